// Defect-targeted zones of the subdomain cycle (paper Sec. II.C, steps 2-4
// and the oscillating zone radius).
//
//  - k_defect_stats: one workgroup.  Mean and population standard deviation
//    of the local energies (fixed-order FP64 sums) and the threshold
//    mu + kappa*sigma_e; k_defect_count, k_defect_list (up to kDefSmall
//    charges the same workgroup): the list of charges above it in increasing
//    index order.
//  - k_zone_pick: one thread per zone.  Centre (a defect charge or the
//    caller's disk point, by the caller's uniform draws) and the radius of
//    the triangle wave.
//  - k_zone_count / k_zone_fill: one to kZoneS workgroups per zone, each wave a
//    contiguous range of the charges.  Every charge within the radius,
//    counted, then listed in increasing index order.
//  - zone_batches: host code.  Greedy assignment of the zones to batches of
//    mutually distant zones (in sequence order, or first fit), with a
//    uniform grid over the centres.
//
// The comparisons that decide membership are taken on separately rounded
// FP64 operations (no contraction), so the lists are reproducible exactly.
#include <algorithm>
#include <cmath>
#include <vector>

#include "common.hpp"

namespace cd {

constexpr int kZT = 1024;  // threads of the one-workgroup kernels
constexpr int kZW = kZT / 64;
constexpr int kDefE = 4 * kZT;  // charges per workgroup of the defect list
// Up to this many charges the one-workgroup kernel writes the list itself: the
// two launches of the spread list cost 4 us (call with 50 zones, us, list in the
// kernel against spread: 1000 charges 33.3 / 38.8, 5000 35.9 / 39.0, 12 000
// 39.8 / 41.3, 16 000 41.6 / 41.5, 24 000 46.6 / 43.7).
constexpr int kDefSmall = 16384;
constexpr int kZoneS = 4;       // workgroups per zone, at most
constexpr int kZoneWaves = kZoneS * kZW;

size_t zones_workspace_bytes(int op, int64_t n, int32_t n_zones) {
  Carve c;
  if (op == CD_OP_DEFECT) {
    c.take<int32_t>((size_t)n);
    c.take<double>(4);
    c.take<int32_t>((size_t)n / kDefE + 1);
  } else {
    c.take<int32_t>((size_t)n_zones * kZoneS);
    c.take<int32_t>((size_t)n_zones * kZoneWaves);
    c.take<int32_t>((size_t)n_zones + 1);
  }
  return c.off + 256;
}

// Sum of one double per thread over a 1024-thread workgroup in a fixed
// order: butterfly inside each wave, then the 16 wave sums in order.
__device__ double block_sum_fixed(double v, double* red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  double s = 0.0;
  for (int q = 0; q < kZW; ++q) s += red[q];
  __syncthreads();
  return s;
}

// Sum of one int per thread over the workgroup, and (scan) the sum of the
// threads before this one.
__device__ int block_sum_int(int v, int* ws, int* before = nullptr) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int s = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(s, off, 64);
    if (lane >= off) s += u;
  }
  if (lane == 63) ws[w] = s;
  __syncthreads();
  int total = 0, b = s - v;
  for (int q = 0; q < kZW; ++q) {
    b += q < w ? ws[q] : 0;
    total += ws[q];
  }
  __syncthreads();
  if (before) *before = b;
  return total;
}

#pragma clang fp contract(off)

// Sum over the thread's charges t, t + kZT, ... in order; up to 16 loads go out
// together (one at a time the two sums and the list took 104 us at n = 1e5), and
// two where fewer are left.
template <int U, class F>
__device__ __forceinline__ void strided_group(const double* __restrict__ e, int n, int b, F f,
                                              double& s) {
  double v[U];
#pragma unroll
  for (int q = 0; q < U; ++q) v[q] = e[min(b + q * kZT + (int)threadIdx.x, n - 1)];
#pragma unroll
  for (int q = 0; q < U; ++q)
    if (b + q * kZT + (int)threadIdx.x < n) s += f(v[q]);
}
template <class F>
__device__ __forceinline__ double strided_sum(const double* __restrict__ e, int n, F f) {
  double s = 0.0;
  int b = 0;
  for (; n - b > 8 * kZT; b += 16 * kZT) strided_group<16>(e, n, b, f, s);
  for (; n - b > 2 * kZT; b += 8 * kZT) strided_group<8>(e, n, b, f, s);
  for (; b < n; b += 2 * kZT) strided_group<2>(e, n, b, f, s);
  return s;
}

// Defects of the thread's four consecutive charges of block `b`, as bits.
__device__ __forceinline__ int defect_bits(const double* __restrict__ e, int n, double thr, int b) {
  const int j0 = b * kDefE + 4 * threadIdx.x;
  int m = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) m |= (j0 + q < n && e[min(j0 + q, n - 1)] > thr) << q;
  return m;
}
__device__ __forceinline__ void defect_write(int m, int b, int pos, int32_t* __restrict__ list) {
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if ((m >> q) & 1) list[pos++] = b * kDefE + 4 * threadIdx.x + q;
}

// LIST: the list too (n up to kDefSmall).
template <bool LIST>
__global__ __launch_bounds__(kZT) void k_defect_stats(const double* __restrict__ e, int n,
                                                      double kappa, double* __restrict__ stats,
                                                      int32_t* __restrict__ list) {
  __shared__ double red[kZW];
  __shared__ int ws[kZW];
  const double s = strided_sum(e, n, [](double v) { return v; });
  const double mu = block_sum_fixed(s, red) / (double)n;
  const double q = strided_sum(e, n, [mu](double v) {
    const double d = v - mu;
    return d * d;
  });
  const double var = block_sum_fixed(q, red) / (double)n;
  const double sigma = __dsqrt_rn(var);
  const double ks = kappa * sigma;
  const double thr = mu + ks;
  int base = 0;
  if (LIST)
    for (int b = 0; b * kDefE < n; ++b) {
      const int m = defect_bits(e, n, thr, b);
      int before;
      const int total = block_sum_int(__popc(m), ws, &before);
      defect_write(m, b, base + before, list);
      base += total;
    }
  if (threadIdx.x == 0) {
    stats[0] = mu;
    stats[1] = sigma;
    stats[2] = thr;
    if (LIST) stats[3] = (double)base;
  }
}

__global__ __launch_bounds__(kZT) void k_defect_count(const double* __restrict__ e, int n,
                                                      const double* __restrict__ stats,
                                                      int32_t* __restrict__ sums) {
  __shared__ int ws[kZW];
  const int t = block_sum_int(__popc(defect_bits(e, n, stats[2], blockIdx.x)), ws);
  if (threadIdx.x == 0) sums[blockIdx.x] = t;
}
__global__ __launch_bounds__(kZT) void k_defect_list(const double* __restrict__ e, int n,
                                                     double* __restrict__ stats,
                                                     const int32_t* __restrict__ sums,
                                                     int32_t* __restrict__ list) {
  __shared__ int ws[kZW];
  int base = 0, before;
  for (int q = threadIdx.x; q < (int)blockIdx.x; q += kZT) base += sums[q];
  base = block_sum_int(base, ws);
  const int m = defect_bits(e, n, stats[2], blockIdx.x);
  const int total = block_sum_int(__popc(m), ws, &before);
  defect_write(m, blockIdx.x, base + before, list);
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) stats[3] = (double)(base + total);
}

__global__ void k_zone_pick(const double* __restrict__ x, const double* __restrict__ y,
                            const double* __restrict__ stats, const int32_t* __restrict__ list,
                            const double* __restrict__ draws, int P, cd_zone_opts o,
                            double* __restrict__ cx, double* __restrict__ cy,
                            double* __restrict__ rz, int32_t* __restrict__ ci) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= P) return;
  const double u = draws[4 * (size_t)t], v = draws[4 * (size_t)t + 1];
  const int64_t nd = (int64_t)stats[3];
  if (u < o.p_defect && nd > 0) {
    const double f = floor(v * (double)nd);
    int64_t k = f < 0.0 ? 0 : (int64_t)f;
    if (k > nd - 1) k = nd - 1;
    const int i = list[k];
    cx[t] = x[i];
    cy[t] = y[i];
    ci[t] = i;
  } else {
    cx[t] = draws[4 * (size_t)t + 2];
    cy[t] = draws[4 * (size_t)t + 3];
    ci[t] = -1;
  }
  const int64_t s = (o.t0 + t) % o.period;
  const int64_t m = s < o.period - s ? s : o.period - s;
  const double tri = (double)(2 * m) / (double)o.period;
  const double span = o.r_hi - o.r_lo;
  const double step = span * tri;
  rz[t] = o.r_lo + step;
}

__device__ __forceinline__ bool in_zone(double xj, double yj, double c0, double c1, double r2) {
  const double dx = xj - c0, dy = yj - c1;
  const double a = dx * dx, b = dy * dy;
  const double d2 = a + b;
  return d2 <= r2;
}

// The calling wave's range of the charges, in blocks of 64: f(index, in the
// zone).  Eight blocks' loads go out together, two where fewer are left.
template <int U, class F>
__device__ __forceinline__ void zone_group(const double* __restrict__ x,
                                           const double* __restrict__ y, double c0, double c1,
                                           double r2, int b, int j1, F f) {
  const int lane = threadIdx.x & 63;
  double vx[U], vy[U];
#pragma unroll
  for (int q = 0; q < U; ++q) {
    const int j = min(b + q * 64 + lane, j1 - 1);
    vx[q] = x[j];
    vy[q] = y[j];
  }
#pragma unroll
  for (int q = 0; q < U; ++q) {
    const int j = b + q * 64 + lane;
    if (b + q * 64 < j1) f(j, j < j1 && in_zone(vx[q], vy[q], c0, c1, r2));
  }
}
template <class F>
__device__ __forceinline__ void zone_sweep(const double* __restrict__ x,
                                           const double* __restrict__ y, int n, double c0,
                                           double c1, double r2, int g, F f) {
  const int waves = gridDim.y * kZW;
  const int per = (n + 64 * waves - 1) / (64 * waves) * 64;
  const int j0 = min(n, g * per), j1 = min(n, j0 + per);
  int b = j0;
  for (; j1 - b > 256; b += 512) zone_group<8>(x, y, c0, c1, r2, b, j1, f);
  for (; b < j1; b += 128) zone_group<2>(x, y, c0, c1, r2, b, j1, f);
}

// Counts per wave (wcnt [zones][kZoneWaves]) and per workgroup (cnt
// [zones][workgroups per zone]).  67 zones at n = 1e5: count and list 16 us each, 33 and 72 by
// one workgroup per zone with two barriers per 1024 charges of the list.
__global__ __launch_bounds__(kZT) void k_zone_count(const double* __restrict__ x,
                                                    const double* __restrict__ y, int n,
                                                    const double* __restrict__ cx,
                                                    const double* __restrict__ cy,
                                                    const double* __restrict__ rz,
                                                    int32_t* __restrict__ cnt,
                                                    int32_t* __restrict__ wcnt) {
  __shared__ int ws[kZW];
  const int p = blockIdx.x, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = blockIdx.y * kZW + w;
  const double r = rz[p], r2 = r * r;
  int c = 0;
  zone_sweep(x, y, n, cx[p], cy[p], r2, g, [&](int, bool in) { c += __popcll(__ballot(in)); });
  if ((threadIdx.x & 63) == 0) {
    ws[w] = c;
    wcnt[(size_t)p * kZoneWaves + g] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int s = 0;
    for (int q = 0; q < kZW; ++q) s += ws[q];
    cnt[p * gridDim.y + blockIdx.y] = s;
  }
}

__global__ __launch_bounds__(kZT) void k_zone_fill(const double* __restrict__ x,
                                                   const double* __restrict__ y, int n,
                                                   const double* __restrict__ cx,
                                                   const double* __restrict__ cy,
                                                   const double* __restrict__ rz,
                                                   const int32_t* __restrict__ ptr,
                                                   const int32_t* __restrict__ wcnt,
                                                   int32_t* __restrict__ out) {
  const int p = blockIdx.x, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, g = blockIdx.y * kZW + w;
  const double r = rz[p], r2 = r * r;
  int before = lane < g ? wcnt[(size_t)p * kZoneWaves + lane] : 0;
  for (int m = 32; m >= 1; m >>= 1) before += __shfl_xor(before, m, 64);
  const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  int32_t* const dst = out + ptr[p];
  const int cap = ptr[p + 1] - ptr[p];
  zone_sweep(x, y, n, cx[p], cy[p], r2, g, [&](int j, bool in) {
    const uint64_t m = __ballot(in);
    const int pos = before + __popcll(m & lt);
    if (in && pos < cap) dst[pos] = j;
    before += __popcll(m);
  });
}
static_assert(kZoneWaves <= 64, "k_zone_fill sums the waves before its own across a wave");
// Workgroups per zone: more where few zones leave the chip idle.  zone_patches,
// us, with one / two / four: 5000 charges and 128 zones 57.5 / 56.3 / 56.8, 256
// 58.2 / 57.7 / 59.5, 1000 68.8 / 70.0 / 76.8; 24 000 and 128 67.4 / 61.4 / 62.6, 256
// 68.0 / 67.5 / 70.9, 512 79.0 / 78.9 / 85.7; 1e5 and 64 103 / 80 / 69, 128 105 / 81 / 81,
// 256 106 / 102 / 102, 1000 232 / 232 / 234.
static int zone_split(int n_zones) { return n_zones <= 128 ? 4 : n_zones <= 256 ? 2 : 1; }

#pragma clang fp contract(on)

}  // namespace cd

using namespace cd;

namespace {

#pragma clang fp contract(off)
// Placed zones, in ranges by cell of the scheduler's grid, each range in
// sequence order.
struct Placed {
  std::vector<double> x, y, r;
  std::vector<uint64_t> bit;  // 1 << (batch mod 64)
  std::vector<int32_t> b;     // batch
  explicit Placed(size_t n) : x(n), y(n), r(n), bit(n), b(n) {}
};
// The OR of bit[q] over the zones q of [q0, q1) that conflict with (x, y, r).
// No branch on a test's outcome, so that the loop vectorises (about one zone in
// five conflicts, in no order: the mispredicted branch costs more than the
// test).  1000 zones with the radii of a cycle at N = 1e5: 0.87 ms with the
// branch, now 0.33 (0.40 in sequence order).
uint64_t conflict_bits(const Placed& p, size_t q0, size_t q1, const uint64_t* bit, double x,
                       double y, double r, double gap) {
  const double *px = p.x.data() + q0, *py = p.y.data() + q0, *pr = p.r.data() + q0;
  const size_t n = q1 - q0;
  uint64_t m = 0;
  for (size_t q = 0; q < n; ++q) {
    const double dx = px[q] - x, dy = py[q] - y;
    const double reach = pr[q] + r + gap;
    const double a = dx * dx, b = dy * dy;
    const double d2 = a + b;
    const double r2 = reach * reach;
    m |= bit[q] & -(uint64_t)(d2 < r2);
  }
  return m;
}
#pragma clang fp contract(on)

// 1 << 0 .. 1 << 63
struct LaneBits {
  uint64_t v[64];
  constexpr LaneBits() : v() {
    for (int q = 0; q < 64; ++q) v[q] = 1ull << q;
  }
};
constexpr LaneBits kLaneBits;
// cells of the scheduler's grid, at most, per zone
constexpr int64_t kCellsPerZone = 4;

}  // namespace

extern "C" {

double zone_radius_holding(int64_t n, int64_t count) {
  if (n < 1 || count < 0) return 0.0;
  return sqrt((double)count / (double)n);
}

int defect_zones(const double* x, const double* y, const double* e, int64_t n, int32_t n_zones,
                 const double* draws, const cd_zone_opts* opts, double* cx, double* cy,
                 double* rz, int32_t* centre_idx, double* stats, int32_t* defect_idx, void* ws,
                 size_t ws_bytes, void* stream) {
  if (!x || !y || !e || !opts || n < 1 || n > (1 << 26) || n_zones < 0 ||
      (n_zones > 0 && (!draws || !cx || !cy || !rz || !centre_idx)) || opts->period < 1 ||
      opts->t0 < 0 || !(opts->r_lo >= 0.0) || !(opts->r_hi >= opts->r_lo) ||
      !std::isfinite(opts->r_hi) || !std::isfinite(opts->kappa))
    return CD_ERR_INVALID_ARG;
  if (!ws || ws_bytes < zones_workspace_bytes(CD_OP_DEFECT, n, 0)) return CD_ERR_WORKSPACE;
  Carve c;
  c.base = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255));
  int32_t* list = c.take<int32_t>((size_t)n);
  double* st_d = c.take<double>(4);
  int32_t* sums = c.take<int32_t>((size_t)n / kDefE + 1);
  if (defect_idx) list = defect_idx;
  if (stats) st_d = stats;
  hipStream_t st = (hipStream_t)stream;
  const int nw = ((int)n + kDefE - 1) / kDefE;
  if (n <= kDefSmall) {
    hipLaunchKernelGGL(k_defect_stats<true>, dim3(1), dim3(kZT), 0, st, e, (int)n, opts->kappa,
                       st_d, list);
  } else {
    hipLaunchKernelGGL(k_defect_stats<false>, dim3(1), dim3(kZT), 0, st, e, (int)n, opts->kappa,
                       st_d, list);
    hipLaunchKernelGGL(k_defect_count, dim3(nw), dim3(kZT), 0, st, e, (int)n, st_d, sums);
    hipLaunchKernelGGL(k_defect_list, dim3(nw), dim3(kZT), 0, st, e, (int)n, st_d, sums, list);
  }
  if (n_zones > 0)
    hipLaunchKernelGGL(k_zone_pick, dim3((n_zones + 255) / 256), dim3(256), 0, st, x, y, st_d,
                       list, draws, n_zones, *opts, cx, cy, rz, centre_idx);
  return hip_status(hipGetLastError());
}

int zone_patches(const double* x, const double* y, int64_t n, int32_t n_zones, const double* cx,
                 const double* cy, const double* rz, int32_t* patch_ptr, int32_t* active_idx,
                 int64_t capacity, void* ws, size_t ws_bytes, void* stream) {
  if (!x || !y || !cx || !cy || !rz || !patch_ptr || n < 1 || n > (1 << 26) || n_zones < 1 ||
      capacity < 0 || (capacity > 0 && !active_idx))
    return CD_ERR_INVALID_ARG;
  if (!ws || ws_bytes < zones_workspace_bytes(CD_OP_ZONES, n, n_zones)) return CD_ERR_WORKSPACE;
  Carve c;
  c.base = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255));
  int32_t* cnt_d = c.take<int32_t>((size_t)n_zones * kZoneS);
  int32_t* wcnt = c.take<int32_t>((size_t)n_zones * kZoneWaves);
  int32_t* ptr_d = c.take<int32_t>((size_t)n_zones + 1);
  hipStream_t st = (hipStream_t)stream;
  const int S = zone_split(n_zones);
  hipLaunchKernelGGL(k_zone_count, dim3(n_zones, S), dim3(kZT), 0, st, x, y, (int)n, cx, cy,
                     rz, cnt_d, wcnt);
  int rc = hip_status(hipGetLastError());
  if (rc) return rc;
  std::vector<int32_t> cnt((size_t)n_zones * S);
  if ((rc = hip_status(hipMemcpyAsync(cnt.data(), cnt_d, sizeof(int32_t) * cnt.size(),
                                      hipMemcpyDeviceToHost, st))))
    return rc;
  if ((rc = hip_status(hipStreamSynchronize(st)))) return rc;
  int64_t total = 0;
  patch_ptr[0] = 0;
  for (int p = 0; p < n_zones; ++p) {
    for (int q = 0; q < S; ++q) total += cnt[(size_t)p * S + q];
    if (total > INT32_MAX) return CD_ERR_INVALID_ARG;
    patch_ptr[p + 1] = (int32_t)total;
  }
  if (total > capacity) return CD_ERR_CAPACITY;
  if (total == 0) return CD_OK;
  if ((rc = hip_status(hipMemcpyAsync(ptr_d, patch_ptr, sizeof(int32_t) * (n_zones + 1),
                                      hipMemcpyHostToDevice, st))))
    return rc;
  hipLaunchKernelGGL(k_zone_fill, dim3(n_zones, S), dim3(kZT), 0, st, x, y, (int)n, cx, cy,
                     rz, ptr_d, wcnt, active_idx);
  if ((rc = hip_status(hipGetLastError()))) return rc;
  // the host offsets were read by the copy above; keep them valid until it ends
  return hip_status(hipStreamSynchronize(st));
}

int zone_batches(const double* cx, const double* cy, const double* rz, int32_t n_zones,
                 double gap, int32_t cap, int32_t keep_order, int32_t* batch,
                 int32_t* n_batches) {
  if (n_zones < 0 || cap < 1 || !(gap >= 0.0) || !std::isfinite(gap) ||
      (n_zones > 0 && (!cx || !cy || !rz || !batch)))
    return CD_ERR_INVALID_ARG;
  if (n_zones == 0) {
    if (n_batches) *n_batches = 0;
    return CD_OK;
  }
  double rmax = 0.0, x0 = 0.0, x1 = 0.0, y0 = 0.0, y1 = 0.0;
  for (int t = 0; t < n_zones; ++t) {
    if (!std::isfinite(cx[t]) || !std::isfinite(cy[t]) || !(rz[t] >= 0.0) ||
        !std::isfinite(rz[t]))
      return CD_ERR_INVALID_ARG;
    rmax = std::max(rmax, rz[t]);
    x0 = t ? std::min(x0, cx[t]) : cx[t];
    x1 = t ? std::max(x1, cx[t]) : cx[t];
    y0 = t ? std::min(y0, cy[t]) : cy[t];
    y1 = t ? std::max(y1, cy[t]) : cy[t];
  }
  // Conflicting centres are closer than 2 rmax + gap: with cells at least
  // that wide only the 3 x 3 neighbourhood of a cell can hold a conflict
  // (1e-6 of slack keeps rounding in the cell index from splitting a
  // conflicting pair two cells apart).
  const double cell = (2.0 * rmax + gap) * (1.0 + 1e-6);
  int gx = 1, gy = 1;
  if (cell > 0.0) {
    gx = (int)std::max(1.0, std::min(1024.0, std::floor((x1 - x0) / cell)));
    gy = (int)std::max(1.0, std::min(1024.0, std::floor((y1 - y0) / cell)));
  }
  // wider cells find the same conflicts: more cells than a few per zone only
  // cost memory and time to clear (1000 zones of radius 0.001: 4 ms and 24 MB
  // with a vector for each of 1024 x 1024 cells, now 0.2 ms)
  while ((int64_t)gx * gy > kCellsPerZone * (int64_t)n_zones) {
    if (gx >= gy) gx = (gx + 1) / 2;
    else gy = (gy + 1) / 2;
  }
  const double wx = gx > 1 ? (x1 - x0) / gx : 1.0;
  const double wy = gy > 1 ? (y1 - y0) / gy : 1.0;
  auto cell_of = [&](double v, double lo, double w, int g) {
    if (g == 1) return 0;
    return std::min(g - 1, std::max(0, (int)((v - lo) / w)));
  };
  // the zones by cell: every cell's range of the flat arrays, filled as its
  // zones are placed
  std::vector<int32_t> cell_id(n_zones), first((size_t)gx * gy + 1), fill((size_t)gx * gy);
  for (int t = 0; t < n_zones; ++t) {
    cell_id[t] = cell_of(cx[t], x0, wx, gx) * gy + cell_of(cy[t], y0, wy, gy);
    ++first[cell_id[t] + 1];
  }
  for (size_t c = 0; c < fill.size(); ++c) {
    first[c + 1] += first[c];
    fill[c] = first[c];
  }
  Placed placed(n_zones);
  std::vector<int32_t> size;
  std::vector<int32_t> mark;  // mark[b] == t + 1: batch b holds a zone in conflict with t
  uint64_t full = 0;          // batches below 64 without room
  int32_t nb = 0;
  for (int t = 0; t < n_zones; ++t) {
    const int ix = cell_id[t] / gy, iy = cell_id[t] % gy;
    const double tx = cx[t], ty = cy[t], tr = rz[t];
    uint64_t hit = 0;  // up to 64 batches: those with a conflicting zone
    int32_t need = 0;  // one past the last batch with one
    for (int a = std::max(0, ix - 1); a <= std::min(gx - 1, ix + 1); ++a)
      for (int b = std::max(0, iy - 1); b <= std::min(gy - 1, iy + 1); ++b) {
        const size_t c = (size_t)a * gy + b, q0 = first[c], q1 = fill[c];
        if (nb <= 64) {
          hit |= conflict_bits(placed, q0, q1, placed.bit.data() + q0, tx, ty, tr, gap);
          continue;
        }
        for (size_t q = q0; q < q1; q += 64) {
          uint64_t m = conflict_bits(placed, q, std::min(q1, q + 64), kLaneBits.v, tx, ty, tr, gap);
          const int32_t* const pb = placed.b.data() + q;
          if (keep_order)
            for (; m; m &= m - 1) need = std::max(need, pb[__builtin_ctzll(m)] + 1);
          else
            for (; m; m &= m - 1) mark[pb[__builtin_ctzll(m)]] = t + 1;
        }
      }
    // ordered: after every conflicting earlier zone; first fit: the first
    // batch without a conflicting zone.  Either way a full batch is passed.
    int32_t b;
    if (nb <= 64) {
      if (keep_order && hit) hit = ~0ull >> __builtin_clzll(hit);  // and all batches before
      const uint64_t room = ~(hit | full);
      b = room ? std::min<int32_t>(nb, __builtin_ctzll(room)) : nb;
    } else {
      b = keep_order ? need : 0;
      while (b < nb && (size[b] >= cap || (!keep_order && mark[b] == t + 1))) ++b;
    }
    if (b == nb) {
      ++nb;
      size.push_back(0);
      mark.push_back(0);
    }
    if (++size[b] >= cap && b < 64) full |= 1ull << b;
    batch[t] = b;
    const size_t q = fill[cell_id[t]]++;
    placed.x[q] = tx;
    placed.y[q] = ty;
    placed.r[q] = tr;
    placed.bit[q] = 1ull << (b & 63);
    placed.b[q] = b;
  }
  if (n_batches) *n_batches = nb;
  return CD_OK;
}

}  // extern "C"
