// Morton order of the charges: 24-bit Morton keys (12 bits per axis over
// [-1, 1]^2), ordered by (key, index).  That order is unique, so both ways to
// it below give the same permutation, and both are deterministic: every
// count is exact and every position is a rank.
//
// Up to kRankMax charges: one launch that counts, for each charge, the
// charges before it.  Above: a stable least-significant-digit radix sort, 3
// passes of 8 bits, two launches each -- per-tile digit counts (the first
// pass also computes the keys), and a stable scatter whose workgroups sum
// the counts they need themselves (beyond kInlineTiles tiles a launch in
// between does).
#include "common.hpp"

namespace cd {

constexpr int kSortThreads = 1024;
constexpr int kSortRounds = 2;
constexpr int kSortTile = kSortThreads * kSortRounds;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortRows = kSortWaves * kSortRounds;  // waves of a tile, in index order
// The scatter of one of T tiles reads the T x 256 count table (1 KiB rows,
// from L2); past this many the table is scanned once, by a launch of its own
// (at 128 tiles, 262 144 charges, 34.9 us without that launch and 47 with it;
// the reads grow with the square of the tiles).
constexpr int kInlineTiles = 128;
constexpr int kRankThreads = 1024;
// The counting grows with n^2, the radix sort's launches do not: 19.8 us
// against 24 at n = 10 000, 22.6 at 12 000, 25.6 at 14 000 (the radix sort of
// nine launches took 36).
constexpr int kRankMax = 12288;

int sort_tiles(int n) { return (n + kSortTile - 1) / kSortTile; }

// Elements of 32-bit scratch the sort needs besides the key/value buffers.
size_t sort_scratch_elems(int n) { return (size_t)256 * sort_tiles(n) + 256; }

__device__ __forceinline__ uint32_t spread12(uint32_t v) {
  v &= 0xfffu;
  v = (v | (v << 8)) & 0x00ff00ffu;
  v = (v | (v << 4)) & 0x0f0f0f0fu;
  v = (v | (v << 2)) & 0x33333333u;
  v = (v | (v << 1)) & 0x55555555u;
  return v;
}

__device__ __forceinline__ uint32_t morton_key(double x, double y) {
  double fx = (x + 1.0) * 2048.0, fy = (y + 1.0) * 2048.0;
  if (!(fx >= 0.0)) fx = 0.0;  // also maps NaN to 0
  if (!(fx <= 4095.0)) fx = 4095.0;
  if (!(fy >= 0.0)) fy = 0.0;
  if (!(fy <= 4095.0)) fy = 4095.0;
  return spread12((uint32_t)fx) | (spread12((uint32_t)fy) << 1);
}

// The position of each charge in the order, counted directly: position of i =
// number of j with key_j < key_i, or key_j = key_i and j < i.  A workgroup
// takes 64 charges (one per lane); it computes all n keys into LDS and its 16
// waves count over a sixteenth of them each, four keys per broadcast read.
// Bound: launch latency up to about 2000 charges (5.9 us at 1000, the nine
// launches of the radix sort before took 27), above it the two instructions
// per comparison and the n keys that each workgroup computes (10.7 us at
// 4097, 19.8 at 10 000, 34 and 36 before).
__global__ __launch_bounds__(kRankThreads) void k_rank(const double* __restrict__ x,
                                                       const double* __restrict__ y, int n,
                                                       int32_t* __restrict__ perm) {
  extern __shared__ __align__(16) uint32_t key[];  // n rounded up to 4 * 16 keys, then the waves' counts
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  constexpr int NW = kRankThreads / 64;
  const int per = (n + 4 * NW - 1) / (4 * NW) * 4;  // keys per wave, a multiple of 4
  uint32_t* cnt = key + per * NW;
  for (int j = t; j < per * NW; j += kRankThreads)
    key[j] = j < n ? morton_key(x[j], y[j]) : 0xffffffffu;  // keys have 24 bits: never counted
  __syncthreads();
  const int i0 = blockIdx.x * 64, i = i0 + lane;
  const uint32_t k = i < n ? key[i] : 0u;
  uint32_t c = 0;
  // j before the block counts at key_j <= k, j after it at key_j < k
  auto count = [&](int a, int b, uint32_t lim) {  // a, b: multiples of 4
#pragma unroll 4
    for (int j = a; j < b; j += 4) {
      const uint4 q = *reinterpret_cast<const uint4*>(key + j);
      c += q.x < lim;
      c += q.y < lim;
      c += q.z < lim;
      c += q.w < lim;
    }
  };
  const int j0 = w * per, j1 = j0 + per;
  count(j0, min(j1, i0), k + 1);
  count(max(j0, i0 + 64), j1, k);
  for (int j = max(j0, i0); j < min(j1, i0 + 64); ++j) c += key[j] < k || (key[j] == k && j < i);
  cnt[t] = c;
  __syncthreads();
  if (t < 64 && i < n) {
    uint32_t r = 0;
    for (int q = 0; q < NW; ++q) r += cnt[q * 64 + lane];
    perm[r] = i;
  }
}

// Digit counts of one tile, hist[tile][digit].  MORTON: the keys are computed
// from (x, y) and written with the identity values first.
template <bool MORTON>
__global__ __launch_bounds__(kSortThreads) void k_sort_hist(const double* __restrict__ x,
                                                            const double* __restrict__ y,
                                                            uint32_t* __restrict__ keys,
                                                            int32_t* __restrict__ vals, int n,
                                                            int shift,
                                                            uint32_t* __restrict__ hist) {
  __shared__ uint32_t cnt[256];
  if (threadIdx.x < 256) cnt[threadIdx.x] = 0;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    const int i = blockIdx.x * kSortTile + r * kSortThreads + threadIdx.x;
    if (i < n) {
      uint32_t k;
      if (MORTON) {
        k = morton_key(x[i], y[i]);
        keys[i] = k;
        vals[i] = i;
      } else {
        k = keys[i];
      }
      atomicAdd(&cnt[(k >> shift) & 255u], 1u);
    }
  }
  __syncthreads();
  if (threadIdx.x < 256) hist[blockIdx.x * 256 + threadIdx.x] = cnt[threadIdx.x];
}

// Where a tile's items of each digit go: the items of smaller digits in all
// tiles, then those of the digit in earlier tiles.  Thread t takes digit t mod
// 256 and a quarter of the tiles.  sum[q][d]: quarter q's count of digit d,
// before[q][d]: its part in tiles below `me`.
struct ColSums {
  uint32_t sum[4][256], before[4][256], wsum[4];
};
__device__ __forceinline__ void col_sums(const uint32_t* __restrict__ hist, int ntiles, int me,
                                         ColSums& s) {
  const int d = threadIdx.x & 255, q = threadIdx.x >> 8;
  const int per = (ntiles + 3) / 4, k0 = min(ntiles, q * per), k1 = min(ntiles, k0 + per);
  uint32_t a = 0, b = 0;
#pragma unroll 8
  for (int k = k0; k < k1; ++k) {
    const uint32_t c = hist[(size_t)k * 256 + d];
    a += c;
    b += k < me ? c : 0u;
  }
  s.sum[q][d] = a;
  s.before[q][d] = b;
  __syncthreads();
}
// Exclusive prefix over the digits of all tiles' counts (threads 0..255; every
// thread takes part in the barrier).
__device__ __forceinline__ uint32_t digit_base(ColSums& s) {
  const int t = threadIdx.x, lane = t & 63;
  uint32_t tot = 0, v = 0;
  if (t < 256) {
    tot = s.sum[0][t] + s.sum[1][t] + s.sum[2][t] + s.sum[3][t];
    v = tot;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t u = __shfl_up(v, off, 64);
      if (lane >= off) v += u;
    }
    if (lane == 63) s.wsum[t >> 6] = v;
  }
  __syncthreads();
  if (t < 256)
    for (int q = 0; q < (t >> 6); ++q) v += s.wsum[q];
  return v - tot;
}

// The count table turned into positions in place, one workgroup: thread
// (digit, quarter of the tiles).
__global__ __launch_bounds__(kSortThreads) void k_sort_cols(uint32_t* __restrict__ hist,
                                                            int ntiles) {
  __shared__ ColSums s;
  __shared__ uint32_t base[256];
  col_sums(hist, ntiles, 0, s);
  const uint32_t b = digit_base(s);
  if (threadIdx.x < 256) base[threadIdx.x] = b;
  __syncthreads();
  const int d = threadIdx.x & 255, q = threadIdx.x >> 8;
  const int per = (ntiles + 3) / 4, k0 = min(ntiles, q * per), k1 = min(ntiles, k0 + per);
  uint32_t pos = base[d];
  for (int p = 0; p < q; ++p) pos += s.sum[p][d];
#pragma unroll 8
  for (int k = k0; k < k1; ++k) {
    const uint32_t c = hist[(size_t)k * 256 + d];
    hist[(size_t)k * 256 + d] = pos;
    pos += c;
  }
}

// Bound of the radix sort: launch latency, six launches of 4 to 5 us (30.5 us
// at 1e5 charges; with the scans in launches of their own and 256-thread
// workgroups that ranked a tile in eight rounds, 50.3).
//
// Stable scatter of one tile.  INLINE: hist holds the counts and the
// workgroup sums its positions from them; otherwise hist holds positions.
template <bool INLINE>
__global__ __launch_bounds__(kSortThreads) void k_sort_scatter(
    const uint32_t* __restrict__ kin, const int32_t* __restrict__ vin, int n, int shift,
    int ntiles, const uint32_t* __restrict__ hist, uint32_t* __restrict__ kout,
    int32_t* __restrict__ vout) {
  __shared__ ColSums s;
  __shared__ uint32_t wcnt[kSortRows][256];  // per wave and digit: count, then position
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  uint32_t key[kSortRounds];
  int32_t val[kSortRounds];
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    const int i = blockIdx.x * kSortTile + r * kSortThreads + t;
    key[r] = i < n ? kin[i] : 0u;
    val[r] = i < n ? vin[i] : 0;
  }
  for (int e = t; e < kSortRows * 256; e += kSortThreads) (&wcnt[0][0])[e] = 0;
  uint32_t base = 0;
  if (INLINE) {
    col_sums(hist, ntiles, blockIdx.x, s);  // its barrier also follows the clearing of wcnt
    base = digit_base(s);
    if (t < 256) base += s.before[0][t] + s.before[1][t] + s.before[2][t] + s.before[3][t];
  } else {
    if (t < 256) base = hist[(size_t)blockIdx.x * 256 + t];
    __syncthreads();
  }
  uint32_t lower[kSortRounds];
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    const bool ok = blockIdx.x * kSortTile + r * kSortThreads + t < n;
    const uint32_t d = (key[r] >> shift) & 255u;
    uint64_t m = __ballot(ok);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const uint64_t bb = __ballot((d >> bit) & 1u);
      m &= ((d >> bit) & 1u) ? bb : ~bb;
    }
    lower[r] = __popcll(m & lt);
    if (ok && lower[r] == 0) wcnt[r * kSortWaves + w][d] = __popcll(m);
  }
  __syncthreads();
  if (t < 256) {
    uint32_t c[kSortRows];
#pragma unroll
    for (int q = 0; q < kSortRows; ++q) c[q] = wcnt[q][t];
#pragma unroll
    for (int q = 0; q < kSortRows; ++q) {
      wcnt[q][t] = base;
      base += c[q];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    if (blockIdx.x * kSortTile + r * kSortThreads + t >= n) continue;
    const uint32_t pos = wcnt[r * kSortWaves + w][(key[r] >> shift) & 255u] + lower[r];
    kout[pos] = key[r];
    vout[pos] = val[r];
  }
}

// Stable Morton order of (x, y): perm[s] = index of the s-th charge.  ka, kb
// and va are scratch of n elements, hist has sort_scratch_elems(n); perm
// (n elements) also serves as scratch in the first two passes.
int morton_order(const double* x, const double* y, int n, uint32_t* ka, uint32_t* kb,
                 int32_t* va, uint32_t* hist, int32_t* perm, hipStream_t st) {
  if (n <= kRankMax) {
    constexpr int NW = kRankThreads / 64;
    const size_t lds = sizeof(uint32_t) * ((size_t)(n + 4 * NW - 1) / (4 * NW) * 4 * NW + kRankThreads);
    hipLaunchKernelGGL(k_rank, dim3((n + 63) / 64), dim3(kRankThreads), lds, st, x, y, n, perm);
    return hip_status(hipGetLastError());
  }
  const int nt = sort_tiles(n);
  // passes: (ka, va) -> (kb, perm) -> (ka, va) -> (kb, perm)
  uint32_t* kin[3] = {ka, kb, ka};
  int32_t* vin[3] = {va, perm, va};
  uint32_t* kout[3] = {kb, ka, kb};
  int32_t* vout[3] = {perm, va, perm};
  const dim3 g(nt), b(kSortThreads);
  for (int p = 0; p < 3; ++p) {
    if (p == 0)
      hipLaunchKernelGGL(k_sort_hist<true>, g, b, 0, st, x, y, ka, va, n, 0, hist);
    else
      hipLaunchKernelGGL(k_sort_hist<false>, g, b, 0, st, nullptr, nullptr, kin[p], nullptr, n,
                         8 * p, hist);
    if (nt <= kInlineTiles) {
      hipLaunchKernelGGL(k_sort_scatter<true>, g, b, 0, st, kin[p], vin[p], n, 8 * p, nt, hist,
                         kout[p], vout[p]);
    } else {
      hipLaunchKernelGGL(k_sort_cols, dim3(1), b, 0, st, hist, nt);
      hipLaunchKernelGGL(k_sort_scatter<false>, g, b, 0, st, kin[p], vin[p], n, 8 * p, nt, hist,
                         kout[p], vout[p]);
    }
  }
  return hip_status(hipGetLastError());
}

}  // namespace cd
