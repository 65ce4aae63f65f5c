// Lanczos check that a configuration is a strict local minimum on the
// tangent space of the hard wall (Eq. 3): the smallest eigenvalue of the
// tangent-space Hessian must be positive.
//
// Operator.  Charges on the wall whose force points outward (F . r_hat > 0)
// are held: they move only along the circle, and moving along a circle adds
// the curvature term F . r_hat to their tangential second derivative.  With
// P the projection that removes the radial component of held charges (and
// every component of inactive charges), the operator is
//     H_t v = P H P v + w o v,   w_i = F_i . r_hat_i for held i, else 0,
// applied with the FP64 Hessian-vector product of the energy.  Optionally
// the rigid rotation (-y, x) -- an exact zero mode of a full disk -- is
// projected out.
//
// Lanczos with full reorthogonalisation (classical Gram-Schmidt, twice; the
// rotation is one more vector of the basis) on the device; the tridiagonal
// eigenproblem is solved by Sturm counts and the Ritz vector by inverse
// iteration with a shift just below the smallest eigenvalue (so the shifted
// matrix is positive definite and the tridiagonal solve needs no pivoting).
// The residual ||H_t u - theta u|| of the unit Ritz vector is measured with
// one more operator application.
//
// All vectors are kept in the sorted, padded order of the pair pass (x part
// [npad], y part [npad], zeros in the pads), so that the product reads a basis
// vector and writes its result in place, with no gather or scatter.  A step is
// eight launches: the product's two, the projection, two passes of (dot
// products, subtraction) and the normalisation.  Bound: the products (70 us at
// 1e4 charges) and the launches; the dot products read the basis at 4 to 5 us a
// pass (with one workgroup per vector, gathers and 16 launches a step took 287 us, now 111).
#include "plan.hpp"

namespace cd {

struct LzDev {
  int n, npad, k;
  size_t len;        // 2 npad
  const double* x;
  const double* y;
  const int32_t* perm;  // caller's index of a sorted place
  const int32_t* mask;
  double *fx, *fy;   // forces at the configuration (caller's order)
  double *ux, *uy;   // [npad] radial unit vector of held charges
  double* wgt;       // [npad] curvature term of held charges
  int32_t* kind;     // [npad] 0 inactive or pad, 1 free, 2 held
  double* Q;         // [k + 2][len]: the unit rotation, then the basis
  double* w;         // [len]
  double* h;         // [len]
  double* part;      // [k + 1][S] partial dot products
  double* nrm;       // [len / kAxE] partial squared norms of w
  double* a1;        // [1] first pass's part of alpha
  double* alpha;     // [k]
  double* beta;      // [k + 1]
  double* tri;       // [k + 4]: Ritz coefficients, then theta_min, theta_max, k_eff, resid^2
  double* scr;       // [2 k] pivots and multipliers of the tridiagonal solve
};

__device__ __forceinline__ uint64_t mix64(uint64_t z) {  // SplitMix64 finaliser
  z += 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

// held set, curvature weights, rotation vector (row 0 of Q, not yet unit),
// random start vector (w), all in sorted order
__global__ void k_lz_setup(LzDev L, uint64_t seed, int deflate) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= L.npad) return;
  int kind = 0;
  double vx = 0.0, vy = 0.0, ux = 0.0, uy = 0.0, fr = 0.0, px = 0.0, py = 0.0;
  if (s < L.n) {
    const int i = L.perm[s];
    const bool act = L.mask ? L.mask[i] != 0 : true;
    px = L.x[i];
    py = L.y[i];
    const double r = sqrt(px * px + py * py);
    fr = r > 0.0 ? (L.fx[i] * px + L.fy[i] * py) / r : 0.0;
    const bool hd = act && r >= 1.0 - 1e-14 && fr > 0.0;
    kind = hd ? 2 : act ? 1 : 0;
    vx = act ? (double)(mix64(seed ^ (2ull * i)) >> 11) * 0x1.0p-52 - 1.0 : 0.0;
    vy = act ? (double)(mix64(seed ^ (2ull * i + 1)) >> 11) * 0x1.0p-52 - 1.0 : 0.0;
    if (hd) {
      ux = px / r;
      uy = py / r;
      const double vr = vx * ux + vy * uy;
      vx -= vr * ux;
      vy -= vr * uy;
    }
  }
  L.kind[s] = kind;
  L.ux[s] = ux;
  L.uy[s] = uy;
  L.wgt[s] = kind == 2 ? fr : 0.0;
  L.w[s] = vx;
  L.w[L.npad + s] = vy;
  if (deflate) {
    L.Q[s] = kind ? -py : 0.0;
    L.Q[L.npad + s] = kind ? px : 0.0;
  }
}

// out = P h + w o v
__global__ void k_lz_post(LzDev L, const double* __restrict__ v, double* __restrict__ out) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= L.npad) return;
  const int kind = L.kind[s];
  double hx = 0.0, hy = 0.0;
  if (kind) {
    hx = L.h[s];
    hy = L.h[L.npad + s];
  }
  if (kind == 2) {
    const double ux = L.ux[s], uy = L.uy[s], hr = hx * ux + hy * uy, g = L.wgt[s];
    hx = hx - hr * ux + g * v[s];
    hy = hy - hr * uy + g * v[L.npad + s];
  }
  out[s] = hx;
  out[L.npad + s] = hy;
}

// part[j][c] = the products of chunk c of A_j (A_j = A + j len) and b.  One
// workgroup per vector and chunk of kDotE elements, fixed order.
constexpr int kDotT = 512, kDotU = 8, kDotE = 2 * kDotT * kDotU;
__global__ __launch_bounds__(kDotT) void k_lz_dots(const double* __restrict__ A, size_t len,
                                                   const double* __restrict__ b,
                                                   double* __restrict__ part) {
  __shared__ double red[kDotT / 64];
  const double2* a2 = reinterpret_cast<const double2*>(A + (size_t)blockIdx.x * len);
  const double2* b2 = reinterpret_cast<const double2*>(b);
  const size_t e0 = (size_t)blockIdx.y * (kDotE / 2) + threadIdx.x, m = len / 2;
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < kDotU; ++q) {
    const size_t e = e0 + (size_t)q * kDotT;
    if (e < m) {
      const double2 u = a2[e], v = b2[e];
      s += u.x * v.x + u.y * v.y;
    }
  }
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int q = 0; q < kDotT / 64; ++q) t += red[q];
    part[(size_t)blockIdx.x * gridDim.y + blockIdx.y] = t;
  }
}

// w -= sum_j c_j A_j, c_j = the sum of part[j][0..S).  A workgroup takes kAxE
// elements, two per lane; its four waves take a quarter of the vectors each,
// added in LDS in wave order.  last: 0; 1 records c of the last vector (the
// first pass's part of alpha), 2 adds it (alpha[step]).  Writes the partial
// squared norm of its elements.
constexpr int kAxE = 128;
__global__ __launch_bounds__(256) void k_lz_axpys(LzDev L, const double* __restrict__ A, int m,
                                                  int S, int last, int step) {
  extern __shared__ double c[];  // [m]
  __shared__ double2 acc[3][64];
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  for (int j = t; j < m; j += 256) {
    double v = 0.0;
    for (int q = 0; q < S; ++q) v += L.part[(size_t)j * S + q];
    c[j] = v;
  }
  __syncthreads();
  if (blockIdx.x == 0 && t == 0 && last) {
    if (last == 1) *L.a1 = c[m - 1];
    else L.alpha[step] = *L.a1 + c[m - 1];
  }
  const size_t e = (size_t)blockIdx.x * (kAxE / 2) + lane, len2 = L.len / 2;  // len: a multiple of kAxE
  const double2* a2 = reinterpret_cast<const double2*>(A) + e;
  const int per = (m + 3) / 4, j0 = min(m, w * per), j1 = min(m, j0 + per);
  double2 v = make_double2(0.0, 0.0);
#pragma unroll 8
  for (int j = j0; j < j1; ++j) {
    const double2 u = a2[(size_t)j * len2];
    v.x += c[j] * u.x;
    v.y += c[j] * u.y;
  }
  if (w > 0) acc[w - 1][lane] = v;
  __syncthreads();
  if (w > 0) return;
  for (int q = 0; q < 3; ++q) {
    v.x += acc[q][lane].x;
    v.y += acc[q][lane].y;
  }
  double2* w2 = reinterpret_cast<double2*>(L.w) + e;
  double2 r = *w2;
  r.x -= v.x;
  r.y -= v.y;
  *w2 = r;
  const double nn = wave_sum(r.x * r.x + r.y * r.y);
  if (lane == 0) L.nrm[blockIdx.x] = nn;
}

// out = w / ||w|| (0 for w = 0); beta (nullable) gets ||w||
__global__ __launch_bounds__(256) void k_lz_next(LzDev L, double* __restrict__ out,
                                                 double* __restrict__ beta) {
  __shared__ double red[4];
  const int t = threadIdx.x, nb = (int)(L.len / kAxE);
  double v = 0.0;
#pragma unroll 4
  for (int q = t; q < nb; q += 256) v += L.nrm[q];
  v = wave_sum(v);
  if ((t & 63) == 0) red[t >> 6] = v;
  __syncthreads();
  const double b = sqrt((red[0] + red[1]) + (red[2] + red[3]));
  const size_t e = (size_t)blockIdx.x * 256 + t;
  if (e < L.len) out[e] = b > 0.0 ? L.w[e] / b : 0.0;
  if (e == 0 && beta) *beta = b;
}

__device__ int sturm_below(const double* a, const double* b, int k, double x) {
  int cnt = 0;
  double d = 1.0;
  for (int i = 0; i < k; ++i) {
    const double bb = i > 0 ? b[i - 1] * b[i - 1] : 0.0;
    d = a[i] - x - (i > 0 ? bb / d : 0.0);
    if (d == 0.0) d = -1e-300;
    cnt += d < 0.0;
  }
  return cnt;
}

// Extreme eigenvalues and the Ritz coefficients of the smallest, one workgroup
// of two waves: wave 0 finds the smallest, wave 1 the largest, each lane
// counting at one of 64 points that split the interval, which shrinks 65-fold
// a pass (a bisection by one thread took 3.5 ms at k = 100, 200 counts for
// each); then thread 0 solves.
__global__ __launch_bounds__(128) void k_lz_tridiag(LzDev L) {
  __shared__ double ends[2];
  const int k = L.k, t = threadIdx.x, lane = t & 63, top = t >> 6;
  const double* a = L.alpha;
  const double* b = L.beta;
  double amax = 0.0;
  for (int i = lane; i < k; i += 64) amax = fmax(amax, fabs(a[i]) + fabs(b[i]));
  amax = wave_max(amax);
  int kk = k;  // the first beta that is negligible ends the matrix
  for (int i = lane; i < k - 1; i += 64)
    if (!(b[i] > 1e-13 * amax)) kk = min(kk, i + 1);
  for (int q = 32; q >= 1; q >>= 1) kk = min(kk, __shfl_xor(kk, q, 64));
  double lo = 1e300, hi = -1e300;
  for (int i = lane; i < kk; i += 64) {
    const double rad = (i > 0 ? fabs(b[i - 1]) : 0.0) + (i < kk - 1 ? fabs(b[i]) : 0.0);
    lo = fmin(lo, a[i] - rad);
    hi = fmax(hi, a[i] + rad);
  }
  lo = wave_min(lo);
  hi = wave_max(hi);
  const int want = top ? kk : 1;  // eigenvalues below the point sought
  for (int it = 0; it < 64; ++it) {
    const double x = lo + (hi - lo) * ((double)(lane + 1) / 65.0);
    const bool above = sturm_below(a, b, kk, x) >= want;
    const uint64_t m = __ballot(above);
    // the first point with enough eigenvalues below it, and the one before
    const int f = m ? __builtin_ctzll(m) : 64;
    const double nlo = f > 0 ? __shfl(x, f - 1, 64) : lo, nhi = f < 64 ? __shfl(x, f, 64) : hi;
    const bool stuck = nlo == lo && nhi == hi;
    lo = nlo;
    hi = nhi;
    if (stuck || !(hi - lo > 0.0)) break;  // uniform in the wave
  }
  if (lane == 0) ends[top] = 0.5 * (lo + hi);
  __syncthreads();
  if (t != 0) return;
  const double tmin = ends[0], tmax = ends[1];
  const double sig = tmin - 1e-10 * (fabs(tmin) + fabs(tmax));
  double* yv = L.tri;
  double *piv = L.scr, *mul = L.scr + k;
  // T - sig I = L D L^T (positive definite), factored once
  double dprev = 0.0;
  for (int i = 0; i < kk; ++i) {
    yv[i] = 1.0;
    mul[i] = i > 0 ? b[i - 1] / dprev : 0.0;
    dprev = a[i] - sig - (i > 0 ? b[i - 1] * mul[i] : 0.0);
    piv[i] = dprev;
  }
  for (int pass = 0; pass < 4; ++pass) {
    double p = yv[0];
    for (int i = 1; i < kk; ++i) yv[i] = p = yv[i] - mul[i] * p;
    yv[kk - 1] = p = yv[kk - 1] / piv[kk - 1];
    for (int i = kk - 2; i >= 0; --i) yv[i] = p = yv[i] / piv[i] - mul[i + 1] * p;
    double q = 0.0;
    for (int i = 0; i < kk; ++i) q += yv[i] * yv[i];
    q = 1.0 / sqrt(q);
    for (int i = 0; i < kk; ++i) yv[i] *= q;
  }
  L.tri[k] = tmin;
  L.tri[k + 1] = tmax;
  L.tri[k + 2] = (double)kk;
}

// u = sum_{j < kk} y_j V_j  (written to w)
__global__ void k_lz_ritz(LzDev L) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= L.len) return;
  const int kk = (int)L.tri[L.k + 2];
  double u = 0.0;
#pragma unroll 8
  for (int j = 0; j < kk; ++j) u += L.tri[j] * L.Q[(size_t)(j + 1) * L.len + e];
  L.w[e] = u;
}

// h = H_t u - theta u (its squared norm is taken by k_lz_dots and k_lz_sum)
__global__ void k_lz_resid(LzDev L) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= L.len) return;
  L.h[e] = L.h[e] - L.tri[L.k] * L.w[e];
}
__global__ void k_lz_sum(const double* __restrict__ p, int m, double* __restrict__ out) {
  double v = 0.0;
  for (int q = threadIdx.x; q < m; q += 64) v += p[q];
  v = wave_sum(v);
  if (threadIdx.x == 0) *out = v;
}

struct LzPlan {
  Plan hv;
  size_t hv_bytes = 0, f_bytes = 0, total = 0;
  char* hvb = nullptr;  // workspace of the staged HVP
  char* fws = nullptr;  // workspace of the force call
  int S = 0;            // chunks of a dot product
  LzDev D;
};

static bool lz_plan(int64_t n, int k, char* base, LzPlan& P) {
  if (n < 2 || n > (1 << 26) || k < 2 || k > 4096) return false;
  P.hv_bytes = hvp64_bytes(n);
  P.f_bytes = coulomb_workspace_bytes(CD_OP_FORCES, n, 0, 0, CD_FP64);
  if (!P.hv_bytes || !P.f_bytes) return false;
  Carve cv;
  cv.base = base;
  P.hvb = cv.take<char>(P.hv_bytes);
  P.fws = cv.take<char>(P.f_bytes);
  LzDev& D = P.D;
  D.n = (int)n;
  D.npad = hvp64_npad(n);
  const size_t np = D.npad, len = 2 * np;
  D.len = len;
  D.k = k;
  P.S = (int)((len + kDotE - 1) / kDotE);
  D.fx = cv.take<double>(n);
  D.fy = cv.take<double>(n);
  D.ux = cv.take<double>(np);
  D.uy = cv.take<double>(np);
  D.wgt = cv.take<double>(np);
  D.kind = cv.take<int32_t>(np);
  D.Q = cv.take<double>(len * (k + 2));
  D.w = cv.take<double>(len);
  D.h = cv.take<double>(len);
  D.part = cv.take<double>((size_t)(k + 1) * P.S);
  D.nrm = cv.take<double>(len / kAxE);
  D.a1 = cv.take<double>(1);
  D.alpha = cv.take<double>(k);
  D.beta = cv.take<double>(k + 1);
  D.tri = cv.take<double>(k + 4);
  D.scr = cv.take<double>(2 * (size_t)k);
  P.total = cv.off + 512;
  return true;
}

size_t lanczos_workspace_bytes(int64_t n, int k) {
  LzPlan P;
  return lz_plan(n, k, nullptr, P) ? P.total : 0;
}

}  // namespace cd

using namespace cd;

extern "C" int tangent_lanczos(const double* x, const double* y, int64_t n, const int32_t* mask,
                               int32_t k, int32_t deflate_rotation, uint64_t seed,
                               double* out_host, void* ws, size_t ws_bytes, void* stream) {
  if (!x || !y || !out_host) return CD_ERR_INVALID_ARG;
  LzPlan P;
  if (!lz_plan(n, k, nullptr, P)) return CD_ERR_INVALID_ARG;
  if (!ws) return CD_ERR_WORKSPACE;
  if (ws_bytes < P.total) return CD_ERR_WORKSPACE;
  char* base = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255));
  lz_plan(n, k, base, P);
  hipStream_t st = (hipStream_t)stream;
  LzDev& D = P.D;
  D.x = x;
  D.y = y;
  D.mask = mask;
  int rc = coulomb_forces(x, y, n, CD_FP64, D.fx, D.fy, nullptr, P.fws, P.f_bytes, stream);
  if (rc) return rc;
  if ((rc = hvp64_stage(P.hv, P.hvb, n, x, y, st))) return rc;
  D.perm = P.hv.perm;
  const size_t len = D.len;
  const int np = D.npad, dfl = deflate_rotation ? 1 : 0;
  const dim3 gn((unsigned)((np + 255) / 256)), g2((unsigned)((len + 255) / 256)), b256(256);
  const dim3 ga((unsigned)(len / kAxE));
  double* const V = D.Q + len;            // the basis
  double* const B = dfl ? D.Q : V;        // what a new vector is made orthogonal to
  auto dots = [&](const double* A, int m, const double* b) {
    if (m) hipLaunchKernelGGL(k_lz_dots, dim3(m, P.S), dim3(kDotT), 0, st, A, len, b, D.part);
  };
  auto axpys = [&](int m, int last, int step) {
    hipLaunchKernelGGL(k_lz_axpys, ga, b256, sizeof(double) * (m ? m : 1), st, D, B, m, P.S, last,
                       step);
  };
  auto next = [&](double* out, double* beta) {
    hipLaunchKernelGGL(k_lz_next, g2, b256, 0, st, D, out, beta);
  };
  hipLaunchKernelGGL(k_lz_setup, gn, b256, 0, st, D, seed, dfl);
  if (dfl) {
    // the unit rotation: w holds the start vector, so its norm goes through h
    LzDev R = D;
    R.w = D.h;
    if ((rc = hip_status(hipMemcpyAsync(D.h, D.Q, sizeof(double) * len, hipMemcpyDeviceToDevice,
                                        st))))
      return rc;
    hipLaunchKernelGGL(k_lz_axpys, ga, b256, sizeof(double), st, R, B, 0, P.S, 0, 0);
    hipLaunchKernelGGL(k_lz_next, g2, b256, 0, st, R, D.Q, nullptr);
  }
  // normalise the start vector
  dots(B, dfl, D.w);
  axpys(dfl, 0, 0);
  next(V, nullptr);
  auto apply = [&](const double* v, double* out) {
    int r = hvp64_sorted(P.hv, v, v + np, D.h, D.h + np, st);
    hipLaunchKernelGGL(k_lz_post, gn, b256, 0, st, D, v, out);
    return r;
  };
  for (int j = 0; j < k; ++j) {
    if ((rc = apply(V + (size_t)j * len, D.w))) return rc;
    for (int pass = 1; pass <= 2; ++pass) {
      dots(B, j + 1 + dfl, D.w);
      axpys(j + 1 + dfl, pass, j);
    }
    next(V + (size_t)(j + 1) * len, D.beta + j);
  }
  hipLaunchKernelGGL(k_lz_tridiag, dim3(1), dim3(128), 0, st, D);
  hipLaunchKernelGGL(k_lz_ritz, g2, b256, 0, st, D);
  if ((rc = apply(D.w, D.h))) return rc;
  hipLaunchKernelGGL(k_lz_resid, g2, b256, 0, st, D);
  dots(D.h, 1, D.h);
  hipLaunchKernelGGL(k_lz_sum, dim3(1), dim3(64), 0, st, D.part, P.S, D.tri + k + 3);
  double host[4];
  if ((rc = hip_status(hipMemcpyAsync(host, D.tri + k, 4 * sizeof(double), hipMemcpyDeviceToHost,
                                      st))))
    return rc;
  if ((rc = hip_status(hipStreamSynchronize(st)))) return rc;
  out_host[0] = host[0];
  out_host[1] = sqrt(host[3]);
  out_host[2] = host[1];
  out_host[3] = host[2];
  return CD_OK;
}
