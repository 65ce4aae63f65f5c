// Structure analysis of a configuration (paper Sec. III: Voronoi
// coordination, the bond-orientational order psi_6, the radial density).
//
// Voronoi cells.  The charges are binned on a uniform grid of cells about
// one mean spacing wide (counting sort; each cell's list is then put in
// index order, so everything downstream is deterministic).  One wave per
// charge i clips a large square around r_i by the bisector half-plane of
// every charge j in the (2R+1)^2 cells around its own (Sutherland-Hodgman in
// coordinates relative to r_i, FP64); each polygon edge remembers the charge
// whose bisector made it.  A charge j outside the searched block lies
// farther than its distance D from r_i (D: the block's margin around r_i,
// unbounded where the block reaches the grid's edge); it can cut a vertex v
// only if |r_j - r_i| < 2|v|.  So a bounded cell is final when every vertex
// satisfies 2|v| <= D; otherwise the search widens (k_voronoi).  Charges on
// the convex hull (host code, monotone chain among the charges outside a
// polygon of extreme ones) have unbounded cells and report z = -2.
// z_i = number of bisector edges = Voronoi (Delaunay) neighbours;
// psi_6(i) = (1/z_i) sum_j u_ij^6, u_ij = (r_j - r_i)/|r_j - r_i| as a complex
// number.
#include <algorithm>
#include <cmath>
#include <vector>

#include "common.hpp"

namespace cd {

constexpr int kVorR = 2;       // cells searched on each side of the charge's cell
constexpr int kVorMaxV = 48;   // polygon vertices
constexpr double kVorBox = 4.0;
constexpr double kGridL = 1.0 + 1e-9;  // the grid covers [-L, L]^2
constexpr int kScanT = 1024;

struct Grid {
  int G;       // cells per side
  double c;    // cell width
};

__host__ __device__ inline Grid make_grid(int64_t n) {
  const double h = sqrt(2.0 * 3.141592653589793 / (sqrt(3.0) * (double)n));
  double g = floor(2.0 * kGridL / h);
  if (g < 1.0) g = 1.0;
  if (g > 4096.0) g = 4096.0;
  Grid q;
  q.G = (int)g;
  q.c = 2.0 * kGridL / q.G;
  return q;
}

constexpr int kScanE = 4 * kScanT;  // counts per workgroup of the scan
// Convex-hull candidates: extreme charges in kHullDirs directions, one row of
// them per wave of kHullPer charges; the candidates' copies.
constexpr int kHullDirs = 64;
constexpr int kHullPer = 128;
struct HullRow {
  double v[kHullDirs];
  int32_t i[kHullDirs];
};
struct HullPoint {
  double x, y;
  int64_t i;  // entry 0 holds the count
};
static int hull_rows(int64_t n) { return (int)((n + kHullPer - 1) / kHullPer); }

size_t structure_workspace_bytes(int64_t n) {
  const Grid g = make_grid(n);
  const size_t cells = (size_t)g.G * g.G;
  Carve cv;
  cv.take<int32_t>(cells + 1);  // counts, then starts
  cv.take<int32_t>(cells);      // fill cursors
  cv.take<int32_t>((size_t)n);  // cell of each charge
  cv.take<int32_t>((size_t)n);  // charges by cell
  cv.take<int32_t>((size_t)n);  // convex-hull flags
  cv.take<int32_t>(cells / kScanE + 1);  // scan sums
  cv.take<HullRow>((size_t)hull_rows(n) + 1);
  cv.take<HullPoint>((size_t)n + 1);
  return cv.off + 256;
}

__device__ __forceinline__ int cell_coord(double v, const Grid& g) {
  int k = (int)floor((v + kGridL) / g.c);
  return k < 0 ? 0 : (k >= g.G ? g.G - 1 : k);
}

__global__ void k_fill_int(int32_t* __restrict__ a, int m, int v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m) a[i] = v;
}

__global__ void k_cell_count(const double* __restrict__ x, const double* __restrict__ y, int n,
                             Grid g, int32_t* __restrict__ count, int32_t* __restrict__ cell) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int c = cell_coord(y[i], g) * g.G + cell_coord(x[i], g);
  cell[i] = c;
  atomicAdd(&count[c], 1);
}

// Exclusive scan of m counts in place, a[m] = the total: one workgroup per
// kScanE counts; the first launch writes each workgroup's sum, the second adds
// up the sums before its own (4096 of them at most: 2 passes over the counts
// instead of one workgroup's 98 rounds at m = 1e5, 104 us).
__device__ __forceinline__ int wg_total(int v, int* ws) {
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = v;
  __syncthreads();
  int t = 0;
  for (int q = 0; q < kScanT / 64; ++q) t += ws[q];
  __syncthreads();
  return t;
}
__global__ __launch_bounds__(kScanT) void k_scan_sums(const int32_t* __restrict__ a, int m,
                                                      int32_t* __restrict__ sums) {
  __shared__ int ws[kScanT / 64];
  int v = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = blockIdx.x * kScanE + q * kScanT + threadIdx.x;
    v += i < m ? a[i] : 0;
  }
  v = wg_total(v, ws);
  if (threadIdx.x == 0) sums[blockIdx.x] = v;
}
__global__ __launch_bounds__(kScanT) void k_scan_write(int32_t* __restrict__ a, int m,
                                                       const int32_t* __restrict__ sums) {
  __shared__ int ws[kScanT / 64];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  int before = 0;
  for (int q = t; q < (int)blockIdx.x; q += kScanT) before += sums[q];
  before = wg_total(before, ws);
  const int i0 = blockIdx.x * kScanE + 4 * t;
  int v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = i0 + q < m ? a[i0 + q] : 0;
  const int own = (v[0] + v[1]) + (v[2] + v[3]);
  int s = own;
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(s, off, 64);
    if (lane >= off) s += u;
  }
  if (lane == 63) ws[w] = s;
  __syncthreads();
  for (int q = 0; q < w; ++q) s += ws[q];
  int e = before + s - own;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (i0 + q < m) a[i0 + q] = e;
    e += v[q];
    if (i0 + q == m - 1) a[m] = e;
  }
}

__global__ void k_cell_fill(int n, const int32_t* __restrict__ cell,
                            const int32_t* __restrict__ start, int32_t* __restrict__ cursor,
                            int32_t* __restrict__ slot) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int c = cell[i];
  slot[start[c] + atomicAdd(&cursor[c], 1)] = i;
}

// Each cell's charges in increasing index order (insertion sort; cells hold
// a handful of charges).
__global__ void k_cell_sort(int m, const int32_t* __restrict__ start, int32_t* __restrict__ slot) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= m) return;
  const int a = start[c], b = start[c + 1];
  for (int k = a + 1; k < b; ++k) {
    const int v = slot[k];
    int q = k - 1;
    while (q >= a && slot[q] > v) {
      slot[q + 1] = slot[q];
      --q;
    }
    slot[q + 1] = v;
  }
}

// Hull candidates.  The extreme charges of kHullDirs directions span a convex
// polygon inside the hull; a charge clearly inside the polygon is no hull
// vertex.  What is left (the outermost rings) goes to the host, whose monotone
// chain decides exactly as it would among all charges (sorting all 1e5 of them
// there took 7 of the call's 11 ms).
// One wave per kHullPer charges, one direction per lane.
__global__ __launch_bounds__(256) void k_hull_rows(const double* __restrict__ x,
                                                   const double* __restrict__ y, int n, int rows,
                                                   HullRow* __restrict__ out) {
  const int r = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  if (r >= rows) return;
  double c, sn;
  sincospi(2.0 * lane / kHullDirs, &sn, &c);
  const int j0 = r * kHullPer, j1 = min(n, j0 + kHullPer);
  double best = -1e300;
  int bi = j0;
#pragma unroll 8
  for (int j = j0; j < j1; ++j) {
    const double v = c * x[j] + sn * y[j];
    if (v > best) {
      best = v;
      bi = j;
    }
  }
  out[r].v[lane] = best;
  out[r].i[lane] = bi;
}
// Row m, one past the m input rows, gets the indices of the extremes of all of
// them (not their values); the candidate count is cleared.
__global__ __launch_bounds__(1024) void k_hull_extremes(HullRow* __restrict__ rows, int m,
                                                        HullPoint* __restrict__ pts) {
  __shared__ double v[16][kHullDirs];
  __shared__ int32_t i[16][kHullDirs];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double best = -1e300;
  int bi = 0;
#pragma unroll 4
  for (int r = w; r < m; r += 16) {
    const double q = rows[r].v[lane];
    const int qi = rows[r].i[lane];
    if (q > best) {
      best = q;
      bi = qi;
    }
  }
  v[w][lane] = best;
  i[w][lane] = bi;
  __syncthreads();
  if (w > 0) return;
  for (int q = 1; q < 16; ++q)
    if (v[q][lane] > best) {
      best = v[q][lane];
      bi = i[q][lane];
    }
  rows[m].i[lane] = bi;
  if (lane == 0) pts[0].i = 0;
}
// Lists the charges not clearly inside the polygon (in any order).
__global__ __launch_bounds__(256) void k_hull_candidates(const double* __restrict__ x,
                                                         const double* __restrict__ y, int n,
                                                         const HullRow* __restrict__ ext,
                                                         HullPoint* __restrict__ pts) {
  __shared__ double ex[kHullDirs], ey[kHullDirs];
  if (threadIdx.x < kHullDirs) {
    const int e = ext->i[threadIdx.x];
    ex[threadIdx.x] = x[e];
    ey[threadIdx.x] = y[e];
  }
  __syncthreads();
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= n) return;
  const double px = x[j], py = y[j];
  // left of every edge by more than rounding (NaN: not inside); repeated
  // extremes have no edge, and fewer than three of them enclose nothing
  bool inside = true;
  int edges = 0;
  for (int k = 0; k < kHullDirs && inside; ++k) {
    const double ax = ex[k], ay = ey[k];
    const double bx = ex[(k + 1) % kHullDirs], by = ey[(k + 1) % kHullDirs];
    const double dx = bx - ax, dy = by - ay;
    if (dx == 0.0 && dy == 0.0) continue;
    ++edges;
    inside = dx * (py - ay) - dy * (px - ax) > 1e-9 * (fabs(dx) + fabs(dy));
  }
  if (inside && edges >= 3) return;
  const unsigned long long e = atomicAdd((unsigned long long*)&pts[0].i, 1ull);
  HullPoint q;
  q.x = px;
  q.y = py;
  q.i = j;
  pts[e + 1] = q;
}
__global__ void k_set_flags(const int32_t* __restrict__ list, int m, int32_t* __restrict__ flags) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < m) flags[list[k]] = 1;
}

// Farthest distance from r_i of a point that could cut vertex v (relative to
// r_i): such a charge lies in the disk about V = r_i + v through r_i (radius
// |v|) and in the disk of radius Rb about the origin that holds every
// charge.  The farthest point of that lens from r_i is the point of circle V
// opposite r_i, the point of circle Rb opposite r_i, or one of the two circle
// intersections (each candidate counted when it lies in the other disk; the
// tests allow slack, which can only add candidates).  Without the Rb disk the
// bound is 2|v|; with it, the long cells of charges next to the hull, whose
// far vertices lie well outside the disk, certify at a short range.
__device__ double lens_reach(double cx, double cy, double vx, double vy, double Rb) {
  const double rho2 = vx * vx + vy * vy, rho = sqrt(rho2);
  const double Vx = cx + vx, Vy = cy + vy;
  const double Ax = Vx + vx, Ay = Vy + vy;
  const double Rb2 = Rb * Rb;
  if (Ax * Ax + Ay * Ay <= Rb2 * (1.0 + 1e-9)) return 2.0 * rho;
  double M = 0.0;
  const double cn = sqrt(cx * cx + cy * cy);
  if (cn > 0.0) {
    const double ex = -Rb * cx / cn - Vx, ey = -Rb * cy / cn - Vy;
    if (ex * ex + ey * ey <= rho2 * (1.0 + 1e-9)) M = Rb + cn;
  } else {
    M = Rb;
  }
  const double d2 = Vx * Vx + Vy * Vy, d = sqrt(d2);
  if (d > 0.0) {
    const double a = (Rb2 - rho2 + d2) / (2.0 * d);
    const double hh = Rb2 - a * a;
    if (hh > -1e-9 * Rb2) {
      const double h = sqrt(fmax(hh, 0.0));
      const double ux = Vx / d, uy = Vy / d;
      const double p1x = a * ux - h * uy - cx, p1y = a * uy + h * ux - cy;
      const double p2x = a * ux + h * uy - cx, p2y = a * uy - h * ux - cy;
      M = fmax(M, fmax(sqrt(p1x * p1x + p1y * p1y), sqrt(p2x * p2x + p2y * p2y)));
    }
  }
  return M;
}
// Charges on the convex hull have unbounded cells: z = -2, psi_6 = 0.  The cell
// of any other charge is clipped by one wave, its polygon in LDS.
//
// The charges around r_i are taken ring by ring of cells around its own, so
// that near charges cut first, 64 of a ring at a time, one per lane.  Each lane
// tests its charge's bisector against the polygon's vertices; the first charge
// that cuts clips the polygon (one vertex per lane, their places by ballots),
// all lanes after it test the new polygon, and so on: the charges act one after
// the other, each on the polygon the ones before it left.  (A charge that
// left the larger polygon whole can still cut a corner of rounding's size off
// the new one, where more than three charges lie on a circle about a vertex.)  A charge of ring k >= 1 lies
// at least (k - 1) c from r_i, so the rings stop once that is beyond every
// vertex's reach (lens_reach).
// The search widens (2, 6, 18, .. cells on each side, then the whole grid) until
// every vertex's reach is within the block's margin: no charge outside can
// cut the polygon.  A certified polygon with an edge on the square belongs to a
// cell that extends beyond it (a charge next to the hull can have far
// vertices): the square grows to 1e4 once, at the same range; z = -1 if even
// that does not hold it, or if the polygon outgrows its vertex arrays.
// Bound: the cuts' chain of LDS reads.  One thread per charge, its polygon in
// scratch memory, took 2.54 ms at n = 1e5, most of it in the few threads next
// to the hull whose search widens; a wave per charge takes 0.46 ms.
constexpr int kVorW = 4;
__global__ __launch_bounds__(64 * kVorW) void k_voronoi(const double* __restrict__ x,
                                                        const double* __restrict__ y, int n, Grid g,
                                                        const int32_t* __restrict__ start,
                                                        const int32_t* __restrict__ slot,
                                                        const int32_t* __restrict__ hullf,
                                                        double Rb, int32_t* __restrict__ zout,
                                                        double* __restrict__ psi) {
  __shared__ double s_px[kVorW][2][kVorMaxV], s_py[kVorW][2][kVorMaxV];
  __shared__ int32_t s_lab[kVorW][2][kVorMaxV], s_pre[kVorW][64], s_st[kVorW][64];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int sl = blockIdx.x * kVorW + w;  // in cell order: neighbours share the caches
  if (sl >= n) return;
  const int i = __builtin_amdgcn_readfirstlane(slot[sl]);
  if (hullf[i]) {  // on the convex hull: unbounded cell
    if (lane == 0) {
      zout[i] = -2;
      if (psi) psi[2 * (size_t)i] = psi[2 * (size_t)i + 1] = 0.0;
    }
    return;
  }
  auto fence = [] {  // the other lanes' LDS writes before this lane's reads
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  const double xi = x[i], yi = y[i];
  const int cx = cell_coord(xi, g), cy = cell_coord(yi, g);
  int R = kVorR, cur = 0, nv = 0, z = -1;
  double B = kVorBox;
  // lens_reach with slack for rounding, over the polygon's vertices
  auto reach = [&] {
    const double m = lane < nv ? lens_reach(xi, yi, s_px[w][cur][lane], s_py[w][cur][lane], Rb) : 0.0;
    return wave_max(m) * (1.0 + 1e-9) + 1e-12;
  };
  for (;;) {
    const int x0 = max(0, cx - R), x1 = min(g.G - 1, cx + R);
    const int y0 = max(0, cy - R), y1 = min(g.G - 1, cy + R);
    // the square of half-width B around r_i
    cur = 0;
    nv = 4;
    if (lane < 4) {
      s_px[w][0][lane] = lane == 1 || lane == 2 ? B : -B;
      s_py[w][0][lane] = lane >= 2 ? B : -B;
      s_lab[w][0][lane] = -1;
    }
    fence();
    const int kmax = max(max(cx - x0, x1 - cx), max(cy - y0, y1 - cy));
    bool over = false;
    for (int k = 0; k <= kmax && !over; ++k) {
      if (k >= 2 && (k - 1) * g.c >= reach()) break;
      // the ring's cells row by row: its first row, two cells of each row
      // between, its last row
      const int row = 2 * k + 1, cells = k ? 8 * k : 1;
      for (int u0 = 0; u0 < cells && !over; u0 += 64) {
        const int u = u0 + lane;
        int qx = cx, qy = cy;
        if (k) {
          const int v = u - row;
          qy = u < row ? cy - k : v < 4 * k - 2 ? cy - k + 1 + (v >> 1) : cy + k;
          qx = u < row ? cx - k + u : v < 4 * k - 2 ? ((v & 1) ? cx + k : cx - k)
                                                    : cx - k + v - (4 * k - 2);
        }
        int st = 0, cnt = 0;
        if (u < cells && qx >= x0 && qx <= x1 && qy >= y0 && qy <= y1) {
          const int c = qy * g.G + qx;
          st = start[c];
          cnt = start[c + 1] - st;
        }
        int pre = cnt;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const int q = __shfl_up(pre, off, 64);
          if (lane >= off) pre += q;
        }
        const int total = __builtin_amdgcn_readlane(pre, 63);
        s_pre[w][lane] = pre - cnt;
        s_st[w][lane] = st;
        fence();
        for (int e0 = 0; e0 < total && !over; e0 += 64) {
          const int e = e0 + lane;
          int l = 0;  // the last cell whose first charge is not beyond e
#pragma unroll
          for (int b = 32; b >= 1; b >>= 1)
            if (s_pre[w][l + b] <= e) l += b;
          const int j = e < total ? slot[s_st[w][l] + e - s_pre[w][l]] : i;
          const double dx = x[j] - xi, dy = y[j] - yi;
          const double hd = 0.5 * (dx * dx + dy * dy);
          // f(v) = v.d - |d|^2/2 <= 0 keeps v; a coincident charge has no bisector
          auto cuts = [&] {
            bool out = false;
            for (int q = 0; q < nv; ++q) out |= s_px[w][cur][q] * dx + s_py[w][cur][q] * dy - hd > 0.0;
            return out;
          };
          const bool real = j != i && hd > 0.0;
          uint64_t m = __ballot(real && cuts());
          while (m) {
            const int f = __builtin_ctzll(m);
            const double ex = lane_f64(dx, f), ey = lane_f64(dy, f), eh = lane_f64(hd, f);
            const int ej = __builtin_amdgcn_readlane(j, f);
            // Sutherland-Hodgman, one vertex per lane: an inside vertex stays,
            // an edge that crosses gives its crossing
            const int q = max(min(lane, nv - 1), 0), r = q + 1 >= nv ? 0 : q + 1;
            const double ax = s_px[w][cur][q], ay = s_py[w][cur][q];
            const double bx = s_px[w][cur][r], by = s_py[w][cur][r];
            const int la = s_lab[w][cur][q];
            const double fa = ax * ex + ay * ey - eh, fb = bx * ex + by * ey - eh;
            const bool in = lane < nv, keep = in && fa <= 0.0;
            const bool cross = in && (fa <= 0.0) != (fb <= 0.0);
            const uint64_t mk = __ballot(keep), mc = __ballot(cross);
            const int nn = __popcll(mk) + __popcll(mc);
            if (nn > kVorMaxV) {
              over = true;
              break;
            }
            int pos = __popcll(mk & lt) + __popcll(mc & lt);
            const int nx = cur ^ 1;
            if (keep) {
              s_px[w][nx][pos] = ax;
              s_py[w][nx][pos] = ay;
              s_lab[w][nx][pos] = la;
              ++pos;
            }
            if (cross) {
              const double t = fa / (fa - fb);
              s_px[w][nx][pos] = ax + t * (bx - ax);
              s_py[w][nx][pos] = ay + t * (by - ay);
              s_lab[w][nx][pos] = keep ? ej : la;
            }
            cur = nx;
            nv = nn;
            fence();
            m = __ballot(real && lane > f && cuts());
          }
        }
        fence();  // s_pre and s_st are written again
      }
    }
    if (over) break;  // z = -1: more vertices than the polygon holds
    // the searched block's margin around r_i (unbounded where it reaches the grid's edge)
    const double inf = 1e300;
    const double ml = x0 == 0 ? inf : xi - (-kGridL + x0 * g.c);
    const double mr = x1 == g.G - 1 ? inf : (-kGridL + (x1 + 1) * g.c) - xi;
    const double mb = y0 == 0 ? inf : yi - (-kGridL + y0 * g.c);
    const double mt = y1 == g.G - 1 ? inf : (-kGridL + (y1 + 1) * g.c) - yi;
    const double D = fmin(fmin(ml, mr), fmin(mb, mt));
    const bool box = __ballot(lane < nv && s_lab[w][cur][min(lane, kVorMaxV - 1)] < 0) != 0;
    const bool full = x0 == 0 && y0 == 0 && x1 == g.G - 1 && y1 == g.G - 1;
    if (full || reach() <= D) {
      if (!box) {
        z = 0;
        break;
      }
      if (B < 1e4) {
        B = 1e4;
        continue;
      }
      break;  // z = -1
    }
    R *= 3;
  }
  double sre = 0.0, sim = 0.0;
  if (z == 0) {
    const int j = lane < nv ? s_lab[w][cur][lane] : -1;
    z = __popcll(__ballot(j >= 0));
    if (psi) {
      if (j >= 0) {
        const double dx = x[j] - xi, dy = y[j] - yi;
        const double r = sqrt(dx * dx + dy * dy);
        const double ur = dx / r, ui = dy / r;
        const double u2r = ur * ur - ui * ui, u2i = 2.0 * ur * ui;
        const double u4r = u2r * u2r - u2i * u2i, u4i = 2.0 * u2r * u2i;
        sre = u4r * u2r - u4i * u2i;
        sim = u4r * u2i + u4i * u2r;
      }
      sre = wave_sum(sre);
      sim = wave_sum(sim);
    }
  }
  if (lane == 0) {
    zout[i] = z;
    if (psi) {
      psi[2 * (size_t)i] = z > 0 ? sre / z : 0.0;
      psi[2 * (size_t)i + 1] = z > 0 ? sim / z : 0.0;
    }
  }
}

// Statistics of a coordination result in one workgroup: per thread a strided
// pass in index order, then a tree over the threads, so the sums do not
// depend on timing.  out[0..4]: fractions of the bounded cells with z = 4..8;
// out[5]: mean |psi_6| over the bounded cells; out[6..8]: the counts of
// bounded cells, hull charges and unresolved cells.
__global__ __launch_bounds__(kScanT) void k_structure_stats(const int32_t* __restrict__ z,
                                                            const double* __restrict__ psi6, int n,
                                                            double* __restrict__ out) {
  __shared__ double s_abs[kScanT];
  __shared__ int32_t s_cnt[8][kScanT];
  const int t = threadIdx.x;
  int32_t c[8] = {0, 0, 0, 0, 0, 0, 0, 0};  // z = 4..8, bounded, hull, unresolved
  double a = 0.0;
  // eight charges' loads go out together (one at a time the pass waited 98
  // times on memory at n = 1e5: 84 us)
  for (int i0 = t; i0 < n; i0 += 8 * kScanT) {
    int zq[8];
    double2 pq[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int i = min(i0 + q * kScanT, n - 1);
      zq[q] = z[i];
      pq[q] = psi6 ? make_double2(psi6[2 * (size_t)i], psi6[2 * (size_t)i + 1])
                   : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (i0 + q * kScanT >= n) continue;
      const int zi = zq[q];
      if (zi >= 0) {
        ++c[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) c[k] += zi == k + 4;
        if (psi6) a += sqrt(pq[q].x * pq[q].x + pq[q].y * pq[q].y);
      } else if (zi == -2) {
        ++c[6];
      } else {
        ++c[7];
      }
    }
  }
  s_abs[t] = a;
  for (int k = 0; k < 8; ++k) s_cnt[k][t] = c[k];
  __syncthreads();
  for (int w = kScanT / 2; w > 0; w >>= 1) {
    if (t < w) {
      s_abs[t] += s_abs[t + w];
      for (int k = 0; k < 8; ++k) s_cnt[k][t] += s_cnt[k][t + w];
    }
    __syncthreads();
  }
  if (t == 0) {
    const int32_t b = s_cnt[5][0];
    const double inv = b > 0 ? 1.0 / (double)b : 0.0;
    for (int k = 0; k < 5; ++k) out[k] = b > 0 ? (double)s_cnt[k][0] * inv : 0.0;
    out[5] = b > 0 && psi6 ? s_abs[0] / (double)b : 0.0;
    out[6] = (double)b;
    out[7] = (double)s_cnt[6][0];
    out[8] = (double)s_cnt[7][0];
  }
}

#pragma clang fp contract(off)
// Up to kRadLds bins: counted per workgroup in LDS, one global add per bin and
// workgroup that has any (every charge adding to global memory took 681 us for
// 50 bins and 1e5 charges, which are few addresses).
constexpr int kRadLds = 8192, kRadT = 1024;
template <bool LDS>
__global__ __launch_bounds__(kRadT) void k_radial(const double* __restrict__ x,
                                                  const double* __restrict__ y, int n, int nbins,
                                                  int32_t* __restrict__ counts) {
  extern __shared__ int32_t loc[];
  if (LDS) {
    for (int k = threadIdx.x; k < nbins; k += kRadT) loc[k] = 0;
    __syncthreads();
  }
  int32_t* const to = LDS ? loc : counts;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const double a = x[i] * x[i], b = y[i] * y[i];
    const double r = sqrt(a + b);
    const double f = floor(r * (double)nbins);
    int k = f < 0.0 ? 0 : (f >= (double)nbins ? nbins - 1 : (int)f);
    if (!(r == r)) k = nbins - 1;  // NaN
    atomicAdd(&to[k], 1);
  }
  if (LDS) {
    __syncthreads();
    for (int k = threadIdx.x; k < nbins; k += kRadT)
      if (loc[k]) atomicAdd(&counts[k], loc[k]);
  }
}
#pragma clang fp contract(on)

}  // namespace cd

using namespace cd;

namespace {

// Vertices of the convex hull (Andrew's monotone chain; points on an edge
// between two vertices are not vertices) among p; their indices.
std::vector<int32_t> hull_of(std::vector<HullPoint>& p) {
  std::sort(p.begin(), p.end(), [](const HullPoint& a, const HullPoint& b) {
    return a.x != b.x ? a.x < b.x : a.y != b.y ? a.y < b.y : a.i < b.i;
  });
  const int n = (int)p.size();
  auto cross = [&](int a, int b, int c) {
    return (p[b].x - p[a].x) * (p[c].y - p[a].y) - (p[b].y - p[a].y) * (p[c].x - p[a].x);
  };
  std::vector<int> h(2 * (size_t)n + 2);
  int k = 0;
  for (int t = 0; t < n; ++t) {  // lower hull
    while (k >= 2 && cross(h[k - 2], h[k - 1], t) <= 0.0) --k;
    h[k++] = t;
  }
  for (int t = n - 2, lo = k + 1; t >= 0; --t) {  // upper hull
    while (k >= lo && cross(h[k - 2], h[k - 1], t) <= 0.0) --k;
    h[k++] = t;
  }
  std::vector<int32_t> out(k);
  for (int t = 0; t < k; ++t) out[t] = (int32_t)p[h[t]].i;
  return out;
}

}  // namespace

extern "C" {

int voronoi_coordination(const double* x, const double* y, int64_t n, int32_t* z, double* psi6,
                         void* ws, size_t ws_bytes, void* stream) {
  if (!x || !y || !z || n < 1 || n > (1 << 26)) return CD_ERR_INVALID_ARG;
  if (!ws || ws_bytes < structure_workspace_bytes(n)) return CD_ERR_WORKSPACE;
  const Grid g = make_grid(n);
  const int cells = g.G * g.G;
  Carve cv;
  cv.base = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255));
  int32_t* start = cv.take<int32_t>((size_t)cells + 1);
  int32_t* cursor = cv.take<int32_t>((size_t)cells);
  int32_t* cell = cv.take<int32_t>((size_t)n);
  int32_t* slot = cv.take<int32_t>((size_t)n);
  int32_t* hullf = cv.take<int32_t>((size_t)n);
  int32_t* sums = cv.take<int32_t>((size_t)cells / kScanE + 1);
  HullRow* rows = cv.take<HullRow>((size_t)hull_rows(n) + 1);
  HullPoint* pts = cv.take<HullPoint>((size_t)n + 1);
  hipStream_t st = (hipStream_t)stream;
  const int nn = (int)n;
  double Rb = 0.0;  // radius of a disk about the origin that holds every charge
  {
    const int m = hull_rows(n);
    hipLaunchKernelGGL(k_hull_rows, dim3((m + 3) / 4), dim3(256), 0, st, x, y, nn, m, rows);
    hipLaunchKernelGGL(k_hull_extremes, dim3(1), dim3(1024), 0, st, rows, m, pts);
    hipLaunchKernelGGL(k_hull_candidates, dim3((nn + 255) / 256), dim3(256), 0, st, x, y, nn,
                       rows + m, pts);
    hipLaunchKernelGGL(k_fill_int, dim3((nn + 255) / 256), dim3(256), 0, st, hullf, nn, 0);
    // the count and, in most cases, all candidates in one copy
    const size_t first = std::min<size_t>((size_t)n, 8192);
    std::vector<HullPoint> p(first + 1);
    auto fetch = [&](size_t at, size_t cnt) {
      int e = hip_status(hipMemcpyAsync(p.data() + at, pts + at, sizeof(HullPoint) * cnt,
                                        hipMemcpyDeviceToHost, st));
      return e ? e : hip_status(hipStreamSynchronize(st));
    };
    int rc = hip_status(hipGetLastError());
    if (rc || (rc = fetch(0, first + 1))) return rc;
    const size_t cnt = (size_t)p[0].i;
    p.resize(cnt + 1);
    if (cnt > first && (rc = fetch(first + 1, cnt - first))) return rc;
    p.erase(p.begin());
    for (const HullPoint& q : p) Rb = fmax(Rb, sqrt(q.x * q.x + q.y * q.y));
    Rb = Rb * (1.0 + 1e-12) + 1e-300;
    const std::vector<int32_t> hull = hull_of(p);
    // the candidates' room holds the list of vertices
    int32_t* list = reinterpret_cast<int32_t*>(pts);
    rc = hip_status(hipMemcpyAsync(list, hull.data(), sizeof(int32_t) * hull.size(),
                                   hipMemcpyHostToDevice, st));
    if (!rc) rc = hip_status(hipStreamSynchronize(st));  // hull is released on return
    if (rc) return rc;
    hipLaunchKernelGGL(k_set_flags, dim3((unsigned)((hull.size() + 255) / 256)), dim3(256), 0, st,
                       list, (int)hull.size(), hullf);
  }
  hipLaunchKernelGGL(k_fill_int, dim3((cells + 256) / 256), dim3(256), 0, st, start, cells + 1, 0);
  hipLaunchKernelGGL(k_fill_int, dim3((cells + 255) / 256), dim3(256), 0, st, cursor, cells, 0);
  hipLaunchKernelGGL(k_cell_count, dim3((nn + 255) / 256), dim3(256), 0, st, x, y, nn, g, start,
                     cell);
  hipLaunchKernelGGL(k_scan_sums, dim3((cells + kScanE - 1) / kScanE), dim3(kScanT), 0, st, start,
                     cells, sums);
  hipLaunchKernelGGL(k_scan_write, dim3((cells + kScanE - 1) / kScanE), dim3(kScanT), 0, st, start,
                     cells, sums);
  hipLaunchKernelGGL(k_cell_fill, dim3((nn + 255) / 256), dim3(256), 0, st, nn, cell, start,
                     cursor, slot);
  hipLaunchKernelGGL(k_cell_sort, dim3((cells + 255) / 256), dim3(256), 0, st, cells, start, slot);
  hipLaunchKernelGGL(k_voronoi, dim3((nn + kVorW - 1) / kVorW), dim3(64 * kVorW), 0, st, x, y, nn,
                     g, start, slot, hullf, Rb, z, psi6);
  return hip_status(hipGetLastError());
}

int radial_histogram(const double* x, const double* y, int64_t n, int32_t nbins, int32_t* counts,
                     void* stream) {
  if (!x || !y || !counts || n < 1 || n > (1 << 26) || nbins < 1 || nbins > (1 << 20))
    return CD_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  hipLaunchKernelGGL(k_fill_int, dim3((nbins + 255) / 256), dim3(256), 0, st, counts, nbins, 0);
  if (nbins <= kRadLds) {
    const unsigned wg = (unsigned)std::min<int64_t>((n + kRadT - 1) / kRadT, 256);
    hipLaunchKernelGGL(k_radial<true>, dim3(wg), dim3(kRadT), sizeof(int32_t) * nbins, st, x, y,
                       (int)n, nbins, counts);
  } else {
    // workgroups of 256: the adds to memory overlap better (9000 bins and a
    // lattice of 1e5 charges 38 us, 44 with workgroups of 1024)
    hipLaunchKernelGGL(k_radial<false>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, x, y,
                       (int)n, nbins, counts);
  }
  return hip_status(hipGetLastError());
}

int structure_stats(const int32_t* z, const double* psi6, int64_t n, double* out, void* stream) {
  if (!z || !out || n < 1 || n > (1 << 26)) return CD_ERR_INVALID_ARG;
  hipLaunchKernelGGL(k_structure_stats, dim3(1), dim3(kScanT), 0, (hipStream_t)stream, z, psi6,
                     (int)n, out);
  return hip_status(hipGetLastError());
}

}  // extern "C"
