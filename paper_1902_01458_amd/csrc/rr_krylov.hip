// LU-free solves of the shifted systems M(omega) X = B and M^H X = B: the
// paper notes (Section 3.2, after Fig. 7) that BiCGStab or GMRES with an
// incomplete-LU or Jacobi preconditioner can stand in for the direct solves;
// that is what lets Algorithm 1 run where the LU no longer fits in
// memory.  Everything here is FP64 and batched: every (shift, column) pair is
// its own linear system, M is applied from the stencil (k_apply).
//
// Preconditioners K ~ M, both built from the 2 x 2 node blocks of M (the two
// velocity components of a grid node couple through the base-flow shear):
//   Jacobi:  K = D = the block diagonal of M.
//   ILU(0):  K = (D + L) D^-1 (D + U) with L, U the strict block triangles of
//            M in natural order (p = j + ny i) and D from the recurrence
//              D_p = M_pp - M_p,p-1 D_p-1^-1 M_p-1,p - M_p,p-ny D_p-ny^-1 M_p-ny,p
//            (block ILU(0): on this stencil the dropped fill is exactly the
//            two cross terms, so L and U keep M's own off-diagonal blocks).
//            Both the recurrence and the triangular sweeps of K^-1 depend on
//            the previous anti-diagonal of the grid only (p - 1 and p - ny lie
//            on i + j - 1), so one workgroup walks the nx + ny - 1
//            anti-diagonals of a system with the previous one in LDS.
// Off-diagonal blocks of M are diagonal 2 x 2 (each component couples to the
// same component of a neighbour), with entries -c from the stencil row.
#include "rr_internal.h"

#include <type_traits>

namespace rr {

namespace {

constexpr int kKChunk = 1024;  // rows per partial sum of the batched dot products
constexpr int kKThreads = 256;

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cmulc(double2 a, double2 b) {  // conj(a) b
  return make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}
__device__ __forceinline__ double2 cscale(double s, double2 a) { return make_double2(s * a.x, s * a.y); }
__device__ __forceinline__ double2 cdiv(double2 a, double2 b) {
  const double d = b.x * b.x + b.y * b.y;
  return make_double2((a.x * b.x + a.y * b.y) / d, (a.y * b.x - a.x * b.y) / d);
}

// 2 x 2 complex matrix, row-major: m[0] m[1] / m[2] m[3]
struct C2 {
  double2 m[4];
};

__device__ __forceinline__ bool inv2(const C2& A, C2& X) {
  const double2 det = csub(cmul(A.m[0], A.m[3]), cmul(A.m[1], A.m[2]));
  const double dd = det.x * det.x + det.y * det.y;
  if (!(dd > 0.0) || !isfinite(dd)) return false;
  const double2 id = make_double2(det.x / dd, -det.y / dd);
  X.m[0] = cmul(A.m[3], id);
  X.m[1] = cmul(make_double2(-A.m[1].x, -A.m[1].y), id);
  X.m[2] = cmul(make_double2(-A.m[2].x, -A.m[2].y), id);
  X.m[3] = cmul(A.m[0], id);
  return true;
}

// y = A x (or A^H x) for a 2-vector x = (x0, x1)
__device__ __forceinline__ void mv2(const C2& A, bool herm, double2 x0, double2 x1, double2& y0,
                                    double2& y1) {
  if (!herm) {
    y0 = cadd(cmul(A.m[0], x0), cmul(A.m[1], x1));
    y1 = cadd(cmul(A.m[2], x0), cmul(A.m[3], x1));
  } else {
    y0 = cadd(cmulc(A.m[0], x0), cmulc(A.m[2], x1));
    y1 = cadd(cmulc(A.m[1], x0), cmulc(A.m[3], x1));
  }
}

// The node block M_pp = i omega I - L_pp of shift (om_r, om_i) from the
// stencil row c (12 coefficients: u row c[0..5], v row c[6..11]).
__device__ __forceinline__ C2 node_block(const double* c, double om_r, double om_i) {
  C2 A;
  A.m[0] = make_double2(-om_i - c[0], om_r);
  A.m[1] = make_double2(-c[5], 0.0);
  A.m[2] = make_double2(-c[11], 0.0);
  A.m[3] = make_double2(-om_i - c[6], om_r);
  return A;
}

__device__ __forceinline__ C2 load_c2(const double2* p) {
  C2 A;
#pragma unroll
  for (int e = 0; e < 4; e++) A.m[e] = p[e];
  return A;
}
__device__ __forceinline__ void store_c2(double2* p, const C2& A) {
#pragma unroll
  for (int e = 0; e < 4; e++) p[e] = A.m[e];
}

// Jacobi: Dinv[w][p] = M_pp^-1 for every node and shift.
__global__ void k_pc_jacobi(int nn, const double* __restrict__ coef,
                            const double* __restrict__ omega, double2* __restrict__ Dinv,
                            uint32_t* status) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x, w = blockIdx.y;
  if (p >= nn) return;
  C2 A = node_block(coef + 12 * (int64_t)p, omega[2 * w], omega[2 * w + 1]), X;
  if (!inv2(A, X)) {
    latch(status, ST_SINGULAR);
    X.m[0] = X.m[3] = make_double2(1, 0);
    X.m[1] = X.m[2] = make_double2(0, 0);
  }
  store_c2(Dinv + ((int64_t)w * nn + p) * 4, X);
}

// Block ILU(0) data of a shift, stored by anti-diagonal: slot (d, j) = d ny +
// j holds node (i, j) = (d - j, j) (slots with i outside 0 .. nx-1 hold the zeros
// that the handle's creation put there: filling them at each setup took as long
// again as the recurrence where ny is well past nx),
// as kIluFields arrays of slots double2 (structure of arrays), so that the
// sweeps, whose threads take consecutive j on one anti-diagonal, read
// consecutive words:
//   0-3   D_p^-1 (row-major 2 x 2)
//   4, 5  forward, K:   (c4, c10) of p, (c2, c8) of p      (blocks to p-1, p-ny)
//   6, 7  forward, K^H: (c3, c9) of p-1, (c1, c7) of p-ny
//   8, 9  backward, K:  (c3, c9) of p, (c1, c7) of p
//   10,11 backward, K^H:(c4, c10) of p+1, (c2, c8) of p+ny
// (the stencil coefficients themselves; the blocks are minus them, and
// neighbours outside the grid hold zeros, whatever the caller's array has
// there: the column sweep multiplies them by the zeros of missing nodes).  In the natural node order every
// operand load of a sweep step touches one cache line per thread, which
// bounds the sweep (measured: 10 ms per apply at 1024 x 512 against 3.9 ms
// with the operands read coalesced).
constexpr int kIluFields = 12;
__host__ __device__ inline int64_t ilu_slots(int nx, int ny) { return (int64_t)(nx + ny - 1) * ny; }

// Block ILU(0) of one shift per workgroup: D_p by the recurrence in the
// header, anti-diagonal by anti-diagonal (d = i + j), the previous
// anti-diagonal's D^-1 in LDS indexed by j.  Stores D^-1 and the
// coefficient pairs in the anti-diagonal layout above.
__global__ __launch_bounds__(kKThreads) void k_pc_ilu0(int nx, int ny,
                                                       const double* __restrict__ coef,
                                                       const double* __restrict__ omega,
                                                       double2* __restrict__ Dinv,
                                                       uint32_t* status) {
  extern __shared__ __align__(16) char kl_smem[];
  C2* ring = reinterpret_cast<C2*>(kl_smem);  // [2][ny]
  const int w = blockIdx.x;
  const double om_r = omega[2 * w], om_i = omega[2 * w + 1];
  const int64_t ns = ilu_slots(nx, ny);
  double2* Fw = Dinv + (int64_t)w * kIluFields * ns;
  for (int d = 0; d < nx + ny - 1; d++) {
    C2* cur = ring + (d & 1) * ny;
    const C2* prev = ring + ((d + 1) & 1) * ny;
    const int j0 = max(0, d - nx + 1), j1 = min(ny - 1, d);
    for (int j = j0 + threadIdx.x; j <= j1; j += blockDim.x) {
      const int i = d - j, p = j + ny * i;
      double c[12];  // (loaded at once, also where a border's masks drop some)
#pragma unroll
      for (int e = 0; e < 12; e++) c[e] = coef[12 * (int64_t)p + e];
      C2 D = node_block(c, om_r, om_i);
      if (j > 0) {  // - M_p,p-1 D_p-1^-1 M_p-1,p: diag(-c4, -c10) E diag(-c3', -c9')
        const double* cq = coef + 12 * (int64_t)(p - 1);
        const C2& E = prev[j - 1];
        const double a[2] = {-c[4], -c[10]}, b[2] = {-cq[3], -cq[9]};
#pragma unroll
        for (int r = 0; r < 2; r++)
#pragma unroll
          for (int s = 0; s < 2; s++) D.m[2 * r + s] = csub(D.m[2 * r + s], cscale(a[r] * b[s], E.m[2 * r + s]));
      }
      if (i > 0) {  // - M_p,p-ny D_p-ny^-1 M_p-ny,p: diag(-c2, -c8) E diag(-c1', -c7')
        const double* cq = coef + 12 * (int64_t)(p - ny);
        const C2& E = prev[j];
        const double a[2] = {-c[2], -c[8]}, b[2] = {-cq[1], -cq[7]};
#pragma unroll
        for (int r = 0; r < 2; r++)
#pragma unroll
          for (int s = 0; s < 2; s++) D.m[2 * r + s] = csub(D.m[2 * r + s], cscale(a[r] * b[s], E.m[2 * r + s]));
      }
      C2 X;
      if (!inv2(D, X)) {
        latch(status, ST_SINGULAR);
        X.m[0] = X.m[3] = make_double2(1, 0);
        X.m[1] = X.m[2] = make_double2(0, 0);
      }
      cur[j] = X;
      const int64_t sl = (int64_t)d * ny + j;
#pragma unroll
      for (int e = 0; e < 4; e++) Fw[e * ns + sl] = X.m[e];
      const double* cl = coef + 12 * (int64_t)(j > 0 ? p - 1 : p);
      const double* cu = coef + 12 * (int64_t)(i > 0 ? p - ny : p);
      const double* cr = coef + 12 * (int64_t)(j < ny - 1 ? p + 1 : p);
      const double* cd = coef + 12 * (int64_t)(i < nx - 1 ? p + ny : p);
      const bool hl = j > 0, hu = i > 0, hr = j < ny - 1, hd = i < nx - 1;
      Fw[4 * ns + sl] = hl ? make_double2(c[4], c[10]) : make_double2(0, 0);
      Fw[5 * ns + sl] = hu ? make_double2(c[2], c[8]) : make_double2(0, 0);
      Fw[6 * ns + sl] = hl ? make_double2(cl[3], cl[9]) : make_double2(0, 0);
      Fw[7 * ns + sl] = hu ? make_double2(cu[1], cu[7]) : make_double2(0, 0);
      Fw[8 * ns + sl] = hr ? make_double2(c[3], c[9]) : make_double2(0, 0);
      Fw[9 * ns + sl] = hd ? make_double2(c[1], c[7]) : make_double2(0, 0);
      Fw[10 * ns + sl] = hr ? make_double2(cr[4], cr[10]) : make_double2(0, 0);
      Fw[11 * ns + sl] = hd ? make_double2(cd[2], cd[8]) : make_double2(0, 0);
    }
    __syncthreads();
  }
}

// Sums of s0, s1 over the workgroup's waves, left in red (two per wave).
__device__ __forceinline__ void block_pair_sum(double2 s0, double2 s1, double2* red) {
  for (int o = 32; o > 0; o >>= 1) {
    s0.x += __shfl_down(s0.x, o, 64);
    s0.y += __shfl_down(s0.y, o, 64);
    s1.x += __shfl_down(s1.x, o, 64);
    s1.y += __shfl_down(s1.y, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[2 * (threadIdx.x >> 6)] = s0;
    red[2 * (threadIdx.x >> 6) + 1] = s1;
  }
  __syncthreads();
}

// Thread e < 2: the workgroup's sum of s_e, after block_pair_sum.
__device__ __forceinline__ double2 pair_total(const double2* red) {
  double2 t = make_double2(0, 0);
  for (int v = 0; v < (int)(blockDim.x >> 6); v++) t = cadd(t, red[2 * v + threadIdx.x]);
  return t;
}

// The sum over a system's partial sums (pairs of complex) by the whole
// workgroup, the same for every thread and in every workgroup of that size.
// red: two complex per wave.
__device__ __forceinline__ void dot_totals(const double2* part, int64_t q, int nparts,
                                           double2* red, double2& t0, double2& t1) {
  double2 s0 = make_double2(0, 0), s1 = make_double2(0, 0);
  for (int ch = threadIdx.x; ch < nparts; ch += blockDim.x) {
    s0 = cadd(s0, part[(q * nparts + ch) * 2]);
    s1 = cadd(s1, part[(q * nparts + ch) * 2 + 1]);
  }
  block_pair_sum(s0, s1, red);
  t0 = t1 = make_double2(0, 0);
  for (int v = 0; v < (int)(blockDim.x >> 6); v++) {
    t0 = cadd(t0, red[2 * v]);
    t1 = cadd(t1, red[2 * v + 1]);
  }
}

// Per-system BiCGStab scalars: rho of the iterations of either parity (a
// kernel that writes one reads the other), alpha, omega.
enum { KS_RHO = 0, KS_ALPHA = 2, KS_OMEGA = 3, KS_N = 4 };

// The vector update in front of a preconditioner apply, and where its scalars
// come from: BICG_P  p <- r + beta (p - omega v),  BICG_S  r <- r - alpha v.
enum { BICG_NONE = 0, BICG_P = 1, BICG_S = 2 };

// A system has ended: the last one to end marks the solve converged, and the
// launches after this one do nothing.
__device__ __forceinline__ void system_ends(const BicgStep& b, int64_t q, uint32_t why) {
  if (why) latch(b.status, why);
  b.active[q] = 0;
  if (atomicSub(b.live, 1u) == 1u) *b.conv = 1u;
}

// The scalar step in front of that update, taken by every workgroup of system
// q from the dot products' partial sums (the owner alone stores): false when
// the system has ended.  c0, c1: beta and omega, or alpha.
//   BICG_P (from the second iteration on) partials <r, r>, <rhat, r>:
//          ||r||^2 <= tol^2 ||b||^2 ends the system; rho, beta
//   BICG_S partials <rhat, v>: alpha = rho / <rhat, v>
// A zero denominator in a live system latches ST_BREAKDOWN and ends it.
template <int MODE>
__device__ __forceinline__ bool bicg_step(const BicgStep& b, int64_t q, bool owner, double2* red,
                                          double2& c0, double2& c1) {
  double2 t0, t1;
  dot_totals((const double2*)b.part, q, b.nparts, red, t0, t1);
  double2* s = (double2*)b.ks + q * KS_N;
  owner = owner && threadIdx.x == 0;
  if (MODE == BICG_P) {
    const bool finite = isfinite(t0.x), done = t0.x <= b.tol2 * b.bnorm2[q];
    const bool broken = t1.x == 0.0 && t1.y == 0.0;
    if (!finite || done || broken) {
      if (owner) system_ends(b, q, !finite ? ST_NONFINITE : done ? 0u : ST_BREAKDOWN);
      return false;
    }
    c1 = s[KS_OMEGA];
    c0 = cmul(cdiv(t1, s[KS_RHO + ((b.it + 1) & 1)]), cdiv(s[KS_ALPHA], c1));
    if (owner) s[KS_RHO + (b.it & 1)] = t1;
  } else {
    if (t0.x == 0.0 && t0.y == 0.0) {
      if (owner) system_ends(b, q, ST_BREAKDOWN);
      return false;
    }
    c0 = cdiv(s[KS_RHO + (b.it & 1)], t0);
    if (owner) s[KS_ALPHA] = c0;
  }
  return true;
}

// Whether system q still runs, the same for every thread of the workgroup.
// Where several workgroups take a system's step, its owner may end the system
// and with it the solve while they start: their waves then see either state,
// and no thread may leave before the vote, as the step has barriers.  A
// workgroup that goes on comes to the owner's decision, from the same sums.
__device__ __forceinline__ bool system_runs(const BicgStep& b, int64_t q) {
  const bool done = __hip_atomic_load(b.conv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return __syncthreads_or(!done && b.active[q] != 0);
}

// r, p, v of one unknown to the updated vector's value
template <int MODE>
__device__ __forceinline__ double2 bicg_update(double2 r, double2 p, double2 v, double2 c0,
                                               double2 c1) {
  if (MODE == BICG_P) return cadd(r, cmul(c0, csub(p, cmul(c1, v))));
  return csub(r, cmul(c0, v));
}

// The update alone, for the sweeps of long lines, whose loads are not coalesced.
template <int MODE>
__global__ __launch_bounds__(kKThreads) void k_bicg_update(int64_t n, int k, double2* X,
                                                           BicgStep b) {
  __shared__ double2 red[2 * kKThreads / 64];
  const int64_t q = (int64_t)blockIdx.z * k + blockIdx.y;
  double2 c0, c1;
  if (!system_runs(b, q)) return;
  if (!bicg_step<MODE>(b, q, blockIdx.x == 0, red, c0, c1)) return;
  const int64_t e0 = (int64_t)blockIdx.x * kKChunk;
  const int rows = (int)min((int64_t)kKChunk, n - e0);
  for (int e = threadIdx.x; e < rows; e += kKThreads) {
    const int64_t o = q * n + e0 + e;
    const double2 x = X[o], v = ((const double2*)b.v)[o];
    X[o] = bicg_update<MODE>(MODE == BICG_P ? ((const double2*)b.r)[o] : x, x, v, c0, c1);
  }
}

// Y = K^-1 X (or K^-H X) with K = D (Jacobi), for every (shift, column).
// MODE: X is the vector of b's update, made here.
template <int MODE>
__global__ __launch_bounds__(256) void k_pc_jacobi_apply(int nn, int k, int adjoint,
                                                         const double2* __restrict__ Dinv,
                                                         double2* X, double2* Y,
                                                         const uint32_t* active,
                                                         const uint32_t* skip, BicgStep b) {
  __shared__ double2 red[8];
  const int p = blockIdx.x * blockDim.x + threadIdx.x, c = blockIdx.y, w = blockIdx.z;
  const int64_t q = (int64_t)w * k + c;
  double2 c0, c1;
  if (MODE == BICG_NONE) {
    if (skip && __hip_atomic_load(skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    if (active && !active[q]) return;
  } else {
    if (!system_runs(b, q)) return;
    if (!bicg_step<MODE>(b, q, blockIdx.x == 0, red, c0, c1)) return;
  }
  if (p >= nn) return;
  const int64_t off = q * 2 * nn + 2 * (int64_t)p;
  const C2 E = load_c2(Dinv + ((int64_t)w * nn + p) * 4);
  double2 x[2], y0, y1;
#pragma unroll
  for (int e = 0; e < 2; e++) {
    x[e] = X[off + e];
    if (MODE == BICG_NONE) continue;
    const double2* v = (const double2*)b.v + off;
    x[e] = MODE == BICG_P ? bicg_update<MODE>(((const double2*)b.r)[off + e], x[e], v[e], c0, c1)
                          : bicg_update<MODE>(x[e], x[e], v[e], c0, c1);
    X[off + e] = x[e];
  }
  mv2(E, adjoint != 0, x[0], x[1], y0, y1);
  Y[off] = y0;
  Y[off + 1] = y1;
}

// Y = K^-1 X (or K^-H X) with the block ILU(0) K, one workgroup per
// (column, shift): the block-lower sweep by ascending anti-diagonals, then the
// block-upper one by descending ones, each node reading its two neighbours of
// the previous anti-diagonal from LDS.  Y may alias X.
//   forward  w_p = D_p^-1 (x_p - M_p,p-1 w_p-1 - M_p,p-ny w_p-ny)
//   backward y_p = w_p - D_p^-1 (M_p,p+1 y_p+1 + M_p,p+ny y_p+ny)
// and for K^H = (D + U)^H D^-H (D + L)^H:
//   forward  w_p = D_p^-H (x_p - M_p-1,p w_p-1 - M_p-ny,p w_p-ny)
//   backward y_p = w_p - D_p^-H (M_p+1,p y_p+1 + M_p+ny,p y_p+ny)
// (the off-diagonal blocks are real and diagonal, so ^H leaves them as they are).
__global__ __launch_bounds__(kKThreads) void k_pc_ilu0_apply(int nx, int ny, int k, int adjoint,
                                                             const double2* __restrict__ Dinv,
                                                             const double2* X, double2* Y,
                                                             const uint32_t* active,
                                                             const uint32_t* skip) {
  if (skip && __hip_atomic_load(skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
  extern __shared__ __align__(16) char ka_smem[];
  double2* ring = reinterpret_cast<double2*>(ka_smem);  // [2][ny][2]
  const int c = blockIdx.x, w = blockIdx.y, nn = nx * ny;
  const int64_t q = (int64_t)w * k + c;
  if (active && !active[q]) return;
  const int64_t off = q * 2 * nn;
  const double2* x = X + off;
  double2* y = Y + off;
  const int64_t ns = ilu_slots(nx, ny);
  const double2* Fw = Dinv + (int64_t)w * kIluFields * ns;
  const bool herm = adjoint != 0;
  const int nd = nx + ny - 1;
  auto dblock = [&](int64_t sl) {
    C2 D;
#pragma unroll
    for (int e = 0; e < 4; e++) D.m[e] = Fw[e * ns + sl];
    return D;
  };
  for (int d = 0; d < nd; d++) {
    double2* cur = ring + (d & 1) * 2 * ny;
    const double2* prev = ring + ((d + 1) & 1) * 2 * ny;
    const int j0 = max(0, d - nx + 1), j1 = min(ny - 1, d);
    for (int j = j0 + threadIdx.x; j <= j1; j += blockDim.x) {
      const int i = d - j, p = j + ny * i;
      const int64_t sl = (int64_t)d * ny + j;
      double2 r0 = x[2 * p], r1 = x[2 * p + 1];
      if (j > 0) {
        const double2 a = Fw[(herm ? 6 : 4) * ns + sl];
        r0 = csub(r0, cscale(-a.x, prev[2 * (j - 1)]));
        r1 = csub(r1, cscale(-a.y, prev[2 * (j - 1) + 1]));
      }
      if (i > 0) {
        const double2 a = Fw[(herm ? 7 : 5) * ns + sl];
        r0 = csub(r0, cscale(-a.x, prev[2 * j]));
        r1 = csub(r1, cscale(-a.y, prev[2 * j + 1]));
      }
      double2 w0, w1;
      mv2(dblock(sl), herm, r0, r1, w0, w1);
      cur[2 * j] = w0;
      cur[2 * j + 1] = w1;
      y[2 * p] = w0;
      y[2 * p + 1] = w1;
    }
    __syncthreads();
  }
  for (int d = nd - 1; d >= 0; d--) {
    double2* cur = ring + (d & 1) * 2 * ny;
    const double2* nxt = ring + ((d + 1) & 1) * 2 * ny;
    const int j0 = max(0, d - nx + 1), j1 = min(ny - 1, d);
    for (int j = j0 + threadIdx.x; j <= j1; j += blockDim.x) {
      const int i = d - j, p = j + ny * i;
      const int64_t sl = (int64_t)d * ny + j;
      double2 t0 = make_double2(0, 0), t1 = make_double2(0, 0);
      if (j < ny - 1) {
        const double2 a = Fw[(herm ? 10 : 8) * ns + sl];
        t0 = cadd(t0, cscale(-a.x, nxt[2 * (j + 1)]));
        t1 = cadd(t1, cscale(-a.y, nxt[2 * (j + 1) + 1]));
      }
      if (i < nx - 1) {
        const double2 a = Fw[(herm ? 11 : 9) * ns + sl];
        t0 = cadd(t0, cscale(-a.x, nxt[2 * j]));
        t1 = cadd(t1, cscale(-a.y, nxt[2 * j + 1]));
      }
      double2 u0, u1;
      mv2(dblock(sl), herm, t0, t1, u0, u1);
      const double2 y0 = csub(y[2 * p], u0), y1 = csub(y[2 * p + 1], u1);
      cur[2 * j] = y0;
      cur[2 * j + 1] = y1;
      y[2 * p] = y0;
      y[2 * p + 1] = y1;
    }
    __syncthreads();
  }
}

// The neighbouring lane's value, lane - 1 (UP) or lane + 1; zero past the wave's end.
template <bool UP>
__device__ __forceinline__ double lane_next(double x) {
  constexpr int ctl = UP ? 0x138 : 0x130;  // wave_shr:1, wave_shl:1
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), ctl, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), ctl, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// The same sweeps with one thread per grid column j (ny <= kIluColMax):
// thread j walks its nodes (i, j), i = 0 .. nx-1 (backward: nx-1 .. 0), at
// anti-diagonal steps d = i + j.  Its own previous node, (i-1, j) (backward
// (i+1, j)), stays in registers; the other neighbour, (i, j-1) (backward
// (i, j+1)), comes from the neighbouring lane's previous step, and between
// waves through LDS and a barrier (ONE: a single wave, no barrier).
//
// What bounds it is the chain of nx + ny - 1 steps each way, a step being the
// instructions that one wave issues, so a step is kept short:
//   - It has no branch, mask or clamp.  Threads without a node at a step read
//     zeros (the preconditioner's unused slots hold them, and vector loads past
//     the buffer's bounds give them), so their results are zeros, which stand
//     for the neighbours that a border node lacks; their stores fall past the
//     bounds and are dropped.
//   - Nothing a node needs depends on the sweep, so each thread holds the loads
//     of its next kIluAhead steps in registers (step d: set d mod kIluAhead,
//     the same for every thread), raw (signs applied at use).
//   - The preconditioner's fields are stored by anti-diagonal, but the vectors
//     by grid line, where the nodes of one step are ny - 1 apart: 64 cache lines
//     a wave and load.  So G neighbouring threads load (and store) G neighbours
//     of one grid line at a time, each at most G - 1 steps before it needs its
//     own (after it has it), and keep them for those steps in LDS, in G places
//     a thread that no other touches.
// 128 x 64 nodes, one shift, 10 columns, with BICG_S: 140 us with masks, clamps
// and 64-bit addresses, 145 instructions a step; 93 us now.  Without the update:
// 130 us with branches, LDS neighbours and one step's loads ahead, 88 now; 4
// shifts at 512 x 256: 2.00 -> 1.00 ms; one at 1024 x 512: 7.3 -> 3.8 ms.
constexpr int kIluColMax = 512;
constexpr int kIluAhead = 4;

template <int MODE>
struct IluOp {
  double2 v0, v1;      // x_p (forward) or w_p (backward), of the line's node
  double2 r0, r1;      // BICG_P: r_p
  double2 u0, u1;      // BICG_P, BICG_S: v_p
  double2 a, b;        // minus the blocks to the (i, j -/+ 1), (i -/+ 1, j) neighbours
  C2 D;
};

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x27000);
}
__device__ __forceinline__ double2 buffer_load(__amdgpu_buffer_rsrc_t b, unsigned at, int base) {
  return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(b, (int)at, base, 0));
}
__device__ __forceinline__ void buffer_store(__amdgpu_buffer_rsrc_t b, unsigned at, double2 s0,
                                             double2 s1) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, s0), b, (int)at, 0, 0);
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, s1), b, (int)at + 16, 0, 0);
}

// s + a x, s + a x (conj: s + conj(a) x), fused
__device__ __forceinline__ double2 rfma(double a, double2 x, double2 s) {
  return make_double2(fma(a, x.x, s.x), fma(a, x.y, s.y));
}
template <bool CONJ>
__device__ __forceinline__ double2 cfma(double2 a, double2 x, double2 s) {
  const double ai = CONJ ? -a.y : a.y;
  return make_double2(fma(-ai, x.y, fma(a.x, x.x, s.x)), fma(ai, x.x, fma(a.x, x.y, s.y)));
}

template <int MODE, bool ONE, bool herm, int G>
__global__ __launch_bounds__(ONE ? 64 : kIluColMax) void k_pc_ilu0_apply_col(
    int nx, int ny, int k, const double2* __restrict__ Dinv, double2* X, double2* Y,
    const uint32_t* active, const uint32_t* skip, BicgStep bs) {
  if (skip && __hip_atomic_load(skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
  extern __shared__ __align__(16) char kc_smem[];
  __shared__ double2 red[2 * kIluColMax / 64];
  constexpr int kEdges = kIluColMax / 64 + 2;
  __shared__ double2 edge[2][kEdges][2];  // [.][v + 1]: wave v's last (first) node of a step
  const int j = threadIdx.x, wave = j >> 6, lane = j & 63;
  const int c = blockIdx.x, w = blockIdx.y, nn = nx * ny;
  const int64_t q = (int64_t)w * k + c;
  if (active && !active[q]) return;
  double2 c0, c1;
  if (MODE != BICG_NONE && !bicg_step<MODE>(bs, q, true, red, c0, c1)) return;
  // the places of this thread in LDS, [G][2][64] a wave: arriving, leaving
  constexpr int kPlace = 2 * 64;
  double2* const fin = reinterpret_cast<double2*>(kc_smem) + wave * 2 * G * kPlace + lane;
  double2* const fout = fin + G * kPlace;
  const int64_t off = q * 2 * nn, ns = ilu_slots(nx, ny);
  const double2* Fw = Dinv + (int64_t)w * kIluFields * ns;
  const int jb = j & ~(G - 1), jt = j | (G - 1), nd = nx + ny - 1;
  const unsigned line = 32u * ny;  // bytes of a grid line
  const auto xb = buffer(X + off, 32u * nn), yb = buffer(Y + off, 32u * nn);
  const auto rb = buffer((const double2*)bs.r + (MODE == BICG_P ? off : 0), 32u * nn);
  const auto vb = buffer((const double2*)bs.v + (MODE != BICG_NONE ? off : 0), 32u * nn);
  auto field = [&](int e) { return buffer(Fw + e * ns, (unsigned)(16 * ns)); };
  const __amdgpu_buffer_rsrc_t dinv[4] = {field(0), field(1), field(2), field(3)};
  // byte offsets: of this thread's unknown pair in grid line i, and of its slot
  // in an anti-diagonal; far past every bound for a thread without a column
  const bool col = j < ny;
  auto at = [&](int i) { return col ? 32u * j + line * (unsigned)i : 0xA0000000u + line * i; };
  const unsigned slot = col ? 16u * j : 0xA0000000u;
  if (!ONE) {
    if (j < 4 * kEdges) (&edge[0][0][0])[j] = make_double2(0, 0);
    __syncthreads();
  }
  // (clamped, so that the offset stays in the field: the slots of the first and
  // last anti-diagonal then meet vectors that are zero, or are not stored)
  auto load = [&](int d, unsigned from, IluOp<MODE>& o, __amdgpu_buffer_rsrc_t v,
                  __amdgpu_buffer_rsrc_t fa, __amdgpu_buffer_rsrc_t fb, bool fwd) {
    const int diag = 16 * ny * min(max(d, 0), nd - 1);
    o.v0 = buffer_load(v, from, 0);
    o.v1 = buffer_load(v, from + 16, 0);
    if (fwd && MODE == BICG_P) {
      o.r0 = buffer_load(rb, from, 0);
      o.r1 = buffer_load(rb, from + 16, 0);
    }
    if (fwd && MODE != BICG_NONE) {
      o.u0 = buffer_load(vb, from, 0);
      o.u1 = buffer_load(vb, from + 16, 0);
    }
    o.a = buffer_load(fa, slot, diag);
    o.b = buffer_load(fb, slot, diag);
#pragma unroll
    for (int e = 0; e < 4; e++) o.D.m[e] = buffer_load(dinv[e], slot, diag);
  };
  auto keep = [&](double2* f, int i, double2 s0, double2 s1) {
    f[(i & (G - 1)) * kPlace] = s0;
    f[(i & (G - 1)) * kPlace + 64] = s1;
  };
  auto kept = [&](const double2* f, int i, double2& s0, double2& s1) {
    s0 = f[(i & (G - 1)) * kPlace];
    s1 = f[(i & (G - 1)) * kPlace + 64];
  };
  // (i, j - 1) or, !UP, (i, j + 1) of the step before, whose parity is par
  auto neighbour = [&](auto up, int par, double2 own0, double2 own1, double2& n0, double2& n1) {
    constexpr bool UP = decltype(up)::value;
    n0 = make_double2(lane_next<UP>(own0.x), lane_next<UP>(own0.y));
    n1 = make_double2(lane_next<UP>(own1.x), lane_next<UP>(own1.y));
    if (!ONE) {
      const double2 e0 = edge[par][wave + (UP ? 0 : 2)][0], e1 = edge[par][wave + (UP ? 0 : 2)][1];
      const bool end = lane == (UP ? 0 : 63);
      n0 = make_double2(end ? e0.x : n0.x, end ? e0.y : n0.y);
      n1 = make_double2(end ? e1.x : n1.x, end ? e1.y : n1.y);
    }
  };
  auto publish = [&](int last, int par, double2 own0, double2 own1) {
    if (ONE) return;
    if (lane == last) {
      edge[par][wave + 1][0] = own0;
      edge[par][wave + 1][1] = own1;
    }
    __syncthreads();
  };
  // s + D_p^-1 r (D_p^-H r)
  auto solve2 = [&](const C2& D, double2 r0, double2 r1, double2 s0, double2 s1, double2& y0,
                    double2& y1) {
    y0 = cfma<herm>(D.m[herm ? 2 : 1], r1, cfma<herm>(D.m[0], r0, s0));
    y1 = cfma<herm>(D.m[3], r1, cfma<herm>(D.m[herm ? 1 : 2], r0, s1));
  };
  IluOp<MODE> op[kIluAhead] = {};
  const double2 zero = make_double2(0, 0);
  double2 own0 = zero, own1 = zero;
  double2 now0 = zero, now1 = zero;  // this step's x_p, w_p
  double2 out0 = zero, out1 = zero;  // the line's results, to be stored
#pragma unroll
  for (int g = 0; g < G; g++) keep(fin, g, zero, zero);
  // forward: w_p = D_p^-1 (x_p - M_p,p-1 w_p-1 - M_p,p-ny w_p-ny).  At step d
  // the group's line d + 1 - jb arrives and line d - 1 - jt leaves.
  const int first = -2 * kIluAhead;
  const auto fa = field(herm ? 6 : 4), fb = field(herm ? 7 : 5);
  unsigned arrive = at(first + 1 - jb), leave = at(first - 1 - jt);
  for (int d0 = first; d0 < nd + G; d0 += kIluAhead) {
#pragma unroll
    for (int u = 0; u < kIluAhead; u++) {
      const int d = d0 + u, i = d - j;
      const IluOp<MODE>& use = op[u];
      double2 n0, n1;
      neighbour(std::true_type{}, (d + 1) & 1, own0, own1, n0, n1);
      const double2 r0 = rfma(use.b.x, own0, rfma(use.a.x, n0, now0));
      const double2 r1 = rfma(use.b.y, own1, rfma(use.a.y, n1, now1));
      solve2(use.D, r0, r1, zero, zero, own0, own1);
      double2 v0 = use.v0, v1 = use.v1;
      if (MODE != BICG_NONE) {
        v0 = bicg_update<MODE>(MODE == BICG_P ? use.r0 : v0, v0, use.u0, c0, c1);
        v1 = bicg_update<MODE>(MODE == BICG_P ? use.r1 : v1, v1, use.u1, c0, c1);
        buffer_store(xb, arrive, v0, v1);
      }
      buffer_store(yb, leave, out0, out1);
      keep(fin, d + 1, v0, v1);  // jb is a multiple of G
      keep(fout, i, own0, own1);
      kept(fin, i + 1, now0, now1);
      kept(fout, d + 1, out0, out1);  // jt one less than one
      load(d + kIluAhead, arrive + kIluAhead * line, op[u], xb, fa, fb, true);
      arrive += line;
      leave += line;
      publish(63, d & 1, own0, own1);
      __builtin_amdgcn_sched_barrier(0);  // keeps a step's loads in front of the next step's
    }
  }
  // backward: y_p = w_p - D_p^-1 (M_p,p+1 y_p+1 + M_p,p+ny y_p+ny); the forward
  // results of a thread's column are its own stores.  At step d the group's
  // line d - 1 - jt arrives and line d + 1 - jb leaves.
  own0 = own1 = now0 = now1 = zero;
#pragma unroll
  for (int u = 0; u < kIluAhead; u++) op[u] = IluOp<MODE>{};
#pragma unroll
  for (int g = 0; g < G; g++) keep(fin, g, zero, zero);
  if (!ONE) {
    __syncthreads();
    if (j < 4 * kEdges) (&edge[0][0][0])[j] = zero;
    __syncthreads();
  }
  const int last = nd - 1 + 2 * kIluAhead + G;
  const auto ga = field(herm ? 10 : 8), gb = field(herm ? 11 : 9);
  arrive = at(last - 1 - jt);
  leave = at(last + 1 - jb);
  for (int d0 = last; d0 >= -1; d0 -= kIluAhead) {
#pragma unroll
    for (int u = 0; u < kIluAhead; u++) {
      const int d = d0 - u, i = d - j;
      const IluOp<MODE>& use = op[u];
      double2 n0, n1;
      neighbour(std::false_type{}, (d + 1) & 1, own0, own1, n0, n1);
      const double2 s0 = rfma(use.b.x, own0, rfma(use.a.x, n0, zero));
      const double2 s1 = rfma(use.b.y, own1, rfma(use.a.y, n1, zero));
      solve2(use.D, s0, s1, now0, now1, own0, own1);
      buffer_store(yb, leave, out0, out1);
      keep(fin, d, use.v0, use.v1);
      keep(fout, i, own0, own1);
      kept(fin, i - 1, now0, now1);
      kept(fout, d, out0, out1);
      load(d - kIluAhead, arrive - kIluAhead * line, op[u], yb, ga, gb, false);
      arrive -= line;
      leave -= line;
      publish(0, d & 1, own0, own1);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// partial[(q * nchunk + chunk) * 2] = sum over the chunk of conj(A) B, per
// system q = w * k + c (and zero beside it, the second of the fused kernels' pairs).
__global__ __launch_bounds__(kKThreads) void k_kdot_partial(int64_t n, int k, const double2* A,
                                                           const double2* B, int nchunk,
                                                           double2* partial,
                                                           const uint32_t* active,
                                                           const uint32_t* skip) {
  if (skip && __hip_atomic_load(skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
  __shared__ double2 red[2 * kKThreads / 64];
  const int chunk = blockIdx.x, c = blockIdx.y, w = blockIdx.z;
  const int64_t q = (int64_t)w * k + c;
  if (active && !active[q]) return;
  const int64_t base = q * n, r0 = (int64_t)chunk * kKChunk, r1 = min(n, r0 + kKChunk);
  double2 s0 = make_double2(0, 0);
  for (int64_t r = r0 + threadIdx.x; r < r1; r += kKThreads)
    s0 = cadd(s0, cmulc(A[base + r], B[base + r]));
  block_pair_sum(s0, make_double2(0, 0), red);
  if (threadIdx.x < 2) partial[(q * nchunk + chunk) * 2 + threadIdx.x] = pair_total(red);
}

__device__ __forceinline__ double2 dot_total(const double2* partial, int64_t q, int nchunk, int e) {
  double2 t = make_double2(0, 0);
  for (int ch = 0; ch < nchunk; ch++) t = cadd(t, partial[(q * nchunk + ch) * 2 + e]);
  return t;
}

// The scalar steps at a solve's ends, one thread per system, from the partial
// sums of ||r||^2 (mode):
//   0  start:  bnorm2 = ||b||^2 (a zero right-hand side is solved by x = 0),
//              rho = <rhat, r> = ||b||^2, the number of live systems
//   1  check:  ||r||^2 <= tol^2 ||b||^2 ends the system
// The solve is marked converged when no system is left (later launches then
// skip).
__global__ __launch_bounds__(kKThreads) void k_krylov_scalars(int N, int nparts, int mode,
                                                             double tol2, const double2* partial,
                                                             double2* ks, double* bnorm2,
                                                             uint32_t* active, uint32_t* live_out,
                                                             uint32_t* conv, uint32_t* status,
                                                             const uint32_t* skip) {
  if (skip && __hip_atomic_load(skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
  __shared__ uint32_t live;
  if (threadIdx.x == 0) live = 0;
  __syncthreads();
  uint32_t mine = 0;
  for (int q = threadIdx.x; q < N; q += blockDim.x) {
    if (mode == 0) {
      const double b2 = dot_total(partial, q, nparts, 0).x;
      bnorm2[q] = b2;
      active[q] = b2 > 0.0 ? 1u : 0u;
      ks[(int64_t)q * KS_N + KS_RHO] = make_double2(b2, 0);
      mine += active[q];
      continue;
    }
    if (!active[q]) continue;
    const double r2 = dot_total(partial, q, nparts, 0).x;
    if (!isfinite(r2)) {
      latch(status, ST_NONFINITE);
      active[q] = 0;
      continue;
    }
    if (r2 <= tol2 * bnorm2[q]) active[q] = 0;
    else mine++;
  }
  atomicAdd(&live, mine);
  __syncthreads();
  if (threadIdx.x == 0) {
    if (mode == 0) *live_out = live;
    if (live == 0) *conv = 1u;
  }
}

// omega = <t, s> / <t, t> (0 when t = 0) from b's partial sums, x += alpha y +
// omega z, r <- s - omega t, and the partial sums of <r, r>, <rhat, r> of the
// next iteration's scalars (kKChunk rows a workgroup).
__global__ __launch_bounds__(kKThreads) void k_bicg_xr(int64_t n, int k, const double2* y,
                                                       const double2* z, const double2* t,
                                                       const double2* rh, double2* x, double2* r,
                                                       double2* part_out, const uint32_t* skip,
                                                       BicgStep b) {
  if (skip && __hip_atomic_load(skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
  __shared__ double2 red[2 * kKThreads / 64];
  const int64_t q = (int64_t)blockIdx.z * k + blockIdx.y;
  if (!b.active[q]) return;
  double2 ts, tt;
  dot_totals((const double2*)b.part, q, b.nparts, red, ts, tt);
  __syncthreads();
  double2* s = (double2*)b.ks + q * KS_N;
  const double2 alpha = s[KS_ALPHA];
  const double2 omega = tt.x > 0.0 ? cscale(1.0 / tt.x, ts) : make_double2(0, 0);
  if (blockIdx.x == 0 && threadIdx.x == 0) s[KS_OMEGA] = omega;
  double2 s0 = make_double2(0, 0), s1 = make_double2(0, 0);
  const int64_t r0 = q * n + (int64_t)blockIdx.x * kKChunk;
  const int rows = (int)min((int64_t)kKChunk, n - (int64_t)blockIdx.x * kKChunk);
#pragma unroll
  for (int u = 0; u < kKChunk / kKThreads; u++) {
    const int e = threadIdx.x + u * kKThreads;
    if (e >= rows) break;
    const int64_t o = r0 + e;
    x[o] = cadd(x[o], cadd(cmul(alpha, y[o]), cmul(omega, z[o])));
    const double2 rn = csub(r[o], cmul(omega, t[o]));
    r[o] = rn;
    s0 = cadd(s0, cmulc(rn, rn));
    s1 = cadd(s1, cmulc(rh[o], rn));
  }
  block_pair_sum(s0, s1, red);
  if (threadIdx.x < 2)
    part_out[(q * gridDim.x + blockIdx.x) * 2 + threadIdx.x] = pair_total(red);
}

// x += d for live systems
__global__ void k_kaxpy(int64_t n, int k, const double2* d, double2* x, const uint32_t* active,
                        const uint32_t* skip) {
  if (skip && __hip_atomic_load(skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t q = (int64_t)blockIdx.z * k + blockIdx.y;
  if (e >= n || !active[q]) return;
  x[q * n + e] = cadd(x[q * n + e], d[q * n + e]);
}

__global__ void k_kcopy(int64_t n, const double2* a, double2* b) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e < n) b[e] = a[e];
}

__global__ void k_latch_live(int N, const uint32_t* active, uint32_t* status, uint32_t bit) {
  for (int q = threadIdx.x; q < N; q += blockDim.x)
    if (active[q]) {
      latch(status, bit);
      break;
    }
}

}  // namespace

int krylov_nchunk(int64_t n) { return (int)((n + kKChunk - 1) / kKChunk); }

size_t ilu0_lds(int ny) { return (size_t)2 * ny * sizeof(C2); }
// Bytes of a Krylov handle's preconditioner data (all shifts).
size_t pc_bytes(int precond, int nx, int ny, int n_omega) {
  if (precond == RR_PRECOND_ILU0)
    return (size_t)n_omega * kIluFields * ilu_slots(nx, ny) * sizeof(double2);
  return (size_t)n_omega * nx * ny * 4 * sizeof(double2);
}
size_t ilu0_apply_lds(int ny) { return (size_t)2 * ny * 2 * sizeof(double2); }

size_t ilu0_col_lds(int G, int threads) { return (size_t)4 * G * threads * sizeof(double2); }

template <int MODE, int G>
static hipError_t prepare_ilu0_col(int threads) {
  hipError_t e = hipSuccess;
  for (const void* fn : {(const void*)k_pc_ilu0_apply_col<MODE, false, true, G>,
                         (const void*)k_pc_ilu0_apply_col<MODE, false, false, G>})
    if (e == hipSuccess)
      e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)ilu0_col_lds(G, threads));
  return e;
}
template <int G>
static hipError_t prepare_ilu0_cols(int threads) {
  hipError_t e = prepare_ilu0_col<BICG_NONE, G>(threads);
  if (e == hipSuccess) e = prepare_ilu0_col<BICG_P, G>(threads);
  if (e == hipSuccess) e = prepare_ilu0_col<BICG_S, G>(threads);
  return e;
}

// Allows the LDS that this grid's kernels ask for beyond the default: a kernel's
// first mention loads it, about 0.2 ms each, so only those.
hipError_t prepare_krylov(int precond, int ny) {
  if (precond != RR_PRECOND_ILU0) return hipSuccess;
  hipError_t e = hipFuncSetAttribute((const void*)k_pc_ilu0,
                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)ilu0_lds(ny));
  if (e == hipSuccess)
    e = hipFuncSetAttribute((const void*)k_pc_ilu0_apply,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)ilu0_apply_lds(ny));
  if (e == hipSuccess && ny > 64 && ny <= 256) e = prepare_ilu0_cols<8>(256);
  if (e == hipSuccess && ny > 256 && ny <= kIluColMax) e = prepare_ilu0_cols<4>(kIluColMax);
  return e;
}

hipError_t launch_pc_setup(const OpDesc& op, int precond, const double* omega, int n_omega,
                           double* Dinv, uint32_t* status, hipStream_t s) {
  const int nn = op.nx * op.ny;
  if (precond == RR_PRECOND_ILU0)
    hipLaunchKernelGGL(k_pc_ilu0, dim3(n_omega), dim3(kKThreads), ilu0_lds(op.ny), s, op.nx,
                       op.ny, op.coef, omega, (double2*)Dinv, status);
  else
    hipLaunchKernelGGL(k_pc_jacobi, dim3((nn + 255) / 256, n_omega), dim3(256), 0, s, nn,
                       op.coef, omega, (double2*)Dinv, status);
  return hipGetLastError();
}

// K^-1 of X (b: X is first updated as MODE says)
template <int MODE>
static hipError_t pc_apply_run(const OpDesc& op, int precond, int n_omega, int k, int adjoint,
                               const double* Dinv, double* X, double* Y, const uint32_t* active,
                               const uint32_t* skip, const BicgStep& b, hipStream_t s) {
  const int nn = op.nx * op.ny;
  const double2* D = (const double2*)Dinv;
  double2 *x = (double2*)X, *y = (double2*)Y;
  if (precond == RR_PRECOND_ILU0 && op.ny <= kIluColMax && op.n <= (1 << 26)) {
    const int threads = (op.ny + 63) / 64 * 64;
    // G = 8 while its places fit in LDS (128 KiB for 256 threads; 4 for 512)
    const int G = threads <= 256 ? 8 : 4;
    auto* kernel = threads == 64
                       ? (adjoint ? k_pc_ilu0_apply_col<MODE, true, true, 8>
                                  : k_pc_ilu0_apply_col<MODE, true, false, 8>)
                   : G == 8 ? (adjoint ? k_pc_ilu0_apply_col<MODE, false, true, 8>
                                       : k_pc_ilu0_apply_col<MODE, false, false, 8>)
                            : (adjoint ? k_pc_ilu0_apply_col<MODE, false, true, 4>
                                       : k_pc_ilu0_apply_col<MODE, false, false, 4>);
    hipLaunchKernelGGL(kernel, dim3(k, n_omega), dim3(threads), ilu0_col_lds(G, threads), s, op.nx,
                       op.ny, k, D, x, y, active, skip, b);
  } else if (precond == RR_PRECOND_ILU0) {
    if constexpr (MODE != BICG_NONE)
      hipLaunchKernelGGL(k_bicg_update<MODE>, dim3(krylov_nchunk(op.n), k, n_omega),
                         dim3(kKThreads), 0, s, op.n, k, x, b);
    hipLaunchKernelGGL(k_pc_ilu0_apply, dim3(k, n_omega), dim3(kKThreads), ilu0_apply_lds(op.ny),
                       s, op.nx, op.ny, k, adjoint, D, x, y, active, skip);
  } else
    hipLaunchKernelGGL(k_pc_jacobi_apply<MODE>, dim3((nn + 255) / 256, k, n_omega), dim3(256), 0,
                       s, nn, k, adjoint, D, x, y, active, skip, b);
  return hipGetLastError();
}

hipError_t launch_pc_apply(const OpDesc& op, int precond, int n_omega, int k, int adjoint,
                           const double* Dinv, const double* X, double* Y,
                           const uint32_t* active, const uint32_t* skip, hipStream_t s) {
  return pc_apply_run<BICG_NONE>(op, precond, n_omega, k, adjoint, Dinv, (double*)X, Y, active,
                                 skip, BicgStep{}, s);
}

hipError_t launch_bicg_p(const OpDesc& op, int precond, int n_omega, int k, int adjoint,
                         const double* Dinv, double* p, double* y, const BicgStep& b,
                         hipStream_t s) {
  return pc_apply_run<BICG_P>(op, precond, n_omega, k, adjoint, Dinv, p, y, b.active, b.conv, b, s);
}
hipError_t launch_bicg_s(const OpDesc& op, int precond, int n_omega, int k, int adjoint,
                         const double* Dinv, double* r, double* z, const BicgStep& b,
                         hipStream_t s) {
  return pc_apply_run<BICG_S>(op, precond, n_omega, k, adjoint, Dinv, r, z, b.active, b.conv, b, s);
}
hipError_t launch_bicg_xr(int64_t n, int n_omega, int k, const double* y, const double* z,
                          const double* t, const double* rh, double* x, double* r,
                          double* part_out, const BicgStep& b, hipStream_t s) {
  hipLaunchKernelGGL(k_bicg_xr, dim3(krylov_nchunk(n), k, n_omega), dim3(kKThreads), 0, s, n, k,
                     (const double2*)y, (const double2*)z, (const double2*)t, (const double2*)rh,
                     (double2*)x, (double2*)r, (double2*)part_out, b.conv, b);
  return hipGetLastError();
}

hipError_t launch_kdot(int64_t n, int n_omega, int k, const double* A, const double* B,
                       double* partial, const uint32_t* active, const uint32_t* skip,
                       hipStream_t s) {
  const int nc = krylov_nchunk(n);
  hipLaunchKernelGGL(k_kdot_partial, dim3(nc, k, n_omega), dim3(kKThreads), 0, s, n, k,
                     (const double2*)A, (const double2*)B, nc, (double2*)partial, active, skip);
  return hipGetLastError();
}

hipError_t launch_krylov_scalars(int N, int64_t n, int mode, double tol, const double* partial,
                                 double* ks, double* bnorm2, uint32_t* active, uint32_t* live,
                                 uint32_t* conv, uint32_t* status, const uint32_t* skip,
                                 hipStream_t s) {
  hipLaunchKernelGGL(k_krylov_scalars, dim3(1), dim3(kKThreads), 0, s, N, krylov_nchunk(n), mode,
                     tol * tol, (const double2*)partial, (double2*)ks, bnorm2, active, live, conv,
                     status, skip);
  return hipGetLastError();
}

hipError_t launch_kaxpy(int64_t n, int n_omega, int k, const double* d, double* x,
                        const uint32_t* active, const uint32_t* skip, hipStream_t s) {
  hipLaunchKernelGGL(k_kaxpy, dim3((unsigned)((n + 255) / 256), k, n_omega), dim3(256), 0, s, n, k,
                     (const double2*)d, (double2*)x, active, skip);
  return hipGetLastError();
}

hipError_t launch_kcopy(int64_t count, const double* a, double* b, hipStream_t s) {
  hipLaunchKernelGGL(k_kcopy, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, count,
                     (const double2*)a, (double2*)b);
  return hipGetLastError();
}

hipError_t launch_latch_live(int N, const uint32_t* active, uint32_t* status, uint32_t bit,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_latch_live, dim3(1), dim3(256), 0, s, N, active, status, bit);
  return hipGetLastError();
}

}  // namespace rr
