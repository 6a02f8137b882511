// Sparse LU of M(omega) in nested-dissection order, batched over shifts, and
// its solves (Section 3.1: one factorisation serves every solve).
//
// Every front (rr_ndplan.hip) is a dense block matrix over its p separator
// unknowns (1) and its q border unknowns (2),
//   F = [ F11 F12 ]   F11, F12, F21: the stencil's entries plus the halves'
//       [ F21 F22 ]   Schur complements; F22: the halves' alone
// and keeps A = F11^-1, B12 = A F12 and F21; S = F22 - F21 B12 goes to the
// front above.  No pivoting.  Solves take products only:
//   forward  up:  z = A b1,  u = (halves' u) - F21 z;     down: x1 = z - B12 x2
//   adjoint  up:  z = b1,    u = (halves' u) - B12^H z;   down: x1 = A^H (z - F21^H x2)
// with b1 the right-hand side plus the halves' updates u at the separator.
// A leaf (a block of grid nodes, no halves) keeps A alone: each of its border
// unknowns has one neighbour in it, so F12 and F21 have one real entry per
// border unknown, S = -F21 A F12 takes no product, and its sweeps apply F12 and
// F21 entry by entry (up z = A b, u = -F21 z, or z = A^H b, u = -F12^H z; down
// x = A (b - F12 x2) or A^H (b - F21^H x2)), straight from and to the caller's
// blocks.
//
// A and F21 are stored column-major and B12 row-major, so that every product
// of the factorisation and of the sweeps up reads 16 consecutive elements of
// either operand per MFMA row, and the sweeps down read 4 consecutive ones
// per lane.
//
// Schur complements and updates are pulled by the front above through the
// border tables (each border unknown belongs to at most one half), so nothing
// is zeroed, scattered or added atomically and every result is bitwise
// repeatable.
//
// Against the band LU in the natural order (half-band 2 ny): at 512 x 256 a
// shift takes 5.8e10 real flops and 4.1e7 factor entries instead of 5.5e11 and
// 2.7e8, and the longest chain of dependent eliminations is about 2.5e3
// unknowns (the separators on one path of the tree) instead of 262144.
#include <algorithm>
#include <type_traits>

#include "rr_mfma.h"

namespace rr {
namespace {

typedef cplx<double> zc;

template <typename R>
struct CAcc {
  typename Mf<R>::v4 re, im;
};
template <typename R>
__device__ __forceinline__ void zero(CAcc<R>& a) {
  a.re = typename Mf<R>::v4{0, 0, 0, 0};
  a.im = typename Mf<R>::v4{0, 0, 0, 0};
}

template <typename R>
__device__ __forceinline__ cplx<R> narrow(zc v) {
  return cplx<R>{(R)v.re, (R)v.im};
}
// An inverse's element as it is kept; one that FP32 does not hold counts as a
// bad pivot.
template <typename R>
__device__ __forceinline__ cplx<R> kept(zc v, bool& bad) {
  const cplx<R> k = narrow<R>(v);
  if constexpr (sizeof(R) < sizeof(double)) bad |= !(isfinite(k.re) && isfinite(k.im));
  return k;
}

// M(omega) between unknowns dr (row) and dc: i omega - L.
template <typename R>
__device__ __forceinline__ cplx<R> entry(const OpDesc& op, double om_r, double om_i, int dr,
                                         int dc) {
  cplx<R> v{(R)0, (R)0};
  const int d = (dc >> 1) - (dr >> 1);
  const bool same = ((dr ^ dc) & 1) == 0;
  if (d != 0 && d != 1 && d != -1 && d != op.ny && d != -op.ny) return v;
  if (d != 0 && !same) return v;
  const double* cf = op.coef + 12 * (int64_t)(dr >> 1) + 6 * (dr & 1);
  double lv = 0.0;
  if (d == 0) lv = same ? cf[0] : cf[5];
  else if (d == op.ny) lv = cf[1];
  else if (d == -op.ny) lv = cf[2];
  else {
    const int j = (dr >> 1) % op.ny;
    if (d == 1 && j < op.ny - 1) lv = cf[3];
    else if (d == -1 && j > 0) lv = cf[4];
  }
  double re = -lv, im = 0.0;
  if (dr == dc) { re -= om_i; im = om_r; }
  v.re = (R)re;
  v.im = (R)im;
  return v;
}

template <typename R>
__device__ __forceinline__ void add(cplx<R>& a, cplx<R> b) {
  a.re += b.re;
  a.im += b.im;
}

// ---------------------------------------------------------------------------
// Inverse of a T x T tile in LDS (T a multiple of 16, at most 64), column
// major with pitch ld, in place: Gauss-Jordan by 16-column blocks.  Per block
// one wave inverts the 16 x 16 pivot block in registers (lane l: row l % 16,
// columns 4 (l / 16) .. + 3; the pivot row comes by DPP row broadcasts); then
// the block row is multiplied by it and the other block rows updated on MFMA,
// a wave per block row.  Bound by its serial chain, so the next pivot block
// is updated and inverted first, by a wave of its own, while the other waves
// update the rest (the pivot row's wave, which has no row to update, takes
// that wave's row).  A zero or non-finite pivot latches ST_SINGULAR and is
// replaced by 1.
//
// In FP64 for FP32 factors too where P <= 64: without pivoting the inverse of a
// leaf's or a small front's block grows now and then, and the FP32 one then loses
// the digits that refinement next to an eigenvalue of L needs.  Over 80 grids at
// 1e-5 |lambda| (emulated), 30 solves missed 1e-10 within six corrections with
// FP32 inverses, 14 of them solves that the band LU finishes; 15 and 4 with FP64
// ones (or pivoted ones: it is the growth).  The band LU misses 28.  The pivot
// tiles of larger fronts are inverted in the factor's type: over 48 grids up to
// 80 x 70 FP64 ones there made no difference (5 misses, 4 without).  The price is
// the FP64 tile's 75 KB of LDS, two workgroups a CU instead of four: 512 x 256, 16
// shifts, FP32, k_nd_leaf 1.69 -> 3.96 ms, 2.87 with narrow leaves apart.
// ---------------------------------------------------------------------------
template <int S>
__device__ __forceinline__ float row_bcast(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + S, 0xf, 0xf, true));
}
template <int S>
__device__ __forceinline__ double row_bcast(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x150 + S, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x150 + S, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
template <int S, typename R>
__device__ __forceinline__ cplx<R> row_bcast(cplx<R> v) {
  return cplx<R>{row_bcast<S>(v.re), row_bcast<S>(v.im)};
}
__device__ __forceinline__ float lane_value(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}
// 1 / x off the division's length, which is on the chain; the division itself
// near the ends of the range
__device__ __forceinline__ double recip(double x) {
  return x > 1e-290 && x < 1e290 ? recip_newton(x) : 1.0 / x;
}
__device__ __forceinline__ float recip(float x) { return 1.0f / x; }

template <typename R, int S>
struct Inv16 {
  static __device__ __forceinline__ void run(cplx<R> (&a)[4], bool& bad) {
    if constexpr (S < 16) {
      constexpr int G = S >> 2, C = S & 3;
      const int l = threadIdx.x & 63, i = l & 15, g = l >> 4;
      const int src = 16 * G + i;
      const cplx<R> f{__shfl(a[C].re, src), __shfl(a[C].im, src)};  // a(i, S)
      cplx<R> d{lane_value(a[C].re, 16 * G + S), lane_value(a[C].im, 16 * G + S)};
      const R mag = d.re * d.re + d.im * d.im;
      R rm = recip(mag);
      if (!(mag > (R)0) || !isfinite(mag)) {
        bad = true;
        d = cplx<R>{(R)1, (R)0};
        rm = (R)1;
      }
      const cplx<R> inv{d.re * rm, -d.im * rm};
      cplx<R> m = cmul(f, inv);
      const bool piv = i == S;
      if (piv) m = cplx<R>{-inv.re, -inv.im};
#pragma unroll
      for (int c = 0; c < 4; c++) {
        const cplx<R> v = row_bcast<S>(a[c]);
        cplx<R> b = a[c];
        if (piv) b = cplx<R>{(R)0, (R)0};
        b.re -= m.re * v.re - m.im * v.im;
        b.im -= m.re * v.im + m.im * v.re;
        a[c] = b;
      }
      if (g == G) a[C] = cplx<R>{-m.re, -m.im};
      Inv16<R, S + 1>::run(a, bad);
    }
  }
};

constexpr int kPv = 17;             // pitch of the 16 x 16 pivot inverses
constexpr int kPvSize = 2 * 16 * kPv;  // two of them, by pivot parity

// (inlined: as a function it would take its LDS operands through generic
// pointers, i.e. flat instead of LDS instructions)
template <typename R>
__device__ __forceinline__ void invert_tile(cplx<R>* F, int ld, int T, cplx<R>* pvs, uint32_t* status) {
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, i = l & 15, g = l >> 4;
  const int nb = T >> 4;
  // invert pivot block kb from LDS into its pv
  auto pivot = [&](int kb) __attribute__((always_inline)) {
    cplx<R> a[4];
#pragma unroll
    for (int c = 0; c < 4; c++) a[c] = F[(16 * kb + 4 * g + c) * ld + 16 * kb + i];
    bool bad = false;
    Inv16<R, 0>::run(a, bad);
    if (bad && l == 0) latch(status, ST_SINGULAR);
#pragma unroll
    for (int c = 0; c < 4; c++) pvs[(kb & 1) * 16 * kPv + i * kPv + 4 * g + c] = a[c];
  };
  auto put = [&](int rb, int j, const CAcc<R>& acc) {
#pragma unroll
    for (int e = 0; e < 4; e++)
      F[(16 * j + i) * ld + 16 * rb + Mf<R>::row(l, e)] = cplx<R>{acc.re[e], acc.im[e]};
  };
  // (one place calls pivot: a second would make it a function, its operands in
  // scratch memory)
  for (int kb = -1;; kb++) {
    const cplx<R>* pv = pvs + (kb & 1) * 16 * kPv;
    const int nx = kb + 1;
    CAcc<R> held;
    int rb = wave;
    bool rows = false;
    if (kb >= 0) {
      if (wave != kb && wave < nb) {  // block row kb: R_j = pv F(kb, j), j = wave
        CAcc<R> acc;
        zero(acc);
        const cplx<R>* col = F + (16 * wave + i) * ld + 16 * kb;
#pragma unroll
        for (int s = 0; s < 4; s++)
          cmfma<R, false, false>(acc.re, acc.im, pv[i * kPv + 4 * s + g], col[4 * s + g]);
        put(kb, wave, acc);
      }
      __syncthreads();
      // block row `rb` of the update: F(rb, j) -= C R_j and, held back until
      // every reader of C = F(rb, kb) is done, F(rb, kb) = -C pv
      if (wave == kb) rb = nx;         // (nx < nb) the next pivot's row, for its wave
      rows = wave < nb && rb < nb && (wave == kb || wave != nx);
      if (wave < nb && (rows || wave == nx)) {
        cplx<R> cf[4];
#pragma unroll
        for (int s = 0; s < 4; s++) cf[s] = F[(16 * kb + 4 * s + g) * ld + 16 * rb + i];
        for (int j = 0; j < nb; j++) {
          if (j == kb || (wave == nx ? j != nx : (rb == nx && j == nx))) continue;
          CAcc<R> acc;
          const cplx<R>* col = F + (16 * j + i) * ld;
#pragma unroll
          for (int e = 0; e < 4; e++) {
            const cplx<R> v = col[16 * rb + Mf<R>::row(l, e)];
            acc.re[e] = v.re;
            acc.im[e] = v.im;
          }
#pragma unroll
          for (int s = 0; s < 4; s++)
            cmfma<R, false, true>(acc.re, acc.im, cf[s], col[16 * kb + 4 * s + g]);
          put(rb, j, acc);
        }
        if (rows) {
          zero(held);
#pragma unroll
          for (int s = 0; s < 4; s++)
            cmfma<R, false, true>(held.re, held.im, cf[s], pv[(4 * s + g) * kPv + i]);
        }
      }
    }
    if (nx < nb && wave == nx) pivot(nx);
    __syncthreads();
    if (kb >= 0) {
      if (rows) put(rb, kb, held);
      if (wave == kb)
#pragma unroll
        for (int c = 0; c < 4; c++)
          F[(16 * kb + 4 * g + c) * ld + 16 * kb + i] = pv[i * kPv + 4 * g + c];
    }
    if (nx >= nb) break;
  }
  __syncthreads();
}

// The task of a workgroup: workgroups are dealt to the eight XCDs in turn, so
// every eighth one takes consecutive tasks.  A front's tiles then share one L2,
// which reads their common operands once: 512 x 256, 16 shifts, FP64, k_nd_schur
// 42 -> 21 GB read, the factor 32.5 -> 32.0 ms; one FP32 shift 3.04 -> 2.88 ms.
__device__ __forceinline__ int xcd_task() {
  const int n = gridDim.x, c = blockIdx.x & 7;
  return c * (n >> 3) + min(c, n & 7) + (blockIdx.x >> 3);
}

// ---------------------------------------------------------------------------
// Factorisation
// ---------------------------------------------------------------------------
template <typename R>
struct FactorArgs {
  OpDesc op;
  const NdFront* fronts;
  const NdTask* tasks;
  const int *pdof, *bmap, *grow;
  const double* omega;
  cplx<R>* factor;
  cplx<R>* schur_in;   // the arena of the halves
  cplx<R>* schur_out;
  cplx<R>* temp;
  int64_t nfactor, nin, nout, ntemp;  // elements per shift
  uint32_t* status;
  int w0;
};

constexpr int kLd = kNdTile + 1;  // pitch of a tile in LDS
template <typename R>
constexpr size_t tile_lds() {
  return (size_t)(kNdTile * kLd + kPvSize) * sizeof(cplx<R>);
}
// A P x P tile with its pivot inverses; k_nd_front (R: the factor's type) keeps
// 4 x 16 rows of P + 1 for F21 in the tile's place.
template <typename R>
__host__ __device__ constexpr int front_tile(int P) {  // in elements of zc
  const int rows = (int)(kNdTile * sizeof(cplx<R>) / sizeof(zc));
  return (P > rows ? P : rows) * (P + 1);
}
size_t leaf_lds(int P) { return (size_t)(P * (P + 1) + kPvSize) * sizeof(zc); }
template <typename R>
size_t front_lds(int P) {
  return (size_t)(front_tile<R>(P) + kPvSize) * sizeof(zc);
}

// A leaf's border: its unknowns' positions in the leaf and their real
// couplings.  At most 32 nodes have at most 66 neighbours around them.
constexpr int kLeafQ = 144;
template <typename R>
struct LeafBorder {
  R f12[kLeafQ], f21[kLeafQ];
  int at[kLeafQ];
};
template <typename R>
__device__ __forceinline__ void leaf_border(LeafBorder<R>& lb, const OpDesc& op, const NdFront& fr,
                                            const int* pdof, const int* bmap, const int* grow) {
  for (int c = threadIdx.x; c < fr.Q; c += 256) {
    const int at = bmap[fr.bor + c];
    const bool real = c < fr.q;
    lb.at[c] = real ? at : 0;
    const int dp = real ? pdof[fr.row + at] : 0, db = real ? pdof[grow[fr.bor + c]] : 0;
    lb.f12[c] = real ? entry<R>(op, 0.0, 0.0, dp, db).re : (R)0;
    lb.f21[c] = real ? entry<R>(op, 0.0, 0.0, db, dp).re : (R)0;
  }
}

// One workgroup per leaf: F11 from the stencil into LDS, its inverse A, and S.
template <typename R>
__global__ __launch_bounds__(256, 2) void k_nd_leaf(FactorArgs<R> g) {
  extern __shared__ __align__(16) char smem_raw[];
  __shared__ LeafBorder<R> lb;
  const int w = g.w0 + blockIdx.y;
  const NdFront fr = g.fronts[g.tasks[blockIdx.x].front];
  const double om_r = g.omega[2 * w], om_i = g.omega[2 * w + 1];
  const int p = fr.p, P = fr.P, Q = fr.Q, ld = P + 1;
  zc* F = reinterpret_cast<zc*>(smem_raw);
  zc* pv = F + P * ld;
  const int* pd = g.pdof + fr.row;
  leaf_border<R>(lb, g.op, fr, g.pdof, g.bmap, g.grow);
  for (int e = threadIdx.x; e < P * ld; e += 256) F[e] = zc{0.0, 0.0};
  __syncthreads();
  if (threadIdx.x < P) {  // one thread a row: its at most six entries in the leaf
    const int r = threadIdx.x;
    if (r < p) {
      const int dof = pd[r], across = fr.across, m = (r >> 1) % across;
      const double* cf = g.op.coef + 12 * (int64_t)(dof >> 1) + 6 * (r & 1);
      F[r * ld + r] = zc{-cf[0] - om_i, om_r};
      F[(r ^ 1) * ld + r] = zc{-cf[5], 0.0};
      if (r + 2 * across < p) F[(r + 2 * across) * ld + r] = zc{-cf[1], 0.0};
      if (r - 2 * across >= 0) F[(r - 2 * across) * ld + r] = zc{-cf[2], 0.0};
      if (m < across - 1) F[(r + 2) * ld + r] = zc{-cf[3], 0.0};
      if (m > 0) F[(r - 2) * ld + r] = zc{-cf[4], 0.0};
    } else {
      F[r * ld + r] = zc{1.0, 0.0};
    }
  }
  __syncthreads();
  invert_tile<double>(F, ld, P, pv, g.status);
  cplx<R>* A = g.factor + w * g.nfactor + fr.a;
  bool bad = false;
  for (int e = threadIdx.x; e < P * P; e += 256) {
    const int c = e / P, r = e - c * P;
    A[e] = kept<R>(F[c * ld + r], bad);
  }
  if (bad) latch(g.status, ST_SINGULAR);
  cplx<R>* S = g.schur_out + w * g.nout + fr.s;
  for (int e = threadIdx.x; e < Q * Q; e += 256) {
    const int r = e / Q, c = e - r * Q;
    const zc v = F[lb.at[c] * ld + lb.at[r]];
    const double f = -lb.f21[r], h = lb.f12[c];
    S[e] = narrow<R>(zc{f * v.re * h, f * v.im * h});
  }
}

// A T x T tile in LDS (T <= TM) to the factor's type in the same place: every
// thread holds its elements over a barrier.
template <int TM, typename R>
__device__ __forceinline__ void tile_narrow(const zc* from, cplx<R>* to, int ld, int T, bool& bad) {
  constexpr int N = (TM * TM + 255) / 256;
  cplx<R> v[N];
#pragma unroll
  for (int u = 0; u < N; u++) {
    const int e = threadIdx.x + 256 * u, c = e / T, r = e - c * T;
    if (e < T * T) v[u] = kept<R>(from[c * ld + r], bad);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < N; u++) {
    const int e = threadIdx.x + 256 * u, c = e / T, r = e - c * T;
    if (e < T * T) to[c * ld + r] = v[u];
  }
  __syncthreads();
}

// A front with halves and P <= 64, one workgroup (blockIdx.z > 0: further ones
// for shares of its border, which invert F11 again): F11 into LDS, its inverse
// A, then B12 = A F12 by 16-column strips (a wave each, F12 pulled straight
// into the MFMA operand) and F21 through LDS into column-major order.  Only a
// border unknown that neither half has (m < 0) can be the stencil's neighbour
// of the separator.
//
// Bound by latency (a chain of loads, the inverse and the products per
// workgroup), so the registers a wave holds, which set how many workgroups a CU
// runs, follow the level's largest P (PM = 16, 32 or 64).
template <typename R, int PM>
__global__ __launch_bounds__(256, PM <= 16 ? 4 : PM <= 32 ? 3 : 2) void k_nd_front(FactorArgs<R> g) {
  extern __shared__ __align__(16) char smem_raw[];
  zc* D = reinterpret_cast<zc*>(smem_raw);            // F11 and its inverse
  cplx<R>* F = reinterpret_cast<cplx<R>*>(smem_raw);  // the inverse as it is kept
  const int w = g.w0 + blockIdx.y;
  const NdFront fr = g.fronts[g.tasks[blockIdx.x].front];
  const double om_r = g.omega[2 * w], om_i = g.omega[2 * w + 1];
  const int p = fr.p, P = fr.P, Q = fr.Q, ld = P + 1;
  zc* pv = D + front_tile<R>(P);
  const int* pd = g.pdof + fr.row;
  const int* bm = g.bmap + fr.bor;
  const int* gr = g.grow + fr.bor;
  const cplx<R>* const sa = g.schur_in + w * g.nin + fr.sA;
  const cplx<R>* const sb = g.schur_in + w * g.nin + fr.sB;
  auto Sh = [&](int h) { return h ? sb : sa; };
  auto Qh = [&](int h) { return h ? fr.QB : fr.QA; };
  auto base = [&](int h) { return h ? fr.baseB : fr.baseA; };
  cplx<R>* A = g.factor + w * g.nfactor + fr.a;
  cplx<R>* B12 = g.factor + w * g.nfactor + fr.b12;
  cplx<R>* F21 = g.factor + w * g.nfactor + fr.f21;
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, i = l & 15, gq = l >> 4;
  {  // rows by waves, columns by lanes (P <= 64); four rows' loads at a time
    const int c = l, cc = min(c, p - 1);
    const cplx<R>* s0 = sa + (int64_t)base(0) * Qh(0) + base(0) + cc;
    const cplx<R>* s1 = sb + (int64_t)base(1) * Qh(1) + base(1) + cc;
    for (int r0 = wave; r0 < P; r0 += 16) {
      cplx<R> x[4], y[4];
#pragma unroll
      for (int u = 0; u < 4; u++) {
        const int rr = min(r0 + 4 * u, p - 1);
        x[u] = s0[(int64_t)rr * Qh(0)];
        y[u] = s1[(int64_t)rr * Qh(1)];
      }
#pragma unroll
      for (int u = 0; u < 4; u++) {
        const int r = r0 + 4 * u;
        if (r >= P || c >= P) continue;
        zc v{r == c ? 1.0 : 0.0, 0.0};
        if (r < p && c < p) {
          v = zc{0.0, 0.0};
          const int d = (r >> 1) - (c >> 1);
          if (d >= -1 && d <= 1) v = entry<double>(g.op, om_r, om_i, pd[r], pd[c]);
          v.re += (double)x[u].re + (double)y[u].re;
          v.im += (double)x[u].im + (double)y[u].im;
        }
        D[c * ld + r] = v;
      }
    }
  }
  __syncthreads();
  invert_tile<double>(D, ld, P, pv, g.status);
  bool bad = false;
  if constexpr (sizeof(R) < sizeof(double)) tile_narrow<PM>(D, F, ld, P, bad);
  if (bad) latch(g.status, ST_SINGULAR);
  if (blockIdx.z == 0)
    for (int e = threadIdx.x; e < P * P; e += 256) {
      const int c = e / P, r = e - c * P;
      A[e] = F[c * ld + r];
    }
  const int step = 4 * gridDim.z;
  for (int t = wave + 4 * blockIdx.z; t < Q / 16; t += step) {
    const int j = 16 * t + i;
    const int m = bm[j];
    const bool real = j < fr.q;
    const int h = m & 1;
    // (a column without a source reads the first half's corner and drops it)
    const cplx<R>* src = m >= 0 ? Sh(h) + (int64_t)base(h) * Qh(h) + (m >> 1) : Sh(0);
    const int lds_ = m >= 0 ? Qh(h) : 0;
    cplx<R> b[PM / 4];
#pragma unroll
    for (int s = 0; s < PM / 4; s++)
      if (4 * s < P) b[s] = src[(int64_t)min(4 * s + gq, p - 1) * lds_];
    CAcc<R> acc[PM / 16];
#pragma unroll
    for (int rb = 0; rb < PM / 16; rb++) zero(acc[rb]);
#pragma unroll
    for (int s = 0; s < PM / 4; s++) {
      if (4 * s >= P) continue;
      const int kk = 4 * s + gq;
      if (m < 0 || kk >= p) b[s] = cplx<R>{(R)0, (R)0};
      if (m < 0 && real && kk < p) b[s] = entry<R>(g.op, om_r, om_i, pd[kk], g.pdof[gr[j]]);
#pragma unroll
      for (int rb = 0; rb < PM / 16; rb++)
        if (16 * rb < P)
          cmfma<R, false, false>(acc[rb].re, acc[rb].im, F[kk * ld + 16 * rb + i], b[s]);
    }
#pragma unroll
    for (int rb = 0; rb < PM / 16; rb++)
      if (16 * rb < P)
#pragma unroll
        for (int e = 0; e < 4; e++)
          B12[(int64_t)(16 * rb + Mf<R>::row(l, e)) * Q + 16 * t + i] =
              cplx<R>{acc[rb].re[e], acc[rb].im[e]};
  }
  __syncthreads();
  // F21, 16 border rows a wave at a time, transposed in the wave's quarter of LDS
  cplx<R>* tr = F + wave * 16 * ld;  // [c][r]
  for (int t0 = 4 * blockIdx.z; t0 < Q / 16; t0 += step) {
    const int t = t0 + wave;
    if (t < Q / 16 && l < P) {
      const int lr = min(l, p - 1);
      cplx<R> v[16];
#pragma unroll
      for (int c = 0; c < 16; c++) {
        const int m = bm[16 * t + c], h = m & 1;
        v[c] = (m >= 0 ? Sh(h) + (int64_t)(m >> 1) * Qh(h) + base(h) : Sh(0))[lr];
      }
#pragma unroll
      for (int c = 0; c < 16; c++) {
        const int cc = 16 * t + c, m = bm[cc];
        if (m < 0 || l >= p) v[c] = cplx<R>{(R)0, (R)0};
        if (m < 0 && cc < fr.q && l < p)
          v[c] = entry<R>(g.op, om_r, om_i, g.pdof[gr[cc]], pd[l]);
        tr[c * ld + l] = v[c];
      }
    }
    __syncthreads();
    if (t < Q / 16)
      for (int r = gq; r < P; r += 4) F21[(int64_t)r * Q + 16 * t + i] = tr[i * ld + r];
    __syncthreads();
  }
}

// Acc (+)= sum over k of X[k][m]^T Y[k][n] for a wave's 2 x 2 blocks of 16 x
// 16: both operands K rows of consecutive m / n.  px, py: the lane's element
// of row l / 16 of each block; four k-steps are loaded ahead.
template <typename R, bool SUB>
__device__ __forceinline__ void gemm32(CAcc<R> (&acc)[2][2], const cplx<R>* const (&px)[2],
                                       int64_t ldx, const cplx<R>* const (&py)[2], int64_t ldy,
                                       int K) {
  cplx<R> x[2][4][2], y[2][4][2];
  const int nc = K >> 4;
  auto load = [&](int buf, int c) {
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
      for (int b = 0; b < 2; b++) {
        x[buf][s][b] = px[b][(16 * c + 4 * s) * ldx];
        y[buf][s][b] = py[b][(16 * c + 4 * s) * ldy];
      }
  };
  auto mul = [&](int buf) {
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
      for (int m = 0; m < 2; m++)
#pragma unroll
        for (int n = 0; n < 2; n++)
          cmfma<R, false, SUB>(acc[m][n].re, acc[m][n].im, x[buf][s][m], y[buf][s][n]);
  };
  load(0, 0);
  for (int c = 0; c < nc; c += 2) {
    load(1, min(c + 1, nc - 1));
    mul(0);
    if (c + 1 >= nc) break;
    load(0, min(c + 2, nc - 1));
    mul(1);
  }
}

// The wave's 32 x 32 quarter of a 64 x 64 tile: block indices, clamped for loads.
struct Quarter {
  int mb[2], nb[2];    // block row / column
  bool mok[2], nok[2];
  int ml[2], nl[2];    // for loads
  __device__ __forceinline__ Quarter(int ti, int tj, int M, int N) {
    const int wave = threadIdx.x >> 6;
#pragma unroll
    for (int b = 0; b < 2; b++) {
      mb[b] = 4 * ti + 2 * (wave >> 1) + b;
      nb[b] = 4 * tj + 2 * (wave & 1) + b;
      mok[b] = 16 * mb[b] < M;
      nok[b] = 16 * nb[b] < N;
      ml[b] = min(mb[b], M / 16 - 1);
      nl[b] = min(nb[b], N / 16 - 1);
    }
  }
  __device__ __forceinline__ bool any() const { return mok[0] && nok[0]; }
};

// S = (the halves' Schur complements at the border) - F21 B12, a 64 x 64 tile
// per workgroup.
template <typename R>
__global__ __launch_bounds__(256, 2) void k_nd_schur(FactorArgs<R> g) {
  const int w = g.w0 + blockIdx.y;
  const NdTask t = g.tasks[xcd_task()];
  const NdFront fr = g.fronts[t.front];
  const int P = fr.P, Q = fr.Q;
  const Quarter q(t.i, t.j, Q, Q);
  if (!q.any()) return;
  const int l = threadIdx.x & 63, i = l & 15, gq = l >> 4;
  const int* bm = g.bmap + fr.bor;
  const cplx<R>* F21 = g.factor + w * g.nfactor + fr.f21;
  const cplx<R>* B12 = g.factor + w * g.nfactor + fr.b12;
  cplx<R>* S = g.schur_out + w * g.nout + fr.s;
  CAcc<R> acc[2][2];
#pragma unroll
  for (int m = 0; m < 2; m++)
#pragma unroll
    for (int n = 0; n < 2; n++) zero(acc[m][n]);
  {
    const cplx<R>* Sa = g.schur_in + w * g.nin + fr.sA;
    const cplx<R>* Sb = g.schur_in + w * g.nin + fr.sB;
#pragma unroll
    for (int n = 0; n < 2; n++) {
      const int mj = bm[16 * q.nl[n] + i];
      const cplx<R>* src = (mj & 1) ? Sb : Sa;
      const int ld = (mj & 1) ? fr.QB : fr.QA;
#pragma unroll
      for (int m = 0; m < 2; m++)
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const int mi = bm[16 * q.ml[m] + Mf<R>::row(l, e)];
          if (mi >= 0 && mj >= 0 && ((mi ^ mj) & 1) == 0) {
            const cplx<R> v = src[(int64_t)(mi >> 1) * ld + (mj >> 1)];
            acc[m][n].re[e] = v.re;
            acc[m][n].im[e] = v.im;
          }
        }
    }
  }
  const cplx<R>* const px[2] = {F21 + (int64_t)gq * Q + 16 * q.ml[0] + i,
                                F21 + (int64_t)gq * Q + 16 * q.ml[1] + i};
  const cplx<R>* const py[2] = {B12 + (int64_t)gq * Q + 16 * q.nl[0] + i,
                                B12 + (int64_t)gq * Q + 16 * q.nl[1] + i};
  gemm32<R, true>(acc, px, Q, py, Q, P);
#pragma unroll
  for (int m = 0; m < 2; m++)
#pragma unroll
    for (int n = 0; n < 2; n++)
      if (q.mok[m] && q.nok[n])
#pragma unroll
        for (int e = 0; e < 4; e++)
          S[(int64_t)(16 * q.mb[m] + Mf<R>::row(l, e)) * Q + 16 * q.nb[n] + i] =
              cplx<R>{acc[m][n].re[e], acc[m][n].im[e]};
}

// B12 = A T12 (P > 64)
template <typename R>
__global__ __launch_bounds__(256, 2) void k_nd_border(FactorArgs<R> g) {
  const int w = g.w0 + blockIdx.y;
  const NdTask t = g.tasks[xcd_task()];
  const NdFront fr = g.fronts[t.front];
  const int P = fr.P, Q = fr.Q;
  const Quarter q(t.i, t.j, P, Q);
  if (!q.any()) return;
  const int l = threadIdx.x & 63, i = l & 15, gq = l >> 4;
  const cplx<R>* A = g.factor + w * g.nfactor + fr.a;
  const cplx<R>* T12 = g.temp + w * g.ntemp + fr.t;
  cplx<R>* B12 = g.factor + w * g.nfactor + fr.b12;
  CAcc<R> acc[2][2];
#pragma unroll
  for (int m = 0; m < 2; m++)
#pragma unroll
    for (int n = 0; n < 2; n++) zero(acc[m][n]);
  const cplx<R>* const px[2] = {A + (int64_t)gq * P + 16 * q.ml[0] + i,
                                A + (int64_t)gq * P + 16 * q.ml[1] + i};
  const cplx<R>* const py[2] = {T12 + (int64_t)gq * Q + 16 * q.nl[0] + i,
                                T12 + (int64_t)gq * Q + 16 * q.nl[1] + i};
  gemm32<R, false>(acc, px, P, py, Q, P);
#pragma unroll
  for (int m = 0; m < 2; m++)
#pragma unroll
    for (int n = 0; n < 2; n++)
      if (q.mok[m] && q.nok[n])
#pragma unroll
        for (int e = 0; e < 4; e++)
          B12[(int64_t)(16 * q.mb[m] + Mf<R>::row(l, e)) * Q + 16 * q.nb[n] + i] =
              cplx<R>{acc[m][n].re[e], acc[m][n].im[e]};
}

// Temporaries of a front with P > 64: T12 (P x Q, row-major), the pivot
// block's row (64 x P, row-major) and column (64 columns of P), and two
// copies (by pivot parity) of the pivot inverse, column- and row-major.
__device__ __forceinline__ int64_t t_row(const NdFront& f) { return f.t + (int64_t)f.P * f.Q; }
__device__ __forceinline__ int64_t t_col(const NdFront& f) {
  return t_row(f) + (int64_t)kNdTile * f.P;
}
__device__ __forceinline__ int64_t t_piv(const NdFront& f, int k, int rowmajor) {
  return t_col(f) + (int64_t)kNdTile * f.P + (2 * (k & 1) + rowmajor) * kNdTile * kNdTile;
}
__device__ __forceinline__ int tile_width(int P, int k) { return min(kNdTile, P - kNdTile * k); }

// Invert the T x T tile in LDS and write it as pivot inverse k.
template <typename R>
__device__ __forceinline__ void pivot_out(cplx<R>* F, cplx<R>* pv, int T, const NdFront& fr, int k,
                          cplx<R>* temp, uint32_t* status) {
  __syncthreads();
  invert_tile<R>(F, kLd, T, pv, status);
  cplx<R>* pc = temp + t_piv(fr, k, 0);
  cplx<R>* pr = temp + t_piv(fr, k, 1);
  for (int e = threadIdx.x; e < T * T; e += 256) {
    const int c = e / T, r = e - c * T;
    pc[c * kNdTile + r] = F[c * kLd + r];
    pr[c * kNdTile + r] = F[r * kLd + c];
  }
}

// A 64 x 64 tile of F11 (kind 0, into A), F12 (1, into T12) or F21 (2).
// F11's first tile is the first pivot: it is inverted at once.
template <typename R>
__global__ __launch_bounds__(256, 2) void k_nd_assemble(FactorArgs<R> g) {
  extern __shared__ __align__(16) char smem_raw[];
  cplx<R>* F = reinterpret_cast<cplx<R>*>(smem_raw);
  cplx<R>* pv = F + kNdTile * kLd;
  const int w = g.w0 + blockIdx.y;
  const NdTask t = g.tasks[xcd_task()];
  const NdFront fr = g.fronts[t.front];
  const double om_r = g.omega[2 * w], om_i = g.omega[2 * w + 1];
  const int p = fr.p, P = fr.P, Q = fr.Q;
  const int* pd = g.pdof + fr.row;
  const int* bm = g.bmap + fr.bor;
  const int* gr = g.grow + fr.bor;
  const cplx<R>* const sa = g.schur_in + w * g.nin + fr.sA;
  const cplx<R>* const sb = g.schur_in + w * g.nin + fr.sB;
  auto Sh = [&](int h) { return h ? sb : sa; };
  auto Qh = [&](int h) { return h ? fr.QB : fr.QA; };
  auto base = [&](int h) { return h ? fr.baseB : fr.baseA; };
  const int M = t.kind == 2 ? Q : P, N = t.kind == 1 ? Q : P;
  const int r0 = kNdTile * t.i, c0 = kNdTile * t.j;
  const int nr = min(kNdTile, M - r0), nc = min(kNdTile, N - c0);
  const int cl = threadIdx.x & 63;
  const int c = c0 + cl;
  cplx<R>* T12 = g.temp + w * g.ntemp + fr.t;
  // Four rows' loads at a time, from valid places also where there is none;
  // the stencil couples a separator's unknowns along its line, and with a
  // border unknown only if neither half has it (m < 0).
  const int cc = min(c, (t.kind == 1 ? fr.q : p) - 1);
  const int mc = t.kind == 1 && cl < nc ? bm[c] : -1;
  const int dc = cl >= nc ? -1 : t.kind == 1 ? (c < fr.q ? g.pdof[gr[c]] : -1) : pd[c];
  const cplx<R>* q0 = Sh(0);
  const cplx<R>* q1 = Sh(1);
  int64_t l0 = 0, l1 = 0;
  if (t.kind == 0) {
    q0 += (int64_t)base(0) * Qh(0) + base(0) + cc;
    q1 += (int64_t)base(1) * Qh(1) + base(1) + cc;
    l0 = Qh(0);
    l1 = Qh(1);
  } else if (t.kind == 1 && mc >= 0) {
    q0 = Sh(mc & 1) + (int64_t)base(mc & 1) * Qh(mc & 1) + (mc >> 1);
    l0 = Qh(mc & 1);
  }
  for (int b0 = threadIdx.x >> 6; b0 < nr; b0 += 16) {
    cplx<R> x[4], y[4];
    int mr[4];
#pragma unroll
    for (int u = 0; u < 4; u++) {
      const int r = min(r0 + b0 + 4 * u, (t.kind == 2 ? fr.q : p) - 1);
      mr[u] = t.kind == 2 ? bm[r] : 0;
      y[u] = cplx<R>{(R)0, (R)0};
      if (t.kind == 2) {
        const int h = mr[u] & 1;
        x[u] = (mr[u] >= 0 ? Sh(h) + (int64_t)(mr[u] >> 1) * Qh(h) + base(h) : Sh(0))[cc];
      } else {
        x[u] = q0[r * l0];
        if (t.kind == 0) y[u] = q1[r * l1];
      }
    }
#pragma unroll
    for (int u = 0; u < 4; u++) {
      const int rl = b0 + 4 * u, r = r0 + rl;
      if (rl >= nr || cl >= nc) continue;
      cplx<R> v{(R)0, (R)0};
      if (t.kind == 0) {
        if (r < p && c < p) {
          const int d = (r >> 1) - (c >> 1);
          if (d >= -1 && d <= 1) v = entry<R>(g.op, om_r, om_i, pd[r], dc);
          add(v, x[u]);
          add(v, y[u]);
        } else {
          v.re = (R)(r == c ? 1 : 0);
        }
      } else if (t.kind == 1) {
        if (r < p && dc >= 0) v = mc >= 0 ? x[u] : entry<R>(g.op, om_r, om_i, pd[r], dc);
      } else if (r < fr.q && c < p) {
        v = mr[u] >= 0 ? x[u] : entry<R>(g.op, om_r, om_i, g.pdof[gr[r]], dc);
      }
      if (t.kind == 1) T12[(int64_t)r * Q + c] = v;
      else F[cl * kLd + rl] = v;
    }
  }
  if (t.kind == 1) return;
  __syncthreads();
  cplx<R>* out = g.factor + w * g.nfactor + (t.kind == 0 ? fr.a : fr.f21);
  const int rl = threadIdx.x & 63;
  if (rl < nr)
    for (int k = threadIdx.x >> 6; k < nc; k += 4)
      out[(int64_t)(c0 + k) * M + r0 + rl] = F[k * kLd + rl];
  if (t.kind == 0 && t.i == 0 && t.j == 0)
    pivot_out<R>(F, pv, nr, fr, 0, g.temp + w * g.ntemp, g.status);
}

// Pivot tile k's block row, R_j = F(k,k)^-1 F(k, j) (kind 0), and a copy of
// its block column (kind 1): what the update reads while it overwrites both.
template <typename R>
__global__ __launch_bounds__(256, 2) void k_nd_panel(FactorArgs<R> g) {
  extern __shared__ __align__(16) char smem_raw[];
  cplx<R>* F = reinterpret_cast<cplx<R>*>(smem_raw);
  const int w = g.w0 + blockIdx.y;
  const NdTask t = g.tasks[xcd_task()];
  const NdFront fr = g.fronts[t.front];
  const int P = fr.P, k = t.j;
  const int T = tile_width(P, k), N = tile_width(P, t.i);  // pivot tile, tile t.i
  const cplx<R>* A = g.factor + w * g.nfactor + fr.a;
  cplx<R>* temp = g.temp + w * g.ntemp;
  const int r = threadIdx.x & 63;
  if (t.kind == 1) {
    if (r < N)
      for (int c = threadIdx.x >> 6; c < T; c += 4)
        temp[t_col(fr) + (int64_t)c * P + kNdTile * t.i + r] =
            A[(int64_t)(kNdTile * k + c) * P + kNdTile * t.i + r];
    return;
  }
  if (r < T)
    for (int c = threadIdx.x >> 6; c < N; c += 4)
      F[c * kLd + r] = A[(int64_t)(kNdTile * t.i + c) * P + kNdTile * k + r];
  __syncthreads();
  const Quarter q(0, 0, T, N);
  if (!q.any()) return;
  const int l = threadIdx.x & 63, i = l & 15, gq = l >> 4;
  const cplx<R>* piv = temp + t_piv(fr, k, 0);
  CAcc<R> acc[2][2];
#pragma unroll
  for (int m = 0; m < 2; m++)
#pragma unroll
    for (int n = 0; n < 2; n++) zero(acc[m][n]);
  const cplx<R>* const px[2] = {piv + gq * kNdTile + 16 * q.ml[0] + i,
                                piv + gq * kNdTile + 16 * q.ml[1] + i};
  const cplx<R>* const py[2] = {F + (16 * q.nl[0] + i) * kLd + gq,
                                F + (16 * q.nl[1] + i) * kLd + gq};
  gemm32<R, false>(acc, px, kNdTile, py, 1, T);
#pragma unroll
  for (int m = 0; m < 2; m++)
#pragma unroll
    for (int n = 0; n < 2; n++)
      if (q.mok[m] && q.nok[n])
#pragma unroll
        for (int e = 0; e < 4; e++)
          temp[t_row(fr) + (int64_t)(16 * q.mb[m] + Mf<R>::row(l, e)) * P + kNdTile * t.i +
               16 * q.nb[n] + i] = cplx<R>{acc[m][n].re[e], acc[m][n].im[e]};
}

// Gauss-Jordan update of tile (i, j) of A for pivot tile k:
//   F(i, j) -= C_i R_j;  F(i, k) = -C_i F(k,k)^-1;  F(k, j) = R_j;  F(k, k) = its inverse
// computed transposed (rows of the product along j), so that lanes hold
// consecutive elements of A's columns.  The next pivot tile is inverted where
// it is updated.
template <typename R>
__global__ __launch_bounds__(256, 2) void k_nd_update(FactorArgs<R> g) {
  extern __shared__ __align__(16) char smem_raw[];
  cplx<R>* F = reinterpret_cast<cplx<R>*>(smem_raw);
  cplx<R>* pv = F + kNdTile * kLd;
  const int w = g.w0 + blockIdx.y;
  const NdTask t = g.tasks[xcd_task()];
  const NdFront fr = g.fronts[t.front];
  const int P = fr.P, k = t.kind;
  const int T = tile_width(P, k), M = tile_width(P, t.j), N = tile_width(P, t.i);
  cplx<R>* temp = g.temp + w * g.ntemp;
  cplx<R>* A = g.factor + w * g.nfactor + fr.a + (int64_t)kNdTile * t.j * P + kNdTile * t.i;
  if (t.i == k) {  // the pivot's block row, through LDS into column-major order
    if (t.j == k) {
      const cplx<R>* piv = temp + t_piv(fr, k, 0);
      const int r = threadIdx.x & 63;
      if (r < T)
        for (int c = threadIdx.x >> 6; c < T; c += 4) A[(int64_t)c * P + r] = piv[c * kNdTile + r];
      return;
    }
    const cplx<R>* row = temp + t_row(fr) + kNdTile * t.j;
    const int x = threadIdx.x & 63;
    if (x < M)
      for (int r = threadIdx.x >> 6; r < T; r += 4) F[x * kLd + r] = row[(int64_t)r * P + x];
    __syncthreads();
    if (x < T)
      for (int c = threadIdx.x >> 6; c < M; c += 4) A[(int64_t)c * P + x] = F[c * kLd + x];
    return;
  }
  const bool next = t.i == k + 1 && t.j == k + 1;
  const Quarter q(0, 0, M, N);
  const int l = threadIdx.x & 63, i = l & 15, gq = l >> 4;
  if (q.any()) {
    CAcc<R> acc[2][2];
#pragma unroll
    for (int m = 0; m < 2; m++)
#pragma unroll
      for (int n = 0; n < 2; n++) {
        zero(acc[m][n]);
        if (t.j != k)
#pragma unroll
          for (int e = 0; e < 4; e++) {
            const cplx<R> v = A[(int64_t)(16 * q.ml[m] + Mf<R>::row(l, e)) * P + 16 * q.nl[n] + i];
            acc[m][n].re[e] = v.re;
            acc[m][n].im[e] = v.im;
          }
      }
    const cplx<R>* X = t.j == k ? temp + t_piv(fr, k, 1) : temp + t_row(fr) + kNdTile * t.j;
    const int64_t ldx = t.j == k ? kNdTile : P;
    const cplx<R>* Y = temp + t_col(fr) + kNdTile * t.i;
    const cplx<R>* const px[2] = {X + gq * ldx + 16 * q.ml[0] + i, X + gq * ldx + 16 * q.ml[1] + i};
    const cplx<R>* const py[2] = {Y + (int64_t)gq * P + 16 * q.nl[0] + i,
                                  Y + (int64_t)gq * P + 16 * q.nl[1] + i};
    gemm32<R, true>(acc, px, ldx, py, P, T);
#pragma unroll
    for (int m = 0; m < 2; m++)
#pragma unroll
      for (int n = 0; n < 2; n++)
        if (q.mok[m] && q.nok[n])
#pragma unroll
          for (int e = 0; e < 4; e++) {
            const int c = 16 * q.mb[m] + Mf<R>::row(l, e), r = 16 * q.nb[n] + i;
            const cplx<R> v{acc[m][n].re[e], acc[m][n].im[e]};
            if (next) F[c * kLd + r] = v;
            else A[(int64_t)c * P + r] = v;
          }
  }
  if (next) pivot_out<R>(F, pv, N, fr, k + 1, temp, g.status);
}

// ---------------------------------------------------------------------------
// Solves
// ---------------------------------------------------------------------------
template <typename R, typename IO>
struct SolveArgs {
  const NdFront* fronts;
  const NdTask* tasks;
  const int *pdof, *bmap, *grow;
  const cplx<R>* factor;
  cplx<R>*w, *z;          // (shift, row, column)
  cplx<R>*uin, *uout;     // the halves' updates, this level's
  int64_t nfactor, nw, nuin, nuout;  // elements per shift
  OpDesc op;
  const cplx<IO>* B;      // the caller's right-hand sides and solutions (their first column)
  cplx<IO>* X;
  int64_t n, bstride, xstride;
  int k, adjoint, qsplit;
  int w0;
  const uint32_t* skip;
};
__device__ __forceinline__ bool skipped(const uint32_t* skip) {
  return skip && __hip_atomic_load(skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The separators' right-hand sides by rows: w[row][j] = B[j][pdof[row]], zero
// for padding and for the row after the last; back for the solution.
constexpr int kRowTile = 32;
template <typename R, typename IO, bool OUT>
__global__ __launch_bounds__(256) void k_nd_permute(const int* pdof, int64_t rows, int64_t n, int k,
                                                    int64_t cstride, const cplx<IO>* B,
                                                    cplx<IO>* X, cplx<R>* W, int w0,
                                                    const uint32_t* skip) {
  if (skipped(skip)) return;
  __shared__ cplx<R> tile[kRowTile][33];
  const int w = w0 + blockIdx.y;
  const int64_t r0 = (int64_t)blockIdx.x * kRowTile;
  const int64_t total = rows + 1;  // with the zero row
  const int nr = (int)min((int64_t)kRowTile, total - r0);
  cplx<R>* Wt = W + (w * total + r0) * k;
  const int r = threadIdx.x & 31;
  const int dof = r0 + r < rows ? pdof[r0 + r] : -1;
  if (OUT) {
    for (int e = threadIdx.x; e < nr * k; e += 256) tile[e / k][e % k] = Wt[e];
    __syncthreads();
    if (dof >= 0)
      for (int j = threadIdx.x >> 5; j < k; j += 8) {
        const cplx<R> v = tile[r][j];
        X[(int64_t)w * cstride + (int64_t)j * n + dof] = cplx<IO>{(IO)v.re, (IO)v.im};
      }
  } else {
    for (int j = threadIdx.x >> 5; j < k; j += 8) {
      cplx<R> v{(R)0, (R)0};
      if (dof >= 0) {
        const cplx<IO> b = B[(int64_t)w * cstride + (int64_t)j * n + dof];
        v = cplx<R>{(R)b.re, (R)b.im};
      }
      tile[r][j] = v;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < nr * k; e += 256) Wt[e] = tile[e / k][e % k];
  }
}

// Columns go through the matrix cores eight at a time in real form: MFMA
// column c < 8 holds the real part of a block's column c and column c + 8 the
// imaginary part, so that a complex product is two real MFMAs,
//   [Yr | Yi] += Xr [Vr | Vi] + Xi [-Vi | Vr],
// and a block of k columns takes 2 ceil(k / 8) of them per 16 rows and 4 inner
// elements instead of 4 ceil(k / 16) (k = 20: 6 instead of 8).
template <typename R>
using v4 = typename Mf<R>::v4;

// acc[b] += X(rows of one 16-row block) * V over the k-chunks of 16 in
// [c0, nc) by step; X element (i, kk) at i + kk * ld (KF false) or
// i * ld + kk (KF true); row(kk): V's row, col[b] the lane's column in it.
// KF takes k in the order 4 (l / 16) + s, so that a lane's four loads are
// consecutive.  LDS: V is in LDS and read when it is used.
template <typename R, int NB, bool KF, bool CONJ, bool LDS, typename RowPtr>
__device__ __forceinline__ void rows_mul(v4<R> (&acc)[NB], const cplx<R>* X, int64_t ld, int c0,
                                         int nc, int step, const int (&col)[NB], RowPtr row) {
  const int l = threadIdx.x & 63, i = l & 15, g = l >> 4;
  const bool hi = i >= 8;
  cplx<R> x[2][4], v[2][4][LDS ? 1 : NB];
  auto at = [&](int c, int s) { return 16 * c + (KF ? 4 * g + s : 4 * s + g); };
  auto load = [&](int buf, int c) {
#pragma unroll
    for (int s = 0; s < 4; s++) {
      const int kk = at(c, s);
      x[buf][s] = X[KF ? i * ld + kk : (int64_t)kk * ld + i];
      if constexpr (!LDS) {
        const cplx<R>* vr = row(kk);
#pragma unroll
        for (int b = 0; b < NB; b++) v[buf][s][b] = vr[col[b]];
      }
    }
  };
  auto mul = [&](int buf, int c) {
#pragma unroll
    for (int s = 0; s < 4; s++) {
      const R xi = CONJ ? -x[buf][s].im : x[buf][s].im;
#pragma unroll
      for (int b = 0; b < NB; b++) {
        cplx<R> y;
        if constexpr (LDS) y = row(at(c, s))[col[b]];
        else y = v[buf][s][b];
        acc[b] = Mf<R>::op(x[buf][s].re, hi ? y.im : y.re, acc[b]);
        acc[b] = Mf<R>::op(xi, hi ? y.re : -y.im, acc[b]);
      }
    }
  };
  if (c0 >= nc) return;
  load(0, c0);
  for (int c = c0; c < nc; c += 2 * step) {
    load(1, c + step < nc ? c + step : c);
    mul(0, c);
    if (c + step >= nc) break;
    load(0, c + 2 * step < nc ? c + 2 * step : c);
    mul(1, c + step);
  }
}
template <typename R, int NB>
__device__ __forceinline__ void zero(v4<R> (&acc)[NB]) {
#pragma unroll
  for (int b = 0; b < NB; b++) acc[b] = v4<R>{0, 0, 0, 0};
}
// the lane's part of element (row(l, e), block b) of a rows x pitch array
template <typename R>
__device__ __forceinline__ R& part(cplx<R>* a, int64_t pitch, int r, int b) {
  const int i = threadIdx.x & 15;
  return reinterpret_cast<R*>(a + r * pitch + 8 * b + (i & 7))[i >> 3];
}

// A leaf, sweep up: z = A b (A^H b) in LDS, u = -F21 z (-F12^H z).
template <typename R, typename IO, int NB, bool ADJ>
__global__ __launch_bounds__(256, 2) void k_nd_leaf_up(SolveArgs<R, IO> a) {
  if (skipped(a.skip)) return;
  extern __shared__ __align__(16) char smem_raw[];
  __shared__ LeafBorder<R> lb;
  constexpr int NC = 8 * NB + 1;  // pitch: columns of one row, and a bank of its own
  const int w = a.w0 + blockIdx.y;
  const NdFront fr = a.fronts[a.tasks[blockIdx.x].front];
  const int P = fr.P, k = a.k;
  cplx<R>* bs = reinterpret_cast<cplx<R>*>(smem_raw);  // P x NC
  leaf_border<R>(lb, a.op, fr, a.pdof, a.bmap, a.grow);
  const int r = threadIdx.x & 63;
  const int dof = r < P ? a.pdof[fr.row + r] : -1;
  const cplx<IO>* B = a.B + (int64_t)w * a.bstride;
  if (r < P)
    for (int j = threadIdx.x >> 6; j < 8 * NB; j += 4) {
      cplx<R> v{(R)0, (R)0};
      if (dof >= 0 && j < k) {
        const cplx<IO> b = B[j * a.n + dof];
        v = cplx<R>{(R)b.re, (R)b.im};
      }
      bs[r * NC + j] = v;
    }
  __syncthreads();
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
  int col[NB];
#pragma unroll
  for (int b = 0; b < NB; b++) col[b] = 8 * b + (l & 7);
  v4<R> acc[NB];
  zero<R, NB>(acc);
  const cplx<R>* A = a.factor + w * a.nfactor + fr.a;
  if (16 * wave < P)
    rows_mul<R, NB, ADJ, ADJ, true>(acc, A + (ADJ ? 16 * wave * P : 16 * wave), P, 0, P / 16, 1, col,
                                    [&](int kk) { return bs + kk * NC; });
  __syncthreads();
  if (16 * wave < P)
#pragma unroll
    for (int b = 0; b < NB; b++)
#pragma unroll
      for (int e = 0; e < 4; e++) part(bs, NC, 16 * wave + Mf<R>::row(l, e), b) = acc[b][e];
  __syncthreads();
  cplx<R>* u = a.uout + w * a.nuout + (int64_t)fr.urow * k;
  for (int e = threadIdx.x; e < fr.Q * k; e += 256) {
    const int c = e / k, j = e - c * k;
    const R f = ADJ ? -lb.f12[c] : -lb.f21[c];
    const cplx<R> z = bs[lb.at[c] * NC + j];
    u[e] = cplx<R>{f * z.re, f * z.im};
  }
}

// A leaf, sweep down: x = A (b - F12 x2) (A^H (b - F21^H x2)) into X.
template <typename R, typename IO, int NB, bool ADJ>
__global__ __launch_bounds__(256, 2) void k_nd_leaf_down(SolveArgs<R, IO> a) {
  if (skipped(a.skip)) return;
  extern __shared__ __align__(16) char smem_raw[];
  __shared__ LeafBorder<R> lb;
  constexpr int NC = 8 * NB + 1;
  const int w = a.w0 + blockIdx.y;
  const NdFront fr = a.fronts[a.tasks[blockIdx.x].front];
  const int P = fr.P, k = a.k;
  cplx<R>* bs = reinterpret_cast<cplx<R>*>(smem_raw);
  leaf_border<R>(lb, a.op, fr, a.pdof, a.bmap, a.grow);
  const int r = threadIdx.x & 63;
  const int dof = r < P ? a.pdof[fr.row + r] : -1;
  const cplx<IO>* B = a.B + (int64_t)w * a.bstride;
  if (r < P)
    for (int j = threadIdx.x >> 6; j < 8 * NB; j += 4) {
      cplx<R> v{(R)0, (R)0};
      if (dof >= 0 && j < k) {
        const cplx<IO> b = B[j * a.n + dof];
        v = cplx<R>{(R)b.re, (R)b.im};
      }
      bs[r * NC + j] = v;
    }
  const cplx<R>* W = a.w + w * a.nw;
  const int* gr = a.grow + fr.bor;
#pragma unroll
  for (int side = 0; side < 4; side++) {  // a leaf unknown has one neighbour a side at most
    __syncthreads();
    const int s0 = fr.side[side], len = fr.side[side + 1] - s0;
    for (int e = threadIdx.x; e < len * k; e += 256) {
      const int c = s0 + e / k, j = e % k;
      const cplx<R> x = W[(int64_t)gr[c] * k + j];
      const R f = ADJ ? lb.f21[c] : lb.f12[c];
      cplx<R>& t = bs[lb.at[c] * NC + j];
      t.re -= f * x.re;
      t.im -= f * x.im;
    }
  }
  __syncthreads();
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
  int col[NB];
#pragma unroll
  for (int b = 0; b < NB; b++) col[b] = 8 * b + (l & 7);
  v4<R> acc[NB];
  zero<R, NB>(acc);
  const cplx<R>* A = a.factor + w * a.nfactor + fr.a;
  if (16 * wave < P)
    rows_mul<R, NB, ADJ, ADJ, true>(acc, A + (ADJ ? 16 * wave * P : 16 * wave), P, 0, P / 16, 1, col,
                                    [&](int kk) { return bs + kk * NC; });
  __syncthreads();
  if (16 * wave < P)
#pragma unroll
    for (int b = 0; b < NB; b++)
#pragma unroll
      for (int e = 0; e < 4; e++) part(bs, NC, 16 * wave + Mf<R>::row(l, e), b) = acc[b][e];
  __syncthreads();
  if (dof >= 0)
    for (int j = threadIdx.x >> 6; j < k; j += 4) {
      const cplx<R> v = bs[r * NC + j];
      a.X[(int64_t)w * a.xstride + j * a.n + dof] = cplx<IO>{(IO)v.re, (IO)v.im};
    }
}

// A 16-row operand block of P <= PM inner elements, all its loads issued at
// once (i + kk * ld, kk = 4 s + l / 16), and its product with V in LDS.
template <typename R, int PM>
struct OperandBlock {
  cplx<R> v[PM / 4];
};
template <typename R, int PM>
__device__ __forceinline__ void load_block(OperandBlock<R, PM>& x, const cplx<R>* X, int64_t ld,
                                           int P) {
  const int l = threadIdx.x & 63, i = l & 15, g = l >> 4;
#pragma unroll
  for (int s = 0; s < PM / 4; s++)
    if (4 * s < P) x.v[s] = X[(int64_t)(4 * s + g) * ld + i];
}
template <typename R, int PM, int NB, bool CONJ>
__device__ __forceinline__ void block_mul(v4<R> (&acc)[NB], const OperandBlock<R, PM>& x, int P,
                                          const int (&col)[NB], const cplx<R>* V, int pitch) {
  const int l = threadIdx.x & 63, g = l >> 4;
  const bool hi = (l & 15) >= 8;
#pragma unroll
  for (int s = 0; s < PM / 4; s++) {
    if (4 * s >= P) continue;
    const R xi = CONJ ? -x.v[s].im : x.v[s].im;
#pragma unroll
    for (int b = 0; b < NB; b++) {
      const cplx<R> y = V[(4 * s + g) * pitch + col[b]];
      acc[b] = Mf<R>::op(x.v[s].re, hi ? y.im : y.re, acc[b]);
      acc[b] = Mf<R>::op(xi, hi ? y.re : -y.im, acc[b]);
    }
  }
}

// A front with P <= 64, sweep up: one workgroup per front (and share of its
// border rows, blockIdx.z).  A chain of short products: each one's operands are
// on their way before the one ahead of it is done, and the halves' updates
// while it runs (8 shifts, 512 x 256, a solve 4.14 -> 4.00 ms).
// PM: the level's largest P, 16, 32 or 64 (the operands held in registers)
template <typename R, typename IO, int NB, bool ADJ, int PM>
__global__ __launch_bounds__(256, 2) void k_nd_up(SolveArgs<R, IO> a) {
  if (skipped(a.skip)) return;
  extern __shared__ __align__(16) char smem_raw[];
  constexpr int NC = 8 * NB;
  const int w = a.w0 + blockIdx.y;
  const NdFront fr = a.fronts[a.tasks[blockIdx.x].front];
  const int P = fr.P, Q = fr.Q, k = a.k;
  cplx<R>* bs = reinterpret_cast<cplx<R>*>(smem_raw);  // b1, P x NC
  cplx<R>* zs = ADJ ? bs : bs + P * NC;                // z
  const cplx<R>* ua = a.uin + w * a.nuin + (int64_t)fr.uA * k;
  const cplx<R>* ub = a.uin + w * a.nuin + (int64_t)fr.uB * k;
  cplx<R>* z = a.z + w * a.nw + (int64_t)fr.row * k;
  const cplx<R>* b = a.w + w * a.nw + (int64_t)fr.row * k;
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int hi = (l >> 3) & 1;
  const cplx<R>* fac = a.factor + w * a.nfactor;
  // the first product's operands, which wait on nothing, before b1's loads
  const int first = ADJ ? wave + 4 * (int)blockIdx.z : wave;
  const bool live = 16 * first < (ADJ ? Q : P);
  const int64_t xld = ADJ ? Q : P;
  const cplx<R>* xp = fac + (ADJ ? fr.b12 : fr.a) + 16 * (live ? first : 0);
  OperandBlock<R, PM> x;
  if (!ADJ || Q > 0) load_block<R, PM>(x, xp, xld, P);
  for (int e0 = threadIdx.x; e0 < P * NC; e0 += 1024) {  // four elements' loads at a time
    cplx<R> v[4], p[4], q[4];
#pragma unroll
    for (int u = 0; u < 4; u++) {
      const int e = min(e0 + 256 * u, P * NC - 1);
      const int r = e / NC, j = min(e % NC, k - 1), rr = min(r, fr.p - 1);
      v[u] = b[r * k + j];
      p[u] = ua[(fr.baseA + rr) * k + j];
      q[u] = ub[(fr.baseB + rr) * k + j];
    }
#pragma unroll
    for (int u = 0; u < 4; u++) {
      const int e = e0 + 256 * u;
      if (e >= P * NC) continue;
      const int r = e / NC, j = e % NC;
      if (r < fr.p) {
        add(v[u], p[u]);
        add(v[u], q[u]);
      }
      if (j >= k) v[u] = cplx<R>{(R)0, (R)0};
      else if (ADJ && blockIdx.z == 0) z[r * k + j] = v[u];
      bs[e] = v[u];
    }
  }
  __syncthreads();
  int col[NB];
#pragma unroll
  for (int c = 0; c < NB; c++) col[c] = 8 * c + (l & 7);
  v4<R> acc[NB];
  if (!ADJ) {
    if (live) {
      zero<R, NB>(acc);
      block_mul<R, PM, NB, false>(acc, x, P, col, bs, NC);
    }
    // F21's first rows, while z is written and read back
    if (Q > 0)
      load_block<R, PM>(x, fac + fr.f21 + 16 * min(wave + 4 * (int)blockIdx.z, Q / 16 - 1), Q, P);
    if (live)
#pragma unroll
      for (int c = 0; c < NB; c++)
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const int r = 16 * wave + Mf<R>::row(l, e);
          part(zs, NC, r, c) = acc[c][e];
          if (blockIdx.z == 0 && col[c] < k) part(z, k, r, c) = acc[c][e];
        }
    __syncthreads();
  }
  const int* bm = a.bmap + fr.bor;
  cplx<R>* uo = a.uout + w * a.nuout + (int64_t)fr.urow * k;
  for (int rb = wave + 4 * blockIdx.z; rb < Q / 16; rb += 4 * a.qsplit) {
    R pulled[4][NB];  // the halves' updates, loaded while the product runs
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int m = bm[16 * rb + Mf<R>::row(l, e)];
      const cplx<R>* src = m < 0 ? ua : ((m & 1) ? ub : ua) + (m >> 1) * k;
#pragma unroll
      for (int c = 0; c < NB; c++) {
        const R v = reinterpret_cast<const R*>(src + min(col[c], k - 1))[hi];
        pulled[e][c] = m >= 0 ? v : (R)0;
      }
    }
    zero<R, NB>(acc);
    block_mul<R, PM, NB, ADJ>(acc, x, P, col, zs, NC);
    const int nx = rb + 4 * a.qsplit;
    if (nx < Q / 16) load_block<R, PM>(x, fac + (ADJ ? fr.b12 : fr.f21) + 16 * nx, Q, P);
#pragma unroll
    for (int e = 0; e < 4; e++)
#pragma unroll
      for (int c = 0; c < NB; c++)
        if (col[c] < k)
          part(uo, k, 16 * rb + Mf<R>::row(l, e), c) = pulled[e][c] - acc[c][e];
  }
}

// A front with P <= kNdDownP, sweep down; the four waves split the inner
// dimension where P leaves them idle.
template <typename R, typename IO, int NB, bool ADJ>
__global__ __launch_bounds__(256, 2) void k_nd_down(SolveArgs<R, IO> a) {
  if (skipped(a.skip)) return;
  extern __shared__ __align__(16) char smem_raw[];
  constexpr int NC = 8 * NB;
  cplx<R>* red = reinterpret_cast<cplx<R>*>(smem_raw);  // 4 x 16 x NC: the waves' sums
  const int w = a.w0 + blockIdx.y;
  const NdFront fr = a.fronts[a.tasks[blockIdx.x].front];
  const int P = fr.P, Q = fr.Q, k = a.k;
  cplx<R>* ts = red + 4 * 16 * NC;  // P x NC (adjoint)
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
  const cplx<R>* fac = a.factor + w * a.nfactor;
  cplx<R>* W = a.w + w * a.nw;
  const cplx<R>* z = a.z + w * a.nw + (int64_t)fr.row * k;
  cplx<R>* x = W + (int64_t)fr.row * k;
  const int* gr = a.grow + fr.bor;
  const int nrb = P / 16, nsplit = 4 / nrb;  // nrb <= 2 (kNdDownP)
  const int rb = wave % nrb, ks = wave / nrb;
  int col[NB];
#pragma unroll
  for (int c = 0; c < NB; c++) col[c] = min(8 * c + (l & 7), k - 1);
  v4<R> acc[NB];
  zero<R, NB>(acc);
  if (ks < nsplit)
    rows_mul<R, NB, true, ADJ, false>(acc, fac + (ADJ ? fr.f21 : fr.b12) + (int64_t)16 * rb * Q, Q,
                                      ks, Q / 16, nsplit, col,
                                      [&](int kk) { return W + (int64_t)gr[kk] * k; });
#pragma unroll
  for (int c = 0; c < NB; c++)
#pragma unroll
    for (int e = 0; e < 4; e++) part(red, NC, wave * 16 + Mf<R>::row(l, e), c) = acc[c][e];
  __syncthreads();
  for (int e = threadIdx.x; e < P * NC; e += 256) {
    const int r = e / NC, j = e % NC;
    cplx<R> v{(R)0, (R)0};
    if (j < k) {
      v = z[r * k + j];
      for (int s = 0; s < nsplit; s++) {
        const cplx<R> d = red[((s * nrb + (r >> 4)) * 16 + (r & 15)) * NC + j];
        v.re -= d.re;
        v.im -= d.im;
      }
      if (!ADJ) x[r * k + j] = v;
    }
    if (ADJ) ts[e] = v;
  }
  if (!ADJ) return;
  __syncthreads();
  if (wave >= nrb) return;
#pragma unroll
  for (int c = 0; c < NB; c++) col[c] = 8 * c + (l & 7);
  zero<R, NB>(acc);
  rows_mul<R, NB, true, true, true>(acc, fac + fr.a + (int64_t)16 * wave * P, P, 0, P / 16, 1, col,
                                    [&](int kk) { return ts + kk * NC; });
#pragma unroll
  for (int c = 0; c < NB; c++)
#pragma unroll
    for (int e = 0; e < 4; e++)
      if (col[c] < k) part(x, k, 16 * wave + Mf<R>::row(l, e), c) = acc[c][e];
}

// P > 64: b1 of 64 rows (into w, or z for the adjoint sweep)
template <typename R, typename IO>
__global__ __launch_bounds__(256) void k_nd_gather(SolveArgs<R, IO> a) {
  if (skipped(a.skip)) return;
  const int w = a.w0 + blockIdx.y;
  const NdTask t = a.tasks[blockIdx.x];
  const NdFront fr = a.fronts[t.front];
  const int k = a.k;
  const cplx<R>* ua = a.uin + w * a.nuin + (int64_t)fr.uA * k;
  const cplx<R>* ub = a.uin + w * a.nuin + (int64_t)fr.uB * k;
  const int r0 = kNdTile * t.i, nr = min(kNdTile, fr.P - r0);
  const int64_t at = w * a.nw + (int64_t)(fr.row + r0) * k;
  for (int e = threadIdx.x; e < nr * k; e += 256) {
    cplx<R> v = a.w[at + e];
    if (r0 + e / k < fr.p) {
      add(v, ua[(fr.baseA + r0) * k + e]);
      add(v, ub[(fr.baseB + r0) * k + e]);
    }
    (a.adjoint ? a.z : a.w)[at + e] = v;
  }
}

// 16 rows of one product, the workgroup's NW waves splitting its inner dimension.
// Eight where it is long (the border, or P > 256): with four, one shift's
// product over 1024 border rows took 34 us against 27.  Four where it is 256 or
// less, two chunks or so a wave (8 shifts, P = 128: 90 us against 137).
enum { ND_Z = 0,    // z = A w               (forward, up)
       ND_U = 1,    // u = pulled - F21 z    (adjoint: B12^H z)
       ND_X = 2,    // w = z - B12 w[border]  (adjoint: z -= F21^H w[border])
       ND_AH = 3 }; // w = A^H z             (adjoint, down)
template <typename R, typename IO, int NB, int MODE, bool ADJ, int NW>
__global__ __launch_bounds__(64 * NW, 2) void k_nd_rows(SolveArgs<R, IO> a) {
  if (skipped(a.skip)) return;
  constexpr int NC = 8 * NB;
  constexpr bool KF = MODE == ND_X || MODE == ND_AH;
  __shared__ cplx<R> red[NW * 16 * NC];
  const int w = a.w0 + blockIdx.y;
  const NdTask t = a.tasks[xcd_task()];
  const NdFront fr = a.fronts[t.front];
  const int P = fr.P, Q = fr.Q, k = a.k;
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
  cplx<R>* W = a.w + w * a.nw;
  cplx<R>* Z = a.z + w * a.nw;
  const int* gr = a.grow + fr.bor;
  const int64_t off = MODE == ND_Z || MODE == ND_AH ? fr.a
                      : (MODE == ND_U) != ADJ        ? fr.f21
                                                     : fr.b12;
  const int64_t ld = MODE == ND_U || MODE == ND_X ? Q : P;
  const int K = MODE == ND_X ? Q : P;
  const cplx<R>* X = a.factor + w * a.nfactor + off + (KF ? 16 * t.i * ld : 16 * t.i);
  int col[NB];
#pragma unroll
  for (int c = 0; c < NB; c++) col[c] = min(8 * c + (l & 7), k - 1);
  v4<R> acc[NB];
  zero<R, NB>(acc);
  const cplx<R>* V = (MODE == ND_Z ? W : Z) + (int64_t)fr.row * k;
  rows_mul<R, NB, KF, ADJ, false>(acc, X, ld, wave, K / 16, NW, col, [&](int kk) {
    return MODE == ND_X ? W + (int64_t)gr[kk] * k : V + (int64_t)kk * k;
  });
#pragma unroll
  for (int c = 0; c < NB; c++)
#pragma unroll
    for (int e = 0; e < 4; e++) part(red, NC, wave * 16 + Mf<R>::row(l, e), c) = acc[c][e];
  __syncthreads();
  for (int e = threadIdx.x; e < 16 * NC; e += 64 * NW) {
    const int r = 16 * t.i + e / NC, j = e % NC;
    if (j >= k) continue;
    cplx<R> v = red[e];
#pragma unroll
    for (int s = 1; s < NW; s++) add(v, red[s * 16 * NC + e]);
    const int64_t at = (int64_t)(fr.row + r) * k + j;
    if (MODE == ND_Z) {
      Z[at] = v;
    } else if (MODE == ND_AH) {
      W[at] = v;
    } else if (MODE == ND_X) {
      const cplx<R> z = Z[at];
      (ADJ ? Z : W)[at] = cplx<R>{z.re - v.re, z.im - v.im};
    } else {
      const int m = a.bmap[fr.bor + r];
      cplx<R> u{(R)0, (R)0};
      if (m >= 0) {
        u = a.uin[w * a.nuin + (int64_t)(((m & 1) ? fr.uB : fr.uA) + (m >> 1)) * k + j];
      }
      a.uout[w * a.nuout + (int64_t)(fr.urow + r) * k + j] = cplx<R>{u.re - v.re, u.im - v.im};
    }
  }
}

constexpr int kMaxY = 32768;  // shifts per launch (grid y)

// Workgroups per small front: its border (64 rows or columns a share at
// least) over several where the level's fronts leave CUs idle (two
// workgroups each on 256 CUs).
int shares(const NdLevel& lv, int64_t nw) {
  const int64_t wgs = std::max<int64_t>(1, lv.small.count * nw);
  return (int)std::max<int64_t>(1, std::min<int64_t>((lv.maxQ + 63) / 64, 512 / wgs));
}

template <typename R>
hipError_t factor_run(const OpDesc& op, const NdPlan& pl, const NdDevice& d, const double* omega,
                      int n_omega, uint32_t* status, hipStream_t s) {
  FactorArgs<R> a{};
  a.op = op;
  a.fronts = d.fronts;
  a.pdof = d.pdof;
  a.bmap = d.bmap;
  a.grow = d.grow;
  a.omega = omega;
  a.factor = (cplx<R>*)d.factor;
  a.temp = (cplx<R>*)d.temp;
  a.nfactor = pl.factor;
  a.ntemp = pl.temp;
  a.status = status;
  const size_t lds = tile_lds<R>();
  for (int w0 = 0; w0 < n_omega; w0 += kMaxY) {
    const unsigned nw = (unsigned)std::min(kMaxY, n_omega - w0);
    a.w0 = w0;
    auto run = [&](auto kernel, const NdSpan& sp, size_t shm, int zs = 1) {
      if (!sp.count) return;
      a.tasks = d.tasks + sp.first;
      hipLaunchKernelGGL(kernel, dim3(sp.count, nw, zs), dim3(256), shm, s, a);
    };
    for (int dep = (int)pl.levels.size() - 1; dep >= 0; dep--) {
      const NdLevel& lv = pl.levels[dep];
      a.schur_out = (cplx<R>*)d.schur[dep & 1];
      a.schur_in = (cplx<R>*)d.schur[~dep & 1];
      a.nout = pl.schur[dep & 1];
      a.nin = pl.schur[~dep & 1];
      if ((int64_t)lv.leafs[0].count * nw >= kNdLeafApart) {
        run(k_nd_leaf<R>, lv.leafs[0], leaf_lds(kNdLeafP));
        run(k_nd_leaf<R>, lv.leafs[1], leaf_lds(lv.leafP));
      } else {
        run(k_nd_leaf<R>, lv.leaf, leaf_lds(lv.leafP));
      }
      const size_t fl = front_lds<R>(lv.maxP);
      if (lv.maxP <= 16) run(k_nd_front<R, 16>, lv.small, fl, shares(lv, nw));
      else if (lv.maxP <= 32) run(k_nd_front<R, 32>, lv.small, fl, shares(lv, nw));
      else run(k_nd_front<R, 64>, lv.small, fl, shares(lv, nw));
      run(k_nd_assemble<R>, lv.assemble, lds);
      for (size_t k = 0; k < lv.panel.size(); k++) {
        run(k_nd_panel<R>, lv.panel[k], (size_t)kNdTile * kLd * sizeof(cplx<R>));
        run(k_nd_update<R>, lv.update[k], lds);
      }
      run(k_nd_border<R>, lv.border, 0);
      run(k_nd_schur<R>, lv.schur, 0);
    }
  }
  return hipGetLastError();
}

template <typename R, typename IO, int NB, bool ADJ>
hipError_t solve_run(const OpDesc& op, const NdPlan& pl, const NdDevice& d, int64_t n, int n_omega,
                     int k, int c0, int ktot, const void* Bm, int64_t bstride, void* X,
                     hipStream_t s, const uint32_t* skip) {
  constexpr int NC = 8 * NB;
  SolveArgs<R, IO> a{};
  a.op = op;
  a.fronts = d.fronts;
  a.pdof = d.pdof;
  a.bmap = d.bmap;
  a.grow = d.grow;
  a.factor = (const cplx<R>*)d.factor;
  a.w = (cplx<R>*)d.w;
  a.z = (cplx<R>*)d.z;
  a.nfactor = pl.factor;
  a.nw = (pl.rows + 1) * k;
  a.k = k;
  a.adjoint = ADJ;
  a.skip = skip;
  const unsigned rb = (unsigned)((pl.rows + 1 + kRowTile - 1) / kRowTile);
  const cplx<IO>* B = (const cplx<IO>*)Bm + (int64_t)c0 * n;
  cplx<IO>* Xo = (cplx<IO>*)X + (int64_t)c0 * n;
  a.B = B;
  a.X = Xo;
  a.n = n;
  a.bstride = bstride;
  a.xstride = (int64_t)ktot * n;
  for (int w0 = 0; w0 < n_omega; w0 += kMaxY) {
    const unsigned nw = (unsigned)std::min(kMaxY, n_omega - w0);
    a.w0 = w0;
    auto run = [&](auto kernel, const NdSpan& sp, size_t shm, int zs = 1, int threads = 256) {
      if (!sp.count) return;
      a.tasks = d.tasks + sp.first;
      a.qsplit = zs;
      hipLaunchKernelGGL(kernel, dim3(sp.count, nw, zs), dim3(threads), shm, s, a);
    };
    auto rows = [&](auto kernel, const NdSpan& sp, int waves) { run(kernel, sp, 0, 1, 64 * waves); };
    auto level = [&](int dep) -> const NdLevel& {
      a.uout = (cplx<R>*)d.u[dep & 1];
      a.uin = (cplx<R>*)d.u[~dep & 1];
      a.nuout = pl.urows[dep & 1] * k;
      a.nuin = pl.urows[~dep & 1] * k;
      return pl.levels[dep];
    };
    hipLaunchKernelGGL((k_nd_permute<R, IO, false>), dim3(rb, nw), dim3(256), 0, s, d.pdof, pl.rows, n,
                       k, bstride, B, (cplx<IO>*)nullptr, a.w, w0, skip);
    for (int dep = (int)pl.levels.size() - 1; dep >= 0; dep--) {
      const NdLevel& lv = level(dep);
      run(k_nd_leaf_up<R, IO, NB, ADJ>, lv.leaf, (size_t)lv.leafP * (NC + 1) * sizeof(cplx<R>));
      if (lv.small.count) {
        const size_t lds = (size_t)lv.maxP * NC * (ADJ ? 1 : 2) * sizeof(cplx<R>);
        if (lv.maxP <= 16) run(k_nd_up<R, IO, NB, ADJ, 16>, lv.small, lds, shares(lv, nw));
        else if (lv.maxP <= 32) run(k_nd_up<R, IO, NB, ADJ, 32>, lv.small, lds, shares(lv, nw));
        else run(k_nd_up<R, IO, NB, ADJ, 64>, lv.small, lds, shares(lv, nw));
      }
      run(k_nd_gather<R, IO>, lv.gather, 0);
      if (lv.largeP <= 256) {
        if (!ADJ) rows(k_nd_rows<R, IO, NB, ND_Z, ADJ, 4>, lv.rowsP, 4);
        rows(k_nd_rows<R, IO, NB, ND_U, ADJ, 4>, lv.rowsQ, 4);
      } else {
        if (!ADJ) rows(k_nd_rows<R, IO, NB, ND_Z, ADJ, 8>, lv.rowsP, 8);
        rows(k_nd_rows<R, IO, NB, ND_U, ADJ, 8>, lv.rowsQ, 8);
      }
    }
    for (int dep = 0; dep < (int)pl.levels.size(); dep++) {
      const NdLevel& lv = level(dep);
      run(k_nd_down<R, IO, NB, ADJ>, lv.down,
          (size_t)(64 + (ADJ ? lv.downP : 0)) * NC * sizeof(cplx<R>));
      rows(k_nd_rows<R, IO, NB, ND_X, ADJ, 8>, lv.rowsX, 8);
      if (ADJ && lv.largeP <= 256) rows(k_nd_rows<R, IO, NB, ND_AH, ADJ, 4>, lv.rowsX, 4);
      if (ADJ && lv.largeP > 256) rows(k_nd_rows<R, IO, NB, ND_AH, ADJ, 8>, lv.rowsX, 8);
      run(k_nd_leaf_down<R, IO, NB, ADJ>, lv.leaf, (size_t)lv.leafP * (NC + 1) * sizeof(cplx<R>));
    }
    hipLaunchKernelGGL((k_nd_permute<R, IO, true>), dim3(rb, nw), dim3(256), 0, s, d.pdof, pl.rows, n, k,
                       (int64_t)ktot * n, (const cplx<IO>*)nullptr, Xo, a.w, w0, skip);
  }
  return hipGetLastError();
}

template <typename R>
hipError_t prepare_r() {
  hipError_t e = hipSuccess;
  auto lds = [&](const void* fn, size_t bytes) {
    if (e == hipSuccess && bytes > 64 * 1024)
      e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  };
  lds((const void*)k_nd_leaf<R>, tile_lds<double>());
  lds((const void*)k_nd_front<R, 64>, tile_lds<double>());
  lds((const void*)k_nd_assemble<R>, tile_lds<R>());
  lds((const void*)k_nd_panel<R>, tile_lds<R>());
  lds((const void*)k_nd_update<R>, tile_lds<R>());
  return e;
}

}  // namespace

hipError_t nd_prepare() {
  const hipError_t e = prepare_r<double>();
  return e != hipSuccess ? e : prepare_r<float>();
}

hipError_t launch_nd_factor(const OpDesc& op, const NdPlan& pl, const NdDevice& d,
                            const double* omega, int n_omega, bool fp32, uint32_t* status,
                            hipStream_t s) {
  return fp32 ? factor_run<float>(op, pl, d, omega, n_omega, status, s)
              : factor_run<double>(op, pl, d, omega, n_omega, status, s);
}

hipError_t launch_nd_solve(const OpDesc& op, const NdPlan& pl, const NdDevice& d, int64_t n,
                           int n_omega, int k, int c0, int ktot, bool fp32, bool io32, int adjoint,
                           const void* Bm, int64_t bstride, void* X, hipStream_t s,
                           const uint32_t* skip) {
  auto go = [&](auto r, auto io, auto nb, auto adj) {
    return solve_run<decltype(r), decltype(io), decltype(nb)::value, decltype(adj)::value>(
        op, pl, d, n, n_omega, k, c0, ktot, Bm, bstride, X, s, skip);
  };
  auto by_adj = [&](auto r, auto io, auto nb) {
    return adjoint ? go(r, io, nb, std::true_type{}) : go(r, io, nb, std::false_type{});
  };
  auto by_nb = [&](auto r, auto io) {
    return k <= 8    ? by_adj(r, io, std::integral_constant<int, 1>{})
           : k <= 16 ? by_adj(r, io, std::integral_constant<int, 2>{})
           : k <= 24 ? by_adj(r, io, std::integral_constant<int, 3>{})
                     : by_adj(r, io, std::integral_constant<int, 4>{});
  };
  return !fp32 ? by_nb(0.0, 0.0) : io32 ? by_nb(0.0f, 0.0f) : by_nb(0.0f, 0.0);
}

}  // namespace rr
