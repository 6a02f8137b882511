// Wide sketches: the k x k steps of Algorithm 1 for 32 < k <= 512.
//
// The paper studies the accuracy against the sketch width k from 2 to 500
// (Section 3.2, Fig. 7).  Past k = 32 the LDS-resident kernels of
// rr_small.hip no longer hold a k x k matrix, so these keep the small
// matrices in global memory (L2-resident at this size) and tile the tall
// products through LDS:
//   * Gram G = Y^H Y in 32 x 32 tiles per row chunk, then summed over chunks;
//   * Cholesky G = R^H R and R^-1 in 32 x 32 blocks, one workgroup per shift;
//   * k x k products (composing the two CholQR passes, R^-1 W) in 32 x 32 tiles;
//   * tall products Y S (n x k by k x k) in 64 x 32 output tiles;
//   * the one-sided Jacobi SVD of R^H, one workgroup per shift, 16 lanes (from
//     k = 361 on 64) per column pair of the round-robin order (in LDS up to k =
//     100);
//   * column norms for eq. (9)'s sigma_j = ||M^-1 v_j||.
// Same steps and outputs as the narrow path (CholQR2, then the SVD of the
// k x k factor), with one difference: a Gram matrix that is not numerically
// positive definite latches ST_BREAKDOWN here (the narrow path falls back to
// shifted CholeskyQR3).
#include <algorithm>

#include "rr_mfma.h"

namespace rr {

namespace {

constexpr int kBT = 32;          // tile edge of the k x k blocks

__device__ __forceinline__ double2 bmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 bmulc(double2 a, double2 b) {  // conj(a) b
  return make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}

// part[w][chunk][i][j] = sum over the chunk's rows of conj(Y_i) Y_j for the
// 32 x 32 tile (I, J), J >= I, of every shift; Y is (n_omega, k, n).
__global__ __launch_bounds__(256) void k_gramb_partial(int64_t n, int k, const double2* Y,
                                                       int64_t rows, int nchunk, double2* part) {
  __shared__ double2 a[kBT][kBT + 1], b[kBT][kBT + 1];  // [row][col]
  const int nt = (k + kBT - 1) / kBT;
  const int I = blockIdx.x / nt, J = blockIdx.x % nt, chunk = blockIdx.y, w = blockIdx.z;
  if (J < I) return;
  const int64_t r0 = chunk * rows, r1 = min(n, r0 + rows);
  const double2* Yw = Y + (int64_t)w * k * n;
  const int t = threadIdx.x, oi = t >> 3, oj = (t & 7) * 4;  // outputs (oi, oj .. oj+3)
  double2 acc[4] = {};
  for (int64_t rb = r0; rb < r1; rb += kBT) {
    for (int e = t; e < kBT * kBT; e += 256) {
      const int c = e / kBT, rr = e % kBT;  // consecutive threads: consecutive rows
      const int64_t row = rb + rr;
      const int ca = kBT * I + c, cb = kBT * J + c;
      a[rr][c] = (row < r1 && ca < k) ? Yw[(int64_t)ca * n + row] : make_double2(0, 0);
      b[rr][c] = (row < r1 && cb < k) ? Yw[(int64_t)cb * n + row] : make_double2(0, 0);
    }
    __syncthreads();
    for (int rr = 0; rr < kBT; rr++) {
      const double2 x = a[rr][oi];
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const double2 p = bmulc(x, b[rr][oj + q]);
        acc[q].x += p.x;
        acc[q].y += p.y;
      }
    }
    __syncthreads();
  }
  double2* out = part + ((int64_t)w * nchunk + chunk) * k * k;
  const int gi = kBT * I + oi;
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const int gj = kBT * J + oj + q;
    if (gi < k && gj < k) out[(int64_t)gi * k + gj] = acc[q];
  }
}

// G[w] (k x k, row-major, leading dimension k) = sum over chunks, the lower
// triangle mirrored from the upper one (G is Hermitian).
__global__ void k_gramb_reduce(int k, int nchunk, const double2* part, int64_t sG, double2* G) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int w = blockIdx.y;
  if (idx >= (int64_t)k * k) return;
  const int i = (int)(idx / k), j = (int)(idx % k);
  const bool up = j >= i;
  const int64_t src = up ? (int64_t)i * k + j : (int64_t)j * k + i;
  double2 s = make_double2(0, 0);
  for (int c = 0; c < nchunk; c++) {
    const double2 p = part[((int64_t)w * nchunk + c) * k * k + src];
    s.x += p.x;
    s.y += p.y;
  }
  G[w * sG + idx] = up ? s : make_double2(s.x, -s.y);
}

// A 32 x 32 complex product of blocks in LDS on the FP64 matrix cores: waves 0
// to 7 of the workgroup take a 16 x 16 tile's real or imaginary part each (the
// others wait).  CT: X^H Y, else X Y.
typedef Mf<double>::v4 BlockAcc;
typedef double2 Block[kBT][kBT + 1];
template <bool CT>
__device__ __forceinline__ void block_mul(BlockAcc& acc, const Block& X, const Block& Y) {
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, i = l & 15, g = l >> 4;
  if (wave >= 8) return;
  const bool im = wave & 1;
  const int r0 = 16 * (wave >> 2), c0 = 16 * ((wave >> 1) & 1);
#pragma unroll
  for (int s = 0; s < kBT / 4; s++) {
    const int kk = 4 * s + g;
    const double2 x = CT ? X[kk][r0 + i] : X[r0 + i][kk], y = Y[kk][c0 + i];
    acc = Mf<double>::op(x.x, im ? y.y : y.x, acc);
    acc = Mf<double>::op(im != CT ? x.y : -x.y, im ? y.x : y.y, acc);
  }
}
__device__ __forceinline__ void block_store(const BlockAcc& acc, Block& Z) {
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
  if (wave >= 8) return;
  const int r0 = 16 * (wave >> 2), c = 16 * ((wave >> 1) & 1) + (l & 15);
#pragma unroll
  for (int e = 0; e < 4; e++) {
    double2& z = Z[r0 + Mf<double>::row(l, e)][c];
    if (wave & 1) z.y = acc[e];
    else z.x = acc[e];
  }
}

// G = R^H R (R upper, real positive diagonal) and R^-1, one workgroup per
// shift, in 32 x 32 blocks: a diagonal block is factored and inverted in LDS
// (one barrier per step, as in the narrow path), its block row multiplied by
// the inverse, the blocks below updated; then R^-1 by block back-substitution
// with the diagonal inverses.  A thread holds one element of a block.  The
// chain is k short steps in LDS and (k / 32)^3 / 3 block products, where the
// unblocked form took k steps through global memory and one thread per column
// of R^-1: 957 us at k = 100; 211 with the products by one thread an element,
// which wait for LDS, and a barrier for each step of the inverses, 154 now.  A
// pivot that is not positive latches ST_BREAKDOWN and is taken as 1 (the results
// stay finite).
__global__ __launch_bounds__(1024) void k_cholb(int k, int64_t sM, const double2* G, double2* R,
                                                double2* Rinv, uint32_t* status) {
  __shared__ Block S0, S1, S2;
  const int w = blockIdx.x, t = threadIdx.x, ti = t >> 5, tj = t & 31;
  const int nt = (k + kBT - 1) / kBT;
  const double2* Gw = G + w * sM;
  double2* Rw = R + w * sM;
  double2* Xw = Rinv + w * sM;
  const double2 none = make_double2(0, 0);
  auto get = [&](const double2* M, int i, int j) {
    return i < k && j < k ? M[(int64_t)i * k + j] : none;
  };
  auto put = [&](double2* M, int i, int j, double2 v) {
    if (i < k && j < k) M[(int64_t)i * k + j] = v;
  };
  for (int64_t e = t; e < (int64_t)k * k; e += 1024) {
    const int i = (int)(e / k), j = (int)(e % k);
    Rw[e] = j >= i ? Gw[e] : none;
    Xw[e] = none;
  }
  __syncthreads();
  bool bad = false;
  for (int J = 0; J < nt; J++) {
    const int j0 = kBT * J, jb = min(kBT, k - j0);
    S0[ti][tj] = ti < jb && tj < jb ? get(Rw, j0 + ti, j0 + tj)
                                    : make_double2(ti == tj ? 1.0 : 0.0, 0.0);
    __syncthreads();
    for (int j = 0; j < jb; j++) {
      const double d = S0[j][j].x;
      const bool no = !(d > 0.0) || !isfinite(d);
      bad |= no;
      const double rd = no ? 1.0 : 1.0 / d;
      if (ti > j && tj >= ti) {
        // (scaled before the product, as in the narrow path)
        const double2 gc = S0[j][tj];
        const double2 p = bmulc(S0[j][ti], make_double2(gc.x * rd, gc.y * rd));
        S0[ti][tj].x -= p.x;
        S0[ti][tj].y -= p.y;
      }
      __syncthreads();
    }
    const double d = S0[ti][ti].x;
    const double r = !(d > 0.0) || !isfinite(d) ? 1.0 : sqrt(d);
    double2 v = S0[ti][tj];
    v = tj > ti ? make_double2(v.x / r, v.y / r) : make_double2(tj == ti ? r : 0.0, 0.0);
    __syncthreads();
    S0[ti][tj] = v;
    put(Rw, j0 + ti, j0 + tj, v);
    __syncthreads();
    invert_upper(S0, S1, kBT);
    __syncthreads();
    put(Xw, j0 + ti, j0 + tj, S1[ti][tj]);
    for (int C = J + 1; C < nt; C++) {  // block row J: R_JC = S1^H G_JC
      S2[ti][tj] = get(Rw, j0 + ti, kBT * C + tj);
      __syncthreads();
      BlockAcc acc = {};
      block_mul<true>(acc, S1, S2);
      __syncthreads();
      block_store(acc, S2);
      __syncthreads();
      put(Rw, j0 + ti, kBT * C + tj, S2[ti][tj]);
      __syncthreads();
    }
    for (int B = J + 1; B < nt; B++) {  // G_BC -= R_JB^H R_JC, C >= B
      S0[ti][tj] = get(Rw, j0 + ti, kBT * B + tj);
      for (int C = B; C < nt; C++) {
        S2[ti][tj] = get(Rw, j0 + ti, kBT * C + tj);
        const double2 g = get(Rw, kBT * B + ti, kBT * C + tj);
        __syncthreads();
        BlockAcc acc = {};
        block_mul<true>(acc, S0, S2);
        __syncthreads();
        block_store(acc, S2);
        __syncthreads();
        const double2 s = S2[ti][tj];
        put(Rw, kBT * B + ti, kBT * C + tj,
            C > B || tj >= ti ? make_double2(g.x - s.x, g.y - s.y) : none);
        __syncthreads();
      }
    }
  }
  for (int J = 1; J < nt; J++)
    for (int I = J - 1; I >= 0; I--) {  // X_IJ = -X_II sum_L R_IL X_LJ
      BlockAcc acc = {};
      for (int L = I + 1; L <= J; L++) {
        S0[ti][tj] = get(Rw, kBT * I + ti, kBT * L + tj);
        S1[ti][tj] = get(Xw, kBT * L + ti, kBT * J + tj);
        __syncthreads();
        block_mul<false>(acc, S0, S1);
        __syncthreads();
      }
      block_store(acc, S2);
      S0[ti][tj] = get(Xw, kBT * I + ti, kBT * I + tj);
      __syncthreads();
      acc = {};
      block_mul<false>(acc, S0, S2);
      block_store(acc, S1);
      __syncthreads();
      const double2 x = S1[ti][tj];
      put(Xw, kBT * I + ti, kBT * J + tj, make_double2(-x.x, -x.y));
      __syncthreads();
    }
  if (t == 0 && bad) latch(status, ST_BREAKDOWN);
}

// C[w] = A[w] B[w] (k x k, row-major, leading dimension k), 32 x 32 tiles.
__global__ __launch_bounds__(256) void k_sgemm(int k, int64_t sM, const double2* A,
                                               const double2* B, double2* C) {
  __shared__ double2 a[kBT][kBT + 1], b[kBT][kBT + 1];
  const int I = blockIdx.x, J = blockIdx.y, w = blockIdx.z;
  const int t = threadIdx.x, oi = t >> 3, oj = (t & 7) * 4;
  const double2* Aw = A + w * sM;
  const double2* Bw = B + w * sM;
  double2 acc[4] = {};
  for (int L = 0; L < k; L += kBT) {
    for (int e = t; e < kBT * kBT; e += 256) {
      const int i = e / kBT, j = e % kBT;
      const int ar = kBT * I + i, ac = L + j, br = L + i, bc = kBT * J + j;
      a[i][j] = (ar < k && ac < k) ? Aw[(int64_t)ar * k + ac] : make_double2(0, 0);
      b[i][j] = (br < k && bc < k) ? Bw[(int64_t)br * k + bc] : make_double2(0, 0);
    }
    __syncthreads();
    for (int l = 0; l < kBT; l++) {
      const double2 x = a[oi][l];
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const double2 p = bmul(x, b[l][oj + q]);
        acc[q].x += p.x;
        acc[q].y += p.y;
      }
    }
    __syncthreads();
  }
  const int gi = kBT * I + oi;
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const int gj = kBT * J + oj + q;
    if (gi < k && gj < k) C[w * sM + (int64_t)gi * k + gj] = acc[q];
  }
}

// Out = Y S per shift: Y (n_omega, k, n), S (k x k, row-major), Out like Y
// (not aliasing it); 64 rows x 32 output columns per workgroup.
__global__ __launch_bounds__(256) void k_applyb(int64_t n, int k, const double2* Y, int64_t sS,
                                                const double2* S, double2* Out) {
  __shared__ double2 ya[kBT][64 + 1];  // [col][row]
  __shared__ double2 sa[kBT][kBT + 1];
  const int64_t r0 = blockIdx.x * (int64_t)64;
  const int J = blockIdx.y, w = blockIdx.z;
  const double2* Yw = Y + (int64_t)w * k * n;
  const double2* Sw = S + w * sS;
  const int t = threadIdx.x, orow = t & 63, oc = (t >> 6) * 8;  // 8 columns per thread
  double2 acc[8] = {};
  for (int L = 0; L < k; L += kBT) {
    for (int e = t; e < kBT * 64; e += 256) {
      const int c = e / 64, rr = e % 64;
      const int64_t row = r0 + rr;
      ya[c][rr] = (row < n && L + c < k) ? Yw[(int64_t)(L + c) * n + row] : make_double2(0, 0);
    }
    for (int e = t; e < kBT * kBT; e += 256) {
      const int i = e / kBT, j = e % kBT;
      sa[i][j] = (L + i < k && kBT * J + j < k) ? Sw[(int64_t)(L + i) * k + kBT * J + j]
                                               : make_double2(0, 0);
    }
    __syncthreads();
    for (int l = 0; l < kBT; l++) {
      const double2 x = ya[l][orow];
#pragma unroll
      for (int q = 0; q < 8; q++) {
        const double2 p = bmul(x, sa[l][oc + q]);
        acc[q].x += p.x;
        acc[q].y += p.y;
      }
    }
    __syncthreads();
  }
  const int64_t row = r0 + orow;
  if (row >= n) return;
#pragma unroll
  for (int q = 0; q < 8; q++) {
    const int col = kBT * J + oc + q;
    if (col < k) Out[((int64_t)w * k + col) * n + row] = acc[q];
  }
}

// One-sided (Hestenes) Jacobi SVD of A = R^H (k x k) per shift, one
// workgroup: the pairs of each round follow the round-robin order, 16 lanes a
// pair (LN), so that a round of up to 64 pairs runs at once.  The rotation is the
// narrow path's: with gamma = a_p^H a_q and e = gamma / |gamma|, the columns
// [a_p, conj(e) a_q] are rotated by the real Jacobi angle of [[alpha,
// |gamma|], [|gamma|, beta]].  The columns start in descending order of their
// norms, a rotation's larger column staying in front (8 sweeps against 10 where
// the iteration has already sorted the spectrum).  Then sigma_c = ||a_c||, sorted
// descending (ranks counted in parallel), Ut = A diag(1/sigma), W = J, both
// permuted; Rinv W is formed by k_sgemm.
//
// Bound by the latency of its rounds (m - 1 a sweep).  In LDS mode (m <= 100:
// 160 KB) A stays in LDS, a pair's columns in registers for the round, and
// kJacobiParts workgroups per shift compute the same rotations of A while each
// applies them to its own rows of J, at most 16 (in global scratch, loaded at
// the round's start): one workgroup's J traffic, 320 KB a round, took longer
// than the rotations.  Beyond m = 100 A is in global scratch too (column c
// contiguous) and one workgroup does everything.  At k = 100: 11.4 ms with A
// in global scratch and a wave per pair, 5.1 ms with all of J in one
// workgroup, 3.85 with the sums by shuffles and the columns unsorted, 2.97 ms
// now; at k = 102, with A in global scratch, 6.9 ms, at 128 11.2.
//
// In global scratch a pair takes 16 lanes up to m = 360 and a wave beyond, where
// the columns no longer stay in the caches near the CU and the longer runs of
// whole lines win (gains of one shift, 16 / 64 lanes: k = 300 165 / 174 ms, 360
// 289 / 307, 372 423 / 369, 450 847 / 723, 500 1146 / 950).
constexpr int kJacobiLds = 100;  // largest m whose A fits the CU's LDS
constexpr int kJacobiNarrow = 360;
constexpr int kJacobiEl = (kJacobiLds + 15) / 16;
constexpr int kJacobiParts = (kJacobiLds + 15) / 16;
// The place of v[c] in the descending order (stable, NaNs first), each place once
__device__ __forceinline__ int descending_rank(const double* v, int n, int c) {
  int r = 0;
  const bool cn = isnan(v[c]);
  for (int d = 0; d < n; d++) {
    const bool dn = isnan(v[d]);
    r += (dn && !cn) || v[d] > v[c] || ((v[d] == v[c] || (dn && cn)) && d < c);
  }
  return r;
}
// The sum over a pair's LN lanes, in every lane.
template <int LN>
__device__ __forceinline__ double pair_sum(double v) {
  v = sum16(v);
  if constexpr (LN == 64) {
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
  }
  return v;
}
template <bool LDS, int LN>
__global__ __launch_bounds__(1024) void k_jacobib(int k, int64_t sM, const double2* R, double2* A,
                                                  double2* Jm, double* sigma, double2* Ut,
                                                  double2* W, double* sv, int* rank,
                                                  uint32_t* status, int max_sweeps) {
  extern __shared__ __align__(16) char smem_raw[];
  __shared__ int rotated;
  const int w = blockIdx.x;
  const int m = (k + 1) & ~1;  // even number of players (a zero column pads odd k)
  const int part = blockIdx.y, nparts = gridDim.y;
  const int j0 = LDS ? m * part / nparts : 0;  // this workgroup's rows of J
  const int j1 = LDS ? m * (part + 1) / nparts : m;
  const double2* Rw = R + w * sM;
  double2* Aw = LDS ? reinterpret_cast<double2*>(smem_raw) : A + (int64_t)w * m * m;
  double2* Jw = Jm + (int64_t)w * m * m;
  double* svw = sv + (int64_t)w * m;
  int* rk = rank + (int64_t)w * m;
  // every part has the same norms and ranks, in scratch of its own
  svw += (int64_t)part * gridDim.x * m;
  rk += (int64_t)part * gridDim.x * m;
  const int group = threadIdx.x / LN, lane = threadIdx.x % LN, ngroup = blockDim.x / LN;
  for (int c = group; c < m; c += ngroup) {
    double s = 0;
    for (int a = lane; a < k && c < k; a += LN) {
      const double2 v = Rw[(int64_t)c * k + a];
      s += v.x * v.x + v.y * v.y;
    }
    s = pair_sum<LN>(s);
    if (lane == 0) svw[c] = c < k ? s : -1.0;  // the zero column comes last
  }
  __syncthreads();
  for (int c = threadIdx.x; c < m; c += blockDim.x) rk[c] = descending_rank(svw, m, c);
  __syncthreads();
  for (int64_t e = threadIdx.x; e < (int64_t)m * m; e += blockDim.x) {
    const int c = (int)(e / m), a = (int)(e % m);  // column c, row a
    const int64_t to = (int64_t)rk[c] * m + a;
    double2 v = make_double2(0, 0);
    if (a < k && c < k) {
      const double2 rc = Rw[(int64_t)c * k + a];  // A[a][c] = conj(R[c][a])
      v = make_double2(rc.x, -rc.y);
    }
    Aw[to] = v;
    if (a >= j0 && a < j1) Jw[to] = make_double2(a == c ? 1.0 : 0.0, 0.0);
  }
  __syncthreads();
  const int npair = m / 2;
  int sweep = 0;
  for (; sweep < max_sweeps; sweep++) {
    if (threadIdx.x == 0) rotated = 0;
    __syncthreads();
    for (int rnd = 0; rnd < m - 1; rnd++) {
      for (int pr = group; pr < npair; pr += ngroup) {
        int p, q;
        if (pr == 0) {
          p = 0;
          q = 1 + rnd % (m - 1);
        } else {
          p = 1 + (pr + rnd) % (m - 1);
          q = 1 + (m - 1 - pr + rnd) % (m - 1);
        }
        if (p > q) { const int tt = p; p = q; q = tt; }
        double2* ap = Aw + (int64_t)p * m;
        double2* aq = Aw + (int64_t)q * m;
        double2* jp = Jw + (int64_t)p * m;
        double2* jq = Jw + (int64_t)q * m;
        double2 ax[kJacobiEl], ay[kJacobiEl], jx, jy;
        double al = 0, be = 0, gr = 0, gi = 0;
        auto gram = [&](double2 x, double2 y) {
          al += x.x * x.x + x.y * x.y;
          be += y.x * y.x + y.y * y.y;
          gr += x.x * y.x + x.y * y.y;
          gi += x.x * y.y - x.y * y.x;
        };
        if constexpr (LDS) {
          const int jr = min(j0 + lane, m - 1);
          jx = jp[jr];
          jy = jq[jr];
#pragma unroll
          for (int u = 0; u < kJacobiEl; u++) {
            const int r = lane + 16 * u;
            ax[u] = r < m ? ap[r] : make_double2(0, 0);
            ay[u] = r < m ? aq[r] : make_double2(0, 0);
            gram(ax[u], ay[u]);
          }
        } else {
          for (int r = lane; r < m; r += LN) gram(ap[r], aq[r]);
        }
        al = pair_sum<LN>(al);
        be = pair_sum<LN>(be);
        gr = pair_sum<LN>(gr);
        gi = pair_sum<LN>(gi);
        double er, ei, c, sn;
        if (jacobi_angle(al, be, gr, gi, er, ei, c, sn)) {
          auto rotate = [&](double2& x, double2& y) {
            const double2 yp = make_double2(y.x * er - y.y * ei, y.x * ei + y.y * er);
            y = make_double2(sn * x.x + c * yp.x, sn * x.y + c * yp.y);
            x = make_double2(c * x.x - sn * yp.x, c * x.y - sn * yp.y);
          };
          if constexpr (LDS) {
#pragma unroll
            for (int u = 0; u < kJacobiEl; u++) {
              const int r = lane + 16 * u;
              rotate(ax[u], ay[u]);
              if (r < m) {
                ap[r] = ax[u];
                aq[r] = ay[u];
              }
            }
            if (j0 + lane < j1) {
              rotate(jx, jy);
              jp[j0 + lane] = jx;
              jq[j0 + lane] = jy;
            }
          } else {
            for (int r = lane; r < m; r += LN) {
              double2 x = ap[r], y = aq[r];
              rotate(x, y);
              ap[r] = x;
              aq[r] = y;
              x = jp[r];
              y = jq[r];
              rotate(x, y);
              jp[r] = x;
              jq[r] = y;
            }
          }
          if (lane == 0) rotated = 1;
        }
      }
      __syncthreads();
    }
    if (!rotated) break;
    __syncthreads();
  }
  if (threadIdx.x == 0 && rotated && part == 0) latch(status, ST_SVD_NOT_CONVERGED);
  for (int c = threadIdx.x; c < k; c += blockDim.x) {
    double s = 0;
    for (int a = 0; a < k; a++) {
      const double2 v = Aw[(int64_t)c * m + a];
      s += v.x * v.x + v.y * v.y;
    }
    svw[c] = sqrt(s);
    if (!isfinite(svw[c])) latch(status, ST_NONFINITE);
  }
  __syncthreads();
  for (int c = threadIdx.x; c < k; c += blockDim.x) rk[c] = descending_rank(svw, k, c);
  __syncthreads();
  for (int64_t e = threadIdx.x; e < (int64_t)k * k; e += blockDim.x) {
    const int src = (int)(e / k), a = (int)(e % k);  // source column, row
    if (a < j0 || a >= j1) continue;
    const int c = rk[src];
    const double s = svw[src];
    const double2 u = Aw[(int64_t)src * m + a];
    Ut[w * sM + (int64_t)a * k + c] = s > 0 ? make_double2(u.x / s, u.y / s) : make_double2(0, 0);
    W[w * sM + (int64_t)a * k + c] = Jw[(int64_t)src * m + a];
    if (a == 0) sigma[(int64_t)w * k + c] = s;
  }
}

// sigma[w][c] = ||X_c|| and, when U != NULL, U_c = X_c / sigma (eq. 9), one
// workgroup per (column, shift).
__global__ __launch_bounds__(256) void k_colnormb(int64_t n, int k, const double2* X,
                                                  double* sigma, double2* U, uint32_t* status) {
  __shared__ double red[4];
  __shared__ double tot;
  const int c = blockIdx.x, w = blockIdx.y;
  const double2* x = X + ((int64_t)w * k + c) * n;
  double s = 0;
  for (int64_t r = threadIdx.x; r < n; r += 256) s += x[r].x * x[r].x + x[r].y * x[r].y;
  for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    tot = sqrt(red[0] + red[1] + red[2] + red[3]);
    sigma[(int64_t)w * k + c] = tot;
    if (!isfinite(tot)) latch(status, ST_NONFINITE);
  }
  __syncthreads();
  if (!U) return;
  const double inv = tot > 0 ? 1.0 / tot : 0.0;
  double2* u = U + ((int64_t)w * k + c) * n;
  for (int64_t r = threadIdx.x; r < n; r += 256) u[r] = make_double2(x[r].x * inv, x[r].y * inv);
}

// Columns [c0, c0 + kg) of a wide block (shift w at w * wstride, k columns)
// to a narrow block (n_omega, kg, n) (gather), or back (scatter).
__global__ void k_cols_copy(int64_t n, int k, int64_t wstride, int c0, int kg, const double2* src,
                            double2* dst, int gather) {
  const int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int c = blockIdx.y, w = blockIdx.z;
  if (r >= n) return;
  const int64_t wide = w * wstride + (int64_t)(c0 + c) * n + r;
  const int64_t narrow = ((int64_t)w * kg + c) * n + r;
  if (gather) dst[narrow] = src[wide];
  else dst[wide] = src[narrow];
}

}  // namespace

// Row chunks of the tiled Gram matrix: at least 128 rows each, and with the
// nt (nt + 1) / 2 tiles about 512 workgroups (at least 16 chunks, at most 64).
// At n = 4096, k = 100 two chunks of 2048 rows (20 workgroups) took 342 us.
int gramb_chunks(int64_t n, int k) {
  const int nt = (k + kBT - 1) / kBT;
  const int want = std::min(64, std::max(16, 1024 / (nt * (nt + 1))));
  return (int)std::min<int64_t>(want, (n + 127) / 128);
}
// complex elements of partial sums per shift for any k <= k_max
size_t gramb_partial(int64_t n, int k_max) {
  size_t most = 0;
  for (int nt = 1; nt <= (k_max + kBT - 1) / kBT; nt++) {
    const size_t k = std::min(kBT * nt, k_max);
    most = std::max(most, (size_t)gramb_chunks(n, (int)k) * k * k);
  }
  return most;
}
// dynamic LDS of the wide kernels, set when a handle is created
hipError_t prepare_big() {
  return hipFuncSetAttribute((const void*)k_jacobib<true, 16>,
                             hipFuncAttributeMaxDynamicSharedMemorySize,
                             kJacobiLds * kJacobiLds * (int)sizeof(double2));
}

namespace {

// Gram, Cholesky and R^-1 of Y into G, R, Rinv (k x k per shift, stride sM)
void gram_chol(int64_t n, int n_omega, int k, const double* Y, SmallWs& ws, double* G, double* R,
               double* Rinv, uint32_t* status, hipStream_t s) {
  const int nt = (k + kBT - 1) / kBT, nc = gramb_chunks(n, k);
  const int64_t rows = (n + nc - 1) / nc, sM = (int64_t)ws.kmax * ws.kmax;
  hipLaunchKernelGGL(k_gramb_partial, dim3(nt * nt, nc, n_omega), dim3(256), 0, s, n, k,
                     (const double2*)Y, rows, nc, (double2*)ws.partial);
  hipLaunchKernelGGL(k_gramb_reduce, dim3((unsigned)(((int64_t)k * k + 255) / 256), n_omega),
                     dim3(256), 0, s, k, nc, (const double2*)ws.partial, sM, (double2*)G);
  hipLaunchKernelGGL(k_cholb, dim3(n_omega), dim3(1024), 0, s, k, sM, (const double2*)G,
                     (double2*)R, (double2*)Rinv, status);
}

void sgemm(int n_omega, int k, int64_t sM, const double* A, const double* B, double* C,
           hipStream_t s) {
  const int nt = (k + kBT - 1) / kBT;
  hipLaunchKernelGGL(k_sgemm, dim3(nt, nt, n_omega), dim3(256), 0, s, k, sM, (const double2*)A,
                     (const double2*)B, (double2*)C);
}

void applyb(int64_t n, int n_omega, int k, const double* Y, int64_t sS, const double* S,
            double* Out, hipStream_t s) {
  const int nt = (k + kBT - 1) / kBT;
  hipLaunchKernelGGL(k_applyb, dim3((unsigned)((n + 63) / 64), nt, n_omega), dim3(256), 0, s, n,
                     k, (const double2*)Y, sS, (const double2*)S, (double2*)Out);
}

}  // namespace

// Y <- Q = Y R^-1 by two Cholesky QR passes (Y = Q R, R = R2 R1 into ws.R,
// R^-1 = R1^-1 R2^-1 into ws.Rinv); tmp: a block like Y.
hipError_t launch_cholqr2_big(int64_t n, int n_omega, int k, double* Y, double* tmp, SmallWs& ws,
                              uint32_t* status, hipStream_t s) {
  if (k > ws.kmax || k > kMaxWideK || !ws.big1 || !ws.big2) return hipErrorInvalidValue;
  const int64_t sM = (int64_t)ws.kmax * ws.kmax;
  gram_chol(n, n_omega, k, Y, ws, ws.G, ws.big1, ws.big2, status, s);   // R1, R1^-1
  applyb(n, n_omega, k, Y, sM, ws.big2, tmp, s);                          // Q1 = Y R1^-1
  gram_chol(n, n_omega, k, tmp, ws, ws.G, ws.W, ws.Ut, status, s);      // R2, R2^-1
  applyb(n, n_omega, k, tmp, sM, ws.Ut, Y, s);                            // Q = Q1 R2^-1
  sgemm(n_omega, k, sM, ws.W, ws.big1, ws.R, s);                          // R = R2 R1
  sgemm(n_omega, k, sM, ws.big2, ws.Ut, ws.Rinv, s);                      // R^-1 = R1^-1 R2^-1
  return hipGetLastError();
}

// The wide counterpart of launch_small_svd: Z = Qz R (two Cholesky QR passes
// on a copy in tmp), the Jacobi SVD R^H = Ut S W^H, V = Z R^-1 W and, when
// Uqu != NULL, U = Q Ut (eq. 8).
hipError_t launch_small_svd_big(int64_t n, int n_omega, int k, const double* Z, const double* Q,
                                double* sigma, double* V, double* Uqu, double* tmp,
                                SmallWs& ws, uint32_t* status, hipStream_t s) {
  if (k > ws.kmax || k > kMaxWideK || !ws.big1 || !ws.big2) return hipErrorInvalidValue;
  const int64_t sM = (int64_t)ws.kmax * ws.kmax;
  hipError_t e = launch_kcopy((int64_t)n_omega * k * n, Z, tmp, s);
  if (e != hipSuccess) return e;
  // V is free until the end: it holds the second pass's Q1 R2^-1 scratch
  gram_chol(n, n_omega, k, tmp, ws, ws.G, ws.big1, ws.big2, status, s);
  applyb(n, n_omega, k, tmp, sM, ws.big2, V, s);
  gram_chol(n, n_omega, k, V, ws, ws.G, ws.W, ws.Ut, status, s);
  sgemm(n_omega, k, sM, ws.W, ws.big1, ws.R, s);      // R = R2 R1
  sgemm(n_omega, k, sM, ws.big2, ws.Ut, ws.Rinv, s);  // R^-1 = R1^-1 R2^-1
  const int m = (k + 1) & ~1;
  // Jacobi scratch: A and J (m x m each; big1 / big2 hold (kmax + 1)^2 per
  // shift), the column norms and ranks in the partial-sum buffer
  const int parts = m <= kJacobiLds ? kJacobiParts : 1;
  double* sv = ws.partial;
  int* rank = reinterpret_cast<int*>(ws.partial + (size_t)parts * n_omega * m);
  auto jacobi = [&](auto kernel, size_t lds) {
    hipLaunchKernelGGL(kernel, dim3(n_omega, parts), dim3(1024), lds, s, k, sM,
                       (const double2*)ws.R, (double2*)ws.big1, (double2*)ws.big2, sigma,
                       (double2*)ws.Ut, (double2*)ws.W, sv, rank, status, ws.jacobi_sweeps);
  };
  if (m <= kJacobiLds) jacobi(k_jacobib<true, 16>, (size_t)m * m * sizeof(double2));
  else if (m <= kJacobiNarrow) jacobi(k_jacobib<false, 16>, 0);
  else jacobi(k_jacobib<false, 64>, 0);
  sgemm(n_omega, k, sM, ws.Rinv, ws.W, ws.G, s);  // Tv = R^-1 W
  applyb(n, n_omega, k, Z, sM, ws.G, V, s);        // V = Z Tv
  if (Uqu) applyb(n, n_omega, k, Q, sM, ws.Ut, Uqu, s);
  return hipGetLastError();
}

hipError_t launch_colnorm_big(int64_t n, int n_omega, int k, const double* X, double* sigma,
                              double* U, uint32_t* status, hipStream_t s) {
  hipLaunchKernelGGL(k_colnormb, dim3(k, n_omega), dim3(256), 0, s, n, k, (const double2*)X,
                     sigma, (double2*)U, status);
  return hipGetLastError();
}

hipError_t launch_cols_copy(int64_t n, int n_omega, int k, int64_t wstride, int c0, int kg,
                            const double* src, double* dst, bool gather, hipStream_t s) {
  hipLaunchKernelGGL(k_cols_copy, dim3((unsigned)((n + 255) / 256), kg, n_omega), dim3(256), 0, s,
                     n, k, wstride, c0, kg, (const double2*)src, (double2*)dst, gather ? 1 : 0);
  return hipGetLastError();
}

}  // namespace rr
