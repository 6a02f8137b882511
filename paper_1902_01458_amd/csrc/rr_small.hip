// Tall-skinny and k x k kernels (all FP64): Cholesky QR applied twice for the
// orthonormal basis of Algorithm 1 step 3, the reduced SVD of step 5 (one-sided
// Jacobi on the k x k triangular factor), the tall-small products that form
// V = Qz W and U = Q Ut (eq. 8), the column norms of steps 7-9 and the
// convergence test of the mixed-precision refinement.
//
// Reductions over n use a fixed chunking and a fixed summation order, so the
// results are bitwise reproducible from run to run.
#include <algorithm>
#include <type_traits>

#include "rr_mfma.h"

namespace rr {

constexpr int kChunkRows = 2048;  // rows per partial-sum chunk (norms)
constexpr int KM = 32;            // largest sketch width the k x k kernels take

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cmulc(double2 a, double2 b) {  // conj(a) * b
  return make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}

// partial[w][chunk] = (Y_c T)^H (Y_c T) over the chunk's rows, where T is the
// k x k matrix Tm[w] (MUL; identity otherwise).  Y: (n_omega, k, n).
//
// In real form on the FP64 matrix cores: with the 2k real columns [re im] of
// every column of Y, H = Yr^T Yr holds all four real products of each complex
// one, and only its 16 x 16 blocks on and above the diagonal are formed (6 at
// k = 20, i.e. 6 MFMAs per 4 rows).  For a Gram matrix both MFMA operands have
// the same lane layout, so each element is loaded once.  With MUL a wave first
// multiplies its 16 rows by T, whose operand stays in registers; the product's
// accumulator layout is the Gram product's operand layout, so nothing moves.
// Each wave takes every fourth group of 16 rows; the waves' sums are added in
// order, so results are bitwise reproducible, and the chunks depend on n
// alone, so a shift's result does not depend on the batch.
// Bound by HBM (one read of Y per pass) once there are enough rows: at n =
// 262144, k = 20 one shift / 16 shifts took 111 / 466 us a pass on the vector
// units with 2048 rows a workgroup.
// With only_if != NULL a shift whose only_if[w] is zero is skipped.
static int gram_rows(int64_t n) {  // rows per chunk: at most 512 chunks
  return (int)std::max<int64_t>(256, ((n + 511) / 512 + 63) / 64 * 64);
}
int gram_chunks(int64_t n) { return (int)((n + gram_rows(n) - 1) / gram_rows(n)); }

template <int NB, bool MUL>  // NB blocks of 16 real columns
__global__ __launch_bounds__(256) void k_gram(int64_t n, int k, const double* __restrict__ Y,
                                              const double2* __restrict__ Tm, int kmax, int rows,
                                              double2* __restrict__ partial,
                                              const uint32_t* __restrict__ only_if) {
  typedef Mf<double>::v4 v4;
  constexpr int NU = NB * (NB + 1) / 2, NH = 16 * NB;
  __shared__ double hs[NH][NH + 1];
  const int w = blockIdx.y, chunk = blockIdx.x;
  if (only_if && only_if[w] == 0) return;
  const double* Yw = Y + 2 * (int64_t)w * k * n;
  const int64_t r0 = (int64_t)chunk * rows, r1 = min(n, r0 + rows);
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, i = l & 15, g = l >> 4;
  v4 h[NU];
#pragma unroll
  for (int u = 0; u < NU; u++) h[u] = v4{0, 0, 0, 0};
  auto accumulate = [&](const double (&z)[NB]) {
    int u = 0;
#pragma unroll
    for (int a = 0; a < NB; a++)
#pragma unroll
      for (int b = a; b < NB; b++, u++) h[u] = Mf<double>::op(z[a], z[b], h[u]);
  };
  if constexpr (!MUL) {
    // lane: real column 16 b + i, rows 4 g + s of the group
    double y[2][4][NB];
    auto load = [&](int buf, int64_t rg) {
#pragma unroll
      for (int s = 0; s < 4; s++) {
        const int64_t r = rg + 4 * g + s;
#pragma unroll
        for (int b = 0; b < NB; b++) {
          const int c = 16 * b + i;
          y[buf][s][b] = r < r1 && c < 2 * k ? Yw[2 * ((int64_t)(c >> 1) * n + r) + (c & 1)] : 0.0;
        }
      }
    };
    int64_t rg = r0 + 16 * wave;
    load(0, rg);
    for (; rg < r1; rg += 128) {
      load(1, rg + 64);  // past the chunk: zeros
#pragma unroll
      for (int s = 0; s < 4; s++) accumulate(y[0][s]);
      load(0, rg + 128);
#pragma unroll
      for (int s = 0; s < 4; s++) accumulate(y[1][s]);
    }
  } else {
    // T in real form, [[tr, ti], [-ti, tr]] per entry: element (4 s + g, 16 b + i)
    double t[4 * NB][NB];
#pragma unroll
    for (int s = 0; s < 4 * NB; s++)
#pragma unroll
      for (int b = 0; b < NB; b++) {
        const int c = 4 * s + g, d = 16 * b + i;
        t[s][b] = 0.0;
        if (c < 2 * k && d < 2 * k) {
          const double2 v = Tm[(int64_t)w * kmax * kmax + (c >> 1) * k + (d >> 1)];
          t[s][b] = (c & 1) == (d & 1) ? v.x : (c & 1) ? -v.y : v.y;
        }
      }
    for (int64_t rg = r0 + 16 * wave; rg < r1; rg += 64) {
      double x[4 * NB];  // row i, real column 4 s + g
#pragma unroll
      for (int s = 0; s < 4 * NB; s++) {
        const int c = 4 * s + g;
        x[s] = rg + i < r1 && c < 2 * k ? Yw[2 * ((int64_t)(c >> 1) * n + rg + i) + (c & 1)] : 0.0;
      }
      v4 z[NB];
#pragma unroll
      for (int b = 0; b < NB; b++) z[b] = v4{0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < 4 * NB; s++)
#pragma unroll
        for (int b = 0; b < NB; b++) z[b] = Mf<double>::op(x[s], t[s][b], z[b]);
#pragma unroll
      for (int e = 0; e < 4; e++) {
        double zb[NB];
#pragma unroll
        for (int b = 0; b < NB; b++) zb[b] = z[b][e];
        accumulate(zb);
      }
    }
  }
  for (int v = 0; v < 4; v++) {  // the waves' sums, in order
    if (wave == v) {
      int u = 0;
#pragma unroll
      for (int a = 0; a < NB; a++)
#pragma unroll
        for (int b = a; b < NB; b++, u++)
#pragma unroll
          for (int e = 0; e < 4; e++) {
            double& d = hs[16 * a + Mf<double>::row(l, e)][16 * b + i];
            d = v ? d + h[u][e] : h[u][e];
          }
    }
    __syncthreads();
  }
  double2* out = partial + ((int64_t)w * gridDim.x + chunk) * k * k;
  for (int e = threadIdx.x; e < k * k; e += 256) {
    const int a = e / k, b = e - a * k;
    if (b >= a)
      out[e] = make_double2(hs[2 * a][2 * b] + hs[2 * a + 1][2 * b + 1],
                            hs[2 * a][2 * b + 1] - hs[2 * a + 1][2 * b]);
  }
}

// G[w] = sum of the chunks' partials (upper triangle), 16 slices of the chunks
// per entry, added in order.
__global__ __launch_bounds__(256) void k_gram_sum(int k, int kmax, int nchunk,
                                                  const double2* __restrict__ partial,
                                                  double2* __restrict__ G,
                                                  const uint32_t* __restrict__ only_if) {
  __shared__ double2 red[16][17];
  const int w = blockIdx.y;
  if (only_if && only_if[w] == 0) return;
  const int e = threadIdx.x & 15, slice = threadIdx.x >> 4;
  const int idx = blockIdx.x * 16 + e;
  double2 s = make_double2(0, 0);
  if (idx < k * k && idx % k >= idx / k) {
    const double2* p = partial + (int64_t)w * nchunk * k * k + idx;
#pragma unroll 4
    for (int c = slice; c < nchunk; c += 16) {
      const double2 v = p[(int64_t)c * k * k];
      s.x += v.x;
      s.y += v.y;
    }
  }
  red[slice][e] = s;
  __syncthreads();
  if (slice == 0 && idx < k * k) {
    s = red[0][e];
    for (int c = 1; c < 16; c++) {
      s.x += red[c][e].x;
      s.y += red[c][e].y;
    }
    G[(int64_t)w * kmax * kmax + idx] = s;
  }
}

// Cholesky G = R^H R (R upper, real positive
// diagonal), Rinv = R^-1.  Passes 1 and 2 compose: R <- Rnew Rold,
// Rinv <- Rinv_old Rinv_new.
//
// Cholesky QR breaks down once cond(Y) passes about u^-1/2 (1e8): the Gram
// matrix is then not numerically positive definite.  Pass 0 then takes the
// Cholesky factor of G + s I instead, with the shift of Fukaya, Kannan,
// Nakatsukasa, Yamamoto & Yanagisawa (shifted CholeskyQR3, SISC 2020),
// s = 11 (m k + k (k + 1)) u ||Y||_F^2 (m + 2 in place of m for complex inner
// products; ||Y||_F^2 = trace G bounds ||Y||_2^2), and sets shifted[w]; Y R^-1
// then has a condition number near (u m k)^-1/2, which the two passes that
// follow make orthonormal.  Pass 2 runs only for shifts with shifted[w] set.
// A breakdown that remains latches ST_BREAKDOWN (the pivot is replaced by 1).
//
// Bound by latency (k dependent steps, one workgroup per shift): one barrier
// per step of the factorisation, which leaves the rows' scaling by the roots
// of the pivots to the end, and none in the inverse, eight threads of a wave
// sharing each of its elements' sums.
//
// Gg: nparts partial sums of G a shift, sG elements apart from shift to shift
// (up to kCholParts straight from k_gram, added in k_gram_sum's order: a launch
// of 4 us less; else k_gram_sum's total, as eight sums of k = 32 already cost 3 us
// more here).
constexpr int kCholParts = 4;
__global__ __launch_bounds__(256) void k_chol(int k, int kmax, int64_t m, int nparts, int64_t sG,
                                              const double2* __restrict__ Gg,
                                              double2* __restrict__ Rg, double2* __restrict__ Rinvg,
                                              int pass, uint32_t* __restrict__ shifted,
                                              uint32_t* status) {
  __shared__ double2 G[KM][KM + 1];
  __shared__ double2 Ri[KM][KM + 1];
  __shared__ double2 Ro[KM][KM + 1];
  const int w = blockIdx.x, t = threadIdx.x;
  if (pass == 2 && shifted[w] == 0) return;
  const int64_t at = (int64_t)w * kmax * kmax;
  double2* Rw = Rg + at;
  double2* Riw = Rinvg + at;
  const double2* Gw = Gg + w * sG;
  auto total = [&](int e) {
    double2 s = Gw[e];
#pragma unroll
    for (int c = 1; c < kCholParts; c++)
      if (c < nparts) {
        const double2 v = Gw[c * k * k + e];
        s.x += v.x;
        s.y += v.y;
      }
    return s;
  };
  bool bad = false;
  int attempt = 0;
  double shift = 0.0;
  for (;; attempt++) {
    for (int e = t; e < k * k; e += 256) {
      const int a = e / k, c = e % k;
      double2 v = c >= a ? total(e) : make_double2(0, 0);
      if (a == c) v.x += shift;
      G[a][c] = v;
      if (pass > 0) Ro[a][c] = Rw[e];
    }
    __syncthreads();
    bad = false;
    for (int j = 0; j < k; j++) {  // rows j of sqrt(pivot) R; `bad` is block-uniform
      const double d = G[j][j].x;
      const bool no = !(d > 0.0) || !isfinite(d);
      bad |= no;
      const double rd = no ? 1.0 : 1.0 / d;
      const int wd = k - 1 - j;
      for (int e = t; e < wd * wd; e += 256) {
        const int a = j + 1 + e / wd, c = j + 1 + e % wd;
        if (c < a) continue;
        // (scaled before the product: entries of G are squares already, and
        // their products leave FP64's range from |Y| ~ 1e77 on)
        const double2 gc = G[j][c];
        const double2 p = cmulc(G[j][a], make_double2(gc.x * rd, gc.y * rd));
        G[a][c].x -= p.x;
        G[a][c].y -= p.y;
      }
      __syncthreads();
    }
    if (!(bad && pass == 0 && attempt == 0)) break;
    // the trace from memory: every thread needs it, and the steps above have
    // overwritten the diagonal in LDS
    double tr = 0;
    for (int j = 0; j < k; j++) tr += total(j * (k + 1)).x;
    shift = 11.0 * ((double)(m + 2) * k + (double)k * (k + 1)) * 0x1p-53 * tr;
  }
  if (pass == 0 && t == 0) shifted[w] = attempt;
  double2 v[4];
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const int e = t + 256 * q;
    if (e >= k * k) break;
    const int a = e / k, c = e % k;
    const double d = G[a][a].x;
    const double r = !(d > 0.0) || !isfinite(d) ? 1.0 : sqrt(d);
    v[q] = c > a ? make_double2(G[a][c].x / r, G[a][c].y / r) : make_double2(c == a ? r : 0.0, 0.0);
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const int e = t + 256 * q;
    if (e < k * k) G[e / k][e % k] = v[q];  // R
  }
  __syncthreads();
  invert_upper(G, Ri, k);  // R X = I
  __syncthreads();
  if (pass > 0) {
    // R <- R Rold ; Rinv <- Riold Ri
    double2 ni[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int e = t + 256 * q;
      if (e >= k * k) break;
      const int a = e / k, c = e % k;
      double2 s = make_double2(0, 0), u = make_double2(0, 0);
      for (int x = 0; x < k; x++) {
        const double2 p = cmul(G[a][x], Ro[x][c]);
        s.x += p.x;
        s.y += p.y;
        const double2 z = cmul(Riw[a * k + x], Ri[x][c]);
        u.x += z.x;
        u.y += z.y;
      }
      v[q] = s;
      ni[q] = u;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int e = t + 256 * q;
      if (e >= k * k) break;
      Rw[e] = v[q];
      Riw[e] = ni[q];
    }
  } else {
    for (int e = t; e < k * k; e += 256) {
      Rw[e] = G[e / k][e % k];
      Riw[e] = Ri[e / k][e % k];
    }
  }
  if (t == 0 && bad) latch(status, ST_BREAKDOWN);
}

// Out = Y * Tm[w]  (n x k times k x k), one row per thread (held in registers);
// Out may alias Y.  With only_if != NULL a shift whose only_if[w] is zero is
// skipped.
__global__ __launch_bounds__(256) void k_apply_small(int64_t n, int k, const double2* Y,
                                                     const double2* __restrict__ Tm, int kmax,
                                                     double2* Out,
                                                     const uint32_t* __restrict__ only_if) {
  __shared__ double2 tm[KM][KM];
  const int w = blockIdx.y;
  if (only_if && only_if[w] == 0) return;
  for (int idx = threadIdx.x; idx < k * k; idx += 256)
    tm[idx / k][idx % k] = Tm[(int64_t)w * kmax * kmax + idx];
  __syncthreads();
  int64_t r = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (r >= n) return;
  const double2* Yw = Y + (int64_t)w * k * n;
  double2* Ow = Out + (int64_t)w * k * n;
  double2 row[KM];
#pragma unroll
  for (int i = 0; i < KM; i++) row[i] = i < k ? Yw[(int64_t)i * n + r] : make_double2(0, 0);
  for (int j = 0; j < k; j++) {
    double2 s = make_double2(0, 0);
#pragma unroll
    for (int i = 0; i < KM; i++) {
      if (i < k) {
        double2 p = cmul(row[i], tm[i][j]);
        s.x += p.x; s.y += p.y;
      }
    }
    Ow[(int64_t)j * n + r] = s;
  }
}

// T[w] = I for the shifts with only_if[w] set.
__global__ __launch_bounds__(256) void k_identity_if(int k, int kmax, double2* Tm,
                                                     const uint32_t* __restrict__ only_if) {
  const int w = blockIdx.x;
  if (only_if[w] == 0) return;
  for (int idx = threadIdx.x; idx < k * k; idx += 256)
    Tm[(int64_t)w * kmax * kmax + idx] = make_double2(idx / k == idx % k ? 1.0 : 0.0, 0.0);
}

static int nchunks(int64_t n) { return (int)((n + kChunkRows - 1) / kChunkRows); }

// Cholesky QR of Y (n_omega blocks of n x k) into ws.R and ws.Rinv: two
// passes, and for shifts whose first Cholesky broke down a shifted first pass
// and a third (shifted CholeskyQR3).  The launch sequence is the same either
// way (the third pass returns at once for the other shifts).  With
// explicit_q, a shifted shift's Y is replaced by Q1 = Y R1^-1 after the first
// pass and its R^-1 reset to I, so the two passes that follow orthonormalise
// Q1 itself and the final Q = Q1 R^-1 is orthonormal to O(u); otherwise Q is
// formed from Y through the composed R^-1 and orthonormal to about u cond(Y).
// R is the composed factor (Y = Q R) either way.
static void chol_passes(int n, int n_omega, int k, double* Y, bool explicit_q, SmallWs& ws,
                        uint32_t* status, hipStream_t s) {
  const int rows = gram_rows(n), nc = gram_chunks(n);
  const dim3 g(nc, n_omega);
  double2* part = (double2*)ws.partial;
  for (int pass = 0; pass < 3; pass++) {
    const uint32_t* only = pass == 2 ? ws.shifted : nullptr;
    auto gram = [&](auto nb) {
      constexpr int NB = decltype(nb)::value;
      if (pass)
        hipLaunchKernelGGL((k_gram<NB, true>), g, dim3(256), 0, s, (int64_t)n, k, Y,
                           (const double2*)ws.Rinv, ws.kmax, rows, part, only);
      else
        hipLaunchKernelGGL((k_gram<NB, false>), g, dim3(256), 0, s, (int64_t)n, k, Y,
                           (const double2*)nullptr, ws.kmax, rows, part, only);
    };
    if (k <= 8) gram(std::integral_constant<int, 1>{});
    else if (k <= 16) gram(std::integral_constant<int, 2>{});
    else if (k <= 24) gram(std::integral_constant<int, 3>{});
    else gram(std::integral_constant<int, 4>{});
    const bool direct = nc <= kCholParts;
    if (!direct)
      hipLaunchKernelGGL(k_gram_sum, dim3((k * k + 15) / 16, n_omega), dim3(256), 0, s, k, ws.kmax,
                         nc, (const double2*)part, (double2*)ws.G, only);
    hipLaunchKernelGGL(k_chol, dim3(n_omega), dim3(256), 0, s, k, ws.kmax, (int64_t)n,
                       direct ? nc : 1, (int64_t)(direct ? nc * k * k : ws.kmax * ws.kmax),
                       (const double2*)(direct ? ws.partial : ws.G), (double2*)ws.R,
                       (double2*)ws.Rinv, pass, ws.shifted, status);
    if (pass == 0 && explicit_q) {
      hipLaunchKernelGGL(k_apply_small, dim3((n + 255) / 256, n_omega), dim3(256), 0, s,
                         (int64_t)n, k, (const double2*)Y, (const double2*)ws.Rinv, ws.kmax,
                         (double2*)Y, (const uint32_t*)ws.shifted);
      hipLaunchKernelGGL(k_identity_if, dim3(n_omega), dim3(256), 0, s, k, ws.kmax,
                         (double2*)ws.Rinv, (const uint32_t*)ws.shifted);
    }
  }
}

hipError_t launch_cholqr2(int n, int n_omega, int k, double* Y, SmallWs& ws, uint32_t* status,
                          hipStream_t s) {
  if (nchunks(n) > ws.nchunk || k > ws.kmax || k > KM) return hipErrorInvalidValue;
  chol_passes(n, n_omega, k, Y, true, ws, status, s);
  hipLaunchKernelGGL(k_apply_small, dim3((n + 255) / 256, n_omega), dim3(256), 0, s,
                     (int64_t)n, k, (const double2*)Y, (const double2*)ws.Rinv, ws.kmax,
                     (double2*)Y, (const uint32_t*)nullptr);
  return hipGetLastError();
}

// One-sided (Hestenes) Jacobi SVD of A = R^H (k x k, one workgroup per shift):
// columns are rotated pairwise until mutually orthogonal, A J = Ut S, so
// R^H = Ut S J^H.  Pairs follow the round-robin (circle) order, k/2 disjoint
// pairs per round, 8 threads per pair.  Outputs sorted by descending sigma.
// Also forms Tv = Rinv * W for V = Z Tv.
// A sweep that still rotated a pair after max_sweeps sweeps means the SVD has
// not converged: ST_SVD_NOT_CONVERGED is latched (the results are returned
// as they stand).
__global__ __launch_bounds__(256) void k_jacobi_svd(int k, int kmax, const double2* __restrict__ Rg,
                                                    const double2* __restrict__ Rinvg,
                                                    double* __restrict__ sigma,
                                                    double2* __restrict__ Utg, double2* __restrict__ Wg,
                                                    double2* __restrict__ Tvg, uint32_t* status,
                                                    int max_sweeps) {
  __shared__ double2 A[KM][KM + 1];  // A[row][col]
  __shared__ double2 J[KM][KM + 1];
  __shared__ double sv[KM];
  __shared__ int perm[KM];
  __shared__ int rotated;
  const int w = blockIdx.x;
  const double2* R = Rg + (int64_t)w * kmax * kmax;
  const int m = (k + 1) & ~1;  // even number of players (a zero column pads odd k)
  for (int idx = threadIdx.x; idx < m * m; idx += 256) {
    int a = idx / m, c = idx % m;
    double2 v = make_double2(0, 0);
    if (a < k && c < k) { double2 rc = R[c * k + a]; v = make_double2(rc.x, -rc.y); }  // R^H
    A[a][c] = v;
    J[a][c] = make_double2(a == c ? 1.0 : 0.0, 0.0);
  }
  __syncthreads();
  const int npair = m / 2;
  const int pair = threadIdx.x >> 3, sub = threadIdx.x & 7;
  for (int sweep = 0; sweep < max_sweeps; sweep++) {
    if (threadIdx.x == 0) rotated = 0;
    __syncthreads();
    for (int rnd = 0; rnd < m - 1; rnd++) {
      if (pair < npair) {
        int p, q;
        if (pair == 0) { p = 0; q = 1 + rnd % (m - 1); }
        else {
          p = 1 + (pair + rnd) % (m - 1);
          q = 1 + (m - 1 - pair + rnd) % (m - 1);
        }
        if (p > q) { int t = p; p = q; q = t; }
        double al = 0, be = 0, gr = 0, gi = 0;
        for (int a = sub; a < m; a += 8) {
          double2 x = A[a][p], y = A[a][q];
          al += x.x * x.x + x.y * x.y;
          be += y.x * y.x + y.y * y.y;
          gr += x.x * y.x + x.y * y.y;  // conj(x) y
          gi += x.x * y.y - x.y * y.x;
        }
        al = sum8(al);
        be = sum8(be);
        gr = sum8(gr);
        gi = sum8(gi);
        double er, ei, c, sn;
        if (jacobi_angle(al, be, gr, gi, er, ei, c, sn)) {  // rotate [a_p, e^{-i phi} a_q]
          for (int a = sub; a < m; a += 8) {
            double2 x = A[a][p], y = A[a][q];
            double2 yp = make_double2(y.x * er - y.y * ei, y.x * ei + y.y * er);
            A[a][p] = make_double2(c * x.x - sn * yp.x, c * x.y - sn * yp.y);
            A[a][q] = make_double2(sn * x.x + c * yp.x, sn * x.y + c * yp.y);
            x = J[a][p]; y = J[a][q];
            yp = make_double2(y.x * er - y.y * ei, y.x * ei + y.y * er);
            J[a][p] = make_double2(c * x.x - sn * yp.x, c * x.y - sn * yp.y);
            J[a][q] = make_double2(sn * x.x + c * yp.x, sn * x.y + c * yp.y);
          }
          if (sub == 0) rotated = 1;
        }
      }
      __syncthreads();
    }
    if (!rotated) break;
    __syncthreads();
  }
  // every thread read `rotated` after the last round's barrier; nothing has
  // written it since
  if (threadIdx.x == 0 && rotated) latch(status, ST_SVD_NOT_CONVERGED);
  for (int c = threadIdx.x; c < k; c += 256) {
    double s = 0;
    for (int a = 0; a < k; a++) s += A[a][c].x * A[a][c].x + A[a][c].y * A[a][c].y;
    sv[c] = sqrt(s);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int c = 0; c < k; c++) perm[c] = c;
    for (int a = 0; a < k; a++) {  // selection sort, descending, stable
      int best = a;
      for (int c = a + 1; c < k; c++)
        if (sv[perm[c]] > sv[perm[best]]) best = c;
      int t = perm[a]; perm[a] = perm[best]; perm[best] = t;
    }
    for (int c = 0; c < k; c++)
      if (!isfinite(sv[c])) latch(status, ST_NONFINITE);
  }
  __syncthreads();
  double* sw = sigma + (int64_t)w * k;
  double2* Ut = Utg + (int64_t)w * kmax * kmax;
  double2* Wm = Wg + (int64_t)w * kmax * kmax;
  double2* Tv = Tvg + (int64_t)w * kmax * kmax;
  const double2* Ri = Rinvg + (int64_t)w * kmax * kmax;
  for (int idx = threadIdx.x; idx < k * k; idx += 256) {
    int a = idx / k, c = idx % k;  // row a, output column c
    int src = perm[c];
    double s = sv[src];
    double2 u = A[a][src];
    Ut[a * k + c] = s > 0 ? make_double2(u.x / s, u.y / s) : make_double2(0, 0);
    Wm[a * k + c] = J[a][src];
    double2 t = make_double2(0, 0);
    for (int b = 0; b < k; b++) {
      double2 p = cmul(Ri[a * k + b], J[b][src]);
      t.x += p.x; t.y += p.y;
    }
    Tv[a * k + c] = t;
    if (a == 0) sw[c] = s;
  }
}

hipError_t launch_small_svd(int n, int n_omega, int k, const double* Z, const double* Q,
                            double* sigma, double* V, double* Uqu, SmallWs& ws, uint32_t* status,
                            hipStream_t s) {
  if (nchunks(n) > ws.nchunk || k > ws.kmax || k > KM) return hipErrorInvalidValue;
  // Z = Qz R by Cholesky QR (R and R^-1 composed; Qz never formed)
  chol_passes(n, n_omega, k, const_cast<double*>(Z), false, ws, status, s);  // Z is not written
  // W and its product with R^-1 (ws.G holds Tv = R^-1 W)
  hipLaunchKernelGGL(k_jacobi_svd, dim3(n_omega), dim3(256), 0, s, k, ws.kmax,
                     (const double2*)ws.R, (const double2*)ws.Rinv, sigma, (double2*)ws.Ut,
                     (double2*)ws.W, (double2*)ws.G, status, ws.jacobi_sweeps);
  // V = Z R^-1 W = Qz W
  hipLaunchKernelGGL(k_apply_small, dim3((n + 255) / 256, n_omega), dim3(256), 0, s,
                     (int64_t)n, k, (const double2*)Z, (const double2*)ws.G, ws.kmax, (double2*)V,
                     (const uint32_t*)nullptr);
  if (Uqu)  // Halko et al.'s response modes U = Q Ut (eq. 8)
    hipLaunchKernelGGL(k_apply_small, dim3((n + 255) / 256, n_omega), dim3(256), 0, s,
                       (int64_t)n, k, (const double2*)Q, (const double2*)ws.Ut, ws.kmax,
                       (double2*)Uqu, (const uint32_t*)nullptr);
  return hipGetLastError();
}

// partial[w][chunk][j] = sum over the chunk of |X_j|^2 (and of |D_j|^2 into
// partial2 when D != NULL, after X += D).  Block (chunk, w, z) takes columns
// 4z .. 4z+3; each thread owns rows r0 + t + 256 i of the chunk and issues
// all of a column's loads before it adds them up (in i order), so a column
// costs one memory round trip.
constexpr int kColGroup = 4;
template <typename RD>
__global__ __launch_bounds__(256) void k_colnorm_partial(int64_t n, int k, double2* X,
                                                         const cplx<RD>* __restrict__ D,
                                                         int nchunk, double* partial,
                                                         double* partial2, const uint32_t* skip) {
  if (skip && __hip_atomic_load(skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
  constexpr int RPT = kChunkRows / 256;
  __shared__ double red[2][256];
  const int w = blockIdx.y, chunk = blockIdx.x;
  const int64_t r0 = (int64_t)chunk * kChunkRows, r1 = min(n, r0 + kChunkRows);
  const int j1 = min(k, kColGroup * ((int)blockIdx.z + 1));
  for (int j = kColGroup * blockIdx.z; j < j1; j++) {
    double2* x = X + ((int64_t)w * k + j) * n;
    const cplx<RD>* d = D ? D + ((int64_t)w * k + j) * n : nullptr;
    double2 xv[RPT], dv[RPT];
#pragma unroll
    for (int i = 0; i < RPT; i++) {
      const int64_t r = r0 + threadIdx.x + 256 * i;
      xv[i] = r < r1 ? x[r] : make_double2(0, 0);
      dv[i] = make_double2(0, 0);
      if (d && r < r1) {
        const cplx<RD> q = d[r];
        dv[i] = make_double2(q.re, q.im);
      }
    }
    double sx = 0, sd = 0;
#pragma unroll
    for (int i = 0; i < RPT; i++) {
      const int64_t r = r0 + threadIdx.x + 256 * i;
      if (r < r1) {
        double2 v = xv[i];
        if (d) {
          sd += dv[i].x * dv[i].x + dv[i].y * dv[i].y;
          v.x += dv[i].x; v.y += dv[i].y;
          x[r] = v;
        }
        sx += v.x * v.x + v.y * v.y;
      }
    }
    red[0][threadIdx.x] = sx;
    red[1][threadIdx.x] = sd;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if (threadIdx.x < o) {
        red[0][threadIdx.x] += red[0][threadIdx.x + o];
        red[1][threadIdx.x] += red[1][threadIdx.x + o];
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      partial[((int64_t)w * nchunk + chunk) * 64 + j] = red[0][0];
      if (partial2) partial2[((int64_t)w * nchunk + chunk) * 64 + j] = red[1][0];
    }
    __syncthreads();
  }
}
static dim3 colnorm_grid(int nc, int n_omega, int k) {
  return dim3(nc, n_omega, (k + kColGroup - 1) / kColGroup);
}

__global__ void k_colnorm_final(int k, int nchunk, const double* partial, double* sigma,
                                uint32_t* status) {
  const int w = blockIdx.x;
  for (int j = threadIdx.x; j < k; j += blockDim.x) {
    double s = 0;
    for (int c = 0; c < nchunk; c++) s += partial[((int64_t)w * nchunk + c) * 64 + j];
    s = sqrt(s);
    if (!isfinite(s)) latch(status, ST_NONFINITE);
    sigma[(int64_t)w * k + j] = s;
  }
}

// U_j = W_j / sigma_j (divide; 0 where sigma_j = 0) or W_j * sigma_j.
// Each thread takes kScaleRows rows, 256 apart.
constexpr int kScaleRows = 8;
__global__ __launch_bounds__(256) void k_scale_cols(int64_t n, int k, const double2* W,
                                                    const double* sigma, double2* U, int divide) {
  const int j = blockIdx.y, w = blockIdx.z;
  const double s = sigma[(int64_t)w * k + j];
  const double c = divide ? (s > 0 ? 1.0 / s : 0.0) : s;
  const int64_t base = ((int64_t)w * k + j) * n;
  const int64_t r0 = blockIdx.x * (int64_t)(256 * kScaleRows) + threadIdx.x;
  double2 v[kScaleRows];
#pragma unroll
  for (int i = 0; i < kScaleRows; i++) {
    const int64_t r = r0 + 256 * i;
    v[i] = r < n ? W[base + r] : make_double2(0, 0);
  }
#pragma unroll
  for (int i = 0; i < kScaleRows; i++) {
    const int64_t r = r0 + 256 * i;
    if (r < n) U[base + r] = make_double2(v[i].x * c, v[i].y * c);
  }
}
static dim3 scale_grid(int n, int k, int n_omega) {
  return dim3((unsigned)((n + 256 * kScaleRows - 1) / (256 * kScaleRows)), k, n_omega);
}

hipError_t launch_scale_cols(int n, int n_omega, int k, const double* W, const double* scale,
                             double* U, hipStream_t s) {
  hipLaunchKernelGGL(k_scale_cols, scale_grid(n, k, n_omega), dim3(256), 0, s,
                     (int64_t)n, k, (const double2*)W, scale, (double2*)U, 0);
  return hipGetLastError();
}

hipError_t launch_colnorm_scale(int n, int n_omega, int k, const double* W, double* sigma,
                                double* U, SmallWs& ws, uint32_t* status, hipStream_t s) {
  int nc = nchunks(n);
  if (nc > ws.nchunk || k > KM) return hipErrorInvalidValue;
  double* part = ws.partial;
  hipLaunchKernelGGL((k_colnorm_partial<double>), colnorm_grid(nc, n_omega, k), dim3(256), 0, s,
                     (int64_t)n, k, (double2*)W, (const cplx<double>*)nullptr, nc, part,
                     (double*)nullptr, (const uint32_t*)nullptr);
  hipLaunchKernelGGL(k_colnorm_final, dim3(n_omega), dim3(64), 0, s, k, nc, part, sigma, status);
  if (U)
    hipLaunchKernelGGL(k_scale_cols, scale_grid(n, k, n_omega), dim3(256), 0, s,
                       (int64_t)n, k, (const double2*)W, (const double*)sigma, (double2*)U, 1);
  return hipGetLastError();
}

// After X += D, per column j: e_j = ||D_j|| / ||X_j||, the size of the
// correction just applied.  Refinement shrinks the error by a contraction
// rho per correction, the rate of the iteration matrix I - M32^-1 M
// (forward) or I - M32^-H M^H (adjoint), so the error left is about rho e_j.
// rho is never assumed: it is measured, and kept per shift as the largest
// value seen since the factorisation (slot kRhoSlot of the shift's row; zero
// = not measured yet).  Two measurements: the ratio of two successive
// corrections, e_j / e_j,prev; and, on the first solve after a
// factorisation when the solve has spare columns, probe systems M x = M z
// with z known, solved beside the caller's columns, whose errors before and
// after the first correction are exact (k_probe_rho).  Both directions share it: the adjoint iteration matrix is
// the conjugate transpose of I - M M32^-1 = M (I - M32^-1 M) M^-1, similar
// to the forward one, so the two have the same eigenvalues and the ratios
// converge to the same rate.  A column has converged when e_j <= tol, or
// when the error it leaves, estimated with rho (this solve's own ratio from
// the second correction on, else the kept one), is at most tol / 2.  So the
// first solve after a factorisation takes a second correction unless the
// first already meets tol or its probes measured rho, and later ones, in
// either direction, stop after one when the measured contraction allows it.  Unconverged columns are
// counted into *fail_count (reset by the caller per correction).
__global__ void k_refine_check(int k, int nchunk, const double* px, const double* pd, double tol,
                               int it, int adjoint, double* rho, uint32_t* fail_count,
                               uint32_t* status, const uint32_t* skip) {
  if (skip && __hip_atomic_load(skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
  __shared__ double ratio_max;
  const int w = blockIdx.x;
  double* rw = rho + (int64_t)w * kRhoStride;
  double e = 0.0, ratio = 0.0;
  const int j = threadIdx.x;
  if (threadIdx.x == 0) ratio_max = 0.0;
  __syncthreads();
  if (j < k) {
    double sx = 0, sd = 0;
    for (int c = 0; c < nchunk; c++) {
      sx += px[((int64_t)w * nchunk + c) * 64 + j];
      sd += pd[((int64_t)w * nchunk + c) * 64 + j];
    }
    if (!isfinite(sx) || !isfinite(sd)) latch(status, ST_NONFINITE);
    e = sx > 0 ? sqrt(sd / sx) : (sd > 0 ? INFINITY : 0.0);
    if (it > 0) {
      const double prev = rw[j];
      ratio = prev > 0 ? e / prev : (e > 0 ? INFINITY : 0.0);
      // doubles compare as their bit patterns when non-negative
      atomicMax(reinterpret_cast<unsigned long long*>(&ratio_max),
                (unsigned long long)__double_as_longlong(ratio));
    }
  }
  __syncthreads();
  double* kept = rw + kRhoSlot;
  (void)adjoint;
  const double rho_kept = *kept;
  if (j < k) {
    rw[j] = e;
    const double r = it > 0 ? fmax(ratio, rho_kept) : rho_kept;
    const bool ok = e <= tol || (r > 0.0 && 2.0 * e * r <= tol);
    if (!ok) atomicAdd(fail_count, 1u);
  }
  __syncthreads();
  if (threadIdx.x == 0 && it > 0) *kept = fmax(rho_kept, ratio_max);
}

// partial[w][chunk][q] = sum over the chunk of |X_{k0+q} - Z_q|^2, q < p: the
// errors of the probe columns (X: kk columns per shift, Z: p per shift).
__global__ __launch_bounds__(256) void k_probe_partial(int64_t n, int kk, int k0, int p,
                                                       const double2* __restrict__ X,
                                                       const double2* __restrict__ Z, int nchunk,
                                                       double* partial, const uint32_t* skip) {
  if (skip && __hip_atomic_load(skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
  constexpr int RPT = kChunkRows / 256;
  __shared__ double red[256];
  const int w = blockIdx.y, chunk = blockIdx.x;
  const int64_t r0 = (int64_t)chunk * kChunkRows, r1 = min(n, r0 + kChunkRows);
  for (int q = 0; q < p; q++) {
    const double2* x = X + ((int64_t)w * kk + k0 + q) * n;
    const double2* z = Z + ((int64_t)w * p + q) * n;
    double2 xv[RPT], zv[RPT];
#pragma unroll
    for (int i = 0; i < RPT; i++) {
      const int64_t r = r0 + threadIdx.x + 256 * i;
      xv[i] = r < r1 ? x[r] : make_double2(0, 0);
      zv[i] = r < r1 ? z[r] : make_double2(0, 0);
    }
    double se = 0;
#pragma unroll
    for (int i = 0; i < RPT; i++) {
      const double dx = xv[i].x - zv[i].x, dy = xv[i].y - zv[i].y;
      se += dx * dx + dy * dy;
    }
    red[threadIdx.x] = se;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
      __syncthreads();
    }
    if (threadIdx.x == 0) partial[((int64_t)w * nchunk + chunk) * 64 + q] = red[0];
    __syncthreads();
  }
}

// The probes' errors e_q: after the first solve (stage 0) kept in the slots
// kProbeSlot + q; after the first correction (stage 1) their ratio to those,
// whose largest is the measured contraction rho (kept as in k_refine_check).
__global__ void k_probe_rho(int p, int nchunk, const double* partial, int stage, double* rho,
                            uint32_t* status, const uint32_t* skip) {
  if (skip && __hip_atomic_load(skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
  __shared__ double ratio_max;
  const int w = blockIdx.x, q = threadIdx.x;
  double* rw = rho + (int64_t)w * kRhoStride;
  if (q == 0) ratio_max = 0.0;
  __syncthreads();
  if (q < p) {
    double s = 0;
    for (int c = 0; c < nchunk; c++) s += partial[((int64_t)w * nchunk + c) * 64 + q];
    if (!isfinite(s)) latch(status, ST_NONFINITE);
    const double e = sqrt(s);
    if (stage == 0) {
      rw[kProbeSlot + q] = e;
    } else {
      const double e0 = rw[kProbeSlot + q];
      const double ratio = e0 > 0 ? e / e0 : (e > 0 ? INFINITY : 0.0);
      atomicMax(reinterpret_cast<unsigned long long*>(&ratio_max),
                (unsigned long long)__double_as_longlong(ratio));
    }
  }
  __syncthreads();
  if (q == 0 && stage == 1) rw[kRhoSlot] = fmax(rw[kRhoSlot], ratio_max);
}

hipError_t launch_probe_errors(int n, int n_omega, int kk, int k0, int p, const double* X,
                               const double* Z, SmallWs& ws, uint32_t* status, hipStream_t s) {
  const int nc = nchunks(n);
  if (nc > ws.nchunk || p < 1 || p > 32 || k0 + p > kk || !ws.rho) return hipErrorInvalidValue;
  double* pz = ws.partial + 2 * (size_t)n_omega * nc * 64;
  hipLaunchKernelGGL(k_probe_partial, dim3(nc, n_omega), dim3(256), 0, s, (int64_t)n, kk, k0, p,
                     (const double2*)X, (const double2*)Z, nc, pz, (const uint32_t*)nullptr);
  hipLaunchKernelGGL(k_probe_rho, dim3(n_omega), dim3(64), 0, s, p, nc, (const double*)pz, 0,
                     ws.rho, status, (const uint32_t*)nullptr);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_cols_place(int64_t n, const double2* src, int64_t sws,
                                                    int sc0, double2* dst, int64_t dws, int dc0) {
  const int c = blockIdx.y, w = blockIdx.z;
  const double2* a = src + w * sws + (int64_t)(sc0 + c) * n;
  double2* b = dst + w * dws + (int64_t)(dc0 + c) * n;
  const int64_t r0 = blockIdx.x * (int64_t)(256 * kScaleRows) + threadIdx.x;
  double2 v[kScaleRows];
#pragma unroll
  for (int i = 0; i < kScaleRows; i++) {
    const int64_t r = r0 + 256 * i;
    v[i] = r < n ? a[r] : make_double2(0, 0);
  }
#pragma unroll
  for (int i = 0; i < kScaleRows; i++) {
    const int64_t r = r0 + 256 * i;
    if (r < n) b[r] = v[i];
  }
}

hipError_t launch_cols_place(int64_t n, int n_omega, int ncols, const double* src, int64_t sws,
                             int sc0, double* dst, int64_t dws, int dc0, hipStream_t s) {
  if (ncols < 1) return hipSuccess;
  hipLaunchKernelGGL(k_cols_place, scale_grid((int)n, ncols, n_omega), dim3(256), 0, s, n,
                     (const double2*)src, sws, sc0, (double2*)dst, dws, dc0);
  return hipGetLastError();
}

// Forget the measured contractions (a new factorisation).
__global__ void k_refine_reset(int n_omega, double* rho) {
  const int w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w < n_omega) {
    rho[(int64_t)w * kRhoStride + kRhoSlot] = 0.0;
    rho[(int64_t)w * kRhoStride + kRhoSlot + 1] = 0.0;
  }
}

hipError_t launch_refine_reset(int n_omega, double* rho, hipStream_t s) {
  hipLaunchKernelGGL(k_refine_reset, dim3((n_omega + 255) / 256), dim3(256), 0, s, n_omega, rho);
  return hipGetLastError();
}

hipError_t launch_refine_update(int n, int n_omega, int k, double* X, const void* D, bool d32,
                                double tol, int it, int adjoint, SmallWs& ws, uint32_t* status,
                                uint32_t* fail_count, hipStream_t s, const uint32_t* skip, int kk,
                                int p, const double* Z) {
  int nc = nchunks(n);
  if (kk < k) kk = k;
  if (nc > ws.nchunk || kk > KM || (p > 0 && (!Z || k + p > kk))) return hipErrorInvalidValue;
  double* px = ws.partial;
  double* pd = ws.partial + (size_t)n_omega * nc * 64;
  if (d32)
    hipLaunchKernelGGL((k_colnorm_partial<float>), colnorm_grid(nc, n_omega, kk), dim3(256), 0, s,
                       (int64_t)n, kk, (double2*)X, (const cplx<float>*)D, nc, px, pd, skip);
  else
    hipLaunchKernelGGL((k_colnorm_partial<double>), colnorm_grid(nc, n_omega, kk), dim3(256), 0, s,
                       (int64_t)n, kk, (double2*)X, (const cplx<double>*)D, nc, px, pd, skip);
  if (p > 0 && it == 0) {  // the probes' errors after the first correction: rho
    double* pz = ws.partial + 2 * (size_t)n_omega * nc * 64;
    hipLaunchKernelGGL(k_probe_partial, dim3(nc, n_omega), dim3(256), 0, s, (int64_t)n, kk, k, p,
                       (const double2*)X, (const double2*)Z, nc, pz, skip);
    hipLaunchKernelGGL(k_probe_rho, dim3(n_omega), dim3(64), 0, s, p, nc, pz, 1, ws.rho, status,
                       skip);
  }
  hipLaunchKernelGGL(k_refine_check, dim3(n_omega), dim3(64), 0, s, k, nc, px, pd, tol, it,
                     adjoint, ws.rho, fail_count, status, skip);
  return hipGetLastError();
}

}  // namespace rr
