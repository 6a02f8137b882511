// Operator-side kernels: Burgers stencil coefficients, matrix-free M X in
// FP64 (residuals of the mixed-precision refinement), and the physics-weighted
// complex Gaussian sketch (Algorithm 1 step 1 with eq. 10 weighting).
#include <algorithm>

#include "rr_internal.h"

namespace rr {

__global__ void k_fill_u32(uint32_t* p, uint32_t v, int64_t count) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < count; i += stride) p[i] = v;
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t v, int64_t count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  int64_t blocks = (count + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, s, p, v, count);
  return hipGetLastError();
}

// Linearised viscous Burgers about (U(x,y), V = 0), central differences:
//   u-row: nu Lap u - U u_x - U_x u - U_y v,    v-row: nu Lap v - U v_x
__global__ void k_burgers_coeffs(int nx, int ny, const double* __restrict__ U, double hx,
                                 double hy, double nu, double* __restrict__ coef,
                                 double* __restrict__ phi) {
  int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= nx * ny) return;
  int i = p / ny + 1, j = p % ny + 1;  // 1-based node in the (nx+2) x (ny+2) array
  int ld = ny + 2;
  double Uc = U[i * ld + j];
  double Ux = (U[(i + 1) * ld + j] - U[(i - 1) * ld + j]) / (2.0 * hx);
  double Uy = (U[i * ld + j + 1] - U[i * ld + j - 1]) / (2.0 * hy);
  double ax = nu / (hx * hx), ay = nu / (hy * hy);
  double* c = coef + 12 * (int64_t)p;
  c[0] = -2.0 * (ax + ay) - Ux;
  c[1] = ax - Uc / (2.0 * hx);
  c[2] = ax + Uc / (2.0 * hx);
  c[3] = ay;
  c[4] = ay;
  c[5] = -Uy;
  c[6] = -2.0 * (ax + ay);
  c[7] = ax - Uc / (2.0 * hx);
  c[8] = ax + Uc / (2.0 * hx);
  c[9] = ay;
  c[10] = ay;
  c[11] = 0.0;
  if (phi) phi[p] = sqrt(Ux * Ux + Uy * Uy) + 0.1;
}

hipError_t launch_burgers_coeffs(int nx, int ny, const double* U, double hx, double hy,
                                 double nu, double* coef, double* phi, hipStream_t s) {
  int nn = nx * ny;
  hipLaunchKernelGGL(k_burgers_coeffs, dim3((nn + 255) / 256), dim3(256), 0, s, nx, ny, U, hx,
                     hy, nu, coef, phi);
  return hipGetLastError();
}

// Y = Bm - M X  (or Y = M X when Bm == NULL), M = i omega I - L, for the
// columns of one group (blockIdx.z) of shift w (blockIdx.y).  Adjoint: M^H =
// conj(i omega) I - L^T, whose stencil reads the transposed coefficients from
// the neighbouring nodes.  Y may be FP32 (the residual of an FP32 correction,
// which rounds it there anyway).
//
// Bound by HBM: x (and b) read once, y written once.  A thread takes one
// unknown's place in kApplyLines consecutive grid lines, so that its loads are
// consecutive across lanes (16 bytes each), a line's neighbours in x are the
// thread's own values, and the node's other unknown is the next lane's; it
// reads its stencil once for all columns.  Consecutive strips of lines go to
// one XCD (workgroups are dealt to the eight in turn), whose L2 then serves
// the lines that two strips share.  At n = 262144, 16 shifts, 20 columns: 0.85
// ms with one thread per node and no strips, 0.54 ms now (2.7 GB).
// DOTS: instead of Bm, D whose dot products with Y are taken on the way, one
// pair of partial sums per workgroup and column: 1 <D, Y>, 2 <Y, D> and <Y, Y>.
// Below kApplyDealt workgroups a shift the strips go out in turn: filling the
// eighths up would start up to seven idle workgroups a shift (16 x 8 nodes, 1000
// shifts: 191 us a call instead of 59).
constexpr int kApplyLines = 4;
constexpr int kApplyDealt = 64;
template <typename OUT, int DOTS>
__global__ __launch_bounds__(256) void k_apply(int nx, int ny, const double* __restrict__ coef,
                                               const double* __restrict__ omega, int k,
                                               int group, int chunks, int adjoint,
                                               const double2* __restrict__ X,
                                               const double2* __restrict__ Bm, int64_t bstride,
                                               cplx<OUT>* __restrict__ Y, const uint32_t* skip,
                                               double2* __restrict__ partial) {
  if (skip && __hip_atomic_load(skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
  constexpr int L = kApplyLines;
  const int chunk = chunks < kApplyDealt
                        ? blockIdx.x
                        : (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (chunk >= chunks) return;
  const int w = blockIdx.y, ld = 2 * ny, strips = (nx + L - 1) / L;
  const int64_t n = (int64_t)nx * ld;
  const int64_t item = chunk * (int64_t)256 + threadIdx.x;
  const bool live = item < (int64_t)strips * ld;
  if (DOTS == 0 && (item & ~int64_t(63)) >= (int64_t)strips * ld) return;  // a wave without work
  const int strip = live ? (int)(item / ld) : strips - 1;
  const int r = live ? (int)(item % ld) : (int)(threadIdx.x & 1);  // unknown within a line
  const int c = r & 1, j = r >> 1, i0 = L * strip;
  const int dn = j < ny - 1 ? 2 : 0, ds = j > 0 ? -2 : 0;
  // couplings of the line's unknown to itself, the node's other unknown, E, W, N, S
  double a[L], ac[L], e[L], wv[L], nv[L], sv[L];
#pragma unroll
  for (int t = 0; t < L; t++) {
    const int i = min(i0 + t, nx - 1), p = i * ny + j;
    const double* cf = coef + 12 * (int64_t)p + 6 * c;
    const bool hE = i < nx - 1, hW = i > 0;
    a[t] = cf[0];
    if (!adjoint) {
      ac[t] = cf[5];
      e[t] = hE ? cf[1] : 0.0;
      wv[t] = hW ? cf[2] : 0.0;
      nv[t] = dn ? cf[3] : 0.0;
      sv[t] = ds ? cf[4] : 0.0;
    } else {
      ac[t] = coef[12 * (int64_t)p + 6 * (1 - c) + 5];
      e[t] = hE ? cf[12 * ny + 2] : 0.0;
      wv[t] = hW ? cf[-12 * ny + 1] : 0.0;
      nv[t] = dn ? cf[12 + 4] : 0.0;
      sv[t] = ds ? cf[-12 + 3] : 0.0;
    }
  }
  // shift: M = (i omega) I - L; i omega = -om_i + i om_r; M^H shift = conj of it
  const double sr = -omega[2 * w + 1], si = adjoint ? -omega[2 * w] : omega[2 * w];
  int64_t at[L + 2];  // this unknown in lines i0 - 1 .. i0 + L (the grid's edge: the line itself)
#pragma unroll
  for (int t = 0; t < L + 2; t++) at[t] = (int64_t)min(max(i0 + t - 1, 0), nx - 1) * ld + r;
  const int j1 = min(k, (int)(blockIdx.z + 1) * group);
  for (int col = blockIdx.z * group; col < j1; col++) {
    const int64_t off = ((int64_t)w * k + col) * n;
    const double2* x = X + off;
    double2 s0 = make_double2(0, 0), s1 = make_double2(0, 0);
    const double2* bb = Bm ? Bm + (int64_t)w * bstride + (int64_t)col * n : nullptr;
    double2 v[L + 2], xn[L], xs[L], b[L];
#pragma unroll
    for (int t = 0; t < L + 2; t++) v[t] = x[at[t]];
#pragma unroll
    for (int t = 0; t < L; t++) {
      xn[t] = x[at[t + 1] + dn];
      xs[t] = x[at[t + 1] + ds];
      b[t] = bb ? bb[at[t + 1]] : make_double2(0, 0);
    }
#pragma unroll
    for (int t = 0; t < L; t++) {
      const double2 xc = v[t + 1];
      const double2 xo = make_double2(__shfl_xor(xc.x, 1), __shfl_xor(xc.y, 1));
      double lr = a[t] * xc.x + ac[t] * xo.x;
      double li = a[t] * xc.y + ac[t] * xo.y;
      lr += e[t] * v[t + 2].x;
      li += e[t] * v[t + 2].y;
      lr += wv[t] * v[t].x;
      li += wv[t] * v[t].y;
      lr += nv[t] * xn[t].x;
      li += nv[t] * xn[t].y;
      lr += sv[t] * xs[t].x;
      li += sv[t] * xs[t].y;
      double mr = sr * xc.x - si * xc.y - lr;
      double mi = sr * xc.y + si * xc.x - li;
      if (DOTS == 0 && bb) {
        mr = b[t].x - mr;
        mi = b[t].y - mi;
      }
      if (live && i0 + t < nx) {
        Y[off + at[t + 1]] = cplx<OUT>{(OUT)mr, (OUT)mi};
        if (DOTS) {
          const double im = b[t].x * mi - b[t].y * mr;
          s0.x += b[t].x * mr + b[t].y * mi;
          s0.y += DOTS == 1 ? im : -im;
          s1.x += mr * mr + mi * mi;
        }
      }
    }
    if (DOTS) {
      for (int o = 32; o > 0; o >>= 1) {
        s0.x += __shfl_down(s0.x, o, 64);
        s0.y += __shfl_down(s0.y, o, 64);
        s1.x += __shfl_down(s1.x, o, 64);
      }
      __shared__ double2 red[2][4];
      __syncthreads();  // the column before has been read
      if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = s0;
        red[1][threadIdx.x >> 6] = s1;
      }
      __syncthreads();
      if (threadIdx.x < 2) {
        double2 sum = make_double2(0, 0);
        for (int u = 0; u < 4; u++) {
          sum.x += red[threadIdx.x][u].x;
          sum.y += red[threadIdx.x][u].y;
        }
        partial[(((int64_t)w * k + col) * chunks + chunk) * 2 + threadIdx.x] = sum;
      }
    }
  }
}

int apply_chunks(int nx, int ny) {
  const int64_t items = (int64_t)((nx + kApplyLines - 1) / kApplyLines) * 2 * ny;
  return (int)((items + 255) / 256);
}

template <typename OUT, int DOTS = 0>
static hipError_t apply_run(const OpDesc& op, const double* omega, int n_omega, int k, int adjoint,
                            const double* X, const double* Bm, int64_t bstride, cplx<OUT>* Y,
                            hipStream_t s, const uint32_t* skip, double* partial = nullptr) {
  const int chunks = apply_chunks(op.nx, op.ny);
  // columns in groups where the chunks alone leave the GPU idle (8 workgroups
  // a CU), two columns at least: each group reads the stencil again
  const int64_t wgs = (int64_t)chunks * n_omega;
  const int groups = (int)std::min<int64_t>((k + 1) / 2, std::max<int64_t>(1, 2048 / wgs));
  const int group = (k + groups - 1) / groups;
  const int dealt = chunks < kApplyDealt ? chunks : (chunks + 7) / 8 * 8;
  hipLaunchKernelGGL((k_apply<OUT, DOTS>), dim3(dealt, n_omega, (k + group - 1) / group),
                     dim3(256), 0, s, op.nx, op.ny, op.coef, omega, k, group, chunks, adjoint,
                     (const double2*)X, (const double2*)Bm, bstride, Y, skip, (double2*)partial);
  return hipGetLastError();
}

hipError_t launch_apply(const OpDesc& op, const double* omega, int n_omega, int k, int adjoint,
                        const double* X, const double* Bm, int64_t bstride, double* Y,
                        hipStream_t s, const uint32_t* skip) {
  return apply_run(op, omega, n_omega, k, adjoint, X, Bm, bstride, (cplx<double>*)Y, s, skip);
}
hipError_t launch_apply_dots(const OpDesc& op, const double* omega, int n_omega, int k, int adjoint,
                             const double* X, double* Y, const double* D, bool norm,
                             double* partial, hipStream_t s, const uint32_t* skip) {
  auto* run = norm ? apply_run<double, 2> : apply_run<double, 1>;
  return run(op, omega, n_omega, k, adjoint, X, D, (int64_t)k * op.n, (cplx<double>*)Y, s, skip,
             partial);
}
hipError_t launch_residual32(const OpDesc& op, const double* omega, int n_omega, int k, int adjoint,
                             const double* X, const double* Bm, int64_t bstride, float* Y,
                             hipStream_t s, const uint32_t* skip) {
  return apply_run(op, omega, n_omega, k, adjoint, X, Bm, bstride, (cplx<float>*)Y, s, skip);
}

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): 10 rounds of two 32x32->64 products
// on counter words 0 and 2, with the key bumped by the Weyl constants.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
  const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
  const uint32_t W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; r++) {
    if (r) { k0 += W0; k1 += W1; }
    uint32_t hi0 = __umulhi(M0, c[0]), lo0 = M0 * c[0];
    uint32_t hi1 = __umulhi(M1, c[2]), lo1 = M1 * c[2];
    uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0; c[1] = lo1; c[2] = n2; c[3] = lo0;
  }
}

__global__ void k_philox_raw(uint32_t* out, int64_t count, uint32_t c1, uint32_t c2,
                             uint32_t k0, uint32_t k1) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= count) return;
  uint32_t c[4] = {(uint32_t)i, c1, c2, 0u};
  philox4x32_10(c, k0, k1);
  out[4 * i + 0] = c[0]; out[4 * i + 1] = c[1]; out[4 * i + 2] = c[2]; out[4 * i + 3] = c[3];
}

// Test matrix entry (r, j), weighted by phi[r/2] when phi is given:
//   Gaussian (and the orthonormal kind before its QR): sqrt(-ln u1) exp(2 pi i u2),
//     u1 = (m1+1) 2^-53, u2 = m2 2^-53 from the top 53 bits of (x0:x1) and
//     (x2:x3) at counter (r, j, 0, 0);
//   Rademacher: +-1, the sign being the top bit of x0 at that counter;
//   sparse sign: that +-1 if column j is among the zeta columns of row r with
//     the smallest keys (x0 at counter (r, j', 1, 0)), ties to the lower
//     column, else 0.
__global__ void k_sketch(int64_t n, int k, const double* __restrict__ phi, uint32_t k0,
                         uint32_t k1, int kind, int zeta, double2* __restrict__ theta) {
  int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  int j = blockIdx.y;
  if (r >= n) return;
  uint32_t c[4] = {(uint32_t)r, (uint32_t)j, 0u, 0u};
  philox4x32_10(c, k0, k1);
  double2 v;
  if (kind == RR_TM_RADEMACHER || kind == RR_TM_SPARSE) {
    bool keep = true;
    if (kind == RR_TM_SPARSE) {
      uint32_t kc[4] = {(uint32_t)r, (uint32_t)j, 1u, 0u};
      philox4x32_10(kc, k0, k1);
      const uint32_t key = kc[0];
      int rank = 0;
      for (int jj = 0; jj < k; jj++) {
        if (jj == j) continue;
        uint32_t oc[4] = {(uint32_t)r, (uint32_t)jj, 1u, 0u};
        philox4x32_10(oc, k0, k1);
        rank += (oc[0] < key) || (oc[0] == key && jj < j);
      }
      keep = rank < zeta;
    }
    v = make_double2(keep ? ((c[0] >> 31) ? -1.0 : 1.0) : 0.0, 0.0);
  } else {
    uint64_t m1 = ((((uint64_t)c[0]) << 32) | c[1]) >> 11;
    uint64_t m2 = ((((uint64_t)c[2]) << 32) | c[3]) >> 11;
    const double two_m53 = 1.1102230246251565404e-16;
    double u1 = ((double)m1 + 1.0) * two_m53;
    double u2 = (double)m2 * two_m53;
    double rad = sqrt(-log(u1));
    double sn, cs;
    sincospi(2.0 * u2, &sn, &cs);
    v = make_double2(rad * cs, rad * sn);
  }
  double w = (phi && kind != RR_TM_ORTHONORMAL) ? phi[r >> 1] : 1.0;
  theta[(int64_t)j * n + r] = make_double2(w * v.x, w * v.y);
}

hipError_t launch_sketch(const OpDesc& op, const double* phi, int k, uint64_t seed, int kind,
                         int zeta, double* Theta, hipStream_t s) {
  int64_t n = op.n;
  dim3 grid((unsigned)((n + 255) / 256), k);
  hipLaunchKernelGGL(k_sketch, grid, dim3(256), 0, s, n, k, phi, (uint32_t)(seed & 0xffffffffu),
                     (uint32_t)(seed >> 32), kind, zeta, (double2*)Theta);
  return hipGetLastError();
}

__global__ void k_weight_rows(int64_t n, const double* __restrict__ phi, double2* theta) {
  int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (r >= n) return;
  const double w = phi[r >> 1];
  double2* t = theta + (int64_t)blockIdx.y * n + r;
  double2 v = *t;
  *t = make_double2(w * v.x, w * v.y);
}

hipError_t launch_weight_rows(int64_t n, int k, const double* phi, double* Theta, hipStream_t s) {
  dim3 grid((unsigned)((n + 255) / 256), k);
  hipLaunchKernelGGL(k_weight_rows, grid, dim3(256), 0, s, n, phi, (double2*)Theta);
  return hipGetLastError();
}

}  // namespace rr

// Raw generator output for the known-answer test of the device generator:
// out[4*i .. 4*i+3] = Philox4x32-10 of counter (i, c1, c2, 0) under (k0, k1).
extern "C" rr_status rr_philox_raw(uint32_t* out_dev, int64_t count, uint32_t c1, uint32_t c2,
                                   uint32_t k0, uint32_t k1, void* stream) {
  if (!out_dev || count < 0) return RR_ERR_INVALID;
  if (count == 0) return RR_OK;
  hipLaunchKernelGGL(rr::k_philox_raw, dim3((unsigned)((count + 255) / 256)), dim3(256), 0,
                     (hipStream_t)stream, out_dev, count, c1, c2, k0, k1);
  return hipGetLastError() == hipSuccess ? RR_OK : RR_ERR_HIP;
}

// Unweighted/weighted sketch written to a caller buffer (tests): Theta (k, n).
extern "C" rr_status rr_sketch(const rr_problem* p, int32_t k, uint64_t seed, rr_test_matrix kind,
                               int32_t zeta, double* theta, void* stream) {
  if (!p || !theta || k < 1 || p->nx < 1 || p->ny < 1) return RR_ERR_INVALID;
  if (kind != RR_TM_GAUSSIAN && kind != RR_TM_RADEMACHER && kind != RR_TM_SPARSE)
    return RR_ERR_INVALID;
  const int z = zeta <= 0 ? (k < 8 ? k : 8) : (zeta < k ? zeta : k);
  rr::OpDesc op{p->nx, p->ny, 2 * p->nx * p->ny, p->coef};
  return rr::launch_sketch(op, p->phi, k, seed, kind, z, theta, (hipStream_t)stream) ==
                 hipSuccess
             ? RR_OK
             : RR_ERR_HIP;
}
