// Fused Gram-Schmidt and small least-squares kernels of the FGMRES iterations
// (outer solve and Sec. 3.3 smoothing).
//
// Classical Gram-Schmidt applied twice to t against V[0..k):
//   launch_dots        partial dots V_q . t                      (pass 1)
//   launch_upd_dots    h = sum partials; t -= V h; partial V_q . t (pass 2)
//   launch_upd_norm    h2 = sum partials; t -= V h2; partial |t|^2
//   launch_scale_red   |t| = sqrt(sum partials); v = t / |t|
// A consumer kernel reduces its producer's per-block partials itself, every
// block in the same fixed order, so the result is deterministic and no
// cross-block synchronisation or atomics are needed; block 0 also records the
// Hessenberg entries.
//
// Batched launches take the system from blockIdx.y: vectors are segments of
// a batch vector (BSeg), and partial sums, Hessenberg columns and norms sit
// at fixed per-system strides; systems whose active flag is 0 are skipped.
#include <type_traits>

#include "internal.hpp"

namespace ibmg {

namespace {

constexpr int kThreads = 256;

// out[q] = sum_b partial[b * k + q], q < k (out in shared memory), eight
// sums at a time in a fixed order.
__device__ void reduce_partials(const double* __restrict__ partial, int nblk, int k, double* out,
                                double* red) {
  const int tid = threadIdx.x;
  for (int q0 = 0; q0 < k; q0 += 8) {
    const int nq = k - q0 < 8 ? k - q0 : 8;
    double a[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) a[q] = 0.0;
    for (int b = tid; b < nblk; b += kThreads) {
      const double* pb = partial + (size_t)b * k + q0;
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (q < nq) a[q] += pb[q];
    }
    block_sums256<8>(a, nq, red, out + q0, tid);
  }
}

// per-block partial sums of up to 8 products at a time, written as
// partial[blockIdx.x * k + q]
template <typename T>
__device__ void block_dots(const T* __restrict__ V, int k, size_t stride, const T* t, size_t n,
                           double* __restrict__ partial, double* red) {
  const int tid = threadIdx.x;
  for (int v0 = 0; v0 < k; v0 += 8) {
    const int nv = k - v0 < 8 ? k - v0 : 8;
    double acc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = 0.0;
#pragma unroll 4
    for (size_t i = blockIdx.x * (size_t)kThreads + tid; i < n; i += (size_t)gridDim.x * kThreads) {
      const double ti = (double)t[i];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (q < nv) acc[q] += (double)V[(size_t)(v0 + q) * stride + i] * ti;
    }
    block_sums256<8>(acc, nv, red, partial + (size_t)blockIdx.x * k + v0, tid);
  }
}

}  // namespace

// t -= V h (h from pass-1 partials, stored into hcol by block 0), then the
// pass-2 partial dots of the updated t.
template <typename T>
__global__ void __launch_bounds__(kThreads) k_upd_dots(T* t, const T* __restrict__ V, int k, size_t stride,
                                                       BSeg sg, const double* __restrict__ pin, int nblk_in,
                                                       size_t pstride, double* __restrict__ hcol,
                                                       size_t hstride, double* __restrict__ pout) {
  __shared__ double red[36];
  __shared__ double h[64];
  const int sy = blockIdx.y;
  if (!seg_on(sg, sy)) return;
  const size_t o = seg_begin(sg, sy), n = seg_len(sg, sy);
  t += o;
  V += o;
  pin += sy * pstride;
  pout += sy * pstride;
  hcol += sy * hstride;
  reduce_partials(pin, nblk_in, k, h, red);
  if (blockIdx.x == 0 && threadIdx.x < k) hcol[threadIdx.x] = h[threadIdx.x];
  if (k <= 8) {
    // one pass: each basis value feeds the update and then the pass-2 dot
    // of the updated entry; every thread visits its entries in the order
    // block_dots would, so the sums are those of the two-pass form
    double acc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = 0.0;
#pragma unroll 2
    for (size_t i = blockIdx.x * (size_t)kThreads + threadIdx.x; i < n; i += (size_t)gridDim.x * kThreads) {
      double vq[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) vq[q] = q < k ? (double)V[(size_t)q * stride + i] : 0.0;
      double a = (double)t[i];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (q < k) a -= h[q] * vq[q];
      const T tn = (T)a;
      t[i] = tn;
      const double ti = (double)tn;
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (q < k) acc[q] += vq[q] * ti;
    }
    block_sums256<8>(acc, k, red, pout + (size_t)blockIdx.x * k, threadIdx.x);
    return;
  }
#pragma unroll 4
  for (size_t i = blockIdx.x * (size_t)kThreads + threadIdx.x; i < n; i += (size_t)gridDim.x * kThreads) {
    double a = (double)t[i];
    for (int q = 0; q < k; ++q) a -= h[q] * (double)V[(size_t)q * stride + i];
    t[i] = (T)a;
  }
  __syncthreads();
  block_dots<T>(V, k, stride, t, n, pout, red);
}

// t -= V h2 (h2 from pass-2 partials, added into hcol by block 0), then the
// partial sums of |t|^2.
template <typename T>
__global__ void __launch_bounds__(kThreads) k_upd_norm(T* t, const T* __restrict__ V, int k, size_t stride,
                                                       BSeg sg, const double* __restrict__ pin, int nblk_in,
                                                       size_t pstride, double* __restrict__ hcol,
                                                       size_t hstride, double* __restrict__ pout) {
  __shared__ double red[32];
  __shared__ double h[64];
  const int sy = blockIdx.y;
  if (!seg_on(sg, sy)) return;
  const size_t o = seg_begin(sg, sy), n = seg_len(sg, sy);
  t += o;
  V += o;
  pin += sy * pstride;
  pout += sy * pstride;
  hcol += sy * hstride;
  reduce_partials(pin, nblk_in, k, h, red);
  if (blockIdx.x == 0 && threadIdx.x < k) hcol[threadIdx.x] += h[threadIdx.x];
  double acc = 0.0;
#pragma unroll 4
  for (size_t i = blockIdx.x * (size_t)kThreads + threadIdx.x; i < n; i += (size_t)gridDim.x * kThreads) {
    double a = (double)t[i];
    for (int q = 0; q < k; ++q) a -= h[q] * (double)V[(size_t)q * stride + i];
    const T tn = (T)a;
    t[i] = tn;
    acc += (double)tn * (double)tn;
  }
  const double a1[1] = {acc};
  block_sums256<1>(a1, 1, red, pout + blockIdx.x, threadIdx.x);
}

// v = t / sqrt(sum partials) (v = 0 on an exact breakdown); block 0 stores the
// norm into *hout.
template <typename T>
__global__ void __launch_bounds__(kThreads) k_scale_red(const T* t, T* v, BSeg sg,
                                                        const double* __restrict__ pin, int nblk_in,
                                                        size_t pstride, double* __restrict__ hout,
                                                        size_t hstride, ScaleCopies<T> cp) {
  __shared__ double red[32];
  __shared__ double nrm;
  const int sy = blockIdx.y;
  if (!seg_on(sg, sy)) return;
  const size_t o = seg_begin(sg, sy), n = seg_len(sg, sy);
  t += o;
  v += o;
  pin += sy * pstride;
  hout += sy * hstride;
  reduce_partials(pin, nblk_in, 1, &nrm, red);
  const double d = sqrt(nrm);
  if (blockIdx.x == 0 && threadIdx.x == 0) hout[0] = d;
  const double inv = d != 0.0 ? 1.0 / d : 0.0;
  for (size_t i = blockIdx.x * (size_t)kThreads + threadIdx.x; i < n; i += (size_t)gridDim.x * kThreads) {
    const T x = (T)((double)t[i] * inv);
    v[i] = x;
    if (cp.v2) {
      cp.v2[i] = x;
      cp.dst[i] = cp.src[i];
    }
  }
}

// A second Gram-Schmidt pass finished with the normalisation, from partial
// sums of h2 = V^T t and |t|^2 (k + 1 per block), for the kernel timer (the solves
// store the updated t before they scale it):
// t2 = t - V h2, whose norm is sqrt(|t|^2 - |h2|^2) (t2 is orthogonal to the
// orthonormal V), and t = t2 / |t2| (0 on an exact breakdown); block 0 adds
// h2 into hcol[0..k) and stores |t2| into hcol[k].
template <typename T>
__global__ void __launch_bounds__(kThreads) k_scale_upd(T* t, const T* __restrict__ V, int k, size_t stride,
                                                        size_t n, const double* __restrict__ pin, int nblk_in,
                                                        double* __restrict__ hcol) {
  __shared__ double red[32];
  __shared__ double h[64];
  reduce_partials(pin, nblk_in, k + 1, h, red);
  double hh = 0.0;
  for (int q = 0; q < k; ++q) hh += h[q] * h[q];
  const double r2 = h[k] - hh;
  const double d = r2 > 0.0 ? sqrt(r2) : 0.0;
  if (blockIdx.x == 0) {
    if (threadIdx.x < k) hcol[threadIdx.x] += h[threadIdx.x];
    if (threadIdx.x == 0) hcol[k] = d;
  }
  const double inv = d != 0.0 ? 1.0 / d : 0.0;
  for (size_t i = blockIdx.x * (size_t)kThreads + threadIdx.x; i < n; i += (size_t)gridDim.x * kThreads) {
    double a = (double)t[i];
    for (int q = 0; q < k; ++q) a -= h[q] * (double)V[(size_t)q * stride + i];
    t[i] = (T)((double)(T)a * inv);
  }
}

// ---------------------------------------------------------------------------
// Smoothing FGMRES (Sec. 3.3) on an unnormalised basis.  One smoothing step
// works on u_0 = the residual itself and u_k = L z_{k-1} after the first
// Gram-Schmidt pass, stored once and never rescaled or swept again.  The
// second pass is carried as coefficients: with w_0 = u_0 and
//   w_k = u_k - sum_{q<k} g_kq w_q,   g_kq = (w_q . u_k) / D_q,
//   D_k = |w_k|^2 = |u_k|^2 - sum_q g_kq^2 D_q
// the w_k are orthogonal as after classical Gram-Schmidt applied twice (the
// g_kq are the second pass's small corrections), every dot with w_k follows
// from dots with the u_q, and the basic smoother takes u_k where it would take
// w_k / |w_k|: FGMRES allows any search direction, and u_k differs from w_k by
// rounding.  That needs one sweep per iteration (the first pass's update with
// the second pass's sums) where a normalised basis takes two, and none to
// normalise the first vector.  Hessenberg: L z_k = sum_q H_qk w_q + w_{k+1}.
//
// S (kGsScal doubles): D_q at q, g_kq at 16 + 8 k + q, H_qk at 96 + 9 k + q.
// Every block reduces its producer's partial sums itself, in the same order,
// and block 0 records what later launches need; no launch reads entries of S
// that another block of the same launch writes.
// These launches last a few microseconds and are bound by their chain of
// dependent steps (partial sums, block sums, the small algebra, one sweep), so
// the sums cross lanes by DPP and the least squares runs in registers of every
// thread, unrolled for the step's length.  Update / combination at k = 2, FP64:
// 64^2 3.6 / 3.3 us, 256^2 4.9 / 4.6, 512^2 6.8 / 6.4 (with shuffles, the
// second sweep's launch and one thread's least squares: 6.3 + 4.6 / 5.6 us at
// 256^2, 9.6 + 7.4 / 8.3 at 512^2).
// ---------------------------------------------------------------------------
// (a NaN stays a NaN; a zero norm is an exact breakdown: no component)
__device__ __forceinline__ double gs_div(double a, double d) { return d != 0.0 ? a / d : 0.0; }

// sums of nb blocks x NS values into v[0..NS)
template <int NS, int NV>
__device__ __forceinline__ void gs_partials(const double* __restrict__ p, int nb, double (&v)[NV], int at, int tid) {
  for (int b0 = tid; b0 < nb; b0 += 4 * kThreads) {
    double r[4][NS];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int q = 0; q < NS; ++q) {
        const int b = b0 + j * kThreads;
        r[j][q] = b < nb ? p[(size_t)b * NS + q] : 0.0;
      }
#pragma unroll
    for (int q = 0; q < NS; ++q) v[at + q] += (r[0][q] + r[1][q]) + (r[2][q] + r[3][q]);
  }
}

// dots with w_q from dots with u_q, q < K (in place)
template <int K>
__device__ __forceinline__ void gs_to_w(double (&d)[K], const double (&g)[K + 1][K]) {
#pragma unroll
  for (int q = 1; q < K; ++q)
#pragma unroll
    for (int i = 0; i < q; ++i) d[q] -= g[q][i] * d[i];
}

// The second pass of u_K from its sums e_q = u_q . u_K (q < K) and |u_K|^2:
// g_Kq, and D_K returned
template <int K>
__device__ __forceinline__ double gs_second(double (&e)[K], double uu, const double* D, double (&g)[K + 1][K]) {
  gs_to_w<K>(e, g);
  double d = uu;
#pragma unroll
  for (int q = 0; q < K; ++q) {
    g[K][q] = gs_div(e[q], D[q]);
    d -= g[K][q] * g[K][q] * D[q];
  }
  return d <= 0.0 ? 0.0 : d;
}

template <typename T, int K, bool SYS>
__global__ void __launch_bounds__(kThreads) k_gs_update(T* __restrict__ t, const T* __restrict__ u0,
                                                        const T* __restrict__ V, size_t stride, size_t n,
                                                        const double* __restrict__ pd, int nd,
                                                        const double* __restrict__ pu, int npu,
                                                        double* __restrict__ S, double* __restrict__ pout,
                                                        Many m) {
  if (SYS) {
    if (m.act && !m.act[blockIdx.y]) return;
    t += blockIdx.y * m.bs;
    u0 += blockIdx.y * m.bs;
    if (K > 1) V += blockIdx.y * m.bs;
    pd += blockIdx.y * m.ps;
    if (K > 1) pu += blockIdx.y * m.ps;
    pout += blockIdx.y * m.ps;
    S += blockIdx.y * kGsScal;
  }
  constexpr int NA = K == 1 ? 2 : K, NB = K == 1 ? 0 : K;
  __shared__ double red[(NA + NB) * 4];
  __shared__ double red2[(K + 1) * 4];
  const int tid = threadIdx.x;
  double v[NA + NB];
#pragma unroll
  for (int q = 0; q < NA + NB; ++q) v[q] = 0.0;
  gs_partials<NA>(pd, nd, v, 0, tid);
  if constexpr (K > 1) gs_partials<K>(pu, npu, v, NA, tid);
  double D[K], g[K + 1][K];
#pragma unroll
  for (int k = 0; k < K - 1; ++k) {
    D[k] = S[k];
#pragma unroll
    for (int q = 0; q < k; ++q) g[k][q] = S[16 + 8 * k + q];
  }
  block_totals<NA + NB>(v, red, tid);
  double h[K];
#pragma unroll
  for (int q = 0; q < K; ++q) h[q] = v[q];
  if constexpr (K == 1) {
    D[0] = v[1];
    if (blockIdx.x == 0 && tid == 0) S[0] = D[0];
  } else {
    // the previous vector's second pass, now that its sums are complete
    double e[K - 1], gp[K][K - 1];
#pragma unroll
    for (int q = 0; q < K - 1; ++q) {
      e[q] = v[NA + q];
#pragma unroll
      for (int i = 0; i < q; ++i) gp[q][i] = g[q][i];
    }
    D[K - 1] = gs_second<K - 1>(e, v[NA + K - 1], D, gp);
#pragma unroll
    for (int q = 0; q < K - 1; ++q) g[K - 1][q] = gp[K - 1][q];
    if (blockIdx.x == 0 && tid == 0) {
      S[K - 1] = D[K - 1];
#pragma unroll
      for (int q = 0; q < K - 1; ++q) {
        S[16 + 8 * (K - 1) + q] = g[K - 1][q];
        S[96 + 9 * (K - 2) + q] += g[K - 1][q];
      }
    }
  }
  gs_to_w<K>(h, g);
#pragma unroll
  for (int q = 0; q < K; ++q) h[q] = gs_div(h[q], D[q]);
  if (blockIdx.x == 0 && tid == 0)
#pragma unroll
    for (int q = 0; q < K; ++q) S[96 + 9 * (K - 1) + q] = h[q];
  // sum_q h_q w_q as a combination of the u_q
#pragma unroll
  for (int q = K - 1; q >= 1; --q)
#pragma unroll
    for (int i = 0; i < q; ++i) h[i] -= h[q] * g[q][i];
  double acc[K + 1];
#pragma unroll
  for (int q = 0; q <= K; ++q) acc[q] = 0.0;
#pragma unroll 2
  for (size_t i = blockIdx.x * (size_t)kThreads + tid; i < n; i += (size_t)gridDim.x * kThreads) {
    double u[K];
    u[0] = (double)u0[i];
#pragma unroll
    for (int q = 1; q < K; ++q) u[q] = (double)V[(size_t)q * stride + i];
    double a = (double)t[i];
#pragma unroll
    for (int q = 0; q < K; ++q) a -= h[q] * u[q];
    const T tn = (T)a;
    t[i] = tn;
    const double ti = (double)tn;
#pragma unroll
    for (int q = 0; q < K; ++q) acc[q] += u[q] * ti;
    acc[K] += ti * ti;
  }
  block_totals<K + 1>(acc, red2, tid);
  if (tid == 0)
#pragma unroll
    for (int q = 0; q <= K; ++q) pout[(size_t)blockIdx.x * (K + 1) + q] = acc[q];
}

// The end of a step of K iterations: the last vector's second pass from its
// partial sums, then the least squares min || sqrt(D_0) e_1 - H y || ((K+1) x K
// Hessenberg in the orthonormal w_q / sqrt(D_q)) by Givens rotations.  y, and
// with RES rho: r = u_0 - sum_k y_k L z_k = sum_q rho_q u_q.
template <int K, bool RES>
__device__ __forceinline__ void gs_solve(const double* __restrict__ pu, int npu, const double* __restrict__ S,
                                         double* red, int tid, double (&y)[K], double (&rho)[K + 1]) {
  double v[K + 1];
#pragma unroll
  for (int q = 0; q <= K; ++q) v[q] = 0.0;
  gs_partials<K + 1>(pu, npu, v, 0, tid);
  double D[K + 1], g[K + 1][K], H[K + 1][K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    D[k] = S[k];
#pragma unroll
    for (int q = 0; q < k; ++q) g[k][q] = S[16 + 8 * k + q];
#pragma unroll
    for (int q = 0; q <= K; ++q) H[q][k] = q <= k ? S[96 + 9 * k + q] : 0.0;
  }
  block_totals<K + 1>(v, red, tid);
  double e[K];
#pragma unroll
  for (int q = 0; q < K; ++q) e[q] = v[q];
  D[K] = gs_second<K>(e, v[K], D, g);
#pragma unroll
  for (int q = 0; q < K; ++q) H[q][K - 1] += g[K][q];
  double sd[K + 1], R[K + 1][K], f[K + 1];
#pragma unroll
  for (int q = 0; q <= K; ++q) {
    sd[q] = sqrt(D[q]);
    f[q] = 0.0;
  }
  f[0] = sd[0];
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int q = 0; q <= K; ++q) R[q][k] = q <= k ? H[q][k] * sd[q] : (q == k + 1 ? sd[q] : 0.0);
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const double a = R[j][j], b = R[j + 1][j];
    const double d = sqrt(a * a + b * b);
    const double c = d != 0.0 ? a / d : 1.0, s = d != 0.0 ? b / d : 0.0;
#pragma unroll
    for (int k = j; k < K; ++k) {
      const double p = R[j][k], q = R[j + 1][k];
      R[j][k] = c * p + s * q;
      R[j + 1][k] = c * q - s * p;
    }
    const double fj = f[j];
    f[j] = c * fj;
    f[j + 1] = -s * fj;
  }
#pragma unroll
  for (int j = K - 1; j >= 0; --j) {
    double a = f[j];
#pragma unroll
    for (int m = j + 1; m < K; ++m) a -= R[j][m] * y[m];
    y[j] = R[j][j] != 0.0 ? a / R[j][j] : 0.0;
  }
  if constexpr (RES) {
#pragma unroll
    for (int q = 0; q <= K; ++q) {
      double a = q == 0 ? 1.0 : -y[q - 1];
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (k >= q) a -= y[k] * H[q][k];
      rho[q] = a;
    }
#pragma unroll
    for (int q = K; q >= 1; --q)
#pragma unroll
      for (int i = 0; i < q; ++i) rho[i] -= rho[q] * g[q][i];
  }
}

template <typename T, int K, bool SYS>
__global__ void __launch_bounds__(kThreads) k_gs_combine(T* __restrict__ x, const T* __restrict__ Z, size_t stride,
                                                         size_t n, const double* __restrict__ pu, int npu,
                                                         const double* __restrict__ S, bool assign, Many m) {
  if (SYS) {
    if (m.act && !m.act[blockIdx.y]) return;
    x += blockIdx.y * m.bs;
    Z += blockIdx.y * m.bs;
    pu += blockIdx.y * m.ps;
    S += blockIdx.y * kGsScal;
  }
  __shared__ double red[(K + 1) * 4];
  double y[K], rho[K + 1];
  gs_solve<K, false>(pu, npu, S, red, threadIdx.x, y, rho);
  for (size_t i = blockIdx.x * (size_t)kThreads + threadIdx.x; i < n; i += (size_t)gridDim.x * kThreads) {
    double a = assign ? 0.0 : (double)x[i];
#pragma unroll
    for (int q = 0; q < K; ++q) a += y[q] * (double)Z[(size_t)q * stride + i];
    x[i] = (T)a;
  }
}

// One thread per coarse point: its 2 x 2 fine points of x = sum_q y_q Z_q, and
// the restriction of r = sum_q rho_q u_q (neighbouring threads share the fine
// values of r through the caches), in place of an operator application, a
// residual and a restriction.
template <typename T, int K, bool SYS>
__global__ void __launch_bounds__(kThreads) k_gs_combine_restrict(T* __restrict__ x, const T* __restrict__ Z,
                                                                  const T* __restrict__ u0, const T* __restrict__ V,
                                                                  size_t stride, int Nc, const double* __restrict__ pu,
                                                                  int npu, const double* __restrict__ S,
                                                                  T* __restrict__ coarse, Many m) {
  if (SYS) {
    if (m.act && !m.act[blockIdx.y]) return;
    x += blockIdx.y * m.bs;
    Z += blockIdx.y * m.bs;
    u0 += blockIdx.y * m.bs;
    V += blockIdx.y * m.bs;
    pu += blockIdx.y * m.ps;
    S += blockIdx.y * kGsScal;
    coarse += blockIdx.y * (m.bs / 4);
  }
  __shared__ double red[(K + 1) * 4];
  double y[K], rho[K + 1];
  gs_solve<K, true>(pu, npu, S, red, threadIdx.x, y, rho);
  const int gx = (Nc + 63) / 64;
  const int i = ((int)blockIdx.x % gx) * 64 + (threadIdx.x & 63), j = ((int)blockIdx.x / gx) * 4 + (threadIdx.x >> 6);
  if (i >= Nc || j >= Nc) return;
  const int Nf = 2 * Nc;
  const size_t nf = (size_t)Nf * Nf;
#pragma unroll
  for (int comp = 0; comp < 3; ++comp)
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
      for (int ii = 0; ii < 2; ++ii) {
        const size_t o = comp * nf + (size_t)(2 * j + jj) * Nf + 2 * i + ii;
        double a = 0.0;
#pragma unroll
        for (int q = 0; q < K; ++q) a += y[q] * (double)Z[(size_t)q * stride + o];
        x[o] = (T)a;
      }
  restrict_point<T>(coarse, Nc, i, j, [&](int comp, int I, int J) -> T {
    const size_t o = comp * nf + (size_t)J * Nf + I;
    double a = rho[0] * (double)u0[o];
#pragma unroll
    for (int q = 1; q <= K; ++q) a += rho[q] * (double)V[(size_t)q * stride + o];
    return (T)a;
  });
}

static int stream_blocks(size_t n) {
  size_t g = (n + kThreads - 1) / kThreads;
  if (g > 1024) g = 1024;
  return (int)(g < 1 ? 1 : g);
}

template <typename T>
void launch_upd_dots_b(T* t, const T* V, int k, size_t stride, BSeg sg, int nsys, const double* pin,
                       int nblk, size_t pstride, double* hcol, size_t hstride, double* pout, hipStream_t s,
                       int nblk_in) {
  if (nsys <= 0) return;
  IBMG_KLAUNCH((k_upd_dots<T>), dim3(nblk, nsys), dim3(kThreads), 0, s, t, V, k, stride, sg, pin,
                     nblk_in > 0 ? nblk_in : nblk, pstride, hcol, hstride, pout);
  IBMG_LAUNCH_CHECK();
}

template <typename T>
void launch_upd_norm_b(T* t, const T* V, int k, size_t stride, BSeg sg, int nsys, const double* pin,
                       int nblk, size_t pstride, double* hcol, size_t hstride, double* pout, hipStream_t s,
                       int nblk_in) {
  if (nsys <= 0) return;
  IBMG_KLAUNCH((k_upd_norm<T>), dim3(nblk, nsys), dim3(kThreads), 0, s, t, V, k, stride, sg, pin,
                     nblk_in > 0 ? nblk_in : nblk, pstride, hcol, hstride, pout);
  IBMG_LAUNCH_CHECK();
}

template <typename T>
void launch_scale_red_b(const T* t, T* v, BSeg sg, int nsys, size_t nmax, const double* pin, int nblk,
                        size_t pstride, double* hout, size_t hstride, hipStream_t s) {
  if (nsys <= 0) return;
  IBMG_KLAUNCH((k_scale_red<T>), dim3(stream_blocks(nmax), nsys), dim3(kThreads), 0, s, t, v, sg, pin,
                     nblk, pstride, hout, hstride, ScaleCopies<T>{});
  IBMG_LAUNCH_CHECK();
}

template <typename T>
void launch_upd_dots(T* t, const T* V, int k, size_t stride, size_t n, const double* pin, int nblk,
                     double* hcol, double* pout, hipStream_t s, int nblk_in) {
  launch_upd_dots_b<T>(t, V, k, stride, seg1(n), 1, pin, nblk, 0, hcol, 0, pout, s, nblk_in);
}

template <typename T>
void launch_upd_norm(T* t, const T* V, int k, size_t stride, size_t n, const double* pin, int nblk,
                     double* hcol, double* pout, hipStream_t s, int nblk_in) {
  launch_upd_norm_b<T>(t, V, k, stride, seg1(n), 1, pin, nblk, 0, hcol, 0, pout, s, nblk_in);
}

template <typename T>
void launch_scale_red(const T* t, T* v, size_t n, const double* pin, int nblk, double* hout, hipStream_t s,
                      ScaleCopies<T> cp) {
  // nblk: blocks of the producer of pin
  IBMG_KLAUNCH((k_scale_red<T>), dim3(stream_blocks(n)), dim3(kThreads), 0, s, t, v, seg1(n), pin, nblk, (size_t)0, hout,
               (size_t)0, cp);
  IBMG_LAUNCH_CHECK();
}

template <typename T>
void launch_scale_upd(T* t, const T* V, int k, size_t stride, size_t n, const double* pin, int nblk_in,
                      double* hcol, hipStream_t s) {
  if (k < 1 || k > 8) throw Error(IBMG_ERR_ARG, "the norm-carrying second pass takes 1..8 basis vectors");
  IBMG_KLAUNCH((k_scale_upd<T>), dim3(stream_blocks(n)), dim3(kThreads), 0, s, t, V, k, stride, n, pin, nblk_in, hcol);
  IBMG_LAUNCH_CHECK();
}

int gs_blocks(size_t n) {
  const size_t g = (n + kThreads - 1) / kThreads;
  return (int)(g < 1 ? 1 : (g > 768 ? 768 : g));
}
static int gs_blocks(size_t n, const Many& m) {
  const int g = gs_blocks(n);
  return m.nblk > 0 && m.nblk < g ? m.nblk : g;
}

// f(std::integral_constant<int, k>) for 1 <= k <= 8
template <typename F>
static void gs_dispatch(int k, F f) {
  switch (k) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 7: f(std::integral_constant<int, 7>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    default: throw Error(IBMG_ERR_ARG, "a smoothing step takes 1..8 iterations");
  }
}

template <typename T>
void launch_gs_update(T* t, const T* u0, const T* V, int k, size_t stride, size_t n, const double* pd, int nd,
                      const double* pu, double* S, double* pout, hipStream_t s, Many m) {
  if (k > 1 && pu == pout) throw Error(IBMG_ERR_ARG, "the update's partial sums need a buffer of their own");
  if (m.nsys <= 0) return;
  const int nb = gs_blocks(n, m);
  gs_dispatch(k, [&](auto kc) {
    constexpr int K = decltype(kc)::value;
    const dim3 grid(nb, m.nsys);
    if (m.bs) IBMG_KLAUNCH((k_gs_update<T, K, true>), grid, dim3(kThreads), 0, s, t, u0, V, stride, n, pd, nd, pu, nb, S, pout, m);
    else IBMG_KLAUNCH((k_gs_update<T, K, false>), grid, dim3(kThreads), 0, s, t, u0, V, stride, n, pd, nd, pu, nb, S, pout, m);
  });
  IBMG_LAUNCH_CHECK();
}

template <typename T>
void launch_gs_combine(T* x, const T* Z, int k, size_t stride, size_t n, const double* pu, double* S, bool assign,
                       hipStream_t s, Many m) {
  if (m.nsys <= 0) return;
  const int nb = gs_blocks(n, m);
  gs_dispatch(k, [&](auto kc) {
    constexpr int K = decltype(kc)::value;
    if (m.bs) IBMG_KLAUNCH((k_gs_combine<T, K, true>), dim3(nb, m.nsys), dim3(kThreads), 0, s, x, Z, stride, n, pu, nb, S, assign, m);
    else IBMG_KLAUNCH((k_gs_combine<T, K, false>), dim3(stream_blocks(n)), dim3(kThreads), 0, s, x, Z, stride, n, pu, nb, S, assign, m);
  });
  IBMG_LAUNCH_CHECK();
}

template <typename T>
void launch_gs_combine_restrict(T* x, const T* Z, const T* u0, const T* V, int k, size_t stride, int Nc,
                                const double* pu, double* S, T* coarse, hipStream_t s, Many m) {
  if (m.nsys <= 0) return;
  const dim3 grid(((Nc + 63) / 64) * ((Nc + 3) / 4), m.nsys);
  const int nb = gs_blocks((size_t)12 * Nc * Nc, m);
  gs_dispatch(k, [&](auto kc) {
    constexpr int K = decltype(kc)::value;
    if (m.bs) IBMG_KLAUNCH((k_gs_combine_restrict<T, K, true>), grid, dim3(kThreads), 0, s, x, Z, u0, V, stride, Nc, pu, nb, S, coarse, m);
    else IBMG_KLAUNCH((k_gs_combine_restrict<T, K, false>), grid, dim3(kThreads), 0, s, x, Z, u0, V, stride, Nc, pu, nb, S, coarse, m);
  });
  IBMG_LAUNCH_CHECK();
}

#define IBMG_INST_KRY(T)                                                                               \
  template void launch_gs_update<T>(T*, const T*, const T*, int, size_t, size_t, const double*, int,   \
                                    const double*, double*, double*, hipStream_t, Many);               \
  template void launch_gs_combine<T>(T*, const T*, int, size_t, size_t, const double*, double*, bool,  \
                                     hipStream_t, Many);                                               \
  template void launch_gs_combine_restrict<T>(T*, const T*, const T*, const T*, int, size_t, int,      \
                                              const double*, double*, T*, hipStream_t, Many);          \
  template void launch_upd_dots<T>(T*, const T*, int, size_t, size_t, const double*, int, double*,     \
                                   double*, hipStream_t, int);                                         \
  template void launch_upd_norm<T>(T*, const T*, int, size_t, size_t, const double*, int, double*,     \
                                   double*, hipStream_t, int);                                         \
  template void launch_scale_red<T>(const T*, T*, size_t, const double*, int, double*, hipStream_t,    \
                                    ScaleCopies<T>);                                                   \
  template void launch_scale_upd<T>(T*, const T*, int, size_t, size_t, const double*, int, double*,    \
                                    hipStream_t);                                                      \
  template void launch_upd_dots_b<T>(T*, const T*, int, size_t, BSeg, int, const double*, int, size_t, \
                                     double*, size_t, double*, hipStream_t, int);                      \
  template void launch_upd_norm_b<T>(T*, const T*, int, size_t, BSeg, int, const double*, int, size_t, \
                                     double*, size_t, double*, hipStream_t, int);                      \
  template void launch_scale_red_b<T>(const T*, T*, BSeg, int, size_t, const double*, int, size_t,     \
                                      double*, size_t, hipStream_t);

IBMG_INST_KRY(double)
IBMG_INST_KRY(float)

}  // namespace ibmg
