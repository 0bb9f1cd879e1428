// Dense pieces of the V-cycle: Schwarz box matrices L_k = R_k L R_k^T
// (Alg. 2) assembled from the level stencils and the Galerkin IB rows, their
// batched inversion, the restricted additive Schwarz application, and the
// coarsest-level direct solve (Alg. 1, coarse-grid equation).
//
// Box local ordering (m = b + 2o cells per side): x-faces jj*(m+1) + ii for
// ii in [0, m], jj in [0, m); y-faces m(m+1) + jj*m + ii for ii in [0, m),
// jj in [0, m]; cells 2m(m+1) + jj*m + ii.  Owned unknowns (b x b cells with
// their left x-face and bottom y-face) are ordered x-faces, y-faces, cells,
// each (oj, oi) row-major.
#include <algorithm>
#include <type_traits>

#include "internal.hpp"

namespace ibmg {

static inline int cdiv(size_t a, int b) { return (int)((a + b - 1) / b); }

__device__ __forceinline__ int pmod(int a, int N) {
  a %= N;
  return a < 0 ? a + N : a;
}

struct CsrView {
  const int* ptr;
  const int* col;
  const double* val;
};

// Box matrices, ld x ld each: row and column at(k) hold local unknown k (its
// position; null maps: k itself).  One work-group per 64 rows: the kept tiles
// (on or below the diagonal) are zeroed, a thread per row writes the stencil,
// and a wave per row adds the IB entries, whose columns are distinct.  Bound by
// the zeroing's writes; with one work-group per matrix it was bound by the rows'
// serial entry loops and by the few work-groups (580 -> 200 us
// on average over the levels of the 512^2 annulus).  Rows [nn, nnp) are the padding: 1 on the diagonal.
__global__ void __launch_bounds__(256) k_patch_assemble(const int* __restrict__ patch_ids, BoxGeom g,
                                                        StokesCoef<double> c, CsrView tu, CsrView tv, BoxOrder bo,
                                                        BoxMat bm, double* __restrict__ mats) {
  const int mat = blockIdx.y, pid = patch_ids[mat], ld = bm.ld, nnp = bm.nnp;
  const int N = g.N, NN = N * N, m = g.m, bb = g.b * g.b;
  const int x0 = (pid % g.npd) * g.b - g.o;
  const int y0 = (pid / g.npd) * g.b - g.o;
  double* A = mats + (size_t)mat * ld * ld;
  const int R0 = blockIdx.x * 64, R1 = R0 + 64 < ld ? R0 + 64 : ld;
  const unsigned short* ord = bo.ord ? bo.ord + (size_t)mat * g.nown : nullptr;
  const unsigned short* own = bo.ord ? bo.own + (size_t)mat * g.nown : nullptr;
  auto at = [&](int k) {
    if (!bo.pos) return k;
    const int p = bo.pos[k];
    return p < nnp ? p : nnp + own[p - nnp];
  };
  const int nu = m * (m + 1), p0 = 2 * nu;
  auto local = [&](int row) {   // -1: padding
    if (!bo.pos) return row;
    if (row < nnp) return row < bm.nn ? bo.nonown[row] : -1;
    const int r = ord[row - nnp], comp = r / bb, oi = r % bb % g.b + g.o, oj = r % bb / g.b + g.o;
    return comp == 0 ? oj * (m + 1) + oi : (comp == 1 ? nu + oj * m + oi : p0 + oj * m + oi);
  };
  for (int r = R0; r < R1; ++r)
    for (int k = threadIdx.x; k < R1; k += 256) A[(size_t)r * ld + k] = 0.0;
  __syncthreads();
  const double dg = c.alpha + 4.0 * c.beta;
  if (threadIdx.x < R1 - R0) {
    const int row = R0 + threadIdx.x, k = local(row);
    double* Ar = A + (size_t)row * ld;
    auto put = [&](int kc, double v) {
      const int q = at(kc);
      if (q < R1) Ar[q] = v;
    };
    if (k < 0) {
      Ar[row] = 1.0;
    } else if (k < nu) {  // x-face (ii, jj)
      const int ii = k % (m + 1), jj = k / (m + 1);
      Ar[row] = dg;
      if (ii >= 1) put(k - 1, -c.beta);
      if (ii <= m - 1) put(k + 1, -c.beta);
      if (jj >= 1) put(k - (m + 1), -c.beta);
      if (jj <= m - 2) put(k + (m + 1), -c.beta);
      if (ii <= m - 1) put(p0 + jj * m + ii, c.gi);
      if (ii >= 1) put(p0 + jj * m + ii - 1, -c.gi);
    } else if (k < p0) {  // y-face (ii, jj)
      const int ii = (k - nu) % m, jj = (k - nu) / m;
      Ar[row] = dg;
      if (ii >= 1) put(k - 1, -c.beta);
      if (ii <= m - 2) put(k + 1, -c.beta);
      if (jj >= 1) put(k - m, -c.beta);
      if (jj <= m - 1) put(k + m, -c.beta);
      if (jj <= m - 1) put(p0 + jj * m + ii, c.gi);
      if (jj >= 1) put(p0 + (jj - 1) * m + ii, -c.gi);
    } else {  // cell (ii, jj): -(D u)
      const int ii = (k - p0) % m, jj = (k - p0) / m;
      put(jj * (m + 1) + ii + 1, -c.gi);
      put(jj * (m + 1) + ii, c.gi);
      put(nu + (jj + 1) * m + ii, -c.gi);
      put(nu + jj * m + ii, c.gi);
    }
  }
  __syncthreads();
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int row = R0 + wave; row < R1; row += 4) {
    const int k = local(row);
    if (k < 0 || k >= p0) continue;
    const bool xf = k < nu;
    const int ii = xf ? k % (m + 1) : (k - nu) % m, jj = xf ? k / (m + 1) : (k - nu) / m;
    const int r = pmod(y0 + jj, N) * N + pmod(x0 + ii, N);
    const CsrView& t = xf ? tu : tv;
    double* Ar = A + (size_t)row * ld;
    // col indexes the level's [u | v] vector; the entry counts when its face
    // lies in the enlarged box
    for (int e = t.ptr[r] + lane; e < t.ptr[r + 1]; e += 64) {
      const int comp = t.col[e] >= NN ? 1 : 0, f = t.col[e] - comp * NN;
      const int li = pmod(f % N - x0, N), lj = pmod(f / N - y0, N);
      int kc = -1;
      if (comp == 0) {
        if (li <= m && lj <= m - 1) kc = lj * (m + 1) + li;
      } else if (li <= m - 1 && lj <= m) {
        kc = nu + lj * m + li;
      }
      if (kc < 0) continue;
      const int q = at(kc);
      if (q < R1) Ar[q] += t.val[e];
    }
  }
}

void launch_patch_assemble(const int* patch_ids, int count, BoxGeom g, StokesCoef<double> c,
                           const int* tptr_u, const int* tcol_u, const double* tval_u,
                           const int* tptr_v, const int* tcol_v, const double* tval_v, BoxOrder bo, BoxMat bm,
                           double* mats, hipStream_t s) {
  if (!count) return;
  CsrView tu{tptr_u, tcol_u, tval_u}, tv{tptr_v, tcol_v, tval_v};
  IBMG_KLAUNCH(k_patch_assemble, dim3((bm.ld + 63) / 64, count), dim3(256), 0, s, patch_ids, g, c, tu, tv, bo, bm, mats);
  IBMG_LAUNCH_CHECK();
}

// Operand layout of the 16x16x4 MFMA: lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16]; its result register v holds D[row][l % 16] with
// row = 4 (l / 16) + v for FP32 and row = l / 16 + 4 v for FP64 (checked on
// gfx950 with a one-wave probe).
template <typename T>
struct Mfma;
template <>
struct Mfma<double> {
  typedef double acc_t __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc_t mma(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int kq, int v) { return kq + 4 * v; }
};
template <>
struct Mfma<float> {
  typedef float acc_t __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc_t mma(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int kq, int v) { return 4 * kq + v; }
};

// ---------------------------------------------------------------------------
// Batched in-place inversion of the symmetric box matrices by block sweeps
// (the symmetric form of Gauss-Jordan elimination, no pivoting), 128 columns
// per step.  The box matrices are ordered velocities first: the velocity
// block R_k A_IB R_k^T is symmetric positive definite (a principal submatrix
// of rho/dt - mu Lap + IB with the periodic constants cut off), and the
// pressure pivots come from the negative definite Schur complement
// -G^T A^{-1} G, so no pivot vanishes.  L_IB is symmetric (G = -D^T,
// S = J^*), so every swept matrix is too, and only the 64 x 64 tiles on or
// below the diagonal (tiles I >= J, diagonal tiles in full) are kept.
// Sweeping block K (columns kb .. kb+127, tiles K0 = kb/64 and K1 = K0 + 1)
// of a symmetric S with D = S_KK:
//   S_IJ <- S_IJ - S_IK D^{-1} S_KJ   (I, J outside K),
//   S_IK <- S_IK D^{-1},  S_KK <- -D^{-1};
// after every block S = -A^{-1}.
// The restricted boxes need less than the whole inverse: with the unknowns
// ordered non-owned first (n), owned last (o), the solution on the owned ones is
//   z_o = S_oo^{-1} (r_o - A_on A_nn^{-1} r_n),  S_oo = A_oo - A_on A_nn^{-1} A_no.
// Sweeping the blocks of n leaves W = A_on A_nn^{-1} in the rows o; rows already
// swept are not needed again, so those steps update the rows below their block
// only (elimination, "partial" below), and the blocks of o are then swept
// within o alone.
// The box matrices are sparse, and a 64-row tile of column K that is zero takes
// no part in step K: panel read flags the tiles that are not, and the other
// launches skip the rest.  The order of the unknowns keeps many zero: n runs
// around the ring, sector by sector (the faces before the cells), so a sector
// meets its neighbours and the wrap only; o runs line by line (faces before
// cells) through the rows that n does not reach and ends with those it does
// (coupled velocities, then the cells beside one).  Every prefix of these orders
// holds, with each of its cells, faces that lead out of the set of those cells,
// so the pressure pivots stay definite as in the velocities-first order.  A 16
// x 16/4 box takes 0.75 GFLOP (1.4 where the structure runs along its edge)
// instead of 3.4, the whole inverse's 5.8.
// Stiff structures leave D with rigid and soft directions side by side, so D^{-1}
// is never applied as a matrix: with D = L D_1 L^T (D_1 diagonal) and Y = S_:K L^{-T},
//   S_IJ <- S_IJ - Y_I D_1^{-1} Y_J^T,   S_IK <- E_I = Y_I D_1^{-1} L^{-1}.
// Step K, five launches over every matrix:
//   pivot      (a work-group per matrix): L and D_1;
//   panel read (64-row tiles): which tiles of C = S_:K are not zero, and those
//              above K, stored in K's tile rows, turned round;
//   scale      (64-row tiles): Y and E by substitution in 16-column blocks, and
//              E_K = D^{-1};
//   update     (kept 64 x 64 tiles outside K): S_IJ <- S_IJ - Y_I D_1^{-1} Y_J^T;
//   panel write: S_IK <- E_I below K, S_KI <- E_I^T above it, S_KK <- -D^{-1}.
// The last block may be narrower (w < 128 columns): D is padded with the
// identity, and the panel columns beyond w are zero, so they change nothing.
// Loads run unconditionally from clamped indices and what lies outside is
// selected away or never stored: a load under a lane condition makes the
// compiler wait for each one in turn (that alone cost the update kernel 2.5x).
// All products run on the FP64 matrix cores (16x16x4 MFMA).
constexpr int GJ_NB = kGjNb;   // 128
static_assert(GJ_NB == 128, "the sweep kernels are written for 128-column blocks of two 64-wide tiles");

// Step K of a 16 x 16 L D L^T factorisation without pivoting, in one wave's
// accumulator layout (d[v]: row kq + 4 v, column ln): rows below K are reduced by
// row K, and L^{-1} grows in place of the zeros (d = D on the diagonal).
template <int K>
__device__ __forceinline__ void ldl16_step(Mfma<double>::acc_t& d, int kq, int ln) {
  const double rk = __shfl(d[K >> 2], (K & 3) * 16 + ln, 64);   // row K at this lane's column
  const double ip = 1.0 / dpp_move<0x150 + K>(rk);              // row_newbcast: lane K of the row of 16
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const double l = dpp_move<0x150 + K>(d[v]) * ip;   // column K at this lane's row
    const double x = ln == K ? -l : d[v] - l * rk;
    d[v] = Mfma<double>::row(kq, v) > K ? x : d[v];
  }
}

// L D L^T of the 128 x 128 pivot block without pivoting, one work-group of 1024
// threads per matrix, 16 columns at a time; wave w holds tiles (w / 2, 4 (w mod 2)
// + t), t < 4, in MFMA accumulators, of which those on or right of the diagonal
// count.  Per step the wave with the diagonal tile factorises it in registers (DPP
// and shuffles, no barrier), and P = L_kk^{-1} S_k: and the update S_ij -= P_i^T
// D^{-1} P_j run on the matrix cores: two barriers a step.  Bound by the eight
// chains of 15 divisions: 51 us for 300 boxes, 41 on average over the sweeps of a
// 512^2 annulus's rebuild.  Out: piv holds L below its 16 x 16 diagonal blocks,
// which are L_kk^{-1} (row-major, 128 wide; nothing above them), then 1 / D.
// (The inverses of the 16 x 16 tiles themselves in place of the factors, which
// are as ill-conditioned as the block, cost all digits on stiff structures: thin
// membrane at 256^2, 16 x 16/4 boxes, kappa = 2.6e8, mu = 0.01: a sweep's error
// 2.5e-2.)
__global__ void __launch_bounds__(1024) k_sw_pivot(const double* __restrict__ mats, int n, int kb, int w,
                                                   double* __restrict__ piv_all) {
  constexpr int LD = 18;            // row stride in LDS: operand reads of 16 rows without bank conflicts
  constexpr int LP = GJ_NB + 2;
  __shared__ double Rs[16 * LP], Ps[16 * LP];
  __shared__ double Ls[2][16 * LD];
  __shared__ double ri[GJ_NB];
  const double* A = mats + (size_t)blockIdx.x * n * n;
  double* Pv = piv_all + (size_t)blockIdx.x * kGjPivot;
  // (the wave's number as a scalar: a branch on it is then a branch, and no exec
  // mask changes while products are in flight)
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, kq = lane >> 4, ln = lane & 15;
  const int rt = wave >> 1, c0 = 4 * (wave & 1);
  // the padding of a narrow last block is the identity, so the pivots stay
  // nonzero; the padded rows and columns never reach the matrix.  Above the
  // diagonal tiles only tile (K1, K0) is kept: D[a][b] with a in the first
  // half and b in the second is read as D[b][a].
  Mfma<double>::acc_t d[4];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int a = 16 * rt + Mfma<double>::row(kq, v), b = 16 * (c0 + t) + ln;
      const int ac = a < w ? a : w - 1, bc = b < w ? b : w - 1;
      const bool upper = (ac >> 6) < (bc >> 6);
      const double x = A[(size_t)(kb + (upper ? bc : ac)) * n + kb + (upper ? ac : bc)];
      d[t][v] = a < w && b < w ? x : (a == b ? 1.0 : 0.0);
    }
  for (int kk = 0; kk < GJ_NB / 16; ++kk) {
    double* L = Ls[kk & 1];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (rt != kk) continue;
      if (c0 + t > kk) {
#pragma unroll
        for (int v = 0; v < 4; ++v) Rs[Mfma<double>::row(kq, v) * LP + 16 * (c0 + t) + ln] = d[t][v];
      } else if (c0 + t == kk) {
        Mfma<double>::acc_t x = d[t];
        ldl16_step<0>(x, kq, ln);
        ldl16_step<1>(x, kq, ln);
        ldl16_step<2>(x, kq, ln);
        ldl16_step<3>(x, kq, ln);
        ldl16_step<4>(x, kq, ln);
        ldl16_step<5>(x, kq, ln);
        ldl16_step<6>(x, kq, ln);
        ldl16_step<7>(x, kq, ln);
        ldl16_step<8>(x, kq, ln);
        ldl16_step<9>(x, kq, ln);
        ldl16_step<10>(x, kq, ln);
        ldl16_step<11>(x, kq, ln);
        ldl16_step<12>(x, kq, ln);
        ldl16_step<13>(x, kq, ln);
        ldl16_step<14>(x, kq, ln);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = Mfma<double>::row(kq, v);
          const double l = ln < i ? x[v] : (ln == i ? 1.0 : 0.0);
          L[i * LD + ln] = l;
          Pv[(size_t)(16 * kk + i) * GJ_NB + 16 * kk + ln] = l;
          if (ln == i) ri[16 * kk + i] = 1.0 / x[v];
        }
      }
    }
    __syncthreads();
    if (wave < GJ_NB / 16 && wave > kk) {   // P for column tile `wave`
      Mfma<double>::acc_t p = {0, 0, 0, 0};
#pragma unroll
      for (int st = 0; st < 4; ++st)
        p = Mfma<double>::mma(L[ln * LD + 4 * st + kq], Rs[(4 * st + kq) * LP + 16 * wave + ln], p);
#pragma unroll
      for (int v = 0; v < 4; ++v) Ps[Mfma<double>::row(kq, v) * LP + 16 * wave + ln] = p[v];
    }
    __syncthreads();
    // R is next written after this barrier, P after the next one; L alternates
    if (wave < GJ_NB / 16 && wave > kk) {   // L's tile (wave, kk) = (D^{-1} P)^T
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = 16 * wave + (lane >> 4) + 4 * q;
        Pv[(size_t)i * GJ_NB + 16 * kk + ln] = Ps[ln * LP + i] * ri[16 * kk + ln];
      }
    }
    if (rt > kk) {
      double a[4];
#pragma unroll
      for (int st = 0; st < 4; ++st)
        a[st] = -Ps[(4 * st + kq) * LP + 16 * rt + ln] * ri[16 * kk + 4 * st + kq];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (c0 + t < rt) continue;
#pragma unroll
        for (int st = 0; st < 4; ++st)
          d[t] = Mfma<double>::mma(a[st], Ps[(4 * st + kq) * LP + 16 * (c0 + t) + ln], d[t]);
      }
    }
  }
  if (tid < GJ_NB) Pv[(size_t)GJ_NB * GJ_NB + tid] = ri[tid];   // (written before the last barriers)
}

struct GjTileSmem {
  double Xs[32][65];   // [reduction index of the chunk][row]
  double Ys[32][65];   // [reduction index of the chunk][column]
};

// flags[I]: whether tile I of S_:K outside K has a nonzero (a NaN counts); above K
// (S_I,Kh = S_Kh,I^T from tile row Kh) the nonzero tiles are turned round into C,
// n x 128 (row stride 128), one 64-column half at a time.
__global__ void __launch_bounds__(256) k_sw_panel_read(const double* __restrict__ mats, int n, int kb, int w, int lo,
                                                       double* __restrict__ work, int* __restrict__ flags) {
  __shared__ double Ts[64][65];   // [row of the tile][column of the half]
  const int I = lo + blockIdx.x, I0 = I * 64, K0 = kb / 64, Ke = (kb + w + 63) / 64;
  if (I >= K0 && I < Ke) return;
  const double* A = mats + (size_t)blockIdx.y * n * n;
  double* C = work + (size_t)blockIdx.y * sweep_panels(n);
  int* flag = flags + (size_t)blockIdx.y * ((n + 63) / 64) + I;
  const int tid = threadIdx.x;
  int any = 0;
  if (I >= Ke) {
    const int k = kb + ((tid & 127) < w ? tid & 127 : w - 1);
#pragma unroll
    for (int q = 0; q < 32; ++q) {
      const int i = I0 + (tid >> 7) + 2 * q;
      any |= !(A[(size_t)(i < n ? i : n - 1) * n + k] == 0.0);
    }
    any = __syncthreads_or(any);
    if (tid == 0) *flag = any;
    return;
  }
  double x[2][16];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int k = 64 * h + (tid >> 6) + 4 * q;
      x[h][q] = A[(size_t)(kb + (k < w ? k : w - 1)) * n + I0 + (tid & 63)];
      x[h][q] = k < w ? x[h][q] : 0.0;
      any |= !(x[h][q] == 0.0);
    }
  any = __syncthreads_or(any);
  if (tid == 0) *flag = any;
  if (!any) return;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int q = 0; q < 16; ++q) Ts[tid & 63][(tid >> 6) + 4 * q] = x[h][q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int a = (tid >> 6) + 4 * q, k = tid & 63;
      C[(size_t)(I0 + a) * GJ_NB + 64 * h + k] = Ts[a][k];
    }
    __syncthreads();
  }
}

// Lanes of a wave exchange a 16 x 16 tile through LDS: from the accumulator layout
// to the MFMA's A operand (a[st]: row ln, column 4 st + kq).
__device__ __forceinline__ void tile_to_a(double* xs, const Mfma<double>::acc_t& x, double (&a)[4], int kq, int ln) {
  constexpr int LD = 18;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int v = 0; v < 4; ++v) xs[Mfma<double>::row(kq, v) * LD + ln] = x[v];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int st = 0; st < 4; ++st) a[st] = xs[ln * LD + 4 * st + kq];
}

// row of entry t of a lower triangle stored row by row
__host__ __device__ constexpr int tri_row(int t) {
  int j = 0;
  while ((j + 1) * (j + 2) / 2 <= t) ++j;
  return j;
}

// Every 64-row tile I >= lo that is not zero: Y_I = C_I L^{-T} (to Yw), and for I
// >= re also E_I = Y_I D^{-1} L^{-1} (in place of C), by substitution in 16-column
// blocks on the matrix cores, with S_KK = L D L^T from k_sw_pivot (L^{-1} of the 16 x
// 16 diagonal blocks only).  A tile of K itself (I >= re) takes the identity for C
// and so gets E_K = S_KK^{-1}.  L's 36 blocks lie in LDS (83 KB); a wave takes 16 rows
// at a time, whose Y and E blocks stay in registers.  Bound by each wave's chain of
// products through LDS, so a work-group (one fits a CU; gpm per matrix, on one XCD)
// has eight waves, which share out the matrix's rows: 207 us a step for 300 boxes,
// 121 to 141 on average over the sweeps of a 512^2 annulus's rebuild (299 with a
// work-group of four waves per tile, 220 with the loads of C under conditions).
constexpr int kSwMaxTiles = 1024;   // most 64-row tiles of a swept matrix
__global__ void __launch_bounds__(512) k_sw_scale(const double* __restrict__ mats, const double* __restrict__ piv_all,
                                                  int n, int kb, int w, int lo, int re, int gpm, int count,
                                                  double* __restrict__ work, const int* __restrict__ flags) {
  constexpr int NB = GJ_NB / 16, LD = 18;
  __shared__ double Lb[NB * (NB + 1) / 2][16 * LD];   // block (j, k), k <= j, at j (j + 1) / 2 + k
  __shared__ double xs[8][16 * LD];
  __shared__ double ri[GJ_NB];
  __shared__ unsigned short act[kSwMaxTiles];
  __shared__ int nact;
  const int slot = blockIdx.x >> 3, mat = (slot / gpm) * 8 + (blockIdx.x & 7), first = slot % gpm;
  if (mat >= count) return;
  // (the wave's number as a scalar: a branch on it is then a branch, and no exec
  // mask changes while products are in flight)
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, kq = lane >> 4, ln = lane & 15;
  const int T = (n + 63) / 64, K0 = kb / 64, Ke = (kb + w + 63) / 64;
  const double* Pv = piv_all + (size_t)mat * kGjPivot;
  {
    double l[NB * (NB + 1) / 4];   // half of the threads a block each
    const int i = (tid >> 4) & 15, c = tid & 15, half = wave >> 2;
#pragma unroll
    for (int u = 0; u < NB * (NB + 1) / 4; ++u) {
      const int j = half ? tri_row(2 * u + 1) : tri_row(2 * u), k = 2 * u + half - j * (j + 1) / 2;
      l[u] = Pv[(size_t)(16 * j + i) * GJ_NB + 16 * k + c];
    }
#pragma unroll
    for (int u = 0; u < NB * (NB + 1) / 4; ++u) Lb[2 * u + half][i * LD + c] = l[u];
  }
  if (tid < GJ_NB) ri[tid] = Pv[(size_t)GJ_NB * GJ_NB + tid];
  if (wave == 7) {   // the tiles to do, in order
    int c = 0;
    for (int i0 = lo; i0 < T; i0 += 64) {
      const int I = i0 + lane;
      const bool on = I < T && (I >= K0 && I < Ke ? I >= re : flags[(size_t)mat * T + I] != 0);
      const unsigned long long m = __ballot(on);
      if (on) act[c + __popcll(m & ((1ull << lane) - 1))] = (unsigned short)I;
      c += __popcll(m);
    }
    if (lane == 0) nact = c;
  }
  __syncthreads();
  double* C = work + (size_t)mat * sweep_panels(n);
  double* Y = C + sweep_panels(n) / 2;
  const double* A = mats + (size_t)mat * n * n;
  const int q1 = __builtin_amdgcn_readfirstlane(4 * nact);
  for (int q = first * 8 + wave; q < q1; q += 8 * gpm) {
    const int I = __builtin_amdgcn_readfirstlane(act[q >> 2]), r0 = 64 * I + 16 * (q & 3);   // the wave's rows r0 ..
    const bool in_k = I >= K0 && I < Ke;
    if (r0 >= n) continue;
    // C in accumulator layout
    Mfma<double>::acc_t y[NB];
    if (in_k) {
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) y[j][v] = r0 + Mfma<double>::row(kq, v) - kb == 16 * j + ln ? 1.0 : 0.0;
    } else {
      const double* c = I >= Ke ? A + kb : C;
      const size_t ld = I >= Ke ? n : GJ_NB;
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = r0 + Mfma<double>::row(kq, v), k = 16 * j + ln;
          y[j][v] = c[(size_t)(r < n ? r : n - 1) * ld + (k < w ? k : w - 1)];
        }
      if (w < GJ_NB)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) y[j][v] = 16 * j + ln < w ? y[j][v] : 0.0;
    }
    double a[NB][4];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      Mfma<double>::acc_t x = y[j];
#pragma unroll
      for (int k = 0; k < j; ++k)
#pragma unroll
        for (int st = 0; st < 4; ++st)
          x = Mfma<double>::mma(a[k][st], Lb[j * (j + 1) / 2 + k][ln * LD + 4 * st + kq], x);
      double t[4];
      tile_to_a(xs[wave], x, t, kq, ln);
      x = Mfma<double>::acc_t{0, 0, 0, 0};
#pragma unroll
      for (int st = 0; st < 4; ++st) x = Mfma<double>::mma(t[st], Lb[j * (j + 1) / 2 + j][ln * LD + 4 * st + kq], x);
      y[j] = x;
      // (the panels have whole blocks of 16 rows, so no store needs a condition)
#pragma unroll
      for (int v = 0; v < 4; ++v) Y[(size_t)(r0 + Mfma<double>::row(kq, v)) * GJ_NB + 16 * j + ln] = x[v];
      x = -x;   // (the next blocks subtract)
      tile_to_a(xs[wave], x, a[j], kq, ln);
    }
    if (I < re) continue;
#pragma unroll
    for (int k = NB - 1; k >= 0; --k) {
      Mfma<double>::acc_t x = y[k] * ri[16 * k + ln];
#pragma unroll
      for (int j = NB - 1; j > k; --j)
#pragma unroll
        for (int st = 0; st < 4; ++st)
          x = Mfma<double>::mma(a[j][st], Lb[j * (j + 1) / 2 + k][(4 * st + kq) * LD + ln], x);
      double t[4];
      tile_to_a(xs[wave], x, t, kq, ln);
      x = Mfma<double>::acc_t{0, 0, 0, 0};
#pragma unroll
      for (int st = 0; st < 4; ++st) x = Mfma<double>::mma(t[st], Lb[k * (k + 1) / 2 + k][(4 * st + kq) * LD + ln], x);
#pragma unroll
      for (int v = 0; v < 4; ++v) C[(size_t)(r0 + Mfma<double>::row(kq, v)) * GJ_NB + 16 * k + ln] = x[v];
      x = -x;
      tile_to_a(xs[wave], x, a[k], kq, ln);
    }
  }
}

// S_IJ <- S_IJ - Y_I D^{-1} Y_J^T over the kept tiles I >= J >= lo outside K (tiles K0
// .. Ke - 1) whose panels are not zero, rows I >= r0 only.  gpm work-groups per
// matrix share out the pairs of its active tiles in row order; a matrix's
// work-groups run on one XCD (work-groups go to the eight in turn), whose L2
// holds its panels.  Both 64 x 128 panels of a pair lie in LDS (133 of its 160
// KB, Y_I D^{-1} kept along a row, rows padded to 130 values so that operand reads meet
// no bank conflicts), the next pair's panels and tile load into registers during
// the MFMA steps, and the accumulators start from the old tile.  Bound by the
// FP64 matrix cores and the turn between pairs: 300 boxes of 55 active pairs
// take 490 us, 35 TFLOP/s (635 us with loads under lane conditions).
__global__ void __launch_bounds__(512) k_sw_update(double* __restrict__ mats, int n, int kb, int w, int lo, int r0,
                                                   int gpm, int count, const double* __restrict__ work,
                                                   const double* __restrict__ piv_all, const int* __restrict__ flags) {
  constexpr int LD = GJ_NB + 2;
  __shared__ double Xs[64 * LD], Ys[64 * LD];
  __shared__ unsigned short act[kSwMaxTiles];
  __shared__ int nact, nskip;
  const int slot = blockIdx.x >> 3, mat = (slot / gpm) * 8 + (blockIdx.x & 7), first = slot % gpm;
  if (mat >= count) return;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int T = (n + 63) / 64, K0 = kb / 64, Ke = (kb + w + 63) / 64;
  if (wave == 0) {   // the active tiles, in order; nskip of them lie above r0
    int c = 0, sk = 0;
    for (int i0 = lo; i0 < T; i0 += 64) {
      const int I = i0 + lane;
      const bool on = I < T && !(I >= K0 && I < Ke) && flags[(size_t)mat * T + I];
      const unsigned long long m = __ballot(on);
      if (on) act[c + __popcll(m & ((1ull << lane) - 1))] = (unsigned short)I;
      sk += __popcll(__ballot(on && I < r0));
      c += __popcll(m);
    }
    if (lane == 0) {
      nact = c;
      nskip = sk;
    }
  }
  __syncthreads();
  const int pa = nskip * (nskip + 1) / 2, pairs = nact * (nact + 1) / 2 - pa;
  const int per = (pairs + gpm - 1) / gpm;
  int p = pa + first * per;
  const int p1 = p + per < pa + pairs ? p + per : pa + pairs;
  if (p >= p1) return;
  double* A = mats + (size_t)mat * n * n;
  const double* Yw = work + (size_t)mat * sweep_panels(n) + sweep_panels(n) / 2;
  const int wr = wave & 1, wc = wave >> 1, kq = lane >> 4, ln = lane & 15;   // rows 32 wr, columns 16 wc
  const int lr = tid >> 7, lk = tid & 127;   // panel loads: rows lr + 4 q, column lk
  const double md = -piv_all[(size_t)mat * kGjPivot + GJ_NB * GJ_NB + lk];   // -1 / D
  double xr[16], yr[16], old[2][4];
  auto load_y = [&](int I, double (&y)[16]) {
    const double* Y = Yw + (size_t)I * 64 * GJ_NB;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int a = lr + 4 * q;
      y[q] = Y[(size_t)(I * 64 + a < n ? a : n - 1 - I * 64) * GJ_NB + lk];
    }
  };
  auto load_old = [&](int I, int J) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = 64 * I + 32 * wr + 16 * a + Mfma<double>::row(kq, v), j = 64 * J + 16 * wc + ln;
        old[a][v] = A[(size_t)(i < n ? i : n - 1) * n + (j < n ? j : n - 1)];
      }
  };
  int ri = (int)((sqrtf(8.0f * (float)p + 1.0f) - 1.0f) * 0.5f);   // row and column of pair p among the active
  while (ri * (ri + 1) / 2 > p) --ri;
  while ((ri + 1) * (ri + 2) / 2 <= p) ++ri;
  int rj = p - ri * (ri + 1) / 2;
  bool fresh = true;   // Y of the current row is in registers, not yet in LDS
  load_y(act[ri], xr);
  load_y(act[rj], yr);
  load_old(act[ri], act[rj]);
  for (; p < p1; ++p) {
    const int I0 = act[ri] * 64, J0 = act[rj] * 64;
    __syncthreads();   // the last pair's operand reads are done
    if (fresh)
#pragma unroll
      for (int q = 0; q < 16; ++q) Xs[(lr + 4 * q) * LD + lk] = md * xr[q];
#pragma unroll
    for (int q = 0; q < 16; ++q) Ys[(lr + 4 * q) * LD + lk] = yr[q];
    Mfma<double>::acc_t acc[2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[a][v] = old[a][v];
    __syncthreads();
    fresh = rj == ri;
    ri += fresh ? 1 : 0;
    rj = fresh ? 0 : rj + 1;
    if (p + 1 < p1) {   // no work-group of this launch writes another's tile or Y
      if (fresh) load_y(act[ri], xr);
      load_y(act[rj], yr);
      load_old(act[ri], act[rj]);
    }
    const double* xa = Xs + (32 * wr + ln) * LD + kq;
    const double* xb = xa + 16 * LD;
    const double* yb = Ys + (16 * wc + ln) * LD + kq;
#pragma unroll 8
    for (int st = 0; st < GJ_NB / 4; ++st) {
      const double b0 = yb[4 * st];
      acc[0] = Mfma<double>::mma(xa[4 * st], b0, acc[0]);
      acc[1] = Mfma<double>::mma(xb[4 * st], b0, acc[1]);
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = I0 + 32 * wr + 16 * a + Mfma<double>::row(kq, v), j = J0 + 16 * wc + ln;
        if (i < n && j < n) A[(size_t)i * n + j] = acc[a][v];
      }
  }
}

// Row and column K of the swept matrix, one 64-row tile I = lo + blockIdx.x per
// work-group: the kept tiles of S_KK <- -E_K; below K, S_I,Kh <- E_I's half h;
// above K, S_Kh,I <- that half transposed.
__global__ void __launch_bounds__(256) k_sw_panel_write(double* __restrict__ mats, int n, int kb, int w, int lo,
                                                        const double* __restrict__ work,
                                                        const int* __restrict__ flags) {
  __shared__ double Ts[64][65];
  const int I = lo + blockIdx.x, I0 = I * 64, K0 = kb / 64, Ke = (kb + w + 63) / 64;
  if (!(I >= K0 && I < Ke) && !flags[(size_t)blockIdx.y * ((n + 63) / 64) + I]) return;   // stays zero
  double* A = mats + (size_t)blockIdx.y * n * n;
  const double* E = work + (size_t)blockIdx.y * sweep_panels(n);
  const int tid = threadIdx.x;
  if (I >= K0 && I < Ke) {
    // row tile I of K's kept lower part: columns 0 .. 64 (I - K0) + 63
    const int r0 = 64 * (I - K0);
    for (int h = 0; h <= I - K0; ++h) {
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int t = tid + 256 * q, a = t >> 6, b = t & 63;
        const int cb = 64 * h + b;
        const double x = -E[(size_t)(r0 + a < w ? I0 + a : n - 1) * GJ_NB + cb];
        if (r0 + a < w && cb < w) A[(size_t)(I0 + a) * n + kb + cb] = x;
      }
    }
    return;
  }
  if (I >= Ke) {    // S_IK <- E_I
    double x[32];
#pragma unroll
    for (int q = 0; q < 32; ++q) {
      const int i = I0 + (tid >> 7) + 2 * q;
      x[q] = E[(size_t)(i < n ? i : n - 1) * GJ_NB + (tid & 127)];
    }
#pragma unroll
    for (int q = 0; q < 32; ++q) {
      const int i = I0 + (tid >> 7) + 2 * q;
      if (i < n && (tid & 127) < w) A[(size_t)i * n + kb + (tid & 127)] = x[q];
    }
    return;
  }
  // above K the kept tiles are S_Kh,I <- (E_I's half h)^T
  for (int h = 0; h < 2; ++h) {
    const int wh = w - 64 * h;
    if (wh <= 0) break;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int t = tid + 256 * q, a = t >> 6, k = t & 63;
      Ts[a][k] = E[(size_t)(I0 + a) * GJ_NB + 64 * h + k];   // above K: whole tiles
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int t = tid + 256 * q, k = t >> 6, c = t & 63, i = I0 + c;
      if (k < wh) A[(size_t)(kb + 64 * h + k) * n + i] = Ts[c][k];
    }
    __syncthreads();
  }
}

// One step of the sweeps: block [kb, kb + w) (w <= 128, kb a multiple of 64, w
// too unless the block ends the matrix) within the tiles from lo on; partial:
// the rows below the block only.
static void sweep_step(double* mats, int n, int kb, int w, int lo, bool partial, int count, double* work, double* piv,
                       int* flags, hipStream_t s) {
  const int T = (n + 63) / 64, Ke = (kb + w + 63) / 64;
  IBMG_KLAUNCH(k_sw_pivot, dim3(count), dim3(1024), 0, s, mats, n, kb, w, piv);
  IBMG_LAUNCH_CHECK();
  IBMG_KLAUNCH(k_sw_panel_read, dim3(T - lo, count), dim3(256), 0, s, mats, n, kb, w, lo, work, flags);
  IBMG_LAUNCH_CHECK();
  const int r0 = partial ? Ke : lo;   // first row tile of E and of the panel
  if (T - r0 > 0) {
    const int gps = std::min((T - lo + 1) / 2, std::max(1, 768 / count)), c8 = (count + 7) / 8 * 8;
    IBMG_KLAUNCH(k_sw_scale, dim3(gps * c8), dim3(512), 0, s, mats, piv, n, kb, w, lo, r0, gps, count, work, flags);
    IBMG_LAUNCH_CHECK();
    // work-groups per matrix (one fits a CU): a pair each for a few matrices,
    // else enough for six rounds of the device, so that matrices with more
    // active pairs even out
    const int t = T - lo, pairs = t * (t + 1) / 2, gpm = std::min(pairs, std::max(4, 1536 / count));
    IBMG_KLAUNCH(k_sw_update, dim3(gpm * c8), dim3(512), 0, s, mats, n, kb, w, lo, r0, gpm, count,
                 work, piv, flags);
    IBMG_LAUNCH_CHECK();
    IBMG_KLAUNCH(k_sw_panel_write, dim3(T - r0, count), dim3(256), 0, s, mats, n, kb, w, r0, work, flags);
    IBMG_LAUNCH_CHECK();
  }
}

// the parts of a sweep's workspace (sweep_work)
static double* sweep_piv(double* work, int n, int count) { return work + (size_t)count * sweep_panels(n); }
static int* sweep_flags(double* work, int n, int count) {
  return reinterpret_cast<int*>(sweep_piv(work, n, count) + (size_t)count * kGjPivot);
}

void launch_gj_invert(double* mats, int n, int count, double* work, hipStream_t s) {
  if (!count) return;
  if (n > 64 * kSwMaxTiles) throw Error(IBMG_ERR_ARG, "matrix too large for the block sweeps");
  for (int kb = 0; kb < n; kb += GJ_NB)
    sweep_step(mats, n, kb, std::min(GJ_NB, n - kb), 0, false, count, work, sweep_piv(work, n, count),
               sweep_flags(work, n, count), s);
}

void launch_box_eliminate(double* mats, BoxMat bm, int count, double* work, hipStream_t s) {
  if (!count) return;
  if (bm.nnp % 64) throw Error(IBMG_ERR_ARG, "the owned unknowns start at a tile");
  if (bm.ld > 64 * kSwMaxTiles) throw Error(IBMG_ERR_ARG, "matrix too large for the block sweeps");
  double* piv = sweep_piv(work, bm.ld, count);
  int* flags = sweep_flags(work, bm.ld, count);
  for (int kb = 0; kb < bm.nnp; kb += GJ_NB)
    sweep_step(mats, bm.ld, kb, std::min(GJ_NB, bm.nnp - kb), 0, true, count, work, piv, flags, s);
  for (int kb = bm.nnp; kb < bm.ld; kb += GJ_NB)
    sweep_step(mats, bm.ld, kb, std::min(GJ_NB, bm.ld - kb), bm.nnp / 64, false, count, work, piv, flags, s);
}

// The inverse's owned rows at the non-owned columns, M_on = S_oo^{-1} (-W), for
// the boxes that keep whole rows: after the elimination the kept tiles of o hold
// -S_oo^{-1} and the rows o hold W, so M_on is their product.  One 64 x 64 tile
// per work-group (four waves of 2 x 2 MFMA tiles, the reduction through LDS 32
// indices at a time); the result goes, transposed, to the unused block right of
// n: M_on[r][j] at (j, nnp + r).
__global__ void __launch_bounds__(256) k_box_on(double* __restrict__ mats, BoxMat bm) {
  __shared__ GjTileSmem sm;
  double* A = mats + (size_t)blockIdx.z * bm.ld * bm.ld;
  const int nown = bm.ld - bm.nnp, R0 = blockIdx.x * 64, J0 = blockIdx.y * 64, ld = bm.ld;
  const double* O = A + (size_t)bm.nnp * ld + bm.nnp;   // the owned block
  const double* W = A + (size_t)bm.nnp * ld;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wr = wave & 1, wc = wave >> 1, kq = lane >> 4, ln = lane & 15;
  Mfma<double>::acc_t acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = Mfma<double>::acc_t{0, 0, 0, 0};
  double xr[8], yr[8];
  auto load = [&](int k0) {
    const bool below = (k0 >> 6) <= (R0 >> 6);   // the tile (R0, k0) is a kept one
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int t = tid + 256 * q;
      const int r = R0 + (below ? t >> 5 : t & 63), k = k0 + (below ? t & 31 : t >> 6);
      const int rc = r < nown ? r : nown - 1, kc = k < nown ? k : nown - 1;
      xr[q] = O[(size_t)(below ? rc : kc) * ld + (below ? kc : rc)];
      xr[q] = k < nown ? xr[q] : 0.0;
      const int kb = k0 + (t >> 6), j = J0 + (t & 63);
      yr[q] = W[(size_t)(kb < nown ? kb : nown - 1) * ld + (j < bm.nn ? j : bm.nn - 1)];
    }
  };
  load(0);
#pragma unroll 1
  for (int k0 = 0; k0 < nown; k0 += 32) {
    const bool below = (k0 >> 6) <= (R0 >> 6);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int t = tid + 256 * q;
      sm.Xs[below ? t & 31 : t >> 6][below ? t >> 5 : t & 63] = xr[q];
      sm.Ys[t >> 6][t & 63] = yr[q];
    }
    __syncthreads();
    if (k0 + 32 < nown) load(k0 + 32);
#pragma unroll
    for (int st = 0; st < 8; ++st) {
      const int kk = 4 * st + kq;
      const double a0 = sm.Xs[kk][32 * wr + ln], a1 = sm.Xs[kk][32 * wr + 16 + ln];
      const double b0 = sm.Ys[kk][32 * wc + ln], b1 = sm.Ys[kk][32 * wc + 16 + ln];
      acc[0][0] = Mfma<double>::mma(a0, b0, acc[0][0]);
      acc[0][1] = Mfma<double>::mma(a0, b1, acc[0][1]);
      acc[1][0] = Mfma<double>::mma(a1, b0, acc[1][0]);
      acc[1][1] = Mfma<double>::mma(a1, b1, acc[1][1]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = R0 + 32 * wr + 16 * a + Mfma<double>::row(kq, v), j = J0 + 32 * wc + 16 * b + ln;
        if (r < nown && j < bm.nn) A[(size_t)j * ld + bm.nnp + r] = acc[a][b][v];
      }
}

void launch_box_on(double* mats, BoxMat bm, int count, hipStream_t s) {
  if (!count) return;
  const int nown = bm.ld - bm.nnp;
  IBMG_KLAUNCH(k_box_on, dim3((nown + 63) / 64, (bm.nn + 63) / 64, count), dim3(256), 0, s, mats, bm);
  IBMG_LAUNCH_CHECK();
}

// entry (owned position r, owned position q) of an eliminated box's inverse
__device__ __forceinline__ double box_oo(const double* A, const BoxMat& bm, int r, int q) {
  const int i = bm.nnp + r, j = bm.nnp + q;
  return -((i >> 6) >= (j >> 6) ? A[(size_t)i * bm.ld + j] : A[(size_t)j * bm.ld + i]);
}
// entry (owned unknown r, local unknown p: non-owned position or nnp + owned
// unknown) of an eliminated box's inverse (launch_box_on for p < nnp); own: the
// owned unknowns' positions
__device__ __forceinline__ double box_inv_at(const double* A, const BoxMat& bm, const unsigned short* own, int r, int p) {
  return p < bm.nnp ? A[(size_t)p * bm.ld + bm.nnp + own[r]] : box_oo(A, bm, own[r], own[p - bm.nnp]);
}

// global index of local unknown k of box pid (periodic wrap)
__device__ __forceinline__ size_t box_glob(const BoxGeom& g, int pid, int k) {
  const int N = g.N, m = g.m, nu = m * (m + 1);
  const int x0 = (pid % g.npd) * g.b - g.o, y0 = (pid / g.npd) * g.b - g.o;
  const size_t nn = (size_t)N * N;
  int ii, jj;
  size_t off;
  if (k < nu) {
    ii = k % (m + 1);
    jj = k / (m + 1);
    off = 0;
  } else if (k < 2 * nu) {
    const int q = k - nu;
    ii = q % m;
    jj = q / m;
    off = nn;
  } else {
    const int q = k - 2 * nu;
    ii = q % m;
    jj = q / m;
    off = 2 * nn;
  }
  return off + (size_t)pmod(y0 + jj, N) * N + pmod(x0 + ii, N);
}

// global index of owned row r of box pid
__device__ __forceinline__ size_t own_glob(const BoxGeom& g, int pid, int r) {
  const int bb = g.b * g.b;
  const int comp = r / bb, q = r % bb;
  const int gi = (pid % g.npd) * g.b + q % g.b, gj = (pid / g.npd) * g.b + q / g.b;
  return (size_t)comp * g.N * g.N + (size_t)gj * g.N + gi;
}

// box and vector offset of an entry (SYS: of many systems); false: its system is
// not active
template <bool SYS>
__device__ __forceinline__ bool box_entry(const BoxGeom& g, int ent, int& pid, size_t& base) {
  pid = ent;
  base = 0;
  if (!SYS) return true;
  const int sys = ent / g.nbs;
  pid = ent - sys * g.nbs;
  base = sys * g.sysn;
  return !g.act || g.act[sys];
}

// Rows of A^{-1}, stored per box as row chunks of 64: element (row, j)
// at (row / 64) * nloc * 64 + j * 64 + row % 64 (rows beyond nown are 0), so
// a chunk's 64 rows of one column are contiguous and a chunk is one
// contiguous stream of nloc * 64 values.  bo.pos = null: every row of a swept
// matrix (the summed combination); else the owned rows of an eliminated one.
template <typename T>
__global__ void k_extract_rows(const double* __restrict__ mats, int count, BoxGeom g, BoxMat bm, BoxOrder bo,
                               T* __restrict__ out) {
  const size_t per = (size_t)g.nch * g.nloc * 64;
  const size_t tot = per * count;
  for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < tot; t += (size_t)gridDim.x * blockDim.x) {
    const size_t blk = t / per;
    size_t rem = t % per;
    const int c = (int)(rem / ((size_t)g.nloc * 64));
    rem %= (size_t)g.nloc * 64;
    const int j = (int)(rem / 64), rr = (int)(rem % 64);
    const int row = c * 64 + rr;
    const double* A = mats + blk * bm.ld * bm.ld;
    T v = 0;
    if (row < g.nown) {
      if (bo.pos) v = (T)box_inv_at(A, bm, bo.own + blk * g.nown, row, bo.pos[j]);
      else v = (T)(-((row >> 6) >= (j >> 6) ? A[(size_t)row * bm.ld + j] : A[(size_t)j * bm.ld + row]));
    }
    out[t] = v;
  }
}

template <typename T>
void launch_extract_rows(const double* mats, int count, BoxGeom g, BoxMat bm, BoxOrder bo, T* out, hipStream_t s) {
  if (!count) return;
  size_t tot = (size_t)g.nch * g.nloc * 64 * count;
  int grid = cdiv(tot, 256);
  if (grid > 16384) grid = 16384;
  IBMG_KLAUNCH((k_extract_rows<T>), dim3(grid), dim3(256), 0, s, mats, count, g, bm, bo, out);
  IBMG_LAUNCH_CHECK();
}

// ---------------------------------------------------------------------------
// Eliminated storage of the IB boxes.  Instead of the owned rows of L_k^{-1} a
// box keeps the two factors the elimination leaves (above):
//   W rows: the owned rows coupled to a non-owned unknown (by the stencil along
//           the box's edge or by the IB rows), nn columns each, row-major with
//           a row stride of nn rounded up to a multiple of 4 (the first pass
//           loads 16 bytes: four FP32 values or two FP64 ones);
//   Q:      S_oo^{-1}, symmetric: chunk c (owned rows 64c .. 64c+63) holds the
//           columns 0 .. 64 (c + 1) - 1 of 64 rows each (the tiles on and below
//           the diagonal; zero beyond nown); the others are the transposes of
//           stored entries.
// z_o = Q (r_o - W r_n): two passes instead of one product, but at 16 x 16/4
// with 268 coupled rows of 768 (the mean of the 512^2 annulus's 172 boxes) 4.7
// MB instead of 8.75 MB (symmetric owned block, whole non-owned columns) or
// 10.9 MB (whole rows).
// ---------------------------------------------------------------------------
__host__ __device__ inline size_t sym_chunk_off(int c) { return (size_t)4096 * ((size_t)c * (c + 1) / 2); }
size_t sym_box_stride(const BoxGeom& g) { return sym_chunk_off(g.nch); }
// partials per box, the chunks' columns cut into ks slices: chunk c's 64
// row sums of each slice, then its 64 c column sums
__host__ __device__ inline int sym_part_off(int c, int ks) { return 64 * ks * c + 32 * c * (c - 1); }
// Column slices: enough work-groups to cover the device twice while a slice
// keeps at least two tiles of the longest chunk.
static int sym_ksplit(const BoxGeom& g, int n_ib) {
  int ks = 1;
  while (ks < 4 && n_ib * g.nch * ks < 512 && g.nch / (2 * ks) >= 2) ks *= 2;
  return ks;
}
int sym_part_len(const BoxGeom& g) { return sym_part_off(g.nch, 4); }

template <typename T>
__global__ void k_extract_sym(const double* __restrict__ mats, int count, BoxGeom g, BoxMat bm, T* __restrict__ out) {
  const size_t per = sym_chunk_off(g.nch);
  const size_t tot = per * count;
  for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < tot; t += (size_t)gridDim.x * blockDim.x) {
    const size_t blk = t / per;
    size_t rem = t % per;
    int c = 0;
    while (c + 1 < g.nch && sym_chunk_off(c + 1) <= rem) ++c;
    rem -= sym_chunk_off(c);
    const int q = (int)(rem / 64), row = c * 64 + (int)(rem % 64);
    out[t] = row < g.nown && q < g.nown ? (T)box_oo(mats + blk * bm.ld * bm.ld, bm, row, q) : T(0);
  }
}

template <typename T>
void launch_extract_sym(const double* mats, int count, BoxGeom g, BoxMat bm, T* out, hipStream_t s) {
  if (!count) return;
  const size_t tot = sym_box_stride(g) * count;
  int grid = cdiv(tot, 256);
  if (grid > 16384) grid = 16384;
  IBMG_KLAUNCH((k_extract_sym<T>), dim3(grid), dim3(256), 0, s, mats, count, g, bm, out);
  IBMG_LAUNCH_CHECK();
}

// the W rows of count boxes: rows wptr[i] .. wptr[i+1] of box i, owned position
// wrow
template <typename T>
__global__ void k_extract_w(const double* __restrict__ mats, BoxMat bm, const int* __restrict__ wptr,
                            const int* __restrict__ wrow, int ws, T* __restrict__ out) {
  const double* A = mats + (size_t)blockIdx.y * bm.ld * bm.ld;
  for (int e = wptr[blockIdx.y] + blockIdx.x; e < wptr[blockIdx.y + 1]; e += gridDim.x) {
    const double* Ar = A + (size_t)(bm.nnp + wrow[e]) * bm.ld;
    for (int j = threadIdx.x; j < ws; j += blockDim.x) out[(size_t)e * ws + j] = j < bm.nn ? (T)Ar[j] : T(0);
  }
}

template <typename T>
void launch_extract_w(const double* mats, int count, BoxMat bm, const int* wptr, const int* wrow, int ws, T* out,
                      hipStream_t s) {
  if (!count) return;
  IBMG_KLAUNCH((k_extract_w<T>), dim3(32, count), dim3(256), 0, s, mats, bm, wptr, wrow, ws, out);
  IBMG_LAUNCH_CHECK();
}

// What the eliminated form costs in accuracy in 32 bits: the roundings of W and of
// r_o - W r_n reach z through Q, so against whole rows the mean square error of a
// kind of unknown grows by sum_ik Q_ik^2 (1 + |W_k|^2) / sum_ik Q_ik^2, i over its
// owned positions.  k_w_weight: the weights 1 + |W_k|^2, a wave per row;
// k_elim_loss: both sums of velocities and pressures, every entry of the symmetric Q
// read once, kLossParts work-groups a box and no atomics (the host adds their sums).
// Bound by reading W and Q once from HBM: 175 boxes of 16 x 16/4 247 and 178 us, in
// the set-up of FP32 smoothers only.
__global__ void k_w_weight(const double* __restrict__ mats, BoxMat bm, int nown, double* __restrict__ wt) {
  const double* A = mats + (size_t)blockIdx.y * bm.ld * bm.ld;
  const int lane = threadIdx.x & 63;
  for (int k = blockIdx.x * 4 + (threadIdx.x >> 6); k < nown; k += gridDim.x * 4) {
    const double* Ar = A + (size_t)(bm.nnp + k) * bm.ld;
    double v = 0.0;
    for (int j = lane; j < bm.nn; j += 64) v = fma(Ar[j], Ar[j], v);
    v = wave_sum(v);
    if (lane == 0) wt[(size_t)blockIdx.y * nown + k] = 1.0 + v;
  }
}

__global__ void __launch_bounds__(256) k_elim_loss(const double* __restrict__ mats, BoxMat bm, int nown, int nvel,
                                                   const unsigned short* __restrict__ ord,
                                                   const double* __restrict__ wt, double* __restrict__ out) {
  __shared__ double red[4][4];
  const double* A = mats + (size_t)blockIdx.y * bm.ld * bm.ld;
  const unsigned short* o = ord + (size_t)blockIdx.y * nown;
  const double* w = wt + (size_t)blockIdx.y * nown;
  double s[4] = {0.0, 0.0, 0.0, 0.0};   // weighted and plain, of velocities and of pressures
  for (int i = blockIdx.x; i < nown; i += gridDim.x) {
    const double* Ar = A + (size_t)(bm.nnp + i) * bm.ld + bm.nnp;
    const double wi = w[i], ui = o[i] < nvel ? 1.0 : 0.0;
    for (int k = threadIdx.x; k <= i; k += 256) {
      const double q = Ar[k] * Ar[k], uk = o[k] < nvel ? 1.0 : 0.0;
      const double a = q * w[k], b = k < i ? q * wi : 0.0, c = k < i ? q : 0.0;
      s[0] += ui * a + uk * b;
      s[1] += ui * q + uk * c;
      s[2] += (1.0 - ui) * a + (1.0 - uk) * b;
      s[3] += (1.0 - ui) * q + (1.0 - uk) * c;
    }
  }
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const double v = wave_sum(s[m]);
    if ((threadIdx.x & 63) == 0) red[wave][m] = v;
  }
  __syncthreads();
  if (threadIdx.x < 4)
    out[((size_t)blockIdx.y * gridDim.x + blockIdx.x) * 4 + threadIdx.x] =
        (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
}

void launch_elim_loss(const double* mats, int count, BoxMat bm, BoxGeom g, const unsigned short* ord, double* wt,
                      double* out, hipStream_t s) {
  if (!count) return;
  IBMG_KLAUNCH(k_w_weight, dim3(16, count), dim3(256), 0, s, mats, bm, g.nown, wt);
  IBMG_LAUNCH_CHECK();
  IBMG_KLAUNCH(k_elim_loss, dim3(kLossParts, count), dim3(256), 0, s, mats, bm, g.nown, 2 * g.nown / 3, ord, wt, out);
  IBMG_LAUNCH_CHECK();
}

// ---------------------------------------------------------------------------
// Restricted additive Schwarz (Alg. 2 from a zero guess):
//   z[G~_k] = (L_k^{-1} R_k r)[G~_k]  for every box k.
// The owned sets partition the unknowns, so every z entry is written by
// exactly one work-group and no atomics are needed.
// ---------------------------------------------------------------------------
template <typename T>
struct Vec16;
template <>
struct Vec16<double> {
  typedef double type __attribute__((ext_vector_type(2)));
  static constexpr int n = 2;
};
template <>
struct Vec16<float> {
  typedef float type __attribute__((ext_vector_type(4)));
  static constexpr int n = 4;
};

// Rows rsub R .. (R = 64 / RS) of one (box, 64-row chunk) item, whole columns, by
// NW waves: a wave streams batches of eight 16-byte loads a lane (CP columns of R
// rows side by side per load), the next batch loading during the current one's
// sums and the first before the residual gather.  RS > 1 spreads few boxes over
// the device: a chunk's rows split between work-groups need no partial sums.
constexpr int kRowsPad = 128;   // zeros behind the gathered residual: batches run past nloc
template <typename T, int NW, int RS>
__device__ __forceinline__ void ras_rows_block(const T* __restrict__ r, T* __restrict__ z, const BoxGeom& g,
                                               const T* __restrict__ Mc, int pid, int chunk, int rsub, T* x, T* part,
                                               bool acc_mode) {
  using V = typename Vec16<T>::type;
  constexpr int VEC = Vec16<T>::n, R = 64 / RS, LPC = R / VEC, CP = 64 / LPC, UNR = 8, B = UNR * CP;
  static_assert(B <= kRowsPad, "a batch reads at most the padding");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int cph = lane / LPC, rl = (lane % LPC) * VEC, n = g.nloc;
  Mc += rsub * R + rl;
  V m0[UNR];
  auto load = [&](int jb) {
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int j = jb + cph + u * CP;
      m0[u] = __builtin_nontemporal_load(reinterpret_cast<const V*>(Mc + (size_t)(j < n ? j : n - 1) * 64));
    }
  };
  int jb = wave * B;
  if (jb < n) load(jb);
  for (int k = tid; k < n + kRowsPad; k += 64 * NW) x[k] = k < n ? r[box_glob(g, pid, k)] : T(0);
  __syncthreads();
  T acc[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) acc[v] = 0;
  for (; jb < n; jb += NW * B) {
    V m[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) m[u] = m0[u];
    if (jb + NW * B < n) load(jb + NW * B);
    T xv[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) xv[u] = x[jb + cph + u * CP];
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      T t[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) t[u] = m[u][v] * xv[u];
      acc[v] += ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
    }
  }
  // the column phases, then the waves
#pragma unroll
  for (int off = 32; off >= LPC; off >>= 1)
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] += __shfl_down(acc[v], off, 64);
  if (lane < LPC)
#pragma unroll
    for (int v = 0; v < VEC; ++v) part[wave * R + rl + v] = acc[v];
  __syncthreads();
  const int row = chunk * 64 + rsub * R + tid;
  if (tid < R && row < g.nown) {
    T a = 0;
#pragma unroll
    for (int q = 0; q < NW; q += 2) a += part[q * R + tid] + part[(q + 1) * R + tid];
    const size_t o = own_glob(g, pid, row);
    z[o] = acc_mode ? z[o] + a : a;
  }
}

// First pass of the eliminated boxes: t = W r_n for the rows [lo, hi) of W (row e
// at Wm + e ws; t by position).  Each lane keeps its share of the box's non-owned
// residual in registers (CH 16-byte groups of columns) and every wave streams its
// rows, 16 bytes a lane and load, the next row loading during the current one's
// sum over the wave.
template <typename T, int CH, int NW>
__device__ __forceinline__ void ras_w_block(const T* __restrict__ r, const BoxGeom& g, int pid, const WBoxView& w,
                                            const T* __restrict__ Wm, int lo, int hi, T* __restrict__ t, T* xs) {
  using V = typename Vec16<T>::type;
  constexpr int VEC = Vec16<T>::n;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  V m[CH], nx[CH];
  int pos = 0, npos = 0;
  auto load = [&](int e) {
    npos = w.wrow[e];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int j = (c * 64 + lane) * VEC;
      nx[c] = __builtin_nontemporal_load(reinterpret_cast<const V*>(Wm + (size_t)e * w.ws + (j < w.ws ? j : 0)));
    }
  };
  int e = lo + wave;
  if (e < hi) load(e);
  for (int k = tid; k < CH * 64 * VEC; k += 64 * NW) xs[k] = k < w.nn ? r[box_glob(g, pid, w.nloc[k])] : T(0);
  __syncthreads();
  V x[CH];   // zero where a lane's columns end: its repeated loads count nothing
#pragma unroll
  for (int c = 0; c < CH; ++c)
#pragma unroll
    for (int v = 0; v < VEC; ++v) x[c][v] = xs[(c * 64 + lane) * VEC + v];
  for (; e < hi; e += NW) {
#pragma unroll
    for (int c = 0; c < CH; ++c) m[c] = nx[c];
    pos = npos;
    if (e + NW < hi) load(e + NW);
    T a = 0;
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int v = 0; v < VEC; ++v) a += m[c][v] * x[c][v];
    a = wave_sum(a);
    if (lane == 0) t[pos] = a;
  }
}

// Second pass, z_o = Q y with y = r_o - t on the coupled rows and r_o on the
// others: work-group = (box, 64-row chunk c, column slice),
// longest chunks first.  The chunk's stored columns are cut into gridDim.z
// slices of whole 64-column tiles; a slice's columns stream in batches of UNR x
// VEC (16-byte loads, eight in flight per lane), batches dealt to the four waves
// in turn.  Every column adds its entries times y_q to the rows (lane sums); a
// column of an earlier tile (q < 64 c) also forms its transposed product, the
// sum over the chunk's rows of Q[row][q] y_row, reduced over the lanes of its
// column phase, which belongs to row q of an earlier chunk.  The box's partials:
// the chunk's row sums per slice at sym_part_off(c, ks), its column sums after
// them (each column in one slice).
template <typename T, bool SYS>
__global__ void __launch_bounds__(256) k_ras_ib_sym(const T* __restrict__ r, const T* __restrict__ t, BoxGeom g,
                                                    const int* __restrict__ boxes, WBoxView w,
                                                    const T* __restrict__ inv, const void* const* __restrict__ qtab,
                                                    T* __restrict__ part) {
  using V = typename Vec16<T>::type;
  constexpr int VEC = Vec16<T>::n;
  constexpr int LPC = 64 / VEC;   // lanes per column
  constexpr int UNR = 8, B = UNR * VEC;
  extern __shared__ char smem_raw[];
  T* xs = reinterpret_cast<T*>(smem_raw);
  T* red = xs + 64 * g.nch;       // 4 waves x 64 row sums
  T* tcol = red + 256;            // the chunk's 64 c column sums
  const int slot = blockIdx.x, c = g.nch - 1 - blockIdx.y, sl = blockIdx.z, ks = gridDim.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int cph = lane / LPC, rl = (lane % LPC) * VEC;
  const int ntr = 64 * c, ncol = 64 * (c + 1);
  const int cs = ((ncol + ks - 1) / ks + 63) / 64 * 64;
  const int cb = sl * cs < ncol ? sl * cs : ncol, ce = cb + cs < ncol ? cb + cs : ncol;
  T* pb = part + (size_t)slot * sym_part_off(g.nch, ks) + sym_part_off(c, ks);
  if (cb >= ce) {   // a short chunk's empty slice
    if (tid < 64) pb[64 * sl + tid] = T(0);
    return;
  }
  int pid;
  size_t base;
  if (!box_entry<SYS>(g, boxes[slot], pid, base)) return;
  r += base;
  const T* Q = SYS ? static_cast<const T*>(qtab[slot]) : inv + (size_t)slot * sym_chunk_off(g.nch);
  const T* Mc = Q + sym_chunk_off(c) + rl;
  // the wave's first batch is issued before the residual, so its trip from
  // memory overlaps that one (columns come in whole batches: ce - cb is a
  // multiple of 64)
  const int jb0 = cb + wave * B;
  V m0[UNR];
  auto load = [&](V (&m)[UNR], int jb) {
#pragma unroll
    for (int u = 0; u < UNR; ++u)
      m[u] = __builtin_nontemporal_load(reinterpret_cast<const V*>(Mc + (size_t)(jb + cph + u * VEC) * 64));
  };
  if (jb0 < ce) load(m0, jb0);
  for (int k = tid; k < ncol; k += 256) {
    const size_t at = (size_t)slot * g.nown + (k < g.nown ? k : 0);
    const T ro = r[own_glob(g, pid, w.ord[at])], tk = t[at];
    xs[k] = k < g.nown ? (w.coupled[at] ? ro - tk : ro) : T(0);
  }
  __syncthreads();
  T xr[VEC];   // this lane's rows' values (owned rows 64 c + rl + v)
#pragma unroll
  for (int v = 0; v < VEC; ++v) xr[v] = xs[64 * c + rl + v];
  T acc[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) acc[v] = 0;
  // one column's contribution; tr: the column also needs its transposed sum
  auto column = [&](const V& m, int q, bool tr) {
    const T* a = reinterpret_cast<const T*>(&m);
    const T x = xs[q];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] += a[v] * x;
    if (tr) {
      T p = 0;
#pragma unroll
      for (int v = 0; v < VEC; ++v) p += a[v] * xr[v];
      // the column phase's LPC lanes: rows of 16 by DPP, then across rows
      p = row16_sum(p);
      if constexpr (LPC == 32) p += __shfl_xor(p, 16, 64);
      if (lane % LPC == 0) tcol[q] = p;
    }
  };
  for (int jb = jb0; jb < ce; jb += 4 * B) {
    V m[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) m[u] = m0[u];
    if (jb + 4 * B < ce) load(m0, jb + 4 * B);
    const bool tr = jb < ntr;   // batches never straddle ntr (multiples of 64)
#pragma unroll
    for (int u = 0; u < UNR; ++u) column(m[u], jb + cph + u * VEC, tr);
  }
  // sum the VEC column phases, then the four waves
#pragma unroll
  for (int off = 32; off >= LPC; off >>= 1)
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] += __shfl_down(acc[v], off, 64);
  if (lane < LPC)
#pragma unroll
    for (int v = 0; v < VEC; ++v) red[wave * 64 + rl + v] = acc[v];
  __syncthreads();
  if (tid < 64) pb[64 * sl + tid] = (red[tid] + red[64 + tid]) + (red[128 + tid] + red[192 + tid]);
  for (int q = cb + tid; q < (ce < ntr ? ce : ntr); q += 256) pb[64 * ks + q] = tcol[q];
}

// z[owned rows] (=, or += with acc) from the partials of ns eliminated boxes, ks
// column slices: the owned unknown at position r = 64 c + i is chunk c's row sums
// i of its slices, in slice order, plus the column sums at r of every later
// chunk, added in chunk order.
template <typename T, bool SYS>
__global__ void k_ras_sum(const T* __restrict__ ps, const int* __restrict__ boxes, int ns, int ks,
                          const unsigned short* __restrict__ ord, T* __restrict__ z, BoxGeom g, bool acc) {
  const size_t tot = (size_t)ns * g.nown;
  for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < tot; t += (size_t)gridDim.x * blockDim.x) {
    const int b = (int)(t / g.nown), row = (int)(t % g.nown);
    int pid;
    size_t base;
    if (!box_entry<SYS>(g, boxes[b], pid, base)) continue;
    const size_t o = base + own_glob(g, pid, ord[t]);
    const int cr = row >> 6;
    const T* pp = ps + (size_t)b * sym_part_off(g.nch, ks);
    const T* pr = pp + sym_part_off(cr, ks) + (row & 63);
    // the row's ks slice sums, then the later chunks' column sums: read eight
    // at a time (past the end the first again), added one by one in that order
    const int m = ks + (g.nch - cr - 1);
    auto val = [&](int i) {
      const T* p = i < ks ? pr + 64 * i : pp + sym_part_off(cr + 1 + i - ks, ks) + 64 * ks + row;
      return *(i < m ? p : pr);
    };
    T a = pr[0];
    for (int i0 = 1; i0 < m; i0 += 8) {
      T v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = val(i0 + j);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (i0 + j < m) a += v[j];
    }
    z[o] = acc ? z[o] + a : a;
  }
}

// ---------------------------------------------------------------------------
// Interior boxes share one inverse (translation invariance of the periodic
// stencil away from the structure), and their matrix commutes with the box's
// two reflections: x -> -x takes x-face (ii, jj) to (m - ii, jj) with a sign
// change of u, and y-face or cell (ii, jj) to (m - 1 - ii, jj); y -> -y
// likewise with v.  So the product splits into the four parity classes
// (+-, +-) of the residual: with the orbits {k, Xk, Yk, XYk} of local
// unknowns,
//   class sums  q_ab[k] = r_k + a s_X r_Xk + b s_Y r_Yk + a b s_XY r_XYk,
//   products    Z_ab = M_ab q_ab over one representative per orbit,
//   results     z_k = sum_ab Z_ab,  z_Xk = s_X sum a Z_ab, ...
// M_ab[k, l] = 1/4 sum over l's distinct images g l of a^i b^j s_g M[k, g l].
// At 16 x 16/4 that is 4 x 208 x 456 multiply-adds a box instead of 768 x
// 1776, at 8 x 8/2 4 x 64 x 120 instead of 192 x 456, from a 3.0 MB (0.25 MB)
// matrix that stays in the caches, and few enough to need no reduction slices.
//
// Work-group = 16 boxes x one 16-row tile, wave = class x part of the chunk (KS
// parts).  The boxes' residuals are gathered 64 KS orbits at a time (a thread
// reads an orbit's four values of one box), split into classes and staged in
// LDS as the 16x16x4 MFMA's B operand; A streams from the class matrices, laid
// out [class][row tile][k][16 rows] so that a wave reads contiguous runs.  The
// next chunk's values load during the MFMAs.  The parts' and classes' results
// meet in LDS and each thread writes its row's owned images.
// Bound by the gathers' latency (one trip per chunk) on few boxes, by their
// address arithmetic beside the MFMAs on many: 852 boxes of 16 x 16/4 38.5 us
// FP64 (22.1 FP32) against 89.7 (58.4) for the dense product with its slices'
// sum launch; 188 boxes 16.5 against 31; 896 boxes of 8 x 8/2 6.7 against 22.
// ---------------------------------------------------------------------------
template <typename T, int KS>
struct RasIntSmem {
  T Xs[4][64 * KS][17];   // [class][orbit of the chunk][box]
  int bid[16];    // a box tile's boxes (-1: none) and their vectors' offsets
  int base[16];
  int kcode[kIntMaxOrbits];
};
template <typename T, int KS, bool SYS>
__device__ __forceinline__ void ras_int_block(RasIntSmem<T, KS>& sm, const T* __restrict__ r, T* __restrict__ z,
                                              const BoxGeom& g, const IntClassView& C, const int* __restrict__ boxes,
                                              int nlist, int bt, int rt, bool acc_mode) {
  constexpr int KC = 64 * KS, NT = 256 * KS, GPT = 4, AS = 16;
  using acc_t = typename Mfma<T>::acc_t;
  auto& Xs = sm.Xs;
  int *bid = sm.bid, *kcode = sm.kcode;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, kq = lane >> 4, bl = lane & 15;
  const int cls = wave & 3, kp = (wave >> 2) * 64;   // the wave's class and part of the chunk
  const int N = g.N, m = g.m, nn = N * N;
  bt *= 16;
  bool on = false;
  if (tid < 16) {
    int pid = -1;
    size_t base = 0;
    on = bt + tid < nlist && box_entry<SYS>(g, boxes[bt + tid], pid, base);
    bid[tid] = on ? pid : -1;
    if (SYS) sm.base[tid] = (int)base;   // (a batch's vectors have fewer than 2^31 entries)
  }
  for (int k = tid; k < C.Kp; k += NT) kcode[k] = k < C.K ? C.kcode[k] : -1;
  // a thread's orbit within a chunk and its four boxes are fixed, the boxes
  // the same for its whole wave
  int xb[GPT], yb[GPT], ob[GPT];
  if (SYS) {
    if (!__syncthreads_or(on)) return;
  } else {
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < GPT; ++u) {
    const int pid = __builtin_amdgcn_readfirstlane(bid[(tid + u * NT) / KC]);
    ob[u] = SYS ? __builtin_amdgcn_readfirstlane(sm.base[(tid + u * NT) / KC]) : 0;
    xb[u] = pid >= 0 ? (pid % g.npd) * g.b - g.o : -N;   // -N: no box
    yb[u] = pid >= 0 ? (pid / g.npd) * g.b - g.o : 0;
  }
  const T* Ma = static_cast<const T*>(C.M) + (((size_t)cls * C.nrt + rt) * C.Kp + kp + kq) * 16 + bl;
  acc_t acc{0, 0, 0, 0};
  T gx[GPT][4], ga[AS];
  auto wrap = [&](int a) { return a < 0 ? a + N : (a >= N ? a - N : a); };
  auto gather = [&](int k0) {
    const int code = kcode[k0 + tid % KC];
    const int comp = code >> 24, ii = code & 0xfff, jj = (code >> 12) & 0xfff;
    const int mi = (comp == 0 ? m : m - 1) - ii, mj = (comp == 1 ? m : m - 1) - jj;
    const int oe = jj * N + ii, ox = jj * N + mi, oy = mj * N + ii, oxy = mj * N + mi;
    const T* rc = r + (size_t)(comp < 0 ? 0 : comp) * nn;
#pragma unroll
    for (int u = 0; u < GPT; ++u) {
      const int x0 = xb[u], y0 = yb[u];
#pragma unroll
      for (int q = 0; q < 4; ++q) gx[u][q] = T(0);
      if (x0 >= 0 && y0 >= 0 && x0 + m < N && y0 + m < N) {   // clear of the periodic edges
        const int at = ob[u] + y0 * N + x0;
        if (code >= 0) {
          gx[u][0] = rc[at + oe];
          gx[u][1] = rc[at + ox];
          gx[u][2] = rc[at + oy];
          gx[u][3] = rc[at + oxy];
        }
      } else if (x0 > -N && code >= 0) {
        const int xe = wrap(x0 + ii), xm = wrap(x0 + mi), ye = ob[u] + wrap(y0 + jj) * N, ym = ob[u] + wrap(y0 + mj) * N;
        gx[u][0] = rc[ye + xe];
        gx[u][1] = rc[ye + xm];
        gx[u][2] = rc[ym + xe];
        gx[u][3] = rc[ym + xm];
      }
    }
  };
  // the signs of the images: u changes under X, v under Y
  auto stage = [&](int k0) {
    const int kk = tid % KC, comp = kcode[k0 + kk] >> 24;
    const T sx = comp == 0 ? T(-1) : T(1), sy = comp == 1 ? T(-1) : T(1);
#pragma unroll
    for (int u = 0; u < GPT; ++u) {
      const int b = (tid + u * NT) / KC;
      const T e = gx[u][0], x = sx * gx[u][1], y = sy * gx[u][2], xy = sx * sy * gx[u][3];
      const T ep = e + x, em = e - x, yp = y + xy, ym = y - xy;
      Xs[0][kk][b] = ep + yp;
      Xs[1][kk][b] = em + ym;
      Xs[2][kk][b] = ep - yp;
      Xs[3][kk][b] = em - ym;
    }
  };
  auto load_a = [&](int k0) {
#pragma unroll
    for (int s = 0; s < AS; ++s) ga[s] = Ma[(size_t)k0 * 16 + s * 64];
  };
  gather(0);
  load_a(0);
  for (int k0 = 0; k0 < C.Kp; k0 += KC) {
    stage(k0);
    __syncthreads();
    T a[AS];
#pragma unroll
    for (int s = 0; s < AS; ++s) a[s] = ga[s];
    if (k0 + KC < C.Kp) {
      gather(k0 + KC);
      load_a(k0 + KC);
    }
#pragma unroll
    for (int s = 0; s < AS; ++s) acc = Mfma<T>::mma(a[s], Xs[cls][kp + 4 * s + kq][bl], acc);
    __syncthreads();
  }
  // the parts' and classes' results: Xs[class][16 part + row][box]
#pragma unroll
  for (int v = 0; v < 4; ++v) Xs[cls][kp / 4 + Mfma<T>::row(kq, v)][bl] = acc[v];
  __syncthreads();
  if (tid < 256) {
    const int row = tid % 16, b = tid / 16;
    const int k = rt * 16 + row, pid = bid[b];
    if (k >= C.R || pid < 0) return;
    const int code = C.rcode[k], comp = (code >> 24) & 3, ii = code & 0xfff, jj = (code >> 12) & 0xfff, own = code >> 26;
    const int mi = (comp == 0 ? m : m - 1) - ii, mj = (comp == 1 ? m : m - 1) - jj;
    const int x0 = (pid % g.npd) * g.b - g.o, y0 = (pid / g.npd) * g.b - g.o;
    const T sx = comp == 0 ? T(-1) : T(1), sy = comp == 1 ? T(-1) : T(1);
    T zc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      zc[q] = Xs[q][row][b];
#pragma unroll
      for (int p = 1; p < KS; ++p) zc[q] += Xs[q][16 * p + row][b];
    }
    const T p = zc[0] + zc[2], q = zc[1] + zc[3], d = zc[0] - zc[2], e = zc[1] - zc[3];
    auto put = [&](int i, int j, T v) {   // an owned image: inside the grid, no wrap
      T* zp = z + (SYS ? sm.base[b] : 0) + (size_t)comp * nn + (size_t)(y0 + j) * N + x0 + i;
      *zp = acc_mode ? *zp + v : v;
    };
    if (own & 1) put(ii, jj, p + q);
    if (own & 2) put(mi, jj, sx * (p - q));
    if (own & 4) put(ii, mj, sy * (d + e));
    if (own & 8) put(mi, mj, sx * sy * (d - e));
  }
}

// One launch of the sweep: the first nib work-groups take the IB boxes (whole
// rows: box, chunk and row part; or the eliminated boxes' W pass: box and rpg rows
// of W), the others the interior ones (box tile and row tile).  The two kinds
// share nothing but r, and one launch lets the interior work-groups' gathers and
// MFMAs run under the IB boxes' streaming; splitting a chunk's rows instead of its
// columns needs no sum.  A coarse level's application is bound by its chain of
// latencies: 28 + 36 boxes of 8 x 8/2 9 us as one launch against 20 as three
// (rows, interior, sum); V-cycle at 64^2 274 -> 225 us.
template <typename T, int KS, int RS, bool SYS>
__global__ void __launch_bounds__(256 * KS) k_ras_rows(const T* __restrict__ r, T* __restrict__ z, BoxGeom g,
                                                       const T* __restrict__ inv, const T* const* __restrict__ inv_tab,
                                                       const int* __restrict__ ib_boxes, int nib, IntClassView C,
                                                       const int* __restrict__ int_boxes, int n_int, bool acc) {
  __shared__ RasIntSmem<T, KS> sm;
  const int p = blockIdx.x;
  if (p < nib) {
    const int item = p / RS, slot = item / g.nch, chunk = item % g.nch;
    T* x = &sm.Xs[0][0][0];
    int pid;
    size_t base;
    if (!box_entry<SYS>(g, ib_boxes[slot], pid, base)) return;
    const T* M = SYS ? inv_tab[slot] : inv + (size_t)slot * g.nch * g.nloc * 64;
    ras_rows_block<T, 4 * KS, RS>(r + base, z + base, g, M + (size_t)chunk * g.nloc * 64, pid, chunk, p % RS, x,
                                  x + g.nloc + kRowsPad, acc);
  } else {
    const int q = p - nib, nt = (n_int + 15) / 16;
    ras_int_block<T, KS, SYS>(sm, r, z, g, C, int_boxes, n_int, q % nt, q / nt, acc);
  }
}
// the rows' residual, its padding and the waves' sums fit in Xs
static_assert(4 * 64 * 17 >= kMaxNloc + kRowsPad + 4 * 64 && 4 * 128 * 17 >= kMaxNloc + kRowsPad + 8 * 64, "");

template <typename T, int KS, int CH, bool SYS>
__global__ void __launch_bounds__(256 * KS) k_ras_w(const T* __restrict__ r, T* __restrict__ z, BoxGeom g,
                                                    WBoxView w, const int* __restrict__ ib_boxes, int n_ib, int nib,
                                                    int rpg, T* __restrict__ t, IntClassView C,
                                                    const int* __restrict__ int_boxes, int n_int, bool acc) {
  __shared__ RasIntSmem<T, KS> sm;
  const int p = blockIdx.x;
  if (p < nib) {
    const int slot = p % n_ib, e1 = w.wptr[slot + 1], lo = w.wptr[slot] + p / n_ib * rpg;
    const int hi = lo + rpg < e1 ? lo + rpg : e1;
    int pid;
    size_t base;
    if (lo >= hi || !box_entry<SYS>(g, ib_boxes[slot], pid, base)) return;
    const T* Wm = SYS ? static_cast<const T*>(w.wtab[slot]) - (size_t)w.wptr[slot] * w.ws : static_cast<const T*>(w.W);
    ras_w_block<T, CH, 4 * KS>(r + base, g, pid, w, Wm, lo, hi, t + (size_t)slot * g.nown, &sm.Xs[0][0][0]);
  } else {
    const int q = p - nib, nt = (n_int + 15) / 16;
    ras_int_block<T, KS, SYS>(sm, r, z, g, C, int_boxes, n_int, q % nt, q / nt, acc);
  }
}
static_assert(4 * 64 * 17 >= kElimMaxNn, "");

// The class matrices of the eliminated interior box (launch_box_on done); kl:
// the four images' positions of every orbit, rl: the owned row of every row
// representative.
template <typename T>
__global__ void k_extract_classes(const double* __restrict__ mat, BoxMat bm, const unsigned short* __restrict__ own,
                                  IntClassView C, const int* __restrict__ kl, const int* __restrict__ rl,
                                  T* __restrict__ out) {
  const size_t tot = (size_t)4 * C.nrt * C.Kp * 16;
  for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < tot; t += (size_t)gridDim.x * blockDim.x) {
    const int rr = (int)(t % 16);
    const size_t t1 = t / 16;
    const int k = (int)(t1 % C.Kp);
    const int rt = (int)(t1 / C.Kp % C.nrt), cls = (int)(t1 / C.Kp / C.nrt), row = rt * 16 + rr;
    double v = 0.0;
    if (row < C.R && k < C.K) {
      const int lr = rl[row], comp = C.kcode[k] >> 24;
      const int e = kl[4 * k], x = kl[4 * k + 1], y = kl[4 * k + 2], xy = kl[4 * k + 3];
      auto at = [&](int j) { return box_inv_at(mat, bm, own, lr, j); };
      const double cx = (comp == 0 ? -1.0 : 1.0) * (cls & 1 ? -1.0 : 1.0), cy = (comp == 1 ? -1.0 : 1.0) * (cls & 2 ? -1.0 : 1.0);
      v = at(e);
      if (x != e) v += cx * at(x);
      if (y != e) v += cy * at(y);
      if (xy != e && xy != x && xy != y) v += cx * cy * at(xy);
      v *= 0.25;
    }
    out[t] = (T)v;
  }
}

template <typename T>
void launch_extract_classes(const double* mat, BoxMat bm, const unsigned short* own, IntClassView C, const int* kl,
                            const int* rl, T* out, hipStream_t s) {
  const size_t tot = (size_t)4 * C.nrt * C.Kp * 16;
  int grid = cdiv(tot, 256);
  if (grid > 4096) grid = 4096;
  IBMG_KLAUNCH((k_extract_classes<T>), dim3(grid), dim3(256), 0, s, mat, bm, own, C, kl, rl, out);
  IBMG_LAUNCH_CHECK();
}
template void launch_extract_classes<double>(const double*, BoxMat, const unsigned short*, IntClassView, const int*,
                                            const int*, double*, hipStream_t);
template void launch_extract_classes<float>(const double*, BoxMat, const unsigned short*, IntClassView, const int*,
                                            const int*, float*, hipStream_t);

template <typename T, int KS, bool SYS>
static void launch_ras(const T* r, T* z, const BoxGeom& g, const T* inv, const T* const* inv_tab, const int* ib_boxes, int n_ib,
                       const IntClassView& C, const int* int_boxes, int n_int, hipStream_t s, bool acc,
                       const SymIB* sym) {
  const int nint = (n_int + 15) / 16 * (n_int ? C.nrt : 0);
  const dim3 block(256 * KS);
  if (n_ib && sym) {
    const WBoxView& w = sym->w;
    T* t = static_cast<T*>(sym->t);
    // rows per work-group: enough work-groups to cover the device
    int rpg = 64;
    while (rpg > 16 && (long long)n_ib * ((w.maxrows + rpg - 1) / rpg) < 768 / KS) rpg /= 2;
    const int nib = n_ib * std::max(1, (w.maxrows + rpg - 1) / rpg);
    const int ch = (w.ws + 64 * Vec16<T>::n - 1) / (64 * Vec16<T>::n);
    if (ch > 8 || w.nn > kElimMaxNn) throw Error(IBMG_ERR_ARG, "eliminated boxes take at most 1024 non-owned unknowns");
    const dim3 grid(nib + nint);
    if (ch <= 2) IBMG_KLAUNCH((k_ras_w<T, KS, 2, SYS>), grid, block, 0, s, r, z, g, w, ib_boxes, n_ib, nib, rpg, t, C, int_boxes, n_int, acc);
    else if (ch <= 4) IBMG_KLAUNCH((k_ras_w<T, KS, 4, SYS>), grid, block, 0, s, r, z, g, w, ib_boxes, n_ib, nib, rpg, t, C, int_boxes, n_int, acc);
    else IBMG_KLAUNCH((k_ras_w<T, KS, 8, SYS>), grid, block, 0, s, r, z, g, w, ib_boxes, n_ib, nib, rpg, t, C, int_boxes, n_int, acc);
    IBMG_LAUNCH_CHECK();
    return;
  }
  // row parts of a chunk: more work-groups where there are few (one fits a CU;
  // each gathers the whole residual).  Solves with the line at 64, 128, 256 and
  // 512 work-groups: 256^2 8 x 8/2 3.68, 3.63, 3.79 and 3.91 ms; multiplicative
  // 256^2 16 x 16/4 19.7, 18.4, 19.5 and 19.5 ms
  const int items = n_ib * g.nch;
  int rs = 1;
  while (rs < 4 && items * rs < 128) rs *= 2;
  const dim3 grid(items * rs + nint);
  if (rs == 1) IBMG_KLAUNCH((k_ras_rows<T, KS, 1, SYS>), grid, block, 0, s, r, z, g, inv, inv_tab, ib_boxes, items, C, int_boxes, n_int, acc);
  else if (rs == 2) IBMG_KLAUNCH((k_ras_rows<T, KS, 2, SYS>), grid, block, 0, s, r, z, g, inv, inv_tab, ib_boxes, 2 * items, C, int_boxes, n_int, acc);
  else IBMG_KLAUNCH((k_ras_rows<T, KS, 4, SYS>), grid, block, 0, s, r, z, g, inv, inv_tab, ib_boxes, 4 * items, C, int_boxes, n_int, acc);
  IBMG_LAUNCH_CHECK();
}

template <typename T, bool SYS>
static void launch_ras_sweep(const T* r, T* z, BoxGeom g, const T* inv, const int* ib_boxes, int n_ib,
                      const IntClassView& C, const int* int_boxes, int n_int, hipStream_t s, int parts, bool acc,
                      const SymIB* sym, const T* const* inv_tab) {
  if (!(parts & 1)) n_ib = 0;
  if (!(parts & 2)) n_int = 0;
  if (n_ib + n_int == 0) return;
  if (g.nloc > kMaxNloc) throw Error(IBMG_ERR_ARG, "box too large");
  if (n_int) {
    if (!C.M || g.nown != 3 * g.b * g.b) throw Error(IBMG_ERR_ARG, "interior boxes without class matrices");
    if (C.Kp > kIntMaxOrbits || C.Kp % 128) throw Error(IBMG_ERR_ARG, "class matrices padded to whole chunks");
  }
  // interior parts: two shorten a work-group's chain of chunks (188 boxes of 16 x
  // 16/4, 156 work-groups: 16.5 us against 22.2 FP64, 11.2 against 16.7 FP32);
  // once the work-groups fill the device their size costs more (852 boxes, 702
  // work-groups: 46.6 against 38.5 FP64, 22.1 against 24.7 FP32; 3584 boxes of
  // 8 x 8/2, 896 work-groups: 20.6 against 16.9, 13.1 against 12.3)
  if ((n_int + 15) / 16 * (n_int ? C.nrt : 0) >= (sizeof(T) == 8 ? 512 : 768))
    launch_ras<T, 1, SYS>(r, z, g, inv, inv_tab, ib_boxes, n_ib, C, int_boxes, n_int, s, acc, sym);
  else
    launch_ras<T, 2, SYS>(r, z, g, inv, inv_tab, ib_boxes, n_ib, C, int_boxes, n_int, s, acc, sym);
  if (!n_ib || !sym) return;
  const int ks = sym_ksplit(g, n_ib);
  const size_t lds = (64 * (size_t)g.nch + 256 + 64 * (size_t)(g.nch - 1)) * sizeof(T);
  IBMG_KLAUNCH((k_ras_ib_sym<T, SYS>), dim3(n_ib, g.nch, ks), dim3(256), lds, s, r, static_cast<const T*>(sym->t), g,
               ib_boxes, sym->w, static_cast<const T*>(sym->inv), sym->qtab, static_cast<T*>(sym->part));
  IBMG_LAUNCH_CHECK();
  const int grid = std::min(4096, cdiv((size_t)n_ib * g.nown, 256));
  IBMG_KLAUNCH((k_ras_sum<T, SYS>), dim3(grid), dim3(256), 0, s, static_cast<const T*>(sym->part), ib_boxes, n_ib, ks,
               sym->w.ord, z, g, acc);
  IBMG_LAUNCH_CHECK();
}

template <typename T>
void launch_ras_apply(const T* r, T* z, BoxGeom g, const T* inv, const int* ib_boxes, int n_ib,
                      const IntClassView& C, const int* int_boxes, int n_int, hipStream_t s, int parts, bool acc,
                      const SymIB* sym, const T* const* inv_tab) {
  if (g.nbs) launch_ras_sweep<T, true>(r, z, g, inv, ib_boxes, n_ib, C, int_boxes, n_int, s, parts, acc, sym, inv_tab);
  else launch_ras_sweep<T, false>(r, z, g, inv, ib_boxes, n_ib, C, int_boxes, n_int, s, parts, acc, sym, inv_tab);
}

// ---------------------------------------------------------------------------
// Summed additive Schwarz (the plain R_k^T combination).  First every box's
// whole local solution y_k = L_k^{-1} R_k r: a work-group per (box, 64-row
// chunk) streams that chunk of the box's full inverse as the IB-box kernel
// does (interior boxes share one inverse) and writes the 64 rows to
// Y[(box * nch + chunk) * 64 + row].  Then every unknown gathers its entries
// from the boxes whose index set holds it: no two work-groups write one
// unknown, and no atomics are needed.
// ---------------------------------------------------------------------------
// One (box, 64-row chunk) item: Mc is the chunk of the box's inverse; x holds nloc
// values (LDS), part 256; the 64 row sums go to out.  The first loads of the
// inverse are issued before the gather.
template <typename T>
__device__ __forceinline__ void asm_chunk(const T* __restrict__ r, const BoxGeom& g, const T* __restrict__ Mc, int pid,
                                          T* x, T* part, T* __restrict__ out) {
  using V = typename Vec16<T>::type;
  constexpr int VEC = Vec16<T>::n;
  constexpr int LPC = 64 / VEC;  // lanes per column
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int cph = lane / LPC;           // column phase 0..VEC-1
  const int rl = (lane % LPC) * VEC;    // first of this lane's VEC rows
  const int per = ((g.nloc + 4 * VEC - 1) / (4 * VEC)) * VEC;
  const int j0 = q * per, j1 = j0 + per < g.nloc ? j0 + per : g.nloc;
  Mc += rl;
  int j = j0 + cph;
  // eight 16-byte loads in flight per lane, summed in a fixed tree; the
  // inverse streams through once per sweep, so its loads are non-temporal
  // and leave the caches to the level's vectors
  constexpr int UNR = 8;
  auto load8 = [&](V* m, int jj) {
#pragma unroll
    for (int u = 0; u < UNR; ++u)
      m[u] = __builtin_nontemporal_load(reinterpret_cast<const V*>(Mc + (size_t)(jj + u * VEC) * 64));
  };
  T acc[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) acc[v] = 0;
  auto fma8 = [&](const V* m, int jj) {
    T xv[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) xv[u] = x[jj + u * VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      T t[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) t[u] = reinterpret_cast<const T*>(&m[u])[v] * xv[u];
      acc[v] += ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
    }
  };
  const bool first = j + (UNR - 1) * VEC < j1;
  V m0[UNR];
  if (first) load8(m0, j);
  for (int k = threadIdx.x; k < g.nloc; k += blockDim.x) x[k] = r[box_glob(g, pid, k)];
  __syncthreads();
  if (first) {
    fma8(m0, j);
    j += UNR * VEC;
  }
  for (; j + (UNR - 1) * VEC < j1; j += UNR * VEC) {
    V m[UNR];
    load8(m, j);
    fma8(m, j);
  }
  for (; j < j1; j += VEC) {
    const V m0 = __builtin_nontemporal_load(reinterpret_cast<const V*>(Mc + (size_t)j * 64));
    const T* a0 = reinterpret_cast<const T*>(&m0);
    const T x0 = x[j];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] += a0[v] * x0;
  }
  // sum the VEC column phases (lanes l, l + LPC, ...)
#pragma unroll
  for (int off = 32; off >= LPC; off >>= 1)
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] += __shfl_down(acc[v], off, 64);
  if (lane < LPC)
#pragma unroll
    for (int v = 0; v < VEC; ++v) part[q * 64 + rl + v] = acc[v];
  __syncthreads();
  if (q == 0) out[lane] = (part[lane] + part[64 + lane]) + (part[128 + lane] + part[192 + lane]);
}

template <typename T>
__global__ void __launch_bounds__(256) k_asm_local(const T* __restrict__ r, BoxGeom g, const T* __restrict__ inv,
                                                   const int* __restrict__ box_inv, T* __restrict__ Y) {
  extern __shared__ char smem_raw[];
  T* x = reinterpret_cast<T*>(smem_raw);
  T* part = x + ((g.nloc + 3) & ~3);
  const int pid = blockIdx.x, chunk = blockIdx.y;
  const T* Mc = inv + ((size_t)box_inv[pid] * g.nch + chunk) * g.nloc * 64;
  asm_chunk<T>(r, g, Mc, pid, x, part, Y + ((size_t)pid * g.nch + chunk) * 64);
}

// z[d] = sum of unknown d's entries over the boxes that hold it.  Along each
// axis the boxes holding a coordinate lie within reach (b + o) / b + 1 of its
// owner box (on levels with fewer boxes than that window, every box is
// tried); they are visited rows of boxes first, in increasing offset from
// the owner, a fixed order per unknown.
template <typename T>
__global__ void k_asm_gather(const T* __restrict__ Y, T* __restrict__ z, BoxGeom g) {
  const int N = g.N, m = g.m, nu = m * (m + 1), npd = g.npd;
  const size_t nn = (size_t)N * N, tot = 3 * nn;
  const int reach = (g.b + g.o) / g.b + 1;
  const bool every = 2 * reach + 1 >= npd;
  const int cnt = every ? npd : 2 * reach + 1;
  for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < tot; t += (size_t)gridDim.x * blockDim.x) {
    const int comp = (int)(t / nn);
    const size_t q = t - (size_t)comp * nn;
    const int i = (int)(q % N), j = (int)(q / N);
    const int ext_x = comp == 0 ? m + 1 : m, ext_y = comp == 1 ? m + 1 : m;
    const int ox = i / g.b, oy = j / g.b;
    T acc = 0;
    for (int ty = 0; ty < cnt; ++ty) {
      const int by = every ? ty : pmod(oy - reach + ty, npd);
      const int jj = pmod(j - (by * g.b - g.o), N);
      if (jj >= ext_y) continue;
      for (int tx = 0; tx < cnt; ++tx) {
        const int bx = every ? tx : pmod(ox - reach + tx, npd);
        const int ii = pmod(i - (bx * g.b - g.o), N);
        if (ii >= ext_x) continue;
        const int k = comp == 0 ? jj * (m + 1) + ii : (comp == 1 ? nu + jj * m + ii : 2 * nu + jj * m + ii);
        acc += Y[((size_t)(by * npd + bx) * g.nch + (k >> 6)) * 64 + (k & 63)];
      }
    }
    z[t] = acc;
  }
}

template <typename T>
void launch_asm_apply(const T* r, T* z, BoxGeom g, const T* inv, const int* box_inv, T* Y, hipStream_t s) {
  const int nbox = g.npd * g.npd;
  const size_t lds = (((size_t)g.nloc + 3) & ~(size_t)3) * sizeof(T) + 256 * sizeof(T);
  IBMG_KLAUNCH((k_asm_local<T>), dim3(nbox, g.nch), dim3(256), lds, s, r, g, inv, box_inv, Y);
  IBMG_LAUNCH_CHECK();
  const size_t tot = 3 * (size_t)g.N * g.N;
  int grid = cdiv(tot, 256);
  if (grid > 8192) grid = 8192;
  IBMG_KLAUNCH((k_asm_gather<T>), dim3(grid), dim3(256), 0, s, Y, z, g);
  IBMG_LAUNCH_CHECK();
}

// ---------------------------------------------------------------------------
// Coarsest level.  Its pseudo-inverse L0^+ (the solution of the system bordered
// by the null vectors: the constant pressure, plus constant u and v when
// rho = 0) comes from the block sweeps of the box matrices: with q the unit
// constant vector of a block, L0 + s q q^T (velocity, rho = 0) - t q q^T
// (pressure) is regular and ordered for sweeps without pivoting (velocities
// positive definite, then a negative definite Schur complement), and its
// inverse is L0^+ + q q^T / s - q q^T / t, so the extraction takes those
// constants off again.  s and t are the sizes of the blocks' diagonals (of the
// Schur complement for the pressure).  Two steps of 128 columns at 8 x 8: 0.5
// ms, where one work-group's pivoted elimination took 4.3 to 5.6; at 15 x 15
// (675 unknowns, 240^2 finest) a whole rebuild went from 248 to 11 ms.
// Tangent springs shorter than their rest length can make the velocity block
// indefinite: such handles eliminate with pivoting, on the bordered matrix
// [[L0, C], [C^T, 0]] augmented by the identity (aug is nn x 2 nn row-major,
// nn = 3 N^2 + nb).
// ---------------------------------------------------------------------------
// ld: row stride; nb: border columns (0: none, and no identity); su, sp: added
// to every entry of the velocity and pressure blocks' constant part
__global__ void k_coarse_assemble(int N, StokesCoef<double> c, CsrView tu, CsrView tv, int nb, int ld, double su,
                                  double sp, double* __restrict__ aug) {
  const int n = 3 * N * N, nn = n + nb;
  const int row = blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= nn) return;
  double* Ar = aug + (size_t)row * ld;
  if (nb) Ar[nn + row] = 1.0;
  const int NN = N * N;
  // block -> border column: rho = 0: u->0, v->1, p->2; else p->0
  auto border = [&](int blk) -> int {
    if (nb == 3) return n + blk;
    return nb == 1 && blk == 2 ? n : -1;
  };
  if (row >= n) {
    const int cidx = row - n;
    const int blk = nb == 3 ? cidx : 2;
    for (int k = 0; k < NN; ++k) Ar[blk * NN + k] = 1.0;
    return;
  }
  const int blk = row / NN, q = row % NN;
  const int i = q % N, j = q / N;
  const int im = pmod(i - 1, N), ip = pmod(i + 1, N), jm = pmod(j - 1, N), jp = pmod(j + 1, N);
  const double dg = c.alpha + 4.0 * c.beta;
  const double shift = blk == 2 ? sp : su;
  if (shift != 0.0)
    for (int k = 0; k < NN; ++k) Ar[blk * NN + k] += shift;
  if (blk == 0) {
    Ar[q] += dg;
    Ar[j * N + im] -= c.beta;
    Ar[j * N + ip] -= c.beta;
    Ar[jm * N + i] -= c.beta;
    Ar[jp * N + i] -= c.beta;
    Ar[2 * NN + j * N + i] += c.gi;
    Ar[2 * NN + j * N + im] -= c.gi;
    for (int k = tu.ptr[q]; k < tu.ptr[q + 1]; ++k) Ar[tu.col[k]] += tu.val[k];
  } else if (blk == 1) {
    Ar[NN + q] += dg;
    Ar[NN + j * N + im] -= c.beta;
    Ar[NN + j * N + ip] -= c.beta;
    Ar[NN + jm * N + i] -= c.beta;
    Ar[NN + jp * N + i] -= c.beta;
    Ar[2 * NN + j * N + i] += c.gi;
    Ar[2 * NN + jm * N + i] -= c.gi;
    for (int k = tv.ptr[q]; k < tv.ptr[q + 1]; ++k) Ar[tv.col[k]] += tv.val[k];
  } else {
    Ar[j * N + ip] -= c.gi;
    Ar[j * N + i] += c.gi;
    Ar[NN + jp * N + i] -= c.gi;
    Ar[NN + j * N + i] += c.gi;
  }
  const int bc = border(blk);
  if (bc >= 0) Ar[bc] += 1.0;
}

void launch_coarse_assemble(int N, StokesCoef<double> c, const int* tptr_u, const int* tcol_u,
                            const double* tval_u, const int* tptr_v, const int* tcol_v,
                            const double* tval_v, int nb, double* aug, hipStream_t s) {
  CsrView tu{tptr_u, tcol_u, tval_u}, tv{tptr_v, tcol_v, tval_v};
  const int nn = 3 * N * N + nb;
  IBMG_KLAUNCH(k_coarse_assemble, dim3(cdiv(nn, 64)), dim3(64), 0, s, N, c, tu, tv, nb, 2 * nn, 0.0, 0.0, aug);
  IBMG_LAUNCH_CHECK();
}

// the constants' sizes: the velocity diagonal (0 when rho > 0: the block is
// regular) and the Schur complement's
CoarseShift coarse_shift(StokesCoef<double> c, bool rho_zero) {
  const double dg = c.alpha + 4.0 * c.beta;
  return CoarseShift{rho_zero ? dg : 0.0, c.gi * c.gi / dg};
}

void launch_coarse_assemble_sym(int N, StokesCoef<double> c, const int* tptr_u, const int* tcol_u,
                                const double* tval_u, const int* tptr_v, const int* tcol_v, const double* tval_v,
                                CoarseShift sh, double* mat, hipStream_t s) {
  CsrView tu{tptr_u, tcol_u, tval_u}, tv{tptr_v, tcol_v, tval_v};
  const int n = 3 * N * N;
  const double inn = 1.0 / ((double)N * N);   // q q^T has entries 1 / N^2
  IBMG_KLAUNCH(k_coarse_assemble, dim3(cdiv(n, 64)), dim3(64), 0, s, N, c, tu, tv, 0, n, sh.vel * inn, -sh.p * inn,
               mat);
  IBMG_LAUNCH_CHECK();
}

// L0^+ from the swept matrix (-X, 64 x 64 tiles on or below the diagonal) and the
// shifted matrix A, with one refinement step: R = I - A X (FINAL false), then X + X R
// less the constants (FINAL true).  The unpivoted sweeps lose up to a digit and a
// half against a pivoted elimination on stiff structures (64^2, kappa = 1e8, mu =
// 1e-3: 3.4e-10 against 1.9e-11); the step takes the error below both.  One 64 x 64
// tile per work-group, four waves of 2 x 2 MFMA tiles, the reduction through LDS 32
// indices at a time.  Bound by latency, a step of 32 indices about 3 us: 20 and 22 us
// at 8^2 (9 work-groups), 72 and 80 at 15^2 or 16^2 (121 or 144), on the stream that
// runs beside the boxes' elimination.
template <bool FINAL>
__global__ void __launch_bounds__(256) k_coarse_refine(const double* __restrict__ S, const double* __restrict__ AR,
                                                       int N, CoarseShift sh, double* __restrict__ out) {
  __shared__ GjTileSmem sm;
  const int NN = N * N, n = 3 * NN, I0 = blockIdx.x * 64, J0 = blockIdx.y * 64;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wr = wave & 1, wc = wave >> 1, kq = lane >> 4, ln = lane & 15;
  // the symmetric X, from clamped indices
  auto x_at = [&](int i, int j) { return -((i >> 6) >= (j >> 6) ? S[(size_t)i * n + j] : S[(size_t)j * n + i]); };
  Mfma<double>::acc_t acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = Mfma<double>::acc_t{0, 0, 0, 0};
  for (int k0 = 0; k0 < n; k0 += 32) {
    double xr[8], yr[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int t = tid + 256 * q;
      const int i = I0 + (t >> 5), k = k0 + (t & 31), kb = k0 + (t >> 6), j = J0 + (t & 63);
      const int ic = i < n ? i : n - 1, kc = k < n ? k : n - 1, kbc = kb < n ? kb : n - 1, jc = j < n ? j : n - 1;
      xr[q] = FINAL ? x_at(ic, kc) : AR[(size_t)ic * n + kc];
      xr[q] = k < n ? xr[q] : 0.0;
      yr[q] = FINAL ? AR[(size_t)kbc * n + jc] : x_at(kbc, jc);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int t = tid + 256 * q;
      sm.Xs[t & 31][t >> 5] = xr[q];
      sm.Ys[t >> 6][t & 63] = yr[q];
    }
    __syncthreads();
#pragma unroll
    for (int st = 0; st < 8; ++st) {
      const int kk = 4 * st + kq;
      const double a0 = sm.Xs[kk][32 * wr + ln], a1 = sm.Xs[kk][32 * wr + 16 + ln];
      const double b0 = sm.Ys[kk][32 * wc + ln], b1 = sm.Ys[kk][32 * wc + 16 + ln];
      acc[0][0] = Mfma<double>::mma(a0, b0, acc[0][0]);
      acc[0][1] = Mfma<double>::mma(a0, b1, acc[0][1]);
      acc[1][0] = Mfma<double>::mma(a1, b0, acc[1][0]);
      acc[1][1] = Mfma<double>::mma(a1, b1, acc[1][1]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = I0 + 32 * wr + 16 * a + Mfma<double>::row(kq, v), j = J0 + 32 * wc + 16 * b + ln;
        if (i >= n || j >= n) continue;
        double x = (i == j ? 1.0 : 0.0) - acc[a][b][v];
        if (FINAL) {
          x = x_at(i, j) + acc[a][b][v];
          const int bi = i / NN;
          if (bi == j / NN) {
            if (bi == 2) x += 1.0 / (sh.p * (double)NN);
            else if (sh.vel > 0.0) x -= 1.0 / (sh.vel * (double)NN);
          }
        }
        out[(size_t)i * n + j] = x;
      }
}

void launch_coarse_refine(const double* swept, const double* A, double* R, int N, CoarseShift sh, double* inv,
                          hipStream_t s) {
  const int T = (3 * N * N + 63) / 64;
  IBMG_KLAUNCH((k_coarse_refine<false>), dim3(T, T), dim3(256), 0, s, swept, A, N, sh, R);
  IBMG_LAUNCH_CHECK();
  IBMG_KLAUNCH((k_coarse_refine<true>), dim3(T, T), dim3(256), 0, s, swept, R, N, sh, inv);
  IBMG_LAUNCH_CHECK();
}

// Gauss-Jordan with partial pivoting on [A | I] in one work-group of 1024
// threads.  Per pivot: the column's largest magnitude (ties to the lower
// row) by a butterfly within each wave and one pass over the 16 wave
// results; the row swap; the scaled pivot row and the column's factors
// staged in LDS; then the elimination over the whole matrix as one flat
// loop, so each thread keeps several independent loads in flight.
__global__ void __launch_bounds__(1024) k_coarse_invert(double* __restrict__ aug, int nn) {
  __shared__ double wmax[16];
  __shared__ int wimax[16];
  __shared__ double fac[1024];
  __shared__ double rowk[2048];   // the scaled pivot row (2 nn <= 2048)
  const int ld = 2 * nn;
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6;
  for (int k = 0; k < nn; ++k) {
    double best = -1.0;
    int bi = k;
    for (int i = k + tid; i < nn; i += nt) {
      const double a = fabs(aug[(size_t)i * ld + k]);
      if (a > best) { best = a; bi = i; }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const double o = __shfl_xor(best, off, 64);
      const int oi = __shfl_xor(bi, off, 64);
      if (o > best || (o == best && oi < bi)) { best = o; bi = oi; }
    }
    if (lane == 0) {
      wmax[wave] = best;
      wimax[wave] = bi;
    }
    __syncthreads();
    double bv = wmax[0];
    int p = wimax[0];
    for (int q = 1; q < (nt >> 6); ++q) {
      const double o = wmax[q];
      const int oi = wimax[q];
      if (o > bv || (o == bv && oi < p)) { bv = o; p = oi; }
    }
    if (p != k) {
      for (int j = tid; j < ld; j += nt) {
        const double t = aug[(size_t)k * ld + j];
        aug[(size_t)k * ld + j] = aug[(size_t)p * ld + j];
        aug[(size_t)p * ld + j] = t;
      }
    }
    __syncthreads();
    const double ip = 1.0 / aug[(size_t)k * ld + k];
    __syncthreads();
    for (int j = tid; j < ld; j += nt) {
      const double v = aug[(size_t)k * ld + j] * ip;
      aug[(size_t)k * ld + j] = v;
      rowk[j] = v;
    }
    for (int i = tid; i < nn; i += nt) fac[i] = aug[(size_t)i * ld + k];
    __syncthreads();
    const int tot = nn * ld;
#pragma unroll 8
    for (int t = tid; t < tot; t += nt) {
      const int i = t / ld, j = t - i * ld;
      if (i != k) aug[(size_t)i * ld + j] -= fac[i] * rowk[j];
    }
    __syncthreads();
  }
}

void launch_coarse_invert(double* aug, int nn, hipStream_t s) {
  if (nn > 1024) throw Error(IBMG_ERR_ARG, "coarsest system too large for one work-group");
  IBMG_KLAUNCH(k_coarse_invert, dim3(1), dim3(1024), 0, s, aug, nn);
  IBMG_LAUNCH_CHECK();
}

__global__ void k_coarse_extract(const double* __restrict__ aug, int nn, int n0, double* __restrict__ inv) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n0 * n0) return;
  const int i = t / n0, j = t % n0;
  inv[t] = aug[(size_t)i * 2 * nn + nn + j];
}

void launch_coarse_extract(const double* aug, int nn, int n0, double* inv, hipStream_t s) {
  IBMG_KLAUNCH(k_coarse_extract, dim3(cdiv((size_t)n0 * n0, 256)), dim3(256), 0, s, aug, nn, n0, inv);
  IBMG_LAUNCH_CHECK();
}

// z = inv r on the coarsest level, FP64 arithmetic whatever T is: one wave
// per row, the lanes reading the row (and r) contiguously, then a butterfly
// over the wave.
template <typename T>
__global__ void __launch_bounds__(256) k_coarse_apply(const double* __restrict__ inv, int n0,
                                                      const T* __restrict__ r, T* __restrict__ z) {
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= n0) return;
  // batched: system blockIdx.y, inverses n0^2 and vectors n0 apart
  inv += (size_t)blockIdx.y * n0 * n0;
  r += (size_t)blockIdx.y * n0;
  z += (size_t)blockIdx.y * n0;
  const double* row = inv + (size_t)i * n0;
  double a = 0.0;
  for (int j = lane; j < n0; j += 64) a += row[j] * (double)r[j];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) a += __shfl_xor(a, off, 64);
  if (lane == 0) z[i] = (T)a;
}

template <typename T>
void launch_coarse_apply_batch(const double* inv, int n0, const T* r, T* z, int nsys, hipStream_t s) {
  if (nsys <= 0) return;
  IBMG_KLAUNCH((k_coarse_apply<T>), dim3(cdiv(n0, 4), nsys), dim3(256), 0, s, inv, n0, r, z);
  IBMG_LAUNCH_CHECK();
}

template <typename T>
void launch_coarse_apply(const double* inv, int n0, const T* r, T* z, hipStream_t s) {
  launch_coarse_apply_batch<T>(inv, n0, r, z, 1, s);
}

template void launch_extract_rows<double>(const double*, int, BoxGeom, BoxMat, BoxOrder, double*, hipStream_t);
template void launch_extract_rows<float>(const double*, int, BoxGeom, BoxMat, BoxOrder, float*, hipStream_t);
template void launch_extract_w<double>(const double*, int, BoxMat, const int*, const int*, int, double*, hipStream_t);
template void launch_extract_w<float>(const double*, int, BoxMat, const int*, const int*, int, float*, hipStream_t);
template void launch_asm_apply<double>(const double*, double*, BoxGeom, const double*, const int*, double*,
                                       hipStream_t);
template void launch_asm_apply<float>(const float*, float*, BoxGeom, const float*, const int*, float*, hipStream_t);
template void launch_ras_apply<double>(const double*, double*, BoxGeom, const double*, const int*, int,
                                       const IntClassView&, const int*, int, hipStream_t, int, bool, const SymIB*,
                                       const double* const*);
template void launch_ras_apply<float>(const float*, float*, BoxGeom, const float*, const int*, int,
                                      const IntClassView&, const int*, int, hipStream_t, int, bool, const SymIB*,
                                       const float* const*);
template void launch_extract_sym<double>(const double*, int, BoxGeom, BoxMat, double*, hipStream_t);
template void launch_extract_sym<float>(const double*, int, BoxGeom, BoxMat, float*, hipStream_t);
template void launch_coarse_apply<double>(const double*, int, const double*, double*, hipStream_t);
template void launch_coarse_apply<float>(const double*, int, const float*, float*, hipStream_t);
template void launch_coarse_apply_batch<double>(const double*, int, const double*, double*, int, hipStream_t);
template void launch_coarse_apply_batch<float>(const double*, int, const float*, float*, int, hipStream_t);

}  // namespace ibmg
