// Host orchestration: hierarchy set-up, the V-cycle of Alg. 1 with
// FGMRES-wrapped smoothing (Sec. 3.3), and the outer flexible GMRES solve.
// Every arithmetic step runs in the kernels; the host builds index structures
// (footprint windows, face -> point lists, IB row patterns, box classes) and
// sequences launches on one stream.
#pragma once

#include <atomic>
#include <exception>
#include <mutex>
#include <map>
#include <numeric>
#include <thread>
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cmath>
#include <type_traits>

#include "sc_smoother.hpp"
#include "solver.hpp"

namespace ibmg {

namespace detail {

constexpr int kMaxNu = 8;
constexpr int kMaxRestart = 64;
// The IB term of L_IB w comes from a level's explicit Galerkin rows (in the
// operator's own launch) up to this many entries for the level's longest face list
// and its number of points.  The rows cost about 4 to 5.9 us per million entries
// (12 bytes each, FP64; 8 in FP32); the other form (interpolate, spring forces,
// gather: three launches) at least 12 to 15 us, and more with the points and with
// the longest list, which one thread walks.  Rows and the other form, FP64 us (FP32):
// 512^2, 2000 scattered points, 3.32 M entries, list 4: 21.7 and 16.2 (17.0, 11.8);
// annuli, 4 x 2048, 2.35 M, 17: 15.3 and 19.5 (10.7, 15.9), with tangent springs
// 4.59 M, 17: 31.5 and 19.9 (26.1, 15.6), 8 x 4096, 4.03 M, 51: 19.5 and 47.3
// (15.1, 34.3); thick shell of 59584 points, 4.57 M, 40: 23.6 and 75.6 (18.7, 52.7);
// 1024^2, suspension of 32768 points, 6.50 M, 10: 55.0 and 42.6 (43.1, 30.9); thick
// shell of 235904 points, 17.65 M, 41: 106 and 368 (56, 339).  Over 244 such levels
// the line costs 0.7 % against the better form each time (3.5 M entries whatever the
// lists: 7.2 %, eleven times at the worst).  IBMG_NO_IB_ROWS in the environment
// takes the other form on every level.
inline size_t ib_rows_max_entries(int longest, int points) {
  return 1500000 + 100000 * (size_t)longest + 100 * (size_t)points;
}
// Blocks of the outer solve's long reductions up to which the next kernel's
// blocks reduce the partial sums themselves: the folding launches cost more than
// the reads until every block reads them all from many.  30 iterations of one
// restart cycle with and without folding, in us: 256^2 (192 blocks) 16301 and 15889,
// 320^2 (300) 22191 and 21796, 416^2 (507) 28024 and 27679, 480^2 (675) 36768 and
// 36482, 512^2 (768) 26055 and 26121, 640^2 (1024) 39678 and 40490.
constexpr int kFoldBlocks = 704;
// The IB boxes are kept eliminated (two passes over W and the symmetric owned
// factor) where their whole rows would take at least this much; see
// prepare_boxes.
constexpr size_t kElimMinBytes = (size_t)192 << 20;
// An FP32 smoother takes the eliminated form only where it is no less accurate
// than whole rows: its two roundings, amplified as launch_elim_loss measures (the
// sums' ratio), against the whole rows' longer sums.  Error of one sweep against
// FP64, eliminated over whole rows, by that ratio (16 x 16/4 and 8 x 8/2 boxes,
// annuli and the thin and thick structures over stiffnesses): velocities 0.55 to
// 0.65 at 1.4 to 1.6, 0.95 at 3.3, 0.98 at 5.0, 1.14 at 8.3, 1.24 at 10, 1.41 at
// 7.3, 6.2 to 33 on the stiffest; pressures 0.6 to 0.8 at 1.1 to 1.3, 0.65 at 1.6,
// 1.7 at 4.2 and 4.4.
constexpr double kElimMaxLossVel = 5.0, kElimMaxLossPre = 1.6;
// Pre-smoothing steps up to which the V-cycle takes the residual it restricts
// from the Arnoldi relation, without an operator application.  That residual
// leaves out what rounding did to L z_q and to w, which grows with the basis:
// 128^2 membrane, kappa = 1e6, FP32 smoother, error of a V-cycle against FP64
// (geometric mean over 40 right-hand sides), Arnoldi relation and b - L w: 1.5e-7
// and 1.5e-7 at two iterations, 2.4e-7 and 2.0e-7 at three, 5.2e-7 and 3.3e-7 at
// four, 3.5e-6 and 5.0e-7 at six, 1.3e-4 and 5.1e-6 at seven.
constexpr int kArnoldiResidualNu = 2;
// lanes per explicit row: a wave where rows are long (crowded coarse levels)
constexpr int kIbLongRow = 96;
// partial-sum buffers: two of kPartStride doubles (blocks x vectors)
constexpr size_t kPartStride = (size_t)256 * 65;
// the outer solve's Gram-Schmidt passes: up to kOuterBlocks blocks of up to
// 65 vectors, folded by one block before their consumers
constexpr int kOuterBlocks = 1024;
constexpr size_t kOuterPartStride = (size_t)kOuterBlocks * 65;

inline int wrapn(int a, int N) {
  a %= N;
  return a < 0 ? a + N : a;
}

inline std::vector<int> level_sizes(int N, int coarse) {
  std::vector<int> s;
  for (int n = N; n >= coarse; n /= 2) {
    s.push_back(n);
    if (n == coarse) break;
  }
  std::reverse(s.begin(), s.end());
  return s;
}

inline void box_params(int N, int box, int overlap, int* b, int* o) {
  *b = std::min(box, N / 2);
  *o = std::min(overlap, (N - *b - 1) / 2);
  if (*o < 0) *o = 0;
}

}  // namespace detail

using namespace detail;

template <typename T>
struct Level {
  int N = 0;
  CompFoot f[2];
  // rows of the IB term (comp N^2 + face) and the faces' flags; ib_lanes = 0:
  // the IB term of L_IB w by interpolation, spring forces and the gather
  std::vector<int> ib_rows;
  size_t n_ib_v = 0;            // of them component 1's (the last ones)
  int ib_lanes = 0;
  DBuf<int> d_ib_rows;
  DBuf<unsigned char> d_ib_flag;
  StokesCoef<double> cd{};
  StokesCoef<T> ct{};
  // restricted additive Schwarz
  BoxGeom g{};
  int n_unique = 0, n_ib = 0;
  std::vector<int> uniq;  // unique box ids (IB boxes, then one interior representative)
  std::vector<int> ib_list, int_list;
  DBuf<int> d_ib, d_int;
  DBuf<T> inv;            // [n_unique][nch][nloc][64], or W and Q
  // the interior boxes' shared inverse in its four parity classes (ras_int_block)
  std::vector<int> kcode, rcode, klocal, rlocal;
  DBuf<int> d_kcode, d_rcode, d_klocal, d_rlocal;
  DBuf<T> cls;
  IntClassView clsv{};
  // layout of the box matrices and the local unknowns' positions in it; the
  // non-owned unknowns in that order
  BoxMat bm{};
  std::vector<int> pos, nonown;
  DBuf<int> d_pos, d_nonown;
  // per unique box: the owned unknowns by position and back
  std::vector<unsigned short> ord, own;
  DBuf<unsigned short> d_ord, d_own;
  // eliminated storage of the IB boxes: the W rows, the symmetric factor, the
  // first pass's result and the per-box partials
  bool use_sym = false, may_sym = false;
  double loss[4] = {0, 0, 0, 0};   // launch_elim_loss's sums (FP32 smoothers)
  std::vector<int> wptr, wrow;
  std::vector<unsigned char> coupled;
  DBuf<int> d_wptr, d_wrow;
  DBuf<unsigned char> d_coupled;
  int w_max = 0, w_stride = 0;
  T *wmat = nullptr, *inv_sym = nullptr;   // W and Q, within inv
  DBuf<T> w_res, sym_part;
  // restricted multiplicative Schwarz: box colours; ib_list and int_list
  // sorted by colour, colour c spanning [ib_off[c], ib_off[c+1]) and
  // [int_off[c], int_off[c+1])
  int ncolour = 0;
  std::vector<int> box_colour, ib_off, int_off;
  DBuf<T> rr;             // residual between colours
  // summed combination (IBMG_COMBINE_SUM): g.nown = nloc, every row of every
  // box inverse is kept; box_inv maps a box id to its inverse (IB boxes their
  // own, interior boxes the shared one), Y holds every box's local solution
  bool sum_mode = false;
  DBuf<int> d_box_inv;
  DBuf<T> Y;
  // work vectors
  DBuf<T> w, b, r, t, V, Z, F;
  DBuf<double> scal, part;   // the smoothing step's state, its partial sums
  // Schur-complement smoother
  std::unique_ptr<ScLevel<T>> sc;
};

template <typename T>
class BatchSolver;

template <typename T>
class Solver final : public SolverBase {
  friend class BatchSolver<T>;

 public:
  // defer_coarse: assemble the coarsest system but leave its inversion to
  // the caller (the batched form inverts every system's in one launch and
  // hands each back through finish_coarse)
  // members: per level, the systems of the batch that have it (a batch member)
  Solver(const ibmg_desc& d, hipStream_t s, bool defer_coarse = false, std::vector<int> members = {})
      : d_(d), defer_coarse_(defer_coarse), members_(std::move(members)) {
    M_ = d.M;
    E_ = d.n_springs;
    X_.assign(d.X, d.X + 2 * (size_t)M_);
    ends_.assign(d.ends, d.ends + 2 * (size_t)E_);
    kappa_.assign(d.kappa, d.kappa + E_);
    tangent_ = d.spring_model == IBMG_SPRING_TANGENT;
    rest_.assign(E_, 0.0);
    if (d.rest) rest_.assign(d.rest, d.rest + E_);
    // the descriptor's host arrays belong to the caller
    d_.X = nullptr;
    d_.ends = nullptr;
    d_.kappa = nullptr;
    d_.rest = nullptr;
    nu_ = std::max(d.nu1, d.nu2);
    sizes_ = level_sizes(d.N, d.coarse_N);
    L_ = (int)sizes_.size() - 1;
    outer_cap_ = d.max_restart > 0 ? d.max_restart : 30;
    alloc_fixed(s);
    build_all(s);
  }

  // Buffers whose sizes do not depend on the structure's positions, placed
  // first in the workspace: a rebuild at moved positions releases everything
  // above them and lays it out again in the same order.  A member of a batch
  // keeps only its hierarchy (the batch has its own work and outer vectors).
  void alloc_fixed(hipStream_t s) {
    (void)s;
    if (defer_coarse_) return;
    const size_t n = 3 * (size_t)d_.N * d_.N, m2 = 2 * (size_t)std::max(M_, 1);
    const int R = outer_cap_;
    Vo_.alloc((size_t)(R + 1) * n);
    Zo_.alloc((size_t)R * n);
    Ho_.alloc((size_t)(R + 1) * R);
    cs_.alloc(R + 1);
    sn_.alloc(R + 1);
    g_.alloc(R + 2);
    y_.alloc(R + 1);
    osc_.alloc(256);
    opart_.alloc(2 * kOuterPartStride);
    ofold_.alloc(2 * 72);
    bp_.alloc(n);
    rr_.alloc(n);
    vin_.alloc(n);
    vout_.alloc(n);
    Fd_.alloc(2 * m2);   // forces [2][M] then J u [2][M]
    Uw_.alloc(m2);
    Ul_.alloc(m2);
    Fs_.alloc(m2);
    fs_.alloc(2 * (size_t)d_.N * d_.N);
    rhs_.alloc(n);
    if (!pinned_) IBMG_HIP(hipHostMalloc((void**)&pinned_, 8 * sizeof(double), hipHostMallocDefault));
  }

  // Every position-dependent part of the set-up, in workspace order.  With
  // IBMG_SETUP_TIMES set in the environment each phase waits for the device
  // and its wall time goes to stderr (a measurement aid; it serialises the
  // phases).
  void build_all(hipStream_t s) {
    const bool timed = std::getenv("IBMG_SETUP_TIMES") != nullptr;
    auto t = std::chrono::steady_clock::now();
    const auto t_begin = t;
    auto mark = [&](const char* what) {
      if (!timed) return;
      IBMG_HIP(hipStreamSynchronize(s));
      const auto now = std::chrono::steady_clock::now();
      std::fprintf(stderr, "[ibmg set-up] %-16s %8.3f ms\n", what,
                   std::chrono::duration<double, std::milli>(now - t).count());
      t = now;
    };
    build_structure(s, mark);
    if (!defer_coarse_) alloc_work(s);
    mark("work buffers");
    build_numeric(s, mark);
    check_breakdown(s);
    mark("breakdown scan");
    IBMG_HIP(hipStreamSynchronize(s));
    setup_ms_ = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_begin).count();
  }

  // Release everything alloc_fixed did not place (the whole hierarchy, the
  // structure's device arrays, the coarsest inverse and the set-up's slice
  // buffer), leaving the workspace as it was right after alloc_fixed.
  void release_dependent() {
    if (coarse_aug_.n) {   // a set-up that stopped before joining the coarsest inversion
      if (side_) IBMG_HIP(hipStreamSynchronize(side_));
      coarse_aug_.release();
    }
    levels_.clear();
    for (DBuf<int>* b : {&d_adj_ptr_, &d_adj_nbr_, &d_ends_, &d_order_}) b->release();
    for (DBuf<double>* b : {&d_adj_k_, &d_X_, &d_adj_k2_, &d_adj_kap_, &d_adj_rest_, &d_gblocks_, &inv0_, &tpart_,
                            &aug0_})
      b->release();
    d_adj_kf_.release();
    d_adj_k2f_.release();
  }

  // A set-up factorisation that broke down leaves non-finite entries in its
  // inverse (a zero pivot divides by zero); so does a non-finite operator.
  // The coarsest inverse and every level's box inverses are scanned once,
  // and the SC Chebyshev bounds must be finite and positive.
  void check_breakdown(hipStream_t s, bool coarse_only = false) {
    DBuf<int> flag(1);
    if (dry_run()) return;
    int bad = 0;
    auto scan = [&](const auto* a, size_t n, const char* what) {
      if (!n) return;
      launch_fill<int>(flag.p, 0, 1, s);
      launch_count_nonfinite(a, n, flag.p, s);
      IBMG_HIP(hipMemcpyAsync(&bad, flag.p, sizeof(int), hipMemcpyDeviceToHost, s));
      IBMG_HIP(hipStreamSynchronize(s));
      if (bad) throw Error(IBMG_ERR_BREAKDOWN, std::string(what) + " has non-finite entries (singular or non-finite matrix)");
    };
    if (inv0_.n) scan(inv0_.p, inv0_.n, "the coarsest inverse");
    for (int l = 1; l <= L_ && !coarse_only; ++l) {
      Level<T>& lev = levels_[l];
      if (lev.use_sym) {
        scan(lev.inv_sym, (size_t)lev.n_ib * sym_box_stride(lev.g), ("the IB box inverses of level " + std::to_string(l)).c_str());
        scan(lev.wmat, lev.wrow.size() * (size_t)lev.w_stride, ("the IB box factors of level " + std::to_string(l)).c_str());
      } else {
        scan(lev.inv.p, rows_held(lev) * box_stride(lev), ("the box inverses of level " + std::to_string(l)).c_str());
      }
      if (lev.cls.n) scan(lev.cls.p, lev.cls.n, ("the interior box inverse of level " + std::to_string(l)).c_str());
      if (lev.sc)
        if (!(std::isfinite(lev.sc->lamA) && lev.sc->lamA > 0.0 && std::isfinite(lev.sc->lamM) && lev.sc->lamM > 0.0))
          throw Error(IBMG_ERR_BREAKDOWN, "Schur-complement Chebyshev bound of level " + std::to_string(l) +
                                              " is not finite and positive");
    }
  }

  ~Solver() override {
    if (est_ev_) (void)hipEventDestroy(est_ev_);
    if (side_) {
      (void)hipStreamSynchronize(side_);
      (void)hipStreamDestroy(side_);
      (void)hipEventDestroy(ev_fork_);
      (void)hipEventDestroy(ev_join_);
    }
    drop_graph();
    if (gstream_) (void)hipStreamDestroy(gstream_);
    if (pinned_) (void)hipHostFree(pinned_);
  }

  int levels() const override { return L_ + 1; }
  int level_n(int l) const override { return sizes_.at(l); }

  // ---------------------------------------------------------------- set-up
  template <typename Mark>
  void build_structure(hipStream_t s, Mark& mark) {
    // spring adjacency (node -> incident springs in spring order)
    adj_ptr_.assign(M_ + 1, 0);
    for (int e = 0; e < E_; ++e) {
      adj_ptr_[ends_[2 * e] + 1]++;
      adj_ptr_[ends_[2 * e + 1] + 1]++;
    }
    for (int l = 0; l < M_; ++l) adj_ptr_[l + 1] += adj_ptr_[l];
    adj_nbr_.assign(adj_ptr_[M_], 0);
    adj_sid_.assign(adj_ptr_[M_], 0);
    {
      std::vector<int> fill(adj_ptr_.begin(), adj_ptr_.end() - 1);
      for (int e = 0; e < E_; ++e) {
        const int a = ends_[2 * e], b = ends_[2 * e + 1];
        adj_nbr_[fill[a]] = b;
        adj_sid_[fill[a]++] = e;
        adj_nbr_[fill[b]] = a;
        adj_sid_[fill[b]++] = e;
      }
    }
    d_adj_ptr_.upload(adj_ptr_, s);
    d_adj_nbr_.upload(adj_nbr_, s);
    d_ends_.upload(ends_, s);
    d_X_.upload(X_, s);
    levels_.resize(L_ + 1);
    for (int l = L_; l >= 0; --l) {
      Level<T>& lev = levels_[l];
      lev.N = sizes_[l];
      const double h = 1.0 / lev.N;
      lev.cd = StokesCoef<double>{d_.rho / d_.dt, d_.mu / (h * h), 1.0 / h, d_.dt / (h * h)};
      lev.ct = StokesCoef<T>{(T)lev.cd.alpha, (T)lev.cd.beta, (T)lev.cd.gi, (T)lev.cd.ibs};
      for (int c = 0; c < 2; ++c) {
        if (l == L_) fine_windows(lev.N, c, lev.f[c]);
        else coarse_windows(levels_[l + 1].f[c], c, levels_[l + 1].N, lev.N, lev.f[c]);
      }
    }
    // every level's and component's lists and the points' order, largest first
    // (512^2 with 8192 points, copies included: 4.7 -> 3.6 ms; the box classes and
    // row lists below 2.8 -> 1.8 ms)
    std::vector<int> order;
    parallel_for(2 * (size_t)(L_ + 1) + 1, [&](size_t i) {
      if (i == 0) order = point_order(levels_[L_].N, levels_[L_].f[0]);
      else spread_lists(levels_[L_ - (i - 1) / 2].N, levels_[L_ - (i - 1) / 2].f[(i - 1) % 2]);
    });
    for (int l = L_; l >= 0; --l) {
      Level<T>& lev = levels_[l];
      for (int c = 0; c < 2; ++c) {
        CompFoot& f = lev.f[c];
        f.d_base.upload(f.base, s);
        f.d_mask.upload(f.mask, s);
        f.w.alloc((size_t)M_ * 16);
        if (l == L_)
          launch_fp_fine(d_X_.p, M_, lev.N, c, f.d_base.p, f.d_mask.p, f.w.p, s);
        else
          launch_fp_coarsen(levels_[l + 1].f[c].d_base.p, levels_[l + 1].f[c].w.p, f.d_base.p, M_, c,
                            levels_[l + 1].N, lev.N, f.w.p, s);
        if (std::is_same<T, float>::value) {
          f.wf.alloc((size_t)M_ * 16);
          launch_cast<double, float>(f.w.p, f.wf.p, (size_t)M_ * 16, s);
        }
        f.d_sp_ptr.upload(f.sp_ptr, s);
        f.d_sp_ent.upload(f.sp_ent, s);
        f.sw.alloc(std::max<size_t>(f.sp_ent.size(), 1));
        launch_gather_weights<double>(f.w.p, f.d_sp_ent.p, f.sp_ent.size(), f.sw.p, s);
        if (std::is_same<T, float>::value) {
          f.swf.alloc(std::max<size_t>(f.sp_ent.size(), 1));
          launch_gather_weights<float>(f.w.p, f.d_sp_ent.p, f.sp_ent.size(), f.swf.p, s);
        }
        if (l == L_ && c == 0) d_order_.upload(order, s);
        // the interpolation walks points in cell order and reads their
        // windows there, so it gets copies laid out in that order
        f.d_obase.alloc(2 * (size_t)M_);
        f.ow.alloc((size_t)M_ * 16);
        launch_walk_order<double>(d_order_.p, f.d_base.p, f.w.p, M_, f.d_obase.p, f.ow.p, s);
        if (std::is_same<T, float>::value) {
          f.owf.alloc((size_t)M_ * 16);
          launch_walk_order<float>(d_order_.p, f.d_base.p, f.wf.p, M_, f.d_obase.p, f.owf.p, s);
        }
      }
    }
    mark("windows, lists");
    ib_patterns();   // IB rows need both components' windows
    mark("IB row patterns");
    std::vector<std::vector<unsigned char>> flags(L_ + 1);
    parallel_for(L_ + 1, [&](size_t i) {
      const int l = L_ - (int)i;
      list_ib_rows(levels_[l], flags[l]);
      if (l >= 1 && (d_.smoother == IBMG_RAS || d_.smoother == IBMG_RMS)) classify_boxes(levels_[l]);
      if (l >= 1 && d_.smoother == IBMG_RMS) colour_boxes(levels_[l]);
    });
    for (int l = L_; l >= 0; --l) {
      Level<T>& lev = levels_[l];
      for (int c = 0; c < 2; ++c) {
        CompFoot& f = lev.f[c];
        f.d_tptr.upload(f.tptr, s);
        f.d_tcol.upload(f.tcol, s);
        f.tval.alloc(f.tcol.size());
        if (std::is_same<T, float>::value) f.tvalf.alloc(f.tcol.size());
      }
      if (lev.ib_lanes) {
        lev.d_ib_rows.upload(lev.ib_rows, s);
        lev.d_ib_flag.upload(flags[l], s);
      }
      if (l >= 1 && d_.smoother == IBMG_SC) sc_structure(lev, s);
    }
    mark("box classes");
  }

  // The level's rows with IB entries, the faces' flags and the lanes a row
  // gets in the operator's launch (0: too many entries, see ib_rows_max_entries).
  void list_ib_rows(Level<T>& lev, std::vector<unsigned char>& flag) const {
    const int nn = lev.N * lev.N;
    const size_t nnz = lev.f[0].tcol.size() + lev.f[1].tcol.size();
    lev.ib_rows.clear();
    lev.n_ib_v = 0;
    lev.ib_lanes = 0;
    const int longest = std::max(lev.f[0].max_list, lev.f[1].max_list);
    // (a batch runs every member's rows in one launch, whatever their number)
    if (!defer_coarse_ && (nnz == 0 || nnz > ib_rows_max_entries(longest, M_) || std::getenv("IBMG_NO_IB_ROWS"))) return;
    flag.assign(nn, 0);
    for (int c = 0; c < 2; ++c)
      for (int q = 0; q < nn && !lev.f[c].tcol.empty(); ++q)
        if (lev.f[c].tptr[q + 1] > lev.f[c].tptr[q]) {
          lev.ib_rows.push_back(c * nn + q);
          lev.n_ib_v += c;
          flag[q] |= (unsigned char)(1 << c);
        }
    lev.ib_lanes = nnz > (size_t)kIbLongRow * lev.ib_rows.size() ? 64 : 16;
  }

  // Points in cell order (row-major by the finest x-window base, ties in
  // index order), the order in which the point-wise kernels walk them.
  std::vector<int> point_order(int N, const CompFoot& f) const {
    std::vector<int> ord(std::max(M_, 1), 0);
    std::iota(ord.begin(), ord.begin() + M_, 0);
    std::stable_sort(ord.begin(), ord.begin() + M_, [&](int a, int b) {
      const long long ka = (long long)f.base[2 * a + 1] * N + f.base[2 * a];
      const long long kb = (long long)f.base[2 * b + 1] * N + f.base[2 * b];
      return ka < kb;
    });
    return ord;
  }

  // Finest windows: t = X N - shift, i0 = floor(t) - 1, slots with |t - k| < 2.
  void fine_windows(int N, int comp, CompFoot& f) {
    f.base.assign(2 * (size_t)M_, 0);
    f.mask.assign(M_, 0);
    const double sx = comp == 0 ? 0.0 : 0.5, sy = comp == 0 ? 0.5 : 0.0;
    for (int l = 0; l < M_; ++l) {
      const double tx = X_[2 * l] * N - sx, ty = X_[2 * l + 1] * N - sy;
      const int i0 = (int)std::floor(tx) - 1, j0 = (int)std::floor(ty) - 1;
      int mk = 0;
      for (int b = 0; b < 4; ++b)
        for (int a = 0; a < 4; ++a)
          if (std::fabs(tx - (i0 + a)) < 2.0 && std::fabs(ty - (j0 + b)) < 2.0) mk |= 1 << (b * 4 + a);
      f.base[2 * l] = wrapn(i0, N);
      f.base[2 * l + 1] = wrapn(j0, N);
      f.mask[l] = mk;
    }
  }

  // Coarse windows: base = fine base / 2; a coarse slot is structural when a
  // structural fine slot is interpolated from it by P_u.
  void coarse_windows(const CompFoot& ff, int comp, int Nf, int Nc, CompFoot& f) {
    (void)Nf;
    f.base.assign(2 * (size_t)M_, 0);
    f.mask.assign(M_, 0);
    for (int l = 0; l < M_; ++l) {
      const int I0 = ff.base[2 * l], J0 = ff.base[2 * l + 1];
      const int ci0 = I0 >> 1, cj0 = J0 >> 1;
      int mk = 0;
      for (int s = 0; s < 16; ++s) {
        if (!((ff.mask[l] >> s) & 1)) continue;
        const int I = I0 + (s & 3), J = J0 + (s >> 2);
        if (comp == 0) {
          const int cj = (J >> 1) - cj0;
          if ((I & 1) == 0) mk |= 1 << (cj * 4 + (I >> 1) - ci0);
          else mk |= (1 << (cj * 4 + ((I - 1) >> 1) - ci0)) | (1 << (cj * 4 + ((I + 1) >> 1) - ci0));
        } else {
          const int ci = (I >> 1) - ci0;
          if ((J & 1) == 0) mk |= 1 << (((J >> 1) - cj0) * 4 + ci);
          else mk |= (1 << ((((J - 1) >> 1) - cj0) * 4 + ci)) | (1 << ((((J + 1) >> 1) - cj0) * 4 + ci));
        }
      }
      f.base[2 * l] = wrapn(ci0, Nc);
      f.base[2 * l + 1] = wrapn(cj0, Nc);
      f.mask[l] = mk;
    }
  }

  static int face_of(const CompFoot& f, int l, int s, int N) {
    int i = f.base[2 * l] + (s & 3), j = f.base[2 * l + 1] + (s >> 2);
    if (i >= N) i -= N;
    if (j >= N) j -= N;
    return j * N + i;
  }

  // faces -> (point, slot) entries, entries of a face in increasing (l, s)
  void spread_lists(int N, CompFoot& f) const {
    const size_t nf = (size_t)N * N;
    f.sp_ptr.assign(nf + 1, 0);
    for (int l = 0; l < M_; ++l)
      for (int s = 0; s < 16; ++s)
        if ((f.mask[l] >> s) & 1) f.sp_ptr[face_of(f, l, s, N) + 1]++;
    f.max_list = 0;
    for (size_t r = 0; r < nf; ++r) {
      f.max_list = std::max(f.max_list, f.sp_ptr[r + 1]);
      f.sp_ptr[r + 1] += f.sp_ptr[r];
    }
    f.sp_ent.assign(f.sp_ptr[nf], 0);
    std::vector<int> fill(f.sp_ptr.begin(), f.sp_ptr.end() - 1);
    for (int l = 0; l < M_; ++l)
      for (int s = 0; s < 16; ++s)
        if ((f.mask[l] >> s) & 1) f.sp_ent[fill[face_of(f, l, s, N)]++] = l * 16 + s;
  }

  // Pattern of the comp rows of dt/h^2 J^T K' J: row r couples to every face
  // of every point that shares a spring (or is itself) with a point whose
  // comp-window holds r, in the same component, and with tangent blocks also
  // in the other one.  Columns index [u | v] (v faces offset by N^2), sorted.
  // The IB rows' columns on every level and component (the Galerkin
  // pattern): one pool of worker threads takes chunks of rows of all (level,
  // component) pairs.  Each chunk keeps its own columns and the chunks join
  // in order, so the pattern does not depend on the thread count.  A worker
  // marks the columns of the row in hand with a tag it never reuses, so one
  // stamp array serves every pair without being cleared.
  void ib_patterns() {
    struct Task {
      int l, comp;
      size_t r0, r1;
    };
    constexpr size_t kChunk = 2048;
    std::vector<Task> tasks;
    std::vector<size_t> first(2 * (size_t)(L_ + 1) + 1, 0);   // first task of pair 2 l + comp
    for (int l = 0; l <= L_; ++l)
      for (int c = 0; c < 2; ++c) {
        first[2 * l + c] = tasks.size();
        const size_t nf = (size_t)levels_[l].N * levels_[l].N;
        for (size_t r0 = 0; r0 < nf; r0 += kChunk) tasks.push_back({l, c, r0, std::min(nf, r0 + kChunk)});
      }
    first[2 * (size_t)(L_ + 1)] = tasks.size();
    std::vector<std::vector<int>> ccols(tasks.size()), clen(tasks.size());
    const size_t nf_max = (size_t)levels_[L_].N * levels_[L_].N;
    std::atomic<size_t> next{0};
    auto worker = [&]() {
      std::vector<int> stamp(2 * nf_max, -1);
      std::vector<int> pstamp(std::max(M_, 1), -1);   // points already taken for this row
      std::vector<int> cols, pts;
      int tag = -1;
      for (;;) {
        const size_t ti = next++;
        if (ti >= tasks.size()) break;
        const Task& tk = tasks[ti];
        const Level<T>& lev = levels_[tk.l];
        const int N = lev.N;
        const size_t nf = (size_t)N * N;
        const CompFoot& f = lev.f[tk.comp];
        auto add_point = [&](int q) {
          for (int c = 0; c < 2; ++c) {
            if (c != tk.comp && !tangent_) continue;
            const CompFoot& fc = lev.f[c];
            for (int sl = 0; sl < 16; ++sl) {
              if (!((fc.mask[q] >> sl) & 1)) continue;
              const int col = c * (int)nf + face_of(fc, q, sl, N);
              if (stamp[col] != tag) {
                stamp[col] = tag;
                cols.push_back(col);
              }
            }
          }
        };
        std::vector<int>& out = ccols[ti];
        std::vector<int>& len = clen[ti];
        len.assign(tk.r1 - tk.r0, 0);
        // the points whose windows the row reaches: each spring-carrying
        // point in the face's list and its spring neighbours, each taken once
        auto take = [&](int q) {
          if (pstamp[q] != tag) {
            pstamp[q] = tag;
            pts.push_back(q);
          }
        };
        for (size_t r = tk.r0; r < tk.r1; ++r) {
          if (f.sp_ptr[r + 1] == f.sp_ptr[r]) continue;
          ++tag;
          cols.clear();
          pts.clear();
          for (int e = f.sp_ptr[r]; e < f.sp_ptr[r + 1]; ++e) {
            const int l = f.sp_ent[e] >> 4;
            if (adj_ptr_[l + 1] == adj_ptr_[l]) continue;
            take(l);
            for (int a = adj_ptr_[l]; a < adj_ptr_[l + 1]; ++a) take(adj_nbr_[a]);
          }
          for (int q : pts) add_point(q);
          std::sort(cols.begin(), cols.end());
          out.insert(out.end(), cols.begin(), cols.end());
          len[r - tk.r0] = (int)cols.size();
        }
      }
    };
    // each worker keeps a stamp over the finest [u | v]: at most 1 GiB in all
    const size_t by_mem = std::max<size_t>(1, ((size_t)1 << 30) / (2 * nf_max * sizeof(int)));
    run_workers(worker, std::min(by_mem, tasks.size()));
    parallel_for(2 * (size_t)(L_ + 1), [&](size_t i) {   // largest first
      const int l = L_ - (int)(i / 2), c = (int)(i % 2);
      CompFoot& f = levels_[l].f[c];
      const size_t nf = (size_t)levels_[l].N * levels_[l].N;
      const size_t t0 = first[2 * l + c], t1 = first[2 * l + c + 1];
      f.tptr.assign(nf + 1, 0);
      size_t tot = 0;
      for (size_t t = t0; t < t1; ++t) tot += ccols[t].size();
      f.tcol.clear();
      f.tcol.reserve(tot);
      for (size_t t = t0; t < t1; ++t) {
        for (size_t i = 0; i < clen[t].size(); ++i) f.tptr[tasks[t].r0 + i + 1] = clen[t][i];
        f.tcol.insert(f.tcol.end(), ccols[t].begin(), ccols[t].end());
      }
      f.max_row = 0;
      for (size_t r = 0; r < nf; ++r) {
        f.max_row = std::max(f.max_row, f.tptr[r + 1]);
        f.tptr[r + 1] += f.tptr[r];
      }
    });
  }

  // A box needs its own inverse when one of its faces carries an IB row;
  // every other box has the same (translation-invariant) matrix.
  void classify_boxes(Level<T>& lev) {
    int b, o;
    box_params(lev.N, d_.box, d_.overlap, &b, &o);
    const int m = b + 2 * o, N = lev.N;
    lev.g = BoxGeom{N, b, o, m, N / b, 2 * m * (m + 1) + m * m, 3 * b * b, (3 * b * b + 63) / 64};
    const int nbox = lev.g.npd * lev.g.npd;
    lev.uniq.clear();
    lev.ib_list.clear();
    lev.int_list.clear();
    for (int p = 0; p < nbox; ++p) {
      const int x0 = (p % lev.g.npd) * b - o, y0 = (p / lev.g.npd) * b - o;
      bool ib = false;
      for (int jj = 0; jj <= m && !ib; ++jj)
        for (int ii = 0; ii <= m && !ib; ++ii) {
          const int r = wrapn(y0 + jj, N) * N + wrapn(x0 + ii, N);
          if (jj < m && lev.f[0].tptr[r + 1] > lev.f[0].tptr[r]) ib = true;   // x-face (ii, jj)
          if (ii < m && lev.f[1].tptr[r + 1] > lev.f[1].tptr[r]) ib = true;   // y-face (ii, jj)
        }
      if (ib) lev.ib_list.push_back(p);
      else lev.int_list.push_back(p);
    }
    const int nloc = lev.g.nloc;
    lev.n_ib = (int)lev.ib_list.size();
    lev.uniq = lev.ib_list;
    if (!lev.int_list.empty()) lev.uniq.push_back(lev.int_list.front());
    lev.n_unique = (int)lev.uniq.size();
    if (d_.combine == IBMG_COMBINE_SUM) {
      // every row of every box inverse: the whole local solution is summed
      lev.sum_mode = true;
      lev.g.nown = nloc;
      lev.g.nch = (nloc + 63) / 64;
      lev.bm = BoxMat{nloc, 0, 0};
      return;
    }
    // matrix positions: the non-owned unknowns around the ring, then the owned
    // ones (each box orders them, order_boxes)
    lev.pos.assign(nloc, -1);
    lev.nonown.clear();
    const int bb = b * b, nown = lev.g.nown, nu = m * (m + 1);
    std::vector<int> own(nown);
    for (int r = 0; r < nown; ++r) {
      const int comp = r / bb, oi = r % bb % b + o, oj = r % bb / b + o;
      own[r] = comp == 0 ? oj * (m + 1) + oi : (comp == 1 ? nu + oj * m + oi : 2 * nu + oj * m + oi);
      lev.pos[own[r]] = r;
    }
    for (int k = 0; k < nloc; ++k)
      if (lev.pos[k] < 0) lev.nonown.push_back(k);
    // the ring's sectors (lines of o cells across it): bottom, right, top, left
    // strip, each with the corner it ends in; a face belongs to the first
    // sector of its non-owned cells, faces before cells within a sector
    auto sector = [&](int i, int j) {
      if (i < 0 || j < 0 || i >= m || j >= m) return INT_MAX;
      if (j < o && i < m - o) return i;
      if (i >= m - o && j < m - o) return m - o + j;
      if (j >= m - o && i >= o) return 2 * (m - o) + m - 1 - i;
      if (i < o && j >= o) return 3 * (m - o) + m - 1 - j;
      return INT_MAX;   // owned
    };
    auto key = [&](int k) {
      if (k < nu) {
        const int i = k % (m + 1), j = k / (m + 1);
        return std::array<int, 3>{std::min(sector(i - 1, j), sector(i, j)), 0, k};
      }
      if (k < 2 * nu) {
        const int i = (k - nu) % m, j = (k - nu) / m;
        return std::array<int, 3>{std::min(sector(i, j - 1), sector(i, j)), 0, k};
      }
      return std::array<int, 3>{sector((k - 2 * nu) % m, (k - 2 * nu) / m), 1, k};
    };
    std::sort(lev.nonown.begin(), lev.nonown.end(), [&](int p, int q) { return key(p) < key(q); });
    const int nn = (int)lev.nonown.size(), nnp = (nn + 63) / 64 * 64;
    lev.bm = BoxMat{nnp + nown, nn, nnp};
    for (int r = 0; r < nown; ++r) lev.pos[own[r]] = nnp + r;
    for (int k = 0; k < nn; ++k) lev.pos[lev.nonown[k]] = k;
  }

  // The order of every unique box's owned unknowns in its matrix, and the owned
  // rows that couple to a non-owned unknown of the box (the rows of W): rows
  // whose stencil reaches one, and IB rows with a column on one.  Line by line
  // (x-faces, y-faces, cells) through the uncoupled faces and the cells with
  // four uncoupled faces, then the coupled faces, then the other cells.  The
  // boxes are shared out over worker threads.
  void order_boxes(Level<T>& lev) {
    const BoxGeom& g = lev.g;
    const int N = g.N, NN = N * N, b = g.b, bb = b * b, nown = g.nown, m = g.m;
    std::vector<unsigned char> edge(nown, 0);   // coupled by the stencil
    for (int r = 0; r < nown; ++r) {
      const int comp = r / bb, i = r % bb % b, j = r % bb / b;
      edge[r] = i == b - 1 || j == b - 1 || (comp < 2 && g.o > 0 && (i == 0 || j == 0));
    }
    lev.coupled.assign((size_t)lev.n_unique * nown, 0);
    lev.ord.resize((size_t)lev.n_unique * nown);
    lev.own.resize((size_t)lev.n_unique * nown);
    std::atomic<int> next{0};
    auto worker = [&]() {
      std::vector<unsigned char> cp(nown), late(nown);
      for (int s = next++; s < lev.n_unique; s = next++) {
        cp = edge;
        if (s < lev.n_ib) {   // the last unique box may be the interior one: no IB rows
          const int pid = lev.ib_list[s], ox = pid % g.npd * b, oy = pid / g.npd * b;
          for (int r = 0; r < 2 * bb; ++r) {
            if (cp[r]) continue;
            const CompFoot& f = lev.f[r / bb];
            const int q = (oy + r % bb / b) * N + ox + r % bb % b;
            for (int k = f.tptr[q]; k < f.tptr[q + 1]; ++k) {
              const int comp = f.tcol[k] >= NN ? 1 : 0, c = f.tcol[k] - comp * NN;
              int lj = c / N, li = c - lj * N - ox;   // from the owned corner
              lj -= oy;
              if (li >= 0 && li < b && lj >= 0 && lj < b) continue;   // owned
              li += g.o;
              lj += g.o;
              li = li < 0 ? li + N : (li >= N ? li - N : li);
              lj = lj < 0 ? lj + N : (lj >= N ? lj - N : lj);
              if (comp == 0 ? (li <= m && lj < m) : (li < m && lj <= m)) {
                cp[r] = 1;
                break;
              }
            }
          }
        }
        late = cp;
        for (int j = 0; j < b; ++j)
          for (int i = 0; i < b; ++i) {
            const int q = j * b + i;
            late[2 * bb + q] = i == b - 1 || j == b - 1 || cp[q] || cp[q + 1] || cp[bb + q] || cp[bb + q + b];
          }
        unsigned short *ord = lev.ord.data() + (size_t)s * nown, *own = lev.own.data() + (size_t)s * nown;
        unsigned char* cpos = lev.coupled.data() + (size_t)s * nown;
        int p = 0;
        auto take = [&](int comp0, int comp1, int which) {
          for (int j = 0; j < b; ++j)
            for (int comp = comp0; comp < comp1; ++comp)
              for (int i = 0; i < b; ++i) {
                const int r = comp * bb + j * b + i;
                if (late[r] != which) continue;
                ord[p] = (unsigned short)r;
                own[r] = (unsigned short)p;
                cpos[p++] = cp[r];
              }
        };
        take(0, 3, 0);
        take(0, 2, 1);
        take(2, 3, 1);
      }
    };
    run_workers(worker, (size_t)lev.n_unique * nown / 16384 + 1);
  }

  // The rows of W of a level's IB boxes (order_boxes done).
  void list_w_rows(Level<T>& lev) {
    const int nown = lev.g.nown;
    lev.wptr.assign(1, 0);
    lev.wrow.clear();
    lev.w_max = 0;
    for (int s = 0; s < lev.n_ib; ++s) {
      for (int r = 0; r < nown; ++r)
        if (lev.coupled[(size_t)s * nown + r]) lev.wrow.push_back(r);
      lev.wptr.push_back((int)lev.wrow.size());
      lev.w_max = std::max(lev.w_max, lev.wptr[s + 1] - lev.wptr[s]);
    }
    lev.w_stride = (lev.bm.nn + 3) / 4 * 4;
  }

  // fn on up to 16 host threads, at most `most` of them
  template <typename F>
  static void run_workers(F& fn, size_t most) {
    const size_t hw = std::max(1u, std::thread::hardware_concurrency());
    const size_t nth = std::min({(size_t)16, hw, most});
    if (nth <= 1) {
      fn();
      return;
    }
    // (an exception in a worker is thrown again here, after all have ended)
    std::exception_ptr err;
    std::mutex mu;
    auto guarded = [&] {
      try {
        fn();
      } catch (...) {
        const std::lock_guard<std::mutex> lock(mu);
        if (!err) err = std::current_exception();
      }
    };
    std::vector<std::thread> th;
    try {
      for (size_t t = 1; t < nth; ++t) th.emplace_back(guarded);
    } catch (...) {   // fewer threads than asked for
    }
    guarded();
    for (auto& t : th) t.join();
    if (err) std::rethrow_exception(err);
  }

  // fn(i) for i < n on the host threads
  template <typename F>
  static void parallel_for(size_t n, F fn) {
    std::atomic<size_t> next{0};
    auto worker = [&] {
      for (size_t i = next++; i < n; i = next++) fn(i);
    };
    run_workers(worker, n);
  }

  size_t box_stride(const Level<T>& lev) const { return (size_t)lev.g.nch * lev.g.nloc * 64; }

  // Every Schwarz launch goes through here: boxes [i0, i1) of the IB list and
  // [k0, k1) of the interior list.
  void ras_launch(Level<T>& lev, const T* r, T* z, int i0, int i1, int k0, int k1, hipStream_t s, int parts, bool acc) {
    const SymIB sy = sym_of(lev, i0);
    launch_ras_apply<T>(r, z, lev.g, lev.inv.p + (lev.use_sym ? 0 : (size_t)i0 * box_stride(lev)), lev.d_ib.p + i0,
                        i1 - i0, lev.clsv, lev.d_int.p + k0, k1 - k0, s, parts, acc, lev.use_sym ? &sy : nullptr);
  }

  // blocks of the fused operator + dots kernel on a level
  static int dot_blocks(const Level<T>& lev) {
    return apply_blocks(lev.N, lev.ib_lanes ? (int)lev.ib_rows.size() : 0, lev.ib_lanes);
  }

  // partial-sum buffers of a level: the reductions' blocks x vectors, and the
  // fused operator kernel's blocks x (nu + 1) vectors
  static size_t part_stride(const Level<T>& lev) {
    return (size_t)std::max({dot_blocks(lev), gs_blocks(3 * (size_t)lev.N * lev.N), 1024}) * (kMaxNu + 1);
  }

  // Orbits of a box's local unknowns under its two reflections (ras_int_block):
  // one representative per orbit for the columns, and for the rows every orbit
  // that holds an owned unknown, represented by an owned one.
  void class_tables(Level<T>& lev) {
    const BoxGeom& g = lev.g;
    const int m = g.m, nu = m * (m + 1);
    auto local = [&](int c, int i, int j) { return c == 0 ? j * (m + 1) + i : (c == 1 ? nu + j * m + i : 2 * nu + j * m + i); };
    auto owned = [&](int i, int j) { return i >= g.o && i < g.o + g.b && j >= g.o && j < g.o + g.b; };
    lev.kcode.clear();
    lev.klocal.clear();
    lev.rcode.clear();
    lev.rlocal.clear();
    for (int c = 0; c < 3; ++c) {
      const int mx = c == 0 ? m : m - 1, my = c == 1 ? m : m - 1;   // images: mx - i, my - j
      for (int j = 0; 2 * j <= my; ++j)
        for (int i = 0; 2 * i <= mx; ++i) {
          lev.kcode.push_back((c << 24) | (j << 12) | i);
          for (int l : {local(c, i, j), local(c, mx - i, j), local(c, i, my - j), local(c, mx - i, my - j)})
            lev.klocal.push_back(lev.pos[l]);
          // an owned image e of the orbit, and which of its images are owned
          // (each unknown once)
          for (const auto& e : {std::pair<int, int>{i, j}, {mx - i, j}, {i, my - j}, {mx - i, my - j}}) {
            if (!owned(e.first, e.second)) continue;
            const int a = e.first, b = e.second, xa = mx - a, yb = my - b;
            int bits = 1;
            if (xa != a && owned(xa, b)) bits |= 2;
            if (yb != b && owned(a, yb)) bits |= 4;
            if (xa != a && yb != b && owned(xa, yb)) bits |= 8;
            lev.rcode.push_back((bits << 26) | (c << 24) | (b << 12) | a);
            lev.rlocal.push_back(lev.pos[local(c, a, b)] - lev.bm.nnp);
            break;
          }
        }
    }
  }

  // Colours of the multiplicative sweep (Alg. 3 in colour-major order).
  // Box p reaches box q when a row of p's enlarged box couples, through the
  // five-point stencil, the IB rows, G or D, to an unknown owned by q
  // (unknowns are owned by the box of their cell: left x-face, bottom
  // y-face, pressure); reaching in either direction is a conflict.  Boxes
  // take, in index order, the smallest colour unused by coloured conflicting
  // boxes; the box lists are then sorted by colour.
  void colour_boxes(Level<T>& lev) {
    const BoxGeom& g = lev.g;
    const int N = g.N, b = g.b, o = g.o, m = g.m, npd = g.npd, nb = npd * npd;
    std::vector<std::vector<int>> adj(nb);
    std::vector<int> stamp(nb, -1);
    auto owner = [&](int i, int j) { return (wrapn(j, N) / b) * npd + wrapn(i, N) / b; };
    for (int p = 0; p < nb; ++p) {
      const int x0 = (p % npd) * b - o, y0 = (p / npd) * b - o;
      auto touch = [&](int q) {
        if (q != p && stamp[q] != p) {
          stamp[q] = p;
          adj[p].push_back(q);
          adj[q].push_back(p);
        }
      };
      auto ib_cols = [&](int comp, int i, int j) {
        const CompFoot& f = lev.f[comp];
        const int r = wrapn(j, N) * N + wrapn(i, N);
        for (int k = f.tptr[r]; k < f.tptr[r + 1]; ++k) {
          const int face = f.tcol[k] % (N * N);   // columns index [u | v]
          touch(owner(face % N, face / N));
        }
      };
      for (int jj = 0; jj <= m; ++jj)
        for (int ii = 0; ii <= m; ++ii) {
          const int i = x0 + ii, j = y0 + jj;
          if (jj < m) {  // x-face (i, j): u stencil, G (cells (i, j), (i-1, j)), IB row
            touch(owner(i, j));
            touch(owner(i - 1, j));
            touch(owner(i + 1, j));
            touch(owner(i, j - 1));
            touch(owner(i, j + 1));
            ib_cols(0, i, j);
          }
          if (ii < m) {  // y-face (i, j): v stencil, G (cells (i, j), (i, j-1)), IB row
            touch(owner(i, j));
            touch(owner(i - 1, j));
            touch(owner(i + 1, j));
            touch(owner(i, j - 1));
            touch(owner(i, j + 1));
            ib_cols(1, i, j);
          }
          if (ii < m && jj < m) {  // cell (i, j): D (faces (i, j), (i+1, j), (i, j+1))
            touch(owner(i, j));
            touch(owner(i + 1, j));
            touch(owner(i, j + 1));
          }
        }
    }
    lev.box_colour.assign(nb, -1);
    std::vector<int> mark;
    lev.ncolour = 0;
    for (int p = 0; p < nb; ++p) {
      for (int q : adj[p])
        if (lev.box_colour[q] >= 0) {
          if ((int)mark.size() <= lev.box_colour[q]) mark.resize(lev.box_colour[q] + 1, -1);
          mark[lev.box_colour[q]] = p;
        }
      int c = 0;
      while (c < (int)mark.size() && mark[c] == p) ++c;
      lev.box_colour[p] = c;
      lev.ncolour = std::max(lev.ncolour, c + 1);
    }
    auto by_colour = [&](std::vector<int>& list, std::vector<int>& off) {
      std::stable_sort(list.begin(), list.end(),
                       [&](int a, int bb) { return lev.box_colour[a] < lev.box_colour[bb]; });
      off.assign(lev.ncolour + 1, 0);
      for (int q : list) off[lev.box_colour[q] + 1]++;
      for (int c = 0; c < lev.ncolour; ++c) off[c + 1] += off[c];
    };
    by_colour(lev.ib_list, lev.ib_off);
    by_colour(lev.int_list, lev.int_off);
    lev.uniq = lev.ib_list;
    if (!lev.int_list.empty()) lev.uniq.push_back(lev.int_list.front());
  }

  // Per spring the unit block B_e = K_e / kappa_e of the tangent model at the
  // current positions: (1 - L/l) I + (L/l) t t^T (B_xx, B_xy, B_yy), the
  // identity for L = 0.
  std::vector<double> unit_blocks() const {
    std::vector<double> B(3 * (size_t)E_);
    for (int e = 0; e < E_; ++e) {
      const double L = rest_[e];
      if (L == 0.0) {
        B[3 * e] = 1.0;
        B[3 * e + 1] = 0.0;
        B[3 * e + 2] = 1.0;
        continue;
      }
      const int a = ends_[2 * e], b = ends_[2 * e + 1];
      double dx = X_[2 * b] - X_[2 * a], dy = X_[2 * b + 1] - X_[2 * a + 1];
      dx -= std::nearbyint(dx);
      dy -= std::nearbyint(dy);
      const double len = std::hypot(dx, dy);
      require(len > 0.0, "spring " + std::to_string(e) + " has zero length and a non-zero rest length");
      const double tx = dx / len, ty = dy / len, g = L / len;
      B[3 * e] = (1.0 - g) + g * tx * tx;
      B[3 * e + 1] = g * tx * ty;
      B[3 * e + 2] = (1.0 - g) + g * ty * ty;
    }
    return B;
  }

  template <typename Mark>
  void build_numeric(hipStream_t s, Mark& mark) {
    // spring stiffness per incidence: kappa_e, or the tangent block K_e
    const size_t na = adj_nbr_.size();
    std::vector<double> ak(na);
    for (size_t a = 0; a < na; ++a) ak[a] = kappa_[adj_sid_[a]];
    if (tangent_) {
      const std::vector<double> B = unit_blocks();
      std::vector<double> k00(na), k2(2 * na), rest(na);
      for (size_t a = 0; a < na; ++a) {
        const int e = adj_sid_[a];
        k00[a] = kappa_[e] * B[3 * e];
        k2[2 * a] = kappa_[e] * B[3 * e + 1];
        k2[2 * a + 1] = kappa_[e] * B[3 * e + 2];
        rest[a] = rest_[e];
      }
      d_adj_kap_.upload(ak, s);
      d_adj_rest_.upload(rest, s);
      d_gblocks_.upload(B, s);
      ak.swap(k00);
      d_adj_k2_.upload(k2, s);
      if (std::is_same<T, float>::value) {
        std::vector<float> k2f(k2.begin(), k2.end());
        d_adj_k2f_.upload(k2f, s);
      }
    }
    d_adj_k_.upload(ak, s);
    if (std::is_same<T, float>::value) {
      std::vector<float> akf(ak.begin(), ak.end());
      d_adj_kf_.upload(akf, s);
    }
    for (int l = L_; l >= 0; --l) {
      Level<T>& lev = levels_[l];
      for (int c = 0; c < 2; ++c) {
        CompFoot& f = lev.f[c];
        if (!f.tcol.empty()) {
          // faces of coarse levels carry thousands of points: their rows'
          // point lists are shared out over several waves, 16 points each (a
          // gradient at 256^2, two solves and a rebuild: 15.5 ms with slices of 64
          // points, 15.1 with 32, 14.9 with 16)
          const size_t nnz = f.tcol.size();
          int nslice = std::min(32, std::max(1, f.max_list / 16));
          while (nslice > 1 && (size_t)nslice * nnz > ((size_t)1 << 27)) nslice /= 2;   // <= 1 GiB of slices
          if (nslice > 1 && tpart_.n < (size_t)nslice * nnz) tpart_.alloc((size_t)nslice * nnz);
          const size_t n_u = lev.ib_rows.size() - lev.n_ib_v;
          launch_t_values(fview<double>(lev.f[0]), fview<double>(lev.f[1]), lev.f[0].d_mask.p, lev.f[1].d_mask.p,
                          sview<double>(), c, lev.N, lev.cd.ibs, f.d_tptr.p, f.d_tcol.p, f.tval.p, nslice, nnz,
                          tpart_.p, lev.ib_lanes ? lev.d_ib_rows.p + (c ? n_u : 0) : nullptr,
                          (int)(c ? lev.n_ib_v : n_u), f.max_row, s);
          if (std::is_same<T, float>::value)
            launch_cast<double, float>(f.tval.p, f.tvalf.p, f.tcol.size(), s);
        }
      }
    }
    mark("IB rows");
    build_coarse(s);
    mark("coarsest (queued)");
    if (d_.smoother == IBMG_RAS || d_.smoother == IBMG_RMS) build_boxes(s);
    if (d_.smoother == IBMG_SC)
      for (int l = 1; l <= L_; ++l) sc_numeric(levels_[l], s);
    join_coarse(s);
    mark("smoother data");
  }

  // ------------------------------------------------ Schur-complement set-up
  void sc_structure(Level<T>& lev, hipStream_t s) {
    const int N = lev.N, NN = N * N;
    lev.sc.reset(new ScLevel<T>());
    ScLevel<T>& sc = *lev.sc;
    sc.N = N;
    sc.its = d_.cheb_its;
    sc.rho_zero = d_.rho == 0.0;
    // velocity colours: five-point stencil plus IB rows, both components in
    // one greedy pass in row order (with uncoupled components this equals
    // colouring each component alone; tangent blocks couple u and v rows)
    std::vector<int> colv = greedy_colours(2 * NN, [&](int r, std::vector<int>& nb) {
      const int comp = r >= NN ? 1 : 0, q = r - comp * NN, o = comp * NN;
      const int i = q % N, j = q / N;
      nb.push_back(o + j * N + (i + 1) % N);
      nb.push_back(o + j * N + (i + N - 1) % N);
      nb.push_back(o + ((j + 1) % N) * N + i);
      nb.push_back(o + ((j + N - 1) % N) * N + i);
      const CompFoot& f = lev.f[comp];
      for (int k = f.tptr[q]; k < f.tptr[q + 1]; ++k) nb.push_back(f.tcol[k]);
    });
    sc.colu.build(colv, [&](int r) {
      const int comp = r >= NN ? 1 : 0, q = r - comp * NN;
      const CompFoot& f = lev.f[comp];
      return f.tptr[q + 1] - f.tptr[q] > kGsLongRow;
    }, s);
    build_band_runs<T>(sc.colu, lev.f[0].tptr, lev.f[0].tcol, lev.f[1].tptr, lev.f[1].tcol, N, sc.runs_u, s);
    std::vector<int> colp = greedy_colours(NN, [&](int r, std::vector<int>& nb) {
      const int i = r % N, j = r / N;
      nb.push_back(j * N + (i + 1) % N);
      nb.push_back(j * N + (i + N - 1) % N);
      nb.push_back(((j + 1) % N) * N + i);
      nb.push_back(((j + N - 1) % N) * N + i);
    });
    sc.colp.build(colp, [](int) { return false; }, s);
    const size_t n2 = 2 * (size_t)NN, n1 = NN;
    sc.diag.alloc(n2);
    sc.dinv.alloc(n2);
    sc.mdiag.alloc(n1);
    for (DBuf<T>* b : {&sc.yu, &sc.ga, &sc.gx, &sc.ad, &sc.ar, &sc.at, &sc.as}) b->alloc(n2);
    for (DBuf<T>* b : {&sc.md, &sc.mr, &sc.mt, &sc.ms, &sc.ones}) b->alloc(n1);
    sc.part.alloc(1024);
    launch_fill<T>(sc.ones.p, T(1), n1, s);
  }

  // Largest Ritz value of ten Arnoldi steps (classical Gram-Schmidt twice)
  // of op from v0 (overwritten).
  template <typename OP>
  double arnoldi_lambda(size_t n, T* v0, OP op, hipStream_t s) {
    constexpr int steps = 10;
    DBuf<T> V((size_t)(steps + 1) * n);
    DBuf<double> part(2 * kPartStride), hd(64);
    if (dry_run()) return 1.0;
    const int nblk = dots_blocks(n, 256);
    std::vector<double> H((steps + 1) * steps, 0.0), h(steps + 1), h2(steps + 1);
    auto norm_of = [&](const T* x) {
      launch_dots<T>(x, 1, n, x, n, part.p, nblk, s);
      launch_dots_finish(part.p, 1, nblk, hd.p, nullptr, 2, s);
      double v;
      IBMG_HIP(hipMemcpyAsync(&v, hd.p, sizeof(double), hipMemcpyDeviceToHost, s));
      IBMG_HIP(hipStreamSynchronize(s));
      return v;
    };
    const double b0 = norm_of(v0);
    launch_scale<T>(v0, V.p, hd.p, n, s);
    int k = steps;
    for (int j = 0; j < steps; ++j) {
      T* w = V.p + (size_t)(j + 1) * n;
      op(V.p + (size_t)j * n, w);
      for (int pass = 0; pass < 2; ++pass) {
        launch_dots<T>(V.p, j + 1, n, w, n, part.p, nblk, s);
        launch_dots_finish(part.p, j + 1, nblk, hd.p, nullptr, 0, s);
        launch_update<T>(w, V.p, j + 1, n, hd.p, -1.0, n, s);
        IBMG_HIP(hipMemcpyAsync(h2.data(), hd.p, (j + 1) * sizeof(double), hipMemcpyDeviceToHost, s));
        IBMG_HIP(hipStreamSynchronize(s));
        for (int i = 0; i <= j; ++i) H[i * steps + j] += h2[i];
      }
      const double hn = norm_of(w);
      H[(j + 1) * steps + j] = hn;
      if (hn == 0.0) {
        k = j + 1;
        break;
      }
      launch_scale<T>(w, w, hd.p, n, s);
    }
    (void)b0;
    std::vector<double> Hk((size_t)k * k);
    for (int i = 0; i < k; ++i)
      for (int j = 0; j < k; ++j) Hk[(size_t)i * k + j] = H[i * steps + j];
    return hessenberg_max_real_eig(Hk, k);
  }

  void sc_numeric(Level<T>& lev, hipStream_t s) {
    ScLevel<T>& sc = *lev.sc;
    const int N = lev.N, NN = N * N;
    const size_t n2 = 2 * (size_t)NN, n1 = NN;
    sc.c = coef<T>(lev);
    sc.tu = csr<T>(lev.f[0]);
    sc.ib_rows = lev.ib_lanes ? lev.d_ib_rows.p : nullptr;
    sc.n_ib_rows = lev.ib_lanes ? (int)lev.ib_rows.size() : 0;
    sc.tv = csr<T>(lev.f[1]);
    sc.ih2 = (T)((double)N * N);
    launch_sc_diag<T>(N, sc.c, sc.tu, sc.tv, sc.ih2, sc.diag.p, sc.dinv.p, sc.mdiag.p, s);
    for (BandRun<T>& run : sc.runs_u) launch_band_values<T>(run, sc.c, sc.tu, sc.tv, N, sc.diag.p, s);
    const int nb1 = dots_blocks(n1, 256);
    // lam for SGS(A_IB)^{-1} A_IB, start vector with the velocity means
    // removed when rho = 0
    DBuf<T> v0(n2);
    launch_weyl<T>(v0.p, n2, s);
    if (sc.rho_zero)
      for (int c = 0; c < 2; ++c) {
        launch_dots<T>(sc.ones.p, 1, n1, v0.p + (size_t)c * n1, n1, sc.part.p, nb1, s);
        launch_sub_mean<T>(v0.p + (size_t)c * n1, n1, sc.part.p, nb1, s);
      }
    sc.lamA = arnoldi_lambda(n2, v0.p, [&](const T* x, T* y) {
      launch_aib_apply<T>(x, sc.at.p, N, sc.c, sc.tu, sc.tv, s);
      sc.sgs_a(sc.at.p, y, s);
    }, s);
    ScLevel<T>::cheb_coefs(sc.lamA, sc.its, &sc.a_theta_inv, sc.a_c1, sc.a_c2);
    // lam for SGS(-M^)^{-1} (-D A~^{-1} G), mean-free start vector
    DBuf<T> q0(n1);
    launch_weyl<T>(q0.p, n1, s);
    launch_dots<T>(sc.ones.p, 1, n1, q0.p, n1, sc.part.p, nb1, s);
    launch_sub_mean<T>(q0.p, n1, sc.part.p, nb1, s);
    sc.lamM = arnoldi_lambda(n1, q0.p, [&](const T* x, T* y) {
      sc.schur_op(x, sc.mt.p, s);
      sc.sgs_m(sc.mt.p, y, s);
    }, s);
    ScLevel<T>::cheb_coefs(sc.lamM, sc.its, &sc.m_theta_inv, sc.m_c1, sc.m_c2);
    IBMG_HIP(hipStreamSynchronize(s));
  }

  // Springs shorter than their rest length (tangent model): the velocity
  // blocks may be indefinite, so the coarsest elimination pivots.
  bool compressed() const {
    if (!tangent_) return false;
    for (int e = 0; e < E_; ++e) {
      double dx = X_[2 * ends_[2 * e + 1]] - X_[2 * ends_[2 * e]], dy = X_[2 * ends_[2 * e + 1] + 1] - X_[2 * ends_[2 * e] + 1];
      dx -= std::nearbyint(dx);
      dy -= std::nearbyint(dy);
      if (rest_[e] > std::hypot(dx, dy)) return true;
    }
    return false;
  }

  void build_coarse(hipStream_t s) {
    Level<T>& lev = levels_[0];
    const int N = lev.N;
    n0_ = 3 * N * N;
    const CoarseShift sh = coarse_shift(lev.cd, d_.rho == 0.0);
    auto assemble_sym = [&](double* mat) {
      launch_fill<double>(mat, 0.0, (size_t)n0_ * n0_, s);
      launch_coarse_assemble_sym(N, lev.cd, lev.f[0].d_tptr.p, lev.f[0].d_tcol.p, lev.f[0].tval.p, lev.f[1].d_tptr.p,
                                 lev.f[1].d_tcol.p, lev.f[1].tval.p, sh, mat, s);
    };
    if (defer_coarse_) {   // (linear springs: no pivoting)
      aug0_.alloc((size_t)n0_ * n0_);
      assemble_sym(aug0_.p);
      IBMG_HIP(hipStreamSynchronize(s));
      return;
    }
    // The inversion is a chain of small latency-bound launches: it runs on a
    // second stream (default priority) beside the box inversions and is
    // joined by join_coarse before anything reads the inverse.
    const bool pivot = compressed();
    const int nb = d_.rho == 0.0 ? 3 : 1, nn = n0_ + nb;
    const size_t mat = pivot ? (size_t)nn * 2 * nn : (size_t)n0_ * n0_;
    // (a tangent handle's rebuilds may change between the two)
    const size_t swept = 2 * (size_t)n0_ * n0_ + sweep_work(n0_, 1);
    DBuf<double> aug(tangent_ ? std::max(swept, (size_t)nn * 2 * nn) : swept);
    if (pivot) {
      launch_fill<double>(aug.p, 0.0, mat, s);
      launch_coarse_assemble(N, lev.cd, lev.f[0].d_tptr.p, lev.f[0].d_tcol.p, lev.f[0].tval.p,
                             lev.f[1].d_tptr.p, lev.f[1].d_tcol.p, lev.f[1].tval.p, nb, aug.p, s);
    } else {
      assemble_sym(aug.p);
    }
    inv0_.alloc((size_t)n0_ * n0_);
    if (!pivot)   // the matrix stays, for the refinement
      IBMG_HIP(hipMemcpyAsync(inv0_.p, aug.p, mat * sizeof(double), hipMemcpyDeviceToDevice, s));
    if (!dry_run() && !side_) {
      IBMG_HIP(hipStreamCreateWithFlags(&side_, hipStreamNonBlocking));
      IBMG_HIP(hipEventCreateWithFlags(&ev_fork_, hipEventDisableTiming));
      IBMG_HIP(hipEventCreateWithFlags(&ev_join_, hipEventDisableTiming));
    }
    IBMG_HIP(hipEventRecord(ev_fork_, s));
    IBMG_HIP(hipStreamWaitEvent(side_, ev_fork_, 0));
    if (pivot) {
      launch_coarse_invert(aug.p, nn, side_);
      launch_coarse_extract(aug.p, nn, n0_, inv0_.p, side_);
    } else {
      launch_gj_invert(aug.p, n0_, 1, aug.p + 2 * mat, side_);
      launch_coarse_refine(aug.p, inv0_.p, aug.p + mat, N, sh, inv0_.p, side_);
    }
    IBMG_HIP(hipEventRecord(ev_join_, side_));
    coarse_aug_ = std::move(aug);
  }

  // The caller's stream waits for the coarsest inversion; its work matrix
  // is then released (later work on the stream is ordered after the join).
  void join_coarse(hipStream_t s) {
    if (!coarse_aug_.n) return;
    IBMG_HIP(hipStreamWaitEvent(s, ev_join_, 0));
    coarse_aug_.release();
  }

  // the coarsest inverse from the caller's swept copy of aug0_ (R: as large)
  void finish_coarse(const double* swept, double* R, hipStream_t s) {
    Level<T>& lev = levels_[0];
    inv0_.alloc((size_t)n0_ * n0_);
    launch_coarse_refine(swept, aug0_.p, R, lev.N, coarse_shift(lev.cd, d_.rho == 0.0), inv0_.p, s);
    aug0_.release();
    defer_coarse_ = false;
  }

  // Box lists, slice buffers and the inverse storage of one level.
  void prepare_boxes(Level<T>& lev, hipStream_t s) {
    const BoxGeom& g = lev.g;
    lev.d_ib.upload(lev.ib_list, s);
    lev.d_int.upload(lev.int_list, s);
    if (lev.sum_mode) {
      std::vector<int> bi((size_t)g.npd * g.npd, lev.n_ib);
      for (int i = 0; i < lev.n_ib; ++i) bi[lev.ib_list[i]] = i;
      lev.d_box_inv.upload(bi, s);
      lev.inv.alloc((size_t)lev.n_unique * box_stride(lev));
      lev.Y.alloc((size_t)g.npd * g.npd * g.nch * 64);
      return;
    }
    if (has_classes(lev)) {
      class_tables(lev);
      lev.d_kcode.upload(lev.kcode, s);
      lev.d_rcode.upload(lev.rcode, s);
      lev.d_klocal.upload(lev.klocal, s);
      lev.d_rlocal.upload(lev.rlocal, s);
      IntClassView& v = lev.clsv;
      v.K = (int)lev.kcode.size();
      v.Kp = (v.K + 127) / 128 * 128;
      v.R = (int)lev.rcode.size();
      v.nrt = (v.R + 15) / 16;
      lev.cls.alloc((size_t)4 * v.nrt * v.Kp * 16);
      v.M = lev.cls.p;
      v.kcode = lev.d_kcode.p;
      v.rcode = lev.d_rcode.p;
    }
    order_boxes(lev);
    lev.d_pos.upload(lev.pos, s);
    lev.d_nonown.upload(lev.nonown, s);
    lev.d_ord.upload(lev.ord, s);
    lev.d_own.upload(lev.own, s);
    // The IB boxes are kept eliminated (three launches over fewer
    // bytes) where the whole rows that one launch of the sweep reads (all boxes,
    // or a colour's) take at least 192 MiB.  Alone, the eliminated form breaks
    // even near 100 MiB (FP64 16 x 16/4: 42 MiB 18.3 against 10.7 us for whole
    // rows, 125 MiB 21.2 against 24.3, 1790 MiB 146 against 286; 8 x 8/2: 75 MiB
    // 20.7 against 15.9, 166 MiB 30.0 against 27.6; FP32 16 x 16/4: 62 MiB 15.9
    // against 13.9, 166 MiB 21.5 against 28.2), but its launches wait for one
    // another where the whole rows' one also covers the interior boxes: a
    // multiplicative 256^2 solve took 18.4 ms with the line at 96 MiB, 17.6 at
    // 192 and 17.7 at 320 (additive 512^2 67.4 ms at all three).  A batch's
    // launches read every member's boxes (taken as the same number each).
    const size_t l = &lev - levels_.data();
    const int per_launch = d_.smoother == IBMG_RMS ? lev.n_ib / std::max(1, lev.ncolour)
                                                   : lev.n_ib * (l < members_.size() ? members_[l] : 1);
    // An FP32 level keeps room for both forms: which one it takes follows from the
    // eliminated boxes (kElimMaxLossVel), in build_boxes.
    lev.may_sym = lev.n_ib > 0 && lev.bm.nn <= kElimMaxNn &&
                  (size_t)per_launch * box_stride(lev) * sizeof(T) >= kElimMinBytes &&
                  std::getenv("IBMG_NO_SYM") == nullptr;
    lev.use_sym = lev.may_sym;
    const size_t rows = rows_held(lev) * box_stride(lev);
    if (!lev.may_sym) {
      lev.inv.alloc(rows);
      return;
    }
    list_w_rows(lev);
    lev.d_wptr.upload(lev.wptr, s);
    lev.d_wrow.upload(lev.wrow, s);
    lev.d_coupled.upload(lev.coupled, s);
    const size_t wlen = (lev.wrow.size() * (size_t)lev.w_stride + 63) / 64 * 64;
    const size_t both = wlen + (size_t)lev.n_ib * sym_box_stride(g);
    lev.inv.alloc(sizeof(T) == 4 ? std::max(rows, both) : both);
    lev.wmat = lev.inv.p;
    lev.inv_sym = lev.inv.p + wlen;
    if (!defer_coarse_) {   // (a batch has its own for all members)
      lev.w_res.alloc((size_t)lev.n_ib * g.nown);
      lev.sym_part.alloc((size_t)lev.n_ib * sym_part_len(g));
    }
  }

  // the box matrices' order from unique box u0 on
  BoxOrder order_of(Level<T>& lev, int u0) {
    if (lev.sum_mode) return BoxOrder{};
    return BoxOrder{lev.d_pos.p, lev.d_nonown.p, lev.d_ord.p + (size_t)u0 * lev.g.nown,
                    lev.d_own.p + (size_t)u0 * lev.g.nown};
  }

  // the eliminated storage from IB box i0 on
  SymIB sym_of(Level<T>& lev, int i0) {
    if (!lev.use_sym) return SymIB{};
    return SymIB{lev.inv_sym + (size_t)i0 * sym_box_stride(lev.g), nullptr, lev.sym_part.p,
                 WBoxView{lev.wmat, nullptr, lev.d_wptr.p + i0, lev.d_wrow.p, lev.d_nonown.p,
                          lev.d_coupled.p + (size_t)i0 * lev.g.nown, lev.d_ord.p + (size_t)i0 * lev.g.nown, lev.bm.nn,
                          lev.w_stride, lev.w_max},
                 lev.w_res.p};
  }

  // The unique boxes whose rows lev.inv holds in chunks where none are eliminated:
  // the IB boxes, and the interior boxes' shared inverse where no parity classes
  // hold it.
  size_t rows_held(const Level<T>& lev) const { return has_classes(lev) ? lev.n_ib : lev.n_unique; }
  // the single-system restricted sweeps take the interior boxes in parity
  // classes; the summed combination and the batched form read whole rows
  bool has_classes(const Level<T>& lev) const { return !lev.sum_mode && !lev.int_list.empty(); }

  // Adds what the eliminated form costs `count` IB boxes from u0 on (m: their
  // matrices, eliminated) to the level's sums, and takes the level to whole rows
  // where that is too much (a NaN from a breakdown included).
  void elim_loss(Level<T>& lev, int u0, int count, const double* m, BoxMat bm, hipStream_t s) {
    const size_t nsum = (size_t)count * kLossParts * 4;
    DBuf<double> buf(nsum + (size_t)count * lev.g.nown);
    if (dry_run()) return;
    launch_elim_loss(m, count, bm, lev.g, order_of(lev, u0).ord, buf.p + nsum, buf.p, s);
    std::vector<double> h(nsum);
    IBMG_HIP(hipMemcpyAsync(h.data(), buf.p, nsum * sizeof(double), hipMemcpyDeviceToHost, s));
    IBMG_HIP(hipStreamSynchronize(s));
    if (u0 == 0) std::fill(lev.loss, lev.loss + 4, 0.0);
    for (size_t i = 0; i < nsum; ++i) lev.loss[i % 4] += h[i];
    lev.use_sym = lev.loss[0] <= kElimMaxLossVel * lev.loss[1] && lev.loss[2] <= kElimMaxLossPre * lev.loss[3];
  }

  // The unique box inverses of every Schwarz level: assembled per level,
  // eliminated (or, for the summed combination, inverted) in batches that mix
  // levels whose boxes have the same number of unknowns (one run of sweeps
  // serves them all), each level's storage extracted.  Batches hold at most
  // 512 matrices and 10 GiB of them with their sweep workspace (a set-up
  // temporary of the handle's workspace), split evenly.
  void build_boxes(hipStream_t s) {
    std::map<std::pair<int, int>, std::vector<std::pair<int, int>>> groups;   // (size, nnp) -> (level, unique index)
    std::vector<DBuf<int>> ids(L_ + 1);
    for (int l = 1; l <= L_; ++l) {
      Level<T>& lev = levels_[l];
      prepare_boxes(lev, s);
      ids[l].upload(lev.uniq, s);
      for (int u = 0; u < lev.n_unique; ++u) groups[{lev.bm.ld, lev.bm.nnp}].push_back({l, u});
    }
    const size_t budget = (size_t)10 << 30;
    for (auto& grp : groups) {
      const int n = grp.first.first;
      const auto& items = grp.second;
      const BoxMat bm = levels_[items[0].first].bm;   // one box shape per group
      const size_t per = ((size_t)n * n + sweep_work(n, 1)) * sizeof(double);
      const size_t cap = std::min<size_t>(std::max<size_t>(1, budget / per), 512);
      const size_t nbatch = (items.size() + cap - 1) / cap;
      const int batch = (int)((items.size() + nbatch - 1) / nbatch);
      DBuf<double> mats((size_t)batch * n * n), work(sweep_work(n, batch));
      for (size_t b0 = 0; b0 < items.size();) {
        const int cnt = (int)std::min<size_t>(batch, items.size() - b0);
        // runs of one level with consecutive unique indices
        auto for_runs = [&](auto fn) {
          size_t i = b0;
          while (i < b0 + cnt) {
            size_t j = i + 1;
            while (j < b0 + cnt && items[j].first == items[i].first && items[j].second == items[j - 1].second + 1) ++j;
            fn(items[i].first, items[i].second, (int)(j - i), i - b0);
            i = j;
          }
        };
        for_runs([&](int l, int u0, int count, size_t slot) {
          Level<T>& lev = levels_[l];
          launch_patch_assemble(ids[l].p + u0, count, lev.g, lev.cd, lev.f[0].d_tptr.p, lev.f[0].d_tcol.p,
                                lev.f[0].tval.p, lev.f[1].d_tptr.p, lev.f[1].d_tcol.p, lev.f[1].tval.p,
                                order_of(lev, u0), bm, mats.p + slot * n * n, s);
        });
        if (bm.nnp) launch_box_eliminate(mats.p, bm, cnt, work.p, s);
        else launch_gj_invert(mats.p, n, cnt, work.p, s);
        // (boxes that an earlier batch put down in the other form come again)
        bool again = false;
        if (sizeof(T) == 4)
          for_runs([&](int l, int u0, int count, size_t slot) {
            Level<T>& lev = levels_[l];
            if (!lev.use_sym || u0 >= lev.n_ib) return;
            elim_loss(lev, u0, std::min(count, lev.n_ib - u0), mats.p + slot * n * n, bm, s);
            again = again || (!lev.use_sym && u0 > 0);
          });
        if (again) {
          b0 = 0;
          continue;
        }
        for_runs([&](int l, int u0, int count, size_t slot) {
          Level<T>& lev = levels_[l];
          double* m0 = mats.p + slot * n * n;
          // unique indices below n_ib are the IB boxes; the eliminated ones
          // come apart into their two factors, the others and the interior
          // representative (the last) get whole rows
          const int nsym = lev.use_sym ? std::min(count, std::max(0, lev.n_ib - u0)) : 0;
          if (bm.nnp) launch_box_on(m0 + (size_t)nsym * n * n, bm, count - nsym, s);
          const int c1 = std::min(u0 + count, (int)rows_held(lev));
          if (!lev.use_sym && c1 > u0)
            launch_extract_rows<T>(m0, c1 - u0, lev.g, bm, order_of(lev, u0), lev.inv.p + (size_t)u0 * box_stride(lev),
                                   s);
          if (has_classes(lev) && u0 + count > lev.n_ib)
            launch_extract_classes<T>(m0 + (size_t)(lev.n_ib - u0) * n * n, bm,
                                      lev.d_own.p + (size_t)lev.n_ib * lev.g.nown, lev.clsv, lev.d_klocal.p,
                                      lev.d_rlocal.p, lev.cls.p, s);
          if (nsym > 0) {
            launch_extract_sym<T>(m0, nsym, lev.g, bm, lev.inv_sym + (size_t)u0 * sym_box_stride(lev.g), s);
            launch_extract_w<T>(m0, nsym, bm, lev.d_wptr.p + u0, lev.d_wrow.p, lev.w_stride, lev.wmat, s);
          }
        });
        b0 += batch;
      }
      IBMG_HIP(hipStreamSynchronize(s));
    }
  }

  void alloc_work(hipStream_t s) {
    (void)s;
    for (int l = 0; l <= L_; ++l) {
      Level<T>& lev = levels_[l];
      const size_t n = 3 * (size_t)lev.N * lev.N;
      lev.w.alloc(n);
      lev.b.alloc(n);
      lev.r.alloc(n);
      lev.t.alloc(n);
      if (l >= 1) {
        lev.V.alloc((size_t)(nu_ + 1) * n);
        lev.Z.alloc((size_t)nu_ * n);
      }
      lev.F.alloc(4 * (size_t)std::max(M_, 1));   // forces [2][M] then J u [2][M]
      if (l >= 1 && d_.smoother == IBMG_RMS) lev.rr.alloc(n);
      lev.scal.alloc(kGsScal);
      lev.part.alloc(3 * part_stride(lev));
    }
  }

  // --------------------------------------------------------------- views
  template <typename U>
  FootView<U> fview(CompFoot& f) {
    if constexpr (std::is_same<U, double>::value)
      return FootView<double>{f.d_base.p, f.w.p, f.d_sp_ptr.p, f.d_sp_ent.p, f.sw.p, d_order_.p, f.d_obase.p,
                              f.ow.p};
    else
      return FootView<float>{f.d_base.p, f.wf.p, f.d_sp_ptr.p, f.d_sp_ent.p, f.swf.p, d_order_.p, f.d_obase.p,
                             f.owf.p};
  }
  template <typename U>
  SpringView<U> sview() {
    if constexpr (std::is_same<U, double>::value)
      return SpringView<double>{M_, d_adj_ptr_.p, d_adj_nbr_.p, d_adj_k_.p, tangent_ ? d_adj_k2_.p : nullptr};
    else
      return SpringView<float>{M_, d_adj_ptr_.p, d_adj_nbr_.p, d_adj_kf_.p, tangent_ ? d_adj_k2f_.p : nullptr};
  }
  template <typename U>
  StokesCoef<U> coef(Level<T>& lev) {
    if constexpr (std::is_same<U, double>::value) return lev.cd;
    else return StokesCoef<float>{(float)lev.cd.alpha, (float)lev.cd.beta, (float)lev.cd.gi, (float)lev.cd.ibs};
  }

  // the level's explicit IB rows, or its nodal forces K' J x formed in F (Fp)
  template <typename U>
  IbRows<U> ib_source(Level<T>& lev, const U* x, U* F, const U** Fp, hipStream_t s) {
    *Fp = nullptr;
    if (lev.ib_lanes)
      return IbRows<U>{lev.d_ib_rows.p, lev.d_ib_flag.p, csr<U>(lev.f[0]), csr<U>(lev.f[1]), (int)lev.ib_rows.size(),
                       lev.ib_lanes};
    if (M_ > 0 && E_ > 0) {
      const size_t nn = (size_t)lev.N * lev.N;
      launch_ib_force<U>(x, x + nn, fview<U>(lev.f[0]), fview<U>(lev.f[1]), sview<U>(), lev.N,
                         F + 2 * (size_t)std::max(M_, 1), F, s);
      *Fp = F;
    }
    return IbRows<U>{};
  }

  // y = L_IB^l x (b != null: y = b - L_IB^l x)
  template <typename U>
  void op(int l, const U* x, U* y, const U* b, bool trans, U* F, hipStream_t s) {
    Level<T>& lev = levels_[l];
    const U* Fp;
    const IbRows<U> R = ib_source<U>(lev, x, F, &Fp, s);
    launch_apply<U>(x, y, b, Fp, R, fview<U>(lev.f[0]), fview<U>(lev.f[1]), lev.N, M_, coef<U>(lev), trans, s);
  }

  // y = L_IB^l x with the first Gram-Schmidt pass fused into the operator
  // kernel: partial holds dot_blocks(lev) blocks of the dots u_q . y, q < nvec
  // (u_0 = u0, u_q = V + q vstride; with nvec = 1 also u_0 . u_0)
  template <typename U>
  void op_dots(int l, const U* x, U* y, const U* u0, const U* V, int nvec, size_t vstride, double* partial, U* F,
               hipStream_t s) {
    Level<T>& lev = levels_[l];
    const U* Fp;
    const IbRows<U> R = ib_source<U>(lev, x, F, &Fp, s);
    launch_apply_dots<U>(x, y, Fp, R, fview<U>(lev.f[0]), fview<U>(lev.f[1]), lev.N, M_, coef<U>(lev), u0, V, nvec,
                         vstride, partial, s);
  }

  template <typename U>
  CsrT<U> csr(CompFoot& f) {
    if constexpr (std::is_same<U, double>::value)
      return CsrT<double>{f.d_tptr.p, f.d_tcol.p, f.tval.p};
    else
      return CsrT<float>{f.d_tptr.p, f.d_tcol.p, f.tvalf.p};
  }
  // ------------------------------------------------------- V-cycle pieces
  void basic_smoother(int l, const T* v, T* z, hipStream_t s) {
    Level<T>& lev = levels_[l];
    if (lev.sc) {
      lev.sc->apply(v, z, s);
      return;
    }
    if (lev.sum_mode) {
      launch_asm_apply<T>(v, z, lev.g, lev.inv.p, lev.d_box_inv.p, lev.Y.p, s);
      return;
    }
    if (d_.smoother == IBMG_RMS) {
      // Alg. 3 colour by colour from z = 0: each colour's boxes add their
      // restricted local solutions of the residual of the current z
      launch_fill<T>(z, T(0), 3 * (size_t)lev.N * lev.N, s);
      for (int c = 0; c < lev.ncolour; ++c) {
        const T* rc = v;
        if (c > 0) {
          op<T>(l, z, lev.rr.p, v, false, lev.F.p, s);
          rc = lev.rr.p;
        }
        ras_launch(lev, rc, z, lev.ib_off[c], lev.ib_off[c + 1], lev.int_off[c], lev.int_off[c + 1], s, 3, true);
      }
      return;
    }
    ras_launch(lev, v, z, 0, lev.n_ib, 0, (int)lev.int_list.size(), s, 3, false);
  }

  // w <- w + e, e = nu FGMRES iterations (classical Gram-Schmidt twice) on
  // L e = b - L w from e = 0, on an unnormalised basis (krylov_kernels.hip).
  // With w_zero, w is not read (the result is stored into it); crs != null
  // (w_zero only) also leaves the restriction of b - L w there, by the Arnoldi
  // relation, and the return value says whether it did (the Richardson steps do
  // not).
  bool smooth_t(int l, T* w, const T* b, int nu, bool w_zero, hipStream_t s, T* crs = nullptr) {
    Level<T>& lev = levels_[l];
    const size_t n = 3 * (size_t)lev.N * lev.N;
    if (d_.sweep_kind == IBMG_SWEEP_RICHARDSON) {
      // nu undamped Richardson steps w <- w + B (b - L w); from w = 0 the
      // first step is w = B b
      for (int k = 0; k < nu; ++k) {
        if (k == 0 && w_zero) {
          basic_smoother(l, b, w, s);
          continue;
        }
        op<T>(l, w, lev.r.p, b, false, lev.F.p, s);
        basic_smoother(l, lev.r.p, lev.t.p, s);
        launch_axpy<T>(w, lev.t.p, n, s);
      }
      return false;
    }
    T* V = lev.V.p;
    T* Z = lev.Z.p;
    const T* u0 = b;
    if (!w_zero) {
      op<T>(l, w, V, b, false, lev.F.p, s);
      u0 = V;
    }
    double* pd = lev.part.p;
    double* pu[2] = {lev.part.p + part_stride(lev), lev.part.p + 2 * part_stride(lev)};
    const int nd = dot_blocks(lev);
    for (int k = 0; k < nu; ++k) {
      const T* uk = k == 0 ? u0 : V + (size_t)k * n;
      T* zk = Z + (size_t)k * n;
      T* t = V + (size_t)(k + 1) * n;
      basic_smoother(l, uk, zk, s);
      op_dots<T>(l, zk, t, u0, V, k + 1, n, pd, lev.F.p, s);
      launch_gs_update<T>(t, u0, V, k + 1, n, n, pd, nd, pu[(k + 1) & 1], lev.scal.p, pu[k & 1], s);
    }
    const double* pl = pu[(nu - 1) & 1];
    if (crs) launch_gs_combine_restrict<T>(w, Z, u0, V, nu, n, lev.N / 2, pl, lev.scal.p, crs, s);
    else launch_gs_combine<T>(w, Z, nu, n, n, pl, lev.scal.p, w_zero, s);
    return crs != nullptr;
  }

  // Classical Gram-Schmidt twice against V[0..k) for the outer solve's long
  // vectors: h (first pass + second pass) into hcol[0..k), the partial sums of
  // |t|^2 left in opart_ for launch_scale_red.  On up to kOuterBlocks blocks:
  // beyond kFoldBlocks of them one block folds each pass's partial sums (the
  // pass-1 dots, then the pass-2 dots) before the next kernel, so that kernel's
  // blocks read k values instead of every block's k partials.
  void orthogonalise_outer(const double* V, int k, size_t n, double* t, double* hcol, int nblk, hipStream_t s) {
    double* pa = opart_.p;
    double* pb = opart_.p + kOuterPartStride;
    const bool fold = nblk > kFoldBlocks;
    launch_dots<double>(V, k, n, t, n, pa, nblk, s);
    if (fold) launch_dots_finish(pa, k, nblk, ofold_.p, nullptr, 0, s);
    launch_upd_dots<double>(t, V, k, n, n, fold ? ofold_.p : pa, nblk, hcol, pb, s, fold ? 1 : nblk);
    if (fold) launch_dots_finish(pb, k, nblk, ofold_.p + 72, nullptr, 0, s);
    launch_upd_norm<double>(t, V, k, n, n, fold ? ofold_.p + 72 : pb, nblk, hcol, pa, s, fold ? 1 : nblk);
  }

  // w = MG(0, b) on level l (Alg. 1)
  void mg(int l, const T* b, T* w, hipStream_t s) {
    if (l == 0) {
      launch_coarse_apply<T>(inv0_.p, n0_, b, w, s);
      return;
    }
    Level<T>& lev = levels_[l];
    Level<T>& crs = levels_[l - 1];
    if (!smooth_t(l, w, b, d_.nu1, true, s, d_.nu1 <= kArnoldiResidualNu ? crs.b.p : nullptr)) {
      op<T>(l, w, lev.r.p, b, false, lev.F.p, s);
      launch_restrict<T>(lev.r.p, crs.b.p, crs.N, s);
    }
    mg(l - 1, crs.b.p, crs.w.p, s);
    launch_prolong_add<T>(crs.w.p, w, crs.N, s);
    smooth_t(l, w, b, d_.nu2, false, s);
  }

  // ------------------------------------------------------------ ABI calls
  void apply(int level, const double* w, double* y, bool trans, hipStream_t s) override {
    op<double>(level, w, y, nullptr, trans, Fd_.p, s);
  }

  void spread(const double* F, double* f, hipStream_t s) override {
    Level<T>& lev = levels_[L_];
    const double h = 1.0 / lev.N;
    launch_spread(F, fview<double>(lev.f[0]), fview<double>(lev.f[1]), M_, lev.N, 1.0 / (h * h), f, s);
  }

  void interp(const double* u, double* U, hipStream_t s) override {
    Level<T>& lev = levels_[L_];
    launch_interp<double>(u, u + (size_t)lev.N * lev.N, fview<double>(lev.f[0]), fview<double>(lev.f[1]),
                          M_, lev.N, U, s);
  }

  void restrict_(int level, const double* fine, double* coarse, hipStream_t s) override {
    launch_restrict<double>(fine, coarse, levels_[level - 1].N, s);
  }

  void prolong_add(int level, const double* coarse, double* fine, hipStream_t s) override {
    launch_prolong_add<double>(coarse, fine, levels_[level - 1].N, s);
  }

  void smoother_apply(int level, const double* r, double* z, hipStream_t s) override {
    Level<T>& lev = levels_[level];
    const size_t n = 3 * (size_t)lev.N * lev.N;
    if constexpr (std::is_same<T, double>::value) {
      basic_smoother(level, r, z, s);
    } else {
      launch_cast<double, T>(r, lev.r.p, n, s);
      basic_smoother(level, lev.r.p, lev.t.p, s);
      launch_cast<T, double>(lev.t.p, z, n, s);
    }
  }

  void smooth(int level, double* w, const double* b, int nu, hipStream_t s) override {
    require(nu >= 1 && nu <= nu_, "nu must lie in [1, max(nu1, nu2)]");
    Level<T>& lev = levels_[level];
    const size_t n = 3 * (size_t)lev.N * lev.N;
    if constexpr (std::is_same<T, double>::value) {
      smooth_t(level, w, b, nu, false, s);
    } else {
      launch_cast<double, T>(w, lev.w.p, n, s);
      launch_cast<double, T>(b, lev.b.p, n, s);
      smooth_t(level, lev.w.p, lev.b.p, nu, false, s);
      launch_cast<T, double>(lev.w.p, w, n, s);
    }
  }

  void coarse_solve(const double* r, double* x, hipStream_t s) override {
    launch_coarse_apply<double>(inv0_.p, n0_, r, x, s);
  }

  void vcycle_body(const double* r, double* z, hipStream_t s) {
    Level<T>& top = levels_[L_];
    const size_t n = 3 * (size_t)top.N * top.N;
    if constexpr (std::is_same<T, double>::value) {
      mg(L_, r, z, s);
    } else {
      launch_cast<double, T>(r, top.b.p, n, s);
      mg(L_, top.b.p, top.w.p, s);
      launch_cast<T, double>(top.w.p, z, n, s);
    }
  }

  // The whole V-cycle (several hundred launches, no host synchronisation)
  // is captured once into a HIP graph reading vin_ and writing vout_, then
  // replayed; the graph holds kernel nodes only.
  void build_graph() {
    if (!gstream_) IBMG_HIP(hipStreamCreateWithFlags(&gstream_, hipStreamNonBlocking));
    IBMG_HIP(hipStreamBeginCapture(gstream_, hipStreamCaptureModeThreadLocal));
    try {
      vcycle_body(vin_.p, vout_.p, gstream_);
    } catch (...) {
      hipGraph_t g = nullptr;
      (void)hipStreamEndCapture(gstream_, &g);
      if (g) (void)hipGraphDestroy(g);
      throw;
    }
    IBMG_HIP(hipStreamEndCapture(gstream_, &graph_));
    IBMG_HIP(hipGraphInstantiate(&gexec_, graph_, nullptr, nullptr, 0));
  }

  void drop_graph() {
    if (gexec_) (void)hipGraphExecDestroy(gexec_);
    if (graph_) (void)hipGraphDestroy(graph_);
    gexec_ = nullptr;
    graph_ = nullptr;
  }

  void vcycle(const double* r, double* z, hipStream_t s) override {
    if (!use_graph_) {
      vcycle_body(r, z, s);
      return;
    }
    const size_t n = 3 * (size_t)d_.N * d_.N;
    IBMG_HIP(hipMemcpyAsync(vin_.p, r, n * sizeof(double), hipMemcpyDeviceToDevice, s));
    replay(s);
    IBMG_HIP(hipMemcpyAsync(z, vout_.p, n * sizeof(double), hipMemcpyDeviceToDevice, s));
  }

  // the captured V-cycle, from vin_ to vout_
  void replay(hipStream_t s) {
    if (!gexec_) build_graph();
    IBMG_HIP(hipGraphLaunch(gexec_, s));
  }

  double read_scalar(const double* dptr, hipStream_t s) {
    IBMG_HIP(hipMemcpyAsync(pinned_, dptr, sizeof(double), hipMemcpyDeviceToHost, s));
    IBMG_HIP(hipStreamSynchronize(s));
    return pinned_[0];
  }

  void project(double* a, hipStream_t s) {
    Level<T>& top = levels_[L_];
    launch_block_sums<double>(a, top.N, opart_.p, 64, s);
    launch_dots_finish(opart_.p, 3, 64, osc_.p + 8, nullptr, 0, s);
    launch_subtract_means<double>(a, top.N, osc_.p + 8, d_.rho == 0.0 ? 1 : 0, s);
  }

  double norm(const double* a, size_t n, hipStream_t s) {
    const int nblk = dots_blocks(n);
    launch_dots<double>(a, 1, n, a, n, opart_.p, nblk, s);
    launch_dots_finish(opart_.p, 1, nblk, osc_.p + 0, nullptr, 2, s);
    return read_scalar(osc_.p + 0, s);
  }

  int fgmres(const double* b, double* x, const ibmg_solve_opts& o, ibmg_solve_info* info,
             hipStream_t s) override {
    const auto t0 = std::chrono::steady_clock::now();
    require(o.restart >= 1 && o.restart <= outer_cap_,
            "restart must lie in [1, max_restart = " + std::to_string(outer_cap_) + "]");
    require(o.max_it >= 1, "max_it must be >= 1");
    require(std::isfinite(o.rtol) && o.rtol > 0.0, "rtol must be finite and > 0");
    // the adjoint system uses the transposed operator path; L_IB is
    // symmetric, so the same V-cycle preconditions it
    const bool trans = o.transpose != 0;
    const int N = d_.N;
    const size_t n = 3 * (size_t)N * N;
    const int gs_nblk = dots_blocks(n, kOuterBlocks);
    const int ldh = o.restart + 1;
    int hist_n = 0;
    auto push_hist = [&](double v) {
      if (info && info->history && hist_n < info->history_cap) info->history[hist_n] = v;
      ++hist_n;
    };
    // projected right-hand side and the removed null-space part
    IBMG_HIP(hipMemcpyAsync(bp_.p, b, n * sizeof(double), hipMemcpyDeviceToDevice, s));
    project(bp_.p, s);
    IBMG_HIP(hipMemcpyAsync(pinned_, osc_.p + 8, 3 * sizeof(double), hipMemcpyDeviceToHost, s));
    IBMG_HIP(hipStreamSynchronize(s));
    const double nn = (double)N * N;
    double null2 = pinned_[2] * pinned_[2] / nn;
    if (d_.rho == 0.0) null2 += (pinned_[0] * pinned_[0] + pinned_[1] * pinned_[1]) / nn;
    const double bnorm = norm(bp_.p, n, s);
    if (info) {
      info->iters = 0;
      info->restarts = 0;
      info->rhs_null_norm = std::sqrt(null2);
      info->setup_ms = setup_ms_;
      info->vcycles = 0;
    }
    if (!std::isfinite(bnorm) || !std::isfinite(null2)) throw Error(IBMG_ERR_NONFINITE, "right-hand side holds NaN/Inf");
    if (!o.use_x0) launch_fill<double>(x, 0.0, n, s);
    if (bnorm == 0.0) {
      launch_fill<double>(x, 0.0, n, s);
      IBMG_HIP(hipStreamSynchronize(s));
      if (info) {
        info->rel_res_est = info->rel_res_true = 0.0;
        info->solve_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
      }
      return IBMG_OK;
    }
    const double target = o.rtol * bnorm;
    int its = 0, restarts = 0, vcycles = 0;
    bool converged = false;
    double est = bnorm, prev_est = 0.0;
    if (!est_ev_) IBMG_HIP(hipEventCreateWithFlags(&est_ev_, hipEventDisableTiming));
    while (its < o.max_it) {
      double* V0 = Vo_.p;
      op<double>(L_, x, V0, bp_.p, trans, Fd_.p, s);
      const double beta = norm(V0, n, s);
      if (!std::isfinite(beta)) throw Error(IBMG_ERR_NONFINITE, "residual is not finite");
      est = beta;
      if (beta <= target) { converged = true; break; }
      launch_scale<double>(V0, V0, osc_.p + 0, n, s);
      launch_fill<double>(g_.p, 0.0, (size_t)o.restart + 2, s);
      IBMG_HIP(hipMemcpyAsync(g_.p, osc_.p + 0, sizeof(double), hipMemcpyDeviceToDevice, s));
      // Replays read vin_ and write vout_: the operator takes z_k from vout_,
      // and the launch that normalises the next basis vector also stores it to
      // vin_ and z_k to its column (two copies fewer an iteration)
      if (use_graph_) IBMG_HIP(hipMemcpyAsync(vin_.p, V0, n * sizeof(double), hipMemcpyDeviceToDevice, s));
      auto precondition = [&](const double* v, double* z) {
        if (use_graph_) replay(s);
        else vcycle_body(v, z, s);
      };
      int k = 0;
      bool queued = false;   // z_k's V-cycle already queued by the previous iteration
      for (; k < o.restart && its < o.max_it;) {
        double* vk = Vo_.p + (size_t)k * n;
        double* zk = Zo_.p + (size_t)k * n;
        double* t = Vo_.p + (size_t)(k + 1) * n;
        if (!queued) precondition(vk, zk);
        queued = false;
        ++vcycles;
        op<double>(L_, use_graph_ ? vout_.p : zk, t, nullptr, trans, Fd_.p, s);
        double* hcol = Ho_.p + (size_t)k * ldh;
        orthogonalise_outer(Vo_.p, k + 1, n, t, hcol, gs_nblk, s);
        launch_scale_red<double>(t, t, n, opart_.p, gs_nblk, hcol + k + 1, s,
                                 use_graph_ ? ScaleCopies<double>{vin_.p, vout_.p, zk} : ScaleCopies<double>{});
        launch_givens(Ho_.p, ldh, k, cs_.p, sn_.p, g_.p, osc_.p + 1, s);
        // The estimate is read on the host after this iteration's work.
        // While the last two estimates say that even one more step at their
        // rate would stay above the target, the next iteration's V-cycle
        // (its input, the normalised t, is already queued) is queued before
        // the host waits, so the device does not idle through the read.  A
        // wrong guess leaves one unused V-cycle behind the solve's tail; it
        // is not counted in vcycles.
        IBMG_HIP(hipMemcpyAsync(pinned_, osc_.p + 1, sizeof(double), hipMemcpyDeviceToHost, s));
        IBMG_HIP(hipEventRecord(est_ev_, s));
        const double rate = prev_est > 0.0 ? std::min(1.0, est / prev_est) : 1.0;
        if (k + 1 < o.restart && its + 1 < o.max_it && its >= 2 && est * rate * rate > target) {
          precondition(t, Zo_.p + (size_t)(k + 1) * n);
          queued = true;
        }
        IBMG_HIP(hipEventSynchronize(est_ev_));
        prev_est = est;
        est = pinned_[0];
        ++k;
        ++its;
        push_hist(est / bnorm);
        if (!std::isfinite(est)) throw Error(IBMG_ERR_NONFINITE, "iteration produced NaN/Inf");
        if (est <= target) { converged = true; break; }
      }
      launch_backsolve(Ho_.p, ldh, k, g_.p, y_.p, s);
      launch_combine<double>(x, Zo_.p, k, n, y_.p, n, s);
      ++restarts;
      if (converged) break;
    }
    project(x, s);
    op<double>(L_, x, rr_.p, bp_.p, trans, Fd_.p, s);
    const double tr = norm(rr_.p, n, s);
    if (info) {
      info->iters = its;
      info->restarts = restarts;
      info->rel_res_est = est / bnorm;
      info->rel_res_true = tr / bnorm;
      info->vcycles = vcycles;
      info->solve_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    }
    if (!std::isfinite(tr)) throw Error(IBMG_ERR_NONFINITE, "solution is not finite");
    return converged ? IBMG_OK : IBMG_NOT_CONVERGED;
  }

  void spring_gradient(const double* w, const double* lam, double* out, hipStream_t s) override {
    spring_gradient_in(w, lam, out, Uw_.p, Ul_.p, s);
  }

  void spring_gradient_in(const double* w, const double* lam, double* out, double* Uw, double* Ul,
                          hipStream_t s) override {
    Level<T>& lev = levels_[L_];
    const size_t nn = (size_t)lev.N * lev.N;
    const double h = 1.0 / lev.N;
    launch_interp<double>(w, w + nn, fview<double>(lev.f[0]), fview<double>(lev.f[1]), M_, lev.N, Uw, s);
    launch_interp<double>(lam, lam + nn, fview<double>(lev.f[0]), fview<double>(lev.f[1]), M_, lev.N, Ul, s);
    launch_spring_grad(Uw, Ul, d_ends_.p, tangent_ ? d_gblocks_.p : nullptr, E_, -d_.dt / (h * h), out, s);
  }

  int points() const override { return M_; }

  void set_kappa(const double* kappa, hipStream_t s) override {
    require(E_ == 0 || kappa != nullptr, "kappa is NULL");
    for (int e = 0; e < E_; ++e)
      require(std::isfinite(kappa[e]) && kappa[e] >= 0.0, "kappa must be finite and >= 0");
    kappa_.assign(kappa, kappa + E_);
    rebuild(s);
  }

  // ------------------------------------------- semi-implicit time step
  // rhs = [(rho/dt) u + S_h F(X); 0] on the finest grid (Eq. matrix-impib),
  // F the nodal spring forces (K_h X for the linear model)
  void step_rhs(const double* w, double* rhs, hipStream_t s) override {
    Level<T>& lev = levels_[L_];
    const double h = 1.0 / lev.N;
    const size_t m2 = 2 * (size_t)std::max(M_, 1);
    launch_fill<double>(Fs_.p, 0.0, m2, s);
    launch_fibre_force(d_X_.p, sview<double>(), tangent_ ? d_adj_kap_.p : d_adj_k_.p,
                       tangent_ ? d_adj_rest_.p : nullptr, Fs_.p, s);
    launch_spread(Fs_.p, fview<double>(lev.f[0]), fview<double>(lev.f[1]), M_, lev.N, 1.0 / (h * h), fs_.p, s);
    launch_step_rhs(w, fs_.p, d_.rho / d_.dt, lev.N, rhs, s);
  }

  // Solve L_IB(X^n) w^{n+1} = rhs, advance X^{n+1} = X^n + dt J_h u^{n+1}
  // (Eq. imp-X-new, wrapped into [0, 1)) and rebuild every level at X^{n+1}.
  int time_step(double* w, const ibmg_solve_opts& o, ibmg_solve_info* info, hipStream_t s) override {
    Level<T>& lev = levels_[L_];
    const size_t nn = (size_t)lev.N * lev.N;
    step_rhs(w, rhs_.p, s);
    const int st = fgmres(rhs_.p, w, o, info, s);
    launch_interp<double>(w, w + nn, fview<double>(lev.f[0]), fview<double>(lev.f[1]), M_, lev.N, Uw_.p, s);
    launch_advance(d_X_.p, Uw_.p, d_.dt, M_, s);
    if (M_ > 0)
      IBMG_HIP(hipMemcpyAsync(X_.data(), d_X_.p, 2 * (size_t)M_ * sizeof(double), hipMemcpyDeviceToHost, s));
    IBMG_HIP(hipStreamSynchronize(s));
    for (double x : X_)
      if (!std::isfinite(x) || x < 0.0 || x >= 1.0) throw Error(IBMG_ERR_NONFINITE, "updated positions are invalid");
    rebuild(s);
    if (info) info->setup_ms = setup_ms_;
    return st;
  }

  // Every level rebuilt for the current positions X_ (host copy) and
  // stiffnesses, laid out again above the fixed buffers.  If the rebuild
  // fails part-way (a workspace too small for the new layout), the handle
  // stays unusable.
  void rebuild(hipStream_t s) {
    drop_graph();
    valid_ = false;
    release_dependent();
    build_all(s);
    valid_ = true;
  }

  bool valid() const override { return valid_; }

  void positions(double* X) const override {
    std::copy(X_.begin(), X_.end(), X);
  }

  void sc_info(int level, double* lam, int32_t* colours) const override {
    require(level >= 1 && level <= L_, "level out of range");
    const Level<T>& lev = levels_[level];
    require(lev.sc != nullptr, "the handle does not use the Schur-complement smoother");
    lam[0] = lev.sc->lamA;
    lam[1] = lev.sc->lamM;
    colours[0] = lev.sc->colu.ncol;
    colours[1] = lev.sc->colp.ncol;
  }

  // One kernel of level `level`, launched alone on the level's work vectors
  // (filled with ones): IB-box Schwarz (k_ras_rows, or k_ras_w and its
  // followers), interior-box Schwarz (k_ras_rows) or the stencil k_apply.  Algorithmic work per launch: every IB
  // box streams its owned rows of the inverse (nown x nloc), gathers nloc
  // values and writes nown; the interior product reads the class matrices once
  // and each box's nloc values and writes nown, four R x K products per box;
  // the stencil reads and writes the three fields once.
  double kernel_time(int kernel, int level, int reps, hipStream_t s, double* bytes, double* flops) override {
    require(level >= 0 && level <= L_, "level out of range");
    require(reps >= 1 && reps <= 100000, "reps must lie in [1, 100000]");
    Level<T>& lev = levels_[level];
    const size_t n = 3 * (size_t)lev.N * lev.N;
    const double ts = sizeof(T);
    launch_fill<T>(lev.r.p, T(1), n, s);
    launch_fill<T>(lev.t.p, T(0), n, s);
    double by = 0, fl = 0, ms = 0;
    const BoxGeom& g = lev.g;
    if (kernel == IBMG_KERNEL_RAS_IB || kernel == IBMG_KERNEL_RAS_INTERIOR) {
      require(level >= 1 && !lev.sc, "Schwarz kernels need a Schwarz smoother level >= 1");
      require(!lev.sum_mode, "the restricted Schwarz kernels do not run with the summed combination");
      const int n_int = (int)lev.int_list.size();
      if (kernel == IBMG_KERNEL_RAS_IB) {
        require(lev.n_ib > 0, "the level has no IB boxes");
        // the eliminated boxes (as the additive sweep runs them, three
        // launches) stream their two factors
        const double stored = lev.use_sym ? (double)lev.n_ib * sym_box_stride(g) + (double)lev.wrow.size() * lev.bm.nn
                                          : (double)lev.n_ib * g.nown * g.nloc;
        by = (stored + (double)lev.n_ib * (g.nloc + g.nown)) * ts;
        fl = lev.use_sym ? 2.0 * ((double)lev.n_ib * g.nown * g.nown + (double)lev.wrow.size() * lev.bm.nn)
                         : 2.0 * lev.n_ib * g.nown * g.nloc;
      } else {
        require(n_int > 0, "the level has no interior boxes");
        by = ((double)lev.cls.n + (double)n_int * (g.nloc + g.nown)) * ts;
        fl = 2.0 * n_int * 4.0 * lev.clsv.R * lev.clsv.K;
      }
      const int part = kernel == IBMG_KERNEL_RAS_IB ? 1 : 2;
      ms = time_launches([&] {
        ras_launch(lev, lev.r.p, lev.t.p, 0, lev.n_ib, 0, n_int, s, part, false);
      }, reps, s);
    } else if (kernel == IBMG_KERNEL_STENCIL) {
      by = 2.0 * (double)n * ts;
      fl = 0;
      ms = time_launches([&] {
        launch_apply<T>(lev.r.p, lev.t.p, nullptr, nullptr, IbRows<T>{}, fview<T>(lev.f[0]), fview<T>(lev.f[1]), lev.N,
                        M_, coef<T>(lev), false, s);
      }, reps, s);
    } else if (kernel == IBMG_KERNEL_RESTRICT || kernel == IBMG_KERNEL_PROLONG) {
      require(level >= 1, "transfers need a level >= 1");
      Level<T>& cl = levels_[level - 1];
      const size_t nc = 3 * (size_t)cl.N * cl.N;
      if (kernel == IBMG_KERNEL_RESTRICT) {
        by = (double)(n + nc) * ts;
        ms = time_launches([&] { launch_restrict<T>(lev.r.p, cl.t.p, cl.N, s); }, reps, s);
      } else {
        by = (double)(nc + 2 * n) * ts;
        launch_fill<T>(cl.r.p, T(1), nc, s);
        ms = time_launches([&] { launch_prolong_add<T>(cl.r.p, lev.t.p, cl.N, s); }, reps, s);
      }
    } else if (kernel == IBMG_KERNEL_SPREAD || kernel == IBMG_KERNEL_INTERP) {
      require(level == L_, "spreading and interpolation run on the finest level");
      require(M_ > 0, "the structure has no points");
      const size_t nn = (size_t)lev.N * lev.N;
      launch_fill<double>(fs_.p, 1.0, 2 * nn, s);
      launch_fill<double>(Fd_.p, 1.0, 2 * (size_t)M_, s);
      size_t ents = 0, touched = 0;
      for (int c = 0; c < 2; ++c) {
        ents += lev.f[c].sp_ent.size();
        for (size_t r = 0; r < nn; ++r) touched += lev.f[c].sp_ptr[r + 1] > lev.f[c].sp_ptr[r];
      }
      const double h = 1.0 / lev.N;
      if (kernel == IBMG_KERNEL_SPREAD) {
        by = (double)ents * 12.0 + (double)(2 * (nn + 1)) * 4.0 + 2.0 * M_ * 8.0 + 2.0 * nn * 8.0;
        ms = time_launches([&] {
          launch_spread(Fd_.p, fview<double>(lev.f[0]), fview<double>(lev.f[1]), M_, lev.N, 1.0 / (h * h), fs_.p, s);
        }, reps, s);
      } else {
        by = 2.0 * M_ * 16 * 8.0 + 2.0 * M_ * 2 * 4.0 + (double)touched * 8.0 + 2.0 * M_ * 8.0;
        ms = time_launches([&] {
          launch_interp<double>(fs_.p, fs_.p + nn, fview<double>(lev.f[0]), fview<double>(lev.f[1]), M_, lev.N,
                                Uw_.p, s);
        }, reps, s);
      }
    } else if (kernel >= IBMG_KERNEL_APPLY_DOTS && kernel <= IBMG_KERNEL_SCALE_UPD) {
      // one smoothing step's Krylov kernels with the basis at its largest
      // (k = nu vectors), and the kernels of a normalised basis (the outer
      // solve's, and k_scale_upd): zero dots leave t as it is and unit
      // norms keep the small algebra well posed, so repeated launches see the
      // same values
      require(level >= 1, "the smoothing kernels run on levels >= 1");
      const int k = nu_;
      const int nblk = dots_blocks(n, 1024), nd = dot_blocks(lev);
      const size_t ps = part_stride(lev);
      double* pa = lev.part.p;
      double* pb = lev.part.p + ps;
      double* pc = lev.part.p + 2 * ps;
      double* S = lev.scal.p;
      T* V = lev.V.p;
      T* Z = lev.Z.p;
      T* t = V + (size_t)k * n;
      launch_fill<T>(V, T(1), (size_t)(k + 1) * n, s);
      launch_fill<T>(Z, T(1), (size_t)k * n, s);
      launch_fill<double>(pa, 0.0, 3 * ps, s);
      launch_fill<double>(S, 0.0, kGsScal, s);
      launch_fill<double>(S, 1.0, k, s);                                           // D_q
      for (int q = 0; q < k; ++q) launch_fill<double>(S + 96 + 9 * q + q, 1.0, 1, s);   // H_qq
      if (k == 1) launch_fill<double>(pa + 1, 1.0, 1, s);                          // u_0 . u_0
      else launch_fill<double>(pb + k - 1, 1.0, 1, s);                             // |u_{k-1}|^2
      double* hcol = S + 96;
      if (kernel == IBMG_KERNEL_APPLY_DOTS) {
        by = (double)(k + 2) * n * ts;
        ms = time_launches([&] { op_dots<T>(level, Z, lev.t.p, V, V, k, n, pa, lev.F.p, s); }, reps, s);
      } else if (kernel == IBMG_KERNEL_UPD_DOTS) {
        by = (double)(k + 2) * n * ts;
        ms = time_launches([&] { launch_gs_update<T>(t, V, V, k, n, n, pa, nd, pb, S, pc, s); }, reps, s);
      } else if (kernel == IBMG_KERNEL_SCALE_UPD) {
        // zero second-pass dots and a unit |t|^2 in every block's partials:
        // t keeps its values and is scaled by the same factor each launch
        by = (double)(k + 2) * n * ts;
        launch_fill<double>(pb, 0.0, (size_t)nblk * (k + 1), s);
        launch_fill<double>(pb + k, 1.0, 1, s);
        ms = time_launches([&] { launch_scale_upd<T>(t, V, k, n, n, pb, nblk, hcol, s); }, reps, s);
      } else if (kernel == IBMG_KERNEL_UPD_NORM) {
        by = (double)(k + 2) * n * ts;
        launch_fill<double>(pb, 0.0, (size_t)nblk * k, s);
        ms = time_launches([&] { launch_upd_norm<T>(t, V, k, n, n, pb, nblk, hcol, pa, s); }, reps, s);
      } else if (kernel == IBMG_KERNEL_SCALE_RED) {
        by = 2.0 * n * ts;
        launch_fill<double>(pb, 1.0, (size_t)nblk, s);
        ms = time_launches([&] { launch_scale_red<T>(t, lev.t.p, n, pb, nblk, hcol, s); }, reps, s);
      } else {
        by = (double)(k + 2) * n * ts;
        launch_fill<double>(pc + k, 1.0, 1, s);                                    // |u_k|^2
        ms = time_launches([&] { launch_gs_combine<T>(lev.w.p, Z, k, n, n, pc, S, false, s); }, reps, s);
      }
    } else {
      require(false, "unknown kernel");
    }
    if (bytes) *bytes = by;
    if (flops) *flops = fl;
    return ms;
  }

  std::vector<int64_t> stats() const override {
    std::vector<int64_t> v;
    v.push_back(L_ + 1);
    for (int l = 0; l <= L_; ++l) {
      const Level<T>& lev = levels_[l];
      v.push_back(lev.N);
      v.push_back((int64_t)lev.g.npd * lev.g.npd);
      v.push_back(lev.n_unique);
      v.push_back(lev.n_ib);
      v.push_back((int64_t)lev.f[0].tcol.size() + (int64_t)lev.f[1].tcol.size());
      v.push_back(lev.ncolour);
    }
    return v;
  }

 private:
  ibmg_desc d_;
  int M_ = 0, E_ = 0, nu_ = 2, L_ = 0, n0_ = 0;
  std::vector<double> X_, kappa_, rest_;
  bool tangent_ = false;   // IBMG_SPRING_TANGENT
  std::vector<int> ends_, sizes_;
  std::vector<int> adj_ptr_, adj_nbr_, adj_sid_;
  DBuf<int> d_adj_ptr_, d_adj_nbr_, d_ends_;
  DBuf<int> d_order_;   // points in cell order
  DBuf<double> d_adj_k_, d_X_;
  DBuf<float> d_adj_kf_;
  // tangent model: (K_e[0][1], K_e[1][1]) per incidence, kappa_e and L_e per
  // incidence (spring forces), unit blocks per spring (gradient)
  DBuf<double> d_adj_k2_, d_adj_kap_, d_adj_rest_, d_gblocks_;
  DBuf<float> d_adj_k2f_;
  std::vector<Level<T>> levels_;
  DBuf<double> inv0_;
  DBuf<double> Fd_, Uw_, Ul_;
  DBuf<double> Fs_, fs_, rhs_;   // time step: nodal forces, spread forces, right-hand side
  // outer FGMRES
  int outer_cap_ = 0;
  DBuf<double> Vo_, Zo_, Ho_, cs_, sn_, g_, y_, osc_, opart_, ofold_, bp_, rr_;
  double* pinned_ = nullptr;
  // V-cycle graph
  bool use_graph_ = graphs_enabled();
  hipStream_t gstream_ = nullptr;
  hipGraph_t graph_ = nullptr;
  hipGraphExec_t gexec_ = nullptr;
  DBuf<double> vin_, vout_;
  DBuf<double> tpart_;   // slice sums of the IB-row values on coarse levels
  hipEvent_t est_ev_ = nullptr;   // the outer loop's estimate copy
  hipStream_t side_ = nullptr;    // the coarsest inversion beside the box inversions
  hipEvent_t ev_fork_ = nullptr, ev_join_ = nullptr;
  DBuf<double> coarse_aug_;       // its work matrix until the join
  bool defer_coarse_ = false;   // a member of a batch: the batch inverts the coarsest system
  std::vector<int> members_;    // and has this many systems on each level
  bool valid_ = true;
  double setup_ms_ = 0.0;   // wall time of the latest build_all (device work included)
  DBuf<double> aug0_;    // the assembled coarsest matrix while its inversion is deferred

  static bool graphs_enabled() {
    const char* e = std::getenv("IBMG_GRAPH");
    return !(e && e[0] == '0');
  }
};

}  // namespace ibmg
