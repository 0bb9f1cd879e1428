// Batched form: many independent Stokes-IB systems (different grid sizes,
// structures and stiffnesses, one fluid and one box configuration) solved
// together.  Each system's hierarchy, IB rows, box inverses and coarsest
// inverse are built by its own single-system set-up; the batch then runs
// Alg. 1 on all of them in lockstep by level.  Level l has the same grid
// size 8 * 2^l (coarse_N * 2^l) in every system, so systems sorted by size,
// largest first, make level l's active systems a prefix [0, nact_l) and a
// level's batch vectors are nact_l level vectors back to back.  A system
// whose finest level is l joins the descent there and leaves the ascent
// there.  Per level and sweep: one launch for L_IB with its IB rows and dots,
// the Schwarz launches over every system's boxes, and the
// Gram-Schmidt update over all systems at once.  The outer FGMRES(m) runs
// per system in lockstep with one host read of all residual estimates per
// iteration; converged systems drop out through device-side active flags.
#include <numeric>

#include "solver_impl.hpp"

namespace ibmg {

// Host checks of a batch's descriptors (every one valid, the shared
// parameters equal, the options the batched form runs).
void validate_batch(int nsys, const ibmg_desc* d) {
  require(nsys >= 1 && nsys <= 4096, "nsys must lie in [1, 4096]");
  require(d != nullptr, "descs is NULL");
  const ibmg_desc& d0 = d[0];
  for (int i = 0; i < nsys; ++i) {
    validate_desc(d[i]);
    require(d[i].smoother == IBMG_RAS, "the batched form uses the additive Schwarz smoother");
    require(d[i].spring_model == IBMG_SPRING_LINEAR, "the batched form takes linear springs");
    require(d[i].combine == IBMG_COMBINE_RESTRICTED && d[i].sweep_kind == IBMG_SWEEP_FGMRES,
            "the batched form runs the restricted combination with FGMRES smoothing");
    require(d[i].coarse_N == d0.coarse_N && d[i].rho == d0.rho && d[i].mu == d0.mu && d[i].dt == d0.dt &&
                d[i].box == d0.box && d[i].overlap == d0.overlap && d[i].nu1 == d0.nu1 &&
                d[i].nu2 == d0.nu2 && d[i].precision == d0.precision && d[i].max_restart == d0.max_restart,
            "batched systems must share coarse_N, rho, mu, dt, box, overlap, nu1, nu2, precision and "
            "max_restart");
  }
}

template <typename T>
class BatchSolver final : public BatchBase {
 public:
  BatchSolver(int nsys, const ibmg_desc* d, hipStream_t s) : ns_(nsys) {
    const auto t_begin = std::chrono::steady_clock::now();
    validate_batch(nsys, d);
    const ibmg_desc& d0 = d[0];
    nu1_ = d0.nu1;
    nu2_ = d0.nu2;
    max_restart_ = d0.max_restart > 0 ? d0.max_restart : 30;
    rho_zero_ = d0.rho == 0.0;
    order_.resize(nsys);
    std::iota(order_.begin(), order_.end(), 0);
    std::stable_sort(order_.begin(), order_.end(), [&](int a, int b) { return d[a].N > d[b].N; });
    // systems per level (coarse_N 2^l has the same size in every system)
    std::vector<int> members;
    for (int p = 0; p < nsys; ++p) {
      int l = 0;
      for (int n = d[order_[p]].N; ; n /= 2, ++l)
        if (n <= d0.coarse_N) break;
      if ((int)members.size() <= l) members.resize(l + 1, 0);
      for (int k = 0; k <= l; ++k) members[k]++;
    }
    for (int p = 0; p < nsys; ++p) sys_.emplace_back(new Solver<T>(d[order_[p]], s, true, members));
    {
      // every system's coarsest matrix has the same size (shared coarse_N):
      // they are swept a group at a time, one run of sweeps per group of up
      // to 1 GiB of matrices
      const int n0 = sys_[0]->n0_;
      const size_t stride = (size_t)n0 * n0;
      const int grp = (int)std::max<size_t>(1, std::min<size_t>(nsys, ((size_t)1 << 27) / stride));
      DBuf<double> mats(stride * grp), work(sweep_work(n0, grp)), res(stride);
      for (int p0 = 0; p0 < nsys; p0 += grp) {
        const int cnt = std::min(grp, nsys - p0);
        for (int p = p0; p < p0 + cnt; ++p) {
          require(sys_[p]->n0_ == n0 && sys_[p]->aug0_.n == stride, "coarsest systems differ in size");
          IBMG_HIP(hipMemcpyAsync(mats.p + (p - p0) * stride, sys_[p]->aug0_.p, stride * sizeof(double),
                                  hipMemcpyDeviceToDevice, s));
        }
        launch_gj_invert(mats.p, n0, cnt, work.p, s);
        for (int p = p0; p < p0 + cnt; ++p) sys_[p]->finish_coarse(mats.p + (p - p0) * stride, res.p, s);
        IBMG_HIP(hipStreamSynchronize(s));
      }
      for (int p = 0; p < nsys; ++p) sys_[p]->check_breakdown(s, true);
    }
    Lmax_ = sys_[0]->L_;
    nact_.assign(Lmax_ + 2, 0);
    for (int p = 0; p < nsys; ++p)
      for (int l = 0; l <= sys_[p]->L_; ++l) nact_[l]++;
    off_.assign(nsys + 1, 0);
    for (int p = 0; p < nsys; ++p) {
      const long long N = sys_[p]->d_.N;
      off_[p + 1] = off_[p] + 3 * N * N;
    }
    ntot_ = (size_t)off_[nsys];
    require(ntot_ < ((size_t)1 << 31), "batch too large for 32-bit indices");
    d_off_.upload(off_, s);
    std::vector<int> ones(nsys, 1);
    d_act_.upload(ones, s);
    IBMG_HIP(hipHostMalloc((void**)&pin_d_, (size_t)(2 * nsys + 8) * sizeof(double), hipHostMallocDefault));
    IBMG_HIP(hipHostMalloc((void**)&pin_i_, (size_t)(2 * nsys + 8) * sizeof(int), hipHostMallocDefault));
    build_levels(s);
    build_outer_rows(s);
    build_coarse(s);
    alloc_outer(max_restart_);
    time_sweeps(s);
    IBMG_HIP(hipStreamSynchronize(s));
    setup_ms_ = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_begin).count();
  }

  ~BatchSolver() override {
    drop_graph();
    if (gstream_) (void)hipStreamDestroy(gstream_);
    if (pin_d_) (void)hipHostFree(pin_d_);
    if (pin_i_) (void)hipHostFree(pin_i_);
  }

  int nsys() const override { return ns_; }

 private:
  struct BLevel {
    int N = 0, nact = 0, nblk = 1;
    size_t n = 0, pst = 0;
    StokesCoef<T> c{};
    DBuf<T> w, b, r, V, Z;
    DBuf<double> scal, part;
    // the systems' explicit IB rows, and the most of one system
    DBuf<IbRows<T>> ib_tab;
    IbRows<T> rows{};
    int nrows = 0;
    // Schwarz boxes: (system, box) entries; IB boxes with whole rows and their
    // inverses, eliminated ones and their factors, interior boxes and the class
    // matrices of the first member that has one
    BoxGeom g{};
    int nbox = 0, n_int = 0, n_rows = 0, n_elim = 0;
    double w_vals = 0;   // values of W over all eliminated boxes
    DBuf<int> int_ents, row_ents, elim_ents, wptr, wrow;
    DBuf<const T*> row_inv;
    DBuf<const void*> wtab, qtab;
    DBuf<unsigned short> ord;
    DBuf<unsigned char> coupled;
    DBuf<T> w_res, sym_part;
    SymIB sym{};
    IntClassView cls{};
    double sweep_us = 0;
  };

  // ---------------------------------------------------------------- set-up
  template <typename U>
  static const U* tvals(const CompFoot& f) {
    if constexpr (std::is_same<U, double>::value) return f.tval.p;
    else return f.tvalf.p;
  }

  // Concatenate the finest levels' IB rows of system positions [0, count) with
  // indices shifted by base.
  template <typename U>
  void gather_rows(int count, const std::vector<size_t>& base, DBuf<int>& rows, DBuf<int>& ptr, DBuf<int>& col,
                   DBuf<U>& val, int* nrows, hipStream_t s) {
    std::vector<int> hr, hp(1, 0), hc;
    std::vector<std::pair<const U*, size_t>> pieces;
    for (int p = 0; p < count; ++p) {
      Solver<T>& S = *sys_[p];
      Level<T>& lev = S.levels_[S.L_];
      const size_t nn = (size_t)lev.N * lev.N;
      for (int c = 0; c < 2; ++c) {
        const CompFoot& f = lev.f[c];
        if (f.tcol.empty()) continue;
        const size_t b0 = base[p] + c * nn;
        for (size_t r = 0; r + 1 < f.tptr.size(); ++r) {
          if (f.tptr[r + 1] == f.tptr[r]) continue;
          hr.push_back((int)(b0 + r));
          hp.push_back(hp.back() + (f.tptr[r + 1] - f.tptr[r]));
        }
        // columns index the system's [u | v] vector
        for (int cc : f.tcol) hc.push_back((int)(base[p] + cc));
        pieces.emplace_back(tvals<U>(f), f.tcol.size());
      }
    }
    *nrows = (int)hr.size();
    rows.upload(hr, s);
    ptr.upload(hp, s);
    col.upload(hc, s);
    val.alloc(hc.size());
    size_t at = 0;
    for (auto& pc : pieces) {
      IBMG_HIP(hipMemcpyAsync(val.p + at, pc.first, pc.second * sizeof(U), hipMemcpyDeviceToDevice, s));
      at += pc.second;
    }
  }

  void build_levels(hipStream_t s) {
    lv_.resize(Lmax_ + 1);
    for (int l = 0; l <= Lmax_; ++l) {
      BLevel& L = lv_[l];
      Level<T>& l0 = sys_[0]->levels_[l];
      L.N = l0.N;
      L.n = 3 * (size_t)L.N * L.N;
      L.nact = nact_[l];
      L.c = sys_[0]->template coef<T>(l0);
      const size_t bn = (size_t)L.nact * L.n;
      L.w.alloc(bn);
      L.b.alloc(bn);
      L.r.alloc(bn);
      launch_fill<T>(L.w.p, T(0), bn, s);
      launch_fill<T>(L.b.p, T(0), bn, s);
      launch_fill<T>(L.r.p, T(0), bn, s);
      if (l == 0) continue;
      const int nv = std::max(nu1_, nu2_);
      L.V.alloc((size_t)(nv + 1) * bn);
      L.Z.alloc((size_t)nv * bn);
      launch_fill<T>(L.V.p, T(0), L.V.n, s);
      launch_fill<T>(L.Z.p, T(0), L.Z.n, s);
      std::vector<IbRows<T>> tab;
      L.rows = IbRows<T>{nullptr, nullptr, {}, {}, 0, 16};
      int blocks = 0;
      for (int p = 0; p < L.nact; ++p) {
        Level<T>& lev = sys_[p]->levels_[l];
        tab.push_back(IbRows<T>{lev.d_ib_rows.p, lev.d_ib_flag.p, sys_[p]->template csr<T>(lev.f[0]),
                                sys_[p]->template csr<T>(lev.f[1]), (int)lev.ib_rows.size(), lev.ib_lanes});
        L.nrows += tab[p].n;
        if (apply_blocks(L.N, tab[p].n, tab[p].lanes) > blocks) {   // the largest grid of one system
          blocks = apply_blocks(L.N, tab[p].n, tab[p].lanes);
          L.rows.n = tab[p].n;
          L.rows.lanes = tab[p].lanes;
        }
      }
      L.ib_tab.upload(tab, s);
      L.rows.each = L.ib_tab.p;
      // blocks per system: the device four times over, shared by the systems
      L.nblk = std::max(8, (4096 + L.nact - 1) / L.nact);
      L.pst = (size_t)std::max(apply_blocks(L.N, L.rows.n, L.rows.lanes, L.nblk), gs_blocks(L.n)) * (kMaxNu + 1);
      L.part.alloc(3 * (size_t)L.nact * L.pst);
      L.scal.alloc((size_t)L.nact * kGsScal);
      // (equal fluid coefficients and box geometry give one interior matrix)
      L.g = l0.g;
      L.nbox = L.g.npd * L.g.npd;
      require((size_t)L.nact * L.nbox < ((size_t)1 << 31), "too many boxes");
      L.g.nbs = L.nbox;
      L.g.sysn = L.n;
      L.g.act = d_act_.p;
      const size_t stride = sys_[0]->box_stride(l0);
      std::vector<int> ie, re, ee, wptr(1, 0), wrow;
      std::vector<const T*> ri;
      std::vector<const void*> wt, qt;
      std::vector<unsigned short> ord;
      std::vector<unsigned char> cpl;
      int wmax = 0;
      for (int p = 0; p < L.nact; ++p) {
        Level<T>& lev = sys_[p]->levels_[l];
        for (int i = 0; i < lev.n_ib; ++i) {
          const int ent = p * L.nbox + lev.ib_list[i];
          if (!lev.use_sym) {
            re.push_back(ent);
            ri.push_back(lev.inv.p + (size_t)i * stride);
            continue;
          }
          ee.push_back(ent);
          wt.push_back(lev.wmat + (size_t)lev.wptr[i] * lev.w_stride);
          qt.push_back(lev.inv_sym + (size_t)i * sym_box_stride(lev.g));
          wrow.insert(wrow.end(), lev.wrow.begin() + lev.wptr[i], lev.wrow.begin() + lev.wptr[i + 1]);
          wptr.push_back((int)wrow.size());
          ord.insert(ord.end(), lev.ord.begin() + (size_t)i * lev.g.nown, lev.ord.begin() + (size_t)(i + 1) * lev.g.nown);
          cpl.insert(cpl.end(), lev.coupled.begin() + (size_t)i * lev.g.nown,
                     lev.coupled.begin() + (size_t)(i + 1) * lev.g.nown);
          wmax = std::max(wmax, lev.wptr[i + 1] - lev.wptr[i]);
        }
        for (int q : lev.int_list) ie.push_back(p * L.nbox + q);
        if (!L.cls.M && !lev.int_list.empty()) L.cls = lev.clsv;
      }
      L.n_int = (int)ie.size();
      L.n_rows = (int)re.size();
      L.n_elim = (int)ee.size();
      L.int_ents.upload(ie, s);
      L.row_ents.upload(re, s);
      L.row_inv.upload(ri, s);
      if (L.n_elim) {
        L.w_vals = (double)wrow.size() * l0.bm.nn;
        L.elim_ents.upload(ee, s);
        L.wtab.upload(wt, s);
        L.qtab.upload(qt, s);
        L.wptr.upload(wptr, s);
        L.wrow.upload(wrow, s);
        L.ord.upload(ord, s);
        L.coupled.upload(cpl, s);
        L.w_res.alloc((size_t)L.n_elim * L.g.nown);
        L.sym_part.alloc((size_t)L.n_elim * sym_part_len(L.g));
        L.sym = SymIB{nullptr, L.qtab.p, L.sym_part.p,
                      WBoxView{nullptr, L.wtab.p, L.wptr.p, L.wrow.p, l0.d_nonown.p, L.coupled.p, L.ord.p, l0.bm.nn,
                               (l0.bm.nn + 3) / 4 * 4, wmax},
                      L.w_res.p};
      }
      // (the sources of asynchronous copies end with this level's scope)
      IBMG_HIP(hipStreamSynchronize(s));
    }
    n0_ = sys_[0]->n0_;
  }

  // IB rows of every system at its finest level, indexed into the ragged
  // outer vectors (FP64: the outer residual stays in double precision).
  void build_outer_rows(hipStream_t s) {
    std::vector<size_t> base(ns_);
    for (int p = 0; p < ns_; ++p) base[p] = (size_t)off_[p];
    gather_rows<double>(ns_, base, orows_, optr_, ocol_, oval_, &onrows_, s);
  }

  void build_coarse(hipStream_t s) {
    inv0_.alloc((size_t)ns_ * n0_ * n0_);
    for (int p = 0; p < ns_; ++p)
      IBMG_HIP(hipMemcpyAsync(inv0_.p + (size_t)p * n0_ * n0_, sys_[p]->inv0_.p, (size_t)n0_ * n0_ * sizeof(double),
                              hipMemcpyDeviceToDevice, s));
  }

  // Time of each level's Schwarz sweep (reported by stats).
  void time_sweeps(hipStream_t s) {
    if (dry_run()) return;
    for (int l = 1; l <= Lmax_; ++l) {
      BLevel& L = lv_[l];
      launch_fill<T>(L.r.p, T(1), (size_t)L.nact * L.n, s);
      L.sweep_us = 1e3 * time_launches([&] { ras(l, L.r.p, L.w.p, s); }, 5, s);
      launch_fill<T>(L.r.p, T(0), (size_t)L.nact * L.n, s);
      launch_fill<T>(L.w.p, T(0), (size_t)L.nact * L.n, s);
    }
  }

  // --------------------------------------------------------- level pieces
  // One sweep over every active system's boxes: the boxes with whole rows and
  // the interior ones in one launch, then the eliminated boxes' three (the first
  // with the interior boxes where no box has whole rows).
  void ras(int l, const T* r, T* z, hipStream_t s) {
    BLevel& L = lv_[l];
    const bool rows = L.n_rows > 0 || !L.n_elim;
    if (rows)
      launch_ras_apply<T>(r, z, L.g, nullptr, L.row_ents.p, L.n_rows, L.cls, L.int_ents.p, L.n_int, s, 3, false,
                          nullptr, L.row_inv.p);
    if (L.n_elim)
      launch_ras_apply<T>(r, z, L.g, nullptr, L.elim_ents.p, L.n_elim, L.cls, L.int_ents.p, rows ? 0 : L.n_int, s, 3,
                          false, &L.sym);
  }

  Many many(const BLevel& L) const {
    Many m;
    m.nsys = L.nact;
    m.bs = L.n;
    m.ps = L.pst;
    m.nblk = L.nblk;
    m.act = d_act_.p;
    return m;
  }

  // Sec. 3.3 smoothing on every active system of level l: w <- w + e, e from
  // nu FGMRES iterations on L e = b - L w, on the unnormalised basis of the
  // single-system form and with its launches.  With w_zero, w is not read; crs
  // (w_zero only): also the restriction of the new residual to the next coarser
  // level, by the Arnoldi relation.
  void smooth(int l, T* w, const T* b, int nu, bool w_zero, T* crs, hipStream_t s) {
    BLevel& L = lv_[l];
    const size_t n = L.n, bn = (size_t)L.nact * n, pn = (size_t)L.nact * L.pst;
    const Many m = many(L);
    const FootView<T> none{};
    T* V = L.V.p;
    const T* u0 = b;
    if (!w_zero) {
      launch_apply<T>(w, V, b, nullptr, L.rows, none, none, L.N, 0, L.c, false, s, m);
      u0 = V;
    }
    double* pd = L.part.p;
    double* pu[2] = {L.part.p + pn, L.part.p + 2 * pn};
    const int nd = apply_blocks(L.N, L.rows.n, L.rows.lanes, L.nblk);
    for (int k = 0; k < nu; ++k) {
      const T* uk = k == 0 ? u0 : V + (size_t)k * bn;
      T* zk = L.Z.p + (size_t)k * bn;
      T* t = V + (size_t)(k + 1) * bn;
      ras(l, uk, zk, s);
      launch_apply_dots<T>(zk, t, nullptr, L.rows, none, none, L.N, 0, L.c, u0, V, k + 1, bn, pd, s, m);
      launch_gs_update<T>(t, u0, V, k + 1, bn, n, pd, nd, pu[(k + 1) & 1], L.scal.p, pu[k & 1], s, m);
    }
    const double* pl = pu[(nu - 1) & 1];
    if (crs) launch_gs_combine_restrict<T>(w, L.Z.p, u0, V, nu, bn, L.N / 2, pl, L.scal.p, crs, s, m);
    else launch_gs_combine<T>(w, L.Z.p, nu, bn, n, pl, L.scal.p, w_zero, s, m);
  }

  // Alg. 1 on every system: r and z are ragged batch vectors (FP64).
  void vcycle_body(const double* r, double* z, hipStream_t s) {
    for (int l = Lmax_; l >= 1; --l) {
      BLevel& L = lv_[l];
      const int p0 = nact_[l + 1], p1 = nact_[l];
      if (p1 > p0) launch_cast<double, T>(r + off_[p0], L.b.p + (size_t)p0 * L.n, (size_t)(p1 - p0) * L.n, s);
      BLevel& C = lv_[l - 1];
      const bool relation = nu1_ <= kArnoldiResidualNu;
      smooth(l, L.w.p, L.b.p, nu1_, true, relation ? C.b.p : nullptr, s);
      if (!relation) {
        const FootView<T> none{};
        launch_apply<T>(L.w.p, L.r.p, L.b.p, nullptr, L.rows, none, none, L.N, 0, L.c, false, s, many(L));
        launch_restrict<T>(L.r.p, C.b.p, C.N, s, many(L));
      }
    }
    launch_coarse_apply_batch<T>(inv0_.p, n0_, lv_[0].b.p, lv_[0].w.p, nact_[0], s);
    for (int l = 1; l <= Lmax_; ++l) {
      BLevel& L = lv_[l];
      const int p0 = nact_[l + 1], p1 = nact_[l];
      launch_prolong_add_batch<T>(lv_[l - 1].w.p, L.w.p, lv_[l - 1].N, p1, d_act_.p, s);
      smooth(l, L.w.p, L.b.p, nu2_, false, nullptr, s);
      if (p1 > p0) launch_cast<T, double>(L.w.p + (size_t)p0 * L.n, z + off_[p0], (size_t)(p1 - p0) * L.n, s);
    }
  }

  // The batched V-cycle is captured once into a HIP graph (kernel nodes
  // only) reading vin_ and writing vout_.
  void build_graph() {
    if (!gstream_) IBMG_HIP(hipStreamCreateWithFlags(&gstream_, hipStreamNonBlocking));
    launch_fill<double>(vin_.p, 0.0, ntot_, gstream_);
    launch_fill<double>(vout_.p, 0.0, ntot_, gstream_);
    IBMG_HIP(hipStreamSynchronize(gstream_));
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

  void vcycle_ragged(const double* r, double* z, hipStream_t s) {
    if (!use_graph_) {
      vcycle_body(r, z, s);
      return;
    }
    if (!gexec_) build_graph();
    IBMG_HIP(hipMemcpyAsync(vin_.p, r, ntot_ * sizeof(double), hipMemcpyDeviceToDevice, s));
    IBMG_HIP(hipGraphLaunch(gexec_, s));
    IBMG_HIP(hipMemcpyAsync(z, vout_.p, ntot_ * sizeof(double), hipMemcpyDeviceToDevice, s));
  }

  void gather(const double* const* src, double* dst, hipStream_t s) {
    for (int p = 0; p < ns_; ++p) {
      require(src[order_[p]] != nullptr, "NULL system vector");
      IBMG_HIP(hipMemcpyAsync(dst + off_[p], src[order_[p]], (size_t)(off_[p + 1] - off_[p]) * sizeof(double),
                              hipMemcpyDeviceToDevice, s));
    }
  }

  void scatter(const double* src, double* const* dst, hipStream_t s) {
    for (int p = 0; p < ns_; ++p) {
      require(dst[order_[p]] != nullptr, "NULL system vector");
      IBMG_HIP(hipMemcpyAsync(dst[order_[p]], src + off_[p], (size_t)(off_[p + 1] - off_[p]) * sizeof(double),
                              hipMemcpyDeviceToDevice, s));
    }
  }

 public:
  void vcycle(const double* const* r, double* const* z, hipStream_t s) override {
    require(r && z, "NULL pointer array");
    set_all_active(s);
    gather(r, io_in_.p, s);
    vcycle_ragged(io_in_.p, io_out_.p, s);
    scatter(io_out_.p, z, s);
  }

 private:

  void set_all_active(hipStream_t s) {
    for (int p = 0; p < ns_; ++p) pin_i_[p] = 1;
    IBMG_HIP(hipMemcpyAsync(d_act_.p, pin_i_, ns_ * sizeof(int), hipMemcpyHostToDevice, s));
    IBMG_HIP(hipStreamSynchronize(s));
  }

  // --------------------------------------------------------- outer solve
  // y = L_IB x (b != null: y = b - L_IB x) on every system's finest level,
  // FP64, over the ragged vectors: one stencil launch per grid size.
  void op_outer(const double* x, double* y, const double* b, hipStream_t s) {
    for (int l = Lmax_; l >= 1; --l) {
      const int p0 = nact_[l + 1], p1 = nact_[l];
      if (p1 <= p0) continue;
      Level<T>& lev = sys_[p0]->levels_[l];
      launch_apply_batch<double>(x + off_[p0], y + off_[p0], b ? b + off_[p0] : nullptr, lev.N, lev.cd, p1 - p0,
                                 lv_[l].n, s);
    }
    launch_ib_rows<double>(x, y, orows_.p, optr_.p, ocol_.p, oval_.p, onrows_, b ? -1.0 : 1.0, s);
  }

  // remove the null-space components of every system's vector; the block
  // sums are left at osums_ + 8 p
  void project(double* a, hipStream_t s) {
    for (int l = Lmax_; l >= 1; --l) {
      const int p0 = nact_[l + 1], p1 = nact_[l];
      if (p1 <= p0) continue;
      const int N = lv_[l].N;
      const size_t n = lv_[l].n;
      launch_block_sums_b<double>(a + off_[p0], N, n, ppart_.p + (size_t)p0 * 64 * 3, 64, 64 * 3, p1 - p0, s);
      launch_dots_finish_b(ppart_.p + (size_t)p0 * 64 * 3, 3, 64, 64 * 3, osums_.p + (size_t)p0 * 8, nullptr, 8,
                           0, p1 - p0, s);
      launch_subtract_means_b<double>(a + off_[p0], N, n, osums_.p + (size_t)p0 * 8, 8, rho_zero_ ? 1 : 0, p1 - p0,
                                      s);
    }
  }

  // per-system 2-norms into onorm_ and pin_d_[0..ns)
  void norms(const double* a, hipStream_t s) {
    const BSeg sg{d_off_.p, 0, nullptr};
    launch_dots_b<double>(a, 1, ntot_, a, sg, ns_, opa_.p, opst_, onblk_, s);
    launch_dots_finish_b(opa_.p, 1, onblk_, opst_, onorm_.p, nullptr, 1, 2, ns_, s);
    IBMG_HIP(hipMemcpyAsync(pin_d_, onorm_.p, ns_ * sizeof(double), hipMemcpyDeviceToHost, s));
    IBMG_HIP(hipStreamSynchronize(s));
  }

  // every buffer of the outer solve and the V-cycle's input and output,
  // for restarts up to max_restart (placed at creation)
  void alloc_outer(int restart) {
    io_in_.alloc(ntot_);
    io_out_.alloc(ntot_);
    vin_.alloc(ntot_);
    vout_.alloc(ntot_);
    Vo_.alloc((size_t)(restart + 1) * ntot_);
    Zo_.alloc((size_t)restart * ntot_);
    launch_fill<double>(Vo_.p, 0.0, Vo_.n, nullptr);
    launch_fill<double>(Zo_.p, 0.0, Zo_.n, nullptr);
    ldh_ = restart + 1;
    hst_ = (size_t)(restart + 1) * restart;
    rst_ = (size_t)restart + 2;
    Ho_.alloc((size_t)ns_ * hst_);
    cs_.alloc((size_t)ns_ * rst_);
    sn_.alloc((size_t)ns_ * rst_);
    g_.alloc((size_t)ns_ * rst_);
    y_.alloc((size_t)ns_ * rst_);
    est_.alloc(ns_);
    onorm_.alloc(ns_);
    osums_.alloc((size_t)ns_ * 8);
    ppart_.alloc((size_t)ns_ * 64 * 3);
    size_t nmax = 0;
    for (int p = 0; p < ns_; ++p) nmax = std::max(nmax, (size_t)(off_[p + 1] - off_[p]));
    onblk_ = dots_blocks(nmax, 256);
    opst_ = (size_t)onblk_ * (restart + 1);
    opa_.alloc((size_t)ns_ * opst_);
    opb_.alloc((size_t)ns_ * opst_);
    bp_.alloc(ntot_);
    xb_.alloc(ntot_);
    rr_.alloc(ntot_);
    kcnt_.alloc(ns_);
    nmax_ = nmax;
    outer_cap_ = restart;
  }

  void upload_flags(const std::vector<int>& act, hipStream_t s) {
    for (int p = 0; p < ns_; ++p) pin_i_[p] = act[p];
    IBMG_HIP(hipMemcpyAsync(d_act_.p, pin_i_, ns_ * sizeof(int), hipMemcpyHostToDevice, s));
  }

 public:
  int fgmres(const double* const* b, double* const* x, const ibmg_solve_opts& o, ibmg_solve_info* infos,
             hipStream_t s) override {
    const auto t0 = std::chrono::steady_clock::now();
    require(b && x, "NULL pointer array");
    require(o.restart >= 1 && o.restart <= outer_cap_,
            "restart must lie in [1, max_restart = " + std::to_string(outer_cap_) + "]");
    require(o.max_it >= 1, "max_it must be >= 1");
    require(std::isfinite(o.rtol) && o.rtol > 0.0, "rtol must be finite and > 0");
    require(o.transpose == 0, "the batched form solves with L_IB only");
    const int m = o.restart;
    set_all_active(s);
    gather(b, bp_.p, s);
    project(bp_.p, s);
    // removed null-space norms
    std::vector<double> sums((size_t)ns_ * 8);
    IBMG_HIP(hipMemcpyAsync(sums.data(), osums_.p, sums.size() * sizeof(double), hipMemcpyDeviceToHost, s));
    norms(bp_.p, s);
    std::vector<double> bnorm(pin_d_, pin_d_ + ns_), target(ns_), est(ns_), null(ns_);
    for (int p = 0; p < ns_; ++p) {
      const double nn = (double)(off_[p + 1] - off_[p]) / 3.0;
      double n2 = sums[8 * p + 2] * sums[8 * p + 2] / nn;
      if (rho_zero_) n2 += (sums[8 * p] * sums[8 * p] + sums[8 * p + 1] * sums[8 * p + 1]) / nn;
      null[p] = std::sqrt(n2);
      if (!std::isfinite(bnorm[p]) || !std::isfinite(n2)) throw Error(IBMG_ERR_NONFINITE, "right-hand side holds NaN/Inf");
      target[p] = o.rtol * bnorm[p];
      est[p] = bnorm[p];
    }
    if (o.use_x0) gather(const_cast<const double* const*>(x), xb_.p, s);
    else launch_fill<double>(xb_.p, 0.0, ntot_, s);
    std::vector<int> its(ns_, 0), conv(ns_, 0), act(ns_, 0), kc(ns_, 0), restarts(ns_, 0), vcyc(ns_, 0);
    std::vector<int> hist_n(ns_, 0);
    auto push_hist = [&](int p, double v) {
      ibmg_solve_info* inf = infos ? &infos[order_[p]] : nullptr;
      if (inf && inf->history && hist_n[p] < inf->history_cap) inf->history[hist_n[p]] = v;
      ++hist_n[p];
    };
    for (int p = 0; p < ns_; ++p)
      if (bnorm[p] == 0.0) conv[p] = 1;
    const BSeg sga{d_off_.p, 0, d_act_.p};
    const BSeg sgall{d_off_.p, 0, nullptr};
    while (true) {
      // restart: V0 = (b - L x) / beta for the systems still running
      op_outer(xb_.p, Vo_.p, bp_.p, s);
      norms(Vo_.p, s);
      int nrun = 0;
      for (int p = 0; p < ns_; ++p) {
        act[p] = 0;
        if (conv[p]) continue;
        const double beta = pin_d_[p];
        if (!std::isfinite(beta)) throw Error(IBMG_ERR_NONFINITE, "residual is not finite");
        est[p] = beta;
        if (beta <= target[p]) {
          conv[p] = 1;
          continue;
        }
        if (its[p] >= o.max_it) continue;
        act[p] = 1;
        ++nrun;
      }
      if (nrun == 0) break;
      upload_flags(act, s);
      launch_scale_b<double>(Vo_.p, Vo_.p, onorm_.p, 1, sga, ns_, nmax_, s);
      launch_fill<double>(g_.p, 0.0, g_.n, s);
      IBMG_HIP(hipMemcpy2DAsync(g_.p, rst_ * sizeof(double), onorm_.p, sizeof(double), sizeof(double), ns_,
                                hipMemcpyDeviceToDevice, s));
      std::fill(kc.begin(), kc.end(), 0);
      for (int k = 0; k < m && nrun > 0; ++k) {
        double* vk = Vo_.p + (size_t)k * ntot_;
        double* zk = Zo_.p + (size_t)k * ntot_;
        double* t = Vo_.p + (size_t)(k + 1) * ntot_;
        vcycle_ragged(vk, zk, s);
        op_outer(zk, t, nullptr, s);
        double* hcol = Ho_.p + (size_t)k * ldh_;
        launch_dots_b<double>(Vo_.p, k + 1, ntot_, t, sga, ns_, opa_.p, opst_, onblk_, s);
        launch_upd_dots_b<double>(t, Vo_.p, k + 1, ntot_, sga, ns_, opa_.p, onblk_, opst_, hcol, hst_, opb_.p, s);
        launch_upd_norm_b<double>(t, Vo_.p, k + 1, ntot_, sga, ns_, opb_.p, onblk_, opst_, hcol, hst_, opa_.p, s);
        launch_scale_red_b<double>(t, t, sga, ns_, nmax_, opa_.p, onblk_, opst_, hcol + k + 1, hst_, s);
        launch_givens_b(Ho_.p, ldh_, hst_, k, cs_.p, sn_.p, g_.p, rst_, est_.p, d_act_.p, ns_, s);
        IBMG_HIP(hipMemcpyAsync(pin_d_, est_.p, ns_ * sizeof(double), hipMemcpyDeviceToHost, s));
        IBMG_HIP(hipStreamSynchronize(s));
        bool changed = false;
        for (int p = 0; p < ns_; ++p) {
          if (!act[p]) continue;
          const double e = pin_d_[p];
          if (!std::isfinite(e)) throw Error(IBMG_ERR_NONFINITE, "iteration produced NaN/Inf");
          est[p] = e;
          ++its[p];
          ++vcyc[p];
          kc[p] = k + 1;
          push_hist(p, e / bnorm[p]);
          if (e <= target[p]) conv[p] = 1;
          if (conv[p] || its[p] >= o.max_it) {
            act[p] = 0;
            --nrun;
            changed = true;
          }
        }
        if (changed && nrun > 0) upload_flags(act, s);
      }
      for (int p = 0; p < ns_; ++p) {
        pin_i_[ns_ + p] = kc[p];
        if (kc[p] > 0) ++restarts[p];
      }
      IBMG_HIP(hipMemcpyAsync(kcnt_.p, pin_i_ + ns_, ns_ * sizeof(int), hipMemcpyHostToDevice, s));
      launch_backsolve_b(Ho_.p, ldh_, hst_, kcnt_.p, g_.p, y_.p, rst_, ns_, s);
      launch_combine_b<double>(xb_.p, Zo_.p, ntot_, y_.p, rst_, kcnt_.p, sgall, ns_, nmax_, s);
      IBMG_HIP(hipStreamSynchronize(s));
      bool more = false;
      for (int p = 0; p < ns_; ++p)
        if (!conv[p] && its[p] < o.max_it) more = true;
      if (!more) break;
    }
    set_all_active(s);
    project(xb_.p, s);
    op_outer(xb_.p, rr_.p, bp_.p, s);
    norms(rr_.p, s);
    std::vector<double> tr(pin_d_, pin_d_ + ns_);
    scatter(xb_.p, x, s);
    IBMG_HIP(hipStreamSynchronize(s));
    const double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    bool all = true;
    for (int p = 0; p < ns_; ++p) {
      if (!std::isfinite(tr[p])) throw Error(IBMG_ERR_NONFINITE, "solution is not finite");
      all = all && conv[p];
      if (!infos) continue;
      ibmg_solve_info& inf = infos[order_[p]];
      inf.iters = its[p];
      inf.restarts = restarts[p];
      inf.rel_res_est = bnorm[p] > 0 ? est[p] / bnorm[p] : 0.0;
      inf.rel_res_true = bnorm[p] > 0 ? tr[p] / bnorm[p] : 0.0;
      inf.rhs_null_norm = null[p];
      inf.setup_ms = setup_ms_;
      inf.solve_ms = ms;
      inf.vcycles = vcyc[p];
    }
    return all ? IBMG_OK : IBMG_NOT_CONVERGED;
  }

  // The Schwarz sweep of a batch level alone, on the level's work vectors
  // (filled with ones).  Algorithmic work: each IB box streams its whole rows or
  // its two factors, the interior product reads the class matrices once; every
  // box gathers nloc values and writes nown.
  double kernel_time(int kernel, int level, int reps, hipStream_t s, double* bytes, double* flops) override {
    require(kernel == IBMG_KERNEL_RAS_BATCH, "batch handles time the batched Schwarz launch only");
    require(level >= 1 && level <= Lmax_, "level out of range");
    require(reps >= 1 && reps <= 100000, "reps must lie in [1, 100000]");
    BLevel& L = lv_[level];
    set_all_active(s);
    launch_fill<T>(L.r.p, T(1), (size_t)L.nact * L.n, s);
    const double ts = sizeof(T);
    const BoxGeom& g = L.g;
    const double n_ib = L.n_rows + L.n_elim, q = (double)L.n_elim * sym_box_stride(g);
    double by = ((double)L.n_rows * g.nown * g.nloc + L.w_vals + q + (n_ib + L.n_int) * (g.nloc + g.nown)) * ts;
    if (L.n_int > 0) by += 4.0 * L.cls.nrt * L.cls.Kp * 16 * ts;
    const double ms = time_launches([&] { ras(level, L.r.p, L.w.p, s); }, reps, s);
    if (bytes) *bytes = by;
    if (flops)
      *flops = 2.0 * ((double)L.n_rows * g.nown * g.nloc + L.w_vals + (double)L.n_elim * g.nown * g.nown +
                      4.0 * L.n_int * L.cls.R * L.cls.K);
    return ms;
  }

  // [nsys, levels, then per level: N, systems, interior boxes, IB boxes, IB
  //  rows, boxes of an interior tile, items of a sweep (interior tiles and IB
  //  row chunks), sweep time (ns)]
  std::vector<int64_t> stats() const override {
    std::vector<int64_t> v{ns_, Lmax_ + 1};
    for (int l = 0; l <= Lmax_; ++l) {
      const BLevel& L = lv_[l];
      v.push_back(L.N);
      v.push_back(L.nact);
      v.push_back(L.n_int);
      v.push_back(L.n_rows + L.n_elim);
      v.push_back(L.nrows);
      v.push_back(l ? 16 : 0);
      v.push_back((L.n_int + 15) / 16 * L.cls.nrt + (L.n_rows + L.n_elim) * L.g.nch);
      v.push_back((int64_t)(L.sweep_us * 1e3));
    }
    return v;
  }

 private:
  int ns_ = 0, Lmax_ = 0, nu1_ = 2, nu2_ = 2, n0_ = 0, max_restart_ = 30;
  double setup_ms_ = 0.0;   // wall time of the constructor's set-up (device work included)
  bool rho_zero_ = false;
  std::vector<int> order_, nact_;
  std::vector<std::unique_ptr<Solver<T>>> sys_;
  std::vector<BLevel> lv_;
  std::vector<long long> off_;
  size_t ntot_ = 0, nmax_ = 0;
  DBuf<long long> d_off_;
  DBuf<int> d_act_, kcnt_;
  DBuf<double> inv0_;
  DBuf<int> orows_, optr_, ocol_;
  DBuf<double> oval_;
  int onrows_ = 0;
  // outer FGMRES
  int outer_cap_ = 0, ldh_ = 0, onblk_ = 1;
  size_t hst_ = 0, rst_ = 0, opst_ = 0;
  DBuf<double> Vo_, Zo_, Ho_, cs_, sn_, g_, y_, est_, onorm_, osums_, ppart_, opa_, opb_, bp_, xb_, rr_;
  DBuf<double> io_in_, io_out_;
  double* pin_d_ = nullptr;
  int* pin_i_ = nullptr;
  // V-cycle graph
  bool use_graph_ = graphs_on();
  hipStream_t gstream_ = nullptr;
  hipGraph_t graph_ = nullptr;
  hipGraphExec_t gexec_ = nullptr;
  DBuf<double> vin_, vout_;

  static bool graphs_on() {
    const char* e = std::getenv("IBMG_GRAPH");
    return !(e && e[0] == '0');
  }
};

BatchBase* make_batch(int nsys, const ibmg_desc* d, hipStream_t s) {
  require(nsys >= 1 && d != nullptr, "nsys must be >= 1 and descs non-NULL");
  if (d[0].precision == IBMG_FP32_SMOOTHER) return new BatchSolver<float>(nsys, d, s);
  return new BatchSolver<double>(nsys, d, s);
}

}  // namespace ibmg
