// Batched periodic solver of eq. (iter) (Sec. 4.2): per-incidence
// periodizer set-up, the operator (I + A_else A_0^+ - B Q^+ C A_0^+) applied
// to a batch of right-hand sides, and the pieces of the recovery.  Used by
// mfs_solve_incident (one batch) and by the serving loop (a fixed pool of
// slots that incident waves enter and leave between GMRES iterations).
#pragma once

#include <algorithm>
#include <cmath>
#include <complex>
#include <memory>
#include <vector>

#include "capi_impl.hpp"
#include "gpinv.hpp"

namespace mfs {

// launch_dft with the input rows ld_in apart and the output bins ldo apart
// (ldo <= 0: X)
void launch_dft_ld(int nr, int P, int X, const double2 *in, size_t ld_in, double2 *out, int sgn,
                   double scale, hipStream_t s, int ldo = 0);

using cplx = std::complex<double>;

// Expansions from this many times the bytes of one wave's matrices in stored
// kernel values on (below, few waves would gain too: 112 MB stored against 57.5
// MB a wave 7.9 -> 5.5 ms for one wave, 17.0 -> 16.8 for 16).
constexpr double kExpMinRatio = 4.0;

// Time of an iteration's near-field sums in bytes at 3.5 TB/s, for the lockstep
// of W waves of a solve.  Stored values: 100 us a launch (one where the surface's
// mirror pairs fill whole tiles, `paired`, else two) and the values, 0.7 of their
// bytes, 1.6 times that above 8 waves; 0.16, 0.22 and 0.38 ms were measured for 289,
// 786 and 1468 MB and 8 waves, 0.25, 0.35 and 0.62 for 16.
inline double stored_cost(double stored, bool paired, int W) {
  return ((paired ? 350e6 : 700e6) + 0.7 * stored) * (W > 8 ? 1.6 : 1.0);
}
// Expansions: the waves' matrices, 0.132 ms for 470 MB, and a tenth of their build
// (ten iterations or so share it), the steps of the 3j recurrences for every eight
// waves: 1.0 ms for eight at degrees 39 and 44, 0.48 at 26 and 29, 0.7 and 0.38 for
// one or two (stored values are filled in 0.4 to 0.6 ms).
inline double expansion_cost(double bytes, int ps, int pt, int W) {
  const double groups = W <= 2 ? 0.6 : (W + 7) / 8;
  return W * bytes + 2.0 * groups * std::pow((double)ps * pt, 2) * std::min(ps, pt);
}

struct Solver {
  const mfs_op *op;
  BodyData &b;
  mfs_lattice lat;
  int W, P, M, N, MP, NH, NQmax, maxit;
  // the two halves of Q (internal.hpp): rows (4 M1^2, more where a half would
  // have more columns than that; zero rows then), leading dimension, columns
  int rows_h, ldq, NQh;
  int Mr, Nc;   // per-mode system rows and columns (2M x 2N for transmission)
  hipStream_t s;
  std::vector<cplx> al, be;
  std::vector<double> kv;
  std::vector<std::vector<RBOrder>> orders;
  // periodizer
  std::vector<DevBuf> Q;            // both halves of a wave's Q, one after the other
  DevBuf qflags, Bvals, Bvals_v, qnodes, qnrb;
  std::vector<MatDesc> h_qdescs;
  std::vector<int> qrank;           // kept rank of every half [2 W]
  GradedPinv gp;
  bool qreflect = false;            // let a full-rank Q keep its QR's reflectors instead of forming U = Q_1
  DevBuf QHW;                       // work of the reflector apply
  const MatDesc *qdesc = nullptr;   // Q^+ factors of every wave (default: gp's)
  size_t near_limit = SIZE_MAX;     // bound on the stored near field besides the operator's
  // plans
  NsumPlan psurf, pwalls;
  DevBuf wsurf, wwalls;
  // low-rank image blocks of the surface sums (when their stored values do not fit)
  std::shared_ptr<NearLowRank> lowrank;
  DevBuf LRW;
  // near field by spherical-wave expansions: tables, the waves' matrices G
  // and their descriptors, moments, products (regular coefficients, then the
  // right-hand sides of Q^+) and partial products
  std::unique_ptr<NearExpansion> ex;
  DevBuf EG, EW, EM, EO, EP;
  int ldo = 0;
  // work
  DevBuf V, Z, XIN, C, SIG, GS, GH, WR, CY, XIH, XI, PART, PART2, YW, H1;
  int nsplit_s = 1, nsplit_w = 1;
  // timing: events around every neighbour-sum launch, the dense bytes each streamed
  std::vector<hipEvent_t> nsum_ev;
  std::vector<double> nsum_bytes, nsum_alg_bytes;
  // where the neighbour sums' kernel values come from: 0 evaluated on the fly
  // (near-field budget 0), 1 stored, 2 on the fly because the stored field
  // did not fit the budget or the free device memory, 3 low-rank image blocks,
  // 4 expansions
  int near_mode = 0;
  bool time_nsum = true;
  double near_fill_ms = 0.0;

  Solver(const mfs_op *o, BodyData &body, const mfs_lattice &l, int nw, int mi, hipStream_t st)
      : op(o), b(body), lat(l), W(nw), maxit(mi), s(st) {
    P = b.P; M = b.M; N = b.N; Mr = b.rows; Nc = b.cols; MP = P * Mr;
    NH = (lat.p + 1) * (lat.p + 1);
    NQmax = NQh = rows_h = ldq = 0;
  }
  // sizes of the halves for waves of at most nrb Rayleigh-Bloch orders
  void size_halves(int nrb) {
    NQmax = NH + 2 * nrb;
    NQh = half_cols(lat.p, 0) + nrb;
    rows_h = std::max(4 * lat.M1 * lat.M1, NQh);
    ldq = round_up(rows_h, 16);
  }
  ~Solver() {
    for (auto e : nsum_ev) (void)hipEventDestroy(e);
  }

  void setup_periodizer(double rel_cutoff) {
    std::vector<double> wall, nodes;
    wall_nodes(lat, wall);
    half_nodes(lat.M1, wall, nodes);
    qnodes.alloc(nodes.size() * sizeof(double));
    upload(qnodes.p, nodes.data(), nodes.size() * sizeof(double), s);
    const int NM = 2 * W;
    qflags.alloc((size_t)2 * NM * sizeof(int));
    int *flags = qflags.as<int>();
    Q.resize(W);
    h_qdescs.resize(NM);
    int nrbmax = 0;
    for (int w = 0; w < W; ++w) {
      const int nrb = (int)orders[w].size();
      nrbmax = std::max(nrbmax, nrb);
      MFS_REQUIRE(NH + 2 * nrb <= 8 * lat.M1 * lat.M1, "periodizer: Q has more columns than rows (raise M1)");
    }
    size_halves(nrbmax);
    std::vector<DevBuf> ordbufs(W);
    std::vector<QFillArgs> qargs(W);
    for (int w = 0; w < W; ++w) {
      const int nrb = (int)orders[w].size();
      const int nc[2] = {half_cols(lat.p, 0) + nrb, half_cols(lat.p, 1) + nrb};
      Q[w].alloc((size_t)ldq * (nc[0] + nc[1]) * sizeof(double2));
      QFillArgs a{};
      for (int par = 0; par < 2; ++par) {
        MatDesc d{};
        d.a = Q[w].as<double2>() + (par ? (size_t)ldq * nc[0] : 0);
        d.m = rows_h; d.n = nc[par]; d.lda = ldq;
        d.rank = flags + NM + 2 * w + par;
        h_qdescs[2 * w + par] = d;
        a.Q[par] = d.a;
      }
      // Rayleigh-Bloch data
      std::vector<double> kx(nrb), ky(nrb);
      std::vector<double2> kz(nrb);
      for (int o = 0; o < nrb; ++o) {
        kx[o] = orders[w][o].kx;
        ky[o] = orders[w][o].ky;
        kz[o] = cz(orders[w][o].kz.real(), orders[w][o].kz.imag());
      }
      ordbufs[w].alloc((size_t)std::max(1, nrb) * (2 * sizeof(double) + sizeof(double2)));
      double2 *kzd = ordbufs[w].as<double2>();
      double *kxd = reinterpret_cast<double *>(kzd + nrb);
      double *kyd = kxd + nrb;
      if (nrb > 0) {
        upload(kxd, kx.data(), nrb * sizeof(double), s);
        upload(kyd, ky.data(), nrb * sizeof(double), s);
        upload(kzd, kz.data(), nrb * sizeof(double2), s);
      }
      a.nrb = nrb;
      a.alpha = cz(al[w].real(), al[w].imag());
      a.beta = cz(be[w].real(), be[w].imag());
      a.kx = kxd; a.ky = kyd; a.kz = kzd;
      a.ldq = ldq;
      qargs[w] = a;
    }
    launch_qfill(qargs, lat.p, lat.M1, rows_h, b.k, qnodes.as<double>(), s);
    progress("periodizer: Q filled for %d waves, two halves of %d x %d at most; factoring", W, rows_h, NQh);
    // Q's columns equilibrated: the harmonics of high degree are smaller than
    // the low ones by far more than the cutoff on the walls, and would
    // otherwise be dropped whatever their use
    graded_pinv(gp, h_qdescs, rel_cutoff, s, true, qreflect, true);
    
    qrank = gp.kept;
    progress("periodizer: factored (%s; %d of %d halves again by column steps; Jacobi %.0f ms, %d launches)",
             gp.direct ? "full rank, no SVD"
             : gp.cod  ? "pivoted triangle, truncated complete orthogonal decomposition"
                       : "pivoted triangle",
             gp.redone, NM, gp.jacobi_ms, gp.jacobi_launches);
  }

  // Take the near field from expansions where they converge and the point
  // sums are long enough for them to pay.  A solve weighs its waves' matrices and
  // their build against stored values, where those would fit: on the small body
  // (N = 40, P = 24, M1 = 20) 2, 4, 8 and 16 waves take 5.9, 7.6, 10.3 and 16.6 ms
  // with expansions, 7.2, 8.0, 9.9 and 15.3 ms with stored values; with one of
  // radius 0.22 (23 MB a wave for 59) 16 waves 13.2 and 14.5; at k = 10 eight 19
  // and 65.  A server's waves come and go one by one and do not (`lockstep`
  // false): expansions are ahead in every case tried, 0.95 of the time a wave at
  // 8 slots on the small body, 0.82 at 1.9 times the bytes.  So the form a wave's
  // sums take depends on how many waves come with it, and on the memory left for
  // their matrices: its results are the same to rounding alone and in any batch.
  // MFS_NEAR_EXPANSION: 0 never, 1 by this rule (default), 2 wherever they converge.
  bool setup_expansion(bool lockstep) {
    const char *e = std::getenv("MFS_NEAR_EXPANSION"), *lr = std::getenv("MFS_NEAR_LOWRANK");
    const int mode = e ? std::atoi(e) : 1;
    const uint64_t budget = std::min<uint64_t>(op->near_budget, (uint64_t)near_limit);
    if (mode == 0 || budget == 0 || (lr && std::atoi(lr) == 2)) return false;
    std::unique_ptr<NearExpansion> x(new NearExpansion);
    if (!x->plan(b, lat)) return false;
    const size_t free_bytes = device_free_bytes(), spare = (size_t)2 << 30;
    const size_t room = std::min<uint64_t>(budget, free_bytes > spare ? free_bytes - spare : 0);
    // values a stored near field would read per iteration (mirror pairs once)
    const double S = (double)P * N;
    const double stored = 16.0 * S * (4.0 * MP + 30.0 * lat.M1 * lat.M1);
    if (mode == 1) {
      if (stored < kExpMinRatio * x->bytes_read) return false;
      const bool paired = (P / 2 * M) % 64 == 0;
      // (twice: without the pairing, and the padding of the tiles)
      if (lockstep && 2.0 * stored <= (double)room &&
          stored_cost(stored, paired, W) < expansion_cost(x->bytes_read, x->x.ps, x->x.pt, W))
        return false;
    }
    if ((size_t)W * x->wave_elems * sizeof(double2) > room) return false;
    ex = std::move(x);
    return true;
  }

  // the matrices of the waves ks (slots of this solver), phases al, be
  void build_expansion(const std::vector<int> &ks, const std::vector<cplx> &a, const std::vector<cplx> &bb,
                       hipStream_t st) const {
    std::vector<ExpWave> h;
    for (size_t i = 0; i < ks.size(); ++i) h.push_back(exp_wave(ks[i], a[i], bb[i]));
    ex->build(h, st);
  }
  ExpWave exp_wave(int k, cplx a, cplx bb) const {
    ExpWave v{};
    v.alpha = cz(a.real(), a.imag());
    v.beta = cz(bb.real(), bb.imag());
    v.G[0] = EG.as<double2>() + (size_t)k * ex->wave_elems;
    v.G[1] = v.G[0] + (size_t)ex->x.ldg * half_cols(ex->pm, 0);
    return v;
  }
  // descriptors of the waves an iteration applies (live[w] = 0: skipped)
  void upload_expansion(const std::vector<char> &live) {
    std::vector<ExpWave> h(W);
    for (int w = 0; w < W; ++w)
      if (live[w]) h[w] = exp_wave(w, al[w], be[w]);
    upload(EW.p, h.data(), W * sizeof(ExpWave), s);
  }

  void setup_sums(bool build_waves = true) {
    if (setup_expansion(build_waves)) {
      hipEvent_t f0, f1;
      HIP_CHECK(hipEventCreate(&f0));
      HIP_CHECK(hipEventCreate(&f1));
      HIP_CHECK(hipEventRecord(f0, s));
      ex->setup(b, lat, s);
      ldo = ex->x.row0 + rows_h;
      EG.alloc((size_t)W * ex->wave_elems * sizeof(double2));
      EW.alloc((size_t)W * sizeof(ExpWave));
      EM.alloc((size_t)2 * W * ex->ldx * sizeof(double2));
      EO.alloc((size_t)2 * W * ldo * sizeof(double2));
      if (ex->splits(W) > 1) EP.alloc((size_t)ex->splits(W) * 2 * W * ldo * sizeof(double2));
      if (build_waves) {
        std::vector<int> ks(W);
        for (int w = 0; w < W; ++w) ks[w] = w;
        build_expansion(ks, al, be, s);
      }
      upload_expansion(std::vector<char>(W, build_waves ? 1 : 0));
      HIP_CHECK(hipEventRecord(f1, s));
      HIP_CHECK(hipEventSynchronize(f1));
      float ms = 0.f;
      HIP_CHECK(hipEventElapsedTime(&ms, f0, f1));
      near_fill_ms = ms;
      near_mode = 4;
      (void)hipEventDestroy(f0);
      (void)hipEventDestroy(f1);
      work_buffers();
      return;
    }
    setup_bvals();
    surface_plan(b, psurf, s);
    walls_plan(lat, b.P, b.N, pwalls, s);
    std::vector<double2> w1, w2;
    image_weights(al, be, psurf, w1);
    walls_weights(al, be, pwalls, w2);
    wsurf.alloc(w1.size() * sizeof(double2));
    upload(wsurf.p, w1.data(), w1.size() * sizeof(double2), s);
    wwalls.alloc(w2.size() * sizeof(double2));
    upload(wwalls.p, w2.data(), w2.size() * sizeof(double2), s);
    const int S = P * N;
    nsplit_s = nsum_splits(psurf, S);
    nsplit_w = nsum_splits(pwalls, S);
    // dense near field, surface first (the larger share of the iteration)
    const uint64_t near_budget = std::min<uint64_t>(op->near_budget, (uint64_t)near_limit);
    if (near_budget > 0) {
      hipEvent_t f0, f1;
      HIP_CHECK(hipEventCreate(&f0));
      HIP_CHECK(hipEventCreate(&f1));
      HIP_CHECK(hipEventRecord(f0, s));
      const size_t budget = (size_t)std::min<uint64_t>(near_budget, (uint64_t)SIZE_MAX);
      if (nsum_build_dense(psurf, b.k, lat.ex, lat.ey, b.src_P.as<double>(), S, budget, s))
        nsum_build_dense(pwalls, b.k, lat.ex, lat.ey, b.src_P.as<double>(), S, budget - psurf.dense_bytes, s);
      HIP_CHECK(hipEventRecord(f1, s));
      HIP_CHECK(hipEventSynchronize(f1));
      float ms = 0.f;
      HIP_CHECK(hipEventElapsedTime(&ms, f0, f1));
      near_fill_ms = (psurf.dense.p || pwalls.dense.p) ? ms : 0.0;
      near_mode = (psurf.dense.p && pwalls.dense.p) ? 1 : 2;
      if (near_mode == 2)
        progress("near field: %s stored; the other sums run on the fly (budget or free memory too small)",
                 psurf.dense.p ? "surface sums" : "nothing");
      (void)hipEventDestroy(f0);
      (void)hipEventDestroy(f1);
    }
    // Surface sums from low-rank factors of the image blocks when their
    // stored values did not fit (MFS_NEAR_LOWRANK: 0 never, 1 then
    // (default), 2 whenever the surface values are not stored).  The factors
    // depend on the body and the lattice only and stay with the operator.
    {
      const char *e = std::getenv("MFS_NEAR_LOWRANK");
      const int mode = e ? std::atoi(e) : 1;
      if (!psurf.dense.p && !b.trans() && W <= 16 && mode > 0 && (near_mode == 2 || mode == 2)) {
        auto &c = b.lowrank;
        if (!(c && c->ex == lat.ex && c->ey == lat.ey && c->k == b.k && c->P == P && c->M == M && c->N == N)) {
          c.reset();
          c = build_near_lowrank(b, psurf, lat.ex, lat.ey, s);
          near_fill_ms = c ? c->build_ms : 0.0;
        } else {
          near_fill_ms = 0.0;
        }
        lowrank = c;
        if (lowrank) {
          LRW.alloc(lowrank_work_bytes(*lowrank, W));
          near_mode = 3;
          progress("near field: surface sums from low-rank image blocks (%.2f GB, built in %.0f ms)",
                   lowrank->bytes / 1e9, lowrank->build_ms);
        }
      }
    }
    // work buffers of the point sums
    SIG.alloc((size_t)W * P * N * sizeof(double2));
    GS.alloc((size_t)W * psurf.ntarget_pad * sizeof(double2));
    GH.alloc((size_t)W * MP * sizeof(double2));
    WR.alloc((size_t)W * pwalls.ntarget_pad * sizeof(double2));
    CY.alloc((size_t)2 * W * rows_h * sizeof(double2));
    const size_t part = std::max((size_t)nsplit_s * W * psurf.ntarget_pad, (size_t)nsplit_w * W * pwalls.ntarget_pad);
    PART.alloc(part * sizeof(double2));
    // the wall sums' slices when they run in the surface sums' launch
    if (nsum_pair_fusable(psurf, pwalls, b.k, b.src_P.as<double>(), P * N, W))
      PART2.alloc((size_t)nsplit_w * W * pwalls.ntarget_pad * sizeof(double2));
    work_buffers();
  }

  void work_buffers() {
    V.alloc((size_t)W * (maxit + 1) * MP * sizeof(double2));
    Z.alloc((size_t)W * MP * sizeof(double2));
    XIN.alloc((size_t)W * MP * sizeof(double2));
    C.alloc((size_t)W * P * Nc * sizeof(double2));
    XIH.alloc((size_t)2 * W * NQh * sizeof(double2));
    XI.alloc((size_t)W * NQmax * sizeof(double2));
    qnrb.alloc((size_t)W * sizeof(int));
    upload_orders();
    YW.alloc(std::max((size_t)b.nd * 2 * W * Nc, (size_t)2 * W * NQh) * sizeof(double2));
    H1.alloc((size_t)W * (maxit + 2) * 2 * sizeof(double2));
  }

  const MatDesc *qpinv_descs() const { return qdesc ? qdesc : gp.apply_descs(); }

  // number of Rayleigh-Bloch orders of every wave (after a wave changes)
  void upload_orders() {
    std::vector<int> n(W);
    for (int w = 0; w < W; ++w) n[w] = (int)orders[w].size();
    upload(qnrb.p, n.data(), W * sizeof(int), s);
  }

  // XIH = Q^+ y for every wave, half by half (y [2 W][ldy]): U^H then W, or,
  // when the factorisation kept the QR's reflectors in place of U = Q_1 (the
  // direct form), Q^H from the reflectors panel by panel, then W
  void apply_qpinv(const double2 *y, int ldy) {
    PinvJob j{};
    j.mode = 1; j.nmat = 2 * W; j.P = P; j.nrhs = 1; j.ldx = ldy; j.ldo = NQh; j.maxcols = 1;
    j.maxr = NQh; j.maxm = rows_h; j.maxn = NQh;
    j.descs = qpinv_descs(); j.x = y; j.out = XIH.as<double2>(); j.ywork = YW.as<double2>();
    if (!qdesc && gp.reflect) {
      if (!QHW.p) QHW.alloc(qh_apply_work(2 * W, rows_h, ldy));
      // the reflector apply's work follows the input's stride
      launch_qh_apply(gp.qr_descs(), 2 * W, rows_h, NQh, gp.qr_nb, y, ldy, QHW.as<double2>(), YW.as<double2>(), NQh,
                      s);
      launch_pinv_apply_w(j, s);
    } else {
      launch_pinv_apply(j, s);
    }
  }
  void merge_xi() {
    launch_merge_xi(W, lat.p, NQmax, qnrb.as<int>(), XIH.as<double2>(), NQh, XI.as<double2>(), NQmax, s);
  }
  // XI = Q^+ of the wall sums WR
  void walls_to_xi() {
    launch_split_walls(W, lat.M1, WR.as<double2>(), CY.as<double2>(), rows_h, s);
    apply_qpinv(CY.as<double2>(), rows_h);
    merge_xi();
  }

  // EO = G (moments of the mode coefficients c), timed like a neighbour sum
  void expansion_sums(const double2 *c) {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (time_nsum) {
      HIP_CHECK(hipEventCreate(&e0));
      HIP_CHECK(hipEventCreate(&e1));
      HIP_CHECK(hipEventRecord(e0, s));
    }
    ex->moments(W, c, Nc, EM.as<double2>(), s);
    ex->apply(W, EW.as<ExpWave>(), EM.as<double2>(), EO.as<double2>(), ldo, EP.as<double2>(), s);
    if (time_nsum) {
      HIP_CHECK(hipEventRecord(e1, s));
      nsum_ev.push_back(e0);
      nsum_ev.push_back(e1);
      nsum_bytes.push_back(W * ex->bytes_read);
      nsum_alg_bytes.push_back(W * ex->bytes_read);
    }
  }

  // phase weights of the neighbour sums from al, be (after a wave changes)
  void upload_weights() {
    if (ex) return;
    std::vector<double2> w1, w2;
    image_weights(al, be, psurf, w1);
    walls_weights(al, be, pwalls, w2);
    upload(wsurf.p, w1.data(), w1.size() * sizeof(double2), s);
    upload(wwalls.p, w2.data(), w2.size() * sizeof(double2), s);
  }

  // B~ (the harmonics' Neumann data on the surface rings, and for a
  // transmission body their values), wave independent; for the point sums (the
  // expansions have tables of their own)
  void setup_bvals() {
    Bvals.alloc((size_t)NH * M * sizeof(double2));
    launch_bfill(M, lat.p, b.k, b.rho, b.z, b.nrho, b.nz, Bvals.as<double2>(), s, 0);
    if (b.trans()) {
      Bvals_v.alloc((size_t)NH * M * sizeof(double2));
      launch_bfill(M, lat.p, b.k, b.rho, b.z, b.nrho, b.nz, Bvals_v.as<double2>(), s, 1);
    }
  }

  // Recovery of the waves w with iters[w] > 0 from their GMRES coefficients
  // y[w] (eta~ = V y): eta = A_0^+ eta~, xi = -Q^+ C eta, and the field at the
  // targets (near sum of the q_field-node point sources + harmonics).
  // xi: host [W][NQmax]; u: host [W][ntargets].  Blocking.
  void recover(const double2 *Vb, size_t ldw, const std::vector<std::vector<cplx>> &y,
               const std::vector<int> &iters, const double *targets, int ntargets, int q_field,
               std::vector<double2> &xi, std::vector<double2> &u) {
    int kmax = 0;
    for (int w = 0; w < W; ++w) kmax = std::max(kmax, iters[w]);
    std::vector<double2> ny((size_t)W * std::max(kmax, 1), cz(0.0, 0.0));
    for (int w = 0; w < W; ++w)
      for (int i = 0; i < iters[w]; ++i) ny[(size_t)w * kmax + i] = cz(-y[w][i].real(), -y[w][i].imag());
    DevBuf X((size_t)W * MP * sizeof(double2)), Yd(ny.size() * sizeof(double2));
    launch_zero(X.as<double2>(), (long)W * MP, s);
    upload(Yd.p, ny.data(), ny.size() * sizeof(double2), s);
    if (kmax > 0) launch_update(W, kmax, MP, Vb, ldw, MP, X.as<double2>(), Yd.as<double2>(), kmax, s);
    pinv_A0(X.as<double2>(), C.as<double2>());
    c_then_qpinv(C.as<double2>());
    xi.assign((size_t)W * NQmax, cz(0.0, 0.0));
    HIP_CHECK(hipMemcpyAsync(xi.data(), XI.p, xi.size() * sizeof(double2), hipMemcpyDeviceToHost, s));
    u.assign((size_t)W * ntargets, cz(0.0, 0.0));
    if (ntargets > 0) {
      DevBuf srcf, sigf((size_t)W * q_field * b.N * sizeof(double2));
      source_points(b, q_field, srcf, s);
      launch_point_strengths(W, b.P, q_field, b.N, C.as<double2>(), sigf.as<double2>(), s, Nc);
      std::vector<double> u6((size_t)6 * ntargets, 0.0);
      for (int t = 0; t < ntargets; ++t)
        for (int k = 0; k < 3; ++k) u6[(size_t)6 * t + k] = targets[(size_t)3 * t + k];
      NsumPlan pu;
      user_plan(u6.data(), ntargets, 0, true, pu, s);
      std::vector<double2> wu;
      image_weights(al, be, pu, wu);
      DevBuf wud(wu.size() * sizeof(double2));
      upload(wud.p, wu.data(), wu.size() * sizeof(double2), s);
      const int Sf = q_field * b.N;
      const int ns = nsum_splits(pu, Sf);
      DevBuf ur((size_t)W * pu.ntarget_pad * (1 + ns) * sizeof(double2));
      launch_nsum(pu, W, b.k, lat.ex, lat.ey, srcf.as<double>(), Sf, sigf.as<double2>(), wud.as<double2>(),
                  ur.as<double2>(), ur.as<double2>() + (size_t)W * pu.ntarget_pad, s);
      DevBuf hf((size_t)W * ntargets * sizeof(double2)), tx((size_t)3 * ntargets * sizeof(double));
      launch_zero(hf.as<double2>(), (long)W * ntargets, s);
      upload(tx.p, targets, (size_t)3 * ntargets * sizeof(double), s);
      launch_harm_field(W, ntargets, tx.as<double>(), lat.p, b.k, XI.as<double2>(), NQmax, hf.as<double2>(), s);
      std::vector<double2> unear((size_t)W * pu.ntarget_pad), uh((size_t)W * ntargets);
      HIP_CHECK(hipMemcpyAsync(unear.data(), ur.p, unear.size() * sizeof(double2), hipMemcpyDeviceToHost, s));
      HIP_CHECK(hipMemcpyAsync(uh.data(), hf.p, uh.size() * sizeof(double2), hipMemcpyDeviceToHost, s));
      HIP_CHECK(hipStreamSynchronize(s));
      for (int w = 0; w < W; ++w)
        for (int t = 0; t < ntargets; ++t) {
          const double2 a = unear[(size_t)w * pu.ntarget_pad + t], h = uh[(size_t)w * ntargets + t];
          u[(size_t)w * ntargets + t] = cz(a.x - h.x, a.y - h.y);   // d = -xi_d
        }
    }
    HIP_CHECK(hipStreamSynchronize(s));
  }

  // Bragg amplitudes a = -xi_a, b = -xi_b of wave w, its orders and eps_flux
  void amplitudes(int w, const double2 *xw, mfs_result &r) const {
    const auto &o = orders[w];
    const int nrb = (int)o.size();
    r.q_rank = qrank.empty() ? 0 : qrank[2 * w] + qrank[2 * w + 1];
    r.nq_cols = NH + 2 * nrb;
    double flux = 0.0, kz00 = 0.0;
    for (int i = 0; i < nrb; ++i) {
      const double2 av = xw[NH + i];
      const double2 bv = xw[NH + nrb + i];
      if (r.m) r.m[i] = o[i].m;
      if (r.n) r.n[i] = o[i].n;
      if (r.kz) r.kz[i] = mfs_c128{o[i].kz.real(), o[i].kz.imag()};
      const cplx a(-av.x, -av.y), bcoef(-bv.x, -bv.y);
      if (r.a) r.a[i] = mfs_c128{a.real(), a.imag()};
      if (r.b) r.b[i] = mfs_c128{bcoef.real(), bcoef.imag()};
      if (o[i].kz.imag() == 0.0 && o[i].kz.real() > 0.0) {
        cplx bb = bcoef;
        if (o[i].m == 0 && o[i].n == 0) {
          bb += std::exp(cplx(0.0, -kv[3 * w + 2] * lat.z0));
          kz00 = o[i].kz.real();
        }
        flux += o[i].kz.real() * (std::norm(a) + std::norm(bb));
      }
    }
    r.eps_flux = std::fabs(flux - kz00);
  }

  void pinv_A0(const double2 *x, double2 *out) {
    PinvJob j{};
    j.mode = 0; j.nmat = b.nd; j.P = P; j.nrhs = W; j.maxcols = 2 * W; j.maxr = Nc; j.maxm = Mr; j.maxn = Nc;
    j.descs = b.descs.as<MatDesc>(); j.x = x; j.out = out; j.ywork = YW.as<double2>();
    launch_pinv_apply(j, s);
  }

  // neighbour sum of the point strengths in SIG over plan (weights w) into out
  void nsum(const NsumPlan &plan, const DevBuf &w, double2 *out) {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (time_nsum) {
      HIP_CHECK(hipEventCreate(&e0));
      HIP_CHECK(hipEventCreate(&e1));
      HIP_CHECK(hipEventRecord(e0, s));
    }
    launch_nsum(plan, W, b.k, lat.ex, lat.ey, b.src_P.as<double>(), P * N, SIG.as<double2>(), w.as<double2>(), out,
                PART.as<double2>(), s);
    if (time_nsum) {
      HIP_CHECK(hipEventRecord(e1, s));
      nsum_ev.push_back(e0);
      nsum_ev.push_back(e1);
      nsum_bytes.push_back((double)plan.dense_bytes);
      nsum_alg_bytes.push_back((double)plan.dense_alg_bytes);
    }
  }

  // the surface sums into GS and the wall sums into WR in one launch over
  // both stored fields, timed like one neighbour sum (bytes: both fields)
  void nsum_surface_and_walls() {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (time_nsum) {
      HIP_CHECK(hipEventCreate(&e0));
      HIP_CHECK(hipEventCreate(&e1));
      HIP_CHECK(hipEventRecord(e0, s));
    }
    launch_nsum_pair(psurf, wsurf.as<double2>(), GS.as<double2>(), PART.as<double2>(), pwalls,
                     wwalls.as<double2>(), WR.as<double2>(), PART2.as<double2>(), W, P * N, SIG.as<double2>(), s);
    if (time_nsum) {
      HIP_CHECK(hipEventRecord(e1, s));
      nsum_ev.push_back(e0);
      nsum_ev.push_back(e1);
      nsum_bytes.push_back((double)(psurf.dense_bytes + pwalls.dense_bytes));
      nsum_alg_bytes.push_back((double)(psurf.dense_alg_bytes + pwalls.dense_alg_bytes));
    }
  }

  // the surface sums of the point strengths in SIG from the low-rank image
  // blocks, timed like the direct sums (bytes: the factors streamed)
  void surface_sum_lowrank(double2 *out) {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (time_nsum) {
      HIP_CHECK(hipEventCreate(&e0));
      HIP_CHECK(hipEventCreate(&e1));
      HIP_CHECK(hipEventRecord(e0, s));
    }
    lowrank_apply(*lowrank, W, SIG.as<double2>(), wsurf.as<double2>(), out, psurf.ntarget_pad, LRW.p, s);
    if (time_nsum) {
      HIP_CHECK(hipEventRecord(e1, s));
      nsum_ev.push_back(e0);
      nsum_ev.push_back(e1);
      nsum_bytes.push_back((double)lowrank->bytes);
      nsum_alg_bytes.push_back((double)lowrank->bytes);
    }
  }

  // XI = Q^+ (C c) for mode coefficients in C
  void c_then_qpinv(const double2 *cmodes) {
    if (ex) {
      expansion_sums(cmodes);
      apply_qpinv(EO.as<double2>() + ex->x.row0, ldo);
      merge_xi();
      return;
    }
    launch_point_strengths(W, P, P, N, cmodes, SIG.as<double2>(), s, Nc);
    nsum(pwalls, wwalls, WR.as<double2>());
    walls_to_xi();
  }

  // out = (I + A_else A_0^+ - B Q^+ C A_0^+) x
  void apply_op(const double2 *x, double2 *out) {
    pinv_A0(x, C.as<double2>());
    if (ex) {
      expansion_sums(C.as<double2>());
      apply_qpinv(EO.as<double2>() + ex->x.row0, ldo);
      ex->local(W, EO.as<double2>(), ldo, XIH.as<double2>(), NQh, x, out, s);
      return;
    }
    launch_point_strengths(W, P, P, N, C.as<double2>(), SIG.as<double2>(), s, Nc);
    // both stored fields in one launch when they can (the wall rows read the
    // same strengths), else the surface sums now and the wall sums below
    const bool fused = !lowrank && PART2.p && nsum_pair_fusable(psurf, pwalls, b.k, b.src_P.as<double>(), P * N, W);
    if (fused) nsum_surface_and_walls();
    else if (lowrank) surface_sum_lowrank(GS.as<double2>());
    else nsum(psurf, wsurf, GS.as<double2>());
    if (!b.trans()) {
      launch_dft_ld(W, P, M, GS.as<double2>(), psurf.ntarget_pad, GH.as<double2>(), -1, 1.0 / P, s, M);
    } else {
      // values (second target group) into rows [0, M), normal derivatives into [M, 2M)
      launch_dft_ld(W, P, M, GS.as<double2>() + psurf.groups[1].t0, psurf.ntarget_pad, GH.as<double2>(), -1,
                    1.0 / P, s, Mr);
      launch_dft_ld(W, P, M, GS.as<double2>() + psurf.groups[0].t0, psurf.ntarget_pad, GH.as<double2>() + M, -1,
                    1.0 / P, s, Mr);
    }
    launch_axpby_op(W, MP, x, GH.as<double2>(), nullptr, out, s);
    // the wall rows reuse SIG computed above
    if (!fused) nsum(pwalls, wwalls, WR.as<double2>());
    walls_to_xi();
    if (!b.trans()) {
      launch_bapply(W, P, M, lat.p, Bvals.as<double2>(), XI.as<double2>(), NQmax, out, s, M);
    } else {
      launch_bapply(W, P, M, lat.p, Bvals_v.as<double2>(), XI.as<double2>(), NQmax, out, s, Mr);
      launch_bapply(W, P, M, lat.p, Bvals.as<double2>(), XI.as<double2>(), NQmax, out + M, s, Mr);
    }
  }

  double nsum_avg_ms() {
    if (nsum_ev.empty()) return 0.0;
    double tot = 0.0;
    for (size_t i = 0; i + 1 < nsum_ev.size(); i += 2) {
      float ms = 0.f;
      HIP_CHECK(hipEventElapsedTime(&ms, nsum_ev[i], nsum_ev[i + 1]));
      tot += ms;
    }
    return tot / (nsum_ev.size() / 2);
  }
};


}  // namespace mfs
