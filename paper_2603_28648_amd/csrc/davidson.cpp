// Davidson eigensolver for the lowest eigenpair of H_eff (Davidson 1975) with
// the diagonal preconditioner and a precision ladder for the sigma products.
//
// Vectors live on the device in FP64; the subspace matrix (k <= 64) is filled
// and diagonalised there (rocSOLVER dsyevj), the Ritz vectors and the
// orthogonalisation take their coefficients from device memory, and a step
// waits for the host twice (eigenvalues and residual; norm of the correction).
// Buffers, solver handle and pinned results stay with the plan.  14 orbitals
// D = 256, six steps: 4.72 ms with a wait per dot product and buffers per
// call, now 3.08, of which 2.1 sigma.  The host has the eigenvectors for the
// restart combinations.  Each ladder stage
// uses one sigma precision until the residual norm drops below the stage
// threshold, reaches the floor that precision allows, or stalls; the
// subspace is then restarted from the current Ritz vector with sigma
// recomputed in the next precision.  The last stage is FP64, and the returned
// energy is the FP64 Rayleigh quotient.  With residual refinement, the FP64
// stage takes its correction vectors from inexact Jacobi-Davidson solves on
// the previous stage's precision (below).
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <vector>

#include <rocsolver/rocsolver.h>

#include "davidson.h"

namespace dmrg {

namespace {
// Relative error of a sigma product per precision, as measured against the
// FP64 sigma (split-BF16x3 1.3e-6 .. 1.4e-6 at CAS(22,22) and CAS(54,36);
// BF16 products carry 2^-8 per operand), with margin.
double sigma_rel_error(int precision) {
  switch (precision) {
    case 1: return 4e-3;   // BF16
    case 2: return 3e-6;   // split-BF16x3
    case 3: return 1e-13;  // Ozaki, 47 bits
    default: return 0.0;   // FP64
  }
}
constexpr double kFloorFactor = 3.0;
constexpr int kStallWindow = 10;
// Residual refinement: relative reduction of the correction equation's
// residual that ends an inner solve, and the inner iterations allowed.
constexpr double kRefineEta = 1e-2;
constexpr int kRefineInner = 60;
}  // namespace

void launch_extract_diag(const DiagTask* tasks, int ntasks, hipStream_t s);
void launch_heff_diag(double* out, int64_t rows, int dr, const int64_t* rowinfo, int64_t offR,
                      int npairs, const double* yd, const double* Ld, int64_t DL,
                      const double* Zd, int64_t DR, hipStream_t s);
void launch_precondition(double* t, const double* r, const double* d, double theta, int64_t n,
                         hipStream_t s);
void launch_ritz(double* u, double* w, double* r, const double* V, const double* W, int64_t n, int k, const double* y,
                 const double* theta, hipStream_t s);
void launch_olsen(double* t, const double* x, const double* c, int64_t n, hipStream_t s);
void launch_scale_to(double* y, double a, const double* x, int64_t n, hipStream_t s);
void launch_subspace(double* G, int kmax, const double* h, int c, double* A, hipStream_t s);
void launch_min(double* out, double* part, const double* x, int64_t n, hipStream_t s);

// ---- diagonal of H_eff (a sum over pairs with diagonal blocks) ------------
void build_diagonal(SigmaPlan& plan, const Bond& bl, const Bond& br, hipStream_t s) {
  const PsiLayout& ps = plan.psi;
  std::vector<int> use;
  for (size_t k = 0; k < plan.pairs.size(); ++k) {
    const SigmaPair& p = plan.pairs[k];
    if (!(p.L.lay->dq == QN{0, 0})) continue;
    if (p.z >= 0 && !(plan.zops[p.z].lay->dq == QN{0, 0})) continue;
    bool any = false;
    for (int n = 0; n < 16; ++n) any = any || p.y.m[n][n] != 0;
    if (any) use.push_back((int)k);
  }
  const int P = (int)use.size();
  const int64_t DL = bl.total, DR = br.total;
  DevBuf yd((size_t)std::max(1, P) * 16 * sizeof(double));
  DevBuf Ld((size_t)std::max<int64_t>(1, (int64_t)P * DL) * sizeof(double));
  DevBuf Zd((size_t)std::max<int64_t>(1, (int64_t)P * DR) * sizeof(double));
  launch_fill(Ld.as<double>(), 0.0, (int64_t)P * DL, s);
  launch_fill(Zd.as<double>(), 0.0, (int64_t)P * DR, s);
  std::vector<double> hy((size_t)P * 16);
  std::vector<DiagTask> tasks;
  for (int q = 0; q < P; ++q) {
    const SigmaPair& p = plan.pairs[use[q]];
    for (int n = 0; n < 16; ++n) hy[(size_t)q * 16 + n] = p.y.m[n][n];
    for (auto& b : p.L.lay->blk)
      if (b.r == b.c) tasks.push_back({p.L.data + b.off, Ld.as<double>() + (int64_t)q * DL + bl.off[b.c], b.dc, b.ld});
    if (p.z >= 0) {
      for (auto& b : plan.zops[p.z].lay->blk)
        if (b.r == b.c) tasks.push_back({plan.zops[p.z].data + b.off, Zd.as<double>() + (int64_t)q * DR + br.off[b.c], b.dc, b.ld});
    } else {
      launch_fill(Zd.as<double>() + (int64_t)q * DR, 1.0, DR, s);
    }
  }
  DMRG_HIP(hipMemcpy(yd.p, hy.data(), hy.size() * sizeof(double), hipMemcpyHostToDevice));
  DevBuf dt((size_t)std::max<size_t>(1, tasks.size()) * sizeof(DiagTask));
  DMRG_HIP(hipMemcpy(dt.p, tasks.data(), tasks.size() * sizeof(DiagTask), hipMemcpyHostToDevice));
  launch_extract_diag(dt.as<DiagTask>(), (int)tasks.size(), s);
  // row info: (global left state, site index n) of every psi row
  std::vector<int64_t> rowinfo;
  std::vector<int64_t> rowbase(br.size(), 0);
  for (size_t r = 0; r < br.size(); ++r) {
    rowbase[r] = (int64_t)rowinfo.size();
    std::vector<int64_t> rows(ps.rows_of[r] * 2, 0);
    for (auto& kv : ps.row_of[r]) {
      const int l = kv.first.first, n = kv.first.second;
      for (int a = 0; a < bl.d[l]; ++a) {
        rows[2 * (kv.second + a)] = bl.off[l] + a;
        rows[2 * (kv.second + a) + 1] = n;
      }
    }
    rowinfo.insert(rowinfo.end(), rows.begin(), rows.end());
  }
  DevBuf ri((size_t)std::max<size_t>(1, rowinfo.size()) * sizeof(int64_t));
  DMRG_HIP(hipMemcpy(ri.p, rowinfo.data(), rowinfo.size() * sizeof(int64_t), hipMemcpyHostToDevice));
  plan.diag.alloc((size_t)std::max<int64_t>(1, ps.size) * sizeof(double));
  for (size_t r = 0; r < br.size(); ++r) {
    if (ps.rows_of[r] == 0) continue;
    launch_heff_diag(plan.diag.as<double>() + ps.off[r], ps.rows_of[r], br.d[r],
                     ri.as<int64_t>() + rowbase[r], br.off[r], P, yd.as<double>(),
                     Ld.as<double>(), DL, Zd.as<double>(), DR, s);
  }
  DMRG_HIP(hipStreamSynchronize(s));
}

namespace {
// What a solve needs besides the plan: kept with the plan between its calls
// (a window's calls have the same sizes), the vectors up to kKeepBytes.
constexpr size_t kKeepBytes = (size_t)256 << 20;
constexpr int kMaxSubspace = 64;
struct DavidsonWork {
  DevBuf buf;              // vectors, then scalars
  double* host = nullptr;  // pinned: a step's results
  rocblas_handle h = nullptr;
  hipEvent_t e0 = nullptr, e1 = nullptr;  // around a sigma
  DavidsonWork() {
    DMRG_HIP(hipHostMalloc(reinterpret_cast<void**>(&host), kHost * sizeof(double)));
    DMRG_HIP(hipEventCreate(&e0));
    DMRG_HIP(hipEventCreate(&e1));
    DMRG_REQUIRE(rocblas_create_handle(&h) == rocblas_status_success, kErrHip,
                 "davidson: rocblas_create_handle failed");
  }
  ~DavidsonWork() {
    if (h) rocblas_destroy_handle(h);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (host) (void)hipHostFree(host);
  }
  // scalars: eigenvalues, 4 dots, solver info (2 int32) and residual, the
  // subspace matrix (then its eigenvectors) | G, coefficients, partial minima
  static constexpr int kEv = 0, kDot = kMaxSubspace, kInfo = kDot + 4, kRes = kInfo + 1, kA = kRes + 1,
                       kHost = kA + kMaxSubspace * kMaxSubspace, kG = kHost, kC = kG + kMaxSubspace * kMaxSubspace,
                       kPart = kC + 2 * kMaxSubspace, kScalars = kPart + 1024;
};
}  // namespace

static double now_ms() {
  return std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

int davidson(SigmaPlan& plan, double* psi, const DavidsonOpts& o, DavidsonResult& res,
             hipStream_t s) {
  const int64_t n = plan.psi.size;
  DMRG_REQUIRE(n > 0, kErrShape, "davidson: empty window");
  const int kmax = std::max(3, std::min(o.max_subspace, 64));
  const double t_start = now_ms();
  res = DavidsonResult();
  if (!plan.davidson_work) plan.davidson_work = std::make_shared<DavidsonWork>();
  DavidsonWork& wk = *static_cast<DavidsonWork*>(plan.davidson_work.get());
  struct Trim {
    DavidsonWork& wk;
    ~Trim() {
      if (wk.buf.bytes > kKeepBytes) wk.buf.release();
    }
  } trim{wk};
  const int64_t np = (n + 31) / 32 * 32;
  const size_t need = ((size_t)2 * kmax * n + 5 * np + 32 + DavidsonWork::kScalars) * sizeof(double);
  if (wk.buf.bytes < need) wk.buf.alloc(need);
  DMRG_REQUIRE(rocblas_set_stream(wk.h, s) == rocblas_status_success, kErrHip,
               "davidson: rocblas_set_stream failed");
  double* sc = wk.buf.as<double>();
  double *u = sc + DavidsonWork::kScalars, *w = u + np, *r = w + np, *t = r + np;
  double* aux = t + n;  // right behind t: both are dotted with u in one launch
  double *V = t + 2 * np, *W = V + (int64_t)kmax * n;
  double *ev_d = sc + DavidsonWork::kEv, *h = sc + DavidsonWork::kC, *cc = h + kMaxSubspace, *A = sc + DavidsonWork::kA;
  const double* d = plan.diag.as<double>();
  bool sigma_pending = false;
  auto sync = [&]() {
    DMRG_HIP(hipStreamSynchronize(s));
    if (!sigma_pending) return;
    float ms = 0;
    DMRG_HIP(hipEventElapsedTime(&ms, wk.e0, wk.e1));
    res.sigma_ms += ms;
    sigma_pending = false;
  };
  auto read = [&](const double* src, int count) {  // into wk.host
    DMRG_HIP(hipMemcpyAsync(wk.host, src, (size_t)count * sizeof(double), hipMemcpyDeviceToHost, s));
    sync();
  };
  DevBuf tmpV, tmpW;
  std::vector<double> ev, Y;
  auto dot = [&](const double* a, const double* b) {
    launch_multidot(h, a, 0, 1, b, n, s);
    read(h, 1);
    return wk.host[0];
  };
  auto sigma = [&](const double* x, double* y, int prec) {
    if (sigma_pending) sync();
    DMRG_HIP(hipEventRecord(wk.e0, s));
    run_sigma(plan, x, y, prec, s);
    DMRG_HIP(hipEventRecord(wk.e1, s));
    sigma_pending = true;
    res.n_sigma[prec]++;
  };
  // column k of G against all previous basis vectors, G[i][k] = V_i . W_k, and
  // G's leading part for the subspace eigenproblem
  auto fill_col = [&](int k) {
    launch_multidot(h, V, n, k + 1, W + (int64_t)k * n, n, s);
    launch_subspace(sc + DavidsonWork::kG, kmax, h, k, A, s);
  };
  // u, w, r of the lowest Ritz pair of the k x k subspace problem; its
  // eigenvalues ascending in ev, eigenvector j in column j of Y, |r|^2
  auto ritz = [&](int k) {
    // cyclic Jacobi (one small-matrix kernel); tolerance: machine precision
    rocblas_int* info = reinterpret_cast<rocblas_int*>(sc + DavidsonWork::kInfo);
    DMRG_REQUIRE(rocsolver_dsyevj(wk.h, rocblas_esort_ascending, rocblas_evect_original, rocblas_fill_upper,
                                  k, A, k, 0.0, sc + DavidsonWork::kRes, 100, info + 1, ev_d,
                                  info) == rocblas_status_success,
                 kErrHip, "davidson: rocsolver_dsyevj failed");
    launch_ritz(u, w, r, V, W, n, k, A, ev_d, s);
    launch_multidot(sc + DavidsonWork::kDot, r, 0, 1, r, n, s);
    read(sc, DavidsonWork::kA + k * k);
    DMRG_REQUIRE(*reinterpret_cast<const rocblas_int*>(wk.host + DavidsonWork::kInfo) == 0, kErrHip,
                 "davidson: subspace eigensolver did not converge");
    ev.assign(wk.host, wk.host + k);
    Y.resize((size_t)k * k);
    for (int i = 0; i < k; ++i)
      for (int j = 0; j < k; ++j) Y[(size_t)i * k + j] = wk.host[DavidsonWork::kA + (size_t)j * k + i];
    return wk.host[DavidsonWork::kDot];
  };
  auto orthogonalise = [&](int k) {  // t against the first k basis vectors, twice
    for (int pass = 0; pass < 2; ++pass) {
      launch_multidot(h, V, n, k, t, n, s);
      launch_lincomb(t, V, n, k, h, n, 1.0, s, -1.0);
    }
  };
  // start: V0 = psi / |psi|
  launch_min(h + 1, sc + DavidsonWork::kPart, d, n, s);
  launch_multidot(h, psi, 0, 1, psi, n, s);
  read(h, 2);
  const double nrm = std::sqrt(wk.host[0]), dmin = wk.host[1];
  DMRG_REQUIRE(nrm > 0 && std::isfinite(nrm), kErrInvalidArg, "davidson: psi has zero or non-finite norm");
  launch_scale_to(V, 1.0 / nrm, psi, n, s);
  int stage = 0;
  const bool verbose = std::getenv("DMRG_VERBOSE") != nullptr;  // one progress line per iteration
  const int nst = std::max(1, o.n_ladder);
  auto prec_of = [&](int st) { return o.n_ladder > 0 ? o.ladder[st] : 0; };
  // Residual refinement after a reduced-precision stage (Jacobi-Davidson
  // with inexact inner solves): the FP64 stage keeps its Davidson subspace,
  // FP64 sigma products and Rayleigh-Ritz, but each correction vector t
  // solves the correction equation
  //   (1 - u u^T)(H - theta)(1 - u u^T) t = -r,  t orthogonal to u,
  // for the Ritz pair (theta, u) and FP64 residual r, by conjugate gradients
  // on the reduced-precision sigma with the diagonal preconditioner
  // (diag(H_eff) - theta, projected), to a relative residual of kRefineEta
  // (looser when |r| is within a few times tol).
  // The reduced-precision error limits how much each correction gains, not
  // the attainable residual, which the FP64 products set.
  DevBuf cgb;
  auto inner_cg = [&](double* x, int lp, double theta_, int& iters_) {
    if (!cgb.p) cgb.alloc((size_t)4 * n * sizeof(double));
    double* rs = cgb.as<double>();  // residual of the correction equation
    double* z = rs + n;             // preconditioned residual
    double* p = z + n;              // search direction
    double* q = p + n;              // projected (H - theta) p
    auto project = [&](double* v) { launch_axpy(v, -dot(u, v), u, n, s); };
    const bool below_ = theta_ < dmin;
    auto precond = [&]() {  // z = P (diag - theta)^-1 rs, or P rs
      if (o.precondition > 0 && below_) {
        launch_precondition(z, rs, d, theta_, n, s);
        launch_scale(z, -1.0, n, s);
      } else {
        DMRG_HIP(hipMemcpyAsync(z, rs, n * sizeof(double), hipMemcpyDeviceToDevice, s));
      }
      project(z);
    };
    DMRG_HIP(hipMemsetAsync(x, 0, n * sizeof(double), s));
    DMRG_HIP(hipMemcpyAsync(rs, r, n * sizeof(double), hipMemcpyDeviceToDevice, s));
    launch_scale(rs, -1.0, n, s);
    project(rs);
    precond();
    DMRG_HIP(hipMemcpyAsync(p, z, n * sizeof(double), hipMemcpyDeviceToDevice, s));
    double rz = dot(rs, z);
    const double r0 = std::sqrt(std::max(0.0, dot(rs, rs)));
    // near the target a looser solve suffices: the correction needs to cut
    // the residual only to a fraction of tol
    const double eta = std::max(kRefineEta, std::min(0.5, 0.3 * o.tol / std::max(r0, 1e-300)));
    for (int it = 0; it < kRefineInner && iters_ < o.max_iter; ++it) {
      ++iters_;
      sigma(p, q, lp);
      launch_axpy(q, -theta_, p, n, s);
      project(q);
      const double pq = dot(p, q);
      if (!(pq > 0) || !(rz > 0)) break;  // the projected operator is not positive here
      const double alpha = rz / pq;
      launch_axpy(x, alpha, p, n, s);
      launch_axpy(rs, -alpha, q, n, s);
      const double rsn = std::sqrt(std::max(0.0, dot(rs, rs)));
      if (verbose)
        fprintf(stderr, "[dmrg] refinement inner %d (precision %d): relative residual %.3e\n", it, lp,
                rsn / r0);
      if (rsn < eta * r0) break;
      precond();
      const double rz1 = dot(rs, z);
      launch_scale(p, rz1 / rz, n, s);
      launch_axpy(p, 1.0, z, n, s);
      rz = rz1;
    }
  };
  int refine_lp = -1;  // reduced precision of the inner solves, once refining
  sigma(V, W, prec_of(stage));
  int k = 1;
  fill_col(0);
  double theta = 0, rnorm = 1e300;
  std::vector<double> hist;
  int iters = 0;
  bool converged = false;
  while (true) {
    rnorm = std::sqrt(std::max(0.0, ritz(k)));
    theta = ev[0];
    if (verbose)
      fprintf(stderr, "[dmrg] davidson iteration %d stage %d (precision %d): theta %.12f residual %.3e\n",
              iters, stage, prec_of(stage), theta, rnorm);
    hist.push_back(rnorm);
    res.residual_history.push_back(rnorm);
    res.stage_history.push_back(stage);
    const bool last = stage == nst - 1;
    const double thr = last ? o.tol : o.ladder_tol[stage];
    // A reduced-precision stage ends at its threshold, near the residual
    // floor its sigma error sets (kFloorFactor times the relative sigma
    // error times |theta|: an inexact sigma cannot give a smaller residual),
    // or when the residual has not dropped by 10% in kStallWindow iterations.
    // A short stall window ends stages early on the plateaus of slow
    // convergence (measured at CAS(54,36): with a 3-iteration window the FP64
    // stage did 224 of 236 iterations; floor factors 10, 3 and 1.5 gave
    // 178, 169 and 173 s to solution against 236 s for FP64 alone).
    bool stalled = false;
    if (!last) {
      const double floor_abs = kFloorFactor * sigma_rel_error(prec_of(stage)) * std::fabs(theta);
      stalled = rnorm < floor_abs;
      if (hist.size() > (size_t)kStallWindow)
        stalled = stalled || rnorm > 0.9 * hist[hist.size() - 1 - kStallWindow];
    }
    if (rnorm < thr || stalled) {
      if (last) { converged = rnorm < o.tol; break; }
      // next ladder stage: restart from the Ritz vector with a fresh sigma
      ++stage;
      hist.clear();
      if (o.refine && stage == nst - 1 && prec_of(stage - 1) != 0) refine_lp = prec_of(stage - 1);
      const double un = std::sqrt(dot(u, u));
      launch_scale_to(V, 1.0 / un, u, n, s);
      sigma(V, W, prec_of(stage));
      k = 1;
      fill_col(0);
      continue;
    }
    if (iters >= o.max_iter) break;
    ++iters;
    // correction t = r / (theta - diag), orthogonalised twice against V.
    // (theta - diag)^-1 is a useful preconditioner only once theta is below
    // the whole diagonal: while theta lies inside its range some
    // denominators pass through zero and the correction is dominated by
    // the few components where diag ~ theta, so those steps take t = r.
    const bool below = theta < dmin;
    double tn0 = 0;
    if (refine_lp >= 0) {
      inner_cg(t, refine_lp, theta, iters);
      tn0 = std::sqrt(std::max(0.0, dot(t, t)));
    }
    if (refine_lp >= 0 && tn0 > 0) {
      // correction from the inner solve
    } else if (o.precondition == 2 && below) {
      // Olsen: t = M^-1 (r - eps u), eps = u.M^-1 r / u.M^-1 u, M = theta - diag;
      // removes the component of M^-1 r along the Ritz vector that makes the
      // plain correction degenerate when diag(H_eff) is a good approximation
      launch_precondition(t, r, d, theta, n, s);
      launch_precondition(aux, u, d, theta, n, s);
      launch_multidot(h, t, n, 2, u, n, s);
      launch_olsen(t, aux, h, n, s);
    } else if (o.precondition == 1 && below) {
      launch_precondition(t, r, d, theta, n, s);
    } else {
      DMRG_HIP(hipMemcpyAsync(t, r, n * sizeof(double), hipMemcpyDeviceToDevice, s));
    }
    orthogonalise(k);
    double tn = std::sqrt(dot(t, t));
    if (k == kmax || !(tn > 1e-14)) {
      // thick restart: keep the m lowest Ritz vectors (V Y_m, W Y_m)
      const int m = std::min(k, std::max(1, std::min(o.restart, kmax - 1)));
      std::vector<int> order(k);
      for (int i = 0; i < k; ++i) order[i] = i;
      std::sort(order.begin(), order.end(), [&](int a, int b) { return ev[a] < ev[b]; });
      if (tmpV.bytes < (size_t)m * n * sizeof(double)) {
        tmpV.alloc((size_t)m * n * sizeof(double));
        tmpW.alloc((size_t)m * n * sizeof(double));
      }
      for (int j = 0; j < m; ++j) {
        std::vector<double> yj(k);
        for (int i = 0; i < k; ++i) yj[i] = Y[(size_t)i * k + order[j]];
        DMRG_HIP(hipMemcpyAsync(cc, yj.data(), k * sizeof(double), hipMemcpyHostToDevice, s));
        launch_lincomb(tmpV.as<double>() + (int64_t)j * n, V, n, k, cc, n, 0.0, s);
        launch_lincomb(tmpW.as<double>() + (int64_t)j * n, W, n, k, cc, n, 0.0, s);
        DMRG_HIP(hipStreamSynchronize(s));
      }
      DMRG_HIP(hipMemcpyAsync(V, tmpV.p, (size_t)m * n * sizeof(double), hipMemcpyDeviceToDevice, s));
      DMRG_HIP(hipMemcpyAsync(W, tmpW.p, (size_t)m * n * sizeof(double), hipMemcpyDeviceToDevice, s));
      k = m;
      for (int j = 0; j < m; ++j) fill_col(j);
      // re-orthogonalise t against the restarted basis
      orthogonalise(k);
      tn = std::sqrt(dot(t, t));
      if (!(tn > 1e-14)) continue;
    }
    launch_scale_to(V + (int64_t)k * n, 1.0 / tn, t, n, s);
    sigma(V + (int64_t)k * n, W + (int64_t)k * n, prec_of(stage));
    fill_col(k);
    ++k;
  }
  // final FP64 Rayleigh quotient of the normalised Ritz vector
  const double un = std::sqrt(dot(u, u));
  launch_scale(u, 1.0 / un, n, s);
  sigma(u, w, 0);
  res.energy = dot(u, w);
  DMRG_HIP(hipMemcpyAsync(r, w, n * sizeof(double), hipMemcpyDeviceToDevice, s));
  launch_axpy(r, -res.energy, u, n, s);
  res.residual = std::sqrt(std::max(0.0, dot(r, r)));
  DMRG_HIP(hipMemcpyAsync(psi, u, n * sizeof(double), hipMemcpyDeviceToDevice, s));
  sync();
  res.iterations = iters;
  res.converged = converged || res.residual < o.tol;
  res.time_ms = now_ms() - t_start;
  return res.converged ? kOk : kWarnNotConverged;
}

}  // namespace dmrg
