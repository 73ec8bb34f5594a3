// Reverse mode of the two-site sigma with respect to the integrals.
//
// For fixed window vectors psi, lam and a fixed MPS, f = <lam, H_eff psi> is
// linear in (h, (pq|rs)); its gradient is the transition 1- and 2-RDM of the
// two full-space states the window vectors stand for (with lam = psi, the
// RDMs that orbital optimisation needs: dE/dh_pq = gamma_pq and
// dE/d(pq|rs) = Gamma_pqrs / 2).
//
// Every integral enters the sigma through exactly one component coefficient:
// of a block Hamiltonian, of a complementary operator, or of a window partial
// sum.  The operator such a coefficient multiplies is always an identity or a
// normal string, which does not depend on the integrals.  So, in reverse:
//   1. window: adjoints of the integral-dependent operators of the pairs,
//        L_bar[l',l] += y s * lam(l',n')[r'] . (Z psi^T)[r'](l,n)   (left)
//        U_bar = y s * L^T lam,  Z_bar[r',r] += a * U_bar^T psi(r)   (right)
//      and the partial sums' coefficient gradients <W_bar, x_L>;
//   2. along each chain, from the window outwards, the adjoint of
//      X -> Proj(X (x) y):
//        left  X_bar[l',l] += y s * A(l',n') N_bar[r',r] A(l,n)^T
//        right X_bar[r',r] += y s * B(l',n')^T N_bar[l',l] B(l,n)
//      carries the adjoints of block Hamiltonians and complementary
//      operators to the operators they were built from, and every
//      coefficient with integral dependence receives <N_bar_t, Proj(x (x) y)>.
// All contractions are grouped GEMMs of the forward's kernels: FP64, or the
// BF16 kernel (BF16 or split-BF16x3 products, FP32 accumulation flushed into
// FP64) for the mixed variant; the blocks are rebuilt in FP64 either way.
#include "backward.h"

#include <algorithm>
#include <array>
#include <chrono>
#include <set>
#include <tuple>

namespace dmrg {
namespace {

double now_ms() {
  return std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now().time_since_epoch())
      .count();
}

using Kinds = std::vector<std::vector<uint8_t>>;
Kinds kinds_of(const Env& e) {
  Kinds k(e.classes.size());
  for (size_t c = 0; c < e.classes.size(); ++c) k[c].assign((size_t)e.classes[c]->nops, 255);
  for (auto& kv : e.ops) k[kv.second.cls][kv.second.idx] = kv.first.kind;
  return k;
}
// Operators whose entries depend on the integrals.
bool dependent(uint8_t kind) { return kind == kHam || kind == kComp || kind == kPsum; }

// Adjoints of the operators of one block: one zeroed array per class.
struct Adj {
  ZeroedStore store;
  std::vector<DevSpan> cls;
  double* op(const Env& e, int c, int i) const {
    return cls[c].as<double>() + (int64_t)i * e.classes[c]->L.nnz;
  }
};
void alloc_adj(const Env& e, Adj& a, hipStream_t s) {
  std::vector<int64_t> n;
  for (auto& c : e.classes) n.push_back((int64_t)c->nops * c->L.nnz);
  a.cls = a.store.allocate(n, s);
}

void grow(DevBuf& b, size_t bytes, hipStream_t s) {
  if (b.bytes >= bytes) return;
  DMRG_HIP(hipStreamSynchronize(s));
  b.alloc(bytes);
}

// dst (old-bond operator, layout dl) += alpha * Proj^T(src, y), the adjoint
// of X -> Proj(X (x) y) applied to the new-bond operator src (layout sl).
// Same chunked two-stage scheme as the forward projections.
void run_adjoint_projections(int side, const Mps& m, int site, const std::vector<Projection>& projs,
                             DevBuf& desc, DevBuf& uws, int64_t budget, hipStream_t s) {
  const SiteTensor& st = m.site[site];
  const double* S = st.data.as<double>();
  const Bond& oldb = side > 0 ? m.bonds[site] : m.bonds[site + 1];
  const Bond& newb = side > 0 ? m.bonds[site + 1] : m.bonds[site];
  // visits every (dst block, n', n) term; f(tb, n', n, yv, idx...) with the
  // sector indices on both bonds
  struct Term {
    const Layout::Blk* tb;
    const Layout::Blk* xb;
    int n, np;
    double yv;
    int o0, o1;        // old-bond sectors (ket, bra)
    int w0, w1;        // new-bond sectors (ket, bra)
    int64_t s0, s1;    // site blocks (ket, bra)
  };
  auto visit = [&](const Projection& pr, auto&& f) {
    for (auto& tb : pr.dl->blk) {
      f.begin(tb);
      for (int n = 0; n < 4; ++n)
        for (int np = 0; np < 4; ++np) {
          const double yv = pr.y.m[np][n];
          if (yv == 0) continue;
          const int o0 = tb.c, o1 = tb.r;
          int w0, w1;
          if (side > 0) {
            w0 = newb.find(oldb.q[o0] + kSiteQN[n]);
            w1 = newb.find(oldb.q[o1] + kSiteQN[np]);
          } else {
            w0 = newb.find(oldb.q[o0] - kSiteQN[n]);
            w1 = newb.find(oldb.q[o1] - kSiteQN[np]);
          }
          if (w0 < 0 || w1 < 0) continue;
          const Layout::Blk* xb = pr.sl->col(w0);
          if (!xb || xb->r != w1) continue;
          const int64_t s0 = side > 0 ? st.off[4 * o0 + n] : st.off[4 * w0 + n];
          const int64_t s1 = side > 0 ? st.off[4 * o1 + np] : st.off[4 * w1 + np];
          if (s0 < 0 || s1 < 0) continue;
          f.term(Term{&tb, xb, n, np, yv, o0, o1, w0, w1, s0, s1});
        }
      f.end(tb);
    }
  };
  size_t p = 0;
  while (p < projs.size()) {
    int64_t need = 0;
    size_t q = p;
    for (; q < projs.size(); ++q) {
      struct {
        int64_t u = 0;
        const Bond *ob, *nb;
        void begin(const Layout::Blk&) {}
        void end(const Layout::Blk&) {}
        void term(const Term& t) {
          u += (int64_t)nb->d[t.w1] * ob->d[t.o0];
        }
      } sz;
      sz.ob = &oldb;
      sz.nb = &newb;
      visit(projs[q], sz);
      if (q > p && need + sz.u > budget) break;
      need += sz.u;
    }
    grow(uws, (size_t)std::max<int64_t>(need, 1) * sizeof(double), s);
    double* U = uws.as<double>();
    int64_t uoff = 0;
    GemmBatch b1, b2;
    for (size_t k = p; k < q; ++k) {
      const Projection& pr = projs[k];
      const int xpar = pr.dl->dq.n & 1;
      struct {
        GemmBatch *b1, *b2;
        const Projection* pr;
        const Bond *ob, *nb;
        const double* S;
        double* U;
        int64_t* uoff;
        int side, xpar;
        size_t s0 = 0;
        void begin(const Layout::Blk&) { s0 = b2->segs.size(); }
        void term(const Term& t) {
          double* u = U + *uoff;
          const size_t t0 = b1->segs.size();
          if (side > 0) {
            // old sectors l = o0, l' = o1; new sectors r = w0, r' = w1
            const int dl = ob->d[t.o0], dlp = ob->d[t.o1], dr = nb->d[t.w0], drp = nb->d[t.w1];
            *uoff += (int64_t)drp * dl;
            // u (r' x l) = N[r', r] A(l, n)^T
            b1->segs.push_back({pr->src + t.xb->off, S + t.s0, t.xb->ld, dr, dr, kTransB, 1.0});
            b1->add_problem(u, dl, drp, dl, t0, t0 + 1, 0);
            const double sg = ((pr->ypar & 1) && (ob->q[t.o0].n & 1)) ? -1.0 : 1.0;
            // X[l', l] += A(l', n') u
            b2->segs.push_back({S + t.s1, u, drp, dl, drp, 0, pr->alpha * t.yv * sg});
          } else {
            // old sectors r = o0, r' = o1; new sectors l = w0, l' = w1
            const int dr = ob->d[t.o0], drp = ob->d[t.o1], dl = nb->d[t.w0], dlp = nb->d[t.w1];
            *uoff += (int64_t)dlp * dr;
            // u (l' x r) = N[l', l] B(l, n)
            b1->segs.push_back({pr->src + t.xb->off, S + t.s0, t.xb->ld, dr, dl, 0, 1.0});
            b1->add_problem(u, dr, dlp, dr, t0, t0 + 1, 0);
            const double sg = (xpar && (kSiteN[t.n] & 1)) ? -1.0 : 1.0;
            // X[r', r] += B(l', n')^T u
            b2->segs.push_back({S + t.s1, u, drp, dr, dlp, kTransA, pr->alpha * t.yv * sg});
          }
        }
        void end(const Layout::Blk& tb) {
          b2->add_problem(pr->dst + tb.off, tb.ld, tb.dr, tb.dc, s0, b2->segs.size(), 1);
        }
      } em;
      em.b1 = &b1;
      em.b2 = &b2;
      em.pr = &pr;
      em.ob = &oldb;
      em.nb = &newb;
      em.S = S;
      em.U = U;
      em.uoff = &uoff;
      em.side = side;
      em.xpar = xpar;
      visit(pr, em);
    }
    launch_gemm(b1, desc, s);
    launch_gemm(b2, desc, s);
    p = q;
  }
}

const int64_t kProjBudget = (int64_t)1 << 27;  // doubles of projection intermediates per chunk
// A batch of component groups: doubles of its projections, and of its
// coefficients and downloaded products (a larger group is a batch by itself).
const int64_t kBatchBudget = (int64_t)1 << 26, kCoefBudget = (int64_t)1 << 24;


struct Work {
  DevBuf desc, uws, tmp, tmp2, coef, gout;
  std::vector<double> host;
};

// Downloads G (rows x cols) after the stream drains.
const std::vector<double>& fetch(Work& w, int64_t n, hipStream_t s) {
  w.host.resize((size_t)n);
  DMRG_HIP(hipStreamSynchronize(s));
  DMRG_HIP(hipMemcpy(w.host.data(), w.gout.p, (size_t)n * sizeof(double), hipMemcpyDeviceToHost));
  return w.host;
}

void upload(DevBuf& d, const std::vector<double>& h, hipStream_t s) {
  grow(d, std::max<size_t>(1, h.size()) * sizeof(double), s);
  DMRG_HIP(hipStreamSynchronize(s));
  DMRG_HIP(hipMemcpy(d.p, h.data(), h.size() * sizeof(double), hipMemcpyHostToDevice));
}

// C (m x n, ldc) = or += alpha * op(A) op(B) as one problem.  An empty
// contraction (k = 0, e.g. an operator class without blocks) still sets C = 0
// when beta = 0.
void gemm(void* c, int ldc, int m, int n, const void* a, int lda, const void* b, int ldb, int k,
          int flags, double alpha, int beta, DevBuf& desc, hipStream_t s) {
  if (m <= 0 || n <= 0) return;
  if (k <= 0) {
    if (!beta) {
      DMRG_REQUIRE(ldc == n, kErrState, "gemm: empty product into a strided output");
      launch_fill(static_cast<double*>(c), 0.0, (int64_t)m * n, s);
    }
    return;
  }
  GemmBatch g;
  g.segs.push_back({a, b, lda, ldb, k, flags, alpha});
  g.add_problem(c, ldc, m, n, 0, 1, beta);
  launch_gemm(g, desc, s);
}

// One renormalisation step backwards: the adjoints an of the new block's
// operators give the gradient of the step's coefficients and the adjoints
// (added to ao) of the old block's integral-dependent operators.
void step_back(const Mps& m, const Env& old, const Env& neu, const CompProv& rec, const Adj& an,
               Adj& ao, std::vector<double>& grad, Work& w, hipStream_t s, BackwardStats& stats) {
  const int side = neu.side;
  const int site = side > 0 ? old.bond : neu.bond;
  const Kinds ko = kinds_of(old), kn = kinds_of(neu);
  using Prov = std::vector<std::pair<int64_t, double>>;
  struct Source {
    int si;
    double coef;
    const Prov* prov;  // null: a source that depends on integrals itself
  };
  struct Group {
    std::map<int, std::vector<Source>> by_t;  // target -> sources
    std::set<int> srcs;
    int64_t coef = 0, gout = 0, proj = 0, x = 0;  // offsets in the batch's buffers (Shape)
  };
  std::map<std::tuple<int, uint64_t, int>, Group> groups;
  for (auto& kv : rec.coef) {
    int tc, ti, sc, si;
    uint64_t yk;
    std::tie(tc, ti, sc, si, yk) = kv.first;
    if (!dependent(kn[tc][ti])) continue;
    const bool dep = dependent(ko[sc][si]);
    const Prov* prov = nullptr;
    if (!dep) {
      auto it = rec.prov.find(kv.first);
      if (it == rec.prov.end()) continue;
      prov = &it->second;
    }
    if (dep && kv.second == 0.0) continue;
    Group& g = groups[std::make_tuple(tc, yk, sc)];
    g.by_t[ti].push_back({si, kv.second, prov});
    g.srcs.insert(si);
  }
  // Groups run in batches, each a handful of launches over all its groups:
  // the projections, the products on them, the projections of their results;
  // one upload of coefficients, one download of the products G that give the
  // gradient, and nothing in between waits for the host.
  struct Shape {
    const OpClass &T, &S;
    std::vector<int> prov, dep;  // sources by what they depend on
    bool adjoint_first;
    // doubles of the projections (M or P), X, coefficients and G
    int64_t proj, x, coef, gout;
  };
  auto shape = [&](const std::tuple<int, uint64_t, int>& key, const Group& g) {
    Shape h{*neu.classes[std::get<0>(key)], *old.classes[std::get<2>(key)], {}, {}, g.by_t.size() <= g.srcs.size(),
            0, 0, 0, 0};
    for (int si : g.srcs) (dependent(ko[std::get<2>(key)][si]) ? h.dep : h.prov).push_back(si);
    const int64_t nt = (int64_t)g.by_t.size(), np = (int64_t)h.prov.size(), nd = (int64_t)h.dep.size();
    if (h.adjoint_first) {
      h.proj = nt * h.S.L.nnz;
      h.gout = np ? nt * h.S.nops : 0;
      h.coef = nd ? nt * h.S.nops : 0;
    } else {
      h.proj = np * h.T.L.nnz;
      h.x = nd * h.T.L.nnz;
      h.gout = np * h.T.nops;
      h.coef = nd * h.T.nops;
    }
    return h;
  };
  for (auto g0 = groups.begin(); g0 != groups.end();) {
    std::vector<double> C;
    int64_t ng = 0, np = 0, nx = 0;
    auto g1 = g0;
    for (; g1 != groups.end(); ++g1) {
      Group& g = g1->second;
      const Shape h = shape(g1->first, g);
      if (g1 != g0 && ((int64_t)C.size() + h.coef > kCoefBudget || ng + h.gout > kCoefBudget ||
                       np + h.proj + nx + h.x > kBatchBudget))
        break;
      g.coef = (int64_t)C.size();
      g.gout = ng;
      g.proj = np;
      g.x = nx;
      ng += h.gout;
      np += h.proj;
      nx += h.x;
      C.resize(C.size() + (size_t)h.coef, 0.0);
      if (!h.coef) continue;
      std::map<int, int> dpos;
      for (int si : h.dep) dpos.emplace(si, (int)dpos.size());
      const size_t nt = g.by_t.size();
      size_t k = 0;
      for (auto& t : g.by_t) {
        for (const Source& e : t.second)
          if (!e.prov)
            C[(size_t)g.coef + (h.adjoint_first ? (size_t)e.si * nt + k
                                                : (size_t)dpos[e.si] * h.T.nops + (size_t)t.first)] += e.coef;
        ++k;
      }
    }
    upload(w.coef, C, s);
    grow(w.gout, (size_t)std::max<int64_t>(1, ng) * sizeof(double), s);
    grow(w.tmp, (size_t)std::max<int64_t>(1, np) * sizeof(double), s);
    grow(w.tmp2, (size_t)std::max<int64_t>(1, nx) * sizeof(double), s);
    launch_fill(w.tmp.as<double>(), 0.0, np, s);
    // adjoint first: M[k] = Proj^T(N_bar[t_k], y) on the old bond; project
    // first: P[k] = Proj(S[s_k], y) on the new one
    std::vector<Projection> adj, fwd, out;
    GemmBatch nt_prod, nn_prod;  // by operand orders
    std::map<int, std::vector<GemmSeg>> into;  // old class -> products added to all its adjoints
    for (auto it = g0; it != g1; ++it) {
      ++stats.n_groups;
      const int tc = std::get<0>(it->first), sc = std::get<2>(it->first);
      const Str ys = Str::from_key(std::get<1>(it->first));
      const Mat4 y = site_matrix(ys);
      const int ypar = ys.parity();
      const Group& g = it->second;
      const Shape h = shape(it->first, g);
      const OpClass &T = h.T, &S = h.S;
      const int64_t nnzS = S.L.nnz, nnzT = T.L.nnz;
      double* Pj = w.tmp.as<double>() + g.proj;
      double* X = w.tmp2.as<double>() + g.x;
      double* G = w.gout.as<double>() + g.gout;
      const double* Ct = w.coef.as<double>() + g.coef;
      auto product = [&](GemmBatch& b, double* c, int ldc, int m2, int n2, const double* a2, int lda, const double* b2,
                         int ldb, int k, int flags) {
        if (m2 <= 0 || n2 <= 0) return;
        if (k <= 0) {  // an empty contraction, e.g. an operator class without blocks
          launch_fill(c, 0.0, (int64_t)m2 * n2, s);
          return;
        }
        const size_t s0 = b.segs.size();
        b.segs.push_back({a2, b2, lda, ldb, k, flags, 1.0});
        b.add_problem(c, ldc, m2, n2, s0, s0 + 1, 0);
      };
      if (h.adjoint_first) {
        const int nt = (int)g.by_t.size();
        int k = 0;
        for (auto& t : g.by_t)
          adj.push_back({an.op(neu, tc, t.first), &T.L, y, ypar, Pj + (int64_t)(k++) * nnzS, &S.L, 1.0});
        // G (nt x nops_S) = M S^T
        if (!h.prov.empty())
          product(nt_prod, G, S.nops, nt, S.nops, Pj, (int)nnzS, S.data.as<double>(), (int)nnzS, (int)nnzS, kTransB);
        // ao[sc] (nops_S x nnz) += C^T M, C[k][s] = coefficient of (t_k, s)
        if (!h.dep.empty()) into[sc].push_back({Ct, Pj, nt, (int)nnzS, nt, 0, 1.0});
        continue;
      }
      for (size_t k = 0; k < h.prov.size(); ++k)
        fwd.push_back({S.op(h.prov[k]), &S.L, y, ypar, Pj + (int64_t)k * nnzT, &T.L, 1.0});
      // G (nops_T x np) = N_bar_T P^T
      if (!h.prov.empty())
        product(nt_prod, G, (int)h.prov.size(), T.nops, (int)h.prov.size(), an.cls[tc].as<double>(), (int)nnzT, Pj,
                (int)nnzT, (int)nnzT, kTransB);
      // X (nd x nnz_T) = C^T N_bar_T, then ao[s] += Proj^T(X_s, y)
      if (!h.dep.empty())
        product(nn_prod, X, (int)nnzT, (int)h.dep.size(), (int)nnzT, Ct, T.nops, an.cls[tc].as<double>(), (int)nnzT,
                T.nops, 0);
      for (size_t k = 0; k < h.dep.size(); ++k)
        out.push_back({X + (int64_t)k * nnzT, &T.L, y, ypar, ao.op(old, sc, h.dep[k]), &S.L, 1.0});
    }
    // (A list holds products of several groups, yet one group's per adjoint:
    // an operator that depends on integrals enters the new block through one
    // site string, the one that closes its open orbitals on the site, and the
    // other groups' coefficients of it are zero.  So no FP32 sum of the low
    // precisions runs over several groups.)
    for (auto& q : into) {
      const OpClass& S = *old.classes[q.first];
      const size_t s0 = nn_prod.segs.size();
      nn_prod.segs.insert(nn_prod.segs.end(), q.second.begin(), q.second.end());
      nn_prod.add_problem(ao.cls[q.first].p, (int)S.L.nnz, S.nops, (int)S.L.nnz, s0, nn_prod.segs.size(), 1);
    }
    run_adjoint_projections(side, m, site, adj, w.desc, w.uws, kProjBudget, s);
    run_projections(side, m, site, fwd, w.desc, w.uws, kProjBudget, s);
    launch_gemm(nt_prod, w.desc, s);
    launch_gemm(nn_prod, w.desc, s);
    // several groups may add to one operator: rounds of distinct targets
    std::stable_sort(out.begin(), out.end(), [](const Projection& x, const Projection& y) { return x.dst < y.dst; });
    std::vector<std::vector<Projection>> rounds;
    for (size_t k = 0; k < out.size();) {
      const size_t k0 = k;
      for (; k < out.size() && out[k].dst == out[k0].dst; ++k) {
        if (rounds.size() <= k - k0) rounds.emplace_back();
        rounds[k - k0].push_back(out[k]);
      }
    }
    for (auto& r : rounds) run_adjoint_projections(side, m, site, r, w.desc, w.uws, kProjBudget, s);
    const std::vector<double>& H = fetch(w, ng, s);
    for (auto it = g0; it != g1; ++it) {
      const Group& g = it->second;
      const Shape h = shape(it->first, g);
      std::map<int, int> ppos;
      for (int si : h.prov) ppos.emplace(si, (int)ppos.size());
      size_t k = 0;
      for (auto& t : g.by_t) {
        for (const Source& e : t.second) {
          if (!e.prov) continue;
          const double x = H[(size_t)g.gout + (h.adjoint_first ? k * h.S.nops + (size_t)e.si
                                                               : (size_t)t.first * ppos.size() + (size_t)ppos[e.si])];
          for (auto& pe : *e.prov) grad[(size_t)pe.first] += pe.second * x;
        }
        ++k;
      }
    }
    g0 = g1;
  }
}

// Window adjoints of the pairs' integral-dependent operators.
void window_back(const Mps& m, const SigmaPlan& plan, const Env& L, const Env& R, const double* lam_pad,
                 Adj& aL, Adj& aW, Adj& aR, int64_t budget, Work& w, hipStream_t s) {
  const int i = plan.window;
  const Bond& bl = m.bonds[i];
  const Bond& br = m.bonds[i + 2];
  const PsiLayout& ps = plan.psi;
  const Env& W = *plan.psums;
  const Kinds kL = kinds_of(L), kR = kinds_of(R);
  const double* Ppad = plan.bufs[plan.buf_psi].f64;
  const double* PT = plan.bufs[plan.buf_psit].f64;
  auto ldep = [&](const SigmaPair& p) {
    return p.lsrc == 1 || dependent(kL[p.lref.cls][p.lref.idx]);
  };
  auto zdep = [&](const SigmaPair& p) {
    return p.z >= 0 && dependent(kR[plan.zrefs[p.z].cls][plan.zrefs[p.z].idx]);
  };
  std::set<int> zl, zz;
  for (auto& p : plan.pairs) {
    if (ldep(p) && p.z >= 0) zl.insert(p.z);
    if (zdep(p)) zz.insert(p.z);
  }
  const int nz = (int)plan.zops.size();
  auto zsize = [&](int z) {
    int64_t n = 0;
    for (auto& blk : plan.zops[z].lay->blk)
      if (ps.rows_of[blk.c] > 0 && ps.rows_of[blk.r] > 0) n += ps.rows_pad[blk.c] * br.d[blk.r];
    return n;
  };
  // chunks over z (each z needs T (left-dependent pairs) and/or U_bar)
  std::vector<std::pair<int, int>> chunks;
  {
    int z0 = 0;
    int64_t acc = 0;
    for (int z = 0; z < nz; ++z) {
      const int64_t need = (zl.count(z) + zz.count(z)) * zsize(z);
      if (z > z0 && acc + need > budget) {
        chunks.push_back({z0, z});
        z0 = z;
        acc = 0;
      }
      acc += need;
    }
    chunks.push_back({z0, std::max(nz, z0 + 1)});
  }
  for (size_t ci = 0; ci < chunks.size(); ++ci) {
    const int z0 = chunks[ci].first, z1 = chunks[ci].second;
    std::map<std::pair<int, int>, int64_t> tloc, uloc;  // (z, r) -> ws offset (d_r' x rows_pad_r)
    int64_t off = 0;
    for (int z = z0; z < std::min(z1, nz); ++z)
      for (auto& blk : plan.zops[z].lay->blk) {
        const int r = blk.c, rp = blk.r;
        if (ps.rows_of[r] == 0 || ps.rows_of[rp] == 0) continue;
        const int64_t n = ps.rows_pad[r] * br.d[rp];
        if (zl.count(z)) { tloc[{z, r}] = off; off += n; }
        if (zz.count(z)) { uloc[{z, r}] = off; off += n; }
      }
    grow(w.tmp, (size_t)std::max<int64_t>(1, off) * sizeof(double), s);
    double* ws = w.tmp.as<double>();
    launch_fill(ws, 0.0, std::max<int64_t>(1, off), s);
    // B1: T^T[z, r] = a Z(r', r) psi_r^T   (as the forward's first stage)
    GemmBatch b1;
    for (auto& t : tloc) {
      const int z = t.first.first, r = t.first.second;
      const OpView& Z = plan.zops[z];
      const Layout::Blk* blk = Z.lay->col(r);
      const double alpha = (plan.zpar[z] && (br.q[r].n & 1)) ? -1.0 : 1.0;
      const size_t s0 = b1.segs.size();
      b1.segs.push_back({Z.data + blk->off, Ppad + ps.off_pad[r], blk->ld, ps.ld[r], br.d[r], kTransB, alpha});
      b1.add_problem(ws + t.second, (int)ps.rows_pad[r], br.d[blk->r], (int)ps.rows_pad[r], s0, s0 + 1, 0);
    }
    launch_gemm(b1, w.desc, s);
    // B2 (left adjoints) and B3 (U_bar), output-stationary
    struct Item {
      double* out;
      int m, n, ldc;
      GemmSeg g;
    };
    std::vector<Item> outL, outU;
    std::vector<std::tuple<int, int, double>> yv;
    for (auto& pr : plan.pairs) {
      const bool dl = ldep(pr) && (pr.z < 0 ? ci == 0 : (pr.z >= z0 && pr.z < z1));
      const bool dz = zdep(pr) && pr.z >= z0 && pr.z < z1;
      if (!dl && !dz) continue;
      const Layout& Ll = *pr.L.lay;
      const Env& LE = pr.lsrc ? W : L;
      const Adj& LA = pr.lsrc ? aW : aL;
      pr.y.nonzeros(yv);
      for (auto& y : yv)
        for (auto& lb : Ll.blk) {
          const int l = lb.c;
          const PsiLayout::RowGroup &k = ps.group[16 * l + std::get<1>(y)], &kp = ps.group[16 * lb.r + std::get<0>(y)];
          const int r = k.r, rp = kp.r;
          if (r < 0 || rp < 0) continue;
          if (pr.z >= 0) {
            const Layout::Blk* zb = plan.zops[pr.z].lay->col(r);
            if (!zb || zb->r != rp) continue;
          } else if (r != rp) {
            continue;
          }
          const double sg = ((pr.ypar & 1) && (bl.q[l].n & 1)) ? -1.0 : 1.0;
          const double* lamb = lam_pad + ps.off_pad[rp] + kp.row * ps.ld[rp];
          if (dl) {
            // L_bar[l', l] += lam(l', n') (d_l' x d_r') . T^T[z, r](:, (l, n)) (d_r' x d_l)
            const double* B = pr.z < 0 ? PT + ps.offT[r] + k.row : ws + tloc.at({pr.z, r}) + k.row;
            outL.push_back({LA.op(LE, pr.lref.cls, pr.lref.idx) + lb.off, lb.dr, lb.dc, lb.ld,
                            {lamb, B, ps.ld[rp], (int)ps.rows_pad[r], br.d[rp], 0, std::get<2>(y) * sg}});
          }
          if (dz) {
            // U_bar^T[z, r](:, (l, n)) += lam(l', n')^T (d_r' x d_l') . L[l', l]
            outU.push_back({ws + uloc.at({pr.z, r}) + k.row, br.d[rp], lb.dc, (int)ps.rows_pad[r],
                            {lamb, pr.L.data + lb.off, ps.ld[rp], lb.ld, lb.dr, kTransA, std::get<2>(y) * sg}});
          }
        }
    }
    GemmBatch b2;
    for (auto* o : {&outL, &outU}) {
      // by output, each output's products in the order found
      std::stable_sort(o->begin(), o->end(), [](const Item& x, const Item& y) { return x.out < y.out; });
      for (size_t q = 0; q < o->size();) {
        const Item& it = (*o)[q];
        const size_t s0 = b2.segs.size();
        for (; q < o->size() && (*o)[q].out == it.out; ++q) b2.segs.push_back((*o)[q].g);
        b2.add_problem(it.out, it.ldc, it.m, it.n, s0, b2.segs.size(), 1);
      }
    }
    launch_gemm(b2, w.desc, s);
    // B4: Z_bar[r', r] += a U_bar^T[z, r] psi_r
    GemmBatch b4;
    for (auto& u : uloc) {
      const int z = u.first.first, r = u.first.second;
      const OpRef& zr = plan.zrefs[z];
      const Layout::Blk* blk = plan.zops[z].lay->col(r);
      const double alpha = (plan.zpar[z] && (br.q[r].n & 1)) ? -1.0 : 1.0;
      const size_t s0 = b4.segs.size();
      b4.segs.push_back({ws + u.second, Ppad + ps.off_pad[r], (int)ps.rows_pad[r], ps.ld[r],
                         (int)ps.rows_pad[r], 0, alpha});
      b4.add_problem(aR.op(R, zr.cls, zr.idx) + blk->off, blk->ld, blk->dr, blk->dc, s0, s0 + 1, 1);
    }
    launch_gemm(b4, w.desc, s);
    DMRG_HIP(hipStreamSynchronize(s));
  }
}

}  // namespace

BackwardStats sigma_backward(const Problem& P0, const Mps& m, int window, const double* psi,
                             const double* lam, double* grad_out, int64_t ws_budget, hipStream_t s,
                             int precision) {
  BackwardStats st;
  const int K = P0.K, i = window;
  DMRG_REQUIRE(i >= 0 && i + 1 < K, kErrInvalidArg, "sigma_backward: bad window");
  Problem P = P0;
  P.all_terms = true;  // every integral entry is an input, zero or not
  std::vector<double> grad((size_t)K * K + (size_t)K * K * K * K, 0.0);
  Work w;
  // ---- rebuild both blocks, recording the components ----------------------
  double t0 = now_ms();
  std::vector<std::unique_ptr<Env>> Ls(i + 1), Rs(K + 1);
  std::vector<CompProv> recL(i + 1), recR(K + 1);
  Ls[0] = left_start(m, s);
  for (int b = 0; b < i; ++b) Ls[b + 1] = grow_left(P, m, *Ls[b], w.desc, s, &recL[b + 1]);
  Rs[K] = right_start(m, s);
  for (int b = K; b > i + 2; --b) Rs[b - 1] = grow_right(P, m, *Rs[b], w.desc, s, &recR[b - 1]);
  auto plan = plan_sigma(P, m, *Ls[i], *Rs[i + 2], ws_budget, s, true);
  DMRG_HIP(hipStreamSynchronize(s));
  st.ms_chain = now_ms() - t0;
  // ---- window ---------------------------------------------------------------
  // Every contraction from here on runs in the requested precision; the
  // gradient itself is accumulated in FP64 on the host.
  GemmPrecisionScope scope(precision);
  t0 = now_ms();
  const int64_t npad = plan->psi.size_pad;
  DevBuf lam_pad((size_t)std::max<int64_t>(1, npad) * sizeof(double));
  plan_load_psi(*plan, lam, s);
  DMRG_HIP(hipMemcpyAsync(lam_pad.p, plan->bufs[plan->buf_psi].f64, (size_t)npad * sizeof(double),
                          hipMemcpyDeviceToDevice, s));
  plan_load_psi(*plan, psi, s);
  std::vector<Adj> aL(i + 1), aR(K + 1);
  Adj aW;
  alloc_adj(*Ls[i], aL[i], s);
  alloc_adj(*Rs[i + 2], aR[i + 2], s);
  alloc_adj(*plan->psums, aW, s);
  window_back(m, *plan, *Ls[i], *Rs[i + 2], lam_pad.as<double>(), aL[i], aW, aR[i + 2], ws_budget, w, s);
  // partial sums: W = C x_L, so dC = W_bar x_L^T
  const Env& W = *plan->psums;
  for (auto& wc : plan->w_src_cls) {
    const OpClass& Wc = *W.classes[wc.first];
    const OpClass& Sc = *Ls[i]->classes[wc.second];
    const int64_t nnz = Wc.L.nnz;
    grow(w.gout, (size_t)std::max(1, Wc.nops * Sc.nops) * sizeof(double), s);
    gemm(w.gout.p, Sc.nops, Wc.nops, Sc.nops, aW.cls[wc.first].p, (int)nnz, Sc.data.p, (int)nnz, (int)nnz,
         kTransB, 1.0, 0, w.desc, s);
    const auto& G = fetch(w, (int64_t)Wc.nops * Sc.nops, s);
    for (auto& wk : plan->wkeys) {
      if (wk.second.cls != wc.first) continue;
      auto it = plan->psum_prov.find(wk.first);
      if (it == plan->psum_prov.end()) continue;
      for (auto& src : it->second)
        for (auto& pe : src.second)
          grad[(size_t)pe.first] += pe.second * G[(size_t)wk.second.idx * Sc.nops + src.first.second];
    }
  }
  DMRG_HIP(hipStreamSynchronize(s));
  plan.reset();
  st.ms_window = now_ms() - t0;
  // ---- adjoint renormalisation along both chains -------------------------------
  t0 = now_ms();
  for (int b = i; b >= 1; --b) {
    alloc_adj(*Ls[b - 1], aL[b - 1], s);
    step_back(m, *Ls[b - 1], *Ls[b], recL[b], aL[b], aL[b - 1], grad, w, s, st);
    aL[b] = Adj();
    Ls[b].reset();
  }
  for (int b = i + 2; b <= K - 1; ++b) {
    alloc_adj(*Rs[b + 1], aR[b + 1], s);
    step_back(m, *Rs[b + 1], *Rs[b], recR[b], aR[b], aR[b + 1], grad, w, s, st);
    aR[b] = Adj();
    Rs[b].reset();
  }
  DMRG_HIP(hipStreamSynchronize(s));
  st.ms_adjoint = now_ms() - t0;
  std::copy(grad.begin(), grad.end(), grad_out);
  return st;
}

}  // namespace dmrg

namespace dmrg {

void orbital_gradient(const Problem& P, const double* dh, const double* deri, double* fock,
                      double* grad, hipStream_t s) {
  const int K = P.K;
  const int64_t K2 = (int64_t)K * K, K3 = K2 * K;
  DMRG_REQUIRE(K3 < ((int64_t)1 << 31), kErrShape, "orbital_gradient: K^3 exceeds the GEMM index range");
  std::vector<double> eye((size_t)K2, 0.0);
  for (int p = 0; p < K; ++p) eye[(size_t)p * K + p] = 1.0;
  DevBuf dH((size_t)K2 * sizeof(double)), dE((size_t)(K3 * K) * sizeof(double)),
      dI((size_t)K2 * sizeof(double)), dF((size_t)K2 * sizeof(double)), desc;
  DMRG_HIP(hipMemcpyAsync(dH.p, P.h.data(), (size_t)K2 * sizeof(double), hipMemcpyHostToDevice, s));
  DMRG_HIP(hipMemcpyAsync(dE.p, P.eri.data(), (size_t)(K3 * K) * sizeof(double), hipMemcpyHostToDevice, s));
  DMRG_HIP(hipMemcpyAsync(dI.p, eye.data(), (size_t)K2 * sizeof(double), hipMemcpyHostToDevice, s));
  double* F = fock ? fock : dF.as<double>();
  // F = gamma h^T + (2 deri)(K x K^3) eri(K x K^3)^T
  GemmBatch f;
  f.segs.push_back({dh, dH.p, K, K, K, kTransB, 1.0});
  f.segs.push_back({deri, dE.p, (int)K3, (int)K3, (int)K3, kTransB, 2.0});
  f.add_problem(F, K, K, K, 0, 2, 0);
  launch_gemm_f64(f, s);
  // g = 2 F^T I - 2 F I
  GemmBatch g;
  g.segs.push_back({F, dI.p, K, K, K, kTransA, 2.0});
  g.segs.push_back({F, dI.p, K, K, K, 0, -2.0});
  g.add_problem(grad, K, K, K, 0, 2, 0);
  launch_gemm_f64(g, s);
  DMRG_HIP(hipStreamSynchronize(s));
}

}  // namespace dmrg
