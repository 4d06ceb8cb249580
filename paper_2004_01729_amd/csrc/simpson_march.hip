// Implicit integral form generated by Simpson's rule (Section III; Table
// tab:numerr and tab:timings, row "Simpson's"): on the uniform grid
// tau_y = y h, h = beta / n_g,
//     s_0 = 0,   s_y = - sum_{x <= y} G^y_x exp(-Delta (tau_y - tau_x)) S[s_x],
// each s_y solved by fixed-point sweeps with the earlier points fixed (G^y_y != 0:
// the implicit method of Section II.C), Omega_CC by Simpson's rule on the same
// grid; the adjoint of the discrete Lagrangian swept backward over the points.
// Storage: grid states s_y in sb[y], their residuals S[s_y] in abuf[y], Lambda
// of point y in lam[y] (y = 0..n_g); the executor has one slot per instance.
#include "api_internal.h"

namespace ftcc {
namespace host {

// C with G^y_x = h C[x] (x = 0..y): cumulative Simpson weights of int_0^{tau_y}.
// y even: composite Simpson (1/3)[1, 4, 2, ..., 4, 1]; y odd >= 3: composite Simpson
// on [0, tau_{y-3}] and the 3/8 rule (3/8)[1, 3, 3, 1] on the last three intervals;
// y = 1: the trapezoid (1/2)[1, 1].
std::vector<double> simpson_row(int y) {
  std::vector<double> C(y + 1, 0.0);
  if (y == 1) {
    C[0] = C[1] = 0.5;
    return C;
  }
  const int even = (y % 2 == 0) ? y : y - 3;
  for (int x = 0; even > 0 && x <= even; ++x) C[x] = ((x == 0 || x == even) ? 1.0 : (x % 2 ? 4.0 : 2.0)) / 3.0;
  if (y % 2) {
    const double w[4] = {1.0, 3.0, 3.0, 1.0};
    for (int k = 0; k < 4; ++k) C[y - 3 + k] += 3.0 * w[k] / 8.0;
  }
  return C;
}

// One exponential-sum launch over both amplitude segments of every instance
// (gated by the run flags).  The descriptor set is built from spec(i) on first
// use of `key` and kept until the next solve (h = beta / n_g may change).
void expsum_run(ftcc_ctx* c, long key, const std::function<ExpSpec(int)>& spec) {
  auto it = c->sp_cache.find(key);
  if (it == c->sp_cache.end()) {
    std::vector<ExpSumProblem> ps;
    std::vector<int> prefix;
    std::vector<std::vector<ExpTerm>> terms;
    int total = 0;
    for (int i = 0; i < c->B; ++i) {
      const ExpSpec sp = spec(i);
      const Instance& I = c->inst[i];
      const long n2 = (long)I.n * I.n;
      for (int seg = 0; seg < 2; ++seg) {
        const long off = seg ? n2 : 0;
        ExpSumProblem p;
        std::memset(&p, 0, sizeof(p));
        p.eps = I.eps;
        p.n = I.n;
        p.rank = seg ? 4 : 2;
        p.len = seg_len(c, i, seg);
        p.idx = I.d_allowed[seg];
        p.pack = c->packed_states ? (unsigned)I.n : 0u;
        p.h = I.beta / c->P;
        p.mode = sp.mode;
        p.base = sp.base ? sp.base + off : nullptr;
        p.x0 = sp.x0;
        p.prod = sp.prod ? sp.prod + off : nullptr;
        p.nterms = (int)sp.terms.size();
        p.out = sp.out + off;
        p.maxbits = sp.track ? c->d_maxbits + 2 * i : nullptr;
        p.active = c->d_run + i * c->slots;
        std::vector<ExpTerm> t;
        for (const auto& x : sp.terms) t.push_back(ExpTerm{std::get<0>(x) + off, std::get<1>(x), std::get<2>(x)});
        terms.push_back(t);
        prefix.push_back(total);
        total += (int)((p.len + 1023) / 1024);
        ps.push_back(p);
      }
    }
    size_t nterm = 0;
    for (const auto& t : terms) nterm += t.size();
    const size_t bytes = ps.size() * sizeof(ExpSumProblem) + prefix.size() * sizeof(int) + 64 +
                         std::max<size_t>(nterm, 1) * sizeof(ExpTerm);
    char* buf = nullptr;
    FTCC_HIP(hipMalloc((void**)&buf, bytes));
    ExpSumProblem* d_ps = (ExpSumProblem*)buf;
    int* d_pre = (int*)(buf + ps.size() * sizeof(ExpSumProblem));
    ExpTerm* d_terms = (ExpTerm*)(((uintptr_t)(d_pre + prefix.size()) + 63) / 64 * 64);
    size_t k = 0;
    for (size_t q = 0; q < ps.size(); ++q) {
      ps[q].terms = d_terms + k;
      if (!terms[q].empty())
        FTCC_LEGACY(hipMemcpy(d_terms + k, terms[q].data(), terms[q].size() * sizeof(ExpTerm), hipMemcpyHostToDevice));
      k += terms[q].size();
    }
    FTCC_LEGACY(hipMemcpy(d_ps, ps.data(), ps.size() * sizeof(ExpSumProblem), hipMemcpyHostToDevice));
    FTCC_LEGACY(hipMemcpy(d_pre, prefix.data(), prefix.size() * sizeof(int), hipMemcpyHostToDevice));
    it = c->sp_cache.emplace(key, SpLaunch{buf, (int)ps.size(), total}).first;
  }
  const SpLaunch& L = it->second;
  const ExpSumProblem* d_ps = (const ExpSumProblem*)L.buf;
  const int* d_pre = (const int*)(L.buf + L.n_prob * sizeof(ExpSumProblem));
  launch_expsum(d_ps, d_pre, L.n_prob, L.blocks, c->stream);
  FTCC_HIP(hipGetLastError());
}

long sp_key(int kind, int y) { return (long)kind * 1000000L + y; }

void simpson_solve(ftcc_ctx* c, std::vector<int>& status, std::vector<int>& total) {
  const int B = c->B, m = c->m, P = c->P;
  std::vector<double> ebuf((size_t)B * (P + 1), 0.0);
  std::vector<bool> ok(B);
  const auto wall0 = std::chrono::steady_clock::now();
  auto energy_to_host = [&](int y) {
    for (int i = 0; i < B; ++i)
      if (c->run_host[i])
        FTCC_HIP(hipMemcpyAsync(&ebuf[(size_t)i * (P + 1) + y], c->e[i * m], sizeof(double), hipMemcpyDeviceToHost,
                                c->stream));
  };
  // s_0 = 0 and its residual
  for (int i = 0; i < B; ++i) {
    zero_d(c, c->inst[i].sb[0], node_len(c, i));
    zero_d(c, c->amp[i * m], node_len(c, i));
  }
  run_all(c);
  forward_one(c, 0);
  for (int i = 0; i < B; ++i) node_copy(c, i, c->inst[i].abuf[0], c->S[i * m]);
  energy_to_host(0);
  for (int y = 1; y <= P; ++y) {
    const std::vector<double> C = simpson_row(y);
    for (int i = 0; i < B; ++i) ok[i] = status[i] == 0;
    set_run(c, ok);
    // the fixed part of point y: H = -sum_{x<y} G^y_x e^{-Delta h (y - x)} S_x
    expsum_run(c, sp_key(1, y), [c, y, &C](int i) {
      ExpSpec sp;
      for (int x = 0; x < y; ++x)
        if (C[x] != 0.0) sp.terms.emplace_back(c->inst[i].abuf[x], -C[x], (double)(y - x));
      sp.out = c->inst[i].rk_tmp[0];
      return sp;
    });
    // start from S_y ~ S_{y-1}
    expsum_run(c, sp_key(2, y), [c, y, &C](int i) {
      ExpSpec sp;
      sp.base = c->inst[i].rk_tmp[0];
      sp.x0 = 1.0;
      sp.terms.emplace_back(c->inst[i].abuf[y - 1], -C[y], 0.0);
      sp.out = c->amp[i * c->m];
      return sp;
    });
    std::vector<bool> active = ok;
    std::vector<DivergenceWatch> watch(B);
    for (int it = 1; it <= c->opt.max_iter; ++it) {
      set_run(c, active);
      forward_one(c, 0);
      reset_maxbits(c);
      expsum_run(c, sp_key(3, y), [c, &C, y](int i) {
        ExpSpec sp;
        sp.base = c->inst[i].rk_tmp[0];
        sp.x0 = 1.0;
        sp.terms.emplace_back(c->S[i * c->m], -C[y], 0.0);
        sp.out = c->amp[i * c->m];
        sp.track = true;
        return sp;
      });
      const std::vector<double> mb = read_maxbits(c);
      bool any = false;
      for (int i = 0; i < B; ++i) {
        if (!active[i]) continue;
        total[i] += 1;
        const double chg = mb[2 * i], val = mb[2 * i + 1];
        if (!std::isfinite(chg) || !std::isfinite(val)) {
          status[i] = FTCC_ENONFINITE;
          active[i] = false;
          continue;
        }
        if (chg <= c->opt.tol * std::max(1.0, val)) {
          active[i] = false;
          continue;
        }
        if (watch[i].diverged(chg)) {
          status[i] = FTCC_EDIVERGE;
          active[i] = false;
          continue;
        }
        any = true;
      }
      if (!any) break;
      if (it == c->opt.max_iter)
        for (int i = 0; i < B; ++i)
          if (active[i]) status[i] = FTCC_ENOCONV;
    }
    // the residual at the converged amplitudes, stored with the state
    for (int i = 0; i < B; ++i) ok[i] = status[i] == 0;
    set_run(c, ok);
    forward_one(c, 0);
    for (int i = 0; i < B; ++i) {
      if (!ok[i]) continue;
      node_copy(c, i, c->inst[i].sb[y], c->amp[i * m]);
      node_copy(c, i, c->inst[i].abuf[y], c->S[i * m]);
    }
    energy_to_host(y);
    if (trace_on()) {
      sync(c);
      trace(c, "forward (Simpson)", y, P, std::vector<int>(1, 0), wall0);
    }
  }
  run_all(c);
  sync(c);
  const std::vector<double> g = simpson_row(P);
  for (int i = 0; i < B; ++i) {
    Instance& I = c->inst[i];
    double om = 0.0;
    for (int y = 0; y <= P; ++y) {
      I.energies[y] = ebuf[(size_t)i * (P + 1) + y];
      om += g[y] / P * I.energies[y];   // (1/beta) G^{n_g}_y = C[y] / n_g
    }
    I.omega_cc = status[i] == 0 ? om : std::nan("");
    I.iters = total[i];
  }
}

// Backward over the points: lam_x = -(g_x/beta) dE/ds(s_x) - J_x^T lamt_x with
// lamt_x = sum_{y >= x} G^y_x e^{-Delta h (y - x)} lam_y (implicit through y = x),
// by fixed-point sweeps on lam_x; lam_0 = 0 (s_0 is not an unknown).
void simpson_lambda(ftcc_ctx* c, std::vector<int>& status, std::vector<int>& total) {
  const int B = c->B, m = c->m, P = c->P;
  std::vector<bool> ok(B);
  const auto wall0 = std::chrono::steady_clock::now();
  for (int i = 0; i < B; ++i) zero_d(c, c->inst[i].lam[0], node_len(c, i));
  for (int x = P; x >= 1; --x) {
    for (int i = 0; i < B; ++i) ok[i] = status[i] == 0;
    set_run(c, ok);
    // the later points' part of lamt_x
    expsum_run(c, sp_key(4, x), [c, x, P](int i) {
      ExpSpec sp;
      for (int y = x + 1; y <= P; ++y) {
        const double cy = simpson_row(y)[x];
        if (cy != 0.0) sp.terms.emplace_back(c->inst[i].lam[y], cy, (double)(y - x));
      }
      sp.out = c->inst[i].rk_tmp[1];
      return sp;
    });
    for (int i = 0; i < B; ++i) {
      if (!ok[i]) continue;
      node_copy(c, i, c->amp[i * m], c->inst[i].sb[x]);
      zero_d(c, c->inst[i].lam[x], node_len(c, i));
    }
    set_ebar(c, 0, x);
    forward(c);   // the tape at s_x, reused by every sweep below
    const double cxx = simpson_row(x)[x];
    std::vector<bool> active = ok;
    std::vector<DivergenceWatch> watch(B);
    for (int it = 1; it <= c->opt.max_iter; ++it) {
      set_run(c, active);
      expsum_run(c, sp_key(5, x), [c, x, cxx](int i) {   // cotangent of S at s_x: lamt_x
        ExpSpec sp;
        sp.base = c->inst[i].rk_tmp[1];
        sp.x0 = 1.0;
        sp.terms.emplace_back(c->inst[i].lam[x], cxx, 0.0);
        sp.out = c->cot[i * c->m];
        return sp;
      });
      backward(c);
      c->vjp_evals += n_running(c);
      reset_maxbits(c);
      expsum_run(c, sp_key(6, x), [c, x](int i) {          // lam_x = -gradient
        ExpSpec sp;
        sp.base = c->gr[i * c->m];
        sp.x0 = -1.0;
        sp.out = c->inst[i].lam[x];
        sp.track = true;
        return sp;
      });
      const std::vector<double> mb = read_maxbits(c);
      bool any = false;
      for (int i = 0; i < B; ++i) {
        if (!active[i]) continue;
        total[i] += 1;
        const double chg = mb[2 * i], val = mb[2 * i + 1];
        if (!std::isfinite(chg) || !std::isfinite(val)) {
          status[i] = FTCC_ENONFINITE;
          active[i] = false;
          continue;
        }
        if (chg <= c->opt.tol * std::max(val, 1e-30) || chg == 0.0) {
          active[i] = false;
          continue;
        }
        if (watch[i].diverged(chg)) {
          status[i] = FTCC_EDIVERGE;
          active[i] = false;
          continue;
        }
        any = true;
      }
      if (!any) break;
      if (it == c->opt.max_iter)
        for (int i = 0; i < B; ++i)
          if (active[i]) status[i] = FTCC_ENOCONV;
    }
    if (trace_on()) {
      sync(c);
      trace(c, "lambda (Simpson)", P - x + 1, P, std::vector<int>(1, 0), wall0);
    }
  }
  run_all(c);
}

// lamt_x of every instance into cot (all later points, the diagonal included)
void simpson_lamt(ftcc_ctx* c, int x) {
  const int P = c->P;
  expsum_run(c, sp_key(7, x), [c, x, P](int i) {
    ExpSpec sp;
    for (int y = std::max(x, 1); y <= P; ++y) {
      const double cy = simpson_row(y)[x];
      if (cy != 0.0) sp.terms.emplace_back(c->inst[i].lam[y], cy, (double)(y - x));
    }
    sp.out = c->cot[i * c->m];
    return sp;
  });
}

// sum_x d[G^y_x e^{-Delta h (y - x)}] S_x for point y into out (mode 1: d/dh, mode 2:
// d/dDelta); with prod, out = base + prod * (that sum)
void simpson_grid_term(ftcc_ctx* c, int y, int mode, const std::function<double*(int)>& out,
                       const std::function<const double*(int)>& prod) {
  const std::vector<double> C = simpson_row(y);
  expsum_run(c, sp_key(mode == 1 ? 8 : 9, y), [c, y, mode, &C, &out, &prod](int i) {
    ExpSpec sp;
    sp.mode = mode;
    for (int x = 0; x <= y; ++x)
      if (C[x] != 0.0) sp.terms.emplace_back(c->inst[i].abuf[x], C[x], (double)(y - x));
    sp.out = out(i);
    if (prod) {
      sp.prod = prod(i);
      sp.base = sp.out;
      sp.x0 = 1.0;
    }
    return sp;
  });
}

}  // namespace host
}  // namespace ftcc
