// Tensor-program engine: lowering of contractions to grouped kernel launches.
#include "engine.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <stdexcept>
#include <unordered_map>

#include "util.h"

namespace ftcc {

// ------------------------------------------------------------------ Program
int Program::tensor(const std::string& name, int rank, TensorKind kind) {
  for (size_t i = 0; i < t.size(); ++i)
    if (t[i].name == name) throw std::runtime_error("duplicate tensor " + name);
  t.push_back({name, rank, kind, false});
  return (int)t.size() - 1;
}

int Program::id(const std::string& name) const {
  for (size_t i = 0; i < t.size(); ++i)
    if (t[i].name == name) return (int)i;
  throw std::runtime_error("unknown tensor " + name);
}

void Program::op(const std::string& out, const std::string& oi, double alpha, const std::string& a,
                 const std::string& ai, const std::string& b, const std::string& bi, bool acc) {
  SymOp o;
  o.out = id(out);
  o.oi = oi;
  o.alpha = alpha;
  o.a = id(a);
  o.ai = ai;
  o.b = b.empty() ? -1 : id(b);
  o.bi = bi;
  o.accumulate = acc;
  if ((int)oi.size() != t[o.out].rank || (int)ai.size() != t[o.a].rank ||
      (o.b >= 0 && (int)bi.size() != t[o.b].rank))
    throw std::runtime_error("rank mismatch in op on " + out);
  o.setup = false;
  ops.push_back(o);
}

// An intermediate is derived (a constant combination) when every op writing it
// reads only constants or derived tensors; those ops form the set-up list.
void Program::set_law(const std::string& name, const std::vector<int>& signs) {
  const int k = id(name);
  if ((int)signs.size() != t[k].rank) throw std::runtime_error("law rank mismatch: " + name);
  if ((int)law.size() < (int)t.size()) law.resize(t.size());
  law[k] = signs;
}

void Program::finalize() {
  law.resize(t.size());
  for (auto& d : t) d.derived = false;
  bool changed = true;
  while (changed) {
    changed = false;
    for (size_t k = 0; k < t.size(); ++k) {
      if (t[k].kind != T_INTER || t[k].derived) continue;
      bool any = false, all_const = true;
      for (const SymOp& o : ops) {
        if (o.out != (int)k) continue;
        any = true;
        auto c = [&](int x) { return x < 0 || t[x].kind == T_CONST || t[x].derived; };
        if (!c(o.a) || !c(o.b)) all_const = false;
      }
      if (any && all_const) {
        t[k].derived = true;
        changed = true;
      }
    }
  }
  for (SymOp& o : ops) o.setup = t[o.out].derived;
  finalized_ = true;
}

// ------------------------------------------------------------------ helpers
static long ipow(long n, int r) {
  long v = 1;
  for (int k = 0; k < r; ++k) v *= n;
  return v;
}

static bool has(const std::string& s, char c) { return s.find(c) != std::string::npos; }

static std::string filter(const std::string& src, const std::string& a, const std::string& b, bool in_a,
                          bool in_b) {
  std::string out;
  for (char c : src)
    if (has(a, c) == in_a && has(b, c) == in_b) out.push_back(c);
  return out;
}

Executor::~Executor() {
  for (void* p : owned_) (void)hipFree(p);
}

void* Executor::upload(const void* host, size_t bytes) {
  constexpr size_t kFirst = (size_t)64 << 10, kLast = (size_t)4 << 20, kAlign = 256;
  if (bytes > kLast / 4) {
    void* d = nullptr;
    FTCC_HIP(hipMalloc(&d, bytes));
    owned_.push_back(d);
    FTCC_LEGACY(hipMemcpy(d, host, bytes, hipMemcpyHostToDevice));
    return d;
  }
  const size_t need = (std::max<size_t>(bytes, 8) + kAlign - 1) / kAlign * kAlign;
  if (chunks_.empty() || chunks_.back().host.size() + need > chunks_.back().size) {
    flush_uploads();
    Chunk c;
    // each twice the one before: at most half of a plan's chunks is left unused
    c.size = std::max(need, chunks_.empty() ? kFirst : std::min(kLast, 2 * chunks_.back().size));
    void* d = nullptr;
    FTCC_HIP(hipMalloc(&d, c.size));
    owned_.push_back(d);
    c.dev = (char*)d;
    c.host.reserve(c.size);
    chunks_.push_back(std::move(c));
  }
  Chunk& c = chunks_.back();
  const size_t at = c.host.size();
  c.host.resize(at + need);
  if (bytes) std::memcpy(c.host.data() + at, host, bytes);
  return c.dev + at;
}

void Executor::flush_uploads() {
  for (Chunk& c : chunks_) {
    if (c.flushed < c.host.size())
      FTCC_LEGACY(hipMemcpy(c.dev + c.flushed, c.host.data() + c.flushed, c.host.size() - c.flushed,
                         hipMemcpyHostToDevice));
    c.flushed = c.host.size();
  }
}

// The plan is complete: its tables are on the device, the host images are not needed.
void Executor::end_uploads() {
  flush_uploads();
  chunks_.clear();
  tuple_cache_.clear();
}

using Ranges = std::vector<std::pair<uintptr_t, uintptr_t>>;

static void add_range(Ranges& v, const void* p, size_t bytes) {
  if (p && bytes) v.emplace_back((uintptr_t)p, (uintptr_t)p + bytes);
}

// sorted, overlapping and touching ranges joined
static void normalize(Ranges& v) {
  if (v.empty()) return;
  std::sort(v.begin(), v.end());
  size_t w = 0;
  for (size_t k = 1; k < v.size(); ++k) {
    if (v[k].first <= v[w].second) v[w].second = std::max(v[w].second, v[k].second);
    else v[++w] = v[k];
  }
  v.resize(w + 1);
}

static bool overlaps(const Ranges& a, const Ranges& b) {
  size_t i = 0, j = 0;
  while (i < a.size() && j < b.size()) {
    if (a[i].second <= b[j].first) ++i;
    else if (b[j].second <= a[i].first) ++j;
    else return true;
  }
  return false;
}

// Which launches of a list lead to the memory in `needed`: a launch is kept if it writes
// what is needed, and what it reads is needed then.
static std::vector<char> leads_to(const std::vector<Launch>& L, Ranges needed) {
  std::vector<char> keep(L.size(), 0);
  normalize(needed);
  for (int i = (int)L.size() - 1; i >= 0; --i) {
    Ranges wr = L[i].wr;
    normalize(wr);
    if (!overlaps(wr, needed)) continue;
    keep[i] = 1;
    needed.insert(needed.end(), L[i].rd.begin(), L[i].rd.end());
    normalize(needed);
  }
  return keep;
}

// must b run after a (a earlier in program order)?
static bool ordered(const Launch& a, const Launch& b) {
  if (!a.ranged || !b.ranged) return true;
  return overlaps(a.wr, b.rd) || overlaps(a.wr, b.wr) || overlaps(a.rd, b.wr);
}

// Task of the first element of every `per`-element block of an element-task list
// (the largest task index whose first element is at or before it), and the last
// task after the final block: the kernels search only between two neighbours.
static std::vector<int> block_first_tasks(const std::vector<ElemTask>& tasks, long long total, int per) {
  const long long nb = (total + per - 1) / per;
  std::vector<int> bf((size_t)nb + 1);
  int t = 0;
  for (long long b = 0; b < nb; ++b) {
    while (t + 1 < (int)tasks.size() && tasks[t + 1].first <= b * per) ++t;
    bf[(size_t)b] = t;
  }
  bf[(size_t)nb] = tasks.empty() ? 0 : (int)tasks.size() - 1;
  return bf;
}

// ------------------------------------------------------------------ lowering: permute / fill
void Executor::perm(std::vector<Launch>& dst, const PerProb& X, const std::string& xi, const PerProb& Y,
                    const std::string& yi, double alpha, double beta, const std::vector<const double*>* scale,
                    const std::string& tag) {
  const int np = (int)probs_.size();
  const int r = (int)yi.size();
  if ((int)xi.size() != r) throw std::runtime_error("permute rank mismatch " + xi + "->" + yi);
  std::vector<PermProblem> ps(np);
  std::vector<int> prefix(np);
  Ranges rd, wr;
  int total = 0;
  for (int p = 0; p < np; ++p) {
    const long n = probs_[p].n;
    PermProblem& q = ps[p];
    q.X = X[p];
    q.Y = Y[p];
    q.scale = scale ? (*scale)[p] : nullptr;
    q.alpha = alpha;
    q.beta = beta;
    q.active = gate_for(dst, p);
    // Y axes padded on the left to 4; X strides of each Y axis
    for (int k = 0; k < 4; ++k) {
      q.d[k] = 1;
      q.xs[k] = 0;
    }
    for (int k = 0; k < r; ++k) {
      const int ya = 4 - r + k;
      const size_t pos = xi.find(yi[k]);
      if (pos == std::string::npos) throw std::runtime_error("permute letter mismatch " + xi + "->" + yi);
      q.d[ya] = (int)n;
      q.xs[ya] = ipow(n, r - 1 - (int)pos);
    }
    q.tb = -1;
    if (q.xs[3] != 1 && q.d[3] > 1) {
      for (int k = 0; k < 3; ++k)
        if (q.xs[k] == 1 && q.d[k] > 1) q.tb = k;
    }
    for (int k = 0; k < 4; ++k) q.div[k] = make_fastdiv((unsigned)q.d[k]);
    prefix[p] = total;
    if (alpha != 0.0) add_range(rd, X[p], sizeof(double) * (size_t)ipow(n, r));
    if (q.scale) add_range(rd, q.scale, sizeof(double));
    add_range(wr, Y[p], sizeof(double) * (size_t)ipow(n, r));
    if (q.tb < 0) {
      const long el = (long)q.d[0] * q.d[1] * q.d[2] * q.d[3];
      total += (int)((el + 1023) / 1024);
    } else {
      int c = 0;
      for (int k = 0; k < 3; ++k)
        if (k != q.tb) q.oth[c++] = k;
      const int nt3 = (q.d[3] + 31) / 32, ntb = (q.d[q.tb] + 31) / 32;
      q.tdiv[0] = make_fastdiv((unsigned)nt3);
      q.tdiv[1] = make_fastdiv((unsigned)ntb);
      total += nt3 * ntb * q.d[q.oth[0]] * q.d[q.oth[1]];
    }
  }
  Launch L;
  L.kind = Launch::PERM;
  L.n_prob = np;
  for (int p = 0; p < np; ++p) L.prob_total.push_back((p + 1 < np ? prefix[p + 1] : total) - prefix[p]);
  L.total = total;
  L.d_desc = upload(ps.data(), sizeof(PermProblem) * np);
  L.d_prefix = (int*)upload(prefix.data(), sizeof(int) * np);
  L.tag = tag;
  for (int p = 0; p < np; ++p)
    L.bytes += sizeof(double) * (double)ipow(probs_[p].n, r) * ((alpha != 0.0) + (beta != 0.0) + 1);
  L.rd = std::move(rd);
  L.wr = std::move(wr);
  L.ranged = true;
  dst.push_back(L);
}

void Executor::fill(std::vector<Launch>& dst, const PerProb& Y, int rank, const std::string& tag, int t_y) {
  // zero fill: the contiguous permute path with alpha = 0 and beta = 0 reads neither X nor Y;
  // with momentum laws only the allowed elements (the others never leave zero)
  if (rank > 0) {
    std::string idx;
    for (int k = 0; k < rank; ++k) idx.push_back((char)('p' + k));
    if (elem_blocked(dst, Y, idx, Y, idx, 0.0, 0.0, t_y, t_y, tag)) return;
  }
  dense_guard(tag, {t_y});
  const int np = (int)probs_.size();
  std::vector<PermProblem> ps(np);
  std::vector<int> prefix(np);
  int total = 0;
  for (int p = 0; p < np; ++p) {
    const long n = probs_[p].n;
    PermProblem& q = ps[p];
    std::memset(&q, 0, sizeof(q));
    q.X = Y[p];
    q.Y = Y[p];
    q.d[0] = 1;
    q.d[1] = 1;
    q.d[2] = 1;
    q.d[3] = (int)ipow(n, rank);
    q.xs[3] = 1;
    q.tb = -1;
    for (int k = 0; k < 4; ++k) q.div[k] = make_fastdiv((unsigned)q.d[k]);
    q.alpha = 0.0;
    q.beta = 0.0;
    q.active = gate_for(dst, p);
    prefix[p] = total;
    total += (int)((q.d[3] + 1023) / 1024);
  }
  Launch L;
  for (int p = 0; p < np; ++p) {
    add_range(L.wr, Y[p], sizeof(double) * (size_t)ipow(probs_[p].n, rank));
    L.bytes += sizeof(double) * (double)ipow(probs_[p].n, rank);
  }
  L.ranged = true;
  L.kind = Launch::FILL;
  L.n_prob = np;
  for (int p = 0; p < np; ++p) L.prob_total.push_back((p + 1 < np ? prefix[p + 1] : total) - prefix[p]);
  L.total = total;
  L.d_desc = upload(ps.data(), sizeof(PermProblem) * np);
  L.d_prefix = (int*)upload(prefix.data(), sizeof(int) * np);
  L.tag = tag;
  dst.push_back(L);
}

// Element offsets, in a tensor of layout `oi` (n per letter), of every index
// tuple of `letters` (first letter most significant): the rows or columns of a
// GEMM written straight into that tensor.  Built once per (n, letters, oi).
const unsigned* Executor::out_offsets(long n, const std::string& letters, const std::string& oi) {
  const std::string key = std::to_string(n) + ":" + letters + ":" + oi;
  auto it = out_tables_.find(key);
  if (it != out_tables_.end()) return it->second;
  const int r = (int)letters.size(), ro = (int)oi.size();
  std::vector<long> stride(r);
  for (int k = 0; k < r; ++k) stride[k] = ipow(n, ro - 1 - (int)oi.find(letters[k]));
  std::vector<unsigned> t((size_t)ipow(n, r));
  for (size_t idx = 0; idx < t.size(); ++idx) {
    long rem = (long)idx, off = 0;
    for (int k = r - 1; k >= 0; --k) {
      off += (rem % n) * stride[k];
      rem /= n;
    }
    t[idx] = (unsigned)off;
  }
  const unsigned* d = (const unsigned*)upload(t.data(), sizeof(unsigned) * std::max<size_t>(t.size(), 1));
  out_tables_[key] = d;
  return d;
}

Executor::PerProb Executor::const_permuted(int tensor, const PerProb& X, const std::string& xi,
                                           const std::string& yi) {
  // canonical key: the permutation as positions
  std::string key;
  for (char c : yi) key.push_back((char)('0' + xi.find(c)));
  auto k = std::make_pair(tensor, key);
  auto it = const_cache_.find(k);
  if (it != const_cache_.end()) return it->second;
  const int np = (int)probs_.size();
  PerProb Y(np);
  std::map<int, double*> per_inst;
  for (int p = 0; p < np; ++p) {
    const int inst = probs_[p].inst;
    if (!per_inst.count(inst)) {
      per_inst[inst] = const_alloc_(inst, (size_t)ipow(probs_[p].n, (int)xi.size()));
      const_bytes_ += sizeof(double) * (size_t)ipow(probs_[p].n, (int)xi.size());
    }
    Y[p] = per_inst[inst];
  }
  // one permute per instance: restrict to the first problem of each instance
  std::vector<ProblemRef> saved = probs_;
  std::vector<ProblemRef> firsts;
  PerProb Xf, Yf;
  std::map<int, bool> seen;
  for (int p = 0; p < np; ++p) {
    if (seen[probs_[p].inst]) continue;
    seen[probs_[p].inst] = true;
    firsts.push_back(probs_[p]);
    Xf.push_back(X[p]);
    Yf.push_back(Y[p]);
  }
  probs_ = firsts;
  perm(setup_, Xf, xi, Yf, yi, 1.0, 0.0, nullptr, "const-permute");
  probs_ = saved;
  const_cache_[k] = Y;
  return Y;
}

// Permuted copy of a non-constant value operand.  Copies are kept and reused by
// later consumers until the tensor is written again (its version changes); the
// operands of the backward program are forward values, fixed during backward.
Executor::PerProb Executor::value_permuted(std::vector<Launch>& dst, int tensor, const PerProb& X,
                                           const std::string& xi, const std::string& yi, const PerProb& scratch,
                                           const std::string& tag) {
  if (tensor < 0 || !cache_alloc_) {
    perm(dst, X, xi, scratch, yi, 1.0, 0.0, nullptr, tag);
    return scratch;
  }
  std::string key;
  for (char c : yi) key.push_back((char)('0' + xi.find(c)));
  auto k = std::make_pair(tensor, key);
  auto it = value_cache_.find(k);
  if (it != value_cache_.end() && it->second.version == version_[tensor]) return it->second.buf;
  const int np = (int)probs_.size();
  PerProb Y;
  if (it != value_cache_.end()) {
    Y = it->second.buf;
  } else {
    size_t bytes = 0;
    for (int p = 0; p < np; ++p) bytes += sizeof(double) * (size_t)ipow(probs_[p].n, (int)xi.size());
    if (cache_bytes_ + bytes > cache_budget_) {
      perm(dst, X, xi, scratch, yi, 1.0, 0.0, nullptr, tag);
      return scratch;
    }
    for (int p = 0; p < np; ++p) {
      double* q = cache_alloc_((size_t)ipow(probs_[p].n, (int)xi.size()));
      if (!q) {   // no room: uncached (buffers taken for earlier problems stay unused)
        perm(dst, X, xi, scratch, yi, 1.0, 0.0, nullptr, tag);
        return scratch;
      }
      cache_bytes_ += sizeof(double) * (size_t)ipow(probs_[p].n, (int)xi.size());
      Y.push_back(q);
    }
  }
  perm(dst, X, xi, Y, yi, 1.0, 0.0, nullptr, tag + "(cached)");
  value_cache_[k] = CacheEntry{Y, version_[tensor]};
  return Y;
}

// ------------------------------------------------------------------ lowering: contraction
void Executor::contract(std::vector<Launch>& dst, const PerProb& out, const std::string& oi, double alpha,
                        const PerProb& A, const std::string& ai, int a_const, const PerProb* B,
                        const std::string& bi, int b_const, bool acc, const std::string& tag, int a_val,
                        int b_val, int t_out, int t_a, int t_b) {
  const double beta = acc ? 1.0 : 0.0;
  const int np = (int)probs_.size();
  if (B && !oi.empty() && !ai.empty() && !bi.empty() && &dst != &setup_ &&
      contract_blocked(dst, out, oi, alpha, A, ai, *B, bi, acc, tag, t_out, t_a, t_b))
    return;
  if (!B) {
    for (char c : ai)
      if (!has(oi, c)) throw std::runtime_error("single-operand reduction unsupported: " + tag);
    if (elem_blocked(dst, A, ai, out, oi, alpha, beta, t_out, t_a, tag)) return;
    dense_guard(tag, {t_out, t_a});
    perm(dst, A, ai, out, oi, alpha, beta, nullptr, tag);
    return;
  }
  // scalar operand: scaled permute with a device scalar (over the allowed elements
  // when the laws are known)
  if (ai.empty() || bi.empty()) {
    const PerProb& S = ai.empty() ? A : *B;
    const PerProb& X = ai.empty() ? *B : A;
    const std::string& xi = ai.empty() ? bi : ai;
    std::vector<const double*> sc(S.begin(), S.end());
    const int t_x = ai.empty() ? t_b : t_a;
    if (&dst != &setup_ && !oi.empty() && elem_blocked(dst, X, xi, out, oi, alpha, beta, t_out, t_x, tag, &sc))
      return;
    dense_guard(tag, {t_out, t_a, t_b});
    perm(dst, X, xi, out, oi, alpha, beta, &sc, tag);
    return;
  }
  for (char c : ai)
    if (!has(bi, c) && !has(oi, c)) throw std::runtime_error("letter summed in one operand only: " + tag);
  for (char c : bi)
    if (!has(ai, c) && !has(oi, c)) throw std::runtime_error("letter summed in one operand only: " + tag);
  for (char c : oi)
    if (has(ai, c) && has(bi, c)) throw std::runtime_error("batch letters unsupported: " + tag);

  // full contraction -> dot
  if (oi.empty()) {
    if (&dst != &setup_ && dot_blocked(dst, A, ai, *B, bi, out, alpha, beta, t_a, t_b, tag)) return;
    dense_guard(tag, {t_a, t_b, t_out});
    PerProb Bp = *B;
    if (bi != ai) {
      if (b_const >= 0) Bp = const_permuted(b_const, *B, bi, ai);
      else Bp = value_permuted(dst, b_val, *B, bi, ai, scratch_->b, tag + ":permB");
    }
    std::vector<DotProblem> ds(np);
    for (int p = 0; p < np; ++p) {
      ds[p].X = A[p];
      ds[p].Y = Bp[p];
      ds[p].out = out[p];
      ds[p].len = ipow(probs_[p].n, (int)ai.size());
      ds[p].alpha = alpha;
      ds[p].beta = beta;
      ds[p].active = gate_for(dst, p);
    }
    Launch L;
    for (int p = 0; p < np; ++p) {
      add_range(L.rd, ds[p].X, sizeof(double) * (size_t)ds[p].len);
      add_range(L.rd, ds[p].Y, sizeof(double) * (size_t)ds[p].len);
      add_range(L.wr, ds[p].out, sizeof(double));
      L.bytes += 2.0 * sizeof(double) * (double)ds[p].len;
    }
    L.ranged = true;
    L.kind = Launch::DOT;
    L.n_prob = np;
    // from a million elements on 64 blocks of 256 threads read less than the memory delivers
    // (57 orbitals: 281 us with 64)
    L.dot_blocks = 64;
    L.d_partial = scratch_->dot_partial;
    for (const DotProblem& d : ds)
      if (d.len >= (1L << 20) && (size_t)np * kMaxDotBlocks <= scratch_->tail_ws_doubles) {
        L.dot_blocks = kMaxDotBlocks;
        L.d_partial = scratch_->tail_ws;
      }
    L.d_desc = upload(ds.data(), sizeof(DotProblem) * np);
    L.tag = tag;
    dst.push_back(L);
    return;
  }

  dense_guard(tag, {t_out, t_a, t_b});
  const std::string M_a = filter(ai, bi, oi, false, true);   // in A and out only
  const std::string K_a = filter(ai, bi, oi, true, false);   // in A and B only
  const std::string N_b = filter(bi, ai, oi, false, true);
  const std::string K_b = filter(bi, ai, oi, true, false);
  const std::string M_o = filter(oi, ai, bi, true, false);
  const std::string N_o = filter(oi, bi, ai, true, false);

  struct Choice {
    std::string M, N, K;
    bool swap;
    double cost;
  };
  Choice best{"", "", "", false, 1e300};
  const long n0 = probs_[0].n;
  auto sz = [&](const std::string& s) { return (double)ipow(n0, (int)s.size()); };
  for (int im = 0; im < 2; ++im)
    for (int in = 0; in < 2; ++in)
      for (int ik = 0; ik < 2; ++ik) {
        std::string M = im ? M_o : M_a, N = in ? N_o : N_b, K = ik ? K_b : K_a;
        double cost = 0.0;
        const bool a_ok = (ai == M + K) || (ai == K + M);
        const bool b_ok = (bi == K + N) || (bi == N + K);
        if (!a_ok && a_const < 0) cost += sz(ai);
        if (!b_ok && b_const < 0) cost += sz(bi);
        bool swap = false;
        if (oi == M + N) {
        } else if (oi == N + M) {
          swap = true;
        } else if (!N.empty() && N.back() == oi.back()) {
          cost += 0.1 * sz(oi);   // written through output offset tables, columns contiguous
        } else if (!M.empty() && M.back() == oi.back()) {
          swap = true;            // the same with C transposed
          cost += 0.1 * sz(oi);
        } else {
          cost += 2.0 * sz(oi);   // GEMM layout, then a permute pass
        }
        if (cost < best.cost) best = {M, N, K, swap, cost};
      }

  // operands in GEMM layout
  auto place = [&](const PerProb& X, const std::string& xi, int xconst, int xval, const std::string& first,
                   const std::string& second, PerProb& scratch, bool& trans, std::string& lay) -> PerProb {
    if (xi == first + second) {
      trans = false;
      lay = xi;
      return X;
    }
    if (xi == second + first) {
      trans = true;
      lay = xi;
      return X;
    }
    trans = false;
    lay = first + second;
    if (xconst >= 0) return const_permuted(xconst, X, xi, lay);
    return value_permuted(dst, xval, X, xi, lay, scratch, tag + ":perm");
  };
  // C[M][N] = A[M][K] B[K][N]; with swap, C^T[N][M] = B^T[N][K] A^T[K][M]
  std::string M = best.M, N = best.N, K = best.K;
  PerProb Ap, Bp;
  bool ta = false, tb = false;
  std::string alay, blay;
  if (!best.swap) {
    Ap = place(A, ai, a_const, a_val, M, K, scratch_->a, ta, alay);     // ta: stored [K][M]
    Bp = place(*B, bi, b_const, b_val, K, N, scratch_->b, tb, blay);    // tb: stored [N][K]
  } else {
    // rows of C = N letters (from B), cols = M letters (from A)
    Ap = place(*B, bi, b_const, b_val, N, K, scratch_->b, ta, alay);
    Bp = place(A, ai, a_const, a_val, K, M, scratch_->a, tb, blay);
    std::swap(M, N);
  }
  const bool c_direct = (oi == M + N);
  // Output in neither [M][N] nor [N][M] but with its fastest letter the GEMM's
  // fastest column letter: the GEMM writes it through row and column offset
  // tables (coalesced along that letter) instead of C plus a permute pass; not
  // when the output aliases an operand, which the GEMM would overwrite while
  // other tiles still read it.
  bool c_table = !c_direct && !N.empty() && N.back() == oi.back();
  for (int p = 0; p < np && c_table; ++p) {
    if (out[p] == A[p] || out[p] == (*B)[p] || out[p] == Ap[p] || out[p] == Bp[p]) c_table = false;
    if (ipow(probs_[p].n, (int)oi.size()) >= (1L << 32)) c_table = false;
  }
  const double galpha = alpha;
  const double gbeta = (c_direct || c_table) ? beta : 0.0;
  const PerProb& Cp = (c_direct || c_table) ? out : scratch_->c;

  int cfg = 0;
  {
    const long m = ipow(n0, (int)M.size()), nn = ipow(n0, (int)N.size()), kk = ipow(n0, (int)K.size());
    cfg = (m >= 128 && nn >= 128) ? (kk >= 512 ? 2 : 0) : 1;
  }
  // descriptors of the grouped launch for one tile configuration; allow_split:
  // split K when the launch would not fill the device
  auto build_gemm = [&](int gcfg, bool allow_split) {
    std::vector<GemmProblem> gs(np);
    std::vector<int> prefix(np), prefix2(np);
    const int BM = gemm_bm(gcfg), BN = gemm_bn(gcfg);
    int total = 0, total2 = 0;
    bool any_split = false;
    double flops = 0.0;
    long tiles_all = 0;
    for (int p = 0; p < np; ++p) {
      const long n = probs_[p].n;
      tiles_all += ((ipow(n, (int)M.size()) + BM - 1) / BM) * ((ipow(n, (int)N.size()) + BN - 1) / BN);
    }
    for (int p = 0; p < np; ++p) {
      const long n = probs_[p].n;
      GemmProblem& g = gs[p];
      g.M = (int)ipow(n, (int)M.size());
      g.N = (int)ipow(n, (int)N.size());
      g.K = (int)ipow(n, (int)K.size());
      g.A = Ap[p];
      g.B = Bp[p];
      g.C = Cp[p];
      g.lda = ta ? g.M : g.K;
      g.ldb = tb ? g.K : g.N;
      g.ldc = g.N;
      g.alpha = galpha;
      g.beta = gbeta;
      g.active = gate_for(dst, p);
      g.tiles_m = (g.M + BM - 1) / BM;
      g.tiles_n = (g.N + BN - 1) / BN;
      if (c_table) {
        g.offM = out_offsets(n, M, oi);
        g.offN = out_offsets(n, N, oi);
      }
      int ks = 1;
      if (allow_split && tiles_all < 512 && g.K >= 512) {
        ks = (int)std::min<long>((512 + tiles_all - 1) / tiles_all, g.K / 256);
        // the partial buffer holds n^4 doubles
        while (ks > 1 && (long)ks * g.M * g.N > ipow(n, 4)) --ks;
        ks = std::max(ks, 1);
      }
      if ((long)g.M * g.K >= (1L << 31) || (long)g.K * g.N >= (1L << 31) || (long)g.M * g.N >= (1L << 31))
        throw std::runtime_error("GEMM operand exceeds 2^31 elements: " + tag);
      g.ksplit = ks;
      g.kchunk = (g.K + ks - 1) / ks;
      g.kchunk = ((g.kchunk + 15) / 16) * 16;
      g.ksplit = (g.K + g.kchunk - 1) / g.kchunk;
      g.partial = scratch_->part[p];
      if (g.ksplit > 1) any_split = true;
      prefix[p] = total;
      total += g.tiles_m * g.tiles_n * g.ksplit;
      prefix2[p] = total2;
      total2 += (int)(((long)g.M * g.N + 63) / 64);
      flops += 2.0 * g.M * (double)g.N * g.K;
    }
    std::vector<double> pf(np);
    std::vector<int> pinst(np);
    Launch L;
    for (int p = 0; p < np; ++p) {
      pf[p] = 2.0 * gs[p].M * (double)gs[p].N * gs[p].K;
      pinst[p] = p;
      L.bytes += sizeof(double) * ((double)gs[p].M * gs[p].K + (double)gs[p].K * gs[p].N +
                                   (double)gs[p].M * gs[p].N * (beta != 0.0 ? 2 : 1));
    }
    L.kind = Launch::GEMM;
    L.n_prob = np;
    for (int p = 0; p < np; ++p) {
      L.prob_total.push_back((p + 1 < np ? prefix[p + 1] : total) - prefix[p]);
      L.prob_total2.push_back((p + 1 < np ? prefix2[p + 1] : total2) - prefix2[p]);
    }
    L.total = total;
    L.min_k = np > 0 ? gs[0].K : 0;
    for (int p = 1; p < np; ++p) L.min_k = std::min(L.min_k, gs[p].K);
    if (&dst != &setup_) {
      L.prob_flops = pf;
      L.prob_gate = pinst;
    }
    L.cfg = gcfg;
    L.ta = ta;
    L.tb = tb;
    L.d_desc = upload(gs.data(), sizeof(GemmProblem) * np);
    L.d_prefix = (int*)upload(prefix.data(), sizeof(int) * np);
    if (any_split) {
      // problems without a split still need their own reduce pass skipped: mark via ksplit
      L.splitk_blocks = total2;
      L.d_prefix2 = (int*)upload(prefix2.data(), sizeof(int) * np);
    }
    L.flops = flops;
    L.tag = tag;
    return L;
  };
  Launch L = build_gemm(cfg, true);
  if (&dst != &setup_) {
    // candidates for the autotuner: 64 x 64 tiles while the 128 x 128 launch is
    // short of four waves of resident blocks (beyond that its edge waste is small
    // and the larger tile wins), and the launch without split-K
    if (gemm_bm(cfg) == 128 && L.total < 4 * gemm_slots(cfg)) L.alts.push_back(build_gemm(1, true));
    if (L.splitk_blocks > 0) L.alts.push_back(build_gemm(cfg, false));
  }
  dst.push_back(L);
  if (!c_direct && !c_table) perm(dst, scratch_->c, M + N, out, oi, 1.0, beta, nullptr, tag + ":permC");
}


// ------------------------------------------------------------------ momentum blocking
// Laws of the intermediates from the ops, in program order: a unary op copies
// its operand's signs; for out = A * B the contracted letters fix the relative
// orientation s of B's law (sign_A * sign_B, the same for every contracted
// letter), and out gets sign_A on A's free letters and -s * sign_B on B's.
// Every op writing a tensor must give the same law up to an overall sign.
bool packing_enabled() {
  const char* e = std::getenv("FTCC_PACK");
  return !(e && e[0] == '0');
}

bool labels_distinct(const InstMomentum& M) {
  const int D = M.dims;
  if (D <= 0) return false;
  const int n = (int)(M.labels.size() / D);
  std::vector<std::vector<int>> keys(n, std::vector<int>(D));
  for (int p = 0; p < n; ++p)
    for (int c = 0; c < D; ++c) {
      int v = M.labels[(size_t)p * D + c];
      if (M.modulus[c] > 0) v = ((v % M.modulus[c]) + M.modulus[c]) % M.modulus[c];
      keys[p][c] = v;
    }
  std::sort(keys.begin(), keys.end());
  return std::adjacent_find(keys.begin(), keys.end()) == keys.end();
}

void Executor::dense_guard(const std::string& tag, std::initializer_list<int> ts) const {
  for (int t : ts)
    if (is_packed(t)) throw std::runtime_error("packed intermediate on a dense path: " + tag);
}

int Executor::n_packed() const {
  int k = 0;
  for (char v : packed_) k += v ? 1 : 0;
  return k;
}

// Which intermediates are stored packed: rank >= 2, a known momentum law, every
// instance's labels distinct, and every op that touches the tensor (forward, and
// its reverse forms when the backward list is built) has known laws on all of
// its tensors, so that it lowers to blocked kernels, which address elements
// through offset tables only.  Derived constants keep dense storage (their set-up
// ops are dense permutes).
void Executor::plan_packing(bool want_backward) {
  const int nt = (int)prog_->t.size();
  packed_.assign(nt, 0);
  pack_on_ = one_per_label_ = false;
  if (mom_.empty()) return;
  for (const ProblemRef& p : probs_)
    if (p.inst < 0 || p.inst >= (int)mom_.size() || !mom_[p.inst] || !labels_distinct(*mom_[p.inst])) return;
  one_per_label_ = true;
  if (!packing_enabled()) return;
  pack_on_ = true;
  for (int k = 0; k < nt; ++k) {
    const TensorDecl& d = prog_->t[k];
    packed_[k] = (d.kind == T_INTER && !d.derived && d.rank >= 2 && law_ok_[k]) ? 1 : 0;
  }
  (void)want_backward;   // the reverse forms of an op lower blocked exactly when the forward does
  for (const SymOp& o : prog_->ops) {
    if (o.setup && !inline_setup_) continue;
    const bool ok = law_ok_[o.out] && law_ok_[o.a] && (o.b < 0 || law_ok_[o.b]);
    if (ok) continue;
    packed_[o.out] = 0;
    packed_[o.a] = 0;
    if (o.b >= 0) packed_[o.b] = 0;
  }
}

std::vector<int> Executor::plan_const_packing(const std::vector<int>& const_grads) const {
  std::vector<int> out;
  if (!pack_on_ || inline_setup_) return out;
  const int nt = (int)prog_->t.size();
  for (int k = 0; k < nt; ++k) {
    const TensorDecl& d = prog_->t[k];
    if (!(d.kind == T_CONST || d.derived) || d.rank < 2 || !law_ok_[k]) continue;
    if (std::find(const_grads.begin(), const_grads.end(), k) != const_grads.end()) continue;
    bool ok = true, used = false;
    for (const SymOp& o : prog_->ops) {
      if (o.setup) continue;
      if (o.out != k && o.a != k && o.b != k) continue;
      used = true;
      if (!(law_ok_[o.out] && law_ok_[o.a] && (o.b < 0 || law_ok_[o.b]))) ok = false;
    }
    if (ok && used) out.push_back(k);
  }
  return out;
}

std::vector<int> Executor::plan_io_packing() const {
  std::vector<int> out;
  if (!pack_on_) return out;
  const int nt = (int)prog_->t.size();
  for (int k = 0; k < nt; ++k) {
    const TensorDecl& d = prog_->t[k];
    if (!(d.kind == T_INPUT || d.kind == T_OUTPUT) || d.rank < 2 || !law_ok_[k]) continue;
    bool ok = true;
    for (const SymOp& o : prog_->ops) {
      if (o.setup || (o.out != k && o.a != k && o.b != k)) continue;
      if (!(law_ok_[o.out] && law_ok_[o.a] && (o.b < 0 || law_ok_[o.b]))) ok = false;
    }
    if (ok) out.push_back(k);
  }
  return out;
}

bool Executor::io_packable(const Program* prog, const std::vector<ProblemRef>& probs) {
  if (mom_.empty()) return false;
  prog_ = prog;
  probs_ = probs;
  infer_laws();
  plan_packing(true);
  int n_io = 0;
  for (const TensorDecl& d : prog->t) n_io += (d.kind == T_INPUT || d.kind == T_OUTPUT) && d.rank >= 2;
  return (int)plan_io_packing().size() == n_io;
}

void Executor::infer_laws() {
  const int nt = (int)prog_->t.size();
  law_.assign(nt, {});
  law_ok_.assign(nt, 0);
  std::vector<char> bad(nt, 0), known(nt, 0);
  for (int k = 0; k < nt; ++k)
    if ((k < (int)prog_->law.size() && !prog_->law[k].empty()) || prog_->t[k].rank == 0) {
      if (k < (int)prog_->law.size()) law_[k] = prog_->law[k];
      known[k] = 1;
    }
  for (const SymOp& o : prog_->ops) {
    bool ok = known[o.a] && !bad[o.a] && (o.b < 0 || (known[o.b] && !bad[o.b]));
    std::vector<int> lc;
    if (ok) {
      auto sg = [&](int t, const std::string& idx, char c) { return law_[t][idx.find(c)]; };
      int s = -1;
      bool first = true;
      if (o.b >= 0)
        for (char c : o.ai)
          if (has(o.bi, c)) {
            const int r = sg(o.a, o.ai, c) * sg(o.b, o.bi, c);
            if (first) {
              s = r;
              first = false;
            } else if (r != s) {
              ok = false;
            }
          }
      if (ok)
        for (char c : o.oi) lc.push_back(has(o.ai, c) ? sg(o.a, o.ai, c) : -s * sg(o.b, o.bi, c));
    }
    const int k = o.out;
    if (!ok) {
      bad[k] = 1;
    } else if (!known[k]) {
      law_[k] = lc;
      known[k] = 1;
    } else {
      std::vector<int> neg(lc);
      for (int& v : neg) v = -v;
      if (law_[k] != lc && law_[k] != neg) bad[k] = 1;
    }
  }
  for (int k = 0; k < nt; ++k) law_ok_[k] = known[k] && !bad[k];
}

static long long pack_momentum(const std::vector<int>& q) {
  long long key = 0;
  for (size_t c = 0; c < q.size(); ++c) key |= (long long)(q[c] + (1 << 19)) << (21 * c);
  return key;
}

// Tuples of `letters` (each 0..n-1) in momentum-block order, with their element
// offsets in the operands indexed by xi and yi (row-major, every axis n) and
// the packed momentum sum_l signs[l] k(index_l) of each block.
const Executor::GroupTable& Executor::group_table(int inst, long n, const std::string& letters,
                                                  const std::string& xi, bool xp, const std::string& yi, bool yp,
                                                  const std::vector<int>& signs, int edge) {
  if (one_per_label_) edge = 0;   // blocks of a few elements: nothing to gain
  inst = same_labels_[inst];
  std::string key = std::to_string(inst) + "|" + letters + "|" + xi + (xp ? "#" : "") + "|" + yi +
                    (yp ? "#" : "") + "|" + std::to_string(edge);
  for (int v : signs) key += (v > 0 ? '+' : '-');
  auto it = group_cache_.find(key);
  if (it != group_cache_.end()) return it->second;
  const InstMomentum& M = *mom_[inst];
  const int g = (int)letters.size(), D = M.dims;
  // row-major strides; a packed tensor drops its last axis (stride 0: that index
  // is fixed by the others on every allowed element)
  auto stride = [&](const std::string& idx, bool packed, char c) -> unsigned long {
    const int pos = (int)idx.find(c), len = (int)idx.size();
    if (!packed) return (unsigned long)ipow(n, len - 1 - pos);
    return pos == len - 1 ? 0ul : (unsigned long)ipow(n, len - 2 - pos);
  };
  std::vector<unsigned long> sx(g), sy(g);
  for (int l = 0; l < g; ++l) {
    sx[l] = stride(xi, xp, letters[l]);
    sy[l] = stride(yi, yp, letters[l]);
  }
  const long count = ipow(n, g);
  struct Row {
    long long key;
    unsigned ox, oy, ord;
  };
  // Order inside a block.  Lanes run along a tuple list, so the letter along which a
  // tensor is contiguous should be the fastest: for rows and columns (edge 1) the
  // operand's, which is read once per tile, before the output's; for the inner list
  // (edge 4), where the two operands may want different letters, the tuples go in patches
  // of edge x edge of those two and both are read in runs of `edge` (27 orbitals, a ring
  // contraction with crossed inner letters: 165 -> 114 us).
  int lx = edge && has(letters, xi.back()) ? (int)letters.find(xi.back()) : -1;
  int ly = edge && has(letters, yi.back()) ? (int)letters.find(yi.back()) : -1;
  if (edge == 1 && lx >= 0) ly = -1;
  auto order_of = [&](const std::vector<int>& idx, long t) -> unsigned {
    if (lx < 0 && ly < 0) return (unsigned)t;
    unsigned long o = 0;
    for (int l = 0; l < g; ++l)
      if (l != lx && l != ly) o = o * n + idx[l];
    if (lx < 0 || ly < 0 || lx == ly) return (unsigned)(o * n + idx[lx >= 0 ? lx : ly]);
    const unsigned long nb = (n + edge - 1) / edge;
    o = (o * nb + idx[lx] / edge) * nb + idx[ly] / edge;
    return (unsigned)((o * edge + idx[lx] % edge) * edge + idx[ly] % edge);
  };
  std::vector<Row> rows(count);
  std::vector<int> idx(g, 0), q(D);
  for (long t = 0; t < count; ++t) {
    unsigned long ox = 0, oy = 0;
    std::fill(q.begin(), q.end(), 0);
    for (int l = 0; l < g; ++l) {
      ox += idx[l] * sx[l];
      oy += idx[l] * sy[l];
      for (int c = 0; c < D; ++c) q[c] += signs[l] * M.labels[(size_t)idx[l] * D + c];
    }
    for (int c = 0; c < D; ++c)
      if (M.modulus[c] > 0) q[c] = ((q[c] % M.modulus[c]) + M.modulus[c]) % M.modulus[c];
    rows[t] = Row{pack_momentum(q), (unsigned)ox, (unsigned)oy, order_of(idx, t)};
    for (int l = g - 1; l >= 0; --l) {   // next tuple, last letter fastest
      if (++idx[l] < n) break;
      idx[l] = 0;
    }
  }
  // into blocks by momentum (a counting sort over the few distinct ones), each block in its order
  std::map<long long, std::pair<int, int>> found;
  std::vector<std::pair<int, int>*> of(count);
  {
    std::unordered_map<long long, std::pair<int, int>*> seen;
    for (long t = 0; t < count; ++t) {
      auto it = seen.find(rows[t].key);
      if (it == seen.end()) it = seen.emplace(rows[t].key, &found.emplace(rows[t].key, std::make_pair(0, 0)).first->second).first;
      of[t] = it->second;
      it->second->second++;
    }
  }
  int first = 0;
  for (auto& f : found) {
    f.second.first = first;
    first += f.second.second;
    f.second.second = 0;
  }
  std::vector<Row> sorted(count);
  for (long t = 0; t < count; ++t) sorted[of[t]->first + of[t]->second++] = rows[t];
  if (lx >= 0 || ly >= 0)
    for (const auto& f : found) {
      auto b = sorted.begin() + f.second.first, e = b + f.second.second;
      auto before = [](const Row& x, const Row& y) { return x.ord < y.ord; };
      if (!std::is_sorted(b, e, before)) std::sort(b, e, before);
    }
  GroupTable T;
  T.blocks = std::move(found);
  std::vector<unsigned> o1(count), o2(count);
  for (long t = 0; t < count; ++t) {
    o1[t] = sorted[t].ox;
    o2[t] = sorted[t].oy;
  }
  T.off1 = upload(o1.data(), sizeof(unsigned) * count);
  T.off2 = upload(o2.data(), sizeof(unsigned) * count);
  return group_cache_.emplace(key, std::move(T)).first->second;
}

// The tuples (one byte per index) with sum_l signs[l] k(index_l) = 0,
// lexicographically: the last index runs over the orbitals of the label that the others
// leave.  At most four letters.
const std::vector<unsigned>& Executor::allowed_tuples(int inst, long n, const std::vector<int>& signs) {
  inst = same_labels_[inst];
  std::string key = std::to_string(inst) + "|";
  for (int v : signs) key += v == signs[0] ? '+' : '-';   // a common sign does not matter
  auto it = tuple_cache_.find(key);
  if (it != tuple_cache_.end()) return it->second;
  const InstMomentum& M = *mom_[inst];
  const int g = (int)signs.size(), D = M.dims;
  auto reduced = [&](int v, int c) { return M.modulus[c] > 0 ? ((v % M.modulus[c]) + M.modulus[c]) % M.modulus[c] : v; };
  // orbital of a label, over the box that the labels span
  std::vector<int> lo(D), len(D);
  std::vector<int> lab((size_t)n * D);
  for (long p = 0; p < n; ++p)
    for (int c = 0; c < D; ++c) lab[p * D + c] = reduced(M.labels[p * D + c], c);
  long box = 1;
  for (int c = 0; c < D; ++c) {
    int mn = lab[c], mx = lab[c];
    for (long p = 1; p < n; ++p) {
      mn = std::min(mn, lab[p * D + c]);
      mx = std::max(mx, lab[p * D + c]);
    }
    lo[c] = mn;
    len[c] = mx - mn + 1;
    box *= len[c];
  }
  // wide label ranges (any integers are allowed) are looked up in a map instead
  const bool dense = box <= (1L << 22);
  std::vector<std::vector<int>> at(dense ? box : 0);   // orbitals of each label, ascending
  std::unordered_map<long, std::vector<int>> far;
  auto slot = [&](const int* v) -> long {
    long o = 0;
    for (int c = 0; c < D; ++c) {
      if (v[c] < lo[c] || v[c] >= lo[c] + len[c]) return -1;
      o = o * len[c] + (v[c] - lo[c]);
    }
    return o;
  };
  for (long p = 0; p < n; ++p) {
    const long o = slot(&lab[p * D]);
    if (dense) at[o].push_back((int)p);
    else far[o].push_back((int)p);
  }
  std::vector<unsigned> out;
  std::vector<int> idx(g, 0), v(D);
  const long count = ipow(n, g - 1);
  for (long t = 0; t < count; ++t) {
    unsigned packed = 0;
    std::fill(v.begin(), v.end(), 0);
    for (int l = 0; l + 1 < g; ++l) {
      packed |= (unsigned)idx[l] << (8 * l);
      for (int c = 0; c < D; ++c) v[c] += signs[l] * M.labels[(size_t)idx[l] * D + c];
    }
    for (int c = 0; c < D; ++c) v[c] = reduced(-signs[g - 1] * v[c], c);
    const long o = slot(v.data());
    const std::vector<int>* last = nullptr;
    if (o >= 0) {
      if (dense) {
        last = &at[o];
      } else {
        auto f = far.find(o);
        if (f != far.end()) last = &f->second;
      }
    }
    if (last)
      for (int p : *last) out.push_back(packed | (unsigned)p << (8 * (g - 1)));
    for (int l = g - 2; l >= 0; --l) {
      if (++idx[l] < n) break;
      idx[l] = 0;
    }
  }
  return tuple_cache_.emplace(key, std::move(out)).first->second;
}

// Element offsets, in a tensor indexed by xi, of the allowed tuples of `letters`.
const unsigned* Executor::offset_list(int inst, long n, const std::string& letters, const std::vector<int>& signs,
                                      const std::string& xi, bool xp) {
  inst = same_labels_[inst];
  const int g = (int)letters.size();
  std::string key = std::to_string(inst) + "|";
  for (int v : signs) key += v == signs[0] ? '+' : '-';
  unsigned long stride[4] = {0, 0, 0, 0};
  for (int l = 0; l < g; ++l) {
    const int pos = (int)xi.find(letters[l]);
    key += (char)('0' + pos);
    stride[l] = !xp ? (unsigned long)ipow(n, g - 1 - pos) : pos == g - 1 ? 0ul : (unsigned long)ipow(n, g - 2 - pos);
  }
  if (xp) key += '#';
  auto it = list_cache_.find(key);
  if (it != list_cache_.end()) return it->second;
  const std::vector<unsigned>& T = allowed_tuples(inst, n, signs);
  std::vector<unsigned> off(T.size());
  for (size_t t = 0; t < T.size(); ++t) {
    unsigned long o = 0;
    for (int l = 0; l < g; ++l) o += ((T[t] >> (8 * l)) & 255u) * stride[l];
    off[t] = (unsigned)o;
  }
  const unsigned* d = (const unsigned*)upload(off.data(), sizeof(unsigned) * off.size());
  return list_cache_.emplace(key, d).first->second;
}

const unsigned* Executor::zero_offset() {
  const unsigned z = 0;
  if (!zero_offset_) zero_offset_ = (const unsigned*)upload(&z, sizeof z);
  return zero_offset_;
}

// Tile shape of one block of a blocked contraction (ml rows, nl columns, kl inner):
// 0 (16 x 16 MFMA tiles) or a lane-mapped shape code, whichever needs fewer wave
// latencies by a simple count: a wave costs 3 dependent memory latencies (task,
// offsets, the store) plus 2 per step of its inner loop; an MFMA step covers 32
// inner indices, a lane-mapped step 8 per lane of the inner slices (at most
// `cap` steps: longer ranges go to MFMA tiles split over several waves).  With
// the operands in cache (packed storage) long lane-mapped chains pay: 1.31 s per
// 123-PW step with a cap of 16 steps against 1.44 s with 2 and 1.79 s without
// lane-mapped tiles; with every operand scattered over dense arrays a cap of 2
// had been the best.
static int sgemm_shape(int ml, int nl, int kl, long cap) {
  auto cdiv = [](long a, long b) { return (a + b - 1) / b; };
  auto steps = [&](long per) { return std::max(1L, cdiv(kl, per)); };
  const long mfma = cdiv(ml, 16) * cdiv(nl, 16) * (3 + 2 * steps(32));
  long best = mfma;
  int shape = 0;
  for (int lr = 0; lr <= 6; ++lr)
    for (int lc = 0; lr + lc <= 6; ++lc) {
      const int ls = 6 - lr - lc;
      if (steps(8L << ls) > cap) continue;   // longer ranges: MFMA tiles split over several waves
      const long c = cdiv(ml, 1L << lr) * cdiv(nl, 1L << lc) * (3 + 2 * steps(8L << ls));
      if (c < best) {
        best = c;
        shape = sgemm_thin_shape(lr, lc, ls);
      }
    }
  return shape;
}

constexpr long kSgemmThinSteps = 16;

// Block-tile shape of one block of a blocked contraction, or 0 (wave tiles).  A
// block tile pays when both its sides exceed one 16-wide MFMA tile and it is long on
// one side (27-orbital step 515 ms with wave tiles only, 265 with block tiles) or over
// the inner range (33 x 33 outputs over 33^3: 100 us in wave tiles of 64 indices plus
// 60 us to add them, 20 us together in block tiles); a narrow side of at most 32 takes
// the 128-long tiles.
constexpr int kTileMin = 64;
constexpr int kTileSpread = 144;
static int sgemm_tile_shape(int ml, int nl, int kl) {
  if (std::min(ml, nl) <= 16 || (std::max(ml, nl) < kTileMin && kl < 512)) return 0;
  if (nl <= 32 && ml > 64) return kTile128x32;
  if (ml <= 32 && nl > 64) return kTile32x128;
  return kTile64x64;
}

// workspace units (256 doubles) of one part of a split tile
static int part_units(int shape) { return shape >= kTile64x64 ? 16 : 1; }

// wave latencies of a task by the same count (the order of a merged task list);
// block tiles stand before every wave task, longest first
static long sgemm_task_cost(const SgemmTask& t) {
  if (t.shape >= kTile64x64) return (t.shape == kTile64x64 ? 2000000000L : 1000000000L) + t.klen;
  const long per = t.shape == kWave32x32 ? 16L : t.shape ? (8L << ((t.shape >> 6) & 7)) : 32L;
  return 3 + 2 * std::max(1L, (t.klen + per - 1) / per);
}

// C[oi] (+)= alpha A[ai] B[bi] over the momentum-allowed blocks: rows M (letters
// of A and C), inner K (A and B), columns N (B and C).  A row tuple of momentum
// q pairs with inner tuples of A-momentum -q and column tuples of B-momentum s q.
// Returns false (dense lowering) when a law is unknown.
bool Executor::contract_blocked(std::vector<Launch>& dst, const PerProb& out, const std::string& oi, double alpha,
                                const PerProb& A, const std::string& ai, const PerProb& B, const std::string& bi,
                                bool acc, const std::string& tag, int t_out, int t_a, int t_b) {
  if (mom_.empty() || t_out < 0 || t_a < 0 || t_b < 0) return false;
  if (!law_ok_[t_out] || !law_ok_[t_a] || !law_ok_[t_b]) return false;
  // the letter along which a tensor is contiguous (a packed tensor drops its last axis)
  auto unit_letter = [&](const std::string& idx, int t) {
    return is_packed(t) ? (idx.size() >= 2 ? idx[idx.size() - 2] : '\0') : idx.back();
  };
  // columns of C are the index group that holds its contiguous letter: the other
  // way round, compute the transpose (with one orbital per momentum the blocks are
  // a few elements wide and the order does not matter)
  if (!one_per_label_ && !has(bi, unit_letter(oi, t_out)) && has(ai, unit_letter(oi, t_out)))
    return contract_blocked(dst, out, oi, alpha, B, bi, A, ai, acc, tag, t_out, t_b, t_a);
  const std::vector<int>&la = law_[t_a], &lb = law_[t_b];
  auto sa = [&](char c) { return la[ai.find(c)]; };
  auto sb = [&](char c) { return lb[bi.find(c)]; };
  const std::string M = filter(ai, bi, oi, false, true);   // A and C
  const std::string K = filter(ai, bi, oi, true, false);   // A and B
  const std::string N = filter(bi, ai, oi, false, true);   // B and C
  int s = -1;
  bool first = true;
  for (char c : K) {
    const int r = sa(c) * sb(c);
    if (first) {
      s = r;
      first = false;
    } else if (r != s) {
      return false;
    }
  }
  std::vector<int> sgM, sgK, sgN;
  for (char c : M) sgM.push_back(sa(c));
  for (char c : K) sgK.push_back(sa(c));
  for (char c : N) sgN.push_back(sb(c));
  const int np = (int)probs_.size();
  std::vector<SgemmProblem> ps(np);
  std::vector<SgemmTask> tasks;
  struct Tile {
    int p, m0, ml, k0, kl, n0, nl, shape;
  };
  std::vector<Tile> tiles;
  // FTCC_SGEMM_THIN=0: 16 x 16 MFMA tiles for every block; =N: at most N inner
  // steps per lane-mapped wave (diagnostics)
  double bytes = 0.0;
  const char* thin_env = std::getenv("FTCC_SGEMM_THIN");
  const long thin_cap = thin_env ? std::atol(thin_env) : kSgemmThinSteps;
  const bool thin_ok = thin_cap > 0;
  std::vector<double> pf(np, 0.0);
  std::vector<int> pinst(np);
  double flops = 0.0;
  for (int p = 0; p < np; ++p) {
    const int inst = probs_[p].inst;
    const long n = probs_[p].n;
    if (inst < 0 || inst >= (int)mom_.size() || !mom_[inst]) throw std::runtime_error("momentum labels missing");
    if (ipow(n, (int)std::max(std::max(ai.size(), bi.size()), oi.size())) >= (1L << 32))
      throw std::runtime_error("tensor exceeds 2^32 elements: " + tag);
    const GroupTable& TM = group_table(inst, n, M, ai, is_packed(t_a), oi, is_packed(t_out), sgM, 1);
    const GroupTable& TK = group_table(inst, n, K, ai, is_packed(t_a), bi, is_packed(t_b), sgK, 4);
    const GroupTable& TN = group_table(inst, n, N, bi, is_packed(t_b), oi, is_packed(t_out), sgN, 1);
    SgemmProblem& P = ps[p];
    P.A = A[p];
    P.B = B[p];
    P.C = out[p];
    P.offAM = (const unsigned*)TM.off1;
    P.offCM = (const unsigned*)TM.off2;
    P.offAK = (const unsigned*)TK.off1;
    P.offBK = (const unsigned*)TK.off2;
    P.offBN = (const unsigned*)TN.off1;
    P.offCN = (const unsigned*)TN.off2;
    P.alpha = alpha;
    P.beta = acc ? 1.0 : 0.0;
    P.active = gate_for(dst, p);
    P.a_inner = has(K, unit_letter(ai, t_a)) ? 1 : 0;
    P.b_inner = has(K, unit_letter(bi, t_b)) ? 1 : 0;
    pinst[p] = p;
    const InstMomentum& Mm = *mom_[inst];
    struct Block {
      int m0, ml, k0, kl, n0, nl;
    };
    std::vector<Block> blocks;
    long n_wave = 0;   // 16 x 16 tiles of the problem
    for (const auto& blk : TM.blocks) {
      std::vector<int> q(Mm.dims), qk(Mm.dims), qn(Mm.dims);
      for (int c = 0; c < Mm.dims; ++c) {
        q[c] = (int)((blk.first >> (21 * c)) & ((1 << 21) - 1)) - (1 << 19);
        qk[c] = -q[c];
        qn[c] = s * q[c];
        if (Mm.modulus[c] > 0) {
          qk[c] = ((qk[c] % Mm.modulus[c]) + Mm.modulus[c]) % Mm.modulus[c];
          qn[c] = ((qn[c] % Mm.modulus[c]) + Mm.modulus[c]) % Mm.modulus[c];
        }
      }
      auto nb = TN.blocks.find(pack_momentum(qn));
      if (nb == TN.blocks.end()) continue;
      auto kb = TK.blocks.find(pack_momentum(qk));
      const int k0 = kb == TK.blocks.end() ? 0 : kb->second.first;
      const int kl = kb == TK.blocks.end() ? 0 : kb->second.second;
      if (kl == 0 && acc) continue;   // nothing to add; a set writes its zeros
      blocks.push_back(Block{blk.second.first, blk.second.second, k0, kl, nb->second.first, nb->second.second});
      n_wave += (long)((blk.second.second + 15) / 16) * ((nb->second.second + 15) / 16);
    }
    // Waves of 32 x 32 gather each operand element half as often; they pay where a
    // problem alone still has a wave for every CU (81 labelled orbitals, forward: 38.4 ->
    // 35.3 ms; 57, step: 48.0 -> 47.0), not where its parallelism is short (33: 216 -> 223).
    // They take inner ranges of up to 192 whole: 16 x 16 tiles in parts of 64 and their sum
    // cost a step of 123 labelled orbitals 750 ms against 716.
    const bool wide = n_wave >= 256;
    for (const Block& b : blocks) {
      const int m0 = b.m0, ml = b.ml, k0 = b.k0, kl = b.kl, n0 = b.n0, nl = b.nl;
      // With one orbital per momentum the few blocks large enough for tiles gather every
      // element from a line of its own, which the tiles do not change, and their blocks
      // only delay the level (81 orbitals, forward: 40.8 ms with tiles, 38.3 without; 57:
      // no difference).
      int shape = one_per_label_ ? 0 : sgemm_tile_shape(ml, nl, kl);
      int R, C;
      if (shape) {
        R = sgemm_tile_rows(shape);
        C = 4096 / R;
      } else {
        shape = thin_ok ? sgemm_shape(ml, nl, kl, thin_cap) : 0;
        R = shape ? 1 << (shape & 7) : 16;
        C = shape ? 1 << ((shape >> 3) & 7) : 16;
        if (wide && !shape && std::min(ml, nl) > 16 && kl <= 3 * kSgemmChunk) {
          shape = kWave32x32;
          R = C = 32;
        }
      }
      // bands of 8 tile rows, down the rows first, so that neighbouring tiles share both
      // operands' panels (see upload_sgemm)
      for (int band = 0; band < ml; band += 8 * R)
        for (int c = 0; c < nl; c += C)
          for (int r = band; r < std::min(ml, band + 8 * R); r += R)
            tiles.push_back(Tile{p, m0 + r, std::min(R, ml - r), k0, kl, n0 + c, std::min(C, nl - c), shape});
      pf[p] += 2.0 * ml * (double)nl * kl;
      bytes += sizeof(double) * ((double)ml * kl + (double)kl * nl + (double)ml * nl * (acc ? 2 : 1));
    }
    flops += pf[p];
  }
  // A tile with a long inner range would be one wave's long serial chain of
  // dependent gathers: its range is cut into chunks whose partial tiles a
  // second kernel adds in order.  The chunk grows (powers of two) until every
  // partial tile fits the workspace.
  // Block tiles: chunks of at least 16 steps, sized so that one problem alone makes
  // about kTileSpread tasks (by the problem's own tiles only, so that a batch and a
  // single instance add in the same order).
  const long ws_tiles = scratch_ && scratch_->tail_ws ? (long)(scratch_->tail_ws_doubles / 256) : 0;
  auto is_tile = [](const Tile& t) { return t.shape >= kTile64x64; };
  auto steps_of = [](int kl) { return (kl + kTileBK - 1) / kTileBK; };
  std::vector<long> prob_steps(np, 0);
  for (const Tile& t : tiles)
    if (is_tile(t)) prob_steps[t.p] += steps_of(t.kl);
  int chunk = kSgemmChunk, grow = 1;
  auto chunk_of = [&](const Tile& t) {   // inner indices per part; kl: not split
    if (!is_tile(t)) return t.shape || t.kl <= chunk + chunk / 2 ? t.kl : chunk;
    const long per = grow * std::max(16L, (prob_steps[t.p] + kTileSpread - 1) / kTileSpread);
    const long st = steps_of(t.kl);
    if (st <= per + per / 2) return t.kl;
    const long parts = (st + per - 1) / per;
    return (int)((st + parts - 1) / parts) * kTileBK;
  };
  auto units_needed = [&] {
    long n = 0;
    for (const Tile& t : tiles) {
      const int ch = chunk_of(t);
      if (ch < t.kl) n += (long)part_units(t.shape) * ((t.kl + ch - 1) / ch);
    }
    return n;
  };
  while (ws_tiles > 0 && units_needed() > ws_tiles) {
    chunk *= 2;
    grow *= 2;
  }
  std::vector<SgemmReduce> reds;
  int units = 0;
  for (const Tile& t : tiles) {
    const int ch = ws_tiles == 0 ? t.kl : chunk_of(t);
    if (ch >= t.kl) {
      tasks.push_back(SgemmTask{t.p, t.m0, t.ml, t.k0, t.kl, t.n0, t.nl, -1, t.shape});
      continue;
    }
    const int first = units, pu = part_units(t.shape);
    for (int k = 0; k < t.kl; k += ch) {
      tasks.push_back(SgemmTask{t.p, t.m0, t.ml, t.k0 + k, std::min(ch, t.kl - k), t.n0, t.nl, units, t.shape});
      units += pu;
    }
    reds.push_back(SgemmReduce{t.p, t.m0, t.ml, t.n0, t.nl, first, (units - first) / pu, t.shape, 0});
  }
  Launch L;
  for (int p = 0; p < np; ++p) {
    const long n = probs_[p].n;
    add_range(L.rd, A[p], sizeof(double) * elems(t_a, n, (int)ai.size()));
    add_range(L.rd, B[p], sizeof(double) * elems(t_b, n, (int)bi.size()));
    add_range(L.wr, out[p], sizeof(double) * elems(t_out, n, (int)oi.size()));
  }
  L.ranged = true;
  L.bytes = bytes;
  L.sprobs = ps;
  L.stasks = tasks;
  L.sreds = reds;
  L.kind = Launch::SGEMM;
  upload_sgemm(L);
  L.flops = flops;
  if (&dst != &setup_) {
    L.prob_flops = pf;
    L.prob_gate = pinst;
  }
  L.tag = tag + "(blocked)";
  dst.push_back(L);
  return true;
}

// Y[yi] = alpha X[xi] + beta Y over the allowed elements of Y (its law known).
bool Executor::elem_blocked(std::vector<Launch>& dst, const PerProb& X, const std::string& xi, const PerProb& Y,
                            const std::string& yi, double alpha, double beta, int t_y, int t_x,
                            const std::string& tag, const std::vector<const double*>* scale, int xp, int yp) {
  std::vector<SumTerm> terms;
  if (alpha != 0.0) {
    SumTerm t{X, xi, t_x, alpha, {}, xp};
    if (scale) t.scale = *scale;
    terms.push_back(t);
  }
  return sum_blocked(dst, terms, Y, yi, beta, t_y, tag, yp);
}

// Elementwise launches address their elements through one list per tensor where every
// orbital has its own label: the pairs of index groups would be a task of a few elements
// each, and finding an element's task took longer than its value.
bool Executor::flat_lists(int rank) const { return one_per_label_ && rank >= 2 && rank <= 4; }

// Sums do so for other problems of at most kFlatElements elements too: their launches are
// as much bound by the chain of dependent loads (6 dense orbitals, a step: 13.35 -> 12.9 ms; a
// spin ring of 12 21.4 -> 20.8); larger ones would read as many offsets as values.
constexpr size_t kFlatElements = 1 << 17;
bool Executor::flat_sums(int rank, const std::vector<int>& signs) {
  if (flat_lists(rank)) return true;
  if (rank < 2 || rank > 4) return false;
  for (const ProblemRef& p : probs_)
    if (ipow(p.n, rank) > (1L << 20) || allowed_tuples(p.inst, p.n, signs).size() > kFlatElements) return false;
  return true;
}

// Y[yi] = beta Y + sum_s alpha_s X_s[xi_s] over the allowed elements of Y (its law known):
// Y's letters split into two halves whose momentum blocks q and -q pair up.
// Returns false (dense lowering) when a law is unknown.
bool Executor::sum_blocked(std::vector<Launch>& dst, const std::vector<SumTerm>& terms, const PerProb& Y,
                           const std::string& yi, double beta, int t_y, const std::string& tag, int yp) {
  const bool ypk = yp >= 0 ? yp != 0 : is_packed(t_y);
  if (mom_.empty() || t_y < 0 || !law_ok_[t_y] || yi.empty()) return false;
  const std::vector<int>& ly = law_[t_y];
  // every operand's law must describe the same allowed set (equal or opposite signs)
  for (const SumTerm& s : terms) {
    if (s.t_x < 0 || !law_ok_[s.t_x]) return false;
    int rel = 0;
    for (size_t a = 0; a < yi.size(); ++a) {
      const int r = ly[a] * law_[s.t_x][s.xi.find(yi[a])];
      if (rel == 0) rel = r;
      else if (r != rel) return false;
    }
  }
  const std::string G1 = yi.substr(0, yi.size() / 2), G2 = yi.substr(yi.size() / 2);
  const std::vector<int> s1(ly.begin(), ly.begin() + G1.size()), s2(ly.begin() + G1.size(), ly.end());
  const int np = (int)probs_.size();
  Launch L;
  double elements = 0.0;
  const bool flat = flat_sums((int)yi.size(), ly);
  for (int p = 0; p < np; ++p) {
    const int inst = probs_[p].inst;
    const long n = probs_[p].n;
    if (ipow(n, (int)yi.size()) >= (1L << 32)) throw std::runtime_error("tensor exceeds 2^32 elements: " + tag);
    ElemProblem P;
    P.Y = Y[p];
    if (flat) {
      P.oy1 = zero_offset();
      P.oy2 = offset_list(inst, n, yi, ly, yi, ypk);
    } else {
      P.oy1 = (const unsigned*)group_table(inst, n, G1, yi, ypk, yi, ypk, s1).off2;
      P.oy2 = (const unsigned*)group_table(inst, n, G2, yi, ypk, yi, ypk, s2).off2;
    }
    P.beta = beta;
    P.active = gate_for(dst, p);
    P.src = (int)L.esrcs.size();
    P.n_src = (int)terms.size();
    const size_t ey = sizeof(double) * (size_t)ipow_l(n, (int)yi.size() - (ypk ? 1 : 0));
    if (beta != 0.0) add_range(L.rd, Y[p], ey);
    add_range(L.wr, Y[p], ey);
    for (const SumTerm& s : terms) {
      const bool xpk = s.xp >= 0 ? s.xp != 0 : is_packed(s.t_x);
      ElemSource q;
      q.X = s.X[p];
      q.ox1 = q.ox2 = nullptr;
      if (flat && (s.xi != yi || xpk != ypk)) {
        q.ox1 = zero_offset();
        q.ox2 = offset_list(inst, n, yi, ly, s.xi, xpk);
      } else if (s.xi != yi || xpk != ypk) {   // the same tuples in the same order, X's offsets
        q.ox1 = (const unsigned*)group_table(inst, n, G1, s.xi, xpk, yi, ypk, s1).off1;
        q.ox2 = (const unsigned*)group_table(inst, n, G2, s.xi, xpk, yi, ypk, s2).off1;
      }
      q.scale = s.scale.empty() ? nullptr : s.scale[p];
      q.alpha = s.alpha;
      L.esrcs.push_back(q);
      add_range(L.rd, q.X, sizeof(double) * (size_t)ipow_l(n, (int)yi.size() - (xpk ? 1 : 0)));
      if (q.scale) add_range(L.rd, q.scale, sizeof(double));
    }
    L.eprobs.push_back(P);
    if (flat) {
      const int count = (int)allowed_tuples(inst, n, ly).size();
      if (count) L.etasks.push_back(ElemTask{L.n_elem, p, 0, 1, 0, count});
      L.n_elem += count;
      elements += (double)count;
      continue;
    }
    const GroupTable& T1 = group_table(inst, n, G1, yi, ypk, yi, ypk, s1);
    const GroupTable& T2 = group_table(inst, n, G2, yi, ypk, yi, ypk, s2);
    const InstMomentum& Mm = *mom_[inst];
    for (const auto& blk : T1.blocks) {
      std::vector<int> q(Mm.dims);
      for (int c = 0; c < Mm.dims; ++c) {
        q[c] = -((int)((blk.first >> (21 * c)) & ((1 << 21) - 1)) - (1 << 19));
        if (Mm.modulus[c] > 0) q[c] = ((q[c] % Mm.modulus[c]) + Mm.modulus[c]) % Mm.modulus[c];
      }
      auto b2 = T2.blocks.find(pack_momentum(q));
      if (b2 == T2.blocks.end()) continue;
      L.etasks.push_back(
          ElemTask{L.n_elem, p, blk.second.first, blk.second.second, b2->second.first, b2->second.second});
      L.n_elem += (long long)blk.second.second * b2->second.second;
      elements += (double)blk.second.second * b2->second.second;
    }
  }
  L.ranged = true;
  L.flat = flat;
  L.kind = Launch::ELEM;
  L.bytes = sizeof(double) * elements * ((double)terms.size() + (beta != 0.0) + 1);
  L.tag = tag + "(blocked)";
  upload_elem(L);
  dst.push_back(L);
  return true;
}

void Executor::upload_elem(Launch& L) {
  if (defer_) return;
  L.n_prob = (int)L.eprobs.size();
  L.d_desc = upload(L.eprobs.data(), sizeof(ElemProblem) * L.eprobs.size());
  L.d_src = upload(L.esrcs.data(), sizeof(ElemSource) * L.esrcs.size());
  L.n_tasks = (int)L.etasks.size();
  // Four elements a thread where the launch's tasks fill blocks of that many on average
  // (dense orbitals: the task is then uniform over a block) and give every CU one; one
  // where the tasks are smaller (labels: a block of 1024 spans tasks, every thread
  // searches for each of its elements in turn and a problem's last block is mostly
  // padding; 10 orbitals, 12 instances: 32.6 ms a step with four, 27.0 with one) or the
  // launch is (6 dense orbitals: 19.2 against 18.6).
  L.elem_per = L.n_elem >= std::max(1024LL * L.n_tasks, 1024LL * 256) ? 4 : 1;
  L.n_flat = 0;
  if (L.flat && L.elem_per == 1) {
    std::vector<ElemBlock> blocks;
    for (const ElemTask& T : L.etasks)
      for (int k = 0; k < T.vlen; k += 256) blocks.push_back(ElemBlock{T.prob, k, T.vlen});
    L.n_flat = L.total = (int)blocks.size();
    L.d_tasks = upload(blocks.data(), sizeof(ElemBlock) * blocks.size());
    return;
  }
  const long long block = 256 * L.elem_per;
  long long first = 0;
  for (size_t t = 0; t < L.etasks.size(); ++t) {
    ElemTask& T = L.etasks[t];
    if (t && T.prob != L.etasks[t - 1].prob) first = (first + block - 1) / block * block;   // a block, one problem
    T.first = first;
    first += (long long)T.ulen * T.vlen;
  }
  L.n_elem = first;
  L.d_tasks = upload(L.etasks.data(), sizeof(ElemTask) * L.etasks.size());
  const std::vector<int> bf = block_first_tasks(L.etasks, L.n_elem, (int)block);
  L.d_bfirst = upload(bf.data(), sizeof(int) * bf.size());
  L.total = (int)std::min<long long>((L.n_elem + block - 1) / block, 1 << 30);
}

bool Executor::dot_blocked(std::vector<Launch>& dst, const PerProb& A, const std::string& ai, const PerProb& B,
                           const std::string& bi, const PerProb& out, double alpha, double beta, int t_a, int t_b,
                           const std::string& tag) {
  if (mom_.empty() || t_a < 0 || !law_ok_[t_a] || ai.empty() || !scratch_ || !scratch_->tail_ws) return false;
  const std::vector<int>& la = law_[t_a];
  const std::string G1 = ai.substr(0, ai.size() / 2), G2 = ai.substr(ai.size() / 2);
  const std::vector<int> s1(la.begin(), la.begin() + G1.size()), s2(la.begin() + G1.size(), la.end());
  const int np = (int)probs_.size();
  std::vector<DotbProblem> ps(np);
  const bool flat = flat_lists((int)ai.size());
  std::vector<ElemTask> tasks;
  long long total = 0;
  for (int p = 0; p < np; ++p) {
    const int inst = probs_[p].inst;
    const long n = probs_[p].n;
    if (ipow(n, (int)ai.size()) >= (1L << 32)) throw std::runtime_error("tensor exceeds 2^32 elements: " + tag);
    DotbProblem& P = ps[p];
    P.X = A[p];
    P.Y = B[p];
    P.out = out[p];
    P.alpha = alpha;
    P.beta = beta;
    P.active = gate_for(dst, p);
    total = (total + 255) / 256 * 256;     // every problem starts on a block boundary
    const long long start = total;
    P.first_block = (int)(start / 256);
    if (flat) {
      const int count = (int)allowed_tuples(inst, n, la).size();
      P.ox1 = P.oy1 = zero_offset();
      P.ox2 = offset_list(inst, n, ai, la, ai, is_packed(t_a));
      P.oy2 = offset_list(inst, n, ai, la, bi, is_packed(t_b));
      if (count) tasks.push_back(ElemTask{total, p, 0, 1, 0, count});
      total += count;
      P.n_blocks = (count + 255) / 256;
      continue;
    }
    // A's allowed elements: index groups G1 of momentum q with G2 of momentum -q
    const GroupTable& T1 = group_table(inst, n, G1, ai, is_packed(t_a), bi, is_packed(t_b), s1);
    const GroupTable& T2 = group_table(inst, n, G2, ai, is_packed(t_a), bi, is_packed(t_b), s2);
    P.ox1 = (const unsigned*)T1.off1;
    P.oy1 = (const unsigned*)T1.off2;
    P.ox2 = (const unsigned*)T2.off1;
    P.oy2 = (const unsigned*)T2.off2;
    const InstMomentum& Mm = *mom_[inst];
    for (const auto& blk : T1.blocks) {
      std::vector<int> q(Mm.dims);
      for (int c = 0; c < Mm.dims; ++c) {
        q[c] = -((int)((blk.first >> (21 * c)) & ((1 << 21) - 1)) - (1 << 19));
        if (Mm.modulus[c] > 0) q[c] = ((q[c] % Mm.modulus[c]) + Mm.modulus[c]) % Mm.modulus[c];
      }
      auto b2 = T2.blocks.find(pack_momentum(q));
      if (b2 == T2.blocks.end()) continue;
      tasks.push_back(ElemTask{total, p, blk.second.first, blk.second.second, b2->second.first, b2->second.second});
      total += (long long)blk.second.second * b2->second.second;
    }
    P.n_blocks = (int)((total - start + 255) / 256);
  }
  if ((total + 255) / 256 > (long long)scratch_->tail_ws_doubles) return false;
  Launch L;
  for (int p = 0; p < np; ++p) {
    const long n = probs_[p].n;
    add_range(L.rd, A[p], sizeof(double) * elems(t_a, n, (int)ai.size()));
    add_range(L.rd, B[p], sizeof(double) * elems(t_b, n, (int)bi.size()));
    add_range(L.wr, out[p], sizeof(double));
  }
  L.ranged = true;
  L.kind = Launch::DOTB;
  L.n_prob = np;
  L.d_desc = upload(ps.data(), sizeof(DotbProblem) * np);
  L.n_tasks = (int)tasks.size();
  L.d_tasks = upload(tasks.data(), sizeof(ElemTask) * std::max<size_t>(tasks.size(), 1));
  {
    const std::vector<int> bf = block_first_tasks(tasks, total, 256);
    L.d_bfirst = upload(bf.data(), sizeof(int) * bf.size());
  }
  L.n_elem = total;
  L.bytes = 2.0 * sizeof(double) * (double)total;
  L.d_partial = scratch_->tail_ws;
  L.tag = tag + "(blocked dot)";
  dst.push_back(L);
  return true;
}

double Executor::sgemm_flops_forward() const {
  double f = 0.0;
  for (const Launch& l : fwd_)
    if (l.kind == Launch::SGEMM) f += l.flops;
  return f;
}

// Order of n block tile tasks from `begin` over the chip: block b runs on XCD b % 8,
// and each XCD has its own L2, so every run of equally long tasks is cut into eight
// contiguous pieces, one per XCD (neighbouring tiles share operand panels), while
// the list as a whole stays longest first.
static void xcd_order(std::vector<SgemmTask>& all, int begin, int n, int n_prob) {
  constexpr int X = 8;
  std::vector<SgemmTask> q[X], tasks(all.begin() + begin, all.begin() + begin + n);
  for (int i = 0, turn = 0; i < n; ++turn) {
    int j = i;
    while (j < n && tasks[j].klen == tasks[i].klen && tasks[j].prob / n_prob == tasks[i].prob / n_prob) ++j;
    for (int x = 0; x < X; ++x) {
      const int lo = i + (int)((long)(j - i) * x / X), hi = i + (int)((long)(j - i) * (x + 1) / X);
      std::vector<SgemmTask>& t = q[(x + turn) % X];
      t.insert(t.end(), tasks.begin() + lo, tasks.begin() + hi);
    }
    i = j;
  }
  size_t at[X] = {};
  for (int i = 0; i < n; ++i) {
    int x = i % X;
    for (int k = 0; k < X && at[x] >= q[x].size(); ++k) x = (x + 1) % X;   // that XCD's share is used up
    all[begin + i] = q[x][at[x]++];
  }
}

// Device lists of an SGEMM launch: block tiles first, longest tasks first (so that
// the last wave of the launch holds short ones), one reduction entry per 256 outputs.
void Executor::upload_sgemm(Launch& L) {
  if (defer_) return;
  std::stable_sort(L.stasks.begin(), L.stasks.end(),
                   [](const SgemmTask& a, const SgemmTask& b) { return sgemm_task_cost(a) > sgemm_task_cost(b); });
  L.n_prob = (int)L.sprobs.size();
  L.d_desc = upload(L.sprobs.data(), sizeof(SgemmProblem) * L.sprobs.size());
  L.n_tasks = (int)L.stasks.size();
  L.n_square = L.n_narrow = 0;
  L.wide = false;
  for (const SgemmTask& t : L.stasks) {
    L.n_square += t.shape == kTile64x64;
    L.wide = L.wide || t.shape == kWave32x32;
    L.n_narrow += t.shape > kTile64x64;
  }
  xcd_order(L.stasks, 0, L.n_square, (int)probs_.size());
  xcd_order(L.stasks, L.n_square, L.n_narrow, (int)probs_.size());
  L.d_tasks = upload(L.stasks.data(), sizeof(SgemmTask) * std::max<size_t>(L.stasks.size(), 1));
  std::vector<SgemmReduce> slices;
  for (const SgemmReduce& r : L.sreds)
    for (int k = 0; k < part_units(r.shape); ++k) {
      slices.push_back(r);
      slices.back().slice = k;
    }
  L.n_red = (int)slices.size();
  if (L.n_red > 0) L.d_red = upload(slices.data(), sizeof(SgemmReduce) * slices.size());
  L.d_partial = scratch_->tail_ws;
  const int blocks = L.n_square + L.n_narrow;
  L.total = blocks + (L.n_tasks - blocks + 3) / 4;
}

Launch Executor::merge_sgemm(const std::vector<Launch*>& parts) {
  Launch M;
  M.kind = Launch::SGEMM;
  M.ranged = true;
  int part_base = 0;
  for (const Launch* l : parts) {
    const int po = (int)M.sprobs.size();
    M.sprobs.insert(M.sprobs.end(), l->sprobs.begin(), l->sprobs.end());
    for (SgemmTask t : l->stasks) {
      t.prob += po;
      if (t.part >= 0) t.part += part_base;
      M.stasks.push_back(t);
    }
    int n_parts = 0;
    for (SgemmReduce r : l->sreds) {
      r.prob += po;
      r.first += part_base;
      n_parts += r.count * part_units(r.shape);
      M.sreds.push_back(r);
    }
    part_base += n_parts;
    M.flops += l->flops;
    M.bytes += l->bytes;
    M.prob_flops.insert(M.prob_flops.end(), l->prob_flops.begin(), l->prob_flops.end());
    M.prob_gate.insert(M.prob_gate.end(), l->prob_gate.begin(), l->prob_gate.end());
    M.rd.insert(M.rd.end(), l->rd.begin(), l->rd.end());
    M.wr.insert(M.wr.end(), l->wr.begin(), l->wr.end());
    M.tag += (M.tag.empty() ? "" : "+") + l->tag;
  }
  normalize(M.rd);
  normalize(M.wr);
  upload_sgemm(M);
  return M;
}

Launch Executor::merge_elem(const std::vector<Launch*>& parts) {
  Launch M;
  M.kind = Launch::ELEM;
  M.ranged = M.flat = true;
  for (const Launch* l : parts) {
    const int po = (int)M.eprobs.size(), so = (int)M.esrcs.size();
    for (ElemProblem q : l->eprobs) {
      q.src += so;
      M.eprobs.push_back(q);
    }
    M.esrcs.insert(M.esrcs.end(), l->esrcs.begin(), l->esrcs.end());
    for (ElemTask t : l->etasks) {
      t.prob += po;
      M.etasks.push_back(t);
    }
    M.n_elem += l->n_elem;
    M.flat = M.flat && l->flat;
    M.bytes += l->bytes;
    M.rd.insert(M.rd.end(), l->rd.begin(), l->rd.end());
    M.wr.insert(M.wr.end(), l->wr.begin(), l->wr.end());
    M.tag += (M.tag.empty() ? "" : "+") + l->tag;
  }
  normalize(M.rd);
  normalize(M.wr);
  upload_elem(M);
  return M;
}

void Executor::fuse_levels(std::vector<Launch>& L) {
  defer_ = false;
  const int nL = (int)L.size();
  for (Launch& l : L) {
    normalize(l.rd);
    normalize(l.wr);
  }
  // level: one more than the highest level of any earlier launch it must follow
  std::vector<int> level(nL, 0);
  int top = 0;
  for (int i = 0; i < nL; ++i) {
    int lv = 0;
    for (int j = i - 1; j >= 0; --j)
      if (level[j] + 1 > lv && ordered(L[j], L[i])) lv = level[j] + 1;
    level[i] = lv;
    top = std::max(top, lv);
  }
  std::vector<std::vector<int>> at(top + 1);
  for (int i = 0; i < nL; ++i) at[level[i]].push_back(i);
  const long ws_tiles = scratch_ && scratch_->tail_ws ? (long)(scratch_->tail_ws_doubles / 256) : 0;
  std::vector<Launch> out;
  for (const std::vector<int>& lv : at) {
    std::vector<Launch*> sg, el;
    for (int i : lv) {
      Launch& l = L[i];
      if (l.kind == Launch::SGEMM && !l.sprobs.empty()) sg.push_back(&l);
      else if (l.kind == Launch::ELEM && !l.eprobs.empty()) el.push_back(&l);
      else out.push_back(std::move(l));
    }
    if (el.size() == 1) {
      out.push_back(std::move(*el[0]));
    } else if (el.size() > 1) {
      out.push_back(merge_elem(el));
    }
    // blocked contractions: one launch while their partial tiles fit the workspace
    size_t k = 0;
    while (k < sg.size()) {
      std::vector<Launch*> grp;
      long parts = 0;
      for (; k < sg.size(); ++k) {
        long np = 0;
        for (const SgemmReduce& r : sg[k]->sreds) np += r.count * part_units(r.shape);
        if (!grp.empty() && parts + np > ws_tiles) break;
        grp.push_back(sg[k]);
        parts += np;
      }
      if (grp.size() == 1) {
        out.push_back(std::move(*grp[0]));
      } else {
        out.push_back(merge_sgemm(grp));
      }
    }
  }
  for (Launch& l : out) {   // upload what was not merged; the host copies are no longer needed
    if (l.kind == Launch::SGEMM && !l.d_desc) upload_sgemm(l);
    if (l.kind == Launch::ELEM && !l.d_desc) upload_elem(l);
    std::vector<SgemmProblem>().swap(l.sprobs);
    std::vector<SgemmTask>().swap(l.stasks);
    std::vector<SgemmReduce>().swap(l.sreds);
    std::vector<ElemProblem>().swap(l.eprobs);
    std::vector<ElemSource>().swap(l.esrcs);
    std::vector<ElemTask>().swap(l.etasks);
  }
  L = std::move(out);
}

// ------------------------------------------------------------------ lowering: op lists
void Executor::lower_one(std::vector<Launch>& dst, const OpInst& o, const PerProb& out, bool acc) {
  contract(dst, out, o.oi, o.alpha, *o.A, o.ai, o.a_const, o.B, o.bi, o.b_const, acc, o.tag, o.a_val, o.b_val,
           o.t_out, o.t_a, o.t_b);
  if (&dst == &fwd_) version_[o.t_out]++;
}

// Lower a list of ops; the buffers of `zeroed` (gradients, key number of tensors + k)
// start at zero.
//
// Without momentum laws: one launch (or GEMM and permute) per op, in order.
// With them the launches later run by dependency level, and the ops that accumulate
// into one buffer would stand in one level each, since its writes keep their order:
// 11 for the doubles residual.  Instead every run of writes with no read in between
// is taken together: contractions write private copies (the first one the buffer
// itself), and one elementwise sum adds the copies and the elementwise terms in op
// order.  A contraction whose operands are ready later than everything else
// accumulates in place after that sum.  27 -> 14 launches per forward pass of the
// restricted program at 6 orbitals (6 sums, 6 contraction levels, 2 dots), 40 -> 13 per
// reverse pass.  Copies are taken only while memory
// is plentiful (cache_alloc); without them the writes are serial.
void Executor::lower(std::vector<Launch>& dst, const std::vector<OpInst>& ops, const std::vector<int>& zeroed,
                     const std::vector<PerProb>& zero_bufs) {
  const int nt = (int)prog_->t.size(), np = (int)probs_.size();
  auto rank_of = [&](int t) { return prog_->t[t].rank; };
  std::map<int, int> fresh;   // key -> index in zeroed, until its first write
  for (size_t k = 0; k < zeroed.size(); ++k) fresh[nt + zeroed[k]] = (int)k;
  if (mom_.empty()) {
    for (size_t k = 0; k < zeroed.size(); ++k)
      fill(dst, zero_bufs[k], rank_of(zeroed[k]), "zero:" + prog_->t[zeroed[k]].name, zeroed[k]);
    for (const OpInst& o : ops) lower_one(dst, o, *o.out, o.acc);
    return;
  }
  // the elementwise form of an op with one operand, or one operand and a scalar
  auto unary = [](const OpInst& o) { return !o.B || o.ai.empty() || o.bi.empty(); };
  auto term_of = [&](const OpInst& o) {   // letters renamed by their place in the output
    const bool sa = o.B && o.ai.empty(), sb = o.B && o.bi.empty();
    SumTerm t{sa ? *o.B : *o.A, sa ? o.bi : o.ai, sa ? o.t_b : o.t_a, o.alpha, {}, -1};
    if (sa) t.scale.assign(o.A->begin(), o.A->end());
    if (sb) t.scale.assign(o.B->begin(), o.B->end());
    for (char& c : t.xi) c = (char)('A' + o.oi.find(c));
    return t;
  };
  std::map<int, int> level;   // of a buffer's last write
  auto lv = [&](int key) {
    auto it = level.find(key);
    return it == level.end() ? 0 : it->second;
  };
  auto ready = [&](const OpInst& o) { return std::max(lv(o.akey), o.bkey >= 0 ? lv(o.bkey) : 0) + 1; };
  std::map<int, std::vector<const OpInst*>> open;
  auto close = [&](int key) {
    auto it = open.find(key);
    if (it == open.end()) {
      auto f = fresh.find(key);   // read before any write: zero
      if (f == fresh.end()) return;
      const int k = f->second;
      fresh.erase(f);
      fill(dst, zero_bufs[k], rank_of(zeroed[k]), "zero:" + prog_->t[zeroed[k]].name, zeroed[k]);
      level[key] = 1;
      return;
    }
    const std::vector<const OpInst*> seg = std::move(it->second);
    open.erase(it);
    const PerProb& out = *seg[0]->out;
    const int t_out = seg[0]->t_out, r = rank_of(t_out);
    const bool acc0 = fresh.count(key) ? false : seg[0]->acc;
    fresh.erase(key);
    std::vector<const OpInst*> un, con;
    for (const OpInst* o : seg) (unary(*o) ? un : con).push_back(o);
    std::string yi;
    for (int k = 0; k < r; ++k) yi.push_back((char)('A' + k));
    // the contraction to accumulate in place, last: the only one ready strictly after the others and their sum
    const OpInst* last = nullptr;
    int top = 0, rest = 0;
    for (const OpInst* o : con) top = std::max(top, ready(*o));
    int at_top = 0;
    for (const OpInst* o : con)
      if (ready(*o) == top) {
        ++at_top;
        last = o;
      } else {
        rest = std::max(rest, ready(*o));
      }
    for (const OpInst* o : un) rest = std::max(rest, ready(*o) - 1);
    if (at_top != 1 || (con.size() > 1 && rest + 1 >= top)) last = nullptr;
    if (last) con.erase(std::find(con.begin(), con.end(), last));
    bool acc = acc0;
    // private copies of every contraction but the first
    std::vector<SumTerm> copies;
    bool serial = false;
    for (size_t k = 1; k < con.size() && !serial; ++k) {
      size_t total = 0;
      for (int p = 0; p < np; ++p) total += (elems(t_out, probs_[p].n, r) + 31) / 32 * 32;
      double* q = cache_alloc_ ? cache_alloc_(total) : nullptr;
      if (!q) {
        serial = true;
        break;
      }
      cache_bytes_ += sizeof(double) * total;
      SumTerm t{PerProb(np), yi, t_out, 1.0, {}, -1};
      for (int p = 0; p < np; ++p) {
        t.X[p] = q;
        q += (elems(t_out, probs_[p].n, r) + 31) / 32 * 32;
      }
      copies.push_back(t);
    }
    if (serial) copies.clear();
    if (!con.empty() && !serial) {
      lower_one(dst, *con[0], out, acc);
      acc = true;
      for (size_t k = 1; k < con.size(); ++k) lower_one(dst, *con[k], copies[k - 1].X, false);
    }
    std::vector<SumTerm> terms;
    {
      size_t c = 0;
      for (const OpInst* o : seg) {
        if (unary(*o)) terms.push_back(term_of(*o));
        else if (o != last && !serial && o != con[0]) terms.push_back(copies[c++]);
      }
    }
    if (!terms.empty()) {
      if (!sum_blocked(dst, terms, out, yi, acc ? 1.0 : 0.0, t_out, seg[0]->tag)) {
        for (const OpInst* o : un) {   // no common law: one dense pass each
          lower_one(dst, *o, out, acc);
          acc = true;
        }
        for (const SumTerm& t : copies) {
          dense_guard(seg[0]->tag, {t_out});
          perm(dst, t.X, yi, out, yi, 1.0, 1.0, nullptr, seg[0]->tag);
        }
      }
      acc = true;
    }
    if (serial)
      for (const OpInst* o : con) {
        lower_one(dst, *o, out, acc);
        acc = true;
      }
    if (last) lower_one(dst, *last, out, acc);
    int done = rest;   // of the others, then their sum, then the contraction in place
    if (!last && !con.empty()) done = std::max(done, top);
    if (!terms.empty()) ++done;
    if (last) done = std::max(top, done + 1);
    level[key] = std::max(done, 1);
  };
  for (const OpInst& o : ops) {
    close(o.akey);
    if (o.bkey >= 0) close(o.bkey);
    if (o.oi.empty()) {   // a full contraction: a dot, in order
      auto f = fresh.find(o.okey);
      const bool acc = f == fresh.end() && o.acc;
      fresh.erase(o.okey);
      lower_one(dst, o, *o.out, acc);
      level[o.okey] = std::max(lv(o.okey), ready(o));
      continue;
    }
    open[o.okey].push_back(&o);
  }
  while (!open.empty()) close(open.begin()->first);
  while (!fresh.empty()) close(fresh.begin()->first);
}

// ------------------------------------------------------------------ build
void Executor::build(const Program* prog, const std::vector<ProblemRef>& probs, Binder bind, Scratch* scratch,
                     std::function<double*(int, size_t)> const_alloc, bool want_backward,
                     const std::vector<int>& const_grads, std::function<double*(size_t)> cache_alloc,
                     size_t cache_budget) {
  cache_alloc_ = cache_alloc;
  cache_budget_ = cache_budget;
  if (!prog->finalized()) throw std::runtime_error("Program::finalize() not called");
  prog_ = prog;
  probs_ = probs;
  scratch_ = scratch;
  const_alloc_ = const_alloc;
  if (!mom_.empty()) infer_laws();
  plan_packing(want_backward);
  {
    const char* fz = std::getenv("FTCC_FUSE");
    defer_ = !mom_.empty() && !(fz && fz[0] == '0');
  }
  same_labels_.clear();
  for (size_t i = 0; i < mom_.size(); ++i) {
    size_t j = 0;
    while (j < i && !(mom_[j] && mom_[i] && mom_[j]->dims == mom_[i]->dims && mom_[j]->modulus == mom_[i]->modulus &&
                      mom_[j]->labels == mom_[i]->labels))
      ++j;
    same_labels_.push_back((int)j);
  }
  const int zero = 0;
  d_zero_ = (int*)upload(&zero, sizeof(int));
  const int np = (int)probs.size();
  const int nt = (int)prog->t.size();
  std::vector<PerProb> fwd(nt, PerProb(np)), grd(nt, PerProb(np));
  std::vector<bool> need_grad(nt, false);
  for (int k = 0; k < nt; ++k) {
    const TensorDecl& d = prog->t[k];
    for (int p = 0; p < np; ++p) fwd[k][p] = bind(k, p, false, elems(k, probs[p].n, d.rank));
    bool g = (d.kind == T_INPUT || d.kind == T_OUTPUT || (d.kind == T_INTER && (!d.derived || inline_setup_)));
    if (std::find(const_grads.begin(), const_grads.end(), k) != const_grads.end()) g = true;
    need_grad[k] = g && want_backward;
    if (need_grad[k])
      for (int p = 0; p < np; ++p) grd[k][p] = bind(k, p, true, elems(k, probs[p].n, d.rank));
  }
  auto cidx = [&](int k) {
    return (k >= 0 && (prog->t[k].kind == T_CONST || (prog->t[k].derived && !inline_setup_))) ? k : -1;
  };
  // set-up ops first (constants only), once per instance
  if (!inline_setup_) {
    std::vector<ProblemRef> firsts;
    std::vector<int> idx;
    std::vector<bool> seen_inst;
    for (int p = 0; p < np; ++p) {
      const int inst = probs[p].inst;
      if (inst >= (int)seen_inst.size()) seen_inst.resize(inst + 1, false);
      if (seen_inst[inst]) continue;
      seen_inst[inst] = true;
      firsts.push_back(probs[p]);
      idx.push_back(p);
    }
    auto sub = [&](const PerProb& v) {
      PerProb r;
      for (int p : idx) r.push_back(v[p]);
      return r;
    };
    Scratch firsts_scratch;
    firsts_scratch.a = sub(scratch->a);
    firsts_scratch.b = sub(scratch->b);
    firsts_scratch.c = sub(scratch->c);
    firsts_scratch.part = sub(scratch->part);
    firsts_scratch.dot_partial = scratch->dot_partial;
    probs_ = firsts;
    scratch_ = &firsts_scratch;
    // with momentum laws: one elementwise sum per derived constant (its ops are elementwise)
    std::map<int, std::vector<const SymOp*>> by_out;
    std::vector<int> order;
    for (const SymOp& o : prog->ops) {
      if (!o.setup) continue;
      if (by_out[o.out].empty()) order.push_back(o.out);
      by_out[o.out].push_back(&o);
    }
    for (int out : order) {
      std::vector<SumTerm> terms;
      const std::vector<const SymOp*>& list = by_out[out];
      for (const SymOp* o : list)
        if (o->b < 0) {
          SumTerm t{sub(fwd[o->a]), o->ai, o->a, o->alpha, {}, -1};
          for (char& ch : t.xi) ch = (char)('A' + o->oi.find(ch));
          terms.push_back(t);
        }
      std::string yi;
      for (int k = 0; k < prog->t[out].rank; ++k) yi.push_back((char)('A' + k));
      if (terms.size() == list.size() && !list[0]->accumulate &&
          sum_blocked(setup_, terms, sub(fwd[out]), yi, 0.0, out, "setup:" + prog->t[out].name))
        continue;
      for (const SymOp* o : list) {
        PerProb ob;
        if (o->b >= 0) ob = sub(fwd[o->b]);
        contract(setup_, sub(fwd[o->out]), o->oi, o->alpha, sub(fwd[o->a]), o->ai, -1, o->b >= 0 ? &ob : nullptr,
                 o->bi, -1, o->accumulate, "setup:" + prog->t[o->out].name, -1, -1, o->out, o->a, o->b);
      }
    }
    // Packed copies of the constants the blocked ops read, gathered from the dense
    // blocks (after the derived ones are made) each time the set-up list runs; the
    // program then reads the copies.
    for (int k : plan_const_packing(const_grads)) {
      const TensorDecl& d = prog->t[k];
      std::string ix;
      for (int a = 0; a < d.rank; ++a) ix.push_back((char)('p' + a));
      PerProb pk;
      std::map<int, double*> of_inst;
      for (const ProblemRef& f : firsts) {
        const size_t cnt = (size_t)ipow_l(f.n, d.rank - 1);
        double* q = const_alloc_(f.inst, cnt);
        const_bytes_ += sizeof(double) * cnt;
        of_inst[f.inst] = q;
        pk.push_back(q);
      }
      if (!elem_blocked(setup_, sub(fwd[k]), ix, pk, ix, 1.0, 0.0, k, k, "setup:pack:" + d.name, nullptr, 0, 1))
        throw std::runtime_error("no packed copy of constant " + d.name);
      for (int p = 0; p < np; ++p) fwd[k][p] = of_inst[probs[p].inst];
      packed_[k] = 1;
    }
    probs_ = probs;
    scratch_ = scratch;
  }
  // rank >= 2 inputs, outputs and their gradients in packed buffers
  if (packed_io_)
    for (int k : plan_io_packing()) packed_[k] = 1;
  version_.assign(nt, 0);
  auto vidx = [&](int k) { return (k >= 0 && cidx(k) < 0) ? k : -1; };
  // buffer keys of the op lists: a tensor's values k, its gradient nt + k
  std::vector<OpInst> ops;
  for (const SymOp& o : prog->ops) {
    if (o.setup && !inline_setup_) continue;
    ops.push_back(OpInst{o.out, o.a, o.b, &fwd[o.out], &fwd[o.a], o.b >= 0 ? &fwd[o.b] : nullptr, o.oi, o.ai, o.bi,
                         o.alpha, o.accumulate, cidx(o.a), cidx(o.b), vidx(o.a), vidx(o.b), o.out, o.a, o.b,
                         prog->t[o.out].name});
  }
  lower(fwd_, ops, {}, {});
  if (!want_backward) {
    const char* fz = std::getenv("FTCC_FUSE");
    if (!mom_.empty() && !(fz && fz[0] == '0')) {
      fuse_levels(setup_);
      fuse_levels(fwd_);
    }
    end_uploads();
    dump_plan();
    return;
  }
  // every gradient buffer except the cotangents of the outputs starts at zero
  std::vector<int> zeroed;
  std::vector<PerProb> zero_bufs;
  for (int k = 0; k < nt; ++k)
    if (need_grad[k] && prog->t[k].kind != T_OUTPUT) {
      zeroed.push_back(k);
      zero_bufs.push_back(grd[k]);
    }
  ops.clear();
  for (int i = (int)prog->ops.size() - 1; i >= 0; --i) {
    const SymOp& o = prog->ops[i];
    if (o.setup && !inline_setup_) continue;
    const std::string tag = "bwd:" + prog->t[o.out].name;
    const bool one = o.b < 0;
    if (need_grad[o.a])
      ops.push_back(OpInst{nt + o.a, nt + o.out, o.b, &grd[o.a], &grd[o.out], one ? nullptr : &fwd[o.b], o.ai, o.oi,
                           o.bi, o.alpha, true, -1, cidx(o.b), -1, vidx(o.b), o.a, o.out, o.b,
                           one ? tag : tag + ":dA"});
    if (!one && need_grad[o.b])
      ops.push_back(OpInst{nt + o.b, o.a, nt + o.out, &grd[o.b], &fwd[o.a], &grd[o.out], o.bi, o.ai, o.oi, o.alpha,
                           true, cidx(o.a), -1, vidx(o.a), -1, o.b, o.a, o.out, tag + ":dB"});
  }
  lower(bwd_, ops, zeroed, zero_bufs);
  // FTCC_FUSE=0 keeps the program order, one launch per contraction (diagnostics)
  const char* fz = std::getenv("FTCC_FUSE");
  if (!mom_.empty() && !(fz && fz[0] == '0')) {
    // The energy's dots and the gradients of the integrals are no part of a fixed-point
    // sweep (step of a spin ring of 12: 23.1 -> 21.7 ms without them, 6 dense orbitals
    // 14.1 -> 13.4, 33 dense orbitals, forward 108.7 -> 107.1).
    bool ranged = true;
    for (const Launch& l : fwd_) ranged = ranged && l.ranged;
    for (const Launch& l : bwd_) ranged = ranged && l.ranged;
    if (ranged) {
      Ranges out, in;
      for (int k = 0; k < nt; ++k) {
        const bool output = prog->t[k].kind == T_OUTPUT, input = prog->t[k].kind == T_INPUT;
        for (int p = 0; p < np; ++p) {
          const size_t sz = sizeof(double) * (size_t)ipow_l(probs[p].n, prog->t[k].rank);
          if (output && prog->t[k].rank > 0) add_range(out, fwd[k][p], sz);
          if (input && need_grad[k]) add_range(in, grd[k][p], sz);
        }
      }
      const std::vector<char> kf = leads_to(fwd_, out), kb = leads_to(bwd_, in);
      bool apart = true;
      for (size_t i = 0; i < fwd_.size(); ++i) {
        if (kf[i]) {
          fwd_sweep_.push_back(fwd_[i]);
          continue;
        }
        fwd_rest_.push_back(fwd_[i]);
        Ranges used = fwd_[i].rd;
        used.insert(used.end(), fwd_[i].wr.begin(), fwd_[i].wr.end());
        normalize(used);
        for (size_t j = i + 1; j < fwd_.size(); ++j) {
          if (!kf[j]) continue;
          Ranges wr = fwd_[j].wr;
          normalize(wr);
          apart = apart && !overlaps(wr, used);
        }
      }
      for (size_t i = 0; i < bwd_.size(); ++i)
        if (kb[i]) bwd_sweep_.push_back(bwd_[i]);
      if (!apart || fwd_rest_.empty() || bwd_sweep_.empty()) {
        fwd_sweep_.clear();
        fwd_rest_.clear();
        bwd_sweep_.clear();
      }
      for (std::vector<Launch>* l : {&fwd_sweep_, &fwd_rest_, &bwd_sweep_}) fuse_levels(*l);
    }
    fuse_levels(setup_);
    fuse_levels(fwd_);
    fuse_levels(bwd_);
  }
  end_uploads();
  dump_plan();
}

// Autotuner: every grouped GEMM launch with 128x128 tiles is timed on its own
// descriptors (the real operand pointers and shapes of the program) with each
// candidate tile configuration, and the fastest is kept.  Outputs written while
// timing are overwritten by the first real sweep (every tensor's first op
// overwrites it; gradient buffers are zero-filled before each backward).
void Executor::autotune(hipStream_t s) {
  const char* env = std::getenv("FTCC_AUTOTUNE");
  hipEvent_t e0, e1;
  FTCC_HIP(hipEventCreate(&e0));
  FTCC_HIP(hipEventCreate(&e1));
  // every candidate of a GEMM launch: its own descriptor set (tile size, split-K)
  // with each tile configuration of that size (BK 16 or 32 for 128 x 128 tiles),
  // timed over two launches after a warm-up (split-K reduce included)
  auto time_one = [&](const Launch& v, int cfg) {
    auto go = [&] {
      launch_gemm(cfg, v.ta, v.tb, (const GemmProblem*)v.d_desc, v.d_prefix, v.n_prob, v.total, tail_of(v, cfg), s);
      if (v.splitk_blocks > 0)
        launch_splitk_reduce((const GemmProblem*)v.d_desc, v.d_prefix2, v.n_prob, v.splitk_blocks, s);
    };
    go();
    FTCC_HIP(hipEventRecord(e0, s));
    for (int r = 0; r < 2; ++r) go();
    FTCC_HIP(hipEventRecord(e1, s));
    FTCC_HIP(hipEventSynchronize(e1));
    float ms = 0.f;
    FTCC_HIP(hipEventElapsedTime(&ms, e0, e1));
    return ms * 0.5f;
  };
  for (std::vector<Launch>* lst : {&fwd_, &bwd_}) {
    for (Launch& l : *lst) {
      if (l.kind != Launch::GEMM) continue;
      if (env && env[0] == '0') {
        l.alts.clear();
        continue;
      }
      int best_v = -1, best_cfg = l.cfg;
      float best_ms = 1e30f;
      for (int v = -1; v < (int)l.alts.size(); ++v) {
        const Launch& cand = v < 0 ? l : l.alts[v];
        const std::vector<int> cfgs = gemm_bm(cand.cfg) == 128 ? std::vector<int>{0, 2} : std::vector<int>{1};
        for (int cfg : cfgs) {
          const float ms = time_one(cand, cfg);
          if (ms < best_ms) {
            best_ms = ms;
            best_v = v;
            best_cfg = cfg;
          }
        }
      }
      if (best_v >= 0) {
        const Launch& w = l.alts[best_v];
        l.d_desc = w.d_desc;
        l.d_prefix = w.d_prefix;
        l.d_prefix2 = w.d_prefix2;
        l.total = w.total;
        l.splitk_blocks = w.splitk_blocks;
        l.prob_total = w.prob_total;
        l.prob_total2 = w.prob_total2;
        l.min_k = w.min_k;
      }
      l.cfg = best_cfg;
      l.tuned_ms = best_ms;
      l.alts.clear();
    }
  }
  FTCC_HIP(hipEventDestroy(e0));
  FTCC_HIP(hipEventDestroy(e1));
  dump_plan();
}

// FTCC_PLAN_DUMP=1 prints the lowered launch lists (diagnostics only)
void Executor::dump_plan() const {
  const char* env = std::getenv("FTCC_PLAN_DUMP");
  if (!env || env[0] != '1') return;
  const char* kinds[] = {"perm", "gemm", "dot", "fill", "sgemm", "elem", "dotb"};
  const std::pair<const char*, const std::vector<Launch>*> lists[] = {
      {"setup", &setup_},       {"forward", &fwd_},      {"backward", &bwd_},
      {"fwd-sweep", &fwd_sweep_}, {"fwd-rest", &fwd_rest_}, {"bwd-sweep", &bwd_sweep_}};
  for (const auto& pl : lists) {
    int counts[7] = {0, 0, 0, 0, 0, 0, 0};
    double fl = 0.0;
    for (const Launch& l : *pl.second) {
      counts[l.kind]++;
      fl += l.flops;
      std::fprintf(stderr, "[plan] %-8s %-4s cfg=%d ta=%d tb=%d blocks=%d split=%d gflop=%.3f ms=%.3f %s\n",
                   pl.first, kinds[l.kind], l.cfg, (int)l.ta, (int)l.tb, l.total, l.splitk_blocks > 0,
                   l.flops * 1e-9, l.tuned_ms, l.tag.c_str());
    }
    std::fprintf(stderr,
                 "[plan] %s: %d perm, %d gemm, %d dot, %d fill, %d blocked, %d blocked-elem, %d blocked-dot, "
                 "%.3f GFLOP\n",
                 pl.first, counts[0], counts[1], counts[2], counts[3], counts[4], counts[5], counts[6], fl * 1e-9);
  }
}

// ------------------------------------------------------------------ run
// algorithmic flops of a GEMM launch over the problems whose instance runs
double Executor::run_flops(const Launch& l) const {
  if (!gate_host_ || l.prob_flops.empty()) return l.flops;
  double f = 0.0;
  for (size_t p = 0; p < l.prob_flops.size(); ++p)
    if (gate_host_[l.prob_gate[p]]) f += l.prob_flops[p];
  return f;
}

void Executor::run(const std::vector<Launch>& L, hipStream_t s) const {
  for (const Launch& l : L) {
    switch (l.kind) {
      case Launch::PERM:
      case Launch::FILL:
        launch_permute((const PermProblem*)l.d_desc, l.d_prefix, l.n_prob, l.total, s);
        break;
      case Launch::GEMM: {
        const bool timed = prof_ && prof_->enabled && gemm_bm(l.cfg) == 128;
        if (timed) prof_->record_begin(s);
        launch_gemm(l.cfg, l.ta, l.tb, (const GemmProblem*)l.d_desc, l.d_prefix, l.n_prob, l.total, tail_of(l, l.cfg),
                    s);
        if (timed) prof_->record_end(s, run_flops(l));
      }
        if (l.splitk_blocks > 0)
          launch_splitk_reduce((const GemmProblem*)l.d_desc, l.d_prefix2, l.n_prob, l.splitk_blocks, s);
        break;
      case Launch::DOT:
        launch_dot((const DotProblem*)l.d_desc, l.n_prob, l.dot_blocks, l.d_partial, s);
        break;
      case Launch::SGEMM:
        launch_sgemm((const SgemmProblem*)l.d_desc, (const SgemmTask*)l.d_tasks, l.n_square, l.n_narrow, l.n_tasks,
                     l.wide, l.d_partial,
                     (const SgemmReduce*)l.d_red, l.n_red, s);
        break;
      case Launch::DOTB:
        launch_dotb((const DotbProblem*)l.d_desc, l.n_prob, (const ElemTask*)l.d_tasks, (const int*)l.d_bfirst,
                    l.n_tasks, l.n_elem,
                    l.d_partial, s);
        break;
      case Launch::ELEM:
        if (l.n_flat > 0)
          launch_elem_flat((const ElemProblem*)l.d_desc, (const ElemSource*)l.d_src, (const ElemBlock*)l.d_tasks,
                           l.n_flat, s);
        else
          launch_elem((const ElemProblem*)l.d_desc, (const ElemSource*)l.d_src, (const ElemTask*)l.d_tasks,
                    (const int*)l.d_bfirst, l.n_tasks, l.n_elem, l.elem_per, s);
        break;
    }
  }
}

bool Executor::run_forward_one(int prob, hipStream_t s) const {
  for (const Launch& l : fwd_)
    if (l.kind != Launch::PERM && l.kind != Launch::FILL && l.kind != Launch::GEMM && l.kind != Launch::DOT) return false;
  for (const Launch& l : fwd_) {
    switch (l.kind) {
      case Launch::PERM:
      case Launch::FILL:
        launch_permute((const PermProblem*)l.d_desc + prob, d_zero_, 1, l.prob_total[prob], s);
        break;
      case Launch::GEMM: {
        const GemmProblem* d = (const GemmProblem*)l.d_desc + prob;
        const int total = l.prob_total[prob];
        launch_gemm(l.cfg, l.ta, l.tb, d, d_zero_, 1, total,
                    plan_gemm_tail(l.cfg, total, l.min_k, l.splitk_blocks > 0, scratch_->tail_ws,
                                   scratch_->tail_ws_doubles),
                    s);
        if (l.splitk_blocks > 0) launch_splitk_reduce(d, d_zero_, 1, l.prob_total2[prob], s);
        break;
      }
      default:
        launch_dot((const DotProblem*)l.d_desc + prob, 1, l.dot_blocks, l.d_partial, s);
    }
  }
  return true;
}

// ------------------------------------------------------------------ profiler
void KernelProfiler::reset() {
  used = 0;
  pending_flops.clear();
  flops = seconds = 0.0;
  launches = 0;
}

void KernelProfiler::record_begin(hipStream_t s) {
  if (used + 2 > (int)ev.size()) {
    // pool full: wait for the stream and harvest before reusing events
    FTCC_HIP(hipStreamSynchronize(s));
    harvest();
    if (ev.size() < 8192) {
      const size_t old = ev.size();
      ev.resize(old ? old * 2 : 512);
      for (size_t k = old; k < ev.size(); ++k) FTCC_HIP(hipEventCreate(&ev[k]));
    }
  }
  FTCC_HIP(hipEventRecord(ev[used], s));
}

void KernelProfiler::record_end(hipStream_t s, double f) {
  FTCC_HIP(hipEventRecord(ev[used + 1], s));
  pending_flops.push_back(f);
  used += 2;
}

void KernelProfiler::harvest() {
  for (size_t k = 0; k < pending_flops.size(); ++k) {
    float ms = 0.f;
    FTCC_HIP(hipEventElapsedTime(&ms, ev[2 * k], ev[2 * k + 1]));
    seconds += ms * 1e-3;
    flops += pending_flops[k];
    ++launches;
  }
  pending_flops.clear();
  used = 0;
}

KernelProfiler::~KernelProfiler() {
  for (hipEvent_t e : ev) (void)hipEventDestroy(e);
}

long Executor::dispatches(const std::vector<Launch>& L) const {
  long k = 0;
  for (const Launch& l : L) {
    switch (l.kind) {
      case Launch::GEMM: {
        const GemmTail t = tail_of(l, l.cfg);
        k += (l.total > 0) + (t.splits > 1 && t.dp_tiles < l.total) + (l.splitk_blocks > 0);
        break;
      }
      case Launch::SGEMM: k += (l.n_square > 0) + (l.n_narrow > 0) + (l.n_tasks > l.n_square + l.n_narrow) + (l.n_tasks > 0 && l.n_red > 0); break;
      case Launch::DOT: k += 2; break;
      case Launch::DOTB: k += 1 + (l.n_elem > 0 && l.n_tasks > 0); break;
      case Launch::ELEM: k += (l.n_tasks > 0 && l.n_elem > 0); break;
      default: k += (l.total > 0); break;
    }
  }
  return k;
}

double Executor::bytes_forward() const {
  double b = 0.0;
  for (const Launch& l : fwd_) b += l.bytes;
  return b;
}

double Executor::gemm_flops_forward() const {
  double f = 0.0;
  for (const Launch& l : fwd_) f += l.flops;
  return f;
}

double Executor::gemm_flops_backward() const {
  double f = 0.0;
  for (const Launch& l : bwd_) f += l.flops;
  return f;
}

}  // namespace ftcc
