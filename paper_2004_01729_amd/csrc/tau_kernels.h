// Imaginary-time kernels: thermal integral blocks and the panel propagator.
#pragma once
#include <hip/hip_runtime.h>

namespace ftcc {

constexpr int kMaxNodes = 6;

// Panel quadrature shared by all instances: m Gauss-Legendre nodes c_x on [0,1],
// weights b_x, and the monomial coefficients of the Lagrange basis,
// l_y(u) = sum_k lc[y][k] u^k.
struct PanelRule {
  int m;
  int lawson;               // 0: exponential collocation, 1: integrating factor
  double c[kMaxNodes];
  double b[kMaxNodes];
  double lc[kMaxNodes][kMaxNodes];
  double A[kMaxNodes][kMaxNodes];   // int_0^{c_x} l_y(u) du (Lawson)
  // gc[x][y][k] = lc[y][k] c_x^(k+1) k!  (x = m: the panel end, c = 1), so that
  // W_xy = h sum_k gc[x][y][k] phi_{k+1}(-D h c_x)
  double gc[kMaxNodes + 1][kMaxNodes][kMaxNodes];
};

enum TauMode {
  TAU_INIT = 0,     // s_x = E_x s_b
  TAU_STEP = 1,     // s_x = E_x s_b - sum_y W_xy S_y   (+ max|change|, max|s|)
  TAU_END = 2,      // out = E_e s_b - sum_y We_y S_y
  TAU_LAMT = 3,     // s_x (lambda tilde) = sum_y W_yx S_y (lambda) + We_x s_b (a)
  TAU_APREV = 4,    // out = E_e s_b (a) + sum_x E_x S_x (lambda)
  TAU_BETA = 5,     // partial += sum_x <S_x(lam), -dE_x sb + sum_y dW_xy R_y> + <a, -dEe sb + sum dWe_y R_y>
  TAU_LSTEP = 6,    // s_x (lambda) = -R_x (gradient), with max|change|, max|lambda|
  TAU_DEPS = 7,     // out[e] += sum_x S_x(lam) (-dE_x sb + sum_y dW_xy R_y) + a (-dEe sb + sum dWe_y R_y),
                    // d/dDelta at fixed h (the orbital-energy response through the propagator)
  TAU_LSWEEP = 8,   // TAU_LSTEP, then lamt_x = TAU_LAMT's sum of the new lambda
};

// One amplitude segment of one instance (t1: n^2 elements, t2: n^4 elements).
struct TauProblem {
  const double* eps;
  int n;
  int rank;           // 2 or 4
  long len;
  double h;           // panel width beta / P
  const double* sb;   // panel-start state s_b (or adjoint a_{p+1})
  const double* S[kMaxNodes];   // residuals (or lambda)
  const double* R[kMaxNodes];   // residuals for TAU_BETA / gradients for TAU_LSTEP
  double* s[kMaxNodes];         // node amplitudes (or lambda-tilde / lambda)
  double* lamt[kMaxNodes];      // lambda-tilde for TAU_LSWEEP
  double* out;                  // end state / previous adjoint state / TAU_DEPS accumulator
  const double* lam_a;          // a_{p+1} for TAU_BETA and TAU_DEPS
  unsigned long long* maxbits;  // [0] max |change|, [1] max |value| (bit patterns of doubles >= 0)
  const int* active;            // STEP / LSTEP: instance still iterating (nullptr: always)
  double* partial;              // TAU_BETA: one partial sum per block
  const unsigned* idx;          // optional: the elements to visit (momentum-allowed ones), len of them;
                                // nullptr: every element 0..len-1
  unsigned pack;                // 0, or n: element e lies at e / n of the segments (the last index,
                                // fixed by the others, is not stored)
};

// elements per block of a launch (per problem); d_rule is a device copy of the rule
inline long tau_block_elements(int mode) { return mode == TAU_BETA ? 1024 : 256; }
void launch_tau(const PanelRule* d_rule, int m, int mode, const TauProblem* d_probs, const int* d_prefix, int n_prob,
                int total_blocks, hipStream_t s);

// Explicit Runge-Kutta march of the differential form (Algorithm alg:diff,
// eqn:smud: ds/dtau = -(Delta s + S[s])) and its reverse: one combination per
// amplitude segment,
//   out = x0 * base + sum_l coef[l] * (-Delta * Y_l + sigma * S_l)
// with Delta the segment's orbital-energy difference.  sigma = -1 makes the
// terms the slopes k_l = -(Delta Y_l + S_l) (stage states, step end);
// sigma = +1 the reverse-mode terms -Delta kbar_l + g_l (g the residual VJP).
// Null base / Y_l / S_l read as zero.  maxbits (optional) receives max |out|.
constexpr int kMaxStages = 4;
struct RKProblem {
  const double* eps;
  int n;
  int rank;                      // 2 or 4
  long len;                      // elements to visit
  const unsigned* idx;           // optional allowed-element list (len entries)
  const double* base;
  double x0;
  int nst;
  double coef[kMaxStages];
  const double* Y[kMaxStages];
  const double* S[kMaxStages];
  double sigma;
  unsigned pack;                 // as in TauProblem
  const double* h_x0;            // optional device factor of x0, of every coef
  const double* h_coef;
  double* out;
  unsigned long long* maxbits;
  const int* active;             // instance runs (nullptr: always)
};
constexpr int kRKBlock = 256;   // elements per block
// blocks: kRKBlock elements each, per problem
void launch_rk_combine(const RKProblem* d_probs, const int* d_prefix, int n_prob, int total_blocks, hipStream_t s);

// Implicit integral form generated by Simpson's rule (Section III): sums of
// exponentially weighted grid tensors, per element with Delta from eps,
//   out = x0 * base + (prod ? prod : 1) * sum_l t_l,
//   t_l = h C_l exp(-Delta h k_l) X_l                    (mode 0: the quadrature G e^{-Delta (tau_y - tau_x)})
//   t_l = C_l exp(-Delta h k_l) (1 - Delta h k_l) X_l     (mode 1: its h-derivative)
//   t_l = -h^2 C_l k_l exp(-Delta h k_l) X_l              (mode 2: its Delta-derivative)
// The terms live in device memory (terms[0..nterms)).  With maxbits, max |out|
// goes to maxbits[1] and max |out - out_before| to maxbits[0] (the fixed-point
// change of an amplitude or Lambda update).
struct ExpTerm {
  const double* X;
  double C;
  double k;
};
struct ExpSumProblem {
  unsigned pack;         // as in TauProblem
  const double* eps;
  int n;
  int rank;                      // 2 or 4
  long len;                      // elements to visit
  const unsigned* idx;           // optional allowed-element list (len entries)
  double h;
  int mode;
  const double* base;
  double x0;
  const double* prod;
  const ExpTerm* terms;
  int nterms;
  double* out;
  unsigned long long* maxbits;
  const int* active;             // instance runs (nullptr: always)
};
// blocks: 1024 elements each, per problem
void launch_expsum(const ExpSumProblem* d_probs, const int* d_prefix, int n_prob, int total_blocks, hipStream_t s);

// dst[o] = src[o] for the element offsets o of a node state listed in a (the t1
// block, na entries) and, shifted by `second`, in b (the t2 block, nb entries):
// the copy of a node state whose other elements are zero in both buffers.
void launch_copy_listed(const unsigned* a, long na, const unsigned* b, long nb, long second, const double* src,
                        double* dst, hipStream_t s);

// Many node states at once: dst = src (null: zero), over the listed elements when a is
// set (as above), else over len contiguous doubles.
struct StateCopy {
  const double* src;
  double* dst;
  long len;
  const unsigned* a;
  const unsigned* b;
  long na, nb, second;
  const int* active;   // optional run flag (0: skip)
  int add;             // dst += src
};
constexpr long kStateCopyBlock = 1024;   // elements per block
void launch_state_copies(const StateCopy* d_copies, const int* d_prefix, int n, int blocks, hipStream_t s);

void launch_repack(const unsigned* list, long count, int n, double* dense, double* packed, bool to_packed,
                   hipStream_t s);

// One instance's thermal set-up: occupations and weights from (mu, beta), the Fock
// operator f_pq = h_pq + sum_r (g <pr|qr> - <pr|rq>) n_r (g = 2: spin-restricted
// spatial orbitals, 1: spin orbitals), u = f - diag(eps), the 4 one-body and 12
// two-body weighted blocks (out = product of the slots' weights times the integral)
// and the mean-field sums; and the same quantities' derivatives.  Every launch takes
// a range of instances, blockIdx.y (or the block prefix) selecting one.
struct SetupProblem {
  int n;
  const double* eps;
  const double* h;      // n x n
  const double* eri;    // n^4, <pq|rs>
  double* occ;          // n_p
  double* wo;           // sqrt(n_p) or 0 when dropped
  double* wv;           // sqrt(1 - n_p) or 0 when dropped
  double* fock;         // n x n
  double* u_raw;        // f - diag(eps)
  double *dn, *dwo, *dwv, *du_raw;   // derivatives
  double* u[4];         // weighted blocks: oo, ov, vo, vv
  double* g[12];        // in the order of kBlockHoles
  double* du[4];        // their derivatives
  double* dg[12];
  const unsigned* idx;  // optional list of the two-body elements to compute (the others stay zero)
  long count;
  double* mf;           // mean-field sums
};
// hole slots (bit k: slot k) of the 12 two-body blocks: oooo ooov oovo oovv ovov ovvo ovvv vovv vvvv vvvo ovoo vvoo
constexpr int kBlockHoles[12] = {15, 7, 11, 3, 5, 9, 1, 2, 0, 8, 13, 12};
constexpr int kBlockHoles1[4] = {3, 1, 2, 0};
// elements one instance's block launch visits, and its blocks of 256
inline long setup_elements(const SetupProblem& p) {
  const long n2 = (long)p.n * p.n;
  return (p.idx ? p.count : n2 * n2) + n2;
}
enum SetupDeriv { SETUP_MU = 0, SETUP_BETA = 1, SETUP_DIR = 2, SETUP_EPS = 3 };

// occupations, Fock operator, blocks and mean-field sums of n_prob instances; mubeta[2 i]
// = mu, [2 i + 1] = beta; prefix: first block of each instance, `blocks` in all
void launch_thermal(const SetupProblem* d_probs, const double* d_mubeta, const int* d_prefix, int n_prob, int n_max,
                    int blocks, double thr, double g, hipStream_t s);
// derivative blocks: along mu, beta, a direction (dirs[2 i] = dh, [2 i + 1] = d<pq|rs>, either may be
// null) or the orbital energy q (occupations and the explicit u; instances with n <= q are left alone)
void launch_setup_deriv(const SetupProblem* d_probs, const double* d_mubeta, const double* const* d_dirs,
                        const int* d_prefix, int n_prob, int n_max, int blocks, int which, int q, double g,
                        hipStream_t s);

// DIIS: coefficients for every instance from its Gram matrix (ld x ld, count entries
// valid), then the extrapolated iterate sum_j c_j (X_j + R_j) of one buffer.
constexpr int kMaxDiis = 8;
struct DiisTerms {
  int k;
  const double* coef;
  const double* X[kMaxDiis];
  const double* R[kMaxDiis];
};
void launch_diis_solve(int n_inst, const int* counts, const int* newest, const double* G, int ld, double* coef,
                       hipStream_t s);
void launch_diis_combine(long len, const DiisTerms& t, double* out, hipStream_t s);

// acc[i][slot] += scale * (sum of instance i's partials [off[i], off[i + 1])), one block per instance
void launch_partial_sums(int n_inst, const double* partial, const int* off, double scale, double* const* acc, int slot,
                         hipStream_t s);
// sum of `count` doubles into *out (single block, deterministic)
void launch_sum(const double* x, int count, double* out, hipStream_t s);
// element-wise: y = a * x + b * y over len doubles
void launch_axpby(long len, double a, const double* x, double b, double* y, hipStream_t s);

}  // namespace ftcc
