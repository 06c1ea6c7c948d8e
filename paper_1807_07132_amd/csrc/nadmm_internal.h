// Internal declarations shared by the translation units of libnadmm (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>
#include <cmath>

#include "nadmm.h"

namespace nadmm {

// Raises a kernel's dynamic-LDS limit to the 160 KB of a gfx950 compute unit (less for kernels with LDS arrays of their own), once per device
// (the attribute belongs to the kernel's code object on the current device).
// done_mask: devices on which this has been done; host threads may race to it, the attribute is then set twice.
typedef std::atomic<uint64_t> LdsLimitMask;
inline hipError_t ensure_lds_limit(const void* kernel, LdsLimitMask* done_mask, int bytes = 160 * 1024) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = (uint64_t)1 << (dev & 63);
  if ((done_mask->load(std::memory_order_acquire) & bit) == 0) {
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
    done_mask->fetch_or(bit, std::memory_order_release);
  }
  return hipSuccess;
}

constexpr int kWave = 64;
constexpr int kMaxCand = NADMM_MAX_LS + 2;  // candidate step sizes 1, gamma, ..., gamma^(max_ls+1)
constexpr int kCandSlots = kMaxCand + 1;    // + one slot for alpha = 0 (objective at X itself)

// CG state after some number of updates, kept twice: a kernel that applies a pending update reads one copy and
// its workgroup 0 writes the other, so that no workgroup reads what another one of the same kernel writes.
struct CgSlot {
  double rr;        // ||r||^2 of the current residual
  int32_t active;   // 0 once CG has stopped (tolerance met, no positive curvature, or nothing to solve)
  int32_t iters;    // updates applied
  int32_t cur;      // which of the two sets of the vectors r, d, p is current
  int32_t pad_;
};

// Device-resident scalars of the Newton / CG / line-search drivers.  Lives at
// the start of the workspace; written only by single-workgroup tail kernels.
// Iterations of one CG solve whose directional logits A d_k the fused path may keep, so that the line search gets
// A p = sum_k alpha_k A d_k without another pass over A.
constexpr int kCgHist = 32;

struct DevState {
  double loss;      // Fhat at the current X
  double gg;        // ||g||^2 at the current X
  double rr;        // CG: ||r||^2 of the current residual
  double gg_cg;     // CG: ||g||^2 of the right-hand side
  double loss_new;  // line search: Fhat(X + alpha p)
  double loss_initial;
  float alpha;      // line search result
  int32_t newton_even;  // see newton_entered
  int32_t cg_active;
  int32_t cg_iters;
  int32_t armijo_ok;
  int32_t ls_evals;
  int32_t cg_go;    // two-kernel CG update: the first kernel's verdict (active and positive curvature)
  int32_t cg_ok;    //   0 if the first kernel met non-positive curvature
  float cg_alpha;   //   step length of this CG iteration
  int32_t newton_odd;
  int32_t pad_[2];  // one slot of cgs to a cache line: a kernel reads one while a workgroup of it writes the other
  double rr_prev;   //   ||r||^2 before this CG iteration
  CgSlot cgs[2];    // CG updates that several workgroups make (CgPend, cg_step_scalars)
  float cg_alphas[kCgHist];  // deferred CG update: step length of every iteration taken (p = sum_k alpha_k d_k)
  nadmm_stats stats;  // copied to the host at the end of nadmm_local_newton
};

static_assert(offsetof(DevState, cgs) / 128 == (offsetof(DevState, cgs) + sizeof(CgSlot) - 1) / 128 && (offsetof(DevState, cgs) + sizeof(CgSlot)) % 128 == 0,
              "the slots' lines");

// Iteration `iter` of Algorithm 3 is entered if its word is not 0.  Its head leaves in the other word whether the iteration goes on,
// and the next iteration is entered by that.  A kernel that makes the head beside other work goes by the first word in all its
// workgroups: none reads what another one of the same kernel writes.
inline __host__ __device__ int32_t* newton_entered(DevState* st, int32_t iter) { return (iter & 1) != 0 ? &st->newton_odd : &st->newton_even; }
inline __host__ __device__ int32_t* newton_goes_on(DevState* st, int32_t iter) { return newton_entered(st, iter + 1); }

// 16 bytes of a row of A that need only start on a 4-byte boundary: the load type of the matrix-core kernels' variants
// for rows that are not 16-byte aligned (any row stride, A 4-byte aligned).
struct __attribute__((packed, aligned(4))) Quad {
  float x, y, z, w;
};

// Row-pass (forward) work description, shared by the two-pass and the fused kernels.
//   kind 0  Hessian-vector rows:  D = P o W - P o rowsum(P o W)         (Section 2.6)
//   kind 1  gradient rows:        R = P - Y, row losses                  (Sections 2.1, 2.2)
//   kind 2  row losses only
//   kind 3  logits only:          Z0 = A B0 and / or Z1 = A B1
//   kind 4  line search:          row losses at Z0 + alpha Z1 for every step size of `alphas` (no logits are stored)
enum RowKind { kRowsHv = 0, kRowsGrad = 1, kRowsLoss = 2, kRowsLogits = 3, kRowsSearch = 4 };
constexpr int kSweepCand = 16;  // step sizes that a sweep of kind 4 evaluates at most: one per class lane of the rows stage

struct RowArgs {
  const float* A;
  int64_t n;
  int32_t p;
  int64_t lda;
  int32_t NC;          // C-1
  const float* B0;     // p x NC, operand of the logits Z = A B0 (X); NULL if P comes from Pin
  const float* B1;     // p x NC, operand of the directional logits W = A B1 (V or p); may be NULL
  const int32_t* labels;
  const float* Pin;    // n x NC, with B0 == NULL: cached probabilities (kind 0) or logits A X (kind 4)
  float* rows_out;     // n x NC: D (kind 0) or R (kind 1); may be NULL
  float* Pout;         // n x NC: probabilities, optional
  float* Z0out;        // n x NC: logits A B0, optional
  float* Z1out;        // n x NC: logits A B1, optional
  double* loss_part;   // per-workgroup partial sums of row losses (kinds 1, 2)
  int32_t kind;
  const int32_t* flag; // if non-NULL and *flag == 0 the kernel does nothing
};

// Kind 4 (not part of RowArgs: its size costs kernels without it registers, the wide-row ones two more spilled in their stream)
struct SearchArgs {
  double* lpart;       // [step size][workgroup] partial sums of row losses
  int32_t ncand;       // step sizes, at most kSweepCand
  float alphas[kSweepCand];
};

// A CG update (Section 2.4) that has not been applied yet, handed to the kernel that needs its result: the
// next Hessian-vector sweep needs the new direction d, the sweep after the last CG iteration the iterate p.
// Every workgroup of that kernel applies the update for itself from q = H d and the partial sums of <d, q>
// (identical arithmetic in every workgroup, so all of them agree bit for bit, also on whether CG stops);
// workgroup 0 writes the new vectors to the other set and the new state to the other CgSlot.
struct CgPend {
  DevState* st;          // NULL: no deferred update (operands come from RowArgs as usual)
  int32_t slot_in;       // st->cgs[slot_in] is read, st->cgs[slot_in ^ 1] written
  int32_t final_p;       // 0: the kernel wants d (Hessian-vector product), 1: it wants p (end of CG)
  float* r[2];
  float* d[2];
  float* p[2];
  const float* q;        // H d of the update
  const double* dot_part;
  int32_t ndot;
  float tol;
  float* p_final;        // final_p: workgroup 0 leaves the iterate here and copies the state to the scalars of DevState
  int64_t dlen;
  int32_t* iters_out;    // the kernels that end a stand-alone CG solve, optional: its results
  float* relres_out;
};

// Column-pass (transpose product) description: partial[k] = (rows of chunk k of A)^T rows_in
struct ColArgs {
  const float* A;
  int64_t n;
  int32_t p;
  int64_t lda;
  int32_t NC;
  const float* rows_in;  // n x NC
  float* partial;        // nparts x (p*NC)
  int32_t rows_per_chunk;
  const int32_t* flag;
};

struct Shape {
  int64_t n;
  int32_t p;
  int32_t NC;
  int64_t d;  // p * NC
};

// ---- launchers, generic two-pass path (nadmm_generic.hip) ----
int generic_row_blocks(int64_t n);
void generic_col_grid(const Shape& s, int* nslabs, int* nchunks, int* rows_per_chunk);
hipError_t launch_generic_rows(const RowArgs& a, hipStream_t st);
hipError_t launch_generic_cols(const ColArgs& a, int nslabs, int nchunks, hipStream_t st);
// rows stage on per-slice partial logits zw[slice][row][Z|W][C-1] (Z only if B0, W only if B1 is given);
// partial losses per block of generic_row_blocks()
// rows_ld: floats between the rows of a.rows_out
hipError_t launch_logit_rows(const RowArgs& a, const float* zw, int nslices, int rows_ld, hipStream_t st);

// ---- vector / tail kernels (nadmm_vec.hip) ----
struct NewtonHeadArgs {
  DevState* st;
  const double* loss_part;
  int32_t nblocks;
  float scale, lambda, rho;
  const float* X;
  const float* z;
  const float* y;
  const float* g;
  float* g_out;        // launch_thin with head: where the gradient is left (g is not read then)
  float* pdir;
  float* r;
  float* dvec;
  int64_t d;
  int32_t iter;        // Newton iteration index
  float grad_tol;
  int32_t newton_mode; // 1: part of Algorithm 3 (stats, grad_tol); 0: plain CG initialisation from g
  const double* pen_part;  // optional (with gg_part): partial sums left by the reduction that formed g, which
  const double* gg_part;   //   has then also written p = 0, r = d = -g
  int32_t npart;
  const float* rho_scale;  // optional device scalar factor on rho
};

// The scalars of an iteration's head, by one thread: objective, ||g||, the stopping test of Algorithm 3 and the state that CG starts from.
inline __host__ __device__ void newton_head_scalars(const NewtonHeadArgs& a, double gg, double loss) {
  DevState* st = a.st;
  st->gg = gg;
  st->rr = gg;
  st->gg_cg = gg;
  st->cg_iters = 0;
  st->cg_active = gg > 0.0 ? 1 : 0;
  int32_t cg_on = st->cg_active;
  if (a.newton_mode && (sqrt(gg) < (double)a.grad_tol || !(gg > 0.0))) cg_on = 0;
  st->cgs[0] = CgSlot{gg, cg_on, 0, 0, 0};
  if (a.newton_mode) {
    const double gn = sqrt(gg);
    st->loss = loss;
    nadmm_stats* s = &st->stats;
    if (a.iter == 0) { st->loss_initial = loss; s->loss_initial = loss; s->loss_final = loss; }
    s->grad_norm_final = gn;
    *newton_goes_on(st, a.iter) = cg_on;
    if (cg_on == 0) {
      st->cg_active = 0;
    } else if (a.iter < NADMM_TRACE_LEN) {
      s->loss[a.iter] = loss;
      s->grad_norm[a.iter] = gn;
    }
  }
}
// The head of an iteration that is not entered: CG stays inactive, the next iteration is not entered either.
inline __host__ __device__ void newton_head_skipped(const NewtonHeadArgs& a) {
  a.st->cgs[0] = CgSlot{0.0, 0, 0, 0, 0};
  *newton_goes_on(a.st, a.iter) = 0;
}

struct ReduceArgs {
  const float* partial;
  int32_t nparts;
  int64_t d;
  float scale;            // s
  int32_t kind;           // 0: out = s*sum + (lambda+rho) V ; 1: out = s*sum + lambda X + rho (X - z) + y
  const float* V;         // kind 0
  union {
    const float* X;       // kind 1
    // kind 0, with dot_part (d <= 2^18), optional: the residual r; behind them as many sums of r t, of t^2 and of r^2, t = out - (lambda + rho) r
    // (Behind the other arguments it cost the kernel a further line of them to wait for, and so did gridDim.x, which lies behind all of them.  7 CG
    // iterations at 30000 x 94, C = 18, with both: 144.8 us, without 139.9.)
    const float* r_dot;
  };
  const float* z;
  const float* y;
  float lambda, rho;
  const float* rho_scale; // optional device scalar: the penalty is rho * *rho_scale (adaptive penalty of the outer solver)
  float* out;
  const float* V_alt;     // kind 0, optional with cur: V is V_alt if *cur != 0 (the two vector sets of a deferred CG update)
  const int32_t* cur;
  double* dot_part;       // kind 0, optional: per-workgroup sums of out[e] * V[e], reduce_out_blocks(d) entries
  double* pen_part;       // kind 1, optional: per-workgroup sums of the penalty terms lambda/2 x^2 + rho/2 (x - z + y/rho)^2
  double* gg_part;        // kind 1, optional: per-workgroup sums of out[e]^2
  float* cg_p;            // kind 1, optional: CG start from the gradient just formed, p = 0, r = d = -out
  float* cg_r;
  float* cg_d;
  const int32_t* flag;
  // kind 1, optional (d <= kReduceFinishMax): one more workgroup finishes the objective beside the reduction,
  // *lf_loss_out = s * sum(lf_loss_part[0 .. lf_nblocks)) + penalty terms of X (from X, z, y themselves)
  const double* lf_loss_part;
  int32_t lf_nblocks;
  double* lf_loss_out;
  // kind 0, optional (d <= kReduceFinishMax): that workgroup does the work of newton_head_kernel instead (the first
  // Hessian-vector product of a CG solve needs nothing of it: its direction is the -g that the gradient's reduction left)
  int32_t has_head;
  NewtonHeadArgs head;
};
constexpr int64_t kReduceFinishMax = 16384;
int reduce_out_blocks(int64_t d);
hipError_t launch_reduce_out(const ReduceArgs& a, hipStream_t st);

struct LossFinishArgs {
  const double* loss_part;
  int32_t nblocks;
  float scale, lambda, rho;
  const float* X;
  const float* z;
  const float* y;
  int64_t d;
  const double* pen_part;  // optional: penalty terms already summed per workgroup by the reduction (npart entries)
  int32_t npart;
  double* loss_out;  // device scalar
  const float* rho_scale;  // optional device scalar factor on rho
};
hipError_t launch_loss_finish(const LossFinishArgs& a, hipStream_t st);

hipError_t launch_newton_head(const NewtonHeadArgs& a, hipStream_t st);
// the same as the start of a stand-alone CG solve (newton_mode 0, no partial sums); part: cg_start_blocks(d) doubles
hipError_t launch_cg_start(const NewtonHeadArgs& a, double* part, hipStream_t st);

struct CgUpdateArgs {
  DevState* st;
  float* pdir;
  float* r;
  float* dvec;
  const float* q;
  const double* dot_part;  // partial sums left by the reduction that formed q: of <d, q>, and behind them for the step those of ReduceArgs.r_dot
  int32_t ndot;            // of each
  double* rr_part;         // two-kernel form: cg_start_blocks(d) partial sums of the new ||r||^2
  int64_t d;
  float tol;
  // the step over several workgroups (cg_one_step): st->cgs[slot_in] is read and the other one written, likewise r and r_out
  int32_t slot_in;
  float* r_out;
  float lambda, rho;       // of H's linear term
  const float* rho_scale;
  float* pack;             // optional: the new direction also as rows of pack_ld floats for each NC elements, as the product with a sparse A reads it
  int32_t pack_ld, NC;
};
bool cg_one_step(int64_t d);
// lambda + rho_scale rho: the same bits wherever the step's sums are formed and used
__host__ __device__ inline float linear_factor(float lambda, float rho, const float* rho_scale) {
  return rho_scale != nullptr ? fmaf(rho, *rho_scale, lambda) : lambda + rho;
}
// the update with as many workgroups as the vectors take, in one launch (cg_one_step) or in two
hipError_t launch_cg_update(const CgUpdateArgs& a, hipStream_t st);
int cg_start_blocks(int64_t d);
// Small problems (d <= 1024 and at most 64 partial sums per thread): the reduction of the partial sums
// of A^T D, the linear term and the whole CG update in one single-workgroup kernel.
bool cg_fused_tail_supported(int64_t d, int nparts);
hipError_t launch_cg_reduce_update(const ReduceArgs& r, const CgUpdateArgs& a, hipStream_t st);

struct CgFinishArgs {
  const DevState* st;
  const float* pdir;
  float* p_out;
  int64_t d;
  int32_t* iters_out;
  float* relres_out;
};
hipError_t launch_cg_finish(const CgFinishArgs& a, hipStream_t st);

struct LsEvalArgs {
  const float* Zx;
  const float* Zp;         // A p; or NULL: A p = sum_{k < st->cg_iters} st->cg_alphas[k] * hist[k * hist_stride + .]
  const float* hist;       // the directional logits A d_k that the CG sweeps left, n x NC each
  int64_t hist_stride;     // elements between two of them
  int32_t nbuf;            // buffers there are (<= kCgHist): the most iterations a solve takes
  int32_t has_pend;        // the last CG update is still pending (pend): workgroup 0 applies it, the others take its
                           // step length from the same scalars; launched with one workgroup more
  CgPend pend;
  const DevState* st;
  const int32_t* labels;
  int64_t n;
  int32_t NC;
  int32_t ncand;           // number of step sizes in alphas[] that are evaluated
  float alphas[kCandSlots];
  double* lpart;           // [candidate slot][workgroup], ls_eval_blocks(n) workgroups
  const int32_t* flag;
};
int ls_eval_blocks(int64_t n);
bool ls_eval_takes_pending(int64_t n);
hipError_t launch_ls_eval(const LsEvalArgs& a, hipStream_t st);

struct LsTailArgs {
  DevState* st;
  const double* lpart;
  int32_t nblocks;
  int32_t ncand;          // candidates of Algorithm 2 (max_ls + 2)
  int32_t zero_slot;      // index in alphas[] of alpha = 0, or -1 if loss_at_X is given
  float alphas[kCandSlots];
  double loss_at_X;       // used if zero_slot < 0 and !use_state_loss
  int32_t use_state_loss; // take Fhat(X) from st->loss
  float scale, lambda, rho, beta;
  const float* X;
  const float* z;
  const float* y;
  const float* pdir;
  const float* g;
  int64_t d;
  float* X_apply;         // if non-NULL: X_apply += alpha * pdir (Newton update)
  float* alpha_out;       // optional device outputs of the stand-alone call
  double* loss_new_out;
  int32_t* ok_out;
  int32_t iter;           // Newton iteration index or -1
  const int32_t* flag;
  const float* rho_scale; // optional device scalar factor on rho
  double* qpart;          // scratch of 2 reduce_out_blocks(d) doubles (long vectors: the sums over d are formed by
                          // several workgroups and pass through it); NULL = single-workgroup form at any length
};
hipError_t launch_ls_tail(const LsTailArgs& a, hipStream_t st);

// outer_flag, if non-NULL, is copied into the words of newton_entered: a stopped outer iteration turns the local solve into no-ops
hipError_t launch_state_init(DevState* st, const int32_t* outer_flag, hipStream_t stream);

// ---- ADMM outer solver (nadmm_admm.hip) ----
struct AdmmState {
  int32_t active;     // 0 once the residual test has stopped the iteration
  float rho_scale;    // common factor on every worker's penalty (residual balancing); written by the finishing
                      // kernel of a consensus step, read by the kernels launched after it
  nadmm_admm_stats stats;
};
struct AdmmConsensusArgs {
  AdmmState* st;           // may be NULL (stand-alone consensus step)
  const float* x;          // N x d
  float* u;                // N x d
  float* z;                // d
  int32_t N;
  int64_t d;
  float rho[NADMM_MAX_WORKERS];
  float lambda, eps_abs, eps_rel;
  int32_t penalty_rule;    // 0 fixed, 1 residual balancing
  float rb_mu, rb_tau;
  double* part;            // admm_blocks(d) x 5 partial sums
  double* out;             // optional: r_norm, d_norm, eps_pri, eps_dual
  int32_t iter;
};
int admm_blocks(int64_t d);
hipError_t launch_admm_init(AdmmState* st, float* u, float* z, int32_t N, int64_t d, hipStream_t stream);
hipError_t launch_admm_consensus(const AdmmConsensusArgs& a, hipStream_t stream);

// ---- fused single-pass path (nadmm_fused.hip) ----
bool fused_supported(const Shape& s, int64_t lda, const void* A);
int fused_num_partials(const Shape& s);
// Runs the rows pass and (if partial != NULL) the transpose product in one sweep
// over A; leaves per-workgroup partial sums of A^T rows in `partial`
// (nparts = fused_num_partials() blocks of d floats) and per-workgroup partial
// losses in a.loss_part[0 .. nparts).
hipError_t launch_fused(const RowArgs& a, float* partial, int nparts, hipStream_t st, const CgPend* cg = nullptr,
                        const SearchArgs* search = nullptr);
// the pending update alone (one workgroup): end of a stand-alone CG solve
hipError_t launch_cg_pending_finish(const CgPend& c, hipStream_t st);

// ---- thin-data single-pass path (nadmm_thin.h, nadmm_thin.hip): p <= 32, C-1 <= 3, at most 3 elements between rows ----
bool thin_supported(const Shape& s, int64_t lda, const void* A);          // p % 4 == 0, lda == p, 16-byte aligned
bool thin_general_supported(const Shape& s, int64_t lda, const void* A);  // other rows of up to 32 columns
bool thin_numbered_2(const Shape& s, int64_t lda);  // of those, 16-byte aligned: whether callers know them by path number 2
int thin_num_partials(const Shape& s);
// cg, prev (both or neither): the sweep first applies the pending CG update, forming q = H d from the previous sweep's
// partial sums prev->partial (prev also carries scale, lambda, rho of the linear terms); see ThinArgs in nadmm_thin.h
hipError_t launch_thin(const RowArgs& a, float* partial, int nparts, hipStream_t st, const CgPend* cg = nullptr,
                       const ReduceArgs* prev = nullptr, const NewtonHeadArgs* head = nullptr, const SearchArgs* search = nullptr);
// the pending update alone (one workgroup): end of a stand-alone CG solve
hipError_t launch_thin_cg_finish(const CgPend& cg, const ReduceArgs& prev, hipStream_t st);

// ---- a whole CG or Newton solve of a small thin problem in one launch (nadmm_small.hip) ----
struct SmallSolve {
  const float* A;
  int64_t n, lda;
  int32_t p, NC;
  int32_t quads;           // set by the launcher: rows are whole aligned quads
  const float* X;
  const float* z;          // as in nadmm_problem; not read by a CG solve
  const float* y;
  const int32_t* labels;   // Newton solve
  float scale, lambda, rho;
  const float* rho_scale;  // optional device scalar factor on rho
  int32_t max_cg;
  float cg_tol;
  // CG solve: from g to p_out, iters_out and relres_out (optional)
  const float* g;
  float* p_out;
  int32_t* iters_out;
  float* relres_out;
  // Newton solve (Algorithm 3): X_out may be X; scalars and statistics go to st
  int32_t newton;
  int32_t max_newton;
  float grad_tol, beta;
  int32_t ncand;           // candidates of the line search
  float alphas[kCandSlots];
  float* X_out;
  DevState* st;
  const int32_t* outer_flag;  // as for launch_state_init
};
bool small_solve_supported(const Shape& s, int32_t max_cg);
hipError_t launch_small_solve(const SmallSolve& c, hipStream_t st);

// ---- column-sliced two-sweep matrix-core path (nadmm_sliced.hip): any p, C-1 <= 32, lda % 4 == 0 ----
bool sliced_supported(const Shape& s, int64_t lda, const void* A);
void sliced_grid(const Shape& s, int* nslices, int* steps_per_slice, int* row_groups);
// sweep 1 and the rows stage in one kernel (the logits never leave the compute unit); partial row losses: one per
// workgroup, sliced_loss_blocks() of them
int sliced_loss_blocks(const Shape& s);
hipError_t launch_sliced_logits(const RowArgs& a, hipStream_t st);
hipError_t launch_sliced_cols(const RowArgs& a, const float* rows_in, float* partial, hipStream_t st);

// ---- matrix-core kernel for narrow rows (nadmm_narrow.hip), on the paths of the fused (C-1 <= 16) and the column-sliced kernels ----
bool narrow_supported(const Shape& s, int64_t lda, const void* A);
bool narrow_takes(const Shape& s, bool has_x, bool has_v);  // whether it makes the sweep with these operands
int64_t narrow_min_rows(int32_t p);                         // C-1 <= 16: fewer rows are faster on the fused kernel, where that takes them
int narrow_num_partials(const Shape& s);
hipError_t launch_narrow(const RowArgs& a, float* partial, int nparts, hipStream_t st, const CgPend* cg);  // as launch_fused

// ---- single-pass matrix-core kernel for wide rows (nadmm_wide.hip): the sweeps of that path that form A^T rows ----
bool wide_supported(const Shape& s, int64_t lda, const void* A);
bool wide_takes(const Shape& s, bool has_x, bool has_v);  // whether it makes the sweep with these operands (else two sweeps)
int wide_num_partials(const Shape& s, int wg_cap);   // workgroups, at most wg_cap if that is > 0
size_t wide_operand_bytes(const Shape& s);
// packs the operands into `operands` and makes the sweep; partial sums and partial losses as launch_fused
// packed: the operands of this call are in place (launch_wide_direction)
hipError_t launch_wide(const RowArgs& a, void* operands, bool packed, float* partial, int nparts, hipStream_t st);
// launch_cg_update that leaves the new direction as the operands of the next product as well (cg_one_step only)
hipError_t launch_wide_direction(const CgUpdateArgs& a, const Shape& s, void* operands, hipStream_t st);

// ---- sparse storage of A (nadmm_sparse.hip) ----
// compressed rows of an nrows x ncols matrix; used for A (row view) and for A^T (column view of A)
struct SparseView {
  const int64_t* ptr;  // nrows + 1
  const int32_t* idx;  // nnz, in 0..ncols-1
  const float* val;    // nnz
  int64_t nrows;
  int32_t ncols;
  int64_t nnz;
};
// Rows of a view in windows of equal cost: the first row of each, n + 1 entries, 1 << shift cost units
struct SparseWindows {
  int32_t* first;
  int32_t n, shift;
};
// out = S B for a packed dense operand B: ncols rows of nops blocks of 4 sparse_group(NC) floats (what lies beyond the first NC of a block does not
// matter); row r of the product goes to out[(r * nops + op) * NC + c], op < nops, c < NC
struct SpmmArgs {
  SparseView S;
  const float* B;
  float* out;
  int32_t NC, nq, nops;  // nq = ceil(NC / 4) quads of a block hold data
  SparseWindows w;
  const int32_t* flag;
  // rows longer than a window are shared by the windows they reach over: sums of the shares, 2 x nwin x nops NC floats, and how many of a row
  // are there, nwin words that are 0 between launches (launch_sparse_plan); NULL: the workgroup in whose window such a row starts takes all of it
  float* share;
  int32_t* arrived;
};
int sparse_group(int NC);
int sparse_window_shift(int64_t nrows, int64_t nnz);
int sparse_windows(int64_t nrows, int64_t nnz);
// the windows of both views, and `arrived` zero for the larger number of them
hipError_t launch_sparse_plan(const SparseView& S0, const SparseWindows& w0, const SparseView& S1, const SparseWindows& w1, int32_t* arrived, hipStream_t st);
// dst[r] = [src0[r] | src1[r]] with every block padded to 4 sparse_group(NC) floats; src1 may be NULL
hipError_t launch_sparse_pack(const float* src0, const float* src1, int64_t rows, int NC, float* dst,
                              const int32_t* flag, hipStream_t st);
hipError_t launch_spmm(const SpmmArgs& a, hipStream_t st);

}  // namespace nadmm
