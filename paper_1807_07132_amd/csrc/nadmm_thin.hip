// Thin data: which rows the path takes, its launches, and the kernel (nadmm_thin.h) for rows of whole quads.
#include <algorithm>
#include <cstring>

#include "nadmm_thin.h"

namespace nadmm {
namespace {

// the pending update alone: end of a stand-alone CG solve
constexpr int kFinishThreads = 1024;
__global__ __launch_bounds__(kFinishThreads) void thin_cg_finish_kernel(const ThinArgs ta) {
  bool go;
  cg_from_partials<kFinishThreads>(ta, threadIdx.x < 64, &go, [] {});
  if (threadIdx.x == 0) cg_solve_results(ta.cg);
}

// the fields of a deferred CG update; false if they do not fit this path
bool set_pending(ThinArgs* ta, const CgPend& cg, const ReduceArgs* prev, int64_t d) {
  if (prev == nullptr || prev->partial == nullptr || prev->nparts < 1 || prev->nparts > kThinMaxPartials || prev->d != d) return false;
  if (cg.st == nullptr || cg.dlen != d || d > kThinMaxD) return false;
  ta->cg = cg;
  ta->prev = prev->partial;
  ta->nprev = prev->nparts;
  ta->scale = prev->scale;
  ta->lambda = prev->lambda;
  ta->rho = prev->rho;
  ta->rho_scale = prev->rho_scale;
  return true;
}

}  // namespace

hipError_t launch_thin_quads(const ThinArgs& ta, int grid, hipStream_t st) { return launch_thin_rows<kQuads>(ta, grid, st); }

bool thin_supported(const Shape& s, int64_t lda, const void* A) {
  if (s.p > 32 || (s.p & 3) != 0 || s.NC > 3 || s.p * s.NC > 64) return false;
  if (lda != s.p || (reinterpret_cast<uintptr_t>(A) & 15) != 0) return false;
  return true;
}

// Any other rows of up to 32 columns: at most 3 elements of padding, so that a chunk of 64 rows is one block of little more than
// 64 p floats; the accumulators of the padded row fit the registers.  The limits on the smallest matrices are those of an earlier form,
// which fetched 16 bytes at a time; the kernel does without them, but callers may go by the path numbers that follow from them.
bool thin_general_supported(const Shape& s, int64_t lda, const void* A) {
  const int64_t pp = (lda + 3) / 4 * 4;
  if (lda < s.p || lda > 32 || s.NC > 3 || pp * s.NC > 64 || s.p <= pp - 4) return false;
  return s.n * lda >= 8 && (s.n - 1) * lda + s.p >= 4 && (reinterpret_cast<uintptr_t>(A) & 3) == 0;
}

// Rows with padding that are 16-byte aligned, of more than one operand piece, on up to 65535 rows (393215 with 32 x 2 accumulators):
// the narrow-row kernel made them under path number 2 until this kernel came to stream chunks straight to LDS and to defer the CG update
// for all rows.  The number is part of what callers may rely on, the kernel is this one: nothing is faster on the other (505 shapes, 2049
// to 393215 rows; single sweeps of up to 65535 rows, which launches bound, equal to 0.3 of 11 us).  Narrow-row kernel against this one (us): lda = 32,
// C = 3: 5000 rows, 6 CG iterations 64.9 : 54.6; 200000 rows, gradient 24.6 : 15.3, 6 CG iterations 112 : 62.5; lda = 8, C = 4: 40000 rows, 2 Newton
// iterations of 5 CG iterations 161 : 117, a line search 20.3 : 17.7.  Both work to the same accuracy (Hessian-vector products within
// 4.0e-8 to 6.0e-8 of 64 bits there, 3.5e-8 to 5.8e-8 here).
bool thin_numbered_2(const Shape& s, int64_t lda) {
  return s.n > 2048 && lda * s.NC > 16 && s.n < (lda * s.NC < 64 ? 65536 : 393216);
}

// one workgroup per compute unit, and every wave with a chunk of 64 rows before any has two
int thin_num_partials(const Shape& s) { return (int)std::min<int64_t>(kThinMaxPartials, (s.n + 63) / 64); }

hipError_t launch_thin(const RowArgs& a, float* partial, int nparts, hipStream_t st, const CgPend* cg, const ReduceArgs* prev,
                       const NewtonHeadArgs* head, const SearchArgs* search) {
  if (nparts < 1 || nparts > kThinMaxPartials) return hipErrorInvalidValue;
  if (a.kind == kRowsSearch &&
      (a.labels == nullptr || search == nullptr || search->lpart == nullptr || search->ncand < 1 || search->ncand > kSweepCand))
    return hipErrorInvalidValue;
  ThinArgs ta;
  std::memset(&ta, 0, sizeof(ta));
  ta.r = a;
  ta.partial = partial;
  if (search != nullptr) ta.search = *search;
  if (cg != nullptr) {
    // the pending update of a CG iteration on cached probabilities (or the line search's logits pass on the final iterate)
    if (a.B0 != nullptr || !set_pending(&ta, *cg, prev, (int64_t)a.p * a.NC)) return hipErrorInvalidValue;
    if (prev->partial == partial) return hipErrorInvalidValue;  // the sweep reads the previous partials while it writes its own
  } else if (head != nullptr) {
    if (a.B0 != nullptr || prev == nullptr || prev->partial == nullptr || prev->partial == partial || prev->nparts < 1 ||
        prev->nparts > kThinMaxPartials || head->st == nullptr || head->newton_mode == 0 || head->d != (int64_t)a.p * a.NC ||
        head->d > kThinMaxD || head->loss_part == nullptr || head->g_out == nullptr || head->nblocks < 1 || head->nblocks > kThinMaxPartials)
      return hipErrorInvalidValue;
    ta.head = *head;
    ta.prev = prev->partial;
    ta.nprev = prev->nparts;
  }
  return (a.lda & 3) == 0 ? launch_thin_quads(ta, nparts, st) : launch_thin_block(ta, nparts, st);
}

hipError_t launch_thin_cg_finish(const CgPend& cg, const ReduceArgs& prev, hipStream_t st) {
  ThinArgs ta;
  std::memset(&ta, 0, sizeof(ta));
  if (cg.final_p == 0 || !set_pending(&ta, cg, &prev, cg.dlen)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(thin_cg_finish_kernel, dim3(1), dim3(kFinishThreads), 0, st, ta);
  return hipGetLastError();
}

}  // namespace nadmm
