// Single-pass kernel for thin data (p <= 32 features, few classes), gfx950.  Compiled for the two layouts of rows in two units
// (nadmm_thin.hip, nadmm_thin_block.hip).
//
// With rows of 4..128 bytes the pass is a pure HBM stream (about 1.5 flop per byte for C = 2), so there is no contraction worth a
// matrix core: one lane owns one sample.  A wave copies chunks of 64 rows -- one block of memory -- straight into its own part of
// LDS (global_load_lds), takes its rows from there into registers and has the next chunk on its way before it computes: logits
// Z = a_i X and W = a_i V with X and V as wave-uniform operands, the probabilities with the log-sum-exp shift (Section 2.2), the row
// of D (Section 2.6) or of P - Y, and a_i^T D into its private p x (C-1) registers.  What is in flight is LDS, not registers
// (16 waves per compute unit with up to 8 KB each), and no barrier is in the loop.  Per-lane accumulators are summed over the
// workgroup once, at the end, in a fixed order.
// In a CG solve the sweep of iteration k also does what lies between two sweeps (Section 2.4): it adds up the partial sums of
// sweep k - 1, forms q = H d and applies the CG update before it reads its operand (kHvCg, kLogitsCg, kSearchCg).
// The first sweep of a Newton iteration's CG solve makes the gradient's reduction and the head of the iteration the same way (kHvHead):
// two Newton iterations of 6 CG iterations at 100000 x 28, C = 2: 149 -> 137 us.
// A line search evaluates its step sizes in the pass that forms A p (kSearch, kSearchCg): a lane has its row's logits in registers, and
// the exponentials run beside the stream.  Against logits to memory and a row kernel on them: line search at 1400000 x 28, C = 2:
// 56.4 -> 42.8 us, 10 x 10 iterations at 1375000 x 28: 3703 -> 3516 us; 2500 rows equal.
//
// What bounds it: HBM.  Against chunks of 256 rows through registers of a whole workgroup (up to 204 of them, and surplus pieces
// past every chunk where rows are no dense quads): objective and gradient at 1375000 x 29, C = 2: 53.5 -> 35.8 us (the floor of one
// read of A is 28 us); Hessian-vector product at 600000 x 30, C = 3: 45.9 -> 20.7 us;
// 10 Newton iterations of 10 CG iterations at 1375000 x 28, C = 2: 4108 -> 3701 us; 6 CG iterations at 600000 x 32, C = 2: 184 -> 110 us.
#pragma once

#include "nadmm_internal.h"
#include "nadmm_cgstep.h"
#include "nadmm_mfma.h"

namespace nadmm {

struct ThinArgs {
  RowArgs r;
  float* partial;      // gridDim.x x (p*NC) or NULL
  SearchArgs search;   // kSearch, kSearchCg
  // Deferred CG update (kHvCg, kLogitsCg): the sweep of the previous CG iteration left only its per-workgroup
  // partial sums of A^T D.  Every workgroup of this sweep adds them up (fixed order), forms q = H d, applies the update of
  // Section 2.4 and takes its operand, the new direction (or, for the line search's pass, the final iterate), from there;
  // workgroup 0 stores the new vectors and state.  No reduction kernel and no CG kernel run between two sweeps.
  CgPend cg;           // cg.q and cg.dot_part are not used: this kernel forms both itself
  // kHvHead: the first sweep of a CG solve inside a Newton iteration.  The gradient's sweep left its partial sums only; every workgroup
  // forms g from them, workgroup 0 stores g and what newton_head_kernel leaves, and the operand is the first direction -g.
  NewtonHeadArgs head;
  const float* prev;   // the previous sweep's partial sums, nprev x (p*NC)
  int32_t nprev;
  float scale, lambda, rho;
  const float* rho_scale;
};

constexpr int kThinMaxPartials = 256;  // one workgroup per compute unit
constexpr int kThinMaxD = 64;          // p (C-1), with padded columns: the vectors fit one wave

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// How the rows lie, with lda <= 4 NQ:
//   kQuads: lda = 4 NQ, rows of whole quads (p = lda, or up to three elements between rows).  The lanes read quads, which lie
//     turned within their rows so that the reads spread over the banks.
//   kBlock: lda is no multiple of 4.  A block of rows lies in LDS as it does in memory, and the lanes read their rows back in
//     4-byte pieces: no bank conflicts where lda is odd, two lanes to a bank where it is even.
enum Rows { kBlock, kQuads };

// Everything a lane does with its row of A once it is in registers: logits, probabilities with the log-sum-exp shift, its row of D
// or of P - Y, the optional outputs, and its share of A^T rows.  P: the cached probabilities on entry (has0 false).
// x(j, c), v(j, c): the operands' entries, uniform in a wave.
template <int PP, int NC, typename OpX, typename OpV>
__device__ __forceinline__ void thin_row(const RowArgs& a, bool has0, bool has1, bool with_cols, bool valid, int64_t row,
                                         const float (&av)[PP], OpX&& x, OpV&& v, float (&P)[NC], int label,
                                         float (&acc)[PP][NC], double& loss_acc) {
  float z[NC], w[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) { z[c] = 0.f; w[c] = 0.f; }
  if (has0) {
#pragma unroll
    for (int j = 0; j < PP; ++j)
#pragma unroll
      for (int c = 0; c < NC; ++c) z[c] = fmaf(av[j], x(j, c), z[c]);
  }
  if (has1) {
#pragma unroll
    for (int j = 0; j < PP; ++j)
#pragma unroll
      for (int c = 0; c < NC; ++c) w[c] = fmaf(av[j], v(j, c), w[c]);
  }
  const size_t ro = (size_t)row * NC;
  if (a.kind == kRowsLogits) {
    if (valid) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        if (has0 && a.Z0out) a.Z0out[ro + c] = z[c];
        if (has1 && a.Z1out) a.Z1out[ro + c] = w[c];
      }
    }
    return;
  }
  float d[NC];
  float M = 0.f, alpha = 1.f;
  if (has0) {
#pragma unroll
    for (int c = 0; c < NC; ++c) M = fmaxf(M, z[c]);
    alpha = expf(-M);
#pragma unroll
    for (int c = 0; c < NC; ++c) { P[c] = expf(z[c] - M); alpha += P[c]; }
    const float inv = 1.f / alpha;
#pragma unroll
    for (int c = 0; c < NC; ++c) P[c] *= inv;
  }
  if (a.kind == kRowsHv) {
    float tt = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) tt = fmaf(P[c], w[c], tt);
#pragma unroll
    for (int c = 0; c < NC; ++c) d[c] = valid ? P[c] * (w[c] - tt) : 0.f;
  } else {
    float zb = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if (c == label) zb = z[c];
      d[c] = valid ? P[c] - (c == label ? 1.f : 0.f) : 0.f;
    }
    if (valid) loss_acc += (double)M + (double)logf(alpha) - (double)zb;
  }
  if (valid) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if (a.Pout) a.Pout[ro + c] = P[c];
      if (has0 && a.Z0out) a.Z0out[ro + c] = z[c];
    }
  }
  if (with_cols) {
#pragma unroll
    for (int j = 0; j < PP; ++j)
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[j][c] = fmaf(av[j], d[c], acc[j][c]);
  }
}

// Sum over the partials of element e = lane: lane e of wave w adds those of w, w + W, ... (requested by request(), all at once), and
// behind one barrier every wave adds up the waves' sums.
template <int THREADS>
struct PartialSum {
  static constexpr int W = THREADS / 64, U = kThinMaxPartials / W;
  float part[U];
  __device__ __forceinline__ void request(const ThinArgs& ta, int dlen, int ec) {
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = w + u * W;
      part[u] = ta.prev[(size_t)(k < ta.nprev ? k : ta.nprev - 1) * dlen + ec];
    }
  }
  __device__ __forceinline__ float sum(const ThinArgs& ta) {
    __shared__ float wave_part[W][64];
    const int e = threadIdx.x & 63, w = threadIdx.x >> 6;
    float s = 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u) s += w + u * W < ta.nprev ? part[u] : 0.f;
    wave_part[w][e] = s;
    lds_barrier();
    float s2 = 0.f;
#pragma unroll
    for (int k = 0; k < W; ++k) s2 += wave_part[k][e];
    return s2;
  }
};

// q = H d and the pending CG update (CgPend, Section 2.4) from the previous sweep's partial sums, which are requested together with
// both sets of vectors, so that nothing waits to learn which set is current; every wave makes the update for itself, one element of
// the vectors per lane.  (By the whole workgroup, as for longer vectors, it took five barriers: 1.3 us more per CG iteration at 2500 to 40000 rows.)
// Returns the lane's element of the new direction or of the final iterate; *go is false if no product is left to form.
// `writer`: this wave stores the new vectors and state.  after_issue(): the caller's first loads.
template <int THREADS, typename F>
__device__ __forceinline__ float cg_from_partials(const ThinArgs& ta, bool writer, bool* go, F&& after_issue) {
  const CgPend& c = ta.cg;
  DevState* st = c.st;
  const int e = threadIdx.x & 63;
  const int dlen = (int)c.dlen, ec = e < dlen ? e : dlen - 1;
  const bool own = e < dlen;
  PartialSum<THREADS> partials;
  partials.request(ta, dlen, ec);
  const float r0 = c.r[0][ec], r1 = c.r[1][ec], d0 = c.d[0][ec], d1 = c.d[1][ec], p0 = c.p[0][ec], p1 = c.p[1][ec];
  const CgSlot in = st->cgs[c.slot_in];
  const double gg = st->gg_cg;
  const float rho_ = ta.rho_scale != nullptr ? ta.rho * *ta.rho_scale : ta.rho;
  __builtin_amdgcn_sched_barrier(0);
  after_issue();
  __builtin_amdgcn_sched_barrier(0);
  const float s2 = partials.sum(ta);
  const int cur = in.cur & 1;
  float r = own ? (cur ? r1 : r0) : 0.f, d = own ? (cur ? d1 : d0) : 0.f, p = own ? (cur ? p1 : p0) : 0.f;
  const float q = own ? fmaf(ta.lambda + rho_, d, ta.scale * s2) : 0.f;
  CgSlot out = in;
  bool updated = false;
  float al = 0.f;
  if (in.active != 0) {  // uniform
    const double dq = mfma_detail::wave64_sum((double)d * (double)q);
    if (!(dq > 0.0) || !isfinite(dq)) {  // no positive curvature: keep the current iterate
      out.active = 0;
    } else {
      al = (float)(in.rr / dq);
      r = fmaf(-al, q, r);
      const double rr_new = mfma_detail::wave64_sum((double)r * (double)r);
      p = fmaf(al, d, p);
      d = fmaf((float)(rr_new / in.rr), d, r);
      out.rr = rr_new;
      out.iters = in.iters + 1;
      out.cur = cur ^ 1;
      // a tolerance of 0 is met by a zero residual only: no square roots in the chain
      if (c.tol > 0.f ? sqrt(rr_new) <= (double)c.tol * sqrt(gg) : rr_new == 0.0) out.active = 0;
      updated = true;
    }
  }
  if (writer) {
    if (own && updated) {
      (cur ? c.r[0] : c.r[1])[e] = r;
      (cur ? c.d[0] : c.d[1])[e] = d;
      (cur ? c.p[0] : c.p[1])[e] = p;
    }
    if (own && c.final_p != 0) c.p_final[e] = p;
    if (e == 0) {
      st->cgs[c.slot_in ^ 1] = out;
      if (updated && in.iters < kCgHist) st->cg_alphas[in.iters] = al;
      if (c.final_p != 0) {  // the scalars that the line search and the statistics read
        st->rr = out.rr;
        st->cg_iters = out.iters;
        st->cg_active = out.active;
      }
    }
  }
  *go = c.final_p != 0 || out.active != 0;
  return c.final_p != 0 ? p : d;
}

// The gradient, the head of a Newton iteration and the start of CG (newton_head_kernel) from the partial sums of the gradient's sweep,
// likewise: returns the lane's element of the first direction -g; *go is false if the iteration has ended.
template <int THREADS, typename F>
__device__ __forceinline__ float head_from_partials(const ThinArgs& ta, bool writer, bool* go, F&& after_issue) {
  const NewtonHeadArgs& h = ta.head;
  const int e = threadIdx.x & 63;
  const int dlen = (int)h.d, ec = e < dlen ? e : dlen - 1;
  const bool own = e < dlen;
  PartialSum<THREADS> partials;
  partials.request(ta, dlen, ec);
  const float x_in = h.X[ec], z_in = h.z != nullptr ? h.z[ec] : 0.f, y_in = h.y != nullptr ? h.y[ec] : 0.f;
  double lp[kThinMaxPartials / 64];  // row losses, one partial sum per workgroup of the gradient's sweep
#pragma unroll
  for (int u = 0; u < kThinMaxPartials / 64; ++u) {
    const int k = e + 64 * u;
    lp[u] = writer ? h.loss_part[k < h.nblocks ? k : h.nblocks - 1] : 0.0;
  }
  const float rho_ = h.rho_scale != nullptr ? h.rho * *h.rho_scale : h.rho;
  __builtin_amdgcn_sched_barrier(0);
  after_issue();
  __builtin_amdgcn_sched_barrier(0);
  const float s = partials.sum(ta);
  const float x = own ? x_in : 0.f, z = own ? z_in : 0.f, y = own ? y_in : 0.f;
  const float g = own ? h.scale * s + (h.lambda * x + rho_ * (x - z) + y) : 0.f;
  const double gg = mfma_detail::wave64_sum((double)g * (double)g);
  *go = gg > 0.0 && !(h.grad_tol > 0.f && sqrt(gg) < (double)h.grad_tol);
  if (writer) {
    const double u = (double)x - (double)z + (double)y / (double)rho_;
    const double pen = mfma_detail::wave64_sum(own ? 0.5 * (double)h.lambda * (double)x * (double)x + 0.5 * (double)rho_ * u * u : 0.0);
    double data = 0.0;
#pragma unroll
    for (int k = 0; k < kThinMaxPartials / 64; ++k) data += e + 64 * k < h.nblocks ? lp[k] : 0.0;
    data = mfma_detail::wave64_sum(data);
    if (own) {
      h.g_out[e] = g;
      h.pdir[e] = 0.f;
      h.r[e] = -g;
      h.dvec[e] = -g;
    }
    if (e == 0) newton_head_scalars(h, gg, (double)h.scale * data + pen);
  }
  return -g;
}

typedef __attribute__((address_space(1))) const void gvoid;
typedef __attribute__((address_space(3))) void lvoid;
template <int BYTES>  // lane l: BYTES from its own address g to l BYTES behind the wave's address to
__device__ __forceinline__ void copy_to_lds(const float* g, float* to) {
  static_assert(BYTES == 16 || BYTES == 4, "sizes that are used here");
  if constexpr (BYTES == 16) __builtin_amdgcn_global_load_lds((gvoid*)g, (lvoid*)to, 16, 0, 0);
  else __builtin_amdgcn_global_load_lds((gvoid*)g, (lvoid*)to, 4, 0, 0);
}

// What the sweep makes, fixed at compile time: chosen inside the loop it cost copies of all accumulators and spills.
// kHvCg, kHvHead: with cached probabilities; kSearchCg: with cached logits A X.
enum StreamOp { kHvX, kHvCg, kHvHead, kGrad, kLoss, kLogits, kLogitsCg, kSearch, kSearchCg };

template <int NQ, int NC, int THREADS, Rows ROWS, StreamOp OP>
__global__ __launch_bounds__(THREADS) void thin_stream_kernel(const ThinArgs ta) {
  constexpr int PP = 4 * NQ, D = PP * NC, W = THREADS / 64;
  RowArgs a = ta.r;
  a.kind = OP == kHvX || OP == kHvCg || OP == kHvHead ? kRowsHv : (OP == kGrad ? kRowsGrad : (OP == kLoss ? kRowsLoss : (OP == kLogits || OP == kLogitsCg ? kRowsLogits : kRowsSearch)));
  if (a.flag != nullptr && *a.flag == 0) {
    if (OP == kHvHead && blockIdx.x == 0 && threadIdx.x == 0) newton_head_skipped(ta.head);
    return;
  }
  extern __shared__ __attribute__((aligned(16))) float tile[];  // [wave][64 rows]
  __shared__ double red[W];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int p = a.p, ld = ROWS == kQuads ? PP : (int)a.lda;
  constexpr bool cg = OP == kHvCg || OP == kLogitsCg || OP == kSearchCg, search = OP == kSearch || OP == kSearchCg;
  const bool has0 = OP == kLogits ? a.B0 != nullptr : (OP == kHvX || OP == kGrad || OP == kLoss || OP == kSearch);
  const bool has1 = OP == kLogits ? a.B1 != nullptr : (OP == kHvX || OP == kHvHead || OP == kSearch || cg);
  constexpr bool with_cols = OP == kHvX || OP == kHvCg || OP == kHvHead || OP == kGrad;
  constexpr bool wants_label = OP == kGrad || OP == kLoss || search, wants_p = OP == kHvCg || OP == kHvHead || OP == kSearchCg;
  float* mine = tile + wave * (64 * PP);

  const bool aligned = (reinterpret_cast<uintptr_t>(a.A) & 15) == 0;
  const int64_t end_el = ROWS == kQuads && aligned ? a.n * ld : (a.n - 1) * ld + p;  // elements that may be read
  const int64_t last_el = (a.n - 1) * ld + p - 1;
  // kQuads: quad q of row r lies (q + turn(r)) % NQ quads behind the row's start, so that the lanes' reads of one quad spread over
  // the banks
  auto turn = [](int r) { return NQ % 8 == 0 ? (r & 7) : (NQ % 4 == 0 ? ((r >> 1) & 3) : (NQ % 2 == 0 ? ((r >> 2) & 1) : 0)); };
  auto source = [&](int slot) {  // kQuads: element of the chunk whose quad lies in this slot
    const int r = slot / NQ, q = slot % NQ - turn(r);
    return (r * NQ + (q < 0 ? q + NQ : q)) * 4;
  };
  auto fetch = [&](int64_t chunk) {
    const int64_t e0 = chunk * 64 * ld;
    if (aligned && e0 + 64 * ld <= end_el) {  // uniform
#pragma unroll
      for (int k = 0; k < NQ; ++k) {
        const int s = k * 64 + lane;
        if (ROWS == kQuads) copy_to_lds<16>(a.A + e0 + source(s), mine + k * 256);
        else if (k < NQ - 1 || s < 16 * ld) copy_to_lds<16>(a.A + e0 + 4 * s, mine + k * 256);  // 4 (NQ - 1) < ld
      }
    } else {
      // The matrix's last rows, or an A that starts between 16-byte boundaries.  The latter costs 6 to 40 % (1375000 rows, product:
      // 28 columns, C = 2: 31.3 us, 29.5 aligned; 32, C = 3: 47.7, 34.1); 16-byte loads through registers, for chunks of 256 rows, took 41.4 and
      // 69.4 there.
#pragma unroll 1
      for (int i = 0; i < ld; ++i) {
        const int s = i * 64 + lane;
        const int64_t e = e0 + (ROWS == kQuads ? source(s >> 2) + (s & 3) : s);
        copy_to_lds<4>(a.A + (e < last_el ? e : last_el), mine + i * 64);
      }
    }
  };

  const int64_t nchunks = (a.n + 63) / 64, step = (int64_t)gridDim.x * W;
  float Pn[NC];
  int label_n = -1;
  auto request = [&](int64_t chunk) {  // what a row needs beside A, ahead of its chunk: loads return in order
    const int64_t row = chunk * 64 + lane;
    const int64_t rc = row < a.n ? row : a.n - 1;
#pragma unroll
    for (int c = 0; c < NC; ++c) Pn[c] = wants_p ? a.Pin[rc * NC + c] : 0.f;
    if (wants_label) label_n = a.labels[rc];
    fetch(chunk);
  };
  int64_t chunk = blockIdx.x + (int64_t)gridDim.x * wave;
  // one entry of X and of V per lane (p (C-1) <= 64); the products read them lane by lane as scalar registers
  const int dlen = p * NC, le = lane < dlen ? lane : dlen - 1;
  float x_in = has0 ? a.B0[le] : 0.f, v_in = 0.f;
  if constexpr (cg || OP == kHvHead) {
    bool go;
    const bool writer = blockIdx.x == 0 && wave == 0;
    auto first = [&] {
      if (chunk < nchunks) request(chunk);
    };
    if constexpr (OP == kHvHead) v_in = head_from_partials<THREADS>(ta, writer, &go, first);
    else v_in = cg_from_partials<THREADS>(ta, writer, &go, first);
    if (!go) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing is on its way to LDS when the workgroup ends
      return;
    }
  } else {
    const float v = has1 ? a.B1[le] : 0.f;
    v_in = lane < dlen ? v : 0.f;
    if (chunk < nchunks) request(chunk);
  }
  x_in = lane < dlen ? x_in : 0.f;
  auto entry = [](float all, int e) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(all), e)); };
  float acc[PP][NC];
#pragma unroll
  for (int j = 0; j < PP; ++j)
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[j][c] = 0.f;
  double loss_acc = 0.0;
  double cand[search ? kSweepCand : 1];  // row losses per step size
#pragma unroll
  for (int k = 0; k < (search ? kSweepCand : 1); ++k) cand[k] = 0.0;

  while (chunk < nchunks) {  // uniform in a wave; no barrier inside
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the chunk is in LDS
    float av[PP], P[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) P[c] = Pn[c];
    const int label = label_n;
    if constexpr (ROWS == kBlock) {
#pragma unroll
      for (int j = 0; j < PP; ++j) av[j] = mine[lane * ld + j];  // at most 63 ld + PP - 1 < 64 PP
    } else {
      const int tr = turn(lane);
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int at = q + tr < NQ ? q + tr : q + tr - NQ;
        const f32x4 v = *reinterpret_cast<const f32x4*>(&mine[lane * PP + 4 * at]);
#pragma unroll
        for (int e = 0; e < 4; ++e) av[4 * q + e] = v[e];
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // and in registers: its place is free
#pragma unroll
    for (int j = PP - 4; j < PP; ++j) av[j] = j < p ? av[j] : 0.f;  // p > PP - 4
    const int64_t row = chunk * 64 + lane;
    if (chunk == nchunks - 1) {  // uniform: rows past the end
#pragma unroll
      for (int j = 0; j < PP; ++j) av[j] = row < a.n ? av[j] : 0.f;
    }
    const int64_t next = chunk + step;
    if (next < nchunks) request(next);
    if constexpr (search) {
      float z[NC], w[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        z[c] = OP == kSearch ? 0.f : P[c];
        w[c] = 0.f;
      }
#pragma unroll
      for (int j = 0; j < PP; ++j)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          if (OP == kSearch) z[c] = fmaf(av[j], entry(x_in, j * NC + c), z[c]);
          w[c] = fmaf(av[j], entry(v_in, j * NC + c), w[c]);
        }
#pragma unroll
      for (int k0 = 0; k0 < kSweepCand; k0 += 4) {
        if (k0 >= ta.search.ncand) continue;  // uniform; four step sizes at a time, those past the last one are 0 and not summed up
#pragma unroll
        for (int k = k0; k < k0 + 4; ++k) {
          float zz[NC], M = 0.f, zb = 0.f, es;
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            zz[c] = fmaf(ta.search.alphas[k], w[c], z[c]);
            M = fmaxf(M, zz[c]);
            zb = c == label ? zz[c] : zb;  // the reference class has logit 0
          }
          if constexpr (NC == 1) {
            es = 1.f + expf(fmaf(-2.f, M, zz[0]));  // of exp(-M) and exp(z - M) one is exp(0), the other exp(-|z|); NaN at z = +inf, as everywhere else
          } else {
            es = expf(-M);
#pragma unroll
            for (int c = 0; c < NC; ++c) es += expf(zz[c] - M);
          }
          cand[k] += row < a.n ? (double)M + (double)logf(es) - (double)zb : 0.0;
        }
      }
    } else {
      thin_row<PP, NC>(a, has0, has1, with_cols, row < a.n, row, av, [&](int j, int c) { return entry(x_in, j * NC + c); },
                       [&](int j, int c) { return entry(v_in, j * NC + c); }, P, label, acc, loss_acc);
    }
    chunk = next;
  }
  if constexpr (search) {  // the step sizes' sums: rows of 16 lanes by rotations, then the workgroup's 4 W row sums in a fixed order
    __syncthreads();
    double* sums = reinterpret_cast<double*>(tile);  // [step size][row of 16 lanes]: 512 W bytes, the smallest tile has 1024 W
#pragma unroll
    for (int k0 = 0; k0 < kSweepCand; k0 += 4) {
      if (k0 >= ta.search.ncand) continue;
      double s[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) s[k] = mfma_detail::row16_sum(cand[k0 + k]);
      if ((lane & 15) == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) sums[(k0 + k) * (4 * W) + 4 * wave + (lane >> 4)] = s[k];
      }
    }
    __syncthreads();
    if (t < 64) {  // four lanes per step size
      const int k = t >> 2;
      double s = 0.0;
      if (k < ta.search.ncand) {
#pragma unroll
        for (int w = 0; w < W; ++w) s += sums[k * (4 * W) + 4 * w + (t & 3)];
      }
      s += __shfl_xor(s, 1, 64);
      s += __shfl_xor(s, 2, 64);
      if ((t & 3) == 0 && k < ta.search.ncand) ta.search.lpart[(size_t)k * gridDim.x + blockIdx.x] = s;
    }
    return;
  }

  // ---- workgroup sums: every accumulator over each row of 16 lanes by rotations (a tree of shuffles each took 5 us here, where
  // nothing overlaps them), then the row sums in a fixed order ----
  __syncthreads();
  float* wsum = tile;  // [wave][row of 16 lanes][D]: 4 D floats of a wave's 64 PP
  if (with_cols) {
#pragma unroll
    for (int j = 0; j < PP; ++j)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const float v = mfma_detail::row16_sum(acc[j][c]);
        if ((lane & 15) == 0) wsum[(wave * 4 + (lane >> 4)) * D + j * NC + c] = v;
      }
  }
  if (a.loss_part != nullptr) {
    loss_acc = mfma_detail::wave64_sum(loss_acc);
    if (lane == 0) red[wave] = loss_acc;
  }
  __syncthreads();
  if (with_cols && t < p * NC) {
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w)
      s += (wsum[(4 * w) * D + t] + wsum[(4 * w + 1) * D + t]) + (wsum[(4 * w + 2) * D + t] + wsum[(4 * w + 3) * D + t]);
    ta.partial[(size_t)blockIdx.x * (p * NC) + t] = s;
  }
  if (a.loss_part != nullptr && t == 0) {
    double s = red[0];
#pragma unroll
    for (int w = 1; w < W; ++w) s += red[w];
    a.loss_part[blockIdx.x] = s;
  }
}

template <int NQ, int NC, Rows ROWS, StreamOp OP>
hipError_t launch_stream_op(const ThinArgs& ta, int grid, hipStream_t st) {
  constexpr int THREADS = 4 * NQ * NC <= 32 ? 1024 : 512;  // accumulators in 128 or 256 registers
  constexpr size_t lds = (size_t)THREADS * 4 * NQ * sizeof(float);
  if constexpr (lds + 1024 > 64 * 1024) {
    static LdsLimitMask done{0};
    const hipError_t e = ensure_lds_limit(reinterpret_cast<const void*>(&thin_stream_kernel<NQ, NC, THREADS, ROWS, OP>), &done, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((thin_stream_kernel<NQ, NC, THREADS, ROWS, OP>), dim3(grid), dim3(THREADS), lds, st, ta);
  return hipGetLastError();
}

template <int NQ, int NC, Rows ROWS>
hipError_t launch_stream(const ThinArgs& ta, int grid, hipStream_t st) {
  const RowArgs& a = ta.r;
  const bool cols = ta.partial != nullptr;
  if constexpr (4 * NQ * NC <= kThinMaxD) {
    if (ta.cg.st != nullptr) {
      if (a.kind == kRowsHv && cols && a.Pin != nullptr) return launch_stream_op<NQ, NC, ROWS, kHvCg>(ta, grid, st);
      if (a.kind == kRowsLogits && !cols && a.Z1out != nullptr) return launch_stream_op<NQ, NC, ROWS, kLogitsCg>(ta, grid, st);
      if (a.kind == kRowsSearch && !cols && a.Pin != nullptr) return launch_stream_op<NQ, NC, ROWS, kSearchCg>(ta, grid, st);
      return hipErrorInvalidValue;
    }
    if (ta.head.st != nullptr) {
      if (a.kind == kRowsHv && cols && a.Pin != nullptr) return launch_stream_op<NQ, NC, ROWS, kHvHead>(ta, grid, st);
      return hipErrorInvalidValue;
    }
    if (a.kind == kRowsHv && cols && a.B0 != nullptr && a.B1 != nullptr) return launch_stream_op<NQ, NC, ROWS, kHvX>(ta, grid, st);
    if (a.kind == kRowsGrad && cols && a.B0 != nullptr) return launch_stream_op<NQ, NC, ROWS, kGrad>(ta, grid, st);
    if (a.kind == kRowsLoss && !cols && a.B0 != nullptr) return launch_stream_op<NQ, NC, ROWS, kLoss>(ta, grid, st);
    if (a.kind == kRowsLogits && !cols) return launch_stream_op<NQ, NC, ROWS, kLogits>(ta, grid, st);
    if (a.kind == kRowsSearch && !cols && a.B0 != nullptr && a.B1 != nullptr) return launch_stream_op<NQ, NC, ROWS, kSearch>(ta, grid, st);
  }
  return hipErrorInvalidValue;
}

template <int NQ, Rows ROWS>
hipError_t launch_thin_nq(const ThinArgs& ta, int grid, hipStream_t st) {
  switch (ta.r.NC) {
    case 1: return launch_stream<NQ, 1, ROWS>(ta, grid, st);
    case 2: return launch_stream<NQ, 2, ROWS>(ta, grid, st);
    case 3: return launch_stream<NQ, 3, ROWS>(ta, grid, st);
    default: return hipErrorInvalidValue;
  }
}

template <Rows ROWS>
hipError_t launch_thin_rows(const ThinArgs& ta, int grid, hipStream_t st) {
  switch ((ta.r.lda + 3) >> 2) {
    case 1: return launch_thin_nq<1, ROWS>(ta, grid, st);
    case 2: return launch_thin_nq<2, ROWS>(ta, grid, st);
    case 3: return launch_thin_nq<3, ROWS>(ta, grid, st);
    case 4: return launch_thin_nq<4, ROWS>(ta, grid, st);
    case 5: return launch_thin_nq<5, ROWS>(ta, grid, st);
    case 6: return launch_thin_nq<6, ROWS>(ta, grid, st);
    case 7: return launch_thin_nq<7, ROWS>(ta, grid, st);
    case 8: return launch_thin_nq<8, ROWS>(ta, grid, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_thin_quads(const ThinArgs& ta, int grid, hipStream_t st);  // lda a multiple of 4
hipError_t launch_thin_block(const ThinArgs& ta, int grid, hipStream_t st);  // the others

}  // namespace nadmm
