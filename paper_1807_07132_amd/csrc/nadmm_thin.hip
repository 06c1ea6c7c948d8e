// Single-pass kernel for thin data (p <= 32 features, few classes), gfx950.
//
// With rows of 16..128 bytes the pass is a pure HBM stream (about 1.5 flop per
// byte for C = 2), so there is no contraction worth a matrix core: one lane owns
// one sample.  A workgroup copies a chunk of 256 consecutive rows -- a contiguous
// block of memory -- with coalesced 16-byte loads into LDS (row stride padded off
// the bank period), each lane reads its own row back, forms its logits Z = a_i X
// and W = a_i V with X and V as wave-uniform operands, the probabilities with the
// log-sum-exp shift (Section 2.2), its row of D (Section 2.6) or of P - Y, and
// accumulates a_i^T D into its private p x (C-1) registers.  The next chunk is
// already in flight in registers while the current one is consumed.  Per-lane
// accumulators are summed over the workgroup once, at the end, in a fixed order.
// Inside a Newton iteration the sweep of CG iteration k also does what lies between
// two sweeps (Section 2.4): it adds up the partial sums of sweep k - 1, forms q = H d
// and applies the CG update before it reads its operand (instantiations with CG).
#include <algorithm>
#include <cstring>

#include "nadmm_internal.h"
#include "nadmm_cgstep.h"
#include "nadmm_mfma.h"

namespace nadmm {
namespace {

constexpr int kThinThreads = 256;
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct ThinArgs {
  RowArgs r;
  float* partial;      // gridDim.x x (p*NC) or NULL
  int32_t rows_per_wg; // multiple of 256
  // Deferred CG update (kernels instantiated with CG): the sweep of the previous CG iteration left only its per-workgroup
  // partial sums of A^T D.  Every workgroup of this sweep adds them up (fixed order), forms q = H d, applies the update of
  // Section 2.4 and takes its operand, the new direction (or, for the line search's pass, the final iterate), from there;
  // workgroup 0 stores the new vectors and state.  No reduction kernel and no CG kernel run between two sweeps.
  CgPend cg;           // cg.q and cg.dot_part are not used: this kernel forms both itself
  const float* prev;   // the previous sweep's partial sums, nprev x (p*NC)
  int32_t nprev;
  float scale, lambda, rho;
  const float* rho_scale;
};

// NQ = p / 4: float4 per row, which is also the float4 per lane in a chunk of 256 rows
// ROWS: how the rows lie.  kDense: lda = p, a multiple of 4, 16-byte aligned.  The others (p odd, a few columns of padding, A
// 4-byte aligned; NQ = ceil(lda / 4)) would go through the matrix-core kernel for narrow rows, where one lane in 16 has work in
// the rows stage (1375000 x 29, C = 2, objective and gradient: 103 us).
//   kBlock: lda is no multiple of 4.  A block of rows lies in LDS as it does in memory, and the lanes read their rows back in
//     4-byte pieces: no bank conflicts where lda is odd, two lanes to a bank where it is even.
//   kQuads: lda = 4 NQ.  The lanes read whole quads, which lie turned within their rows.
enum Rows { kDense, kBlock, kQuads };

// floats per row in LDS, off the bank period
constexpr int tile_stride(int pp) { return pp % 8 == 0 ? pp + 4 : pp; }

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

template <int NQ, int NC, bool CG>
__global__ __launch_bounds__(kThinThreads) void thin_kernel(const ThinArgs ta) {
  constexpr int PP = 4 * NQ;
  constexpr int kMaxQuads = NQ;
  constexpr int nquads = NQ;
  const RowArgs& a = ta.r;
  if (a.flag != nullptr && *a.flag == 0) return;
  extern __shared__ __attribute__((aligned(16))) float tile[];  // 256 rows, see tile_stride
  __shared__ double red[4];
  const int t = threadIdx.x;
  constexpr int p = PP, PS = tile_stride(PP);
  const bool has0 = !CG && a.B0 != nullptr;
  const bool has1 = CG || a.B1 != nullptr;
  const bool with_cols = ta.partial != nullptr;

  const int64_t r_begin = (int64_t)blockIdx.x * ta.rows_per_wg;
  int64_t r_end = r_begin + ta.rows_per_wg;
  if (r_end > a.n) r_end = a.n;
  const f32x4* A4 = reinterpret_cast<const f32x4*>(a.A);
  const int64_t last4 = a.n * nquads - 1;  // last float4 of the matrix (lda == p)

  // X and V are the same for every lane: keep them as wave-uniform (scalar) registers
  float xs[PP][NC], vs[PP][NC];
  if constexpr (CG) {
    constexpr int D = PP * NC;      // length of the vectors, a multiple of 4
    constexpr int NQV = D / 4;      // quads per partial
    constexpr int GROUPS = kThinThreads / NQV;
    constexpr int U = 24;           // partials per thread and memory round trip
    __shared__ __attribute__((aligned(16))) float cgv[D];
    __shared__ __attribute__((aligned(16))) float cgq[D];
    __shared__ double cgdot[1];
    __shared__ double cgsm[kThinThreads / 64 + 1];
    const CgPend& c = ta.cg;
    const int cur = c.st->cgs[c.slot_in].cur & 1;
    const float* __restrict__ d_in = cur ? c.d[1] : c.d[0];
    const float rho_ = ta.rho_scale != nullptr ? ta.rho * *ta.rho_scale : ta.rho;
    const float dv = d_in[t < D ? t : D - 1];
    // thread (group g, quad qd) adds the partials g, g + GROUPS, ... of its quad, in that order
    const int qd = t % NQV, g = t / NQV;
    const int gc = g < GROUPS ? g : GROUPS - 1;
    const f32x4* __restrict__ pq = reinterpret_cast<const f32x4*>(ta.prev) + qd;
    f32x4 s4 = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k = gc; k < ta.nprev; k += U * GROUPS) {
      f32x4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int idx = k + u * GROUPS;
        v[u] = pq[(size_t)(idx < ta.nprev ? idx : ta.nprev - 1) * NQV];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k + u * GROUPS < ta.nprev) s4 += v[u];
    }
    f32x4* gs = reinterpret_cast<f32x4*>(tile);  // [group][quad]: at most 256 quads, the smallest tile holds them
    if (g < GROUPS) gs[g * NQV + qd] = s4;
    __syncthreads();
    if (t < 64) {  // the vectors fit one wave
      double prod = 0.0;
      if (t < D) {
        float s2 = 0.f;
        for (int g2 = 0; g2 < GROUPS; ++g2) s2 += tile[(g2 * NQV + (t >> 2)) * 4 + (t & 3)];
        const float qv = fmaf(ta.lambda + rho_, dv, ta.scale * s2);
        cgq[t] = qv;
        prod = (double)dv * (double)qv;
      }
      prod = mfma_detail::wave64_sum(prod);
      if (t == 0) cgdot[0] = prod;
    }
    __syncthreads();
    CgPend c2 = c;
    c2.q = cgq;
    c2.dot_part = cgdot;
    c2.ndot = 1;
    if (!cg_pending_update<kThinThreads, 1>(c2, blockIdx.x == 0, cgv, cgsm, [] {})) return;
#pragma unroll
    for (int j = 0; j < PP; ++j)
#pragma unroll
      for (int c1 = 0; c1 < NC; ++c1) {
        xs[j][c1] = 0.f;
        vs[j][c1] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(cgv[j * NC + c1])));
      }
    __syncthreads();  // the tile is about to be overwritten by the first chunk
  } else {
#pragma unroll
    for (int j = 0; j < PP; ++j)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        xs[j][c] = has0 ? __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(a.B0[j * NC + c]))) : 0.f;
        vs[j][c] = has1 ? __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(a.B1[j * NC + c]))) : 0.f;
      }
  }

  float acc[PP][NC];
#pragma unroll
  for (int j = 0; j < PP; ++j)
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[j][c] = 0.f;
  double loss_acc = 0.0;

  // position of this lane's k-th float4 inside a chunk: element 4 (t + 256 k) = row * PP + col
  int prow[kMaxQuads], pcol[kMaxQuads];
  {
    int row = (4 * t) / PP, col = (4 * t) % PP;
#pragma unroll
    for (int k = 0; k < kMaxQuads; ++k) {
      prow[k] = row;
      pcol[k] = col;
      row += 1024 / PP;
      col += 1024 % PP;
      if (col >= PP) { col -= PP; row += 1; }
    }
  }

  // Two chunks are in flight per workgroup: registers pf[0] and pf[1] alternate.  Loads are
  // unconditional (addresses clamped to the workgroup's own last float4), so the compiler can
  // wait for exactly the chunk it needs.
  f32x4 pf[2][kMaxQuads];
  const int64_t own_last4 = (r_end > r_begin ? r_end : r_begin + 1) * nquads - 1;
  auto load_chunk = [&](int b, int64_t row0) {
    const int64_t base4 = row0 * nquads + t;
#pragma unroll
    for (int k = 0; k < kMaxQuads; ++k) {
      int64_t i4 = base4 + (int64_t)k * kThinThreads;
      i4 = i4 < own_last4 ? i4 : own_last4;
      i4 = i4 < last4 ? i4 : last4;
      pf[b][k] = A4[i4];
    }
  };
  auto process = [&](int b, int64_t row0) {
    __syncthreads();  // rows of the previous chunk have been read
#pragma unroll
    for (int k = 0; k < kMaxQuads; ++k) {
      *reinterpret_cast<f32x4*>(__builtin_assume_aligned(&tile[prow[k] * PS + pcol[k]], 16)) = pf[b][k];
    }
    load_chunk(b, row0 + 2 * kThinThreads);
    __syncthreads();

    const int64_t row = row0 + t;
    const bool valid = row < r_end;
    float av[PP];
#pragma unroll
    for (int q = 0; q < PP / 4; ++q) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(__builtin_assume_aligned(&tile[t * PS + 4 * q], 16));
      av[4 * q + 0] = v[0]; av[4 * q + 1] = v[1]; av[4 * q + 2] = v[2]; av[4 * q + 3] = v[3];
    }
    float P[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) P[c] = (!has0 && valid && a.Pin != nullptr) ? a.Pin[(size_t)row * NC + c] : 0.f;
    const int label = (valid && a.kind != kRowsHv && a.kind != kRowsLogits) ? a.labels[row] : -1;
    thin_row<PP, NC>(a, has0, has1, with_cols, valid, row, av, [&](int j, int c) { return xs[j][c]; },
                     [&](int j, int c) { return vs[j][c]; }, P, label, acc, loss_acc);
  };

  if (r_begin < r_end) {
    load_chunk(0, r_begin);
    load_chunk(1, r_begin + kThinThreads);
  }
  for (int64_t row0 = r_begin; row0 < r_end; row0 += 2 * kThinThreads) {
    process(0, row0);
    if (row0 + kThinThreads < r_end) process(1, row0 + kThinThreads);
  }

  // ---- workgroup sums: every accumulator over each row of 16 lanes by rotations (no shuffles: 28 trees of six
  // shuffles each took 5 us here, where nothing overlaps them), then the 16 row sums in a fixed order ----
  __syncthreads();
  float* wsum = tile;  // [wave][row of 16 lanes][PP*NC]: 16 sums per accumulator (at most 4 KB, the smallest tile)
  const int lane = t & 63, wave = t >> 6;
  if (with_cols) {
#pragma unroll
    for (int j = 0; j < PP; ++j)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const float v = mfma_detail::row16_sum(acc[j][c]);
        if ((lane & 15) == 0) wsum[(wave * 4 + (lane >> 4)) * (PP * NC) + j * NC + c] = v;
      }
  }
  if (a.loss_part != nullptr) {
    loss_acc = mfma_detail::wave64_sum(loss_acc);
    if (lane == 0) red[wave] = loss_acc;
  }
  __syncthreads();
  if (with_cols && t < p * NC) {
    float w4[4];
#pragma unroll
    for (int w = 0; w < 4; ++w)
      w4[w] = (wsum[(4 * w) * (PP * NC) + t] + wsum[(4 * w + 1) * (PP * NC) + t]) +
              (wsum[(4 * w + 2) * (PP * NC) + t] + wsum[(4 * w + 3) * (PP * NC) + t]);
    ta.partial[(size_t)blockIdx.x * (p * NC) + t] = ((w4[0] + w4[1]) + w4[2]) + w4[3];
  }
  if (a.loss_part != nullptr && t == 0) a.loss_part[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

// The same for the other rows (kBlock, kQuads): no barrier and no prefetch registers.  A wave copies chunks of 64 rows -- one block
// of memory -- straight into its own part of LDS (global_load_lds), takes its rows from there into registers and has the next chunk
// on its way before it computes.  What is in flight is LDS, not registers: 16 waves per compute unit with up to 8 KB each.
// What bounds it: HBM.  Against chunks of 256 rows through registers (204 of them, so that only 512 of the 768 workgroups fitted,
// and surplus pieces past every chunk): objective and gradient at 1375000 x 29, C = 2: 53.5 -> 35.8 us (4.46 TB/s with the reduction's
// launch; the floor of one read of A is 28 us); Hessian-vector product at 600000 x 30, C = 3: 45.9 -> 20.7 us.
typedef __attribute__((address_space(1))) const void gvoid;
typedef __attribute__((address_space(3))) void lvoid;
template <int BYTES>  // lane l: BYTES from its own address g to l BYTES behind the wave's address to
__device__ __forceinline__ void copy_to_lds(const float* g, float* to) {
  static_assert(BYTES == 16 || BYTES == 4, "sizes that are used here");
  if constexpr (BYTES == 16) __builtin_amdgcn_global_load_lds((gvoid*)g, (lvoid*)to, 16, 0, 0);
  else __builtin_amdgcn_global_load_lds((gvoid*)g, (lvoid*)to, 4, 0, 0);
}

// What the sweep makes, fixed at compile time: chosen inside the loop it cost copies of all accumulators and spills.
enum StreamOp { kHvX, kHvP, kGrad, kLoss, kLogits };  // kHvP: with cached probabilities

template <int NQ, int NC, int THREADS, Rows ROWS, StreamOp OP>
__global__ __launch_bounds__(THREADS) void thin_stream_kernel(const ThinArgs ta) {
  constexpr int PP = 4 * NQ, D = PP * NC, W = THREADS / 64;
  RowArgs a = ta.r;
  a.kind = OP == kHvX || OP == kHvP ? kRowsHv : (OP == kGrad ? kRowsGrad : (OP == kLoss ? kRowsLoss : kRowsLogits));
  if (a.flag != nullptr && *a.flag == 0) return;
  extern __shared__ __attribute__((aligned(16))) float tile[];  // [wave][64 rows]
  __shared__ double red[W];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int p = a.p, ld = ROWS == kQuads ? PP : (int)a.lda;
  const bool has0 = OP == kLogits ? a.B0 != nullptr : OP != kHvP;
  const bool has1 = OP == kLogits ? a.B1 != nullptr : (OP == kHvX || OP == kHvP);
  constexpr bool with_cols = OP == kHvX || OP == kHvP || OP == kGrad;
  constexpr bool wants_label = OP == kGrad || OP == kLoss, wants_p = OP == kHvP;
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
    } else {  // the matrix's last rows, or rows that start between 16-byte boundaries
#pragma unroll 1
      for (int i = 0; i < ld; ++i) {
        const int s = i * 64 + lane;
        const int64_t e = e0 + (ROWS == kQuads ? source(s >> 2) + (s & 3) : s);
        copy_to_lds<4>(a.A + (e < last_el ? e : last_el), mine + i * 64);
      }
    }
  };

  // one entry of X and of V per lane (p (C-1) <= 64); the products read them lane by lane as scalar registers
  const int le = lane < p * NC ? lane : p * NC - 1;
  float x_in = has0 ? a.B0[le] : 0.f, v_in = has1 ? a.B1[le] : 0.f;
  x_in = lane < p * NC ? x_in : 0.f;
  v_in = lane < p * NC ? v_in : 0.f;
  auto entry = [](float all, int e) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(all), e)); };
  float acc[PP][NC];
#pragma unroll
  for (int j = 0; j < PP; ++j)
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[j][c] = 0.f;
  double loss_acc = 0.0;

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
  if (chunk < nchunks) request(chunk);
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
    thin_row<PP, NC>(a, has0, has1, with_cols, row < a.n, row, av, [&](int j, int c) { return entry(x_in, j * NC + c); },
                     [&](int j, int c) { return entry(v_in, j * NC + c); }, P, label, acc, loss_acc);
    chunk = next;
  }

  // ---- workgroup sums as in thin_kernel ----
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
  if constexpr (4 * NQ * NC <= 64) {
    if (a.kind == kRowsHv && cols && a.B1 != nullptr && (a.B0 != nullptr || a.Pin != nullptr))
      return a.B0 != nullptr ? launch_stream_op<NQ, NC, ROWS, kHvX>(ta, grid, st) : launch_stream_op<NQ, NC, ROWS, kHvP>(ta, grid, st);
    if (a.kind == kRowsGrad && cols && a.B0 != nullptr) return launch_stream_op<NQ, NC, ROWS, kGrad>(ta, grid, st);
    if (a.kind == kRowsLoss && !cols && a.B0 != nullptr) return launch_stream_op<NQ, NC, ROWS, kLoss>(ta, grid, st);
    if (a.kind == kRowsLogits && !cols) return launch_stream_op<NQ, NC, ROWS, kLogits>(ta, grid, st);
  }
  return hipErrorInvalidValue;
}

template <int NQ, int NC, bool CG>
hipError_t launch_rows(const ThinArgs& ta, int grid, hipStream_t st) {
  const size_t lds = (size_t)kThinThreads * tile_stride(4 * NQ) * sizeof(float);
  hipLaunchKernelGGL((thin_kernel<NQ, NC, CG>), dim3(grid), dim3(kThinThreads), lds, st, ta);
  return hipGetLastError();
}

template <int NQ, int NC>
hipError_t launch_thin_t(const ThinArgs& ta, int grid, bool cg, Rows rows, hipStream_t st) {
  if (rows != kDense && cg) return hipErrorInvalidValue;
  if (rows == kQuads) return launch_stream<NQ, NC, kQuads>(ta, grid, st);
  if (rows == kBlock) return launch_stream<NQ, NC, kBlock>(ta, grid, st);
  return cg ? launch_rows<NQ, NC, true>(ta, grid, st) : launch_rows<NQ, NC, false>(ta, grid, st);
}

template <int NQ>
hipError_t launch_thin_nq(const ThinArgs& ta, int grid, bool cg, Rows rows, hipStream_t st) {
  switch (ta.r.NC) {
    case 1: return launch_thin_t<NQ, 1>(ta, grid, cg, rows, st);
    case 2: return launch_thin_t<NQ, 2>(ta, grid, cg, rows, st);
    case 3: return launch_thin_t<NQ, 3>(ta, grid, cg, rows, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

bool thin_supported(const Shape& s, int64_t lda, const void* A) {
  if (s.p > 32 || (s.p & 3) != 0 || s.NC > 3 || s.p * s.NC > 64) return false;
  if (lda != s.p || (reinterpret_cast<uintptr_t>(A) & 15) != 0) return false;
  return true;
}

// Any other rows of up to 32 columns: at most 3 elements of padding, so that 256 rows are one
// block of about 256 p floats; the accumulators of the padded row fit the registers.
bool thin_general_supported(const Shape& s, int64_t lda, const void* A) {
  const int64_t pp = (lda + 3) / 4 * 4;
  if (lda < s.p || lda > 32 || s.NC > 3 || pp * s.NC > 64 || s.p <= pp - 4) return false;
  return s.n * lda >= 8 && (s.n - 1) * lda + s.p >= 4 && (reinterpret_cast<uintptr_t>(A) & 3) == 0;
}

// Rows with padding that are 16-byte aligned, of more than one operand piece: up to 65536 of them are faster on the narrow-row kernel,
// which works to the same accuracy (Hessian-vector products within 4.0e-8 to 6.0e-8 of 64 bits, here 3.5e-8 to 5.8e-8) and defers the
// CG update into the next sweep (here the vectors, p (C-1) long, are no whole quads).  With more rows the stream counts, one lane
// per row against one in 16 with work in the rows stage; 32 x 2 accumulators leave so few waves in flight here that it takes 393216.
// Measured, this kernel against the narrow one (us, 3 to 8 CG iterations): lda = 32, C = 3: 5000 rows 139 : 98, 60000 rows
// 1.40 times, 220000 rows 1.70 times as fast on the narrow one, one gradient at 300000 rows 1.03, at 400000 0.92 times; lda = 20,
// C = 4: 2500 rows 1.37, 60000 rows 1.28, gradient at 80000 rows 0.96; lda = 12, C = 3: 20000 rows 1.06, 80000 rows 0.89; lda = 16, C = 2:
// 2500 rows 0.94, 20000 rows 1.02.  Single sweeps are equal up to 65536 rows.  Up to 2048 rows all CG iterations are one launch
// (nadmm_small.hip): 300 rows 0.32 to 0.80.
bool thin_padded_narrow(const Shape& s, int64_t lda) {
  return s.n > 2048 && lda * s.NC > 16 && s.n < (lda * s.NC < 64 ? 65536 : 393216);
}

int thin_num_partials(const Shape& s) {
  // 3 resident workgroups per compute unit for small accumulator sets, else 2 (register budget);
  // every workgroup gets the same whole number of 256-row chunks
  const int64_t cap = (s.p * s.NC <= 32) ? 768 : 512;
  const int64_t chunks = (s.n + kThinThreads - 1) / kThinThreads;
  const int64_t g = chunks < cap ? chunks : cap;
  const int64_t per = (chunks + g - 1) / g;
  return (int)((chunks + per - 1) / per);
}

// other rows (thin_stream_kernel): one workgroup per compute unit, and every wave with a chunk of 64 rows before any has two
int thin_stream_partials(const Shape& s) { return (int)std::min<int64_t>(256, (s.n + 63) / 64); }

hipError_t launch_thin(const RowArgs& a, float* partial, int nparts, hipStream_t st, const CgPend* cg, const ReduceArgs* prev) {
  ThinArgs ta;
  std::memset(&ta, 0, sizeof(ta));
  ta.r = a;
  ta.partial = partial;
  const int64_t chunks = (a.n + kThinThreads - 1) / kThinThreads;
  ta.rows_per_wg = (int32_t)((chunks + nparts - 1) / nparts) * kThinThreads;
  const bool with_cg = cg != nullptr;
  if (with_cg) {
    // the pending update of a CG iteration on cached probabilities (or the line search's logits pass on the final iterate)
    if (prev == nullptr || prev->partial == nullptr || prev->nparts < 1 || prev->d != (int64_t)a.p * a.NC) return hipErrorInvalidValue;
    if (a.B0 != nullptr || (a.kind != kRowsHv && a.kind != kRowsLogits) || cg->dlen != prev->d || cg->st == nullptr) return hipErrorInvalidValue;
    if (prev->partial == partial) return hipErrorInvalidValue;  // the sweep reads the previous partials while it writes its own
    ta.cg = *cg;
    ta.prev = prev->partial;
    ta.nprev = prev->nparts;
    ta.scale = prev->scale;
    ta.lambda = prev->lambda;
    ta.rho = prev->rho;
    ta.rho_scale = prev->rho_scale;
  }
  const bool dense = thin_supported(Shape{a.n, a.p, a.NC, (int64_t)a.p * a.NC}, a.lda, a.A);
  const Rows rows = dense ? kDense : ((a.lda & 3) == 0 ? kQuads : kBlock);
  switch ((a.lda + 3) >> 2) {
    case 1: return launch_thin_nq<1>(ta, nparts, with_cg, rows, st);
    case 2: return launch_thin_nq<2>(ta, nparts, with_cg, rows, st);
    case 3: return launch_thin_nq<3>(ta, nparts, with_cg, rows, st);
    case 4: return launch_thin_nq<4>(ta, nparts, with_cg, rows, st);
    case 5: return launch_thin_nq<5>(ta, nparts, with_cg, rows, st);
    case 6: return launch_thin_nq<6>(ta, nparts, with_cg, rows, st);
    case 7: return launch_thin_nq<7>(ta, nparts, with_cg, rows, st);
    case 8: return launch_thin_nq<8>(ta, nparts, with_cg, rows, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace nadmm
