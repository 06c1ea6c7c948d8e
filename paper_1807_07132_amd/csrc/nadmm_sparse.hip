// Kernels for A in sparse storage (gfx950): both products with A are the same operation, a
// compressed-rows matrix S times a dense matrix B with few columns,
//   pass 1:  [Z | W] = A [X | V]      S = row view of A,    B = [X | V]   (Sections 2.1, 2.6)
//   pass 2:  A^T D                    S = column view of A, B = D         (Section 2.6)
// followed by the rows stage on logits and the fixed-order reduction that the dense paths use.
//
// The rows of B are first copied into a buffer in which every row takes a power-of-two number G of
// 16-byte quads (zero padded), so that a row lies in one 128-byte cache line.  A wave reads 64 (index,
// value) pairs with two coalesced loads and hands them out by lane shuffles; as many neighbouring lanes
// as a row of B has quads then share an entry, each loading one quad of the row that the entry points to,
// so that a load instruction touches each of its rows once, and each lane keeps the partial sums of its quad; at the
// end of a row of S the lanes holding the same quad are added across the wave.  Work is cut into
// windows of equal cost (stored entries plus a fixed cost per row) by a binary search over the row
// pointers; a workgroup owns the rows that start in its window: rows of fewer than 48 entries go to 16 lanes each, others to single waves, long
// ones are shared by its four waves and combined in LDS in wave order.  A row longer than a window is cut where the windows are: every one
// it reaches over sums its share (the windows inside such a row have no rows of their own), and whichever arrives last adds the shares in their
// order; where the caller's memory has no room for the shares, one workgroup does both.  Before, one workgroup took such a row whole, 0.9 us for
// 240 entries, while the others had long ended: columns of the 60000 x 9000 counts of the benchmark's kind (200 a row, C = 28) 241 us for the
// product with A^T, 62 for the one with A.  The order of additions depends on the matrix only: results are reproducible bit for bit.
// What each of the forms gives, the others in place (us a Hessian-vector product, without and with): cutting 2012 and 1938 at 40628 x 279998, C = 20, 385 and 274 at
// 60000 x 9000, C = 28; 16 lanes for short rows 105 and 71 at 50000 x 200000, C = 4 (30 a row), but 65 and 67 at 6000 x 4000, C = 20, where few rows are short;
// windows by size 48 and 31 at 2000 x 2000, C = 3, 80 and 67 at 6000 x 4000.
#include "nadmm_internal.h"
#include "nadmm_mfma.h"

namespace nadmm {
namespace {

constexpr int kSpThreads = 256;
constexpr int kSpWaves = kSpThreads / 64;
constexpr int kMinShift = 9, kMaxShift = 12;  // windows of 512 to 4096 cost units per workgroup
constexpr int kRowCost = 8;    // cost of a row beyond its entries (bounds the rows per window)
constexpr int kLong = 512;     // rows with at least this many entries are shared by the waves of the workgroup; as long as a window, they are cut at its ends
constexpr int kShort = 48;     // rows with fewer entries are summed by 16 lanes (16 and 24: up to 16 % slower at 30 entries a row; 80: equal)
constexpr int kMaxLong = (1 << kMaxShift) / (kLong + kRowCost) + 3;  // long rows that start in a window, and one that reaches into it

// Per window of either view (the first n0 blocks are of view 0): the first row r in [0, nrows] whose cost prefix ptr[r] + kRowCost r reaches it
__global__ __launch_bounds__(256) void plan_kernel(const SparseView S0, const SparseWindows w0, const SparseView S1, const SparseWindows w1, int blocks0,
                                                   int32_t* __restrict__ arrived) {
  const bool second = (int)blockIdx.x >= blocks0;
  const SparseView& S = second ? S1 : S0;
  const SparseWindows& w = second ? w1 : w0;
  const int k = ((int)blockIdx.x - (second ? blocks0 : 0)) * 256 + threadIdx.x;
  if (k > w.n) return;
  if (k < w.n && arrived != nullptr) arrived[k] = arrived[w.n + k] = 0;  // both operands' passes
  if (k == w.n) {
    w.first[k] = (int32_t)S.nrows;
    return;
  }
  const int64_t target = (int64_t)k << w.shift;
  int64_t lo = 0, hi = S.nrows;  // answer in [lo, hi]
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (S.ptr[mid] + (int64_t)kRowCost * mid >= target) hi = mid;
    else lo = mid + 1;
  }
  w.first[k] = (int32_t)lo;
}

// dst[r][op][slot] = src_op[r][NC], zero in the padding (slot = 4 G floats); one thread per group of 4 floats
__global__ __launch_bounds__(256) void pack_kernel(const float* __restrict__ src0, const float* __restrict__ src1,
                                                   int64_t rows, int NC, int G, int nops,
                                                   float* __restrict__ dst, const int32_t* flag) {
  if (flag != nullptr && *flag == 0) return;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = rows * nops * G;
  if (t >= total) return;
  const int q = (int)(t % G);
  const int64_t ro = t / G;
  const int op = (int)(ro % nops);
  const int64_t r = ro / nops;
  const float* __restrict__ src = (op == 0 ? src0 : src1) + (size_t)r * NC;
  mfma_detail::f32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = (4 * q + e < NC) ? src[4 * q + e] : 0.f;
  reinterpret_cast<mfma_detail::f32x4*>(dst)[t] = v;
}

struct RowSpan {
  int64_t k0, k1;
};
__device__ __forceinline__ RowSpan row_span(const SparseView& S, int64_t r) {
  int64_t k0 = S.ptr[r], k1 = S.ptr[r + 1];
  k0 = k0 < 0 ? 0 : (k0 > S.nnz ? S.nnz : k0);
  k1 = k1 < k0 ? k0 : (k1 > S.nnz ? S.nnz : k1);
  return RowSpan{k0, k1};
}

// A row that is cut: its entries inside window k (as costs go, the entries come first and kRowCost behind them), and the first and last window
// that holds any
struct Cut {
  RowSpan here;
  int first, last;
};
__device__ __forceinline__ Cut cut_span(const RowSpan& sp, int64_t r, int k, int wshift) {
  const int64_t c0 = sp.k0 + (int64_t)kRowCost * r, len = sp.k1 - sp.k0;
  const int64_t w0 = ((int64_t)k << wshift) - c0, w1 = w0 + ((int64_t)1 << wshift);
  Cut c;
  c.first = (int)(c0 >> wshift);
  c.last = (int)((c0 + len - 1) >> wshift);
  c.here.k0 = sp.k0 + (w0 < 0 ? 0 : (w0 > len ? len : w0));
  c.here.k1 = sp.k0 + (w1 < 0 ? 0 : (w1 > len ? len : w1));
  return c;
}

// the stored entries of a chunk from kb on, one per lane (value 0 and a valid index beyond the end)
struct Chunk {
  int col;
  float v;
};
__device__ __forceinline__ Chunk fetch_chunk(const SparseView& S, int64_t kb, int64_t k1, int size, int lane) {
  const int64_t k = kb + lane;
  const bool ok = k < k1 && lane < size;  // lanes beyond the chunk hold no entry
  const int64_t kc = k < k1 ? k : k1 - 1;
  const int c = S.idx[kc];
  Chunk ch;
  ch.v = ok ? S.val[kc] : 0.f;
  ch.col = c < 0 ? 0 : (c >= S.ncols ? S.ncols - 1 : c);
  return ch;
}

// Lanes per wave that hold entries, for rows of NQ quads: S = 64 / NQ entries share a load instruction
// (lane = s NQ + q reads quad q of the B row of entry s), a chunk is T = 64 / S such groups.
template <int NQ>
struct Shape64 {
  static constexpr int S = 64 / NQ;
  static constexpr int T = 64 / S;
  static constexpr int CE = S * T;  // entries per chunk: 64, or a little less where NQ does not divide 64
};

// The sum of value * (row of B) over the entries of the chunks kb0, kb0 + stride, ... of [.., k1).
// NQ neighbouring lanes share an entry, one quad of its B row each, so that one load instruction touches
// every row once (several loads of one lane to one cache line would wait on each other in the vector
// L1).  Returns, in lanes 0 .. NQ-1, the sums of quad q = lane over the whole wave.
template <int NQ, int NPER, int NOPS>
__device__ __forceinline__ void row_sum(const SpmmArgs& a, const mfma_detail::f32x4* __restrict__ B, int64_t kb0, int64_t k1, int stride, int lane,
                                        mfma_detail::f32x4 (&acc)[NPER]) {
  using mfma_detail::f32x4;
  constexpr int S = Shape64<NQ>::S, T = Shape64<NQ>::T, CE = Shape64<NQ>::CE;
  constexpr int G = NQ <= 1 ? 1 : (NQ <= 2 ? 2 : (NQ <= 4 ? 4 : 8));  // quads per row slot of B
  const int s = lane / NQ, q = lane - s * NQ;
  const bool active = lane < S * NQ;
  const f32x4* __restrict__ Bq = B + q;
#pragma unroll
  for (int op = 0; op < NPER; ++op) acc[op] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (kb0 >= k1) return;
  Chunk cur = fetch_chunk(a.S, kb0, k1, CE, lane);
  for (int64_t kb = kb0; kb < k1; kb += stride) {
    const int64_t left = k1 - kb;
    const int nsub = left >= CE ? T : (int)((left + S - 1) / S);
    f32x4 b[T][NPER];
    float vv[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int c = __shfl(cur.col, t * S + s, 64);
      vv[t] = __shfl(cur.v, t * S + s, 64);
      const f32x4* __restrict__ row = Bq + (size_t)c * (NOPS * G);
#pragma unroll
      for (int op = 0; op < NPER; ++op) b[t][op] = (t < nsub && active) ? row[op * G] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if (kb + stride < k1) cur = fetch_chunk(a.S, kb + stride, k1, CE, lane);  // in flight during the products
#pragma unroll
    for (int t = 0; t < T; ++t) {
#pragma unroll
      for (int op = 0; op < NPER; ++op) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[op][e] = fmaf(vv[t], b[t][op][e], acc[op][e]);
      }
    }
  }
  // add the S lanes of each quad: halving tree over s, fixed order
  int cnt = S;
#pragma unroll
  for (int h = 32; h >= 1; h >>= 1) {
    if (h < cnt) {
      const bool take = s + h < cnt;
#pragma unroll
      for (int op = 0; op < NPER; ++op) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float o = __shfl_down(acc[op][e], h * NQ, 64);
          acc[op][e] += take ? o : 0.f;
        }
      }
      cnt = h;
    }
  }
}

// The same for four short rows at once, 16 lanes each (row k0 .. k0 + len is the same in all of them): a tree over 16 lanes instead of 64 and a quarter
// of the waits.  Returns the sums of quad q in lane q of the 16.
template <int NQ, int NPER, int NOPS>
__device__ __forceinline__ void short_rows_sum(const SpmmArgs& a, const mfma_detail::f32x4* __restrict__ B, int64_t k0, int len, int lane,
                                               mfma_detail::f32x4 (&acc)[NPER]) {
  using mfma_detail::f32x4;
  constexpr int S = 16 / NQ, T = (16 + S - 1) / S;  // entries of a row per load instruction, such loads per 16 entries
  constexpr int G = NQ <= 1 ? 1 : (NQ <= 2 ? 2 : (NQ <= 4 ? 4 : 8));
  const int l = lane & 15, s = l / NQ, q = l - s * NQ;
  const f32x4* __restrict__ Bq = B + q;
#pragma unroll
  for (int op = 0; op < NPER; ++op) acc[op] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int kb = 0; __any(kb < len); kb += 16) {
    int64_t k = k0 + kb + l;
    k = k < a.S.nnz ? k : a.S.nnz - 1;
    const int c0 = a.S.idx[k];
    const float v0 = kb + l < len ? a.S.val[k] : 0.f;
    const int c = c0 < 0 ? 0 : (c0 >= a.S.ncols ? a.S.ncols - 1 : c0);
    constexpr int U = (T + 1) / 2 < 4 / NPER ? (T + 1) / 2 : 4 / NPER;  // loads in flight: more would cost the kernel waves
#pragma unroll
    for (int t0 = 0; t0 < T; t0 += U) {
      if (!__any(kb + t0 * S < len)) break;
      f32x4 b[U][NPER];
      float vv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = (t0 + u) * S + s;
        const int cc = __shfl(c, (lane & 48) + (e & 15), 64);
        const float w = __shfl(v0, (lane & 48) + (e & 15), 64);
        const bool ok = s < S && e < 16 && kb + e < len;
        vv[u] = ok ? w : 0.f;
        const f32x4* __restrict__ row = Bq + (size_t)cc * (NOPS * G);
#pragma unroll
        for (int op = 0; op < NPER; ++op) b[u][op] = ok ? row[op * G] : f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int op = 0; op < NPER; ++op) {
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[op][e] = fmaf(vv[u], b[u][op][e], acc[op][e]);
        }
      }
    }
  }
  int cnt = S;
#pragma unroll
  for (int h = 8; h >= 1; h >>= 1) {
    if (h < cnt) {
      const bool take = s + h < cnt;
#pragma unroll
      for (int op = 0; op < NPER; ++op) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float o = __shfl_down(acc[op][e], h * NQ, 64);
          acc[op][e] += take ? o : 0.f;
        }
      }
      cnt = h;
    }
  }
}

template <int NPER>
__device__ __forceinline__ void store_row(const SpmmArgs& a, float* __restrict__ out, int row, int q, const mfma_detail::f32x4 (&acc)[NPER]) {
  float* __restrict__ orow = out + (size_t)row * (a.nops * a.NC);
#pragma unroll
  for (int op = 0; op < NPER; ++op) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int c = 4 * q + e;
      if (c < a.NC) orow[op * a.NC + c] = acc[op][e];
    }
  }
}

__device__ __forceinline__ int64_t lane_of(int64_t x, int i) {
  return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), i) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)x, i));
}

// NPER of the NOPS operands are multiplied together, the others by further workgroups (blockIdx.y).
// 5 to 7 quads: a wave more per SIMD than the compiler would leave room for, at 1 to 2 spilled registers with 6 and 7 (6000 x 4000, 400 a row, C = 20: 70 -> 67 us a
// Hessian-vector product; 40000 x 100000, 300 a row, C = 20: 291 -> 296; 60000 x 9000, C = 28, and 40628 x 279998, C = 20: within 1 %; fewer or more quads, or
// two operands, are slower with that, 2 to 25 %)
// SHARED: rows as long as a window are shared by the workgroups of the windows they reach over.  Without room for the shares the one in whose
// window such a row starts takes all of it, window by window and in the same order of additions: the results are the same bit for bit.
template <int NQ, int NPER, int NOPS, bool SHARED>
__global__ __launch_bounds__(kSpThreads, NPER == 1 && NQ >= 5 && NQ <= 7 ? 7 : 1) void spmm_kernel(const SpmmArgs a) {
  constexpr int G = 8;  // bound of NQ, for the LDS staging of long rows
  constexpr int CE = Shape64<NQ>::CE;
  using mfma_detail::f32x4;
  if (a.flag != nullptr && *a.flag == 0) return;
  __shared__ int long_rows[kMaxLong];
  __shared__ int nlong_sh;
  __shared__ float part[kMaxLong][kSpWaves][NPER][G][4];
  __shared__ int last_sh[2];
  const int win = blockIdx.x;
  const int r0 = a.w.first[win], r1 = a.w.first[win + 1];
  const int wshift = a.w.shift;
  const int64_t kCut = (int64_t)1 << wshift;
  // the cut row that reaches into this window from before it, and the one that starts here and reaches beyond it (the last that starts here)
  bool into = false, beyond = false;
  if (SHARED && r0 > 0) {
    const RowSpan sp = row_span(a.S, r0 - 1);
    into = sp.k1 - sp.k0 >= kCut && cut_span(sp, r0 - 1, win, wshift).last >= win;
  }
  if (SHARED && r1 > r0) {
    const RowSpan sp = row_span(a.S, r1 - 1);
    beyond = sp.k1 - sp.k0 >= kCut && cut_span(sp, r1 - 1, win, wshift).last > win;
  }
  if (r1 <= r0 && !into) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int kSlot = NQ <= 1 ? 1 : (NQ <= 2 ? 2 : (NQ <= 4 ? 4 : 8));  // quads per row slot of an operand
  const f32x4* __restrict__ B = reinterpret_cast<const f32x4*>(a.B) + blockIdx.y * kSlot;
  float* __restrict__ out = a.out + blockIdx.y * a.NC;
  const int ldo = NOPS * a.NC, width = NPER * a.NC;
  float* share = SHARED ? a.share + (size_t)blockIdx.y * 2 * a.w.n * width : nullptr;

  if (threadIdx.x == 0) {
    nlong_sh = into ? 1 : 0;
    if (into) long_rows[0] = r0 - 1;
  }
  __syncthreads();
  for (int r = r0 + (int)threadIdx.x; r < r1; r += kSpThreads) {
    const RowSpan sp = row_span(a.S, r);
    if (sp.k1 - sp.k0 >= kLong) {
      const int slot = atomicAdd(&nlong_sh, 1);
      if (slot < kMaxLong) long_rows[slot] = r;
    }
  }
  __syncthreads();
  const int nlong = nlong_sh < kMaxLong ? nlong_sh : kMaxLong;

  // long rows: wave w takes chunks w, w + 4, ...; partial sums to LDS
  constexpr int kPer = NPER * G * 4;
  auto wave_sums = [&](const RowSpan& sp, int sl) {
    f32x4 acc[NPER];
    row_sum<NQ, NPER, NOPS>(a, B, sp.k0 + CE * wave, sp.k1, CE * kSpWaves, lane, acc);
    if (lane < NQ) {
#pragma unroll
      for (int op = 0; op < NPER; ++op) {
#pragma unroll
        for (int e = 0; e < 4; ++e) part[sl][wave][op][lane][e] = acc[op][e];
      }
    }
  };
  auto add_waves = [&](int sl, int j) {
    const float* pj = &part[sl][0][0][0][0] + j;
    float sum = pj[0];
#pragma unroll
    for (int w = 1; w < kSpWaves; ++w) sum += pj[w * kPer];
    return sum;
  };
  for (int sl = 0; sl < nlong; ++sl) {
    const int row = long_rows[sl];
    RowSpan sp = row_span(a.S, row);
    if (sp.k1 - sp.k0 >= kCut) {  // uniform
      if constexpr (!SHARED) {
        const Cut c = cut_span(sp, row, win, wshift);
        const int j = threadIdx.x, op = j / (4 * G), cl = j - op * (4 * G);
        float sum = c.first == c.last ? -0.f : 0.f;  // x + -0 is x
        for (int w = c.first; w <= c.last; ++w) {
          wave_sums(cut_span(sp, row, w, wshift).here, sl);
          __syncthreads();
          if (j < kPer) sum += add_waves(sl, j);
          __syncthreads();
        }
        if (j < kPer && cl < a.NC) out[(size_t)row * ldo + op * a.NC + cl] = sum;
        continue;
      }
      sp = cut_span(sp, row, win, wshift).here;
    }
    wave_sums(sp, sl);
  }
  // the other rows, those of a wave one per lane: 16 lanes sum a short one, the wave a longer one
  for (int rb = r0 + wave; rb < r1; rb += 64 * kSpWaves) {
    const int rl = rb + kSpWaves * lane;
    int64_t from = 0;
    int len = -1;  // none, or a long row
    if (rl < r1) {
      const RowSpan sp = row_span(a.S, rl);
      from = sp.k0;
      if (sp.k1 - sp.k0 < kLong) len = (int)(sp.k1 - sp.k0);
    }
    if (len == 0)
      for (int c = 0; c < width; ++c) out[(size_t)rl * ldo + c] = 0.f;
    uint64_t todo = __ballot(len >= kShort);
    for (; todo != 0; todo &= todo - 1) {
      const int i = __builtin_ctzll(todo);
      const int64_t k0 = lane_of(from, i);
      f32x4 acc[NPER];
      row_sum<NQ, NPER, NOPS>(a, B, k0, k0 + __builtin_amdgcn_readlane(len, i), CE, lane, acc);
      if (lane < NQ) store_row<NPER>(a, out, rb + kSpWaves * i, lane, acc);
    }
    todo = __ballot(len > 0 && len < kShort);
    while (todo != 0) {
      int mine = -1;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        if (todo != 0 && (lane >> 4) == g) mine = __builtin_ctzll(todo);
        todo &= todo - 1;
      }
      const int src = mine < 0 ? 0 : mine;
      const int64_t s0 = __shfl(from, src, 64);
      const int slen = __shfl(len, src, 64);
      f32x4 acc[NPER];
      short_rows_sum<NQ, NPER, NOPS>(a, B, s0, mine < 0 ? 0 : slen, lane, acc);
      if (mine >= 0 && (lane & 15) < NQ) store_row<NPER>(a, out, rb + kSpWaves * mine, lane & 15, acc);
    }
  }
  if (nlong == 0) return;
  __syncthreads();
  for (int t = threadIdx.x; t < nlong * kPer; t += kSpThreads) {
    const int sl = t / kPer, j = t - sl * kPer;
    const int op = j / (4 * G), c = j - op * (4 * G);
    const float sum = add_waves(sl, j);
    if (c >= a.NC) continue;
    const int row = long_rows[sl];
    if constexpr (!SHARED) {
      const RowSpan sp = row_span(a.S, row);
      if (sp.k1 - sp.k0 >= kCut) continue;  // summed above
    }
    // share of a cut row: past the L2, which other XCDs do not see
    if ((into && sl == 0) || (beyond && row == r1 - 1))
      __hip_atomic_store(share + (size_t)(2 * win + (row < r0 ? 0 : 1)) * width + op * a.NC + c, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
      out[(size_t)row * ldo + op * a.NC + c] = sum;
  }
  if (!SHARED || (!into && !beyond)) return;
  int32_t* arrived = a.arrived + (size_t)blockIdx.y * a.w.n;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the shares are where every XCD reads them
  __syncthreads();
  if (threadIdx.x < 2) {
    const int row = threadIdx.x == 0 ? r0 - 1 : r1 - 1;
    int last = 0;
    if (threadIdx.x == 0 ? into : beyond) {
      const Cut c = cut_span(row_span(a.S, row), row, win, wshift);
      last = __hip_atomic_fetch_add(arrived + c.first, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == c.last - c.first;
      if (last) __hip_atomic_store(arrived + c.first, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    last_sh[threadIdx.x] = last;
  }
  __syncthreads();
  const int side = threadIdx.x >> 7, j = threadIdx.x & 127;  // width <= 64
  if (last_sh[side] != 0 && j < width) {
    const int row = side == 0 ? r0 - 1 : r1 - 1;
    const Cut c = cut_span(row_span(a.S, row), row, win, wshift);
    auto share_of = [&](int w) {
      return __hip_atomic_load(share + (size_t)(2 * w + (w == c.first ? 1 : 0)) * width + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    float sum = 0.f;
    for (int w = c.first; w <= c.last; w += 8) {
      float x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = share_of(w + u <= c.last ? w + u : c.last);
#pragma unroll
      for (int u = 0; u < 8; ++u) sum += w + u <= c.last ? x[u] : 0.f;
    }
    out[(size_t)row * ldo + j] = sum;
  }
}

template <int NQ, int NPER, int NOPS>
hipError_t launch_q(const SpmmArgs& a, hipStream_t st) {
  const dim3 grid(a.w.n, NOPS / NPER);
  if (a.arrived != nullptr) hipLaunchKernelGGL((spmm_kernel<NQ, NPER, NOPS, true>), grid, dim3(kSpThreads), 0, st, a);
  else hipLaunchKernelGGL((spmm_kernel<NQ, NPER, NOPS, false>), grid, dim3(kSpThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace

// lanes (16-byte quads) per operand row: the smallest power of two that holds C-1 floats
int sparse_group(int NC) {
  const int nq = (NC + 3) >> 2;
  return nq <= 1 ? 1 : (nq <= 2 ? 2 : (nq <= 4 ? 4 : 8));
}

// Eight workgroups for every compute unit, as many as are resident, where there is that much work: 126 windows of 4096 for half a million entries
// left half the chip idle (2000 x 2000, 250 a row, C = 3: Hessian-vector product 58 -> 37 us).
int sparse_window_shift(int64_t nrows, int64_t nnz) {
  const int64_t total = nnz + (int64_t)kRowCost * nrows;
  int s = kMaxShift;
  while (s > kMinShift && (total >> s) < 2048) --s;
  return s;
}

int sparse_windows(int64_t nrows, int64_t nnz) {
  const int64_t total = nnz + (int64_t)kRowCost * nrows;
  const int s = sparse_window_shift(nrows, nnz);
  const int64_t w = (total + ((int64_t)1 << s) - 1) >> s;
  return (int)(w < 1 ? 1 : w);
}

hipError_t launch_sparse_plan(const SparseView& S0, const SparseWindows& w0, const SparseView& S1, const SparseWindows& w1, int32_t* arrived, hipStream_t st) {
  const int b0 = (w0.n + 1 + 255) / 256, b1 = (w1.n + 1 + 255) / 256;
  hipLaunchKernelGGL(plan_kernel, dim3(b0 + b1), dim3(256), 0, st, S0, w0, S1, w1, b0, arrived);
  return hipGetLastError();
}

hipError_t launch_sparse_pack(const float* src0, const float* src1, int64_t rows, int NC, float* dst,
                              const int32_t* flag, hipStream_t st) {
  const int nops = src1 != nullptr ? 2 : 1;
  const int G = sparse_group(NC);
  const int64_t total = rows * nops * G;
  hipLaunchKernelGGL(pack_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, src0, src1, rows, NC, G,
                     nops, dst, flag);
  return hipGetLastError();
}

hipError_t launch_spmm(const SpmmArgs& a, hipStream_t st) {
  // two operands in one pass only where both rows share a 128-byte line (C-1 <= 16): for wider ones two passes over the entries, which fetch a line
  // per entry, take 2 x 620 us where one pass that fetches two takes 1523 (40628 x 279998, C = 20)
  if (a.nq != (a.NC + 3) / 4 || a.nq < 1 || a.nq > 8 || a.nops < 1 || a.nops > 2) return hipErrorInvalidValue;
  switch (a.nq * 2 + (a.nops - 1)) {
    case 2: return launch_q<1, 1, 1>(a, st);
    case 3: return launch_q<1, 2, 2>(a, st);
    case 4: return launch_q<2, 1, 1>(a, st);
    case 5: return launch_q<2, 2, 2>(a, st);
    case 6: return launch_q<3, 1, 1>(a, st);
    case 7: return launch_q<3, 2, 2>(a, st);
    case 8: return launch_q<4, 1, 1>(a, st);
    case 9: return launch_q<4, 2, 2>(a, st);
    case 10: return launch_q<5, 1, 1>(a, st);
    case 11: return launch_q<5, 1, 2>(a, st);
    case 12: return launch_q<6, 1, 1>(a, st);
    case 13: return launch_q<6, 1, 2>(a, st);
    case 14: return launch_q<7, 1, 1>(a, st);
    case 15: return launch_q<7, 1, 2>(a, st);
    case 16: return launch_q<8, 1, 1>(a, st);
    case 17: return launch_q<8, 1, 2>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace nadmm
