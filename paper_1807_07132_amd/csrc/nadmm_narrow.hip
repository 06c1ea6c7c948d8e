// Matrix-core kernel for narrow rows (gfx950): p <= 128 with C-1 <= 16, p <= 96 with up to 32 free classes; any row stride.
//
// The fused kernel splits the columns of a tile over the 8 waves of a workgroup in steps of 32: with 70 columns three waves
// work and five wait at the barriers (100000 x 70, C = 7: 19.7 us per sweep of 28 MB).  Here a wave owns whole rows: it
// takes tiles of 16 rows with all their columns, its operands and accumulators are the whole of X, V and A^T D, and nothing
// is exchanged between waves until the end of the kernel -- no barrier in the loop.  A lane's logits are those of four
// rows and one class, which is also the layout in which the second product takes D: no exchange of D either.
// What bounds it: the stream of A where there are many rows (Hessian-vector product at 700000 x 120, C = 10: 127 -> 86 us, 3.9 TB/s
// over the call; 581012 x 54, C = 7: 111 -> 49 us), the rows stage where few of the 16 class lanes are used, the chain of one
// tile on few rows.  RT tiles are in flight per wave, so that narrow rows keep as many bytes on their way as wider ones.
// More than 16 free classes took two sweeps, unaligned rows below 48 columns the vector kernels: 1000000 x 33, C = 22,
// objective and gradient: 747 -> 110 us; 500000 x 84, C = 29: 196 -> 67 us.
// Arithmetic: every operand is split into three bf16 parts (the whole float32 significand) and each product takes the six
// terms of weight >= 2^-16, for A X, A V and A^T D alike: as accurate as float32 products, which is what narrow rows that are
// not 16-byte aligned had from the vector kernels.
#include "nadmm_internal.h"
#include "nadmm_cgstep.h"
#include "nadmm_mfma.h"

namespace nadmm {
namespace {

using namespace mfma_detail;

constexpr int kThreads = 256;
constexpr int kWaves = 4;
constexpr int kStepCols = 32;
constexpr int kSlotBytes = 3072;  // one step of a tile of 16 rows: high, middle and low part

struct NarrowArgs {
  RowArgs r;
  float* partial;       // gridDim.x x (p*NC), or NULL (no transpose product)
  int32_t rounds, more; // rounds of a workgroup (a tile for each of its waves); the first `more` workgroups make one more
  CgPend cg;            // cg.st != NULL: the operand B1 is the result of a pending CG update (kernels without B0 only)
};

// bytes of LDS: the waves' tiles, and at the end their accumulators side by side
__host__ __device__ constexpr int wave_lds_bytes(int S, int RT, int NB) {
  const int tiles = S * RT * kSlotBytes, accs = S * kStepCols * NB * 16 * 4;
  return tiles > accs ? tiles : accs;
}

template <int S, int RT, int NB, int KIND, bool HAS0, bool HAS1, bool STORES, bool ANY>
__global__ __launch_bounds__(kThreads, 2) void narrow_kernel(const NarrowArgs na) {
  const RowArgs& a = na.r;
  if (a.flag != nullptr && *a.flag == 0) return;
  constexpr bool with_cols = KIND == kRowsHv || KIND == kRowsGrad;
  constexpr int kWaveLds = wave_lds_bytes(S, RT, NB);
  constexpr int kTile = 16 * RT;             // rows of a wave's round
  __shared__ __attribute__((aligned(16))) char lds[kWaves * kWaveLds];
  __shared__ double red[2 * kWaves];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = lane & 15, kg = lane >> 4;
  const int NC = a.NC, p = a.p;
  char* slots = lds + wave * kWaveLds;
  const int col_max = ANY ? p - 4 : ((p + 3) & ~3) - 4;  // the last column a 16-byte piece is fetched from

  const int wg = blockIdx.x;
  const int64_t r_begin = ((int64_t)wg * na.rounds + (wg < na.more ? wg : na.more)) * (kWaves * kTile);
  int64_t r_end = r_begin + (int64_t)(na.rounds + (wg < na.more ? 1 : 0)) * (kWaves * kTile);
  if (r_end > a.n) r_end = a.n;

  // ---- rows of A, RT tiles of 16; a step's columns lie in the k-slots as two pieces of four, so that the four lanes of a
  //      row fetch 64 consecutive bytes ----
  float4 pf[RT][S][2];
  auto load_tile = [&](int64_t row0) {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      int64_t row = row0 + 16 * t + m;
      row = row < r_end ? row : r_end - 1;
      const float* src = a.A + row * a.lda;
#pragma unroll
      for (int i = 0; i < S; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int c0 = kStepCols * i + 16 * h + 4 * kg;
          const float* at = src + ((i < S - 1 || c0 < col_max) ? c0 : col_max);  // all but the last step are whole
          if constexpr (ANY) {
            const Quad q = *reinterpret_cast<const Quad*>(at);
            pf[t][i][h] = float4{q.x, q.y, q.z, q.w};
          } else {
            pf[t][i][h] = *reinterpret_cast<const float4*>(at);
          }
        }
    }
  };
  const int64_t first = r_begin + (int64_t)wave * kTile;
  auto load_first = [&]() { load_tile(first < r_end ? first : r_begin); };

  // ---- operands: lane (class 16 nb + m, k-group kg); padded classes and columns past p read some other entry and only ever
  //      meet zeros (D = 0, the tile's columns past p are zeroed) ----
  bool cv[NB];
  int cl[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    cv[nb] = 16 * nb + m < NC;
    cl[nb] = cv[nb] ? 16 * nb + m : NC - 1;
  }
  // The waves share the work of gathering and splitting: unit u (operand, step, class block) is prepared by wave u mod 4 and
  // handed to the others through LDS.  (Every wave for itself took 32 gathers per step count of 4 and operand: a launch on few
  // rows spent most of its time there.)
  constexpr int kOps = (HAS0 ? 1 : 0) + (HAS1 ? 1 : 0), kUnits = kOps * S * NB, kPerWave = (kUnits + kWaves - 1) / kWaves;
  constexpr int kVecBytes = (!HAS0 && HAS1 && NB == 1) ? S * kStepCols * 16 * 4 : 0;  // room for the vector of a deferred update
  static_assert(kVecBytes + kUnits * 3072 <= kWaves * kWaveLds, "operands fit the tiles' LDS");
  u32x4 bx[HAS0 ? S : 1][NB][3], bv[HAS1 ? S : 1][NB][3];
  bool deferred = false;
  if constexpr (!HAS0 && HAS1 && NB == 1) {
    deferred = na.cg.st != nullptr;
    static_assert(S * kStepCols * 16 <= 2 * 4 * kThreads, "the longest vector of this kernel fits the update's registers");
    if (deferred && !cg_pending_update<kThreads, 2>(na.cg, blockIdx.x == 0, reinterpret_cast<float*>(lds), red, load_first)) return;
  }
  {
    float raw[kPerWave][8];
#pragma unroll
    for (int k = 0; k < kPerWave; ++k) {
      const int u = wave + kWaves * k < kUnits ? wave + kWaves * k : kUnits - 1;  // uniform
      const int nb = u % NB, i = (u / NB) % S;
      const float* src = (HAS0 && u < S * NB) ? a.B0 : a.B1;
      const int clu = (NB == 2 && nb == 1) ? cl[NB - 1] : cl[0];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int j = kStepCols * i + 16 * (e >> 2) + 4 * kg + (e & 3);
        const int at = (j < p ? j : p - 1) * NC + clu;
        raw[k][e] = deferred ? reinterpret_cast<const float*>(lds)[at] : src[at];
      }
    }
    if (!deferred) load_first();  // behind the operands: loads return in order
#pragma unroll
    for (int k = 0; k < kPerWave; ++k) {
      const int u = wave + kWaves * k;
      u32x4 q[3];
      split8_3(raw[k], q[0], q[1], q[2]);
      if (u < kUnits) {
#pragma unroll
        for (int t = 0; t < 3; ++t) *reinterpret_cast<u32x4*>(lds + kVecBytes + u * 3072 + t * 1024 + lane * 16) = q[t];
      }
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          if (HAS0) bx[HAS0 ? i : 0][nb][t] = *reinterpret_cast<const u32x4*>(lds + kVecBytes + (i * NB + nb) * 3072 + t * 1024 + lane * 16);
          if (HAS1)
            bv[HAS1 ? i : 0][nb][t] = *reinterpret_cast<const u32x4*>(lds + kVecBytes + ((kOps - 1) * S * NB + i * NB + nb) * 3072 + t * 1024 + lane * 16);
        }
    lds_barrier();  // every wave has its operands: the tiles may overwrite them
  }

  f32x4 acc[S][2][NB];
#pragma unroll
  for (int i = 0; i < S; ++i)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[i][h][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  double loss_acc = 0.0;

  // tile in LDS: blocks of 16 rows x 16 columns (512 bytes; part, column half), written and read back to back
  const int wr_off = m * 32 + kg * 8;
  const int rd_off = (4 * kg + (m >> 2)) * 32 + (m & 3) * 8;

  for (int64_t row0 = first; row0 < r_end; row0 += kWaves * kTile) {
    // cached probabilities or labels: rows row0 + 16 t + 4 kg + e
    const int left = r_end - row0 < kTile ? (int)(r_end - row0) : kTile;
    float pin[RT][NB][4];
    int label[RT][4];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 16 * t + 4 * kg + e < left ? 16 * t + 4 * kg + e : left - 1;
        if (KIND == kRowsHv && !HAS0) {
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) pin[t][nb][e] = (a.Pin + row0 * NC)[(unsigned)(r * NC + cl[nb])];
        }
        if (KIND == kRowsGrad || KIND == kRowsLoss) label[t][e] = (a.labels + row0)[(unsigned)r];
      }

    // ---------------- logits; the tile goes to LDS as it is converted ----------------
    f32x4 accZ[RT][NB], accW[RT][NB];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) accZ[t][nb] = accW[t][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int i = 0; i < S; ++i) {
        float av[8] = {pf[t][i][0].x, pf[t][i][0].y, pf[t][i][0].z, pf[t][i][0].w,
                       pf[t][i][1].x, pf[t][i][1].y, pf[t][i][1].z, pf[t][i][1].w};
        if (i == S - 1 && kStepCols * S > p) {  // uniform: zero what lies past column p
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int c0 = kStepCols * i + 16 * h + 4 * kg;
            if constexpr (ANY) {
              const int shift = c0 - (c0 < col_max ? c0 : col_max);  // 0: the piece is its own; >= 4: all of it is past p
              const float q0 = av[4 * h], q1 = av[4 * h + 1], q2 = av[4 * h + 2], q3 = av[4 * h + 3];
              av[4 * h + 0] = shift == 0 ? q0 : (shift == 1 ? q1 : (shift == 2 ? q2 : (shift == 3 ? q3 : 0.f)));
              av[4 * h + 1] = shift == 0 ? q1 : (shift == 1 ? q2 : (shift == 2 ? q3 : 0.f));
              av[4 * h + 2] = shift == 0 ? q2 : (shift == 1 ? q3 : 0.f);
              av[4 * h + 3] = shift == 0 ? q3 : 0.f;
            } else {
              const int nv = c0 <= col_max ? p - c0 : 0;
#pragma unroll
              for (int e = 0; e < 4; ++e) av[4 * h + e] = e < nv ? av[4 * h + e] : 0.f;
            }
          }
        }
        u32x4 ap[3];
        split8_3(av, ap[0], ap[1], ap[2]);
        // smallest terms first (see mfma6), Z and W and the class blocks taking turns
        constexpr int ta[6] = {2, 0, 1, 1, 0, 0}, tb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int k = 0; k < 6; ++k)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            if (HAS0) accZ[t][nb] = mfma(ap[ta[k]], bx[HAS0 ? i : 0][nb][tb[k]], accZ[t][nb]);
            if (HAS1) accW[t][nb] = mfma(ap[ta[k]], bv[HAS1 ? i : 0][nb][tb[k]], accW[t][nb]);
          }
        if (with_cols) {
          char* base = slots + (t * S + i) * kSlotBytes + wr_off;
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            *reinterpret_cast<u32x2*>(base + 1024 * k) = u32x2{ap[k][0], ap[k][1]};
            *reinterpret_cast<u32x2*>(base + 1024 * k + 512) = u32x2{ap[k][2], ap[k][3]};
          }
        }
      }
    __builtin_amdgcn_sched_barrier(0);
    load_tile(row0 + kWaves * kTile);  // past the range: its last row again
    __builtin_amdgcn_sched_barrier(0);

#pragma unroll
    for (int t = 0; t < RT; ++t) {
      // ---------------- rows: lane (m, kg) holds rows row0 + 16 t + 4 kg + e, classes 16 nb + m ----------------
      float d[NB][4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 16 * t + 4 * kg + e;
        const bool valid = r < left;
        float P[NB];
        if (KIND != kRowsLogits) {
          float M = 0.f, alpha = 1.f;
          if (HAS0) {
            float mx = 0.f;  // the reference class has logit 0
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) mx = fmaxf(mx, cv[nb] ? accZ[t][nb][e] : 0.f);
            M = row16_max(mx);
            float es = 0.f;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
              P[nb] = cv[nb] ? expf(accZ[t][nb][e] - M) : 0.f;
              es += P[nb];
            }
            alpha = row16_sum(es) + expf(-M);
            const float inv = 1.f / alpha;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) P[nb] *= inv;
          } else {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) P[nb] = cv[nb] ? pin[t][nb][e] : 0.f;
          }
          if (KIND == kRowsHv) {
            float s = 0.f;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) s = fmaf(P[nb], cv[nb] ? accW[t][nb][e] : 0.f, s);
            s = row16_sum(s);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) d[nb][e] = (valid && cv[nb]) ? P[nb] * (accW[t][nb][e] - s) : 0.f;
          } else {
            float zb = 0.f;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
              const bool mine = cv[nb] && 16 * nb + m == label[t][e];
              zb += mine ? accZ[t][nb][e] : 0.f;
              d[nb][e] = (valid && cv[nb]) ? P[nb] - (mine ? 1.f : 0.f) : 0.f;
            }
            zb = row16_sum(zb);
            if (valid && m == 0) loss_acc += (double)M + (double)logf(alpha) - (double)zb;
          }
        }
        if (STORES && valid) {
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            if (cv[nb]) {
              const unsigned at = (unsigned)(r * NC + cl[nb]);
              if (KIND != kRowsLogits && a.Pout) (a.Pout + row0 * NC)[at] = P[nb];
              if (HAS0 && a.Z0out) (a.Z0out + row0 * NC)[at] = accZ[t][nb][e];
              if (HAS1 && (KIND == kRowsLogits || KIND == kRowsHv) && a.Z1out) (a.Z1out + row0 * NC)[at] = accW[t][nb][e];
            }
        }
      }
      if (!with_cols) continue;
      // ---------------- out^T += D^T tile: the six terms in three instructions, two parts of the same 16 rows each ----------------
      u32x4 dhh[NB], dmm[NB], dhl[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        unsigned h[2], mm[2], l[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const float d0 = d[nb][2 * k], d1 = d[nb][2 * k + 1];
          h[k] = pack2(d0, d1);
          const float r0 = d0 - low_as_float(h[k]), r1 = d1 - high_as_float(h[k]);
          mm[k] = pack2(r0, r1);
          l[k] = pack2(r0 - low_as_float(mm[k]), r1 - high_as_float(mm[k]));
        }
        dhh[nb] = u32x4{h[0], h[1], h[0], h[1]};
        dmm[nb] = u32x4{mm[0], mm[1], mm[0], mm[1]};
        dhl[nb] = u32x4{h[0], h[1], l[0], l[1]};
      }
#pragma unroll
      for (int i = 0; i < S; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          char* base = slots + (t * S + i) * kSlotBytes + 512 * h + rd_off;
          const u32x2 th = read_transposed(base), tm = read_transposed(base + 1024), tl = read_transposed(base + 2048);
          const u32x4 hm = u32x4{th[0], th[1], tm[0], tm[1]}, lh = u32x4{tl[0], tl[1], th[0], th[1]};
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            acc[i][h][nb] = mfma(dhl[nb], lh, acc[i][h][nb]);
            acc[i][h][nb] = mfma(dmm[nb], hm, acc[i][h][nb]);
            acc[i][h][nb] = mfma(dhh[nb], hm, acc[i][h][nb]);
          }
        }
    }
  }

  // ---- the workgroup's partial: the waves' accumulators side by side in LDS in the order of the result, added in wave order ----
  if (with_cols) {
    float* mine = reinterpret_cast<float*>(slots);
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int j = kStepCols * i + 16 * h + m, c = 16 * nb + 4 * kg + e;
            if (j < p && c < NC) mine[j * NC + c] = acc[i][h][nb][e];
          }
    __syncthreads();
    float* out = na.partial + (size_t)blockIdx.x * ((size_t)p * NC);
    const float* all = reinterpret_cast<const float*>(lds);
    constexpr int stride = kWaveLds / 4;
    for (int q = threadIdx.x; q < p * NC; q += kThreads)
      out[q] = ((all[q] + all[stride + q]) + all[2 * stride + q]) + all[3 * stride + q];
  }
  if (KIND == kRowsGrad || KIND == kRowsLoss) {
    loss_acc = wave64_sum(loss_acc);
    if (lane == 0) red[wave] = loss_acc;
    __syncthreads();
    if (threadIdx.x == 0) a.loss_part[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
  }
}

int steps_of(int p) { return (p + kStepCols - 1) / kStepCols; }
constexpr int tiles_of(int steps, int nb) { return steps == 1 ? 4 / nb : (steps == 2 ? 2 / nb : 1); }  // RT: what the registers hold

bool rows_16_byte_aligned(const RowArgs& a) { return (a.lda & 3) == 0 && (reinterpret_cast<uintptr_t>(a.A) & 15) == 0; }

template <int S, int NB, int KIND, bool HAS0, bool HAS1, bool STORES>
hipError_t launch_s(const NarrowArgs& na, int grid, hipStream_t st) {
  constexpr int RT = tiles_of(S, NB);
  if (rows_16_byte_aligned(na.r))
    hipLaunchKernelGGL((narrow_kernel<S, RT, NB, KIND, HAS0, HAS1, STORES, false>), dim3(grid), dim3(kThreads), 0, st, na);
  else
    hipLaunchKernelGGL((narrow_kernel<S, RT, NB, KIND, HAS0, HAS1, STORES, true>), dim3(grid), dim3(kThreads), 0, st, na);
  return hipGetLastError();
}

template <int S, int NB>
hipError_t launch_steps(const NarrowArgs& na, int grid, hipStream_t st) {
  const RowArgs& a = na.r;
  const bool h0 = a.B0 != nullptr, h1 = a.B1 != nullptr;
  const bool stores = a.Pout != nullptr || a.Z0out != nullptr || a.Z1out != nullptr;
  switch (a.kind) {
    case kRowsHv:
      if (na.partial == nullptr || !h1) return hipErrorInvalidValue;
      if constexpr (NB == 1 || S <= 2) {
        if (h0) return stores ? launch_s<S, NB, kRowsHv, true, true, true>(na, grid, st) : launch_s<S, NB, kRowsHv, true, true, false>(na, grid, st);
      }
      if (h0 || a.Pin == nullptr) return hipErrorInvalidValue;
      return stores ? launch_s<S, NB, kRowsHv, false, true, true>(na, grid, st) : launch_s<S, NB, kRowsHv, false, true, false>(na, grid, st);
    case kRowsGrad:
      if (na.partial == nullptr || !h0 || h1 || a.labels == nullptr || a.loss_part == nullptr) return hipErrorInvalidValue;
      return stores ? launch_s<S, NB, kRowsGrad, true, false, true>(na, grid, st) : launch_s<S, NB, kRowsGrad, true, false, false>(na, grid, st);
    case kRowsLoss:
      if (!h0 || h1 || a.labels == nullptr || a.loss_part == nullptr) return hipErrorInvalidValue;
      return launch_s<S, NB, kRowsLoss, true, false, false>(na, grid, st);
    case kRowsLogits:
      if constexpr (NB == 1 || S <= 2) {
        if (h0 && h1) return launch_s<S, NB, kRowsLogits, true, true, true>(na, grid, st);
      }
      if (h1 && !h0) return launch_s<S, NB, kRowsLogits, false, true, true>(na, grid, st);
      if (h0 && !h1) return launch_s<S, NB, kRowsLogits, true, false, true>(na, grid, st);
      return hipErrorInvalidValue;
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace

bool narrow_supported(const Shape& s, int64_t lda, const void* A) {
  if (s.p < 4 || s.p > (s.NC > 16 ? 96 : 128) || s.NC > 32) return false;  // whole 16-byte pieces inside a row
  return (reinterpret_cast<uintptr_t>(A) & 3) == 0 && lda >= s.p;
}

// A wave needs a tile or more of its own; below that the fused kernel, which spreads a tile over 8 waves, has the shorter
// chain: a wave's grows with its steps.  Measured at C = 10, fused against this kernel (us), Hessian-vector product / 10 CG
// iterations: p = 64: 33000 rows 13.6 : 14.1 / 113 : 114, 50000 rows 14.2 : 13.0 / 125 : 117, 100000 rows 20.5 : 17.0 / 174 : 144;
// p = 96: 33000 rows 12.8 : 13.6 / 115 : 119, 50000 rows 15.0 : 14.4 / 135 : 128, 100000 rows 21.9 : 19.3 / 192 : 158;
// p = 112: 50000 rows 15.4 : 16.0 / 137 : 139, 57600 rows 16.6 : 16.1 / 145 : 141, 70000 rows 17.9 : 18.3 / 157 : 154, 100000 rows
// 22.6 : 21.9 / 198 : 178.  Unaligned rows slow the fused kernel down: p = 97: 50000 rows 17.6 : 16.7, 8 iterations 148 : 145.
// The line for more than 96 columns is not moved up to where the times cross: three terms against six of A V and A^T D, errors of
// 5.1e-7 against 5.0e-8 at 55541 x 124, C = 10.
int64_t narrow_min_rows(int32_t p) { return steps_of(p) <= 2 ? 32768 : 49152; }

// Two blocks of classes: X and V together fit the registers up to two steps only (else two sweeps).
bool narrow_takes(const Shape& s, bool has_x, bool has_v) { return s.NC <= 16 || s.p <= 2 * kStepCols || !(has_x && has_v); }

// Workgroups: two per compute unit, each with equally many rounds of its waves as far as that goes with fewer of them; with 3 to 8
// rounds each, 512 of which some make a round less, since then the compute units that had a single one count: 100000 x 70, C = 7,
// Hessian-vector product 18.9 -> 16.9 us, 10 CG iterations 184 -> 172 us (391 workgroups of 4 rounds before); 150000 x 64, C = 7:
// 19.8 -> 17.2 us.  With 2 rounds the larger number of partial sums costs what it gains (50000 x 70: 14.7 : 14.9), beyond 8 equal.
// With two blocks of classes the same (72 shapes of 3 to 8 rounds: gradient, product and 4 CG iterations 0.86 to 1.01 of the time with
// equal rounds): 137625 x 16, C = 20, product 19.8 -> 17.4 us, gradient 21.8 -> 18.8; 101580 x 84, C = 29, gradient 24.8 -> 22.8, 4 CG
// iterations 137 -> 132; 232652 x 64, C = 22, product 31.3 -> 29.3.
int narrow_num_partials(const Shape& s) {
  const int64_t round = (int64_t)kWaves * 16 * tiles_of(steps_of(s.p), s.NC > 16 ? 2 : 1);
  const int64_t rounds = (s.n + round - 1) / round;
  const int64_t g = rounds < 512 ? rounds : 512;
  const int64_t per = (rounds + g - 1) / g;
  if (per >= 3 && per <= 8) return 512;
  return (int)((rounds + per - 1) / per);
}

hipError_t launch_narrow(const RowArgs& a, float* partial, int nparts, hipStream_t st, const CgPend* cg) {
  NarrowArgs na;
  na.r = a;
  na.partial = partial;
  if (cg != nullptr) {  // only kernels with one block of classes, without X and with V apply a pending update
    if (a.NC > 16 || a.B0 != nullptr || a.B1 == nullptr || (a.kind != kRowsHv && a.kind != kRowsLogits)) return hipErrorInvalidValue;
    if (cg->st == nullptr || cg->ndot < 1 || cg->ndot > kThreads || cg->dlen != (int64_t)a.p * a.NC) return hipErrorInvalidValue;
    na.cg = *cg;
  } else {
    na.cg = CgPend{};
  }
  const int steps = steps_of(a.p);
  const int64_t round = (int64_t)kWaves * 16 * tiles_of(steps, a.NC > 16 ? 2 : 1);
  const int64_t rounds = (a.n + round - 1) / round;
  na.rounds = (int32_t)(rounds / nparts);
  na.more = (int32_t)(rounds % nparts);
  if (a.NC <= 16) {
    switch (steps) {
      case 1: return launch_steps<1, 1>(na, nparts, st);
      case 2: return launch_steps<2, 1>(na, nparts, st);
      case 3: return launch_steps<3, 1>(na, nparts, st);
      case 4: return launch_steps<4, 1>(na, nparts, st);
      default: return hipErrorInvalidValue;
    }
  }
  switch (steps) {
    case 1: return launch_steps<1, 2>(na, nparts, st);
    case 2: return launch_steps<2, 2>(na, nparts, st);
    case 3: return launch_steps<3, 2>(na, nparts, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace nadmm
