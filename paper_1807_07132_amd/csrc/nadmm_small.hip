// A whole CG solve or a whole local Newton solve of a small thin problem in one kernel (gfx950): n <= 2048 rows of up to 32
// columns and up to 3 free classes.
//
// Such a solve is bound by launches: at 1000 x 20, C = 3 a CG iteration as a launch of its own takes 7.4 us for less than 1 us of
// work, and the gradient, the head, the line search's two kernels and the state's initialisation 27 us per Newton iteration.
// Here one workgroup keeps its rows of A (up to four per thread), their logits and probabilities in registers for the whole
// solve.  Vectors of at most 64 elements lie one element per lane, in every wave the same: a pass over the rows leaves the sums of
// every wave in LDS, and after one barrier each wave adds them up and makes the update (Section 2.4) for itself, so that a CG
// iteration has a single barrier and the direction reaches the products as scalar registers.  The line search (Algorithm 2)
// evaluates its candidates one after the other from the logits in registers and stops at the first that is taken.
// What bounds it: the serial chain of an iteration (row products, the sum over lanes and waves, the inner products in float64).
// Measured: 1.9 us per CG iteration at 1000 x 20, C = 3 (3.3 us with two barriers per iteration and sums of 16 lanes by rotations);
// a Newton iteration with 10 CG iterations there 62 -> 29 us (CG alone in one launch before), 10 CG iterations 41 -> 25 us.
// float32 products and sums over rows, float64 inner products and objectives; every sum in a fixed order.
#include <cstring>

#include "nadmm_internal.h"
#include "nadmm_mfma.h"

namespace nadmm {
namespace {

using mfma_detail::wave64_sum;
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kRowsPerThread = 4;

// floats per row of the staging tile: off the bank period where rows lie in whole quads
constexpr int small_stride(int pp) { return pp % 8 == 0 ? pp + 4 : pp; }

__device__ __forceinline__ float lane_f(float v, int lane) {  // lane: a constant
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

template <int NQ, int NC, int THREADS, int R>
__global__ __launch_bounds__(THREADS) void small_solve_kernel(const SmallSolve c) {
  constexpr int PP = 4 * NQ, D = PP * NC;          // padded columns, vector length with them (<= 64)
  constexpr int W = THREADS / 64;
  constexpr int DEPTH = THREADS <= 256 || R < 4 ? R : 2;  // chunks of rows in flight while they are staged
  if (c.outer_flag != nullptr && *c.outer_flag == 0) {  // the outer iteration has stopped: the solve is not made
    if (c.newton && threadIdx.x == 0) {
      c.st->newton_even = 0;
      c.st->cg_active = 0;
    }
    return;
  }
  extern __shared__ __attribute__((aligned(16))) float tile[];  // staging of THREADS rows, then the waves' partial sums
  __shared__ float wsum[2][W][D];     // sums of a wave, two passes in turn
  __shared__ double red[2][W];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int p = c.p, n = (int)c.n, dlen = p * NC, ld = (int)c.lda;
  DevState* st = c.st;
  const bool newton = c.newton != 0;

  // one element of the vectors per lane, element lane = j NC + class
  const int le = lane < dlen ? lane : dlen - 1;
  const bool own = lane < dlen;
  float xv = 0.f, zv = 0.f, yv = 0.f, g = 0.f;
  {
    const float x_in = c.X[le], z_in = c.z != nullptr ? c.z[le] : 0.f, y_in = c.y != nullptr ? c.y[le] : 0.f;
    const float g_in = newton ? 0.f : c.g[le];
    xv = own ? x_in : 0.f;
    zv = own ? z_in : 0.f;
    yv = own ? y_in : 0.f;
    g = own ? g_in : 0.f;
  }
  const float rho_ = c.rho_scale != nullptr ? c.rho * *c.rho_scale : c.rho;
  int lab[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int row = t + k * THREADS;
    lab[k] = newton ? c.labels[row < n ? row : n - 1] : 0;
  }

  // ---- rows t, t + THREADS, ... into registers, zeros past the end and past column p: fetched as one block of memory, in
  // 16-byte pieces where rows are whole quads (stride 4 NQ, aligned), else element by element, and dealt out through LDS ----
  float a[R][PP];
  const int nchunks = (n + THREADS - 1) / THREADS;  // <= R
  auto take_row = [&](int k, const float* src) {
    const bool valid = t + k * THREADS < n;
#pragma unroll
    for (int j = 0; j < PP; ++j) {
      const float v = src[j];
      a[k][j] = valid && (j < PP - 4 || j < p) ? v : 0.f;  // p > PP - 4
    }
  };
  if (c.quads != 0) {
    constexpr int PS = small_stride(PP);
    const f32x4* A4 = reinterpret_cast<const f32x4*>(c.A);
    const int last4 = n * NQ - 1;
    f32x4 pf[DEPTH][NQ];
    auto fetch = [&](int b, int k) {
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        const int i4 = k * THREADS * NQ + t + i * THREADS;
        pf[b][i] = A4[i4 < last4 ? i4 : last4];
      }
    };
#pragma unroll
    for (int k = 0; k < DEPTH; ++k) fetch(k, k);
#pragma unroll
    for (int k = 0; k < R; ++k) {
      if (k < nchunks) {  // uniform
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
          const int e = 4 * (t + i * THREADS);
          *reinterpret_cast<f32x4*>(&tile[(e / PP) * PS + e % PP]) = pf[k % DEPTH][i];
        }
        if (k + DEPTH < R) fetch(k % DEPTH, k + DEPTH);
        __syncthreads();
        take_row(k, &tile[t * PS]);
      } else {
#pragma unroll
        for (int j = 0; j < PP; ++j) a[k][j] = 0.f;
      }
    }
  } else {
    const int last = (n - 1) * ld + p - 1;
#pragma unroll
    for (int k = 0; k < R; ++k) {
      if (k < nchunks) {  // uniform
        float pf[PP];
#pragma unroll
        for (int i = 0; i < PP; ++i) {
          const int e = k * THREADS * ld + t + i * THREADS;  // i < ld: the chunk; beyond, never stored
          pf[i] = c.A[e < last ? e : last];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PP; ++i)
          if (i < ld) tile[t + i * THREADS] = pf[i];  // < THREADS ld
        __syncthreads();
        take_row(k, &tile[t * ld]);  // at most (THREADS - 1) ld + PP - 1 < THREADS PP
      } else {
#pragma unroll
        for (int j = 0; j < PP; ++j) a[k][j] = 0.f;
      }
    }
  }
  __syncthreads();  // the tile becomes the waves' partial sums

  // A v for the vector whose elements the lanes hold
  auto products = [&](float v, float (&w)[R][NC]) {
#pragma unroll
    for (int k = 0; k < R; ++k)
#pragma unroll
      for (int q = 0; q < NC; ++q) w[k][q] = 0.f;
#pragma unroll
    for (int j = 0; j < PP; ++j)
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const float s = lane_f(v, j * NC + q);
#pragma unroll
        for (int k = 0; k < R; ++k) w[k][q] = fmaf(a[k][j], s, w[k][q]);
      }
  };
  // A^T d, element lane of it, in every wave: sums of four lanes by rotations, of a wave through its part of the tile, of the
  // waves after the barrier.  `par` alternates: a wave is at most one barrier ahead of another.
  int par = 0;
  constexpr int kPart = D + 4;
  float* mine = tile + wave * 16 * kPart;  // 16 partial sums per element and wave (16 (D + 4) floats <= 64 rows of the tile, D >= 4)
  auto col_sums = [&](const float (&dk)[R][NC]) -> float {
    constexpr int B = 8;  // quads written together: what lies between is registers
#pragma unroll
    for (int v0 = 0; v0 < D / 4; v0 += B) {
      f32x4 s4[B];
#pragma unroll
      for (int v = v0; v < v0 + B && v < D / 4; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int j = (4 * v + e) / NC, q = (4 * v + e) % NC;
          float s = a[0][j] * dk[0][q];
#pragma unroll
          for (int k = 1; k < R; ++k) s = fmaf(a[k][j], dk[k][q], s);
          s += mfma_detail::row_ror<8>(s);
          s += mfma_detail::row_ror<4>(s);
          s4[v - v0][e] = s;
        }
      if ((lane & 15) < 4) {
        f32x4* at = reinterpret_cast<f32x4*>(mine + ((lane >> 4) * 4 + (lane & 3)) * kPart);
#pragma unroll
        for (int v = v0; v < v0 + B && v < D / 4; ++v) at[v] = s4[v - v0];
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    const int ld_ = lane < D ? lane : D - 1;
    float u[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 16; ++k) u[k & 3] += mine[k * kPart + ld_];
    if (lane < D) wsum[par][wave][lane] = (u[0] + u[1]) + (u[2] + u[3]);
    __syncthreads();
    float s = wsum[par][0][ld_];
#pragma unroll
    for (int w = 1; w < W; ++w) s += wsum[par][w][ld_];
    par ^= 1;
    return s;
  };
  // sum of a double over the workgroup, in every thread
  int dpar = 0;
  auto block_sum = [&](double v) -> double {
    v = wave64_sum(v);
    if (lane == 0) red[dpar][wave] = v;
    __syncthreads();
    double s = red[dpar][0];
#pragma unroll
    for (int w = 1; w < W; ++w) s += red[dpar][w];
    dpar ^= 1;
    return s;
  };

  float z[R][NC], P[R][NC], dk[R][NC];
  const int max_newton = newton ? c.max_newton : 1;
  double loss = 0.0, gg = 0.0, rr = 0.0, loss_new = 0.0, loss_initial = 0.0;
  float pv = 0.f, r = 0.f, alpha = 0.f;
  int iters = 0, active = 1, ok = 1, evals = 0, newton_active = 1;
  // statistics, kept by thread 0
  int s_newton = 0, s_cg = 0, s_ls = 0, s_failed = 0;
  double s_loss_final = 0.0, s_gn = 0.0;
  if (newton)
    for (int i = t; i < NADMM_TRACE_LEN; i += THREADS) {
      st->stats.alpha[i] = 0.f; st->stats.cg_iters[i] = 0; st->stats.loss[i] = 0.0; st->stats.grad_norm[i] = 0.0;
    }

  for (int nt = 0; nt < max_newton; ++nt) {
    // ---- logits, probabilities (log-sum-exp shift, Section 2.2), row losses, rows of P - Y ----
    products(xv, z);
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const bool valid = t + k * THREADS < n;
      float M = 0.f, zb = 0.f;
#pragma unroll
      for (int q = 0; q < NC; ++q) M = fmaxf(M, z[k][q]);
      float al = expf(-M);
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        P[k][q] = expf(z[k][q] - M);
        al += P[k][q];
      }
      const float inv = 1.f / al;
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        P[k][q] = valid ? P[k][q] * inv : 0.f;
        if (q == lab[k]) zb = z[k][q];
        dk[k][q] = valid ? P[k][q] - (q == lab[k] ? 1.f : 0.f) : 0.f;
      }
      if (valid) acc += (double)M + (double)logf(al) - (double)zb;
    }
    if (newton) {
      // ---- gradient, objective, stopping test of Algorithm 3 ----
      const float s = col_sums(dk);
      g = own ? c.scale * s + (c.lambda * xv + rho_ * (xv - zv) + yv) : 0.f;
      const double data = block_sum(acc);
      const double u = (double)xv - (double)zv + (double)yv / (double)rho_;
      const double pen = wave64_sum(own ? 0.5 * (double)c.lambda * (double)xv * (double)xv + 0.5 * (double)rho_ * u * u : 0.0);
      gg = wave64_sum((double)g * (double)g);
      loss = (double)c.scale * data + pen;
      rr = gg;
      iters = 0;
      active = gg > 0.0 ? 1 : 0;
      const double gn = sqrt(gg);
      s_gn = gn;
      if (nt == 0) {
        loss_initial = loss;
        s_loss_final = loss;
      }
      if (gn < (double)c.grad_tol || !(gg > 0.0)) {
        newton_active = 0;
        active = 0;
        break;
      }
      if (t == 0 && nt < NADMM_TRACE_LEN) {
        st->stats.loss[nt] = loss;
        st->stats.grad_norm[nt] = gn;
      }
    } else {
      gg = wave64_sum((double)g * (double)g);
      rr = gg;
      active = gg > 0.0 ? 1 : 0;
    }

    // ---- CG on H p = -g (Section 2.4) ----
    r = -g;
    pv = 0.f;
    float dv = r;
    const double bound = (double)c.cg_tol * sqrt(gg);
    for (int it = 0; it < c.max_cg && active != 0; ++it) {  // uniform
      const double inv_rr = 1.0 / rr;  // here and not at its use, where the next direction waits for it (ten iterations 29.7 -> 29.1 us at 1000 x 20, C = 3)
      // rows of D = P o W - P o rowsum(P o W), W = A d
      products(dv, dk);
#pragma unroll
      for (int k = 0; k < R; ++k) {
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < NC; ++q) s = fmaf(P[k][q], dk[k][q], s);
#pragma unroll
        for (int q = 0; q < NC; ++q) dk[k][q] = P[k][q] * (dk[k][q] - s);
      }
      const float s = col_sums(dk);
      const float q = own ? fmaf(c.lambda + rho_, dv, c.scale * s) : 0.f;
      const double dq = wave64_sum((double)dv * (double)q);
      if (!(dq > 0.0) || !isfinite(dq)) {  // no positive curvature: keep the current iterate
        active = 0;
      } else {
        const float al = (float)(rr / dq);
        r = fmaf(-al, q, r);
        const double rr_new = wave64_sum((double)r * (double)r);
        pv = fmaf(al, dv, pv);
        // a bound of 0 is met by a zero residual only: no square root in the chain
        const bool stop = bound > 0.0 ? sqrt(rr_new) <= bound : rr_new == 0.0;
        if (stop) active = 0;
        else dv = fmaf((float)(rr_new * inv_rr), dv, r);
        rr = rr_new;
        iters += 1;
      }
    }
    if (!newton) break;

    // ---- Armijo backtracking on Z + alpha A p (Algorithm 2), then X += alpha p ----
    products(pv, dk);
    double q0 = 0.0, q1 = 0.0, q2 = 0.0, sl = 0.0;
    if (own) {  // penalty along the line: q0 + alpha q1 + alpha^2 q2, and the slope <p, g>
      const double x = xv, pd = pv, uu = x - (double)zv + (double)yv * (1.0 / (double)rho_);
      q0 = 0.5 * (double)c.lambda * x * x + 0.5 * (double)rho_ * uu * uu;
      q1 = (double)c.lambda * x * pd + (double)rho_ * uu * pd;
      q2 = 0.5 * ((double)c.lambda + (double)rho_) * pd * pd;
      sl = pd * (double)g;
    }
    q0 = wave64_sum(q0); q1 = wave64_sum(q1); q2 = wave64_sum(q2); sl = wave64_sum(sl);
    ok = 1;
    for (int k = 0;; ++k) {  // uniform
      alpha = c.alphas[k];
      double la = 0.0;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        if (i >= nchunks) continue;  // uniform
        float zz[NC], M = 0.f, zb = 0.f;
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          zz[q] = fmaf(alpha, dk[i][q], z[i][q]);
          M = fmaxf(M, zz[q]);
          if (q == lab[i]) zb = zz[q];
        }
        float s = expf(-M);
#pragma unroll
        for (int q = 0; q < NC; ++q) s += expf(zz[q] - M);
        if (t + i * THREADS < n) la += (double)M + (double)logf(s) - (double)zb;
      }
      const double al = (double)alpha;
      loss_new = (double)c.scale * block_sum(la) + q0 + al * q1 + al * al * q2;
      evals = k + 1;
      if (!(loss_new > loss + al * (double)c.beta * sl)) break;  // Armijo holds (eq. armijo)
      if (k + 1 >= c.ncand) {                                    // the i > i_max break of Algorithm 2
        ok = 0;
        break;
      }
    }
    xv = own ? fmaf(alpha, pv, xv) : 0.f;
    s_newton += 1;
    s_cg += iters;
    s_ls += evals;
    s_failed += ok ? 0 : 1;
    s_loss_final = loss_new;
    if (t == 0 && nt < NADMM_TRACE_LEN) {
      st->stats.alpha[nt] = alpha;
      st->stats.cg_iters[nt] = iters;
    }
  }

  if (!newton) {
    if (t < dlen) c.p_out[t] = pv;  // dlen <= 64: wave 0
    if (t == 0) {
      if (c.iters_out) *c.iters_out = iters;
      if (c.relres_out) *c.relres_out = gg > 0.0 ? (float)sqrt(rr / gg) : 0.f;
    }
    return;
  }
  if (t < dlen) c.X_out[t] = xv;
  if (t == 0) {
    st->loss = loss; st->gg = gg; st->rr = rr; st->gg_cg = gg; st->loss_new = loss_new; st->loss_initial = loss_initial;
    st->alpha = alpha;
    st->newton_even = newton_active; st->cg_active = active; st->cg_iters = iters; st->armijo_ok = ok; st->ls_evals = evals;
    nadmm_stats* s = &st->stats;
    s->newton_iters = s_newton; s->cg_iters_total = s_cg; s->ls_evals_total = s_ls; s->armijo_failed = s_failed;
    s->loss_initial = loss_initial; s->loss_final = s_loss_final; s->grad_norm_final = s_gn;
  }
}

template <int NQ, int NC, int THREADS, int R>
hipError_t launch_n(const SmallSolve& c, hipStream_t st) {
  constexpr size_t lds = (size_t)THREADS * small_stride(4 * NQ) * sizeof(float);
  static_assert(lds >= (size_t)(THREADS / 64) * 16 * (4 * NQ * NC + 4) * sizeof(float), "the waves' partial sums fit the tile");
  if constexpr (lds + 8192 > 64 * 1024) {
    static LdsLimitMask done{0};
    const hipError_t e = ensure_lds_limit(reinterpret_cast<const void*>(&small_solve_kernel<NQ, NC, THREADS, R>), &done, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((small_solve_kernel<NQ, NC, THREADS, R>), dim3(1), dim3(THREADS), lds, st, c);
  return hipGetLastError();
}

template <int NQ, int NC>
hipError_t launch_t(const SmallSolve& c, hipStream_t st) {
  if constexpr (4 * NQ * NC <= 64) {
    // As many rows per thread as there are, on one wave per SIMD while that holds them (rounds with half the rows per thread on twice the waves take
    // longer: 1000 x 20, C = 3, a Newton iteration of 10 CG iterations 32.7 us for 29.5, on 1024 threads 55).  Padding four rows for two: 500 x 8, C = 4,
    // two Newton iterations of 5: 26.3 us, 23.0 without; 1400 x 14, C = 4, ten CG iterations with four rows for three 40.7, 36.5.
    if (c.n <= 512) return launch_n<NQ, NC, 256, 2>(c, st);
    if (c.n <= 768) return launch_n<NQ, NC, 256, 3>(c, st);
    if (c.n <= 1024) return launch_n<NQ, NC, 256, 4>(c, st);
    if (c.n <= 1536) return launch_n<NQ, NC, 512, 3>(c, st);
    return launch_n<NQ, NC, 512, 4>(c, st);
  }
  return hipErrorInvalidValue;
}

template <int NQ>
hipError_t launch_nq(const SmallSolve& c, hipStream_t st) {
  switch (c.NC) {
    case 1: return launch_t<NQ, 1>(c, st);
    case 2: return launch_t<NQ, 2>(c, st);
    case 3: return launch_t<NQ, 3>(c, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// One workgroup of 512 threads with four rows each; the limits on columns and classes are those of the thin-data kernel.
// Any number of iterations: the rows come in through one compute unit, but as one block of memory, which costs less than the
// launches of a single iteration.  Measured, launches against this kernel (us): 2048 x 32, C = 2: a CG solve of 1 iteration
// 25.3 : 15.6, of 4 47.7 : 18.1, a Newton iteration of 1 CG iteration 38.4 : 17.6; 2048 x 31, C = 3: 25.2 : 16.9, 68 : 28 and 54 : 26.
bool small_solve_supported(const Shape& s, int32_t max_cg) {
  const int64_t pp = (s.p + 3) / 4 * 4;
  return max_cg >= 1 && s.n <= 512 * kRowsPerThread && s.p <= 32 && s.NC <= 3 && pp * s.NC <= 64;
}

hipError_t launch_small_solve(const SmallSolve& c, hipStream_t st) {
  if (c.max_cg < 1 || c.A == nullptr || c.X == nullptr || c.n < 1 || c.n > 512 * kRowsPerThread || c.p < 1 || c.p > 32 ||
      c.lda < c.p || c.lda > (c.p + 3) / 4 * 4)
    return hipErrorInvalidValue;
  if (c.newton != 0 ? (c.labels == nullptr || c.X_out == nullptr || c.st == nullptr || c.ncand < 1 || c.max_newton < 1)
                    : (c.g == nullptr || c.p_out == nullptr))
    return hipErrorInvalidValue;
  SmallSolve s = c;
  s.quads = (c.lda & 3) == 0 && (reinterpret_cast<uintptr_t>(c.A) & 15) == 0 ? 1 : 0;
  switch ((c.p + 3) / 4) {
    case 1: return launch_nq<1>(s, st);
    case 2: return launch_nq<2>(s, st);
    case 3: return launch_nq<3>(s, st);
    case 4: return launch_nq<4>(s, st);
    case 5: return launch_nq<5>(s, st);
    case 6: return launch_nq<6>(s, st);
    case 7: return launch_nq<7>(s, st);
    case 8: return launch_nq<8>(s, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace nadmm
