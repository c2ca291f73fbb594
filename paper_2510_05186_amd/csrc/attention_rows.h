// One row of causal attention by one wave, any storage type, head_dim 64 DPL: fp32 arithmetic, online softmax.  A row reads no
// key above the diagonal (dK / dV: no query below it), so a value that is not finite reaches the rows that attend to it
// and no other.  The general kernels are made of these rows, and the matrix-unit kernels that multiply whole tiles, a key above the
// diagonal by a probability of zero (zero times infinity is NaN), redo rows that came out non-finite with them.
// All 64 lanes take part; the LDS pointers are the wave's own.
#pragma once
#include "common.h"

// LDS written by lanes of this wave is read by others of the same wave: LDS operations of a wave run in order, so only the compiler
// has to keep theirs
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Columns k and k + d / 2 of a gradient row, turned back by the angle of the row's position (the transposed rotary rotation)
__device__ __forceinline__ void rope_back(float& lo, float& hi, float cs, float sn) {
  const float a = lo;
  lo = a * cs + hi * sn;
  hi = hi * cs - a * sn;
}
// the same for a row spread over a wave: lane l holds the columns l + 64 e; table row of the position, d / 2 (cos, sin) pairs
template <int DPL> __device__ __forceinline__ void rope_back_row(float (&v)[DPL], const float2* row, int lane) {
  if constexpr (DPL == 2) {
    rope_back(v[0], v[1], row[lane].x, row[lane].y);
  } else {
    const float other = __shfl_xor(v[0], 32, 64);
    const float2 t = row[lane & 31];
    v[0] = lane < 32 ? v[0] * t.x + other * t.y : v[0] * t.x - other * t.y;
  }
}

// qs: 64 DPL floats
template <typename T, int DPL>
__device__ __forceinline__ void attn_fwd_row(const T* __restrict__ qkv, T* __restrict__ o, float* __restrict__ lse, int seq, int n_q,
                                             int n_kv, int t, int a, int b, float* qs) {
  constexpr int D = 64 * DPL;
  const int lane = threadIdx.x & 63, g = a * n_kv / n_q;
  const int ld = (n_q + 2 * n_kv) * D;
  const T* base = qkv + (size_t)b * seq * ld;
  const float scale = rsqrtf((float)D);
#pragma unroll
  for (int e = 0; e < DPL; ++e) qs[lane + 64 * e] = to_f32(base[(size_t)t * ld + a * D + lane + 64 * e]) * scale;
  wave_lds_fence();
  const T* Kp = base + (size_t)(n_q + g) * D;
  const T* Vp = base + (size_t)(n_q + n_kv + g) * D;
  float m = -INFINITY, l = 0.f, acc[DPL];
#pragma unroll
  for (int e = 0; e < DPL; ++e) acc[e] = 0.f;
  for (int c0 = 0; c0 <= t; c0 += 64) {
    const int key = c0 + lane;
    const bool valid = key <= t;
    float s = -INFINITY;
    if (valid) {
      const T* kr = Kp + (size_t)key * ld;
      s = 0.f;
      for (int dd = 0; dd < D; ++dd) s = fmaf(qs[dd], to_f32(kr[dd]), s);
    }
    const float mn = fmaxf(m, wave_max(s));
    const float p = valid ? expf(s - mn) : 0.f;
    const float alpha = expf(m - mn);
    l = l * alpha + wave_sum(p);
#pragma unroll
    for (int e = 0; e < DPL; ++e) acc[e] *= alpha;
    const int nj = min(64, t - c0 + 1);
    for (int j = 0; j < nj; ++j) {
      const float pj = __shfl(p, j, 64);
      const T* vr = Vp + (size_t)(c0 + j) * ld;
#pragma unroll
      for (int e = 0; e < DPL; ++e) acc[e] = fmaf(pj, to_f32(vr[lane + 64 * e]), acc[e]);
    }
    m = mn;
  }
  T* orow = o + ((size_t)b * seq + t) * (n_q * D) + a * D;
#pragma unroll
  for (int e = 0; e < DPL; ++e) orow[lane + 64 * e] = from_f32<T>(acc[e] / l);
  if (lane == 0) lse[((size_t)b * n_q + a) * seq + t] = m + logf(l);
}

// D_t = <dO_t, O_t> (stored where Dws is given), dQ_t = scale * sum_j dS_tj K_j, turned back by the rotary angle where a table is given.
// dqkv may be qkv itself: the row's Q is read before its dQ is written.  qs, dos: 64 DPL floats each
template <typename T, int DPL>
__device__ __forceinline__ void attn_bwd_dq_row(const T* qkv, const T* __restrict__ o, const T* __restrict__ dout,
                                                const float* __restrict__ lse, T* dqkv, float* __restrict__ Dws,
                                                int seq, int n_q, int n_kv, int t, int a, int b, float* qs, float* dos,
                                                const float2* rope = nullptr) {
  constexpr int D = 64 * DPL;
  const int lane = threadIdx.x & 63, g = a * n_kv / n_q;
  const int ld = (n_q + 2 * n_kv) * D;
  const T* base = qkv + (size_t)b * seq * ld;
  const float scale = rsqrtf((float)D);
  const size_t orow = ((size_t)b * seq + t) * (n_q * D) + a * D;
  float dsum = 0.f;
#pragma unroll
  for (int e = 0; e < DPL; ++e) {
    qs[lane + 64 * e] = to_f32(base[(size_t)t * ld + a * D + lane + 64 * e]) * scale;
    float dv = to_f32(dout[orow + lane + 64 * e]);
    dos[lane + 64 * e] = dv;
    dsum += dv * to_f32(o[orow + lane + 64 * e]);
  }
  dsum = wave_sum(dsum);
  wave_lds_fence();
  const float L = lse[((size_t)b * n_q + a) * seq + t];
  if (lane == 0 && Dws) Dws[((size_t)b * n_q + a) * seq + t] = dsum;
  const T* Kp = base + (size_t)(n_q + g) * D;
  const T* Vp = base + (size_t)(n_q + n_kv + g) * D;
  float acc[DPL];
#pragma unroll
  for (int e = 0; e < DPL; ++e) acc[e] = 0.f;
  for (int c0 = 0; c0 <= t; c0 += 64) {
    const int key = c0 + lane;
    float dS = 0.f;
    if (key <= t) {
      const T* kr = Kp + (size_t)key * ld;
      const T* vr = Vp + (size_t)key * ld;
      float s = 0.f, dp = 0.f;
      for (int dd = 0; dd < D; ++dd) {
        s = fmaf(qs[dd], to_f32(kr[dd]), s);
        dp = fmaf(dos[dd], to_f32(vr[dd]), dp);
      }
      dS = expf(s - L) * (dp - dsum);
    }
    const int nj = min(64, t - c0 + 1);
    for (int j = 0; j < nj; ++j) {
      const float dj = __shfl(dS, j, 64);
      const T* kr = Kp + (size_t)(c0 + j) * ld;
#pragma unroll
      for (int e = 0; e < DPL; ++e) acc[e] = fmaf(dj, to_f32(kr[lane + 64 * e]), acc[e]);
    }
  }
  T* dq = dqkv + ((size_t)b * seq + t) * ld + a * D;
#pragma unroll
  for (int e = 0; e < DPL; ++e) acc[e] *= scale;
  if (rope) rope_back_row<DPL>(acc, rope + (size_t)t * (D / 2), lane);
#pragma unroll
  for (int e = 0; e < DPL; ++e) dq[lane + 64 * e] = from_f32<T>(acc[e]);
}

// Key row tk of kv head g: dV = sum_t P_t dO_t, dK = scale * sum_t dS_t Q_t over the group's q heads, dK turned back by the rotary angle
// where a table is given.  Q comes from q rows of ldq elements (qkv itself, or a copy where dqkv is qkv and holds dQ by now).  Dws
// holds D, or -D where NEG_D.  ks, vs: 64 DPL floats each
template <typename T, int DPL, bool NEG_D>
__device__ __forceinline__ void attn_bwd_dkv_row(const T* qkv, const T* q, int ldq, const T* __restrict__ dout, const float* __restrict__ lse,
                                                 const float* __restrict__ Dws, T* dqkv, int seq, int n_q, int n_kv,
                                                 int tk, int g, int b, float* ks, float* vs, const float2* rope = nullptr) {
  constexpr int D = 64 * DPL;
  const int lane = threadIdx.x & 63;
  const int ld = (n_q + 2 * n_kv) * D;
  const T* base = qkv + (size_t)b * seq * ld;
  const float scale = rsqrtf((float)D);
#pragma unroll
  for (int e = 0; e < DPL; ++e) {
    ks[lane + 64 * e] = to_f32(base[(size_t)tk * ld + (n_q + g) * D + lane + 64 * e]) * scale;
    vs[lane + 64 * e] = to_f32(base[(size_t)tk * ld + (n_q + n_kv + g) * D + lane + 64 * e]);
  }
  wave_lds_fence();
  float dk[DPL], dv[DPL];
#pragma unroll
  for (int e = 0; e < DPL; ++e) { dk[e] = 0.f; dv[e] = 0.f; }
  const int rep = n_q / n_kv;
  for (int a = g * rep; a < (g + 1) * rep; ++a) {
    const float* Lp = lse + ((size_t)b * n_q + a) * seq;
    const float* Dp = Dws + ((size_t)b * n_q + a) * seq;
    for (int c0 = (tk / 64) * 64; c0 < seq; c0 += 64) {
      const int tq = c0 + lane;
      float p = 0.f, dS = 0.f;
      if (tq >= tk && tq < seq) {
        const T* qr = q + ((size_t)b * seq + tq) * ldq + a * D;
        const T* dor = dout + ((size_t)b * seq + tq) * (n_q * D) + a * D;
        float s = 0.f, dp = 0.f;
        for (int dd = 0; dd < D; ++dd) {
          s = fmaf(ks[dd], to_f32(qr[dd]), s);
          dp = fmaf(vs[dd], to_f32(dor[dd]), dp);
        }
        p = expf(s - Lp[tq]);
        dS = p * (NEG_D ? dp + Dp[tq] : dp - Dp[tq]);
      }
      const int j0 = max(0, tk - c0), j1 = min(64, seq - c0);
      for (int j = j0; j < j1; ++j) {
        const float pj = __shfl(p, j, 64), dj = __shfl(dS, j, 64);
        const T* qr = q + ((size_t)b * seq + c0 + j) * ldq + a * D;
        const T* dor = dout + ((size_t)b * seq + c0 + j) * (n_q * D) + a * D;
#pragma unroll
        for (int e = 0; e < DPL; ++e) {
          dv[e] = fmaf(pj, to_f32(dor[lane + 64 * e]), dv[e]);
          dk[e] = fmaf(dj, to_f32(qr[lane + 64 * e]), dk[e]);
        }
      }
    }
  }
  T* dkr = dqkv + ((size_t)b * seq + tk) * ld + (n_q + g) * D;
  T* dvr = dqkv + ((size_t)b * seq + tk) * ld + (n_q + n_kv + g) * D;
#pragma unroll
  for (int e = 0; e < DPL; ++e) dk[e] *= scale;
  if (rope) rope_back_row<DPL>(dk, rope + (size_t)tk * (D / 2), lane);
#pragma unroll
  for (int e = 0; e < DPL; ++e) {
    dkr[lane + 64 * e] = from_f32<T>(dk[e]);
    dvr[lane + 64 * e] = from_f32<T>(dv[e]);
  }
}
