// Causal attention forward / backward in fp32 on the fp32 matrix instruction v_mfma_f32_16x16x4_f32 (fp32 products and sums),
// head_dim 64 or 128.  q-head a reads kv-head a * n_kv / n_q; dK and dV are summed over the q-heads of a group.  Packed qkv
// rows: [q heads | k heads | v heads].  lse is [batch][n_q][seq], natural log.
//
// A workgroup owns 16 rows (queries, or keys for dK / dV) of one head; its four waves split the tiles of 16 rows on the other side
// (wave w takes tiles w, w + 4, ...) and their partial results are combined through LDS at the end.  With a few hundred tokens
// that is what gives most of the 256 compute units work, and several workgroups share one, so loads go straight from memory
// (L2) into registers: no LDS in the loop, no barrier.  What bounds it is the latency of those loads between dependent
// products; the general kernels (one wave per row, 64 partial sums by shuffles) are an order of magnitude above that.
//
// Fragment layouts (lane = 16 g + r).  An MFMA takes A[row r][k g] and B[k g][column r] and leaves D[row 4 g + v][column r].
//  rows     4 floats at row r, columns 16 s + 4 g .. + 3: element e is the operand of MFMA (s, e), which contracts the columns
//           16 s + 4 g + e; the same on both sides.
//  columns  (the operand contracted over its rows) 4 floats at row 4 g + e, columns 64 h + 4 r .. + 3: element i belongs to the
//           output tile 4 h + i, whose row r is column 64 h + 4 r + i.  Rows 4 g + e are where the probabilities of MFMA e sit: a lane
//           holds D[4 g + e][r], which is B[k g][column r] for the contraction over 4 g + e.
//  Result   tile 4 h + i, register v: column 64 h + 4 (4 g + v) + i of row r, i.e. 4 consecutive columns over i.
// A tile on the diagonal multiplies keys above it by a probability of zero, and rows past the end repeat the last one: with finite
// operands that adds nothing, with others it makes NaN of rows that do not depend on them.  Where a result is not finite the
// workgroup therefore redoes its rows one by one (attention_rows.h): one barrier more, nothing else, for finite ones.
// Measured (us, general kernels -> these): 512 tokens, 16 heads of 64: forward 188 -> 17.8, dQ 275 -> 19.5, dK / dV 286 -> 29.5;
// 128 tokens, 4 heads: 35.1 -> 7.0, 21.2 -> 7.4, 22.0 -> 9.0.
#include "attention_rows.h"

namespace {

constexpr int ROWS = 16;

template <int D> struct F32 {
  static constexpr int S = D / 16, H = D / 64, NT = D / 16;   // k-steps of a row, 64-column groups, output tiles
  static __device__ __forceinline__ void rows(f32x4_t (&v)[S], const float* row, int g) {
#pragma unroll
    for (int s = 0; s < S; ++s) v[s] = *reinterpret_cast<const f32x4_t*>(row + 16 * s + 4 * g);
  }
  // v[e][h]: base + (row 4 g + e) * ld, rows clamped to `last`
  static __device__ __forceinline__ void columns(f32x4_t (&v)[4][H], const float* base, size_t ld, int first, int last, int g, int r) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float* p = base + (size_t)min(first + 4 * g + e, last) * ld + 4 * r;
#pragma unroll
      for (int h = 0; h < H; ++h) v[e][h] = *reinterpret_cast<const f32x4_t*>(p + 64 * h);
    }
  }
  // D[4 g + v][r] = sum over columns of a-rows times b-rows
  static __device__ __forceinline__ f32x4_t product(const f32x4_t (&a)[S], const f32x4_t (&b)[S]) {
    f32x4_t d0 = {0.f, 0.f, 0.f, 0.f}, d1 = {0.f, 0.f, 0.f, 0.f};   // two chains: consecutive MFMAs do not wait for one another
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s][e], b[s][e], d0, 0, 0, 0);
        d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s][e + 1], b[s][e + 1], d1, 0, 0, 0);
      }
    return f32x4_t{d0[0] + d1[0], d0[1] + d1[1], d0[2] + d1[2], d0[3] + d1[3]};
  }
  static __device__ __forceinline__ void accumulate(f32x4_t (&acc)[NT], const f32x4_t (&c)[4][H], const f32x4_t& p) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(c[e][t >> 2][t & 3], p[e], acc[t], 0, 0, 0);
  }
  // this lane's part of the 16 x D result into LDS rows of D + 4 floats
  static __device__ __forceinline__ void put(float (*dst)[D + 4], const f32x4_t (&acc)[NT], int g, int r) {
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        *reinterpret_cast<f32x4_t*>(&dst[r][64 * h + 16 * g + 4 * v]) =
            f32x4_t{acc[4 * h][v], acc[4 * h + 1][v], acc[4 * h + 2][v], acc[4 * h + 3][v]};
  }
  static __device__ __forceinline__ void clear(f32x4_t (&acc)[NT]) {
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  // columns c .. c + 3 of a result row, out of the four partial results, rotated back: the partner columns lie d / 2 away
  static __device__ __forceinline__ void turn_back(f32x4_t& v, const float (*part)[ROWS][D + 4], float scale, const float2* angle, int row, int c) {
    const int k = c % (D / 2), other = c < D / 2 ? c + D / 2 : c - D / 2;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float x = (((part[0][row][other + e] + part[1][row][other + e]) + part[2][row][other + e]) + part[3][row][other + e]) * scale;
      const float2 t = angle[k + e];
      float own = v[e];
      if (c < D / 2) rope_back(own, x, t.x, t.y);
      else rope_back(x, own, t.x, t.y);
      v[e] = own;
    }
  }
  static __device__ __forceinline__ void scaled(f32x4_t (&v)[S], float f) {
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[s][e] *= f;
  }
};

__device__ __forceinline__ bool all_finite(const f32x4_t& v) {
  const float z = (v[0] * 0.f + v[1] * 0.f) + (v[2] * 0.f + v[3] * 0.f);   // 0 times infinity or NaN is NaN
  return z == 0.f;
}
// sum or maximum over the four lanes that hold a column's rows
__device__ __forceinline__ float sum_g(float x) { x += __shfl_xor(x, 16, 64); return x + __shfl_xor(x, 32, 64); }
__device__ __forceinline__ float max_g(float x) { x = fmaxf(x, __shfl_xor(x, 16, 64)); return fmaxf(x, __shfl_xor(x, 32, 64)); }

// longest rows (last query tiles) are dispatched first, for every head: grid (n_q, batch, tiles)
template <int D>
__global__ __launch_bounds__(256) void attn_fwd_f32(const float* __restrict__ qkv, float* __restrict__ o, float* __restrict__ lse,
                                                    int seq, int n_q, int n_kv) {
  typedef F32<D> F;
  __shared__ __attribute__((aligned(16))) float part[4][ROWS][D + 4];
  __shared__ float pm[4][ROWS], pl[4][ROWS];
  __shared__ int redo;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
  const int tile = gridDim.z - 1 - blockIdx.z, a = blockIdx.x, b = blockIdx.y, kvh = a * n_kv / n_q;
  const int q0 = tile * ROWS, last = seq - 1;
  const size_t ld = (size_t)(n_q + 2 * n_kv) * D;
  const float* base = qkv + (size_t)b * seq * ld;
  const float *Kp = base + (size_t)(n_q + kvh) * D, *Vp = base + (size_t)(n_q + n_kv + kvh) * D;
  f32x4_t q[F::S], acc[F::NT];
  F::rows(q, base + (size_t)min(q0 + r, last) * ld + (size_t)a * D, g);
  F::scaled(q, rsqrtf((float)D));
  F::clear(acc);
  float m = -INFINITY, l = 0.f;
  for (int t = wave; t <= tile; t += 4) {
    f32x4_t k[F::S], v[4][F::H];
    F::rows(k, Kp + (size_t)min(16 * t + r, last) * ld, g);
    F::columns(v, Vp, ld, 16 * t, last, g, r);
    f32x4_t s = F::product(k, q);                            // s[e]: key 16 t + 4 g + e, query q0 + r
    if (t == tile) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * g + e > r) s[e] = -INFINITY;
    }
    // every tile up to the diagonal holds a key of every query, so the maximum is finite from the first one on
    const float mn = fmaxf(m, max_g(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))));
    const float alpha = expf(m - mn);
    f32x4_t p;
#pragma unroll
    for (int e = 0; e < 4; ++e) p[e] = expf(s[e] - mn);
    l = l * alpha + (p[0] + p[1]) + (p[2] + p[3]);           // this lane's keys; summed over the four lanes at the end
#pragma unroll
    for (int i = 0; i < F::NT; ++i)
#pragma unroll
      for (int x = 0; x < 4; ++x) acc[i][x] *= alpha;
    F::accumulate(acc, v, p);
    m = mn;
  }
  l = sum_g(l);
  F::put(part[wave], acc, g, r);
  if (g == 0) { pm[wave][r] = m; pl[wave][r] = l; }
  if (threadIdx.x == 0) redo = 0;
  __syncthreads();
  f32x4_t out[F::H];
  float ls[F::H];
#pragma unroll
  for (int h = 0; h < F::H; ++h) {
    const int i = threadIdx.x + 256 * h, row = i / (D / 4), c = (i % (D / 4)) * 4;
    const float M = fmaxf(fmaxf(pm[0][row], pm[1][row]), fmaxf(pm[2][row], pm[3][row]));
    float L = 0.f;
    f32x4_t v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float f = expf(pm[w][row] - M);                  // a wave without tiles: exp(-inf) = 0 times zeros
      L += pl[w][row] * f;
      const f32x4_t x = *reinterpret_cast<const f32x4_t*>(&part[w][row][c]);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += x[e] * f;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] /= L;
    out[h] = v;
    ls[h] = M + logf(L);
    if (q0 + row < seq && !(all_finite(v) && fabsf(ls[h]) < INFINITY)) redo = 1;
  }
  __syncthreads();
  if (redo) {
    for (int row = wave; row < ROWS && q0 + row < seq; row += 4)
      attn_fwd_row<float, F::H>(qkv, o, lse, seq, n_q, n_kv, q0 + row, a, b, &part[wave][0][0]);
    return;
  }
#pragma unroll
  for (int h = 0; h < F::H; ++h) {
    const int i = threadIdx.x + 256 * h, row = i / (D / 4), c = (i % (D / 4)) * 4, t = q0 + row;
    if (t >= seq) continue;
    *reinterpret_cast<f32x4_t*>(o + ((size_t)b * seq + t) * ((size_t)n_q * D) + (size_t)a * D + c) = out[h];
    if (c == 0) lse[((size_t)b * n_q + a) * seq + t] = ls[h];
  }
}

// D_t = <dO_t, O_t> (stored for the dK / dV kernel), dQ_t = scale * sum_j dS_tj K_j
template <int D>
__global__ __launch_bounds__(256) void attn_bwd_dq_f32(const float* qkv, const float* __restrict__ o,
                                                       const float* __restrict__ dout, const float* __restrict__ lse,
                                                       float* dqkv, float* __restrict__ qcopy, const float2* __restrict__ rope,
                                                       float* __restrict__ Dws, int seq, int n_q, int n_kv) {
  typedef F32<D> F;
  __shared__ __attribute__((aligned(16))) float part[4][ROWS][D + 4];
  __shared__ int redo;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
  const int tile = gridDim.z - 1 - blockIdx.z, a = blockIdx.x, b = blockIdx.y, kvh = a * n_kv / n_q;
  const int q0 = tile * ROWS, last = seq - 1, row_q = min(q0 + r, last);
  const size_t ld = (size_t)(n_q + 2 * n_kv) * D, ldo = (size_t)n_q * D;
  const float* base = qkv + (size_t)b * seq * ld;
  const float *Kp = base + (size_t)(n_q + kvh) * D, *Vp = base + (size_t)(n_q + n_kv + kvh) * D;
  const float scale = rsqrtf((float)D);
  f32x4_t q[F::S], dO[F::S], x[F::S], acc[F::NT];
  F::rows(q, base + (size_t)row_q * ld + (size_t)a * D, g);
  F::rows(dO, dout + ((size_t)b * seq + row_q) * ldo + (size_t)a * D, g);
  F::rows(x, o + ((size_t)b * seq + row_q) * ldo + (size_t)a * D, g);
  if (qcopy && wave == 0 && q0 + r < seq) {                  // dQ will take Q's place: the dK / dV kernel reads this copy
    float* p = qcopy + ((size_t)b * seq + row_q) * ldo + (size_t)a * D;
#pragma unroll
    for (int s = 0; s < F::S; ++s) *reinterpret_cast<f32x4_t*>(p + 16 * s + 4 * g) = q[s];
  }
  F::scaled(q, scale);
  F::clear(acc);
  float dsum = 0.f;
#pragma unroll
  for (int s = 0; s < F::S; ++s)
#pragma unroll
    for (int e = 0; e < 4; ++e) dsum = fmaf(dO[s][e], x[s][e], dsum);
  dsum = sum_g(dsum);
  const size_t stat = ((size_t)b * n_q + a) * seq + row_q;
  const float L = lse[stat];
  if (wave == 0 && g == 0 && q0 + r < seq) Dws[stat] = dsum;
  for (int t = wave; t <= tile; t += 4) {
    f32x4_t k[F::S], v[F::S], kc[4][F::H];
    F::rows(k, Kp + (size_t)min(16 * t + r, last) * ld, g);
    F::rows(v, Vp + (size_t)min(16 * t + r, last) * ld, g);
    F::columns(kc, Kp, ld, 16 * t, last, g, r);
    const f32x4_t s = F::product(k, q), dp = F::product(v, dO);
    f32x4_t ds;
#pragma unroll
    for (int e = 0; e < 4; ++e) ds[e] = t == tile && 4 * g + e > r ? 0.f : expf(s[e] - L) * (dp[e] - dsum);
    F::accumulate(acc, kc, ds);
  }
  F::put(part[wave], acc, g, r);
  if (threadIdx.x == 0) redo = 0;
  __syncthreads();
  f32x4_t out[F::H];
#pragma unroll
  for (int h = 0; h < F::H; ++h) {
    const int i = threadIdx.x + 256 * h, row = i / (D / 4), c = (i % (D / 4)) * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      out[h][e] = (((part[0][row][c + e] + part[1][row][c + e]) + part[2][row][c + e]) + part[3][row][c + e]) * scale;
    if (q0 + row < seq && !all_finite(out[h])) redo = 1;
    if (rope && q0 + row < seq) F::turn_back(out[h], part, scale, rope + (size_t)(q0 + row) * (D / 2), row, c);
  }
  __syncthreads();
  if (redo) {
    for (int row = wave; row < ROWS && q0 + row < seq; row += 4)
      attn_bwd_dq_row<float, F::H>(qkv, o, dout, lse, dqkv, nullptr, seq, n_q, n_kv, q0 + row, a, b, &part[wave][0][0], &part[wave][2][0], rope);
    return;
  }
#pragma unroll
  for (int h = 0; h < F::H; ++h) {
    const int i = threadIdx.x + 256 * h, row = i / (D / 4), c = (i % (D / 4)) * 4, t = q0 + row;
    if (t < seq) *reinterpret_cast<f32x4_t*>(dqkv + ((size_t)b * seq + t) * ld + (size_t)a * D + c) = out[h];
  }
}

// per 16 keys and kv head: dV = sum_t P_t dO_t, dK = scale * sum_t dS_t Q_t over the group's q heads
template <int D>
__global__ __launch_bounds__(256) void attn_bwd_dkv_f32(const float* qkv, const float* qsrc, int ldq, const float* __restrict__ dout,
                                                        const float* __restrict__ lse, const float* __restrict__ Dws,
                                                        float* dqkv, const float2* __restrict__ rope, int seq, int n_q, int n_kv) {
  typedef F32<D> F;
  __shared__ __attribute__((aligned(16))) float part[4][ROWS][D + 4];
  __shared__ int redo;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
  const int tile = blockIdx.z, kvh = blockIdx.x, b = blockIdx.y, k0 = tile * ROWS, last = seq - 1;
  const size_t ld = (size_t)(n_q + 2 * n_kv) * D, ldo = (size_t)n_q * D;
  const float* base = qkv + (size_t)b * seq * ld;
  const float scale = rsqrtf((float)D);
  f32x4_t k[F::S], v[F::S], ak[F::NT], av[F::NT];
  F::rows(k, base + (size_t)min(k0 + r, last) * ld + (size_t)(n_q + kvh) * D, g);
  F::rows(v, base + (size_t)min(k0 + r, last) * ld + (size_t)(n_q + n_kv + kvh) * D, g);
  F::scaled(k, scale);
  F::clear(ak);
  F::clear(av);
  const int rep = n_q / n_kv, tiles = (seq + ROWS - 1) / ROWS - tile;   // query tiles at or after these keys
  for (int it = wave; it < rep * tiles; it += 4) {
    const int a = kvh * rep + it / tiles, t = tile + it % tiles;
    const float *Qp = qsrc + (size_t)b * seq * ldq + (size_t)a * D, *dOp = dout + (size_t)b * seq * ldo + (size_t)a * D;
    const float *Lp = lse + ((size_t)b * n_q + a) * seq, *Dp = Dws + ((size_t)b * n_q + a) * seq;
    f32x4_t q[F::S], dO[F::S], c[4][F::H];
    F::rows(q, Qp + (size_t)min(16 * t + r, last) * ldq, g);
    F::rows(dO, dOp + (size_t)min(16 * t + r, last) * ldo, g);
    const f32x4_t s = F::product(q, k), dp = F::product(dO, v);   // [e]: query 16 t + 4 g + e, key k0 + r
    f32x4_t p, ds;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int tq = 16 * t + 4 * g + e, at = min(tq, last);
      p[e] = tq >= seq || tq < k0 + r ? 0.f : expf(s[e] - Lp[at]);
      ds[e] = tq >= seq || tq < k0 + r ? 0.f : p[e] * (dp[e] - Dp[at]);
    }
    F::columns(c, dOp, ldo, 16 * t, last, g, r);
    F::accumulate(av, c, p);
    F::columns(c, Qp, ldq, 16 * t, last, g, r);
    F::accumulate(ak, c, ds);
  }
  if (threadIdx.x == 0) redo = 0;
  f32x4_t out[2][F::H];
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    if (which) __syncthreads();
    F::put(part[wave], which ? av : ak, g, r);
    __syncthreads();
#pragma unroll
    for (int h = 0; h < F::H; ++h) {
      const int i = threadIdx.x + 256 * h, row = i / (D / 4), c = (i % (D / 4)) * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x = ((part[0][row][c + e] + part[1][row][c + e]) + part[2][row][c + e]) + part[3][row][c + e];
        out[which][h][e] = which ? x : x * scale;
      }
      if (k0 + row < seq && !all_finite(out[which][h])) redo = 1;
      if (!which && rope && k0 + row < seq) F::turn_back(out[0][h], part, scale, rope + (size_t)(k0 + row) * (D / 2), row, c);
    }
  }
  __syncthreads();
  if (redo) {
    for (int row = wave; row < ROWS && k0 + row < seq; row += 4)
      attn_bwd_dkv_row<float, F::H, false>(qkv, qsrc, ldq, dout, lse, Dws, dqkv, seq, n_q, n_kv, k0 + row, kvh, b, &part[wave][0][0],
                                           &part[wave][2][0], rope);
    return;
  }
#pragma unroll
  for (int which = 0; which < 2; ++which)
#pragma unroll
    for (int h = 0; h < F::H; ++h) {
      const int i = threadIdx.x + 256 * h, row = i / (D / 4), c = (i % (D / 4)) * 4, t = k0 + row;
      if (t < seq) *reinterpret_cast<f32x4_t*>(dqkv + ((size_t)b * seq + t) * ld + (size_t)(n_q + which * n_kv + kvh) * D + c) = out[which][h];
    }
}

}  // namespace

// rows of 16-byte pieces: head_dim 64 or 128 makes every stride one, so only the base addresses decide; the tile count must
// fit the grid's third dimension
bool attn_f32_applies(int dtype, int d, int seq, const void* p0, const void* p1, const void* p2, const void* p3) {
  return dtype == DT_FP32 && (d == 64 || d == 128) && (seq + ROWS - 1) / ROWS < 65536 &&
         (((uintptr_t)p0 | (uintptr_t)p1 | (uintptr_t)p2 | (uintptr_t)p3) & 15) == 0;
}

hipError_t launch_attn_fwd_f32(const void* qkv, void* o, float* lse, int seq, int batch, int n_q, int n_kv, int d, hipStream_t s) {
  const dim3 grid(n_q, batch, (seq + ROWS - 1) / ROWS);
  if (d == 64) hipLaunchKernelGGL(attn_fwd_f32<64>, grid, dim3(256), 0, s, (const float*)qkv, (float*)o, lse, seq, n_q, n_kv);
  else hipLaunchKernelGGL(attn_fwd_f32<128>, grid, dim3(256), 0, s, (const float*)qkv, (float*)o, lse, seq, n_q, n_kv);
  return hipGetLastError();
}

hipError_t launch_attn_bwd_f32(const void* qkv, const void* o, const void* dout, const float* lse, void* dqkv, float* ws, int seq,
                               int batch, int n_q, int n_kv, int d, hipStream_t s, void* qcopy, const float2* rope) {
  const int tiles = (seq + ROWS - 1) / ROWS;
  const float *q = (const float*)qkv, *op = (const float*)o, *dop = (const float*)dout;
  float *dq = (float*)dqkv, *qc = (float*)qcopy;
  const float* qsrc = qc ? qc : q;
  const int ldq = (qc ? n_q : n_q + 2 * n_kv) * d;
  if (d == 64) hipLaunchKernelGGL(attn_bwd_dq_f32<64>, dim3(n_q, batch, tiles), dim3(256), 0, s, q, op, dop, lse, dq, qc, rope, ws, seq, n_q, n_kv);
  else hipLaunchKernelGGL(attn_bwd_dq_f32<128>, dim3(n_q, batch, tiles), dim3(256), 0, s, q, op, dop, lse, dq, qc, rope, ws, seq, n_q, n_kv);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (d == 64) hipLaunchKernelGGL(attn_bwd_dkv_f32<64>, dim3(n_kv, batch, tiles), dim3(256), 0, s, q, qsrc, ldq, dop, lse, ws, dq, rope, seq, n_q, n_kv);
  else hipLaunchKernelGGL(attn_bwd_dkv_f32<128>, dim3(n_kv, batch, tiles), dim3(256), 0, s, q, qsrc, ldq, dop, lse, ws, dq, rope, seq, n_q, n_kv);
  return hipGetLastError();
}
