// Causal attention forward / backward, general path (any storage type, head_dim 64 or 128): one wave
// per query row (forward, dQ) or per key row (dK, dV), fp32 arithmetic, online softmax.  The fallback
// where the MFMA kernels do not apply (operands that are not 16-byte aligned, sequences past 32-bit offsets) or gain nothing (a few tokens).  q-head a reads kv-head
// a * n_kv / n_q; dK and dV are summed over the q-heads of a group.  Packed qkv rows:
// [q heads | k heads | v heads].  lse is [batch][n_q][seq], natural log.
#include "attention_rows.h"

namespace {

template <typename T, int DPL>   // DPL = head_dim / 64
__global__ __launch_bounds__(256) void attn_fwd_simple(const T* __restrict__ qkv, T* __restrict__ o,
                                                       float* __restrict__ lse, int seq, int n_q, int n_kv) {
  __shared__ float qs[4][64 * DPL];
  const int wave = threadIdx.x >> 6, t = blockIdx.x * 4 + wave;
  if (t < seq) attn_fwd_row<T, DPL>(qkv, o, lse, seq, n_q, n_kv, t, blockIdx.y, blockIdx.z, qs[wave]);
}

// per query row: D_t = <dO_t, O_t>, dQ_t = scale * sum_j dS_tj K_j
template <typename T, int DPL>
__global__ __launch_bounds__(256) void attn_bwd_dq_simple(const T* __restrict__ qkv, const T* __restrict__ o,
                                                          const T* __restrict__ dout, const float* __restrict__ lse,
                                                          T* __restrict__ dqkv, float* __restrict__ Dws, int seq,
                                                          int n_q, int n_kv) {
  __shared__ float qs[4][64 * DPL];
  __shared__ float dos[4][64 * DPL];
  const int wave = threadIdx.x >> 6, t = blockIdx.x * 4 + wave;
  if (t < seq) attn_bwd_dq_row<T, DPL>(qkv, o, dout, lse, dqkv, Dws, seq, n_q, n_kv, t, blockIdx.y, blockIdx.z, qs[wave], dos[wave]);
}

// per key row and kv head: dV = sum_t P_t dO_t, dK = scale * sum_t dS_t Q_t over the group's q heads
template <typename T, int DPL>
__global__ __launch_bounds__(256) void attn_bwd_dkv_simple(const T* __restrict__ qkv, const T* __restrict__ dout,
                                                           const float* __restrict__ lse, const float* __restrict__ Dws,
                                                           T* __restrict__ dqkv, int seq, int n_q, int n_kv) {
  __shared__ float ks[4][64 * DPL];
  __shared__ float vs[4][64 * DPL];
  const int wave = threadIdx.x >> 6, tk = blockIdx.x * 4 + wave;
  if (tk < seq) attn_bwd_dkv_row<T, DPL, false>(qkv, qkv, (n_q + 2 * n_kv) * 64 * DPL, dout, lse, Dws, dqkv, seq, n_q, n_kv, tk, blockIdx.y, blockIdx.z, ks[wave], vs[wave]);
}

template <typename T, int DPL>
hipError_t fwd_t(const void* qkv, void* o, float* lse, int seq, int batch, int n_q, int n_kv, hipStream_t s) {
  hipLaunchKernelGGL((attn_fwd_simple<T, DPL>), dim3((seq + 3) / 4, n_q, batch), dim3(256), 0, s, (const T*)qkv, (T*)o, lse, seq, n_q, n_kv);
  return hipGetLastError();
}
template <typename T, int DPL>
hipError_t bwd_t(const void* qkv, const void* o, const void* dout, const float* lse, void* dqkv, float* ws, int seq,
                 int batch, int n_q, int n_kv, hipStream_t s) {
  hipLaunchKernelGGL((attn_bwd_dq_simple<T, DPL>), dim3((seq + 3) / 4, n_q, batch), dim3(256), 0, s, (const T*)qkv,
      (const T*)o, (const T*)dout, lse, (T*)dqkv, ws, seq, n_q, n_kv);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_bwd_dkv_simple<T, DPL>), dim3((seq + 3) / 4, n_kv, batch), dim3(256), 0, s, (const T*)qkv,
      (const T*)dout, lse, ws, (T*)dqkv, seq, n_q, n_kv);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_fwd_simple(int dtype, const void* qkv, void* o, float* lse, int seq, int batch, int n_q,
                                  int n_kv, int d, hipStream_t s) {
  if (dtype == DT_BF16) {
    if (d == 64) return fwd_t<bf16_t, 1>(qkv, o, lse, seq, batch, n_q, n_kv, s);
    if (d == 128) return fwd_t<bf16_t, 2>(qkv, o, lse, seq, batch, n_q, n_kv, s);
  } else {
    if (d == 64) return fwd_t<float, 1>(qkv, o, lse, seq, batch, n_q, n_kv, s);
    if (d == 128) return fwd_t<float, 2>(qkv, o, lse, seq, batch, n_q, n_kv, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_attn_bwd_simple(int dtype, const void* qkv, const void* o, const void* dout, const float* lse,
                                  void* dqkv, float* ws, int seq, int batch, int n_q, int n_kv, int d, hipStream_t s) {
  if (dtype == DT_BF16) {
    if (d == 64) return bwd_t<bf16_t, 1>(qkv, o, dout, lse, dqkv, ws, seq, batch, n_q, n_kv, s);
    if (d == 128) return bwd_t<bf16_t, 2>(qkv, o, dout, lse, dqkv, ws, seq, batch, n_q, n_kv, s);
  } else {
    if (d == 64) return bwd_t<float, 1>(qkv, o, dout, lse, dqkv, ws, seq, batch, n_q, n_kv, s);
    if (d == 128) return bwd_t<float, 2>(qkv, o, dout, lse, dqkv, ws, seq, batch, n_q, n_kv, s);
  }
  return hipErrorInvalidValue;
}
