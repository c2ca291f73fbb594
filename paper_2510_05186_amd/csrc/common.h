// Shared device/host helpers for the optstage kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>

// Raises a kernel's dynamic LDS limit, once per device (the attribute belongs to the function on one device; a
// process that drives several GPUs needs it on each).  One slot of flags per kernel at the call site.
struct LdsAttrOnce {
  std::atomic<unsigned long long> done{0};        // bit d: set on device d (devices past 63 set it on every launch)
  hipError_t ensure(const void* kernel, int bytes) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const unsigned long long bit = dev < 64 ? 1ull << dev : 0ull;
    if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess && bit) done.fetch_or(bit, std::memory_order_release);
    return e;
  }
};

typedef __bf16 bf16_t;
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

enum { DT_FP32 = 0, DT_BF16 = 1 };
enum { FAM_GPT = 0, FAM_LLAMA = 1 };

// GEMM operand layouts: C[M,N] = sum_k A(m,k) * B(n,k)
//   NT: A is [M,K] row-major, B is [N,K] row-major  (both contiguous along the contraction)
//   TN: A is [K,M] row-major, B is [K,N] row-major  (both contiguous along their output index)
// GEMM_NT_SLAB: C = A B^T with B stored in slabs of 256 rows x 64 columns, slab (n / 256, k / 64) at element offset
// ((n / 256) * (K / 64) + k / 64) * 16384, row-major inside, rows padded to a multiple of 256
enum { GEMM_NT = 0, GEMM_TN = 1, GEMM_NT_SLAB = 2 };
// epilogues: store C (stage dtype); store C + R (R like C); C (fp32) += product; C (fp32) = product;
// EPI_ROPE: store C with the q and k head columns rotated by position (rotary embedding fused into the QKV projection);
// EPI_SWIGLU: B holds the gate / up weight in paired slabs (GEMM_NT_SLAB with rows paired, see launch_slabs): stores the
// product in the plain [gate | up] layout AND a = silu(gate) * up (the MLP activation fused into the gate / up projection)
// EPI_GELU: store C and gelu(C as stored) to R, rows like C's; EPI_DGELU, EPI_DSWIGLU: the product is the gradient of the MLP
// activation's output; C holds the activation's input ([gate | up] for SwiGLU, up at column N + n) and receives its gradient
enum { EPI_STORE = 0, EPI_RESID = 1, EPI_ACCUM = 2, EPI_STOREF = 3, EPI_ROPE = 4, EPI_SWIGLU = 5, EPI_GELU = 6, EPI_DGELU = 7, EPI_DSWIGLU = 8 };
// what the two fused epilogues need beyond C: the rotary table [seq][64] (cos, sin), the sequence length (position =
// row % seq) and the number of leading columns that are q / k heads; the activation output [M, f] and f
struct GemmExtra {
  const float2* table = nullptr; int seq = 0; int rot_cols = 0;
  void* a_out = nullptr; int f = 0;
};

template <typename T> __device__ __forceinline__ float to_f32(T v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<bf16_t>(bf16_t v) { return (float)v; }
template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float v) { return (bf16_t)v; }

// MLP activations: GELU (Phi, the normal distribution) and SwiGLU = silu(gate) * up.  The sums of products are written out, so that
// every kernel rounds alike.
__device__ __forceinline__ float sigmoidf_(float x) { return 1.f / (1.f + expf(-x)); }
__device__ __forceinline__ float gelu(float x) { return 0.5f * x * (1.f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float dgelu(float x, float d) {
  const float Phi = 0.5f * (1.f + erff(x * 0.70710678118654752f));
  const float phi = 0.39894228040143268f * expf(-0.5f * x * x);
  return d * fmaf(x, phi, Phi);
}
__device__ __forceinline__ void dswiglu(float gate, float up, float d, float& dgate, float& dup) {
  const float s = sigmoidf_(gate);
  dgate = d * up * s * fmaf(gate, 1.f - s, 1.f);
  dup = d * gate * s;
}

// 16-byte vector of T (4 floats or 8 bf16) with element access in fp32
template <typename T> struct Vec16;
template <> struct Vec16<float> {
  static constexpr int N = 4;
  f32x4_t v;
  __device__ __forceinline__ float get(int i) const { return v[i]; }
  __device__ __forceinline__ void set(int i, float x) { v[i] = x; }
};
template <> struct Vec16<bf16_t> {
  static constexpr int N = 8;
  bf16x8_t v;
  __device__ __forceinline__ float get(int i) const { return (float)v[i]; }
  __device__ __forceinline__ void set(int i, float x) { v[i] = (bf16_t)x; }
};

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// launchers implemented in the .hip files; all return hipError_t from the launch
int attn_dkv_split(int seq, int batch, int n_q, int n_kv);
struct GemmProblem { const void* A; const void* B; void* C; const void* R; int M, N, lda, ldb, ldc; };
bool gemm_bf16_grouped_applies(int layout, int n, const GemmProblem* problems, int K);
hipError_t launch_gemm_bf16_grouped(int layout, int epi, int n, const GemmProblem* problems, int K, hipStream_t s);
hipError_t launch_gemm_bf16(int layout, int epi, const void* A, const void* B, void* C, const void* R, int M, int N,
                            int K, int lda, int ldb, int ldc, hipStream_t s, const GemmExtra* extra = nullptr);
// whether a product y = x W^T (dense operands) is served with the activation in its epilogue (EPI_GELU, EPI_DGELU, EPI_DSWIGLU)
bool gemm_bf16_act_applies(int M, int N, int K);
bool gemm_f32_act_applies(int M, int N, int K);
// the form that an fp32 product takes by its sizes: matrix-instruction kernel on tiles of 64 x 64, 64 x 32, 32 x 32, 16 x 32, 16 x 16 (0 - 4), plain
// kernel (5); vec: operand rows load 16 bytes at a time
int gemm_f32_form(bool tn, bool vec, int epi, int M, int N, int K, int ldc);
// tiles of 128 or 64, for products of up to 256 tiles of 128 x 128 and for what is cut off a grouped TN set; bf16 alignment rules as
// for launch_gemm_bf16
bool gemm_bf16_small_applies(int M, int N, int K, int lda, int ldb);
hipError_t launch_gemm_bf16_small(int layout, int epi, const GemmProblem& problem, int K, hipStream_t s);
bool gemm_bf16_fused_applies(int epi, int M, int N, int K, int lda, int head_dim);
hipError_t launch_gemm_f32(int layout, int epi, const void* A, const void* B, void* C, const void* R, int M, int N,
                           int K, int lda, int ldb, int ldc, hipStream_t s);
// n (up to 16) independent fp32 TN products with the same K in one launch
bool gemm_f32_grouped_applies(int n, const GemmProblem* problems, int K);
hipError_t launch_gemm_f32_grouped(int epi, int n, const GemmProblem* problems, int K, hipStream_t s);
// x_copy / dres_copy: where given, the kernel also stores the x / dres that it reads there
hipError_t launch_norm_fwd(int dtype, int family, const void* x, const void* gamma, const void* beta, void* out,
                           float* stats, int rows, int h, float eps, hipStream_t s, void* x_copy = nullptr);
hipError_t launch_norm_bwd(int dtype, int family, const void* dn, const void* x, const float* stats,
                           const void* gamma, const void* dres, void* dx, float* partial, float* dgamma,
                           float* dbeta, int rows, int h, hipStream_t s, int overwrite = 0, void* dres_copy = nullptr, bool reduce = true);
// the sums that launch_norm_bwd(reduce = false) left in `partial` of up to MAX norms of the same rows and h, in one launch
struct NormReduce {
  static constexpr int MAX = 8;
  const float* partial[MAX];
  float* dgamma[MAX];
  float* dbeta[MAX];
  int n;
};
hipError_t launch_norm_reduce(int family, const NormReduce& list, int rows, int h, int overwrite, hipStream_t s);
int norm_bwd_partial_rows(int rows);
hipError_t launch_act_fwd(int dtype, int family, const void* gu, void* a, int rows, int f, hipStream_t s);
hipError_t launch_act_bwd(int dtype, int family, const void* da, const void* gu, void* dgu, int rows, int f,
                          hipStream_t s);
hipError_t launch_rope_table(float* table, int seq, int d, float base, hipStream_t s);
hipError_t launch_rope(int dtype, const void* src, void* dst, const float* table, int rows, int seq, int n_q, int n_kv,
                       int d, int backward, int do_rotate, hipStream_t s);
hipError_t launch_transpose(int dtype, const void* src, void* dst, int rows, int cols, hipStream_t s);
// bf16 weight into the slab layout of GEMM_NT_SLAB: B[n][k] = src[n * K + k], or src[k * N + n] when transposed = 1.
// transposed = 2 (paired): src is a [gate | up] weight of N = 2 f rows; slab row 256 t + 128 w + 64 q + o holds source
// row q f + 128 t + 64 w + o, so that each wave of an output tile owns 64 gate columns and the 64 matching up columns
// (f % 128 == 0)
hipError_t launch_slabs(const void* src, void* dst, int N, int K, int transposed, hipStream_t s);
bool gemm_bf16_slab_applies(int M, int N, int K, int lda);
// up to MAX copies of 16-byte units in one launch, between memory that the device can address
struct CopyList {
  static constexpr int MAX = 10;
  const void* src[MAX];
  void* dst[MAX];
  unsigned long long units[MAX];
  int n;
};
hipError_t launch_copy_list(const CopyList& list, hipStream_t s);
hipError_t launch_checksum(const void* buf, uint64_t bytes, uint64_t* out_dev, hipStream_t s);
hipError_t launch_attn_fwd(int dtype, const void* qkv, void* o, float* lse, int seq, int batch, int n_q, int n_kv,
                           int d, hipStream_t s);
// ws: fp32 scratch of attn_bwd_ws_floats() elements
hipError_t launch_attn_bwd(int dtype, const void* qkv, const void* o, const void* dout, const float* lse, void* dqkv,
                           float* ws, int seq, int batch, int n_q, int n_kv, int d, hipStream_t s);
// the same with the gradient written over qkv, rotated back where a rotary table is given; qcopy: scratch for rows x n_q x d elements of
// the storage type.  Which calls it serves: attn_bwd_inplace_applies
bool attn_bwd_inplace_applies(int dtype, int d, int seq, int batch, int n_q, int n_kv, const void* qkv, const void* o, const void* dout,
                              const void* qcopy);
hipError_t launch_attn_bwd_inplace(int dtype, void* qkv, const void* o, const void* dout, const float* lse, void* qcopy, const float* rope_table,
                                   float* ws, int seq, int batch, int n_q, int n_kv, int d, hipStream_t s);
uint64_t attn_bwd_ws_floats(int seq, int batch, int n_q, int n_kv, int d);
// heads of 64: how many groups of waves share the keys of a dK / dV workgroup
int attn_d64_key_groups(int seq, int batch, int n_q, int n_kv);
