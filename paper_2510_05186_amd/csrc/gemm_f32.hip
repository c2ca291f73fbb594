// fp32 GEMM of the fp32 workload: C[M,N] = sum_k A(m,k) * B(n,k) with the same layouts and epilogues as the bf16 kernels
// (Sec. 2.2: Y = X W^T, dX = dY W, dW += dY^T X), on the fp32 matrix instruction v_mfma_f32_16x16x4_f32 (fp32 products and sums).
//
// What bounds it: an fp32 MFMA does 64 flop per cycle and SIMD, so operands are cheap to feed and what counts is how many compute
// units have work.  A workgroup owns an RM x RN tile (64 x 64 to 16 x 16, see pick_tile), its four waves split the contraction in
// steps of 16 k (wave w takes the steps w, w + 4, ...) and the four partial tiles are added through LDS in wave order.  No
// operand is shared between waves, so nothing is staged through LDS: every lane loads its part of the fragments straight into
// registers, 16 bytes at a time, several steps ahead (DEPTH), and the loop has no barrier.
//  * NT (contiguous along k): lane = row (lane & 15), 4 consecutive k at 4 (lane >> 4); element e of the four goes to MFMA e of
//    the step, the same k on both sides.  One load is 16 rows of 64 bytes.
//  * TN (contiguous along the output index): a lane loads T = rows / 16 consecutive rows (columns) T r .. of one k, r = lane & 15,
//    and element i belongs to MFMA tile i: tile i holds the rows T r + i, which costs nothing but the index in the epilogue.
//    One load is 4 k-rows of 4 RM (RN) bytes.
// Loads go through the buffer range check: rows past the operand and, by a lane offset out of range, k past K read as zero.
// The loads ahead only help if every step waits for its own: the vectors that come back are kept as they are (as single floats, the
// compiler copied them all at the top of the loop, behind one wait for every load in flight) and each step's loads are fenced in behind its
// MFMAs.  That and the 64 x 32 and 16 x 32 tiles, us: NT 512 x 1024 x 4096 62.7 -> 45.5, 512 x 1024 x 1024 19.8 -> 14.2, 512 x 4096 x 1024 45.4 -> 40.2,
// 128 x 768 x 256 4.9 -> 3.8, 2048 x 2048 x 2048 154 -> 138 (124 TFLOP/s); TN 1024 x 4096 x 512 45.8 -> 42.0; 80 products drawn between 100 and 2048
// 1.26x (geometric mean; least .98, of 4 us).
#include "common.h"

namespace {

typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
constexpr unsigned OUT_OF_RANGE = 0xFFFFFF00u;
constexpr int STEP = 16;                                     // k per step

// One operand: R rows of the tile (RM or RN) by 16 k per step, T = R / 16 MFMA tiles
template <int R, bool TNL, bool VEC> struct Operand {
  static constexpr int T = R / 16;
  __amdgpu_buffer_rsrc_t rsrc;
  unsigned off[T];             // NT: row 16 i + r of the tile at this lane's k; TN: off[0] = this lane's rows at k-row g
  unsigned kstep;              // bytes per k
  int k0;                      // first k of this lane within a step

  __device__ __forceinline__ void init(const float* p, int ld, int first, int extent, int K, int lane) {
    const int r = lane & 15, g = lane >> 4;
    const float* base = TNL ? p + first : p + (size_t)first * ld;
    const unsigned long long bytes = TNL ? ((unsigned long long)(K - 1) * ld + extent - first) * 4
                                         : ((unsigned long long)(extent - 1 - first) * ld + K) * 4;
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, (int)(unsigned)(bytes > OUT_OF_RANGE ? OUT_OF_RANGE : bytes), 0x00020000);
    if constexpr (TNL) {
      k0 = g;                                                // rows g, g + 4, g + 8, g + 12 of a step
      kstep = (unsigned)ld * 4u;
      off[0] = first + r * T < extent ? (unsigned)(r * T) * 4u : OUT_OF_RANGE;
    } else {
      k0 = 4 * g;
      kstep = 4u;
#pragma unroll
      for (int i = 0; i < T; ++i) off[i] = first + i * 16 + r < extent ? (unsigned)(i * 16 + r) * (unsigned)ld * 4u : OUT_OF_RANGE;
    }
  }
  __device__ __forceinline__ float one(unsigned o) const {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, o, 0, 0));
  }
  // A step's operands as they are loaded: NT a vector of four k per MFMA tile, TN a vector of the lane's T rows per k
  struct Frag {
    typedef float vec_t __attribute__((ext_vector_type(TNL ? (T == 1 ? 2 : T) : 4)));   // T = 1: the second element is not used
    vec_t v[TNL ? 4 : T];
    // operand of MFMA e (k-set e) of tile i
    __device__ __forceinline__ float get(int i, int e) const { return TNL ? v[e][i] : v[i][e]; }
  };
  __device__ __forceinline__ void load(Frag& f, int k, int K, int rows_left) const {
    if constexpr (TNL) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int kk = k + k0 + 4 * e;
        const unsigned o = kk < K && off[0] != OUT_OF_RANGE ? off[0] + (unsigned)kk * kstep : OUT_OF_RANGE;
        if constexpr (VEC && T == 4) {
          f.v[e] = __builtin_bit_cast(typename Frag::vec_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc, o, 0, 0));
        } else if constexpr (VEC && T == 2) {
          f.v[e] = __builtin_bit_cast(typename Frag::vec_t, __builtin_amdgcn_raw_buffer_load_b64(rsrc, o, 0, 0));
        } else {
#pragma unroll
          for (int i = 0; i < T; ++i) f.v[e][i] = one(o != OUT_OF_RANGE && i < rows_left ? o + i * 4u : OUT_OF_RANGE);
        }
      }
    } else {
      const int kk = k + k0;
#pragma unroll
      for (int i = 0; i < T; ++i) {
        if constexpr (VEC) {                                 // K % 4 == 0: the four k are inside or outside together
          const unsigned o = kk < K && off[i] != OUT_OF_RANGE ? off[i] + (unsigned)kk * 4u : OUT_OF_RANGE;
          f.v[i] = __builtin_bit_cast(typename Frag::vec_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc, o, 0, 0));
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            f.v[i][e] = one(kk + e < K && off[i] != OUT_OF_RANGE ? off[i] + (unsigned)(kk + e) * 4u : OUT_OF_RANGE);
        }
      }
    }
  }
};

template <int RM, int RN, bool TNL, bool VEC>
__device__ __forceinline__ void f32_tile(const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ C,
                                         const float* __restrict__ Res, int M, int N, int K, int lda, int ldb, int ldc, int id,
                                         int tiles_m, int tiles_n, int epi) {
  constexpr int TA = RM / 16, TB = RN / 16, DEPTH = TA * TB >= 16 ? 2 : TA * TB >= 8 ? 3 : TA * TB >= 4 ? 4 : 8;
  __shared__ __attribute__((aligned(16))) float part[4][RM][RN + 4];
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // consecutive workgroup ids go to different XCDs: every XCD takes one contiguous eighth of the tiles, row by row
  const int n_tiles = tiles_m * tiles_n;
  if ((n_tiles & 7) == 0) id = (id & 7) * (n_tiles >> 3) + (id >> 3);
  const int m0 = (id / tiles_n) * RM, n0 = (id % tiles_n) * RN;
  Operand<RM, TNL, VEC> a;
  Operand<RN, TNL, VEC> b;
  a.init(A, lda, m0, M, K, lane);
  b.init(B, ldb, n0, N, K, lane);
  const int a_left = TNL ? M - m0 - r * TA : 0, b_left = TNL ? N - n0 - r * TB : 0;   // rows of this lane inside the operand
  f32x4_t acc[TA][TB];
#pragma unroll
  for (int i = 0; i < TA; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  typename Operand<RM, TNL, VEC>::Frag av[DEPTH];
  typename Operand<RN, TNL, VEC>::Frag bv[DEPTH];
  const int steps = (K + STEP - 1) / STEP, count = (steps - wave + 3) >> 2;   // this wave's steps: wave + 4 s
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) {
    __builtin_amdgcn_sched_barrier(0);
    a.load(av[d], (wave + 4 * d) * STEP, K, a_left);
    b.load(bv[d], (wave + 4 * d) * STEP, K, b_left);
  }
  auto multiply = [&](int d) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j)
          // in assembly the sums stay where they are: of the builtin's results the compiler moves all to other registers and back, every time
          // round.  Its operands come straight from loads; no vector instruction writes them
          if constexpr (VEC) asm volatile("v_mfma_f32_16x16x4_f32 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(bv[d].get(j, e)), "v"(av[d].get(i, e)));
          else acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv[d].get(j, e), av[d].get(i, e), acc[i][j], 0, 0, 0);
  };
  if constexpr (VEC) {                                       // the zeros are in place, some cycles ahead of the first product
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int j = 0; j < TB; ++j) asm volatile("" : "+a"(acc[i][j]));
    asm volatile("s_nop 3" ::: "memory");
  }
  int s = 0;
  for (; s + DEPTH <= count; s += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      // a step's loads stay behind its MFMAs: left alone the compiler gathers those of all DEPTH steps at the end of the loop, right ahead of
      // one wait for all of them
      __builtin_amdgcn_sched_barrier(0);
      multiply(d);
      __builtin_amdgcn_sched_barrier(0);
      a.load(av[d], (wave + 4 * (s + d + DEPTH)) * STEP, K, a_left);
      b.load(bv[d], (wave + 4 * (s + d + DEPTH)) * STEP, K, b_left);
    }
  }
#pragma unroll
  for (int d = 0; d < DEPTH - 1; ++d)                        // the steps left over are loaded
    if (s + d < count) multiply(d);
  if constexpr (VEC) asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");   // the last results have left the matrix unit
  // partial tiles into LDS in the order of C: acc[i][j][v] is row r of tile i, column 4 g + v of tile j
#pragma unroll
  for (int i = 0; i < TA; ++i) {
    const int row = TNL ? TA * r + i : 16 * i + r;
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      if constexpr (TNL) {
#pragma unroll
        for (int v = 0; v < 4; ++v) part[wave][row][TB * (4 * g + v) + j] = acc[i][j][v];
      } else {
        *reinterpret_cast<f32x4_t*>(&part[wave][row][16 * j + 4 * g]) = acc[i][j];
      }
    }
  }
  __syncthreads();
  // RM * RN / 4 pieces of four columns over 256 threads, partial tiles added in wave order
  for (int q = tid; q < RM * RN / 4; q += 256) {
    const int row = q / (RN / 4), col = (q % (RN / 4)) * 4, m = m0 + row, n = n0 + col;
    f32x4_t v = *reinterpret_cast<const f32x4_t*>(&part[0][row][col]);
#pragma unroll
    for (int p = 1; p < 4; ++p) {
      const f32x4_t o = *reinterpret_cast<const f32x4_t*>(&part[p][row][col]);
      v[0] += o[0]; v[1] += o[1]; v[2] += o[2]; v[3] += o[3];
    }
    if (m >= M || n >= N) continue;
    float* dst = C + (size_t)m * ldc + n;
    if (epi >= EPI_GELU) {                                   // N and ldc are multiples of four
      f32x4_t o;
      if (epi == EPI_GELU) {
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = gelu(v[e]);
        *reinterpret_cast<f32x4_t*>(dst) = v;
        *reinterpret_cast<f32x4_t*>(const_cast<float*>(Res) + (size_t)m * ldc + n) = o;
        continue;
      }
      const f32x4_t x = *reinterpret_cast<const f32x4_t*>(dst);
      if (epi == EPI_DGELU) {
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = dgelu(x[e], v[e]);
      } else {
        const f32x4_t u = *reinterpret_cast<const f32x4_t*>(dst + N);
        f32x4_t du;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float dg, d1;
          dswiglu(x[e], u[e], v[e], dg, d1);
          o[e] = dg;
          du[e] = d1;
        }
        *reinterpret_cast<f32x4_t*>(dst + N) = du;
      }
      *reinterpret_cast<f32x4_t*>(dst) = o;
      continue;
    }
    const float* add = epi == EPI_RESID ? Res + (size_t)m * ldc + n : epi == EPI_ACCUM ? dst : nullptr;
    if (n + 4 <= N && (ldc & 3) == 0) {
      if (add) { const f32x4_t o = *reinterpret_cast<const f32x4_t*>(add); v[0] += o[0]; v[1] += o[1]; v[2] += o[2]; v[3] += o[3]; }
      *reinterpret_cast<f32x4_t*>(dst) = v;
    } else {
      for (int e = 0; e < 4 && n + e < N; ++e) dst[e] = add ? v[e] + add[e] : v[e];
    }
  }
}

template <int RM, int RN, bool TNL, bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_mfma_kernel(const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ C,
                                                            const float* __restrict__ Res, int M, int N, int K, int lda, int ldb,
                                                            int ldc, int tiles_m, int tiles_n, int epi) {
  f32_tile<RM, RN, TNL, VEC>(A, B, C, Res, M, N, K, lda, ldb, ldc, blockIdx.x, tiles_m, tiles_n, epi);
}

// The weight-gradient products of a W op in one launch: none depends on another, and at a few hundred tokens each is a launch
// of 5 us that leaves most of the compute units idle (W of the two-layer hidden-256 stage: eight launches 44 us, one 15).
constexpr int MAX_GROUP = 16;
struct GroupedF32 { const float* A; const float* B; float* C; int M, N, lda, ldb, ldc, tiles_m, tiles_n, first; };
struct GroupedF32Args { int n, K, epi; GroupedF32 p[MAX_GROUP]; };
template <int RM, int RN>
__global__ __launch_bounds__(256) void gemm_f32_grouped_tn_kernel(const GroupedF32Args g) {
  int q = 0;
  for (int i = 1; i < g.n; ++i)
    if ((int)blockIdx.x >= g.p[i].first) q = i;
  const GroupedF32& p = g.p[q];
  f32_tile<RM, RN, true, true>(p.A, p.B, p.C, p.C /* no residual; a null constant here crashes the compiler */, p.M, p.N, g.K, p.lda, p.ldb, p.ldc, blockIdx.x - p.first, p.tiles_m, p.tiles_n, g.epi);
}

// General path: 64 x 64 tile through LDS, 256 threads, 4 x 4 outputs per thread, any strides.  Takes what 32-bit offsets within
// a tile do not reach, and short contractions of many tiles (plain_is_faster).
template <int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ B,
                                                       float* __restrict__ C, const float* __restrict__ R, int M, int N,
                                                       int K, long sam, long sak, long sbn, long sbk, int ldc) {
  constexpr int T = 64, KT = 16;
  __shared__ float As[KT][T + 4];
  __shared__ float Bs[KT][T + 4];
  const int tid = threadIdx.x;
  const int m0 = blockIdx.y * T, n0 = blockIdx.x * T;
  const int ty = tid >> 4, tx = tid & 15;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += KT) {
    for (int e = tid; e < T * KT; e += 256) {
      int r, k;
      if (sak == 1) { r = e / KT; k = e % KT; } else { r = e % T; k = e / T; }   // walk the contiguous index fastest
      int gm = m0 + r, gk = k0 + k;
      As[k][r] = (gm < M && gk < K) ? A[gm * sam + gk * sak] : 0.f;
    }
    for (int e = tid; e < T * KT; e += 256) {
      int r, k;
      if (sbk == 1) { r = e / KT; k = e % KT; } else { r = e % T; k = e / T; }
      int gn = n0 + r, gk = k0 + k;
      Bs[k][r] = (gn < N && gk < K) ? B[gn * sbn + gk * sbk] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < KT; ++k) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[k][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[k][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int m = m0 + ty * 4 + i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int n = n0 + tx * 4 + j;
      if (n >= N) continue;
      size_t off = (size_t)m * ldc + n;
      float v = acc[i][j];
      if (EPI == EPI_RESID) v += R[off];
      if (EPI == EPI_ACCUM) v += C[off];
      C[off] = v;
    }
  }
}


template <int RM, int RN, bool TNL, bool VEC>
hipError_t launch_mfma(int epi, const float* A, const float* B, float* C, const float* R_, int M, int N, int K, int lda, int ldb,
                       int ldc, hipStream_t s) {
  const int tiles_m = (M + RM - 1) / RM, tiles_n = (N + RN - 1) / RN;
  hipLaunchKernelGGL((gemm_f32_mfma_kernel<RM, RN, TNL, VEC>), dim3((unsigned)tiles_m * (unsigned)tiles_n), dim3(256), 0, s, A, B, C, R_,
                     M, N, K, lda, ldb, ldc, tiles_m, tiles_n, epi);
  return hipGetLastError();
}

// The tile that needs the least time.  Workgroups come to the compute units evenly, n = ceil(tiles / 256) to the fullest, and share its matrix
// units: start, first loads and epilogue once, and n contractions.  Both from 256 and 1024 k and one to eight workgroups per unit, us:
// 512 x 4096 x 1024 40.1 in tiles of 64 x 64, 48.0 of 64 x 32, 61.3 of 32 x 32; 512 x 3072 x 1024 39.4 / 37.0 / 46.8; 512 x 1024 x 4096 65.7 / 45.3 /
// 58.9; 512 x 1024 x 1024 20.0 / 14.2 / 17.4; 128 x 768 x 256 8.2 / 5.7 / 4.3, of 16 x 32 3.7, of 16 x 16 4.1; 128 x 256 x 1024 19.7 / 13.7 / 9.4 / 7.8 / 5.9.
struct TileShape { int rows, cols; double start_us, first_ns, next_ns; };   // ns per k: a unit's only workgroup, each of several
constexpr TileShape TILES[] = {{64, 64, 4.0, 16.8, 16.8}, {64, 32, 3.0, 10.9, 11.2}, {32, 32, 2.6, 6.8, 7.2}, {16, 32, 2.6, 5.0, 5.7}, {16, 16, 2.6, 2.6, 3.75}};
int pick_tile(int n, const GemmProblem* pr, int K) {
  int best = 0;
  double least = 1e30;
  for (int t = 0; t < 5; ++t) {
    const TileShape& s = TILES[t];
    long long tiles = 0;
    for (int i = 0; i < n; ++i) tiles += (long long)((pr[i].M + s.rows - 1) / s.rows) * ((pr[i].N + s.cols - 1) / s.cols);
    const double us = s.start_us + 1e-3 * K * (tiles <= 256 ? s.first_ns : (double)((tiles + 255) / 256) * s.next_ns);
    if (us < least) { least = us; best = t; }
  }
  return best;
}

template <bool TNL, bool VEC>
hipError_t launch_sized(int epi, const float* A, const float* B, float* C, const float* R, int M, int N, int K, int lda, int ldb,
                        int ldc, hipStream_t s) {
  const GemmProblem pr = {A, B, C, R, M, N, lda, ldb, ldc};
  switch (pick_tile(1, &pr, K)) {
    case 0: return launch_mfma<64, 64, TNL, VEC>(epi, A, B, C, R, M, N, K, lda, ldb, ldc, s);
    case 1: return launch_mfma<64, 32, TNL, VEC>(epi, A, B, C, R, M, N, K, lda, ldb, ldc, s);
    case 2: return launch_mfma<32, 32, TNL, VEC>(epi, A, B, C, R, M, N, K, lda, ldb, ldc, s);
    case 3: return launch_mfma<16, 32, TNL, VEC>(epi, A, B, C, R, M, N, K, lda, ldb, ldc, s);
    default: return launch_mfma<16, 16, TNL, VEC>(epi, A, B, C, R, M, N, K, lda, ldb, ldc, s);
  }
}

// With a contraction of one or two steps of 16 the four waves have little to share, and adding their partial tiles through LDS costs more
// than the products: what is left is the writing of C, which the plain kernel does at once where there are many tiles.  Operands that do not
// load, or a C that does not store, 16 bytes at a time (vec = false) move that point up.  Time of the matrix-instruction kernel over the plain one:
//  vec   NT 8192 tiles of 64 (8192 x 4096), K 16 / 32 / 40 1.10 / 1.05 / .83; 2048 tiles, K 8 / 32 .81 / .94; 1024 tiles, K 8 .95; 384 tiles .75
//        TN 8192 tiles, K 16 / 32 / 40 1.11 / 1.01 / .87; 2048 tiles, K 8 / 16 / 32 1.11 / 1.04 / .84; 1024 tiles 1.59 / 1.01 / .81; 384 tiles 1.11 / 1.05 / .82;
//        28 tiles, K 4 / 16 .93 / .81 (accumulating, the old values are read in either kernel: .7 - .86)
//  else  NT 560 tiles (1760 x 1262), K 6 / 17 / 41 1.09 / 1.01 / .99; 256 tiles, K 6 .89
//        TN 560 tiles, K 6 / 17 / 41 1.27 / 1.12 / .96; 256 tiles, K 6 / 17 1.22 / .94
bool plain_is_faster(bool tn, bool vec, int epi, long tiles64, int K) {
  if (tn && epi == EPI_ACCUM) return vec ? K <= 32 && tiles64 >= 4096 : K <= 24 && tiles64 >= 512;
  if (tn) return vec ? K <= 16 ? tiles64 >= 256 : K <= 32 && tiles64 >= 4096 : K <= 12 ? tiles64 >= 128 : K <= 24 && tiles64 >= 512;
  return vec ? K <= 32 && tiles64 >= 4096 : K <= 12 && tiles64 >= 512;
}
long tiles64_of(int n, const GemmProblem* pr) {
  long tiles = 0;
  for (int i = 0; i < n; ++i) tiles += (long)((pr[i].M + 63) / 64) * ((pr[i].N + 63) / 64);
  return tiles;
}

}  // namespace

namespace {
// lane offsets of the matrix-instruction kernels: NT 64 rows of a tile, TN all k-rows of the operand's column strip
bool mfma_reaches(bool tn, int K, int lda, int ldb) {
  const unsigned long long reach = 0xF0000000ull / 4;
  const unsigned long long span = (unsigned long long)(tn ? K + 64ull * 16 : 64ull) * (unsigned long long)(lda > ldb ? lda : ldb) + 64;
  return span < reach && (tn || (unsigned long long)K < reach / 2);
}

template <int RM, int RN>
hipError_t launch_grouped(int epi, int n, const GemmProblem* pr, int K, hipStream_t s) {
  GroupedF32Args g;
  g.n = n; g.K = K; g.epi = epi;
  int total = 0;
  for (int i = 0; i < n; ++i) {
    const int tm = (pr[i].M + RM - 1) / RM, tn = (pr[i].N + RN - 1) / RN;
    g.p[i] = {(const float*)pr[i].A, (const float*)pr[i].B, (float*)pr[i].C, pr[i].M, pr[i].N, pr[i].lda, pr[i].ldb, pr[i].ldc, tm, tn, total};
    total += tm * tn;
  }
  hipLaunchKernelGGL((gemm_f32_grouped_tn_kernel<RM, RN>), dim3(total), dim3(256), 0, s, g);
  return hipGetLastError();
}
}  // namespace

bool gemm_f32_grouped_applies(int n, const GemmProblem* pr, int K) {
  if (n < 1 || n > MAX_GROUP || K <= 0) return false;
  for (int i = 0; i < n; ++i)
    if (pr[i].M <= 0 || pr[i].N <= 0 || ((pr[i].lda | pr[i].ldb | pr[i].M | pr[i].N) & 3) || !mfma_reaches(true, K, pr[i].lda, pr[i].ldb)) return false;
  return !plain_is_faster(true, true, EPI_ACCUM, tiles64_of(n, pr), K);
}

// n independent TN products with the same K: C (fp32) += product (EPI_ACCUM) or = product
hipError_t launch_gemm_f32_grouped(int epi, int n, const GemmProblem* pr, int K, hipStream_t s) {
  if (!gemm_f32_grouped_applies(n, pr, K) || (epi != EPI_ACCUM && epi != EPI_STOREF)) return hipErrorInvalidValue;
  switch (pick_tile(n, pr, K)) {
    case 0: return launch_grouped<64, 64>(epi, n, pr, K, s);
    case 1: return launch_grouped<64, 32>(epi, n, pr, K, s);
    case 2: return launch_grouped<32, 32>(epi, n, pr, K, s);
    case 3: return launch_grouped<16, 32>(epi, n, pr, K, s);
    default: return launch_grouped<16, 16>(epi, n, pr, K, s);
  }
}

// The activation's epilogues are in the matrix-instruction kernels only
bool gemm_f32_act_applies(int M, int N, int K) {
  if (M <= 0 || N <= 0 || K <= 0 || (N & 3) || !mfma_reaches(false, K, K, K)) return false;
  const GemmProblem pr = {nullptr, nullptr, nullptr, nullptr, M, N, K, K, N};
  return !((K & 3) == 0 && plain_is_faster(false, true, EPI_STORE, tiles64_of(1, &pr), K)) &&
         !((K & 3) && plain_is_faster(false, false, EPI_STORE, tiles64_of(1, &pr), K));
}

hipError_t launch_gemm_f32(int layout, int epi, const void* A, const void* B, void* C, const void* R, int M, int N,
                           int K, int lda, int ldb, int ldc, hipStream_t s) {
  if (M <= 0 || N <= 0 || K <= 0) return hipErrorInvalidValue;
  if ((layout != GEMM_NT && layout != GEMM_TN) || epi < EPI_STORE || epi > EPI_DSWIGLU || epi == EPI_ROPE || epi == EPI_SWIGLU)
    return hipErrorInvalidValue;
  if (epi >= EPI_GELU && (layout != GEMM_NT || lda != K || ldb != K || (ldc & 3) || !gemm_f32_act_applies(M, N, K))) return hipErrorInvalidValue;
  const bool tn = layout == GEMM_TN;
  const float *a = (const float*)A, *b = (const float*)B, *r = (const float*)R;
  float* c = (float*)C;
  const GemmProblem pr = {A, B, C, R, M, N, lda, ldb, ldc};
  const bool vec = (lda & 3) == 0 && (ldb & 3) == 0 && (tn ? (M & 3) == 0 && (N & 3) == 0 : (K & 3) == 0);
  const bool plain = epi < EPI_GELU && plain_is_faster(tn, vec && (ldc & 3) == 0, epi, tiles64_of(1, &pr), K) && (M + 63) / 64 < 65536;   // the second dimension of its grid
  if (!plain && mfma_reaches(tn, K, lda, ldb)) {
    if (tn) return vec ? launch_sized<true, true>(epi, a, b, c, r, M, N, K, lda, ldb, ldc, s)
                       : launch_sized<true, false>(epi, a, b, c, r, M, N, K, lda, ldb, ldc, s);
    return vec ? launch_sized<false, true>(epi, a, b, c, r, M, N, K, lda, ldb, ldc, s)
               : launch_sized<false, false>(epi, a, b, c, r, M, N, K, lda, ldb, ldc, s);
  }
  const long sam = tn ? 1 : lda, sak = tn ? lda : 1, sbn = tn ? 1 : ldb, sbk = tn ? ldb : 1;
  dim3 grid((N + 63) / 64, (M + 63) / 64), block(256);
  if (epi == EPI_RESID) hipLaunchKernelGGL(gemm_f32_kernel<EPI_RESID>, grid, block, 0, s, a, b, c, r, M, N, K, sam, sak, sbn, sbk, ldc);
  else if (epi == EPI_ACCUM) hipLaunchKernelGGL(gemm_f32_kernel<EPI_ACCUM>, grid, block, 0, s, a, b, c, r, M, N, K, sam, sak, sbn, sbk, ldc);
  else hipLaunchKernelGGL(gemm_f32_kernel<EPI_STORE>, grid, block, 0, s, a, b, c, r, M, N, K, sam, sak, sbn, sbk, ldc);
  return hipGetLastError();
}
