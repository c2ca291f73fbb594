// fp32 GEMM of the fp32 workload: C[M,N] = sum_k A(m,k) * B(n,k) with the same layouts and epilogues as the bf16 kernels
// (Sec. 2.2: Y = X W^T, dX = dY W, dW += dY^T X), on the fp32 matrix instruction v_mfma_f32_16x16x4_f32 (fp32 products and sums).
//
// What bounds it: an fp32 MFMA does 64 flop per cycle and SIMD, so operands are cheap to feed and what counts is how many compute
// units have work, and that nothing is issued while no MFMA runs.  A workgroup owns an RM x RN tile (64 x 64 to 16 x 16, see pick_form), its
// four waves split the contraction in steps of 16 k (wave w takes the steps w, w + 4, ...) and the four partial tiles are added through LDS
// in wave order.  No operand is shared between waves, so the loop has no barrier.
//  * NT (contiguous along k) with 16-byte rows: loads go straight into a ring in LDS, each wave's its own (staged_loop).
//  * TN (contiguous along the output index): into registers, several steps ahead (DEPTH).  A lane loads T = rows / 16 consecutive
//    rows (columns) T r .. of one k, r = lane & 15, and element i belongs to MFMA tile i: tile i holds the rows T r + i, which costs
//    nothing but the index in the epilogue.  One load is 4 k-rows of 4 RM (RN) bytes.
//  * rows that do not load 16 bytes at a time: the same into registers, element by element.
// Loads go through the buffer range check: rows past the operand and k past K read as zero.
// An MFMA takes 32 cycles and leaves room for other instructions of its wave, but only for those that stand between it and the next:
// with a step's loads and their address arithmetic (some 90 instructions) in one place behind its MFMAs, 512 x 1024 x 4096 kept the matrix units
// busy for 64 % of the time.  Now the loads and reads stand one by one between the MFMAs, their addresses are a scalar offset, and NT rows
// go through LDS, where 16 lanes fetch four rows instead of sixteen (4 % of it).  us, before -> after: NT 512 x 1024 x 4096 45.7 -> 39.4,
// 512 x 3072 x 1024 37.1 -> 32.4, 2048 x 2048 x 2048 135 -> 129 (133 TFLOP/s), 333 x 1000 x 512 8.7 -> 7.8, 128 x 256 x 1024 5.9 -> 4.6; TN 1024 x 1024 x
// 1024 20.9 -> 19.1, 4096 x 1024 x 512 40.2 -> 38.5, 2048 x 2048 x 2048 134 -> 123.
// The sums keep their registers and every step waits for its own loads: the vectors that come back are kept as they are (as single
// floats the compiler copied them all at the top of the loop, behind one wait for every load in flight).
#include <algorithm>
#include <utility>

#include "common.h"

namespace {

typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
constexpr unsigned OUT_OF_RANGE = 0xFFFFFF00u;
constexpr int STEP = 16;                                     // k per step
// slots of a wave's ring: some 2000 cycles of MFMAs ahead (TA * TB of 128 cycles per step) within the LDS of two workgroups per compute unit
constexpr int ring_slots(int rm, int rn) { return rm * rn >= 4096 ? 2 : rm * rn >= 2048 ? 3 : rm * rn >= 1024 ? 4 : rm * rn >= 512 ? 6 : 8; }

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
      if constexpr (VEC) {                                   // for load_k: rows past the end take others in their place, and no sum of theirs is stored
        if (off[0] == OUT_OF_RANGE) off[0] = 0;
        off[0] += (unsigned)g * kstep;
      }
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
  // TN, 16-byte rows: k-set e of the step at k.  k-rows past K lie past the operand and read as zero: the range check adds the scalar offset to the
  // lane's, also where the scalar one is past the end by itself.
  __device__ __forceinline__ void load_k(Frag& f, int k, int e) const {
    const unsigned at = (unsigned)(k + 4 * e) * kstep;
    if constexpr (T == 4) f.v[e] = __builtin_bit_cast(typename Frag::vec_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off[0], at, 0));
    else if constexpr (T == 2) f.v[e] = __builtin_bit_cast(typename Frag::vec_t, __builtin_amdgcn_raw_buffer_load_b64(rsrc, off[0], at, 0));
    else f.v[e][0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, off[0], at, 0));
  }
  __device__ __forceinline__ void load(Frag& f, int k, int K, int rows_left) const {
    if constexpr (TNL && VEC) {
#pragma unroll
      for (int e = 0; e < 4; ++e) load_k(f, k, e);
    } else if constexpr (TNL) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int kk = k + k0 + 4 * e;
        const unsigned o = kk < K && off[0] != OUT_OF_RANGE ? off[0] + (unsigned)kk * kstep : OUT_OF_RANGE;
#pragma unroll
        for (int i = 0; i < T; ++i) f.v[e][i] = one(o != OUT_OF_RANGE && i < rows_left ? o + i * 4u : OUT_OF_RANGE);
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

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(3))) f32x4_t lds_f32x4_t;
typedef int i32x4_t __attribute__((ext_vector_type(4)));

// One NT operand by way of LDS: R rows of the tile, a step (64 bytes of each row) per slot, in the wave's own ring.  A load
// takes 16 rows, four lanes to a row; the 16-byte chunk that lands at place p of its row is p ^ (row / 4 % 4), so that the 16 rows at
// one k that an MFMA operand reads fall on all banks.
template <int R> struct Staged {
  static constexpr int T = R / 16;
  // The range check adds the scalar offset (4 k) to the lane's, and the sum wraps: PAST + 4 k has to stay past the end (mfma_reaches)
  static constexpr unsigned PAST = 0xF8000000u;
  unsigned voff[T];            // this lane's byte offset within a step
  unsigned frag;               // where it reads MFMA tile 0
  int k0;                      // first k it fetches
  i32x4_t desc;                // from the tile's corner to the operand's end: what lies past it reads as zero

  __device__ __forceinline__ void init(const float* p, int ld, int first, int extent, int K, int lane) {
    const unsigned long long at = (unsigned long long)(p + (size_t)first * ld), bytes = ((unsigned long long)(extent - 1 - first) * ld + K) * 4;
    desc[0] = __builtin_amdgcn_readfirstlane((int)(unsigned)at);
    desc[1] = __builtin_amdgcn_readfirstlane((int)(unsigned)(at >> 32) & 0xffff);
    desc[2] = __builtin_amdgcn_readfirstlane((int)(unsigned)(bytes > PAST ? PAST : bytes));
    desc[3] = 0x00020000;
    const int chunk = (lane & 3) ^ (lane >> 4);
    k0 = chunk * 4;
#pragma unroll
    for (int i = 0; i < T; ++i)
      voff[i] = first + i * 16 + (lane >> 2) < extent ? (unsigned)(i * 16 + (lane >> 2)) * (unsigned)ld * 4u + (unsigned)chunk * 16u : PAST;
    frag = (unsigned)((lane & 15) * 64 + (((lane >> 4) ^ ((lane >> 2) & 3)) << 4));
  }
  // the last step of a K that is no multiple of 16: chunks past K go out of range, for good
  __device__ __forceinline__ void cut(int k, int K) {
#pragma unroll
    for (int i = 0; i < T; ++i)
      if (k + k0 >= K) voff[i] = PAST;
  }
  __device__ __forceinline__ void issue(unsigned slot, unsigned kbytes, int i) const {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(slot + i * 1024), "v"(voff[i]), "s"(desc), "s"(kbytes) : "memory", "m0");
  }
  __device__ __forceinline__ f32x4_t read(unsigned slot, int i) const { return *(const lds_f32x4_t*)(slot + frag + i * 1024); }
};

// f(0), f(1), ...: a loop that is unrolled at any length, its index a constant
template <int... I, class F> __device__ __forceinline__ void each(std::integer_sequence<int, I...>, F f) {
  (f(std::integral_constant<int, I>{}), ...);
}

// The sums leave the matrix unit before a path ends: where paths meet, the compiler may copy them, and knows nothing of products in assembly
template <int TA, int TB> __device__ __forceinline__ void drain(f32x4_t (&acc)[TA][TB]) {
  asm volatile("s_nop 15\n\ts_nop 7" : "+a"(acc[0][0]) :: "memory");
#pragma unroll
  for (int i = 0; i < TA; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j) asm volatile("" : "+a"(acc[i][j]));
}

// acc[i][j] += this wave's share of the contraction (steps wave, wave + 4, ...)
template <int RM, int RN>
__device__ __forceinline__ void staged_loop(char* smem, f32x4_t (&acc)[RM / 16][RN / 16], const float* A, const float* B, int M, int N,
                                            int K, int lda, int ldb, int m0, int n0, int wave, int lane) {
  constexpr int TA = RM / 16, TB = RN / 16, L = TA + TB, NM = 4 * TA * TB, SLOTS = ring_slots(RM, RN), SLOT = L * 1024;
  Staged<RM> a;
  Staged<RN> b;
  a.init(A, lda, m0, M, K, lane);
  b.init(B, ldb, n0, N, K, lane);
  const unsigned ring = (unsigned)(size_t)(lds_void_t*)smem + wave * (SLOTS * SLOT);
  f32x4_t av[2][TA], bv[2][TB];
  const int steps = (K + STEP - 1) / STEP, count = (steps - wave + 3) >> 2;
  // Past its last step a wave loads the last of all again, which nobody reads: as many loads are in flight on every trip, and none
  // reaches further.
  auto first_k = [&](int n) __attribute__((always_inline)) {
    const int k = min(wave + 4 * n, steps - 1) * STEP;
    if (k + STEP > K) { a.cut(k, K); b.cut(k, K); }
    return k;
  };
  auto issue = [&](unsigned slot, int k, int l) __attribute__((always_inline)) {
    if (l < TA) a.issue(slot, k * 4u, l); else b.issue(slot + TA * 1024, k * 4u, l - TA);
  };
  auto read = [&](int set, unsigned slot, int q) __attribute__((always_inline)) {
    if (q < TA) av[set][q] = a.read(slot, q); else bv[set][q - TA] = b.read(slot + TA * 1024, q - TA);
  };
#pragma unroll
  for (int u = 0; u < SLOTS; ++u) {
    const int k = first_k(u);
#pragma unroll
    for (int l = 0; l < L; ++l) issue(ring + u * SLOT, k, l);
  }
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"((SLOTS - 1) * L) : "memory");
#pragma unroll
  for (int q = 0; q < L; ++q) read(0, ring, q);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  {
    const int k = first_k(SLOTS);
#pragma unroll
    for (int l = 0; l < L; ++l) issue(ring, k, l);
  }
  unsigned slot = ring;
  // A step: its MFMAs (fragment set `set`) in the order written.  Between those of the first half the next step's fragments are
  // read, which have landed; between the others the slot that they have left is filled again.
  auto trip = [&](int set, int n) __attribute__((always_inline)) {
    slot = slot + SLOT == ring + SLOTS * SLOT ? ring : slot + SLOT;
    const int k = first_k(n + 1 + SLOTS);
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"((SLOTS - 1) * L) : "memory");
    each(std::make_integer_sequence<int, NM>(), [&](auto at) __attribute__((always_inline)) {
      constexpr int t = decltype(at)::value, H = NM / 2;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < L; ++q)
        if (q * H / L == t) read(set ^ 1, slot, q);
      if (t == H) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int l = 0; l < L; ++l)
        if (H + l * H / L == t) issue(slot, k, l);
      __builtin_amdgcn_sched_barrier(0);
      constexpr int e = t / (TA * TB), i = t / TB % TA, j = t % TB;
      // in assembly the sums stay where they are (see f32_tile)
      f32x4_t& sum = acc[i][j];
      const float bf = bv[set][j][e], af = av[set][i][e];
      asm volatile("v_mfma_f32_16x16x4_f32 %0, %1, %2, %0" : "+a"(sum) : "v"(bf), "v"(af));
    });
    __builtin_amdgcn_sched_barrier(0);
  };
  int n = 0;
  for (; n + 2 <= count; n += 2) {
    trip(0, n);
    trip(1, n + 1);
  }
  drain<TA, TB>(acc);
  if (n < count) {
    trip(0, n);
    drain<TA, TB>(acc);
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // nothing may land in LDS any more
}

template <int RM, int RN, bool TNL, bool VEC>
__device__ __forceinline__ void f32_tile(const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ C,
                                         const float* __restrict__ Res, int M, int N, int K, int lda, int ldb, int ldc, int id,
                                         int tiles_m, int tiles_n, int epi) {
  constexpr int TA = RM / 16, TB = RN / 16, DEPTH = TA * TB >= 16 ? 2 : TA * TB >= 8 ? 3 : TA * TB >= 4 ? 4 : 8;
  constexpr bool STAGED = !TNL && VEC;
  constexpr int PART = 4 * RM * (RN + 4) * 4, RING = STAGED ? 4 * ring_slots(RM, RN) * (TA + TB) * 1024 : 0;
  __shared__ __attribute__((aligned(1024))) char smem[PART > RING ? PART : RING];
  float (&part)[4][RM][RN + 4] = *reinterpret_cast<float (*)[4][RM][RN + 4]>(smem);
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // consecutive workgroup ids go to different XCDs: every XCD takes one contiguous eighth of the tiles, row by row
  const int n_tiles = tiles_m * tiles_n;
  if ((n_tiles & 7) == 0) id = (id & 7) * (n_tiles >> 3) + (id >> 3);
  const int m0 = (id / tiles_n) * RM, n0 = (id % tiles_n) * RN;
  Operand<RM, TNL, VEC> a;
  Operand<RN, TNL, VEC> b;
  if constexpr (!STAGED) {
    a.init(A, lda, m0, M, K, lane);
    b.init(B, ldb, n0, N, K, lane);
  }
  const int a_left = TNL ? M - m0 - r * TA : 0, b_left = TNL ? N - n0 - r * TB : 0;   // rows of this lane inside the operand
  f32x4_t acc[TA][TB];
#pragma unroll
  for (int i = 0; i < TA; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  if constexpr (VEC) {                                       // the zeros are in place, some cycles ahead of the first product
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int j = 0; j < TB; ++j) asm volatile("" : "+a"(acc[i][j]));
    asm volatile("s_nop 3" ::: "memory");
  }
  if constexpr (STAGED) {
    staged_loop<RM, RN>(smem, acc, A, B, M, N, K, lda, ldb, m0, n0, wave, lane);
  } else {
    typename Operand<RM, TNL, VEC>::Frag av[DEPTH];
    typename Operand<RN, TNL, VEC>::Frag bv[DEPTH];
    const int steps = (K + STEP - 1) / STEP, count = (steps - wave + 3) >> 2;   // this wave's steps: wave + 4 s
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      __builtin_amdgcn_sched_barrier(0);
      a.load(av[d], (wave + 4 * d) * STEP, K, a_left);
      b.load(bv[d], (wave + 4 * d) * STEP, K, b_left);
    }
    auto multiply_k = [&](int d, int e) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j)
          // in assembly the sums stay where they are: of the builtin's results the compiler moves all to other registers and back, every time
          // round.  Its operands come straight from loads; no vector instruction writes them
          if constexpr (VEC) asm volatile("v_mfma_f32_16x16x4_f32 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(bv[d].get(j, e)), "v"(av[d].get(i, e)));
          else acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv[d].get(j, e), av[d].get(i, e), acc[i][j], 0, 0, 0);
    };
    auto multiply = [&](int d) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 4; ++e) multiply_k(d, e);
    };
    int s = 0;
    for (; s + DEPTH <= count; s += DEPTH) {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        // a step's loads stay behind the MFMAs that free their registers: left alone the compiler gathers those of all DEPTH steps at the
        // end of the loop, right ahead of one wait for all of them
        const int k = (wave + 4 * (s + d + DEPTH)) * STEP;
        if constexpr (TNL && VEC) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            __builtin_amdgcn_sched_barrier(0);
            multiply_k(d, e);
            __builtin_amdgcn_sched_barrier(0);
            a.load_k(av[d], k, e);
            b.load_k(bv[d], k, e);
          }
        } else {
          __builtin_amdgcn_sched_barrier(0);
          multiply(d);
          __builtin_amdgcn_sched_barrier(0);
          a.load(av[d], k, K, a_left);
          b.load(bv[d], k, K, b_left);
        }
      }
    }
    if constexpr (VEC) drain<TA, TB>(acc);
#pragma unroll
    for (int d = 0; d < DEPTH - 1; ++d)                      // the steps left over are loaded
      if (s + d < count) {
        multiply(d);
        if constexpr (VEC) drain<TA, TB>(acc);
      }
  }
  if constexpr (STAGED) __syncthreads();                     // every wave's ring is read
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
// a tile do not reach, and short contractions of many tiles (pick_form).
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

// The form that needs the least time: the matrix-instruction kernel on one of five tiles, or the plain kernel.  Workgroups come to the compute units
// evenly, n = ceil(tiles / 256) of them to the fullest.  Their contractions share its units, ns per k each; while the contraction is short, a
// workgroup's start, first loads and the way of its tile through LDS to memory bound them instead, a time per workgroup that no k shortens
// (16 x 16 tiles: 756 x 2056 of any K up to 64 takes 25 us, 64 x 64 tiles 6.6, and the plain kernel, which writes its sums at once, 7).  The plain
// kernel also waits for the loads of every step of 16, however many workgroups share a unit.  Measured from 4 to 4096 k on one to 128
// workgroups per unit (2052 products of 24 sizes, both layouts, 16-byte rows and others, storing and accumulating): the form picked takes 1.5 %
// longer than the fastest on average, 31 % at most, and 1.8 % on 832 others of any size up to 50 GFLOP.  With the start counted once for all workgroups, and fixed limits to the plain kernel,
// it was 15 % and up to three times, e.g. us before -> now: NT 756 x 2056 x 4 15.6 -> 6.8, 2208 x 2316 x 16 25.4 -> 14.5, 1760 x 1264 x 1023 166 -> 112,
// TN 4095 x 4095 x 128 accumulating 144 -> 98, 1760 x 1264 x 64 accumulating 14.3 -> 10.6; 512 x 4096 x 1024 37.8, 512 x 1024 x 1024 13.9 as before.
struct Form { int rows, cols; };
constexpr Form FORMS[] = {{64, 64}, {64, 32}, {32, 32}, {16, 32}, {16, 16}, {64, 64}};
constexpr int PLAIN = 5;
struct Cost { double start_us, group_us, k_ns, once_ns; };
// Consecutive workgroups go to different XCDs; where the number of tiles is a multiple of 8, each XCD has neighbours (f32_tile).  Elsewhere
// small TN tiles, which read most per product, take `scattered` times as long: 596 x 3724 x 3008 on 32 x 32 tiles 224 us, 640 x 3840 x 3072 145.
struct Costs { double scattered; Cost form[6]; };
constexpr Costs COSTS[] = {                                  // by layout, rows, epilogue (costs_of); by form
  {1, {{2.43, 2.33, 16.7}, {2.67, 2.07, 8.64}, {1.78, 1.37, 4.95}, {1.78, 0.91, 4.89}, {1.72, 0.98, 3.07}, {4.11, 1.65, 44.3, 92.1}}},   // NT
  {1, {{3.37, 1.86, 43.1}, {2.82, 1.19, 29.9}, {3.08, 0.67, 15.1}, {3.04, 0.66, 11.3}, {2.45, 0.42, 10}, {4.39, 1.76, 36, 90}}},   // NT, element by element
  {1.3, {{3.74, 2.57, 17.2}, {3.31, 0.81, 9.76}, {2.87, 0.81, 5.42}, {2.3, 1.07, 3.95}, {2.38, 0.74, 3.84}, {3.75, 1.59, 55.9, 81.2}}},   // TN
  {1.3, {{3.45, 3.65, 16.4}, {2.76, 1.07, 10.8}, {2.28, 0.76, 5.51}, {2.41, 0.91, 3.96}, {2.46, 0.89, 3.82}, {5.84, 1.87, 55.6, 108}}},   // TN, accumulating
  {1, {{4.15, 2.46, 36.3}, {3.39, 1.59, 25.1}, {2.74, 1.06, 10.8}, {2.73, 1.06, 7.44}, {2.99, 1.03, 4.02}, {3.9, 2.08, 31.8, 73.5}}},   // TN, element by element
  {1, {{3.93, 5.5, 35.7}, {4.78, 1.96, 24}, {3.22, 1.22, 9.72}, {2.84, 1.78, 6.9}, {2.11, 1.18, 4.35}, {5.4, 2.75, 30.4, 108}}},   // TN, element by element, accumulating
  {1, {{3.68, 3.14, 16.7}, {2.88, 1.97, 8.64}, {2, 1.39, 4.95}, {1.92, 1.49, 4.89}, {1.68, 0.85, 3.07}, {2.84, 2.03, 44.3, 92.1}}},   // NT, rows of C off 16 bytes
  {1, {{5.84, 4.22, 16.7}, {2.88, 3.4, 8.64}, {1.77, 2.24, 4.95}, {2.12, 1.44, 4.89}, {1.62, 1.49, 3.07}, {6.59, 3.18, 44.3, 92.1}}},   // the same with a residual
};
const Costs& costs_of(bool tn, bool vec, int epi, int ldc) {
  return COSTS[tn ? (vec ? 2 : 4) + (epi == EPI_ACCUM) : !vec ? 1 : ldc & 3 ? 6 + (epi == EPI_RESID) : 0];
}
int pick_form(const Costs& costs, int n, const GemmProblem* pr, int K, int forms = PLAIN + 1) {
  int best = 0;
  double least = 1e30;
  for (int t = 0; t < forms; ++t) {
    const Cost& c = costs.form[t];
    long long tiles = 0;
    for (int i = 0; i < n; ++i) tiles += (long long)((pr[i].M + FORMS[t].rows - 1) / FORMS[t].rows) * ((pr[i].N + FORMS[t].cols - 1) / FORMS[t].cols);
    const double each = (double)((tiles + 255) / 256), k = t == PLAIN ? (K + 15) / 16 * 16.0 : K;
    const double k_ns = c.k_ns * (FORMS[t].rows < 64 && each > 1 && (tiles & 7) ? costs.scattered : 1);
    const double us = c.start_us + std::max(each * c.group_us, 1e-3 * k * (c.once_ns + each * k_ns));
    if (us < least) { least = us; best = t; }
  }
  return best;
}

template <bool TNL, bool VEC>
hipError_t launch_sized(int form, int epi, const float* A, const float* B, float* C, const float* R, int M, int N, int K, int lda, int ldb,
                        int ldc, hipStream_t s) {
  switch (form) {
    case 0: return launch_mfma<64, 64, TNL, VEC>(epi, A, B, C, R, M, N, K, lda, ldb, ldc, s);
    case 1: return launch_mfma<64, 32, TNL, VEC>(epi, A, B, C, R, M, N, K, lda, ldb, ldc, s);
    case 2: return launch_mfma<32, 32, TNL, VEC>(epi, A, B, C, R, M, N, K, lda, ldb, ldc, s);
    case 3: return launch_mfma<16, 32, TNL, VEC>(epi, A, B, C, R, M, N, K, lda, ldb, ldc, s);
    default: return launch_mfma<16, 16, TNL, VEC>(epi, A, B, C, R, M, N, K, lda, ldb, ldc, s);
  }
}

}  // namespace

namespace {
// lane offsets of the matrix-instruction kernels: NT 64 rows of a tile, TN all k-rows of the operand's column strip
bool mfma_reaches(bool tn, int K, int lda, int ldb) {
  const unsigned long long reach = 0xF0000000ull / 4;
  const unsigned long long span = (unsigned long long)(tn ? K + 64ull * 16 : 64ull) * (unsigned long long)(lda > ldb ? lda : ldb) + 64;
  return span < reach && (tn || K < 1 << 25);                // 4 k below 2^27 (Staged::PAST)
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
  return pick_form(costs_of(true, true, EPI_ACCUM, 0), n, pr, K) != PLAIN;
}

// n independent TN products with the same K: C (fp32) += product (EPI_ACCUM) or = product
hipError_t launch_gemm_f32_grouped(int epi, int n, const GemmProblem* pr, int K, hipStream_t s) {
  if (!gemm_f32_grouped_applies(n, pr, K) || (epi != EPI_ACCUM && epi != EPI_STOREF)) return hipErrorInvalidValue;
  switch (pick_form(costs_of(true, true, epi, 0), n, pr, K, PLAIN)) {
    case 0: return launch_grouped<64, 64>(epi, n, pr, K, s);
    case 1: return launch_grouped<64, 32>(epi, n, pr, K, s);
    case 2: return launch_grouped<32, 32>(epi, n, pr, K, s);
    case 3: return launch_grouped<16, 32>(epi, n, pr, K, s);
    default: return launch_grouped<16, 16>(epi, n, pr, K, s);
  }
}

int gemm_f32_form(bool tn, bool vec, int epi, int M, int N, int K, int ldc) {
  const GemmProblem pr = {nullptr, nullptr, nullptr, nullptr, M, N, 0, 0, ldc};
  return pick_form(costs_of(tn, vec, epi, ldc), 1, &pr, K);
}

// The activation's epilogues are in the matrix-instruction kernels only
bool gemm_f32_act_applies(int M, int N, int K) {
  if (M <= 0 || N <= 0 || K <= 0 || (N & 3) || !mfma_reaches(false, K, K, K)) return false;
  return gemm_f32_form(false, (K & 3) == 0, EPI_STORE, M, N, K, N) != PLAIN;
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
  // the plain kernel also where the other does not reach; its grid's second dimension ends at 65535
  const bool reaches = mfma_reaches(tn, K, lda, ldb), plain_too = epi < EPI_GELU && (M + 63) / 64 < 65536;
  const int form = plain_too ? gemm_f32_form(tn, vec, epi, M, N, K, ldc) : pick_form(costs_of(tn, vec, epi, ldc), 1, &pr, K, PLAIN);
  if (form != PLAIN && reaches) {
    if (tn) return vec ? launch_sized<true, true>(form, epi, a, b, c, r, M, N, K, lda, ldb, ldc, s)
                       : launch_sized<true, false>(form, epi, a, b, c, r, M, N, K, lda, ldb, ldc, s);
    return vec ? launch_sized<false, true>(form, epi, a, b, c, r, M, N, K, lda, ldb, ldc, s)
               : launch_sized<false, false>(form, epi, a, b, c, r, M, N, K, lda, ldb, ldc, s);
  }
  const long sam = tn ? 1 : lda, sak = tn ? lda : 1, sbn = tn ? 1 : ldb, sbk = tn ? ldb : 1;
  dim3 grid((N + 63) / 64, (M + 63) / 64), block(256);
  if (epi == EPI_RESID) hipLaunchKernelGGL(gemm_f32_kernel<EPI_RESID>, grid, block, 0, s, a, b, c, r, M, N, K, sam, sak, sbn, sbk, ldc);
  else if (epi == EPI_ACCUM) hipLaunchKernelGGL(gemm_f32_kernel<EPI_ACCUM>, grid, block, 0, s, a, b, c, r, M, N, K, sam, sak, sbn, sbk, ldc);
  else hipLaunchKernelGGL(gemm_f32_kernel<EPI_STORE>, grid, block, 0, s, a, b, c, r, M, N, K, sam, sak, sbn, sbk, ldc);
  return hipGetLastError();
}
