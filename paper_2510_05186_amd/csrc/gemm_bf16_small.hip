// bf16 MFMA GEMM for products too small for the 256 x 256 kernels (gemm_bf16.hip): the same three linear maps (paper
// Sec. 2.2) on square tiles of 128 or 64, so that a few hundred tokens or a narrow layer still give work to most of
// the 256 compute units.  Tiles go straight from global memory into LDS (`buffer_load_dwordx4 ... lds`), products run on
// v_mfma_f32_16x16x32_bf16 (first operand = B fragment: a lane owns 4 consecutive columns of one row).
//  * NT (operands contiguous along k): LDS [rows][64 k], 16-byte chunks XOR-swizzled by the row; chunks past K are fetched
//    out of range and read as zero, so K needs to be a multiple of 8 only.
//  * TN (operands contiguous along their output index): LDS [64 k][columns] as in memory, fragments through the transposing
//    read; k-rows past K lie past the operand and read as zero, so K may be anything.
//  * Descriptors start at the tile's own corner (64-bit address), so operands may be larger than 4 GiB; the lane offsets
//    need (rows of a tile) * ld to stay below 2^31 elements, which the host checks.
// Two kernels:
//  shared  the four waves of a workgroup take the quarters of the tile.  Every fragment is read by two waves and every
//          k-tile costs a barrier, so the 64 k of a tile take 640 cycles at 64 x 64 and 1050 at 128 x 128 (LDS reads and
//          their latency) against 128 and 512 cycles of matrix work, however deep the prefetch.  The sums run over k in the
//          order of the 256 x 256 kernels, bit for bit.
//  split   (NT, few tiles) the waves split the contraction instead: wave w computes the whole 64 x 64 tile over the k-tiles w, w + 4, ... and
//          the four partial tiles are added through LDS at the end.  No wave reads what another has loaded: no barrier in the
//          loop, half the LDS reads, 250 cycles per 64 k.
// Measured (us, register-staged 128 x 128 kernel -> this file): NT 320 x 1024 x 3584 44.3 -> 11.0 (split; shared 64 18.8,
// shared 128 30.6), 1000 x 1024 x 3072 40.7 -> 12.6, 1024 x 1024 x 8192 96.7 -> 24.8, 2048 x 2048 x 2048 30.9 -> 21.7 (shared
// 128; split 31.6); TN 1024 x 1024 x 320 12.0 -> 5.2 (shared 64), 2048 x 2048 x 2048 42.3 -> 24.9 (shared 128).
#include <utility>

#include "common.h"

namespace {

constexpr int BK = 64;
constexpr unsigned OUT_OF_RANGE = 0xFFFFFF00u;
typedef __attribute__((address_space(3))) void lds_void_t;
typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
typedef __attribute__((address_space(3))) bf16x8_t lds_bf16x8_t;
typedef int i32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int swz(int row) { return (row ^ (row >> 3)) & 7; }

// One operand of an R-wide tile by 64 k: R rows (NT) or columns (TN), R * 128 bytes of LDS per k-tile.  A wave issues LOADS of
// the loads that fill it (1 KB each, from load `first_load`) and reads FRAGS 16-wide fragments from `first_frag`.
template <int R, bool TNL, int LOADS, int FRAGS> struct Operand {
  unsigned voff[LOADS];      // this lane's byte offset within the k-tile
  int fa[FRAGS][TNL ? 1 : 2];
  int load0;
  const char* base;          // corner of k-tile 0
  unsigned long long bytes;  // from there to the operand's end
  unsigned long long step;   // bytes from one k-tile to the next

  // which XOR of the 16-byte chunk index k-row k carries (TN): the 16 lanes-by-8-bytes pieces of a transposing read, k-rows
  // e = 0..3 of two groups 8 rows apart, must fall on all 64 banks (a row is one 256-byte bank window at R = 128, half of
  // one at R = 64)
  __device__ __forceinline__ static int tn_xor(int k) {
    return (R == 128 ? (k & 3) << 2 : ((k >> 1) & 1) << 2) ^ (((k >> 3) & 1) << 1);
  }
  // NT: the 16-byte chunk of its row that this lane fetches with load l
  __device__ __forceinline__ int nt_chunk(int l, int lane) const { return (lane & 7) ^ swz((load0 + l) * 8 + (lane >> 3)); }

  __device__ __forceinline__ void init(const bf16_t* p, int ld, int first, int extent, int K, int first_load, int first_frag, int lane) {
    load0 = first_load;
    if constexpr (TNL) {
      base = reinterpret_cast<const char*>(p + first);
      bytes = ((unsigned long long)(K - 1) * ld + extent - first) * 2;
      step = (unsigned long long)BK * ld * 2;
    } else {
      base = reinterpret_cast<const char*>(p + (size_t)first * ld);
      bytes = ((unsigned long long)(extent - 1 - first) * ld + K) * 2;
      step = BK * 2;
    }
#pragma unroll
    for (int l = 0; l < LOADS; ++l) {
      if constexpr (TNL) {
        constexpr int CPR = R / 8;                           // chunks per k-row
        const int k = (load0 + l) * (64 / CPR) + lane / CPR, c = (lane % CPR) ^ tn_xor(k);
        voff[l] = first + c * 8 < extent ? (unsigned)k * (unsigned)ld * 2u + (unsigned)c * 16u : OUT_OF_RANGE;
      } else {                                               // rows past the end lie past `bytes`
        voff[l] = (unsigned)((load0 + l) * 8 + (lane >> 3)) * (unsigned)ld * 2u + (unsigned)nt_chunk(l, lane) * 16u;
      }
    }
    const int g = lane >> 4;
#pragma unroll
    for (int i = 0; i < FRAGS; ++i) {
      if constexpr (TNL) {
        const int e = (lane >> 2) & 3, r = lane & 3, k = g * 8 + e;
        fa[i][0] = k * (R * 2) + (((2 * (first_frag + i) + (r >> 1)) ^ tn_xor(k)) << 4) + (r & 1) * 8;
      } else {
        const int row = (first_frag + i) * 16 + (lane & 15);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) fa[i][ks] = row * 128 + (((ks * 4 + g) ^ swz(row)) << 4);
      }
    }
  }
  // Descriptor of k-tile kt.  Past the last tile its length is zero: the loads zero-fill their slot, so that the number in
  // flight is the same on every trip.  The last tile of an NT operand with K % 64 != 0: chunks past K go out of range (for
  // good: no later tile is read).
  __device__ __forceinline__ i32x4_t desc(int kt, int K, int lane) {
    const unsigned long long off = (unsigned long long)kt * step, a = (unsigned long long)base + off;
    const unsigned long long left = kt * BK < K ? bytes - off : 0;
    i32x4_t d;
    d[0] = __builtin_amdgcn_readfirstlane((int)(unsigned)a);
    d[1] = __builtin_amdgcn_readfirstlane((int)(unsigned)(a >> 32) & 0xffff);
    d[2] = __builtin_amdgcn_readfirstlane((int)(unsigned)(left > 0xFFFFFF00ull ? 0xFFFFFF00ull : left));
    d[3] = 0x00020000;
    if constexpr (!TNL) {
      if (kt * BK < K && kt * BK + BK > K) {
        const int valid = (K - kt * BK) >> 3;
#pragma unroll
        for (int l = 0; l < LOADS; ++l)
          if (nt_chunk(l, lane) >= valid) voff[l] = OUT_OF_RANGE;
      }
    }
    return d;
  }
  __device__ __forceinline__ void issue(const i32x4_t& d, unsigned dst, int l) const {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(dst + l * 1024), "v"(voff[l]), "s"(d) : "memory", "m0");
  }
  __device__ __forceinline__ bf16x8_t frag(unsigned slot, int i, int ks) const {
    if constexpr (TNL) {
      const unsigned ad = slot + fa[i][0] + ks * (32 * R * 2);
      const i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t*)ad);
      const i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t*)(ad + 4 * R * 2));
      return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    } else {
      return *(const lds_bf16x8_t*)(slot + fa[i][ks]);
    }
  }
};

// four consecutive columns of one row of the result
template <int EPI> __device__ __forceinline__ void finish(const GemmProblem& pr, int m, int n, f32x4_t v) {
  if (m >= pr.M || n >= pr.N) return;
  const size_t off = (size_t)m * pr.ldc + n;
  if (EPI == EPI_STOREF || EPI == EPI_ACCUM) {
    f32x4_t* c = reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(pr.C) + off);
    if (EPI == EPI_ACCUM) { const f32x4_t o = *c; v[0] += o[0]; v[1] += o[1]; v[2] += o[2]; v[3] += o[3]; }
    // stored straight from the accumulation registers, the accumulators push the fragments of the loop into those, and every MFMA
    // waits for copies
    else asm volatile("" : "+v"(v));
    *c = v;
  } else if (EPI == EPI_DGELU || EPI == EPI_DSWIGLU) {       // of the gradient rounded as a product of its own would store it
    bf16x4_t* c = reinterpret_cast<bf16x4_t*>(reinterpret_cast<bf16_t*>(pr.C) + off);
    const bf16x4_t x = *c;
    bf16x4_t o;
    if (EPI == EPI_DGELU) {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (bf16_t)dgelu((float)x[e], (float)(bf16_t)v[e]);
    } else {
      bf16x4_t* cu = reinterpret_cast<bf16x4_t*>(reinterpret_cast<bf16_t*>(pr.C) + off + pr.N);
      const bf16x4_t u = *cu;
      bf16x4_t ou;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float dg, du;
        dswiglu((float)x[e], (float)u[e], (float)(bf16_t)v[e], dg, du);
        o[e] = (bf16_t)dg;
        ou[e] = (bf16_t)du;
      }
      *cu = ou;
    }
    *c = o;
  } else {
    if (EPI == EPI_RESID) {
      const bf16x4_t r = *reinterpret_cast<const bf16x4_t*>(reinterpret_cast<const bf16_t*>(pr.R) + off);
      v[0] += (float)r[0]; v[1] += (float)r[1]; v[2] += (float)r[2]; v[3] += (float)r[3];
    }
    bf16x4_t o;
    o[0] = (bf16_t)v[0]; o[1] = (bf16_t)v[1]; o[2] = (bf16_t)v[2]; o[3] = (bf16_t)v[3];
    *reinterpret_cast<bf16x4_t*>(reinterpret_cast<bf16_t*>(pr.C) + off) = o;
    if (EPI == EPI_GELU) {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (bf16_t)gelu((float)o[e]);
      *reinterpret_cast<bf16x4_t*>(const_cast<bf16_t*>(reinterpret_cast<const bf16_t*>(pr.R)) + off) = o;
    }
  }
}

// shared: ring of five k-tiles; while tile kt is multiplied, kt + 1 has landed (its first fragments are read under kt's last
// MFMAs) and kt + 2 .. kt + 4 are in flight.  One barrier per k-tile.
template <int R, bool TNL, int EPI>
__device__ __forceinline__ void shared_tile(char* smem, const GemmProblem& pr, int K, int tile_m, int tile_n) {
  constexpr int T = R / 32;                                  // 16 x 16 MFMA tiles per wave and direction
  constexpr int SLOT = 2 * R * 128, SHARE = R * 32;          // a k-tile of both operands; a wave's share of one operand
  constexpr int STAGES = 5, NL = R / 32, L = 2 * NL;         // loads of a wave per operand and per k-tile
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int m0 = tile_m * R, n0 = tile_n * R;
  Operand<R, TNL, NL, T> A, B;
  A.init((const bf16_t*)pr.A, pr.lda, m0, pr.M, K, wave * NL, wm * T, lane);
  B.init((const bf16_t*)pr.B, pr.ldb, n0, pr.N, K, wave * NL, wn * T, lane);
  const unsigned lds0 = (unsigned)(size_t)(lds_void_t*)smem;
  f32x4_t acc[T][T];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  bf16x8_t fa[2][T], fb[2][T];
  // fragment q (0 .. T - 1 A, T .. 2 T - 1 B) of k-step ks
  auto read = [&](int set, unsigned slot, int ks, int q) __attribute__((always_inline)) {
    if (q < T) fa[set][q] = A.frag(lds0 + slot, q, ks);
    else fb[set][q - T] = B.frag(lds0 + slot + R * 128, q - T, ks);
  };
  // Half a trip: the T * T MFMAs of fragment set `set`, in the order the compiler must keep.  Ahead of each of the first 2 T
  // goes one fragment read of the next half (they have landed when it starts), the loads of one operand of k-tile kt + 4
  // sit behind them (T = 4) or between them (T = 2).
  auto half = [&](int set, unsigned slot, int ks, auto& op, const i32x4_t& d, unsigned dst) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < T * T; ++t) {
      __builtin_amdgcn_sched_barrier(0);
      if (t < 2 * T) read(set ^ 1, slot, ks, (t & 1) * T + (t >> 1));
      if (t & 1) {
        const int l = T == 4 ? (t - 9) >> 1 : t >> 1;
        if (l >= 0 && l < NL) op.issue(d, dst, l);
      }
      __builtin_amdgcn_sched_barrier(0);
      const int i = t / T, j = i & 1 ? T - 1 - t % T : t % T;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][j], fa[set][i], acc[i][j], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  const int nk = (K + BK - 1) / BK;
  const unsigned lds_a = lds0 + wave * SHARE, lds_b = lds_a + R * 128;
#pragma unroll
  for (int u = 0; u < STAGES - 1; ++u) {
    const i32x4_t da = A.desc(u, K, lane), db = B.desc(u, K, lane);
#pragma unroll
    for (int l = 0; l < NL; ++l) { A.issue(da, lds_a + u * SLOT, l); B.issue(db, lds_b + u * SLOT, l); }
  }
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"((STAGES - 2) * L) : "memory");
#pragma unroll
  for (int q = 0; q < 2 * T; ++q) read(0, 0, 0, q);
  unsigned cur = 0, free_slot = (STAGES - 1) * SLOT;
  for (int kt = 0; kt < nk; ++kt) {
    const unsigned next = cur + SLOT == STAGES * SLOT ? 0 : cur + SLOT;
    const i32x4_t da = A.desc(kt + STAGES - 1, K, lane), db = B.desc(kt + STAGES - 1, K, lane);
    // tile kt + 1 has landed (this wave's part; the barrier covers the rest) and nobody still reads tile kt - 1
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"((STAGES - 3) * L) : "memory");
    half(0, cur, 1, A, da, lds_a + free_slot);
    half(1, next, 0, B, db, lds_b + free_slot);
    free_slot = cur;
    cur = next;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // no load may land in LDS that is no longer ours
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j)
      finish<EPI>(pr, m0 + (wm * T + i) * 16 + (lane & 15), n0 + (wn * T + j) * 16 + (lane >> 4) * 4, acc[i][j]);
}

// split: a wave has two 16 KB slots (64 k of both operands).  While block n is multiplied out of registers, the fragments of
// block n + 1 are read, the slot they leave is refilled with block n + 3, and block n + 2 is in flight.
template <int EPI>
__device__ __forceinline__ void split_tile(char* smem, const GemmProblem& pr, int K, int tile_m, int tile_n) {
  constexpr int R = 64, F = 4, NL = 8, SLOT = 16384, MF = 2 * F * F;   // fragments and loads per operand, MFMAs per block
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = tile_m * R, n0 = tile_n * R;
  Operand<R, false, NL, F> A, B;
  A.init((const bf16_t*)pr.A, pr.lda, m0, pr.M, K, 0, 0, lane);
  B.init((const bf16_t*)pr.B, pr.ldb, n0, pr.N, K, 0, 0, lane);
  const unsigned mine = (unsigned)(size_t)(lds_void_t*)smem + wave * 2 * SLOT;
  f32x4_t acc[F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  bf16x8_t fa[2][2 * F], fb[2][2 * F];                       // [set][ks * F + i]
  // fragments in the order their first MFMA comes: per k-step A0, B0 .. B3, A1 ..
  auto read = [&](int set, unsigned slot, int q) __attribute__((always_inline)) {
    const int ks = q / (2 * F), r = q % (2 * F);
    if (r == 0 || r > F) { const int i = r == 0 ? 0 : r - F; fa[set][ks * F + i] = A.frag(slot, i, ks); }
    else fb[set][ks * F + r - 1] = B.frag(slot + SLOT / 2, r - 1, ks);
  };
  const int nkb = (K + BK - 1) / BK, count = (nkb - wave + 3) >> 2;   // this wave's blocks: wave + 4 n
  auto fill = [&](int n, unsigned slot) __attribute__((always_inline)) {
    const i32x4_t da = A.desc(wave + 4 * n, K, lane), db = B.desc(wave + 4 * n, K, lane);
#pragma unroll
    for (int l = 0; l < NL; ++l) { A.issue(da, slot, l); B.issue(db, slot + SLOT / 2, l); }
  };
  fill(0, mine);
  fill(1, mine + SLOT);
  asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
#pragma unroll
  for (int q = 0; q < 4 * F; ++q) read(0, mine, q);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  fill(2, mine);
  // One block: its MFMAs (fragment set `set`) in the order written; ahead of each of the first half of them a fragment read
  // of block n + 1 (slot s), ahead of each of the others a load that refills that slot with block n + 3.
  auto trip = [&](int set, unsigned s, int n) __attribute__((always_inline)) {
    const i32x4_t da = A.desc(wave + 4 * (n + 3), K, lane), db = B.desc(wave + 4 * (n + 3), K, lane);
    asm volatile("s_waitcnt vmcnt(16)" ::: "memory");        // block n + 1 has landed; n + 2 stays in flight
#pragma unroll
    for (int t = 0; t < MF; ++t) {
      __builtin_amdgcn_sched_barrier(0);
      if (t < MF / 2) {
        read(set ^ 1, s, t);
      } else {
        if (t == MF / 2) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        const int l = t - MF / 2;
        if (l & 1) B.issue(db, s + SLOT / 2, l >> 1); else A.issue(da, s, l >> 1);
      }
      __builtin_amdgcn_sched_barrier(0);
      const int ks = t / (F * F), i = t / F % F, j = i & 1 ? F - 1 - t % F : t % F;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][ks * F + j], fa[set][ks * F + i], acc[i][j], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  for (int n = 0; n < count; n += 2) {
    trip(0, mine + SLOT, n);
    trip(1, mine, n + 1);                                    // past the last block: zeros
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // nothing may land in LDS any more
  __syncthreads();
  // add the four partial tiles ([wave][64 rows][64] fp32, 16-byte chunks XOR-swizzled by the row): wave w adds rows
  // 16 w .. 16 w + 15, in wave order, and finishes them
  constexpr int RB = R * 4, PART = R * RB;
#pragma unroll
  for (int i = 0; i < F; ++i) {
    const int row = i * 16 + (lane & 15);
#pragma unroll
    for (int j = 0; j < F; ++j)
      *reinterpret_cast<f32x4_t*>(smem + wave * PART + row * RB + (((j * 4 + (lane >> 4)) ^ (row & 15)) << 4)) = acc[i][j];
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int row = wave * 16 + it * 4 + (lane >> 4), c = lane & 15;
    const char* at = smem + row * RB + ((c ^ (row & 15)) << 4);
    f32x4_t v = *reinterpret_cast<const f32x4_t*>(at);
#pragma unroll
    for (int p = 1; p < 4; ++p) {
      const f32x4_t o = *reinterpret_cast<const f32x4_t*>(at + p * PART);
      v[0] += o[0]; v[1] += o[1]; v[2] += o[2]; v[3] += o[3];
    }
    finish<EPI>(pr, m0 + row, n0 + c * 4, v);
  }
}

// Consecutive workgroup ids go to different XCDs: every XCD takes one contiguous eighth of the tile sequence, which walks
// groups of 8 tile rows column by column, so that the tiles of an XCD share operand panels in its L2.
__device__ __forceinline__ void tile_at(int id, int n, int tiles_m, int tiles_n, int& tile_m, int& tile_n) {
  if ((n & 7) == 0) id = (id & 7) * (n >> 3) + (id >> 3);
  constexpr int GM = 8;
  const int grp = id / (GM * tiles_n), first_m = grp * GM, gsz = min(tiles_m - first_m, GM), in_grp = id - grp * GM * tiles_n;
  tile_m = first_m + in_grp % gsz;
  tile_n = in_grp / gsz;
}

template <int R, bool TNL, int EPI>
__global__ __launch_bounds__(256) void gemm_bf16_shared_kernel(const GemmProblem pr, int K, int tiles_m, int tiles_n) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int tile_m, tile_n;
  tile_at(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, tile_m, tile_n);
  shared_tile<R, TNL, EPI>(smem, pr, K, tile_m, tile_n);
}

template <int EPI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_bf16_split_kernel(const GemmProblem pr, int K,
                                                                                                       int tiles_m, int tiles_n) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int tile_m, tile_n;
  tile_at(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, tile_m, tile_n);
  split_tile<EPI>(smem, pr, K, tile_m, tile_n);
}

template <int R, int SMEM, typename Kernel>
hipError_t launch(Kernel kern, LdsAttrOnce& lds_attr, const GemmProblem& pr, int K, hipStream_t s) {
  if (hipError_t e = lds_attr.ensure(reinterpret_cast<const void*>(kern), SMEM); e != hipSuccess) return e;
  const int tiles_m = (pr.M + R - 1) / R, tiles_n = (pr.N + R - 1) / R;
  hipLaunchKernelGGL(kern, dim3((unsigned)tiles_m * (unsigned)tiles_n), dim3(256), SMEM, s, pr, K, tiles_m, tiles_n);
  return hipGetLastError();
}

// Which kernel, by the number of 64 x 64 tiles.  Two workgroups of the shared kernel with tiles of 64 fit a compute unit, one of the others.
// Times over those of the register-staged 128 x 128 kernel:
//  * up to 256 (a tile per compute unit), NT: split from K = 768 on (K 904 / 1536 / 4800 .44 / .32 / .24, shared .48 / .42 /
//    .38), shared below (K 64 / 256 / 704 .53 - .98 / .47 - .64 / .44; split .71 - 1.11 / .59 - .78 / .46).  TN: shared.
//  * up to 512 the shared kernel with tiles of 64, one round for the chip: NT .53 - .77 (tiles of 128 .65 - .95, split, now two rounds, .57 -
//    1.63), TN .40 - .95 (tiles of 128 .52 - .97).  NT towards the end of that range, where it is fully loaded, tiles of 128
//    with a long contraction (490 tiles, K 1472 .73 / .83; 468, K 1352 .77 / .77; 452, K 5536 .70 / .59).
//  * beyond, where tiles of 64 take a second round, tiles of 128: NT 550 to 986 tiles .73 - .95 (64: .83 - 1.29; K 24, 40: .93 /
//    .83, .95 / .92), TN 528 to 890 .52 - .90 (64: .66 - 1.17; accumulating, K 102 / 279, .88 / .82, .79 / .77: with short contractions
//    the line is 700).
template <bool TNL, int EPI>
hipError_t launch_sized(const GemmProblem& pr, int K, hipStream_t s) {
  const long tiles64 = (long)((pr.M + 63) / 64) * ((pr.N + 63) / 64);
  static LdsAttrOnce big, small, split;
  if constexpr (!TNL)
    if (tiles64 <= 256 && K >= 768) return launch<64, 4 * 32768>(gemm_bf16_split_kernel<EPI>, split, pr, K, s);
  const long round64 = TNL ? (K <= 160 ? 700 : 512) : K >= 1024 ? 480 : 512;
  if (tiles64 > round64) return launch<128, 5 * 32768>(gemm_bf16_shared_kernel<128, TNL, EPI>, big, pr, K, s);
  return launch<64, 5 * 16384>(gemm_bf16_shared_kernel<64, TNL, EPI>, small, pr, K, s);
}

}  // namespace

bool gemm_bf16_small_applies(int M, int N, int K, int lda, int ldb) {
  return (unsigned long long)lda < (1ull << 23) && (unsigned long long)ldb < (1ull << 23) && M > 0 && N > 0 && K > 0;
}

hipError_t launch_gemm_bf16_small(int layout, int epi, const GemmProblem& pr, int K, hipStream_t s) {
  if (!gemm_bf16_small_applies(pr.M, pr.N, K, pr.lda, pr.ldb)) return hipErrorInvalidValue;
  if (layout == GEMM_NT) {
    if (epi == EPI_STORE) return launch_sized<false, EPI_STORE>(pr, K, s);
    if (epi == EPI_RESID) return launch_sized<false, EPI_RESID>(pr, K, s);
    if (epi == EPI_ACCUM) return launch_sized<false, EPI_ACCUM>(pr, K, s);
    if (epi == EPI_GELU) return launch_sized<false, EPI_GELU>(pr, K, s);
    if (epi == EPI_DGELU) return launch_sized<false, EPI_DGELU>(pr, K, s);
    if (epi == EPI_DSWIGLU) return launch_sized<false, EPI_DSWIGLU>(pr, K, s);
  } else if (layout == GEMM_TN) {
    if (epi == EPI_STORE) return launch_sized<true, EPI_STORE>(pr, K, s);
    if (epi == EPI_ACCUM) return launch_sized<true, EPI_ACCUM>(pr, K, s);
    if (epi == EPI_STOREF) return launch_sized<true, EPI_STOREF>(pr, K, s);
  }
  return hipErrorInvalidValue;
}
