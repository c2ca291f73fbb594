// bf16 MFMA GEMM for gfx950: C[M,N] = sum_k A(m,k) * B(n,k), fp32 accumulation.
//
// These are the three linear maps of a stage (paper Sec. 2.2): forward Y = X W^T (NT), backward for
// activations dX = dY W (NT against the transposed weight copy), backward for weights dW += dY^T X (TN).
//
// Design (CDNA4): three kernels by size (launch_layout).  Large products take the direct kernels below: one workgroup of
// 4 waves per tile, the K loop advances 64 elements at a time, operand tiles go straight from global memory into a ring of
// five LDS slots, one barrier per step.  Smaller products run on tiles of 128 or 64 (gemm_bf16_small.hip).  What neither can
// address (rows of one tile spread over more than 32-bit offsets), and some products between their sizes (direct_on_few_tiles),
// go through the register-staged kernel: 128 x 128 tiles, global
// -> registers -> LDS, two buffers, operands that are contiguous along their output index (TN) transposed in registers on the
// way into LDS.  Everywhere the LDS tiles' 16-byte chunk index is XOR-swizzled by the row so that operand reads and tile writes
// are free of bank conflicts, and the MFMA is issued with the B fragment as its first operand: each lane then owns
// 4 consecutive n of one m, which gives 8-byte (bf16) / 16-byte (fp32) row-major global accesses in the epilogue.  Workgroup
// ids are remapped so that the tiles resident on one XCD (ids congruent mod 8) form a compact patch of the output and share
// A/B panels in that XCD's L2.
#include <utility>

#include "common.h"

namespace {

constexpr int BK = 64;           // k elements per LDS tile
constexpr int ROW_BYTES = 128;   // 64 bf16

__device__ __forceinline__ int swz(int row) { return (row ^ (row >> 3)) & 7; }

// ---- global -> register staging -------------------------------------------------------------------
// K-contiguous operand: element (r, k) at p[r * ld + k].  Thread handles R_T/32 16-byte chunks.
template <int R_T, int NTH> struct StageKC {
  static constexpr int NCH = R_T * 8 / NTH;
  uint4 reg[NCH];
  __device__ __forceinline__ void load(const bf16_t* p, int ld, int row0, int rows, int k0, int K, int tid) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      int q = tid + NTH * i;
      int row = q >> 3, c = q & 7;
      int gr = row0 + row, gk = k0 + c * 8;
      if (gr < rows && gk < K)
        reg[i] = *reinterpret_cast<const uint4*>(p + (size_t)gr * ld + gk);
      else
        reg[i] = make_uint4(0, 0, 0, 0);
    }
  }
  __device__ __forceinline__ void store(char* lds, int tid) const {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      int q = tid + NTH * i;
      int row = q >> 3, c = q & 7;
      *reinterpret_cast<uint4*>(lds + row * ROW_BYTES + ((c ^ swz(row)) << 4)) = reg[i];
    }
  }
};

// Row-contiguous operand: element (r, k) at p[k * ld + r].  Thread gathers KV k-rows x 8 r and writes
// 8 pieces of KV k-contiguous elements.
template <int R_T, int NTH> struct StageRC {
  static constexpr int KV = R_T * 8 / NTH;   // k-rows per thread
  static_assert(KV == 4, "unsupported tile / thread-count combination");
  uint4 reg[KV];
  // 8-byte LDS stores: lanes 0-7 vary the row chunk, lane bit 3 the half of the 16-byte chunk
  __device__ __forceinline__ static void coords(int tid, int& rc, int& kg) {
    const int hi = tid >> 4;
    rc = (tid & 7) | ((hi % (R_T / 64)) << 3);
    kg = ((tid >> 3) & 1) | ((hi / (R_T / 64)) << 1);
  }
  __device__ __forceinline__ void load(const bf16_t* p, int ld, int row0, int rows, int k0, int K, int tid) {
    int rc, kg;
    coords(tid, rc, kg);
    int gr = row0 + rc * 8;
#pragma unroll
    for (int kk = 0; kk < KV; ++kk) {
      int gk = k0 + kg * KV + kk;
      if (gr < rows && gk < K)
        reg[kk] = *reinterpret_cast<const uint4*>(p + (size_t)gk * ld + gr);
      else
        reg[kk] = make_uint4(0, 0, 0, 0);
    }
  }
  __device__ __forceinline__ void store(char* lds, int tid) const {
    int rc, kg;
    coords(tid, rc, kg);
    const uint32_t* w = reinterpret_cast<const uint32_t*>(reg);   // w[kk*4 + i/2] holds elements i, i+1 of k-row kk
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      uint32_t out[KV / 2];
#pragma unroll
      for (int pr = 0; pr < KV / 2; ++pr) {
        uint32_t a = w[(2 * pr) * 4 + (i >> 1)], b = w[(2 * pr + 1) * 4 + (i >> 1)];
        out[pr] = (i & 1) ? ((a >> 16) | (b & 0xffff0000u)) : ((a & 0xffffu) | (b << 16));
      }
      int row = rc * 8 + i;
      int koff = kg * KV;
      char* dst = lds + row * ROW_BYTES + ((((koff >> 3)) ^ swz(row)) << 4) + (koff & 7) * 2;
      *reinterpret_cast<uint2*>(dst) = make_uint2(out[0], out[1]);
    }
  }
};

template <int R_T, int NTH, bool RC> struct StageSel { typedef StageKC<R_T, NTH> type; };
template <int R_T, int NTH> struct StageSel<R_T, NTH, true> { typedef StageRC<R_T, NTH> type; };

// ---- kernel ---------------------------------------------------------------------------------------
template <bool RC, int EPI>
__global__ __launch_bounds__(256) void gemm_bf16_staged_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B,
                                                        void* __restrict__ Cv, const bf16_t* __restrict__ R, int M,
                                                        int N, int K, int lda, int ldb, int ldc, int tiles_m,
                                                        int tiles_n) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr int BM = 128, BN = 128, WM = 2, WN = 2;
  constexpr int A_BYTES = BM * ROW_BYTES, B_BYTES = BN * ROW_BYTES, BUF = A_BYTES + B_BYTES;
  constexpr int NTH = 64 * WM * WN;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;   // 32x32 MFMA tiles per wave in m and n

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;

  // XCD-aware tile order: consecutive hardware ids go to different XCDs, so give every XCD one
  // contiguous range of the tile sequence, and walk that sequence in groups of 8 tile rows.
  int pid = blockIdx.x;
  const int nblk = tiles_m * tiles_n;
  if ((nblk & 7) == 0) pid = (pid & 7) * (nblk >> 3) + (pid >> 3);
  constexpr int GM = 8;
  const int grp = pid / (GM * tiles_n);
  const int first_m = grp * GM;
  const int gsz = min(tiles_m - first_m, GM);
  const int in_grp = pid - grp * GM * tiles_n;
  const int tile_m = first_m + in_grp % gsz, tile_n = in_grp / gsz;
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  typename StageSel<BM, NTH, RC>::type sa;
  typename StageSel<BN, NTH, RC>::type sb;

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // per-lane LDS read offsets (row part); the k chunk is added per k-step
  int a_off[TM], a_sw[TM], b_off[TN], b_sw[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    int row = wm * (BM / WM) + i * 32 + (lane & 31);
    a_off[i] = row * ROW_BYTES;
    a_sw[i] = swz(row);
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    int row = wn * (BN / WN) + j * 32 + (lane & 31);
    b_off[j] = A_BYTES + row * ROW_BYTES;
    b_sw[j] = swz(row);
  }
  const int khalf = lane >> 5;

  const int nk = (K + BK - 1) / BK;
  char* const buf0 = smem;
  char* const buf1 = smem + BUF;

  // operand fragments of one 16-wide k-step
  auto load_frags = [&](bf16x8_t (&af)[TM], bf16x8_t (&bfr)[TN], const char* buf, int ks) {
    const int chunk = ks * 2 + khalf;
#pragma unroll
    for (int i = 0; i < TM; ++i) af[i] = *reinterpret_cast<const bf16x8_t*>(buf + a_off[i] + ((chunk ^ a_sw[i]) << 4));
#pragma unroll
    for (int j = 0; j < TN; ++j) bfr[j] = *reinterpret_cast<const bf16x8_t*>(buf + b_off[j] + ((chunk ^ b_sw[j]) << 4));
  };
  auto mma = [&](const bf16x8_t (&af)[TM], const bf16x8_t (&bfr)[TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
  };

  // Software pipeline.  LDS holds tiles kt (cur) and kt+1 (nxt); registers hold tile kt+2 in flight.
  // Fragments are double-buffered so the LDS reads of k-step ks+1 run under the MFMAs of k-step ks, and
  // the one barrier per tile sits before the last k-step, with a full k-step of MFMAs already queued;
  // after it the freed cur buffer takes tile kt+2 and the first fragments of tile kt+1 are fetched.
  sa.load(A, lda, m0, M, 0, K, tid);
  sb.load(B, ldb, n0, N, 0, K, tid);
  sa.store(buf0, tid);
  sb.store(buf0 + A_BYTES, tid);
  sa.load(A, lda, m0, M, BK, K, tid);
  sb.load(B, ldb, n0, N, BK, K, tid);
  sa.store(buf1, tid);
  sb.store(buf1 + A_BYTES, tid);
  __syncthreads();

  bf16x8_t fa0[TM], fb0[TN], fa1[TM], fb1[TN];
  load_frags(fa0, fb0, buf0, 0);
  for (int kt = 0; kt < nk; ++kt) {
    char* cur = (kt & 1) ? buf1 : buf0;
    char* nxt = (kt & 1) ? buf0 : buf1;
    sa.load(A, lda, m0, M, (kt + 2) * BK, K, tid);
    sb.load(B, ldb, n0, N, (kt + 2) * BK, K, tid);
    __builtin_amdgcn_sched_barrier(0);
    load_frags(fa1, fb1, cur, 1);
    __builtin_amdgcn_sched_barrier(0);
    mma(fa0, fb0);
    __builtin_amdgcn_sched_barrier(0);
    load_frags(fa0, fb0, cur, 2);
    __builtin_amdgcn_sched_barrier(0);
    mma(fa1, fb1);
    __builtin_amdgcn_sched_barrier(0);
    load_frags(fa1, fb1, cur, 3);
    __builtin_amdgcn_sched_barrier(0);
    mma(fa0, fb0);
    __builtin_amdgcn_sched_barrier(0);
    // every wave has issued its last read of cur and its writes of nxt: wait for LDS traffic only
    // (global loads of tile kt+2 stay in flight), then meet
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    load_frags(fa0, fb0, nxt, 0);
    __builtin_amdgcn_sched_barrier(0);
    mma(fa1, fb1);
    __builtin_amdgcn_sched_barrier(0);
    sa.store(cur, tid);
    sb.store(cur + A_BYTES, tid);
  }

  // epilogue: lane owns m = .. + (lane & 31) and, per register group g, n = .. + 8 g + 4 (lane >> 5) + 0..3
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + wm * (BM / WM) + i * 32 + (lane & 31);
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int n = n0 + wn * (BN / WN) + j * 32 + g * 8 + khalf * 4;
        if (n >= N) continue;
        const size_t off = (size_t)m * ldc + n;
        float v0 = acc[i][j][g * 4 + 0], v1 = acc[i][j][g * 4 + 1], v2 = acc[i][j][g * 4 + 2], v3 = acc[i][j][g * 4 + 3];
        if (EPI == EPI_STOREF) {
          f32x4_t c = {v0, v1, v2, v3};
          *reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(Cv) + off) = c;
        } else if (EPI == EPI_ACCUM) {
          float* C = reinterpret_cast<float*>(Cv);
          f32x4_t c = *reinterpret_cast<const f32x4_t*>(C + off);
          c[0] += v0; c[1] += v1; c[2] += v2; c[3] += v3;
          *reinterpret_cast<f32x4_t*>(C + off) = c;
        } else {
          if (EPI == EPI_RESID) {
            bf16x4_t r = *reinterpret_cast<const bf16x4_t*>(R + off);
            v0 += (float)r[0]; v1 += (float)r[1]; v2 += (float)r[2]; v3 += (float)r[3];
          }
          bf16x4_t o;
          o[0] = (bf16_t)v0; o[1] = (bf16_t)v1; o[2] = (bf16_t)v2; o[3] = (bf16_t)v3;
          *reinterpret_cast<bf16x4_t*>(reinterpret_cast<bf16_t*>(Cv) + off) = o;
        }
      }
    }
  }
}

// ---- kernels with direct global -> LDS tile loads (NT and TN) -----------------------------------------
// 256 x 256 x 64 tiles, 2 x 2 waves (one per SIMD; each owns 128 x 128 of the output in 256 accumulator
// registers).  The tiles never pass through registers: every wave issues 16 `buffer_load_dwordx4 ... lds` per
// k-tile, each filling 1 KB of LDS (lane i writes 16 bytes at base + 16 i); which global address a lane loads
// realises the LDS swizzle.  Requires operands below 4 GiB (checked on the host); rows, columns and k past the operand read
// as zero through the buffer range check.
//
// What bounds them is power: the board holds its limit by lowering the clock, so time goes with the energy per flop.
// v_mfma_f32_16x16x32_bf16 moves half the accumulator traffic per flop of v_mfma_f32_32x32x16_bf16 and runs 15 % faster in
// a loop that does nothing else (2070 against 1806 TFLOP/s, operands drawn at random); in these kernels, 32x32x16 -> 16x16x32:
// 4096 x 12288 x 4096 1358 -> 1479 TFLOP/s, 4096 x 4096 x 11008 1400 -> 1528, 4096 x 8192 x 28672 1430 -> 1503, the
// grouped TN set of a hidden-8192 layer 1233 -> 1285 (fp32 store 1316 -> 1370).  The clock rises from 1.59 to 1.81 GHz, the matrix
// pipe is busy 81 % of the cycles (88 % before); with the trip's scalar work spread between the MFMAs (below) the four reach
// 1522, 1563, 1566 and 1331 (1427) on a box where the start gave 1355, 1377, 1413 and 1235 (1305).  Walking j to and fro (consecutive MFMAs share an operand) is worth 0.7 %.
//
//  NT (operands contiguous along k): a stage holds [256 rows][64 k]; the load for rows 8 q .. 8 q + 7 has lane i
//     fetch row 8 q + i / 8, logical 16-byte chunk (i % 8) ^ swz(row); fragments are plain 16-byte reads: 16 rows by 4
//     chunks, the 16 lanes of a pass on 16 rows of one chunk, which the swizzle spreads over all banks.
//  TN (operands contiguous along their output index): a stage holds the tile as it lies in memory,
//     [64 k][256 columns]; one load fills k-rows 2 b, 2 b + 1, lane i fetching k-row 2 b + i / 32, logical chunk
//     (i % 32) ^ ((k & 3) << 2) ^ (((k >> 3) & 1) << 1).  Fragments come from the transposing read ds_read_b64_tr_b16: in
//     every 16-lane group lane 4 e + r reads 8 bytes of k-row e, columns 4 r .. 4 r + 3, and the instruction hands lane i
//     the 4 k values of column i; two of them make the 8 k of an MFMA operand.  The first XOR spreads the 4 k-rows of
//     such a read over the four 64-byte bank groups, the second puts the two 16-lane groups of a pass, which read
//     k-rows 8 apart, in the two halves of a group.
//
// With a single wave per SIMD nothing hides an instruction that waits, so the main loop is laid out by hand
// (the scheduling barriers pin the order):
//  * LDS is a ring of five 32 KB slots that the operand tiles take in the order A0 B0 A1 B1 A2 ...; a tile's
//    operands may lie in any two of them, so the per-lane fragment addresses are rebuilt (one add each) for
//    the next tile under MFMAs that have nothing else to issue.
//  * The fragments of k-step s + 1 are read under the MFMAs of k-step s; those of the last k-step of a tile are
//    requested early in the k-step before, so they have landed when the tile barrier is reached.
//  * The loop is rotated so that the one barrier per tile (next tile landed, two slots free to refill) sits at
//    the top of the trip; it waits for all of this wave's loads but the newest eight, which belong to the tile
//    after the next one.
//  * One tile load goes out ahead of every eighth MFMA.  Issued back to back (16 loads by each of four waves at
//    the same point of the loop) they fill the address queue of the texture unit, which blocks the waves that
//    issue them and the MFMAs behind; the uneven request stream also cost a third more L2 misses.
//  * An MFMA leaves room for the issue of two or three other instructions, so the scalar work of a trip (descriptors, ring
//    slots) and the address adds are pinned between MFMAs too, at the positions that carry no read: gathered at the top of
//    the trip, as the compiler leaves them, they cost 4 %.
//  * A tile index past the end is fetched through a zero-length descriptor, which zero-fills its slot, so the
//    number of loads in flight is the same on every trip and the waits need no second code path.  The trip of the last tile
//    loads nothing, so that all loads have landed well before the epilogue takes LDS over.
//  * The tile loads are written in assembly: issued through the compiler builtin, every later transposing
//    read is ordered after them with a full vmcnt(0) wait, which serialises the loop.  The one wait + barrier
//    per tile orders them instead.
typedef __attribute__((address_space(3))) void lds_void_t;
typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
typedef int i32x4_t __attribute__((ext_vector_type(4)));

// Accumulators of a wave of the direct kernels: 128 x 128 of the output as 8 x 8 MFMA tiles of 16 x 16.  Of tile (i, j)
// this lane holds row 16 i + (lane & 15), columns 16 j + 4 (lane >> 4) .. + 3.
typedef f32x4_t acc_tile_t[8][8];

// Epilogue of the direct kernels for bf16 outputs: the wave converts its 128 x 128 accumulator tile to bf16
// (after adding the residual, given in accumulator layout, when there is one), transposes it through its own
// 32 KB of LDS ([128 rows][256 B], 16-byte chunks XOR-swizzled by the row: a 32-lane 8-byte write, 16 rows by the two
// halves of a chunk, touches all 64 banks once) and writes whole 256-byte row segments, 16 bytes per lane.
template <int EPI>
__device__ __forceinline__ void epilogue_bf16_rows(acc_tile_t& acc, const bf16x4_t (&res)[EPI == EPI_RESID ? 64 : 1], char* smem, int wave,
                                                   int lane, bf16_t* C, int M, int N, int ldc, int mw, int nw) {
  char* const wl = smem + wave * 32768;
  const int g = lane >> 4;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int row = i * 16 + (lane & 15);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      f32x4_t v = acc[i][j];
      if (EPI == EPI_RESID) {
        const bf16x4_t rv = res[i * 8 + j];
        v[0] += (float)rv[0]; v[1] += (float)rv[1]; v[2] += (float)rv[2]; v[3] += (float)rv[3];
      }
      bf16x4_t o;
      o[0] = (bf16_t)v[0]; o[1] = (bf16_t)v[1]; o[2] = (bf16_t)v[2]; o[3] = (bf16_t)v[3];
      const int chunk = j * 2 + (g >> 1);
      *reinterpret_cast<bf16x4_t*>(wl + row * 256 + ((chunk ^ (row & 15)) << 4) + (g & 1) * 8) = o;
    }
  }
  // every wave reads back only what it wrote itself: no workgroup barrier
  const int c = lane & 15, rsub = lane >> 4;
  const int n = nw + c * 8;
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  auto fetch = [&](int row) {
    return *reinterpret_cast<const u32x4*>(wl + row * 256 + ((c ^ (row & 15)) << 4));
  };
  if (mw + 128 <= M && nw + 128 <= N && (ldc & 7) == 0) {        // interior wave tile: 16-byte stores, no checks
    bf16_t* dst = C + (size_t)(mw + rsub) * ldc + n;
    const size_t step = (size_t)4 * ldc;
#pragma unroll 8
    for (int it = 0; it < 32; ++it) {
      *reinterpret_cast<u32x4*>(dst) = fetch(it * 4 + rsub);
      dst += step;
    }
  } else {
    for (int it = 0; it < 32; ++it) {
      const int row = it * 4 + rsub;
      const u32x4 v = fetch(row);
      const int m = mw + row;
      if (m < M) {
        bf16_t* dst = C + (size_t)m * ldc + n;
        if (n + 4 <= N) { u32x2 lo; lo[0] = v[0]; lo[1] = v[1]; *reinterpret_cast<u32x2*>(dst) = lo; }
        if (n + 8 <= N) { u32x2 hi; hi[0] = v[2]; hi[1] = v[3]; *reinterpret_cast<u32x2*>(dst + 4) = hi; }
      }
    }
  }
}

// old value p2 (0..63, two rows each) of C += product for this lane: row 2 p2 + lane / 32, columns 4 (lane % 32) ..  An ordinary load:
// non-temporal ones are the slower the fewer tiles there are (TN, 128 tiles, 64 / 512 / 2048 tokens: 16.8 / 25.6 / 47.3 us
// non-temporal, 15.9 / 22.7 / 44.4 so; 256 tiles, 512: 34.4 / 33.5; sets of 3088 and 13056 tiles the same).
__device__ __forceinline__ f32x4_t old_value(const float* C, int p2, int lane, int M, int N, int ldc, int mw, int nw) {
  const int m = min(mw + 2 * p2 + (lane >> 5), M - 1), n = min(nw + (lane & 31) * 4, N - 4);
  return *reinterpret_cast<const f32x4_t*>(C + (size_t)m * ldc + n);
}

// Epilogue of the direct kernels for fp32 outputs (C = product or C += product): 64 rows at a time go through the wave's
// 32 KB of LDS ([64 rows][512 B], 16-byte chunks XOR-swizzled by the row) so that global memory sees whole 512-byte row
// segments.  The old values of the first 64 rows come in `old`; each is replaced by one of the second 64 when it has been
// used, so that those arrive under the stores.  Stores are non-temporal: nothing reads a row again in this launch.
template <int EPI>
__device__ __forceinline__ void epilogue_f32_rows(acc_tile_t& acc, f32x4_t (&old)[EPI == EPI_ACCUM ? 32 : 1], char* smem, int wave, int lane,
                                                  float* C, int M, int N, int ldc, int mw, int nw) {
  char* const wl = smem + wave * 32768;
  const int khalf = lane >> 5, c = lane & 31, n = nw + c * 4;
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = i * 16 + (lane & 15);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        *reinterpret_cast<f32x4_t*>(wl + row * 512 + (((j * 4 + (lane >> 4)) ^ (row & 31)) << 4)) = acc[pass * 4 + i][j];
    }
#pragma unroll
    for (int p2 = 0; p2 < 32; ++p2) {
      const int row = 2 * p2 + khalf, m = mw + pass * 64 + row;
      f32x4_t v = *reinterpret_cast<const f32x4_t*>(wl + row * 512 + ((c ^ (row & 31)) << 4));
      if constexpr (EPI == EPI_ACCUM) {
        v[0] += old[p2][0]; v[1] += old[p2][1]; v[2] += old[p2][2]; v[3] += old[p2][3];
        if (pass == 0) old[p2] = old_value(C, 32 + p2, lane, M, N, ldc, mw, nw);
      }
      if (m < M && n < N) __builtin_nontemporal_store(v, reinterpret_cast<f32x4_t*>(C + (size_t)m * ldc + n));
    }
  }
}

// Rotary embedding on the accumulators of a wave tile that is one attention head (128 columns starting at a multiple
// of 128): column c < 64 pairs with column c + 64, which the same lane holds in the same register of acc[i][j + 4]
// (j = 0..3), so the rotation by position * theta_c happens in registers, in fp32, before the one conversion to bf16.
// table[pos * 64 + c] = (cos, sin); pos = row % seq.  Every lane reads the 32-byte pieces of its own row's table row
// straight from memory (the table stays in L2); staging the rows through LDS with coalesced loads measured slower.
__device__ __forceinline__ void rope_rotate_acc(acc_tile_t& acc, const float2* __restrict__ table, int seq, int M,
                                                int mw, int lane) {
  const int g = lane >> 4;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    int m = mw + i * 16 + (lane & 15);
    m = m < M ? m : M - 1;                                 // rows past the end are never stored; keep the table read in bounds
    const float4* row = reinterpret_cast<const float4*>(table + (size_t)(m % seq) * 64);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = j * 16 + g * 4;                        // this lane's 4 consecutive frequencies
      const float4 t0 = row[c / 2], t1 = row[c / 2 + 1];   // (cos, sin) of c, c + 1 and of c + 2, c + 3
      const float cs[4] = {t0.x, t0.z, t1.x, t1.z}, sn[4] = {t0.y, t0.w, t1.y, t1.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float lo = acc[i][j][e], hi = acc[i][j + 4][e];
        acc[i][j][e] = lo * cs[e] - hi * sn[e];
        acc[i][j + 4][e] = hi * cs[e] + lo * sn[e];
      }
    }
  }
}

// Epilogue of the gate / up projection with the MLP activation fused in.  B is in paired slabs, so the wave tile's
// columns 0..63 are gate columns base..base + 63 (base = 128 tile_n + 64 wn) and its columns 64..127 the up columns of
// the same indices: a = silu(gate) * up is formed from the fp32 accumulators.  Stored: gate and up (bf16) where the
// plain [gate | up] layout has them (GU[m][base + c], GU[m][f + base + c]) and a (bf16) at A[m][base + c]; each of
// the three is a 128-byte row segment.  32 rows at a time go through the wave's own LDS ([32][400 B]).
__device__ __forceinline__ void epilogue_swiglu_rows(acc_tile_t& acc, char* smem, int wave, int lane, bf16_t* GU,
                                                     bf16_t* Aout, int M, int f, int ldgu, int mw, int base) {
  char* const wl = smem + wave * 32768;
  constexpr int RS = 400;                                  // row stride: 3 x 128 B + 16 (16 rows start at 16 different chunks)
  const int g = lane >> 4;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bf16x4_t og, ou, oa;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float gv = acc[2 * i + h][j][e], uv = acc[2 * i + h][j + 4][e];
          og[e] = (bf16_t)gv;
          ou[e] = (bf16_t)uv;
          // silu(g) u = g u / (1 + 2^(-g log2 e)): hardware exp2 and reciprocal (1 ulp each), far below bf16's 2^-9
          oa[e] = (bf16_t)(gv * uv * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.44269504088896f * gv)));
        }
        const int r = h * 16 + (lane & 15), cb = (j * 16 + g * 4) * 2;   // byte offset of the 4 columns within a 128-byte segment
        *reinterpret_cast<bf16x4_t*>(wl + r * RS + cb) = og;
        *reinterpret_cast<bf16x4_t*>(wl + r * RS + 128 + cb) = ou;
        *reinterpret_cast<bf16x4_t*>(wl + r * RS + 256 + cb) = oa;
      }
    // the wave reads back only what it wrote itself: no workgroup barrier (the compiler orders LDS accesses of a wave)
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int it = 0; it < 12; ++it) {                      // 32 rows x 24 chunks of 16 bytes
      const int q = it * 64 + lane, row = q / 24, cc = q % 24, seg = cc >> 3, w8 = (cc & 7) * 8;
      const u32x4 v = *reinterpret_cast<const u32x4*>(wl + row * RS + seg * 128 + (cc & 7) * 16);
      const int m = mw + i * 32 + row;
      if (m < M) {
        bf16_t* dst = seg == 2 ? Aout + (size_t)m * f + base + w8 : GU + (size_t)m * ldgu + (seg == 1 ? f : 0) + base + w8;
        *reinterpret_cast<u32x4*>(dst) = v;
      }
    }
  }
}

// f(std::integral_constant<int, P0>{}), ..., f(std::integral_constant<int, P1 - 1>{}): a loop whose index is a
// constant expression inside the body
template <int P0, class F, int... I>
__device__ __forceinline__ void for_range_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, P0 + I>{}), ...);
}
template <int P0, int P1, class F>
__device__ __forceinline__ void for_range(F&& f) {
  for_range_impl<P0>(f, std::make_integer_sequence<int, P1 - P0>{});
}

// Main loop of the direct kernels: position t (0..63) within a phase of 64 MFMAs.  Tile load n (0..7) of the phase goes
// out ahead of position LOAD_POS[n]: every eighth, moved to t % 3 == 2, the positions that carry no fragment read
__device__ constexpr int load_at(int t) {
  constexpr int LOAD_POS[8] = {5, 14, 20, 29, 38, 44, 53, 62};
  for (int n = 0; n < 8; ++n)
    if (LOAD_POS[n] == t) return n;
  return -1;
}

// One output tile.  TNL = false: A(m, k) at A[m * lda + k], B(n, k) at B[n * ldb + k].  TNL = true: A[k * lda + m],
// B[k * ldb + n]; there K may be anything (k-rows past it lie past the operand and read as zero).  Otherwise K % 64 == 0 unless
// RAGGED (then K % 8 == 0): the 16-byte chunks of the last k-tile that lie past K are fetched out of range.
template <bool TNL, int EPI, bool RAGGED = false>
__device__ __forceinline__ void direct_tile(char* smem, const bf16_t* __restrict__ A, const bf16_t* __restrict__ B,
                                            void* __restrict__ Cv, const bf16_t* __restrict__ R, int M, int N, int K, int lda,
                                            int ldb, int ldc, unsigned a_bytes, unsigned b_bytes, int tile_m, int tile_n,
                                            bool b_slab = false, const GemmExtra& ex = GemmExtra()) {
  constexpr int BM = 256, BN = 256, WM = 2, WN = 2;
  constexpr int OPB = 32768;                    // one operand of one stage
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;

  const int m0 = tile_m * BM, n0 = tile_n * BN;

  acc_tile_t acc;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;

  // Fragment i (0..7) of an operand = its 16 rows 16 i .. (wave part of 128 rows); lane = row (lane & 15), k-group
  // lane >> 4 of 8 k.  Byte address of this lane's read within a slot, without the wave part:
  //  NT: faddr[(i & 3) * 2 + ks]; the swizzle repeats every 64 rows, so i + 4 is an immediate offset of 8192
  //  TN: faddr[i]; k-step and k-quad are immediates (16384 and 2048 bytes)
  int faddr[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int g = lane >> 4;
    if (TNL) {
      const int e = (lane >> 2) & 3, r = lane & 3;
      faddr[q] = (g * 8 + e) * 512 + (((2 * q + (r >> 1)) ^ (e << 2) ^ ((g & 1) << 1)) << 4) + (r & 1) * 8;
    } else {
      const int row = (q >> 1) * 16 + (lane & 15), ks = q & 1;
      faddr[q] = row * ROW_BYTES + (((ks * 4 + g) ^ swz(row)) << 4);
    }
  }
  // tile loads: 16 per wave and tile, t even -> A, t odd -> B, each 1 KB of LDS; voff = this lane's byte offset
  // within the k-tile (out of range for rows or columns past the operand); the k-tile moves the descriptor's base
  unsigned voff[16];
  unsigned a_tile, b_tile;
  if (TNL) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = 2 * (wave * 8 + j) + (lane >> 5);
      const int c16 = (lane & 31) ^ ((k & 3) << 2) ^ (((k >> 3) & 1) << 1);
      const int ca = m0 + c16 * 8, cb = n0 + c16 * 8;
      voff[2 * j] = ca < M ? (unsigned)k * (unsigned)lda * 2u + (unsigned)ca * 2u : 0xFFFFFF00u;
      voff[2 * j + 1] = cb < N ? (unsigned)k * (unsigned)ldb * 2u + (unsigned)cb * 2u : 0xFFFFFF00u;
    }
    a_tile = 64u * (unsigned)lda * 2u;
    b_tile = 64u * (unsigned)ldb * 2u;
  } else {
    const int lrow = lane >> 3, c0 = (lane & 7) ^ lrow;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const unsigned coff = (unsigned)((c0 ^ j) << 4);
      voff[2 * j] = (unsigned)(m0 + wave * 64 + j * 8 + lrow) * (unsigned)lda * 2u + coff;
      // B in slabs: the 256 rows x 64 columns of tile column tile_n and k-tile kt lie together (32 KB, row-major
      // inside), so one load instruction covers 1 KB of consecutive memory instead of 128 bytes of 8 rows each
      voff[2 * j + 1] = b_slab ? (unsigned)tile_n * (unsigned)(K / BK) * 32768u + (unsigned)(wave * 64 + j * 8 + lrow) * 128u + coff
                               : (unsigned)(n0 + wave * 64 + j * 8 + lrow) * (unsigned)ldb * 2u + coff;
    }
    a_tile = BK * 2;
    b_tile = b_slab ? 32768u : BK * 2;
  }
  const int nk = (K + BK - 1) / BK;
  auto drop_tail = [&](bool is_b) __attribute__((always_inline)) {       // ahead of the loads of the last k-tile
    const int c0 = (lane & 7) ^ (lane >> 3), valid = (K % BK) >> 3;
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if ((c0 ^ j) >= valid) voff[2 * j + (is_b ? 1 : 0)] = 0xFFFFFF00u;
  };
  // Descriptor of an operand: base and length both move with the k-tile, so that what lies past the operand's end reads as
  // zero whatever the range check makes of a scalar offset.  Past the last tile the length is zero (the load then moves
  // nothing from memory and zero-fills its slot, so the count of loads in flight is the same on every trip).
  // The scalar steps of the main loop are written in assembly so that they stay at the positions they are written at: left to
  // the compiler they gather at the top of the trip, 40 instructions during which the matrix unit has nothing to do.
  struct Desc { unsigned lo, hi, left, len; };          // left = bytes from the tile's base to the operand's end
  auto start = [&](const void* p, unsigned bytes) __attribute__((always_inline)) {
    const unsigned long long a = (unsigned long long)p;
    Desc d;
    d.lo = __builtin_amdgcn_readfirstlane((int)(unsigned)a);
    d.hi = __builtin_amdgcn_readfirstlane((int)(unsigned)(a >> 32)) & 0xffff;
    d.left = d.len = __builtin_amdgcn_readfirstlane((int)bytes);
    return d;
  };
  auto move_base = [](Desc& d, unsigned step) __attribute__((always_inline)) {
    asm volatile("s_add_u32 %0, %0, %2\n\ts_addc_u32 %1, %1, 0" : "+s"(d.lo), "+s"(d.hi) : "s"(step) : "scc");
  };
  auto move_end = [](Desc& d, unsigned step, int tile, int tiles) __attribute__((always_inline)) {
    asm volatile("s_sub_u32 %0, %0, %2\n\ts_cmp_lt_i32 %3, %4\n\ts_cselect_b32 %1, %0, 0"
                 : "+s"(d.left), "=&s"(d.len) : "s"(step), "s"(tile), "s"(tiles) : "scc");
  };
  auto add = [](unsigned& r, unsigned x, unsigned y) __attribute__((always_inline)) {
    asm volatile("s_add_u32 %0, %1, %2" : "=s"(r) : "s"(x), "s"(y) : "scc");
  };
  // ring arithmetic on byte offsets of slots
  auto slot_after = [](unsigned& r, unsigned x) __attribute__((always_inline)) {
    asm volatile("s_add_u32 %0, %1, %2\n\ts_cmp_eq_u32 %0, %3\n\ts_cselect_b32 %0, 0, %0"
                 : "=&s"(r) : "s"(x), "n"(32768), "n"(163840) : "scc");
  };
  auto slot_before = [](unsigned& r, unsigned x) __attribute__((always_inline)) {
    asm volatile("s_sub_u32 %0, %1, %2\n\ts_cselect_b32 %0, %3, %0" : "=&s"(r) : "s"(x), "n"(32768), "n"(131072) : "scc");
  };
  auto slot_after_next = [](unsigned& x) __attribute__((always_inline)) {
    unsigned y;
    asm volatile("s_add_u32 %0, %0, %2\n\ts_sub_u32 %1, %0, %3\n\ts_cselect_b32 %0, %0, %1"
                 : "+s"(x), "=&s"(y) : "n"(65536), "n"(163840) : "scc");
  };
  auto words = [](const Desc& d) __attribute__((always_inline)) { return i32x4_t{(int)d.lo, (int)d.hi, (int)d.len, 0x00020000}; };
  const unsigned lds0 = (unsigned)(size_t)(lds_void_t*)smem;
  // load idx (0..7) of this wave for one operand: set_m0 gives the ring slot's address plus this wave's 8 KB share as
  // `base`; m0 = LDS address of the load, written one position ahead of the load (the hardware wants an instruction in between)
  unsigned m0v;
  auto set_m0 = [](unsigned base, auto idx_c) __attribute__((always_inline)) {
    constexpr int idx = decltype(idx_c)::value;
    unsigned r;
    asm volatile("s_add_u32 %0, %1, %2" : "={m0}"(r) : "s"(base), "n"(idx * 1024) : "scc");
    return r;
  };
  auto issue_one = [&](i32x4_t desc, bool is_b, auto idx_c) __attribute__((always_inline)) {
    constexpr int idx = decltype(idx_c)::value;
    const unsigned vo = voff[2 * idx + (is_b ? 1 : 0)];
    const unsigned mm = m0v;
    asm volatile("buffer_load_dwordx4 %0, %1, 0 offen lds" :: "v"(vo), "s"(desc), "{m0}"(mm) : "memory");
  };
  const unsigned lds_wave = lds0 + wave * 8192;
  // LDS is a ring of five 32 KB slots which the operands take in the order A0 B0 A1 B1 A2 ... (operand u in slot
  // u % 5).  While tile kt is computed its two slots are read, the two that tile kt - 1 has left are refilled with
  // B of tile kt + 1 and A of tile kt + 2, and A of tile kt + 1 sits in the fifth.  The sync at the top of tile kt
  // wants both operands of tile kt landed: every load but this wave's last 8 (A of tile kt + 1), which stay in
  // flight across the barrier, so the memory pipe never runs empty.  The slots of a tile change from trip to
  // trip: cur[] = LDS addresses of the fragments of the tile being read (0..7 A, 8..15 B), rebuilt for the next tile
  // under the MFMAs that end the trip, when nothing reads the old ones any more.
  constexpr int WPART = TNL ? 256 : 16384;           // the 128 rows (NT) or columns (TN) of a wave within a slot
  const unsigned base_fa = lds0 + wm * WPART, base_fb = lds0 + wn * WPART;
  int cur[16];
  bf16x8_t fr[2][16];                                // [k-step parity][0..7 A, 8..15 B]
  i16x4_t half0;                                     // TN: first half of the fragment being read
  // TN: the two 8-byte halves of fragment q are one transposing read each; NT: one 16-byte read
  auto read_nt = [&](int ks, int q) __attribute__((always_inline)) {
    typedef __attribute__((address_space(3))) bf16x8_t lds_bf16x8_t;
    const int i = q & 7;
    fr[ks][q] = *(const lds_bf16x8_t*)(unsigned)(cur[(q & 8) + (i & 3) * 2 + ks] + (i >> 2) * 8192);
  };
  auto read_tn = [&](int ks, int q, int half) __attribute__((always_inline)) {
    const i16x4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t*)(unsigned)(cur[q] + ks * 16384 + half * 2048));
    if (half == 0) half0 = v;
    else fr[ks][q] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(half0, v, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  // order in which a phase needs its fragments (MFMA t of a phase: i = t / 8, j walks to and fro, so that consecutive
  // MFMAs share an operand): A0, B0 .. B7, A1 .. A7
  constexpr int RQ[16] = {0, 8, 9, 10, 11, 12, 13, 14, 15, 1, 2, 3, 4, 5, 6, 7};
  auto mma_one = [&](int set, int t) __attribute__((always_inline)) {
    const int i = t >> 3, j = (i & 1) ? 7 - (t & 7) : (t & 7);
    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[set][8 + j], fr[set][i], acc[i][j], 0, 0, 0);
  };
  // One trip of the loop = two phases of 64 MFMAs: phase 0 multiplies k-step 1 of the previous tile (fragment set 1, in
  // registers) while the fragments of k-step 0 of tile kt are read, phase 1 multiplies k-step 0 of tile kt while those of
  // k-step 1 are read.  An MFMA occupies the matrix pipe for 16 cycles, which is room for the issue of two or three other
  // instructions, so no position carries more than one of:
  //  * fragment reads, out by position 47 of the phase (t % 3 == 0, for TN, which has two per fragment, also 1), so that
  //    they have landed when the tile barrier is reached;
  //  * the 16 tile loads of the trip (t % 3 == 2): in phase 0 the 8 of B of tile kt + 1 into the slot at pa, in phase 1
  //    those of A of tile kt + 2 into the slot at pb;
  //  * the fragment addresses of the next tile, one each at positions 48..63 of phase 1.
  // The ring in the trip of tile kt, as byte offsets: pa = slot that A of tile kt - 1 has left, which takes B of kt + 1 (operand
  // 2 kt + 3); the one after it takes A of kt + 2; the one before it holds A of kt + 1.
  unsigned pa = 0, pb = 0, na = 0;
  unsigned ld_b = 0, ld_a = 0;                       // LDS addresses (this wave's share) of the two slots to refill
  unsigned at_a = base_fa + 2 * OPB, at_b = base_fb + 3 * OPB;   // where the next tile's fragments are
  Desc da = start(A, a_bytes), db = start(B, b_bytes);
  const int nk2 = nk - 2;
  int kt = 0;
  auto position = [&](auto p_c, bool refill, bool next) __attribute__((always_inline)) {
    constexpr int p = decltype(p_c)::value, ph = p >> 6, t = p & 63;
    constexpr int n = load_at(t);
    __builtin_amdgcn_sched_barrier(0);
    // every fragment of this phase has landed (requested 16 MFMAs ago at the latest): said once, so that the compiler
    // does not put a wait ahead of each fragment's first use (lgkmcnt(0), the other counters left alone)
    if (t == 0) __builtin_amdgcn_s_waitcnt(0xC07F);
    if (RAGGED && t == 0 && refill) {
      if (kt + 1 + ph == nk - 1) drop_tail(ph == 0);
    }
    if constexpr (n >= 0) {
      if (refill) issue_one(words(ph == 0 ? db : da), ph == 0, std::integral_constant<int, n>{});
    }
    if (next && t < 48) {
      if (TNL) { if (t % 3 < 2) read_tn(ph, RQ[t / 3], t % 3); }
      else if (t % 3 == 0) read_nt(ph, RQ[t / 3]);
    }
    if (next && ph == 0) {                           // for phase 1: A's descriptor and slot, the next tile's fragments
      if (t == 48) move_base(da, a_tile);
      if (t == 49) move_end(da, a_tile, kt, nk2);
      if (t == 50) slot_after(pb, pa);
      if (t == 51) add(ld_a, lds_wave, pb);
      if (t == 54) slot_before(na, pa);
      if (t == 55) { add(at_a, base_fa, na); add(at_b, base_fb, pa); }
      if (t == 56) slot_after_next(pa);
    }
    if (next && ph == 1) {                           // for the next trip: B's descriptor and slot
      if (t == 48) move_base(db, b_tile);
      if (t == 49) move_end(db, b_tile, kt, nk2);
      if (t == 50) add(ld_b, lds_wave, pa);
    }
    if (ph == 1 && t >= 48) {
      constexpr int q = t >= 48 ? t - 48 : 0;
      cur[q] = faddr[q & 7] + (int)(q < 8 ? at_a : at_b);
      asm volatile("" : "+v"(cur[q]));               // here, not where the address is first used
    }
    if constexpr (t < 63 && load_at(t + 1) >= 0) {
      if (refill) m0v = set_m0(ph == 0 ? ld_b : ld_a, std::integral_constant<int, load_at(t + 1)>{});
    }
    __builtin_amdgcn_sched_barrier(0);
    mma_one(ph ^ 1, t);
  };
  auto trip = [&](auto p0, auto p1, bool refill, bool next) __attribute__((always_inline)) {
    for_range<decltype(p0)::value, decltype(p1)::value>([&](auto p) __attribute__((always_inline)) { position(p, refill, next); });
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr std::integral_constant<int, 0> P0{};
  constexpr std::integral_constant<int, 64> P64{};
  constexpr std::integral_constant<int, 128> P128{};
#define OPTSTAGE_TILE_SYNC(n) asm volatile("s_waitcnt vmcnt(" #n ") lgkmcnt(0)\n\ts_barrier" ::: "memory")
#pragma unroll
  for (int u = 0; u < 5; ++u) {
    Desc& d = u & 1 ? db : da;
    if (u >= 2) { move_base(d, u & 1 ? b_tile : a_tile); move_end(d, u & 1 ? b_tile : a_tile, u >> 1, nk); }
    if (RAGGED && (u >> 1) == nk - 1) drop_tail((u & 1) != 0);
    for_range<0, 8>([&](auto idx) __attribute__((always_inline)) {
      m0v = set_m0(lds_wave + u * OPB, idx);
      asm volatile("s_nop 0");
      issue_one(words(d), (u & 1) != 0, idx);
    });
  }
#pragma unroll
  for (int q = 0; q < 16; ++q) cur[q] = faddr[q & 7] + (int)(q < 8 ? base_fa : base_fb + OPB);
  OPTSTAGE_TILE_SYNC(24);
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    if (TNL) { read_tn(0, RQ[q], 0); read_tn(0, RQ[q], 1); }
    else read_nt(0, RQ[q]);
  }
  trip(P64, P128, false, true);
  for (kt = 1; kt < nk - 1; ++kt) {
    OPTSTAGE_TILE_SYNC(8);
    trip(P0, P128, true, true);
  }
  if (nk > 1) {                                      // the last tile: nothing is left to load
    OPTSTAGE_TILE_SYNC(8);
    trip(P0, P128, false, true);
  }
  const int mw = m0 + wm * (BM / WM), nw = n0 + wn * (BN / WN);
  // No tile load is in flight from here on: the last ones went out a trip ago, so this waits for nothing, and what the epilogue
  // requests below can neither be mistaken for a tile load nor has to be counted, wherever the compiler puts it.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  // What the epilogue adds is requested ahead of the last 64 MFMAs, which read and load nothing any more: the residual, or
  // the old values of the first 64 rows (rows and columns past the end read a value that is not used).
  // (4096 x 8192 x 8192 with residual 1467 -> 1513 TFLOP/s, grouped TN set of a hidden-8192 layer 1352 -> 1366.)
  f32x4_t old[EPI == EPI_ACCUM ? 32 : 1];
  bf16x4_t res[EPI == EPI_RESID ? 64 : 1];
  if constexpr (EPI == EPI_ACCUM) {
#pragma unroll
    for (int p2 = 0; p2 < 32; ++p2) old[p2] = old_value(reinterpret_cast<const float*>(Cv), p2, lane, M, N, ldc, mw, nw);
  }
  if constexpr (EPI == EPI_RESID) {
#pragma unroll
    for (int q = 0; q < 64; ++q) {
      const int m = min(mw + (q >> 3) * 16 + (lane & 15), M - 1), n = min(nw + (q & 7) * 16 + (lane >> 4) * 4, N - 4);
      res[q] = *reinterpret_cast<const bf16x4_t*>(R + (size_t)m * ldc + n);
    }
  }
  trip(P0, P64, false, false);
  // every wave is done with the operand tiles, and none of them has a tile load in flight: LDS is the epilogue's
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#undef OPTSTAGE_TILE_SYNC
  if constexpr (EPI == EPI_ACCUM || EPI == EPI_STOREF) {
    epilogue_f32_rows<EPI>(acc, old, smem, wave, lane, reinterpret_cast<float*>(Cv), M, N, ldc, mw, nw);
  } else if constexpr (EPI == EPI_SWIGLU) {
    epilogue_swiglu_rows(acc, smem, wave, lane, reinterpret_cast<bf16_t*>(Cv), reinterpret_cast<bf16_t*>(ex.a_out), M, ex.f, ldc,
                         mw, tile_n * 128 + wn * 64);
  } else {
    if (EPI == EPI_ROPE && nw < ex.rot_cols)         // this wave's 128 columns are a q or k head
      rope_rotate_acc(acc, ex.table, ex.seq, M, mw, lane);
    epilogue_bf16_rows<(EPI == EPI_ROPE ? EPI_STORE : EPI)>(acc, res, smem, wave, lane, reinterpret_cast<bf16_t*>(Cv), M, N, ldc, mw, nw);
  }
}

// Consecutive hardware workgroup ids go to different XCDs: give every XCD one contiguous range of the sequence
__device__ __forceinline__ int xcd_remap(int id, int n) { return (n & 7) == 0 ? (id & 7) * (n >> 3) + (id >> 3) : id; }

// Which output tile workgroup `id` of a problem computes (id counted from the problem's first workgroup; n = the
// problem's tile count).
//  order 0: the tile sequence walks groups of 8 tile rows column by column, and every XCD takes one contiguous
//           eighth of it: the 32 tiles an XCD has in flight form an 8 x 4 patch that shares 12 operand panels in its
//           L2, but the eight XCDs work far apart and share nothing.
//  order 1: every round of 256 workgroups covers one 16 x 16 patch of tiles; XCD x (= id % 8) takes the 4 x 8 part
//           at rows 4 (x % 4), columns 8 (x / 4) of it (12 panels in its L2 as before), so the chip as a whole touches
//           32 panels per round instead of 96 and two thirds of the L2 misses can hit in the memory-side cache.
//           Tiles outside the whole patches (a strip on the right, one at the bottom) come last, column by column.
__device__ __forceinline__ void tile_coords(int id, int n, int tiles_m, int tiles_n, int order, int& tile_m, int& tile_n) {
  if (order == 1) {
    const int nfm = tiles_m >> 4, nfn = tiles_n >> 4, whole = nfm * nfn * 256;
    if (id < whole) {
      const int sp = id >> 8, x = id & 7, w = (id >> 3) & 31;
      tile_m = (sp % nfm) * 16 + (x & 3) * 4 + (w & 3);
      tile_n = (sp / nfm) * 16 + (x >> 2) * 8 + (w >> 2);
      return;
    }
    int q = id - whole;
    const int rn = tiles_n - nfn * 16, rm = tiles_m - nfm * 16;
    if (q < tiles_m * rn) { tile_m = q % tiles_m; tile_n = nfn * 16 + q / tiles_m; return; }
    q -= tiles_m * rn;
    tile_m = nfm * 16 + q % rm;
    tile_n = q / rm;
    return;
  }
  const int pid = xcd_remap(id, n);
  constexpr int GM = 8;
  const int grp = pid / (GM * tiles_n);
  const int first_m = grp * GM;
  const int gsz = min(tiles_m - first_m, GM);
  const int in_grp = pid - grp * GM * tiles_n;
  tile_m = first_m + in_grp % gsz;
  tile_n = in_grp / gsz;
}

template <bool TNL, int EPI, bool RAGGED>
__global__ __launch_bounds__(256) void gemm_bf16_direct_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B,
                                                               void* __restrict__ Cv, const bf16_t* __restrict__ R, int M, int N,
                                                               int K, int lda, int ldb, int ldc, int tiles_m, int tiles_n,
                                                               unsigned a_bytes, unsigned b_bytes, int b_slab, const GemmExtra ex,
                                                               int order) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int tile_m, tile_n;
  tile_coords(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, order, tile_m, tile_n);
  direct_tile<TNL, EPI, RAGGED>(smem, A, B, Cv, R, M, N, K, lda, ldb, ldc, a_bytes, b_bytes, tile_m, tile_n, !TNL && b_slab != 0, ex);
}

// Several independent products with the same K in one launch (the weight-gradient GEMMs of a W op: four per
// layer, none depending on another): their tiles form one sequence, so the partly filled last round of
// workgroups that every product would leave behind on its own happens once.
constexpr int MAX_GROUP = 16;
struct GroupedProblem {
  const bf16_t* A; const bf16_t* B; void* C; const bf16_t* R;
  int M, N, lda, ldb, ldc, tiles_m, tiles_n, first_tile;
  unsigned a_bytes, b_bytes;
};
struct GroupedArgs { int n, K, total, order; GroupedProblem p[MAX_GROUP]; };

template <bool TNL, int EPI>
__global__ __launch_bounds__(256) void gemm_bf16_direct_grouped_kernel(const GroupedArgs g) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  // order 1 within each problem: workgroups with equal (id - first_tile) % 8 are on one XCD whatever first_tile is,
  // and any 256 consecutive ids are in flight together, which is all the patch mapping relies on
  const int id = g.order == 1 ? (int)blockIdx.x : xcd_remap(blockIdx.x, g.total);
  int q = 0;
  for (int i = 1; i < g.n; ++i)
    if (id >= g.p[i].first_tile) q = i;
  const GroupedProblem& pr = g.p[q];
  int tile_m, tile_n;
  if (g.order == 1) {
    tile_coords(id - pr.first_tile, pr.tiles_m * pr.tiles_n, pr.tiles_m, pr.tiles_n, 1, tile_m, tile_n);
  } else {                                   // the sequence position is already XCD-mapped over the whole launch
    constexpr int GM = 8;
    const int pid = id - pr.first_tile, grp = pid / (GM * pr.tiles_n), first_m = grp * GM;
    const int gsz = min(pr.tiles_m - first_m, GM), in_grp = pid - grp * GM * pr.tiles_n;
    tile_m = first_m + in_grp % gsz;
    tile_n = in_grp / gsz;
  }
  direct_tile<TNL, EPI>(smem, pr.A, pr.B, pr.C, pr.R, pr.M, pr.N, g.K, pr.lda, pr.ldb, pr.ldc, pr.a_bytes, pr.b_bytes, tile_m, tile_n);
}

// Measured on the weight-gradient set of the grouped-query stage (8 products, one launch): order 1 1229 TFLOP/s against
// 1187 for order 0 (TN with the fp32 read-add-store, whose operand panels are re-read most: 2.6 x the algorithmic bytes
// miss the L2); the NT products are within 0.5 % either way and keep order 0.
constexpr int tile_order(bool tnl) { return tnl ? 1 : 0; }

template <bool TNL, int EPI, bool RAGGED = false>
hipError_t launch_direct(const void* A, const void* B, void* C, const void* R, int M, int N, int K, int lda, int ldb,
                         int ldc, hipStream_t s, bool b_slab = false, const GemmExtra& ex = GemmExtra()) {
  auto kern = gemm_bf16_direct_kernel<TNL, EPI, RAGGED>;
  constexpr int smem = 163840;
  static LdsAttrOnce lds_attr;
  if (hipError_t e = lds_attr.ensure(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  const int tiles_m = (M + 255) / 256, tiles_n = (N + 255) / 256;
  // byte extent of each operand: whatever lies past it reads as zero
  const unsigned a_bytes = (unsigned)(TNL ? ((size_t)(K - 1) * lda + M) * 2 : ((size_t)(M - 1) * lda + K) * 2);
  const unsigned b_bytes = b_slab ? (unsigned)((size_t)tiles_n * (K / 64) * 32768)
                                  : (unsigned)(TNL ? ((size_t)(K - 1) * ldb + N) * 2 : ((size_t)(N - 1) * ldb + K) * 2);
  hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(256), smem, s, (const bf16_t*)A, (const bf16_t*)B, C, (const bf16_t*)R,
                     M, N, K, lda, ldb, ldc, tiles_m, tiles_n, a_bytes, b_bytes, b_slab ? 1 : 0, ex, tile_order(TNL));
  return hipGetLastError();
}

// the direct path needs 32-bit byte offsets (including what a partial edge tile reaches past the operand)
bool direct_applies(bool tnl, int M, int N, int K, int lda, int ldb) {
  const unsigned long long lim = 0xF0000000ull;
  if (tnl) return ((unsigned long long)(K + 63) * lda * 2 < lim) && ((unsigned long long)(K + 63) * ldb * 2 < lim);
  return ((unsigned long long)(M + 256) * lda * 2 < lim) && ((unsigned long long)(N + 256) * ldb * 2 < lim);
}
template <bool TNL, int EPI>
hipError_t launch_direct_grouped(int n, const GemmProblem* pr, int K, hipStream_t s) {
  auto kern = gemm_bf16_direct_grouped_kernel<TNL, EPI>;
  constexpr int smem = 163840;
  static LdsAttrOnce lds_attr;
  if (hipError_t e = lds_attr.ensure(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  GroupedArgs g;
  g.n = n;
  g.K = K;
  int total = 0;
  for (int i = 0; i < n; ++i) {
    GroupedProblem& q = g.p[i];
    q.A = (const bf16_t*)pr[i].A; q.B = (const bf16_t*)pr[i].B; q.C = pr[i].C; q.R = (const bf16_t*)pr[i].R;
    q.M = pr[i].M; q.N = pr[i].N; q.lda = pr[i].lda; q.ldb = pr[i].ldb; q.ldc = pr[i].ldc;
    q.tiles_m = (q.M + 255) / 256;
    q.tiles_n = (q.N + 255) / 256;
    q.first_tile = total;
    total += q.tiles_m * q.tiles_n;
    q.a_bytes = (unsigned)(TNL ? ((size_t)(K - 1) * q.lda + q.M) * 2 : ((size_t)(q.M - 1) * q.lda + K) * 2);
    q.b_bytes = (unsigned)(TNL ? ((size_t)(K - 1) * q.ldb + q.N) * 2 : ((size_t)(q.N - 1) * q.ldb + K) * 2);
  }
  g.total = total;
  g.order = tile_order(TNL);
  hipLaunchKernelGGL(kern, dim3(total), dim3(256), smem, s, g);
  return hipGetLastError();
}

template <bool RC, int EPI>
hipError_t launch_staged(const void* A, const void* B, void* C, const void* R, int M, int N, int K, int lda, int ldb,
                         int ldc, hipStream_t s) {
  auto kern = gemm_bf16_staged_kernel<RC, EPI>;
  constexpr int smem = 2 * (128 + 128) * ROW_BYTES;
  static LdsAttrOnce lds_attr;
  if (hipError_t e = lds_attr.ensure(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  const int tiles_m = (M + 127) / 128, tiles_n = (N + 127) / 128;
  hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(256), smem, s, (const bf16_t*)A, (const bf16_t*)B, C,
                     (const bf16_t*)R, M, N, K, lda, ldb, ldc, tiles_m, tiles_n);
  return hipGetLastError();
}

// Products of more than 256 tiles of 128 x 128 but fewer than 128 of 256 x 256: the direct kernel leaves half the chip idle and more, but
// its loop is 5 (NT) to 15 % (TN) cheaper than that of the register-staged kernel, two of whose workgroups share a compute
// unit.  Both give the same bits.  Time of the direct kernel over the staged one:
//  * rows that do not start on 128 bytes (NT): every 128-byte piece of a tile is two cache lines.  K 1624: 1.03 to 1.18.
//  * residual: loads and stores of a whole tile by one compute unit.  K 64 / 512 / 1024 / 2048: 1.15 - 1.33 / 1.00 - 1.08 /
//    .98 - 1.04 / .97 - 1.00.
//  * no more work than one full tile of 128 per compute unit, in many cut ones (1053 x 3664, 300 x 12000): store, NT, K 64 / 1024 /
//    2048: 1.09 - 1.23 / .97 - 1.05 / .96 - .99; accumulate, TN, K 64 / 512 / 768: .95 - 1.25 / .86 - 1.02 / .86 - .99.
//  * otherwise, whole tiles along N: .77 - 1.02 at every K; cut ones: accumulate .84 - 1.02; store, NT, K 64 / 768 / 1024:
//    1.00 - 1.04 / .92 - 1.04 / .92 - 1.01; store, TN, K 64 / 128 / 256: .98 - 1.14 / .95 - 1.05 / .95 - .98.
bool direct_on_few_tiles(bool tnl, int epi, int M, int N, int K, int lda, int ldb) {
  const bool spare = (long long)M * N <= 256ll * 128 * 128;
  if (!tnl && ((K | lda | ldb) & 63)) return false;
  if (epi == EPI_RESID) return !spare && K >= 2048;
  const int from = spare ? (tnl ? 768 : 2048) : N % 256 == 0 || epi == EPI_ACCUM ? 0 : tnl ? 256 : 1024;
  return K >= from;
}

// The direct kernels from 128 tiles of 256 x 256 on.  Up to 256 tiles of 128 x 128 (one per compute unit) the small kernels, on tiles
// of 128 and 64; between the two the rule above.  The register-staged kernel also takes leading dimensions of 2^23
// elements and more, whose rows within one tile span more than 32-bit offsets reach.
enum Route { ROUTE_DIRECT, ROUTE_SMALL, ROUTE_STAGED };
Route route(bool rc, int epi, int M, int N, int K, int lda, int ldb) {
  const long tiles256 = (long)((M + 255) / 256) * ((N + 255) / 256), tiles128 = (long)((M + 127) / 128) * ((N + 127) / 128);
  const bool between = tiles256 < 128 && tiles128 > 256;
  if ((tiles256 >= 128 || (between && direct_on_few_tiles(rc, epi, M, N, K, lda, ldb))) && direct_applies(rc, M, N, K, lda, ldb)) return ROUTE_DIRECT;
  return !between && gemm_bf16_small_applies(M, N, K, lda, ldb) ? ROUTE_SMALL : ROUTE_STAGED;
}
template <bool RC, int EPI>
hipError_t launch_layout(const void* A, const void* B, void* C, const void* R, int M, int N, int K, int lda, int ldb,
                         int ldc, hipStream_t s) {
  switch (route(RC, EPI, M, N, K, lda, ldb)) {
    case ROUTE_DIRECT:
      if (!RC && K % BK) return launch_direct<RC, EPI, !RC>(A, B, C, R, M, N, K, lda, ldb, ldc, s);
      return launch_direct<RC, EPI>(A, B, C, R, M, N, K, lda, ldb, ldc, s);
    case ROUTE_SMALL: return launch_gemm_bf16_small(RC ? GEMM_TN : GEMM_NT, EPI, GemmProblem{A, B, C, R, M, N, lda, ldb, ldc}, K, s);
    default: return launch_staged<RC, EPI>(A, B, C, R, M, N, K, lda, ldb, ldc, s);
  }
}

}  // namespace

// B in slabs is served by the direct kernel only: shapes that the dispatcher would send elsewhere do not qualify
bool gemm_bf16_slab_applies(int M, int N, int K, int lda) {
  if (M <= 0 || N <= 0 || K <= 0 || (K % 64) || (lda & 7) || (N & 3)) return false;
  const long tiles_n = (N + 255) / 256, big_tiles = (long)((M + 255) / 256) * tiles_n;
  if (big_tiles < 128 || (unsigned long long)tiles_n * (K / 64) * 32768ull >= 0xF0000000ull) return false;
  return direct_applies(false, M, N, K, lda, 8);
}

// The fused epilogues run on the direct kernel only, on whole heads / whole gate-up pairs: what must hold for them
bool gemm_bf16_fused_applies(int epi, int M, int N, int K, int lda, int head_dim) {
  if (epi == EPI_ROPE) return head_dim == 128 && (N % 128) == 0 && (N & 3) == 0 && direct_applies(false, M, N, K, lda, K) &&
                              (long)((M + 255) / 256) * ((N + 255) / 256) >= 128 && (lda & 7) == 0 && (K % 64) == 0;
  if (epi == EPI_SWIGLU) return (N % 256) == 0 && gemm_bf16_slab_applies(M, N, K, lda);
  return false;
}

// The activation runs in the epilogue of the small kernels: at their sizes its own pass is a launch of 4 us, most of it start and end
// (320 tokens, hidden 1024, ffn 1792, SwiGLU backward 4.8 us of 13 with its product).
// The product's weight must have its plain layout: not at a size where it is kept in slabs.
bool gemm_bf16_act_applies(int M, int N, int K) {
  if (M <= 0 || N <= 0 || K <= 0 || (K & 7) || (N & 3) || gemm_bf16_slab_applies(M, N, K, K)) return false;
  return route(false, EPI_STORE, M, N, K, K, K) == ROUTE_SMALL;
}

hipError_t launch_gemm_bf16(int layout, int epi, const void* A, const void* B, void* C, const void* R, int M, int N,
                            int K, int lda, int ldb, int ldc, hipStream_t s, const GemmExtra* extra) {
  // host-side shape checks: 16-byte vector accesses need these
  if (M <= 0 || N <= 0 || K <= 0) return hipErrorInvalidValue;
  if (epi == EPI_ROPE) {
    // whole heads per wave tile, rotated columns a whole number of heads, table and sequence length given
    if (!extra || !extra->table || extra->seq <= 0 || extra->rot_cols < 0 || extra->rot_cols > N || (extra->rot_cols % 128) ||
        (ldc & 7) || (layout != GEMM_NT && layout != GEMM_NT_SLAB) || !gemm_bf16_fused_applies(epi, M, N, K, lda, 128))
      return hipErrorInvalidValue;
    if (layout == GEMM_NT_SLAB) {
      if (!gemm_bf16_slab_applies(M, N, K, lda)) return hipErrorInvalidValue;
      return launch_direct<false, EPI_ROPE>(A, B, C, R, M, N, K, lda, 64, ldc, s, true, *extra);
    }
    if ((ldb & 7) || ldb < K) return hipErrorInvalidValue;
    return launch_direct<false, EPI_ROPE>(A, B, C, R, M, N, K, lda, ldb, ldc, s, false, *extra);
  }
  if (epi == EPI_SWIGLU) {
    // N = 2 f columns in paired slabs; GU rows of ldc elements, a rows of f elements, 16-byte row segments
    if (!extra || !extra->a_out || extra->f <= 0 || N != 2 * extra->f || (extra->f % 128) || (ldc & 7) || ldc < N ||
        layout != GEMM_NT_SLAB || !gemm_bf16_fused_applies(epi, M, N, K, lda, 0))
      return hipErrorInvalidValue;
    return launch_direct<false, EPI_SWIGLU>(A, B, C, R, M, N, K, lda, 64, ldc, s, true, *extra);
  }
  if (layout == GEMM_NT_SLAB) {
    if ((ldc & 3) || !gemm_bf16_slab_applies(M, N, K, lda)) return hipErrorInvalidValue;
    if (epi == EPI_STORE) return launch_direct<false, EPI_STORE>(A, B, C, R, M, N, K, lda, 64, ldc, s, true);
    if (epi == EPI_RESID) return launch_direct<false, EPI_RESID>(A, B, C, R, M, N, K, lda, 64, ldc, s, true);
    return hipErrorInvalidValue;
  }
  if ((lda & 7) || (ldb & 7) || (ldc & 3) || (N & 3)) return hipErrorInvalidValue;
  if (epi == EPI_GELU || epi == EPI_DGELU || epi == EPI_DSWIGLU) {
    if (layout != GEMM_NT || lda != K || ldb != K || !gemm_bf16_act_applies(M, N, K)) return hipErrorInvalidValue;
    return launch_gemm_bf16_small(GEMM_NT, epi, GemmProblem{A, B, C, R, M, N, lda, ldb, ldc}, K, s);
  }
  if (layout == GEMM_NT) {
    if (K & 7) return hipErrorInvalidValue;
    if (epi == EPI_STORE) return launch_layout<false, EPI_STORE>(A, B, C, R, M, N, K, lda, ldb, ldc, s);
    if (epi == EPI_RESID) return launch_layout<false, EPI_RESID>(A, B, C, R, M, N, K, lda, ldb, ldc, s);
    if (epi == EPI_ACCUM) return launch_layout<false, EPI_ACCUM>(A, B, C, R, M, N, K, lda, ldb, ldc, s);
  } else if (layout == GEMM_TN) {
    if ((M & 7) || (N & 7)) return hipErrorInvalidValue;
    if (epi == EPI_STORE) return launch_layout<true, EPI_STORE>(A, B, C, R, M, N, K, lda, ldb, ldc, s);
    if (epi == EPI_ACCUM) return launch_layout<true, EPI_ACCUM>(A, B, C, R, M, N, K, lda, ldb, ldc, s);
    if (epi == EPI_STOREF) return launch_layout<true, EPI_STOREF>(A, B, C, R, M, N, K, lda, ldb, ldc, s);
  }
  return hipErrorInvalidValue;
}

// n independent products sharing layout, epilogue and K in one launch: whether the set qualifies (every product
// on the direct path, operands aligned as the kernels need, at least half a round of tiles in total)
bool gemm_bf16_grouped_applies(int layout, int n, const GemmProblem* pr, int K) {
  if (n <= 0 || n > MAX_GROUP || K <= 0) return false;
  long tiles = 0;
  for (int i = 0; i < n; ++i) {
    const GemmProblem& q = pr[i];
    if (q.M <= 0 || q.N <= 0) return false;
    if ((q.lda & 7) || (q.ldb & 7) || (q.ldc & 3) || (q.N & 3)) return false;
    if (layout == GEMM_TN && ((q.M & 7) || (q.N & 7))) return false;
    if (layout == GEMM_NT && (K % 64)) return false;
    if (!direct_applies(layout == GEMM_TN, q.M, q.N, K, q.lda, q.ldb)) return false;
    tiles += (long)((q.M + 255) / 256) * ((q.N + 255) / 256);
  }
  return tiles >= 128;
}

// A set that leaves a few tiles for a last round of workgroups (one per compute unit) pays a whole round for them.  Up to 64 such
// tiles are cut off as columns of one product and go to the small kernels, whose sums run over k in the same order; more than 32
// only from K = 1024 on, since a short round costs little (256 tiles and `left` more, store fp32, uncut / cut us: left 16, K 64
// 22.7 / 19.7, K 512 36.2 / 29.7, K 4096 156 / 118; left 32 22.8 / 21.7, 36.3 / 32.5, 156 / 127; left 64 22.7 / 25.8, 36.7 /
// 38.7, K 1024 53.6 / 54.0, K 2048 87.4 / 84.5, K 4096 155 / 148; accumulating and bf16 sets gain more).  The four products of a
// hidden-4096 layer (3088 tiles = 12 rounds and 16 tiles) at 4096 tokens: 1308 -> 1278 us.
constexpr long ROUND = 256, TAIL_TILES = 64, TAIL_TILES_SHORT = 32, TAIL_LONG_K = 1024;
static bool cut_tail(int n, GemmProblem* pr, int epi, int K, GemmProblem* tail) {
  auto up = [](int x) { return (long)(x + 255) / 256; };
  long total = 0, best = TAIL_TILES + 1;
  for (int i = 0; i < n; ++i) total += up(pr[i].M) * up(pr[i].N);
  const long left = total % ROUND;
  if (total < ROUND || !left || left > (K < TAIL_LONG_K ? TAIL_TILES_SHORT : TAIL_TILES)) return false;
  int at = -1;
  long cols = 0;
  for (int i = 0; i < n; ++i) {
    const long tm = up(pr[i].M), c = (left + tm - 1) / tm;
    if (c < up(pr[i].N) && c * tm < best && gemm_bf16_small_applies(pr[i].M, pr[i].N, K, pr[i].lda, pr[i].ldb)) { best = c * tm; at = i; cols = c; }
  }
  if (at < 0) return false;
  const int n0 = (int)(up(pr[at].N) - cols) * 256;
  *tail = pr[at];
  tail->B = (const bf16_t*)pr[at].B + n0;
  tail->C = epi == EPI_STORE ? (void*)((bf16_t*)pr[at].C + n0) : (void*)((float*)pr[at].C + n0);
  tail->N = pr[at].N - n0;
  pr[at].N = n0;
  return true;
}

hipError_t launch_gemm_bf16_grouped(int layout, int epi, int n, const GemmProblem* problems, int K, hipStream_t s) {
  if (!gemm_bf16_grouped_applies(layout, n, problems, K)) return hipErrorInvalidValue;
  GemmProblem set[MAX_GROUP], tail;
  const GemmProblem* pr = problems;
  if (layout == GEMM_TN && (epi == EPI_ACCUM || epi == EPI_STORE || epi == EPI_STOREF)) {
    for (int i = 0; i < n; ++i) set[i] = problems[i];
    if (cut_tail(n, set, epi, K, &tail)) {
      pr = set;
      if (hipError_t e = launch_gemm_bf16_small(layout, epi, tail, K, s); e != hipSuccess) return e;
    }
  }
  if (layout == GEMM_TN && epi == EPI_ACCUM) return launch_direct_grouped<true, EPI_ACCUM>(n, pr, K, s);
  if (layout == GEMM_TN && epi == EPI_STORE) return launch_direct_grouped<true, EPI_STORE>(n, pr, K, s);
  if (layout == GEMM_TN && epi == EPI_STOREF) return launch_direct_grouped<true, EPI_STOREF>(n, pr, K, s);
  if (layout == GEMM_NT && epi == EPI_STORE) return launch_direct_grouped<false, EPI_STORE>(n, pr, K, s);
  if (layout == GEMM_NT && epi == EPI_ACCUM) return launch_direct_grouped<false, EPI_ACCUM>(n, pr, K, s);
  return hipErrorInvalidValue;
}
