// Fused causal attention, bf16 MFMA path for head_dim 128 and 64 (gfx950): forward (online softmax, writes
// lse) and backward (dQ kernel + dK/dV kernel, both recomputing the probabilities from lse; no atomics,
// so results are bitwise reproducible).  q-head a reads kv-head a * n_kv / n_q; dK, dV are summed over
// the q-heads of a group inside the dK/dV kernel.
//
// Register / LDS scheme.  Every product is issued on v_mfma_f32_32x32x16_bf16 in the orientation whose
// accumulator layout (one column per lane, 4-row groups along registers) already has the shape of the
// next product's 8-element operand, so probabilities never move between lanes:
//   forward / dQ:  S^T = K Q^T (lane = query, registers = keys)  ->  O^T += V^T P^T,  dQ^T += K^T dS^T
//   dK/dV:         S   = Q K^T (lane = key,   registers = queries) -> dV^T += dO^T P,  dK^T += Q^T dS
// Tiles go from global memory straight into LDS, row-major; operands that are contracted over their row
// index (V^T, K^T, dO^T, Q^T) come out of the same tile through transposing LDS reads.  All LDS tiles are
// XOR-swizzled so that both kinds of operand reads are bank-conflict free.
//
// Tiles are multiplied whole: what causality leaves out enters as zero times a row, which is NaN where that row is not finite, and an
// infinity that does belong to a row meets both parts of a split probability.  Heads of 64 keep such values to the rows that
// depend on them: a wave that finds a result that is not finite redoes its rows one by one (attention_rows.h).  Heads of 128 do
// not: there one such value makes NaN of up to 256 rows around it.
#include "attention_rows.h"

namespace {

constexpr float LOG2E = 1.4426950408889634f;

typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(3))) bf16x8_t lds_bf16x8_t;
typedef __attribute__((address_space(3))) f32x4_t lds_f32x4_t;

// What depends on the head size: rows of ROWB bytes = CH 16-byte chunks in the LDS tiles of 64 rows, NKS k-steps of an MFMA over
// a row, NDT 32-wide pieces of it, NLD loads of 1 KB (RPL rows) by which a wave fills its quarter of a tile.
// SPLIT: the probabilities and dS, fp32 numbers, enter the second product as the sum of two bf16 numbers (16 significant bits
// between them, a rounding of 2^-17 at most) and not as one.  The general kernels multiply them in fp32; the error against 64
// bits is no larger here (o 1.6e-3, dqkv 1.8e-3: the rounding of the results), where one bf16 number would raise it by a quarter.
// The exponentials themselves are v_exp_f32 (1 ulp) of x = c s - c m rounded once, |x| 2^-24: p is off by at most 2^-23 +
// 0.7 |x| 2^-24 of itself, as expf of a rounded difference is.
// Measured for heads of 64 at 4 x 1024 tokens, 16 heads, forward and backward: 4466 us on the general kernels (one wave per row,
// no matrix unit), 97 us here.
template <int D> struct Head {
  static constexpr int ROWB = 2 * D, TILE = 64 * ROWB, CH = D / 8, NKS = D / 16, NDT = D / 32, RPL = 64 / CH, NLD = 16 / RPL;
  static constexpr bool SPLIT = D == 64;
  // rows with a result that is not finite are redone one by one (needs all of a key's queries in one workgroup: split == 1);
  // ROW_LDS: bytes of LDS that they need behind the tiles, two rows of fp32 per wave
  static constexpr bool ROW_EXACT = D == 64;
  static constexpr int ROW_LDS = ROW_EXACT ? 4 * 2 * D * 4 : 0;
  // 16-byte chunk c of tile row r is stored at chunk c ^ swz(r).  Row reads: the 16 rows that a pass touches at one chunk fall on
  // all banks; transposing reads: the 4 rows of one differ in the 64-byte group (D = 64: so do rows two apart, which share
  // the half of the 256-byte bank window)
  __device__ __forceinline__ static constexpr int swz(int r) {
    return D == 128 ? ((r & 3) << 2) | ((r >> 2) & 3) : (((r >> 1) & 1) << 2) | (((r >> 2) & 1) << 1) | ((r >> 3) & 1);
  }
};

__device__ __forceinline__ bf16x8_t pack8(const f32x16_t& s, int u) {
  bf16x8_t r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = (bf16_t)s[8 * u + e];
  return r;
}
// what pack8 has rounded away, rounded
__device__ __forceinline__ bf16x8_t pack8_rest(const f32x16_t& s, const bf16x8_t& hi, int u) {
  bf16x8_t r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = (bf16_t)(s[8 * u + e] - (float)hi[e]);
  return r;
}

// NaN where any of the values is not finite, 0 otherwise
__device__ __forceinline__ float not_finite(const f32x16_t& s, float z = 0.f) {
#pragma unroll
  for (int v = 0; v < 16; ++v) z = fmaf(s[v], 0.f, z);
  return z;
}

// 4 columns of a gradient row from column `col` on and the 4 columns d / 2 away, scaled, turned back by the rotary angle of the row's
// position where there is one (fp32, ahead of the one rounding) and stored
template <int D> __device__ __forceinline__ void store_turned4(bf16_t* row, const float2* angle, int col, f32x4_t lo, f32x4_t hi, float scale) {
  f32x4_t t0 = {1.f, 0.f, 1.f, 0.f}, t1 = t0;
  if (angle) {
    t0 = *reinterpret_cast<const f32x4_t*>(angle + col);
    t1 = *reinterpret_cast<const f32x4_t*>(angle + col + 2);
  }
  bf16x4_t l, h;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float a = lo[i] * scale, b = hi[i] * scale;
    if (angle) rope_back(a, b, i < 2 ? t0[2 * (i & 1)] : t1[2 * (i & 1)], i < 2 ? t0[2 * (i & 1) + 1] : t1[2 * (i & 1) + 1]);
    l[i] = (bf16_t)a;
    h[i] = (bf16_t)b;
  }
  *reinterpret_cast<bf16x4_t*>(row + col) = l;
  *reinterpret_cast<bf16x4_t*>(row + col + D / 2) = h;
}
template <int D> __device__ __forceinline__ void store_turned(bf16_t* row, const float2* angle, int col, const f32x16_t& lo, const f32x16_t& hi,
                                                              int v, float scale) {
  store_turned4<D>(row, angle, col, f32x4_t{lo[v], lo[v + 1], lo[v + 2], lo[v + 3]}, f32x4_t{hi[v], hi[v + 1], hi[v + 2], hi[v + 3]}, scale);
}

// Two groups of waves hold partial sums of the same rows: the second group's waves leave theirs in LDS (16 bytes per lane and access), the
// first group's add them to their own
template <int TT, int NDT> __device__ __forceinline__ void meet_give(char* lds, int wave, int lane, const f32x16_t (&x)[TT][NDT]) {
  f32x4_t* p = reinterpret_cast<f32x4_t*>(lds) + wave * (TT * NDT * 4 * 64) + lane;
#pragma unroll
  for (int i = 0; i < TT * NDT * 4; ++i) {
    const f32x16_t& y = x[i / 4 / NDT][i / 4 % NDT];
    p[i * 64] = f32x4_t{y[4 * (i & 3)], y[4 * (i & 3) + 1], y[4 * (i & 3) + 2], y[4 * (i & 3) + 3]};
  }
}
template <int TT, int NDT> __device__ __forceinline__ void meet_take(const char* lds, int wave, int lane, f32x16_t (&x)[TT][NDT]) {
  const f32x4_t* p = reinterpret_cast<const f32x4_t*>(lds) + wave * (TT * NDT * 4 * 64) + lane;
#pragma unroll
  for (int i = 0; i < TT * NDT * 4; ++i) {
    const f32x4_t o = p[i * 64];
    f32x16_t& y = x[i / 4 / NDT][i / 4 % NDT];
#pragma unroll
    for (int e = 0; e < 4; ++e) y[4 * (i & 3) + e] += o[e];
  }
}

__device__ __forceinline__ void store4(bf16_t* p, const f32x16_t& x, int v, float scale) {
  bf16x4_t r;
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = (bf16_t)(x[v + i] * scale);
  *reinterpret_cast<bf16x4_t*>(p) = r;
}

// max over the two lanes 32 apart (the two halves of a score row), in both of them: v_permlane32_swap exchanges
// the upper half of its first operand with the lower half of its second, so swapping x with itself gives
// (x.low, x.low) and (x.high, x.high).  A vector instruction: no trip through the LDS crossbar.
__device__ __forceinline__ float pair_max32(float x) {
  const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

// ---- forward: grid (n_q, batch, ceil(seq / (32 NW))); NW NG waves, two per SIMD of a filled compute unit -------------------------------
// Same frame as the dQ kernel below: wave w owns the 32 queries from q0 + 32 w on, Q operand fragments and O^T ([d 128][32 queries]) in
// accumulator registers, key blocks of 64 (K and V rows) streaming through LDS straight from global memory: two stages of K (the
// scores of the next block's first tile are issued before the current block's last tile is finished) and two of V.  Per 32-key tile:
//   S^T = K Q^T (8 MFMAs), p = exp2(c s - c m_ref) with row sums, O^T += V^T P^T (8 MFMAs, V^T through
//   transposing LDS reads of the row-major V tile).
// An MFMA keeps the matrix unit for 32 cycles, in which a SIMD issues about eight vector instructions; a tile has four of those per MFMA
// (multiply-add, exponential at half rate, row sum, half a maximum and a conversion).  So the steps of consecutive tiles are interleaved by
// hand: the exponentials of tile i run between the score MFMAs of tile i + 1, the row maxima of tile i + 1 between the O^T MFMAs of
// tile i; the loop has no address arithmetic (stages are constants of the unrolled blocks: 15 of 107 vector instructions per step,
// and 2-5 % of the time, as sums); and a second wave on the SIMD takes the waits that are left.  On long sequences the board's power limit
// holds the clock at 1.7-1.9 GHz while the matrix unit is busy 54 % of the cycles, so fewer cycles save less than their share.
// The softmax reference m_ref is not the running maximum: it is raised (and O^T and the row sums rescaled)
// only when some row of the wave finds a score more than FWD_TAU / c above it, so p <= 2^FWD_TAU and the
// rescaling, which would sit between consecutive tiles' MFMAs on the same accumulators, is rare after the first
// tiles.  softmax does not depend on the reference: o = (sum p v) / (sum p), lse = m_ref scale + log(sum p).
// NG = 2: a second group of NW waves has the same queries; the groups share every block's keys, 32 each, and meet at the end.
constexpr float FWD_TAU = 8.f;

template <int D, int NW, int NG>
__global__ __launch_bounds__(64 * NW * NG) void attn_fwd_mfma(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ o,
                                                     float* __restrict__ lse, int seq, int n_q, int n_kv) {
  typedef Head<D> H;
  constexpr int ROWB = H::ROWB, TILE = H::TILE, NKS = H::NKS, NDT = H::NDT;
  constexpr int WROWS = 64 / (NW * NG), NLD = WROWS / H::RPL;        // rows of a tile that a wave loads, and its loads
  constexpr int V_RING = 2 * TILE;             // LDS: two K tiles of 64 keys, then two V tiles
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, c32 = lane & 31;
  const int id = __builtin_amdgcn_readfirstlane(tid >> 6), wave = id % NW, grp = id / NW;
  const int half = grp * 32;                   // NG = 2: a wave takes one half of every block's keys, which is in its addresses
  constexpr int GQ = 32 * NW;                  // queries of the workgroup
  const int nqb = (seq + GQ - 1) / GQ;
  const int q0 = (nqb - 1 - (int)blockIdx.z) * GQ;          // longest rows are dispatched first, for every head
  const int a = blockIdx.x, b = blockIdx.y, kvh = a * n_kv / n_q;
  const int ld = (n_q + 2 * n_kv) * D, ldo = n_q * D;
  const bf16_t* base = qkv + (size_t)b * seq * ld;
  const int wave_first_q = q0 + 32 * wave, qglob = wave_first_q + c32;
  const float scale = rsqrtf((float)D), c = scale * LOG2E, thr = FWD_TAU / c;

  bf16x8_t Qf[NKS];
  {
    const bf16_t* qp = base + (size_t)min(qglob, seq - 1) * ld + (size_t)a * D + 8 * g;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) Qf[ks] = *reinterpret_cast<const bf16x8_t*>(qp + 16 * ks);
  }
  f32x16_t acc[1][NDT];                         // [d tile]: lane = query, registers = d
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][dt][v] = 0.f;
  // the second group may meet rows that none of its first keys belong to: its reference starts at a finite value, which minus infinity
  // lies below (minus infinity from minus infinity is NaN)
  float mref = grp == 0 ? -INFINITY : -3.402823466e38f, lsum = 0.f;

  // LDS addressing as in the dQ kernel: 64 rows of ROWB bytes per tile, 16-byte chunk c of row r stored at chunk c ^ swz(r)
  int rm_addr[NKS];
  {
    const int f = H::swz(c32);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) rm_addr[ks] = half * ROWB + c32 * ROWB + (((2 * ks + g) ^ f) << 4);
  }
  int tr_addr[NDT][2];
  {
    const int cg = (lane >> 4) & 1, e = (lane >> 2) & 3, r = lane & 3;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int kq = 0; kq < 2; ++kq)
        tr_addr[dt][kq] = V_RING + half * ROWB + (4 * g + e) * ROWB + (((4 * dt + 2 * cg + (r >> 1)) ^ H::swz(8 * kq + 4 * g + e)) << 4) + (r & 1) * 8;
  }
  unsigned voff[NLD];
#pragma unroll
  for (int j = 0; j < NLD; ++j) {
    const int row = WROWS * id + H::RPL * j + lane / H::CH;
    const int chunk = (lane % H::CH) ^ H::swz(row);
    voff[j] = (unsigned)row * (unsigned)ld * 2u + (unsigned)chunk * 16u;
  }
  i32x4_t rs;
  {
    const unsigned long long ad = (unsigned long long)base;
    rs[0] = __builtin_amdgcn_readfirstlane((int)(unsigned)ad);
    rs[1] = __builtin_amdgcn_readfirstlane((int)(unsigned)(ad >> 32) & 0xffff);
    rs[2] = (int)((unsigned)seq * ld * 2u);                   // rows at or past seq read zero
    rs[3] = 0x00020000;
  }
  const unsigned lds0 = (unsigned)(size_t)(lds_void_t*)smem;
  const unsigned k_off = (unsigned)(n_q + kvh) * D * 2u, v_off = (unsigned)(n_q + n_kv + kvh) * D * 2u;
  auto issue_tile = [&](int kb, unsigned off, int lds) {
    const unsigned rowoff = (unsigned)(64 * kb) * (unsigned)ld * 2u + off;
    const unsigned dst = lds0 + lds + (WROWS * id) * ROWB;
#pragma unroll
    for (int j = 0; j < NLD; ++j)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                   :: "s"(dst + j * 1024), "v"(voff[j] + rowoff), "s"(rs) : "memory", "m0");
  };
  typedef short i16x4_t __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
  auto tr_frag = [&](const char* tile, int dt, int t, int u) {
    const i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t*)(tile + (32 * t + 16 * u) * ROWB + tr_addr[dt][0]));
    const i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t*)(tile + (32 * t + 16 * u + 8) * ROWB + tr_addr[dt][1]));
    return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto rm_frag = [&](const char* tile, int t, int ks) {
    return *reinterpret_cast<const bf16x8_t*>(tile + t * 32 * ROWB + rm_addr[ks]);
  };

  const int nkb = min((q0 + GQ - 1) / 64 + 1, (seq + 63) / 64);

#define OPTSTAGE_SB() __builtin_amdgcn_sched_barrier(0)
#define OPTSTAGE_MFMA_V(acc, a, b) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b))
  // O^T and the Q fragments stay in the accumulation half of the register file (an MFMA takes its A / B operands
  // from either half): the vector half holds two score tiles, the streaming operand fragments and addresses.  A
  // compiler-chosen form would shuttle O^T between the halves at every tile.
#define OPTSTAGE_MFMA_A(acc, a, b) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b))
  // Every wave runs every tile of the workgroup's 2 nkb, with no branch around a step: a tile above a wave's
  // diagonal is masked entirely (p = 0 adds nothing), and its SIMD would wait for the workgroup's last wave
  // anyway.  The scores issued in the very last step read a stage that holds no tile of this workgroup's; they
  // are never used.
  //
  // scores of the next tile into nxt (K half t of the tile in `stage_k`), between them the exponentials of the
  // current tile in cur
  // The first operand fragment of every step is read during the step before it (kf_first, trf_first), so that no
  // step starts with the matrix unit idle for an LDS round trip.
  constexpr int PF = 3, PT = 3;
  bf16x8_t kf[PF], trf[PT];
  auto step_scores = [&](bool with_exp, int stage_k, int t, f32x16_t& cur, f32x16_t& nxt, int stage_v, int tv) {
    const char* sK = smem + stage_k * TILE;
    const float mc = mref * c;
    float ls = 0.f;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      OPTSTAGE_SB();
      if (ks + PF - 1 < NKS) kf[(ks + PF - 1) % PF] = rm_frag(sK, t, ks + PF - 1);
      if (stage_v >= 0 && ks + PT - 1 >= NKS) trf[ks + PT - 1 - NKS] = tr_frag(smem + stage_v * TILE, (ks + PT - 1 - NKS) % NDT, tv, (ks + PT - 1 - NKS) / NDT);
      OPTSTAGE_SB();
      // The compiler does not see into the MFMA statements, so it keeps no distance between a vector instruction
      // that produces an operand (a copy, a read of an accumulation register that holds part of Q) and the MFMA
      // that consumes it: have the operands in place, then two idle cycles
      asm volatile("s_nop 1" :: "v"(kf[ks % PF]));
      // One MFMA, then vector work for about as long as it occupies the matrix unit, then the next: a wave that
      // reaches an MFMA while the unit is busy waits there and issues nothing else, so two MFMAs back to back
      // followed by all of the vector work run one after the other instead of side by side.
      if (ks == 0)                                               // the first k-step starts from C = 0
        asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(nxt) : "v"(kf[0]), "a"(Qf[0]));
      else
        asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(nxt) : "v"(kf[ks % PF]), "a"(Qf[ks]));
      OPTSTAGE_SB();
      if (with_exp) {                                            // compile-time after inlining
        constexpr int PV = 16 / NKS;                             // registers per MFMA
#pragma unroll
        for (int x = 0; x < PV; ++x) {
          const int v = ks * PV + x;
          cur[v] = __builtin_amdgcn_exp2f(fmaf(cur[v], c, -mc));
          ls += cur[v];
          // keeps these instructions here, between the MFMAs: without a use at this point the compiler sinks
          // them to where the probabilities are packed
          asm volatile("" : "+v"(cur[v]), "+v"(ls));
        }
      }
      OPTSTAGE_SB();
    }
    OPTSTAGE_SB();
    lsum += ls;
  };
  // scores above the diagonal (and keys past the sequence, which lie above every stored query) leave the softmax
  auto mask_tile = [&](int i, f32x16_t& sc) {
    const int key0 = 32 * i + half;
    if (key0 + 31 <= wave_first_q) return;                     // wave-uniform: the tile lies below the diagonal
    asm volatile("s_nop 7" ::: "memory");                        // the scores' last MFMA has written its results
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int key = key0 + 8 * (v >> 2) + 4 * g + (v & 3);
      if (key > qglob) sc[v] = -INFINITY;
    }
  };
  auto max_part = [&](int n, const f32x16_t& sc, float& mx) {    // n: one of the 2 NDT positions of a step
#pragma unroll
    for (int x = 0; x < 4 / NDT; ++x) {
      const int v = 2 * (n * (4 / NDT) + x);
      mx = fmaxf(mx, fmaxf(sc[v], sc[v + 1]));
    }
    asm volatile("" : "+v"(mx));                                // stays between the MFMAs it is written between
  };
  // the rare raise of m_ref, with O^T and the row sums rescaled
  auto raise_reference = [&](float mx) {
    mx = pair_max32(mx);                                        // the two lanes of a row hold 16 keys each
    if (__any(mx > mref + thr)) {
      asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");         // the last O^T MFMAs have left the matrix unit
      const float mn = fmaxf(mref, mx);
      const float alpha = mn == mref ? 1.f : __builtin_amdgcn_exp2f((mref - mn) * c);
      mref = mn;
      lsum *= alpha;
      // one accumulator tile at a time: they pass through vector registers for the multiplication
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
        OPTSTAGE_SB();
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[0][dt][v] *= alpha;
      }
      OPTSTAGE_SB();
    }
  };
  // O^T += V^T P^T of the current tile (probabilities in cur, V half t of the tile in `stage_v`), between the MFMAs
  // the row maxima of the next tile i1 (scores in nxt, already masked)
  auto step_output = [&](bool fill, int stage_v, int t, int i1, f32x16_t& cur, f32x16_t& nxt, int stage_k, int tk) {
    const char* sV = smem + stage_v * TILE;
    if (fill) {
#pragma unroll
      for (int i = 0; i < PT - 1; ++i) trf[i] = tr_frag(sV, i % NDT, t, i / NDT);
    }
    mask_tile(i1, nxt);
    float mx = -INFINITY;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const bf16x8_t p = pack8(cur, u);
      bf16x8_t rest;
      if constexpr (H::SPLIT) rest = pack8_rest(cur, p, u);
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
        const int n = u * NDT + dt, n2 = n + PT - 1, k2 = n + PF - 1 - 2 * NDT;
        OPTSTAGE_SB();
        if (n2 < 2 * NDT) trf[n2 % PT] = tr_frag(sV, n2 % NDT, t, n2 / NDT);
        if (stage_k >= 0 && k2 >= 0) kf[k2] = rm_frag(smem + stage_k * TILE, tk, k2);
        if (dt == 0) asm volatile("s_nop 1" :: "v"(p) : "memory");           // packed operands settled
        if constexpr (H::SPLIT) { if (dt == 0) asm volatile("s_nop 1" :: "v"(rest) : "memory"); }
        OPTSTAGE_SB();
        OPTSTAGE_MFMA_A(acc[0][dt], trf[n % PT], p);
        if constexpr (H::SPLIT) OPTSTAGE_MFMA_A(acc[0][dt], trf[n % PT], rest);
        OPTSTAGE_SB();
        max_part(n, nxt, mx);
      }
    }
    OPTSTAGE_SB();
    raise_reference(mx);
  };
#define OPTSTAGE_BLOCK_SYNC() asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory")

  auto fill_k = [&](int stage, int t) {
#pragma unroll
    for (int i = 0; i < PF - 1; ++i) kf[i] = rm_frag(smem + stage * TILE, t, i);
  };
  f32x16_t sA, sB;
  issue_tile(0, k_off, 0);
  OPTSTAGE_BLOCK_SYNC();
  if (nkb > 1) issue_tile(1, k_off, TILE);
  issue_tile(0, v_off, V_RING);
  fill_k(0, 0);
  step_scores(false, 0, 0, sB, sA, -1, 0);                      // scores of tile 0 into sA
  {
    // nothing to hide behind yet: results of the matrix unit may be read by the vector unit only some cycles
    // after the last pass
    asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
    mask_tile(0, sA);
    float mx = -INFINITY;
#pragma unroll
    for (int n = 0; n < 2 * NDT; ++n) max_part(n, sA, mx);
    raise_reference(mx);
    if (NG == 1) fill_k(0, 1);
  }
  if constexpr (NG == 1) {
    auto block = [&](int kb, int st) __attribute__((always_inline)) {   // st: the stage of block kb, a constant: LDS addresses need no arithmetic
      step_scores(true, st, 1, sA, sB, -1, 0);                   // exponentials of tile 2 kb, scores of tile 2 kb + 1
      // K of block kb + 1 and V of block kb have landed (this wave's part; the barrier covers the rest; they were requested a whole
      // block ago) and nobody still reads K of block kb or V of block kb - 1
      OPTSTAGE_BLOCK_SYNC();
      if (kb + 2 < nkb) issue_tile(kb + 2, k_off, st * TILE);
      if (kb + 1 < nkb) issue_tile(kb + 1, v_off, V_RING + (st ^ 1) * TILE);
      step_output(true, st, 0, 2 * kb + 1, sA, sB, st ^ 1, 0);
      step_scores(true, st ^ 1, 0, sB, sA, st, 1);               // exponentials of tile 2 kb + 1, scores of tile 2 kb + 2
      step_output(false, st, 1, 2 * kb + 2, sB, sA, st ^ 1, 1);
    };
    for (int kb = 0; kb < nkb; kb += 2) {
      block(kb, 0);
      if (kb + 1 < nkb) block(kb + 1, 1);
    }
  } else {
    // one tile of 32 keys per block: the exponentials of block kb's tile, the scores of the next one's, the output of block kb's
    auto block = [&](int kb, int st, f32x16_t& cur, f32x16_t& nxt) __attribute__((always_inline)) {
      OPTSTAGE_BLOCK_SYNC();                                   // K of block kb + 1 and V of block kb have landed
      if (kb + 2 < nkb) issue_tile(kb + 2, k_off, st * TILE);
      if (kb + 1 < nkb) issue_tile(kb + 1, v_off, V_RING + (st ^ 1) * TILE);
      fill_k(st ^ 1, 0);
      step_scores(true, st ^ 1, 0, cur, nxt, st, 0);
      step_output(false, st, 0, 2 * kb + 2, cur, nxt, -1, 0);
    };
    for (int kb = 0; kb < nkb; kb += 2) {
      block(kb, 0, sA, sB);
      if (kb + 1 < nkb) block(kb + 1, 1, sB, sA);
    }
  }
#undef OPTSTAGE_BLOCK_SYNC
#undef OPTSTAGE_MFMA_V
#undef OPTSTAGE_MFMA_A
  asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");

  if constexpr (NG == 2) {
    // the second group's sums, relative to its own reference, join the first group's: the larger reference of the two holds
    float* ref = reinterpret_cast<float*>(smem + NW * NDT * 4096) + wave * 128 + lane;
    __syncthreads();
    if (grp == 1) {
      meet_give<1, NDT>(smem, wave, lane, acc);
      ref[0] = mref;
      ref[64] = lsum;
    }
    __syncthreads();
    if (grp == 1) return;
    const float m1 = ref[0], M = fmaxf(mref, m1);
    const float f0 = __builtin_amdgcn_exp2f((mref - M) * c), f1 = __builtin_amdgcn_exp2f((m1 - M) * c);
    mref = M;
    lsum = lsum * f0 + ref[64] * f1;
    const f32x4_t* p = reinterpret_cast<const f32x4_t*>(smem) + wave * (NDT * 4 * 64) + lane;
#pragma unroll
    for (int i = 0; i < NDT * 4; ++i) {
      const f32x4_t o1 = p[i * 64];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[0][i / 4][4 * (i & 3) + e] = acc[0][i / 4][4 * (i & 3) + e] * f0 + o1[e] * f1;
    }
  }
  const float lt = lsum + __shfl_xor(lsum, 32, 64);
  const float inv = 1.f / lt;
  float row_lse = mref * scale + logf(lt);
  if constexpr (H::SPLIT) {
    // One fp32 rounding of lse and little more: the exponents were formed as c s - (c m_ref rounded), and what that rounding
    // left out scaled every p of the row alike (o does not see it); log(sum p) is larger than lse where m_ref is not the
    // maximum, so its integer part is added in fp64.  RMS-relative error at 1024 tokens 2.3e-8, 4.9e-8 as the plain sum
    // above, 4.3e-8 in the general kernels; 3.4e-8 is the most that rounding the exact value gives.
    const float mc = mref * c;
    int k;
    const float f = frexpf(lt, &k);
    row_lse = (float)((double)mref * scale + k * 0.6931471805599453 + (double)(logf(f) - fmaf(mref, c, -mc) * 0.6931471805599453f));
  }
  if constexpr (H::ROW_EXACT) {
    float z = fmaf(row_lse, 0.f, inv * 0.f);
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) z = not_finite(acc[0][dt], z);
    if (__any(qglob < seq && z != 0.f)) {
      for (int t = wave_first_q; t < min(wave_first_q + 32, seq); ++t)
        attn_fwd_row<bf16_t, D / 64>(qkv, o, lse, seq, n_q, n_kv, t, a, b, reinterpret_cast<float*>(smem + V_RING + 2 * TILE) + wave * D);
      return;
    }
  }
  if (qglob >= seq) return;
  bf16_t* orow = o + ((size_t)b * seq + qglob) * ldo + (size_t)a * D;
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt) {
    OPTSTAGE_SB();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      bf16x4_t r;
#pragma unroll
      for (int i = 0; i < 4; ++i) r[i] = (bf16_t)(acc[0][dt][4 * j + i] * inv);
      *reinterpret_cast<bf16x4_t*>(orow + 32 * dt + 8 * j + 4 * g) = r;
    }
  }
  if (g == 0) lse[((size_t)b * n_q + a) * seq + qglob] = row_lse;
#undef OPTSTAGE_SB
}


// ---- backward, dQ: grid (n_q, batch, ceil(seq / (32 NW))); NW NG waves --------------------------------------------------------------
// Mirror image of the dK/dV kernel below.  Wave w owns the 32 queries from q0 + 32 w on: their Q and dO operand fragments stay in registers
// (64) and dQ^T ([d 128][32 queries]) in accumulator registers.  Key blocks of 64 (K and V rows) stream through a
// two-stage LDS ring loaded straight from global memory; one copy of the K tile serves S^T = K Q^T (16-byte row
// reads) and dQ^T += K^T dS^T (transposing reads), through the same chunk swizzle as in the dK/dV kernel.
// Also produces D_t = <dO_t, O_t> per query row and head (from the dO fragments it holds anyway) and stores it
// for the dK/dV kernel, which runs after this one.  qcopy: see attn_bwd_inplace_applies.  NG as in the forward kernel.
template <int D, int NW, int NG>
__global__ __launch_bounds__(64 * NW * NG) void attn_bwd_dq_mfma(const bf16_t* qkv, const bf16_t* __restrict__ o,
                                                        const bf16_t* __restrict__ dout, const float* __restrict__ lse,
                                                        float* __restrict__ delta, bf16_t* dqkv, bf16_t* __restrict__ qcopy,
                                                        const float2* __restrict__ rope, int seq, int n_q, int n_kv) {
  typedef Head<D> H;
  constexpr int ROWB = H::ROWB, TILE = H::TILE, NKS = H::NKS, NDT = H::NDT;
  constexpr int WROWS = 64 / (NW * NG), NLD = WROWS / H::RPL;        // rows of a tile that a wave loads, and its loads
  constexpr int DQ_STAGE = 2 * TILE;           // K tile, V tile of 64 keys
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, c32 = lane & 31;
  const int id = __builtin_amdgcn_readfirstlane(tid >> 6), wave = id % NW, grp = id / NW;
  const int half = grp * 32;                   // NG = 2: a wave takes one half of every block's keys, which is in its addresses
  constexpr int GQ = 32 * NW;                  // queries of the workgroup
  const int nqb = (seq + GQ - 1) / GQ;
  const int q0 = (nqb - 1 - (int)blockIdx.z) * GQ;          // longest rows are dispatched first, for every head
  const int a = blockIdx.x, b = blockIdx.y, kvh = a * n_kv / n_q;
  const int ld = (n_q + 2 * n_kv) * D, ldo = n_q * D;
  const bf16_t* base = qkv + (size_t)b * seq * ld;
  const int wave_first_q = q0 + 32 * wave, wave_last_q = wave_first_q + 31, qglob = wave_first_q + c32;
  const float scale = rsqrtf((float)D), c = scale * LOG2E;

  // Q, dO operand fragments of this wave's queries (rows past the end are clamped: their results are not stored),
  // lse * log2(e) and D per query
  bf16x8_t Qf[NKS], dOf[NKS];
  float Lc, Dq;
  {
    const int qrow = min(qglob, seq - 1);
    const bf16_t* qp = base + (size_t)qrow * ld + (size_t)a * D + 8 * g;
    const bf16_t* dop = dout + ((size_t)b * seq + qrow) * ldo + (size_t)a * D + 8 * g;
    const bf16_t* op = o + ((size_t)b * seq + qrow) * ldo + (size_t)a * D + 8 * g;
    float dsum = 0.f;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      Qf[ks] = *reinterpret_cast<const bf16x8_t*>(qp + 16 * ks);
      dOf[ks] = *reinterpret_cast<const bf16x8_t*>(dop + 16 * ks);
      const bf16x8_t of = *reinterpret_cast<const bf16x8_t*>(op + 16 * ks);
#pragma unroll
      for (int e = 0; e < 8; ++e) dsum = fmaf((float)dOf[ks][e], (float)of[e], dsum);
    }
    if (qcopy && grp == 0 && qglob < seq) {
      bf16_t* cp = qcopy + ((size_t)b * seq + qrow) * ldo + (size_t)a * D + 8 * g;
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) *reinterpret_cast<bf16x8_t*>(cp + 16 * ks) = Qf[ks];
    }
    Lc = -lse[((size_t)b * n_q + a) * seq + qrow] * LOG2E;
    Dq = dsum + __shfl_xor(dsum, 32, 64);                  // the two lanes of a row hold 64 columns each
    // stored negated: both backward kernels use -D as the initial value of their dP accumulators
    if (grp == 0 && g == 0 && qglob < seq) delta[((size_t)b * n_q + a) * seq + qglob] = -Dq;
  }
  // -D of this lane's query in every register of an accumulator-shaped tuple: the initial value of the dP^T
  // MFMAs, which then deliver dP^T - D
  f32x16_t negD;
#pragma unroll
  for (int v = 0; v < 16; ++v) negD[v] = -Dq;
  // from here on the fragments are operands of MFMAs only: they move to the accumulation half of the register file
  // for good (the empty statements are where the move happens)
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) asm volatile("" : "+a"(Qf[ks]), "+a"(dOf[ks]));
  f32x16_t acc[1][NDT];                         // [d tile]: lane = query, registers = d
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][dt][v] = 0.f;

  const unsigned lds0 = (unsigned)(size_t)(lds_void_t*)smem;
  int rm_addr[NKS];                             // LDS addresses as numbers: the tile's place is a constant of each read
  {
    const int f = H::swz(c32);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      rm_addr[ks] = (int)lds0 + half * ROWB + c32 * ROWB + (((2 * ks + g) ^ f) << 4);
      asm volatile("" : "+v"(rm_addr[ks]));                    // one number per read, not the terms of a sum to be added at every read
    }
  }
  int tr_addr[NDT][2];
  {
    const int cg = (lane >> 4) & 1, e = (lane >> 2) & 3, r = lane & 3;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int kq = 0; kq < 2; ++kq) {
        tr_addr[dt][kq] = (int)lds0 + half * ROWB + (4 * g + e) * ROWB + (((4 * dt + 2 * cg + (r >> 1)) ^ H::swz(8 * kq + 4 * g + e)) << 4) + (r & 1) * 8;
        asm volatile("" : "+v"(tr_addr[dt][kq]));
      }
  }
  // tile loads: one instruction fills 4 rows (1 KB); wave w loads rows 16 w .. 16 w + 15 of the K and of the V tile
  unsigned voff[NLD];
#pragma unroll
  for (int j = 0; j < NLD; ++j) {
    const int row = WROWS * id + H::RPL * j + lane / H::CH;
    const int chunk = (lane % H::CH) ^ H::swz(row);
    voff[j] = (unsigned)row * (unsigned)ld * 2u + (unsigned)chunk * 16u;
  }
  auto make_desc = [](const void* p, unsigned bytes) {
    const unsigned long long ad = (unsigned long long)p;
    i32x4_t d;
    d[0] = __builtin_amdgcn_readfirstlane((int)(unsigned)ad);
    d[1] = __builtin_amdgcn_readfirstlane((int)(unsigned)(ad >> 32) & 0xffff);
    d[2] = (int)bytes;
    d[3] = 0x00020000;
    return d;
  };
  const i32x4_t rs = make_desc(base, (unsigned)seq * ld * 2u);
  const unsigned k_off = (unsigned)(n_q + kvh) * D * 2u, v_off = (unsigned)(n_q + n_kv + kvh) * D * 2u;
  // All offsets are the lane's (the range check would count a scalar one too): rows at or past seq read zero.
  auto issue_block = [&](int kb, int stage) {
    const unsigned rowoff = (unsigned)(64 * kb) * (unsigned)ld * 2u;
    const unsigned dst = lds0 + stage * DQ_STAGE + (WROWS * id) * ROWB;
#pragma unroll
    for (int j = 0; j < NLD; ++j) {
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                   :: "s"(dst + j * 1024), "v"(voff[j] + rowoff + k_off), "s"(rs) : "memory", "m0");
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                   :: "s"(dst + TILE + j * 1024), "v"(voff[j] + rowoff + v_off), "s"(rs) : "memory", "m0");
    }
  };
  typedef short i16x4_t __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
  auto tr_frag = [&](int tile, int dt, int t, int u) {
    const i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t*)(unsigned)(tr_addr[dt][0] + tile + (32 * t + 16 * u) * ROWB));
    const i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t*)(unsigned)(tr_addr[dt][1] + tile + (32 * t + 16 * u + 8) * ROWB));
    return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto rm_frag = [&](int tile, int t, int ks) { return *(const lds_bf16x8_t*)(unsigned)(rm_addr[ks] + tile + t * 32 * ROWB); };

#define OPTSTAGE_SB() __builtin_amdgcn_sched_barrier(0)
  // the register-resident operands (Q, dO) sit in the accumulation half of the register file, next to dQ^T: an
  // MFMA takes its A / B operands from either half, and the vector half is left to the score tiles, the streaming
  // fragments and the addresses
#define OPTSTAGE_MFMA_V(acc, a, b) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "a"(b))
#define OPTSTAGE_MFMA_0(acc, a, b) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "a"(b))
  auto block = [&](int kb, int stage) {
    if (64 * kb > wave_last_q) return;                           // block above this wave's diagonal
    const int sK = stage * DQ_STAGE, sV = sK + TILE;             // constants: they become the offsets of the LDS reads
#pragma unroll
    for (int t = 0; t < 2 / NG; ++t) {
      const int key0 = 64 * kb + half + 32 * t;
      if (key0 > wave_last_q) continue;                          // wave-uniform
      const bool edge = key0 + 31 > wave_first_q;                // touches the diagonal (keys past seq are masked by it)
      // lane = query, registers = keys key0 + 8 (v / 4) + 4 g + v % 4
      f32x16_t s, dp;
      bf16x8_t kf[2], vf[2];
      // ---- S^T = K Q^T (the first k-step starts from C = 0)
      kf[0] = rm_frag(sK, t, 0);
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        OPTSTAGE_SB();
        if (ks < NKS - 1) kf[(ks + 1) & 1] = rm_frag(sK, t, ks + 1);
        else vf[0] = rm_frag(sV, t, 0);
        OPTSTAGE_SB();
        if (ks == 0) OPTSTAGE_MFMA_0(s, kf[0], Qf[0]);
        else OPTSTAGE_MFMA_V(s, kf[ks & 1], Qf[ks]);
      }
      // ---- dP^T = V dO^T, with the exponentials of S^T under its MFMAs
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        OPTSTAGE_SB();
        if (ks < NKS - 1) vf[(ks + 1) & 1] = rm_frag(sV, t, ks + 1);
        OPTSTAGE_SB();
        if (ks == 0) {                                             // dP^T - D: the first k-step starts from C = -D
          asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(dp) : "v"(vf[0]), "a"(dOf[0]), "v"(negD));
          asm volatile("s_nop 7" ::: "memory");                    // the exponentials read S^T a few cycles after the matrix unit has written it
        } else {
          OPTSTAGE_MFMA_V(dp, vf[ks & 1], dOf[ks]);
        }
        OPTSTAGE_SB();
#pragma unroll
        for (int e = 0; e < 16 / NKS; ++e) {
          const int v = (16 / NKS) * ks + e;
          s[v] = __builtin_amdgcn_exp2f(fmaf(s[v], c, Lc));
        }
      }
      OPTSTAGE_SB();
      if (edge) {
        asm volatile("" ::: "memory");                             // a real branch: only diagonal tiles pay for the mask
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = key0 + 8 * (v >> 2) + 4 * g + (v & 3);
          if (key > qglob) s[v] = 0.f;
        }
      }
      // results of the matrix unit may be read by the vector unit only some cycles after the last pass
      asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
      OPTSTAGE_SB();
      // ---- dQ^T += K^T dS^T; dS^T = P^T (dP^T - D) of the second half runs under the MFMAs of the first (D is
      // already subtracted: it was the accumulator's initial value)
      bf16x8_t trf[2];
      trf[0] = tr_frag(sK, 0, t, 0);
#pragma unroll
      for (int v = 0; v < 8; ++v) dp[v] = s[v] * dp[v];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const bf16x8_t d = pack8(dp, u);
        bf16x8_t rest;
        if constexpr (H::SPLIT) rest = pack8_rest(dp, d, u);
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
          const int n = u * NDT + dt;
          OPTSTAGE_SB();
          if (n < 2 * NDT - 1) trf[(n + 1) & 1] = tr_frag(sK, (dt + 1) % NDT, t, dt == NDT - 1 ? 1 : u);
          OPTSTAGE_SB();
          acc[0][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(trf[n & 1], d, acc[0][dt], 0, 0, 0);
          if constexpr (H::SPLIT) acc[0][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(trf[n & 1], rest, acc[0][dt], 0, 0, 0);
          OPTSTAGE_SB();
          if (u == 0) {
#pragma unroll
            for (int e = 0; e < 8 / NDT; ++e) {
              const int v = 8 + (8 / NDT) * dt + e;
              dp[v] = s[v] * dp[v];
            }
          }
        }
      }
      OPTSTAGE_SB();
    }
  };
#undef OPTSTAGE_MFMA_V
#undef OPTSTAGE_MFMA_0
#undef OPTSTAGE_SB

  const int nkb = min((q0 + GQ - 1) / 64 + 1, (seq + 63) / 64);
  issue_block(0, 0);
  for (int kb = 0; kb < nkb; kb += 2) {
    // block kb has landed (this wave's part; the barrier covers the rest) and nobody still reads stage 1
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    if (kb + 1 < nkb) issue_block(kb + 1, 1);
    block(kb, 0);
    if (kb + 1 < nkb) {
      asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
      if (kb + 2 < nkb) issue_block(kb + 2, 0);
      block(kb + 1, 1);
    }
  }

  if constexpr (NG == 2) {
    __syncthreads();
    if (grp == 1) meet_give<1, NDT>(smem, wave, lane, acc);
    __syncthreads();
    if (grp == 1) return;
    meet_take<1, NDT>(smem, wave, lane, acc);
  }
  if constexpr (H::ROW_EXACT) {
    float z = 0.f;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) z = not_finite(acc[0][dt], z);
    if (__any(qglob < seq && z != 0.f)) {
      float* own = reinterpret_cast<float*>(smem + 2 * DQ_STAGE) + wave * 2 * D;
      for (int t = wave_first_q; t < min(wave_first_q + 32, seq); ++t)
        attn_bwd_dq_row<bf16_t, D / 64>(qkv, o, dout, lse, dqkv, nullptr, seq, n_q, n_kv, t, a, b, own, own + D, rope);
      return;
    }
  }
  if (qglob >= seq) return;
  bf16_t* dq = dqkv + ((size_t)b * seq + qglob) * ld + (size_t)a * D;
  if (rope) {
    const float2* angle = rope + (size_t)qglob * (D / 2);
#pragma unroll
    for (int dt = 0; dt < NDT / 2; ++dt)
#pragma unroll
      for (int j = 0; j < 4; ++j) store_turned<D>(dq, angle, 32 * dt + 8 * j + 4 * g, acc[0][dt], acc[0][dt + NDT / 2], 4 * j, scale);
    return;
  }
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      __builtin_amdgcn_sched_barrier(0);                     // one piece after the other: no more registers than the loop
      store4(dq + 32 * dt + 8 * j + 4 * g, acc[0][dt], 4 * j, scale);
    }
}

// ---- backward, dK / dV: grid (n_kv, batch, ceil(seq / (128 KT))); 4 NG waves; text for KT = 2, NG = 1 (one wave per SIMD) ----------------
// Wave w owns keys k0 + 64 w .. + 63 as two 32-key tiles: their K operand fragments stay in registers for the
// whole kernel (the V rows of the workgroup's 256 keys stay in LDS: both operand sets do not fit beside the
// accumulators) and dK^T, dV^T ([d 128][64 keys] each) in the 256 accumulator registers, so every Q / dO
// fragment read from LDS feeds two MFMAs.  Query blocks of 64 (Q and dO rows plus their lse and D)
// stream through a two-stage LDS ring, loaded straight from global memory (`buffer_load ... lds`); one copy
// of a tile serves both contractions: over head_dim with 16-byte row reads (S = Q K^T, dP = dO V^T) and over
// the queries with transposing reads (dV^T += dO^T P, dK^T += Q^T dS).  16-byte chunk c of tile row r is
// stored at chunk c ^ f(r), f(r) = ((r & 3) << 2) | ((r >> 2) & 3): 16 consecutive rows get 16 different
// values (row reads of one chunk hit every bank once) and 4 consecutive rows differ in the 64-byte group
// (the 4 rows of a transposing read do too).

// With grouped-query attention a kv head's gradient sums over n_q / n_kv query heads and the grid has only
// n_kv * batch * ceil(seq / 256) workgroups; `split` > 1 deals the query heads of a group to that many
// workgroups, each writing an fp32 partial ([part][batch][seq][kv head][K|V][128]) that attn_bwd_dkv_reduce sums
// in a fixed order.
// KT = 1, NG = 2: one key tile per wave, and a second group of four waves for the other 32 queries of every block, whose sums the first group
// adds at the end: two waves per SIMD in 246 registers each, half the chain of queries.  4096 tokens, 8 heads: this kernel 130 -> 107 us.
template <int D, int KT, int NG>
__global__ __launch_bounds__(256 * NG) void attn_bwd_dkv_mfma(const bf16_t* qkv, const bf16_t* qsrc, int ldq, const bf16_t* __restrict__ dout,
                                                         const float* __restrict__ lse, const float* __restrict__ delta,
                                                         bf16_t* dqkv, float* __restrict__ partial, const float2* __restrict__ rope,
                                                         int split, int seq, int n_q, int n_kv) {
  typedef Head<D> H;
  constexpr int ROWB = H::ROWB, TILE = H::TILE, NKS = H::NKS, NDT = H::NDT;
  constexpr int WROWS = 16 / NG, NLD = WROWS / H::RPL;        // rows of a tile that a wave loads, and its loads
  constexpr int DKV_STAGE = 2 * TILE + 512;    // Q tile, dO tile, 64 lse, 64 D; behind two of them V rows of 256 keys
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, c32 = lane & 31;
  const int id = __builtin_amdgcn_readfirstlane(tid >> 6), wave = id & 3, grp = NG == 1 ? 0 : id >> 2;
  constexpr int WK = 32 * KT, GK = 4 * WK;       // keys of a wave, of the workgroup
  const int k0 = blockIdx.z * GK;               // first key blocks (most queries) are dispatched first, for every head
  const int kvh = blockIdx.x / split, part = blockIdx.x % split, b = blockIdx.y;
  const int ld = (n_q + 2 * n_kv) * D, ldo = n_q * D;
  const bf16_t* base = qkv + (size_t)b * seq * ld;
  const int wave_first_k = k0 + WK * wave;
  const float scale = rsqrtf((float)D), c = scale * LOG2E;

  // K, V operand fragments of this wave's keys (rows past the end are clamped: their results are not stored)
  bf16x8_t Kf[KT][NKS];
#pragma unroll
  for (int kk = 0; kk < KT; ++kk) {
    const int krow = min(wave_first_k + 32 * kk + c32, seq - 1);
    const bf16_t* kp = base + (size_t)krow * ld + (size_t)(n_q + kvh) * D + 8 * g;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) Kf[kk][ks] = *reinterpret_cast<const bf16x8_t*>(kp + 16 * ks);
  }
  f32x16_t accK[KT][NDT], accV[KT][NDT];          // [key tile][d tile]: lane = key, registers = d
#pragma unroll
  for (int kk = 0; kk < KT; ++kk)
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int v = 0; v < 16; ++v) { accK[kk][dt][v] = 0.f; accV[kk][dt][v] = 0.f; }

  // per-lane LDS addresses within a tile.  Row read of k-step ks: row c32 (+ 32 t), chunk 2 ks + g.
  const unsigned lds0 = (unsigned)(size_t)(lds_void_t*)smem;
  // NG = 2: a wave takes one half of every block's queries, which is in its addresses
  const int half = grp * 32, row4 = (int)lds0 + 16 * g + half * 4;
  int rm_addr[NKS];
  {
    const int f = H::swz(c32);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      rm_addr[ks] = (int)lds0 + half * ROWB + c32 * ROWB + (((2 * ks + g) ^ f) << 4);
      asm volatile("" : "+v"(rm_addr[ks]));                    // one number per read, not the terms of a sum to be added at every read
    }
  }
  // Transposing read (dt, kq): in each 16-lane group lane 4 e + r reads 8 bytes of row 4 g + e (+ 32 t + 16 u
  // + 8 kq), columns 32 dt + 16 cg + 4 r ..; f(row) = (e << 2) | (2 kq + g)
  int tr_addr[NDT][2];
  {
    const int cg = (lane >> 4) & 1, e = (lane >> 2) & 3, r = lane & 3;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int kq = 0; kq < 2; ++kq) {
        tr_addr[dt][kq] = (int)lds0 + half * ROWB + (4 * g + e) * ROWB + (((4 * dt + 2 * cg + (r >> 1)) ^ H::swz(8 * kq + 4 * g + e)) << 4) + (r & 1) * 8;
        asm volatile("" : "+v"(tr_addr[dt][kq]));
      }
  }
  // tile loads: one instruction fills 4 rows (1 KB); wave w loads rows 16 w .. 16 w + 15 of Q and of dO.
  // Lane i: row 4 b + i / 16, stored chunk i % 16 = logical chunk ^ f(row), f = ((i / 16) << 2) | (b & 3).
  unsigned voff_q[NLD], voff_do[NLD];
#pragma unroll
  for (int j = 0; j < NLD; ++j) {
    const int row = WROWS * id + H::RPL * j + lane / H::CH;
    const int chunk = (lane % H::CH) ^ H::swz(row);
    voff_q[j] = (unsigned)row * (unsigned)ldq * 2u + (unsigned)chunk * 16u;
    voff_do[j] = (unsigned)row * (unsigned)ldo * 2u + (unsigned)chunk * 16u;
  }
  auto make_desc = [](const void* p, unsigned bytes) {
    const unsigned long long a = (unsigned long long)p;
    i32x4_t d;
    d[0] = __builtin_amdgcn_readfirstlane((int)(unsigned)a);
    d[1] = __builtin_amdgcn_readfirstlane((int)(unsigned)(a >> 32) & 0xffff);
    d[2] = (int)bytes;
    d[3] = 0x00020000;
    return d;
  };
  const i32x4_t rs_q = make_desc(qsrc + (size_t)b * seq * ldq, (unsigned)seq * ldq * 2u);
  const i32x4_t rs_do = make_desc(dout + (size_t)b * seq * ldo, (unsigned)seq * ldo * 2u);
  const i32x4_t rs_l = make_desc(lse + (size_t)b * n_q * seq, (unsigned)n_q * seq * 4u);
  const i32x4_t rs_d = make_desc(delta + (size_t)b * n_q * seq, (unsigned)n_q * seq * 4u);

  // V rows of this wave's 64 keys -> LDS (16 loads of 4 rows), same layout as the streamed tiles
  const i32x4_t rs_v = make_desc(base, (unsigned)seq * ld * 2u);
  const int sV = 2 * DKV_STAGE + wave * WK * ROWB - half * ROWB;
#pragma unroll
  for (int j0 = 0; j0 < 2 * KT * NLD; ++j0) {                   // both groups of waves read them: each loads its share
    const int j = j0 + grp * 2 * KT * NLD, row = H::RPL * j + lane / H::CH;
    const int chunk = (lane % H::CH) ^ H::swz(row);
    const unsigned vo = ((unsigned)(wave_first_k + row) * (unsigned)ld + (unsigned)(n_q + n_kv + kvh) * D) * 2u + (unsigned)chunk * 16u;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(lds0 + 2 * DKV_STAGE + wave * WK * ROWB + j * 1024), "v"(vo), "s"(rs_v) : "memory", "m0");
  }
  const int rep = n_q / n_kv / split;                          // query heads of the group handled here
  const int qb0 = k0 / 64, nqb = (seq + 63) / 64 - qb0;       // query blocks at or after the first key
  const int iters = rep * nqb;
  // All offsets are the lane's (the range check would count a scalar one too): rows at or past seq read zero.
  auto issue_block = [&](int it, int stage) {
    const int a = (kvh * split + part) * rep + it / nqb;
    const int r0 = 64 * (qb0 + it % nqb);
    const unsigned oq = ((unsigned)r0 * (unsigned)ldq + (unsigned)a * D) * 2u;
    const unsigned od = ((unsigned)r0 * (unsigned)ldo + (unsigned)a * D) * 2u;
    const unsigned dst = lds0 + stage * DKV_STAGE + (WROWS * id) * ROWB;
#pragma unroll
    for (int j = 0; j < NLD; ++j) {
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                   :: "s"(dst + j * 1024), "v"(voff_q[j] + oq), "s"(rs_q) : "memory", "m0");
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                   :: "s"(dst + TILE + j * 1024), "v"(voff_do[j] + od), "s"(rs_do) : "memory", "m0");
    }
    if (id < 2) {                              // wave 0: lse of the 64 queries, wave 1: D
      const unsigned vo = ((unsigned)a * (unsigned)seq + (unsigned)min(r0 + lane, seq - 1)) * 4u;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                   :: "s"(lds0 + stage * DKV_STAGE + 2 * TILE + id * 256), "v"(vo), "s"(id == 0 ? rs_l : rs_d) : "memory", "m0");
    }
  };
  typedef short i16x4_t __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
  auto tr_frag = [&](int tile, int dt, int t, int u) {
    const i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t*)(unsigned)(tr_addr[dt][0] + tile + (32 * t + 16 * u) * ROWB));
    const i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t*)(unsigned)(tr_addr[dt][1] + tile + (32 * t + 16 * u + 8) * ROWB));
    return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto rm_frag = [&](int tile, int t, int ks) { return *(const lds_bf16x8_t*)(unsigned)(rm_addr[ks] + tile + t * 32 * ROWB); };

#define OPTSTAGE_SB() __builtin_amdgcn_sched_barrier(0)
  // VGPR-result MFMA in assembly: the compiler would place the score tiles in accumulator registers, all 256
  // of which hold dK, dV.  Readers of the result keep >= 2 MFMAs (or an s_nop) behind the last write.
#define OPTSTAGE_MFMA_V(acc, a, b) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b))
#define OPTSTAGE_MFMA_0(acc, a, b) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "v"(b))
  auto block = [&](int it, int stage) {
    const int r0 = 64 * (qb0 + it % nqb);
    if (r0 + 63 < wave_first_k) return;                          // all queries precede this wave's keys
    const int sQ = stage * DKV_STAGE, sDO = sQ + TILE;           // constants: they become the offsets of the LDS reads
    const int sL = sQ + 2 * TILE, sD = sL + 256;
#pragma unroll
    for (int t = 0; t < 2 / NG; ++t) {
      const int q0 = r0 + half + 32 * t;
      if (q0 + 31 < wave_first_k) continue;                      // wave-uniform
      const bool edge = q0 < wave_first_k + WK - 1 || q0 + 32 > seq;   // touches the diagonal or the ragged tail
      // lane = key, registers = queries q0 + 8 (v / 4) + 4 g + v % 4
      f32x16_t s[KT], dp[KT];
      f32x4_t nL[4];                                               // -lse * log2(e) of this lane's queries
      f32x16_t negD;                                               // -D of this lane's queries, in accumulator order
      bf16x8_t qf[2], df[2], vf[2][KT];
      // ---- S = Q K^T: fragment of k-step ks + 1 requested before the MFMAs of k-step ks
      qf[0] = rm_frag(sQ, t, 0);
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        OPTSTAGE_SB();
        if (ks < NKS - 1) {
          qf[(ks + 1) & 1] = rm_frag(sQ, t, ks + 1);
        } else {
          df[0] = rm_frag(sDO, t, 0);
#pragma unroll
          for (int kk = 0; kk < KT; ++kk) vf[0][kk] = rm_frag(sV, kk, 0);
        }
        if (KT == 2 ? ks < 4 : ks == NKS - 1) nL[KT == 2 ? ks : 0] = *(const lds_f32x4_t*)(unsigned)(row4 + sL + (32 * t + 8 * (KT == 2 ? ks : 0)) * 4);
        if (ks >= NKS - 4) {
          const f32x4_t d4 = *(const lds_f32x4_t*)(unsigned)(row4 + sD + (32 * t + 8 * (ks - (NKS - 4))) * 4);
#pragma unroll
          for (int i = 0; i < 4; ++i) (KT == 2 ? negD : dp[0])[4 * (ks - (NKS - 4)) + i] = d4[i];
        }
        OPTSTAGE_SB();
        if (ks == 0) {                                             // the first k-step starts from C = 0
#pragma unroll
          for (int kk = 0; kk < KT; ++kk) OPTSTAGE_MFMA_0(s[kk], qf[0], Kf[kk][0]);
        } else {
#pragma unroll
          for (int kk = 0; kk < KT; ++kk) OPTSTAGE_MFMA_V(s[kk], qf[ks & 1], Kf[kk][ks]);
        }
        OPTSTAGE_SB();
        if (KT == 2 && ks >= NKS - 4) {
#pragma unroll
          for (int i = 0; i < 4; ++i) nL[ks - (NKS - 4)][i] *= -LOG2E;
        }
      }
      // ---- dP = dO V^T, with the exponentials of S (2 registers x 2 key tiles per k-step) under its MFMAs
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        OPTSTAGE_SB();
        if (ks < NKS - 1) {
          df[(ks + 1) & 1] = rm_frag(sDO, t, ks + 1);
#pragma unroll
          for (int kk = 0; kk < KT; ++kk) vf[(ks + 1) & 1][kk] = rm_frag(sV, kk, ks + 1);
        }
        // one key tile: lse of the next four queries one k-step ahead of its exponentials (16 registers fewer, two waves per SIMD)
        constexpr int KL = NKS / 4;                                // k-steps per four queries
        if (KT == 1 && ks % KL == KL - 1 && ks / KL < 3)
          nL[ks / KL + 1] = *(const lds_f32x4_t*)(unsigned)(row4 + sL + (32 * t + 8 * (ks / KL + 1)) * 4);
        OPTSTAGE_SB();
        if (ks == 0) {                                             // dP - D: the first k-step starts from C = -D
#pragma unroll
          for (int kk = 0; kk < KT; ++kk) {
            if constexpr (KT == 2) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(dp[kk]) : "v"(df[0]), "v"(vf[0][kk]), "v"(negD));
            else OPTSTAGE_MFMA_V(dp[kk], df[0], vf[0][kk]);
          }
          // the exponentials read S a few cycles after the matrix unit has written it: a second key tile's MFMA is that long
          if (KT == 1) asm volatile("s_nop 7" ::: "memory");
        } else {
#pragma unroll
          for (int kk = 0; kk < KT; ++kk) OPTSTAGE_MFMA_V(dp[kk], df[ks & 1], vf[ks & 1][kk]);
        }
        OPTSTAGE_SB();
#pragma unroll
        for (int e = 0; e < 16 / NKS; ++e) {
          const int v = (16 / NKS) * ks + e;
#pragma unroll
          for (int kk = 0; kk < KT; ++kk) s[kk][v] = __builtin_amdgcn_exp2f(fmaf(s[kk][v], c, KT == 2 ? nL[v >> 2][v & 3] : nL[v >> 2][v & 3] * -LOG2E));
        }
      }
      OPTSTAGE_SB();
      if (edge) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int qg = q0 + 8 * (v >> 2) + 4 * g + (v & 3);
#pragma unroll
          for (int kk = 0; kk < KT; ++kk)
            if (qg < wave_first_k + 32 * kk + c32 || qg >= seq) s[kk][v] = 0.f;
        }
      }
      OPTSTAGE_SB();
      // ---- dV^T += dO^T P, with dS = P (dP - D) under its MFMAs (the first two MFMAs cover the dP latency)
      bf16x8_t trf[2];
      trf[0] = tr_frag(sDO, 0, t, 0);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        bf16x8_t p[KT], rest[KT];
#pragma unroll
        for (int kk = 0; kk < KT; ++kk) p[kk] = pack8(s[kk], u);
        if constexpr (H::SPLIT) {
#pragma unroll
          for (int kk = 0; kk < KT; ++kk) rest[kk] = pack8_rest(s[kk], p[kk], u);
        }
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
          const int n = u * NDT + dt;
          OPTSTAGE_SB();
          if (n < 2 * NDT - 1) trf[(n + 1) & 1] = tr_frag(sDO, (dt + 1) % NDT, t, dt == NDT - 1 ? 1 : u);
          else trf[0] = tr_frag(sQ, 0, t, 0);
          OPTSTAGE_SB();
#pragma unroll
          for (int kk = 0; kk < KT; ++kk) accV[kk][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(trf[n & 1], p[kk], accV[kk][dt], 0, 0, 0);
          if constexpr (H::SPLIT) {
#pragma unroll
            for (int kk = 0; kk < KT; ++kk) accV[kk][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(trf[n & 1], rest[kk], accV[kk][dt], 0, 0, 0);
          }
          OPTSTAGE_SB();
          if (KT == 1 && n == 0) asm volatile("s_nop 7" ::: "memory");   // dP has left the matrix unit
#pragma unroll
          for (int e = 0; e < 8 / NDT; ++e) {
            const int v = (8 / NDT) * n + e;
#pragma unroll
            for (int kk = 0; kk < KT; ++kk) dp[kk][v] = s[kk][v] * dp[kk][v];
          }
        }
      }
      // ---- dK^T += Q^T dS
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        bf16x8_t d[KT], rest[KT];
#pragma unroll
        for (int kk = 0; kk < KT; ++kk) d[kk] = pack8(dp[kk], u);
        if constexpr (H::SPLIT) {
#pragma unroll
          for (int kk = 0; kk < KT; ++kk) rest[kk] = pack8_rest(dp[kk], d[kk], u);
        }
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
          const int n = u * NDT + dt;
          OPTSTAGE_SB();
          if (n < 2 * NDT - 1) trf[(n + 1) & 1] = tr_frag(sQ, (dt + 1) % NDT, t, dt == NDT - 1 ? 1 : u);
          OPTSTAGE_SB();
#pragma unroll
          for (int kk = 0; kk < KT; ++kk) accK[kk][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(trf[n & 1], d[kk], accK[kk][dt], 0, 0, 0);
          if constexpr (H::SPLIT) {
#pragma unroll
            for (int kk = 0; kk < KT; ++kk) accK[kk][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(trf[n & 1], rest[kk], accK[kk][dt], 0, 0, 0);
          }
        }
      }
      OPTSTAGE_SB();
    }
  };
#undef OPTSTAGE_MFMA_V
#undef OPTSTAGE_MFMA_0
#undef OPTSTAGE_SB

  if (iters > 0) issue_block(0, 0);
  for (int it = 0; it < iters; it += 2) {
    // block `it` has landed (this wave's part; the barrier covers the rest) and nobody still reads stage 1
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    if (it + 1 < iters) issue_block(it + 1, 1);
    block(it, 0);
    if (it + 1 < iters) {
      asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
      if (it + 2 < iters) issue_block(it + 2, 0);
      block(it + 1, 1);
    }
  }

  if constexpr (NG == 2) {
    __syncthreads();
    if (grp == 1) meet_give<KT, NDT>(smem, wave, lane, accV);
    __syncthreads();
    if (grp == 0) meet_take<KT, NDT>(smem, wave, lane, accV);
    __syncthreads();
    if (grp == 1) meet_give<KT, NDT>(smem, wave, lane, accK);
    __syncthreads();
    if (grp == 1) return;
    meet_take<KT, NDT>(smem, wave, lane, accK);
  }

#pragma unroll
  for (int kk = 0; kk < KT; ++kk) {
    const int kglob = wave_first_k + 32 * kk + c32;
    if constexpr (H::ROW_EXACT) {
      float z = 0.f;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) z = not_finite(accV[kk][dt], not_finite(accK[kk][dt], z));
      if (__any(kglob < seq && z != 0.f)) {
        float* own = reinterpret_cast<float*>(smem + 2 * DKV_STAGE + 4 * WK * ROWB) + wave * 2 * D;
        for (int t = wave_first_k + 32 * kk; t < min(wave_first_k + 32 * kk + 32, seq); ++t)
          attn_bwd_dkv_row<bf16_t, D / 64, true>(qkv, qsrc, ldq, dout, lse, delta, dqkv, seq, n_q, n_kv, t, kvh, b, own, own + D, rope);
        continue;
      }
    }
    if (kglob >= seq) continue;
    if (split > 1) {
      float* prow = partial + ((((size_t)part * gridDim.y + b) * seq + kglob) * n_kv + kvh) * 2 * D;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          f32x4_t rk, rv;
#pragma unroll
          for (int i = 0; i < 4; ++i) { rk[i] = accK[kk][dt][4 * j + i]; rv[i] = accV[kk][dt][4 * j + i]; }
          *reinterpret_cast<f32x4_t*>(prow + 32 * dt + 8 * j + 4 * g) = rk;
          *reinterpret_cast<f32x4_t*>(prow + D + 32 * dt + 8 * j + 4 * g) = rv;
        }
      continue;
    }
    bf16_t* krow = dqkv + ((size_t)b * seq + kglob) * ld + (size_t)(n_q + kvh) * D;
    bf16_t* vrow = dqkv + ((size_t)b * seq + kglob) * ld + (size_t)(n_q + n_kv + kvh) * D;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (!rope) store4(krow + 32 * dt + 8 * j + 4 * g, accK[kk][dt], 4 * j, scale);
        store4(vrow + 32 * dt + 8 * j + 4 * g, accV[kk][dt], 4 * j, 1.f);
      }
    if (rope) {
      const float2* angle = rope + (size_t)kglob * (D / 2);
#pragma unroll
      for (int dt = 0; dt < NDT / 2; ++dt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          __builtin_amdgcn_sched_barrier(0);                   // no registers to spare for several table reads in flight
          store_turned<D>(krow, angle, 32 * dt + 8 * j + 4 * g, accK[kk][dt], accK[kk][dt + NDT / 2], 4 * j, scale);
        }
    }
  }
}

// sums the `split` partials of dK, dV (fixed order), scales dK by 1 / sqrt(d), turns it back by the rotary angle where a table is given,
// and stores bf16 into the packed gradient rows: one thread per 4 columns of one (token, kv head, K|V) and the 4 columns d / 2 away
__global__ void attn_bwd_dkv_reduce(const float* __restrict__ partial, bf16_t* __restrict__ dqkv, const float2* __restrict__ rope,
                                    int split, int rows, int seq, int n_q, int n_kv) {
  constexpr int D = 128, Q = D / 8;                           // threads per (token, kv head, K|V)
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t per_part = (size_t)rows * n_kv * 2 * D;
  if (idx * 8 >= per_part) return;
  const int col = (int)(idx % Q) * 4, kv = (int)((idx / Q) % 2);
  const int h = (int)((idx / (2 * Q)) % n_kv);
  const size_t row = idx / ((size_t)2 * Q * n_kv);
  const float* p = partial + idx / Q * D + col;
  f32x4_t lo = *reinterpret_cast<const f32x4_t*>(p), hi = *reinterpret_cast<const f32x4_t*>(p + D / 2);
  for (int i = 1; i < split; ++i) {
    const f32x4_t v = *reinterpret_cast<const f32x4_t*>(p + i * per_part), w = *reinterpret_cast<const f32x4_t*>(p + i * per_part + D / 2);
#pragma unroll
    for (int e = 0; e < 4; ++e) { lo[e] += v[e]; hi[e] += w[e]; }
  }
  const int ld = (n_q + 2 * n_kv) * D;
  store_turned4<D>(dqkv + row * ld + (size_t)(n_q + kv * n_kv + h) * D, kv == 0 && rope ? rope + row % seq * (D / 2) : nullptr, col, lo, hi,
                   kv == 0 ? rsqrtf((float)D) : 1.f);
}

}  // namespace

// how many workgroups share the query heads of one kv head in the dK/dV kernel, a divisor of n_q / n_kv: enough to give every compute
// unit about two workgroups of 256 keys.  Callers size their scratch by it, so it does not look at the tile count that the launch picks:
// with one tile per wave the same split makes twice as many workgroups of half the size (8192 tokens, 8 / 1 heads: 512 of 128
// keys; dK / dV 382 -> 278 us).
int attn_dkv_split(int seq, int batch, int n_q, int n_kv) {
  const int rep = n_q / n_kv;
  const long wgs = (long)n_kv * batch * ((seq + 255) / 256);
  int split = 1;
  while (split < rep && wgs * split < 448 && rep % (split * 2) == 0) split *= 2;
  return split;
}

// bf16, head_dim 128 or 64, per-sequence tensors addressable with 32-bit byte offsets (buffer loads), 16-byte aligned rows, row blocks
// that fit the grid's third dimension (a few narrow heads reach it before the offsets do)
bool attn_mfma_applies(int dtype, int d, int seq, int n_q, int n_kv, const void* p0, const void* p1, const void* p2, const void* p3) {
  return dtype == DT_BF16 && (d == 128 || d == 64) && (seq + 127) / 128 < 65536 && (unsigned long long)(seq + 256) * (n_q + 2 * n_kv) * d * 2 < 0xF0000000ull &&
         (((uintptr_t)p0 | (uintptr_t)p1 | (uintptr_t)p2 | (uintptr_t)p3) & 15) == 0;
}

namespace {
template <int D, int NW, int NG> hipError_t fwd_d(const void* qkv, void* o, float* lse, int seq, int batch, int n_q, int n_kv, hipStream_t s) {
  constexpr int smem = 4 * Head<D>::TILE + Head<D>::ROW_LDS + (NG - 1) * NW * 512, GQ = 32 * NW;
  static LdsAttrOnce lds_attr;
  auto kern = attn_fwd_mfma<D, NW, NG>;
  if (hipError_t e = lds_attr.ensure(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(n_q, batch, (seq + GQ - 1) / GQ), dim3(64 * NW * NG), smem, s, (const bf16_t*)qkv, (bf16_t*)o, lse, seq, n_q, n_kv);
  return hipGetLastError();
}

struct BwdArgs {
  const void *qkv, *o, *dout;
  const float* lse;
  void* dqkv;
  float* ws;
  int seq, batch, n_q, n_kv;
  hipStream_t s;
  void* qcopy;
  const float2* rope;
};

template <int D, int NW, int NG> hipError_t dq_d(const BwdArgs& a) {
  constexpr int smem = 2 * 2 * Head<D>::TILE + Head<D>::ROW_LDS, GQ = 32 * NW;
  static LdsAttrOnce lds_attr;
  auto kern = attn_bwd_dq_mfma<D, NW, NG>;
  if (hipError_t e = lds_attr.ensure(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(a.n_q, a.batch, (a.seq + GQ - 1) / GQ), dim3(64 * NW * NG), smem, a.s, (const bf16_t*)a.qkv, (const bf16_t*)a.o,
      (const bf16_t*)a.dout, a.lse, a.ws, (bf16_t*)a.dqkv, (bf16_t*)a.qcopy, a.rope, a.seq, a.n_q, a.n_kv);
  return hipGetLastError();
}

// after dq_d, whose D array it reads
template <int D, int KT, int NG> hipError_t dkv_d(const BwdArgs& a) {
  constexpr int smem = 2 * (2 * Head<D>::TILE + 512) + 2 * KT * Head<D>::TILE + Head<D>::ROW_LDS, GK = 128 * KT;
  static LdsAttrOnce lds_attr;
  auto kern = attn_bwd_dkv_mfma<D, KT, NG>;
  if (hipError_t e = lds_attr.ensure(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  // partials of several workgroups per kv head need scratch that callers have for head size 128 only
  const int split = D == 128 ? attn_dkv_split(a.seq, a.batch, a.n_q, a.n_kv) : 1;
  float* partial = a.ws + (size_t)a.batch * a.n_q * a.seq;     // behind the D array
  hipLaunchKernelGGL(kern, dim3(a.n_kv * split, a.batch, (a.seq + GK - 1) / GK), dim3(256 * NG), smem, a.s, (const bf16_t*)a.qkv,
      (const bf16_t*)(a.qcopy ? a.qcopy : a.qkv), (a.qcopy ? a.n_q : a.n_q + 2 * a.n_kv) * D, (const bf16_t*)a.dout, a.lse, a.ws, (bf16_t*)a.dqkv,
      partial, a.rope, split, a.seq, a.n_q, a.n_kv);
  if (split > 1) {
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    const size_t items = (size_t)a.batch * a.seq * a.n_kv * 2 * D / 8;
    hipLaunchKernelGGL(attn_bwd_dkv_reduce, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, a.s, partial, (bf16_t*)a.dqkv, a.rope,
        split, a.batch * a.seq, a.seq, a.n_q, a.n_kv);
  }
  return hipGetLastError();
}

// Which division of the rows.  A wave has 32 query rows (forward, dQ) or 32 or 64 key rows (dK / dV); what varies is how many waves make a
// workgroup (NW: every row block of 32 NW queries reads its own K and V tiles) and whether two groups of waves share every block's
// 64 keys (queries) and add up at the end (NG = 2).  W = workgroups of 128 query rows = heads x sequences x blocks; one compute unit holds 8
// waves of these kernels, two per SIMD, and a lone wave leaves its SIMD idle for half of the time.
//  * Up to W = 256 a workgroup per compute unit is all there is: 64 rows and two groups, i.e. twice the workgroups and half the chain of
//    the longest row.  Forward, us, one group of 4 waves -> 2 x 2 waves: 4096 tokens, 8 heads 73.8 -> 55.2, 512, 16 heads 14.8 -> 10.9, 7673, 2 heads
//    132.6 -> 86.4; backward (both kernels) 8192, 8 / 1 heads 502.9 -> 434.8, 4096, 8 216.6 -> 162.4.  Rows of one or two tiles
//    have no chain to halve and pay for the addition: one group of 2 waves (109 tokens 6.4 / 6.3, 92 tokens 5.9 / 6.0).
//  * Up to two workgroups of four waves per compute unit, W = 512, long rows still gain from the halved chain: 6408 tokens, 8 heads (408)
//    126.0 -> 101.3, 4096, 16 heads (512, 4 x 2 waves) 91.1 -> 79.3; short ones do not: 280 tokens, 64 heads x 2 (384) 12.9 -> 17.2, 1237
//    tokens x 3, 16 heads (480) 33.6 -> 35.8.
//  * Beyond, 4 waves and two workgroups per compute unit: 2111 tokens x 8, 8 heads (1088) 90.6, 8 waves 100.6; 617 x 8, 32 heads 58.9 / 70.4.
//    Eight waves on one set of tiles, which read half as much, where their workgroups fill the chip twice or many times: 4096
//    tokens, 32 heads (512 of 256 rows) 146.6 / 137.0, 7298, 16 heads (464) 227.8 / 212.7, 16384, 40 heads 2607 / 2568; between, as above.
// Measured against two 32-row tiles per wave on four waves, the former kernels, in turn in one process on two cards: 16384 tokens, 40 heads forward
// 2765 -> 2603 and 2674 -> 2551, backward 8510 -> 8377 and 8417 -> 8219 (a third card 8265 -> 8293); 4096, 32 heads 148.6 -> 143.7 and 152.6 -> 140.9,
// 453 -> 439 and 442 -> 430; they are never the better ones in forward and dQ.
long row_workgroups(int seq, int batch, int n_q) { return (long)n_q * batch * ((seq + 127) / 128); }
}  // namespace

hipError_t launch_attn_fwd_mfma(const void* qkv, void* o, float* lse, int seq, int batch, int n_q, int n_kv, int d, hipStream_t s) {
  const long W = row_workgroups(seq, batch, n_q), wide = (long)n_q * batch * ((seq + 255) / 256);
  // heads of 64: three workgroups of four waves fit a compute unit; 246 tokens x 2, 16 heads (64) 9.3 -> 8.4 us, 1993, 16 heads (256) 42.5 -> 41.3,
  // 5661 x 8, one head (360) 108.7 -> 115.6
  if (d == 64) return W <= 256 ? fwd_d<64, 2, 1>(qkv, o, lse, seq, batch, n_q, n_kv, s) : fwd_d<64, 4, 1>(qkv, o, lse, seq, batch, n_q, n_kv, s);
  // one group of 2 waves over two where the compute units are full of rows of a few tiles: 192 tokens, W = 256 9.1 / 9.7 us, 256 10.9 / 11.2; W = 128 8.4 / 7.9, 9.4 /
  // 8.7; 320 tokens, W = 192 11.5 / 10.3
  if (W <= 256 && seq <= (W > 192 ? 256 : 128)) return fwd_d<128, 2, 1>(qkv, o, lse, seq, batch, n_q, n_kv, s);
  if (W <= 256 || (W <= 448 && seq > 640)) return fwd_d<128, 2, 2>(qkv, o, lse, seq, batch, n_q, n_kv, s);
  if (W > 448 && W <= 512 && seq > 1600) return fwd_d<128, 4, 2>(qkv, o, lse, seq, batch, n_q, n_kv, s);
  return (wide > 416 && wide <= 512) || wide >= 2048 ? fwd_d<128, 8, 1>(qkv, o, lse, seq, batch, n_q, n_kv, s)
                                                     : fwd_d<128, 4, 1>(qkv, o, lse, seq, batch, n_q, n_kv, s);
}

// Heads of 64, dK / dV: groups of waves that share a workgroup's keys.  WK = workgroups.  Up to two of them per compute unit two groups pay, with
// grouped heads also on short sequences, since a workgroup has all of a group's queries; us, one group -> two: 7298 tokens, 16 / 4 heads 1020 ->
// 887, 100 x 8, 16 / 4 26.2 -> 23.9, 1000 x 4, 64 / 8 (256) 325 -> 281, 1600 x 4, 32 / 8 (416) 289 -> 252.  Not beyond: 256 x 16, 32 / 16 (512) 62.1 -> 73.5,
// 640 x 16, 32 / 8 (640) 175 -> 199, 3000 x 4, 32 / 8 (768) 746 -> 809, 2048 x 8, 64 / 8 (1024) 1479 -> 1602; at 512 from some 1000 tokens on: 4096 x 2,
// 32 / 8 790 -> 688.  Without grouped heads 6426, 8 heads (408) 326 -> 293, 1024 x 4, 16 heads (512) 65.7 -> 66.8, 2111 x 8, 8 heads (1088) 205 ->
// 223, 128 x 16, 16 heads (256) 16.1 -> 17.1.
int attn_d64_key_groups(int seq, int batch, int n_q, int n_kv) {
  const long WK = row_workgroups(seq, batch, n_kv);
  return WK <= 480 ? (n_q > n_kv || seq > 128 ? 2 : 1) : n_q > n_kv && WK <= 512 && seq > 640 ? 2 : 1;
}

hipError_t launch_attn_bwd_mfma(const void* qkv, const void* o, const void* dout, const float* lse, void* dqkv, float* ws,
                                int seq, int batch, int n_q, int n_kv, int d, hipStream_t s, void* qcopy, const float2* rope) {
  const long W = row_workgroups(seq, batch, n_q);
  const BwdArgs a = {qkv, o, dout, lse, dqkv, ws, seq, batch, n_q, n_kv, s, qcopy, rope};
  hipError_t e;
  if (d == 64) {
    // dQ as in the forward pass: 1993 tokens, 16 heads (256) 101.2 -> 87.5 of both kernels' time, 6408, 8 heads (408) 418.6 -> 387.2, 361 x 3, 32 heads
    // (288) 37.2 -> 38.8, 1108, 64 heads (576) 138.7 -> 144.1; 192 tokens x 4, 32 heads (256) 18.6 -> 19.2
    if (W <= 256 && seq < (W > 128 ? 200 : 110)) e = dq_d<64, 2, 1>(a);
    else if (W <= 256 || (W <= 448 && seq > 640)) e = dq_d<64, 2, 2>(a);
    else e = dq_d<64, 4, 1>(a);
    if (e != hipSuccess) return e;
    return attn_d64_key_groups(seq, batch, n_q, n_kv) == 2 ? dkv_d<64, 1, 2>(a) : dkv_d<64, 1, 1>(a);
  }
  // dQ: 5661 tokens x 8, one head (360) 2 waves 271.6, 4 x 2 254.2, 2 x 2 275.5; 671 x 3, 16 heads (288) 48.2 / 54.7 / 54.5; 2048, 32 heads (512) 133.7 /
  // 137.3; 5096 x 8, 2 heads (640) 404 / 395, 8 waves 402; 2742 x 2, 16 heads (704) 265 / 265, 8 waves 254; 4096, 32 heads (1024) 474 / 459, 8 waves 426
  if (W <= 256) e = seq <= (W > 128 ? 400 : 192) ? dq_d<128, 2, 1>(a) : dq_d<128, 2, 2>(a);
  else if (W <= 640) e = seq > 2560 ? dq_d<128, 4, 2>(a) : dq_d<128, 2, 1>(a);
  else e = dq_d<128, 8, 1>(a);
  if (e != hipSuccess) return e;
  // dK / dV: two key tiles per wave feed every fragment read from LDS to two MFMAs, which a full chip wants, and leave one wave per SIMD; one tile
  // and two groups of waves, two per SIMD, for less.  Two tiles / two groups: 6745 tokens, 16 heads (848) 660 / 655, 7298 (928) 727 / 742, 2742 x 2, 16 heads
  // (704) 273 / 265, 2111 x 8, 8 heads (1088) 291 / 300.  Few blocks of queries: one group, 156 tokens x 2, 4 heads 23.0, two groups 23.4, 361 x 3, 32
  // heads 45.7 / 48.3, 296, 8 heads 30.0 / 29.9.
  if (W > 896) return dkv_d<128, 2, 1>(a);
  return seq <= 256 || (seq <= 384 && W > 256) ? dkv_d<128, 1, 1>(a) : dkv_d<128, 1, 2>(a);
}
