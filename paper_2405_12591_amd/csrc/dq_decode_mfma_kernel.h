// Matrix-core decode attention over the compressed cache for the formats
//   bits in {2, 4, 8};  group = 128 with 1, 2 or 4 query heads of a kv head per workgroup, 8 in large launches,
//                       group = 64  with 1 or 2, 4 in large launches (see HP below),
// with head_dim = 128, j1 = 16, j2 = 8, block_tokens % 128 == 0, two or three local tensors.
// More query heads per kv head are served by several workgroups (head groups) over the same codes.
// Heads of 64 channels (j1 = 8, j2 = 8, group = 64) ride in pairs: two neighbouring kv heads are
// worked as one head of 128 channels whose small tensors are block-diagonal and whose query heads are
// the real ones (one or two of each kv head) padded with zeros (see P2 below).
//
// This is the fusion of dequantization with the product of the local tensors of Section 3.2 (arXiv
// 2405.12591) carried through the attention that follows it.  The low-bit codes never become
// floating point: a 32-bit word of codes is split into words of four bytes each
// (4-bit: x & 0x0F0F0F0F, (x >> 4) & 0x0F0F0F0F; 2-bit: (x >> 2k) & 0x03030303; 8-bit: x ^ 0x80808080) and fed to the
// int8 matrix cores; the other operand (the folded query, then the softmax weights times the
// value steps) is expressed as signed bytes, its limbs (four and three), relative to a per-tile power of two,
// one B column per limb, so the contraction is exact integer arithmetic.  Per 128-token tile,
// one wavefront
//   1. folds the keys' small tensor into the query,  q'[r, b2] = sum_b1 T_S^K[b1, r] q[b1, b2]
//      (one 16x16x16 f16 MFMA per two heads; T_S and q are fp16, so the products are exact),
//      and writes the limbs of q' * scale * log2(e) as B operands;
//   2. streams the key codes: S[t][limb] = sum_c (u[t, c] - offset) limb[c]  (16x16x64 i8 MFMA; limbs on the left where all sixteen
//      columns are in use or one head's stand in all of them, see TURN and SPREAD;
//      u = code + offset as stored; the offset's share comes from a constant-A MFMA and is the
//      accumulators' starting value);
//   3. online softmax with two tokens per lane (scores cross from the MFMA layout through wave-private LDS; SPREAD: they are
//      there already), or with eight tokens of one head per lane (TURN); w_t = p_t * step^V_t is cut into limbs, again B columns;
//   4. streams the value codes (stored token-contiguous): o'[r, b2] = sum_t u[t, r, b2] limb[t]
//      (several heads, two tensors: with the limbs as the left operand, which leaves a head's limbs in one lane);
//   5. applies the values' small tensor with fp32 16x16x4 MFMAs,
//      acc[b1, b2] = alpha * acc + sum_r T_S^V[b1, r] o'[r, b2]
//      (several b2 side by side first, so that the sixteen columns of these MFMAs are all in use).
// With two step groups per token row (group = 64: rows r < 8 and r >= 8 of the large tensor)
// every limb gets one B column per group: the key side zeroes the limbs of the other group's
// channels, the value side takes each row of o' from the column of that row's group.
// A query head takes 4 (one group) or 8 (two groups) of the sixteen B columns.
//
// MFMA operand layouts (lane l: n = l % 16, g = l / 16):
//   A[m][k]: lane holds row m = n, k = S*g + i (S values per lane);  B[k][n]: column n, same k;
//   D[m][n]: lane holds column n, rows m = 4*g + i.
#pragma once

#include <hip/hip_ext.h>

#include <type_traits>

#include "dq_decode.h"
#include "dq_tail.h"

namespace dq {

typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr float kLog2e = 1.4426950408889634f;
// Limbs are signed bytes: adding kDigitBias to an integer and taking it off by an exclusive or leaves in every lower byte a digit
// from -128 to 127, with the carries settled, for two cheap instructions (seven-bit limbs took a shift and a mask each).  With the
// steps' scales taken once per tile, a tile of four heads has 120 ns of issue less of 1310: 16 x 32 heads (8 kv heads) x 32768 tokens
// 93.3 -> 92.2 us, a serving step of 16 sequences of 3000 to 8000 tokens 33.1 -> 32.5.  The results' error against 64 bits over 900
// random caches: 1.9e-6 of the output's rms, 3.8e-6 with 21 and 28 bits in seven-bit limbs.
constexpr uint32_t kDigitBias = 0x00808080u;
constexpr int kMantBits = 22;             // weights: 22-bit integers, limb0 * 2^16 + limb1 * 2^8 + limb2
// The folded query takes all four columns of its group of four: 31 bits with the sign relative to the tile's
// largest |q'|, every bit its fp32 values have.  With three limbs of seven bits the rounding of the small entries of q' (2^-21 of
// the largest one, times 128 channels) was the largest error of the whole kernel on peaked softmaxes.
constexpr int kQueryBits = 31;
// With three local tensors the weights are signed mixtures over a run of tokens and what they
// multiply cancels across the run: they take all four columns as well.
constexpr int kSignedWeightBits = 31;

// ---- per-bit-width pieces -------------------------------------------------------------------
// Chunk: what one lane loads of a 16-row piece of codes (32 bytes at 8 bits, 16 at 4, 8 at 2); it
// feeds two int8 MFMAs of 16 codes per lane each.  `slot(e)` is the byte position, inside the 16
// bytes a lane hands to one MFMA, of the e-th of its 16 consecutive codes.
template <int BITS> struct Codec;
template <> struct Codec<4> {
  typedef u32x4 chunk_t;
  static constexpr int kOffset = 8;
  // first MFMA: words x, y (codes 0..15 of the lane's 32); second: words z, w
  static __device__ __forceinline__ i32x4 half(const chunk_t& c, int which) {
    const uint32_t M = 0x0F0F0F0Fu;
    const uint32_t x0 = which ? c.z : c.x, x1 = which ? c.w : c.y;
    i32x4 v;
    v.x = (int)(x0 & M);          // codes 0, 2, 4, 6
    v.y = (int)((x0 >> 4) & M);   // codes 1, 3, 5, 7
    v.z = (int)(x1 & M);          // codes 8, 10, 12, 14
    v.w = (int)((x1 >> 4) & M);   // codes 9, 11, 13, 15
    return v;
  }
  static __device__ __forceinline__ int slot(int e) { return (e & 8) + (e & 1) * 4 + ((e & 7) >> 1); }
};
template <> struct Codec<2> {
  typedef u32x2 chunk_t;
  static constexpr int kOffset = 2;
  static __device__ __forceinline__ i32x4 half(const chunk_t& c, int which) {
    const uint32_t M = 0x03030303u;
    const uint32_t x = which ? c.y : c.x;
    i32x4 v;
    v.x = (int)(x & M);           // codes 0, 4, 8, 12
    v.y = (int)((x >> 2) & M);    // codes 1, 5, 9, 13
    v.z = (int)((x >> 4) & M);    // codes 2, 6, 10, 14
    v.w = (int)((x >> 6) & M);    // codes 3, 7, 11, 15
    return v;
  }
  static __device__ __forceinline__ int slot(int e) { return (e & 3) * 4 + (e >> 2); }
};

template <> struct Codec<8> {
  typedef uint32_t chunk_t __attribute__((ext_vector_type(8)));
  static constexpr int kOffset = 0;   // the stored byte becomes the signed code by flipping its top bit
  static __device__ __forceinline__ i32x4 half(const chunk_t& c, int which) {
    const uint32_t F = 0x80808080u;
    i32x4 v;
    v.x = (int)((which ? c.s4 : c.s0) ^ F);
    v.y = (int)((which ? c.s5 : c.s1) ^ F);
    v.z = (int)((which ? c.s6 : c.s2) ^ F);
    v.w = (int)((which ? c.s7 : c.s3) ^ F);
    return v;
  }
  static __device__ __forceinline__ int slot(int e) { return e; }
};

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_f(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
// Maximum over the wave, taken on integer keys that order like the floats (for v >= 0 the bit
// pattern itself; otherwise the low 31 bits of negative values are flipped): an integer maximum
// takes its partner lane's value straight from the DPP operand, where a floating-point one needs
// the value copied and quieted first.  All-reduce over the 16 lanes of a row, then over the four rows.
__device__ __forceinline__ int wave_allmax_key(int x) {
  x = max(x, dpp_i<0xB1>(x));    // quad_perm [1,0,3,2]
  x = max(x, dpp_i<0x4E>(x));    // quad_perm [2,3,0,1]
  x = max(x, dpp_i<0x141>(x));   // row_half_mirror
  x = max(x, dpp_i<0x140>(x));   // row_mirror
  return max(max(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
             max(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}
__device__ __forceinline__ float wave_allmax(float v) {          // any finite values and -inf
  int x = __builtin_bit_cast(int, v);
  x ^= (x >> 31) & 0x7FFFFFFF;
  x = wave_allmax_key(x);
  x ^= (x >> 31) & 0x7FFFFFFF;
  return __builtin_bit_cast(float, x);
}
__device__ __forceinline__ float wave_allmax_nonneg(float v) {   // v >= 0 (+0 only)
  return __builtin_bit_cast(float, wave_allmax_key(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ float wave_allsum(float v) {
  v += dpp_f<0xB1>(v);
  v += dpp_f<0x4E>(v);
  v += dpp_f<0x141>(v);
  v += dpp_f<0x140>(v);
  return (lane_f(v, 0) + lane_f(v, 16)) + (lane_f(v, 32) + lane_f(v, 48));
}

// The same over the sixteen lanes of a row.
__device__ __forceinline__ float row_allmax(float v) {
  int x = __builtin_bit_cast(int, v);
  x ^= (x >> 31) & 0x7FFFFFFF;
  x = max(x, dpp_i<0xB1>(x));
  x = max(x, dpp_i<0x4E>(x));
  x = max(x, dpp_i<0x141>(x));
  x = max(x, dpp_i<0x140>(x));
  x ^= (x >> 31) & 0x7FFFFFFF;
  return __builtin_bit_cast(float, x);
}
__device__ __forceinline__ float row_allsum(float v) {
  v += dpp_f<0xB1>(v);
  v += dpp_f<0x4E>(v);
  v += dpp_f<0x141>(v);
  v += dpp_f<0x140>(v);
  return v;
}

// 2^e as a float for -126 <= e <= 127
__device__ __forceinline__ float pow2i(int e) {
  return __builtin_bit_cast(float, (uint32_t)(e + 127) << 23);
}

// BITS: code width.  NG: step groups per token row (group = 128 / NG).  R: query heads per kv head.  NW: wavefronts per workgroup (4 or 8); the tiles
// of one (sequence, kv head) are dealt round-robin to the NW waves of each of its n_split workgroups.
// TM: what to do about the fp16 tail (tokens not yet compressed).  0: there is none.  1, 2: its rows are
// dealt over all waves of the (sequence, kv head), which work them off while their first codes are on
// their way (1: the launch has one workgroup per (sequence, kv head); 2: several, so fewer rows per
// wave are requested up front).
// N3: three local tensors (format.i3 == 8).  Row a2*8 + e of the codes then belongs to the bond
// index e of the third tensor instead of a token: the tile's 128 row sums y are computed as
// before, the scores of the eight tokens of a run are s[a3] = sum_e T_3^K[e, a3] y[e], and the
// value rows are weighted with p'[e] = sum_a3 T_3^V[e, a3] p[a3] (signed, so these weights get a
// signed top limb like the query's).  The lanes that hold the eight rows of a run form a quad,
// so both products are quad broadcasts and fused multiply-adds.
// P2: a pair of kv heads of 64 channels each (j1 = 8), R / 2 query heads of each, as one virtual
// head of 128 channels and two step groups (NG = 2).  Virtual row r of the large tensors is row
// r % 8 of head r / 8, a virtual token row is the two heads' rows side by side, virtual query head hd
// is a real query head in the 64 channels of its kv head hd / (R / 2) and zero in the other's, and the
// small tensors are the heads' 8 x 8 ones on the diagonal of a 16 x 16 one.  Scores, softmax and the
// epilogue then run unchanged: head hd's scores come from its own channels only, and its output sits
// in the virtual channels of its own half (the other half, the other kv head's values under this
// head's weights, is dropped).  Only addresses (each lane reads its own head's arrays), the masks that
// realise the zeros, and the mapping of the output differ.  A head needs the four columns of one
// step group, so two query heads of each kv head share a code stream; more come in head groups of
// two.  Batch 8, 32 query on 8 kv heads, 2048 to 4096 tokens (15 MB): 74 + 7 us in the plain kernel
// these shapes used to take, 12 us here.
//
// HP = 2: two sets of four heads (two step groups: of two) in one workgroup, each with sixteen columns of its own.  What bounded more than four heads per kv head
// was the stream: every head group asked for the same codes (8 x 64 heads, 8 kv heads, x 32768 tokens: 587 MB through the L2s for 294 MB
// of cache; 68.5 us with one wave a SIMD, 66.2 with two) and unpacked them.  Here a chunk is asked for and unpacked once and multiplied with both
// sets: 221 registers, two waves a SIMD.  4 bits 65.4 -> 56 us, 2 bits 52.9 -> 45.5, 8 bits x 8192 tokens 47.4 -> 32.7; two step
// groups, 64 x 4 heads x 32768 tokens, 4 bits 65.5 -> 55.2.  Which launches take it: mfma_two_groups (dq_decode_mfma.hip).
// (two step groups: R counts the heads of both sets)
template <int BITS, int NG, int RQ, int NW, int TM, bool N3, bool P2, int HP = 1, bool KEEP = false, bool SP = true>
__global__ __launch_bounds__(64 * NW, (NW == 4 && BITS < 8) ? 2 : 1) void decode_mfma_kernel(DecodeArgs a) {
  constexpr int R = (NG == 2 && HP == 2) ? RQ / 2 : RQ;   // query heads of a set of columns
  static_assert(!P2 || (NG == 2 && (R == 2 || R == 4) && !N3), "a pair of heads is two step groups and two or four query heads");
  static_assert(HP == 1 || (HP == 2 && NG * R == 4 && R >= 2 && TM == 0 && !N3 && !P2), "sets of sixteen columns: no tail, two tensors");
  constexpr int RW = R * HP;                  // query heads per workgroup, in HP sets of sixteen columns
  typedef Codec<BITS> C;
  typedef typename C::chunk_t chunk_t;
  constexpr int CG = P2 ? 1 : NG;             // column groups per head (a pair: a head has channels of one step group only)
  constexpr int HPK = P2 ? R / 2 : RW;        // query heads per kv head of the workgroup
  constexpr int CPH = 4 * CG;                 // B columns per head: column CPH*head + 4*group + limb
  constexpr int NC = CPH * R;
  static_assert(NC <= 16, "too many heads for sixteen B columns");
  constexpr int F = (RW + 1) / 2;             // fold MFMAs (two heads each)
  constexpr int D = 128, J1 = 16, J2 = 8;
  // The epilogue multiplies o'[r] of every head and b2 by the values' small tensor, sixteen (head, b2) columns at a time.
  // With one head, or three tensors, one b2 fills only 3 R of the columns (one limb triple per head, once the two step groups'
  // columns have been merged): the columns of PK = 4 / R successive b2 are packed side by side first.
  // With several heads the value product has its operands the other way round (see step 4): a lane's result
  // registers are then the limbs of one head, which it joins as floats, two multiply-adds, and the rows r, now down the lanes, are
  // turned through LDS: 16 / R b2 of a head fill a set, 4 R / 2 matrix instructions per tile.  (Limbs joined by lane shifts, from
  // columns, took 176 vector instructions a tile with four heads where this takes 40; with two heads it was 16 matrix instructions
  // instead of 4.  64 query on 8 kv heads, 8 x 32768 tokens: 72.2 us, 66.0 so; 32 on 8, mixed lengths with tails: whole step 34.2,
  // 33.1; four 64-channel heads of 256 tokens: 6.0, 5.7.)
  constexpr bool JOIN = (R >= 2 && !N3);
  // Four heads, or two of two step groups, fill all sixteen columns: the score product has its operands the other way round as well.  A lane then holds the limbs
  // of one head's scores of eight tokens, joins them in registers and goes on with them; the steps reach it from the lanes
  // that asked for them by lane swaps.  Through LDS (8 writes and 32 reads a tile, four reductions' checks instead of one) the wave
  // waited for them: 16 x 32 heads (8 kv heads) x 32768 tokens 92.2 -> 90.5 us, so turned and with the folded query in 8 writes instead of
  // 32; a serving step of 16 sequences of 3000 to 8000 tokens 32.5 -> 31.4; 8 x 32 on 8 heads of 64 channels, 2048 to 4096 tokens
  // 11.5 -> 11.0 (10.6 with KEEP).  (Two heads of one step group would leave half the lanes idle in the softmax.)  Two step groups add a swap a token, for the
  // other group's share: 64 x 2 heads x 8192 tokens of two step groups, 4 bits, 24.1 -> 22.1, 64 x 2 x 128 6.1 -> 5.4.
  // (Pairs in 8 bits keep the other order: a lane's two tokens are neighbours there and lie in one line of two 64-byte rows, which two chunks would each ask for half
  // of: 128 units x 64 tiles 66.8 us turned, 50.6 so, 64 x 128 61.1, 47.5.  In 4 and 2 bits turning gains more than that costs, in 4 bits with several
  // head groups only if the halves meet in the caches: see KEEP.)
  constexpr bool TURN = (NC == 16 && R >= 2 && !N3 && !(P2 && BITS == 8));
  // One head of one step group fills four of the sixteen columns.  Its limbs stand in all four groups of columns, so that with the score product
  // turned every lane holds the limbs of every eighth token's score, and keeps those of its own two.  Through LDS (8 writes and 8 reads a
  // tile): 1 x 32 heads x 2999 tokens 7.54 -> 7.41 us, 8 x 32 x 4096 4 bits 24.6 -> 24.4, 8 bits the same.  (Three tensors: 8-bit codes would
  // drop to one wave a SIMD.  Two heads, their limbs in both halves of the columns and a lane swap between them: 14 x 32 64-channel heads x
  // 8442 tokens, 2 bits, 29.5 -> 30.1, so these go through LDS.)
  // (SP = false: large launches in 8 bits, see mfma_spread)
  constexpr bool SPREAD = (NC == 4 && !N3 && SP);
  constexpr int PK = JOIN ? 16 / R : 4 / R, NSET = J2 / PK;
  constexpr int TS = 20;                      // floats per (head, b2) of the joined values on their way through LDS (16 rows + pad)
  constexpr int RD = P2 ? 64 : D;             // channels of a real head (output, partials, cache rows)
  constexpr int RJ1 = P2 ? 8 : J1;            // rows of a real head's large tensors
  constexpr int ROWB = RD * BITS / 8;         // bytes of a key row in memory
  constexpr int VROWB = kTileTokens * BITS / 8;   // bytes of a value row (one r, one b2) in a tile
  constexpr int CHUNKB = sizeof(chunk_t);
  constexpr int SS = 132;                     // ints per column of the score staging (128 tokens + pad)
  constexpr int LS = 144;                     // bytes from column to column of the limbs (128 and a pad that keeps the b128 reads off each other's banks)
  constexpr int QS_BYTES = HP * NC * LS, PS_BYTES = HP * NC * LS, SS_BYTES = TURN ? RW * J2 * TS * 4 : SPREAD ? 1024 : NC * SS * 4;
  constexpr int MC = JOIN ? RW : NC;           // columns of a wave's result in the merge (JOIN: the limbs are joined already)
  constexpr int WAVE_LDS = QS_BYTES + PS_BYTES + SS_BYTES;
  static_assert(WAVE_LDS >= MC * D * 4 + 2 * RW * 4, "merge area must fit the wave's LDS");
  static_assert(!JOIN || RW * J2 * TS * 4 <= SS_BYTES, "the joined values take the scores' place");
  __shared__ __attribute__((aligned(16))) unsigned char smem[NW * WAVE_LDS];
  // the waves' partial results over the fp16 tail
  // (128 rows requested up front, by two workgroups if TM == 2; fewer where the heads leave fewer registers)
  constexpr int kTailBatch = TM == 1 ? 32 / NW : 16 / NW, kTailMost = R == 1 ? 8 : (R == 4 && (P2 || N3)) ? 2 : 4;
  typedef TailWave<R, kTailBatch < kTailMost ? kTailBatch : kTailMost, P2> Tail;
  __shared__ float s_tail[TM ? NW * Tail::kResultFloats : 1];
  __shared__ int s_last;
  __shared__ float s_wgt[HP * 4][kMaxSplits];
  __shared__ float s_sum[HP * 4];

  const int tid = threadIdx.x, lane = tid & 63;
#ifdef DQ_TIMELINE
  // time line of this wave (instrumented build only): slot numbers in dq_decode.h
  unsigned long long* const tl_wave = a.timeline
      ? a.timeline + ((long)(blockIdx.y * gridDim.x + blockIdx.x) * NW + (tid >> 6)) * kTimelineSlots : nullptr;
#define DQ_STAMP(slot)                                                          \
  do {                                                                          \
    if (tl_wave && lane == 0) tl_wave[slot] = __builtin_amdgcn_s_memrealtime(); \
  } while (0)
#else
#define DQ_STAMP(slot) \
  do {                 \
  } while (0)
#endif
  DQ_STAMP(0);
#ifdef DQ_TIMELINE
  if (tl_wave && lane == 0) tl_wave[20] = NW;
#endif
  // the wave's number as a scalar: everything derived from it (its tiles, their addresses) is then
  // computed once per wave on the scalar unit instead of once per lane
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, g = lane >> 4;
  // More query heads per kv head than the sixteen B columns hold (R of them per workgroup) are
  // served in head groups: head_groups workgroups per (sequence, kv head, split), each streaming
  // the same codes for its own R heads.  The groups are the slow part of the grid's y index, so the
  // workgroups of one (sequence, kv head) are a multiple of eight apart in launch order (whenever
  // the number of units is one) and land on the same XCD: while they run side by side, the second
  // to ask for a line finds it in that XCD's L2.
  // (rows normally ride on the grid's y index, splits of a row next to each other in launch order;
  // more rows than a y extent takes ride on x)
  const int split = a.rows_on_x ? blockIdx.y : blockIdx.x;
  const int row = a.rows_on_x ? blockIdx.x : blockIdx.y;
  const int n_units = (a.rows_on_x ? gridDim.x : gridDim.y) / a.head_groups;
  const int hgrp = row / n_units;
  const int bh = unit_of_row(row % n_units, n_units, a.unit_map);
  const int H = a.cache.kv_heads, NB = a.cache.block_capacity;
  constexpr int HPU = P2 ? 2 : 1;              // kv heads per unit
  const int b = bh / (H / HPU), h = (bh % (H / HPU)) * HPU;
  const long bh0 = (long)b * H + h;            // the unit's (first) kv head among all (sequence, kv head) pairs
  const int tpb = a.fmt.block_tokens / kTileTokens;
  const long codes_per_block = (long)a.fmt.block_tokens * ROWB;
  constexpr int MG = P2 ? 1 : NG;              // step groups per row in memory
  const long scales_per_block = (long)a.fmt.block_tokens * MG;

  // The sequence length lives in device memory and takes a memory round trip to read.  Tiles are dealt round-robin over all waves of all splits of this (sequence, kv head), so a wave's
  // first tile does not depend on the sequence length and its loads can start before the length is
  // known; they are wasted only if the sequence is shorter than that tile.
  const int first_tile = split * NW + wave;
  const int tile_stride = a.n_split * NW;
  const bool spec_ok = first_tile * kTileTokens < a.max_seq_len;
  int S = 0;  // the sequence's real length, read after the speculative loads are on their way

  // ---- the last workgroup of this (sequence, kv head) to finish merges the partial results ----
  const int heads_per_kv = a.q_heads / H;
  const long hq_first = (long)h * heads_per_kv + (long)hgrp * HPK;   // this workgroup's first query head
  // the last group may hold fewer than HPK heads of a kv head (3 = 3, 7 = 4 + 3): the columns of the
  // missing ones compute on a zero query and are never written out
  const int nhk = min(HPK, heads_per_kv - hgrp * HPK);
  const long bhq0 = (long)b * a.q_heads + hq_first;
  // virtual head hd: head hd of the group, or (a pair) head hd % HPK of kv head h + hd / HPK
  auto head_live = [&](int hd) -> bool { return (P2 ? hd % HPK : hd) < nhk; };
  auto head_row = [&](int hd) -> long {   // its row among all (sequence, query head) pairs; a missing one: the last one's
    return P2 ? bhq0 + (long)(hd / HPK) * heads_per_kv + min(hd % HPK, nhk - 1) : bhq0 + min(hd, nhk - 1);
  };
  int32_t* const ticket_counter = a.counters + (long)bh * a.head_groups + hgrp;
  const int n_contrib = a.n_split;   // workgroups that hand in partials
  auto ticket_and_merge = [&]() __attribute__((always_inline)) {
    // Ordering of the hand-over.  Producer: the partials above are device-scope (sc1) stores, which
    // write through the XCD's L2; every wave waits here until all of its own stores have been
    // acknowledged (the vector memory counter counts stores on this chip), and only after the
    // barrier that follows, i.e. after every wave of the workgroup has done so, does one thread take
    // a ticket, itself a device-scope read-modify-write performed at the memory side.  Consumer: the
    // workgroup that draws the last ticket knows that every other workgroup's increment, and so
    // every store ahead of it, has been performed; its loads of the partials are device-scope
    // loads (never served from this XCD's stale lines) issued after the second barrier, which the
    // compiler may not move them across.  No cache write-back or invalidation is involved.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __syncthreads();
    if (tid == 0) {
      const int ticket = __hip_atomic_fetch_add(ticket_counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_last = (ticket == n_contrib - 1);
      if (s_last) __hip_atomic_store(ticket_counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // clean for the next call
    }
    __syncthreads();
    if (!s_last) return;
    // Wave hd requests the maxima and sums of head hd's partials, one slot per lane, and every
    // thread the first eight slots of its output element, all in flight together; wave hd leaves
    // each slot's weight in LDS; then every thread adds up
    // its element over the slots, eight device-scope loads at a time (slots past the last one are
    // not read and weigh nothing).
    const int ns = a.n_slots;   // the splits: <= kMaxSplits = 64, a slot per lane (the waves' shares of the tail are in them)
    static_assert(kMaxSplits <= 64, "one slot per lane");
    auto load_slots = [&](const float* col, int sp, float (&v)[8]) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < 8; ++k)
        v[k] = (sp + k < ns) ? __hip_atomic_load(col + (sp + k) * (RD + 2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.f;
    };
    float v_first[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    constexpr int kHeadsAWave = (RW + NW - 1) / NW;
    float m0[kHeadsAWave], l0[kHeadsAWave];
#pragma unroll
    for (int k = 0; k < kHeadsAWave; ++k) {
      const int hd = wave + k * NW;
      m0[k] = -INFINITY; l0[k] = 0.f;
      if (hd < RW && head_live(hd)) {
        const float* base = a.partials + head_row(hd) * ns * (RD + 2);
        if (lane < ns) {
          m0[k] = __hip_atomic_load(base + lane * (RD + 2) + RD, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          l0[k] = __hip_atomic_load(base + lane * (RD + 2) + RD + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
    if (tid < RW * RD && head_live(tid / RD)) load_slots(a.partials + head_row(tid / RD) * ns * (RD + 2) + tid % RD, 0, v_first);
#pragma unroll
    for (int k = 0; k < kHeadsAWave; ++k) {
      const int hd = wave + k * NW;
      if (hd < RW && head_live(hd)) {
        const float M = wave_allmax(m0[k]);
        const float w0 = (m0[k] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m0[k] - M);
        if (lane < ns) s_wgt[hd][lane] = w0;
        const float L = wave_allsum(l0[k] * w0);
        if (lane == 0) s_sum[hd] = L;
      }
    }
    __syncthreads();
    for (int idx = tid; idx < RW * RD; idx += 64 * NW) {
      const int hd = idx / RD, c = idx % RD;
      if (!head_live(hd)) continue;
      const float* col = a.partials + head_row(hd) * ns * (RD + 2) + c;
      float o = 0.f;
      for (int sp = 0; sp < ns; sp += 8) {
        float v[8];
        if (idx == tid && sp == 0) {
#pragma unroll
          for (int k = 0; k < 8; ++k) v[k] = v_first[k];
        } else {
          load_slots(col, sp, v);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float wk = (sp + k < ns) ? s_wgt[hd][sp + k] : 0.f;
          o = (wk != 0.f) ? fmaf(v[k], wk, o) : o;   // an empty slot contributes nothing whatever it holds
        }
      }
      const float L = s_sum[hd];
      const float r = (L > 0.f) ? o / L : 0.f;
      a.out[head_row(hd) * RD + c] = f2h_rne(r);
      if (a.out_f32) a.out_f32[head_row(hd) * RD + c] = r;
    }
  };


  unsigned char* wl = smem + wave * WAVE_LDS;
  unsigned char* Qs = wl;                                        // [NC][8 row pairs][16 slots] bytes
  unsigned char* Ps = wl + QS_BYTES;                             // [NC][8 token groups][16 slots] bytes
  int* Ss = reinterpret_cast<int*>(wl + QS_BYTES + PS_BYTES);    // [NC][SS] ints
  const bool col_live = (n < NC) && (N3 || (n & 3) != 3);   // value side: three limbs per group of four columns (four with three local tensors)
  const bool col_live_k = n < NC;                      // key side: four
  // the epilogue's packed columns (see PK): column n holds head packed_head, slot packed_slot of its set
  const int packed_head = JOIN ? n / PK : (R == 1) ? 0 : (R == 4) ? (n >> 2) : (CG == 1) ? ((n >> 2) & 1) : (n >> 3);
  const int packed_slot = JOIN ? n % PK : (R == 1) ? (n >> 2) : (R == 4) ? 0 : (CG == 1) ? (n >> 3) : ((n >> 2) & 1);
  // JOIN: lane (row r = n, g) holds the limbs of head g (two step groups: of head g / 2, rows of group g % 2)
  const bool join_live = (CG == 1) ? g < R : (g & 1) == (n >> 3);
  float* const Ts = reinterpret_cast<float*>(Ss);                // [R * 8][TS]
  float* const join_to = Ts + (g / CG) * (J2 * TS) + n;
  const float* const join_from = Ts + (packed_head * J2 + packed_slot) * TS + 4 * g;

  // softmax layout: lane = 8*G16 + pi owns the two tokens of token group G16 whose weights sit in
  // B slots 2*pi and 2*pi + 1
  // (with three tensors and 2-bit codes the low lane bits are dealt the other way round, which
  // puts the eight rows of a run into one quad of lanes)
  const int G16 = lane >> 3, pi = (N3 && BITS == 2) ? (((lane & 3) << 1) | ((lane >> 2) & 1)) : (lane & 7);
  int tA, tB;
  if (BITS == 4) { tA = 16 * G16 + 8 * (pi >> 2) + ((0x5140 >> (4 * (pi & 3))) & 7); tB = tA + 2; }
  else if (BITS == 2) { tA = 16 * G16 + 8 * (pi & 1) + (pi >> 1); tB = tA + 4; }
  else { tA = 16 * G16 + 2 * pi; tB = tA + 1; }

  // key rows of the chunks.  TURN: chunks 2 k and 2 k + 1 hold the lane's tokens tA and tB of the k-th 32, the pair whose weights
  // share a 16-bit word of B slots; a chunk still asks for whole lines (two rows at 4 bits, four at 2, one at 8)
  const int key_row = (TURN || SPREAD) ? tA - 32 * g : n;
  constexpr int kPairRows = BITS == 4 ? 2 : BITS == 2 ? 4 : 1;   // tB - tA
  static_assert(!(TURN || SPREAD) || BITS < 8 || kPairRows * ROWB == 128, "8 bits: a chunk asks for whole lines");
  auto chunk_rows = [](int j) constexpr -> int { return (TURN || SPREAD) ? 32 * (j >> 1) + (j & 1) * kPairRows : 16 * j; };

  // KEEP: not past the caches (see launch_bits)
  auto load_key = [](const unsigned char* from) __attribute__((always_inline)) {
    const chunk_t* const at = reinterpret_cast<const chunk_t*>(from);
    return KEEP ? *at : __builtin_nontemporal_load(at);
  };

  // The fold has its operands the other way round as well, and its columns are dealt so that the four a lane gets lie side by side in B slots
  // (2-bit codes: two and two).  Three tensors, four heads and a tail do without in 4 and 2 bits: turned, small calls took longer (1 x 32 heads on
  // 4 x 640 tokens 13.6 us, 13.0 so; over 180 sizes 2.5 %), without a tail shorter (1 x 16 on 4 x 128 7.6, 7.8), in 8 bits 1.3 %.
  constexpr bool FOLD_TURN = !(N3 && R == 4 && TM != 0 && BITS < 8);
  auto fold_b2 = [](int c) constexpr -> int {   // the b2 of column c (mod 8)
    return !FOLD_TURN ? c : BITS == 4 ? 2 * (c & 3) + (c >> 2) : BITS == 2 ? (c >> 2) * 2 + ((c >> 1) & 1) + 4 * (c & 1) : c;
  };

  // loop-invariant operands of the fold, q[(b2, head)][k = b1].  The loads go out first (the
  // memory counter retires in issue order and q is needed before the first codes); the values are
  // packed further down, after the first tile's codes have been requested, so that the wait for q
  // does not sit in front of those requests.
  half4 bq[F];
  uint32_t q_raw[F][4];
  {
    const int b2 = fold_b2(n & 7);
#pragma unroll
    for (int f = 0; f < F; ++f) {
      const int hd = 2 * f + (n >> 3);
      // no branch here (columns past the last head read the last one and are zeroed when packed):
      // across a branch the compiler loses count of the loads in flight and waits for all of them
      // (a pair of heads: virtual row b1 = 4g + i of virtual head hd is row b1 % 8 of the real head;
      // the rows of the other head's half are zeroed when packed)
      const uint16_t* qp = a.q + head_row(min(hd, RW - 1)) * RD;
#pragma unroll
      for (int i = 0; i < 4; ++i) q_raw[f][i] = qp[((4 * g + i) & (RJ1 - 1)) * J2 + b2];
    }
  }

  float m_run[TURN ? HP : R], l_run[TURN ? HP : R];   // TURN: of head g, the sum over the lane's own tokens
#pragma unroll
  for (int hd = 0; hd < (TURN ? HP : R); ++hd) { m_run[hd] = -INFINITY; l_run[hd] = 0.f; }
  f32x4 acc[HP * NSET];
#pragma unroll
  for (int st = 0; st < HP * NSET; ++st) acc[st] = (f32x4){0.f, 0.f, 0.f, 0.f};

  const float qk_scale = a.scale * kLog2e;
  constexpr int kMinusWord = (int)((uint32_t)((256 - C::kOffset) & 255) * 0x01010101u);  // four bytes of -offset
  const i32x4 a_minus = {kMinusWord, kMinusWord, kMinusWord, kMinusWord};
  const i32x4 izero = {0, 0, 0, 0};

  // ---- the code stream of one wave: 16 chunks per tile (keys j = 0..7 in slots 0..7, values
  // b2 = 0..7 in slots 8..15) flow through a 16-slot register ring; a slot is refilled in place
  // with the same chunk of the wave's next tile as soon as it has been unpacked, so one whole
  // tile per wave is in flight at all times.  The memory counter retires loads in issue order,
  // so everything is requested in the order it will be used: the next tile's small tensors and
  // steps first (needed before its first key chunk), then the refills.
  chunk_t ring[16];
  struct Side { u32x2 ksm, vsm; uint32_t dkA, dkB, dvA, dvB; };   // small tensors + the lane's steps
  Side cur = {{0, 0}, {0, 0}, 0, 0, 0, 0};
  // three tensors: the columns of T_3^K of the lane's two tokens and the rows of T_3^V of its two
  // rows, eight fp16 each (kept apart from Side so that the other instances carry nothing of it)
  struct Side3 { u32x4 k3A, k3B, v3A, v3B; };
  Side3 cur3 = {{0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}};
  // a pair of heads: the second head's steps of the lane's two tokens (its step group 1)
  struct SideP { uint32_t dkA, dkB, dvA, dvB; };
  SideP curP = {0, 0, 0, 0};
  // the lane's part of a block-diagonal small tensor lies on the diagonal
  const bool small_live = !P2 || (g >> 1) == (n >> 3);
  // the kv head (0 or 1) of the head in the lane's column of fold f, and whether the lane's rows are its own
  auto fold_half = [&](int f) -> int { return (2 * f + (n >> 3)) / HPK; };
  auto fold_live = [&](int f) -> bool { return !P2 || (g >> 1) == fold_half(f); };
  // the same of the fold's result: columns 4 g + i, row n
  auto folded_half = [&](int f) -> int { return (2 * f + (g >> 1)) / HPK; };

  auto tile_ptrs = [&](int tile, const unsigned char*& kc, const unsigned char*& vc, long& blkid, int& tib) {
    blkid = bh0 * NB + tile / tpb;
    tib = tile % tpb;
    if (P2) {
      // keys: a virtual row is the two heads' rows side by side, two chunks each; values: virtual
      // row r of a b2 is row r % 8 of head r / 8 (the second head's blocks lie NB blocks further on)
      kc = a.cache.k_codes + (blkid + (g >> 1) * NB) * codes_per_block + (long)tib * kTileTokens * ROWB + key_row * ROWB + CHUNKB * (g & 1);
      vc = a.cache.v_codes + (blkid + (n >> 3) * NB) * codes_per_block + (long)tib * kTileTokens * ROWB + (n & 7) * VROWB + CHUNKB * g;
    } else {
      kc = a.cache.k_codes + blkid * codes_per_block + (long)tib * kTileTokens * ROWB + key_row * ROWB + CHUNKB * g;
      vc = a.cache.v_codes + blkid * codes_per_block + (long)tib * kTileTokens * ROWB + n * VROWB + CHUNKB * g;
    }
  };
  auto load_steps = [&](const uint16_t* p, int t) -> uint32_t {   // the fp16 steps of token t as stored
    if (MG == 1) return p[t];
    return *reinterpret_cast<const uint32_t*>(p + 2 * t);
  };
  auto load_side = [&](Side& sd, long blkid, int tib) {
    if (P2) {
      // the lane's row of its own head's 8 x 8 small tensor (used only where small_live)
      const long sb = (blkid + (n >> 3) * NB) * (RJ1 * RJ1) + (n & 7) * RJ1 + 4 * (g & 1);
      sd.ksm = *reinterpret_cast<const u32x2*>(a.cache.k_small + sb);
      sd.vsm = *reinterpret_cast<const u32x2*>(a.cache.v_small + sb);
    } else {
      sd.ksm = *reinterpret_cast<const u32x2*>(a.cache.k_small + blkid * (J1 * J1) + n * J1 + 4 * g);
      sd.vsm = *reinterpret_cast<const u32x2*>(a.cache.v_small + blkid * (J1 * J1) + n * J1 + 4 * g);
    }
    const uint16_t* ksc = a.cache.k_scales + blkid * scales_per_block + tib * kTileTokens * MG;
    const uint16_t* vsc = a.cache.v_scales + blkid * scales_per_block + tib * kTileTokens * MG;
    sd.dkA = load_steps(ksc, tA); sd.dkB = load_steps(ksc, tB);
    sd.dvA = load_steps(vsc, tA); sd.dvB = load_steps(vsc, tB);
  };
  auto load_sideP = [&](SideP& sd, long blkid, int tib) {   // the same steps of the pair's second head
    const uint16_t* ksc = a.cache.k_scales + (blkid + NB) * scales_per_block + tib * kTileTokens;
    const uint16_t* vsc = a.cache.v_scales + (blkid + NB) * scales_per_block + tib * kTileTokens;
    sd.dkA = ksc[tA]; sd.dkB = ksc[tB];
    sd.dvA = vsc[tA]; sd.dvB = vsc[tB];
  };
  auto load_side3 = [&](Side3& sd, long blkid) {
    const uint16_t* k3 = a.cache.k_small3 + blkid * (kRun * kRun);   // [a3][e]
    const uint16_t* v3 = a.cache.v_small3 + blkid * (kRun * kRun);   // [e][a3]
    sd.k3A = *reinterpret_cast<const u32x4*>(k3 + (tA & 7) * kRun);
    sd.k3B = *reinterpret_cast<const u32x4*>(k3 + (tB & 7) * kRun);
    sd.v3A = *reinterpret_cast<const u32x4*>(v3 + (tA & 7) * kRun);
    sd.v3B = *reinterpret_cast<const u32x4*>(v3 + (tB & 7) * kRun);
  };
  auto issue_tile = [&](int tile) {
    const unsigned char *kc, *vc;
    long blkid;
    int tib;
    tile_ptrs(tile, kc, vc, blkid, tib);
    load_side(cur, blkid, tib);
    if (N3) load_side3(cur3, blkid);
    if (P2) load_sideP(curP, blkid, tib);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 8; ++j) ring[j] = load_key(kc + chunk_rows(j) * ROWB);
#pragma unroll
    for (int b2 = 0; b2 < 8; ++b2) ring[8 + b2] = __builtin_nontemporal_load(reinterpret_cast<const chunk_t*>(vc + b2 * (RJ1 * VROWB)));
  };
  // fp16 step of group grp: from the packed word, or (a pair of heads) from the second head's word
  auto step_of = [&](uint32_t packed, uint32_t second, int grp) -> float {
    if (P2) return h2f((uint16_t)(grp ? second : packed));
    return h2f((uint16_t)(grp ? (packed >> 16) : (packed & 0xFFFFu)));
  };

  // Three tensors: outA = sum over the run of coefA[row] * x[row] (and outB with coefB), where the
  // eight values x of a run sit in a quad of lanes, two per lane (xA, xB), and the coefficient
  // vectors hold one fp16 per row of the run.  Quad lane k holds the rows offA(k) and offB(k).
  auto quad_mix = [&](float xA, float xB, const u32x4& coefA, const u32x4& coefB, float& outA, float& outB)
                      __attribute__((always_inline)) {
    typedef _Float16 half8 __attribute__((ext_vector_type(8)));
    const half8 cA = __builtin_bit_cast(half8, coefA), cB = __builtin_bit_cast(half8, coefB);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int offA = (BITS == 4) ? ((0x5140 >> (4 * k)) & 7) : (BITS == 2) ? k : 2 * k;
      const int offB = (BITS == 4) ? offA + 2 : (BITS == 2) ? k + 4 : 2 * k + 1;
      float a_k, b_k;
      switch (k) {   // the DPP control must be a literal
        case 0: a_k = dpp_f<0x00>(xA); b_k = dpp_f<0x00>(xB); break;
        case 1: a_k = dpp_f<0x55>(xA); b_k = dpp_f<0x55>(xB); break;
        case 2: a_k = dpp_f<0xAA>(xA); b_k = dpp_f<0xAA>(xB); break;
        default: a_k = dpp_f<0xFF>(xA); b_k = dpp_f<0xFF>(xB); break;
      }
      outA = fmaf((float)cA[offA], a_k, outA);
      outA = fmaf((float)cA[offB], b_k, outA);
      outB = fmaf((float)cB[offA], a_k, outB);
      outB = fmaf((float)cB[offB], b_k, outB);
    }
  };

  // One tile.  HAS_NEXT: the wave has another tile after this one.
  auto compute_tile = [&](const int tile, auto has_next_tag) __attribute__((always_inline)) {
    constexpr bool HAS_NEXT = decltype(has_next_tag)::value;
    const int tok0 = tile * kTileTokens;
    const unsigned char *kc_next = nullptr, *vc_next = nullptr;
    long blkid_next = 0;
    int tib_next = 0;
    if (HAS_NEXT) tile_ptrs(tile + tile_stride, kc_next, vc_next, blkid_next, tib_next);
    Side nxt = cur;
    if (HAS_NEXT) load_side(nxt, blkid_next, tib_next);
    Side3 nxt3;
    if (N3) {
      nxt3 = cur3;
      if (HAS_NEXT) load_side3(nxt3, blkid_next);
    }
    SideP nxtP;
    if (P2) {
      nxtP = curP;
      if (HAS_NEXT) load_sideP(nxtP, blkid_next, tib_next);
    }
    __builtin_amdgcn_sched_barrier(0);
    // (a tile with another one after it is full)
    const bool okA = HAS_NEXT || (tok0 + tA) < S, okB = HAS_NEXT || (tok0 + tB) < S;
    // three tensors: a row counts as soon as its run of eight holds a valid token
    const bool rowA = N3 && !HAS_NEXT ? (tok0 + (tA & ~7)) < S : okA, rowB = N3 && !HAS_NEXT ? (tok0 + (tB & ~7)) < S : okB;
    float dvA[NG], dvB[NG], dkA[NG], dkB[NG];
#pragma unroll
    for (int gr = 0; gr < NG; ++gr) {
      dvA[gr] = rowA ? step_of(cur.dvA, curP.dvA, gr) : 0.f;
      dvB[gr] = rowB ? step_of(cur.dvB, curP.dvB, gr) : 0.f;
      dkA[gr] = step_of(cur.dkA, curP.dkA, gr);
      dkB[gr] = step_of(cur.dkB, curP.dkB, gr);
    }
    const half4 vsm_h = __builtin_bit_cast(half4, small_live ? cur.vsm : u32x2{0u, 0u});

    // ---- 1. fold T_S^K into q; limbs of q' relative to 2^e >= max |q'| ----
    float q_unscale;
    float q_unscale_second = 0.f;   // a pair of heads: each head's query gets a scale of its own
    {
      const half4 aK = __builtin_bit_cast(half4, small_live ? cur.ksm : u32x2{0u, 0u});
      f32x4 fd[F];
      float amax = 0.f, amax_second = 0.f;
#pragma unroll
      for (int f = 0; f < F; ++f) {
        fd[f] = FOLD_TURN ? __builtin_amdgcn_mfma_f32_16x16x16f16(bq[f], aK, (f32x4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0)
                          : __builtin_amdgcn_mfma_f32_16x16x16f16(aK, bq[f], (f32x4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        // a pair of heads: rows r = n of the other head's half are zero by construction; they
        // are set to zero outright so that nothing the other head holds (a NaN, say) gets across
        if (P2 && (n >> 3) != folded_half(f)) fd[f] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (P2) amax_second = fmaxf(amax_second, folded_half(f) ? fabsf(fd[f][i]) : 0.f);
          amax = fmaxf(amax, (P2 && folded_half(f)) ? 0.f : fabsf(fd[f][i]));
        }
      }
      auto exponent_of = [&](float m) -> int {
        int e = 0;
        if (m > 0.f && m < INFINITY) e = __builtin_amdgcn_frexp_expf(m);  // m = f * 2^e, f in [0.5, 1)
        return max(min(e, 100), -90);
      };
      const int e = exponent_of(wave_allmax_nonneg(amax) * qk_scale);
      q_unscale = pow2i(e - (kQueryBits - 1));
      const float qn_first = qk_scale * pow2i(kQueryBits - 1 - e);   // |q' * qn| < 2^30
      float qn_second = 0.f;
      if (P2) {   // one scale per kv head
        const int e_second = exponent_of(wave_allmax_nonneg(amax_second) * qk_scale);
        q_unscale_second = pow2i(e_second - (kQueryBits - 1));
        qn_second = qk_scale * pow2i(kQueryBits - 1 - e_second);
      }
      // the fold's D layout: lane (n, g) holds row r = n of the columns 4 g + i, four b2 of head 2 f + (g >> 1).  Channel (r, b2) is
      // code number (r & 1)*8 + b2 of the 16 codes that row pair r >> 1 contributes to one MFMA: four channels side by side in
      // B slots go out in one word per limb (byte by byte: 32 writes instead of 8 with four heads).
#pragma unroll
      for (int f = 0; f < F; ++f) {
        if constexpr (!FOLD_TURN) {   // lane (n, g) holds rows r = 4 g + i of column n, b2 = n % 8
          const int hd = 2 * f + (n >> 3);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t v = ((uint32_t)(int)__builtin_rintf(fd[f][i] * qn_first) + kDigitBias) ^ kDigitBias;
            const int r = 4 * g + i;
            unsigned char* const dst = Qs + CPH * hd * LS + (r >> 1) * 16 + C::slot((r & 1) * 8 + (n & 7));
            dst[0] = (unsigned char)(v >> 24);
            dst[LS] = (unsigned char)(v >> 16);
            dst[2 * LS] = (unsigned char)(v >> 8);
            dst[3 * LS] = (unsigned char)v;
          }
          continue;
        }
        const int hd = 2 * f + (g >> 1);
        const float qn = (P2 && folded_half(f)) ? qn_second : qn_first;
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = ((uint32_t)(int)__builtin_rintf(fd[f][i] * qn) + kDigitBias) ^ kDigitBias;
        // the four words' bytes by limb
        const uint32_t low01 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), high01 = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
        const uint32_t low23 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u), high23 = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
        if (hd < RW) {
          const int grp = (CG == 2) ? (n >> 3) : 0;
          unsigned char* dst = Qs + (CPH * hd + 4 * grp) * LS + (n >> 1) * 16 + C::slot((n & 1) * 8 + fold_b2(4 * (g & 1)));
          if (BITS == 2) {   // two and two: b2, b2 + 4 and b2 + 1, b2 + 5
            *reinterpret_cast<uint16_t*>(dst) = (uint16_t)(high01 >> 16);
            *reinterpret_cast<uint16_t*>(dst + LS) = (uint16_t)high01;
            *reinterpret_cast<uint16_t*>(dst + 2 * LS) = (uint16_t)(low01 >> 16);
            *reinterpret_cast<uint16_t*>(dst + 3 * LS) = (uint16_t)low01;
            *reinterpret_cast<uint16_t*>(dst + 4) = (uint16_t)(high23 >> 16);
            *reinterpret_cast<uint16_t*>(dst + 4 + LS) = (uint16_t)high23;
            *reinterpret_cast<uint16_t*>(dst + 4 + 2 * LS) = (uint16_t)(low23 >> 16);
            *reinterpret_cast<uint16_t*>(dst + 4 + 3 * LS) = (uint16_t)low23;
          } else {
            *reinterpret_cast<uint32_t*>(dst) = __builtin_amdgcn_perm(high23, high01, 0x07060302u);
            *reinterpret_cast<uint32_t*>(dst + LS) = __builtin_amdgcn_perm(high23, high01, 0x05040100u);
            *reinterpret_cast<uint32_t*>(dst + 2 * LS) = __builtin_amdgcn_perm(low23, low01, 0x07060302u);
            *reinterpret_cast<uint32_t*>(dst + 3 * LS) = __builtin_amdgcn_perm(low23, low01, 0x05040100u);
          }
        }
      }
    }
    // (powers of two: the steps take the query's scale along, once per tile)
#pragma unroll
    for (int gr = 0; gr < NG; ++gr) {
      const float unscale = (P2 && gr) ? q_unscale_second : q_unscale;
      dkA[gr] = (N3 || okA) ? dkA[gr] * unscale : 0.f;
      dkB[gr] = (N3 || okB) ? dkB[gr] * unscale : 0.f;
    }
    // a token past the end scores minus infinity (its step, which may be anything, counts as zero)
    const float pastA = (N3 || okA) ? 0.f : -INFINITY, pastB = (N3 || okB) ? 0.f : -INFINITY;
    __builtin_amdgcn_wave_barrier();
    i32x4 bqs[HP][2];
#pragma unroll
    for (int hp = 0; hp < HP; ++hp) {
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        i32x4 t = izero;
        if (col_live_k || SPREAD) t = *reinterpret_cast<const i32x4*>(Qs + (hp * NC + (SPREAD ? n & 3 : n)) * LS + (2 * g + w) * 16);
        bqs[hp][w] = t;
      }
    }

    // ---- 2. scores: S[t][col] = sum_c (u[t, c] - offset) limb[col][c] ----
    [[maybe_unused]] int highA = 0, lowA = 0, highB = 0, lowB = 0;   // SPREAD: the limb pairs of the lane's two tokens
    [[maybe_unused]] float sc[HP][8];   // TURN: of head g (two step groups: of head g / 2, the share of group g % 2), the lane's tokens tA and tB of each 32
    // (the offset's share, the same for every token, is the accumulators' starting value)
    {
      i32x4 cinitk[HP];
      auto product = [&](const i32x4& codes, const i32x4& limbs, const i32x4& c) __attribute__((always_inline)) {
        return (TURN || SPREAD) ? __builtin_amdgcn_mfma_i32_16x16x64_i8(limbs, codes, c, 0, 0, 0) : __builtin_amdgcn_mfma_i32_16x16x64_i8(codes, limbs, c, 0, 0, 0);
      };
#pragma unroll
      for (int hp = 0; hp < HP; ++hp) {
        cinitk[hp] = izero;
        if (C::kOffset != 0) {
          cinitk[hp] = product(a_minus, bqs[hp][0], izero);
          cinitk[hp] = product(a_minus, bqs[hp][1], cinitk[hp]);
        }
      }
      // limb pairs are joined as integers (|S| <= 2^21 per limb: 128 channels x 128 x 128), then as floats
      auto keep = [&](int hp, int j, const i32x4& v) __attribute__((always_inline)) {
        if (TURN) sc[hp][j] = fmaf((float)(v[0] * 256 + v[1]), 65536.f, (float)(v[2] * 256 + v[3]));
        else if (SPREAD) {
          const int high = v[0] * 256 + v[1], low = v[2] * 256 + v[3];
          const bool own = g == (j >> 1);
          if (j & 1) { highB = own ? high : highB; lowB = own ? low : lowB; }
          else { highA = own ? high : highA; lowA = own ? low : lowA; }
        } else if (col_live_k) *reinterpret_cast<i32x4*>(Ss + n * SS + 16 * j + 4 * g) = v;
      };
      i32x4 s_prev[HP];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const i32x4 a0 = C::half(ring[j], 0), a1 = C::half(ring[j], 1);
        __builtin_amdgcn_sched_barrier(0);   // the slot is dead from here on: refill it in place
        if (HAS_NEXT) ring[j] = load_key(kc_next + chunk_rows(j) * ROWB);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int hp = 0; hp < HP; ++hp) {
          i32x4 s = product(a0, bqs[hp][0], cinitk[hp]);
          s = product(a1, bqs[hp][1], s);
          // the previous chunk's scores are taken while this chunk's MFMAs run
          if (j > 0) keep(hp, j - 1, s_prev[hp]);
          s_prev[hp] = s;
        }
      }
#pragma unroll
      for (int hp = 0; hp < HP; ++hp) keep(hp, 7, s_prev[hp]);
    }
    if (!TURN && !SPREAD) __builtin_amdgcn_wave_barrier();

    // ---- 3. online softmax, tokens tA and tB per lane (TURN: of head g, the pair of each 32 tokens) ----
    float v_unscale, vs = 0.f;
    float vs_second = 0.f;   // a pair of heads: the second head's steps get a scale of their own
    if (!N3) {
      float dvm = fmaxf(dvA[0], dvB[0]);
      if (NG == 2 && !P2) dvm = fmaxf(dvm, fmaxf(dvA[NG - 1], dvB[NG - 1]));
      const float dvmax = wave_allmax_nonneg(dvm);
      int e = 0;
      if (dvmax > 0.f && dvmax < INFINITY) e = __builtin_amdgcn_frexp_expf(dvmax);
      vs = pow2i(kMantBits - e);   // p * step * vs < 2^22 - 2^11
      v_unscale = pow2i(e - kMantBits);
      if (P2) {
        const float dvmax2 = wave_allmax_nonneg(fmaxf(dvA[NG - 1], dvB[NG - 1]));
        int e2 = 0;
        if (dvmax2 > 0.f && dvmax2 < INFINITY) e2 = __builtin_amdgcn_frexp_expf(dvmax2);
        vs_second = pow2i(kMantBits - e2);
        // the epilogue's rows b1 = n of the second head (n >= 8) undo the second head's scale
        if (n >> 3) v_unscale = pow2i(e2 - kMantBits);
      }
    }
    // the steps in units of the weights' integers (an infinite one counts as the largest; a NaN stays one and its weight becomes zero)
    float dvsA[NG], dvsB[NG];
#pragma unroll
    for (int gr = 0; gr < NG; ++gr) {
      constexpr float kMost = (float)((1 << kMantBits) - (1 << (kMantBits - 11)));
      const float vsg = (P2 && gr) ? vs_second : vs;
      dvsA[gr] = dvA[gr] * vsg;
      dvsB[gr] = dvB[gr] * vsg;
      dvsA[gr] = dvsA[gr] > kMost ? kMost : dvsA[gr];
      dvsB[gr] = dvsB[gr] > kMost ? kMost : dvsB[gr];
    }
    if constexpr (TURN) {
      // lane (n, g) has its pair's steps of the g-th 32 tokens; it needs those of all four for its own head (a pair of heads:
      // its kv head's; two step groups: of its own group).  Three swaps deal a register of each row of lanes to all of them.
      float kA[4], kB[4], wA[4], wB[4];
      auto deal = [&](const float (&x)[NG], float (&to)[4]) __attribute__((always_inline)) {
        const uint32_t x0 = __builtin_bit_cast(uint32_t, x[0]), x1 = __builtin_bit_cast(uint32_t, x[NG - 1]);
        if (CG == 2) {   // (odd rows of lanes take the second step group's)
          const auto h = __builtin_amdgcn_permlane16_swap(x0, x1, false, false);   // rows 0, 2; rows 1, 3
          const auto lo = __builtin_amdgcn_permlane32_swap(h[0], h[0], false, false), hi = __builtin_amdgcn_permlane32_swap(h[1], h[1], false, false);
          to[0] = __builtin_bit_cast(float, (uint32_t)lo[0]); to[2] = __builtin_bit_cast(float, (uint32_t)lo[1]);
          to[1] = __builtin_bit_cast(float, (uint32_t)hi[0]); to[3] = __builtin_bit_cast(float, (uint32_t)hi[1]);
        } else {
          const auto h = __builtin_amdgcn_permlane32_swap(x0, x1, false, false);   // rows 0, 1 twice; rows 2, 3 twice
          const auto lo = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false), hi = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);
          to[0] = __builtin_bit_cast(float, (uint32_t)lo[0]); to[1] = __builtin_bit_cast(float, (uint32_t)lo[1]);
          to[2] = __builtin_bit_cast(float, (uint32_t)hi[0]); to[3] = __builtin_bit_cast(float, (uint32_t)hi[1]);
        }
      };
      deal(dkA, kA);
      deal(dkB, kB);
      deal(dvsA, wA);
      deal(dvsB, wB);
#pragma unroll
      for (int hp = 0; hp < HP; ++hp) {
        float mt_lane = -INFINITY;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          // a token past the end scores minus infinity (its step counts as zero)
          const int t = tok0 + 32 * k + key_row;
          sc[hp][2 * k] = fmaf(sc[hp][2 * k], kA[k], (HAS_NEXT || t < S) ? 0.f : -INFINITY);
          sc[hp][2 * k + 1] = fmaf(sc[hp][2 * k + 1], kB[k], (HAS_NEXT || t + kPairRows < S) ? 0.f : -INFINITY);
          if (CG == 2) {   // the head's other step group is in the neighbouring row of lanes
#pragma unroll
            for (int i = 2 * k; i < 2 * k + 2; ++i) {
              const uint32_t w = __builtin_bit_cast(uint32_t, sc[hp][i]);
              const auto both = __builtin_amdgcn_permlane16_swap(w, w, false, false);
              sc[hp][i] = __builtin_bit_cast(float, (uint32_t)both[0]) + __builtin_bit_cast(float, (uint32_t)both[1]);
            }
          }
          mt_lane = fmaxf(mt_lane, fmaxf(sc[hp][2 * k], sc[hp][2 * k + 1]));
        }
        // the running maxima move in a sequence's first tiles and rarely afterwards: they are reduced only when some lane
        // holds a score above its head's
        if (__any(mt_lane > m_run[hp])) {
          const float m_new = fmaxf(m_run[hp], row_allmax(mt_lane));   // finite after the first tile (it has a valid token)
          const float alpha = __builtin_amdgcn_exp2f(m_run[hp] - m_new);
          m_run[hp] = m_new;
          l_run[hp] *= alpha;
          const float alpha_col = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(64 * CG * packed_head, __builtin_bit_cast(int, alpha)));
#pragma unroll
          for (int st = 0; st < NSET; ++st) acc[hp * NSET + st] *= alpha_col;
        }
        float p_sum = 0.f;
        unsigned char* const dst0 = Ps + (hp * NC + 4 * g) * LS + (n >> 3) * 16 + 2 * (n & 7);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float pA = __builtin_amdgcn_exp2f(sc[hp][2 * k] - m_run[hp]), pB = __builtin_amdgcn_exp2f(sc[hp][2 * k + 1] - m_run[hp]);
          p_sum += pA + pB;
          const uint32_t iA = ((uint32_t)fmaf(pA, wA[k], 0.5f) + kDigitBias) ^ kDigitBias;
          const uint32_t iB = ((uint32_t)fmaf(pB, wB[k], 0.5f) + kDigitBias) ^ kDigitBias;
          const uint32_t low = __builtin_amdgcn_perm(iB, iA, 0x05010400u);   // the two lowest limbs of both tokens
          unsigned char* const dst = dst0 + 32 * k;
          *reinterpret_cast<uint16_t*>(dst) = (uint16_t)__builtin_amdgcn_perm(iB, iA, 0x0C0C0602u);
          *reinterpret_cast<uint16_t*>(dst + LS) = (uint16_t)(low >> 16);
          *reinterpret_cast<uint16_t*>(dst + 2 * LS) = (uint16_t)low;
        }
        l_run[hp] += p_sum;
      }
    }
    float alpha[R];
    float wA[R][NG], wB[R][NG];   // three tensors: the weights, kept until their common scale is known
    float wmax = 0.f;
#pragma unroll
    for (int hd = 0; hd < (TURN ? 0 : R); ++hd) {
      float sA = pastA, sB = pastB;
#pragma unroll
      for (int gr = 0; gr < NG; ++gr) {
        if (P2 && gr != hd / HPK) continue;   // a head of a pair has its channels in its own step group only
        if (SPREAD) {
          sA = fmaf(fmaf((float)highA, 65536.f, (float)lowA), dkA[gr], sA);
          sB = fmaf(fmaf((float)highB, 65536.f, (float)lowB), dkB[gr], sB);
          continue;
        }
        const int* s0 = Ss + (CPH * hd + (P2 ? 0 : 4 * gr)) * SS;
        const int* s1 = s0 + SS;
        const int* s2 = s1 + SS;
        const int* s3 = s2 + SS;
        sA = fmaf(fmaf((float)(s0[tA] * 256 + s1[tA]), 65536.f, (float)(s2[tA] * 256 + s3[tA])), dkA[gr], sA);
        sB = fmaf(fmaf((float)(s0[tB] * 256 + s1[tB]), 65536.f, (float)(s2[tB] * 256 + s3[tB])), dkB[gr], sB);
      }
      if (N3) {   // rows -> tokens with T_3^K
        const float yA = sA, yB = sB;
        sA = 0.f; sB = 0.f;
        quad_mix(yA, yB, cur3.k3A, cur3.k3B, sA, sB);
        sA = okA ? sA : -INFINITY;
        sB = okB ? sB : -INFINITY;
      }
      // the running maximum moves in a sequence's first tiles and rarely afterwards: the wave-wide
      // reduction runs only when some lane holds a score above it
      const float mt_lane = fmaxf(sA, sB);
      float m_new = m_run[hd];                           // finite after the first tile (it has a valid token)
      alpha[hd] = 1.f;
      if (__any(mt_lane > m_new)) {
        m_new = wave_allmax(mt_lane);
        alpha[hd] = __builtin_amdgcn_exp2f(m_run[hd] - m_new);
      }
      const float pA = __builtin_amdgcn_exp2f(sA - m_new);
      const float pB = __builtin_amdgcn_exp2f(sB - m_new);
      l_run[hd] = l_run[hd] * alpha[hd] + (pA + pB);
      m_run[hd] = m_new;
      if (N3) {   // tokens -> rows with T_3^V; the weights are signed
        float qA = 0.f, qB = 0.f;
        quad_mix(pA, pB, cur3.v3A, cur3.v3B, qA, qB);
#pragma unroll
        for (int gr = 0; gr < NG; ++gr) {
          wA[hd][gr] = rowA ? qA * dvA[gr] : 0.f;
          wB[hd][gr] = rowB ? qB * dvB[gr] : 0.f;
          wmax = fmaxf(wmax, fmaxf(fabsf(wA[hd][gr]), fabsf(wB[hd][gr])));
        }
      } else {
#pragma unroll
        for (int gr = 0; gr < NG; ++gr) {
          // a pair of heads: only the head's own rows are kept, so the weights carry their steps
          if (P2 && gr != hd / HPK) continue;
          const uint32_t iA = ((uint32_t)fmaf(pA, dvsA[gr], 0.5f) + kDigitBias) ^ kDigitBias;
          const uint32_t iB = ((uint32_t)fmaf(pB, dvsB[gr], 0.5f) + kDigitBias) ^ kDigitBias;
          const uint32_t low = __builtin_amdgcn_perm(iB, iA, 0x05010400u);   // the two lowest limbs of both tokens
          unsigned char* dst = Ps + (CPH * hd + (P2 ? 0 : 4 * gr)) * LS + G16 * 16 + 2 * pi;
          *reinterpret_cast<uint16_t*>(dst) = (uint16_t)__builtin_amdgcn_perm(iB, iA, 0x0C0C0602u);
          *reinterpret_cast<uint16_t*>(dst + LS) = (uint16_t)(low >> 16);
          *reinterpret_cast<uint16_t*>(dst + 2 * LS) = (uint16_t)low;
        }
      }
    }
    if (N3) {
      // limbs relative to the largest weight of the tile: |w * vs| < 2^30
      wmax = wave_allmax_nonneg(wmax);
      int e = 0;
      if (wmax > 0.f && wmax < INFINITY) e = __builtin_amdgcn_frexp_expf(wmax);
      e = max(min(e, 100), -90);
      vs = pow2i(kSignedWeightBits - 1 - e);
      v_unscale = pow2i(e - (kSignedWeightBits - 1));
#pragma unroll
      for (int hd = 0; hd < R; ++hd) {
#pragma unroll
        for (int gr = 0; gr < NG; ++gr) {
          const uint32_t iA = ((uint32_t)(int)__builtin_rintf(wA[hd][gr] * vs) + kDigitBias) ^ kDigitBias;
          const uint32_t iB = ((uint32_t)(int)__builtin_rintf(wB[hd][gr] * vs) + kDigitBias) ^ kDigitBias;
          const uint32_t low = __builtin_amdgcn_perm(iB, iA, 0x05010400u), high = __builtin_amdgcn_perm(iB, iA, 0x07030602u);
          unsigned char* dst = Ps + (CPH * hd + 4 * gr) * LS + G16 * 16 + 2 * pi;
          *reinterpret_cast<uint16_t*>(dst) = (uint16_t)(high >> 16);
          *reinterpret_cast<uint16_t*>(dst + LS) = (uint16_t)high;
          *reinterpret_cast<uint16_t*>(dst + 2 * LS) = (uint16_t)(low >> 16);
          *reinterpret_cast<uint16_t*>(dst + 3 * LS) = (uint16_t)low;
        }
      }
    }
    __builtin_amdgcn_wave_barrier();

    // ---- 4 + 5. o' = sum_t u limb per b2, then the small-tensor epilogue ----
    i32x4 bp[HP][2];
#pragma unroll
    for (int hp = 0; hp < HP; ++hp) {
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        i32x4 t = izero;
        if (col_live) t = *reinterpret_cast<const i32x4*>(Ps + (hp * NC + n) * LS + (2 * g + v) * 16);
        bp[hp][v] = t;
      }
    }
    float alpha_col = 1.f;
#pragma unroll
    for (int hd = 0; hd < (TURN ? 0 : R); ++hd) alpha_col = (packed_head == hd) ? alpha[hd] : alpha_col;
    float aT[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) aT[i] = (float)vsm_h[i] * v_unscale;
    i32x4 cinitv[HP];
#pragma unroll
    for (int hp = 0; hp < HP; ++hp) {
      cinitv[hp] = izero;
      if (C::kOffset != 0) {
        cinitv[hp] = JOIN ? __builtin_amdgcn_mfma_i32_16x16x64_i8(bp[hp][0], a_minus, izero, 0, 0, 0) : __builtin_amdgcn_mfma_i32_16x16x64_i8(a_minus, bp[hp][0], izero, 0, 0, 0);
        cinitv[hp] = JOIN ? __builtin_amdgcn_mfma_i32_16x16x64_i8(bp[hp][1], a_minus, cinitv[hp], 0, 0, 0) : __builtin_amdgcn_mfma_i32_16x16x64_i8(a_minus, bp[hp][1], cinitv[hp], 0, 0, 0);
      }
    }
    if (!TURN && __any(alpha_col != 1.f)) {   // the running maximum moved: rare after the first tiles
#pragma unroll
      for (int st = 0; st < NSET; ++st) acc[st] *= alpha_col;
    }
    // o' of one b2 arrives with column 4*(NG*head + group) + limb.  pack() puts it into the
    // set's B operand: with two step groups a column's weights carry the step of one group only,
    // so rows r = 4g + i < 8 are taken from the first group's column and rows >= 8 from the second
    // group's (four lanes further on), which leaves one limb triple per head; then the triple
    // moves to the bank of four columns that slot k = b2 % PK owns.
    auto pack = [&](i32x4& pk, i32x4 o, auto k_tag) __attribute__((always_inline)) {
      constexpr int K = decltype(k_tag)::value % PK;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        int v = o[i];
        if (CG == 2) v = __builtin_amdgcn_update_dpp(v, v, 0x104 /* row_shl:4 */, 0xC, 0x5, false);
        if (K == 0) {
          pk[i] = v;
        } else {
          // live banks after the merge: R = 1: {0};  R = 2: {0, 1} (one group), {0, 2} (two groups)
          constexpr int kShift = (R == 2 && CG == 1) ? 8 * K : 4 * K;
          constexpr int kBanks = ((R == 1) ? 0x1 : (CG == 1) ? 0x3 : 0x5) << (kShift / 4);
          pk[i] = __builtin_amdgcn_update_dpp(pk[i], v, 0x110 + kShift /* row_shr */, 0xF, kBanks, false);
        }
      }
    };
    // JOIN: the limbs of o' joined as floats (one fp32 rounding, of the size of the accumulation's own)
    auto join = [&](int hp, int b2, const i32x4& o) __attribute__((always_inline)) {
      const float v = fmaf((float)o[0], 65536.f, fmaf((float)o[1], 256.f, (float)o[2]));
      if (join_live) join_to[(hp * R * J2 + b2) * TS] = v;
    };
    auto epilogue_joined = [&](int hp, int st) __attribute__((always_inline)) {   // b2 = st * PK .. + PK - 1 of every head
      const f32x4 v = *reinterpret_cast<const f32x4*>(join_from + (hp * R * J2 + st * PK) * TS);   // rows r = 4 g + i
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[hp * NSET + st] = __builtin_amdgcn_mfma_f32_16x16x4f32(aT[i], v[i], acc[hp * NSET + st], 0, 0, 0);
    };
    auto epilogue = [&](int st, const i32x4& pk) __attribute__((always_inline)) {
      f32x4 c = acc[st];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int word = pk[i];   // (a copy: the bit cast below wants an object, not an element of a vector)
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(aT[i], (float)word, c, 0, 0, 0);
      }
      acc[st] = c;
    };
    i32x4 pk_cur = izero, pk_done = izero, o_prev[HP];
#pragma unroll
    for (int b2 = 0; b2 < J2; ++b2) {
      const i32x4 a0 = C::half(ring[8 + b2], 0), a1 = C::half(ring[8 + b2], 1);
      __builtin_amdgcn_sched_barrier(0);
      if (HAS_NEXT) ring[8 + b2] = __builtin_nontemporal_load(reinterpret_cast<const chunk_t*>(vc_next + b2 * (RJ1 * VROWB)));
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (JOIN) {
#pragma unroll
        for (int hp = 0; hp < HP; ++hp) {
          i32x4 o = __builtin_amdgcn_mfma_i32_16x16x64_i8(bp[hp][0], a0, cinitv[hp], 0, 0, 0);
          o = __builtin_amdgcn_mfma_i32_16x16x64_i8(bp[hp][1], a1, o, 0, 0, 0);
          // the b2 before this one is joined, and a set that has gone through LDS multiplied, while this b2's integer MFMAs run
          if (b2 > 0) join(hp, b2 - 1, o_prev[hp]);
          if (b2 > PK && (b2 - 1) % PK == 0) epilogue_joined(hp, (b2 - 1) / PK - 1);
          o_prev[hp] = o;
        }
      } else {
        i32x4 o = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0, bp[0][0], cinitv[0], 0, 0, 0);
        o = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1, bp[0][1], o, 0, 0, 0);
        // the previous set's epilogue runs while this b2's integer MFMAs do
        if (b2 > 0 && b2 % PK == 0) epilogue(b2 / PK - 1, pk_done);
        if (b2 % PK == 0) pack(pk_cur, o, std::integral_constant<int, 0>{});
        else if (b2 % PK == 1) pack(pk_cur, o, std::integral_constant<int, 1>{});
        else if (b2 % PK == 2) pack(pk_cur, o, std::integral_constant<int, 2>{});
        else pack(pk_cur, o, std::integral_constant<int, 3>{});
        if (b2 % PK == PK - 1) pk_done = pk_cur;
      }
    }
    if constexpr (JOIN) {
#pragma unroll
      for (int hp = 0; hp < HP; ++hp) join(hp, J2 - 1, o_prev[hp]);
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int hp = 0; hp < HP; ++hp) epilogue_joined(hp, NSET - 1);
    } else {
      epilogue(NSET - 1, pk_done);
    }
    cur = nxt;
    if (N3) cur3 = nxt3;
    if (P2) curP = nxtP;
    __builtin_amdgcn_wave_barrier();
  };

  // The first requests go out in one straight line of code, without a branch: across a branch the
  // compiler loses count of the loads in flight and makes every later wait a wait for all of them.
  // So a wave whose first tile lies past max_seq_len reads tile 0 instead (in bounds: the cache
  // holds at least one block) and throws it away, and the tail's rows below its capacity are requested
  // whatever its length.  The tail's rows go first: they are worked off while the codes are on
  // their way.
  Tail tb;
  if (TM) tb.issue(a, b, h, hq_first, nhk, heads_per_kv, first_tile, tile_stride);
  issue_tile(spec_ok ? first_tile : 0);
  // Both lengths are requested only now (a scalar load that is still out holds up every wait on
  // scalar data, the addresses of the loads above among them) and before the asm statements below
  // (after them the compiler no longer treats memory as unchanged and would fetch these with vector
  // loads, whose wait covers the requests above).
  const int seq_len_raw = a.seq_lens[b];
  const int tail_len_raw = TM ? a.tail.tail_lens[b] : 0;
#pragma unroll
  for (int f = 0; f < F; ++f) {
    const int fold_head = 2 * f + (n >> 3);
    const bool live = fold_head < RW && head_live(fold_head) && fold_live(f);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      asm volatile("" : "+v"(q_raw[f][i]));   // nothing derived from q may move above the requests
      bq[f][i] = __builtin_bit_cast(_Float16, (uint16_t)(live ? q_raw[f][i] : 0u));
    }
  }
  if (TM) tb.finish(tail_len_raw, nhk, s_tail + wave * Tail::kResultFloats);

  if (CG == 2) {
    // A channel contributes nothing to the other group's columns: those bytes of the query limbs
    // are the same in every tile and are zeroed once (the fold writes only its own group's).
    static_assert(QS_BYTES % 16 == 0, "");
    for (int o = lane * 16; o < QS_BYTES; o += 64 * 16) *reinterpret_cast<i32x4*>(Qs + o) = izero;
    __builtin_amdgcn_wave_barrier();
  }
  S = min(max(seq_len_raw, 0), a.max_seq_len);
  const int tiles_total = (S + kTileTokens - 1) / kTileTokens;
  DQ_STAMP(1);
  {
    int tile = first_tile;
    [[maybe_unused]] int nth = 0;
    if (tile < tiles_total) {
      if (!spec_ok) issue_tile(tile);   // cannot happen while seq_len <= max_seq_len; kept for safety
      for (; tile + tile_stride < tiles_total; tile += tile_stride) {
        DQ_STAMP(2 + min(nth++, 15));
        compute_tile(tile, std::true_type{});
      }
      DQ_STAMP(2 + min(nth++, 15));
      compute_tile(tile, std::false_type{});
    }
  }
  DQ_STAMP(18);

  // ---- merge the waves of the workgroup ----
  float* Macc = reinterpret_cast<float*>(wl);            // [MC][128] per wave (reuses the wave's LDS)
  float* Mml = Macc + MC * D;                            // [RW] m, [RW] l
#pragma unroll
  for (int hd = 0; hd < (TURN ? HP : R); ++hd) l_run[hd] = TURN ? row_allsum(l_run[hd]) : wave_allsum(l_run[hd]);
  if (JOIN) {                 // [head][channel b1 * 8 + b2]
#pragma unroll
    for (int st = 0; st < HP * NSET; ++st) {
#pragma unroll
      for (int i = 0; i < 4; ++i) Macc[(st / NSET * R + packed_head) * D + (4 * g + i) * J2 + st % NSET * PK + packed_slot] = acc[st][i];
    }
  } else if (N3 || (n & 3) != 3) {   // [head][limb][channel b1 * 8 + b2]
#pragma unroll
    for (int st = 0; st < NSET; ++st) {
#pragma unroll
      for (int i = 0; i < 4; ++i) Macc[(4 * packed_head + (n & 3)) * D + (4 * g + i) * J2 + st * PK + packed_slot] = acc[st][i];
    }
  }
  if (TURN) {
#pragma unroll
    for (int hp = 0; hp < HP; ++hp) {
      if (n == 0 && g % CG == 0) { Mml[hp * R + g / CG] = m_run[hp]; Mml[RW + hp * R + g / CG] = l_run[hp]; }
    }
  } else if (lane == 0) {
#pragma unroll
    for (int hd = 0; hd < R; ++hd) { Mml[hd] = m_run[hd]; Mml[RW + hd] = l_run[hd]; }
  }
  __syncthreads();
  for (int idx = tid; idx < RW * RD; idx += 64 * NW) {
    // c: the real head's channel; cv: where it sits among the 128 channels the waves worked on
    const int hd = idx / RD, c = idx % RD, cv = P2 ? c + RD * (hd / HPK) : c;
    if (!head_live(hd)) continue;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      M = fmaxf(M, reinterpret_cast<const float*>(smem + w * WAVE_LDS)[MC * D + hd]);
      if (TM) M = fmaxf(M, s_tail[w * Tail::kResultFloats + hd * (D + 2) + D]);
    }
    float o = 0.f, L = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float* base = reinterpret_cast<const float*>(smem + w * WAVE_LDS);
      const float mw = base[MC * D + hd];
      const float wgt = (mw == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mw - M);
      const float* col = base + (JOIN ? hd : 4 * hd) * D + cv;
      const float v = JOIN ? col[0]
                      : N3 ? ((col[0] * 256.f + col[D]) * 256.f + col[2 * D]) * 256.f + col[3 * D]
                           : col[0] * 65536.f + col[D] * 256.f + col[2 * D];
      o = fmaf(v, wgt, o);
      L = fmaf(base[MC * D + RW + hd], wgt, L);
      if (TM) {   // the wave's share of the fp16 tail
        const float* tp = s_tail + w * Tail::kResultFloats + hd * (D + 2);
        const float wt = (tp[D] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(tp[D] - M);
        o = fmaf(tp[cv], wt, o);
        L = fmaf(tp[D + 1], wt, L);
      }
    }
    if (a.n_split == 1) {   // this workgroup saw the whole sequence: finish here
      const float r = (L > 0.f) ? o / L : 0.f;
      a.out[head_row(hd) * RD + c] = f2h_rne(r);
      if (a.out_f32) a.out_f32[head_row(hd) * RD + c] = r;
    } else {
      // device-scope stores: they go through to memory, past the per-XCD L2, so that a workgroup
      // on another XCD can read them without any cache write-back or invalidation
      float* part = a.partials + (head_row(hd) * a.n_slots + split) * (RD + 2);
      __hip_atomic_store(part + c, o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (c == 0) {
        __hip_atomic_store(part + RD, M, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // M in log2 units
        __hip_atomic_store(part + RD + 1, L, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
  if (a.n_split == 1) {
    DQ_STAMP(19);
    return;
  }

  ticket_and_merge();
  DQ_STAMP(19);
}
#undef DQ_STAMP
template <int BITS, int NG, int R, int TM, bool N3, bool P2, int HP = 1, bool KEEP = false, bool SP = true>
inline void launch_tm(const DecodeArgs& a, hipStream_t st) {
  const int units = a.cache.batch * a.cache.kv_heads / (P2 ? 2 : 1);
  const dim3 grid = a.rows_on_x ? dim3(units * a.head_groups, a.n_split) : dim3(a.n_split, units * a.head_groups);
  // the events, when given, receive the kernel's own begin and end timestamps
  // (8-bit codes: a wave's ring of chunks is twice as large and an 8-wave workgroup runs out of
  // registers, so that width always takes 4 waves)
  if constexpr (BITS < 8) {
    if (a.nw == 8) {
      hipExtLaunchKernelGGL((decode_mfma_kernel<BITS, NG, R, 8, TM, N3, P2, HP, KEEP, SP>), grid, dim3(512), 0, st, a.ev_start, a.ev_stop, 0, a);
      return;
    }
  }
  hipExtLaunchKernelGGL((decode_mfma_kernel<BITS, NG, R, 4, TM, N3, P2, HP, KEEP, SP>), grid, dim3(256), 0, st, a.ev_start, a.ev_stop, 0, a);
}

template <int BITS, int NG, int R, bool N3, bool P2 = false, bool KEEP = false, bool SP = true>
inline void launch_n3(const DecodeArgs& a, hipStream_t st) {
  if (!a.tail.k_tail) launch_tm<BITS, NG, R, 0, N3, P2, 1, KEEP, SP>(a, st);
  else if (a.n_split == 1) launch_tm<BITS, NG, R, 1, N3, P2, 1, KEEP, SP>(a, st);
  else launch_tm<BITS, NG, R, 2, N3, P2, 1, KEEP, SP>(a, st);
}

template <int BITS, int NG, int R>
inline void launch_r(const DecodeArgs& a, hipStream_t st) {
  if (a.fmt.i3 == kRun) return launch_n3<BITS, NG, R, true>(a, st);
  if constexpr (BITS == 8 && NG == 1 && R == 1) {
    if (!mfma_spread(a.cache.batch * a.cache.kv_heads, (a.max_seq_len + kTileTokens - 1) / kTileTokens))
      return launch_n3<BITS, NG, R, false, false, false, false>(a, st);
  }
  launch_n3<BITS, NG, R, false>(a, st);
}

template <int BITS>
int32_t launch_bits(const DecodeArgs& a, hipStream_t st) {
  if (a.pair_heads) {   // two kv heads of 64 channels per workgroup, one or two query heads of each
    if (a.heads_per_group == 1) launch_n3<BITS, 2, 2, false, true>(a, st);
    // 4 bits, turned: two chunks ask for half of every line of keys.  Requested past the caches, a line was fetched for each half; where several
    // head groups read it as well, plain loads are never slower (17 x 48 heads on 8 x 32768 tokens 143 us, 118 so; 8 x 96 on 32
    // x 2048 15.3, 14.2), with one group they lose up to 4 % beyond 64 MB of codes (8 x 64 on 32 x 32768 87.3, 90.9).  2 bits: the same within 1 %.
    else if (BITS == 4 && a.head_groups > 1) launch_n3<BITS, 2, 4, false, true, BITS == 4>(a, st);
    else launch_n3<BITS, 2, 4, false, true>(a, st);
    return DQ_OK;
  }
  const int rep = a.heads_per_group;   // query heads per workgroup (the last group may hold fewer)
  // two sets of columns know neither a tail nor a third tensor: a rule that sent such a call there must not be answered without them
  const bool two_sets_ok = !a.tail.k_tail && a.fmt.i3 == 1;
  if (a.fmt.group == 128) {
    switch (rep) {
      case 1: launch_r<BITS, 1, 1>(a, st); break;
      case 2: launch_r<BITS, 1, 2>(a, st); break;
      case 4: launch_r<BITS, 1, 4>(a, st); break;
      case 8:
        if (!two_sets_ok) return DQ_EINVAL;
        launch_tm<BITS, 1, 4, 0, false, false, 2>(a, st);
        break;
      default: return DQ_EINVAL;
    }
  } else {
    switch (rep) {
      case 1: launch_r<BITS, 2, 1>(a, st); break;
      case 2: launch_r<BITS, 2, 2>(a, st); break;
      case 4:
        if (!two_sets_ok) return DQ_EINVAL;
        launch_tm<BITS, 2, 4, 0, false, false, 2>(a, st);
        break;
      default: return DQ_EINVAL;
    }
  }
  return DQ_OK;
}


}  // namespace dq
