// Shared host/device helpers of libdecoquant (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "decoquant.h"

namespace dq {

constexpr int kTileTokens = 128;   // tokens per value-code tile and per decode work tile
constexpr int kMaxSplits = 64;     // upper bound on split-sequence partials per (b, head)
constexpr int kWsHeaderBytes = 256;
constexpr int kMaxCompressUnits = 1 << 22;   // blocks (keys and values counted apart) one compression call takes
constexpr int kMaxHeadGroups = 16; // matrix-core decode: groups of query heads per kv head
constexpr int kMaxGridY = 65535;   // largest y extent of a launch; more rows than that ride on the x index
constexpr int kMaxDecodeRows = 1 << 24;   // (sequence, query head) pairs one decode call takes (index arithmetic stays in 32 bits)
constexpr int kMaxTailRows = 1024; // rows of the fp16 tail a decode call takes per sequence and kv head
constexpr int kRun = 8;            // side of the third local tensor: tokens per run it mixes

constexpr uint32_t kCompressMostlyIdle = 1u << 31;   // internal flag of a compression call, see CompressJob
// The compression launch of dq_cache_append (dq_compress.hip): one block per (sequence, kv head) whose
// tail has filled, blk_idx[b] < 0 for all others.
int32_t compress_filled_tails(const dq_format* fmt, dq_cache* cache, const uint16_t* k_tail, const uint16_t* v_tail,
                              const int32_t* blk_idx, void* workspace, size_t workspace_bytes, hipStream_t st);

// Record a failed HIP runtime call for dq_last_hip_error().
void set_last_hip_error(hipError_t e);

#define DQ_HIP_CHECK(expr)                         \
  do {                                             \
    hipError_t _e = (expr);                        \
    if (_e != hipSuccess) {                        \
      ::dq::set_last_hip_error(_e);                \
      return DQ_EHIP;                              \
    }                                              \
  } while (0)

inline bool format_ok(const dq_format* f) {
  if (!f) return false;
  if (f->bits != 2 && f->bits != 4 && f->bits != 8) return false;
  if (f->head_dim != 64 && f->head_dim != 128) return false;
  if (f->j1 != 8 && f->j1 != 16 && f->j1 != 32) return false;
  if (f->j2 <= 0 || f->j1 * f->j2 != f->head_dim) return false;
  if (f->group <= 0 || f->head_dim % f->group) return false;
  const int seg = f->head_dim / 2;
  if (!(f->group == f->head_dim || (f->group <= seg && seg % f->group == 0))) return false;
  if ((f->group * f->bits) % 32) return false;  // a group covers whole 32-bit words
  if (f->block_tokens <= 0 || f->block_tokens % kTileTokens) return false;
  if (f->i3 != 1 && f->i3 != kRun) return false;
  if (f->levels != 0 && f->levels != 1) return false;
  if (f->i1 != 1 && f->i1 != 2 && f->i1 != 4) return false;
  if (f->i1 > 1 && (f->i3 != 1 || f->i1 * f->j1 > 32)) return false;
  return true;
}

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// ---- cache geometry (element strides, in units of the array's element type) ----
struct Geometry {
  int bits, G, d, j1, j2, Tb;
  int row_bytes;        // d*bits/8
  int groups;           // d/G
  int tiles_per_block;  // Tb/128
  int vrow_bytes;       // 128*bits/8: bytes of one (b2, r) value row inside a tile
  long codes_per_block; // bytes of k_codes (== v_codes) per block
  long scales_per_block;
  long small_per_block;
  int NB, H;
};

__host__ __device__ inline Geometry make_geometry(const dq_format& f, int kv_heads, int block_capacity) {
  Geometry g;
  g.bits = f.bits; g.G = f.group; g.d = f.head_dim; g.j1 = f.j1; g.j2 = f.j2; g.Tb = f.block_tokens;
  g.row_bytes = f.head_dim * f.bits / 8;
  g.groups = f.head_dim / f.group;
  g.tiles_per_block = f.block_tokens / kTileTokens;
  g.vrow_bytes = kTileTokens * f.bits / 8;
  g.codes_per_block = (long)f.block_tokens * g.row_bytes;
  g.scales_per_block = (long)f.block_tokens * g.groups;
  g.small_per_block = (long)(f.i1 * f.j1) * (f.i1 * f.j1);
  g.NB = block_capacity; g.H = kv_heads;
  return g;
}

// ---- fp16 bit helpers ----
__device__ inline float h2f(uint16_t h) {
  return (float)__builtin_bit_cast(_Float16, h);
}
__host__ __device__ inline uint16_t f2h_rne(float x) {
  return __builtin_bit_cast(uint16_t, (_Float16)x);
}

// fp64 -> fp16 bits with a single round-to-nearest-even; saturating variant clamps to +-65504.  The value
// is first rounded to odd in fp32 (13 more bits than fp16), which makes the second rounding land
// where a single one would.
__host__ __device__ inline uint16_t f64_to_f16_rne(double x, bool saturate, bool* saturated) {
  const float f = (float)x;
  const double e = x - (double)f;                       // what the first rounding dropped
  uint32_t bits = __builtin_bit_cast(uint32_t, f);
  // even and not exact (an infinity, whose e is a NaN, is): one further from zero where x is (e and f, a zero too, have the same
  // sign), one nearer otherwise.  No branches: a solver's lane converts 32 values in a row.
  const uint32_t unlike = (uint32_t)(__builtin_bit_cast(uint64_t, e) >> 32) ^ bits;
  const bool move = ((e > 0.0) | (e < 0.0)) & !(bits & 1u);
  bits += move ? (uint32_t)((int32_t)unlike >> 31) | 1u : 0u;
  const float odd = __builtin_bit_cast(float, bits);
  uint16_t h = f2h_rne(odd);
  if (saturate) {
    const bool over = __builtin_fabsf(odd) >= 65520.f;  // rounds to infinity
    if (saturated) *saturated |= over;
    h = over ? (uint16_t)((h & 0x8000u) | 0x7BFFu) : h;
  }
  return h;
}

}  // namespace dq
