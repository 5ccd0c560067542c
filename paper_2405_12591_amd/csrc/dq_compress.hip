// Compression of K/V blocks into DecoQuant form (Section 3.1 of arXiv 2405.12591):
//   step 1  two-site MPO split of the regrouped block, M = T_S * T_L            (Eq. 2, Eq. 3)
//   step 2  per-group round-to-nearest quantization of T_L, T_S kept in fp16   (Eq. 1)
// Plain shapes, two kernels: `decompose_kernel` (Gram matrix, Jacobi eigen-solver, projection; one wave per block) writes the
// small tensor into the cache and the fp32 large tensor into the workspace;
// `quantize_tiles_kernel` turns fp32 rows into packed codes and fp16 steps.
#include "dq_common.h"
#include "dq_unit.h"

namespace dq {

// ------------------------------------------------------------------------------------------
// Quantize + pack one tile of 128 token rows (Eq. 1 per group).  256 threads.
// ------------------------------------------------------------------------------------------

// Step of a group: fp16(amax / qmax), the exact quotient rounded once (nearest, ties to even).
// The quotient is first rounded to odd in fp32 (13 more bits than fp16), which makes the second
// rounding to fp16 land where a single rounding of the exact quotient would.
template <int QMAX>
__device__ __forceinline__ uint16_t group_step_bits(float amax) {
  if (QMAX == 1) return f2h_rne(amax);
  const float q = amax / (float)QMAX;                  // correctly rounded fp32 division
  const float e = fmaf(-(float)QMAX, q, amax);         // sign of (exact quotient - q); 0 iff q is exact
  uint32_t bits = __builtin_bit_cast(uint32_t, q);
  if (e > 0.f) bits |= 1u;                             // exact lies above q: odd end of [q, next]
  else if (e < 0.f) bits -= (bits & 1u) ? 0u : 1u;     // exact lies below q: odd end of [prev, q]
  return f2h_rne(__builtin_bit_cast(float, bits));
}

// Code of one element: nearest integer of the exact x / step, ties to even, clamped.
// `q` = x * (1/step) from the fp32 reciprocal estimate is within 4e-5 of the exact quotient
// (|q| <= 128, three roundings of 2^-23), so rint(q) is the answer unless q sits that close to a
// half-integer.  Only then the exact path runs: the residual x - c*step is exact in fp64 (24-bit x,
// 7-bit c, 11-bit step) and settles the candidate, ties included.
constexpr float kNearTie = 0.5f - 0x1p-12f;

// Value of another lane by a fixed data-parallel-primitive pattern (no LDS round trip).
template <int CTRL>
__device__ __forceinline__ float lane_exchange(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}

__device__ __forceinline__ int settle_code(float x, float c0, float step, double half_step) {
  const double r = fma(-(double)c0, (double)step, (double)x);
  int c = (int)c0;
  const double ar = fabs(r);
  const bool move = (ar > half_step) | ((ar == half_step) & ((c & 1) != 0));   // false when r is NaN (step = inf)
  c += move ? (r > 0.0 ? 1 : -1) : 0;
  return c;
}

// The stored fields (code + bias, one byte each) of four elements that share a step; the same
// arithmetic as in quantize_tile: the reciprocal estimate decides unless the quotient sits within
// 2^-12 of a half-integer, then the exact residual does.
template <int BITS, bool FULL>
__device__ __forceinline__ uint32_t fields_of_four(float x0, float x1, float x2, float x3, float step, float inv) {
  constexpr int QMAX = (1 << (BITS - 1)) - 1;
  constexpr int QMIN = FULL ? -QMAX - 1 : -QMAX;
  constexpr int BIAS = 1 << (BITS - 1);
  const float xs[4] = {x0, x1, x2, x3};
  uint32_t fields = 0;
  bool near = false;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float q = xs[e] * inv;
    const float cf = __builtin_rintf(q);
    near |= fabsf(q - cf) > kNearTie;
    fields |= (uint32_t)(min(max((int)cf, QMIN), QMAX) + BIAS) << (8 * e);
  }
  if (near) {   // rare
    const double hs = 0.5 * (double)step;
    fields = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int c = settle_code(xs[e], __builtin_rintf(xs[e] * inv), step, hs);
      fields |= (uint32_t)(min(max(c, QMIN), QMAX) + BIAS) << (8 * e);
    }
  }
  return fields;
}

// Second half of the quantizer: the tile's stored fields, one byte per element in lds_u[128][D],
// leave as packed codes in key layout (rows of D elements) or value layout ([b2][r][128 tokens]).
// All NT threads of the workgroup call it, after a barrier that follows the last field's store;
// it ends with a barrier (lds_u may be reused).  The value layout needs D * (128 * BITS / 32 + 1)
// words of staging behind the fields.
// Parts of a tile whose value rows are collected before they are stored: enough for 32 bytes.
__host__ __device__ constexpr int pack_parts(int bits, int qt) {
  const int want = bits == 8 ? 64 : 32;   // bytes per store and row
  return (qt * bits / 8 >= want || qt >= kTileTokens) ? 1 : (want * 8 / (qt * bits) < kTileTokens / qt ? want * 8 / (qt * bits) : kTileTokens / qt);
}

// QT < 128: lds_u holds QT rows, the rows [part * QT, (part + 1) * QT) of the tile that begins at
// codes_out (staging D * (pack_parts(BITS, QT) * QT * BITS / 32 + 1) words).
template <int BITS, int D, int NT, int QT = kTileTokens>
__device__ __forceinline__ void pack_fields(uint8_t* __restrict__ lds_u, int j1, int j2, int value_layout,
                                            uint8_t* __restrict__ codes_out, int part = 0) {
  constexpr int d = D;
  const int tid = threadIdx.x;
  constexpr int PER_WORD = 32 / BITS;
  constexpr int total_words = QT * d / PER_WORD;
  uint32_t* out32 = reinterpret_cast<uint32_t*>(codes_out);
  if (!value_layout) {
    // key layout: rows of d elements, element index contiguous
    out32 += part * total_words;
    for (int w = tid; w < total_words; w += NT) {
      const uint32_t* f = reinterpret_cast<const uint32_t*>(lds_u + w * PER_WORD);
      uint32_t word = 0;
#pragma unroll
      for (int k4 = 0; k4 < PER_WORD / 4; ++k4) {
        const uint32_t x = f[k4];
#pragma unroll
        for (int k = 0; k < 4; ++k) word |= ((x >> (8 * k)) & 0xFFu) << ((4 * k4 + k) * BITS);
      }
      out32[w] = word;
    }
  } else {
    // value layout: [b2][r][128 tokens], tokens contiguous.  Consecutive lanes take consecutive
    // columns (conflict-free byte reads), the words are transposed through a padded LDS buffer and
    // leave in output order.
    constexpr int WPR = QT / PER_WORD;            // words per (b2, r) row held here
    constexpr int WPR_TILE = kTileTokens / PER_WORD;   // ... and in the tile
    // A row's words of AP successive parts are collected in the staging area (it lies behind the
    // fields and survives from part to part) and leave together, so that no store is shorter
    // than 32 bytes: shorter pieces of a row cost the memory system a whole request each.
    constexpr int AP = pack_parts(BITS, QT);
    constexpr int WST = AP * WPR;                 // words per row in the staging area
    uint32_t* stage = reinterpret_cast<uint32_t*>(lds_u + QT * d);
    const int sub = part % AP;
    for (int idx = tid; idx < total_words; idx += NT) {
      const int col = idx % d, wi = idx / d;
      const int b2 = col % j2, r = col / j2;
      uint32_t word = 0;
#pragma unroll
      for (int k = 0; k < PER_WORD; ++k)
        word |= (uint32_t)lds_u[(wi * PER_WORD + k) * d + col] << (k * BITS);
      stage[(b2 * j1 + r) * (WST + 1) + sub * WPR + wi] = word;
    }
    __syncthreads();
    if (sub == AP - 1) {
      const int first = (part - sub) * WPR;       // the collected words' place in the tile's row
      for (int w = tid; w < AP * total_words; w += NT)
        out32[(w / WST) * WPR_TILE + first + w % WST] = stage[(w / WST) * (WST + 1) + w % WST];
    }
  }
  __syncthreads();
}

// FULL: the non-default level set (format.levels == 1): codes in [-QMAX - 1, QMAX], and the step is
// the larger of max(x) / QMAX and max(-x) / (QMAX + 1), each rounded once to fp16 (rounding is
// monotonic, so that is the rounded larger quotient; the second divisor is a power of two).
template <int BITS, int D, bool FULL>
__device__ __forceinline__ void quantize_tile(const float* __restrict__ src,  // [128, D] fp32
                              int G, int j1, int j2, int value_layout,
                              uint8_t* __restrict__ codes_out,    // tile's code bytes
                              uint16_t* __restrict__ scales_out,  // [128, D/G]
                              uint8_t* __restrict__ lds_u) {      // [128 * D] stored fields (+ value staging)
  constexpr int QMAX = (1 << (BITS - 1)) - 1;
  constexpr int QMIN = FULL ? -QMAX - 1 : -QMAX;
  constexpr int BIAS = 1 << (BITS - 1);
  constexpr int d = D;
  constexpr int LPR = D / 4;                 // lanes per row, 4 elements each: 32 or 16
  constexpr int ROWS_PER_PASS = 256 / LPR;
  constexpr int PASSES = kTileTokens / ROWS_PER_PASS;
  const int tid = threadIdx.x;
  const int li = tid & (LPR - 1), rp = tid / LPR;
  const int gl = G >> 2;                     // lanes per group, a power of two
  const int groups = d / G;

  // Straight-line over the passes, stage by stage, so that the 8 or 16 independent rows a thread
  // handles overlap their latencies (loads, cross-lane steps, the division) instead of queueing.
  float4 v[PASSES];                          // the whole tile in flight before the first use
#pragma unroll
  for (int ps = 0; ps < PASSES; ++ps)
    v[ps] = *reinterpret_cast<const float4*>(src + (long)(ps * ROWS_PER_PASS + rp) * d + 4 * li);
  // amax: max |x| of the group (FULL: max x, at least 0); amin (FULL only): max -x, at least 0
  float amax[PASSES], amin[PASSES];
#pragma unroll
  for (int ps = 0; ps < PASSES; ++ps) {
    if (FULL) {
      amax[ps] = fmaxf(fmaxf(fmaxf(v[ps].x, v[ps].y), fmaxf(v[ps].z, v[ps].w)), 0.f);
      amin[ps] = fmaxf(fmaxf(fmaxf(-v[ps].x, -v[ps].y), fmaxf(-v[ps].z, -v[ps].w)), 0.f);
    } else {
      amax[ps] = fmaxf(fmaxf(fabsf(v[ps].x), fabsf(v[ps].y)), fmaxf(fabsf(v[ps].z), fabsf(v[ps].w)));
      amin[ps] = 0.f;
    }
  }
  // group maximum over gl lanes: lane exchanges inside a row of 16 lanes, then across the two rows
  auto group_max = [&](float (&m)[PASSES]) __attribute__((always_inline)) {
    if (gl > 1) {
#pragma unroll
      for (int ps = 0; ps < PASSES; ++ps) m[ps] = fmaxf(m[ps], lane_exchange<0xB1>(m[ps]));    // i ^ 1
    }
    if (gl > 2) {
#pragma unroll
      for (int ps = 0; ps < PASSES; ++ps) m[ps] = fmaxf(m[ps], lane_exchange<0x4E>(m[ps]));    // i ^ 2
    }
    if (gl > 4) {
#pragma unroll
      for (int ps = 0; ps < PASSES; ++ps) m[ps] = fmaxf(m[ps], lane_exchange<0x141>(m[ps]));   // 7 - i in 8
    }
    if (gl > 8) {
#pragma unroll
      for (int ps = 0; ps < PASSES; ++ps) m[ps] = fmaxf(m[ps], lane_exchange<0x140>(m[ps]));   // 15 - i in 16
    }
    if (LPR > 16 && gl > 16) {
#pragma unroll
      for (int ps = 0; ps < PASSES; ++ps) m[ps] = fmaxf(m[ps], __shfl_xor(m[ps], 16));
    }
  };
  group_max(amax);
  if (FULL) group_max(amin);
  float step[PASSES], inv[PASSES];
#pragma unroll
  for (int ps = 0; ps < PASSES; ++ps) {
    uint16_t sbits = group_step_bits<QMAX>(amax[ps]);
    if (FULL) {
      // both are bit patterns of non-negative fp16 values (or +inf), which order like integers
      const uint16_t down = f2h_rne(amin[ps] * (1.0f / (float)(QMAX + 1)));   // exact: a power of two
      sbits = sbits > down ? sbits : down;
    }
    step[ps] = h2f(sbits);
    inv[ps] = step[ps] > 0.f ? __builtin_amdgcn_rcpf(step[ps]) : 0.f;   // step 0 (and inf): every code 0
    if ((li & (gl - 1)) == 0) scales_out[(ps * ROWS_PER_PASS + rp) * groups + li / gl] = sbits;
  }
  uint32_t near_mask = 0;
#pragma unroll
  for (int ps = 0; ps < PASSES; ++ps) {
    const float xs[4] = {v[ps].x, v[ps].y, v[ps].z, v[ps].w};
    uint32_t fields = 0;
    bool near = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float q = xs[e] * inv[ps];
      const float cf = __builtin_rintf(q);
      near |= fabsf(q - cf) > kNearTie;
      fields |= (uint32_t)(min(max((int)cf, QMIN), QMAX) + BIAS) << (8 * e);
    }
    near_mask |= (near ? 1u : 0u) << ps;
    *reinterpret_cast<uint32_t*>(lds_u + (ps * ROWS_PER_PASS + rp) * d + 4 * li) = fields;
  }
  if (near_mask) {   // rare: some quotient sits within 2^-12 of a half-integer
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      if ((near_mask >> ps) & 1u) {
        const float xs[4] = {v[ps].x, v[ps].y, v[ps].z, v[ps].w};
        const double hs = 0.5 * (double)step[ps];
        uint32_t fields = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int c = settle_code(xs[e], __builtin_rintf(xs[e] * inv[ps]), step[ps], hs);
          fields |= (uint32_t)(min(max(c, QMIN), QMAX) + BIAS) << (8 * e);
        }
        *reinterpret_cast<uint32_t*>(lds_u + (ps * ROWS_PER_PASS + rp) * d + 4 * li) = fields;
      }
    }
  }
  __syncthreads();
  pack_fields<BITS, D, 256>(lds_u, j1, j2, value_layout, codes_out);
}

// LDS bytes quantize_tile needs: one byte per element plus the padded transpose buffer.
__host__ __device__ inline size_t quantize_lds_bytes(int d, int bits) {
  return (size_t)kTileTokens * d + (size_t)d * (kTileTokens * bits / 32 + 1) * sizeof(uint32_t);
}

// Stand-alone entry: contiguous input rows, contiguous outputs (dq_quantize_pack).
template <int BITS, int D, bool FULL>
__global__ __launch_bounds__(256) void quantize_pack_kernel(const float* __restrict__ t_large, int G, int j1,
                                                            int j2, int value_layout,
                                                            uint8_t* __restrict__ codes,
                                                            uint16_t* __restrict__ scales) {
  extern __shared__ uint8_t lds_u[];
  const long tile = blockIdx.x;
  const long tile_code_bytes = (long)kTileTokens * D * BITS / 8;
  quantize_tile<BITS, D, FULL>(t_large + tile * kTileTokens * D, G, j1, j2, value_layout,
                         codes + tile * tile_code_bytes, scales + tile * kTileTokens * (D / G), lds_u);
}

// The per-block status words of the decomposition become the call's two status words (flags OR-ed,
// sweeps at their maximum).  One workgroup of NT threads.
template <int NT>
__device__ __forceinline__ void fold_status(const int32_t* __restrict__ unit_status, int n_units,
                                            int32_t* __restrict__ status) {
  __shared__ int red[2];
  if (threadIdx.x < 2) red[threadIdx.x] = 0;
  __syncthreads();
  int flags = 0, sweeps = 0;
  for (int u = threadIdx.x; u < n_units; u += NT) {
    const int w = unit_status[u];
    flags |= w & 0xFF;
    sweeps = max(sweeps, w >> 8);
  }
  atomicOr(&red[0], flags);
  atomicMax(&red[1], sweeps);
  __syncthreads();
  if (threadIdx.x < 2) status[threadIdx.x] = red[threadIdx.x];
}

// Whether a call of the mostly idle kind (CompressJob) skips every sequence; all lanes of a wave ask.  Such
// a call leaves zero in its two status words.
__device__ __forceinline__ bool call_is_idle(const CompressJob& job) {
  if (!job.mostly_idle) return false;
  bool any = false;
  for (int i = threadIdx.x & 63; i < job.batch; i += 64) any |= job.blk_idx[i] >= 0;
  return !__any(any);
}

// Compress path: tile `blockIdx.x % tiles_per_block` of work unit `blockIdx.x / tiles_per_block`.
template <int BITS, int D, bool FULL>
__global__ __launch_bounds__(256) void quantize_tiles_kernel(const float* __restrict__ large_ws,
                                                             dq_format fmt, dq_cache cache,
                                                             CompressJob job,
                                                             const int32_t* __restrict__ unit_status,
                                                             int n_units, int32_t* __restrict__ status) {
  extern __shared__ uint8_t lds_u[];
  const Geometry g = make_geometry(fmt, cache.kv_heads, cache.block_capacity);
  if (blockIdx.x == 0) {
    if (call_is_idle(job)) {   // (hundreds of zero words need not be read: the same answer in every wave)
      if (threadIdx.x < 2) status[threadIdx.x] = 0;
      return;
    }
    fold_status<256>(unit_status, n_units, status);
  }
  const int tile = blockIdx.x % g.tiles_per_block;
  const int unit = blockIdx.x / g.tiles_per_block;
  const UnitRef ur = unit_ref(g, job, unit);
  const int which = ur.which, slot = ur.slot;
  if (slot < 0) return;
  const long blk = ur.bh * g.NB + slot;
  const float* src = large_ws + ((long)unit * g.Tb + (long)tile * kTileTokens) * D;
  uint8_t* codes = (which ? cache.v_codes : cache.k_codes) + blk * g.codes_per_block +
                   (long)tile * kTileTokens * g.row_bytes;
  uint16_t* scales = (which ? cache.v_scales : cache.k_scales) + blk * g.scales_per_block +
                     (long)tile * kTileTokens * g.groups;
  quantize_tile<BITS, D, FULL>(src, g.G, g.j1, g.j2, which, codes, scales, lds_u);
}

// ------------------------------------------------------------------------------------------
// Decomposition: Gram matrix in fp64, parallel cyclic Jacobi, projection.  One wavefront per
// (sequence, kv head, K|V) block, so all synchronisation is inside one wave.
// ------------------------------------------------------------------------------------------
constexpr int kGramTile = 8;  // tokens staged in LDS per Gram step

// Reciprocal and reciprocal square root in fp64 from the hardware estimates plus Newton steps
// (relative error about 1e-16).  The Jacobi rotations sit on a serial path of a few lanes, where the
// compiler's IEEE-exact division and square root sequences cost several times more.
__device__ __forceinline__ double fast_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = r * (2.0 - x * r);
  r = r * (2.0 - x * r);
  return r;
}
__device__ __forceinline__ double fast_rsqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = y * (1.5 - 0.5 * x * y * y);
  y = y * (1.5 - 0.5 * x * y * y);
  return y;
}

// n: side of the small tensor (i1 * j1); i1 rows are staged per token position
__host__ __device__ inline size_t decompose_lds_bytes(int n, int d, int i1) {
  const size_t mat = (size_t)n * (n + 1);
  return (5 * mat + 5 * (size_t)n) * sizeof(double) + 3 * (size_t)n * sizeof(int) +
         (size_t)kGramTile * d * i1 * sizeof(float) + 64;
}

// I1 > 1: a token factor on the small tensor (Eq. 2 with n = 2, i_1 = I1).  The regrouped matrix has
// rows (a1, b1) and columns (a2, b2), M[(a1, b1), (a2, b2)] = X[a1*i2 + a2, b1*j2 + b2]; everything
// below runs on its side I1*J1 instead of J1, and row a2*I1 + rho of the large tensor holds the
// elements T_L[rho*J1 + r', (a2, b2)].
template <int J1, int DD, int I1 = 1>
__global__ __launch_bounds__(64) void decompose_kernel(dq_format fmt, dq_cache cache, CompressJob job,
                                                       float* __restrict__ large_ws,
                                                       int32_t* __restrict__ unit_status) {
  const Geometry g = make_geometry(fmt, cache.kv_heads, cache.block_capacity);
  const int unit = blockIdx.x;
  const UnitRef ur = unit_ref(g, job, unit);
  const int which = ur.which, slot = ur.slot, nv = ur.nv;
  const long bh = ur.bh;
  if (slot < 0) {
    if (threadIdx.x == 0) unit_status[unit] = 0;
    return;
  }
  const int tid = threadIdx.x;
  constexpr int cj1 = J1, d = DD, j2 = DD / J1;   // compile-time shapes: loops unroll, no divisions
  constexpr int j1 = I1 * J1;            // side of the regrouped matrix's row index (a1, b1)
  constexpr int ld = j1 + 1;             // padded leading dimension of the small matrices
  constexpr int nent = j1 * j1;
  const int i2 = g.Tb / I1;              // positions a2 per block
  const uint16_t* X = ur.X;  // [nv, d] fp16 bits

  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  double* A0 = reinterpret_cast<double*>(lds_raw);   // Gram matrix, double buffered
  double* A1 = A0 + j1 * ld;
  double* V0 = A1 + j1 * ld;                         // accumulated rotations, double buffered
  double* V1 = V0 + j1 * ld;
  double* W = V1 + j1 * ld;                          // W[r][b1] = U[b1][order r] / sigma_r
  double* rc = W + j1 * ld;                          // rotation (c, s) per index (both partners)
  double* rs = rc + j1;
  double* lam = rs + j1;
  double* sigma = lam + j1;
  double* offarr = sigma + j1;                       // per rotating lane: largest relative off-diagonal
  int* partner = reinterpret_cast<int*>(offarr + j1);
  int* is_p = partner + j1;                          // 1 if the index is the first member of its pair
  int* order = is_p + j1;
  float* xs = reinterpret_cast<float*>(order + j1 + (j1 & 1));   // [I1][kGramTile][d]

  // ---- Gram matrix: Gm[p][q] = sum_{a2, b2} M[p, (a2, b2)] M[q, (a2, b2)], p = (a1, b1) ----
  // lane (pb, qb) of an 8 x 8 grid owns a (j1/8) x (j1/8) block of entries
  constexpr int BS = j1 / 8;
  const int pb = (tid >> 3) * BS, qb = (tid & 7) * BS;
  double acc[BS][BS];
#pragma unroll
  for (int i = 0; i < BS; ++i)
#pragma unroll
    for (int j = 0; j < BS; ++j) acc[i][j] = 0.0;
  // row p = (a1, b1) of M takes channel b1*j2 + b2 of token group a1's staged row
  int off_p[BS], off_q[BS];
#pragma unroll
  for (int i = 0; i < BS; ++i) {
    off_p[i] = ((pb + i) / cj1) * kGramTile * d + ((pb + i) % cj1) * j2;
    off_q[i] = ((qb + i) / cj1) * kGramTile * d + ((qb + i) % cj1) * j2;
  }
  // (positions past the last valid row of the first token group hold zeros in every group)
  const int np = min(i2, nv);
  for (int t0 = 0; t0 < np; t0 += kGramTile) {
    const int nt = min(kGramTile, np - t0);
    for (int i = tid; i < I1 * nt * d; i += 64) {
      const int a1 = i / (nt * d), rest = i % (nt * d);
      const int row = a1 * i2 + t0 + rest / d;
      xs[a1 * kGramTile * d + rest] = row < nv ? h2f(X[(long)row * d + rest % d]) : 0.f;
    }
    __syncthreads();
    for (int t = 0; t < nt; ++t) {
      const float* xr = xs + t * d;
#pragma unroll
      for (int b2 = 0; b2 < j2; ++b2) {
        double xp[BS], xq[BS];
#pragma unroll
        for (int i = 0; i < BS; ++i) {
          xp[i] = (double)xr[off_p[i] + b2];
          xq[i] = (double)xr[off_q[i] + b2];
        }
        // every product of two fp16 values is exact in fp64; only the sum rounds
#pragma unroll
        for (int i = 0; i < BS; ++i)
#pragma unroll
          for (int j = 0; j < BS; ++j) acc[i][j] = fma(xp[i], xq[j], acc[i][j]);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < BS; ++i)
#pragma unroll
    for (int j = 0; j < BS; ++j) A0[(pb + i) * ld + qb + j] = acc[i][j];
  for (int idx = tid; idx < nent; idx += 64) V0[(idx / j1) * ld + idx % j1] = (idx / j1 == idx % j1) ? 1.0 : 0.0;
  __syncthreads();

  // ---- parallel cyclic Jacobi: j1-1 rounds of j1/2 disjoint rotations per sweep ----
  double* Ac = A0; double* An = A1; double* Vc = V0; double* Vn = V1;
  const int nm1 = j1 - 1;
  int sweeps = 0;
  for (int sweep = 0; sweep < 16; ++sweep) {
    ++sweeps;
    if (tid < j1) offarr[tid] = 0.0;
    __syncthreads();
    for (int round = 0; round < nm1; ++round) {
      if (tid < j1 / 2) {
        int p, q;
        if (tid == 0) { p = nm1; q = round; }
        else { p = (round + tid) % nm1; q = (round - tid + nm1) % nm1; }
        if (p > q) { const int t = p; p = q; q = t; }
        const double app = Ac[p * ld + p], aqq = Ac[q * ld + q], apq = Ac[p * ld + q];
        double c = 1.0, s = 0.0;
        // skip off-diagonals that are already negligible against the diagonal (also keeps tau finite)
        if (fabs(apq) > 1e-300 && fabs(apq) > 1e-40 * (fabs(app) + fabs(aqq))) {
          const double tau = (aqq - app) * 0.5 * fast_rcp(apq);
          const double w = 1.0 + tau * tau;                       // sqrt(w) = w * rsqrt(w)
          const double t = (tau >= 0.0 ? 1.0 : -1.0) * fast_rcp(fabs(tau) + w * fast_rsqrt(w));
          c = fast_rsqrt(1.0 + t * t);
          s = t * c;
          const double rel2 = apq * apq * fast_rcp(fabs(app * aqq) + 1e-300);   // squared relative size
          if (rel2 > offarr[tid]) offarr[tid] = rel2;
        }
        rc[p] = c; rs[p] = s; rc[q] = c; rs[q] = s;
        partner[p] = q; partner[q] = p;
        is_p[p] = 1; is_p[q] = 0;
      }
      __syncthreads();
      // J has J[p][p] = c, J[p][q] = s, J[q][p] = -s, J[q][q] = c for each pair.
      // A' = J^T A J ; V' = V J.  Entry (i, j) needs A at {i, pi} x {j, pj}.
      for (int idx = tid; idx < nent; idx += 64) {
        const int i = idx / j1, j = idx % j1;
        const int pi = partner[i], pj = partner[j];
        // column j of J: J[j][j] = c_j, J[pj][j] = (is_p[j] ? -s : +s)
        const double cj = rc[j], sj = is_p[j] ? -rs[j] : rs[j];
        const double ci = rc[i], si = is_p[i] ? -rs[i] : rs[i];
        const double aj_i = Ac[i * ld + j] * cj + Ac[i * ld + pj] * sj;     // (A J)[i][j]
        const double aj_pi = Ac[pi * ld + j] * cj + Ac[pi * ld + pj] * sj;  // (A J)[pi][j]
        An[i * ld + j] = ci * aj_i + si * aj_pi;                            // (J^T (A J))[i][j]
        Vn[i * ld + j] = Vc[i * ld + j] * cj + Vc[i * ld + pj] * sj;
      }
      __syncthreads();
      double* t = Ac; Ac = An; An = t;
      t = Vc; Vc = Vn; Vn = t;
    }
    double om = 0.0;
    for (int i = 0; i < j1 / 2; ++i) om = fmax(om, offarr[i]);
    __syncthreads();
    if (om < 1e-24) break;   // every rotated off-diagonal was below 1e-12 of its diagonal pair
  }

  // ---- singular values, ordering, small tensor ----
  if (tid < j1) lam[tid] = Ac[tid * ld + tid];
  __syncthreads();
  if (tid < j1) {
    int rank = 0;
    const double me = lam[tid];
    for (int s = 0; s < j1; ++s) rank += (lam[s] > me) || (lam[s] == me && s < tid);
    order[rank] = tid;
  }
  __syncthreads();
  if (tid < j1) {
    const double lmax = fmax(lam[order[0]], 0.0);
    const double l = lam[order[tid]];
    sigma[tid] = (l > 1e-12 * lmax && l > 0.0) ? sqrt(l) : 0.0;
  }
  __syncthreads();
  {
    const long blk = (long)bh * g.NB + slot;
    uint16_t* small = (which ? cache.v_small : cache.k_small) + blk * g.small_per_block;
    bool sat = false;
    for (int idx = tid; idx < nent; idx += 64) {
      // neighbouring lanes write neighbouring entries of the stored array (keys are stored transposed)
      const int b1 = which ? idx / j1 : idx % j1, r = which ? idx % j1 : idx / j1;
      const double u = Vc[b1 * ld + order[r]];
      const double sg = sigma[r];
      W[r * ld + b1] = sg > 0.0 ? u / sg : 0.0;
      const uint16_t hb = f64_to_f16_rne(u * sg, true, &sat);
      if (which) small[b1 * j1 + r] = hb;   // values: natural [b1][r]
      else small[r * j1 + b1] = hb;         // keys: transposed [r][b1]
    }
    // this block's status word: bit 0 = T_S saturated, bits 8.. = Jacobi sweeps used
    const bool any_sat = __any(sat);
    if (tid == 0) unit_status[unit] = (any_sat ? 1 : 0) | (sweeps << 8);
  }
  __syncthreads();

  // ---- projection: T_L[r, (a2, b2)] = sum_p W[r][p] M[p, (a2, b2)], fp64 -> fp32, to row
  // a2*I1 + r / J1, element (r % J1)*j2 + b2 ----
  float* out = large_ws + (long)unit * g.Tb * d;
  for (int item = tid; item < i2 * j2; item += 64) {
    const int t = item / j2, b2 = item % j2;
    if (t < nv) {
      double xv[j1];
#pragma unroll
      for (int p = 0; p < j1; ++p) {
        const int row = (p / cj1) * i2 + t;
        xv[p] = row < nv ? (double)h2f(X[(long)row * d + (p % cj1) * j2 + b2]) : 0.0;
      }
      for (int r = 0; r < j1; ++r) {
        double a = 0.0;
#pragma unroll
        for (int p = 0; p < j1; ++p) a = fma(W[r * ld + p], xv[p], a);
        out[((long)t * I1 + r / cj1) * d + (r % cj1) * j2 + b2] = (float)a;
      }
    } else {
      for (int r = 0; r < j1; ++r) out[((long)t * I1 + r / cj1) * d + (r % cj1) * j2 + b2] = 0.f;
    }
  }
}

// ------------------------------------------------------------------------------------------
// Fast decomposition for the common shape d = 128, j1 = 16, j2 = 8: one wave per block, the two
// dense contractions (Gram matrix, projection) on the fp64 matrix cores, the eigen-solver in
// registers.
//
// v_mfma_f64_16x16x4_f64 operand layout (one double per lane for A and B, four for D):
//   A[m][k]: lane l -> m = l % 16, k = l / 16;  B[k][n]: lane l -> n = l % 16, k = l / 16;
//   D[m][n]: lane l, register i -> n = l % 16, m = l / 16 + 4 i.
// ------------------------------------------------------------------------------------------
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// Rotation (c, s) that annihilates entry (p, q) of a symmetric matrix; `big` reports whether that
// entry was still above kSettled relative to its diagonal pair.  The angle comes from the hardware
// estimates alone (relative error near 1e-7: the entry shrinks by that factor instead of
// vanishing, which does not slow the quadratic convergence); c is refined to full precision so
// that c^2 + s^2 = 1 and the accumulated rotations stay orthogonal.
constexpr double kSettled2 = 1e-9;   // (3e-5)^2: one more sweep squares 3e-5 to about 1e-9

__device__ __forceinline__ void jacobi_rotation(double app, double aqq, double apq, double floor_abs,
                                                double& c, double& s, bool& big) {
  // Entries at the rounding level of the whole matrix (floor_abs = 1e-17 * trace) or negligible
  // against their own diagonal pair are skipped: rotating them changes nothing that is kept, and
  // between two numerically zero eigenvalues they would never settle.  Written without branches.
  const bool live = fabs(apq) > floor_abs && fabs(apq) > 1e-40 * (fabs(app) + fabs(aqq));
  const double tau = (aqq - app) * 0.5 * __builtin_amdgcn_rcp(apq);
  const double root = __builtin_amdgcn_sqrt(fma(tau, tau, 1.0));
  const double t = copysign(__builtin_amdgcn_rcp(fabs(tau) + root), tau);
  const double cc = fast_rsqrt(fma(t, t, 1.0));
  c = live ? cc : 1.0;
  s = live ? t * cc : 0.0;
  big = live && apq * apq > kSettled2 * fabs(app * aqq);
}

// ---- eigen-decomposition of the 16 x 16 Gram matrix: one-sided Jacobi in registers ----
// Columns of G are rotated against each other until they are orthogonal: G Q = U Lambda, so the
// normalised columns are the eigenvectors and the columns' norms the eigenvalues; no matrix of
// accumulated rotations is needed.  A lane holds a pair of columns (x, y) and derives their
// rotation once; eight lanes hold the sixteen columns.  ROWS of the sixteen rows sit in a lane:
// ROWS = 2 spreads one block over the wave (lane = pair + 8 * row group; the shortest chain), ROWS = 4 and 8 two and
// four, ROWS = 16 works eight blocks per wave (lane = pair + 8 * block; no sum over lanes, every
// rotation derived once per block).  Between rounds the y columns move to another lane of the eight
// by a data-parallel-primitive pattern, so a round touches no LDS at all: on one wave per SIMD, which
// issues an instruction every 5.3 cycles whatever it is, a round of about 55 instructions takes 320
// cycles, against 550 for a two-sided iteration in LDS (100 instructions, two LDS round trips and a lane
// exchange through LDS).  Whole call on one block per compute unit (256 blocks): 40 -> 30 us; on 320: 61
// -> 38 us (four waves per block instead of two in the latter, now that the solver is shorter).
// All sums over rows run over the same tree whatever ROWS is, so every build of the kernels that
// calls this gets the same bits.
// Accuracy, replayed on the CPU over blocks whose singular values span 0 to 5.8 decades (600 to 2000 each),
// against the two-sided iteration: rows of T_L orthonormal to 3e-9 / 7e-9 on flat spectra, both at the
// fp32 rounding of T_L once it is stored (9e-9 to 8e-8); T_S T_L before any rounding 5e-10 / 2e-15 off,
// because the normalised columns are orthogonal to 2e-9 only, and 2.6e-8 for both with T_L in fp32.
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppXor3 = 0x1B, kDppXor7 = 0x141, kDppXor8 = 0x128;
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  u32x2 w = __builtin_bit_cast(u32x2, v);
  w.x = (unsigned)__builtin_amdgcn_update_dpp(0, (int)w.x, CTRL, 0xF, 0xF, true);
  w.y = (unsigned)__builtin_amdgcn_update_dpp(0, (int)w.y, CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, w);
}
// v of this lane plus v of the lane 16 (32) further on or back
__device__ __forceinline__ double add_xor16(double v) {
  const u32x2 w = __builtin_bit_cast(u32x2, v);
  const auto lo = __builtin_amdgcn_permlane16_swap(w.x, w.x, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(w.y, w.y, false, false);
  return __builtin_bit_cast(double, u32x2{lo[0], hi[0]}) + __builtin_bit_cast(double, u32x2{lo[1], hi[1]});
}
__device__ __forceinline__ double add_xor32(double v) {
  const u32x2 w = __builtin_bit_cast(u32x2, v);
  const auto lo = __builtin_amdgcn_permlane32_swap(w.x, w.x, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(w.y, w.y, false, false);
  return __builtin_bit_cast(double, u32x2{lo[0], hi[0]}) + __builtin_bit_cast(double, u32x2{lo[1], hi[1]});
}

// sum over the sixteen rows of u * v: products in pairs of rows, then a balanced tree over the
// eight pairs, whose upper levels are lanes when ROWS < 16
template <int ROWS>
__device__ __forceinline__ double dot16(const double (&u)[ROWS], const double (&v)[ROWS]) {
  double s[ROWS / 2];
#pragma unroll
  for (int i = 0; i < ROWS / 2; ++i) s[i] = fma(u[2 * i + 1], v[2 * i + 1], u[2 * i] * v[2 * i]);
#pragma unroll
  for (int n = ROWS / 4; n >= 1; n >>= 1)
#pragma unroll
    for (int i = 0; i < n; ++i) s[i] = s[2 * i] + s[2 * i + 1];
  double r = s[0];
  if (ROWS <= 8) r += dpp_d<kDppXor8>(r);
  if (ROWS <= 4) r = add_xor16(r);
  if (ROWS <= 2) r = add_xor32(r);
  return r;
}

constexpr int kMostSweeps = 24;

// Make a pair's columns orthogonal.  tan of the angle is 2 x.y over d + sign(d) sqrt(d^2 + (2 x.y)^2)
// with d the difference of the squared norms a, b; hardware estimates (about 1e-7) do for it: what is
// left of x.y shrinks by that factor and the next sweep deals with it.  cos gets a Newton step, so that
// rotations stay orthogonal to 1e-14.  The tiny addend keeps a pair of zero columns (0 / 0) from
// producing a NaN and is far below any pair that matters.  TEST: report whether the pair was
// still apart (the first sweeps do not ask); `floor`: squared norm below which that does not matter.
template <int ROWS, bool TEST>
__device__ __forceinline__ void rotate_pair(double (&x)[ROWS], double (&y)[ROWS], double& a, double& b, double floor, bool& unsettled) {
  const double g = dot16<ROWS>(x, y);
  if (TEST) unsettled |= (g * g > kSettled2 * (a * b)) & (a > floor) & (b > floor);
  const double d = b - a, g2 = g + g;
  const double root = __builtin_amdgcn_sqrt(fma(g2, g2, fma(d, d, 1e-240)));
  const double t = g2 * __builtin_amdgcn_rcp(d + copysign(root, d));
  const double w = fma(t, t, 1.0);
  const double r0 = __builtin_amdgcn_rsq(w);
  const double c = r0 * fma(-0.5 * w, r0 * r0, 1.5);
  const double tc = t * c;
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    const double xi = x[i], yi = y[i];
    x[i] = fma(-tc, yi, c * xi);
    y[i] = fma(tc, xi, c * yi);
  }
  a = fma(-t, g, a);
  b = fma(t, g, b);
}

// The sum over the eight places of a column pair (DPP lanes 0..7 of each eight).
__device__ __forceinline__ double over_eight(double v) {
  v += dpp_d<kDppXor1>(v);
  v += dpp_d<kDppXor2>(v);
  return v + dpp_d<kDppXor7>(v);
}

// a, or b where the lane's bit of `mask` is set.  The select that names VCC takes 9.5 ns where several follow each other (1.85 in
// the form with a pair of scalar registers, which the compiler gives up for the shorter one wherever it can).
__device__ __forceinline__ int select_i(unsigned long long mask, int a, int b) {
  int r;
  // (the mask is a constant; said so that a build without optimization has it in scalar registers, too)
  asm("v_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b),
      "s"((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(mask >> 32)) << 32 |
          (unsigned)__builtin_amdgcn_readfirstlane((int)mask)));
  return r;
}
__device__ __forceinline__ double select_d(unsigned long long mask, double a, double b) {
  const u32x2 u = __builtin_bit_cast(u32x2, a), v = __builtin_bit_cast(u32x2, b);
  return __builtin_bit_cast(double, u32x2{(unsigned)select_i(mask, (int)u.x, (int)v.x), (unsigned)select_i(mask, (int)u.y, (int)v.y)});
}

template <int ROWS>
struct Jacobi16 {
  double x[ROWS], y[ROWS];   // the lane's rows of its two columns
  double a, b;               // their squared norms
  int ix, iy;                // what they are ranked by: where they end up or (a pair of heads) where they began, which tells the head

  template <int CTRL, bool PAIR>
  __device__ __forceinline__ void move() {   // the y columns to lane ^ mask
#pragma unroll
    for (int i = 0; i < ROWS; ++i) y[i] = dpp_d<CTRL>(y[i]);
    b = dpp_d<CTRL>(b);
    if (PAIR) iy = __builtin_amdgcn_update_dpp(0, iy, CTRL, 0xF, 0xF, true);
  }
  // The lanes whose bit of `upper` is not set collect the x columns of both partners (lane, lane ^ mask), the
  // others the y columns.
  template <int CTRL, bool PAIR>
  __device__ __forceinline__ void split(unsigned long long upper) {
    auto cross = [&](double& u, double& v) __attribute__((always_inline)) {
      const double uo = dpp_d<CTRL>(u), vo = dpp_d<CTRL>(v);
      u = select_d(upper, u, vo);
      v = select_d(upper, uo, v);
    };
#pragma unroll
    for (int i = 0; i < ROWS; ++i) cross(x[i], y[i]);
    cross(a, b);
    if (PAIR) {
      const int ixo = __builtin_amdgcn_update_dpp(0, ix, CTRL, 0xF, 0xF, true);
      const int iyo = __builtin_amdgcn_update_dpp(0, iy, CTRL, 0xF, 0xF, true);
      ix = select_i(upper, ix, iyo);
      iy = select_i(upper, ixo, iy);
    }
  }

  // PAIR: the floor of the columns' own head counts (two columns of different heads have no row in common: their
  // product is zero and nothing is to settle).
  template <bool TEST, bool PAIR>
  __device__ __forceinline__ void rotate(double floor_lo, double floor_hi, bool& unsettled) {
    rotate_pair<ROWS, TEST>(x, y, a, b, (PAIR && ix >= 8) ? floor_hi : floor_lo, unsettled);
  }

  // Fifteen rounds of eight disjoint pairs: x columns against y columns, then the two halves of each
  // among themselves, and so on; every exchange is one data-parallel-primitive pattern.  Of the orders
  // that leave the columns where the next sweep can start from them, this one converges soonest (5.9
  // sweeps on the synthetic workloads' blocks; with the first eight rounds the other way round, 6.9).
  template <bool TEST, bool PAIR>
  __device__ __forceinline__ void sweep(double floor_lo, double floor_hi, bool& unsettled) {
    move<kDppXor7, PAIR>(); rotate<TEST, PAIR>(floor_lo, floor_hi, unsettled);
    move<kDppXor3, PAIR>(); rotate<TEST, PAIR>(floor_lo, floor_hi, unsettled);
    move<kDppXor1, PAIR>(); rotate<TEST, PAIR>(floor_lo, floor_hi, unsettled);
    move<kDppXor3, PAIR>(); rotate<TEST, PAIR>(floor_lo, floor_hi, unsettled);
    move<kDppXor7, PAIR>(); rotate<TEST, PAIR>(floor_lo, floor_hi, unsettled);
    move<kDppXor3, PAIR>(); rotate<TEST, PAIR>(floor_lo, floor_hi, unsettled);
    move<kDppXor1, PAIR>(); rotate<TEST, PAIR>(floor_lo, floor_hi, unsettled);
    move<kDppXor3, PAIR>(); rotate<TEST, PAIR>(floor_lo, floor_hi, unsettled);
    split<kDppXor7, PAIR>(0xF0F0F0F0F0F0F0F0ull); rotate<TEST, PAIR>(floor_lo, floor_hi, unsettled);
    move<kDppXor1, PAIR>(); rotate<TEST, PAIR>(floor_lo, floor_hi, unsettled);
    move<kDppXor2, PAIR>(); rotate<TEST, PAIR>(floor_lo, floor_hi, unsettled);
    move<kDppXor1, PAIR>(); rotate<TEST, PAIR>(floor_lo, floor_hi, unsettled);
    split<kDppXor3, PAIR>(0xCCCCCCCCCCCCCCCCull); move<kDppXor1, PAIR>(); rotate<TEST, PAIR>(floor_lo, floor_hi, unsettled);
    move<kDppXor1, PAIR>(); rotate<TEST, PAIR>(floor_lo, floor_hi, unsettled);
    split<kDppXor1, PAIR>(0xAAAAAAAAAAAAAAAAull); rotate<TEST, PAIR>(floor_lo, floor_hi, unsettled);
  }

  // Called with x = column j, y = column j + 8 of the matrix, j = lane % 8.  Returns the sweeps used.  All
  // eight lanes of a block (and, for ROWS < 16, all its row groups) leave together.
  template <bool PAIR>
  __device__ __forceinline__ int run() {
    const int lane = threadIdx.x & 63, j = lane & 7;
    ix = j; iy = j + 8;
    a = dot16<ROWS>(x, x);
    b = dot16<ROWS>(y, y);
    // columns of eigenvalues below 1e-14 of the largest are dropped later: whether they have settled
    // does not matter.  (A pair: of the largest of the same head, as order() drops them.  x are the first
    // head's columns here, y the second's.  One floor over both left a head a thousand times smaller
    // than its partner unsettled: up to 88 % of its block lost where its singular values span 1e5.)
    const double floor_lo = over_eight(PAIR ? a : a + b) * 1e-28, floor_hi = PAIR ? over_eight(b) * 1e-28 : 0.0;
    bool unsettled = true;
    int sweeps = 0;
    // no block with anything off the diagonal settles in three sweeps: they do not test
    while (sweeps < 3) {
      ++sweeps;
      sweep<false, PAIR>(floor_lo, floor_hi, unsettled);
      a = dot16<ROWS>(x, x);
      b = dot16<ROWS>(y, y);
    }
    // (blocks in general position settle in 6, graded ones in up to 17: five decades and a half)
    while (unsettled && sweeps < kMostSweeps) {
      ++sweeps;
      unsettled = false;
      sweep<true, PAIR>(floor_lo, floor_hi, unsettled);
      a = dot16<ROWS>(x, x);
      b = dot16<ROWS>(y, y);
      // every pair of this sweep was within 3e-5 of orthogonal when it was rotated, so the sweep (one
      // more quadratic step) has left them near 1e-9, two orders under the fp32 rounding of T_L
      const unsigned long long open = __ballot(unsettled);
      if (ROWS == 2) {
        unsettled = open != 0;
      } else {
        constexpr int LPB = 128 / (ROWS == 2 ? 4 : ROWS);   // lanes per block
        unsettled = ((open >> (lane & ~(LPB - 1))) & ((1ull << LPB) - 1)) != 0;
      }
    }
    return sweeps;
  }

  // The columns' places in descending order of eigenvalue, and the factors of the two results: column
  // times rx (ry) is the column of T_S = U Sigma, times rx^3 the row of W = Sigma^-1 U^T; 0 if the
  // direction is dropped.  `lam`: sixteen doubles of LDS of this block.  PAIR: the columns of each half
  // are ranked among themselves.
  template <bool PAIR>
  __device__ __forceinline__ void order(double* lam, int& px, int& py, double& rx, double& ry, double& lx, double& ly) {
    const int lane = threadIdx.x & 63;
    lx = a > 0.0 ? a * fast_rsqrt(a) : a;   // (a NaN stays one)
    ly = b > 0.0 ? b * fast_rsqrt(b) : b;
    lam[ix] = lx;
    lam[iy] = ly;
    __builtin_amdgcn_wave_barrier();
    int places = 0;                        // of x in the low half, of y in the high half
    double mx = 0.0, my = 0.0;
    const int row0 = first_row(lane);
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {       // the lane's share of the sixteen columns
      const int s = row0 + i;
      const double o = lam[s];
      const bool sx = !PAIR || (s >> 3) == (ix >> 3), sy = !PAIR || (s >> 3) == (iy >> 3);
      places += (sx & ((o > lx) | ((o == lx) & (s < ix)))) ? 1 : 0;
      places += (sy & ((o > ly) | ((o == ly) & (s < iy)))) ? 0x10000 : 0;
      mx = sx ? fmax(mx, o) : mx;
      if (PAIR) my = sy ? fmax(my, o) : my;
    }
    if (ROWS <= 8) {
      places += __builtin_amdgcn_update_dpp(0, places, kDppXor8, 0xF, 0xF, true);
      mx = fmax(mx, dpp_d<kDppXor8>(mx));
      if (PAIR) my = fmax(my, dpp_d<kDppXor8>(my));
    }
#pragma unroll
    for (int o = 16; o < 128 / ROWS; o <<= 1) {
      places += __shfl_xor(places, o);
      mx = fmax(mx, __shfl_xor(mx, o));
      if (PAIR) my = fmax(my, __shfl_xor(my, o));
    }
    if (!PAIR) my = mx;
    px = (places & 0xFFFF) + (PAIR ? (ix & 8) : 0);
    py = (places >> 16) + (PAIR ? (iy & 8) : 0);
    const bool kx = (lx > 1e-12 * mx) & (lx > 0.0), ky = (ly > 1e-12 * my) & (ly > 0.0);
    rx = kx ? fast_rsqrt(lx) : 0.0;
    ry = ky ? fast_rsqrt(ly) : 0.0;
    if (!kx) lx = 0.0;
    if (!ky) ly = 0.0;
  }
  static __device__ __forceinline__ int first_row(int lane) { return ROWS == 16 ? 0 : ROWS * ((lane >> 3) & (16 / ROWS - 1)); }
};

// W[r][b1] from the solver's registers (lam2[r]: the eigenvalue, 0 if the direction is dropped)
template <int ROWS, bool PAIR, int LD>
__device__ __forceinline__ void store_factors(Jacobi16<ROWS>& jac, double* lam, double* lam2, double* W) {
  int px, py;
  double rx, ry, lx, ly;
  jac.template order<PAIR>(lam, px, py, rx, ry, lx, ly);
  const int row0 = jac.first_row(threadIdx.x & 63);
  lam2[px] = lx;
  lam2[py] = ly;
  const double fx = rx * rx * rx, fy = ry * ry * ry;
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    W[px * LD + row0 + i] = rx > 0.0 ? jac.x[i] * fx : 0.0;
    W[py * LD + row0 + i] = ry > 0.0 ? jac.y[i] * fy : 0.0;
  }
  __builtin_amdgcn_wave_barrier();
}

// ------------------------------------------------------------------------------------------
// Projection and quantizer on the fp16 matrix cores, for 2- and 4-bit codes of two local tensors.
//
// The codes and steps are those of the fp64 projection, bit for bit, but few tokens need it: a first pass
// projects on fp16 matrix instructions (the rows are fp16 as they are, W is cut into two fp16 pieces, 22
// bits; fp32 accumulation) with an error bound that is derived from a measured model of the instruction, and a token with a step or a code within that bound
// of a rounding boundary is in doubt.  Those of a group of sixteen go through the fp64 projection
// itself at once, two at a time, their 2 x 8 columns side by side in one product, from the rows that lie in LDS (a block whose
// bound is wide goes there as a whole).  DIRECT builds keep no rows in LDS: they list the tokens in doubt of a tile and fetch
// them again behind its first pass.
// A 16 x 16 x 16 product takes one matrix instruction of 16 cycles (16x16x32: both pieces side by side), instead of four fp64 ones of
// 64 cycles each, and no fp16 value is widened.  14720 blocks with outlier channels (4-bit, d = 128): 280 us all in fp64; 192 with
// three pieces in three instructions and the rows in the matrix cores' order, 146 with them in memory order; one instruction instead
// of three leaves that as it is (fewer cycles, but a wider bound: without the tokens in doubt 139 and 134); 139 since
// they are settled from LDS, without a round trip to memory.  Rows from cache instead of memory: 118,
// so what is left is both, 670 MB and the instructions.
//
// Keys (W as the left operand): lane (token n = l % 16, g = l / 16) gets rows r = 4 g + i of its token, eight
// b2 each, i.e. whole words of the key layout, which it stores as they are.  Values (operands
// swapped): lane (row r = n, g) gets tokens 4 g + i of a group of sixteen; its four codes of one b2 are
// neighbours in the value layout and go through LDS once, 8 or 16 bits at a time, to be stored in rows.
// In both a lane's elements belong to one step group per token (rows r < 8, r >= 8).
//
// Error bound.  T[r] = sum_b1 W[r, b1] X[b1] of a token and a b2, S = sum |W X|, amax = the token's largest |T|.
//  - A 16x16x32 fp16 matrix instruction adds its products in four groups of eight (those of a lane): each product is cut to 24
//    bits below the group's largest exponent E (an fp16 subnormal counts with exponent -14); the sum is added to
//    the accumulator, which is cut there as well, 28 bits below the accumulator's exponent, and rounded to fp32 (found by
//    comparing with that model over random and adversarial operands: 98 to 99 of 100 results are its own, the others differ by
//    one unit in the last place).  The largest product of a group loses nothing, seven others and the accumulator at most 2^(E - 24)
//    each, so the groups' cuts come to 8 * 2^-24 S.  Each of the four additions may round by one unit, 2^-23 of its
//    result: three of them are within S, the last is the result itself.  In all 14.2 * 2^-24 S + 2 * 2^-24 amax: kRoundings = 14.5
//    (the largest error seen is 7.2 * 2^-24 S; test_gpu_mfma_f16.py holds the
//    instruction to the 14.2 and 2 on operands that strain them).  A subnormal X adds at most 32 * 2^-24 * 2^-14 max |W[r]|.
//  - The pieces leave out what is known exactly when they are cut (`left`): 2^-23 of an element at the most, a tenth of the above.
//  - S <= C amax + sum |W[r]| d.  X = T_S T + what directions that were dropped carry, so |X[b1]| <= s[b1] amax + d,
//    s[b1] = sum_r |T_S[b1, r]|, d <= sqrt(15e-12 lambda_max) (0 if none was dropped): C = sum |W[r, b1]| s[b1];
//    and by Cauchy and Schwarz C = |W[r]| sqrt(sum lambda) as well.
//  - The value that is quantized is the fp64 sum rounded to fp32, and the comparisons round, too: 4 * 2^-24 amax, 6 with the above.
// So |error| <= eps amax + eps_abs with the block's constants eps, eps_abs.  With three pieces, under a
// bound of 12 C + 4 instead of 14.5 C + 6, 3 to 5 of a tile's 128 tokens were in doubt with one step per token on a synthetic
// prompt, 8 to 10 with two.
// ------------------------------------------------------------------------------------------
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr float kRoundings = 14.5f;
// eps beyond which a block skips the first pass: about half of its tokens would be listed
constexpr float kHardEps = 0x1p-13f;
// Where a block's constants lie, in doubles from its Gram matrix on (behind G, W and the eigenvalues): the pieces of W,
// then floats.
constexpr int kFastPieces = 2 * 256 + 16, kFastScales = kFastPieces + 2 * 64;

__device__ __forceinline__ float max_xor16(float v) {
  const uint32_t w = __builtin_bit_cast(uint32_t, v);
  const auto x = __builtin_amdgcn_permlane16_swap(w, w, false, false);
  return fmaxf(__builtin_bit_cast(float, (uint32_t)x[0]), __builtin_bit_cast(float, (uint32_t)x[1]));
}
__device__ __forceinline__ float max_xor32(float v) {
  const uint32_t w = __builtin_bit_cast(uint32_t, v);
  const auto x = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return fmaxf(__builtin_bit_cast(float, (uint32_t)x[0]), __builtin_bit_cast(float, (uint32_t)x[1]));
}

// Between steps of NWV waves that share LDS; NWV = 1: of one wave on its own, whose LDS operations execute in order.
template <int NWV>
__device__ __forceinline__ void team_barrier() {
  if (NWV > 1) {
    __syncthreads();
  } else {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

template <int QB, bool FULL, bool PAIR, bool DIRECT>
struct FastProject {
  static constexpr int QMAX = (1 << (QB - 1)) - 1, QMIN = FULL ? -QMAX - 1 : -QMAX, BIAS = 1 << (QB - 1);
  static constexpr float kBase = 128.f + (float)BIAS + 0.5f;   // between 128 and 256 a float's low sixteen bits are its fraction, the next byte the integer
  static constexpr int ROWB = 16 * QB, STRIDE = ROWB + 4;     // bytes of a value row of a tile, and of its place in LDS
  static constexpr int kStageBytes = 128 * STRIDE, kRowBytes = DIRECT ? 0 : 16 * 256;

  f16x8 w;           // row r = l % 16 of W, columns b1 = 4 j + l / 16, scaled by 2^(15 - e): four upper pieces, four lower ones
  float sc;          // 2^(e - 15) of row l % 16
  float sck[4];      // ... of rows 4 (l / 16) + i
  float eps, eps_abs;   // the error bound (see above)
  const double* W64; // [16][16], in the workspace
  const uint16_t* X; // the block's rows
  int nv;
  long head_gap;
  bool one_group;
  bool hard;         // the first pass is not worth its while

  // X[t][b1 * 8 + b2], the 16-byte piece of one b1
  __device__ __forceinline__ const uint16_t* piece(int t, int b1) const {
    return PAIR ? X + (b1 >> 3) * head_gap + (long)t * 64 + (b1 & 7) * 8 : X + (long)t * 128 + b1 * 8;
  }
  // Sixteen tokens' rows, as they lie in memory: lane l gets piece b1 = l % 16 of token t0 + 4 u + l / 16 (past the last valid
  // row: that row again; the caller clears it).  What bounds a prompt's projection is memory: without its quantizer it
  // takes the same time.  Requested in the matrix cores' order, lanes 256 bytes apart, the rows took four times the
  // accesses to the first-level cache, and each of its lines was asked for four times; in memory order no line is,
  // so that they can pass the caches by.  14720 blocks, steady clocks: 179 us in the other order (215 non-temporal),
  // 172 so, 148 non-temporal; two groups ahead instead of one 161.
  // DIRECT: in the matrix cores' order all the same, pieces b1 = 4 j + l / 16 of token t0 + l % 16.
  __device__ __forceinline__ void load(u32x4 (&x)[4], int t0) const {
    int l = threadIdx.x & 63;
    if (DIRECT && PAIR) asm volatile("" : "+v"(l));   // (the pieces' places, kept from call to call, would be a spill)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (DIRECT) x[u] = *reinterpret_cast<const u32x4*>(piece(min(t0 + (l & 15), nv - 1), 4 * u + (l >> 4)));
      else x[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(piece(min(t0 + 4 * u + (l >> 4), nv - 1), l & 15)));
    }
  }
  // ... those of tokens past the last valid one are zero
  __device__ __forceinline__ void clear(u32x4 (&x)[4], int t0) const {
    if (t0 + 16 <= nv) return;
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (t0 + (DIRECT ? l & 15 : 4 * u + (l >> 4)) >= nv) x[u] = u32x4{0u, 0u, 0u, 0u};
  }
  // ... and through LDS (kRowBytes) into the matrix cores' order: lane (n = l % 16, g = l / 16) gets pieces b1 = 4 j + g
  // of token n.  Piece b1 of token n lies at place b1 ^ n of its row, so that neither side meets a bank twice.
  static __device__ __forceinline__ void turn(u32x4 (&x)[4], uint8_t* rows) {
    const int l = threadIdx.x & 63, n = l & 15, g = l >> 4;
#pragma unroll
    for (int u = 0; u < 4; ++u) *reinterpret_cast<u32x4*>(rows + (4 * u + g) * 256 + ((n ^ (4 * u + g)) * 16)) = x[u];
    team_barrier<1>();
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = *reinterpret_cast<const u32x4*>(rows + n * 256 + (((4 * j + g) ^ n) * 16));
    team_barrier<1>();
  }

  static __device__ __forceinline__ float max8(float v) {      // over eight lanes
    v = fmaxf(v, lane_exchange<0xB1>(v));
    v = fmaxf(v, lane_exchange<0x4E>(v));
    v = fmaxf(v, lane_exchange<0x141>(v));
    return v;
  }

  // (what store_fast_factors left)
  __device__ __forceinline__ void setup(const double* G) {
    W64 = G + 256;
    const uint16_t* const pieces = reinterpret_cast<const uint16_t*>(G + kFastPieces);
    const float* const scales = reinterpret_cast<const float*>(G + kFastScales);
    const int l = threadIdx.x & 63, r = l & 15, g = l >> 4;
    w = *reinterpret_cast<const f16x8*>(pieces + (g * 16 + r) * 8);
    sc = scales[r];
    const f32x4 s4 = *reinterpret_cast<const f32x4*>(scales + 4 * g);
#pragma unroll
    for (int i = 0; i < 4; ++i) sck[i] = s4[i];
    eps = scales[16];
    eps_abs = scales[17];
    hard = scales[18] != 0.f;
  }

  __device__ __forceinline__ static uint16_t step_bits(float up, float dn) {
    uint16_t s = group_step_bits<QMAX>(up);
    if (FULL) {
      const uint16_t down = f2h_rne(dn * (1.0f / (float)(QMAX + 1)));
      s = s > down ? s : down;
    }
    return s;
  }

  template <bool VALUES>
  __device__ __forceinline__ void project(const u32x4 (&x)[4], f32x4 (&acc)[8]) const {
    f16x8 h[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) h[j] = __builtin_bit_cast(f16x8, x[j]);
#pragma unroll
    for (int b2 = 0; b2 < 8; ++b2) {
      // (slots 0 to 3 of a lane's eight meet the upper pieces of W, slots 4 to 7, the same values, the lower ones)
      const f16x8 x8 = {h[0][b2], h[1][b2], h[2][b2], h[3][b2], h[0][b2], h[1][b2], h[2][b2], h[3][b2]};
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      acc[b2] = VALUES ? __builtin_amdgcn_mfma_f32_16x16x32_f16(x8, w, zero, 0, 0, 0) : __builtin_amdgcn_mfma_f32_16x16x32_f16(w, x8, zero, 0, 0, 0);
    }
  }

  // Largest value over a step group.  Keys: over the lanes of a token (16 and, for one group, 32 apart);
  // values: over the rows of a token (within 8 and, for one group, 16 lanes).
  template <bool VALUES>
  __device__ __forceinline__ float group_max(float v, bool both) const {
    if (VALUES) {
      v = max8(v);
      if (both) v = fmaxf(v, lane_exchange<0x140>(v));
    } else {
      v = max_xor16(v);
      if (both) v = max_xor32(v);
    }
    return v;
  }

  // Fields of NT = 1 (keys) or 4 (values) tokens of the lane: element (i, b2) belongs to row 4 g + i of token
  // n of the sixteen, or to row n of token 4 g + i.  Steps come back in `sbits` (values: of token 4 g + n % 4), the
  // fields, QB bits each, in `part`: keys: element 8 i + b2 in index order (part[i]: eight of them);
  // values: part[b2]: the four tokens.  Returns the tokens that are in doubt, one bit each, the same in all lanes.
  template <bool VALUES>
  __device__ __forceinline__ uint32_t quantize(const f32x4 (&acc)[8], uint16_t& sbits, uint32_t (&part)[VALUES ? 8 : 4]) const {
    const int l = threadIdx.x & 63, n = l & 15;
    constexpr int NT = VALUES ? 4 : 1;
    auto scale = [&](int i) -> float { return VALUES ? sc : sck[i]; };
    // ---- largest values per token and group, and the step ----
    float up[NT], dn[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) { up[k] = 0.f; dn[k] = 0.f; }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float u = 0.f, m = 0.f;
#pragma unroll
      for (int b2 = 0; b2 < 8; ++b2) {
        u = fmaxf(u, FULL ? acc[b2][i] : fabsf(acc[b2][i]));
        if (FULL) m = fmaxf(m, -acc[b2][i]);
      }
      up[VALUES ? i : 0] = fmaxf(up[VALUES ? i : 0], u * scale(i));
      if (FULL) dn[VALUES ? i : 0] = fmaxf(dn[VALUES ? i : 0], m * scale(i));
    }
    float all[NT];   // of both groups: what the error bound refers to (a pair: of the head alone)
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      up[k] = group_max<VALUES>(up[k], one_group);
      if (FULL) dn[k] = group_max<VALUES>(dn[k], one_group);
      all[k] = FULL ? fmaxf(up[k], dn[k]) : up[k];
      if (!PAIR && !one_group) all[k] = VALUES ? fmaxf(all[k], lane_exchange<0x140>(all[k])) : max_xor32(all[k]);
    }
    // values: the lane's quad shares the four tokens, lane n % 4 = i settles token i
    float my_up = up[0], my_dn = dn[0], my_all = all[0];
    if (VALUES) {
#pragma unroll
      for (int k = 1; k < NT; ++k) {
        my_up = (n & 3) == k ? up[k] : my_up;
        my_dn = (n & 3) == k ? dn[k] : my_dn;
        my_all = (n & 3) == k ? all[k] : my_all;
      }
    }
    const float err = fmaf(eps, my_all, eps_abs);
    // The step of the exact sums lies between those of the ends of the interval: the quotients' own rounding widens
    // it by 2^-22 (an exact division costs twenty instructions); a tie or a step that depends on it is in doubt.
    constexpr float kDown = QMAX == 1 ? 1.f : (1.f - 0x1p-22f) / QMAX, kUp = QMAX == 1 ? 1.f : (1.f + 0x1p-22f) / QMAX;
    float hi = (my_up + err) * kUp, lo = (my_up - err) * kDown;
    if (FULL) {
      hi = fmaxf(hi, (my_dn + err) * (1.f / (QMAX + 1)));
      lo = fmaxf(lo, (my_dn - err) * (1.f / (QMAX + 1)));
    }
    sbits = f2h_rne(hi);
    const bool doubt = sbits != f2h_rne(fmaxf(lo, 0.f));
    const float my_step = h2f(sbits);
    const float my_inv = my_step > 0.f ? __builtin_amdgcn_rcpf(my_step) : 0.f;
    // A quotient further than this from a half-integer is on the right side of it: the bound above, the
    // reciprocal's error and the rounding of the product.  In units of 2^-16, with one for the rounding below.
    const float my_margin = err * my_inv + (float)(QMAX + 1) * 0x1p-21f;
    const float my_base = fmaf((float)((int)(fminf(my_margin, 0.25f) * 0x1p16f) + 2), 0x1p-16f, kBase);   // (exact)
    // the step of a group of subnormal size may be rounded so far down that a quotient leaves the range
    // (FULL: whose negative end has one more code)
    const bool wide = ((FULL ? fmaxf(my_up, my_dn - my_step) : my_up) * my_inv > (float)QMAX + 0.25f) | !(my_margin < 0.2f);
    float inv[NT], base[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      if (!VALUES) {
        inv[k] = my_inv;
        base[k] = my_base;
      } else if (k == 0) {
        inv[k] = lane_exchange<0x00>(my_inv);
        base[k] = lane_exchange<0x00>(my_base);
      } else if (k == 1) {
        inv[k] = lane_exchange<0x55>(my_inv);
        base[k] = lane_exchange<0x55>(my_base);
      } else if (k == 2) {
        inv[k] = lane_exchange<0xAA>(my_inv);
        base[k] = lane_exchange<0xAA>(my_base);
      } else {
        inv[k] = lane_exchange<0xFF>(my_inv);
        base[k] = lane_exchange<0xFF>(my_base);
      }
    }
    // ---- fields: quotient + base has the code + BIAS as its integer, in one byte of the float, unless the fraction is less than
    // twice the margin.  An element costs an addition, a 16-bit minimum (half the price of the other kinds) and 0.75 of a
    // byte permutation; a magic number for the code, the distance from it and its maximum cost 1.7 times that: whole call of
    // 14720 blocks 318.4 us, 313.4 so. ----
    // bit i: token 4 g + i is in doubt (keys: bit 0)
    uint32_t near = wide ? (VALUES ? 15u : 1u) : doubt ? (VALUES ? 1u << (n & 3) : 1u) : 0u;
    uint32_t t[4][8], least[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) least[k] = 0xFFFFu;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float f = inv[VALUES ? i : 0] * scale(i);
#pragma unroll
      for (int b2 = 0; b2 < 8; ++b2) {
        t[i][b2] = __builtin_bit_cast(uint32_t, fmaf(acc[b2][i], f, base[VALUES ? i : 0]));
        asm("v_min_u16 %0, %0, %1" : "+v"(least[VALUES ? i : 0]) : "v"(t[i][b2]));
      }
    }
#pragma unroll
    for (int k = 0; k < NT; ++k)   // (the fraction of `base` is a half and the margin)
      near |= (uint16_t)least[k] < (uint16_t)(__builtin_bit_cast(uint32_t, base[k]) << 1) ? 1u << k : 0u;
    // the integers of a and b (bytes 0 and 1; with `high`: 2 and 3)
    auto two = [](uint32_t a, uint32_t b, bool high = false) __attribute__((always_inline)) {
      return __builtin_amdgcn_perm(b, a, high ? 0x06020C0Cu : 0x0C0C0602u);
    };
    if (VALUES) {
#pragma unroll
      for (int b2 = 0; b2 < 8; ++b2) {
        const uint32_t w = (two(t[1][b2], t[3][b2]) << QB) | two(t[0][b2], t[2][b2]);
        part[b2] = QB == 4 ? w : (w >> 4) | w;   // (the lowest 4 QB bits count)
      }
    } else {
#pragma unroll
      for (int i = 0; i < (VALUES ? 1 : 4); ++i) {
        if (QB == 4)
          part[i] = ((two(t[i][1], t[i][3]) | two(t[i][5], t[i][7], true)) << 4) | (two(t[i][0], t[i][2]) | two(t[i][4], t[i][6], true));
        else
          part[i] = (((two(t[i][3], t[i][7]) << 2 | two(t[i][2], t[i][6])) << 2 | two(t[i][1], t[i][5])) << 2) | two(t[i][0], t[i][4]);
      }
    }
    const unsigned long long any = __ballot(near != 0);
    if (any == 0) return 0;
    if (!VALUES) return (uint32_t)(any | (any >> 16) | (any >> 32) | (any >> 48)) & 0xFFFFu;
    near |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)near, 0xB1, 0xF, 0xF, true);
    near |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)near, 0x4E, 0xF, 0xF, true);
    near |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)near, 0x141, 0xF, 0xF, true);
    near |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)near, 0x140, 0xF, 0xF, true);
    return (uint32_t)__builtin_amdgcn_readlane((int)near, 0) | (uint32_t)__builtin_amdgcn_readlane((int)near, 16) << 4 |
           (uint32_t)__builtin_amdgcn_readlane((int)near, 32) << 8 | (uint32_t)__builtin_amdgcn_readlane((int)near, 48) << 12;
  }

  // ---- second pass: two tokens at a time through the fp64 projection, all their 2 x 8 columns side by side in
  // one product.  The sums, their order and so every bit are those of the build that keeps the fp32 rows.
  // Lane (n = l % 16, g = l / 16): token n / 8 of the two, b2 = n % 8, rows r = 4 g + i (the rows of W are dealt so).
  __device__ __forceinline__ void load_factor(double (&w)[4], int l) const {
    const int n = l & 15, g = l >> 4;
#pragma unroll
    for (int s = 0; s < 4; ++s) w[s] = W64[(4 * (n & 3) + (n >> 2)) * 16 + 4 * s + g];
  }
  // x[s]: the lane's token's X[b1 = 4 s + g][b2] (t < 0: none)
  __device__ __forceinline__ void load_column(uint16_t (&x)[4], int t, int l) const {
    const int g = l >> 4;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      x[s] = 0;
      if (t >= 0 && t < nv) x[s] = piece(t, 4 * s + g)[l & 7];
    }
  }
  // ... of token n of the sixteen whose rows `turn` left in LDS
  static __device__ __forceinline__ void row_column(uint16_t (&x)[4], int n, const uint8_t* rows) {
    const int l = threadIdx.x & 63, g = l >> 4;
#pragma unroll
    for (int s = 0; s < 4; ++s) x[s] = *reinterpret_cast<const uint16_t*>(rows + n * 256 + (((4 * s + g) ^ n) * 16) + (l & 7) * 2);
  }
  // The fields of the lane's four rows, a byte each, and the step of the group that holds them.
  __device__ __forceinline__ uint32_t settle(const double (&w)[4], const uint16_t (&x)[4], uint16_t& sbits) const {
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(w[s], (double)h2f(x[s]), acc, 0, 0, 0);
    float f[4], up = 0.f, dn = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[i] = (float)acc[i];
      up = fmaxf(up, FULL ? f[i] : fabsf(f[i]));
      if (FULL) dn = fmaxf(dn, -f[i]);
    }
    up = group_max<false>(max8(up), one_group);   // (the token's eight b2, then its rows)
    if (FULL) dn = group_max<false>(max8(dn), one_group);
    sbits = step_bits(up, dn);
    const float step = h2f(sbits), inv = step > 0.f ? __builtin_amdgcn_rcpf(step) : 0.f;
    return fields_of_four<QB, FULL>(f[0], f[1], f[2], f[3], step, inv);
  }
};

// Gram matrix of a block's sixteen rows b1 (1024 columns (t, b2) each at 128 tokens), NWV waves, wave wv
// taking every NWV-th group of four tokens: lane (b1 = l % 16, k = l / 16) loads the 8 b2 of token k of a group
// as one 16-byte piece; 16 lanes cover a 256-byte row.
//
// The sums are exact integers: an fp16 value is a multiple of 2^-24, and x * 2^24 = 254 * 2^24 * d4 + v with v a
// 32-bit integer, |v| <= 127.5 * 2^24.  v is cut into four signed digits d0..d3 of eight bits; d4 is zero
// unless |x| >= 127.5, which a step of eight tokens asks of all its elements at once (one step in ten on prompts
// with outlier channels).  A digit of the lane's sixteen elements is one operand of the int8 matrix cores; of the
// sixteen products of digits ten are formed (the others are their transposes), those of one weight in
// one accumulator: at most 2^18 a token (eight columns, two products of 2^14), and 32 bits would wrap from 8192 tokens a
// wave on, so every kDrainTokens tokens of a wave the accumulators are added to two doubles an entry in LDS, a low
// and a high half.  Tokens add less than 1.04 * 2^42 each to the low half of an entry and of its transpose together, in
// halves of one: 256 of them stay far under 2^52, and what goes beyond 2^32 is carried to the high half (2^32 a token,
// in halves: 2^20 tokens) before more is added.  The halves are therefore exact, are joined and rounded
// once, and G does not depend on the number of waves or the order of the sums, whatever the size of the block (a sum of
// squares beyond 2^30 whose rows hold values of 127.5 and more has more bits than the high half holds: it takes up to
// three roundings more each time the accumulators are drained).  A block that holds values
// beyond kMostDigits (infinities and NaN among them) takes the fp64 matrix instructions below, whose sums round, in an
// order that depends on the number of waves.
// Bound by vector instructions: six and a half an element, and 160 matrix instructions of 16 cycles a block, where
// the fp64 matrix cores take two an element and 256 of 64 cycles (and round their sums).
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
constexpr float kPlainMost = 127.4375f;   // the largest fp16 value below 127.5
constexpr float kMostDigits = 32256.f;
constexpr int kDrainTokens = 256;         // tokens a wave adds up in 32 bits (see above)

// The sums of products of digits: p[w]: digits i < j <= 3, total weight w + 1; e[i]: digit i with itself; f[i]: d4
// with digit i.
struct GramSums {
  i32x4 p[5], e[5], f[4];
  f16x2 most = {(_Float16)0.f, (_Float16)0.f};   // the largest |x| so far, of even and odd elements
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < 5; ++i) p[i] = e[i] = i32x4{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = i32x4{0, 0, 0, 0};
  }
  // four 32-bit integers -> their digits, a word of four elements each
  static __device__ __forceinline__ void cut(const int (&v)[4], int& q0, int& q1, int& q2, int& q3) {
    constexpr uint32_t kBias = 0x00808080u;   // every lower byte of v + kBias is a digit + 128, the top one a digit
    const uint32_t a = (uint32_t)v[0] + kBias, b = (uint32_t)v[1] + kBias, c = (uint32_t)v[2] + kBias, d = (uint32_t)v[3] + kBias;
    const uint32_t ab_lo = __builtin_amdgcn_perm(b, a, 0x05010400u), cd_lo = __builtin_amdgcn_perm(d, c, 0x05010400u);
    const uint32_t ab_hi = __builtin_amdgcn_perm(b, a, 0x07030602u), cd_hi = __builtin_amdgcn_perm(d, c, 0x07030602u);
    q0 = (int)(__builtin_amdgcn_perm(cd_lo, ab_lo, 0x05040100u) ^ 0x80808080u);
    q1 = (int)(__builtin_amdgcn_perm(cd_lo, ab_lo, 0x07060302u) ^ 0x80808080u);
    q2 = (int)(__builtin_amdgcn_perm(cd_hi, ab_hi, 0x05040100u) ^ 0x80808080u);
    q3 = (int)__builtin_amdgcn_perm(cd_hi, ab_hi, 0x07060302u);
  }
  // eight tokens: the lane's row's eight b2 of two of them
  __device__ __forceinline__ void add(const u32x4& v0, const u32x4& v1) {
    const u32x4 x[2] = {v0, v1};
    f16x2 m = {(_Float16)0.f, (_Float16)0.f};
#pragma unroll
    for (int i = 0; i < 8; ++i)   // largest of m, x, -x; a NaN stays
      asm("v_pk_maximum3_f16 %0, %0, %1, %1 neg_lo:[0,0,1] neg_hi:[0,0,1]" : "+v"(m) : "v"(x[i >> 2][i & 3]));
    asm("v_pk_maximum3_f16 %0, %0, %1, %1" : "+v"(most) : "v"(m));
    i32x4 q[4];   // digit i of the lane's sixteen elements
    const bool plain = (float)m.x <= kPlainMost && (float)m.y <= kPlainMost;
    if (__all(plain)) {
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        int v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          v[i] = (int)fmaf((float)__builtin_bit_cast(f16x2, (uint32_t)x[w >> 1][2 * (w & 1) + (i >> 1)])[i & 1], 0x1p24f, 0.f);
        int d0, d1, d2, d3;
        cut(v, d0, d1, d2, d3);
        q[0][w] = d0; q[1][w] = d1; q[2][w] = d2; q[3][w] = d3;
      }
    } else {
      i32x4 q4;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        int v[4];
        uint32_t top[4];   // d4 in the low byte
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          // all exact: where d4 is not zero, x is a multiple of 2^-4, and |x - 254 d4| <= 127
          constexpr float kRound = 12582912.f;   // 1.5 * 2^23: the nearest integer appears in the low bits
          const float h = fmaf((float)__builtin_bit_cast(f16x2, (uint32_t)x[w >> 1][2 * (w & 1) + (i >> 1)])[i & 1], 0x1p24f, 0.f);
          const float t = fmaf(h, 0x1p-24f / 254.f, kRound);
          v[i] = (int)fmaf(t - kRound, -254.f * 0x1p24f, h);
          top[i] = __builtin_bit_cast(uint32_t, t);
        }
        int d0, d1, d2, d3;
        cut(v, d0, d1, d2, d3);
        q[0][w] = d0; q[1][w] = d1; q[2][w] = d2; q[3][w] = d3;
        q4[w] = (int)__builtin_amdgcn_perm(__builtin_amdgcn_perm(top[3], top[2], 0x0C0C0400u),
                                           __builtin_amdgcn_perm(top[1], top[0], 0x0C0C0400u), 0x05040100u);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) f[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q4, q[i], f[i], 0, 0, 0);
      e[4] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q4, q4, e[4], 0, 0, 0);
    }
    p[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q[0], q[1], p[0], 0, 0, 0);
    p[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q[0], q[2], p[1], 0, 0, 0);
    p[2] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q[0], q[3], p[2], 0, 0, 0);
    p[3] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q[1], q[3], p[3], 0, 0, 0);
    p[4] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q[2], q[3], p[4], 0, 0, 0);
    e[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q[0], q[0], e[0], 0, 0, 0);
    e[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q[1], q[1], e[1], 0, 0, 0);
    e[2] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q[2], q[2], e[2], 0, 0, 0);
    e[3] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q[3], q[3], e[3], 0, 0, 0);
    p[2] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q[1], q[2], p[2], 0, 0, 0);
  }
  __device__ __forceinline__ bool fits() const { return (float)most.x <= kMostDigits && (float)most.y <= kMostDigits; }
  // The sums so far into their low and high (2^32) half (`first`: there is nothing in these yet).  Products of a digit
  // with itself count half: the sum with the transpose makes them whole.
  __device__ __forceinline__ void drain(double* lo, double* hi, int ld, bool first) const {
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 4; ++i) {   // lane (column l % 16) holds rows 4 (l / 16) + i
      const int at = (4 * (l >> 4) + i) * ld + (l & 15);
      double w = fma((double)p[2][i], 0x1p24, fma((double)p[1][i], 0x1p16, (double)p[0][i] * 0x1p8)) +
                 fma((double)e[1][i], 0x1p15, (double)e[0][i] * 0.5);
      const double h = fma((double)p[4][i], 0x1p8, (double)p[3][i]) + fma((double)e[3][i], 0x1p15, (double)e[2][i] * 0.5);
      // (d4's weight: 254 * 2^24)
      const double t = fma((double)f[3][i], 0x1p16, fma((double)f[2][i], 0x1p8, (double)f[1][i])) +
                       fma((double)e[4][i], 127.0 * 0x1p16, (double)f[0][i] * 0x1p-8);
      double v = fma(t, 254.0, h);
      if (!first) {
        w += lo[at];
        const double carry = __builtin_rint(w * 0x1p-32);
        w = fma(carry, -0x1p32, w);
        v += hi[at] + carry;
      }
      lo[at] = w;
      hi[at] = v;
    }
  }
};

// N groups of four tokens from token t0 on, wave wv of NWV taking every NWV-th
template <int NWV, bool PAIR, bool CACHED, int N>
__device__ __forceinline__ void load_groups(u32x4 (&v)[N], const uint16_t* row, int t0, int nv) {
  constexpr int d = PAIR ? 64 : 128;
  const int t1 = t0 + 4 * (threadIdx.x >> 6) + ((threadIdx.x & 63) >> 4);
  auto piece = [&](int u) __attribute__((always_inline)) {
    const u32x4* p = reinterpret_cast<const u32x4*>(row + (long)(t1 + 4 * u * NWV) * d);
    return NWV == 1 && !CACHED ? __builtin_nontemporal_load(p) : *p;   // (see kMostCached)
  };
  if (t0 + 4 * N * NWV <= nv) {   // (whole pieces without a branch per load)
#pragma unroll
    for (int u = 0; u < N; ++u) v[u] = piece(u);
  } else {
#pragma unroll
    for (int u = 0; u < N; ++u) {
      v[u] = u32x4{0u, 0u, 0u, 0u};
      if (t1 + 4 * u * NWV < nv) v[u] = piece(u);
    }
  }
}

// On the fp64 matrix cores: A and B operand of one instruction are the same register (lane (b1, k) holds
// X[t0 + k][b1*8 + b2] for the 4 tokens of a group and one b2); products of fp16 values are exact, sums round.
template <int NWV, bool PAIR, bool CACHED>
__device__ __forceinline__ void gram16_fp64(const uint16_t* row, int nv, double* mats, double* out, int ldo) {
  constexpr int ld = 17, kMat = 16 * ld, GP = 4;
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
  f64x4 acc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int t0 = 0; t0 < nv; t0 += 4 * GP * NWV) {
    u32x4 y[GP];
    load_groups<NWV, PAIR, CACHED>(y, row, t0, nv);
#pragma unroll
    for (int u = 0; u < GP; ++u) {
      const f16x8 h = __builtin_bit_cast(f16x8, y[u]);
#pragma unroll
      for (int b2 = 0; b2 < 8; ++b2) {
        const double a = (double)(float)h[b2];
        acc[b2 & 3] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, a, acc[b2 & 3], 0, 0, 0);
      }
    }
  }
  double* const dst = mats + wv * kMat;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = (l >> 4) + 4 * i, c = l & 15;
    const double sum = (acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i]);
    dst[r * ld + c] = (PAIR && (r >> 3) != (c >> 3)) ? 0.0 : sum;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4 / NWV; ++k) {
    const int idx = (int)threadIdx.x + 64 * NWV * k, at = (idx >> 4) * ld + (idx & 15);
    double sum = mats[at];
#pragma unroll
    for (int w = 1; w < NWV; ++w) sum += mats[w * kMat + at];   // fixed order: reproducible
    out[(idx >> 4) * ldo + (idx & 15)] = sum;
  }
}

// mats: 2 * NWV matrices of 16 x 17 doubles in LDS; s_fits: NWV words.  out may be mats (ldo 17).  All waves call it; it
// ends with a barrier.
template <int NWV, bool PAIR, bool CACHED>
__device__ __forceinline__ void gram16(const uint16_t* __restrict__ X, int nv, long head_gap, double* mats,
                                       int* s_fits, double* out, int ldo) {
  constexpr int ld = 17, kMat = 16 * ld;
  constexpr int GP = NWV == 1 ? 4 : 8;   // groups requested together
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6, b1 = l & 15;
  const uint16_t* const row = PAIR ? X + (b1 >> 3) * head_gap + (b1 & 7) * 8 : X + b1 * 8;
  static_assert(kDrainTokens % (4 * GP) == 0, "a wave's share is whole steps");
  GramSums sums;
  u32x4 x[GP], y[GP];
  load_groups<NWV, PAIR, CACHED>(x, row, 0, nv);
  int t0 = 0;
  bool more = true;
#pragma unroll 1
  for (bool first = true; more; first = false) {
    sums.clear();
#pragma unroll 1
    do {
      t0 += 4 * GP * NWV;
      more = t0 < nv;
      if (more) load_groups<NWV, PAIR, CACHED>(y, row, t0, nv);
#pragma unroll
      for (int u = 0; u < GP; u += 2) sums.add(x[u], x[u + 1]);
      if (!more) break;
#pragma unroll
      for (int u = 0; u < GP; ++u) x[u] = y[u];
    } while (t0 % (kDrainTokens * NWV) != 0);
    sums.drain(mats + 2 * wv * kMat, mats + (2 * wv + 1) * kMat, ld, first);
  }
  bool fits = __all(sums.fits());
  if (NWV > 1 && l == 0) s_fits[wv] = fits;
  __syncthreads();
  if (NWV > 1) {
#pragma unroll
    for (int w = 0; w < NWV; ++w) fits &= s_fits[w] != 0;
  }
  if (fits) {   // (the same answer in every wave)
    double val[4 / NWV];
#pragma unroll
    for (int k = 0; k < 4 / NWV; ++k) {
      const int idx = (int)threadIdx.x + 64 * NWV * k, p = idx >> 4, q = idx & 15;
      double s_lo = 0.0, s_hi = 0.0;
#pragma unroll
      for (int w = 0; w < NWV; ++w) {
        const double* m = mats + 2 * w * kMat;
        s_lo += m[p * ld + q] + m[q * ld + p];
        s_hi += m[kMat + p * ld + q] + m[kMat + q * ld + p];
      }
      // (no products across the heads of a pair)
      val[k] = (PAIR && (p >> 3) != (q >> 3)) ? 0.0 : fma(s_hi, 0x1p32, s_lo) * 0x1p-48;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4 / NWV; ++k) {
      const int idx = (int)threadIdx.x + 64 * NWV * k;
      out[(idx >> 4) * ldo + (idx & 15)] = val[k];
    }
  } else {
    gram16_fp64<NWV, PAIR, CACHED>(row, nv, mats, out, ldo);
  }
  __syncthreads();
}

// The unit of workgroup wg of n, in launches of many workgroups: they go round-robin to the eight XCDs and, in each, to
// its four shader engines, whatever these have left to do, so workgroup wg runs on engine wg % 32.  Keys and values
// (units 2 i and 2 i + 1), which take 25 and 32 us a wave, and the blocks past a sequence's end would each fall to the
// same few engines; a group of 32 units is dealt five places further on than the one before it.
// 14720 of 16384 blocks valid: projection 149 us, 160 in plain order.
__device__ __forceinline__ int dealt_unit(int wg, int n) {
  return wg < (n & ~31) ? (wg & ~31) | ((wg + 5 * (wg >> 5)) & 31) : wg;
}

// NWV waves per block: the two contractions are split over the waves by token, the eigen-solver
// runs in one of them.  The host picks NWV so that the launch has about one wave per SIMD.
// PAIR: heads of 64 channels with j1 = 8.  The same block (keys or values, same sequence and block
// position) of two neighbouring kv heads is worked as one block of 128 channels: the two 8 x T_b*8
// regrouped matrices on top of each other.  The 16 x 16 Gram matrix then holds the heads' own 8 x 8
// Gram matrices on its diagonal; the blocks off the diagonal (products across heads) are set to
// zero, after which every rotation between the two halves is the identity and the iteration solves
// the two 8 x 8 problems side by side (the rotations, their order and the stopping rule are those of
// the 16 x 16 case).  Ordering, small tensors, projection and outputs are per head.
// QB, FULL: QB != 0 quantizes the large tensor here, straight from the projection's registers, to
// QB-bit codes (FULL: all 2^QB of them) and writes codes and steps into the cache; the fp32 rows do
// not go to the workspace then and no quantizer launch follows (d = 128, one or two step groups per
// row).  QB == 0 leaves the fp32 rows in the workspace for quantize_tiles_kernel.
// Then the kernel also ends the call: the last workgroup to finish (a ticket counter in the third
// word of the workspace header, zero between calls) folds the blocks' status words into the call's
// two; status words travel as device-scope stores and loads, as the counter does, so no cache
// write-back or invalidation is needed between the XCDs.
// PART: calls of thousands of blocks (a prompt) are bound by throughput, not by one block's latency, and
// run as three launches, each with one wave per block or less and several waves per SIMD: PART 1 is the
// Gram matrix alone (left in the block's region of the workspace), then solve16_kernel, two to eight blocks
// per wave, then PART 3, the projection and quantizer.  In one launch every block derives each of its
// rotations in eight lanes at once and its solver, a chain of dependent instructions, holds the
// registers of the contractions.  The arithmetic, and so every bit written, is that of the other builds.
// 14720 blocks (4-bit, d = 128): 670 us in one launch, 163 + 100 + 280 us in three when both contractions were fp64, 98 + 87 +
// 137 now (steady clocks).
// Launch bounds: one launch (PART 0) asks for two waves per SIMD, or its products' accumulators go to registers of
// their own and calls of more than one workgroup a compute unit hold one (1024 blocks of 64 channels, 8 bits: 56 us, 37).
// N3 (PART 3 with the quantizer, d = 128): three local tensors (Eq. 2 with n = 3, factor shapes
// 1 * (T_b/8) * 8 by j1 * j2 * 1) in the same kernel.  The first cut's right factor R is never
// stored: a first pass over the rows forms it 16 tokens at a time (rounded to fp32, the precision
// the three-kernel path keeps it in) and adds it to the 8 x 8 Gram matrix of the second cut,
// A^T A with A[(r, a2, b2), a3]; the same wave solves that 8 x 8 problem and writes T_3; a second
// pass forms R again, this time with the tokens down the rows of the matrix-core result, which is
// the operand layout that lets a second matrix product contract over the eight tokens of a run
// (T_2 = A V' diag(1/sigma')), and hands the rows of T_2 to the quantizer in the registers it
// expects them in.  job.keep_large: the fp32 rows of T_2 also go to the workspace.
// CACHED: PART 1 requests the rows with plain loads (see kMostCached), PART 3 (2 or 4 bits) in the matrix cores' order (see
// kLeastDirect).
template <int NWV, bool PAIR, int QB = 0, bool FULL = false, int PART = 0, bool N3 = false, bool CACHED = false>
__global__ __launch_bounds__(64 * NWV, PART == 1 ? 3 : PART == 3 ? (!CACHED && (PAIR || N3 || QB == 4 || QB == 2) ? 3 : 4) : 2) void decompose16_kernel(dq_format fmt, dq_cache cache, CompressJob job,
                                                               float* __restrict__ large_ws,
                                                               int32_t* __restrict__ unit_status,
                                                               int32_t* __restrict__ call_status) {
  constexpr bool LEAN = PART != 0;
  // Projection and quantizer of a prompt's 2- and 4-bit codes: FastProject.  (Eight bits put 1 in 700
  // elements near a decision, and a small call, whose block has four waves, gains nothing: 320 blocks
  // 39.8 us with it, 39.3 without.)
  constexpr bool FAST = PART == 3 && (QB == 2 || QB == 4) && !N3;
  __shared__ int s_last_block;
  auto end_call = [&]() __attribute__((always_inline)) {   // QB != 0 only; every workgroup, once, at its end
    // every wave waits for its own device-scope stores (the status words) to be acknowledged; after
    // the barrier all of the workgroup's have been, and only then is the ticket taken
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __syncthreads();
    if (threadIdx.x == 0) {
      const int ticket = __hip_atomic_fetch_add(call_status + 2, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_last_block = (ticket == (int)gridDim.x - 1);
      if (s_last_block) __hip_atomic_store(call_status + 2, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!s_last_block || threadIdx.x >= 64) return;
    int flags = 0, sweeps = 0;
    const int n_units = (PAIR ? 2 : 1) * (int)gridDim.x;
    for (int u = threadIdx.x; u < n_units; u += 64) {
      const int w = __hip_atomic_load(unit_status + u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      flags |= w & 0xFF;
      sweeps = max(sweeps, w >> 8);
    }
    for (int o = 32; o > 0; o >>= 1) {
      flags |= __shfl_xor(flags, o);
      sweeps = max(sweeps, __shfl_xor(sweeps, o));
    }
    if (threadIdx.x == 0) { call_status[0] = flags; call_status[1] = sweeps; }
  };
  if (QB != 0 && PART == 0 && call_is_idle(job)) {
    // A call that skips every sequence ends here, without a ticket: hundreds of workgroups drawing
    // theirs from one counter at the same time took 4.1 us of the 6.1 such a launch cost (2.0 now).
    if (blockIdx.x == 0 && threadIdx.x < 2) call_status[threadIdx.x] = 0;
    return;
  }
  const Geometry g = make_geometry(fmt, cache.kv_heads, cache.block_capacity);
  // the work unit (of the pair's first head); the second head's unit lies `unit_gap` further on
  const int wg = PART != 0 ? dealt_unit(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  int unit = wg;
  const int unit_gap = 2 * job.n_blocks;
  if (PAIR) {
    const int pb = wg >> 1, j = pb % job.n_blocks, hp = pb / job.n_blocks;   // hp = b * (H/2) + head pair
    const int half_h = g.H >> 1;
    unit = (((hp / half_h) * g.H + 2 * (hp % half_h)) * job.n_blocks + j) * 2 + (wg & 1);
  }
  const UnitRef ur = unit_ref(g, job, unit);
  const int which = ur.which, slot = ur.slot, nv = ur.nv;
  const long bh = ur.bh;
  // (the three launches of a prompt: the solver's launch has left the status words)
  if (PART == 3 && QB != 0 && blockIdx.x == 0) {
    if (call_is_idle(job)) {
      if (threadIdx.x < 2) call_status[threadIdx.x] = 0;
      return;
    }
    fold_status<64>(unit_status, (PAIR ? 2 : 1) * (int)gridDim.x, call_status);
  }
  if (PART != 0 && slot < 0) return;
  if (slot < 0) {
    if (threadIdx.x == 0) {
      if (QB != 0) {
        __hip_atomic_store(unit_status + unit, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (PAIR) __hip_atomic_store(unit_status + unit + unit_gap, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        unit_status[unit] = 0;
        if (PAIR) unit_status[unit + unit_gap] = 0;
      }
    }
    if constexpr (QB != 0 && PART == 0) end_call();
    return;
  }
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int solver = blockIdx.x % NWV;   // the wave that runs the eigen-solver (spread over the SIMDs)
  constexpr int j1 = 16, ld = 17;
  constexpr int d = PAIR ? 64 : 128;     // halves per row in memory
  const uint16_t* X = ur.X;  // [nv, d] fp16 bits
  const long head_gap = (long)job.t_new * d;   // PAIR: from a row of the first head to the same row of the second
  double* const gram_ws = reinterpret_cast<double*>(large_ws + (long)unit * g.Tb * d);   // PART: G, then W, of this block

  static_assert(!LEAN || NWV == 1, "one wave per block");
  static_assert(!N3 || (LEAN && !PAIR && QB != 0), "three tensors: PART 3 with the quantizer, d = 128");
  constexpr int kMat = j1 * ld;                              // doubles per 16 x 16 matrix (padded rows)
  constexpr int kMatBytes = 2 * NWV * kMat * (int)sizeof(double);   // the waves' Gram partials; then G and W
  // fused quantizer: one byte per element of QT token rows, then the value layout's staging
  // (a pair: one such area per head, of 64 channels each)
  constexpr int QT = LEAN ? 32 : kTileTokens;                // rows quantized and packed at a time
  constexpr int kHeadArea = QT * d + d * (pack_parts(QB ? QB : 8, QT) * QT * (QB ? QB : 8) / 32 + 1) * 4;
  typedef FastProject<QB == 2 ? 2 : 4, FULL, PAIR, CACHED> FP;
  constexpr int kFieldBytes = FAST ? FP::kStageBytes + FP::kRowBytes : QB ? (PAIR ? 2 : 1) * kHeadArea : 16;
  // (the three launches: no matrices in LDS, but the second cut's)
  constexpr int kPoolBytes = LEAN ? (kMatBytes > kFieldBytes ? kMatBytes : kFieldBytes) : kMatBytes + kFieldBytes;
  __shared__ __attribute__((aligned(16))) unsigned char pool[kPoolBytes];
  double* const A = reinterpret_cast<double*>(pool);
  double* const W = A + kMat;
  uint8_t* const lds_u = LEAN ? pool : pool + kMatBytes;
  __shared__ double lam[j1], lam2[j1];
  __shared__ uint8_t s_list[FAST && CACHED ? kTileTokens : 1];   // the tile's tokens that are settled in fp64

  // ---- Gram matrix G[p][q] = sum_{t, b2} X[t, p*8+b2] X[t, q*8+b2] ----
  if constexpr (PART != 3) {
    __shared__ int s_fits[NWV];
    gram16<NWV, PAIR, CACHED>(X, nv, head_gap, A, s_fits, PART == 1 ? gram_ws : A, PART == 1 ? j1 : ld);
  }
  if constexpr (PART == 1) return;
  if constexpr (PART == 0) {
  if (wv == solver) {
    // lane (pair j = l % 8, row group l / 8) holds rows 2 (l / 8) + i of columns j and j + 8
    Jacobi16<2> jac;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      jac.x[i] = A[(2 * (l >> 3) + i) * ld + (l & 7)];
      jac.y[i] = A[(2 * (l >> 3) + i) * ld + (l & 7) + 8];
    }
    const int sweeps = jac.template run<PAIR>();

    // ---- singular values, ordering, small tensor ----
    store_factors<2, PAIR, ld>(jac, lam, lam2, W);
    const long blk = (long)bh * g.NB + slot;
    uint16_t* small = (which ? cache.v_small : cache.k_small) + blk * g.small_per_block;
    bool sat = false;
    for (int idx = l; idx < j1 * j1; idx += 64) {
      // neighbouring lanes write neighbouring entries of the stored array (keys are stored transposed)
      const int b1 = which ? idx >> 4 : idx & 15, r = which ? idx & 15 : idx >> 4;
      const double ts = W[r * ld + b1] * lam2[r];   // T_S = U Sigma = W Lambda
      if (PAIR) {
        // the heads' 8 x 8 small tensors are the diagonal blocks (the second head's blocks lie NB
        // blocks further on in the cache); the entries off the diagonal are zero and go nowhere
        if ((b1 >> 3) == (r >> 3)) {
          const uint16_t hb = f64_to_f16_rne(ts, true, &sat);
          uint16_t* sm = small + (long)(b1 >> 3) * g.NB * g.small_per_block;
          if (which) sm[(b1 & 7) * 8 + (r & 7)] = hb;
          else sm[(r & 7) * 8 + (b1 & 7)] = hb;
        }
      } else {
        const uint16_t hb = f64_to_f16_rne(ts, true, &sat);
        if (which) small[b1 * j1 + r] = hb;   // values: natural [b1][r]
        else small[r * j1 + b1] = hb;         // keys: transposed [r][b1]
      }
    }
    // this block's status word: bit 0 = T_S saturated, bits 8.. = Jacobi sweeps used
    const bool any_sat = __any(sat);
    if (l == 0) {
      const int word = (any_sat ? 1 : 0) | (sweeps << 8);
      // (a pair: one word for both heads)
      if (QB != 0) {
        __hip_atomic_store(unit_status + unit, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (PAIR) __hip_atomic_store(unit_status + unit + unit_gap, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        unit_status[unit] = word;
        if (PAIR) unit_status[unit + unit_gap] = word;
      }
    }
  }
  __syncthreads();
  }

  if constexpr (FAST) {
    FP fp;
    fp.X = X; fp.nv = nv; fp.head_gap = head_gap; fp.one_group = !PAIR && g.groups == 1;
    fp.setup(gram_ws);
    const int n = l & 15, q4 = l >> 4;
    const long blk = bh * g.NB + slot;
    uint8_t* const codes = (which ? cache.v_codes : cache.k_codes) + blk * g.codes_per_block;
    uint16_t* const scales = (which ? cache.v_scales : cache.k_scales) + blk * g.scales_per_block;
    const long codes_gap = (long)g.NB * g.codes_per_block, scales_gap = (long)g.NB * g.scales_per_block;   // PAIR: to the second head's
    uint8_t* const stage = lds_u;
    // the lane's 32 elements of a key token's row: words 4 q4 .. of 4-bit codes, 2 q4 .. of 2-bit codes
    auto store_key = [&](int t, const uint32_t (&part)[4], uint16_t sb) __attribute__((always_inline)) {
      uint8_t* const dst = codes + (PAIR ? (q4 >> 1) * codes_gap + (long)t * (8 * QB) + (q4 & 1) * (4 * QB)
                                         : (long)t * (16 * QB) + q4 * (4 * QB));
      if (QB == 4) __builtin_nontemporal_store(u32x4{part[0], part[1], part[2], part[3]}, reinterpret_cast<u32x4*>(dst));
      else *reinterpret_cast<u32x2*>(dst) = u32x2{part[0] | (part[1] << 16), part[2] | (part[3] << 16)};
      if (PAIR) {
        if (!(q4 & 1)) scales[(q4 >> 1) * scales_gap + t] = sb;
      } else if (q4 == 0 || (!fp.one_group && q4 == 2)) {
        scales[(long)t * g.groups + (q4 >> 1)] = sb;
      }
    };
    // the step of a value token's group that holds the lane's row n
    auto store_value_step = [&](int t, uint16_t sb) __attribute__((always_inline)) {
      if (PAIR) scales[(n >> 3) * scales_gap + t] = sb;
      else if (!fp.one_group || n < 8) scales[(long)t * g.groups + (n >> 3)] = sb;
    };
    double w64[4];
    if (!CACHED) fp.load_factor(w64, l);
    // Two tokens through fp64: lane (n, q4) has column b2 = n % 8 of token n / 8 of the two, the t-th of the tile (t < 0: none)
    auto settle = [&](const uint16_t (&xc)[4], int tile, int t, int lane) __attribute__((always_inline)) {
      const int n = lane & 15, q4 = lane >> 4, b2 = n & 7;
      uint16_t sb;
      const uint32_t fields = fp.settle(w64, xc, sb);   // rows 4 q4 + i, b2 = n % 8
      if (which) {
        // the token's field in its row's word (the other token's may be in the same one)
        uint32_t* const word = reinterpret_cast<uint32_t*>(stage + (b2 * 16 + 4 * q4) * FP::STRIDE) + max(t, 0) * QB / 32;
        const int shift = (t * QB) & 31;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (t >= 0) {
            atomicAnd(word + i * (FP::STRIDE / 4), ~(((1u << QB) - 1u) << shift));
            atomicOr(word + i * (FP::STRIDE / 4), ((fields >> (8 * i)) & 0xFFu) << shift);
          }
      } else {
        // row r's eight b2 are neighbours: lane b2 = i collects those of row 4 q4 + i
        uint32_t mine = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          uint32_t v = ((fields >> (8 * i)) & 0xFFu) << (QB * b2);
          v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);
          v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);
          v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);
          mine = b2 == i ? v : mine;
        }
        const int r = 4 * q4 + b2;
        uint8_t* const dst = codes + (PAIR ? (q4 >> 1) * codes_gap + (long)(tile + t) * (8 * QB) + (r & 7) * QB
                                           : (long)(tile + t) * (16 * QB) + r * QB);
        if (t >= 0 && b2 < 4) {
          if (QB == 4) *reinterpret_cast<uint32_t*>(dst) = mine;
          else *reinterpret_cast<uint16_t*>(dst) = (uint16_t)mine;
        }
      }
      if (t >= 0 && b2 == 0) {
        if (PAIR) {
          if (!(q4 & 1)) scales[(q4 >> 1) * scales_gap + tile + t] = sb;
        } else if (q4 == 0 || (!fp.one_group && q4 == 2)) {
          scales[(long)(tile + t) * g.groups + (q4 >> 1)] = sb;
        }
      }
    };
    u32x4 next[4];
    fp.load(next, 0);
    for (int tile = 0; tile < g.Tb; tile += kTileTokens) {
      int listed = fp.hard ? kTileTokens : 0;   // DIRECT: tokens of the tile in s_list (a hard block: all of them)
#pragma unroll 1
      for (int t0 = CACHED && fp.hard ? kTileTokens : 0; t0 < kTileTokens; t0 += 16) {
        u32x4 x[4] = {next[0], next[1], next[2], next[3]};
        fp.clear(x, tile + t0);
        if (!CACHED) FP::turn(x, stage + FP::kStageBytes);
        if (tile + t0 + 16 < nv) {   // (the next sixteen tokens of the block, if there are any)
          fp.load(next, tile + t0 + 16);
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) next[u] = u32x4{0u, 0u, 0u, 0u};
        }
        uint32_t doubt = 0xFFFFu;
        if (!fp.hard) {
          f32x4 acc[8];
          uint16_t sb;
          if (!which) {
            fp.template project<false>(x, acc);
            uint32_t part[4];
            doubt = fp.template quantize<false>(acc, sb, part);
            if (!((doubt >> n) & 1u)) store_key(tile + t0 + n, part, sb);
          } else {
            fp.template project<true>(x, acc);
            uint32_t part[8];
            doubt = fp.template quantize<true>(acc, sb, part);
            // row (b2, r = n) of the tile, tokens t0 + 4 q4 .. + 3
#pragma unroll
            for (int b2 = 0; b2 < 8; ++b2) {
              uint8_t* const dst = stage + (b2 * 16 + n) * FP::STRIDE + (t0 / 4 + q4) * (QB / 2);
              if (QB == 4) *reinterpret_cast<uint16_t*>(dst) = (uint16_t)part[b2];
              else *dst = (uint8_t)part[b2];
            }
            if ((n & 4) == 0 && !((doubt >> (4 * q4 + (n & 3))) & 1u)) store_value_step(tile + t0 + 4 * q4 + (n & 3), sb);
          }
          __builtin_amdgcn_wave_barrier();   // (one wave: its LDS operations execute in order)
        }
        if constexpr (CACHED) {
          if (l < 16 && ((doubt >> l) & 1u)) s_list[listed + __builtin_popcount(doubt & ((1u << l) - 1u))] = (uint8_t)(t0 + l);
          listed += __builtin_popcount(doubt);
        } else {
          // the tokens in doubt, two at a time, while their rows lie in LDS
#pragma unroll 1
          while (doubt) {
            const int first = __builtin_ctz(doubt);
            doubt &= doubt - 1;
            const int tok = (n >> 3) == 0 ? first : doubt ? __builtin_ctz(doubt) : -1;
            doubt &= doubt - 1;
            uint16_t xc[4];
            FP::row_column(xc, max(tok, 0), stage + FP::kStageBytes);
            settle(xc, tile, tok < 0 ? -1 : t0 + tok, l);
          }
        }
      }
      if constexpr (CACHED) {
      __builtin_amdgcn_wave_barrier();
      if (listed > 0) {
        // (the lane's number anew: addresses formed from it ahead of the first pass would cost that pass its
        // registers, of which it has 122 to 128 for four waves a SIMD)
        int lane = l;
        asm volatile("" : "+v"(lane));
        const int n = lane & 15;
        fp.load_factor(w64, lane);
        // Pairs of tokens whose rows are requested together, while the ones before them are settled: one request after the
        // other, a block that is settled here as a whole was a chain of 32 round trips to memory.
        constexpr int PAIRS = 2;
        int tok_next[PAIRS];
        uint16_t x_next[PAIRS][4];
        auto request = [&](int base) __attribute__((always_inline)) {
#pragma unroll
          for (int k = 0; k < PAIRS; ++k) {
            const int at = base + 2 * k + (n >> 3);
            tok_next[k] = at >= listed ? -1 : fp.hard ? at : (int)s_list[at];
            fp.load_column(x_next[k], tok_next[k] < 0 ? -1 : tile + tok_next[k], lane);
          }
        };
        request(0);
#pragma unroll 1
        for (int base = 0; base < listed; base += 2 * PAIRS) {
          int tok[PAIRS];
          uint16_t xc[PAIRS][4];
#pragma unroll
          for (int k = 0; k < PAIRS; ++k) {
            tok[k] = tok_next[k];
#pragma unroll
            for (int s = 0; s < 4; ++s) xc[k][s] = x_next[k][s];
          }
          request(base + 2 * PAIRS);
#pragma unroll
          for (int k = 0; k < PAIRS; ++k) settle(xc[k], tile, tok[k], lane);
        }
      }
      }
      if (which) {
        __syncthreads();
        // the tile's rows in memory: [b2][r], or per head [b2][r % 8]
        constexpr int CPR = FP::ROWB / 16;   // 16-byte pieces per row
        int lane = l;
        asm volatile("" : "+v"(lane));
        for (int idx = lane; idx < 128 * CPR; idx += 64) {
          const int rw = idx / CPR, pc = idx % CPR;
          const uint32_t* src = reinterpret_cast<const uint32_t*>(stage + rw * FP::STRIDE + 16 * pc);
          const u32x4 v = {src[0], src[1], src[2], src[3]};
          uint8_t* const dst = codes + (PAIR ? ((rw >> 3) & 1) * codes_gap + (long)tile * (8 * QB) + ((rw >> 4) * 8 + (rw & 7)) * FP::ROWB + 16 * pc
                                             : (long)tile * (16 * QB) + rw * FP::ROWB + 16 * pc);
          __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(dst));
        }
        __syncthreads();
      }
    }
  } else
  // ---- projection: K'[t, r*8+b2] = sum_b1 W[r][b1] X[t, b1*8+b2], fp64 -> fp32 ----
  // One MFMA chain per b2: rows r, columns 16 tokens, contraction over b1 in 4 steps of 4.
  // Wave wv takes every NWV-th group of 16 tokens.
  {
    constexpr int NT = QT / 16 / NWV;   // token groups per wave in a chunk of QT tokens
    constexpr int TB = LEAN ? 1 : NT;   // groups whose rows are requested together
    double wreg[4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
      wreg[s] = PART == 3 ? gram_ws[j1 * j1 + (l & 15) * j1 + 4 * s + (l >> 4)] : W[(l & 15) * ld + 4 * s + (l >> 4)];
    double w3reg[4] = {0.0, 0.0, 0.0, 0.0};
    if constexpr (N3) {
      // ---- second cut: Gram matrix of A[(r, a2, b2), a3] from the right factor, 16 tokens at a time ----
      constexpr int N = kRun, LD3 = N + 1;
      double* const Dm = reinterpret_cast<double*>(pool);        // 16 x 16 token products, padded rows
      double* A0 = Dm + kMat;
      double* A1 = A0 + N * LD3;
      double* V0 = A1 + N * LD3;
      double* V1 = V0 + N * LD3;
      double* const W3 = V1 + N * LD3;                           // [e][a3] = V'[a3, e] / sigma'_e
      double* const rc = W3 + N * N;
      double* const rs = rc + N;
      double* const lam3 = rs + N;
      double* const sigma3 = lam3 + N;
      int* const partner = reinterpret_cast<int*>(sigma3 + N);
      int* const is_p = partner + N;
      int* const order3 = is_p + N;
      static_assert((kMat + 4 * N * LD3 + N * N + 4 * N) * (int)sizeof(double) + 3 * N * (int)sizeof(int) <= kPoolBytes,
                    "the second cut's matrices fit the pool");
      f64x4 g3[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) g3[i] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
      for (int t0 = 0; t0 < nv; t0 += 16) {
        const int t = t0 + (l & 15);
        u32x4 x[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          x[s] = u32x4{0u, 0u, 0u, 0u};
          if (t < nv) x[s] = *reinterpret_cast<const u32x4*>(X + (long)t * d + (4 * s + (l >> 4)) * 8);
        }
        f64x4 acc[8];
#pragma unroll
        for (int b2 = 0; b2 < 8; ++b2) acc[b2] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const f16x8 h = __builtin_bit_cast(f16x8, x[s]);
#pragma unroll
          for (int b2 = 0; b2 < 8; ++b2)
            acc[b2] = __builtin_amdgcn_mfma_f64_16x16x4f64(wreg[s], (double)(float)h[b2], acc[b2], 0, 0, 0);
        }
        // lane (token l % 16, k = l / 16) holds R[r = k + 4 i][token][b2]: both operands of a product
        // of the 16 tokens with themselves over four r; the runs' own 8 x 8 blocks are kept below
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int b2 = 0; b2 < 8; ++b2) {
            const double v = (double)(float)acc[b2][i];
            g3[b2 & 3] = __builtin_amdgcn_mfma_f64_16x16x4f64(v, v, g3[b2 & 3], 0, 0, 0);
          }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
        Dm[((l >> 4) + 4 * i) * ld + (l & 15)] = (g3[0][i] + g3[1][i]) + (g3[2][i] + g3[3][i]);
      __builtin_amdgcn_wave_barrier();
      {
        const int p = l >> 3, q = l & 7;
        A0[p * LD3 + q] = Dm[p * ld + q] + Dm[(p + 8) * ld + q + 8];
        V0[p * LD3 + q] = (p == q) ? 1.0 : 0.0;
      }
      __builtin_amdgcn_wave_barrier();
      double trace3 = 0.0;
#pragma unroll
      for (int i = 0; i < N; ++i) trace3 += A0[i * LD3 + i];
      const double floor3 = 1e-17 * trace3;
      // parallel cyclic Jacobi: 7 rounds of 4 disjoint rotations per sweep (the iteration of the
      // three-kernel path's second cut, in this one wave)
      double* Ac = A0; double* An = A1; double* Vc = V0; double* Vn = V1;
      constexpr int NM1 = N - 1;
      for (int sweep = 0; sweep < 16; ++sweep) {
        bool any_big = false;
#pragma unroll 1
        for (int round = 0; round < NM1; ++round) {
          bool big = false;
          if (l < N / 2) {
            int p, q;
            if (l == 0) { p = NM1; q = round; }
            else { p = (round + l) % NM1; q = (round - l + NM1) % NM1; }
            if (p > q) { const int tmp = p; p = q; q = tmp; }
            double c, sn;
            jacobi_rotation(Ac[p * LD3 + p], Ac[q * LD3 + q], Ac[p * LD3 + q], floor3, c, sn, big);
            rc[p] = c; rs[p] = sn; rc[q] = c; rs[q] = sn;
            partner[p] = q; partner[q] = p;
            is_p[p] = 1; is_p[q] = 0;
          }
          any_big = any_big || __any(big);
          __builtin_amdgcn_wave_barrier();
          {
            const int i = l >> 3, j = l & 7;
            const int pi = partner[i], pj = partner[j];
            const double cj = rc[j], sj = is_p[j] ? -rs[j] : rs[j];
            const double ci = rc[i], si = is_p[i] ? -rs[i] : rs[i];
            const double aj_i = Ac[i * LD3 + j] * cj + Ac[i * LD3 + pj] * sj;
            const double aj_pi = Ac[pi * LD3 + j] * cj + Ac[pi * LD3 + pj] * sj;
            An[i * LD3 + j] = ci * aj_i + si * aj_pi;
            Vn[i * LD3 + j] = Vc[i * LD3 + j] * cj + Vc[i * LD3 + pj] * sj;
          }
          __builtin_amdgcn_wave_barrier();
          double* tp = Ac; Ac = An; An = tp;
          tp = Vc; Vc = Vn; Vn = tp;
        }
        if (!any_big) break;
      }
      if (l < N) lam3[l] = Ac[l * LD3 + l];
      __builtin_amdgcn_wave_barrier();
      if (l < N) {
        int rank = 0;
        const double me = lam3[l];
        for (int s2 = 0; s2 < N; ++s2) rank += (lam3[s2] > me) || (lam3[s2] == me && s2 < l);
        order3[rank] = l;
      }
      __builtin_amdgcn_wave_barrier();
      if (l < N) {
        const double lmax = fmax(lam3[order3[0]], 0.0);
        const double lv = lam3[order3[l]];
        sigma3[l] = (lv > 1e-12 * lmax && lv > 0.0) ? sqrt(lv) : 0.0;
      }
      __builtin_amdgcn_wave_barrier();
      {
        const int e = l >> 3, a3 = l & 7;
        const double v = Vc[a3 * LD3 + order3[e]];
        const double sg = sigma3[e];
        W3[e * N + a3] = sg > 0.0 ? v / sg : 0.0;
        const long b3 = ((long)bh * g.NB + slot) * (N * N);
        const uint16_t hb = f64_to_f16_rne(v * sg, true, nullptr);   // |T_3| <= sqrt(j1): far inside fp16
        if (which) cache.v_small3[b3 + e * N + a3] = hb;   // values: natural [e][a3]
        else cache.k_small3[b3 + a3 * N + e] = hb;         // keys: transposed [a3][e]
      }
      __builtin_amdgcn_wave_barrier();
      // the token mix as the right-hand operand of a product over four tokens (k = l / 16, token
      // k + 4 i of the group): column n = l % 16 is row e = n % 8 of run n / 8; a token of the other
      // run contributes nothing
#pragma unroll
      for (int i = 0; i < 4; ++i)
        w3reg[i] = ((i >> 1) == ((l & 15) >> 3)) ? W3[(l & 7) * N + (((l >> 4) + 4 * i) & 7)] : 0.0;
      __builtin_amdgcn_wave_barrier();   // W3 is read; the fields may take the pool
    }
    float* out = large_ws + (long)unit * g.Tb * d;
    const long out_gap = (long)unit_gap * g.Tb * d;   // PAIR: to the second head's rows in the workspace
    for (int t0 = 0; t0 < g.Tb; t0 += QT) {
#pragma unroll 1
     for (int tg0 = 0; tg0 < NT; tg0 += TB) {
      u32x4 x[TB][4];
#pragma unroll
      for (int tgi = 0; tgi < TB; ++tgi) {
        const int t = t0 + 16 * ((tg0 + tgi) * NWV + wv) + (l & 15);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          x[tgi][s] = u32x4{0u, 0u, 0u, 0u};
          // b1 = 4 s + l / 16 (a pair: row b1 % 8 of head b1 / 8 = s / 2)
          if (t < nv)
            x[tgi][s] = *reinterpret_cast<const u32x4*>(PAIR ? X + (s >> 1) * head_gap + (long)t * d + ((4 * s + (l >> 4)) & 7) * 8
                                                             : X + (long)t * d + (4 * s + (l >> 4)) * 8);
        }
      }
#pragma unroll
      for (int tgi = 0; tgi < TB; ++tgi) {
        const int tg = tg0 + tgi;
        const int t = t0 + 16 * (tg * NWV + wv) + (l & 15);
        f64x4 acc[8];
#pragma unroll
        for (int b2 = 0; b2 < 8; ++b2) acc[b2] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const f16x8 h = __builtin_bit_cast(f16x8, x[tgi][s]);
#pragma unroll
          for (int b2 = 0; b2 < 8; ++b2) {
            // (three tensors: operands swapped, so that the result has the 16 tokens down its rows)
            if (N3) acc[b2] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)(float)h[b2], wreg[s], acc[b2], 0, 0, 0);
            else acc[b2] = __builtin_amdgcn_mfma_f64_16x16x4f64(wreg[s], (double)(float)h[b2], acc[b2], 0, 0, 0);
          }
        }
        if constexpr (N3) {
          // lane (r = l % 16, k = l / 16) holds R[r][token k + 4 i][b2], rounded to fp32 as in the first
          // pass: left operand of the product over the tokens; the result has rows r = l / 16 + 4 i and
          // columns (run, e), which is where the quantizer below expects a row of the large tensor
#pragma unroll
          for (int b2 = 0; b2 < 8; ++b2) {
            f64x4 o = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int i = 0; i < 4; ++i)
              o = __builtin_amdgcn_mfma_f64_16x16x4f64((double)(float)acc[b2][i], w3reg[i], o, 0, 0, 0);
            acc[b2] = o;
          }
        }
        if constexpr (QB == 0) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            // row r = l / 16 + 4 i of the large tensor (a pair: row r % 8 of head r / 8 = i / 2)
            float* dst = PAIR ? out + (i >> 1) * out_gap + (long)t * d + (((l >> 4) + 4 * i) & 7) * 8
                              : out + (long)t * d + ((l >> 4) + 4 * i) * 8;
            *reinterpret_cast<float4*>(dst) = make_float4((float)acc[0][i], (float)acc[1][i], (float)acc[2][i], (float)acc[3][i]);
            *reinterpret_cast<float4*>(dst + 4) = make_float4((float)acc[4][i], (float)acc[5][i], (float)acc[6][i], (float)acc[7][i]);
          }
        } else {
          // ---- Eq. 1 on the token's row, from the registers: the lane holds rows r = l / 16 + 4 i
          // (i = 0..3) of token t, eight b2 each; the token's other rows sit in the lanes 16, 32 and
          // 48 further on.  Step groups: the whole row, or rows r < 8 (i < 2) and r >= 8.
          constexpr int QMAX = (1 << (QB - 1)) - 1;
          float f[4][8];
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int b2 = 0; b2 < 8; ++b2) f[i][b2] = (float)acc[b2][i];
          if (N3 && job.keep_large) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              float* dst = out + (long)t * d + ((l >> 4) + 4 * i) * 8;
              *reinterpret_cast<float4*>(dst) = make_float4(f[i][0], f[i][1], f[i][2], f[i][3]);
              *reinterpret_cast<float4*>(dst + 4) = make_float4(f[i][4], f[i][5], f[i][6], f[i][7]);
            }
          }
          float up[2] = {0.f, 0.f}, dn[2] = {0.f, 0.f};   // max |x| (FULL: max x and max -x) per group
#pragma unroll
          for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int b2 = 0; b2 < 8; ++b2) {
              if (FULL) {
                up[i >> 1] = fmaxf(up[i >> 1], f[i][b2]);
                dn[i >> 1] = fmaxf(dn[i >> 1], -f[i][b2]);
              } else {
                up[i >> 1] = fmaxf(up[i >> 1], fabsf(f[i][b2]));
              }
            }
          }
          if (!PAIR && g.groups == 1) {   // (a pair: group i / 2 is head i / 2's row, its only group)
            up[0] = up[1] = fmaxf(up[0], up[1]);
            dn[0] = dn[1] = fmaxf(dn[0], dn[1]);
          }
          uint16_t sb[2];
          float step[2], inv[2];
#pragma unroll
          for (int gi = 0; gi < 2; ++gi) {
            up[gi] = fmaxf(up[gi], __shfl_xor(up[gi], 16));
            up[gi] = fmaxf(up[gi], __shfl_xor(up[gi], 32));
            sb[gi] = group_step_bits<QMAX>(up[gi]);
            if (FULL) {
              dn[gi] = fmaxf(dn[gi], __shfl_xor(dn[gi], 16));
              dn[gi] = fmaxf(dn[gi], __shfl_xor(dn[gi], 32));
              const uint16_t down = f2h_rne(dn[gi] * (1.0f / (float)(QMAX + 1)));
              sb[gi] = sb[gi] > down ? sb[gi] : down;
            }
            step[gi] = h2f(sb[gi]);
            inv[gi] = step[gi] > 0.f ? __builtin_amdgcn_rcpf(step[gi]) : 0.f;
          }
          const int tl = 16 * (tg * NWV + wv) + (l & 15);   // the token's row among the QT rows in LDS
          if ((l >> 4) == 0) {
            uint16_t* sc = (which ? cache.v_scales : cache.k_scales) + ((long)bh * g.NB + slot) * g.scales_per_block +
                           (long)(t0 + tl) * g.groups;
            sc[0] = sb[0];
            if (PAIR) sc[(long)g.NB * g.scales_per_block] = sb[1];   // the second head's block, NB blocks further on
            else if (g.groups == 2) sc[1] = sb[1];
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            uint2 w;
            w.x = fields_of_four<QB, FULL>(f[i][0], f[i][1], f[i][2], f[i][3], step[i >> 1], inv[i >> 1]);
            w.y = fields_of_four<QB, FULL>(f[i][4], f[i][5], f[i][6], f[i][7], step[i >> 1], inv[i >> 1]);
            uint8_t* dst = PAIR ? lds_u + (i >> 1) * kHeadArea + tl * d + (((l >> 4) + 4 * i) & 7) * 8
                                : lds_u + tl * d + ((l >> 4) + 4 * i) * 8;
            *reinterpret_cast<uint2*>(dst) = w;
          }
        }
      }
     }
      if constexpr (QB != 0) {
        // every wave has left the fields of its tokens: pack these rows of the tile and send them off
        __syncthreads();
        uint8_t* codes = (which ? cache.v_codes : cache.k_codes) + ((long)bh * g.NB + slot) * g.codes_per_block +
                         (long)(t0 & ~(kTileTokens - 1)) * g.row_bytes;
        const int part = (t0 & (kTileTokens - 1)) / QT;
        if (PAIR) {
          pack_fields<QB, d, 64 * NWV, QT>(lds_u, 8, 8, which, codes, part);
          pack_fields<QB, d, 64 * NWV, QT>(lds_u + kHeadArea, 8, 8, which, codes + (long)g.NB * g.codes_per_block, part);
        } else {
          pack_fields<QB, d, 64 * NWV, QT>(lds_u, 16, 8, which, codes, part);
        }
      }
    }
  }
  if constexpr (QB != 0 && PART == 0) end_call();
}

// The constants of FastProject, from the solver's registers (a lane: ROWS of the rows b1 of two columns of W^T, places
// px and py; their sums cross eight lanes at most, where the projection's wave, one block in 64 lanes, took 850
// instructions for them, a fifth of its own: 14720 blocks 177 us for the projection, 193 before, and 7 more here then): the two fp16 pieces
// of W scaled by 2^(15 - e), |W[r]| < 2^e, as [b1 % 4][r][piece][b1 / 4]; 2^(e - 15) of every row; eps, eps_abs, hard.  They go
// to the block's place in LDS, on their way to G + kFastPieces.
constexpr int kFastPieceBytes = 2 * 256 * 2, kFastBytes = kFastPieceBytes + 20 * 4;   // (of the latter 19 floats are used)
template <int ROWS, bool PAIR>
__device__ __forceinline__ void store_fast_factors(const Jacobi16<ROWS>& jac, const double (&wx)[ROWS], const double (&wy)[ROWS],
                                                   int px, int py, double lx, double ly, unsigned char* dst) {
  static_assert(ROWS % 4 == 0, "a lane's rows are whole pieces");
  const int lane = threadIdx.x & 63, row0 = jac.first_row(lane);
  uint16_t* const pieces = reinterpret_cast<uint16_t*>(dst);
  float* const scales = reinterpret_cast<float*>(dst + kFastPieceBytes);
  auto over_rows = [&](float v, auto op) __attribute__((always_inline)) {   // the lanes that hold the column's other rows
    if (ROWS <= 8) v = op(v, lane_exchange<kDppXor8>(v));
    if (ROWS <= 4) v = op(v, __shfl_xor(v, 16));
    return v;
  };
  auto over_columns = [&](float v, auto op) __attribute__((always_inline)) {
    v = op(v, lane_exchange<kDppXor1>(v));
    v = op(v, lane_exchange<kDppXor2>(v));
    return op(v, lane_exchange<kDppXor7>(v));
  };
  auto add = [](float a, float b) { return a + b; };
  auto most = [](float a, float b) { return fmaxf(a, b); };
  const float lam[2] = {(float)lx, (float)ly};
  // s[b1] = sum_r |T_S[b1][r]|  (a pair: W is block-diagonal, the other head's columns add nothing)
  float s[ROWS];
#pragma unroll
  for (int i = 0; i < ROWS; ++i)
    s[i] = over_columns(fabsf((float)wx[i]) * lam[0] + fabsf((float)wy[i]) * lam[1], add);
  // sum, largest and least eigenvalue (a pair: of the column's own head)
  float total[2], top[2], least[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int head = (c ? py : px) >> 3;
    const bool sx = !PAIR || (px >> 3) == head, sy = !PAIR || (py >> 3) == head;
    if (PAIR) {
      // both heads' figures in every lane, then the column's own
      float t[2], m[2], n[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const bool hx = (px >> 3) == h, hy = (py >> 3) == h;
        t[h] = over_columns((hx ? lam[0] : 0.f) + (hy ? lam[1] : 0.f), add);
        m[h] = over_columns(fmaxf(hx ? lam[0] : 0.f, hy ? lam[1] : 0.f), most);
        n[h] = over_columns(fmaxf(hx ? -lam[0] : -INFINITY, hy ? -lam[1] : -INFINITY), most);
      }
      total[c] = head ? t[1] : t[0];
      top[c] = head ? m[1] : m[0];
      least[c] = -(head ? n[1] : n[0]);
    } else {
      total[c] = over_columns((sx ? lam[0] : 0.f) + (sy ? lam[1] : 0.f), add);
      top[c] = over_columns(fmaxf(lam[0], lam[1]), most);
      least[c] = -over_columns(fmaxf(-lam[0], -lam[1]), most);
    }
  }
  float rel = 0.f, abs = 0.f;
  bool soft = true;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int r = c ? py : px;
    float wm = 0.f, one = 0.f, two = 0.f, cs = 0.f;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const float ab = fabsf((float)(c ? wy[i] : wx[i]));
      wm = fmaxf(wm, ab);
      one += ab;
      two = fmaf(ab, ab, two);
      cs = fmaf(ab, s[i], cs);
    }
    wm = over_rows(wm, most);
    // |w| < 2^e (the rounding of wm to fp32 may only raise it); the smallest scale keeps 2^(15 - e) a float
    const int e = wm > 0.f ? max(__builtin_amdgcn_frexp_expf(wm * (1.f + 0x1p-22f)), -100) : 0;
    const float scale = __builtin_amdgcn_ldexpf(1.f, e - 15);
    float rest = 0.f;
    _Float16 h[2][ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      double left = __builtin_amdgcn_ldexp(c ? wy[i] : wx[i], 15 - e);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        float f = (float)left;
        asm("" : "+v"(f));   // (two conversions: of a double straight to fp16 there is only a long sequence)
        h[k][i] = (_Float16)f;
        left -= (double)(float)h[k][i];
      }
      // (a subnormal piece counts with exponent -14 as well: the addend)
      rest = fmaf((fabsf((float)left) + 0x1p-35f) * scale, s[i], rest);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int i = 0; i < ROWS; ++i)
        reinterpret_cast<_Float16*>(pieces)[((i & 3) * 16 + r) * 8 + 4 * k + ((row0 + i) >> 2)] = h[k][i];
    one = over_rows(one, add);
    two = over_rows(two, add);
    cs = over_rows(cs, add);
    rest = over_rows(rest, add);
    cs = fminf(cs, __builtin_sqrtf(two) * __builtin_sqrtf(total[c]));
    const float dropped = least[c] > 0.f ? 0.f : 4.1e-6f * __builtin_sqrtf(top[c]);
    // (2 % for the rounding of these sums themselves)
    const float re = 1.02f * (0x1p-24f * (kRoundings * cs + 6.f) + rest);
    const float ae = 1.02f * (0x1p-24f * kRoundings * one * dropped + scale * 0x1p-18f);
    soft = soft && re + 32.f * ae <= kHardEps;   // all of the block's rows; false for a NaN (a block that holds one)
    rel = fmaxf(rel, re);
    abs = fmaxf(abs, ae);
    if (row0 == 0) scales[r] = scale;
  }
  rel = over_columns(rel, most);
  abs = over_columns(abs, most);
  const float all_soft = -over_columns(soft ? -1.f : 0.f, most);
  if (row0 == 0 && (lane & 7) == 0) {
    scales[16] = rel;
    scales[17] = abs;
    scales[18] = all_soft != 0.f ? 0.f : 1.f;
  }
}

// The eigen-solver of a call of thousands of blocks: ROWS / 2 blocks per wave (eight at ROWS = 16:
// every rotation is derived once, no sum crosses lanes, nothing touches LDS in the sweeps).  Reads the
// Gram matrices and writes W, the eigenvalues and FastProject's constants behind them, the small tensors into the cache, the
// blocks' status words.
// Bound by instruction issue in its sweeps; what comes before and after them is a burst of all waves at once, bound by requests:
// a lane's rows lie 64 bytes apart from its neighbour's, and from the registers they would take an instruction of 64 lines for
// every 16 bytes.  They pass through LDS and cross as they lie in memory, 1 KB an instruction.
// 14720 blocks, eight a wave: 87 us, 99 with four a wave, factors stored from the registers and selects by VCC.  Tried: four
// columns a lane (the same pairs and bits, a third of the exchanges, 2 x 1260 instead of 2 x 1440 instructions a sweep of
// eight blocks): 94, too few waves to cover one another's waits.
// Workgroups of four waves, so that the waves spread evenly over the SIMDs.
constexpr int kSolveWaves = 4;
constexpr int kFactorBytes = (16 * 16 + 16) * 8;             // a block's place in LDS: W and the eigenvalues
static_assert(kFactorBytes == (kFastPieces - 16 * 16) * 8 && kFactorBytes >= kFastBytes, "a block's place in LDS");
template <int ROWS, bool PAIR, bool FAST>
__device__ __forceinline__ void solve16(const dq_format& fmt, const dq_cache& cache, const CompressJob& job, float* __restrict__ large_ws,
                                        int32_t* __restrict__ unit_status, int n_groups, unsigned char (*s_stage)[kFactorBytes]) {
  constexpr int LPB = 128 / ROWS, BPW = 64 / LPB, BPG = kSolveWaves * BPW;   // lanes per block, blocks per wave and workgroup
  constexpr int j1 = 16, d = PAIR ? 64 : 128;
  const Geometry g = make_geometry(fmt, cache.kv_heads, cache.block_capacity);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, blk = threadIdx.x / LPB, j = lane & 7;
  unsigned char* const stage = s_stage[blk];
  const int gi = blockIdx.x * BPG + blk;
  int unit = min(gi, n_groups - 1);
  const int unit_gap = 2 * job.n_blocks;
  if (PAIR) {
    const int pb = unit >> 1, jb = pb % job.n_blocks, hp = pb / job.n_blocks, half_h = g.H >> 1;
    unit = (((hp / half_h) * g.H + 2 * (hp % half_h)) * job.n_blocks + jb) * 2 + (unit & 1);
  }
  const UnitRef ur = unit_ref(g, job, unit);
  const bool live = gi < n_groups && ur.slot >= 0;
  // A wave none of whose blocks is live has nothing to solve (without this it swept four times over
  // zeros: an append that fills no tail, 1280 blocks, 38 us with that, 19 without).
  if (!__any(live)) {
    if (gi < n_groups && lane % LPB == 0) {
      unit_status[unit] = 0;
      if (PAIR) unit_status[unit + unit_gap] = 0;
    }
    return;
  }
  // the wave's b-th block: its part of the workspace (a block that is skipped has no matrix)
  auto there = [&](int b) __attribute__((always_inline)) { return __builtin_amdgcn_readlane((int)live, b * LPB) != 0; };
  auto region = [&](int b) __attribute__((always_inline)) {
    return reinterpret_cast<unsigned char*>(large_ws + (long)__builtin_amdgcn_readlane(unit, b * LPB) * g.Tb * d);
  };
  Jacobi16<ROWS> jac;
  const int row0 = jac.first_row(lane);
  {
    u32x4 x[2 * BPW];
#pragma unroll
    for (int b = 0; b < BPW; ++b) {
      const bool any = there(b);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        x[2 * b + k] = u32x4{0u, 0u, 0u, 0u};
        if (any) x[2 * b + k] = *reinterpret_cast<const u32x4*>(region(b) + 1024 * k + 16 * lane);
      }
    }
#pragma unroll
    for (int b = 0; b < 2 * BPW; ++b) *reinterpret_cast<u32x4*>(s_stage[BPW * wave + b / 2] + 1024 * (b & 1) + 16 * lane) = x[b];
    team_barrier<1>();
    const double* const G = reinterpret_cast<const double*>(stage);
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {   // (symmetric: column j is row j)
      jac.x[i] = G[j * j1 + row0 + i];
      jac.y[i] = G[(j + 8) * j1 + row0 + i];
    }
    team_barrier<1>();
  }
  const int sweeps = jac.template run<PAIR>();
  int px, py;
  double rx, ry, lx, ly;
  jac.template order<PAIR>(reinterpret_cast<double*>(stage), px, py, rx, ry, lx, ly);
  team_barrier<1>();
  // `bytes` of every block, from its place in LDS to `at` bytes behind its Gram matrix' begin
  auto flush = [&](int bytes, int at) __attribute__((always_inline)) {
    team_barrier<1>();
#pragma unroll 1
    for (int b = 0; b < BPW; ++b) {
      if (!there(b)) continue;
      unsigned char* const to = region(b) + at;
      for (int i = 16 * lane; i < bytes; i += 16 * 64)
        *reinterpret_cast<u32x4*>(to + i) = *reinterpret_cast<const u32x4*>(s_stage[BPW * wave + b] + i);
    }
    team_barrier<1>();
  };
  const double fx = rx * rx * rx, fy = ry * ry * ry;
  double wx[ROWS], wy[ROWS];   // columns px and py of W^T
  {
    double* const to = reinterpret_cast<double*>(stage);
    to[j1 * j1 + px] = lx;
    to[j1 * j1 + py] = ly;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      wx[i] = rx > 0.0 ? jac.x[i] * fx : 0.0;
      wy[i] = ry > 0.0 ? jac.y[i] * fy : 0.0;
      to[px * j1 + row0 + i] = wx[i];
      to[py * j1 + row0 + i] = wy[i];
    }
  }
  flush(kFactorBytes, j1 * j1 * 8);
  if constexpr (FAST) {
    store_fast_factors<ROWS, PAIR>(jac, wx, wy, px, py, lx, ly, stage);
    flush(kFastBytes, kFastPieces * 8);
  }
  bool sat = false;
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    const int b1 = row0 + i;
    auto put = [&](int r, double ts) __attribute__((always_inline)) {
      uint16_t* const to = reinterpret_cast<uint16_t*>(stage);
      if (PAIR) {   // the heads' 8 x 8 tensors one after the other; across heads there is nothing
        if ((b1 >> 3) != (r >> 3)) return;
        to[(b1 >> 3) * 64 + (ur.which ? (b1 & 7) * 8 + (r & 7) : (r & 7) * 8 + (b1 & 7))] = f64_to_f16_rne(ts, true, &sat);
      } else {      // values: [b1][r]; keys: transposed [r][b1]
        to[ur.which ? b1 * j1 + r : r * j1 + b1] = f64_to_f16_rne(ts, true, &sat);
      }
    };
    put(px, wx[i] * lx);   // T_S = U Sigma = W Lambda
    put(py, wy[i] * ly);
  }
  team_barrier<1>();
  const unsigned long long sat_lanes = __ballot(sat);
  if (live) {
    const int lb = lane % LPB;
    uint16_t* const small = (ur.which ? cache.v_small : cache.k_small) + (ur.bh * g.NB + ur.slot) * g.small_per_block;
    constexpr int CHUNKS = (PAIR ? 128 : j1 * j1) / 8;   // of eight entries
#pragma unroll
    for (int c = lb; c < CHUNKS; c += LPB) {
      uint16_t* dst = PAIR ? small + (long)(c / 8) * g.NB * g.small_per_block + (c % 8) * 8 : small + c * 8;
      *reinterpret_cast<u32x4*>(dst) = *reinterpret_cast<const u32x4*>(stage + c * 16);
    }
  }
  if (gi < n_groups && lane % LPB == 0) {
    const bool any_sat = ((sat_lanes >> (lane & ~(LPB - 1))) & ((1ull << LPB) - 1)) != 0;
    const int word = live ? (any_sat ? 1 : 0) | (sweeps << 8) : 0;
    unit_status[unit] = word;
    if (PAIR) unit_status[unit + unit_gap] = word;
  }
}

// ROWS / 2 blocks a wave, half as many where at most `few` of the call's blocks (pairs of them) are live: the host, which sees
// neither the slots nor the lengths, launches workgroups for the latter, and those that are not wanted leave.
template <int ROWS, bool PAIR, bool FAST>
__global__ __launch_bounds__(64 * kSolveWaves, ROWS == 16 ? 2 : 4) void solve16_kernel(dq_format fmt, dq_cache cache, CompressJob job,
                                                     float* __restrict__ large_ws, int32_t* __restrict__ unit_status,
                                                     int n_groups, int few) {
  __shared__ __attribute__((aligned(16))) unsigned char s_stage[kSolveWaves * ROWS / 2][kFactorBytes];
  if constexpr (ROWS > 4) {
    const Geometry g = make_geometry(fmt, cache.kv_heads, cache.block_capacity);
    int live = 0;
    for (int b = threadIdx.x & 63; b < job.batch; b += 64) live += live_blocks(g, job, b);
    live += __builtin_amdgcn_update_dpp(0, live, kDppXor1, 0xF, 0xF, true);
    live += __builtin_amdgcn_update_dpp(0, live, kDppXor2, 0xF, 0xF, true);
    live += __builtin_amdgcn_update_dpp(0, live, kDppXor7, 0xF, 0xF, true);
    live += __builtin_amdgcn_update_dpp(0, live, kDppXor8, 0xF, 0xF, true);
    live = (__builtin_amdgcn_readlane(live, 0) + __builtin_amdgcn_readlane(live, 16)) +
           (__builtin_amdgcn_readlane(live, 32) + __builtin_amdgcn_readlane(live, 48));
    if (live * (PAIR ? g.H : 2 * g.H) <= few) {
      solve16<ROWS / 2, PAIR, FAST>(fmt, cache, job, large_ws, unit_status, n_groups, s_stage);
      return;
    }
    if ((int)blockIdx.x * (kSolveWaves * ROWS / 2) >= n_groups) return;
  }
  solve16<ROWS, PAIR, FAST>(fmt, cache, job, large_ws, unit_status, n_groups, s_stage);
}

// ------------------------------------------------------------------------------------------
// Second cut of the three-tensor form (Eq. 2 with n = 3; factor shapes 1 * (T_b/8) * 8 by
// j1 * j2 * 1).  The first cut left its right factor R[(a2, a3), c'] (orthonormal over r) as fp32
// rows in the workspace.  Regrouped as A[(a2, c'), a3] it is cut again,
//   A = T_2 diag(sigma') V'^T,   T_3[e, a3] = sigma'_e V'[a3, e],   T_2 = A V' diag(1/sigma'),
// through the 8 x 8 Gram matrix A^T A (fp64; the fp32 inputs make every product exact), the same
// Jacobi iteration as the first cut, and a projection that overwrites the eight rows of every run
// a2 in place: row a2*8 + e becomes T_2[., a2, ., e].  One workgroup of four waves per block.
// ------------------------------------------------------------------------------------------
template <int DD>
__global__ __launch_bounds__(256) void split3_kernel(dq_format fmt, dq_cache cache, CompressJob job,
                                                     float* __restrict__ large_ws) {
  constexpr int N = kRun, LD = N + 1;
  const Geometry g = make_geometry(fmt, cache.kv_heads, cache.block_capacity);
  const int unit = blockIdx.x;
  const UnitRef ur = unit_ref(g, job, unit);
  const int which = ur.which, slot = ur.slot;
  const long bh = ur.bh;
  if (slot < 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float* blk = large_ws + (long)unit * g.Tb * DD;
  const int runs = g.Tb / N;

  __shared__ double gpart[4][16 * 16];
  __shared__ double A0[N * LD], A1[N * LD], V0[N * LD], V1[N * LD], W3[N * N];
  __shared__ double rc[N], rs[N], lam[N], sigma[N];
  __shared__ int partner[N], is_p[N], order[N];

  // ---- Gram matrix on the fp64 matrix cores: a 16 x 16 product of two runs side by side, whose
  // two diagonal 8 x 8 blocks are the runs' contributions.  Lane (n, k): row a2 = 2*pair + n/8,
  // token a3 = n % 8, elements c' = 16*S + 4*k + j for the j-th of four successive products.
  {
    const int n = lane & 15, k = lane >> 4;
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int pair = wave; pair < runs / 2; pair += 4) {
      const float* row = blk + (long)((2 * pair + (n >> 3)) * N + (n & 7)) * DD + 4 * k;
      float4 v[DD / 16];
#pragma unroll
      for (int S = 0; S < DD / 16; ++S) v[S] = *reinterpret_cast<const float4*>(row + 16 * S);
#pragma unroll
      for (int S = 0; S < DD / 16; ++S) {
        const double x0 = v[S].x, x1 = v[S].y, x2 = v[S].z, x3 = v[S].w;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, x0, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, x1, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x2, x2, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x3, x3, acc, 0, 0, 0);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) gpart[wave][(k + 4 * i) * 16 + n] = acc[i];
  }
  __syncthreads();
  if (tid < N * N) {
    const int p = tid >> 3, q = tid & 7;
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < 4; ++w) s += gpart[w][p * 16 + q] + gpart[w][(p + 8) * 16 + q + 8];   // fixed order
    A0[p * LD + q] = s;
    V0[p * LD + q] = (p == q) ? 1.0 : 0.0;
  }
  __syncthreads();
  // ---- wave 0 alone: Jacobi, ordering, T_3.  A wave's LDS operations execute in order, so
  // inside it a compiler barrier (no hardware one) separates the steps. ----
  if (wave == 0) {
    double trace = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i) trace += A0[i * LD + i];
    const double floor_abs = 1e-17 * trace;
    // parallel cyclic Jacobi: 7 rounds of 4 disjoint rotations per sweep
    double* Ac = A0; double* An = A1; double* Vc = V0; double* Vn = V1;
    constexpr int NM1 = N - 1;
    for (int sweep = 0; sweep < 16; ++sweep) {
      bool any_big = false;
      for (int round = 0; round < NM1; ++round) {
        bool big = false;
        if (lane < N / 2) {
          int p, q;
          if (lane == 0) { p = NM1; q = round; }
          else { p = (round + lane) % NM1; q = (round - lane + NM1) % NM1; }
          if (p > q) { const int t = p; p = q; q = t; }
          double c, sn;
          jacobi_rotation(Ac[p * LD + p], Ac[q * LD + q], Ac[p * LD + q], floor_abs, c, sn, big);
          rc[p] = c; rs[p] = sn; rc[q] = c; rs[q] = sn;
          partner[p] = q; partner[q] = p;
          is_p[p] = 1; is_p[q] = 0;
        }
        any_big = any_big || __any(big);
        __builtin_amdgcn_wave_barrier();
        // J[p][p] = c, J[p][q] = s, J[q][p] = -s, J[q][q] = c per pair;  A' = J^T A J,  V' = V J
        {
          const int i = lane >> 3, j = lane & 7;
          const int pi = partner[i], pj = partner[j];
          const double cj = rc[j], sj = is_p[j] ? -rs[j] : rs[j];
          const double ci = rc[i], si = is_p[i] ? -rs[i] : rs[i];
          const double aj_i = Ac[i * LD + j] * cj + Ac[i * LD + pj] * sj;
          const double aj_pi = Ac[pi * LD + j] * cj + Ac[pi * LD + pj] * sj;
          An[i * LD + j] = ci * aj_i + si * aj_pi;
          Vn[i * LD + j] = Vc[i * LD + j] * cj + Vc[i * LD + pj] * sj;
        }
        __builtin_amdgcn_wave_barrier();
        double* t = Ac; Ac = An; An = t;
        t = Vc; Vc = Vn; Vn = t;
      }
      if (!any_big) break;   // no rotated entry was above 3e-5 of its diagonal pair: this sweep finished them
    }

    // singular values in descending order, T_3, and W3[e][a3] = V'[a3, e] / sigma'_e
    if (lane < N) lam[lane] = Ac[lane * LD + lane];
    __builtin_amdgcn_wave_barrier();
    if (lane < N) {
      int rank = 0;
      const double me = lam[lane];
      for (int s2 = 0; s2 < N; ++s2) rank += (lam[s2] > me) || (lam[s2] == me && s2 < lane);
      order[rank] = lane;
    }
    __builtin_amdgcn_wave_barrier();
    if (lane < N) {
      const double lmax = fmax(lam[order[0]], 0.0);
      const double l = lam[order[lane]];
      sigma[lane] = (l > 1e-12 * lmax && l > 0.0) ? sqrt(l) : 0.0;
    }
    __builtin_amdgcn_wave_barrier();
    {
      const int e = lane >> 3, a3 = lane & 7;
      const double v = Vc[a3 * LD + order[e]];
      const double sg = sigma[e];
      W3[e * N + a3] = sg > 0.0 ? v / sg : 0.0;
      const long b3 = ((long)bh * g.NB + slot) * (N * N);
      const uint16_t hb = f64_to_f16_rne(v * sg, true, nullptr);   // |T_3| <= sqrt(j1): far inside fp16
      if (which) cache.v_small3[b3 + e * N + a3] = hb;   // values: natural [e][a3]
      else cache.k_small3[b3 + a3 * N + e] = hb;         // keys: transposed [a3][e]
    }
  }
  __syncthreads();

  // ---- projection in place: a thread owns one (a2, c') column of eight rows ----
  for (int idx = tid; idx < runs * DD; idx += 256) {
    const int a2 = idx / DD, c = idx % DD;
    float* col = blk + (long)a2 * N * DD + c;
    double x[N];
#pragma unroll
    for (int a3 = 0; a3 < N; ++a3) x[a3] = (double)col[a3 * DD];
#pragma unroll
    for (int e = 0; e < N; ++e) {
      double y = 0.0;
#pragma unroll
      for (int a3 = 0; a3 < N; ++a3) y = fma(W3[e * N + a3], x[a3], y);
      col[e * DD] = (float)y;
    }
  }
}

}  // namespace dq

// ------------------------------------------------------------------------------------------
// C ABI
// ------------------------------------------------------------------------------------------
using namespace dq;

static size_t compress_workspace_bytes(const dq_format* fmt, int batch, int kv_heads, int n_blocks) {
  // header (status words), the fp32 large tensors, one status word per block
  const size_t units = (size_t)batch * kv_heads * 2 * n_blocks;
  return (size_t)kWsHeaderBytes + units * fmt->block_tokens * fmt->head_dim * sizeof(float) +
         align_up(units * sizeof(int32_t), 256);
}

extern "C" size_t dq_compress_workspace_bytes(const dq_format* fmt, int32_t batch, int32_t kv_heads) {
  if (!format_ok(fmt) || batch <= 0 || kv_heads <= 0) return 0;
  return compress_workspace_bytes(fmt, batch, kv_heads, 1);
}

extern "C" size_t dq_compress_blocks_workspace_bytes(const dq_format* fmt, int32_t batch, int32_t kv_heads,
                                                     int32_t t_new) {
  if (!format_ok(fmt) || batch <= 0 || kv_heads <= 0 || t_new < 1) return 0;
  const int n_blocks = (t_new + fmt->block_tokens - 1) / fmt->block_tokens;
  if ((long)batch * kv_heads * 2 * n_blocks > (long)kMaxCompressUnits) return 0;
  return compress_workspace_bytes(fmt, batch, kv_heads, n_blocks);
}

extern "C" int32_t dq_quantize_pack(const dq_format* fmt, const float* t_large, int64_t n_rows,
                                    int32_t value_layout, uint8_t* codes, uint16_t* scales,
                                    void* hip_stream) {
  if (!format_ok(fmt) || !t_large || !codes || !scales) return DQ_EINVAL;
  if (n_rows < 0 || n_rows % kTileTokens) return DQ_EINVAL;
  if (n_rows == 0) return DQ_OK;
  hipStream_t st = (hipStream_t)hip_stream;
  const int tiles = (int)(n_rows / kTileTokens);
  const size_t lds = quantize_lds_bytes(fmt->head_dim, fmt->bits);
  const int d = fmt->head_dim, G = fmt->group, j1 = fmt->j1, j2 = fmt->j2;
#define DQ_LAUNCH_QPACK(B_, D_)                                                                                  \
  do {                                                                                                           \
    if (fmt->levels)                                                                                             \
      hipLaunchKernelGGL((quantize_pack_kernel<B_, D_, true>), dim3(tiles), dim3(256), lds, st, t_large, G, j1,  \
                         j2, value_layout, codes, scales);                                                       \
    else                                                                                                         \
      hipLaunchKernelGGL((quantize_pack_kernel<B_, D_, false>), dim3(tiles), dim3(256), lds, st, t_large, G, j1, \
                         j2, value_layout, codes, scales);                                                       \
  } while (0)
  if (d == 128) {
    if (fmt->bits == 2) DQ_LAUNCH_QPACK(2, 128);
    else if (fmt->bits == 4) DQ_LAUNCH_QPACK(4, 128);
    else DQ_LAUNCH_QPACK(8, 128);
  } else {
    if (fmt->bits == 2) DQ_LAUNCH_QPACK(2, 64);
    else if (fmt->bits == 4) DQ_LAUNCH_QPACK(4, 64);
    else DQ_LAUNCH_QPACK(8, 64);
  }
#undef DQ_LAUNCH_QPACK
  DQ_HIP_CHECK(hipGetLastError());
  return DQ_OK;
}

// Waves per block of the tuned decomposition kernel for a launch of `groups` workgroups (0: the
// three launches of a prompt).  The two contractions and the quantizer shrink with the waves, the
// solver runs in one of them; beyond two workgroups per compute unit the waves of different blocks
// queue for the SIMDs.  Measured, us per call with four / two waves (4-bit, d = 128): 256 blocks
// 30 / 38, 512 blocks 40 / 51, 768 blocks 63 / 53, 1024 blocks 76 / 61.
static int waves_per_block(int groups, int want_waves) {
  if (want_waves) return want_waves == 1 ? 0 : want_waves;
  return groups <= 512 ? 4 : groups <= 1024 ? 2 : 0;
}

// Blocks per wave of the eigen-solver's launch: two up to kMostTwoBlocks blocks, four up to kMostFourBlocks, eight beyond.  More
// blocks share a wave's instructions, fewer give more waves, and the launch takes whole rounds of the chip's 1024 SIMDs: the
// lines lie where a SIMD would get a second wave of two blocks, and a fourth of four.
// Whole call in us, 4 bits, two / four blocks per wave: 2048 blocks 63.9 / 71.8, 3072 95.5 / 87.9, 4096 111.0 / 106.8, graded over
// three decades 207 / 193; four / eight: 4096 107 / 127, 8192 184.1 / 185.5, 9216 228 / 242, 12288 271 / 286, 14720 326.7 / 320.3, graded
// 669 / 657, 32768 665 / 648; 8192 pairs of heads 210 / 214, 16384 401 / 398.
// Where most sequences are skipped, the chain of one wave is what counts: the launch alone for 16384 blocks, four / eight a wave, one
// sequence of sixteen left 30.6 / 47, four 53 / 50, eight 71 / 53.  A launch of eight (four) a wave takes four (two) where at most
// kFewFourBlocks (kFewTwoBlocks) are live, seven eighths of a wave a SIMD: the waves that are left do not spread evenly.  3328 of 14336
// live: 79.7 us, 50.6 so, whole call 200 and 161; 1536 of 3072 78.2 and 71.5; where all are live the count costs 0.4.
constexpr int kMostTwoBlocks = 2048, kMostFourBlocks = 12288, kFewTwoBlocks = 1792, kFewFourBlocks = 3584;

// Blocks (of sixteen rows of channels: pairs of 64-channel heads count once) up to which the Gram matrices' launch requests
// its rows with plain loads: the projection then finds them in the 256 MB last-level cache, 32 KB a block (kMostCachedFast: 2- and
// 4-bit codes).  Where the rows do not fit, or the fp32 rows, 64 KB a block, displace them (kMostCached: kept large tensors;
// 8 bits and three tensors, bound by instructions, gain nothing), loads that pass the caches by are faster.  Whole call in us,
// non-temporal / plain: 4 bits, 2048 blocks 70.0 / 67.2, 4096 126 / 115, 8192 214 / 202, 9216 254 / 249, 13312 324 / 324, 14720
// 339 / 346; 4096 pairs 142 / 128; large tensors kept, 2048 blocks 138 / 128, 3072 199 / 211; 8 bits, 1152 blocks 83.1 /
// 82.7, 8192 285 / 300.
constexpr int kMostCachedFast = 8192, kMostCached = 2048;

// Workgroups of a prompt's projection (2 or 4 bits) that request their rows in the matrix cores' order: of these four fit a
// SIMD, of those that turn their rows in LDS three, which takes launches of more than 2816 in two rounds instead of one.  It
// matters where many tokens are settled in fp64 and a wave takes long; the rows still come from the last-level cache (see
// kMostCachedFast), whose lines are asked for four times in this order.  Whole call in us, turned / direct, blocks with outlier
// channels and blocks graded over three decades, 4 bits: 2048 blocks 67.6 / 69.4 and 125 / 128, 2816 85.1 / 87.0 and 166 / 167, 2944
// 87.4 / 88.9 and 191 / 165, 4096 105 / 108 and 228 / 195, 5120 137 / 132 and 287 / 264, 6144 153 / 153 and 322 / 289, 7168 166 / 175
// and 357 / 323, 14720 315 / 354 and 630 / 604; 2 bits 2944 86.5 / 89.4 and 161 / 161, 4096 106 / 108 and 200 / 190, 5120 140 / 134 and
// 261 / 258, 7168 168 / 172 and 326 / 314; pairs of heads, 4 bits, 4096 121 / 128 and 213 / 187, 5120 154 / 154 and 259 / 247, 2 bits 4096 120 / 124
// and 186 / 183.
constexpr int kLeastDirect = 2817, kMostDirect = 6144;

// LDS that the projection of pairs of heads (2 or 4 bits) is given beyond what it uses from 6145 workgroups on, to hold six of them
// per compute unit instead of the twelve its registers would let in: more rows on their way are slower, not faster.  Whole call
// without / with, outlier channels: 8192 pairs 212 / 205 us in 4 bits, 212 / 206 in 2; 14720 pairs 370 / 362 and 364 / 353; 32768
// 763 / 742 and 763 / 725.  Blocks graded over three decades, most of whose tokens are settled in fp64, lose by it: 8192 pairs 356 / 442 and
// 329 / 432, 14720 581 / 745 and 557 / 727.
static size_t prompt_projection_pad(int groups, bool pair_heads, int bits) {
  if (groups <= kMostDirect || !pair_heads || bits == 8) return 0;
  const size_t used = 128 * (16 * bits + 4) + 4096 + 1024;
  return 160 * 1024 / 6 > used ? 160 * 1024 / 6 - used : 0;
}

static int32_t compress_impl(const dq_format* fmt, dq_cache* cache, const uint16_t* k_new,
                             const uint16_t* v_new, int32_t t_new, int n_blocks, const int32_t* blk_idx,
                             const int32_t* n_valid, void* workspace, size_t workspace_bytes, uint32_t flags,
                             void* hip_stream) {
  if (!cache->k_codes || !cache->k_scales || !cache->k_small || !cache->v_codes || !cache->v_scales ||
      !cache->v_small)
    return DQ_EINVAL;
  if (fmt->i3 != 1 && (!cache->k_small3 || !cache->v_small3)) return DQ_EINVAL;
  if (cache->batch <= 0 || cache->kv_heads <= 0 || cache->block_capacity <= 0) return DQ_EINVAL;
  if ((long)cache->batch * cache->kv_heads * 2 * n_blocks > (long)kMaxCompressUnits) return DQ_EINVAL;
  const size_t need = compress_workspace_bytes(fmt, cache->batch, cache->kv_heads, n_blocks);
  if (workspace_bytes < need) return DQ_ENOSPACE;
  hipStream_t st = (hipStream_t)hip_stream;
  int32_t* status = reinterpret_cast<int32_t*>(workspace);
  float* large_ws = reinterpret_cast<float*>(reinterpret_cast<char*>(workspace) + kWsHeaderBytes);
  const int units = cache->batch * cache->kv_heads * 2 * n_blocks;
  int32_t* unit_status = reinterpret_cast<int32_t*>(large_ws + (size_t)units * fmt->block_tokens * fmt->head_dim);
  const CompressJob job = {k_new, v_new, t_new, n_blocks, blk_idx, n_valid, (flags & DQ_COMPRESS_NO_LARGE) ? 0 : 1,
                           (flags & kCompressMostlyIdle) ? 1 : 0, cache->batch};
  const size_t dlds = decompose_lds_bytes(fmt->i1 * fmt->j1, fmt->head_dim, fmt->i1);
#define DQ_LAUNCH_DECOMPOSE(J, DD_)                                                                      \
  hipLaunchKernelGGL((decompose_kernel<J, DD_>), dim3(units), dim3(64), dlds, st, *fmt, *cache, job, large_ws, \
                     unit_status)
#define DQ_LAUNCH_DECOMPOSE_I1(J, DD_, I_)                                                               \
  hipLaunchKernelGGL((decompose_kernel<J, DD_, I_>), dim3(units), dim3(64), dlds, st, *fmt, *cache, job, \
                     large_ws, unit_status)
  const bool force_general = (flags & DQ_COMPRESS_PLAIN) != 0;
  const int want_waves = (int)((flags >> 8) & 0xFu);   // 0: the library's choice
  // heads of 64 channels with j1 = 8 go through the same kernel two at a time
  const bool pair_heads = fmt->head_dim == 64 && fmt->j1 == 8 && (cache->kv_heads & 1) == 0 && fmt->i1 == 1;
  // Where the caller does not need the fp32 large tensors the decomposition kernel quantizes them
  // itself, which saves their trip through memory (four times the bytes the method needs) and the
  // quantizer's launch.  Calls of a few hundred blocks are bound by the latency of one block's chain
  // and give a block several waves; calls of more than 1024 blocks are bound by throughput and take
  // three launches.
  const bool fused = (flags & DQ_COMPRESS_NO_LARGE) && fmt->i3 == 1 && fmt->i1 == 1 && !force_general &&
                     ((fmt->head_dim == 128 && fmt->j1 == 16 && (fmt->group == 128 || fmt->group == 64)) ||
                      (pair_heads && fmt->group == 64));
  // Three local tensors (d = 128, j1 = 16): the last of the three launches makes the second cut and quantizes, and leaves the fp32 rows of T_2 in the workspace if the caller wants them.  It is one wave
  // per block, so a call of a few hundred blocks, which is bound by the latency of one block's
  // chain, keeps the three launches (first cut with several waves per block, second cut,
  // quantizer); larger calls, and a forced wave count of one, take the one-kernel build.
  const bool fused3 = fmt->i3 == kRun && fmt->i1 == 1 && !force_general && fmt->head_dim == 128 && fmt->j1 == 16 &&
                      (fmt->group == 128 || fmt->group == 64) && (want_waves == 1 || (want_waves == 0 && units > 512));
  // The first two launches of a call of thousands of blocks: Gram matrices, eigen-solver.  `fast`: the fp16 projection follows and wants its constants.
  auto launch_factor = [&](bool fast) {
    const int groups = pair_heads ? units / 2 : units;
    const bool cached = groups <= (fast ? kMostCachedFast : kMostCached);
#define DQ_LAUNCH_GRAM(P_, C_)                                                                                       \
  hipLaunchKernelGGL((decompose16_kernel<1, P_, 0, false, 1, false, C_>), dim3(groups), dim3(64), 0, st, *fmt, *cache, \
                     job, large_ws, unit_status, (int32_t*)nullptr)
    if (pair_heads && cached) DQ_LAUNCH_GRAM(true, true);
    else if (pair_heads) DQ_LAUNCH_GRAM(true, false);
    else if (cached) DQ_LAUNCH_GRAM(false, true);
    else DQ_LAUNCH_GRAM(false, false);
#undef DQ_LAUNCH_GRAM
    // (workgroups for half as many blocks a wave, see solve16_kernel)
    constexpr int kFewPerGroup16 = kSolveWaves * 4, kFewPerGroup8 = kSolveWaves * 2, kFewPerGroup4 = kSolveWaves * 2;
#define DQ_LAUNCH_SOLVE(R_, P_, F_)                                                                               \
  hipLaunchKernelGGL((solve16_kernel<R_, P_, F_>), dim3((groups + kFewPerGroup##R_ - 1) / kFewPerGroup##R_),      \
                     dim3(64 * kSolveWaves), 0, st, *fmt,                                                         \
                     *cache, job, large_ws, unit_status, groups, R_ == 16 ? kFewFourBlocks : kFewTwoBlocks)
#define DQ_LAUNCH_SOLVE_F(R_, P_)          \
  do {                                     \
    if (fast) DQ_LAUNCH_SOLVE(R_, P_, true); \
    else DQ_LAUNCH_SOLVE(R_, P_, false);   \
  } while (0)
    if (groups > kMostFourBlocks) {
      if (pair_heads) DQ_LAUNCH_SOLVE_F(16, true);
      else DQ_LAUNCH_SOLVE_F(16, false);
    } else if (groups > kMostTwoBlocks) {
      if (pair_heads) DQ_LAUNCH_SOLVE_F(8, true);
      else DQ_LAUNCH_SOLVE_F(8, false);
    } else {
      if (pair_heads) DQ_LAUNCH_SOLVE_F(4, true);
      else DQ_LAUNCH_SOLVE_F(4, false);
    }
#undef DQ_LAUNCH_SOLVE_F
#undef DQ_LAUNCH_SOLVE
  };
  if (fused3) {
    launch_factor(false);
#define DQ_LAUNCH_FUSED3(B_)                                                                                     \
  do {                                                                                                           \
    if (fmt->levels)                                                                                             \
      hipLaunchKernelGGL((decompose16_kernel<1, false, B_, true, 3, true>), dim3(units), dim3(64), 0, st, *fmt,  \
                         *cache, job, large_ws, unit_status, status);                                            \
    else                                                                                                         \
      hipLaunchKernelGGL((decompose16_kernel<1, false, B_, false, 3, true>), dim3(units), dim3(64), 0, st,       \
                         *fmt, *cache, job, large_ws, unit_status, status);                                      \
  } while (0)
    if (fmt->bits == 2) DQ_LAUNCH_FUSED3(2);
    else if (fmt->bits == 4) DQ_LAUNCH_FUSED3(4);
    else DQ_LAUNCH_FUSED3(8);
#undef DQ_LAUNCH_FUSED3
    DQ_HIP_CHECK(hipGetLastError());
    return DQ_OK;
  }
  if (fused) {
#define DQ_LAUNCH_FUSED(N_, B_)                                                                                 \
  do {                                                                                                          \
    if (pair_heads && fmt->levels)                                                                              \
      hipLaunchKernelGGL((decompose16_kernel<N_, true, B_, true>), dim3(units / 2), dim3(64 * N_), 0, st, *fmt, \
                         *cache, job, large_ws, unit_status, status);                                           \
    else if (pair_heads)                                                                                        \
      hipLaunchKernelGGL((decompose16_kernel<N_, true, B_, false>), dim3(units / 2), dim3(64 * N_), 0, st,      \
                         *fmt, *cache, job, large_ws, unit_status, status);                                     \
    else if (fmt->levels)                                                                                       \
      hipLaunchKernelGGL((decompose16_kernel<N_, false, B_, true>), dim3(units), dim3(64 * N_), 0, st, *fmt,    \
                         *cache, job, large_ws, unit_status, status);                                           \
    else                                                                                                        \
      hipLaunchKernelGGL((decompose16_kernel<N_, false, B_, false>), dim3(units), dim3(64 * N_), 0, st, *fmt,   \
                         *cache, job, large_ws, unit_status, status);                                           \
  } while (0)
#define DQ_LAUNCH_FUSED_PART3(B_, D_)                                                                              \
  do {                                                                                                          \
    if (pair_heads && fmt->levels)                                                                              \
      hipLaunchKernelGGL((decompose16_kernel<1, true, B_, true, 3, false, D_>), dim3(units / 2), dim3(64), pad, st, *fmt, \
                         *cache, job, large_ws, unit_status, status);                                           \
    else if (pair_heads)                                                                                        \
      hipLaunchKernelGGL((decompose16_kernel<1, true, B_, false, 3, false, D_>), dim3(units / 2), dim3(64), pad, st,      \
                         *fmt, *cache, job, large_ws, unit_status, status);                                     \
    else if (fmt->levels)                                                                                       \
      hipLaunchKernelGGL((decompose16_kernel<1, false, B_, true, 3, false, D_>), dim3(units), dim3(64), pad, st, *fmt,    \
                         *cache, job, large_ws, unit_status, status);                                           \
    else                                                                                                        \
      hipLaunchKernelGGL((decompose16_kernel<1, false, B_, false, 3, false, D_>), dim3(units), dim3(64), pad, st, *fmt,   \
                         *cache, job, large_ws, unit_status, status);                                           \
  } while (0)
    const int fused_groups = pair_heads ? units / 2 : units;
    int fused_waves = waves_per_block(fused_groups, want_waves);
    const size_t pad = prompt_projection_pad(fused_groups, pair_heads, fmt->bits);
    if (fused_waves == 0) {
      launch_factor(fmt->bits != 8);
      const bool direct = fused_groups >= kLeastDirect && fused_groups <= kMostDirect;
      if (fmt->bits == 2 && direct) DQ_LAUNCH_FUSED_PART3(2, true);
      else if (fmt->bits == 2) DQ_LAUNCH_FUSED_PART3(2, false);
      else if (fmt->bits == 4 && direct) DQ_LAUNCH_FUSED_PART3(4, true);
      else if (fmt->bits == 4) DQ_LAUNCH_FUSED_PART3(4, false);
      else DQ_LAUNCH_FUSED_PART3(8, false);
    } else if (fused_waves == 4) {
      if (fmt->bits == 2) DQ_LAUNCH_FUSED(4, 2);
      else if (fmt->bits == 4) DQ_LAUNCH_FUSED(4, 4);
      else DQ_LAUNCH_FUSED(4, 8);
    } else {
      if (fmt->bits == 2) DQ_LAUNCH_FUSED(2, 2);
      else if (fmt->bits == 4) DQ_LAUNCH_FUSED(2, 4);
      else DQ_LAUNCH_FUSED(2, 8);
    }
#undef DQ_LAUNCH_FUSED
#undef DQ_LAUNCH_FUSED_PART3
    DQ_HIP_CHECK(hipGetLastError());
    return DQ_OK;
  }
  if (fmt->i1 > 1) {   // a token factor on the small tensor: the plain kernel on the side i1 * j1
    const int dd = fmt->head_dim, jj = fmt->j1;
    if (fmt->i1 == 2) {
      if (dd == 128 && jj == 16) DQ_LAUNCH_DECOMPOSE_I1(16, 128, 2);
      else if (dd == 128 && jj == 8) DQ_LAUNCH_DECOMPOSE_I1(8, 128, 2);
      else if (dd == 64 && jj == 16) DQ_LAUNCH_DECOMPOSE_I1(16, 64, 2);
      else if (dd == 64 && jj == 8) DQ_LAUNCH_DECOMPOSE_I1(8, 64, 2);
      else return DQ_EINVAL;
    } else {
      if (dd == 128 && jj == 8) DQ_LAUNCH_DECOMPOSE_I1(8, 128, 4);
      else if (dd == 64 && jj == 8) DQ_LAUNCH_DECOMPOSE_I1(8, 64, 4);
      else return DQ_EINVAL;
    }
  } else if (((fmt->head_dim == 128 && fmt->j1 == 16) || pair_heads) && !force_general) {
#define DQ_LAUNCH_D16(N_)                                                                                     \
  do {                                                                                                        \
    if (pair_heads)                                                                                           \
      hipLaunchKernelGGL((decompose16_kernel<N_, true>), dim3(units / 2), dim3(64 * N_), 0, st, *fmt, *cache, \
                         job, large_ws, unit_status, (int32_t*)nullptr);                                      \
    else                                                                                                      \
      hipLaunchKernelGGL((decompose16_kernel<N_, false>), dim3(units), dim3(64 * N_), 0, st, *fmt, *cache,    \
                         job, large_ws, unit_status, (int32_t*)nullptr);                                      \
  } while (0)
    const int groups16 = pair_heads ? units / 2 : units;
    // (a call that mostly skips everything keeps to one launch here: idle, 1280 blocks with groups of 32,
    // 17.7 us against 22.5 with three)
    const int nwv = waves_per_block(groups16, (flags & kCompressMostlyIdle) && groups16 > 1024 ? 2 : want_waves);
    if (nwv == 0) {
      launch_factor(false);
      if (pair_heads)
        hipLaunchKernelGGL((decompose16_kernel<1, true, 0, false, 3>), dim3(units / 2), dim3(64), 0, st, *fmt, *cache,
                           job, large_ws, unit_status, (int32_t*)nullptr);
      else
        hipLaunchKernelGGL((decompose16_kernel<1, false, 0, false, 3>), dim3(units), dim3(64), 0, st, *fmt, *cache,
                           job, large_ws, unit_status, (int32_t*)nullptr);
    } else if (nwv == 4) DQ_LAUNCH_D16(4);
    else DQ_LAUNCH_D16(2);
#undef DQ_LAUNCH_D16
  } else if (fmt->head_dim == 128) {
    if (fmt->j1 == 8) DQ_LAUNCH_DECOMPOSE(8, 128);
    else if (fmt->j1 == 16) DQ_LAUNCH_DECOMPOSE(16, 128);
    else DQ_LAUNCH_DECOMPOSE(32, 128);
  } else {
    if (fmt->j1 == 8) DQ_LAUNCH_DECOMPOSE(8, 64);
    else if (fmt->j1 == 16) DQ_LAUNCH_DECOMPOSE(16, 64);
    else DQ_LAUNCH_DECOMPOSE(32, 64);
  }
#undef DQ_LAUNCH_DECOMPOSE
#undef DQ_LAUNCH_DECOMPOSE_I1
  DQ_HIP_CHECK(hipGetLastError());
  if (fmt->i3 == kRun) {   // three local tensors: cut the right factor again before it is quantized
    if (fmt->head_dim == 128)
      hipLaunchKernelGGL((split3_kernel<128>), dim3(units), dim3(256), 0, st, *fmt, *cache, job, large_ws);
    else
      hipLaunchKernelGGL((split3_kernel<64>), dim3(units), dim3(256), 0, st, *fmt, *cache, job, large_ws);
    DQ_HIP_CHECK(hipGetLastError());
  }
  const int tiles = units * (fmt->block_tokens / kTileTokens);
  const size_t lds = quantize_lds_bytes(fmt->head_dim, fmt->bits);
#define DQ_LAUNCH_QTILES(B_, D_)                                                                              \
  do {                                                                                                        \
    if (fmt->levels)                                                                                          \
      hipLaunchKernelGGL((quantize_tiles_kernel<B_, D_, true>), dim3(tiles), dim3(256), lds, st, large_ws,    \
                         *fmt, *cache, job, unit_status, units, status);                                      \
    else                                                                                                      \
      hipLaunchKernelGGL((quantize_tiles_kernel<B_, D_, false>), dim3(tiles), dim3(256), lds, st, large_ws,   \
                         *fmt, *cache, job, unit_status, units, status);                                      \
  } while (0)
  if (fmt->head_dim == 128) {
    if (fmt->bits == 2) DQ_LAUNCH_QTILES(2, 128);
    else if (fmt->bits == 4) DQ_LAUNCH_QTILES(4, 128);
    else DQ_LAUNCH_QTILES(8, 128);
  } else {
    if (fmt->bits == 2) DQ_LAUNCH_QTILES(2, 64);
    else if (fmt->bits == 4) DQ_LAUNCH_QTILES(4, 64);
    else DQ_LAUNCH_QTILES(8, 64);
  }
#undef DQ_LAUNCH_QTILES
  DQ_HIP_CHECK(hipGetLastError());
  return DQ_OK;
}

extern "C" int32_t dq_compress_kv(const dq_format* fmt, dq_cache* cache, const uint16_t* k_new,
                                  const uint16_t* v_new, int32_t t_new, const int32_t* blk_idx,
                                  const int32_t* n_valid, void* workspace, size_t workspace_bytes,
                                  void* hip_stream) {
  if (!format_ok(fmt) || !cache || !k_new || !v_new || !blk_idx || !workspace) return DQ_EINVAL;
  if (t_new < 1 || t_new > fmt->block_tokens) return DQ_EINVAL;
  return compress_impl(fmt, cache, k_new, v_new, t_new, 1, blk_idx, n_valid, workspace, workspace_bytes,
                       DQ_COMPRESS_KEEP_LARGE, hip_stream);
}

extern "C" int32_t dq_compress_kv_blocks(const dq_format* fmt, dq_cache* cache, const uint16_t* k_new,
                                         const uint16_t* v_new, int32_t t_new, const int32_t* blk_idx,
                                         const int32_t* n_valid, void* workspace, size_t workspace_bytes,
                                         void* hip_stream) {
  if (!format_ok(fmt) || !cache || !k_new || !v_new || !blk_idx || !workspace) return DQ_EINVAL;
  if (t_new < 1) return DQ_EINVAL;
  const int n_blocks = (t_new + fmt->block_tokens - 1) / fmt->block_tokens;
  if (n_blocks > cache->block_capacity) return DQ_EINVAL;
  return compress_impl(fmt, cache, k_new, v_new, t_new, n_blocks, blk_idx, n_valid, workspace,
                       workspace_bytes, DQ_COMPRESS_KEEP_LARGE, hip_stream);
}

namespace dq {
int32_t compress_filled_tails(const dq_format* fmt, dq_cache* cache, const uint16_t* k_tail, const uint16_t* v_tail,
                              const int32_t* blk_idx, void* workspace, size_t workspace_bytes, hipStream_t st) {
  return compress_impl(fmt, cache, k_tail, v_tail, fmt->block_tokens, 1, blk_idx, nullptr, workspace, workspace_bytes,
                       DQ_COMPRESS_NO_LARGE | kCompressMostlyIdle, st);
}
}  // namespace dq

extern "C" int32_t dq_compress_kv_ex(const dq_format* fmt, dq_cache* cache, const uint16_t* k_new,
                                     const uint16_t* v_new, int32_t t_new, const int32_t* blk_idx,
                                     const int32_t* n_valid, void* workspace, size_t workspace_bytes,
                                     uint32_t flags, void* hip_stream) {
  if (!format_ok(fmt) || !cache || !k_new || !v_new || !blk_idx || !workspace) return DQ_EINVAL;
  if (t_new < 1 || (flags & ~(DQ_COMPRESS_NO_LARGE | DQ_COMPRESS_PLAIN | DQ_COMPRESS_WAVES(0xF)))) return DQ_EINVAL;
  {
    const uint32_t wv = (flags >> 8) & 0xFu;
    if (wv != 0 && wv != 1 && wv != 2 && wv != 4) return DQ_EINVAL;
  }
  const int n_blocks = (t_new + fmt->block_tokens - 1) / fmt->block_tokens;
  if (n_blocks > cache->block_capacity) return DQ_EINVAL;
  return compress_impl(fmt, cache, k_new, v_new, t_new, n_blocks, blk_idx, n_valid, workspace,
                       workspace_bytes, flags, hip_stream);
}
