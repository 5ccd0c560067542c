// Host side of the C ABI: argument checks, workspace carve-up, kernel selection.
#include <atomic>
#include <mutex>

#include "dq_decode.h"

namespace dq {

static std::atomic<int> g_last_hip_error{0};
void set_last_hip_error(hipError_t e) { g_last_hip_error.store((int)e); }

// Waves per SIMD that choose_mfma_shape counts on: what the registers of the 4-wave kernels hold in a launch of several splits (one split
// holds a tail's rows in more of them).  Six kinds of launch are counted with one fewer than they hold.  Five hold three and are counted with two: the estimate takes a third workgroup
// on a compute unit for cheaper than it is, and with three picked finer splits that lost more than others won.  Kernel times, counted with
// two / three: four heads of one step group, 4 bits, 192 units x 64 tiles 36.0 / 45.0 us, 96 x 128 37.5 / 41.8, 2 bits 96 x 128
// 30.4 / 32.8; two heads of two step groups, 4 bits, 96 x 128 37.6 / 40.0, 384 x 32 40.1 / 38.6; pairs of four heads, 2 bits, 160 x 64
// 26.0 / 28.6, 96 x 24 14.4 / 12.4; two heads, three tensors, 2 bits, 160 x 64 27.7 / 30.4, 96 x 24 15.3 / 13.4.  Two heads of one step group in 2 bits
// hold four and are counted with three: 128 x 256 55.1 / 64.6, 392 x 124 83.4 / 89.4 (416 x 152 100 / 107), but 272 x 168 92.0 / 76.4; the 90 of 670 launches
// that differ, measured in both, 1 % slower on average.  (8 bits with two waves where
// one was counted: four heads 96 x 64 49.4 -> 43.8, two heads and a tail 48.8 -> 41.2.)
static int resident_waves(int bits, int heads, bool two_groups, bool three, bool two_sets, bool tail) {
  if (bits == 8) {
    if (two_sets) return 1;
    if (heads == 1) return three && two_groups ? 1 : 2;
    if (heads == 2) return three || (tail && two_groups) ? 1 : 2;
    return three || tail || two_groups ? 1 : 2;   // (four heads; of two step groups: pairs)
  }
  if (two_sets || heads == 4) return 2;
  if (bits == 4) return !three && (heads == 1 || (!tail && !two_groups)) ? 3 : 2;
  if (heads == 1) return three ? 3 : 4;
  if (three) return 2;
  return 3;
}

// (for tests)
extern "C" int32_t dq_debug_resident_waves(int32_t bits, int32_t heads, int32_t two_groups, int32_t three,
                                           int32_t two_sets, int32_t tail) {
  return resident_waves(bits, heads, two_groups != 0, three != 0, two_sets != 0, tail != 0);
}

// Launch shape of the matrix-core kernel: n splits of every (sequence, kv head) unit and nw waves per
// workgroup, the pair with the least estimated time.  The estimate is meant to rank shapes, not to give
// their time; it was fitted to the kernel timestamps of 2302 launches (1 to 640 units, 1 to 256
// tiles of 128 tokens, 2, 4 and 8 bits, one to four heads per workgroup, two and three tensors, with
// and without a tail), each in up to 24 shapes:
//   the busiest compute unit works k = ceil(units n / 256) workgroups, as many at a time as its registers
//   hold, the rest in further rounds;
//   in a round a wave works ceil(tiles / (n nw)) tiles, each of which takes the longer of one wave's
//   chain (requests, unpacking, two contractions, softmax) and the SIMD's issue of all its waves'
//   tiles, which grows with the code width, and something for every wave beside it; a pair of
//   64-channel heads counts a chain 0.2 us shorter than two heads of 128 channels (256 units of 32 tiles
//   in 4 bits: 26.1 us in one split of 4 waves, 27.5 in the 8 waves that are picked without it);
//   every wave on a SIMD and every split (partial, ticket, merge) costs a fixed amount, and so does the
//   tail per wave and per load of its rows;
//   a finer split has to promise 8.6 % to be taken.
// The picks were 0.9 % slower than the fastest shape measured on average, 19 % at worst.  The kernels of several heads have become
// faster since: over 4361 launches of the present ones, 55 formats and options, the picks are 1.1 % slower on average and 31 % at
// worst (160 units of 12 tiles, four heads, 4 bits, a tail: 17.1 us in 3 splits of 4 waves, 13.0 in 1 of 4), 93 of them over 10 %.  All constants
// fitted again to these, with no launch slower than it was, gained 0.04 %.
static void choose_mfma_shape(int units, int max_tiles, int heads, int bits, bool two_groups, bool three, bool pair,
                              bool two_sets, bool tail, int* n_out, int* nw_out) {
  static const int kSplits[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64};
  const int resident = resident_waves(bits, heads, two_groups, three, two_sets, tail);
  const float h = (float)(heads - 1), n3 = three ? 1.f : 0.f;
  // (two sets of columns: fitted by themselves, 276 sizes in three code widths; the picks are 0.25 % behind the fastest
  // shape on average, 7.5 % at worst, and with the constants of the others, extended to eight heads, 0.8 % and 28 %;
  // two step groups, the 74 of 219 sizes that take it: 3.8 % at worst)
  const float chain = two_sets ? 3.623f : 1.955f + 0.626f * h + 2.847f * n3 - (pair ? 0.2f : 0.f);
  const float issue = two_sets ? 1.247f : 0.018f + 0.483f * bits + 0.008f * h + 0.758f * n3;
  const float per_wave = two_sets ? 2.087f : 2.172f + (tail ? 0.024f * (1 + heads) : 0.f);
  float best = 3.0e38f;
  for (const int n : kSplits) {
    if (n > kMaxSplits || n > max_tiles) break;
    // (8-bit codes: a wave's ring of chunks is twice as large and an 8-wave workgroup would run out of
    // registers)
    for (int nw = 4; nw <= (bits == 8 ? 4 : 8); nw += 4) {
      const int tiles = (max_tiles + n * nw - 1) / (n * nw);           // of the busiest wave
      auto round = [&](int groups) -> float {                          // so many workgroups on a compute unit at a time
        if (groups == 0) return 0.f;
        const float waves = 0.25f * (float)(groups * nw);               // per SIMD
        return tiles * (fmaxf(chain, waves * issue) + (two_sets ? 0.911f : 0.289f) * waves) + per_wave * waves + 0.072f;
      };
      const int together = resident * 4 / nw > 1 ? resident * 4 / nw : 1;
      const long per_cu = ((long)units * n + 255) / 256;
      float t = (float)(per_cu / together) * round(together) + round((int)(per_cu % together));
      if (n > 1) t += two_sets ? 2.038f + 0.233f * n : 1.606f + 0.112f * n;
      if (tail) t += 0.136f * (float)((16 + n * nw - 1) / (n * nw));    // (64 rows, four a load)
      if (t < 0.914f * best) { best = t; *n_out = n; *nw_out = nw; }
    }
  }
}

int choose_splits(const dq_format* f, int batch, int q_heads, int kv_heads, int max_seq_len, bool mfma, bool tail,
                  uint32_t flags, int* nw_out, int* head_groups_out, int* heads_per_group_out) {
  const int max_tiles = (max_seq_len + kTileTokens - 1) / kTileTokens;
  int n = 1, nw = 4;
  int per_group = q_heads / kv_heads;
  int hg = mfma ? mfma_head_groups(f, q_heads, kv_heads, &per_group) : 1;   // each head group is a workgroup of its own
  const bool two_sets = mfma && mfma_two_groups(f, batch, q_heads, kv_heads, max_tiles, tail);   // ... or two of them are
  if (two_sets) { hg /= 2; per_group *= 2; }
  if (max_tiles > 0) {
    if (mfma) {
      if (mfma_pair_heads(f, q_heads, kv_heads))   // two kv heads per workgroup
        choose_mfma_shape(batch * kv_heads / 2 * hg, max_tiles, 2 * per_group, f->bits, true, false, true, false, tail, &n, &nw);
      else
        choose_mfma_shape(batch * kv_heads * hg, max_tiles, per_group, f->bits, f->group == 64, f->i3 == kRun, false, two_sets,
                          tail, &n, &nw);
    } else {
      const int units = batch * q_heads;
      n = (2048 + units - 1) / units;
      const int by_len = (max_tiles + 1) / 2;
      if (n > by_len) n = by_len;
    }
  }
  // the caller's overrides (validated by the entry point)
  if (const int v = (int)((flags >> 8) & 0x7Fu)) n = v;
  if (const int v = (int)((flags >> 16) & 0xFu)) nw = v;
  if (n < 1) n = 1;
  if (n > kMaxSplits) n = kMaxSplits;
  if (max_tiles > 0 && n > max_tiles) n = max_tiles;
  *nw_out = nw;
  *head_groups_out = hg;
  *heads_per_group_out = per_group;
  return n;
}

__global__ void fill_zero_kernel(uint4* p, size_t n16) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Each wave reads its own contiguous slice with sixteen 1 KB loads in flight: the access shape
// that gave the highest read rate of the shapes tried on this chip.
__global__ __launch_bounds__(256) void stream_read_kernel(const u32x4* __restrict__ src, size_t n16,
                                                          uint32_t* __restrict__ sink) {
  constexpr int INF = 16;
  const size_t waves = (size_t)gridDim.x * 4;
  const size_t wave = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  // slices are multiples of one load group (INF * 64 elements); what is left over after the
  // slices is dealt out in 64-element pieces
  const size_t group = (size_t)INF * 64;
  const size_t per_wave = (n16 / waves) / group * group;
  const size_t begin = wave * per_wave;
  const size_t end = begin + per_wave;
  u32x4 acc = {0, 0, 0, 0};
  for (size_t i = begin + lane; i < end; i += group) {
    u32x4 v[INF];
#pragma unroll
    for (int k = 0; k < INF; ++k) v[k] = __builtin_nontemporal_load(src + i + k * 64);
#pragma unroll
    for (int k = 0; k < INF; ++k) acc ^= v[k];
  }
  for (size_t i = waves * per_wave + wave * 64 + lane; i < n16; i += waves * 64)
    acc ^= __builtin_nontemporal_load(src + i);
  // a data-dependent store that practically never happens keeps the loads alive
  if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9E3779B9u) {
    sink[0] = acc.x; sink[1] = acc.y; sink[2] = acc.z; sink[3] = acc.w;
  }
}

}  // namespace dq

using namespace dq;

#ifdef DQ_TIMELINE
namespace dq { unsigned long long* g_timeline = nullptr; }
// Instrumented build only: the device buffer ([workgroups * waves, kTimelineSlots] u64, zero-filled by the
// caller) the matrix-core decode kernel's waves stamp their time line into; NULL switches it off.
extern "C" void dq_debug_timeline(void* buffer) { dq::g_timeline = reinterpret_cast<unsigned long long*>(buffer); }
extern "C" int32_t dq_debug_timeline_slots(void) { return dq::kTimelineSlots; }
#endif

extern "C" int32_t dq_version(void) { return 6; }

extern "C" const char* dq_status_string(int32_t status) {
  switch (status) {
    case DQ_OK: return "ok";
    case DQ_EINVAL: return "invalid argument or unsupported format";
    case DQ_ENOSPACE: return "workspace too small";
    case DQ_EHIP: return "HIP runtime error";
    case DQ_ELIMIT: return "sizes beyond the limit of the allocation-free entry point";
    default: return "unknown status";
  }
}

extern "C" int32_t dq_last_hip_error(void) { return g_last_hip_error.load(); }

extern "C" int32_t dq_decode_mfma_supported(const dq_format* fmt, int32_t q_heads, int32_t kv_heads) {
  return mfma_supported(fmt, q_heads, kv_heads) ? 1 : 0;
}

extern "C" size_t dq_decode_workspace_bytes(const dq_format* fmt, int32_t batch, int32_t q_heads,
                                            int32_t kv_heads, int32_t max_seq_len) {
  if (!format_ok(fmt) || batch <= 0 || q_heads <= 0 || kv_heads <= 0 || q_heads % kv_heads ||
      max_seq_len < 0)
    return 0;
  return (size_t)kWsHeaderBytes + decode_counter_bytes(batch, q_heads) +
         decode_partial_bytes(fmt, batch, q_heads);
}

extern "C" int32_t dq_workspace_init(void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!workspace || workspace_bytes % 16 || ((uintptr_t)workspace & 15)) return DQ_EINVAL;
  if (workspace_bytes == 0) return DQ_OK;
  const size_t n16 = workspace_bytes / 16;
  size_t blocks = (n16 + 255) / 256;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)hip_stream,
                     reinterpret_cast<uint4*>(workspace), n16);
  DQ_HIP_CHECK(hipGetLastError());
  return DQ_OK;
}

static int32_t decode_impl(const dq_format* fmt, const dq_cache* cache, const uint16_t* q,
                           int32_t q_heads, const int32_t* seq_lens, int32_t max_seq_len,
                           const dq_tail* tail, float softmax_scale, uint16_t* out, float* out_f32,
                           void* workspace, size_t workspace_bytes, uint32_t flags, void* hip_stream,
                           void* ev_kernel_start, void* ev_kernel_stop) {
  if (!format_ok(fmt) || !cache || !q || !seq_lens || !out || !workspace) return DQ_EINVAL;
  if (!cache->k_codes || !cache->k_scales || !cache->k_small || !cache->v_codes || !cache->v_scales ||
      !cache->v_small)
    return DQ_EINVAL;
  if (fmt->i3 != 1 && (!cache->k_small3 || !cache->v_small3)) return DQ_EINVAL;
  if (cache->batch <= 0 || cache->kv_heads <= 0 || cache->block_capacity <= 0) return DQ_EINVAL;
  if (q_heads <= 0 || q_heads % cache->kv_heads) return DQ_EINVAL;
  if ((long)cache->batch * q_heads > kMaxDecodeRows) return DQ_EINVAL;
  if (max_seq_len < 0 || (long)max_seq_len > (long)cache->block_capacity * fmt->block_tokens) return DQ_EINVAL;
  if ((flags & DQ_DECODE_FORCE_GENERIC) && (flags & DQ_DECODE_FORCE_MFMA)) return DQ_EINVAL;
  {
    const uint32_t splits = (flags >> 8) & 0x7Fu, waves = (flags >> 16) & 0xFu, umap = (flags >> 20) & 0xFu;
    if (flags & ~(3u | DQ_DECODE_SPLITS(0x7F) | DQ_DECODE_WAVES(0xF) | (0xFu << 20))) return DQ_EINVAL;
    if (splits > (uint32_t)kMaxSplits || (waves != 0 && waves != 4 && waves != 8) || umap > 6) return DQ_EINVAL;
  }
  const size_t need = dq_decode_workspace_bytes(fmt, cache->batch, q_heads, cache->kv_heads, max_seq_len);
  if (need == 0) return DQ_EINVAL;
  if (workspace_bytes < need) return DQ_ENOSPACE;
  if (tail && (!tail->k_tail || !tail->v_tail || !tail->tail_lens || tail->capacity < 1 || tail->capacity > kMaxTailRows))
    return DQ_EINVAL;
  const bool can_mfma = mfma_supported(fmt, q_heads, cache->kv_heads);
  if ((flags & DQ_DECODE_FORCE_MFMA) && !can_mfma) return DQ_EINVAL;
  const bool use_mfma = mfma_takes(fmt, q_heads, cache->kv_heads) && !(flags & DQ_DECODE_FORCE_GENERIC);

  DecodeArgs a;
  a.fmt = *fmt;
  a.cache = *cache;
  a.q = q;
  a.q_heads = q_heads;
  a.seq_lens = seq_lens;
  a.max_seq_len = max_seq_len;
  a.scale = softmax_scale > 0.f ? softmax_scale : 1.0f / sqrtf((float)fmt->head_dim);
  a.out = out;
  a.out_f32 = out_f32;
  char* ws = reinterpret_cast<char*>(workspace);
  a.counters = reinterpret_cast<int32_t*>(ws + kWsHeaderBytes);
  a.partials = reinterpret_cast<float*>(ws + kWsHeaderBytes + decode_counter_bytes(cache->batch, q_heads));
  a.n_split = choose_splits(fmt, cache->batch, q_heads, cache->kv_heads, max_seq_len, use_mfma, tail != nullptr, flags, &a.nw,
                            &a.head_groups, &a.heads_per_group);
  // With one workgroup per compute unit and equal shares, a launch ends with its slowest XCD.
  // Dealing the units so that every XCD sees every residue class of them (mod 8) brings the XCDs
  // closer together: measured 4 - 5 % faster on the 256-unit benchmark shapes (4- and 8-bit), neutral
  // or within half a percent either way on the other workloads, where the plain order stays.
  a.pair_heads = (use_mfma && mfma_pair_heads(fmt, q_heads, cache->kv_heads)) ? 1 : 0;
  const int units = cache->batch * cache->kv_heads / (a.pair_heads ? 2 : 1);
  a.unit_map = (a.n_split == 1 && a.head_groups == 1 && units <= 256) ? 3 : 0;
  if (const uint32_t umap = (flags >> 20) & 0xFu) a.unit_map = (int)umap - 1;   // the caller's override
  a.rows_on_x = ((long)cache->batch * q_heads > kMaxGridY) ? 1 : 0;   // rows: at most batch * q_heads of them
  a.n_slots = a.n_split + (tail && !use_mfma ? 1 : 0);   // the matrix-core kernel's waves take the tail along
  if (tail) a.tail = *tail;
  else a.tail = dq_tail{nullptr, nullptr, nullptr, 0};
#ifdef DQ_TIMELINE
  a.timeline = g_timeline;
#endif
  a.ev_start = (hipEvent_t)ev_kernel_start;
  a.ev_stop = (hipEvent_t)ev_kernel_stop;
  hipStream_t st = (hipStream_t)hip_stream;
  return use_mfma ? launch_decode_mfma(a, st) : launch_decode_generic(a, st);
}

// (for tests) How decode_impl would launch these sizes: out = {matrix-core kernel or not, splits, waves, query heads per workgroup}.
extern "C" int32_t dq_debug_decode_shape(const dq_format* fmt, int32_t batch, int32_t q_heads, int32_t kv_heads, int32_t max_seq_len,
                                         int32_t tail, uint32_t flags, int32_t* out) {
  if (!format_ok(fmt) || batch <= 0 || kv_heads <= 0 || q_heads <= 0 || q_heads % kv_heads || max_seq_len < 0 || !out) return DQ_EINVAL;
  const bool mfma = mfma_takes(fmt, q_heads, kv_heads) && !(flags & DQ_DECODE_FORCE_GENERIC);
  int nw = 0, groups = 0, heads = 0;
  out[1] = choose_splits(fmt, batch, q_heads, kv_heads, max_seq_len, mfma, tail != 0, flags, &nw, &groups, &heads);
  out[0] = mfma;
  out[2] = nw;
  out[3] = heads;
  return DQ_OK;
}

extern "C" int32_t dq_attn_decode_timed(const dq_format* fmt, const dq_cache* cache, const uint16_t* q,
                                        int32_t q_heads, const int32_t* seq_lens, int32_t max_seq_len,
                                        float softmax_scale, uint16_t* out, float* out_f32, void* workspace,
                                        size_t workspace_bytes, uint32_t flags, void* hip_stream,
                                        void* ev_kernel_start, void* ev_kernel_stop) {
  return decode_impl(fmt, cache, q, q_heads, seq_lens, max_seq_len, nullptr, softmax_scale, out, out_f32,
                     workspace, workspace_bytes, flags, hip_stream, ev_kernel_start, ev_kernel_stop);
}

extern "C" int32_t dq_attn_decode_tail(const dq_format* fmt, const dq_cache* cache, const uint16_t* q,
                                       int32_t q_heads, const int32_t* seq_lens, int32_t max_seq_len,
                                       const dq_tail* tail, float softmax_scale, uint16_t* out,
                                       float* out_f32, void* workspace, size_t workspace_bytes,
                                       uint32_t flags, void* hip_stream) {
  return decode_impl(fmt, cache, q, q_heads, seq_lens, max_seq_len, tail, softmax_scale, out, out_f32,
                     workspace, workspace_bytes, flags, hip_stream, nullptr, nullptr);
}

extern "C" int32_t dq_attn_decode(const dq_format* fmt, const dq_cache* cache, const uint16_t* q,
                                  int32_t q_heads, const int32_t* seq_lens, int32_t max_seq_len,
                                  float softmax_scale, uint16_t* out, float* out_f32, void* workspace,
                                  size_t workspace_bytes, uint32_t flags, void* hip_stream) {
  return dq_attn_decode_timed(fmt, cache, q, q_heads, seq_lens, max_seq_len, softmax_scale, out, out_f32,
                              workspace, workspace_bytes, flags, hip_stream, nullptr, nullptr);
}

// ---- decode without a workspace argument: for callers that cannot allocate -------------------
// The split partials and tickets live in a file-scope device array.  Every GPU the library runs on
// holds its own copy at its own address, which is looked up once per device; host code uses that
// address only, never the array's name.
constexpr int kStaticMaxPairs = 512;   // (sequence, query head) pairs one call may hold
constexpr size_t kStaticScratchBytes =
    (size_t)kWsHeaderBytes + (size_t)kStaticMaxPairs * sizeof(int32_t) /* tickets, a multiple of 256 */ +
    (size_t)kStaticMaxPairs * (kMaxSplits + 1) * (128 + 2) * sizeof(float);
static_assert(((size_t)kStaticMaxPairs * sizeof(int32_t)) % 256 == 0, "ticket area is a multiple of 256 bytes");
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[kMaxDevices];   // the array's device address, per device; null until looked up

// The current device's copy of the array; on its first use the ticket area is cleared on `st` (a
// small kernel, safe under stream capture).  The kernels leave the tickets at zero afterwards.
static int32_t static_scratch(hipStream_t st, void** out) {
  int dev = -1;
  DQ_HIP_CHECK(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return DQ_EINVAL;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    DQ_HIP_CHECK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return DQ_EHIP;
    const size_t head = (size_t)kWsHeaderBytes + (size_t)kStaticMaxPairs * sizeof(int32_t);
    hipLaunchKernelGGL(fill_zero_kernel, dim3(1), dim3(256), 0, st, reinterpret_cast<uint4*>(ptr), head / 16);
    DQ_HIP_CHECK(hipGetLastError());
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return DQ_OK;
}

extern "C" int32_t dq_attn_decode_static(const dq_format* fmt, const dq_cache* cache, const uint16_t* q,
                                         int32_t q_heads, const int32_t* seq_lens, int32_t max_seq_len,
                                         const dq_tail* tail, float softmax_scale, uint16_t* out,
                                         float* out_f32, uint32_t flags, void* hip_stream) {
  if (!format_ok(fmt) || !cache || cache->batch <= 0 || q_heads <= 0) return DQ_EINVAL;
  if ((long)cache->batch * q_heads > kStaticMaxPairs) return DQ_ELIMIT;
  const size_t need = dq_decode_workspace_bytes(fmt, cache->batch, q_heads, cache->kv_heads, max_seq_len);
  if (need == 0) return DQ_EINVAL;
  if (need > kStaticScratchBytes) return DQ_ELIMIT;
  void* ptr = nullptr;
  const int32_t rc = static_scratch((hipStream_t)hip_stream, &ptr);
  if (rc != DQ_OK) return rc;
  return decode_impl(fmt, cache, q, q_heads, seq_lens, max_seq_len, tail, softmax_scale, out, out_f32, ptr,
                     kStaticScratchBytes, flags, hip_stream, nullptr, nullptr);
}

extern "C" int32_t dq_stream_read(const void* src, size_t bytes, uint32_t* sink, void* hip_stream) {
  if (!src || !sink || bytes % 16 || ((uintptr_t)src & 15)) return DQ_EINVAL;
  if (bytes == 0) return DQ_OK;
  const size_t n16 = bytes / 16;
  size_t blocks = n16 / (16 * 64 * 4);   // at least one full load group per wave
  if (blocks > 1024) blocks = 1024;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(stream_read_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)hip_stream,
                     reinterpret_cast<const u32x4*>(src), n16, sink);
  DQ_HIP_CHECK(hipGetLastError());
  return DQ_OK;
}
