// Host side of the matrix-core decode path: which formats it takes, and the launch.  The kernel
// template lives in dq_decode_mfma_kernel.h; its instantiations are spread over one source file per
// code width so that they compile in parallel.
#include "dq_decode.h"

namespace dq {

// Query heads per kv head that one workgroup takes: four B columns per head and step group of the
// sixteen, so at most 4 (one step group) or 2 (two); the kernel is built for 1, 2 and 4 in a set of columns.  More heads
// are served in groups of that many, the last group taking what is left (7 = 4 + 3); a number that
// is not a power of two takes the next size up (3 heads run in a workgroup built for 4).
static int heads_per_workgroup(const dq_format* f, int rep) {
  const int most = (f->group == 128) ? 4 : 2;
  int r = 1;
  while (r < rep && r < most) r <<= 1;
  return ((rep + r - 1) / r <= kMaxHeadGroups) ? r : 0;
}

// Heads of 64 channels are worked in pairs of neighbouring kv heads (as one head of 128 channels and
// two step groups): j1 = j2 = 8, one step per row, an even number of heads, two local tensors.  One or
// two query heads of each of the two ride in a workgroup (four B columns each); more are served in
// head groups of two, the last one taking what is left.
bool mfma_pair_heads(const dq_format* f, int q_heads, int kv_heads) {
  if (!format_ok(f) || kv_heads <= 0 || q_heads <= 0 || q_heads % kv_heads || (kv_heads & 1)) return false;
  if (q_heads / kv_heads > 2 * kMaxHeadGroups) return false;
  return f->head_dim == 64 && f->j1 == 8 && f->j2 == 8 && f->group == 64 && f->i3 == 1 && f->i1 == 1;
}

// Whether the matrix-core kernel takes a call that leaves the choice to the library.  (Grouped query
// heads of 64 channels are taken here but not where the caller names the kernel: dq_decode_mfma_supported
// and DQ_DECODE_FORCE_MFMA keep the set they were defined with.)
bool mfma_takes(const dq_format* f, int q_heads, int kv_heads) {
  return mfma_supported(f, q_heads, kv_heads) || mfma_pair_heads(f, q_heads, kv_heads);
}

bool mfma_supported(const dq_format* f, int q_heads, int kv_heads) {
  if (!format_ok(f) || kv_heads <= 0 || q_heads <= 0 || q_heads % kv_heads) return false;
  if (f->i1 != 1) return false;   // a token factor on the small tensor: the plain kernel's
  if (q_heads == kv_heads && mfma_pair_heads(f, q_heads, kv_heads)) return true;
  if (f->head_dim != 128 || f->j1 != 16 || f->j2 != 8) return false;
  if (f->bits != 8 && f->bits != 4 && f->bits != 2) return false;
  if (f->group != 128 && f->group != 64) return false;
  return heads_per_workgroup(f, q_heads / kv_heads) > 0;
}

int mfma_head_groups(const dq_format* f, int q_heads, int kv_heads, int* heads_per_group) {
  if (mfma_pair_heads(f, q_heads, kv_heads)) {
    const int per_kv = q_heads / kv_heads, r = per_kv >= 2 ? 2 : 1;
    if (heads_per_group) *heads_per_group = r;
    return (per_kv + r - 1) / r;
  }
  const int rep = q_heads / kv_heads;
  const int r = heads_per_workgroup(f, rep);
  if (heads_per_group) *heads_per_group = r;
  return (rep + r - 1) / r;
}

// Whether the head groups (of four heads, with two step groups of two) go two to a workgroup: the kernel with two sets of columns, for an even
// number of groups, two local tensors and no fp16 tail.  The codes are then requested and unpacked once for both, but a wave's chain over a
// tile is longer and there are half the workgroups, so a launch that leaves the chip part idle loses by it.  The line lies where
// single groups take more than one workgroup a compute unit already (kv heads of all sequences x 8 query heads x tokens, 4 bits: 256 x 8 x
// 512 9.7 us one by one, 8.6 by two; 128 x 8 x 1024: 8.2, 11.3), or there are tiles enough to fill the chip either way (64 x 8 x 32768:
// 64.5, 56; 64 x 8 x 8192: 22.2, 22.8; two step groups 64 x 4 x 16384: 35.0, 32.1; 96 x 4 x 8192: 31.8, 28.1; 128 x 4 x 4096: 20.2,
// 21.0; 8 bits, whose stream, twice through the L2, bounds it sooner: 64 x 8 x 3072: 22.3, 20.7; 64 x 8 x 1024: 12.4, 15.1).  8 bits
// hold one wave a SIMD, so 257 workgroups and more take a second round; with two step groups and up to three tiles one by one was up to
// 5 % faster there up to 400 (136 x 8 x 256: 17.3, 18.0; 208 x 8 x 256, 416 workgroups: 22.6, 19.2).  Over 729 sizes measured in both: none
// slower than one by one by more than 2 %, at most 11 % behind the better of the two.
bool mfma_two_groups(const dq_format* f, int batch, int q_heads, int kv_heads, int max_tiles, bool tail) {
  int per_group = 0;
  const int groups = mfma_head_groups(f, q_heads, kv_heads, &per_group);
  if (tail || mfma_pair_heads(f, q_heads, kv_heads) || per_group != (f->group == 128 ? 4 : 2) || groups % 2 || f->i3 != 1) return false;
  const long units = (long)batch * kv_heads * (groups / 2);
  if (f->bits == 8 && f->group == 64 && max_tiles < 4 && units > 256 && units <= 400) return false;
  return (2 * units > 256 && (max_tiles >= 4 || f->bits == 8)) || units * max_tiles > (f->bits == 8 ? 1024 : f->group == 64 ? 5000 : 8192);
}

// One head of one step group in 8 bits (two tensors): whether scores are joined in registers (SPREAD in dq_decode_mfma_kernel.h) or go through LDS.
// Registers shorten a tile's chain, which counts while a wave has few of them; a launch of more than about 40 tiles a compute unit only waits for
// memory, which answers the requests of SPREAD (a chunk's key rows are every other line) a little slower.  us, in registers / through LDS, codes from HBM:
// 64 units x 32 tiles 18.3 / 18.7, 128 x 55 45.1 / 45.3, 256 x 32 48.5 / 48.7, 256 x 40 (10240) 0.2 % for registers; 440 x 59 149.8 / 148.7, 512 x 64
// 185.5 / 184.5, 200 x 157, lengths from 6000 on, 204.2 / 201.7.  Of 40 sizes measured beyond the line three are slower through LDS, by 0.3 % at most.  (2 bits:
// 440 x 59 39.4 / 38.7, but 512 x 64 49.0 / 49.6 and 256 x 32 15.3 / 15.5: in registers throughout.)
bool mfma_spread(int units, int max_tiles) { return (long)units * max_tiles <= 10240; }

// (for tests)
extern "C" int32_t dq_debug_mfma_spread(int32_t units, int32_t max_tiles) { return mfma_spread(units, max_tiles); }

// defined in dq_decode_mfma_b8.hip, _b4.hip, _b2.hip
int32_t launch_decode_mfma_b8(const DecodeArgs& a, hipStream_t st);
int32_t launch_decode_mfma_b4(const DecodeArgs& a, hipStream_t st);
int32_t launch_decode_mfma_b2(const DecodeArgs& a, hipStream_t st);

int32_t launch_decode_mfma(const DecodeArgs& a, hipStream_t st) {
  const int32_t rc = (a.fmt.bits == 8) ? launch_decode_mfma_b8(a, st)
                     : (a.fmt.bits == 4) ? launch_decode_mfma_b4(a, st) : launch_decode_mfma_b2(a, st);
  if (rc != DQ_OK) return rc;
  DQ_HIP_CHECK(hipGetLastError());
  return DQ_OK;
}

}  // namespace dq
