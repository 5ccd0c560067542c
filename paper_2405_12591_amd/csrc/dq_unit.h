// What a compression call works on, and which of the caller's rows a block of it reads.
#pragma once
#include "dq_common.h"

namespace dq {

// What one dq_compress_kv call works on: t_new rows per (sequence, kv head), cut into n_blocks
// blocks of T_b rows (the last one may be short); block j of sequence b goes to slot blk_idx[b] + j.
struct CompressJob {
  const uint16_t* k_new;     // [B, H, t_new, d] fp16 bits
  const uint16_t* v_new;
  int t_new;
  int n_blocks;              // ceil(t_new / T_b)
  const int32_t* blk_idx;    // [B]
  const int32_t* n_valid;    // [B] or null
  int keep_large;            // the one-kernel three-tensor build also leaves its fp32 rows in the workspace
  int mostly_idle;           // most calls skip every sequence (a serving step whose tails rarely fill)
  int batch;
};

// Work unit `unit` = (((b * H + h) * n_blocks) + j) * 2 + which.  slot < 0: nothing to do (sequence
// skipped, slot past the cache's capacity, or a block none of whose rows is valid).
struct UnitRef {
  int which, b, slot, nv;    // nv: valid rows of this block (the rest count as zero)
  long bh;                   // b * H + h
  const uint16_t* X;         // the block's first row; null where there is nothing to do
};
// The address of the rows comes with their number and only from here, so no row is asked for before the lengths are known: rows past the
// valid ones and those of skipped sequences need not be there, and a call that skips most of its sequences does not read them.  (With
// the first rows requested ahead of the lengths a call of 512 blocks took 36.8 us, 37.1 so, one of 3072 pairs of heads 62.5 and 64.7; but one
// that skips 31 of 32 sequences 10.9 and 10.6, and a prompt of 16384 blocks, fifteen sequences of sixteen skipped, 151 and 141.)
__host__ __device__ __forceinline__ UnitRef unit_ref(const Geometry& g, const CompressJob& job, int unit) {
  UnitRef u;
  u.which = unit & 1;
  const int ub = unit >> 1;
  const int j = ub % job.n_blocks;
  u.bh = ub / job.n_blocks;
  u.b = (int)(u.bh / g.H);
  const int first = job.blk_idx[u.b];
  int rows = job.t_new;
  if (job.n_valid) {
    const int valid = job.n_valid[u.b];
    rows = valid < 0 ? 0 : valid < job.t_new ? valid : job.t_new;
  }
  const int left = rows - j * g.Tb;
  u.nv = left < 0 ? 0 : left < g.Tb ? left : g.Tb;
  u.slot = (first < 0 || first + j >= g.NB || u.nv == 0) ? -1 : first + j;
  u.X = u.slot < 0 ? nullptr : (u.which ? job.v_new : job.k_new) + (u.bh * job.t_new + (long)j * g.Tb) * g.d;
  return u;
}

}  // namespace dq
