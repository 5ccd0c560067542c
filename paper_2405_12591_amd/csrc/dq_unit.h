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

__host__ __device__ __forceinline__ int valid_rows(const CompressJob& job, int b) {
  if (!job.n_valid) return job.t_new;
  const int valid = job.n_valid[b];
  return valid < 0 ? 0 : valid < job.t_new ? valid : job.t_new;
}

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
  const int left = valid_rows(job, u.b) - j * g.Tb;
  u.nv = left < 0 ? 0 : left < g.Tb ? left : g.Tb;
  u.slot = (first < 0 || first + j >= g.NB || u.nv == 0) ? -1 : first + j;
  u.X = u.slot < 0 ? nullptr : (u.which ? job.v_new : job.k_new) + (u.bh * job.t_new + (long)j * g.Tb) * g.d;
  return u;
}

// Blocks of sequence b, per head and side, for which unit_ref() has something to do.
__host__ __device__ __forceinline__ int live_blocks(const Geometry& g, const CompressJob& job, int b) {
  const int first = job.blk_idx[b], blocks = (valid_rows(job, b) + g.Tb - 1) / g.Tb, room = g.NB - first;
  return first < 0 || room < 0 ? 0 : blocks < room ? blocks : room;
}

}  // namespace dq
