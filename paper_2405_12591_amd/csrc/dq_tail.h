// The fp16 tail of a sequence (tokens appended since the last compressed block, Section 3.2 of
// arXiv 2405.12591) as one more partial result of the decode step: plain fp32 attention of the
// query heads of one kv head over at most kMaxTailRows rows, computed by one workgroup (TailBlock) or by
// waves on their own (TailWave).
//
// TailBlock (the plain path): a row of D halves is read by D/8 lanes, 16 bytes each, so a wave covers 4
// (D = 128) or 8 (D = 64) whole rows per load; the query heads of the group share every row that is read.
//   issue_keys()  starts the loads of q and of the first batch of key and value rows;
//   finish()      scores, softmax over the rows, weighted sum of the value rows; leaves
//                 out[head][0..D) (unnormalised), out[head][D] = max score in log2 units
//                 (-inf for an empty tail) and out[head][D + 1] = sum of weights in `result`.
#pragma once

#include "dq_decode.h"

namespace dq {

typedef _Float16 tail_h8 __attribute__((ext_vector_type(8)));
typedef uint32_t tail_u4 __attribute__((ext_vector_type(4)));

template <int CTRL>
__device__ __forceinline__ float tail_dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

// D: head dimension.  NWV: waves in the workgroup (all of them must call both functions).
// HEADS: query heads handled together (every row read serves all of them).
template <int D, int NWV, int HEADS>
struct TailBlock {
  static constexpr int LPR = D / 8;      // lanes per row
  static constexpr int RPI = 64 / LPR;   // rows per wave-wide load
  static constexpr int HB = HEADS;
  static constexpr int BATCH = 8;        // row loads a lane keeps in flight
  static constexpr int ROWS_PER_BATCH = BATCH * RPI * NWV;
  // floats of LDS scratch finish() needs, and of the result it leaves
  static constexpr int kScratchFloats = HB * kMaxTailRows + NWV * HB * D + 2 * HB * NWV;
  static constexpr int kResultFloats = HB * (D + 2);

  tail_u4 kreg[BATCH], vreg[BATCH], qraw[HB];
  float qreg[HB][8];
  float qk;
  const uint16_t* kt;
  const uint16_t* vt;
  int lane, wave, chunk, rsub, cap;

  __device__ __forceinline__ int batch_row(int batch, int it) const {
    return batch * ROWS_PER_BATCH + RPI * (wave + NWV * it) + rsub;
  }

  // heads [hq0, hq0 + nh) of sequence b are the query heads of kv head h (nh <= HB)
  __device__ __forceinline__ void issue_keys(const DecodeArgs& a, int b, int h, long hq0, int nh) {
    lane = threadIdx.x & 63; wave = threadIdx.x >> 6;
    chunk = lane % LPR; rsub = lane / LPR;
    cap = a.tail.capacity;
    const int H = a.cache.kv_heads;
    // the lane's 8 halves of a row: kt + row * D
    kt = a.tail.k_tail + ((long)b * H + h) * cap * D + 8 * chunk;
    vt = a.tail.v_tail + ((long)b * H + h) * cap * D + 8 * chunk;
    qk = a.scale * 1.4426950408889634f;
#pragma unroll
    for (int hd = 0; hd < HB; ++hd)
      qraw[hd] = *reinterpret_cast<const tail_u4*>(a.q + ((long)b * a.q_heads + hq0 + min(hd, nh - 1)) * D + 8 * chunk);
    // Rows below the capacity are readable whatever the tail's length, which is not known yet; rows
    // past the capacity read the last row instead.  No branches: the caller may have other loads in
    // flight whose count the compiler has to keep.
#pragma unroll
    for (int it = 0; it < BATCH; ++it)
      kreg[it] = *reinterpret_cast<const tail_u4*>(kt + (long)min(batch_row(0, it), cap - 1) * D);
#pragma unroll
    for (int it = 0; it < BATCH; ++it)
      vreg[it] = *reinterpret_cast<const tail_u4*>(vt + (long)min(batch_row(0, it), cap - 1) * D);
  }

  __device__ __forceinline__ void score_rows(const tail_u4 (&rows)[BATCH], int batch, int n_tail, float* sc) {
#pragma unroll
    for (int it = 0; it < BATCH; ++it) {
      const int row = batch_row(batch, it);
      const tail_h8 kv = __builtin_bit_cast(tail_h8, rows[it]);
      float part[HB];
#pragma unroll
      for (int hd = 0; hd < HB; ++hd) part[hd] = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float kf = (float)kv[i];
#pragma unroll
        for (int hd = 0; hd < HB; ++hd) part[hd] = fmaf(kf, qreg[hd][i], part[hd]);
      }
#pragma unroll
      for (int hd = 0; hd < HB; ++hd) {
        float v = part[hd];
        v += tail_dpp<0xB1>(v);                    // lane ^ 1
        v += tail_dpp<0x4E>(v);                    // lane ^ 2
        v += tail_dpp<0x141>(v);                   // 7 - lane within 8
        if (LPR == 16) v += tail_dpp<0x140>(v);    // 15 - lane within 16
        if (chunk == 0 && row < n_tail) sc[hd * kMaxTailRows + row] = v;
      }
    }
  }

  // tail_len: the caller's read of tail_lens[b] (requested early, so that it has arrived by now)
  __device__ __forceinline__ void finish(int tail_len, int nh, float* scratch, float* result) {
    float* sc = scratch;                       // [HB][kMaxTailRows] scores, then weights
    float* red = scratch + HB * kMaxTailRows;  // [NWV][HB][D]
    float* stat = red + NWV * HB * D;          // [2][HB][NWV]
    const int tid = threadIdx.x;
    const int n_tail = min(max(tail_len, 0), cap);
#pragma unroll
    for (int hd = 0; hd < HB; ++hd) {
      // nothing derived from q may move above loads the caller issued after issue_keys()
      asm volatile("" : "+v"(qraw[hd].x), "+v"(qraw[hd].y), "+v"(qraw[hd].z), "+v"(qraw[hd].w));
      const tail_h8 qv = __builtin_bit_cast(tail_h8, qraw[hd]);
#pragma unroll
      for (int i = 0; i < 8; ++i) qreg[hd][i] = hd < nh ? (float)qv[i] * qk : 0.f;
    }
    const int n_batches = (n_tail + ROWS_PER_BATCH - 1) / ROWS_PER_BATCH;
    // ---- scores ----
    if (n_batches > 0) score_rows(kreg, 0, n_tail, sc);
    for (int batch = 1; batch < n_batches; ++batch) {
      tail_u4 rows[BATCH];
#pragma unroll
      for (int it = 0; it < BATCH; ++it) {
        const int row = batch_row(batch, it);
        rows[it] = tail_u4{0u, 0u, 0u, 0u};
        if (row < n_tail) rows[it] = *reinterpret_cast<const tail_u4*>(kt + (long)row * D);
      }
      score_rows(rows, batch, n_tail, sc);
    }
    __syncthreads();
    // ---- softmax over the rows: thread t owns rows t, t + 64 NWV, ... ----
    float m[HB];
#pragma unroll
    for (int hd = 0; hd < HB; ++hd) {
      float v = -INFINITY;
      for (int t = tid; t < n_tail; t += 64 * NWV) v = fmaxf(v, sc[hd * kMaxTailRows + t]);
      for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
      if (lane == 0) stat[hd * NWV + wave] = v;
    }
    __syncthreads();
#pragma unroll
    for (int hd = 0; hd < HB; ++hd) {
      float mm = -INFINITY;
#pragma unroll
      for (int w = 0; w < NWV; ++w) mm = fmaxf(mm, stat[hd * NWV + w]);
      m[hd] = mm;
      float v = 0.f;
      for (int t = tid; t < n_tail; t += 64 * NWV) {
        const float p = __builtin_amdgcn_exp2f(sc[hd * kMaxTailRows + t] - mm);
        sc[hd * kMaxTailRows + t] = p;
        v += p;
      }
      for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
      if (lane == 0) stat[(HB + hd) * NWV + wave] = v;
    }
    __syncthreads();
    // ---- weighted sum of the value rows ----
    float acc[HB][8];
#pragma unroll
    for (int hd = 0; hd < HB; ++hd)
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[hd][i] = 0.f;
    for (int batch = 0; batch < n_batches; ++batch) {
      tail_u4 rows[BATCH];
#pragma unroll
      for (int it = 0; it < BATCH; ++it) {
        const int row = batch_row(batch, it);
        // batch 0 was requested by issue_keys() for every row below the capacity: rows past the
        // tail's length hold whatever the caller left there and are dropped here
        rows[it] = (row < n_tail) ? vreg[it] : tail_u4{0u, 0u, 0u, 0u};
        if (batch > 0 && row < n_tail) rows[it] = *reinterpret_cast<const tail_u4*>(vt + (long)row * D);
      }
#pragma unroll
      for (int it = 0; it < BATCH; ++it) {
        const int row = batch_row(batch, it);
        const tail_h8 vv = __builtin_bit_cast(tail_h8, rows[it]);
        float w[HB];
#pragma unroll
        for (int hd = 0; hd < HB; ++hd) w[hd] = (row < n_tail) ? sc[hd * kMaxTailRows + row] : 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float vf = (float)vv[i];
#pragma unroll
          for (int hd = 0; hd < HB; ++hd) acc[hd][i] = fmaf(w[hd], vf, acc[hd][i]);
        }
      }
    }
    // lanes with the same chunk (different rows) add up, then the waves
#pragma unroll
    for (int hd = 0; hd < HB; ++hd) {
      if (hd < nh) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          float v = acc[hd][i];
          for (int o = LPR; o < 64; o <<= 1) v += __shfl_xor(v, o);
          if (rsub == 0) red[(wave * HB + hd) * D + 8 * chunk + i] = v;
        }
      }
    }
    __syncthreads();
    for (int idx = tid; idx < nh * D; idx += 64 * NWV) {
      const int hd = idx / D, c = idx % D;
      float o = 0.f;
#pragma unroll
      for (int w = 0; w < NWV; ++w) o += red[(w * HB + hd) * D + c];
      result[hd * (D + 2) + c] = o;
      if (c == 0) {
        float l = 0.f;
#pragma unroll
        for (int w = 0; w < NWV; ++w) l += stat[(HB + hd) * NWV + w];
        result[hd * (D + 2) + D] = (n_tail > 0) ? m[hd] : -INFINITY;
        result[hd * (D + 2) + D + 1] = l;
      }
    }
    __syncthreads();
  }
};


// The same attention by single waves, for the matrix-core kernel: the rows are dealt over all waves of
// all workgroups of the (sequence, kv head), four rows per wave-wide load, and every wave leaves a
// partial of its own for the workgroup's merge.  No barrier, no exchange through LDS but the result.
// (One workgroup working the whole tail between barriers, with lane exchanges through LDS, took 7 to
// 9 us of a 30 us launch that its tiles had to wait for; the rows' bytes are worth 1.5.)
//   issue()   starts the loads of q and of the wave's first BATCH keys and values (rows below the
//             capacity are readable whatever the tail's length, which is not known yet; rows past it
//             read the last row instead: no branches, the caller may have other loads in flight whose
//             count the compiler has to keep);
//   finish()  leaves out[head][0..128) (unnormalised), out[head][128] = largest score in log2 units (-inf:
//             no row, or none that weighs anything) and out[head][129] = sum of weights in the wave's `result`.
// HEADS query heads share every row.  PAIR: the 128 channels are two neighbouring kv heads of 64, each
// with HEADS / 2 query heads: the lanes of each half read their own head's arrays, query head hd is zero
// outside the half p = hd / (HEADS / 2), and its partial is channels [64 p, 64 p + 64) of result[hd].
template <int HEADS, int BATCH, bool PAIR>
struct TailWave {
  static constexpr int D = 128, RD = PAIR ? 64 : 128, LPR = 16, RPI = 4;
  static constexpr int HPK = PAIR ? HEADS / 2 : HEADS;   // query heads per kv head
  static constexpr int kResultFloats = HEADS * (D + 2);
  tail_u4 kreg[BATCH], vreg[BATCH], qraw[HEADS];
  const uint16_t* kt;
  const uint16_t* vt;
  int chunk, rsub, cap, first, stride;
  float qk;

  __device__ __forceinline__ int row_of(int it) const { return RPI * (first + stride * it) + rsub; }

  // `nth` of `waves`: the wave among all that share the rows; nh query heads per kv head are present
  __device__ __forceinline__ void issue(const DecodeArgs& a, int b, int h, long hq0, int nh, int heads_per_kv, int nth, int waves) {
    const int lane = threadIdx.x & 63;
    chunk = lane & 15; rsub = lane >> 4;
    cap = a.tail.capacity;
    first = nth; stride = waves;
    const int H = a.cache.kv_heads;
    const int own = PAIR ? chunk >> 3 : 0, part = PAIR ? chunk & 7 : chunk;
    kt = a.tail.k_tail + ((long)b * H + h + own) * cap * RD + 8 * part;
    vt = a.tail.v_tail + ((long)b * H + h + own) * cap * RD + 8 * part;
    qk = a.scale * 1.4426950408889634f;
#pragma unroll
    for (int hd = 0; hd < HEADS; ++hd) {
      const long head = hq0 + (PAIR ? (hd / HPK) * heads_per_kv : 0) + min(hd % HPK, nh - 1);
      qraw[hd] = *reinterpret_cast<const tail_u4*>(a.q + ((long)b * a.q_heads + head) * RD + 8 * part);
    }
#pragma unroll
    for (int it = 0; it < BATCH; ++it) kreg[it] = *reinterpret_cast<const tail_u4*>(kt + (long)min(row_of(it), cap - 1) * RD);
#pragma unroll
    for (int it = 0; it < BATCH; ++it) vreg[it] = *reinterpret_cast<const tail_u4*>(vt + (long)min(row_of(it), cap - 1) * RD);
  }

  static __device__ __forceinline__ float over_rows_max(float v) {   // over the four rows of a load
    const uint32_t w = __builtin_bit_cast(uint32_t, v);
    const auto x = __builtin_amdgcn_permlane16_swap(w, w, false, false);
    const uint32_t m = __builtin_bit_cast(uint32_t, fmaxf(__builtin_bit_cast(float, (uint32_t)x[0]), __builtin_bit_cast(float, (uint32_t)x[1])));
    const auto y = __builtin_amdgcn_permlane32_swap(m, m, false, false);
    return fmaxf(__builtin_bit_cast(float, (uint32_t)y[0]), __builtin_bit_cast(float, (uint32_t)y[1]));
  }

  __device__ __forceinline__ void finish(int tail_len, int nh, float* result) {
    const int n_tail = min(max(tail_len, 0), cap);
    float qreg[HEADS][8], acc[HEADS][8], m_run[HEADS], l_run[HEADS];
#pragma unroll
    for (int hd = 0; hd < HEADS; ++hd) {
      // nothing derived from q may move above loads the caller issued after issue()
      asm volatile("" : "+v"(qraw[hd].x), "+v"(qraw[hd].y), "+v"(qraw[hd].z), "+v"(qraw[hd].w));
      const tail_h8 qv = __builtin_bit_cast(tail_h8, qraw[hd]);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        qreg[hd][i] = (hd % HPK < nh && (!PAIR || (chunk >> 3) == hd / HPK)) ? (float)qv[i] * qk : 0.f;
        acc[hd][i] = 0.f;
      }
      m_run[hd] = -INFINITY;
      l_run[hd] = 0.f;
    }
    // (wave-uniform: row_of(it) - rsub is the first of the load's four rows)
    for (int it0 = 0; RPI * (first + stride * it0) < n_tail; it0 += BATCH) {
      if (it0 > 0) {   // more rows than were requested up front
#pragma unroll
        for (int it = 0; it < BATCH; ++it) kreg[it] = *reinterpret_cast<const tail_u4*>(kt + (long)min(row_of(it0 + it), cap - 1) * RD);
#pragma unroll
        for (int it = 0; it < BATCH; ++it) vreg[it] = *reinterpret_cast<const tail_u4*>(vt + (long)min(row_of(it0 + it), cap - 1) * RD);
      }
      float sc[BATCH][HEADS], m_ref[HEADS];
#pragma unroll
      for (int it = 0; it < BATCH; ++it) {
        const tail_h8 kv = __builtin_bit_cast(tail_h8, kreg[it]);
        const bool live = row_of(it0 + it) < n_tail;
#pragma unroll
        for (int hd = 0; hd < HEADS; ++hd) {
          float v = 0.f;
#pragma unroll
          for (int i = 0; i < 8; ++i) v = fmaf((float)kv[i], qreg[hd][i], v);
          // a pair: the lanes on the other head's half of the row add an outright zero (their query is
          // zero, but zero times whatever that head's row holds need not be)
          if (PAIR && (chunk >> 3) != hd / HPK) v = 0.f;
          v += tail_dpp<0xB1>(v);     // lane ^ 1
          v += tail_dpp<0x4E>(v);     // lane ^ 2
          v += tail_dpp<0x141>(v);    // 7 - lane within 8
          v += tail_dpp<0x140>(v);    // 15 - lane within 16
          sc[it][hd] = live ? v : -INFINITY;
        }
      }
#pragma unroll
      for (int hd = 0; hd < HEADS; ++hd) {
        float m = sc[0][hd];
#pragma unroll
        for (int it = 1; it < BATCH; ++it) m = fmaxf(m, sc[it][hd]);
        m = fmaxf(over_rows_max(m), m_run[hd]);
        // (-inf where every row so far scored that, as an infinite key makes it: such rows weigh nothing,
        // whatever the other waves' rows do.  The weights are then taken against zero: exp2(-inf) = 0)
        m_ref[hd] = m == -INFINITY ? 0.f : m;
        const float alpha = __builtin_amdgcn_exp2f(m_run[hd] - m_ref[hd]);
        m_run[hd] = m;
        l_run[hd] *= alpha;
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[hd][i] *= alpha;
      }
#pragma unroll
      for (int it = 0; it < BATCH; ++it) {
        // rows past the tail's length hold whatever the caller left there and are dropped here
        const bool live = row_of(it0 + it) < n_tail;
        const tail_h8 vv = __builtin_bit_cast(tail_h8, live ? vreg[it] : tail_u4{0u, 0u, 0u, 0u});
#pragma unroll
        for (int hd = 0; hd < HEADS; ++hd) {
          const float p = __builtin_amdgcn_exp2f(sc[it][hd] - m_ref[hd]);
          l_run[hd] += p;
#pragma unroll
          for (int i = 0; i < 8; ++i) acc[hd][i] = fmaf(p, (float)vv[i], acc[hd][i]);
        }
      }
    }
    // Add up the four rows' lanes: after the first exchange a lane holds four of its eight channels
    // for two rows' lanes, after the second two for all four.
    const int b4 = rsub & 1, b5 = rsub >> 1;
#pragma unroll
    for (int hd = 0; hd < HEADS; ++hd) {
      float half[4], out[2];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const auto x = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, acc[hd][i]),
                                                        __builtin_bit_cast(uint32_t, acc[hd][i + 4]), false, false);
        half[i] = __builtin_bit_cast(float, (uint32_t)x[0]) + __builtin_bit_cast(float, (uint32_t)x[1]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const auto x = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, half[i]),
                                                        __builtin_bit_cast(uint32_t, half[i + 2]), false, false);
        out[i] = __builtin_bit_cast(float, (uint32_t)x[0]) + __builtin_bit_cast(float, (uint32_t)x[1]);
      }
      // the sixteen lanes of a row hold the same p: one lane per row contributes to the sum of weights
      float l = l_run[hd];
      const uint32_t lw = __builtin_bit_cast(uint32_t, l);
      const auto x = __builtin_amdgcn_permlane16_swap(lw, lw, false, false);
      l = __builtin_bit_cast(float, (uint32_t)x[0]) + __builtin_bit_cast(float, (uint32_t)x[1]);
      const uint32_t lw2 = __builtin_bit_cast(uint32_t, l);
      const auto y = __builtin_amdgcn_permlane32_swap(lw2, lw2, false, false);
      l = __builtin_bit_cast(float, (uint32_t)y[0]) + __builtin_bit_cast(float, (uint32_t)y[1]);
      float* dst = result + hd * (D + 2);
      dst[8 * chunk + 4 * b5 + 2 * b4] = out[0];
      dst[8 * chunk + 4 * b5 + 2 * b4 + 1] = out[1];
      if (rsub == 0 && chunk == 0) { dst[D] = m_run[hd]; dst[D + 1] = l; }
    }
  }
};

}  // namespace dq
