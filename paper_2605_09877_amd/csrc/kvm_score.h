// Similarity and winners of a block's tokens, the generic form (any dtype and block length): a kernel of its own (fold.hip)
// or workgroups of a prefill's attention launch (attn_rows.hip, attn_mfma.hip).
#pragma once

#include "kvm_device.h"
#include "kvm_internal.h"

namespace kvm {

// One wave per token, four tokens per workgroup (number `blk` of unit u); lanes stride over state rows [row0, row1); each
// dot product is an fp64 sum of the I/O-dtype operands.  first_pass: rows are the pre-append state,
// writes s_j (all rows) and the best eligible row.  Otherwise rows are the ones appended in this fold and
// only tokens that were not appended themselves may move to them (strictly larger score only).
// What bounds it is latency: a row is a lane's chain of D dependent fp64 additions behind a round trip to memory, so a
// lane has two rows under way, eight pieces of each: 2 x 4173 tokens, 16 heads of 64 channels on 4, 256 rows, 458 us a call;
// with one row whole 522, with four rows of four pieces 25 more than with two.  But fp32 rows of 128 channels one by
// one, sixteen pieces at a time: 1500 tokens, 4 heads, 300 rows 333 us, two rows 353.
// And with many workgroups (2560: bf16, 32 units, 320-token blocks, 1100 rows) the registers of two rows cost more than they buy,
// 1846 us a call with one, 2054 with two: score_kernel has both forms.
template <typename T, int D, bool kTwo = true>
__device__ __forceinline__ void score_tokens(const Dev &dv, int slot, int row0, int row1, int first_pass, int blk, int u) {
  constexpr int VEC = Vec16<T>::kN, kPieces = D / VEC;          // 16-byte pieces of a row
  constexpr int kRows = kPieces > 16 || !kTwo ? 1 : 2;          // rows under way
  constexpr int kInFlight = kRows == 2 || kPieces < 16 ? 8 : 16;  // pieces of each
  static_assert(kPieces % kInFlight == 0, "");
  __shared__ double kb[4][D];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = blk * 4 + wave;
  const int64_t tj = (int64_t)u * dv.C + j;
  const bool active = j < dv.C && (first_pass || dv.app[tj] < 0);
  if (active) {
    const T *kbar = (const T *)dv.kbar + tj * D;
    for (int c = lane; c < D; c += 64) kb[wave][c] = (double)Io<T>::load(kbar + c);
  }
  __syncthreads();
  if (!active) return;
  double best_all = -INFINITY, best = -INFINITY;
  int best_i = 0x7fffffff;
  const T *kh = (const T *)dv.khat + slot * dv.slot_elems + (int64_t)u * dv.Mcap * D;
  for (int i0 = row0 + lane; i0 < row1; i0 += 64 * kRows) {
    const T *row[kRows];
    double acc[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      const int i = i0 + 64 * r;
      row[r] = kh + (int64_t)(i < row1 ? i : i0) * D;
      acc[r] = 0.0;
    }
#pragma unroll 1
    for (int c0 = 0; c0 < D; c0 += kInFlight * VEC) {
      uint4 raw[kRows][kInFlight];
#pragma unroll
      for (int r = 0; r < kRows; ++r)
#pragma unroll
        for (int n = 0; n < kInFlight; ++n) raw[r][n] = *reinterpret_cast<const uint4 *>(row[r] + c0 + n * VEC);
#pragma unroll
      for (int n = 0; n < kInFlight; ++n) {
        float x[kRows][VEC];
#pragma unroll
        for (int r = 0; r < kRows; ++r) unpack16<T>(raw[r][n], x[r]);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const double k = kb[wave][c0 + n * VEC + e];
#pragma unroll
          for (int r = 0; r < kRows; ++r) acc[r] += k * (double)x[r][e];
        }
      }
    }
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      const int i = i0 + 64 * r;
      if (i < row1) {
        best_all = acc[r] > best_all ? acc[r] : best_all;
        if (i >= dv.S && acc[r] > best) {
          best = acc[r];
          best_i = i;
        }
      }
    }
  }
  best_all = wave_max(best_all);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double ob = __shfl_xor(best, o, kWave);
    const int oi = __shfl_xor(best_i, o, kWave);
    if (ob > best || (ob == best && oi < best_i)) {
      best = ob;
      best_i = oi;
    }
  }
  if (lane == 0) {
    if (first_pass) {
      dv.score[tj] = make_float2((float)best_all, (float)best);
      dv.pi[tj] = best_i;
      dv.app[tj] = -1;
    } else if (best_i != 0x7fffffff && (float)best > dv.score[tj].y) {
      // compare in the stored (fp32) precision so both passes rank alike
      dv.score[tj].y = (float)best;
      dv.pi[tj] = best_i;
    }
  }
}

}  // namespace kvm
