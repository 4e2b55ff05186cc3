// Top-k lists and sums that lanes keep of a state row's logits, and their merge, of the kernels whose workgroups copy their operands
// straight into LDS (tile, one-round and panel kernel).
#pragma once
#include "device_utils.h"
#include "spec_internal.h"

namespace specdraft {

typedef __attribute__((address_space(3))) unsigned char lds_byte;
typedef const __attribute__((address_space(3))) u32x4 lds_word;

// ---- a list's entry: one float64 (high word = the logit, low word breaks ties: smaller index, larger key), as in the wide kernel ----
__device__ __forceinline__ double list_key(float x, int32_t not_index) {
  const int32_t b = __float_as_int(x);
  return __hiloint2double(b, not_index ^ (b >> 31));
}
__device__ __forceinline__ float list_logit(double key) { return __int_as_float(__double2hiint(key)); }
__device__ __forceinline__ int32_t list_index(double key) { return ~(__double2loint(key) ^ (__double2hiint(key) >> 31)); }
__device__ __forceinline__ uint64_t list_best_key(double key) { return best_key(list_logit(key), list_index(key)); }
// What a row's exponentials are relative to: its best logit so far, or where it has none (-inf and NaN only; weight rows past
// the vocabulary) a number below every logit whose product with log2(e) is still finite, so that exp(-inf) is 0 there too.
__device__ __forceinline__ float list_reference(double best) { return fmaxf(-2e38f, list_logit(best)); }

// N = copies of this wave that may still be in flight; LDS: all its LDS reads have returned.  Then the barrier.
template <int N, bool LDS>
__device__ __forceinline__ void copies_landed_barrier() {
  static_assert(N >= 0 && N < 64, "the counter has six bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (LDS ? 0 : 15 << 8));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// over eight neighbouring lanes
__device__ __forceinline__ float row8_max(float x) {
  x = fmaxf(x, dpp_f<kDppXor1>(x));
  x = fmaxf(x, dpp_f<kDppXor2>(x));
  return fmaxf(x, dpp_f<kDppHalfMirror>(x));
}
__device__ __forceinline__ float row8_sum(float x) {
  x += dpp_f<kDppXor1>(x);
  x += dpp_f<kDppXor2>(x);
  return x + dpp_f<kDppHalfMirror>(x);
}
__device__ __forceinline__ uint64_t row8_best_key(uint64_t key) {
  key = key_step<kDppXor1>(key);
  key = key_step<kDppXor2>(key);
  return key_step<kDppHalfMirror>(key);
}

// ---- merge of a workgroup of 2 x 4 waves: wave (wn, wm) holds, for state row 16 * (wm * MB + m) + lane % 16 of the block, one of
// the eight lists (4 lane groups x 2 waves) and sums that become the row's partial.  The lists go through LDS, from its start: the
// caller has seen all copies into it land and all reads of it return, for all waves.
constexpr size_t list_merge_bytes(int mb, int kt) { return (size_t)64 * mb * ((8 * kt + 1) * 8 + 8 * 8); }

template <int MB, int KT>
__device__ __forceinline__ void merge_lane_lists(unsigned char* smem, const double (&lk)[MB][KT], const float (&sum)[MB],
                                                 int wave, int lane, int row0, int R, const Partials& part, int k_top,
                                                 int nparts, int range) {
  constexpr int ROWS = 64 * MB, RS = 8 * KT + 1;
  uint64_t* sk = reinterpret_cast<uint64_t*>(smem);            // [ROWS][RS]
  float* sm = reinterpret_cast<float*>(sk + ROWS * RS);        // [ROWS][8]
  float* ss = sm + ROWS * 8;
  const int wn = wave / 4, wm = wave % 4, col = lane & 15, list = wn * 4 + (lane >> 4);
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    const int rl = (wm * MB + m) * 16 + col;
#pragma unroll
    for (int q = 0; q < KT; ++q) sk[rl * RS + list * KT + q] = list_best_key(lk[m][q]);
    sm[rl * 8 + list] = list_reference(lk[m][0]);
    ss[rl * 8 + list] = sum[m];
  }
  __syncthreads();
  const uint64_t kEmpty = best_key(SPEC_NEG_INF, kIdxNone);
  const int rows = min(ROWS, R - row0);
#pragma unroll 1
  for (int r0 = wave * 8; r0 < rows; r0 += 64) {   // eight lanes to a row
    const int rl = min(r0 + (lane >> 3), rows - 1), s8 = lane & 7;
    const bool live = r0 + (lane >> 3) < rows;
    uint64_t hk[KT];
#pragma unroll
    for (int q = 0; q < KT; ++q) hk[q] = sk[rl * RS + s8 * KT + q];
    const float m = sm[rl * 8 + s8], s = ss[rl * 8 + s8];
    const float mx = row8_max(m), tot = row8_sum(s * __expf(m - mx));
    const int64_t slot = (int64_t)(row0 + rl) * nparts + range;
    if (live && s8 == 0) {
      part.m[slot] = mx;
      part.s[slot] = tot;
    }
#pragma unroll
    for (int j = 0; j < KT; ++j) {
      if (j < k_top) {
        const uint64_t best = row8_best_key(hk[0]);
        const bool won = hk[0] == best;   // the owner of the winner pops it
#pragma unroll
        for (int q = 0; q + 1 < KT; ++q) {
          const uint64_t up = opaque_key(hk[q + 1]);
          hk[q] = won ? up : hk[q];
        }
        hk[KT - 1] = won ? kEmpty : hk[KT - 1];
        if (live && s8 == j) {
          float bv;
          int32_t bi;
          best_unkey(best, bv, bi);
          part.val[slot * k_top + j] = bv;
          part.idx[slot * k_top + j] = bi;
        }
      }
    }
  }
}

}  // namespace specdraft
