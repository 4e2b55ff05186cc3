// Wave-level merge of the per-part results of a head contraction into the
// row's log-sum-exp and its k best (logit, token) pairs.
#pragma once
#include "device_utils.h"
#include "spec_internal.h"

namespace specdraft {

// All 64 lanes of a wave call this for the same row; every lane receives the
// result.  out_val / out_idx must be indexed with compile-time constants by the
// caller (they live in registers).  Candidates of different parts never share a
// vocabulary index, so (value, index) is a strict total order.
//
// Latency matters here (this sits on the serial chain between two heads at
// batch 1): every lane first issues the loads of UN parts at once, then folds
// them into a sorted register list; the k results are popped with wave-wide
// reductions, no memory traffic in between.  UN is as large as the parts need: with the
// 17 .. 128 parts of the dense kernel four per lane are mostly masked work (tree kernel, 72 rows of 17 parts
// per sequence: 23.8 -> 19.1 us; 24 rows of 64 parts: 16.5 -> 13.7 us).
template <int K, int UN>
__device__ __forceinline__ void wave_merge_partials_un(const Partials& p, int64_t row, int nparts, int k,
                                                    float (&out_val)[kMaxTopK], int32_t (&out_idx)[kMaxTopK],
                                                    float& lse) {
  const int lane = opaque_tid() & 63;
  const float* pm = p.m + row * nparts;
  const float* ps = p.s + row * nparts;
  const float* pv = p.val + row * (int64_t)nparts * k;
  const int32_t* pi = p.idx + row * (int64_t)nparts * k;

  // the lane's list, as 64-bit keys (best_key): sorted, empty slots hold the key of (-inf, none)
  const uint64_t kEmpty = best_key(SPEC_NEG_INF, kIdxNone);
  uint64_t tk[K];
#pragma unroll
  for (int q = 0; q < K; ++q) tk[q] = kEmpty;
  float run_m = SPEC_NEG_INF, run_s = 0.f;

  for (int p0 = 0; p0 < nparts; p0 += 64 * UN) {
    float lm[UN], ls[UN], lv[UN][K];
    int32_t li[UN][K];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      // every load is unconditional (clamped to a valid slot) so that all of them are
      // in flight together; what does not exist is masked after it arrives
      const int part = p0 + u * 64 + lane;
      const bool ok = part < nparts;
      const int pc = ok ? part : nparts - 1;
      const float m_ = pm[pc], s_ = ps[pc];
      lm[u] = ok ? m_ : SPEC_NEG_INF;
      ls[u] = ok ? s_ : 0.f;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const int jc = j < k ? j : k - 1;
        const float v_ = pv[(int64_t)pc * k + jc];
        const int32_t i_ = pi[(int64_t)pc * k + jc];
        const bool okj = ok && j < k;
        lv[u][j] = okj ? v_ : SPEC_NEG_INF;
        li[u][j] = okj ? i_ : kIdxNone;
      }
    }
    // softmax pieces of this lane's UN parts: one exponential per part (the fast one: its 1e-6
    // relative error is far inside what separates float32 from float64 accumulation)
    float mloc = lm[0];
#pragma unroll
    for (int u = 1; u < UN; ++u) mloc = fmaxf(mloc, lm[u]);
    float sloc = 0.f;
#pragma unroll
    for (int u = 0; u < UN; ++u) sloc += lm[u] > SPEC_NEG_INF ? ls[u] * __expf(lm[u] - mloc) : 0.f;
    if (p0 == 0) {
      run_m = mloc;
      run_s = sloc;
    } else if (mloc > SPEC_NEG_INF) {
      const float mn = fmaxf(run_m, mloc);
      run_s = run_s * __expf(run_m - mn) + sloc * __expf(mloc - mn);
      run_m = mn;
    }
    // branch-free insertion: a chain of compare-exchanges down the list (an entry that does not
    // belong, the empty key included, falls through and changes nothing)
#pragma unroll
    for (int u = 0; u < UN; ++u) {
#pragma unroll
      for (int j = 0; j < K; ++j) {
        uint64_t x = best_key(lv[u][j], li[u][j]);
#pragma unroll
        for (int q = 0; q < K; ++q) {
          const bool gt = x > tk[q];
          const uint64_t lower = gt ? tk[q] : x;
          tk[q] = gt ? x : tk[q];
          x = lower;
        }
      }
    }
  }

  const float mx = wave_max(run_m);
  const float sum = wave_sum(run_m > SPEC_NEG_INF ? run_s * __expf(run_m - mx) : 0.f);
  lse = mx + logf(sum);

#pragma unroll
  for (int j = 0; j < kMaxTopK; ++j) {
    out_val[j] = SPEC_NEG_INF;
    out_idx[j] = kIdxNone;
  }
#pragma unroll
  for (int j = 0; j < K; ++j) {
    if (j < k) {
      const uint64_t best = wave_best_key(tk[0]);
      const bool won = tk[0] == best;   // the owner of the winner pops it (keys of real entries are unique)
#pragma unroll
      for (int q = 0; q + 1 < K; ++q) {
        const uint64_t up = opaque_key(tk[q + 1]);
        tk[q] = won ? up : tk[q];
      }
      tk[K - 1] = won ? kEmpty : tk[K - 1];
      best_unkey(best, out_val[j], out_idx[j]);
    }
  }
}

template <int K>
__device__ __forceinline__ void wave_merge_partials_k(const Partials& p, int64_t row, int nparts, int k,
                                                    float (&out_val)[kMaxTopK], int32_t (&out_idx)[kMaxTopK],
                                                    float& lse) {
  if (nparts <= 64) wave_merge_partials_un<K, 1>(p, row, nparts, k, out_val, out_idx, lse);
  else if (nparts <= 128) wave_merge_partials_un<K, 2>(p, row, nparts, k, out_val, out_idx, lse);
  else wave_merge_partials_un<K, 4>(p, row, nparts, k, out_val, out_idx, lse);
}

// The same merge for the ONE row that a whole workgroup wants, by its first 256 threads: with at most
// 256 parts every thread holds exactly one part's (already sorted) list, so nothing has
// to be inserted.  Two levels, ONE exchange: every wave reduces its 64 parts to its own
// (max, sum-exp, k best) with wave-wide reductions only, the four waves' results go
// through LDS behind a single barrier, and there every one of the 4 K candidates is given to
// a lane that counts the candidates before it: its rank.  (A pop per round across the whole group
// - one barrier and one LDS exchange per result - took 0.65 us per round on the batch-1 chain; the four
// lists merged in registers by every thread, K shifts of 4 K keys each, made the stage kernel take 7.5 us
// for 5 rows (256 parts, top-5), 21.7 for 960 rows and 34.4 for 2304, against 6.8, 19.5 and 27.1.)
// The other threads of a larger workgroup wait at the barrier: they would only take issue slots, eight waves on four SIMDs
// (stage kernel, 5 rows of top-5, 7.0 us with both groups of 256 merging, 6.0 with one; 96 rows of top-6 9.6 and 8.5; top-1 4.8
// either way).  EVERY thread of the workgroup must call, with the same k and nparts.  Lane c < 4 K of every wave receives
// candidate c (value, index, rank; the k best have ranks 0 .. k - 1), the other lanes rank kNoRank; every thread receives
// lse.  `lds` is scratch of kMergeLds words, 8-byte aligned, that nobody has used before.
constexpr int kMergeWave = 2 + 2 * kMaxTopK;   // words per wave: max, sum-exp, k keys
constexpr int kMergeLds = 4 * kMergeWave;
constexpr int kNoRank = 1 << 20;
// What a thread reads for it, its own part's list: to be requested before anything else that a caller wants from memory.
template <int K>
struct MergePart {
  float m, s, v[K];
  int32_t i[K];
};
template <int K>
__device__ __forceinline__ void group_merge_load(const Partials& p, int64_t row, int nparts, int k, MergePart<K>& x) {
  const int pc = min(opaque_tid() & 255, nparts - 1);   // (past the last part: that one again, masked below)
  x.m = p.m[row * nparts + pc];
  x.s = p.s[row * nparts + pc];
  const float* pv = p.val + (row * nparts + pc) * (int64_t)k;
  const int32_t* pi = p.idx + (row * nparts + pc) * (int64_t)k;
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const int jc = j < k ? j : k - 1;
    x.v[j] = pv[jc];
    x.i[j] = pi[jc];
  }
}
template <int K>
__device__ __forceinline__ void group_merge_loaded(const MergePart<K>& x, const Partials& p, int64_t row, int nparts, int k,
                                                 float& out_val, int32_t& out_idx, int& rank,
                                                 float& lse, float* lds) {
  const int tid = opaque_tid(), gt = tid & 255, lane = gt & 63, w = gt >> 6;

  if (__builtin_amdgcn_readfirstlane(tid >> 8) == 0) {
    uint64_t tk[K];   // the thread's list as keys (best_key)
    const bool ok = gt < nparts;
    float run_m = ok ? x.m : SPEC_NEG_INF, run_s = ok ? x.s : 0.f;
    const uint64_t kEmpty = best_key(SPEC_NEG_INF, kIdxNone);
#pragma unroll
    for (int j = 0; j < K; ++j) tk[j] = ok && j < k ? best_key(x.v[j], x.i[j]) : kEmpty;
    const float* pm = p.m + row * nparts;
    const float* ps = p.s + row * nparts;
    const float* pv = p.val + row * (int64_t)nparts * k;
    const int32_t* pi = p.idx + row * (int64_t)nparts * k;
    for (int part = gt + 256; part < nparts; part += 256) {   // more parts than threads: fold the rest in
      const float m_ = pm[part], s_ = ps[part];
      if (m_ > SPEC_NEG_INF) {
        const float mn = fmaxf(run_m, m_);
        run_s = run_s * __expf(run_m - mn) + s_ * __expf(m_ - mn);
        run_m = mn;
      }
      for (int j = 0; j < k; ++j) {
        uint64_t c = best_key(pv[(int64_t)part * k + j], pi[(int64_t)part * k + j]);
#pragma unroll
        for (int q = 0; q < K; ++q) {   // (an entry that does not belong falls through and changes nothing)
          const bool gt_q = c > tk[q];
          const uint64_t lower = gt_q ? tk[q] : c;
          tk[q] = gt_q ? c : tk[q];
          c = lower;
        }
      }
    }

    // ---- this wave's 64 parts
    const float wm = wave_max(run_m);
    const float wsum = wave_sum(run_m > SPEC_NEG_INF ? run_s * __expf(run_m - wm) : 0.f);
    uint64_t won_key[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
      won_key[j] = kEmpty;
      if (j < k) {
        won_key[j] = wave_best_key(tk[0]);
        const bool won = tk[0] == won_key[j];   // the owner of the winner pops it (keys of real entries are unique)
#pragma unroll
        for (int q = 0; q + 1 < K; ++q) {
          const uint64_t up = opaque_key(tk[q + 1]);
          tk[q] = won ? up : tk[q];
        }
        tk[K - 1] = won ? kEmpty : tk[K - 1];
      }
    }
    // ---- the four waves' results through LDS
    float* mine = lds + w * kMergeWave;
    if (lane == 0) {
      mine[0] = wm;
      mine[1] = wsum;
#pragma unroll
      for (int j = 0; j < K; ++j)   // (empty entries are told apart, so that every candidate has its own rank)
        reinterpret_cast<uint64_t*>(mine + 2)[j] =
            won_key[j] == kEmpty ? best_key(SPEC_NEG_INF, kIdxNone - (w * kMaxTopK + j)) : won_key[j];
    }
  }
  __syncthreads();
  float m4[4], s4[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) { m4[q] = lds[q * kMergeWave]; s4[q] = lds[q * kMergeWave + 1]; }
  const float mx = fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3]));
  float sum = 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q) sum += m4[q] > SPEC_NEG_INF ? s4[q] * __expf(m4[q] - mx) : 0.f;
  lse = mx + logf(sum);

  const int c = min(lane, 4 * K - 1);
  const uint64_t key = reinterpret_cast<const uint64_t*>(lds + (c / K) * kMergeWave + 2)[c % K];
  int before_me = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int t = 0; t < K; ++t)
      before_me += reinterpret_cast<const uint64_t*>(lds + q * kMergeWave + 2)[t] > key ? 1 : 0;
  best_unkey(key, out_val, out_idx);
  if (out_idx > kIdxNone - 4 * kMaxTopK) out_idx = kIdxNone;   // (an empty entry: no token has such an index)
  rank = lane < 4 * K ? before_me : kNoRank;
}

// k is uniform over the launch: pick the list size that just holds it, so that
// the common narrow heads (k = 1..3) do not pay for eight slots.
__device__ __forceinline__ void wave_merge_partials(const Partials& p, int64_t row, int nparts, int k,
                                                    float (&out_val)[kMaxTopK], int32_t (&out_idx)[kMaxTopK],
                                                    float& lse) {
  switch (k) {
    case 1: wave_merge_partials_k<1>(p, row, nparts, k, out_val, out_idx, lse); break;
    case 2: wave_merge_partials_k<2>(p, row, nparts, k, out_val, out_idx, lse); break;
    case 3: wave_merge_partials_k<3>(p, row, nparts, k, out_val, out_idx, lse); break;
    case 4: wave_merge_partials_k<4>(p, row, nparts, k, out_val, out_idx, lse); break;
    case 5:
    case 6: wave_merge_partials_k<6>(p, row, nparts, k, out_val, out_idx, lse); break;
    default: wave_merge_partials_k<8>(p, row, nparts, k, out_val, out_idx, lse); break;
  }
}

}  // namespace specdraft
