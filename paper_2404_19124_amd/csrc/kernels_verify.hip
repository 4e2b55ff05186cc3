// Verification (Sec. 1, 3.1, 5 of the paper), greedy:
//   greedy[b,c,p]  = first maximum of base_logits[b,c,p,:]
//   accept[b,c]    = number of leading positions p with greedy[b,c,p] == cand[b,c,p]
//   best[b]        = first candidate with the longest accepted prefix
//   out            = cand[b,best,:a] ++ greedy[b,best,a]   (the bonus token)
// The row scan is the only part that touches real memory: one workgroup (NT threads) per
// (b,c,p) row, 16-byte loads, (value, index) reduced with "larger value, then
// smaller index".
#include <type_traits>

#include "device_utils.h"
#include "spec_internal.h"

namespace specdraft {

template <bool BF16, int NT, int U>
__global__ __launch_bounds__(NT) void argmax_rows_kernel(const void* logits, int V, int B, int n1,
                                                           const int32_t* n_cand, int32_t* greedy) {
  __shared__ float sv[16];
  __shared__ int32_t si[16];
  const int64_t row = blockIdx.x;
  const int tid = threadIdx.x;
  if (n_cand) {
    // per-sequence candidate counts: rows of padding candidates are not read at all
    const int p = (int)(row % n1);
    const int64_t qc = row / n1;
    const int c = (int)(qc % B), nc = n_cand[qc / B];
    if (c >= max(nc, 1) || (nc == 0 && p > 0)) {
      if (tid == 0) greedy[row] = -1;
      return;
    }
  }
  // (a thread meets its elements in increasing index order, so a strict "larger" keeps the first maximum;
  // the (value, smaller index) order only matters between threads)
  float bv = SPEC_NEG_INF;
  int32_t bi = kIdxNone;
  // 16-byte loads from the row's first 16-byte boundary on; the few elements before it (a vocabulary whose rows do
  // not start on one) and behind the last whole word go one to a thread, requested with the rest: at small batch the
  // kernel is a chain of memory round trips, not a stream.  U words of a thread are in flight.  Non-temporal: the
  // logits are read once.
  typedef typename std::conditional<BF16, uint16_t, float>::type elem;
  constexpr int PER = BF16 ? 8 : 4;
  const elem* x = static_cast<const elem*>(logits) + row * V;
  auto take = [&](float v, int i) {
    if (v > bv) { bv = v; bi = i; }
  };
  auto value = [](elem e) {
    if constexpr (BF16) return bf16_bits_to_f32(e);
    else return e;
  };
  if constexpr (U == 0) {
    for (int i = tid; i < V; i += NT) take(value(x[i]), i);
  }
  const uint32_t past = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(x)) & 15;
  const int lead = min(V, (int)(((16 - past) & 15) / (uint32_t)sizeof(elem)));
  const u32x4* xv = reinterpret_cast<const u32x4*>(x + lead);
  const int nvec = U == 0 ? 0 : (int)((uint32_t)(V - lead) / PER), rest = lead + nvec * PER;
  const bool ends = U > 0 && lead + (V - rest) > 0;   // (the same for every thread)
  elem first = 0, last = 0;
  if (ends) {
    if (tid < lead) first = x[tid];
    if (tid < V - rest) last = x[rest + tid];
  }
  for (int c0 = tid; c0 < nvec; c0 += NT * U) {
    u32x4 raw[U > 0 ? U : 1];
#pragma unroll
    for (int u = 0; u < U; ++u) raw[u] = __builtin_nontemporal_load(xv + min(c0 + u * NT, nvec - 1));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = c0 + u * NT, i0 = lead + c * PER;
      if (c < nvec) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if constexpr (BF16) {
            take(bf16_bits_to_f32(raw[u][q] & 0xffffu), i0 + 2 * q);
            take(bf16_bits_to_f32(raw[u][q] >> 16), i0 + 2 * q + 1);
          } else {
            take(__uint_as_float(raw[u][q]), i0 + q);
          }
        }
      }
    }
  }
  if (ends) {
    if (tid < V - rest) take(value(last), rest + tid);
    // (the element before the boundary comes before the thread's others: it wins a tie)
    if (tid < lead && value(first) > SPEC_NEG_INF && value(first) >= bv) { bv = value(first); bi = tid; }
  }
  block_best<NT>(bv, bi, sv, si);
  // a row of NaNs (or of -inf) has no "larger" element: report index 0 like a first-maximum scan
  if (tid == 0) greedy[row] = (bi == kIdxNone) ? 0 : bi;
}

// As many words of a thread in flight as a row has: a row of fewer loads its last word over and over in the others (4096
// rows of 1001 floats with 16 in flight: 20.1 us).  Two elements of a thread and less: no words at all, the row's ends
// would cost more than they save (the same rows: 10.1 us by words, 9.8 by elements).  4096 rows of 8001 floats: 30.8 us
// by elements, 35.2 with 16 words in flight, 22.4 with 4; of 32003: 157 by elements, 80 now.
template <bool BF16, int NT>
static void launch_argmax_t(const void* logits, int64_t rows, int V, int B, int n1, const int32_t* n_cand,
                            int32_t* greedy, hipStream_t st) {
  const int words = V / (BF16 ? 8 : 4);
#define LAUNCH_ARGMAX(U) \
  hipLaunchKernelGGL((argmax_rows_kernel<BF16, NT, U>), dim3((unsigned)rows), dim3(NT), 0, st, logits, V, B, n1, n_cand, greedy)
  if (V <= 2 * NT) LAUNCH_ARGMAX(0);
  else if (words <= NT) LAUNCH_ARGMAX(1);
  else if (words <= 2 * NT) LAUNCH_ARGMAX(2);
  else if (words <= 4 * NT) LAUNCH_ARGMAX(4);
  else LAUNCH_ARGMAX(8192 / NT);
#undef LAUNCH_ARGMAX
}

hipError_t launch_argmax_rows(const void* logits, int bf16, int64_t rows, int V, int B, int n1, const int32_t* n_cand,
                              int32_t* greedy, hipStream_t st) {
  // a few rows (small batch): a chain of memory round trips, the more loads in flight per row the better;
  // thousands of rows: a stream, which runs a little faster from 512-thread workgroups (7B batch 64: 81 -> 79.4 us)
  if (rows >= 1024) {
    if (bf16) launch_argmax_t<true, 512>(logits, rows, V, B, n1, n_cand, greedy, st);
    else launch_argmax_t<false, 512>(logits, rows, V, B, n1, n_cand, greedy, st);
  } else {
    if (bf16) launch_argmax_t<true, 1024>(logits, rows, V, B, n1, n_cand, greedy, st);
    else launch_argmax_t<false, 1024>(logits, rows, V, B, n1, n_cand, greedy, st);
  }
  return hipGetLastError();
}

__global__ __launch_bounds__(64) void accept_kernel(const int32_t* greedy, const int32_t* cand, const int32_t* n_cand,
                                                    int B, int n, int32_t* accept_len, int32_t* best_cand,
                                                    int32_t* out_tokens, int32_t* n_out, int32_t* accept_all) {
  const int q = blockIdx.x, lane = threadIdx.x;
  // candidates of this sequence (the rest of its B slots is padding); none = speculation off: the
  // first slot stands for the empty candidate, whose accepted length is 0
  const int nc = n_cand ? n_cand[q] : B;
  // (accepted length, candidate): longer first, then smaller candidate index
  float bv = -1.f;
  int32_t bi = kIdxNone;
  for (int c = lane; c < B; c += 64) {
    const int32_t* g = greedy + ((int64_t)q * B + c) * (n + 1);
    const int32_t* t = cand + ((int64_t)q * B + c) * n;
    // all positions are requested at once (one round trip, not one per accepted token)
    int32_t gg[kMaxStages], tt[kMaxStages];
#pragma unroll
    for (int p = 0; p < kMaxStages; ++p) {
      gg[p] = p < n ? g[p] : 0;
      tt[p] = p < n ? t[p] : -1;
    }
    int a = 0;
    bool run = c < nc;
#pragma unroll
    for (int p = 0; p < kMaxStages; ++p) {
      run = run && p < n && gg[p] == tt[p];
      a += run ? 1 : 0;
    }
    if (accept_all) accept_all[(int64_t)q * B + c] = a;
    if (c < max(nc, 1) && before((float)a, c, bv, bi)) { bv = (float)a; bi = c; }
  }
  wave_best(bv, bi);
  const int a = (int)bv, best = bi;
  if (lane == 0) {
    accept_len[q] = a;
    best_cand[q] = best;
    n_out[q] = a + 1;
  }
  const int32_t* g = greedy + ((int64_t)q * B + best) * (n + 1);
  const int32_t* t = cand + ((int64_t)q * B + best) * n;
  for (int p = lane; p <= n; p += 64) out_tokens[(int64_t)q * (n + 1) + p] = p < a ? t[p] : (p == a ? g[a] : -1);
}

hipError_t launch_accept(const int32_t* greedy, const int32_t* cand, const int32_t* n_cand, int batch, int B, int n,
                         int32_t* accept_len, int32_t* best_cand, int32_t* out_tokens, int32_t* n_out,
                         int32_t* accept_all, hipStream_t st) {
  hipLaunchKernelGGL(accept_kernel, dim3(batch), dim3(64), 0, st, greedy, cand, n_cand, B, n, accept_len, best_cand,
                     out_tokens, n_out, accept_all);
  return hipGetLastError();
}

}  // namespace specdraft
