// Stage kernel (Sec. 3.1 of the paper): for every node of the current depth,
//   state = GELU(LayerNorm(w_s * (W s_parent) + w_e * Emb[token]))
// The token a node carries is the j-th best of its parent's head row; that row's
// partial results are merged here (which saves a separate launch on the latency-critical batch-1 chain).
#include "stage_body.h"

#include <cstring>

namespace specdraft {

// Parents from which siblings share a workgroup: one for every CU.  With fewer, what a CU saves others do not lend (a child is
// 2 us of arithmetic on one CU).  Together and one by one, us: D = 4096, 16 parents of 6 11.2 and 8.5, 64 of 5 11.6 and 10.9, 96 of
// 4 11.9 and 10.2, 320 of 3 16.9 and 17.1; D = 3072, 32 of 6 12.2 and 10.0, 192 of 4 12.8 and 13.8, 768 of 3 21.0 and 29.4.
constexpr int kSiblingParents = 256;

// K: the width that registers are kept for, see stage_rows; NCH = 8-element chunks per thread (D <= NCH * NT * 8).  One
// row per workgroup (every sibling repeats its parent's merge).
template <bool BF16, int K, int NCH, int NT>
__global__ __launch_bounds__(NT) void stage_kernel(StageJob j) {
  __shared__ __align__(16) float lds[32 + kMergeLds];
  int r = blockIdx.x;
  if (j.xcd_rows) {
    // Workgroup ids go round-robin over the 8 XCDs, and a row's state is stored as one 16-byte slot in
    // each of D / 8 lines that it shares with the other rows of its 16-row tile.  Rows of one tile on
    // eight XCDs leave every L2 with an eighth of each line to write back; here the 16 rows of a tile
    // run on one XCD, whose L2 puts the lines together (7B shape, 64 sequences: -7 us per step).
    const int xcd = blockIdx.x & 7, s = blockIdx.x >> 3;
    r = (((s >> 4) << 3) + xcd) * 16 + (s & 15);
    if (r >= j.R) return;
  }
  int parent = r / j.k_prev, rank = r - parent * j.k_prev;
  if (j.row_parent) {  // per-sequence trees: the host laid the rows out
    parent = j.row_parent[r];
    rank = j.row_rank[r];
  }
  stage_rows<BF16, K, NCH, NT, 1>(j, parent, rank, r, 1, lds);
}

// KC siblings per workgroup, `per` workgroups per parent (uniform trees, packed states).  The merge and the parent's
// projection are read and computed once for the siblings, which are a third to a half of a row's instructions.
// Bound: vector ALU (38 instructions per element of a row).  2304 rows of 3 siblings, D = 3072: 28.3 us one by one, 21.0 so.
template <int K, int NCH, int NT, int KC>
__global__ __launch_bounds__(NT) void stage_siblings_kernel(StageJob j, int per, int group) {
  __shared__ __align__(16) float lds[32 * KC + kMergeLds];
  // `group` parents have whole 16-row tiles of children: they run on one XCD (see above)
  const int xcd = blockIdx.x & 7, s = blockIdx.x >> 3, span = group * per;
  const int g = s / span, in = s - g * span, pin = in / per;
  const int parent = (g * 8 + xcd) * group + pin;
  const int rank0 = (in - pin * per) * KC, r0 = parent * j.k_prev + rank0;
  if (r0 >= j.R) return;
  stage_rows<true, K, NCH, NT, KC>(j, parent, rank0, r0, min(KC, j.k_prev - rank0), lds);
}

template <int K, int NCH, int NT>
static hipError_t launch_siblings(const StageJob& job, hipStream_t st) {
  constexpr int KC = K <= 4 ? K : K / 2;   // (widths 5 and 6: 3 of 6, 7 and 8: 4 of 8)
  const int k = job.k_prev, parents = job.R / k, per = (k + KC - 1) / KC;
  const int group = 16 / ((k & 1) ? 1 : (k & 2) ? 2 : (k & 4) ? 4 : 8);
  const int groups = (parents + group - 1) / group;
  const dim3 grid((groups + 7) / 8 * 8 * group * per);
  hipLaunchKernelGGL((stage_siblings_kernel<K, NCH, NT, KC>), grid, dim3(NT), 0, st, job, per, group);
  return hipGetLastError();
}

template <bool BF16, int K, int NCH, int NT>
static hipError_t launch_stage_n(const StageJob& job, hipStream_t st) {
  if constexpr (BF16 && K >= 2 && NCH <= 2)
    if (job.xcd_rows && !job.row_parent && job.R / job.k_prev >= kSiblingParents) return launch_siblings<K, NCH, NT>(job, st);
  // tile-per-XCD order: whole groups of 8 tiles, the workgroups past the last row leave at once
  const dim3 grid(job.xcd_rows ? (job.R + 127) / 128 * 128 : job.R);
  hipLaunchKernelGGL((stage_kernel<BF16, K, NCH, NT>), grid, dim3(NT), 0, st, job);
  return hipGetLastError();
}

template <bool BF16, int K>
static hipError_t launch_stage_k(const StageJob& job, hipStream_t st) {
  const int nchunk = job.D / 8;
  // 512 threads per row from D = 4096 on: the row's LayerNorm / GELU arithmetic is what a workgroup spends its
  // time on once its loads are back, and eight waves halve it (7B batch 1: -1 us per step; 7-stage chain: -3.6 us)
  if (nchunk <= 256) return launch_stage_n<BF16, K, 1, 256>(job, st);
  if (nchunk <= 512) return launch_stage_n<BF16, K, 1, 512>(job, st);
  if (nchunk <= 1024) return launch_stage_n<BF16, K, 2, 512>(job, st);
  if (nchunk <= 2048) return launch_stage_n<BF16, K, 4, 512>(job, st);
  return hipErrorInvalidValue;
}

template <bool BF16>
static hipError_t launch_stage_t(const StageJob& job, hipStream_t st) {
  if (job.stage == 0) return launch_stage_k<BF16, 0>(job, st);
  switch (job.k_prev) {
    case 1: return launch_stage_k<BF16, 1>(job, st);
    case 2: return launch_stage_k<BF16, 2>(job, st);
    case 3: return launch_stage_k<BF16, 3>(job, st);
    case 4: return launch_stage_k<BF16, 4>(job, st);
    case 5:
    case 6: return launch_stage_k<BF16, 6>(job, st);
    default: return launch_stage_k<BF16, 8>(job, st);
  }
}

hipError_t launch_stage(const StageJob& job, hipStream_t st) {
  return job.bf16 ? launch_stage_t<true>(job, st) : launch_stage_t<false>(job, st);
}

// Row maps of a call with per-sequence trees: a few KB straight from pinned host memory, every word requested at
// once (one trip over PCIe), and the candidate counts to the caller's array.  Two copies by the runtime in its place
// delayed the draft's first kernel by 15 us.  A workgroup that has read its words says so in pinned memory (`read`, one word
// each): an event behind the launch, or its own, made the draft's first kernel wait 6 or 5 us for its release to the host.
__global__ __launch_bounds__(kFetchWords) void fetch_maps_kernel(const int32_t* __restrict__ maps, int32_t* __restrict__ dev,
                                                                 int n, int32_t* __restrict__ n_cand, int batch, uint32_t* read,
                                                                 uint32_t ticket) {
  const int i = blockIdx.x * kFetchWords + threadIdx.x;
  if (i < n + batch) {
    const int32_t v = maps[i];
    if (i < n) dev[i] = v;
    else n_cand[i - n] = v;
  }
  __syncthreads();   // (a word has arrived where it has been stored)
  if (threadIdx.x == 0) __hip_atomic_store(read + blockIdx.x, ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

hipError_t launch_fetch_maps(const int32_t* maps, int32_t* dev, int n, int32_t* n_cand, int batch, uint32_t* read,
                             uint32_t ticket, hipStream_t st) {
  hipLaunchKernelGGL(fetch_maps_kernel, dim3(fetch_groups(n + batch)), dim3(kFetchWords), 0, st, maps, dev, n, n_cand, batch, read,
                     ticket);
  return hipGetLastError();
}

// The same for a call that is being recorded into a graph: the words travel in the arguments of the launches, which the graph keeps,
// so every replay finds those of its call, whatever later calls have put into the pinned memory.  One workgroup per launch and
// a launch per kMapWords words (3840 bytes of arguments): 24 sequences of a 5/3/2 tree are two.
struct MapWords {
  int32_t w[kMapWords];
};
__global__ __launch_bounds__(kMapWords) void store_maps_kernel(MapWords words, int count, int at, int32_t* __restrict__ dev, int n,
                                                               int32_t* __restrict__ n_cand) {
  const int i = threadIdx.x;
  if (i >= count) return;
  if (at + i < n) dev[at + i] = words.w[i];
  else n_cand[at + i - n] = words.w[i];
}

hipError_t launch_store_maps(const int32_t* maps, int32_t* dev, int n, int32_t* n_cand, int batch, hipStream_t st) {
  for (int at = 0; at < n + batch; at += kMapWords) {
    MapWords words = {};
    const int count = n + batch - at < kMapWords ? n + batch - at : kMapWords;
    memcpy(words.w, maps + at, (size_t)count * 4);
    hipLaunchKernelGGL(store_maps_kernel, dim3(1), dim3(kMapWords), 0, st, words, count, at, dev, n, n_cand);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// ---------------------------------------------------------------------------
// Tree kernel (Sec. 3.1, 4.1): merge the last head's partial results, score
// every leaf by the sum of its tokens' log-probabilities (added in stage order),
// keep the B best.  One workgroup per sequence.
// ---------------------------------------------------------------------------
// NT = 512: eight waves merge eight rows at a time and each wave may use 256 registers (the
// widest merges need more than the 128 a 1024-thread workgroup would leave).  NT = 1024 for
// last-stage top-k <= 4 (KWAVE = 4): sixteen rows per pass.
// KWAVE = 0: merge_rows_kernel has been here.
template <int NT, int KWAVE>
__global__ __launch_bounds__(NT) void tree_kernel(TreeJob j) {
  __shared__ __align__(16) uint64_t sk[kMaxLeaves];
  __shared__ int s_k[kMaxStages], s_kw[kMaxStages];
  __shared__ int64_t s_off[kMaxStages], s_rbase[kMaxStages];
  __shared__ int32_t c_tok[KWAVE ? kMaxLeaves : 1];
  __shared__ float c_logp[KWAVE ? kMaxLeaves : 1];
  TreeArgs a;
  tree_args_for_sequence(j, blockIdx.x, a, s_k, s_off, s_rbase, s_kw);
  // (no barrier here: a wave reads back only what it wrote itself, so it starts its loads while the later waves
  // of the workgroup are still being launched)
  tree_body<NT, KWAVE>(a, blockIdx.x, s_k, s_off, s_rbase, s_kw, sk, c_tok, c_logp);
}

// The last head's tables ahead of the tree kernel, one row per wave and workgroup, over the whole chip.  Bound: latency, one trip
// to memory and the merge's chain (4.6 us for 2304 rows as for 15).  A wave alone on its SIMD: no reason for larger workgroups.
template <int K>
__global__ __launch_bounds__(64) void merge_rows_kernel(TreeJob j) {
  const int64_t row = blockIdx.x;
  const int lane = threadIdx.x, kw = j.kstride[j.n - 1];
  const int64_t at = j.off[j.n - 1] + row * kw, row_at = j.row_off[j.n - 1] + row;
  float v[kMaxTopK], lse;
  int32_t ix[kMaxTopK];
  wave_merge_partials_k<K>(j.part, row, j.nparts, kw, v, ix, lse);
#pragma unroll
  for (int t = 0; t < K; ++t)
    if (lane == t && t < kw) {
      j.tok[at + t] = ix[t];
      j.logp[at + t] = v[t] - lse;
    }
  if (lane == 0) j.lse[row_at] = lse;
}

static void launch_merge_rows(const TreeJob& job, hipStream_t st) {
  const dim3 grid(job.rows_last), block(64);
  switch (job.kstride[job.n - 1]) {
    case 1: hipLaunchKernelGGL(merge_rows_kernel<1>, grid, block, 0, st, job); break;
    case 2: hipLaunchKernelGGL(merge_rows_kernel<2>, grid, block, 0, st, job); break;
    case 3: hipLaunchKernelGGL(merge_rows_kernel<3>, grid, block, 0, st, job); break;
    case 4: hipLaunchKernelGGL(merge_rows_kernel<4>, grid, block, 0, st, job); break;
    case 5:
    case 6: hipLaunchKernelGGL(merge_rows_kernel<6>, grid, block, 0, st, job); break;
    default: hipLaunchKernelGGL(merge_rows_kernel<8>, grid, block, 0, st, job); break;
  }
}

hipError_t launch_tree(const TreeJob& job, hipStream_t st) {
  // (per-sequence trees: the widest table decides the merge variant, rows_last is then an upper bound)
  const int kw_last = job.kstride[job.n - 1];
  const int rows_last = job.seq_desc ? kMaxLeaves : job.L / job.top_k[job.n - 1];
  // More rows per sequence than one pass of sixteen waves: a pass is 3 us and more of arithmetic on one CU while others
  // are idle, and the rows get a launch of their own.  Tree kernel alone, and both launches, us: 24 rows x 16 sequences
  // 16.2 and 13.0, 72 x 32 19.8 and 13.4; in one pass 15 x 64 12.2 and 11.8, 15 x 5 10.3 and 10.5, 15 x 1 8.5 and 9.6: the
  // line goes by the rows of a sequence alone, and from some dozens of sequences of 15 rows on it leaves 0.4 us behind.
  // The tree kernel then only scores and ranks: a leaf per thread up to 256, since small workgroups share a CU (256 leaves,
  // 256 and 1024 threads, us: 600 sequences 10.0 and 21.3, 32 sequences 8.3 and 8.0, 1 sequence 7.3 and 7.1); with more
  // leaves 1024 threads (320 leaves 15.3 and 9.1, 512 20.9 and 11.9).
  if (!job.seq_desc && rows_last > 16) {
    launch_merge_rows(job, st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (job.L <= 256) hipLaunchKernelGGL((tree_kernel<256, 0>), dim3(job.batch), dim3(256), 0, st, job);
    else hipLaunchKernelGGL((tree_kernel<1024, 0>), dim3(job.batch), dim3(1024), 0, st, job);
  } else if (kw_last <= 4 && rows_last > 8) {
    hipLaunchKernelGGL((tree_kernel<1024, 4>), dim3(job.batch), dim3(1024), 0, st, job);
  } else {
    hipLaunchKernelGGL((tree_kernel<512, kMaxTopK>), dim3(job.batch), dim3(512), 0, st, job);
  }
  return hipGetLastError();
}

}  // namespace specdraft
