// Token tree of a sequence's candidates and the hand-over to the next step
// (Sec. 3.1 of the paper: multi-candidate decoding with tree attention; the base model
// is stage 0 of the next draft).
#include "device_utils.h"
#include "spec_internal.h"

namespace specdraft {

// One workgroup per sequence.  Item i = (c, p) stands for the prefix cand[c, :p+1].
//   first(c, p) = the smallest c' whose prefix of the same length is equal
//   a prefix is a node where first(c, p) == c; nodes are numbered in item order.
// Bound: a chain of LDS passes of one workgroup (nothing to stream but the mask).  Depth by depth, a candidate
// looks for the first one with the same first(., p - 1) and the same token: two words per comparison whatever the
// depth, four comparisons per trip; the numbering is a scan over ballots; the mask is cleared in 16-byte stores while
// that runs.  (Whole prefixes compared token by token, a count over all earlier items per item and single-byte
// stores: 18 us for 16 sequences of 32 candidates x 3, calls back to back; one word after the other per comparison:
// 9.4, and slower than that on chains and trees of a few candidates; now 6.4.)
// M = B * n <= kMaxTreeItems.  Dynamic LDS: 3 * M ints.
__global__ __launch_bounds__(256) void tree_meta_kernel(const int32_t* __restrict__ cand, int B, int n,
                                                        int32_t* node_tok, int32_t* node_parent, int32_t* node_depth,
                                                        int32_t* n_nodes, int32_t* cand_node, uint8_t* mask) {
  extern __shared__ int32_t lds[];
  __shared__ int s_wave[4];
  const int M = B * n;
  // depth-major: entry (c, p) at [p * B + c]
  int32_t* tok = lds;            // [M]
  int32_t* first = lds + M;      // [M] candidate first(c, p)
  int32_t* nid = lds + 2 * M;    // [M] node number of a prefix, where first(c, p) == c
  const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int32_t* cq = cand + (int64_t)q * M;
  if (B == 1) {   // a chain: every prefix is a node (24 chains of 7: 4.5 us through the passes below, 2.2 here)
    for (int p = tid; p < n; p += 256) {
      node_tok[(int64_t)q * M + p] = cq[p];
      node_parent[(int64_t)q * M + p] = p - 1;
      node_depth[(int64_t)q * M + p] = p + 1;
      cand_node[(int64_t)q * M + p] = p;
    }
    if (tid == 0) n_nodes[q] = n;
    if (mask)
      for (int i = tid; i < n * n; i += 256) mask[(int64_t)q * n * n + i] = i % n <= i / n ? 1 : 0;
    return;
  }
  // item i -> candidate i / n by a reciprocal: (i + 0.5) / n is at least 0.5 / n from every whole number, the product at
  // most 4096 / n * 2^-22 off
  const float rn = 1.0f / (float)n;
  auto cand_of = [&](int i) { return (int)(((float)i + 0.5f) * rn); };
  for (int i = tid; i < M; i += 256) {
    const int c = cand_of(i), p = i - c * n;
    tok[p * B + c] = cq[i];
  }
  if (mask) {
    uint8_t* mq = mask + (int64_t)q * M * M;
    const int64_t bytes = (int64_t)M * M;
    const int64_t lead0 = (int64_t)((16 - (reinterpret_cast<uintptr_t>(mq) & 15)) & 15);
    const int64_t lead = lead0 < bytes ? lead0 : bytes, n16 = (bytes - lead) / 16;
    if (tid < lead) mq[tid] = 0;
    u32x4* mv = reinterpret_cast<u32x4*>(mq + lead);
#pragma unroll 4
    for (int i = tid; i < (int)n16; i += 256) mv[i] = (u32x4){0, 0, 0, 0};
    if (tid < bytes - lead - n16 * 16) mq[lead + n16 * 16 + tid] = 0;
  }
  __syncthreads();
  for (int p = 0; p < n; ++p) {
    const int32_t* tp = tok + p * B;
    const int32_t* fp = first + (p - 1) * B;   // (at depth 0: the tail of tok[], read and not used)
    for (int c = tid; c < B; c += 256) {
      const int t = tp[c], f0 = p ? fp[c] : 0;
      int f = c;
      // (the first candidate of the longer prefix is not before the first of the shorter one)
      for (int c2 = f0; c2 < f; c2 += 4) {
        int ot[4], of[4];   // all eight words are requested before the first is looked at
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          ot[u] = tp[min(c2 + u, c)];
          of[u] = fp[min(c2 + u, c)];
        }
#pragma unroll
        for (int u = 3; u >= 0; --u)
          if ((ot[u] == t) & ((p == 0) | (of[u] == f0))) f = min(f, c2 + u);
      }
      first[p * B + c] = f;
    }
    __syncthreads();
  }
  // numbering in item order
  int total = 0;
  for (int i0 = 0; i0 < M; i0 += 256) {
    const int i = i0 + tid, c = cand_of(i), p = i - c * n;
    const bool node = i < M && first[p * B + c] == c;
    const uint64_t votes = __ballot(node);
    if (lane == 0) s_wave[wave] = __popcll(votes);
    __syncthreads();
    int before = total;
    for (int w = 0; w < 4; ++w) {
      if (w < wave) before += s_wave[w];
      total += s_wave[w];
    }
    if (node) nid[p * B + c] = before + __popcll(votes & (((uint64_t)1 << lane) - 1));
    __syncthreads();
  }
  if (tid == 0) n_nodes[q] = total;
  for (int i = tid; i < M; i += 256) {
    const int c = cand_of(i), p = i - c * n, f = first[p * B + c];
    const int me = nid[p * B + f];
    cand_node[(int64_t)q * M + i] = me;
    if (f == c) {
      node_tok[(int64_t)q * M + me] = tok[p * B + c];
      node_depth[(int64_t)q * M + me] = p + 1;
      node_parent[(int64_t)q * M + me] = p == 0 ? -1 : nid[(p - 1) * B + first[(p - 1) * B + c]];
      if (mask) {
        uint8_t* row = mask + ((int64_t)q * M + me) * M;
        for (int j = 0; j <= p; ++j) row[nid[j * B + first[j * B + c]]] = 1;
      }
    }
  }
  // entries past the last node
  for (int i = total + tid; i < M; i += 256) {
    node_tok[(int64_t)q * M + i] = -1;
    node_parent[(int64_t)q * M + i] = -1;
    node_depth[(int64_t)q * M + i] = 0;
  }
}

hipError_t launch_tree_meta(const int32_t* cand, int batch, int B, int n, int32_t* node_tok, int32_t* node_parent,
                            int32_t* node_depth, int32_t* n_nodes, int32_t* cand_node, uint8_t* mask,
                            hipStream_t st) {
  const size_t smem = (size_t)3 * B * n * sizeof(int32_t);
  hipLaunchKernelGGL(tree_meta_kernel, dim3(batch), dim3(256), smem, st, cand, B, n, node_tok, node_parent, node_depth,
                     n_nodes, cand_node, mask);
  return hipGetLastError();
}

// next_state[q] = hidden[q, best[q], accept[q], :], next_tok[q] = out_tokens[q, accept[q]].
// Indices are clamped to their ranges (a corrupted accept length must not leave the tensor).
__global__ __launch_bounds__(256) void advance_kernel(const uint8_t* __restrict__ hidden, int64_t row_bytes, int B, int n,
                                                      const int32_t* best, const int32_t* accept,
                                                      const int32_t* out_tokens, uint8_t* next_state,
                                                      int32_t* next_tok) {
  const int q = blockIdx.x;
  const int c = min(max(best[q], 0), B - 1), a = min(max(accept[q], 0), n);
  const uint8_t* src = hidden + (((int64_t)q * B + c) * (n + 1) + a) * row_bytes;
  uint8_t* dst = next_state + (int64_t)q * row_bytes;
  if ((row_bytes & 15) == 0 && ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15) == 0) {
    for (int64_t i = threadIdx.x; i < row_bytes / 16; i += 256)
      reinterpret_cast<u32x4*>(dst)[i] = reinterpret_cast<const u32x4*>(src)[i];
  } else {
    for (int64_t i = threadIdx.x; i < row_bytes; i += 256) dst[i] = src[i];
  }
  if (threadIdx.x == 0) next_tok[q] = out_tokens[(int64_t)q * (n + 1) + a];
}

hipError_t launch_advance(const void* hidden, int64_t row_bytes, int batch, int B, int n, const int32_t* best,
                          const int32_t* accept, const int32_t* out_tokens, void* next_state, int32_t* next_tok,
                          hipStream_t st) {
  hipLaunchKernelGGL(advance_kernel, dim3(batch), dim3(256), 0, st, static_cast<const uint8_t*>(hidden), row_bytes, B, n,
                     best, accept, out_tokens, static_cast<uint8_t*>(next_state), next_tok);
  return hipGetLastError();
}

}  // namespace specdraft
