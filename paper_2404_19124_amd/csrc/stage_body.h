// Device-side bodies of the stage step and of the tree step (Sec. 3.1, 4.1 of the
// paper).
#pragma once
#include "merge.h"
#include "spec_internal.h"

namespace specdraft {

// KC sibling nodes of a stage, computed by a whole workgroup of NT threads: the children rank0 .. of row `parent` of
// the stage before, as rows r0 .. of this one (those past the parent's last child, `live` < KC, are not stored):
//   state = GELU(LayerNorm(w_s * (W s_parent) + w_e * Emb[token]))
// The token a node carries is the rank-th best of its parent's head row; that row's partial results are merged here, once
// for the KC siblings (which saves a separate launch on the latency-critical batch-1 chain).
// K: entries per partial list that registers are kept for (>= k_prev; 0: stage 0, where the token is given).
// NCH = 8-element chunks per thread held in registers (D <= NCH * NT * 8).
// `lds`: 32 * KC + kMergeLds words of scratch.  Contains workgroup barriers.
// A chain of trips to memory is what a row takes, so what hangs on nothing is requested up front, the partial lists
// before all else, without a branch between two requests (the compiler waits for what is on its way where paths join);
// the other parts of a split projection come with the embedding row.
// (Lists requested behind a wait for the projection, its parts one trip each: 24 rows of top-1, D = 4096, 5.8 us, now 5.1;
// 15 rows of top-3 6.4, now 5.5.)
// States are stored as whole 16-byte slots; the L2 gathers the eight rows that share a 128-byte line.
template <bool BF16, int K, int NCH, int NT, int KC>
__device__ __forceinline__ void stage_rows(const StageJob& j, int parent, int rank0, int r0, int live, float* lds) {
  const int tid = opaque_tid();
  const int D = j.D, nchunk = D / 8;

  MergePart<K ? K : 1> list;
  if (K) group_merge_load<K ? K : 1>(j.part, parent, j.nparts, j.k_prev, list);
  const float* pz = j.pz + (int64_t)parent * D;
  float zp[NCH][8], ga[NCH][8], be[NCH][8];
  auto load8 = [](float (&x)[8], const float* src) {
    const float4 a = *reinterpret_cast<const float4*>(src), b = *reinterpret_cast<const float4*>(src + 4);
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
  };
  int at8[NCH];   // the thread's chunks (past the row: its last one again, masked where it would count)
#pragma unroll
  for (int ci = 0; ci < NCH; ++ci) {
    at8[ci] = min(tid + ci * NT, nchunk - 1) * 8;
    load8(zp[ci], pz + at8[ci]);
    load8(ga[ci], j.gamma + at8[ci]);
    load8(be[ci], j.beta + at8[ci]);
  }

  int tok[KC], at = kNoRank;
  float v = 0.f, lse = 0.f;
  int32_t ix = 0;
  if (K == 0) {
#pragma unroll
    for (int h = 0; h < KC; ++h) tok[h] = j.last_tok[parent];   // (uniform tree: parent == r)
  } else {
    group_merge_loaded<K ? K : 1>(list, j.part, parent, j.nparts, j.k_prev, v, ix, at, lse, lds + 32 * KC);
#pragma unroll
    for (int h = 0; h < KC; ++h) {
      const int rank = h < live ? rank0 + h : rank0;
      tok[h] = __builtin_amdgcn_readlane(ix, __ffsll((unsigned long long)__ballot(at == rank)) - 1);
    }
  }

  // gather
  uint4 raw[KC][NCH][BF16 ? 1 : 2];
#pragma unroll
  for (int h = 0; h < KC; ++h) {
    const int64_t t = min(max(tok[h], 0), j.V - 1);  // a wild token from the caller must not leave the table
    const uint4* row = reinterpret_cast<const uint4*>(static_cast<const char*>(j.emb) + t * D * (BF16 ? 2 : 4));
#pragma unroll
    for (int ci = 0; ci < NCH; ++ci)
#pragma unroll
      for (int u = 0; u < (BF16 ? 1 : 2); ++u) raw[h][ci][u] = row[(at8[ci] >> 3) * (BF16 ? 1 : 2) + u];
  }
  // a projection split along K: its other parts, added in order.  All three there can be on their way at once; rows past 4096
  // elements, whose threads hold two chunks: as many as leave the kernel below 129 registers, so that two workgroups share a
  // CU.  (Four in both cases, 130 to 166 registers: D = 6144, 255 parents of 6 36.0 us, 255 rows of stage 0 9.9, and now 26.5 and
  // 8.1; one chunk, D = 4096, 255 parents of 3 11.4, now 10.0.  Three siblings of 6144 together with two parts 18.4, with one 16.1.)
  static_assert(kMaxKSplit == 4, "three other parts");
  constexpr int PU = NCH == 1 ? 3 : NCH == 2 && KC == 3 ? 1 : 2;
  for (int q0 = 1; q0 < j.pz_parts; q0 += PU) {
    float pq[PU][NCH][8];
#pragma unroll
    for (int u = 0; u < PU; ++u)
#pragma unroll
      for (int ci = 0; ci < NCH; ++ci)
        load8(pq[u][ci], pz + min(q0 + u, j.pz_parts - 1) * j.pz_part_stride + at8[ci]);
#pragma unroll
    for (int u = 0; u < PU; ++u)
#pragma unroll
      for (int ci = 0; ci < NCH; ++ci)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const float sum = zp[ci][q] + pq[u][ci][q];
          zp[ci][q] = q0 + u < j.pz_parts ? sum : zp[ci][q];
        }
  }
  if (K && rank0 == 0 && tid < 64 && at < j.k_prev) {   // (behind the requests: a wait for those would wait for these)
    j.prev_tok[(int64_t)parent * j.k_prev + at] = ix;
    j.prev_logp[(int64_t)parent * j.k_prev + at] = v - lse;
    if (at == 0) j.prev_lse[parent] = lse;
  }
  // mix
  float z[KC][NCH][8], lsum[KC];
#pragma unroll
  for (int h = 0; h < KC; ++h) {
    lsum[h] = 0.f;
#pragma unroll
    for (int ci = 0; ci < NCH; ++ci) {
      const bool counts = tid + ci * NT < nchunk;
      float sum = lsum[h];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const uint4 w = raw[h][ci][BF16 ? 0 : q >> 2];
        const uint32_t word = (BF16 ? q >> 1 : q & 3) == 0 ? w.x : (BF16 ? q >> 1 : q & 3) == 1 ? w.y
                              : (BF16 ? q >> 1 : q & 3) == 2 ? w.z : w.w;
        const float e = !BF16 ? __uint_as_float(word)
                        : (q & 1) ? bf16_bits_to_f32(word >> 16) : bf16_bits_to_f32(word & 0xffffu);
        z[h][ci][q] = stage_mix(j.w_s, zp[ci][q], j.w_e, e);
        sum += z[h][ci][q];
      }
      lsum[h] = counts ? sum : lsum[h];
    }
  }
  float mean[KC], lvar[KC], rstd[KC];
  block_sums<NT, KC>(lsum, lds);
#pragma unroll
  for (int h = 0; h < KC; ++h) {
    mean[h] = lsum[h] / (float)D;
    lvar[h] = 0.f;
#pragma unroll
    for (int ci = 0; ci < NCH; ++ci) {
      const bool counts = tid + ci * NT < nchunk;
      float sum = lvar[h];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float d = z[h][ci][q] - mean[h];
        sum += d * d;
      }
      lvar[h] = counts ? sum : lvar[h];
    }
  }
  block_sums<NT, KC>(lvar, lds + 16 * KC);
#pragma unroll
  for (int h = 0; h < KC; ++h) rstd[h] = 1.0f / sqrtf(lvar[h] / (float)D + j.eps);

#pragma unroll
  for (int h = 0; h < KC; ++h) {
    if (h >= live) break;
    const int r = r0 + h;
#pragma unroll
    for (int ci = 0; ci < NCH; ++ci) {
      const int c = tid + ci * NT;
      if (c < nchunk) {
        float s[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const float y = (z[h][ci][q] - mean[h]) * rstd[h] * ga[ci][q] + be[ci][q];
          s[q] = 0.5f * y * (1.0f + erf_as(y * 0.70710678118654752440f));
        }
        if (BF16) {
          uint4 o;
          o.x = f32_to_bf16_pair(s[0], s[1]);
          o.y = f32_to_bf16_pair(s[2], s[3]);
          o.z = f32_to_bf16_pair(s[4], s[5]);
          o.w = f32_to_bf16_pair(s[6], s[7]);
          // tiled layout: row tile r/16, column fragment c/4, lane slot (c%4)*16 + r%16
          const int64_t slot = ((int64_t)(r >> 4) * (D / 32) + (c >> 2)) * 64 + ((c & 3) << 4) + (r & 15);
          reinterpret_cast<uint4*>(j.state_out)[slot] = o;
          if (j.state_dbg) reinterpret_cast<uint4*>(j.state_dbg)[((int64_t)r * D) / 8 + c] = o;
        } else {
          float* so = static_cast<float*>(j.state_out) + (int64_t)r * D + c * 8;
          *reinterpret_cast<float4*>(so) = make_float4(s[0], s[1], s[2], s[3]);
          *reinterpret_cast<float4*>(so + 4) = make_float4(s[4], s[5], s[6], s[7]);
          if (j.state_dbg) {
            float* sd = static_cast<float*>(j.state_dbg) + (int64_t)r * D + c * 8;
            *reinterpret_cast<float4*>(sd) = make_float4(s[0], s[1], s[2], s[3]);
            *reinterpret_cast<float4*>(sd + 4) = make_float4(s[4], s[5], s[6], s[7]);
          }
        }
      }
    }
  }
}

// Tree step for one sequence q, by a whole workgroup of NT threads: merge the last
// head's partial results, score every leaf by the sum of its tokens' log-probabilities
// (added in stage order), keep the B best.
struct TreeArgs {
  int n, B, B_pad, L, k_last, kw_last, nparts;
  int64_t off_last, row_off_last;   // the last stage's offsets in tok / logp and in lse
  int64_t rbase_last;               // first row of this sequence at the last stage
  Partials part;                    // last head
  int32_t* tok;                     // per-stage tables [R_i][width_i], concatenated
  float* logp;
  float* lse;
  int32_t* cand_tokens;
  float* cand_scores;
  int32_t* cand_leaf;
};

// One sequence q of the tree step, by a whole workgroup of NT threads.
// B candidates are kept out of L = prod(k_i) leaves; k_last = this sequence's branching at the last
// stage, kw_last = width of the last stage's tables and partial lists (>= k_last; equal for a uniform
// tree).  B = 0 (speculation off): only padding is written.
// s_k / s_off / s_rbase / s_kw: per stage, in LDS (indexing kernel arguments with a run-time stage
// number would make the compiler spill the argument block to scratch): this sequence's branching,
// the table's element offset, this sequence's first row, the table's width.
// sk: kMaxLeaves 64-bit words of LDS (the leaves' scores as keys, see best_key); c_tok / c_logp: kMaxLeaves words
// each, the last stage's tables of this sequence for the leaf scores (the tables in memory are written all
// the same: the debug outputs and the caller's next step read them).
// KWAVE: widest kw_last there is (merged one row per wave: register-hungry for wide lists, a wave of a 1024-thread
// workgroup has 128 registers); 0: the tables of the last stage are there already.  Contains workgroup barriers.
template <int NT, int KWAVE>
__device__ __forceinline__ void tree_body(const TreeArgs& j, int q, const int* s_k, const int64_t* s_off,
                                          const int64_t* s_rbase, const int* s_kw, uint64_t* sk,
                                          int32_t* c_tok, float* c_logp) {
  const int tid = opaque_tid(), lane = tid & 63, wave = tid >> 6;
  const int n = j.n, L = j.L, kw = j.kw_last;
  const int rows_last = j.B > 0 ? L / j.k_last : 0;
  const int nleaf = j.B > 0 ? L : 0;

  // A leaf's path, walking up from the leaf: q_{n-1} = leaf, q_{i-1} = q_i / k_i; its node at stage i is
  // row q_{i-1} of the sequence with rank q_i - q_{i-1} k_i.  at[i] = element of stage i's table.
  // All of a leaf's table reads are issued together: one round trip, not one per stage.
  auto path_of = [&](int leaf, int64_t (&at)[kMaxStages]) {
    int q = leaf;
#pragma unroll
    for (int i = kMaxStages - 1; i >= 0; --i) {
      at[i] = 0;
      if (i < n) {
        const int k = s_k[i];
        // q < 4096, k <= 8: the float quotient of q + 1/2 is farther from an integer than its rounding error
        const int up = (int)(((float)q + 0.5f) * __frcp_rn((float)k));
        at[i] = s_off[i] + (s_rbase[i] + up) * s_kw[i] + (q - up * k);
        q = up;
      }
    }
  };
  // One leaf per thread and the last stage's tables small enough for LDS (the paper's trees): a leaf's
  // entries of the EARLIER stages are requested before the merge and arrive under it; the last stage's
  // come from the merge through LDS.  The leaf scores then wait for no memory at all.
  const bool one_pass = nleaf <= NT;   // every thread has at most one leaf: its tokens stay in registers
  constexpr int kEarly = 3;            // earlier stages whose entries a thread holds across the merge (registers)
  const bool early = KWAVE > 0 && one_pass && n - 1 <= kEarly && (int64_t)rows_last * kw <= kMaxLeaves;
  float lp_e[kEarly];
  int32_t tk_e[kEarly];
  int last_at = 0;
  if (early && tid < nleaf) {
    int64_t at[kMaxStages];
    path_of(tid, at);
#pragma unroll
    for (int i = 0; i < kMaxStages; ++i) {
      if (i < kEarly) {
        lp_e[i] = i < n - 1 ? j.logp[at[i]] : 0.f;
        tk_e[i] = i < n - 1 ? j.tok[at[i]] : 0;
      }
      if (i == n - 1) last_at = (int)(at[i] - (j.off_last + j.rbase_last * kw));
    }
  }

  if (KWAVE > 0) {
    // (the first wave has just spent its time on the leaves' paths: it stays out of the merge when the
    // other waves cover the rows in one pass)
    const int w0 = (early && rows_last <= NT / 64 - 1) ? 1 : 0;
    for (int rl = wave - w0; rl >= 0 && rl < rows_last; rl += NT / 64 - w0) {
      const int64_t row = j.rbase_last + rl;
      float v[kMaxTopK];
      int32_t ix[kMaxTopK];
      float lse;
      if (KWAVE >= kMaxTopK) {
        wave_merge_partials(j.part, row, j.nparts, kw, v, ix, lse);
      } else {
        switch (kw) {
          case 1: wave_merge_partials_k<1>(j.part, row, j.nparts, kw, v, ix, lse); break;
          case 2: wave_merge_partials_k<2>(j.part, row, j.nparts, kw, v, ix, lse); break;
          case 3: wave_merge_partials_k<3>(j.part, row, j.nparts, kw, v, ix, lse); break;
          default: wave_merge_partials_k<4>(j.part, row, j.nparts, kw, v, ix, lse); break;
        }
      }
#pragma unroll
      for (int t = 0; t < kMaxTopK; ++t)
        if (lane == t && t < kw) {
          j.tok[j.off_last + row * kw + t] = ix[t];
          j.logp[j.off_last + row * kw + t] = v[t] - lse;
          if (early) {
            c_tok[rl * kw + t] = ix[t];
            c_logp[rl * kw + t] = v[t] - lse;
          }
        }
      if (lane == 0) j.lse[j.row_off_last + row] = lse;
    }
    __threadfence_block();
    __syncthreads();
  }

  int32_t tk[kMaxStages];
  if (early) {
    if (tid < nleaf) {
      float score = 0.f;   // added in stage order
#pragma unroll
      for (int i = 0; i < kMaxStages; ++i) {
        tk[i] = 0;
        if (i < kEarly && i < n - 1) {
          score += lp_e[i];
          tk[i] = tk_e[i];
        }
        if (i == n - 1) {
          score += c_logp[last_at];
          tk[i] = c_tok[last_at];
        }
      }
      sk[tid] = best_key(score, tid);
    }
  } else {
    for (int leaf = tid; leaf < nleaf; leaf += NT) {
      int64_t at[kMaxStages];
      path_of(leaf, at);
      float lp[kMaxStages];
#pragma unroll
      for (int i = 0; i < kMaxStages; ++i) {
        lp[i] = i < n ? j.logp[at[i]] : 0.f;
        tk[i] = (one_pass && i < n) ? j.tok[at[i]] : 0;
      }
      float score = 0.f;
#pragma unroll
      for (int i = 0; i < kMaxStages; ++i)
        if (i < n) score += lp[i];
      sk[leaf] = best_key(score, leaf);
    }
  }
  // (the ranking reads two keys at a time: fill the last pair)
  if (tid == 0 && (nleaf & 1) && nleaf < kMaxLeaves) sk[nleaf] = 0;
  __syncthreads();

  // rank of a leaf = number of leaves before it in (score, then smaller leaf index): one 64-bit compare each
  for (int leaf = tid; leaf < nleaf; leaf += NT) {
    const uint64_t mine = sk[leaf];
    int pos = 0;
#pragma unroll 4
    for (int o = 0; o < nleaf; o += 2) {
      const uint64_t k0 = sk[o], k1 = sk[o + 1];
      pos += k0 > mine ? 1 : 0;
      pos += k1 > mine ? 1 : 0;
    }
    float s;
    int32_t self;
    best_unkey(mine, s, self);
    if (pos < j.B) {
      const int64_t c = (int64_t)q * j.B_pad + pos;
      j.cand_leaf[c] = leaf;
      j.cand_scores[c] = s;
      if (!one_pass) {
        int64_t at[kMaxStages];
        path_of(leaf, at);
#pragma unroll
        for (int i = 0; i < kMaxStages; ++i) tk[i] = i < n ? j.tok[at[i]] : 0;
      }
#pragma unroll
      for (int i = 0; i < kMaxStages; ++i)
        if (i < n) j.cand_tokens[c * n + i] = tk[i];
    }
  }
  // slots past this sequence's candidates: padding
  for (int pos = j.B + tid; pos < j.B_pad; pos += NT) {
    const int64_t c = (int64_t)q * j.B_pad + pos;
    j.cand_leaf[c] = -1;
    j.cand_scores[c] = SPEC_NEG_INF;
    for (int i = 0; i < n; ++i) j.cand_tokens[c * n + i] = -1;
  }
}

// Fills the per-sequence arguments of tree_body for sequence q from a TreeJob: lanes 0 .. n-1 of EVERY wave
// write the LDS arrays (the same values: a wave may then read them back without a workgroup barrier, its own
// LDS accesses execute in order), every thread computes the scalars.  Call with all threads.
__device__ __forceinline__ void tree_args_for_sequence(const TreeJob& j, int q, TreeArgs& a, int* s_k, int64_t* s_off,
                                                       int64_t* s_rbase, int* s_kw) {
  const int tid = opaque_tid();
  const int n = j.n;
  a.n = n; a.B_pad = j.B_pad; a.nparts = j.nparts;
  a.part = j.part; a.tok = j.tok; a.logp = j.logp; a.lse = j.lse;
  a.cand_tokens = j.cand_tokens; a.cand_scores = j.cand_scores; a.cand_leaf = j.cand_leaf;
  a.B = j.B; a.L = j.L; a.k_last = 1; a.kw_last = 1; a.off_last = 0; a.row_off_last = 0; a.rbase_last = 0;
  const int32_t* d = j.seq_desc ? j.seq_desc + (int64_t)q * (2 * n + 1) : nullptr;
  if (d) {
    a.B = d[2 * n];
    a.L = 1;
  }
  int64_t cnt = 1;   // rows of one sequence at stage i (uniform tree)
#pragma unroll
  for (int i = 0; i < kMaxStages; ++i) {
    if (i < n) {
      const int k = d ? d[i] : j.top_k[i];
      const int64_t rbase = d ? (int64_t)d[n + i] : (int64_t)q * cnt;
      if (d) a.L *= k;
      if ((tid & 63) == i) { s_k[i] = k; s_off[i] = j.off[i]; s_rbase[i] = rbase; s_kw[i] = j.kstride[i]; }
      if (i == n - 1) {
        a.k_last = k; a.kw_last = j.kstride[i]; a.off_last = j.off[i]; a.row_off_last = j.row_off[i];
        a.rbase_last = rbase;
      }
      cnt *= k;
    }
  }
}

}  // namespace specdraft
