// float32 path (the small exact configuration: every tensor and every sum in float32, none
// rounded to 16 bits) and the bf16 tiling kernel.  A row's partial sums are joined with the fast
// exponential (1e-6): over 40 models of 500 .. 8000 x 128 .. 768 the log-sum-exp is 9.2e-8 off 64 bits
// (root mean square, relative), 2.3e-7 when a row was one sum over all of its logits.
#include "merge.h"
#include "spec_internal.h"

namespace specdraft {

// ---- tiling of a row-major bf16 matrix into matrix-core fragment order -------
__global__ __launch_bounds__(256) void pack_bf16_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst,
                                                        int n_rows, int kt, int64_t n_slots, int weights) {
  const int64_t slot = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (slot >= n_slots) return;
  const int lane = (int)(slot & 63);
  const int64_t frag = slot >> 6;
  const int t = (int)(frag % kt);
  const int64_t nt = frag / kt;
  const int64_t row = nt * 16 + (lane & 15);
  uint4* const d = dst + (weights ? nt * packed_tile_slots(kt) : nt * kt * 64) + t * 64 + lane;
  if (row < n_rows) {
    *d = src[row * (kt * 4) + t * 4 + (lane >> 4)];   // 8 bf16 = one 16-byte unit
  } else if (weights) {
    *d = make_uint4(0, 0, 0, 0);
  }
}

hipError_t launch_pack_bf16(const void* src, void* dst, int n_rows, int k, bool weights, hipStream_t st) {
  const int kt = k / 32;
  const int64_t n_slots = (int64_t)((n_rows + 15) / 16) * kt * 64;
  const unsigned grid = (unsigned)((n_slots + 255) / 256);
  hipLaunchKernelGGL(pack_bf16_kernel, dim3(grid), dim3(256), 0, st, static_cast<const uint4*>(src),
                     static_cast<uint4*>(dst), n_rows, kt, n_slots, weights ? 1 : 0);
  return hipGetLastError();
}

// ---- float32 contraction on the float32 matrix instruction -------------------
// Workgroup = 16 waves = 4 tiles of 16 weight rows x 4 parts of K, against 16 state rows (blockIdx.y, z).
// A wave multiplies its 16 x 16 tile over its K part with v_mfma_f32_16x16x4_f32 (float32 products and
// sums), both operands straight from memory in 16-byte pieces: lane l holds row l % 16, columns
// 16 s + 4 (l / 16) .. + 4 of step s, and the four instructions of a step take element 0 .. 3 of every
// lane, the same assignment of K to lanes on both sides.  The K parts are summed through LDS in order;
// then wave r holds state row r, lane c the logit of weight row c of the 64: log-sum-exp pieces and the
// k best leave as one partial per (row, workgroup), logits are not written.  The next stage's projection
// is a second list of tiles in the same launch.
//
// Bound: launch latency and one trip through memory per stage (256 x 1024 model: 1 MB per head).  A vector-ALU
// contraction with logits in memory and a scan per row took 24 + 6 us per stage, and 22 us for its projection; the
// whole draft of that model 177.5 -> 46.9 us.  A stage of at most 16 rows is computed inside the head's launch by every workgroup
// (fold_row_f32): its launch, 2.8 to 4.6 us of a few rows, was a start, two trips to memory and a drain; inside, the head's weights
// arrive with the row's last loads.  That, and lists as short as what a lane sees: the draft of that model 43.6 -> 36.2 us.
constexpr int kF32Tiles = 4, kF32Parts = 4, kF32Cols = 16 * kF32Tiles;
constexpr int kF32GridY = 32768;   // row tiles along y; more go along z
constexpr int kF32Batch = 4;   // steps whose loads are in flight together

struct F32Args {
  const float* a;            // states [R][K]
  const float* w[2];         // weights [n][K]: head, projection (or the only matrix)
  int n[2], blocks[2];       // rows; workgroups along the weight rows
  int per;                   // 64-row blocks a head workgroup covers
  float* out[2];             // store target of the matrix (head: null = partials)
  int64_t ldo[2];
  int R, K, k_top, nparts;
  int vec;                   // rows start on 16 bytes
  Partials part;
};

__device__ __forceinline__ f32x4 load_f32x4(const float* row, int k, int K, int vec) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (vec) {                 // K is a multiple of 4
    if (k < K) v = *reinterpret_cast<const f32x4*>(row + k);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (k + i < K) v[i] = row[k + i];
  }
  return v;
}

// The stage step for one row by one wave, into `row` (LDS): the merge of its parent's partials (at most 64, one per lane), the
// gather, LayerNorm and GELU of the stage kernel in that kernel's order of sums, so the same bits.  A lane holds NC chunks of
// eight elements (D <= 512 NC).  K as in stage_rows; `behind` is called when the last loads that the row waits for have been
// requested.
constexpr int kFoldF32Dim = 1024, kFoldF32Rows = 16, kFoldF32Parts = 64;
template <int K, int NC, typename F>
__device__ __forceinline__ void fold_row_f32(const StageJob& j, int r, float* row, bool tables, F&& behind) {
  const int lane = threadIdx.x & 63, D = j.D, nchunk = D / 8;
  int parent = r / j.k_prev, rank = r - parent * j.k_prev;
  if (j.row_parent) {
    parent = j.row_parent[r];
    rank = j.row_rank[r];
  }
  constexpr int KM = K > 0 ? K : 1;
  const int k = j.k_prev, part = min(lane, j.nparts - 1);
  float pm = 0.f, ps = 0.f, pv[KM];
  int32_t pi[KM], tok = 0;
  if (K > 0) {
    const int64_t at = (int64_t)parent * j.nparts + part;
    pm = j.part.m[at];
    ps = j.part.s[at];
#pragma unroll
    for (int e = 0; e < KM; ++e) {
      pv[e] = j.part.val[at * k + min(e, k - 1)];
      pi[e] = j.part.idx[at * k + min(e, k - 1)];
    }
  } else {
    tok = j.last_tok[parent];
  }
  float zp[NC][8], ga[NC][8], be[NC][8];
  auto load8 = [](float (&x)[8], const float* src) {
    const float4 lo = *reinterpret_cast<const float4*>(src), hi = *reinterpret_cast<const float4*>(src + 4);
    x[0] = lo.x; x[1] = lo.y; x[2] = lo.z; x[3] = lo.w;
    x[4] = hi.x; x[5] = hi.y; x[6] = hi.z; x[7] = hi.w;
  };
  int at8[NC];   // (past the row: its last chunk again, masked where it would count)
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    at8[c] = min(lane + 64 * c, nchunk - 1) * 8;
    load8(zp[c], j.pz + (int64_t)parent * D + at8[c]);
    load8(ga[c], j.gamma + at8[c]);
    load8(be[c], j.beta + at8[c]);
  }

  float best_v[KM], lse = 0.f;
  int32_t best_i[KM];
  if (K > 0) {
    const uint64_t kEmpty = best_key(SPEC_NEG_INF, kIdxNone);
    const bool ok = lane < j.nparts;
    uint64_t hk[KM];
#pragma unroll
    for (int e = 0; e < KM; ++e) hk[e] = ok && e < k ? best_key(pv[e], pi[e]) : kEmpty;
    const float m = ok ? pm : SPEC_NEG_INF, mx = wave_max(m);
    lse = mx + logf(wave_sum(m > SPEC_NEG_INF ? (ok ? ps : 0.f) * __expf(m - mx) : 0.f));
#pragma unroll
    for (int e = 0; e < KM; ++e) {
      best_v[e] = SPEC_NEG_INF;
      best_i[e] = kIdxNone;
      if (e < k) {
        const uint64_t top = wave_best_key(hk[0]);
        const bool won = hk[0] == top;   // the owner of the winner pops it
#pragma unroll
        for (int q = 0; q + 1 < KM; ++q) {
          const uint64_t up = opaque_key(hk[q + 1]);
          hk[q] = won ? up : hk[q];
        }
        hk[KM - 1] = won ? kEmpty : hk[KM - 1];
        best_unkey(top, best_v[e], best_i[e]);
        tok = e == rank ? best_i[e] : tok;
      }
    }
  }
  const int64_t t = min(max(tok, 0), j.V - 1);   // a wild token from the caller must not leave the table
  float em[NC][8];
#pragma unroll
  for (int c = 0; c < NC; ++c) load8(em[c], static_cast<const float*>(j.emb) + t * D + at8[c]);
  behind();
  if (K > 0 && tables && rank == 0) {
#pragma unroll
    for (int e = 0; e < KM; ++e)
      if (lane == e && e < k) {
        j.prev_tok[(int64_t)parent * k + e] = best_i[e];
        j.prev_logp[(int64_t)parent * k + e] = best_v[e] - lse;
      }
    if (lane == 0) j.prev_lse[parent] = lse;
  }
  float z[NC][8], mean = 0.f, var = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      z[c][q] = stage_mix(j.w_s, zp[c][q], j.w_e, em[c][q]);
      sum += z[c][q];
    }
    mean += wave_sum(lane + 64 * c < nchunk ? sum : 0.f);
  }
  mean /= (float)D;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float d = z[c][q] - mean;
      sum += d * d;
    }
    var += wave_sum(lane + 64 * c < nchunk ? sum : 0.f);
  }
  const float rstd = 1.0f / sqrtf(var / (float)D + j.eps);
#pragma unroll
  for (int c = 0; c < NC; ++c) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float y = (z[c][q] - mean) * rstd * ga[c][q] + be[c][q];
      z[c][q] = 0.5f * y * (1.0f + erf_as(y * 0.70710678118654752440f));
    }
    if (lane + 64 * c < nchunk) {
      *reinterpret_cast<float4*>(row + at8[c]) = make_float4(z[c][0], z[c][1], z[c][2], z[c][3]);
      *reinterpret_cast<float4*>(row + at8[c] + 4) = make_float4(z[c][4], z[c][5], z[c][6], z[c][7]);
    }
  }
}

// LIST: entries of a lane's list, at most as many as it sees logits of a row (p.per).  FOLD: >= 0: the states are not in memory
// yet; every workgroup computes the stage's rows itself, one per wave, FOLD = K of fold_row_f32.
template <int LIST, int FOLD, int NC>
__global__ __launch_bounds__(1024) void contract_f32_kernel(F32Args p, StageJob j) {
  __shared__ f32x4 lds[kF32Tiles * kF32Parts * 64];
  extern __shared__ __align__(16) float folded[];   // [R][K + 4]: rows of neighbouring lanes 16 bytes apart in the banks
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tile = wave & (kF32Tiles - 1), kp = wave / kF32Tiles;
  const int mat = (int)blockIdx.x >= p.blocks[0] ? 1 : 0;
  const int block = blockIdx.x - (mat ? p.blocks[0] : 0);
  const int n = p.n[mat], per = mat ? 1 : p.per;
  const int r0 = (int)(blockIdx.z * kF32GridY + blockIdx.y) * 16;
  if (r0 >= p.R) return;
  const int steps = (p.K + 15) / 16, s0 = kp * steps / kF32Parts, s1 = (kp + 1) * steps / kF32Parts;
  const int arow_at = min(r0 + (lane & 15), p.R - 1);
  const float* arow = FOLD >= 0 ? folded + arow_at * (p.K + 4) : p.a + (int64_t)arow_at * p.K;
  const int kl = 4 * (lane >> 4);

  f32x4 wv[kF32Batch];
  auto load_w = [&](const float* wrow, int s) {
#pragma unroll
    for (int u = 0; u < kF32Batch; ++u)   // (past the part: zeros)
      wv[u] = load_f32x4(wrow, s + u < s1 ? (s + u) * 16 + kl : p.K, p.K, p.vec);
  };
  auto weight_row = [&](int v0) { return p.w[mat] + (int64_t)min(v0 + tile * 16 + (lane & 15), n - 1) * p.K; };
  if (FOLD >= 0) {
    auto first = [&]() { load_w(weight_row(block * per * kF32Cols), s0); };
    const int row_w = __builtin_amdgcn_readfirstlane(wave);
    if (row_w < p.R) fold_row_f32<FOLD < 0 ? 0 : FOLD, NC>(j, row_w, folded + row_w * (p.K + 4), blockIdx.x == 0, first);
    else first();
    __syncthreads();
  }

  float run_m = kLowest, run_s = 0.f;
  const uint64_t kEmpty = best_key(SPEC_NEG_INF, kIdxNone);
  uint64_t best[LIST];
#pragma unroll
  for (int q = 0; q < LIST; ++q) best[q] = kEmpty;
  const int row = r0 + wave;             // of the closing part

  for (int b = 0; b < per; ++b) {
    const int v0 = (block * per + b) * kF32Cols;
    if (v0 >= n) break;
    const float* wrow = weight_row(v0);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s = s0; s < s1; s += kF32Batch) {
      f32x4 av[kF32Batch];
      if (FOLD < 0 || b > 0 || s > s0) load_w(wrow, s);
#pragma unroll
      for (int u = 0; u < kF32Batch; ++u)
        av[u] = load_f32x4(arow, s + u < s1 ? (s + u) * 16 + kl : p.K, p.K, FOLD >= 0 ? 1 : p.vec);
#pragma unroll
      for (int u = 0; u < kF32Batch; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[u][i], av[u][i], acc, 0, 0, 0);
    }
    // accumulator lane l: state row l % 16, weight rows (l / 16) * 4 + i of the tile
    __syncthreads();                     // (the previous block's sums have been read)
    lds[wave * 64 + lane] = acc;
    __syncthreads();
    const int c = lane;                  // weight row of the block: tile c / 16, (c % 16) / 4 * 16 + state row, entry c % 4
    const float* P = reinterpret_cast<const float*>(lds) + ((c >> 4) * 64 + ((c & 15) >> 2) * 16 + wave) * 4 + (c & 3);
    float x = 0.f;
#pragma unroll
    for (int q = 0; q < kF32Parts; ++q) x += P[q * kF32Tiles * 64 * 4];
    const int v = v0 + c;
    if (row < p.R && v < n) {
      if (p.out[mat]) {
        p.out[mat][(int64_t)row * p.ldo[mat] + v] = x;
      } else {
        const float m = fmaxf(run_m, x);
        run_s = run_s * expf(run_m - m) + expf(x - m);
        run_m = m;
        uint64_t key = best_key(x, v);
#pragma unroll
        for (int q = 0; q < LIST; ++q) {   // down the list, the smaller of each pair moves on
          const uint64_t old = best[q];
          best[q] = key > old ? key : old;
          key = key > old ? old : key;
        }
      }
    }
  }
  if (p.out[mat] || row >= p.R) return;  // (a whole wave)
  const float mx = wave_max(run_m);
  const float sum = wave_sum(run_s * expf(run_m - mx));
  const int64_t slot = (int64_t)row * p.nparts + block;
  if (lane == 0) {
    p.part.m[slot] = mx;
    p.part.s[slot] = sum;
  }
#pragma unroll
  for (int j = 0; j < kMaxTopK; ++j) {
    if (j < p.k_top) {
      const uint64_t top = wave_best_key(best[0]);
      const bool won = best[0] == top && top != kEmpty;   // the owner of the winner pops it
#pragma unroll
      for (int q = 0; q + 1 < LIST; ++q) {
        const uint64_t up = opaque_key(best[q + 1]);
        best[q] = won ? up : best[q];
      }
      best[LIST - 1] = won ? kEmpty : best[LIST - 1];
      if (lane == j) {
        float bv;
        int32_t bi;
        best_unkey(top, bv, bi);
        p.part.val[slot * p.k_top + j] = bv;
        p.part.idx[slot * p.k_top + j] = bi;
      }
    }
  }
}

template <int FOLD, int NC>
static hipError_t launch_folded_f32_t(const F32Args& p, dim3 grid, const StageJob& fold, hipStream_t st) {
  constexpr size_t most = (size_t)kFoldF32Rows * (512 * NC + 4) * 4;   // with the static part more than the 64 KiB of the default
  static bool attr_set = NC == 1;  // per instantiation
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(contract_f32_kernel<1, FOLD, NC>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL((contract_f32_kernel<1, FOLD, NC>), grid, dim3(1024), (size_t)p.R * (p.K + 4) * 4, st, p, fold);
  return hipGetLastError();
}
template <int NC>
static hipError_t launch_folded_f32(const F32Args& p, dim3 grid, const StageJob& fold, hipStream_t st) {
  switch (fold.stage == 0 ? 0 : fold.k_prev) {
    case 0: return launch_folded_f32_t<0, NC>(p, grid, fold, st);
    case 1: return launch_folded_f32_t<1, NC>(p, grid, fold, st);
    case 2: return launch_folded_f32_t<2, NC>(p, grid, fold, st);
    case 3: return launch_folded_f32_t<3, NC>(p, grid, fold, st);
    case 4: return launch_folded_f32_t<4, NC>(p, grid, fold, st);
    case 5:
    case 6: return launch_folded_f32_t<6, NC>(p, grid, fold, st);
    default: return launch_folded_f32_t<8, NC>(p, grid, fold, st);
  }
}

static hipError_t launch_contract_f32(F32Args& p, hipStream_t st, const StageJob* fold = nullptr) {
  // 16-byte loads need every row of both operands on a 16-byte boundary
  p.vec = (p.K % 4 == 0 && ((reinterpret_cast<uintptr_t>(p.a) | reinterpret_cast<uintptr_t>(p.w[0]) |
                             reinterpret_cast<uintptr_t>(p.w[1])) & 15) == 0) ? 1 : 0;
  const int rt = (p.R + 15) / 16;
  dim3 grid(p.blocks[0] + p.blocks[1], rt < kF32GridY ? rt : kF32GridY, (rt + kF32GridY - 1) / kF32GridY);
  StageJob none = {};
  if (!fold) {
    if (p.per == 1) hipLaunchKernelGGL((contract_f32_kernel<1, -1, 1>), grid, dim3(1024), 0, st, p, none);
    else hipLaunchKernelGGL((contract_f32_kernel<kMaxTopK, -1, 1>), grid, dim3(1024), 0, st, p, none);
    return hipGetLastError();
  }
  return p.per != 1 ? hipErrorInvalidValue : p.K <= 512 ? launch_folded_f32<1>(p, grid, *fold, st) : launch_folded_f32<2>(p, grid, *fold, st);
}

hipError_t launch_store_f32(const float* a, const float* w, float* out, int64_t ldo, int R, int N, int K, hipStream_t st) {
  F32Args p = {};
  p.a = a; p.R = R; p.K = K;
  p.w[0] = w; p.n[0] = N; p.blocks[0] = (N + kF32Cols - 1) / kF32Cols; p.out[0] = out; p.ldo[0] = ldo;
  p.per = 1;
  return launch_contract_f32(p, st);
}

// Fold where every workgroup can hold the stage's rows (one per wave, a merge of one partial per lane) and the head has one
// block per workgroup.  Drafts with such stages, 315 of D = 64 to 768, 500 to 8000 x 1 to 16 sequences: 1.10 times as fast on
// average, D = 512, 16 chains of four 73 -> 57 us; none slower than its repetition.  With more than 16 rows the blocks of every row
// tile would repeat the work.
bool f32_fold_fits(int R, int D, int V, int nparts, int max_parts, int64_t half) {
  return R <= kFoldF32Rows && D <= kFoldF32Dim && nparts <= kFoldF32Parts && (V + kF32Cols - 1) / kF32Cols <= max_parts &&
         (int64_t)kFoldF32Rows * max_parts <= half;
}

hipError_t launch_head_f32(const float* a, const float* w_head, int n_head, int k_top, Partials part, int max_parts,
                           const float* w_proj, int n_proj, float* out_proj, int R, int K, int* nparts, hipStream_t st,
                           const StageJob* fold) {
  F32Args p = {};
  p.a = a; p.R = R; p.K = K;
  p.w[0] = w_head; p.n[0] = n_head; p.k_top = k_top; p.part = part;
  // as many parts per row as the partial results' buffer holds: longer heads take several blocks per workgroup
  const int nb = (n_head + kF32Cols - 1) / kF32Cols;
  p.per = (nb + max_parts - 1) / max_parts;
  p.blocks[0] = (nb + p.per - 1) / p.per;
  p.nparts = *nparts = p.blocks[0];
  if (n_proj > 0) {
    p.w[1] = w_proj; p.n[1] = n_proj; p.blocks[1] = (n_proj + kF32Cols - 1) / kF32Cols;
    p.out[1] = out_proj; p.ldo[1] = n_proj;
  }
  return launch_contract_f32(p, st, fold);
}

__global__ __launch_bounds__(256) void row_log_softmax_kernel(const float* __restrict__ logits,
                                                              float* __restrict__ logp, int64_t ld, int V) {
  __shared__ float scratch[8];
  const int64_t row = blockIdx.x;
  const int tid = threadIdx.x;
  const float* x = logits + row * ld;
  float mx = SPEC_NEG_INF;
  for (int i = tid; i < V; i += 256) mx = fmaxf(mx, x[i]);
  mx = block_max<256>(mx, scratch);
  float s = 0.f;
  for (int i = tid; i < V; i += 256) s += expf(x[i] - mx);
  s = block_sum<256>(s, scratch);
  const float lse = mx + logf(s);
  float* y = logp + row * ld;
  for (int i = tid; i < V; i += 256) y[i] = x[i] - lse;
}

hipError_t launch_row_log_softmax(const float* logits, float* logp, int64_t ld, int R, int V, hipStream_t st) {
  hipLaunchKernelGGL(row_log_softmax_kernel, dim3(R), dim3(256), 0, st, logits, logp, ld, V);
  return hipGetLastError();
}

// Plain copy of n 16-byte words, grid-stride: a launch whose HBM traffic is known
// exactly (n * 16 bytes read, n * 16 written), used to calibrate traffic counters.
__global__ __launch_bounds__(256) void copy_probe_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst,
                                                         int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) dst[i] = src[i];
}

hipError_t launch_copy_probe(const void* src, void* dst, int64_t n16, hipStream_t st) {
  const int64_t want = (n16 + 255) / 256;
  const int grid = (int)(want < 1 ? 1 : (want > 16384 ? 16384 : want));
  hipLaunchKernelGGL(copy_probe_kernel, dim3(grid), dim3(256), 0, st, static_cast<const u32x4*>(src),
                     static_cast<u32x4*>(dst), n16);
  return hipGetLastError();
}

}  // namespace specdraft
