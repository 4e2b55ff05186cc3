// Vocabulary head (and the next stage's projection) for 17 .. 32 state rows: the
// bandwidth-bound regime of a handful of sequences, or of a chain on a loaded server.
//
// Bound: HBM (each weight is used for at most 32 rows).  The streaming kernel of <= 16 rows keeps its
// states in LDS; 32 rows of K = 4096 are 256 KB and do not fit.  They fit the register file: K is split
// over the 16 waves of the CU's one workgroup, so a wave only ever needs ITS K slice of the states, NS
// fragments per 16-row tile, and holds them in 8 * NS registers for the whole launch (64 of its 128 at
// K = 4096).  The rest is the streaming design: tile = 16 weight rows x all of K, workgroup g takes tiles
// g, g + G, ... of [head | projection], weights go straight to a register ring of DEPTH tiles (128 KB per CU and
// tile in flight), the 16 partial accumulators are summed through double-buffered LDS, one barrier per tile, and
// the running (max, sum-exp, top-k) never leaves the CU.  No state traffic after the start.
// Measured against the dense kernel's 64-row tiles, which re-read the states with every tile and leave a launch of
// 1.1 .. 1.6 tiles per range two tiles long: 32000 + 4096 weight rows x 4096, 25 rows: 70.9 -> 48.5 us
// (6.1 TB/s); 49152 + 4096 x 4096, 24 rows: 86.0 -> 66.8 us (6.5 TB/s).  What is
// left beside the stream (7.6 TB/s between those two sizes) is about 10 us per launch of start, last tile and merge.
#include <hip/hip_ext.h>

#include "device_utils.h"
#include "spec_internal.h"

namespace specdraft {

constexpr int kS32Waves = 16;
constexpr int kS32Steps = 8;   // K-steps (of 32) per wave -> K <= 4096
// Longest head: a line of results, not of speed.  Against 128256 rows of 3072 this kernel takes 128 us and the dense one
// 150, but its sums over 16 slices of K (error against 64 bits 0.9 .. 1.0 of the other's) turned the order of near-tied
// candidates of a 6, 4, 3, 2 tree in 1 of 10 seeds: 3 % of the whole numbers of its token tree, where 1 % is the bound
// that such a draft is held to.  With 32000 and 49152 rows ten seeds stayed within it; between 65536 and 128256 nothing
// was measured.
constexpr int kS32MaxHead = 65536;
// slots of one wave's 16x16 accumulator in LDS: the four 16-lane groups are 20 slots apart, so that the
// 16 threads that read one state row's sums hit distinct banks
constexpr int kS32Group = 20;
constexpr int kS32Acc = 3 * kS32Group + 16;
constexpr size_t kS32LdsP = (size_t)2 * kS32Waves * 2 * kS32Acc * 16;
constexpr size_t kS32Lds = kS32LdsP + (size_t)kMaxTopK * 512 * 8;   // + the epilogue threads' top-k lists

// A tile costs 0.9 us of 16 waves, a barrier and an epilogue however short K is, so many tiles of few columns stay with
// the dense kernel, whose waves share nothing.  24 rows, us here / there:  16000 rows of K = 64, 256:  9.2 / 9.9,
// 9.9 / 10.5;  32000 of 64, 256, 384, 512:  12.5 / 10.2, 13.2 / 11.5, 13.2 / 13.4, 14.1 / 14.9;  65536 of 64, 256, 512,
// 768, 1024:  19.4 / 13.2, 19.8 / 15.9, 21.5 / 18.9 (with a projection 21.1 / 21.6), 22.0 / 22.7, 25.5 / 27.6.
// Hence four tiles per workgroup, or one per 48 columns.
bool skinny32_fits(int R, int kt, int n_head, int n_cu) {
  const int tiles = kt * 32 / 48 > 4 ? kt * 32 / 48 : 4;   // of a workgroup
  return R > 16 && R <= 32 && n_head > 0 && n_head <= kS32MaxHead && (kt + kS32Waves - 1) / kS32Waves <= kS32Steps &&
         (n_head + 15) / 16 <= (int64_t)tiles * skinny_grid(n_cu);
}
size_t skinny32_lds_bytes() { return kS32Lds; }

template <int NS, int DEPTH>
__global__ __launch_bounds__(kS32Waves * 64) void head_skinny32_kernel(HeadJob p) {
  extern __shared__ __align__(16) unsigned char smem[];
  f32x4* ldsP = reinterpret_cast<f32x4*>(smem);   // [2][waves][2][kS32Acc]
  // an epilogue thread's sorted list of 64-bit keys (best_key), entry q at [q * 512 + tid]: beside the states
  // and the weight ring it has no registers left, and it is touched once per tile of several thousand cycles
  uint64_t* ldsK = reinterpret_cast<uint64_t*>(smem + kS32LdsP);
  const int wg = blockIdx.x, G = gridDim.x;
  const int kt = p.kt, R = p.R, slots = p.tile_slots;
  const int tid = opaque_tid(), lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: tile addresses stay in scalar registers

  // ---- this wave's slice of K: steps [s0, s0 + ns), ns <= NS
  const int spw = (kt + kS32Waves - 1) / kS32Waves;
  const int s0 = min(w * spw, kt), ns = min(kt, s0 + spw) - s0;
  const int total = p.vt_head + p.vt_proj;
  // The wave's slice of a tile as a buffer of ns KiB: fragments past the slice, and every fragment of a tile
  // past the last one (0 records), read as zero without touching memory.  So the refill of the ring has no
  // branch, and the compiler's wait counters leave the whole ring in flight.
  const u32x4* wh = static_cast<const u32x4*>(p.w_head);
  const u32x4* wp = static_cast<const u32x4*>(p.w_proj);
  auto tile_slice = [&](int tile) {
    const int t = min(tile, total - 1);
    const u32x4* base = t < p.vt_head ? wh + packed_tile_start(t, slots) : wp + packed_tile_start(t - p.vt_head, slots);
    return weight_buffer(base + (int64_t)s0 * 64, tile < total ? ns * 1024 : 0);
  };

  // ---- the slice of the states: fragment (row tile, K-step), lane l = row l % 16, columns 8 (l / 16) .. + 8
  // (requested before the weights: the first matrix instruction needs both)
  u32x4 st[2][NS];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    // packed tiles: one K-step is 64 16-byte words; row-major rows: 4 words of the row
    const int row = min(rt * 16 + (lane & 15), R - 1);
    const int64_t at = p.b_rowmajor ? ((int64_t)row * p.b_ld) / 8 + (lane >> 4) : (int64_t)rt * kt * 64 + lane;
    const u32x4* src = static_cast<const u32x4*>(p.b_src) + at;
    const int step = p.b_rowmajor ? 4 : 64;
#pragma unroll
    for (int t = 0; t < NS; ++t) st[rt][t] = src[(int64_t)min(s0 + min(t, max(ns - 1, 0)), kt - 1) * step];
  }
  // ---- the first DEPTH tiles
  u32x4 a[DEPTH][NS];
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) {
    const auto buf = tile_slice(wg + d * G);
#pragma unroll
    for (int t = 0; t < NS; ++t) a[d][t] = load_weight(buf, lane * 16 + t * 1024);
  }

  // running state of the 512 epilogue threads: state row en, weight row vi of the tile (16 consecutive
  // threads own one state row: their closing merge runs on DPP)
  const int en = (tid >> 4) & 31, vi = tid & 15;
  float run_m = kLowest, run_s = 0.f;
  const uint64_t kEmpty = best_key(SPEC_NEG_INF, kIdxNone);
  if (tid < 512) {
#pragma unroll
    for (int q = 0; q < kMaxTopK; ++q) ldsK[q * 512 + tid] = kEmpty;
  }

  int buf = 0;
  auto one_tile = [&](u32x4 (&ad)[NS], int tile) {
        const auto nbuf = tile_slice(tile + DEPTH * G);
        __builtin_amdgcn_sched_barrier(0);
        f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < NS; ++t) {
          const bf16x8 wf = __builtin_bit_cast(bf16x8, ad[t]);
          acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, __builtin_bit_cast(bf16x8, st[0][t]), acc0, 0, 0, 0);
          acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, __builtin_bit_cast(bf16x8, st[1][t]), acc1, 0, 0, 0);
          ad[t] = load_weight(nbuf, lane * 16 + t * 1024);
        }
#pragma unroll
        for (int t = 0; t < NS; ++t) {   // a fragment is requested again as soon as it is consumed
          __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        f32x4* mine = ldsP + (buf * kS32Waves + w) * 2 * kS32Acc + (lane >> 4) * kS32Group + (lane & 15);
        mine[0] = acc0;
        mine[kS32Acc] = acc1;
        __syncthreads();
        if (tid < 512) {
          // accumulator lane l holds state row l % 16 and weight rows (l / 16) * 4 + i
          const float* P = reinterpret_cast<const float*>(ldsP + buf * kS32Waves * 2 * kS32Acc) +
                           ((en >> 4) * kS32Acc + (vi >> 2) * kS32Group + (en & 15)) * 4 + (vi & 3);
          float sum = 0.f;
#pragma unroll 4
          for (int ww = 0; ww < kS32Waves; ++ww) sum += P[ww * 2 * kS32Acc * 4];
          if (en < R) {
            if (tile < p.vt_head) {
              const int v = tile * 16 + vi;
              if (v < p.n_head) {
                if (p.out_head) {
                  p.out_head[(int64_t)en * p.ld_head + v] = sum;
                } else {
                  const float m_new = fmaxf(run_m, sum);
                  run_s = run_s * __expf(run_m - m_new) + __expf(sum - m_new);
                  run_m = m_new;
                  uint64_t x = best_key(sum, v);
#pragma unroll 1
                  for (int q = 0; q < p.k_top; ++q) {   // down the list, the smaller of each pair moves on
                    const uint64_t old = ldsK[q * 512 + tid];
                    ldsK[q * 512 + tid] = x > old ? x : old;
                    x = x > old ? old : x;
                  }
                }
              }
            } else {
              const int d2 = (tile - p.vt_head) * 16 + vi;
              if (d2 < p.n_proj) p.out_proj[(int64_t)en * p.ld_proj + d2] = sum;
            }
          }
        }
        buf ^= 1;
  };
  int base = wg;
  for (; base + (DEPTH - 1) * G < total; base += DEPTH * G) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) one_tile(a[d], base + d * G);
  }
#pragma unroll
  for (int d = 0; d + 1 < DEPTH; ++d)   // the last round, if it is not a whole one
    if (base + d * G < total) one_tile(a[d], base + d * G);

  if (p.out_head || p.vt_head == 0) return;

  // ---- merge the 16 residue lists of each row (16 consecutive lanes) into the workgroup's partial
  if (tid < 512) {
    const float mx = row16_max(run_m);
    // (always true; the product is rounded before it is added, not fused into one of the sum's two sides)
    const float s = row16_sum(run_m > SPEC_NEG_INF ? run_s * __expf(run_m - mx) : 0.f);
    const int64_t slot = (int64_t)en * p.nparts + wg;
    if (en < R && vi == 0) {
      p.part.m[slot] = mx;
      p.part.s[slot] = s;
    }
    uint64_t hk[kMaxTopK];
#pragma unroll
    for (int q = 0; q < kMaxTopK; ++q) hk[q] = ldsK[q * 512 + tid];
#pragma unroll
    for (int j = 0; j < kMaxTopK; ++j) {
      if (j < p.k_top) {
        const uint64_t best = row16_best_key(hk[0]);
        const bool won = hk[0] == best;   // the owner of the winner pops it
#pragma unroll
        for (int q = 0; q + 1 < kMaxTopK; ++q) {
          const uint64_t up = opaque_key(hk[q + 1]);
          hk[q] = won ? up : hk[q];
        }
        hk[kMaxTopK - 1] = won ? kEmpty : hk[kMaxTopK - 1];
        if (en < R && vi == j) {
          float bv;
          int32_t bi;
          best_unkey(best, bv, bi);
          p.part.val[slot * p.k_top + j] = bv;
          p.part.idx[slot * p.k_top + j] = bi;
        }
      }
    }
  }
}

template <int NS, int DEPTH>
static hipError_t launch_skinny32_t(const HeadJob& job, int grid, hipStream_t st, hipEvent_t ev_start,
                                    hipEvent_t ev_stop) {
  static bool attr_set = false;  // per instantiation
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(head_skinny32_kernel<NS, DEPTH>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kS32Lds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipExtLaunchKernelGGL((head_skinny32_kernel<NS, DEPTH>), dim3(grid), dim3(kS32Waves * 64), kS32Lds, st,
                        ev_start, ev_stop, 0, job);
  return hipGetLastError();
}

hipError_t launch_head_skinny32(const HeadJob& job, int n_cu, hipStream_t st, hipEvent_t ev_start,
                                hipEvent_t ev_stop) {
  const int grid = skinny_grid(n_cu);
  // 8 fragments of a wave in flight, or as near as whole tiles come, are 128 KiB of a CU and saturate HBM; half as much again
  // only queues there.  Launches of 17 to 32 rows with 12 and now 8 (K = 2048) or 6 (3072) of them, us: 32003 rows of 2048
  // 25.4 -> 23.7, 65024 of 2048 44.3 -> 43.1, 32000 of 3072 32.7 -> 31.8, 65024 of 3072 65.9 -> 64.9.  Shorter K within an
  // instance leaves fragments of a tile unused: there the deeper ring.
  const int ns = (job.kt + kS32Waves - 1) / kS32Waves;
  if (ns == 4) return launch_skinny32_t<4, 2>(job, grid, st, ev_start, ev_stop);
  if (ns < 4) return launch_skinny32_t<4, 3>(job, grid, st, ev_start, ev_stop);
  if (ns == 6) return launch_skinny32_t<6, 1>(job, grid, st, ev_start, ev_stop);
  if (ns < 6) return launch_skinny32_t<6, 2>(job, grid, st, ev_start, ev_stop);
  return launch_skinny32_t<kS32Steps, 1>(job, grid, st, ev_start, ev_stop);
}

}  // namespace specdraft
