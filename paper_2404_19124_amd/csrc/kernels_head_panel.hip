// Vocabulary head (and the next stage's projection) for some dozens of state rows, up to 128: the middle stages of a batched draft.
//
// Bound: HBM, each weight is used for at most 128 rows; what the streaming kernels of 32 rows and fewer do with states that stay
// in the CU, states that do not fit it (64 rows of 4096 are 512 KB) have to do from L2.
//  * Workgroup = 12 waves, one workgroup per CU; tile = up to nine 16-row weight tiles against all state rows.  Nine waves
//    multiply, one weight tile each: its fragments go from HBM straight into the wave's registers, D = 8 K-steps ahead (72 KiB of
//    a CU; 16 steps are 1 to 3 % slower where a CU has all nine tiles, the queue in front of the states grows), and
//    nothing else is in such a wave's queue, whose loads land in order.
//  * Three waves copy the states, a slab of KS K-steps at a time, straight into one of two LDS buffers (buffer loads to LDS); one
//    barrier per slab, not per step.  (Built and measured before, 64 / 96 / 320 rows of 32000 + 4096 x 4096: weights through LDS as
//    well, a barrier per K-step, 59 / 72 / 114 us; the time of a step was neither copies, nor LDS reads, nor matrix work: each
//    taken out alone leaves nine tenths of it.)
//  * The logits of a tile pass through LDS once, then eight lanes own a state row: 18 logits each, log-sum-exp and top-k merged by
//    DPP, one row group per wave.  (16 lanes to a row on nine waves: 3 us more per launch of 64 rows.)  Across the tiles of a range a
//    row carries its k best, one per lane, its maximum and its sum.
// A logit is one accumulator over K, in K order, as in the dense kernel of 32-row blocks: the same bits.
// Launches, dense kernels before and this one, us: 64 rows x 36096 x 4096 59.5 / 55.3, 96 rows 65.6 / 59.6, 75 rows x 32000 53.6 / 51.5,
// 48 rows x 36096 60.0 / 53.5, 32 rows x 131328 x 3072 151 / 131 (6.1 TB/s).  Left beside the stream (7.65 TB/s and 9.6 us of
// start and end in the streaming kernels): about 3 us of the states' copies and as much of the closing rows.
#include <hip/hip_ext.h>

#include <cstring>

#include "lane_lists.h"

namespace specdraft {

constexpr int kPanelWaves = 12;
constexpr int kPanelFrags = 9;    // 16-row weight fragments of a tile = waves that multiply, one fragment each
constexpr int kPanelCopy = kPanelWaves - kPanelFrags;   // waves that copy states
constexpr int kPanelCols = 16 * kPanelFrags;
constexpr int kPanelLd = kPanelCols + 8;                // floats between two rows of logits in LDS: eight rows of eight lanes, 64 banks
constexpr size_t kPanelLds = 160 * 1024;

struct PanelArgs {
  const u32x4* w[2];   // packed weights: head, projection
  int n_frags[2];      // their 16-row tiles
  int n_tiles[2];      // workgroup tiles of `ts` of them
  int ts, n_valid, kt, tile_slots;
  const u32x4* b;      // packed states
  int mt_total, R;
  int n_ranges;
  float* out;          // projection
  int64_t ldo;
  int k_top, nparts;
  Partials part;
};

// MF = 16-row state fragments.  (MF = 8 keeps 19 to 59 scalar registers, what the closing rows need of them, in lanes of a vector
// register: written once in front of the tiles, read back 2 to 6 at a time in the closing blocks of 350 to 750 instructions, none in a
// block that multiplies.  No more than some forty instructions of a wave's life, so nothing was given up for them.)
template <int MF>
struct PanelGeo {
  static constexpr int D = 8;                     // K-steps (of 32) of weights that a wave has on their way
  static constexpr int KS = MF <= 6 ? 8 : 4;      // K-steps of states in one of two LDS buffers
  static constexpr int SLAB = MF * KS * 1024;
  static constexpr int CP = (MF * KS + kPanelCopy - 1) / kPanelCopy;   // copies per slab of a copying wave
  static constexpr int PASS = (2 * MF + kPanelWaves - 1) / kPanelWaves;   // groups of eight rows per wave in the epilogue
  static constexpr int LOGITS_AT = 2 * SLAB;
  static constexpr int BYTES = LOGITS_AT + 16 * MF * kPanelLd * 4;
  static_assert(D % KS == 0 && BYTES <= (int)kPanelLds && CP < 64, "");
};

__device__ __forceinline__ void wait_copies() { __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8)); }   // vmcnt(0)
__device__ __forceinline__ void wave_barrier() {   // every LDS access of this wave has returned
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The lane, asked for anew: what hangs on it is then not computed ahead of the K loop and held across it.
__device__ __forceinline__ int lane_anew() {
  uint32_t none = 0;
  asm volatile("" : "+s"(none));
  return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, none));
}

template <int MF, int KT>
__global__ __launch_bounds__(kPanelWaves * 64) void head_panel_kernel(PanelArgs p) {
  extern __shared__ __align__(16) unsigned char smem[];
  using G = PanelGeo<MF>;
  constexpr int D = G::D, KS = G::KS;
  constexpr int NX = kPanelCols / 8;   // logits of a row that a lane closes
  const int range = blockIdx.x;
  const int total = p.n_tiles[0] + p.n_tiles[1];
  const int t0 = (int)((int64_t)range * total / p.n_ranges);
  const int t1 = (int)((int64_t)(range + 1) * total / p.n_ranges);

  const int tid = threadIdx.x, lane = tid & 63, lane16 = lane * 16;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kt = p.kt, groups = (kt + D - 1) / D, slabs = groups * (D / KS);   // of a tile
  lds_byte* const lds = (lds_byte*)smem;
  float* const logits = reinterpret_cast<float*>(smem + G::LOGITS_AT);

  // ---- weights of wave w: fragment w of the tile; past the tile, the matrix or the range: no records, zeros without memory
  auto tile_buf = [&](int t) {
    const int mat = t >= p.n_tiles[0] ? 1 : 0;
    const int f = (t - (mat ? p.n_tiles[0] : 0)) * p.ts + wave;
    const bool ok = t < t1 && wave < p.ts && f < p.n_frags[mat];
    return weight_buffer(p.w[mat] + packed_tile_start(ok ? f : 0, p.tile_slots), ok ? kt * 1024 : 0);
  };
  // ---- states: slab s (K-steps KS s .. of the tile) into LDS buffer of the running count, by the copying waves
  const auto states = weight_buffer(p.b, p.mt_total * kt * 1024);
  auto copy_slab = [&](int s, int at) {
#pragma unroll
    for (int i = 0; i < G::CP; ++i) {
      const int f = min(wave - kPanelFrags + i * kPanelCopy, MF * KS - 1);   // (the last one again: the same bytes)
      const int m = f / KS, k = s * KS + f % KS;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(states, (__attribute__((address_space(3))) void*)(lds + at + f * 1024), 16, lane16,
                                               (min(m, p.mt_total - 1) * kt + min(k, kt - 1)) * 1024, 0, 0);
    }
  };

  // running result of the rows this wave closes: eight lanes to a row, lane j of them the j-th best so far
  uint64_t run_key[G::PASS];
  float run_m[G::PASS], run_s[G::PASS];
  const uint64_t kEmpty = best_key(SPEC_NEG_INF, kIdxNone);
#pragma unroll
  for (int q = 0; q < G::PASS; ++q) { run_key[q] = kEmpty; run_m[q] = kLowest; run_s[q] = 0.f; }

  // Closes the rows whose logits are in LDS: eight lanes to a row, 18 logits each, log-sum-exp and the k best with those so far.
  auto close_rows = [&](int tile) {
    const int lane_e = lane_anew(), j = lane_e & 7;
    const int v0 = tile * p.ts * 16, v_end = min(p.n_valid, v0 + p.ts * 16);
    constexpr float kLog2e = 1.4426950408889634f;
#pragma unroll
    for (int q = 0; q < G::PASS; ++q) {
      const int r0 = (wave + q * kPanelWaves) * 8;
      if (r0 >= p.R) break;
      const float* row = logits + (r0 + (lane_e >> 3)) * kPanelLd + j;
      float x[NX];
#pragma unroll
      for (int i = 0; i < NX; ++i) x[i] = row[8 * i];
      float mx = run_m[q];
#pragma unroll
      for (int i = 0; i < NX; ++i) {
        x[i] = v0 + 8 * i + j < v_end ? x[i] : SPEC_NEG_INF;
        mx = fmaxf(mx, x[i]);
      }
      mx = row8_max(mx);
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < NX; ++i) s += __builtin_amdgcn_exp2f((x[i] - mx) * kLog2e);
      s = row8_sum(s);
      run_s[q] = run_s[q] * __builtin_amdgcn_exp2f((run_m[q] - mx) * kLog2e) + s;
      run_m[q] = mx;
      float lowest = SPEC_NEG_INF, highest = -SPEC_NEG_INF;
      asm volatile("" : "+v"(lowest), "+v"(highest));
      double lk[KT];
#pragma unroll
      for (int e = 0; e < KT; ++e) lk[e] = __hiloint2double(__float_as_int(SPEC_NEG_INF), kIdxNone);
#pragma unroll
      for (int i = 0; i < NX; ++i) {
        double key = list_key(__builtin_amdgcn_fmed3f(x[i], lowest, highest), ~(v0 + 8 * i + j));
#pragma unroll
        for (int e = 0; e < KT; ++e) {   // down the list, the smaller of each pair moves on
          const double old = lk[e];
          lk[e] = __builtin_fmax(old, key);
          if (e + 1 < KT) key = __builtin_fmin(old, key);
        }
      }
      uint64_t hk[KT + 1];   // with the one carried along
#pragma unroll
      for (int e = 0; e < KT; ++e) hk[e] = list_best_key(lk[e]);
      uint64_t c = run_key[q];
#pragma unroll
      for (int e = 0; e < KT; ++e) {
        const bool gt = c > hk[e];
        const uint64_t lower = gt ? hk[e] : c;
        hk[e] = gt ? c : hk[e];
        c = lower;
      }
      hk[KT] = c;
      uint64_t mine = kEmpty;
#pragma unroll
      for (int e = 0; e < KT; ++e) {
        if (e < p.k_top) {
          const uint64_t best = row8_best_key(hk[0]);
          const bool won = hk[0] == best;   // the owner of the winner pops it
#pragma unroll
          for (int u = 0; u < KT; ++u) {
            const uint64_t up = opaque_key(hk[u + 1]);
            hk[u] = won ? up : hk[u];
          }
          mine = j == e ? best : mine;
        }
      }
      run_key[q] = mine;
    }
  };
  auto write_partials = [&]() {
    if (t0 >= p.n_tiles[0]) return;   // a range of the projection only
    const int lane_e = lane_anew(), j = lane_e & 7;
#pragma unroll
    for (int q = 0; q < G::PASS; ++q) {
      const int r = (wave + q * kPanelWaves) * 8 + (lane_e >> 3);
      if (r >= p.R) break;
      const int64_t slot = (int64_t)r * p.nparts + range;
      if (j == 0) {
        p.part.m[slot] = run_m[q];
        p.part.s[slot] = run_s[q];
      }
      if (j < p.k_top) {
        float bv;
        int32_t bi;
        best_unkey(run_key[q], bv, bi);
        p.part.val[slot * p.k_top + j] = bv;
        p.part.idx[slot * p.k_top + j] = bi;
      }
    }
  };

  // ---- waves 9 .. 11: the states' slabs, one ahead of the others, and every barrier of the others
  if (wave >= kPanelFrags) {
    copy_slab(0, 0);
    int at = 0;
    for (int t = t0; t < t1; ++t) {
      for (int s = 0; s < slabs; ++s) {
        wait_copies();
        wave_barrier();
        at ^= G::SLAB;
        if (s + 1 < slabs || t + 1 < t1) copy_slab(s + 1 < slabs ? s + 1 : 0, at);
      }
      if (t < p.n_tiles[0]) {
        wave_barrier();
        close_rows(t);
      }
    }
    write_partials();
    return;
  }

  u32x4 a[D], bf[MF];
  int slab_at = 0;   // LDS buffer of the slab that is read next
  {
    const auto buf = tile_buf(t0);
#pragma unroll
    for (int d = 0; d < D; ++d) {
      a[d] = load_weight(buf, lane16 + d * 1024);
      __builtin_amdgcn_sched_barrier(0);   // (in this order: the K loop then waits for one at a time)
    }
  }

  for (int t = t0; t < t1; ++t) {
    const bool head = t < p.n_tiles[0];
    const int tile = t - (head ? 0 : p.n_tiles[0]);
    f32x4 acc[MF];
#pragma unroll
    for (int m = 0; m < MF; ++m) acc[m] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const auto here = tile_buf(t), next = tile_buf(t + 1);
    // one K-step: the fragments of the next are read as soon as this one's are used, its weights requested D steps ahead
    auto step = [&](int d, bool live, __amdgpu_buffer_rsrc_t src, int off) {
      auto read = [&](int m, int dd) { return *reinterpret_cast<lds_word*>(lds + slab_at + lane16 + (m * KS + dd % KS) * 1024); };
      if (d % KS == 0) {   // the slab has landed, and the other one has been read by all
        wave_barrier();
#pragma unroll
        for (int m = 0; m < MF; ++m) bf[m] = read(m, d);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (live) {
#pragma unroll
        for (int m = 0; m < MF; ++m) {
          acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[d]), __builtin_bit_cast(bf16x8, bf[m]),
                                                           acc[m], 0, 0, 0);
          if (d % KS != KS - 1) bf[m] = read(m, d + 1);
        }
      }
      a[d] = load_weight(src, lane16 + off + d * 1024);
      __builtin_amdgcn_sched_barrier(0);
      if (d % KS == KS - 1) slab_at ^= G::SLAB;
    };
    const int full = kt / D;
    for (int g = 0; g < full; ++g) {
      const bool last = g + 1 == groups;
      const auto src = last ? next : here;
      const int off = last ? 0 : (g + 1) * D * 1024;
#pragma unroll
      for (int d = 0; d < D; ++d) step(d, true, src, off);
    }
    if (full < groups) {   // K is not a multiple of 32 D
#pragma unroll
      for (int d = 0; d < D; ++d) step(d, full * D + d < kt, next, 0);
    }

    const int lane_e = lane_anew(), j = lane_e & 15, quad = lane_e >> 4;
    if (!head) {
      // ---- store: lane = state row lane % 16 of every state fragment, four consecutive columns
      const int f = tile * p.ts + wave;
      if (wave < p.ts && f < p.n_frags[1]) {
#pragma unroll
        for (int m = 0; m < MF; ++m) {
          const int r = m * 16 + j;
          if (r < p.R) *reinterpret_cast<f32x4*>(p.out + (int64_t)r * p.ldo + f * 16 + quad * 4) = acc[m];
        }
      }
      continue;
    }
    // ---- the tile's logits through LDS (read by all before the next tile's first barrier)
#pragma unroll
    for (int m = 0; m < MF; ++m)
      *reinterpret_cast<f32x4*>(logits + (m * 16 + j) * kPanelLd + wave * 16 + quad * 4) = acc[m];
    wave_barrier();
    close_rows(tile);
  }
  write_partials();
}

template <int MF, int KT>
static hipError_t launch_panel_t(const PanelArgs& a, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  constexpr size_t smem = PanelGeo<MF>::BYTES;
  static bool attr_set = false;  // per instantiation
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(head_panel_kernel<MF, KT>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipExtLaunchKernelGGL((head_panel_kernel<MF, KT>), dim3(a.n_ranges), dim3(kPanelWaves * 64), smem, st, ev_start, ev_stop, 0, a);
  return hipGetLastError();
}

// Which launches come here.  Drafts of two stages of top-1 or one of top-3 to 5, 20 to 128 rows, K = 256 to 8192, 2000 to 128256
// weight rows, the kernels there were before / this one:
//  * 17 to 32 rows that the streaming kernel does not take: 1.02 to 1.31 times as fast at any number of tiles per CU;
//  * more rows: where no CU has more than one tile, 0.99 to 1.27.  With more, the states come from L2 once per tile, and the
//    narrower tiles that even rounds want keep less in flight: 49152 rows x 4096 against 48, 75, 112 rows 158.7 / 172.5,
//    191.8 / 197.0, 200.9 / 220.4 us, 128256 x 3072 against 64, 128 156 / 160, 182 / 177;
//  * up to 64 rows against at most 64 weight rows per CU: the narrow dense kernel's two 32-row blocks per tile keep twice the
//    workgroups busy where K is long (8000 + K rows, 48 state rows, K = 1024, 2048, 4096, 8192: 46.5 / 40.1, 53.2 / 53.7,
//    68.3 / 81.3, 135 / 130; 2000 + K: 41.5 / 39.3, 47.2 / 49.3, 59.7 / 72.1, 88.5 / 123), so K <= 1024 there;
//  * more than 128 rows: one fragment of weights per wave reads all states from LDS for it (168 rows x 32000 x 4096: 66 / 76).
PanelPlan plan_panel(int R, int k_top, int n_head, int n_proj, int kt, int n_cu) {
  PanelPlan pl;
  memset(&pl, 0, sizeof(pl));
  const int cus = n_cu > 0 ? n_cu : 256;
  if (R <= 16 || R > 128 || n_head <= 0 || k_top < 1 || k_top > kMaxTopK || skinny32_fits(R, kt, n_head, n_cu)) return pl;
  if (R <= 64 && kt > 32 && (int64_t)n_head + n_proj <= (int64_t)64 * cus) return pl;
  const int64_t frags_head = (n_head + 15) / 16, frags_proj = (n_proj + 15) / 16;
  auto tiles = [&](int ts) { return (frags_head + ts - 1) / ts + (frags_proj + ts - 1) / ts; };
  const int64_t rounds = (tiles(kPanelFrags) + cus - 1) / cus;
  if (R > 32 && rounds > 1) return pl;
  // the fewest weight tiles per workgroup tile that need no more rounds: all CUs stream
  pl.ts = kPanelFrags;
  while (pl.ts > 1 && tiles(pl.ts - 1) <= cus * rounds) --pl.ts;
  const int mf = (R + 15) / 16;
  pl.block = mf == 7 ? 8 : mf;
  pl.kcap = k_top < 2 ? 2 : k_top == 5 ? 6 : k_top == 7 ? 8 : k_top;
  pl.n_head = (int)((frags_head + pl.ts - 1) / pl.ts);
  pl.n_tiles = (int)tiles(pl.ts);
  pl.n_ranges = pl.n_tiles < cus ? pl.n_tiles : cus;
  // ranges that start inside the head hold head tiles
  while (pl.nparts < pl.n_ranges && (int64_t)pl.nparts * pl.n_tiles / pl.n_ranges < pl.n_head) ++pl.nparts;
  return pl;
}

size_t panel_lds_bytes(const PanelPlan& pl) {
  switch (pl.block) {
    case 2: return PanelGeo<2>::BYTES;
    case 3: return PanelGeo<3>::BYTES;
    case 4: return PanelGeo<4>::BYTES;
    case 5: return PanelGeo<5>::BYTES;
    case 6: return PanelGeo<6>::BYTES;
    default: return PanelGeo<8>::BYTES;
  }
}

hipError_t launch_head_panel(const HeadJob& job, const PanelPlan& pl, hipStream_t st, hipEvent_t ev_start,
                             hipEvent_t ev_stop) {
  if (job.vt_head <= 0 || job.out_head || job.b_rowmajor || job.kt < 1 || job.k_top > pl.kcap || job.nparts != pl.nparts ||
      16 * pl.block < job.R)
    return hipErrorInvalidValue;
  PanelArgs a;
  memset(&a, 0, sizeof(a));
  a.w[0] = static_cast<const u32x4*>(job.w_head);
  a.w[1] = static_cast<const u32x4*>(job.w_proj);
  a.n_frags[0] = job.vt_head;
  a.n_frags[1] = job.vt_proj;
  a.n_tiles[0] = pl.n_head;
  a.n_tiles[1] = pl.n_tiles - pl.n_head;
  a.ts = pl.ts;
  a.n_valid = job.n_head;
  a.kt = job.kt;
  a.tile_slots = job.tile_slots;
  a.b = static_cast<const u32x4*>(job.b_src);
  a.mt_total = (job.R + 15) / 16;
  a.R = job.R;
  a.n_ranges = pl.n_ranges;
  a.out = job.out_proj;
  a.ldo = job.ld_proj;
  a.k_top = job.k_top;
  a.nparts = job.nparts;
  a.part = job.part;
  switch (pl.block * 10 + pl.kcap) {
#define PANEL(MF_)                                                          \
  case (MF_) * 10 + 2: return launch_panel_t<MF_, 2>(a, st, ev_start, ev_stop); \
  case (MF_) * 10 + 3: return launch_panel_t<MF_, 3>(a, st, ev_start, ev_stop); \
  case (MF_) * 10 + 4: return launch_panel_t<MF_, 4>(a, st, ev_start, ev_stop); \
  case (MF_) * 10 + 6: return launch_panel_t<MF_, 6>(a, st, ev_start, ev_stop); \
  case (MF_) * 10 + 8: return launch_panel_t<MF_, 8>(a, st, ev_start, ev_stop);
    PANEL(2) PANEL(3) PANEL(4) PANEL(5) PANEL(6) PANEL(8)
#undef PANEL
    default: return hipErrorInvalidValue;
  }
}

}  // namespace specdraft
