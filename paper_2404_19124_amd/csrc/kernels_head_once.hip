// Vocabulary head, alone or with the next stage's projection, against 129 to 320 state rows, where every CU has at most one tile
// of weight rows: the middle stages of a batched draft (320 rows of 64 sequences with a 5/3/2 tree), the last of a small batch.
//
// The two were two launches (head alone, one round of tiles; projection split along K, its four partial sums added by the stage
// kernel) or one whose tile list was a little longer than a round.  160 weight rows to a tile put both into one round of a
// launch whose blocks hold all state rows, so no weight is read twice.
// Bound: the requests a CU may have outstanding.  Its L1 keeps about 90 lines of 128 bytes on their way whatever the kernel has
// asked for (averages of the counters in these launches: 87 to 92, 640 to 950 cycles each), so a line from HBM costs a CU about
// 700 / 90 cycles and one from L2 300 / 90, and the two add up: copies of the states alone take 42 us of the launch below, of the
// weights alone 55, of both 95, with the matrix work 103, which alone would take 55.
//  * Workgroup = 8 waves; tile = 160 (NB = 5) weight rows x 64 * MB state rows, a wave 80 x 16 * MB of it (MB = 5: 100 accumulators
//    of v_mfma_f32_16x16x32_bf16, two sets of fragments beside them).  Tiles of 128 weight rows (NB = 4) where they too are one
//    round: a launch lasts as long as a tile, and 32000 rows are 200 tiles of 160 for 256 CUs.
//  * Both operands are copied straight into LDS (buffer loads to LDS), the weights eight K-steps ahead, the states four, by
//    different waves: a wave's copies land in order, and a wait for its states would be one for its youngest weights.
//    One barrier per K-step; LDS reads and copies are issued one by one between the matrix instructions.
// 320 rows x (32000 + 4096) x 4096: 89.5 + 24.4 us in two launches, 103 in one; 4096 + 32000 rows, drafts of two
// stages against 130, 192, 256 rows 1.15, 1.19, 1.09 times as fast.
#include <hip/hip_ext.h>

#include <cstring>
#include <type_traits>

#include "lane_lists.h"
#include "once_steps.h"

namespace specdraft {

constexpr int kOnceWaves = 8;      // two along the weight rows, four along the state rows
constexpr int kOnceWM = 4;
constexpr int kOnceCopyW = 2;      // waves that copy weights; the others copy states
constexpr int kOnceLds = 160 * 1024;

struct OnceArgs {
  const u32x4* w[2];   // packed weights: head, projection
  int n_frags[2];      // their 16-row tiles
  int n_head;          // workgroup tiles of the head; the projection's follow
  int n_valid, kt, tile_slots;
  const u32x4* b;      // packed states
  int mt_total, R;
  float* out;          // projection
  int64_t ldo;
  int k_top, nparts;
  Partials part;
};

// NB = 16-row weight fragments of a wave, MB = its state fragments.
template <int NB, int MB>
struct OnceGeo {
  static constexpr int WF = 2 * NB, SF = kOnceWM * MB;       // fragments of a K-step
  static constexpr int W_STEP = WF * 1024, S_STEP = SF * 1024;
  static constexpr int WC = WF / kOnceCopyW;                 // copies of a wave per step
  static constexpr int SC = (SF + kOnceWaves - kOnceCopyW - 1) / (kOnceWaves - kOnceCopyW);
  static constexpr int S_AT = kOnceDW * W_STEP;
  static constexpr int BYTES = S_AT + kOnceDS * S_STEP;
  static_assert(BYTES <= kOnceLds, "a CU has no more");
};

// WEIGHTS: what this wave copies.  The slots of that ring are distinct objects to the compiler (restrict): a read of one then waits
// only for this wave's copies into that one, which the counted wait in front of the barrier has already seen land, and not for
// every copy in flight.  The other ring, which this wave only reads, goes by the plain pointer: what it holds changes behind
// every barrier.  Nothing else is kept in that memory before this returns.
template <int NB, int MB, int KT, bool WEIGHTS>
__device__ __forceinline__ void once_contract(const OnceArgs& p, lds_byte* lds, lds_byte* __restrict c0, lds_byte* __restrict c1,
                                              lds_byte* __restrict c2, lds_byte* __restrict c3, lds_byte* __restrict c4,
                                              lds_byte* __restrict c5, lds_byte* __restrict c6, lds_byte* __restrict c7,
                                              f32x4 (&acc)[MB][NB]) {
  using G = OnceGeo<NB, MB>;
  static_assert(kOnceDW == 8 && kOnceDS == 4, "the slots");
  lds_byte* const mine[8] = {c0, c1, c2, c3, c4, c5, c6, c7};   // (four of them for the states)
  constexpr int C = WEIGHTS ? G::WC : G::SC, DEPTH = WEIGHTS ? kOnceDW : kOnceDS;
  const int lane = threadIdx.x & 63, lane16 = lane * 16;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wn = wave / kOnceWM, wm = wave % kOnceWM;
  const int kt = p.kt, range = blockIdx.x;
  const bool head = range < p.n_head;
  const int mat = head ? 0 : 1, f0 = (range - (head ? 0 : p.n_head)) * G::WF;   // first fragment of the tile

  // ---- copies: 1 KiB = one fragment of the packed layout.  A fragment past the matrix or the block repeats the last one.
  const int tile_bytes = p.tile_slots * 16, w_last = min(G::WF, p.n_frags[mat] - f0) - 1, s_last = min(G::SF, p.mt_total) - 1;
  const unsigned char* const src = WEIGHTS ? reinterpret_cast<const unsigned char*>(p.w[mat]) + (int64_t)f0 * tile_bytes
                                           : reinterpret_cast<const unsigned char*>(p.b);
  const int span = WEIGHTS ? w_last * tile_bytes + kt * 1024 : (s_last + 1) * kt * 1024;
  int from[C], to[C];
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const int f = WEIGHTS ? wave * G::WC + i : min((wave - kOnceCopyW) + i * (kOnceWaves - kOnceCopyW), G::SF - 1);
    from[i] = WEIGHTS ? min(f, w_last) * tile_bytes : min(f, s_last) * kt * 1024;
    to[i] = f * 1024;
  }
  const auto buf = weight_buffer(src, span);   // (the scalar offset is not part of its check: no copy reaches past it)
  auto copy = [&](int i, int u, int step) {   // K-step `step` into slot u
    lds_byte* const dst = mine[u % DEPTH] + to[i];
    __builtin_amdgcn_raw_ptr_buffer_load_lds(buf, (__attribute__((address_space(3))) void*)dst, 16, lane16, from[i] + step * 1024, 0,
                                             WEIGHTS ? 2 : 0);
  };
#pragma unroll
  for (int u = 0; u < DEPTH; ++u)
#pragma unroll
    for (int i = 0; i < C; ++i) copy(i, u, u);

  // ---- fragments of two K-steps in registers
  u32x4 aw[2][NB], bf[2][MB];
  const int a_at = wn * NB * 1024 + lane16, b_at = wm * MB * 1024 + lane16;
  auto read_a = [&](int u, int n) {
    lds_byte* const slot = WEIGHTS ? mine[u % kOnceDW] : lds + (u % kOnceDW) * G::W_STEP;
    aw[u & 1][n] = *reinterpret_cast<lds_word*>(slot + a_at + n * 1024);
  };
  auto read_b = [&](int u, int m) {
    lds_byte* const slot = WEIGHTS ? lds + G::S_AT + (u % kOnceDS) * G::S_STEP : mine[u % kOnceDS];
    bf[u & 1][m] = *reinterpret_cast<lds_word*>(slot + b_at + m * 1024);
  };
  copies_landed_barrier<(DEPTH - 1) * C, false>();
#pragma unroll
  for (int n = 0; n < NB; ++n) read_a(0, n);
#pragma unroll
  for (int m = 0; m < MB; ++m) read_b(0, m);

  // (weight rows past the vocabulary start, and stay, at -inf: no mask in the epilogue)
  const int v0 = (f0 + wn * NB) * 16 + (lane >> 4) * 4;   // this lane's weight rows: v0 + 16 n + i
  const int v_end = head ? p.n_valid : 0x7fffffff;
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    f32x4 z;
#pragma unroll
    for (int i = 0; i < 4; ++i) z[i] = v0 + n * 16 + i < v_end ? 0.f : SPEC_NEG_INF;
#pragma unroll
    for (int m = 0; m < MB; ++m) acc[m][n] = z;
  }

  // FULL: all steps of the group count.  Else those before kt, K not being a multiple of 32 * 8.
  auto group = [&](auto full, int base) {
    constexpr bool FULL = decltype(full)::value;
#pragma unroll
    for (int u = 0; u < kOnceDW; ++u) {
      if (!FULL && base + u >= kt) break;
      // every wave has read step u's slots, and step u + 1 has landed for all of them
      copies_landed_barrier<(DEPTH - 2) * C, true>();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < MB; ++m) read_b(u + 1, m);
#pragma unroll
      for (int n = 0; n < NB; ++n) read_a(u + 1, n);
#pragma unroll
      for (int i = 0; i < C; ++i) copy(i, u, once_next_step(base + u, DEPTH, kt));
#pragma unroll
      for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int m = 0; m < MB; ++m)
          acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, aw[u & 1][n]),
                                                              __builtin_bit_cast(bf16x8, bf[u & 1][m]), acc[m][n], 0, 0, 0);
      // a wave issues in order: the reads, then the copies, one by one between the matrix instructions
      constexpr int NM = MB * NB, NR = MB + NB, NT = NR + C;
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
#pragma unroll
        for (int j = i * NT / NM; j < (i + 1) * NT / NM; ++j) {
          if (j < NR) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          else __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  int base = 0;
  for (; base + kOnceDW <= kt; base += kOnceDW) group(std::true_type{}, base);
  if (base < kt) group(std::false_type{}, base);
}

// What becomes of a tile's products: a projection's are stored, a head's closed.
template <int NB, int MB, int KT>
__device__ __forceinline__ void once_close(const OnceArgs& p, const f32x4 (&acc)[MB][NB], unsigned char* smem) {
  using G = OnceGeo<NB, MB>;
  const int lane = threadIdx.x & 63, col = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wn = wave / kOnceWM, wm = wave % kOnceWM;
  const int range = blockIdx.x;
  const bool head = range < p.n_head;
  const int f0 = (range - (head ? 0 : p.n_head)) * G::WF, v0 = (f0 + wn * NB) * 16 + (lane >> 4) * 4;
  if (!head) {
    // ---- store: lane = state row lane % 16 of every state fragment, four consecutive columns of each weight fragment
    copies_landed_barrier<0, true>();   // (LDS goes back with nothing on its way into it)
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      if (f0 + wn * NB + n < p.n_frags[1]) {
#pragma unroll
        for (int m = 0; m < MB; ++m) {
          const int r = (wm * MB + m) * 16 + col;
          if (r < p.R) *reinterpret_cast<f32x4*>(p.out + (int64_t)r * p.ldo + v0 + n * 16) = acc[m][n];
        }
      }
    }
    return;
  }

  // ---- epilogue: a row's 4 NB logits of this lane into its list, and their exponentials into its sum.  The MB rows are
  // independent chains: one logit each in turn.
  float sum[MB];
  double lk[MB][KT];
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int q = 0; q < KT; ++q) lk[m][q] = __hiloint2double(__float_as_int(SPEC_NEG_INF), kIdxNone);
  constexpr float kLog2e = 1.4426950408889634f;
  // NaN counts as -inf in the lists: the median with the two infinities is the smaller of them then.  (In registers the
  // optimiser cannot look through: it would take the median of x and known infinities for x.)
  float lowest = SPEC_NEG_INF, highest = -SPEC_NEG_INF;
  asm volatile("" : "+v"(lowest), "+v"(highest));
#pragma unroll
  for (int n = 0; n < NB; ++n)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int32_t not_index = ~(v0 + n * 16 + i);
      asm volatile("" : "+v"(not_index));   // (one value for the MB rows)
      double key[MB];
#pragma unroll
      for (int m = 0; m < MB; ++m) key[m] = list_key(__builtin_amdgcn_fmed3f(acc[m][n][i], lowest, highest), not_index);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < KT; ++q) {   // down the lists, the smaller of each pair moves on
#pragma unroll
        for (int m = 0; m < MB; ++m) {
          const double old = lk[m][q];
          lk[m][q] = __builtin_fmax(old, key[m]);
          if (q + 1 < KT) key[m] = __builtin_fmin(old, key[m]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  float ml[MB];
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    sum[m] = 0.f;
    ml[m] = -list_reference(lk[m][0]) * kLog2e;
  }
#pragma unroll
  for (int n = 0; n < NB; ++n)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int m = 0; m < MB; ++m) sum[m] += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[m][n][i], kLog2e, ml[m]));

  copies_landed_barrier<0, true>();   // nothing is on its way into LDS any more, for all waves
  merge_lane_lists<MB, KT>(smem, lk, sum, wave, lane, 0, p.R, p.part, p.k_top, p.nparts, range);
}

template <int NB, int MB, int KT>
__global__ __launch_bounds__(kOnceWaves * 64) void head_once_kernel(OnceArgs p) {
  extern __shared__ __align__(16) unsigned char smem[];
  using G = OnceGeo<NB, MB>;
  lds_byte* const l = (lds_byte*)smem;
  lds_byte* const s = l + G::S_AT;
  f32x4 acc[MB][NB];
  if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) < kOnceCopyW) {
    once_contract<NB, MB, KT, true>(p, l, l, l + G::W_STEP, l + 2 * G::W_STEP, l + 3 * G::W_STEP, l + 4 * G::W_STEP,
                                    l + 5 * G::W_STEP, l + 6 * G::W_STEP, l + 7 * G::W_STEP, acc);
    once_close<NB, MB, KT>(p, acc, smem);
  } else {
    once_contract<NB, MB, KT, false>(p, l, s, s + G::S_STEP, s + 2 * G::S_STEP, s + 3 * G::S_STEP, nullptr, nullptr, nullptr,
                                     nullptr, acc);
    once_close<NB, MB, KT>(p, acc, smem);
  }
}

static constexpr size_t once_lds(int nb, int mb, int kt) {
  const size_t rings = (size_t)kOnceDW * 2 * nb * 1024 + (size_t)kOnceDS * kOnceWM * mb * 1024;
  return list_merge_bytes(mb, kt) > rings ? list_merge_bytes(mb, kt) : rings;
}

template <int NB, int MB, int KT>
static hipError_t launch_once_t(const OnceArgs& a, int grid, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  constexpr size_t smem = once_lds(NB, MB, KT);
  static_assert(smem <= kOnceLds && smem >= (size_t)OnceGeo<NB, MB>::BYTES, "a CU has no more");
  static bool attr_set = false;  // per instantiation
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(head_once_kernel<NB, MB, KT>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipExtLaunchKernelGGL((head_once_kernel<NB, MB, KT>), dim3(grid), dim3(kOnceWaves * 64), smem, st, ev_start, ev_stop, 0, a);
  return hipGetLastError();
}

// Which launches come here: lists of at most 4, K of one group of eight steps and more, all tiles in one round.  Tiles of 128 weight
// rows where that is one round, else of 160.  Drafts of one stage of top-2 (a head alone) and of two of top-1, weights of 800 MB in
// turn so that none stay in the memory-side cache, the kernels there were before / this one, times as fast against 130, 192, 256,
// 320 rows:
//  * 160-row tiles, head alone: 38000 x 1024 1.18, 1.14, 1.21, 1.17;  x 2048 1.15, 1.17, 1.17, 1.13;  x 3072 1.19, 1.21, 1.28, 1.21;
//    40000 x 4096 1.19, 1.24, 1.22, 1.18;  x 8192 1.11, 1.21, 1.15, 1.17.  With the projection, its launches by difference: 32000 +
//    1024 31 / 25, 39 / 28, 42 / 30, 44 / 36 us;  + 2048 45 / 40, 61 / 47, 64 / 54, 66 / 59;  + 3072 63 / 54, 82 / 59, 85 / 67, 92 / 74.
//  * 128-row tiles, head alone: 32000 x 1024 1.04, 1.03, 1.02, 0.99;  x 2048 1.14, 1.09, 1.02, 0.98;  x 4096 1.18, 1.12, 1.02, 0.96;
//    x 6144 1.15, 1.07, 1.00, 0.97;  28000 x 4096 1.13, 1.08, 1.00, 0.96;  24000 1.05, 1.03, 0.97, 0.95;  20000 1.02, 1.01, 0.93,
//    0.88: up to 192 rows from 96 weight rows per CU on, up to 256 from 120.
//  * 128-row tiles with the projection, by difference: 28000 + 4096 76 / 63, 74 / 67, 84 / 78, 93 / 91 us;  20000 + 4096 63 / 59, 68 /
//    65, 77 / 74, 87 / 87;  18000 + 6144 89 / 80, 93 / 82, 106 / 96, 123 / 119;  28000 + 2048 39 / 35, 45 / 44, 48 / 49, 51 / 55;  18000 +
//    8192 112 / 107, 132 / 129, 142 / 146, 159 / 163: up to 192 rows, from 84 weight rows per CU on.
//  * The same against 193 and 256 rows, two stages, us: K = 1536 92.2 / 92.5, 96.6 / 97.5;  1792 106.0 / 105.6, 112.1 / 112.3;  2048
//    114.2 / 112.9, 119.5 / 120.0;  2112 116.4 / 114.7, 123.8 / 121.8;  2560 132.1 / 129.2, 140.1 / 138.1;  3072 133.6 / 127.1, 140.3 /
//    135.2;  4096 167.0 / 163.0, 176.5 / 176.9;  6080 231.0 / 224.4, 245.3 / 240.7;  6144 232.2 / 234.1, 247.6 / 252.4;  6208 235.4 /
//    230.4, 250.7 / 246.7;  7168 268.2 / 263.7, 286.5 / 281.5;  8128 313.6 / 309.1, 334.7 / 330.7;  8192 304.6 / 306.5, 324.7 / 329.6;  8704
//    321.3 / 313.8, 343.1 / 338.0;  10240 367.0 / 370.0, 392.5 / 402.5;  12288 467 / 472, 509 / 519.  It gains above K = 2048, and
//    loses where weight tiles lie a whole number of 64 KiB apart (6144, 8192, ..; those of 2048 and 4096 lie 4 KiB further): the
//    eight fragments of a K-step then ask the same channels at once.  So up to 256 rows for the K above 2048 without that.
//  * K that ends within a group, times as fast, head alone and two stages: 33000 x 3136 1.22, 1.45, 1.27, 1.24 and 1.28, 1.53, 1.32, 1.28;
//    38000 x 2496 1.24, 1.43, 1.21, 1.19 and 1.25, 1.48, 1.25, 1.21;  28000 x 1600 1.15, 1.11, - and 1.15, 1.11, -;  30000 x 4160
//    1.19, 1.14, - and 1.19, 1.23, 1.11, 1.12.
OncePlan plan_once(int R, int k_top, int n_head, int n_proj, int kt, int n_cu) {
  OncePlan pl;
  memset(&pl, 0, sizeof(pl));
  const int64_t cus = n_cu > 0 ? n_cu : 256;
  constexpr int kSlots64K = 65536 / 16;
  if (R <= 128 || R > 320 || n_head <= 0 || k_top < 1 || k_top > 4 || kt < kOnceDW) return pl;
  auto head_tiles = [&](int nb) { return ((int64_t)n_head + 32 * nb - 1) / (32 * nb); };
  auto all_tiles = [&](int nb) { return head_tiles(nb) + (n_proj > 0 ? ((int64_t)n_proj + 32 * nb - 1) / (32 * nb) : 0); };
  const int nb = all_tiles(4) <= cus ? 4 : 5;
  if (all_tiles(nb) > cus) return pl;
  if (nb == 4) {
    const int64_t weight_rows = (int64_t)n_head + (n_proj > 0 ? n_proj : 0);
    if (n_proj > 0 ? R > (kt > 64 && packed_tile_slots(kt) % kSlots64K ? 256 : 192) || weight_rows <= 84 * cus
                   : R > 256 || weight_rows <= (R > 192 ? 120 : 96) * cus)
      return pl;
  }
  pl.nb = nb;
  pl.block = (R + 63) / 64;
  pl.kcap = k_top < 2 ? 2 : k_top;
  pl.n_head = (int)head_tiles(nb);
  pl.n_tiles = (int)all_tiles(nb);
  return pl;
}

size_t once_lds_bytes(const OncePlan& pl) { return once_lds(pl.nb, pl.block, pl.kcap); }

hipError_t launch_head_once(const HeadJob& job, const OncePlan& pl, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (job.vt_head <= 0 || job.out_head || job.b_rowmajor || job.kt < kOnceDW || job.k_top > pl.kcap ||
      job.nparts != pl.n_head || job.R > 64 * pl.block)
    return hipErrorInvalidValue;
  OnceArgs a;
  memset(&a, 0, sizeof(a));
  a.w[0] = static_cast<const u32x4*>(job.w_head);
  a.w[1] = static_cast<const u32x4*>(job.w_proj);
  a.n_frags[0] = job.vt_head;
  a.n_frags[1] = job.vt_proj;
  a.n_head = pl.n_head;
  a.n_valid = job.n_head;
  a.kt = job.kt;
  a.tile_slots = job.tile_slots;
  a.b = static_cast<const u32x4*>(job.b_src);
  a.mt_total = (job.R + 15) / 16;
  a.R = job.R;
  a.out = job.out_proj;
  a.ldo = job.ld_proj;
  a.k_top = job.k_top;
  a.nparts = job.nparts;
  a.part = job.part;
  switch (pl.nb * 100 + pl.block * 10 + pl.kcap) {
#define ONCE(NB_, MB_)                                                                             \
  case (NB_) * 100 + (MB_) * 10 + 2: return launch_once_t<NB_, MB_, 2>(a, pl.n_tiles, st, ev_start, ev_stop); \
  case (NB_) * 100 + (MB_) * 10 + 3: return launch_once_t<NB_, MB_, 3>(a, pl.n_tiles, st, ev_start, ev_stop); \
  case (NB_) * 100 + (MB_) * 10 + 4: return launch_once_t<NB_, MB_, 4>(a, pl.n_tiles, st, ev_start, ev_stop);
    ONCE(4, 3) ONCE(4, 4) ONCE(5, 3) ONCE(5, 4) ONCE(5, 5)
#undef ONCE
    default: return hipErrorInvalidValue;
  }
}

}  // namespace specdraft
