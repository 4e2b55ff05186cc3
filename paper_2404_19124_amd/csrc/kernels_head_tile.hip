// Vocabulary head alone against many state rows: the compute-bound launches of a batched draft (960 rows of the last stage for
// 64 sequences with a 5/3/2 tree; 192, 768 and 2304 per stage for 32 sequences with a 6/4/3/2 tree).
//
// Bound: the power the matrix cores may draw, then what a CU pulls through its L2.  So the tile is as tall as the
// accumulators allow, and the cheaper matrix instruction is taken:
//  * workgroup = 8 waves, two per SIMD; tile = 256 weight rows x 64 * MB state rows, split 2 x 4: a wave owns 128 weight rows x
//    16 * MB state rows, i.e. 8 * MB accumulators of v_mfma_f32_16x16x32_bf16 (MB = 4: 128 of its 256 registers).  Bare K
//    loop, 2304 rows x 128256 x 3072, one card: 1328 us with the 32x32x16 instruction, which moves the accumulators twice as
//    often per product (the clock falls to 1.6 GHz), 1220 with 16x16x32 (1.8 GHz, matrix cores 76 % busy).  The dense kernel's
//    1 x 4 split of a 160-row block reads an operand byte from LDS up to twice as often, and its epilogue (vector ALU)
//    runs alone on its SIMD;
//  * no instance uses scratch memory.  Blocks of 256 rows did (18 registers of a wave, 22 with lists of three): written in front
//    of every K loop, read behind it, and a reload waits for every copy in flight.  So there the weight fragments are read in
//    place, the lane index is asked for anew and the third entries of the lists wait in LDS.  960 rows x 32000, us, with scratch
//    and now: K = 128 26.0 and 22.7, 512 42.1 and 39.2, 4096 190.0 and 189.3; 768 x 128256 x 3072 445.5 and 440.0; 2304 rows
//    1270 and 1274; 4096 x 128256 x 8192, 6 ms, 1 to 3 % more;
//  * both operands are copied from memory straight into LDS (buffer loads to LDS), kSteps K-steps ahead and across the tiles
//    of a range, one barrier per K-step.  The fragments of the next step are read into registers while the matrix
//    cores work on this one's, and the copies and reads are issued one by one between the matrix instructions.  The cursor of
//    the copies moves by groups of steps: recomputed at every step it cost 6 % (1385 -> 1297 us);
//  * a workgroup is persistent over a contiguous range of weight tiles; every lane keeps a running sum of
//    exponentials and a top-k list per state row of its own, merged at the end of the range, as in the wide kernel.
// Launches, against the dense kernel: see plan_tile.
#include <hip/hip_ext.h>

#include <cstring>

#include "lane_lists.h"

namespace specdraft {

constexpr int kSteps = 4;        // LDS buffers = K-steps (of 32) in flight
constexpr int kWM = 4;           // waves along the state rows; two along the weight rows
constexpr int kWaves = 2 * kWM;
constexpr int kNB = 8;           // 16-row weight fragments per wave
constexpr int kWF = 2 * kNB;     // weight fragments of a tile

struct TileArgs {
  const u32x4* w;    // packed head weights
  const u32x4* b;    // packed states
  int kt, tile_slots, nt_total, n_valid, mt_total, R;
  int m_tiles, n_tiles, n_ranges, chunk;
  int k_top, nparts;
  Partials part;
};

// The accumulators stay where they are across the K loop: left to itself the register allocator lets them change places
// there for the sake of the epilogue (230 moves in a loop of 160 matrix instructions).
template <int MB>
__device__ __forceinline__ void pin_accumulators(f32x4 (&acc)[MB][kNB]) {
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < kNB; ++n) asm volatile("" : "+v"(acc[m][n]));
}

template <int MB>
struct TileGeo {
  static constexpr int SF = kWM * MB;                 // state fragments (16 rows) of a block
  static constexpr int STEP = (kWF + SF) * 1024;     // LDS bytes of one K-step
  static constexpr int WP = kWF / kWaves;                // weight / state fragments a wave copies per step
  static constexpr int SP = (SF + kWaves - 1) / kWaves;
  static constexpr int COPIES = WP + SP;
  static constexpr int KEEP = MB == 4 ? 8 : 0;
};

constexpr bool tile_parks(int mb, int kt) { return mb == 4 && kt == 3; }

// The four buffers are distinct objects to the compiler (restrict): a read of one then waits only for the copies into that
// one, which the counted wait in front of the barrier has already seen land, and not for every copy in flight.  Nothing else is
// kept in that memory before this returns.
template <int MB, int KT>
__device__ __forceinline__ void tile_range(const TileArgs& p, int t0, int t1, int mtile, int wave,
                                           lds_byte* __restrict b0, lds_byte* __restrict b1, lds_byte* __restrict b2,
                                           lds_byte* __restrict b3, lds_byte* park, float (&sum)[MB], double (&lk)[MB][KT]) {
  using G = TileGeo<MB>;
  static_assert(kSteps == 4, "four buffers");
  lds_byte* const bufs[kSteps] = {b0, b1, b2, b3};
  // The lane is asked for anew where it is needed: held across the K loop it is what does not fit the registers.
  auto lane_id = []() {
    uint32_t none = 0;
    asm volatile("" : "+s"(none));   // (or the first answer is kept)
    return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, none));
  };
  const int wn = wave / kWM, wm = wave % kWM;
  const int kt = p.kt;

  // ---- copies: 1 KiB = one fragment of the packed layout per instruction; wave w takes fragments w, w + 8, ...
  // A fragment past the matrix or the block repeats the last one (its results are masked).
  const int lane16 = lane_id() * 16;
  const unsigned char* const wb = reinterpret_cast<const unsigned char*>(p.w);
  const int mt0 = mtile * G::SF, mt_last = min(G::SF, p.mt_total - mt0) - 1;
  const unsigned char* const sb = reinterpret_cast<const unsigned char*>(p.b) + (int64_t)mt0 * kt * 1024;
  int s_off[G::SP], w_off[G::WP];
#pragma unroll
  for (int i = 0; i < G::SP; ++i) s_off[i] = min(min(i * kWaves + wave, G::SF - 1), mt_last) * kt * 1024;
  // The cursor moves by whole groups of kSteps steps: scalar work at every step would leave the matrix cores waiting.
  int c_step = 0, c_tile = t0;   // first step of the group that is copied, and its tile
  const int tile_bytes = p.tile_slots * 16;
  auto group_bufs = [&](auto& w, auto& s) {
    const int last = min(kWF, p.nt_total - c_tile * kWF) - 1;
#pragma unroll
    for (int i = 0; i < G::WP; ++i) w_off[i] = min(i * kWaves + wave, last) * tile_bytes;
    w = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<unsigned char*>(wb + (int64_t)c_tile * kWF * tile_bytes + c_step * 1024), 0,
        (last + 1) * tile_bytes - c_step * 1024, 0x00020000);
    s = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(sb + c_step * 1024), 0,
                                          (mt_last + 1) * kt * 1024 - c_step * 1024, 0x00020000);
  };
  __amdgpu_buffer_rsrc_t w_buf, s_buf;
  group_bufs(w_buf, s_buf);
  auto copy = [&](int i, int u) {
    if (i < G::WP) {
      lds_byte* const to = bufs[u] + (i * kWaves + wave) * 1024;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(w_buf, (__attribute__((address_space(3))) void*)to, 16, lane16,
                                               w_off[i] + u * 1024, 0, 0);
    } else {
      const int q = i - G::WP;
      lds_byte* const to = bufs[u] + (kWF + min(q * kWaves + wave, G::SF - 1)) * 1024;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(s_buf, (__attribute__((address_space(3))) void*)to, 16, lane16,
                                               s_off[q] + u * 1024, 0, 0);
    }
  };
  // (past the range's last tile its last steps again: nobody reads them, and they are in the L2)
  auto next_group = [&]() {
    const bool wrap = c_step + kSteps == kt, more = c_tile + 1 < t1;
    c_step = wrap ? (more ? 0 : c_step) : c_step + kSteps;
    c_tile += wrap && more ? 1 : 0;
    group_bufs(w_buf, s_buf);
  };
#pragma unroll
  for (int u = 0; u < kSteps; ++u)
#pragma unroll
    for (int i = 0; i < G::COPIES; ++i) copy(i, u);
  next_group();

  // ---- fragments of one K-step in registers: two sets of the states and of the last weight fragments; each of the first
  // G::KEEP weight fragments makes room for the next step's as soon as its matrix instructions are issued
  u32x4 aw[2][kNB], bf[2][MB];
  const int a_at = wn * kNB * 1024 + lane16, b_at = (kWF + wm * MB) * 1024 + lane16;
  auto read_a = [&](int u, int n) {   // fragment n of step u
    aw[n < G::KEEP ? 0 : u & 1][n] = *reinterpret_cast<lds_word*>(bufs[u % kSteps] + a_at + n * 1024);
  };
  auto read_b = [&](int u, int m) {
    bf[u & 1][m] = *reinterpret_cast<lds_word*>(bufs[u % kSteps] + b_at + m * 1024);
  };
  copies_landed_barrier<(kSteps - 1) * G::COPIES, false>();
#pragma unroll
  for (int n = 0; n < kNB; ++n) read_a(0, n);
#pragma unroll
  for (int m = 0; m < MB; ++m) read_b(0, m);

  // running state of this lane, per state row 16 * (wm * MB + m) + col of the block: its best logits so far, and the sum of
  // exponentials relative to the first of them
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    sum[m] = 0.f;
#pragma unroll
    for (int q = 0; q < KT; ++q) lk[m][q] = __hiloint2double(__float_as_int(SPEC_NEG_INF), kIdxNone);
  }

  // The third entries of the lists wait in LDS while the K loop runs (blocks of 256 rows: 8 registers of 256).
  constexpr bool PARK = tile_parks(MB, KT);
  volatile __attribute__((address_space(3))) double* const parked =
      (volatile __attribute__((address_space(3))) double*)(park + (wave * 64 + lane_id()) * (MB * 8));
  auto put = [&]() {
#pragma unroll
    for (int m = 0; m < MB; ++m) parked[m] = lk[m][KT - 1];
  };
  if (PARK) put();

  for (int t = t0; t < t1; ++t) {
    f32x4 acc[MB][kNB];
    // (weight rows past the vocabulary start, and stay, at -inf: no mask in the epilogue)
    const int v0 = t * 256 + wn * 128 + (lane_id() >> 4) * 4;   // this lane's weight rows: v0 + 16 n + i
#pragma unroll
    for (int n = 0; n < kNB; ++n) {
      f32x4 z;
#pragma unroll
      for (int i = 0; i < 4; ++i) z[i] = v0 + n * 16 + i < p.n_valid ? 0.f : SPEC_NEG_INF;
#pragma unroll
      for (int m = 0; m < MB; ++m) acc[m][n] = z;
    }
    pin_accumulators<MB>(acc);

    for (int base = 0; base < kt; base += kSteps) {
#pragma unroll
      for (int u = 0; u < kSteps; ++u) {
        // every wave has read step u's buffer, and step u + 1 has landed for all of them
        copies_landed_barrier<(kSteps - 2) * G::COPIES, true>();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < MB; ++m) read_b(u + 1, m);
#pragma unroll
        for (int n = G::KEEP; n < kNB; ++n) read_a(u + 1, n);
#pragma unroll
        for (int i = 0; i < G::COPIES; ++i) copy(i, u);
#pragma unroll
        for (int n = 0; n < kNB; ++n) {
#pragma unroll
          for (int m = 0; m < MB; ++m)
            acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, aw[n < G::KEEP ? 0 : u & 1][n]), __builtin_bit_cast(bf16x8, bf[u & 1][m]), acc[m][n], 0, 0, 0);
          if (n < G::KEEP) read_a(u + 1, n);
        }
        // a wave issues in order: the reads, then the copies, one by one between the matrix instructions
        constexpr int NM = MB * kNB, NR = MB + kNB, NT = NR + G::COPIES;
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
      next_group();
    }

    pin_accumulators<MB>(acc);
    if (PARK) {
#pragma unroll
      for (int m = 0; m < MB; ++m) lk[m][KT - 1] = parked[m];
    }

    // ---- epilogue: a row's 32 logits of this lane into its list, whose first entry is then the running maximum, and their
    // exponentials into its sum.  The MB rows are independent chains: one logit each in turn.  No branch: the
    // accumulators would be copied in front of it.
    constexpr float kLog2e = 1.4426950408889634f;
    // NaN counts as -inf in the lists: the median with the two infinities is the smaller of them then.  (In registers the
    // optimiser cannot look through: it would take the median of x and known infinities for x.)
    float lowest = SPEC_NEG_INF, highest = -SPEC_NEG_INF;
    asm volatile("" : "+v"(lowest), "+v"(highest));
    float ml[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) ml[m] = list_reference(lk[m][0]);
#pragma unroll
    for (int n = 0; n < kNB; ++n)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        int32_t not_index = ~(v0 + n * 16 + i);
        asm volatile("" : "+v"(not_index));   // (one value for the MB rows)
        float x[MB];
        double key[MB];
#pragma unroll
        for (int m = 0; m < MB; ++m) x[m] = __builtin_amdgcn_fmed3f(acc[m][n][i], lowest, highest);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < MB; ++m) key[m] = list_key(x[m], not_index);
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
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      const float mx = list_reference(lk[m][0]);
      sum[m] *= __builtin_amdgcn_exp2f((ml[m] - mx) * kLog2e);
      ml[m] = -mx * kLog2e;
    }
#pragma unroll
    for (int n = 0; n < kNB; ++n)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int m = 0; m < MB; ++m) sum[m] += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[m][n][i], kLog2e, ml[m]));
    if (PARK && t + 1 < t1) put();
  }

  copies_landed_barrier<0, true>();   // nothing is on its way into LDS any more, for all waves
}

template <int MB, int KT>
__global__ __launch_bounds__(kWaves * 64) void head_tile_kernel(TileArgs p) {
  extern __shared__ __align__(16) unsigned char smem[];
  using G = TileGeo<MB>;
  // XCD-aware workgroup id: ids go round-robin over 8 XCDs; the row blocks of one range run on one of them
  const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
  if (seq >= p.chunk) return;
  const int wg = xcd * p.chunk + seq;
  if (wg >= p.m_tiles * p.n_ranges) return;
  const int range = wg / p.m_tiles, mtile = wg - range * p.m_tiles;
  const int t0 = (int)((int64_t)range * p.n_tiles / p.n_ranges);
  const int t1 = (int)((int64_t)(range + 1) * p.n_tiles / p.n_ranges);
  lds_byte* l = (lds_byte*)smem;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float sum[MB];
  double lk[MB][KT];
  tile_range<MB, KT>(p, t0, t1, mtile, wave, l, l + G::STEP, l + 2 * G::STEP, l + 3 * G::STEP, l + 4 * G::STEP, sum, lk);
  // (the lane is asked for anew here too: see tile_range)
  uint32_t none = 0;
  asm volatile("" : "+s"(none));
  const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, none));
  merge_lane_lists<MB, KT>(smem, lk, sum, wave, lane, mtile * 64 * MB, p.R, p.part, p.k_top, p.nparts, range);
}

template <int MB, int KT>
static hipError_t launch_tile_t(const TileArgs& a, size_t smem, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  static bool attr_set = false;  // per instantiation
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(head_tile_kernel<MB, KT>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipExtLaunchKernelGGL((head_tile_kernel<MB, KT>), dim3(a.chunk * 8), dim3(kWaves * 64), smem, st, ev_start, ev_stop, 0, a);
  return hipGetLastError();
}

// Which head launches come here, of those that the panel kernel and head_once_kernel leave: alone (no projection), more than 64 rows, lists of at most 4, K in whole groups of kSteps
// steps (the cursor of the copies moves by groups; other widths stay with the dense kernel), and cheaper than the dense
// kernel by its own estimate.  Both estimates count tile rounds of the longest range; the unit is the dense kernel's 96-row
// tile, as in plan_gemm.  Launches of 4096 x 32000 (320, 384, 960 rows) and 3072 x 128256 (192, 768, 2304), us, dense kernel /
// blocks of 192, 256 rows here:  320: 91 / 94, 116;  384: 120 / 97, 121;  960: 229 / 239, 216;  192: 192 / 162, -;  768: 551 /
// 473, 454;  2304: 1569 / 1383, 1299 (another card: dense 103, 210, 201, 543, 1551; here, the better block, 84, 189, 160, 440,
// 1274).  So a tile costs 1.55 and 1.95.  The quotient holds for short K too: drafts of one stage, 272 shapes of 128 to 4096 rows,
// K = 128 to 8192 and 8000 to 128256 weight rows, and 260 random ones up to 26000 rows, are 1.007 to 1.38 times as fast where
// the rule comes here (960 rows x 32000: K = 128 58.8 / 55.7, 512 79.8 / 74.1, 1024 105.2 / 96.5); the least, 0.99 and 1.0, are
// 17000 and 20000 rows x 8000, where row blocks nearly fill the CUs by themselves.  One round each, as at 320 rows, is bound by the
// weights' way from memory in both, and the dense kernel keeps what is not 5 % better here; so it does where it shortens its
// tiles to reach more CUs, and where its blocks outnumber the CUs, whose rounds its estimate does not count.  (256 rows with
// lists of 4 do not fit the registers: 36 bytes of scratch a lane, parked entries and all.)
TilePlan plan_tile(int R, int k_top, int n_head, int kt, int n_cu) {
  TilePlan best;
  memset(&best, 0, sizeof(best));
  if (R <= 64 || R > (1 << 22) || n_head <= 0 || k_top < 1 || k_top > 4 || kt % kSteps) return best;
  const int cus = n_cu > 0 ? n_cu : 256, tiles = (n_head + 255) / 256;
  double cost = 0.95 * dense_head_cost(R, k_top, n_head, kt, n_cu);
  for (int block = 6; block <= 8; block += 2) {
    if (block == 8 && k_top > 3) continue;
    TilePlan c;
    c.block = block;
    c.kcap = k_top < 2 ? 2 : k_top;
    c.m_tiles = (R + 32 * block - 1) / (32 * block);
    c.n_tiles = tiles;
    c.n_ranges = cus / c.m_tiles < 1 ? 1 : cus / c.m_tiles;
    if (c.n_ranges > tiles) c.n_ranges = tiles;
    // (more row blocks than CUs: whole rounds of workgroups)
    const double here = (block == 6 ? 1.55 : 1.95) * ((tiles + c.n_ranges - 1) / c.n_ranges) *
                        ((c.m_tiles * c.n_ranges + cus - 1) / cus);
    if (here < cost) {
      best = c;
      cost = here;
    }
  }
  return best;
}

size_t tile_lds_bytes(const TilePlan& pl) {
  const size_t steps = (size_t)kSteps * (kWF + 2 * pl.block) * 1024 +
                       (tile_parks(pl.block / 2, pl.kcap) ? (size_t)kWaves * 64 * (pl.block / 2) * 8 : 0);
  const size_t merge = list_merge_bytes(pl.block / 2, pl.kcap);
  return steps > merge ? steps : merge;
}

hipError_t launch_head_tile(const HeadJob& job, const TilePlan& pl, hipStream_t st, hipEvent_t ev_start,
                            hipEvent_t ev_stop) {
  if (job.vt_proj > 0 || job.vt_head <= 0 || job.out_head || job.b_rowmajor || job.kt % kSteps || job.kt < kSteps ||
      job.k_top > pl.kcap || job.nparts != pl.n_ranges)
    return hipErrorInvalidValue;
  TileArgs a;
  memset(&a, 0, sizeof(a));
  a.w = static_cast<const u32x4*>(job.w_head);
  a.b = static_cast<const u32x4*>(job.b_src);
  a.kt = job.kt;
  a.tile_slots = job.tile_slots;
  a.nt_total = job.vt_head;
  a.n_valid = job.n_head;
  a.mt_total = (job.R + 15) / 16;
  a.R = job.R;
  a.m_tiles = pl.m_tiles;
  a.n_tiles = pl.n_tiles;
  a.n_ranges = pl.n_ranges;
  a.chunk = (pl.m_tiles * pl.n_ranges + 7) / 8;
  a.k_top = job.k_top;
  a.nparts = job.nparts;
  a.part = job.part;
  const size_t smem = tile_lds_bytes(pl);
  switch (pl.block * 10 + pl.kcap) {
    case 62: return launch_tile_t<3, 2>(a, smem, st, ev_start, ev_stop);
    case 63: return launch_tile_t<3, 3>(a, smem, st, ev_start, ev_stop);
    case 64: return launch_tile_t<3, 4>(a, smem, st, ev_start, ev_stop);
    case 82: return launch_tile_t<4, 2>(a, smem, st, ev_start, ev_stop);
    case 83: return launch_tile_t<4, 3>(a, smem, st, ev_start, ev_stop);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace specdraft
