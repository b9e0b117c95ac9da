// Pooled scores in ONE pass over the keys (Section 3.3; Algorithm 1's per-query-block loop), for callers
// that have no row log-sum-exp to hand over.
//
//   A'[I, J] = 1 / (rows x keys) * sum_{r in I} (1 / Z_r) * sum_{j in J} exp(s_rj - m_r),   Z_r = sum_j exp(s_rj - m_r)
//
// The normaliser Z_r of a query row is known only after its last key, so the per-row block sums
// E[r, J] = sum_{j in J} exp(s_rj - m_r) are parked in a scratch slab that belongs to the work-group (columns J of 128
// floats: O(L) per work-group, never O(L^2) in total; a wave stores two columns' worth of its 32 rows at a time) and,
// once the rows are complete, weighted by 1 / Z_r and summed over the rows of each query block. Work-groups are
// persistent: each walks the units (128 consecutive rows of a head: one, two or four query blocks) wg, wg + G, ... and
// reuses its slab.
//
// Reference m_r: the maximum logit of the row's first 32 keys. It is never above the row's true maximum, so
// nothing underflows that the two-pass form (reference = log-sum-exp) would keep. A later logit more than
// 100 octaves above it (never, on real attention logits) is caught by the overflow test on every 32-key
// sub-tile and handled out of line: the reference is raised, and the row's running sums and its parked block
// sums are rescaled.
//
// Bound: the vector unit. A 32-key sub-tile is 8 matrix instructions (256 cycles at head dim 128) and 16 fma, 16 exp2 and
// 16 adds, and an exp2 takes as long as 3.5 to 3.9 fma (about 380 cycles together). The slab is read and written
// by one work-group only, so its order is kept by work-group fences; the columns are read back as whole 16-byte pieces,
// eight in flight per wave.
// 32 heads of 16384 x 128, 64 x 64 blocks: 2.52 -> 2.19 ms (1.00 PFLOP/s); 3 samples (3000, 2100, 1200) x 8 heads of 64: 62 ->
// 39 us (41 with the two parts of a boundary block, which were a launch of 8.6). (Before: block sums staged in LDS row by row, a cache write-back at the end of every unit, four reads in flight in
// the closing pass, 48 to 76 bytes of spills.)
//
// Matrix work, K tile copies, fragment layouts and the 32-key software pipeline are those of pool_bf16_kernel
// (select.hip); exponentials, sums and weights are fp32 throughout, summed in a fixed order.
#include "kernels.hpp"
#include "tile_bf16.hpp"

namespace sparsed {

namespace {

[[maybe_unused]] constexpr float kOverflow = 1.2676506e30f;  // 2^100: a 32-key partial sum at or above this triggers the re-reference path

// Work-groups per compute unit the kernel is built for: two K tiles are under a quarter of the LDS.
constexpr int groups_per_cu(int) { return 4; }

}  // namespace

// QBW: waves per query block. A work-group always has 128 consecutive rows of a head, four waves: one query block of
// 128 rows, two of 64 or four of 32, which share its K tiles and its slab.
// The lane number and the kernel's arguments are worked out / read again where they are used late (fresh_lane,
// fresh_kernel_args): 128 registers a lane are all that four waves per SIMD leave, and a spill in the tile loop waits
// for the copies in flight.
// KS: runs that the keys are cut into, four waves each; all with the same rows.
template <int D, int KS, int BK, int QBW>
__global__ __launch_bounds__(KS * 256) __attribute__((amdgpu_waves_per_eu(4, 4))) void pool1p_bf16_kernel(const PoolArgs) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass only needs the launch stub (the body uses device-only types)
  constexpr int NW = 4, NT = NW * 64, QT = 32 * NW;  // waves and threads of a run, rows of a slab column
  constexpr int kKBytes = KLayout<D>::kTileBytes;
  __shared__ __attribute__((aligned(1024))) char kbuf0[KS * kKBytes];  // run r: its tile at r * kKBytes, which is part of kaddr
  __shared__ __attribute__((aligned(1024))) char kbuf1[KS * kKBytes];
  __shared__ __attribute__((aligned(16))) float inv_z[KS * QT];
  __shared__ float run_max[KS > 1 ? KS * QT : 1], run_sum[KS > 1 ? KS * QT : 1];  // reference and sum of a row in each run
  __shared__ float part_sum[2][NW];  // a wave's share of the two parts of the boundary's key block
  static_assert(NW % QBW == 0, "whole query blocks per work-group");
  constexpr int kBlocksPerGroup = NW / QBW, kBlockRows = 32 * QBW;

  const int wave_of_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave = wave_of_all % NW, run = KS > 1 ? wave_of_all / NW : 0;

  int unit = xcd_remap(blockIdx.x, gridDim.x), units = 0;  // a unit: QT consecutive rows of one head
  do {
    const KernelArgs<PoolArgs>& a = fresh_kernel_args<PoolArgs>();
    const int lane = fresh_lane();
    const int groups_per_head = (a.nqb + kBlocksPerGroup - 1) / kBlocksPerGroup;
    units = a.B * a.Hq * groups_per_head;
    const int gq = unit % groups_per_head;
    const Slab slab_of = slab_at(unit / groups_per_head, a);
    const int b = slab_of.b, h = slab_of.h, hk = slab_of.hk, bh = b * a.Hq + h;
    int L = a.L;  // length of this batch element
    if (a.seq_lens != nullptr) {
      const int len = a.seq_lens[b];
      L = len < a.L ? len : a.L;
    }
    if (gq * QT >= L) continue;  // rows this sample does not have (uniform over the work-group)
    const __bf16* qbase = static_cast<const __bf16*>(a.q.ptr) + b * a.q.sb + h * a.q.sh;
    const __bf16* kbase = static_cast<const __bf16*>(a.k.ptr) + b * a.k.sb + hk * a.k.sh;
    const int row0 = gq * QT + wave * 32;
    const float c = a.scale_log2;

    TileDma<D, NT, false> kdma;
    kdma.init(a.k.sl, wave, lane);
    KFragAddr<D> kaddr;
    kaddr.init(lane);
    if (KS > 1)
#pragma unroll
      for (int i = 0; i < KFragAddr<D>::kBases; ++i) kaddr.base[i] += run * kKBytes;
    QFrag<D, 1> qf;
    // This run's tiles: tile0 and the n - 1 behind it (an even tile0: a run's columns are its own and begin with a pair).
    const int n_all = (L - 1) / kTileK + 1;             // 64-key tiles that exist
    const int n_first = KS == 1 ? n_all : n_all < 2 ? n_all : ((n_all + 3) >> 2) * 2;  // tiles of the first run, no fewer than of the second
    const int tile0 = run * n_first, n = run == 0 ? n_first : n_all - n_first;
    const int last_blk = n - 1;
    const int tail_keys = tile0 + n == n_all ? L - (n_all - 1) * kTileK : kTileK;  // keys in the last of them
    auto keys_at = [&](int tile) -> int { return tile >= n ? 0 : tile == last_blk ? tail_keys : kTileK; };
    const int first_key = n > 0 ? tile0 * kTileK : 0;
    const __amdgpu_buffer_rsrc_t krsrc = make_rsrc(kbase + first_key * a.k.sl, ((int64_t)(L - 1 - first_key) * a.k.sl + D) * 2);
    const int64_t k_sl = a.k.sl;
    const int32_t k_tile_bytes = (int32_t)(kTileK * k_sl * 2);
    char* const kdst0 = kbuf0 + run * kKBytes;
    char* const kdst1 = kbuf1 + run * kKBytes;
    auto copy_k_any = [&](int tile, char* dst) {  // any tile: past the end repeats the last one, which may be partial
      const int blk = tile < n ? tile : n - 1;
      if (blk == last_blk && tail_keys < kTileK) kdma.issue_partial(krsrc, blk * k_tile_bytes, dst, wave, fresh_lane(), k_sl, tail_keys);
      else kdma.issue(krsrc, blk * k_tile_bytes, dst, wave);
    };

    f32x16 s_even[1], s_odd[1];
    float M = 0.f;                  // reference of this lane's row, in octaves (log2 units)
    float lsum = 0.f;               // this lane's share of Z_r
    float carry = 0.f, hold = 0.f;  // its share of the sub-tile before the one being summed / of the block before the one being completed

    // masked: apply `valid`, the number of keys of the sub-tile that exist (>= 32: all, <= 0: none)
    auto mask_sub = [&](f32x16(&s)[1], int valid) {
      const int mine = valid - 8 * (fresh_lane() >> 5);  // register x of lane (j, g) holds key 16*(x/8) + 8*g + x%8
#pragma unroll
      for (int x = 0; x < 16; ++x)
        if (16 * (x >> 3) + (x & 7) >= mine) s[0][x] = -__builtin_inff();
    };
    auto row_max = [&](const f32x16(&s)[1]) -> float {
      float mx = fmaxf(s[0][0], s[0][1]);
#pragma unroll
      for (int x = 2; x < 16; x += 2) mx = fmaxf(fmaxf(mx, s[0][x]), s[0][x + 1]);
      return pair_max(mx) * c;
    };
    auto exp_sum = [&](const f32x16(&s)[1]) -> float {
      float part = 0.f;
#pragma unroll
      for (int x = 0; x < 16; ++x) part += __builtin_amdgcn_exp2f(__builtin_fmaf(s[0][x], c, -M));
      asm volatile("" : "+v"(part));  // keep the vector work inside the block that holds the matrix work
      return part;
    };
    // The slab: columns J of QT floats, stored two at a time (both halves of a wave), or once per two tiles with 128-key blocks.
    const int col0 = BK == kTileK / 2 ? 2 * tile0 : BK == kTileK ? tile0 : tile0 >> 1;  // this run's first column
    float* const slab = a.slab + ((int64_t)blockIdx.x * a.slab_ld + col0) * QT;
    const __amdgpu_buffer_rsrc_t slab_rsrc = make_rsrc(slab, (int64_t)QT * (a.slab_ld - col0) * 4);
    auto park_store = [&](int col, float v) {
      const int ln = fresh_lane();
      const int off = 4 * ((BK == 2 * kTileK ? 0 : (ln >> 5) * QT) + (ln & 31));
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), slab_rsrc, off, (col * QT + wave * 32) * 4, 0);
    };
    // after sub-tile 2t+1 (sum `part`): key tile t is complete. P = t & 1.
    auto park_tile = [&](const int P, const bool maybe_last, int t, float part) {
      if (BK == kTileK / 2) {
        park_store(2 * t, two_pair_sums(carry, part));
        return;
      }
      const float e = carry + part;
      if (BK == kTileK) {
        if (P) park_store(t - 1, two_pair_sums(hold, e));
        else if (maybe_last && t == n - 1) park_store(t, two_pair_sums(e, 0.f));
        else hold = e;
      } else {
        if (P) park_store(t >> 1, pair_sum(hold + e));
        else if (maybe_last && t == n - 1) park_store(t >> 1, pair_sum(e));
        else hold = e;
      }
    };
    // Out of line: some partial sum overflowed the reference. Raise the reference of the rows concerned to their new
    // maximum, rescale everything they have accumulated (tiles_done key tiles are complete), redo the sub-tile's sum.
    auto re_reference = [&](const f32x16(&s)[1], float& part, int tiles_done) {
      const float Mn = fmaxf(M, row_max(s));
      // 2^(M - Mn) in two factors: the sums are up to 2^100, so that what is left of them counts where the one factor were zero
      const float half = __builtin_amdgcn_exp2f(0.5f * (M - Mn));  // <= 1; exactly 1 where nothing changes
      M = Mn;
      auto rescaled = [&](float x) -> float { return x * half * half; };
      lsum = rescaled(lsum);
      carry = rescaled(carry);
      hold = rescaled(hold);
      const int cols = BK == kTileK / 2 ? 2 * tiles_done : BK == kTileK ? tiles_done & ~1 : tiles_done >> 1;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // this wave's parked sums have been written
      if (half < 1.0f)  // (not for a NaN: the row is lost anyway)
        for (int J = fresh_lane() >> 5; J < cols; J += 2) {
          float* const e = slab + (int64_t)J * QT + wave * 32 + (fresh_lane() & 31);
          *e = rescaled(*e);
        }
      part = exp_sum(s);
    };
    auto overflowed = [&](float part) -> bool { return __builtin_amdgcn_ballot_w64(!(part < kOverflow)) != 0; };

    // Tile step t (LDS parity P = t & 1) = sub-tiles 2t+1 and 2t+2. On entry S(2t+1) is in s_odd, K(t+1) in
    // kbuf[1-P]; kbuf[P] is free and receives K(t+2). Tiles past the end are phantoms (a repeated copy, every key
    // masked); MASKED steps (the last few) count the keys that exist in each sub-tile.
#define SPARSED_POOL1P_STEP(P, MASKED, T)                                                          \
  {                                                                                                \
    char* const kb_free = (P) ? kdst1 : kdst0;                                                     \
    char* const kb_next = (P) ? kbuf0 : kbuf1;                                                     \
    if (MASKED) copy_k_any((T) + 2, kb_free);                                                      \
    else kdma.issue(krsrc, ((T) + 2 < n ? (T) + 2 : n - 1) * k_tile_bytes, kb_free, wave);         \
    logits_sub<D, 1, false>(kb_next, 0, kaddr, qf, s_even);                                        \
    if (MASKED) mask_sub(s_odd, keys_at(T) - 32);                                                  \
    float part = exp_sum(s_odd);                                                                   \
    sched_substep_interleave<D, 1, false>();                                                       \
    if (__builtin_expect(overflowed(part), 0)) re_reference(s_odd, part, (T));                     \
    lsum += part;                                                                                  \
    park_tile((P), (MASKED), (T), part);                                                           \
    __builtin_amdgcn_sched_barrier(0);                                                             \
    logits_sub<D, 1, false>(kb_next, 1, kaddr, qf, s_odd);                                         \
    if (MASKED) mask_sub(s_even, keys_at((T) + 1));                                                \
    part = exp_sum(s_even);                                                                        \
    sched_substep_interleave<D, 1, false>();                                                       \
    if (__builtin_expect(overflowed(part), 0)) re_reference(s_even, part, (T) + 1);                \
    lsum += part;                                                                                  \
    carry = part;                                                                                  \
    __syncthreads();                                                                               \
  }

    // prologue: K(0), K(1) (a repeat of K(0) for a one-tile range) into LDS; S(0); reference and sums of sub-tile 0
    if (KS == 1 || n > 0) {
      copy_k_any(0, kdst0);
      copy_k_any(1, kdst1);
      qf.load(qbase, row0, L, a.q.sl, lane);
    }
    __syncthreads();
    if (KS == 1 || n > 0) {
      logits_sub<D, 1, true>(kbuf0, 0, kaddr, qf, s_even);
      logits_sub<D, 1, true>(kbuf0, 1, kaddr, qf, s_odd);
      mask_sub(s_even, keys_at(0));
      M = row_max(s_even);  // at least one key exists, so this is finite
      if (KS > 1 && run > 0) M = fmaxf(M, -1e30f);  // (keys of logit -inf behind others: their sums are 0)
      carry = exp_sum(s_even);
      lsum = carry;
    }
    __syncthreads();  // everyone is done with K(0) before tile step 0 lets K(2) overwrite it

    const int steady_reach = (tail_keys < kTileK) ? 4 : 2;
    int t = 0;
    while (t + steady_reach < n) {
      SPARSED_POOL1P_STEP(0, false, t);
      SPARSED_POOL1P_STEP(1, false, t + 1);
      t += 2;
    }
    for (; t < n; ++t) {
      if (t & 1) {
        SPARSED_POOL1P_STEP(1, true, t);
      } else {
        SPARSED_POOL1P_STEP(0, true, t);
      }
    }
#undef SPARSED_POOL1P_STEP
    if (KS > 1)
      for (t = n > 0 ? n : 0; t < n_first; ++t) __syncthreads();  // a shorter run keeps step

    // The rows are complete: 1 / Z_r (0 for rows past the end), and then
    // A'[I, J] = sum_r E[r, J] / Z_r over the rows of the block, divided by the entries that exist: a lane weighs the same
    // four rows of every column, and the lanes of a query block (8, 16 or 32) are summed in a fixed order.
    const KernelArgs<PoolArgs>& ae = fresh_kernel_args<PoolArgs>();
    const int lane_e = fresh_lane();
    const float ltot = pair_sum(lsum);
    float weight = 1.0f / ltot;
    if (KS > 1) {
      // 1 / Z_r against this run's reference, Z_r from both runs' sums. A run without a sum has no say in the common reference.
      const int at = wave * 32 + (lane_e & 31);
      if (lane_e < 32) {
        run_max[run * QT + at] = M;
        run_sum[run * QT + at] = ltot;
      }
      __syncthreads();
      const float l0 = run_sum[at], l1 = run_sum[QT + at];
      const float m0 = l0 == 0.f ? -3e38f : run_max[at], m1 = l1 == 0.f ? -3e38f : run_max[QT + at];
      const float m = fmaxf(m0, m1), mine = run ? m1 : m0;
      const float a0 = __builtin_amdgcn_exp2f(m0 - m), a1 = __builtin_amdgcn_exp2f(m1 - m);
      weight = (run ? a1 : a0) / (l0 * a0 + l1 * a1);
      // A run's later logits may lie up to 100 octaves above its reference before that is raised, so its sums can count beside
      // the other run's where the factor between the references alone is near or below the smallest float. Rows whose
      // references are that far apart (out of line, practically never) take it in two steps, their parked sums right here.
      const bool apart = l0 != 0.f && l1 != 0.f && fabsf(m0 - m1) > 100.f;
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(apart) != 0, 0)) {
        const float h = __builtin_amdgcn_exp2f(0.5f * (mine - m)), h0 = __builtin_amdgcn_exp2f(0.5f * (m0 - m)),
                    h1 = __builtin_amdgcn_exp2f(0.5f * (m1 - m));
        if (apart) {
          weight = 1.0f / (l0 * h0 * h0 + l1 * h1 * h1);
          M = m;
        }
        const int cols = BK == kTileK / 2 ? 2 * n : BK == kTileK ? n : (n + 1) >> 1;
        wait_vector_memory();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // this wave's parked sums have been written
        if (apart && mine < m)
          for (int J = lane_e >> 5; J < cols; J += 2) {
            float* const e = slab + (int64_t)J * QT + at;
            *e = *e * h * h;
          }
      }
    }
    const bool splits = ae.part != nullptr && L > ae.boundary;
    if (splits) {
      // The key block that holds the prefill boundary once more, its keys before the boundary and the others apart: one or two
      // tiles against the row statistics that are at hand here, instead of a launch that reads Q and the statistics again.
      // 3 samples (3000, 2100, 1200) x 8 heads of 64, 128 x 128 blocks, 30 % kept: 73.2 -> 68.5 us with
      // the sparse step (the launch: 8.3 us).
      const int begin = ae.boundary / BK * BK / kTileK, end = (ae.boundary / BK * BK + BK - 1) / kTileK;
      const bool mine = KS == 1 || (begin >= n_first) == (run == 1);  // the run that has the block
      float before = 0.f, behind = 0.f;
      for (int tile = begin; tile <= end && tile < n_all; ++tile) {
        if (mine) copy_k_any(tile - tile0, kdst0);
        __syncthreads();
#pragma unroll 1
        for (int sub = 0; sub < 2; ++sub) {
          const int key0 = tile * kTileK + 32 * sub;
          if (!mine || (BK < kTileK && (key0 & ~(BK - 1)) != ae.boundary / BK * BK)) continue;  // (the other block of the tile)
          logits_sub<D, 1, false>(kbuf0, sub, kaddr, qf, s_even);
          int first = key0 + 8 * (lane_e >> 5);  // key of register 0
          asm volatile("" : "+v"(first));  // the comparisons below stay here: sixteen masks at once do not fit
#pragma unroll
          for (int x = 0; x < 16; ++x) {
            const int key = first + 16 * (x >> 3) + (x & 7);
            const float e = key < L ? __builtin_amdgcn_exp2f(__builtin_fmaf(s_even[0][x], c, -M)) : 0.f;
            if (key < ae.boundary) before += e;
            else behind += e;
          }
        }
        __syncthreads();  // the tile may be overwritten
      }
      const float z = row0 + (lane_e & 31) < L ? weight : 0.f;
      before = lane_group_sum_to_last(pair_sum(before) * z, 32);
      behind = lane_group_sum_to_last(pair_sum(behind) * z, 32);
      if (lane_e == 31 && mine) {
        part_sum[0][wave] = before;
        part_sum[1][wave] = behind;
      }
    }
    if (lane_e < 32) {
      const bool exists = row0 + lane_e < L;
      inv_z[run * QT + wave * 32 + lane_e] = exists ? weight : 0.f;
    }
    wait_vector_memory();  // this wave's parked sums have been written
    __syncthreads();  // all parked sums and weights of the group are written
    if (splits && (int)threadIdx.x < 2 * kBlocksPerGroup) {
      const int which = threadIdx.x & 1, blk = threadIdx.x >> 1, Ib = gq * kBlocksPerGroup + blk;
      const int rows = L - Ib * kBlockRows < kBlockRows ? L - Ib * kBlockRows : kBlockRows;
      const int begin = ae.boundary / BK * BK, end = begin + BK < L ? begin + BK : L;
      float x = 0.f;
#pragma unroll
      for (int w = 0; w < QBW; ++w) x += part_sum[which][blk * QBW + w];
      if (rows > 0) ae.part[((int64_t)bh * ae.nqb + Ib) * 2 + which] = x * (1.0f / (float)(rows * (which ? end - ae.boundary : ae.boundary - begin)));
    }
    constexpr int kLanes = QT / 4, kCols = 64 / kLanes, kUnroll = 8;  // lanes per column, columns per wave load
    const int li = lane_e % kLanes, sub_col = lane_e / kLanes;
    const f32x4v w0 = *reinterpret_cast<const f32x4v*>(&inv_z[4 * li]);
    f32x4v w1 = w0;
    if (KS > 1) w1 = *reinterpret_cast<const f32x4v*>(&inv_z[(KS - 1) * QT + 4 * li]);
    const int col1 = (n_first * kTileK + BK - 1) / BK;  // the second run's first column
    const float* const all = slab - (int64_t)col0 * QT;
    const int I = gq * kBlocksPerGroup + 4 * li / kBlockRows;
    const int rows_here = L - I * kBlockRows < kBlockRows ? L - I * kBlockRows : kBlockRows;
    const bool writes = (4 * li + 4) % kBlockRows == 0 && rows_here > 0;  // the last lane of a query block that exists
    float* const arow = ae.apool + ((int64_t)bh * ae.nqb + I) * ae.out_stride;
    const int nkb_here = (L + BK - 1) / BK;  // key blocks this sample has
    for (int J0 = wave_of_all * (kCols * kUnroll); J0 < nkb_here; J0 += KS * NW * kCols * kUnroll) {
      f32x4v e[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int J = J0 + u * kCols + sub_col;
        e[u] = *reinterpret_cast<const f32x4v*>(all + (int64_t)(J < nkb_here ? J : nkb_here - 1) * QT + 4 * li);
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int J = J0 + u * kCols + sub_col;
        const f32x4v w = KS > 1 && J >= col1 ? w1 : w0;
        float x = e[u][0] * w[0] + e[u][1] * w[1] + e[u][2] * w[2] + e[u][3] * w[3];
        x = lane_group_sum_to_last(x, kBlockRows / 4);
        const int keys_here = L - J * BK < BK ? L - J * BK : BK;
        if (writes && J < nkb_here) arow[J] = x * (1.0f / (float)(rows_here * keys_here));  // mean over the entries that exist
      }
    }
    __syncthreads();  // the K buffers, the weights and the slab are free for the next unit
  } while ((unit += gridDim.x) < units);
#endif
}

int pool1p_groups(int) { return 256 * groups_per_cu(4); }

int64_t pool1p_units(int B, int Hq, int nqb, int block_q) {
  const int per = 128 / block_q;  // query blocks per work-group
  return (int64_t)B * Hq * ((nqb + per - 1) / per);
}

template <int D, int KS, int QBW>
static hipError_t launch_pool1p_bk(const PoolArgs& a, int groups, hipStream_t s) {
  const dim3 grid((unsigned)groups), block(KS * 256);
  switch (a.block_k) {
    case 32: hipLaunchKernelGGL((pool1p_bf16_kernel<D, KS, 32, QBW>), grid, block, 0, s, a); break;
    case 64: hipLaunchKernelGGL((pool1p_bf16_kernel<D, KS, 64, QBW>), grid, block, 0, s, a); break;
    case 128: hipLaunchKernelGGL((pool1p_bf16_kernel<D, KS, 128, QBW>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int D, int KS>
static hipError_t launch_pool1p_q(int block_q, const PoolArgs& a, int groups, hipStream_t s) {
  if (block_q == 128) return launch_pool1p_bk<D, KS, 4>(a, groups, s);
  if (block_q == 64) return launch_pool1p_bk<D, KS, 2>(a, groups, s);
  return launch_pool1p_bk<D, KS, 1>(a, groups, s);
}

// Two key runs: the same number of waves in flight, half as many units at a time and each in half the time. It pays with at most a
// unit a compute unit, where it is twice the waves, and where one to three whole rounds of the chip (1024 units) leave
// a last one that is at most half full, but not empty, if the runs are long enough for what merging them costs every unit. Selections, two runs
// against one, by 128-row units and tokens. Head dim 64, up to 256 units: 1500 0.95, 2000 to 3000 0.92, longer 0.86; 1025 to 1280:
// 250 to 1000 1.23, 1000 to 2000 0.92, longer 0.88; to 1536 1.05, 0.93, 0.84; a round more 1.27, 0.98, 0.93; two more 1.23, 1.02,
// 0.93; three more 1.0 at best. Head dim 128: 1.01, 0.96, 0.89; 1.1, 1.02, 0.94; 1.1, 0.93, 0.85; a round more 1.33, 1.11, 1.05 and
// (from 2305 units) 1.26, 1.01, 0.96; two more 1.0 at best. 257 to 1024 units: 1.0 to 1.4 (32 heads of 3000 x 128 96 -> 131 us). With
// fewer slabs than a round the rounds are others; with lengths per sample they are a guess (0.97 on average, 0.79 to 1.18).
static int key_runs(int D, const PoolArgs& a, int64_t units, int groups) {
  const int tiles = (a.L + kTileK - 1) / kTileK;
  if (units <= 256) return tiles >= (D == 64 ? 24 : 30) ? 2 : 1;
  if (units <= 1024 || groups < 1024) return 1;
  const int64_t full = (units - 1) / 1024, left = units - full * 1024;
  if (left <= 64 || left > 512 || full > (D == 64 ? 3 : 2)) return 1;  // (a few units more than a round: 1.05 to 1.14)
  if (D == 64 || left > 256) return tiles >= 16 * full ? 2 : 1;
  return full == 1 && tiles >= 32 ? 2 : 1;
}

// One-pass pooled scores over the whole key range of every sample. a.slab holds `groups` slabs of
// 128 x a.slab_ld floats; a.part (optional) receives the scores of the two parts of the boundary block.
hipError_t launch_pool1p_bf16(int D, int block_q, const PoolArgs& a, int groups, hipStream_t s) {
  if (block_q != 128 && block_q != 64 && block_q != 32) return hipErrorInvalidValue;
  const int64_t units = pool1p_units(a.B, a.Hq, a.nqb, block_q);
  if (units <= 0 || units > 0x7fffffff || groups < 1 || a.slab == nullptr || a.slab_ld < a.out_stride) return hipErrorInvalidValue;
  if (groups > units) groups = (int)units;
  if (key_runs(D, a, units, groups) == 2) {
    if (groups > 512) groups = 512;  // two a compute unit
    if (D == 128) return launch_pool1p_q<128, 2>(block_q, a, groups, s);
    if (D == 64) return launch_pool1p_q<64, 2>(block_q, a, groups, s);
  } else {
    if (D == 128) return launch_pool1p_q<128, 1>(block_q, a, groups, s);
    if (D == 64) return launch_pool1p_q<64, 1>(block_q, a, groups, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace sparsed
