// Pattern selection for gfx950 (Section 3.3; Algorithm 1's per-query-block loop; Eq. 6):
//   pool_*_kernel  A'[I, J] = mean over the block_q x block_k rectangle of the softmax
//                  probabilities of Eq. 1 (every row normalised over all L keys, via the row
//                  log-sum-exp of the statistics pass, or what a dense call left). A work-group walks
//                  all key tiles, or those of a segment, once; the L x L matrix never exists.
//   topk_kernel    per pooled row, the k largest entries (ties: lower block index), written
//                  ascending into the per-head CSR block index. One wavefront per row.
// Pooled scores are fp32 from the logits on: the exponentials, the normaliser and every partial
// sum, with a fixed summation order (lane, then wave tree, then waves in order).
#include <type_traits>

#include "kernels.hpp"
#include "tile_bf16.hpp"
#include "tile_f32.hpp"
#include "topk_row.hpp"

namespace sparsed {

// ---------------------------------------------------------------------------- pooled scores, bf16
// Sum of one value per lane over the 64 lanes of a wave with DPP row operations (no LDS traffic);
// the total ends up in lane 63.
__device__ __forceinline__ float wave_sum_to_last_lane(float x) {
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x111, 0xf, 0xf, true));  // row_shr:1
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x112, 0xf, 0xf, true));  // row_shr:2
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x114, 0xf, 0xf, true));  // row_shr:4
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x118, 0xf, 0xf, true));  // row_shr:8
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x142, 0xa, 0xf, true));  // row_bcast:15
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x143, 0xc, 0xf, true));  // row_bcast:31
  return x;
}

// One work-group of NW waves, 32 query rows each, covers NW / QBW consecutive query blocks of QBW waves (one block
// of 128 rows, two of 64 or four of 32 with NW = 4: small query blocks share the work-group's K tiles and keep four
// waves on every SIMD). Same 32-key software pipeline as
// the attention kernels: sub-step u interleaves the matrix work S(u+1) = K(u+1) Q^T with the vector
// work of sub-tile u (p = 2^(s*c - lse), summed per lane). A key block is two sub-tiles; its
// per-lane sums are reduced over the wave, then over the waves of its query block through LDS in a fixed order.
// HALF: key blocks of 32 (the two 32-key sub-tiles of a tile are pooled separately).
template <int D, int NW, bool HALF, int QBW = NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(NW >= 4 ? 4 : NW >= 2 ? 2 : 1, NW >= 4 ? 4 : NW >= 2 ? 2 : 1)))
void pool_bf16_kernel(const PoolArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass only needs the launch stub (the body uses device-only types)
  constexpr int NT = NW * 64;
  constexpr int kKBytes = KLayout<D>::kTileBytes;
  __shared__ __attribute__((aligned(1024))) char kbuf0[kKBytes];
  __shared__ __attribute__((aligned(1024))) char kbuf1[kKBytes];
  __shared__ float wsum[2][NW];
  __shared__ float wsum_even[2][NW];  // HALF only: the even sub-tile's sums (wsum then holds the odd one's)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 31;
  static_assert(NW % QBW == 0, "whole query blocks per work-group");
  constexpr int kBlocksPerGroup = NW / QBW, kBlockRows = 32 * QBW;
  const int lid = xcd_remap(blockIdx.x, gridDim.x);
  const int groups_per_head = (a.nqb + kBlocksPerGroup - 1) / kBlocksPerGroup;
  const int gq = lid % groups_per_head;  // which run of 32 * NW rows of the head
  const Slab slab_of = slab_at(lid / groups_per_head, a);
  const int b = slab_of.b, h = slab_of.h, hk = slab_of.hk, bh = b * a.Hq + h;
  const int first_wave = (wave / QBW) * QBW;            // first wave of this wave's query block
  const int I = gq * kBlocksPerGroup + wave / QBW;      // this wave's query block

  // length of this batch element (per-sample lengths shorten the whole-sequence key range with it)
  int L = a.L;
  // which part of the keys: the whole range, one of the launch's two ranges, or a segment of the range
  int key_begin = a.key_begin, key_len = a.key_len, first_col = 0;
  if (a.seg_len > 0) {
    const int skip = blockIdx.y * a.seg_len;
    key_begin += skip;
    key_len = key_len - skip < a.seg_len ? key_len - skip : a.seg_len;
    first_col = skip / a.block_k;
  } else if (blockIdx.y) {
    key_begin += key_len;
    key_len = a.key_len2;
    first_col = 1;
  }
  if (a.seq_lens != nullptr) {
    const int len = a.seq_lens[b];
    L = len < a.L ? len : a.L;
    key_len = L - key_begin < key_len ? L - key_begin : key_len;
  }
  if (gq * (32 * NW) >= L || key_len <= 0) return;  // uniform over the work-group
  const __bf16* qbase = static_cast<const __bf16*>(a.q.ptr) + b * a.q.sb + h * a.q.sh;
  const __bf16* kbase = static_cast<const __bf16*>(a.k.ptr) + b * a.k.sb + hk * a.k.sh + (int64_t)key_begin * a.k.sl;
  const int row0 = gq * (32 * NW) + wave * 32;
  // a query block of the group that the head (or this sample) does not have: its waves run along with all-zero terms
  const bool block_exists = I < a.nqb && I * kBlockRows < L;

  QFrag<D, 1> qf;
  qf.load(qbase, row0, L, a.q.sl, lane);
  // What a term is relative to, and what the sums of a row are weighed by: its log-sum-exp and 1, or its reference and 1 / its sum
  // where the dense call left those (the log-sum-exp, rounded to fp32, is off by 2^-24 of its size: 4 heads of 2048 x 128, scores
  // to 4e-7 of themselves with it, to 5e-8 so). A query row past L (partial last query block): infinitely far, all its terms are 0.
  float ref = __builtin_inff(), weight = 1.f;
  if (row0 + j < L) {
    const int64_t at = (int64_t)bh * a.L + row0 + j;
    if (a.row_stat != nullptr) {
      const f32x2 stat = *reinterpret_cast<const f32x2*>(a.row_stat + 2 * at);
      ref = stat[0];
      weight = stat[1];
    } else {
      ref = a.lse[at] * 1.4426950408889634f;
    }
  }
  float* arow = a.apool + ((int64_t)bh * a.nqb + I) * a.out_stride + first_col;
  const int rows_here = (L - I * kBlockRows < kBlockRows) ? L - I * kBlockRows : kBlockRows;  // query rows of the block that exist
  const int last_blk = (key_len - 1) / kTileK;
  const int tail_keys = key_len - last_blk * kTileK;  // keys that exist in the last key block of the range
  auto keys_of = [&](int blk) -> int { return blk == last_blk ? tail_keys : kTileK; };

  TileDma<D, NT, false> kdma;
  kdma.init(a.k.sl, wave, lane);
  KFragAddr<D> kaddr;
  kaddr.init(lane);
  const __amdgpu_buffer_rsrc_t krsrc = make_rsrc(kbase, ((int64_t)(key_len - 1) * a.k.sl + D) * 2);
  const int32_t k_tile_bytes = (int32_t)(kTileK * a.k.sl * 2);
  const int n = last_blk + 1;
  const float c = a.scale_log2;

  auto copy_k_any = [&](int tile, char* dst) {  // any tile: past the end repeats the last one, which may be partial
    const int blk = tile < n ? tile : n - 1;
    if (blk == last_blk && tail_keys < kTileK) kdma.issue_partial(krsrc, blk * k_tile_bytes, dst, wave, lane, a.k.sl, tail_keys);
    else kdma.issue(krsrc, blk * k_tile_bytes, dst, wave);
  };
  auto keys_at = [&](int tile) -> int { return tile < n ? keys_of(tile) : 0; };  // keys that exist in a tile (none in a phantom)
  f32x16 s_even[1], s_odd[1];
  float carry = 0.f;  // per-lane sum of the even sub-tile of the key block in progress
  const int g = lane >> 5;
  // masked: apply `valid`, the number of keys of the sub-tile that exist (>= 32: all, <= 0: none)
  auto expsum_sub = [&](f32x16(&s)[1], const bool masked, int valid) -> float {
    if (masked) {
      const int mine = valid - 8 * g;  // register x of lane (j, g) holds key 16*(x/8) + 8*g + x%8
#pragma unroll
      for (int x = 0; x < 16; ++x)
        if (16 * (x >> 3) + (x & 7) >= mine) s[0][x] = -__builtin_inff();
    }
    float part = 0.f;
#pragma unroll
    for (int x = 0; x < 16; ++x) part += __builtin_amdgcn_exp2f(__builtin_fmaf(s[0][x], c, -ref));
    part *= weight;
    asm volatile("" : "+v"(part));  // keep the vector work inside the block that holds the matrix work
    return part;
  };
  const int tile_shift = a.block_k == 2 * kTileK ? 1 : 0;  // a 128-key block is pooled over two consecutive tiles
  float block_acc = 0.f;                                   // first thread of a query block: sum over the tiles of the key block in progress
  auto flush_block = [&](int t, float part) {  // after the tile barrier: key tile t is complete
    (void)part;
    if (tid == first_wave * 64 && block_exists) {
      if (HALF) {  // two 32-key blocks per tile; the second may not exist in the last tile
        float ev = 0.f, od = 0.f;
#pragma unroll
        for (int w = 0; w < QBW; ++w) {
          ev += wsum_even[t & 1][first_wave + w];
          od += wsum[t & 1][first_wave + w];
        }
        const int left = key_len - t * kTileK;  // keys from this tile's first on
        arow[2 * t] = ev * (1.0f / (float)(rows_here * (left < 32 ? left : 32)));
        if (left > 32) arow[2 * t + 1] = od * (1.0f / (float)(rows_here * (left - 32 < 32 ? left - 32 : 32)));
        return;
      }
      float tot = block_acc;
#pragma unroll
      for (int w = 0; w < QBW; ++w) tot += wsum[t & 1][first_wave + w];
      if ((t & tile_shift) == tile_shift || t == n - 1) {  // last tile of its key block
        const int J = t >> tile_shift;
        const int keys_here = key_len - J * a.block_k < a.block_k ? key_len - J * a.block_k : a.block_k;
        arow[J] = tot * (1.0f / (float)(rows_here * keys_here));  // mean over the entries that exist
        tot = 0.f;
      }
      block_acc = tot;
    }
  };

  // Tile step t (LDS parity P = t & 1) = sub-steps 2t+1 and 2t+2. On entry S(2t+1) is in s_odd, the
  // per-lane sum of sub-tile 2t in `carry`, K(t+1) in kbuf[1-P]; kbuf[P] is free and receives K(t+2).
  // Tiles past the end of the range are phantoms (a repeated copy, every key masked), so one branch-free
  // step serves the whole range; MASKED steps (the last few) count the keys that exist in each sub-tile.
#define SPARSED_POOL_STEP(P, MASKED, T)                                                            \
  {                                                                                                \
    char* const kb_free = (P) ? kbuf1 : kbuf0;                                                     \
    char* const kb_next = (P) ? kbuf0 : kbuf1;                                                     \
    if (MASKED) copy_k_any((T) + 2, kb_free);                                                      \
    else kdma.issue(krsrc, ((T) + 2 < n ? (T) + 2 : n - 1) * k_tile_bytes, kb_free, wave);         \
    logits_sub<D, 1, false>(kb_next, 0, kaddr, qf, s_even);                                        \
    float part = (HALF ? 0.f : carry) + expsum_sub(s_odd, (MASKED), keys_at(T) - 32);              \
    sched_substep_interleave<D, 1, false>();                                                       \
    part = wave_sum_to_last_lane(part);                                                            \
    if (lane == 63) wsum[(P)][wave] = part;                                                        \
    if (HALF) {                                                                                    \
      const float ev = wave_sum_to_last_lane(carry);                                               \
      if (lane == 63) wsum_even[(P)][wave] = ev;                                                   \
    }                                                                                              \
    __builtin_amdgcn_sched_barrier(0);                                                             \
    logits_sub<D, 1, false>(kb_next, 1, kaddr, qf, s_odd);                                         \
    carry = expsum_sub(s_even, (MASKED), keys_at((T) + 1));                                        \
    sched_substep_interleave<D, 1, false>();                                                       \
    __syncthreads();                                                                               \
    flush_block((T), part);                                                                        \
  }

  // prologue: K(0), K(1) (a repeat of K(0) for a one-tile range) into LDS; S(0); the sums of sub-tile 0
  copy_k_any(0, kbuf0);
  copy_k_any(1, kbuf1);
  __syncthreads();
  logits_sub<D, 1, true>(kbuf0, 0, kaddr, qf, s_even);
  logits_sub<D, 1, true>(kbuf0, 1, kaddr, qf, s_odd);
  carry = expsum_sub(s_even, true, keys_at(0));
  __syncthreads();  // everyone is done with K(0) before tile step 0 lets K(2) overwrite it

  // an unmasked step at tile t touches tiles t, t+1 (sums) and t+2 (copy, possibly a repeat); a partial last
  // block must stay out of its reach on all three counts, a full one only as far as t+1
  const int steady_reach = (tail_keys < kTileK) ? 4 : 2;
  int t = 0;
  while (t + steady_reach < n) {
    SPARSED_POOL_STEP(0, false, t);
    SPARSED_POOL_STEP(1, false, t + 1);
    t += 2;
  }
  for (; t < n; ++t) {
    if (t & 1) {
      SPARSED_POOL_STEP(1, true, t);
    } else {
      SPARSED_POOL_STEP(0, true, t);
    }
  }
#undef SPARSED_POOL_STEP
#endif
}

// ---------------------------------------------------------------------------- pooled scores, fp32
// One work-group of eight waves per query block: RW = block_q / 32 row groups times KW = 8 / RW key groups. Wave
// (rw, kw) sums, for its 32 rows, the key blocks kw, kw + KW, ...; the row groups' sums of a block meet in LDS (in row
// group order), a segment of blocks at a time. Products on split operands (tile_f32.hpp); every wave has its own K tile in LDS,
// copied again as soon as its last chunk has been read, so there is no barrier inside a segment.
// Bound: the vector unit (440 instructions a tile, 350 of them to split K). 8 heads of 2000 x 128, 64 x 64 blocks: 84 -> 61 us;
// 2 heads of 256 x 64: 7.4 -> 6.6 us.
template <int D, int RW>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void pool_f32_kernel(const PoolArgs a) {
  constexpr int KW = 8 / RW, kChunks = D / 8, kSteps = D / 16, kSeg = 512;
  __shared__ float sums[RW][kSeg];
  __shared__ __attribute__((aligned(1024))) char ktiles[8 * KTileF32<D>::kBytes];  // every wave's own

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rw = wave % RW, kw = wave / RW;
  char* const ktile = ktiles + wave * KTileF32<D>::kBytes;
  const int j = lane & 31, g = lane >> 5;
  const int lid = xcd_remap_f(blockIdx.x, gridDim.x);
  const int I = lid % a.nqb;
  const Slab slab_of = slab_at(lid / a.nqb, a);
  const int b = slab_of.b, h = slab_of.h, hk = slab_of.hk, bh = b * a.Hq + h;

  int L = a.L;                    // length of this batch element
  const int second = blockIdx.y;  // which of the launch's key ranges
  const int key_begin = second ? a.key_begin + a.key_len : a.key_begin;
  int key_len = second ? a.key_len2 : a.key_len;
  if (a.seq_lens != nullptr) {
    const int len = a.seq_lens[b];
    L = len < a.L ? len : a.L;
    key_len = L - key_begin < key_len ? L - key_begin : key_len;
  }
  if (I * (32 * RW) >= L || key_len <= 0) return;  // uniform over the work-group
  SlabF32<D> ks;
  ks.init(static_cast<const float*>(a.k.ptr) + b * a.k.sb + hk * a.k.sh + (int64_t)key_begin * a.k.sl, a.k.sl, key_len);
  const int row = I * (32 * RW) + rw * 32 + j;
  const float* const qrow = static_cast<const float*>(a.q.ptr) + b * a.q.sb + h * a.q.sh + (int64_t)(row < L ? row : L - 1) * a.q.sl + 4 * g;
  // a query row past L (partial last query block) gets an infinite normaliser: all its terms are 0
  const float lse2 = row < L ? a.lse[(int64_t)bh * a.L + row] * 1.4426950408889634f : __builtin_inff();
  float* arow = a.apool + ((int64_t)bh * a.nqb + I) * a.out_stride + second;
  const int rows_here = (L - I * (32 * RW) < 32 * RW) ? L - I * (32 * RW) : 32 * RW;  // query rows that exist
  const int nkb = (key_len + a.block_k - 1) / a.block_k;
  const float c = a.scale_log2;

  // The wave's key blocks of all segments. SPLIT: on the bf16 matrix instruction; else on the fp32 one. Returns whether some
  // sum of this lane is infinite or not a number, or the logits may be short of bits (tile_f32.hpp).
  auto walk = [&](auto split_tag) __attribute__((always_inline)) -> bool {
    constexpr bool SPLIT = decltype(split_tag)::value;
    f32x4 kf[SPLIT ? 1 : kChunks], qf[SPLIT ? 1 : kChunks];
    Split8 qs[SPLIT ? kSteps : 1];
    float probe = 0.f;
    if constexpr (SPLIT) {
      SplitRange range;
#pragma unroll
      for (int s2 = 0; s2 < kSteps; ++s2) {
        const f32x4 lo = *reinterpret_cast<const f32x4*>(qrow + 16 * s2), hi = *reinterpret_cast<const f32x4*>(qrow + 16 * s2 + 8);
        qs[s2] = split8(lo, hi);
        range.add(lo);
        range.add(hi);
      }
      if (range.outside()) probe = __builtin_nanf("");
    } else {
#pragma unroll
      for (int ch = 0; ch < kChunks; ++ch) qf[ch] = *reinterpret_cast<const f32x4*>(qrow + 8 * ch);
    }
    int J = kw, key = kw * a.block_k;  // block and first key of the tile to come
    if constexpr (SPLIT) {
      KTileF32<D>::copy(ks, key, ktile, lane);
    } else {
      const uint32_t off = ks.k_offset(key, lane);
#pragma unroll
      for (int ch = 0; ch < kChunks; ++ch) kf[ch] = ks.k_chunk(off, ch);
    }
    for (int seg = 0; seg < nkb; seg += kSeg) {
      const int seg_end = seg + kSeg < nkb ? seg + kSeg : nkb;
      float acc = 0.f;  // this lane's share of block J
      while (J < seg_end) {
        const int left = (J + 1) * a.block_k < key_len ? (J + 1) * a.block_k - key : key_len - key;  // keys of the block from `key` on (>= 1)
        const bool last = left <= kTileKF;                                                           // last tile of its block
        const int key_next = last ? (J + KW) * a.block_k : key + kTileKF;  // (past the last block: rows that read as zeros)
        f32x16 s;
#pragma unroll
        for (int x = 0; x < 16; ++x) s[x] = 0.f;
        if constexpr (SPLIT) {
          vector_memory_done_but_f<0>();  // the tile is there
          auto chunk = [&](int ch) -> f32x4 { return KTileF32<D>::chunk(ktile, ch, lane); };
          Split8 now = split8(chunk(0), chunk(1));
          f32x4 lo = chunk(2), hi = chunk(3);
#pragma unroll
          for (int s2 = 0; s2 < kSteps; ++s2) {
            Split8 next;
            if (s2 + 1 < kSteps) next = split8(lo, hi);
            if (s2 + 2 < kSteps) {
              lo = chunk(2 * s2 + 4);
              hi = chunk(2 * s2 + 5);
            }
            s = mfma_split(now, qs[s2], s);
            if (s2 + 2 < kSteps) sched_split_interleave<2>();
            else if (s2 + 1 < kSteps) sched_split_interleave<0>();
            __builtin_amdgcn_sched_barrier(0);
            if (s2 + 1 < kSteps) now = next;
            if (s2 == kSteps - 2) {
              lds_reads_done_f();
              KTileF32<D>::copy(ks, key_next, ktile, lane);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        } else {
          const uint32_t off_next = ks.k_offset(key_next, lane);
#pragma unroll
          for (int ch = 0; ch < kChunks; ++ch) {
#pragma unroll
            for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[ch][e], qf[ch][e], s, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);  // the reload stays behind its fragment's last use, so it can take its registers
            kf[ch] = ks.k_chunk(off_next, ch);
          }
        }
        if (left < kTileKF) {
#pragma unroll
          for (int x = 0; x < 16; ++x)
            if (8 * (x / 4) + 4 * g + (x % 4) >= left) s[x] = -__builtin_inff();
        }
        float least = 0.f, part = 0.f;
#pragma unroll
        for (int x = 0; x < 16; ++x) {
          s[x] = __builtin_fmaf(s[x], c, -lse2);
          least = fminf(least, s[x]);
        }
        if (__builtin_amdgcn_ballot_w64(least < -126.f) == 0) {
#pragma unroll
          for (int x = 0; x < 16; ++x) part += __builtin_amdgcn_exp2f(s[x]);
        } else {  // masked keys, or probabilities that the instruction alone would give as zero
#pragma unroll
          for (int x = 0; x < 16; ++x) part += exp2f(s[x]);
        }
        acc += part;
        key = key_next;
        if (last) {
          if (SPLIT) probe = __builtin_fmaf(acc, 0.f, probe);
          acc = wave_sum_f(acc);
          if (lane == 0) sums[rw][J - seg] = acc;
          acc = 0.f;
          J += KW;
        }
      }
      __syncthreads();
      for (int x = tid; x < seg_end - seg; x += 512) {
        float tot = 0.f;
#pragma unroll
        for (int w = 0; w < RW; ++w) tot += sums[w][x];
        const int first = (seg + x) * a.block_k;
        const int keys_here = key_len - first < a.block_k ? key_len - first : a.block_k;
        arow[seg + x] = tot * (1.0f / (float)(rows_here * keys_here));  // mean over the entries that exist
      }
      __syncthreads();  // the sums may be overwritten
    }
    vector_memory_done_but_f<0>();  // the last copy into LDS, of a tile past the range, has landed
    return probe != probe;
  };
  if (__builtin_expect(__syncthreads_or(walk(std::true_type{})), 0)) walk(std::false_type{});
}

// ---------------------------------------------------------------------------- per-row top-k
template <int R>
__global__ __launch_bounds__(64) void topk_kernel(const TopkArgs a) {
  extern __shared__ uint32_t lds[];  // the row (R = 0), then the kept entries of a row with a straddling boundary block
  const int lane = threadIdx.x;
  TopkRow<R> row;
  row.lds = lds;
  row.lane = lane;
  const int r = blockIdx.x;
  if (r >= a.rows) return;
  const int bh = r / a.nqb, I = r % a.nqb;
  const uint32_t* src = reinterpret_cast<const uint32_t*>(a.apool) + (int64_t)r * a.nkb;
  const int keep = a.keep_lo + a.keep_hi;
  auto kept = [&](int nblocks) -> int { return kept_blocks_of(a.rho, nblocks); };
  if (a.straddle >= 0) {
    // Prefill boundary at key token a.boundary, inside key block a.straddle. A row is one entry shorter where both of its
    // ranges keep that block, so its place depends on the rows before it. Either the wave works out which of those are
    // short (rows_tmp null, see places_rows_itself), or the rows are staged at a fixed stride (the host's keep_lo + keep_hi)
    // with their lengths and compact_kernel builds the CSR.
    int L = a.L;  // length of this batch element
    if (a.seq_lens != nullptr) {
      const int len = a.seq_lens[bh / a.heads_per_batch];
      L = len < a.L ? len : a.L;
    }
    const int nkb_b = L > 0 ? (L + a.block_k - 1) / a.block_k : 0, nqb_b = L > 0 ? (L + a.block_q - 1) / a.block_q : 0;
    // The ranked row has nkb_b + 1 entries: blocks before the one that holds the boundary, that block's
    // prefill part, its generation part, the blocks after it. Entries [0, Js] are the prefill range.
    // A sample no longer than the prefill has one range over the key blocks it has, none of them split.
    const int Js = a.straddle, nv = nkb_b + 1;
    const bool one_range = L <= a.boundary;
    const int keep_lo = kept(one_range ? nkb_b : Js + 1), keep_hi = one_range ? 0 : kept(nkb_b - Js), keep_b = keep_lo + keep_hi;
    const uint32_t* part = reinterpret_cast<const uint32_t*>(a.part) + (int64_t)r * 2;
    int32_t* tmp = nullptr;
    int begin = 0;
    auto finish = [&](int n) {  // the row has n entries
      if (lane != 0) return;
      if (R == 0 || R > 4 || a.rows_tmp != nullptr) {
        a.counts[r] = n;
        return;
      }
      int32_t* rp = a.row_ptr + (int64_t)bh * (a.nqb + 1);
      rp[I] = begin;
      if (I == a.nqb - 1) rp[a.nqb] = begin + n;
    };
    if (R == 0 || R > 4 || a.rows_tmp != nullptr) {
      tmp = a.rows_tmp + (int64_t)r * keep;
    } else {
      // A lane per earlier row (at most 64): both parts of its boundary block are kept if, in their range, fewer entries than
      // it keeps rank before them. The first part is the last of its range, so equal entries rank before it; the second
      // part is the first of its.
      const int earlier = I < nqb_b ? I : nqb_b;
      int before_lo = 0, before_hi = 0;
      if (!one_range && lane < earlier) {
        const uint32_t* mine = src + (int64_t)(lane - I) * a.nkb;
        const uint32_t p_lo = part[2 * (lane - I)], p_hi = part[2 * (lane - I) + 1];
#pragma unroll 8
        for (int J = 0; J < Js; ++J) before_lo += mine[J] >= p_lo;
#pragma unroll 8
        for (int J = Js + 1; J < nkb_b; ++J) before_hi += mine[J] > p_hi;
      }
      const bool is_short = !one_range && lane < earlier && before_lo < keep_lo && before_hi < keep_hi;
      begin = earlier * keep_b - __builtin_popcountll(__ballot(is_short));
      tmp = a.col_idx + (int64_t)bh * a.cap_per_head + begin;
    }
    if (I >= nqb_b) {  // a query block this sample does not have: an empty row
      finish(0);
      return;
    }
    if (one_range) {
      row.load(nkb_b, [&](int J) { return src[J]; });
      row.emit(0, nkb_b, keep_b, tmp);
      finish(keep_b);
      return;
    }
    row.load(nv, [&](int v) { return v == Js ? part[0] : v == Js + 1 ? part[1] : src[v < Js ? v : v - 1]; });
    int32_t* sel = reinterpret_cast<int32_t*>(lds + (R > 0 ? 0 : nv));  // the kept entries of both ranges
    row.emit(0, Js + 1, keep_lo, sel);
    row.emit(Js + 1, nv, keep_hi, sel + keep_lo);
    __syncthreads();
    // entries -> key blocks; the only possible duplicate is the boundary block, at the junction of the two ranges
    const bool dup = keep_lo > 0 && keep_hi > 0 && sel[keep_lo - 1] == Js && sel[keep_lo] == Js + 1;
    for (int t = lane; t < keep_b; t += 64) {
      if (dup && t == keep_lo) continue;
      const int v = sel[t];
      tmp[t - ((dup && t > keep_lo) ? 1 : 0)] = v > Js ? v - 1 : v;
    }
    finish(keep_b - (dup ? 1 : 0));
    return;
  }
  if (a.seq_lens != nullptr) {
    // per-sample length: this sample ranks the key blocks it has and keeps its own "top rho%" of them
    const int len = a.seq_lens[bh / a.heads_per_batch];
    const int L = len < a.L ? len : a.L;
    const int nkb_b = L > 0 ? (L + a.block_k - 1) / a.block_k : 0, nqb_b = L > 0 ? (L + a.block_q - 1) / a.block_q : 0;
    // With a prefill / generation split (Eq. 5) the sample's two ranges are [0, split) and [split, nkb_b), the
    // first cut to the blocks the sample has; a sample no longer than the prefill has one range only.
    const int split_b = a.split < nkb_b ? a.split : nkb_b;
    const int keep_lo_b = kept(split_b), keep_hi_b = kept(nkb_b - split_b);
    const int keep_b = keep_lo_b + keep_hi_b;
    int32_t* rp = a.row_ptr + (int64_t)bh * (a.nqb + 1);
    if (I < nqb_b) {
      row.load(nkb_b, [&](int J) { return src[J]; });
      int32_t* out_b = a.col_idx + (int64_t)bh * a.cap_per_head + (int64_t)I * keep_b;
      row.emit(0, split_b, keep_lo_b, out_b);
      row.emit(split_b, nkb_b, keep_hi_b, out_b + keep_lo_b);
    }
    if (lane == 0) {
      rp[I] = (I < nqb_b ? I : nqb_b) * keep_b;  // query blocks the sample does not have get empty rows
      if (I == a.nqb - 1) rp[a.nqb] = nqb_b * keep_b;
    }
    return;
  }
  row.load(a.nkb, [&](int J) { return src[J]; });
  int32_t* out = a.col_idx + (int64_t)bh * a.cap_per_head + (int64_t)I * keep;
  row.emit(0, a.split, a.keep_lo, out);
  row.emit(a.split, a.nkb, a.keep_hi, out + a.keep_lo);
  if (lane == 0) {
    int32_t* rp = a.row_ptr + (int64_t)bh * (a.nqb + 1);
    rp[I] = I * keep;
    if (I == a.nqb - 1) rp[a.nqb] = a.nqb * keep;
  }
}

// Exclusive scan over the 256 threads of a work-group (each brings the sum of its own consecutive rows): returns
// this thread's offset, leaves the grand total in partial[255].
__device__ __forceinline__ int scan_256(int sum, int32_t (&partial)[256], int tid) {
  partial[tid] = sum;
  __syncthreads();
  for (int off = 1; off < 256; off <<= 1) {
    const int add = tid >= off ? partial[tid - off] : 0;
    __syncthreads();
    partial[tid] += add;
    __syncthreads();
  }
  return partial[tid] - sum;
}

// One work-group per head: exclusive scan of the row lengths into row_ptr, then the waves copy the rows to their
// places, a wave per row and a lane per entry.
__global__ __launch_bounds__(256) void compact_kernel(const CompactArgs a) {
  __shared__ int32_t partial[256];
  const int head = blockIdx.x, tid = threadIdx.x;
  const int per = (a.nqb + 255) / 256;  // consecutive rows per thread
  const int first = tid * per, last = first + per < a.nqb ? first + per : a.nqb;
  const int32_t* counts = a.counts + (int64_t)head * a.nqb;
  int sum = 0;
  for (int I = first; I < last; ++I) sum += counts[I];
  int offset = scan_256(sum, partial, tid);
  int32_t* rp = a.row_ptr + (int64_t)head * (a.nqb + 1);
  int32_t* ci = a.col_idx + (int64_t)head * a.cap_per_head;
  for (int I = first; I < last; ++I) {
    rp[I] = offset;
    offset += counts[I];
  }
  if (tid == 255) rp[a.nqb] = partial[255];
  __syncthreads();  // the row pointer written above is visible to the whole work-group
  const int wave = tid >> 6, lane = tid & 63;
  for (int I = wave; I < a.nqb; I += 4) {
    const int beg = rp[I], n = rp[I + 1] - beg;
    const int32_t* src = a.rows_tmp + ((int64_t)head * a.nqb + I) * a.stride;
    for (int t = lane; t < n; t += 64) ci[beg + t] = src[t];
  }
}

// ---------------------------------------------------------------------------- index validation
__global__ __launch_bounds__(256) void validate_kernel(const ValidateArgs a) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= a.rows) return;
  const int bh = r / a.nqb, I = r % a.nqb;
  const int32_t* rp = a.row_ptr + (int64_t)bh * (a.nqb + 1);
  const int32_t beg = rp[I], end = rp[I + 1];
  bool ok = (beg >= 0) && (end >= beg) && (end <= a.cap_per_head) && (I != 0 || beg == 0);
  if (ok) {
    const int32_t* ci = a.col_idx + (int64_t)bh * a.cap_per_head;
    int32_t prev = -1;
    for (int t = beg; t < end; ++t) {
      const int32_t J = ci[t];
      if (J <= prev || J >= a.nkb) ok = false;
      prev = J;
    }
  }
  if (!ok) atomicAdd(a.bad, 1);
}

// ---------------------------------------------------------------------------- fixed patterns
// Sliding window plus attention sinks as a block index (the fixed patterns the paper compares
// against, Section 4.1): query block I keeps the leading `sink_blocks` key blocks and every key
// block that holds a key within `half_window` tokens of one of its queries. One work-group per head: row lengths
// scanned into the row pointer, then a wave per row.
__global__ __launch_bounds__(256) void window_index_kernel(const WindowArgs a) {
  __shared__ int32_t partial[256];
  const int bh = blockIdx.x, tid = threadIdx.x;
  const int per = (a.nqb + 255) / 256;  // consecutive rows per thread
  const int first_row = tid * per, last_row = first_row + per < a.nqb ? first_row + per : a.nqb;
  int sum = 0;
  for (int I = first_row; I < last_row; ++I) sum += window_row_length(I, a.block_q, a.block_k, a.L, a.half_window, a.sink_blocks);
  int offset = scan_256(sum, partial, tid);
  int32_t* rp = a.row_ptr + (int64_t)bh * (a.nqb + 1);
  int32_t* ci = a.col_idx + (int64_t)bh * a.cap_per_head;
  for (int I = first_row; I < last_row; ++I) {
    rp[I] = offset;
    offset += window_row_length(I, a.block_q, a.block_k, a.L, a.half_window, a.sink_blocks);
  }
  if (tid == 255) rp[a.nqb] = partial[255];
  __syncthreads();  // the row pointer written above is visible to the whole work-group
  const int wave = tid >> 6, lane = tid & 63;
  for (int I = wave; I < a.nqb; I += 4) {  // a wave per row, a lane per entry: the sinks, then the window
    int sink_end, first, last;
    window_row_runs(I, a.block_q, a.block_k, a.L, a.half_window, a.sink_blocks, &sink_end, &first, &last);
    int32_t* dst = ci + rp[I];
    for (int J = lane; J < sink_end; J += 64) dst[J] = J;
    for (int J = first + lane; J <= last; J += 64) dst[sink_end + J - first] = J;
  }
}

// ---------------------------------------------------------------------------- launchers
// Tokens per segment where there are too few query rows to fill the chip: the key range is cut into segments, four tiles or
// more each (0: one segment), whose scores are independent given the row statistics. What a launch takes, in hundredths of a
// microsecond, is a fixed part and a part per tile of a segment, by the work-groups of the busiest compute unit, one to four
// (fitted to 2300 calls with and without segments, to 5 %); the number of segments is the one that takes least. Pooling and top-k,
// us: 4 heads of 2048 x 128 27 -> 14.7 (7 segments), of 600 x 64 13.7 -> 10.0 (2); where the units nearly fill the chip, segments
// pay by the work-groups they leave on the busiest unit: 300 units of 2000 tokens 0.82 (head dim 64), 0.92 (128) of the time, 450
// units of 1000 tokens, head dim 128, 1.09, and are left whole.
static int pool_segment(int D, int64_t groups, int key_len, int block_k) {
  constexpr int kCus = 256, kLeast = 4 * kTileK;
  struct Line {
    int fixed, per_tile;
  };
  static constexpr Line kLines[2][2][4] = {  // [head dim 128][key blocks of 32]
      {{{740, 49}, {810, 74}, {830, 105}, {860, 138}}, {{730, 69}, {790, 92}, {860, 124}, {840, 163}}},
      {{{770, 57}, {840, 98}, {990, 153}, {1120, 199}}, {{770, 74}, {880, 110}, {900, 172}, {1180, 213}}}};
  auto cost = [&](int64_t parts, int len) -> int64_t {
    const int64_t k = (groups * parts - 1) / kCus;
    if (k > 3) return INT64_MAX;
    const Line& c = kLines[D == 128][block_k == 32][k];
    return c.fixed + (int64_t)c.per_tile * ((len + kTileK - 1) / kTileK);
  };
  if (groups > 2 * kCus) return 0;
  int64_t least = cost(1, key_len);
  int best = 0;
  for (int parts = 2; parts <= 4 * kCus / groups && key_len > kLeast; ++parts) {
    int len = (key_len + parts - 1) / parts;
    len = (len + 127) / 128 * 128;  // a multiple of every block_k
    if (len < kLeast) break;
    const int64_t c = cost((key_len + len - 1) / len, len);
    if (c * 100 < least * 99) least = c, best = len;
  }
  return best;
}

template <int D>
static hipError_t launch_pool_bf16_d(int block_q, PoolArgs a, hipStream_t s) {
  // every work-group is four waves = 128 consecutive rows of a head: one, two or four query blocks
  if (block_q != 128 && block_q != 64 && block_q != 32) return hipErrorInvalidValue;
  const int blocks_per_group = 128 / block_q;
  const int64_t total = (int64_t)a.B * a.Hq * ((a.nqb + blocks_per_group - 1) / blocks_per_group);
  if (total <= 0 || total > 0x7fffffff) return hipErrorInvalidValue;
  a.seg_len = a.key_len2 > 0 ? 0 : pool_segment(D, total, a.key_len, a.block_k);
  const dim3 grid((unsigned)total, a.key_len2 > 0 ? 2 : a.seg_len > 0 ? (a.key_len + a.seg_len - 1) / a.seg_len : 1), block(256);
  switch (block_q) {
    case 128:
      if (a.block_k == 32) hipLaunchKernelGGL((pool_bf16_kernel<D, 4, true, 4>), grid, block, 0, s, a);
      else hipLaunchKernelGGL((pool_bf16_kernel<D, 4, false, 4>), grid, block, 0, s, a);
      break;
    case 64:
      if (a.block_k == 32) hipLaunchKernelGGL((pool_bf16_kernel<D, 4, true, 2>), grid, block, 0, s, a);
      else hipLaunchKernelGGL((pool_bf16_kernel<D, 4, false, 2>), grid, block, 0, s, a);
      break;
    case 32:
      if (a.block_k == 32) hipLaunchKernelGGL((pool_bf16_kernel<D, 4, true, 1>), grid, block, 0, s, a);
      else hipLaunchKernelGGL((pool_bf16_kernel<D, 4, false, 1>), grid, block, 0, s, a);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_pool_bf16(int D, int block_q, const PoolArgs& a, hipStream_t s) {
  if (D == 128) return launch_pool_bf16_d<128>(block_q, a, s);
  if (D == 64) return launch_pool_bf16_d<64>(block_q, a, s);
  return hipErrorInvalidValue;
}

template <int D>
static hipError_t launch_pool_f32_d(int block_q, const PoolArgs& a, hipStream_t s) {
  const int64_t total = (int64_t)a.B * a.Hq * a.nqb;
  if (total <= 0 || total > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid((unsigned)total, a.key_len2 > 0 ? 2 : 1);
  switch (block_q) {
    case 128: hipLaunchKernelGGL((pool_f32_kernel<D, 4>), grid, dim3(512), 0, s, a); break;
    case 64: hipLaunchKernelGGL((pool_f32_kernel<D, 2>), grid, dim3(512), 0, s, a); break;
    case 32: hipLaunchKernelGGL((pool_f32_kernel<D, 1>), grid, dim3(512), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_pool_f32(int D, int block_q, const PoolArgs& a, hipStream_t s) {
  if (D == 128) return launch_pool_f32_d<128>(block_q, a, s);
  if (D == 64) return launch_pool_f32_d<64>(block_q, a, s);
  return hipErrorInvalidValue;
}

// A lane per earlier row: up to 64 rows a head; rows in at most four registers a lane. A wave then reads the scores of all the
// rows before its own, which is quicker than a second launch everywhere here. Whole selection (statistics given) with head dim
// 64, us, staged and compacted -> placed: 4 heads of 64 rows x 64 blocks 39.7 -> 32.3, 64 x 128 78.1 -> 70.0, 4 x 4 20.0 -> 17.3;
// 32 heads 48 x 192 268 -> 262, 64 x 128 140.0 -> 138.4 (64-row blocks) and 402.5 -> 402.4 (128-row blocks).
bool places_rows_itself(int nqb, int nkb) { return nqb <= 64 && nkb < 256; }

hipError_t launch_topk(const TopkArgs& a, hipStream_t s) {
  if (a.rows <= 0) return hipErrorInvalidValue;
  const int entries = a.nkb + (a.straddle >= 0 ? 1 : 0);                 // ranked entries of a row
  const int sel = a.straddle >= 0 ? a.keep_lo + a.keep_hi : 0;           // kept entries staged in LDS
  const dim3 grid((unsigned)a.rows), block(64);
  if (entries <= 64) hipLaunchKernelGGL(topk_kernel<1>, grid, block, sel * sizeof(uint32_t), s, a);
  else if (entries <= 128) hipLaunchKernelGGL(topk_kernel<2>, grid, block, sel * sizeof(uint32_t), s, a);
  else if (entries <= 256) hipLaunchKernelGGL(topk_kernel<4>, grid, block, sel * sizeof(uint32_t), s, a);
  else if (entries <= 512) hipLaunchKernelGGL(topk_kernel<8>, grid, block, sel * sizeof(uint32_t), s, a);
  else if (entries <= 1024) hipLaunchKernelGGL(topk_kernel<16>, grid, block, sel * sizeof(uint32_t), s, a);
  else hipLaunchKernelGGL(topk_kernel<0>, grid, block, (entries + sel) * sizeof(uint32_t), s, a);
  return hipGetLastError();
}

hipError_t launch_window_index(const WindowArgs& a, hipStream_t s) {
  if (a.heads <= 0 || a.nqb <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(window_index_kernel, dim3((unsigned)a.heads), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_compact(const CompactArgs& a, hipStream_t s) {
  if (a.heads <= 0 || a.nqb <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(compact_kernel, dim3((unsigned)a.heads), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_validate(const ValidateArgs& a, hipStream_t s) {
  if (a.rows <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(validate_kernel, dim3((unsigned)((a.rows + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace sparsed
