// fp32 flash-attention forward for gfx950: dense (Eq. 1), block-sparse (Eq. 3 / Eq. 4) and the
// statistics-only pass. fp32 inputs, fp32 softmax, fp32 output; products on the bf16 matrix instruction with operands split in
// three (tile_f32.hpp), or on the fp32 one (32x32x2): where the parts would not do, and for lists that one wave walks.
// This is the path held to 1e-5 against the fp64 reference.
//
// One work-group owns 32 query rows of one (batch, head); its KW waves share the rows and split the keys: wave w takes
// the 32-key tiles w, w + KW, ... of the list with its own reference, sum and output accumulator, and the parts
// are merged once, through LDS, at the end. The waves need nothing from each other in between (tile_f32.hpp), so the tile
// loop has no barrier, and a short sequence still spreads over many waves. The next tile is requested as soon as what it
// replaces has been used: every load has most of a tile's work to arrive.
//
// Bound: the vector unit, which splits every K and V value into its three bf16 parts for 32 rows of queries (700 of the 890
// vector instructions of a tile at head dim 128, 2 ns each), and the matrix cores (96 instructions of 16 ns), which hardly
// overlap: 60 % and 42 % busy in a dense call of 8 heads of 2000 x 128; then what a work-group spends before its first and after
// its last tile. 8 heads of 2000 x 128: dense 164 -> 111 us, sparse (64 x 64 blocks, 20 % kept) 48 -> 37 us, pooling (select.hip)
// 84 -> 61 us; 2 heads of 256 x 64: dense 11.5 -> 9.4 us. (Before: the fp32 matrix instruction alone. Of these times 1 to 3 %
// are the looks at values that three parts do not hold, see tile_f32.hpp.) Error against 64 bits, largest of an output over its
// root mean square, random inputs of both: 8 x 2000 x 128 3.2e-6 -> 2.7e-6, 4 x 600 x 64 1.5e-6 -> 1.2e-6, peaked rows (logits of
// variance 16) 2.1e-5 -> 1.7e-5, log-normal inputs (sigma 1.5 and 3) 3.5e-4 -> 9.0e-5; log-sum-exp 8.7e-6 -> 8.1e-6 where rows are
// peaked, the same elsewhere.
#include <type_traits>

#include "kernels.hpp"
#include "tile_f32.hpp"
#include "topk_row.hpp"

namespace sparsed {

// Pooling (kDensePool). The step at which the pattern is selected needs A'[I, J], the mean of the probabilities over query block
// I and key block J, beside the attention output, and the tile loop already forms the sums of a row's probabilities. A
// work-group is then a query block, RW = block_q / 32 row groups times KW = 8 / RW key groups; a wave takes whole key
// blocks and parks, per row and block, the sum and the reference it is relative to in LDS. When the rows are complete, the
// parts' references and sums are known to all, and the work-group weighs and adds up its parked sums. Against the dense call
// and a pooling kernel that computes every logit again (short fp32 schedules, switch step and top-k): 8 heads of 2000 x 128,
// 64 x 64 blocks 174 -> 121 us; 2 of 256 x 64, 32 x 32 blocks 18.1 -> 13.3 us.
template <int D, int RW>
struct PoolLdsF32 {
  static constexpr int kBytes = 157 * 1024;  // a compute unit's, less the statistics
  static constexpr int kUsed = RW * (D / 16) * 3 * 64 * 16 + (D == 64 ? 8 * KTileF32<D>::kBytes : 0);  // queries, K tiles
  static constexpr int kBlocks = (kBytes - kUsed) / (RW * 32 * 8);                                       // key blocks that can be parked
};

// RANKS (kDensePool): the work-group also ranks the row it has pooled and writes its part of the index (ranks_own_rows_f32).
template <int D, int KW, Mode MODE, bool SPLIT_FIRST, int RW = 1, bool RANKS = false>
__global__ __launch_bounds__(RW * KW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_f32_kernel(const AttnArgs a) {
  constexpr bool kPool = MODE == Mode::kDensePool;
  static_assert(!RANKS || kPool, "the rows ranked are the pooled ones");
  static_assert(RW == 1 || kPool, "several row groups: only where a work-group is a query block");
  constexpr int NW = RW * KW, NT = NW * 64;
  constexpr bool kHasV = MODE != Mode::kStats;
  constexpr int kChunks = D / 8, kSteps = D / 16, kV = D / 32;
  using VRow = typename SlabF32<D>::VRow;
  // K through LDS (tile_f32.hpp), or straight into registers as V. Through LDS at head dim 64, where two waves per SIMD find
  // room for their tiles beside another work-group's (2 heads of 256, dense: 10.2 us straight, 9.3 through LDS); at 128 a
  // work-group of eight waves would fill the LDS, and nothing is left to run while it begins and ends (8 heads of 2000, dense:
  // 115 us, straight 110).
  constexpr bool KLDS = SPLIT_FIRST && D == 64;
  // The query fragments ([row group][step][part][lane], 16 bytes each), the waves' K tiles, the parked sums ([block][row], sum
  // and reference) and, once the keys are done, the waves' accumulators ([wave][row][32 pieces of D/32 columns], piece i of
  // row j at position i ^ j so that neither side has bank conflicts).
  constexpr int kQBytes = SPLIT_FIRST ? kSteps * 3 * 64 * 16 : kChunks * 64 * 16;  // of a row group
  constexpr int kKBytes = KLDS ? NW * KTileF32<D>::kBytes : 0, kAccBytes = kHasV ? NW * 32 * D * 4 : 16;
  constexpr int kTileBytes = RW * kQBytes + kKBytes > kAccBytes ? RW * kQBytes + kKBytes : kAccBytes;
  __shared__ __attribute__((aligned(1024))) char lds[kPool ? PoolLdsF32<D, RW>::kBytes : kTileBytes];
  static_assert(!kPool || (kTileBytes <= PoolLdsF32<D, RW>::kBytes && RW * kQBytes + kKBytes == PoolLdsF32<D, RW>::kUsed), "layout");
  f32x2f* const parked = reinterpret_cast<f32x2f*>(lds + (kPool ? PoolLdsF32<D, RW>::kUsed : 0));
  __shared__ float stat_m[NW][32], stat_l[NW][32];
  __shared__ int verdicts[SPLIT_FIRST ? NW : 1];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rw = RW == 1 ? 0 : wave % RW, kw = RW == 1 ? wave : wave / RW;  // row group and key group of this wave
  const int j = lane & 31, g = lane >> 5;

  const int lid = xcd_remap_f(blockIdx.x, gridDim.x);
  const int qt = lid % a.n_qtiles;
  const Slab slab_of = slab_at(lid / a.n_qtiles, a);
  const int b = slab_of.b, h = slab_of.h, hk = slab_of.hk, bh = b * a.Hq + h;
  int L = a.L;  // length of this batch element
  if (a.seq_lens != nullptr) {
    const int len = a.seq_lens[b];
    L = len < a.L ? len : a.L;
  }
  const int wg_row0 = qt * (32 * RW), row0 = wg_row0 + rw * 32;
  // RANKS: the place of row qt, every row of a sample keeping as many blocks
  auto place_row = [&](int keep) {
    const KernelArgs<AttnArgs>& ae = fresh_kernel_args<AttnArgs>();
    const int rows = L > 0 ? (L + 32 * RW - 1) / (32 * RW) : 0;  // query blocks of the sample; those behind them are empty
    if (tid != 0) return;
    int32_t* const rp = ae.row_ptr_out + (int64_t)bh * (ae.nqb + 1);
    rp[qt] = (qt < rows ? qt : rows) * keep;
    if (qt == ae.nqb - 1) rp[ae.nqb] = rows * keep;
  };
  if (wg_row0 >= L) {  // a query tile wholly past the end (uniform over the work-group)
    if (RANKS) place_row(L > 0 ? kept_blocks_of(a.rho, (L + a.block_k - 1) / a.block_k) : 0);
    return;
  }

  SlabF32<D> ks, vs;
  ks.init(static_cast<const float*>(a.k.ptr) + b * a.k.sb + hk * a.k.sh, a.k.sl, L);
  if (kHasV) vs.init(static_cast<const float*>(a.v.ptr) + b * a.v.sb + hk * a.v.sh, a.v.sl, L);

  // tiles of the list: every 32 keys (dense), or those of the listed key blocks
  const int tile_shift = (MODE == Mode::kSparse || kPool) ? (a.block_k == 128 ? 2 : a.block_k == 64 ? 1 : 0) : 0;
  int n;
  const int32_t* cols = nullptr;
  if (MODE == Mode::kSparse) {
    const int32_t* rp = a.row_ptr + (int64_t)bh * (a.nqb + 1) + row0 / a.block_q;
    const int beg = rp[0], end = rp[1];
    n = (end - beg) << tile_shift;
    cols = a.col_idx + (int64_t)bh * a.cap_per_head + beg;
  } else {
    n = (L + kTileKF - 1) / kTileKF;
  }
  int opaque_zero;  // keeps the list reads on the vector path: a scalar load would share its counter with the LDS reads
  asm volatile("v_mov_b32 %0, 0" : "=v"(opaque_zero));
  // kPool: a wave's tiles are those of the key blocks kw, kw + KW, ..., numbered kw, kw + KW, ... as if they were every KW-th
  // tile; a partial last block counts as a whole one (its last tiles may hold no key)
  const int nkb = kPool ? (n + (1 << tile_shift) - 1) >> tile_shift : 0;
  if (kPool) n = ((nkb - kw + KW - 1) / KW << tile_shift) * KW;  // (no tile: at most zero)
  auto first_key = [&](int t) -> int {  // of tile t of the list; past the end: of the last one (a harmless repeat)
    if (kPool) {
      const int i = (t < n ? t : n - 1) / KW;  // this wave's i-th tile
      return (((kw + (i >> tile_shift) * KW) << tile_shift) + (i & ((1 << tile_shift) - 1))) * kTileKF;
    }
    const int u = t < n ? t : n - 1;
    if (MODE != Mode::kSparse) return u * kTileKF;
    return cols[(u >> tile_shift) + opaque_zero] * a.block_k + (u & ((1 << tile_shift) - 1)) * kTileKF;
  };

  float M = -1e30f, lsum = 0.f;
  f32x16 o[kV];
  const float c = a.scale_log2;
  const float* const qhead = static_cast<const float*>(a.q.ptr) + b * a.q.sb + h * a.q.sh;

  char* const qlds = lds + rw * kQBytes;
  bool queries_outside = false;  // some query value of this wave's share (SplitRange)
  uint32_t v_top = 0;            // bits of the largest |V| of tiles with probabilities below 2^-108 (tile_f32.hpp)

  // The wave's share of the tile list. SPLIT: on the bf16 matrix instruction; else on the fp32 one.
  auto walk = [&](auto split_tag) __attribute__((always_inline)) {
    constexpr bool SPLIT = decltype(split_tag)::value;
    // query fragments into LDS: lane (j, g) of chunk ch holds columns 8 ch + 4g .. + 3 of row j
    {
      const int row = row0 + j < L ? row0 + j : L - 1;
      const float* qrow = qhead + (int64_t)row * a.q.sl + 4 * g;
      if constexpr (SPLIT) {
        SplitRange range;
        for (int s2 = kw; s2 < kSteps; s2 += KW) {
          const f32x4 lo = *reinterpret_cast<const f32x4*>(qrow + 16 * s2), hi = *reinterpret_cast<const f32x4*>(qrow + 16 * s2 + 8);
          const Split8 w = split8(lo, hi);
          range.add(lo);
          range.add(hi);
          u32x4f* const dst = reinterpret_cast<u32x4f*>(qlds) + s2 * 3 * 64 + lane;
          dst[0] = w.h;
          dst[64] = w.m;
          dst[128] = w.l;
        }
        queries_outside = __builtin_amdgcn_ballot_w64(range.outside()) != 0;
      } else {
        for (int ch = kw; ch < kChunks; ch += KW)
          *reinterpret_cast<f32x4*>(qlds + (ch * 64 + lane) * 16) = *reinterpret_cast<const f32x4*>(qrow + 8 * ch);
      }
    }
    M = -1e30f;
    lsum = 0.f;
#pragma unroll
    for (int dt = 0; dt < kV; ++dt)
#pragma unroll
      for (int x = 0; x < 16; ++x) o[dt][x] = 0.f;
    constexpr bool VIA_LDS = SPLIT && KLDS;
    char* const ktile = lds + (VIA_LDS ? RW * kQBytes + wave * KTileF32<D>::kBytes : 0);
    float block_sum = 0.f;  // kPool: this lane's share of the key block in progress
    f32x4 kf[VIA_LDS ? 1 : kChunks];
    VRow vf[16];

    int t = kw, key = 0, key_next = 0;
    if (t < n) {
      key = __builtin_amdgcn_readfirstlane(first_key(t));
      key_next = __builtin_amdgcn_readfirstlane(first_key(t + KW));
      const uint32_t off = ks.k_offset(key, lane), voff = kHasV ? vs.v_offset(key, lane) : 0;
      if constexpr (VIA_LDS) {
        KTileF32<D>::copy(ks, key, ktile, lane);
        __builtin_amdgcn_sched_barrier(0);
      } else {
#pragma unroll
        for (int ch = 0; ch < kChunks; ++ch) kf[ch] = ks.k_chunk(off, ch);
      }
      if (kHasV) {
#pragma unroll
        for (int x = 0; x < 16; ++x) vf[x] = vs.v_row(voff, x);
      }
    }
    __syncthreads();
    for (; t < n; t += KW) {
      const int key_after = first_key(t + 2 * KW);
      const uint32_t off_next = ks.k_offset(key_next, lane), voff_next = kHasV ? vs.v_offset(key_next, lane) : 0;
      f32x16 s;
#pragma unroll
      for (int x = 0; x < 16; ++x) s[x] = 0.f;
      if constexpr (SPLIT) {
        // A tile's copy is followed by the V rows of the same tile, whose loads may stay in flight.
        if constexpr (VIA_LDS) vector_memory_done_but_f<kHasV ? 16 : 0>();
        auto chunk = [&](int ch) -> f32x4 {
          if constexpr (VIA_LDS) return KTileF32<D>::chunk(ktile, ch, lane);
          else return kf[ch];
        };
        Split8 now = split8(chunk(0), chunk(1));
        f32x4 lo = chunk(2), hi = chunk(3);
        __builtin_amdgcn_sched_barrier(0);  // a reload stays behind its fragment's last use, so it can take its registers
#pragma unroll
        for (int s2 = 0; s2 < kSteps; ++s2) {
          if constexpr (!VIA_LDS) {
            kf[2 * s2] = ks.k_chunk(off_next, 2 * s2);
            kf[2 * s2 + 1] = ks.k_chunk(off_next, 2 * s2 + 1);
          }
          const u32x4f* const src = reinterpret_cast<const u32x4f*>(qlds) + s2 * 3 * 64 + lane;
          const Split8 qw = {src[0], src[64], src[128]};
          Split8 next;
          if (s2 + 1 < kSteps) next = split8(lo, hi);
          if (s2 + 2 < kSteps) {
            lo = chunk(2 * s2 + 4);
            hi = chunk(2 * s2 + 5);
          }
          s = mfma_split(now, qw, s);
          if (s2 + 2 < kSteps) sched_split_interleave<VIA_LDS ? 5 : 3>();
          else if (s2 + 1 < kSteps) sched_split_interleave<3>();
          __builtin_amdgcn_sched_barrier(0);
          if (s2 + 1 < kSteps) now = next;
          if (VIA_LDS && s2 == kSteps - 2) {
            lds_reads_done_f();
            KTileF32<D>::copy(ks, key_next, ktile, lane);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      } else {
#pragma unroll
        for (int ch = 0; ch < kChunks; ++ch) {
          const f32x4 qf = *reinterpret_cast<const f32x4*>(qlds + (ch * 64 + lane) * 16);
#pragma unroll
          for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[ch][e], qf[e], s, 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          kf[ch] = ks.k_chunk(off_next, ch);
        }
      }
      // this lane's least logit, of keys that do not exist as well (rows that mostly read as zeros)
      float least = fminf(s[0], s[1]);
      if (kHasV) {
#pragma unroll
        for (int x = 2; x < 16; x += 2) least = fminf(fminf(least, s[x]), s[x + 1]);
      }
      // keys of this tile that exist: fewer than 32 at the end of a sequence whose length is not a multiple of the tile,
      // none in the later tiles of a partial last key block
      const int valid = L - key;
      if (valid < kTileKF) {
#pragma unroll
        for (int x = 0; x < 16; ++x)
          if (8 * (x / 4) + 4 * g + (x % 4) >= valid) {
            s[x] = -__builtin_inff();
            // (a row past the end mostly reads as zeros, but where rows are 16 MB and more apart its offset wraps)
            if (kHasV) vf[x] = VRow{};
          }
      }
      // The row's reference M stays within an octave of its maximum: probabilities stay at or below 2, and the output is
      // rescaled for the few tiles that raise a row's maximum by more.
      float mx = fmaxf(s[0], s[1]);
#pragma unroll
      for (int x = 2; x < 16; x += 2) mx = fmaxf(fmaxf(mx, s[x]), s[x + 1]);
      mx = pair_max_f(mx) * c;
      if (__builtin_amdgcn_ballot_w64(mx > M + 1.0f) != 0) {
        const float Mn = fmaxf(M, mx);
        const float alpha = __builtin_amdgcn_exp2f(M - Mn);
        M = Mn;
        lsum *= alpha;
        if (kPool) block_sum *= alpha;
        if (kHasV) {
#pragma unroll
          for (int dt = 0; dt < kV; ++dt)
#pragma unroll
            for (int x = 0; x < 16; ++x) o[dt][x] *= alpha;
        }
      }
      float part = 0.f;
#pragma unroll
      for (int x = 0; x < 16; ++x) s[x] = __builtin_fmaf(s[x], c, -M);
      if (!kHasV || __builtin_expect(__builtin_amdgcn_ballot_w64(__builtin_fmaf(least, c, -M) < (SPLIT ? -108.f : -126.f)) == 0, 1)) {
#pragma unroll
        for (int x = 0; x < 16; ++x) s[x] = __builtin_amdgcn_exp2f(s[x]);
      } else {  // probabilities that the instruction alone would give as zero, or that three parts do not hold whole
#pragma unroll
        for (int x = 0; x < 16; ++x) s[x] = exp2f(s[x]);
        if constexpr (SPLIT && kHasV) {
          float top = 0.f;
#pragma unroll
          for (int x = 0; x < 16; ++x)
#pragma unroll
            for (int dt = 0; dt < kV; ++dt) top = fmaxf(top, fabsf(vf[x][dt]));
#pragma unroll
          for (int d = 32; d >= 1; d >>= 1) top = fmaxf(top, __shfl_xor(top, d, 64));
          const uint32_t bits = (uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(top));
          v_top = bits > v_top ? bits : v_top;
        }
      }
#pragma unroll
      for (int x = 0; x < 16; ++x) part += s[x];
      lsum += part;
      if (kPool) {
        block_sum += part;
        const int i = t / KW;
        if (((i + 1) & ((1 << tile_shift) - 1)) == 0) {  // the last tile of its block
          const float e = pair_sum_f(block_sum);
          const f32x2f v = {e, M};
          if (g == 0) parked[(kw + (i >> tile_shift) * KW) * (RW * 32) + rw * 32 + j] = v;
          block_sum = 0.f;
        }
      }
      if (kHasV) {
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (SPLIT) {
          Split8 p[2];
#pragma unroll
          for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i) p[m].pair(i, s[8 * m + 2 * i], s[8 * m + 2 * i + 1]);
          auto split_v = [&](int u) -> Split8 {  // u = m * kV + dt
            const int m = u / kV, dt = u % kV;
            Split8 w;
#pragma unroll
            for (int i = 0; i < 4; ++i) w.pair(i, vf[8 * m + 2 * i][dt], vf[8 * m + 2 * i + 1][dt]);
            return w;
          };
          Split8 now = split_v(0);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < 2 * kV; ++u) {
            Split8 next;
            if (u + 1 < 2 * kV) next = split_v(u + 1);
            o[u % kV] = mfma_split(now, p[u / kV], o[u % kV]);
            if (u + 1 < 2 * kV) sched_split_interleave<0>();
            __builtin_amdgcn_sched_barrier(0);
            if (u % kV == kV - 2 || kV == 1) {  // every column of these eight rows has been split
#pragma unroll
              for (int x = 0; x < 8; ++x) vf[u / kV * 8 + x] = vs.v_row(voff_next, u / kV * 8 + x);
            }
            if (u + 1 < 2 * kV) now = next;
          }
        } else {
#pragma unroll
          for (int x = 0; x < 16; ++x) {
#pragma unroll
            for (int dt = 0; dt < kV; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[x][dt], s[x], o[dt], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            vf[x] = vs.v_row(voff_next, x);
          }
        }
      }
      key = key_next;
      key_next = __builtin_amdgcn_readfirstlane(key_after);
    }
    vector_memory_done_but_f<0>();  // the last copy into LDS, of a tile past the list, has landed
  };
  auto leave_statistics = [&]() {
    const float ltot = pair_sum_f(lsum);
    if (g == 0) {
      stat_m[wave][j] = M;
      stat_l[wave][j] = ltot;
    }
  };
  if constexpr (!SPLIT_FIRST) {
    walk(std::false_type{});
    leave_statistics();
    __syncthreads();  // everyone is done with the query fragments
  } else {
    walk(std::true_type{});
    // Whether this wave's results may show what the parts do not carry (tile_f32.hpp).
    float least = __builtin_inff(), probe = 0.f * lsum;  // probe: not a number if any sum is infinite or not a number
    bool small = false;
    if (kHasV) {
#pragma unroll
      for (int dt = 0; dt < kV; ++dt)
#pragma unroll
        for (int x = 0; x < 16; ++x) {
          probe = __builtin_fmaf(o[dt][x], 0.f, probe);
          least = fminf(least, fabsf(o[dt][x]));
        }
      const float good = fmaxf(0x1p-90f, __uint_as_float(v_top) * 0x1p-92f);  // the least sum that is good
      small = least < good;
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(least == 0.f) != 0, 0)) {  // the least of those that are not zero
        float next = __builtin_inff();
#pragma unroll
        for (int dt = 0; dt < kV; ++dt)
#pragma unroll
          for (int x = 0; x < 16; ++x) next = fminf(next, o[dt][x] == 0.f ? __builtin_inff() : fabsf(o[dt][x]));
        small = next < good || (least == 0.f && good >= 0x1p-60f);
        // zeros are good where V is zero: its values again, for any that are small and not zero
        SplitRange range;
        for (int t = kw; t < n; t += KW) {
          const uint32_t off = vs.v_offset(__builtin_amdgcn_readfirstlane(first_key(t)), lane);
#pragma unroll 4
          for (int x = 0; x < 16; ++x) {
            const VRow w = vs.v_row(off, x);
#pragma unroll
            for (int dt = 0; dt < kV; ++dt) range.add_low(w[dt]);
          }
        }
        small |= range.below();
      }
    }
    int verdict = queries_outside || __builtin_amdgcn_ballot_w64(small || probe != probe) != 0 ? 1 : 0;
    if (lane == 0) verdicts[wave] = verdict;
    leave_statistics();
    __syncthreads();  // everyone is done with the query fragments
#pragma unroll
    for (int w = 0; w < NW; ++w) verdict |= verdicts[w];
    if (__builtin_expect(verdict, 0)) {
      walk(std::false_type{});
      leave_statistics();
      __syncthreads();
    }
  }

  // Merge the waves' parts: O = sum_w O_w 2^(M_w - M) / sum_w l_w 2^(M_w - M), M = max_w M_w.
  auto factors = [&](int group, int row, float (&f)[KW], float* m) -> float {  // every part's factor and the common maximum; returns l
    float mm = stat_m[group][row], l = 0.f;
#pragma unroll
    for (int w = 1; w < KW; ++w) mm = fmaxf(mm, stat_m[w * RW + group][row]);
#pragma unroll
    for (int w = 0; w < KW; ++w) {
      f[w] = exp2f(stat_m[w * RW + group][row] - mm);
      l += stat_l[w * RW + group][row] * f[w];
    }
    *m = mm;
    return l;
  };
  TopkRow<4> row;
  row.lane = lane;
  if constexpr (kPool) {
    // A'[I, J] = sum over the rows of E 2^(M_parked - M) / l, divided by the entries that exist. A wave takes a key block (two
    // with 32 rows) at a time, a lane one row of it, or two; the lanes are added up in a fixed order.
    constexpr int kRowsPerLane = RW == 4 ? 2 : 1;
    float ref[kRowsPerLane], weight[kRowsPerLane];
    int at[kRowsPerLane];
#pragma unroll
    for (int u = 0; u < kRowsPerLane; ++u) {
      at[u] = RW == 1 ? j : lane + 64 * u;
      float f[KW];
      const float l = factors(at[u] >> 5, at[u] & 31, f, &ref[u]);
      weight[u] = wg_row0 + at[u] < L ? 1.0f / l : 0.f;
    }
    const int rows_here = L - wg_row0 < 32 * RW ? L - wg_row0 : 32 * RW;
    float* const arow = a.apool + ((int64_t)bh * a.nqb + qt) * a.nkb;
    constexpr int kAtOnce = RW == 1 ? 2 : 1;
    for (int J0 = wave * kAtOnce; J0 < nkb; J0 += NW * kAtOnce) {
      const int J = J0 + (RW == 1 ? g : 0);
      float x = 0.f;
#pragma unroll
      for (int u = 0; u < kRowsPerLane; ++u) {
        const f32x2f v = parked[(J < nkb ? J : nkb - 1) * (RW * 32) + at[u]];
        x += v[0] * exp2f(v[1] - ref[u]) * weight[u];
      }
#pragma unroll
      for (int d = RW == 1 ? 16 : 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
      const int keys_here = L - J * a.block_k < a.block_k ? L - J * a.block_k : a.block_k;
      if ((RW == 1 ? j : lane) == 0 && J < nkb) {
        x *= 1.0f / (float)(rows_here * keys_here);
        arow[J] = x;
        if (RANKS) parked[J * (RW * 32)][0] = x;  // (this wave alone has read the block's sums)
      }
    }
    if (RANKS) {
      __syncthreads();
      if (wave == 0) row.load(nkb, [&](int J) { return __float_as_uint(parked[J * (RW * 32)][0]); });
    }
    __syncthreads();  // the accumulators may take the parked sums' place
  }
  if (kHasV) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      VRow w;
#pragma unroll
      for (int dt = 0; dt < kV; ++dt) w[dt] = o[dt][v];
      const int piece = 8 * (v / 4) + 4 * g + (v % 4);  // columns kV * piece .. + kV - 1 of row j
      *reinterpret_cast<VRow*>(lds + ((wave * 32 + j) * 32 + (piece ^ j)) * sizeof(VRow)) = w;
    }
  }
  __syncthreads();
  if (a.lse != nullptr && tid < 32 * RW && wg_row0 + tid < L) {
    float f[KW], m;
    const float l = factors(tid >> 5, tid & 31, f, &m);
    a.lse[(int64_t)bh * a.L + wg_row0 + tid] = (m + log2f(l)) * 0.6931471805599453f;
  }
  if (kHasV) {
    for (int id = tid; id < RW * 32 * 32; id += NT) {
      const int group = id >> 10, row = (id >> 5) & 31, piece = id & 31;
      if (wg_row0 + group * 32 + row >= L) break;  // partial last query tile (rows ascend with id)
      float f[KW], m;
      const float l = factors(group, row, f, &m);
      const float inv = l > 0.f ? 1.0f / l : 0.f;
      VRow acc;
#pragma unroll
      for (int dt = 0; dt < kV; ++dt) acc[dt] = 0.f;
#pragma unroll
      for (int w = 0; w < KW; ++w) {
        const VRow part = *reinterpret_cast<const VRow*>(lds + (((w * RW + group) * 32 + row) * 32 + (piece ^ row)) * sizeof(VRow));
#pragma unroll
        for (int dt = 0; dt < kV; ++dt) acc[dt] += part[dt] * f[w];
      }
#pragma unroll
      for (int dt = 0; dt < kV; ++dt) acc[dt] *= inv;
      float* orow = static_cast<float*>(a.o) + b * a.o_sb + h * a.o_sh + (int64_t)(wg_row0 + group * 32 + row) * a.o_sl;
      *reinterpret_cast<VRow*>(orow + kV * piece) = acc;
    }
  }
  if constexpr (RANKS) {
    // The row's kept blocks, from the scores in the first wave's registers.
    const KernelArgs<AttnArgs>& ae = fresh_kernel_args<AttnArgs>();
    if (wave == 0) {
      const int keep = kept_blocks_of(ae.rho, nkb);
      row.emit(0, nkb, keep, ae.col_idx_out + (int64_t)bh * ae.cap_per_head + (int64_t)qt * keep);
      place_row(keep);
    }
  }
}

template <int D, int KW, Mode MODE, bool SPLIT_FIRST = true>
static hipError_t launch_one_f32(const AttnArgs& a, hipStream_t s) {
  const int64_t total = (int64_t)a.B * a.Hq * a.n_qtiles;
  if (total <= 0 || total > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL((attn_f32_kernel<D, KW, MODE, SPLIT_FIRST>), dim3((unsigned)total), dim3(KW * 64), 0, s, a);
  return hipGetLastError();
}

// Waves per work-group, dense and statistics: a compute unit holds eight waves of this kernel, as two work-groups of four or
// one of eight. Eight where there are no more work-groups than compute units (short sequences: the keys split eight ways), else four.
template <int D, Mode MODE>
static hipError_t launch_by_fill_f32(const AttnArgs& a, hipStream_t s) {
  if ((int64_t)a.B * a.Hq * a.n_qtiles <= 256) return launch_one_f32<D, 8, MODE>(a, s);
  return launch_one_f32<D, 4, MODE>(a, s);
}

// Sparse: a short list does not feed four waves, and what a work-group spends around its tiles (splitting the queries,
// merging the waves) grows with its waves. Two waves of a SIMD share its matrix core in about the time of 1.6 that run alone,
// one after the other, so the time goes with the waves of the busiest SIMD (2 a pair, 1.25 for an odd one) times, in quarters of
// a tile on the fp32 instruction, 4 a tile and 17 for a wave alone with its list on that instruction (its queries need no
// splitting, and eight such work-groups fit a compute unit), 2 a step and 11 for one of two waves, 2 a step and 6 for one of
// four. The average list comes from the capacity, which is exact or an upper bound. Fitted to 362 calls (280 to 3008
// work-groups, 1 to 32 tiles, both head dims; the form chosen is 0.6 % from the best on average, 10 % at most): head dim 128, 2048
// work-groups, 1, 4, 16 tiles: alone 27.3, 51.5, 143 us; two 32.8, 53.5, 129; four 38.4, 55.2, 123; 400 work-groups of
// 16 tiles: 73, 45, 32.
template <int D>
static hipError_t launch_sparse_f32(const AttnArgs& a, hipStream_t s) {
  const int64_t groups = (int64_t)a.B * a.Hq * a.n_qtiles;
  if (groups <= 256) return launch_one_f32<D, 8, Mode::kSparse>(a, s);
  const int64_t tiles = ((int64_t)a.cap_per_head * (a.block_k / kTileKF) + a.nqb - 1) / a.nqb;
  auto busiest_simd = [](int64_t waves) -> int64_t {  // in quarters
    const int64_t n = (waves + 1023) / 1024;
    return n / 2 * 8 + n % 2 * 5;
  };
  const int64_t one = busiest_simd(groups) * (4 * tiles + 17), two = busiest_simd(2 * groups) * (2 * ((tiles + 1) / 2) + 11),
                four = busiest_simd(4 * groups) * (2 * ((tiles + 3) / 4) + 6);
  if (four <= one && four <= two) return launch_one_f32<D, 4, Mode::kSparse>(a, s);
  return two <= one ? launch_one_f32<D, 2, Mode::kSparse>(a, s) : launch_one_f32<D, 1, Mode::kSparse, false>(a, s);
}

template <int D, int RW>
static hipError_t launch_pool_rw_f32(const AttnArgs& a, hipStream_t s) {
  const int64_t total = (int64_t)a.B * a.Hq * a.n_qtiles;
  if (total <= 0 || total > 0x7fffffff || a.nkb > PoolLdsF32<D, RW>::kBlocks) return hipErrorInvalidValue;
  if constexpr (RW <= 2) {
    if (a.row_ptr_out != nullptr) {
      if (a.nkb > 256) return hipErrorInvalidValue;
      hipLaunchKernelGGL((attn_f32_kernel<D, 8 / RW, Mode::kDensePool, true, RW, true>), dim3((unsigned)total), dim3(512), 0, s, a);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((attn_f32_kernel<D, 8 / RW, Mode::kDensePool, true, RW>), dim3((unsigned)total), dim3(512), 0, s, a);
  return hipGetLastError();
}
template <int D>
static hipError_t launch_pool_d_f32(const AttnArgs& a, hipStream_t s) {
  switch (a.block_q) {
    case 32: return launch_pool_rw_f32<D, 1>(a, s);
    case 64: return launch_pool_rw_f32<D, 2>(a, s);
    case 128: return launch_pool_rw_f32<D, 4>(a, s);
    default: return hipErrorInvalidValue;
  }
}
hipError_t launch_attn_f32_dense_pool(int D, AttnArgs a, hipStream_t s) {
  if (a.L <= 0 || !a.apool || (a.block_k != 32 && a.block_k != 64 && a.block_k != 128)) return hipErrorInvalidValue;
  a.n_qtiles = a.nqb;  // a work-group is a query block
  if (D == 128) return launch_pool_d_f32<128>(a, s);
  if (D == 64) return launch_pool_d_f32<64>(a, s);
  return hipErrorInvalidValue;
}

template <int D>
static int parked_blocks_f32(int block_q) {
  return block_q == 32 ? PoolLdsF32<D, 1>::kBlocks : block_q == 64 ? PoolLdsF32<D, 2>::kBlocks : PoolLdsF32<D, 4>::kBlocks;
}
// Whether the kernel above takes a call: its sums must fit the LDS, and its coarser work-groups must cost less than computing the
// logits a second time. In tiles that a wave walks, times the rounds of the chip: FUSED here; DENSE in the dense call, whose
// waves split a query tile's keys four or eight ways whatever block_q; a pooling kernel walks as many tiles as this one, in half the
// time each. Of 152 calls (1 to 32 heads of 130 to 4000 tokens) none is slower for it by more than 1 %; where it is left, four
// heads of 600 x 128, 128 x 64 blocks, 56.2 us so and 64.3 in one kernel (10 tiles here, 3 there).
bool dense_pool_pays_f32(int D, int64_t heads, int L, int block_q, int block_k) {
  const int nkb = (L + block_k - 1) / block_k, rw = block_q / 32, kw = 8 / rw;
  if (nkb > (D == 128 ? parked_blocks_f32<128>(block_q) : parked_blocks_f32<64>(block_q))) return false;
  const int64_t tiles = (L + 31) / 32, groups = heads * ((L + block_q - 1) / block_q), dense_groups = heads * tiles;
  const int64_t fused = (int64_t)((nkb + kw - 1) / kw) * (block_k / 32) * ((groups + 255) / 256);
  const int64_t dense = dense_groups <= 256 ? (tiles + 7) / 8 : (tiles + 3) / 4 * ((dense_groups + 511) / 512);
  return fused <= 2 * dense + 1;
}

// One wave ranks while the rest of its compute unit, which holds one such work-group, waits: about as long as a launch takes, so
// it is for calls of one round of the chip. Switch step, us, launch of its own -> ranked here, (heads, tokens, head dim) and
// blocks: (2, 256, 64) 32 x 32 13.5 -> 12.8, (8, 100, 64) 32 x 32 11.4 -> 10.3, (28, 100, 128) 64 x 64 17.7 -> 16.4, (8, 2000, 128)
// 64 x 64 115.5 -> 114.3; with two rounds (28, 600, 64) 32 x 32 45.6 and 47.6; 128-row blocks 22.4 and 22.5, 103.3 and 106.4.
bool ranks_own_rows_f32(int64_t heads, int nqb, int nkb, int block_q) { return block_q <= 64 && heads * nqb <= 256 && nkb <= 256; }

hipError_t launch_attn_f32(Mode mode, int D, int block_q, AttnArgs a, hipStream_t s) {
  if (a.L <= 0 || (mode == Mode::kSparse && block_q % 32 != 0)) return hipErrorInvalidValue;
  a.block_q = block_q;
  a.n_qtiles = (a.L + 31) / 32;
  if (D == 128) {
    if (mode == Mode::kDense) return launch_by_fill_f32<128, Mode::kDense>(a, s);
    if (mode == Mode::kSparse) return launch_sparse_f32<128>(a, s);
    return launch_by_fill_f32<128, Mode::kStats>(a, s);
  }
  if (D == 64) {
    if (mode == Mode::kDense) return launch_by_fill_f32<64, Mode::kDense>(a, s);
    if (mode == Mode::kSparse) return launch_sparse_f32<64>(a, s);
    return launch_by_fill_f32<64, Mode::kStats>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace sparsed
