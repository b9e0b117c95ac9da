// bf16 attention with the keys split over the waves of a work-group: block-sparse (Eq. 3 / Eq. 4) for SMALL query blocks (32 or
// 64 rows), and dense (Eq. 1) and sparse calls with too few rows to fill the chip (the rule is at splitk_takes).
//
// The general kernel (attn_bf16_kernel.hpp) gives every wave 32 query rows and all the keys of a tile, so a
// 64-row query block is a work-group of two waves; its K/V double buffers fill the LDS of a compute
// unit after two such groups, which leaves one wave per SIMD and nothing to overlap a wave's softmax
// with. Here a query block gets twice the waves: wave (rw, kh) owns rows 32*rw .. 32*rw+31 and, of
// every 64-key tile, only the 32 keys of half kh. The two key halves of a row keep their own running
// maximum, sum and output accumulator (flash-decoding style) and are merged once, through LDS, at the
// end. Same LDS footprint per group, twice the waves per compute unit. With SG tile streams a row's keys are in 2 SG parts.
//
// Per tile step t a wave computes  S(t+1) = K(t+1)[half] Q^T  interleaved with the softmax of S(t),
// then  O += P(t) V(t)[half].  K(t+2) and V(t+1) are copied global -> LDS meanwhile; one barrier per tile.
// The last step or two (TAIL) copy and multiply nothing past the end of the list (the last barrier would wait for it, and
// a list of 13 tiles moved three tiles of 29 for nothing. 32 heads of 2000 x 128, 32 x 32 blocks, half kept: 76.5 -> 71.5 us);
// a partial last key block is masked in the last steps, the only ones that apply key counts.
// Query blocks of 32 rows (RW = 1) have two forms. Where the launch fills the chip, PRIVATE: a wave copies and reads its own key
// half only, so nothing is shared until the merge, and the tile loop has no barrier. One K and one V buffer (a wave refills its
// half as soon as its reads are done) instead of two of each put four query blocks on a compute unit, two waves per SIMD,
// where two blocks fitted: the second wave covers what the shorter lead of the copies leaves open. 32 heads of 2000 x 128,
// 32 x 32 blocks, half kept: 71.5 -> 60.9 us (469 -> 551 TFLOP/s). With no second wave there the lead is what counts, and the
// double buffers are the better form (the rule is at launch_splitk_d).
// Listed blocks of 128 keys are walked as two tiles, listed blocks of 32 keys are paired up two to a tile
// (see the notes at `tile_shift` / `half_blocks` below).
#include "kernels.hpp"
#include "tile_bf16.hpp"

namespace sparsed {

// KB: keys per listed block (32, 64 or 128), a compile-time choice so that the common 64 pays nothing for the others.
// PRIVATE: the barrier-free form (RW = 1). SG: tile streams; stream sg walks the tiles sg, sg + SG, ... with 2 RW waves and
// buffers of its own. LIST: sparse (the listed blocks), else dense (every tile).
template <int D, int RW, int KB, bool PRIVATE, int SG, bool LIST>
__global__ __launch_bounds__(RW * SG * 128)
    __attribute__((amdgpu_waves_per_eu(RW * SG == 1 && !PRIVATE ? 1 : 2, RW * SG == 1 && !PRIVATE ? 1 : 2))) void attn_bf16_splitk_kernel(const AttnArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass only needs the launch stub (the body uses device-only types)
  static_assert(LIST || KB == kTileK, "dense walks 64-key tiles");
  constexpr int NW = 2 * RW, NT = NW * 64, QT = 32 * RW;  // waves and threads of a stream
  constexpr int KW = 2 * SG;                              // parts that the keys of a row are split into
  constexpr int kKBytes = KLayout<D>::kTileBytes, kVBytes = VLayout<D>::kTileBytes;
  constexpr float kOverflow = 1.152921504606847e18f;  // 2^60: a 16-key partial sum at or above this re-references the row
  __shared__ __attribute__((aligned(1024))) char kbufs0[SG * kKBytes];
  __shared__ __attribute__((aligned(1024))) char kbufs1[PRIVATE ? 16 : SG * kKBytes];
  __shared__ __attribute__((aligned(1024))) char vbufs0[SG * kVBytes];
  __shared__ __attribute__((aligned(1024))) char vbufs1[PRIVATE ? 16 : SG * kVBytes];
  __shared__ float stat_m[SG > 1 ? RW : 1][SG > 1 ? KW : 1][32], stat_l[SG > 1 ? RW : 1][SG > 1 ? KW : 1][32];
  __shared__ float half_m[RW == 4 ? RW : 1][64], half_l[RW == 4 ? RW : 1][64];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_of_group = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int sg = SG == 1 ? 0 : wave_of_group / NW, wave = SG == 1 ? wave_of_group : wave_of_group % NW;
  const int rw = wave % RW, kh = wave / RW;  // row group and key half of this wave
  char* const kbuf0 = kbufs0 + sg * kKBytes;
  char* const kbuf1 = kbufs1 + (PRIVATE ? 0 : sg * kKBytes);
  char* const vbuf0 = vbufs0 + sg * kVBytes;
  char* const vbuf1 = vbufs1 + (PRIVATE ? 0 : sg * kVBytes);
  const int j = lane & 31, g = lane >> 5;

  const int lid = xcd_remap(blockIdx.x, gridDim.x);
  const int qt = lid % a.n_qtiles;
  const Slab slab_of = slab_at(lid / a.n_qtiles, a);
  const int b = slab_of.b, h = slab_of.h, hk = slab_of.hk, bh = b * a.Hq + h;
  int L = a.L;  // length of this batch element
  if (a.seq_lens != nullptr) {
    const int len = a.seq_lens[b];
    L = len < a.L ? len : a.L;
  }
  if (qt * QT >= L) return;  // a query block wholly past the end (uniform over the work-group)

  const __bf16* qbase = static_cast<const __bf16*>(a.q.ptr) + b * a.q.sb + h * a.q.sh;
  const __bf16* kbase = static_cast<const __bf16*>(a.k.ptr) + b * a.k.sb + hk * a.k.sh;
  const __bf16* vbase = static_cast<const __bf16*>(a.v.ptr) + b * a.v.sb + hk * a.v.sh;
  const int row0 = qt * QT + rw * 32;

  int beg = 0, end = 0;
  if (LIST) {  // the rows of a query block may be spread over several work-groups
    const int32_t* rp = a.row_ptr + (int64_t)bh * (a.nqb + 1) + ((qt * QT) >> __builtin_ctz(a.block_q));
    beg = rp[0];
    end = rp[1];
  }
  // A listed 128-key block is two consecutive tiles. Listed 32-key blocks are paired up in list order:
  // tile t holds entries 2t and 2t + 1, one in each 32-key half, wherever in the sequence they come from
  // (the key half a wave owns is then exactly one listed block; an odd count leaves the last half empty).
  constexpr int tile_shift = KB == 2 * kTileK ? 1 : 0;
  constexpr bool half_blocks = KB == kTileK / 2;
  const int entries = end - beg;
  const int n = !LIST ? (L + kTileK - 1) / kTileK : half_blocks ? (entries + 1) >> 1 : entries << tile_shift;
  // steps of this wave: the same for all where they meet at barriers (streams short of a tile end with a masked repeat)
  const int n_steps = SG == 1 ? n : PRIVATE ? (n - sg + SG - 1) / SG : (n + SG - 1) / SG;
  const int32_t* cols = LIST ? a.col_idx + (int64_t)bh * a.cap_per_head + beg : nullptr;
  constexpr int unit = half_blocks ? kTileK / 2 : kTileK;  // keys per copy unit: a 32-key block or a 64-key tile
  const int last_blk = (L - 1) / unit;                 // last unit that exists
  const int tail_keys = L - last_blk * unit;           // keys in it

  float M = SG > 1 ? -1e30f : 0.f, lsum = 0.f;  // (a stream without a tile must not set the row's reference)
  f32x16 o[1][D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int x = 0; x < 16; ++x) o[0][dt][x] = 0.f;
  f32x16 s_a[1], s_b[1];  // logits of the tile being normalised and of the next one
  bf16x8 p[1][2];

  TileDma<D, NT, false> kdma;
  TileDma<D, NT, true> vdma;
  if (half_blocks) {
    kdma.init_half(a.k.sl, wave, lane);
    vdma.init_half(a.v.sl, wave, lane);
  } else {
    kdma.init(a.k.sl, wave, lane);
    vdma.init(a.v.sl, wave, lane);
  }
  KFragAddr<D> kaddr;
  VFragAddr<D> vaddr;
  kaddr.init(lane);
  vaddr.init(lane);

  // Block numbers of this stream's next 64 steps, one a lane; a step reads the ones it needs from there. (A load a step, even
  // four tiles ahead, is waited for by count, and the count takes the copies in flight with it.) Past the end: the last one.
  int list_base = 0;
  auto list_from = [&](int from) -> int {
    const int t = (from + lane) * SG + sg;
    if (half_blocks) {  // the block of this wave's half of the tile; a missing half repeats the last block, masked
      const int e = 2 * t + kh;
      return cols[e < entries ? e : entries - 1];
    }
    const int idx = t < n ? t : n - 1;
    return (cols[idx >> tile_shift] << tile_shift) + (idx & tile_shift);
  };
  int list = LIST && n > 0 ? list_from(0) : 0;
  auto blk_at = [&](int step) -> int {  // key TILE number of this stream's tile at a step; with 32-key blocks: the block of this wave's half
    if (!LIST) {
      const int t = step * SG + sg;
      return t < n ? t : n - 1;
    }
    return __builtin_amdgcn_readlane(list, step - list_base);
  };
  // before steps that need the numbers up to step `last`
  auto reach_list = [&](int t, int last) {
    if (LIST && last - list_base > 63) {
      list_base = t;
      list = list_from(t);
      asm volatile("" : "+v"(list));
      __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0), in a form that the compiler counts: no wait is left for the reads
    }
  };
  QFrag<D, 1> qf;  // loaded after the first K/V copies have been issued (see attn_bf16_kernel.hpp)

  const int64_t slab_rows = (int64_t)(a.L - 1);
  auto rsrc_of = [](const void* base, int64_t bytes) {
    if constexpr (PRIVATE) return untracked_rsrc(base, bytes);
    else return make_rsrc(base, bytes);
  };
  const auto krsrc = rsrc_of(kbase, (slab_rows * a.k.sl + D) * 2);
  const auto vrsrc = rsrc_of(vbase, (slab_rows * a.v.sl + D) * 2);
  const int32_t k_tile_bytes = (int32_t)(unit * a.k.sl * 2), v_tile_bytes = (int32_t)(unit * a.v.sl * 2);  // bytes per copy unit
  // (the second tile of a partial 128-key block may lie wholly past the end: any real tile is copied, all keys masked)
  // a whole unit
  auto copy_whole_k = [&](int ub, char* dst) { kdma.issue(krsrc, ub * k_tile_bytes, dst, wave); };
  auto copy_whole_v = [&](int ub, char* dst) { vdma.issue(vrsrc, ub * v_tile_bytes, dst, wave); };
  auto copy_k = [&](int blk, char* dst) {
    const int ub = blk < last_blk ? blk : last_blk;
    if (ub == last_blk && tail_keys < unit) {
      if (half_blocks) kdma.issue_partial_half(krsrc, ub * k_tile_bytes, dst, wave, lane, a.k.sl, tail_keys);
      else kdma.issue_partial(krsrc, ub * k_tile_bytes, dst, wave, lane, a.k.sl, tail_keys);
    } else {
      copy_whole_k(ub, dst);
    }
  };
  auto copy_v = [&](int blk, char* dst) {
    const int ub = blk < last_blk ? blk : last_blk;
    if (ub == last_blk && tail_keys < unit) {
      if (half_blocks) vdma.issue_partial_half(vrsrc, ub * v_tile_bytes, dst, wave, lane, a.v.sl, tail_keys);
      else vdma.issue_partial(vrsrc, ub * v_tile_bytes, dst, wave, lane, a.v.sl, tail_keys);
    } else {
      copy_whole_v(ub, dst);
    }
  };

  const float c = a.scale_log2;

  // Softmax of this wave's 32 keys of one tile against the row's fixed reference M (same arithmetic as the
  // general kernel: the reference is set once, from the first tile, and a sub-tile whose probabilities leave
  // the range that is good for is redone out of line): s -> p and this lane's share of the row sum.
  auto mask_half = [&](f32x16(&s)[1], int valid) {
    const int mine = valid - 8 * g;  // register x of lane (j, g) holds key 16*(x/8) + 8*g + x%8 of the half
#pragma unroll
    for (int x = 0; x < 16; ++x)
      if (16 * (x >> 3) + (x & 7) >= mine) s[0][x] = -__builtin_inff();
  };
  auto exp_half = [&](const f32x16(&s)[1], float& part) {
    part = 0.f;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      u32x4 pk;
#pragma unroll
      for (int x = 0; x < 8; x += 2) {
        const f32x2 two = {__builtin_amdgcn_exp2f(__builtin_fmaf(s[0][8 * m + x], c, -M)),
                           __builtin_amdgcn_exp2f(__builtin_fmaf(s[0][8 * m + x + 1], c, -M))};
        pk[x >> 1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(two, bf16x2));
        part += two[0];
        part += two[1];
      }
      asm volatile("" : "+v"(pk));  // keep the probabilities inside the block that holds the matrix instructions
      p[0][m] = __builtin_bit_cast(bf16x8, pk);
    }
    asm volatile("" : "+v"(part));
  };
  auto row_max = [&](const f32x16(&s)[1]) -> float {
    float mx = fmaxf(s[0][0], s[0][1]);
#pragma unroll
    for (int x = 2; x < 16; x += 2) mx = fmaxf(fmaxf(mx, s[0][x]), s[0][x + 1]);
    return pair_max(mx) * c;
  };
  auto softmax_half = [&](f32x16(&s)[1], float& part, const bool masked, int valid) {
    if (masked) mask_half(s, valid);
    exp_half(s, part);
  };
  // Out of line, practically never taken: raise the reference to at least this tile's maximum, bring the
  // row's sum and output to it, redo the tile's probabilities.
  auto re_reference = [&](const f32x16(&s)[1], float& part) {
    const float Mn = fmaxf(M, row_max(s));
    const float alpha = __builtin_amdgcn_exp2f(M - Mn);  // <= 1; exactly 1 where nothing changes
    M = Mn;
    lsum *= alpha;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int x = 0; x < 16; ++x) o[0][dt][x] *= alpha;
    exp_half(s, part);
  };
  // keys of this wave's half that exist in its stream's tile at a step
  auto valid_in = [&](int step) -> int {
    const int T = step * SG + sg;
    if (SG > 1 && T >= n) return 0;
    const int tile0 = blk_at(step);
    return half_blocks ? (2 * T + kh < entries ? (tile0 == last_blk ? tail_keys : 32) : 0)
                       : (tile0 > last_blk ? 0 : tile0 == last_blk ? tail_keys : kTileK) - 32 * kh;
  };

  // Tile step t (LDS parity P = t & 1). On entry: S(t) in S_CUR, K(t+1) in kbuf[1-P], V(t) in vbuf[P];
  // kbuf[P] (held K(t)) and vbuf[1-P] (held V(t-1)) are free and receive K(t+2) and V(t+1).
#define SPARSED_SPLITK_STEP(P, MASKED, TAIL, T, S_CUR, S_NEXT)                                       \
  {                                                                                                \
    char* const kb_free = (P) ? kbuf1 : kbuf0;                                                     \
    char* const kb_next = (P) ? kbuf0 : kbuf1;                                                     \
    char* const vb_this = (P) ? vbuf1 : vbuf0;                                                     \
    char* const vb_free = (P) ? vbuf0 : vbuf1;                                                     \
    if (!(TAIL) || (T) + 2 < n_steps) copy_k(blk_at((T) + 2), kb_free);                            \
    if (!(TAIL) || (T) + 1 < n_steps) copy_v(blk_at((T) + 1), vb_free);                            \
    const int valid = !(MASKED) ? 32 : valid_in(T);                                               \
    float part;                                                                                    \
    if (!(TAIL) || (T) + 1 < n_steps) logits_sub<D, 1, false>(kb_next, kh, kaddr, qf, S_NEXT);     \
    softmax_half(S_CUR, part, (MASKED), valid);                                                    \
    sched_substep_interleave<D, 1, false>();                                                       \
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(part < kOverflow)) != 0, 0)) re_reference(S_CUR, part);  \
    lsum += part;                                                                                  \
    __builtin_amdgcn_sched_barrier(0);                                                             \
    if (SG == 1 || !(TAIL) || (T) * SG + sg < n) pv_sub<D, 1, true>(vb_this, kh, vaddr, p, o);     \
    __syncthreads();                                                                               \
  }

  // PRIVATE. On entry: S(t) in S_CUR, K(t+1) on its way to this wave's half of kbuf0, then V(t) to its half of vbuf0.
  // A counted wait leaves exactly one tile copy in flight, the one issued since the fence in front of it (V(t) behind
  // K(t+1); K(t+2) behind V(t)). The copies are issued so that the compiler does not count them: it cannot tell those into
  // kbuf0 from those into vbuf0 and would wait for V(t) in front of the K reads of a step as well, half a step after it was
  // asked for (32 heads of 2000 x 128, 32 x 32 blocks, half kept: 57.9 ->
  // 55.9 us with the list read from registers; 32 heads of 7428 x 128, 32 x 128 blocks, 12 tiles a row: 183 -> 169).
  auto wait_copy = [&](bool all) {
    constexpr int kPer = TileDma<D, NT, false>::kPerWave;
    if (all) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kPer) : "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto reads_done = [&]() {  // this wave's LDS reads have returned: what they read may be overwritten
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
#define SPARSED_PRIVATE_STEP(TAIL, T, S_CUR, S_NEXT)                                               \
  {                                                                                                \
    const int valid = !(TAIL) ? 32 : valid_in(T);                                                \
    float part;                                                                                    \
    if (!(TAIL) || (T) + 1 < n_steps) wait_copy(false); /* K(t+1) */                                     \
    if (!(TAIL) || (T) + 1 < n_steps) {                                                                  \
      logits_sub<D, 1, false>(kbuf0, kh, kaddr, qf, S_NEXT);                                       \
    }                                                                                              \
    softmax_half(S_CUR, part, (TAIL), valid);                                                      \
    sched_substep_interleave<D, 1, false>();                                                       \
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(part < kOverflow)) != 0, 0)) re_reference(S_CUR, part);  \
    lsum += part;                                                                                  \
    reads_done();                                                                                  \
    if (!(TAIL)) copy_whole_k(blk_at((T) + 2), kbuf0);                                             \
    else if ((T) + 2 < n_steps) copy_k(blk_at((T) + 2), kbuf0);                                                     \
    wait_copy((TAIL) && (T) + 2 >= n_steps); /* V(t) */                                                  \
    pv_sub<D, 1, true>(vbuf0, kh, vaddr, p, o);                                                    \
    reads_done();                                                                                  \
    if (!(TAIL)) copy_whole_v(blk_at((T) + 1), vbuf0);                                             \
    else if ((T) + 1 < n_steps) copy_v(blk_at((T) + 1), vbuf0);                                                     \
  }

  if constexpr (PRIVATE) if (n_steps > 0) {
    copy_k(blk_at(0), kbuf0);
    qf.load(qbase, row0, L, a.q.sl, lane);
    wait_vector_memory();
    logits_sub<D, 1, true>(kbuf0, kh, kaddr, qf, s_a);
    reads_done();
    if (n_steps > 1) copy_k(blk_at(1), kbuf0);
    copy_v(blk_at(0), vbuf0);
    {
      f32x16 first[1] = {s_a[0]};  // the first tile fixes the reference, as below
      mask_half(first, valid_in(0));
      M = fmaxf(row_max(first), -1e30f);
    }
    int t = 0;
    // a steady step at tile t copies K(t+2), which must exist and be whole: the last block of the list may be partial
    // (with 128-key blocks its second tile may not exist at all); its copies have no branch, so that
    // a wait has exactly one of them behind it
    const int reach = 3 + ((tail_keys < unit || (tile_shift && !(last_blk & 1))) ? 1 + tile_shift : 0);
    while (t + reach < n_steps) {
      reach_list(t, t + 3);
      SPARSED_PRIVATE_STEP(false, t, s_a, s_b);
      SPARSED_PRIVATE_STEP(false, t + 1, s_b, s_a);
      t += 2;
    }
    for (; t < n_steps; ++t) {
      reach_list(t, t + 2);
      if (t & 1) {
        SPARSED_PRIVATE_STEP(true, t, s_b, s_a);
      } else {
        SPARSED_PRIVATE_STEP(true, t, s_a, s_b);
      }
    }
  }
#undef SPARSED_PRIVATE_STEP

  if constexpr (!PRIVATE) if (n > 0) {
    copy_k(blk_at(0), kbuf0);
    if (n_steps > 1) copy_k(blk_at(1), kbuf1);
    copy_v(blk_at(0), vbuf0);
    qf.load(qbase, row0, L, a.q.sl, lane);
    __syncthreads();
    logits_sub<D, 1, true>(kbuf0, kh, kaddr, qf, s_a);
    {
      // The first tile fixes the reference: the maximum over the keys of this wave's half that exist. A half
      // with no such key (a short first block) starts from a floor that the first real key re-references.
      f32x16 first[1] = {s_a[0]};
      mask_half(first, valid_in(0));
      M = fmaxf(row_max(first), -1e30f);
    }
    __syncthreads();  // everyone is done with K(0) before step 0 lets K(2) overwrite it

    int t = 0;
    while (t + 2 < n_steps) {
      reach_list(t, t + 3);
      SPARSED_SPLITK_STEP(0, false, false, t, s_a, s_b);
      SPARSED_SPLITK_STEP(1, false, false, t + 1, s_b, s_a);
      t += 2;
    }
    reach_list(t, t + 2);
    if (n_steps - t == 2) {  // with 128-key blocks the last two tiles may both be short (a partial last block)
      SPARSED_SPLITK_STEP(0, (tile_shift != 0), true, t, s_a, s_b);
      SPARSED_SPLITK_STEP(1, true, true, t + 1, s_b, s_a);
    } else {
      SPARSED_SPLITK_STEP(0, true, true, t, s_a, s_b);
    }
  }
#undef SPARSED_SPLITK_STEP

  auto row_results = [&](float reference, float ltot) {  // of this lane's row
    if (LIST || (a.lse == nullptr && a.row_stat == nullptr) || g != 0 || row0 + j >= L) return;
    const int64_t at = (int64_t)bh * a.L + row0 + j;
    if (a.lse != nullptr) a.lse[at] = (reference + __builtin_amdgcn_logf(ltot)) * 0.6931471805599453f;
    if (a.row_stat != nullptr) *reinterpret_cast<f32x2*>(a.row_stat + 2 * at) = f32x2{reference, 1.0f / ltot};  // (not a number where the sum is not)
  };
  if constexpr (SG > 1) {
    // Merge the KW parts of every row. Wave `part` of a row group finishes 1/KW of the columns: every wave leaves its
    // accumulator's groups of 8 columns with the wave that owns them, four values a lane, lane after lane, in a region of the
    // (now idle) buffers that belongs to the owner, and the owner adds the parts up, each by its factor, normalises and stores.
    constexpr int kGroups = D / 8, kOwn = kGroups / KW;             // groups of 8 columns, and those of a wave
    constexpr int kRegionBytes = (KW - 1) * kOwn * 1024;
    static_assert(RW <= 2 && (!PRIVATE || RW == 1), "a buffer per wave of a stream");
    static_assert(kRegionBytes <= kVBytes && kVBytes <= kKBytes, "a region a buffer");
    const int part = 2 * sg + kh;
    auto region = [&](int p) -> char* {  // of the wave of this row group that owns part p
      const int w = (p & 1) * RW + rw;   // its number in its stream
      char* const bufs[4] = {kbufs0 + (p >> 1) * kKBytes, PRIVATE || RW == 1 ? vbufs0 + (p >> 1) * kVBytes : kbufs1 + (p >> 1) * kKBytes,
                             vbufs0 + (p >> 1) * kVBytes, vbufs1 + (PRIVATE ? 0 : (p >> 1) * kVBytes)};
      return bufs[w];
    };
    const float ltot_mine = pair_sum(lsum);
    if (PRIVATE) __syncthreads();  // the regions overlap the buffers of waves that may still be reading them
    if (g == 0) {
      stat_m[rw][part][j] = M;
      stat_l[rw][part][j] = ltot_mine;
    }
    f32x4v own[kOwn];
#pragma unroll
    for (int p = 0; p < KW; ++p) {
      f32x4v v[kOwn];
#pragma unroll
      for (int i = 0; i < kOwn; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[i][e] = o[0][(p * kOwn + i) / 4][4 * ((p * kOwn + i) % 4) + e];
      if (p == part) {
#pragma unroll
        for (int i = 0; i < kOwn; ++i) own[i] = v[i];
      } else {
        char* const dst = region(p) + (part < p ? part : part - 1) * (kOwn * 1024) + lane * 16;
#pragma unroll
        for (int i = 0; i < kOwn; ++i) *reinterpret_cast<f32x4v*>(dst + i * 1024) = v[i];
      }
    }
    __syncthreads();
    float Mn = M, ltot = 0.f;
#pragma unroll
    for (int p = 0; p < KW; ++p) Mn = fmaxf(Mn, stat_m[rw][p][j]);
    char* const mine = region(part);
    {
      const float f = __builtin_amdgcn_exp2f(M - Mn);
#pragma unroll
      for (int i = 0; i < kOwn; ++i) own[i] *= f;
    }
#pragma unroll
    for (int p = 0; p < KW; ++p) {
      const float f = __builtin_amdgcn_exp2f(stat_m[rw][p][j] - Mn);
      ltot += stat_l[rw][p][j] * f;
      if (p != part) {
        const char* const src = mine + (p < part ? p : p - 1) * (kOwn * 1024) + lane * 16;
#pragma unroll
        for (int i = 0; i < kOwn; ++i) own[i] += *reinterpret_cast<const f32x4v*>(src + i * 1024) * f;
      }
    }
    const float inv = ltot > 0.f ? 1.0f / ltot : 0.f;
    if (part == 0) row_results(Mn, ltot);

    // stores of whole runs of a row, through an LDS transpose in the wave's own region (its slots of 16 bytes, one per group,
    // at position slot ^ (row mod slots))
    constexpr int kRowBytes = 16 * kOwn;
    static_assert(32 * kRowBytes <= kRegionBytes, "staging fits the region");
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
      const f32x2 lo = {own[i][0] * inv, own[i][1] * inv}, hi = {own[i][2] * inv, own[i][3] * inv};
      u32x2 w;
      w[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, bf16x2));
      w[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, bf16x2));
      *reinterpret_cast<u32x2*>(mine + j * kRowBytes + ((i ^ (j & (kOwn - 1))) << 4) + 8 * g) = w;
    }
    __bf16* const obase = static_cast<__bf16*>(a.o) + b * a.o_sb + h * a.o_sh + part * (8 * kOwn);
#pragma unroll
    for (int it = 0; it < (32 * kOwn + 63) / 64; ++it) {
      const int piece = it * 64 + lane, r = piece / kOwn, slot = piece % kOwn;
      if (r < 32 && row0 + r < L) {
        const u32x4 w = *reinterpret_cast<const u32x4*>(mine + r * kRowBytes + ((slot ^ (r & (kOwn - 1))) << 4));
        *reinterpret_cast<u32x4*>(obase + (int64_t)(row0 + r) * a.o_sl + slot * 8) = w;
      }
    }
  } else {
    // Merge the two key halves of every row. The waves of half 1 leave their accumulator, reference
    // maximum and sum in the (now idle) K buffers, laid out [value][lane] so that both sides touch
    // consecutive words; the waves of half 0 fold them in, normalise and store.
    static_assert(!PRIVATE || RW == 1, "a wave per key half");
    static_assert(RW == 1 || RW == 2 || RW == 4, "a K buffer and a V buffer per wave of the second key half, or a buffer");
    static_assert(D / 32 * 16 * 64 * 4 <= kKBytes && 2 * 64 * 4 <= kVBytes, "exchange areas must fit the buffers");
    float* const xchg = reinterpret_cast<float*>(rw == 0 ? kbuf0 : RW <= 2 || rw == 1 ? kbuf1 : rw == 2 ? vbuf0 : vbuf1);  // the accumulator
    float* const xchg_m = RW == 4 ? half_m[rw] : reinterpret_cast<float*>(rw == 0 ? vbuf0 : vbuf1);  // reference maximum
    float* const xchg_l = RW == 4 ? half_l[rw] : xchg_m + 64;                                        // and sum
    const float ltot_mine = pair_sum(lsum);
    if (PRIVATE) __syncthreads();  // the exchange overlaps the other wave's halves
    if (kh == 1) {
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int x = 0; x < 16; ++x) xchg[(dt * 16 + x) * 64 + lane] = o[0][dt][x];
      xchg_m[lane] = M;
      xchg_l[lane] = ltot_mine;
    }
    __syncthreads();
    if (kh == 1) return;
    const float M_other = xchg_m[lane], l_other = xchg_l[lane];
    const float Mn = fmaxf(M, M_other);
    const float f_mine = __builtin_amdgcn_exp2f(M - Mn), f_other = __builtin_amdgcn_exp2f(M_other - Mn);
    const float ltot = ltot_mine * f_mine + l_other * f_other;
    const float inv = ltot > 0.f ? 1.0f / ltot : 0.f;
    row_results(Mn, ltot);
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int x = 0; x < 16; ++x) o[0][dt][x] = (o[0][dt][x] * f_mine + xchg[(dt * 16 + x) * 64 + lane] * f_other) * inv;

    // whole-row stores through an LDS transpose (see the epilogue of attn_bf16_kernel.hpp); the staging slice is this
    // row group's V buffer, whose two exchanged values this wave has already read (with four row groups: where its exchange was)
    constexpr int kRowBytes = 2 * D, kSlots = D / 8, kRowsPerStore = 64 / kSlots;
    static_assert(32 * kRowBytes <= kVBytes, "staging slice must fit a V buffer");
    char* const stage = RW == 4 ? reinterpret_cast<char*>(xchg) : rw == 0 ? vbuf0 : vbuf1;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const f32x2 lo = {o[0][dt][4 * q4], o[0][dt][4 * q4 + 1]};
        const f32x2 hi = {o[0][dt][4 * q4 + 2], o[0][dt][4 * q4 + 3]};
        u32x2 w;
        w[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, bf16x2));
        w[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, bf16x2));
        *reinterpret_cast<u32x2*>(stage + j * kRowBytes + (((4 * dt + q4) ^ (j & (kSlots - 1))) << 4) + 8 * g) = w;
      }
    __bf16* const obase = static_cast<__bf16*>(a.o) + b * a.o_sb + h * a.o_sh;
#pragma unroll
    for (int it = 0; it < 32 / kRowsPerStore; ++it) {
      const int r = it * kRowsPerStore + lane / kSlots, slot = lane % kSlots;
      const u32x4 w = *reinterpret_cast<const u32x4*>(stage + r * kRowBytes + ((slot ^ (r & (kSlots - 1))) << 4));
      const int grow = row0 + r;
      if (grow < L) *reinterpret_cast<u32x4*>(obase + (int64_t)grow * a.o_sl + slot * 8) = w;
    }
  }
#endif
}

template <int D, int RW, bool PRIVATE, int SG>
static hipError_t launch_splitk(Mode mode, AttnArgs a, hipStream_t s) {
  a.n_qtiles = (a.L + 32 * RW - 1) / (32 * RW);
  const int64_t total = (int64_t)a.B * a.Hq * a.n_qtiles;
  if (total <= 0 || total > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid((unsigned)total), block(RW * SG * 128);
  if (mode == Mode::kDense) {
    if constexpr (RW * SG == 1) return hipErrorInvalidValue;  // no rule takes dense there
    else hipLaunchKernelGGL((attn_bf16_splitk_kernel<D, RW, 64, PRIVATE, SG, false>), grid, block, 0, s, a);
    return hipGetLastError();
  }
  switch (a.block_k) {
    case 32: hipLaunchKernelGGL((attn_bf16_splitk_kernel<D, RW, 32, PRIVATE, SG, true>), grid, block, 0, s, a); break;
    case 64: hipLaunchKernelGGL((attn_bf16_splitk_kernel<D, RW, 64, PRIVATE, SG, true>), grid, block, 0, s, a); break;
    case 128: hipLaunchKernelGGL((attn_bf16_splitk_kernel<D, RW, 128, PRIVATE, SG, true>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Whether and how a dense or sparse call is split over the keys. What counts is how many runs of 32 query rows there are (the
// chip holds 2048 waves of 256 registers) and how many tiles each walks. Dense, and sparse with 128-row query blocks, up to
// 1024 runs: the general kernel's work-groups of 128 or 256 rows leave compute units idle or with one wave a SIMD. The fewer the
// runs, the smaller the work-group's share of rows and the more parts of the keys, as long as a part has a few tiles; rows of
// one query block in several work-groups walk the same list. Beyond, K and V copied for 32 to 128 rows instead of 128 or 256
// cost more than the idle units (1504 runs of 94 tiles, head dim 128, dense: 146.5 us general, 164.7 split).
// Dense, us, general -> split, (heads, tokens, head dim): (4, 2048, 64) 33.0 -> 13.6, (4, 2048, 128) 43.6 -> 19.9,
// (8, 600, 64) 12.9 -> 8.5, (16, 600, 64) 13.1 -> 9.7, (4, 4096, 64) 61.4 -> 27.9, (8, 4096, 128) 84.0 -> 71.0,
// (28, 600, 64) 13.5 -> 11.9. Sparse 128 x 128, 30 % kept: (4, 2048, 64) 12.4 -> 8.8, (4, 2048, 128) 15.1 -> 11.9,
// (4, 4096, 64) 19.6 -> 13.9, (8, 3000, 64) 19.1 -> 17.0 (head dim 128: 24.0 and 23.6, with longer lists the general kernel is
// the faster one; with lists of fewer than 8 tiles it is at 64). Sparse 32 x 32, half kept: (4, 2048, 64) 13.3 -> 9.8,
// (4, 4096, 128) 35.6 -> 30.2. Sparse 64 x 64, 7 tiles, 256 runs: 8.2 split in two, 7.8 in four.
bool splitk_takes(Mode mode, int D, int block_q, const AttnArgs& a) {
  if (mode == Mode::kSparse && block_q <= 64) return true;
  if (mode != Mode::kDense && mode != Mode::kSparse) return false;
  const int64_t runs = (int64_t)a.B * a.Hq * ((a.L + 31) / 32);
  if (runs <= 512) return true;
  return runs <= 1024 && (mode == Mode::kDense || (D == 64 && (int64_t)a.cap_per_head * a.block_k >= (int64_t)8 * kTileK * a.nqb));
}

template <int D>
static hipError_t launch_splitk_d(Mode mode, int block_q, const AttnArgs& a, hipStream_t s) {
  const bool dense = mode == Mode::kDense;
  const int64_t runs = (int64_t)a.B * a.Hq * ((a.L + 31) / 32);
  // tiles that a row walks; the host does not know the lists: their capacity is the average length where it is exact, and an
  // upper bound of it otherwise
  const int64_t tiles = dense ? (a.L + kTileK - 1) / kTileK : ((int64_t)a.cap_per_head * a.block_k / kTileK + a.nqb - 1) / a.nqb;
  if (!dense && block_q == 32) {
    if (tiles >= (runs <= 256 ? 4 : 12) && runs <= 512) return launch_splitk<D, 1, true, 2>(mode, a, s);
    // Double buffers while every compute unit has at most the two work-groups that they allow: 448 work-groups, 14 tiles a row:
    // head dim 64 11.5 us against 13.4 private, 128 18.3 against 19.2; 528 work-groups, 8 tiles: 14.4 against 10.3, 21.7 against
    // 15.3.
    if (runs <= 512) return launch_splitk<D, 1, false, 1>(mode, a, s);
    return launch_splitk<D, 1, true, 1>(mode, a, s);
  }
  if (runs <= 256 && tiles >= (dense ? 8 : 10)) return launch_splitk<D, 1, true, 2>(mode, a, s);
  // An index with room for every block says nothing of the length of its lists, and eight waves a work-group lose more on short ones
  // than they gain on long ones. Against four waves, lists of less than 6 tiles and of 14 and more: 64 x 64 blocks 1.18 (up to 1.46) and
  // 0.95 of the time, 64 x 128 1.13 (up to 1.37) and 0.88, 128 x 64 1.17 and 1.02; 128 x 128 blocks gain (general kernel 1, eight
  // waves 0.84 and 0.68).
  const bool any_length = !dense && (block_q == 64 || a.block_k < 128) &&
                          (int64_t)a.cap_per_head >= (int64_t)a.nqb * ((a.L + a.block_k - 1) / a.block_k);
  if (runs > 256 && runs <= 512 && !any_length && tiles >= (!dense ? 16 : D == 64 ? 12 : 20)) return launch_splitk<D, 2, false, 2>(mode, a, s);
  if (runs > 512 && (dense || block_q == 128)) {
    if constexpr (D == 64) return launch_splitk<D, 4, false, 1>(mode, a, s);
    else if (dense) return launch_splitk<D, 4, false, 1>(mode, a, s);
  }
  return launch_splitk<D, 2, false, 1>(mode, a, s);
}

hipError_t launch_attn_bf16_splitk(Mode mode, int D, int block_q, const AttnArgs& a, hipStream_t s) {
  if (mode == Mode::kSparse && block_q != 32 && block_q != 64 && block_q != 128) return hipErrorInvalidValue;
  if (D == 128) return launch_splitk_d<128>(mode, block_q, a, s);
  if (D == 64) return launch_splitk_d<64>(mode, block_q, a, s);
  return hipErrorInvalidValue;
}

}  // namespace sparsed
