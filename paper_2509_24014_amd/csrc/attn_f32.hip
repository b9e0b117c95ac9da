// fp32 flash-attention forward for gfx950: dense (Eq. 1), block-sparse (Eq. 3 / Eq. 4) and the
// statistics-only pass. fp32 inputs, fp32 matrix cores (32x32x2), fp32 softmax, fp32 output:
// this is the path held to 1e-5 against the fp64 reference.
//
// One work-group owns 32 query rows of one (batch, head); its KW waves share the rows and split the keys: wave w takes
// the 32-key tiles w, w + KW, ... of the list with its own running maximum, sum and output accumulator, and the parts
// are merged once, through LDS, at the end. The waves need nothing from each other in between (K and V are loaded
// straight into registers, see tile_f32.hpp), so the tile loop has no barrier, and a short sequence still spreads over
// many waves. A fragment of the next tile is requested as soon as the fragment it replaces has been used: every load
// has a whole tile of matrix work (8192 cycles at head dim 128) to arrive.
//
// Bound: the fp32 matrix rate (157 TFLOP/s nominal). 8 heads of 2000 x 128: dense 440 -> 167 us (98 TFLOP/s), sparse
// (64 x 64 blocks, 20 % kept) 122 -> 50 us; 2 heads of 256 x 64: dense 33 -> 12 us, sparse 18 -> 8 us. (Before: tiles staged
// through LDS by all waves, two barriers per tile, one LDS read per matrix instruction and operand, rows not split.)
#include "kernels.hpp"
#include "tile_f32.hpp"

namespace sparsed {

template <int D, int KW, Mode MODE>
__global__ __launch_bounds__(KW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_f32_kernel(const AttnArgs a) {
  constexpr int NT = KW * 64;
  constexpr bool kHasV = MODE != Mode::kStats;
  constexpr int kChunks = D / 8, kV = D / 32;
  using VRow = typename SlabF32<D>::VRow;
  // The query fragments ([chunk][lane], 16 bytes each) and, once the keys are done, the waves' accumulators
  // ([wave][row][32 pieces of D/32 columns], piece i of row j at position i ^ j so that neither side has bank conflicts).
  constexpr int kQBytes = kChunks * 64 * 16, kAccBytes = kHasV ? KW * 32 * D * 4 : 16;
  __shared__ __attribute__((aligned(16))) char lds[kQBytes > kAccBytes ? kQBytes : kAccBytes];
  __shared__ float stat_m[KW][32], stat_l[KW][32];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
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
  const int row0 = qt * 32;
  if (row0 >= L) return;  // a query tile wholly past the end (uniform over the work-group)

  const SlabF32<D> ks{reinterpret_cast<const char*>(static_cast<const float*>(a.k.ptr) + b * a.k.sb + hk * a.k.sh), (uint32_t)(a.k.sl * 4), L};
  const SlabF32<D> vs{reinterpret_cast<const char*>(kHasV ? static_cast<const float*>(a.v.ptr) + b * a.v.sb + hk * a.v.sh : nullptr),
                      (uint32_t)(a.v.sl * 4), L};

  // tiles of the list: every 32 keys (dense), or those of the listed key blocks
  const int tile_shift = (MODE == Mode::kSparse) ? (a.block_k == 128 ? 2 : a.block_k == 64 ? 1 : 0) : 0;
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
  auto first_key = [&](int t) -> int {  // of tile t of the list; past the end: of the last one (a harmless repeat)
    const int u = t < n ? t : n - 1;
    if (MODE != Mode::kSparse) return u * kTileKF;
    return cols[(u >> tile_shift) + opaque_zero] * a.block_k + (u & ((1 << tile_shift) - 1)) * kTileKF;
  };

  {  // query fragments into LDS: lane (j, g) of chunk c holds columns 8c + 4g .. + 3 of row j
    const int row = row0 + j < L ? row0 + j : L - 1;
    const float* qrow = static_cast<const float*>(a.q.ptr) + b * a.q.sb + h * a.q.sh + (int64_t)row * a.q.sl + 4 * g;
    for (int c = wave; c < kChunks; c += KW)
      *reinterpret_cast<f32x4*>(lds + (c * 64 + lane) * 16) = *reinterpret_cast<const f32x4*>(qrow + 8 * c);
  }

  float M = -1e30f, lsum = 0.f;
  f32x16 o[kV];
#pragma unroll
  for (int dt = 0; dt < kV; ++dt)
#pragma unroll
    for (int x = 0; x < 16; ++x) o[dt][x] = 0.f;
  f32x4 kf[kChunks];
  VRow vf[16];
  const float c = a.scale_log2;

  int t = wave, key = 0, key_next = 0;
  if (t < n) {
    key = __builtin_amdgcn_readfirstlane(first_key(t));
    key_next = __builtin_amdgcn_readfirstlane(first_key(t + KW));
    const uint32_t off = ks.row_offset(key + j) + 16 * g;
#pragma unroll
    for (int ch = 0; ch < kChunks; ++ch) kf[ch] = ks.k_chunk(off, ch);
    if (kHasV) {
#pragma unroll
      for (int x = 0; x < 16; ++x) vf[x] = vs.v_row(key, x, lane);
    }
  }
  __syncthreads();
  for (; t < n; t += KW) {
    const int key_after = first_key(t + 2 * KW);
    const uint32_t off_next = ks.row_offset(key_next + j) + 16 * g;
    f32x16 s;
#pragma unroll
    for (int x = 0; x < 16; ++x) s[x] = 0.f;
#pragma unroll
    for (int ch = 0; ch < kChunks; ++ch) {
      const f32x4 qf = *reinterpret_cast<const f32x4*>(lds + (ch * 64 + lane) * 16);
#pragma unroll
      for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[ch][e], qf[e], s, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);  // the reload stays behind its fragment's last use, so it can take its registers
      kf[ch] = ks.k_chunk(off_next, ch);
    }
    // keys of this tile that exist: fewer than 32 at the end of a sequence whose length is not a multiple of the tile,
    // none in the later tiles of a partial last key block
    const int valid = L - key;
    if (valid < kTileKF) {
#pragma unroll
      for (int x = 0; x < 16; ++x)
        if (8 * (x / 4) + 4 * g + (x % 4) >= valid) s[x] = -__builtin_inff();
      if (kHasV && valid <= 0) {  // no key at all: the rows stand for none, and 0 times an infinity of theirs would be NaN
#pragma unroll
        for (int x = 0; x < 16; ++x)
#pragma unroll
          for (int dt = 0; dt < kV; ++dt) vf[x][dt] = 0.f;
      }
    }
    float mx = s[0];
#pragma unroll
    for (int x = 1; x < 16; ++x) mx = fmaxf(mx, s[x]);
    mx = fmaxf(mx, other_half_f(mx));
    const float Mn = fmaxf(M, mx * c);
    const float alpha = exp2f(M - Mn);
    M = Mn;
    float part = 0.f;
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      s[x] = exp2f(__builtin_fmaf(s[x], c, -Mn));
      part += s[x];
    }
    lsum = lsum * alpha + part;
    if (kHasV) {
      if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
        for (int dt = 0; dt < kV; ++dt)
#pragma unroll
          for (int x = 0; x < 16; ++x) o[dt][x] *= alpha;
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int x = 0; x < 16; ++x) {
#pragma unroll
        for (int dt = 0; dt < kV; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[x][dt], s[x], o[dt], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        vf[x] = vs.v_row(key_next, x, lane);
      }
    }
    key = key_next;
    key_next = __builtin_amdgcn_readfirstlane(key_after);
  }

  // Merge the waves' parts: O = sum_w O_w 2^(M_w - M) / sum_w l_w 2^(M_w - M), M = max_w M_w.
  const float ltot = lsum + other_half_f(lsum);
  __syncthreads();  // everyone is done with the query fragments
  if (g == 0) {
    stat_m[wave][j] = M;
    stat_l[wave][j] = ltot;
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
  auto factors = [&](int row, float (&f)[KW], float* m) -> float {  // every wave's factor and the common maximum; returns l
    float mm = stat_m[0][row], l = 0.f;
#pragma unroll
    for (int w = 1; w < KW; ++w) mm = fmaxf(mm, stat_m[w][row]);
#pragma unroll
    for (int w = 0; w < KW; ++w) {
      f[w] = exp2f(stat_m[w][row] - mm);
      l += stat_l[w][row] * f[w];
    }
    *m = mm;
    return l;
  };
  if (a.lse != nullptr && tid < 32 && row0 + tid < L) {
    float f[KW], m;
    const float l = factors(tid, f, &m);
    a.lse[(int64_t)bh * a.L + row0 + tid] = (m + log2f(l)) * 0.6931471805599453f;
  }
  if (kHasV) {
    for (int id = tid; id < 32 * 32; id += NT) {
      const int row = id >> 5, piece = id & 31;
      if (row0 + row >= L) break;  // partial last query tile (rows ascend with id)
      float f[KW], m;
      const float l = factors(row, f, &m);
      const float inv = l > 0.f ? 1.0f / l : 0.f;
      VRow acc;
#pragma unroll
      for (int dt = 0; dt < kV; ++dt) acc[dt] = 0.f;
#pragma unroll
      for (int w = 0; w < KW; ++w) {
        const VRow part = *reinterpret_cast<const VRow*>(lds + ((w * 32 + row) * 32 + (piece ^ row)) * sizeof(VRow));
#pragma unroll
        for (int dt = 0; dt < kV; ++dt) acc[dt] += part[dt] * f[w];
      }
#pragma unroll
      for (int dt = 0; dt < kV; ++dt) acc[dt] *= inv;
      float* orow = static_cast<float*>(a.o) + b * a.o_sb + h * a.o_sh + (int64_t)(row0 + row) * a.o_sl;
      *reinterpret_cast<VRow*>(orow + kV * piece) = acc;
    }
  }
}

template <int D, int KW, Mode MODE>
static hipError_t launch_one_f32(const AttnArgs& a, hipStream_t s) {
  const int64_t total = (int64_t)a.B * a.Hq * a.n_qtiles;
  if (total <= 0 || total > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL((attn_f32_kernel<D, KW, MODE>), dim3((unsigned)total), dim3(KW * 64), 0, s, a);
  return hipGetLastError();
}

// Waves per work-group, dense and statistics: a compute unit holds eight waves of this kernel, as two work-groups of four or
// one of eight. Eight where there are no more work-groups than compute units (short sequences: the keys split eight ways), else four.
template <int D, Mode MODE>
static hipError_t launch_by_fill_f32(const AttnArgs& a, hipStream_t s) {
  if ((int64_t)a.B * a.Hq * a.n_qtiles <= 256) return launch_one_f32<D, 8, MODE>(a, s);
  return launch_one_f32<D, 4, MODE>(a, s);
}

// Sparse: a short list does not feed four waves, and a work-group of one wave leaves its compute unit to seven others. Two
// waves of a SIMD share its matrix core in about the time of 1.6 that run alone, one after the other, so the time goes with
// the waves of the busiest SIMD (2 a pair, 1.25 for an odd one) times the steps of a wave, plus 1.5 steps of prologue and
// epilogue for a wave that walks its list alone and 0.5 for one of four (theirs overlap). One wave where that is less; two
// came out best only between the others. The average list comes from the capacity, which is exact or an upper bound. 544
// calls (352 to 4080 work-groups, 1 to 16 tiles, both head dims): never slower than four waves for all, 2 % from the best of
// one, two and four on average. At 64 columns a head, 128 x 32 blocks: 2048 work-groups with one tile 32.8 -> 17.8 us, with 5
// tiles 54.7 -> 38.1 us, 1000 with two tiles 19.4 -> 13.5 us.
template <int D>
static hipError_t launch_sparse_f32(const AttnArgs& a, hipStream_t s) {
  const int64_t groups = (int64_t)a.B * a.Hq * a.n_qtiles;
  if (groups <= 256) return launch_one_f32<D, 8, Mode::kSparse>(a, s);
  const int64_t tiles = ((int64_t)a.cap_per_head * (a.block_k / kTileKF) + a.nqb - 1) / a.nqb;
  auto busiest_simd = [](int64_t waves) -> int64_t {  // in quarters
    const int64_t n = (waves + 1023) / 1024;
    return n / 2 * 8 + n % 2 * 5;
  };
  const int64_t one = busiest_simd(groups) * (2 * tiles + 3), four = busiest_simd(4 * groups) * (2 * ((tiles + 3) / 4) + 1);
  return one < four ? launch_one_f32<D, 1, Mode::kSparse>(a, s) : launch_one_f32<D, 4, Mode::kSparse>(a, s);
}

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
