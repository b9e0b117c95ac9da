// Device-side building blocks of the fp32 kernels for gfx950 (wave64; v_mfma_f32_32x32x16_bf16 on split operands, and
// v_mfma_f32_32x32x2_f32).
//
// Same transposed formulation as the bf16 kernels: S^T[key, query] = K . Q^T puts one query in
// each lane (lane = 32*g + j holds query j; register v holds key row 8*(v/4) + 4*g + (v%4) of the
// 32-key tile). Inputs, accumulators and softmax are fp32, and the products as good as fp32 ones:
//
// Products. The fp32 matrix instruction contracts 2 columns in 64 cycles, the bf16 one 16 in 32. An fp32 value is the sum of
// three bf16 values to 2^-26 of itself (each the nearest to what the ones before it leave, all of them exact differences),
// so a product of two fp32 numbers is six bf16 products, exact in the fp32 accumulator: those of the parts whose orders add up
// to at most 2^-17 of the whole (h h, h m, m h, m m, h l, l h); the three left out are below 2^-26 of it, a quarter of half
// an fp32 unit in the last place. Six bf16 instructions take 192 cycles for what the fp32 one takes 512, and their sums are
// rounded less often: error against 64 bits see attn_f32.hip. An operand that is infinite, not a number or beyond the
// largest bf16 number splits into parts that are not numbers; and parts end at 2^-133, so a value is carried to 2^-26 of itself
// or to 2^-134, whichever is more. A work-group whose results either may show does its work again on the fp32 instruction, so
// such inputs give what they give there. It can tell at little cost:
//   logits  A query value below 2^-108 (and not zero) is short of bits, and one of 2^80 or more would show that a key value is
//           (SplitRange, where the queries are split); with neither, a logit is off by 2^-47 at most.
//   output  Probabilities add up to 2^-134 of an error for every value of V. A sum below 2^-90 (and not zero) may show it.
//           Probabilities below 2^-108 of the row's largest are short of bits themselves; a tile that has any notes the largest
//           value of V there, and the least sum that is good rises to 2^-92 of it (2^16 keys that are off by 2^-134 each, 2^-26
//           of the sum). A sum of zero is good where V is zero: a wave with one reads its V again and asks for a repeat if a value
//           is below 2^-108 and not zero, or may be 2^32 or more at such probabilities. Dense calls with columns of zeros, 8
//           heads of 2000 x 128: 109 -> 124 us, 2 of 256 x 64 9.1 -> 10.0; V all zeros, which used to be a repeat, 218 -> 109, 16.2 -> 10.1.
//
// K and V go from global memory straight into the registers that feed the matrix cores: the vector memory path delivers
// them with room to spare, and nothing is gained by passing a tile through LDS (and a barrier) to reorder it. Both products
// sum over an index whose order is free, so the order is chosen to make the loads wide:
//   first product:  lane (i, g) holds columns 8c + 4g .. + 3 of key row i, one 16-byte load: four steps of the fp32
//                   instruction, half the operand of a step of the bf16 one (whose other half is chunk c + 1);
//   second product: accumulator register x of the first product is, as it stands, the B operand for the key pair
//                   {8*(x/4) + (x%4), + 4} of the fp32 instruction, eight of them that of the bf16 one; tile dt of the
//                   output takes columns (D/32)*i + dt, so lane (i, g) needs D/32 consecutive columns of one V row: one
//                   load per key pair, a whole row per half wave.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sparsed {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2f;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8f;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2f;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4f;

constexpr int kTileKF = 32;  // keys per K/V tile of the fp32 kernels

// Of the two lanes j and j + 32 that share a query: the larger value, the sum of both.
__device__ __forceinline__ float pair_max_f(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum_f(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ float wave_sum_f(float x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

__device__ __forceinline__ int xcd_remap_f(int wg, int total) {
  const int q = total >> 3, r = total & 7;
  const int x = wg & 7, n = wg >> 3;
  return x * q + (x < r ? x : r) + n;
}

// Eight fp32 values as the sums of three bf16 values each: one operand of the bf16 matrix instruction per part.
struct Split8 {
  u32x4f h, m, l;
  __device__ __forceinline__ void pair(int i, float a, float b) {  // values 2i and 2i + 1
    auto take = [&]() -> uint32_t {  // the nearest bf16 values; a and b become what they leave
      const f32x2f two = {a, b};
      const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector(two, bf16x2f));
      a -= __uint_as_float(w << 16);
      b -= __uint_as_float(w & 0xffff0000u);
      return w;
    };
    h[i] = take();
    m[i] = take();
    l[i] = take();
  }
};
__device__ __forceinline__ Split8 split8(f32x4 lo, f32x4 hi) {
  Split8 w;
  w.pair(0, lo[0], lo[1]);
  w.pair(1, lo[2], lo[3]);
  w.pair(2, hi[0], hi[1]);
  w.pair(3, hi[2], hi[3]);
  return w;
}
// Whether values lie where their three parts stand for them to 2^-26 and products with parts that are cut off stay small.
struct SplitRange {
  static constexpr uint32_t kLeast = (127u - 108u) << 24;  // 2^-108, doubled bits
  uint32_t low = ~0u;                                      // least doubled bits less one: zero comes last
  float high = 0.f;
  __device__ __forceinline__ void add_low(float v) {
    const uint32_t u = (__float_as_uint(v) << 1) - 1u;
    low = u < low ? u : low;
  }
  __device__ __forceinline__ void add(f32x4 v) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      add_low(v[e]);
      high = fmaxf(high, fabsf(v[e]));
    }
  }
  __device__ __forceinline__ bool below() const { return low < kLeast - 1u; }
  __device__ __forceinline__ bool outside() const { return below() || !(high < 0x1p80f); }
};
// acc += A . B, the six products of the parts that matter, smallest first
__device__ __forceinline__ f32x16 mfma_split(const Split8& a, const Split8& b, f32x16 acc) {
  auto mul = [&](const u32x4f& x, const u32x4f& y) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8f, x), __builtin_bit_cast(bf16x8f, y), acc, 0, 0, 0);
  };
  mul(a.l, b.h);
  mul(a.h, b.l);
  mul(a.m, b.m);
  mul(a.m, b.h);
  mul(a.h, b.m);
  mul(a.h, b.h);
  return acc;
}
// The layout of a block of `mfma_split` calls and the splitting of the next one's operand: vector instructions behind every
// matrix instruction, which occupies the matrix core for the time of sixteen of them.
template <int READS>
__device__ __forceinline__ void sched_split_interleave() {
  if (READS) __builtin_amdgcn_sched_group_barrier(0x100, READS, 0);
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
  }
}

// A (batch, head) slab of K or V and this lane's way of reading 32-key tiles of it, through a buffer descriptor that ends with
// the slab: rows at or past its end (a tile at the end of the sequence, or wholly past it) read as zeros, unless the rows are so
// far apart that their 32-bit offsets wrap; they then read as something inside the slab. The caller masks their logits and
// clears their V.
template <int D>
struct SlabF32 {
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t row_bytes;
  __device__ __forceinline__ void init(const float* base, int64_t stride_l, int rows) {
    row_bytes = (uint32_t)(stride_l * 4);
    const int64_t bytes = ((int64_t)(rows - 1) * stride_l + D) * 4;
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, (int32_t)bytes, 0x00020000);
  }
  // K: byte offset of chunk 0 of the key row of lane (j, g) in the tile that begins at `key`
  __device__ __forceinline__ uint32_t k_offset(int key, int lane) const { return (uint32_t)(key + (lane & 31)) * row_bytes + 16 * (lane >> 5); }
  // chunk c of the first product's operand: columns 8c + 4g .. + 3 of that row
  __device__ __forceinline__ f32x4 k_chunk(uint32_t off, int c) const {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off + 32 * c, 0, 0));
  }
  // V: byte offset of this lane's columns of key pair 0 in the tile that begins at `key`
  __device__ __forceinline__ uint32_t v_offset(int key, int lane) const {
    return (uint32_t)(key + 4 * (lane >> 5)) * row_bytes + (lane & 31) * (uint32_t)sizeof(VRow);
  }
  // key pair x of the second product's operand: D/32 consecutive columns of key row key + 8*(x/4) + 4g + (x%4)
  typedef __attribute__((ext_vector_type(D / 32))) float VRow;
  __device__ __forceinline__ VRow v_row(uint32_t off, int x) const {
    const uint32_t at = off + (uint32_t)(8 * (x / 4) + (x % 4)) * row_bytes;
    if constexpr (D == 128) return __builtin_bit_cast(VRow, __builtin_amdgcn_raw_buffer_load_b128(rsrc, at, 0, 0));
    else return __builtin_bit_cast(VRow, __builtin_amdgcn_raw_buffer_load_b64(rsrc, at, 0, 0));
  }
};

// A wave's own K tile in LDS. A load that hands a lane 16 bytes of its own key row touches 32 rows, and the address path takes
// about four times as long for it as for whole rows (pool_f32_kernel, 8 heads of 2000 x 128: 74 us so, 61 us through
// LDS); so the tile is copied in whole rows, global -> LDS directly, and the lanes read their chunks there. Chunk c (16 bytes) of
// row r sits at position c ^ (r & 15) of the row: 16 consecutive lanes, the same chunk of 16 rows, read 16 different positions.
template <int D>
struct KTileF32 {
  static constexpr int kBytes = kTileKF * D * 4, kLoads = kBytes / 1024, kRowsPerLoad = 256 / D;
  // copy of the tile that begins at `key`; rows that do not exist leave zeros or what was there
  __device__ __forceinline__ static void copy(const SlabF32<D>& s, int key, char* tile, int lane) {
    const int hi = lane / (D / 4);
    const uint32_t row0 = (uint32_t)(key + hi) * s.row_bytes, pos = (uint32_t)((lane % (D / 4)) ^ hi) << 4;
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const uint32_t at = row0 + (uint32_t)(u * kRowsPerLoad) * s.row_bytes + (pos ^ (uint32_t)(((u * kRowsPerLoad) & 15) << 4));
      __builtin_amdgcn_raw_ptr_buffer_load_lds(s.rsrc, (__attribute__((address_space(3))) void*)(tile + u * 1024), 16, at, 0, 0, 0);
    }
  }
  // chunk ch of the first product's operand (as SlabF32::k_chunk)
  __device__ __forceinline__ static f32x4 chunk(const char* tile, int ch, int lane) {
    const int i = lane & 31, x = (lane >> 5) ^ (i & 15);
    return *reinterpret_cast<const f32x4*>(tile + i * (4 * D) + ((x ^ ((2 * ch) & 15)) << 4) + ((2 * ch) & 16) * 16);
  }
};
// Every LDS read this wave has issued has returned: what it read may be overwritten.
__device__ __forceinline__ void lds_reads_done_f() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// All vector memory operations of this wave but the newest N have completed.
template <int N>
__device__ __forceinline__ void vector_memory_done_but_f() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
  __builtin_amdgcn_sched_barrier(0);
}

}  // namespace sparsed
