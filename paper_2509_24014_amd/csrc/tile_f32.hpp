// Device-side building blocks of the fp32 kernels for gfx950 (wave64, v_mfma_f32_32x32x2_f32).
//
// Same transposed formulation as the bf16 kernels: S^T[key, query] = K . Q^T puts one query in
// each lane (lane = 32*g + j holds query j; register v holds key row 8*(v/4) + 4*g + (v%4) of the
// 32-key tile). Everything stays fp32: inputs, both products, softmax.
//
// K and V go from global memory straight into the registers that feed the matrix cores. An fp32 32x32x2 product
// occupies the matrix core for 64 cycles and takes one register of each operand, so a wave needs 16 KB of K in
// 4096 cycles: the vector memory path delivers that with room to spare, and nothing is gained by passing a tile
// through LDS (and a barrier) to reorder it. Both products sum over an index whose order is free, so the order is
// chosen to make the loads wide:
//   first product:  step 4c + e contracts columns 8c + e (lanes g = 0) and 8c + 4 + e (g = 1): lane (i, g) holds
//                   columns 8c + 4g .. + 3 of key row i, one 16-byte load per four steps;
//   second product: accumulator register x of the first product is, as it stands, the B operand for the key pair
//                   {8*(x/4) + (x%4), + 4}; tile dt of the output takes columns (D/32)*i + dt, so lane (i, g) needs
//                   D/32 consecutive columns of one V row: one load per key pair, a whole row per half wave.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sparsed {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kTileKF = 32;  // keys per K/V tile of the fp32 kernels

__device__ __forceinline__ float other_half_f(float x) { return __shfl_xor(x, 32, 64); }

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

// A (batch, head) slab of K or V and this lane's way of reading 32-key tiles of it. Rows at or past `rows` (a tile at
// the end of the sequence, or wholly past it) are read from the last row that exists; the caller masks their logits.
template <int D>
struct SlabF32 {
  const char* base;    // row 0
  uint32_t row_bytes;  // fits: a slab is below 2^31 bytes
  int rows;
  __device__ __forceinline__ uint32_t row_offset(int row) const { return (uint32_t)(row < rows ? row : rows - 1) * row_bytes; }
  // chunk c of the first product's operand: columns 8c + 4g .. + 3 of the row at byte offset `off` (which includes 16g)
  __device__ __forceinline__ f32x4 k_chunk(uint32_t off, int c) const {
    return *reinterpret_cast<const f32x4*>(base + off + 32 * c);
  }
  // key pair x of the second product's operand: D/32 consecutive columns of key row key0 + 8*(x/4) + 4g + (x%4)
  typedef __attribute__((ext_vector_type(D / 32))) float VRow;
  __device__ __forceinline__ VRow v_row(int key0, int x, int lane) const {
    const int row = key0 + 8 * (x / 4) + 4 * (lane >> 5) + (x % 4);
    return *reinterpret_cast<const VRow*>(base + row_offset(row) + (lane & 31) * (uint32_t)sizeof(VRow));
  }
};

}  // namespace sparsed
