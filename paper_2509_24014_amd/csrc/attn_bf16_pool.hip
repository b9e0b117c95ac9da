// The dense bf16 attention step that also leaves the pooled scores of pattern selection (Mode::kDensePool of
// attn_bf16_kernel.hpp): launch shape and launch.
#include "attn_bf16_kernel.hpp"

namespace sparsed {

// Rows per work-group: 256 (8 waves, one work-group per compute unit) or 128 (4 waves, two per compute unit); both are multiples
// of every block_q. Head dim 64: 128 while every work-group has a compute unit to itself (16 heads of 2048: 33.6 us, 41.3 with
// 256), beyond that as for the dense call that does not pool (dense_qtile_bf16; 32 heads of 2300, 1.1 rounds of 256 rows: 73 and
// 89 us, 16 heads of 3000, 0.75 rounds: 61 and 56). Head dim 128: the kernel of 128 rows is 8 to 19 % slower on a full chip
// (32 heads of 2300: 133 and 126 us, 28 of 1500: 53 and 46) and 3 to 10 % on an emptier one (4 of 6000: 140 and 130), but for
// the shortest sequences (16 of 256: 15.7 and 16.4).
DensePoolShape dense_pool_shape(int D, int B, int Hq, int L, int block_k, int max_rows) {
  DensePoolShape s;
  constexpr int kCus = 256;
  const bool alone = (int64_t)B * Hq * ((L + 127) / 128) <= kCus;
  const bool small = D == 128 ? alone && L <= 512 : alone || dense_qtile_bf16(D, (int64_t)B * Hq, L, false) <= 128;
  s.rows = max_rows < 256 || small ? 128 : 256;
  const int64_t units = (int64_t)B * Hq * ((L + s.rows - 1) / s.rows), resident = s.rows == 256 ? kCus : 2 * kCus;
  s.groups = (int)(units < resident ? units : resident);
  const int n = (L + kTileK - 1) / kTileK;  // key tiles; columns are stored in pairs, or once per tile pair
  s.slab_cols = block_k == kTileK / 2 ? 2 * n : block_k == kTileK ? (n + 1) & ~1 : (n + 1) >> 1;
  return s;
}

template <int D, int NW>
static hipError_t launch_nw(const AttnArgs& a, int groups, hipStream_t s) {
  const dim3 grid((unsigned)groups), block(NW * 64);
  switch (a.block_k) {
    case 32: hipLaunchKernelGGL((attn_bf16_kernel<D, 1, NW, Mode::kDensePool, 32>), grid, block, 0, s, a); break;
    case 64: hipLaunchKernelGGL((attn_bf16_kernel<D, 1, NW, Mode::kDensePool, 64>), grid, block, 0, s, a); break;
    case 128: hipLaunchKernelGGL((attn_bf16_kernel<D, 1, NW, Mode::kDensePool, 128>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_attn_bf16_dense_pool(int D, AttnArgs a, const DensePoolShape& sh, hipStream_t s) {
  a.n_qtiles = (a.L + sh.rows - 1) / sh.rows;
  a.slab_cols = sh.slab_cols;
  if ((int64_t)a.B * a.Hq * a.n_qtiles > 0x7fffffff - 1024 || !a.slab || !a.apool) return hipErrorInvalidValue;
  if (a.block_q != 32 && a.block_q != 64 && a.block_q != 128) return hipErrorInvalidValue;
  if (D == 128) return sh.rows == 256 ? launch_nw<128, 8>(a, sh.groups, s) : launch_nw<128, 4>(a, sh.groups, s);
  if (D == 64) return sh.rows == 256 ? launch_nw<64, 8>(a, sh.groups, s) : launch_nw<64, 4>(a, sh.groups, s);
  return hipErrorInvalidValue;
}

}  // namespace sparsed
