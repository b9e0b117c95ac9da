// Dense, sparse and statistics launches of the bf16 attention kernel (attn_bf16_kernel.hpp).
#include "attn_bf16_kernel.hpp"

namespace sparsed {

int dense_qtile_bf16(int L) {
  if (L <= 0) return 0;
  if (L % 256 == 0) return 256;
  if (L % 128 == 0) return 128;
  if (L % 64 == 0) return 64;
  return L >= 1024 ? 256 : L >= 256 ? 128 : 64;  // partial last tile: waste at most one tile of rows
}

template <int D, int NQ, int NW, Mode MODE, int KB = kTileK>
static hipError_t launch_one(const AttnArgs& a, hipStream_t s) {
  const int64_t total = (int64_t)a.B * a.Hq * a.n_qtiles;
  if (total <= 0 || total > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid((unsigned)total), block(NW * 64);
  hipLaunchKernelGGL((attn_bf16_kernel<D, NQ, NW, MODE, KB>), grid, block, 0, s, a);
  return hipGetLastError();
}

template <int D, Mode MODE>
static hipError_t launch_by_qtile(int qtile, const AttnArgs& a, hipStream_t s) {
  switch (qtile) {
    case 256: return launch_one<D, 1, 8, MODE>(a, s);
    case 128:
      if (MODE == Mode::kSparse && a.block_k == 2 * kTileK) return launch_one<D, 1, 4, MODE, 2 * kTileK>(a, s);
      if (MODE == Mode::kSparse && a.block_k == kTileK / 2) return launch_one<D, 1, 4, MODE, kTileK / 2>(a, s);
      return launch_one<D, 1, 4, MODE>(a, s);
    case 64: return launch_one<D, 1, 2, MODE>(a, s);
    case 32: return launch_one<D, 1, 1, MODE>(a, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_attn_bf16(Mode mode, int D, int block_q, AttnArgs a, hipStream_t s) {
  const int qtile = (mode == Mode::kSparse) ? block_q : dense_qtile_bf16(a.L);
  if (qtile == 0) return hipErrorInvalidValue;
  a.n_qtiles = (a.L + qtile - 1) / qtile;
  a.block_q = block_q;
  if (splitk_takes(mode, D, block_q, a)) return launch_attn_bf16_splitk(mode, D, block_q, a, s);
  if (D == 128) {
    if (mode == Mode::kDense) return launch_by_qtile<128, Mode::kDense>(qtile, a, s);
    if (mode == Mode::kSparse) return launch_by_qtile<128, Mode::kSparse>(qtile, a, s);
    return launch_by_qtile<128, Mode::kStats>(qtile, a, s);
  }
  if (D == 64) {
    if (mode == Mode::kDense) return launch_by_qtile<64, Mode::kDense>(qtile, a, s);
    if (mode == Mode::kSparse) return launch_by_qtile<64, Mode::kSparse>(qtile, a, s);
    return launch_by_qtile<64, Mode::kStats>(qtile, a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace sparsed
