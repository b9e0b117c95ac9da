// Dense, sparse and statistics launches of the bf16 attention kernel (attn_bf16_kernel.hpp).
#include "attn_bf16_kernel.hpp"

namespace sparsed {

// Rows per work-group of a call that walks every tile. 256 (8 waves, alone on a compute unit) copies a tile for twice the rows
// of 128 (4 waves, two work-groups a unit) and is the faster form of a chip that is full for the whole launch: 5 % at head dim
// 128, 1 to 4 % at 64. But its launch ends with a round of its own length, however few units have work in it, where a 128-row
// work-group that is alone on its unit takes 0.7 of a pair's time. Dense, us, 256 -> 128 rows, 1.1, 1.25, 1.5, 2.25, 3.1, 4.1
// rounds of 256: head dim 64 143 -> 122, 157 -> 135, 98 -> 87, 219 -> 198, 405 -> 376, 755 -> 716; 128 210 -> 184, 232 -> 206,
// 145 -> 139, 336 -> 314, 630 -> 601, 1182 -> 1154; above half a round left over, 256 rows throughout. (A length that is a
// multiple of 64 and not of 128 once had work-groups of 64 rows, two waves: 16 heads of 3776 x 128 148 us, 102 with 256 rows.)
// With lengths per sample (`padded`) the rounds of full samples are no more than a guess: the forms that lose least by a wrong one,
// 128 rows below 1024 tokens at head dim 64 (by rounds 0.80 to 1.20 times the time of what was taken before there were rounds, so
// 0.68 to 1.03), 256 rows from there to 4096 tokens (0.92 to 1.08, so 0.99 to 1.02); longer ones by rounds (0.82 to 1.05).
int dense_qtile_bf16(int D, int64_t heads, int L, bool padded) {
  if (L <= 0) return 0;
  if (L <= 64) return 64;
  if (padded && L < 1024 && D == 64) return 128;
  if (padded && L >= 1024 && L < 4096) return 256;
  constexpr int64_t kCus = 256;
  const int64_t n256 = heads * ((L + 255) / 256), n128 = heads * ((L + 127) / 128), left = n128 % (2 * kCus);
  const int64_t cost256 = (n256 + kCus - 1) / kCus * 1000;
  const int64_t cost128 = (n128 / (2 * kCus) * 10 + (left == 0 ? 0 : left <= kCus ? 7 : 10)) * (D == 64 ? 101 : 105);
  return cost128 < cost256 ? 128 : 256;
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
  const int qtile = (mode == Mode::kSparse) ? block_q : dense_qtile_bf16(D, (int64_t)a.B * a.Hq, a.L, a.seq_lens != nullptr);
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
