// The ranking of one row of pooled scores by one wave (Eq. 6), for the kernel that does only that (select.hip) and for those that
// have just made the row.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sparsed {

// The host's count rule, in the same double arithmetic.
__device__ __forceinline__ int kept_blocks_of(double rho, int nblocks) {
  if (nblocks <= 0) return 0;
  double x = ceil(rho * (double)nblocks - 1e-9);
  if (!(x >= 1.0)) x = 1.0;
  if (x > (double)nblocks) x = (double)nblocks;
  return (int)x;
}

// Scores are non-negative floats, so their bit patterns order like unsigned integers. For one range [lo, hi) of the row: a
// descent over the bits finds the keep-th largest value T and how many entries equal to T are still needed (it ends
// early once a threshold is met by exactly `keep` entries); then one ascending sweep emits every entry above T plus the
// first `need` entries equal to T (lower block index wins ties).
// Bound: latency. The descent is a chain of up to 32 compare - count - branch steps; a row of up to 64 * R entries stays
// in R registers a lane, so that a step does not wait for LDS reads. Rows longer than the widest register form (16) are
// held in LDS (R = 0). 8192 rows of 256 entries: 40.8 -> 20.8 us;
// 576 rows of at most 25 entries in two ranges: 12.0 -> 5.9 us; 16 rows of 8: 6.3 -> 3.4 us. (Before: every row in LDS, all 32 steps.)
template <int R>
struct TopkRow {
  uint32_t x[R > 0 ? R : 1];
  uint32_t* lds;  // R = 0: the row; else unused
  int lane;
  template <typename Get>
  __device__ __forceinline__ void load(int n, Get get) {
    if constexpr (R > 0) {
#pragma unroll
      for (int r = 0; r < R; ++r) x[r] = r * 64 + lane < n ? get(r * 64 + lane) : 0u;
    } else {
      for (int J = lane; J < n; J += 64) lds[J] = get(J);
      __syncthreads();
    }
  }
  // visit(J, value, exists) for this lane's entry of every 64-entry chunk that meets [lo, hi), in ascending order
  template <typename Visit>
  __device__ __forceinline__ void chunks(int lo, int hi, Visit visit) const {
    if constexpr (R > 0) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int J = r * 64 + lane;
        if (r * 64 < hi && r * 64 + 64 > lo) visit(J, x[r], J >= lo && J < hi);
      }
    } else {
      for (int base = lo; base < hi; base += 64) {
        const int J = base + lane;
        visit(J, lds[J < hi ? J : lo], J < hi);
      }
    }
  }
  __device__ __forceinline__ void emit(int lo, int hi, int keep, int32_t* out) const {
    if (keep <= 0 || hi <= lo) return;
    uint32_t T = 0;
    int need = 0;       // entries equal to T to take
    bool exact = false;  // exactly `keep` entries lie above T
    for (int bit = 31; bit >= 0; --bit) {
      const uint32_t cand = T | (1u << bit);
      int cnt = 0;
      chunks(lo, hi, [&](int, uint32_t v, bool exists) { cnt += __builtin_popcountll(__ballot(exists && v >= cand)); });
      if (cnt == keep) {
        T = cand - 1;
        exact = true;
        break;
      }
      if (cnt > keep) T = cand;
    }
    if (!exact) {
      int above = 0;
      chunks(lo, hi, [&](int, uint32_t v, bool exists) { above += __builtin_popcountll(__ballot(exists && v > T)); });
      need = keep - above;
    }
    const unsigned long long lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    int n_out = 0, eq_seen = 0;
    chunks(lo, hi, [&](int J, uint32_t v, bool exists) {
      const bool gt = exists && v > T;
      const bool eq = exists && v == T;
      const unsigned long long eq_mask = __ballot(eq);
      const int eq_rank = eq_seen + __builtin_popcountll(eq_mask & lt_mask);
      const bool take = gt || (eq && eq_rank < need);
      const unsigned long long take_mask = __ballot(take);
      if (take) out[n_out + __builtin_popcountll(take_mask & lt_mask)] = J;
      n_out += __builtin_popcountll(take_mask);
      eq_seen += __builtin_popcountll(eq_mask);
    });
  }
};

}  // namespace sparsed
