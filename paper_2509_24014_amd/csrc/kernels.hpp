// Internal interface between the host-side C ABI (api.hip) and the gfx950 kernels.
// Not installed; include/sparsed.h is the public boundary.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sparsed {

// One [B, H, L, D] operand: base pointer and element strides (stride of D is 1).
struct TensorArg {
  const void* ptr;
  int64_t sb, sh, sl;
};

// Arguments of the attention kernels (dense, sparse, and the statistics-only pass).
struct AttnArgs {
  TensorArg q, k, v;
  void* o;
  int64_t o_sb, o_sh, o_sl;
  float* lse;              // optional [B, Hq, L]: natural-log sum-exp of each row's scaled logits
  float* row_stat;         // optional [B, Hq, L, 2] (dense calls that splitk_takes): a row's reference in octaves, and 1 / its sum against that
  const int32_t* row_ptr;  // sparse only: [B, Hq, nqb + 1]
  const int32_t* col_idx;  // sparse only: [B, Hq, cap_per_head]
  int32_t B, Hq, group, L;  // group: query heads per key/value head
  const int32_t* seq_lens; // optional [B]: rows and keys of batch element b at or past seq_lens[b] do not exist
  int32_t nqb, cap_per_head, block_k;
  int32_t n_qtiles;        // query tiles per head = ceil(L / rows per work-group)
  float scale_log2;        // log2(e) / sqrt(D)
  int32_t block_q;         // rows per query block (sparse; kDensePool)
  // kDensePool only (nqb, block_q and block_k then describe the pooled blocks)
  float* slab;             // scratch: one slab of (rows per work-group) x slab_cols floats per work-group of the launch
  float* apool;            // [B, Hq, nqb, nkb] pooled scores
  int32_t slab_cols, nkb;
  // kDensePool of fp32 only: where the kept blocks go if the kernel ranks its rows itself (ranks_own_rows), else null; the
  // capacity per head is cap_per_head
  int32_t *row_ptr_out, *col_idx_out;
  double rho;
};

// Arguments of the pooled-score kernels (Section 3.3: A' = avgpool(A, block)). The keys pooled are
// the tokens [key_begin, key_begin + key_len), cut into blocks of block_k from key_begin on (the whole
// sequence for plain selection; one part of the block that holds the prefill boundary otherwise).
struct PoolArgs {
  TensorArg q, k;
  const float* lse;        // [B, Hq, L] natural-log sum-exp of each row over ALL L keys
  const float* row_stat;   // bf16: instead of lse, as AttnArgs::row_stat
  float* apool;            // [B, Hq, nqb, out_stride]; block t of the range lands in column t
  int32_t B, Hq, group, L;  // group: query heads per key/value head
  const int32_t* seq_lens; // optional [B] per-sample lengths (they cut the key ranges too)
  int32_t nqb, block_k;
  int32_t key_begin, key_len;
  int32_t key_len2;        // > 0: a second range, the key_len2 tokens behind the first, pooled into column 1 (a
                           // grid of two rows; both parts of the block that holds the prefill boundary in one launch)
  int32_t seg_len;         // set by the bf16 launcher: > 0: the range is cut into segments of so many tokens, one per grid row
  int32_t out_stride;
  float scale_log2;        // log2(e) / sqrt(D)
  // one-pass form only (pool1p_bf16_kernel; whole key range, lse unused):
  float* slab;             // scratch, one slab of 128 x slab_ld floats per work-group of the launch
  int32_t slab_ld;         // columns of a slab: the key-block count rounded up to a multiple of 16
  float* part;             // optional [B, Hq, nqb, 2]: the key block that holds the key token `boundary`, pooled over its keys
  int32_t boundary;        // before that token and over the others (rows of samples that end before the token: not written)
};

// Arguments of the per-row top-k kernel (Eq. 6): one wavefront per pooled row.
struct TopkArgs {
  const float* apool;      // [rows, nkb]
  int32_t* row_ptr;        // [B*H, nqb + 1]
  int32_t* col_idx;        // [B*H, cap_per_head]
  int32_t rows, nqb, nkb;
  int32_t split;           // key blocks [0, split) and [split, nkb) are ranked separately
  int32_t keep_lo, keep_hi;  // kept in each range (keep_hi = 0 and split = nkb for one range)
  int32_t cap_per_head;
  // Prefill boundary inside key block `straddle` (else straddle < 0): that block enters the first range
  // with score part[2r] (its prefill keys) and the second with part[2r+1] (its generation keys); it is
  // listed once even if both keep it, so rows differ in length. Without rows_tmp (places_rows_itself) the kernel writes
  // the CSR; else entries go to rows_tmp [rows, keep_lo + keep_hi] and counts [rows], and compact_kernel builds it.
  // Per-sample lengths (optional): sample b ranks the key blocks it has, ceil(len/block_k) of them, with its own
  // counts kept_blocks(rho, size of each of its ranges), and its query blocks past ceil(len/block_q) get empty rows.
  const int32_t* seq_lens;
  int32_t heads_per_batch, block_q, block_k, L;
  double rho;
  int32_t straddle;
  int32_t boundary;        // the boundary's key token (only with straddle >= 0)
  const float* part;
  int32_t* rows_tmp;
  int32_t* counts;
};

// Builds row_ptr / col_idx of every head from fixed-stride rows and their lengths.
struct CompactArgs {
  const int32_t* rows_tmp;  // [heads * nqb, stride]
  const int32_t* counts;    // [heads * nqb]
  int32_t* row_ptr;         // [heads, nqb + 1]
  int32_t* col_idx;         // [heads, cap_per_head]
  int32_t heads, nqb, stride, cap_per_head;
};

struct ValidateArgs {
  const int32_t* row_ptr;
  const int32_t* col_idx;
  int32_t rows, nqb, nkb, cap_per_head;
  int32_t* bad;            // device counter of malformed rows
};

// Arguments of the fixed-pattern index builder (sliding window + attention sinks).
struct WindowArgs {
  int32_t* row_ptr;
  int32_t* col_idx;
  int32_t heads, nqb, nkb, block_q, block_k, L, cap_per_head;
  int32_t half_window;  // tokens on either side of a query that stay visible
  int32_t sink_blocks;  // leading key blocks that are always visible
};

// The (batch, head) slab that the work-groups of position `pos` in the launch order take. Every XCD walks a contiguous range
// of positions, and in plain order (batch outermost) that is one or two samples: of a padded batch, the XCDs with the
// longest sample finish last and the others wait. With per-sample lengths the samples therefore alternate inside every
// group of heads that shares K and V, so each XCD gets its share of each length. Both orders are the same two divisions,
// by other numbers.
// 3 samples (3000, 2100, 1200) x 8 heads of 64, 128 x 128 blocks, 30 % kept: pooling 97 -> 62 us, sparse step 41 -> 24 us.
struct Slab {
  int b, h, hk;  // sample, query head, key/value head
};
template <typename Args>
__device__ __forceinline__ Slab slab_at(int pos, const Args& a) {
  const int group = a.group;
  const bool alternate = a.seq_lens != nullptr;
  const int outer = alternate ? a.B * group : a.Hq;
  const int x = pos / outer, rest = pos - x * outer, y = rest / group;
  return alternate ? Slab{y, x * group + rest - y * group, x} : Slab{x, rest, y};
}

// The kernel's argument struct (its only argument), read from the argument segment at the point of the call. Reading
// it again where it is used late keeps two dozen scalars from living, or being spilled into vector registers, in between.
template <typename Args>
using KernelArgs = const __attribute__((address_space(4))) Args;
template <typename Args>
__device__ __forceinline__ KernelArgs<Args>& fresh_kernel_args() {
  auto p = (KernelArgs<Args>*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *p;
}

enum class Mode : int { kDense = 0, kSparse = 1, kStats = 2, kDensePool = 3 };

// Launchers. Each returns the HIP error of the launch. block_q selects the work-group shape for
// the sparse and pooled kernels; dense and stats pick their own query tile from L.
hipError_t launch_attn_bf16(Mode mode, int D, int block_q, AttnArgs a, hipStream_t s);
hipError_t launch_attn_f32(Mode mode, int D, int block_q, AttnArgs a, hipStream_t s);
// bf16 attention with the keys split over the waves of a work-group (a.block_q set; block_q = 0 for dense), and the calls it
// is for: sparse with query blocks of 32 or 64 rows, dense and sparse calls with few rows in all.
bool splitk_takes(Mode mode, int D, int block_q, const AttnArgs& a);
hipError_t launch_attn_bf16_splitk(Mode mode, int D, int block_q, const AttnArgs& a, hipStream_t s);
// The dense call that also pools (bf16): shape of its launch for q [B, Hq, L, .] and blocks of block_q x block_k, and the
// launch itself (a.slab of groups * rows * slab_cols floats, a.apool, a.nqb, a.nkb, a.block_q, a.block_k set by the caller).
struct DensePoolShape {
  int rows;       // query rows per work-group: a multiple of every block_q
  int groups;     // persistent work-groups
  int slab_cols;  // columns of a work-group's slab
};
DensePoolShape dense_pool_shape(int D, int B, int Hq, int L, int block_k, int max_rows);  // max_rows: 256 or 128
hipError_t launch_attn_bf16_dense_pool(int D, AttnArgs a, const DensePoolShape& sh, hipStream_t s);
// The same for fp32 (a.apool, a.nqb, a.nkb, a.block_q, a.block_k set by the caller; no scratch), and whether it is the form for
// a call with heads = B * Hq (else: the dense call with its log-sum-exp, then pooling with it).
hipError_t launch_attn_f32_dense_pool(int D, AttnArgs a, hipStream_t s);
bool dense_pool_pays_f32(int D, int64_t heads, int L, int block_q, int block_k);
// Whether that launch is to rank the rows as well (a.row_ptr_out, a.col_idx_out, a.cap_per_head and a.rho set), or launch_topk after it.
bool ranks_own_rows_f32(int64_t heads, int nqb, int nkb, int block_q);
hipError_t launch_pool_bf16(int D, int block_q, const PoolArgs& a, hipStream_t s);
hipError_t launch_pool_f32(int D, int block_q, const PoolArgs& a, hipStream_t s);
// Pooled scores of bf16 inputs in one pass over the keys (no row statistics needed): `groups` persistent work-groups,
// each with its own slab in a.slab. pool1p_groups: the number of work-groups that fills the chip for this block_q.
hipError_t launch_pool1p_bf16(int D, int block_q, const PoolArgs& a, int groups, hipStream_t s);
int pool1p_groups(int block_q);
// Units of work of that launch: runs of 128 consecutive rows of one head (one, two or four query blocks).
int64_t pool1p_units(int B, int Hq, int nqb, int block_q);
hipError_t launch_topk(const TopkArgs& a, hipStream_t s);
// Whether launch_topk is to write the CSR itself (rows_tmp null) where rows differ in length, or staged rows for launch_compact.
bool places_rows_itself(int nqb, int nkb);
hipError_t launch_compact(const CompactArgs& a, hipStream_t s);
hipError_t launch_validate(const ValidateArgs& a, hipStream_t s);
hipError_t launch_window_index(const WindowArgs& a, hipStream_t s);
// Row I of the window + sink pattern as two disjoint ascending runs of key blocks: the sink blocks
// [0, *sink_end) and the window blocks [*first, *last] that are not sinks already (empty if *first > *last).
// Shared by the host-side sizing and the kernel.
__host__ __device__ inline void window_row_runs(int I, int block_q, int block_k, int L, int half_window, int sink_blocks,
                                                int* sink_end, int* first, int* last) {
  long lo = (long)I * block_q - half_window, hi = (long)(I + 1) * block_q - 1 + half_window;
  if (lo < 0) lo = 0;
  if (hi > L - 1) hi = L - 1;
  const int nkb = (L + block_k - 1) / block_k;
  *sink_end = sink_blocks < nkb ? sink_blocks : nkb;
  *first = (int)(lo / block_k);
  *last = (int)(hi / block_k);
  if (*first < *sink_end) *first = *sink_end;
}
__host__ __device__ inline int window_row_length(int I, int block_q, int block_k, int L, int half_window, int sink_blocks) {
  int sink_end, first, last;
  window_row_runs(I, block_q, block_k, L, half_window, sink_blocks, &sink_end, &first, &last);
  return sink_end + (last >= first ? last - first + 1 : 0);
}
// Matrix-core rate probe: kProbeGroups work-groups x 8 waves, each wave issues 32 MFMAs per iteration.
constexpr int kProbeGroups = 256;
constexpr int kProbeFloats = kProbeGroups * 512;
hipError_t launch_mfma_rate(float* scratch, int iters, int random_operands, hipStream_t s);
// Vector-unit rate probe, same launch shape: each wave issues 64 fp32 instructions per iteration (op 0: fma, 1: exp2).
hipError_t launch_valu_rate(float* scratch, int iters, int op, hipStream_t s);
// Matrix instructions together with vector_per_mfma (0, 2, 3, 4, 5, 6 or 8) vector instructions each, a quarter of them
// exp2, and optionally one LDS operand read each; same launch shape and matrix work as launch_mfma_rate.
hipError_t launch_mix_rate(float* scratch, int iters, int vector_per_mfma, int lds_operands, hipStream_t s);

// Rows per work-group the bf16 dense / stats kernels use for heads = B * Hq and this L (0 if L is unsupported); padded: the samples
// have lengths of their own.
int dense_qtile_bf16(int D, int64_t heads, int L, bool padded);

}  // namespace sparsed
