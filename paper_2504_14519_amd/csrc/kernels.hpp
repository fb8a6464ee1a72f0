// Host-visible argument blocks and launchers of the gfx950 kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace slimpipe {

// The cached keys / values as the paper stores them (Sec. 5): a list of slice-sized chunks rather than
// one buffer.  Row j of the prefix is row j % len of chunk j / len; inside a chunk rows follow the kv
// strides.  A contiguous prefix is the list of one chunk (any length).  With more than one chunk `len`
// is a multiple of 256 and the kernels walk key tiles on an absolute grid, so that no tile straddles two
// chunks.
constexpr int kMaxChunks = 64;
struct KvChunks {
  const __bf16* k[kMaxChunks];
  const __bf16* v[kMaxChunks];
  int64_t len;
  int32_t n;
};
// keys one workgroup of the dk/dv kernel owns
inline __host__ __device__ constexpr int dkdv_keys_per_workgroup() { return 8 * 32; }
// first key of the tile grid for tiles of `tile` keys
inline __host__ __device__ int64_t kv_grid_origin(int64_t kv_begin, int32_t n_chunks, int tile) {
  return n_chunks > 1 ? kv_begin / tile * tile : kv_begin;
}

// Key ranges one forward launch covers (paper Sec. 4.2.2: the pieces of a context exchange).  Range r
// of a launch writes its (out, lse) at out + r * out_range_stride, lse + r * lse_range_stride.
constexpr int kMaxRanges = 16;

// Query blocks.  A forward / dq workgroup is 8 waves of 32 query rows.  The waves of all query heads that share a
// K/V head are numbered through, head_waves per head, and cut into blocks of 8.  head_waves is the host's choice: a multiple of
// 8 gives every head blocks of its own, the last one with waves past the slice; ceil(s_q / 32) packs the heads, so that only
// the last block of a K/V head can hold waves without rows (777 rows, 8 heads on one K/V head: 25 blocks instead of 32).
inline __host__ __device__ int packed_head_waves(int s_q) { return (int)(((unsigned)s_q + 31u) / 32u); }
inline __host__ __device__ int padded_head_waves(int s_q) { return (int)(((unsigned)s_q + 255u) / 256u * 8u); }
inline __host__ __device__ int64_t query_blocks(int head_waves, int group) { return ((int64_t)group * head_waves + 7) / 8; }

// The memory from the first element of a [batch, rows, heads, head_dim] tensor (strides in elements, all positive) to its last.
struct Span {
  uintptr_t begin, end;      // [begin, end); empty without elements
};
inline Span span_of(const void* first, int64_t elem_bytes, int64_t batch, int64_t rows, int64_t heads, int64_t head_dim, int64_t stride_b, int64_t stride_s,
                    int64_t stride_h) {
  const uintptr_t p = reinterpret_cast<uintptr_t>(first);
  if (batch < 1 || rows < 1 || heads < 1 || head_dim < 1) return {p, p};
  return {p, p + (uintptr_t)(((batch - 1) * stride_b + (rows - 1) * stride_s + (heads - 1) * stride_h + head_dim) * elem_bytes)};
}
inline bool share_memory(const Span& a, const Span& b) { return a.begin < a.end && b.begin < b.end && a.begin < b.end && b.begin < a.end; }

struct FwdArgs {
  const __bf16* q;
  KvChunks kv;
  void* out;
  float* lse;
  int32_t s_q, n_q_heads, group, causal, out_f32;
  int32_t n_ranges;                                   // >= 1; third item coordinate = batch index * n_ranges + range
  // [range_begin, range_end): without the keys behind the last one that any row sees.  No key outside is read (rows of a tile that
  // lie outside are clamped): the cache may hold anything there, and a weight of 0 times a NaN is a NaN
  int64_t range_begin[kMaxRanges], range_end[kMaxRanges];
  int64_t out_range_stride, lse_range_stride;         // in elements of the output type / floats
  // work items = (query block, kv head, batch index x range), items[0] * [1] * [2] of them; with `ticket` (eight counters
  // set to zero before the launch, one per XCD) the grid holds more workgroups than items and each takes the next item
  // from the counters (see next_item and BwdArgs::ticket_dkdv); nullptr: workgroup index = item
  unsigned* ticket;
  int32_t items[3];
  int32_t items_by_group;      // an XCD takes all query blocks of a (head, batch index x range) (see next_item)
  int32_t head_waves;          // of the query blocks
  int64_t q_offset, kv_capacity;
  float scale_log2e;
  int64_t q_stride_b, q_stride_s, q_stride_h;
  int64_t kv_stride_b, kv_stride_s, kv_stride_h;
  int64_t o_stride_b, o_stride_s, o_stride_h;
};

struct BwdArgs {
  const __bf16* q;
  KvChunks kv;
  const __bf16* out;
  const __bf16* d_out;
  const float* lse;
  float* delta;            // workspace [batch, n_q_heads, s_q]: -rowsum(dO * O) (negated: initial accumulator of dP in dk/dv)
  float* lse2;             // workspace [batch, n_q_heads, s_q]: lse * log2(e), +inf where lse = -inf
  void* dq;
  float* dk_acc[kMaxChunks];   // float32 accumulators, chunked like the keys / values
  float* dv_acc[kMaxChunks];
  float* part;             // workspace [n_split][2][batch][n_kv_heads][nkeys_pad][head_dim]: partial dk, dv (n_split > 1)
  // dq kernel: key ranges of one launch (third item coordinate = batch index * n_dq_ranges + range).  With one range dq is the
  // caller's buffer; with several it is the float32 workspace [range][batch, s_q, heads, head_dim] that
  // dq_reduce_kernel adds up into dq_final.
  int32_t n_dq_ranges;
  int64_t dq_range_begin[kMaxRanges], dq_range_end[kMaxRanges];      // (as in FwdArgs)
  int64_t dq_range_stride;                       // elements between the partial dq of two ranges
  int64_t dq_stride_b, dq_stride_s, dq_stride_h; // of `dq` as the dq kernel writes it
  void* dq_final;                                // the caller's dq (q strides) when n_dq_ranges > 1
  int32_t dq_final_f32, dq_final_accumulate;
  int32_t n_split;         // chunks the query stream of a key tile is cut into (one workgroup each)
  int64_t nkeys_pad;       // key rows per (batch, kv head) plane of `part`
  // dk/dv work items = (key tile x chunk, kv head, batch index), dkdv_items[0] * [1] * [2] of them.  With `ticket`
  // (a counter in the workspace that the delta kernel sets to zero) workgroups take the next item from the counter
  // instead of deriving it from their index: the hardware hands workgroups to the eight XCDs round-robin whatever
  // their speed, and this lets a faster XCD take more items.  The dk/dv launch then has dkdv_wgs workgroups (one per
  // compute unit) that loop over items, with ticket_dkdv[0..7] one counter per XCD; the dq launch has a quarter more
  // workgroups than items, one item each, and eight counters too.
  // nullptr: workgroup index = item (no room for the counters in the workspace, or no more items than compute units, when
  // every workgroup starts at once and there is nothing to even out, or dq and dk/dv in one launch).
  unsigned* ticket_dkdv;
  unsigned* ticket_dq;
  int32_t dkdv_wgs;
  int32_t dkdv_items[3];
  int32_t items_by_group;   // of the dq launch, as in FwdArgs
  int32_t head_waves;       // of the dq query blocks, as in FwdArgs
  int32_t dq_first;         // dq and dk/dv in one launch: the dq items come first
  int32_t dq_items[3];      // dq work items = (query block, kv head, batch index x key range), handed out the same way
  int32_t s_q, n_q_heads, n_kv_heads, group, causal;
  int32_t dq_f32, dq_accumulate, dkv_accumulate;
  int64_t q_offset, kv_begin, kv_end, kv_capacity;
  int64_t seen_end;         // keys of [seen_end, kv_end) are seen by no row: their dk, dv are 0, whatever the cache holds there
  float scale, scale_log2e;
  int64_t q_stride_b, q_stride_s, q_stride_h;
  int64_t kv_stride_b, kv_stride_s, kv_stride_h;
  int64_t o_stride_b, o_stride_s, o_stride_h;
  int64_t do_stride_b, do_stride_s, do_stride_h;
  int32_t dq_tile_keys, dkdv_tile_rows;      // keys of a dq tile, query rows of a dk/dv tile (head_dim 64 has two of each)
};

struct MergeArgs {
  const void* outs[16];
  const float* lses[16];
  int32_t n_parts, part_f32, out_f32, head_dim, n_q_heads, s_q;
  int64_t rows;            // batch * s_q
  void* out;               // strides o_* (parts are contiguous [batch, s_q, heads, head_dim])
  float* lse;
  int64_t o_stride_b, o_stride_s, o_stride_h;
};

// The attention kernels use more than 64 KB of dynamic LDS, which a kernel has to be allowed once per device
// (hipFuncSetAttribute; the attribute belongs to the function on the CURRENT device).  These two set it for
// every instantiation of the forward / backward kernels; api.hip calls them once per device.
hipError_t opt_in_fwd_kernels();
hipError_t opt_in_bwd_kernels();
hipError_t opt_in_small_kernels();

hipError_t launch_fwd(const FwdArgs& a, int batch, int head_dim, hipStream_t st);
hipError_t launch_fwd_small(const FwdArgs& a, int batch, int head_dim, hipStream_t st);
hipError_t launch_zero_counters(unsigned* counters, hipStream_t st);
hipError_t launch_delta(const BwdArgs& a, int batch, int head_dim, hipStream_t st);
hipError_t launch_bwd_dq(const BwdArgs& a, int batch, int head_dim, hipStream_t st);
hipError_t launch_bwd_dkdv(const BwdArgs& a, int batch, int head_dim, hipStream_t st);
hipError_t launch_dkdv_reduce(const BwdArgs& a, int batch, int head_dim, hipStream_t st);
hipError_t launch_dq_reduce(const BwdArgs& a, int batch, int head_dim, hipStream_t st);
hipError_t launch_bwd_both(const BwdArgs& a, int head_dim, hipStream_t st);
int small_dq_tile_keys(int head_dim);
// own_stats: no delta launch before; key_blocks: of 32 keys that a dk/dv item owns (1; head_dim 64: or 2)
hipError_t launch_bwd_small(const BwdArgs& a, int batch, int head_dim, bool own_stats, int key_blocks, hipStream_t st);
hipError_t launch_both_reduce(const BwdArgs& a, int batch, int head_dim, hipStream_t st);
hipError_t launch_merge(const MergeArgs& a, hipStream_t st);
hipError_t launch_finalize(const float* acc, __bf16* dst, int64_t n, hipStream_t st);
hipError_t launch_dq_atomic_probe(float* dq, int s_q, int heads, int key_tiles, int rows_per_step, int placement, int rotate,
                                  int filler_mfma, int with_atomics, unsigned* xcc_mismatch, hipStream_t st);
hipError_t launch_xcd_rate(int iters, int workgroups, long long* t_start, long long* t_end, unsigned* xcc, hipStream_t st);
hipError_t launch_mfma_rate(int random, int iters, int workgroups, float* sink, hipStream_t st);

}  // namespace slimpipe
