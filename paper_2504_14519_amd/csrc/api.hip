// C ABI of the library: host-only validation, launch planning, error mapping.
#include <math.h>
#include <string.h>

#include <atomic>
#include <mutex>
#include <vector>

#include "../../include/slimpipe_attn.h"
#include "../../include/slimpipe_attn_bench.h"
#include "kernels.hpp"

using namespace slimpipe;

// Fixed device memory of the entry point that allocates nothing (slimpipe_attn_bwd_noalloc): the backward's row
// statistics live here instead of in a caller's workspace.  Every GPU the library runs on holds its own copy
// until the process ends.  Host code never uses this name as an address: it asks the runtime for the device
// address once per device (ensure_device_ready) and passes that pointer to the kernels.
constexpr size_t kScratchBytes = (size_t)4 << 20;          // the two statistics arrays
constexpr size_t kScratchTicketBytes = 256;                // + the counters the workgroups take their work items from
static __device__ __align__(256) unsigned char scratch[kScratchBytes + kScratchTicketBytes];

namespace {

bool stride_ok(int64_t s) { return s > 0 && (s % 8) == 0; }
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// one float array per row statistic (delta, lse in log2 units), each rounded up to 256 bytes
size_t stat_bytes(const slimpipe_attn_params* p) {
  size_t n = (size_t)p->batch * (size_t)p->n_q_heads * (size_t)p->s_q * sizeof(float);
  return (n + 255) & ~(size_t)255;
}
size_t delta_bytes(const slimpipe_attn_params* p) { return 2 * stat_bytes(p); }

// ---- per-device state: the only state the library keeps besides the benchmark's profiling switch ----
// For each device the dynamic-LDS opt-in of the kernels (done once, under std::call_once) and the number of
// compute units.  Both are functions of the device alone, so concurrent callers agree on them.
constexpr int kMaxDevices = 64;
struct DeviceState {
  std::once_flag once;
  hipError_t status = hipSuccess;
  void* scratch = nullptr;       // this device's copy of `scratch` below (its address differs from device to device)
};
DeviceState g_device[kMaxDevices];
std::atomic<int> g_compute_units[kMaxDevices];

// Makes the current device ready for launches: SLIMPIPE_OK, or SLIMPIPE_ELAUNCH when the runtime refuses.
int ensure_device_ready(void** scratch_ptr = nullptr) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SLIMPIPE_ELAUNCH;
  DeviceState& d = g_device[dev];
  std::call_once(d.once, [&d] {
    d.status = opt_in_fwd_kernels();
    if (d.status == hipSuccess) d.status = opt_in_bwd_kernels();
    if (d.status == hipSuccess) d.status = opt_in_small_kernels();
    if (d.status == hipSuccess) d.status = hipGetSymbolAddress(&d.scratch, HIP_SYMBOL(scratch));
    if (d.status == hipSuccess && d.scratch == nullptr) d.status = hipErrorInvalidSymbol;
  });
  if (scratch_ptr) *scratch_ptr = d.scratch;
  return d.status == hipSuccess ? SLIMPIPE_OK : SLIMPIPE_ELAUNCH;
}

// Compute units of the current device (256 on MI355X, also assumed when no device can be asked, so that the
// workspace query stays a pure host function).
int compute_units() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
  int cus = g_compute_units[dev].load(std::memory_order_relaxed);
  if (cus > 0) return cus;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return 256;
  g_compute_units[dev].store(cus, std::memory_order_relaxed);
  return cus;
}

// The dk/dv kernel runs one workgroup per compute unit; a call with W key tiles takes ceil(W / CUs)
// rounds of one tile's query stream each.  Cutting every stream into S chunks makes W*S workgroups of
// 1/S the length: S is the smallest of 1, 2, 4, 8 that comes within 3% of the best rounds/S, as long
// as a chunk keeps at least 64 query tiles (the prologue and epilogue of a workgroup cost a few tiles).
int64_t dkdv_key_tiles(const slimpipe_attn_params* p, int n_chunks) {
  if (p->kv_end <= p->kv_begin) return 0;
  const int64_t per = dkdv_keys_per_workgroup();
  return (p->kv_end - kv_grid_origin(p->kv_begin, n_chunks, (int)per) + per - 1) / per;
}
int preferred_split(const slimpipe_attn_params* p, int n_chunks, bool ticket) {
  const int64_t tiles = dkdv_key_tiles(p, n_chunks);
  const int64_t w = tiles * p->n_kv_heads * p->batch;
  if (w <= 0) return 1;
  const int64_t stream = ((int64_t)p->s_q + 31) / 32 * (p->n_q_heads / p->n_kv_heads);
  const int cus = compute_units();
  double best = 1e30;
  double cost[4];
  for (int i = 0; i < 4; ++i) {
    const int s = 1 << i;
    cost[i] = (s > 1 && stream / s < 64) ? 1e30 : (double)((w * s + cus - 1) / cus) / s;
    if (cost[i] < best) best = cost[i];
  }
  int split = 1;
  for (int i = 3; i >= 0; --i)
    if (cost[i] <= best * 1.03) split = 1 << i;
  // Items handed out through a counter: a compute unit that finishes early takes another one, so more items even out
  // compute units (and XCDs) of unequal speed and key tiles of unequal streams (the causal diagonal).  Up to about 8
  // items per compute unit, as long as a chunk keeps at least 512 query tiles (a workgroup's prologue and epilogue
  // cost about 8 tiles' time, and every chunk adds a plane of partial sums to the reduce kernel's work).
  // And no split for the sake of whole rounds once there are two items per compute unit anyway: the counter evens out
  // most of what the rounding would cost, and the partial sums with their reduce kernel cost more than the rest.
  if (ticket) {
    if (w >= 2 * (int64_t)cus) split = 1;
    while (split < 8 && w * split < 8 * (int64_t)cus && stream / (2 * split) >= 512) split *= 2;
  }
  return split;
}
// room for the ticket counter of the dk/dv kernel behind the two statistics arrays
constexpr size_t kTicketBytes = 256;
size_t split_bytes(const slimpipe_attn_params* p, int n_chunks, int split) {
  if (split <= 1) return 0;
  return (size_t)split * 2 * (size_t)p->batch * (size_t)p->n_kv_heads *
         (size_t)(dkdv_key_tiles(p, n_chunks) * dkdv_keys_per_workgroup()) * (size_t)p->head_dim * sizeof(float);
}

// ---- key ranges of one forward launch --------------------------------------------------------------
// Visible (query, key) pairs of the call with keys in [p->kv_begin, e).
double visible_pairs_upto(const slimpipe_attn_params* p, int64_t e) {
  if (e > p->kv_end) e = p->kv_end;
  if (e <= p->kv_begin) return 0.0;
  const int64_t s = p->s_q;
  if (!p->causal) return (double)s * (double)(e - p->kv_begin);
  // row i sees keys below q_offset + i + 1: rows from i0 on see all of [kv_begin, e), rows i1 .. i0-1 a part
  int64_t i0 = e - p->q_offset - 1;
  i0 = i0 < 0 ? 0 : (i0 > s ? s : i0);
  int64_t i1 = p->kv_begin - p->q_offset;
  i1 = i1 < 0 ? 0 : (i1 > i0 ? i0 : i1);
  const double full = (double)(s - i0) * (double)(e - p->kv_begin);
  const double cnt = (double)(i0 - i1);
  const double first = (double)(p->q_offset + i1 + 1 - p->kv_begin), last = (double)(p->q_offset + i0 - p->kv_begin);
  return full + (cnt > 0 ? 0.5 * cnt * (first + last) : 0.0);
}

// How the query rows are cut into blocks (see kernels.hpp) for a call on `keys` keys that may be cut into up to `ranges` key
// ranges.  Heads are packed where that takes a tenth of the blocks or more, the blocks (times the ranges) fill the chip, so that
// fewer blocks are fewer rounds or more ranges, and little of the work is at the causal diagonal: a block that holds the end
// of one head and the start of the next walks the keys of the one with masked tiles for the other (about 1.1 us per 128-key
// tile of the forward), and on an idle chip 8 full waves load and store 2 to 3 us longer than 2.  Packed against padded over
// 160 shapes: where the rule packs, forward 0.68 to 1.00 and backward call 0.69 to 1.00 of the time (777 rows on 33777 keys 0.88
// and 0.86); packing everything costs up to 1.45 (4679 rows on 8817 keys, 4/1 heads of 64: 87 against 127 us).
int head_waves_of(const slimpipe_attn_params* p, int64_t keys, int ranges) {
  const int packed = packed_head_waves(p->s_q), padded = padded_head_waves(p->s_q), group = p->n_q_heads / p->n_kv_heads;
  const int64_t rows_packed = query_blocks(packed, group), rows_padded = query_blocks(padded, group);
  const bool pack = 10 * rows_packed <= 9 * rows_padded && (!p->causal || keys >= 12 * (int64_t)p->s_q) &&
                    rows_padded * p->n_kv_heads * p->batch * ranges >= compute_units();
  return pack ? packed : padded;
}
// Key ranges of at least min_keys a call can be cut into.
int most_ranges(const slimpipe_attn_params* p, int64_t min_keys) {
  const int64_t r = (p->kv_end - p->kv_begin) / min_keys;
  return r < 1 ? 1 : (r > kMaxRanges ? kMaxRanges : (int)r);
}
constexpr int64_t min_range_keys(int head_dim) { return head_dim == 64 ? 256 : 1024; }
int64_t all_query_blocks(const slimpipe_attn_params* p, int head_waves) {
  return query_blocks(head_waves, p->n_q_heads / p->n_kv_heads) * p->n_kv_heads * p->batch;
}

// Microseconds of a call with w < compute units query blocks of 256 rows in r key ranges (see fwd_preferred_ranges).
double fwd_blocks_us(const slimpipe_attn_params* p, int64_t cus, int64_t w, int r) {
  const int64_t keys = p->kv_end - p->kv_begin;
  return (double)((w * r + cus - 1) / cus) * (10.0 + (p->head_dim == 64 ? 1.8 : 2.5) * (double)keys / (128.0 * r)) +
         (r > 1 ? 4.5 + (double)(r + 1) * p->s_q * p->n_q_heads * p->batch * p->head_dim * 4 / 4e6 : 0.0);
}
// One forward workgroup owns 256 query rows and walks the whole key range; a short slice over a
// long cache leaves compute units idle.  Cutting the key range into R ranges of equal work (one launch,
// partial (out, lse) per range, then the online-softmax merge) makes R times the workgroups.  With a block per compute
// unit or more, R is the smallest count that comes within 3% of the best rounds/R, ranges keeping at least 1024 keys;
// with less, the smallest within 3% of the shortest time of the sum below, ranges keeping min_range_keys.
int fwd_preferred_ranges(const slimpipe_attn_params* p, int head_waves) {
  const int64_t w = all_query_blocks(p, head_waves);
  const int64_t keys = p->kv_end - p->kv_begin;
  if (w <= 0 || keys <= 0) return 1;
  const int cus = compute_units();
  // Less than one block per compute unit: every compute unit runs a chain of ceil(w r / CUs) items, each of about 10 us plus
  // 2.5 us (head_dim 128; 1.8 us at 64) per 128-key tile, and the merge is a launch of 4.5 us plus its bytes at 4 TB/s (fwd_blocks_us).
  // The tile times are those of a half-filled chip; measured are 2.2 us (32 items) to 3.4 us (247 items; 3.7 in short chains)
  // at head_dim 128 and 1.7 to 2.2 at 64, so the sum is a fifth to a quarter short where it fills the chip.  What counts is the pick:
  // over 35 shapes of 1 to 247 blocks, every count up to 16 timed, it is within 3% of the best allowed count in 30, and in
  // five small calls 15 ranges are taken where 16 cut the keys evenly (2 to 4 us).  With tile times that grow with the busy share (2.2 +
  // share) the sum comes within 15%, but the picks are the same on the 20 shapes it was fitted to and 0.6% slower at
  // head_dim 128 where they differ.  (By rounds alone 192 blocks of head_dim 64 on 4238 keys were cut into 4 ranges, three
  // full rounds, which took 262 us of a backward call instead of 220.)  Ranges of head_dim 64 may be as short as 256 keys:
  // 512 rows on 2048 keys and 4 heads are 8 blocks.
  if (w < cus) {
    int pick = 1;
    double best_us = 1e30;
    for (int r = 1; r <= kMaxRanges && (r == 1 || keys / r >= min_range_keys(p->head_dim)) && (int64_t)p->batch * r <= 65535; ++r) {
      const double us = fwd_blocks_us(p, cus, w, r);
      if (us < best_us * 0.97) { best_us = us; pick = r; }
    }
    return pick;
  }
  double best = 1e30, cost[kMaxRanges + 1];
  for (int r = 1; r <= kMaxRanges; ++r) {
    // (a range keeps at least 1024 keys; batch * ranges is the grid's z dimension)
    cost[r] = (r > 1 && (keys / r < 1024 || (int64_t)p->batch * r > 65535)) ? 1e30 : (double)((w * r + cus - 1) / cus) / r;
    if (cost[r] < best) best = cost[r];
  }
  for (int r = 1; r <= kMaxRanges; ++r)
    if (cost[r] <= best * 1.03) return r;
  return 1;
}
// Whether the query blocks that share keys go to one XCD (next_item).  At least 8 groups of them read keys of their own, so
// that every XCD has one; with fewer, an XCD would be without, and the keys of so few groups are streamed by
// all L2s at a rate the memory-side cache does not notice (0.2 TB/s at one K/V head against 2.4 at 40).  And only for
// items that walk 3072 keys or more: a surplus workgroup finds all eight classes used up one after the other, about 10 us,
// which short items do not win back.  By group against one counter over 110 shapes: forward 0.80 to 1.02 of the time where the rule
// says yes (16/16 heads of 128, 2 x 6089 rows on 10389 keys 718 -> 674 us; 40/40 heads, 4096 rows on 20480 keys in 2 ranges 1395 ->
// 1368), but up to 1.15 on shorter items (64/8 heads of 64, 4 x 307 rows on 858 keys; 40/40, 3 x 1367 rows on 7804 in 6 ranges 1.10).
bool items_by_group(const slimpipe_attn_params* p, int64_t keys, int ranges) {
  return (int64_t)p->n_kv_heads * p->batch >= 8 && keys >= 3072 * (int64_t)ranges;
}
size_t fwd_part_out_bytes(const slimpipe_attn_params* p) {
  size_t n = (size_t)p->batch * (size_t)p->s_q * (size_t)p->n_q_heads * (size_t)p->head_dim * sizeof(float);
  return (n + 255) & ~(size_t)255;
}
size_t fwd_parts_bytes(const slimpipe_attn_params* p, int ranges) {
  return ranges <= 1 ? 0 : (size_t)ranges * (fwd_part_out_bytes(p) + stat_bytes(p));
}
// Microseconds of a call through the small kernel (32 query rows a workgroup, the 8 waves sharing out the keys of its range) in
// r key ranges: 8.7 (head_dim 64: 7) + 1.3 (1.4) per step of a wave, which is 32 (64) keys, times the rounds of workgroups, + the merge.
double fwd_small_us(const slimpipe_attn_params* p, int64_t cus, int r) {
  const bool d64 = p->head_dim == 64;
  const int64_t keys = p->kv_end - p->kv_begin;
  const int64_t wgs = ((int64_t)p->s_q + 31) / 32 * p->n_q_heads * p->batch * r, per_step = 8 * (d64 ? 64 : 32);
  const double steps = (double)((keys + r * per_step - 1) / (r * per_step)), rounds = (double)((wgs + cus - 1) / cus);
  return (d64 ? 7.0 : 8.7) + 2 * (rounds - 1) + rounds * steps * (d64 ? 1.4 : 1.3) +
         (r > 1 ? 4.5 + (double)(r + 1) * p->s_q * p->n_q_heads * p->batch * p->head_dim * 4 / 4e6 : 0.0);
}
// One past the last key before `end` that any row sees (`begin` when none does).
int64_t seen_end(const slimpipe_attn_params* p, int64_t begin, int64_t end) {
  if (p->causal && p->q_offset + p->s_q < end) end = p->q_offset + p->s_q;
  return end > begin ? end : begin;
}
struct FwdPlan {
  int head_waves;    // of the query blocks
  int ranges;        // key ranges
  bool small;        // 32-row workgroups (attn_fwd_small_kernel)
};
// The plan with 256-row blocks when the partial results of the ranges take at most `room` bytes.
FwdPlan fwd_blocks_plan(const slimpipe_attn_params* p, size_t room) {
  const int hw = head_waves_of(p, p->kv_end - p->kv_begin, fwd_parts_bytes(p, 2) > room ? 1 : most_ranges(p, min_range_keys(p->head_dim)));
  int ranges = fwd_preferred_ranges(p, hw);
  while (ranges > 1 && (fwd_parts_bytes(p, ranges) > room || (int64_t)p->batch * ranges > 65535)) --ranges;
  return {hw, ranges, false};
}
// What the forward would do with all the room it wants.
// With less than one 256-row block per compute unit the small kernel is taken, in the number of ranges (none shorter than the
// 256-row blocks may have) that makes it fastest, where its time is shorter.  Over 567 calls, both kernels timed in 1 to 8 ranges, the pick is within 1 %
// of the best in the mean (1.58 and 1.74 times its time at worst, at head_dim 64 and 128: long keys left on the blocks), and where it is the
// small kernel 1.61 and 1.95 times as fast as the 256-row blocks, 0.99 at worst, 3.1 at best (256 rows of 8 heads on 2648 keys 42.4 -> 16.9 us).
// It loses where keys are long: every workgroup reads all its keys for 32 rows (676 rows of 8 heads on 17519 keys: 98 us against 69).
FwdPlan fwd_plan_wanted(const slimpipe_attn_params* p) {
  const FwdPlan blocks = fwd_blocks_plan(p, SIZE_MAX);
  const int64_t w = all_query_blocks(p, blocks.head_waves), keys = p->kv_end - p->kv_begin, cus = compute_units();
  if (w >= cus || keys <= 0) return blocks;
  double best_us = fwd_blocks_us(p, cus, w, blocks.ranges) * 0.97;
  int pick = 0;
  for (int r = 1; r <= kMaxRanges && (r == 1 || keys / r >= min_range_keys(p->head_dim)) && (int64_t)p->batch * r <= 65535; ++r) {
    const double us = fwd_small_us(p, cus, r);
    if (us < best_us) { best_us = us * 0.99; pick = r; }
  }
  return pick ? FwdPlan{blocks.head_waves, pick, true} : blocks;
}
// The plan of a call with a workspace of this many bytes (0: none): [ticket counter, 256 bytes][partial results of the ranges].
// The small kernel is taken only when it is what the call wants with all the room, and has that room.  With less, or without
// a workspace, the call keeps the kernel of slimpipe_attn_fwd_ranges, in as many ranges as fit: undivided, it
// returns what a range of that call returns, bit for bit.  (Choosing anew for the room there is would take the small kernel wherever
// the lack of ranges makes the 256-row blocks slow: other bits with every other size of the workspace.)
FwdPlan fwd_plan_within(const slimpipe_attn_params* p, size_t workspace_bytes) {
  const bool lent = workspace_bytes >= kTicketBytes;
  const size_t room = lent ? workspace_bytes - kTicketBytes : workspace_bytes;
  if (lent) {
    const FwdPlan wanted = fwd_plan_wanted(p);
    if (wanted.small && fwd_parts_bytes(p, wanted.ranges) <= room) return wanted;
  }
  return fwd_blocks_plan(p, room);
}
// The dq kernel has the forward's launch shape and is cut into key ranges the same way; its partial results are
// float32 [range][batch, s_q, heads, head_dim].
size_t dq_parts_bytes(const slimpipe_attn_params* p, int ranges) {
  return ranges <= 1 ? 0 : (size_t)ranges * fwd_part_out_bytes(p);
}

// ---- the backward's launches -------------------------------------------------------------------------
struct BwdPlan {
  int head_waves;    // of the dq query blocks
  int split;         // chunks of a key tile's query stream
  int dq_ranges;     // key ranges of the dq items
  bool both;         // dq and dk/dv items in one launch
  bool dq_first;     // ... the dq items first
  double us;         // (one launch) its time and that of the reduce by the model of bwd_plan
  bool full;         // what is wanted whatever the workspace, not cut down to it
};

// Time at which `na` items of length ta, then `nb` items of length tb, each started on the unit that is free first, are
// all done on `units` units.
double list_makespan(int64_t units, int64_t na, double ta, int64_t nb, double tb) {
  const int64_t full = na / units, extra = na % units;                 // `extra` units hold one item more
  const double load0 = (double)full * ta, load1 = load0 + (extra ? ta : 0.0);
  const int64_t n0 = units - extra;
  if (nb <= 0) return load1;
  // the smallest finishing time m at which the units hold nb items of length tb between them
  double best = 1e30;
  for (int g = 0; g < (extra ? 2 : 1); ++g) {
    const double load = g ? load1 : load0;
    for (int k = 1; k <= 64; ++k) {
      const double m = load + k * tb;
      if (m >= best) break;
      const int64_t room = (int64_t)((m - load0) / tb + 1e-9) * n0 + (m > load1 ? (int64_t)((m - load1) / tb + 1e-9) * extra : 0);
      if (room >= nb) { best = m; break; }
    }
  }
  return best > load1 ? best : load1;
}

// A call with fewer than two items per compute unit (query blocks + key tiles) runs dq and dk/dv in one launch, with the
// cuts that finish first by the times below; a larger one runs them one after the other through the ticket counters.
// Microseconds measured on MI355X with the chip full: a dq item is about 8 + 2.4 per 64 keys (head_dim 128; 1.4 at 64; 1.3 to
// 1.5 at 128 with 25 to 130 units busy), a dk/dv item about 10 + 1.6 (1.1) per 32 query rows; a reduce launch 4 + its
// bytes at 5 TB/s.
// The partial sums of the cuts take at most `room` bytes (SIZE_MAX: all that are wanted): a small call chooses among the
// pairs that fit, a large one takes first as many chunks and then as many key ranges as fit.
BwdPlan bwd_plan(const slimpipe_attn_params* p, int n_chunks, bool ticket, size_t room) {
  const int64_t cus = compute_units();
  const int hw = head_waves_of(p, p->kv_end - p->kv_begin, dq_parts_bytes(p, 2) > room ? 1 : most_ranges(p, 256));
  const int64_t wq = all_query_blocks(p, hw);
  const int64_t wk = dkdv_key_tiles(p, n_chunks) * p->n_kv_heads * p->batch;
  if (wk <= 0 || wq + wk >= 2 * cus) {
    BwdPlan plan{hw, preferred_split(p, n_chunks, ticket), fwd_preferred_ranges(p, hw), false, false, 0.0, room == SIZE_MAX};
    while (plan.split > 1 && split_bytes(p, n_chunks, plan.split) > room) plan.split /= 2;
    const size_t used = split_bytes(p, n_chunks, plan.split);
    while (plan.dq_ranges > 1 && (dq_parts_bytes(p, plan.dq_ranges) > room - used || (int64_t)p->batch * plan.dq_ranges > 65535)) --plan.dq_ranges;
    return plan;
  }
  const int64_t keys = p->kv_end - p->kv_begin;
  const double dq_tiles = (double)keys / 64, dq_tile = p->head_dim == 128 ? 2.4 : 1.4;
  const double stream = (double)(((int64_t)p->s_q + 31) / 32 * (p->n_q_heads / p->n_kv_heads)), dkdv_tile = p->head_dim == 128 ? 1.6 : 1.1;
  static const int kCuts[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16};
  BwdPlan best{hw, 1, 1, true, false, 0.0, room == SIZE_MAX};
  double best_us = 1e30;
  for (int s : kCuts) {
    if (s > 8 || (s > 1 && stream / s < 4)) break;             // a chunk keeps at least 4 query tiles
    for (int r : kCuts) {
      if (r > 1 && (keys / r < 256 || (int64_t)p->batch * r > 65535)) break;      // a range keeps at least 256 keys
      if (split_bytes(p, n_chunks, s) + dq_parts_bytes(p, r) > room) break;       // (1, 1) needs none
      const double tq = 8 + dq_tile * dq_tiles / r, tk = 10 + dkdv_tile * stream / s;
      double us = tq > tk ? list_makespan(cus, wq * r, tq, wk * s, tk) : list_makespan(cus, wk * s, tk, wq * r, tq);
      // Where no cut fits and the items are long, one launch can have as long a tail as two, and then two are faster: a
      // kind that has part of a power-limited chip to itself runs at a higher clock (dq items alone on 128 of 256 units take 0.55
      // of the time above).  Measured without cuts, two launches / one: 2856 / 3094, 759 / 788, 4332 / 4669, 4029 / 4178 us
      // where the model gives one launch 0.87, 0.96, 1.00, 1.00 of two; at 0.63 to 0.80 of it one is faster by 9 to 48 %, and by
      // up to 11 % where items are short.  With a cut of either kind two launches were never faster.
      bool both = true;
      if (room != SIZE_MAX && s == 1 && r == 1 && tq >= 300 && tk >= 300)
        both = us <= 0.85 * (list_makespan(cus, wq, tq, 0, 0) + list_makespan(cus, wk, tk, 0, 0));
      double bytes = s > 1 ? (double)(s + 2) * keys * p->n_kv_heads * p->batch * p->head_dim * 8 : 0.0;
      if (r > 1) bytes += (double)(r + 1) * p->s_q * p->n_q_heads * p->batch * p->head_dim * 4;
      if (bytes > 0) us += 4 + bytes / 5e6;
      if (us < best_us * 0.99) { best_us = us; best = {hw, s, r, both, tq > tk, us, room == SIZE_MAX}; }
    }
  }
  return best;
}
// The plan of a call with a workspace of this many bytes: the best one when its partial sums fit, otherwise the best of
// those that do.  (Cutting the best plan down to the room there is leaves its order of the two kinds: 2387 rows on 52005 keys
// planned 10 ranges of short dq items behind the dk/dv items; undivided, the dq items are the longer kind and came last.)
BwdPlan bwd_plan_within(const slimpipe_attn_params* p, int n_chunks, size_t workspace_bytes) {
  const bool ticket = workspace_bytes >= delta_bytes(p) + kTicketBytes;
  const size_t room = workspace_bytes - delta_bytes(p) - (ticket ? kTicketBytes : 0);
  const BwdPlan plan = bwd_plan(p, n_chunks, ticket, SIZE_MAX);
  return split_bytes(p, n_chunks, plan.split) + dq_parts_bytes(p, plan.dq_ranges) <= room ? plan : bwd_plan(p, n_chunks, ticket, room);
}
// Whether a call that bwd_plan puts into one launch goes through the small kernel instead (32 query rows or 32 keys a workgroup, the
// eight waves sharing out the other side, no partial sums in memory), and which items come first there.  Only a call that is
// given the workspace it is asked for: with less, and where nothing would be cut, it keeps the sums of the undivided items.
// Microseconds: a dq item 6 (head_dim 64: 5) + 1.6 (1.4) per step of a wave, which is 32 (64) keys, a dk/dv item 6 (5) + 2 (1) per 32
// query rows of a wave, and 4 (5.5) for the launch; against the model of bwd_plan + 7, what the delta and reduce launches
// cost beyond it.  These are the times of the first small kernel, which took longer: they err towards the 256-row items.  Of random calls,
// both kernels timed, the small kernel takes 1 / 1.56 of their time at head_dim 64 where it is picked (1170 calls, 0.86 at worst; 512 rows on 2048
// keys, 4 heads, 30.2 -> 13.4 us) and 1 / 1.41 at 128 (159 calls, 0.92; 100 rows of 8/2 heads on 448 keys, batch 2, 31.9 -> 17.1); where it is not it
// would be 0.96 and 0.87 times as fast (412 and 96 calls), by up to 1.44 and 1.27 faster.  Long calls stay out: a workgroup reads
// the whole other side for 32 rows or keys, and the model does not know what that costs a full chip (1969 rows on 4976 keys, 8/1 heads of
// 64: 80 us by the model, 104 measured, 90 through the 256-row items).
// The line at 32 dq items is no line of speed: below it the small kernel wins too (318 calls of 17 to 32 items of head_dim 64: 1.62 times as fast in
// the mean), but the launches of a call of 32 items are what the per-kernel timing is pinned to, kind by kind.  With 33 to 63 items (280
// calls) it is 1.78 times as fast in the mean, 0.96 at worst.
// key_blocks: at head_dim 64 a dk/dv item can own two blocks of 32 keys, four waves each: half the items, of twice the steps.
// own_stats: the items work out the row statistics themselves and no delta kernel runs before.  That saves its launch, 3 us and the
// host's 4, and costs each step of a dk/dv wave 0.5 us (O comes along with Q and dO); at head_dim 128 1 us (256 rows on 512 keys, 8/1 heads, 8
// steps, 30.9 with / 24.9 without), so only head_dim 64 has it.  (A call whose gradients lie over its out or lse has the delta kernel all the
// same: bwd_impl.)  Where every item has a compute unit to itself, the steps decide: calls of up to 6 have no delta kernel (with / without it
// 1.27, 1.15, 1.09, 1.04, 1.00, 0.98, 0.94 of the time at 2 to 8 steps, in the mean).  Otherwise small_bwd_us does, and so it does between one
// block and two: one block, with more items than units behind a delta kernel, unless another way is 5 % faster (the sums are 4 % off in the
// mean).  Over 1170 calls, all four ways timed, the pick takes 1.007 of the best one's time in the mean, 1.19 at worst, and 0.93 of that of one
// block behind a delta kernel, 1.09 at worst, more than 1.05 twice.  (Two blocks by makespans of other times, and no delta kernel up to 6
// steps whatever the items: 1.014, 1.41; 0.935, 1.36, more than 1.05 in 34 calls.)  One block with / without delta kernel, two blocks with / without, us:
// 512 rows on 2048 keys, 4/4 heads, 17.6 / 16.6, - / 13.4; 1024 on 1061, 2 x 2/2, 14.2 / 12.5, 17.6 / 19.6; 1334 on 12925, 2/2, not causal, 54.9 /
// 64.8, 57.2 / 64.4.
struct BwdSmallPlan { bool use, dq_first, own_stats; int key_blocks; };
// Microseconds of a call of head_dim 64 through the small kernel: its launch (with the delta launch's), and the longest item, or with more items
// than compute units what each unit gets in the mean and two thirds of a short item for the uneven end, if that is longer.  sq, sk: steps
// of a wave of a dq item and of a dk/dv item of one block, were every row to see every key; seen: the share that it does see.
double small_bwd_us(int64_t cus, int64_t nq, int64_t nk, double sq, double sk, double seen, int key_blocks, bool own_stats, bool* dq_first) {
  const double step = (key_blocks == 2 ? 1.1 : 1.15) + (own_stats ? 0.5 : 0.0);
  auto dq = [](double steps) { return 3.4 + 1.32 * steps; };
  auto dkdv = [&](double steps) { return (key_blocks == 2 ? 4.5 : 3.6) + step * steps; };
  const double tq = dq(ceil(sq)), tk = dkdv(ceil(key_blocks * sk)), mean_q = dq(sq * seen + 0.4), mean_k = dkdv(key_blocks * sk * seen + 0.4);
  *dq_first = tq > tk;
  double t = tq > tk ? tq : tk;
  if (nq + nk > cus) {
    const double even = (nq * mean_q + nk * mean_k) / cus + 0.67 * (mean_q < mean_k ? mean_q : mean_k);
    if (even > t) t = even;
  }
  return (own_stats ? 2.7 : 5.4) + t;
}
BwdSmallPlan bwd_small_plan(const slimpipe_attn_params* p, const BwdPlan& plan) {
  if (!plan.both || !plan.full || (plan.split == 1 && plan.dq_ranges == 1)) return {false, false, false, 1};
  const bool d64 = p->head_dim == 64;
  const int64_t keys = p->kv_end - p->kv_begin, cus = compute_units();
  const int64_t row_blocks = ((int64_t)p->s_q + 31) / 32, key_blocks = (keys + 31) / 32;
  const int64_t nq = row_blocks * p->n_q_heads * p->batch, nk = key_blocks * p->n_kv_heads * p->batch;
  // steps of the longest item where every item has a compute unit to itself, otherwise of the mean one
  const double seen = visible_pairs_upto(p, p->kv_end) / ((double)p->s_q * (double)keys);
  const double sq = (double)keys / (d64 ? 512 : 256), sk = (double)(row_blocks * (p->n_q_heads / p->n_kv_heads)) / 8;
  const double tq = (d64 ? 5 : 6) + (d64 ? 1.4 : 1.6) * (nq > cus ? sq * seen + 0.5 : ceil(sq));
  const double tk = (d64 ? 5 : 6) + (d64 ? 1.0 : 2.0) * (nk > cus ? sk * seen + 0.5 : ceil(sk));
  const double us = (d64 ? 5.5 : 4) + (tq > tk ? list_makespan(cus, nq, tq, nk, tk) : list_makespan(cus, nk, tk, nq, tq));
  BwdSmallPlan best{nq > 32 && us < 60 && us * 1.05 < plan.us + 7, tq > tk, false, 1};
  if (!best.use || !d64) return best;
  const int64_t items[2] = {nk, (key_blocks + 1) / 2 * p->n_kv_heads * p->batch};
  auto one_round = [&](int blocks) { return nq + items[blocks - 1] <= cus; };
  auto few_steps = [&](int blocks) { return blocks * sk <= 6; };
  double best_us = 0.0;
  auto consider = [&](int blocks, bool own, double factor) {
    BwdSmallPlan other{true, false, own, blocks};
    const double t = factor * small_bwd_us(cus, nq, items[blocks - 1], sq, sk, seen, blocks, own, &other.dq_first);
    if (best_us == 0.0 || t < best_us) { best_us = t; best = other; }
  };
  consider(1, one_round(1) && few_steps(1), 0.95);
  for (int blocks = 1; blocks <= 2; ++blocks)
    for (int own = 0; own < 2; ++own)
      if (!one_round(blocks) || (own != 0) == few_steps(blocks)) consider(blocks, own != 0, 1.0);
  return best;
}
// Tiles of the large backward at head_dim 64: 128 or 64 keys (dq), 64 or 32 query rows (dk/dv).  The larger ones have half the
// barriers and copies per pair; a short walk pays for them in its first and last tile, which nothing hides, and in padding.
// Over 470 calls of random sizes in two launches, larger against smaller tile: dq 0.93 to 1.01 of the time where the rule says 128, always
// taking 128 costs up to 1.21 (64 rows of 40 heads on 141 keys, batch 8).
int dq_tile_keys(const slimpipe_attn_params* p, const BwdPlan& plan) {
  if (p->head_dim == 128 || plan.both) return 64;
  const double walk = visible_pairs_upto(p, p->kv_end) / ((double)p->s_q * plan.dq_ranges);      // keys that an item's row sees, in the mean
  return walk >= 3072 || (walk >= 1024 && p->s_q >= 512) ? 128 : 64;
}
// dk/dv in two launches: 0.89 to 1.01 of the time where the rule says 64 rows (1400 rows an item and more, with padding more);
// always taking 64 costs up to 1.75 (40 rows of 40 heads on 5278 keys, batch 4) and 1.13 to 1.19 at 512 rows.  In one launch, where a long
// item ends the call, the line is lower: 512 rows a chunk (256 rows of 4 heads on 5073 keys, 128 rows a chunk: 27.3 us with 32-row tiles,
// 29.7 with 64) and 4 % of padding (400 rows are 416 or 448: 73.3 us against 77.3 on 12400 keys, 8/2 heads); over 360 calls 0.88 to
// 1.05 of the time where it says 64.
int dkdv_tile_rows(const slimpipe_attn_params* p, const BwdPlan& plan) {
  if (p->head_dim == 128 || p->kv_end <= p->kv_begin) return 32;
  const int64_t group = p->n_q_heads / p->n_kv_heads, t32 = ((int64_t)p->s_q + 31) / 32, t64 = (t32 + 1) / 2;
  const double padding = (double)(2 * t64 - t32) / (double)t32;
  if (plan.both) return p->s_q * group >= 512 * (int64_t)plan.split && padding <= 0.04 ? 64 : 32;
  const double walk = visible_pairs_upto(p, p->kv_end) / (double)(p->kv_end - p->kv_begin) * (double)group / plan.split;      // rows that see an item's key
  return walk * (0.08 - padding) >= 112 ? 64 : 32;
}
// Cut points of equal work on multiples of 256 keys (no range boundary inside a chunk-grid tile).
void equal_work_ranges(const slimpipe_attn_params* p, int ranges, int64_t* begin, int64_t* end) {
  const double total = visible_pairs_upto(p, p->kv_end);
  int64_t prev = p->kv_begin;
  for (int r = 0; r < ranges; ++r) {
    int64_t cut = p->kv_end;
    if (r + 1 < ranges) {
      const double want = total * (double)(r + 1) / (double)ranges;
      int64_t lo = prev / 256, hi = (p->kv_end + 255) / 256;        // smallest multiple of 256 with enough pairs below it
      while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (visible_pairs_upto(p, mid * 256) >= want) hi = mid; else lo = mid + 1;
      }
      cut = lo * 256;
      if (cut < prev) cut = prev;
      if (cut > p->kv_end) cut = p->kv_end;
    }
    begin[r] = prev;
    end[r] = cut;
    prev = cut;
  }
}

// A chunk list is legal when it covers kv_capacity rows; with more than one chunk the chunk length is a
// multiple of the dk/dv key tile (256), so that no key tile of any kernel straddles two chunks.
int check_chunks(const slimpipe_attn_params* p, int32_t n_chunks, int64_t chunk_len) {
  if (n_chunks < 1 || n_chunks > kMaxChunks || chunk_len < 1) return SLIMPIPE_EINVAL_SHAPE;
  if (n_chunks * chunk_len < p->kv_capacity) return SLIMPIPE_EINVAL_RANGE;
  if (n_chunks > 1 && chunk_len % dkdv_keys_per_workgroup() != 0) return SLIMPIPE_EINVAL_SHAPE;
  return SLIMPIPE_OK;
}



// ---- optional per-kernel event timing (benchmark aid) ----------------------------------------------
struct ProfRecord { int kind; hipEvent_t start, stop; };
std::atomic<bool> g_prof_on{false};
std::mutex g_prof_mutex;                     // guards the two vectors
std::vector<ProfRecord> g_prof_records;
std::vector<hipEvent_t> g_prof_free;

hipEvent_t prof_event() {                    // (caller holds g_prof_mutex)
  if (!g_prof_free.empty()) { hipEvent_t e = g_prof_free.back(); g_prof_free.pop_back(); return e; }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

template <class F>
hipError_t timed(int kind, hipStream_t st, F&& launch, bool allow = true) {
  if (!allow || !g_prof_on.load(std::memory_order_relaxed)) return launch();
  std::lock_guard<std::mutex> lock(g_prof_mutex);
  ProfRecord r{kind, prof_event(), prof_event()};
  if (!r.start || !r.stop) return launch();
  (void)hipEventRecord(r.start, st);
  hipError_t e = launch();
  (void)hipEventRecord(r.stop, st);
  g_prof_records.push_back(r);
  return e;
}

}  // namespace

extern "C" {

int slimpipe_attn_init(void) { return ensure_device_ready(); }

int slimpipe_attn_profile_enable(int enable) {
  g_prof_on.store(enable != 0, std::memory_order_relaxed);
  return SLIMPIPE_OK;
}

int slimpipe_attn_profile_read(double total_ms[SLIMPIPE_KERNEL_KINDS], int64_t launches[SLIMPIPE_KERNEL_KINDS]) {
  if (!total_ms || !launches) return SLIMPIPE_EINVAL_NULL;
  for (int i = 0; i < SLIMPIPE_KERNEL_KINDS; ++i) { total_ms[i] = 0.0; launches[i] = 0; }
  int rc = SLIMPIPE_OK;
  std::lock_guard<std::mutex> lock(g_prof_mutex);
  for (const ProfRecord& r : g_prof_records) {
    float ms = 0.f;
    if (hipEventSynchronize(r.stop) != hipSuccess || hipEventElapsedTime(&ms, r.start, r.stop) != hipSuccess)
      rc = SLIMPIPE_ELAUNCH;
    else if (r.kind >= 0 && r.kind < SLIMPIPE_KERNEL_KINDS) { total_ms[r.kind] += ms; launches[r.kind] += 1; }
    g_prof_free.push_back(r.start);
    g_prof_free.push_back(r.stop);
  }
  g_prof_records.clear();
  return rc;
}

int slimpipe_attn_bwd_plan(const slimpipe_attn_params* p, int32_t n_chunks, size_t workspace_bytes, slimpipe_bwd_plan* out) {
  if (!p || !out) return SLIMPIPE_EINVAL_NULL;
  int rc = slimpipe_attn_validate(p, 1);
  if (rc != SLIMPIPE_OK) return rc;
  if (n_chunks < 1 || n_chunks > kMaxChunks) return SLIMPIPE_EINVAL_SHAPE;
  if (workspace_bytes < delta_bytes(p)) return SLIMPIPE_EWORKSPACE;
  const BwdPlan plan = bwd_plan_within(p, n_chunks, workspace_bytes);
  out->one_launch = plan.both;
  out->dq_first = plan.both && plan.dq_first;
  out->dkdv_split = plan.split;
  out->dq_ranges = plan.dq_ranges;
  out->dkdv_items = dkdv_key_tiles(p, n_chunks) * plan.split * p->n_kv_heads * p->batch;
  out->dq_items = all_query_blocks(p, plan.head_waves) * plan.dq_ranges;
  out->compute_units = compute_units();
  out->dq_by_xcd = !plan.both && out->dq_items > out->compute_units && workspace_bytes >= delta_bytes(p) + kTicketBytes &&
                   items_by_group(p, p->kv_end - p->kv_begin, plan.dq_ranges);
  return SLIMPIPE_OK;
}

int slimpipe_attn_call_path(const slimpipe_attn_params* p, int is_bwd, int32_t n_chunks, size_t workspace_bytes, slimpipe_call_path* path) {
  if (!p || !path) return SLIMPIPE_EINVAL_NULL;
  int rc = slimpipe_attn_validate(p, is_bwd);
  if (rc != SLIMPIPE_OK) return rc;
  if (n_chunks < 1 || n_chunks > kMaxChunks) return SLIMPIPE_EINVAL_SHAPE;
  memset(path, 0, sizeof(*path));
  if (!is_bwd) {
    const FwdPlan plan = fwd_plan_within(p, workspace_bytes);
    path->small = plan.small;
    path->ranges = plan.ranges;
    return SLIMPIPE_OK;
  }
  if (workspace_bytes < delta_bytes(p)) return SLIMPIPE_EWORKSPACE;
  const BwdPlan plan = bwd_plan_within(p, n_chunks, workspace_bytes);
  path->small = bwd_small_plan(p, plan).use;
  path->ranges = path->small ? 1 : plan.dq_ranges;
  path->dq_tile_keys = path->small ? small_dq_tile_keys(p->head_dim) : dq_tile_keys(p, plan);
  path->dkdv_tile_rows = path->small ? 32 : dkdv_tile_rows(p, plan);
  return SLIMPIPE_OK;
}

int slimpipe_attn_small_bwd_plan(const slimpipe_attn_params* p, int32_t n_chunks, size_t workspace_bytes, slimpipe_small_bwd_plan* out) {
  if (!p || !out) return SLIMPIPE_EINVAL_NULL;
  int rc = slimpipe_attn_validate(p, 1);
  if (rc != SLIMPIPE_OK) return rc;
  if (n_chunks < 1 || n_chunks > kMaxChunks) return SLIMPIPE_EINVAL_SHAPE;
  if (workspace_bytes < delta_bytes(p)) return SLIMPIPE_EWORKSPACE;
  memset(out, 0, sizeof(*out));
  const BwdSmallPlan sm = bwd_small_plan(p, bwd_plan_within(p, n_chunks, workspace_bytes));
  if (sm.use) *out = {1, sm.key_blocks, sm.own_stats, sm.dq_first};
  return SLIMPIPE_OK;
}

int slimpipe_attn_validate(const slimpipe_attn_params* p, int is_bwd) {
  if (!p) return SLIMPIPE_EINVAL_NULL;
  if (p->batch <= 0 || p->s_q <= 0 || p->n_q_heads <= 0 || p->n_kv_heads <= 0) return SLIMPIPE_EINVAL_SHAPE;
  if (p->n_q_heads % p->n_kv_heads != 0) return SLIMPIPE_EINVAL_SHAPE;
  if (p->head_dim != 64 && p->head_dim != 128) return SLIMPIPE_EINVAL_SHAPE;
  if (!(p->scale > 0.0f) || !isfinite(p->scale)) return SLIMPIPE_EINVAL_SHAPE;
  if (p->causal != 0 && p->causal != 1) return SLIMPIPE_EINVAL_SHAPE;
  if (p->out_dtype != SLIMPIPE_BF16 && p->out_dtype != SLIMPIPE_F32) return SLIMPIPE_EINVAL_SHAPE;
  if (p->batch > 65535 || p->n_q_heads > 65535) return SLIMPIPE_EINVAL_SHAPE;   /* limits stated in the header */
  if (p->kv_capacity < 0 || p->q_offset < 0 || p->kv_begin < 0) return SLIMPIPE_EINVAL_RANGE;
  if (p->kv_begin > p->kv_end || p->kv_end > p->kv_capacity) return SLIMPIPE_EINVAL_RANGE;
  if (p->q_offset > (int64_t)1 << 40 || p->kv_capacity > (int64_t)1 << 40) return SLIMPIPE_EINVAL_RANGE;
  const int64_t s[9] = {p->q_stride_b, p->q_stride_s, p->q_stride_h, p->kv_stride_b, p->kv_stride_s,
                        p->kv_stride_h, p->o_stride_b, p->o_stride_s, p->o_stride_h};
  for (int i = 0; i < 9; ++i)
    if (!stride_ok(s[i])) return SLIMPIPE_EINVAL_STRIDE;
  if (is_bwd && (!stride_ok(p->do_stride_b) || !stride_ok(p->do_stride_s) || !stride_ok(p->do_stride_h) ||
                 p->do_stride_h < p->head_dim))
    return SLIMPIPE_EINVAL_STRIDE;
  if (p->q_stride_h < p->head_dim || p->kv_stride_h < p->head_dim || p->o_stride_h < p->head_dim)
    return SLIMPIPE_EINVAL_STRIDE;
  /* row strides enter 32-bit byte offsets inside a tile */
  if (p->q_stride_s >= (1 << 22) || p->kv_stride_s >= (1 << 22) || p->o_stride_s >= (1 << 22) ||
      (is_bwd && p->do_stride_s >= (1 << 22)))
    return SLIMPIPE_EINVAL_STRIDE;
  return SLIMPIPE_OK;
}

int slimpipe_attn_workspace_bytes(const slimpipe_attn_params* p, int is_bwd, size_t* bytes) {
  if (!bytes) return SLIMPIPE_EINVAL_NULL;
  int rc = slimpipe_attn_validate(p, is_bwd);
  if (rc != SLIMPIPE_OK) return rc;
  if (!is_bwd) { *bytes = kTicketBytes + fwd_parts_bytes(p, fwd_plan_wanted(p).ranges); return SLIMPIPE_OK; }
  // the tile grid of a chunked call can start up to 255 keys before kv_begin: room for whichever of the
  // two variants asks for more
  const BwdPlan plan1 = bwd_plan(p, 1, true, SIZE_MAX), plan2 = bwd_plan(p, 2, true, SIZE_MAX);
  const size_t one = split_bytes(p, 1, plan1.split) + dq_parts_bytes(p, plan1.dq_ranges);
  const size_t many = split_bytes(p, 2, plan2.split) + dq_parts_bytes(p, plan2.dq_ranges);
  *bytes = delta_bytes(p) + kTicketBytes + (one > many ? one : many);
  return SLIMPIPE_OK;
}

// Forward over `n_ranges` key ranges in one launch.  With parts == nullptr there is one range and the result
// goes straight to (out, lse); otherwise range r writes float32 partials at part_out + r * part_out_elems,
// part_lse + r * part_lse_elems (contiguous [batch, s_q, heads, head_dim] / [batch, heads, s_q]) and, when
// `out` is given, the merge kernel folds them into (out, lse).
static int fwd_impl(const slimpipe_attn_params* p, const void* q_slice, const void* const* k_chunks,
                    const void* const* v_chunks, int32_t n_chunks, int64_t chunk_len, int32_t n_ranges,
                    const int64_t* range_begin, const int64_t* range_end, float* part_out, int64_t part_out_elems,
                    float* part_lse, int64_t part_lse_elems, void* out, float* lse, void* hip_stream, unsigned* ticket = nullptr,
                    int head_waves = 0, bool small = false) {      // (head_waves 0: chosen here)
  int rc = slimpipe_attn_validate(p, 0);
  if (rc != SLIMPIPE_OK) return rc;
  const bool parts = part_out != nullptr;
  if (!q_slice || !k_chunks || !v_chunks || !range_begin || !range_end) return SLIMPIPE_EINVAL_NULL;
  if (parts ? !part_lse || ((out == nullptr) != (lse == nullptr)) : (!out || !lse)) return SLIMPIPE_EINVAL_NULL;
  if (n_ranges < 1 || n_ranges > kMaxRanges || (!parts && n_ranges != 1)) return SLIMPIPE_EINVAL_SHAPE;
  if ((int64_t)p->batch * n_ranges > 65535) return SLIMPIPE_EINVAL_SHAPE;
  rc = check_chunks(p, n_chunks, chunk_len);
  if (rc != SLIMPIPE_OK) return rc;
  if (!aligned16(q_slice) || (out && (!aligned16(out) || (reinterpret_cast<uintptr_t>(lse) & 3u)))) return SLIMPIPE_EINVAL_ALIGN;
  if (parts && (!aligned16(part_out) || (reinterpret_cast<uintptr_t>(part_lse) & 3u) || part_out_elems % 4 != 0)) return SLIMPIPE_EINVAL_ALIGN;
  FwdArgs a;
  memset(&a.kv, 0, sizeof(a.kv));
  int64_t last_key = 0, keys = 0;
  for (int r = 0; r < kMaxRanges; ++r) {
    a.range_begin[r] = a.range_end[r] = 0;
    if (r >= n_ranges) continue;
    if (range_begin[r] < 0 || range_begin[r] > range_end[r] || range_end[r] > p->kv_capacity) return SLIMPIPE_EINVAL_RANGE;
    a.range_begin[r] = range_begin[r];
    a.range_end[r] = seen_end(p, range_begin[r], range_end[r]);
    if (range_end[r] > last_key) last_key = range_end[r];
    keys += range_end[r] - range_begin[r];
  }
  for (int i = 0; i < n_chunks; ++i) {
    if (last_key > 0 && (!k_chunks[i] || !v_chunks[i])) return SLIMPIPE_EINVAL_NULL;
    if (!aligned16(k_chunks[i]) || !aligned16(v_chunks[i])) return SLIMPIPE_EINVAL_ALIGN;
    a.kv.k[i] = static_cast<const __bf16*>(k_chunks[i]);
    a.kv.v[i] = static_cast<const __bf16*>(v_chunks[i]);
  }
  a.kv.len = chunk_len;
  a.kv.n = n_chunks;
  a.q = static_cast<const __bf16*>(q_slice);
  a.n_ranges = n_ranges;
  a.s_q = p->s_q; a.n_q_heads = p->n_q_heads; a.group = p->n_q_heads / p->n_kv_heads;
  a.causal = p->causal;
  a.q_offset = p->q_offset; a.kv_capacity = p->kv_capacity;
  a.scale_log2e = p->scale * 1.4426950408889634f;
  a.q_stride_b = p->q_stride_b; a.q_stride_s = p->q_stride_s; a.q_stride_h = p->q_stride_h;
  a.kv_stride_b = p->kv_stride_b; a.kv_stride_s = p->kv_stride_s; a.kv_stride_h = p->kv_stride_h;
  if (parts) {
    a.out = part_out; a.lse = part_lse; a.out_f32 = 1;
    a.out_range_stride = part_out_elems; a.lse_range_stride = part_lse_elems;
    a.o_stride_h = p->head_dim; a.o_stride_s = (int64_t)p->n_q_heads * p->head_dim; a.o_stride_b = a.o_stride_s * p->s_q;
  } else {
    a.out = out; a.lse = lse; a.out_f32 = (p->out_dtype == SLIMPIPE_F32);
    a.out_range_stride = 0; a.lse_range_stride = 0;
    a.o_stride_b = p->o_stride_b; a.o_stride_s = p->o_stride_s; a.o_stride_h = p->o_stride_h;
  }
  a.head_waves = head_waves ? head_waves : head_waves_of(p, keys, n_ranges);
  const int64_t blocks = query_blocks(a.head_waves, a.group);
  // (32-row workgroups are at most 8 times as many)
  if (blocks * p->n_kv_heads * p->batch * n_ranges > (int64_t)1 << 30) return SLIMPIPE_EINVAL_SHAPE;
  a.items[0] = (int32_t)blocks;
  a.items[1] = p->n_kv_heads;
  a.items[2] = p->batch * n_ranges;
  // a counter only where there are more items than compute units (otherwise every workgroup starts at once)
  if ((int64_t)a.items[0] * a.items[1] * a.items[2] <= compute_units()) ticket = nullptr;
  a.ticket = ticket;
  a.items_by_group = items_by_group(p, keys, n_ranges);
  if (ensure_device_ready() != SLIMPIPE_OK) return SLIMPIPE_ELAUNCH;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  if (small) a.items[0] = (int32_t)(((int64_t)p->s_q + 31) / 32);
  else if (ticket && launch_zero_counters(ticket, st) != hipSuccess) return SLIMPIPE_ELAUNCH;
  hipError_t e = timed(SLIMPIPE_KERNEL_FWD, st, [&] { return small ? launch_fwd_small(a, p->batch, p->head_dim, st) : launch_fwd(a, p->batch, p->head_dim, st); });
  if (e != hipSuccess) return SLIMPIPE_ELAUNCH;
  if (parts && out) {
    MergeArgs m;
    memset(&m, 0, sizeof(m));
    for (int r = 0; r < n_ranges; ++r) {
      m.outs[r] = part_out + (int64_t)r * part_out_elems;
      m.lses[r] = part_lse + (int64_t)r * part_lse_elems;
    }
    m.n_parts = n_ranges; m.part_f32 = 1; m.out_f32 = (p->out_dtype == SLIMPIPE_F32);
    m.head_dim = p->head_dim; m.n_q_heads = p->n_q_heads; m.s_q = p->s_q; m.rows = (int64_t)p->batch * p->s_q;
    m.out = out; m.lse = lse;
    m.o_stride_b = p->o_stride_b; m.o_stride_s = p->o_stride_s; m.o_stride_h = p->o_stride_h;
    e = timed(SLIMPIPE_KERNEL_MERGE, st, [&] { return launch_merge(m, st); });
    if (e != hipSuccess) return SLIMPIPE_ELAUNCH;
  }
  return SLIMPIPE_OK;
}

// One range, or - when the caller lends a workspace and the launch would leave compute units idle - the
// range cut into pieces of equal work whose partial results are merged in the same call.
static int fwd_auto(const slimpipe_attn_params* p, const void* q_slice, const void* const* k_chunks,
                    const void* const* v_chunks, int32_t n_chunks, int64_t chunk_len, void* out, float* lse,
                    void* workspace, size_t workspace_bytes, void* hip_stream) {
  int rc = slimpipe_attn_validate(p, 0);
  if (rc != SLIMPIPE_OK) return rc;
  // workspace: [ticket counter, 256 bytes][partial out of the ranges][partial lse of the ranges]
  if (workspace && !aligned16(workspace)) return SLIMPIPE_EINVAL_ALIGN;
  unsigned* ticket = (workspace && workspace_bytes >= kTicketBytes) ? static_cast<unsigned*>(workspace) : nullptr;
  char* parts_base = ticket ? static_cast<char*>(workspace) + kTicketBytes : static_cast<char*>(workspace);
  const FwdPlan plan = fwd_plan_within(p, workspace ? workspace_bytes : 0);
  const int ranges = plan.ranges;
  if (ranges <= 1)
    return fwd_impl(p, q_slice, k_chunks, v_chunks, n_chunks, chunk_len, 1, &p->kv_begin, &p->kv_end, nullptr, 0, nullptr, 0, out,
                    lse, hip_stream, ticket, plan.head_waves, plan.small);
  int64_t begin[kMaxRanges], end[kMaxRanges];
  equal_work_ranges(p, ranges, begin, end);
  float* part_out = reinterpret_cast<float*>(parts_base);
  float* part_lse = reinterpret_cast<float*>(parts_base + (size_t)ranges * fwd_part_out_bytes(p));
  return fwd_impl(p, q_slice, k_chunks, v_chunks, n_chunks, chunk_len, ranges, begin, end, part_out,
                  (int64_t)(fwd_part_out_bytes(p) / sizeof(float)), part_lse, (int64_t)(stat_bytes(p) / sizeof(float)), out, lse,
                  hip_stream, ticket, plan.head_waves, plan.small);
}

int slimpipe_attn_fwd(const slimpipe_attn_params* p, const void* q_slice, const void* k_prefix,
                      const void* v_prefix, void* out, float* lse, void* workspace, size_t workspace_bytes,
                      void* hip_stream) {
  if (!p) return SLIMPIPE_EINVAL_NULL;
  return fwd_auto(p, q_slice, &k_prefix, &v_prefix, 1, p->kv_capacity > 0 ? p->kv_capacity : 1, out, lse, workspace,
                  workspace_bytes, hip_stream);
}

int slimpipe_attn_fwd_chunked(const slimpipe_attn_params* p, const void* q_slice, const void* const* k_chunks,
                              const void* const* v_chunks, int32_t n_chunks, int64_t chunk_len, void* out, float* lse,
                              void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!p) return SLIMPIPE_EINVAL_NULL;
  return fwd_auto(p, q_slice, k_chunks, v_chunks, n_chunks, chunk_len, out, lse, workspace, workspace_bytes, hip_stream);
}

int slimpipe_attn_fwd_ranges(const slimpipe_attn_params* p, const void* q_slice, const void* const* k_chunks,
                             const void* const* v_chunks, int32_t n_chunks, int64_t chunk_len, int32_t n_ranges,
                             const int64_t* kv_begin, const int64_t* kv_end, float* part_out, float* part_lse, void* out,
                             float* lse, void* hip_stream) {
  if (!p) return SLIMPIPE_EINVAL_NULL;
  if (!part_out || !part_lse) return SLIMPIPE_EINVAL_NULL;
  const int64_t out_elems = (int64_t)p->batch * p->s_q * p->n_q_heads * p->head_dim;
  const int64_t lse_elems = (int64_t)p->batch * p->n_q_heads * p->s_q;
  return fwd_impl(p, q_slice, k_chunks, v_chunks, n_chunks, chunk_len, n_ranges, kv_begin, kv_end, part_out, out_elems, part_lse,
                  lse_elems, out, lse, hip_stream);
}

// Whether a gradient of the call may lie over its out or lse (by the memory they span: tensors that interleave count as well).
static bool gradients_over_saved(const slimpipe_attn_params* p, int32_t n_chunks, int64_t chunk_len, const void* out, const float* lse, const void* dq,
                                 int32_t dq_dtype, float* const* dk_chunks, float* const* dv_chunks) {
  const Span saved[2] = {span_of(out, 2, p->batch, p->s_q, p->n_q_heads, p->head_dim, p->o_stride_b, p->o_stride_s, p->o_stride_h),
                         span_of(lse, 4, 1, 1, 1, (int64_t)p->batch * p->n_q_heads * p->s_q, 1, 1, 1)};
  auto over = [&](const Span& g) { return share_memory(g, saved[0]) || share_memory(g, saved[1]); };
  if (over(span_of(dq, dq_dtype == SLIMPIPE_F32 ? 4 : 2, p->batch, p->s_q, p->n_q_heads, p->head_dim, p->q_stride_b, p->q_stride_s, p->q_stride_h))) return true;
  for (int i = 0; i < n_chunks; ++i) {
    // rows of the chunk that the range holds
    const int64_t lo = p->kv_begin - i * chunk_len, hi = p->kv_end - i * chunk_len;
    const int64_t r0 = lo > 0 ? lo : 0, rows = (hi < chunk_len ? hi : chunk_len) - r0;
    for (float* g : {dk_chunks[i], dv_chunks[i]})
      if (rows > 0 && over(span_of(g + r0 * p->kv_stride_s, 4, p->batch, rows, p->n_kv_heads, p->head_dim, p->kv_stride_b, p->kv_stride_s, p->kv_stride_h)))
        return true;
  }
  return false;
}

static int bwd_impl(const slimpipe_attn_params* p, const void* q_slice, const void* const* k_chunks,
                    const void* const* v_chunks, int32_t n_chunks, int64_t chunk_len, const void* out,
                    const void* d_out, const float* lse, void* dq, int32_t dq_dtype, int32_t dq_accumulate,
                    float* const* dk_chunks, float* const* dv_chunks, int32_t dkv_accumulate, void* workspace,
                    size_t workspace_bytes, void* hip_stream, bool events = true) {
  int rc = slimpipe_attn_validate(p, 1);
  if (rc != SLIMPIPE_OK) return rc;
  if (!q_slice || !out || !d_out || !lse || !dq || !k_chunks || !v_chunks || !dk_chunks || !dv_chunks) return SLIMPIPE_EINVAL_NULL;
  rc = check_chunks(p, n_chunks, chunk_len);
  if (rc != SLIMPIPE_OK) return rc;
  if (dq_dtype != SLIMPIPE_BF16 && dq_dtype != SLIMPIPE_F32) return SLIMPIPE_EINVAL_SHAPE;
  if (dq_accumulate && dq_dtype != SLIMPIPE_F32) return SLIMPIPE_EINVAL_SHAPE;
  if (!aligned16(q_slice) || !aligned16(out) || !aligned16(d_out) || !aligned16(dq) || (reinterpret_cast<uintptr_t>(lse) & 3u))
    return SLIMPIPE_EINVAL_ALIGN;
  if (!workspace || workspace_bytes < delta_bytes(p)) return SLIMPIPE_EWORKSPACE;
  if (!aligned16(workspace)) return SLIMPIPE_EINVAL_ALIGN;
  BwdArgs a;
  memset(&a.kv, 0, sizeof(a.kv));
  memset(a.dk_acc, 0, sizeof(a.dk_acc));
  memset(a.dv_acc, 0, sizeof(a.dv_acc));
  for (int i = 0; i < n_chunks; ++i) {
    if (!dk_chunks[i] || !dv_chunks[i]) return SLIMPIPE_EINVAL_NULL;
    if (p->kv_end > 0 && (!k_chunks[i] || !v_chunks[i])) return SLIMPIPE_EINVAL_NULL;
    if (!aligned16(k_chunks[i]) || !aligned16(v_chunks[i]) || !aligned16(dk_chunks[i]) || !aligned16(dv_chunks[i])) return SLIMPIPE_EINVAL_ALIGN;
    a.kv.k[i] = static_cast<const __bf16*>(k_chunks[i]);
    a.kv.v[i] = static_cast<const __bf16*>(v_chunks[i]);
    a.dk_acc[i] = dk_chunks[i];
    a.dv_acc[i] = dv_chunks[i];
  }
  a.kv.len = chunk_len;
  a.kv.n = n_chunks;
  a.q = static_cast<const __bf16*>(q_slice);
  a.out = static_cast<const __bf16*>(out);
  a.d_out = static_cast<const __bf16*>(d_out);
  a.lse = lse;
  a.delta = static_cast<float*>(workspace);
  a.lse2 = reinterpret_cast<float*>(static_cast<char*>(workspace) + stat_bytes(p));
  // behind the statistics: the ticket counter of the dk/dv kernel (when there is room for it), the partial dk/dv sums
  // of a split query stream, the partial dq of key ranges
  const bool ticket = workspace_bytes >= delta_bytes(p) + kTicketBytes;
  const size_t fixed = delta_bytes(p) + (ticket ? kTicketBytes : 0);
  unsigned* const counters = ticket ? reinterpret_cast<unsigned*>(static_cast<char*>(workspace) + delta_bytes(p)) : nullptr;
  const BwdPlan plan = bwd_plan_within(p, n_chunks, workspace_bytes);
  const int split = plan.split, dq_ranges = plan.dq_ranges;
  a.n_split = split;
  a.part = reinterpret_cast<float*>(static_cast<char*>(workspace) + fixed);
  // the partial dq behind the partial dk/dv
  const size_t used = fixed + split_bytes(p, n_chunks, split);
  a.n_dq_ranges = dq_ranges;
  for (int r = 0; r < kMaxRanges; ++r) a.dq_range_begin[r] = a.dq_range_end[r] = 0;
  if (dq_ranges > 1) {
    equal_work_ranges(p, dq_ranges, a.dq_range_begin, a.dq_range_end);
    a.dq = static_cast<char*>(workspace) + used;
    a.dq_range_stride = (int64_t)(fwd_part_out_bytes(p) / sizeof(float));
    a.dq_stride_h = p->head_dim; a.dq_stride_s = (int64_t)p->n_q_heads * p->head_dim; a.dq_stride_b = a.dq_stride_s * p->s_q;
  } else {
    a.dq_range_begin[0] = p->kv_begin; a.dq_range_end[0] = p->kv_end;
    a.dq = dq;
    a.dq_range_stride = 0;
    a.dq_stride_b = p->q_stride_b; a.dq_stride_s = p->q_stride_s; a.dq_stride_h = p->q_stride_h;
  }
  for (int r = 0; r < dq_ranges; ++r) a.dq_range_end[r] = seen_end(p, a.dq_range_begin[r], a.dq_range_end[r]);
  a.seen_end = seen_end(p, p->kv_begin, p->kv_end);
  a.dq_final = dq;
  a.dq_final_f32 = (dq_dtype == SLIMPIPE_F32); a.dq_final_accumulate = dq_accumulate ? 1 : 0;
  a.nkeys_pad = dkdv_key_tiles(p, n_chunks) * dkdv_keys_per_workgroup();
  a.dkdv_items[0] = (int32_t)(dkdv_key_tiles(p, n_chunks) * split);
  a.dkdv_items[1] = p->n_kv_heads;
  a.dkdv_items[2] = p->batch;
  a.head_waves = plan.head_waves;
  const int64_t blocks = query_blocks(plan.head_waves, p->n_q_heads / p->n_kv_heads);
  if (blocks * p->n_kv_heads * p->batch * dq_ranges > (int64_t)1 << 30) return SLIMPIPE_EINVAL_SHAPE;
  a.dq_items[0] = (int32_t)blocks;
  a.dq_items[1] = p->n_kv_heads;
  a.dq_items[2] = p->batch * dq_ranges;
  // a counter only where there are more items than compute units (otherwise every workgroup starts at once)
  const int64_t cus = compute_units();
  a.dkdv_wgs = (int32_t)cus;
  a.dq_first = plan.dq_first;
  a.dq_tile_keys = dq_tile_keys(p, plan);
  a.dkdv_tile_rows = dkdv_tile_rows(p, plan);
  const bool counted = counters && !plan.both;
  a.ticket_dkdv = (counted && (int64_t)a.dkdv_items[0] * a.dkdv_items[1] * a.dkdv_items[2] > cus) ? counters : nullptr;
  a.ticket_dq = (counted && (int64_t)a.dq_items[0] * a.dq_items[1] * a.dq_items[2] > cus) ? counters + 8 : nullptr;     // [0..7]: dk/dv, [8..15]: dq, one per XCD
  a.items_by_group = items_by_group(p, p->kv_end - p->kv_begin, dq_ranges);
  if ((int64_t)a.dkdv_items[0] * a.dkdv_items[1] * a.dkdv_items[2] > (int64_t)1 << 30) return SLIMPIPE_EINVAL_SHAPE;
  a.s_q = p->s_q; a.n_q_heads = p->n_q_heads; a.n_kv_heads = p->n_kv_heads;
  a.group = p->n_q_heads / p->n_kv_heads; a.causal = p->causal;
  a.dq_f32 = dq_ranges > 1 ? 1 : a.dq_final_f32; a.dq_accumulate = dq_ranges > 1 ? 0 : a.dq_final_accumulate;
  a.dkv_accumulate = dkv_accumulate ? 1 : 0;
  a.q_offset = p->q_offset; a.kv_begin = p->kv_begin; a.kv_end = p->kv_end; a.kv_capacity = p->kv_capacity;
  a.scale = p->scale; a.scale_log2e = p->scale * 1.4426950408889634f;
  a.q_stride_b = p->q_stride_b; a.q_stride_s = p->q_stride_s; a.q_stride_h = p->q_stride_h;
  a.kv_stride_b = p->kv_stride_b; a.kv_stride_s = p->kv_stride_s; a.kv_stride_h = p->kv_stride_h;
  a.o_stride_b = p->o_stride_b; a.o_stride_s = p->o_stride_s; a.o_stride_h = p->o_stride_h;
  a.do_stride_b = p->do_stride_b; a.do_stride_s = p->do_stride_s; a.do_stride_h = p->do_stride_h;
  if (ensure_device_ready() != SLIMPIPE_OK) return SLIMPIPE_ELAUNCH;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  BwdSmallPlan sm = bwd_small_plan(p, plan);
  // out and lse are read before any gradient is written, so that gradients may lie over them: by the delta kernel, ahead of the others; items
  // that read them are in one launch with items that write gradients.
  if (sm.own_stats && gradients_over_saved(p, n_chunks, chunk_len, out, lse, dq, dq_dtype, dk_chunks, dv_chunks)) sm.own_stats = false;
  if (!sm.own_stats &&
      timed(SLIMPIPE_KERNEL_DELTA, st, [&] { return launch_delta(a, p->batch, p->head_dim, st); }, events) != hipSuccess)
    return SLIMPIPE_ELAUNCH;
  if (sm.use) {
    a.dq_first = sm.dq_first;
    return timed(SLIMPIPE_KERNEL_BWD_BOTH, st, [&] { return launch_bwd_small(a, p->batch, p->head_dim, sm.own_stats, sm.key_blocks, st); }, events) == hipSuccess
               ? SLIMPIPE_OK : SLIMPIPE_ELAUNCH;
  }
  if (plan.both) {
    if (timed(SLIMPIPE_KERNEL_BWD_BOTH, st, [&] { return launch_bwd_both(a, p->head_dim, st); }, events) != hipSuccess) return SLIMPIPE_ELAUNCH;
    if ((split > 1 || dq_ranges > 1) &&
        timed(SLIMPIPE_KERNEL_BOTH_REDUCE, st, [&] { return launch_both_reduce(a, p->batch, p->head_dim, st); }, events) != hipSuccess)
      return SLIMPIPE_ELAUNCH;
    return SLIMPIPE_OK;
  }
  if (timed(SLIMPIPE_KERNEL_DQ, st, [&] { return launch_bwd_dq(a, p->batch, p->head_dim, st); }, events) != hipSuccess) return SLIMPIPE_ELAUNCH;
  if (dq_ranges > 1 &&
      timed(SLIMPIPE_KERNEL_DQ_REDUCE, st, [&] { return launch_dq_reduce(a, p->batch, p->head_dim, st); }, events) != hipSuccess)
    return SLIMPIPE_ELAUNCH;
  if (timed(SLIMPIPE_KERNEL_DKDV, st, [&] { return launch_bwd_dkdv(a, p->batch, p->head_dim, st); }, events) != hipSuccess) return SLIMPIPE_ELAUNCH;
  if (split > 1 &&
      timed(SLIMPIPE_KERNEL_DKDV_REDUCE, st, [&] { return launch_dkdv_reduce(a, p->batch, p->head_dim, st); }, events) != hipSuccess)
    return SLIMPIPE_ELAUNCH;
  return SLIMPIPE_OK;
}

int slimpipe_attn_bwd(const slimpipe_attn_params* p, const void* q_slice, const void* k_prefix,
                      const void* v_prefix, const void* out, const void* d_out, const float* lse, void* dq,
                      int32_t dq_dtype, int32_t dq_accumulate, float* dk_acc, float* dv_acc,
                      int32_t dkv_accumulate, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!p) return SLIMPIPE_EINVAL_NULL;
  return bwd_impl(p, q_slice, &k_prefix, &v_prefix, 1, p->kv_capacity > 0 ? p->kv_capacity : 1, out, d_out, lse, dq, dq_dtype,
                  dq_accumulate, &dk_acc, &dv_acc, dkv_accumulate, workspace, workspace_bytes, hip_stream);
}

int slimpipe_attn_bwd_noalloc(const slimpipe_attn_params* p, const void* q_slice, const void* k_prefix,
                              const void* v_prefix, const void* out, const void* d_out, const float* lse, void* dq,
                              int32_t dq_dtype, int32_t dq_accumulate, float* dk_acc, float* dv_acc,
                              int32_t dkv_accumulate, void* hip_stream) {
  if (!p) return SLIMPIPE_EINVAL_NULL;
  int rc = slimpipe_attn_validate(p, 1);
  if (rc != SLIMPIPE_OK) return rc;
  if (delta_bytes(p) > kScratchBytes) return SLIMPIPE_ETOOLARGE;
  void* ws = nullptr;
  if (ensure_device_ready(&ws) != SLIMPIPE_OK || !ws) return SLIMPIPE_ELAUNCH;
  // the two statistics arrays and the ticket counter behind them: no split of the dk/dv query stream, no key ranges for
  // dq (the sums of slimpipe_attn_bwd given a workspace of the minimum size), and no event records of the benchmark switch
  static_assert(kScratchTicketBytes == kTicketBytes, "the counter sits right behind the statistics");
  return bwd_impl(p, q_slice, &k_prefix, &v_prefix, 1, p->kv_capacity > 0 ? p->kv_capacity : 1, out, d_out, lse, dq, dq_dtype,
                  dq_accumulate, &dk_acc, &dv_acc, dkv_accumulate, ws, delta_bytes(p) + kTicketBytes, hip_stream, false);
}

int slimpipe_attn_noalloc_max_rows(void) { return (int)(kScratchBytes / (2 * sizeof(float))); }

int slimpipe_attn_bwd_chunked(const slimpipe_attn_params* p, const void* q_slice, const void* const* k_chunks,
                              const void* const* v_chunks, int32_t n_chunks, int64_t chunk_len, const void* out,
                              const void* d_out, const float* lse, void* dq, int32_t dq_dtype, int32_t dq_accumulate,
                              float* const* dk_chunks, float* const* dv_chunks, int32_t dkv_accumulate, void* workspace,
                              size_t workspace_bytes, void* hip_stream) {
  return bwd_impl(p, q_slice, k_chunks, v_chunks, n_chunks, chunk_len, out, d_out, lse, dq, dq_dtype, dq_accumulate, dk_chunks,
                  dv_chunks, dkv_accumulate, workspace, workspace_bytes, hip_stream);
}

int slimpipe_attn_merge(int32_t n_parts, const void* const* outs, const float* const* lses, int32_t part_dtype,
                        int32_t batch, int32_t s_q, int32_t n_q_heads, int32_t head_dim, void* out,
                        int32_t out_dtype, float* lse, void* hip_stream) {
  if (!outs || !lses || !out || !lse) return SLIMPIPE_EINVAL_NULL;
  if (n_parts < 1 || n_parts > 16) return SLIMPIPE_EINVAL_SHAPE;
  if (batch <= 0 || s_q <= 0 || n_q_heads <= 0 || head_dim <= 0 || head_dim % 8 != 0) return SLIMPIPE_EINVAL_SHAPE;
  if ((part_dtype != SLIMPIPE_BF16 && part_dtype != SLIMPIPE_F32) ||
      (out_dtype != SLIMPIPE_BF16 && out_dtype != SLIMPIPE_F32))
    return SLIMPIPE_EINVAL_SHAPE;
  MergeArgs a;
  memset(&a, 0, sizeof(a));
  for (int i = 0; i < n_parts; ++i) {
    if (!outs[i] || !lses[i]) return SLIMPIPE_EINVAL_NULL;
    if (!aligned16(outs[i]) || (reinterpret_cast<uintptr_t>(lses[i]) & 3u)) return SLIMPIPE_EINVAL_ALIGN;
    a.outs[i] = outs[i];
    a.lses[i] = lses[i];
  }
  if (!aligned16(out) || (reinterpret_cast<uintptr_t>(lse) & 3u)) return SLIMPIPE_EINVAL_ALIGN;
  a.n_parts = n_parts; a.part_f32 = (part_dtype == SLIMPIPE_F32); a.out_f32 = (out_dtype == SLIMPIPE_F32);
  a.head_dim = head_dim; a.n_q_heads = n_q_heads; a.s_q = s_q; a.rows = (int64_t)batch * s_q;
  a.out = out; a.lse = lse;
  a.o_stride_h = head_dim; a.o_stride_s = (int64_t)n_q_heads * head_dim; a.o_stride_b = a.o_stride_s * s_q;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  hipError_t e = timed(SLIMPIPE_KERNEL_MERGE, st, [&] { return launch_merge(a, st); });
  return e == hipSuccess ? SLIMPIPE_OK : SLIMPIPE_ELAUNCH;
}

int slimpipe_attn_finalize_bf16(const float* acc, void* dst_bf16, int64_t n_elems, void* hip_stream) {
  if (!acc || !dst_bf16) return SLIMPIPE_EINVAL_NULL;
  if (n_elems < 0) return SLIMPIPE_EINVAL_SHAPE;
  if (!aligned16(acc) || (reinterpret_cast<uintptr_t>(dst_bf16) & 7u)) return SLIMPIPE_EINVAL_ALIGN;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  hipError_t e = timed(SLIMPIPE_KERNEL_FINALIZE, st, [&] { return launch_finalize(acc, static_cast<__bf16*>(dst_bf16), n_elems, st); });
  return e == hipSuccess ? SLIMPIPE_OK : SLIMPIPE_ELAUNCH;
}

int slimpipe_attn_mfma_rate(int random_operands, float* sink, double* tflops, void* hip_stream) {
  if (!sink || !tflops) return SLIMPIPE_EINVAL_NULL;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const int iters = 20000, wgs = 8 * compute_units();
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) return SLIMPIPE_ELAUNCH;
  int rc = SLIMPIPE_OK;
  float ms = 0.f;
  // one untimed launch to get the clocks where they settle, then the timed one
  if (launch_mfma_rate(random_operands, iters, wgs, sink, st) != hipSuccess) rc = SLIMPIPE_ELAUNCH;
  if (rc == SLIMPIPE_OK && (hipEventRecord(e0, st) != hipSuccess || launch_mfma_rate(random_operands, iters, wgs, sink, st) != hipSuccess ||
                            hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                            hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
    rc = SLIMPIPE_ELAUNCH;
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc == SLIMPIPE_OK) *tflops = (double)wgs * 8 * 4 * iters * 32768.0 / (ms * 1e-3) / 1e12;
  return rc;
}

int slimpipe_attn_xcd_rate(int32_t iters, int32_t workgroups, int64_t* t_start, int64_t* t_end, uint32_t* xcc, void* hip_stream) {
  if (!t_start || !t_end || !xcc) return SLIMPIPE_EINVAL_NULL;
  if (iters < 1 || workgroups < 1 || workgroups > 1 << 16) return SLIMPIPE_EINVAL_SHAPE;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  if (launch_xcd_rate(iters, workgroups, reinterpret_cast<long long*>(t_start), reinterpret_cast<long long*>(t_end), xcc, st) != hipSuccess)
    return SLIMPIPE_ELAUNCH;
  return hipStreamSynchronize(st) == hipSuccess ? SLIMPIPE_OK : SLIMPIPE_ELAUNCH;
}

int slimpipe_attn_dq_atomic_probe(float* dq, int32_t s_q, int32_t heads, int32_t key_tiles, int32_t rows_per_step,
                                  int32_t placement, int32_t rotate, int32_t filler_mfma, int32_t with_atomics,
                                  uint32_t* xcc_mismatch, double* ms, void* hip_stream) {
  if (!dq || !xcc_mismatch || !ms) return SLIMPIPE_EINVAL_NULL;
  if (s_q <= 0 || heads <= 0 || key_tiles <= 0 || (rows_per_step != 32 && rows_per_step != 64) || s_q % rows_per_step != 0 ||
      filler_mfma < 0 || filler_mfma % 4 != 0 || (int64_t)key_tiles * heads > 1 << 20)
    return SLIMPIPE_EINVAL_SHAPE;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  // on failure *ms = -(1000 * step + HIP error code), so that a benchmark log names the call that failed
  float t = 0.f;
  int step = 0;
  hipError_t e = hipSuccess;
  auto run = [&](hipError_t r) { ++step; if (e == hipSuccess && r != hipSuccess) { e = r; return false; } return e == hipSuccess; };
  run(hipEventCreate(&e0)) && run(hipEventCreate(&e1)) && run(hipEventRecord(e0, st)) &&
      run(launch_dq_atomic_probe(dq, s_q, heads, key_tiles, rows_per_step, placement, rotate, filler_mfma, with_atomics, xcc_mismatch, st)) &&
      run(hipEventRecord(e1, st)) && run(hipEventSynchronize(e1)) && run(hipEventElapsedTime(&t, e0, e1));
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  *ms = e == hipSuccess ? (double)t : -(1000.0 * step + (double)(int)e);
  return e == hipSuccess ? SLIMPIPE_OK : SLIMPIPE_ELAUNCH;
}

const char* slimpipe_attn_strerror(int code) {
  switch (code) {
    case SLIMPIPE_OK: return "ok";
    case SLIMPIPE_EINVAL_NULL: return "a required pointer is NULL";
    case SLIMPIPE_EINVAL_SHAPE: return "invalid shape, head_dim, scale, flag or dtype";
    case SLIMPIPE_EINVAL_RANGE: return "invalid q_offset / kv range / kv_capacity";
    case SLIMPIPE_EINVAL_STRIDE: return "strides must be positive multiples of 8 elements and cover head_dim";
    case SLIMPIPE_EINVAL_ALIGN: return "pointer not 16-byte aligned";
    case SLIMPIPE_EWORKSPACE: return "workspace missing or too small";
    case SLIMPIPE_ELAUNCH: return "HIP launch failed";
    case SLIMPIPE_ETOOLARGE: return "batch * heads * rows exceeds the fixed scratch of slimpipe_attn_bwd_noalloc";
    default: return "unknown slimpipe status";
  }
}

}  // extern "C"
