// Small calls.  Forward: a workgroup owns 32 query rows of one head and its 8 wavefronts share out their keys.
//
// What bounds a small call is a chain: a 256-row block walks its keys tile after tile behind barriers on a chip that is mostly idle, and
// key ranges shorten the chain only at the price of a merge launch.  Here eight waves walk eight tiles of the keys at the same time,
// each with a K and a V tile of its own in LDS, copied by itself and waited for by itself (no barrier in the loop), and their
// partial results meet in LDS.  512 rows on 2048 keys, 4 heads of 64 (64 workgroups): 18.1 -> 10.9 us; 512 rows of 8 heads of 128 on one
// K/V head, 2048 keys: 34.6 -> 15.9.  A wave's step (32 keys, 64 at head_dim 64) takes 1.3 us, 1 of which is the compute unit's path to
// memory: eight K and V tiles are 128 KB at 64 bytes a clock.  One K and one V tile per wave are all of LDS, so K of the next step is
// copied during softmax and P V, V during the scores and the softmax; what a wave does not need it does not ask for (a last tile copied
// once more, and Q by loads that the compiler waits for together with every copy: 11.9 and 18.1 us).  Touching the lines of later
// tiles ahead of their copies makes it slower (12.5), the path being what is short.  Which calls come here: fwd_plan_within in api.hip.
// A wave's probabilities are rounded to bf16 relative to the maximum of the wave's own keys, so the roundings of P V fall elsewhere than in
// the 256-row blocks (2.5e-3 of the result in the 2-norm).  There are as many bits; the error against 64 bits is smaller: float32 out,
// 512 rows on 512 keys of 64, 1.12e-3 (blocks 1.17e-3), 280 rows on 1486 keys of 128, 1.32e-3 (1.52e-3), at scores of 4 times the size 2.4e-4 (5.1e-4).
#include "kernels.hpp"
#include "tile_common.hpp"

namespace slimpipe {

// Row of a key in the chunk that holds it; `first` is the first chunk's base, asked for ahead (the only one, as a rule): a pointer that is looked
// up by a computed chunk number is a second trip to the kernel's arguments before the first copy (with the block index as a grid of three
// dimensions instead of two divisions 512 rows on 2048 keys, 8/1 heads of 128, 16.9 -> 15.9 us).
SP_DEV const bf16_t* kv_row(const bf16_t* const* table, const bf16_t* first, const KvChunks& kv, int64_t key, int64_t stride_s) {
  if (kv.n <= 1) return first + key * stride_s;
  const int chunk = kv_chunk_of(kv, key);
  return table[chunk] + (key - (int64_t)chunk * kv.len) * stride_s;
}

template <int D>
struct FwdSmall {
  static constexpr int NW = 8, BN = D == 64 ? 64 : 32, KB = BN / 32, KS = D / 16, DB = D / 32;
  static constexpr int TILE_BYTES = BN * D * 2, WAVE_BYTES = 2 * TILE_BYTES;
  static constexpr int ROW = D + 4;                      // floats per row of a wave's partial output (padded against bank conflicts)
  static constexpr int PART_BYTES = 32 * ROW * 4, STAT_BASE = NW * PART_BYTES, COMBINE_BYTES = STAT_BASE + NW * 64 * 4;
  static constexpr int Q_BASE = NW * WAVE_BYTES, TILES_END = Q_BASE + 32 * D * 2;      // the query rows, behind the tiles
  static constexpr int LDS = TILES_END > COMBINE_BYTES ? TILES_END : COMBINE_BYTES;
};

template <int D>
__global__ __launch_bounds__(512) void attn_fwd_small_kernel(const FwdArgs a) {
  using F = FwdSmall<D>;
  constexpr int NW = F::NW, BN = F::BN, KB = F::KB, KS = F::KS, DB = F::DB;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, ql = lane & 31;
  const int wave_u = __builtin_amdgcn_readfirstlane(tid >> 6);
  // block index = (query head, 32-row block of a head, batch index x range), row blocks with the longest key ranges first
  const int row_blocks = a.items[0], h = blockIdx.x, rb = blockIdx.y;
  int b = blockIdx.z, range = 0;
  if (a.n_ranges > 1) {
    b = __builtin_amdgcn_readfirstlane(b / a.n_ranges);
    range = blockIdx.z - b * a.n_ranges;
  }
  const int row0 = (row_blocks - 1 - rb) * 32, hk = __builtin_amdgcn_readfirstlane(h / a.group);
  const int myrow = row0 + ql;
  const int64_t kv_begin = a.range_begin[range], kv_end = a.range_end[range];
  int64_t hi = kv_end;
  if (a.causal) {
    const int64_t lim = a.q_offset + (row0 + 32 < a.s_q ? row0 + 32 : a.s_q);
    hi = hi < lim ? hi : lim;
  }
  const int64_t lo = kv_grid_origin(kv_begin, a.kv.n, BN);
  const int nt = hi > kv_begin ? (int)((hi - lo + BN - 1) / BN) : 0;
  const int before = (int)(kv_begin - lo);               // rows of tile 0 before the range
  const float c = a.scale_log2e;

  f32x16 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  const unsigned smem_lds = lds_addr(smem), k_lds = smem_lds + wave_u * F::WAVE_BYTES, v_lds = k_lds + F::TILE_BYTES;
  RpBase<D> lo_k;
  TrBase<D> lo_v;
  lo_k.init(lane, (int)k_lds);
  lo_v.init(lane, (int)v_lds);
  const int64_t head_off = (int64_t)b * a.kv_stride_b + (int64_t)hk * a.kv_stride_h;
  const uint32_t row_bytes = (uint32_t)a.kv_stride_s * 2;
  WaveDma<D, BN> dma;
  dma.init(lane, row_bytes);
  const bf16_t *const k_first = a.kv.k[0], *const v_first = a.kv.v[0];
  auto copy = [&](bool k, int t, int first) {
    // (a tile lies inside one chunk; rows outside the range are clamped to its first and last key)
    const int64_t key0 = lo + (int64_t)t * BN, left = kv_end - key0;
    const bf16_t* base = uniform_ptr(kv_row(k ? a.kv.k : a.kv.v, k ? k_first : v_first, a.kv, key0, a.kv_stride_s) + head_off);
    dma.copy(k ? k_lds : v_lds, base, row_bytes, first, left < BN ? (int)left : BN, lane);
  };
  constexpr int PASSES = WaveDma<D, BN>::PASSES;
  // The query rows, one copy instruction per wave (as far as there are any).  Not by ordinary loads: the compiler counts those alone, so
  // that in front of the first use of Q, in the loop, it would wait for every copy that is under way.
  if (wave_u < WaveDma<D, 32>::PASSES) {
    const bf16_t* qbase = uniform_ptr(a.q + (int64_t)b * a.q_stride_b + (int64_t)row0 * a.q_stride_s + (int64_t)h * a.q_stride_h);
    WaveDma<D, 32>::copy_pass(smem_lds + F::Q_BASE, qbase, (uint32_t)a.q_stride_s * 2, a.s_q - row0, lane, wave_u);
  }
  int t = wave_u;                                        // tiles w, w + 8, w + 16, .. are this wave's
  if (t < nt) {
    const int first = t == 0 ? before : 0;
    copy(true, t, first);
    copy(false, t, first);
    wait_copies<2 * PASSES>();
  } else {
    wait_async();
  }
  __syncthreads();                                       // the query rows have landed
  RpBase<D> lo_q;
  lo_q.init(lane, (int)smem_lds + F::Q_BASE);
  bf16x8 q[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) q[ks] = lds_rp<D>(lo_q, ks, 0);
  for (; t < nt; t += NW) {
    const int tn = t + NW;
    wait_copies<PASSES>();                               // K has landed (the copies of V may still be under way)
    f32x16 s[KB];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const f32x16 zero = {0};
        s[kb] = mfma32(lds_rp<D>(lo_k, ks, kb * 32 * D * 2), q[ks], ks == 0 ? zero : s[kb]);
      }
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) asm volatile("" : "+v"(s[kb]));      // the reads of K are done before K is copied over
    if (tn < nt) copy(true, tn, 0);
    const int64_t key0 = lo + (int64_t)t * BN;
    if (key0 < kv_begin || key0 + BN > kv_end || (a.causal && key0 + BN - 1 > a.q_offset + row0)) {
      const int64_t kmin = kv_begin - key0;
      int64_t kmax = kv_end - 1;
      if (a.causal && a.q_offset + myrow < kmax) kmax = a.q_offset + myrow;
      kmax -= key0;
      const int kmin_lane = (kmin < 0 ? 0 : (int)kmin) - 4 * g, kmax_lane = (kmax < -1 ? -1 : (kmax > BN ? BN : (int)kmax)) - 4 * g;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int key = kb * 32 + 8 * (i >> 2) + (i & 3);
          s[kb][i] = ((key >= kmin_lane) & (key <= kmax_lane)) ? s[kb][i] : -INFINITY;
        }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int i = 0; i < 16; i += 2) mx = fmaxf(fmaxf(s[kb][i], s[kb][i + 1]), mx);
    mx = xhalf_max(mx);
    const float m_new = fmaxf(m_run, mx * c), m_eff = m_new == -INFINITY ? 0.f : m_new;
    if (__builtin_amdgcn_ballot_w64(m_new != m_run) != 0) {
      const float alpha = exp2_fast(m_run - m_eff);      // m_run = -inf -> 0
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
    }
    m_run = m_new;
    bf16x8 p[KB][2];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
      for (int i = 0; i < 16; ++i) s[kb][i] = __builtin_fmaf(s[kb][i], c, -m_eff);
#pragma unroll
      for (int i = 0; i < 16; ++i) s[kb][i] = exp2_fast(s[kb][i]);
      float sum[4] = {s[kb][0], s[kb][1], s[kb][2], s[kb][3]};
#pragma unroll
      for (int i = 4; i < 16; ++i) sum[i & 3] += s[kb][i];
      l_run += (sum[0] + sum[1]) + (sum[2] + sum[3]);
      p[kb][0] = pack8(s[kb], 0);
      p[kb][1] = pack8(s[kb], 8);
    }
    // V has landed (the copies of the next K may still be under way)
    if (tn < nt) wait_copies<PASSES>();
    else wait_copies<0>();
#pragma unroll
    for (int blk = 0; blk < 2 * KB; ++blk)
#pragma unroll
      for (int db = 0; db < DB; ++db) o[db] = mfma32(lds_tr<D>(lo_v, db, blk * 16 * D * 2), p[blk / 2][blk % 2], o[db]);
#pragma unroll
    for (int db = 0; db < DB; ++db) asm volatile("" : "+v"(o[db]));      // the reads of V are done before V is copied over
    if (tn < nt) copy(false, tn, 0);
  }
  __syncthreads();                                       // nobody reads or copies a tile any more
  // the eight partial results meet in LDS: out = sum of exp2(m_w - m) o_w over sum of exp2(m_w - m) l_w
  float* const part = reinterpret_cast<float*>(smem) + wave_u * (F::PART_BYTES / 4);
  float* const stat = reinterpret_cast<float*>(smem + F::STAT_BASE);
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const f32x4 v = {o[db][4 * i4], o[db][4 * i4 + 1], o[db][4 * i4 + 2], o[db][4 * i4 + 3]};
      *reinterpret_cast<f32x4*>(part + ql * F::ROW + 32 * db + 8 * i4 + 4 * g) = v;
    }
  const float l_tot = xhalf_sum(l_run);
  if (g == 0) {
    stat[wave_u * 64 + ql] = m_run;
    stat[wave_u * 64 + 32 + ql] = l_tot;
  }
  __syncthreads();
  constexpr int PER = D / 16;                            // head_dim elements of a thread, 16 threads a row
  const int r = tid >> 4, d0 = (tid & 15) * PER;
  float mw[NW], m = -INFINITY;
#pragma unroll
  for (int w = 0; w < NW; ++w) { mw[w] = stat[w * 64 + r]; m = fmaxf(m, mw[w]); }
  const float m_eff = m == -INFINITY ? 0.f : m;
  float l = 0.f;
  f32x4 acc[PER / 4];
#pragma unroll
  for (int j = 0; j < PER / 4; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const float e = exp2_fast(mw[w] - m_eff);
    l += e * stat[w * 64 + 32 + r];
#pragma unroll
    for (int j = 0; j < PER / 4; ++j) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(smem) + w * (F::PART_BYTES / 4) + r * F::ROW + d0 + 4 * j);
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[j][k] += e * v[k];
    }
  }
  const int row = row0 + r;
  if (row < a.s_q) {
    const bool has = l > 0.f;
    const float inv = has ? 1.0f / l : 0.f;
    if (d0 == 0) a.lse[(int64_t)range * a.lse_range_stride + ((int64_t)b * a.n_q_heads + h) * a.s_q + row] = has ? (m + __builtin_log2f(l)) * kLn2 : -INFINITY;
    const int64_t ob = (int64_t)range * a.out_range_stride + (int64_t)b * a.o_stride_b + (int64_t)row * a.o_stride_s + (int64_t)h * a.o_stride_h + d0;
#pragma unroll
    for (int j = 0; j < PER / 4; ++j) {
      const f32x4 v = {acc[j][0] * inv, acc[j][1] * inv, acc[j][2] * inv, acc[j][3] * inv};
      if (a.out_f32) *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.out) + ob + 4 * j) = v;
      else *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16_t*>(a.out) + ob + 4 * j) = __builtin_convertvector(v, bf16x4);
    }
  }
}

hipError_t launch_fwd_small(const FwdArgs& a, int batch, int head_dim, hipStream_t st) {
  const dim3 grid((unsigned)a.n_q_heads, (unsigned)a.items[0], (unsigned)(batch * a.n_ranges)), block(512);      // (y: of less than 256 blocks of 256 rows; z: fwd_impl checks it)
  if (head_dim == 128) hipLaunchKernelGGL(attn_fwd_small_kernel<128>, grid, block, FwdSmall<128>::LDS, st, a);
  else hipLaunchKernelGGL(attn_fwd_small_kernel<64>, grid, block, FwdSmall<64>::LDS, st, a);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------ backward
// The same idea for both gradients, in one launch: a workgroup owns 32 query rows (dq) or 32 keys
// (dk/dv) and its eight waves share out the keys, or the query tiles of all heads of the group, each with tiles of its own; the
// eight partial sums meet in LDS and are added up in wave order (bit-reproducible).  No partial sums in memory, no reduce launch.
// 512 rows on 2048 keys, 4 heads of 64: 30.2 -> 13.4 us for the call (16.6 with one key block an item; 17.2 with rows of Q, dO and K loaded by
// every wave, a row a lane, and a delta kernel before it; 512 rows on 512 keys 13.3 -> 10.8).  A step of dk/dv (32 query rows of a wave) takes 1 us at
// head_dim 64, where the tiles are double-buffered, and 2 us at 128, where one Q and one dO tile per wave are all of LDS and the
// copy of the next waits for the sums of this one.  Which calls come here: bwd_small_plan in api.hip.
template <int D>
struct BwdSmall {
  static constexpr int NW = 8, KS = D / 16, DB = D / 32;
  static constexpr int ROW = D + 4, PART_BYTES = 32 * ROW * 4;
  // dq: a K and a V tile of BN keys per wave
  static constexpr int BN = D == 64 ? 64 : 32, KB = BN / 32, KV_BYTES = BN * D * 2;
  // ... and the workgroup's rows of Q, dO and (own statistics) O
  static constexpr int ROWS_BYTES = 32 * D * 2, Q_BASE = NW * 2 * KV_BYTES, DO_BASE = Q_BASE + ROWS_BYTES, O_BASE = DO_BASE + ROWS_BYTES;
  // dk/dv: BUF x (Q and dO tile of 32 rows, their statistics) per wave, and the V and K rows of the workgroup
  static constexpr int BUF = D == 64 ? 2 : 1, TILE_BYTES = 32 * D * 2, SET_BYTES = 2 * TILE_BYTES + 256;
  static constexpr int MAX_BLOCKS = D == 64 ? 2 : 1;      // of 32 keys a workgroup can own
  static constexpr int V_BASE = NW * BUF * SET_BYTES, K_BASE = V_BASE + MAX_BLOCKS * TILE_BYTES;
  static constexpr int max3(int a, int b, int c) { return a > b ? (a > c ? a : c) : (b > c ? b : c); }
  static constexpr int LDS = max3(O_BASE + ROWS_BYTES, K_BASE + MAX_BLOCKS * TILE_BYTES, NW * PART_BYTES);
  static constexpr int GRADS = 2 * NW * PART_BYTES <= LDS ? 2 : 1;      // of dk and dv, whose partial sums fit LDS at a time
};

// Elements d0 .. d0 + 4 * N - 1 of row r of the sum of WAVES waves' partial results, the first at `parts`.
template <int D, int WAVES, int N>
SP_DEV void sum_parts(const char* parts, int r, int d0, f32x4 (&sum)[N]) {
  using S = BwdSmall<D>;
#pragma unroll
  for (int j = 0; j < N; ++j) sum[j] = *reinterpret_cast<const f32x4*>(parts + (r * S::ROW + d0 + 4 * j) * 4);
#pragma unroll
  for (int w = 1; w < WAVES; ++w)
#pragma unroll
    for (int j = 0; j < N; ++j) sum[j] += *reinterpret_cast<const f32x4*>(parts + w * S::PART_BYTES + (r * S::ROW + d0 + 4 * j) * 4);
}
// A wave's accumulators (lane = column of the C layout, registers = head_dim) into its partial result, `factor` times.
template <int D>
SP_DEV void put_part(char* part, const f32x16 (&acc)[D / 32], float factor, int ql, int g) {
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const f32x4 v = {acc[db][4 * i4] * factor, acc[db][4 * i4 + 1] * factor, acc[db][4 * i4 + 2] * factor, acc[db][4 * i4 + 3] * factor};
      *reinterpret_cast<f32x4*>(part + (ql * BwdSmall<D>::ROW + 32 * db + 8 * i4 + 4 * g) * 4) = v;
    }
}

// c + a . b
SP_DEV float dot8(bf16x8 a, bf16x8 b, float c) {
#pragma unroll
  for (int j = 0; j < 8; j += 2) c = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{a[j], a[j + 1]}, bf16x2{b[j], b[j + 1]}, c, false);
  return c;
}
// Sum over aligned groups of N = 8 or 16 lanes, in all of them.
template <int N>
SP_DEV float row_sum(float x) {
  static_assert(N == 8 || N == 16, "within a DPP row");
  x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, true));       // lane ^ 1
  x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x4E, 0xF, 0xF, true));       // lane ^ 2
  x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x141, 0xF, 0xF, true));      // the other quad of eight lanes
  if constexpr (N == 16) x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x140, 0xF, 0xF, true));      // the other half of 16
  return x;
}
// lse in log2 units; +inf for a row that saw no key, so that its p are exp2(-inf) = 0
SP_DEV float lse_log2(float l) { return l == -INFINITY ? INFINITY : l * kLog2e; }

// index -> (query head, 32-row block of a head, batch index).  OWN_STATS: the item works out -dO . O of its rows from out and lse;
// otherwise the delta kernel has (and nothing of this launch reads out or lse: gradients may lie over them).
template <int D, bool OWN_STATS>
SP_DEV void dq_small_item(const BwdArgs& a, int item, char* smem) {
  using S = BwdSmall<D>;
  constexpr int NW = S::NW, BN = S::BN, KB = S::KB, KS = S::KS, DB = S::DB;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, ql = lane & 31;
  const int wave_u = __builtin_amdgcn_readfirstlane(tid >> 6);
  item = __builtin_amdgcn_readfirstlane(item);
  const int row_blocks = (int)(((int64_t)a.s_q + 31) / 32), per_b = row_blocks * a.n_q_heads;
  const int b = __builtin_amdgcn_readfirstlane(item / per_b), hb = item - b * per_b;
  const int rb = __builtin_amdgcn_readfirstlane(hb / a.n_q_heads), h = hb - rb * a.n_q_heads;
  const int row0 = (row_blocks - 1 - rb) * 32, hk = __builtin_amdgcn_readfirstlane(h / a.group);
  const int myrow = row0 + ql, myrow_c = myrow < a.s_q ? myrow : a.s_q - 1;
  const int64_t kv_end = a.seen_end;
  int64_t hi = kv_end;
  if (a.causal) {
    const int64_t lim = a.q_offset + (row0 + 32 < a.s_q ? row0 + 32 : a.s_q);
    hi = hi < lim ? hi : lim;
  }
  const int64_t lo = kv_grid_origin(a.kv_begin, a.kv.n, BN);
  const int nt = hi > a.kv_begin ? (int)((hi - lo + BN - 1) / BN) : 0;
  const int before = (int)(a.kv_begin - lo);             // rows of tile 0 before the range
  const float c = a.scale_log2e;

  const unsigned smem_lds = lds_addr(smem);
  // The rows of Q, dO and (OWN_STATS) O, one copy instruction of each per wave (as far as there are any): eight waves that each load their
  // lane's row of them are 64 lines an instruction, a lane a clock.
  if (wave_u < WaveDma<D, 32>::PASSES) {
    const int rows = a.s_q - row0;
    WaveDma<D, 32>::copy_pass(smem_lds + S::Q_BASE, uniform_ptr(a.q + (int64_t)b * a.q_stride_b + (int64_t)row0 * a.q_stride_s + (int64_t)h * a.q_stride_h),
                              (uint32_t)a.q_stride_s * 2, rows, lane, wave_u);
    WaveDma<D, 32>::copy_pass(smem_lds + S::DO_BASE, uniform_ptr(a.d_out + (int64_t)b * a.do_stride_b + (int64_t)row0 * a.do_stride_s + (int64_t)h * a.do_stride_h),
                              (uint32_t)a.do_stride_s * 2, rows, lane, wave_u);
    if constexpr (OWN_STATS)
      WaveDma<D, 32>::copy_pass(smem_lds + S::O_BASE, uniform_ptr(a.out + (int64_t)b * a.o_stride_b + (int64_t)row0 * a.o_stride_s + (int64_t)h * a.o_stride_h),
                                (uint32_t)a.o_stride_s * 2, rows, lane, wave_u);
  }
  f32x16 dq[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) dq[db][i] = 0.f;

  const unsigned k_lds = smem_lds + wave_u * 2 * S::KV_BYTES, v_lds = k_lds + S::KV_BYTES;
  RpBase<D> lo_k, lo_v;
  TrBase<D> lo_kt;
  lo_k.init(lane, (int)k_lds);
  lo_v.init(lane, (int)v_lds);
  lo_kt.init(lane, (int)k_lds);
  // statistics of the lane's row: lse in log2 units (+inf for a row that saw no key) and -dO . O, the initial accumulator of dP
  const int64_t stat = ((int64_t)b * a.n_q_heads + h) * a.s_q + myrow_c;
  float lse2 = OWN_STATS ? a.lse[stat] : a.lse2[stat], ndelta = OWN_STATS ? 0.f : a.delta[stat];
  const int64_t head_off = (int64_t)b * a.kv_stride_b + (int64_t)hk * a.kv_stride_h;
  const uint32_t row_bytes = (uint32_t)a.kv_stride_s * 2;
  WaveDma<D, BN> dma;
  dma.init(lane, row_bytes);
  const bf16_t *const k_first = a.kv.k[0], *const v_first = a.kv.v[0];
  auto copy = [&](bool k, int t, int first) {
    const int64_t key0 = lo + (int64_t)t * BN, left = kv_end - key0;      // (a tile lies inside one chunk; clamped as in the forward)
    const bf16_t* base = uniform_ptr(kv_row(k ? a.kv.k : a.kv.v, k ? k_first : v_first, a.kv, key0, a.kv_stride_s) + head_off);
    dma.copy(k ? k_lds : v_lds, base, row_bytes, first, left < BN ? (int)left : BN, lane);
  };
  int t = wave_u;                                        // tiles w, w + 8, w + 16, .. are this wave's
  if (t < nt) {
    const int first = t == 0 ? before : 0;
    copy(true, t, first);
    copy(false, t, first);
    wait_copies<2 * WaveDma<D, BN>::PASSES>();
  } else {
    wait_async();
  }
  __syncthreads();                                       // the rows have landed
  bf16x8 q[KS], dO[KS];
  {
    RpBase<D> lo_r;
    lo_r.init(lane, (int)smem_lds + S::Q_BASE);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      q[ks] = lds_rp<D>(lo_r, ks, 0);
      dO[ks] = lds_rp<D>(lo_r, ks, S::ROWS_BYTES);
      if constexpr (OWN_STATS) ndelta = dot8(lds_rp<D>(lo_r, ks, 2 * S::ROWS_BYTES), dO[ks], ndelta);
    }
  }
  if constexpr (OWN_STATS) {
    ndelta = -xhalf_sum(ndelta);
    lse2 = lse_log2(lse2);
  }
  for (; t < nt; t += NW) {
    const int tn = t + NW;
    wait_copies<0>();
    f32x16 s[KB], dp[KB];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const f32x16 zero = {0};
        s[kb] = mfma32(lds_rp<D>(lo_k, ks, kb * 32 * D * 2), q[ks], ks == 0 ? zero : s[kb]);
      }
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) dp[kb][i] = ndelta;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) dp[kb] = mfma32(lds_rp<D>(lo_v, ks, kb * 32 * D * 2), dO[ks], dp[kb]);
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) asm volatile("" : "+v"(dp[kb]));      // the reads of V are done before V is copied over
    if (tn < nt) copy(false, tn, 0);
    const int64_t key0 = lo + (int64_t)t * BN;
    if (key0 < a.kv_begin || key0 + BN > kv_end || (a.causal && key0 + BN - 1 > a.q_offset + row0)) {
      const int64_t kmin = a.kv_begin - key0;
      int64_t kmax = kv_end - 1;
      if (a.causal && a.q_offset + myrow < kmax) kmax = a.q_offset + myrow;
      kmax -= key0;
      const int kmin_lane = (kmin < 0 ? 0 : (int)kmin) - 4 * g, kmax_lane = (kmax < -1 ? -1 : (kmax > BN ? BN : (int)kmax)) - 4 * g;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int key = kb * 32 + 8 * (i >> 2) + (i & 3);
          s[kb][i] = ((key >= kmin_lane) & (key <= kmax_lane)) ? s[kb][i] : -INFINITY;      // exp2(-inf) = 0
        }
    }
    bf16x8 ds[KB][2];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
      for (int i = 0; i < 16; ++i) s[kb][i] = __builtin_fmaf(s[kb][i], c, -lse2);
#pragma unroll
      for (int i = 0; i < 16; ++i) s[kb][i] = exp2_fast(s[kb][i]);
#pragma unroll
      for (int i = 0; i < 16; ++i) s[kb][i] *= dp[kb][i];                  // dp holds dP - delta
      ds[kb][0] = pack8(s[kb], 0);
      ds[kb][1] = pack8(s[kb], 8);
    }
#pragma unroll
    for (int blk = 0; blk < 2 * KB; ++blk)
#pragma unroll
      for (int db = 0; db < DB; ++db) dq[db] = mfma32(lds_tr<D>(lo_kt, db, blk * 16 * D * 2), ds[blk / 2][blk % 2], dq[db]);
#pragma unroll
    for (int db = 0; db < DB; ++db) asm volatile("" : "+v"(dq[db]));      // the reads of K are done before K is copied over
    if (tn < nt) copy(true, tn, 0);
  }
  __syncthreads();                                       // nobody reads or copies a tile any more
  put_part<D>(smem + wave_u * S::PART_BYTES, dq, a.scale, ql, g);
  __syncthreads();
  const int r = tid >> 4, d0 = (tid & 15) * (D / 16), row = row0 + r;
  if (row < a.s_q) {
    f32x4 sum[D / 64];
    sum_parts<D, NW>(smem, r, d0, sum);
    const int64_t base = (int64_t)b * a.q_stride_b + (int64_t)row * a.q_stride_s + (int64_t)h * a.q_stride_h + d0;
#pragma unroll
    for (int j = 0; j < D / 64; ++j) {
      if (a.dq_final_f32) {
        f32x4* dst = reinterpret_cast<f32x4*>(static_cast<float*>(a.dq_final) + base + 4 * j);
        if (a.dq_final_accumulate) sum[j] += *dst;
        *dst = sum[j];
      } else {
        *reinterpret_cast<bf16x4*>(static_cast<bf16_t*>(a.dq_final) + base + 4 * j) = __builtin_convertvector(sum[j], bf16x4);
      }
    }
  }
}

// index -> (BLOCKS blocks of 32 keys, kv head, batch index).  With two blocks four of the waves belong to each and walk its query tiles.
// OWN_STATS: the wave works out the statistics of a tile's rows itself; otherwise the delta kernel has, and they are copied with the tile.
template <int D, bool OWN_STATS, int BLOCKS>
SP_DEV void dkdv_small_item(const BwdArgs& a, int item, char* smem) {
  using S = BwdSmall<D>;
  constexpr int NW = S::NW / BLOCKS, KS = S::KS, DB = S::DB, BUF = S::BUF, TILE_BYTES = S::TILE_BYTES;      // NW: waves of a key block
  static_assert(BLOCKS <= S::MAX_BLOCKS && WaveDma<D, 32>::PASSES <= NW, "");
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, ql = lane & 31;
  const int wave_u = __builtin_amdgcn_readfirstlane(tid >> 6);
  item = __builtin_amdgcn_readfirstlane(item);
  const int64_t grid0 = kv_grid_origin(a.kv_begin, a.kv.n, 32);
  const int key_blocks = (int)((a.kv_end - grid0 + 32 * BLOCKS - 1) / (32 * BLOCKS)), per_b = key_blocks * a.n_kv_heads;
  const int b = __builtin_amdgcn_readfirstlane(item / per_b), hb = item - b * per_b;
  const int hk = __builtin_amdgcn_readfirstlane(hb / key_blocks), kblk = hb - hk * key_blocks;
  const int block = wave_u / NW, wave_b = wave_u % NW;   // the wave's key block and its number among the waves of that
  int64_t key0 = grid0 + (int64_t)(kblk * BLOCKS + block) * 32;
  const bool exists = BLOCKS == 1 || key0 < a.kv_end;    // (a last, second block may lie behind the range: its waves copy and store nothing)
  if (!exists) key0 -= 32;
  const int64_t mykey = key0 + ql;
  const int chunk = kv_chunk_of(a.kv, key0);
  const int64_t chunk_row0 = key0 - (int64_t)chunk * a.kv.len, left = a.kv_end - key0;      // (>= 1)
  const int64_t head_off = (int64_t)b * a.kv_stride_b + (int64_t)hk * a.kv_stride_h;
  const float c = a.scale_log2e;

  f32x16 dk[DB], dv[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) { dk[db][i] = 0.f; dv[db][i] = 0.f; }

  const unsigned smem_lds = lds_addr(smem);
  // K and V rows of the workgroup: one copy instruction of each per wave (as far as there are any)
  {
    const bf16_t* kbase = uniform_ptr(a.kv.k[chunk] + head_off + chunk_row0 * a.kv_stride_s);
    if (wave_b < WaveDma<D, 32>::PASSES)
      WaveDma<D, 32>::copy_pass(smem_lds + S::K_BASE + block * TILE_BYTES, kbase, (uint32_t)a.kv_stride_s * 2, left < 32 ? (int)left : 32, lane, wave_b);
    const bf16_t* vbase = uniform_ptr(a.kv.v[chunk] + head_off + chunk_row0 * a.kv_stride_s);
    // (rows that some row sees: dS of the others is P = 0 times dP, and what the cache holds there must not reach dP)
    const int64_t seen = a.seen_end - key0;
    if (wave_b < WaveDma<D, 32>::PASSES && seen > 0)
      WaveDma<D, 32>::copy_pass(smem_lds + S::V_BASE + block * TILE_BYTES, vbase, (uint32_t)a.kv_stride_s * 2, seen < 32 ? (int)seen : 32, lane, wave_b);
  }
  // query tiles that see the block: [qt0, nqt) of every head of the group, tile j of this list for wave j mod NW of the block
  const int nqt = (int)(((int64_t)a.s_q + 31) / 32);
  int qt0 = 0;
  if (a.causal && key0 > a.q_offset) {
    const int64_t first = key0 - a.q_offset;
    qt0 = first >= a.s_q ? nqt : (int)(first / 32);
  }
  const int nv = nqt - qt0, total = exists ? nv * a.group : 0;
  const uint32_t q_bytes = (uint32_t)a.q_stride_s * 2, do_bytes = (uint32_t)a.do_stride_s * 2;
  WaveDma<D, 32> dma_q, dma_do;
  dma_q.init(lane, q_bytes);
  dma_do.init(lane, do_bytes);
  // the delta kernel's two statistics are arrays of one workspace (far below 4 GB): one uniform base and a 32-bit lane offset
  const int64_t stat_gap = a.delta - a.lse2;
  const float* const stat_base = stat_gap < 0 ? a.delta : a.lse2;
  const uint32_t off_lse2 = stat_gap < 0 ? (uint32_t)(-stat_gap) * 4u : 0u, off_delta = stat_gap < 0 ? 0u : (uint32_t)stat_gap * 4u;
  const unsigned set_lds = smem_lds + wave_u * BUF * S::SET_BYTES;
  auto head_of = [&](int j) { return __builtin_amdgcn_readfirstlane(j / nv); };
  auto copy_tile = [&](int j, int buf, bool with_q, bool with_do) {
    const int hh = head_of(j), row0 = (qt0 + j - hh * nv) * 32, h = hk * a.group + hh, rows = a.s_q - row0;
    const unsigned dst = set_lds + buf * S::SET_BYTES;
    if (with_q) {
      if constexpr (!OWN_STATS) {
        // lanes 0..31: lse2 of the rows, lanes 32..63: -delta (clamped to the slice)
        const int rr = ql < rows ? ql : rows - 1;
        dma4(uniform_ptr(stat_base + ((int64_t)b * a.n_q_heads + h) * a.s_q + row0), (g ? off_delta : off_lse2) + (uint32_t)rr * 4u,
             __builtin_amdgcn_readfirstlane(dst + 2 * TILE_BYTES));
      }
      dma_q.copy(dst, uniform_ptr(a.q + (int64_t)b * a.q_stride_b + (int64_t)h * a.q_stride_h + (int64_t)row0 * a.q_stride_s), q_bytes, 0, rows < 32 ? rows : 32, lane);
    }
    if (with_do)
      dma_do.copy(dst + TILE_BYTES, uniform_ptr(a.d_out + (int64_t)b * a.do_stride_b + (int64_t)h * a.do_stride_h + (int64_t)row0 * a.do_stride_s), do_bytes,
                  0, rows < 32 ? rows : 32, lane);
  };
  // For the row statistics of a tile, asked for a step ahead: lse of row ql, and the 16 bytes of O that sit where lane and pass are in the
  // copy of the dO tile (8 or 16 lanes a row; a row a lane would be 64 lines an instruction)
  constexpr int NP = WaveDma<D, 32>::PASSES, NC = WaveDma<D, 32>::NC;
  const uint32_t o_bytes = (uint32_t)a.o_stride_s * 2;
  bf16x8 o_part[NP];
  float lse_row = 0.f;
  auto fetch_rows = [&](int j) {
    const int hh = head_of(j), row0 = (qt0 + j - hh * nv) * 32, h = hk * a.group + hh, rows = a.s_q - row0;
    const char* op = reinterpret_cast<const char*>(uniform_ptr(a.out + (int64_t)b * a.o_stride_b + (int64_t)row0 * a.o_stride_s + (int64_t)h * a.o_stride_h));
#pragma unroll
    for (int n = 0; n < NP; ++n) o_part[n] = *reinterpret_cast<const bf16x8*>(op + WaveDma<D, 32>::pass_off(lane, n, o_bytes, rows));
    lse_row = a.lse[((int64_t)b * a.n_q_heads + h) * a.s_q + row0 + (ql < rows ? ql : rows - 1)];
  };
  int j = wave_b;
  if (j < total) {
    copy_tile(j, 0, true, true);
    if constexpr (OWN_STATS) fetch_rows(j);
  }
  wait_async();
  __syncthreads();                                       // K and V have landed
  bf16x8 k[KS];
  {
    RpBase<D> lo_k;
    lo_k.init(lane, (int)smem_lds + S::K_BASE + block * TILE_BYTES);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) k[ks] = lds_rp<D>(lo_k, ks, 0);
  }
  RpBase<D> lo_q, lo_v;
  TrBase<D> lo_qt;
  lo_q.init(lane, (int)set_lds);
  lo_qt.init(lane, (int)set_lds);
  lo_v.init(lane, (int)smem_lds + S::V_BASE + block * TILE_BYTES);
  int buf = 0;
  for (; j < total; j += NW) {
    const int jn = j + NW;
    const int hh = head_of(j), row0 = (qt0 + j - hh * nv) * 32;
    const int o = buf * S::SET_BYTES;
    RpBase<D> lq = lo_q;
    TrBase<D> lqt = lo_qt;
    lq.add(o);
    lqt.add(o);
    // statistics of the tile's rows: lse in log2 units, then -dO . O; through LDS to where the scores need them
    float* const stats = reinterpret_cast<float*>(smem + (set_lds - smem_lds) + o + 2 * TILE_BYTES);
    if constexpr (OWN_STATS) {
      const char* dO = smem + (set_lds - smem_lds) + o + TILE_BYTES + lane * 16;
      if (g == 0) stats[ql] = lse_log2(lse_row);
#pragma unroll
      for (int n = 0; n < NP; ++n) {
        const float d = row_sum<NC>(dot8(*reinterpret_cast<const bf16x8*>(dO + n * 1024), o_part[n], 0.f));
        if (lane % NC == 0) stats[32 + lane / NC + 64 / NC * n] = -d;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    const float* stat = stats + 4 * g;
    if constexpr (BUF == 2) {
      if (jn < total) {
        copy_tile(jn, buf ^ 1, true, true);
        if constexpr (OWN_STATS) fetch_rows(jn);
      }
      SP_FENCE();
    }
    f32x16 s, dp;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const f32x16 zero = {0};
      s = mfma32(lds_rp<D>(lq, ks, 0), k[ks], ks == 0 ? zero : s);
    }
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const f32x4 nd = *reinterpret_cast<const f32x4*>(stat + 32 + 8 * i4);
#pragma unroll
      for (int e = 0; e < 4; ++e) dp[4 * i4 + e] = nd[e];
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) dp = mfma32(lds_rp<D>(lq, ks, TILE_BYTES), lds_rp<D>(lo_v, ks, 0), dp);
    if ((a.causal && a.q_offset + row0 < key0 + 31) || row0 + 32 > a.s_q) {
      const int64_t rl = a.causal ? mykey - a.q_offset - row0 : 0;      // first row of the tile that sees this lane's key
      const int lo = (rl < 0 ? 0 : (rl > 32 ? 32 : (int)rl)) - 4 * g, hi = (a.s_q - row0 > 32 ? 32 : a.s_q - row0) - 4 * g;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int r = 8 * (i >> 2) + (i & 3);
        s[i] = ((r >= lo) & (r < hi)) ? s[i] : -INFINITY;      // exp2(-inf) = 0
      }
    }
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const f32x4 l2 = *reinterpret_cast<const f32x4*>(stat + 8 * i4);
#pragma unroll
      for (int e = 0; e < 4; ++e) s[4 * i4 + e] = __builtin_fmaf(s[4 * i4 + e], c, -l2[e]);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = exp2_fast(s[i]);
#pragma unroll
    for (int i = 0; i < 16; ++i) dp[i] *= s[i];
    const bf16x8 pb[2] = {pack8(s, 0), pack8(s, 8)}, dsb[2] = {pack8(dp, 0), pack8(dp, 8)};
    // dK first: with one buffer, Q of the next tile is copied while dV is computed
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int db = 0; db < DB; ++db) dk[db] = mfma32(lds_tr<D>(lqt, db, hf * 16 * D * 2), dsb[hf], dk[db]);
#pragma unroll
    for (int db = 0; db < DB; ++db) asm volatile("" : "+v"(dk[db]));      // the reads of Q are done before Q is copied over
    if constexpr (BUF == 1) {
      if (jn < total) copy_tile(jn, 0, true, false);
    }
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int db = 0; db < DB; ++db) dv[db] = mfma32(lds_tr<D>(lqt, db, TILE_BYTES + hf * 16 * D * 2), pb[hf], dv[db]);
#pragma unroll
    for (int db = 0; db < DB; ++db) asm volatile("" : "+v"(dv[db]));
    if constexpr (BUF == 1) {
      if (jn < total) copy_tile(jn, 0, false, true);
    }
    SP_FENCE();
    wait_async();
    asm volatile("" ::: "memory");
    SP_FENCE();
    if constexpr (BUF == 2) buf ^= 1;
  }
  wait_async();
  // the waves' sums meet in LDS and are added up in wave order, 16 / BLOCKS threads a row; what the accumulators hold is asked for before
  constexpr int PER = D * BLOCKS / 16, N4 = PER / 4;     // head_dim elements of a thread
  const int tb = tid & (NW * 64 - 1), r = tb / (16 / BLOCKS), d0 = tb % (16 / BLOCKS) * PER;
  const int64_t key = key0 + r;
  const bool mine = exists && key >= a.kv_begin && key < a.kv_end;
  const int64_t dst_off = head_off + (chunk_row0 + r) * a.kv_stride_s + d0;
  f32x4 old[2][N4];
  if (a.dkv_accumulate && mine) {
#pragma unroll
    for (int grad = 0; grad < 2; ++grad)
#pragma unroll
      for (int j4 = 0; j4 < N4; ++j4) old[grad][j4] = *reinterpret_cast<const f32x4*>((grad ? a.dv_acc[chunk] : a.dk_acc[chunk]) + dst_off + 4 * j4);
  }
  constexpr int GRADS = S::GRADS, PLANE = S::NW * S::PART_BYTES;
#pragma unroll
  for (int g0 = 0; g0 < 2; g0 += GRADS) {
    __syncthreads();                                     // nobody reads what is there any more
#pragma unroll
    for (int grad = g0; grad < g0 + GRADS; ++grad)
      put_part<D>(smem + (grad - g0) * PLANE + wave_u * S::PART_BYTES, grad ? dv : dk, grad ? 1.0f : a.scale, ql, g);
    __syncthreads();
    if (mine) {
#pragma unroll
      for (int grad = g0; grad < g0 + GRADS; ++grad) {
        f32x4 sum[N4];
        sum_parts<D, NW>(smem + (grad - g0) * PLANE + block * NW * S::PART_BYTES, r, d0, sum);
        float* dst = (grad ? a.dv_acc[chunk] : a.dk_acc[chunk]) + dst_off;
#pragma unroll
        for (int j4 = 0; j4 < N4; ++j4) {
          if (a.dkv_accumulate) sum[j4] += old[grad][j4];
          *reinterpret_cast<f32x4*>(dst + 4 * j4) = sum[j4];
        }
      }
    }
  }
}

// dq and dk/dv items, the kind that takes longer first.
template <int D, bool OWN_STATS, int BLOCKS>
__global__ __launch_bounds__(512) void attn_bwd_small_kernel(const BwdArgs a, int n_dq, int n_dkdv) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int i = blockIdx.x, first = a.dq_first ? n_dq : n_dkdv;
  if ((i < first) == (a.dq_first != 0)) dq_small_item<D, OWN_STATS>(a, a.dq_first ? i : i - n_dkdv, smem);
  else dkdv_small_item<D, OWN_STATS, BLOCKS>(a, a.dq_first ? i - n_dq : i, smem);
}

template <int D, bool OWN_STATS, int BLOCKS>
static hipError_t launch_bwd_small_t(const BwdArgs& a, int batch, hipStream_t st) {
  const int64_t n_dq = ((int64_t)a.s_q + 31) / 32 * a.n_q_heads * batch;
  const int64_t n_dkdv = (a.kv_end - kv_grid_origin(a.kv_begin, a.kv.n, 32) + 32 * BLOCKS - 1) / (32 * BLOCKS) * a.n_kv_heads * batch;
  hipLaunchKernelGGL((attn_bwd_small_kernel<D, OWN_STATS, BLOCKS>), dim3((unsigned)(n_dq + n_dkdv)), dim3(512), BwdSmall<D>::LDS, st, a, (int)n_dq, (int)n_dkdv);
  return hipGetLastError();
}
hipError_t launch_bwd_small(const BwdArgs& a, int batch, int head_dim, bool own_stats, int key_blocks, hipStream_t st) {
  if (head_dim == 128) return launch_bwd_small_t<128, false, 1>(a, batch, st);
  if (key_blocks == 2) return own_stats ? launch_bwd_small_t<64, true, 2>(a, batch, st) : launch_bwd_small_t<64, false, 2>(a, batch, st);
  return own_stats ? launch_bwd_small_t<64, true, 1>(a, batch, st) : launch_bwd_small_t<64, false, 1>(a, batch, st);
}

int small_dq_tile_keys(int head_dim) { return head_dim == 128 ? BwdSmall<128>::BN : BwdSmall<64>::BN; }

hipError_t opt_in_small_kernels() {
  const hipFuncAttribute attr = hipFuncAttributeMaxDynamicSharedMemorySize;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_fwd_small_kernel<128>), attr, FwdSmall<128>::LDS);
  if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_fwd_small_kernel<64>), attr, FwdSmall<64>::LDS);
  if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_bwd_small_kernel<128, false, 1>), attr, BwdSmall<128>::LDS);
  if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_bwd_small_kernel<64, true, 1>), attr, BwdSmall<64>::LDS);
  if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_bwd_small_kernel<64, false, 1>), attr, BwdSmall<64>::LDS);
  if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_bwd_small_kernel<64, true, 2>), attr, BwdSmall<64>::LDS);
  if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_bwd_small_kernel<64, false, 2>), attr, BwdSmall<64>::LDS);
  return e;
}

}  // namespace slimpipe
