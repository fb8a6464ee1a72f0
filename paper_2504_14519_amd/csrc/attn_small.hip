// Forward of small calls: a workgroup owns 32 query rows of one head and its 8 wavefronts share out their keys.
//
// What bounds a small call is a chain: a 256-row block walks its keys tile after tile behind barriers on a chip that is mostly idle, and
// key ranges shorten the chain only at the price of a merge launch.  Here eight waves walk eight tiles of the keys at the same time,
// each with a K and a V tile of its own in LDS, copied by itself and waited for by itself (no barrier in the loop), and their
// partial results meet in LDS.  512 rows on 2048 keys, 4 heads of 64 (64 workgroups): 18.1 -> 11.9 us; 512 rows of 8 heads of 128 on one
// K/V head, 2048 keys: 34.6 -> 19.1; 1024 rows: 35.5 -> 19.8.  A wave's step (32 keys, 64 at head_dim 64) takes 1.3 us, most of it
// latency of the copies: one K and one V tile per wave are all of LDS, so K of the next step is copied during softmax and P V, V
// during the scores and the softmax.  Which calls come here: fwd_plan in api.hip.
#include "kernels.hpp"
#include "tile_common.hpp"

namespace slimpipe {

// A wave's own tile copy (64 lanes, 1 KB an instruction): 64 / (D / 8) rows per pass.  The lane's offset inside the rows of a pass
// is the same in every pass but for the swizzle (head_dim 128: bits 0..1 of the chunk alternate with the pass), so a full tile
// costs scalar additions only; in a tile with fewer rows they are clamped to those that exist.
template <int D, int ROWS>
struct WaveDma {
  static constexpr int NC = D / 8, RPP = 64 / NC, PASSES = ROWS / RPP, PHASES = D == 128 ? 4 : 1;
  uint32_t off[PHASES];
  SP_DEV void init(int lane, uint32_t row_bytes) {
    const int r = lane / NC, p = lane % NC;
    const int c = D == 128 ? (((p >> 2) ^ r) & 3) << 2 | (p & 3) : (p ^ r) & (NC - 1);
#pragma unroll
    for (int n = 0; n < PHASES; ++n) off[n] = __umul24((uint32_t)r, row_bytes) + (uint32_t)((c ^ n) * 16);
  }
  SP_DEV void copy(unsigned lds_tile, const bf16_t* tile_base, uint32_t row_bytes, int rows_avail, int lane) const {
    lds_tile = __builtin_amdgcn_readfirstlane(lds_tile);
    if (rows_avail >= ROWS) {
      const char* base = reinterpret_cast<const char*>(tile_base);
#pragma unroll
      for (int n = 0; n < PASSES; ++n, base += (uint64_t)RPP * row_bytes) dma16(base, off[n % PHASES], lds_tile + n * 1024);
    } else {
      const int r0 = lane / NC;
#pragma unroll
      for (int n = 0; n < PASSES; ++n) {
        const int r = r0 + RPP * n, rr = r < rows_avail ? r : rows_avail - 1;
        dma16(tile_base, off[n % PHASES] + __umul24((uint32_t)rr, row_bytes) - __umul24((uint32_t)r0, row_bytes), lds_tile + n * 1024);
      }
    }
  }
};

template <int D>
struct FwdSmall {
  static constexpr int NW = 8, BN = D == 64 ? 64 : 32, KB = BN / 32, KS = D / 16, DB = D / 32;
  static constexpr int TILE_BYTES = BN * D * 2, WAVE_BYTES = 2 * TILE_BYTES;
  static constexpr int ROW = D + 4;                      // floats per row of a wave's partial output (padded against bank conflicts)
  static constexpr int PART_BYTES = 32 * ROW * 4, STAT_BASE = NW * PART_BYTES, COMBINE_BYTES = STAT_BASE + NW * 64 * 4;
  static constexpr int LDS = NW * WAVE_BYTES > COMBINE_BYTES ? NW * WAVE_BYTES : COMBINE_BYTES;
};

template <int D>
__global__ __launch_bounds__(512) void attn_fwd_small_kernel(const FwdArgs a) {
  using F = FwdSmall<D>;
  constexpr int NW = F::NW, BN = F::BN, KB = F::KB, KS = F::KS, DB = F::DB;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, ql = lane & 31;
  const int wave_u = __builtin_amdgcn_readfirstlane(tid >> 6);
  // block index -> (query head, 32-row block of a head, batch index x range), row blocks with the longest key ranges first
  const int row_blocks = a.items[0], per_z = row_blocks * a.n_q_heads;
  const int bz = __builtin_amdgcn_readfirstlane((int)(blockIdx.x / (unsigned)per_z)), hb = blockIdx.x - bz * per_z;
  const int b = __builtin_amdgcn_readfirstlane(bz / a.n_ranges), range = bz - b * a.n_ranges;
  const int rb = __builtin_amdgcn_readfirstlane(hb / a.n_q_heads), h = hb - rb * a.n_q_heads;
  const int row0 = (row_blocks - 1 - rb) * 32, hk = h / a.group;
  const int myrow = row0 + ql, myrow_c = myrow < a.s_q ? myrow : a.s_q - 1;
  const int64_t kv_begin = a.range_begin[range], kv_end = a.range_end[range];
  int64_t hi = kv_end;
  if (a.causal) {
    const int64_t lim = a.q_offset + (row0 + 32 < a.s_q ? row0 + 32 : a.s_q);
    hi = hi < lim ? hi : lim;
  }
  const int64_t lo = kv_grid_origin(kv_begin, a.kv.n, BN);
  const int nt = hi > lo ? (int)((hi - lo + BN - 1) / BN) : 0;
  const float c = a.scale_log2e;

  bf16x8 q[KS];
  {
    const bf16_t* qp = a.q + (int64_t)b * a.q_stride_b + (int64_t)myrow_c * a.q_stride_s + (int64_t)h * a.q_stride_h;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) q[ks] = *reinterpret_cast<const bf16x8*>(qp + 16 * ks + 8 * g);
  }
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
  auto copy = [&](bool k, int t) {
    const int64_t key0 = lo + (int64_t)t * BN;
    const int chunk = kv_chunk_of(a.kv, key0);
    const int64_t row = key0 - (int64_t)chunk * a.kv.len, left = a.kv.len - row;
    const bf16_t* base = uniform_ptr((k ? a.kv.k[chunk] : a.kv.v[chunk]) + head_off + row * a.kv_stride_s);
    dma.copy(k ? k_lds : v_lds, base, row_bytes, left < BN ? (int)left : BN, lane);
  };
  constexpr int PASSES = WaveDma<D, BN>::PASSES;
  int t = wave_u;                                        // tiles w, w + 8, w + 16, .. are this wave's
  if (t < nt) {
    copy(true, t);
    copy(false, t);
  }
  for (; t < nt; t += NW) {
    const int tn = t + NW < nt ? t + NW : t;             // (past the end the last tile is copied again)
    // K has landed (the copies of V may still be under way)
    SP_FENCE();
    __builtin_amdgcn_s_waitcnt(0x0F70 | PASSES);
    asm volatile("" ::: "memory");
    SP_FENCE();
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
    copy(true, tn);
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
    SP_FENCE();
    __builtin_amdgcn_s_waitcnt(0x0F70 | PASSES);
    asm volatile("" ::: "memory");
    SP_FENCE();
#pragma unroll
    for (int blk = 0; blk < 2 * KB; ++blk)
#pragma unroll
      for (int db = 0; db < DB; ++db) o[db] = mfma32(lds_tr<D>(lo_v, db, blk * 16 * D * 2), p[blk / 2][blk % 2], o[db]);
#pragma unroll
    for (int db = 0; db < DB; ++db) asm volatile("" : "+v"(o[db]));      // the reads of V are done before V is copied over
    copy(false, tn);
  }
  wait_async();
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
  const dim3 grid((unsigned)((int64_t)a.items[0] * a.n_q_heads * batch * a.n_ranges)), block(512);
  if (head_dim == 128) hipLaunchKernelGGL(attn_fwd_small_kernel<128>, grid, block, FwdSmall<128>::LDS, st, a);
  else hipLaunchKernelGGL(attn_fwd_small_kernel<64>, grid, block, FwdSmall<64>::LDS, st, a);
  return hipGetLastError();
}

hipError_t opt_in_small_kernels() {
  const hipFuncAttribute attr = hipFuncAttributeMaxDynamicSharedMemorySize;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_fwd_small_kernel<128>), attr, FwdSmall<128>::LDS);
  if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_fwd_small_kernel<64>), attr, FwdSmall<64>::LDS);
  return e;
}

}  // namespace slimpipe
