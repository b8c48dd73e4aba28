// MFMA attention for grids that leave CUs idle (the rule and both sides' times: attn_mfma_plan): the same products, types and roundings as
// attn_mfma.hip and attn_mfma_dq.hip, but a workgroup owns 32 rows and its wavefronts take the 32-row blocks of the other side in turn,
// without a barrier in the walk; their sums meet in LDS and are added in wavefront order.  With few rows and heads the time of
// the other kernels is one wavefront's serial walk over the whole other side behind a barrier per step (2 us per 64 keys in the
// forward, 3 per 64 queries of every head of a group in dK/dV) on a handful of CUs.  What bounds these: the latency of launch, first loads, one to a few
// blocks (about 1 us each) and the exchange; with more rows the blocks, read by every workgroup of the head, through the L2.
// Blocks come straight from memory: a lane loads the 16-byte chunks of one row, which are at once the row fragments of the products over the
// head dimension and, put to a wavefront-private LDS tile, the source of the transposed fragments of the others.
// dS goes through the scratch of attn_mfma.hip in its layout, every block of the pairs the dQ kernel reads written in full.
#include "attn_mfma_common.h"

namespace rrfp {
namespace {

template <int D>
struct SplitCfg {
  static constexpr int DP = (D + 31) / 32 * 32, NDS = D / 16, NDB = DP / 32;
  static constexpr int NW = D == 128 ? 4 : 8;           // wavefronts: what the LDS of two workgroups (D 128) or one and a half holds
  static constexpr int PITCH = DP * 2 + 32;             // bytes per row of a staged block: the value tile's pitch of attn_mfma.hip
  static constexpr int TILE = 32 * PITCH;
  static constexpr int SUM_PITCH = DP + 4;              // floats per row of a wavefront's sums
  static constexpr int SUMS = 32 * SUM_PITCH * 4;
  static constexpr int area(int bytes) { return bytes > SUMS ? bytes : SUMS; }
};

// The rows of a block of 32 at row0 (at or past row_end: the last one again): lane gets chunks 2 ds + h of row li.
template <int D>
__device__ __forceinline__ void rows_load(uint4 (&r)[D / 16], const el_t* __restrict__ p, int ld, int row0, int row_end, int lane) {
  const el_t* row = p + (size_t)min(row0 + (lane & 31), row_end - 1) * ld + (lane >> 5) * 8;
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int ds = 0; ds < D / 16; ++ds) r[ds] = __builtin_bit_cast(uint4, *reinterpret_cast<const u32x4*>(row + ds * 16));
}
template <int D>
__device__ __forceinline__ void rows_put(const uint4 (&r)[D / 16], char* tile, int lane) {
#pragma unroll
  for (int ds = 0; ds < D / 16; ++ds) *reinterpret_cast<uint4*>(tile + (lane & 31) * SplitCfg<D>::PITCH + (ds * 2 + (lane >> 5)) * 16) = r[ds];
}
// Columns D .. DP - 1 of a tile: zero, for good.
template <int D>
__device__ __forceinline__ void pad_zero(char* tile, int lane) {
  if constexpr (SplitCfg<D>::DP != D) {
    static_assert(SplitCfg<D>::DP - D == 16, "two chunks of padding");
    *reinterpret_cast<uint4*>(tile + (lane & 31) * SplitCfg<D>::PITCH + (D / 8 + (lane >> 5)) * 16) = make_uint4(0, 0, 0, 0);
  }
}
// Transposed sums (rows = head dimension, columns = this workgroup's rows) of this wavefront to its area.
template <int D>
__device__ __forceinline__ void sums_put(float* area, const floatx16 (&acc)[SplitCfg<D>::NDB], int lane) {
  wave_lds_sync();
#pragma unroll
  for (int db = 0; db < SplitCfg<D>::NDB; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<float4*>(area + (lane & 31) * SplitCfg<D>::SUM_PITCH + db * 32 + g * 8 + (lane >> 5) * 4) =
          make_float4(acc[db][g * 4], acc[db][g * 4 + 1], acc[db][g * 4 + 2], acc[db][g * 4 + 3]);
}
// Four values of a row, added over the wavefronts in order, each times its factor (null: 1).
template <int D, int AREA>
__device__ __forceinline__ float4 sums_get(const char* smem, int row, int c, const float* factor) {
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int w = 0; w < SplitCfg<D>::NW; ++w) {
    const float4 x = *reinterpret_cast<const float4*>(smem + w * AREA + (row * SplitCfg<D>::SUM_PITCH + c) * 4);
    const float f = factor ? factor[w * 32 + row] : 1.0f;
    v.x += x.x * f; v.y += x.y * f; v.z += x.z * f; v.w += x.w * f;
  }
  return v;
}
__device__ __forceinline__ uint2 pack_bf16x4(float4 v) { return make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w)); }

// Sub-tile of 32 rows; per_tile of them are launched for each tile: as many as the longest segment has (r0 >= r1: nothing to do).  The last
// rows of a tile first (under a causal mask they have the longest walk), from another start in every tile: with few heads a
// sub-tile's place in its tile would decide its XCD, and segments that end early would leave some of them without work.
__device__ __forceinline__ AttnTile split_tile(const AttnTile* __restrict__ tiles, int i, int per_tile) {
  const int tile = i / per_tile;
  AttnTile t = tiles[tile];
  t.r0 += (per_tile - 1 - i % per_tile + tile) % per_tile * 32;
  t.r1 = min(t.r1, t.r0 + 32);
  return t;
}
int split_per_tile(const AttnArgs& a, int tile_rows) { return (std::min(a.longest, tile_rows) + 31) / 32; }

template <int D>
__global__ __launch_bounds__(64 * SplitCfg<D>::NW, 2) void attn_fwd_split_kernel(const el_t* __restrict__ qkv, bf16_t* __restrict__ o,
                                                                             float* __restrict__ o32, el_t* __restrict__ o16,
                                                                             float* __restrict__ lse, const AttnTile* __restrict__ tiles, int per_tile, int Tn,
                                                                             int nq, int nkv, int causal, float scale_log2e) {
  using C = SplitCfg<D>;
  constexpr int NDS = C::NDS, NDB = C::NDB, NW = C::NW, AREA = C::area(C::TILE);
  extern __shared__ __attribute__((aligned(16))) char smem[];
  float* const ms = reinterpret_cast<float*>(smem + NW * AREA);
  float* const ls = ms + NW * 32;
  const int a = blockIdx.x % nq, b = a / (nq / nkv);
  const AttnTile tl = split_tile(tiles, blockIdx.x / nq, per_tile);
  if (tl.r0 >= tl.r1) return;
  const int ld = (nq + 2 * nkv) * D;
  const el_t *kp = qkv + (nq + b) * D, *vp = qkv + (nq + nkv + b) * D;
  const int lane = threadIdx.x & 63, h = lane >> 5, li = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  char* const tile = smem + wave * AREA;
  const int i = tl.r0 + li;                             // this lane's query
  uint4 qr[NDS], kr[NDS], vr[NDS];
  rows_load<D>(qr, qkv + a * D, ld, tl.r0, tl.r1, lane);
  floatx16 acc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[db][e] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const int kv_end = causal ? tl.r1 : tl.s1;
  int k0 = tl.s0 + wave * 32;
  if (k0 < kv_end) {
    rows_load<D>(kr, kp, ld, k0, kv_end, lane);
    rows_load<D>(vr, vp, ld, k0, kv_end, lane);
  }
  pad_zero<D>(tile, lane);
  for (; k0 < kv_end; k0 += 32 * NW) {
    wave_lds_sync();                                    // the reads of the block before precede these writes
    rows_put<D>(vr, tile, lane);
    floatx16 s;                                         // S^T: rows = keys, columns = queries
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
    for (int ds = 0; ds < NDS; ++ds) s = mfma16(__builtin_bit_cast(frag_t, kr[ds]), __builtin_bit_cast(frag_t, qr[ds]), s);
    if (k0 + 32 * NW < kv_end) {
      rows_load<D>(kr, kp, ld, k0 + 32 * NW, kv_end, lane);
      rows_load<D>(vr, vp, ld, k0 + 32 * NW, kv_end, lane);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int j = k0 + (e >> 2) * 8 + h * 4 + (e & 3);
      if (j >= kv_end || (causal && j > i)) s[e] = -INFINITY;
      mx = fmaxf(mx, s[e]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m_run, mx * scale_log2e);   // finite: the first key of a block is no later than any of the queries
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
    m_run = m_new;
    l_run *= alpha;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[db][e] *= alpha;
    float p[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      p[e] = __builtin_amdgcn_exp2f(fmaf(s[e], scale_log2e, -m_run));
      l_run += p[e];
    }
    wave_lds_sync();                                    // the value rows are in place
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const frag_t pf = pack8(p + u * 8);
#pragma unroll
      for (int db = 0; db < NDB; ++db) acc[db] = mfma16(frag_cols_tr(tile, C::PITCH, u * 16, db * 32, lane), pf, acc[db]);
    }
  }
  l_run += __shfl_xor(l_run, 32, 64);                   // the halves of the wavefront hold disjoint keys of a query
  sums_put<D>(reinterpret_cast<float*>(tile), acc, lane);
  if (h == 0) {
    ms[wave * 32 + li] = m_run;
    ls[wave * 32 + li] = l_run;
  }
  __syncthreads();
  if (threadIdx.x < 32) {                               // factors that bring the wavefronts to one reference point, over the row's sum
    const int row = threadIdx.x;
    float m = ms[row];
#pragma unroll
    for (int w = 1; w < NW; ++w) m = fmaxf(m, ms[w * 32 + row]);
    float f[NW], l = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      f[w] = __builtin_amdgcn_exp2f(ms[w * 32 + row] - m);     // a wavefront without keys: 0
      l += ls[w * 32 + row] * f[w];
    }
    const float inv = 1.0f / l;
#pragma unroll
    for (int w = 0; w < NW; ++w) ms[w * 32 + row] = f[w] * inv;
    if (tl.r0 + row < tl.r1) lse[(size_t)a * Tn + tl.r0 + row] = (m + log2f(l)) * 0.69314718055994531f;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < 32 * D / 4; q += 64 * NW) {
    const int row = q / (D / 4), c = (q - row * (D / 4)) * 4;
    if (tl.r0 + row >= tl.r1) continue;
    const float4 v = sums_get<D, AREA>(smem, row, c, ms);
    const size_t off = (size_t)(tl.r0 + row) * nq * D + a * D + c;
    *reinterpret_cast<uint2*>(o + off) = pack_bf16x4(v);
    if (o32) *reinterpret_cast<float4*>(o32 + off) = v;
    if (o16) *reinterpret_cast<uint2*>(o16 + off) = make_uint2(pack_f16x2(v.x, v.y), pack_f16x2(v.z, v.w));
  }
}

// A workgroup owns 32 keys of a KV head; its wavefronts take the (query head of the subset, 32-query block) pairs in turn.
template <int D>
__global__ __launch_bounds__(64 * SplitCfg<D>::NW) void attn_dkv_split_kernel(const el_t* __restrict__ qkv, const el_t* __restrict__ d_o,
                                                                             const float* __restrict__ lse, const float* __restrict__ delta,
                                                                             bf16_t* __restrict__ dqkv, const AttnTile* __restrict__ tiles, int per_tile, int Tn,
                                                                             int nq, int nkv, int causal, float scale,
                                                                             const float* __restrict__ grad_scale, el_t* __restrict__ ds,
                                                                             int ds_rows, int ds_nqs, int n_sub, float* __restrict__ part) {
  using C = SplitCfg<D>;
  constexpr int NDS = C::NDS, NDB = C::NDB, NW = C::NW, AREA = C::area(2 * C::TILE + 256);
  constexpr float LOG2E = 1.4426950408889634f;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int heads = nkv * n_sub, b = blockIdx.x % heads / n_sub, sub = blockIdx.x % heads % n_sub;
  const int G = nq / nkv / n_sub, a0 = b * (nq / nkv) + sub * G;
  const AttnTile tl = split_tile(tiles, blockIdx.x / heads, per_tile);
  if (tl.r0 >= tl.r1) return;
  const int ld = (nq + 2 * nkv) * D;
  const int lane = threadIdx.x & 63, h = lane >> 5, li = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  char* const tq = smem + wave * AREA;                  // Q rows, dO rows, row statistics of the block
  char* const td = tq + C::TILE;
  float* const stat = reinterpret_cast<float*>(td + C::TILE);
  const int j = tl.r0 + li;                             // this lane's key
  const float scale_log2e = scale * LOG2E;
  const int ds_krow = tl.kb0 + ((tl.r0 - tl.s0) >> 5);
  uint4 kr[NDS], vr[NDS], qr[NDS], dr[NDS];
  rows_load<D>(kr, qkv + (nq + b) * D, ld, tl.r0, tl.r1, lane);
  rows_load<D>(vr, qkv + (nq + nkv + b) * D, ld, tl.r0, tl.r1, lane);
  floatx16 dk[NDB], dv[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) { dk[db][e] = 0.f; dv[db][e] = 0.f; }
  const int qb0 = causal ? (tl.r0 - tl.s0) >> 5 : 0, per = ((tl.s1 - tl.s0 + 31) >> 5) - qb0, pairs = G * per;
  float r_stat = 0.f;
  auto fetch = [&](int p) {
    const int a = a0 + p / per, q0 = tl.s0 + (qb0 + p % per) * 32;
    rows_load<D>(qr, qkv + a * D, ld, q0, tl.s1, lane);
    rows_load<D>(dr, d_o + a * D, nq * D, q0, tl.s1, lane);
    r_stat = (h ? delta : lse)[(size_t)a * Tn + min(q0 + li, tl.s1 - 1)];
  };
  int p = wave;
  if (p < pairs) fetch(p);
  pad_zero<D>(tq, lane);
  pad_zero<D>(td, lane);
  for (; p < pairs; p += NW) {
    const int a = a0 + p / per, qb = qb0 + p % per, q0 = tl.s0 + qb * 32;
    wave_lds_sync();                                    // the reads of the block before precede these writes
    rows_put<D>(qr, tq, lane);
    rows_put<D>(dr, td, lane);
    stat[lane] = h ? r_stat : r_stat * LOG2E;
    floatx16 s, dp;                                     // rows = queries, columns = keys
#pragma unroll
    for (int e = 0; e < 16; ++e) { s[e] = 0.f; dp[e] = 0.f; }
#pragma unroll
    for (int i = 0; i < NDS; ++i) {
      s = mfma16(__builtin_bit_cast(frag_t, qr[i]), __builtin_bit_cast(frag_t, kr[i]), s);
      dp = mfma16(__builtin_bit_cast(frag_t, dr[i]), __builtin_bit_cast(frag_t, vr[i]), dp);
    }
    if (p + NW < pairs) fetch(p + NW);
    wave_lds_sync();                                    // the rows and statistics are in place
    el_t* ds_block = ds + (((size_t)a * ds_rows + ds_krow) * ds_nqs + (qb >> 1)) * 2048 + (qb & 1) * 1024 + lane * 8;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      float pv[8], dsv[8];
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const int row = (u * 2 + g) * 8 + h * 4;        // of the four accumulator values from e = 8 u + 4 g
        const float4 l4 = *reinterpret_cast<const float4*>(stat + row), d4 = *reinterpret_cast<const float4*>(stat + 32 + row);
        const float lv[4] = {l4.x, l4.y, l4.z, l4.w}, dl[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int e = u * 8 + g * 4 + c, i = q0 + row + c;
          float x = __builtin_amdgcn_exp2f(fmaf(s[e], scale_log2e, -lv[c]));
          if (i >= tl.s1 || j >= tl.r1 || (causal && j > i)) x = 0.f;
          pv[g * 4 + c] = x;
          dsv[g * 4 + c] = x * (dp[e] - dl[c]);         // masked entries: P = 0 and dP finite, so dS = 0
        }
      }
      const frag_t pf = pack8(pv), dsf = pack8(dsv);
      *reinterpret_cast<uint4*>(ds_block + u * 512) = __builtin_bit_cast(uint4, dsf);
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        dv[db] = mfma16(frag_cols_tr(td, C::PITCH, u * 16, db * 32, lane), pf, dv[db]);
        dk[db] = mfma16(frag_cols_tr(tq, C::PITCH, u * 16, db * 32, lane), dsf, dk[db]);
      }
    }
  }
  const float inv_s = grad_scale ? grad_scale[1] : 1.0f;     // d_o held s * dO: undo it (a power of two: exact)
#pragma unroll
  for (int tensor = 0; tensor < 2; ++tensor) {
    if (tensor) __syncthreads();
    sums_put<D>(reinterpret_cast<float*>(tq), tensor ? dv : dk, lane);
    __syncthreads();
    const float mul = tensor ? inv_s : scale * inv_s;
    for (int q = threadIdx.x; q < 32 * D / 4; q += 64 * NW) {
      const int row = q / (D / 4), c = (q - row * (D / 4)) * 4, jr = tl.r0 + row;
      if (jr >= tl.r1) continue;
      const float4 v = sums_get<D, AREA>(smem, row, c, nullptr);
      if (n_sub > 1) *reinterpret_cast<float4*>(part + ((size_t)(tensor * n_sub + sub) * Tn + jr) * (nkv * D) + b * D + c) = v;
      else *reinterpret_cast<uint2*>(dqkv + (size_t)jr * ld + (nq + tensor * nkv + b) * D + c) =
               pack_bf16x4(make_float4(v.x * mul, v.y * mul, v.z * mul, v.w * mul));
    }
  }
}

template <int D>
__global__ __launch_bounds__(64 * SplitCfg<D>::NW) void attn_dq_split_kernel(const el_t* __restrict__ qkv, const el_t* __restrict__ ds,
                                                                            bf16_t* __restrict__ dqkv, const AttnTile* __restrict__ tiles, int per_tile, int nq,
                                                                            int nkv, int causal, float scale, const float* __restrict__ grad_scale,
                                                                            int ds_rows, int ds_nqs) {
  using C = SplitCfg<D>;
  // dS of the 32 queries and 32 keys of a block, as the dQ kernel of attn_mfma_dq.hip lays it out
  constexpr int DS_HALF = 512 + 64, DS_PAIR = 2 * DS_HALF;
  constexpr int NDS = C::NDS, NDB = C::NDB, NW = C::NW, AREA = C::area(C::TILE + 2 * DS_PAIR);
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int a = blockIdx.x % nq, b = a / (nq / nkv);
  const AttnTile tl = split_tile(tiles, blockIdx.x / nq, per_tile);
  if (tl.r0 >= tl.r1) return;
  const int ld = (nq + 2 * nkv) * D;
  const el_t* kp = qkv + (nq + b) * D;
  const int lane = threadIdx.x & 63, h = lane >> 5, li = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  char* const tile = smem + wave * AREA;
  char* const dsw = tile + C::TILE;
  const int qb = (tl.r0 - tl.s0) >> 5, nblk = causal ? qb + 1 : (tl.s1 - tl.s0 + 31) >> 5;
  const el_t* ds0 = ds + (((size_t)a * ds_rows + tl.kb0) * ds_nqs + (qb >> 1)) * 2048 + (qb & 1) * 1024 + lane * 8;
  const size_t ds_step = (size_t)ds_nqs * 2048;
  floatx16 acc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[db][e] = 0.f;
  uint4 kr[NDS], dr0, dr1;
  auto fetch = [&](int kb) {
    rows_load<D>(kr, kp, ld, tl.s0 + kb * 32, tl.s1, lane);
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    dr0 = __builtin_bit_cast(uint4, *reinterpret_cast<const u32x4*>(ds0 + kb * ds_step));
    dr1 = __builtin_bit_cast(uint4, *reinterpret_cast<const u32x4*>(ds0 + kb * ds_step + 512));
  };
  int kb = wave;
  if (kb < nblk) fetch(kb);
  pad_zero<D>(tile, lane);
  // lane roles of the transposed read of dS: see attn_mfma_dq.hip
  const int tr_krow = h * 4 + ((lane & 15) >> 2), tr_qg = ((lane >> 4) & 1) * 4 + (lane & 3);
  const char* tr = dsw + (tr_qg >> 2) * DS_PAIR + (tr_qg & 1) * DS_HALF + ((tr_qg >> 1) & 1) * 8 + tr_krow * 16;
  for (; kb < nblk; kb += NW) {
    wave_lds_sync();
    rows_put<D>(kr, tile, lane);
    *reinterpret_cast<uint4*>(dsw + h * DS_HALF + li * 16) = dr0;
    *reinterpret_cast<uint4*>(dsw + DS_PAIR + h * DS_HALF + li * 16) = dr1;
    if (kb + NW < nblk) fetch(kb + NW);
    wave_lds_sync();
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {                    // 16 keys each
      union { short4v hh[2]; frag_t v; } f;
      f.hh[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(tr + s2 * 256));
      f.hh[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(tr + s2 * 256 + 128));
#pragma unroll
      for (int db = 0; db < NDB; ++db) acc[db] = mfma16(frag_cols_tr(tile, C::PITCH, s2 * 16, db * 32, lane), f.v, acc[db]);
    }
  }
  sums_put<D>(reinterpret_cast<float*>(tile), acc, lane);
  __syncthreads();
  const float mul = scale * (grad_scale ? grad_scale[1] : 1.0f);
  for (int q = threadIdx.x; q < 32 * D / 4; q += 64 * NW) {
    const int row = q / (D / 4), c = (q - row * (D / 4)) * 4;
    if (tl.r0 + row >= tl.r1) continue;
    const float4 v = sums_get<D, AREA>(smem, row, c, nullptr);
    *reinterpret_cast<uint2*>(dqkv + (size_t)(tl.r0 + row) * ld + a * D + c) = pack_bf16x4(make_float4(v.x * mul, v.y * mul, v.z * mul, v.w * mul));
  }
}

template <int D>
hipError_t fwd_launch(const AttnArgs& a, hipStream_t s) {
  using C = SplitCfg<D>;
  constexpr int smem = C::NW * (C::area(C::TILE) + 2 * 32 * 4);
  static std::once_flag once;
  static hipError_t once_status = hipSuccess;
  if (hipError_t e = set_max_dynamic_lds_once(once, once_status, (const void*)attn_fwd_split_kernel<D>, smem); e != hipSuccess) return e;
  const int per_tile = split_per_tile(a, ATTN_TILE_Q);
  hipLaunchKernelGGL(attn_fwd_split_kernel<D>, dim3(a.n_q_tiles * per_tile * a.nq), dim3(64 * C::NW), smem, s, (const el_t*)a.qkv,
                     (bf16_t*)a.o, a.o32, (el_t*)a.o16, a.lse, a.q_tiles, per_tile, a.T, a.nq, a.nkv, a.causal, 1.4426950408889634f / sqrtf((float)D));
  return hipGetLastError();
}

template <int D>
hipError_t dkv_launch(const AttnArgs& a, int n_sub, hipStream_t s) {
  using C = SplitCfg<D>;
  constexpr int smem = C::NW * C::area(2 * C::TILE + 256);
  static std::once_flag once;
  static hipError_t once_status = hipSuccess;
  if (hipError_t e = set_max_dynamic_lds_once(once, once_status, (const void*)attn_dkv_split_kernel<D>, smem); e != hipSuccess) return e;
  const int per_tile = split_per_tile(a, ATTN_TILE_KV);
  hipLaunchKernelGGL(attn_dkv_split_kernel<D>, dim3(a.n_kv_tiles * per_tile * a.nkv * n_sub), dim3(64 * C::NW), smem, s,
                     (const el_t*)a.qkv, (const el_t*)a.d_o, a.lse, a.delta, (bf16_t*)a.dqkv, a.kv_tiles, per_tile, a.T, a.nq, a.nkv, a.causal,
                     1.0f / sqrtf((float)D), a.grad_scale, (el_t*)a.ds, a.ds_rows, a.ds_nqs, n_sub, a.dkv_part);
  return hipGetLastError();
}

template <int D>
hipError_t dq_launch(const AttnArgs& a, hipStream_t s) {
  using C = SplitCfg<D>;
  constexpr int smem = C::NW * C::area(C::TILE + 4 * (512 + 64));
  static std::once_flag once;
  static hipError_t once_status = hipSuccess;
  if (hipError_t e = set_max_dynamic_lds_once(once, once_status, (const void*)attn_dq_split_kernel<D>, smem); e != hipSuccess) return e;
  const int per_tile = split_per_tile(a, ATTN_TILE_Q);
  hipLaunchKernelGGL(attn_dq_split_kernel<D>, dim3(a.n_q_tiles * per_tile * a.nq), dim3(64 * C::NW), smem, s, (const el_t*)a.qkv,
                     (const el_t*)a.ds, (bf16_t*)a.dqkv, a.q_tiles, per_tile, a.nq, a.nkv, a.causal, 1.0f / sqrtf((float)D), a.grad_scale, a.ds_rows, a.ds_nqs);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_fwd_split(const AttnArgs& a, hipStream_t s) {
  if (a.d == 64) return fwd_launch<64>(a, s);
  if (a.d == 80) return fwd_launch<80>(a, s);
  if (a.d == 128) return fwd_launch<128>(a, s);
  return hipErrorInvalidValue;
}
hipError_t launch_attn_dkv_split(const AttnArgs& a, int n_sub, hipStream_t s) {
  return a.d == 64 ? dkv_launch<64>(a, n_sub, s) : hipErrorInvalidValue;
}
hipError_t launch_attn_dq_split(const AttnArgs& a, hipStream_t s) {
  if (a.d == 64) return dq_launch<64>(a, s);
  if (a.d == 80) return dq_launch<80>(a, s);
  if (a.d == 128) return dq_launch<128>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace rrfp
