// fp32 attention forward and backward over packed segments (head_dim a multiple of 16, up to 128; GQA; causal or
// bidirectional), the attention of the fp32 path, on the fp32 matrix instruction v_mfma_f32_16x16x4_f32: every product
// and sum is fp32.
//
// Operand layout of the instruction: lane l carries row (or column) l & 15 and k = l >> 4 of an operand, and rows
// 4 (l >> 4) .. + 3 of column l & 15 of the 16x16 result.  Two consequences shape all kernels here:
//   - the contraction index may be permuted as long as both operands agree, so over the head dimension lane l takes
//     the four consecutive values 16 s + 4 (l >> 4) + i for the i-th of four MFMAs: 16-byte reads of rows as stored;
//   - the score block is formed in the orientation in which its 4 values per lane are, unchanged, the k operand of the
//     next product (k = row 4 (l >> 4) + r for the r-th of four MFMAs): P and dS never leave the registers.
//
// A workgroup has four wavefronts of 16 rows (queries in the forward and dQ kernels, keys in the dK/dV kernel); the
// other side streams through LDS in steps of 32 rows, double buffered, the next step's global loads in flight under
// the current one's MFMAs.  The grid has one workgroup per 64-row sub-tile of the host's tiles, so that small stages
// still spread over the chip: heads in grid x (sub-tiles there and heads in y were 2.5 % slower on an iteration of a 16-head
// stage at 1024 tokens), sub-tiles in y and, past 65535 of them (many segments of a few tokens), in z.  Bound by the fp32 matrix rate (157
// TFLOP/s) once the sequences are long enough, by the
// latency of the key loop before that, where the split kernels below take over (see attn_f32_plan for both at each size).  16 query
// heads of 64, T = 2048: forward 155 us, dQ 189, dK/dV 248.
// No atomics: sums run over ascending steps; with grouped heads every query head leaves its own dK, dV plane and the
// planes are added in head order.
#include <algorithm>

#include "kernels.h"
#include "numeric.h"

namespace rrfp {
namespace {

typedef float f32x4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4v mfma4(float a, float b, f32x4v c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

constexpr int SUB = 64;      // rows a workgroup owns
constexpr int STEP = 32;     // rows of the streamed side per step

template <int D>
struct F32Cfg {
  static constexpr int NS = D / 16;                        // 16-wide slices of the head dimension
  static constexpr int PITCH = D + 4;                      // floats: rows 4 apart sit 16 banks apart
  static constexpr int N4 = (STEP * D / 4 + 255) / 256;    // float4 per thread and tile
};

// Rows row0 .. row0 + STEP - 1 of a [*, ld] tensor (rows at or past row_end repeat row_end - 1: finite, masked later).
template <int D>
__device__ __forceinline__ void tile_fetch(f32x4v (&r)[F32Cfg<D>::N4], const float* __restrict__ p, int ld, int row0, int row_end) {
#pragma unroll
  for (int i = 0; i < F32Cfg<D>::N4; ++i) {
    const int q = min(i * 256 + (int)threadIdx.x, STEP * D / 4 - 1);
    const int row = q / (D / 4), c = q - row * (D / 4);
    r[i] = *reinterpret_cast<const f32x4v*>(p + (size_t)min(row0 + row, row_end - 1) * ld + c * 4);
  }
}
template <int D>
__device__ __forceinline__ void tile_put(const f32x4v (&r)[F32Cfg<D>::N4], float* lds) {
#pragma unroll
  for (int i = 0; i < F32Cfg<D>::N4; ++i) {
    const int q = i * 256 + (int)threadIdx.x;
    const int row = q / (D / 4), c = q - row * (D / 4);
    if (STEP * D / 4 % 256 == 0 || q < STEP * D / 4) *reinterpret_cast<f32x4v*>(lds + row * F32Cfg<D>::PITCH + c * 4) = r[i];
  }
}

// Row fragments kept in registers: row `row` of a [*, ld] tensor (zero if !exists).
template <int D>
__device__ __forceinline__ void row_frags(f32x4v (&f)[F32Cfg<D>::NS], const float* __restrict__ p, int ld, int row, bool exists, int lane) {
#pragma unroll
  for (int s = 0; s < F32Cfg<D>::NS; ++s) {
    f[s] = f32x4v{0.f, 0.f, 0.f, 0.f};
    if (exists) f[s] = *reinterpret_cast<const f32x4v*>(p + (size_t)row * ld + s * 16 + (lane >> 4) * 4);
  }
}

// acc[i] += (rows i*16 .. +15 of the LDS tile) x (register fragments), contraction over the head dimension; the two
// blocks of a step are independent chains.
template <int D>
__device__ __forceinline__ void rows_times_frags(f32x4v (&acc)[2], const float* lds, const f32x4v (&f)[F32Cfg<D>::NS], int lane) {
#pragma unroll
  for (int i = 0; i < 2; ++i) acc[i] = f32x4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < F32Cfg<D>::NS; ++s) {
    f32x4v a[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
      a[i] = *reinterpret_cast<const f32x4v*>(lds + (i * 16 + (lane & 15)) * F32Cfg<D>::PITCH + s * 16 + (lane >> 4) * 4);
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int i = 0; i < 2; ++i) acc[i] = mfma4(a[i][c], f[s][c], acc[i]);
  }
}

// out[db][d, col] += sum over the 32 rows of the LDS tile of tile[row][d] * w[row][col], w in the score layout.
template <int D>
__device__ __forceinline__ void cols_times_scores(f32x4v (&out)[F32Cfg<D>::NS], const float* lds, const f32x4v (&w)[2], int lane) {
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float* row = lds + (i * 16 + (lane >> 4) * 4 + r) * F32Cfg<D>::PITCH + (lane & 15);
#pragma unroll
      for (int db = 0; db < F32Cfg<D>::NS; ++db) out[db] = mfma4(row[db * 16], w[i][r], out[db]);
    }
}

struct SubTile { int r0, r1, s0, s1; };
// Sub-tile of SUB rows; r0 >= r1: nothing to do.
__device__ __forceinline__ SubTile sub_tile(const AttnTile* __restrict__ tiles, int n_tiles, int per_tile) {
  const int i = (int)(blockIdx.z * gridDim.y + blockIdx.y);
  if (i >= n_tiles * per_tile) return SubTile{0, 0, 0, 0};
  const AttnTile t = tiles[i / per_tile];
  const int r0 = t.r0 + i % per_tile * SUB;
  return SubTile{r0, min(r0 + SUB, t.r1), t.s0, t.s1};
}

// ------------------------------------------------------------------------- forward
template <int D>
__global__ __launch_bounds__(256) void attn_fwd_f32_kernel(const float* __restrict__ qkv, float* __restrict__ o, float* __restrict__ lse,
                                                           const AttnTile* __restrict__ tiles, int n_tiles, int Tn, int nq, int nkv, int causal) {
  constexpr int NS = F32Cfg<D>::NS;
  __shared__ __attribute__((aligned(16))) float sk[2][STEP * F32Cfg<D>::PITCH], sv[2][STEP * F32Cfg<D>::PITCH];
  const SubTile tl = sub_tile(tiles, n_tiles, ATTN_TILE_Q / SUB);
  if (tl.r0 >= tl.r1) return;
  const int a = blockIdx.x, b = a / (nq / nkv);
  const int ld = (nq + 2 * nkv) * D;
  const float* kp = qkv + (nq + b) * D;
  const float* vp = qkv + (nq + nkv + b) * D;
  const float scale = 1.0f / sqrtf((float)D);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int w0 = tl.r0 + wave * 16, qi = w0 + (lane & 15);       // this lane's query
  f32x4v qf[NS], out[NS];
  row_frags<D>(qf, qkv + a * D, ld, qi, qi < tl.r1, lane);
#pragma unroll
  for (int db = 0; db < NS; ++db) out[db] = f32x4v{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  const int kv_end = causal ? tl.r1 : tl.s1;
  const int steps = (kv_end - tl.s0 + STEP - 1) / STEP;
  const int n_active = w0 >= tl.r1 ? 0 : (causal ? min(steps, (min(w0 + 15, tl.r1 - 1) - tl.s0) / STEP + 1) : steps);
  f32x4v rk[F32Cfg<D>::N4], rv[F32Cfg<D>::N4];
  tile_fetch<D>(rk, kp, ld, tl.s0, kv_end);
  tile_fetch<D>(rv, vp, ld, tl.s0, kv_end);
  tile_put<D>(rk, sk[0]);
  tile_put<D>(rv, sv[0]);
  __syncthreads();
  for (int st = 0; st < steps; ++st) {
    const int k0 = tl.s0 + st * STEP, cur = st & 1;
    if (st + 1 < steps) {
      tile_fetch<D>(rk, kp, ld, k0 + STEP, kv_end);
      tile_fetch<D>(rv, vp, ld, k0 + STEP, kv_end);
    }
    if (st < n_active) {
      f32x4v s[2];
      rows_times_frags<D>(s, sk[cur], qf, lane);
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int j = k0 + i * 16 + (lane >> 4) * 4 + r;
          s[i][r] = (j < kv_end && (!causal || j <= qi)) ? s[i][r] * scale : -INFINITY;
          mx = fmaxf(mx, s[i][r]);
        }
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      // a step always holds an unmasked key of a query inside the tile; the guards are for the lanes past its end
      const float m_new = fmaxf(m_run, mx);
      const float alpha = m_run == -INFINITY ? 0.f : __expf(m_run - m_new);
      float ps = 0.f;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          s[i][r] = s[i][r] == -INFINITY ? 0.f : __expf(s[i][r] - m_new);
          ps += s[i][r];
        }
      ps += __shfl_xor(ps, 16, 64);
      ps += __shfl_xor(ps, 32, 64);
      l_run = l_run * alpha + ps;
      m_run = m_new;
#pragma unroll
      for (int db = 0; db < NS; ++db) out[db] *= alpha;
      cols_times_scores<D>(out, sv[cur], s, lane);
    }
    if (st + 1 < steps) {
      tile_put<D>(rk, sk[cur ^ 1]);
      tile_put<D>(rv, sv[cur ^ 1]);
    }
    __syncthreads();
  }
  if (qi < tl.r1) {
    const float inv = 1.0f / l_run;
#pragma unroll
    for (int db = 0; db < NS; ++db)
      *reinterpret_cast<f32x4v*>(o + (size_t)qi * nq * D + a * D + db * 16 + (lane >> 4) * 4) = out[db] * inv;
    if (lane < 16) lse[(size_t)a * Tn + qi] = m_run + __logf(l_run);
  }
}

// ------------------------------------------------------------------------- delta = rowsum(dO * O)
// 16 lanes per (token, head) pair.
__global__ __launch_bounds__(256) void attn_delta_f32_kernel(const float* __restrict__ o, const float* __restrict__ d_o,
                                                             float* __restrict__ delta, int Tn, int nq, int d) {
  const int pair = blockIdx.x * 16 + (threadIdx.x >> 4);
  float s = 0.f;
  if (pair < Tn * nq)
    for (int c = (threadIdx.x & 15) * 4; c < d; c += 64) {
      const f32x4v x = *reinterpret_cast<const f32x4v*>(o + (size_t)pair * d + c), y = *reinterpret_cast<const f32x4v*>(d_o + (size_t)pair * d + c);
      s += x[0] * y[0] + x[1] * y[1] + x[2] * y[2] + x[3] * y[3];
    }
#pragma unroll
  for (int off = 1; off < 16; off <<= 1) s += __shfl_xor(s, off, 64);
  if ((threadIdx.x & 15) == 0 && pair < Tn * nq) {
    const int i = pair / nq, a = pair - i * nq;
    delta[(size_t)a * Tn + i] = s;
  }
}

// ------------------------------------------------------------------------- dQ
template <int D>
__global__ __launch_bounds__(256) void attn_dq_f32_kernel(const float* __restrict__ qkv, const float* __restrict__ d_o,
                                                          const float* __restrict__ lse, const float* __restrict__ delta,
                                                          float* __restrict__ dqkv, const AttnTile* __restrict__ tiles, int n_tiles, int Tn, int nq,
                                                          int nkv, int causal) {
  constexpr int NS = F32Cfg<D>::NS;
  __shared__ __attribute__((aligned(16))) float sk[2][STEP * F32Cfg<D>::PITCH], sv[2][STEP * F32Cfg<D>::PITCH];
  const SubTile tl = sub_tile(tiles, n_tiles, ATTN_TILE_Q / SUB);
  if (tl.r0 >= tl.r1) return;
  const int a = blockIdx.x, b = a / (nq / nkv);
  const int ld = (nq + 2 * nkv) * D;
  const float* kp = qkv + (nq + b) * D;
  const float* vp = qkv + (nq + nkv + b) * D;
  const float scale = 1.0f / sqrtf((float)D);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int w0 = tl.r0 + wave * 16, qi = w0 + (lane & 15);
  f32x4v qf[NS], df[NS], out[NS];
  row_frags<D>(qf, qkv + a * D, ld, qi, qi < tl.r1, lane);
  row_frags<D>(df, d_o + a * D, nq * D, qi, qi < tl.r1, lane);
  const float lse_q = qi < tl.r1 ? lse[(size_t)a * Tn + qi] : 0.f, delta_q = qi < tl.r1 ? delta[(size_t)a * Tn + qi] : 0.f;
#pragma unroll
  for (int db = 0; db < NS; ++db) out[db] = f32x4v{0.f, 0.f, 0.f, 0.f};
  const int kv_end = causal ? tl.r1 : tl.s1;
  const int steps = (kv_end - tl.s0 + STEP - 1) / STEP;
  const int n_active = w0 >= tl.r1 ? 0 : (causal ? min(steps, (min(w0 + 15, tl.r1 - 1) - tl.s0) / STEP + 1) : steps);
  f32x4v rk[F32Cfg<D>::N4], rv[F32Cfg<D>::N4];
  tile_fetch<D>(rk, kp, ld, tl.s0, kv_end);
  tile_fetch<D>(rv, vp, ld, tl.s0, kv_end);
  tile_put<D>(rk, sk[0]);
  tile_put<D>(rv, sv[0]);
  __syncthreads();
  for (int st = 0; st < steps; ++st) {
    const int k0 = tl.s0 + st * STEP, cur = st & 1;
    if (st + 1 < steps) {
      tile_fetch<D>(rk, kp, ld, k0 + STEP, kv_end);
      tile_fetch<D>(rv, vp, ld, k0 + STEP, kv_end);
    }
    if (st < n_active) {
      f32x4v s[2], dp[2];
      rows_times_frags<D>(s, sk[cur], qf, lane);
      rows_times_frags<D>(dp, sv[cur], df, lane);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int j = k0 + i * 16 + (lane >> 4) * 4 + r;
          const float p = (qi < tl.r1 && j < kv_end && (!causal || j <= qi)) ? __expf(s[i][r] * scale - lse_q) : 0.f;
          s[i][r] = p * (dp[i][r] - delta_q);
        }
      cols_times_scores<D>(out, sk[cur], s, lane);
    }
    if (st + 1 < steps) {
      tile_put<D>(rk, sk[cur ^ 1]);
      tile_put<D>(rv, sv[cur ^ 1]);
    }
    __syncthreads();
  }
  if (qi < tl.r1)
#pragma unroll
    for (int db = 0; db < NS; ++db)
      *reinterpret_cast<f32x4v*>(dqkv + (size_t)qi * ld + a * D + db * 16 + (lane >> 4) * 4) = out[db] * scale;
}

// ------------------------------------------------------------------------- dK, dV
// One workgroup per 64 keys and QUERY head.  part == null (one query head per KV head): dK, dV go to dqkv; otherwise
// the unscaled sums go to this head's plane [tensor][head of the group][token][KV head * D + d].
template <int D>
__global__ __launch_bounds__(256) void attn_dkv_f32_kernel(const float* __restrict__ qkv, const float* __restrict__ d_o,
                                                           const float* __restrict__ lse, const float* __restrict__ delta,
                                                           float* __restrict__ dqkv, const AttnTile* __restrict__ tiles, int n_tiles, int Tn, int nq,
                                                           int nkv, int causal, float* __restrict__ part) {
  constexpr int NS = F32Cfg<D>::NS;
  __shared__ __attribute__((aligned(16))) float sq[2][STEP * F32Cfg<D>::PITCH], sd[2][STEP * F32Cfg<D>::PITCH];
  __shared__ __attribute__((aligned(16))) float stat[2][2 * STEP];      // lse, delta of the step's rows
  const SubTile tl = sub_tile(tiles, n_tiles, ATTN_TILE_KV / SUB);
  if (tl.r0 >= tl.r1) return;
  const int a = blockIdx.x, G = nq / nkv, b = a / G;
  const int ld = (nq + 2 * nkv) * D;
  const float scale = 1.0f / sqrtf((float)D);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int w0 = tl.r0 + wave * 16, kj = w0 + (lane & 15);              // this lane's key
  f32x4v kf[NS], vf[NS], dk[NS], dv[NS];
  row_frags<D>(kf, qkv + (nq + b) * D, ld, kj, kj < tl.r1, lane);
  row_frags<D>(vf, qkv + (nq + nkv + b) * D, ld, kj, kj < tl.r1, lane);
#pragma unroll
  for (int db = 0; db < NS; ++db) { dk[db] = f32x4v{0.f, 0.f, 0.f, 0.f}; dv[db] = dk[db]; }
  const int q_begin = causal ? tl.r0 : tl.s0;
  const int steps = (tl.s1 - q_begin + STEP - 1) / STEP;
  const bool wave_has_keys = w0 < tl.r1;
  f32x4v rq[F32Cfg<D>::N4], rd[F32Cfg<D>::N4];
  float rs = 0.f;
  auto fetch = [&](int st) {
    const int q0 = q_begin + st * STEP;
    tile_fetch<D>(rq, qkv + a * D, ld, q0, tl.s1);
    tile_fetch<D>(rd, d_o + a * D, nq * D, q0, tl.s1);
    const int i = min(q0 + (int)(threadIdx.x & (STEP - 1)), tl.s1 - 1);
    if (threadIdx.x < 2 * STEP) rs = (threadIdx.x < STEP ? lse : delta)[(size_t)a * Tn + i];
  };
  auto put = [&](int buf) {
    tile_put<D>(rq, sq[buf]);
    tile_put<D>(rd, sd[buf]);
    if (threadIdx.x < 2 * STEP) stat[buf][threadIdx.x] = rs;
  };
  fetch(0);
  put(0);
  __syncthreads();
  for (int st = 0; st < steps; ++st) {
    const int q0 = q_begin + st * STEP, cur = st & 1;
    if (st + 1 < steps) fetch(st + 1);
    if (wave_has_keys && (!causal || q0 + STEP > w0)) {
      f32x4v s[2], dp[2];
      rows_times_frags<D>(s, sq[cur], kf, lane);
      rows_times_frags<D>(dp, sd[cur], vf, lane);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const f32x4v l4 = *reinterpret_cast<const f32x4v*>(&stat[cur][i * 16 + (lane >> 4) * 4]);
        const f32x4v d4 = *reinterpret_cast<const f32x4v*>(&stat[cur][STEP + i * 16 + (lane >> 4) * 4]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int qi = q0 + i * 16 + (lane >> 4) * 4 + r;
          const float p = (qi < tl.s1 && kj < tl.r1 && (!causal || kj <= qi)) ? __expf(s[i][r] * scale - l4[r]) : 0.f;
          s[i][r] = p;
          dp[i][r] = p * (dp[i][r] - d4[r]);
        }
      }
      cols_times_scores<D>(dv, sd[cur], s, lane);
      cols_times_scores<D>(dk, sq[cur], dp, lane);
    }
    if (st + 1 < steps) put(cur ^ 1);
    __syncthreads();
  }
  if (kj >= tl.r1) return;
#pragma unroll
  for (int db = 0; db < NS; ++db) {
    const int c = db * 16 + (lane >> 4) * 4;
    if (part) {
      const size_t plane = (size_t)Tn * nkv * D, off = (size_t)kj * nkv * D + b * D + c;
      *reinterpret_cast<f32x4v*>(part + (size_t)(a - b * G) * plane + off) = dk[db];
      *reinterpret_cast<f32x4v*>(part + (size_t)(G + a - b * G) * plane + off) = dv[db];
    } else {
      *reinterpret_cast<f32x4v*>(dqkv + (size_t)kj * ld + (nq + b) * D + c) = dk[db] * scale;
      *reinterpret_cast<f32x4v*>(dqkv + (size_t)kj * ld + (nq + nkv + b) * D + c) = dv[db];
    }
  }
}

// ------------------------------------------------------------------------- short grids: the streamed side dealt to the wavefronts
// When 64-row sub-tiles leave CUs idle, the time of the kernels above is one wavefront's serial walk over the other side (2.2 us per
// 32 rows).  Here a workgroup owns 16 rows and its eight wavefronts take the 16-row blocks of the other side in turn, straight from
// memory (no LDS, no barrier in the walk); their sums meet in LDS and are added in wavefront order.
constexpr int SPLIT = 8, ROWS = 16;                     // wavefronts of a workgroup; rows it owns

// Sub-tile of ROWS rows; per_tile of them are launched for each tile: as many as the longest segment has (r0 >= r1: nothing to do).  Every
// tile starts at another one: with few heads a sub-tile's place in its tile would decide its XCD, and segments that end early would
// leave some of them without work.
__device__ __forceinline__ SubTile split_tile(const AttnTile* __restrict__ tiles, int n_tiles, int per_tile) {
  const int i = (int)(blockIdx.z * gridDim.y + blockIdx.y), tile = i / per_tile;
  if (tile >= n_tiles) return SubTile{0, 0, 0, 0};
  const AttnTile t = tiles[tile];
  const int r0 = t.r0 + (i + tile) % per_tile * ROWS;
  return SubTile{r0, min(r0 + ROWS, t.r1), t.s0, t.s1};
}

// Block of 16 rows at row0 of a [*, ld] tensor, rows at or past row_end repeat row_end - 1.  Rows: lane l has row l & 15, the values
// 16 s + 4 (l >> 4) .. + 3 of slice s.  Columns: lane l has value 16 db + (l & 15) of row 4 (l >> 4) + r.
template <int D>
__device__ __forceinline__ void block_rows(f32x4v (&f)[F32Cfg<D>::NS], const float* __restrict__ p, int ld, int row0, int row_end, int lane) {
  const float* row = p + (size_t)min(row0 + (lane & 15), row_end - 1) * ld + (lane >> 4) * 4;
#pragma unroll
  for (int s = 0; s < F32Cfg<D>::NS; ++s) f[s] = *reinterpret_cast<const f32x4v*>(row + s * 16);
}
template <int D>
__device__ __forceinline__ void block_cols(f32x4v (&f)[F32Cfg<D>::NS], const float* __restrict__ p, int ld, int row0, int row_end, int lane) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float* row = p + (size_t)min(row0 + (lane >> 4) * 4 + r, row_end - 1) * ld + (lane & 15);
#pragma unroll
    for (int db = 0; db < F32Cfg<D>::NS; ++db) f[db][r] = row[db * 16];
  }
}
// a (16 rows) x b's fragments over the head dimension, in two chains
template <int D>
__device__ __forceinline__ f32x4v block_scores(const f32x4v (&a)[F32Cfg<D>::NS], const f32x4v (&b)[F32Cfg<D>::NS]) {
  f32x4v acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int s = 0; s < F32Cfg<D>::NS; ++s)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c & 1] = mfma4(a[s][c], b[s][c], acc[c & 1]);
  return acc[0] + acc[1];
}
// out[db] += columns x weights w in the score layout
template <int D>
__device__ __forceinline__ void block_outer(f32x4v (&out)[F32Cfg<D>::NS], const f32x4v (&cols)[F32Cfg<D>::NS], const f32x4v& w) {
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int db = 0; db < F32Cfg<D>::NS; ++db) out[db] = mfma4(cols[db][r], w[r], out[db]);
}
// This wavefront's sums to its part of the exchange area [SPLIT][ROWS][D + 4].
template <int D>
__device__ __forceinline__ void put_sums(float* area, const f32x4v (&out)[F32Cfg<D>::NS], int wave, int lane) {
  float* mine = area + (wave * ROWS + (lane & 15)) * F32Cfg<D>::PITCH + (lane >> 4) * 4;
#pragma unroll
  for (int db = 0; db < F32Cfg<D>::NS; ++db) *reinterpret_cast<f32x4v*>(mine + db * 16) = out[db];
}
// Sum over the wavefronts of four values of a row, each times its factor.
template <int D>
__device__ __forceinline__ f32x4v get_sum(const float* area, int row, int c, const float* factor) {
  f32x4v v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < SPLIT; ++w) {
    const f32x4v x = *reinterpret_cast<const f32x4v*>(area + (w * ROWS + row) * F32Cfg<D>::PITCH + c);
    v += factor ? x * factor[w * ROWS + row] : x;
  }
  return v;
}

template <int D>
__global__ __launch_bounds__(64 * SPLIT) void attn_fwd_f32_split_kernel(const float* __restrict__ qkv, float* __restrict__ o, float* __restrict__ lse,
                                                                        const AttnTile* __restrict__ tiles, int n_tiles, int per_tile, int Tn, int nq, int nkv,
                                                                        int causal) {
  constexpr int NS = F32Cfg<D>::NS;
  __shared__ __attribute__((aligned(16))) float area[SPLIT * ROWS * F32Cfg<D>::PITCH];
  __shared__ float ms[SPLIT * ROWS], ls[SPLIT * ROWS];
  const SubTile tl = split_tile(tiles, n_tiles, per_tile);
  if (tl.r0 >= tl.r1) return;
  const int a = blockIdx.x, b = a / (nq / nkv);
  const int ld = (nq + 2 * nkv) * D;
  const float* kp = qkv + (nq + b) * D;
  const float* vp = qkv + (nq + nkv + b) * D;
  const float scale = 1.0f / sqrtf((float)D);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int qi = tl.r0 + (lane & 15);                   // this lane's query
  f32x4v qf[NS], out[NS], kf[NS], vf[NS];
  float m_run = -INFINITY, l_run = 0.f;
  block_rows<D>(qf, qkv + a * D, ld, tl.r0, tl.r1, lane);
#pragma unroll
  for (int db = 0; db < NS; ++db) out[db] = f32x4v{0.f, 0.f, 0.f, 0.f};
  const int kv_end = causal ? tl.r1 : tl.s1;
  int k0 = tl.s0 + wave * 16;
  if (k0 < kv_end) block_rows<D>(kf, kp, ld, k0, kv_end, lane);
  for (; k0 < kv_end; k0 += 16 * SPLIT) {
    block_cols<D>(vf, vp, ld, k0, kv_end, lane);
    f32x4v s = block_scores<D>(kf, qf);
    if (k0 + 16 * SPLIT < kv_end) block_rows<D>(kf, kp, ld, k0 + 16 * SPLIT, kv_end, lane);
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = k0 + (lane >> 4) * 4 + r;
      s[r] = (j < kv_end && (!causal || j <= qi)) ? s[r] * scale : -INFINITY;
      mx = fmaxf(mx, s[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m_run, mx);              // -inf while every key so far is masked
    const float alpha = m_run == -INFINITY ? 0.f : __expf(m_run - m_new);
    float ps = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[r] = s[r] == -INFINITY ? 0.f : __expf(s[r] - m_new);
      ps += s[r];
    }
    ps += __shfl_xor(ps, 16, 64);
    ps += __shfl_xor(ps, 32, 64);
    l_run = l_run * alpha + ps;
    m_run = m_new;
#pragma unroll
    for (int db = 0; db < NS; ++db) out[db] *= alpha;
    block_outer<D>(out, vf, s);
  }
  put_sums<D>(area, out, wave, lane);
  if (lane < 16) {
    ms[wave * ROWS + lane] = m_run;
    ls[wave * ROWS + lane] = l_run;
  }
  __syncthreads();
  if (threadIdx.x < ROWS) {                            // factors that bring the wavefronts to one reference point, over the row's sum
    const int row = threadIdx.x;
    float m = ms[row];
#pragma unroll
    for (int w = 1; w < SPLIT; ++w) m = fmaxf(m, ms[w * ROWS + row]);
    float l = 0.f;
#pragma unroll
    for (int w = 0; w < SPLIT; ++w) l += ls[w * ROWS + row] == 0.f ? 0.f : ls[w * ROWS + row] * __expf(ms[w * ROWS + row] - m);
    const float inv = 1.0f / l;
#pragma unroll
    for (int w = 0; w < SPLIT; ++w) ms[w * ROWS + row] = ls[w * ROWS + row] == 0.f ? 0.f : __expf(ms[w * ROWS + row] - m) * inv;
    if (tl.r0 + row < tl.r1) lse[(size_t)a * Tn + tl.r0 + row] = m + __logf(l);
  }
  __syncthreads();
  for (int q = threadIdx.x; q < ROWS * D / 4; q += 64 * SPLIT) {
    const int row = q / (D / 4), c = (q - row * (D / 4)) * 4;
    if (tl.r0 + row < tl.r1) *reinterpret_cast<f32x4v*>(o + (size_t)(tl.r0 + row) * nq * D + a * D + c) = get_sum<D>(area, row, c, ms);
  }
}

template <int D>
__global__ __launch_bounds__(64 * SPLIT) void attn_dq_f32_split_kernel(const float* __restrict__ qkv, const float* __restrict__ d_o,
                                                                       const float* __restrict__ lse, const float* __restrict__ delta,
                                                                       float* __restrict__ dqkv, const AttnTile* __restrict__ tiles, int n_tiles, int per_tile,
                                                                       int Tn, int nq, int nkv, int causal) {
  constexpr int NS = F32Cfg<D>::NS;
  __shared__ __attribute__((aligned(16))) float area[SPLIT * ROWS * F32Cfg<D>::PITCH];
  const SubTile tl = split_tile(tiles, n_tiles, per_tile);
  if (tl.r0 >= tl.r1) return;
  const int a = blockIdx.x, b = a / (nq / nkv);
  const int ld = (nq + 2 * nkv) * D;
  const float* kp = qkv + (nq + b) * D;
  const float* vp = qkv + (nq + nkv + b) * D;
  const float scale = 1.0f / sqrtf((float)D);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int qi = min(tl.r0 + (lane & 15), tl.r1 - 1);   // this lane's query; past the end the last one, not stored
  f32x4v qf[NS], df[NS], out[NS], kf[NS], vf[NS], kc[NS];
  block_rows<D>(qf, qkv + a * D, ld, tl.r0, tl.r1, lane);
  block_rows<D>(df, d_o + a * D, nq * D, tl.r0, tl.r1, lane);
  const float lse_q = lse[(size_t)a * Tn + qi], delta_q = delta[(size_t)a * Tn + qi];
#pragma unroll
  for (int db = 0; db < NS; ++db) out[db] = f32x4v{0.f, 0.f, 0.f, 0.f};
  const int kv_end = causal ? tl.r1 : tl.s1;
  for (int k0 = tl.s0 + wave * 16; k0 < kv_end; k0 += 16 * SPLIT) {
    block_rows<D>(kf, kp, ld, k0, kv_end, lane);
    block_rows<D>(vf, vp, ld, k0, kv_end, lane);
    block_cols<D>(kc, kp, ld, k0, kv_end, lane);
    f32x4v s = block_scores<D>(kf, qf);
    const f32x4v dp = block_scores<D>(vf, df);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = k0 + (lane >> 4) * 4 + r;
      const float p = (j < kv_end && (!causal || j <= qi)) ? __expf(s[r] * scale - lse_q) : 0.f;
      s[r] = p * (dp[r] - delta_q);
    }
    block_outer<D>(out, kc, s);
  }
  put_sums<D>(area, out, wave, lane);
  __syncthreads();
  for (int q = threadIdx.x; q < ROWS * D / 4; q += 64 * SPLIT) {
    const int row = q / (D / 4), c = (q - row * (D / 4)) * 4;
    if (tl.r0 + row < tl.r1)
      *reinterpret_cast<f32x4v*>(dqkv + (size_t)(tl.r0 + row) * ld + a * D + c) = get_sum<D>(area, row, c, nullptr) * scale;
  }
}

template <int D>
__global__ __launch_bounds__(64 * SPLIT) void attn_dkv_f32_split_kernel(const float* __restrict__ qkv, const float* __restrict__ d_o,
                                                                        const float* __restrict__ lse, const float* __restrict__ delta,
                                                                        float* __restrict__ dqkv, const AttnTile* __restrict__ tiles, int n_tiles, int per_tile,
                                                                        int Tn, int nq, int nkv, int causal, float* __restrict__ part) {
  constexpr int NS = F32Cfg<D>::NS;
  __shared__ __attribute__((aligned(16))) float area[SPLIT * ROWS * F32Cfg<D>::PITCH];
  const SubTile tl = split_tile(tiles, n_tiles, per_tile);
  if (tl.r0 >= tl.r1) return;
  const int a = blockIdx.x, G = nq / nkv, b = a / G;
  const int ld = (nq + 2 * nkv) * D;
  const float scale = 1.0f / sqrtf((float)D);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int key = tl.r0 + (lane & 15);                  // of this lane; not stored when past the end
  f32x4v kf[NS], vf[NS], dk[NS], dv[NS], x[NS], y[NS];
  block_rows<D>(kf, qkv + (nq + b) * D, ld, tl.r0, tl.r1, lane);
  block_rows<D>(vf, qkv + (nq + nkv + b) * D, ld, tl.r0, tl.r1, lane);
#pragma unroll
  for (int db = 0; db < NS; ++db) { dk[db] = f32x4v{0.f, 0.f, 0.f, 0.f}; dv[db] = dk[db]; }
  for (int q0 = (causal ? tl.r0 : tl.s0) + wave * 16; q0 < tl.s1; q0 += 16 * SPLIT) {
    f32x4v l4, d4;
    block_rows<D>(x, qkv + a * D, ld, q0, tl.s1, lane);
    block_rows<D>(y, d_o + a * D, nq * D, q0, tl.s1, lane);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const size_t qi = (size_t)a * Tn + min(q0 + (lane >> 4) * 4 + r, tl.s1 - 1);
      l4[r] = lse[qi];
      d4[r] = delta[qi];
    }
    f32x4v s = block_scores<D>(x, kf), dp = block_scores<D>(y, vf);
    block_cols<D>(x, qkv + a * D, ld, q0, tl.s1, lane);
    block_cols<D>(y, d_o + a * D, nq * D, q0, tl.s1, lane);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int qi = q0 + (lane >> 4) * 4 + r;
      const float p = (qi < tl.s1 && (!causal || key <= qi)) ? __expf(s[r] * scale - l4[r]) : 0.f;
      s[r] = p;
      dp[r] = p * (dp[r] - d4[r]);
    }
    block_outer<D>(dk, x, dp);
    block_outer<D>(dv, y, s);
  }
#pragma unroll
  for (int tensor = 0; tensor < 2; ++tensor) {
    if (tensor) __syncthreads();
    put_sums<D>(area, tensor ? dv : dk, wave, lane);
    __syncthreads();
    for (int q = threadIdx.x; q < ROWS * D / 4; q += 64 * SPLIT) {
      const int row = q / (D / 4), c = (q - row * (D / 4)) * 4, kj = tl.r0 + row;
      if (kj >= tl.r1) continue;
      const f32x4v v = get_sum<D>(area, row, c, nullptr);
      if (part) *reinterpret_cast<f32x4v*>(part + ((size_t)(tensor * G + a - b * G) * Tn + kj) * nkv * D + b * D + c) = v;
      else *reinterpret_cast<f32x4v*>(dqkv + (size_t)kj * ld + (nq + tensor * nkv + b) * D + c) = tensor ? v : v * scale;
    }
  }
}

// dK, dV = sum of the G planes of a group in head order.
__global__ __launch_bounds__(256) void dkv_combine_f32_kernel(const float* __restrict__ part, float* __restrict__ dqkv, int Tn, int nq,
                                                              int nkv, int D, float scale) {
  const int W = nkv * D, G = nq / nkv;
  const size_t plane = (size_t)Tn * W, idx = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (idx >= plane) return;
  const int j = (int)(idx / W), c = (int)(idx - (size_t)j * W);
#pragma unroll
  for (int tensor = 0; tensor < 2; ++tensor) {
    const float* p = part + (size_t)tensor * G * plane + idx;
    f32x4v acc = *reinterpret_cast<const f32x4v*>(p);
    for (int g = 1; g < G; ++g) acc += *reinterpret_cast<const f32x4v*>(p + (size_t)g * plane);
    *reinterpret_cast<f32x4v*>(dqkv + (size_t)j * (nq + 2 * nkv) * D + (nq + tensor * nkv) * D + c) = tensor == 0 ? acc * scale : acc;
  }
}

int split_per_tile(const AttnArgs& a, int tile_rows) { return (std::min(a.longest, tile_rows) + ROWS - 1) / ROWS; }
dim3 sub_tile_grid(int nq, int n) {
  const int z = (n + 65534) / 65535;
  return dim3(nq, (n + z - 1) / z, z);
}

template <int D>
hipError_t fwd_launch(const AttnArgs& a, hipStream_t s) {
  if (attn_f32_plan(a, device_cu_count()).fwd) {
    const int per_tile = split_per_tile(a, ATTN_TILE_Q);
    hipLaunchKernelGGL(attn_fwd_f32_split_kernel<D>, sub_tile_grid(a.nq, a.n_q_tiles * per_tile), dim3(64 * SPLIT), 0, s, (const float*)a.qkv,
                       (float*)a.o, a.lse, a.q_tiles, a.n_q_tiles, per_tile, a.T, a.nq, a.nkv, a.causal);
  } else {
    hipLaunchKernelGGL(attn_fwd_f32_kernel<D>, sub_tile_grid(a.nq, a.n_q_tiles * (ATTN_TILE_Q / SUB)), dim3(256), 0, s, (const float*)a.qkv,
                       (float*)a.o, a.lse, a.q_tiles, a.n_q_tiles, a.T, a.nq, a.nkv, a.causal);
  }
  return hipGetLastError();
}

template <int D>
hipError_t bwd_launch(const AttnArgs& a, hipStream_t s) {
  float* part = a.nq > a.nkv ? a.dkv_part : nullptr;
  const AttnPlan plan = attn_f32_plan(a, device_cu_count());
  hipLaunchKernelGGL(attn_delta_f32_kernel, dim3((a.T * a.nq + 15) / 16), dim3(256), 0, s, (const float*)a.o, (const float*)a.d_o, a.delta, a.T,
                     a.nq, a.d);
  if (plan.dkv) {
    const int per_tile = split_per_tile(a, ATTN_TILE_KV);
    hipLaunchKernelGGL(attn_dkv_f32_split_kernel<D>, sub_tile_grid(a.nq, a.n_kv_tiles * per_tile), dim3(64 * SPLIT), 0, s, (const float*)a.qkv,
                       (const float*)a.d_o, a.lse, a.delta, (float*)a.dqkv, a.kv_tiles, a.n_kv_tiles, per_tile, a.T, a.nq, a.nkv, a.causal, part);
  } else {
    hipLaunchKernelGGL(attn_dkv_f32_kernel<D>, sub_tile_grid(a.nq, a.n_kv_tiles * (ATTN_TILE_KV / SUB)), dim3(256), 0, s, (const float*)a.qkv,
                       (const float*)a.d_o, a.lse, a.delta, (float*)a.dqkv, a.kv_tiles, a.n_kv_tiles, a.T, a.nq, a.nkv, a.causal, part);
  }
  if (part)
    hipLaunchKernelGGL(dkv_combine_f32_kernel, dim3((unsigned)(((size_t)a.T * a.nkv * D / 4 + 255) / 256)), dim3(256), 0, s, part,
                       (float*)a.dqkv, a.T, a.nq, a.nkv, D, 1.0f / sqrtf((float)D));
  if (plan.dq) {
    const int per_tile = split_per_tile(a, ATTN_TILE_Q);
    hipLaunchKernelGGL(attn_dq_f32_split_kernel<D>, sub_tile_grid(a.nq, a.n_q_tiles * per_tile), dim3(64 * SPLIT), 0, s, (const float*)a.qkv,
                       (const float*)a.d_o, a.lse, a.delta, (float*)a.dqkv, a.q_tiles, a.n_q_tiles, per_tile, a.T, a.nq, a.nkv, a.causal);
  } else {
    hipLaunchKernelGGL(attn_dq_f32_kernel<D>, sub_tile_grid(a.nq, a.n_q_tiles * (ATTN_TILE_Q / SUB)), dim3(256), 0, s, (const float*)a.qkv,
                       (const float*)a.d_o, a.lse, a.delta, (float*)a.dqkv, a.q_tiles, a.n_q_tiles, a.T, a.nq, a.nkv, a.causal);
  }
  return hipGetLastError();
}

}  // namespace

#define RRFP_HEAD_DIMS(CALL) \
  switch (a.d) {             \
    case 16: return CALL<16>(a, s);   \
    case 32: return CALL<32>(a, s);   \
    case 48: return CALL<48>(a, s);   \
    case 64: return CALL<64>(a, s);   \
    case 80: return CALL<80>(a, s);   \
    case 96: return CALL<96>(a, s);   \
    case 112: return CALL<112>(a, s); \
    case 128: return CALL<128>(a, s); \
    default: return hipErrorInvalidValue; \
  }

// Where the split kernels are launched (attn_deal; measured below two 64-row sub-tiles of a query head per CU, and kept from there on
// where the tiled ones win: 2048 x 16 heads 248 -> 258 us in dK/dV, 4096 x 16 543 -> 682 in dQ).  A bidirectional row counts twice,
// in the forward also a row of more than 64 columns, whose sums leave a CU two workgroups instead of four.  us, tiled -> split, forward, dK/dV,
// dQ, in brackets where it is not launched; 16 heads of 64, causal, rows in segments of one length: 1269 of 1024 69.6 -> 42.4, 102.4 -> 84.4, 82.6 -> 57.2;
// 1024 of 512 34.5 -> 25.7, 51.6 -> 49.1, 39.6 -> 35.0; of 256 19.4 -> 20.3, (28.8 -> 34.9), (21.5 -> 25.2); of 128 16.5 -> 14.6, (17.9 -> 25.5), (18.9 -> 17.1);
// 614 of 128 15.1 -> 10.5, (16.7 -> 18.8), 18.8 -> 12.3; 409 of 32 7.1 -> 6.4, 9.2 -> 9.6, 8.5 -> 6.1; 1986 of 512 41.6 -> 42.6, (66.6 -> 88.6), (49.8 -> 60.1).
// 4 heads of 128, bidirectional: 983 of 128 17.6 -> 12.0, 28.2 -> 16.5, 20.7 -> 11.3; 3276 of 512 (56.5 -> 69.4), (93.5 -> 117.5), (70.4 -> 89.1); 7946 of 32
// 54 -> 38, (75 -> 59), 71 -> 47.  32 rows a workgroup: slower up to 1024 x 16.
AttnPlan attn_f32_plan(const AttnArgs& a, int n_cu) {
  if ((long long)a.T * a.nq >= 2LL * SUB * n_cu) return AttnPlan{false, false, false};
  const float both = a.causal ? 1.0f : 2.0f, wide = a.d > 64 ? 2.0f : 1.0f;
  return AttnPlan{attn_deal(a, n_cu, AttnLine{64.f, 4.0f, 64}, both * wide, ROWS), attn_deal(a, n_cu, AttnLine{28.f, 2.5f, 16}, both, ROWS),
                  attn_deal(a, n_cu, AttnLine{48.f, 1.5f, 64}, both, ROWS)};
}

hipError_t launch_attn_fwd_f32(const AttnArgs& a, hipStream_t s) {
  if (a.dtype != F32 || a.n_q_tiles < 1) return hipErrorInvalidValue;
  RRFP_HEAD_DIMS(fwd_launch)
}

hipError_t launch_attn_bwd_f32(const AttnArgs& a, hipStream_t s) {
  if (a.dtype != F32 || a.n_q_tiles < 1 || a.n_kv_tiles < 1 || (a.nq > a.nkv && !a.dkv_part)) return hipErrorInvalidValue;
  RRFP_HEAD_DIMS(bwd_launch)
}

}  // namespace rrfp
