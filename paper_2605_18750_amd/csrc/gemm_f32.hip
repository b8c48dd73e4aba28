// fp32 GEMM on the fp32 matrix instruction v_mfma_f32_32x32x2_f32: C[M,N] = A(m,k) B(k,n) (+ bias) (+ R), the
// GEMM of the fp32 path for every operand orientation, size and alignment.
//
// Why MFMA: without packed arithmetic the vector pipes reach half of the chip's fp32 rate (157 TFLOP/s), and an
// fp32-FMA kernel needs an LDS read for every few FMAs; one 32x32x2 MFMA takes two registers and keeps the matrix
// pipe busy for 64 cycles, so neither LDS nor issue slots limit anything here.  Products and sums stay fp32.
//
// Three tile routines, chosen by the size of the output alone (see f32_tile_edge):
//   f32_tile   tiles of 64 x 64, eight wavefronts, 32-deep k steps through three LDS buffers (global loads four steps
//     ahead, one barrier per step).  1024 x 1024 x 5504: 98 us = 117 TFLOP/s, 4096^3: 1033 us = 133 (this card's vendor product: 154).
//     With two buffers, loads two steps ahead behind branches and the reads of a step behind its barrier: 113 and 1157 us.  (128 x 128 tiles:
//     5 % faster than those at 4096^3, two to four times slower on outputs of up to 1024 rows.  Sixteen wavefronts and 64-deep steps:
//     93 us at 1024 x 1024 x 5504, but 129 against 112 at 1024 x 5504 x 1024.)
//   f32_small  tiles of 32 x 32 whose eight wavefronts split the contraction and read their
//     fragments straight from global memory (L2): for outputs with too few tiles to fill the chip the time is the
//     latency of the serial k loop, and this cuts the loop and takes the barriers out of it (128 x 256 x 688: 95 -> 8 us).
//   f32_tiny   the same with tiles of 16 x 16 for the smallest outputs (128 x 256 x 688: 8 -> 5 us).
//
// The contraction index is free to be permuted as long as both operands agree: in a chunk of 8 k the half h of a
// wavefront holds k = 4h + i for the i-th of four MFMAs, so a K-contiguous operand is read 16 bytes at a time.
// Every output element is summed in one fixed order (k chunks ascending inside a wavefront, the ranges of
// the wavefronts added in order), so a call always gives the same bits.
#include <algorithm>
#include <climits>

#include "kernels.h"
#include "numeric.h"

namespace rrfp {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// Four consecutive values at p[0..3], of which the first n (<= 0: none) exist.  VEC: they exist together and p is
// 16-byte aligned.
template <bool VEC>
__device__ __forceinline__ f32x4v load4(const float* __restrict__ p, int n) {
  f32x4v v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (VEC) {
    if (n > 0) v = *reinterpret_cast<const f32x4v*>(p);
  } else {
    if (n > 0) v.x = p[0];
    if (n > 1) v.y = p[1];
    if (n > 2) v.z = p[2];
    if (n > 3) v.w = p[3];
  }
  return v;
}

constexpr int FK = 32;       // k per step of the tile kernel (64 measured the same at K >= 1024, 6 to 15 % slower in the weight-gradient form)
constexpr int KC_PITCH = FK + 4;   // floats per row of a K-contiguous tile: 16 rows of a b128 read fall into 16 bank groups

// One operand tile of ROWS rows x FK k, moved by NT threads.  KC: stored [rows][K] in memory and [rows][KC_PITCH] in LDS; else stored
// [K][rows] and [FK][ROWS + 8] in LDS (the two halves of a wavefront read k rows 4 apart: 4 * pitch = 32 mod 64).
template <bool KC, int ROWS, bool VEC, int NT>
struct F32Tile {
  static constexpr int N4 = ROWS * FK / 4 / NT;                // float4 per thread
  static constexpr int KS_PITCH = ROWS + 8;
  static constexpr int FLOATS = KC ? ROWS * KC_PITCH : FK * KS_PITCH;
  __device__ static __forceinline__ void load(f32x4v (&r)[N4], const float* __restrict__ p, int ld, int row0, int n_rows, int k0, int K) {
#pragma unroll
    for (int i = 0; i < N4; ++i) {
      const int q = i * NT + threadIdx.x;
      if constexpr (KC) {
        const int row = row0 + (q / (FK / 4)), k = k0 + (q % (FK / 4)) * 4;
        r[i] = load4<VEC>(p + (size_t)row * ld + k, row < n_rows ? K - k : 0);
      } else {
        const int k = k0 + q / (ROWS / 4), row = row0 + (q % (ROWS / 4)) * 4;
        r[i] = load4<VEC>(p + (size_t)k * ld + row, k < K ? n_rows - row : 0);
      }
    }
  }
  __device__ static __forceinline__ void store(const f32x4v (&r)[N4], float* lds) {
#pragma unroll
    for (int i = 0; i < N4; ++i) {
      const int q = i * NT + threadIdx.x;
      if constexpr (KC) *reinterpret_cast<f32x4v*>(lds + (q / (FK / 4)) * KC_PITCH + (q % (FK / 4)) * 4) = r[i];
      else *reinterpret_cast<f32x4v*>(lds + (q / (ROWS / 4)) * KS_PITCH + (q % (ROWS / 4)) * 4) = r[i];
    }
  }
  // Operand of the four MFMAs of k chunk s (8 k) for the 32 rows at row0: lane l has row l & 31, k = 8s + 4 (l >> 5) + i.
  __device__ static __forceinline__ f32x4v frag(const float* lds, int row0, int s, int lane) {
    const int row = row0 + (lane & 31), k = s * 8 + (lane >> 5) * 4;
    if constexpr (KC) {
      return *reinterpret_cast<const f32x4v*>(lds + row * KC_PITCH + k);
    } else {
      const float* p = lds + k * KS_PITCH + row;
      return f32x4v{p[0], p[KS_PITCH], p[2 * KS_PITCH], p[3 * KS_PITCH]};
    }
  }
};

// The tiles of an operand along K, for F32Tile::store.  VEC: buffer loads without a branch (what does not exist carries an offset past the
// buffer and reads as zero), so that the waits for them count exactly; the base moves with the step, offsets stay within one tile.
constexpr int VEC_MAX_LD = 1 << 22;
template <bool KC, int ROWS, bool VEC, int NT>
struct F32Stream {
  using Tile = F32Tile<KC, ROWS, VEC, NT>;
  static constexpr int N4 = Tile::N4;
  const float* p;
  int ld, row0, n_rows, K;
  int voff[N4], k_in[N4];                              // byte offset inside a tile (or past it), k inside the step
  // pair_f > 0 (K-strided, VEC): the columns of a SwiGLU forward of pair_f features, as f32_column
  __device__ __forceinline__ F32Stream(const float* p_, int ld_, int row0_, int n_rows_, int K_, int pair_f = 0)
      : p(p_), ld(ld_), row0(pair_f > 0 ? 0 : row0_), n_rows(n_rows_), K(K_) {
#pragma unroll
    for (int i = 0; i < N4; ++i) {
      const int q = i * NT + threadIdx.x;
      int row = KC ? q / (FK / 4) : q % (ROWS / 4) * 4;
      if (pair_f > 0) {
        const int f = (row0_ >> 1) + row % (ROWS / 2);
        row = f < pair_f ? f + (row >= ROWS / 2 ? pair_f : 0) : n_rows;
      }
      k_in[i] = KC ? q % (FK / 4) * 4 : q / (ROWS / 4);
      voff[i] = row0 + row < n_rows ? (KC ? row * ld + k_in[i] : k_in[i] * ld + row) * 4 : (int)0x80000000;
    }
  }
  __device__ __forceinline__ void load(f32x4v (&r)[N4], int t) const {
    if constexpr (VEC) {
      const float* base = KC ? p + (size_t)row0 * ld + t * FK : p + (size_t)t * FK * ld + row0;
      const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7fffffff, 0x00020000);
      typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
      for (int i = 0; i < N4; ++i) {
        const int vo = t * FK + k_in[i] < K ? voff[i] : (int)0x80000000;
        r[i] = __builtin_bit_cast(f32x4v, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(rsrc, vo, 0, 0));
      }
    } else {
      Tile::load(r, p, ld, row0, n_rows, t * FK, K);
    }
  }
};

// Accumulator value r of a 32x32 block: row 8 (r / 4) + 4 (lane >> 5) + r % 4, column lane & 31: a store instruction
// writes 128 contiguous bytes of two rows.
// ACT: the activation of GemmArgs on the sum (SwiGLU forward needs two sums and is put by put_swiglu).  The formulas of the stand-alone kernels
// of elementwise.hip; what the fusion saves is their launch and the trip of the tensor through memory: an iteration of one layer, hidden 256,
// ffn 688, four microbatches of 128 tokens 437 -> 420 us; two layers, hidden 1024, ffn 2752, 1541 tokens 2802 -> 2775 us.
struct F32Out {
  float* C; const float* R; const float* bias; float* E;
  int ldc, ldr, lde;
};
__device__ __forceinline__ float sigmoid_f32(float z) { return 1.0f / (1.0f + __expf(-z)); }
// What the sum of row m, column n meets: the residual, or the saved tensor of an activation's backward (x; SwiGLU: gate x, up y).
template <int ACT>
__device__ __forceinline__ void get_operands(float& x, float& y, const F32Out& o, int m, int n, int N) {
  x = y = 0.f;
  if constexpr (ACT == ACT_GELU_BWD || ACT == ACT_SWIGLU_BWD) {
    x = o.E[(size_t)m * o.lde + n];
    if constexpr (ACT == ACT_SWIGLU_BWD) y = o.E[(size_t)m * o.lde + N + n];
  } else if (o.R) {
    x = o.R[(size_t)m * o.ldr + n];
  }
}
template <int ACT>
__device__ __forceinline__ void put_f32(float v, float x, float y, const F32Out& o, int m, int n, int N) {
  if (o.bias) v += o.bias[n];
  float* c = o.C + (size_t)m * o.ldc + n;
  if constexpr (ACT == ACT_GELU_FWD) {
    o.E[(size_t)m * o.lde + n] = 0.5f * v * (1.0f + erff(v * 0.70710678118654752f));
  } else if constexpr (ACT == ACT_GELU_BWD) {
    const float Phi = 0.5f * (1.0f + erff(x * 0.70710678118654752f)), phi = 0.39894228040143268f * __expf(-0.5f * x * x);
    v *= Phi + x * phi;
  } else if constexpr (ACT == ACT_SWIGLU_BWD) {
    const float sg = sigmoid_f32(x);
    c[N] = v * x * sg;
    v = v * y * sg * (1.0f + x * (1.0f - sg));
  } else {
    v += x;
  }
  *c = v;
}
// Row m, feature f of a SwiGLU forward of F features: the sums of its gate and up columns.
__device__ __forceinline__ void put_swiglu(float g, float up, const F32Out& o, int m, int f, int F) {
  if (o.bias) { g += o.bias[f]; up += o.bias[F + f]; }
  float* c = o.C + (size_t)m * o.ldc + f;
  c[0] = g;
  c[F] = up;
  o.E[(size_t)m * o.lde + f] = g * sigmoid_f32(g) * up;
}
// Column of C that column c of the tile at n0 stands for; SwiGLU forward: the first half of the tile is gate, the second the up columns of
// the same features (those past the last feature: the last one again).
template <int ACT, int EDGE>
__device__ __forceinline__ int f32_column(int n0, int c, int N) {
  if constexpr (ACT == ACT_SWIGLU_FWD) {
    const int F = N >> 1;
    return min((n0 >> 1) + c % (EDGE / 2), F - 1) + (c >= EDGE / 2 ? F : 0);
  }
  return min(n0 + c, N - 1);
}

// Tile of 64 x 64, eight wavefronts: two groups of 2 x 2 (32 x 32 of C each), each group contracting one half of every
// step's k; the groups' sums are added at the end, group 0 first.  Eight instead of four wavefronts because a grid of
// about one tile per CU would otherwise leave a single wavefront per SIMD to cover its own LDS reads and barriers.
constexpr int KG = 2, TILE_THREADS = 256 * KG;
template <bool TA, bool TB, bool VEC, int ACT = ACT_NONE>
__device__ __forceinline__ void f32_tile(const float* __restrict__ A, const float* __restrict__ B, const F32Out& out, int M, int N, int K,
                                         int lda, int ldb, int m0, int n0) {
  using TileA = F32Tile<!TA, 64, VEC, TILE_THREADS>;
  using TileB = F32Tile<TB, 64, VEC, TILE_THREADS>;
  constexpr int CHUNKS = FK / 8 / KG;                 // 8-deep k chunks of a step per wavefront
  constexpr int BUF = TileA::FLOATS + TileB::FLOATS;
  static_assert(3 * BUF >= 4 * 1024, "the second group's sums reuse the tile buffers");
  __shared__ __attribute__((aligned(16))) float pool[3 * BUF];
  const int lane = threadIdx.x & 63, wave = (threadIdx.x >> 6) & 3, group = threadIdx.x >> 8;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;

  // Three buffers: while step t is contracted, step t + 2 goes from registers to LDS and step t + 4 is requested from memory, and the first
  // fragments of step t + 1, complete since the barrier before, are read under the last MFMAs: what the step's one barrier waits for has
  // MFMAs running beside it, and the MFMAs behind it have their operands.  (1024 x 1024 x 1024: 24 us = 91 TFLOP/s.)
  f32x4v ra[2][TileA::N4], rb[2][TileB::N4];
  const int steps = (K + FK - 1) / FK;
  const F32Stream<!TA, 64, VEC, TILE_THREADS> sa(A, lda, m0, M, K);
  const F32Stream<TB, 64, VEC, TILE_THREADS> sb(B, ldb, n0, N, K, ACT == ACT_SWIGLU_FWD ? N >> 1 : 0);
  auto fetch = [&](int set, int t) {                   // a step past the end: zeros
    sa.load(ra[set], t);
    sb.load(rb[set], t);
  };
  auto put = [&](int set, int buf) {
    TileA::store(ra[set], pool + buf * BUF);
    TileB::store(rb[set], pool + buf * BUF + TileA::FLOATS);
  };
  static_assert(CHUNKS == 2, "two chunks of a step per wavefront");
  f32x4v fa[2], fb[2];
  auto frags = [&](int c8, int buf) {
    fa[c8] = TileA::frag(pool + buf * BUF, wm, group * CHUNKS + c8, lane);
    fb[c8] = TileB::frag(pool + buf * BUF + TileA::FLOATS, wn, group * CHUNKS + c8, lane);
  };
  auto multiply = [&](int c8) {
#pragma unroll
    for (int c = 0; c < 4; ++c) acc = mfma_f32(fa[c8][c], fb[c8][c], acc);
  };
  auto step = [&](int t, int set, int buf) {           // set = t % 2, buf = t % 3: constants at every call
    frags(1, buf);
    multiply(0);
    __builtin_amdgcn_sched_barrier(0);
    put(set, (buf + 2) % 3);
    fetch(set, t + 4);
    frags(0, (buf + 1) % 3);
    multiply(1);
    __builtin_amdgcn_sched_barrier(0);                 // the MFMAs stay on this side: they run while the reads and writes land
    __syncthreads();
  };
  fetch(0, 0);
  fetch(1, 1);
  put(0, 0);
  fetch(0, 2);
  put(1, 1);
  fetch(1, 3);
  __syncthreads();
  frags(0, 0);
  for (int t = 0;; t += 6) {
    step(t, 0, 0);
    if (t + 1 >= steps) break;
    step(t + 1, 1, 1);
    if (t + 2 >= steps) break;
    step(t + 2, 0, 2);
    if (t + 3 >= steps) break;
    step(t + 3, 1, 0);
    if (t + 4 >= steps) break;
    step(t + 4, 0, 1);
    if (t + 5 >= steps) break;
    step(t + 5, 1, 2);
    if (t + 6 >= steps) break;
  }
  // operands of the epilogue, requested together before the sums are exchanged (one by one each row would wait for its own)
  float x[16], y[16];
  auto row_of = [&](int r) { return m0 + wm + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3); };
  if (ACT != ACT_SWIGLU_FWD && group == 0)
#pragma unroll
    for (int r = 0; r < 16; ++r) get_operands<ACT>(x[r], y[r], out, min(row_of(r), M - 1), min(n0 + wn + (lane & 31), N - 1), N);
  if (group > 0)
#pragma unroll
    for (int e = 0; e < 16; ++e) pool[wave * 1024 + e * 64 + lane] = acc[e];
  __syncthreads();
  if (group == 0)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] += pool[wave * 1024 + r * 64 + lane];
  if constexpr (ACT == ACT_SWIGLU_FWD) {              // the up columns' wavefronts hand their sums to the gate columns'
    static_assert(3 * BUF >= (4 + 2) * 1024, "room for them");
    if (group == 0 && wn > 0)
#pragma unroll
      for (int e = 0; e < 16; ++e) pool[(4 + (wave >> 1)) * 1024 + e * 64 + lane] = acc[e];
    __syncthreads();
    if (wn > 0) return;
  }
  if (group > 0) return;
  const int n = ACT == ACT_SWIGLU_FWD ? (n0 >> 1) + (lane & 31) : n0 + wn + (lane & 31);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = row_of(r);
    if constexpr (ACT == ACT_SWIGLU_FWD) {
      if (m < M && n < (N >> 1)) put_swiglu(acc[r], pool[(4 + (wave >> 1)) * 1024 + r * 64 + lane], out, m, n, N >> 1);
    } else {
      if (m < M && n < N) put_f32<ACT>(acc[r], x[r], y[r], out, m, n, N);
    }
  }
}

constexpr int SMALL_WAVES = 8, SMALL_CHUNKS = 4;     // k ranges of a tile, one per wavefront; chunks of 8 k in flight together

// Fragment of 8 k at k0 for rows row0 .. row0+31 straight from memory (rows past the end repeat the last one: their
// results are never stored; k past the end reads as zero).
template <bool KC, bool VEC>
__device__ __forceinline__ f32x4v small_frag(const float* __restrict__ p, int ld, int row, int k, int K) {
  if constexpr (KC) return load4<VEC>(p + (size_t)row * ld + k, K - k);
  f32x4v v;
  v.x = k < K ? p[(size_t)k * ld + row] : 0.f;
  v.y = k + 1 < K ? p[(size_t)(k + 1) * ld + row] : 0.f;
  v.z = k + 2 < K ? p[(size_t)(k + 2) * ld + row] : 0.f;
  v.w = k + 3 < K ? p[(size_t)(k + 3) * ld + row] : 0.f;
  return v;
}

// The wavefronts' sums of a tile, [SMALL_WAVES][EDGE][EDGE], added in order and put.
template <int ACT, int EDGE>
__device__ __forceinline__ void put_sums(const float* red, const F32Out& out, int M, int N, int m0, int n0) {
  constexpr int W = ACT == ACT_SWIGLU_FWD ? EDGE / 2 : EDGE;          // values (features) per row
  for (int q = threadIdx.x; q < EDGE * W; q += 64 * SMALL_WAVES) {
    const int at = q / W * EDGE + q % W;
    float v = red[at], up = ACT == ACT_SWIGLU_FWD ? red[at + EDGE / 2] : 0.f;
#pragma unroll
    for (int w = 1; w < SMALL_WAVES; ++w) {
      v += red[w * EDGE * EDGE + at];
      if (ACT == ACT_SWIGLU_FWD) up += red[w * EDGE * EDGE + at + EDGE / 2];
    }
    const int m = m0 + q / W;
    if constexpr (ACT == ACT_SWIGLU_FWD) {
      const int f = (n0 >> 1) + q % W;
      if (m < M && f < (N >> 1)) put_swiglu(v, up, out, m, f, N >> 1);
    } else {
      const int n = n0 + q % W;
      float x, y;
      if (m < M && n < N) {
        get_operands<ACT>(x, y, out, m, n, N);
        put_f32<ACT>(v, x, y, out, m, n, N);
      }
    }
  }
}

template <bool TA, bool TB, bool VEC, int ACT = ACT_NONE>
__device__ __forceinline__ void f32_small(const float* __restrict__ A, const float* __restrict__ B, const F32Out& out, int M, int N, int K,
                                          int lda, int ldb, int m0, int n0) {
  __shared__ float red[SMALL_WAVES][32 * 32];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m = min(m0 + (lane & 31), M - 1), n = f32_column<ACT, 32>(n0, lane & 31, N);
  const int chunks = (K + 7) / 8, per = (chunks + SMALL_WAVES - 1) / SMALL_WAVES;
  const int k_end = min(K, (wave + 1) * per * 8);
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  f32x4v fa[2][SMALL_CHUNKS], fb[2][SMALL_CHUNKS];
  auto fetch = [&](f32x4v (&a)[SMALL_CHUNKS], f32x4v (&b)[SMALL_CHUNKS], int k0) {
#pragma unroll
    for (int c = 0; c < SMALL_CHUNKS; ++c) {
      const int k = k0 + c * 8 + (lane >> 5) * 4;
      a[c] = small_frag<!TA, VEC>(A, lda, m, k, k_end);
      b[c] = small_frag<TB, VEC>(B, ldb, n, k, k_end);
    }
  };
  auto multiply = [&](const f32x4v (&a)[SMALL_CHUNKS], const f32x4v (&b)[SMALL_CHUNKS]) {
#pragma unroll
    for (int c = 0; c < SMALL_CHUNKS; ++c) {
      acc = mfma_f32(a[c].x, b[c].x, acc);
      acc = mfma_f32(a[c].y, b[c].y, acc);
      acc = mfma_f32(a[c].z, b[c].z, acc);
      acc = mfma_f32(a[c].w, b[c].w, acc);
    }
  };
  constexpr int KB = SMALL_CHUNKS * 8;
  int k0 = wave * per * 8;
  if (k0 < k_end) {
    fetch(fa[0], fb[0], k0);
    for (; k0 < k_end; k0 += 2 * KB) {
      if (k0 + KB < k_end) fetch(fa[1], fb[1], k0 + KB);
      multiply(fa[0], fb[0]);
      if (k0 + KB < k_end) {
        if (k0 + 2 * KB < k_end) fetch(fa[0], fb[0], k0 + 2 * KB);
        multiply(fa[1], fb[1]);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) red[wave][((r >> 2) * 8 + (lane >> 5) * 4 + (r & 3)) * 32 + (lane & 31)] = acc[r];
  __syncthreads();
  put_sums<ACT, 32>(&red[0][0], out, M, N, m0, n0);
}

// Tiles of 16 x 16 on v_mfma_f32_16x16x4_f32, otherwise as f32_small: four times the workgroups for the smallest outputs.  In a
// chunk of 16 k lane l holds row l & 15 and k = 4 (l >> 4) + i for the i-th of four MFMAs.
constexpr int TINY = 16, TINY_CHUNKS = 4;
__device__ __forceinline__ f32x4v mfma_f32_16(float a, float b, f32x4v c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
template <bool TA, bool TB, bool VEC, int ACT = ACT_NONE>
__device__ __forceinline__ void f32_tiny(const float* __restrict__ A, const float* __restrict__ B, const F32Out& out, int M, int N, int K,
                                         int lda, int ldb, int m0, int n0) {
  __shared__ float red[SMALL_WAVES][TINY * TINY];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m = min(m0 + (lane & 15), M - 1), n = f32_column<ACT, TINY>(n0, lane & 15, N);
  const int chunks = (K + 15) / 16, per = (chunks + SMALL_WAVES - 1) / SMALL_WAVES;
  const int k_end = min(K, (wave + 1) * per * 16);
  f32x4v acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  f32x4v fa[2][TINY_CHUNKS], fb[2][TINY_CHUNKS];
  auto fetch = [&](f32x4v (&a)[TINY_CHUNKS], f32x4v (&b)[TINY_CHUNKS], int k0) {
#pragma unroll
    for (int c = 0; c < TINY_CHUNKS; ++c) {
      const int k = k0 + c * 16 + (lane >> 4) * 4;
      a[c] = small_frag<!TA, VEC>(A, lda, m, k, k_end);
      b[c] = small_frag<TB, VEC>(B, ldb, n, k, k_end);
    }
  };
  auto multiply = [&](const f32x4v (&a)[TINY_CHUNKS], const f32x4v (&b)[TINY_CHUNKS]) {
#pragma unroll
    for (int c = 0; c < TINY_CHUNKS; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[c & 1] = mfma_f32_16(a[c][i], b[c][i], acc[c & 1]);
  };
  constexpr int KB = TINY_CHUNKS * 16;
  int k0 = wave * per * 16;
  if (k0 < k_end) {
    fetch(fa[0], fb[0], k0);
    for (; k0 < k_end; k0 += 2 * KB) {
      if (k0 + KB < k_end) fetch(fa[1], fb[1], k0 + KB);
      multiply(fa[0], fb[0]);
      if (k0 + KB < k_end) {
        if (k0 + 2 * KB < k_end) fetch(fa[0], fb[0], k0 + 2 * KB);
        multiply(fa[1], fb[1]);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) red[wave][((lane >> 4) * 4 + r) * TINY + (lane & 15)] = acc[0][r] + acc[1][r];
  __syncthreads();
  put_sums<ACT, TINY>(&red[0][0], out, M, N, m0, n0);
}

template <bool TA, bool TB, bool VEC, int EDGE, int ACT>
__global__ __launch_bounds__(EDGE < 64 ? 64 * SMALL_WAVES : TILE_THREADS) void gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ B,
                                                                                         const F32Out out, int M, int N, int K, int lda, int ldb) {
  const int m0 = blockIdx.y * EDGE, n0 = blockIdx.x * EDGE;
  if constexpr (EDGE == TINY) f32_tiny<TA, TB, VEC, ACT>(A, B, out, M, N, K, lda, ldb, m0, n0);
  else if constexpr (EDGE == 32) f32_small<TA, TB, VEC, ACT>(A, B, out, M, N, K, lda, ldb, m0, n0);
  else f32_tile<TA, TB, VEC, ACT>(A, B, out, M, N, K, lda, ldb, m0, n0);
}

// Weight gradients of a whole task in one launch: the products are independent (A stored [K, M], B [K, N]), and a small
// stage's are a few tiles each, so launched one by one they leave most of the chip idle and cost a launch each.  One iteration of
// a 2-layer hidden-128 stage 667 -> 619 us, of a 2-layer hidden-1024 one 3615 -> 3475 us.
constexpr int F32_GROUP_MAX = 32;
struct F32Problem {
  const float *A, *B;
  float* C;
  int M, N, lda, ldb, ldc, tiles_n;
};
struct F32Group {
  int start[F32_GROUP_MAX];                            // index of each product's first tile; INT_MAX past the last product
  F32Problem p[F32_GROUP_MAX];
  int K;
};
template <bool VEC, bool SMALL>
__global__ __launch_bounds__(SMALL ? 64 * SMALL_WAVES : TILE_THREADS) void gemm_f32_group_kernel(const F32Group g) {
  constexpr int EDGE = SMALL ? 32 : 64;
  static_assert(F32_GROUP_MAX <= 64, "a lane per product");
  const int lane = threadIdx.x & 63;                   // all starts at once: a walk is a chain of loads from host memory
  const int i = __builtin_amdgcn_readfirstlane(__popcll(__ballot(lane < F32_GROUP_MAX && g.start[lane] <= (int)blockIdx.x)) - 1);
  const F32Problem& p = g.p[i];
  const int t = blockIdx.x - g.start[i], m0 = t / p.tiles_n * EDGE, n0 = t % p.tiles_n * EDGE;
  const F32Out out{p.C, nullptr, nullptr, nullptr, p.ldc, 0, 0};
  if constexpr (SMALL) f32_small<true, false, VEC>(p.A, p.B, out, p.M, p.N, g.K, p.lda, p.ldb, m0, n0);
  else f32_tile<true, false, VEC>(p.A, p.B, out, p.M, p.N, g.K, p.lda, p.ldb, m0, n0);
}

// Which kernel (us, 32 x 32 against 64 x 64 tiles): up to 64 tiles of 64 x 64 the small kernel's fill one round and win clearly (256 x 1024 x 1024
// 12.7 / 21.6, x 4096 37.6 / 74.7); from there to 127 they win where K is short (448 x 1024 x 256 7.0 / 8.6), tie at K = 1024 (22.0 / 21.6) and lose
// at longer K over a K-strided B (x 2752 57 / 50); from 128 they need three rounds.
// Sixteen k ranges instead of eight change nothing: the operand rows then bound it through the L1.
// So below 97 tiles of 32 x 32 the tiles are 16 x 16, which spreads those rows over four times the CUs (us, 32 -> 16): 128 x 256 x 1376 15.3 ->
// 7.5, x 256 4.4 -> 3.2, 32 x 1024 x 2752 28.9 -> 12.7, 128 x 768 x 256 (96 tiles) 4.5 -> 4.4; but 128 x 1376 x 256 (172 tiles) 4.9 -> 6.5.
int f32_tile_edge(int M, int N) {
  auto tiles = [&](int edge) { return (long long)((M + edge - 1) / edge) * ((N + edge - 1) / edge); };
  return tiles(64) >= 128 ? 64 : tiles(32) > 96 ? 32 : TINY;
}

template <bool TA, bool TB, bool VEC, int ACT = ACT_NONE>
hipError_t launch_f32(const GemmArgs& g, hipStream_t s) {
  const F32Out out{(float*)g.C, g.R, (const float*)g.bias, (float*)g.E, g.ldc, g.ldr, g.lde};
  const int t = f32_tile_edge(g.M, g.N);
  const int columns = ACT == ACT_SWIGLU_FWD ? (g.N / 2 + t / 2 - 1) / (t / 2) : (g.N + t - 1) / t;
  const dim3 grid(columns, (g.M + t - 1) / t);
#define RRFP_GO(EDGE, THREADS) \
  hipLaunchKernelGGL((gemm_f32_kernel<TA, TB, VEC, EDGE, ACT>), grid, dim3(THREADS), 0, s, (const float*)g.A, (const float*)g.B, out, g.M, g.N, g.K, g.lda, g.ldb)
  if (t == 64) RRFP_GO(64, TILE_THREADS);
  else if (t == 32) RRFP_GO(32, 64 * SMALL_WAVES);
  else RRFP_GO(TINY, 64 * SMALL_WAVES);
#undef RRFP_GO
  return hipGetLastError();
}

// 16-byte loads need aligned rows and a contiguous extent of whole float4s (M or N when K-strided, K when K-contiguous)
bool vec_ok(const GemmArgs& g) {
  return g.lda < VEC_MAX_LD && g.ldb < VEC_MAX_LD && !((g.lda | g.ldb) & 3) && !((uintptr_t)g.A & 15) && !((uintptr_t)g.B & 15) && !((g.transA ? g.M : g.K) & 3) &&
         !((g.transB ? g.K : g.N) & 3);
}
template <bool TA, bool TB>
hipError_t launch_f32_aligned(const GemmArgs& g, hipStream_t s) {
  return vec_ok(g) ? launch_f32<TA, TB, true>(g, s) : launch_f32<TA, TB, false>(g, s);
}

// 64 x 64 tiles from 128 of them in the whole group on, else 32 x 32: f32_tile_edge without its 16 x 16 tiles, which no group has been built with.
hipError_t launch_f32_group(const GemmArgs* g, int n, hipStream_t s) {
  F32Group grp{};
  grp.K = g[0].K;
  for (int i = n; i < F32_GROUP_MAX; ++i) grp.start[i] = INT_MAX;
  bool vec = true;
  auto tiles = [&](int edge) {
    int t = 0;
    for (int i = 0; i < n; ++i) {
      const int tn = (g[i].N + edge - 1) / edge;
      grp.p[i] = F32Problem{(const float*)g[i].A, (const float*)g[i].B, (float*)g[i].C, g[i].M, g[i].N, g[i].lda, g[i].ldb, g[i].ldc, tn};
      grp.start[i] = t;
      t += (g[i].M + edge - 1) / edge * tn;
    }
    return t;
  };
  for (int i = 0; i < n; ++i) vec = vec && vec_ok(g[i]);
  int t = tiles(64);
  const bool small = t < 128;
  if (small) t = tiles(32);
#define RRFP_GO(VEC, SMALL, THREADS) hipLaunchKernelGGL((gemm_f32_group_kernel<VEC, SMALL>), dim3(t), dim3(THREADS), 0, s, grp)
  if (vec && small) RRFP_GO(true, true, 64 * SMALL_WAVES);
  else if (vec) RRFP_GO(true, false, TILE_THREADS);
  else if (small) RRFP_GO(false, true, 64 * SMALL_WAVES);
  else RRFP_GO(false, false, TILE_THREADS);
#undef RRFP_GO
  return hipGetLastError();
}

}  // namespace

bool gemm_f32_act_supported(const GemmArgs& g) {
  if (g.in_dtype != F32 || g.out_dtype != F32 || g.transA || g.R || !g.E || !vec_ok(g)) return false;
  switch (g.act) {
    case ACT_SWIGLU_FWD: return !g.transB && g.N % 8 == 0;              // the vectors of B's columns lie in one half
    case ACT_GELU_FWD: return !g.transB;
    case ACT_SWIGLU_BWD: case ACT_GELU_BWD: return g.transB;
    default: return false;
  }
}

hipError_t launch_gemm_f32(const GemmArgs& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.K <= 0 || g.in_dtype != F32 || g.out_dtype != F32) return hipErrorInvalidValue;
  if (g.act != ACT_NONE) {
    if (!gemm_f32_act_supported(g)) return hipErrorInvalidValue;
    switch (g.act) {
      case ACT_SWIGLU_FWD: return launch_f32<false, false, true, ACT_SWIGLU_FWD>(g, s);
      case ACT_GELU_FWD: return launch_f32<false, false, true, ACT_GELU_FWD>(g, s);
      case ACT_SWIGLU_BWD: return launch_f32<false, true, true, ACT_SWIGLU_BWD>(g, s);
      default: return launch_f32<false, true, true, ACT_GELU_BWD>(g, s);
    }
  }
  if (!g.transA && !g.transB) return launch_f32_aligned<false, false>(g, s);
  if (!g.transA) return launch_f32_aligned<false, true>(g, s);
  if (!g.transB) return launch_f32_aligned<true, false>(g, s);
  return launch_f32_aligned<true, true>(g, s);
}

bool gemm_f32_groupable(const GemmArgs& g) {
  return g.transA && !g.transB && !g.R && !g.bias && g.act == ACT_NONE && g.in_dtype == F32 && g.out_dtype == F32 && g.M > 0 && g.N > 0 && g.K > 0 &&
         (long long)((g.M + 31) / 32) * ((g.N + 31) / 32) < (1 << 24);
}

hipError_t launch_gemm_f32_group(const GemmArgs* g, int n, hipStream_t s) {
  for (int i = 0; i < n; i += F32_GROUP_MAX)
    if (hipError_t e = launch_f32_group(g + i, std::min(F32_GROUP_MAX, n - i), s); e != hipSuccess) return e;
  return hipSuccess;
}

}  // namespace rrfp
