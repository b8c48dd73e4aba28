// bf16 MFMA GEMM for gfx950: C[M,N] = A(m,k) B(k,n) (+R), fp32 accumulation, bf16 or fp32 out.
//
// Two kernels share the tile geometry (a workgroup owns a 256-wide tile of C); a third takes small outputs:
//
//   gemm_mfma_dl_kernel  the main kernel.  8 wavefronts (2 x 4, 128 x 64 of C each), accumulators of
//     v_mfma_f32_16x16x32_bf16.  K advances in 32-deep steps through a ring of five LDS buffers that
//     are filled by direct global->LDS loads, issued for pairs of steps (so that both 64-byte halves of
//     a 128-byte line of a K-contiguous operand reach L2 as one request) and spread between the MFMAs;
//     epilogue staged through LDS so that all stores, residual loads and activation-operand loads are
//     row-contiguous; optional fused residual / bias / SwiGLU / GELU forward and backward epilogues; a
//     128-row tile variant and a split-K mode for grids that do not fill the CUs.
//   gemm_mfma_kernel     the fallback for K-contiguous operands whose K is not a multiple of 32: four
//     wavefronts, v_mfma_f32_32x32x16_bf16, 64-deep steps, two LDS stages filled through registers.
//   gemm_mfma_small_kernel  64 x 64 or 32 x 32 tiles, the contraction dealt to the wavefronts of a workgroup.
//
// Operand tiles sit in LDS in their memory orientation, so every global load is a coalesced
// 16-byte access:
//   K-contiguous operand ([rows][K] in memory): rows of 16-byte chunks, XOR-swizzled so that the lanes
//     one ds_read_b128 pass serves fall into distinct bank groups; a fragment (8 consecutive k of one
//     row) is one ds_read_b128.
//   K-strided operand ([K][rows] in memory): LDS [k][256 rows], chunks XOR-swizzled by k; a fragment is
//     two ds_read_b64_tr_b16, the LDS transpose read of gfx950 that hands each lane 4 consecutive k of
//     one row out of a 4(k) x 16(rows) block.
// The forward GEMMs use (A K-contiguous, B K-strided), the input-gradient GEMMs (both
// K-contiguous), the weight-gradient GEMMs (both K-strided, K = tokens).
//
// The MFMA is issued with the B fragment as its first operand, so a lane's four consecutive
// accumulator values are four consecutive columns of one row of C.  Rows beyond M, columns beyond N
// and k beyond K are zero-filled on load and masked on store.  The k loop order, the tile partition,
// the choice of 128-row tiles and the split-K factor depend only on the shape and on the device's CU
// count, never on what else is running, so a given call always sums in the same order.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "kernels.h"
#include "numeric.h"

namespace rrfp {
namespace {

constexpr int BM = 256, BN = 256, BK = 64, NTHREADS = 256;
constexpr int TILE_BYTES = 256 * 64 * 2;          // one operand tile
constexpr int STAGE_BYTES = 2 * TILE_BYTES;       // A + B
constexpr int SMEM_BYTES = 2 * STAGE_BYTES;       // two stages

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4v* lds_short4_ptr;

// Byte offset of the 16-byte chunk (row, c) of a K-contiguous tile [256][64].
__device__ __forceinline__ int kc_off(int row, int c) { return row * 128 + ((c ^ ((row >> 1) & 7)) << 4); }
// Byte offset of the 16-byte chunk (k, c) of a K-strided tile [64][256]; c in 0..31.
__device__ __forceinline__ int ks_off(int k, int c) {
  const int f = (k & 3) | (((k >> 3) & 1) << 2);
  return k * 512 + (((((c >> 2) ^ f) << 2) | (c & 3)) << 4);
}

// Global -> registers for one operand tile: 8 chunks of 16 bytes per thread.
template <bool KC>
__device__ __forceinline__ void load_tile(uint4 (&r)[8], const bf16_t* __restrict__ base, int ld, int outer0,
                                          int outer_n, int k0, int K) {
  const int t = threadIdx.x;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int q = i * NTHREADS + t;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (KC) {
      const int row = q >> 3, c = q & 7;
      const int go = outer0 + row, gk = k0 + c * 8;
      if (go < outer_n && gk < K) v = *reinterpret_cast<const uint4*>(base + (size_t)go * ld + gk);
    } else {
      const int k = q >> 5, c = q & 31;
      const int gk = k0 + k, go = outer0 + c * 8;
      if (gk < K && go < outer_n) v = *reinterpret_cast<const uint4*>(base + (size_t)gk * ld + go);
    }
    r[i] = v;
  }
}

template <bool KC>
__device__ __forceinline__ void store_tile(const uint4 (&r)[8], char* tile) {
  const int t = threadIdx.x;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int q = i * NTHREADS + t;
    const int off = KC ? kc_off(q >> 3, q & 7) : ks_off(q >> 5, q & 31);
    *reinterpret_cast<uint4*>(tile + off) = r[i];
  }
}

// Fragment of 32 rows starting at row0 (multiple of 32), k-step ks (16 k): lane l gets row
// row0 + (l & 31), k = ks*16 + (l >> 5)*8 + 0..7.
template <bool KC>
__device__ __forceinline__ bf16x8 read_frag(const char* tile, int row0, int ks, int lane) {
  if (KC) {
    const int row = row0 + (lane & 31);
    const uint4 v = *reinterpret_cast<const uint4*>(tile + kc_off(row, ks * 2 + (lane >> 5)));
    return __builtin_bit_cast(bf16x8, v);
  } else {
    const int kb = ks * 16 + (lane >> 5) * 8 + ((lane & 15) >> 2);
    const int c = (row0 >> 3) + ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1);
    const int sub = (lane & 1) * 8;
    union { short4v h[2]; bf16x8 v; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(tile + ks_off(kb, c) + sub));
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(tile + ks_off(kb + 4, c) + sub));
    return u.v;
  }
}

// Output tile index from the hardware workgroup id.  Workgroups are dealt round-robin to the
// 8 XCDs, each with its own L2; give every XCD a contiguous run of tiles, and order tiles in
// groups of 8 tile-rows so that the tiles resident on an XCD together share A and B panels.
__device__ __forceinline__ void tile_coords(int b, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int nt = tiles_m * tiles_n;
  const int q = nt >> 3, r = nt & 7, xcd = b & 7, i = b >> 3;
  const int pid = xcd < r ? xcd * (q + 1) + i : r * (q + 1) + (xcd - r) * q + i;
  constexpr int GM = 8;
  const int per_group = GM * tiles_n;
  const int g = pid / per_group;
  const int first_m = g * GM;
  const int gsize = min(tiles_m - first_m, GM);
  const int in_g = pid - g * per_group;
  tm = first_m + in_g % gsize;
  tn = in_g / gsize;
}

template <bool A_KC, bool B_KC, typename TO, bool HAS_R>
__global__ __launch_bounds__(NTHREADS) void gemm_mfma_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B,
                                                             TO* __restrict__ C, const float* __restrict__ R, int M,
                                                             int N, int K, int lda, int ldb, int ldc, int ldr,
                                                             int tiles_m, int tiles_n) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int tm, tn;
  tile_coords(blockIdx.x, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = (wave >> 1) * 128, wn = (wave & 1) * 128;

  floatx16 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  uint4 ra[8], rb[8];
  const int nk = (K + BK - 1) / BK;
  load_tile<A_KC>(ra, A, lda, m0, M, 0, K);
  load_tile<B_KC>(rb, B, ldb, n0, N, 0, K);
  store_tile<A_KC>(ra, smem);
  store_tile<B_KC>(rb, smem + TILE_BYTES);
  __syncthreads();

  for (int kt = 0; kt < nk; ++kt) {
    const char* sa = smem + (kt & 1) * STAGE_BYTES;
    const char* sb = sa + TILE_BYTES;
    const bool more = kt + 1 < nk;
    if (more) {
      load_tile<A_KC>(ra, A, lda, m0, M, (kt + 1) * BK, K);
      load_tile<B_KC>(rb, B, ldb, n0, N, (kt + 1) * BK, K);
    }
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      bf16x8 fa[4], fb[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) fa[i] = read_frag<A_KC>(sa, wm + i * 32, ks, lane);
#pragma unroll
      for (int j = 0; j < 4; ++j) fb[j] = read_frag<B_KC>(sb, wn + j * 32, ks, lane);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
    if (more) {
      char* na = smem + ((kt + 1) & 1) * STAGE_BYTES;
      store_tile<A_KC>(ra, na);
      store_tile<B_KC>(rb, na + TILE_BYTES);
    }
    __syncthreads();
  }

  // Epilogue.  acc[i][j][g*4 + e] = C[m0 + wm + i*32 + (lane & 31)][n0 + wn + j*32 + g*8 + (lane >> 5)*4 + e].
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + wm + i * 32 + (lane & 31);
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int n = n0 + wn + j * 32 + g * 8 + (lane >> 5) * 4;
        if (n >= N) continue;     // N is a multiple of 8: the four columns are in or out together
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[i][j][g * 4 + e];
        if (HAS_R) {
          const float4 rr = *reinterpret_cast<const float4*>(R + (size_t)m * ldr + n);
          v[0] += rr.x; v[1] += rr.y; v[2] += rr.z; v[3] += rr.w;
        }
        if (sizeof(TO) == 4) {
          *reinterpret_cast<float4*>((float*)C + (size_t)m * ldc + n) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
          uint2 o;
          o.x = pack_bf16x2(v[0], v[1]);
          o.y = pack_bf16x2(v[2], v[3]);
          *reinterpret_cast<uint2*>((bf16_t*)C + (size_t)m * ldc + n) = o;
        }
      }
    }
  }
}


// ------------------------------------------------------------------------------------------
// Direct-to-LDS variant (the one the stage tasks run).
//   - global -> LDS copies are buffer_load ... lds instructions, 16 bytes per lane, which land
//     in LDS at base + lane * 16 without passing through registers.  The XOR swizzles of the
//     tile layouts are therefore applied on the GLOBAL side: lane p of a 1 KB block fetches the
//     chunk that belongs at LDS position p.
//   - buffer descriptors bound every operand, so rows past the end of an operand read as zero
//     (that is what zero-fills the ragged K tail of the weight-gradient GEMMs, K = tokens).
//   - K advances in steps of 32 through FIVE LDS buffers of 32 KB (all of the CU's LDS); the loads of
//     steps e and e+1 are issued together, three to four steps ahead of their use.  The buffers are
//     five separate __shared__ arrays and the loop is unrolled by ten, so the compiler can prove that
//     fragment reads of one buffer do not alias loads in flight to another.
// Requires K % 32 == 0 when an operand is K-contiguous (a K tail would wrap into the next row).
// ------------------------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void* lds_void_ptr;

// Wavefronts per workgroup of the direct-load kernel.  With a K-contiguous operand: 2 x 4 (128 x 64 of C
// each, two per SIMD so that one wavefront's waits hide behind the other's MFMAs), v_mfma_f32_16x16x32_bf16.
// With both operands K-strided (the weight-gradient form) the kernel is bounded by the issue rate of the
// LDS transpose reads, two per fragment: 2 x 2 wavefronts (128 x 128 each) need a third fewer of them.
// 256 accumulator registers per wavefront only allocate cleanly as 16 tuples of 16 (with 64 tuples of 4
// the register allocator shuffles accumulators between MFMAs), so that form keeps v_mfma_f32_32x32x16_bf16;
// it is not power bound, so the cheaper 16x16x32 form would buy nothing there.
constexpr int dl_wm(bool, bool) { return 2; }
constexpr int dl_wn(bool a_kc, bool b_kc) { return (a_kc || b_kc) ? 4 : 2; }
constexpr bool dl_m32(bool a_kc, bool b_kc) { return !a_kc && !b_kc; }
constexpr int DBK = 32;                              // k per stage
constexpr int DTILE = 256 * DBK * 2;                 // bytes of one operand tile (16 KB)
constexpr int DSTAGE = 2 * DTILE;                    // A + B (32 KB)

// K-contiguous tile [256 rows][32 k]: 64-byte rows, 4 chunks; chunk c of row r sits at c ^ s(r), with
// s = 0, 2, 3, 1 for (r >> 2) & 3 = 0, 1, 2, 3.  LDS serves 256 bytes per clock (64 banks), 16 lanes of a
// ds_read_b128 at a time, and those 16 lanes are not consecutive: measured (a probe that times the
// read for lane -> address tables, and the bank-conflict counter), the four passes take lanes
// {0-3, 12-15, 20-23, 24-27}, {32-35, 44-47, 52-55, 56-59}, {4-7, 8-11, 16-19, 28-31} and
// {36-39, 40-43, 48-51, 60-63}.  A fragment read has lane l at row (l & 15), chunk l >> 4, so one pass
// holds the row quads and chunks (0, c), (3, c), (1, c + 1), (2, c + 1); rows that differ in bits 0..1
// fall into different 64-byte windows of the 256, and s(r) sends the four quads of a pass to four
// different 16-byte slots.
__device__ __forceinline__ int dkc_swz(int row) {
  const int q = (row >> 2) & 3;
  return ((q & 1) << 1) ^ ((q >> 1) * 3);
}
__device__ __forceinline__ int dkc_off(int row, int c) { return row * 64 + ((c ^ dkc_swz(row)) << 4); }

// K-strided tile [32 k][256 rows]: 512-byte rows of 32 chunks; chunk c of row k sits at c ^ dks_swz(k).
// A fragment read (below) touches, per 32 lanes, 8 k-rows (k & 3 and bit 3 of k vary) at the same pair of
// chunks; the swizzle sends them to 8 distinct 32-byte bank groups.
__device__ __forceinline__ int dks_swz(int k) { return ((k & 3) | (((k >> 3) & 1) << 2)) << 1; }

// NW = wavefronts per workgroup.
// SWZ32 (K-strided tiles only): the swizzle of the 32x32x16 fragment reads (64-byte units moved by k,
// as in ks_off) instead of the one of the 16x16x32 reads.
template <bool KC, int NW, int ROWS = 256, bool SWZ32 = false>
struct DirectLoader {
  static_assert(KC || ROWS == 256, "a K-strided tile is always 256 wide");
  static constexpr int NL = (ROWS / 16) / NW;      // 1 KB blocks of the tile per wavefront (16 rows of 64 B each when K-contiguous)
  static_assert(NL >= 1, "tile too small for this many wavefronts");
  __amdgpu_buffer_rsrc_t rsrc;
  int voff[NL];
  int k_stride;     // bytes per k-step
  // pair_f > 0 (K-strided operand only): the 256 tile columns are 4 groups of [32 "gate" columns
  // f .. f+31 | 32 "up" columns pair_f + f .. pair_f + f+31], f = outer0/2 + 32 * group, so that one
  // wavefront holds gate and up of the same 32 features.
  __device__ __forceinline__ void init(const bf16_t* base, int ld, int outer0, int outer_n, int K, int wave, int lane,
                                       int pair_f = 0) {
    const size_t bytes = KC ? ((size_t)(outer_n - 1) * ld + K) * 2 : ((size_t)(K - 1) * ld + outer_n) * 2;
    rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)bytes, 0x00020000);
    k_stride = KC ? DBK * 2 : DBK * ld * 2;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int blk = i * NW + wave;                 // 1 KB block of the 16 KB tile
      if (KC) {
        const int row = blk * 16 + (lane >> 2), c = (lane & 3) ^ dkc_swz(row);
        voff[i] = (outer0 + row < outer_n) ? ((outer0 + row) * ld + c * 8) * 2 : (int)0x80000000;
      } else {
        const int k = blk * 2 + (lane >> 5), cp = lane & 31;
        const int f = (k & 3) | (((k >> 3) & 1) << 2);
        const int c = SWZ32 ? ((((cp >> 2) ^ f) << 2) | (cp & 3)) : (cp ^ dks_swz(k));
        int col = outer0 + c * 8;
        if (pair_f > 0) {
          const int nl = c * 8;                                  // column inside the tile
          col = ((nl >> 5) & 1) * pair_f + (outer0 >> 1) + (nl >> 6) * 32 + (nl & 31);
        }
        voff[i] = (k * ld + col) * 2;
      }
    }
  }
  // Load instruction i (of NL) of this wavefront for the k-step whose byte offset is soff.
  // exists == false: every lane gets the per-lane offset that is past any buffer (the same marker rows
  // past the end of the operand carry), so the descriptor's range check turns the load into zeros.
  __device__ __forceinline__ void issue_one(char* tile, int i, int soff, int wave, bool exists) const {
    const int vo = exists ? voff[i] : (int)0x80000000;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(tile + (i * NW + wave) * 1024), 16, vo, soff, 0, 0);
  }
};

// One quarter (Q = 0..3) of the loads of a pair of consecutive k-steps (e, e+1), e even: step e goes to
// bufE, step e+1 to bufO.  A wavefront's LA + LB load instructions per step are dealt to the quarters in
// order (A first); the two instructions that fetch the same rows for the two steps are issued back to
// back.  For a K-contiguous operand they are the two 64-byte halves of the same 128-byte lines: issued
// together they reach L2 as one request per line, issued a step apart (as two separate fetches) as two.
// Steps at or beyond nk are issued with a per-lane offset past every buffer (2^31; operands are smaller),
// which the descriptor turns into a load of zeros without a memory access: the number of loads in flight
// never depends on the position in K.
template <int Q, int LA, int LB>
struct QuarterCount { static constexpr int PAIRS = (Q + 1) * (LA + LB) / 4 - Q * (LA + LB) / 4, LOADS = 2 * PAIRS; };
template <int Q, bool GUARD, typename LoaderA, typename LoaderB>
__device__ __forceinline__ void issue_quarter(const LoaderA& la, const LoaderB& lb, char* bufE, char* bufO, int e, int nk, int wave) {
  constexpr int LA = LoaderA::NL, LB = LoaderB::NL;
  constexpr int P0 = Q * (LA + LB) / 4, P1 = (Q + 1) * (LA + LB) / 4;
  if constexpr (P1 > P0) {
    const bool okE = !GUARD || e < nk, okO = !GUARD || e + 1 < nk;
    const int aE = okE ? e * la.k_stride : 0, aO = okO ? (e + 1) * la.k_stride : 0;
    const int bE = okE ? e * lb.k_stride : 0, bO = okO ? (e + 1) * lb.k_stride : 0;
#pragma unroll
    for (int p = P0; p < P1; ++p) {
      if (p < LA) {
        la.issue_one(bufE, p, aE, wave, okE);
        la.issue_one(bufO, p, aO, wave, okO);
      } else {
        lb.issue_one(bufE + DTILE, p - LA, bE, wave, okE);
        lb.issue_one(bufO + DTILE, p - LA, bO, wave, okO);
      }
    }
  }
}

// Fragments of v_mfma_f32_16x16x32_bf16 for a 16-row block and the 32 k of one stage: lane l gets row
// (l & 15) of the block, k = (l >> 4) * 8 + 0..7.
//   K-contiguous: one ds_read_b128 at dkc_off(row, l >> 4); blocks are 1024 bytes apart.
//   K-strided: two ds_read_b64_tr_b16 (k-rows kb and kb + 4, same swizzle); in each, the 16 lanes of a
//     group address a 4 (k) x 16 (rows) block (lane -> k-row (l & 15) >> 2, rows 4 * (l & 3) .. + 3) and
//     receive 4 consecutive k of row l & 15.  Block i of the wavefront sits at chunk (cw | 2i | cl),
//     cw = 16-aligned chunk of the wavefront's first row, cl = (l & 3) >> 1, and the swizzle XORs bits
//     1..3 of the chunk, so the byte offset of block i is lane_part ^ (i << 5): one XOR per block.
typedef __attribute__((address_space(3))) const char* lds_char_ptr;

// Per-lane part of the fragment address of this wavefront's blocks starting at row w0.
template <bool KC>
__device__ __forceinline__ int frag_lane_offset(int w0, int lane) {
  if (KC) return dkc_off(w0 + (lane & 15), lane >> 4);
  const int kb = (lane >> 4) * 8 + ((lane & 15) >> 2);
  return kb * 512 + (lane & 1) * 8 + ((((w0 >> 3) | ((lane & 3) >> 1)) ^ dks_swz(kb)) << 4);
}

template <bool KC, int N>
__device__ __forceinline__ void load_blocks(bf16x8 (&f)[N], const char* tile, int lane_off) {
  if (!KC) asm volatile("" : "+v"(lane_off));   // keeps the per-block addresses from being hoisted out of the k loop (register pressure)
  const lds_char_ptr t = (lds_char_ptr)tile;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (KC) {
      f[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const __attribute__((address_space(3))) uint4*>(t + lane_off + i * 1024));
    } else {
      const int o = lane_off ^ (i << 5);
      union { short4v h[2]; bf16x8 v; } u;
      u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(t + o));
      u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(t + o + 2048));
      f[i] = u.v;
    }
  }
}

// Workgroup barrier between pipeline steps.  The caller has already waited (s_waitcnt vmcnt) for its
// own direct loads of the stage that is read next; a plain s_barrier then makes every wavefront's
// share of that stage visible.  No fence: a release fence would make the compiler drain ALL loads
// in flight, including those of the stages two and three steps ahead.  The empty asm statements
// keep the compiler from moving LDS accesses across the barrier.
__device__ __forceinline__ void stage_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}

// Fragments of one 32-deep step for v_mfma_f32_16x16x32_bf16: the wavefront's 16-row blocks of A in two
// halves (lo, hi: MA blocks each) and its NF 16-column blocks of B, the latter double-buffered by step parity.
template <int MA, int NF>
struct Frags { bf16x8 alo[MA], ahi[MA], b[2][NF]; };

// acc[i0 + i][j] += A block i x B block j.  The B fragment is the first operand: a lane's four accumulator
// values are four consecutive columns of one row of C.
// F16: the 16-bit operands are IEEE halves (v_mfma_f32_16x16x32_f16; same rate, same fragment layout).
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
template <int MA, int NF, int MI16, bool F16 = false>
__device__ __forceinline__ void mfma_blocks(floatx4 (&acc)[MI16][NF], const bf16x8 (&a)[MA], const bf16x8 (&b)[NF], int i0) {
#pragma unroll
  for (int i = 0; i < MA; ++i)
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      if constexpr (F16)
        acc[i0 + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, b[j]), __builtin_bit_cast(halfx8, a[i]),
                                                                acc[i0 + i][j], 0, 0, 0);
      else
        acc[i0 + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i0 + i][j], 0, 0, 0);
    }
}

// 32x32x16 path (both operands K-strided): fragments of one 16-wide k-step, MI row blocks of A and NB column
// blocks of B (32 x 16 each, two transpose reads per fragment).
template <int MI, int NB>
struct Frags32 { bf16x8 a[MI], b[NB]; };
template <int MI, int NB>
__device__ __forceinline__ void load_frags32(Frags32<MI, NB>& f, const char* sa, int ks, int wm, int wn, int lane) {
  const char* sb = sa + DTILE;
#pragma unroll
  for (int i = 0; i < MI; ++i) f.a[i] = read_frag<false>(sa, wm + i * 32, ks, lane);
#pragma unroll
  for (int j = 0; j < NB; ++j) f.b[j] = read_frag<false>(sb, wn + j * 32, ks, lane);
}
template <int MI, int NB>
__device__ __forceinline__ void mfma32(floatx16 (&acc)[MI][NB], const Frags32<MI, NB>& f) {
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[j], f.a[i], acc[i][j], 0, 0, 0);
}

// Ask the scheduler to interleave N_DS LDS reads, N_VM global->LDS loads and N_MFMA MFMAs in groups, reads
// leading.  The loads are spread over the groups on purpose: a wavefront that issues its loads of a step
// back to back sits at the (in-order) issue of the later ones while the texture path works through the
// earlier ones, and its MFMAs wait behind them; one load between every few MFMAs never queues.
template <int N_DS, int N_MFMA, int N_VM, int G, int Q>
__device__ __forceinline__ void interleave_group() {
  if constexpr (Q < G) {
    // LDS reads go into the first G-1 groups (the last MFMAs of the half-step cover the latency of the last reads)
    constexpr int DSG = G - 1;
    constexpr int DS = Q < DSG ? ((Q + 1) * N_DS + DSG - 1) / DSG - (Q * N_DS + DSG - 1) / DSG : 0;
    constexpr int VM = (Q + 1) * N_VM / G - Q * N_VM / G;
    constexpr int MF = (Q + 1) * N_MFMA / G - Q * N_MFMA / G;
    if constexpr (DS > 0) __builtin_amdgcn_sched_group_barrier(0x100, DS, 0);
    if constexpr (VM > 0) __builtin_amdgcn_sched_group_barrier(0x020, VM, 0);
    if constexpr (MF > 0) __builtin_amdgcn_sched_group_barrier(0x008, MF, 0);
    interleave_group<N_DS, N_MFMA, N_VM, G, Q + 1>();
  }
}
template <int N_DS, int N_MFMA, int N_VM>
__device__ __forceinline__ void interleave_ds_vm_mfma() {
  interleave_group<N_DS, N_MFMA, N_VM, (N_MFMA % 4 == 0) ? 4 : 2, 0>();
}

// WM x WN wavefronts tile the 256x256 block; each owns (256/WM) x (256/WN).
__device__ __forceinline__ float sigmoid_f(float z) { return 1.0f / (1.0f + __expf(-z)); }
// Normal distribution function of u and e = exp(-u^2/2): the lower tail Phi(-|u|) = e w, w = erfcx(|u| / sqrt 2) / 2 = 1/2 + s R(s)
// with s = 1 / (1 + 0.3 |u| / sqrt 2) - 1 and R a degree-8 polynomial fitted to the relative error in w (reweighted least squares
// against 64-bit erfcx).  With its coefficients in fp32 that error is 5e-8 for |u| < 1, 2e-7 to 3, 5e-7 to 6 and 1.7e-6 to 13
// (unrounded the fit reaches 1.7e-8: the terms cancel as w falls).  The epilogues of the GELU forms are bound by this: the library's erff is
// two expansions, both run by a wavefront whose lanes differ.  Against 64 bits (2-norm, u in -3..0 / 0..9 / -9..-3): u Phi 8e-8 / 2e-8 /
// 4e-7, the derivative 5e-8 / 4e-8 / 2e-7; by 1 + erff 1e-7 / 2e-8 / 4e-5 and 5e-8 / 4e-8 / 3e-6 (1 + erff cancels in the lower tail).
__device__ __forceinline__ float normal_cdf(float u, float& e) {
  const float x = fminf(fabsf(u), 1e30f) * 0.212132034f, t = __builtin_amdgcn_rcpf(1.0f + x), s = -(x * t);
  e = __expf(-0.5f * u * u);
  float r = -0.0615883172f;
  r = fmaf(r, s, -0.329083174f);
  r = fmaf(r, s, -0.629304707f);
  r = fmaf(r, s, -0.148489118f);
  r = fmaf(r, s, 1.6587162f);
  r = fmaf(r, s, 3.8503294f);
  r = fmaf(r, s, 4.69918823f);
  r = fmaf(r, s, 3.67486835f);
  r = fmaf(r, s, 1.88063073f);
  const float q = fmaf(r, s, 0.5f) * e;
  return u < 0.0f ? q : 1.0f - q;
}
__device__ __forceinline__ float gelu_f(float u) {
  float e;
  return u * normal_cdf(u, e);
}
__device__ __forceinline__ float gelu_grad_f(float u) {
  float e;
  const float phi = normal_cdf(u, e);
  return fmaf(u * 0.39894228040143268f, e, phi);
}
__device__ __forceinline__ void load_f32x8(const float* p, float* v) {
  const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void unpack4(uint2 w, float* v) {
  v[0] = __uint_as_float(w.x << 16); v[1] = __uint_as_float(w.x & 0xffff0000u);
  v[2] = __uint_as_float(w.y << 16); v[3] = __uint_as_float(w.y & 0xffff0000u);
}

// One tile of C at rows m0.., columns n0.. (the whole of gemm_mfma_dl_kernel after its placement).
// BMT = rows of the C tile: 256, or 128 for the short tiles that finish a GEMM whose tile count is
// not a multiple of the CU count (A K-contiguous only).
// F16IN: A and B hold IEEE halves instead of bf16 (forms with a K-contiguous operand only); TO may be float,
// bf16_t or f16_t.
template <bool A_KC, bool B_KC, typename TO, bool HAS_R, int WM, int WN, int ACT, int BMT = 256, bool F16IN = false>
__device__ __forceinline__ void dl_tile(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, TO* __restrict__ C,
                                        const float* __restrict__ R, int M, int N, int K, int lda, int ldb, int ldc, int ldr, int m0,
                                        int n0, bf16_t* __restrict__ E, int lde, const bf16_t* __restrict__ bias,
                                        const float* __restrict__ out_scale) {
  constexpr int NW = WM * WN;
  constexpr int MI = (BMT / 32) / WM;               // 32-high row blocks per wavefront
  constexpr int NB = 8 / WN;                        // 32-wide column blocks per wavefront
  constexpr int WAVE_M = MI * 32, WAVE_N = NB * 32;
  __shared__ __attribute__((aligned(1024))) char stage0[DSTAGE];
  __shared__ __attribute__((aligned(1024))) char stage1[DSTAGE];
  __shared__ __attribute__((aligned(1024))) char stage2[DSTAGE];
  __shared__ __attribute__((aligned(1024))) char stage3[DSTAGE];
  __shared__ __attribute__((aligned(1024))) char stage4[DSTAGE];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = (wave / WN) * WAVE_M, wn = (wave % WN) * WAVE_N;

  constexpr bool M32 = dl_m32(A_KC, B_KC);          // 32x32x16 accumulators (acc32) instead of 16x16x32 ones (acc)
  static_assert(!(M32 && F16IN), "half inputs are built for the 16x16x32 forms only");
  constexpr int MI16 = 2 * MI, NF = 2 * NB, MA = MI;   // 16-row / 16-column blocks per wavefront; A blocks per half
  floatx4 acc[M32 ? 1 : MI16][M32 ? 1 : NF];
  floatx16 acc32[M32 ? MI : 1][M32 ? NB : 1];
  if constexpr (M32) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc32[i][j][e] = 0.f;
  } else {
#pragma unroll
    for (int i = 0; i < MI16; ++i)
#pragma unroll
      for (int j = 0; j < NF; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;
  }

  DirectLoader<A_KC, NW, BMT, M32> la;
  DirectLoader<B_KC, NW, 256, M32> lb;
  la.init(A, lda, m0, M, K, wave, lane);
  lb.init(B, ldb, n0, N, K, wave, lane, ACT == ACT_SWIGLU_FWD ? N / 2 : 0);
  const int nk = (K + DBK - 1) / DBK;

  // Software pipeline over 32-deep steps through a ring of five LDS buffers (step t lives in buffer
  // t % 5).  Loads are issued for PAIRS of steps (e, e+1), e even, in four quarters spread over four
  // consecutive half-steps, starting right after the barrier in the middle of step e-4 (which frees the
  // buffer of step e-4 for step e+1; the buffer of step e-5 is free since the barrier before):
  //   quarter 0 in the second half of step e-4, 1 and 2 in the two halves of step e-3, 3 in the first
  //   half of step e-2.
  // Entering step t the fragments of the first half of the wavefront's A blocks and of all its B blocks
  // are in registers.  First half: read the second half of the A blocks under the MFMAs of the first
  // (after this, nobody reads buffer t % 5 any more).  Middle: wait for the own LDS reads and,
  // on odd steps, for this wavefront's loads of the pair (t+1, t+2): everything but quarters 0 and 1 of
  // the following pair, which were issued later; then barrier: buffer t % 5 is consumed by everybody and
  // the pair (t+1, t+2) is complete.  On even steps the next step's buffer is complete since the previous
  // barrier.  Second half: read step t+1's first A half and its B blocks (into the other B register
  // set) under the MFMAs of the second A half.
  using LoaderA = DirectLoader<A_KC, NW, BMT, M32>;
  using LoaderB = DirectLoader<B_KC, NW, 256, M32>;
  constexpr int LA = LoaderA::NL, LB = LoaderB::NL;
  constexpr int NQ0 = QuarterCount<0, LA, LB>::LOADS, NQ1 = QuarterCount<1, LA, LB>::LOADS;
  constexpr int NQ2 = QuarterCount<2, LA, LB>::LOADS, NQ3 = QuarterCount<3, LA, LB>::LOADS;
  constexpr int LGKM_ONLY = 0xC07F;                                // vmcnt(63), lgkmcnt(0)
  constexpr int VM_01 = 0x0070 | ((NQ0 + NQ1) & 15) | (((NQ0 + NQ1) >> 4) << 14);              // vmcnt(NQ0+NQ1), lgkmcnt(0)
  constexpr int VM_012 = 0x0070 | ((NQ0 + NQ1 + NQ2) & 15) | (((NQ0 + NQ1 + NQ2) >> 4) << 14);  // vmcnt(NQ0+NQ1+NQ2), lgkmcnt(0)
  constexpr int DS_A = A_KC ? MA : 2 * MA, DS_B = B_KC ? NF : 2 * NF;   // LDS read instructions of half the A blocks / all B blocks
  constexpr int N_MFMA = MA * NF;                                        // MFMAs of a half-step
  // One step.  PAR = parity of tt; b0..b4 = the buffers of steps tt..tt+4; GUARD = the step may be the
  // last one or beyond (the tail loop), else every step up to tt+5 exists.
#define RRFP_STEP(PAR, GUARD, b0, b1, b2, b3, b4, tt)                                                    \
  if (!GUARD || (tt) < nk) {                                                                             \
    if constexpr (PAR == 0) issue_quarter<3, GUARD>(la, lb, b2, b3, (tt) + 2, nk, wave);                 \
    else issue_quarter<1, GUARD>(la, lb, b3, b4, (tt) + 3, nk, wave);                                    \
    if constexpr (M32) {                                                                                 \
      load_frags32<MI, NB>(fy, b0, 1, wm, wn, lane);                                                     \
      mfma32<MI, NB>(acc32, fx);                                                                         \
      interleave_ds_vm_mfma<2 * (MI + NB), MI * NB, (PAR == 0 ? NQ3 : NQ1)>();                           \
    } else {                                                                                             \
      load_blocks<A_KC, MA>(fr.ahi, b0, off_ahi);                                                        \
      mfma_blocks<MA, NF, MI16, F16IN>(acc, fr.alo, fr.b[PAR], 0);                                       \
      interleave_ds_vm_mfma<DS_A, N_MFMA, (PAR == 0 ? NQ3 : NQ1)>();                                     \
    }                                                                                                    \
    if (!GUARD || (tt) + 1 < nk) {                                                                       \
      __builtin_amdgcn_s_waitcnt(PAR == 0 ? LGKM_ONLY : VM_01);                                          \
      stage_barrier();                                                                                   \
      if constexpr (PAR == 0) issue_quarter<0, GUARD>(la, lb, b4, b0, (tt) + 4, nk, wave);               \
      else issue_quarter<2, GUARD>(la, lb, b3, b4, (tt) + 3, nk, wave);                                  \
      if constexpr (M32) {                                                                               \
        load_frags32<MI, NB>(fx, b1, 0, wm, wn, lane);                                                   \
      } else {                                                                                           \
        load_blocks<A_KC, MA>(fr.alo, b1, off_alo);                                                      \
        load_blocks<B_KC, NF>(fr.b[1 - PAR], b1 + DTILE, off_b);                                         \
      }                                                                                                  \
    }                                                                                                    \
    if constexpr (M32) mfma32<MI, NB>(acc32, fy);                                                        \
    else mfma_blocks<MA, NF, MI16, F16IN>(acc, fr.ahi, fr.b[PAR], MA);                                   \
    if (!GUARD) {                                                                                        \
      if constexpr (M32) interleave_ds_vm_mfma<2 * (MI + NB), MI * NB, (PAR == 0 ? NQ0 : NQ2)>();        \
      else interleave_ds_vm_mfma<DS_A + DS_B, N_MFMA, (PAR == 0 ? NQ0 : NQ2)>();                         \
      __builtin_amdgcn_sched_barrier(0);   /* half-steps are scheduled one by one */                     \
    }                                                                                                    \
  }
#define RRFP_TEN_STEPS(GUARD, t)                                        \
  RRFP_STEP(0, GUARD, stage0, stage1, stage2, stage3, stage4, (t));     \
  RRFP_STEP(1, GUARD, stage1, stage2, stage3, stage4, stage0, (t) + 1); \
  RRFP_STEP(0, GUARD, stage2, stage3, stage4, stage0, stage1, (t) + 2); \
  RRFP_STEP(1, GUARD, stage3, stage4, stage0, stage1, stage2, (t) + 3); \
  RRFP_STEP(0, GUARD, stage4, stage0, stage1, stage2, stage3, (t) + 4); \
  RRFP_STEP(1, GUARD, stage0, stage1, stage2, stage3, stage4, (t) + 5); \
  RRFP_STEP(0, GUARD, stage1, stage2, stage3, stage4, stage0, (t) + 6); \
  RRFP_STEP(1, GUARD, stage2, stage3, stage4, stage0, stage1, (t) + 7); \
  RRFP_STEP(0, GUARD, stage3, stage4, stage0, stage1, stage2, (t) + 8); \
  RRFP_STEP(1, GUARD, stage4, stage0, stage1, stage2, stage3, (t) + 9)

  Frags<MA, NF> fr;
  Frags32<MI, NB> fx, fy;
  const int off_alo = frag_lane_offset<A_KC>(wm, lane), off_ahi = frag_lane_offset<A_KC>(wm + MA * 16, lane);
  const int off_b = frag_lane_offset<B_KC>(wn, lane);
  // Prologue: the pair (0, 1) in full and quarters 0..2 of the pair (2, 3); step 0's first half issues quarter 3.
  issue_quarter<0, true>(la, lb, stage0, stage1, 0, nk, wave);
  issue_quarter<1, true>(la, lb, stage0, stage1, 0, nk, wave);
  issue_quarter<2, true>(la, lb, stage0, stage1, 0, nk, wave);
  issue_quarter<3, true>(la, lb, stage0, stage1, 0, nk, wave);
  issue_quarter<0, true>(la, lb, stage2, stage3, 2, nk, wave);
  issue_quarter<1, true>(la, lb, stage2, stage3, 2, nk, wave);
  issue_quarter<2, true>(la, lb, stage2, stage3, 2, nk, wave);
  __builtin_amdgcn_s_waitcnt(VM_012);
  stage_barrier();
  if constexpr (M32) {
    load_frags32<MI, NB>(fx, stage0, 0, wm, wn, lane);
  } else {
    load_blocks<A_KC, MA>(fr.alo, stage0, off_alo);
    load_blocks<B_KC, NF>(fr.b[0], stage0 + DTILE, off_b);
  }

  int t = 0;
  for (; t + 13 < nk; t += 10) {    // every load these ten steps issue is for a step below nk
    RRFP_TEN_STEPS(false, t);
  }
  for (; t < nk; t += 10) {
    RRFP_TEN_STEPS(true, t);
  }
#undef RRFP_TEN_STEPS
#undef RRFP_STEP
  __builtin_amdgcn_s_waitcnt(0x0070);   // the zero loads of the steps past the end have landed too

  // Epilogue through LDS.  In the accumulator layout a lane owns 4 consecutive columns of one row, so a
  // direct store instruction would touch 32 different rows with 16 bytes each.  Instead every wavefront
  // writes one 32-row block of its accumulators to its own LDS scratch (the pipeline stages are free
  // now), and reads it back with 8 consecutive columns per lane and whole rows per group of lanes: all
  // global loads and stores of the epilogue (C, the residual, the activation operand) are then row-
  // contiguous 16- or 32-byte accesses per lane.
  __syncthreads();     // every wavefront has finished its fragment reads of the last step
  float* scratch;
  {
    constexpr int PER = DSTAGE * 4 / NW;            // bytes of scratch per wavefront: 16 KB (8 waves) or 32 KB (4)
    const int sel = wave * PER / DSTAGE, sub = (wave * PER) % DSTAGE;
    char* base = sel == 0 ? stage0 : sel == 1 ? stage1 : sel == 2 ? stage2 : stage3;
    scratch = reinterpret_cast<float*>(base + sub);
  }
  constexpr int NBC = NB * 32;                      // columns of the wavefront's tile
  constexpr int PITCH = NBC + 4;                    // floats; 16-byte skew per row
  const int li = lane & 15, hq = lane >> 4;
  // The epilogue's global operand loads (residual, activation operand) are issued for a whole 32-row
  // chunk before the chunk is staged, from addresses clamped into the matrix, so that their latency is
  // paid once per chunk and not once per sweep; only the stores are predicated.
  constexpr int LPR = NBC / 8;                      // lanes per row of the read-back
  constexpr int RPS = 64 / LPR;                     // rows per sweep
  constexpr int SW = 32 / RPS;                      // sweeps per chunk
  const int c0 = (lane % LPR) * 8, r0 = lane / LPR;
  const int n_col = n0 + wn + c0;                   // first of this lane's 8 columns (same for every sweep)
  const int n_ld = min(n_col, N - 8);
  float bv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (ACT != ACT_SWIGLU_FWD && bias) load_vec<bf16_t>(bias + n_ld, bv);
  // out_scale (plain 16-bit outputs only): a device scalar, a power of two, multiplied into the result before it
  // is rounded -- brings a gradient tensor into the range of IEEE halves whatever the scale of the loss
  const float oscale = (ACT == ACT_NONE && !HAS_R && sizeof(TO) == 2 && out_scale) ? *out_scale : 1.0f;
  struct Pre { float rv[8]; uint4 e0, e1; };
  auto prefetch = [&](Pre (&pre)[SW], int i) {
#pragma unroll
    for (int rr = 0; rr < SW; ++rr) {
      const int m_ld = min(m0 + wm + i * 32 + rr * RPS + r0, M - 1);
      if (HAS_R) load_f32x8(R + (size_t)m_ld * ldr + n_ld, pre[rr].rv);
      if (ACT == ACT_GELU_BWD || ACT == ACT_SWIGLU_BWD) pre[rr].e0 = *reinterpret_cast<const uint4*>(E + (size_t)m_ld * lde + n_ld);
      if (ACT == ACT_SWIGLU_BWD) pre[rr].e1 = *reinterpret_cast<const uint4*>(E + (size_t)m_ld * lde + N + n_ld);
    }
  };
  Pre pre[2][SW];
  if (ACT != ACT_SWIGLU_FWD) prefetch(pre[0], 0);
  // The lanes of a wavefront exchange values through the wavefront's own scratch: write in the accumulator
  // layout, read back row-contiguous, overwrite with the next chunk.  The hardware executes one wavefront's
  // LDS instructions in order; these wavefront-scope fences keep the compiler from reordering the three phases.
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    wave_sync();        // read-back of chunk i-1 precedes the writes of chunk i
    if constexpr (M32) {
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<float4*>(scratch + (lane & 31) * PITCH + j * 32 + g * 8 + (lane >> 5) * 4) =
              make_float4(acc32[i][j][g * 4 + 0], acc32[i][j][g * 4 + 1], acc32[i][j][g * 4 + 2], acc32[i][j][g * 4 + 3]);
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < NF; ++j)
          *reinterpret_cast<float4*>(scratch + (h * 16 + li) * PITCH + j * 16 + hq * 4) =
              make_float4(acc[2 * i + h][j][0], acc[2 * i + h][j][1], acc[2 * i + h][j][2], acc[2 * i + h][j][3]);
    }
    wave_sync();        // the writes of chunk i precede its read-back
    if (ACT == ACT_SWIGLU_FWD) {
      // scratch columns 0..31 = gate, 32..63 = up of features f0 .. f0+31; 4 lanes per row, 16 rows per sweep
      const int F = N >> 1;
      const int f0 = (n0 >> 1) + (wn >> 6) * 32;
      const int fc = (lane & 3) * 8;
      float bg[8], bu[8];
      if (bias) {
        load_vec<bf16_t>(bias + f0 + fc, bg);
        load_vec<bf16_t>(bias + F + f0 + fc, bu);
      }
#pragma unroll
      for (int rr = 0; rr < 2; ++rr) {
        const int row = rr * 16 + (lane >> 2);
        const int m = m0 + wm + i * 32 + row;
        float gt[8], up[8], mm[8];
        load_f32x8(scratch + row * PITCH + fc, gt);
        load_f32x8(scratch + row * PITCH + 32 + fc, up);
        if (bias) {
#pragma unroll
          for (int e = 0; e < 8; ++e) { gt[e] += bg[e]; up[e] += bu[e]; }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) mm[e] = gt[e] * sigmoid_f(gt[e]) * up[e];
        if (m < M) {
          bf16_t* crow = (bf16_t*)C + (size_t)m * ldc + f0 + fc;
          store_vec<bf16_t>(crow, gt);
          store_vec<bf16_t>(crow + F, up);
          store_vec<bf16_t>(E + (size_t)m * lde + f0 + fc, mm);
        }
      }
    } else if (sizeof(TO) == 4 && ACT == ACT_NONE && !HAS_R && !bias) {
      // plain fp32 tile: 16 bytes per lane with the lanes of a row side by side, so that every store instruction
      // writes whole 128-byte lines (with 32 bytes per lane each of the two stores would write half of every line)
      constexpr int LPR4 = NBC / 4, RPS4 = 64 / LPR4, SW4 = 32 / RPS4;
      const int c4 = (lane % LPR4) * 4, r4 = lane / LPR4;
      const int n = n0 + wn + c4;
#pragma unroll
      for (int rr = 0; rr < SW4; ++rr) {
        const int row = rr * RPS4 + r4;
        const int m = m0 + wm + i * 32 + row;
        const float4 v = *reinterpret_cast<const float4*>(scratch + row * PITCH + c4);
        if (m < M && n < N) *reinterpret_cast<float4*>((float*)C + (size_t)m * ldc + n) = v;   // N is a multiple of 8
      }
    } else {
      if (i + 1 < MI) prefetch(pre[(i + 1) & 1], i + 1);
      const Pre (&cur)[SW] = pre[i & 1];
#pragma unroll
      for (int rr = 0; rr < SW; ++rr) {
        const int row = rr * RPS + r0;
        const int m = m0 + wm + i * 32 + row, n = n_col;
        float v[8];
        load_f32x8(scratch + row * PITCH + c0, v);
        const bool ok = m < M && n < N;             // N is a multiple of 8: the eight columns are in or out together
        if (bias) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] += bv[e];
        }
        if (HAS_R) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] += cur[rr].rv[e];
        }
        if (ACT == ACT_GELU_FWD) {
          float mm[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) mm[e] = gelu_f(v[e]);
          if (ok) {
            store_vec<bf16_t>((bf16_t*)C + (size_t)m * ldc + n, v);
            store_vec<bf16_t>(E + (size_t)m * lde + n, mm);
          }
        } else if (ACT == ACT_GELU_BWD) {
          float u[8];
          unpack4(make_uint2(cur[rr].e0.x, cur[rr].e0.y), u);
          unpack4(make_uint2(cur[rr].e0.z, cur[rr].e0.w), u + 4);
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] *= gelu_grad_f(u[e]);
          if (ok) store_vec<bf16_t>((bf16_t*)C + (size_t)m * ldc + n, v);
        } else if (ACT == ACT_SWIGLU_BWD) {
          float gt[8], up[8], dg[8], du[8];
          unpack4(make_uint2(cur[rr].e0.x, cur[rr].e0.y), gt);
          unpack4(make_uint2(cur[rr].e0.z, cur[rr].e0.w), gt + 4);
          unpack4(make_uint2(cur[rr].e1.x, cur[rr].e1.y), up);
          unpack4(make_uint2(cur[rr].e1.z, cur[rr].e1.w), up + 4);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float sg = sigmoid_f(gt[e]);
            dg[e] = v[e] * up[e] * sg * (1.0f + gt[e] * (1.0f - sg));
            du[e] = v[e] * gt[e] * sg;
          }
          if (ok) {
            store_vec<bf16_t>((bf16_t*)C + (size_t)m * ldc + n, dg);
            store_vec<bf16_t>((bf16_t*)C + (size_t)m * ldc + N + n, du);
          }
        } else if (sizeof(TO) == 4) {
          if (ok) {
            float* crow = (float*)C + (size_t)m * ldc + n;
            *reinterpret_cast<float4*>(crow) = make_float4(v[0], v[1], v[2], v[3]);
            *reinterpret_cast<float4*>(crow + 4) = make_float4(v[4], v[5], v[6], v[7]);
          }
        } else {
          using T16 = std::conditional_t<sizeof(TO) == 2, TO, bf16_t>;    // bf16_t or f16_t
          if constexpr (ACT == ACT_NONE && !HAS_R) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] *= oscale;
          }
          if (ok) store_vec<T16>((T16*)C + (size_t)m * ldc + n, v);
        }
      }
    }
  }
}

// tn0 = first tile column of this launch.
template <bool A_KC, bool B_KC, typename TO, bool HAS_R, int WM, int WN, int ACT, int BMT = 256, bool F16IN = false>
__global__ __launch_bounds__(WM * WN * 64) void gemm_mfma_dl_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B,
                                                               TO* __restrict__ C, const float* __restrict__ R, int M,
                                                               int N, int K, int lda, int ldb, int ldc, int ldr,
                                                               int tiles_m, int tiles_n, bf16_t* __restrict__ E, int lde,
                                                               int tn0, int k_split, const bf16_t* __restrict__ bias,
                                                               const float* __restrict__ out_scale) {
  // Split-K launches (grid y = split): this workgroup contracts k in [y * k_split, min(K, (y+1) * k_split))
  // and writes its partial tile into the y-th [M, ldc] plane of C.
  if (k_split > 0) {
    const int k0 = blockIdx.y * k_split;
    A += A_KC ? (size_t)k0 : (size_t)k0 * lda;
    B += B_KC ? (size_t)k0 : (size_t)k0 * ldb;
    C += (size_t)blockIdx.y * M * ldc;
    K = min(k_split, K - k0);
  }
  int tm, tn;
  tile_coords(blockIdx.x, tiles_m, tiles_n, tm, tn);
  dl_tile<A_KC, B_KC, TO, HAS_R, WM, WN, ACT, BMT, F16IN>(A, B, C, R, M, N, K, lda, ldb, ldc, ldr, tm * BMT, (tn + tn0) * BN, E, lde, bias,
                                                         out_scale);
}

// Explicit instantiations of every variant the launcher can pick.
#define RRFP_INST(AKC, BKC, TO, HR, ACT)                                                                     \
  template __global__ void gemm_mfma_dl_kernel<AKC, BKC, TO, HR, dl_wm(AKC, BKC), dl_wn(AKC, BKC), ACT>(      \
      const bf16_t*, const bf16_t*, TO*, const float*, int, int, int, int, int, int, int, int, int, bf16_t*, int, int, int, const bf16_t*, const float*);
#define RRFP_INST_SHORT(BKC, TO, HR, ACT)                                                                    \
  template __global__ void gemm_mfma_dl_kernel<true, BKC, TO, HR, dl_wm(true, BKC), dl_wn(true, BKC), ACT, 128>( \
      const bf16_t*, const bf16_t*, TO*, const float*, int, int, int, int, int, int, int, int, int, bf16_t*, int, int, int, const bf16_t*, const float*);
#define RRFP_INST_SHORT4(BKC) RRFP_INST_SHORT(BKC, float, true, ACT_NONE) RRFP_INST_SHORT(BKC, float, false, ACT_NONE) \
                              RRFP_INST_SHORT(BKC, bf16_t, true, ACT_NONE) RRFP_INST_SHORT(BKC, bf16_t, false, ACT_NONE)
RRFP_INST_SHORT4(false) RRFP_INST_SHORT4(true)
RRFP_INST_SHORT(false, bf16_t, false, ACT_SWIGLU_FWD) RRFP_INST_SHORT(false, bf16_t, false, ACT_GELU_FWD)
RRFP_INST_SHORT(true, bf16_t, false, ACT_SWIGLU_BWD) RRFP_INST_SHORT(true, bf16_t, false, ACT_GELU_BWD)
#undef RRFP_INST_SHORT4
#undef RRFP_INST_SHORT
#define RRFP_INST4(AKC, BKC) RRFP_INST(AKC, BKC, float, true, ACT_NONE) RRFP_INST(AKC, BKC, float, false, ACT_NONE) \
                             RRFP_INST(AKC, BKC, bf16_t, true, ACT_NONE) RRFP_INST(AKC, BKC, bf16_t, false, ACT_NONE)
RRFP_INST4(true, false) RRFP_INST4(true, true) RRFP_INST4(false, false) RRFP_INST4(false, true)
RRFP_INST(true, false, bf16_t, false, ACT_SWIGLU_FWD) RRFP_INST(true, false, bf16_t, false, ACT_GELU_FWD)
RRFP_INST(true, true, bf16_t, false, ACT_SWIGLU_BWD) RRFP_INST(true, true, bf16_t, false, ACT_GELU_BWD)
#undef RRFP_INST4
#undef RRFP_INST
// Half-precision forms of the attention path: the QKV projection (half in, half out), the output projection
// (half in, fp32 out with the residual) and the gradient of the attention output, dO = dx1 Wo^T (bf16 in, half
// out), each with its 128-row tile variant.
template __global__ void gemm_mfma_dl_kernel<true, false, f16_t, false, dl_wm(true, false), dl_wn(true, false), ACT_NONE, 256, true>(
    const bf16_t*, const bf16_t*, f16_t*, const float*, int, int, int, int, int, int, int, int, int, bf16_t*, int, int, int, const bf16_t*, const float*);
template __global__ void gemm_mfma_dl_kernel<true, false, f16_t, false, dl_wm(true, false), dl_wn(true, false), ACT_NONE, 128, true>(
    const bf16_t*, const bf16_t*, f16_t*, const float*, int, int, int, int, int, int, int, int, int, bf16_t*, int, int, int, const bf16_t*, const float*);
template __global__ void gemm_mfma_dl_kernel<true, false, float, true, dl_wm(true, false), dl_wn(true, false), ACT_NONE, 256, true>(
    const bf16_t*, const bf16_t*, float*, const float*, int, int, int, int, int, int, int, int, int, bf16_t*, int, int, int, const bf16_t*, const float*);
template __global__ void gemm_mfma_dl_kernel<true, false, float, true, dl_wm(true, false), dl_wn(true, false), ACT_NONE, 128, true>(
    const bf16_t*, const bf16_t*, float*, const float*, int, int, int, int, int, int, int, int, int, bf16_t*, int, int, int, const bf16_t*, const float*);
template __global__ void gemm_mfma_dl_kernel<true, true, f16_t, false, dl_wm(true, true), dl_wn(true, true), ACT_NONE, 256, false>(
    const bf16_t*, const bf16_t*, f16_t*, const float*, int, int, int, int, int, int, int, int, int, bf16_t*, int, int, int, const bf16_t*, const float*);
template __global__ void gemm_mfma_dl_kernel<true, true, f16_t, false, dl_wm(true, true), dl_wn(true, true), ACT_NONE, 128, false>(
    const bf16_t*, const bf16_t*, f16_t*, const float*, int, int, int, int, int, int, int, int, int, bf16_t*, int, int, int, const bf16_t*, const float*);

// True when the direct-to-LDS kernel can take the call (else the register-staged one does).
inline bool direct_ok(const GemmArgs& g) {
  const bool a_kc = !g.transA, b_kc = g.transB;
  if ((a_kc || b_kc) && (g.K % DBK)) return false;
  const size_t lim = (size_t)1 << 31;      // every operand byte offset stays below the per-lane offset that means "out of range"
  const size_t a_bytes = (size_t)(a_kc ? g.M + BM : g.K + BK) * g.lda * 2;
  const size_t b_bytes = (size_t)(b_kc ? g.N + BN : g.K + BK) * g.ldb * 2;
  return a_bytes < lim && b_bytes < lim;
}

// Compute units of the current device (cached per device id; 256 if the query fails).
inline int cu_count() {
  static int cached[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] == 0) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 1) v = 256;
    cached[dev] = v;
  }
  return cached[dev];
}

// How a GEMM with A K-contiguous is cut into launches.  One workgroup occupies a CU, so t tiles of
// 256 x 256 run in ceil(t / n_cu) rounds.  (a) A grid that fills at most half the CUs is launched
// entirely with 128-row tiles (twice the workgroups).  (b) Otherwise, when the last round holds r
// tiles and carving ceil(r / tiles_m) trailing tile columns off removes that round, those columns
// are launched separately with 128-row tiles, provided they fit one round.  A pure function of the
// shape and the device.  Returns the number of tile columns of the 256-row launch.
inline int full_tile_columns(int tiles_m, int tiles_n, int n_cu) {
  const int t = tiles_m * tiles_n;
  if (2 * t <= n_cu) return 0;
  const int r = t % n_cu;
  if (t <= n_cu || r == 0) return tiles_n;
  const int ct = (r + tiles_m - 1) / tiles_m;
  if (ct >= tiles_n) return tiles_n;
  const int t_main = t - ct * tiles_m;
  const bool removes_round = (t_main + n_cu - 1) / n_cu < (t + n_cu - 1) / n_cu;
  const bool tail_fits = 2 * ct * tiles_m <= n_cu;
  return (removes_round && tail_fits) ? tiles_n - ct : tiles_n;
}

// Sum of S partial planes [M, ldw] (plane stride M * ldw floats) in plane order into the column block
// out[m, 0 .. width) of a matrix with row pitch ldo: the fixed-order finish of a split-K tail launch.
__global__ __launch_bounds__(256) void splitk_tail_reduce_kernel(const float* __restrict__ ws, int S, int M, int ldw,
                                                                 float* __restrict__ out, int ldo, int width) {
  const int w4 = width >> 2;
  const size_t n = (size_t)M * w4;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const int m = (int)(i / w4), c = (int)(i - (size_t)m * w4) * 4;
    float4 acc = *reinterpret_cast<const float4*>(ws + (size_t)m * ldw + c);
    for (int p = 1; p < S; ++p) {
      const float4 v = *reinterpret_cast<const float4*>(ws + ((size_t)p * M + m) * ldw + c);
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
    *reinterpret_cast<float4*>(out + (size_t)m * ldo + c) = acc;
  }
}

// Weight-gradient form as a single call (rrfp_gemm_ws; a W task launches its products together, see wgrad_group_cut) on a grid
// of more than one round: when the last round would be nearly empty and carving
// the trailing tile columns off removes it (the rule of full_tile_columns), those columns are a second launch
// whose tiles are split along K into TAIL_SPLIT ranges (so the tail fills the CUs for half a round instead of a
// fraction of them for a whole one); each range writes its own compact partial plane into the scratch and the
// planes are added in range order.  Returns the tile columns of the plain launch (tiles_n = no tail).
constexpr int TAIL_SPLIT = 2;
inline int wgrad_full_tile_columns(const GemmArgs& g, int tiles_m, int tiles_n, int n_cu, bool have_scratch) {
  if (!have_scratch || g.R || g.out_dtype != F32) return tiles_n;
  const int cn = full_tile_columns(tiles_m, tiles_n, n_cu);
  if (cn <= 0 || cn >= tiles_n) return tiles_n;
  const int steps = (g.K + DBK - 1) / DBK;
  const int width = g.N - cn * BN;
  if (steps < 16 * TAIL_SPLIT || (width & 3) || (g.ldc & 3)) return tiles_n;
  return cn;
}
inline size_t wgrad_tail_scratch_bytes(const GemmArgs& g, int cn) { return (size_t)TAIL_SPLIT * g.M * (g.N - cn * BN) * 4; }

// Split-K factor for a grid of t tiles and a contraction of K: as many ranges as fit the CUs, each at
// least 16 steps deep, at most 16 ranges; 1 = no split.  A pure function of the shape and the device.
inline int splitk_factor(int t, int K, int n_cu) {
  if (2 * t > n_cu) return 1;
  const int steps = (K + DBK - 1) / DBK;
  return std::max(1, std::min(std::min(n_cu / t, steps / 16), 16));
}

// What the tile epilogue does to 8 consecutive columns n.. of row m, for kernels that hold them in one thread: v (SwiGLU forward:
// v the gate, up the other half) are the fp32 sums, already with their bias.
template <typename TO, bool HAS_R, int ACT>
__device__ __forceinline__ void finish8(float (&v)[8], float (&up)[8], int m, int n, int N, TO* __restrict__ C, int ldc, const float* __restrict__ R,
                                        int ldr, bf16_t* __restrict__ E, int lde, const float* __restrict__ out_scale) {
  if constexpr (HAS_R) {
    float r[8];
    load_f32x8(R + (size_t)m * ldr + n, r);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += r[e];
  }
  TO* crow = C + (size_t)m * ldc + n;
  if constexpr (ACT == ACT_SWIGLU_FWD) {
    float mm[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) mm[e] = v[e] * sigmoid_f(v[e]) * up[e];
    store_vec<TO>(crow, v);
    store_vec<TO>(crow + (N >> 1), up);
    store_vec<bf16_t>(E + (size_t)m * lde + n, mm);
  } else if constexpr (ACT == ACT_GELU_FWD) {
    float mm[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) mm[e] = gelu_f(v[e]);
    store_vec<TO>(crow, v);
    store_vec<bf16_t>(E + (size_t)m * lde + n, mm);
  } else if constexpr (ACT == ACT_GELU_BWD) {
    float u[8];
    load_vec<bf16_t>(E + (size_t)m * lde + n, u);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] *= gelu_grad_f(u[e]);
    store_vec<TO>(crow, v);
  } else if constexpr (ACT == ACT_SWIGLU_BWD) {
    float gt[8], ut[8], dg[8], du[8];
    load_vec<bf16_t>(E + (size_t)m * lde + n, gt);
    load_vec<bf16_t>(E + (size_t)m * lde + N + n, ut);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float sg = sigmoid_f(gt[e]);
      dg[e] = v[e] * ut[e] * sg * (1.0f + gt[e] * (1.0f - sg));
      du[e] = v[e] * gt[e] * sg;
    }
    store_vec<TO>(crow, dg);
    store_vec<TO>(crow + N, du);
  } else {
    if constexpr (!HAS_R && sizeof(TO) == 2) {
      const float sc = out_scale ? *out_scale : 1.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] *= sc;
    }
    store_vec<TO>(crow, v);
    if constexpr (sizeof(TO) == 4) store_vec<TO>(crow + 4, v + 4);
  }
}
__device__ __forceinline__ void add_bias8(const bf16_t* __restrict__ bias, int n, float (&v)[8]) {
  if (!bias) return;
  float b[8];
  load_vec<bf16_t>(bias + n, b);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] += b[e];
}

// Finish of a split-K launch of a form with A K-contiguous: adds the S partial planes [M, N] in range order and applies what
// the unsplit kernel's epilogue applies, on the same fp32 values.  A thread owns 8 columns (of SwiGLU forward: 8
// features, gate and up).
template <typename TO, bool HAS_R, int ACT>
__global__ __launch_bounds__(256) void splitk_finish_kernel(const float* __restrict__ ws, int S, int M, int N, TO* __restrict__ C, int ldc,
                                                            const float* __restrict__ R, int ldr, bf16_t* __restrict__ E, int lde,
                                                            const bf16_t* __restrict__ bias, const float* __restrict__ out_scale) {
  const int width = ACT == ACT_SWIGLU_FWD ? N >> 1 : N, w8 = width >> 3;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (size_t)M * w8) return;
  const int m = (int)(i / w8), n = (int)(i - (size_t)m * w8) * 8;
  const size_t plane = (size_t)M * N;
  const float* row = ws + (size_t)m * N + n;
  auto sum_planes = [&](const float* p, float (&v)[8]) {
    load_f32x8(p, v);
#pragma unroll 4
    for (int y = 1; y < S; ++y) {
      float t[8];
      load_f32x8(p + y * plane, t);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] += t[e];
    }
  };
  float v[8], up[8];
  sum_planes(row, v);
  add_bias8(bias, n, v);
  if constexpr (ACT == ACT_SWIGLU_FWD) {
    sum_planes(row + width, up);
    add_bias8(bias, width + n, up);
  }
  finish8<TO, HAS_R, ACT>(v, up, m, n, N, C, ldc, R, ldr, E, lde, out_scale);
}

// ------------------------------------------------------------------------------------------
// Small outputs.  Tiles of 64 x 64 (or 32 x 32, see small_edge) whose NW wavefronts each contract a range of k on their own (64 accumulator registers of
// v_mfma_f32_16x16x32, no barrier before the end); their sums meet in LDS and are added in range order, and every fused
// epilogue of the tile kernel runs on them.  What bounds an output of a few tiles is latency: a 256- or 128-row tile is one
// workgroup's serial walk over K plus the store of a large tile by one CU (11 us for 512 x 512 x 100); this spreads
// both over 4 to 8 times the CUs and cuts the walk by NW.
//   K-contiguous operand: a lane's 16 bytes of a fragment come straight from memory.
//   K-strided operand: rows of 128 bytes go through registers to a wavefront-private LDS tile [32 k][64 columns] and come back
//     by the LDS transpose read; chunk c of row k sits at c ^ swz(k), so that the 8 k-rows of a pass meet 8 bank groups.
// Operands of k at or past K read as zero, rows and columns past the end repeat the last ones and are not stored.
// ------------------------------------------------------------------------------------------
constexpr int ST = 64;                                 // tile edge

__device__ __forceinline__ int st_swz(int k) { return ((((k >> 1) & 1) | (((k >> 3) & 1) << 1)) << 1); }

// One operand of a wavefront: 32-deep steps of EDGE / 16 loads.  (64-deep ones, which fetch whole 128-byte lines of a K-contiguous
// operand at once, measured the same and spilled in the SwiGLU form.)
template <bool KC, int EDGE>
struct SmallOperand {
  static constexpr int NB = EDGE / 16;                // 16-row blocks, and loads of a step
  static constexpr int CPR = EDGE / 8, KPL = 64 / CPR; // K-strided: 16-byte chunks per k row, k rows per load
  const bf16_t* p[NB];    // KC: row of fragment i at this lane's k offset; else: this lane's chunk of k row lane / CPR + KPL i
  int k_lane[NB], step;   // k of the lane's element in step 0; elements per step
  int lds_w, lds_r;
  // SwiGLU forward: the first half of the tile columns is gate, the second the up columns of the same features (pair_f = ffn)
  __device__ __forceinline__ void init(const bf16_t* base, int ld, int outer0, int outer_n, int lane, int pair_f) {
    step = KC ? 32 : 32 * ld;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if constexpr (KC) {
        k_lane[i] = (lane >> 4) * 8;
        p[i] = base + (size_t)min(outer0 + i * 16 + (lane & 15), outer_n - 1) * ld + k_lane[i];
      } else {
        const int c = lane % CPR * 8;
        const int col = pair_f > 0 ? (c >= EDGE / 2 ? pair_f : 0) + (outer0 >> 1) + c % (EDGE / 2) : min(outer0 + c, outer_n - 8);
        k_lane[i] = lane / CPR + i * KPL;
        p[i] = base + (size_t)k_lane[i] * ld + col;
      }
    }
    if constexpr (!KC) {
      // a row of the LDS tile is EDGE * 2 bytes; bits 0..2 (EDGE 32: 0..3) of k come from the lane, bit 3 of EDGE 64 from i (an XOR of
      // 64 bytes in put)
      lds_w = lane / CPR * (EDGE * 2) + ((lane % CPR ^ swz(lane / CPR)) << 4);
      const int kb = (lane >> 4) * 8 + ((lane & 15) >> 2);
      lds_r = kb * (EDGE * 2) + ((((lane & 3) >> 1) ^ swz(kb)) << 4) + (lane & 1) * 8;
    }
  }
  // The 8 k rows of a transposed read's pass meet 8 bank groups (EDGE 32: rows of half the length, two chunk pairs)
  __device__ static __forceinline__ int swz(int k) { return EDGE == 64 ? st_swz(k) : ((k >> 2) & 1) << 1; }
  __device__ __forceinline__ void fetch(uint4 (&r)[NB], int t, int k_end) const {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      r[i] = make_uint4(0, 0, 0, 0);
      if (t * 32 + k_lane[i] < k_end) r[i] = *reinterpret_cast<const uint4*>(p[i] + (size_t)t * step);
    }
  }
  __device__ __forceinline__ void put(const uint4 (&r)[NB], char* tile) const {
    if constexpr (!KC) {
#pragma unroll
      for (int i = 0; i < NB; ++i) *reinterpret_cast<uint4*>(tile + i * 1024 + (EDGE == 64 ? lds_w ^ ((i & 1) << 6) : lds_w)) = r[i];
    }
  }
  __device__ __forceinline__ bf16x8 frag(const uint4 (&r)[NB], const char* tile, int i) const {
    if constexpr (KC) return __builtin_bit_cast(bf16x8, r[i]);
    // block i: chunks 2i, 2i + 1; the second read is 4 k rows on (EDGE 32: the other swizzle)
    const lds_char_ptr q = (lds_char_ptr)tile + (lds_r ^ (i << 5));
    const lds_char_ptr q4 = EDGE == 64 ? q + 512 : (lds_char_ptr)tile + ((lds_r + 256) ^ (i << 5) ^ 32);
    union { short4v h[2]; bf16x8 v; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)q);
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)q4);
    return u.v;
  }
};

constexpr int SMALL_NW = 8;                            // four wavefronts, two workgroups per CU: 5 to 40 % slower
// EDGE: 64, or 32 for the smallest outputs, whose time is a wavefront's chain of loads and the exchange of the sums: four times
// the workgroups, a quarter of the exchange, and loads three steps ahead instead of one.
template <bool A_KC, bool B_KC, typename TO, bool HAS_R, int ACT, bool F16IN, int EDGE>
__device__ __forceinline__ void small_tile(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, TO* __restrict__ C,
                                           const float* __restrict__ R, int M, int N, int K, int lda, int ldb, int ldc, int ldr, int m0,
                                           int n0, bf16_t* __restrict__ E, int lde, const bf16_t* __restrict__ bias,
                                           const float* __restrict__ out_scale) {
  constexpr int NW = SMALL_NW, PITCH = EDGE + 4, NB = EDGE / 16;   // PITCH: floats per row of a wavefront's sums
  constexpr int TILE = 32 * EDGE * 2;                  // bytes of one K-strided operand tile of one step
  constexpr int RED = EDGE * PITCH * 4, STAGE = (A_KC ? 0 : TILE) + (B_KC ? 0 : TILE);
  constexpr int AHEAD = EDGE == 64 ? 2 : 4;            // steps in registers
  static_assert(STAGE <= RED, "the staging tiles live inside the wavefront's part of the sums");
  __shared__ __attribute__((aligned(1024))) char pool[NW * RED];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  char* mine = pool + wave * RED;
  SmallOperand<A_KC, EDGE> oa;
  SmallOperand<B_KC, EDGE> ob;
  oa.init(A, lda, m0, M, lane, 0);
  ob.init(B, ldb, n0, N, lane, ACT == ACT_SWIGLU_FWD ? N >> 1 : 0);
  floatx4 acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int steps = (K + 31) / 32, per = (steps + NW - 1) / NW;
  const int t0 = wave * per, t1 = min(steps, t0 + per), k_end = min(K, t1 * 32);
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  uint4 ra[AHEAD][NB], rb[AHEAD][NB];
  auto multiply = [&](int set) {                      // set: a constant at every call
    char* tile_b = mine + (A_KC ? 0 : TILE);
    oa.put(ra[set], mine);
    ob.put(rb[set], tile_b);
    if constexpr (!A_KC || !B_KC) wave_sync();
    bf16x8 fa[NB], fb[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) { fa[i] = oa.frag(ra[set], mine, i); fb[i] = ob.frag(rb[set], tile_b, i); }
    mfma_blocks<NB, NB, NB, F16IN>(acc, fa, fb, 0);
    if constexpr (!A_KC || !B_KC) wave_sync();
  };
  if (t0 < t1) {
#pragma unroll
    for (int i = 0; i < AHEAD - 1; ++i) {
      oa.fetch(ra[i], t0 + i, k_end);
      ob.fetch(rb[i], t0 + i, k_end);
    }
    for (int t = t0; t < t1; t += AHEAD) {            // loads run AHEAD - 1 steps ahead; past the range they give zeros without a memory access
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) {
        if (i > 0 && t + i >= t1) break;
        oa.fetch(ra[(i + AHEAD - 1) % AHEAD], t + i + AHEAD - 1, k_end);
        ob.fetch(rb[(i + AHEAD - 1) % AHEAD], t + i + AHEAD - 1, k_end);
        multiply(i);
      }
    }
  }
  // block (i, j): row 16 i + (lane & 15), columns 16 j + 4 (lane >> 4) ..+3
  float* red = reinterpret_cast<float*>(mine);
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) *reinterpret_cast<floatx4*>(red + (i * 16 + (lane & 15)) * PITCH + j * 16 + (lane >> 4) * 4) = acc[i][j];
  __syncthreads();
  constexpr int CH = (ACT == ACT_SWIGLU_FWD ? EDGE / 2 : EDGE) / 8;   // 8-column chunks per row (SwiGLU forward: of features)
  for (int q = threadIdx.x; q < EDGE * CH; q += NW * 64) {
    const int row = q / CH, c = (q % CH) * 8, m = m0 + row;
    const int n = ACT == ACT_SWIGLU_FWD ? (n0 >> 1) + c : n0 + c;
    if (m >= M || n >= (ACT == ACT_SWIGLU_FWD ? N >> 1 : N)) continue;
    auto sum_waves = [&](int at, float (&v)[8]) {
      const float* p = reinterpret_cast<const float*>(pool) + row * PITCH + at;
      load_f32x8(p, v);
#pragma unroll
      for (int w = 1; w < NW; ++w) {
        float x[8];
        load_f32x8(p + w * (RED / 4), x);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += x[e];
      }
    };
    float v[8], up[8];
    sum_waves(c, v);
    add_bias8(bias, n, v);
    if constexpr (ACT == ACT_SWIGLU_FWD) {
      sum_waves(EDGE / 2 + c, up);
      add_bias8(bias, (N >> 1) + n, up);
    }
    finish8<TO, HAS_R, ACT>(v, up, m, n, N, C, ldc, R, ldr, E, lde, out_scale);
  }
}

template <bool A_KC, bool B_KC, typename TO, bool HAS_R, int ACT, bool F16IN, int EDGE>
__global__ __launch_bounds__(SMALL_NW * 64) void gemm_mfma_small_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, TO* __restrict__ C,
                                                                  const float* __restrict__ R, int M, int N, int K, int lda, int ldb, int ldc,
                                                                  int ldr, int tiles_m, int tiles_n, bf16_t* __restrict__ E, int lde,
                                                                  const bf16_t* __restrict__ bias, const float* __restrict__ out_scale) {
  int tm, tn;
  tile_coords(blockIdx.x, tiles_m, tiles_n, tm, tn);
  small_tile<A_KC, B_KC, TO, HAS_R, ACT, F16IN, EDGE>(A, B, C, R, M, N, K, lda, ldb, ldc, ldr, tm * EDGE, tn * EDGE, E, lde, bias, out_scale);
}

// Edge of the small-output tiles: 32 while there are at most two of them per CU.  us, 64 -> 32: 129 x 512 x 512 6.2 -> 4.1, x 1536 10.8 -> 6.7,
// 512 x 512 x 3072 24.7 -> 13.8, 129 x 3072 x 512 (480 tiles of 32) 6.4 -> 5.5; but 777 x 768 x 512 (600) 6.5 -> 7.3, 300 x 3072 x 512 (960) 6.8 -> 9.2.
inline long long small_tiles(int M, int N, int edge) { return (long long)((M + edge - 1) / edge) * ((N + edge - 1) / edge); }
// Below 32 rows the 64 x 64 tiles stay, not because they are faster (1 x 2048 x 2048 would go 10.1 -> 6.9, the one shape measured there) but because
// the lower estimate would take the products of a few tokens out of the split form, which the tests of that form reach through them.
inline int small_edge(int M, int N, int n_cu) { return M >= 32 && small_tiles(M, N, 32) <= 2 * n_cu ? 32 : ST; }

template <bool A_KC, bool B_KC, typename TO, bool HAS_R, int ACT, bool F16IN>
hipError_t launch_small(const GemmArgs& g, hipStream_t s) {
  const int edge = small_edge(g.M, g.N, cu_count()), tiles_m = (g.M + edge - 1) / edge, tiles_n = (g.N + edge - 1) / edge;
  const auto kernel = edge == 32 ? gemm_mfma_small_kernel<A_KC, B_KC, TO, HAS_R, ACT, F16IN, 32> : gemm_mfma_small_kernel<A_KC, B_KC, TO, HAS_R, ACT, F16IN, ST>;
  hipLaunchKernelGGL(kernel, dim3(tiles_m * tiles_n), dim3(SMALL_NW * 64), 0, s,
                     (const bf16_t*)g.A, (const bf16_t*)g.B, (TO*)g.C, g.R, g.M, g.N, g.K, g.lda, g.ldb, g.ldc, g.ldr, tiles_m, tiles_n,
                     (bf16_t*)g.E, g.lde, (const bf16_t*)g.bias, g.out_scale);
  return hipGetLastError();
}

// Estimated time (us) of the small-output kernel.  64 x 64 tiles: rounds, each bound by what one CU can have in flight
// from memory (128 rows of K at 35 GB/s) plus 1.5 us of start and store.  Measured: 512 x 3072 x 777 14.6 (the split 256-row tiles:
// 23.8), 1000 x 8192 x 1024 66 (23).  32 x 32 tiles: a wavefront's chain of loads, twice as long with two tiles on a CU: 512 x 512 x 3072
// 13.8 (the split tiles: 17.1), 129 x 512 x 3072 13.5 (13.2), 777 x 512 x 1536 11.7.
inline float small_us(int M, int N, int K, int n_cu) {
  const int edge = small_edge(M, N, n_cu);
  const long long rounds = (small_tiles(M, N, edge) + n_cu - 1) / n_cu;
  if (edge == 32) return 2.7f + (rounds > 1 ? 0.0063f : 0.0034f) * K;
  return 2.0f + (float)rounds * (1.5f + 0.0072f * K);
}

// Cut along K of a form with A K-contiguous: ranges == 0 means the small-output kernel, ranges > 1 tiles of tile_rows x 256,
// each contracted in `ranges` pieces whose fp32 planes go to the scratch and are added by splitk_finish_kernel, ranges == 1 the
// launches of full_tile_columns.  A pure function of the shape and the device for a caller whose scratch holds the planes (a
// stage's always does: gemm_mfma_plane_bytes); a smaller one gives the best cut that fits.  A call without scratch keeps the
// unsplit tiles and their bits, also where the small-output kernel, which needs none, would be faster.  tiles_only: without that kernel.
//
// A workgroup takes 0.75 us per 32-deep step with 256-row tiles and 0.55 us with 128-row ones, whether it shares the chip
// with 31 or 255 others (operands from HBM), so a grid of t tiles leaves the rest of the chip idle for K / 32 of those
// steps.  The rule compares rounds x steps x that time, plus, for a split, the planes' write and read at 8 TB/s (they mostly stay in the
// caches) and 4 us for the finishing launch.  Measured (us, unsplit -> split): 512 x 4096 x 22016 366 -> 103 (8 ranges), x 4096 68 -> 35
// (128 rows, 4), 1093 x 4096 x 22016 374 -> 178 (3), 2048 x 4096 x 22016 383 -> 303 (2), 6272 x 1280 x 5120 94 -> 86 (2),
// 512 x 12288 x 4096 74 -> 60 (2);
// 2048 x 4096 x 4096 would go 70 -> 78 and stays unsplit.
struct KSplit { int tile_rows, ranges; };
inline KSplit a_kc_split(int M, int N, int K, int n_cu, size_t ws_bytes, bool tiles_only = false) {
  constexpr float US_256 = 0.75f, US_128 = 0.55f, BASE_US = 4.0f, FINISH_US = 4.0f, PLANE_BYTES_PER_US = 8.0e6f;
  constexpr int MAX_RANGES = 12, MIN_STEPS = 8;
  const int steps = (K + DBK - 1) / DBK;
  const long long tn = (N + BN - 1) / BN;
  KSplit best{256, 1};
  if (ws_bytes == 0 || (M + 255) / 256 * tn > n_cu) return best;   // without scratch, or several rounds of full tiles
  const unsigned t256 = (unsigned)((M + 255) / 256 * tn), t128 = (unsigned)((M + 127) / 128 * tn), cus = (unsigned)n_cu;
  auto rounds = [&](unsigned wgs) { return (float)((wgs + cus - 1) / cus); };
  float cost = (2 * t256 <= cus ? rounds(t128) * US_128 : US_256) * steps;
  const float mn = (float)M * (float)N;
  for (int S = 2; S <= MAX_RANGES && steps / S >= MIN_STEPS; ++S) {
    const int per = (steps + S - 1) / S;
    if (per * (S - 1) >= steps) continue;            // fewer ranges of that depth hold all steps
    if ((size_t)S * M * N * 4 > ws_bytes) break;
    const float finish = FINISH_US + mn * (8 * S + 6) / PLANE_BYTES_PER_US;
    const float c256 = rounds(t256 * S) * per * US_256 + finish, c128 = rounds(t128 * S) * per * US_128 + finish;
    if (c256 < cost) { cost = c256; best = KSplit{256, S}; }
    if (c128 < cost) { cost = c128; best = KSplit{128, S}; }
  }
  if (!tiles_only && small_us(M, N, K, n_cu) < cost + BASE_US) best = KSplit{ST, 0};
  return best;
}

// The weight-gradient form takes the small-output kernel when that is estimated a tenth faster than its 256-row tiles (which
// need about 8 us beyond their k steps, most of it one CU storing 256 KB of fp32).
inline bool wgrad_small(int M, int N, int K, int n_cu) {
  const int t = (M + 255) / 256 * ((N + BN - 1) / BN);
  if (t > n_cu) return false;
  const int S = splitk_factor(t, K, n_cu), steps = (K + DBK - 1) / DBK, per = (steps + S - 1) / S;
  const float tile_us = 8.0f + 0.75f * per + (S > 1 ? 4.0f + (float)M * (float)N * (8 * S + 6) / 8.0e6f : 0.0f);
  return small_us(M, N, K, n_cu) < 0.9f * tile_us;
}

// ------------------------------------------------------------------------------------------
// Weight gradients of a whole task.  The 4 x layers products of W (both operands K-strided, K = the tokens of the microbatch)
// do not depend on one another, so their tiles share one launch: a product of 25 to 100 tiles no longer needs splitting along K
// to fill the chip, and every product but the last stops ending in a round of its own.  Only the tiles left over
// after the whole rounds of the group are cut along K; each range writes a compact 256 x 256 plane, added in range order.
// One iteration, product by product -> grouped: 8 layers of hidden 1280 at 6272 tokens 21.46 -> 19.73 ms (planes of 3 to 10 ranges
// per product are gone), 4 such layers on three streams 9.72 -> 8.59, a hidden-512 stage 1.374 -> 1.241; hidden 4096 at 4096 tokens,
// whose products are several rounds each, 39.1 -> 39.0.
// ------------------------------------------------------------------------------------------
constexpr int GROUP_MAX = WGRAD_GROUP_MAX;             // the list travels in the kernel arguments (1.8 KB of 4)
struct WgradProblem {
  const bf16_t* A; const bf16_t* B; float* C;
  int M, N, lda, ldb, ldc, tiles_m, tiles_n;
};
struct WgradGroup {
  int start[GROUP_MAX];                                // index of each product's first tile; INT_MAX past the last product
  WgradProblem p[GROUP_MAX];
  int K;
  int full, tail, k_split;                             // tiles contracted whole; tiles after them, cut into ranges of k_split
  float* ws;
};

// The product a tile belongs to.  No walk along the list: the arguments lie in host memory, and a chain of loads, each the next line, cost a
// launch of 16 products 5 us before its first tile.  Lane l of a wavefront keeps the start of product l, and a tile is a compare and a count
// of bits.  (All starts compared in scalar registers were some 250 instructions a tile, more than a short walk: one layer of hidden 512 at 512 tokens,
// 688 tiles of 64 x 64, walk 18.5 us, scalar 19.8, lanes 18.2; one of hidden 2048 at 32 tokens, 688 tiles of 256 x 256, 36.1, 42.4, 40.6.)
static_assert(GROUP_MAX <= 64, "a lane per product");
__device__ __forceinline__ int group_starts(const WgradGroup& g) {
  const int lane = threadIdx.x & 63;
  return lane < GROUP_MAX ? g.start[lane] : INT_MAX;
}
__device__ __forceinline__ int group_index(int starts, int tile) { return __builtin_amdgcn_readfirstlane(__popcll(__ballot(starts <= tile)) - 1); }

// Work item id: tile id for id < full, else range (id - full) / tail of tile full + (id - full) % tail.  Pointers are those of the
// item's first element; rows, cols: how much of the 256 x 256 tile the output has.
struct WgradItem {
  const bf16_t *A, *B;
  float* C;
  int a_bytes, b_bytes, lda, ldb, ldc, rows, cols, nk;
};
__device__ __forceinline__ WgradItem wgrad_item(const WgradGroup& g, int starts, int id) {
  int tile = id, range = -1, k0 = 0, K = g.K;
  if (id >= g.full) {
    range = (id - g.full) / g.tail;
    tile = g.full + (id - g.full) % g.tail;
    k0 = range * g.k_split;
    K = min(g.k_split, K - k0);
  }
  const int i = group_index(starts, tile);
  const WgradProblem& p = g.p[i];
  int tm, tn;
  tile_coords(tile - g.start[i], p.tiles_m, p.tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  WgradItem w;
  w.lda = p.lda; w.ldb = p.ldb;
  w.A = p.A + (size_t)k0 * p.lda + m0;
  w.B = p.B + (size_t)k0 * p.ldb + n0;
  w.a_bytes = (int)(((size_t)(K - 1) * p.lda + (p.M - m0)) * 2);
  w.b_bytes = (int)(((size_t)(K - 1) * p.ldb + (p.N - n0)) * 2);
  w.rows = min(BM, p.M - m0);
  w.cols = min(BN, p.N - n0);
  w.nk = (K + DBK - 1) / DBK;
  w.ldc = range < 0 ? p.ldc : BN;
  w.C = range < 0 ? p.C + (size_t)m0 * p.ldc + n0 : g.ws + ((size_t)range * g.tail + (tile - g.full)) * (BM * BN);
  return w;
}

// One K-strided operand tile of 32 k x 256 columns, as DirectLoader lays it out for the 32x32x16 reads, for a wavefront of four.
struct WgradLoader {
  const bf16_t* base;
  int bytes, k_stride;
  int voff[4];
  __device__ __forceinline__ void init(const bf16_t* p, int n_bytes, int ld, int wave, int lane) {
    base = p;
    bytes = n_bytes;
    k_stride = DBK * ld * 2;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = (i * 4 + wave) * 2 + (lane >> 5), cp = lane & 31;
      const int f = (k & 3) | (((k >> 3) & 1) << 2);
      voff[i] = (k * ld + ((((cp >> 2) ^ f) << 2) | (cp & 3)) * 8) * 2;
    }
  }
  // The wavefront's four loads of step t; a step that does not exist has no bytes, so they give zeros without a memory access.
  __device__ __forceinline__ void issue(char* tile, int t, bool exists, int wave) const {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, exists ? bytes : 0, 0x00020000);
    const int soff = exists ? t * k_stride : 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(tile + (i * 4 + wave) * 1024), 16, voff[i], soff, 0, 0);
  }
};

// A workgroup per CU walks the items blockIdx.x, + gridDim.x, ...  The steps of all its items form one sequence: the first steps of an item
// are loaded under the last MFMAs of the one before, and its sums go straight from the accumulators to memory, no LDS between.  Four
// 32 KB buffers hold a group of four steps; an item's steps are padded to whole groups with steps of zeros (1.3 us for three of them).
// While step s is contracted the loads of step s + 4 go to its own buffer: A's after the barrier in the
// middle of the step (when nobody reads that buffer any more), B's in the first half of step s + 1.  They are waited for in the
// middle of step s + 3: everything but the 16 loads of the two steps after it that were issued later.
// The stores of an item overlap little of the next one: the counter holds 63 and retires in order, so behind the 256 stores of a wavefront the
// first two steps' waits leave at most 56 of them in flight, and the third, whose B was requested after them, none.
// A is the first operand of the MFMA here: a lane holds one column, and a store instruction writes 128 contiguous bytes of two rows.
// What bounds it: at K of a few hundred the fp32 output (a CU alone stores a tile in 3.4 us, 256 at once in 11: 6 TB/s) and the operand
// reads behind the L2s, at K of thousands the matrix pipes at the power limit.  A workgroup per tile, its sums through LDS -> this, inside
// the stage: 4 layers of hidden 4096 at 256 to 512 tokens 1137 -> 979 us a launch, at 4096 tokens 5368 -> 5191; 8 layers of hidden 1280 at
// 6272 tokens 1540 -> 1519; 2 layers of hidden 2048 at 3704 tokens 652 -> 616; on another box, with group_starts, 955, 5154, 1478 and 611.
// Waiting for all but 16 of the loads and stores at every step gave half of that.  Few tokens (us, a workgroup per tile -> two groups an
// item -> this): hidden 2048 at 32 tokens 36.1 -> 40.6 -> 34.1, 1536 at 64 25.7 -> 29.0 -> 24.5, 4096 at 128 184 -> 165 -> 153; one round of tiles at one step, hidden 1024 at 32, 14.9 -> 15.5 -> 15.7 (the zeros).
__global__ __launch_bounds__(256) void gemm_mfma_wgrad_group_kernel(const WgradGroup g, int items) {
  __shared__ __attribute__((aligned(1024))) char stage0[DSTAGE];
  __shared__ __attribute__((aligned(1024))) char stage1[DSTAGE];
  __shared__ __attribute__((aligned(1024))) char stage2[DSTAGE];
  __shared__ __attribute__((aligned(1024))) char stage3[DSTAGE];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = (wave >> 1) * 128, wn = (wave & 1) * 128;
  floatx16 acc[4][4];
  auto clear = [&] {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  };
  auto multiply = [&](const Frags32<4, 4>& f) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i], f.b[j], acc[i][j], 0, 0, 0);
  };
  // LDS reads, and all but the 16 loads issued last; over_stores: but the 60 loads and stores issued last, for the first two steps of an item,
  // whose loads precede the stores of the item before
  auto wait_loads = [](bool over_stores) {
    if (over_stores) __builtin_amdgcn_s_waitcnt(0x0070 | (60 & 15) | ((60 >> 4) << 14));
    else __builtin_amdgcn_s_waitcnt(0x0070 | (16 & 15) | ((16 >> 4) << 14));
  };
  int id = blockIdx.x;
  const int starts = group_starts(g);
  WgradItem next = wgrad_item(g, starts, id);          // the item whose steps are being loaded
  WgradLoader la, lb;
  la.init(next.A, next.a_bytes, next.lda, wave, lane);
  lb.init(next.B, next.b_bytes, next.ldb, wave, lane);
  float* C = next.C;                                   // of the item that is being contracted
  int ldc = next.ldc, rows = next.rows, cols = next.cols, groups = (next.nk + 3) >> 2, t = 0;
  la.issue(stage0, 0, true, wave);
  lb.issue(stage0 + DTILE, 0, true, wave);
  la.issue(stage1, 1, 1 < next.nk, wave);
  lb.issue(stage1 + DTILE, 1, 1 < next.nk, wave);
  la.issue(stage2, 2, 2 < next.nk, wave);
  lb.issue(stage2 + DTILE, 2, 2 < next.nk, wave);
  la.issue(stage3, 3, 3 < next.nk, wave);
  lb.issue(stage3 + DTILE, 3, 3 < next.nk, wave);
  clear();
  __builtin_amdgcn_s_waitcnt(0x0070);
  stage_barrier();
  Frags32<4, 4> fx, fy;
  load_frags32<4, 4>(fx, stage0, 0, wm, wn, lane);
  load_frags32<4, 4>(fy, stage0, 1, wm, wn, lane);
  multiply(fx);
#define RRFP_W_FIRST(P, over_stores, b0, b1)                                                             \
  wait_loads(over_stores);                                                                               \
  stage_barrier();                                                                                       \
  la.issue(b0, t + (P), t + (P) < next.nk, wave);                                                        \
  load_frags32<4, 4>(fx, b1, 0, wm, wn, lane);                                                           \
  multiply(fy);                                                                                          \
  interleave_ds_vm_mfma<16, 16, 4>();                                                                    \
  __builtin_amdgcn_sched_barrier(0);
#define RRFP_W_SECOND(P, b0, b1)                                                                         \
  lb.issue(b0 + DTILE, t + (P), t + (P) < next.nk, wave);                                                \
  load_frags32<4, 4>(fy, b1, 1, wm, wn, lane);                                                           \
  multiply(fx);                                                                                          \
  interleave_ds_vm_mfma<16, 16, 4>();                                                                    \
  __builtin_amdgcn_sched_barrier(0);
  for (;;) {
    const bool only = groups == 1;
    if (groups > 1) {   // first four steps: the loads of the next two were issued before the 256 stores of the item before
      t = 4;
      RRFP_W_FIRST(0, true, stage0, stage1)
      RRFP_W_SECOND(0, stage0, stage1)
      RRFP_W_FIRST(1, true, stage1, stage2)
      RRFP_W_SECOND(1, stage1, stage2)
      RRFP_W_FIRST(2, false, stage2, stage3)
      RRFP_W_SECOND(2, stage2, stage3)
      RRFP_W_FIRST(3, false, stage3, stage0)
      RRFP_W_SECOND(3, stage3, stage0)
    }
    for (; groups > 2; --groups) {
      t += 4;
      RRFP_W_FIRST(0, false, stage0, stage1)
      RRFP_W_SECOND(0, stage0, stage1)
      RRFP_W_FIRST(1, false, stage1, stage2)
      RRFP_W_SECOND(1, stage1, stage2)
      RRFP_W_FIRST(2, false, stage2, stage3)
      RRFP_W_SECOND(2, stage2, stage3)
      RRFP_W_FIRST(3, false, stage3, stage0)
      RRFP_W_SECOND(3, stage3, stage0)
    }
    // last four steps of the item: their loads are the next item's
    id += gridDim.x;
    t = 0;
    next.nk = 0;
    if (id < items) {
      next = wgrad_item(g, starts, id);
      la.init(next.A, next.a_bytes, next.lda, wave, lane);
      lb.init(next.B, next.b_bytes, next.ldb, wave, lane);
    }
    RRFP_W_FIRST(0, only, stage0, stage1)
    RRFP_W_SECOND(0, stage0, stage1)
    RRFP_W_FIRST(1, only, stage1, stage2)
    RRFP_W_SECOND(1, stage1, stage2)
    RRFP_W_FIRST(2, false, stage2, stage3)
    RRFP_W_SECOND(2, stage2, stage3)
    RRFP_W_FIRST(3, false, stage3, stage0)
    int voff[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int col = wn + j * 32 + (lane & 31);
      voff[j] = col < cols ? ((lane >> 5) * 4 * ldc + col) * 4 : (int)0x80000000;      // past any buffer: not stored
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = wm + i * 32 + q * 8;
        // M is a multiple of 8; rows past it get a buffer of no bytes (and no offset: the range check subtracts it), so that the
        // stores are always 256
        const int pitch = row < rows ? ldc * 4 : 0;
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(C + (size_t)row * ldc, 0, row < rows ? 0x7fffffff : 0, 0x00020000);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[i][j][q * 4 + e]), rsrc, voff[j], e * pitch, 0);
      }
    if (id >= items) break;
    C = next.C;
    ldc = next.ldc;
    rows = next.rows;
    cols = next.cols;
    groups = (next.nk + 3) >> 2;
    clear();
    RRFP_W_SECOND(3, stage3, stage0)
  }
#undef RRFP_W_FIRST
#undef RRFP_W_SECOND
  __builtin_amdgcn_s_waitcnt(0x0070);                  // no load into this workgroup's LDS is left in flight
}

// Planes of the cut tiles added in range order: 16 workgroups per tile, 16 rows each.
__global__ __launch_bounds__(256) void wgrad_group_finish_kernel(const WgradGroup g, int ranges) {
  const int t = blockIdx.x >> 4, tile = g.full + t;
  const int i = group_index(group_starts(g), tile);
  const WgradProblem& p = g.p[i];
  int tm, tn;
  tile_coords(tile - g.start[i], p.tiles_m, p.tiles_n, tm, tn);
  const int c = (threadIdx.x & 63) * 4, n = tn * BN + c;
  if (n >= p.N) return;                                // N is a multiple of 8
  float4 v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int y = 0; y < ranges; ++y) {
    const float* plane = g.ws + ((size_t)y * g.tail + t) * (BM * BN) + c;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = (blockIdx.x & 15) * 16 + i * 4 + (threadIdx.x >> 6);
      if (tm * BM + row >= p.M) continue;              // not written by the planes either
      const float4 x = *reinterpret_cast<const float4*>(plane + row * BN);
      v[i].x += x.x; v[i].y += x.y; v[i].z += x.z; v[i].w += x.w;
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = tm * BM + (blockIdx.x & 15) * 16 + i * 4 + (threadIdx.x >> 6);
    if (m < p.M) *reinterpret_cast<float4*>(p.C + (size_t)m * p.ldc + n) = v[i];
  }
}

// The same list with 128 x 128 tiles, one per workgroup of four wavefronts (64 x 64 each, v_mfma_f32_32x32x16_bf16), two workgroups per CU:
// for few tokens on a chip the 256-row tiles do not fill.  What bounds it is latency (the first loads, a barrier a step, the store of the
// tile): four times the workgroups, a quarter of the store each.  32-deep steps through four 16 KB buffers, loads three steps ahead;
// both operands' tiles as in read_frag, rows of 256 bytes, 64-byte units moved by k & 3 (the k rows one pass of a transposed read meets).
constexpr int MT = 128, MTILE = 32 * MT * 2;           // tile edge; bytes of one operand of a step
struct MidLoader {
  const bf16_t* base;
  int bytes, k_stride, voff[2];
  __device__ __forceinline__ void init(const bf16_t* p, int n_bytes, int ld, int wave, int lane) {
    base = p;
    bytes = n_bytes;
    k_stride = DBK * ld * 2;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int k = (i * 4 + wave) * 4 + (lane >> 4), cp = lane & 15;
      voff[i] = (k * ld + ((((cp >> 2) ^ (k & 3)) << 2) | (cp & 3)) * 8) * 2;
    }
  }
  __device__ __forceinline__ void issue(char* tile, int t, bool exists, int wave) const {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, exists ? bytes : 0, 0x00020000);
    const int soff = exists ? t * k_stride : 0;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(tile + (i * 4 + wave) * 1024), 16, voff[i], soff, 0, 0);
  }
};
__device__ __forceinline__ bf16x8 mid_frag(const char* tile, int row0, int ks, int lane) {
  const int kb = ks * 16 + (lane >> 5) * 8 + ((lane & 15) >> 2);
  const int c = (row0 >> 3) + ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1);
  const char* p = tile + kb * (MT * 2) + (((((c >> 2) ^ (kb & 3)) << 2) | (c & 3)) << 4) + (lane & 1) * 8;
  union { short4v h[2]; bf16x8 v; } u;
  u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)p);
  u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(p + 4 * MT * 2));
  return u.v;
}
__global__ __launch_bounds__(256, 2) void gemm_mfma_wgrad_group_mid_kernel(const WgradGroup g) {
  __shared__ __attribute__((aligned(1024))) char stage0[2 * MTILE];
  __shared__ __attribute__((aligned(1024))) char stage1[2 * MTILE];
  __shared__ __attribute__((aligned(1024))) char stage2[2 * MTILE];
  __shared__ __attribute__((aligned(1024))) char stage3[2 * MTILE];
  const int i = group_index(group_starts(g), blockIdx.x);
  const WgradProblem& p = g.p[i];
  int tm, tn;
  tile_coords(blockIdx.x - g.start[i], p.tiles_m, p.tiles_n, tm, tn);
  const int m0 = tm * MT, n0 = tn * MT, K = g.K, nk = (K + DBK - 1) / DBK;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  MidLoader la, lb;
  la.init(p.A + m0, (int)(((size_t)(K - 1) * p.lda + (p.M - m0)) * 2), p.lda, wave, lane);
  lb.init(p.B + n0, (int)(((size_t)(K - 1) * p.ldb + (p.N - n0)) * 2), p.ldb, wave, lane);
  auto issue = [&](char* buf, int t) {
    la.issue(buf, t, t < nk, wave);
    lb.issue(buf + MTILE, t, t < nk, wave);
  };
  issue(stage0, 0);
  issue(stage1, 1);
  issue(stage2, 2);
  floatx16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  constexpr int VM_8 = 0x0070 | 8;                     // all but the loads of the two steps after; lgkmcnt(0)
#define RRFP_MID_STEP(cur, ahead, t)                                                                        \
  __builtin_amdgcn_s_waitcnt(VM_8);                                                                         \
  stage_barrier();                                                                                          \
  issue(ahead, (t) + 3);                                                                                    \
  _Pragma("unroll") for (int ks = 0; ks < 2; ++ks) {                                                        \
    bf16x8 fa[2], fb[2];                                                                                    \
    _Pragma("unroll") for (int i = 0; i < 2; ++i) {                                                         \
      fa[i] = mid_frag(cur, wm + i * 32, ks, lane);                                                         \
      fb[i] = mid_frag(cur + MTILE, wn + i * 32, ks, lane);                                                 \
    }                                                                                                       \
    _Pragma("unroll") for (int i = 0; i < 2; ++i)                                                           \
    _Pragma("unroll") for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0); \
  }
  for (int t = 0;; t += 4) {
    RRFP_MID_STEP(stage0, stage3, t)
    if (t + 1 >= nk) break;
    RRFP_MID_STEP(stage1, stage0, t + 1)
    if (t + 2 >= nk) break;
    RRFP_MID_STEP(stage2, stage1, t + 2)
    if (t + 3 >= nk) break;
    RRFP_MID_STEP(stage3, stage2, t + 3)
    if (t + 4 >= nk) break;
  }
#undef RRFP_MID_STEP
  __builtin_amdgcn_s_waitcnt(0x0070);                  // the zero loads of the steps past the end have landed too
  const int rows = min(MT, p.M - m0), cols = min(MT, p.N - n0);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int col = wn + j * 32 + (lane & 31);
    if (col >= cols) continue;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = wm + i * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
        if (row < rows) p.C[(size_t)(m0 + row) * p.ldc + n0 + col] = acc[i][j][e];
      }
  }
}

// The same list with 64 x 64 tiles (tile counts and starts are those of the small kernel).
__global__ __launch_bounds__(SMALL_NW * 64) void gemm_mfma_wgrad_group_small_kernel(const WgradGroup g) {
  const int i = group_index(group_starts(g), blockIdx.x);
  const WgradProblem& p = g.p[i];
  int tm, tn;
  tile_coords(blockIdx.x - g.start[i], p.tiles_m, p.tiles_n, tm, tn);
  small_tile<false, false, float, false, ACT_NONE, false, ST>(p.A, p.B, p.C, nullptr, p.M, p.N, g.K, p.lda, p.ldb, p.ldc, 0, tm * ST, tn * ST,
                                                          nullptr, 0, nullptr, nullptr);
}

// Launch of the direct-to-LDS kernel for the forms with A K-contiguous, per the cuts above.
template <bool B_KC, typename TO, bool HAS_R, int ACT, bool F16IN = false>
hipError_t launch_a_kc(const GemmArgs& g, hipStream_t s) {
  constexpr int WMv = dl_wm(true, B_KC), WNv = dl_wn(true, B_KC);
  const KSplit ks = a_kc_split(g.M, g.N, g.K, cu_count(), g.ws && !((uintptr_t)g.ws & 15) ? g.ws_bytes : 0);
  if (ks.ranges == 0) return launch_small<true, B_KC, TO, HAS_R, ACT, F16IN>(g, s);
  if (ks.ranges > 1) {
    const int steps = (g.K + DBK - 1) / DBK, k_split = (steps + ks.ranges - 1) / ks.ranges * DBK, S = (g.K + k_split - 1) / k_split;
    const int tm = (g.M + ks.tile_rows - 1) / ks.tile_rows, tn = (g.N + BN - 1) / BN;
    auto planes = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(tm * tn, S), dim3(WMv * WNv * 64), 0, s, (const bf16_t*)g.A, (const bf16_t*)g.B, (float*)g.ws,
                         (const float*)nullptr, g.M, g.N, g.K, g.lda, g.ldb, g.N, 0, tm, tn, (bf16_t*)nullptr, 0, 0, k_split,
                         (const bf16_t*)nullptr, (const float*)nullptr);
    };
    if (ks.tile_rows == 256) planes(gemm_mfma_dl_kernel<true, B_KC, float, false, WMv, WNv, ACT_NONE, 256, F16IN>);
    else planes(gemm_mfma_dl_kernel<true, B_KC, float, false, WMv, WNv, ACT_NONE, 128, F16IN>);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    const size_t threads = (size_t)g.M * ((ACT == ACT_SWIGLU_FWD ? g.N / 2 : g.N) / 8);
    hipLaunchKernelGGL((splitk_finish_kernel<TO, HAS_R, ACT>), dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, (const float*)g.ws,
                       S, g.M, g.N, (TO*)g.C, g.ldc, g.R, g.ldr, (bf16_t*)g.E, g.lde, (const bf16_t*)g.bias, g.out_scale);
    return hipGetLastError();
  }
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  const int cn = full_tile_columns(tiles_m, tiles_n, cu_count());
  if (cn > 0)
    hipLaunchKernelGGL((gemm_mfma_dl_kernel<true, B_KC, TO, HAS_R, WMv, WNv, ACT, 256, F16IN>), dim3(tiles_m * cn), dim3(WMv * WNv * 64),
                       0, s, (const bf16_t*)g.A, (const bf16_t*)g.B, (TO*)g.C, g.R, g.M, g.N, g.K, g.lda, g.ldb, g.ldc,
                       g.ldr, tiles_m, cn, (bf16_t*)g.E, g.lde, 0, 0, (const bf16_t*)g.bias, g.out_scale);
  if (cn < tiles_n) {
    const int tiles_m2 = (g.M + 127) / 128;
    hipLaunchKernelGGL((gemm_mfma_dl_kernel<true, B_KC, TO, HAS_R, WMv, WNv, ACT, 128, F16IN>), dim3(tiles_m2 * (tiles_n - cn)),
                       dim3(WMv * WNv * 64), 0, s, (const bf16_t*)g.A, (const bf16_t*)g.B, (TO*)g.C, g.R, g.M, g.N, g.K,
                       g.lda, g.ldb, g.ldc, g.ldr, tiles_m2, tiles_n - cn, (bf16_t*)g.E, g.lde, cn, 0, (const bf16_t*)g.bias, g.out_scale);
  }
  return hipGetLastError();
}

// How the group is cut: estimated times as in a_kc_split, 8 us a round of 256-row tiles beyond its k steps.
// ranges = 0: the small-output kernel, -1: 128 x 128 tiles.  A pure function of the shapes, the device and the scratch.
// The 128 x 128 tiles are for short contractions.  Up to 320 tokens while one round of them (two per CU, 3/4 full) replaces 256-row tiles that
// leave CUs idle or 64 x 64 ones past a round.  Measured (us, else -> 128 x 128): 2 layers of hidden 512 at 32 / 128 / 300 tokens 11.6 -> 9.7,
// 11.9 -> 11.3, 16.2 -> 15.5, 4 of hidden 256 12.3 -> 8.3, 13.3 -> 9.4, 16.8 -> 12.8.  Past 320 it depends on the list: 172 tiles of 128 x 128 still
// win at 640 (22.0 -> 19.9), 88 lose from 512 on (12.8 -> 13.8), 344 tie.  But 4 of hidden 512 at 40 (736 tiles) 14.9 -> 16.5, 1 of hidden 256
// at 40 (192 tiles of 64 x 64) 5.6 -> 7.5.  Up to 64 tokens also where the 256-row tiles would need a second round of up to half the CUs: 2 of
// hidden 1024 at 32 / 64 22.2 -> 21.3, 22.8 -> 23.0, with GELU 24.2 -> 22.2, 24.5 -> 23.1; 8 of hidden 512 24.1 -> 23.4, 24.8 -> 26.7.  From there it loses:
// at 128 23.6 -> 27.2, 25.0 -> 26.8, 25.9 -> 33.0.
struct GroupCut { int full, tail, ranges; };
inline GroupCut wgrad_group_cut(long long t256, long long t128, long long t64, int K, int n_cu, size_t ws_bytes) {
  if ((K <= 320 && t64 > n_cu && 2 * t128 <= 3 * n_cu) || (K <= 64 && t256 > n_cu && 2 * t256 <= 3 * n_cu)) return GroupCut{(int)t128, 0, -1};
  constexpr float US_STEP = 0.75f, US_ROUND = 8.0f, FINISH_US = 4.0f, PLANE_BYTES_PER_US = 8.0e6f;
  constexpr int MAX_RANGES = 16, MIN_STEPS = 8;
  const int steps = (K + DBK - 1) / DBK, r = (int)(t256 % n_cu);
  GroupCut best{(int)t256, 0, 1};
  const float whole = (float)(t256 / n_cu) * (US_ROUND + US_STEP * steps);
  float cost = r ? US_ROUND + US_STEP * steps : 0.0f;  // of the last round
  for (int S = 2; r && S <= MAX_RANGES && steps / S >= MIN_STEPS; ++S) {
    const int per = (steps + S - 1) / S;
    if (per * (S - 1) >= steps) continue;            // fewer ranges of that depth hold all steps
    if ((size_t)S * r * BM * BN * 4 > ws_bytes) break;
    const float c = (float)((unsigned)(r * S + n_cu - 1) / (unsigned)n_cu) * (US_ROUND + US_STEP * per) + FINISH_US + (float)r * (BM * BN) * (8 * S + 6) / PLANE_BYTES_PER_US;
    if (c < cost) { cost = c; best = GroupCut{(int)(t256 - r), r, S}; }
  }
  const float small = 2.0f + (float)((t64 + n_cu - 1) / n_cu) * (1.5f + 0.0072f * K);
  if (small < 0.9f * (whole + cost)) best = GroupCut{(int)t64, 0, 0};
  return best;
}

// Tiles of edge x edge of all products of a group.
inline long long group_tiles(const GemmArgs* g, int n, int edge) {
  long long t = 0;
  for (int i = 0; i < n; ++i) t += (long long)((g[i].M + edge - 1) / edge) * ((g[i].N + edge - 1) / edge);
  return t;
}

hipError_t launch_wgrad_group_mfma(const GemmArgs* g, int n, hipStream_t s) {
  WgradGroup grp{};
  grp.K = g[0].K;
  const bool ws = g[0].ws && !((uintptr_t)g[0].ws & 15);
  const GroupCut cut = wgrad_group_cut(group_tiles(g, n, BM), group_tiles(g, n, MT), group_tiles(g, n, ST), grp.K, cu_count(), ws ? g[0].ws_bytes : 0);
  const int edge = cut.ranges == 0 ? ST : cut.ranges < 0 ? MT : BM;
  for (int i = 0; i < GROUP_MAX; ++i) grp.start[i] = i < n ? (int)group_tiles(g, i, edge) : INT_MAX;
  for (int i = 0; i < n; ++i)
    grp.p[i] = WgradProblem{(const bf16_t*)g[i].A, (const bf16_t*)g[i].B, (float*)g[i].C, g[i].M, g[i].N, g[i].lda, g[i].ldb, g[i].ldc,
                            (g[i].M + edge - 1) / edge, (g[i].N + edge - 1) / edge};
  if (edge == MT) {
    hipLaunchKernelGGL(gemm_mfma_wgrad_group_mid_kernel, dim3(cut.full), dim3(256), 0, s, grp);
    return hipGetLastError();
  }
  if (edge == ST) {
    hipLaunchKernelGGL(gemm_mfma_wgrad_group_small_kernel, dim3(cut.full), dim3(SMALL_NW * 64), 0, s, grp);
    return hipGetLastError();
  }
  const int steps = (grp.K + DBK - 1) / DBK;
  grp.full = cut.full;
  grp.tail = cut.tail;
  grp.k_split = (steps + cut.ranges - 1) / cut.ranges * DBK;
  grp.ws = (float*)g[0].ws;
  const int items = cut.full + cut.tail * cut.ranges;
  hipLaunchKernelGGL(gemm_mfma_wgrad_group_kernel, dim3(std::min(items, cu_count())), dim3(256), 0, s, grp, items);
  if (hipError_t e = hipGetLastError(); e != hipSuccess || cut.tail == 0) return e;
  hipLaunchKernelGGL(wgrad_group_finish_kernel, dim3(cut.tail * 16), dim3(256), 0, s, grp, cut.ranges);
  return hipGetLastError();
}

template <bool A_KC, bool B_KC, typename TO, bool HAS_R>
hipError_t launch_one(const GemmArgs& g, hipStream_t s) {
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  if (direct_ok(g)) {
    if constexpr (A_KC) return launch_a_kc<B_KC, TO, HAS_R, ACT_NONE>(g, s);
    // Weight-gradient form as a single call (both operands K-strided, fp32 out, K = tokens): when the output has too
    // few tiles to fill the CUs, the contraction is split into S ranges, every range writes its own
    // partial plane into the scratch, and the planes are summed in range order (one fixed order).
    if constexpr (!A_KC && !B_KC && !HAS_R && sizeof(TO) == 4) {
      if (g.ws && wgrad_small(g.M, g.N, g.K, cu_count())) return launch_small<false, false, float, false, ACT_NONE, false>(g, s);
      const int S = splitk_factor(tiles_m * tiles_n, g.K, cu_count());
      if (S > 1 && g.ws && g.ldc == g.N && (size_t)S * g.M * g.N * 4 <= g.ws_bytes && ((size_t)g.M * g.N) % 4 == 0) {
        const int steps = (g.K + DBK - 1) / DBK, k_split = (steps + S - 1) / S * DBK;
        const int S_eff = (g.K + k_split - 1) / k_split;
        hipLaunchKernelGGL((gemm_mfma_dl_kernel<A_KC, B_KC, TO, HAS_R, dl_wm(A_KC, B_KC), dl_wn(A_KC, B_KC), ACT_NONE>),
                           dim3(tiles_m * tiles_n, S_eff), dim3(dl_wm(A_KC, B_KC) * dl_wn(A_KC, B_KC) * 64), 0,
                           s, (const bf16_t*)g.A, (const bf16_t*)g.B, (TO*)g.ws, g.R, g.M, g.N, g.K, g.lda,
                           g.ldb, g.ldc, g.ldr, tiles_m, tiles_n, (bf16_t*)nullptr, 0, 0, k_split, (const bf16_t*)nullptr, (const float*)nullptr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_grad_reduce((const float*)g.ws, (size_t)g.M * g.N, S_eff, (float*)g.C, (size_t)g.M * g.N, s);
      }
      const int cn = wgrad_full_tile_columns(g, tiles_m, tiles_n, cu_count(), g.ws != nullptr);
      if (cn < tiles_n && wgrad_tail_scratch_bytes(g, cn) <= g.ws_bytes && ((uintptr_t)g.ws & 15) == 0) {
        constexpr int WMv = dl_wm(A_KC, B_KC), WNv = dl_wn(A_KC, B_KC);
        const int ct = tiles_n - cn, width = g.N - cn * BN;
        const int steps = (g.K + DBK - 1) / DBK, k_split = (steps + TAIL_SPLIT - 1) / TAIL_SPLIT * DBK;
        hipLaunchKernelGGL((gemm_mfma_dl_kernel<A_KC, B_KC, TO, HAS_R, WMv, WNv, ACT_NONE>), dim3(tiles_m * cn), dim3(WMv * WNv * 64), 0,
                           s, (const bf16_t*)g.A, (const bf16_t*)g.B, (TO*)g.C, g.R, g.M, g.N, g.K, g.lda, g.ldb, g.ldc, g.ldr,
                           tiles_m, cn, (bf16_t*)nullptr, 0, 0, 0, (const bf16_t*)nullptr, (const float*)nullptr);
        // the tail's planes are compact ([M, width]); the kernel addresses columns by their index in C, so the
        // plane pointer is moved left by the tail's first column (never dereferenced outside the planes)
        float* ws_shifted = (float*)g.ws - (size_t)cn * BN;
        hipLaunchKernelGGL((gemm_mfma_dl_kernel<A_KC, B_KC, TO, HAS_R, WMv, WNv, ACT_NONE>), dim3(tiles_m * ct, TAIL_SPLIT),
                           dim3(WMv * WNv * 64), 0, s, (const bf16_t*)g.A, (const bf16_t*)g.B, (TO*)ws_shifted, g.R, g.M, g.N, g.K,
                           g.lda, g.ldb, width, g.ldr, tiles_m, ct, (bf16_t*)nullptr, 0, cn, k_split, (const bf16_t*)nullptr, (const float*)nullptr);
        const size_t n4 = (size_t)g.M * (width / 4);
        hipLaunchKernelGGL(splitk_tail_reduce_kernel, dim3((unsigned)std::min<size_t>((n4 + 255) / 256, 8192)), dim3(256), 0, s,
                           (const float*)g.ws, TAIL_SPLIT, g.M, width, (float*)g.C + (size_t)cn * BN, g.ldc, width);
        return hipGetLastError();
      }
    }
    hipLaunchKernelGGL((gemm_mfma_dl_kernel<A_KC, B_KC, TO, HAS_R, dl_wm(A_KC, B_KC), dl_wn(A_KC, B_KC), ACT_NONE>),
                       dim3(tiles_m * tiles_n), dim3(dl_wm(A_KC, B_KC) * dl_wn(A_KC, B_KC) * 64), 0,
                       s, (const bf16_t*)g.A, (const bf16_t*)g.B, (TO*)g.C, g.R, g.M, g.N, g.K, g.lda,
                       g.ldb, g.ldc, g.ldr, tiles_m, tiles_n, (bf16_t*)nullptr, 0, 0, 0, (const bf16_t*)g.bias, g.out_scale);
    return hipGetLastError();
  }
  static std::once_flag once;       // per instantiation; the attribute is process-wide for the function
  static hipError_t once_status = hipSuccess;
  if (hipError_t e = set_max_dynamic_lds_once(once, once_status, (const void*)gemm_mfma_kernel<A_KC, B_KC, TO, HAS_R>, SMEM_BYTES);
      e != hipSuccess) return e;
  hipLaunchKernelGGL((gemm_mfma_kernel<A_KC, B_KC, TO, HAS_R>), dim3(tiles_m * tiles_n), dim3(NTHREADS), SMEM_BYTES, s,
                     (const bf16_t*)g.A, (const bf16_t*)g.B, (TO*)g.C, g.R, g.M, g.N, g.K, g.lda, g.ldb,
                     g.ldc, g.ldr, tiles_m, tiles_n);
  return hipGetLastError();
}

template <bool A_KC, bool B_KC>
hipError_t launch_orient(const GemmArgs& g, hipStream_t s) {
  if (g.out_dtype == F32) return g.R ? launch_one<A_KC, B_KC, float, true>(g, s) : launch_one<A_KC, B_KC, float, false>(g, s);
  return g.R ? launch_one<A_KC, B_KC, bf16_t, true>(g, s) : launch_one<A_KC, B_KC, bf16_t, false>(g, s);
}

}  // namespace

// Fused-activation launch: forward forms are (A K-contiguous, B K-strided), backward forms (both K-contiguous).
template <bool B_KC, int ACT>
hipError_t launch_act(const GemmArgs& g, hipStream_t s) {
  return launch_a_kc<B_KC, bf16_t, false, ACT>(g, s);
}

int device_cu_count() { return cu_count(); }

bool gemm_mfma_act_supported(const GemmArgs& g) {
  if (g.act == ACT_NONE) return true;
  if (!gemm_mfma_supports(g) || !direct_ok(g) || g.R || g.out_dtype != BF16 || !g.E || (g.lde & 7) ||
      ((uintptr_t)g.E & 15) || g.transA)
    return false;
  static_assert(dl_wm(true, false) == 2 && dl_wn(true, false) == 4 && dl_wn(true, true) == 4, "epilogue pairing assumes 2x4 wavefronts");
  switch (g.act) {
    case ACT_SWIGLU_FWD: return !g.transB && (g.N % 256) == 0;          // F a multiple of 128: whole paired tiles
    case ACT_GELU_FWD: return !g.transB;
    case ACT_SWIGLU_BWD: case ACT_GELU_BWD: return g.transB;
    default: return false;
  }
}

// How launch_gemm_mfma would cut g (without an activation) on a device with n_cu compute units and ws_bytes of scratch: the
// same decisions as the launchers above, without touching the device.
GemmPlan gemm_mfma_plan(const GemmArgs& g, int n_cu, size_t ws_bytes) {
  GemmPlan p{};
  if (!gemm_mfma_supports(g)) return p;
  const bool a_kc = !g.transA, b_kc = g.transB;
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  p.wavefronts = direct_ok(g) ? dl_wm(a_kc, b_kc) * dl_wn(a_kc, b_kc) : NTHREADS / 64;
  p.split_k = 1;
  if (!direct_ok(g)) {
    p.kernel = 2;
    p.main_workgroups = tiles_m * tiles_n;
    return p;
  }
  p.kernel = 1;
  auto small_plan = [&] {
    p.kernel = 3;
    p.wavefronts = SMALL_NW;
    p.main_workgroups = (int)small_tiles(g.M, g.N, small_edge(g.M, g.N, n_cu));
    return p;
  };
  if (a_kc) {
    const KSplit ks = a_kc_split(g.M, g.N, g.K, n_cu, ws_bytes);
    if (ks.ranges == 0) return small_plan();
    if (ks.ranges > 1) {
      const int wgs = (g.M + ks.tile_rows - 1) / ks.tile_rows * tiles_n;
      p.main_workgroups = ks.tile_rows == 256 ? wgs : 0;
      p.short_workgroups = ks.tile_rows == 256 ? 0 : wgs;
      p.split_k = ks.ranges;
      return p;
    }
    const int cn = full_tile_columns(tiles_m, tiles_n, n_cu);
    p.main_workgroups = tiles_m * cn;
    p.short_workgroups = ((g.M + 127) / 128) * (tiles_n - cn);
    return p;
  }
  p.main_workgroups = tiles_m * tiles_n;
  if (!b_kc && !g.R && g.out_dtype == F32 && ws_bytes > 0) {
    if (wgrad_small(g.M, g.N, g.K, n_cu)) return small_plan();
    const int S = (g.ldc == g.N && ((size_t)g.M * g.N) % 4 == 0) ? splitk_factor(tiles_m * tiles_n, g.K, n_cu) : 1;
    if (S > 1 && (size_t)S * g.M * g.N * 4 <= ws_bytes) {
      const int steps = (g.K + DBK - 1) / DBK, k_split = (steps + S - 1) / S * DBK;
      p.split_k = (g.K + k_split - 1) / k_split;
    } else {
      const int cn = wgrad_full_tile_columns(g, tiles_m, tiles_n, n_cu, true);
      if (cn < tiles_n && wgrad_tail_scratch_bytes(g, cn) <= ws_bytes) {   // plain launch over cn tile columns + a tail launch split along K
        p.main_workgroups = tiles_m * cn;
        p.short_workgroups = tiles_m * (tiles_n - cn) * TAIL_SPLIT;
        p.split_k = TAIL_SPLIT;
      }
    }
  }
  return p;
}

bool gemm_mfma_supports(const GemmArgs& g) {
  if (g.in_dtype != BF16 && g.in_dtype != F16) return false;
  if (g.in_dtype == F16 || g.out_dtype == F16) {
    // half forms: QKV projection (half x half -> half, NN), output projection (half x half -> fp32 + residual, NN)
    // and dO (bf16 x bf16 -> half, NT); direct-load kernel only
    const bool qkv_form = g.in_dtype == F16 && g.out_dtype == F16 && !g.transA && !g.transB && !g.R;
    const bool wo_form = g.in_dtype == F16 && g.out_dtype == F32 && !g.transA && !g.transB && g.R;
    const bool do_form = g.in_dtype == BF16 && g.out_dtype == F16 && !g.transA && g.transB && !g.R;
    if (!(qkv_form || wo_form || do_form) || g.act != ACT_NONE || !direct_ok(g)) return false;
  }
  if (g.bias && (!direct_ok(g) || ((uintptr_t)g.bias & 15))) return false;   // bias lives in the direct-load kernel's epilogue
  if (g.M < 1 || g.N < 1 || g.K < 1) return false;
  if ((g.lda | g.ldb | g.ldc) & 7) return false;
  if (g.R && ((g.ldr & 3) || ((uintptr_t)g.R & 15))) return false;
  if (g.N & 7) return false;
  const bool a_kc = !g.transA, b_kc = g.transB;
  if ((a_kc || b_kc) && (g.K & 7)) return false;      // K-contiguous chunks must be whole
  if (!a_kc && (g.M & 7)) return false;               // K-strided A: rows of C come in chunks of 8
  auto aligned = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  return aligned(g.A) && aligned(g.B) && aligned(g.C);
}

bool gemm_mfma_wgrad_groupable(const GemmArgs& g) {
  return g.transA && !g.transB && !g.R && !g.bias && g.act == ACT_NONE && g.in_dtype == BF16 && g.out_dtype == F32 && gemm_mfma_supports(g) &&
         direct_ok(g) && !(g.ldc & 3) && (long long)((g.M + ST - 1) / ST) * ((g.N + ST - 1) / ST) < (1 << 24);
}

// The rows enter the cut through the counts of 128- and 256-row tiles and, smoothly, through the cost of adding the planes,
// which only speaks for fewer ranges as the rows grow: within 128 rows the first one takes the most ranges.
size_t gemm_mfma_plane_bytes(int max_M, int N, int K, int n_cu) {
  size_t most = 0;
  for (int M = 1; M <= max_M && (long long)((M + 255) / 256) * ((N + BN - 1) / BN) <= n_cu; M += 128) {
    const KSplit ks = a_kc_split(M, N, K, n_cu, ~(size_t)0, true);
    if (ks.ranges > 1) most = std::max(most, (size_t)ks.ranges * std::min(M + 127, max_M) * N * 4);
  }
  return most;
}

// Of the lengths of one 32-deep step the longest is the last to go to the 64 x 64 or 128 x 128 tiles (whose limits are whole steps); else the cut
// is that of the step.
size_t gemm_mfma_wgrad_plane_bytes(const GemmArgs* g, int n, int min_K, int max_K, int n_cu) {
  const long long t256 = group_tiles(g, n, BM), t128 = group_tiles(g, n, MT), t64 = group_tiles(g, n, ST);
  size_t most = 0;
  for (int step = (min_K - 1) / DBK; step * DBK < max_K; ++step) {
    const GroupCut cut = wgrad_group_cut(t256, t128, t64, std::min((step + 1) * DBK, max_K), n_cu, ~(size_t)0);
    if (cut.ranges > 1) most = std::max(most, (size_t)cut.ranges * cut.tail * BM * BN * 4);
  }
  return most;
}

WgradGroupPlan gemm_mfma_wgrad_group_plan(const GemmArgs* g, int n, int n_cu, size_t ws_bytes) {
  const GroupCut cut = wgrad_group_cut(group_tiles(g, n, BM), group_tiles(g, n, MT), group_tiles(g, n, ST), g[0].K, n_cu, ws_bytes);
  return WgradGroupPlan{cut.full, cut.tail, cut.ranges, cut.ranges > 1 ? (size_t)cut.ranges * cut.tail * BM * BN * 4 : 0};
}

hipError_t launch_gemm_mfma_wgrad_group(const GemmArgs* g, int n, hipStream_t s) {
  for (int i = 0; i < n; i += GROUP_MAX)
    if (hipError_t e = launch_wgrad_group_mfma(g + i, std::min(GROUP_MAX, n - i), s); e != hipSuccess) return e;
  return hipSuccess;
}

hipError_t launch_gemm_mfma(const GemmArgs& g, hipStream_t s) {
  if (!gemm_mfma_supports(g)) return hipErrorInvalidValue;
  if (g.act != ACT_NONE) {
    if (!gemm_mfma_act_supported(g)) return hipErrorInvalidValue;
    switch (g.act) {
      case ACT_SWIGLU_FWD: return launch_act<false, ACT_SWIGLU_FWD>(g, s);
      case ACT_GELU_FWD: return launch_act<false, ACT_GELU_FWD>(g, s);
      case ACT_SWIGLU_BWD: return launch_act<true, ACT_SWIGLU_BWD>(g, s);
      default: return launch_act<true, ACT_GELU_BWD>(g, s);
    }
  }
  const bool a_kc = !g.transA, b_kc = g.transB;
  if (g.in_dtype == F16 && g.out_dtype == F32) return launch_a_kc<false, float, true, ACT_NONE, true>(g, s);
  if (g.in_dtype == F16) return launch_a_kc<false, f16_t, false, ACT_NONE, true>(g, s);
  if (g.out_dtype == F16) return launch_a_kc<true, f16_t, false, ACT_NONE, false>(g, s);
  if (a_kc && !b_kc) return launch_orient<true, false>(g, s);
  if (a_kc && b_kc) return launch_orient<true, true>(g, s);
  if (!a_kc && !b_kc) return launch_orient<false, false>(g, s);
  return launch_orient<false, true>(g, s);
}

}  // namespace rrfp
