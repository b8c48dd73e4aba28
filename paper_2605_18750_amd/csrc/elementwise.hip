// HBM-bound kernels of the stage tasks: RMSNorm forward/backward, SwiGLU and GELU
// forward/backward, the fixed-order column sum for norm-gain gradients and the
// index-ordered gradient reduction.  All arithmetic is fp32; storage is fp32 or bf16.
// None of these kernels uses atomics: every sum has one fixed order.
#include <algorithm>

#include "kernels.h"
#include "numeric.h"

namespace rrfp {
namespace {

constexpr int WAVE = 64;

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}

// Vec<T>::N consecutive fp32 values (the residual stream is fp32 whatever the storage type).
template <int V>
__device__ inline void load_f32(const float* p, float* out) {
#pragma unroll
  for (int i = 0; i < V; i += 4) {
    const float4 v = *reinterpret_cast<const float4*>(p + i);
    out[i] = v.x; out[i + 1] = v.y; out[i + 2] = v.z; out[i + 3] = v.w;
  }
}
template <int V>
__device__ inline void store_f32(float* p, const float* in) {
#pragma unroll
  for (int i = 0; i < V; i += 4) *reinterpret_cast<float4*>(p + i) = make_float4(in[i], in[i + 1], in[i + 2], in[i + 3]);
}

// ---------------------------------------------------------------- storage type -> fp32 copy
// copy, when given, also receives the values unchanged, and partial the largest magnitude each workgroup met (one read of src serves
// all outputs; a maximum has no summation order, so the result does not depend on how the work was cut).
// words: as many 32-bit words copied along, from pinned host memory: what a task brings with it costs no launch of its own (two copies of
// 2.4 us a forward task before).
template <typename T>
__global__ __launch_bounds__(256) void widen_kernel(const T* __restrict__ src, float* __restrict__ dst, size_t n, T* __restrict__ copy,
                                                    float* __restrict__ partial, const int* __restrict__ words_src, int* __restrict__ words_dst,
                                                    int words) {
  constexpr int V = Vec<T>::N;
  __shared__ float red[4];
  const size_t nv = n / V, first = (size_t)blockIdx.x * 256 + threadIdx.x, stride = (size_t)gridDim.x * 256;
  for (size_t i = first; i < (size_t)words; i += stride) words_dst[i] = words_src[i];
  float mx = 0.f;
  for (size_t i = first; i < nv; i += stride) {
    float v[V];
    load_vec<T>(src + i * V, v);
    store_f32<V>(dst + i * V, v);
    if (copy) store_vec<T>(copy + i * V, v);     // widening and rounding back is the identity
#pragma unroll
    for (int e = 0; e < V; ++e) mx = fmaxf(mx, fabsf(v[e]));      // fmaxf drops NaNs: a NaN in dy shows in the results, not here
  }
  for (size_t i = nv * V + first; i < n; i += stride) {
    const float v = to_float(src[i]);
    dst[i] = v;
    if (copy) copy[i] = src[i];
    mx = fmaxf(mx, fabsf(v));
  }
  if (!partial) return;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, WAVE));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) partial[blockIdx.x] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// ---------------------------------------------------------------- gradient scale
// from the workgroups' maxima of widen_kernel
__global__ __launch_bounds__(256) void grad_scale_kernel(const float* __restrict__ partial, int n_partial, float* __restrict__ scale) {
  __shared__ float red[4];
  float mx = 0.f;
  for (int i = threadIdx.x; i < n_partial; i += 256) mx = fmaxf(mx, partial[i]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, WAVE));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    float s = 1.0f;
    if (mx > 0.f && mx < INFINITY) {
      int ex;
      frexpf(mx, &ex);                               // mx = f * 2^ex, f in [0.5, 1)
      ex = max(-100, min(100, ex - 1));              // 2^ex <= mx < 2^(ex+1)
      s = ldexpf(1.0f, -ex);                         // s * mx in [1, 2)
    }
    scale[0] = s;
    scale[1] = 1.0f / s;                             // exact: s is a power of two
  }
}

// ---------------------------------------------------------------- RMSNorm forward
// One wavefront per row; 4 rows per workgroup.  Two sweeps over the row (the second is
// served by cache): sum of squares, then scale.  x is the fp32 residual stream.
// h16, when given (bf16 storage only), receives the same values rounded to IEEE half: the copy the QKV
// projection reads (the bf16 one then serves the weight-gradient GEMM, whose other operand is a bf16 gradient).
template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_fwd_kernel(const float* __restrict__ x, const T* __restrict__ g,
                                                          T* __restrict__ h, float* __restrict__ r_out,
                                                          int Tn, int H, float eps, f16_t* __restrict__ h16) {
  constexpr int V = Vec<T>::N;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= Tn) return;
  const float* xr = x + (size_t)row * H;
  T* hr = h + (size_t)row * H;
  float ss = 0.f;
  const bool vec = (H % V) == 0;
  if (vec) {
    for (int c = lane * V; c < H; c += WAVE * V) {
      float v[V];
      load_f32<V>(xr + c, v);
#pragma unroll
      for (int i = 0; i < V; ++i) ss += v[i] * v[i];
    }
  } else {
    for (int c = lane; c < H; c += WAVE) { float v = xr[c]; ss += v * v; }
  }
  ss = wave_sum(ss);
  const float r = 1.0f / sqrtf(ss / (float)H + eps);
  if (lane == 0) r_out[row] = r;
  if (vec) {
    for (int c = lane * V; c < H; c += WAVE * V) {
      float v[V], gv[V];
      load_f32<V>(xr + c, v);
      load_vec<T>(g + c, gv);
#pragma unroll
      for (int i = 0; i < V; ++i) v[i] = v[i] * r * gv[i];
      store_vec<T>(hr + c, v);
      if constexpr (V == 8) {
        if (h16) store_vec<f16_t>(h16 + (size_t)row * H + c, v);
      }
    }
  } else {
    for (int c = lane; c < H; c += WAVE) {
      const float v = xr[c] * r * to_float(g[c]);
      hr[c] = from_float<T>(v);
      if (h16) h16[(size_t)row * H + c] = from_float<f16_t>(v);
    }
  }
}

// The same for rows of up to NV * 64 vectors (H % Vec<T>::N == 0): the row is read once, all its loads issued
// before the first use, and stays in registers between the two sweeps.  Same arithmetic in the same order as the
// kernel above (bit-identical results).
template <typename T, int NV>
__global__ __launch_bounds__(256) void rmsnorm_fwd_rows_kernel(const float* __restrict__ x, const T* __restrict__ g,
                                                               T* __restrict__ h, float* __restrict__ r_out,
                                                               int Tn, int H, float eps, f16_t* __restrict__ h16) {
  constexpr int V = Vec<T>::N;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= Tn) return;
  const float* xr = x + (size_t)row * H;
  float a[NV][V];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int c = (v * WAVE + lane) * V;
    if (c < H) load_f32<V>(xr + c, a[v]);
  }
  float ss = 0.f;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    if ((v * WAVE + lane) * V < H) {
#pragma unroll
      for (int i = 0; i < V; ++i) ss += a[v][i] * a[v][i];
    }
  }
  ss = wave_sum(ss);
  const float r = 1.0f / sqrtf(ss / (float)H + eps);
  if (lane == 0) r_out[row] = r;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int c = (v * WAVE + lane) * V;
    if (c < H) {
      float gv[V];
      load_vec<T>(g + c, gv);
#pragma unroll
      for (int i = 0; i < V; ++i) a[v][i] = a[v][i] * r * gv[i];
      store_vec<T>(h + (size_t)row * H + c, a[v]);
      if constexpr (V == 8) {
        if (h16) store_vec<f16_t>(h16 + (size_t)row * H + c, a[v]);
      }
    }
  }
}

// ---------------------------------------------------------------- RMSNorm backward, rows
// dx = add_in + r * (w - xhat * mean(w * xhat)),  w = dh * g,  xhat = x * r.
// dh (a GEMM output consumed only here), x and add_in (residual stream) are fp32.  dx goes to out32 (fp32, next link of the residual-gradient
// chain) and/or out_t (storage type: GEMM operand, or the task's dx output); either may be null.
template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_bwd_rows_kernel(const float* __restrict__ dh, const float* __restrict__ x,
                                                               const float* __restrict__ r, const T* __restrict__ g,
                                                               const float* __restrict__ add_in, float* __restrict__ out32,
                                                               T* __restrict__ out_t, int Tn, int H) {
  constexpr int V = Vec<T>::N;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= Tn) return;
  const size_t off = (size_t)row * H;
  const float rr = r[row];
  float dot = 0.f;
  const bool vec = (H % V) == 0;
  if (vec) {
    for (int c = lane * V; c < H; c += WAVE * V) {
      float a[V], b[V], gv[V];
      load_f32<V>(dh + off + c, a);
      load_f32<V>(x + off + c, b);
      load_vec<T>(g + c, gv);
#pragma unroll
      for (int i = 0; i < V; ++i) dot += a[i] * gv[i] * (b[i] * rr);
    }
  } else {
    for (int c = lane; c < H; c += WAVE) dot += dh[off + c] * to_float(g[c]) * (x[off + c] * rr);
  }
  dot = wave_sum(dot) / (float)H;
  if (vec) {
    for (int c = lane * V; c < H; c += WAVE * V) {
      float a[V], b[V], gv[V], ad[V];
      load_f32<V>(dh + off + c, a);
      load_f32<V>(x + off + c, b);
      load_vec<T>(g + c, gv);
      load_f32<V>(add_in + off + c, ad);
#pragma unroll
      for (int i = 0; i < V; ++i) a[i] = ad[i] + rr * (a[i] * gv[i] - (b[i] * rr) * dot);
      if (out32) store_f32<V>(out32 + off + c, a);
      if (out_t) store_vec<T>(out_t + off + c, a);
    }
  } else {
    for (int c = lane; c < H; c += WAVE) {
      const float w = dh[off + c] * to_float(g[c]);
      const float v = add_in[off + c] + rr * (w - (x[off + c] * rr) * dot);
      if (out32) out32[off + c] = v;
      if (out_t) out_t[off + c] = from_float<T>(v);
    }
  }
}

// ---------------------------------------------------------------- RMSNorm backward, gain partials
// partial[chunk][c] = sum over the chunk's rows (ascending) of dh[t][c] * x[t][c] * r[t].
template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_bwd_gain_kernel(const float* __restrict__ dh, const float* __restrict__ x,
                                                               const float* __restrict__ r, float* __restrict__ partial,
                                                               int Tn, int H) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  const int chunk = blockIdx.y;
  if (c >= H) return;
  const int t0 = chunk * NORM_BWD_ROWS;
  const int t1 = min(t0 + NORM_BWD_ROWS, Tn);
  float acc = 0.f;
  for (int t = t0; t < t1; ++t) acc += dh[(size_t)t * H + c] * (x[(size_t)t * H + c] * r[t]);
  partial[(size_t)chunk * H + c] = acc;
}

// ---------------------------------------------------------------- RMSNorm backward, fused
// Rows and gain partials in one pass over dh and x.  A workgroup owns `rows` consecutive rows (norm_bwd_rows), dealt to up to
// four wavefronts; every lane keeps the running sums of dh * xhat of its own columns (NV vectors of
// Vec<T>::N columns) in registers, the wavefronts are added in wavefront order through LDS, and
// the workgroup writes one partial row.  H <= NV * 64 * Vec<T>::N and H % Vec<T>::N == 0.
template <typename T, int NV>
__global__ __launch_bounds__(256) void rmsnorm_bwd_fused_kernel(const float* __restrict__ dh, const float* __restrict__ x,
                                                                const float* __restrict__ r, const T* __restrict__ g,
                                                                const float* __restrict__ add_in, float* __restrict__ out32,
                                                                T* __restrict__ out_t, float* __restrict__ partial,
                                                                int Tn, int H, int rows) {
  constexpr int V = Vec<T>::N;
  extern __shared__ float red[];                 // [wavefronts][H]
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, waves = blockDim.x >> 6, per = rows / waves;
  float gsum[NV][V];
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int i = 0; i < V; ++i) gsum[v][i] = 0.f;
  for (int rr_ = 0; rr_ < per; ++rr_) {
    const int row = blockIdx.x * rows + wave * per + rr_;
    if (row >= Tn) break;
    const size_t off = (size_t)row * H;
    const float rr = r[row];
    float dot = 0.f;
    if constexpr (NV <= 8) {
      // rows of up to 4096 values: dh and x stay in registers between the two sweeps (each is read from memory
      // once; 254 registers, two wavefronts per SIMD).  Measured at hidden 4096: 84 -> 78 us stand-alone, B task -0.8 %.
      float a[NV][V], b[NV][V];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int c = (v * WAVE + lane) * V;
        if (c < H) {
          load_f32<V>(dh + off + c, a[v]);
          load_f32<V>(x + off + c, b[v]);
        }
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int c = (v * WAVE + lane) * V;
        if (c < H) {
          float gv[V];
          load_vec<T>(g + c, gv);
#pragma unroll
          for (int i = 0; i < V; ++i) {
            b[v][i] *= rr;                       // xhat
            dot += a[v][i] * gv[i] * b[v][i];
            gsum[v][i] += a[v][i] * b[v][i];
          }
        }
      }
      dot = wave_sum(dot) / (float)H;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int c = (v * WAVE + lane) * V;
        if (c < H) {
          float gv[V], ad[V];
          load_vec<T>(g + c, gv);
          load_f32<V>(add_in + off + c, ad);
#pragma unroll
          for (int i = 0; i < V; ++i) ad[i] += rr * (a[v][i] * gv[i] - b[v][i] * dot);
          if (out32) store_f32<V>(out32 + off + c, ad);
          if (out_t) store_vec<T>(out_t + off + c, ad);
        }
      }
    } else {
      // longer rows (hidden 8192): keeping them would leave one wavefront per SIMD, measured slower (174 -> 197 us);
      // the second sweep re-reads the row, served by cache
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int c = (v * WAVE + lane) * V;
        if (c < H) {
          float a[V], b[V], gv[V];
          load_f32<V>(dh + off + c, a);
          load_f32<V>(x + off + c, b);
          load_vec<T>(g + c, gv);
#pragma unroll
          for (int i = 0; i < V; ++i) {
            const float xh = b[i] * rr;
            dot += a[i] * gv[i] * xh;
            gsum[v][i] += a[i] * xh;
          }
        }
      }
      dot = wave_sum(dot) / (float)H;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int c = (v * WAVE + lane) * V;
        if (c < H) {
          float a[V], b[V], gv[V], ad[V];
          load_f32<V>(dh + off + c, a);
          load_f32<V>(x + off + c, b);
          load_vec<T>(g + c, gv);
          load_f32<V>(add_in + off + c, ad);
#pragma unroll
          for (int i = 0; i < V; ++i) ad[i] += rr * (a[i] * gv[i] - (b[i] * rr) * dot);
          if (out32) store_f32<V>(out32 + off + c, ad);
          if (out_t) store_vec<T>(out_t + off + c, ad);
        }
      }
    }
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int c = (v * WAVE + lane) * V;
    if (c < H) store_f32<V>(red + (size_t)wave * H + c, gsum[v]);
  }
  __syncthreads();
  for (int c = threadIdx.x; c < H; c += blockDim.x) {
    float t = red[c];
    for (int w = 1; w < waves; ++w) t += red[(size_t)w * H + c];
    partial[(size_t)blockIdx.x * H + c] = t;
  }
}

// Column sums of `partial` [n_partial][width], rows ld apart, in one fixed order: 16 contiguous slices of the rows are
// summed front to back by 16 thread groups (4 columns per thread), then added in slice order.  64 columns from c0 per workgroup.
__device__ __forceinline__ void colsum_block(const float* __restrict__ partial, int n_partial, int ld, int width, int c0,
                                             float* __restrict__ out) {
  __shared__ float red[16][64];
  const int cv = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const int c = c0 + cv * 4;
  const int per = (n_partial + 15) / 16;
  const int p0 = grp * per, p1 = min(p0 + per, n_partial);
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  if (c + 3 < width && (ld & 3) == 0 && ((uintptr_t)partial & 15) == 0) {
    // eight loads in flight at a time, added in row order (the loop is bound by the latency of its loads)
    int p = p0;
    for (; p + 8 <= p1; p += 8) {
      float4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const float4*>(partial + (size_t)(p + u) * ld + c);
#pragma unroll
      for (int u = 0; u < 8; ++u) { acc[0] += v[u].x; acc[1] += v[u].y; acc[2] += v[u].z; acc[3] += v[u].w; }
    }
    for (; p < p1; ++p) {
      const float4 v = *reinterpret_cast<const float4*>(partial + (size_t)p * ld + c);
      acc[0] += v.x; acc[1] += v.y; acc[2] += v.z; acc[3] += v.w;
    }
  } else {
    for (int p = p0; p < p1; ++p)
      for (int i = 0; i < 4; ++i)
        if (c + i < width) acc[i] += partial[(size_t)p * ld + c + i];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) red[grp][cv * 4 + i] = acc[i];
  __syncthreads();
  if (threadIdx.x < 64) {
    const int cc = c0 + threadIdx.x;
    if (cc < width) {
      float t = red[0][threadIdx.x];
#pragma unroll
      for (int q = 1; q < 16; ++q) t += red[q][threadIdx.x];
      out[cc] = t;
    }
  }
}
__global__ __launch_bounds__(256) void colsum_kernel(const float* __restrict__ partial, int n_partial, int H, float* __restrict__ out) {
  colsum_block(partial, n_partial, H, H, blockIdx.x * 64, out);
}
// Entry of a list (at most 64) that workgroup `block` belongs to, from the entries' first workgroups: all are loaded at once, for a walk would be a
// chain of loads from the arguments in host memory.
__device__ __forceinline__ int list_index(const int* start, int n, int block) {
  const int lane = threadIdx.x & 63;
  return __builtin_amdgcn_readfirstlane(__popcll(__ballot(lane < n && start[lane] <= block)) - 1);
}
// The vector gradients of a whole B task: each sum is 2 to 5 us of latency (a few workgroups that walk some hundred rows), so one launch
// takes up to COLSUM_LIST_MAX of them, workgroup after workgroup.  4 layers with LayerNorm and biases: 32 launches of 4.7 us a task -> 1 (with the
// chunk sums of the bias gradients below, also one launch).
struct ColsumList {
  ColsumJob job[COLSUM_LIST_MAX];
  int start[COLSUM_LIST_MAX + 1];      // first workgroup of each, and the end
  int n;
};
__global__ __launch_bounds__(256) void colsum_list_kernel(const ColsumList list) {
  const int i = list_index(list.start, list.n, blockIdx.x);
  const ColsumJob& j = list.job[i];
  colsum_block(j.partial, j.n_partial, j.ld, j.width, ((int)blockIdx.x - list.start[i]) * 64, j.out);
}

// ---------------------------------------------------------------- SwiGLU / GELU
__device__ inline float sigmoidf_(float z) { return 1.0f / (1.0f + __expf(-z)); }

template <typename T>
__global__ __launch_bounds__(256) void swiglu_fwd_kernel(const T* __restrict__ gu, T* __restrict__ m, int Tn, int F) {
  constexpr int V = Vec<T>::N;
  const int fv = F / V;
  const size_t n = (size_t)Tn * fv;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const size_t t = i / fv;
    const int f = (int)(i % fv) * V;
    float a[V], b[V];
    load_vec<T>(gu + t * 2 * F + f, a);
    load_vec<T>(gu + t * 2 * F + F + f, b);
#pragma unroll
    for (int k = 0; k < V; ++k) a[k] = a[k] * sigmoidf_(a[k]) * b[k];
    store_vec<T>(m + t * F + f, a);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void swiglu_bwd_kernel(const float* __restrict__ dm, const T* __restrict__ gu,
                                                         T* __restrict__ dgu, int Tn, int F) {
  constexpr int V = Vec<T>::N;
  const int fv = F / V;
  const size_t n = (size_t)Tn * fv;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const size_t t = i / fv;
    const int f = (int)(i % fv) * V;
    float a[V], b[V], d[V], da[V], db[V];
    load_vec<T>(gu + t * 2 * F + f, a);
    load_vec<T>(gu + t * 2 * F + F + f, b);
    load_f32<V>(dm + t * F + f, d);
#pragma unroll
    for (int k = 0; k < V; ++k) {
      const float sg = sigmoidf_(a[k]);
      da[k] = d[k] * b[k] * sg * (1.0f + a[k] * (1.0f - sg));
      db[k] = d[k] * a[k] * sg;
    }
    store_vec<T>(dgu + t * 2 * F + f, da);
    store_vec<T>(dgu + t * 2 * F + F + f, db);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void gelu_fwd_kernel(const T* __restrict__ u, T* __restrict__ m, size_t nv) {
  constexpr int V = Vec<T>::N;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < nv; i += (size_t)gridDim.x * 256) {
    float a[V];
    load_vec<T>(u + i * V, a);
#pragma unroll
    for (int k = 0; k < V; ++k) a[k] = 0.5f * a[k] * (1.0f + erff(a[k] * 0.70710678118654752f));
    store_vec<T>(m + i * V, a);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void gelu_bwd_kernel(const float* __restrict__ dm, const T* __restrict__ u,
                                                       T* __restrict__ du, size_t nv) {
  constexpr int V = Vec<T>::N;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < nv; i += (size_t)gridDim.x * 256) {
    float a[V], d[V];
    load_vec<T>(u + i * V, a);
    load_f32<V>(dm + i * V, d);
#pragma unroll
    for (int k = 0; k < V; ++k) {
      const float Phi = 0.5f * (1.0f + erff(a[k] * 0.70710678118654752f));
      const float phi = 0.39894228040143268f * __expf(-0.5f * a[k] * a[k]);
      d[k] = d[k] * (Phi + a[k] * phi);
    }
    store_vec<T>(du + i * V, d);
  }
}

// ---------------------------------------------------------------- LayerNorm (model-fidelity variant)
// Plain kernels, one wavefront per row: h = (x - mu) * r * g + b with r = (var + eps)^-1/2 (biased
// variance, two passes over the row: mean first, then squared deviations).
template <typename T>
__global__ __launch_bounds__(256) void layernorm_fwd_kernel(const float* __restrict__ x, const T* __restrict__ g,
                                                            const T* __restrict__ b, T* __restrict__ h,
                                                            float* __restrict__ r_out, float* __restrict__ mu_out,
                                                            int Tn, int H, float eps, f16_t* __restrict__ h16) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= Tn) return;
  const float* xr = x + (size_t)row * H;
  float sum = 0.f;
  for (int c = lane; c < H; c += WAVE) sum += xr[c];
  const float mu = wave_sum(sum) / (float)H;
  float ss = 0.f;
  for (int c = lane; c < H; c += WAVE) { const float dlt = xr[c] - mu; ss += dlt * dlt; }
  const float r = 1.0f / sqrtf(wave_sum(ss) / (float)H + eps);
  if (lane == 0) { r_out[row] = r; mu_out[row] = mu; }
  T* hr = h + (size_t)row * H;
  for (int c = lane; c < H; c += WAVE) {
    const float v = (xr[c] - mu) * r * to_float(g[c]) + to_float(b[c]);
    hr[c] = from_float<T>(v);
    if (h16) h16[(size_t)row * H + c] = from_float<f16_t>(v);
  }
}

// The same for rows of whole vectors, read once (32 bytes per lane, every load issued before the first use) and kept in
// registers through the two sums.  H <= NV * 64 * Vec<T>::N and H % Vec<T>::N == 0.  The scalar kernel reads a row three times, four
// bytes per lane: 18.9 us for 2380 rows of 1280 on average; one iteration of the workload named at colsum_groups 5518 -> 5378 us.
template <typename T, int NV>
__global__ __launch_bounds__(256) void layernorm_fwd_vec_kernel(const float* __restrict__ x, const T* __restrict__ g,
                                                                const T* __restrict__ b, T* __restrict__ h,
                                                                float* __restrict__ r_out, float* __restrict__ mu_out,
                                                                int Tn, int H, float eps, f16_t* __restrict__ h16) {
  constexpr int V = Vec<T>::N;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= Tn) return;
  const size_t off = (size_t)row * H;
  float xv[NV][V];
  float sum = 0.f, ss = 0.f;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int c = (v * WAVE + lane) * V;
    if (c < H) load_f32<V>(x + off + c, xv[v]);
  }
#pragma unroll
  for (int v = 0; v < NV; ++v)
    if ((v * WAVE + lane) * V < H)
#pragma unroll
      for (int i = 0; i < V; ++i) sum += xv[v][i];
  const float mu = wave_sum(sum) / (float)H;
#pragma unroll
  for (int v = 0; v < NV; ++v)
    if ((v * WAVE + lane) * V < H)
#pragma unroll
      for (int i = 0; i < V; ++i) { xv[v][i] -= mu; ss += xv[v][i] * xv[v][i]; }
  const float r = 1.0f / sqrtf(wave_sum(ss) / (float)H + eps);
  if (lane == 0) { r_out[row] = r; mu_out[row] = mu; }
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int c = (v * WAVE + lane) * V;
    if (c < H) {
      float gv[V], bv[V];
      load_vec<T>(g + c, gv);
      load_vec<T>(b + c, bv);
#pragma unroll
      for (int i = 0; i < V; ++i) gv[i] = xv[v][i] * r * gv[i] + bv[i];
      store_vec<T>(h + off + c, gv);
      if constexpr (V == 8) {
        if (h16) store_vec<f16_t>(h16 + off + c, gv);
      }
    }
  }
}

// dx = add_in + r * (w - mean(w) - xhat * mean(w * xhat)),  w = dh * g,  xhat = (x - mu) * r.
template <typename T>
__global__ __launch_bounds__(256) void layernorm_bwd_rows_kernel(const float* __restrict__ dh, const float* __restrict__ x,
                                                                 const float* __restrict__ r, const float* __restrict__ mu,
                                                                 const T* __restrict__ g, const float* __restrict__ add_in,
                                                                 float* __restrict__ out32, T* __restrict__ out_t, int Tn, int H) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= Tn) return;
  const size_t off = (size_t)row * H;
  const float rr = r[row], m = mu[row];
  float s1 = 0.f, s2 = 0.f;
  for (int c = lane; c < H; c += WAVE) {
    const float w = dh[off + c] * to_float(g[c]);
    s1 += w;
    s2 += w * ((x[off + c] - m) * rr);
  }
  s1 = wave_sum(s1) / (float)H;
  s2 = wave_sum(s2) / (float)H;
  for (int c = lane; c < H; c += WAVE) {
    const float w = dh[off + c] * to_float(g[c]);
    const float v = add_in[off + c] + rr * (w - s1 - ((x[off + c] - m) * rr) * s2);
    if (out32) out32[off + c] = v;
    if (out_t) out_t[off + c] = from_float<T>(v);
  }
}

// The same for rows of whole vectors: dh and x are read once, 32 bytes per lane and every load issued before the first use, and
// stay in registers between the sums and the result.  H <= NV * 64 * Vec<T>::N and H % Vec<T>::N == 0.
template <typename T, int NV>
__global__ __launch_bounds__(256) void layernorm_bwd_rows_vec_kernel(const float* __restrict__ dh, const float* __restrict__ x,
                                                                     const float* __restrict__ r, const float* __restrict__ mu,
                                                                     const T* __restrict__ g, const float* __restrict__ add_in,
                                                                     float* __restrict__ out32, T* __restrict__ out_t, int Tn, int H) {
  constexpr int V = Vec<T>::N;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= Tn) return;
  const size_t off = (size_t)row * H;
  const float rr = r[row], m = mu[row];
  float w[NV][V], xh[NV][V];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int c = (v * WAVE + lane) * V;
    if (c < H) {
      load_f32<V>(dh + off + c, w[v]);
      load_f32<V>(x + off + c, xh[v]);
    }
  }
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int c = (v * WAVE + lane) * V;
    if (c < H) {
      float gv[V];
      load_vec<T>(g + c, gv);
#pragma unroll
      for (int i = 0; i < V; ++i) {
        w[v][i] *= gv[i];
        xh[v][i] = (xh[v][i] - m) * rr;
        s1 += w[v][i];
        s2 += w[v][i] * xh[v][i];
      }
    }
  }
  s1 = wave_sum(s1) / (float)H;
  s2 = wave_sum(s2) / (float)H;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int c = (v * WAVE + lane) * V;
    if (c < H) {
      float o[V];
      load_f32<V>(add_in + off + c, o);
#pragma unroll
      for (int i = 0; i < V; ++i) o[i] += rr * (w[v][i] - s1 - xh[v][i] * s2);
      if (out32) store_f32<V>(out32 + off + c, o);
      if (out_t) store_vec<T>(out_t + off + c, o);
    }
  }
}

// Column sums over chunks of NORM_BWD_ROWS rows, one chunk of 32 column vectors per workgroup.  One thread per column, walking its 64
// rows, is bound by the latency of a load at a time; here eight groups of threads take eight rows each with all loads in
// flight, and the groups are added in row order through LDS.  With the vector kernel above, one iteration of 4 layers of hidden 1280
// with LayerNorm and biases, two microbatches of 2641 and 2120 tokens: 6455 -> 5518 us.
constexpr int CS_GROUPS = 8, CS_ROWS = NORM_BWD_ROWS / CS_GROUPS, CS_VECS = 256 / CS_GROUPS;
template <int V>
__device__ __forceinline__ void colsum_groups(float (&acc)[V], float (*red)[CS_VECS * V], float* __restrict__ out, int c0, int n) {
  const int cv = threadIdx.x % CS_VECS, grp = threadIdx.x / CS_VECS;
#pragma unroll
  for (int i = 0; i < V; ++i) red[grp][cv * V + i] = acc[i];
  __syncthreads();
  if (threadIdx.x < CS_VECS * V && c0 + (int)threadIdx.x < n) {
    float t = red[0][threadIdx.x];
#pragma unroll
    for (int q = 1; q < CS_GROUPS; ++q) t += red[q][threadIdx.x];
    out[c0 + threadIdx.x] = t;
  }
  __syncthreads();
}

template <typename T>
__device__ __forceinline__ void colsum_rows_block(const T* __restrict__ src, int ld, float* __restrict__ partial, int Tn, int N, int block) {
  constexpr int V = Vec<T>::N;
  __shared__ float red[CS_GROUPS][CS_VECS * V];
  const int c0 = block * CS_VECS * V, c = c0 + (threadIdx.x % CS_VECS) * V;
  const int r0 = blockIdx.y * NORM_BWD_ROWS + threadIdx.x / CS_VECS * CS_ROWS;
  float acc[V] = {}, v[CS_ROWS][V] = {};
  if (c < N) {
#pragma unroll
    for (int i = 0; i < CS_ROWS; ++i)
      if (r0 + i < Tn) load_vec<T>(src + (size_t)(r0 + i) * ld + c, v[i]);
  }
#pragma unroll
  for (int i = 0; i < CS_ROWS; ++i)
#pragma unroll
    for (int k = 0; k < V; ++k) acc[k] += v[i][k];
  colsum_groups<V>(acc, red, partial + (size_t)blockIdx.y * N, c0, N);
}
template <typename T>
__global__ __launch_bounds__(256) void colsum_rows_vec_kernel(const T* __restrict__ src, int ld, float* __restrict__ partial, int Tn, int N) {
  colsum_rows_block<T>(src, ld, partial, Tn, N, blockIdx.x);
}
struct ColsumRowsList {
  ColsumRowsJob job[COLSUM_LIST_MAX];
  int start[COLSUM_LIST_MAX + 1];
  int n;
};
template <typename T>
__global__ __launch_bounds__(256) void colsum_rows_list_kernel(const ColsumRowsList list, int Tn) {
  const int i = list_index(list.start, list.n, blockIdx.x);
  const ColsumRowsJob& j = list.job[i];
  colsum_rows_block<T>((const T*)j.src, j.N, j.partial, Tn, j.N, (int)blockIdx.x - list.start[i]);
}

__global__ __launch_bounds__(256) void layernorm_bwd_partials_vec_kernel(const float* __restrict__ dh, const float* __restrict__ x,
                                                                         const float* __restrict__ r, const float* __restrict__ mu,
                                                                         float* __restrict__ partial_g, float* __restrict__ partial_b,
                                                                         int Tn, int H) {
  constexpr int V = 4;
  __shared__ float red[CS_GROUPS][CS_VECS * V];
  const int c0 = blockIdx.x * CS_VECS * V, c = c0 + (threadIdx.x % CS_VECS) * V;
  const int r0 = blockIdx.y * NORM_BWD_ROWS + threadIdx.x / CS_VECS * CS_ROWS;
  float sg[V] = {}, sb[V] = {}, d[CS_ROWS][V] = {}, xv[CS_ROWS][V] = {}, m[CS_ROWS] = {}, rr[CS_ROWS] = {};
  if (c < H) {
#pragma unroll
    for (int i = 0; i < CS_ROWS; ++i)
      if (r0 + i < Tn) {
        load_f32<V>(dh + (size_t)(r0 + i) * H + c, d[i]);
        load_f32<V>(x + (size_t)(r0 + i) * H + c, xv[i]);
        m[i] = mu[r0 + i];
        rr[i] = r[r0 + i];
      }
  }
#pragma unroll
  for (int i = 0; i < CS_ROWS; ++i)
#pragma unroll
    for (int k = 0; k < V; ++k) {
      sg[k] += d[i][k] * ((xv[i][k] - m[i]) * rr[i]);
      sb[k] += d[i][k];
    }
  colsum_groups<V>(sg, red, partial_g + (size_t)blockIdx.y * H, c0, H);
  colsum_groups<V>(sb, red, partial_b + (size_t)blockIdx.y * H, c0, H);
}

// Per-chunk partial sums for the LayerNorm gain and bias gradients: partial_g[chunk][c] = sum over the
// chunk's rows (ascending) of dh * xhat, partial_b[chunk][c] = sum of dh.  One thread per column.
__global__ __launch_bounds__(256) void layernorm_bwd_partials_kernel(const float* __restrict__ dh, const float* __restrict__ x,
                                                                     const float* __restrict__ r, const float* __restrict__ mu,
                                                                     float* __restrict__ partial_g, float* __restrict__ partial_b,
                                                                     int Tn, int H) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= H) return;
  const int r0 = blockIdx.y * NORM_BWD_ROWS, r1 = min(r0 + NORM_BWD_ROWS, Tn);
  float sg = 0.f, sb = 0.f;
  for (int row = r0; row < r1; ++row) {
    const float d = dh[(size_t)row * H + c];
    sg += d * ((x[(size_t)row * H + c] - mu[row]) * r[row]);
    sb += d;
  }
  partial_g[(size_t)blockIdx.y * H + c] = sg;
  partial_b[(size_t)blockIdx.y * H + c] = sb;
}

// Per-chunk column sums of a [Tn, N] tensor of the storage type (row pitch ld): partial[chunk][c] = sum
// over the chunk's rows in ascending order.  With launch_colsum this gives the bias gradients.
template <typename T>
__global__ __launch_bounds__(256) void colsum_rows_kernel(const T* __restrict__ src, int ld, float* __restrict__ partial,
                                                          int Tn, int N) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= N) return;
  const int r0 = blockIdx.y * NORM_BWD_ROWS, r1 = min(r0 + NORM_BWD_ROWS, Tn);
  float acc = 0.f;
  for (int row = r0; row < r1; ++row) acc += to_float(src[(size_t)row * ld + c]);
  partial[(size_t)blockIdx.y * N + c] = acc;
}

// ---------------------------------------------------------------- head norm (QK-norm variant)
// RMSNorm over head_dim (a multiple of 16, at most 128) of every (token, head) d-vector of the first n_heads heads of a [T, ld]
// tensor, in place: x <- xhat * g, with xhat = x * r saved (storage type) and r saved (fp32) for the backward.
// Heads [0, nq) use gq, heads [nq, n_heads) use gk.  A head is one 16-byte vector per lane of a group of HN_LANES lanes (two values per
// lane of a wavefront before): bound by memory, 2048 tokens x 40 heads of 128: 28.5 -> 12 us, the backward 43 -> 19.
// TP = type of the gains (the parameter storage type); T = type of the tensor and of the saved xhat.
template <typename T> constexpr int HN_LANES = 128 / Vec<T>::N;
template <int LANES>
__device__ __forceinline__ float group_sum(float v) {
#pragma unroll
  for (int o = LANES / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}
template <typename T, typename TP>
__global__ __launch_bounds__(256) void headnorm_fwd_kernel(T* __restrict__ x, int ld, int nq, int n_heads, int d,
                                                           const TP* __restrict__ gq, const TP* __restrict__ gk,
                                                           T* __restrict__ xhat, float* __restrict__ r_out, int Tn, float eps) {
  constexpr int V = Vec<T>::N, L = HN_LANES<T>;
  static_assert(Vec<TP>::N == V, "one vector of each");
  const size_t pair = (size_t)blockIdx.x * (256 / L) + threadIdx.x / L;
  const int c = threadIdx.x % L * V;
  if (pair >= (size_t)Tn * n_heads) return;
  const int t = (int)(pair / n_heads), hd = (int)(pair - (size_t)t * n_heads);
  T* p = x + (size_t)t * ld + hd * d + c;
  float v[V] = {}, gv[V], ss = 0.f;
  if (c < d) {
    load_vec<T>(p, v);
    load_vec<TP>((hd < nq ? gq : gk) + c, gv);
  }
#pragma unroll
  for (int i = 0; i < V; ++i) ss += v[i] * v[i];
  const float r = 1.0f / sqrtf(group_sum<L>(ss) / (float)d + eps);
  if (c == 0) r_out[pair] = r;
  if (c < d) {
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] *= r;
    store_vec<T>(xhat + pair * d + c, v);
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] *= gv[i];
    store_vec<T>(p, v);
  }
}

// Backward, in place on the gradient tensor: dx = r * (w - xhat * mean(w * xhat)), w = dy * g.  A workgroup
// handles 64 consecutive (token, head) pairs of ONE kind (grid y = 0: query heads, 1: key heads) and writes
// one partial row of the gain gradient, sum over its pairs (each group of lanes its own ascending, the groups in order) of dy * xhat.
// TX = type of the saved xhat (the forward's tensor type); T = type of the gradient tensor and of the gains.
template <typename T, typename TX>
__global__ __launch_bounds__(256) void headnorm_bwd_kernel(T* __restrict__ dy, int ld, int nq, int n_heads, int d,
                                                           const T* __restrict__ gq, const T* __restrict__ gk,
                                                           const TX* __restrict__ xhat, const float* __restrict__ r_in,
                                                           float* __restrict__ partial_q, float* __restrict__ partial_k, int Tn,
                                                           float* __restrict__ dk32) {
  constexpr int V = Vec<T>::N, L = HN_LANES<T>, GROUPS = 256 / L, PER = 64 / GROUPS;
  static_assert(Vec<TX>::N == V, "one vector of each");
  __shared__ float red[GROUPS][128];
  const int kind = blockIdx.y, nh = kind == 0 ? nq : n_heads - nq, h0 = kind == 0 ? 0 : nq;
  float* partial = kind == 0 ? partial_q : partial_k;
  const size_t n_pairs = (size_t)Tn * nh;
  if ((size_t)blockIdx.x * 64 >= n_pairs) return;
  const int grp = threadIdx.x / L, c = threadIdx.x % L * V;
  float gv[V] = {}, gs[V] = {}, dv[PER][V] = {}, xh[PER][V] = {}, rr[PER] = {};
  if (c < d) load_vec<T>((kind == 0 ? gq : gk) + c, gv);
  auto place = [&](int i, size_t& pair, T*& p, float*& p32) -> bool {
    const size_t q = (size_t)blockIdx.x * 64 + grp * PER + i;      // pair index inside this kind
    if (q >= n_pairs) return false;
    const int t = (int)(q / nh), hd = (int)(q - (size_t)t * nh);
    pair = (size_t)t * n_heads + h0 + hd;
    p = dy + (size_t)t * ld + (h0 + hd) * d + c;
    p32 = dk32 + ((size_t)t * nh + hd) * d + c;
    return true;
  };
#pragma unroll
  for (int i = 0; i < PER; ++i) {                      // every load in flight before the first use
    size_t pair; T* p; float* p32;
    if (place(i, pair, p, p32) && c < d) {
      load_vec<T>(p, dv[i]);
      load_vec<TX>(xhat + pair * d + c, xh[i]);
      rr[i] = r_in[pair];
    }
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    float w[V], dot = 0.f;
#pragma unroll
    for (int k = 0; k < V; ++k) {
      w[k] = dv[i][k] * gv[k];
      dot += w[k] * xh[i][k];
      gs[k] += dv[i][k] * xh[i][k];
    }
    dot = group_sum<L>(dot) / (float)d;
    size_t pair; T* p; float* p32;
    if (place(i, pair, p, p32) && c < d) {
#pragma unroll
      for (int k = 0; k < V; ++k) w[k] = rr[i] * (w[k] - xh[i][k] * dot);
      store_vec<T>(p, w);
      // un-rounded copy of the key-head gradients [Tn, nk * d]: their column sum (the key bias gradient) is a
      // small remainder of cancelling terms and would lose its leading digits to the storage rounding
      if (dk32 && kind == 1) store_f32<V>(p32, w);
    }
  }
#pragma unroll
  for (int k = 0; k < V; ++k) red[grp][c + k] = gs[k];
  __syncthreads();
  if ((int)threadIdx.x < d) {
    float t = red[0][threadIdx.x];
#pragma unroll
    for (int q = 1; q < GROUPS; ++q) t += red[q][threadIdx.x];
    partial[(size_t)blockIdx.x * d + threadIdx.x] = t;
  }
}

// ---------------------------------------------------------------- rotary embedding
// The angle is formed in double precision and reduced to [0, 2 pi) before the single-precision sine and cosine, so that the
// fp32 path keeps its 1e-4 budget at positions in the thousands.  A thread turns one vector of pairs of one row in up to ROPE_HEADS
// heads, which share its angles.  Workgroup: 256 / (half / V) rows of a query tile, blocks_per_tile of them launched for each: as many as the longest
// segment has.  What bounds it: memory at some thousand rows, before that the serial work of a thread, 0.4 us a head (with all loads in flight the same;
// the angles, formed in double, cost nothing beside it), so two heads and not eight.  us, a lane per pair and a workgroup per head and tile -> eight heads a
// thread -> this: bf16, 40 heads of 128, 2048 rows 25 -> 9.0 -> 8.1, 512 rows 23 -> 7.2 -> 4.4, 300 in three segments 11.3 -> 6.8 -> 4.1; 40 of 64, 61 rows in
// segments of 4 3.0 -> 7.2 -> 4.1; 8 of 128, 3973 segments of a row 16 -> 58 -> 17 (four heads: 15.7); 72 of 128, 4096 rows 54 -> 31 -> 26.6; fp32,
// 8 of 128, 983 rows in segments of 16 4.4 -> 10.1 -> 4.0; 2 of 64, 8000 in segments of 2 6.6 -> 22.5 -> 5.2.
constexpr int ROPE_HEADS = 2;
template <typename T>
__global__ __launch_bounds__(256) void rope_kernel(T* __restrict__ x, const AttnTile* __restrict__ tiles, int blocks_per_tile, int n_heads, int d,
                                                   int ld, double log2_base, float sign) {
  constexpr int V = Vec<T>::N;
  __shared__ double theta[64];
  const AttnTile tl = tiles[blockIdx.x / blocks_per_tile];
  const int half = d >> 1, chunks = half / V, rows = 256 / chunks;
  const int row0 = tl.r0 + (int)(blockIdx.x % blocks_per_tile) * rows, row = row0 + (int)threadIdx.x / chunks;
  const int c = threadIdx.x % chunks * V;
  if (row0 >= tl.r1) return;
  if ((int)threadIdx.x < half) theta[threadIdx.x] = exp2(-2.0 * (double)threadIdx.x / (double)d * log2_base);
  __syncthreads();
  if (row >= tl.r1 || (int)threadIdx.x >= rows * chunks) return;
  float sn[V], cs[V];
#pragma unroll
  for (int i = 0; i < V; ++i) {
    double ang = (double)(row - tl.s0) * theta[c + i];
    ang -= 6.283185307179586476925 * floor(ang * 0.1591549430918953357689);
    __sincosf((float)ang, &sn[i], &cs[i]);
    sn[i] *= sign;
  }
  T* p = x + (size_t)row * ld + c;
#pragma unroll
  for (int u = 0; u < ROPE_HEADS; ++u) {
    const int h = blockIdx.y * ROPE_HEADS + u;
    if (h >= n_heads) break;
    float a[V], b[V], ra[V], rb[V];
    load_vec<T>(p + h * d, a);
    load_vec<T>(p + h * d + half, b);
#pragma unroll
    for (int i = 0; i < V; ++i) {
      ra[i] = a[i] * cs[i] - b[i] * sn[i];
      rb[i] = b[i] * cs[i] + a[i] * sn[i];
    }
    store_vec<T>(p + h * d, ra);
    store_vec<T>(p + h * d + half, rb);
  }
}

// ---------------------------------------------------------------- gradient reduction
// Slots are streamed once: all loads of a group of up to 8 slots are issued before the first add (the
// adds then run in microbatch index order, which is what fixes the result bit for bit), and the loads
// bypass temporal caching.
typedef float f32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void grad_reduce_kernel(const f32x4* __restrict__ slots, size_t stride4, int M,
                                                          f32x4* __restrict__ out, size_t n4) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (size_t)gridDim.x * 256) {
    f32x4 acc = __builtin_nontemporal_load(slots + i);
    for (int j0 = 1; j0 < M; j0 += 8) {
      f32x4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (j0 + u < M) v[u] = __builtin_nontemporal_load(slots + (size_t)(j0 + u) * stride4 + i);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (j0 + u < M) acc += v[u];
    }
    __builtin_nontemporal_store(acc, out + i);
  }
}

inline int grid_for(size_t n, int cap = 256 * 32) {
  size_t b = (n + 255) / 256;
  return (int)(b < 1 ? 1 : (b > (size_t)cap ? cap : b));
}

}  // namespace

#define DISPATCH_T(dtype, ...)                       \
  if ((dtype) == F32) { using T = float; __VA_ARGS__; } \
  else { using T = bf16_t; __VA_ARGS__; }

// bf16 -> IEEE half, element by element (exact except below half's normal range; saturating), for a list of tensors: a workgroup converts
// HALF_COPY_VECS vectors, all its loads in flight.
constexpr int HALF_COPIES_MAX = 64, HALF_COPY_VECS = 4 * 256;
struct HalfCopies {
  HalfCopy c[HALF_COPIES_MAX];
  int start[HALF_COPIES_MAX + 1];      // first workgroup of each, and the end
  int n;
};
__global__ __launch_bounds__(256) void bf16_to_f16_kernel(const HalfCopies list) {
  const int t = list_index(list.start, list.n, blockIdx.x);
  const bf16_t* src = (const bf16_t*)list.c[t].src;
  f16_t* dst = (f16_t*)list.c[t].dst;
  const size_t n8 = list.c[t].n / 8, i0 = (size_t)((int)blockIdx.x - list.start[t]) * HALF_COPY_VECS + threadIdx.x;
  float v[4][8];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (i0 + k * 256 < n8) load_vec<bf16_t>(src + (i0 + k * 256) * 8, v[k]);
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (i0 + k * 256 < n8) store_vec<f16_t>(dst + (i0 + k * 256) * 8, v[k]);
}

hipError_t launch_widen(const void* src, float* dst, size_t n, int dtype, hipStream_t s, void* copy, float* scale, float* partial,
                        const void* host, void* device, size_t bytes) {
  const int blocks = scale ? grad_scale_partials(n) : grid_for(n / (dtype == F32 ? 4 : 8) + 1);
  DISPATCH_T(dtype, hipLaunchKernelGGL(widen_kernel<T>, dim3(blocks), dim3(256), 0, s, (const T*)src, dst, n, (T*)copy, scale ? partial : nullptr,
                                       (const int*)host, (int*)device, (int)(bytes / 4)));
  if (scale) hipLaunchKernelGGL(grad_scale_kernel, dim3(1), dim3(256), 0, s, (const float*)partial, blocks, scale);
  return hipGetLastError();
}

hipError_t launch_rope(void* x, const AttnTile* q_tiles, int n_q_tiles, int longest, int n_heads, int d, int ld, float base,
                       float sign, int dtype, hipStream_t s) {
  if (n_q_tiles < 1 || n_heads < 1 || d % 16 || d < 16 || d > 128 || !(base > 1.0f)) return hipErrorInvalidValue;
  const int rows = 256 / (d / 2 / (dtype == F32 ? 4 : 8)), per_tile = (std::min(longest, ATTN_TILE_Q) + rows - 1) / rows;
  const dim3 grid(n_q_tiles * per_tile, (n_heads + ROPE_HEADS - 1) / ROPE_HEADS);
  if (dtype == F16) {
    hipLaunchKernelGGL(rope_kernel<f16_t>, grid, dim3(256), 0, s, (f16_t*)x, q_tiles, per_tile, n_heads, d, ld, log2((double)base), sign);
    return hipGetLastError();
  }
  DISPATCH_T(dtype, hipLaunchKernelGGL(rope_kernel<T>, grid, dim3(256), 0, s, (T*)x, q_tiles, per_tile, n_heads, d, ld, log2((double)base), sign));
  return hipGetLastError();
}

hipError_t launch_rmsnorm_fwd(const float* x, const void* g, void* h, float* r_out, int Tn, int H, float eps,
                              int dtype, hipStream_t s, void* h16) {
  if (h16 && dtype != BF16) return hipErrorInvalidValue;
  const int V = dtype == F32 ? 4 : 8;
  if ((H % V) == 0) {
    const int nv = (H + WAVE * V - 1) / (WAVE * V);
#define RRFP_ROWS(NVV)                                                                                              \
  if (nv <= NVV) {                                                                                                  \
    DISPATCH_T(dtype, hipLaunchKernelGGL((rmsnorm_fwd_rows_kernel<T, NVV>), dim3((Tn + 3) / 4), dim3(256), 0, s, x, \
                                         (const T*)g, (T*)h, r_out, Tn, H, eps, (f16_t*)h16));                      \
    return hipGetLastError();                                                                                       \
  }
    RRFP_ROWS(1) RRFP_ROWS(2) RRFP_ROWS(4) RRFP_ROWS(8) RRFP_ROWS(16)
#undef RRFP_ROWS
  }
  DISPATCH_T(dtype, hipLaunchKernelGGL(rmsnorm_fwd_kernel<T>, dim3((Tn + 3) / 4), dim3(256), 0, s, x, (const T*)g, (T*)h,
                                       r_out, Tn, H, eps, (f16_t*)h16));
  return hipGetLastError();
}

template <typename T, int NV>
hipError_t launch_bwd_fused(const float* dh, const float* x, const float* r, const void* g, const float* add_in,
                            float* out32, void* out_t, float* dg_partial, int Tn, int H, int rows, hipStream_t s) {
  auto kern = rmsnorm_bwd_fused_kernel<T, NV>;
  const int waves = std::min(rows, 4);
  const size_t smem = (size_t)waves * H * sizeof(float);
  static std::once_flag once;
  static hipError_t once_status = hipSuccess;
  if (hipError_t e = set_max_dynamic_lds_once(once, once_status, (const void*)kern, 4 * NV * WAVE * Vec<T>::N * 4); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((Tn + rows - 1) / rows), dim3(waves * WAVE), smem, s, dh, x, r, (const T*)g, add_in, out32,
                     (T*)out_t, dg_partial, Tn, H, rows);
  return hipGetLastError();
}

static bool norm_bwd_fused(int H, int dtype) {
  const int V = dtype == F32 ? 4 : 8;
  return (H % V) == 0 && H <= 16 * WAVE * V && (dtype != F32 || H <= 8 * WAVE * V);
}

int norm_bwd_partials(int Tn, int H, int dtype, int rows) {
  const int per = norm_bwd_fused(H, dtype) ? rows : NORM_BWD_ROWS;
  return (Tn + per - 1) / per;
}

// A row of 4096 costs 74 KB of traffic, and one CU moves about 35 KB a microsecond: workgroups of 8 rows that do not reach every CU leave
// the time to the few that work.  So below one workgroup per CU the rows per workgroup are halved, down to 2.  Measured, one B
// task of 4 layers of hidden 4096 with 256 to 675 tokens, 8 rows -> this rule: 1400 -> 1336 us.  The line: 4 workgroups per CU
// instead of one adds partial rows for nothing (4096 tokens 7.43 -> 7.52 ms a task, 3272 tokens of hidden 2048 1109 -> 1130 us); rows
// below 1024 values are too short to matter (hidden 512: 658 against 660).
constexpr int NORM_BWD_MAX_CUS = 256;   // of the chip: bounds the partial rows
int norm_bwd_rows(int Tn, int H, int dtype, int n_cu) {
  int rows = NORM_BWD_FUSED_ROWS;
  if (H < 1024 || !norm_bwd_fused(H, dtype)) return rows;
  while (rows > 2 && (Tn + rows - 1) / rows < std::min(n_cu, NORM_BWD_MAX_CUS)) rows /= 2;
  return rows;
}
size_t norm_bwd_few_rows_bytes(int Tn, int H, int dtype) {
  if (H < 1024 || !norm_bwd_fused(H, dtype)) return 0;
  return (size_t)std::min((Tn + 1) / 2, 2 * NORM_BWD_MAX_CUS) * H * 4;   // halving less than a workgroup per CU gives less than two
}

hipError_t launch_rmsnorm_bwd(const float* dh, const float* x, const float* r, const void* g, const float* add_in,
                              float* out32, void* out_t, float* dg_partial, int Tn, int H, int dtype, hipStream_t s, int rows) {
  const int V = dtype == F32 ? 4 : 8;
  if (norm_bwd_fused(H, dtype)) {
    const int nv = (H + WAVE * V - 1) / (WAVE * V);
#define RRFP_FUSED(NVV)                                                                                         \
  if (nv <= NVV) {                                                                                              \
    DISPATCH_T(dtype, return (launch_bwd_fused<T, NVV>(dh, x, r, g, add_in, out32, out_t, dg_partial, Tn, H, rows, s))); \
  }
    RRFP_FUSED(1) RRFP_FUSED(2) RRFP_FUSED(3) RRFP_FUSED(4) RRFP_FUSED(6) RRFP_FUSED(8)
    if (dtype != F32) { RRFP_FUSED(16) }
#undef RRFP_FUSED
  }
  const int chunks = (Tn + NORM_BWD_ROWS - 1) / NORM_BWD_ROWS;
  DISPATCH_T(dtype, {
    hipLaunchKernelGGL(rmsnorm_bwd_gain_kernel<T>, dim3((H + 255) / 256, chunks), dim3(256), 0, s, dh, x, r,
                       dg_partial, Tn, H);
    hipLaunchKernelGGL(rmsnorm_bwd_rows_kernel<T>, dim3((Tn + 3) / 4), dim3(256), 0, s, dh, x, r, (const T*)g,
                       add_in, out32, (T*)out_t, Tn, H);
  });
  return hipGetLastError();
}

int headnorm_partials(int Tn, int n_heads_of_kind) { return (int)(((size_t)Tn * n_heads_of_kind + 63) / 64); }

hipError_t launch_headnorm_fwd(void* x, int ld, int nq, int n_heads, int d, const void* gq, const void* gk, void* xhat,
                               float* r_out, int Tn, float eps, int dtype, hipStream_t s) {
  if (d > 128 || d % 16) return hipErrorInvalidValue;
  const int per = dtype == F32 ? 256 / HN_LANES<float> : 256 / HN_LANES<f16_t>;
  const dim3 grid((unsigned)(((size_t)Tn * n_heads + per - 1) / per));
  if (dtype == F16) {   // half tensor, bf16 gains
    hipLaunchKernelGGL((headnorm_fwd_kernel<f16_t, bf16_t>), grid, dim3(256), 0, s, (f16_t*)x, ld, nq,
                       n_heads, d, (const bf16_t*)gq, (const bf16_t*)gk, (f16_t*)xhat, r_out, Tn, eps);
    return hipGetLastError();
  }
  DISPATCH_T(dtype, hipLaunchKernelGGL((headnorm_fwd_kernel<T, T>), grid, dim3(256), 0, s, (T*)x, ld, nq,
                                       n_heads, d, (const T*)gq, (const T*)gk, (T*)xhat, r_out, Tn, eps));
  return hipGetLastError();
}

hipError_t launch_headnorm_bwd(void* dy, int ld, int nq, int n_heads, int d, const void* gq, const void* gk, const void* xhat,
                               const float* r_in, float* partial_q, float* partial_k, int Tn, int dtype, hipStream_t s,
                               float* dk32, int xhat_dtype) {
  if (d > 128 || d % 16) return hipErrorInvalidValue;
  const int nb = std::max(headnorm_partials(Tn, nq), headnorm_partials(Tn, n_heads - nq));
  if (xhat_dtype == F16) {
    if (dtype != BF16) return hipErrorInvalidValue;
    hipLaunchKernelGGL((headnorm_bwd_kernel<bf16_t, f16_t>), dim3(nb, 2), dim3(256), 0, s, (bf16_t*)dy, ld, nq, n_heads, d,
                       (const bf16_t*)gq, (const bf16_t*)gk, (const f16_t*)xhat, r_in, partial_q, partial_k, Tn, dk32);
    return hipGetLastError();
  }
  DISPATCH_T(dtype, hipLaunchKernelGGL((headnorm_bwd_kernel<T, T>), dim3(nb, 2), dim3(256), 0, s, (T*)dy, ld, nq, n_heads, d,
                                       (const T*)gq, (const T*)gk, (const T*)xhat, r_in, partial_q, partial_k, Tn, dk32));
  return hipGetLastError();
}

int colsum_chunks(int Tn) { return (Tn + NORM_BWD_ROWS - 1) / NORM_BWD_ROWS; }

hipError_t launch_layernorm_fwd(const float* x, const void* g, const void* b, void* h, float* r_out, float* mu_out,
                                int Tn, int H, float eps, int dtype, hipStream_t s, void* h16) {
  if (h16 && dtype != BF16) return hipErrorInvalidValue;
  // as in the backward: rows of whole vectors up to 4096 values (fp32 2048) stay in registers
  const int V = dtype == F32 ? 4 : 8, nv = (H + WAVE * V - 1) / (WAVE * V);
  const bool vec = H % V == 0 && !(((uintptr_t)x | (uintptr_t)g | (uintptr_t)b | (uintptr_t)h | (uintptr_t)h16) & 15);
#define RRFP_LN(NVV)                                                                                                            \
  if (vec && nv <= NVV) {                                                                                                       \
    DISPATCH_T(dtype, hipLaunchKernelGGL((layernorm_fwd_vec_kernel<T, NVV>), dim3((Tn + 3) / 4), dim3(256), 0, s, x, (const T*)g, \
                                         (const T*)b, (T*)h, r_out, mu_out, Tn, H, eps, (f16_t*)h16));                          \
    return hipGetLastError();                                                                                                   \
  }
  RRFP_LN(1) RRFP_LN(3) RRFP_LN(8)
#undef RRFP_LN
  DISPATCH_T(dtype, hipLaunchKernelGGL(layernorm_fwd_kernel<T>, dim3((Tn + 3) / 4), dim3(256), 0, s, x, (const T*)g,
                                       (const T*)b, (T*)h, r_out, mu_out, Tn, H, eps, (f16_t*)h16));
  return hipGetLastError();
}

hipError_t launch_layernorm_bwd(const float* dh, const float* x, const float* r, const float* mu, const void* g,
                                const float* add_in, float* out32, void* out_t, float* partial_g, float* partial_b,
                                int Tn, int H, int dtype, hipStream_t s) {
  if ((H & 3) == 0)
    hipLaunchKernelGGL(layernorm_bwd_partials_vec_kernel, dim3((H + CS_VECS * 4 - 1) / (CS_VECS * 4), colsum_chunks(Tn)), dim3(256), 0, s, dh, x,
                       r, mu, partial_g, partial_b, Tn, H);
  else
    hipLaunchKernelGGL(layernorm_bwd_partials_kernel, dim3((H + 255) / 256, colsum_chunks(Tn)), dim3(256), 0, s, dh, x, r, mu,
                       partial_g, partial_b, Tn, H);
  // rows of whole vectors up to 4096 values (fp32 2048) stay in registers; longer and odd ones take the scalar kernel
  const int V = dtype == F32 ? 4 : 8, nv = (H + WAVE * V - 1) / (WAVE * V);
  auto aligned = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
#define RRFP_LN(NVV)                                                                                                        \
  if (nv <= NVV) {                                                                                                          \
    DISPATCH_T(dtype, hipLaunchKernelGGL((layernorm_bwd_rows_vec_kernel<T, NVV>), dim3((Tn + 3) / 4), dim3(256), 0, s, dh, x, r, mu, \
                                         (const T*)g, add_in, out32, (T*)out_t, Tn, H));                                    \
    return hipGetLastError();                                                                                               \
  }
  if (H % V == 0 && aligned(out_t) && aligned(out32) && aligned(g)) { RRFP_LN(1) RRFP_LN(3) RRFP_LN(8) }
#undef RRFP_LN
  DISPATCH_T(dtype, hipLaunchKernelGGL(layernorm_bwd_rows_kernel<T>, dim3((Tn + 3) / 4), dim3(256), 0, s, dh, x, r, mu,
                                       (const T*)g, add_in, out32, (T*)out_t, Tn, H));
  return hipGetLastError();
}

hipError_t launch_colsum_rows(const void* src, int ld, float* partial, int Tn, int N, int dtype, hipStream_t s) {
  const int V = dtype == F32 ? 4 : 8;
  if (N % V == 0 && ld % V == 0 && ((uintptr_t)src & 15) == 0) {
    DISPATCH_T(dtype, hipLaunchKernelGGL(colsum_rows_vec_kernel<T>, dim3((N + CS_VECS * V - 1) / (CS_VECS * V), colsum_chunks(Tn)), dim3(256), 0, s,
                                         (const T*)src, ld, partial, Tn, N));
    return hipGetLastError();
  }
  DISPATCH_T(dtype, hipLaunchKernelGGL(colsum_rows_kernel<T>, dim3((N + 255) / 256, colsum_chunks(Tn)), dim3(256), 0, s,
                                       (const T*)src, ld, partial, Tn, N));
  return hipGetLastError();
}

hipError_t launch_colsum(const float* partial, int n_partial, int H, float* out, hipStream_t s) {
  hipLaunchKernelGGL(colsum_kernel, dim3((H + 63) / 64), dim3(256), 0, s, partial, n_partial, H, out);
  return hipGetLastError();
}

hipError_t launch_colsum_list(const ColsumJob* jobs, int n, hipStream_t s) {
  for (int i0 = 0; i0 < n; i0 += COLSUM_LIST_MAX) {
    ColsumList list;
    list.n = std::min(COLSUM_LIST_MAX, n - i0);
    list.start[0] = 0;
    for (int i = 0; i < list.n; ++i) {
      list.job[i] = jobs[i0 + i];
      list.start[i + 1] = list.start[i] + (jobs[i0 + i].width + 63) / 64;
    }
    hipLaunchKernelGGL(colsum_list_kernel, dim3(list.start[list.n]), dim3(256), 0, s, list);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_colsum_rows_list(const ColsumRowsJob* jobs, int n, int Tn, int dtype, hipStream_t s) {
  const int V = dtype == F32 ? 4 : 8, chunks = colsum_chunks(Tn);
  ColsumRowsList list;
  list.n = 0;
  list.start[0] = 0;
  auto flush = [&]() -> hipError_t {
    if (list.n > 0) {
      DISPATCH_T(dtype, hipLaunchKernelGGL(colsum_rows_list_kernel<T>, dim3(list.start[list.n], chunks), dim3(256), 0, s, list, Tn));
    }
    list.n = 0;
    return hipGetLastError();
  };
  for (int i = 0; i < n; ++i) {
    const ColsumRowsJob& j = jobs[i];
    if (j.N % V || ((uintptr_t)j.src & 15)) {          // the kernel of single columns, by itself
      if (hipError_t e = launch_colsum_rows(j.src, j.N, j.partial, Tn, j.N, dtype, s); e != hipSuccess) return e;
      continue;
    }
    list.job[list.n] = j;
    list.start[list.n + 1] = list.start[list.n] + (j.N + CS_VECS * V - 1) / (CS_VECS * V);
    if (++list.n == COLSUM_LIST_MAX)
      if (hipError_t e = flush(); e != hipSuccess) return e;
  }
  return flush();
}

hipError_t launch_swiglu_fwd(const void* gu, void* m, int Tn, int F, int dtype, hipStream_t s) {
  DISPATCH_T(dtype, {
    if (F % Vec<T>::N) return hipErrorInvalidValue;
    hipLaunchKernelGGL(swiglu_fwd_kernel<T>, dim3(grid_for((size_t)Tn * F / Vec<T>::N)), dim3(256), 0, s, (const T*)gu,
                       (T*)m, Tn, F);
  });
  return hipGetLastError();
}

hipError_t launch_swiglu_bwd(const float* dm, const void* gu, void* dgu, int Tn, int F, int dtype, hipStream_t s) {
  DISPATCH_T(dtype, {
    if (F % Vec<T>::N) return hipErrorInvalidValue;
    hipLaunchKernelGGL(swiglu_bwd_kernel<T>, dim3(grid_for((size_t)Tn * F / Vec<T>::N)), dim3(256), 0, s, dm,
                       (const T*)gu, (T*)dgu, Tn, F);
  });
  return hipGetLastError();
}

hipError_t launch_gelu_fwd(const void* u, void* m, int Tn, int F, int dtype, hipStream_t s) {
  DISPATCH_T(dtype, {
    if (F % Vec<T>::N) return hipErrorInvalidValue;
    const size_t nv = (size_t)Tn * F / Vec<T>::N;
    hipLaunchKernelGGL(gelu_fwd_kernel<T>, dim3(grid_for(nv)), dim3(256), 0, s, (const T*)u, (T*)m, nv);
  });
  return hipGetLastError();
}

hipError_t launch_gelu_bwd(const float* dm, const void* u, void* du, int Tn, int F, int dtype, hipStream_t s) {
  DISPATCH_T(dtype, {
    if (F % Vec<T>::N) return hipErrorInvalidValue;
    const size_t nv = (size_t)Tn * F / Vec<T>::N;
    hipLaunchKernelGGL(gelu_bwd_kernel<T>, dim3(grid_for(nv)), dim3(256), 0, s, dm, (const T*)u, (T*)du, nv);
  });
  return hipGetLastError();
}

int grad_scale_partials(size_t n) { return grid_for(n / 8 + 1, 1024); }

hipError_t launch_bf16_to_f16(const HalfCopy* list, int n, hipStream_t s) {
  for (int i0 = 0; i0 < n; i0 += HALF_COPIES_MAX) {
    HalfCopies c;
    c.n = std::min(HALF_COPIES_MAX, n - i0);
    c.start[0] = 0;
    for (int i = 0; i < c.n; ++i) {
      c.c[i] = list[i0 + i];
      if (c.c[i].n % 8 || ((uintptr_t)c.c[i].src & 15) || ((uintptr_t)c.c[i].dst & 15)) return hipErrorInvalidValue;
      c.start[i + 1] = c.start[i] + (int)((c.c[i].n / 8 + HALF_COPY_VECS - 1) / HALF_COPY_VECS);
    }
    hipLaunchKernelGGL(bf16_to_f16_kernel, dim3(c.start[c.n]), dim3(256), 0, s, c);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_grad_reduce(const float* slots, size_t slot_stride, int M, float* out, size_t n, hipStream_t s) {
  if (n % 4 || slot_stride % 4) return hipErrorInvalidValue;
  // one 16-byte element per thread where the grid allows it: measured 5.3 TB/s against 4.6 TB/s for a grid-stride
  // loop over 8192 workgroups (8 slots of 1 GiB; a pure read of the same bytes runs at 5.7 TB/s on this chip)
  hipLaunchKernelGGL(grad_reduce_kernel, dim3(grid_for(n / 4, 1 << 24)), dim3(256), 0, s, (const f32x4*)slots, slot_stride / 4,
                     M, (f32x4*)out, n / 4);
  return hipGetLastError();
}

}  // namespace rrfp
