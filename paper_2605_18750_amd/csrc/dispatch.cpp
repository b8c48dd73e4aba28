// Chooses the kernel family for each GEMM and attention call.  The choice is a pure function
// of dtype and shape, never of machine state, so a task always runs the same kernels.
#include "kernels.h"

#include <algorithm>

namespace rrfp {

bool gemm_act_supported(const GemmArgs& g) {
  return g.act == ACT_NONE || (g.in_dtype == F32 ? gemm_f32_act_supported(g) : gemm_mfma_act_supported(g));
}
hipError_t launch_gemm(const GemmArgs& g, hipStream_t s) {
  if (!gemm_act_supported(g)) return hipErrorInvalidValue;
  if (g.act != ACT_NONE) return g.in_dtype == F32 ? launch_gemm_f32(g, s) : launch_gemm_mfma(g, s);
  if (g.in_dtype == F32 && g.out_dtype == F32) return launch_gemm_f32(g, s);
  return gemm_mfma_supports(g) ? launch_gemm_mfma(g, s) : launch_gemm_simt(g, s);
}
// Length of the longest run of products at the front of the list that one kernel family takes together.
static int wgrad_run(const GemmArgs* g, int n) {
  bool (*const fits)(const GemmArgs&) = g[0].in_dtype == F32 ? gemm_f32_groupable : gemm_mfma_wgrad_groupable;
  int j = 0;
  while (j < n && g[j].K == g[0].K && g[j].in_dtype == g[0].in_dtype && fits(g[j])) ++j;
  return j;
}
hipError_t launch_wgrad_group(const GemmArgs* g, int n, hipStream_t s) {
  for (int i = 0; i < n;) {
    int j = i + wgrad_run(g + i, n - i);
    hipError_t e;
    if (j > i) e = (g[i].in_dtype == F32 ? launch_gemm_f32_group : launch_gemm_mfma_wgrad_group)(g + i, j - i, s);
    else e = launch_gemm(g[j++], s);
    if (e != hipSuccess) return e;
    i = j;
  }
  return hipSuccess;
}
size_t wgrad_group_plane_bytes(GemmArgs* g, int n, int max_K, const int* n_cu, int n_counts) {
  if (g[0].in_dtype == F32) return 0;
  auto fitting = [&](int K) {
    for (int i = 0; i < n; ++i) g[i].K = K;
    return (int)std::count_if(g, g + n, gemm_mfma_wgrad_groupable);
  };
  // a product leaves the list for good once an operand reaches 2 GiB: the lengths between such points share one list
  size_t most = 0;
  for (int K = 1; K <= max_K;) {
    const int here = fitting(K);
    int lo = max_K;
    if (fitting(max_K) != here) {
      lo = K;
      for (int hi = max_K - 1; lo < hi;) {
        const int mid = hi - (hi - lo) / 2;
        if (fitting(mid) == here) lo = mid;
        else hi = mid - 1;
      }
    }
    fitting(K);
    for (int i = 0; i < n;) {
      const int run = wgrad_run(g + i, n - i);
      for (int j = 0; j < run; j += WGRAD_GROUP_MAX)
        for (int c = 0; c < n_counts; ++c)
          most = std::max(most, gemm_mfma_wgrad_plane_bytes(g + i + j, std::min(WGRAD_GROUP_MAX, run - j), K, lo, n_cu[c]));
      i += std::max(run, 1);
    }
    K = lo + 1;
  }
  return most;
}
AttnPlan attn_plan(const AttnArgs& a, int n_cu) { return attn_mfma_supports(a) ? attn_mfma_plan(a, n_cu) : attn_f32_plan(a, n_cu); }
hipError_t launch_attn_fwd(const AttnArgs& a, hipStream_t s) {
  return attn_mfma_supports(a) ? launch_attn_fwd_mfma(a, s) : launch_attn_fwd_f32(a, s);
}
hipError_t launch_attn_bwd(const AttnArgs& a, hipStream_t s) {
  return attn_mfma_supports(a) ? launch_attn_bwd_mfma(a, s) : launch_attn_bwd_f32(a, s);
}

}  // namespace rrfp
