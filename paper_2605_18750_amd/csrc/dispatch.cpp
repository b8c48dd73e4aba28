// Chooses the kernel family for each GEMM and attention call.  The choice is a pure function
// of dtype and shape, never of machine state, so a task always runs the same kernels.
#include "kernels.h"

namespace rrfp {

hipError_t launch_gemm(const GemmArgs& g, hipStream_t s) {
  if (g.act != ACT_NONE) return gemm_act_supported(g) ? launch_gemm_mfma(g, s) : hipErrorInvalidValue;
  if (g.in_dtype == F32 && g.out_dtype == F32) return launch_gemm_f32(g, s);
  return gemm_mfma_supports(g) ? launch_gemm_mfma(g, s) : launch_gemm_simt(g, s);
}
hipError_t launch_wgrad_group(const GemmArgs* g, int n, hipStream_t s) {
  for (int i = 0; i < n;) {
    // the longest run of products that one kernel family takes together
    bool (*const fits)(const GemmArgs&) = g[i].in_dtype == F32 ? gemm_f32_groupable : gemm_mfma_wgrad_groupable;
    int j = i;
    while (j < n && g[j].K == g[i].K && g[j].in_dtype == g[i].in_dtype && fits(g[j])) ++j;
    hipError_t e;
    if (j > i) e = (g[i].in_dtype == F32 ? launch_gemm_f32_group : launch_gemm_mfma_wgrad_group)(g + i, j - i, s);
    else e = launch_gemm(g[j++], s);
    if (e != hipSuccess) return e;
    i = j;
  }
  return hipSuccess;
}
hipError_t launch_attn_fwd(const AttnArgs& a, hipStream_t s) {
  return attn_mfma_supports(a) ? launch_attn_fwd_mfma(a, s) : launch_attn_fwd_f32(a, s);
}
hipError_t launch_attn_bwd(const AttnArgs& a, hipStream_t s) {
  return attn_mfma_supports(a) ? launch_attn_bwd_mfma(a, s) : launch_attn_bwd_f32(a, s);
}

}  // namespace rrfp
