// The masked-edge flavours of the bf16 GEMM (gemm_mfma_kernel.h with EDGE): any M, N, K, in the three
// orientations and with the epilogues that the block and the training step use.
#include "gemm_mfma_kernel.h"

namespace fax {

template <int BM, int BN>
static int dispatch_edge(const GemmArgs& g, const EpiArgs& e, hipStream_t s) {
  const bool erf = g.gelu_form == FAX_GELU_ERF;
  if (g.epi == EPI_GELU && g.value_only)
    return erf ? launch_mfma<BM, BN, true, false, EK_VALUE_ERF, true>(g, e, s) : launch_mfma<BM, BN, true, false, EK_VALUE_TANH, true>(g, e, s);
  if (g.epi == EPI_GELU)
    return erf ? launch_mfma<BM, BN, true, false, EK_GELU_ERF, true>(g, e, s)
               : launch_mfma<BM, BN, true, false, EK_GELU_TANH, true>(g, e, s);
  if (g.epi == EPI_DGELU) return launch_mfma<BM, BN, true, true, EK_DGELU, true>(g, e, s);
  if (g.c_f32 && g.colsum)
    return g.accumulate ? launch_mfma<BM, BN, false, false, EK_F32 | EM_RES | EM_COLSUM, true>(g, e, s)
                        : launch_mfma<BM, BN, false, false, EK_F32 | EM_COLSUM, true>(g, e, s);
  if (g.c_f32 && !g.ta) return launch_mfma<BM, BN, true, false, EK_F32, true>(g, e, s);  // partial products of a bf16 output
  if (g.c_f32)
    return g.accumulate ? launch_mfma<BM, BN, false, false, EK_F32 | EM_RES, true>(g, e, s)
                        : launch_mfma<BM, BN, false, false, EK_F32, true>(g, e, s);
  if (g.tb) return launch_mfma<BM, BN, true, true, EK_STORE, true>(g, e, s);
  if (g.C2)
    return g.R ? launch_mfma<BM, BN, true, false, EK_STORE | EM_RES | EM_C2, true>(g, e, s)
               : launch_mfma<BM, BN, true, false, EK_STORE | EM_C2, true>(g, e, s);
  return g.R ? launch_mfma<BM, BN, true, false, EK_STORE | EM_RES, true>(g, e, s)
             : launch_mfma<BM, BN, true, false, EK_STORE, true>(g, e, s);
}

int gemm_mfma_edge(const GemmArgs& g, const EpiArgs& e, const GemmSplitPlan& plan, hipStream_t s) {
  if (plan.tile_n == 256) return dispatch_edge<256, 256>(g, e, s);
  if (plan.tile_m == 256) return dispatch_edge<256, 128>(g, e, s);
  return dispatch_edge<128, 128>(g, e, s);
}

}  // namespace fax
