// The grouped flavours of the bf16 GEMM (gemm_mfma_kernel.h with GROUP): the weight gradients of one layer in one launch.
#include "gemm_mfma_kernel.h"

namespace fax {

template <int BM, bool EDGE>
static int group_t(const GemmArgs* g, int n, const EpiArgs* e, hipStream_t s) {
  GemmList<true> list;
  list.count = n;
  list.items = 0;
  for (int i = 0; i < n; i++) {
    const int tiles_m = (g[i].M + BM - 1) / BM, tiles_n = (g[i].N + BM - 1) / BM;
    list.p[i] = GemmItem{(const bf16_t*)g[i].A, (const bf16_t*)g[i].B, (float*)g[i].C, g[i].colsum, g[i].lda, g[i].ldb, g[i].ldc, g[i].M, g[i].N,
                         tiles_m, tiles_n, e[i].group ? e[i].group : 4,  // (the side-by-side walk belongs to launches of one product)
                         e[i].a_lim, e[i].b_lim, list.items};
    list.items += tiles_m * tiles_n;
  }
  return g[0].accumulate ? launch_mfma<BM, BM, false, false, EK_F32 | EM_RES | EM_COLSUM, EDGE, true>(g[0], e[0], s, list)
                         : launch_mfma<BM, BM, false, false, EK_F32 | EM_COLSUM, EDGE, true>(g[0], e[0], s, list);
}

int gemm_mfma_group(const GemmArgs* g, int n, const EpiArgs* e, int tile, bool edge, hipStream_t s) {
  if (tile == 256) return edge ? group_t<256, true>(g, n, e, s) : group_t<256, false>(g, n, e, s);
  return edge ? group_t<128, true>(g, n, e, s) : group_t<128, false>(g, n, e, s);
}

}  // namespace fax
