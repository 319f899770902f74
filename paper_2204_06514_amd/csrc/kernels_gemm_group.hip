// The grouped flavours of the bf16 GEMM (gemm_mfma_kernel.h with GROUP): the weight gradients of one layer in one launch.
#include "gemm_mfma_kernel.h"

namespace fax {

template <int BM>
static GemmList<true> group_list(const GemmArgs* g, int n, const EpiArgs* e) {
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
  return list;
}

template <int BM, bool EDGE>
static int group_t(const GemmArgs* g, int n, const EpiArgs* e, hipStream_t s) {
  const GemmList<true> list = group_list<BM>(g, n, e);
  return g[0].accumulate ? launch_mfma<BM, BM, false, false, EK_F32 | EM_RES | EM_COLSUM, EDGE, true>(g[0], e[0], s, list)
                         : launch_mfma<BM, BM, false, false, EK_F32 | EM_COLSUM, EDGE, true>(g[0], e[0], s, list);
}

int gemm_mfma_group(const GemmArgs* g, int n, const EpiArgs* e, int tile, bool edge, hipStream_t s) {
  if (tile == 256) return edge ? group_t<256, true>(g, n, e, s) : group_t<256, false>(g, n, e, s);
  return edge ? group_t<128, true>(g, n, e, s) : group_t<128, false>(g, n, e, s);
}

// The same with an input-gradient product that does not depend on them, on the CUs that the weight gradients' rounds leave over: the
// first workgroups share the weight gradients' tiles, the others the input gradient's, each with the code and the bits of a launch of its own.
struct InputProduct {
  int M, N, K;
  const bf16_t* A;
  int lda;
  const bf16_t* B;
  int ldb;
  EpiArgs e;
  int tiles_m, tiles_n;
};

// Bound, with every CU busy, by the chip's power like the large products.  8192 tokens x 1024, F 4096: the 192 tiles of weight gradients took
// 213 us on as many CUs and the input gradient of the QKV projection 51 after them; together 230 (1.1 PFLOP/s).
template <int BN, int EM, bool EDGE>
__global__ __launch_bounds__(256) void gemm_group_input_kernel(int first, int K, EpiArgs we, GemmList<true> list, InputProduct d) {
  const int block = blockIdx.x;
  if (block < first) {
    const GemmItem& g = list.p[0];
    mfma_tiles<256, 256, false, false, EM, EDGE, true>(block, first, g.M, g.N, K, g.A, g.lda, g.B, g.ldb, we, g.tiles_m, g.tiles_n, list);
  } else {
    mfma_tiles<256, BN, true, true, EK_STORE, EDGE, false>(block - first, gridDim.x - first, d.M, d.N, d.K, d.A, d.lda, d.B, d.ldb, d.e, d.tiles_m,
                                                           d.tiles_n, GemmList<false>());
  }
}

template <int BN, int EM, bool EDGE>
static int group_input_t(const GemmArgs* g, int n, const EpiArgs* e, int first, int blocks, const InputProduct& d, hipStream_t s) {
  constexpr size_t lds = mfma_lds<256, 256>();
  auto kern = gemm_group_input_kernel<BN, EM, EDGE>;
  static bool configured = false;  // benign race: the attribute is idempotent
  if (!configured) {
    FAX_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    configured = true;
  }
  hipLaunchKernelGGL(kern, dim3(first + blocks), dim3(256), lds, s, first, g[0].K, e[0], group_list<256>(g, n, e), d);
  FAX_LAUNCH_CHECK("gemm_group_input");
  return FAX_OK;
}

int gemm_mfma_group_input(const GemmArgs* g, int n, const EpiArgs* e, int first, int blocks, const GemmArgs& d, const EpiArgs& de, int tile_n, bool edge,
                          hipStream_t s) {
  InputProduct p{d.M, d.N, d.K, (const bf16_t*)d.A, d.lda, (const bf16_t*)d.B, d.ldb, de, (d.M + 255) / 256, (d.N + tile_n - 1) / tile_n};
  if (p.e.group == 0) p.e.group = 4;
  constexpr int EM = EK_F32 | EM_COLSUM;
  auto by_edge = [&](auto bn, auto em) -> int {
    constexpr int BN = decltype(bn)::value, E = decltype(em)::value;
    return edge ? group_input_t<BN, E, true>(g, n, e, first, blocks, p, s) : group_input_t<BN, E, false>(g, n, e, first, blocks, p, s);
  };
  if (tile_n == 256) return g[0].accumulate ? by_edge(I<256>{}, I<EM | EM_RES>{}) : by_edge(I<256>{}, I<EM>{});
  return g[0].accumulate ? by_edge(I<128>{}, I<EM | EM_RES>{}) : by_edge(I<128>{}, I<EM>{});
}

}  // namespace fax
