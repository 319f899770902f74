// dK, dV of the causal flash attention at head widths above 64: the kernel on its own (attn_dkv16.h).
#include "attn_dkv16.h"

namespace fax {

template <int DW, bool EDGE, int G, int WPG>
__global__ __launch_bounds__(64 * G * WPG, 2) void attn_bwd_dkv16_mfma_kernel(int S, int H, int BH, int dh, const bf16_t* __restrict__ qkv,
                                                                          const float* __restrict__ lse, const float* __restrict__ delta,
                                                                          const bf16_t* __restrict__ dctx, bf16_t* __restrict__ dqkv) {
  attn_bwd_dkv16_mfma_body<DW, EDGE, G, WPG>(blockIdx.x, S, H, BH, dh, qkv, lse, delta, dctx, dqkv);
}

template <int DW, bool EDGE, int G, int WPG>
static int dkv16_t(int B, int S, int H, int dh, const bf16_t* qkv, const float* lse, const float* delta, const bf16_t* dctx,
                   bf16_t* dqkv, hipStream_t s) {
  constexpr size_t lds_kv = G * 2 * (2 * (size_t)TR * row_width<DW>() * 2 + 4 * 256);  // two stages of Q tile | dO tile | lse, delta
  FAX_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(attn_bwd_dkv16_mfma_kernel<DW, EDGE, G, WPG>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_kv));
  const int n_kt = (S + 16 * WPG - 1) / (16 * WPG);
  const dim3 grid((G == 1 ? (n_kt + 1) / 2 : n_kt) * B * H);
  hipLaunchKernelGGL((attn_bwd_dkv16_mfma_kernel<DW, EDGE, G, WPG>), grid, dim3(64 * G * WPG), lds_kv, s, S, H, B * H, dh, qkv, lse, delta, dctx,
                     dqkv);
  return FAX_OK;
}

int attn_bwd_dkv16_mfma(int B, int S, int H, int dh, bool edge, int groups, int waves, const bf16_t* qkv, const float* lse, const float* delta,
                        const bf16_t* dctx, bf16_t* dqkv, hipStream_t s) {
  auto run = [&](auto g, auto wpg) -> int {
    constexpr int G = decltype(g)::value, WPG = decltype(wpg)::value;
    if (!edge) return dkv16_t<128, false, G, WPG>(B, S, H, dh, qkv, lse, delta, dctx, dqkv, s);
    if (dh <= 96) return dkv16_t<96, true, G, WPG>(B, S, H, dh, qkv, lse, delta, dctx, dqkv, s);
    return dkv16_t<128, true, G, WPG>(B, S, H, dh, qkv, lse, delta, dctx, dqkv, s);
  };
  return groups == 1 ? run(I<1>{}, I<4>{}) : waves == 4 ? run(I<2>{}, I<4>{}) : run(I<2>{}, I<2>{});
}

}  // namespace fax
