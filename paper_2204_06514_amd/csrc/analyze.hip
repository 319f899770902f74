// Host-side static analysis of a model on a data x tensor device mesh: what one device holds and
// does per training step, and how long this library would take for it on one MI355X.
//
// The paper observes that such figures follow from the model's description alone (Sec. 2.1:
// memory requirements, latency estimates) and places tensors on a logical device mesh by naming
// the mesh axis each tensor axis is split over (Sec. 2.2); its tensor parallelism splits heads and
// every large weight over the model axis and requires the head count to divide (Sec. 3.2).
// Nothing here touches a GPU; sizes come from the same layout functions the entry points use and
// product times from the planners of the kernels that run them, and attention is priced by the form that takes it, so the
// analysis cannot drift from the code.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "fax_internal.h"

namespace fax {

// Microseconds of one layer's attention, forward and backward, by the form that attention_fwd and attention_bwd take: the
// larger of what the chip needs for all (query, key) pairs under the causal mask (nanoseconds per 1000 pairs, measured at S =
// 2000 to 2048 with 128 (b, h) problems) and what one workgroup needs for its chain of tiles, with its launches (from shapes of 1 to
// 180 workgroups).  The bf16 kernels give two 128-row tiles of a head to a workgroup, one after the other, in steps of 64 of the
// other index, or share a tile of few heads among two or four groups of waves; the fp32 ones 32 rows, a quarter of whose 32-wide steps
// fall to each wave.  Measured and predicted, us: bf16, 4 x 777, 8 heads of 64 17 + 45 / 18 + 61, 45 heads of 1000 x 80 33 + 102 /
// 31 + 86, 5 of 2048 x 128 23 + 48 / 24 + 59, 8 of 256 x 64 8 + 11 / 8 + 19; fp32, 64
// heads of 512 x 64 39 + 111 / 23 + 80, 4 of 2000 x 128 89 + 180 / 88 + 185.  Scalar kernels: 64 heads of 1000 x 60 1559 + 3632 /
// 1760 + 4288, of 1000 x 256 4875 + 13815 / 4896 + 13069.
struct AttnCost {
  double fwd, bwd;
};
static AttnCost attn_cost_us(const FaxBlockDims& b) {
  const double pairs = (double)b.B * b.H * b.S * b.S / 2.0;
  AttnCost rate, chain{0.0, 0.0};
  if (attn_edge_supported(b.dtype, b.B, b.S, b.H, b.dh)) {
    const double tiles = 2.0 * ((b.S + 127) / 128 + 1);
    const bool fwd_split = attn_fwd_form(b.B, b.S, b.H, b.dh).groups > 1, bwd_split = attn_bwd_form(b.B, b.S, b.H, b.dh).groups > 1;
    if (attn_mfma_supported(b.dtype, b.B, b.S, b.H, b.dh)) {
      rate = b.dh == 64 ? AttnCost{0.32, 1.05} : AttnCost{0.59, 2.32};
      chain = {fwd_split ? 4.0 + 0.6 * tiles : 3.0 + 1.1 * tiles, bwd_split ? 10.0 + 1.45 * tiles : 9.0 + 2.7 * tiles};
    } else {
      rate = b.dh <= 64 ? AttnCost{0.70, 2.2} : b.dh <= 96 ? AttnCost{0.81, 2.6} : AttnCost{1.0, 3.2};
      chain = {fwd_split ? 4.0 + (b.dh <= 64 ? 0.9 : 1.5) * tiles : 3.0 + (b.dh <= 64 ? 1.6 : 2.1) * tiles,
               bwd_split ? 10.0 + (b.dh <= 64 ? 3.2 : 4.2) * tiles : 9.0 + 5.2 * tiles};
    }
  } else if (attn_f32_supported(b.dtype, b.dh, nullptr, nullptr, nullptr, nullptr)) {
    const int width = (b.dh + 31) / 32 * 32;
    const double tiles = ((b.S + 31) / 32 + 3) / 4, whole = b.dh == width ? 1.0 : 1.15;
    rate = width == 32 ? AttnCost{1.6, 5.7} : width == 64 ? AttnCost{2.8, 9.6} : width == 96 ? AttnCost{4.5, 18.0} : AttnCost{5.7, 23.0};
    rate = {rate.fwd * whole, rate.bwd * whole};
    chain = {3.0 + (1.5 + 0.03 * width) * tiles, 9.0 + (2.0 + 0.07 * width) * tiles};
  } else {
    rate = b.dtype == FAX_BF16 ? AttnCost{25.0 + 0.5 * b.dh, 50.0 + 1.4 * b.dh} : AttnCost{30.0 + 0.6 * b.dh, 40.0 + 2.55 * b.dh};
  }
  return {std::max(pairs * rate.fwd * 1e-6, chain.fwd), std::max(pairs * rate.bwd * 1e-6, chain.bwd)};
}

static double block_params(double D, double Hd, double F) {
  return D * 3 * Hd + 3 * Hd + Hd * D + D + 4 * D + D * F + F + F * D + D;
}

}  // namespace fax

using namespace fax;

extern "C" int fax_analyze(const FaxModelDims* g, const FaxMesh* mesh, FaxAnalysis* out) {
  if (!g || !mesh || !out) {
    set_error("fax_analyze: NULL argument");
    return FAX_ERR_INVALID_ARG;
  }
  FAX_TRY(fax_block_dims_check(&g->blk));
  if (g->L <= 0 || g->V <= 0 || g->S_max < g->blk.S) {
    set_error("model dims: L=%d V=%d S_max=%d (S=%d)", g->L, g->V, g->S_max, g->blk.S);
    return FAX_ERR_INVALID_ARG;
  }
  const int dp = mesh->data, tp = mesh->tensor;
  if (dp <= 0 || tp <= 0) {
    set_error("mesh %d x %d", dp, tp);
    return FAX_ERR_INVALID_ARG;
  }
  if (g->blk.B % dp) {
    set_error("batch %d is not divisible by the data axis (%d)", g->blk.B, dp);
    return FAX_ERR_INVALID_ARG;
  }
  if (g->blk.H % tp) {
    set_error("%d attention heads are not divisible by the tensor axis (%d)", g->blk.H, tp);
    return FAX_ERR_INVALID_ARG;
  }
  if (g->blk.F % tp) {
    set_error("feed-forward width %d is not divisible by the tensor axis (%d)", g->blk.F, tp);
    return FAX_ERR_INVALID_ARG;
  }
  FaxAnalysis a;
  memset(&a, 0, sizeof(a));
  a.local = *g;
  a.local.blk.B = g->blk.B / dp;
  a.local.blk.H = g->blk.H / tp;
  a.local.blk.F = g->blk.F / tp;
  // rows of the token table: split only into slices of whole 128-row tiles (other sizes run on the masked-edge form)
  a.local.V = g->V % (tp * 128) == 0 ? g->V / tp : g->V;
  if (tp > 1) a.local.blk.flags |= FAX_FLAG_TP_PARTIAL;
  const FaxBlockDims& b = a.local.blk;
  const int L = g->L, V = a.local.V;
  const double es = b.dtype == FAX_F32 ? 4.0 : 2.0;
  const int T = b.B * b.S, D = b.D, Hd = b.H * b.dh, F = b.F;

  // parameters
  a.params_global = L * block_params(g->blk.D, (double)g->blk.H * g->blk.dh, g->blk.F) + (double)g->V * D +
                    (double)g->S_max * D + 2.0 * D;
  a.params_local = L * block_params(D, Hd, F) + (double)V * D + (double)g->S_max * D + 2.0 * D;

  // memory, as the entry points size it
  FaxSavedLayout sl;
  FAX_TRY(fax_block_saved_layout(&b, &sl));
  size_t train_ws = 0;
  FAX_TRY(fax_train_workspace_bytes(&a.local, &train_ws));
  a.bytes_master = 4.0 * a.params_local;
  a.bytes_moments = 8.0 * a.params_local;
  a.bytes_grads = 4.0 * a.params_local;
  a.bytes_lowp = b.dtype == FAX_BF16 ? 2.0 * a.params_local : 0.0;
  a.bytes_saved = (double)L * (double)sl.total;
  a.bytes_workspace = (double)train_ws - a.bytes_saved;
  a.bytes_total = a.bytes_master + a.bytes_moments + a.bytes_grads + a.bytes_lowp + (double)train_ws;

  // work: forward GEMMs [M, N, K] of a block, the head, and their two backward products each
  const int fwd[4][3] = {{T, 3 * Hd, D}, {T, D, Hd}, {T, F, D}, {T, D, F}};
  double gemm_flop_fwd = 0, us_gemm = 0;
  for (const auto& s : fwd) {
    gemm_flop_fwd += 2.0 * s[0] * s[1] * s[2];
    us_gemm += gemm_time_estimate_us(dense_product(b.dtype, false, false, s[0], s[1], s[2], false));  // forward
    us_gemm += gemm_time_estimate_us(dense_product(b.dtype, false, true, s[0], s[2], s[1], false));   // input gradient: contraction over N
    us_gemm += gemm_time_estimate_us(dense_product(b.dtype, true, false, s[2], s[1], s[0], true));    // weight gradient: contraction over the tokens
  }
  gemm_flop_fwd *= L;
  us_gemm *= L;
  gemm_flop_fwd += 2.0 * T * (double)D * V;
  us_gemm += gemm_time_estimate_us(logits_product(a.local, nullptr, nullptr, nullptr)) +
             gemm_time_estimate_us(hidden_grad_product(a.local, nullptr, nullptr, nullptr)) +
             gemm_time_estimate_us(embedding_grad_product(a.local, nullptr, nullptr, nullptr));
  const double pairs = (double)b.B * b.H * b.S * b.S / 2.0;  // (query, key) pairs under the mask, per layer
  const double attn_flop_fwd = L * 4.0 * pairs * b.dh;
  a.flop_step = 3.0 * (gemm_flop_fwd + attn_flop_fwd);
  a.flop_step_unhalved = 3.0 * (gemm_flop_fwd + 2.0 * attn_flop_fwd);
  const AttnCost ac = attn_cost_us(b);
  a.ms_attention = L * (ac.fwd + ac.bwd) * 1e-3;
  a.ms_gemm = us_gemm * 1e-3;

  // bandwidth-bound kernels: algorithmic bytes and launches
  const double act = (double)T * D * es;
  const int n_ln = 2 * L + 1;
  double bytes = n_ln * (2 * act)              // LayerNorm forward: read x, write h
                 + n_ln * (4 * act)            // backward: read dh, x, residual gradient; write dx
                 + 2.0 * T * (double)V * es    // loss: read the logits, write their gradient over them
                 + 2 * act + 2 * act           // embedding forward and backward
                 + (28.0 + (b.dtype == FAX_BF16 ? 2.0 : 0.0)) * a.params_local;  // AdamW
  a.hbm_bytes_step = bytes;
  const int n_tensors = 12 * L + 4;
  const int bw_launches = n_ln + 2 * n_ln + 1 + 3 + n_tensors;
  a.launches = L * (4 * 3 + 3) + 3 + bw_launches;
  a.ms_bandwidth = bytes / 4.5e9 + bw_launches * 0.006;  // 4.5 TB/s sustained, ~6 us per small launch
  a.ms_step = a.ms_gemm + a.ms_attention + a.ms_bandwidth;

  // exchange volume per step and device
  a.bytes_tensor_axis = tp > 1 ? L * 4.0 * act : 0.0;       // p_attn, p_mlp forward; dh1, dh2 backward
  a.bytes_data_axis = dp > 1 ? 4.0 * a.params_local : 0.0;  // one pass over the fp32 gradients
  *out = a;
  return FAX_OK;
}
