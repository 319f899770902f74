// The loss of a validation step without its logits: the output projection's tiles leave, of every row, a maximum and a sum of exponentials for
// each 128 (64) columns (gemm_mfma_kernel.h, EK_LSE), and one kernel makes the row's loss of them.
#include "gemm_mfma_kernel.h"

namespace fax {

static constexpr int LSE_ROWS = 64, LSE_WAVES = 16;

// A workgroup takes 64 rows: its waves share the parts, a row to a lane, and then the rows' label logits, which are 64-wide dot products of the hidden
// state with the label's row of the embedding.  Bound by reading both and the parts: 16384 rows, 394 parts, D 768: 100 MB in
// 17 us.
__global__ __launch_bounds__(64 * LSE_WAVES) void lse_row_loss_kernel(int M, int N, int D, int parts, const float2* __restrict__ part, const bf16_t* __restrict__ hf,
                                                                      const bf16_t* __restrict__ emb, const int32_t* __restrict__ labels,
                                                                      float* __restrict__ row_loss) {
  __shared__ float tops[LSE_WAVES][LSE_ROWS], sums[LSE_WAVES][LSE_ROWS], label_logit[LSE_ROWS];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m0 = blockIdx.x * LSE_ROWS, m = min(m0 + lane, M - 1);
  auto join = [](float& top, float& sum, float2 p) {  // a part with -infinity has no elements, or none that count
    const float t = __builtin_elementwise_maximum(top, p.x);
    sum = (top == -INFINITY ? 0.f : sum * __builtin_amdgcn_exp2f((top - t) * LSE_LOG2E)) +
          (p.x == -INFINITY ? 0.f : p.y * __builtin_amdgcn_exp2f((p.x - t) * LSE_LOG2E));
    top = t;
  };
  float top = -INFINITY, sum = 0.f;
#pragma unroll 4
  for (int p = wave; p < parts; p += LSE_WAVES) join(top, sum, part[(size_t)p * M + m]);
  tops[wave][lane] = top;
  sums[wave][lane] = sum;
  for (int r = wave; r < LSE_ROWS && m0 + r < M; r += LSE_WAVES) {
    const bf16_t *x = hf + (size_t)(m0 + r) * D, *w = emb + (size_t)min(max(labels[m0 + r], 0), N - 1) * D;
    float z = 0.f;
    for (int d = lane * 8; d < D; d += 512) {
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(x + d), b = *reinterpret_cast<const bf16x8*>(w + d);
#pragma unroll
      for (int k = 0; k < 8; k++) z = fmaf((float)a[k], (float)b[k], z);
    }
    z = wave_sum(z);
    if (lane == 0) label_logit[r] = z;
  }
  __syncthreads();
  if (wave == 0 && m0 + lane < M) {
    for (int w = 1; w < LSE_WAVES; w++) join(top, sum, make_float2(tops[w][lane], sums[w][lane]));
    // The label's logit is summed in another order than the tiles' and may come out above the largest of them: no loss below zero.  v_log_f32 is log2.
    const float loss = (top - label_logit[lane]) + __builtin_amdgcn_logf(sum) * 0.6931471805599453f;
    row_loss[m0 + lane] = loss < 0.f ? 0.f : loss;
  }
}

// Bulk and strip of the output projection: whole 256 x 256 tiles with the last 128 columns on 256 x 128 ones (128 columns: nothing but those), or
// masked tiles, also for those columns where their tiles find room in the others' last round.  The strip's launch takes as long as a round
// of its tiles, us, strip and masked: 256 x 50304 x 2048 73 and 52, 4096 x 3200 x 768 37 and 27, 2048 x 16768 x 768 78 and 71; with a round more the other way, 4096 x
// 4224 x 768 40 and 47, 8192 x 8320 x 768 108 and 117.
struct LsePlan { bool edge; int bulk, parts; };
static LsePlan lse_plan(int M, int N, int K) {
  const int rows = (M + 255) / 256;
  auto rounds = [&](int n) { return ((long long)rows * ((n + 255) / 256) + 255) / 256; };
  const bool edge = M % 256 || N % 128 || K % GK || (N % 256 && rounds(N) == rounds(N / 256 * 256));
  const int bulk = edge ? N : N / 256 * 256;
  return LsePlan{edge, bulk, 2 * ((bulk + 255) / 256) + (bulk < N ? 2 : 0)};
}

// hf [M, K], emb [N, K], both densely stored; `logits` the product with them stored.  What it saves is the logits' way to memory and back: 16384 x 50304 x
// 768 1450 -> 1160 us.  From 192 tiles on, below which 256 x 256 ones leave too many CUs idle, and where the tiles and the rows' kernel (11 us and 2.7 for every 1000 of
// width) are predicted to take less than the product in the tiles it takes by itself and the kernel over its rows (9 us, 0.27 a megabyte and 0.8 for every 1000 rows).
// Validation steps of one narrow layer, stored logits and this, us (tokens x columns x width): 256 x 50304 x 768 75.2 and 72.5, 1024 x 12928 x 2048 121 and 118, 1024 x 21938 x
// 1600 142.5 and 141.7, 4096 x 8448 x 768 153 and 141, 2048 x 13000 x 768 119 and 106, 4096 x 12672 x 2048 332 and 307;  on the other side,
// where the product takes other tiles, 4096 x 8448 x 2048 239 and 241, 4096 x 8576 x 2048 246 and 255, 1111 x 16000 x 2048 164 and
// 162, 4096 x 4224 x 2048 184.5 either way.
bool lse_loss_supported(const GemmArgs& logits, int N) {
  const int M = logits.M, K = logits.K;
  const uintptr_t at = reinterpret_cast<uintptr_t>(logits.A) | reinterpret_cast<uintptr_t>(logits.B);
  if (!(logits.dtype == FAX_BF16 && K % 8 == 0 && (at & 15) == 0 && (long long)((M + 255) / 256) * ((N + 255) / 256) >= 192)) return false;
  const LsePlan plan = lse_plan(M, N, K);
  double us = 11.0 + 2.7e-3 * K;
  if (plan.bulk) us += 3.0 + gemm_tiles_us(256, 256, M, plan.bulk, K);
  if (plan.bulk < N) us += 3.0 + gemm_tiles_us(256, 128, M, N - plan.bulk, K);
  return us < 0.98 * (gemm_time_estimate_us(logits) + 9.0 + 0.27 * (2e-6 * M * N) + 0.8e-3 * M);
}
size_t lse_loss_ws_bytes(int M, int N, int K) { return (size_t)lse_plan(M, N, K).parts * M * sizeof(float2); }

int lse_loss(int M, int N, int K, const void* hf, const void* emb, const int32_t* labels, void* ws, float* row_loss, float* loss_out, hipStream_t s) {
  const LsePlan plan = lse_plan(M, N, K);
  {
    Timed t("gemm_mfma_Ak_Bk_lse", WORK_FLOP, 2.0 * M * N * K, s);
    GemmArgs g = dense_product(FAX_BF16, false, true, M, plan.bulk, K, false);
    g.A = hf; g.B = emb; g.C = ws; g.ldc = M;
    EpiArgs e{};
    e.C = g.C; e.ldc = M; e.splits = 1; e.group = gemm_walk_group((M + 255) / 256, (plan.bulk + 255) / 256, K, 1); e.a_lim = M; e.b_lim = N;
    if (plan.edge) {
      FAX_TRY((launch_mfma<256, 256, true, true, EK_LSE, true>(g, e, s)));
    } else {
      if (plan.bulk) FAX_TRY((launch_mfma<256, 256, true, true, EK_LSE>(g, e, s)));
      if (plan.bulk < N) {
        g.N = N - plan.bulk;
        g.B = (const bf16_t*)emb + (size_t)plan.bulk * K;
        e.C = (float2*)ws + (size_t)(plan.parts - 2) * M;
        FAX_TRY((launch_mfma<256, 128, true, true, EK_LSE>(g, e, s)));
      }
    }
  }
  Timed t("lse_row_loss", WORK_BYTE, (double)plan.parts * M * sizeof(float2) + 4.0 * M * K, s);
  hipLaunchKernelGGL(lse_row_loss_kernel, dim3((M + LSE_ROWS - 1) / LSE_ROWS), dim3(64 * LSE_WAVES), 0, s, M, N, K, plan.parts, (const float2*)ws,
                     (const bf16_t*)hf, (const bf16_t*)emb, labels, row_loss);
  FAX_LAUNCH_CHECK("lse_row_loss");
  return mean_loss(M, row_loss, loss_out, s);
}

}  // namespace fax
