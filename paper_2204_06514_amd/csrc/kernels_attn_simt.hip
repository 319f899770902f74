// Causal attention with scalar FMAs: the fallback for head widths and alignments that the matrix-core kernels do not
// cover, and the form a caller gets by asking for it.  One wavefront per query row (forward, dQ) or per key row (dK, dV);
// the rows themselves are in attn_rows.h.
// No atomics: every output element has exactly one writer.
#include "attn_rows.h"

namespace fax {

static constexpr int AT_MAXDH = 256;  // lane owns d = lane + 64 r, r < 4

template <typename T>
__global__ __launch_bounds__(256) void attn_fwd_simt_kernel(int S, int H, int dh, const T* __restrict__ qkv,
                                                            T* __restrict__ ctx, float* __restrict__ lse) {
  __shared__ float qs[4][AT_MAXDH];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int b = blockIdx.y / H, h = blockIdx.y % H;
  const int Hd = H * dh, ld = 3 * Hd;
  const int i = blockIdx.x * 4 + wave;
  const T* base = qkv + (size_t)b * S * ld + h * dh;
  if (i < S)
    for (int d = lane; d < dh; d += 64) qs[wave][d] = to_f(base[(size_t)i * ld + d]);
  __syncthreads();
  if (i >= S) return;
  attn_fwd_row<AT_MAXDH / 64>(qs[wave], i, lane, base, ld, Hd, dh, ctx + ((size_t)b * S + i) * Hd + h * dh,
                              lse + ((size_t)b * H + h) * S + i);
}

// delta[b,h,i] = sum_d dO[i,d] O[i,d]
template <typename T>
__global__ __launch_bounds__(256) void attn_delta_kernel(int S, int H, int dh, const T* __restrict__ ctx,
                                                         const T* __restrict__ dctx, float* __restrict__ delta) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int b = blockIdx.y / H, h = blockIdx.y % H;
  const int i = blockIdx.x * 4 + wave;
  if (i >= S) return;
  const size_t off = ((size_t)b * S + i) * H * dh + h * dh;
  float s = 0.f;
  for (int d = lane; d < dh; d += 64) s += to_f(ctx[off + d]) * to_f(dctx[off + d]);
  s = wave_sum(s);
  if (lane == 0) delta[((size_t)b * H + h) * S + i] = s;
}

template <typename T>
__global__ __launch_bounds__(256) void attn_bwd_dq_simt_kernel(int S, int H, int dh, const T* __restrict__ qkv,
                                                               const float* __restrict__ lse,
                                                               const float* __restrict__ delta,
                                                               const T* __restrict__ dctx, T* __restrict__ dqkv) {
  __shared__ float qs[4][AT_MAXDH];
  __shared__ float dos[4][AT_MAXDH];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int b = blockIdx.y / H, h = blockIdx.y % H;
  const int Hd = H * dh, ld = 3 * Hd;
  const int i = blockIdx.x * 4 + wave;
  const T* base = qkv + (size_t)b * S * ld + h * dh;
  if (i < S)
    for (int d = lane; d < dh; d += 64) {
      qs[wave][d] = to_f(base[(size_t)i * ld + d]);
      dos[wave][d] = to_f(dctx[((size_t)b * S + i) * Hd + h * dh + d]);
    }
  __syncthreads();
  if (i >= S) return;
  attn_bwd_dq_row<AT_MAXDH / 64>(qs[wave], dos[wave], i, lane, lse[((size_t)b * H + h) * S + i], delta[((size_t)b * H + h) * S + i],
                                 base, ld, Hd, dh, dqkv + ((size_t)b * S + i) * ld + h * dh);
}

template <typename T>
__global__ __launch_bounds__(256) void attn_bwd_dkv_simt_kernel(int S, int H, int dh, const T* __restrict__ qkv,
                                                                const float* __restrict__ lse,
                                                                const float* __restrict__ delta,
                                                                const T* __restrict__ dctx, T* __restrict__ dqkv) {
  __shared__ float ks[4][AT_MAXDH];
  __shared__ float vs[4][AT_MAXDH];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int b = blockIdx.y / H, h = blockIdx.y % H;
  const int Hd = H * dh, ld = 3 * Hd;
  const int j = blockIdx.x * 4 + wave;
  const T* base = qkv + (size_t)b * S * ld + h * dh;
  const T* dob = dctx + (size_t)b * S * Hd + h * dh;
  if (j < S)
    for (int d = lane; d < dh; d += 64) {
      ks[wave][d] = to_f(base[(size_t)j * ld + Hd + d]);
      vs[wave][d] = to_f(base[(size_t)j * ld + 2 * Hd + d]);
    }
  __syncthreads();
  if (j >= S) return;
  T* out = dqkv + ((size_t)b * S + j) * ld + h * dh;
  attn_bwd_dkv_row<AT_MAXDH / 64>(ks[wave], vs[wave], j, S, lane, base, ld, dob, Hd, dh, lse + ((size_t)b * H + h) * S,
                                  delta + ((size_t)b * H + h) * S, out + Hd, out + 2 * Hd);
}

int attn_delta(int dtype, int B, int S, int H, int dh, const void* ctx, const void* dctx, float* delta, hipStream_t s) {
  dim3 grid((S + 3) / 4, B * H);
  if (dtype == FAX_F32)
    hipLaunchKernelGGL((attn_delta_kernel<float>), grid, dim3(256), 0, s, S, H, dh, (const float*)ctx, (const float*)dctx,
                       delta);
  else
    hipLaunchKernelGGL((attn_delta_kernel<bf16_t>), grid, dim3(256), 0, s, S, H, dh, (const bf16_t*)ctx,
                       (const bf16_t*)dctx, delta);
  FAX_LAUNCH_CHECK("attn_delta");
  return FAX_OK;
}

template <typename T>
static int attn_fwd_simt_t(int B, int S, int H, int dh, const T* qkv, T* ctx, float* lse, hipStream_t s) {
  dim3 grid((S + 3) / 4, B * H);
  hipLaunchKernelGGL((attn_fwd_simt_kernel<T>), grid, dim3(256), 0, s, S, H, dh, qkv, ctx, lse);
  FAX_LAUNCH_CHECK("attn_fwd_simt");
  return FAX_OK;
}

int attn_fwd_simt(int dtype, int B, int S, int H, int dh, const void* qkv, void* ctx, float* lse, hipStream_t s) {
  if (dh > AT_MAXDH) {
    set_error("attention: head width %d exceeds %d", dh, AT_MAXDH);
    return FAX_ERR_UNSUPPORTED;
  }
  if (B * H == 0 || S == 0) return FAX_OK;
  if (dtype == FAX_F32) return attn_fwd_simt_t<float>(B, S, H, dh, (const float*)qkv, (float*)ctx, lse, s);
  return attn_fwd_simt_t<bf16_t>(B, S, H, dh, (const bf16_t*)qkv, (bf16_t*)ctx, lse, s);
}

template <typename T>
static int attn_bwd_simt_t(int B, int S, int H, int dh, const T* qkv, const T* ctx, const float* lse, const T* dctx,
                           T* dqkv, float* delta, hipStream_t s) {
  dim3 grid((S + 3) / 4, B * H);
  hipLaunchKernelGGL((attn_delta_kernel<T>), grid, dim3(256), 0, s, S, H, dh, ctx, dctx, delta);
  hipLaunchKernelGGL((attn_bwd_dq_simt_kernel<T>), grid, dim3(256), 0, s, S, H, dh, qkv, lse, delta, dctx, dqkv);
  hipLaunchKernelGGL((attn_bwd_dkv_simt_kernel<T>), grid, dim3(256), 0, s, S, H, dh, qkv, lse, delta, dctx, dqkv);
  FAX_LAUNCH_CHECK("attn_bwd_simt");
  return FAX_OK;
}

int attn_bwd_simt(int dtype, int B, int S, int H, int dh, const void* qkv, const void* ctx, const float* lse,
                  const void* dctx, void* dqkv, float* delta, hipStream_t s) {
  if (dh > AT_MAXDH) {
    set_error("attention: head width %d exceeds %d", dh, AT_MAXDH);
    return FAX_ERR_UNSUPPORTED;
  }
  if (B * H == 0 || S == 0) return FAX_OK;
  if (dtype == FAX_F32)
    return attn_bwd_simt_t<float>(B, S, H, dh, (const float*)qkv, (const float*)ctx, lse, (const float*)dctx,
                                  (float*)dqkv, delta, s);
  return attn_bwd_simt_t<bf16_t>(B, S, H, dh, (const bf16_t*)qkv, (const bf16_t*)ctx, lse, (const bf16_t*)dctx,
                                 (bf16_t*)dqkv, delta, s);
}

}  // namespace fax
