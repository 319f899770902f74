// One row of causal attention with scalar FMAs, by one wavefront: the bodies of the scalar kernels, and what the masked-edge
// matrix-core kernels run again for a row that came out as NaN.  Scores are never materialised: a 64-key (64-query) chunk at a time,
// a lane per pair, and only pairs under the mask are touched.  The own rows (`q`, `dorow`, `krow`, `vrow`: fp32 in LDS or the tensors
// themselves) are read at the same place by all lanes.  R: 64-wide pieces of the head width.
#pragma once
#include "fax_internal.h"

namespace fax {

template <typename A, typename T>
__device__ __forceinline__ float dot_row(const A* __restrict__ a, const T* __restrict__ row, int dh) {
  float s = 0.f;
  for (int d = 0; d < dh; d++) s = fmaf(to_f(a[d]), to_f(row[d]), s);
  return s;
}

// Query i: `base` is the head's Q, row 0, rows `ld` apart; K and V follow at +Hd and +2 Hd.
template <int R, typename A, typename T>
__device__ __forceinline__ void attn_fwd_row(const A* q, int i, int lane, const T* __restrict__ base, size_t ld, int Hd, int dh,
                                             T* __restrict__ out, float* __restrict__ lse_i) {
  const float scale = rsqrtf((float)dh);
  float m = -INFINITY, l = 0.f, acc[R];
#pragma unroll
  for (int r = 0; r < R; r++) acc[r] = 0.f;
  for (int j0 = 0; j0 <= i; j0 += 64) {
    const int j = j0 + lane;
    const bool ok = j <= i;
    float sc = ok ? dot_row(q, base + (size_t)j * ld + Hd, dh) * scale : -INFINITY;
    const float mn = fmaxf(m, wave_max(sc));
    const float p = ok ? expf(sc - mn) : 0.f;
    const float corr = expf(m - mn);
    l = l * corr + wave_sum(p);
#pragma unroll
    for (int r = 0; r < R; r++) acc[r] *= corr;
    const int nj = min(64, i - j0 + 1);
    for (int jj = 0; jj < nj; jj++) {
      const float pj = __shfl(p, jj, 64);
      const T* vr = base + (size_t)(j0 + jj) * ld + 2 * Hd;
#pragma unroll
      for (int r = 0; r < R; r++) {
        const int d = lane + 64 * r;
        if (d < dh) acc[r] = fmaf(pj, to_f(vr[d]), acc[r]);
      }
    }
    m = mn;
  }
  const float inv = 1.f / l;
#pragma unroll
  for (int r = 0; r < R; r++) {
    const int d = lane + 64 * r;
    if (d < dh) out[d] = from_f<T>(acc[r] * inv);
  }
  if (lane == 0) *lse_i = m + logf(l);
}

// dQ of query i, whose log-sum-exp and delta are li and di.
template <int R, typename A, typename T>
__device__ __forceinline__ void attn_bwd_dq_row(const A* q, const A* dorow, int i, int lane, float li, float di,
                                                const T* __restrict__ base, size_t ld, int Hd, int dh, T* __restrict__ out) {
  const float scale = rsqrtf((float)dh);
  float acc[R];
#pragma unroll
  for (int r = 0; r < R; r++) acc[r] = 0.f;
  for (int j0 = 0; j0 <= i; j0 += 64) {
    const int j = j0 + lane;
    float ds = 0.f;
    if (j <= i) {
      const float sc = dot_row(q, base + (size_t)j * ld + Hd, dh) * scale;
      const float p = expf(sc - li);
      const float dp = dot_row(dorow, base + (size_t)j * ld + 2 * Hd, dh);
      ds = p * (dp - di);
    }
    const int nj = min(64, i - j0 + 1);
    for (int jj = 0; jj < nj; jj++) {
      const float dsj = __shfl(ds, jj, 64);
      const T* kr = base + (size_t)(j0 + jj) * ld + Hd;
#pragma unroll
      for (int r = 0; r < R; r++) {
        const int d = lane + 64 * r;
        if (d < dh) acc[r] = fmaf(dsj, to_f(kr[d]), acc[r]);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < R; r++) {
    const int d = lane + 64 * r;
    if (d < dh) out[d] = from_f<T>(acc[r] * scale);
  }
}

// dK and dV of key j; `dob`, `lrow`, `drow`: the head's dO, log-sum-exps and deltas from row 0.
template <int R, typename A, typename T>
__device__ __forceinline__ void attn_bwd_dkv_row(const A* krow, const A* vrow, int j, int S, int lane, const T* __restrict__ base,
                                                 size_t ld, const T* __restrict__ dob, int Hd, int dh,
                                                 const float* __restrict__ lrow, const float* __restrict__ drow,
                                                 T* __restrict__ dk_out, T* __restrict__ dv_out) {
  const float scale = rsqrtf((float)dh);
  float ak[R], av[R];
#pragma unroll
  for (int r = 0; r < R; r++) ak[r] = av[r] = 0.f;
  for (int i0 = j; i0 < S; i0 += 64) {
    const int i = i0 + lane;
    float p = 0.f, ds = 0.f;
    if (i < S) {
      const float sc = dot_row(krow, base + (size_t)i * ld, dh) * scale;
      p = expf(sc - lrow[i]);
      const float dp = dot_row(vrow, dob + (size_t)i * Hd, dh);
      ds = p * (dp - drow[i]);
    }
    const int ni = min(64, S - i0);
    for (int ii = 0; ii < ni; ii++) {
      const float pi = __shfl(p, ii, 64), dsi = __shfl(ds, ii, 64);
      const T* qr = base + (size_t)(i0 + ii) * ld;
      const T* dor = dob + (size_t)(i0 + ii) * Hd;
#pragma unroll
      for (int r = 0; r < R; r++) {
        const int d = lane + 64 * r;
        if (d < dh) {
          av[r] = fmaf(pi, to_f(dor[d]), av[r]);
          ak[r] = fmaf(dsi, to_f(qr[d]), ak[r]);
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < R; r++) {
    const int d = lane + 64 * r;
    if (d < dh) {
      dk_out[d] = from_f<T>(ak[r] * scale);
      dv_out[d] = from_f<T>(av[r]);
    }
  }
}

}  // namespace fax
