// Causal flash attention on the CDNA4 matrix cores: bf16 operands, fp32 scores and statistics.  How the three kernels lay out their
// products, registers and LDS tiles: attn_mfma_common.h.
#include "attn_dkv16.h"

namespace fax {

// dK, dV at head widths above 64: kernels_attn_dkv16.hip (16 keys per wave, its own LDS swizzle)
int attn_bwd_dkv16_mfma(int B, int S, int H, int dh, bool edge, int groups, int waves, const bf16_t* qkv, const float* lse, const float* delta, const bf16_t* dctx,
                        bf16_t* dqkv, hipStream_t s);

// ---------------------------------------------------------------------------------------------
// Forward.  Wave w owns queries 128 qt + 32 w .. + 31 (B operand, in registers); 64-key tiles of
// K and V stream through two LDS buffers.  Per tile: P1 = S^T for both 32-key halves, V = online
// softmax over the 64 keys, P3 = O^T += V^T P^T.
// ---------------------------------------------------------------------------------------------
template <int DW, bool EDGE, int G, int WPG>
__global__ __launch_bounds__(64 * G * WPG, DW == 64 && !EDGE && G == 1 ? 3 : 2) void attn_fwd_mfma_kernel(int S, int H, int BH, int dh, const bf16_t* __restrict__ qkv,
                                                            bf16_t* __restrict__ ctx, float* __restrict__ lse) {
  constexpr int DH = row_width<DW>();  // row length in LDS
  constexpr int KS = DW / 16, DT = DW / 32, TB = TR * DH * 2;
  constexpr int N = 2 * KS;            // MFMAs per phase (P3: 2 halves x 2 k-steps x DT = 2 KS as well)
  constexpr int LEAD = N < 8 ? N : 8;  // fragments in flight
  constexpr int NSEG = DH / 8 / WPG;        // 1 KB load instructions per wave per tile
  constexpr int LPS = (2 * NSEG + N - 1) / N;  // loads per slot of P1
  extern __shared__ __attribute__((aligned(16))) char smem_all[];  // 2 x [K tile | V tile]
  constexpr int RT = 32 * WPG, DIAG = WPG == 4 ? 2 : 1;  // rows of a workgroup, tiles that straddle its diagonal
  const int n_qt = EDGE ? (S + RT - 1) / RT : S / RT;
  int pair, bh;
  if (G == 1) pair_of_tiles(blockIdx.x, n_qt, BH, pair, bh);
  else longest_first(blockIdx.x, BH, pair, bh);
  const int b = bh / H, h = bh % H;
  const int hw = EDGE ? dh : DW, nch = hw / 8;  // head width, in elements and in 16-byte chunks
  const int Hd = H * hw;
  const size_t ld = 3 * (size_t)Hd;
  const bf16_t* base = qkv + (size_t)b * S * ld + h * hw;
  const int lane = threadIdx.x & 63, wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 5;
  const float scale = rsqrtf((float)hw);
  const float c = scale * LOG2E;
  const int grp = G == 1 ? 0 : wave_all / WPG, wave = G == 1 ? wave_all : wave_all % WPG;
  char* const smem = smem_all + grp * (4 * TB);
  const unsigned sm = lds_addr(smem);
  if (EDGE) clear_lds(smem_all, G * 4 * TB);

  for (int pass = 0; pass < (G == 1 ? 2 : 1); pass++) {
    const int qt = pass == 0 ? n_qt - 1 - pair : pair;  // the long one first
    if (pass == 1 && qt == n_qt - 1 - pair) break;      // odd number of tiles: the middle one stands alone
    const int q0w = qt * RT + wave * 32, iq = q0w + (lane & 31);
    bf16x8 qf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ks++)
      qf[ks] = __builtin_bit_cast(bf16x8, EDGE ? edge_load16(base + (size_t)iq * ld + ks * 16 + g * 8, iq < S && ks * 2 + g < nch)
                                               : *reinterpret_cast<const uint4*>(base + (size_t)iq * ld + ks * 16 + g * 8));
#pragma unroll
    for (int ks = 0; ks < KS; ks++) settle(qf[ks]);
    // (G > 1: a group may not meet a key that some query sees for a while, or at all)
    float m = G == 1 ? -INFINITY : -3.4028235e38f, l = 0.f;
    f32x16 oacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; dt++)
#pragma unroll
      for (int v = 0; v < 16; v++) oacc[dt][v] = 0.f;

    const int n_kv = G == 1 && !EDGE ? 2 * (qt + 1) : (min((qt + 1) * RT, S) + TR - 1) / TR;
    auto tile_load = [&](int j0, int buf, int i) {
      const unsigned st = sm + buf * 2 * TB;
      if (i < NSEG) tile_dma_seg<DH, EDGE, WPG>(st, base + (size_t)j0 * ld + Hd, ld, wave, i, S - j0, nch);
      else tile_dma_seg<DH, EDGE, WPG>(st + TB, base + (size_t)j0 * ld + 2 * Hd, ld, wave, i - NSEG, S - j0, nch);
    };
    bf16x8 fr[LEAD], fc[LEAD];
    // One 64-key tile.  MASK: the tile may reach past the wave's first query.
    auto tile = [&](auto mask_c, int t) {
      constexpr bool MASK = decltype(mask_c)::value;
      const char* kt_ = smem + (t / G & 1) * 2 * TB;
      const char* vt_ = kt_ + TB;
      const int j0 = t * TR;
      const int j0n = min(t + G, n_kv - 1) * TR;  // past the end: the last tile again, into the buffer nobody reads
      auto row_frag = [&](int i) { return frag_rows<DH>(kt_, (i % 2) * 32, i / 2, lane); };
      // P3 slot i: d-tile dt = i % DT (so that MFMAs on the same accumulator are DT slots apart),
      // then key half jt and k-step hh from i / DT
      auto col_frag = [&](int i) {
        return frag_cols<DH>(vt_, (i % DT) * 32, ((i / DT) % 2) * 32 + ((i / DT) / 2) * 16, lane);
      };
#pragma unroll
      for (int i = 0; i < LEAD; i++) fr[i] = row_frag(i);  // cold start: exposed once per tile
      f32x16 s[2];
#pragma unroll
      for (int jt = 0; jt < 2; jt++)
#pragma unroll
        for (int v = 0; v < 16; v++) s[jt][v] = 0.f;
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int i = 0; i < N; i++) {
        s[i % 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % LEAD], qf[i / 2], s[i % 2], 0, 0, 0);
        if (i + LEAD < N) fr[i % LEAD] = row_frag(i + LEAD);
        else fc[i + LEAD - N] = col_frag(i + LEAD - N);
#pragma unroll
        for (int n = i * LPS; n < (i + 1) * LPS; n++)
          if (n < 2 * NSEG) tile_load(j0n, (t / G + 1) & 1, n);
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_s_setprio(0);
      // Scores stay unscaled; the softmax scale rides in the exponent: p = 2^(c s - c m), c = scale log2 e.
      if (MASK) {
#pragma unroll
        for (int jt = 0; jt < 2; jt++)
#pragma unroll
          for (int v = 0; v < 16; v++) {
            const int key = j0 + jt * 32 + (v >> 2) * 8 + g * 4 + (v & 3);
            if (key > iq) s[jt][v] = -INFINITY;
          }
      }
      float mx = -INFINITY;
#pragma unroll
      for (int jt = 0; jt < 2; jt++)
#pragma unroll
        for (int v = 0; v < 16; v++) mx = fmaxf(mx, s[jt][v]);
      mx = max32(mx);
      // The reference point of the exponentials, m, follows the running maximum lazily: it moves
      // (and the accumulators are rescaled) only when some query's maximum has risen more than
      // MAX_LAG octaves above it, which after the first few tiles is rare.  Probabilities are then
      // at most 2^MAX_LAG instead of 1; numerator, denominator and lse all use the same m, so
      // the result is the same softmax.
      // EDGE: m is in units of the scaled score.
      const float mn = fmaxf(m, EDGE ? mx * scale : mx);  // finite (G = 1): key 0 is visible to every query and comes in the first tile
      const float octaves = EDGE ? LOG2E : c;
      if (__builtin_amdgcn_ballot_w64((mn - m) * octaves > MAX_LAG) != 0) {
        const float corr = __builtin_amdgcn_exp2f((m - mn) * octaves);
        l *= corr;
#pragma unroll
        for (int dt = 0; dt < DT; dt++)
#pragma unroll
          for (int v = 0; v < 16; v++) oacc[dt][v] *= corr;
        m = mn;
      }
      const float mc = m * c;
      float rs = 0.f;
      bf16x8 pb[2][2];  // probabilities (EDGE: pc below, from the fp32 numbers in s)
#pragma unroll
      for (int jt = 0; jt < 2; jt++)
#pragma unroll
        for (int v = 0; v < 16; v++) {
          const float p = EDGE ? edge_exp(s[jt][v], scale, m) : __builtin_amdgcn_exp2f(fmaf(s[jt][v], c, -mc));
          rs += p;
          if (EDGE) s[jt][v] = p;
          else pb[jt][v >> 3][v & 7] = (__bf16)p;
        }
      rs = sum32(rs);
      l += rs;
      bf16x8 pc[2][3];  // EDGE: eight keys' probabilities in three terms, and the next eight's as they are formed between the MFMAs
      if constexpr (EDGE) {
#pragma unroll
        for (int n = 0; n < 4; n++) split3(s[0][2 * n], s[0][2 * n + 1], pc[0], n);
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int i = 0; i < N; i++) {
        const int dt = i % DT, ch = i / DT;
        if constexpr (EDGE) {
#pragma unroll
          for (int k = 0; k < 3; k++) {
            oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fc[i % LEAD], pc[ch & 1][k], oacc[dt], 0, 0, 0);
#pragma unroll
            for (int n = 0; n < 4; n++) {
              const int v = (ch + 1) / 2 * 8 + 2 * n;
              if (ch < 3 && n * 3 * DT / 4 == dt * 3 + k) split3(s[(ch + 1) % 2][v], s[(ch + 1) % 2][v + 1], pc[(ch + 1) & 1], n);
            }
            if (k < 2) __builtin_amdgcn_sched_barrier(0);
          }
        } else {
          oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fc[i % LEAD], pb[ch % 2][ch / 2], oacc[dt], 0, 0, 0);
        }
        if (i + LEAD < N) fc[i % LEAD] = col_frag(i + LEAD);
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_s_setprio(0);
      lds_dma_wait();
      __syncthreads();
    };

#pragma unroll
    for (int i = 0; i < 2 * NSEG; i++) tile_load(min(grp, n_kv - 1) * TR, 0, i);
    lds_dma_wait();
    __syncthreads();
    if (G == 1) {
      for (int t = 0; t < n_kv - 2; t++) tile(F_{}, t);
      // the last two tiles (128 keys) straddle the diagonal of this workgroup's 128 queries
      if (EDGE) {
        for (int t = max(n_kv - 2, 0); t < n_kv; t++) tile(T_{}, t);
      } else {
        tile(T_{}, n_kv - 2);
        tile(T_{}, n_kv - 1);
      }
    } else {
      int t = grp;
      for (; t < n_kv - DIAG; t += G) tile(F_{}, t);
      for (; t < n_kv; t += G) tile(T_{}, t);
      // every group meets as many barriers as the one with the most tiles
      for (t = (n_kv + G - 1) / G - (n_kv - grp + G - 1) / G; t > 0; t--) __syncthreads();
    }
    if (G > 1) {
      constexpr int U = DT * 4 + 1;
      float* x = reinterpret_cast<float*>(smem_all);
      if (grp) {
        group_put<U>(x, wave_all - WPG, 0, oacc);
        reinterpret_cast<float4*>(x)[((wave_all - WPG) * U + U - 1) * 64 + lane] = make_float4(m, l, 0.f, 0.f);
      }
      __syncthreads();
      if (grp) return;
      const float octaves = EDGE ? LOG2E : c;
#pragma unroll
      for (int o = 0; o < G - 1; o++) {
        const int slot = o * WPG + wave;
        const float4 ml = reinterpret_cast<const float4*>(x)[(slot * U + U - 1) * 64 + lane];
        const float mn = fmaxf(m, ml.x);
        const float a0 = __builtin_amdgcn_exp2f((m - mn) * octaves), a1 = __builtin_amdgcn_exp2f((ml.x - mn) * octaves);
        l = fmaf(l, a0, ml.y * a1);
        m = mn;
        group_add<U>(x, slot, 0, oacc, a0, a1);
      }
    }

    bool store = true;
    unsigned again = 0;  // rows to compute a second time, by their lane in the lower half
    if (EDGE) {
      store = iq < S;
      const unsigned long long odd = __builtin_amdgcn_ballot_w64(store && not_finite(oacc, l * 0.f) != 0.f);
      again = (unsigned)odd | (unsigned)(odd >> 32);
      store = store && !((again >> (lane & 31)) & 1);
    }
    if (store) {
      store_rows<DW, EDGE>(ctx + ((size_t)b * S + iq) * Hd + h * hw, oacc, 1.f / l, g, hw);
      if (g == 0) lse[((size_t)b * H + h) * S + iq] = EDGE ? m + logf(l) : m * scale + logf(l);
    }
    if (EDGE) {
      for (; again; again &= again - 1) {
        int lane_r = lane;
        settle(lane_r);  // nothing derived from it here is worth a register in the loops above
        const int i = q0w + __builtin_ctz(again);
        attn_fwd_row<(DW + 63) / 64>(base + (size_t)i * ld, i, lane_r, base, ld, Hd, hw, ctx + ((size_t)b * S + i) * Hd + h * hw,
                                               lse + ((size_t)b * H + h) * S + i);
      }
    }
  }  // pass
}

// ---------------------------------------------------------------------------------------------
// dQ (and delta).  Wave w owns queries 128 qt + 32 w .. + 31 (Q and dO rows in registers as B
// operands); 64-key tiles of K and V stream through two LDS buffers.  One 32-key half after the
// other:
//   P1: S^T = K Q^T and dP^T = V dO^T, alternating (row fragments of K and V, 2 KS MFMAs)
//   V:  dS^T = P^T (dP^T - delta), P^T = 2^(c S^T - lse log2 e), packed to bf16
//   P3: dQ^T += K^T dS^T (transpose-read fragments of K)
// One barrier per 64-key tile.  Registers budgeted for two waves per SIMD, LDS for two workgroups
// per CU (see above).
// ---------------------------------------------------------------------------------------------
template <int DW, bool EDGE, int G, int WPG>
__device__ __forceinline__ void attn_bwd_dq_mfma_body(int block, int S, int H, int BH, int dh, const bf16_t* __restrict__ qkv,
                                                                         const float* __restrict__ lse,
                                                                         const bf16_t* __restrict__ ctx,
                                                                         const bf16_t* __restrict__ dctx,
                                                                         float* __restrict__ delta, bool have_delta,
                                                                         bf16_t* __restrict__ dqkv) {
  constexpr int DH = row_width<DW>();  // row length in LDS
  constexpr int KS = DW / 16, DT = DW / 32, TB = TR * DH * 2;
  constexpr int N1 = 2 * KS;   // score MFMAs per 32-key half: S and dP, KS each
  constexpr int N3 = 2 * DT;   // dQ MFMAs per half: two k-steps x DT
  constexpr int LEAD = N3;     // fragments in flight
  constexpr int NSEG = DH / 8 / WPG;
  constexpr int LPS = (2 * NSEG + N1 - 1) / N1;  // loads per slot of P1
  static_assert(N1 % LEAD == 0, "slot plan");
  extern __shared__ __attribute__((aligned(16))) char smem_all[];  // 2 x [K tile | V tile]
  constexpr int RT = 32 * WPG, DIAG = WPG == 4 ? 2 : 1;  // rows of a workgroup, tiles that straddle its diagonal
  const int n_qt = EDGE ? (S + RT - 1) / RT : S / RT;
  int pair, bh;
  if (G == 1) pair_of_tiles(block, n_qt, BH, pair, bh);
  else longest_first(block, BH, pair, bh);
  const int b = bh / H, h = bh % H;
  const int hw = EDGE ? dh : DW, nch = hw / 8;  // head width, in elements and in 16-byte chunks
  const int Hd = H * hw;
  const size_t ld = 3 * (size_t)Hd;
  const bf16_t* base = qkv + (size_t)b * S * ld + h * hw;
  const int lane = threadIdx.x & 63, wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 5;
  const float scale = rsqrtf((float)hw);
  const float c = scale * LOG2E;
  const int grp = G == 1 ? 0 : wave_all / WPG, wave = G == 1 ? wave_all : wave_all % WPG;
  char* const smem = smem_all + grp * (4 * TB);
  const unsigned sm = lds_addr(smem);
  if (EDGE) clear_lds(smem_all, G * 4 * TB);

  for (int pass = 0; pass < (G == 1 ? 2 : 1); pass++) {
    const int qt = pass == 0 ? n_qt - 1 - pair : pair;
    if (pass == 1 && qt == n_qt - 1 - pair) break;
    const int q0w = qt * RT + wave * 32, iq = q0w + (lane & 31);
    bf16x8 qf[KS], dof[KS];
    const bf16_t* dorow = dctx + ((size_t)b * S + iq) * Hd + h * hw;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      const bool ok = !EDGE || (iq < S && ks * 2 + g < nch);
      const bf16_t* qp = base + (size_t)iq * ld + ks * 16 + g * 8;
      qf[ks] = __builtin_bit_cast(bf16x8, EDGE ? edge_load16(qp, ok) : *reinterpret_cast<const uint4*>(qp));
      dof[ks] = __builtin_bit_cast(bf16x8, EDGE ? edge_load16(dorow + ks * 16 + g * 8, ok)
                                                : *reinterpret_cast<const uint4*>(dorow + ks * 16 + g * 8));
    }
    float li = EDGE ? (iq >= S ? 0.f : lse[((size_t)b * H + h) * S + iq]) : lse[((size_t)b * H + h) * S + iq] * LOG2E;
    float di = 0.f;  // delta_i = sum_d dO[i, d] O[i, d], half of the row per lane
    if (have_delta) {
      if (!EDGE || iq < S) di = delta[((size_t)b * H + h) * S + iq];
    } else {
      const bf16_t* orow = ctx + ((size_t)b * S + iq) * Hd + h * hw;
#pragma unroll
      for (int ks = 0; ks < KS; ks++) {
        const bf16x8 o = __builtin_bit_cast(bf16x8, EDGE ? edge_load16(orow + ks * 16 + g * 8, iq < S && ks * 2 + g < nch)
                                                         : *reinterpret_cast<const uint4*>(orow + ks * 16 + g * 8));
#pragma unroll
        for (int e = 0; e < 8; e++) di = fmaf((float)o[e], (float)dof[ks][e], di);
      }
      di = sum32(di);
      if (g == 0 && grp == 0 && (!EDGE || iq < S)) delta[((size_t)b * H + h) * S + iq] = di;
    }
#pragma unroll
    for (int ks = 0; ks < KS; ks++) { settle(qf[ks]); settle(dof[ks]); }
    settle(li); settle(di);
    f32x16 dq[DT];
#pragma unroll
    for (int dt = 0; dt < DT; dt++)
#pragma unroll
      for (int v = 0; v < 16; v++) dq[dt][v] = 0.f;

    const int n_kv = G == 1 && !EDGE ? 2 * (qt + 1) : (min((qt + 1) * RT, S) + TR - 1) / TR;
    auto tile_load = [&](int j0, int buf, int i) {
      const unsigned st = sm + buf * 2 * TB;
      if (i < NSEG) tile_dma_seg<DH, EDGE, WPG>(st, base + (size_t)j0 * ld + Hd, ld, wave, i, S - j0, nch);
      else tile_dma_seg<DH, EDGE, WPG>(st + TB, base + (size_t)j0 * ld + 2 * Hd, ld, wave, i - NSEG, S - j0, nch);
    };
    bf16x8 f[LEAD];  // one ring for both kinds of fragment: slot i reloads the register it has just used
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // One 64-key tile, a 32-key half at a time.  MASK: the tile may reach past the wave's first query.
    auto tile = [&](auto mask_c, int t) {
      constexpr bool MASK = decltype(mask_c)::value;
      const char* kt_ = smem + (t / G & 1) * 2 * TB;
      const char* vt_ = kt_ + TB;
      const int j0n = min(t + G, n_kv - 1) * TR;  // past the end: the last tile again, into the buffer nobody reads
      // P1 slot i of half jt: S (K rows x Q) or dP (V rows x dO) by bit 0, k-step i / 2
      auto row_frag = [&](int jt, int i) { return frag_rows<DH>((i & 1) ? vt_ : kt_, jt * 32, i / 2, lane); };
      // P3 slot i of half jt: d-tile i % DT, k-step i / DT
      auto col_frag = [&](int jt, int i) { return frag_cols<DH>(kt_, (i % DT) * 32, jt * 32 + (i / DT) * 16, lane); };
#pragma unroll
      for (int i = 0; i < LEAD; i++) f[i] = row_frag(0, i);  // cold start: exposed once per tile
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int jt = 0; jt < 2; jt++) {
        f32x16 sc, dp;
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int i = 0; i < N1; i++) {
          const int ks = i / 2;
          if (i & 1) dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % LEAD], dof[ks], i < 2 ? zero : dp, 0, 0, 0);
          else sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % LEAD], qf[ks], i < 2 ? zero : sc, 0, 0, 0);
          if (i + LEAD < N1) f[i % LEAD] = row_frag(jt, i + LEAD);
          else f[i % LEAD] = col_frag(jt, i + LEAD - N1);  // (N1 is a multiple of LEAD)
#pragma unroll
          for (int n = i * LPS; n < (i + 1) * LPS; n++)
            if (jt == 0 && n < 2 * NSEG) tile_load(j0n, (t / G + 1) & 1, n);
          __builtin_amdgcn_sched_barrier(0);
        }
        bf16x8 db[2], dc[2][3];  // dS; EDGE: in three terms, the second eight keys' formed between the first one's MFMAs
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int v = 0; v < 16; v++) {
          float p = EDGE ? edge_exp(sc[v], scale, li) : __builtin_amdgcn_exp2f(fmaf(sc[v], c, -li));
          if (MASK && t * TR + jt * 32 + (v >> 2) * 8 + g * 4 + (v & 3) > iq) p = 0.f;
          const float d = p * (dp[v] - di);
          if (EDGE) dp[v] = d;
          else db[v >> 3][v & 7] = (__bf16)d;
        }
        if constexpr (EDGE) {
#pragma unroll
          for (int n = 0; n < 4; n++) split3(dp[2 * n], dp[2 * n + 1], dc[0], n);
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int i = 0; i < N3; i++) {
          if constexpr (EDGE) {
#pragma unroll
            for (int k = 0; k < 3; k++) {
              dq[i % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % LEAD], dc[i / DT][k], dq[i % DT], 0, 0, 0);
#pragma unroll
              for (int n = 0; n < 4; n++)
                if (n * 3 * DT / 4 == i * 3 + k) split3(dp[8 + 2 * n], dp[9 + 2 * n], dc[1], n);
              if (k < 2) __builtin_amdgcn_sched_barrier(0);
            }
          } else {
            dq[i % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % LEAD], db[i / DT], dq[i % DT], 0, 0, 0);
          }
          if (jt == 0) f[i % LEAD] = row_frag(1, i);  // the second half's first rows (N3 = LEAD)
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __builtin_amdgcn_s_setprio(0);
      lds_dma_wait();
      __syncthreads();
    };

#pragma unroll
    for (int i = 0; i < 2 * NSEG; i++) tile_load(min(grp, n_kv - 1) * TR, 0, i);
    lds_dma_wait();
    __syncthreads();
    if (G == 1) {
      for (int t = 0; t < n_kv - 2; t++) tile(F_{}, t);
      // the last two tiles (128 keys) straddle the diagonal of this workgroup's 128 queries
      if (EDGE) {
        for (int t = max(n_kv - 2, 0); t < n_kv; t++) tile(T_{}, t);
      } else {
        tile(T_{}, n_kv - 2);
        tile(T_{}, n_kv - 1);
      }
    } else {
      int t = grp;
      for (; t < n_kv - DIAG; t += G) tile(F_{}, t);
      for (; t < n_kv; t += G) tile(T_{}, t);
      // every group meets as many barriers as the one with the most tiles
      for (t = (n_kv + G - 1) / G - (n_kv - grp + G - 1) / G; t > 0; t--) __syncthreads();
    }
    if (G > 1) {
      constexpr int U = DT * 4;
      float* x = reinterpret_cast<float*>(smem_all);
      if (grp) group_put<U>(x, wave_all - WPG, 0, dq);
      __syncthreads();
      if (grp) return;
#pragma unroll
      for (int o = 0; o < G - 1; o++) group_add<U>(x, o * WPG + wave, 0, dq);
    }

    bool store = true;
    unsigned again = 0;  // as in the forward kernel
    if (EDGE) {
      store = iq < S;
      const unsigned long long odd = __builtin_amdgcn_ballot_w64(store && not_finite(dq, 0.f) != 0.f);
      again = (unsigned)odd | (unsigned)(odd >> 32);
      store = store && !((again >> (lane & 31)) & 1);
    }
    if (store) store_rows<DW, EDGE>(dqkv + ((size_t)b * S + iq) * ld + h * hw, dq, scale, g, hw);
    if (EDGE) {
      for (; again; again &= again - 1) {
        int lane_r = lane;
        settle(lane_r);
        const int r = __builtin_ctz(again), i = q0w + r;
        attn_bwd_dq_row<(DW + 63) / 64>(base + (size_t)i * ld, dctx + ((size_t)b * S + i) * Hd + h * hw, i, lane_r,
                                                  lse[((size_t)b * H + h) * S + i], __shfl(di, r, 64), base, ld, Hd, hw,
                                                  dqkv + ((size_t)b * S + i) * ld + h * hw);
      }
    }
  }  // pass
}

template <int DW, bool EDGE, int G, int WPG>
__global__ __launch_bounds__(64 * G * WPG, 2) void attn_bwd_dq_mfma_kernel(int S, int H, int BH, int dh, const bf16_t* __restrict__ qkv,
                                                                         const float* __restrict__ lse, const bf16_t* __restrict__ ctx,
                                                                         const bf16_t* __restrict__ dctx, float* __restrict__ delta,
                                                                         bf16_t* __restrict__ dqkv) {
  attn_bwd_dq_mfma_body<DW, EDGE, G, WPG>(blockIdx.x, S, H, BH, dh, qkv, lse, ctx, dctx, delta, false, dqkv);
}

// ---------------------------------------------------------------------------------------------
// dK, dV without the skew (used for DH = 64, where the kernel then fits the register budget of
// two waves per SIMD and several workgroups share a CU).  The same arithmetic as the kernel above,
// a 32-query half at a time: P1 = S and dP (2 KS MFMAs), V = P and dS packed to bf16, P3 = dV^T and
// dK^T (2 KS MFMAs); two LDS buffers, one barrier per 64-query tile.
// ---------------------------------------------------------------------------------------------
template <int DW, bool EDGE, int G, int WPG>
__device__ __forceinline__ void attn_bwd_dkv_phased_mfma_body(int block, int S, int H, int BH, int dh, const bf16_t* __restrict__ qkv,
                                                                          const float* __restrict__ lse,
                                                                          const float* __restrict__ delta,
                                                                          const bf16_t* __restrict__ dctx,
                                                                          bf16_t* __restrict__ dqkv) {
  constexpr int DH = row_width<DW>();  // row length in LDS
  constexpr int KS = DW / 16, DT = DW / 32, TB = TR * DH * 2;
  constexpr int LD_OFF = 2 * TB, STAGE = 2 * TB + 4 * 256;  // Q tile | dO tile | lse and delta as above
  constexpr int N = 2 * KS;                   // MFMAs per phase and half
  constexpr int LEAD = N < 8 ? N : 8;         // fragments in flight
  constexpr int NSEG = DH / 8 / WPG;
  static_assert(N % LEAD == 0 && N > 0, "slot plan");
  constexpr int LOADS = 2 * NSEG + 4 / WPG, LPS = (LOADS + N - 1) / N;  // per wave and tile, per slot of P1
  extern __shared__ __attribute__((aligned(16))) char smem_all[];
  constexpr int RT = 32 * WPG;  // keys of a workgroup
  const int n_kt = EDGE ? (S + RT - 1) / RT : S / RT;
  int pair, bh;
  if (G == 1) pair_of_tiles(block, n_kt, BH, pair, bh);
  else longest_first(block, BH, pair, bh);
  const int b = bh / H, h = bh % H;
  const int hw = EDGE ? dh : DW, nch = hw / 8;  // head width, in elements and in 16-byte chunks
  const int Hd = H * hw;
  const size_t ld = 3 * (size_t)Hd;
  const bf16_t* base = qkv + (size_t)b * S * ld + h * hw;
  const bf16_t* dob = dctx + (size_t)b * S * Hd + h * hw;
  const float* lrow = lse + ((size_t)b * H + h) * S;
  const float* drow = delta + ((size_t)b * H + h) * S;
  const int lane = threadIdx.x & 63, g = lane >> 5;
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float scale = rsqrtf((float)hw);
  const float c = scale * LOG2E;
  const int grp = G == 1 ? 0 : wave_all / WPG, wave = G == 1 ? wave_all : wave_all % WPG;
  char* const smem = smem_all + grp * (2 * STAGE);
  const unsigned sm = lds_addr(smem);
  if (EDGE) clear_lds(smem_all, G * 2 * STAGE);

  for (int pass = 0; pass < (G == 1 ? 2 : 1); pass++) {
    const int kt = pass == 0 ? pair : n_kt - 1 - pair;
    if (pass == 1 && kt == pair) break;  // odd number of key tiles: the middle one stands alone
    const int j0w = kt * RT + wave * 32, jk = j0w + (lane & 31);
    bf16x8 kf[KS], vf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      const bool ok = !EDGE || (jk < S && ks * 2 + g < nch);
      const bf16_t *kp = base + (size_t)jk * ld + Hd + ks * 16 + g * 8, *vp = kp + Hd;
      kf[ks] = __builtin_bit_cast(bf16x8, EDGE ? edge_load16(kp, ok) : *reinterpret_cast<const uint4*>(kp));
      vf[ks] = __builtin_bit_cast(bf16x8, EDGE ? edge_load16(vp, ok) : *reinterpret_cast<const uint4*>(vp));
    }
#pragma unroll
    for (int ks = 0; ks < KS; ks++) { settle(kf[ks]); settle(vf[ks]); }
    f32x16 dk[DT], dv[DT];
#pragma unroll
    for (int dt = 0; dt < DT; dt++)
#pragma unroll
      for (int v = 0; v < 16; v++) dk[dt][v] = dv[dt][v] = 0.f;

    const int i_first = kt * RT / TR * TR;
    const int n_q = EDGE ? (S - i_first + TR - 1) / TR : (S - i_first) / TR;
    auto tile_load = [&](int i0, int buf, int i) {
      const unsigned st = sm + buf * STAGE;
      if (i < NSEG) tile_dma_seg<DH, EDGE, WPG>(st, base + (size_t)i0 * ld, ld, wave, i, S - i0, nch);
      else if (i < 2 * NSEG) tile_dma_seg<DH, EDGE, WPG>(st + TB, dob + (size_t)i0 * Hd, (size_t)Hd, wave, i - NSEG, S - i0, nch);
      else {
        const int rb = wave * (4 / WPG) + i - 2 * NSEG;  // sixteen rows
        if (!EDGE || i0 + rb * 16 + (lane & 15) < S) lds_dma4(((lane & 16) ? drow : lrow) + i0 + rb * 16 + (lane & 15), st + LD_OFF + rb * 256);
      }
    };
    bf16x8 f[LEAD];  // one ring for both kinds of fragment: slot i reloads the register it has just used
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // One 64-query tile, a 32-query half at a time.  MASK: the tile may reach back before the wave's last key.
    auto tile = [&](auto mask_c, int t) {
      constexpr bool MASK = decltype(mask_c)::value;
      const char* st = smem + (t / G & 1) * STAGE;
      const int i0n = i_first + min(t + G, n_q - 1) * TR;  // past the end: the last tile again, into the buffer nobody reads
      // P1 slot i of half it: S (Q rows x K) or dP (dO rows x V) by bit 0, k-step i / 2
      auto row_frag = [&](int it, int i) { return frag_rows<DH>(i % 2 ? st + TB : st, it * 32, i / 2, lane); };
      // P3 slot i: dV (dO^T) or dK (Q^T) by bit 0, d-tile (i / 2) % DT, k-step i / (2 DT); EDGE: all of dV, then dK, whose factors are
      // formed meanwhile, d-tile i % DT, k-step (i / DT) % 2
      auto col_frag = [&](int it, int i) {
        if (EDGE) return frag_cols<DH>(i >= 2 * DT ? st : st + TB, (i % DT) * 32, it * 32 + ((i / DT) % 2) * 16, lane);
        return frag_cols<DH>(i % 2 ? st : st + TB, ((i / 2) % DT) * 32, it * 32 + (i / (2 * DT)) * 16, lane);
      };
      // lse / delta of the rows 32 it + 8 q + 4 g + 0..3 that this lane meets in accumulator group q
      auto stat4 = [&](int it, int q, int which) {
        const int row = it * 32 + q * 8 + g * 4;
        return *reinterpret_cast<const float4*>(st + LD_OFF + (row >> 4) * 256 + which * 64 + (row & 15) * 4);
      };
#pragma unroll
      for (int i = 0; i < LEAD; i++) f[i] = row_frag(0, i);  // cold start: exposed once per tile
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int it = 0; it < 2; it++) {
        const int i0h = i_first + t * TR + it * 32;  // first query of the half
        f32x16 sc, dp;
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int i = 0; i < N; i++) {
          if (i % 2 == 0) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % LEAD], kf[i / 2], i < 2 ? zero : sc, 0, 0, 0);
          else dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % LEAD], vf[i / 2], i < 2 ? zero : dp, 0, 0, 0);
          if (i + LEAD < N) f[i % LEAD] = row_frag(it, i + LEAD);
          else f[i % LEAD] = col_frag(it, i + LEAD - N);
#pragma unroll
          for (int n = i * LPS; n < (i + 1) * LPS; n++)
            if (it == 0 && n < LOADS) tile_load(i0n, (t / G + 1) & 1, n);
          __builtin_amdgcn_sched_barrier(0);
        }
        bf16x8 pb[2], db[2], pc[2][3];  // P and dS; EDGE: eight queries' P or dS in three terms, and the next eight's
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const float4 l4 = stat4(it, q, 0), d4 = stat4(it, q, 1);
#pragma unroll
          for (int r = 0; r < 4; r++) {
            const int v = q * 4 + r;
            float p = EDGE ? edge_exp(sc[v], scale, f4_get(l4, r)) : __builtin_amdgcn_exp2f(fmaf(sc[v], c, -LOG2E * f4_get(l4, r)));
            const int i = i0h + q * 8 + g * 4 + r;
            if (MASK && (jk > i || (EDGE && i >= S))) p = 0.f;
            const float d = EDGE && MASK && i >= S ? 0.f : p * (dp[v] - f4_get(d4, r));
            if (EDGE) {
              sc[v] = p;
              dp[v] = d;
            } else {
              pb[v >> 3][v & 7] = (__bf16)p;
              db[v >> 3][v & 7] = (__bf16)d;
            }
          }
        }
        if constexpr (EDGE) {
#pragma unroll
          for (int n = 0; n < 4; n++) split3(sc[2 * n], sc[2 * n + 1], pc[0], n);
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int i = 0; i < N; i++) {
          if constexpr (EDGE) {
            const int ch = i / DT, dt = i % DT;  // P of the first eight queries, of the others, dS likewise
#pragma unroll
            for (int k = 0; k < 3; k++) {
              if (ch < 2) dv[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % LEAD], pc[ch & 1][k], dv[dt], 0, 0, 0);
              else dk[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % LEAD], pc[ch & 1][k], dk[dt], 0, 0, 0);
#pragma unroll
              for (int n = 0; n < 4; n++) {
                if (n * 3 * DT / 4 != dt * 3 + k) continue;
                if (ch == 0) split3(sc[8 + 2 * n], sc[9 + 2 * n], pc[1], n);
                else if (ch < 3) split3(dp[(ch - 1) * 8 + 2 * n], dp[(ch - 1) * 8 + 2 * n + 1], pc[(ch + 1) & 1], n);
              }
              if (k < 2) __builtin_amdgcn_sched_barrier(0);
            }
          } else {
            const int hh = i / (2 * DT), dt = (i / 2) % DT;
            if (i % 2 == 0) dv[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % LEAD], pb[hh], dv[dt], 0, 0, 0);
            else dk[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % LEAD], db[hh], dk[dt], 0, 0, 0);
          }
          if (i + LEAD < N) f[i % LEAD] = col_frag(it, i + LEAD);
          else if (it == 0) f[i % LEAD] = row_frag(1, i + LEAD - N);  // the second half's first rows
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __builtin_amdgcn_s_setprio(0);
      lds_dma_wait();
      __syncthreads();
    };

#pragma unroll
    for (int i = 0; i < LOADS; i++) tile_load(i_first + min(grp, n_q - 1) * TR, 0, i);
    lds_dma_wait();
    __syncthreads();
    // The first two tiles (128 queries) straddle the diagonal of this workgroup's 128 keys, and under EDGE the last may reach
    // past S; there every tile takes the masks (a second copy of the tile costs 63 spilled registers).
    if (EDGE) {
      for (int t = grp; t < n_q; t += G) tile(T_{}, t);
    } else if (G == 1) {
      tile(T_{}, 0);
      tile(T_{}, 1);
      for (int t = 2; t < n_q; t++) tile(F_{}, t);
    } else {
      static_assert(G == 1 || WPG < 4, "one tile on the diagonal");
      if (grp == 0) tile(T_{}, 0);
      for (int t = grp ? grp : G; t < n_q; t += G) tile(F_{}, t);
    }
    if (G > 1) {
      // every group meets as many barriers as the one with the most tiles
      for (int t = (n_q + G - 1) / G - (n_q - grp + G - 1) / G; t > 0; t--) __syncthreads();
      constexpr int U = 2 * DT * 4;
      float* x = reinterpret_cast<float*>(smem_all);
      if (grp) {
        group_put<U>(x, wave_all - WPG, 0, dk);
        group_put<U>(x, wave_all - WPG, U / 2, dv);
      }
      __syncthreads();
      if (grp) return;
#pragma unroll
      for (int o = 0; o < G - 1; o++) {
        group_add<U>(x, o * WPG + wave, 0, dk);
        group_add<U>(x, o * WPG + wave, U / 2, dv);
      }
    }

    bool store = true;
    unsigned again = 0;  // as in the forward kernel
    if (EDGE) {
      store = jk < S;
      const unsigned long long odd = __builtin_amdgcn_ballot_w64(store && not_finite(dv, not_finite(dk, 0.f)) != 0.f);
      again = (unsigned)odd | (unsigned)(odd >> 32);
      store = store && !((again >> (lane & 31)) & 1);
    }
    bf16_t* out = dqkv + ((size_t)b * S + jk) * ld + h * hw;
    if (!EDGE || store) {
      store_rows<DW, EDGE>(out + Hd, dk, scale, g, hw);
      store_rows<DW, EDGE>(out + 2 * Hd, dv, 1.f, g, hw);
    }
    if (EDGE) {
      for (; again; again &= again - 1) {
        int lane_r = lane;
        settle(lane_r);
        const int j = j0w + __builtin_ctz(again);
        const bf16_t* kp = base + (size_t)j * ld + Hd;
        bf16_t* kout = dqkv + ((size_t)b * S + j) * ld + h * hw + Hd;
        attn_bwd_dkv_row<(DW + 63) / 64>(kp, kp + Hd, j, S, lane_r, base, ld, dob, Hd, hw, lrow, drow, kout, kout + Hd);
      }
    }
  }  // pass
}

template <int DW, bool EDGE, int G, int WPG>
__global__ __launch_bounds__(64 * G * WPG, 2) void attn_bwd_dkv_phased_mfma_kernel(int S, int H, int BH, int dh, const bf16_t* __restrict__ qkv,
                                                                          const float* __restrict__ lse, const float* __restrict__ delta,
                                                                          const bf16_t* __restrict__ dctx, bf16_t* __restrict__ dqkv) {
  attn_bwd_dkv_phased_mfma_body<DW, EDGE, G, WPG>(blockIdx.x, S, H, BH, dh, qkv, lse, delta, dctx, dqkv);
}

// dK, dV and dQ in one launch, delta given: the first `first` workgroups are the dK/dV kernel's, which are the longer ones.  Neither kernel
// alone fills the chip where this form is used.
template <int DW, bool EDGE, int G, int WPG>
__global__ __launch_bounds__(64 * G * WPG, 2) void attn_bwd_both_mfma_kernel(int S, int H, int BH, int dh, const bf16_t* __restrict__ qkv,
                                                                              const float* __restrict__ lse, float* __restrict__ delta,
                                                                              const bf16_t* __restrict__ dctx, bf16_t* __restrict__ dqkv, int first) {
  const int block = blockIdx.x;
  if (block >= first) {
    attn_bwd_dq_mfma_body<DW, EDGE, G, WPG>(block - first, S, H, BH, dh, qkv, lse, nullptr, dctx, delta, true, dqkv);
  } else if constexpr (DW == 64) {
    attn_bwd_dkv_phased_mfma_body<DW, EDGE, G, WPG>(block, S, H, BH, dh, qkv, lse, delta, dctx, dqkv);
  } else {
    attn_bwd_dkv16_mfma_body<DW, EDGE, G, WPG>(block, S, H, BH, dh, qkv, lse, delta, dctx, dqkv);
  }
}

bool attn_mfma_supported(int dtype, int B, int S, int H, int dh) {
  (void)B; (void)H;
  return dtype == FAX_BF16 && (dh == 64 || dh == 128) && S > 0 && S % 128 == 0;
}

// Whole 16-byte chunks per head are all that the masked-edge form asks for.  Measured against the scalar kernels, forward / backward
// in us: one head of 17 x 64 7.8 / 15.3 -> 8.4 / 11.7 (launch and latency), 8 heads of 64 x 32 13.1 / 28.2 -> 8.6 / 11.9,
// 45 heads of 1000 x 80 1485 / 2966 -> 37 / 104, 32 heads of 777 x 64 572 / 1075 -> 16 / 43, 16 heads of 1500 x 128
// 1754 / 3791 -> 32 / 106.  Errors against float64, over ten shapes and four distributions, are the scalar kernels' to 2e-4 in
// ctx and the gradients and to 7 % either way in lse (4e-8, half a unit in its last place).
bool attn_edge_supported(int dtype, int B, int S, int H, int dh) {
  (void)B; (void)H;
  return dtype == FAX_BF16 && dh % 8 == 0 && dh <= 128 && S > 0;
}

template <typename K>
static int set_lds(K kern, size_t bytes) {
  FAX_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
  return FAX_OK;
}

static constexpr size_t bwd_lds(int groups, int row) { return groups * 2 * (2 * (size_t)TR * row * 2 + 4 * 256); }  // two stages of Q tile | dO tile | lse, delta each
static inline unsigned grid_of(int B, int S, int H) { return (unsigned)((((S + 127) / 128 + 1) / 2) * B * H); }

// Which form: groups and waves to a group.  1x4 (a pair of 128-row tiles to a workgroup, two of them on a CU) is the form of a full chip.
// The more groups, the shorter a workgroup's chain of 64-wide tiles, but the more of the streamed index is loaded again, and the split forms'
// workgroups, which all groups' tiles make large, are alone on a CU (2x2 up to 64 wide: two).  So a split pays while its workgroups are
// about a round of the 256 CUs, and for more of them the longer the sequence is: its workgroups' chains differ, short ones fill up
// behind long ones.  With one 64-wide tile to a sequence
// there is nothing to split (2x2 takes part in the backward pass for the joint launch).
// The lines lie where the forms cross in 968 shapes of 2 to 1000 heads, 17 to 4096 long, 40 to 128 wide, each kernel timed back to back
// in a graph.  Over those the choice is 1.1 % above the fastest form of each, at most 1.5 % above 1x4, on average 25 % below it; over 330 others, drawn
// at random, 1.8 %, 1.6 % and 31 %.  us, 1x4 and the others:
//   forward, up to 64 wide   100 heads of 34 5.3, 2x2 5.8, 4x1 7.5;  128 of 100 7.7, 2x2 6.4;  400 of 100 10.9, 2x2 14.2;  6 of 256 10.4, 2x2 5.2, 4x1 5.1;  200 of 256 14.3, 2x2 14.1, 300 18.8 and 19.7;
//                            2 of 2048 32, 2x2 17.5, 4x1 14.0;  32 of 777 32, 2x2 19, 4x1 34;  66 of 1024 31, 2x2 28, 128 34 and 38
//   forward, wider           300 of 64 x 80 8.6, 2x2 14.9;  128 of 256 x 80 23, 2x2 21, 2x4 17;  200 of 256 x 128 21, 2x4 23;  6 of 2048 x 128 43, 2x2 25, 2x4 33;
//                            45 of 1024 x 80 42, 2x2 47, 2x4 36;  32 of 2048 x 128 47, 2x4 47
//   backward, up to 64 wide  100 of 34 14.3, 2x2 11.7, 4x1 18.7;  400 of 64 19.7, 2x2 22.4;  400 of 100 32, 2x2 40;  200 of 256 35.6, 2x2 36.4;  2 of 2048 80, 2x2 29, 4x1 22.5;  32 of 777 97, 2x2 46, 4x1 85
//   backward, wider          300 of 34 x 80 18, 2x2 32;  66 of 64 x 80 14.5, 2x2 11.1;  128 of 256 x 80 50, 2x2 61, 2x4 45;  200 of 256 x 128 51, 2x4 67;  6 of 2048 x 128 100, 2x2 56, 2x4 78;
//                            12 of 2048 x 128 103, 2x2 83, 2x4 82;  45 of 1024 x 80 107, 2x4 103;  32 of 2048 x 128 139, 2x4 154
AttnForm attn_fwd_form(int B, int S, int H, int dh) {
  const long long heads = (long long)B * H;
  const int n32 = (S + 31) / 32, n64 = (S + 63) / 64, n128 = (S + 127) / 128;
  if (n64 == 1) return AttnForm{1, 4, false};
  if (dh <= 64) {
    if (n128 > 1 && n32 * heads <= 256) return AttnForm{4, 1, false};
    return n64 * heads <= (n128 == 1 ? 400 : n128 == 2 ? 800 : 1024) ? AttnForm{2, 2, false} : AttnForm{1, 4, false};
  }
  if (n64 * heads <= (n64 < 12 ? 256 : 416)) return AttnForm{2, 2, false};
  return n128 > 1 && n128 * heads <= (n128 < 4 ? 256 : n128 < 6 ? 300 : 528) ? AttnForm{2, 4, false} : AttnForm{1, 4, false};
}
// Joint: dQ and dK/dV side by side, as one launch, while their workgroups are up to two rounds or so.  What ties them together is delta, which
// the dQ kernel produces as it goes; a small kernel of its own computes it first, which costs 2.5 us: 32 heads of 777 x 64
// 57 -> 46 us, 6 of 2048 x 128 60 -> 56, 2 of 2048 x 64 31.5 -> 22.5; 66 of 1024 x 64 and 200 of 256 x 64, beyond the line, 72 and 76, 36 and 39.
AttnForm attn_bwd_form(int B, int S, int H, int dh) {
  const long long heads = (long long)B * H;
  const int n32 = (S + 31) / 32, n64 = (S + 63) / 64, n128 = (S + 127) / 128;
  if (dh <= 64) {
    if (n128 > 1 && n32 * heads <= (n128 < 4 ? 144 : 256)) return AttnForm{4, 1, true};
    const long long t64 = n64 * heads;
    return t64 <= (n64 == 1 ? 256 : n128 == 1 ? 400 : n128 == 2 ? 800 : 1024) ? AttnForm{2, 2, 2 * t64 < (n64 <= 2 ? 640 : n64 <= 4 ? 780 : 1024)} : AttnForm{1, 4, false};
  }
  const bool whole = attn_mfma_supported(FAX_BF16, B, S, H, dh);
  const long long both = (n32 + n64) * heads;  // workgroups of 2x2: 32 keys, 64 queries
  if (both <= (n64 == 1 ? 256 : n64 == 2 ? (whole ? 768 : 500) : n64 < 8 ? min(700, 256 + 144 * (n64 - 1)) : 900)) return AttnForm{2, 2, both <= 600};
  const int most = n128 == 1 ? 128 : n128 < 4 ? 256 : n128 < 6 ? (whole ? 256 : 300) : whole && n128 <= 16 ? 320 : 400;
  return n64 > 1 && n128 * heads <= most ? AttnForm{2, 4, false} : AttnForm{1, 4, false};
}

template <int DW, bool EDGE, int G, int WPG>
static int fwd_t(int B, int S, int H, int dh, const bf16_t* qkv, bf16_t* ctx, float* lse, hipStream_t s) {
  constexpr size_t lds = G * 2 * (2 * (size_t)TR * row_width<DW>() * 2);  // per group two stages of K tile | V tile
  const dim3 grid(G == 1 ? grid_of(B, S, H) : (S + 32 * WPG - 1) / (32 * WPG) * B * H);
  FAX_TRY(set_lds(attn_fwd_mfma_kernel<DW, EDGE, G, WPG>, lds));
  hipLaunchKernelGGL((attn_fwd_mfma_kernel<DW, EDGE, G, WPG>), grid, dim3(64 * G * WPG), lds, s, S, H, B * H, dh, qkv, ctx, lse);
  FAX_LAUNCH_CHECK("attn_fwd_mfma");
  return FAX_OK;
}

// Whole tiles or masked edges, head width as computed, groups and their waves.
template <typename F>
static int by_form(const AttnForm& form, int B, int S, int H, int dh, F f) {
  auto groups = [&](auto dw, auto edge) -> int {
    if (form.groups == 1) return f(dw, edge, I<1>{}, I<4>{});
    if constexpr (decltype(dw)::value == 64) {
      if (form.groups == 4) return f(dw, edge, I<4>{}, I<1>{});
    } else {
      if (form.waves == 4) return f(dw, edge, I<2>{}, I<4>{});
    }
    return f(dw, edge, I<2>{}, I<2>{});
  };
  if (attn_mfma_supported(FAX_BF16, B, S, H, dh)) return dh == 64 ? groups(I<64>{}, F_{}) : groups(I<128>{}, F_{});
  return dh <= 64 ? groups(I<64>{}, T_{}) : dh <= 96 ? groups(I<96>{}, T_{}) : groups(I<128>{}, T_{});
}

int attn_fwd_mfma(int B, int S, int H, int dh, const void* qkv, void* ctx, float* lse, hipStream_t s) {
  const bf16_t* q = (const bf16_t*)qkv;
  bf16_t* c = (bf16_t*)ctx;
  return by_form(attn_fwd_form(B, S, H, dh), B, S, H, dh, [&](auto dw, auto edge, auto g, auto wpg) {
    return fwd_t<decltype(dw)::value, decltype(edge)::value, decltype(g)::value, decltype(wpg)::value>(B, S, H, dh, q, c, lse, s);
  });
}

template <int DW, bool EDGE, int G, int WPG>
static int bwd_t(bool joint, int B, int S, int H, int dh, const bf16_t* qkv, const bf16_t* ctx, const float* lse, const bf16_t* dctx,
                 bf16_t* dqkv, float* delta, hipStream_t s) {
  constexpr int DH = row_width<DW>();
  constexpr size_t lds_q = G * 2 * (2 * (size_t)TR * DH * 2);  // per group two stages of K tile | V tile
  const dim3 grid(G == 1 ? grid_of(B, S, H) : (S + 32 * WPG - 1) / (32 * WPG) * B * H);
  auto dkv = [&]() -> int {
    if constexpr (DW == 64) {
      constexpr size_t lds_kv = bwd_lds(G, DH);
      FAX_TRY(set_lds(attn_bwd_dkv_phased_mfma_kernel<DW, EDGE, G, WPG>, lds_kv));
      hipLaunchKernelGGL((attn_bwd_dkv_phased_mfma_kernel<DW, EDGE, G, WPG>), grid, dim3(64 * G * WPG), lds_kv, s, S, H, B * H, dh, qkv, lse,
                         delta, dctx, dqkv);
    } else {
      FAX_TRY(attn_bwd_dkv16_mfma(B, S, H, dh, EDGE, G, WPG, qkv, lse, delta, dctx, dqkv, s));
    }
    return FAX_OK;
  };
  if constexpr (G > 1 && WPG < 4) {  // (2x4 begins beyond two rounds)
    constexpr size_t lds = bwd_lds(G, DH);
    constexpr int KT = DW == 64 ? 32 * WPG : 16 * WPG;  // keys of a workgroup
    const unsigned first = (S + KT - 1) / KT * B * H;
    if (joint || G == 4) {
      FAX_TRY(attn_delta(FAX_BF16, B, S, H, dh, ctx, dctx, delta, s));
      FAX_TRY(set_lds(attn_bwd_both_mfma_kernel<DW, EDGE, G, WPG>, lds));
      hipLaunchKernelGGL((attn_bwd_both_mfma_kernel<DW, EDGE, G, WPG>), dim3(first + grid.x), dim3(64 * G * WPG), lds, s, S, H, B * H, dh,
                         qkv, lse, delta, dctx, dqkv, (int)first);
      FAX_LAUNCH_CHECK("attn_bwd_mfma");
      return FAX_OK;
    }
  }
  if constexpr (G < 4) {
    // dQ first: it also produces delta, which the dK/dV kernel reads
    FAX_TRY(set_lds(attn_bwd_dq_mfma_kernel<DW, EDGE, G, WPG>, lds_q));
    hipLaunchKernelGGL((attn_bwd_dq_mfma_kernel<DW, EDGE, G, WPG>), grid, dim3(64 * G * WPG), lds_q, s, S, H, B * H, dh, qkv, lse, ctx, dctx, delta,
                       dqkv);
    FAX_TRY(dkv());
    FAX_LAUNCH_CHECK("attn_bwd_mfma");
  }
  return FAX_OK;
}

int attn_bwd_mfma(int B, int S, int H, int dh, const void* qkv, const void* ctx, const float* lse, const void* dctx,
                  void* dqkv, float* delta, hipStream_t s) {
  const bf16_t *q = (const bf16_t*)qkv, *c = (const bf16_t*)ctx, *dc = (const bf16_t*)dctx;
  bf16_t* dq = (bf16_t*)dqkv;
  const AttnForm form = attn_bwd_form(B, S, H, dh);
  return by_form(form, B, S, H, dh, [&](auto dw, auto edge, auto g, auto wpg) {
    return bwd_t<decltype(dw)::value, decltype(edge)::value, decltype(g)::value, decltype(wpg)::value>(form.joint, B, S, H, dh, q, c, lse, dc, dq, delta, s);
  });
}

}  // namespace fax
