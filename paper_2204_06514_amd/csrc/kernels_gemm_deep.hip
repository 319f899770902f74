// bf16 GEMM on the matrix cores for products that leave CUs without a tile: small tiles (128 x 64 or 64 x 64), eight
// wavefronts per tile and five slabs in LDS.
//
// gemm_mfma_kernel.h is built for a full chip, where one wave per SIMD with 128 x 128 of the output each moves the fewest bytes
// through the LDS.  With few tiles its slab time is not bandwidth but the wait from one phase to the next: fragment reads that a
// lone wave per SIMD has to sit out, and slabs requested little more than a slab ahead, too late for operands that have to
// come from memory.  Here a workgroup has two waves per SIMD: waves 0-3 share the tile 2 x 2 and take the first 32 of a slab's 64
// contraction indices, waves 4-7 share it likewise and take the other 32 (half the MFMAs each, the same LDS traffic in all).
// Fragments are read a whole slab ahead into a second register set, and slabs are requested four ahead into the buffer that
// the slab before the current one has left.  At the end the two halves swap 32-row halves of their accumulators through LDS, add
// (first half + second half, whoever adds) and store one half each.
// Any M, N, K that the masked-edge form takes, with the same clamps, and its operand layouts, fragment reads and epilogue.
#include "gemm_mfma_kernel.h"

namespace fax {

static constexpr int DEEP_STAGES = 5;
template <int ROWS>
struct DeepLds {
  static constexpr int BYTES = ROWS * GK * 2;
  static constexpr int NSEG = BYTES / 1024 / 8;  // 1 KB loads per wave per slab
};

// Bound, with one or two workgroups per CU, by the LDS (fragment reads and arriving slabs, about 0.3 us a slab at 128 x 64 where the
// MFMAs take 0.1) and the barrier; with many more by what the L2s deliver into the LDS, which is where larger tiles take over.
// Operands from memory, us, against the best of the other classes: 3108 x 512 x 2048 17 (26 at 128 x 128), 2048 x 640 x 5120 39 (58),
// 3108 x 512 x 32000 225 (336), weight gradients 512 x 512 x 3108 18 (36), 1024 x 1024 x 8192 44 (86, or 32 in four K ranges and a
// fold), 512 x 256 x 1024 6.2 (11).  From the caches: 3108 x 512 x 2048 13, 2048 x 640 x 5120 27, 512 x 512 x 3108 11, 512 x 256 x 1024 4.9.  The other way round 3000 x 1200 x 4800: 61 at 128 x 64, 81 at 64 x 64, 59 at 128 x 128.
// 128 x 128 tiles in this form, with tests and cases still in the loop over slabs, were slower than in the other at every size tried (16-24 waves' worth of LDS reads per slab
// either way, and one workgroup per CU instead of two).
template <int BM, int BN, bool A_KC, bool B_KC, int EM>
__device__ __forceinline__ void deep_tile(int block, int M, int N, int K, const bf16_t* __restrict__ A, int lda,
                                          const bf16_t* __restrict__ B, int ldb, const EpiArgs& e, int tiles_m, int tiles_n) {
  using LA = DeepLds<BM>;
  using LB = DeepLds<BN>;
  constexpr int TM = BM / 64, TN = BN / 64, NSA = LA::NSEG, NSB = LB::NSEG, NS = NSA + NSB;
  constexpr int STAGE = LA::BYTES + LB::BYTES;
  extern __shared__ __attribute__((aligned(16))) char smem[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = wave >> 2;  // of every slab's contraction indices
  const int wm = ((wave >> 1) & 1) * (BM / 2), wn = (wave & 1) * (BN / 2);

  // work item = (K range, tile), as in gemm_mfma_kernel; undivided products skip the divisions, a tenth of a microsecond of a launch's three
  const int nt = tiles_m * tiles_n, nk_total = (int)((unsigned)(K + GK - 1) / GK);
  int tile = block, range = 0, k_first = 0, nk = nk_total;
  if (e.splits > 1) {
    tile = block % nt;
    range = block / nt;
    k_first = (int)((unsigned)range * (unsigned)nk_total / (unsigned)e.splits);
    nk = (int)((unsigned)(range + 1) * (unsigned)nk_total / (unsigned)e.splits) - k_first;
  }
  int tm_i, tn_i;
  tile_walk(tile, tiles_m, tiles_n, e.group, tm_i, tn_i);
  const int m0 = tm_i * BM, n0 = tn_i * BN;
  const int k_end = K - k_first * GK;  // contraction indices from this item's first to the end of the operands
  EpiArgs et = e;
  if (em_kind(EM) == EK_F32) {
    et.C = (float*)e.C + (size_t)range * e.split_stride;
    if (EM & EM_COLSUM) et.colsum = e.colsum + (size_t)range * e.colsum_stride;
  }

  unsigned a_off[NSA], b_off[NSB];
#pragma unroll
  for (int q = 0; q < NSA; q++) a_off[q] = slab_lane_offset<BM, A_KC, true>(lda, (wave * NSA + q) * 1024 + lane * 16, e.a_lim - m0);
#pragma unroll
  for (int q = 0; q < NSB; q++) b_off[q] = slab_lane_offset<BN, B_KC, true>(ldb, (wave * NSB + q) * 1024 + lane * 16, e.b_lim - n0);
  const size_t a_kstride = A_KC ? 1 : (size_t)lda, b_kstride = B_KC ? 1 : (size_t)ldb;
  const bf16_t* const a_tile = A + (A_KC ? (size_t)m0 * lda : (size_t)m0) + (size_t)k_first * GK * a_kstride;
  const bf16_t* const b_tile = B + (B_KC ? (size_t)n0 * ldb : (size_t)n0) + (size_t)k_first * GK * b_kstride;
  const unsigned smem_addr = lds_addr(smem);
  // This wave's NS loads of a slab: `a`, `b` its first elements, `place` the offset of its stage.
  auto request_at = [&](const bf16_t* a, const bf16_t* b, unsigned place) __attribute__((always_inline)) {
    const unsigned da = smem_addr + place + wave * NSA * 1024, db = smem_addr + place + LA::BYTES + wave * NSB * 1024;
#pragma unroll
    for (int q = 0; q < NSA; q++) lds_dma16(a, a_off[q], da + q * 1024);
#pragma unroll
    for (int q = 0; q < NSB; q++) lds_dma16(b, b_off[q], db + q * 1024);
  };
  // The same of slab kt, which may be the one in which K ends: zeros for what lies beyond.
  auto request = [&](int kt, unsigned place) __attribute__((always_inline)) {
    const int k_left = k_end - kt * GK;
    const bf16_t* const a0 = a_tile + (size_t)kt * GK * a_kstride;
    const bf16_t* const b0 = b_tile + (size_t)kt * GK * b_kstride;
    if (k_left >= GK) {
      request_at(a0, b0, place);
    } else {
      const char *a = reinterpret_cast<const char*>(a0), *b = reinterpret_cast<const char*>(b0);
      const unsigned da = smem_addr + place + wave * NSA * 1024, db = smem_addr + place + LA::BYTES + wave * NSB * 1024;
#pragma unroll
      for (int q = 0; q < NSA; q++)
        lds_dma16(slab_lane_k<BM, A_KC>((wave * NSA + q) * 1024 + lane * 16) < k_left ? (const void*)(a + a_off[q]) : (const void*)&gemm_zero16,
                  da + q * 1024);
#pragma unroll
      for (int q = 0; q < NSB; q++)
        lds_dma16(slab_lane_k<BN, B_KC>((wave * NSB + q) * 1024 + lane * 16) < k_left ? (const void*)(b + b_off[q]) : (const void*)&gemm_zero16,
                  db + q * 1024);
    }
  };
  // of this wave's loads only those of the NEWER youngest slabs may still be in flight; everybody's older ones are visible
  auto landed = [&](auto newer_c) __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" : : "n"(decltype(newer_c)::value * NS) : "memory");
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;
  constexpr bool CS = (EM & EM_COLSUM) != 0;
  static_assert(!CS || !B_KC, "column sums are taken from [K, N] fragments");
  const bool cs_on = CS && tm_i == 0 && wm == 0;  // the waves that see every B fragment of their columns once
  float cs[TN];
#pragma unroll
  for (int j = 0; j < TN; j++) cs[j] = 0.f;

  auto main_loop = [&](auto cs_c) {
    constexpr bool CSON = decltype(cs_c)::value;
    bf16x8 fa[2][2][TM], fb[2][2][TN];  // [register set][k-step of this wave's half][tile]
    auto read_one = [&](auto set_c, auto n_c, const char* st) {
      constexpr int SET = decltype(set_c)::value, n = decltype(n_c)::value, ks = n / (TM + TN), t = n % (TM + TN);
      if constexpr (t < TM) fa[SET][ks][t] = frag_load<BM, A_KC>(st, wm + t * 32, half * 2 + ks, lane);
      else fb[SET][ks][t - TM] = frag_load<BN, B_KC>(st + LA::BYTES, wn + (t - TM) * 32, half * 2 + ks, lane);
    };
    constexpr int READS = 2 * (TM + TN), MFMAS = 2 * TM * TN;
    // products of the slab in register set P; meanwhile the fragments of the next one, from stage st, into the other set
    auto step = [&](auto set_c, auto read_c, const char* st) {
      constexpr int P = decltype(set_c)::value;
      constexpr bool READ = decltype(read_c)::value;
      auto slot = [&](auto t_c) {
        constexpr int t = decltype(t_c)::value, ks = t / (TM * TN), i = t % (TM * TN) / TN, j = t % TN;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[P][ks][j], fa[P][ks][i], acc[i][j], 0, 0, 0);  // C^T tile
        if constexpr (READ) {
          constexpr int r0 = t * READS / MFMAS, r1 = (t + 1) * READS / MFMAS;
          if constexpr (r0 < r1) read_one(I<P ^ 1>{}, I<r0>{}, st);
          if constexpr (r0 + 1 < r1) read_one(I<P ^ 1>{}, I<r0 + 1>{}, st);
        }
        if constexpr (CSON && i == 0) {
#pragma unroll
          for (int k = 0; k < 8; k++) cs[j] += (float)fb[P][ks][j][k];
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      slot(I<0>{}); slot(I<1>{});
      if constexpr (MFMAS == 4) { slot(I<2>{}); slot(I<3>{}); }
    };
    static_assert(MFMAS == 2 || MFMAS == 4, "slots of a step");
    auto first = [&](auto set_c) __attribute__((always_inline)) {
      read_one(set_c, I<0>{}, smem); read_one(set_c, I<1>{}, smem); read_one(set_c, I<2>{}, smem); read_one(set_c, I<3>{}, smem);
      if constexpr (READS == 6) { read_one(set_c, I<4>{}, smem); read_one(set_c, I<5>{}, smem); }
    };
    // Slab kt + 1 has landed for everyone, and the fragments of slab kt - 1 have been used by everyone (their waits lie
    // before this barrier), so its buffer is free for slab kt + 4.
    unsigned rd = 0, wr = 4 * STAGE;  // where slabs kt + 1 (after the step below) and kt + 4 are
    const bf16_t *a_next = a_tile + (size_t)4 * GK * a_kstride, *b_next = b_tile + (size_t)4 * GK * b_kstride;
    auto next = [](unsigned& place) { place = place == (DEEP_STAGES - 1) * STAGE ? 0u : place + STAGE; };
    auto turn = [&](auto set_c, auto newer_c, auto request_c) __attribute__((always_inline)) {
      landed(newer_c);
      if constexpr (decltype(request_c)::value) {
        request_at(a_next, b_next, wr);
        a_next += GK * a_kstride;
        b_next += GK * b_kstride;
        next(wr);
      }
      next(rd);
      step(set_c, T_{}, smem + rd);
    };
    // The end of the loop is written out: the turn that requests the last slab, three that request none and the last products, from
    // register sets 0, 1, 0, 1, 0; so sets are known without a test, and the turns before have neither a test nor a case.  With both in every turn, and
    // the stage number modulo five, some sixty instructions and six branches that waited for each other, a slab of a 64 x 64 tile took 0.235 us where
    // it takes 0.13: 512 x 256 x 1024 6.4 -> 4.85 us, 512 x 1024 x 256 3.8 -> 3.5; a block of 512 tokens x 256, forward and backward, 80.9 -> 76.6.
#pragma unroll
    for (int s = 0; s < 4; s++)
      if (s < nk) request(s, s * STAGE);
    if (nk >= 4) landed(I<3>{});
    else if (nk == 3) landed(I<2>{});
    else if (nk == 2) landed(I<1>{});
    else landed(I<0>{});
    if (nk & 1) first(I<0>{});
    else first(I<1>{});
    if (nk > 4) {
      int left = nk - 5;
      if (left & 1) {
        turn(I<1>{}, I<2>{}, T_{});
        left--;
      }
      for (; left > 0; left -= 2) {
        turn(I<0>{}, I<2>{}, T_{});
        turn(I<1>{}, I<2>{}, T_{});
      }
      landed(I<2>{});
      request(nk - 1, wr);
      next(rd);
      step(I<0>{}, T_{}, smem + rd);
    }
    if (nk > 3) turn(I<1>{}, I<2>{}, F_{});
    if (nk > 2) turn(I<0>{}, I<1>{}, F_{});
    if (nk > 1) turn(I<1>{}, I<0>{}, F_{});
    step(I<0>{}, F_{}, smem);
  };
  if constexpr (CS) {
    if (cs_on) main_loop(T_{});
    else main_loop(F_{});
  } else {
    main_loop(F_{});
  }
  __syncthreads();  // every wave is done with the slabs (none is in flight: the last wait was for all)

  // The halves' accumulators: each wave hands over the rows that the wave with the same place in the other half stores.
  constexpr int XF = (TM == 2 ? 1 : TM) * TN * 16 * 64;  // floats per wave
  float* const xch = reinterpret_cast<float*>(smem);
  float* const cs_x = xch + 8 * XF;
  auto hand = [&](int i) {
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) xch[wave * XF + (j * 16 + v) * 64 + lane] = acc[i][j][v];
  };
  if constexpr (TM == 2) {
    if (half) hand(0);
    else hand(1);
  } else {
    if (half) hand(0);
  }
  if constexpr (CS) {
#pragma unroll
    for (int j = 0; j < TN; j++) cs[j] += __shfl_xor(cs[j], 32, 64);
    if (cs_on && half && lane < 32) {
#pragma unroll
      for (int j = 0; j < TN; j++) cs_x[wn + j * 32 + lane] = cs[j];
    }
  }
  __syncthreads();
  if constexpr (CS) {
    if (cs_on && !half && lane < 32) {
#pragma unroll
      for (int j = 0; j < TN; j++) {
        const int n = n0 + wn + j * 32 + lane;
        const float v = cs[j] + cs_x[wn + j * 32 + lane];
        if (n < N) et.colsum[n] = e.accumulate ? et.colsum[n] + v : v;
      }
    }
  }
  f32x16 out[1][TN];
  auto take = [&](int i) {
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) out[0][j][v] = acc[i][j][v] + xch[(wave ^ 4) * XF + (j * 16 + v) * 64 + lane];
  };
  int mw = m0 + wm;
  if constexpr (TM == 2) {
    if (half) take(1);
    else take(0);
    mw += half * 32;
  } else {
    if (half) return;  // (no barrier below)
    take(0);
  }
  float* const wbuf = cs_x + BN + wave * 32 * TN * 32;
  if (m0 + BM > M || n0 + BN > N) tile_epilogue<EM, true, 1, TN>(e, et, out, wbuf, mw, n0 + wn, M, N, lane);
  else tile_epilogue<EM, false, 1, TN>(e, et, out, wbuf, mw, n0 + wn, M, N, lane);
}

template <int BM, int BN, bool A_KC, bool B_KC, int EM>
__global__ __launch_bounds__(512) void gemm_deep_kernel(int M, int N, int K, const bf16_t* __restrict__ A, int lda,
                                                        const bf16_t* __restrict__ B, int ldb, EpiArgs e, int tiles_m,
                                                        int tiles_n) {
  deep_tile<BM, BN, A_KC, B_KC, EM>(blockIdx.x, M, N, K, A, lda, B, ldb, e, tiles_m, tiles_n);
}

template <int BM, int BN>
constexpr size_t deep_lds() {
  return (size_t)DEEP_STAGES * (DeepLds<BM>::BYTES + DeepLds<BN>::BYTES);
}

template <int BM, int BN, bool A_KC, bool B_KC, int EM>
static int launch_deep(const GemmArgs& g, const EpiArgs& e, hipStream_t s) {
  constexpr size_t lds = deep_lds<BM, BN>();
  // exchange (8 waves x 32 x BN/2 floats), column sums, staging (the same again)
  static_assert(2 * 8 * 32 * (BN / 2) * 4 + BN * 4 <= lds, "the epilogue's areas fit the slabs'");
  auto kern = gemm_deep_kernel<BM, BN, A_KC, B_KC, EM>;
  static bool configured = false;  // benign race: the attribute is idempotent
  if (!configured) {
    FAX_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    configured = true;
  }
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  EpiArgs ek = e;
  if (ek.group == 0) ek.group = 4;  // the side-by-side walk belongs to the persistent kernel
  hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n * (e.splits > 1 ? e.splits : 1)), dim3(512), lds, s, g.M, g.N, g.K,
                     (const bf16_t*)g.A, g.lda, (const bf16_t*)g.B, g.ldb, ek, tiles_m, tiles_n);
  FAX_LAUNCH_CHECK("gemm_deep");
  return FAX_OK;
}

// The orientations of gemm_edge_supported().
template <int BM, int BN>
static int dispatch_deep(const GemmArgs& g, const EpiArgs& e, hipStream_t s) {
  const bool erf = g.gelu_form == FAX_GELU_ERF;
  if (g.epi == EPI_GELU)
    return erf ? launch_deep<BM, BN, true, false, EK_GELU_ERF>(g, e, s) : launch_deep<BM, BN, true, false, EK_GELU_TANH>(g, e, s);
  if (g.epi == EPI_DGELU) return launch_deep<BM, BN, true, true, EK_DGELU>(g, e, s);
  if (g.c_f32 && g.colsum)
    return g.accumulate ? launch_deep<BM, BN, false, false, EK_F32 | EM_RES | EM_COLSUM>(g, e, s)
                        : launch_deep<BM, BN, false, false, EK_F32 | EM_COLSUM>(g, e, s);
  if (g.c_f32)
    return g.accumulate ? launch_deep<BM, BN, false, false, EK_F32 | EM_RES>(g, e, s)
                        : launch_deep<BM, BN, false, false, EK_F32>(g, e, s);
  if (g.tb) return launch_deep<BM, BN, true, true, EK_STORE>(g, e, s);
  if (g.C2)
    return g.R ? launch_deep<BM, BN, true, false, EK_STORE | EM_RES | EM_C2>(g, e, s)
               : launch_deep<BM, BN, true, false, EK_STORE | EM_C2>(g, e, s);
  return g.R ? launch_deep<BM, BN, true, false, EK_STORE | EM_RES>(g, e, s) : launch_deep<BM, BN, true, false, EK_STORE>(g, e, s);
}

int gemm_mfma_deep(const GemmArgs& g, const EpiArgs& e, const GemmSplitPlan& plan, hipStream_t s) {
  if (plan.tile_m == 128) return dispatch_deep<128, 64>(g, e, s);
  return dispatch_deep<64, 64>(g, e, s);
}

// A weight-gradient product and the input-gradient product of the same layer in one launch: the first workgroups take the tiles
// of the first, the others those of the second, each exactly as it would in a launch of its own.
struct DeepProduct {
  int M, N, K;
  const bf16_t* A;
  int lda;
  const bf16_t* B;
  int ldb;
  EpiArgs e;
  int tiles_m, tiles_n;
};

// Bound like gemm_deep_kernel; what it saves is a launch's ramp and tail, and the CUs that either product alone leaves idle.
// 512 tokens x 256, F = 1024: 6 us a pair, where the two launches take 5 each and the gap between them; the block forward and
// backward 132.2 -> 114.8 us (75 with what came after).
template <int BM, int WEM, int DM, int DEM>
__global__ __launch_bounds__(512) void gemm_deep_pair_kernel(DeepProduct w, DeepProduct d, int first) {
  const int block = blockIdx.x;
  if (block < first)
    deep_tile<BM, 64, false, false, WEM>(block, w.M, w.N, w.K, w.A, w.lda, w.B, w.ldb, w.e, w.tiles_m, w.tiles_n);
  else
    deep_tile<DM, 64, true, true, DEM>(block - first, d.M, d.N, d.K, d.A, d.lda, d.B, d.ldb, d.e, d.tiles_m, d.tiles_n);
}

static DeepProduct deep_product(const GemmArgs& g, const EpiArgs& e, const GemmSplitPlan& plan) {
  DeepProduct p{g.M, g.N, g.K, (const bf16_t*)g.A, g.lda, (const bf16_t*)g.B, g.ldb, e,
                (g.M + plan.tile_m - 1) / plan.tile_m, (g.N + plan.tile_n - 1) / plan.tile_n};
  if (p.e.group == 0) p.e.group = 4;
  return p;
}

template <int BM, int WEM, int DM, int DEM>
static int launch_deep_pair(const DeepProduct& w, const DeepProduct& d, hipStream_t s) {
  constexpr size_t lds = deep_lds<(BM > DM ? BM : DM), 64>();
  auto kern = gemm_deep_pair_kernel<BM, WEM, DM, DEM>;
  static bool configured = false;  // benign race: the attribute is idempotent
  if (!configured) {
    FAX_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    configured = true;
  }
  const int first = w.tiles_m * w.tiles_n;
  hipLaunchKernelGGL(kern, dim3(first + d.tiles_m * d.tiles_n), dim3(512), lds, s, w, d, first);
  FAX_LAUNCH_CHECK("gemm_deep_pair");
  return FAX_OK;
}

template <int BM, int WEM>
static int dispatch_deep_pair(bool dgelu, int tile_m, const DeepProduct& w, const DeepProduct& d, hipStream_t s) {
  if (tile_m == 128)
    return dgelu ? launch_deep_pair<BM, WEM, 128, EK_DGELU>(w, d, s) : launch_deep_pair<BM, WEM, 128, EK_STORE>(w, d, s);
  return dgelu ? launch_deep_pair<BM, WEM, 64, EK_DGELU>(w, d, s) : launch_deep_pair<BM, WEM, 64, EK_STORE>(w, d, s);
}

int gemm_mfma_deep_pair(const GemmArgs& wg, const EpiArgs& we, const GemmSplitPlan& wp, const GemmArgs& dg, const EpiArgs& de,
                        const GemmSplitPlan& dp, hipStream_t s) {
  const DeepProduct w = deep_product(wg, we, wp), d = deep_product(dg, de, dp);
  const bool dgelu = dg.epi == EPI_DGELU;
  if (wp.tile_m == 128)
    return wg.accumulate ? dispatch_deep_pair<128, EK_F32 | EM_RES | EM_COLSUM>(dgelu, dp.tile_m, w, d, s)
                         : dispatch_deep_pair<128, EK_F32 | EM_COLSUM>(dgelu, dp.tile_m, w, d, s);
  return wg.accumulate ? dispatch_deep_pair<64, EK_F32 | EM_RES | EM_COLSUM>(dgelu, dp.tile_m, w, d, s)
                       : dispatch_deep_pair<64, EK_F32 | EM_COLSUM>(dgelu, dp.tile_m, w, d, s);
}

}  // namespace fax
