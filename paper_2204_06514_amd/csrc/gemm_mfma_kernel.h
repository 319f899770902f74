// bf16 GEMM on the CDNA4 matrix cores: v_mfma_f32_32x32x16_bf16, fp32 accumulate.
//
// One 256-thread workgroup (4 wavefronts, 2x2) computes a BM x BN tile of C, stepping over K in
// slabs of 64.  Slabs of A and B go from global memory straight into LDS
// (global_load_lds_dwordx4: no staging registers, no LDS store instructions), three buffers for
// A and two for B, each slab requested about a slab of MFMAs before it is needed and its load
// instructions spread over that time.
//
// An operand whose contraction index is contiguous in memory ("KC": A stored [M,K], B stored
// [N,K]) is kept in LDS as [row][64] with the 16-byte chunk index XOR-ed with ((row >> 1) & 7):
// measured on gfx950, the 128-bit fragment reads of 32 consecutive rows then run at the full LDS
// rate (XOR with row & 7 is 15 % slower, no swizzle 4x slower).
// An operand whose M/N index is contiguous ("MC": A stored [K,M], B stored [K,N]) is kept as
// [k][rows] and fetched with ds_read_b64_tr_b16, the LDS transpose read: 16 lanes pick up four
// k-rows x 16 columns and each lane receives 4 consecutive k for its own column; two such reads
// make one MFMA operand.  There the 32-byte column-group index is XOR-ed with mc_swizzle(k), which
// spreads the eight k-rows that two 16-lane blocks read in one pass over all banks (see there;
// SQ_LDS_BANK_CONFLICT reads 0 for every flavour of the kernel, where XOR with (k & 3) left 31 %
// of the LDS cycles in conflicts with one such operand and 49 % with two -- at the same kernel
// time: these kernels do not wait for the LDS).  A direct-to-LDS load writes 1024
// consecutive LDS bytes per wave instruction (lane i at +16 i), so both swizzles are applied on
// the global side: each lane fetches the chunk that belongs at its LDS position.
//
// MFMA 32x32x16 lane layout (lane l): first/second operand = row/column (l & 31) of the product,
// k = 8 (l >> 5) + 0..7; accumulator v = 0..15 holds element [8 (v >> 2) + 4 (l >> 5) + (v & 3)][l & 31].
// The kernel feeds the B fragment as first operand and the A fragment as second, i.e. it
// accumulates C^T tiles: a lane then owns row m = l & 31 of C and, in v = 4 g .. 4 g + 3, the four
// consecutive columns n = 8 g + 4 (l >> 5) + 0..3 -- a 16-byte unit for the epilogue.
#pragma once
#include <type_traits>

#include "fax_internal.h"

namespace fax {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) short short4v;
typedef __attribute__((ext_vector_type(8))) short short8v;
typedef __attribute__((ext_vector_type(16))) float f32x16;
template <int V> using I = std::integral_constant<int, V>;
using T_ = std::true_type;
using F_ = std::false_type;

static constexpr int GK = 64;  // K slab

template <int ROWS, bool KC>
struct TileLds {
  static constexpr int BYTES = ROWS * GK * 2;
  static constexpr int NSEG = BYTES / 1024 / 4;  // 1 KB segments (= load instructions) per wave per slab
};

// Byte offset, from the slab's first element, of the 16 bytes that belong at LDS byte offset `b`
// of the slab.  Inverse of the layouts that frag_load() reads.  Does not depend on the slab's
// position: each lane computes its offsets once and only the (wave-uniform) slab base moves.
// XOR applied to the 32-byte column-group index of k-row kr of an M/N-contiguous operand.  A
// transpose read has each 16-lane block fetch four k-rows x 32 bytes; blocks 0 and 1 take the same
// k-rows at neighbouring groups, blocks 2 and 3 the k-rows eight further down.  Whichever two
// blocks the LDS serves in one pass, (0, 1) or (0, 2), their eight 32-byte pieces must fall into
// eight different groups of the 256-byte bank window: bits 0-1 of kr go to bits 1-2 of the XOR
// (four rows, two apart), bit 3 of kr to bit 0.
// A 64-wide operand has four groups per k-row and two k-rows per bank window: bit 0 of kr picks the half of the window
// already, bit 1 goes to bit 1 of the XOR.  The same for a 192-wide one, whose k-rows are a window and a half long.
template <int ROWS>
__device__ __forceinline__ int mc_swizzle(int kr) {
  return ROWS % 128 ? (kr & 2) | ((kr >> 3) & 1) : ((kr & 3) << 1) | ((kr >> 3) & 1);
}

// EDGE: the operand ends `lim` rows (KC) or columns (MC, at least 8 of them) after the slab's first; a
// lane whose chunk lies beyond fetches the last one instead: finite or not, what it brings only
// reaches outputs that are not stored.
template <int ROWS, bool KC, bool EDGE>
__device__ __forceinline__ unsigned slab_lane_offset(int ld, int b, int lim) {
  if (KC) {
    const int row = b >> 7, pc = (b >> 4) & 7;
    const int chunk = pc ^ ((row >> 1) & 7);
    return (unsigned)((EDGE ? min(row, lim - 1) : row) * ld + (chunk << 3)) * 2u;
  }
  constexpr int RB = ROWS * 2;  // bytes per k-row
  const int kr = b / RB, pc = (b % RB) >> 4;
  const int lc = (((pc >> 1) ^ mc_swizzle<ROWS>(kr)) << 1) | (pc & 1);
  return (unsigned)(kr * ld + (EDGE ? min(lc << 3, lim - 8) : lc << 3)) * 2u;
}
// First contraction index, within the slab, of that chunk.
template <int ROWS, bool KC>
__device__ __forceinline__ int slab_lane_k(int b) {
  if (KC) return (((b >> 4) & 7) ^ ((b >> 8) & 7)) << 3;
  return b / (ROWS * 2);
}

// Where lanes of an EDGE kernel fetch from whose contraction index lies beyond the end.
static __device__ const uint4 gemm_zero16 = {0u, 0u, 0u, 0u};

// One MFMA operand (8 bf16 per lane) for the 32 rows starting at rb, k-step ks (16 wide).
template <int ROWS, bool KC>
__device__ __forceinline__ bf16x8 frag_load(const char* lds, int rb, int ks, int lane) {
  if (KC) {
    const int row = rb + (lane & 31);
    const int chunk = ks * 2 + (lane >> 5);
    const uint4 v = *reinterpret_cast<const uint4*>(lds + row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4));
    return __builtin_bit_cast(bf16x8, v);
  } else {
    const int blk = lane >> 4, i = lane & 15;
    const int kr = ks * 16 + (blk >> 1) * 8 + (i >> 2);  // kr + 4 has the same swizzle
    const int col = rb + (blk & 1) * 16 + (i & 3) * 4;
    const char* p = lds + kr * (ROWS * 2) + (((col >> 4) ^ mc_swizzle<ROWS>(kr)) << 5) + (col & 15) * 2;
    typedef __attribute__((address_space(3))) short4v lds_s4;
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(p));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(p + 4 * ROWS * 2));
    const short8v v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
  }
}

// Epilogue flavours, fixed at compile time: a kind, plus flags for the optional operands.  Nothing
// in the store loop may hang on a run-time condition: stores count towards the same counter as
// loads on this target, so the conservative wait the compiler places where branches that contain
// loads rejoin would also wait for every earlier store to be acknowledged, once per row.
// VALUE: GELU without the derivative.  LSE: no output at all but what a softmax over the columns needs (lse_epilogue).
enum { EK_STORE = 0, EK_GELU_TANH = 1, EK_GELU_ERF = 2, EK_DGELU = 3, EK_LSE = 4, EK_F32 = 5, EK_VALUE_TANH = 6, EK_VALUE_ERF = 7 };
enum {
  EM_RES = 8,  // bf16 kinds: add the residual R;  EK_F32: add to what C already holds
  EM_C2 = 16,  // EK_STORE: also write the plain product (before bias and residual) to C2
  EM_COLSUM = 32  // EK_F32, B stored [K, N]: also colsum[n] (+)= sum_k B[k, n]
};
constexpr int em_kind(int em) { return em & 7; }
constexpr bool em_dgelu(int em) { return em_kind(em) == EK_DGELU; }
constexpr bool em_value(int em) { return em_kind(em) == EK_VALUE_TANH || em_kind(em) == EK_VALUE_ERF; }
constexpr bool em_gelu(int em) { return em_kind(em) == EK_GELU_TANH || em_kind(em) == EK_GELU_ERF || em_value(em); }

// tanh-form GELU through the logistic function: (1 + tanh z) / 2 = 1 / (1 + exp(-2 z)), one
// v_exp_f32 and one v_rcp_f32 per element.  In fp32, over N(0, 1) and against tanhf, which the scalar kernel has: the value
// 4.6e-8 from float64 in the 2-norm (tanhf 3.8e-8), the derivative 7.1e-8 (4.7e-8; 2e-6 at most, near u = 4, where 1 - s
// cancels); in the lower tail, u from -6 to -3, 2.6e-7 (4e-5, 1 + tanh cancels).  After the rounding to bf16 that follows both
// are equally far from float64, 1.7e-3 and 1.9e-3, to eight digits.
// This runs in the GEMM's epilogue with the matrix cores idle, so the operation count matters:
// 18 issue slots per element (the two quarter-rate instructions count four each), with u^2
// shared between the argument and the derivative and every constant folded:
//   -2 z log2(e) = u (A + B u^2),  A = -2 sqrt(2/pi) log2(e),  B = 0.044715 A
//   gelu = u s,  gelu' = s + (gelu - gelu s) (C + D u^2),  C = 2 sqrt(2/pi),  D = 3 * 0.044715 C
__device__ __forceinline__ void gelu_tanh_both(float u, float& g, float& dg) {
  const float u2 = u * u;
  const float e = __builtin_amdgcn_exp2f(u * fmaf(-0.10294324f, u2, -2.3022082f));
  const float sg = __builtin_amdgcn_rcpf(1.f + e);
  g = u * sg;
  dg = fmaf(fmaf(-g, sg, g), fmaf(0.21406445f, u2, 1.5957691216057308f), sg);
}

// erf-form GELU.  With x = |u| / sqrt(2), erfc(x) / 2 = e^(-x^2) Q(t), t = 1 / (1 + 0.33 x), Q a polynomial of degree 8 without
// constant term fitted here to the smallest largest relative error over x < 9.5: 1.06e-7 with the coefficients rounded as
// they stand, at x = 0 where they add up to 0.499999947.  In fp32 the value is within 6e-7 of itself for |u| < 3 and
// 4.5e-6 down to u = -9 (the rounding of the exponent), the derivative within 3e-7 of 1.  e^(-x^2) = e^(-u^2 / 2) is the
// density's exponential as well, so value and derivative share one v_exp_f32 and one v_rcp_f32: 26 issue slots per element
// where the library's erf and exp are over a hundred with both of their branches.  The lower tail has no cancellation
// (1 + erf loses it below u = -3); elsewhere the error is that of fp32 sums near 1 either way (4e-8 of the values' norm).  The
// FFN-in product of 3000 tokens x 4800 x 1200: 154 -> 59 us.
__device__ __forceinline__ void gelu_erf_both(float u, float& g, float& dg) {
  const float t = __builtin_amdgcn_rcpf(fmaf(0.23334524f, fabsf(u), 1.f));
  const float e = __builtin_amdgcn_exp2f(u * u * -0.72134752f);
  float q = fmaf(-0.067964382f, t, 0.23134403f);
  q = fmaf(q, t, -0.17771934f);
  q = fmaf(q, t, 0.20627069f);
  q = fmaf(q, t, 0.022505369f);
  q = fmaf(q, t, 0.10096190f);
  q = fmaf(q, t, 0.091418624f);
  q = fmaf(q, t, 0.093183056f);
  const float c = q * t * e;
  const float cdf = u < 0.f ? c : 1.f - c;
  g = u * cdf;
  dg = fmaf(u * 0.39894228f, e, cdf);
}

// Four consecutive columns n..n+3 of row m at once: 8-byte bf16 loads and stores.
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
__device__ __forceinline__ float4 ld_bf16x4(const void* base, size_t idx) {
  const bf16x4 v = *reinterpret_cast<const bf16x4*>((const bf16_t*)base + idx);
  return make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
}
__device__ __forceinline__ void st_bf16x4(void* base, size_t idx, float4 a) {
  bf16x4 v;
  v[0] = (__bf16)a.x; v[1] = (__bf16)a.y; v[2] = (__bf16)a.z; v[3] = (__bf16)a.w;
  // Streaming store: the tile is not read again by this kernel, and a round of tiles is as large as the
  // L2s (32 x 128 KB per XCD against 4 MB), where it would push out the operand panels that the
  // XCD's workgroups share.  Measured against plain stores, A-B-A-B on one box: the 768-wide model
  // 64.8-66.2 -> 63.9-64.0 ms (forward 21.4-22.1 -> 20.55 ms), the 1024-wide one -0.6 %, d_model 4096
  // unchanged.
  __builtin_nontemporal_store(v, reinterpret_cast<bf16x4*>((bf16_t*)base + idx));
}
// `side` is the row's residual (R) or, for the GELU' flavour, the stored derivative (U), fetched by
// the caller ahead of time so that its latency overlaps the LDS turn-around.
// For the fp32 flavour (plain product, optionally added to what C holds) `side` is the old C.
template <int EM>
__device__ __forceinline__ void mfma_epilogue4(const EpiArgs& e, int m, int n, float4 a, float4 bias, float4 side) {
  constexpr int KIND = em_kind(EM);
  if (KIND == EK_F32) {
    if (EM & EM_RES) { a.x += side.x; a.y += side.y; a.z += side.z; a.w += side.w; }
    typedef __attribute__((ext_vector_type(4))) float f32x4s;
    const f32x4s av = {a.x, a.y, a.z, a.w};
    __builtin_nontemporal_store(av, reinterpret_cast<f32x4s*>((float*)e.C + (size_t)m * e.ldc + n));  // as st_bf16x4
    return;
  }
  if (EM & EM_C2) st_bf16x4(e.C2, (size_t)m * e.ldc2 + n, a);
  a.x += bias.x; a.y += bias.y; a.z += bias.z; a.w += bias.w;
  if (!em_dgelu(EM) && (EM & EM_RES)) {
    a.x += side.x; a.y += side.y; a.z += side.z; a.w += side.w;
  }
  if (em_gelu(EM)) {  // C = gelu'(acc), C2 = gelu(acc); VALUE: C2 alone (16384 x 3072 x 768, whose stores are half of a round: 104 -> 90 us)
    float4 g, dg;
    if (KIND == EK_GELU_TANH || KIND == EK_VALUE_TANH) {
      gelu_tanh_both(a.x, g.x, dg.x); gelu_tanh_both(a.y, g.y, dg.y);
      gelu_tanh_both(a.z, g.z, dg.z); gelu_tanh_both(a.w, g.w, dg.w);
    } else {
      gelu_erf_both(a.x, g.x, dg.x); gelu_erf_both(a.y, g.y, dg.y);
      gelu_erf_both(a.z, g.z, dg.z); gelu_erf_both(a.w, g.w, dg.w);
    }
    if (!em_value(EM)) st_bf16x4(e.C, (size_t)m * e.ldc + n, dg);
    st_bf16x4(e.C2, (size_t)m * e.ldc2 + n, g);
    return;
  }
  if (em_dgelu(EM)) { a.x *= side.x; a.y *= side.y; a.z *= side.z; a.w *= side.w; }
  st_bf16x4(e.C, (size_t)m * e.ldc + n, a);
}

// Tile number -> tile of the persistent kernel (comment at its use below).  Host and device: the
// host copy lets the tests check that every walk visits every tile exactly once.
__host__ __device__ inline void tile_walk(int id, int tiles_m, int tiles_n, int group, int& tm_i, int& tn_i) {
  if (group == 0) {
    // 256 workgroups, tile counts that are multiples of 16 both ways: round number id >> 8 is a
    // 16 x 16 block of tiles (walked down the tile rows first), XCD x takes the 4 x 8 block at
    // (x & 3, x >> 2) of it, its workgroup j the tile (j & 3, j >> 2) of that.  The eight XCDs then
    // work on 16 + 16 operand panels at any time instead of 32 + 8.
    const int x = id & 7, j = (id >> 3) & 31, sb = id >> 8;
    const int sbm = tiles_m >> 4;
    tm_i = ((sb % sbm) << 4) + ((x & 3) << 2) + (j & 3);
    tn_i = ((sb / sbm) << 4) + ((x >> 2) << 3) + (j >> 2);
    return;
  }
  const int nt = tiles_m * tiles_n;
  if (nt % 8 == 0) id = (id % 8) * (nt / 8) + id / 8;
  const int per_group = group * tiles_n;
  const int g = id / per_group;
  const int gm0 = g * group;
  const int gsz = group < tiles_m - gm0 ? group : tiles_m - gm0;
  tm_i = gm0 + (id % per_group) % gsz;
  tn_i = (id % per_group) / gsz;
}

// Epilogue of one wave's TM x TN accumulators, whose first element is C[mw][nw].  The wave turns 32 rows of its tile at a time
// through LDS (fp32, `wbuf`: 32 x 32 TN floats of its own) and reads them
// back row-wise, four consecutive columns per lane, so that a row of the wave tile leaves as
// one contiguous run and bias, residual and the GELU side inputs move as 8-byte vectors.  On
// the way in a lane writes the 16-byte units it owns (row l & 31); the 16-byte chunk index is
// XOR-ed with (row & 7) so that neither those writes (8 lanes = 8 rows, same chunk) nor the
// row-wise reads (8 lanes = 8 consecutive chunks) collide on LDS banks.  Reads are issued eight
// rows ahead of the arithmetic and stores that consume them.
// MASK: the tile reaches beyond the output; side inputs are fetched from clamped places (no branch
// around a load), stores are predicated.  `et`: the epilogue operands of this work item (e of the launch).
template <int EM, bool MASK, int TM, int TN>
__device__ __forceinline__ void tile_epilogue(const EpiArgs& e, const EpiArgs& et, const f32x16 (&acc)[TM][TN], float* wbuf,
                                              int mw, int nw, int M, int N, int lane_e) {
  constexpr int WC = TN * 32;     // columns of the wave tile
  constexpr int LPR = WC / 4;     // lanes per row on the way out
  constexpr int RPI = 64 / LPR;   // rows per store instruction
  constexpr int NIT = 32 / RPI;   // store instructions per 32 rows
  constexpr int BATCH = NIT < 8 ? NIT : 8;
  static_assert(NIT % BATCH == 0, "batching of the read-back");
  const int c4 = (lane_e % LPR) * 4;
  const int rsub = lane_e / LPR;
  const int ncol = nw + c4;
  const int ncol_r = MASK ? min(ncol, N - 4) : ncol;  // where the side inputs are read
  auto mrow_r = [&](int m) { return MASK ? min(m, M - 1) : m; };
  constexpr bool F32 = em_kind(EM) == EK_F32, DG = em_dgelu(EM);
  constexpr bool SIDE = !F32 && (DG || (EM & EM_RES));  // a bf16 side input: pre-activation U or residual R
  float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
  if (!F32 && e.bias) bias = ld_bf16x4(e.bias, ncol_r);
  const bf16_t* sp = (const bf16_t*)(DG ? e.U : e.R);
  const int lds_ = DG ? e.ldu : e.ldr;
  // the side input of 32 rows is requested one round ahead: the loads fly while the previous
  // rows turn through LDS
  bf16x4 side[2][SIDE ? NIT : 1];
  auto side_request = [&](int i, bf16x4 (&dst)[SIDE ? NIT : 1]) {
    if (SIDE) {
#pragma unroll
      for (int k = 0; k < NIT; k++)
        dst[k] = *reinterpret_cast<const bf16x4*>(sp + (size_t)mrow_r(mw + i * 32 + rsub + k * RPI) * lds_ + ncol_r);
    }
  };
  side_request(0, side[0]);
#pragma unroll
  for (int i = 0; i < TM; i++) {
    const int mrow = mw + i * 32 + rsub;
    if (i + 1 < TM) side_request(i + 1, side[(i + 1) & 1]);
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int g = 0; g < 4; g++) {
        const int row = lane_e & 31;
        const int chunk = j * 8 + g * 2 + (lane_e >> 5);
        const f32x16& t = acc[i][j];
        *reinterpret_cast<float4*>(wbuf + row * WC + ((chunk ^ (row & 7)) << 2)) =
            make_float4(t[g * 4], t[g * 4 + 1], t[g * 4 + 2], t[g * 4 + 3]);
      }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int k0 = 0; k0 < NIT; k0 += BATCH) {
      constexpr bool ADD_C = F32 && (EM & EM_RES);
      float4 a[BATCH], old_c[ADD_C ? BATCH : 1];
#pragma unroll
      for (int u = 0; u < BATCH; u++) {
        const int row = (k0 + u) * RPI + rsub;
        a[u] = *reinterpret_cast<const float4*>(wbuf + row * WC + (((c4 >> 2) ^ (row & 7)) << 2));
        if (ADD_C) old_c[u] = *reinterpret_cast<const float4*>((const float*)et.C + (size_t)mrow_r(mrow + (k0 + u) * RPI) * e.ldc + ncol_r);
      }
#pragma unroll
      for (int u = 0; u < BATCH; u++) {
        float4 sd = make_float4(0.f, 0.f, 0.f, 0.f);
        if (ADD_C) {
          sd = old_c[u];
        } else if (SIDE) {
          const bf16x4 v = side[i & 1][k0 + u];
          sd = make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
        }
        const int m = mrow + (k0 + u) * RPI;
        if (!MASK || (m < M && ncol < N)) mfma_epilogue4<EM>(et, m, ncol, a[u], bias, sd);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// The same for a wave tile 96 columns wide, whole and with a bf16 output: 24 lanes to a row, so that a store instruction takes two
// rows and two thirds and a lane's place repeats after three of them, eight rows on.  (A function of its own: with both walks
// in one the compiler needed a hundred more address instructions for the other widths, 1.4 % of a step of 1024-wide layers.)
template <int EM, int TM>
__device__ __forceinline__ void tile_epilogue96(const EpiArgs& e, const f32x16 (&acc)[TM][3], float* wbuf, int mw, int nw, int lane_e) {
  constexpr int WC = 96, LPR = WC / 4, PER = 3, NIT = 12, BATCH = 6;
  constexpr bool DG = em_dgelu(EM), SIDE = DG || (EM & EM_RES);
  int c[PER], rsub[PER], ncol[PER];
  float4 bias[PER];
#pragma unroll
  for (int j = 0; j < PER; j++) {
    c[j] = (j * 64 + lane_e) % LPR;
    rsub[j] = (j * 64 + lane_e) / LPR;
    ncol[j] = nw + c[j] * 4;
    bias[j] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (e.bias) {
#pragma unroll
    for (int j = 0; j < PER; j++) bias[j] = ld_bf16x4(e.bias, ncol[j]);
  }
  const bf16_t* sp = (const bf16_t*)(DG ? e.U : e.R);
  const int lds_ = DG ? e.ldu : e.ldr;
  bf16x4 side[2][SIDE ? NIT : 1];
  auto side_request = [&](int i, bf16x4 (&dst)[SIDE ? NIT : 1]) {
    if (SIDE) {
#pragma unroll
      for (int k = 0; k < NIT; k++)
        dst[k] = *reinterpret_cast<const bf16x4*>(sp + (size_t)(mw + i * 32 + rsub[k % PER] + k / PER * 8) * lds_ + ncol[k % PER]);
    }
  };
  side_request(0, side[0]);
#pragma unroll
  for (int i = 0; i < TM; i++) {
    if (i + 1 < TM) side_request(i + 1, side[(i + 1) & 1]);
#pragma unroll
    for (int j = 0; j < 3; j++)
#pragma unroll
      for (int g = 0; g < 4; g++) {
        const int row = lane_e & 31;
        const int chunk = j * 8 + g * 2 + (lane_e >> 5);
        const f32x16& t = acc[i][j];
        *reinterpret_cast<float4*>(wbuf + row * WC + ((chunk ^ (row & 7)) << 2)) =
            make_float4(t[g * 4], t[g * 4 + 1], t[g * 4 + 2], t[g * 4 + 3]);
      }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int k0 = 0; k0 < NIT; k0 += BATCH) {
      float4 a[BATCH];
#pragma unroll
      for (int u = 0; u < BATCH; u++) {
        const int k = k0 + u, row = rsub[k % PER] + k / PER * 8;  // rsub < 8
        a[u] = *reinterpret_cast<const float4*>(wbuf + row * WC + ((c[k % PER] ^ rsub[k % PER]) << 2));
      }
#pragma unroll
      for (int u = 0; u < BATCH; u++) {
        const int k = k0 + u;
        float4 sd = make_float4(0.f, 0.f, 0.f, 0.f);
        if (SIDE) {
          const bf16x4 v = side[i & 1][k];
          sd = make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
        }
        mfma_epilogue4<EM>(e, mw + i * 32 + rsub[k % PER] + k / PER * 8, ncol[k % PER], a[u], bias[k % PER], sd);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// EK_LSE: of every row of the wave tile its largest element and the sum of e^(element - largest); to C as float2, one run of M rows for every
// 32 TN columns (ldc = M).  In place of the stores of 128 KB a tile, which a kernel of its own would read again.  A lane has half of a row in its
// accumulators and lane l ^ 32 the other: nothing goes through LDS.  A NaN gets through the maximum and the sum; a part without elements has
// -infinity and 0.  An element costs one fma and one exponential, of its difference from the largest to base 2 (the difference first and then the scale:
// 16384 x 50304 x 768 25 us more, of 1230); what the largest lost to rounding when it was scaled is put right in the sum.  From 2^30 on that may be more than
// the exponential can hold, and numbers that differ do so by 64 or more: their differences are left unscaled, since only those equal to the largest count.
static constexpr float LSE_LOG2E = 1.4426950408889634f;
template <bool MASK, int TM, int TN>
__device__ __forceinline__ void lse_epilogue(const EpiArgs& e, const f32x16 (&acc)[TM][TN], int mw, int nw, int M, int N, int lane) {
  float2 part[TM];
#pragma unroll
  for (int i = 0; i < TM; i++) {
    float z[TN * 16];
    int left = N - nw - (lane >> 5 << 2);  // columns from this lane's first on
    if (MASK) asm volatile("" : "+v"(left));  // opaque: one comparison a column for all rows would take 128 scalar registers
#pragma unroll
    for (int j = 0; j < TN; j++) {
      f32x16 a = acc[i][j];
      asm volatile("" : "+a"(a));  // read here and not before
#pragma unroll
      for (int v = 0; v < 16; v++) {
        z[j * 16 + v] = a[v];
        if (MASK) z[j * 16 + v] = j * 32 + 8 * (v >> 2) + (v & 3) < left ? z[j * 16 + v] : -INFINITY;
      }
    }
    float top = z[0];
#pragma unroll
    for (int t = 1; t < TN * 16; t++) top = __builtin_elementwise_maximum(top, z[t]);
    top = __builtin_elementwise_maximum(top, __shfl_xor(top, 32, 64));
    const float from = top == -INFINITY ? 0.f : top, scale = fabsf(top) < 1073741824.f ? LSE_LOG2E : 1.f, ref = from * scale;
    float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < TN * 16; t++) sum[t & 3] += __builtin_amdgcn_exp2f(fmaf(z[t], scale, -ref));
    float s = (sum[0] + sum[1]) + (sum[2] + sum[3]);
    s += __shfl_xor(s, 32, 64);
    s *= __builtin_amdgcn_exp2f(fmaf(-from, scale, ref));
    part[i] = make_float2(top, s);
    __builtin_amdgcn_sched_barrier(0);
  }
  // One group of rows in vector registers at a time, and no branch between: with the accumulators of all read ahead of the first, the tile loop's offsets
  // went to scratch and came back for every tile (216 bytes a lane with masks).  2048 x 13000 x 768, masked, 53 -> 48 us, where the stored product takes 49;
  // a validation step of one 768-wide layer, 16384 tokens, under 50304 columns 1586 -> 1534.
#pragma unroll
  for (int i = 0; i < TM; i++) {
    const int m = mw + i * 32 + (lane & 31);
    if (lane < 32 && (!MASK || m < M)) reinterpret_cast<float2*>(e.C)[(size_t)(nw / (TN * 32)) * e.ldc + m] = part[i];
  }
}

// Products of a grouped launch: weight gradients of one layer, which contract over the same tokens and do not depend on each other.
struct GemmItem {
  const bf16_t *A, *B;
  float *C, *colsum;
  int lda, ldb, ldc, M, N, tiles_m, tiles_n, group, a_lim, b_lim;
  int first;  // number of this product's first tile
};
static constexpr int GEMM_GROUP = 4;
template <bool GROUP>
struct GemmList {};
template <>
struct GemmList<true> {
  GemmItem p[GEMM_GROUP];
  int count, items;
};

// EDGE = false: M, N are multiples of the tile, K of the slab.  EDGE = true: any M, N, K.  Rows and
// columns beyond the operands' ends are fetched from their last row or column group (e.a_lim, e.b_lim:
// how far the operands reach) and never stored; contraction indices beyond K are fetched as zeros
// for both operands, by the last slab's loads only (the full slabs keep the scalar-base addressing).  Tiles inside the output keep the unmasked epilogue.
// Bound like the plain form by the rounds of tiles, padding included.  Against the scalar kernel that
// these shapes ran on before, a block at 3000 tokens x 1200 wide (F = 4800): forward products 1440 ->
// 180 us, input gradients 1610 -> 152, weight gradients with their bias sums 2470 -> 200, FFN-in with
// the GELU epilogue 680 -> 136, GELU' 528 -> 57.
// GROUP: the tiles of several products with the same K, one after the other (GemmList); the products' own sizes and operands
// take the place of the arguments, which are those of the first.
// `block` of `blocks` workgroups that share the tiles.
template <int BM, int BN, bool A_KC, bool B_KC, int EM, bool EDGE, bool GROUP>
__device__ __forceinline__ void mfma_tiles(int block, int blocks, int M, int N, int K, const bf16_t* __restrict__ A, int lda,
                                           const bf16_t* __restrict__ B, int ldb, EpiArgs e, int tiles_m, int tiles_n,
                                           const GemmList<GROUP>& list) {
  using LA = TileLds<BM, A_KC>;
  using LB = TileLds<BN, B_KC>;
  using EDGE_ = std::integral_constant<bool, EDGE>;
  constexpr int TM = BM / 64, TN = BN / 64;  // 32x32 MFMA tiles per wave in each direction
  extern __shared__ __attribute__((aligned(16))) char smem[];
  // LDS: three buffers for A slabs, then two for B slabs (see the pipeline below).
  constexpr int A_BUFS = 3;  // and two for B
  constexpr int B_BASE = A_BUFS * LA::BYTES;

  // Persistent workgroups: workgroup b works through tiles b, b + blocks, ...  (the host
  // launches one workgroup per CU, or fewer when there are fewer tiles).  The point is the seam
  // between two tiles: the first slabs of the next tile are requested before the epilogue of the
  // finished one, so their latency (about 3 us from a cold start) runs behind the epilogue.
  //
  // Tile number -> tile.  Consecutive workgroup ids land on different XCDs (8 of them, each with
  // its own L2) and `blocks` is a multiple of 8 whenever that matters, so a workgroup's tile
  // numbers all have its own residue mod 8; the number is first re-dealt so that each XCD owns a
  // contiguous run of tiles, then tiles are walked in column-major groups of e.group (4 or 8, chosen
  // on the host) tile-rows to keep the working set of A and B panels small.  e.group = 0 selects the
  // walk in which the XCDs' blocks of a round lie side by side (below).
  const int nt = tiles_m * tiles_n;
  int first = 0;  // GROUP: tile numbers before the current product's
  auto tile_of = [&](int id, int& tm_i, int& tn_i) { tile_walk(GROUP ? id - first : id, tiles_m, tiles_n, e.group, tm_i, tn_i); };
  auto product_of = [&](int id) {  // GROUP: the product that tile number `id` belongs to takes the arguments' place
    if constexpr (GROUP) {
      int n = 0;
#pragma unroll
      for (int q = 1; q < GEMM_GROUP; q++) n += q < list.count && id >= list.p[q].first;
      const GemmItem& g = list.p[n];
      A = g.A; B = g.B; lda = g.lda; ldb = g.ldb; M = g.M; N = g.N; tiles_m = g.tiles_m; tiles_n = g.tiles_n;
      e.C = g.C; e.colsum = g.colsum; e.ldc = g.ldc; e.group = g.group; e.a_lim = g.a_lim; e.b_lim = g.b_lim;
      first = g.first;
    }
  };

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // in a scalar register: LDS segment addresses stay scalar
  const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);

  // This wave's share of a slab: segments wave*NSEG .. +NSEG-1 of A and likewise of B.  Segment
  // q of a slab is bytes [1024 q, 1024 q + 1024) of its buffer; this lane's 16 bytes sit at
  // +16 lane.  The global address of a segment is (uniform slab base) + (this lane's offset,
  // fixed for the whole kernel), so stepping along K is scalar arithmetic only.
  constexpr int NSA = LA::NSEG, NSB = LB::NSEG;
  // (EDGE: where the tile lies against the operands' ends matters as well, GROUP: the product; recomputed per tile)
  constexpr bool PER_TILE = EDGE || GROUP;
  unsigned a_lane_off[NSA], b_lane_off[NSB];
  auto set_lane_offsets = [&](int tm, int tn) {
    int lane_o = lane;
    if (PER_TILE) asm volatile("" : "+v"(lane_o));  // opaque: the parts of the offsets that no tile changes are not worth a register each
#pragma unroll
    for (int q = 0; q < NSA; q++)
      a_lane_off[q] = slab_lane_offset<BM, A_KC, EDGE>(lda, (wave * NSA + q) * 1024 + lane_o * 16, e.a_lim - tm * BM);
#pragma unroll
    for (int q = 0; q < NSB; q++)
      b_lane_off[q] = slab_lane_offset<BN, B_KC, EDGE>(ldb, (wave * NSB + q) * 1024 + lane_o * 16, e.b_lim - tn * BN);
  };
  if (!PER_TILE) set_lane_offsets(0, 0);
  size_t a_kstride = A_KC ? 1 : (size_t)lda, b_kstride = B_KC ? 1 : (size_t)ldb;
  const unsigned smem_addr = lds_addr(smem);
  auto a_tile_of = [&](int tm_i) { return A + (A_KC ? (size_t)tm_i * BM * lda : (size_t)tm_i * BM); };
  auto b_tile_of = [&](int tn_i) { return B + (B_KC ? (size_t)tn_i * BN * ldb : (size_t)tn_i * BN); };
  // segment q of the A (B) slab at k0 of the tile at `tile_base` -> A (B) buffer number `buf`; of the
  // slab's contraction indices only the first `k_left` exist (cut: that may be fewer than a whole slab's)
  auto dma_from = [&](auto cut_c, const bf16_t* slab, unsigned lane_off, auto lane_k, int seg, int k_left, unsigned dst) {
    if constexpr (decltype(cut_c)::value) {
      int lane_t = lane;  // opaque: what is derived from it is rarely needed and must not occupy registers in the main loop
      asm volatile("" : "+v"(lane_t));
      const char* p = reinterpret_cast<const char*>(slab) + lane_off;
      lds_dma16(lane_k(seg * 1024 + lane_t * 16) < k_left ? (const void*)p : (const void*)&gemm_zero16, dst);
    } else {
      lds_dma16(slab, lane_off, dst);
    }
  };
  auto dma_a_from = [&](auto cut_c, const bf16_t* tile_base, int q, int k0, int buf, int k_left) {
    dma_from(cut_c, tile_base + k0 * a_kstride, a_lane_off[q], slab_lane_k<BM, A_KC>, wave * NSA + q, k_left,
             smem_addr + buf * LA::BYTES + (wave * NSA + q) * 1024);
  };
  auto dma_b_from = [&](auto cut_c, const bf16_t* tile_base, int q, int k0, int buf, int k_left) {
    dma_from(cut_c, tile_base + k0 * b_kstride, b_lane_off[q], slab_lane_k<BN, B_KC>, wave * NSB + q, k_left,
             smem_addr + B_BASE + buf * LB::BYTES + (wave * NSB + q) * 1024);
  };
  // With the contraction split (fp32-output form) the work items are (K range, tile) pairs: item
  // v is tile v % nt over slabs [r nkt / splits, (r + 1) nkt / splits), r = v / nt, nkt = K / GK,
  // and writes the partial product r (and the partial column sums r).
  const int splits = !GROUP && e.splits > 1 ? e.splits : 1;
  const int n_items = nt * splits;
  auto items = [&] {
    if constexpr (GROUP) return list.items;
    else return n_items;
  };
  const int nk_total = EDGE ? (K + GK - 1) / GK : K / GK;
  auto k_range = [&](int item, int& first, int& count) {
    const int r = GROUP ? 0 : item / nt;
    first = (int)((unsigned)r * (unsigned)nk_total / (unsigned)splits);  // r < 32, nk_total < 2^25
    count = (int)((unsigned)(r + 1) * (unsigned)nk_total / (unsigned)splits) - first;
  };
  // A tile starts with slab 0 in A[0], B[0] and slab 1 in A[1], B[1].  Everything but B of slab 1
  // can be requested while the previous tile's epilogue still uses A[2] and B[1].
  auto request_first_slabs = [&](const bf16_t* a_base, const bf16_t* b_base, int nk, int k_left) {
#pragma unroll
    for (int q = 0; q < NSA; q++) dma_a_from(EDGE_{}, a_base, q, 0, 0, k_left);
#pragma unroll
    for (int q = 0; q < NSB; q++) dma_b_from(EDGE_{}, b_base, q, 0, 0, k_left);
    if (nk > 1) {
#pragma unroll
      for (int q = 0; q < NSA; q++) dma_a_from(EDGE_{}, a_base, q, GK, 1, k_left - GK);
    }
  };

  int tm_i, tn_i;
  int k_first, nk_item;
  // of tile number `id`: product, tile, K range
  auto item_of = [&](int id) {
    product_of(id);
    if (GROUP) { a_kstride = A_KC ? 1 : (size_t)lda; b_kstride = B_KC ? 1 : (size_t)ldb; }
    tile_of(GROUP ? id : id % nt, tm_i, tn_i);
    k_range(id, k_first, nk_item);
  };
  item_of(block);
  size_t k_begin = (size_t)k_first * GK;
  if (PER_TILE) set_lane_offsets(tm_i, tn_i);
  request_first_slabs(a_tile_of(tm_i) + k_begin * a_kstride, b_tile_of(tn_i) + k_begin * b_kstride, nk_item, K - k_first * GK);
  for (int tile = block; tile < items(); tile += blocks) {
  const int nk = nk_item;
  const int k_end = K - k_first * GK;  // contraction indices from this item's first to the end of the operands
  const int m0 = tm_i * BM, n0 = tn_i * BN;
  const bf16_t* const a_tile = a_tile_of(tm_i) + k_begin * a_kstride;
  const bf16_t* const b_tile = b_tile_of(tn_i) + k_begin * b_kstride;
  EpiArgs et = e;  // this item's view of the epilogue operands
  const int M_item = M, N_item = N;
  if (!GROUP && em_kind(EM) == EK_F32) {
    et.C = (float*)e.C + (size_t)(tile / nt) * e.split_stride;
    if (EM & EM_COLSUM) et.colsum = e.colsum + (size_t)(tile / nt) * e.colsum_stride;
  }
  auto dma_a = [&](auto cut_c, int q, int k0, int buf) { dma_a_from(cut_c, a_tile, q, k0, buf, k_end - k0); };
  auto dma_b = [&](auto cut_c, int q, int k0, int buf) { dma_b_from(cut_c, b_tile, q, k0, buf, k_end - k0); };
  lds_dma_wait();   // slab 0 and A of slab 1 (requested a whole epilogue ago, except for the first tile)
  __syncthreads();  // ... are visible; every wave is done with the previous tile's epilogue staging
  if (nk > 1) {
#pragma unroll
    for (int q = 0; q < NSB; q++) dma_b(EDGE_{}, q, GK, 1);  // B of slab 1: needed at the first in-loop barrier, waited for there
  }
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;

  // Software pipeline.  A slab is four k-steps ("phases") of TM x TN MFMAs each.  Operand
  // fragments are double buffered in registers: phase s issues the LDS reads for phase s+1.
  //
  // With one wave per SIMD nothing else can fill the matrix core while this wave issues other
  // instructions, so they are slotted between MFMAs: slot t of a phase follows MFMA t and holds
  // at most one fragment read and one slab load.  sched_barrier after each slot keeps the
  // compiler from regrouping them.
  //
  // The slab loads set the pace of the schedule.  The CU's address unit takes 16 cycles per
  // 1 KB load instruction and is shared by the four waves, so a slab (64 instructions at 256^2)
  // keeps it busy for half of the slab's MFMA time: requested in one burst, the loads block the
  // issuing waves and with them the matrix cores.  They are therefore spread over the whole slab,
  // which needs somewhere to put them while both resident slabs are still being read: A gets a
  // third buffer.  While slab kt is multiplied,
  //   phases 0-1:          request A(kt+2) into the spare A buffer, a load every few slots;
  //   phase 2, slot PB:    all fragment reads of slab kt are done; wait until everything older
  //                        than the A loads just issued has landed (that is slab kt+1), barrier:
  //                        slab kt+1 is published and the B buffer of slab kt is free;
  //   rest of phase 2, 3:  request B(kt+2) into that buffer; phase 3 also reads the first
  //                        fragments of slab kt+1.
  // One barrier per slab.  PB leaves four MFMAs between the last fragment read and the wait.
  static_assert(GK / 16 == 4, "pipeline below is written for four k-steps per slab");
  constexpr int NSLOT = TM * TN;
  static_assert(TM + TN <= NSLOT, "slots per phase");
  static_assert(TN != 3 || (!EDGE && !GROUP && em_kind(EM) != EK_F32), "tile_epilogue96");
  constexpr int PB = (TM + TN + 4 < NSLOT) ? TM + TN + 4 : NSLOT;  // barrier position within phase 2
  constexpr int SLOTS_A = 2 * NSLOT;             // slots open to the A loads
  constexpr int SLOTS_B = NSLOT - PB + NSLOT;    // ... and to the B loads
  static_assert(NSA <= SLOTS_A && NSB <= SLOTS_B && NSA < 64, "load schedule");
  // Optional by-product (EM_COLSUM, B stored [K, N]): colsum[n] (+)= sum over k of B[k, n], which for
  // a weight-gradient product is the bias gradient.  Every workgroup sweeps all of K, so the
  // workgroups of tile row 0 between them see every column of B in full; their waves add up the
  // B fragments they feed to the matrix core anyway (lane = column, 8 k's per fragment).  The
  // two waves that share a column range (wm = 0 and wm != 0) take alternate elements, one
  // element per wave and slot at 256^2, and combine through LDS after the loop.  The main loop
  // exists in three copies (no sums, even elements, odd elements) so that the other workgroups
  // pay nothing and the element indices stay compile-time constants.
  constexpr bool CS = (EM & EM_COLSUM) != 0;
  static_assert(!CS || !B_KC, "column sums are taken from [K, N] fragments");
  const bool cs_on = CS && tm_i == 0;
  const int cs_half = wm != 0;
  float cs[TN];
#pragma unroll
  for (int j = 0; j < TN; j++) cs[j] = 0.f;
  auto main_loop = [&](auto cs_c, auto half_c) {
  constexpr bool CSON = decltype(cs_c)::value;
  constexpr int CS_HALF = decltype(half_c)::value;  // which element of each pair this wave sums
  constexpr int EPSL = 8 * TN / NSLOT;  // fragment elements summed per slot
  static_assert(EPSL % 2 == 0, "two waves share the elements of a slot");
  bf16x8 fa[2][TM], fb[2][TN];
  // Slots [T0, T1) of one phase: MFMA t on fragment buffer USE, then fragment read t of k-step ks
  // from (srcA, srcB) into buffer USE ^ 1 (when LOADF), then the slab loads that the schedule
  // puts at this slot: LOADS 1 = A loads, slot number t + OFS of SLOTS_A; LOADS 2 = B loads,
  // slot number t + OFS of SLOTS_B; segment q goes to slot floor(q * SLOTS / NSEG).
  auto phase = [&](auto cut_c, auto use_c, auto loadf_c, auto loads_c, auto ofs_c, auto t0_c, auto t1_c, const char* srcA,
                   const char* srcB, int ks, int k_next, int buf) {
    constexpr int USE = decltype(use_c)::value, LOADS = decltype(loads_c)::value, OFS = decltype(ofs_c)::value;
    constexpr int T0 = decltype(t0_c)::value, T1 = decltype(t1_c)::value;
    constexpr bool LOADF = decltype(loadf_c)::value;
#pragma unroll
    for (int t = T0; t < T1; t++) {
      const int i = t / TN, j = t % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[USE][j], fa[USE][i], acc[i][j], 0, 0, 0);  // C^T tile
      if (CSON) {  // this wave's half of the slot's elements: the wave with the other wm takes the rest
#pragma unroll
        for (int k = 0; k < EPSL / 2; k++) {
          const int el = t * EPSL + 2 * k + CS_HALF;
          cs[el / 8] += (float)fb[USE][el / 8][el % 8];
        }
      }
      if (LOADF) {
        if (t < TM) fa[USE ^ 1][t] = frag_load<BM, A_KC>(srcA, wm + t * 32, ks, lane);
        else if (t < TM + TN) fb[USE ^ 1][t - TM] = frag_load<BN, B_KC>(srcB, wn + (t - TM) * 32, ks, lane);
      }
      if (LOADS == 1) {
#pragma unroll
        for (int q = 0; q < NSA; q++)
          if (q * SLOTS_A / NSA == t + OFS) dma_a(cut_c, q, k_next, buf);
      }
      if (LOADS == 2) {
#pragma unroll
        for (int q = 0; q < NSB; q++)
          if (q * SLOTS_B / NSB == t + OFS) dma_b(cut_c, q, k_next, buf);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto a_buf = [&](int i) { return smem + i * LA::BYTES; };
  auto b_buf = [&](int i) { return smem + B_BASE + i * LB::BYTES; };

#pragma unroll
  for (int i = 0; i < TM; i++) fa[0][i] = frag_load<BM, A_KC>(a_buf(0), wm + i * 32, 0, lane);
#pragma unroll
  for (int j = 0; j < TN; j++) fb[0][j] = frag_load<BN, B_KC>(b_buf(0), wn + j * 32, 0, lane);
  int ia = 0;  // A buffer of the current slab: kt mod 3
  auto slab = [&](auto cut_c, int kt) {
    const int ia1 = ia == 2 ? 0 : ia + 1, ia2 = ia1 == 2 ? 0 : ia1 + 1;
    const int ib = kt & 1;
    const char* curA = a_buf(ia);
    const char* curB = b_buf(ib);
    const int k_next = min(kt + 2, nk - 1) * GK;  // past the end: the last slab again, into buffers nobody reads
    phase(cut_c, I<0>{}, T_{}, I<1>{}, I<0>{}, I<0>{}, I<NSLOT>{}, curA, curB, 1, k_next, ia2);
    phase(cut_c, I<1>{}, T_{}, I<1>{}, I<NSLOT>{}, I<0>{}, I<NSLOT>{}, curA, curB, 2, k_next, ia2);
    phase(cut_c, I<0>{}, T_{}, I<0>{}, I<0>{}, I<0>{}, I<PB>{}, curA, curB, 3, 0, 0);
    // Every fragment read of slab kt has returned (lgkmcnt) and, of this wave's loads, only the
    // NSA newest (A of slab kt+2) may still be in flight: slab kt+1 has landed.
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(NSA) : "memory");
    phase(cut_c, I<0>{}, F_{}, I<2>{}, I<-PB>{}, I<PB>{}, I<NSLOT>{}, curA, curB, 3, k_next, ib);
    phase(cut_c, I<1>{}, T_{}, I<2>{}, I<NSLOT - PB>{}, I<0>{}, I<NSLOT>{}, a_buf(ia1), b_buf(ib ^ 1), 0, k_next, ib);
    ia = ia1;
  };
  // EDGE: the loads of the last slab look at where K ends, in the two or three iterations that request it; the loop before
  // them is the plain form's (a branch around every load, as here once, cuts it into two dozen pieces: 34 us
  // instead of 24 at 3108 x 512 x 2048, 72 instead of 50 at 3000 x 1200 x 4800).
  int kt = 0;
  for (const int n = EDGE && k_end < nk * GK ? nk - 3 : nk - 1; kt < n; kt++) slab(F_{}, kt);
  if constexpr (EDGE) {
#pragma unroll 1
    for (; kt < nk - 1; kt++) slab(T_{}, kt);
  }
  {
    const char* curA = a_buf(ia);
    const char* curB = b_buf((nk - 1) & 1);
    phase(F_{}, I<0>{}, T_{}, I<0>{}, I<0>{}, I<0>{}, I<NSLOT>{}, curA, curB, 1, 0, 0);
    phase(F_{}, I<1>{}, T_{}, I<0>{}, I<0>{}, I<0>{}, I<NSLOT>{}, curA, curB, 2, 0, 0);
    phase(F_{}, I<0>{}, T_{}, I<0>{}, I<0>{}, I<0>{}, I<NSLOT>{}, curA, curB, 3, 0, 0);
    phase(F_{}, I<1>{}, F_{}, I<0>{}, I<0>{}, I<0>{}, I<NSLOT>{}, curA, curB, 0, 0, 0);
  }
  };  // main_loop
  if constexpr (CS) {
    if (!cs_on) main_loop(F_{}, I<0>{});
    else if (cs_half) main_loop(T_{}, I<1>{});
    else main_loop(T_{}, I<0>{});
  } else {
    main_loop(F_{}, I<0>{});
  }
  lds_dma_wait();  // the re-requested last slab: nothing may be in flight when LDS is reused or the wave ends

  // Epilogue (tile_epilogue).  The staging areas are A[2] (waves 0, 1) and B[1] (waves 2, 3): A[0], A[1] and B[0] are
  // already receiving the next tile.
  constexpr int WC = TN * 32;     // columns of the wave tile
  static_assert(2 * 32 * WC * 4 <= LA::BYTES && 2 * 32 * WC * 4 <= LB::BYTES, "two waves stage in one slab buffer");
  __syncthreads();                // every wave is done with the operand slabs
  float* wbuf = reinterpret_cast<float*>(smem + (wave < 2 ? 2 * LA::BYTES : B_BASE + LB::BYTES)) + (wave & 1) * 32 * WC;
  if constexpr (CS) {
    if (cs_on) {  // uniform over the workgroup
      // lanes l and l ^ 32 hold different k's of the same column; waves wm = 0 and wm != 0 different
      // elements.  Exchange through the start of the receiving wave's own staging area.
      float* xch = reinterpret_cast<float*>(smem + 2 * LA::BYTES) + (wave & 1) * 32 * WC;
#pragma unroll
      for (int j = 0; j < TN; j++) cs[j] += __shfl_xor(cs[j], 32, 64);
      if (cs_half && lane < 32) {
#pragma unroll
        for (int j = 0; j < TN; j++) xch[j * 32 + lane] = cs[j];
      }
      __syncthreads();
      if (!cs_half && lane < 32) {
#pragma unroll
        for (int j = 0; j < TN; j++) {
          const float v = cs[j] + xch[j * 32 + lane];
          float* o = et.colsum + n0 + wn + j * 32 + lane;
          if (!EDGE || n0 + wn + j * 32 + lane < N_item) *o = e.accumulate ? *o + v : v;
        }
      }
    }
  }
  // the next tile's first slabs, before anything else of the epilogue
  if (tile + blocks < items()) {
    item_of(tile + blocks);
    k_begin = (size_t)k_first * GK;
    if (PER_TILE) set_lane_offsets(tm_i, tn_i);
    request_first_slabs(a_tile_of(tm_i) + k_begin * a_kstride, b_tile_of(tn_i) + k_begin * b_kstride, nk_item, K - k_first * GK);
  }
  // (lane index through an opaque copy: otherwise everything derived from it below is hoisted out of
  // the tile loop and kept in registers across the main loop, which has none to spare)
  int lane_e = lane;
  asm volatile("" : "+v"(lane_e));
  auto epilogue = [&](auto mask_c) {
    if constexpr (em_kind(EM) == EK_LSE) lse_epilogue<decltype(mask_c)::value, TM, TN>(e, acc, m0 + wm, n0 + wn, M_item, N_item, lane_e);
    else if constexpr (TN == 3) tile_epilogue96<EM, TM>(e, acc, wbuf, m0 + wm, n0 + wn, lane_e);
    else tile_epilogue<EM, decltype(mask_c)::value, TM, TN>(GROUP ? et : e, et, acc, wbuf, m0 + wm, n0 + wn, M_item, N_item, lane_e);
  };  // epilogue
  if constexpr (EDGE) {
    if (m0 + BM > M_item || n0 + BN > N_item) epilogue(T_{});
    else epilogue(F_{});
  } else {
    epilogue(F_{});
  }
  }  // tile loop
  lds_dma_wait();  // nothing is in flight here; stated for whoever reads the assembly in a straight line
}

template <int BM, int BN, bool A_KC, bool B_KC, int EM, bool EDGE, bool GROUP>
__global__ __launch_bounds__(256) void gemm_mfma_kernel(int M, int N, int K, const bf16_t* __restrict__ A, int lda,
                                                        const bf16_t* __restrict__ B, int ldb, EpiArgs e, int tiles_m,
                                                        int tiles_n, GemmList<GROUP> list) {
  mfma_tiles<BM, BN, A_KC, B_KC, EM, EDGE, GROUP>(blockIdx.x, gridDim.x, M, N, K, A, lda, B, ldb, e, tiles_m, tiles_n, list);
}

template <int BM, int BN>
constexpr size_t mfma_lds() {  // 160 KB at 256^2; also covers the epilogue's staging
  return 3 * (size_t)TileLds<BM, true>::BYTES + 2 * (size_t)TileLds<BN, true>::BYTES;
}

// Workgroups of a launch.  Persistent: one per CU.  A 128^2 workgroup needs 80 KB of LDS and under 256 registers,
// so two fit on a CU; they share its LDS bandwidth, which bounds that kernel, and gain little
// (measured: +-0.4 % with many tiles) except when that saves a second round for a few left-over
// tiles (320 tiles: -4 % on the whole step).
static inline int mfma_grid(int bm, int items, int* grid) {
  static int n_cu = 0;  // benign race: same value from every thread
  if (n_cu == 0) {
    int dev = 0, v = 0;
    FAX_HIP(hipGetDevice(&dev));
    FAX_HIP(hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev));
    n_cu = v > 0 ? v : 256;
  }
  const int slots = (bm == 128 && items <= 2 * n_cu) ? 2 * n_cu : n_cu;
  *grid = items < slots ? items : slots;
  return FAX_OK;
}

template <int BM, int BN, bool A_KC, bool B_KC, int EM, bool EDGE = false, bool GROUP = false>
static int launch_mfma(const GemmArgs& g, const EpiArgs& e, hipStream_t s, const GemmList<GROUP>& list = GemmList<GROUP>()) {
  constexpr size_t lds = mfma_lds<BM, BN>();
  auto kern = gemm_mfma_kernel<BM, BN, A_KC, B_KC, EM, EDGE, GROUP>;
  static bool configured = false;  // benign race: the attribute is idempotent
  if (!configured) {
    FAX_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    configured = true;
  }
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  int items = tiles_m * tiles_n * (e.splits > 1 ? e.splits : 1), grid = 0;
  if constexpr (GROUP) items = list.items;
  FAX_TRY(mfma_grid(BM, items, &grid));
  EpiArgs ek = e;
  if (ek.group == 0 && grid != 256) ek.group = 4;  // the side-by-side walk is written for 8 XCDs x 32 workgroups
  hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, s, g.M, g.N, g.K, (const bf16_t*)g.A, g.lda,
                     (const bf16_t*)g.B, g.ldb, ek, tiles_m, tiles_n, list);
  FAX_LAUNCH_CHECK("gemm_mfma");
  return FAX_OK;
}

}  // namespace fax
