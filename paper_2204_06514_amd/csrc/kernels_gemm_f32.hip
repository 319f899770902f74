// fp32 GEMM on the CDNA4 matrix cores through their bf16 instruction: every fp32 factor is cut into three bf16 numbers, and
// v_mfma_f32_32x32x16_bf16 multiplies the pieces and adds the products in fp32.
//
// 2^24 x = hi + mid + lo, each the bf16 nearest to what the ones before leave: 8 + 8 + 8 significant bits, so the sum is 2^24 x itself.  The
// factor 2^24, taken out of the sums again, is what makes that so for every x: without it lo's last bits fall off the end of bf16 below
// 2^-110; with it every piece, of subnormal x too, is a multiple of 2^-125.  Of the nine products of two such sums the kernel
// forms the six that matter: hi hi, hi mid, mid hi, mid mid, hi lo, lo hi.  The three others are below 2^-24 of |x y| together
// (|mid| <= 2^-8 |x|, |lo| <= 2^-17 |x|), 2^-27 in the mean.  hi hi has accumulators of its own, the five small ones share
// others: of the additions that round at the size of the result there is one for sixteen contraction indices, where
// v_mfma_f32_32x32x2_f32 had one for two.  N(0, 1) factors, against float64 in the 2-norm, this kernel and that instruction: 16 contraction
// indices 3.3e-8 and 7.4e-8, 256 6e-8 and 1.5e-7, 1024 1.3e-7 and 5.7e-7 (2.9e-7 in its smallest tiles), 4096 2.7e-7 and 1.15e-6; factors
// of one sign, 4096: 1.8e-7 and 2.5e-7.
// Six of these instructions take 192 clocks for 16 contraction indices of a 32 x 32 tile where v_mfma_f32_32x32x2_f32 takes 512.
//
// A 512-thread workgroup (8 wavefronts, two per SIMD) computes a BM x BN tile: WM x WN waves share the tile, KS such groups of
// waves share the contraction indices of a slab (16 each) and add their accumulators up through LDS at the end.
// Slabs come as fp32 through registers, one or two ahead, are cut there (13 vector instructions for a pair of numbers, once per
// workgroup) and stored as three bf16 planes to the other LDS buffer while the current slab is multiplied; one barrier per slab.
// Any M, N, K and orientation: rows and columns beyond the operands are fetched from their last
// row or column and never stored, contraction indices beyond K become zeros on the way into LDS.
//
// A plane of an operand whose contraction index is contiguous in memory is kept as [row][k], its 16-byte chunks XOR-ed with the row's
// place so that sixteen consecutive rows meet sixteen different places of the 256-byte bank window; the other kind as [k][row], as
// in the bf16 kernel, and read with the LDS transpose read (frag_load, mc_swizzle).  No bank conflicts either way (SQ_LDS_BANK_CONFLICT).
//
// What the pieces cannot carry is computed again, by the wave that finds it in its own partial sums, with v_mfma_f32_32x32x2_f32 on the
// factors as they are, straight from memory: sums that are not finite (an infinite factor's remainder is NaN, and an infinity times a
// piece that is zero is NaN where the product is an infinity; a factor that is not finite, or 2^104 and more, always leaves such a sum, and
// so does a partial sum of 2^80 and more).  A sum that is finite stays as it is, whatever its neighbours are: which of the two an
// element gets hangs on its own row and column alone.  So are contractions over fewer than four indices, whose sums are so short that the
// instruction rounds less: over 1 index 2.5e-8 and 2.6e-8 in the pieces, at most 1.0 and 1.8 x 2^-24 of |x y|, over 2 at most 1.9 and 2.4 of
// the sum of |x y|, over 4 3.3 and 2.4.
//
// Lane layout (lane l): operands = row / column l & 31, k = 8 (l >> 5) + 0..7; accumulator v holds element
// [8 (v >> 2) + 4 (l >> 5) + (v & 3)][l & 31]: 32 lanes store 32 consecutive columns.
#include "gemm_mfma_kernel.h"

namespace fax {

// One chunk of four consecutive floats of a slab.  KC: chunk c is four k's of row c / (BK / 4); otherwise four rows of k-row
// c / (ROWS / 4).  What lies beyond `rows` is fetched from the last row; what lies beyond `K` from the last k
// and zeroed by chunk_mask() before it is used.
template <int ROWS, int BK, bool KC, bool VEC>
__device__ __forceinline__ float4 chunk_load(const float* __restrict__ p, int ld, int rows, int K, int r0, int k0, int c) {
  if (KC) {
    const int row = min(r0 + c / (BK / 4), rows - 1), k = k0 + c % (BK / 4) * 4;
    const float* q = p + (size_t)row * ld;
    if (VEC) return *reinterpret_cast<const float4*>(q + min(k, K - 4));
    return make_float4(q[min(k, K - 1)], q[min(k + 1, K - 1)], q[min(k + 2, K - 1)], q[min(k + 3, K - 1)]);
  }
  const int k = min(k0 + c / (ROWS / 4), K - 1), row = r0 + c % (ROWS / 4) * 4;
  const float* q = p + (size_t)k * ld;
  if (VEC) return *reinterpret_cast<const float4*>(q + min(row, rows - 4));
  return make_float4(q[min(row, rows - 1)], q[min(row + 1, rows - 1)], q[min(row + 2, rows - 1)], q[min(row + 3, rows - 1)]);
}
// The same for whole vectors, as bytes from the slab's first element (row r0, index k0): fixed but for the slab in which K ends, so that a load needs
// a scalar address and this, where working the place out for each took as much of the vector unit as two thirds of the cutting: 4096 x 4096 x 4096
// 742 -> 662 us with both operands [row][k], 2048 x 4096 x 1024 104 -> 97, [K, N] weights 107 -> 103.
template <int ROWS, int BK, bool KC>
__device__ __forceinline__ unsigned chunk_offset(int ld, int rows, int k_left, int c) {  // rows, k_left: how many there are from the slab's first
  if (KC) return 4u * ((unsigned)min(c / (BK / 4), rows - 1) * (unsigned)ld + (unsigned)min(c % (BK / 4) * 4, k_left - 4));
  return 4u * ((unsigned)min(c / (ROWS / 4), k_left - 1) * (unsigned)ld + (unsigned)min(c % (ROWS / 4) * 4, rows - 4));
}
static constexpr int CHUNK_MAX_LD = 1 << 22;  // 128 rows of it are 2^31 bytes
template <int ROWS, int BK, bool KC, bool VEC>
__device__ __forceinline__ float4 chunk_mask(float4 v, int K, int k0, int c) {
  if (KC) {
    const int left = K - (k0 + c % (BK / 4) * 4);
    return make_float4(left > 0 ? v.x : 0.f, left > (VEC ? 0 : 1) ? v.y : 0.f, left > (VEC ? 0 : 2) ? v.z : 0.f,
                       left > (VEC ? 0 : 3) ? v.w : 0.f);
  }
  return k0 + c / (ROWS / 4) < K ? v : make_float4(0.f, 0.f, 0.f, 0.f);
}

static constexpr float SPLIT_UP = 16777216.f, SPLIT_DOWN = 1.f / SPLIT_UP / SPLIT_UP;  // 2^24 of each factor, 2^-48 of a product
static constexpr int SPLIT_MIN_K = 4;

// Four numbers, times SPLIT_UP, as 3 x 4 bf16.
__device__ __forceinline__ void split4(float4 v, uint2 (&p)[3]) {
  float r[4] = {v.x * SPLIT_UP, v.y * SPLIT_UP, v.z * SPLIT_UP, v.w * SPLIT_UP};
#pragma unroll
  for (int q = 0; q < 3; q++) {
    unsigned w[2];
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const bf16x2 t = {(__bf16)r[2 * i], (__bf16)r[2 * i + 1]};
      w[i] = __builtin_bit_cast(unsigned, t);
      asm("" : "+v"(w[i]));  // opaque: the compiler would convert the lower of the two once more by itself
      if (q < 2) {
        r[2 * i] -= __uint_as_float(w[i] << 16);
        r[2 * i + 1] -= __uint_as_float(w[i] & 0xffff0000u);
      }
    }
    p[q] = make_uint2(w[0], w[1]);
  }
}
// Eight numbers as an MFMA operand's three pieces.
__device__ __forceinline__ void split8(const float (&x)[8], bf16x8 (&f)[3]) {
  uint2 lo[3], hi[3];
  split4(make_float4(x[0], x[1], x[2], x[3]), lo);
  split4(make_float4(x[4], x[5], x[6], x[7]), hi);
#pragma unroll
  for (int q = 0; q < 3; q++) f[q] = __builtin_bit_cast(bf16x8, make_uint4(lo[q].x, lo[q].y, hi[q].x, hi[q].y));
}

// One operand's slab in LDS: three planes.
template <int ROWS, int BK, bool KC>
struct SplitSlab {
  static constexpr int PLANE = ROWS * BK * 2;  // bytes
  static constexpr int BYTES = 3 * PLANE;
  static constexpr int CHUNKS = ROWS * BK / 4 / 512;  // per thread
  static __device__ __forceinline__ int swz(int row) {  // 16-byte chunks of a [row][k] plane: 4, 8 or 16 to a row
    return BK == 32 ? (row >> 2) & 3 : BK == 64 ? (row >> 1) & 7 : row & 15;
  }
  static __device__ __forceinline__ int place(int c) {
    if (KC) {
      const int row = c / (BK / 4), k4 = c % (BK / 4);
      return row * (BK * 2) + (((k4 >> 1) ^ swz(row)) << 4) + (k4 & 1) * 8;
    }
    const int k = c / (ROWS / 4), r4 = c % (ROWS / 4);
    return k * (ROWS * 2) + (((r4 >> 2) ^ mc_swizzle<ROWS>(k)) << 5) + (r4 & 3) * 8;
  }
  static __device__ __forceinline__ bf16x8 frag(const char* plane, int rb, int ks, int lane) {
    if constexpr (KC) {
      const int row = rb + (lane & 31), chunk = ks * 2 + (lane >> 5);
      return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(plane + row * (BK * 2) + ((chunk ^ swz(row)) << 4)));
    } else {
      return frag_load<ROWS, false>(plane, rb, ks, lane);
    }
  }
};

// Work items in eight runs, one per XCD (consecutive workgroup ids land on different ones), each walked
// down column-major groups of eight tile rows, so that what an XCD works on at a time shares operand panels.
__device__ __forceinline__ void f32_tile(int id, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int nt = tiles_m * tiles_n;
  if (nt % 8 == 0) id = (id % 8) * (nt / 8) + id / 8;
  const int per_group = 8 * tiles_n, g = id / per_group, rest = id % per_group;
  const int gsz = min(8, tiles_m - 8 * g);
  tm = 8 * g + rest % gsz;
  tn = rest / gsz;
}

// Bound, with a full chip, by the matrix cores at the clock that their power leaves (4096 x 4096 x 4096: 199 to 208 TFLOP/s counted once, 1.2
// to 1.25 bf16 PFLOP/s), with one workgroup on a CU by the chain from barrier to barrier: loads, cutting, LDS and back, 24
// MFMAs.  In the block below the matrix cores are busy 37 to 59 % of the busy CUs' clocks, the vector unit, mostly with the cutting, 41 to 56 %, and
// waits are 19 to 24 % of the waves' time.  v_mfma_f32_32x32x2_f32 sustains 154 from registers alone; the kernel on it that this one replaces, us: 2048 x 3072 x 1024 145, here
// 91; 2048 x 1024 x 1024 52, 30; 2048 x 4096 x 1024 160, 92 to 96; 2048 x 1024 x 4096 172, 104; its block of 2048 tokens x 1024 wide,
// forward and backward, 1625, 1150.
// Phases the other way round in one or both waves of a SIMD, s_setprio around the cutting, requests further ahead: within 2 %.
// Fragments requested before the slab is cut instead of where they are used: 3 %, 128 x 64 8 %.  128 x 64 as 64 x 32 per wave and slabs of 32: 6 % slower.
template <int WM, int WN, int KS, int TM, int TN>
struct SplitShape {
  static constexpr int BM = WM * TM * 32, BN = WN * TN * 32, BK = 16 * KS;
  static constexpr int NV = TM * TN * 16;                               // accumulators per lane
  static constexpr int XCH = (KS == 8 ? NV : NV - NV / KS) * 8 * 64;     // floats of the exchange at the end
  static constexpr int AHEAD = (BM + BN) >= 192 ? 1 : 2;                // slabs requested ahead
};

// GELU: forward orientation with EPI_GELU, its transcendental code kept out of the other instances.
template <int WM, int WN, int KS, int TM, int TN, bool TA, bool TB, bool VEC, bool GELU>
__device__ __forceinline__ void f32_product_tile(int block, int M, int N, int K, const float* __restrict__ A, int lda,
                                                 const float* __restrict__ B, int ldb, const EpiArgs& e, int tiles_m, int tiles_n) {
  using S = SplitShape<WM, WN, KS, TM, TN>;
  static_assert(WM * WN * KS == 8, "eight waves");
  constexpr int BM = S::BM, BN = S::BN, BK = S::BK, NV = S::NV, AHEAD = S::AHEAD;
  using SA = SplitSlab<BM, BK, !TA>;
  using SB = SplitSlab<BN, BK, TB>;
  constexpr int BUF = SA::BYTES + SB::BYTES;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  float* const smem_f = reinterpret_cast<float*>(smem);

  int tm_i, tn_i;
  f32_tile(block, tiles_m, tiles_n, tm_i, tn_i);
  const int m0 = tm_i * BM, n0 = tn_i * BN;
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l31 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / (WM * WN);  // this wave's 16 contraction indices of a slab
  const int wm = wave / WN % WM * (TM * 32), wn = wave % WN * (TN * 32);
  const int a_rows = TA ? e.a_lim : M, a_k = TA ? K : e.a_lim;  // how far A may be read

  // Optional by-product of the weight-gradient form: colsum[n] (+)= sum over k of B[k, n], from the slabs as they pass through the
  // registers (a thread has the same four columns, in the smallest tiles one column, of every slab); what each addition to the running sum rounds off is carried along.
  // 2048 rows of N(0, 1): 0.6e-7 from float64, 1.3e-7 in the separate pass that this stands in for.
  constexpr bool CS = TA && !TB;
  const bool cs_on = CS && e.colsum && tm_i == 0;  // uniform over the workgroup
  float cs[4] = {0.f, 0.f, 0.f, 0.f}, cs_lost[4] = {0.f, 0.f, 0.f, 0.f};

  // In the smallest tiles, which are all latency, a lane stores two elements whose side inputs can be on their way from the start.
  static_assert(KS < 8 || NV == 16, "one tile, shared by all waves");
  const int mb8 = m0 + wave / 2 * 8 + 4 * h + wave % 2 * 2;
  float pre_bias = 0.f, pre_r[2], pre_u[2], pre_c[2];
  if (KS == 8) {
    const int nr = min(n0 + l31, N - 1);
    if (e.bias) pre_bias = ((const float*)e.bias)[nr];
#pragma unroll
    for (int t = 0; t < 2; t++) {
      const size_t m = min(mb8 + t, M - 1);
      if (e.R) pre_r[t] = ((const float*)e.R)[m * e.ldr + nr];
      if (e.epi == EPI_DGELU) pre_u[t] = ((const float*)e.U)[m * e.ldu + nr];
      if (e.accumulate) pre_c[t] = ((const float*)e.C)[m * e.ldc + nr];
    }
  }

  // hi hi goes to `acc`, the other products to `small`, which is 2^-8 of it and rounds off that much less.
  f32x16 acc[TM][TN], small[TM][TN];
  auto clear = [&](f32x16 (&t)[TM][TN]) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++)
#pragma unroll
        for (int v = 0; v < 16; v++) t[i][j][v] = 0.f;
  };
  clear(acc);
  clear(small);
  const int ns = (K + BK - 1) / BK;
  if constexpr (KS == 8) {
    // No fragment is used by two waves here: each takes its own from memory, cuts it in registers and multiplies, a slab ahead in
    // flight, with neither LDS nor barriers.
    float xa[2][8], xb[2][8];
    auto get = [&](bool kc, const float* p, int ld, int row, int lim, int k, float (&x)[8]) __attribute__((always_inline)) {
      if (kc && VEC) {
        const float* q = p + (size_t)row * ld;
        const float4 u = *reinterpret_cast<const float4*>(q + min(k, lim - 4)), w = *reinterpret_cast<const float4*>(q + min(k + 4, lim - 4));
        x[0] = u.x; x[1] = u.y; x[2] = u.z; x[3] = u.w; x[4] = w.x; x[5] = w.y; x[6] = w.z; x[7] = w.w;
      } else {
#pragma unroll
        for (int t = 0; t < 8; t++) x[t] = kc ? p[(size_t)row * ld + min(k + t, lim - 1)] : p[(size_t)min(k + t, lim - 1) * ld + row];
      }
    };
    const int row_a = min(m0 + l31, M - 1), row_b = min(n0 + l31, N - 1);
    auto request = [&](auto set_c, int s) __attribute__((always_inline)) {
      constexpr int SET = decltype(set_c)::value;
      const int k = s * BK + kg * 16 + 8 * h;
      get(!TA, A, lda, row_a, TA ? K : a_k, k, xa[SET]);
      get(TB, B, ldb, row_b, K, k, xb[SET]);
    };
    auto take_in = [&](auto set_c, int s) __attribute__((always_inline)) {
      constexpr int SET = decltype(set_c)::value;
      const int left = K - (s * BK + kg * 16 + 8 * h);
      if (s * BK + BK > K) {  // the slab in which K ends
#pragma unroll
        for (int t = 0; t < 8; t++) {
          xa[SET][t] = t < left ? xa[SET][t] : 0.f;
          xb[SET][t] = t < left ? xb[SET][t] : 0.f;
        }
      }
      bf16x8 ga[3], gb[3];
      split8(xa[SET], ga);
      split8(xb[SET], gb);
      if (CS && cs_on) {
        const float* x = xb[SET];
        const float c = ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
        const float t = cs[0] + c, was = t - c;
        cs_lost[0] += (cs[0] - was) + (c - (t - was));
        cs[0] = t;
      }
      constexpr int QA[6] = {2, 0, 0, 1, 1, 0}, QB[6] = {0, 2, 0, 1, 0, 1};
#pragma unroll
      for (int q = 0; q < 6; q++) {
        f32x16& t = q == 2 ? acc[0][0] : small[0][0];
        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ga[QA[q]], gb[QB[q]], t, 0, 0, 0);
      }
    };
    if (ns > 0) request(I<0>{}, 0);
    int s = 0;
    for (; s + 2 < ns; s += 2) {
      request(I<1>{}, s + 1);
      take_in(I<0>{}, s);
      request(I<0>{}, s + 2);
      take_in(I<1>{}, s + 1);
    }
    if (s + 1 < ns) {
      request(I<1>{}, s + 1);
      take_in(I<0>{}, s);
      take_in(I<1>{}, s + 1);
    } else if (s < ns) {
      take_in(I<0>{}, s);
    }
  } else {
    float4 ra[AHEAD][SA::CHUNKS], rb[AHEAD][SB::CHUNKS];  // slabs on their way from memory to LDS
    // Not for weight gradients, whose two operands are both [k][row] (3072 x 1024 x 2048 81 us, 84 with it), and of the smaller tiles only where both are [row][k].
    constexpr bool PLACES = VEC && !TA && (TB || BM + BN >= 192);
    unsigned oa[SA::CHUNKS], ob[SB::CHUNKS];
    auto places = [&](int k0) {
#pragma unroll
      for (int i = 0; i < SA::CHUNKS; i++) oa[i] = chunk_offset<BM, BK, !TA>(lda, a_rows - m0, a_k - k0, tid + i * 512);
#pragma unroll
      for (int i = 0; i < SB::CHUNKS; i++) ob[i] = chunk_offset<BN, BK, TB>(ldb, N - n0, K - k0, tid + i * 512);
    };
    if (PLACES) places(0);
    auto request = [&](auto set_c, int s) {
      constexpr int SET = decltype(set_c)::value;
      const int k0 = s * BK;
      if constexpr (PLACES) {
        if (s > 0 && s == ns - 1) places(k0);  // (no load in a branch)
        const char* a = reinterpret_cast<const char*>(A + (TA ? (size_t)k0 * lda + m0 : (size_t)m0 * lda + k0));
        const char* b = reinterpret_cast<const char*>(B + (TB ? (size_t)n0 * ldb + k0 : (size_t)k0 * ldb + n0));
#pragma unroll
        for (int i = 0; i < SA::CHUNKS; i++) ra[SET][i] = *reinterpret_cast<const float4*>(a + oa[i]);
#pragma unroll
        for (int i = 0; i < SB::CHUNKS; i++) rb[SET][i] = *reinterpret_cast<const float4*>(b + ob[i]);
      } else {
#pragma unroll
        for (int i = 0; i < SA::CHUNKS; i++) ra[SET][i] = chunk_load<BM, BK, !TA, VEC>(A, lda, a_rows, a_k, m0, k0, tid + i * 512);
#pragma unroll
        for (int i = 0; i < SB::CHUNKS; i++) rb[SET][i] = chunk_load<BN, BK, TB, VEC>(B, ldb, N, K, n0, k0, tid + i * 512);
      }
    };
    auto publish = [&](auto set_c, int s) {
      constexpr int SET = decltype(set_c)::value;
      const int k0 = s * BK;
      char* const buf = smem + (s & 1) * BUF;
      if (k0 + BK > K) {  // the slab in which K ends
#pragma unroll
        for (int i = 0; i < SA::CHUNKS; i++) ra[SET][i] = chunk_mask<BM, BK, !TA, VEC>(ra[SET][i], K, k0, tid + i * 512);
#pragma unroll
        for (int i = 0; i < SB::CHUNKS; i++) rb[SET][i] = chunk_mask<BN, BK, TB, VEC>(rb[SET][i], K, k0, tid + i * 512);
      }
      auto put = [&](char* p, int plane, float4 v) {
        uint2 w[3];
        split4(v, w);
#pragma unroll
        for (int q = 0; q < 3; q++) *reinterpret_cast<uint2*>(p + q * plane) = w[q];
      };
#pragma unroll
      for (int i = 0; i < SA::CHUNKS; i++) put(buf + SA::place(tid + i * 512), SA::PLANE, ra[SET][i]);
#pragma unroll
      for (int i = 0; i < SB::CHUNKS; i++) put(buf + SA::BYTES + SB::place(tid + i * 512), SB::PLANE, rb[SET][i]);
      if (CS && cs_on) {
        float t4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < SB::CHUNKS; i++) { t4[0] += rb[SET][i].x; t4[1] += rb[SET][i].y; t4[2] += rb[SET][i].z; t4[3] += rb[SET][i].w; }
#pragma unroll
        for (int j = 0; j < 4; j++) {
          const float t = cs[j] + t4[j], was = t - t4[j];
          cs_lost[j] += (cs[j] - was) + (t4[j] - (t - was));
          cs[j] = t;
        }
      }
    };

    bf16x8 fa[3][TM], fb[3][TN];
    auto fetch = [&](int s) {  // the fragments of slab s
      const char* const a = smem + (s & 1) * BUF;
      const char* const b = a + SA::BYTES;
      constexpr int QA[3] = {2, 0, 1}, QB[3] = {0, 2, 1};  // in the order of their use
#pragma unroll
      for (int q = 0; q < 3; q++) {
#pragma unroll
        for (int i = 0; i < TM; i++) fa[QA[q]][i] = SA::frag(a + QA[q] * SA::PLANE, wm + i * 32, kg, lane);
#pragma unroll
        for (int j = 0; j < TN; j++) fb[QB[q]][j] = SB::frag(b + QB[q] * SB::PLANE, wn + j * 32, kg, lane);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&] {
      constexpr int QA[6] = {2, 0, 0, 1, 1, 0}, QB[6] = {0, 2, 0, 1, 0, 1};
#pragma unroll
      for (int q = 0; q < 6; q++)
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
          for (int j = 0; j < TN; j++) {
            f32x16& t = q == 2 ? acc[i][j] : small[i][j];
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[QA[q]][i], fb[QB[q]][j], t, 0, 0, 0);
          }
      __builtin_amdgcn_sched_barrier(0);
    };

    // Slab s + 1 is cut and stored while slab s is multiplied; its registers then take slab s + 1 + AHEAD.  Of the two waves of a
    // SIMD one multiplies first and the other cuts first.  The requests are unconditional (past the end the last slab again, never
    // used): around conditional ones the compiler would wait for all loads in flight.
    const bool early = wave < 4;
    auto turn = [&](auto set_c, int s) {  // set_c: (s + 1) % AHEAD
      fetch(s);
      if (!early) multiply();
      publish(set_c, s + 1);
      request(set_c, min(s + 1 + AHEAD, ns - 1));
      __builtin_amdgcn_sched_barrier(0);
      if (early) multiply();
      __syncthreads();
    };
    if (ns == 1) {
      request(I<0>{}, 0);
      publish(I<0>{}, 0);
      __syncthreads();
      fetch(0);
      multiply();
    } else if (ns > 1) {
      request(I<0>{}, 0);
      if (AHEAD > 1) request(I<1 % AHEAD>{}, min(1, ns - 1));
      if (AHEAD > 2) request(I<2 % AHEAD>{}, min(2, ns - 1));
      publish(I<0>{}, 0);
      request(I<0>{}, min(AHEAD, ns - 1));
      __syncthreads();
      int s = 0;
      for (; s + AHEAD < ns; s += AHEAD) {
        turn(I<1 % AHEAD>{}, s);
        if (AHEAD > 1) turn(I<2 % AHEAD>{}, s + 1);
        if (AHEAD > 2) turn(I<0>{}, s + 2);
      }
      if (s + 1 < ns) turn(I<1 % AHEAD>{}, s++);
      if (s + 1 < ns) turn(I<2 % AHEAD>{}, s++);
      fetch(s);
      multiply();
    }
  }

  // The sums of this wave's contraction indices; again, of the same indices, on the fp32 instruction where they are not finite.  The wave loads
  // its fragments from memory as it multiplies.  2048 x 4096 x 1024, 98 to 126 us by orientation, takes 224 to 266 with one
  // infinite factor, 306 to 540 with one in every row; the kernel on that instruction alone 143 to 161.
  bool finite = K >= SPLIT_MIN_K;
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) {
        acc[i][j][v] = (acc[i][j][v] + small[i][j][v]) * SPLIT_DOWN;
        finite = finite && fabsf(acc[i][j][v]) <= 3.4028235e38f;
      }
  if (__ballot(!finite)) {
    clear(small);
    for (int k0 = kg * 16; k0 < K; k0 += k0 % 16 ? BK - 8 : 8) {  // a slab's sixteen in two eights
      float xa[TM][4], xb[TN][4];
#pragma unroll
      for (int t = 0; t < 4; t++) {
        const int k = k0 + 4 * h + t, kr = min(k, K - 1);
#pragma unroll
        for (int i = 0; i < TM; i++) {
          const int row = min(m0 + wm + i * 32 + l31, M - 1);
          const float x = A[TA ? (size_t)kr * lda + row : (size_t)row * lda + kr];
          xa[i][t] = k < K ? x : 0.f;
        }
#pragma unroll
        for (int j = 0; j < TN; j++) {
          const int row = min(n0 + wn + j * 32 + l31, N - 1);
          const float x = B[TB ? (size_t)row * ldb + kr : (size_t)kr * ldb + row];
          xb[j][t] = k < K ? x : 0.f;
        }
      }
#pragma unroll
      for (int t = 0; t < 4; t++)
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
          for (int j = 0; j < TN; j++) small[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(xa[i][t], xb[j][t], small[i][j], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++)
#pragma unroll
        for (int v = 0; v < 16; v++)
          if (K < SPLIT_MIN_K || !(fabsf(acc[i][j][v]) <= 3.4028235e38f)) acc[i][j][v] = small[i][j][v];
  }

  // The end: accumulators that other groups store and column sums go through LDS together.
  float* const cs_x = smem_f + S::XCH;
  constexpr int NH = NV / KS;  // accumulators of a lane that its group stores: tiles of 16, or a part of one
  constexpr int GW = WM * WN;  // waves of a group
  auto mine = [&](int t) { return acc[t / 16 / TN][t / 16 % TN][t % 16]; };
  auto hand = [&](auto keep_c) __attribute__((always_inline)) {  // group KEEP's wave: what group o stores, at the place of the giver
    constexpr int KEEP = decltype(keep_c)::value;
#pragma unroll
    for (int o = 0; o < KS; o++) {
      if (o == KEEP) continue;
#pragma unroll
      for (int t = 0; t < NH; t++) smem_f[((wave * (KS - 1) + (o < KEEP ? o : o - 1)) * NH + t) * 64 + lane] = mine(o * NH + t);
    }
    asm volatile("" : : "n"(KEEP));  // the groups' copies stay apart: merged, they would index the accumulators at run time
  };
  float v[NH];
  auto take = [&](auto keep_c) __attribute__((always_inline)) {
    constexpr int KEEP = decltype(keep_c)::value;
    auto from = [&](int g, int t) {
      return g == KEEP ? mine(KEEP * NH + t)
                       : smem_f[((((wave & (GW - 1)) + g * GW) * (KS - 1) + (KEEP < g ? KEEP : KEEP - 1)) * NH + t) * 64 + lane];
    };
#pragma unroll
    for (int t = 0; t < NH; t++) {
      v[t] = from(0, t) + from(1, t);
      if constexpr (KS == 4) v[t] += from(2, t) + from(3, t);
    }
    asm volatile("" : : "n"(KEEP));
  };
  auto by_group = [&](auto f) __attribute__((always_inline)) {
    if constexpr (KS == 4) {
      if (kg == 3) f(I<3>{});
      else if (kg == 2) f(I<2>{});
      else if (kg == 1) f(I<1>{});
      else f(I<0>{});
    } else {
      if (kg) f(I<1>{});
      else f(I<0>{});
    }
  };
  auto exchange = [&]() __attribute__((always_inline)) {
    if constexpr (KS < 8) {
      by_group(hand);
    } else {
#pragma unroll
      for (int t = 0; t < 16; t++) smem_f[(wave * 16 + t) * 64 + lane] = acc[0][0][t];
    }
  };
  if (KS < 8) __syncthreads();  // every wave is done with the slabs
  exchange();
  if (CS && cs_on) {  // lanes CL apart have the same columns, and so have the waves
    constexpr int CC = KS == 8 ? 1 : 4, CL = BN / CC;
#pragma unroll
    for (int j = 0; j < CC; j++) {
      if (fabsf(cs[j]) <= 3.4028235e38f) cs[j] += cs_lost[j];  // (of an infinity, what was lost is NaN)
#pragma unroll
      for (int o = 32; o >= CL; o >>= 1) cs[j] += __shfl_xor(cs[j], o, 64);
      if (lane < CL) cs_x[wave * BN + lane * CC + j] = cs[j];
    }
  }
  __syncthreads();
  if (CS && cs_on && tid < BN && n0 + tid < N) {
    const float* q = cs_x + tid;
    const float c = ((q[0] + q[BN]) + (q[2 * BN] + q[3 * BN])) + ((q[4 * BN] + q[5 * BN]) + (q[6 * BN] + q[7 * BN]));
    e.colsum[n0 + tid] = e.accumulate ? e.colsum[n0 + tid] + c : c;
  }

  // Epilogue of NE elements of one column n: rows mb + (t & 3) + 8 (t >> 2).  Side inputs are fetched from clamped places
  // (all of them in flight together), stores are predicated.
  auto emit = [&](auto ne_c, float* v, int mb, int n) {
    constexpr int NE = decltype(ne_c)::value;
    const int nr = min(n, N - 1);
    auto row = [&](int t) { return mb + (t & 3) + 8 * (t >> 2); };
    auto fetch = [&](const void* p, int ld, float (&d)[NE], const float* pre) {
#pragma unroll
      for (int t = 0; t < NE; t++) d[t] = KS == 8 ? pre[t] : ((const float*)p)[(size_t)min(row(t), M - 1) * ld + nr];
    };
    auto store = [&](void* p, int ld, const float* d) {
#pragma unroll
      for (int t = 0; t < NE; t++)
        if (n < N && row(t) < M) ((float*)p)[(size_t)row(t) * ld + n] = d[t];
    };
    const float bias = KS == 8 ? pre_bias : e.bias ? ((const float*)e.bias)[nr] : 0.f;
    if (GELU) {
      // one element at a time out of the lane's own LDS slots: sixteen copies of tanh and erf would not fit the instruction cache
      float* slot = smem_f + S::XCH + 8 * BN + wave * 64 * NE + lane;
#pragma unroll
      for (int t = 0; t < NE; t++) slot[t * 64] = v[t];
#pragma unroll 1
      for (int t = 0; t < NE; t++) {
        const float u = slot[t * 64] + bias;
        const float g = gelu_f(u, e.gelu_form), dg = gelu_grad_f(u, e.gelu_form);
        if (n < N && row(t) < M) {
          ((float*)e.C)[(size_t)row(t) * e.ldc + n] = dg;
          ((float*)e.C2)[(size_t)row(t) * e.ldc2 + n] = g;
        }
      }
      return;
    }
    float side[NE];
    if (e.C2) store(e.C2, e.ldc2, v);
#pragma unroll
    for (int t = 0; t < NE; t++) v[t] += bias;
    if (e.R) {
      fetch(e.R, e.ldr, side, pre_r);
#pragma unroll
      for (int t = 0; t < NE; t++) v[t] += side[t];
    }
    if (e.epi == EPI_DGELU) {
      fetch(e.U, e.ldu, side, pre_u);
#pragma unroll
      for (int t = 0; t < NE; t++) v[t] *= side[t];
    }
    if (e.accumulate) {
      fetch(e.C, e.ldc, side, pre_c);
#pragma unroll
      for (int t = 0; t < NE; t++) v[t] += side[t];
    }
    store(e.C, e.ldc, v);
  };
  if constexpr (KS < 8) {
    by_group(take);
    constexpr int NE = NH < 16 ? NH : 16;
#pragma unroll
    for (int u = 0; u < NH / NE; u++) {
      float w[NE];
#pragma unroll
      for (int t = 0; t < NE; t++) w[t] = v[u * NE + t];
      const int first = kg * NH + u * NE;  // of the lane's accumulators
      emit(I<NE>{}, w, m0 + wm + first / 16 / TN * 32 + first % 16 / 4 * 8 + 4 * h, n0 + wn + first / 16 % TN * 32 + l31);
    }
  } else {
#pragma unroll
    for (int t = 0; t < 2; t++) {
      const float* q = smem_f + (wave * 2 + t) * 64 + lane;
      v[t] = ((q[0] + q[1024]) + (q[2048] + q[3072])) + ((q[4096] + q[5120]) + (q[6144] + q[7168]));
    }
    emit(I<2>{}, v, mb8, n0 + l31);
  }
}

template <int WM, int WN, int KS, int TM, int TN, bool TA, bool TB, bool VEC, bool GELU>
__global__ __launch_bounds__(512, 2) void gemm_f32_kernel(int M, int N, int K, const float* __restrict__ A, int lda,
                                                       const float* __restrict__ B, int ldb, EpiArgs e, int tiles_m,
                                                       int tiles_n) {
  f32_product_tile<WM, WN, KS, TM, TN, TA, TB, VEC, GELU>(blockIdx.x, M, N, K, A, lda, B, ldb, e, tiles_m, tiles_n);
}

template <int WM, int WN, int KS, int TM, int TN, bool TA, bool TB, bool GELU>
static constexpr size_t f32_lds() {
  using S = SplitShape<WM, WN, KS, TM, TN>;
  constexpr size_t slabs = 2 * (SplitSlab<S::BM, S::BK, !TA>::BYTES + SplitSlab<S::BN, S::BK, TB>::BYTES);
  constexpr size_t tail = (S::XCH + 8 * S::BN + (GELU ? 8 * 64 * (S::NV / KS < 16 ? S::NV / KS : 16) : 0)) * sizeof(float);
  return slabs > tail && KS < 8 ? slabs : tail;
}

template <int WM, int WN, int KS, int TM, int TN, bool TA, bool TB, bool VEC, bool GELU>
static int launch_f32(const GemmArgs& g, const EpiArgs& e, hipStream_t s) {
  using S = SplitShape<WM, WN, KS, TM, TN>;
  constexpr size_t lds = f32_lds<WM, WN, KS, TM, TN, TA, TB, GELU>();
  auto kern = gemm_f32_kernel<WM, WN, KS, TM, TN, TA, TB, VEC, GELU>;
  static bool configured = false;  // benign race: the attribute is idempotent
  if (!configured) {
    FAX_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    configured = true;
  }
  const int tiles_m = (g.M + S::BM - 1) / S::BM, tiles_n = (g.N + S::BN - 1) / S::BN;
  hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(512), lds, s, g.M, g.N, g.K, (const float*)g.A, g.lda,
                     (const float*)g.B, g.ldb, e, tiles_m, tiles_n);
  FAX_LAUNCH_CHECK("gemm_f32");
  return FAX_OK;
}

template <int WM, int WN, int KS, int TM, int TN, bool VEC>
static int dispatch_f32(const GemmArgs& g, const EpiArgs& e, hipStream_t s) {
  if (g.epi == EPI_GELU) return launch_f32<WM, WN, KS, TM, TN, false, false, VEC, true>(g, e, s);
  if (g.ta) return launch_f32<WM, WN, KS, TM, TN, true, false, VEC, false>(g, e, s);
  if (g.tb) return launch_f32<WM, WN, KS, TM, TN, false, true, VEC, false>(g, e, s);
  return launch_f32<WM, WN, KS, TM, TN, false, false, VEC, false>(g, e, s);
}

template <bool VEC>
static int dispatch_f32_class(int cls, const GemmArgs& g, const EpiArgs& e, hipStream_t s) {
  switch (cls) {
    case 0: return dispatch_f32<2, 2, 2, 2, 2, VEC>(g, e, s);
    case 1: return dispatch_f32<2, 1, 4, 2, 2, VEC>(g, e, s);
    case 2: return dispatch_f32<2, 2, 2, 1, 1, VEC>(g, e, s);
    default: return dispatch_f32<1, 1, 8, 1, 1, VEC>(g, e, s);
  }
}

// Tile class with the smallest predicted time: rounds of one workgroup per CU (workgroups that share a CU take turns on its
// matrix cores), each slabs x slab time + a share of prologue and epilogue.  Measured, us, at 128 x 128, 128 x 64, 64 x 64 and 32 x 32 with its
// K in eighths: 2048 x 4096 x 1024 96, 120, 124, 255; 2048 x 1024 x 4096 150, 103, 123, 215; 1024 x 1024 x 2048 72, 47, 37, 55; 1000 x 640 x
// 640 -, 19, 14, 18; 777 x 512 x 2048 -, 50, 37, 28; 512 x 512 x 512 -, 17, 12, 8.
struct F32Class { int m, n, k; double slab_us, tile_us; };
static constexpr F32Class kF32Classes[] = {{128, 128, 32, 1.35, 4.0}, {128, 64, 64, 1.7, 4.0}, {64, 64, 32, 0.48, 1.5}, {32, 32, 128, 0.85, 1.6}};
static int gemm_f32_class(int M, int N, int K, double* time_us = nullptr) {
  int best = 0;
  double best_t = 1e30;
  for (int c = 0; c < 4; c++) {
    const F32Class& k = kF32Classes[c];
    const long long tiles = (long long)((M + k.m - 1) / k.m) * ((N + k.n - 1) / k.n);
    const double t = (double)((tiles + 255) / 256) * (((K + k.k - 1) / k.k) * k.slab_us + k.tile_us);
    if (t < best_t) { best_t = t; best = c; }
  }
  if (time_us) *time_us = best_t;
  return best;
}
// What a product takes inside a pass: the classes' times are those of one product back to back, with its operands in the caches and
// the clock up.  The four of a forward block of 2048 tokens x 1024 wide: 322 us predicted for them that way, 420 measured in a pass.
double gemm_f32_time_us(int M, int N, int K) {
  double t = 0.0;
  gemm_f32_class(M, N, K, &t);
  return 1.3 * t;
}
void gemm_f32_tile(int M, int N, int K, int* tile_m, int* tile_n) {
  const F32Class& c = kF32Classes[gemm_f32_class(M, N, K)];
  *tile_m = c.m;
  *tile_n = c.n;
}

// What the kernel has no instance for: both operands transposed, GELU other than forward.
bool gemm_f32_supported(const GemmArgs& g) {
  return g.dtype == FAX_F32 && !(g.ta && g.tb) && !(g.epi == EPI_GELU && (g.ta || g.tb)) && !(g.colsum && !g.ta);
}

struct F32Operands {
  EpiArgs e;
  bool vec;
};
static F32Operands f32_operands(const GemmArgs& g) {
  auto vec_ok = [](const void* p, int ld, int extent) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0 && ld % 4 == 0 && extent % 4 == 0 && ld < CHUNK_MAX_LD; };
  const int a_row = g.ta ? g.M : g.K, a_lim = g.a_padded ? (a_row + 3) / 4 * 4 : a_row;  // how far A's rows may be read
  F32Operands o{{g.bias, g.R, g.ldr, g.C, g.ldc, g.C2, g.ldc2, g.U, g.ldu, g.epi, g.gelu_form, 1, g.accumulate ? 1 : 0, g.colsum},
                vec_ok(g.A, g.lda, a_lim) && vec_ok(g.B, g.ldb, g.tb ? g.K : g.N)};
  o.e.a_lim = a_lim;
  return o;
}

int gemm_f32(const GemmArgs& g, hipStream_t s) {
  const F32Operands o = f32_operands(g);
  const int cls = gemm_f32_class(g.M, g.N, g.K);
  return o.vec ? dispatch_f32_class<true>(cls, g, o.e, s) : dispatch_f32_class<false>(cls, g, o.e, s);
}

// A layer's weight gradient and input gradient in one launch: the first workgroups take the tiles of the first, the others those of the
// second, each as it would in a launch of its own (the same bits).
struct F32Product {
  int M, N, K;
  const float* A;
  int lda;
  const float* B;
  int ldb;
  EpiArgs e;
  int tiles_m, tiles_n;
};

// Bound like gemm_f32_kernel; what it saves is a launch's ramp and tail, which are most of a product of one short round.
template <int WKS, int WT, int DKS, int DT>
__global__ __launch_bounds__(512, 2) void gemm_f32_pair_kernel(F32Product w, F32Product d, int first) {
  const int block = blockIdx.x;
  if (block < first)
    f32_product_tile<WT, WT, WKS, 1, 1, true, false, true, false>(block, w.M, w.N, w.K, w.A, w.lda, w.B, w.ldb, w.e, w.tiles_m, w.tiles_n);
  else
    f32_product_tile<DT, DT, DKS, 1, 1, false, true, true, false>(block - first, d.M, d.N, d.K, d.A, d.lda, d.B, d.ldb, d.e, d.tiles_m, d.tiles_n);
}

template <int WKS, int WT, int DKS, int DT>
static int launch_f32_pair(const GemmArgs& wg, const GemmArgs& dg, hipStream_t s) {
  constexpr size_t lw = f32_lds<WT, WT, WKS, 1, 1, true, false, false>(), ld = f32_lds<DT, DT, DKS, 1, 1, false, true, false>(), lds = lw > ld ? lw : ld;
  auto product = [](const GemmArgs& g, int tile) {
    return F32Product{g.M, g.N, g.K, (const float*)g.A, g.lda, (const float*)g.B, g.ldb, f32_operands(g).e, (g.M + tile - 1) / tile, (g.N + tile - 1) / tile};
  };
  const F32Product w = product(wg, 32 * WT), d = product(dg, 32 * DT);
  auto kern = gemm_f32_pair_kernel<WKS, WT, DKS, DT>;
  static bool configured = false;  // benign race: the attribute is idempotent
  if (!configured) {
    FAX_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    configured = true;
  }
  const int first = w.tiles_m * w.tiles_n;
  hipLaunchKernelGGL(kern, dim3(first + d.tiles_m * d.tiles_n), dim3(512), lds, s, w, d, first);
  FAX_LAUNCH_CHECK("gemm_f32_pair");
  return FAX_OK;
}

// For products that take 64 x 64 or 32 x 32 tiles by themselves (larger ones fill the chip alone), operands in whole vectors.
bool gemm_f32_pair_supported(const GemmArgs& w, const GemmArgs& d) {
  auto small = [](const GemmArgs& g) { return gemm_f32_supported(g) && gemm_f32_class(g.M, g.N, g.K) >= 2 && f32_operands(g).vec; };
  return w.ta && !w.tb && w.epi == EPI_NONE && !d.ta && d.tb && (d.epi == EPI_NONE || d.epi == EPI_DGELU) && !d.colsum && small(w) && small(d);
}
int gemm_f32_pair(const GemmArgs& w, const GemmArgs& d, hipStream_t s) {
  const bool w32 = gemm_f32_class(w.M, w.N, w.K) == 3, d32 = gemm_f32_class(d.M, d.N, d.K) == 3;
  if (w32) return d32 ? launch_f32_pair<8, 1, 8, 1>(w, d, s) : launch_f32_pair<8, 1, 2, 2>(w, d, s);
  return d32 ? launch_f32_pair<2, 2, 8, 1>(w, d, s) : launch_f32_pair<2, 2, 2, 2>(w, d, s);
}

}  // namespace fax
