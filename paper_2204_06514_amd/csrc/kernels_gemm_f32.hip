// fp32 GEMM on the CDNA4 matrix cores: v_mfma_f32_32x32x2_f32, which multiplies and adds in fp32 like
// the scalar kernel does, at 256 instead of 128 flop per clock and CU, and with one operand
// register per lane for 4096 flop where a scalar FMA needs two for 2.
//
// A 256-thread workgroup (4 wavefronts) computes a BM x BN tile.  KS = 1: the waves share the tile
// 2 x 2 and step over K in slabs of 32.  KS = 4: every wave computes the whole 32 x 32 tile over its
// own quarter of a 128-wide slab, and the four partial tiles are added up through LDS, in pairs.
// Any M, N, K and orientation: rows and columns beyond the operands are fetched from their last
// row or column and never stored, contraction indices beyond K become zeros on the way into LDS.
//
// The instruction takes 64 clocks, so the fragment reads (1 KB per 256 clocks and wave at a 64 x 64
// wave tile) are far below the LDS's rate and slabs can go through registers: slab s + 1 is requested
// before the products of slab s and stored to the other LDS buffer after them, one barrier per slab.
// An operand whose contraction index is contiguous in memory is kept as [row][k] with rows 4 floats
// longer than a slab: a lane reads four consecutive k's at once, rows l & 31 of a 16-lane
// group at 16 different 16-byte places of the 256-byte bank window.  The other kind is kept as [k][row]
// with rows 8 floats longer: the two halves of a wave read k-rows four apart, 32 banks from each other.
// Which four k's of a group of eight go into one instruction pair (j of the lower half, 4 + j of the
// upper) is the kernel's choice, as long as both operands agree.
//
// Lane layout (lane l): operands = row / column l & 31, k = l >> 5; accumulator v holds element
// [8 (v >> 2) + 4 (l >> 5) + (v & 3)][l & 31]: 32 lanes store 32 consecutive columns.
#include <type_traits>

#include "fax_internal.h"

namespace fax {

typedef __attribute__((ext_vector_type(16))) float f32x16;

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
template <int ROWS, int BK, bool KC, bool VEC>
__device__ __forceinline__ float4 chunk_mask(float4 v, int K, int k0, int c) {
  if (KC) {
    const int left = K - (k0 + c % (BK / 4) * 4);
    return make_float4(left > 0 ? v.x : 0.f, left > (VEC ? 0 : 1) ? v.y : 0.f, left > (VEC ? 0 : 2) ? v.z : 0.f,
                       left > (VEC ? 0 : 3) ? v.w : 0.f);
  }
  return k0 + c / (ROWS / 4) < K ? v : make_float4(0.f, 0.f, 0.f, 0.f);
}
template <int ROWS, int BK, bool KC>
struct F32Slab {
  static constexpr int STRIDE = KC ? BK + 4 : ROWS + 8;
  static constexpr int FLOATS = (KC ? ROWS : BK) * STRIDE;
  static constexpr int CHUNKS = ROWS * BK / 4 / 256;  // per thread
  static __device__ __forceinline__ int place(int c) {
    return KC ? c / (BK / 4) * STRIDE + c % (BK / 4) * 4 : c / (ROWS / 4) * STRIDE + c % (ROWS / 4) * 4;
  }
  // the four k's kb + 4 h + 0..3 of row `row`
  static __device__ __forceinline__ void frag(const float* s, int row, int kb, float (&f)[4]) {
    if (KC) {
      const float4 v = *reinterpret_cast<const float4*>(s + row * STRIDE + kb);
      f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    } else {
#pragma unroll
      for (int j = 0; j < 4; j++) f[j] = s[(kb + j) * STRIDE + row];
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

// Bound by the matrix cores, which sustain 154 TFLOP/s in fp32 on register operands (132 to 136 in the first milliseconds of a run): 2048 x
// 4096 x 1024 runs at 118 (146 us back to back, 173 to 181 inside a block's pass), 2048 x 1024 x 4096 at 99, 4001 x 31003 x 512 at 94.  In the
// block of 2048 tokens x 1024 wide they are busy 64 to 76 % of the clocks of the CUs at work; the rest is waits for the next slab
// and the launch's ramp and tail.  On the scalar kernel that block ran its products at 20 to 60 TFLOP/s.  Requesting slabs two
// ahead instead of one changed nothing (187 us both ways at 2048 x 1024 x 4096) and cost weight gradients 10 %.
// GELU: forward orientation with EPI_GELU, its transcendental code kept out of the other instances.
template <int BM, int BN, int KS, bool TA, bool TB, bool VEC, bool GELU>
__global__ __launch_bounds__(256, 2) void gemm_f32_kernel(int M, int N, int K, const float* __restrict__ A, int lda,
                                                       const float* __restrict__ B, int ldb, EpiArgs e, int tiles_m,
                                                       int tiles_n) {
  constexpr int W = KS == 1 ? 2 : 1;  // waves along M and along N
  static_assert(W * W * KS == 4, "four waves");
  constexpr int TM = BM / W / 32, TN = BN / W / 32, BK = 32 * KS;
  using SA = F32Slab<BM, BK, !TA>;
  using SB = F32Slab<BN, BK, TB>;
  constexpr int BUF = SA::FLOATS + SB::FLOATS;
  extern __shared__ __attribute__((aligned(16))) float smem_f[];

  int tm_i, tn_i;
  f32_tile(blockIdx.x, tiles_m, tiles_n, tm_i, tn_i);
  const int m0 = tm_i * BM, n0 = tn_i * BN;
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l31 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = KS == 1 ? (wave >> 1) * (BM / 2) : 0, wn = KS == 1 ? (wave & 1) * (BN / 2) : 0;
  const int kw = KS == 1 ? 0 : wave * 32;  // this wave's part of a slab

  float4 ra[SA::CHUNKS], rb[SB::CHUNKS];  // the slab on its way from memory to LDS
  auto request = [&](int k0) {
#pragma unroll
    for (int i = 0; i < SA::CHUNKS; i++) ra[i] = chunk_load<BM, BK, !TA, VEC>(A, lda, TA ? e.a_lim : M, TA ? K : e.a_lim, m0, k0, tid + i * 256);
#pragma unroll
    for (int i = 0; i < SB::CHUNKS; i++) rb[i] = chunk_load<BN, BK, TB, VEC>(B, ldb, N, K, n0, k0, tid + i * 256);
  };
  auto publish = [&](int k0, float* buf) {
#pragma unroll
    for (int i = 0; i < SA::CHUNKS; i++)
      *reinterpret_cast<float4*>(buf + SA::place(tid + i * 256)) = chunk_mask<BM, BK, !TA, VEC>(ra[i], K, k0, tid + i * 256);
#pragma unroll
    for (int i = 0; i < SB::CHUNKS; i++)
      *reinterpret_cast<float4*>(buf + SA::FLOATS + SB::place(tid + i * 256)) =
          chunk_mask<BN, BK, TB, VEC>(rb[i], K, k0, tid + i * 256);
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;
  // Optional by-product of the weight-gradient form: colsum[n] (+)= sum over k of B[k, n], from the fragments as they are
  // fed to the matrix core; a slab's sixteen terms first, then the slabs, whose sum carries along what each addition rounds off.
  // 2048 rows of N(0, 1): 0.7e-7 from float64, 1.8e-7 as a plain sum, 1.3e-7 in the separate pass that this stands in for.
  constexpr bool CS = TA && !TB;
  float cs[TN], cs_lost[TN];
#pragma unroll
  for (int j = 0; j < TN; j++) cs[j] = cs_lost[j] = 0.f;

  const int ns = (K + BK - 1) / BK;
  if (ns > 0) {
    request(0);
    publish(0, smem_f);
  }
  __syncthreads();
  for (int s = 0; s < ns; s++) {
    const float* a = smem_f + (s & 1) * BUF;
    const float* b = a + SA::FLOATS;
    if (s + 1 < ns) request((s + 1) * BK);
    float cs1[TN];
#pragma unroll
    for (int j = 0; j < TN; j++) cs1[j] = 0.f;
#pragma unroll
    for (int kb = 0; kb < 32; kb += 8) {
      float fa[TM][4], fb[TN][4];
#pragma unroll
      for (int i = 0; i < TM; i++) SA::frag(a, wm + i * 32 + l31, kw + kb + 4 * h, fa[i]);
#pragma unroll
      for (int j = 0; j < TN; j++) SB::frag(b, wn + j * 32 + l31, kw + kb + 4 * h, fb[j]);
#pragma unroll
      for (int k = 0; k < 4; k++) {
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
          for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][k], fb[j][k], acc[i][j], 0, 0, 0);
      }
      if (CS) {
#pragma unroll
        for (int j = 0; j < TN; j++) cs1[j] += (fb[j][0] + fb[j][1]) + (fb[j][2] + fb[j][3]);
      }
    }
#pragma unroll
    for (int j = 0; j < TN; j++) {
      const float t = cs[j] + cs1[j], was = t - cs1[j];
      cs_lost[j] += (cs[j] - was) + (cs1[j] - (t - was));
      cs[j] = t;
    }
    if (s + 1 < ns) publish((s + 1) * BK, smem_f + ((s + 1) & 1) * BUF);
    __syncthreads();
  }

  if (CS && e.colsum && tm_i == 0) {  // uniform over the workgroup
#pragma unroll
    for (int j = 0; j < TN; j++) {
      if (fabsf(cs[j]) <= 3.4028235e38f) cs[j] += cs_lost[j];  // (of an infinity, what was lost is NaN)
      cs[j] += __shfl_xor(cs[j], 32, 64);
    }
    if (KS > 1) {
      if (lane < 32) smem_f[wave * 32 + lane] = cs[0];
      __syncthreads();
      cs[0] = (smem_f[l31] + smem_f[32 + l31]) + (smem_f[64 + l31] + smem_f[96 + l31]);
      __syncthreads();
    }
    if (lane < 32 && (KS == 1 ? wm == 0 : wave == 0)) {
#pragma unroll
      for (int j = 0; j < TN; j++) {
        const int n = n0 + wn + j * 32 + lane;
        if (n < N) e.colsum[n] = e.accumulate ? e.colsum[n] + cs[j] : cs[j];
      }
    }
  }

  // Epilogue of NE elements of one column n: rows mb + (t & 3) + 8 (t >> 2).  Side inputs are fetched from clamped places
  // (all of them in flight together), stores are predicated.
  auto emit = [&](auto ne_c, float* v, int mb, int n) {
    constexpr int NE = decltype(ne_c)::value;
    const int nr = min(n, N - 1);
    auto row = [&](int t) { return mb + (t & 3) + 8 * (t >> 2); };
    auto fetch = [&](const void* p, int ld, float (&d)[NE]) {
#pragma unroll
      for (int t = 0; t < NE; t++) d[t] = ((const float*)p)[(size_t)min(row(t), M - 1) * ld + nr];
    };
    auto store = [&](void* p, int ld, const float* d) {
#pragma unroll
      for (int t = 0; t < NE; t++)
        if (n < N && row(t) < M) ((float*)p)[(size_t)row(t) * ld + n] = d[t];
    };
    const float bias = e.bias ? ((const float*)e.bias)[nr] : 0.f;
    if (GELU) {
      // one element at a time out of the lane's own LDS slots: sixteen copies of tanh and erf would not fit the instruction cache
      float* slot = smem_f + wave * 64 * NE + lane;
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
      fetch(e.R, e.ldr, side);
#pragma unroll
      for (int t = 0; t < NE; t++) v[t] += side[t];
    }
    if (e.epi == EPI_DGELU) {
      fetch(e.U, e.ldu, side);
#pragma unroll
      for (int t = 0; t < NE; t++) v[t] *= side[t];
    }
    if (e.accumulate) {
      fetch(e.C, e.ldc, side);
#pragma unroll
      for (int t = 0; t < NE; t++) v[t] += side[t];
    }
    store(e.C, e.ldc, v);
  };
  if constexpr (KS == 1) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) {
        float v[16];
#pragma unroll
        for (int t = 0; t < 16; t++) v[t] = acc[i][j][t];
        emit(std::integral_constant<int, 16>{}, v, m0 + wm + i * 32 + 4 * h, n0 + wn + j * 32 + l31);
      }
  } else {
#pragma unroll
    for (int t = 0; t < 16; t++) smem_f[(wave * 16 + t) * 64 + lane] = acc[0][0][t];
    __syncthreads();
    float v[4];
#pragma unroll
    for (int t = 0; t < 4; t++) {
      const float* q = smem_f + (wave * 4 + t) * 64 + lane;
      v[t] = (q[0] + q[1024]) + (q[2048] + q[3072]);
    }
    if (GELU) __syncthreads();  // the slots of the other waves are read before they are used again
    emit(std::integral_constant<int, 4>{}, v, m0 + 8 * wave + 4 * h, n0 + l31);
  }
}

template <int BM, int BN, int KS, bool TA, bool TB, bool VEC, bool GELU>
static int launch_f32(const GemmArgs& g, const EpiArgs& e, hipStream_t s) {
  constexpr int BK = 32 * KS;
  constexpr size_t slabs = 2 * sizeof(float) * (F32Slab<BM, BK, !TA>::FLOATS + F32Slab<BN, BK, TB>::FLOATS);
  constexpr size_t lds = slabs > 16384 ? slabs : 16384;  // the epilogue's exchange: 4 waves x 16 x 64 floats
  auto kern = gemm_f32_kernel<BM, BN, KS, TA, TB, VEC, GELU>;
  static bool configured = false;  // benign race: the attribute is idempotent
  if (!configured) {
    FAX_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    configured = true;
  }
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(256), lds, s, g.M, g.N, g.K, (const float*)g.A, g.lda,
                     (const float*)g.B, g.ldb, e, tiles_m, tiles_n);
  FAX_LAUNCH_CHECK("gemm_f32");
  return FAX_OK;
}

template <int BM, int BN, int KS, bool VEC>
static int dispatch_f32(const GemmArgs& g, const EpiArgs& e, hipStream_t s) {
  if (g.epi == EPI_GELU) return launch_f32<BM, BN, KS, false, false, VEC, true>(g, e, s);
  if (g.ta) return launch_f32<BM, BN, KS, true, false, VEC, false>(g, e, s);
  if (g.tb) return launch_f32<BM, BN, KS, false, true, VEC, false>(g, e, s);
  return launch_f32<BM, BN, KS, false, false, VEC, false>(g, e, s);
}

template <bool VEC>
static int dispatch_f32_class(int cls, const GemmArgs& g, const EpiArgs& e, hipStream_t s) {
  switch (cls) {
    case 0: return dispatch_f32<128, 128, 1, VEC>(g, e, s);
    case 1: return dispatch_f32<128, 64, 1, VEC>(g, e, s);
    case 2: return dispatch_f32<64, 64, 1, VEC>(g, e, s);
    default: return dispatch_f32<32, 32, 4, VEC>(g, e, s);
  }
}

// Tile class with the smallest predicted time: rounds of one workgroup per CU (workgroups that share a CU take turns on its
// matrix cores), each slabs x slab time + a share of prologue and epilogue.  Slab times measured with one or more
// workgroups per CU: 128 x 128 2.4 us, 128 x 64 1.43, 64 x 64 0.73 with several and 0.85 with one, 32 x 32 with its K in
// quarters 0.88 to 1.07 for four times as many k's.  The small tiles fetch more operand bytes per product (64 x 64
// reaches 90-100 TFLOP/s, 32 x 32 65-80) and win where larger ones leave CUs without work: 2048 x 1024 x 1024 95 us at
// 128 x 128, 47 at 128 x 64, 49 at 64 x 64, 60 at 32 x 32; 128 x 128 x 512 42, 24, 16 and under 9.
struct F32Class { int m, n, k; double slab_us, tile_us; };
static constexpr F32Class kF32Classes[] = {{128, 128, 32, 2.40, 3.0}, {128, 64, 32, 1.43, 2.0}, {64, 64, 32, 0.75, 1.5}, {32, 32, 128, 0.95, 1.5}};
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
double gemm_f32_time_us(int M, int N, int K) {
  double t = 0.0;
  gemm_f32_class(M, N, K, &t);
  return t;
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

int gemm_f32(const GemmArgs& g, hipStream_t s) {
  auto vec_ok = [](const void* p, int ld, int extent) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0 && ld % 4 == 0 && extent % 4 == 0; };
  const int a_row = g.ta ? g.M : g.K, a_lim = g.a_padded ? (a_row + 3) / 4 * 4 : a_row;  // how far A's rows may be read
  const bool vec = vec_ok(g.A, g.lda, a_lim) && vec_ok(g.B, g.ldb, g.tb ? g.K : g.N);
  EpiArgs e{g.bias, g.R, g.ldr, g.C, g.ldc, g.C2, g.ldc2, g.U, g.ldu, g.epi, g.gelu_form, 1, g.accumulate ? 1 : 0, g.colsum};
  e.a_lim = a_lim;
  const int cls = gemm_f32_class(g.M, g.N, g.K);
  return vec ? dispatch_f32_class<true>(cls, g, e, s) : dispatch_f32_class<false>(cls, g, e, s);
}

}  // namespace fax
