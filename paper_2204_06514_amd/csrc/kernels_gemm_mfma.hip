// bf16 GEMM on the CDNA4 matrix cores: launch plans (tile class, split contraction, tile walk), the
// choice of kernel flavour and the launches.  The kernel itself is in gemm_mfma_kernel.h.
#include <algorithm>

#include "gemm_mfma_kernel.h"

namespace fax {

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// Tile rows per group of the tile walk (see tile_of in the kernel): the 32 tiles an XCD works on
// at a time form a block of `group` tile rows x 32 / group tile columns.  8 x 4 and 4 x 8 fetch the
// same twelve operand panels; measured inside the benchmark steps, 4 x 8 is the faster one wherever
// the output is wide enough to hold whole blocks of eight columns and the contraction is long
// (d_model 4096 block -0.8 %, the 12288-wide share -2 %, the 2048-wide model -1.2 %, the 1024-wide
// one -1.6 %), and the slower one (+0.3 to 0.5 %) for the 768-wide model with its 3 to 12 tile
// columns and K = 768, which therefore keeps 8 x 4.
// Where both tile counts are multiples of 16 (and the product is not split) the blocks of the eight
// XCDs are laid side by side as well, 4 x 2 of them to a 16 x 16 block of tiles per round (group 0;
// the launch falls back to 4 when it does not run 256 workgroups): the d_model 4096 block another
// -0.4 % (8.065 -> 8.03 ms, A-B on one box), the others unchanged.
int gemm_walk_group(int tiles_m, int tiles_n, int K, int splits) {
  if (K < 1024 || !(tiles_n >= 16 || tiles_n % 8 == 0)) return 8;
  return (splits == 1 && tiles_m % 16 == 0 && tiles_n % 16 == 0) ? 0 : 4;
}

// Both heuristics are written for the 256 CUs of the MI355X.  No device query here on purpose:
// plans decide workspace sizes, and those are computed on hosts without a GPU too (the launch
// itself sizes its grid from the device's own CU count, see launch_mfma).
static constexpr int kCUs = 256;

// Tile classes, largest first, and what a workgroup pays per 64-wide K slab and per
// tile (microseconds, fitted to timings with operands that come from memory, as the previous kernel or the optimizer left them).
// The slab time is given for a full chip (`full_us`) and falls with the share of busy CUs towards `floor_us`: with fewer CUs
// busy the clock is higher (256^2: 1.55 us with all CUs busy, 1.1 with half of them) and each gets more of
// the L2s' bandwidth, which is what bounds the 256 x 128 class on a full chip (13.7 TB/s into LDS
// over all CUs: 0.90 us a slab on 256 CUs, 0.78 on 50).  The smaller the tile, the more LDS
// fragment traffic per flop (4 + 4 fragments per 16 MFMAs at 256^2, 4 + 2 per 8 at 256 x 128,
// 2 + 2 per 4 at 128^2).  Measured and predicted, us, 256 x 192 left out: 3108 x 512 x 2048 40 / 30 / 26 / 17 / 19 in
// that order, predicted 43 / 29 / 24 / 17 / 28; 3000 x 1200 x 4800 86 / 63 / 59 / 61 / 81, predicted 90 / 63 / 53 / 65 / 116.  From the caches the smaller classes gain more, 38 / 23 / 16 / 13
// / 16 and 80 / 53 / 45 / 54 / 70: the prices are those of operands from memory.
struct TileClass {
  int m, n;
  bool deep;  // kernels_gemm_deep.hip: any shape
  double full_us, idle_share, floor_us;  // slab time = max(floor, full * (idle_share + (1 - idle_share) * busy share))
  double epi_bf16_us, epi_f32_us;
};
static constexpr TileClass kTiles[] = {{256, 256, false, 1.55, 0.48, 1.10, 7.0, 8.0},
                                       {256, 192, false, 1.20, 0.40, 0.85, 6.0, 6.0},
                                       {256, 128, false, 0.90, 0.25, 0.78, 4.0, 4.5},
                                       {128, 128, false, 0.66, 1.00, 0.66, 3.0, 3.0},
                                       {128, 64, true, 0.42, 0.85, 0.37, 3.5, 3.5},
                                       {64, 64, true, 0.36, 0.75, 0.28, 3.5, 3.5}};

// Predicted duration of one launch: workgroups run in rounds of one per CU, the last one possibly
// partly filled (a 128^2 launch of at most two per CU runs them side by side, at shared LDS
// bandwidth); folding s partial products costs a launch plus their bytes, written once and read once.
static double tile_time_us(const TileClass& tc, int M, int N, int K, bool f32_out, int s) {
  const int slabs = ((K + GK - 1) / GK + s - 1) / s;
  const long long items = (long long)((M + tc.m - 1) / tc.m) * ((N + tc.n - 1) / tc.n) * s;
  const double epi = f32_out ? tc.epi_f32_us : tc.epi_bf16_us;
  auto round_us = [&](double busy_share) {
    return slabs * std::max(tc.floor_us, tc.full_us * (tc.idle_share + (1.0 - tc.idle_share) * busy_share)) + epi;
  };
  double t;
  if (tc.m == 128 && !tc.deep && items > kCUs && items <= 2 * kCUs && !(f32_out && s > 1)) {
    t = 1.6 * round_us(1.0);
  } else if (tc.m == 64) {  // two workgroups per CU: one's epilogue runs behind the other's products
    const long long rounds = (items + kCUs - 1) / kCUs;
    t = rounds * (round_us(items < kCUs ? (double)items / kCUs : 1.0) - 2.0) + 2.0;
  } else {
    // (weight-gradient products, both operands through the LDS transpose read, gain nothing from a
    // partly filled round: every round at the full-chip price reproduces their measured plans)
    const long long full = items / kCUs, rest = items % kCUs;
    t = full * round_us(1.0) + (rest ? round_us(f32_out ? 1.0 : (double)rest / kCUs) : 0.0);
  }
  if (s > 1) t += 10.0 + (2.0 * s + 1.0) * M * N * 4.0 / 3.0e6;
  return t;
}

// Shapes whose tiles and slabs all come out whole; the others take the masked-edge form of the kernel.
static bool tiles_whole(int M, int N, int K) { return M % 128 == 0 && N % 128 == 0 && K % GK == 0; }

// Tile class (and, when `may_split`, number of K ranges) with the smallest predicted time; a
// smaller tile or a split has to be 3 % better than what is already chosen.  `edge`: the masked-edge
// form, for which every class will do and the padding counts as work; otherwise tile_m = 0 says that
// no class divides the shape.  The 256 x 128 class is used for bf16 outputs only: on weight-gradient
// products (both operands through the LDS transpose read, with or without K ranges) it measured
// 10-50 % above this model.
// The 256 x 192 class: whole tiles with bf16 outputs, where 256^2 tiles leave CUs idle.  It moves a seventh more bytes per flop than
// 256^2 and a seventh fewer than 256 x 128.  One product, us, against the class it takes over from: 16384 x 768 x 3072 64 (73 at 256^2), 16384 x
// 2304 x 768 60 (70), 8192 x 3072 x 3072 124 (135), 4096 x 9216 x 3072 175 (200), 8192 x 2304 x 2304 83 (93 at 256 x 128), 8192 x 1152 x 3456
// 61 (83); nothing or a little the other way 16384 x 1920 x 1920 112 (109), 8192 x 3072 x 768 41.5 (40.6).
// `beside`: another stream's kernels have the CUs that this product leaves idle, so 256^2 stays where it is the best of the others.
// Forward and backward pass against a planner without the class, with that line and with 256 x 192 there as well: 16384 tokens x 768 -1.2 % and
// +0.7 %, 32768 x 768 -1.0 % and +1.2 %, 2048 x 768 -0.7 % and +1.3 %; the other way 4096 x 3072 -1.7 % and -2.4 %.
static GemmSplitPlan plan_tiles(int M, int N, int K, bool f32_out, bool may_split, bool edge, bool deep, bool beside, bool with_192 = true) {
  if (beside && with_192) {
    const GemmSplitPlan p = plan_tiles(M, N, K, f32_out, may_split, edge, deep, beside, false);
    if (p.tile_m == 256 && p.tile_n == 256) return p;
  }
  GemmSplitPlan best{0, 0, 1, false};
  if (M <= 0 || N <= 0 || K <= 0 || (K % GK && !edge)) return best;
  const int nkt = (K + GK - 1) / GK;
  double best_t = 1e30;
  for (const TileClass& tc : kTiles) {
    if (tc.deep ? !deep : (M % tc.m || N % tc.n) && !edge) continue;
    if (f32_out && tc.m != tc.n && !tc.deep) continue;
    if (tc.n == 192 && (edge || !with_192)) continue;
    for (int s = 1; s <= (may_split ? 32 : 1) && (s == 1 || nkt / s >= 8); s++) {
      const double t = tile_time_us(tc, M, N, K, f32_out, s);
      if (t < best_t * 0.97) {
        best_t = t;
        best = GemmSplitPlan{tc.m, tc.n, s, tc.deep};
      }
    }
  }
  // A single slab: the small-tile form's shorter way into and out of its loop decides (512 x 256 x 64 3.8 us at 128 x 128, 2.6 at 64 x 64).
  if (deep && nkt == 1 && best.tile_m == 128 && !best.deep && (long long)((M + 63) / 64) * ((N + 63) / 64) <= kCUs) best = GemmSplitPlan{64, 64, 1, true};
  return best;
}

GemmSplitPlan gemm_split_plan(int M, int N, int K) { return plan_tiles(M, N, K, true, true, !tiles_whole(M, N, K), true, false); }

// One dimension an odd multiple of 128 and the rest big enough to fill the chip with 256^2 tiles:
// the product is computed as two, the bulk on 256^2 tiles and the last 128 rows (1) or columns (2)
// on smaller ones.
static int tail_dim(int M, int N) {
  auto fills = [](int m, int n) { return m > 0 && n > 0 && m % 256 == 0 && n % 256 == 0 && (long long)(m / 256) * (n / 256) >= 2 * kCUs; };
  if (M % 256 == 128 && fills(M - 128, N)) return 1;
  if (N % 256 == 128 && fills(M, N - 128)) return 2;
  return 0;
}

// What gemm_mfma() does with a densely stored product, for inspection from the host: the strip
// decomposition (0, or 1 / 2 = last 128 rows / columns apart) and the plan of the bulk.
GemmSplitPlan gemm_plan_query(int M, int N, int K, bool f32_out, int* tail) {
  const int td = tail_dim(M, N);
  *tail = td;
  const bool deep = tiles_whole(M, N, K);
  if (td == 1) return plan_tiles(M - 128, N, K, f32_out, f32_out, false, deep, false);
  if (td == 2) return plan_tiles(M, N - 128, K, f32_out, false, false, deep, false);  // the strip keeps C's leading dimension: no split
  return plan_tiles(M, N, K, f32_out, f32_out, false, deep, false);
}

// The tile walk of the main launch of a product (not of the 128-wide strip an odd multiple of 128
// leaves over), as a table: tile number -> (tile row, tile column).  For the tests.
int gemm_tile_walk_query(int M, int N, int K, bool f32_out, int* tm, int* tn, int capacity, int* count, int* group) {
  int tail = 0;
  const GemmSplitPlan plan = gemm_plan_query(M, N, K, f32_out, &tail);
  if (plan.tile_m == 0) { *count = 0; *group = -1; return 0; }
  const int tiles_m = (tail == 1 ? M - 128 : M) / plan.tile_m, tiles_n = (tail == 2 ? N - 128 : N) / plan.tile_n;
  int grp = gemm_walk_group(tiles_m, tiles_n, K, plan.splits);
  const int nt = tiles_m * tiles_n;
  const int slots = (plan.tile_m == 128 && nt * plan.splits <= 2 * kCUs) ? 2 * kCUs : kCUs;
  if (grp == 0 && (plan.deep || (nt < slots ? nt : slots) != 256)) grp = 4;  // as launch_mfma and launch_deep decide
  *group = grp; *count = nt;
  for (int id = 0; id < nt && id < capacity; id++) tile_walk(id, tiles_m, tiles_n, grp, tm[id], tn[id]);
  return 0;
}

// partial products, then partial column sums
static size_t split_ws_bytes_1(int M, int N, int K) {
  const int s = gemm_split_plan(M, N, K).splits;
  return s > 1 ? (size_t)s * ((size_t)M * N + N) * sizeof(float) : 0;
}

size_t gemm_split_ws_bytes(int M, int N, int K) {
  if (tiles_whole(M, N, K) && tail_dim(M, N) == 1) return std::max(split_ws_bytes_1(M - 128, N, K), split_ws_bytes_1(128, N, K));
  return split_ws_bytes_1(M, N, K);  // a column strip keeps the leading dimension of C: no split there
}

// A plain bf16 output with few tiles and a very long contraction (the gradient of the hidden states: tokens x width, contracted over
// the vocabulary) is likewise cut into K ranges: fp32 partial products in larger tiles, their sum rounded to bf16 once.  A workgroup
// for every tile of the whole product spends K / 64 slabs one after another, at 25 to 200 workgroups on 256 CUs; the ranges fill them.
// 3108 x 512 x 32003: 189 us as 128 x 64 tiles over all of K, 92 + 15 (fold) as 256 x 256 tiles in 9 ranges.  The line is where the
// predicted times are equal (predicted split / unsplit time; what a whole one-layer training step changes, us): 0.18 128 x 256 x 32000
// 316 -> 206, 0.40 600 x 256 x 16000 271 -> 225, 0.68 6000 x 256 x 32000 1033 -> 922, 0.95 600 x 768 x 6000 342 -> 335, 0.98
// 6000 x 1600 x 32000 4043 -> 3979, 0.99 2048 x 256 x 6000 266 -> 257;  on the other side 1.16 600 x 1600 x 6000 722 -> 724 and
// 6000 x 1600 x 16000 3023 -> 3006, 1.38 600 x 256 x 2500 175 -> 175, 1.45 2048 x 1600 x 6000 1098 -> 1116, 2.6 6000 x 1600 x 2500 2189 -> 2224.
static GemmSplitPlan store_split_plan(int M, int N, int K) {
  const bool edge = !tiles_whole(M, N, K);
  GemmSplitPlan best{0, 0, 1, false};
  double t1 = 1e30;
  for (const TileClass& tc : kTiles)
    if (edge ? tc.n != 192 : tc.deep || !(M % tc.m || N % tc.n)) t1 = std::min(t1, tile_time_us(tc, M, N, K, false, 1));
  double best_t = t1;
  const int nkt = (K + GK - 1) / GK;
  for (const TileClass& tc : kTiles) {
    if (tc.deep || tc.m != tc.n || ((M % tc.m || N % tc.n) && !edge)) continue;
    for (int s = 2; s <= 32 && nkt / s >= 8; s++) {
      const double t = tile_time_us(tc, M, N, K, true, s);
      if (t < best_t) {
        best_t = t;
        best = GemmSplitPlan{tc.m, tc.n, s, false};
      }
    }
  }
  return best;
}
static bool store_split_ok(const GemmArgs& g) {
  return g.store_split && !g.c_f32 && !g.ta && !g.tb && g.epi == EPI_NONE && !g.bias && !g.R && !g.C2 && !g.colsum && g.path == PATH_AUTO &&
         g.ldc == g.N && g.N % 4 == 0 && !g.b_rows;
}
size_t gemm_store_split_ws_bytes(int M, int N, int K) {
  const int s = store_split_plan(M, N, K).splits;
  return s > 1 ? (size_t)s * M * N * sizeof(float) : 0;
}

// What both forms of the kernel ask of a product, apart from its sizes.
static bool mfma_layout_ok(const GemmArgs& g) {
  if (g.dtype != FAX_BF16) return false;
  if (g.c_f32 && (g.bias || g.R || g.C2 || g.epi != EPI_NONE)) return false;  // fp32 C is the plain weight-gradient form
  if (g.colsum && !(g.c_f32 && g.ta && !g.tb)) return false;  // the column sums of B ride only on that form, A [K, M], B [K, N]
  // the GELU epilogues exist for the orientations the block uses them in: forward (A [M,K], B [K,N])
  // and input-gradient (A [M,K], B [N,K])
  if (g.epi == EPI_GELU && (g.ta || g.tb || g.R)) return false;
  if (g.epi == EPI_DGELU && (g.ta || !g.tb || g.R)) return false;
  // the second output likewise: forward orientation only
  if (g.epi == EPI_NONE && g.C2 && (g.ta || g.tb)) return false;
  if (g.M <= 0 || g.N <= 0 || g.K <= 0) return false;
  if (g.lda % 8 || g.ldb % 8 || !aligned16(g.A) || !aligned16(g.B)) return false;
  if (g.c_f32) {  // the epilogue moves four columns at a time: 16-byte fp32 units ...
    if (g.ldc % 4 || !aligned16(g.C)) return false;
  } else {        // ... or 8-byte bf16 units
    auto vec_ok = [](const void* p, int ld) { return !p || (ld % 4 == 0 && (reinterpret_cast<uintptr_t>(p) & 7) == 0); };
    if (!vec_ok(g.C, g.ldc) || !vec_ok(g.C2, g.ldc2) || !vec_ok(g.R, g.ldr) || !vec_ok(g.U, g.ldu) || !vec_ok(g.bias, 4))
      return false;
  }
  return true;
}

// B may have fewer rows than the product has columns (GemmArgs::b_rows): only the masked-edge form stops there.
static bool b_short(const GemmArgs& g) { return g.b_rows && g.b_rows < g.N; }

bool gemm_mfma_supported(const GemmArgs& g) {
  return mfma_layout_ok(g) && tiles_whole(g.M, g.N, g.K) && !b_short(g);  // 128: the smallest tile class
}

// The masked-edge form moves the operands in whole 16-byte chunks and the output in groups of four
// columns, so what is contiguous in memory has to be a multiple of those (the rows of an operand the
// caller has padded may end inside one); the orientations are those of forward, input-gradient and
// weight-gradient products.
bool gemm_edge_supported(const GemmArgs& g) {
  if (!mfma_layout_ok(g) || g.N % 4) return false;
  if (g.c_f32 ? !g.ta || g.tb : g.ta) return false;
  if (g.tb && !g.ta && (g.R || g.C2)) return false;
  const bool a_whole = g.a_padded || (g.ta ? g.M : g.K) % 8 == 0;
  const bool b_whole = (g.tb ? g.K : g.N) % 8 == 0;
  return a_whole && b_whole;
}

template <int BM, int BN>
static int dispatch(const GemmArgs& g, const EpiArgs& e, hipStream_t s) {
  const bool a_kc = !g.ta, b_kc = g.tb;
  const bool erf = g.gelu_form == FAX_GELU_ERF;
  if (g.epi == EPI_GELU && g.value_only)
    return erf ? launch_mfma<BM, BN, true, false, EK_VALUE_ERF>(g, e, s) : launch_mfma<BM, BN, true, false, EK_VALUE_TANH>(g, e, s);
  if (g.epi == EPI_GELU)
    return erf ? launch_mfma<BM, BN, true, false, EK_GELU_ERF>(g, e, s) : launch_mfma<BM, BN, true, false, EK_GELU_TANH>(g, e, s);
  if (g.epi == EPI_DGELU)
    return launch_mfma<BM, BN, true, true, EK_DGELU>(g, e, s);
  if constexpr (BN == 192) {  // bf16 outputs only (plan_tiles)
    if (g.c_f32) {
      set_error("gemm_mfma: no fp32 output on 256 x 192 tiles");
      return FAX_ERR_UNSUPPORTED;
    }
  } else if (g.c_f32 && g.colsum) {
    return g.accumulate ? launch_mfma<BM, BN, false, false, EK_F32 | EM_RES | EM_COLSUM>(g, e, s)
                        : launch_mfma<BM, BN, false, false, EK_F32 | EM_COLSUM>(g, e, s);
  } else if (g.c_f32) {
    if (g.accumulate) {
      if (a_kc && b_kc) return launch_mfma<BM, BN, true, true, EK_F32 | EM_RES>(g, e, s);
      if (a_kc && !b_kc) return launch_mfma<BM, BN, true, false, EK_F32 | EM_RES>(g, e, s);
      if (!a_kc && b_kc) return launch_mfma<BM, BN, false, true, EK_F32 | EM_RES>(g, e, s);
      return launch_mfma<BM, BN, false, false, EK_F32 | EM_RES>(g, e, s);
    }
    if (a_kc && b_kc) return launch_mfma<BM, BN, true, true, EK_F32>(g, e, s);
    if (a_kc && !b_kc) return launch_mfma<BM, BN, true, false, EK_F32>(g, e, s);
    if (!a_kc && b_kc) return launch_mfma<BM, BN, false, true, EK_F32>(g, e, s);
    return launch_mfma<BM, BN, false, false, EK_F32>(g, e, s);
  }
  if (g.C2)  // forward orientation (checked by gemm_mfma_supported)
    return g.R ? launch_mfma<BM, BN, true, false, EK_STORE | EM_RES | EM_C2>(g, e, s)
               : launch_mfma<BM, BN, true, false, EK_STORE | EM_C2>(g, e, s);
  if (g.R) {
    if (a_kc && b_kc) return launch_mfma<BM, BN, true, true, EK_STORE | EM_RES>(g, e, s);
    if (a_kc && !b_kc) return launch_mfma<BM, BN, true, false, EK_STORE | EM_RES>(g, e, s);
    if (!a_kc && b_kc) return launch_mfma<BM, BN, false, true, EK_STORE | EM_RES>(g, e, s);
    return launch_mfma<BM, BN, false, false, EK_STORE | EM_RES>(g, e, s);
  }
  if (a_kc && b_kc) return launch_mfma<BM, BN, true, true, EK_STORE>(g, e, s);
  if (a_kc && !b_kc) return launch_mfma<BM, BN, true, false, EK_STORE>(g, e, s);
  if (!a_kc && b_kc) return launch_mfma<BM, BN, false, true, EK_STORE>(g, e, s);
  return launch_mfma<BM, BN, false, false, EK_STORE>(g, e, s);
}

static const void* offset(const void* p, size_t elements, size_t elem_bytes) {
  return p ? (const char*)p + elements * elem_bytes : nullptr;
}
static void* offset(void* p, size_t elements, size_t elem_bytes) { return p ? (char*)p + elements * elem_bytes : nullptr; }

static EpiArgs epi_args(const GemmArgs& g, const GemmSplitPlan& plan) {
  return EpiArgs{g.bias, g.R, g.ldr, g.C, g.ldc, g.C2, g.ldc2, g.U, g.ldu, g.epi, g.gelu_form, g.c_f32 ? 1 : 0,
                 g.accumulate ? 1 : 0, g.colsum, plan.splits, (size_t)g.M * g.N, (size_t)g.N,
                 gemm_walk_group((g.M + plan.tile_m - 1) / plan.tile_m, (g.N + plan.tile_n - 1) / plan.tile_n, g.K, plan.splits),
                 g.ta ? (g.M + 7) / 8 * 8 : g.M, g.b_rows ? g.b_rows : g.N};
}

// The plan gemm_mfma() would launch, if that is the small-tile form in one launch.
static bool deep_alone(const GemmArgs& g, GemmSplitPlan* plan) {
  if (g.path != PATH_AUTO || !gemm_edge_supported(g)) return false;
  const bool edge = !tiles_whole(g.M, g.N, g.K) || b_short(g);
  if (!edge && tail_dim(g.M, g.N)) return false;
  *plan = plan_tiles(g.M, g.N, g.K, g.c_f32, g.c_f32 && g.split_ws && g.ldc == g.N, edge, true, g.beside);
  return plan->deep && plan->splits == 1;
}

// Launch included; with scratch for a split where the form may have one.
// small: whether (the bulk of) it takes the small-tile form.
static double mfma_time_us(const GemmArgs& g, bool* small) {
  *small = false;
  const bool edge = !tiles_whole(g.M, g.N, g.K) || b_short(g);
  if (store_split_ok(g) && gemm_edge_supported(g)) {
    const GemmSplitPlan plan = store_split_plan(g.M, g.N, g.K);
    for (const TileClass& tc : kTiles)
      if (plan.splits > 1 && tc.m == plan.tile_m && tc.n == plan.tile_n && !tc.deep) return 3.0 + tile_time_us(tc, g.M, g.N, g.K, true, plan.splits);
  }
  auto one = [&](int M, int N, bool bulk) {
    const GemmSplitPlan plan = plan_tiles(M, N, g.K, g.c_f32, g.c_f32 && g.ldc == N, edge, gemm_edge_supported(g), g.beside);
    if (bulk) *small = plan.deep;
    for (const TileClass& tc : kTiles)
      if (tc.m == plan.tile_m && tc.n == plan.tile_n && tc.deep == plan.deep) return 3.0 + tile_time_us(tc, M, N, g.K, g.c_f32, plan.splits);
    return 0.0;
  };
  switch (edge ? 0 : tail_dim(g.M, g.N)) {
    case 1: return one(g.M - 128, g.N, true) + one(128, g.N, false);
    case 2: return one(g.M, g.N - 128, true) + one(g.M, 128, false);
  }
  return one(g.M, g.N, true);
}
double gemm_mfma_time_us(const GemmArgs& g) {
  bool small;
  return mfma_time_us(g, &small);
}
// Of a product with 16-bit outputs in tiles of one class, without the launch.
double gemm_tiles_us(int tile_m, int tile_n, int M, int N, int K) {
  for (const TileClass& tc : kTiles)
    if (tc.m == tile_m && tc.n == tile_n) return tile_time_us(tc, M, N, K, false, 1);
  return 0.0;
}

// The pair takes one launch where both products take the small-tile form by themselves, undivided (in fp32: 64 x 64 or 32 x 32 tiles): those
// leave CUs idle or last little longer than a launch.  The results are the same bits.  (Larger tiles fill the chip alone.)  And where the 64 x 64 tiles
// of both are no more than a round together and so take less than the launches that each would have by itself: forward and backward pass of
// 41 tokens x 64 89 -> 69 us, of 415 x 64 95 -> 85.  Not where the weight gradient would have K ranges: 4096 x 64 123, 145 in pairs.
static bool pair_plan(const GemmArgs& w, const GemmArgs& d, GemmSplitPlan* wp, GemmSplitPlan* dp) {
  if (!(w.c_f32 && w.ta && !w.tb && w.colsum && !d.c_f32 && !d.ta && d.tb && !d.C2 && !d.R && !d.bias && (d.epi == EPI_NONE || d.epi == EPI_DGELU)))
    return false;
  if (deep_alone(w, wp) && deep_alone(d, dp)) return true;
  if (w.path != PATH_AUTO || d.path != PATH_AUTO || !gemm_edge_supported(w) || !gemm_edge_supported(d)) return false;
  const TileClass& tc = kTiles[sizeof(kTiles) / sizeof(kTiles[0]) - 1];
  auto tiles = [&](const GemmArgs& g) { return (long long)((g.M + tc.m - 1) / tc.m) * ((g.N + tc.n - 1) / tc.n); };
  if (tiles(w) + tiles(d) > kCUs || gemm_route(w, w.split_ws != nullptr).splits > 1) return false;
  auto us = [&](const GemmArgs& g) { return tile_time_us(tc, g.M, g.N, g.K, g.c_f32, 1); };
  *wp = *dp = GemmSplitPlan{tc.m, tc.n, 1, true};
  return 3.0 + std::max(us(w), us(d)) < 0.95 * (gemm_mfma_time_us(w) + gemm_mfma_time_us(d));
}
bool gemm_pair_supported(const GemmArgs& w, const GemmArgs& d) {
  if (w.dtype == FAX_F32) return d.dtype == FAX_F32 && gemm_f32_pair_supported(w, d);
  GemmSplitPlan wp, dp;
  return pair_plan(w, d, &wp, &dp);
}

int gemm_pair(const GemmArgs& w, const GemmArgs& d, hipStream_t s) {
  if (w.dtype == FAX_F32) {
    if (!gemm_pair_supported(w, d)) {
      set_error("gemm_pair: not two fp32 products of small tiles");
      return FAX_ERR_UNSUPPORTED;
    }
    Timed t("gemm_f32_pair", WORK_FLOP, 2.0 * w.M * w.N * w.K + 2.0 * d.M * d.N * d.K, s);
    return gemm_f32_pair(w, d, s);
  }
  GemmSplitPlan wp, dp;
  if (!pair_plan(w, d, &wp, &dp)) {
    set_error("gemm_pair: not two products of the small-tile form");
    return FAX_ERR_UNSUPPORTED;
  }
  Timed t("gemm_mfma_pair", WORK_FLOP, 2.0 * w.M * w.N * w.K + 2.0 * d.M * d.N * d.K, s);
  return gemm_mfma_deep_pair(w, epi_args(w, wp), wp, d, epi_args(d, dp), dp, s);
}

// Weight gradients of one layer in one launch, whose tiles share the rounds: by themselves each ends in a partly filled one, takes tiles
// too small for it, or cuts its contraction and folds.  The class with the smaller predicted time.
struct GroupPlan { int tile; bool edge; double us; };
static bool group_plan(const GemmArgs* g, int n, GroupPlan* plan) {
  if (n < 1 || n > GEMM_GROUP) return false;
  for (int i = 0; i < n; i++)
    if (g[i].path != PATH_AUTO || !gemm_edge_supported(g[i]) || !g[i].c_f32 || !g[i].colsum || g[i].K != g[0].K || g[i].accumulate != g[0].accumulate)
      return false;
  plan->us = 1e30;
  for (const TileClass& tc : kTiles) {
    if (tc.m != tc.n || tc.deep) continue;
    long long items = 0;
    bool cut = g[0].K % GK != 0;
    for (int i = 0; i < n; i++) {
      items += (long long)((g[i].M + tc.m - 1) / tc.m) * ((g[i].N + tc.n - 1) / tc.n);
      cut = cut || g[i].M % tc.m || g[i].N % tc.n;
    }
    const double round = (g[0].K + GK - 1) / GK * tc.full_us + tc.epi_f32_us;
    const double t = 3.0 + (tc.m == 128 && items > kCUs && items <= 2 * kCUs ? 1.6 * round : (double)((items + kCUs - 1) / kCUs) * round);
    if (t < plan->us) *plan = GroupPlan{tc.m, cut, t};
  }
  return true;
}

// Weight gradients and an input gradient in one launch: as many workgroups for the former as share their tiles in no more rounds than the whole
// chip would; the latter has the others, in tiles 256 or 128 columns wide, if it is through by then.  On two streams each keeps to its CUs as
// well: weight gradients on all 256 leave the input gradient none before their last round.  Several rounds, us, forward and backward, tokens x width x heads' width
// x F: the two one after the other, the input gradient alone confined, both confined: 8192 x 1920 x 960 x 7680 1963, 2020, 1912; 15872 x 3456 x 640 x
// 10880 7245, 8290, 7154; 12800 x 2176 x 1408 x 8704 4016, 4285, 3909; 17920 x 896 x 896 x 12544 3062, 3020, 3023.  On one stream, one after the other
// and in one launch: the first 1978 and 1945, the last 3104 and 3076.
struct GroupInputPlan { int rounds, first, blocks, tile_n; bool edge; };
static bool group_input_plan(const GemmArgs* g, int n, const GemmArgs& d, GroupInputPlan* plan) {
  GroupPlan gp;
  if (!group_plan(g, n, &gp) || gp.tile != 256) return false;
  if (d.path != PATH_AUTO || !gemm_edge_supported(d) || d.ta || !d.tb || d.c_f32 || d.epi != EPI_NONE || d.bias || d.R || d.C2 || d.colsum || b_short(d))
    return false;
  int items = 0;
  for (int i = 0; i < n; i++) items += ((g[i].M + 255) / 256) * ((g[i].N + 255) / 256);
  plan->rounds = (items + kCUs - 1) / kCUs;
  plan->first = ((items + plan->rounds - 1) / plan->rounds + 7) / 8 * 8;  // a multiple of the XCDs, which the tile walk deals in
  const int left = kCUs - plan->first;
  if (left <= 0) return false;
  double best = 1e30;
  for (const TileClass& tc : kTiles) {
    if (tc.m != 256 || tc.n == 192) continue;
    const long long tiles = (long long)((d.M + 255) / 256) * ((d.N + tc.n - 1) / tc.n);
    const double t = (double)((tiles + left - 1) / left) * ((d.K + GK - 1) / GK * tc.full_us + tc.epi_bf16_us);
    if (t < best) {
      best = t;
      plan->tile_n = tc.n;
      plan->blocks = (int)std::min<long long>(tiles, left);
    }
  }
  plan->edge = gp.edge || !tiles_whole(d.M, d.N, d.K) || d.M % 256 || d.N % plan->tile_n;
  if (items < plan->first) plan->first = items;  // (one round)
  return best < gp.us;
}
bool gemm_group_input_supported(const GemmArgs* w, int n, const GemmArgs& d) {
  GroupInputPlan plan;
  return group_input_plan(w, n, d, &plan);
}
bool gemm_group_input_pays(const GemmArgs* w, int n, const GemmArgs& d, double* group_us) {
  GroupInputPlan plan;
  GroupPlan gp;
  if (!group_input_plan(w, n, d, &plan) || plan.rounds != 1 || !group_plan(w, n, &gp)) return false;
  *group_us = gp.us;
  return true;
}
int gemm_group_input(const GemmArgs* w, int n, const GemmArgs& d, GroupPart part, hipStream_t s) {
  GroupInputPlan plan;
  if (!group_input_plan(w, n, d, &plan)) {
    set_error("gemm_group_input: not products for one launch");
    return FAX_ERR_UNSUPPORTED;
  }
  EpiArgs e[GEMM_GROUP];
  double work = part == PART_WEIGHTS ? 0.0 : 2.0 * d.M * d.N * d.K;
  for (int i = 0; i < n; i++) {
    e[i] = epi_args(w[i], GemmSplitPlan{256, 256, 1, false});
    if (part != PART_INPUT) work += 2.0 * w[i].M * w[i].N * w[i].K;
  }
  if (part == PART_INPUT) plan.first = 0;
  if (part == PART_WEIGHTS) plan.blocks = 0;
  Timed t(part == PART_INPUT ? "gemm_mfma_group_input" : "gemm_mfma_group", WORK_FLOP, work, s);
  return gemm_mfma_group_input(w, n, e, plan.first, plan.blocks, d, epi_args(d, GemmSplitPlan{256, plan.tile_n, 1, false}), plan.tile_n, plan.edge, s);
}

// The lines, with the block's forward and backward pass (us, tokens x width, F = 4 x width) before and after:
// All four: 256^2 tiles, input gradients of at least a round of 256 x 128 tiles each, and 30 % less predicted time than apart.  8192 x 1024 980 -> 904
//   (the feed-forward's two and attention's two by themselves 970); where the input gradients leave CUs idle the other way round, 3108 x 512
//   271 -> 285, 16384 x 512 684 -> 766, 2048 x 5120 in an eighth's share 695 -> 728.
// The feed-forward's two: any gain predicted for whole tiles, a quarter for masked edges (whose small tiles by themselves run 30 % over the
//   model beside other kernels).  3108 x 512 271 -> 253, 4500 x 640 465 -> 438, 3000 x 1200 654 -> 626, 4096 x 1024 470 -> 460; 4200 x 968,
//   beyond the line, 676 and 691.  Not in 128^2 tiles where each alone fills whole rounds of 256^2 ones, which load half as much: apart and
//   together, with attention's two apart, 14336 x 1024 1387 and 1444, 16384 x 1024 1527 and 1593, 24576 x 1024 2216 and 2369, 32768 x 1024
//   2861 and 2867; where they leave CUs idle 12288 x 768 925 and 910, 16384 x 768 1040 and 1037.
//   Within the line and slower 6000 x 3072 with F 6144, 2017 and 2069, where 5000, 8000 and 10000 rows of it are within 0.3 %.
// Attention's two: at 128^2 tiles, and not much longer than the QKV one alone (the other one would start before the attention kernels and run
//   beside them).  4096 x 1024 470 -> 449, 2222 x 1280 563 -> 552, 4096 x 768 380 -> 372; beyond the line 3108 x 512 271 and 277, 1999 x
//   2000 843 and 854, 3600 x 1536 908 and 915.  With the feed-forward's two apart, apart and together: 2500 x 968 472 and 458, 3500 x 768 406 and
//   392, 3000 x 1024 491 and 485, 4000 x 968 699 and 691, 5000 x 800 652 and 639; the other way 2500 x 768 318 and 325, and around 4200 to 4560 rows
//   960 to 1024 wide up to 1 % where attention is a split form, whose workgroups leave no room beside them, and 2 to 3.5 % against apart beside
//   the unsplit one (66 heads of 700 x 88 688 and 700, of 760 x 88 730 and 757): each choice alone is within 1 % there, and no size tells them from 4000 x 968.
//   Nor longer than 92 us by itself: the output projection's share of it, the longer the more, would have run beside the attention kernels.
//   Apart and together, 1024 wide: 6144 708 and 696, 7168 780 and 782, 8000 921 and 924, 8448 920 and 956, 9000 1129 and 1165, 10240 1060 and
//   1079, 12288 1192 and 1243, 14336 1409 and 1513, 20480 1998 and 2108; 9000 x 968 1136 and 1179, 9216 x 1280 1283 and 1301, 6144 x 1280 942 and 940.
int gemm_groups(const GemmArgs (&w)[4], const GemmArgs (&in)[4]) {
  bool pairs = true, full = true;
  for (int i = 0; i < 4; i++) {
    const GemmArgs& g = in[i];
    if (!gemm_edge_supported(g)) return 0;
    pairs = pairs && gemm_pair_supported(i < 2 ? w[i] : w[5 - i], g);  // with the weight gradient of this layer
    if (!full) continue;
    const GemmSplitPlan p = plan_tiles(g.M, g.N, g.K, false, false, !tiles_whole(g.M, g.N, g.K), true, g.beside);
    full = p.tile_m == 256 && (long long)((g.M + 255) / 256) * ((g.N + p.tile_n - 1) / p.tile_n) >= kCUs;
  }
  if (pairs) return 0;  // short products: one launch for a layer's weight and input gradient instead
  GroupPlan all, ffn, att;
  if (!group_plan(w, 4, &all)) return 0;
  group_plan(w, 2, &ffn);
  group_plan(w + 2, 2, &att);
  double apart[4];
  for (int i = 0; i < 4; i++) {
    bool small;
    apart[i] = mfma_time_us(w[i], &small);
    if (i == 2 && !(att.us < 1.45 * apart[2])) att.tile = 0;
    if (small) apart[i] *= 1.3;
  }
  if (full && all.tile == 256 && all.us < 0.7 * (apart[0] + apart[1] + apart[2] + apart[3])) return GROUP_ALL;
  const bool filled = ffn.tile == 128 && gemm_fill(w[0]).rounds && gemm_fill(w[1]).rounds;
  return (!filled && ffn.us < (ffn.edge ? 0.76 : 0.97) * (apart[0] + apart[1]) ? GROUP_FFN : 0) |
         (att.tile == 128 && att.us < 92.0 && att.us < 0.97 * (apart[2] + apart[3]) ? GROUP_ATTENTION : 0);
}

int gemm_group(const GemmArgs* g, int n, hipStream_t s) {
  GroupPlan plan;
  if (!group_plan(g, n, &plan)) {
    set_error("gemm_group: not products for one launch");
    return FAX_ERR_UNSUPPORTED;
  }
  EpiArgs e[GEMM_GROUP];
  double work = 0.0;
  for (int i = 0; i < n; i++) {
    e[i] = epi_args(g[i], GemmSplitPlan{plan.tile, plan.tile, 1, false});
    work += 2.0 * g[i].M * g[i].N * g[i].K;
  }
  Timed t("gemm_mfma_group", WORK_FLOP, work, s);
  return gemm_mfma_group(g, n, e, plan.tile, plan.edge, s);
}

GemmRoute gemm_route(const GemmArgs& g, bool scratch) {
  GemmRoute r{gemm_form(g), false, 0, 0, 0, 1, 0, 0, -1};
  if (r.form == GEMM_F32) gemm_f32_tile(g.M, g.N, g.K, &r.tile_m, &r.tile_n);
  if (r.form != GEMM_MFMA && r.form != GEMM_EDGE) return r;
  if (scratch && store_split_ok(g) && gemm_edge_supported(g)) {
    const GemmSplitPlan p = store_split_plan(g.M, g.N, g.K);
    if (p.splits > 1) return GemmRoute{r.form, false, 0, p.tile_m, p.tile_n, p.splits, (g.M + p.tile_m - 1) / p.tile_m, (g.N + p.tile_n - 1) / p.tile_n,
                                       gemm_walk_group((g.M + p.tile_m - 1) / p.tile_m, (g.N + p.tile_n - 1) / p.tile_n, g.K, p.splits)};
  }
  const bool edge = r.form == GEMM_EDGE;
  r.tail = edge ? 0 : tail_dim(g.M, g.N);
  const int M = r.tail == 1 ? g.M - 128 : g.M, N = r.tail == 2 ? g.N - 128 : g.N;
  const GemmSplitPlan p = plan_tiles(M, N, g.K, g.c_f32, g.c_f32 && scratch && g.ldc == N, edge, gemm_edge_supported(g), g.beside);
  r.small = p.deep; r.tile_m = p.tile_m; r.tile_n = p.tile_n; r.splits = p.splits;
  r.tiles_m = (M + p.tile_m - 1) / p.tile_m;
  r.tiles_n = (N + p.tile_n - 1) / p.tile_n;
  r.group = gemm_walk_group(r.tiles_m, r.tiles_n, g.K, p.splits);
  const int nt = r.tiles_m * r.tiles_n, slots = (p.tile_m == 128 && nt * p.splits <= 2 * kCUs) ? 2 * kCUs : kCUs;
  if (r.group == 0 && (p.deep || std::min(nt * p.splits, slots) != 256)) r.group = 4;  // as launch_mfma and launch_deep decide
  return r;
}

GemmFill gemm_fill(const GemmArgs& g) {
  const GemmRoute r = gemm_route(g, true);
  if (r.form != GEMM_MFMA && r.form != GEMM_EDGE) return GemmFill{1.0, false};
  const long long items = (long long)r.tiles_m * r.tiles_n * r.splits;
  const long long slots = r.tile_m == 128 && !r.small && items > kCUs && items <= 2 * kCUs ? 2 * kCUs : kCUs;
  const long long rounds = (items + slots - 1) / slots;
  return GemmFill{std::max(1.0 - (double)items / (double)(rounds * slots), r.tail ? 0.05 : 0.0), !r.tail && r.tile_m == 256 && items % kCUs == 0};
}

void gemm_route_tile(const GemmRoute& r, int item, int* tile_row, int* tile_col) {
  tile_walk(item, r.tiles_m, r.tiles_n, r.group, *tile_row, *tile_col);
}

int gemm_mfma(const GemmArgs& g0, hipStream_t s) {
  const bool edge = !tiles_whole(g0.M, g0.N, g0.K) || b_short(g0);
  if (store_split_ok(g0) && g0.split_ws && gemm_edge_supported(g0)) {
    const GemmSplitPlan plan = store_split_plan(g0.M, g0.N, g0.K);
    if (plan.splits > 1) {
      GemmArgs g = g0;
      g.c_f32 = true;
      g.C = g0.split_ws;
      const EpiArgs e = epi_args(g, plan);
      if (edge) FAX_TRY(gemm_mfma_edge(g, e, plan, s));
      else if (plan.tile_n == 256) FAX_TRY((dispatch<256, 256>(g, e, s)));
      else FAX_TRY((dispatch<128, 128>(g, e, s)));
      return fold_partials_bf16(plan.splits, (size_t)g.M * g.N, (const float*)g0.split_ws, g0.C, s);
    }
  }
  if (const int td = edge ? 0 : tail_dim(g0.M, g0.N)) {
    const size_t cb = g0.c_f32 ? 4 : 2;
    for (int part = 0; part < 2; part++) {
      GemmArgs h = g0;
      if (td == 1) {  // rows [m0, m0 + M')
        const size_t m0 = part ? g0.M - 128 : 0;
        h.M = part ? 128 : g0.M - 128;
        h.A = offset(g0.A, g0.ta ? m0 : m0 * g0.lda, 2);
        h.C = offset(g0.C, m0 * g0.ldc, cb);
        h.R = offset(g0.R, m0 * g0.ldr, 2);
        h.C2 = offset(g0.C2, m0 * g0.ldc2, 2);
        h.U = offset(g0.U, m0 * g0.ldu, 2);
        if (part) h.colsum = nullptr;  // the column sums of B are complete after the first product
      } else {        // columns [n0, n0 + N')
        const size_t n0 = part ? g0.N - 128 : 0;
        h.N = part ? 128 : g0.N - 128;
        h.B = offset(g0.B, g0.tb ? n0 * g0.ldb : n0, 2);
        h.C = offset(g0.C, n0, cb);
        h.bias = offset(g0.bias, n0, 2);
        h.R = offset(g0.R, n0, 2);
        h.C2 = offset(g0.C2, n0, 2);
        h.U = offset(g0.U, n0, 2);
        if (g0.colsum) h.colsum = g0.colsum + n0;
      }
      FAX_TRY(gemm_mfma(h, s));  // (neither part has a tail of its own)
    }
    return FAX_OK;
  }
  GemmArgs g = g0;
  // Split the contraction?  Only the fp32-output form, with scratch from the caller and C stored
  // densely; the partial products (and partial column sums) are then folded in a fixed order.
  const GemmSplitPlan plan = plan_tiles(g.M, g.N, g.K, g.c_f32, g.c_f32 && g.split_ws && g.ldc == g.N, edge,
                                        gemm_edge_supported(g), g.beside);
  if (plan.tile_m == 0) {
    set_error("gemm_mfma: %d x %d x %d fits no tile class", g.M, g.N, g.K);
    return FAX_ERR_UNSUPPORTED;
  }
  const int splits = plan.splits;
  const size_t mn = (size_t)g.M * g.N;
  float* const part_c = (float*)g.split_ws;
  float* const part_cs = part_c + (size_t)splits * mn;
  if (splits > 1) {
    g.C = part_c;
    if (g.colsum) g.colsum = part_cs;
    g.accumulate = false;
  }
  const EpiArgs e = epi_args(g, plan);
  if (plan.deep) FAX_TRY(gemm_mfma_deep(g, e, plan, s));
  else if (edge) FAX_TRY(gemm_mfma_edge(g, e, plan, s));
  else if (plan.tile_n == 256) FAX_TRY((dispatch<256, 256>(g, e, s)));
  else if (plan.tile_n == 192) FAX_TRY((dispatch<256, 192>(g, e, s)));
  else if (plan.tile_m == 256) FAX_TRY((dispatch<256, 128>(g, e, s)));
  else FAX_TRY((dispatch<128, 128>(g, e, s)));
  if (splits > 1) {
    FAX_TRY(fold_partials(splits, mn, part_c, (float*)g0.C, g0.accumulate, s, g0.colsum ? g.N : 0, part_cs, g0.colsum));
  }
  return FAX_OK;
}

}  // namespace fax
