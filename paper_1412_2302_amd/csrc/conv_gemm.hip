// Convolution forward, backward-data and backward-weight as implicit GEMMs, and the dense layers, on three cores: fp32
// operands on the bf16 matrix cores (gemm_split.h: pointwise, first and dense layers that can be read 16 bytes at a
// time), fp32 matrix instructions (gemm.h: everything else in fp32) and bf16 operands (gemm_bf16.h, gemm16.h, gemm_direct.h).
#include <algorithm>

#include "fc_epilogue.h"
#include "gemm16.h"
#include "gemm_direct.h"
#include "kernels.h"

namespace ax {

constexpr int kBK = 16;  // depth of a k-tile
typedef Tile<128, 128, kBK, 2, 2> T128;  // wave tile 64 x 64
typedef Tile<128, 96, kBK, 4, 1> T96;    // wave tile 32 x 96
typedef Tile<128, 64, kBK, 4, 1> T64;    // wave tile 32 x 64
// 48 columns out of 16x16x4 blocks (wave tile 32 x 48), k-tile 32; only with the whole-tile loaders
constexpr int kBK48 = 32;
typedef Tile<128, 48, kBK48, 4, 1, 16> T48;
// (256 x 128 and 256 x 96 tiles were measured too: their 128 accumulator
// registers leave one wave per SIMD, and with nobody to cover barrier and LDS
// latency they ran 8-12 % slower than 128 x 128 on every AlexNet layer.)

// ------------------------------------------------------------ tile + split-k ---
// A launch is as slow as its busiest compute unit.  With few output tiles (338
// for a 21632 x 256 output at 128 x 128) a third of the chip idles while the
// rest runs a second tile, so the reduction can be cut into `ns` slices whose
// partial tiles go to slabs and are added by a finishing kernel in a fixed
// order.  Larger tiles spend fewer non-MFMA instructions per MFMA but make
// that quantisation worse.  plan_gemm() prices every (tile, ns) pair with a
// small model -- rounds of tiles over 256 compute units at the tile's measured
// MFMA efficiency, padded columns, slab traffic -- and takes the cheapest.
struct GemmPlan {
  int bm, bn, ns, kchunk;
};
// what the second launch of a product in slices costs besides its traffic: the small nets' 15 us products are better
// sliced than whole (346 against 357 us a step with the price at 6 us); between 2 and 6 us every larger pass, fp32 or
// bf16, stays within 0.3 %
constexpr double kSecondLaunch = 4e-6;
struct TileOption {
  int bm, bn, bk;
  double eff;  // fraction of the per-CU fp32 MFMA rate this tile reaches on a long reduction
};
static const TileOption kTileOptions[] = {{128, 128, kBK, 0.80}, {128, 96, kBK, 0.68}, {128, 64, kBK, 0.62},
                                          {128, 48, kBK48, 0.60}};
// bf16 MFMA tiles: k-tile of 32; no longer MFMA-bound, priced at ~4x the fp32 rate
constexpr int kBKbf = 32;
typedef Tile<128, 128, kBKbf, 2, 2> B128;
typedef Tile<128, 64, kBKbf, 4, 1> B64;
// 256 x 128 (wave tile 128 x 64): three fragment reads for every four MFMAs instead of four for four -- these
// kernels are paced by LDS, not by the matrix cores; only with operands stored as bf16 (half the staging registers)
typedef Tile<256, 128, kBKbf, 2, 2> B256;
// 256 x 96 (wave tile 64 x 96) for the first layer's 96 output channels, which the 128-wide tiles pad by a third
typedef Tile<256, 96, kBKbf, 4, 1> B256n96;
static const TileOption kTileOptionsBf[] = {{128, 128, kBKbf, 3.2}, {128, 64, kBKbf, 2.2}, {256, 128, kBKbf, 4.2}};

// precision of the GEMMs launched by the calling thread: 0 fp32 operands, 1 operands rounded to bf16; fp32 accumulation
static thread_local int g_bf16 = 0;
void set_gemm_precision(int bf16) { g_bf16 = bf16 ? 1 : 0; }

static GemmPlan plan_gemm(int M, int N, int K, int groups, double out_bytes, int max_s, bool bf = false,
                          bool allow48 = false, int max_chunk = 0, bool allow256 = false, double* t_out = nullptr) {
  const TileOption* opts = bf ? kTileOptionsBf : kTileOptions;
  const int nopts = bf ? (allow256 ? 3 : 2) : (allow48 ? 4 : 3);
  GemmPlan best{128, 128, 1, ceil_div(K, opts[0].bk) * opts[0].bk};
  double best_t = 1e30;
  for (int o = 0; o < nopts; ++o) {
    const TileOption& to = opts[o];
    const int bk = to.bk, ktiles = ceil_div(K, bk);
    const long tiles = (long)ceil_div(M, to.bm) * ceil_div(N, to.bn) * groups;
    const double t_tile = 2.0 * to.bm * to.bn * (double)ktiles * bk / (0.614e12 * to.eff);
    for (int s = 1; s <= max_s && s <= ktiles; ++s) {
      const int per = ceil_div(ktiles, s);
      if (ceil_div(ktiles, per) != s) continue;
      if (s > 1 && per * bk < 96) break;
      if (max_chunk && per * bk > max_chunk) continue;  // the workgroup's k range must fit its pixel table
      const double rounds = (double)ceil_div(tiles * s, 256);
      double t = rounds * t_tile * per / ktiles + 4e-6;
      if (s > 1) t += (s + 1) * out_bytes / 2.5e12 + kSecondLaunch;
      if (t < best_t * 0.98) {  // prefer earlier (larger, unsplit) candidates unless clearly better
        best_t = t;
        best = GemmPlan{to.bm, to.bn, s, per * bk};
      }
    }
  }
  if (t_out) *t_out = best_t;
  return best;
}

// Algorithmic flops of the launch being prepared (2 x multiply-adds of the
// operation, not of the padded GEMM); 0 means "use 2*M*N*K".
static thread_local double g_algo_flops = 0;
// Algorithmic bytes of the same launch: every operand tensor read once and the result written once (for a
// convolution the activation tensor itself, not its im2col expansion); 0 means "(M*K + K*N + M*N) floats".
static thread_local double g_algo_bytes = 0;
struct AlgoFlops {
  explicit AlgoFlops(double f, double b = 0) { g_algo_flops = f; g_algo_bytes = b; }
  ~AlgoFlops() { g_algo_flops = 0; g_algo_bytes = 0; }
};
static inline double conv_flops(const ConvGeom& c) { return 2.0 * c.P() * c.Cout * c.cg() * c.k * c.k; }
static inline double conv_bytes(const ConvGeom& c) {
  return 4.0 * ((double)c.in_elems() + (double)c.w_elems() + (double)c.out_elems());
}
static inline double gemm_bytes(int M, int N, int K, int groups) {
  return g_algo_bytes > 0 ? g_algo_bytes : 4.0 * groups * ((double)M * K + (double)K * N + (double)M * N);
}

template <class T, class AL, class BL, class Epi>
static int launch_tile(const typename AL::Params& ap, const typename BL::Params& bp, const Epi& ep, int M, int N, int K,
                       int kchunk, int nsplit, int groups, hipStream_t st, size_t dyn_lds = 0) {
  if (M <= 0 || N <= 0) return ALEXNET_OK;
  dim3 grid(ceil_div(M, T::BM), ceil_div(N, T::BN), groups * nsplit);
  if (grid.y > 65535 || grid.z > 65535) {
    set_error("GEMM grid too large (%u,%u,%u)", grid.x, grid.y, grid.z);
    return ALEXNET_ESHAPE;
  }
  KernelScope ks("gemm", g_algo_flops > 0 ? g_algo_flops : 2.0 * M * N * (double)K * groups,
                 gemm_bytes(M, N, K, groups), st);
  hipLaunchKernelGGL((gemm_kernel<T, AL, BL, Epi>), grid, dim3(kThreads), dyn_lds, st, ap, bp, ep, M, N, K, kchunk,
                     nsplit);
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}

template <class T, class AL, class BL, class Epi>
static int launch_tile_bf(const typename AL::Params& ap, const typename BL::Params& bp, const Epi& ep, int M, int N,
                          int K, int kchunk, int nsplit, int groups, hipStream_t st, size_t dyn_lds = 0) {
  if (M <= 0 || N <= 0) return ALEXNET_OK;
  // one-dimensional launch: the kernel deals the tiles to the XCDs itself (xcd_tile)
  const int gx = ceil_div(M, T::BM), gy = ceil_div(N, T::BN), gz = groups * nsplit;
  const long total = (long)gx * gy * gz;
  if (total > 0x7fffffffL) {
    set_error("GEMM grid too large (%d,%d,%d)", gx, gy, gz);
    return ALEXNET_ESHAPE;
  }
  KernelScope ks("gemm_bf16", g_algo_flops > 0 ? g_algo_flops : 2.0 * M * N * (double)K * groups,
                 gemm_bytes(M, N, K, groups), st);
  hipLaunchKernelGGL((gemm_bf16_kernel<T, AL, BL, Epi>), dim3((unsigned)total), dim3(kThreads), dyn_lds, st, ap, bp, ep,
                     M, N, K, kchunk, nsplit, gx, gy);
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}

static inline int round_up(int v, int m) { return (v + m - 1) / m * m; }

// One struct per GEMM flavour: names the loaders for a tile and a pair of
// vector/scalar choices, so that the dispatch below stays a table.
template <int MODE>
struct ConvGather {  // rows = pixels (forward, backward-data)
  template <class T, bool AV, bool BV, class Epi>
  static int go(const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d, int kchunk, int ns,
                hipStream_t st) {
    return launch_tile<T, Im2colKInner<T::BM, T::BK, AV, MODE>, DenseRowInner<T::BN, T::BK, BV>, Epi>(
        a, b, e, d.M, d.N, d.K, kchunk, ns, d.groups, st);
  }
};
struct ConvWeightGrad {  // rows = taps (backward-weight)
  template <class T, bool AV, bool BV, class Epi>
  static int go(const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d, int kchunk, int ns,
                hipStream_t st) {
    return launch_tile<T, Im2colRowInner<T::BM, T::BK, AV>, DenseRowInner<T::BN, T::BK, BV>, Epi>(
        a, b, e, d.M, d.N, d.K, kchunk, ns, d.groups, st);
  }
};

// backward-weight with the pixel table in LDS (see Im2colRowTable): 16-byte loads, whole k-tiles
struct ConvWeightGradTable {
  template <class T, class Epi>
  static int go(const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d, int kchunk, int ns,
                hipStream_t st) {
    return launch_tile<T, Im2colRowTable<T::BM, T::BK>, DenseRowWhole<T::BN, T::BK>, Epi>(
        a, b, e, d.M, d.N, d.K, kchunk, ns, d.groups, st, (size_t)std::min(kchunk, d.K) * sizeof(PixelEntry));
  }
};
static inline bool table_ok(const Im2colParams& a, const GemmDims& d) {
  return a.kh * a.kw <= 31 && d.K % kBK == 0;
}

// a k-tile inside one tap (see Im2colKTap): 16-byte loads, whole k-tiles
template <int MODE>
struct ConvGatherTap {
  template <class T, class Epi>
  static int go(const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d, int kchunk, int ns,
                hipStream_t st) {
    return launch_tile<T, Im2colKTap<T::BM, T::BK, MODE>, DenseRowWhole<T::BN, T::BK>, Epi>(
        a, b, e, d.M, d.N, d.K, kchunk, ns, d.groups, st);
  }
};
static inline bool tap_ok(const Im2colParams& a, const GemmDims& d, int bk = kBK) {
  return a.Cg % bk == 0 && a.kh * a.kw <= 32 && d.K % bk == 0;
}

// bf16 flavours (vector loads only)
template <int MODE>
struct ConvGatherBf {
  template <class T, class Epi>
  static int go(const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d, int kchunk, int ns,
                hipStream_t st) {
    return launch_tile_bf<T, BfRowMajor<Im2colKInner<T::BM, T::BK, true, MODE>, T::BM, T::BK>,
                          BfDenseRowInner<T::BN, T::BK>, Epi>(a, b, e, d.M, d.N, d.K, kchunk, ns, d.groups, st);
  }
};
struct ConvWeightGradBf {
  template <class T, class Epi>
  static int go(const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d, int kchunk, int ns,
                hipStream_t st) {
    return launch_tile_bf<T, BfIm2colRowInner<T::BM, T::BK>, BfDenseRowInner<T::BN, T::BK>, Epi>(
        a, b, e, d.M, d.N, d.K, kchunk, ns, d.groups, st);
  }
};
// bf16 with the uniform-tap / whole-tile / pixel-table loaders
template <int MODE>
struct ConvGatherTapBf {
  template <class T, class Epi>
  static int go(const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d, int kchunk, int ns,
                hipStream_t st) {
    return launch_tile_bf<T, BfRowMajor<Im2colKTap<T::BM, T::BK, MODE>, T::BM, T::BK>, BfDenseRowWhole<T::BN, T::BK>,
                          Epi>(a, b, e, d.M, d.N, d.K, kchunk, ns, d.groups, st);
  }
};
struct ConvWeightGradTableBf {
  template <class T, class Epi>
  static int go(const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d, int kchunk, int ns,
                hipStream_t st) {
    return launch_tile_bf<T, BfIm2colRowTable<T::BM, T::BK>, BfDenseRowWhole<T::BN, T::BK>, Epi>(
        a, b, e, d.M, d.N, d.K, kchunk, ns, d.groups, st, (size_t)std::min(kchunk, d.K) * sizeof(PixelEntry));
  }
};
// bf16 MFMA over operands that are stored as bf16 (gemm_bf16.h, "16" loaders)
template <int MODE>
struct ConvGather16 {
  template <class T, class Epi>
  static int go(const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d, int kchunk, int ns,
                hipStream_t st) {
    return launch_tile_bf<T, Im2colKInner16<T::BM, T::BK, MODE>, DenseKInner16<T::BN, T::BK>, Epi>(
        a, b, e, d.M, d.N, d.K, kchunk, ns, d.groups, st);
  }
};
template <int MODE>
struct ConvGatherTap16 {
  template <class T, class Epi>
  static int go(const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d, int kchunk, int ns,
                hipStream_t st) {
    return launch_tile_bf<T, Im2colKTap16<T::BM, T::BK, MODE>, DenseKInner16<T::BN, T::BK>, Epi>(
        a, b, e, d.M, d.N, d.K, kchunk, ns, d.groups, st);
  }
};
// 192 columns per group and enough 128 x 192 tiles for two workgroups per CU (at batch 64, 172 tiles, the 128 x 64 tile of
// gemm_bf16.h is the faster one, 33 against 38 us; at batch 256, 676 tiles, 83 against 107)
typedef Tile<128, 192, kBKbf, 2, 2> B192;
static bool tile192_ok(const GemmDims& d) {
  return d.N % 192 == 0 && d.N % 128 != 0 && (long)ceil_div(d.M, 128) * (d.N / 192) * d.groups >= 512;
}
template <int MODE, class Epi>
static int launch_tile192(const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d, hipStream_t st) {
  typedef Unit16<Im2colKTap16<128, kBKbf, MODE>, 128, kBKbf> AL;
  typedef Unit16<DenseKInner16<192, kBKbf>, 192, kBKbf> BL;
  const int gx = ceil_div(d.M, 128), gy = d.N / 192;
  KernelScope ks("gemm_bf16", g_algo_flops > 0 ? g_algo_flops : 2.0 * d.M * d.N * (double)d.K * d.groups,
                 gemm_bytes(d.M, d.N, d.K, d.groups), st);
  hipLaunchKernelGGL((gemm16_kernel<B192, AL, BL, Epi>), dim3((unsigned)(gx * gy * d.groups)), dim3(kThreads), 0, st, a, b,
                     e, d.M, d.N, d.K, make_fastdiv((uint32_t)gx), make_fastdiv((uint32_t)gy));
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}
// ---- operands straight to LDS (gemm_direct.h) ----
// Workgroups on the busiest compute unit run in rounds of as many as it holds; a round of n takes first[n-1] + each[n-1] * the
// megaflops of a tile microseconds.  Fitted to (tile, workgroups, MFLOP a tile, us): 128 x 64: 2028 37.7 97.8, 2028 28.3 81.8,
// 510 37.7 29.1, 510 18.9 19.1, 132 28.3 18, 132 37.7 24.1, 128 56.6 29.2, 66 18.9 12; 128 x 128: 1014 75.5 87.8, 676 56.6 59.5,
// 255 75.5 31.8, 170 56.6 24.6, 340 56.6 33.1; 192 x 128: 452 169.9 82.3, 452 84.9 49.6, 171 113 39.2, 114 84.9 31.3.
// Slices only where 128 x 64 tiles leave compute units without one (the sums move 4 to 6 TB/s; third layer, 258 tiles and more,
// forward of 37 pictures 26 us either way, data gradient of 64 31 whole, 34 in slices).
struct DirectTile {
  int bm, bn, occ;
  double first[3], each[3];
};
static const DirectTile kDirectTiles[] = {{128, 64, 3, {5, 9.1, 12.2}, {0.46, 0.53, 0.585}},
                                          {128, 128, 2, {3, 8, 0}, {0.38, 0.476, 0}},
                                          {192, 128, 2, {7.5, 17, 0}, {0.28, 0.385, 0}}};
struct DirectPlan {
  int tile, ns, per;  // per: k-tiles of a slice
};
static DirectPlan plan_direct(const GemmDims& d, double out_bytes, double* t_out = nullptr) {
  DirectPlan best{0, 1, ceil_div(d.K, kBKd)};
  double best_t = 1e30;
  const int ktiles = ceil_div(d.K, kBKd);
  const int most = (long)ceil_div(d.M, 128) * ceil_div(d.N, 64) * d.groups > 256 ? 1 : 8;
  for (int o = 0; o < 3; ++o) {
    const DirectTile& to = kDirectTiles[o];
    const long tiles = (long)ceil_div(d.M, to.bm) * ceil_div(d.N, to.bn) * d.groups;
    for (int s = 1; s <= most && s <= ktiles; ++s) {
      const int per = ceil_div(ktiles, s);
      if (ceil_div(ktiles, per) != s || (s > 1 && per < 4)) continue;
      const int c = ceil_div(tiles * s, 256), rest = c % to.occ;
      const double f = 2e-6 * to.bm * to.bn * (double)per * kBKd;
      double t = c / to.occ * (to.first[to.occ - 1] + to.each[to.occ - 1] * f);
      if (rest) t += to.first[rest - 1] + to.each[rest - 1] * f;
      t *= 1e-6;
      if (s > 1) t += (s + 1) * out_bytes / 6e12 + kSecondLaunch;
      if (t < 0.98 * best_t) {
        best_t = t;
        best = DirectPlan{o, s, per};
      }
    }
  }
  if (t_out) *t_out = best_t + 2e-6;
  return best;
}
// Channels per group that are no multiple of 64 cost instructions for every k-tile: there the tiles of gemm_bf16.h have to be
// a fifth slower by their planner (measured on the second layer, 48 channels, whose forward product has a kernel of its own now,
// patch_conv.hip: at batch 256 six full rounds of 256-row tiles stayed; at 37, 100 and 128 three rounds, the last one part
// empty, inference 374 and 610 us, training 1943, went to 360, 586, 1917).
static bool direct_pays(const GemmDims& d, int Cg, int taps, double out_bytes) {
  if (taps > kDirectTaps) return false;
  if (Cg % kBKd == 0) return true;
  double direct, tiles;
  plan_direct(d, out_bytes, &direct);
  plan_gemm(d.M, d.N, d.K, d.groups, out_bytes, 8, true, false, 0, d.N % 128 == 0, &tiles);
  return 1.2 * direct < tiles;
}
static bool direct_fwd_ok(const ConvGeom& c) {
  const GemmDims d = fwd_dims(c);
  return conv_bf16_stored_ok(c) && !(c.cg() % kBKbf == 0 && tile192_ok(d)) &&
         direct_pays(d, c.cg(), c.k * c.k, (double)c.out_elems() * 4);
}
static bool direct_bwd_data_ok(const ConvGeom& c) {
  return conv_bf16_stored_ok(c) && direct_pays(bwdd_dims(c), c.og(), c.k * c.k, (double)c.in_elems() * 4);
}
template <int BM, int BN, int WM, int WN, int MINB, int MODE, class Epi>
static int launch_direct_tile(const DirectPlan& p, const Im2colParams& a, const DenseParams& b, const Epi& e,
                              const GemmDims& d, hipStream_t st) {
  DirectJob j;
  j.a = a;
  j.b = b;
  j.M = d.M;
  j.N = d.N;
  j.K = d.K;
  j.tiles_per_slice = p.per;
  const int gx = ceil_div(d.M, BM), gy = ceil_div(d.N, BN);
  j.gx = make_fastdiv((uint32_t)gx);
  j.gy = make_fastdiv((uint32_t)gy);
  j.ns = make_fastdiv((uint32_t)p.ns);
  KernelScope ks("gemm_bf16", g_algo_flops > 0 ? g_algo_flops : 2.0 * d.M * d.N * (double)d.K * d.groups,
                 gemm_bytes(d.M, d.N, d.K, d.groups), st);
  const dim3 grid((unsigned)((long)gx * gy * d.groups * p.ns));
  if (a.Cg % kBKd == 0)
    hipLaunchKernelGGL((gemm_direct_kernel<BM, BN, WM, WN, MINB, true, MODE, Epi>), grid, dim3(kThreads), 0, st, j, e);
  else
    hipLaunchKernelGGL((gemm_direct_kernel<BM, BN, WM, WN, MINB, false, MODE, Epi>), grid, dim3(kThreads), 0, st, j, e);
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}
template <int MODE, class Epi>
static int launch_direct(const DirectPlan& p, const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d,
                         hipStream_t st) {
  if (p.tile == 0) return launch_direct_tile<128, 64, 4, 1, 3, MODE, Epi>(p, a, b, e, d, st);
  if (p.tile == 1) return launch_direct_tile<128, 128, 2, 2, 2, MODE, Epi>(p, a, b, e, d, st);
  return launch_direct_tile<192, 128, 2, 2, 2, MODE, Epi>(p, a, b, e, d, st);
}
template <class F, class Epi>
static int by_tile_16(const GemmPlan& p, const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d,
                      hipStream_t st) {
  if (p.bm == 256) return F::template go<B256, Epi>(a, b, e, d, p.kchunk, p.ns, st);
  if (p.bn == 128) return F::template go<B128, Epi>(a, b, e, d, p.kchunk, p.ns, st);
  return F::template go<B64, Epi>(a, b, e, d, p.kchunk, p.ns, st);
}
template <class F, class Epi>
static int by_tile_bf(const GemmPlan& p, const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d,
                      hipStream_t st) {
  if (p.bn == 128) return F::template go<B128, Epi>(a, b, e, d, p.kchunk, p.ns, st);
  return F::template go<B64, Epi>(a, b, e, d, p.kchunk, p.ns, st);
}

// vector loads on both operands, on B only, or on neither
template <class F, class T, class Epi>
static int by_vec(bool av, bool bv, const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d,
                  int kchunk, int ns, hipStream_t st) {
  if (av && bv) return F::template go<T, true, true, Epi>(a, b, e, d, kchunk, ns, st);
  if (bv) return F::template go<T, false, true, Epi>(a, b, e, d, kchunk, ns, st);
  return F::template go<T, false, false, Epi>(a, b, e, d, kchunk, ns, st);
}
template <class F, class Epi>
static int by_tile(const GemmPlan& p, bool av, bool bv, const Im2colParams& a, const DenseParams& b, const Epi& e,
                   const GemmDims& d, hipStream_t st) {
  if (p.bn == 128) return by_vec<F, T128, Epi>(av, bv, a, b, e, d, p.kchunk, p.ns, st);
  if (p.bn == 96) return by_vec<F, T96, Epi>(av, bv, a, b, e, d, p.kchunk, p.ns, st);
  return by_vec<F, T64, Epi>(av, bv, a, b, e, d, p.kchunk, p.ns, st);
}

// out[m][g*N + n] = post(sum_s ws[(g*ns + s)][m][n]); post = +bias, ReLU, or gate by a forward activation
__global__ void slab_finish_kernel(const float* __restrict__ ws, int ns, int groups, long M, int N,
                                   const float* __restrict__ bias, int relu, const float* __restrict__ gate,
                                   float* __restrict__ out) {
  const size_t total = (size_t)M * groups * N;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;  // index into out
  if (i >= total) return;
  const int col = (int)(i % ((size_t)groups * N));
  const size_t m = i / ((size_t)groups * N);
  const int g = col / N, n = col - g * N;
  const size_t slab = (size_t)M * N;
  const float* p = ws + (size_t)g * ns * slab + m * N + n;
  float v = 0.f;
#pragma unroll 8
  for (int k = 0; k < ns; ++k) v += p[(size_t)k * slab];  // loads in flight together, added in order
  if (bias) v += bias[col];
  if (relu) v = v > 0.f ? v : 0.f;
  if (gate && !(gate[i] > 0.f)) v = 0.f;
  out[i] = v;
}
int launch_slab_finish(const float* ws, int ns, int groups, long M, int N, const float* bias, int relu,
                              const float* gate, float* out, hipStream_t st) {
  const size_t total = (size_t)M * groups * N;
  KernelScope ks("slab_finish", 0, (double)total * 4.0 * (ns + 1 + (gate ? 1 : 0)), st);
  hipLaunchKernelGGL(slab_finish_kernel, dim3(ceil_div(total, 256)), dim3(256), 0, st, ws, ns, groups, M, N, bias,
                     relu, gate, out);
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}

// ----------------------------------------- fp32 products on the bf16 matrix cores ---
// (gemm_split.h)  Dense operands, 16-byte loads.
typedef Tile<128, 128, kBKs, 2, 2> S128;
typedef Tile<128, 96, kBKs, 4, 1> S96;
typedef Tile<128, 64, kBKs, 2, 2> S64;
typedef Tile<64, 128, kBKs, 2, 2> S64m;
// rate of a tile on a long reduction over the fp32 matrix rate of a compute unit, measured at 4096 x 4608 x 2048
// (147, 140, 125 and 127 TFLOP/s; the fp32 kernels reach 101 there)
static const TileOption kTileOptionsSplit[] = {
    {128, 128, kBKs, 0.94}, {128, 96, kBKs, 0.89}, {128, 64, kBKs, 0.80},
    {64, 128, kBKs, 0.81}};  // the last one for dense layers on at most 64 rows, where a 128-row tile is half empty
// Cheapest (tile, slices) for a launch of the split kernel, as plan_gemm(), with one difference: these kernels fetch
// one k-tile ahead only, and a workgroup that has its compute unit to itself waits for memory about half the time (a
// weight gradient of 192 x 128 x 2048 x 72: 105 us in 216 workgroups, see fill), so slices are worth having until two
// or three workgroups share every unit.
// rows (may be null): each of the 36 positions has its own number of rows.
static GemmPlan plan_split(int M, int N, int K, int groups, double out_bytes, int max_s, double* t_out = nullptr,
                           bool allow64 = false, const TileRows* rows = nullptr) {
  GemmPlan best{128, 128, 1, ceil_div(K, kBKs) * kBKs};
  double best_t = 1e30;
  const int ktiles = ceil_div(K, kBKs);
  for (const TileOption& to : kTileOptionsSplit) {
    if (to.bm == 64 && !allow64) continue;
    long row_tiles = (long)ceil_div(M, to.bm) * groups;
    if (rows) {
      row_tiles = 0;
      for (int p = 0; p < 36; ++p) {
        const RowRange r = wino_rows(p, rows->short_y, rows->whole, rows->short_x, rows->tiles);
        row_tiles += (long)ceil_div(r.hi - r.lo, to.bm) * (groups / 36);
      }
    }
    const long tiles = row_tiles * ceil_div(N, to.bn);
    const double t_tile = 2.0 * to.bm * to.bn * (double)ktiles * kBKs / (0.614e12 * to.eff);
    for (int s = 1; s <= max_s && s <= ktiles; ++s) {
      const int per = ceil_div(ktiles, s);
      if (ceil_div(ktiles, per) != s) continue;
      if (s > 1 && per * kBKs < 96) break;
      // workgroups per unit: of the launch, at once (see SplitMinBlocks)
      const int c = ceil_div(tiles * s, 256), most = to.bm * to.bn < 128 * 128 ? 3 : 2;
      if (s > 1 && c > 4 * most) break;  // more slices only add traffic
      const double fill = c >= most ? 1.0 : c == 2 ? 0.85 : 0.5;
      // positions with few rows leave room early: half way between the busiest unit and the average (37 to 128 pictures, third
      // to fifth layer, three tiles each: the best of them, or within 7 %; by the busiest unit up to 38 % over it)
      const double share = rows ? 0.5 * (c + tiles * s / 256.0) : c;
      double t = share * t_tile * per / ktiles / fill + 4e-6;
      if (s > 1) t += (s + 1) * out_bytes / 2.5e12 + kSecondLaunch;
      if (t < best_t * 0.98) {
        best_t = t;
        best = GemmPlan{to.bm, to.bn, s, per * kBKs};
      }
    }
  }
  if (t_out) *t_out = best_t;
  return best;
}
template <class T, class AL, class BL, class Epi>
static int launch_tile_split(const typename AL::Params& ap, const typename BL::Params& bp, const Epi& ep, int M, int N,
                             int K, int kchunk, int nsplit, int groups, hipStream_t st, const TileRows* rows = nullptr,
                             int of = 0) {
  if (M <= 0 || N <= 0) return ALEXNET_OK;
  const int gx = ceil_div(M, T::BM), gy = ceil_div(N, T::BN), gz = groups * nsplit;
  const long total = (long)gx * gy * gz;
  if (total > 0x7fffffffL) {
    set_error("GEMM grid too large (%d,%d,%d)", gx, gy, gz);
    return ALEXNET_ESHAPE;
  }
  SplitGrid grid{make_fastdiv((uint32_t)gx), make_fastdiv((uint32_t)gy), make_fastdiv((uint32_t)nsplit), 0, {}, 0, 0, 0, 0};
  if (rows) {
    grid.of = of;
    grid.positions = make_fastdiv((uint32_t)(groups / 36));
    grid.short_y = rows->short_y; grid.whole = rows->whole; grid.short_x = rows->short_x; grid.tiles = rows->tiles;
  }
  KernelScope ks("gemm", g_algo_flops > 0 ? g_algo_flops : 2.0 * M * N * (double)K * groups,
                 gemm_bytes(M, N, K, groups), st);
  hipLaunchKernelGGL((gemm_split_kernel<T, AL, BL, Epi>), dim3((unsigned)total), dim3(kThreads), 0, st, ap, bp, ep, M,
                     N, K, kchunk, grid);
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}
// ALT / BLT: loaders by number of rows
template <template <int> class ALT, template <int> class BLT, class Epi>
static int by_tile_split(const GemmPlan& p, const DenseParams& a, const DenseParams& b, const Epi& e, int M, int N, int K,
                         int groups, hipStream_t st, const TileRows* rows = nullptr, int of = 0) {
#define AX_SPLIT(T) \
  return launch_tile_split<T, ALT<T::BM>, BLT<T::BN>, Epi>(a, b, e, M, N, K, p.kchunk, p.ns, groups, st, rows, of)
  if (p.bm == 64) AX_SPLIT(S64m);
  if (p.bn == 96) AX_SPLIT(S96);
  if (p.bn == 64) AX_SPLIT(S64);
  AX_SPLIT(S128);
#undef AX_SPLIT
}
// The first layer in run mode: a k-tile passes at most one run's end and one row's end of the loaders SplitRun and
// SplitRunT.
static inline bool split_run_ok(const ConvGeom& c) { return run_mode(c) && run_len(c) >= kBKs && c.Wo >= kBKs && c.Cout % 4 == 0; }
static GemmPlan split_run_fwd_plan(const ConvGeom& c, double* t_out = nullptr) {
  return plan_split((int)c.P(), c.Cout, run_k(c), 1, (double)c.out_elems() * 4, 8, t_out);
}
static GemmPlan split_run_bwdw_plan(const ConvGeom& c, double* t_out = nullptr) {
  return plan_split(c.k * c.k * c.Cin, c.Cout, (int)c.P(), 1, (double)c.w_elems() * 4, 256, t_out);
}
// A of either product by tile, B = packed weights or output gradient
template <template <int> class ALT, class AP, class Epi>
static int by_tile_run(const GemmPlan& p, const AP& a, const DenseParams& b, const Epi& e, int M, int N, int K,
                       hipStream_t st) {
#define AX_SPLIT(T) \
  return launch_tile_split<T, ALT<T::BM>, SplitRowInner<T::BN>, Epi>(a, b, e, M, N, K, p.kchunk, p.ns, 1, st)
  if (p.bn == 96) AX_SPLIT(S96);
  if (p.bn == 64) AX_SPLIT(S64);
  AX_SPLIT(S128);
#undef AX_SPLIT
}
// A pointwise convolution (the products of a transformed layer among them) is a dense product per group.
static inline bool pointwise(const ConvGeom& c) { return c.k == 1 && c.stride == 1 && c.pad == 0; }
static inline DenseParams pointwise_A(const ConvGeom& c, const float* x) {
  return DenseParams{x, c.Cin, c.cg(), (int)c.P(), (uint32_t)(c.in_elems() * 4)};
}
static inline bool split_fwd_ok(const ConvGeom& c) {
  return pointwise(c) && c.cg() % 4 == 0 && c.og() % 4 == 0 && c.cg() >= kSplitMinK;
}
static inline bool split_bwdw_ok(const ConvGeom& c) {
  return pointwise(c) && c.cg() % 4 == 0 && c.og() % 4 == 0 && c.P() >= kSplitMinK;
}
static GemmPlan split_fwd_plan(const ConvGeom& c, double* t_out = nullptr, const TileRows* rows = nullptr) {
  const GemmDims d = fwd_dims(c);
  return plan_split(d.M, d.N, d.K, d.groups, (double)c.out_elems() * 4, 8, t_out, false, rows);
}
// weight gradient: the operands may change places, whichever way the tiles cover the result with less padding
static GemmPlan split_bwdw_plan(const ConvGeom& c, bool* swapped, double* t_out = nullptr) {
  const GemmDims d = bwdw_dims(c);
  double t[2];
  const GemmPlan p = plan_split(d.M, d.N, d.K, d.groups, (double)c.w_elems() * 4, 256, &t[0]);
  const GemmPlan q = plan_split(d.N, d.M, d.K, d.groups, (double)c.w_elems() * 4, 256, &t[1]);
  *swapped = t[1] < 0.98 * t[0];
  if (t_out) *t_out = t[*swapped];
  return *swapped ? q : p;
}

bool conv_products_split(const ConvGeom& c) {
  return split_fwd_ok(c) && split_bwdw_ok(c) && !wave_conv_fwd_ok(c, false) && !wave_conv_bwd_weight_ok(c, false);
}

// ------------------------------------------------------------- convolution ---
template <class F, class Epi>
static int by_tile_tap(const GemmPlan& p, const Im2colParams& a, const DenseParams& b, const Epi& e,
                       const GemmDims& d, hipStream_t st) {
  if (p.bn == 128) return F::template go<T128, Epi>(a, b, e, d, p.kchunk, p.ns, st);
  if (p.bn == 96) return F::template go<T96, Epi>(a, b, e, d, p.kchunk, p.ns, st);
  if (p.bn == 48) return F::template go<T48, Epi>(a, b, e, d, p.kchunk, p.ns, st);
  return F::template go<T64, Epi>(a, b, e, d, p.kchunk, p.ns, st);
}

// t48: the 48-column tile may be used (its loaders need a k-tile of 32 inside one tap)
static GemmPlan run16_fwd_plan(const ConvGeom& c, double* t_out = nullptr);
// t256: the 256-row tile may be used (bf16-stored operands)
static GemmPlan fwd_plan(const ConvGeom& c, bool run, bool bf, bool t48 = false, bool t256 = false,
                         double* t_out = nullptr) {
  const GemmDims d = fwd_dims(c);
  return plan_gemm(d.M, d.N, run ? run_k(c) : d.K, d.groups, (double)c.out_elems() * 4, 8, bf, t48, 0, t256, t_out);
}
static GemmPlan bwdd_plan(const ConvGeom& c, bool bf, bool t48 = false, bool t256 = false, double* t_out = nullptr) {
  const GemmDims d = bwdd_dims(c);
  return plan_gemm(d.M, d.N, d.K, d.groups, (double)c.in_elems() * 4, 8, bf, t48, 0, t256, t_out);
}
static GemmPlan bwdw_plan(const ConvGeom& c, bool run, bool bf, bool table = false, double* t_out = nullptr) {
  const GemmDims d = bwdw_dims(c);
  return plan_gemm(run ? run_k(c) : d.M, d.N, d.K, d.groups, (double)(run ? run_w_elems(c) : c.w_elems()) * 4, 256,
                   bf, false, table ? kMaxTableK : 0, false, t_out);
}
// What a product takes in tiles, by the planners of this file.  bf: forward products and data gradients over stored operands
// where there are such kernels; weight gradients and dense layers over fp32 ones.
double tile_seconds_fwd(const ConvGeom& c, bool bf) {
  double t = 0;
  if (bf && run16_mode(c))
    run16_fwd_plan(c, &t);
  else if (bf && direct_fwd_ok(c))
    plan_direct(fwd_dims(c), (double)c.out_elems() * 4, &t);
  else if (!bf && split_fwd_ok(c))
    split_fwd_plan(c, &t);
  else if (!bf && split_run_ok(c))
    split_run_fwd_plan(c, &t);
  else
    fwd_plan(c, run_mode(c) && c.Cout % 4 == 0, bf, false, false, &t);
  return t;
}
double tile_seconds_bwd_data(const ConvGeom& c, bool bf) {
  double t = 0;
  if (bf && direct_bwd_data_ok(c))
    plan_direct(bwdd_dims(c), (double)c.in_elems() * 4, &t);
  else
    bwdd_plan(c, bf, false, false, &t);
  return t;
}
double tile_seconds_bwd_weight(const ConvGeom& c, bool bf) {
  double t = 0;
  bool swapped;
  if (!bf && split_bwdw_ok(c))
    split_bwdw_plan(c, &swapped, &t);
  else if (!bf && split_run_ok(c))
    split_run_bwdw_plan(c, &t);
  else
    bwdw_plan(c, run_mode(c), bf, false, &t);
  return t;
}
// scratch sizes cover every variant (generic / run mode, fp32 / bf16) of the op
size_t conv_fwd_ws_floats(const ConvGeom& c, const TileRows* rows) {
  int ns = 0;
  if (rows) ns = split_fwd_plan(c, nullptr, rows).ns;
  for (int run = 0; run < 2; ++run)
    for (int bf = 0; bf < 2; ++bf) ns = std::max(ns, fwd_plan(c, run && run_mode(c), bf).ns);
  ns = std::max(ns, fwd_plan(c, false, false, true).ns);
  ns = std::max(ns, fwd_plan(c, false, true, false, true).ns);
  if (run16_mode(c)) ns = std::max(ns, run16_fwd_plan(c).ns);
  if (split_fwd_ok(c)) ns = std::max(ns, split_fwd_plan(c).ns);
  if (split_run_ok(c)) ns = std::max(ns, split_run_fwd_plan(c).ns);
  if (direct_fwd_ok(c)) ns = std::max(ns, plan_direct(fwd_dims(c), (double)c.out_elems() * 4).ns);
  ns = std::max(ns, wave_conv_fwd_slices(c));
  return ns > 1 ? (size_t)ns * c.out_elems() : 0;
}
size_t conv_bwd_data_ws_floats(const ConvGeom& c) {
  int ns = std::max(std::max(bwdd_plan(c, false).ns, bwdd_plan(c, true).ns),
                          std::max(std::max(bwdd_plan(c, false, true).ns, bwdd_plan(c, true, false, true).ns),
                                   wave_conv_bwd_data_slices(c)));
  if (direct_bwd_data_ok(c)) ns = std::max(ns, plan_direct(bwdd_dims(c), (double)c.in_elems() * 4).ns);
  return ns > 1 ? (size_t)ns * c.in_elems() : 0;
}
size_t conv_bwd_weight_ws_floats(const ConvGeom& c) {
  size_t n = 0;
  for (int bf = 0; bf < 2; ++bf)
    for (int table = 0; table < 2; ++table) {
      const GemmPlan p = bwdw_plan(c, false, bf, table);
      if (p.ns > 1) n = std::max(n, (size_t)p.ns * c.w_elems());
      if (run_mode(c)) n = std::max(n, (size_t)bwdw_plan(c, true, bf, table).ns * run_w_elems(c));
    }
  if (split_bwdw_ok(c)) {
    bool swapped;
    const int ns = split_bwdw_plan(c, &swapped).ns;
    if (ns > 1) n = std::max(n, (size_t)ns * c.w_elems());
  }
  if (split_run_ok(c)) n = std::max(n, (size_t)split_run_bwdw_plan(c).ns * c.w_elems());
  if (direct_bwd_weight_ok(c)) n = std::max(n, (size_t)direct_bwd_weight_slices(c) * c.w_elems());
  return std::max(n, wave_conv_bwd_weight_ws_floats(c));
}

// ---- run mode helpers: padded copies of the forward weights / of their gradient ----
bool conv_run_mode(const ConvGeom& c) { return run_mode(c); }
size_t conv_run_w_floats(const ConvGeom& c) { return run_mode(c) ? (size_t)run_w_elems(c) : 0; }
// dir 0: wrun[(r,j)][o] = j < k*Cin ? wf[(r, j)][o] : 0;  dir 1: wf[(r,j)][o] = wrun[(r,j)][o] for j < k*Cin
__global__ void run_repack_kernel(const float* __restrict__ src, float* __restrict__ dst, int k, int kc, int run,
                                  int cout, int dir) {
  const size_t total = (size_t)k * run * cout;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;  // index into the padded layout
  if (i >= total) return;
  const int o = (int)(i % cout);
  const size_t q = i / cout;
  const int j = (int)(q % run), r = (int)(q / run);
  const size_t packed = ((size_t)r * kc + j) * cout + o;
  if (dir == 0)
    dst[i] = j < kc ? src[packed] : 0.f;
  else if (j < kc)
    dst[packed] = src[i];
}
int launch_conv_run_pack(const ConvGeom& c, const float* wf, float* wrun, hipStream_t st) {
  const size_t total = (size_t)run_w_elems(c);
  KernelScope ks("run_repack", 0, (double)total * 8.0, st);
  hipLaunchKernelGGL(run_repack_kernel, dim3(ceil_div(total, 256)), dim3(256), 0, st, wf, wrun, c.k, c.k * c.Cin,
                     run_len(c), c.Cout, 0);
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}
static int launch_conv_run_unpack(const ConvGeom& c, const float* dwrun, float* dwf, hipStream_t st) {
  const size_t total = (size_t)run_w_elems(c);
  KernelScope ks("run_repack", 0, (double)total * 8.0, st);
  hipLaunchKernelGGL(run_repack_kernel, dim3(ceil_div(total, 256)), dim3(256), 0, st, dwrun, dwf, c.k, c.k * c.Cin,
                     run_len(c), c.Cout, 1);
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}

bool conv_bf16_stored_ok(const ConvGeom& c) { return conv16_ok(c) && c.Cin % 8 == 0 && c.Cout % 8 == 0; }

int launch_conv_fwd(const ConvGeom& c, const float* x, const float* wf, const float* wrun, const float* bias,
                    int relu, float* y, float* ws, hipStream_t st, const uint16_t* x16, const uint16_t* wf16,
                    uint16_t* y16, const TileRows* rows) {
  // y16: also leave a bf16 copy of y there -- written by the epilogue of a single-pass product, else converted
  struct Copy16 {
    const float* y; uint16_t* y16; size_t n; hipStream_t st; bool pending;
  } copy{y, y16, (size_t)c.out_elems(), st, false};
  auto finish = [&copy](int rc) { return rc == ALEXNET_OK && copy.pending ? launch_to_bf16(copy.y, copy.y16, copy.n, copy.st) : rc; };
  if (wave_conv_fwd_ok(c, g_bf16))
    return launch_wave_conv_fwd(c, x, wf, bias, relu, y, y16, ws,
                                g_bf16 && (run_mode(c) ? c.Cout % 4 == 0 : fwd_A_vec(c, x) && fwd_B_vec(c, wf)), st);
  const bool run = wrun && run_mode(c) && c.Cout % 4 == 0;
  AlgoFlops af(conv_flops(c) * (rows ? rows->share : 1.0), conv_bytes(c) * (rows ? rows->share : 1.0));
  GemmDims d = fwd_dims(c);
  if (g_bf16 && x16 && wf16 && !run && conv_bf16_stored_ok(c) && aligned16(x16) && aligned16(wf16)) {
    const Im2colParams a = im2col16(fwd_A(c, nullptr), x16);
    const DenseParams b = fwd_B16k(c, wf16);
    if (patch_fwd_ok(c)) return launch_patch_fwd(c, x16, wf16, bias, relu, y, y16, st);
    if (direct_fwd_ok(c)) {
      const DirectPlan p = plan_direct(d, (double)c.out_elems() * 4);
      if (p.ns == 1)
        return launch_direct<IM2COL_FWD>(p, a, b, EpiBiasAct{y, c.Cout, bias, relu, c.og(), 0, 0, y16}, d, st);
      copy.pending = y16 != nullptr;
      AX_TRY(launch_direct<IM2COL_FWD>(p, a, b, EpiSlab{ws, (long)d.M * d.N, d.N, nullptr}, d, st));
      return finish(launch_slab_finish(ws, p.ns, d.groups, d.M, d.N, bias, relu, nullptr, y, st));
    }
    const GemmPlan p = fwd_plan(c, false, true, false, d.N % 128 == 0);  // 256-row tiles only without padded columns
    const bool tap = tap_ok(a, d, kBKbf);
    if (tap && tile192_ok(d))
      return launch_tile192<IM2COL_FWD>(a, b, EpiBiasAct{y, c.Cout, bias, relu, c.og(), 0, 0, y16}, d, st);
    if (p.ns == 1) {
      EpiBiasAct ep{y, c.Cout, bias, relu, c.og(), 0, 0, y16};
      if (tap) return by_tile_16<ConvGatherTap16<IM2COL_FWD>>(p, a, b, ep, d, st);
      return by_tile_16<ConvGather16<IM2COL_FWD>>(p, a, b, ep, d, st);
    }
    copy.pending = y16 != nullptr;
    EpiSlab ep{ws, (long)d.M * d.N, d.N, nullptr};
    if (tap)
      AX_TRY((by_tile_16<ConvGatherTap16<IM2COL_FWD>>(p, a, b, ep, d, st)));
    else
      AX_TRY((by_tile_16<ConvGather16<IM2COL_FWD>>(p, a, b, ep, d, st)));
    return finish(launch_slab_finish(ws, p.ns, d.groups, d.M, d.N, bias, relu, nullptr, y, st));
  }
  if (!g_bf16 && split_fwd_ok(c) && fwd_A_vec(c, x) && fwd_B_vec(c, wf)) {
    const GemmPlan p = split_fwd_plan(c, nullptr, rows);
    const DenseParams a = pointwise_A(c, x), b = fwd_B(c, wf);
    copy.pending = y16 != nullptr;
    if (p.ns == 1) {
      EpiBiasAct ep{y, c.Cout, bias, relu, c.og(), 0, 0, nullptr};
      return finish(by_tile_split<SplitKInner, SplitRowInner>(p, a, b, ep, d.M, d.N, d.K, d.groups, st, rows, 1));
    }
    EpiSlab ep{ws, (long)d.M * d.N, d.N, nullptr};
    AX_TRY((by_tile_split<SplitKInner, SplitRowInner>(p, a, b, ep, d.M, d.N, d.K, d.groups, st, rows, 1)));
    return finish(launch_slab_finish(ws, p.ns, d.groups, d.M, d.N, bias, relu, nullptr, y, st));
  }
  if (rows) {
    set_error("products of short tiles: no kernel for these operands");
    return ALEXNET_EINVAL;
  }
  if (run) d.K = run_k(c);
  if (!g_bf16 && run && split_run_ok(c) && aligned16(wrun)) {
    const GemmPlan p = split_run_fwd_plan(c);
    copy.pending = y16 != nullptr;
    if (p.ns == 1) {
      EpiBiasAct ep{y, c.Cout, bias, relu, c.og(), 0, 0, nullptr};
      return finish(by_tile_run<SplitRun>(p, run_A(c, x), run_B(c, wrun), ep, d.M, d.N, d.K, st));
    }
    EpiSlab ep{ws, (long)d.M * d.N, d.N, nullptr};
    AX_TRY((by_tile_run<SplitRun>(p, run_A(c, x), run_B(c, wrun), ep, d.M, d.N, d.K, st)));
    return finish(launch_slab_finish(ws, p.ns, 1, d.M, d.N, bias, relu, nullptr, y, st));
  }
  const bool av = run || fwd_A_vec(c, x), bv = run || fwd_B_vec(c, wf);
  const bool bf = g_bf16 && av && bv;
  const Im2colParams a = run ? run_A(c, x) : fwd_A(c, x);
  const DenseParams b = run ? run_B(c, wrun) : fwd_B(c, wf);
  const bool t48 = !run && !bf && av && bv && tap_ok(a, d, kBK48);
  const GemmPlan p = fwd_plan(c, run, bf, t48);
  const bool tap = !run && !bf && av && bv && tap_ok(a, d);
  const bool tapbf = bf && !run && tap_ok(a, d, kBKbf);
  if (p.ns == 1) {
    EpiBiasAct ep{y, c.Cout, bias, relu, c.og(), 0, 0, y16};
    if (tapbf) return by_tile_bf<ConvGatherTapBf<IM2COL_FWD>>(p, a, b, ep, d, st);
    if (bf) return by_tile_bf<ConvGatherBf<IM2COL_FWD>>(p, a, b, ep, d, st);
    if (tap) return by_tile_tap<ConvGatherTap<IM2COL_FWD>>(p, a, b, ep, d, st);
    return by_tile<ConvGather<IM2COL_FWD>>(p, av, bv, a, b, ep, d, st);
  }
  EpiSlab ep{ws, (long)d.M * d.N, d.N, nullptr};
  if (tapbf)
    AX_TRY((by_tile_bf<ConvGatherTapBf<IM2COL_FWD>>(p, a, b, ep, d, st)));
  else if (bf)
    AX_TRY((by_tile_bf<ConvGatherBf<IM2COL_FWD>>(p, a, b, ep, d, st)));
  else if (tap)
    AX_TRY((by_tile_tap<ConvGatherTap<IM2COL_FWD>>(p, a, b, ep, d, st)));
  else
    AX_TRY((by_tile<ConvGather<IM2COL_FWD>>(p, av, bv, a, b, ep, d, st)));
  copy.pending = y16 != nullptr;
  return finish(launch_slab_finish(ws, p.ns, d.groups, d.M, d.N, bias, relu, nullptr, y, st));
}

// ---- the first layer over bf16 pictures with four channels per pixel (conv_plan.h, run16) ----
bool conv_run16_ok(const ConvGeom& c) { return run16_mode(c); }
size_t conv_run16_x_elems(const ConvGeom& c) { return run16_mode(c) ? (size_t)run16_x_elems(c) : 0; }
size_t conv_run16_w_elems(const ConvGeom& c) { return run16_mode(c) ? (size_t)run16_w_elems(c) : 0; }
static GemmPlan run16_fwd_plan(const ConvGeom& c, double* t_out) {
  const GemmDims d = fwd_dims(c);
  return plan_gemm(d.M, d.N, run16_k(c), 1, (double)c.out_elems() * 4, 8, true, false, 0, true, t_out);
}
struct ConvRun16 {
  template <class T, class Epi>
  static int go(const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d, int kchunk, int ns,
                hipStream_t st) {
    return launch_tile_bf<T, Im2colKInner16<T::BM, T::BK, IM2COL_FWD>, DenseKInner16<T::BN, T::BK>, Epi>(
        a, b, e, d.M, d.N, d.K, kchunk, ns, d.groups, st);
  }
};
int launch_conv_fwd_run16(const ConvGeom& c, const uint16_t* x4, const uint16_t* wk, const float* bias, int relu,
                          float* y, float* ws, hipStream_t st, uint16_t* y16) {
  if (!run16_mode(c) || !aligned16(x4) || !aligned16(wk)) {
    set_error("conv run16: geometry or alignment does not allow it");
    return ALEXNET_EINVAL;
  }
  if (first16_ok(c)) return launch_first16(c, x4, wk, bias, relu, y, y16, st);
  AlgoFlops af(conv_flops(c), conv_bytes(c));
  GemmDims d = fwd_dims(c);
  d.K = run16_k(c);
  const Im2colParams a = run16_A(c, x4);
  const DenseParams b = run16_Bk(c, wk);
  const GemmPlan p = run16_fwd_plan(c);
  if (p.ns == 1) {
    EpiBiasAct ep{y, c.Cout, bias, relu, c.og(), 0, 0, y16};
    if (p.bm == 256 && d.N % 96 == 0 && d.N % 128 != 0)  // whole 96-column tiles instead of padded 128-column ones
      return ConvRun16::go<B256n96, EpiBiasAct>(a, b, ep, d, round_up(d.K, kBKbf), 1, st);
    return by_tile_16<ConvRun16>(p, a, b, ep, d, st);
  }
  EpiSlab ep{ws, (long)d.M * d.N, d.N, nullptr};
  AX_TRY((by_tile_16<ConvRun16>(p, a, b, ep, d, st)));
  AX_TRY(launch_slab_finish(ws, p.ns, 1, d.M, d.N, bias, relu, nullptr, y, st));
  return y16 ? launch_to_bf16(y, y16, (size_t)c.out_elems(), st) : ALEXNET_OK;
}
// ---- strided backward data by phases (conv_plan.h) ----
bool conv_phase_mode(const ConvGeom& c) { return phase_mode(c) && c.Cout % 4 == 0 && phase_n(c) % 4 == 0; }
size_t conv_phase_w_floats(const ConvGeom& c) { return conv_phase_mode(c) ? (size_t)phase_w_elems(c) : 0; }
__global__ void phase_pack_kernel(const float* __restrict__ wf, float* __restrict__ wp, int k, int st, int ka, int cin,
                                  int cout) {
  const int pn = st * st * cin;
  const size_t total = (size_t)ka * ka * cout * pn;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;  // index into wp[(a,b,o)][(py,px,c)]
  if (i >= total) return;
  const int col = (int)(i % pn);
  size_t q = i / pn;
  const int o = (int)(q % cout);
  q /= cout;
  const int b = (int)(q % ka), a = (int)(q / ka);
  const int c = col % cin, pp = col / cin, px = pp % st, py = pp / st;
  const int r = py + st * a, s = px + st * b;
  wp[i] = (r < k && s < k) ? wf[((size_t)(r * k + s) * cin + c) * cout + o] : 0.f;
}
static int launch_conv_bwd_data_phases(const ConvGeom& c, const float* dy, const float* wf, float* wphase, float* dx,
                                       hipStream_t st) {
  const size_t total = (size_t)phase_w_elems(c);
  {
    KernelScope ks("phase_pack", 0, (double)total * 8.0, st);
    hipLaunchKernelGGL(phase_pack_kernel, dim3(ceil_div(total, 256)), dim3(256), 0, st, wf, wphase, c.k, c.stride,
                       phase_taps(c), c.Cin, c.Cout);
    AX_LAUNCH_CHECK();
  }
  const GemmDims d = phase_dims(c);
  AlgoFlops af(conv_flops(c), conv_bytes(c));
  GemmPlan p = plan_gemm(d.M, d.N, d.K, 1, 0, 1, false);  // never split: the epilogue scatters; fp32 only
  return by_tile<ConvGather<IM2COL_T1>>(p, true, true, phase_A(c, dy), phase_B(c, wphase), phase_epilogue(c, dx), d,
                                        st);
}

int launch_conv_bwd_data(const ConvGeom& c, const float* dy, const float* wf, const float* wb, float* wphase,
                         const float* gate, float* dx, float* ws, hipStream_t st, const uint16_t* dy16,
                         const uint16_t* wb16, uint16_t* dx16, bool small) {
  // dx16: also leave a bf16 copy of dx there (see launch_conv_fwd)
  struct Copy16 {
    const float* y; uint16_t* y16; size_t n; hipStream_t st; bool pending;
  } copy{dx, dx16, (size_t)c.in_elems(), st, false};
  auto finish = [&copy](int rc) { return rc == ALEXNET_OK && copy.pending ? launch_to_bf16(copy.y, copy.y16, copy.n, copy.st) : rc; };
  if (wphase && !gate && conv_phase_mode(c) && aligned16(dy)) {
    copy.pending = dx16 != nullptr;
    return finish(launch_conv_bwd_data_phases(c, dy, wf, wphase, dx, st));
  }
  if (small && wave_conv_bwd_data_ok(c, g_bf16))
    return launch_wave_conv_bwd_data(c, dy, wf, gate, dx, dx16, ws, g_bf16 && bwdd_A_vec(c, dy) && bwdd_B_vec(c, wf), st);
  const GemmDims d = bwdd_dims(c);
  AlgoFlops af(conv_flops(c), conv_bytes(c));
  if (g_bf16 && dy16 && wb16 && conv_bf16_stored_ok(c) && aligned16(dy16) && aligned16(wb16)) {
    const Im2colParams a = im2col16(bwdd_A(c, nullptr), dy16);
    const DenseParams b = bwdd_B16k(c, wb16);
    if (direct_bwd_data_ok(c)) {
      const DirectPlan p = plan_direct(d, (double)c.in_elems() * 4);
      if (p.ns == 1) return launch_direct<IM2COL_T1>(p, a, b, EpiGate{dx, c.Cin, gate, c.cg(), 0, 0, dx16}, d, st);
      copy.pending = dx16 != nullptr;
      AX_TRY(launch_direct<IM2COL_T1>(p, a, b, EpiSlab{ws, (long)d.M * d.N, d.N, nullptr}, d, st));
      return finish(launch_slab_finish(ws, p.ns, d.groups, d.M, d.N, nullptr, 0, gate, dx, st));
    }
    const GemmPlan p = bwdd_plan(c, true, false, d.N % 128 == 0);
    const bool tap = tap_ok(a, d, kBKbf);
    if (tap && tile192_ok(d))
      return launch_tile192<IM2COL_T1>(a, b, EpiGate{dx, c.Cin, gate, c.cg(), 0, 0, dx16}, d, st);
    if (p.ns == 1) {
      EpiGate ep{dx, c.Cin, gate, c.cg(), 0, 0, dx16};
      if (tap) return by_tile_16<ConvGatherTap16<IM2COL_T1>>(p, a, b, ep, d, st);
      return by_tile_16<ConvGather16<IM2COL_T1>>(p, a, b, ep, d, st);
    }
    copy.pending = dx16 != nullptr;
    EpiSlab ep{ws, (long)d.M * d.N, d.N, nullptr};
    if (tap)
      AX_TRY((by_tile_16<ConvGatherTap16<IM2COL_T1>>(p, a, b, ep, d, st)));
    else
      AX_TRY((by_tile_16<ConvGather16<IM2COL_T1>>(p, a, b, ep, d, st)));
    return finish(launch_slab_finish(ws, p.ns, d.groups, d.M, d.N, nullptr, 0, gate, dx, st));
  }
  const bool av = bwdd_A_vec(c, dy) && bwdd_B_vec(c, wb), bv = bwdd_B_vec(c, wb);
  const bool bf = g_bf16 && av && bv && c.stride == 1;
  const Im2colParams a = bwdd_A(c, dy);
  const DenseParams b = bwdd_B(c, wb);
  const bool t48 = !bf && c.stride == 1 && av && bv && tap_ok(a, d, kBK48);
  const GemmPlan p = bwdd_plan(c, bf, t48);
  const bool tap = !bf && c.stride == 1 && av && bv && tap_ok(a, d);
  const bool tapbf = bf && tap_ok(a, d, kBKbf);
  if (p.ns == 1) {
    EpiGate ep{dx, c.Cin, gate, c.cg(), 0, 0, dx16};
    if (tapbf) return by_tile_bf<ConvGatherTapBf<IM2COL_T1>>(p, a, b, ep, d, st);
    if (bf) return by_tile_bf<ConvGatherBf<IM2COL_T1>>(p, a, b, ep, d, st);
    if (tap) return by_tile_tap<ConvGatherTap<IM2COL_T1>>(p, a, b, ep, d, st);
    if (c.stride == 1) return by_tile<ConvGather<IM2COL_T1>>(p, av, bv, a, b, ep, d, st);
    return by_tile<ConvGather<IM2COL_TS>>(p, av, bv, a, b, ep, d, st);
  }
  EpiSlab ep{ws, (long)d.M * d.N, d.N, nullptr};
  if (tapbf)
    AX_TRY((by_tile_bf<ConvGatherTapBf<IM2COL_T1>>(p, a, b, ep, d, st)));
  else if (bf)
    AX_TRY((by_tile_bf<ConvGatherBf<IM2COL_T1>>(p, a, b, ep, d, st)));
  else if (tap)
    AX_TRY((by_tile_tap<ConvGatherTap<IM2COL_T1>>(p, a, b, ep, d, st)));
  else if (c.stride == 1)
    AX_TRY((by_tile<ConvGather<IM2COL_T1>>(p, av, bv, a, b, ep, d, st)));
  else
    AX_TRY((by_tile<ConvGather<IM2COL_TS>>(p, av, bv, a, b, ep, d, st)));
  copy.pending = dx16 != nullptr;
  return finish(launch_slab_finish(ws, p.ns, d.groups, d.M, d.N, nullptr, 0, gate, dx, st));
}

bool conv_bwd_weight_bf16(const ConvGeom& c, const float* x, const float* dy) {
  return g_bf16 && (run_mode(c) || bwdw_A_vec(c, x)) && bwdw_B_vec(c, dy);
}

// defer_ns (generic layout only): the split-k slices are left in ws, [group][slice][slab], and their number is
// returned there for the caller to add them up later (1: the result is in dwf already)
int launch_conv_bwd_weight(const ConvGeom& c, const float* x, const float* dy, float* dwf, float* dwrun, float* ws,
                           hipStream_t st, int* defer_ns, bool small, WgradTail* tail, const TileRows* rows) {
  if (small && wave_conv_bwd_weight_ok(c, g_bf16)) {
    if (defer_ns) *defer_ns = 1;
    return launch_wave_conv_bwd_weight(c, x, dy, dwf, ws, conv_bwd_weight_bf16(c, x, dy), st);
  }
  const bool run = dwrun && run_mode(c) && bwdw_B_vec(c, dy);
  AlgoFlops af(conv_flops(c) * (rows ? rows->share : 1.0), conv_bytes(c) * (rows ? rows->share : 1.0));
  GemmDims d = bwdw_dims(c);
  if (run) d.M = run_k(c);
  const bool av = run || bwdw_A_vec(c, x), bv = bwdw_B_vec(c, dy);
  if (!g_bf16 && !run && split_bwdw_ok(c) && av && bv) {
    bool swapped;
    const GemmPlan p = split_bwdw_plan(c, &swapped);
    const long slab = (long)d.M * d.N;
    DenseParams a = pointwise_A(c, x);
    a.R = c.cg();
    float* out = p.ns > 1 ? ws : dwf;
    if (swapped) {
      EpiSlabSwapped ep{out, slab, d.N, nullptr};
      AX_TRY((by_tile_split<SplitRowInner, SplitRowInner>(p, bwdw_B(c, dy), a, ep, d.N, d.M, d.K, d.groups, st, rows, 2)));
    } else {
      EpiSlab ep{out, slab, d.N, nullptr};
      AX_TRY((by_tile_split<SplitRowInner, SplitRowInner>(p, a, bwdw_B(c, dy), ep, d.M, d.N, d.K, d.groups, st, rows, 2)));
    }
    if (defer_ns) *defer_ns = p.ns;
    return defer_ns || p.ns == 1 ? ALEXNET_OK : launch_reduce_slabs(ws, p.ns, slab, d.groups, dwf, st);
  }
  if (rows) {
    set_error("products of short tiles: no kernel for these operands");
    return ALEXNET_EINVAL;
  }
  const bool bf = g_bf16 && av && bv;
  const Im2colParams a = run ? run_A(c, x) : bwdw_A(c, x);
  if (!g_bf16 && run && split_run_ok(c)) {  // compact rows, see SplitRunT
    const GemmPlan p = split_run_bwdw_plan(c);
    const int kc = c.k * c.Cin;
    const long slab = (long)c.k * kc * c.Cout;
    EpiSlab ep{p.ns > 1 ? ws : dwrun, slab, c.Cout, nullptr};
    AX_TRY((by_tile_run<SplitRunT>(p, run_t_params(a, kc), bwdw_B(c, dy), ep, c.k * kc, c.Cout, d.K, st)));
    if (defer_ns) *defer_ns = 1;
    if (tail && tail->n < kMaxWgradJobs) {
      WgradJob j{};
      j.slices = p.ns > 1 ? ws : dwrun;
      j.dU = dwf;
      j.slab = slab;
      j.nsplit = p.ns; j.groups36 = 1; j.k = c.k; j.head = kc / 4 * 4; j.kc = kc; j.cout = c.Cout;
      wgrad_tail_add(*tail, j);
      return ALEXNET_OK;
    }
    return launch_reduce_slabs_unpack(p.ns > 1 ? ws : dwrun, p.ns, slab, c.k, kc / 4 * 4, kc, c.Cout, dwf, st);
  }
  bool table = av && bv && table_ok(a, d) && (!bf || d.K % kBKbf == 0);
  GemmPlan p = bwdw_plan(c, run, bf, table);
  if (table && p.kchunk > kMaxTableK) {  // no split count within reach keeps the k range inside the table
    table = false;
    p = bwdw_plan(c, run, bf, false);
  }
  const long slab = (long)d.M * d.N;
  float* out = run ? dwrun : dwf;
  EpiSlab ep{p.ns > 1 ? ws : out, slab, d.N, nullptr};
  if (bf && table)
    AX_TRY((by_tile_bf<ConvWeightGradTableBf>(p, a, bwdw_B(c, dy), ep, d, st)));
  else if (bf)
    AX_TRY((by_tile_bf<ConvWeightGradBf>(p, a, bwdw_B(c, dy), ep, d, st)));
  else if (table)
    AX_TRY((by_tile_tap<ConvWeightGradTable>(p, a, bwdw_B(c, dy), ep, d, st)));
  else
    AX_TRY((by_tile<ConvWeightGrad>(p, av, bv, a, bwdw_B(c, dy), ep, d, st)));
  if (defer_ns && !run) {
    *defer_ns = p.ns;
    return ALEXNET_OK;
  }
  if (defer_ns) *defer_ns = 1;
  if (run && p.ns > 1)  // slices of the padded layout straight to the packed one
    return launch_reduce_slabs_unpack(ws, p.ns, slab, c.k, run_len(c), c.k * c.Cin, c.Cout, dwf, st);
  if (p.ns > 1) AX_TRY(launch_reduce_slabs(ws, p.ns, slab, d.groups, out, st));
  if (run) AX_TRY(launch_conv_run_unpack(c, dwrun, dwf, st));
  return ALEXNET_OK;
}

// ------------------------------------------------------------ dense layers ---
// y = act(x w^T + b),  dx = gate(dy w),  dw = dy^T x.  The batch is the small
// dimension, so forward and backward-data split the reduction over several
// workgroups and finish in a second kernel that also applies the activation.
// fp32 products use fc_plan, those that gemm_split.h does not take the 128 x 128 tile (fc_split), as do bf16 products over
// fp32 operands; over stored ones dense_plan() (gemm_direct.h).

static int fc_split(int B, int N, int K, int* kchunk, bool bf, double* t_out = nullptr) {
  const int bk = bf ? kBKbf : kBK;
  const int ktiles = ceil_div(K, bk);
  const long tiles = (long)ceil_div(B, 128) * ceil_div(N, 128);
  const double t_tile = 2.0 * 128 * 128 * (double)ktiles * bk / (0.614e12 * (bf ? 3.2 : 0.8));
  int best = 1, best_per = ktiles;
  double best_t = 1e30;
  for (int s = 1; s <= 64 && s <= ktiles; ++s) {
    const int per = ceil_div(ktiles, s);
    if (ceil_div(ktiles, per) != s) continue;
    if (s > 1 && per < 6) break;
    double t = (double)ceil_div(tiles * s, 256) * t_tile * per / ktiles;
    if (s > 1) t += (s + 1) * (double)B * N * 4 / 2.5e12 + kSecondLaunch;
    if (t < best_t * 0.98) {
      best_t = t;
      best = s;
      best_per = per;
    }
  }
  *kchunk = best_per * bk;
  if (t_out) *t_out = best_t;
  return best;
}
static GemmPlan fc_plan(int B, int N, int K, double* t_out = nullptr) {
  return plan_split(B, N, K, 1, (double)B * N * 4, 64, t_out, B <= 64);
}
double tile_seconds_dense(int M, int N, int K, bool bf) {
  double t = 0;
  int kc;
  if (bf)
    fc_split(M, N, K, &kc, true, &t);
  else
    fc_plan(M, N, K, &t);
  return t;
}
size_t fc_ws_floats(int B, int in, int out) {
  int kc;
  size_t n = 0;
  if (fc_bf16_stored_ok(in, out)) {
    n = std::max(n, (size_t)dense_plan(B, out, in).ns * B * out);
    n = std::max(n, (size_t)dense_plan(B, in, out).ns * B * in);
  }
  for (int bf = 0; bf < 2; ++bf) {
    n = std::max(n, (size_t)fc_split(B, out, in, &kc, bf) * B * out);
    n = std::max(n, (size_t)fc_split(B, in, out, &kc, bf) * B * in);
  }
  n = std::max(n, (size_t)fc_plan(B, out, in).ns * B * out);
  n = std::max(n, (size_t)fc_plan(B, in, out).ns * B * in);
  return n;
}

__global__ void fc_fwd_finish_kernel(const float* __restrict__ ws, int nsplit, int B, int out, FcAct act,
                                     float* __restrict__ y, uint16_t* __restrict__ y16) {
  const size_t total = (size_t)B * out;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  float s = 0.f;
#pragma unroll 8
  for (int k = 0; k < nsplit; ++k) s += ws[(size_t)k * total + i];  // loads in flight together, added in order
  const int o = (int)(i % out);
  if (act.bias) s += act.bias[o];
  if (act.relu) s = s > 0.f ? s : 0.f;
  if (act.dropout && !dropout_keep(act.key, act.tag, i, act.thresh24)) s = 0.f;
  y[i] = s * act.scale;
  if (y16) store_bf16(y16 + i, s * act.scale);
}
__global__ void fc_bwd_finish_kernel(const float* __restrict__ ws, int nsplit, size_t total,
                                     const float* __restrict__ gate, float* __restrict__ dx,
                                     uint16_t* __restrict__ dx16) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  float s = 0.f;
#pragma unroll 8
  for (int k = 0; k < nsplit; ++k) s += ws[(size_t)k * total + i];  // loads in flight together, added in order
  if (gate && !(gate[i] > 0.f)) s = 0.f;
  dx[i] = s;
  if (dx16) store_bf16(dx16 + i, s);
}

// y = act(x w^T + b) for at most kFcRows rows of x: the weights are read once, and that is all the time there is -- a
// matrix tile would be 1/16 full at best and needs slices of the reduction, and a second kernel to add them, to reach
// every compute unit.  A wave owns two outputs and runs along k, 1024 values at a time, with eight 16-byte loads of
// weights in flight per lane; the rows of x pass through LDS, shared by the workgroup's four waves.  The sums stay in
// fp32: one chain of in/64 products per lane, then a tree over the lanes.  BF: both operands rounded to bf16 first, as
// the bf16 products have them (a handle's bf16 copy of the weights, twice the traffic of reading them, is not needed).
// fc6 + fc7 of one picture: 111 + 9 us (products in slices, finish) -> 37, 5.9 TB/s.  The line is at four rows: with
// more the multiplies bound it.  One-pass inference, tiles | here: 1 row 163 | 143 us, 2 178 | 165, 4 209 | 206, 6 252 |
// 267, 8 279 | 298; bf16 handles, which need no copy of the weights here, 4 241 | 229, 8 264 | 289.
constexpr int kFcRows = 4;
template <int BB, bool BF>
__global__ void __launch_bounds__(256)
fc_rows_kernel(const float* __restrict__ x, const float* __restrict__ w, int B, int in, int out, FcAct act,
               float* __restrict__ y, uint16_t* __restrict__ y16) {
  constexpr int R = 2, CH = 1024, Q = CH / 256;  // outputs per wave; k per chunk; 16-byte loads per lane and chunk
  __shared__ float4 xs[BB][CH / 4];
  const int tid = threadIdx.x, lane = tid & 63, row0 = (blockIdx.x * 4 + (tid >> 6)) * R, in4 = in / 4;
  auto prep = [](float4 v) {
    if (BF) {
      const uint32_t a = pack_bf16(v.x, v.y), b = pack_bf16(v.z, v.w);
      v = make_float4(bf_lo(a), bf_hi(a), bf_lo(b), bf_hi(b));
    }
    return v;
  };
  const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
  float acc[R][BB];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int b = 0; b < BB; ++b) acc[r][b] = 0.f;
  for (int c0 = 0; c0 < in4; c0 += CH / 4) {
    float4 wv[R][Q];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float4* wr = reinterpret_cast<const float4*>(w) + (size_t)min(row0 + r, out - 1) * in4;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int k = c0 + q * 64 + lane;
        wv[r][q] = zero;
        if (k < in4) wv[r][q] = wr[k];
      }
    }
    __syncthreads();  // the waves are done with the last chunk of x
    for (int i = tid; i < BB * (CH / 4); i += 256) {
      const int b = i / (CH / 4), k = c0 + i % (CH / 4);
      float4 v = zero;
      if (b < B && k < in4) v = reinterpret_cast<const float4*>(x)[(size_t)b * in4 + k];
      xs[b][i % (CH / 4)] = prep(v);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      float4 wq[R];
#pragma unroll
      for (int r = 0; r < R; ++r) wq[r] = prep(wv[r][q]);
#pragma unroll
      for (int b = 0; b < BB; ++b) {
        const float4 xv = xs[b][q * 64 + lane];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          acc[r][b] = fmaf(wq[r].x, xv.x, acc[r][b]);
          acc[r][b] = fmaf(wq[r].y, xv.y, acc[r][b]);
          acc[r][b] = fmaf(wq[r].z, xv.z, acc[r][b]);
          acc[r][b] = fmaf(wq[r].w, xv.w, acc[r][b]);
        }
      }
    }
  }
  float mine = 0.f;  // lane r*BB + b keeps the sum of output row0 + r, row b
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int b = 0; b < BB; ++b) {
      float s = acc[r][b];
#pragma unroll
      for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d);
      if (lane == r * BB + b) mine = s;
    }
  const int b = lane % BB, o = row0 + lane / BB;
  if (lane >= R * BB || b >= B || o >= out) return;
  const size_t i = (size_t)b * out + o;
  if (act.bias) mine += act.bias[o];
  if (act.relu) mine = mine > 0.f ? mine : 0.f;
  if (act.dropout && !dropout_keep(act.key, act.tag, i, act.thresh24)) mine = 0.f;
  y[i] = mine * act.scale;
  if (y16) store_bf16(y16 + i, mine * act.scale);
}
bool fc_rows_ok(int B, int in) { return B <= kFcRows && in % 4 == 0; }
template <bool BF>
static int launch_fc_rows(int B, int in, int out, const float* x, const float* w, const FcAct& act, float* y,
                          uint16_t* y16, hipStream_t st) {
  KernelScope ks("fc_rows", 2.0 * B * in * (double)out, 4.0 * ((double)in * out + (double)B * (in + out)), st);
  const dim3 grid(ceil_div(out, 8)), block(256);
  if (B <= 1) hipLaunchKernelGGL((fc_rows_kernel<1, BF>), grid, block, 0, st, x, w, B, in, out, act, y, y16);
  else if (B <= 2) hipLaunchKernelGGL((fc_rows_kernel<2, BF>), grid, block, 0, st, x, w, B, in, out, act, y, y16);
  else hipLaunchKernelGGL((fc_rows_kernel<kFcRows, BF>), grid, block, 0, st, x, w, B, in, out, act, y, y16);
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}

static inline bool vec_ok(const float* p, long ld) { return aligned16(p) && ld % 4 == 0; }

// Which kernels take a dense fp32 product, and its tile and slices
static inline bool fc_split_ok(bool vec, int K) { return vec && K >= kSplitMinK; }
static GemmPlan fc_product_plan(int B, int N, int K, bool vec, bool bf) {
  if (!bf && fc_split_ok(vec, K)) return fc_plan(B, N, K);
  GemmPlan p{128, 128, 0, 0};
  p.ns = fc_split(B, N, K, &p.kchunk, bf);
  return p;
}
// 16-byte loads and K long enough: on the bf16 matrix cores; else on the fp32 ones
template <template <int> class SA, template <int> class SB, template <int, int, bool> class ALT,
          template <int, int, bool> class BLT, class Epi>
static int launch_dense(bool vec, const GemmPlan& p, const DenseParams& a, const DenseParams& b, const Epi& ep, int M,
                        int N, int K, hipStream_t st) {
  if (fc_split_ok(vec, K)) return by_tile_split<SA, SB>(p, a, b, ep, M, N, K, 1, st);
  if (vec)
    return launch_tile<T128, ALT<128, kBK, true>, BLT<128, kBK, true>, Epi>(a, b, ep, M, N, K, p.kchunk, p.ns, 1, st);
  return launch_tile<T128, ALT<128, kBK, false>, BLT<128, kBK, false>, Epi>(a, b, ep, M, N, K, p.kchunk, p.ns, 1, st);
}

typedef BfRowMajor<DenseKInner<128, kBKbf, true>, 128, kBKbf> BfDenseK;
typedef BfDenseRowInner<128, kBKbf> BfDenseR;

bool fc_bf16_stored_ok(int in, int out) { return in % 8 == 0 && out % 8 == 0; }

// A dense layer is a 1 x 1 convolution over pictures of one pixel
static int launch_dense_direct(const DensePlan& dp, int B, int in, int out, const uint16_t* x16, const uint16_t* w16,
                               const EpiSlab& e, hipStream_t st) {
  const ConvGeom c{B, 1, 1, in, out, 1, 1, 0, 1, 1, 1};
  const Im2colParams a = im2col16(fwd_A(c, nullptr), x16);
  const DenseParams b = fwd_B16k(c, w16);
  const GemmDims d = fwd_dims(c);
  const DirectPlan p{0, dp.ns, dp.per};
  if (dp.tall) return launch_direct_tile<128, 128, 2, 2, 2, IM2COL_FWD>(p, a, b, e, d, st);
  return launch_direct_tile<64, 128, 2, 2, 3, IM2COL_FWD>(p, a, b, e, d, st);
}

int launch_fc_fwd(int B, int in, int out, const float* x, const float* w, const FcAct& act, float* y, float* ws,
                  hipStream_t st, const uint16_t* x16, const uint16_t* w16, uint16_t* y16) {
  const bool vec = vec_ok(x, in) && vec_ok(w, in), bf = g_bf16 && vec;
  if (vec && fc_rows_ok(B, in))
    return bf ? launch_fc_rows<true>(B, in, out, x, w, act, y, y16, st) : launch_fc_rows<false>(B, in, out, x, w, act, y, y16, st);
  if (wave_fc_fwd_ok(B, in, out, g_bf16)) return launch_wave_fc_fwd(B, in, out, x, w, act, y, y16, bf, st);
  const bool s16 = bf && x16 && w16 && fc_bf16_stored_ok(in, out) && aligned16(x16) && aligned16(w16);
  const GemmPlan p = fc_product_plan(B, out, in, vec, bf);
  const DensePlan dp = dense_plan(B, out, in);
  const int ns = s16 ? dp.ns : p.ns, kchunk = p.kchunk;
  DenseParams a{x, in, 0, B, (uint32_t)((size_t)B * in * 4)};
  DenseParams b{w, in, 0, out, (uint32_t)((size_t)out * in * 4)};
  // both operands run along k = in
  auto product = [&](const auto& ep) -> int {
    typedef std::decay_t<decltype(ep)> Epi;
    if (bf) return launch_tile_bf<B128, BfDenseK, BfDenseK, Epi>(a, b, ep, B, out, in, kchunk, ns, 1, st);
    return launch_dense<SplitKInner, SplitKInner, DenseKInner, DenseKInner>(vec, p, a, b, ep, B, out, in, st);
  };
  // A full tile that finishes itself works through 32 to 64 values per lane, one after the other: the mask's hash costs more
  // there than a second launch (128 rows 256 wide: 456 against 434 us per small training step), and so do mask and gate in the
  // bf16 kernels (438 against 434; 30 rows 200 wide 363 against 357).  (Measured when fp32 tiles were stored four columns of 32
  // rows at a time; a row at a time, as they are now, a product of 1000 x 1000 over 512 takes 22.9 us, 22.8 then, of 64 x 4096
  // 17.0 and 17.8.)
  if (ns == 1 && !bf && (B <= 32 || !act.dropout)) return product(EpiFcAct{y, out, act, y16});
  const EpiSlab slabs{ws, (long)B * out, out, nullptr};
  if (s16)
    AX_TRY(launch_dense_direct(dp, B, in, out, x16, w16, slabs, st));
  else
    AX_TRY(product(slabs));
  const size_t total = (size_t)B * out;
  KernelScope ks("fc_finish", 0, (double)total * 4.0 * (ns + 1), st);
  hipLaunchKernelGGL(fc_fwd_finish_kernel, dim3(ceil_div(total, 256)), dim3(256), 0, st, ws, ns, B, out, act, y, y16);
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}

int launch_fc_bwd_data(int B, int in, int out, const float* dy, const float* w, const float* gate, float* dx,
                       float* ws, hipStream_t st, const uint16_t* dy16, const uint16_t* w16, uint16_t* dx16) {
  const bool vec = vec_ok(dy, out) && vec_ok(w, in), bf = g_bf16 && vec;
  const bool s16 = bf && dy16 && w16 && fc_bf16_stored_ok(in, out) && aligned16(dy16) && aligned16(w16);
  const GemmPlan p = fc_product_plan(B, in, out, vec, bf);
  const int ns = s16 ? dense_plan(B, in, out).ns : p.ns, kchunk = p.kchunk;
  DenseParams a{dy, out, 0, B, (uint32_t)((size_t)B * out * 4)};
  DenseParams b{w, in, 0, in, (uint32_t)((size_t)out * in * 4)};
  // A runs along k = out, B along its rows = in
  auto product = [&](const auto& ep) -> int {
    typedef std::decay_t<decltype(ep)> Epi;
    if (bf) return launch_tile_bf<B128, BfDenseK, BfDenseR, Epi>(a, b, ep, B, in, out, kchunk, ns, 1, st);
    return launch_dense<SplitKInner, SplitRowInner, DenseKInner, DenseRowInner>(vec, p, a, b, ep, B, in, out, st);
  };
  if (ns == 1 && !bf) return product(EpiGate{dx, in, gate, in, 0, 0, dx16});  // see launch_fc_fwd
  if (s16)
    AX_TRY(launch_direct_dense_bwd_data(B, in, out, dy16, w16, ws, st));
  else
    AX_TRY(product(EpiSlab{ws, (long)B * in, in, nullptr}));
  const size_t total = (size_t)B * in;
  KernelScope ks("fc_finish", 0, (double)total * 4.0 * (ns + 1 + (gate ? 1 : 0)), st);
  hipLaunchKernelGGL(fc_bwd_finish_kernel, dim3(ceil_div(total, 256)), dim3(256), 0, st, ws, ns, total, gate, dx,
                     dx16);
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}

int launch_fc_bwd(int B, int in, int out, const float* x, const float* dy, const float* w, const float* gate, float* dx,
                  float* dw, hipStream_t st, uint16_t* dx16) {
  const bool bf = g_bf16 && vec_ok(dy, out) && vec_ok(w, in) && vec_ok(x, in);
  return launch_wave_fc_bwd(B, in, out, x, dy, w, gate, dx, dx16, dw, bf, st);
}

static bool fc_stored_ok(bool vec, int in, int out, const uint16_t* x16, const uint16_t* dy16) {
  return g_bf16 && vec && x16 && dy16 && fc_bf16_stored_ok(in, out) && aligned16(x16) && aligned16(dy16);
}
bool fc_bwd_weight_updates(int B, int in, int out, const float* x, const float* dy, const uint16_t* x16, const uint16_t* dy16) {
  const bool vec = vec_ok(dy, out) && vec_ok(x, in);
  return g_bf16 ? fc_stored_ok(vec, in, out, x16, dy16) : fc_split_ok(vec, B);
}
int launch_fc_bwd_weight(int B, int in, int out, const float* x, const float* dy, float* dw, hipStream_t st,
                         const uint16_t* x16, const uint16_t* dy16, const SgdArgs* u) {
  DenseParams a{dy, out, 0, out, (uint32_t)((size_t)B * out * 4)};
  DenseParams b{x, in, 0, in, (uint32_t)((size_t)B * in * 4)};
  EpiSlab ep{dw, (long)out * in, in, nullptr};
  const bool vec = vec_ok(dy, out) && vec_ok(x, in);
  if (u && !fc_bwd_weight_updates(B, in, out, x, dy, x16, dy16)) {
    set_error("fc weight gradient: no kernel updates these weights");
    return ALEXNET_EINVAL;
  }
  if (fc_stored_ok(vec, in, out, x16, dy16)) return launch_direct_dense_bwd_weight(B, in, out, x16, dy16, dw, st, u);
  if (g_bf16 && vec)
    return launch_tile_bf<B128, BfDenseR, BfDenseR, EpiSlab>(a, b, ep, out, in, B, round_up(B, kBKbf), 1, 1, st);
  const GemmPlan p = fc_split_ok(vec, B) ? plan_split(out, in, B, 1, 0, 1) : GemmPlan{128, 128, 1, round_up(B, kBK)};
  if (u) {
    // weights and momentum are read and written beside the gradient
    const AlgoFlops af(2.0 * B * in * (double)out, 4.0 * ((double)B * (in + out) + 5.0 * in * (double)out));
    return by_tile_split<SplitRowInner, SplitRowInner>(p, a, b, EpiSgd{dw, u->w, u->v, in, u->lr, u->mu, u->wd}, out, in, B, 1, st);
  }
  return launch_dense<SplitRowInner, SplitRowInner, DenseRowInner, DenseRowInner>(vec, p, a, b, ep, out, in, B, st);
}

}  // namespace ax
