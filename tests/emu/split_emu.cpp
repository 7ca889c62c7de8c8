// CPU emulation of the workgroup program in csrc/gemm_split.h: the real loaders, three-way splits, LDS stores and
// fragment index maps run thread by thread with the MFMA replaced by its definition, and the products are compared
// with plain double-precision loops.  Built with -fsanitize=address,undefined, so an access outside an operand or an
// LDS tile aborts here.  Also checks that the split is exact.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <vector>

struct float4 {
  float x, y, z, w;
};
#define AX_HOST_EMU 1
#include "../../paper_1412_2302_amd/csrc/conv_plan.h"
namespace ax {
inline void emu_fail(const char* what) {
  fprintf(stderr, "EMULATION FAULT: %s\n", what);
  abort();
}
}  // namespace ax

#include "../../paper_1412_2302_amd/csrc/gemm16.h"

using namespace ax;

static int failures = 0;
static bool force_redo = false;  // every tile a second time, as if its sums were not finite
static float frand() { return (float)rand() / RAND_MAX * 2.f - 1.f; }

template <class T, class AL, class BL, class Epi>
static void emu_split(typename AL::Params ap, typename BL::Params bp, Epi ep, int M, int N, int K, int kchunk,
                      int nsplit, int groups, SplitGrid grid = {}, const std::vector<int>& only = {}) {
  grid.nsplit = make_fastdiv((uint32_t)nsplit);
  const int gx = (M + T::BM - 1) / T::BM, gy = (N + T::BN - 1) / T::BN, gz = groups * nsplit;
  std::vector<uint32_t> As(AL::UNITS * 4), Bs(BL::UNITS * 4);
  std::vector<float> acc((size_t)T::BM * T::BN), lo(acc.size());
  for (int bz = 0; bz < gz; ++bz)
    for (int by = 0; by < gy; ++by)
      for (int bx = 0; bx < gx; ++bx) {
        const int turn = bz / nsplit, split = bz - turn * nsplit, g = (int)split_group(grid, (uint32_t)turn);
        if (!only.empty() && std::find(only.begin(), only.end(), g) == only.end()) continue;
        const int n0 = by * T::BN;
        const SplitPlace at = split_place<T>(grid, (uint32_t)g, split, bx * T::BM, M, K, kchunk);
        const int m0 = at.m0, kbeg = at.kbeg, kend = at.kend;
        typename AL::Params mine = ap;
        if (grid.of == 1) {
          if (m0 >= at.M) continue;
          split_row_limit(mine, at.M);
        }
        const int nt = kend > kbeg ? (kend - kbeg + T::BK - 1) / T::BK : 0;
        std::fill(acc.begin(), acc.end(), 0.f);
        std::fill(lo.begin(), lo.end(), 0.f);
        Epi e = ep;
        e.set_group(g, g * nsplit + split);
        for (int t = 0; t < nt; ++t) {
          std::fill(As.begin(), As.end(), 0x7fc07fc0u);  // two bf16 NaNs: an unwritten slot shows up
          std::fill(Bs.begin(), Bs.end(), 0x7fc07fc0u);
          for (int tid = 0; tid < kThreads; ++tid) {
            AL al(mine, g, tid, m0, kbeg);
            BL bl(bp, g, tid, n0, kbeg);
            float4 ra[AL::NL], rb[BL::NL];
            for (int u = 0; u <= t; ++u) {  // offsets run along with k
              al.fetch(ra, kend - kbeg - u * T::BK);
              bl.fetch(rb, kend - kbeg - u * T::BK);
            }
            split_store_all(al, As.data(), ra);
            split_store_all(bl, Bs.data(), rb);
          }
          // fragments as the kernel addresses them: the unit of the wave's first block, block t further on
          auto val = [](const std::vector<uint32_t>& lds, int unit, int e) {
            const uint32_t w = lds.at((size_t)unit * 4 + e / 2);
            return (e & 1) ? bf_hi(w) : bf_lo(w);
          };
          for (int i = 0; i < T::BM; ++i)
            for (int j = 0; j < T::BN; ++j) {
              const int wa = i / (T::TM * 32), ta = i / 32 % T::TM, wb = j / (T::TN * 32), tb = j / 32 % T::TN;
              for (int q = 0; q < kSplitProducts; ++q) {
                float& c = (q == 0 ? acc : lo)[(size_t)i * T::BN + j];
                float s = 0.f;
                for (int kh = 0; kh < 2; ++kh) {
                  const int ua = split_unit<AL>(0, kh, wa * (T::TM * 32) + i % 32) + split_plane_a(q) * 2 * AL::RP + AL::block_units(ta);
                  const int ub = split_unit<BL>(0, kh, wb * (T::TN * 32) + j % 32) + split_plane_b(q) * 2 * BL::RP + BL::block_units(tb);
                  for (int x = 0; x < 8; ++x) s += val(As, ua, x) * val(Bs, ub, x);
                }
                c += s;
              }
            }
        }
        bool redo = force_redo;
        for (size_t i = 0; i < acc.size(); ++i) {
          acc[i] = (acc[i] + lo[i]) * kSplitUnscale;
          redo = redo || !std::isfinite(acc[i]);
        }
        if (redo) std::fill(acc.begin(), acc.end(), 0.f);
        for (int t = 0; redo && t < nt; ++t) {
          std::fill(As.begin(), As.end(), 0x7fc00000u);
          std::fill(Bs.begin(), Bs.end(), 0x7fc00000u);
          float *ar = reinterpret_cast<float*>(As.data()), *br = reinterpret_cast<float*>(Bs.data());
          for (int tid = 0; tid < kThreads; ++tid) {
            AL al(mine, g, tid, m0, kbeg);
            BL bl(bp, g, tid, n0, kbeg);
            float4 ra[AL::NL], rb[BL::NL];
            for (int u = 0; u <= t; ++u) {
              al.fetch(ra, kend - kbeg - u * T::BK);
              bl.fetch(rb, kend - kbeg - u * T::BK);
            }
            raw_store_all(al, ar, ra);
            raw_store_all(bl, br, rb);
          }
          for (int i = 0; i < T::BM; ++i)
            for (int j = 0; j < T::BN; ++j)
              for (int k = 0; k < T::BK; k += 2)
                acc[(size_t)i * T::BN + j] += ar[i * kRawLd + k] * br[j * kRawLd + k] + ar[i * kRawLd + k + 1] * br[j * kRawLd + k + 1];
        }
        for (int i = 0; i < T::BM && m0 + i < at.M; ++i)
          for (int j = 0; j < T::BN && n0 + j < N; ++j) e.apply(m0 + i, n0 + j, acc[(size_t)i * T::BN + j]);
      }
}

static void check(const char* what, int M, int N, int K, const std::vector<float>& got, const std::vector<double>& want) {
  double num = 0, den = 0;
  bool nan = false;
  for (size_t i = 0; i < want.size(); ++i) {
    if (!(got[i] == got[i])) nan = true;
    num += (got[i] - want[i]) * (got[i] - want[i]);
    den += want[i] * want[i];
  }
  const double rel = sqrt(num / (den > 0 ? den : 1));
  const bool ok = !nan && rel < 5e-7;  // fp32 accumulation; a lost or doubled term pair is at least 2^-17
  printf("%-10s %4d x %4d x %4d rel_l2=%.3e %s\n", what, M, N, K, rel, ok ? "ok" : "FAIL");
  if (!ok) ++failures;
}

static void split_is_exact() {
  long bad = 0;
  for (int i = 0; i < 2000000; ++i) {
    uint32_t u = ((uint32_t)rand() << 16) ^ (uint32_t)rand() ^ ((uint32_t)rand() << 31);
    const int e = (u >> 23) & 255;
    if (e >= 127 + 103) continue;  // the first term stays finite
    float x;
    memcpy(&x, &u, 4);
    const SplitPair s = split_pair(x, -x);
    if ((double)bf_lo(s.t[0]) + bf_lo(s.t[1]) + bf_lo(s.t[2]) != (double)x * kSplitScale) ++bad;
    if ((double)bf_hi(s.t[0]) + bf_hi(s.t[1]) + bf_hi(s.t[2]) != -(double)x * kSplitScale) ++bad;
  }
  const SplitPair z = split_pair(0.f, -0.f);
  for (int p = 0; p < kPlanes; ++p)
    if (bf_lo(z.t[p]) != 0.f || bf_hi(z.t[p]) != 0.f) ++bad;
  // an operand the terms cannot hold leaves a NaN among them, which no product loses: that is how it is found
  for (float x : {INFINITY, 2.028240961e31f, 3.4028235e38f, (float)NAN}) {
    const SplitPair s = split_pair(x, -x);
    if (!std::isnan(bf_lo(s.t[2])) || !std::isnan(bf_hi(s.t[2]))) ++bad;
  }
  printf("exact split %s\n", bad ? "FAIL" : "ok");
  if (bad) ++failures;
}

// M x N x K with the operands of the four kinds of product: A and B contiguous along k or along their rows;
// ns slices of the reduction, ng groups side by side in memory (the layout of the transformed convolutions)
template <class T>
static void dense_case(int M, int N, int K, int ns, int ng) {
  typedef SplitKInner<T::BM> AK;
  typedef SplitRowInner<T::BM> AR;
  typedef SplitRowInner<T::BN> BR;
  // exact-size heap buffers: the sanitizer flags any access past either end
  float *a = new float[(size_t)M * K * ng], *b = new float[(size_t)K * N * ng];
  for (size_t i = 0; i < (size_t)M * K * ng; ++i) a[i] = frand();
  for (size_t i = 0; i < (size_t)K * N * ng; ++i) b[i] = frand();
  const int ktiles = (K + 15) / 16, kc = (ktiles + ns - 1) / ns * 16;
  const long slab = (long)M * N;
  auto run = [&](const char* what, bool a_k, bool b_k) {
    std::vector<double> ref(slab * ng, 0.0);
    // groups side by side along k (a_k: a[m][g*K + k]) or along rows (a[k][g*M + m]); b_k: b[g][n][k], else b[g][k][n]
    auto A = [&](int g, int m, int k) { return (double)(a_k ? a[(size_t)m * K * ng + g * K + k] : a[((size_t)k * ng + g) * M + m]); };
    auto Bv = [&](int g, int k, int n) { return (double)(b_k ? b[((size_t)g * N + n) * K + k] : b[((size_t)g * K + k) * N + n]); };
    for (int g = 0; g < ng; ++g)
      for (int m = 0; m < M; ++m)
        for (int n = 0; n < N; ++n)
          for (int k = 0; k < K; ++k) ref[(g * (size_t)M + m) * N + n] += A(g, m, k) * Bv(g, k, n);
    std::vector<float> ws((size_t)slab * ns * ng, NAN), c(slab * ng, 0.f);
    DenseParams pa{a, a_k ? (long)K * ng : (long)M * ng, a_k ? K : M, M, (uint32_t)((size_t)M * K * ng * 4)};
    DenseParams pb{b, b_k ? K : N, (long)K * N, N, (uint32_t)((size_t)K * N * ng * 4)};
    EpiSlab e{ws.data(), slab, N, nullptr};
    if (a_k && b_k) {
      emu_split<T, AK, SplitKInner<T::BN>, EpiSlab>(pa, pb, e, M, N, K, kc, ns, ng);
    } else if (a_k) {
      emu_split<T, AK, BR, EpiSlab>(pa, pb, e, M, N, K, kc, ns, ng);
    } else {
      emu_split<T, AR, BR, EpiSlab>(pa, pb, e, M, N, K, kc, ns, ng);
    }
    for (int g = 0; g < ng; ++g)
      for (int s = 0; s < ns; ++s)
        for (long i = 0; i < slab; ++i) c[g * slab + i] += ws[((size_t)g * ns + s) * slab + i];
    check(what, M, N, K, c, ref);
  };
  run("k,k", true, true);
  run("k,rows", true, false);
  run("rows,rows", false, false);
  delete[] a;
  delete[] b;
}

// Products of a transformed layer with short tiles: rows (of 1) or the reduction (of 2) run over the rows of a group's position only.
// What lies outside those is NaN, in operands and results, and stays so.
template <class T>
static void short_case(int of, int short_y, int whole, int short_x, int both, int G, int K, int N, int ns) {
  const int tiles = short_y + whole + short_x + both, Z = 36 * G;
  const std::vector<int> groups = {0, 2 * G, 3 * G + G - 1, 18 * G, 35 * G + G - 1};  // both in, once more, row only, column only, neither
  SplitGrid grid{};
  grid.of = of;
  grid.positions = make_fastdiv((uint32_t)G);
  grid.short_y = short_y; grid.whole = whole; grid.short_x = short_x; grid.tiles = tiles;
  std::vector<float> a((size_t)tiles * Z * K, NAN), b(of == 1 ? (size_t)Z * K * N : (size_t)tiles * Z * N, NAN);
  for (int g : groups) {
    const RowRange r = wino_rows(g / G, short_y, whole, short_x, tiles);
    for (int t = r.lo; t < r.hi; ++t)
      for (int k = 0; k < K; ++k) a[((size_t)t * Z + g) * K + k] = frand();
    if (of == 1)
      for (size_t i = 0; i < (size_t)K * N; ++i) b[(size_t)g * K * N + i] = frand();
    else
      for (int t = r.lo; t < r.hi; ++t)
        for (int n = 0; n < N; ++n) b[((size_t)t * Z + g) * N + n] = frand();
  }
  std::vector<float> got;
  std::vector<double> want;
  if (of == 1) {  // c[t][g][n] = sum_k a[t][g][k] b[g][k][n]
    std::vector<float> c((size_t)tiles * Z * N, NAN);
    const DenseParams pa{a.data(), (long)Z * K, K, tiles, (uint32_t)(a.size() * 4)}, pb{b.data(), N, (long)K * N, N, (uint32_t)(b.size() * 4)};
    emu_split<T, SplitKInner<T::BM>, SplitRowInner<T::BN>, EpiBiasAct>(pa, pb, EpiBiasAct{c.data(), (long)Z * N, nullptr, 0, N, 0, 0, nullptr},
                                                                       tiles, N, K, (K + 15) / 16 * 16, 1, Z, grid, groups);
    for (int g : groups) {
      const RowRange r = wino_rows(g / G, short_y, whole, short_x, tiles);
      for (int t = 0; t < tiles; ++t)
        for (int n = 0; n < N; ++n) {
          const float v = c[((size_t)t * Z + g) * N + n];
          if (t < r.lo || t >= r.hi) {
            if (!std::isnan(v)) ++failures, printf("short rows FAIL: row %d of group %d was written\n", t, g);
            continue;
          }
          double s = 0;
          for (int k = 0; k < K; ++k) s += (double)a[((size_t)t * Z + g) * K + k] * b[((size_t)g * K + k) * N + n];
          got.push_back(v);
          want.push_back(s);
        }
    }
  } else {  // c[g][k][n] = sum_t a[t][g][k] b[t][g][n], in slices
    const long slab = (long)K * N;
    std::vector<float> c((size_t)Z * ns * slab, NAN);
    const DenseParams pa{a.data(), (long)Z * K, K, K, (uint32_t)(a.size() * 4)}, pb{b.data(), (long)Z * N, N, N, (uint32_t)(b.size() * 4)};
    emu_split<T, SplitRowInner<T::BM>, SplitRowInner<T::BN>, EpiSlab>(pa, pb, EpiSlab{c.data(), slab, N, nullptr}, K, N, tiles,
                                                                      (tiles + 16 * ns - 1) / (16 * ns) * 16, ns, Z, grid, groups);
    for (int g : groups) {
      const RowRange r = wino_rows(g / G, short_y, whole, short_x, tiles);
      for (long i = 0; i < slab; ++i) {
        float v = 0.f;
        for (int z = 0; z < ns; ++z) v += c[((size_t)g * ns + z) * slab + i];
        double s = 0;
        for (int t = r.lo; t < r.hi; ++t) s += (double)a[((size_t)t * Z + g) * K + i / N] * b[((size_t)t * Z + g) * N + i % N];
        got.push_back(v);
        want.push_back(s);
      }
    }
  }
  check(of == 1 ? "short rows" : "short sums", tiles, N, K, got, want);
}

// first-layer shapes in run mode: forward and weight gradient of an unpadded convolution over three-channel pictures
template <class T>
static void run_case(int B, int H, int W, int Cout, int k, int st, int ns) {
  ConvGeom c;
  c.B = B; c.H = H; c.W = W; c.Cin = 3; c.Cout = Cout; c.k = k; c.stride = st; c.pad = 0; c.groups = 1;
  c.Ho = (H - k) / st + 1;
  c.Wo = (W - k) / st + 1;
  const int run = run_len(c), kc = k * 3, K = run_k(c), P = (int)c.P();
  if (!run_mode(c) || run < 16 || c.Wo < 16) emu_fail("not a case of the run loaders");
  float *x = new float[c.in_elems()], *w = new float[run_w_elems(c)], *dy = new float[c.out_elems()];
  for (long i = 0; i < c.in_elems(); ++i) x[i] = frand();
  for (long i = 0; i < c.out_elems(); ++i) dy[i] = frand();
  for (int r = 0; r < k; ++r)
    for (int j = 0; j < run; ++j)
      for (int o = 0; o < Cout; ++o) w[((long)r * run + j) * Cout + o] = j < kc ? frand() : 0.f;
  std::vector<double> y_ref(c.out_elems(), 0.0), dw_ref(run_w_elems(c), 0.0);
  for (int p = 0; p < P; ++p) {
    const int n = p / (c.Ho * c.Wo), oy = p / c.Wo % c.Ho, ox = p % c.Wo;
    for (int r = 0; r < k; ++r)
      for (int j = 0; j < kc; ++j) {
        const double v = x[(((long)n * H + oy * st + r) * W + ox * st) * 3 + j];
        for (int o = 0; o < Cout; ++o) {
          y_ref[(long)p * Cout + o] += v * w[((long)r * run + j) * Cout + o];
          dw_ref[((long)r * run + j) * Cout + o] += v * dy[(long)p * Cout + o];
        }
      }
  }
  auto chunk = [&](int len) { return ((len + 15) / 16 + ns - 1) / ns * 16; };
  {
    std::vector<float> ws((size_t)ns * c.out_elems(), NAN), y(c.out_elems(), 0.f);
    EpiSlab e{ws.data(), (long)P * Cout, Cout, nullptr};
    emu_split<T, SplitRun<T::BM>, SplitRowInner<T::BN>, EpiSlab>(run_A(c, x), run_B(c, w), e, P, Cout, K, chunk(K), ns, 1);
    for (int s = 0; s < ns; ++s)
      for (long i = 0; i < c.out_elems(); ++i) y[i] += ws[s * c.out_elems() + i];
    check("run fwd", P, Cout, K, y, y_ref);
  }
  {  // rows of the weight gradient: whole quads of every kernel row, then the floats left over
    const int M = k * kc, head = kc / 4 * 4, left = kc - head;
    std::vector<float> ws((size_t)ns * M * Cout, NAN), dw(run_w_elems(c), 0.f);
    EpiSlab e{ws.data(), (long)M * Cout, Cout, nullptr};
    emu_split<T, SplitRunT<T::BM>, SplitRowInner<T::BN>, EpiSlab>(run_t_params(run_A(c, x), kc), bwdw_B(c, dy), e, M, Cout, P, chunk(P), ns, 1);
    for (int m = 0; m < M; ++m) {
      const int r = m < k * head ? m / head : (m - k * head) / left, j = m < k * head ? m % head : head + (m - k * head) % left;
      for (int s = 0; s < ns; ++s)
        for (int o = 0; o < Cout; ++o) dw[((long)r * run + j) * Cout + o] += ws[((long)s * M + m) * Cout + o];
    }
    check("run bwd_w", M, Cout, P, dw, dw_ref);
  }
  delete[] x; delete[] w; delete[] dy;
}

// gemm16.h: a 3x3 layer over bf16 tensors, one tap per k-tile, LDS units of eight k
template <class T, int MODE>
static void conv16_case(int B, int H, int Cin, int Cout, int groups) {
  ConvGeom c;
  c.B = B; c.H = H; c.W = H + 1; c.Cin = Cin; c.Cout = Cout; c.k = 3; c.stride = 1; c.pad = 1; c.groups = groups;
  c.Ho = c.H;
  c.Wo = c.W;
  typedef Unit16<Im2colKTap16<T::BM, T::BK, MODE>, T::BM, T::BK> AL;
  typedef Unit16<DenseKInner16<T::BN, T::BK>, T::BN, T::BK> BL;
  const bool fwd = MODE == IM2COL_FWD;
  const GemmDims d = fwd ? fwd_dims(c) : bwdd_dims(c);
  const long nx = fwd ? c.in_elems() : c.out_elems();
  uint16_t *x = new uint16_t[nx], *w = new uint16_t[c.w_elems()];  // w: [g][column][(tap, channel)]
  for (long i = 0; i < nx; ++i) x[i] = (uint16_t)bf16_bits(frand());
  for (long i = 0; i < c.w_elems(); ++i) w[i] = (uint16_t)bf16_bits(frand());
  const Im2colParams ap = im2col16(fwd ? fwd_A(c, nullptr) : bwdd_A(c, nullptr), x);
  const DenseParams bp = fwd ? fwd_B16k(c, w) : bwdd_B16k(c, w);
  const int Ctot = fwd ? Cin : Cout, Cg = Ctot / groups, ncol = fwd ? Cout : Cin;
  std::vector<double> ref((size_t)d.M * ncol, 0.0);
  std::vector<float> y((size_t)d.M * ncol, NAN);
  for (int m = 0; m < d.M; ++m)
    for (int g = 0; g < groups; ++g)
      for (int n = 0; n < d.N; ++n)
        for (int r = 0; r < 3; ++r)
          for (int s = 0; s < 3; ++s) {
            const int py = m / c.W % c.H, px = m % c.W, iy = fwd ? py - 1 + r : py + 1 - r, ix = fwd ? px - 1 + s : px + 1 - s;
            if (iy < 0 || iy >= c.H || ix < 0 || ix >= c.W) continue;
            for (int k = 0; k < Cg; ++k)
              ref[(size_t)m * ncol + g * d.N + n] +=
                  (double)bf_lo(x[(((long)(m / (c.H * c.W)) * c.H + iy) * c.W + ix) * Ctot + g * Cg + k]) *
                  bf_lo(w[((long)g * d.N + n) * d.K + (r * 3 + s) * Cg + k]);
          }
  EpiGate e{y.data(), ncol, nullptr, d.N, 0, 0, nullptr};
  std::vector<uint32_t> As(AL::UNITS * 4), Bs(BL::UNITS * 4);
  for (int g = 0; g < groups; ++g)
    for (int m0 = 0; m0 < d.M; m0 += T::BM)
      for (int n0 = 0; n0 < d.N; n0 += T::BN) {
        std::vector<float> acc((size_t)T::BM * T::BN, 0.f);
        e.set_group(g, g);
        for (int k0 = 0; k0 < d.K; k0 += T::BK) {
          std::fill(As.begin(), As.end(), 0x7fc07fc0u);
          std::fill(Bs.begin(), Bs.end(), 0x7fc07fc0u);
          for (int tid = 0; tid < kThreads; ++tid) {
            AL al(ap, g, tid, m0);
            BL bl(bp, g, tid, n0);
            float4 ra[AL::NL], rb[BL::NL];
            plan_all(al, k0, d.K);
            plan_all(bl, k0, d.K);
            al.fetch(ra);
            bl.fetch(rb);
            split_store_all(al, As.data(), ra);
            split_store_all(bl, Bs.data(), rb);
          }
          for (int i = 0; i < T::BM; ++i)
            for (int j = 0; j < T::BN; ++j)
              for (int o = 0; o < T::BK / 8; ++o)
                for (int q = 0; q < 4; ++q) {
                  const uint32_t a = As.at((o * AL::RP + i) * 4 + q), b = Bs.at((o * BL::RP + j) * 4 + q);
                  acc[(size_t)i * T::BN + j] += bf_lo(a) * bf_lo(b) + bf_hi(a) * bf_hi(b);
                }
        }
        for (int i = 0; i < T::BM && m0 + i < d.M; ++i)
          for (int j = 0; j < T::BN && n0 + j < d.N; ++j) e.apply(m0 + i, n0 + j, acc[(size_t)i * T::BN + j]);
      }
  check(fwd ? "conv16" : "conv16 T", d.M, d.N, d.K, y, ref);
  delete[] x;
  delete[] w;
}

int main() {
  srand(4321);
  SplitGrid spread{};
  spread.of = 1;
  spread.positions = make_fastdiv(3);
  std::vector<int> turns(108, 0);
  for (uint32_t t = 0; t < 108; ++t) ++turns.at(split_group(spread, t));
  if (std::count(turns.begin(), turns.end(), 1) != 108) ++failures, printf("FAIL: a group has no turn of its own\n");
  split_is_exact();
  typedef Tile<128, 128, 16, 2, 2> S128;
  typedef Tile<128, 192, 16, 2, 2> S192;
  typedef Tile<128, 96, 16, 4, 1> S96;
  typedef Tile<128, 64, 16, 2, 2> S64;
  for (int redo = 0; redo < 2; ++redo) {
    force_redo = redo;
    // one tile with room to spare, whole tiles, one row and one quad past a tile; k below, at and past a k-tile
    dense_case<S128>(4, 4, 4, 1, 1);
    dense_case<S128>(128, 128, 32, 1, 2);
    dense_case<S128>(132, 260, 52, 2, 2);
    dense_case<S192>(132, 196, 20, 1, 2);
    dense_case<S192>(64, 192, 48, 3, 3);
    dense_case<S96>(132, 100, 36, 2, 2);
    dense_case<S96>(128, 96, 16, 1, 3);
    dense_case<S64>(60, 68, 36, 2, 2);
    dense_case<Tile<64, 128, 16, 2, 2>>(50, 132, 40, 2, 1);
    short_case<S128>(1, 27, 81, 27, 9, 1, 20, 36, 1);  // a row tile that ends inside a range, and one that starts inside
    short_case<S64>(1, 5, 128, 7, 3, 2, 12, 8, 1);
    short_case<S64>(1, 0, 30, 10, 0, 1, 8, 4, 1);      // one direction only
    short_case<S64>(2, 27, 81, 27, 9, 1, 20, 12, 1);   // sums that start and end between k-tiles
    short_case<S64>(2, 3, 9, 3, 1, 2, 8, 8, 3);        // a slice without a k-tile
    short_case<S64>(2, 10, 50, 0, 0, 1, 8, 8, 4);
    run_case<S96>(2, 75, 76, 96, 11, 4, 1);   // 17 pixels a row: a k-tile crosses a row's end, and a picture's
    run_case<S96>(3, 41, 45, 20, 7, 2, 3);    // runs of 24, slices that start inside a run and inside a row
    run_case<S128>(1, 22, 36, 132, 5, 1, 2);  // runs of 16, 32 pixels a row
    run_case<S96>(2, 40, 44, 20, 8, 2, 2);    // rows of 24 floats, none left over behind the whole quads
    run_case<S96>(2, 38, 42, 100, 6, 2, 1);   // rows of 18 floats, two left over
  }
  conv16_case<Tile<128, 192, 32, 2, 2>, IM2COL_FWD>(3, 7, 64, 384, 2);
  conv16_case<Tile<128, 192, 32, 2, 2>, IM2COL_T1>(3, 7, 384, 128, 2);
  printf(failures ? "FAILED %d\n" : "ALL OK\n", failures);
  return failures ? 1 : 0;
}
