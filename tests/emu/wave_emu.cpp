// CPU emulation of the small products' workgroup program (csrc/gemm_wave.h): its tables and loaders run lane by lane, the
// eight values of a lane are multiplied as the matrix core's definition has them, and the sums are compared with plain loops.
// Built with -fsanitize=address,undefined and operands of exact size, so an access outside one aborts here.  Also the masks
// of taps inside the tensor and the walk over the taps (csrc/gemm_direct.h), against their definition.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <vector>

struct float4 {
  float x, y, z, w;
};
inline float4 make_float4(float x, float y, float z, float w) { return float4{x, y, z, w}; }
#define AX_HOST_EMU 1
#include "../../paper_1412_2302_amd/csrc/conv_plan.h"
namespace ax {
inline void emu_fail(const char* what) {
  fprintf(stderr, "EMULATION FAULT: %s\n", what);
  abort();
}
}  // namespace ax

#include "../../paper_1412_2302_amd/csrc/gemm_direct.h"
#include "../../paper_1412_2302_amd/csrc/gemm_wave.h"

using namespace ax;

static int failures = 0;
static float frand() { return (float)rand() / RAND_MAX * 2.f - 1.f; }
static float* filled(long n) {
  float* p = new float[n];
  for (long i = 0; i < n; ++i) p[i] = frand();
  return p;
}

// out[group][slice][m][n], as EpiSlab has it
template <class AL, class BL, bool EXACT = false>
static std::vector<double> product(const typename AL::Params& ap, const typename BL::Params& bp, int M, int N, int K, int groups,
                                   int ns) {
  const int kchunk = ((K + 15) / 16 + ns - 1) / ns * 16, threads = 64 * 4;
  std::vector<double> out((size_t)groups * ns * M * N, 0.0);
  for (int g = 0; g < groups; ++g)
    for (int z = 0; z < ns; ++z) {
      const int kbeg = std::min(K, z * kchunk), kend = std::min(K, kbeg + kchunk), len = kend - kbeg;
      std::vector<uint32_t> ta(AL::kWords, 0xdeadbeefu), tb(BL::kWords, 0xdeadbeefu);
      for (int t = 0; t < threads; ++t) {
        AL::build(ap, ta.data(), kbeg, kend, t, threads);
        BL::build(bp, tb.data(), kbeg, kend, t, threads);
      }
      double* slab = out.data() + ((size_t)g * ns + z) * M * N;
      for (int m0 = 0; m0 < M; m0 += kWaveTile)
        for (int n0 = 0; n0 < N; n0 += kWaveTile)
          for (int k = 0; k < len; k += 16) {
            float a[32][16], b[32][16];
            for (int lane = 0; lane < 64; ++lane) {
              const int row = lane & 31, kh = 8 * (lane >> 5);
              float4 ra[2], rb[2];
              const AL al(ap, g, m0 + row, kbeg, kend, ta.data());
              if (EXACT) wave_load_exact(al, ra, k + kh, 0);
              else al.load(ra, k + kh);
              BL(bp, g, n0 + row, kbeg, kend, tb.data()).load(rb, k + kh);
              memcpy(&a[row][kh], ra, 32);
              memcpy(&b[row][kh], rb, 32);
            }
            for (int m = 0; m < std::min(32, M - m0); ++m)
              for (int n = 0; n < std::min(32, N - n0); ++n)
                for (int e = 0; e < 16; ++e) slab[(size_t)(m0 + m) * N + n0 + n] += (double)a[m][e] * b[n][e];
          }
    }
  return out;
}
static void check(const char* what, const ConvGeom& c, const std::vector<double>& slabs, const std::vector<double>& want,
                  int ns) {
  const size_t slab = slabs.size() / (c.groups * ns);
  double worst = 0, top = 0;
  for (int g = 0; g < c.groups; ++g)
    for (size_t i = 0; i < slab; ++i) {
      double s = 0;
      for (int z = 0; z < ns; ++z) s += slabs[((size_t)g * ns + z) * slab + i];
      worst = std::max(worst, fabs(s - want[g * slab + i]));
      top = std::max(top, fabs(want[g * slab + i]));
    }
  const bool ok = worst <= 1e-12 * top;  // both in 64 bits
  if (!ok) ++failures;
  printf("%-12s %dx%dx%d k%d s%d p%d g%d slices %d: %.2e %s\n", what, c.Cin, c.H, c.Cout, c.k, c.stride, c.pad, c.groups, ns,
         worst / top, ok ? "ok" : "FAIL");
}

static void conv(ConvGeom c, int ns) {
  c.Ho = (c.H + 2 * c.pad - c.k) / c.stride + 1;
  c.Wo = (c.W + 2 * c.pad - c.k) / c.stride + 1;
  const int cg = c.cg(), og = c.og();
  float *x = filled(c.in_elems()), *wf = filled(c.w_elems()), *dy = filled(c.out_elems());
  // [group][pixel][o], [group][pixel][c], [group][(r, s, c)][o]
  std::vector<double> y((size_t)c.P() * c.Cout, 0.0), dx((size_t)c.in_elems(), 0.0), dw(c.w_elems(), 0.0);
  for (int g = 0; g < c.groups; ++g)
    for (long p = 0; p < c.P(); ++p)
      for (int r = 0; r < c.k; ++r)
        for (int s = 0; s < c.k; ++s) {
          const int n = (int)(p / (c.Ho * c.Wo)), iy = (int)(p / c.Wo % c.Ho) * c.stride - c.pad + r;
          const int ix = (int)(p % c.Wo) * c.stride - c.pad + s;
          if (iy < 0 || ix < 0 || iy >= c.H || ix >= c.W) continue;
          const long q = ((long)n * c.H + iy) * c.W + ix;
          for (int i = 0; i < cg; ++i)
            for (int o = 0; o < og; ++o) {
              const long w = ((long)g * c.kf() + (r * c.k + s) * cg + i) * og + o;
              const double xv = x[q * c.Cin + g * cg + i], dv = dy[p * c.Cout + g * og + o];
              y[((size_t)g * c.P() + p) * og + o] += xv * wf[w];
              dx[((size_t)g * c.Q() + q) * cg + i] += dv * wf[w];
              dw[w] += xv * dv;
            }
        }
  DenseParams wb = fwd_B(c, wf), gb = bwdw_B(c, dy);
  wb.bytes = (uint32_t)(c.w_elems() / c.groups * 4);  // of a group
  gb.bytes -= (uint32_t)(c.Cout - og) * 4u;           // what lies behind the last group's origin
  const GemmDims f = fwd_dims(c), d = bwdd_dims(c), w = bwdw_dims(c);
  if (run_mode(c)) {
    const WaveRunParams rb{DenseParams{wf, c.Cout, 0, c.Cout, (uint32_t)(c.w_elems() * 4)}, c.k * c.Cin, run_len(c),
                           make_fastdiv((uint32_t)run_len(c))};
    const WaveRunAParams ra{run_A(c, x), c.k * c.Cin};
    check("run forward", c, product<WaveRunA, WaveRunB>(ra, rb, f.M, f.N, run_k(c), 1, ns), y, ns);
    check("run exact", c, product<WaveRunA, WaveRunB, true>(ra, rb, f.M, f.N, run_k(c), 1, ns), y, ns);
  } else if (cg % 4 == 0) {
    check("forward", c, product<WaveIm2col<IM2COL_FWD>, WaveRow>(fwd_A(c, x), wb, f.M, f.N, f.K, f.groups, ns), y, ns);
  }
  if (c.stride == 1 && og % 4 == 0) {
    const WaveTapParams tb{DenseParams{wf, og, (long)c.kf() * og, cg, wb.bytes}, cg, og, make_fastdiv((uint32_t)og)};
    check("data", c, product<WaveIm2col<IM2COL_T1>, WaveTapB>(bwdd_A(c, dy), tb, d.M, d.N, d.K, d.groups, ns), dx, ns);
  }
  if (c.P() <= kWaveMaxPixels * ns)
    check("weight", c, product<WaveIm2colT, WaveRow>(fwd_A(c, x), gb, w.M, w.N, w.K, w.groups, ns), dw, ns);
  delete[] x; delete[] wf; delete[] dy;
}

template <bool VEC>
static void dense(int B, int in, int out) {
  float *x = filled((long)B * in), *w = filled((long)in * out), *dy = filled((long)B * out);
  const ConvGeom c{B, 1, 1, in, out, 1, 1, 0, 1, 1, 1};
  std::vector<double> y((size_t)B * out, 0.0), dx((size_t)B * in, 0.0), dw((size_t)out * in, 0.0);
  for (int b = 0; b < B; ++b)
    for (int o = 0; o < out; ++o)
      for (int i = 0; i < in; ++i) {
        y[b * out + o] += (double)x[b * in + i] * w[o * in + i];
        dx[b * in + i] += (double)dy[b * out + o] * w[o * in + i];
        dw[o * in + i] += (double)dy[b * out + o] * x[b * in + i];
      }
  const DenseParams xk{x, in, 0, B, (uint32_t)(B * in * 4)}, wk{w, in, 0, out, (uint32_t)(in * out * 4)};
  const DenseParams dk{dy, out, 0, B, (uint32_t)(B * out * 4)}, wr{w, in, 0, in, (uint32_t)(in * out * 4)};
  const DenseParams dr{dy, out, 0, out, (uint32_t)(B * out * 4)}, xr{x, in, 0, in, (uint32_t)(B * in * 4)};
  check("dense", c, product<WaveK<VEC>, WaveK<VEC>>(xk, wk, B, out, in, 1, 1), y, 1);
  if (!VEC || out % 4 == 0) check("dense data", c, product<WaveK<VEC>, WaveRow>(dk, wr, B, in, out, 1, 1), dx, 1);
  check("dense weight", c, product<WaveRow, WaveRow>(dr, xr, out, in, B, 1, 1), dw, 1);
  delete[] x; delete[] w; delete[] dy;
}

static void masks() {
  long bad = 0, seen = 0;
  for (int k = 1; k <= 5; ++k)
    for (int H = 1; H <= 7; ++H)
      for (int W = 1; W <= 7; ++W)
        for (int y0 = -6; y0 <= 12; ++y0)
          for (int x0 = -6; x0 <= 12; ++x0) {
            Im2colParams g{};
            g.H = H; g.W = W; g.kh = g.kw = k;
            uint32_t fwd = 0, back = 0;
            for (int r = 0; r < k; ++r)
              for (int s = 0; s < k; ++s) {
                const uint32_t bit = 1u << (r * k + s);
                if (y0 + r >= 0 && y0 + r < H && x0 + s >= 0 && x0 + s < W) fwd |= bit;
                if (y0 - r >= 0 && y0 - r < H && x0 - s >= 0 && x0 - s < W) back |= bit;
              }
            bad += taps_inside<IM2COL_FWD>(g, y0, x0) != fwd;
            bad += taps_inside<IM2COL_T1>(g, y0, x0) != back;
            ++seen;
          }
  failures += bad != 0;
  printf("masks: %ld, %ld wrong\n", 2 * seen, bad);
}

// k-tile by k-tile from every first one, against the division of k
template <bool ONE_TAP>
static void walk(int Cg, int k, int W) {
  Im2colParams g{};
  g.W = W; g.kh = g.kw = k; g.Cg = Cg; g.Ctot = 2 * Cg;
  g.d_cg = make_fastdiv((uint32_t)Cg); g.d_kw = make_fastdiv((uint32_t)k);
  const int K = k * k * Cg;
  long bad = 0, seen = 0;
  for (int first = 0; first * kBKd < K; ++first)
    for (int oct = 0; oct < (ONE_TAP ? 1 : 8); ++oct) {
      int at = first * kBKd + 8 * oct;
      for (TapWalk<ONE_TAP> w(g, at); at < K; at += kBKd, w.next(g), ++seen) {
        const TapCoord t = decode_tap(at, g);
        bad += w.ch != t.c || w.bit != t.r * k + t.s || w.offset(g) != ((uint32_t)t.r * W + t.s) * g.Ctot * 2u;
      }
    }
  failures += bad != 0;
  printf("walk of %d channels, %dx%d: %ld, %ld wrong\n", Cg, k, k, seen, bad);
}

int main() {
  srand(5);
  // B, H, W, Cin, Cout, k, stride, pad, groups
  conv({2, 17, 17, 3, 10, 5, 2, 0, 1, 0, 0}, 1);
  conv({3, 14, 14, 2, 6, 3, 1, 0, 1, 0, 0}, 2);
  conv({2, 9, 11, 1, 33, 3, 1, 0, 1, 0, 0}, 1);
  conv({1, 19, 19, 3, 9, 13, 2, 0, 1, 0, 0}, 3);
  conv({2, 7, 7, 20, 36, 3, 1, 1, 1, 0, 0}, 1);
  conv({2, 7, 7, 36, 44, 3, 1, 2, 4, 0, 0}, 2);
  conv({3, 5, 5, 44, 28, 3, 1, 0, 2, 0, 0}, 1);
  conv({1, 9, 9, 8, 16, 15, 1, 7, 2, 0, 0}, 4);
  conv({5, 1, 1, 32, 40, 3, 1, 1, 1, 0, 0}, 1);
  conv({2, 11, 8, 12, 24, 4, 3, 2, 3, 0, 0}, 2);
  conv({2, 6, 6, 3, 8, 3, 1, 1, 1, 0, 0}, 1);
  conv({4, 33, 33, 4, 4, 2, 1, 0, 1, 0, 0}, 3);
  dense<true>(6, 72, 36);
  dense<true>(33, 40, 200);
  dense<false>(5, 37, 11);
  dense<false>(17, 10, 33);
  masks();
  for (int k = 1; k <= 5; ++k) {
    for (int cg = 8; cg <= 136; cg += 8) walk<false>(cg, k, k + 3);
    for (int cg = 64; cg <= 192; cg += 64) walk<true>(cg, k, k);
  }
  printf(failures ? "FAILURES: %d\n" : "ALL OK\n", failures);
  return failures != 0;
}
