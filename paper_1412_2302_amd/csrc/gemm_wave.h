// Small products: the waves of a workgroup share one 32 x 32 tile of the result and deal its reduction among themselves.
//
// A layer of a small net, or of a single picture, is a few hundred 32 x 32 tiles at most: in 128-row tiles it fills a tenth
// of the chip, its loop of k-tiles is a chain of loads, barriers and LDS stores of about a microsecond a link, and to shorten
// the chain the reduction had to go to slabs that a second launch added up.  Here wave w takes the 16-deep steps w, w + 8, ...
// of the reduction: no operand is shared between the waves, so there is nothing to stage -- every lane loads the eight
// values that it feeds to the matrix core straight from memory, with no barrier in the loop -- and the eight partial tiles meet in LDS once, where they are added in wave order and finished in the same kernel.
//
// Arithmetic: fp32 operands as three bf16 terms, six term products in two sets of accumulators, tiles whose sums are not
// finite computed again with the fp32 matrix instructions, as in gemm_split.h; or both operands rounded to bf16 (BF).
//
// What bounds it: below ten microseconds the launch, the tables and a chain of two or three loads; above, a compute unit's
// tenth of a microsecond per step of a 32 x 32 tile -- 16 values a lane to split, about a hundred vector instructions beside
// six MFMAs, where a 128 x 128 tile shares that work among four times as many, and 4 KB through L2.  Which products take it:
// wave_plan().  Measured, tiles with slices and finishing launches | here: forward of the small nets' 6 x 6 layers at batch
// 16 13.0 | 5.5 us, both gradients of one 26 | 7.5, a whole step 351 | 139 us; mini net at batch 256 636 | 311; in bf16 at
// batch 128 411 | 193; inference of one picture, full net, 145 | 114.
//
#pragma once

#include "conv_plan.h"
#include "gemm_split.h"

namespace ax {

constexpr int kWaveTile = 32;
constexpr int kWaveMaxK = 4096;      // longest reduction over taps and channels
constexpr int kWaveMaxPixels = 2048; // pixels of a weight gradient per workgroup
constexpr int kWaveMaxSide = 15;     // largest kernel side: see TapBits

// ---- loaders --------------------------------------------------------------------
// One row of the operand per lane, rows past the end repeated (their sums are not stored); load(r, k) brings elements (row,
// kbeg + k .. kbeg + k + 7), zero from kend on.  A 16-byte buffer load needs 4-byte alignment only, and an operand spans less
// than 2 GiB.  What an address owes to k alone is worked out once per workgroup, by all threads, into a table in LDS
// (build(), kWords words): with the divisions and 32-bit multiplications in the loop a weight gradient's step took twice
// as long (mini net, batch 128 in bf16: a step of 220 us, 190 with the tables).

// Which taps of a kernel of at most 15 x 15 lie inside the tensor, seen from a pixel: bit r for a row, bit 16 + s for a column;
// a tap needs both of its bits.  Nothing has bits 15 and 31, so ~0 asks for a tap that no pixel has.
constexpr uint32_t kNoTap = 0xffffffffu;
AX_HD uint32_t tap_bits(int r, int s) { return (1u << r) | (0x10000u << s); }
// bits lo .. hi-1, both cut to 0 .. 15
AX_HD uint32_t bit_range(int lo, int hi) {
  lo = lo < 0 ? 0 : lo;
  hi = hi > 15 ? 15 : hi;
  return hi > lo ? (1u << hi) - (1u << lo) : 0u;
}
template <int MODE>
AX_HD uint32_t pixel_taps(const Im2colParams& g, int y0, int x0) {
  if (MODE == IM2COL_FWD) return bit_range(-y0, g.H - y0) | bit_range(-x0, g.W - x0) << 16;
  return bit_range(y0 - g.H + 1, y0 + 1) | bit_range(x0 - g.W + 1, x0 + 1) << 16;
}
AX_HD int wave_steps16(int n) { return (n + 15) / 16 * 16; }

// elem(row, k) = p[row*ld + k]; VEC: K a multiple of four
template <bool VEC>
struct WaveK {
  static constexpr int kWords = 0;
  typedef DenseParams Params;
  BufView v;
  uint32_t base;
  int n;
  AX_HD WaveK(const Params& a, int g, int row, int kbeg, int kend, const uint32_t* /*table*/)
      : v(make_view(a.p + (long)g * a.gstride, a.bytes - (uint32_t)(g * a.gstride * 4))), n(kend - kbeg) {
    row = row < a.R ? row : a.R - 1;
    base = ((uint32_t)row * (uint32_t)a.ld + (uint32_t)kbeg) * 4u;
  }
  static AX_HD void build(const Params&, uint32_t*, int, int, int, int) {}
  AX_HD void load(float4* r, int k) const {
    const uint32_t o = base + (uint32_t)k * 4u;
    if (VEC) {
      r[0] = buf_ld4(v, k < n ? o : kOob);
      r[1] = buf_ld4(v, k + 4 < n ? o + 16u : kOob);
    } else {
      float t[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) t[e] = buf_ld1(v, k + e < n ? o + 4u * e : kOob);
      r[0] = make_float4(t[0], t[1], t[2], t[3]);
      r[1] = make_float4(t[4], t[5], t[6], t[7]);
    }
  }
};

// elem(row, k) = p[k*ld + row]; the extent ends with the group's last k, so that what lies past it reads as zero
struct WaveRow {
  static constexpr int kWords = 0;
  typedef DenseParams Params;
  BufView v;
  uint32_t base, ld4;
  AX_HD WaveRow(const Params& a, int g, int row, int kbeg, int /*kend*/, const uint32_t* /*table*/)
      : v(make_view(a.p + (long)g * a.gstride, a.bytes)), ld4((uint32_t)a.ld * 4u) {
    row = row < a.R ? row : a.R - 1;
    base = (uint32_t)row * 4u + (uint32_t)kbeg * ld4;
  }
  static AX_HD void build(const Params&, uint32_t*, int, int, int, int) {}
  AX_HD void load(float4* r, int k) const {
    const uint32_t o = base + (uint32_t)k * ld4;
    float t[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) t[e] = buf_ld1(v, o + (uint32_t)e * ld4);
    r[0] = make_float4(t[0], t[1], t[2], t[3]);
    r[1] = make_float4(t[4], t[5], t[6], t[7]);
  }
};

// implicit im2col, rows = pixels, k = (r, s, c); channels per group a multiple of four.  Table: per quad of k its byte offset
// from a pixel's origin and the bits of its tap.
template <int MODE>
struct WaveIm2col {
  static_assert(MODE == IM2COL_FWD || MODE == IM2COL_T1, "unit-step gathers only");
  static constexpr int kWords = kWaveMaxK / 4 * 2;
  typedef Im2colParams Params;
  BufView v;
  uint32_t base, taps;
  const uint32_t* table;
  AX_HD WaveIm2col(const Params& a, int grp, int row, int /*kbeg*/, int /*kend*/, const uint32_t* table_)
      : v(make_view(a.x, a.bytes)), table(table_) {
    const PixCoord c = decode_pixel(row < a.P ? row : a.P - 1, a);
    const int y0 = MODE == IM2COL_FWD ? c.y * a.stride - a.pad : c.y + a.pad;
    const int x0 = MODE == IM2COL_FWD ? c.x * a.stride_x - a.pad_x : c.x + a.pad;
    base = row_base<MODE>(a, c.n, y0, x0, grp * a.c_stride_g);
    taps = pixel_taps<MODE>(a, y0, x0);
  }
  static AX_HD void build(const Params& g, uint32_t* table, int kbeg, int kend, int tid, int threads) {
    for (int q = tid; q < wave_steps16(kend - kbeg) / 4; q += threads) {
      const int k = kbeg + 4 * q;
      const TapCoord t = decode_tap(k, g);
      const uint32_t tap = ((uint32_t)t.r * (uint32_t)g.W + (uint32_t)t.s) * (uint32_t)g.Ctot;
      table[2 * q] = ((MODE == IM2COL_FWD ? tap : 0u - tap) + (uint32_t)t.c) * 4u;
      table[2 * q + 1] = k < kend ? tap_bits(t.r, t.s) : kNoTap;
    }
  }
  AX_HD void load(float4* r, int k) const {
    const uint32_t* t = table + k / 2;  // two quads
#pragma unroll
    for (int q = 0; q < 2; ++q) r[q] = buf_ld4(v, (taps & t[2 * q + 1]) == t[2 * q + 1] ? base + t[2 * q] : kOob);
  }
};

// The same with k = a run-mode (r, j < run).  The quad at a run's end may hold floats of the pixels behind the window, of the
// next row's or the next picture's: they meet zero weights, but an infinity or a NaN among them would still reach the sum.
// load_exact() reads them as zero; load(), which costs the small nets' steps 0.7 % less, is for sums that are looked at and
// made again if they are not finite.  Table: also, in an offset's two lowest bits, how many of its floats after the first are
// the window's.
struct WaveRunAParams {
  Im2colParams g;
  int kc;  // floats of a kernel row's window; run = g.Cg: kc rounded up to a multiple of four
};
struct WaveRunA {
  typedef WaveIm2col<IM2COL_FWD> Gather;
  static constexpr int kWords = Gather::kWords;
  typedef WaveRunAParams Params;
  Gather in;
  AX_HD WaveRunA(const Params& a, int grp, int row, int kbeg, int kend, const uint32_t* table)
      : in(a.g, grp, row, kbeg, kend, table) {}
  static AX_HD void build(const Params& p, uint32_t* table, int kbeg, int kend, int tid, int threads) {
    for (int q = tid; q < wave_steps16(kend - kbeg) / 4; q += threads) {
      const int k = kbeg + 4 * q, r = (int)fdiv((uint32_t)k, p.g.d_cg), j = k - r * p.g.Cg, n = p.kc - j;
      table[2 * q] = ((uint32_t)r * (uint32_t)p.g.W + (uint32_t)j) * 4u | (uint32_t)(n < 4 ? n - 1 : 3);
      table[2 * q + 1] = k < kend ? tap_bits(r, 0) : kNoTap;
    }
  }
  AX_HD float4 quad(const uint32_t* t) const {
    return buf_ld4(in.v, (in.taps & t[1]) == t[1] ? in.base + (t[0] & ~3u) : kOob);
  }
  AX_HD void load(float4* r, int k) const {
    const uint32_t* t = in.table + k / 2;
#pragma unroll
    for (int q = 0; q < 2; ++q) r[q] = quad(t + 2 * q);
  }
  AX_HD void load_exact(float4* r, int k) const {
    const uint32_t* t = in.table + k / 2;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const uint32_t last = t[2 * q] & 3u;
      r[q] = quad(t + 2 * q);
      r[q].y = last > 0 ? r[q].y : 0.f;
      r[q].z = last > 1 ? r[q].z : 0.f;
      r[q].w = last > 2 ? r[q].w : 0.f;
    }
  }
};

// the transpose of the im2col, rows = (r, s, c), k = pixels.  Table: per pixel the byte offset of its origin and the taps inside.
struct WaveIm2colT {
  static constexpr int kWords = kWaveMaxPixels * 2;
  typedef Im2colParams Params;
  BufView v;
  uint32_t base, tap;
  const uint32_t* table;
  AX_HD WaveIm2colT(const Params& a, int grp, int row, int /*kbeg*/, int /*kend*/, const uint32_t* table_)
      : v(make_view(a.x, a.bytes)), table(table_) {
    const int rows = a.kh * a.kw * a.Cg;
    const TapCoord t = decode_tap(row < rows ? row : rows - 1, a);
    base = (((uint32_t)t.r * (uint32_t)a.W + (uint32_t)t.s) * (uint32_t)a.Ctot + (uint32_t)(t.c + grp * a.c_stride_g)) * 4u;
    tap = tap_bits(t.r, t.s);
  }
  static AX_HD void build(const Params& g, uint32_t* table, int kbeg, int kend, int tid, int threads) {
    for (int e = tid; e < wave_steps16(kend - kbeg); e += threads) {
      const bool in = kbeg + e < kend;
      const PixCoord c = decode_pixel(in ? kbeg + e : 0, g);
      const int y0 = c.y * g.stride - g.pad, x0 = c.x * g.stride_x - g.pad_x;
      table[2 * e] = row_base<IM2COL_FWD>(g, c.n, y0, x0, 0);
      table[2 * e + 1] = in ? pixel_taps<IM2COL_FWD>(g, y0, x0) : 0u;
    }
  }
  AX_HD void load(float4* r, int k) const {
    const uint32_t* t = table + 2 * k;
    float f[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = buf_ld1(v, (t[2 * e + 1] & tap) == tap ? base + t[2 * e] : kOob);
    r[0] = make_float4(f[0], f[1], f[2], f[3]);
    r[1] = make_float4(f[4], f[5], f[6], f[7]);
  }
};

// run-mode weights from the packed ones: k = (r, j < run), row = output channel; zero for j >= kc.  Table: per quad its byte
// offset, a multiple of four, and in its two lowest bits how many of its elements after the first are there.
struct WaveRunParams {
  DenseParams w;  // packed weights [(r, j < kc)][o]
  int kc, run;    // run: kc rounded up to a multiple of four
  FastDiv d_run;
};
struct WaveRunB {
  static constexpr int kWords = kWaveMaxK / 4;
  typedef WaveRunParams Params;
  BufView v;
  uint32_t base, ld4;
  const uint32_t* table;
  AX_HD WaveRunB(const Params& a, int /*g*/, int row, int /*kbeg*/, int /*kend*/, const uint32_t* table_)
      : v(make_view(a.w.p, a.w.bytes)), ld4((uint32_t)a.w.ld * 4u), table(table_) {
    base = (uint32_t)(row < a.w.R ? row : a.w.R - 1) * 4u;
  }
  static AX_HD void build(const Params& p, uint32_t* table, int kbeg, int kend, int tid, int threads) {
    for (int q = tid; q < wave_steps16(kend - kbeg) / 4; q += threads) {
      const int k = kbeg + 4 * q, r = (int)fdiv((uint32_t)k, p.d_run), j = k - r * p.run, n = p.kc - j;
      table[q] = k < kend ? (uint32_t)(r * p.kc + j) * (uint32_t)p.w.ld * 4u + (uint32_t)(n < 4 ? n - 1 : 3) : kOob;
    }
  }
  AX_HD void load(float4* r, int k) const {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const uint32_t t = table[k / 4 + q], last = t & 3u, o = base + (t & ~3u);
      float f[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) f[e] = buf_ld1(v, e <= (int)last ? o + (uint32_t)e * ld4 : kOob);
      r[q] = make_float4(f[0], f[1], f[2], f[3]);
    }
  }
};

// packed weights wf[g][(r, s, c)][o] as the operand of a data gradient: k = (r, s, o), row = c; og a multiple of four.
// Table: per quad its byte offset.
struct WaveTapParams {
  DenseParams w;  // gstride: floats per group
  int Cg, og;
  FastDiv d_og;
};
struct WaveTapB {
  static constexpr int kWords = kWaveMaxK / 4;
  typedef WaveTapParams Params;
  BufView v;
  uint32_t base;
  const uint32_t* table;
  AX_HD WaveTapB(const Params& a, int g, int row, int /*kbeg*/, int /*kend*/, const uint32_t* table_)
      : v(make_view(a.w.p + (long)g * a.w.gstride, a.w.bytes)), table(table_) {
    base = (uint32_t)(row < a.Cg ? row : a.Cg - 1) * (uint32_t)a.og * 4u;
  }
  static AX_HD void build(const Params& p, uint32_t* table, int kbeg, int kend, int tid, int threads) {
    for (int q = tid; q < wave_steps16(kend - kbeg) / 4; q += threads) {
      const int k = kbeg + 4 * q, rs = (int)fdiv((uint32_t)k, p.d_og), o = k - rs * p.og;
      table[q] = k < kend ? ((uint32_t)rs * (uint32_t)p.Cg * (uint32_t)p.og + (uint32_t)o) * 4u : kOob;
    }
  }
  AX_HD void load(float4* r, int k) const {
#pragma unroll
    for (int q = 0; q < 2; ++q) r[q] = buf_ld4(v, base + table[k / 4 + q]);
  }
};

// One product: its operands, epilogue, sizes and grid of ceil(M/32) * ceil(N/32) * groups * ns workgroups
template <class AL_, class BL_, class Epi_, bool BF_>
struct WaveJob {
  typedef AL_ AL;
  typedef BL_ BL;
  typedef Epi_ Epi;
  static constexpr bool BF = BF_;
  typename AL::Params a;
  typename BL::Params b;
  Epi ep;
  int M, N, K, kchunk;
  FastDiv gx, gy, ns;
  uint32_t blocks;
};

// load_exact() where a loader has one
template <class L>
AX_HD auto wave_load_exact(const L& l, float4* r, int k, int) -> decltype(l.load_exact(r, k)) {
  l.load_exact(r, k);
}
template <class L>
AX_HD void wave_load_exact(const L& l, float4* r, int k, long) {
  l.load(r, k);
}

// ================================= kernel ====================================
#ifndef AX_HOST_EMU
// What the epilogue reads for an element is asked for in front of the products and handed to it behind the sums: at the end it
// was one more trip to the cache or to memory in a chain of two or three.
template <class Epi>
__device__ __forceinline__ float wave_ask(const Epi&, int /*m*/, int /*n*/) { return 0.f; }
template <class Epi>
__device__ __forceinline__ void wave_put(const Epi& e, int m, int n, float v, float /*asked*/) { e.apply(m, n, v); }
__device__ __forceinline__ float wave_ask(const EpiBiasAct& e, int, int n) { return e.bias ? e.bias[e.col_off + n] : -0.f; }
__device__ __forceinline__ void wave_put(const EpiBiasAct& e, int m, int n, float v, float bias) {
  const long o = (long)m * e.ldc + e.col_off + n;
  v += bias;
  if (e.relu) v = v > 0.f ? v : 0.f;
  e.y[o] = v;
  if (e.y16) store_bf16(e.y16 + o, v);
}
__device__ __forceinline__ float wave_ask(const EpiGate& e, int m, int n) {
  return e.gate ? e.gate[(long)m * e.ldc + e.col_off + n] : 1.f;
}
__device__ __forceinline__ void wave_put(const EpiGate& e, int m, int n, float v, float gate) {
  const long o = (long)m * e.ldc + e.col_off + n;
  v = gate > 0.f ? v : 0.f;
  e.dx[o] = v;
  if (e.dx16) store_bf16(e.dx16 + o, v);
}

// Whether an operand without a table is asked for while the other's table is made.  In front of a weight gradient's table it was in
// the way (us without | with: 16 channels, 5 x 5 on 14 x 14, 128 maps 14.4 | 14.9; 24, 3 x 3 on 13 x 13, 64 maps 9.2 | 9.6; 224, 5 x 5
// on 9 x 9, 40 maps 43.3 | 45.2; steps of the small nets 1 % longer); in front of a forward product's, with the bias, it saves a
// trip (32 channels, 14 x 14, 60 maps 15.4 | 15.2; 64, 9 x 9, 50 maps 11.8 | 11.5; steps of the small nets 1 to 3 % shorter).
template <class J>
constexpr bool kOtherFirst = J::BL::kWords == 0 && !std::is_same<typename J::AL, WaveIm2colT>::value;

template <int W, int WORDS>
struct WaveLds {
  float part[W][kWaveTile * kWaveTile];
  uint32_t bad[W];
  __attribute__((aligned(16))) uint32_t table[WORDS ? WORDS : 4];
};
template <class J>
constexpr int kJobWords = J::AL::kWords + J::BL::kWords;

// the three terms of eight values, as the matrix core's operands
struct WaveTerms {
  v8bf t[kPlanes];
};
__device__ __forceinline__ WaveTerms wave_split(const float4* r) {
  const SplitPair p[4] = {split_pair(r[0].x, r[0].y), split_pair(r[0].z, r[0].w), split_pair(r[1].x, r[1].y),
                          split_pair(r[1].z, r[1].w)};
  WaveTerms w;
#pragma unroll
  for (int q = 0; q < kPlanes; ++q) {
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    v4u u;
#pragma unroll
    for (int i = 0; i < 4; ++i) u[i] = p[i].t[q];
    w.t[q] = __builtin_bit_cast(v8bf, u);
  }
  return w;
}
__device__ __forceinline__ v8bf wave_round(const float4* r) {
  typedef uint32_t v4u __attribute__((ext_vector_type(4)));
  v4u u;
  u[0] = split_pack(r[0].x, r[0].y);
  u[1] = split_pack(r[0].z, r[0].w);
  u[2] = split_pack(r[1].x, r[1].y);
  u[3] = split_pack(r[1].z, r[1].w);
  return __builtin_bit_cast(v8bf, u);
}
__device__ __forceinline__ void wave_store(const v16f& acc, float* part, int lane) {
#pragma unroll
  for (int r = 0; r < 16; ++r) part[acc_row(lane, r) * kWaveTile + (lane & 31)] = acc[r];
}

template <int W, class J, class Lds>
__device__ __forceinline__ void wave_tile(const J& j, uint32_t block, Lds& lds) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t rest = fdiv(block, j.gy), z = fdiv(rest, j.gx), g = fdiv(z, j.ns);
  const int split = (int)(z - g * j.ns.d);
  const int m0 = (int)(rest - z * j.gx.d) * kWaveTile, n0 = (int)(block - rest * j.gy.d) * kWaveTile;
  const int kbeg = split * j.kchunk, kend = min(j.K, kbeg + j.kchunk), len = kend - kbeg;
  uint32_t* const ta = lds.table;
  uint32_t* const tb = lds.table + J::AL::kWords;
  const int kh = 8 * (lane >> 5), kfirst = 16 * wave;
  constexpr int kStep = 16 * W;
  // see kOtherFirst
  const typename J::BL bl(j.b, (int)g, n0 + (lane & 31), kbeg, kend, tb);
  float4 rb[2];
  if (kOtherFirst<J> && kfirst < len) bl.load(rb, kfirst + kh);
  typename J::Epi ep = j.ep;
  ep.set_group((int)g, (int)z);
  constexpr int kMine = kWaveTile * kWaveTile / (64 * W);  // of the tile's elements, tid + i * 64 * W
  float asked[kMine];
#pragma unroll
  for (int i = 0; i < kMine; ++i) {
    const int e = tid + i * 64 * W, m = m0 + e / kWaveTile, n = n0 + e % kWaveTile;
    asked[i] = m < j.M && n < j.N ? wave_ask(ep, m, n) : 0.f;
  }
  J::AL::build(j.a, ta, kbeg, kend, tid, 64 * W);
  J::BL::build(j.b, tb, kbeg, kend, tid, 64 * W);
  const typename J::AL al(j.a, (int)g, m0 + (lane & 31), kbeg, kend, ta);
  if (kJobWords<J> > 0) __syncthreads();

  v16f hi, lo;
#pragma unroll
  for (int r = 0; r < 16; ++r) hi[r] = lo[r] = 0.f;
  if (kfirst < len) {  // uniform
    float4 ra[2];
    auto load_a = [&](int k) {  // rounded products are not looked at afterwards
      if (J::BF) wave_load_exact(al, ra, k, 0);
      else al.load(ra, k);
    };
    load_a(kfirst + kh);
    if (!kOtherFirst<J>) bl.load(rb, kfirst + kh);
    for (int k = kfirst; k < len; k += kStep) {
      // the registers are free once their values are split: the next step's loads run under this step's products
      const bool more = k + kStep < len;
      if (J::BF) {
        const v8bf a = wave_round(ra), b = wave_round(rb);
        if (more) {
          load_a(k + kStep + kh);
          bl.load(rb, k + kStep + kh);
        }
        hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, hi, 0, 0, 0);
      } else {
        const WaveTerms a = wave_split(ra), b = wave_split(rb);
        if (more) {
          load_a(k + kStep + kh);
          bl.load(rb, k + kStep + kh);
        }
#pragma unroll
        for (int q = 0; q < kSplitProducts; ++q) {
          v16f& c = q == 0 ? hi : lo;
          c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.t[split_plane_a(q)], b.t[split_plane_b(q)], c, 0, 0, 0);
        }
      }
    }
  }
  if (!J::BF) {
    float top = 0.f;  // as in gemm_split_kernel
#pragma unroll
    for (int r = 0; r < 16; ++r) hi[r] = (hi[r] + lo[r]) * kSplitUnscale;
#pragma unroll
    for (int r = 0; r < 16; r += 2)
      top = __builtin_elementwise_maximum(__builtin_elementwise_maximum(top, fabsf(hi[r])), fabsf(hi[r + 1]));
    const bool bad = __any(!(top <= 3.402823466e38f));
    if (lane == 0) lds.bad[wave] = bad;
  }
  wave_store(hi, lds.part[wave], lane);
  __syncthreads();
  if (!J::BF) {
    uint32_t bad = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) bad |= lds.bad[w];
    if (bad) {  // the same for every wave; each rewrites its own part
#pragma unroll
      for (int r = 0; r < 16; ++r) hi[r] = 0.f;
      for (int k = kfirst; k < len; k += kStep) {
        float4 ra[2], rb[2];
        wave_load_exact(al, ra, k + kh, 0);
        bl.load(rb, k + kh);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          hi = MfmaBlock<32>::mma(ra[q].x, rb[q].x, hi);
          hi = MfmaBlock<32>::mma(ra[q].y, rb[q].y, hi);
          hi = MfmaBlock<32>::mma(ra[q].z, rb[q].z, hi);
          hi = MfmaBlock<32>::mma(ra[q].w, rb[q].w, hi);
        }
      }
      wave_store(hi, lds.part[wave], lane);
      __syncthreads();
    }
  }
  const int parts = min(W, (len + 15) / 16);  // waves that had a step
#pragma unroll
  for (int i = 0; i < kMine; ++i) {
    const int e = tid + i * 64 * W, m = m0 + e / kWaveTile, n = n0 + e % kWaveTile;
    float s = 0.f;
    for (int w = 0; w < parts; ++w) s += lds.part[w][e];
    if (m < j.M && n < j.N) wave_put(ep, m, n, s, asked[i]);
  }
}

template <int W, class J>
__global__ void __launch_bounds__(64 * W, 4) gemm_wave_kernel(J j) {
  __shared__ WaveLds<W, kJobWords<J>> lds;
  wave_tile<W>(j, blockIdx.x, lds);
}
// Two products that do not depend on each other: the weight and the data gradient of a layer, which read the same output
// gradient
template <int W, class J, class K>
__global__ void __launch_bounds__(64 * W, 4) gemm_wave_pair_kernel(J j, K k) {
  __shared__ WaveLds<W, (kJobWords<J> > kJobWords<K> ? kJobWords<J> : kJobWords<K>)> lds;
  if (blockIdx.x < j.blocks)  // uniform
    wave_tile<W>(j, blockIdx.x, lds);
  else
    wave_tile<W>(k, blockIdx.x - j.blocks, lds);
}
#endif  // AX_HOST_EMU

}  // namespace ax
