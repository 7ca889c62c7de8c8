// fp32 products on the bf16 matrix cores: every fp32 operand value is split into three bf16 terms,
//
//   2^24 x = h + m + l,   h = bf16(2^24 x), m = bf16(2^24 x - h), l = 2^24 x - h - m     (8 + 8 + 8 significand bits)
//
// exact for every |x| below 2^103: the factor puts the last bit of the smallest number, 2^-149, where bf16 has one too.
// (Without it the terms of operands below 2^-110 lost bits, 2.6e-5 of the value at 1e-36; the multiplication costs 2 to
// 3 % of a product.)  The sums are multiplied by 2^-48 in return.  A product a*b is the sum of the six term products that
// matter,
//
//   hh + hm + mh + mm + hl + lh,
//
// each exact in the matrix core, accumulated in fp32: hh in one set of accumulators, the other five, 2^-8 of it and
// less, in a second one, and the two are added at the end.  What is dropped (ml, lm, ll) is below 2^-24 of |a*b| and of
// either sign.  An accumulator is rounded once per MFMA, and only hh's roundings count: one per 16 products, where the
// fp32 MFMA rounds its sum once per two.  (All six terms in one set of accumulators round six times per 16: 2.2e-7 of
// the result at K = 192 and 7.1e-7 at 2048 against 7.7e-8 and 2.8e-7 so, 2.5e-7 and 8.3e-7 for the fp32 MFMA -- but
// where half the products are zero, as behind a ReLU, the fp32 MFMA rounds less often and a single set was less exact
// than it at every length, 1.28 times its error at K = 64, 1.14 at 9216.)
//
// An operand that is infinite, or becomes so (from 2^103 up), has a NaN among its terms (inf - inf), and sums from 2^80
// up overflow: either way a sum is not finite.  A workgroup that finds one in its tile computes the tile once more with
// the fp32 matrix instructions, so infinities, NaNs and large numbers come out as those give them; finite sums prove that
// nothing was lost.  The look at the sums costs about 1 % of a product (72 of 6272 x 128 x 192: 171 -> 174 us).
//
// Why: v_mfma_f32_32x32x16_bf16 does 1024 flop per SIMD and clock, v_mfma_f32_32x32x2_f32 does 64; six of the
// former are 16/6 = 2.7 times as fast as the latter for the same contraction.
//
// Measured inside a batch-128 training step against the fp32 MFMA kernels: forward products 282 -> 205 us (first layer),
// 216 -> 185 (second, transformed), 128 -> 106 (third), 97 -> 94 (fourth); weight gradients 353 -> 226, 239 -> 153, 154 ->
// 96, 87 -> 55 us (fifth); dense layers, forward, 116 -> 98 us.  4096 x 4608 x 2048 alone: 101 -> 150 TFLOP/s at half the
// matrix cores' issue rate; the clock falls from 2.2 to 1.7 GHz in such a run, so power bounds it as much as the splitting
// (104 vector instructions per 24 MFMAs and wave) does.  The products of the transformed layers are short (K = 128 .. 256)
// and move 2.5 - 3.5 TB/s as well.
//
// The second set of accumulators costs registers: the 128 x 128 tile fits a compute unit twice instead of three times
// (its LDS with two row-contiguous operands, 55,296 bytes, allows no more anyway), 128 x 96 and 128 x 64 three times.
// Alone, one set -> two: 128 x 128 151 -> 147 TFLOP/s on 4096 x 4608 x 2048, 176 -> 182 us on 72 products of 6272 x 128 x
// 192; 128 x 96 and 128 x 64 within 2 %.  A 128 x 192 tile no longer fits (72 products of 6272 x 192 x 128 took 202 us with
// it, 233 with 128 x 96).
//
// Addressing, zero fill, split-k and epilogues are those of gemm.h; operands are fetched as fp32 and split once per
// workgroup, on their way into LDS.
//
// LDS layout, in 16-byte units of eight consecutive k of one row: unit (plane, k octet, position of the row).
//   k-contiguous operands    position = row; a load of four k is one 8-byte store per plane, and an octet's rows
//                            are padded so that the two octets of a 16-deep step lie half the banks apart
//   row-contiguous operands  a thread fetches k and k+1 of four rows and stores one word per row and plane; row
//                            4q + j sits at position j*(ROWS/4 + 4) + q, so that the lanes of a store are 16 bytes apart
// A fragment is one 16-byte read per plane in both, without bank conflicts.
#pragma once

#include "gemm_bf16.h"
#include "wino_rows.h"

namespace ax {

constexpr int kPlanes = 3;
constexpr int kBKs = 16;  // depth of a k-tile: one MFMA step
// Reductions of fewer than eight values stay on the fp32 matrix instructions.  Those round once per two products, K/2
// times; here, whatever the length, the sum of the two sets of accumulators is rounded, and the dropped terms count as
// much as one rounding again.  A single product is to be correctly rounded (K = 1: 0.43 units of 2^-24 against 0.42, at
// worst 1.5 against 1.0); from K = 4 on the split products are the closer ones at worst too (2.0 against 2.6).
constexpr int kSplitMinK = 8;

AX_HD float bf_lo(uint32_t w) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __uint_as_float(w << 16);
#else
  const uint32_t u = w << 16;
  float f;
  memcpy(&f, &u, 4);
  return f;
#endif
}
AX_HD float bf_hi(uint32_t w) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __uint_as_float(w & 0xffff0000u);
#else
  const uint32_t u = w & 0xffff0000u;
  float f;
  memcpy(&f, &u, 4);
  return f;
#endif
}
constexpr float kSplitScale = 16777216.f, kSplitUnscale = 1.f / 281474976710656.f;  // 2^24, 2^-48
// the three terms of 2^24 x (low halves) and 2^24 y (high halves)
struct SplitPair {
  uint32_t t[kPlanes];
};
// two values rounded to bf16 (nearest even) by one instruction: through pack_bf16() the compiler, which sees that the
// halves are widened again, converts every value a second time on its own
AX_HD uint32_t split_pack(float lo, float hi) {
#if defined(__HIP_DEVICE_COMPILE__)
  uint32_t w;
  asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(w) : "v"(lo), "v"(hi));
  return w;
#else
  return pack_bf16(lo, hi);
#endif
}
AX_HD SplitPair split_pair(float x, float y) {
  SplitPair s;
  x *= kSplitScale;
  y *= kSplitScale;
  s.t[0] = split_pack(x, y);
  const float rx = x - bf_lo(s.t[0]), ry = y - bf_hi(s.t[0]);
  s.t[1] = split_pack(rx, ry);
  s.t[2] = split_pack(rx - bf_lo(s.t[1]), ry - bf_hi(s.t[1]));
  return s;
}

// The tile as plain fp32 in LDS, [row][k], for the second computation of a tile whose sums are not finite
constexpr int kRawLd = kBKs + 1;
AX_HD void raw_store_quad(float* lds, int row, int kq, const float4& v) {
  float* d = lds + row * kRawLd + 4 * kq;
  d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
}
// four consecutive k (quad kq of the tile) of one row of a k-contiguous operand
template <int RP>
AX_HD void split_store_quad(uint32_t* lds, int row, int kq, const float4& v) {
  uint32_t* d = lds + ((kq >> 1) * RP + row) * 4 + 2 * (kq & 1);
  const SplitPair a = split_pair(v.x, v.y), b = split_pair(v.z, v.w);
#pragma unroll
  for (int p = 0; p < kPlanes; ++p) {
#if defined(__HIP_DEVICE_COMPILE__)
    typedef uint32_t v2u __attribute__((ext_vector_type(2)));
    v2u w;
    w[0] = a.t[p];
    w[1] = b.t[p];
    *reinterpret_cast<v2u*>(d + p * 2 * RP * 4) = w;
#else
    d[p * 2 * RP * 4] = a.t[p];
    d[p * 2 * RP * 4 + 1] = b.t[p];
#endif
  }
}
// a unit of a row-contiguous operand: rows 4*rq .. 4*rq+3 at k = 2*kp (a) and 2*kp + 1 (b), two rows at a time
template <int ROWS>
struct SplitRowStore {
  static constexpr int SP = ROWS / 4 + 4, RP = 4 * SP;
  static AX_HD int pos(int row) { return (row & 3) * SP + (row >> 2); }
  // unit idx of the tile: its row quad and pair of k.  Four lanes take the four pairs of an octet, so that the words
  // a wave stores at once lie side by side.
  static AX_HD int quad(int idx) { return (idx >> 2) % (ROWS / 4); }
  static AX_HD int pair(int idx) { return (idx & 3) + 4 * (idx / ROWS); }
  static AX_HD void store_half(uint32_t* lds, int rq, int kp, int half, const float4& a, const float4& b) {
    uint32_t* d = lds + ((kp >> 2) * RP + 2 * half * SP + rq) * 4 + (kp & 3);
    const SplitPair s0 = half ? split_pair(a.z, b.z) : split_pair(a.x, b.x);
    const SplitPair s1 = half ? split_pair(a.w, b.w) : split_pair(a.y, b.y);
#pragma unroll
    for (int p = 0; p < kPlanes; ++p) {
      d[p * 2 * RP * 4] = s0.t[p];
      d[(p * 2 * RP + SP) * 4] = s1.t[p];
    }
  }
  static AX_HD void raw_half(float* lds, int rq, int kp, int half, const float4& a, const float4& b) {
    float* d = lds + (4 * rq + 2 * half) * kRawLd + 2 * kp;
    d[0] = half ? a.z : a.x;
    d[1] = half ? b.z : b.x;
    d[kRawLd] = half ? a.w : a.y;
    d[kRawLd + 1] = half ? b.w : b.y;
  }
};

// ---- loaders --------------------------------------------------------------------
//   fetch(r, kleft)        issue the loads of the next k-tile, of which kleft k are left, and step on; a k-tile past
//                          the end (kleft <= 0) reads nothing and returns zeros
//   store_step(s, lds, r)  split and store part s of what fetch() brought
//   raw_step(s, lds, r)    store it as it is, [row][k] with rows kRawLd apart
// Byte offsets run along with k; rows outside the operand start at kOob and stay outside: a reduction spans less
// than 2 GiB.

// elem(row, k) = p[row*ld + k]; ld and K multiples of four, 16-byte aligned
template <int ROWS>
struct SplitKInner {
  static constexpr int QK = kBKs / 4, NQ = ROWS * QK, NL = (NQ + kThreads - 1) / kThreads, NS = NL;
  static constexpr bool kWhole = NQ % kThreads == 0;  // else some threads own no quad in the last round
  static constexpr int RP = ROWS + 8, UNITS = kPlanes * 2 * RP;
  static AX_HD int pos(int row) { return row; }
  static constexpr int block_units(int t) { return 32 * t; }  // pos(row + 32 t) - pos(row)
  typedef DenseParams Params;
  BufView v;
  int tid, kq;
  uint32_t off[NL];
  AX_HD SplitKInner(const Params& a, int g, int tid_, int row0, int kbeg)
      : v(make_view(a.p + (long)g * a.gstride, a.bytes - (uint32_t)(g * a.gstride * 4))), tid(tid_) {
    kq = tid % QK;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int idx = tid + i * kThreads, row = row0 + idx / QK;
      off[i] = (kWhole || idx < NQ) && row < a.R ? ((uint32_t)row * (uint32_t)a.ld + (uint32_t)(kbeg + 4 * kq)) * 4u : kOob;
    }
  }
  AX_HD void fetch(float4* r, int kleft) {
    const bool in = 4 * kq < kleft;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      r[i] = buf_ld4(v, in ? off[i] : kOob);
      off[i] += kBKs * 4;
    }
  }
  AX_HD void store_step(int s, uint32_t* lds, const float4* r) const {
    const int idx = tid + s * kThreads;
    if (kWhole || idx < NQ) split_store_quad<RP>(lds, idx / QK, kq, r[s]);
  }
  AX_HD void raw_step(int s, float* lds, const float4* r) const {
    const int idx = tid + s * kThreads;
    if (kWhole || idx < NQ) raw_store_quad(lds, idx / QK, kq, r[s]);
  }
};

// elem(row, k) = p[k*ld + row]; rows and ld multiples of four, 16-byte aligned
template <int ROWS>
struct SplitRowInner {
  typedef SplitRowStore<ROWS> St;
  static constexpr int QR = ROWS / 4, NU = QR * (kBKs / 2), NUT = (NU + kThreads - 1) / kThreads, NL = 2 * NUT,
                       NS = 2 * NUT;
  static constexpr bool kWhole = NU % kThreads == 0;  // else some threads own no unit in the last round
  static constexpr int RP = St::RP, UNITS = kPlanes * 2 * RP;
  static AX_HD int pos(int row) { return St::pos(row); }
  static constexpr int block_units(int t) { return 8 * t; }
  typedef DenseParams Params;
  BufView v;
  int tid;
  uint32_t ld4, off[NUT];  // ld4: bytes between consecutive k
  AX_HD SplitRowInner(const Params& a, int g, int tid_, int row0, int kbeg)
      : v(make_view(a.p + (long)g * a.gstride, a.bytes - (uint32_t)(g * a.gstride * 4))), tid(tid_) {
    ld4 = (uint32_t)a.ld * 4u;
#pragma unroll
    for (int u = 0; u < NUT; ++u) {
      const int idx = tid + u * kThreads, row = row0 + 4 * St::quad(idx), kp = St::pair(idx);
      off[u] = (kWhole || idx < NU) && row < a.R ? (uint32_t)(kbeg + 2 * kp) * ld4 + (uint32_t)row * 4u : kOob;
    }
  }
  AX_HD void fetch(float4* r, int kleft) {
#pragma unroll
    for (int u = 0; u < NUT; ++u) {
      const int k = 2 * St::pair(tid + u * kThreads);
      r[2 * u] = buf_ld4(v, k < kleft ? off[u] : kOob);
      r[2 * u + 1] = buf_ld4(v, k + 1 < kleft ? off[u] + ld4 : kOob);
      off[u] += kBKs * ld4;
    }
  }
  AX_HD void store_step(int s, uint32_t* lds, const float4* r) const {
    const int u = s >> 1, idx = tid + u * kThreads;
    if (kWhole || idx < NU) St::store_half(lds, St::quad(idx), St::pair(idx), s & 1, r[2 * u], r[2 * u + 1]);
  }
  AX_HD void raw_step(int s, float* lds, const float4* r) const {
    const int u = s >> 1, idx = tid + u * kThreads;
    if (kWhole || idx < NU) St::raw_half(lds, St::quad(idx), St::pair(idx), s & 1, r[2 * u], r[2 * u + 1]);
  }
};

// The implicit im2col operand of run mode (Im2colParams): row = output pixel, k = (kernel row, position in its run).
// Runs of at least one k-tile (run_len() >= 16), so that a step of one k-tile passes at most one run's end.
template <int ROWS>
struct SplitRun {
  static constexpr int QK = kBKs / 4, NQ = ROWS * QK, NL = NQ / kThreads, NS = NL;
  static_assert(NQ % kThreads == 0, "tile must be a whole number of loads per thread");
  static constexpr int RP = ROWS + 8, UNITS = kPlanes * 2 * RP;
  static AX_HD int pos(int row) { return row; }
  static constexpr int block_units(int t) { return 32 * t; }
  typedef Im2colParams Params;
  BufView v;
  int tid, kq, run, j;   // j: position in the run of the thread's quad
  uint32_t skip;         // bytes from a run's end to the next kernel row's run
  uint32_t off[NL];
  AX_HD SplitRun(const Params& a, int /*g*/, int tid_, int row0, int kbeg) : v(make_view(a.x, a.bytes)), tid(tid_) {
    kq = tid % QK;
    run = a.Cg;
    skip = (uint32_t)(a.W - run) * 4u;
    const int k = kbeg + 4 * kq, r = (int)fdiv((uint32_t)k, a.d_cg);
    j = k - r * run;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int p = row0 + (tid + i * kThreads) / QK;
      const PixCoord c = decode_pixel(p < a.P ? p : 0, a);
      const uint32_t base = row_base<IM2COL_FWD>(a, c.n, c.y * a.stride + r, c.x * a.stride_x + j, 0);
      off[i] = p < a.P ? base : kOob;
    }
  }
  AX_HD void fetch(float4* r, int kleft) {
    const bool in = 4 * kq < kleft;
    j += kBKs;
    const bool over = j >= run;
    const uint32_t step = kBKs * 4u + (over ? skip : 0u);
    if (over) j -= run;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      r[i] = buf_ld4(v, in ? off[i] : kOob);
      off[i] += step;
    }
  }
  AX_HD void store_step(int s, uint32_t* lds, const float4* r) const {
    split_store_quad<RP>(lds, (tid + s * kThreads) / QK, kq, r[s]);
  }
  AX_HD void raw_step(int s, float* lds, const float4* r) const {
    raw_store_quad(lds, (tid + s * kThreads) / QK, kq, r[s]);
  }
};
// Its transpose (weight gradient): k = output pixel, row = one of the k*C floats of a kernel row.  The whole quads of
// every kernel row come first and the floats left over at the runs' ends behind them, (3 mod 4 channels of the last
// tap), as quads gathered one float at a time: 11 rows of 33 floats are 363 rows, three tiles of 128, where runs padded
// to 36 are 396 and need a fourth tile for 12 of them.
struct RunTParams {
  Im2colParams g;     // run mode
  int quads, left;    // whole quads and floats left over per kernel row
  FastDiv d_quads, d_left;
};
inline RunTParams run_t_params(const Im2colParams& g, int floats) {
  return RunTParams{g, floats / 4, floats % 4, make_fastdiv((uint32_t)(floats / 4)), make_fastdiv((uint32_t)(floats % 4))};
}
// A thread owns one row quad and a pair of pixels that moves on by one k-tile at a time; rows of at least one k-tile of
// pixels (OW >= 16), so that a step passes at most one row's end.
template <int ROWS>
struct SplitRunT {
  typedef SplitRowStore<ROWS> St;
  static constexpr int QR = ROWS / 4, NU = QR * (kBKs / 2), NL = 2, NS = 2;
  static_assert(NU <= kThreads, "at most one unit per thread");
  static constexpr int RP = St::RP, UNITS = kPlanes * 2 * RP;
  static AX_HD int pos(int row) { return St::pos(row); }
  static constexpr int block_units(int t) { return 8 * t; }
  typedef RunTParams Params;
  BufView v;
  int tid, OW, OH, x, y;                 // (y, x): the first pixel of the pair
  uint32_t off, pix, row, img;           // byte offset of its origin; steps to the next pixel, past a row's, a picture's end
  uint32_t tap[4];                       // of the quad's rows from a pixel's origin, kOob for a row past the end
  bool gather;                           // rows that do not lie side by side
  AX_HD SplitRunT(const Params& a, int /*g*/, int tid_, int row0, int kbeg)
      : v(make_view(a.g.x, a.g.bytes)), tid(tid_), OW(a.g.OW), OH(a.g.OH) {
    const Im2colParams& g = a.g;
    const int q = row0 / 4 + St::quad(tid), rest = 4 * (q - g.kh * a.quads);
    gather = rest >= 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      int r, j;
      if (gather) {
        r = a.left ? (int)fdiv((uint32_t)(rest + e), a.d_left) : g.kh;
        j = 4 * a.quads + (rest + e - r * a.left);
      } else {
        r = (int)fdiv((uint32_t)q, a.d_quads);
        j = 4 * (q - r * a.quads) + e;
      }
      tap[e] = r < g.kh ? (uint32_t)(r * g.W + j) * 4u : kOob;
    }
    const PixCoord c = decode_pixel(kbeg + 2 * St::pair(tid), g);
    y = c.y;
    x = c.x;
    off = row_base<IM2COL_FWD>(g, c.n, c.y * g.stride, c.x * g.stride_x, 0);
    pix = (uint32_t)g.stride_x * 4u;
    row = (uint32_t)(g.stride * g.W - g.OW * g.stride_x) * 4u;
    img = (uint32_t)((g.H - g.OH * g.stride) * g.W) * 4u;
  }
  // off of a pixel px of row py that may lie past the row's end
  AX_HD uint32_t wrap(uint32_t o, int px, int py) const {
    return px < OW ? o : o + row + (py + 1 < OH ? 0u : img);
  }
  AX_HD void load(float4& r, uint32_t o, bool in) const {
    if (gather) {  // o + kOob stays outside
      r.x = buf_ld1(v, in ? o + tap[0] : kOob);
      r.y = buf_ld1(v, in ? o + tap[1] : kOob);
      r.z = buf_ld1(v, in ? o + tap[2] : kOob);
      r.w = buf_ld1(v, in ? o + tap[3] : kOob);
    } else {
      r = buf_ld4(v, in ? o + tap[0] : kOob);
    }
  }
  AX_HD void fetch(float4* r, int kleft) {
    const int k = 2 * St::pair(tid);
    load(r[0], off, k < kleft);
    load(r[1], wrap(off + pix, x + 1, y), k + 1 < kleft);
    off = wrap(off + kBKs * pix, x + kBKs, y);
    x += kBKs;
    if (x >= OW) {
      x -= OW;
      y = y + 1 < OH ? y + 1 : 0;
    }
  }
  AX_HD void store_step(int s, uint32_t* lds, const float4* r) const {
    if (NU == kThreads || tid < NU) St::store_half(lds, St::quad(tid), St::pair(tid), s & 1, r[0], r[1]);
  }
  AX_HD void raw_step(int s, float* lds, const float4* r) const {
    if (NU == kThreads || tid < NU) St::raw_half(lds, St::quad(tid), St::pair(tid), s & 1, r[0], r[1]);
  }
};

template <class L>
AX_HD void split_store_all(const L& l, uint32_t* lds, const float4* r) {
#pragma unroll
  for (int s = 0; s < L::NS; ++s) l.store_step(s, lds, r);
}
template <class L>
AX_HD void raw_store_all(const L& l, float* lds, const float4* r) {
#pragma unroll
  for (int s = 0; s < L::NS; ++s) l.raw_step(s, lds, r);
}
// 16-byte unit that holds k octet kh of `row` in plane p
template <class L>
AX_HD int split_unit(int p, int kh, int row) {
  return (p * 2 + kh) * L::RP + L::pos(row);
}
// the six term products, hh first, by planes of B: planes of A and B
AX_HD int split_plane_a(int q) { return q < 3 ? q : q < 5 ? q - 3 : 0; }
AX_HD int split_plane_b(int q) { return q < 3 ? 0 : q < 5 ? 1 : 2; }
constexpr int kSplitProducts = 6;

// A weight gradient with its operands exchanged (rows of the product = columns of the result): ws[z][n][m] = v.  The
// lanes of a store run along m, the result's contiguous direction.
struct EpiSlabSwapped {
  float* ws;
  long slab;  // M*N
  long ldc;   // M
  float* base;
  AX_HD void set_group(int /*g*/, int z) { base = ws + (long)z * slab; }
};
// Whether the lanes of a block run along the product's rows (the MFMA's operands exchanged) and not along its columns.  Only here
// are the rows what lies side by side in memory.  Everything else is stored 32 columns at a time; 16-byte stores of four columns
// of 32 rows, which these kernels had, touched 32 lines each: transformed products of batch 128 182 -> 164 us (second layer
// forward), 200 -> 176 (its data gradient), first layer forward 206 -> 189.
template <class Epi>
constexpr bool kRowsAcross = std::is_same<Epi, EpiSlabSwapped>::value;
#ifndef AX_HOST_EMU
template <int TM, int TN>
__device__ __forceinline__ void store_rows(const EpiSlabSwapped& e, const v16f (&acc)[TM][TN], int m, int n, int M, int N, int lane) {
  const uint32_t ld = (uint32_t)e.ldc * 4u;
  const BufView out = make_view(e.base, (uint32_t)N * ld);
  uint32_t at[TM];
  column_offsets<TM>(at, ld, 0, n, m, M, lane);
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int i = 0; i < TM; ++i) buf_st1(out, at[i] + (uint32_t)(j * 32 + block_row(r)) * ld, acc[i][j][r]);
}
#endif

// The one-dimensional grid of gx * gy * (groups * nsplit) workgroups (see xcd_tile).  The divisors are constants of the
// launch, so that a workgroup's place is worked out on the scalar unit and the buffer descriptors that depend on it
// stay in scalar registers.
// of: rows (1) or the reduction (2) of the product run over the rows that a group's position has in a transformed layer with short
// tiles (wino_rows(), group = position * positions.d + group of channels); the sizes of the launch are those of all rows.  Tiles of
// rows that a group does not have are nobody's, and slices share what there is.
struct SplitGrid {
  FastDiv gx, gy, nsplit;
  int of;
  FastDiv positions;
  int short_y, whole, short_x, tiles;
};
// the launch's `turn`-th group
AX_HD uint32_t split_group(const SplitGrid& grid, uint32_t turn) {
  if (grid.of == 0) return turn;
  const uint32_t s = fdiv(turn, grid.positions);
  return (uint32_t)wino_spread((int)s) * grid.positions.d + (turn - s * grid.positions.d);
}
// A workgroup's first row and k, and the ends of both; m0 >= M: nobody's tile
struct SplitPlace {
  int m0, M, kbeg, kend;
};
template <class T>
AX_HD SplitPlace split_place(const SplitGrid& grid, uint32_t g, int split, int m0, int M, int K, int kchunk) {
  SplitPlace p{m0, M, split * kchunk, 0};
  p.kend = K < p.kbeg + kchunk ? K : p.kbeg + kchunk;
  if (grid.of == 0) return p;  // uniform
  const RowRange r = wino_rows((int)fdiv(g, grid.positions), grid.short_y, grid.whole, grid.short_x, grid.tiles);
  if (grid.of == 1) {
    p.m0 += r.lo;
    p.M = r.hi;
  } else {
    const uint32_t steps = (uint32_t)(r.hi - r.lo + T::BK - 1) / T::BK;
    const int per = (int)fdiv(steps + grid.nsplit.d - 1, grid.nsplit) * T::BK;
    p.kbeg = r.lo + split * per;
    p.kend = r.hi < p.kbeg + per ? r.hi : p.kbeg + per;
  }
  return p;
}
AX_HD void split_row_limit(DenseParams& a, int rows) { a.R = rows; }
template <class P>
AX_HD void split_row_limit(P&, int) {}

// ================================= kernel ====================================
#ifndef AX_HOST_EMU
template <class L, int TT>
struct SplitFrags {
  v8bf f[kPlanes][TT];
  template <int P>
  __device__ __forceinline__ void read(const uint32_t* lane_base) {  // lane_base: the lane's unit in plane 0, block 0
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int t = 0; t < TT; ++t)
      f[P][t] = __builtin_bit_cast(v8bf, *reinterpret_cast<const v4u*>(lane_base + (P * 2 * L::RP + L::block_units(t)) * 4));
  }
};

// Side work of one k-tile, dealt over the first four of its six groups of MFMAs: split and store tile t+1.  Its
// registers are then free for the loads of tile t+2, which have the rest of this tile and the next barrier to arrive.
template <class AL, class BL, int SLOT, int W = 0>
__device__ __forceinline__ void split_side_slot(AL& al, BL& bl, uint32_t* as_next, uint32_t* bs_next, float4* ra,
                                                float4* rb, int kleft) {
  constexpr int TOTAL = AL::NS + BL::NS, SLOTS = 4, PER = (TOTAL + SLOTS - 1) / SLOTS, IDX = SLOT * PER + W;
  if constexpr (SLOT < SLOTS && W < PER) {
    if constexpr (IDX < AL::NS)
      al.store_step(IDX, as_next, ra);
    else if constexpr (IDX < TOTAL)
      bl.store_step(IDX - AL::NS, bs_next, rb);
    if constexpr (IDX == AL::NS - 1) al.fetch(ra, kleft);
    if constexpr (IDX == TOTAL - 1) bl.fetch(rb, kleft);
    split_side_slot<AL, BL, SLOT, W + 1>(al, bl, as_next, bs_next, ra, rb, kleft);
  }
}
template <class T, class AL, class BL, bool TR, int Q = 0>
__device__ __forceinline__ void split_groups(const uint32_t* as, const uint32_t* bs, SplitFrags<AL, T::TM>& fa,
                                             SplitFrags<BL, T::TN>& fb, v16f (&hi)[T::TM][T::TN],
                                             v16f (&lo)[T::TM][T::TN], AL& al, BL& bl, uint32_t* as_next, uint32_t* bs_next, float4* ra, float4* rb, int kleft) {
  if constexpr (Q < kSplitProducts) {
    // the terms of a plane are read shortly before their first use, so that three planes of A and two of B are live at
    // a time (with both by turns it was three of each, and 128 x 96 spilled)
    if constexpr (Q == 0) {
      fa.template read<0>(as);
      fb.template read<0>(bs);
      fa.template read<1>(as);
    }
    if constexpr (Q == 1) fa.template read<2>(as);
    if constexpr (Q == 2) fb.template read<1>(bs);
    if constexpr (Q == 4) fb.template read<2>(bs);
#pragma unroll
    for (int i = 0; i < T::TM; ++i)
#pragma unroll
      for (int j = 0; j < T::TN; ++j) {
        const v8bf a = fa.f[split_plane_a(Q)][i], b = fb.f[split_plane_b(Q)][j];
        v16f& c = Q == 0 ? hi[i][j] : lo[i][j];
        c = TR ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, c, 0, 0, 0)
               : __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
      }
    split_side_slot<AL, BL, Q>(al, bl, as_next, bs_next, ra, rb, kleft);
    __builtin_amdgcn_sched_barrier(0);
    split_groups<T, AL, BL, TR, Q + 1>(as, bs, fa, fb, hi, lo, al, bl, as_next, bs_next, ra, rb, kleft);
  }
}

// acc = the tile once more, by the fp32 matrix instructions (see above): rarely run, so short rather than fast
template <class T, class AL, class BL, bool TR>
__device__ __forceinline__ void split_redo(const typename AL::Params& ap, const typename BL::Params& bp, int g, int m0,
                                           int n0, int kbeg, int kend, float* as, float* bs,
                                           v16f (&acc)[T::TM][T::TN]) {
  static_assert(AL::UNITS * 4 >= T::BM * kRawLd && BL::UNITS * 4 >= T::BN * kRawLd, "the fp32 tile fits the terms' LDS");
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // so that nothing derived from it is kept from before the main loop: 10 registers a lane
  AL al(ap, g, tid, m0, kbeg);
  BL bl(bp, g, tid, n0, kbeg);
  const int lane = tid & 63, wave = tid >> 6;
  const float* a = as + ((wave % T::WAVES_M) * (T::TM * 32) + (lane & 31)) * kRawLd + (lane >> 5);
  const float* b = bs + ((wave / T::WAVES_M) * (T::TN * 32) + (lane & 31)) * kRawLd + (lane >> 5);
#pragma unroll
  for (int i = 0; i < T::TM; ++i)
#pragma unroll
    for (int j = 0; j < T::TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  for (int kleft = kend - kbeg; kleft > 0; kleft -= T::BK) {
    float4 ra[AL::NL], rb[BL::NL];
    al.fetch(ra, kleft);
    bl.fetch(rb, kleft);
    __syncthreads();  // the waves are done with what was there
    raw_store_all(al, as, ra);
    raw_store_all(bl, bs, rb);
    __syncthreads();
#pragma unroll 1
    for (int k = 0; k < T::BK; k += 2)
#pragma unroll
      for (int i = 0; i < T::TM; ++i)
#pragma unroll
        for (int j = 0; j < T::TN; ++j) {
          const float x = a[32 * i * kRawLd + k], y = b[32 * j * kRawLd + k];
          acc[i][j] = TR ? MfmaBlock<32>::mma(y, x, acc[i][j]) : MfmaBlock<32>::mma(x, y, acc[i][j]);
        }
  }
}

// Workgroups per compute unit: 128 x 128 has 128 accumulators a lane, which with everything else is 212 registers; 96 or
// 64 leave room for three.
template <class T>
struct SplitMinBlocks {
  static constexpr int value = T::BM * T::BN < 128 * 128 ? 3 : 2;
};

template <class T, class AL, class BL, class Epi>
__global__ void __launch_bounds__(kThreads, (SplitMinBlocks<T>::value))
gemm_split_kernel(typename AL::Params ap, typename BL::Params bp, Epi ep, int M, int N, int K, int kchunk,
                  SplitGrid grid) {
  static_assert(T::BK == kBKs && T::RB == 32, "16-deep k-tiles of 32 x 32 blocks");
  __shared__ __attribute__((aligned(16))) uint32_t As[2][AL::UNITS * 4];
  __shared__ __attribute__((aligned(16))) uint32_t Bs[2][BL::UNITS * 4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % T::WAVES_M, wn = wave / T::WAVES_M;
  const uint32_t total = gridDim.x, L = blockIdx.x, q8 = total >> 3, r8 = total & 7, xcd = L & 7;
  const uint32_t tile = xcd * q8 + min(xcd, r8) + (L >> 3);  // as in xcd_tile
  const uint32_t rest = fdiv(tile, grid.gy), place = fdiv(rest, grid.gx), turn = fdiv(place, grid.nsplit);
  const int split = (int)(place - turn * grid.nsplit.d);
  const uint32_t g = split_group(grid, turn), z = g * grid.nsplit.d + (uint32_t)split;
  const int n0 = (int)(tile - rest * grid.gy.d) * T::BN;
  const SplitPlace at = split_place<T>(grid, g, split, (int)(rest - place * grid.gx.d) * T::BM, M, K, kchunk);
  const int m0 = at.m0, kbeg = at.kbeg, kend = at.kend;
  if (grid.of == 1) {
    if (m0 >= at.M) return;
    split_row_limit(ap, at.M);
  }
  const int nt = kend > kbeg ? (kend - kbeg + T::BK - 1) / T::BK : 0;

  AL al(ap, (int)g, tid, m0, kbeg);
  BL bl(bp, (int)g, tid, n0, kbeg);
  ep.set_group((int)g, (int)z);

  v16f acc[T::TM][T::TN], lo[T::TM][T::TN];  // hh; the other term products
#pragma unroll
  for (int i = 0; i < T::TM; ++i)
#pragma unroll
    for (int j = 0; j < T::TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = lo[i][j][r] = 0.f;

  if (nt > 0) {
    const int kh = lane >> 5;
    const int a_off = split_unit<AL>(0, kh, wm * (T::TM * 32) + (lane & 31)) * 4;
    const int b_off = split_unit<BL>(0, kh, wn * (T::TN * 32) + (lane & 31)) * 4;
    // tile t is multiplied from LDS buffer t&1 while tile t+1 goes from registers to the other buffer and tile t+2
    // is fetched
    float4 ra[AL::NL], rb[BL::NL];
    al.fetch(ra, kend - kbeg);
    bl.fetch(rb, kend - kbeg);
    split_store_all(al, As[0], ra);
    split_store_all(bl, Bs[0], rb);
    al.fetch(ra, kend - kbeg - T::BK);
    bl.fetch(rb, kend - kbeg - T::BK);
    __syncthreads();
    for (int t = 0; t < nt; ++t) {
      const int p = t & 1;
      SplitFrags<AL, T::TM> fa;
      SplitFrags<BL, T::TN> fb;
      split_groups<T, AL, BL, kRowsAcross<Epi>>(As[p] + a_off, Bs[p] + b_off, fa, fb, acc, lo, al, bl, As[p ^ 1], Bs[p ^ 1],
                                                ra, rb, kend - kbeg - (t + 2) * T::BK);
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < T::TM; ++i)
#pragma unroll
      for (int j = 0; j < T::TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = (acc[i][j][r] + lo[i][j][r]) * kSplitUnscale;
    float top = 0.f;  // the largest magnitude, NaN if there is one: one v_maximum3_f32 for two sums
#pragma unroll
    for (int i = 0; i < T::TM; ++i)
#pragma unroll
      for (int j = 0; j < T::TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; r += 2)
          top = __builtin_elementwise_maximum(__builtin_elementwise_maximum(top, fabsf(acc[i][j][r])),
                                              fabsf(acc[i][j][r + 1]));
    const bool bad = __any(!(top <= 3.402823466e38f));
    if (lane == 0) As[0][wave] = bad;
    __syncthreads();
    if ((As[0][0] | As[0][1] | As[0][2] | As[0][3]) != 0)
      split_redo<T, AL, BL, kRowsAcross<Epi>>(ap, bp, (int)g, m0, n0, kbeg, kend, reinterpret_cast<float*>(As[0]),
                                              reinterpret_cast<float*>(Bs[0]), acc);
  }

  store_rows(ep, acc, m0 + wm * (T::TM * 32), n0 + wn * (T::TN * 32), at.M, N, lane);
}
#endif  // AX_HOST_EMU

}  // namespace ax
