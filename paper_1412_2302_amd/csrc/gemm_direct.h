// bf16 products whose operands go from memory to LDS directly (buffer_load ... lds): the convolutions of bf16 handles whose
// channels per group are a multiple of 64 (or of eight, at some cost), forward and backward-data, over operands stored as
// bf16 (the "16" tensors of gemm_bf16.h).
//
// What paces gemm_bf16.h's kernels is neither memory nor the matrix cores but the way through the workgroup: loads to
// registers, registers to LDS, an address per load and k-tile, a barrier per 32 k.  Here a load names its LDS destination, so
// the operands pass no register; a k-tile is 64 deep, the 128 bytes of one pixel's channels that a cache line holds, and lies
// inside one tap, so that an address is an add and a test of the tap's bit -- for the weights nothing, k runs in the scalar
// offset.
//
// LDS: rows of eight 16-byte units, unit (row, slot).  A load instruction fills 64 consecutive units, so eight lanes bring one
// row; the lane of slot s brings octet s ^ (row & 7) of it, and a fragment read of one octet of eight rows touches all banks.
// Two stages: the next k-tile is on its way during the whole of this one's products, with a second workgroup on the compute
// unit to fill the waits.  Each stage is an array of its own and the wait a builtin, which is what tells the compiler that
// reads of one stage need not wait for the loads of the other (with the wait in asm every second k-tile waited for the loads
// it had just issued: 107 us instead of 92).
//
// Alone, batch 256 (gemm_bf16.h and gemm16.h | here): third layer forward 112 | 88 us (870 TFLOP/s), its data gradient 111 |
// 82, fourth forward 83 | 82, fifth 62 | 50, second layer's data gradient (48 of 64 columns) 235 | 187; batch 64: 38 | 29,
// 49 | 36, 38 | 24, 29 | 22.  In a pass with real weights the clock is lower: 113 | 105, 101 | 79, 91 | 95, 66 | 59, 235 |
// 172, the data gradients of the fourth and fifth layers beside the dense layers' update 422 | 361; so forward products of
// 192 columns with many tiles stay with gemm16.h (inference of 256 pictures 92 | 100 us).  Forward products over 16 or 48
// channels are patch_conv.hip's where they fit.  With the results stored a row of the matrix at a time (epi_rows.h) a pass
// of 256 pictures has 105 | 87, 78, 95 | 78 and 59 | 46 us.  Three stages of 32 k, 256-row tiles of eight waves and 192 x 192
// tiles (spills) were slower.  What bounds it: power, and a tile's first and last microseconds, about nine of the 26 of a 192
// x 128 tile with K = 1728; see plan_direct().
#pragma once

#include "conv_plan.h"
#include "epi_rows.h"
#include "gemm_bf16.h"

namespace ax {

constexpr int kBKd = 64;
constexpr int kDirectTaps = 32;  // bits of a lane's mask

// One product; ns slices of the reduction in units of kBKd
struct DirectJob {
  Im2colParams a;
  DenseParams b;
  int M, N, K, tiles_per_slice;
  FastDiv gx, gy, ns;
};

// Products of dense layers, rows = pictures: they wait for the weights, which come from memory once, so that what counts is how
// many loads are on their way.  Two workgroups per compute unit by slices of the reduction (at least two k-tiles each), from
// 64-row tiles unless there are more than 32 of 128 rows.  With sums and activation in front of gemm_bf16.h's 128 x 128 | here,
// us, 4096 and 1000 outputs: batch 256 of 9216, 4096, 4096 inputs 57, 32, 21 | 41, 27, 16, data gradients 64, 34, 19 | 52, 25,
// 17; batch 64 35, 22, 15 | 31, 20, 12 and 51, 21, 16 | 37, 16, 12.  One workgroup per compute unit (256 rows, 9216 inputs):
// 72; four: 49 and more.
struct DensePlan {
  bool tall;  // 128 x 128, else 64 x 128
  int ns, per;
};
inline DensePlan dense_plan(int rows, int cols, int K) {
  const int ktiles = (K + kBKd - 1) / kBKd;
  DensePlan p;
  p.tall = (long)((rows + 127) / 128) * ((cols + 127) / 128) > 32;
  const long tiles = (long)((rows + (p.tall ? 127 : 63)) / (p.tall ? 128 : 64)) * ((cols + 127) / 128);
  long ns = 512 / tiles;
  ns = ns > 32 ? 32 : ns;
  ns = ns > ktiles / 2 ? ktiles / 2 : ns;
  ns = ns < 1 ? 1 : ns;
  p.per = (int)((ktiles + ns - 1) / ns);
  p.ns = (ktiles + p.per - 1) / p.per;
  return p;
}

// Taps of a kernel (at most 32) that lie inside the tensor, seen from (y0, x0): bit r*kw + s
template <int MODE>
AX_HD uint32_t taps_inside(const Im2colParams& g, int y0, int x0) {
  int lo = MODE == IM2COL_FWD ? -x0 : x0 - g.W + 1, hi = MODE == IM2COL_FWD ? g.W - x0 : x0 + 1;
  lo = lo < 0 ? 0 : lo;
  hi = hi > g.kw ? g.kw : hi;
  const uint32_t xs = hi > lo ? (uint32_t)((1ull << hi) - (1ull << lo)) : 0u;
  uint32_t inside = 0;
  for (int r = 0; r < g.kh; ++r) {
    const int iy = MODE == IM2COL_FWD ? y0 + r : y0 - r;
    inside |= (uint32_t)iy < (uint32_t)g.H ? xs << (r * g.kw) : 0u;
  }
  return inside;
}

// The tap (bit r*kw + s) and the channel of a lane's octet, k-tile by k-tile.  ONE_TAP: k-tiles divide the channels, the tap's
// column is carried along.  Otherwise a k-tile goes one step through whole taps and the rest of one, without a branch: lanes
// stand at different taps (with a loop over the taps passed the second layer's forward product of 64 pictures, 48 channels,
// took 90 us).
template <bool ONE_TAP>
struct TapWalk {
  int bit, ch, tx;
  uint32_t tap;
  int step_taps, step_ch;
  AX_HD TapWalk(const Im2colParams& a, int k) {
    bit = (int)fdiv((uint32_t)k, a.d_cg);
    ch = k - bit * a.Cg;
    const int ty = (int)fdiv((uint32_t)bit, a.d_kw);
    tx = bit - ty * a.kw;
    tap = ((uint32_t)ty * (uint32_t)a.W + (uint32_t)tx) * (uint32_t)a.Ctot * 2u;
    step_taps = (int)fdiv(kBKd, a.d_cg);
    step_ch = kBKd - step_taps * a.Cg;
  }
  // of the tap, in bytes from a pixel's origin
  AX_HD uint32_t offset(const Im2colParams& a) const {
    if (ONE_TAP) return tap;
    return ((uint32_t)bit + fdiv((uint32_t)bit, a.d_kw) * (uint32_t)(a.W - a.kw)) * (uint32_t)a.Ctot * 2u;
  }
  AX_HD void next(const Im2colParams& a) {
    if (ONE_TAP) {
      ch += kBKd;
      if (ch == a.Cg) {
        ch = 0;
        ++bit;
        const bool row = ++tx == a.kw;
        tap += (uint32_t)(row ? a.W - a.kw + 1 : 1) * (uint32_t)a.Ctot * 2u;
        tx = row ? 0 : tx;
      }
      return;
    }
    ch += step_ch;
    const int over = ch >= a.Cg;
    bit += step_taps + over;
    ch -= over ? a.Cg : 0;
  }
};

#ifndef AX_HOST_EMU
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void load_lds16(const BufView& v, v4u* dst, uint32_t off, uint32_t soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(v, (__attribute__((address_space(3))) void*)dst, 16, (int)off, (int)soff, 0, 0);
}
// every load to LDS of this wave has arrived and every LDS read is done; then the workgroup meets
__device__ __forceinline__ void direct_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// ONE_TAP: channels per group are a multiple of 64, so a k-tile lies inside one tap; else a multiple of eight, and an octet
// does.
template <int BM, int BN, int WAVES_M, int WAVES_N, int MINB, bool ONE_TAP, int MODE, class Epi>
__global__ void __launch_bounds__(256, MINB) gemm_direct_kernel(DirectJob j, Epi ep) {
  static_assert(WAVES_M * WAVES_N == 4, "four waves");
  constexpr int TM = BM / (32 * WAVES_M), TN = BN / (32 * WAVES_N);
  constexpr int NA = BM / 32, NB = BN / 32;  // loads per lane and k-tile
  __shared__ __attribute__((aligned(16))) v4u stage0[(BM + BN) * 8];
  __shared__ __attribute__((aligned(16))) v4u stage1[(BM + BN) * 8];
  const Im2colParams& ap = j.a;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WAVES_M, wn = wave / WAVES_M;
  const uint32_t total = gridDim.x, L = blockIdx.x, q8 = total >> 3, r8 = total & 7, xcd = L & 7;
  const uint32_t tile = xcd * q8 + min(xcd, r8) + (L >> 3);  // as in xcd_tile
  const uint32_t rest = fdiv(tile, j.gy), z = fdiv(rest, j.gx), g = fdiv(z, j.ns);
  const int m0 = (int)(rest - z * j.gx.d) * BM, n0 = (int)(tile - rest * j.gy.d) * BN;
  const int first = (int)(z - g * j.ns.d) * j.tiles_per_slice;
  const int nt = min((j.K + kBKd - 1) / kBKd - first, j.tiles_per_slice);

  const BufView av = make_view(ap.x, ap.bytes);
  const BufView bv = make_view(reinterpret_cast<const float*>(reinterpret_cast<const uint16_t*>(j.b.p) + (long)g * j.b.gstride),
                               j.b.bytes - (uint32_t)(g * j.b.gstride * 2));
  const int sub = lane >> 3, oct = (lane & 7) ^ sub;  // row of the eight that a load brings, and the octet of it
  uint32_t rowbase[NA], outside[NA], brow[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int n = min(n0 + (i * 4 + wave) * 8 + sub, j.N - 1);  // columns past the end repeat the last one and are not stored
    brow[i] = ((uint32_t)n * (uint32_t)j.b.ld + 8u * oct) * 2u;
  }
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int p = m0 + (i * 4 + wave) * 8 + sub;
    const PixCoord c = decode_pixel(p < ap.P ? p : 0, ap);
    const int y0 = MODE == IM2COL_FWD ? c.y * ap.stride - ap.pad : c.y + ap.pad;
    const int x0 = MODE == IM2COL_FWD ? c.x * ap.stride_x - ap.pad_x : c.x + ap.pad;
    rowbase[i] = row_base<MODE, 2>(ap, c.n, y0, x0, (int)g * ap.c_stride_g + (ONE_TAP ? 8 * oct : 0));
    outside[i] = p < ap.P ? ~taps_inside<MODE>(ap, y0, x0) : 0xffffffffu;
  }
  ep.set_group((int)g, (int)z);

  // The octet to load next: of the k-tile, the same for every lane (ONE_TAP; the lane's octet is in rowbase then), or the lane's own.
  int k = first * kBKd + (ONE_TAP ? 0 : 8 * oct);
  TapWalk<ONE_TAP> walk(ap, k);
  uint32_t bk = (uint32_t)(first * kBKd) * 2u;
  auto load = [&](v4u* st) {
    const uint32_t tap = walk.offset(ap), off = (MODE == IM2COL_FWD ? tap : 0u - tap) + (uint32_t)walk.ch * 2u;
    const bool in = ONE_TAP || k < j.K;  // the last k-tile may lie partly past the end
    const uint32_t bit = 1u << (walk.bit & 31), b_off = in ? bk : kOob;  // kOob and less than 2^31: outside
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const uint32_t out = ONE_TAP ? outside[i] & bit : (in ? outside[i] : 0xffffffffu) & bit;
      load_lds16(av, st + (i * 4 + wave) * 64, out ? kOob : rowbase[i] + off, 0);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if (ONE_TAP)
        load_lds16(bv, st + BM * 8 + (i * 4 + wave) * 64, brow[i], bk);
      else
        load_lds16(bv, st + BM * 8 + (i * 4 + wave) * 64, brow[i] + b_off, 0);
    }
    bk += kBKd * 2;
    k += kBKd;
    walk.next(ap);
  };

  v16f acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int jj = 0; jj < TN; ++jj)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][jj][r] = 0.f;
  const int row = lane & 31, kh = lane >> 5;
  const int a_row = (wm * (TM * 32) + row) * 8, b_row = (BM + wn * (TN * 32) + row) * 8;
  auto multiply = [&](const v4u* st) {
#pragma unroll
    for (int ks = 0; ks < kBKd / 16; ++ks) {
      const int slot = (2 * ks + kh) ^ (row & 7);
      v8bf a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = __builtin_bit_cast(v8bf, st[a_row + slot + i * 256]);
#pragma unroll
      for (int jj = 0; jj < TN; ++jj) b[jj] = __builtin_bit_cast(v8bf, st[b_row + slot + jj * 256]);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jj = 0; jj < TN; ++jj)
          acc[i][jj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[jj], acc[i][jj], 0, 0, 0);
    }
  };
  if (nt > 0) {
    load(stage0);
    int t = 0;
    for (; t + 2 < nt; t += 2) {
      direct_barrier();
      load(stage1);
      multiply(stage0);
      direct_barrier();
      load(stage0);
      multiply(stage1);
    }
    direct_barrier();
    if (t + 1 < nt) {
      load(stage1);
      multiply(stage0);
      direct_barrier();
      multiply(stage1);
    } else {
      multiply(stage0);
    }
  }

  store_rows(ep, acc, m0 + wm * (TM * 32), n0 + wn * (TN * 32), j.M, j.N, lane);
}
#endif  // AX_HOST_EMU

}  // namespace ax
