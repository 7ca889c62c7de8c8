// Weight gradients of the convolutions of bf16 handles, over operands stored as bf16 (see gemm_bf16.h).
//
// The reduction runs over pixels, along which neither operand is contiguous: in LDS they stand as in memory, rows of 64
// channels per pixel, while a matrix instruction wants eight pixels of one channel in a lane.  gemm_bf16.h's kernel, which this
// one replaces, fetched two pixels into registers, interleaved them and wrote pairs to LDS, to read a fragment in four words.
// Here the loads go to LDS directly (gemm_direct.h: two stages of 64 k, a builtin for the wait), and ds_read_b64_tr_b16
// transposes on the way out.
//
// LDS: blocks of 64 rows (channels of a tap, output channels), a row of 128 bytes per pixel, eight 16-byte slots; slot s of
// pixel k holds octet s ^ 4*((k >> 1) & 1), so that the four pixels x 64 bytes that half a wave reads lie in different banks.
// A load fills eight pixels of one block; its lane keeps one octet of rows, hence one tap, whatever the pixel.  A wave decodes
// the 64 pixels of its next four k-tiles at once, one per lane, and passes origin and mask of the taps outside on by shuffles:
// no table, so no limit on the length of a slice and no k-tile left to other kernels.
//
// Product alone, batch 256 and 64, us: second layer 144 and 39 (797 TFLOP/s at 256), third 90 and 29, fourth 84 and 27, fifth
// 46 and 20.  In a training pass, gemm_bf16.h's kernel | here: batch 256 second layer 248 | 137, third 136 | 86, fourth 137 |
// 87, fifth, beside the dense layers' update, 106 | 84; batch 64 70 | 45, 67 | 32, 97 | 77, 49 | 32.  What bounds it: at 128 x
// 128 the reads from LDS (a kilobyte for each matrix instruction of a wave, as much as LDS gives), at 192 x 128 power.
//
// A training pass adds up the slices of all layers at its end, see WgradTail: the sums of a layer, in a launch of their own
// beside the dense layers' update, took 14 to 450 us, by where that kernel's workgroups had found room.
#include <algorithm>

#include "gemm_direct.h"
#include "kernels.h"

namespace ax {

// One weight-gradient product: C[(r,s,c)][o] = sum over pixels of x[pixel + tap][c] * dy[pixel][o]
struct DirectTJob {
  Im2colParams a;
  DenseParams b;
  int M, N, K, tiles_per_slice;
  FastDiv gx, gy, ns;
};

typedef short v4s __attribute__((ext_vector_type(4)));
// Sixteen lanes read a block of 4 k x 16 rows (lane i: four rows from 4*(i%4) at k i/4); lane i gets row i at the four k.
__device__ __forceinline__ v4s read_transposed(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)p);
}

// A_K: the first operand is contiguous along the reduction, a.x[row][k] with a.Cg values of k (gradients of dense layers'
// inputs), and stands in LDS as in gemm_direct.h; the second one is transposed on the way out all the same.
template <int BM, int BN, int WAVES_M, int WAVES_N, int MINB, bool A_K, class Epi>
__global__ void __launch_bounds__(256, MINB) gemm_direct_t_kernel(DirectTJob j, Epi ep) {
  static_assert(WAVES_M * WAVES_N == 4 && BM % 64 == 0 && BN % 64 == 0, "four waves, blocks of 64");
  constexpr int TM = BM / (32 * WAVES_M), TN = BN / (32 * WAVES_N);
  constexpr int CA = BM / 64, CB = BN / 64;  // blocks of 64 rows
  constexpr int kBlock = kBKd * 8;           // units of a block: 64 k of eight octets
  __shared__ __attribute__((aligned(16))) v4u stage0[(CA + CB) * kBlock];
  __shared__ __attribute__((aligned(16))) v4u stage1[(CA + CB) * kBlock];
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

  // A load brings the octets of eight pixels in one block: lane = (pixel, slot).  A wave loads pixels 16*wave .. 16*wave + 15.
  const int sub = lane >> 3, oct = (lane & 7) ^ (4 * ((sub >> 1) & 1));
  constexpr int NA = BM / 32;  // A_K: loads per lane and k-tile, eight rows each
  const int k_oct = (lane & 7) ^ sub;
  uint32_t tapoff[CA], tapmask[CA], bcol[CB], arow[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int m = m0 + (i * 4 + wave) * 8 + sub;
    arow[i] = m < j.M ? ((uint32_t)m * (uint32_t)ap.Cg + 8u * k_oct) * 2u : kOob;
  }
#pragma unroll
  for (int b = 0; b < CA; ++b) {
    const int m = m0 + 64 * b + 8 * oct;
    const bool in = m < j.M;
    const TapCoord t = decode_tap(in ? m : 0, ap);
    tapoff[b] = (((uint32_t)t.r * (uint32_t)ap.W + (uint32_t)t.s) * (uint32_t)ap.Ctot + (uint32_t)t.c +
                 (uint32_t)((int)g * ap.c_stride_g)) * 2u;
    tapmask[b] = in ? 1u << (t.r * ap.kw + t.s) : 0x80000000u;
  }
#pragma unroll
  for (int b = 0; b < CB; ++b) {
    const int n = n0 + 64 * b + 8 * oct;
    bcol[b] = n < j.N ? (uint32_t)n * 2u : kOob;  // less than 2^31 is added: stays outside
  }
  ep.set_group((int)g, (int)z);

  uint32_t pbase = 0, poutside = 0;  // of this lane's pixel: 16*wave + lane % 16 of k-tile t + lane / 16, t a multiple of four
  auto load = [&](v4u* st, int t) {
    const int k0 = (first + t) * kBKd + 16 * wave;
    if (A_K) {
      const uint32_t k = (uint32_t)(first + t) * kBKd;
      const bool in = (int)k + 8 * k_oct < j.K;
#pragma unroll
      for (int i = 0; i < NA; ++i) load_lds16(av, st + (i * 4 + wave) * 64, in ? arow[i] + 2u * k : kOob, 0);
    } else if ((t & 3) == 0) {
      const int p = k0 + (lane >> 4) * kBKd + (lane & 15);
      const bool in = p < ap.P;
      const PixCoord c = decode_pixel(in ? p : 0, ap);
      const int y0 = c.y * ap.stride - ap.pad, x0 = c.x * ap.stride_x - ap.pad_x;
      pbase = row_base<IM2COL_FWD, 2>(ap, c.n, y0, x0, 0);
      poutside = in ? ~taps_inside<IM2COL_FWD>(ap, y0, x0) | 0x80000000u : 0xffffffffu;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if (!A_K) {
        const int from = (t & 3) * 16 + i * 8 + sub;
        const uint32_t base = (uint32_t)__shfl((int)pbase, from), outside = (uint32_t)__shfl((int)poutside, from);
#pragma unroll
        for (int b = 0; b < CA; ++b)
          load_lds16(av, st + b * kBlock + (2 * wave + i) * 64, outside & tapmask[b] ? kOob : base + tapoff[b], 0);
      }
      const uint32_t brow = (uint32_t)(k0 + i * 8 + sub) * (uint32_t)j.b.ld * 2u;  // past the last pixel: outside
#pragma unroll
      for (int b = 0; b < CB; ++b) load_lds16(bv, st + (CA + b) * kBlock + (2 * wave + i) * 64, brow + bcol[b], 0);
    }
  };

  v16f acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int jj = 0; jj < TN; ++jj)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][jj][r] = 0.f;
  // Element e of a lane's eight values is k = 8*(e/4) + 4*kh + e%4 of a step, in both operands; A_K: k = 8*kh + e.  Bytes of lane
  // (k, rows) in a block, for its first and its second 32 rows:
  constexpr int kSecond = A_K ? 512 : 1024;  // from the first four of them to the second
  const int l16 = lane & 15, kk = l16 >> 2, half_row = ((lane >> 4) & 1) * 2 + ((l16 & 3) >> 1);
  const int kh = lane >> 5, lane_k = ((A_K ? 8 : 4) * kh + kk) * 128 + (l16 & 1) * 8;
  const int at0 = lane_k + (half_row ^ (4 * (kk >> 1))) * 16, at1 = at0 ^ 64;
  int a_at[TM], b_at[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int blk = wm * TM + i;
    a_at[i] = A_K ? (blk * 32 + (lane & 31)) * 128 : (blk >> 1) * (kBlock * 16) + (blk & 1 ? at1 : at0);
  }
#pragma unroll
  for (int jj = 0; jj < TN; ++jj) {
    const int blk = wn * TN + jj;
    b_at[jj] = (CA + (blk >> 1)) * (kBlock * 16) + (blk & 1 ? at1 : at0);
  }
  auto multiply = [&](const v4u* st) {
    const char* s = reinterpret_cast<const char*>(st);
    struct Two {
      v4s lo, hi;
    };
#pragma unroll
    for (int ks = 0; ks < kBKd / 16; ++ks) {
      v8bf a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i)
        a[i] = A_K ? __builtin_bit_cast(v8bf, *reinterpret_cast<const v4u*>(s + a_at[i] + ((2 * ks + kh) ^ (lane & 7)) * 16))
                   : __builtin_bit_cast(v8bf, Two{read_transposed(s + a_at[i] + ks * 2048), read_transposed(s + a_at[i] + ks * 2048 + kSecond)});
#pragma unroll
      for (int jj = 0; jj < TN; ++jj)
        b[jj] = __builtin_bit_cast(v8bf, Two{read_transposed(s + b_at[jj] + ks * 2048), read_transposed(s + b_at[jj] + ks * 2048 + kSecond)});
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jj = 0; jj < TN; ++jj)
          acc[i][jj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[jj], acc[i][jj], 0, 0, 0);
    }
  };
  if (nt > 0) {
    load(stage0, 0);
    int t = 0;
    for (; t + 2 < nt; t += 2) {
      direct_barrier();
      load(stage1, t + 1);
      multiply(stage0);
      direct_barrier();
      load(stage0, t + 2);
      multiply(stage1);
    }
    direct_barrier();
    if (t + 1 < nt) {
      load(stage1, t + 1);
      multiply(stage0);
      direct_barrier();
      multiply(stage1);
    } else {
      multiply(stage0);
    }
  }

  store_rows(ep, acc, m0 + wm * (TM * 32), n0 + wn * (TN * 32), j.M, j.N, lane);
}

// Time of a product in slices, as plan_direct() has it: workgroups on the busiest compute unit in rounds of as many as it
// holds, n of them first[n-1] + each[n-1] * MFLOP of a tile's slice.  Fitted to 330 launches (second to fifth layer, batch 64
// and 256, 1 to 48 slices), which it meets within 7 %.  Adding the slabs up takes 2.6 us and, right behind the product, 8 TB/s; a training pass adds up all
// layers' slabs at its end, when they have gone to memory and back: 3 TB/s.
struct DirectTTile {
  int bm, bn, occ;
  double first[3], each[3];
};
static const DirectTTile kDirectTTiles[] = {{128, 64, 3, {0.9, 4.0, 3.0}, {0.636, 0.765, 0.97}},
                                            {128, 128, 2, {4.0, 4.5, 0}, {0.388, 0.50, 0}},
                                            {192, 128, 2, {5.2, 7.6, 0}, {0.328, 0.437, 0}}};
constexpr int kDirectTSlices = 64;
struct DirectTPlan {
  int tile, ns, per;  // per: k-tiles of a slice
};
static DirectTPlan plan_direct_t(const GemmDims& d) {
  const int ktiles = ceil_div(d.K, kBKd);
  DirectTPlan best{0, 1, ktiles};
  double best_t = 1e30;
  for (int o = 0; o < 3; ++o) {
    const DirectTTile& to = kDirectTTiles[o];
    const long tiles = (long)ceil_div(d.M, to.bm) * ceil_div(d.N, to.bn) * d.groups;
    for (int s = 1; s <= kDirectTSlices && s <= ktiles; ++s) {
      const int per = ceil_div(ktiles, s);
      if (ceil_div(ktiles, per) != s) continue;
      const int c = ceil_div(tiles * s, 256), rest = c % to.occ;
      const double f = 2e-6 * to.bm * to.bn * (double)per * kBKd;
      double t = c / to.occ * (to.first[to.occ - 1] + to.each[to.occ - 1] * f);
      if (rest) t += to.first[rest - 1] + to.each[rest - 1] * f;
      if (s > 1) t += 2.6 + (s + 1) * 4e-6 * d.M * d.N * (double)d.groups / 3;
      if (t < best_t) {
        best_t = t;
        best = DirectTPlan{o, s, per};
      }
    }
  }
  return best;
}
bool direct_bwd_weight_ok(const ConvGeom& c) { return conv_bf16_stored_ok(c) && c.k * c.k < kDirectTaps; }
int direct_bwd_weight_slices(const ConvGeom& c) { return plan_direct_t(bwdw_dims(c)).ns; }
template <int BM, int BN, int WM, int WN, int MINB, bool A_K = false, class Epi>
static int launch_direct_t_tile(const DirectTPlan& p, const Im2colParams& a, const DenseParams& b, const Epi& e,
                                const GemmDims& d, double bytes, hipStream_t st) {
  DirectTJob j;
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
  KernelScope ks("gemm_bf16", 2.0 * d.M * d.N * (double)d.K * d.groups,
                 bytes, st);
  hipLaunchKernelGGL((gemm_direct_t_kernel<BM, BN, WM, WN, MINB, A_K, Epi>), dim3((unsigned)((long)gx * gy * d.groups * p.ns)),
                     dim3(kThreads), 0, st, j, e);
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}
template <class Epi>
static int launch_direct_t(const DirectTPlan& p, const Im2colParams& a, const DenseParams& b, const Epi& e, const GemmDims& d,
                           double bytes, hipStream_t st) {
  if (p.tile == 0) return launch_direct_t_tile<128, 64, 4, 1, 3>(p, a, b, e, d, bytes, st);
  if (p.tile == 1) return launch_direct_t_tile<128, 128, 2, 2, 2>(p, a, b, e, d, bytes, st);
  return launch_direct_t_tile<192, 128, 2, 2, 2>(p, a, b, e, d, bytes, st);
}

int launch_direct_bwd_weight(const ConvGeom& c, const uint16_t* x16, const uint16_t* dy16, float* out, hipStream_t st) {
  const GemmDims d = bwdw_dims(c);
  const EpiSlab ep{out, (long)d.M * d.N, d.N, nullptr};
  const double bytes = 4.0 * ((double)c.in_elems() + (double)c.w_elems() + (double)c.out_elems());
  return launch_direct_t(plan_direct_t(d), im2col16(bwdw_A(c, nullptr), x16),
                         dense16(bwdw_B(c, nullptr), dy16), ep, d, bytes, st);
}

// ---- dense layers ----
int launch_direct_dense_bwd_data(int B, int in, int out, const uint16_t* dy16, const uint16_t* w16, float* slabs, hipStream_t st) {
  const GemmDims d{B, in, out, 1};
  const ConvGeom rows{B, 1, 1, out, in, 1, 1, 0, 1, 1, 1};
  DenseParams b;
  b.p = reinterpret_cast<const float*>(w16); b.ld = in; b.gstride = 0; b.R = in; b.bytes = (uint32_t)((size_t)in * out * 2);
  const Im2colParams a = im2col16(fwd_A(rows, nullptr), dy16);
  const EpiSlab e{slabs, (long)B * in, in, nullptr};
  const double bytes = 4.0 * ((double)B * (in + out) + (double)in * out);
  const DensePlan dp = dense_plan(B, in, out);
  const DirectTPlan p{0, dp.ns, dp.per};
  if (dp.tall) return launch_direct_t_tile<128, 128, 2, 2, 2, true>(p, a, b, e, d, bytes, st);
  return launch_direct_t_tile<64, 128, 2, 2, 3, true>(p, a, b, e, d, bytes, st);
}
// The weight gradient of a 1 x 1 convolution over pictures of one pixel, with the operands' parts exchanged.  Its reduction is
// the batch, so that it waits for its stores; 128-row tiles from 65 pictures up (batch 64, 9216 x 4096: 28 us in those, 26 in
// these; 256: 50 and 59).  gemm_bf16.h | here: batch 256 49, 27, 13 | 50, 20, 11 us, batch 64 33, 18, 10 | 26, 13, 7.
int launch_direct_dense_bwd_weight(int B, int in, int out, const uint16_t* x16, const uint16_t* dy16, float* dw, hipStream_t st,
                                   const SgdArgs* u) {
  const GemmDims d{out, in, B, 1};
  const ConvGeom c{B, 1, 1, out, in, 1, 1, 0, 1, 1, 1};
  const Im2colParams a = im2col16(bwdw_A(c, nullptr), dy16);
  const DenseParams b = dense16(bwdw_B(c, nullptr), x16);
  const double bytes = 4.0 * ((double)B * (in + out) + (u ? 5.0 : 1.0) * (double)in * out);
  const DirectTPlan p{0, 1, ceil_div(B, kBKd)};
  if (u) {
    const EpiSgd e{dw, u->w, u->v, in, u->lr, u->mu, u->wd};
    if (B > 64) return launch_direct_t_tile<128, 128, 2, 2, 2>(p, a, b, e, d, bytes, st);
    return launch_direct_t_tile<64, 128, 2, 2, 3>(p, a, b, e, d, bytes, st);
  }
  const EpiSlab e{dw, (long)out * in, in, nullptr};
  if (B > 64) return launch_direct_t_tile<128, 128, 2, 2, 2>(p, a, b, e, d, bytes, st);
  return launch_direct_t_tile<64, 128, 2, 2, 3>(p, a, b, e, d, bytes, st);
}

}  // namespace ax
