// Forward products of bf16 handles over layers with 16 or 48 channels per group, from pictures in LDS.
//
// With channels that are no multiple of 64 the taps' octets lie in pieces of 32 and 96 bytes across cache lines, and a tile that
// gathers them tap by tap (gemm_direct.h) waits for the second-level cache: 192 x 128 tiles of the second layer moved 160 KB a
// k-tile and compute unit, 3 us for 0.7 us of products.  Here a workgroup loads the rows of the picture under a band of output
// rows once and reads every tap's fragments from LDS; only the weights stream, a tap at a time, three stages.
//
// LDS: pixels of U = channels / 8 units of 16 bytes, an odd multiple of two; a pixel whose number has bit 2 set has its units
// exchanged in pairs, so that a fragment read of one octet of eight neighbouring pixels touches all banks.  The same for the
// weights' columns.  Two workgroups to a compute unit.
//
// Second layer (27 x 27, 48 channels, 5 x 5, 128 columns a group), gathered | here: 256 pictures 161 | 104 us (1100 TFLOP/s), 64
// 55 | 33.  With two stages, whose loads had a tap's products alone to arrive under, 118 and 46.  What bounds it: power at 256
// pictures; at 64, one round of two workgroups a unit, the picture's way in and the results' way out.
#include <algorithm>

#include "gemm_direct.h"
#include "kernels.h"

namespace ax {

// units of a picture's rows beside three stages of the weights, of 64 or 128 columns: 80 KiB together
constexpr int patch_units(bool tall) { return tall ? 3584 : 2560; }

struct PatchGeom {
  const uint16_t *x, *w;  // w[g][column][(r, s, c)]
  uint32_t x_bytes, w_bytes;
  int H, W, Ctot, Ho, Wo, pad, k, N, rows;  // rows: output rows of a band
  int PW;                                   // W + 2 pad
  int bands, groups;
  uint32_t wgroup;                          // bytes between groups of w
  FastDiv d_pw, d_wo, d_cols, d_groups, d_bands;
};

template <int U, int WAVES_M, int WAVES_N, int TM, int TN, class Epi>
__global__ void __launch_bounds__(256, 2) patch_conv_kernel(PatchGeom g, Epi ep) {
  static_assert(WAVES_M * WAVES_N == 4 && U % 4 == 2, "four waves; an odd number of pairs");
  constexpr int BN = WAVES_N * TN * 32;
  constexpr int NB = (BN * U + 255) / 256;  // loads of a lane and tap; what they bring past the last column is zero
  __shared__ __attribute__((aligned(16))) v4u patch[patch_units(WAVES_N == 1)];
  __shared__ __attribute__((aligned(16))) v4u stage0[NB * 256];
  __shared__ __attribute__((aligned(16))) v4u stage1[NB * 256];
  __shared__ __attribute__((aligned(16))) v4u stage2[NB * 256];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WAVES_M, wn = wave / WAVES_M;
  const uint32_t total = gridDim.x, L = blockIdx.x, q8 = total >> 3, r8 = total & 7, xcd = L & 7;
  const uint32_t tile = xcd * q8 + min(xcd, r8) + (L >> 3);  // as in xcd_tile
  const uint32_t t1 = fdiv(tile, g.d_cols), t2 = fdiv(t1, g.d_groups), n = fdiv(t2, g.d_bands);
  const int n0 = (int)(tile - t1 * g.d_cols.d) * BN, grp = (int)(t1 - t2 * g.d_groups.d);
  const int y0 = (int)(t2 - n * g.d_bands.d) * g.rows, valid = min(g.rows, g.Ho - y0);
  const BufView xv = make_view(reinterpret_cast<const float*>(g.x), g.x_bytes);
  const BufView wv = make_view(reinterpret_cast<const float*>(g.w), g.w_bytes);

  // a picture's rows y0 - pad .. y0 - pad + valid + k - 2, zero outside it
  const int units = (valid + g.k - 1) * g.PW * U;
  for (int u0 = wave * 64; u0 < units; u0 += 256) {  // uniform
    const int u = u0 + lane, p = u / U, c = (u - p * U) ^ (p >> 2 & 1);
    const int py = (int)fdiv((uint32_t)p, g.d_pw), px = p - py * g.PW;
    const int iy = y0 + py - g.pad, ix = px - g.pad;
    const bool in = u < units && (uint32_t)iy < (uint32_t)g.H && (uint32_t)ix < (uint32_t)g.W;
    const uint32_t at = (((n * (uint32_t)g.H + (uint32_t)iy) * (uint32_t)g.W + (uint32_t)ix) * (uint32_t)g.Ctot + (uint32_t)(grp * 8 * U + 8 * c)) * 2u;
    load_lds16(xv, patch + u0, in ? at : kOob, 0);
  }
  // a tap's weights: units of this lane
  uint32_t wat[NB];
  const uint32_t K2 = (uint32_t)(g.k * g.k * 8 * U) * 2u;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int u = (i * 4 + wave) * 64 + lane, col = u / U, c = (u - col * U) ^ (col >> 2 & 1);
    wat[i] = u < BN * U ? (uint32_t)grp * g.wgroup + (uint32_t)(n0 + col) * K2 + 16u * c : kOob;
  }
  auto load = [&](v4u* st, int tap) {
#pragma unroll
    for (int i = 0; i < NB; ++i) load_lds16(wv, st + (i * 4 + wave) * 64, wat[i] + (uint32_t)tap * (16u * U), 0);
  };
  ep.set_group(grp, grp);

  v16f acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  const int kh = lane >> 5;
  int pix[TM];  // of the lane's output pixels, seen from the first tap
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = min((wm * TM + i) * 32 + (lane & 31), valid * g.Wo - 1), y = (int)fdiv((uint32_t)m, g.d_wo);
    pix[i] = y * g.PW + m - y * g.Wo;
  }
  int b_at[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int col = (wn * TN + j) * 32 + (lane & 31);
    b_at[j] = col * U + (kh ^ (col >> 2 & 1));
  }
  int r = 0, s = 0;
  auto multiply = [&](const v4u* st) {
    const int off = r * g.PW + s;
    int a_at[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int p = pix[i] + off;
      a_at[i] = p * U + (kh ^ (p >> 2 & 1));
    }
    // one set of fragments is read while the other is multiplied
    v8bf a[2][TM], b[2][TN];
    auto read = [&](int ks) {
#pragma unroll
      for (int i = 0; i < TM; ++i) a[ks & 1][i] = __builtin_bit_cast(v8bf, patch[a_at[i] + 2 * ks]);
#pragma unroll
      for (int j = 0; j < TN; ++j) b[ks & 1][j] = __builtin_bit_cast(v8bf, st[b_at[j] + 2 * ks]);
      __builtin_amdgcn_sched_barrier(0);
    };
    read(0);
#pragma unroll
    for (int ks = 0; ks < U / 2; ++ks) {
      if (ks + 1 < U / 2) read(ks + 1);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks & 1][i], b[ks & 1][j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    const bool row = ++s == g.k;
    r += row;
    s = row ? 0 : s;
  };
  // Tap t is multiplied while the next two are on their way.
  const int taps = g.k * g.k;
  auto step = [&](v4u* cur, v4u* far, int t) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070 | NB);  // all but the next tap's; lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    load(far, t + 2);  // past the last tap: the next column's or outside, and nobody reads it
    multiply(cur);
  };
  load(stage0, 0);
  load(stage1, 1);
  int t = 0;
  for (; t + 3 <= taps; t += 3) {
    step(stage0, stage2, t);
    step(stage1, stage0, t + 1);
    step(stage2, stage1, t + 2);
  }
  if (t < taps) step(stage0, stage2, t);
  if (t + 1 < taps) step(stage1, stage0, t + 1);
  __builtin_amdgcn_s_waitcnt(0x0070);  // no load is out when the workgroup ends
  const int m0 = (int)(n * (uint32_t)g.Ho + (uint32_t)y0) * g.Wo;
  store_rows(ep, acc, m0 + wm * (TM * 32), n0 + wn * (TN * 32), m0 + valid * g.Wo, g.N, lane);
}

// Output rows of a band and which tile; rows = 0: the layer does not fit
struct PatchPlan {
  int rows, bands;
  bool tall;  // 384 x 64, else 192 x 128
};
static int patch_rows(const ConvGeom& c, bool tall) {
  const int pixels = tall ? 384 : 192;
  const int U = c.cg() / 8, PW = c.W + 2 * c.pad;
  const int fit = patch_units(tall) / (PW * U) - (c.k - 1), rows = std::min(std::min(pixels / c.Wo, fit), c.Ho);
  if (rows < 1) return 0;
  return ceil_div(c.Ho, ceil_div(c.Ho, rows));  // bands of nearly the same height
}
static bool patch_full(const ConvGeom& c, int rows, int pixels) { return rows > 0 && rows * c.Wo * 4 >= pixels * 3; }
// 384 x 64 tiles, which read half the weights for a product, from two of them to a compute unit on (second layer, 192 x 128 | 384
// x 64: 24 pictures 21.8 | 22.2 us, 40 29.5 | 29.4, 64 33.9 | 32.6, 256 110 | 104; 48 channels of 50 x 50, 3 x 3, 32: 24.7 |
// 18.5), if they are mostly full (13 x 13, 512 maps: 19.5 | 26.4).  Not with 16 channels, where a tap is one product long (27 x
// 27, 256 maps: 22.9 | 24.3).
static PatchPlan patch_plan(const ConvGeom& c) {
  PatchPlan p{c.cg() == 48 ? patch_rows(c, true) : 0, 0, true};
  if (!patch_full(c, p.rows, 384) || (long)ceil_div(c.Ho, p.rows) * (c.og() / 64) * c.groups * c.B < 512) {
    p.rows = patch_rows(c, false);
    p.tall = false;
  }
  if (p.rows) p.bands = ceil_div(c.Ho, p.rows);
  return p;
}
// An odd number of pairs of octets is what the kernel can do, and whole columns of tiles; 16 and 48 channels have an instance.
// us, gathered (and stored in the order of the accumulators, as it was then) | here: 16 channels, 3 x 3 on 27 x 27, 64, 128, 256
// maps 33.7 | 12.6, 25.4 | 15.5, 63.2 | 22.9; 1 x 1 on 28 x 28, 256: 60.9 | 20.8; 5 x 5, two groups, 14 x 14, 128: 37.4 | 17.9;
// 48 channels, 3 x 3 on 13 x 13, 300: 38.3 | 17.0, on 28 x 28, 128: 46.9 | 25.1; gathered and stored by rows 13 x 13, 512: 22.4 |
// 19.7, 28 x 28, 256: 47.1 | 39.1.  Tiles mostly full, and a workgroup to every compute unit.
bool patch_fwd_ok(const ConvGeom& c) {
  if (!conv_bf16_stored_ok(c) || (c.cg() != 16 && c.cg() != 48) || c.og() % 128 != 0) return false;
  const PatchPlan p = patch_plan(c);
  return patch_full(c, p.rows, p.tall ? 384 : 192) && (long)p.bands * (c.og() / (p.tall ? 64 : 128)) * c.groups * c.B >= 256;
}
template <int U, int WM, int WN, int TM, int TN>
static int launch_patch(const PatchGeom& g, const EpiBiasAct& e, const ConvGeom& c, hipStream_t st) {
  KernelScope ks("gemm_bf16", 2.0 * c.P() * c.Cout * c.cg() * c.k * c.k,
                 4.0 * ((double)c.in_elems() + (double)c.w_elems() + (double)c.out_elems()), st);
  hipLaunchKernelGGL((patch_conv_kernel<U, WM, WN, TM, TN, EpiBiasAct>),
                     dim3((unsigned)((long)c.B * g.bands * c.groups * (c.og() / (WN * TN * 32)))), dim3(256), 0, st, g, e);
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}
int launch_patch_fwd(const ConvGeom& c, const uint16_t* x16, const uint16_t* wf16, const float* bias, int relu, float* y,
                     uint16_t* y16, hipStream_t st) {
  const PatchPlan p = patch_plan(c);
  PatchGeom g;
  g.x = x16; g.w = wf16;
  g.x_bytes = (uint32_t)(c.in_elems() * 2);
  g.w_bytes = (uint32_t)(c.w_elems() * 2);
  g.H = c.H; g.W = c.W; g.Ctot = c.Cin; g.Ho = c.Ho; g.Wo = c.Wo; g.pad = c.pad; g.k = c.k; g.N = c.og(); g.rows = p.rows;
  g.PW = c.W + 2 * c.pad;
  g.bands = p.bands; g.groups = c.groups;
  g.wgroup = (uint32_t)((long)c.og() * c.kf() * 2);
  g.d_pw = make_fastdiv((uint32_t)g.PW);
  g.d_wo = make_fastdiv((uint32_t)c.Wo);
  g.d_cols = make_fastdiv((uint32_t)(c.og() / (p.tall ? 64 : 128)));
  g.d_groups = make_fastdiv((uint32_t)c.groups);
  g.d_bands = make_fastdiv((uint32_t)p.bands);
  const EpiBiasAct e{y, c.Cout, bias, relu, c.og(), 0, 0, y16};
  if (c.cg() == 48) return p.tall ? launch_patch<6, 4, 1, 3, 2>(g, e, c, st) : launch_patch<6, 2, 2, 3, 2>(g, e, c, st);
  return launch_patch<2, 2, 2, 3, 2>(g, e, c, st);
}

}  // namespace ax
