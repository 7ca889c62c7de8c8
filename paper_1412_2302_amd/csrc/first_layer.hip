// Forward product of the first layer over pictures stored as bf16 with four channels per pixel (conv_plan.h, run16): the
// weights stay in LDS, and so does the piece of the picture under a few output rows.
//
// As a gather GEMM every kernel row reads its piece of the picture again, k times in all, through L1, registers and LDS, and
// all weights pass through LDS once per 256 pixels.  Here a workgroup of eight waves, one per compute unit, keeps all weights
// (k * run * Cout, 101 KB for 96 11 x 11 kernels) and walks over tiles of R whole output rows, at most 256 pixels: the
// (R - 1) * stride + k picture rows under them lie in LDS as they are in memory, a wave owns 32 pixels and all channels, and
// both fragments of a product are one 16-byte LDS read per lane.  The next tile's rows are on their way to registers
// meanwhile.
//
// LDS, in 16-byte units.  Weights: unit (octet of k, channel).  Picture: unit (row, octet of the row, two pixels), the octets
// of a row in stride/2 planes by octet modulo stride/2, because neighbouring output pixels are stride/2 octets apart: the
// lanes of a read then touch neighbouring units.
//
// What bounds it: memory -- the result, 4 bytes a value, and what runs on the side stream meanwhile -- and 4 KB of fragments
// per wave and three products, a third above what LDS gives in the products' time.  256 pictures of 3 x 227 x 227, 96 kernels
// of 11 x 11, beside the conversion of the dense weights: 284 us as a gather GEMM with 256 x 96 tiles, 170 here (4.4 TB/s with
// the 350 MB of the conversion), the same bits.  It is the faster one wherever it fits: inference of 8, 16, 37 and 100 pictures
// 266, 315, 411 and 694 us as a gather GEMM, 263, 302, 410 and 656 here, stores still in one
// piece (184 us above).
#include <algorithm>

#include "gemm_split.h"
#include "conv_plan.h"
#include "kernels.h"

namespace ax {

constexpr int kFirstWaves = 8, kFirstThreads = 64 * kFirstWaves, kFirstPixels = 32 * kFirstWaves;
constexpr int kFirstLoads = 8;                // picture units per thread
constexpr int kFirstUnits = 157 * 1024 / 16;  // LDS

struct FirstGeom {
  const uint16_t* x4;
  const uint16_t* wk;
  const float* bias;
  float* y;
  uint16_t* y16;  // may be null
  uint32_t x_bytes, y_bytes;
  int W, Ho, Wo, Cout, stride, relu;
  int rows, tiles;          // output rows per tile; tiles per picture
  int patch_rows, row_oct;  // picture rows per tile, octets per picture row
  int planes, plane_units;  // stride/2; units per plane of a row
  int run_oct, octets;      // octets per kernel row, in all (k * run_oct)
  int items;                // tiles in all
  uint32_t img_bytes, row_bytes;  // of the pictures
  FastDiv d_tiles, d_row_oct, d_wo, d_planes, d_run_oct;
};

// R, or 0 if the layer does not fit
static int first16_rows(const ConvGeom& c) {
  if (!run16_mode(c) || c.stride % 2 || c.Cout > 128 || c.Wo > kFirstPixels) return 0;
  const int nb = ceil_div(c.Cout, 32), octets = c.k * (run16_len(c) / 8), weights = (octets + 1) / 2 * 2 * nb * 32;
  if (octets > 128) return 0;  // unit_tab
  const int row_oct = (c.W + 1) / 2, planes = c.stride / 2, row_units = ceil_div(row_oct, planes) * planes;
  for (int r = std::min(kFirstPixels / c.Wo, c.Ho); r > 0; --r) {
    const int rows = (r - 1) * c.stride + c.k;
    // a lane's last octet may start run_oct octets behind its pixel: those units exist too
    if (rows * row_oct <= kFirstLoads * kFirstThreads && weights + rows * row_units + run16_len(c) / 8 <= kFirstUnits) return r;
  }
  return 0;
}

// a barrier that orders LDS only: global loads and stores stay in flight across it
__device__ __forceinline__ void first_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ODD: an odd number of octets, whose last step has one of its own only
template <int NB, bool Y16, bool ODD>
__global__ void __launch_bounds__(kFirstThreads, 2) first_layer_kernel(FirstGeom g) {
  typedef uint32_t v4u __attribute__((ext_vector_type(4)));
  __shared__ __attribute__((aligned(16))) v4u lds[kFirstUnits];
  constexpr int NP = NB * 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), kh = lane >> 5;
  const int steps = (g.octets + 1) / 2;
  v4u* const wl = lds;
  v4u* const pl = lds + steps * 2 * NP;
  const int row_units = g.plane_units * g.planes;
  const BufView xv = make_view(reinterpret_cast<const float*>(g.x4), g.x_bytes);
  const BufView yv = make_view(g.y, g.y_bytes);
  const BufView y16v = make_view(Y16 ? reinterpret_cast<const float*>(g.y16) : g.y, g.y_bytes / 2);
  const BufView wv = make_view(reinterpret_cast<const float*>(g.wk), (uint32_t)g.Cout * (uint32_t)g.octets * 16u);

  // weights, zero past the last channel and octet
  for (int u = tid; u < steps * 2 * NP; u += kFirstThreads) {
    const int q = u / NP, n = u - q * NP;
    const bool in = q < g.octets && n < g.Cout;
    wl[u] = __builtin_bit_cast(v4u, buf_ld4(wv, in ? ((uint32_t)n * (uint32_t)g.octets + (uint32_t)q) * 16u : kOob));
  }
  // whatever lies between and behind the picture's units meets zero weights: it has to be finite
  for (int u = tid; u < g.patch_rows * row_units + g.run_oct; u += kFirstThreads) pl[u] = v4u{0, 0, 0, 0};
  // picture units of this thread: where they go, and their offset from a tile's first row
  uint32_t src[kFirstLoads];
  int dst[kFirstLoads];
  const int total = g.patch_rows * g.row_oct;
#pragma unroll
  for (int i = 0; i < kFirstLoads; ++i) {
    const int u = tid + i * kFirstThreads;
    const int row = (int)fdiv((uint32_t)u, g.d_row_oct), e = u - row * g.row_oct;
    const int pos = (int)fdiv((uint32_t)e, g.d_planes), plane = e - pos * g.planes;
    const bool in = u < total;
    src[i] = in ? (uint32_t)row * g.row_bytes + (uint32_t)e * 16u : kOob;
    dst[i] = in ? row * row_units + plane * g.plane_units + pos : -1;
  }
  // this workgroup's tiles, one after the other
  const uint32_t G = gridDim.x, q8 = G >> 3, r8 = G & 7, xcd = blockIdx.x & 7;
  const uint32_t place = xcd * q8 + min(xcd, r8) + (blockIdx.x >> 3);  // neighbours in memory on one XCD, as in xcd_tile
  int item = (int)((uint64_t)place * g.items / G);
  const int last = (int)((uint64_t)(place + 1) * g.items / G);
  float4 r[kFirstLoads];
  auto fetch = [&](int item) {
    const int n = (int)fdiv((uint32_t)item, g.d_tiles), y0 = (item - n * g.tiles) * g.rows;
    const bool any = item < last;
    const uint32_t base = (uint32_t)n * g.img_bytes + (uint32_t)(y0 * g.stride) * g.row_bytes;
#pragma unroll
    for (int i = 0; i < kFirstLoads; ++i) r[i] = buf_ld4(xv, any && src[i] != kOob ? base + src[i] : kOob);
  };
  auto store = [&]() {
#pragma unroll
    for (int i = 0; i < kFirstLoads; ++i)
      if (dst[i] >= 0) pl[dst[i]] = __builtin_bit_cast(v4u, r[i]);
  };
  // the lane's pixel in a tile and the unit of its first octet
  const int p = wave * 32 + (lane & 31), ly = min((int)fdiv((uint32_t)p, g.d_wo), g.rows - 1);
  const int lx = min(p - ly * g.Wo, g.Wo - 1);
  const v4u* const a0 = pl + ly * g.stride * row_units + lx;
  const v4u* const b0 = wl + kh * NP + (lane & 31);
  // unit of octet q of k relative to that, kept by lane q % 64
  int unit_tab[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int q = lane + 64 * h < g.octets ? lane + 64 * h : 0;
    const int rr = (int)fdiv((uint32_t)q, g.d_run_oct), o = q - rr * g.run_oct, pos = (int)fdiv((uint32_t)o, g.d_planes);
    unit_tab[h] = rr * row_units + (o - pos * g.planes) * g.plane_units + pos;
  }
  // ODD: the octet behind the last one meets zero weights, and a picture's infinity must not: it is a unit behind the picture,
  // which stays zero.
  const int zero = g.patch_rows * row_units - (int)(a0 - pl);
  auto unit_at = [&](int s) {  // of octet 2s + kh
    const int t = s < 32 ? unit_tab[0] : unit_tab[1], l = 2 * s & 63;
    const int u0 = __builtin_amdgcn_readlane(t, l), u1 = __builtin_amdgcn_readlane(t, l + 1);
    return kh ? (!ODD || s + 1 < steps ? u1 : zero) : u0;
  };
  float bias[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) bias[j] = g.bias && j * 32 + (lane & 31) < g.Cout ? g.bias[j * 32 + (lane & 31)] : 0.f;

  // The next tile's loads are issued in front of a tile's products and wait behind them; a tile's results are stored a quarter at
  // a time between the products of the tile after it.  The wait for the loads takes the stores too, although they are the younger
  // ones: the first tile has none, and the compiler counts for the way without them.  By then they have had up to a tile's
  // products to leave.  (Stored all at once behind the products, all compute units wrote at
  // one time and multiplied at another: 13 us a tile of 220 pixels, 5 of products, 3 of arithmetic for the stores and 4 for 84
  // KB to leave at a compute unit's share of the memory; 256 pictures 184 us.)
  float out[NB][16];
  uint32_t out_first = 0;
  int out_valid = 0;  // pixels of the tile that waits to be stored
  auto put = [&](int q) {
    const int pix = wave * 32 + acc_row(lane, q);
    const uint32_t o = ((out_first + (uint32_t)pix) * (uint32_t)g.Cout + (uint32_t)(lane & 31)) * 4u;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const bool in = pix < out_valid && j * 32 + (lane & 31) < g.Cout;
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(out[j][q]), yv, in ? (int)(o + 128u * j) : (int)kOob, 0, 0);
      if (Y16) buf_st_bf16(y16v, in ? (o + 128u * j) / 2 : kOob, out[j][q]);
    }
  };
  fetch(item);
  first_barrier();
  store();
  first_barrier();
  for (; item < last; ++item) {
    fetch(item + 1);
    v16f acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[j][q] = 0.f;
    // one set of fragments is read while the other is multiplied
    v8bf a[2], b[2][NB];
    auto read = [&](int set, int s) {
      a[set] = __builtin_bit_cast(v8bf, a0[unit_at(s)]);
      const v4u* const bs = b0 + s * 2 * NP;
#pragma unroll
      for (int j = 0; j < NB; ++j) b[set][j] = __builtin_bit_cast(v8bf, bs[j * 32]);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int set) {
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[set], b[set][j], acc[j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    read(0, 0);
    int s = 0;
#pragma unroll
    for (int part = 0; part < 4; ++part) {
      if (out_valid > 0) {  // uniform
#pragma unroll
        for (int q = 4 * part; q < 4 * part + 4; ++q) put(q);
      }
      const int end = part == 3 ? steps : (steps * (part + 1) / 4) & ~1;
      for (; s < end; s += 2) {
        read(1, min(s + 1, steps - 1));
        multiply(0);
        if (s + 1 == steps) break;
        read(0, min(s + 2, steps - 1));
        multiply(1);
      }
    }

    first_barrier();  // the waves are done with the picture
    store();
    const int n = (int)fdiv((uint32_t)item, g.d_tiles), y0 = (item - n * g.tiles) * g.rows;
    out_valid = min(g.rows, g.Ho - y0) * g.Wo;
    out_first = (uint32_t)((n * g.Ho + y0) * g.Wo);
#pragma unroll
    for (int q = 0; q < 16; ++q)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const float v = acc[j][q] + bias[j];
        out[j][q] = v > 0.f || !g.relu ? v : 0.f;
      }
    first_barrier();
  }
  if (out_valid > 0) {
#pragma unroll
    for (int q = 0; q < 16; ++q) put(q);
  }
}

bool first16_ok(const ConvGeom& c) { return first16_rows(c) > 0; }

int launch_first16(const ConvGeom& c, const uint16_t* x4, const uint16_t* wk, const float* bias, int relu, float* y,
                   uint16_t* y16, hipStream_t st) {
  FirstGeom g;
  g.x4 = x4; g.wk = wk; g.bias = bias; g.y = y; g.y16 = y16;
  g.x_bytes = (uint32_t)(run16_x_elems(c) * 2);
  g.y_bytes = (uint32_t)(c.out_elems() * 4);
  g.W = c.W; g.Ho = c.Ho; g.Wo = c.Wo; g.Cout = c.Cout; g.stride = c.stride; g.relu = relu;
  g.rows = first16_rows(c);
  if (!g.rows) {
    set_error("first layer: geometry does not fit");
    return ALEXNET_EINVAL;
  }
  g.tiles = ceil_div(c.Ho, g.rows);
  g.patch_rows = (g.rows - 1) * c.stride + c.k;
  g.row_oct = (c.W + 1) / 2;
  g.planes = c.stride / 2;
  g.plane_units = ceil_div(g.row_oct, g.planes);
  g.run_oct = run16_len(c) / 8;
  g.octets = c.k * g.run_oct;
  g.items = c.B * g.tiles;
  g.img_bytes = (uint32_t)c.H * c.W * 8u;
  g.row_bytes = (uint32_t)c.W * 8u;
  g.d_tiles = make_fastdiv((uint32_t)g.tiles);
  g.d_row_oct = make_fastdiv((uint32_t)g.row_oct);
  g.d_wo = make_fastdiv((uint32_t)c.Wo);
  g.d_planes = make_fastdiv((uint32_t)g.planes);
  g.d_run_oct = make_fastdiv((uint32_t)g.run_oct);
  KernelScope ks("gemm_bf16", 2.0 * c.P() * c.Cout * c.cg() * c.k * c.k,
                 4.0 * ((double)c.in_elems() + (double)c.w_elems() + (double)c.out_elems()), st);
  const dim3 grid(std::min(g.items, 256)), block(kFirstThreads);
  const int nb = ceil_div(c.Cout, 32);
  const bool odd = g.octets % 2 != 0;
#define AX_FIRST_AS(NB, ODD)                                                                            \
  if (y16) hipLaunchKernelGGL((first_layer_kernel<NB, true, ODD>), grid, block, 0, st, g);              \
  else hipLaunchKernelGGL((first_layer_kernel<NB, false, ODD>), grid, block, 0, st, g)
#define AX_FIRST(NB)                       \
  if (odd) { AX_FIRST_AS(NB, true); }      \
  else { AX_FIRST_AS(NB, false); }
  if (nb == 1) { AX_FIRST(1); }
  else if (nb == 2) { AX_FIRST(2); }
  else if (nb == 3) { AX_FIRST(3); }
  else { AX_FIRST(4); }
#undef AX_FIRST
#undef AX_FIRST_AS
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}

}  // namespace ax
