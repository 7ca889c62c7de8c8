// Weight gradient of the first layer over pictures stored as bf16 with four channels per pixel (conv_plan.h, run16).
//
// As a gather GEMM the gradient's 363 rows were padded to 512 and its 96 columns to 128, and every 128 rows read the output
// gradient again, 297 MB in fp32 for 256 pictures.  Here a workgroup of eight waves, one per compute unit, holds the whole
// gradient in accumulators (k * ceil(k/4) groups of 16 rows: four taps of four channels) and walks over output rows: each
// row of the output gradient is read once, rounded and put to LDS as it is, [pixel][channel], and of the picture rows under it
// only the stride rows that the row before did not have.  Both fragments come from LDS by ds_read_b64_tr_b16 (see
// weight_direct.hip): four pixels x four taps of the picture are 128 contiguous bytes, so the gather costs nothing.
//
// What bounds it: the output gradient and the pictures from memory (402 MB for 256 pictures, 3.4 TB/s), with one output row of
// them on its way under a row's products, and the fragments from LDS (five or six for six to nine products of a wave).  256
// pictures of 3 x 227 x 227, 96 kernels of 11 x 11: 212 us as a gather GEMM, 117 here; 64 pictures 92 and 41.  The sums of the
// 256 slices, in the launch that adds up all layers', cost 7 to 15 us more than the few of before.
#include <algorithm>

#include "gemm_direct.h"
#include "kernels.h"

namespace ax {

constexpr int kFwThreads = 512, kFwRing = 16, kFwRow = 2048;  // ring of picture rows, bytes of one
constexpr int kFwPixels = 64, kFwCols = 96, kFwBlocks = 3;    // output pixels of a row, columns, 32-row blocks of a wave

struct FirstWeight {
  const uint16_t* x4;
  const float* dy;
  float* slabs;
  uint32_t x_bytes, dy_bytes;
  int H, Ho, Wo, Cin, Cout, k, stride, per_row;  // per_row: groups of 16 rows of a kernel row
  int items;                                      // output rows in all
  uint32_t row_bytes;                             // of the pictures
  FastDiv d_per_row, d_ho;
};

typedef short fw4s __attribute__((ext_vector_type(4)));
__device__ __forceinline__ fw4s fw_read(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) fw4s*)p);
}

__global__ void __launch_bounds__(kFwThreads) first_weight_kernel(FirstWeight g) {
  __shared__ __attribute__((aligned(16))) char ring[kFwRing * kFwRow + 64];  // 64: taps past the kernel, whose rows are dropped
  __shared__ __attribute__((aligned(16))) char grad[2][kFwPixels * kFwCols * 2 + kFwCols * 2];
  __shared__ __attribute__((aligned(16))) char zero[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wgs = gridDim.x, first = (int)((long)g.items * blockIdx.x / wgs), last = (int)((long)g.items * (blockIdx.x + 1) / wgs);
  const BufView xv = make_view(reinterpret_cast<const float*>(g.x4), g.x_bytes), dv = make_view(g.dy, g.dy_bytes);
  const int quads = g.Wo * g.Cout / 4;  // of an output row
  const int groups = g.k * g.per_row, blocks = (groups + 1) / 2;

  // pixels past the row's end: zero in both operands, whatever the picture holds
  for (int i = tid; i < 2 * (int)sizeof(grad[0]) / 4; i += kFwThreads) reinterpret_cast<uint32_t*>(grad)[i] = 0u;
  if (tid < 4) reinterpret_cast<uint32_t*>(zero)[tid] = 0u;
  __syncthreads();

  auto picture_load = [&](int n, int row) {  // 16 bytes of picture row `row`, this thread's unit of four rows
    const int iy = row + (tid >> 7);
    const bool in = iy < g.H && (uint32_t)(tid & 127) * 16 < g.row_bytes;
    return buf_ld4(xv, in ? ((uint32_t)(n * g.H + iy)) * g.row_bytes + (uint32_t)(tid & 127) * 16 : kOob);
  };
  auto picture_store = [&](int row, const float4& v) {
    *reinterpret_cast<float4*>(ring + ((row + (tid >> 7)) & (kFwRing - 1)) * kFwRow + (tid & 127) * 16) = v;
  };
  float4 d[3];
  auto grad_load = [&](int item) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int q = tid + i * kFwThreads;
      d[i] = buf_ld4(dv, q < quads ? ((uint32_t)item * (uint32_t)quads + (uint32_t)q) * 16u : kOob);
    }
  };
  auto grad_store = [&](char* to) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int q = tid + i * kFwThreads;
      if (q < quads) {
        uint2 w;
        w.x = pack_bf16(d[i].x, d[i].y);
        w.y = pack_bf16(d[i].z, d[i].w);
        *reinterpret_cast<uint2*>(to + q * 8) = w;
      }
    }
  };

  v16f acc[kFwBlocks][3];
#pragma unroll
  for (int i = 0; i < kFwBlocks; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  // of this lane in a fragment read: pixel 4*(lane/32) + l16/4, tap l16%4 of its group (picture) or columns 4*(l16%4) (gradient)
  const int l16 = lane & 15, pix = 4 * (lane >> 5) + (l16 >> 2), half = (lane >> 4) & 1;
  int kr[kFwBlocks], at[kFwBlocks];
#pragma unroll
  for (int i = 0; i < kFwBlocks; ++i) {
    const int gid = min(2 * (wave + 8 * i) + half, groups - 1), r = (int)fdiv((uint32_t)gid, g.d_per_row);
    kr[i] = r;
    at[i] = (pix * g.stride + 4 * (gid - r * g.per_row) + (l16 & 3)) * 8;
  }
  const int b_at = pix * g.Cout * 2 + (16 * half + 4 * (l16 & 3)) * 2;

  auto multiply = [&](const char* gr, int y) {
    int a_at[kFwBlocks];
#pragma unroll
    for (int i = 0; i < kFwBlocks; ++i) a_at[i] = ((y * g.stride + kr[i]) & (kFwRing - 1)) * kFwRow + at[i];
    for (int p0 = 0; p0 < g.Wo; p0 += 16) {
      struct Two {
        fw4s lo, hi;
      };
      const bool in0 = p0 + pix < g.Wo, in1 = p0 + 8 + pix < g.Wo;
      v8bf b[3];
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const char* s = gr + b_at + p0 * g.Cout * 2 + j * 64;
        b[j] = __builtin_bit_cast(v8bf, Two{fw_read(s), fw_read(s + 8 * g.Cout * 2)});
      }
#pragma unroll
      for (int i = 0; i < kFwBlocks; ++i) {
        if (wave + 8 * i >= blocks) continue;  // uniform
        const char* s = ring + a_at[i] + p0 * g.stride * 8;
        const v8bf a = __builtin_bit_cast(v8bf, Two{fw_read(in0 ? s : zero), fw_read(in1 ? s + 8 * g.stride * 8 : zero)});
#pragma unroll
        for (int j = 0; j < 3; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b[j], acc[i][j], 0, 0, 0);
      }
    }
  };

  int cur = 0;
  for (int item = first; item < last;) {
    const int n = (int)fdiv((uint32_t)item, g.d_ho), y0 = item - n * g.Ho, rows = min(last - item, g.Ho - y0);
    for (int r = 0; r < g.k; r += 4) picture_store(y0 * g.stride + r, picture_load(n, y0 * g.stride + r));
    grad_load(item);
    grad_store(grad[cur]);
    __syncthreads();
    for (int y = 0; y < rows; ++y) {
      // the rows that the next output row adds lie in slots that this one does not read (k + stride <= ring)
      const int next = (y0 + y) * g.stride + g.k;
      const bool more = y + 1 < rows;
      float4 p = make_float4(0.f, 0.f, 0.f, 0.f);
      if (more) {
        p = picture_load(n, next);
        grad_load(item + y + 1);
      }
      multiply(grad[cur], y0 + y);
      if (more) {
        if ((tid >> 7) < g.stride) picture_store(next, p);
        grad_store(grad[cur ^ 1]);
      }
      cur ^= 1;
      __syncthreads();
    }
    item += rows;
  }

  float* out = g.slabs + (size_t)blockIdx.x * g.k * g.k * g.Cin * g.Cout;
#pragma unroll
  for (int i = 0; i < kFwBlocks; ++i) {
    if (wave + 8 * i >= blocks) continue;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = acc_row(lane, r), gid = 2 * (wave + 8 * i) + (row >> 4);
      const int kr_ = (int)fdiv((uint32_t)gid, g.d_per_row), s = 4 * (gid - kr_ * g.per_row) + ((row & 15) >> 2), c = row & 3;
      if (gid >= groups || s >= g.k || c >= g.Cin) continue;
      float* o = out + (size_t)((kr_ * g.k + s) * g.Cin + c) * g.Cout;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const int col = 32 * j + (lane & 31);
        if (col < g.Cout) o[col] = acc[i][j][r];
      }
    }
  }
}

// Rows of at most 64 outputs and 256 pixels, 96 columns, 24 blocks of 32 rows, and a ring that holds what two output rows need
bool first_weight_ok(const ConvGeom& c) {
  const int per_row = (c.k + 3) / 4;
  return run16_mode(c) && c.Wo <= kFwPixels && c.W * 8 <= kFwRow && c.Cout <= kFwCols && c.Cout % 4 == 0 && c.stride <= 4 &&
         (c.k + 3) / 4 * 4 + c.stride <= kFwRing && (c.k * per_row + 1) / 2 <= 8 * kFwBlocks;
}
int first_weight_slices(const ConvGeom& c) { return std::min(256, c.B * c.Ho); }
int launch_first_weight(const ConvGeom& c, const uint16_t* x4, const float* dy, float* slabs, hipStream_t st) {
  FirstWeight g;
  g.x4 = x4;
  g.dy = dy;
  g.slabs = slabs;
  g.row_bytes = (uint32_t)c.W * 8u;
  g.x_bytes = (uint32_t)((size_t)c.B * c.H * c.W * 8);
  g.dy_bytes = (uint32_t)(c.out_elems() * 4);
  g.H = c.H; g.Ho = c.Ho; g.Wo = c.Wo; g.Cin = c.Cin; g.Cout = c.Cout; g.k = c.k; g.stride = c.stride;
  g.per_row = (c.k + 3) / 4;
  g.items = c.B * c.Ho;
  g.d_per_row = make_fastdiv((uint32_t)g.per_row);
  g.d_ho = make_fastdiv((uint32_t)c.Ho);
  KernelScope ks("gemm_bf16", 2.0 * c.P() * c.Cout * c.cg() * c.k * c.k,
                 4.0 * ((double)c.in_elems() + (double)c.w_elems() + (double)c.out_elems()), st);
  hipLaunchKernelGGL(first_weight_kernel, dim3((unsigned)first_weight_slices(c)), dim3(kFwThreads), 0, st, g);
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}

}  // namespace ax
