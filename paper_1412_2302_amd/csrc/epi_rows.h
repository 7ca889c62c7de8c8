// The last step of the bf16 kernels: a wave writes its accumulator blocks where the epilogue says.
//
// Blocks are not transposed: register r of a lane is C[acc_row(lane, r)][lane % 32], so that a 4-byte store fills whole 128-byte
// lines.  Offsets are 32 bits from the tensor's start, one addition an element, and the buffer's range check takes rows past the
// last; columns past the last start from kOob.  What the epilogue reads is asked for before the first store: bias and gate may be
// the same memory as the output for all the compiler knows, and read element by element, each load waited for the one before it
// (192 x 128 tiles: 96 trips to the cache or, for a gate, to memory behind one another, 7 to 30 us of a launch).
#pragma once

#include <type_traits>

#include "gemm.h"

#ifndef AX_HOST_EMU
namespace ax {

__device__ __forceinline__ void buf_st1(const BufView& v, uint32_t off, float x) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), v, (int)off, 0, 0);
}
__device__ __forceinline__ void buf_st_bf16(const BufView& v, uint32_t off, float x) {
  __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, (__bf16)x), v, (int)off, 0, 0);
}
// Row of register r within a block, without the lane's part (4 * (lane / 32))
__device__ constexpr int block_row(int r) { return 8 * (r >> 2) + (r & 3); }

// Byte offsets of a lane's column of every block in row m + 4 * (lane / 32) of a tensor with ld bytes a row
template <int TN>
__device__ __forceinline__ void column_offsets(uint32_t (&at)[TN], uint32_t ld, int col_off, int m, int n, int N, int lane) {
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int c = n + j * 32 + (lane & 31);
    at[j] = c < N ? (uint32_t)(m + 4 * (lane >> 5)) * ld + (uint32_t)(col_off + c) * 4u : kOob;
  }
}

// m, n: first row and column of the wave's blocks; M, N: extents of the product.  In general, element by element:
template <class Epi, int TM, int TN>
__device__ __forceinline__ void store_rows(const Epi& e, const v16f (&acc)[TM][TN], int m, int n, int M, int N, int lane) {
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int c = n + j * 32 + (lane & 31);
      if (c >= N) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = m + i * 32 + 4 * (lane >> 5) + block_row(r);
        if (row < M) e.apply(row, c, acc[i][j][r]);
      }
    }
}

template <int TM, int TN>
__device__ __forceinline__ void store_rows(const EpiBiasAct& e, const v16f (&acc)[TM][TN], int m, int n, int M, int N, int lane) {
  const uint32_t ld = (uint32_t)e.ldc * 4u;
  const BufView y = make_view(e.y, (uint32_t)M * ld);
  uint32_t at[TN];
  column_offsets<TN>(at, ld, e.col_off, m, n, N, lane);
  float b[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) b[j] = e.bias && at[j] != kOob ? e.bias[e.col_off + n + j * 32 + (lane & 31)] : -0.f;  // v + -0 is v
  const bool any = !e.relu;
  auto put = [&](auto copy) {
    const BufView y16 = make_view(reinterpret_cast<const float*>(e.y16), (uint32_t)M * (ld / 2));
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          float v = acc[i][j][r] + b[j];
          v = any || v > 0.f ? v : 0.f;
          const uint32_t o = at[j] + (uint32_t)(i * 32 + block_row(r)) * ld;
          buf_st1(y, o, v);
          if constexpr (decltype(copy)::value) buf_st_bf16(y16, at[j] == kOob ? kOob : o / 2, v);
        }
  };
  if (e.y16)
    put(std::true_type{});
  else
    put(std::false_type{});
}

template <int TM, int TN>
__device__ __forceinline__ void store_rows(const EpiGate& e, const v16f (&acc)[TM][TN], int m, int n, int M, int N, int lane) {
  const uint32_t ld = (uint32_t)e.ldc * 4u;
  const BufView dx = make_view(e.dx, (uint32_t)M * ld);
  uint32_t at[TN];
  column_offsets<TN>(at, ld, e.col_off, m, n, N, lane);
  auto put = [&](auto gated, auto copy) {
    const BufView gate = make_view(e.gate, (uint32_t)M * ld);
    const BufView dx16 = make_view(reinterpret_cast<const float*>(e.dx16), (uint32_t)M * (ld / 2));
    float q[2][16];  // of the block at hand and of the next
    auto ask = [&](int b) {
#pragma unroll
      for (int r = 0; r < 16; ++r) q[b & 1][r] = buf_ld1(gate, at[b % TN] + (uint32_t)(b / TN * 32 + block_row(r)) * ld);
    };
    if constexpr (decltype(gated)::value) ask(0);
#pragma unroll
    for (int b = 0; b < TM * TN; ++b) {
      const int i = b / TN, j = b % TN;
      if constexpr (decltype(gated)::value)
        if (b + 1 < TM * TN) ask(b + 1);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float v = acc[i][j][r];
        if constexpr (decltype(gated)::value) v = q[b & 1][r] > 0.f ? v : 0.f;
        const uint32_t o = at[j] + (uint32_t)(i * 32 + block_row(r)) * ld;
        buf_st1(dx, o, v);
        if constexpr (decltype(copy)::value) buf_st_bf16(dx16, at[j] == kOob ? kOob : o / 2, v);
      }
    }
  };
  if (e.gate && e.dx16)
    put(std::true_type{}, std::true_type{});
  else if (e.gate)
    put(std::true_type{}, std::false_type{});
  else if (e.dx16)
    put(std::false_type{}, std::true_type{});
  else
    put(std::false_type{}, std::false_type{});
}

template <int TM, int TN>
__device__ __forceinline__ void store_rows(const EpiSlab& e, const v16f (&acc)[TM][TN], int m, int n, int M, int N, int lane) {
  const uint32_t ld = (uint32_t)e.ldc * 4u;
  const BufView out = make_view(e.base, (uint32_t)M * ld);
  uint32_t at[TN];
  column_offsets<TN>(at, ld, 0, m, n, N, lane);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int j = 0; j < TN; ++j) buf_st1(out, at[j] + (uint32_t)(i * 32 + block_row(r)) * ld, acc[i][j][r]);
}

template <int TM, int TN>
__device__ __forceinline__ void store_rows(const EpiSgd& e, const v16f (&acc)[TM][TN], int m, int n, int M, int N, int lane) {
  const uint32_t ld = (uint32_t)e.ldc * 4u;
  const BufView g = make_view(e.g, (uint32_t)M * ld), w = make_view(e.w, (uint32_t)M * ld), v = make_view(e.v, (uint32_t)M * ld);
  uint32_t at[TN];
  column_offsets<TN>(at, ld, 0, m, n, N, lane);
  float wb[2][16], vb[2][16];  // of the block at hand and of the next
  auto ask = [&](int b) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const uint32_t o = at[b % TN] + (uint32_t)(b / TN * 32 + block_row(r)) * ld;
      wb[b & 1][r] = buf_ld1(w, o);
      vb[b & 1][r] = buf_ld1(v, o);
    }
  };
  ask(0);
#pragma unroll
  for (int b = 0; b < TM * TN; ++b) {
    if (b + 1 < TM * TN) ask(b + 1);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const uint32_t o = at[b % TN] + (uint32_t)(b / TN * 32 + block_row(r)) * ld;
      const float x = acc[b / TN][b % TN][r];
      buf_st1(g, o, x);
      sgd_one(wb[b & 1][r], vb[b & 1][r], x, e.wd, e.lr, e.mu);
      buf_st1(v, o, vb[b & 1][r]);
      buf_st1(w, o, wb[b & 1][r]);
    }
  }
}

}  // namespace ax
#endif  // AX_HOST_EMU
