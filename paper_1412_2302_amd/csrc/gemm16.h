// bf16 products of operands that are stored as bf16 and contiguous along k (the forward and data-gradient products of a
// bf16 handle's convolutions).  Same arithmetic and addressing as gemm_bf16.h; what differs is how the operands pass
// through the workgroup:
//
//  * LDS holds 16-byte units of eight consecutive k of one row, unit (k octet, row): a load is stored as it is, and a
//    fragment is one read, both without bank conflicts (an octet's rows are padded by four units, so that the four
//    octets that a load instruction's lanes hold lie a quarter of the banks apart).
//  * One register set between memory and LDS: a k-tile's loads are stored to LDS first thing in the iteration before
//    it is needed, and the next ones are issued at once into the same registers, addresses ready, with the whole
//    k-tile to arrive.  That leaves room for a third workgroup per CU beside 96 accumulators.
//  * The place of a workgroup in the grid is worked out on the scalar unit, as in gemm_split.h.
//
// Measured against gemm_bf16.h on the convolutions of a batch of 256 (bit for bit the same results): tiles of 256 x 128
// and 128 x 128 within 2 %, 128 x 64 3 % slower, so those stay there.  What it is for is 128 x 192 (wave tile 64 x 96: five
// fragment reads for six MFMAs) at three workgroups per CU, for products with 192 columns, which neither 128- nor
// 256-row tiles of 128 columns cover without padding: conv4 forward 107 -> 83 us (690 TFLOP/s).
#pragma once

#include "gemm_split.h"

namespace ax {

// L: one of the k-contiguous "16" loaders of gemm_bf16.h
template <class L, int ROWS, int BK>
struct Unit16 : L {
  using L::L;
  static constexpr int OCT = BK / 8, RP = ROWS + 4, UNITS = OCT * RP;
  AX_HD void store_step(int s, uint32_t* lds, const float4* r) const {
    const int idx = this->tid + s * kThreads;
    if (ROWS * OCT % kThreads == 0 || idx < ROWS * OCT)
      *reinterpret_cast<float4*>(lds + (this->kq * RP + idx / OCT) * 4) = r[s];
  }
};

#ifndef AX_HOST_EMU
template <class L, int TT>
struct Frags16 {
  v8bf f[TT];
  __device__ __forceinline__ void read(const uint32_t* lane_base) {  // lane_base: the lane's unit in block 0
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int t = 0; t < TT; ++t) f[t] = __builtin_bit_cast(v8bf, *reinterpret_cast<const v4u*>(lane_base + 32 * t * 4));
  }
};

// Side work of a k-tile, step IDX of: store tile t+1, fetch tile t+2 (one step), addresses of tile t+3
template <class AL, class BL>
constexpr int kSide16 = AL::NL + BL::NL + 1 + AL::NA + BL::NA;
template <class AL, class BL, int IDX>
__device__ __forceinline__ void side16_step(AL& al, BL& bl, uint32_t* as_next, uint32_t* bs_next, float4* ra, float4* rb,
                                            int k_plan, int kend) {
  constexpr int S0 = AL::NL, S1 = S0 + BL::NL, S2 = S1 + 1, S3 = S2 + AL::NA, S4 = S3 + BL::NA;
  if constexpr (IDX < S0) {
    al.store_step(IDX, as_next, ra);
  } else if constexpr (IDX < S1) {
    bl.store_step(IDX - S0, bs_next, rb);
  } else if constexpr (IDX < S2) {
    al.fetch(ra);
    bl.fetch(rb);
  } else if constexpr (IDX < S3) {
    al.template addr_step<IDX - S2>(k_plan, kend);
  } else if constexpr (IDX < S4) {
    bl.template addr_step<IDX - S3>(k_plan, kend);
  }
}
// the first slot stores and fetches, the others share the address steps
template <class AL, class BL, int SLOT, int SLOTS, int W = 0>
__device__ __forceinline__ void side16_slot(AL& al, BL& bl, uint32_t* as_next, uint32_t* bs_next, float4* ra, float4* rb,
                                            int k_plan, int kend) {
  constexpr int HEAD = AL::NL + BL::NL + 1, REST = AL::NA + BL::NA, PER = (REST + SLOTS - 2) / (SLOTS - 1);
  if constexpr (SLOT == 0 ? W < HEAD : W < PER) {
    constexpr int IDX = SLOT == 0 ? W : HEAD + (SLOT - 1) * PER + W;
    if constexpr (IDX < kSide16<AL, BL>) side16_step<AL, BL, IDX>(al, bl, as_next, bs_next, ra, rb, k_plan, kend);
    side16_slot<AL, BL, SLOT, SLOTS, W + 1>(al, bl, as_next, bs_next, ra, rb, k_plan, kend);
  }
}
// the MFMAs of a k-tile, one row block of one 16-deep step at a time
template <class T, class AL, class BL, int G = 0>
__device__ __forceinline__ void tile16(const uint32_t* as, const uint32_t* bs, Frags16<AL, T::TM>& fa,
                                       Frags16<BL, T::TN>& fb, v16f (&acc)[T::TM][T::TN], AL& al, BL& bl,
                                       uint32_t* as_next, uint32_t* bs_next, float4* ra, float4* rb, int k_plan, int kend) {
  constexpr int KS = T::BK / 16, SLOTS = KS * T::TM;
  if constexpr (G < SLOTS) {
    constexpr int ks = G / T::TM, i = G % T::TM;
    if constexpr (i == 0) {
      fa.read(as + ks * 2 * AL::RP * 4);
      fb.read(bs + ks * 2 * BL::RP * 4);
    }
#pragma unroll
    for (int j = 0; j < T::TN; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.f[i], fb.f[j], acc[i][j], 0, 0, 0);
    side16_slot<AL, BL, G, SLOTS>(al, bl, as_next, bs_next, ra, rb, k_plan, kend);
    tile16<T, AL, BL, G + 1>(as, bs, fa, fb, acc, al, bl, as_next, bs_next, ra, rb, k_plan, kend);
  }
}

template <class T, class AL, class BL, class Epi>
__global__ void __launch_bounds__(kThreads, 3)
gemm16_kernel(typename AL::Params ap, typename BL::Params bp, Epi ep, int M, int N, int K, FastDiv gx, FastDiv gy) {
  __shared__ __attribute__((aligned(16))) uint32_t As[2][AL::UNITS * 4];
  __shared__ __attribute__((aligned(16))) uint32_t Bs[2][BL::UNITS * 4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % T::WAVES_M, wn = wave / T::WAVES_M;
  const uint32_t total = gridDim.x, L = blockIdx.x, q8 = total >> 3, r8 = total & 7, xcd = L & 7;
  const uint32_t tile = xcd * q8 + min(xcd, r8) + (L >> 3);  // as in xcd_tile
  const uint32_t rest = fdiv(tile, gy), g = fdiv(rest, gx);
  const int m0 = (int)(rest - g * gx.d) * T::BM, n0 = (int)(tile - rest * gy.d) * T::BN;
  const int nt = (K + T::BK - 1) / T::BK;

  AL al(ap, (int)g, tid, m0);
  BL bl(bp, (int)g, tid, n0);
  ep.set_group((int)g, (int)g);

  v16f acc[T::TM][T::TN];
#pragma unroll
  for (int i = 0; i < T::TM; ++i)
#pragma unroll
    for (int j = 0; j < T::TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  if (nt > 0) {
    const int kh = lane >> 5;
    const int a_off = (kh * AL::RP + wm * (T::TM * 32) + (lane & 31)) * 4;
    const int b_off = (kh * BL::RP + wn * (T::TN * 32) + (lane & 31)) * 4;
    float4 ra[AL::NL], rb[BL::NL];
    plan_all(al, 0, K);
    plan_all(bl, 0, K);
    al.fetch(ra);
    bl.fetch(rb);
    plan_all(al, T::BK, K);
    plan_all(bl, T::BK, K);
#pragma unroll
    for (int s = 0; s < AL::NL; ++s) al.store_step(s, As[0], ra);
#pragma unroll
    for (int s = 0; s < BL::NL; ++s) bl.store_step(s, Bs[0], rb);
    al.fetch(ra);
    bl.fetch(rb);
    plan_all(al, 2 * T::BK, K);
    plan_all(bl, 2 * T::BK, K);
    __syncthreads();
    for (int t = 0; t < nt; ++t) {
      const int p = t & 1;
      Frags16<AL, T::TM> fa;
      Frags16<BL, T::TN> fb;
      tile16<T, AL, BL>(As[p] + a_off, Bs[p] + b_off, fa, fb, acc, al, bl, As[p ^ 1], Bs[p ^ 1], ra, rb,
                        (t + 3) * T::BK, K);
      __syncthreads();
    }
  }

  store_rows(ep, acc, m0 + wm * (T::TM * 32), n0 + wn * (T::TN * 32), M, N, lane);
}
#endif  // AX_HOST_EMU

}  // namespace ax
