// Epilogue of the dense layers' forward products.
#pragma once

#include "gemm.h"
#include "kernels.h"

namespace ax {

// An unsliced dense product finishes itself: y = act(v + bias), as fc_fwd_finish_kernel does behind slices.
struct EpiFcAct {
  static constexpr bool kTransposed = true;
  float* y;
  long ldc;
  FcAct act;
  uint16_t* y16;  // may be null
  AX_HD void set_group(int /*g*/, int /*z*/) {}
  __device__ void apply(int m, int n, float v) const {
    const size_t i = (size_t)m * ldc + n;
    if (act.bias) v += act.bias[n];
    if (act.relu) v = v > 0.f ? v : 0.f;
    if (act.dropout && !dropout_keep(act.key, act.tag, i, act.thresh24)) v = 0.f;
    y[i] = v * act.scale;
    if (y16) store_bf16(y16 + i, v * act.scale);
  }
  __device__ void apply4(int m, int n, float4 v) const {
    apply(m, n, v.x); apply(m, n + 1, v.y); apply(m, n + 2, v.z); apply(m, n + 3, v.w);
  }
};

// as a small product's epilogue (gemm_wave.h)
__device__ __forceinline__ float wave_ask(const EpiFcAct& e, int, int n) { return e.act.bias ? e.act.bias[n] : -0.f; }
__device__ __forceinline__ void wave_put(const EpiFcAct& e, int m, int n, float v, float bias) {
  const size_t i = (size_t)m * e.ldc + n;
  v += bias;
  if (e.act.relu) v = v > 0.f ? v : 0.f;
  if (e.act.dropout && !dropout_keep(e.act.key, e.act.tag, i, e.act.thresh24)) v = 0.f;
  e.y[i] = v * e.act.scale;
  if (e.y16) store_bf16(e.y16 + i, v * e.act.scale);
}

}  // namespace ax
