// What two kernels at the end of a backward pass share: the second half of the column sums that make the bias gradients.
#pragma once

#include "kernels.h"

namespace ax {

__device__ __forceinline__ void colsum_stage2_block(const float* __restrict__ part, int nparts, int cols,
                                                    float* __restrict__ out, int stripe, const SgdArgs& u) {
  __shared__ float sh[4][64];
  const int cl = threadIdx.x & 63, pl = threadIdx.x >> 6;
  const int col = stripe * 64 + cl;
  float s = 0.f;
  if (col < cols) {
#pragma unroll 8
    for (int p = pl; p < nparts; p += 4) s += part[(size_t)p * cols + col];  // eight loads in flight, added in order
  }
  sh[pl][cl] = s;
  __syncthreads();
  if (pl == 0 && col < cols) {
    const float g = (sh[0][cl] + sh[1][cl]) + (sh[2][cl] + sh[3][cl]);
    out[col] = g;
    if (u.w) {  // biases are not decayed
      const size_t i = (size_t)(out + col - u.g);
      sgd_one(u.w[i], u.v[i], g, 0.f, u.lr, u.mu);
    }
  }
}
// Several column sums in two launches (the bias gradients of a backward pass, whose inputs all still exist at
// its end).  The jobs' grids are laid end to end: a workgroup finds its job from the running totals (first1,
// first2) and its place in that job's own grid.  Same arithmetic and order per job as colsum_stage1 +
// colsum_stage2.
__device__ __forceinline__ int colsum_job_of(const int* first, int n, int block) {
  int j = 0;
#pragma unroll
  for (int k = 1; k < kMaxColsumJobs; ++k)
    if (k < n && block >= first[k]) j = k;
  return j;
}
__device__ __forceinline__ void colsum_batch_block2(const ColsumBatch& b, int block, const SgdArgs& u) {
  const int ji = colsum_job_of(b.first2, b.n, block);
  const ColsumJob& j = b.job[ji];
  colsum_stage2_block(j.part, j.nparts, j.cols, j.out, block - b.first2[ji], u);
}

}  // namespace ax
