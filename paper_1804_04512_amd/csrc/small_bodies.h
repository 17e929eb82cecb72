// Bodies of the small reduction kernels, shared by their stand-alone launches (gemm.hip) and by
// the training step's closing kernel (conv_wgrad.hip), which runs all of a step's deferred
// reductions in one launch.  One workgroup of 256 threads per call; `blk` is the workgroup's
// index inside its job.
#pragma once

#include "dll_internal.h"

namespace dllk {

constexpr int kSmallThreads = 256;
constexpr int kColsumCols = 16, kColsumSlices = kSmallThreads / kColsumCols;

// out[n] = scale * sum_m (A - A2)[m][n] (A2 may be NULL): 16 columns per workgroup, 16 row slices added in a fixed order
// (small inputs: many short independent load chains beat few long ones).
__device__ __forceinline__ void colsum_block(const float *A, int M, int N, float *out, float *update, float step, float *vel,
                                             float mu, int blk, const float *A2 = nullptr, float scale = 1.0f) {
  __shared__ float part[kColsumSlices][kColsumCols + 1];
  const int col = threadIdx.x % kColsumCols, slice = threadIdx.x / kColsumCols;
  const int n = blk * kColsumCols + col;
  float s = 0.0f;
  if (n < N) {
    if (A2) {
#pragma unroll 4
      for (int m = slice; m < M; m += kColsumSlices) s += A[(long)m * N + n] - A2[(long)m * N + n];
    } else {
#pragma unroll 4
      for (int m = slice; m < M; m += kColsumSlices) s += A[(long)m * N + n];
    }
  }
  part[slice][col] = s;
  __syncthreads();
  if (slice == 0 && n < N) {
    float q[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      q[g] = 0.0f;
#pragma unroll
      for (int i = 0; i < kColsumSlices / 4; ++i) q[g] += part[g * (kColsumSlices / 4) + i][col];
    }
    s = ((q[0] + q[1]) + (q[2] + q[3])) * scale;
    if (out) out[n] = s;
    if (update) update_param(update + n, vel ? vel + n : nullptr, s, step, mu, 0.0f);
  }
}

// Sum or maximum over the workgroup's 256 threads, the same value in every thread: lane exchanges
// inside a wavefront (a butterfly, so every lane adds the same pairs in the same order), then the
// four wavefronts' results in wavefront order.  Two barriers instead of the nine of a tree in LDS,
// which were most of what the small row kernels spent.  sh: at least 4 floats, free again on return.
__device__ __forceinline__ float block_reduce(float v, float *sh, bool is_max) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float w = __shfl_xor(v, o);
    v = is_max ? fmaxf(v, w) : v + w;
  }
  const int tid = threadIdx.x;
  if ((tid & 63) == 0) sh[tid >> 6] = v;
  __syncthreads();
  float r = sh[0];
#pragma unroll
  for (int w = 1; w < kSmallThreads / 64; ++w) r = is_max ? fmaxf(r, sh[w]) : r + sh[w];
  __syncthreads();
  return r;
}

// *out = (sum of v[0 .. n)) / count
__device__ __forceinline__ void mean_block(const float *v, int n, float *out, double count) {
  __shared__ double sh[kSmallThreads / 64];
  double s = 0.0;
  for (int j = threadIdx.x; j < n; j += kSmallThreads) s += (double)v[j];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) *out = (float)(((sh[0] + sh[1]) + (sh[2] + sh[3])) / count);
}

// The CRBM's visible sums, kStatBlocks workgroups per channel: scratch[ch][b] = sum over the block's slice of (v0 - v1);
// scratch[C*32 + ch*32 + b] = sum of squares.  blk: channel and slice; sh: kSmallThreads floats of LDS.  Small batches fill
// the first slices only; the others' sums are zero without a reduction.
constexpr int kStatBlocks = 32;
__device__ __forceinline__ void visible_block(const float *v0, const float *v1, int N, int C, int HW, float *scratch, int blk, float *sh) {
  const int b = blk % kStatBlocks, ch = blk / kStatBlocks;
  const long per = (long)N * HW;
  if ((long)b * kSmallThreads >= per) {   // uniform
    if (threadIdx.x == 0) scratch[ch * kStatBlocks + b] = scratch[(C + ch) * kStatBlocks + b] = 0.0f;
    return;
  }
  float s = 0.0f, q = 0.0f;
  for (long e = (long)b * kSmallThreads + threadIdx.x; e < per; e += (long)kStatBlocks * kSmallThreads) {
    const long nn = e / HW, r = e - nn * HW;
    const long o = (nn * C + ch) * HW + r;
    const float d = v0[o] - v1[o];
    s += d;
    q += d * d;
  }
  s = block_reduce(s, sh, false);
  q = block_reduce(q, sh, false);
  if (threadIdx.x == 0) {
    scratch[ch * kStatBlocks + b] = s;
    scratch[(C + ch) * kStatBlocks + b] = q;
  }
}

// Their last sums, in one wavefront: a lane per slice (32 sums, 32 sums of squares), added by lane exchanges in double.
__device__ __forceinline__ void visible_final(const float *scratch, int N, int C, int HW, float scale, float *dc, float *mse, float *c_update,
                                              float step) {
  const int lane = threadIdx.x, b = lane & (kStatBlocks - 1);
  static_assert(kStatBlocks == 32, "half a wavefront per kind of sum");
  double sq = 0.0;
  for (int ch = 0; ch < C; ++ch) {
    double s = (double)scratch[((lane < 32 ? 0 : C) + ch) * kStatBlocks + b];
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) {
      const float g = (float)(s * (double)scale);
      if (dc) dc[ch] = g;
      if (c_update) c_update[ch] += step * g;
    }
    sq += s;   // lanes 32 ..: the channel's squares
  }
  if (mse && lane == 32) *mse = (float)(sq / ((double)N * C * HW));
}

}  // namespace dllk
