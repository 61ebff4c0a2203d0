// The LSTM cell, shared by the gate kernels' epilogues, and the heads' maximum.
// Every operation of the cell is spelled out (no contraction left to the
// compiler), so that the kernels' tile shapes all give the same bits.
#pragma once
#include <hip/hip_runtime.h>

namespace zo {

// 1 / d for d >= 1 (up to infinity) to within one rounding: the hardware's
// reciprocal and one Newton step (IEEE division takes 10 instructions, and a
// cell has five). d is held below 2^126 first, where the step's 1 - d r would
// be 0 times infinity; minimum keeps a NaN.
__device__ __forceinline__ float rcp_ge1(float d) {
  d = __builtin_elementwise_minimum(d, 0x1p126f);
  const float r = __builtin_amdgcn_rcpf(d);
  return fmaf(fmaf(-d, r, 1.0f), r, r);
}
__device__ __forceinline__ float cell_sigmoid(float x) { return rcp_ge1(1.0f + __expf(-x)); }
__device__ __forceinline__ float cell_tanh(float x) { return fmaf(-2.0f, rcp_ge1(__expf(2.0f * x) + 1.0f), 1.0f); }

// The larger of two logits, NaN if either is: a vocabulary tile's maximum must
// not pass over a NaN logit, or a tile of nothing else would count as empty.
__device__ __forceinline__ float max_or_nan(float a, float b) { return __builtin_elementwise_maximum(a, b); }

// c <- f c + i g; returns h = o tanh(c), from the gates' pre-activations.
__device__ __forceinline__ float lstm_cell(float ai, float af, float ag, float ao, float& c) {
#pragma clang fp contract(off)
  const float ig = cell_sigmoid(ai) * cell_tanh(ag);
  c = fmaf(cell_sigmoid(af), c, ig);
  return cell_sigmoid(ao) * cell_tanh(c);
}

}  // namespace zo
