// Epilogues of the GEMMs that keep fp32 results (gemm.hip and
// gemm_split.hip): one output element (r, c) from its accumulated sum v0
// (and v1 in the dual kernels).  apply() returns the value that a later GEMM
// takes as an operand (the logits for an output layer), 0 where there is
// none.
#pragma once

#include "act.h"
#include "hf_internal.h"

namespace hfk {
namespace {

struct EFwd {
  static __device__ __forceinline__ float apply(const EpiArgs& e, int r, int c,
                                               float v0, float) {
    const float z = v0 + e.bias[c];
    const float a = e.hidden ? act_f(e.act, z) : z;
    e.out0[(size_t)r * e.ldo + c] = a;
    return a;
  }
};
struct EFwdRFwd {
  static __device__ __forceinline__ float apply(const EpiArgs& e, int r, int c,
                                               float v0, float v1) {
    const size_t o = (size_t)r * e.ldo + c;
    const float z = v0 + e.bias[c];
    const float rz = v1 + e.rbias[c];
    if (e.hidden) {
      const float a = act_f(e.act, z);
      e.out0[o] = a;
      e.out1[o] = rz;
      e.out2[o] = act_d1(e.act, a) * rz;
    } else {
      e.out0[o] = z;
      e.out1[o] = rz;
    }
    return 0.0f;
  }
};
struct ERFwd {
  static __device__ __forceinline__ float apply(const EpiArgs& e, int r, int c,
                                               float v0, float) {
    const size_t o = (size_t)r * e.ldo + c;
    const float rz = v0 + e.rbias[c];
    if (e.out1) e.out1[o] = rz;      // null: RZ not needed downstream
    if (!e.hidden) return rz;
    const float ra = act_d1(e.act, e.aux0[(size_t)r * e.lda + c]) * rz;
    e.out2[o] = ra;
    return ra;
  }
};
struct EBwd {
  static __device__ __forceinline__ float apply(const EpiArgs& e, int r, int c,
                                               float v0, float) {
    const float d = v0 * act_d1(e.act, e.aux0[(size_t)r * e.lda + c]);
    e.out0[(size_t)r * e.ldo + c] = d;
    return d;
  }
};
// backward data that also caches E * phi''(A) for the Hessian product
struct EBwdE2 {
  static __device__ __forceinline__ float apply(const EpiArgs& e, int r, int c,
                                               float v0, float) {
    const size_t o = (size_t)r * e.ldo + c;
    const float a = e.aux0[(size_t)r * e.lda + c];
    const float d = v0 * act_d1(e.act, a);
    e.out0[o] = d;
    e.out2[o] = v0 * act_d2(e.act, a);
    return d;
  }
};
struct EBwdRBwd {
  static __device__ __forceinline__ float apply(const EpiArgs& e, int r, int c,
                                               float v0, float v1) {
    const size_t o = (size_t)r * e.ldo + c;
    const size_t ia = (size_t)r * e.lda + c;
    const float a = e.aux0[ia];
    const float d1 = act_d1(e.act, a);
    e.out0[o] = v0 * d1;
    e.out1[o] = v1 * d1 + v0 * act_d2(e.act, a) * e.aux1[ia];
    return 0.0f;
  }
};
struct ERBwd {
  static __device__ __forceinline__ float apply(const EpiArgs& e, int r, int c,
                                               float v0, float) {
    const size_t ia = (size_t)r * e.lda + c;
    const float d = v0 * act_d1(e.act, e.aux0[ia]) + e.aux2[ia] * e.aux1[ia];
    e.out1[(size_t)r * e.ldo + c] = d;
    return d;
  }
};
struct EGNBwd {
  static __device__ __forceinline__ float apply(const EpiArgs& e, int r, int c,
                                               float v0, float) {
    const float d = v0 * act_d1(e.act, e.aux0[(size_t)r * e.lda + c]);
    e.out1[(size_t)r * e.ldo + c] = d;
    return d;
  }
};
struct EStore {
  static __device__ __forceinline__ float apply(const EpiArgs& e, int r, int c,
                                               float v0, float) {
    e.out0[(size_t)blockIdx.z * e.split_stride + (size_t)r * e.ldo + c] = v0;
    return 0.0f;
  }
};

}  // namespace
}  // namespace hfk
