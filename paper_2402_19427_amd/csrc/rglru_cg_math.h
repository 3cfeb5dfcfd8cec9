// Complex arithmetic of the complex-gated layer (Appendix B) in bf16 storage.
#pragma once
#include "rglru_pass.h"

namespace rglru {
namespace pass {

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(fmaf(a.x, b.x, -a.y * b.y), fmaf(a.x, b.y, a.y * b.x));
}
// (A2, E2) o (A1, E1): A1, E1 applied first
__device__ __forceinline__ void cthen(float2 &A, float2 &E, float2 A2, float2 E2) {
  const float2 t = cmul(A2, E);
  E = make_float2(t.x + E2.x, t.y + E2.y);
  A = cmul(A2, A);
}
// a~_t from the pre-activation p: base-2 logarithm of |a~_t| per r_t and phase (in revolutions) per r_t
struct Decay {
  float l2, rev;
  __device__ __forceinline__ Decay() {}
  __device__ __forceinline__ Decay(const Problem &p, int h) {
    l2 = neg_c_softplus(p.Lambda[h], p.c) * LOG2E;
    rev = p.c * p.theta[h] * 0.15915494309189535f;
  }
};
__device__ __forceinline__ float2 cdecay(const Decay &k, float rg, float &l2, float &mod) {
  l2 = k.l2 * rg;
  mod = __builtin_amdgcn_exp2f(l2);
  const float ph = __builtin_amdgcn_fractf(k.rev * rg);
  return make_float2(mod * __builtin_amdgcn_cosf(ph), mod * __builtin_amdgcn_sinf(ph));
}
// 1 - |a~_t|^2 to fp32's own accuracy (with the forward's form, which may be 2^-22 too small, db_x was
// 5.2e-6 off instead of 2.6e-6): six terms of -expm1(z) down to z = -0.35, where z^7 / 8! is below 2e-8
__device__ __forceinline__ float one_minus_mod2(float mod, float l2) {
  const float z = 2.f * LN2 * l2;
  float s = fmaf(z, 1.f / 5040.f, 1.f / 720.f);
  s = fmaf(s, z, 1.f / 120.f);
  s = fmaf(s, z, 1.f / 24.f);
  s = fmaf(s, z, 1.f / 6.f);
  s = fmaf(s, z, 0.5f);
  s = fmaf(s, z, 1.f);
  return z > -0.35f ? -z * s : fmaf(-mod, mod, 1.f);
}
__device__ __forceinline__ float sigm(float v) { return __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-LOG2E * v)); }

}  // namespace pass
}  // namespace rglru
