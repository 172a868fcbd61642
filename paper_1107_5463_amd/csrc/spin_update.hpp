// spin_update.hpp -- one Metropolis attempt of a continuous spin and the
// couplings of its bonds, shared by the kernels of continuous.hip and
// brick.hip (internal).
#pragma once

#include "device.hpp"

namespace smc {

// Metropolis acceptance of a continuous-spin move (Eq. (2)): the accurate
// path is metropolis_fp32; fast math takes the library's __expf.
template <bool FAST>
__device__ __forceinline__ bool cont_accept(float dE, uint32_t wacc, float beta, float bl2e) {
  if (FAST) return (dE <= 0.0f) | (u01f(wacc) < __expf(-beta * dE));
  return metropolis_fp32(dE, u01f(wacc), bl2e);
}
template <bool FAST>
__device__ __forceinline__ void sincos_f(float x, float* s, float* c) {
  if (FAST) {
    *s = __sinf(x);
    *c = __cosf(x);
  } else {
    sincosf(x, s, c);
  }
}

// sin and cos of the angle 2 pi f (f in turns).  Exact quadrant reduction
// f = q/4 + r with q = rint(4 f) and |r| <= 1/8, then the Taylor series of sin
// (to x^9) and cos (to x^10) at x = 2 pi r, |x| <= pi/4, whose truncation
// errors (x^11/11! < 2e-9, x^12/12! < 2e-10) lie below FP32 rounding.
__device__ __forceinline__ void sincos_turns(float f, float* s, float* c) {
  const float q = rintf(4.0f * f);
  const float r = fmaf(-0.25f, q, f);
  const float x = 6.28318530717958647692f * r;
  const float x2 = x * x;
  float ps = fmaf(x2, 1.0f / 362880.0f, -1.0f / 5040.0f);
  ps = fmaf(x2, ps, 1.0f / 120.0f);
  ps = fmaf(x2, ps, -1.0f / 6.0f);
  const float sx = fmaf(x * x2, ps, x);
  float pc = fmaf(x2, -1.0f / 3628800.0f, 1.0f / 40320.0f);
  pc = fmaf(x2, pc, -1.0f / 720.0f);
  pc = fmaf(x2, pc, 1.0f / 24.0f);
  pc = fmaf(x2, pc, -0.5f);
  const float cx = fmaf(x2, pc, 1.0f);
  // angle = q pi/2 + x
  const int qi = (int)q & 3;
  const float a = (qi & 1) ? cx : sx;
  const float b = (qi & 1) ? sx : cx;
  *s = (qi & 2) ? -a : a;
  *c = (qi == 1 || qi == 2) ? -b : b;
}

// Coupling of the bond from site (cc, jj) to its +mu neighbour.
template <int JK>
__device__ __forceinline__ float bond(const void* J, float J0, int64_t Nh, int mu, uint32_t cc,
                                      int64_t jj) {
  if (JK == 1) return J0 * (float)((const int8_t*)J)[((int64_t)mu * 2 + cc) * Nh + jj];
  if (JK == 2) return ((const float*)J)[((int64_t)mu * 2 + cc) * Nh + jj];
  return J0;
}

// One XY Metropolis attempt at a site with spin (s0, s1) in field h: rotate
// by delta (2 u_prop - 1), accept iff dE <= 0 or u_acc < exp(-beta dE).
template <bool FAST>
__device__ __forceinline__ bool xy_update(float& s0, float& s1, const float h[3],
                                          const uint32_t wacc, const uint32_t wprop,
                                          const float beta, const float bl2e,
                                          const float delta) {
  // rotation angle delta (2u - 1): in radians for the hardware sin / cos of
  // the fast path, in turns for the series otherwise
  float sD, cD;
  if (FAST)
    sincos_f<true>(delta * (2.0f * u01f(wprop) - 1.0f), &sD, &cD);
  else
    sincos_turns((delta * 0.159154943091895335769f) * (2.0f * u01f(wprop) - 1.0f), &sD, &cD);
  // (the fused products written out: left to the compiler, which of two products
  // is fused depends on the code around them, and kernels must agree in all bits)
  const float n0 = fmaf(s0, cD, -(s1 * sD));
  const float n1 = fmaf(s0, sD, s1 * cD);
  const float dE = -fmaf(n0 - s0, h[0], (n1 - s1) * h[1]);
  const bool accept = cont_accept<FAST>(dE, wacc, beta, bl2e);
  if (accept) {
    s0 = n0;
    s1 = n1;
  }
  return accept;
}

// One Heisenberg Metropolis attempt: a point uniform on the cap of
// 1 - cos(theta_max) = omc around sv (w1: cos alpha, w2: azimuth), accepted
// with u_acc = u(w0).
template <bool FAST>
__device__ __forceinline__ bool heis_update(float sv[3], const float h[3], const uint32_t w0,
                                            const uint32_t w1, const uint32_t w2,
                                            const float beta, const float bl2e,
                                            const float omc) {
  // sin alpha from 1 - cos alpha directly: (1 - c)(1 + c) keeps its relative
  // precision for small caps, where 1 - c^2 would cancel.  The argument is at
  // least omc 2^-24 (a normal number), so the hardware square root (about one
  // ulp) needs no denormal scaling.
  // (the fused products are written out here too, as in xy_update)
  const float u1 = u01f(w1);
  const float omca = u1 * omc;
  const float ca = fmaf(-u1, omc, 1.0f);
  const float sa = __builtin_amdgcn_sqrtf(omca * fmaf(-u1, omc, 2.0f));
  // frame axis: smallest |s_k|, lowest k on ties
  const float a0 = fabsf(sv[0]), a1 = fabsf(sv[1]), a2 = fabsf(sv[2]);
  int k = 0;
  float am = a0;
  if (a1 < am) { k = 1; am = a1; }
  if (a2 < am) { k = 2; }
  const float sk = k == 0 ? sv[0] : (k == 1 ? sv[1] : sv[2]);
  float e1[3] = {-sk * sv[0], -sk * sv[1], -sk * sv[2]};
  if (k == 0) e1[0] = fmaf(-sk, sv[0], 1.0f);
  if (k == 1) e1[1] = fmaf(-sk, sv[1], 1.0f);
  if (k == 2) e1[2] = fmaf(-sk, sv[2], 1.0f);
  const float inv = rsqrtf(fmaf(e1[2], e1[2], fmaf(e1[0], e1[0], e1[1] * e1[1])));
  e1[0] *= inv; e1[1] *= inv; e1[2] *= inv;
  const float e2[3] = {fmaf(sv[1], e1[2], -(sv[2] * e1[1])), fmaf(sv[2], e1[0], -(sv[0] * e1[2])),
                       fmaf(sv[0], e1[1], -(sv[1] * e1[0]))};
  // azimuth 2 pi u(w2)
  float sph, cph;
  if (FAST)
    sincos_f<true>(6.28318530717958647692f * u01f(w2), &sph, &cph);
  else
    sincos_turns(u01f(w2), &sph, &cph);
  float nv[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) nv[q] = fmaf(ca, sv[q], sa * fmaf(cph, e1[q], sph * e2[q]));
  const float dE = -fmaf(nv[2] - sv[2], h[2], fmaf(nv[0] - sv[0], h[0], (nv[1] - sv[1]) * h[1]));
  const bool accept = cont_accept<FAST>(dE, w0, beta, bl2e);
  if (accept) {
    sv[0] = nv[0];
    sv[1] = nv[1];
    sv[2] = nv[2];
  }
  return accept;
}

}  // namespace smc
