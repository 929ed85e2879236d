// Detector-level sum, residual and split on an oversampled internal grid, for the kernels that
// form the per-line predictions there (the splat and the local closure).  As a pass of its own it
// read every line's predictions back and rewrote them: 53 us of 350 an iteration at 2048 x 2048
// internal pixels and 8 lines; from the LDS sums of the splat it costs about 20.
#pragma once

#include <hip/hip_runtime.h>

#include "dev_common.h"

namespace epr {

// One detector pixel, whose F x F internal pixels start at (y, x); P(r, c, s) is line s's
// prediction at internal pixel (y + r, x + c).  Bins every line (the mean), sums the lines, forms
// e = d - P and the positivity-weighted split, and writes e_s to the F x F internal pixels; without
// data (p.d null) writes the binned prediction to p.out instead.  Adds e^2 and d^2 to se, sd.
// The images' rows and lines are multiples of F pixels and at least 16-byte aligned, so a row of
// F values is one store.
template <int NL, int F, bool XDEP, class Pred>
__device__ __forceinline__ void split_bin(const ProbDesc& p, int y, int x, Pred P_at, float& se,
                                          float& sd) {
  const int nx = p.nx, L = p.lp.n;
  float Pv[NL];
  float P = 0.f, S = 0.f;
#pragma unroll
  for (int s = 0; s < NL; ++s) {
    Pv[s] = 0.f;
    if (s < L) {
      float acc = 0.f;
#pragma unroll
      for (int r = 0; r < F; ++r)
#pragma unroll
        for (int c = 0; c < F; ++c) acc += P_at(r, c, s);
      Pv[s] = acc * (1.f / (F * F));
    }
    P += Pv[s];
    S += fmaxf(Pv[s], 0.f);
  }
  const unsigned det = (unsigned)(__mul24(y / F, nx / F) + x / F);
  if (p.d == nullptr) {
    stg(G(p.out), det, P);  // forward model only: the detector intensity, no residual
    return;
  }
  const float dv = ldg(G((const float*)p.d), det);
  const float ev = dv - P;
  se += ev * ev;
  sd += dv * dv;
  const bool hole = !(S > 1e-30f);
  const float inv = hole ? 0.f : 1.f / S;
  const unsigned pix = (unsigned)(__mul24(y, nx) + x);
  const int plane = nx * p.ny;
#pragma unroll
  for (int s = 0; s < NL; ++s) {
    if (s < L) {
      float fw = p.lp.w[s];
      if constexpr (XDEP) {
        if (hole) {
          // x-dependent spectrum: the line's weight averaged over the F internal columns
          fw = 0.f;
#pragma unroll
          for (int c = 0; c < F; ++c) fw += xcol_at(p, x + c, s).x;
          fw *= 1.f / F;
        }
      }
      const float v = (hole ? fw : fmaxf(Pv[s], 0.f) * inv) * ev;
      const unsigned o = (unsigned)(s * plane) + pix;
#pragma unroll
      for (int r = 0; r < F; ++r) {
        if constexpr (F == 2)
          stg((gptr<float2>)G(p.e), (o + (unsigned)(r * nx)) / 2, make_float2(v, v));
        else
          stg((gptr<float4>)G(p.e), (o + (unsigned)(r * nx)) / 4, make_float4(v, v, v, v));
      }
    }
  }
}

}  // namespace epr
