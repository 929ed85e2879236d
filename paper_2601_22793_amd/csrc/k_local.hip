// Local O(L^2) closure (Eq. 1, Methods 4.1) with the fused spectral sum, residual and split.
//
// Per line s, with u = b_s D Y (pixels), I = w_s exp(-a_s X), A = sqrt(I):
//   P_s = I - [D_x(I u_x) + D_y(I u_y)]
//       + 1/2 [D_x D_x(I u_x^2) + D_x D_y(I u_x u_y) + D_y D_x(I u_y u_x) + D_y D_y(I u_y^2)]
//       - q_s [D_x(I D_x Q) + D_y(I D_y Q)],     Q = (D_x D_x A + D_y D_y A) / A,
// with D the central difference inside the image and the one-sided difference on its edges,
// exactly as the composition of derivatives is written in Eq. 1 (D_x and D_y commute, so the two
// mixed terms are one, taken twice).  Order 1 keeps the first bracket only.  Order 3 is the
// second-order non-local model: the transported prediction M_s[I_s], already in e (the splat's
// per-line output), plus the diffraction-pressure term.
//
// One wave computes one line on a strip of kLocalCols output columns x R output rows, alone: each
// lane owns one image column (kLocalHalo lanes of halo on either side), the column neighbours come
// from the adjacent lanes with the wave-shift DPP modes, and the row neighbours stay in registers
// as the wave moves down the R + 2 kLocalHalo rows (fully unrolled).  The nested derivatives so
// need no LDS and no barrier; LDS only carries the finished P_s to the per-pixel sum over lines
// at the end (one barrier).  A workgroup holds one wave per line and strip: local_strips(L)
// strips of every line, so that few-line problems still fill a workgroup.
//
// Bound by vector issue (about 80 instructions per row, line and wave).  Against a version that
// walked the levels of derivatives over 24 x 24 LDS regions with five barriers per line:
// 1080 x 1200, 4 lines: 159 -> 33 us a launch; 256 x 256, 1 line: 8.4 -> 7.0 us.  (An A from its own
// hardware exponential and v_rcp_f32 in the quotients ran in 32 and 6.5 us, with ten times the
// error in the pressure term at optical depth 30.)
#include <hip/hip_runtime.h>

#include <type_traits>

#include "dev_common.h"
#include "epr_internal.h"
#include "split_bin.h"

namespace epr {

constexpr int kLH = kLocalHalo;

// P_s of line s on the strip whose first output pixel is (y0, xs), into Pl[R][64] (lane columns).
// EDGE: some derivative of the strip is one-sided (or a row or column lies off the image: the
// values there are clamped reads that no output uses).  Otherwise every difference is central
// and its halving is folded into the coefficients (exact).
// XDEP: x-dependent spectrum, the line constants are those of the lane's column.
template <int R, int ORDER, bool XDEP, bool EDGE>
__device__ __forceinline__ void local_strip(const ProbDesc& p, int s, int y0, int xs, float* Pl) {
  constexpr int N = R + 2 * kLH;
  const int nx = p.nx, ny = p.ny;
  const int lane = threadIdx.x & 63;
  const int x = xs - kLH + lane;
  const int xc = EDGE ? min(max(x, 0), nx - 1) : x;
  gptr<const float> X = G(p.X);
  gptr<const float> Y = G(p.Y);
  float cw, ca, cb, cq;
  if constexpr (XDEP) {
    const float4 c = xcol_at(p, xc, s);
    cw = c.x; ca = c.y; cb = c.z; cq = c.w;
  } else {
    cw = p.lp.w[s]; ca = p.lp.a[s]; cb = p.lp.b[s]; cq = p.lp.q[s];
  }

  // input row i is image row y0 - kLH + i
  float Xv[N], Yv[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int y = y0 - kLH + i;
    const int yc = EDGE ? min(max(y, 0), ny - 1) : y;
    Xv[i] = ldg(X + yc * nx, (unsigned)xc);
    if constexpr (ORDER != kOrderTransportWkb1) Yv[i] = ldg(Y + yc * nx, (unsigned)xc);
  }

  const bool xfirst = x == 0, xlast = x == nx - 1;
  const float sx = (xfirst || xlast) ? 1.f : 0.5f;
  // D_x f; !EDGE: 2 D_x f
  auto dx = [&](float f) {
    float l = lane_left(f), r = lane_right(f);
    if constexpr (EDGE) {
      l = xfirst ? f : l;
      r = xlast ? f : r;
      return sx * (r - l);
    }
    return r - l;
  };
  // D_y at input row i from the values of rows i - 1, i, i + 1; !EDGE: 2 D_y
  auto dy = [&](int i, float fm, float f0, float fp) {
    if constexpr (EDGE) {
      const int y = y0 - kLH + i;
      const float t = y == 0 ? f0 : fm, b = y == ny - 1 ? f0 : fp;
      return ((y == 0 || y == ny - 1) ? 1.f : 0.5f) * (b - t);
    }
    return fp - fm;
  };
  // coefficients of once, twice and four times differentiated terms
  constexpr float k1 = EDGE ? 1.f : 0.5f, k2 = k1 * k1, k4 = k2 * k2;
  const float cbg = cb * k1, cqg = cq * k4;

  float I[N], dyA[N], Q[N], GY[N], Ix[N], Iy[N], Pxx[N], Pxy[N], Pyy[N], dyP[N];
  Root A[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    // the fourth differences of A amplify its rounding, so A is the root of expf's I: an exp2 of
    // the scaled argument would be off by the argument's rounding, which grows with the depth
    I[i] = cw * expf(-ca * Xv[i]);
    if constexpr (ORDER >= 2) {
      A[i] = root_of(fmaxf(I[i], kRootMin));
      if (i >= 2) dyA[i - 1] = dy(i - 1, A[i - 2].a, A[i - 1].a, A[i].a);
    }
    const int j = i - 2;
    if constexpr (ORDER != kOrderTransportWkb1) {
      if (j >= 2 && j < N - 2) {
        const float ux = cbg * dx(Yv[j]), uy = cbg * dy(j, Yv[j - 1], Yv[j], Yv[j + 1]);
        Ix[j] = I[j] * ux;
        Iy[j] = I[j] * uy;
        if constexpr (ORDER >= 2) {
          Pxx[j] = Ix[j] * ux;
          Pxy[j] = Ix[j] * uy;
          Pyy[j] = Iy[j] * uy;
        }
      }
    }
    if constexpr (ORDER >= 2) {
      if (j >= 2 && j < N - 2)
        Q[j] = over_root(dx(dx(A[j].a)) + dy(j, dyA[j - 1], dyA[j], dyA[j + 1]), A[j]);
      const int k = i - 3;
      if (k >= 3 && k < N - 3) {
        GY[k] = I[k] * dy(k, Q[k - 1], Q[k], Q[k + 1]);
        if constexpr (ORDER == 2) dyP[k] = dy(k, Pyy[k - 1], Pyy[k], Pyy[k + 1]);
      }
    }
    const int m = i - kLH;
    if (m >= kLH && m < N - kLH) {
      float P;
      if constexpr (ORDER == kOrderTransportWkb1) {
        const int y = y0 - kLH + m;
        const int yc = EDGE ? min(max(y, 0), ny - 1) : y;
        P = ldg(G((const float*)p.e) + ((size_t)s * ny + yc) * nx, (unsigned)xc);
      } else {
        P = I[m] - k1 * (dx(Ix[m]) + dy(m, Iy[m - 1], Iy[m], Iy[m + 1]));
        if constexpr (ORDER >= 2) {
          const float xy = dx(dy(m, Pxy[m - 1], Pxy[m], Pxy[m + 1]));
          const float t2 = dx(dx(Pxx[m])) + 2.f * xy + dy(m, dyP[m - 1], dyP[m], dyP[m + 1]);
          P += (0.5f * k2) * t2;
        }
      }
      if constexpr (ORDER >= 2) {
        const float t3 = dx(I[m] * dx(Q[m])) + dy(m, GY[m - 1], GY[m], GY[m + 1]);
        P -= cqg * t3;
      }
      Pl[(m - kLH) * 64 + lane] = P;
    }
  }
}

template <int R, int ORDER, bool XDEP>
__device__ __forceinline__ void local_body(const ProbDesc& p, int local, int mode) {
  extern __shared__ float Pl[];  // [line][strip][R][64]
  const int nx = p.nx, ny = p.ny, L = p.lp.n;
  const int ns = local_strips(L);
  const int ntx = (nx + ns * kLocalCols - 1) / (ns * kLocalCols);
  const int y0 = (local / ntx) * R, tx0 = (local - (local / ntx) * ntx) * (ns * kLocalCols);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  // the short strips (small images, latency) read the data before the closure; a wave sums the
  // rows q = w + k nw, at most R of them
  float dpre[R <= 8 ? R : 1];
  if constexpr (R <= 8) {
    if (mode == kLocalSplit) {
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int q = w + k * nw;
        if (q < R * ns) {
          const int r = q / ns, j = q - r * ns;
          const int y = min(y0 + r, ny - 1);
          const int x = min(max(tx0 + j * kLocalCols + lane - kLH, 0), nx - 1);
          dpre[k] = ldg(G((const float*)p.d), (unsigned)(__mul24(y, nx) + x));
        }
      }
    }
  }
  for (int u = w; u < L * ns; u += nw) {
    const int s = u / ns, xs = tx0 + (u - s * ns) * kLocalCols;
    if (xs >= nx) continue;
    const bool inner = xs >= kLH && xs + kLocalCols + kLH <= nx && y0 >= kLH && y0 + R + kLH <= ny;
    if (inner)
      local_strip<R, ORDER, XDEP, false>(p, s, y0, xs, Pl + u * R * 64);
    else
      local_strip<R, ORDER, XDEP, true>(p, s, y0, xs, Pl + u * R * 64);
  }
  __syncthreads();

  // sum over the lines, residual and split: one strip row per wave and step
  float se = 0.f, sd = 0.f;
  auto sum_row = [&](int q, float dq) {
    const int r = q / ns, j = q - r * ns;
    const int y = y0 + r, x = tx0 + j * kLocalCols + lane - kLH;
    if (lane < kLH || lane >= kLH + kLocalCols || y >= ny || x >= nx) return;
    const unsigned pix = (unsigned)(__mul24(y, nx) + x);
    const float* Pr = Pl + (j * R + r) * 64 + lane;
    const int ls = ns * R * 64;  // line stride
    float P = 0.f, S = 0.f;
    for (int s = 0; s < L; ++s) {
      const float v = Pr[s * ls];
      P += v;
      S += fmaxf(v, 0.f);
    }
    if (mode == kLocalForward) {
      stg(G(p.out), pix, P);
    } else {
      const float dv = R <= 8 ? dq : ldg(G((const float*)p.d), pix);
      const float e = dv - P;
      se += e * e;
      sd += dv * dv;
      const bool hole = !(S > 1e-30f);
      const float inv = hole ? 0.f : 1.f / S;
      for (int s = 0; s < L; ++s) {
        float fw = p.lp.w[s];
        if constexpr (XDEP) fw = xcol_at(p, x, s).x;
        const float share = hole ? fw : fmaxf(Pr[s * ls], 0.f) * inv;
        stg(G(p.e) + (size_t)s * nx * ny, pix, share * e);
      }
    }
  };
  if (mode == kLocalBin) {
    // an oversampled internal grid: the residual and split at the detector pixels (strips are
    // whole detector pixels), one detector row of a strip per wave and step
    auto bin = [&](auto factor) {
      constexpr int F = decltype(factor)::value;
      static_assert(kLocalCols % F == 0 && R % F == 0, "whole detector pixels");
      for (int q = w; q < R / F * ns; q += nw) {
        const int r0 = q / ns * F, j = q - q / ns * ns;
        const int y = y0 + r0, x = tx0 + j * kLocalCols + lane * F;
        if (lane >= kLocalCols / F || y >= ny || x >= nx) continue;
        const float* Pr = Pl + (j * R + r0) * 64 + kLH + lane * F;
        split_bin<kMaxLines, F, XDEP>(p, y, x, [&](int r, int c, int s) {
          return Pr[s * ns * R * 64 + r * 64 + c];
        }, se, sd);
      }
    };
    if (p.os == 2)
      bin(std::integral_constant<int, 2>{});
    else
      bin(std::integral_constant<int, 4>{});
  } else if constexpr (R <= 8) {
#pragma unroll
    for (int k = 0; k < R; ++k)
      if (w + k * nw < R * ns) sum_row(w + k * nw, dpre[k]);
  } else {
    for (int q = w; q < R * ns; q += nw) sum_row(q, 0.f);
  }
  if ((mode == kLocalSplit || mode == kLocalBin) && p.resid != nullptr) {
    __shared__ float red[2][kMaxLines];
    se = wave_sum(se);
    sd = wave_sum(sd);
    if (lane == 0) {
      red[0][w] = se;
      red[1][w] = sd;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      float te = 0.f, td = 0.f;
      for (int i = 0; i < nw; ++i) {
        te += red[0][i];
        td += red[1][i];
      }
      G(p.resid)[2 * local] = te;
      G(p.resid)[2 * local + 1] = td;
    }
  }
}

template <bool B, int R, int ORDER, bool XDEP>
__global__ __launch_bounds__(64 * kMaxLines) void k_local(KArgs a, const ProbDesc* __restrict__ table) {
  EPR_DISPATCH(B, a, table, xcd_remap(blockIdx.x, gridDim.x), (local_body<R, ORDER, XDEP>), a.mode);
}

template <int R, int ORDER>
void launch_local_ro(const KArgs& a, int total_blocks, hipStream_t s, int lines) {
  const int waves = lines * local_strips(lines);
  const size_t lds = sizeof(float) * 64 * (size_t)R * waves;
  const dim3 grid(total_blocks), block(64 * waves);
  if (a.xdep && a.table)
    hipLaunchKernelGGL((k_local<true, R, ORDER, true>), grid, block, lds, s, a, a.table);
  else if (a.table)
    hipLaunchKernelGGL((k_local<true, R, ORDER, false>), grid, block, lds, s, a, a.table);
  else if (a.p.xcol)
    hipLaunchKernelGGL((k_local<false, R, ORDER, true>), grid, block, lds, s, a, a.table);
  else
    hipLaunchKernelGGL((k_local<false, R, ORDER, false>), grid, block, lds, s, a, a.table);
}

// lines: the line count of the launch's problems; rows: their rows per strip (ProbDesc::lrows).
hipError_t launch_local(const KArgs& a, int total_blocks, hipStream_t s, int order, int lines,
                        int rows) {
  if (lines < 1 || lines > kMaxLines || (rows != 4 && rows != 8 && rows != 16)) return hipErrorInvalidValue;
  if (rows == 4) {
    if (order == 1) launch_local_ro<4, 1>(a, total_blocks, s, lines);
    else if (order == 2) launch_local_ro<4, 2>(a, total_blocks, s, lines);
    else launch_local_ro<4, 3>(a, total_blocks, s, lines);
  } else if (rows == 8) {
    if (order == 1) launch_local_ro<8, 1>(a, total_blocks, s, lines);
    else if (order == 2) launch_local_ro<8, 2>(a, total_blocks, s, lines);
    else launch_local_ro<8, 3>(a, total_blocks, s, lines);
  } else {
    if (order == 1) launch_local_ro<16, 1>(a, total_blocks, s, lines);
    else if (order == 2) launch_local_ro<16, 2>(a, total_blocks, s, lines);
    else launch_local_ro<16, 3>(a, total_blocks, s, lines);
  }
  return hipGetLastError();
}

}  // namespace epr
