// Vector-Jacobian products of the forward models (Eqs. 1-5) with respect to the phase and
// absorption maps, for the autograd backward.
//
// Non-local model: P = sum_s M_s(u_s)[I_s], I_s = w_s exp(-a_s A), u_s = b_s D phase.  With
// g = dL/dP:
//   dL/dI_s  = M_s^* g   (bilinear interpolation of g at the mapped point, Eq. 4)
//   dL/du_s  = I_s * gradient of that interpolant with respect to the mapped point
//              (constant inside a cell: the splat is piecewise linear in u)
//   grad_A   = sum_s -a_s I_s dL/dI_s
//   grad_phi = D_x^T Gx + D_y^T Gy,  G = sum_s b_s dL/du_s
// The ray map is recomputed from the phase; nothing is kept from the forward call.
//
// XDEP: x-dependent spectrum (Methods 4.3 remark).  Both maps are the thickness tau, and
// w_s, a_s (= mu_s), b_s and q_s are read at each pixel's column; dL/dtau is then
// grad_A + D_x^T G_x + D_y^T G_y (`accumulate`).
#include <hip/hip_runtime.h>

#include "dev_common.h"
#include "epr_internal.h"

namespace epr {

// {w_s, a_s, b_s, q_s} of line s at column x
template <bool XDEP>
__device__ __forceinline__ float4 line_wabq(const ProbDesc& p, int x, int s) {
  if constexpr (XDEP) return xcol_at(p, x, s);
  else return make_float4(p.lp.w[s], p.lp.a[s], p.lp.b[s], p.lp.q[s]);
}

// Transpose of D along one axis of length n at index j, from the values at j - 1, j and j + 1:
// D has rows (-1, 1) at 0, (-1/2, 0, 1/2) inside and (-1, 1) at n - 1.
__device__ __forceinline__ float d_transpose3(float l, float m, float r, int j, int n) {
  if (j == 0) return -m - 0.5f * r;
  if (j == n - 1) return 0.5f * l + m;
  return (j == 1 ? l : 0.5f * l) - (j == n - 2 ? r : 0.5f * r);
}

// ---------------------------------------------------------------------------------------------
// Non-local model.  A workgroup of 8 waves computes G and the absorption gradient on a region of
// 64 x 32 pixels, a lane one column of 4 consecutive rows, and writes both gradients on the
// 62 x 30 pixels inside: D_x^T G_x from the neighbouring lanes, D_y^T G_y through LDS, so G is never
// in memory (the 10 % computed twice cost less than a pass that reads G back).  All lines sample the
// same g: the region's window of it, zero off the image, is staged in LDS with the halo that the
// region's own shifts need, and the taps come from there; shifts too large for the window read g
// itself.  (Taps from memory take the L1 36 accesses per 64 pixels and line beside 44 vector
// issue slots.)  32 KB of LDS and 64 VGPRs hold four workgroups a CU.
// 2048 x 2048, 8 lines: 76 + 16 us (taps from memory, transposes as a second pass) -> 67 us with the
// transposes here -> 58 us with the window; bound by vector issue (41 us).
// ---------------------------------------------------------------------------------------------
constexpr int kVjpRows = 4, kVjpWaves = 8;
constexpr int kVjpWindow = 8192;  // floats: shifts of 6 pixels take 78 x 46, of 20 pixels 106 x 74
constexpr int kVjpTX = 62, kVjpTY = kVjpRows * kVjpWaves - 2;

template <bool XDEP>
__global__ __launch_bounds__(64 * kVjpWaves) void k_vjp(KArgs a, float* __restrict__ gphi,
                                                        float* __restrict__ gA, int accumulate) {
  __shared__ float W[kVjpWindow];  // the window of g, then G_y
  __shared__ float red[2][kVjpWaves];
  const ProbDesc& p = a.p;
  const int nx = p.nx, ny = p.ny, L = p.lp.n;
  const int local = xcd_remap(blockIdx.x, gridDim.x);
  const int ntx = (nx + kVjpTX - 1) / kVjpTX;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int x = (local % ntx) * kVjpTX - 1 + lane;
  const int y0 = (local / ntx) * kVjpTY - 1 + w * kVjpRows;
  // region pixels off the image compute the nearest image pixel's values, which nothing reads
  const int xc = min(max(x, 0), nx - 1);
  const int xl = max(xc - 1, 0), xh = min(xc + 1, nx - 1);
  const float cx = xh - xl == 2 ? 0.5f : 1.f;
  gptr<const float> g = G(p.d);  // incoming gradient dL/dP
  gptr<const float> X = G(p.X);
  gptr<const float> Y = G(p.Y);
  int yc[kVjpRows];
  float px[kVjpRows], py[kVjpRows], av[kVjpRows];
#pragma unroll
  for (int r = 0; r < kVjpRows; ++r) {
    yc[r] = min(max(y0 + r, 0), ny - 1);
    const int yl = max(yc[r] - 1, 0), yh = min(yc[r] + 1, ny - 1);
    px[r] = cx * (ldg(Y + yc[r] * nx, (unsigned)xh) - ldg(Y + yc[r] * nx, (unsigned)xl));
    py[r] = (yh - yl == 2 ? 0.5f : 1.f) * (ldg(Y + yh * nx, (unsigned)xc) - ldg(Y + yl * nx, (unsigned)xc));
    av[r] = ldg(X + yc[r] * nx, (unsigned)xc);
  }
  // window of g that every tap of the region falls into (halo from the region's own largest shifts;
  // NaNs drop out of the maxima and sample their own pixel)
  float mx = 0.f, my = 0.f;
#pragma unroll
  for (int r = 0; r < kVjpRows; ++r) {
    mx = fmaxf(mx, fabsf(px[r]));
    my = fmaxf(my, fabsf(py[r]));
  }
  mx = lane64_max(mx);
  my = lane64_max(my);
  if (lane == 0) {
    red[0][w] = mx;
    red[1][w] = my;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kVjpWaves; ++k) {
    mx = fmaxf(mx, red[0][k]);
    my = fmaxf(my, red[1][k]);
  }
  const int hx = halo_from(p.lp.b_absmax, mx), hy = halo_from(p.lp.b_absmax, my);
  const int pitch = 64 + 2 * hx, rows = kVjpRows * kVjpWaves + 2 * hy;
  const int wx0 = (local % ntx) * kVjpTX - 1 - hx, wy0 = (local / ntx) * kVjpTY - 1 - hy;
  const bool windowed = (hx < 64 && hy < 64) && pitch * rows <= kVjpWindow;
  if (windowed) {
    for (int q = w; q < rows; q += kVjpWaves) {
      const int y = wy0 + q;
      const bool yin = (unsigned)y < (unsigned)ny;
      gptr<const float> grow = g + min(max(y, 0), ny - 1) * nx;
      for (int cc = lane; cc < pitch; cc += 64) {
        const int xx = wx0 + cc;
        const float v = ldg(grow, (unsigned)min(max(xx, 0), nx - 1));
        W[q * pitch + cc] = yin && (unsigned)xx < (unsigned)nx ? v : 0.f;
      }
    }
    __syncthreads();
  }

  float sa[kVjpRows] = {}, sx[kVjpRows] = {}, sy[kVjpRows] = {};
  for (int s = 0; s < L; ++s) {
    const float4 c = line_wabq<XDEP>(p, xc, s);
    float dx[kVjpRows], dy[kVjpRows], g00[kVjpRows], g10[kVjpRows], g01[kVjpRows], g11[kVjpRows];
#pragma unroll
    for (int r = 0; r < kVjpRows; ++r) {
      // cell and in-cell position as the splat forms them
      const float ux = c.z * px[r], uy = c.z * py[r];
      dx[r] = __builtin_amdgcn_fractf(ux);
      dy[r] = __builtin_amdgcn_fractf(uy);
      const int xt = xc + floor_to_int(ux), yt = yc[r] + floor_to_int(uy);
      if (windowed) {
        const float* q = W + (__mul24(yt - wy0, pitch) + xt - wx0);
        g00[r] = q[0];
        g10[r] = q[1];
        g01[r] = q[pitch];
        g11[r] = q[pitch + 1];
      } else {
        const bool xi0 = (unsigned)xt < (unsigned)nx, xi1 = (unsigned)(xt + 1) < (unsigned)nx;
        const bool yi0 = (unsigned)yt < (unsigned)ny, yi1 = (unsigned)(yt + 1) < (unsigned)ny;
        const int x0 = min(max(xt, 0), nx - 1), x1 = min(max(xt + 1, 0), nx - 1);
        const int r0 = __mul24(min(max(yt, 0), ny - 1), nx);
        const int r1 = __mul24(min(max(yt + 1, 0), ny - 1), nx);
        const float v00 = ldg(g, (unsigned)(r0 + x0)), v10 = ldg(g, (unsigned)(r0 + x1));
        const float v01 = ldg(g, (unsigned)(r1 + x0)), v11 = ldg(g, (unsigned)(r1 + x1));
        g00[r] = xi0 && yi0 ? v00 : 0.f;
        g10[r] = xi1 && yi0 ? v10 : 0.f;
        g01[r] = xi0 && yi1 ? v01 : 0.f;
        g11[r] = xi1 && yi1 ? v11 : 0.f;
      }
    }
#pragma unroll
    for (int r = 0; r < kVjpRows; ++r) {
      const float I = c.x * expf(-c.y * av[r]);
      const float d0 = g10[r] - g00[r], d1 = g11[r] - g01[r], e0 = g01[r] - g00[r], cc = d1 - d0;
      const float gux = fmaf(dy[r], cc, d0), guy = fmaf(dx[r], cc, e0);
      const float gI = fmaf(dy[r], guy, fmaf(dx[r], d0, g00[r]));
      sa[r] = fmaf(-c.y * I, gI, sa[r]);
      sx[r] = fmaf(c.z * I, gux, sx[r]);
      sy[r] = fmaf(c.z * I, guy, sy[r]);
    }
  }
  float(*Gy)[64] = reinterpret_cast<float(*)[64]>(W);
  __syncthreads();  // every wave has read its taps
#pragma unroll
  for (int r = 0; r < kVjpRows; ++r) Gy[w * kVjpRows + r][lane] = sy[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kVjpRows; ++r) {
    const int q = w * kVjpRows + r, y = y0 + r;
    const float l = lane_left(sx[r]), h = lane_right(sx[r]);
    if (q == 0 || q == kVjpRows * kVjpWaves - 1 || y >= ny) continue;
    if (lane == 0 || lane == 63 || x >= nx) continue;
    const float t = d_transpose3(l, sx[r], h, x, nx) +
                    d_transpose3(Gy[q - 1][lane], sy[r], Gy[q + 1][lane], y, ny);
    const unsigned o = (unsigned)(__mul24(y, nx) + x);
    if (accumulate) {
      stg(G(gphi), o, sa[r] + t);
    } else {
      stg(G(gphi), o, t);
      stg(G(gA), o, sa[r]);
    }
  }
}

// gphi = D_x^T Gx + D_y^T Gy, or (accumulate) that added to gphi.
constexpr int kTrThreads = 256;
__global__ __launch_bounds__(kTrThreads) void k_vjp_transpose(KArgs a, const float* __restrict__ Gx,
                                                              const float* __restrict__ Gy,
                                                              float* __restrict__ gphi,
                                                              int accumulate) {
  const ProbDesc& p = a.p;
  const int nx = p.nx, ny = p.ny;
  const int i = blockIdx.x * kTrThreads + threadIdx.x;
  if (i >= nx * ny) return;
  const int y = i / nx, x = i - y * nx;
  // neighbours off the image are clamped reads that the one-sided rows do not use
  const unsigned row = (unsigned)__mul24(y, nx);
  const int xl = max(x - 1, 0), xh = min(x + 1, nx - 1), yl = max(y - 1, 0), yh = min(y + 1, ny - 1);
  gptr<const float> gx = G(Gx);
  gptr<const float> gy = G(Gy);
  const float t = d_transpose3(ldg(gx, row + xl), ldg(gx, row + x), ldg(gx, row + xh), x, nx) +
                  d_transpose3(ldg(gy, (unsigned)(__mul24(yl, nx) + x)), ldg(gy, row + x),
                               ldg(gy, (unsigned)(__mul24(yh, nx) + x)), y, ny);
  gphi[i] = accumulate ? gphi[i] + t : t;
}

// ---------------------------------------------------------------------------------------------
// Local closures (Eq. 1) and the diffraction-pressure term of the second-order non-local model.
// Per line s, with u = b_s D Y, I = w_s exp(-a_s X), A = sqrt(I), Q = (D_x D_x A + D_y D_y A) / A,
// k = D^T G and h_ab = the transpose of D_a D_b applied to G (G = dL/dP, common to all lines):
//   first order    dI = G - (u_x k_x + u_y k_y),      du_x = -I k_x,  du_y = -I k_y
//   second order   dI += 1/2 (u_x^2 h_xx + u_x u_y (h_xy + h_yx) + u_y^2 h_yy)
//                  du_x += 1/2 I (2 u_x h_xx + u_y (h_xy + h_yx)),  du_y likewise
//   pressure       dI += -q_s (D_x Q k_x + D_y Q k_y)
//                  dQ = -q_s (D_x^T(I k_x) + D_y^T(I k_y)),  t = dQ / A
//                  dI += (lap^T t - t Q) / (2 A)
// then grad_A += -a_s I dI and G_x += b_s du_x, G_y += b_s du_y (grad_phi = D_x^T G_x + D_y^T G_y
// by k_vjp_transpose).
//
// As in the closure itself, a wave works on a strip of kLocalCols output columns x kVsRows rows
// alone: column neighbours from the adjacent lanes, row neighbours in registers, so the chain of
// derivatives (four deep in t) needs no planes in memory.  The waves of a workgroup share the lines
// of one strip and add their sums through LDS at the end.
// Bound by vector issue.  1024 x 1280, 4 lines, pressure term: 138 us (four passes over per-line
// planes of A, Q and t) -> 28 us.  The registers are held to what three waves per SIMD allow
// (two with ORDER 2), or one wave fewer with a spectrum per column, where that would spill.
// ---------------------------------------------------------------------------------------------
constexpr int kVsRows = 8;
constexpr int kVsWavesMax = 4;

// ORDER 1 or 2 (local closures), or 3 (the pressure term alone, added to the transport's
// gradient already in gA).  EDGE: the strip meets the image border (see local_strip).
template <int ORDER, bool XDEP, bool EDGE>
__device__ __forceinline__ void vjp_strip_line(const ProbDesc& p, int s, int y0, int x, int xc,
                                               const float (&Xv)[kVsRows + 2 * kLocalHalo],
                                               const float (&Gv)[kVsRows + 2 * kLocalHalo],
                                               const float (&px)[kVsRows], const float (&py)[kVsRows],
                                               float (&sa)[kVsRows], float (&sx)[kVsRows],
                                               float (&sy)[kVsRows]) {
  constexpr int H = kLocalHalo, N = kVsRows + 2 * H;
  const int nx = p.nx, ny = p.ny;
  const float4 c = line_wabq<XDEP>(p, xc, s);
  const bool xfirst = x == 0, xlast = x == nx - 1;
  auto dx = [&](float f) {  // D_x
    float l = lane_left(f), r = lane_right(f);
    if constexpr (EDGE) {
      l = xfirst ? f : l;
      r = xlast ? f : r;
      return ((xfirst || xlast) ? 1.f : 0.5f) * (r - l);
    }
    return 0.5f * (r - l);
  };
  auto dy = [&](int i, float fm, float f0, float fp) {  // D_y at input row i
    if constexpr (EDGE) {
      const int y = y0 - H + i;
      const float t = y == 0 ? f0 : fm, b = y == ny - 1 ? f0 : fp;
      return ((y == 0 || y == ny - 1) ? 1.f : 0.5f) * (b - t);
    }
    return 0.5f * (fp - fm);
  };
  auto dxt = [&](float f) {  // D_x^T
    const float l = lane_left(f), r = lane_right(f);
    if constexpr (EDGE) return d_transpose3(l, f, r, x, nx);
    return 0.5f * (l - r);
  };
  auto dyt = [&](int i, float fm, float f0, float fp) {  // D_y^T at input row i
    if constexpr (EDGE) return d_transpose3(fm, f0, fp, y0 - H + i, ny);
    return 0.5f * (fm - fp);
  };
  Root A[N];
  float I[N], dyA[N], Q[N], kx[N], ky[N], vx[N], vy[N], t[N], ut[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    I[i] = c.x * expf(-c.y * Xv[i]);
    kx[i] = dxt(Gv[i]);
    if constexpr (ORDER >= 2) {
      A[i] = root_of(fmaxf(I[i], kRootMin));
      if (i >= 2) dyA[i - 1] = dy(i - 1, A[i - 2].a, A[i - 1].a, A[i].a);
      // XDEP: q_s scales the pressure term after its outer derivative, so the row factor is
      // D_x^T(q_s g) and the column factor q_s(x) D_y^T g
      vx[i] = I[i] * (XDEP ? dxt(c.w * Gv[i]) : kx[i]);
    }
    if (i >= 2) {
      ky[i - 1] = dyt(i - 1, Gv[i - 2], Gv[i - 1], Gv[i]);
      if constexpr (ORDER >= 2) vy[i - 1] = I[i - 1] * ky[i - 1];
    }
    if constexpr (ORDER >= 2) {
      const int j = i - 2;
      if (j >= 2 && j < N - 2) {
        Q[j] = over_root(dx(dx(A[j].a)) + dy(j, dyA[j - 1], dyA[j], dyA[j + 1]), A[j]);
        const float tx = dxt(vx[j]), ty = dyt(j, vy[j - 1], vy[j], vy[j + 1]);
        t[j] = over_root(XDEP ? -fmaf(c.w, ty, tx) : -c.w * (tx + ty), A[j]);
      }
      const int k = i - 3;
      if (k >= 3 && k < N - 3) ut[k] = dyt(k, t[k - 1], t[k], t[k + 1]);
    }
    const int m = i - H;
    if (m >= H && m < N - H) {
      const int o = m - H;
      float dI = 0.f;
      if constexpr (ORDER != kOrderTransportWkb1) {
        const float ux = c.z * px[o], uy = c.z * py[o];
        dI = Gv[m] - (ux * kx[m] + uy * ky[m]);
        float dux = -I[m] * kx[m], duy = -I[m] * ky[m];
        if constexpr (ORDER == 2) {
          const float hxx = dxt(kx[m]), hyy = dyt(m, ky[m - 1], ky[m], ky[m + 1]);
          const float hm = 2.f * dxt(ky[m]);  // h_xy + h_yx (the transposes commute)
          dI += 0.5f * (ux * ux * hxx + ux * uy * hm + uy * uy * hyy);
          dux += 0.5f * I[m] * (2.f * ux * hxx + uy * hm);
          duy += 0.5f * I[m] * (ux * hm + 2.f * uy * hyy);
        }
        sx[o] += c.z * dux;
        sy[o] += c.z * duy;
      }
      if constexpr (ORDER >= 2) {
        const float dqx = dx(Q[m]), dqy = dy(m, Q[m - 1], Q[m], Q[m + 1]);
        if constexpr (XDEP)
          dI += -(dqx * dxt(c.w * Gv[m]) + dqy * (c.w * ky[m]));
        else
          dI += -c.w * (dqx * kx[m] + dqy * ky[m]);
        const float lap = dxt(dxt(t[m])) + dyt(m, ut[m - 1], ut[m], ut[m + 1]);
        dI += 0.5f * over_root(lap - t[m] * Q[m], A[m]);
      }
      sa[o] -= c.y * I[m] * dI;
    }
  }
}

template <int ORDER, bool XDEP, bool EDGE>
__device__ __forceinline__ void vjp_strip(const ProbDesc& p, int w, int nw, int y0, int xs,
                                          float (&sa)[kVsRows], float (&sx)[kVsRows],
                                          float (&sy)[kVsRows]) {
  constexpr int H = kLocalHalo, N = kVsRows + 2 * H;
  const int nx = p.nx, ny = p.ny;
  const int x = xs - H + (int)(threadIdx.x & 63);
  const int xc = EDGE ? min(max(x, 0), nx - 1) : x;
  gptr<const float> X = G(p.X);
  gptr<const float> Y = G(p.Y);
  gptr<const float> g = G(p.d);
  float Xv[N], Gv[N], px[kVsRows] = {}, py[kVsRows] = {};
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int y = y0 - H + i, yc = EDGE ? min(max(y, 0), ny - 1) : y;
    Xv[i] = ldg(X + yc * nx, (unsigned)xc);
    Gv[i] = ldg(g + yc * nx, (unsigned)xc);
  }
  if constexpr (ORDER != kOrderTransportWkb1) {
#pragma unroll
    for (int o = 0; o < kVsRows; ++o) {
      const int yc = min(y0 + o, ny - 1);
      const int xl = max(xc - 1, 0), xh = min(xc + 1, nx - 1);
      const int yl = max(yc - 1, 0), yh = min(yc + 1, ny - 1);
      px[o] = (xh - xl == 2 ? 0.5f : 1.f) * (ldg(Y + yc * nx, (unsigned)xh) - ldg(Y + yc * nx, (unsigned)xl));
      py[o] = (yh - yl == 2 ? 0.5f : 1.f) * (ldg(Y + yh * nx, (unsigned)xc) - ldg(Y + yl * nx, (unsigned)xc));
    }
  }
  for (int s = w; s < p.lp.n; s += nw)
    vjp_strip_line<ORDER, XDEP, EDGE>(p, s, y0, x, xc, Xv, Gv, px, py, sa, sx, sy);
}

template <int ORDER, bool XDEP>
__global__ __launch_bounds__(64 * kVsWavesMax) __attribute__((
    amdgpu_waves_per_eu((ORDER == 1 ? 4 : ORDER == 2 ? 2 : 3) - (XDEP ? 1 : 0)))) void k_vjp_local(
    KArgs a, float* __restrict__ Gx, float* __restrict__ Gy, float* __restrict__ gA) {
  constexpr int NQ = ORDER == kOrderTransportWkb1 ? 1 : 3;  // sums: A alone, or A, G_x, G_y
  __shared__ float red[kVsWavesMax][NQ][kVsRows][64];
  const ProbDesc& p = a.p;
  const int nx = p.nx, ny = p.ny;
  const int local = xcd_remap(blockIdx.x, gridDim.x);
  const int ntx = (nx + kLocalCols - 1) / kLocalCols;
  const int y0 = (local / ntx) * kVsRows, xs = (local % ntx) * kLocalCols;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6;
  float sa[kVsRows] = {}, sx[kVsRows] = {}, sy[kVsRows] = {};
  const bool inner = xs >= kLocalHalo + 1 && xs + kLocalCols + kLocalHalo + 1 <= nx &&
                     y0 >= kLocalHalo + 1 && y0 + kVsRows + kLocalHalo + 1 <= ny;
  if (inner)
    vjp_strip<ORDER, XDEP, false>(p, w, nw, y0, xs, sa, sx, sy);
  else
    vjp_strip<ORDER, XDEP, true>(p, w, nw, y0, xs, sa, sx, sy);
#pragma unroll
  for (int o = 0; o < kVsRows; ++o) {
    red[w][0][o][lane] = sa[o];
    if constexpr (NQ == 3) {
      red[w][1][o][lane] = sx[o];
      red[w][2][o][lane] = sy[o];
    }
  }
  __syncthreads();
  const int x = xs - kLocalHalo + lane;
  if (lane < kLocalHalo || lane >= kLocalHalo + kLocalCols || x >= nx) return;
  for (int o = w; o < kVsRows; o += nw) {
    const int y = y0 + o;
    if (y >= ny) break;
    float v[NQ] = {};
    for (int k = 0; k < nw; ++k)
#pragma unroll
      for (int q = 0; q < NQ; ++q) v[q] += red[k][q][o][lane];
    const unsigned i = (unsigned)(__mul24(y, nx) + x);
    if constexpr (NQ == 1) {
      stg(G(gA), i, ldg(G((const float*)gA), i) + v[0]);
    } else {
      stg(G(gA), i, v[0]);
      stg(G(Gx), i, v[1]);
      stg(G(Gy), i, v[2]);
    }
  }
}

template <bool XDEP>
hipError_t launch_vjp_local_t(const KArgs& a, hipStream_t s, int order, float* gx, float* gy,
                              float* ga) {
  const dim3 grid(((a.p.ny + kVsRows - 1) / kVsRows) * ((a.p.nx + kLocalCols - 1) / kLocalCols));
  const dim3 block(64 * (a.p.lp.n < kVsWavesMax ? a.p.lp.n : kVsWavesMax));
  if (order == 1)
    hipLaunchKernelGGL((k_vjp_local<1, XDEP>), grid, block, 0, s, a, gx, gy, ga);
  else if (order == 2)
    hipLaunchKernelGGL((k_vjp_local<2, XDEP>), grid, block, 0, s, a, gx, gy, ga);
  else
    hipLaunchKernelGGL((k_vjp_local<3, XDEP>), grid, block, 0, s, a, gx, gy, ga);
  return hipGetLastError();
}

hipError_t launch_vjp_local(const KArgs& a, hipStream_t s, int order, float* gx, float* gy,
                            float* ga) {
  return a.p.xcol ? launch_vjp_local_t<true>(a, s, order, gx, gy, ga)
                  : launch_vjp_local_t<false>(a, s, order, gx, gy, ga);
}

hipError_t launch_vjp(const KArgs& a, hipStream_t s, float* gphi, float* ga, int accumulate) {
  const dim3 grid(((a.p.ny + kVjpTY - 1) / kVjpTY) * ((a.p.nx + kVjpTX - 1) / kVjpTX));
  const dim3 block(64 * kVjpWaves);
  if (a.p.xcol)
    hipLaunchKernelGGL(k_vjp<true>, grid, block, 0, s, a, gphi, ga, accumulate);
  else
    hipLaunchKernelGGL(k_vjp<false>, grid, block, 0, s, a, gphi, ga, accumulate);
  return hipGetLastError();
}

hipError_t launch_vjp_transpose(const KArgs& a, hipStream_t s, const float* gx, const float* gy,
                                float* gphase, int accumulate) {
  const int nb = (a.p.nx * a.p.ny + kTrThreads - 1) / kTrThreads;
  hipLaunchKernelGGL(k_vjp_transpose, dim3(nb), dim3(kTrThreads), 0, s, a, gx, gy, gphase,
                     accumulate);
  return hipGetLastError();
}

}  // namespace epr
