// Non-local transport kernels (Methods 4.2): max-shift reduction, the transpose of the detector
// binning, the residual-norm reduction, and the launches of the splat (k_splat.h).
#include <hip/hip_runtime.h>

#include "dev_common.h"
#include "epr_internal.h"
#include "k_splat.h"

namespace epr {

// ---------------------------------------------------------------------------------------------
// max |D_x Y|, max |D_y Y| and min X over the image, one partial triple per workgroup (a band of
// rows), and the largest positive and negative parts of both differences on every segment of
// kSegCols columns of the band (p.segs): from the former the splat bounds how far away a
// tile's sources can lie, from the latter how far those it can actually meet are displaced.
// ---------------------------------------------------------------------------------------------
constexpr int kMaxgThreads = 1024;  // (a band is a few rows: many loads in flight per workgroup)

__device__ __forceinline__ void maxgrad_body(const ProbDesc& p, int local, int) {
  const int nx = p.nx, ny = p.ny;
  gptr<const float> Y = G(p.Y);
  gptr<const float> X = G(p.X);
  const int nseg = seg_cols(nx);
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int kWaves = kMaxgThreads / 64;
  // {max D_x Y, max -D_x Y, max D_y Y, max -D_y Y}, at least 0, per segment, as float bits (whose
  // order is that of the values for non-negative floats); NaNs drop out of the maxima
  __shared__ unsigned seg[kMaxDim / kSegCols * 4];
  __shared__ float red[kWaves];
  for (int i = tid; i < nseg * 4; i += kMaxgThreads) seg[i] = 0u;
  __syncthreads();
  float mn = INFINITY;
  // each workgroup takes one band of whole rows, so that the rows above and below a pixel are
  // read by the same workgroup (from its caches) rather than fetched again by others
  const int y0 = (int)(((long long)local * ny) / kMaxgBlocks);
  const int y1 = (int)(((long long)(local + 1) * ny) / kMaxgBlocks);
  // the lanes of an aligned group of 8 (four pixels each) or 16 (one each) lie in one segment
  auto deposit = [&](int x, int group, float xp, float xm, float yp, float ym) {
    if (group == 8) {
      xp = lane8_max(xp);
      xm = lane8_max(xm);
      yp = lane8_max(yp);
      ym = lane8_max(ym);
    } else {
      xp = lane16_max(xp);
      xm = lane16_max(xm);
      yp = lane16_max(yp);
      ym = lane16_max(ym);
    }
    if ((lane & (group - 1)) == 0 && x < nx) {
      unsigned* s = seg + (x / kSegCols) * 4;
      atomicMax(s, __float_as_uint(xp));
      atomicMax(s + 1, __float_as_uint(xm));
      atomicMax(s + 2, __float_as_uint(yp));
      atomicMax(s + 3, __float_as_uint(ym));
    }
  };
  if ((nx & 3) == 0 && ((reinterpret_cast<uintptr_t>(p.Y) | reinterpret_cast<uintptr_t>(p.X)) & 15) == 0) {
    // 4 consecutive pixels per lane: three float4 loads (rows y-1, y, y+1) and the two
    // neighbours of the segment; clamping reproduces the one-sided edge differences.  A wave
    // takes 256 columns of every (kWaves / nc)-th row of the band and reduces over lanes once.
    const int nc = (nx + 255) >> 8;
    static_assert((kMaxDim + 255) / 256 <= kWaves, "a column block per wave");
    const int ng = kWaves / nc, g = w / nc;
    const int x = ((w - g * nc) << 8) + 4 * lane;
    float xp = 0.f, xm = 0.f, yp = 0.f, ym = 0.f;
    if (g < ng && x < nx) {
#pragma unroll 2
      for (int y = y0 + g; y < y1; y += ng) {
        const int yl = max(y - 1, 0), yh = min(y + 1, ny - 1);
        const float sy = (yh - yl == 2) ? 0.5f : 1.f;
        const float4 c = ldg((gptr<const float4>)Y, (unsigned)(__mul24(y, nx) + x) >> 2);
        const float4 u = ldg((gptr<const float4>)Y, (unsigned)(__mul24(yl, nx) + x) >> 2);
        const float4 d = ldg((gptr<const float4>)Y, (unsigned)(__mul24(yh, nx) + x) >> 2);
        const float4 xv = ldg((gptr<const float4>)X, (unsigned)(__mul24(y, nx) + x) >> 2);
        const float l = ldg(Y, (unsigned)(__mul24(y, nx) + max(x - 1, 0)));
        const float r = ldg(Y, (unsigned)(__mul24(y, nx) + min(x + 4, nx - 1)));
        // x differences: the first/last pixel of the row use one-sided differences
        const float g0 = (x == 0) ? c.y - c.x : 0.5f * (c.y - l);
        const float g1 = 0.5f * (c.z - c.x);
        const float g2 = 0.5f * (c.w - c.y);
        const float g3 = (x + 4 == nx) ? c.w - c.z : 0.5f * (r - c.z);
        const float h0 = sy * (d.x - u.x), h1 = sy * (d.y - u.y);
        const float h2 = sy * (d.z - u.z), h3 = sy * (d.w - u.w);
        xp = fmaxf(xp, fmaxf(fmaxf(g0, g1), fmaxf(g2, g3)));
        xm = fmaxf(xm, fmaxf(fmaxf(-g0, -g1), fmaxf(-g2, -g3)));
        yp = fmaxf(yp, fmaxf(fmaxf(h0, h1), fmaxf(h2, h3)));
        ym = fmaxf(ym, fmaxf(fmaxf(-h0, -h1), fmaxf(-h2, -h3)));
        mn = fminf(mn, fminf(fminf(xv.x, xv.y), fminf(xv.z, xv.w)));
      }
    }
    if (g < ng) deposit(x, 8, xp, xm, yp, ym);
  } else {
    const int nc = (nx + 63) >> 6;
    for (int t = w; t < nc * (y1 - y0); t += kWaves) {
      const int yb = t / nc;
      const int y = y0 + yb, x = ((t - yb * nc) << 6) + lane;
      float gx = 0.f, gy = 0.f;
      if (x < nx) {
        gx = d_x(Y, y, x, nx);
        gy = d_y(Y, y, x, ny, nx);
        mn = fminf(mn, ldg(X, (unsigned)(__mul24(y, nx) + x)));
      }
      deposit(x, 16, fmaxf(gx, 0.f), fmaxf(-gx, 0.f), fmaxf(gy, 0.f), fmaxf(-gy, 0.f));
    }
  }
  mn = -wave_max(-mn);
  if (lane == 0) red[w] = mn;
  __syncthreads();
  if (w == 0) {
    float a = 0.f, b = 0.f, c = lane < kWaves ? red[lane] : INFINITY;
    for (int i = lane; i < nseg; i += 64) {
      float4 s;
      s.x = __uint_as_float(seg[4 * i]);
      s.y = __uint_as_float(seg[4 * i + 1]);
      s.z = __uint_as_float(seg[4 * i + 2]);
      s.w = __uint_as_float(seg[4 * i + 3]);
      a = fmaxf(a, fmaxf(s.x, s.y));
      b = fmaxf(b, fmaxf(s.z, s.w));
      if (y1 > y0) stg(G(p.segs), (unsigned)(seg_band(y0, ny) * nseg + i), s);
    }
    a = wave_max(a);
    b = wave_max(b);
    c = -wave_max(-c);
    if (lane == 0) {
      gptr<float> mg = G(p.maxg);
      mg[3 * local] = a;
      mg[3 * local + 1] = b;
      mg[3 * local + 2] = c;
    }
  }
}

template <bool B>
__global__ __launch_bounds__(kMaxgThreads) void k_maxgrad(KArgs a, const ProbDesc* __restrict__ table) {
  EPR_DISPATCH(B, a, table, blockIdx.x, maxgrad_body, 0);
}

// Transpose of the detector binning for every line: the detector values r[s] copied to their
// f x f internal pixels, divided by f^2 (one internal pixel per thread).
__global__ __launch_bounds__(256) void k_unbin_lines(const float* __restrict__ r,
                                                     float* __restrict__ out, int ny, int nx,
                                                     int f, int lines) {
  const int n = ny * nx;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n * lines) return;
  const int s = i / n, j = i - s * n;
  const int y = j / nx, x = j - y * nx;
  const int nxd = nx / f;
  const float inv = 1.f / (float)(f * f);
  out[i] = inv * r[(size_t)s * (n / (f * f)) + (size_t)(y / f) * nxd + x / f];
}

hipError_t launch_unbin_lines(const float* r, float* out, int ny, int nx, int f, int lines,
                              hipStream_t s) {
  const long long total = (long long)ny * nx * lines;
  hipLaunchKernelGGL(k_unbin_lines, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, r, out,
                     ny, nx, f, lines);
  return hipGetLastError();
}

// Reduce the nb residual partials of the problem into hist_slot = ||e|| / ||d||.
__global__ __launch_bounds__(256) void k_resid_reduce(KArgs a, float* hist_slot, int nb) {
  const float* __restrict__ resid = a.p.resid;
  float te = 0.f, td = 0.f;
  for (int i = threadIdx.x; i < nb; i += 256) {
    te += resid[2 * i];
    td += resid[2 * i + 1];
  }
  __shared__ float red[2][4];
  te = wave_sum(te);
  td = wave_sum(td);
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = te;
    red[1][threadIdx.x >> 6] = td;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    te = red[0][0] + red[0][1] + red[0][2] + red[0][3];
    td = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    hist_slot[0] = td > 0.f ? sqrtf(te / td) : 0.f;
  }
}

hipError_t launch_maxgrad(const KArgs& a, int total_blocks, hipStream_t s) {
  if (a.table)
    hipLaunchKernelGGL(k_maxgrad<true>, dim3(total_blocks), dim3(kMaxgThreads), 0, s, a, a.table);
  else
    hipLaunchKernelGGL(k_maxgrad<false>, dim3(total_blocks), dim3(kMaxgThreads), 0, s, a, a.table);
  return hipGetLastError();
}

EPR_SPLAT_LINES(EPR_SPLAT_DECLARE)

// `lines` is the line count of every problem in the launch.
hipError_t launch_splat(const KArgs& a, int total_blocks, size_t lds, hipStream_t s, int lines) {
  switch (lines) {
#define EPR_SPLAT_CASE(N) \
  case N: launch_splat_nl<N>(a, total_blocks, lds, s); break;
    EPR_SPLAT_LINES(EPR_SPLAT_CASE)
#undef EPR_SPLAT_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_resid_reduce(const KArgs& a, float* hist_slot, int nb, hipStream_t s) {
  hipLaunchKernelGGL(k_resid_reduce, dim3(1), dim3(256), 0, s, a, hist_slot, nb);
  return hipGetLastError();
}

hipError_t set_transport_attributes() {
  hipError_t e = hipSuccess;
#define EPR_SPLAT_SET(N) \
  if (e == hipSuccess) e = set_splat_attributes_nl<N>();
  EPR_SPLAT_LINES(EPR_SPLAT_SET)
#undef EPR_SPLAT_SET
  return e;
}

}  // namespace epr
