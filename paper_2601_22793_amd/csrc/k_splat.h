// Splat kernels (Methods 4.2): the LDS-tiled conservative bilinear splat with the fused spectral
// sum, residual and split (Eq. 5, Methods 4.4), one instance per line count.
// The instances are compiled in units of about the same size (k_splat_<unit>.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "dev_common.h"
#include "epr_internal.h"
#include "split_bin.h"

namespace epr {

// Every line count has an instance: its constants sit in registers, and no line is tested for in the
// loops.  A count that runs a larger instance pays for the spare lines' registers and tests: 2048 x
// 2048, 64 x 32 tile, us a launch, 9 lines 133 and 12 lines 165 in the instance for 16 (79 and 131 in
// their own).  Instances for even counts alone, with a test for the last line, cost odd counts 3 %
// and slowed a whole solve with 8 lines by 1 %.  (The sixteen take 12 MB of library, eight 8 MB.)
#define EPR_SPLAT_LINES(M) \
  M(1) M(2) M(3) M(4) M(5) M(6) M(7) M(8) M(9) M(10) M(11) M(12) M(13) M(14) M(15) M(16)

// ---------------------------------------------------------------------------------------------
// Splat.  A workgroup owns a TY x TX tile of the detector and accumulates, for every line, the
// bilinear deposits of all sources whose mapped footprint can reach the tile (sources within
// the halo derived on the device from the max-gradient partials and segments) in LDS with LDS atomics.
// Each detector pixel is written by exactly one workgroup: no global atomics.
//   forward mode: out = sum_s P_s
//   split mode  : e = d - sum_s P_s, e_s = pi_s e with pi_s = max(P_s,0)/sum max(P_s',0)
//                 (w_s where that sum is zero), written to e[s]; optional residual partials.
//   bin mode    : the same on an oversampled internal grid (split_bin): P_s is the mean over the
//                 f x f internal pixels of a detector pixel, e_s goes to all of them.
// NL is the line count, at compile time so that the per-line constants sit in registers
// for the whole source loop: a scalar load inside the loop would make every iteration wait
// for all outstanding LDS atomics (they share one counter).
// ---------------------------------------------------------------------------------------------
// Stencil of D Y at a source (y, x) and X there, as loaded: the gradient is formed where the
// sample is used, so the loads of the next source stay in flight meanwhile.  Clamped
// neighbours make the differences one-sided on the edges (same values as d_x / d_y).
struct SourceSample {
  float xr, xl, yr, yl, xv;
};

__device__ __forceinline__ SourceSample load_source(gptr<const float> X, gptr<const float> Y,
                                                    int y, int x, int ny, int nx) {
  const int xl = max(x - 1, 0), xr = min(x + 1, nx - 1);
  const int yl = max(y - 1, 0), yr = min(y + 1, ny - 1);
  const int row = __mul24(y, nx);
  SourceSample s;
  s.xr = ldg(Y, (unsigned)(row + xr));
  s.xl = ldg(Y, (unsigned)(row + xl));
  s.yr = ldg(Y, (unsigned)(__mul24(yr, nx) + x));
  s.yl = ldg(Y, (unsigned)(__mul24(yl, nx) + x));
  s.xv = ldg(X, (unsigned)(row + x));
  return s;
}

// The same samples for a source at least one pixel inside every edge: one offset per lane, the
// neighbours at fixed distances from it (central differences everywhere).
__device__ __forceinline__ SourceSample load_source_inner(gptr<const float> X, gptr<const float> Y,
                                                          int y, int x, int nx) {
  const unsigned o = (unsigned)(__mul24(y, nx) + x);
  SourceSample s;
  s.xr = ldg(Y, o + 1);
  s.xl = ldg(Y, o - 1);
  s.yr = ldg(Y + nx, o);
  s.yl = ldg(Y, o - (unsigned)nx);
  s.xv = ldg(X, o);
  return s;
}

// a * b + c with a 24-bit signed multiply (full rate; b wave-uniform).  Written as the
// instruction itself: the optimiser would otherwise widen an index multiply whose operand range
// it has narrowed (from a bounds test) into a quarter-rate 32-bit multiply.
__device__ __forceinline__ int mad24(int a, int b, int c) {
  int d;
  asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(d) : "v"(a), "s"(b), "v"(c));
  return d;
}

// Largest footprint window (pixels) accumulated in fixed point; wider windows fall back to
// LDS float atomics.
constexpr float kFixedWindowMax = 4096.f;

// XDEP: x-dependent spectrum, the line constants of every source and target come from its
// column (lp.w, lp.a and lp.a_hi then bound them over the columns).
template <int NL, bool XDEP>
__device__ __forceinline__ void splat_body(const ProbDesc& p, int local, int mode) {
  // Per line, accumulators for the tile plus a one-pixel border (TY+2) x (TX+2), origin
  // (ty0-1, tx0-1): a source whose 2x2 footprint touches the tile deposits all four weights
  // without per-corner bounds checks; the border is discarded.
  extern __shared__ unsigned int acc_u[];
  float* acc_f = reinterpret_cast<float*>(acc_u);
  // the reductions of the prologue and of the residual, in turn: no more than that, so that every
  // tile whose accumulators fit kSplatLdsMax launches
  __shared__ __attribute__((aligned(16))) float scratch[kSplatScratch];
  const int nx = p.nx, ny = p.ny;
  const int TX = p.splat_tx, TY = p.splat_ty;
  const int ptile = (TX + 2) * (TY + 2);
  constexpr int L = NL;
  const int ntx = (nx + TX - 1) / TX;
  const int ty0 = (local / ntx) * TY;
  const int tx0 = (local - (local / ntx) * ntx) * TX;
  const int tid = threadIdx.x;

  float lw[NL], la2[NL], lb[NL];
#pragma unroll
  for (int s = 0; s < NL; ++s) {
    lw[s] = p.lp.w[s];
    la2[s] = p.lp.a[s] * 1.4426950408889634f;  // exp(-a x) = exp2(-a log2(e) x)
    lb[s] = p.lp.b[s];
  }

  // Halo of the tile and minimum of X.  The segment maxima around the tile (kGuessX columns and
  // kGuessY rows away) bound the shifts of the sources there, by sign; the
  // partials' maximum bounds every shift of the image.  When the latter keeps all sources that
  // reach the tile within the former's surroundings, the former gives the tile's halo: a tile
  // away from the steepest edges reads few sources that it does not need.  The first three waves
  // read the segments and the fourth the partials, with one barrier.
  // 2048 x 2048, 8 lines, shifts up to 6 pixels: splat 84 -> 66 us a launch (73 us of it by the
  // halo and this prologue, the rest by reading the detector data before the source loop);
  // max-gradient 7.5 -> 8.3 us for the signed segment maxima.
  constexpr int kGuessX = kSegCols, kGuessY = kSplatTileY / 2;
  constexpr int kScanWaves = 3, kScanMax = 256;
  static_assert(kMaxgBlocks == 4 * 64, "four partials (three float4) a lane");
  static_assert(4 * kScanWaves + 3 <= kSplatScratch && 4 * 4 <= kSplatScratch &&
                2 * (kSplatThreads / 64) <= kSplatScratch, "scratch");
  float4* const red4 = reinterpret_cast<float4*>(scratch);
  const int nseg = seg_cols(nx);
  gptr<const float4> segs = G((const float4*)p.segs);
  const int gs0 = max(tx0 - kGuessX, 0) / kSegCols;
  const int gns = min(tx0 + TX - 1 + kGuessX, nx - 1) / kSegCols - gs0 + 1;
  const int gb0 = seg_band(max(ty0 - kGuessY, 0), ny);
  const int gn = gns * (seg_band(min(ty0 + TY - 1 + kGuessY, ny - 1), ny) - gb0 + 1);
  if (tid < kScanWaves * 64) {
    float4 m = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int k = 0; k * kScanWaves * 64 < kScanMax; ++k) {
      const int i = tid + k * kScanWaves * 64;
      if (i < min(gn, kScanMax)) {
        const float4 v = ldg(segs, (unsigned)((gb0 + i / gns) * nseg + gs0 + i % gns));
        m = make_float4(fmaxf(m.x, v.x), fmaxf(m.y, v.y), fmaxf(m.z, v.z), fmaxf(m.w, v.w));
      }
    }
    m = make_float4(lane64_max(m.x), lane64_max(m.y), lane64_max(m.z), lane64_max(m.w));
    if ((tid & 63) == 0) red4[tid >> 6] = m;
  } else if (tid < (kScanWaves + 1) * 64) {
    // partials {x, y, min} of four bands: a.x a.y a.z, a.w b.x b.y, b.z b.w c.x, c.y c.z c.w
    gptr<const float4> mg = (gptr<const float4>)G(p.maxg);
    const unsigned i = 3u * (unsigned)(tid & 63);
    const float4 a = ldg(mg, i), b = ldg(mg, i + 1), c = ldg(mg, i + 2);
    const float gx = lane64_max(fmaxf(fmaxf(a.x, a.w), fmaxf(b.z, c.y)));
    const float gy = lane64_max(fmaxf(fmaxf(a.y, b.x), fmaxf(b.w, c.z)));
    const float xm = -lane64_max(-fminf(fminf(a.z, b.y), fminf(c.x, c.w)));
    if ((tid & 63) == 0) {
      scratch[4 * kScanWaves] = gx;
      scratch[4 * kScanWaves + 1] = gy;
      scratch[4 * kScanWaves + 2] = xm;
    }
  }
  {
    // clear the accumulators, 16 bytes at a time
    const int n = L * ptile;
    uint4* a4 = reinterpret_cast<uint4*>(acc_u);
    for (int i = tid; i < (n >> 2); i += kSplatThreads) a4[i] = make_uint4(0u, 0u, 0u, 0u);
    if (tid < (n & 3)) acc_u[(n & ~3) + tid] = 0u;
  }
  __syncthreads();
  float4 sm = red4[0];
#pragma unroll
  for (int w = 1; w < kScanWaves; ++w) {
    const float4 a = red4[w];
    sm = make_float4(fmaxf(sm.x, a.x), fmaxf(sm.y, a.y), fmaxf(sm.z, a.z), fmaxf(sm.w, a.w));
  }
  const float gmx = scratch[4 * kScanWaves], gmy = scratch[4 * kScanWaves + 1];
  const float xmin = scratch[4 * kScanWaves + 2];
  const int hx = halo_from(p.lp.b_absmax, gmx);
  const int hy = halo_from(p.lp.b_absmax, gmy);
  if (hx > kGuessX || hy > kGuessY || gn > kScanMax) {
    // sources from further away (or too many entries above): the segments the image's halo spans
    const int s0 = max(tx0 - hx, 0) / kSegCols, s1 = min(tx0 + TX - 1 + hx, nx - 1) / kSegCols;
    const int b0 = seg_band(max(ty0 - hy, 0), ny), b1 = seg_band(min(ty0 + TY - 1 + hy, ny - 1), ny);
    const int ns = s1 - s0 + 1;
    constexpr int kFarWaves = 4;
    __syncthreads();  // every wave has read the scratch
    if (tid < kFarWaves * 64) {
      float4 m = make_float4(0.f, 0.f, 0.f, 0.f);
      for (int i = tid; i < ns * (b1 - b0 + 1); i += kFarWaves * 64) {
        const float4 v = ldg(segs, (unsigned)((b0 + i / ns) * nseg + s0 + i % ns));
        m = make_float4(fmaxf(m.x, v.x), fmaxf(m.y, v.y), fmaxf(m.z, v.z), fmaxf(m.w, v.w));
      }
      m = make_float4(lane64_max(m.x), lane64_max(m.y), lane64_max(m.z), lane64_max(m.w));
      if ((tid & 63) == 0) red4[tid >> 6] = m;
    }
    __syncthreads();
    sm = red4[0];
#pragma unroll
    for (int w = 1; w < kFarWaves; ++w) {
      const float4 a = red4[w];
      sm = make_float4(fmaxf(sm.x, a.x), fmaxf(sm.y, a.y), fmaxf(sm.z, a.z), fmaxf(sm.w, a.w));
    }
  }
  // Sources to the left (above) reach the tile with positive shifts, to the right (below) with
  // negative ones; one pixel of halo each way at least (halo_from).  The shifts are b_s D Y with
  // every b_s of one sign: positive for a phase map, negative for a thickness.
  bool bneg = XDEP;
#pragma unroll
  for (int s = 0; s < NL; ++s) bneg = bneg || lb[s] < 0.f;
  const int hxl = halo_from(p.lp.b_absmax, bneg ? sm.y : sm.x);
  const int hxr = halo_from(p.lp.b_absmax, bneg ? sm.x : sm.y);
  const int hyt = halo_from(p.lp.b_absmax, bneg ? sm.w : sm.z);
  const int hyb = halo_from(p.lp.b_absmax, bneg ? sm.z : sm.w);

  // Fixed-point accumulation (integer LDS atomics: several times the throughput of float
  // atomics, and order-independent).  Every source deposits at most its intensity, which is at
  // most w_s exp(-a_s min X), into one pixel, and at most (hxl+hxr+2)(hyt+hyb+2) sources reach it,
  // so with scale_s = 4.29e9 / (w_s exp(-a_s min X) window) no sum exceeds 4.29e9, and with up to
  // one unit more per deposit (rounding) none reaches 2^32.
  const float window = (float)(hxl + hxr + 2) * (float)(hyt + hyb + 2);
  float scale[NL], inv_scale[NL];
  bool fixed = window <= kFixedWindowMax;
#pragma unroll
  for (int s = 0; s < NL; ++s) {
    // (x-dependent: the largest w_s with the a_s bound that maximises exp(-a_s min X))
    const float la2b = (XDEP && xmin < 0.f) ? p.lp.a_hi[s] * 1.4426950408889634f : la2[s];
    const float imax = lw[s] * __builtin_amdgcn_exp2f(-la2b * xmin);
    scale[s] = 4.29e9f / (imax * window);
    inv_scale[s] = 1.f / scale[s];
    if (!(scale[s] > 0.f && scale[s] < 3.0e38f && inv_scale[s] > 0.f)) fixed = false;
  }
  // deposits are formed directly in accumulator units: w_s scale_s (fixed point) or w_s
  float lws[NL];
#pragma unroll
  for (int s = 0; s < NL; ++s) lws[s] = fixed ? lw[s] * scale[s] : lw[s];

  const int sy0 = max(ty0 - hyt, 0), sy1 = min(ty0 + TY - 1 + hyb, ny - 1);
  const int sx0 = max(tx0 - hxl, 0), sx1 = min(tx0 + TX - 1 + hxr, nx - 1);
  const int wsrc = sx1 - sx0 + 1;
  const int nsrc = wsrc * (sy1 - sy0 + 1);
  gptr<const float> X = G(p.X);
  gptr<const float> Y = G(p.Y);

  // The source loop and the read-back, specialised for the common case (fixed-point accumulation,
  // the default or the small tile).
  float se = 0.f, sd = 0.f;
  auto tile = [&](auto full_x, auto full_y, auto inner) {
    constexpr int FX = decltype(full_x)::value, FY = decltype(full_y)::value;
    constexpr bool FULL = FX > 0;
    // INNER: every source of the tile lies at least one pixel inside the image
    constexpr bool INNER = decltype(inner)::value;
    // the full specialisations' tile sizes are compile-time constants, so a footprint's second
    // row and each line's accumulator are immediate offsets
    const int TXk = FULL ? FX : TX, TYk = FULL ? FY : TY;
    // their detector data, read before the source loop that hides the latency
    constexpr int kPre = FULL ? FX * FY / kSplatThreads : 1;
    float dpre[kPre];
    if constexpr (FULL) {
      static_assert(kPre * kSplatThreads == FX * FY, "whole pixels per thread");
      if (mode == kSplatSplit) {
#pragma unroll
        for (int k = 0; k < kPre; ++k) {
          const int i = tid + k * kSplatThreads;
          const int y = min(ty0 + i / FX, ny - 1), x = min(tx0 + i % FX, nx - 1);
          dpre[k] = ldg(G((const float*)p.d), (unsigned)(__mul24(y, nx) + x));
        }
      }
    }
    const int PXk = TXk + 2, ptk = (TXk + 2) * (TYk + 2);
    const int pxm = __builtin_amdgcn_readfirstlane(PXk);  // row stride, a scalar operand
    const int plane = nx * ny;  // line stride of e (every offset below 2^31: L nx ny <= 16 * 4096^2)
    // source index i = r * wsrc + c, advanced incrementally (no division in the loop)
    const int step_r = kSplatThreads / wsrc, step_c = kSplatThreads - step_r * wsrc;
    int r = tid / wsrc, c = tid - r * wsrc;
    SourceSample cur;
    if (tid < nsrc)
      cur = INNER ? load_source_inner(X, Y, sy0 + r, sx0 + c, nx)
                  : load_source(X, Y, sy0 + r, sx0 + c, ny, nx);
    for (int i = tid; i < nsrc; i += kSplatThreads) {
      // The loads of `cur` were issued one iteration ago: wait for them here, before the next
      // source's loads are issued (the vector-memory counter is in order, so a wait placed at
      // the first use of `cur` would also wait for the next source's loads).  LDS atomics are
      // not waited for.
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0) expcnt(7) lgkmcnt(15)
      __builtin_amdgcn_sched_barrier(0);
      const int sy = sy0 + r, sx = sx0 + c;
      // footprint corner for a zero shift, relative to the bordered tile origin (ty0-1, tx0-1)
      const int rx = sx - tx0 + 1, ry = sy - ty0 + 1;
      const float dgx = cur.xr - cur.xl, dgy = cur.yr - cur.yl;
      // central differences inside, one-sided on the edges; INNER: central everywhere, with the
      // halving folded into the line constant ((b / 2) g == b (g / 2) exactly)
      float cgx = dgx, cgy = dgy;
      if constexpr (!INNER) {
        if (sx > 0 && sx < nx - 1) cgx = 0.5f * dgx;
        if (sy > 0 && sy < ny - 1) cgy = 0.5f * dgy;
      }
      r += step_r;
      c += step_c;
      if (c >= wsrc) {
        c -= wsrc;
        ++r;
      }
      SourceSample nxt;
      if (i + kSplatThreads < nsrc)
        nxt = INNER ? load_source_inner(X, Y, sy0 + r, sx0 + c, nx)
                    : load_source(X, Y, sy0 + r, sx0 + c, ny, nx);
#pragma unroll
      for (int s = 0; s < NL; ++s) {
        float sb = INNER ? 0.5f * lb[s] : lb[s], sw = lws[s], sa2 = la2[s];
        if constexpr (XDEP) {
          const float4 c = xcol_at(p, sx, s);
          sb = INNER ? 0.5f * c.z : c.z;
          sw = (FULL || fixed) ? c.x * scale[s] : c.x;
          sa2 = c.y * 1.4426950408889634f;
        }
        const float ux = sb * cgx, uy = sb * cgy;
        const int lx = rx + floor_to_int(ux), ly = ry + floor_to_int(uy);
        if ((unsigned)lx <= (unsigned)TXk && (unsigned)ly <= (unsigned)TYk) {
          // hardware exp2 (v_exp_f32, about one ulp for the normal results met here)
          const float I = sw * __builtin_amdgcn_exp2f(-sa2 * cur.xv);
          // fractional parts x - floor(x) in one instruction each (v_fract_f32, which keeps
          // them below 1 where the subtraction would round up to 1)
          const float dx = __builtin_amdgcn_fractf(ux), dy = __builtin_amdgcn_fractf(uy);
          const int o = s * ptk + mad24(ly, pxm, lx);
          // bilinear weights, all >= 0: w10 + w00 = i0, w11 + w01 = i1, i0 + i1 = I
          const float i1 = I * dy, i0 = I - i1;
          if (FULL || fixed) {
            // nearest accumulator unit (the weights are non-negative): w + 1/2 is formed
            // directly, h10 = i0 dx + 1/2 and h00 = (i0 + 1) - h10 = i0 (1 - dx) + 1/2, then
            // truncated
            const float h10 = fmaf(i0, dx, 0.5f), h00 = (i0 + 1.f) - h10;
            const float h11 = fmaf(i1, dx, 0.5f), h01 = (i1 + 1.f) - h11;
            atomicAdd(&acc_u[o], (unsigned)h00);
            atomicAdd(&acc_u[o + 1], (unsigned)h10);
            atomicAdd(&acc_u[o + PXk], (unsigned)h01);
            atomicAdd(&acc_u[o + PXk + 1], (unsigned)h11);
          } else {
            const float w10 = i0 * dx, w00 = i0 - w10, w11 = i1 * dx, w01 = i1 - w11;
            atomicAdd(&acc_f[o], w00);
            atomicAdd(&acc_f[o + 1], w10);
            atomicAdd(&acc_f[o + PXk], w01);
            atomicAdd(&acc_f[o + PXk + 1], w11);
          }
        }
      }
      cur = nxt;
    }
    __syncthreads();

    auto read_back = [&](int i, float dq) {
      const int ly = i / TXk, lx = i - ly * TXk;
      const int y = ty0 + ly, x = tx0 + lx;
      if (y >= ny || x >= nx) return;
      const unsigned pix = (unsigned)(__mul24(y, nx) + x);
      const int o = (ly + 1) * PXk + lx + 1;
      float Pv[NL];
      float P = 0.f, S = 0.f;
#pragma unroll
      for (int s = 0; s < NL; ++s) {
        Pv[s] = 0.f;
        Pv[s] = (FULL || fixed) ? (float)acc_u[s * ptk + o] * inv_scale[s] : acc_f[s * ptk + o];
        P += Pv[s];
        if (!FULL) S += fmaxf(Pv[s], 0.f);
      }
      // fixed-point sums are never negative: the positive parts are the predictions themselves
      if (FULL) S = P;
      if (mode == kSplatForward) {
        stg(G(p.out), pix, P);
      } else if (mode == kSplatLines) {
#pragma unroll
        for (int s = 0; s < NL; ++s)
          stg(G(p.e), (unsigned)(s * plane) + pix, Pv[s]);
      } else {
        const float dv = FULL ? dq : ldg(G((const float*)p.d), pix);
        const float e = dv - P;
        se += e * e;
        sd += dv * dv;
        const bool hole = !(S > 1e-30f);
        const float inv = hole ? 0.f : 1.f / S;
#pragma unroll
        for (int s = 0; s < NL; ++s) {
          float fw = lw[s];
          if constexpr (XDEP) fw = xcol_at(p, x, s).x;
          const float share = hole ? fw : (FULL ? Pv[s] : fmaxf(Pv[s], 0.f)) * inv;
          stg(G(p.e), (unsigned)(s * plane) + pix, share * e);
        }
      }
    };
    if (mode == kSplatBin) {
      // (tiles are whole detector pixels: bin_tile)
      auto line_at = [&](int o, int s) {
        return (FULL || fixed) ? (float)acc_u[s * ptk + o] * inv_scale[s] : acc_f[s * ptk + o];
      };
      auto bin = [&](auto factor) {
        constexpr int F = decltype(factor)::value;
        const int tw = TXk / F;
        for (int i = tid; i < tw * (TYk / F); i += kSplatThreads) {
          const int ly = i / tw * F, lx = (i - i / tw * tw) * F;
          const int y = ty0 + ly, x = tx0 + lx;
          if (y < ny && x < nx)
            split_bin<NL, F, XDEP>(p, y, x, [&](int r, int c, int s) {
              return line_at((ly + 1 + r) * PXk + lx + 1 + c, s);
            }, se, sd);
        }
      };
      if (p.os == 2)
        bin(std::integral_constant<int, 2>{});
      else
        bin(std::integral_constant<int, 4>{});
    } else if constexpr (FULL) {
#pragma unroll
      for (int k = 0; k < kPre; ++k) read_back(tid + k * kSplatThreads, dpre[k]);
    } else {
      for (int i = tid; i < TXk * TYk; i += kSplatThreads) read_back(i, 0.f);
    }
  };
  const bool inner = sy0 >= 1 && sy1 <= ny - 2 && sx0 >= 1 && sx1 <= nx - 2;
  using std::false_type;
  using std::true_type;
  constexpr std::integral_constant<int, 0> kAny{};
  constexpr std::integral_constant<int, kSplatTileX> kTX{};
  constexpr std::integral_constant<int, kSplatTileY> kTY{};
  constexpr std::integral_constant<int, kSplatSmallX> kSX{};
  constexpr std::integral_constant<int, kSplatSmallY> kSY{};
  if (fixed && TX == kSplatTileX && TY == kSplatTileY) {
    if (inner)
      tile(kTX, kTY, true_type{});
    else
      tile(kTX, kTY, false_type{});
  } else if (fixed && TX == kSplatSmallX && TY == kSplatSmallY) {
    if (inner)
      tile(kSX, kSY, true_type{});
    else
      tile(kSX, kSY, false_type{});
  } else {
    tile(kAny, kAny, false_type{});
  }
  if (mode != kSplatForward && mode != kSplatLines && p.resid != nullptr) {
    __syncthreads();
    se = wave_sum(se);
    sd = wave_sum(sd);
    if ((tid & 63) == 0) {
      scratch[2 * (tid >> 6)] = se;
      scratch[2 * (tid >> 6) + 1] = sd;
    }
    __syncthreads();
    if (tid == 0) {
      float te = 0.f, td = 0.f;
      for (int w = 0; w < kSplatThreads / 64; ++w) {
        te += scratch[2 * w];
        td += scratch[2 * w + 1];
      }
      G(p.resid)[2 * local] = te;
      G(p.resid)[2 * local + 1] = td;
    }
  }
}

template <bool B, int NL>
__global__ __launch_bounds__(kSplatThreads) void k_splat(KArgs a,
                                                        const ProbDesc* __restrict__ table) {
  EPR_DISPATCH(B, a, table, xcd_remap(blockIdx.x, gridDim.x), (splat_body<NL, false>), a.mode);
}
// x-dependent spectrum
template <bool B, int NL>
__global__ __launch_bounds__(kSplatThreads) void k_splat_x(KArgs a,
                                                          const ProbDesc* __restrict__ table) {
  EPR_DISPATCH(B, a, table, xcd_remap(blockIdx.x, gridDim.x), (splat_body<NL, true>), a.mode);
}

template <int NL>
void launch_splat_nl(const KArgs& a, int total_blocks, size_t lds, hipStream_t s) {
  if (a.xdep && a.table)
    hipLaunchKernelGGL((k_splat_x<true, NL>), dim3(total_blocks), dim3(kSplatThreads), lds, s,
                       a, a.table);
  else if (a.table)
    hipLaunchKernelGGL((k_splat<true, NL>), dim3(total_blocks), dim3(kSplatThreads), lds, s, a,
                       a.table);
  else if (a.p.xcol)
    hipLaunchKernelGGL((k_splat_x<false, NL>), dim3(total_blocks), dim3(kSplatThreads), lds, s,
                       a, a.table);
  else
    hipLaunchKernelGGL((k_splat<false, NL>), dim3(total_blocks), dim3(kSplatThreads), lds, s, a,
                       a.table);
}

// Allow the instance its dynamic LDS.
template <int NL>
hipError_t set_splat_attributes_nl() {
  for (const void* f : {(const void*)k_splat<false, NL>, (const void*)k_splat<true, NL>,
                        (const void*)k_splat_x<false, NL>, (const void*)k_splat_x<true, NL>}) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kSplatLdsMax);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Instantiate the host functions (and with them the kernels) of one line count, or declare them.
#define EPR_SPLAT_UNIT(N)                                                                   \
  template void launch_splat_nl<N>(const KArgs&, int, size_t, hipStream_t);                \
  template hipError_t set_splat_attributes_nl<N>();
#define EPR_SPLAT_DECLARE(N)                                                                \
  extern template void launch_splat_nl<N>(const KArgs&, int, size_t, hipStream_t);         \
  extern template hipError_t set_splat_attributes_nl<N>();

}  // namespace epr
