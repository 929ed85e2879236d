// Row pass: back-transport (Eq. 4) and the row real FFT.
#include <hip/hip_runtime.h>

#include "spectral.h"

#ifndef EPR_ROWFFT_WAVES
#define EPR_ROWFFT_WAVES 8
#endif

namespace epr {

// Bilinear interpolation weights and taps of e at (x + ux, y + uy), zero off the grid
// (Eq. 4): v = w00 e(y0,x0) + w10 e(y0,x0+1) + w01 e(y0+1,x0) + w11 e(y0+1,x0+1).
struct Taps {
  float v00, v10, v01, v11, dx, dy;
};

__device__ __forceinline__ Taps load_taps(gptr<const float> e, int ny, int nx, int y, int x,
                                          float ux, float uy) {
  Taps t;
  t.dx = __builtin_amdgcn_fractf(ux);  // x - floor(x), kept below 1 (as the splat forms it)
  t.dy = __builtin_amdgcn_fractf(uy);
  const int x0 = x + floor_to_int(ux), y0 = y + floor_to_int(uy);
  const bool xin0 = (unsigned)x0 < (unsigned)nx, xin1 = (unsigned)(x0 + 1) < (unsigned)nx;
  const bool yin0 = (unsigned)y0 < (unsigned)ny, yin1 = (unsigned)(y0 + 1) < (unsigned)ny;
  // clamp the addresses, zero the values: every lane issues the same four loads
  const int cx0 = min(max(x0, 0), nx - 1), cx1 = min(max(x0 + 1, 0), nx - 1);
  const int cy0 = min(max(y0, 0), ny - 1), cy1 = min(max(y0 + 1, 0), ny - 1);
  const int r0 = __mul24(cy0, nx), r1 = __mul24(cy1, nx);
  const float a = ldg(e, (unsigned)(r0 + cx0)), b = ldg(e, (unsigned)(r0 + cx1));
  const float c = ldg(e, (unsigned)(r1 + cx0)), d = ldg(e, (unsigned)(r1 + cx1));
  t.v00 = (yin0 && xin0) ? a : 0.f;
  t.v10 = (yin0 && xin1) ? b : 0.f;
  t.v01 = (yin1 && xin0) ? c : 0.f;
  t.v11 = (yin1 && xin1) ? d : 0.f;
  return t;
}

// (1 - dy)((1 - dx) v00 + dx v10) + dy((1 - dx) v01 + dx v11), as three linear interpolations
// (a subtraction and a multiply-add each)
__device__ __forceinline__ float taps_value(const Taps& t) {
  const float a = fmaf(t.dx, t.v10 - t.v00, t.v00);
  const float b = fmaf(t.dx, t.v11 - t.v01, t.v01);
  return fmaf(t.dy, b - a, a);
}

// Back-transport of line s at column x = tid + j NT of the kRows rows from y0 (Eq. 4, the
// adjoint of the splat): v[r] = bilinear sample of e_s at (x, y0 + r) + b_s D Y, zero off the
// grid.  A wave whose stencil lies inside the image (wave-uniform test) reads it at one column
// offset per lane from wave-uniform row pointers; if then every tap of the wave is inside the
// image too (a wave vote), the four taps are read at one offset per lane from four
// wave-uniform base pointers, with no clamps or selects.  Every path computes the same values.
template <int NT, bool XDEP>
__device__ __forceinline__ void gather_column(const ProbDesc& p, gptr<const float> es,
                                              gptr<const float> Y, int s, float bs, int y0, int j,
                                              float (&v)[kRows]) {
  const int nx = p.nx, ny = p.ny;
  const int tid = threadIdx.x;
  const int xw = __builtin_amdgcn_readfirstlane((tid & ~63) + j * NT);  // the wave's first column
  const int x = min(tid + j * NT, nx - 1);  // columns past the row: a clamped pixel, discarded
  float cb = bs;
  if constexpr (XDEP) cb = xcol_at(p, x, s).z;
  if (xw >= 1 && xw + 64 <= nx - 1 && y0 >= 1 && y0 + kRows <= ny - 1) {
    // central differences everywhere: D Y = (Y(x+1) - Y(x-1)) / 2, likewise in y.  One load per
    // row y0 - 1 .. y0 + kRows from wave-uniform row pointers; the column neighbours are those of
    // the adjacent lanes, and the two at the wave's ends come with a load of those lanes alone.
    // (The L1 takes about ten accesses per load: reading both neighbours of every row as well
    // made the stencil 14 loads beside the 8 of the taps; 2048 x 2048, 8 lines: 113 -> 110 us.)
    const unsigned xo = (unsigned)x;
    const int lane = tid & 63;
    float c[kRows + 2], ge[kRows] = {};
#pragma unroll
    for (int r = 0; r < kRows + 2; ++r) c[r] = ldg(Y + (y0 + r - 1) * nx, xo);
    if (lane == 0 || lane == 63) {
      const unsigned xe = lane == 0 ? xo - 1 : xo + 1;
#pragma unroll
      for (int r = 0; r < kRows; ++r) ge[r] = ldg(Y + (y0 + r) * nx, xe);
    }
    float ga[kRows], gb[kRows], gc[kRows], gd[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      ga[r] = lane_right_or(c[r + 1], ge[r]);
      gb[r] = lane_left_or(c[r + 1], ge[r]);
      gc[r] = c[r + 2];
      gd[r] = c[r];
    }
    // b (0.5 (a - b)) == (0.5 b) (a - b): the halving is exact, so this is the value the
    // clamped path computes
    const float hb = 0.5f * cb;
    float ux[kRows], uy[kRows];
    unsigned off[kRows];
    bool inside = true;
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      ux[r] = hb * (ga[r] - gb[r]);
      uy[r] = hb * (gc[r] - gd[r]);
      const int xt = x + floor_to_int(ux[r]), yt = y0 + r + floor_to_int(uy[r]);
      inside = inside && (unsigned)xt <= (unsigned)(nx - 2) && (unsigned)yt <= (unsigned)(ny - 2);
      off[r] = (unsigned)(__mul24(yt, nx) + xt);
    }
    if (__all(inside)) {
      const gptr<const float> e10 = es + 1, e01 = es + nx, e11 = es + nx + 1;
      Taps t[kRows];
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        t[r].v00 = ldg(es, off[r]);
        t[r].v10 = ldg(e10, off[r]);
        t[r].v01 = ldg(e01, off[r]);
        t[r].v11 = ldg(e11, off[r]);
        t[r].dx = __builtin_amdgcn_fractf(ux[r]);
        t[r].dy = __builtin_amdgcn_fractf(uy[r]);
      }
#pragma unroll
      for (int r = 0; r < kRows; ++r) v[r] = taps_value(t[r]);
    } else {
      Taps t[kRows];
#pragma unroll
      for (int r = 0; r < kRows; ++r) t[r] = load_taps(es, ny, nx, y0 + r, x, ux[r], uy[r]);
#pragma unroll
      for (int r = 0; r < kRows; ++r) v[r] = taps_value(t[r]);
    }
    return;
  }
  // near the edges: clamped stencil (one-sided differences on the first and last row and
  // column), clamped taps; rows past the image sample a clamped pixel, discarded
  float ga[kRows], gb[kRows], gc[kRows], gd[kRows];
  bool cy[kRows];
  const int xl = max(x - 1, 0), xh = min(x + 1, nx - 1);
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const int y = min(y0 + r, ny - 1);
    const int yl = max(y - 1, 0), yh = min(y + 1, ny - 1);
    ga[r] = ldg(Y, (unsigned)(__mul24(y, nx) + xh));
    gb[r] = ldg(Y, (unsigned)(__mul24(y, nx) + xl));
    gc[r] = ldg(Y, (unsigned)(__mul24(yh, nx) + x));
    gd[r] = ldg(Y, (unsigned)(__mul24(yl, nx) + x));
    cy[r] = yh - yl == 2;
  }
  const bool cx = xh - xl == 2;
  Taps t[kRows];
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const float gx = cx ? 0.5f * (ga[r] - gb[r]) : ga[r] - gb[r];
    const float gy = cy[r] ? 0.5f * (gc[r] - gd[r]) : gc[r] - gd[r];
    t[r] = load_taps(es, ny, nx, min(y0 + r, ny - 1), x, cb * gx, cb * gy);
  }
#pragma unroll
  for (int r = 0; r < kRows; ++r) v[r] = taps_value(t[r]);
}

// ---------------------------------------------------------------------------------------------
// Row pass: per (line s, block of kRows rows) compute r_s (gather of e_s at the mapped points,
// or a copy of e_s), then the real FFT of each row, stored as column blocks of the half
// spectrum.  In gather-only mode r_s goes to p.out and no transform is done (epr_adjoint).
// ---------------------------------------------------------------------------------------------
// XDEP: x-dependent spectrum, b_s of the gather is read at each pixel's column.
template <int NT, bool XDEP>
__device__ __forceinline__ void rowfft_body(const ProbDesc& p, int local, int mode) {
  using SC = SizeClass<NT>;
  extern __shared__ float2 buf[];
  const int nx = p.nx, ny = p.ny, M = nx >> 1;
  // lines vary fastest: the blocks of one row block (all lines) share the thickness stencil,
  // and with the XCD-contiguous block order they run behind one L2
  const int L = p.lp.n;
  const int rb = local / L;
  const int s = local - rb * L;
  const int y0 = rb * kRows;
  gptr<const float> es = G(p.e) + (size_t)s * nx * ny;
  gptr<const float> Y = G(p.Y);
  const float bs = p.lp.b[s];
  const int tid = threadIdx.x;
  float* fb = reinterpret_cast<float*>(buf);
  const bool gather = mode != kRowCopyFft;
  // twiddle table after the transform buffer; its loads overlap the gather
  const TwTable tw = load_twiddles(kRows * lds_rows(M), p.row, tid, NT);

  // the thread's pixels: column x = tid + j NT of each of the kRows rows; the kRows values of
  // one column are loaded together and go straight into the transform buffer (complex index
  // x/2, real part for even x, imaginary for odd x)
  constexpr int kPerRow = SC::kMaxNx / NT;
  const RowPix<NT> pix(tid);
#pragma unroll
  for (int j = 0; j < kPerRow; ++j) {
    // a wave whose columns all lie past the row (narrow images in a size class) has nothing
    // to load or store in this column chunk
    if (__builtin_amdgcn_readfirstlane((tid & ~63) + j * NT) >= nx) continue;
    float v[kRows];
    if (gather) {
      gather_column<NT, XDEP>(p, es, Y, s, bs, y0, j, v);
    } else {
      // columns or rows past the image read a clamped in-bounds pixel; the value is discarded
      const int x = min(tid + j * NT, nx - 1);
#pragma unroll
      for (int r = 0; r < kRows; ++r)
        v[r] = ldg(es, (unsigned)(__mul24(min(y0 + r, ny - 1), nx) + x));
    }
    const int x = tid + j * NT;
    if (x < nx) {
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        const int y = y0 + r;
        const float val = (y < ny) ? v[r] : 0.f;
        fb[pix.at(r, j)] = val;
        if (mode == kRowGatherOnly && y < ny) stg(G(p.out) + (size_t)s * nx * ny, (unsigned)(__mul24(y, nx) + x), val);
      }
    }
  }
  if (mode == kRowGatherOnly) return;
  __syncthreads();
  fft_lds<kRows, NT, SC::kRowEmax, 1>(0, p.row, tw);

  // Split of the half-length transform Z into the half spectrum X, one pair (k, M - k) per
  // item: with A = (Z[k] + conj Z[M-k]) / 2, B = (Z[k] - conj Z[M-k]) / 2 and W = W_nx,
  //   X[k] = A - i W^k B,   X[M-k] = conj(A) - i conj(W^k B)
  // (W^(M-k) = -conj W^k).  Items k = 0 .. M/2 cover every frequency 0 .. M; for even M the
  // item k = M/2 is its own mirror.  Then the unused columns of the last block are zeroed.
  // Item i: column c = i % 4 of block i / 16, row (i / 4) % 4, so that the X[k] of 16
  // consecutive items form one 128-byte tile row group.
  const float2 w1 = G(p.row_tw)[1];
  gptr<float2> out = G(p.spec) + (size_t)s * p.nblk * ny * kColBlock;
  const int nk = M / 2 + 1;
  const int npair = (nk + kColBlock - 1) / kColBlock * (kColBlock * kRows);
  const int nitem = npair + (p.nblk * kColBlock - (M + 1)) * kRows;
  for (int i = tid; i < nitem; i += NT) {
    if (i < npair) {
      const int c = i % kColBlock;
      const int r = (i / kColBlock) % kRows;
      const int k = (i / (kColBlock * kRows)) * kColBlock + c;
      const int y = y0 + r;
      if (k >= nk || y >= ny) continue;
      const int km = M - k;
      const float2 zk = buf[lds_index<kRows>(k, r)];
      const float2 zm = cconj(buf[lds_index<kRows>(k == 0 ? 0 : km, r)]);
      const float2 A = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y + zm.y));
      const float2 B = make_float2(0.5f * (zk.x - zm.x), 0.5f * (zk.y - zm.y));
      const float2 WB = cmul(half_tw(tw, w1, k), B);
      stg(out, (unsigned)(((k >> 2) * ny + y) * kColBlock + (k & 3)),
          make_float2(A.x + WB.y, A.y - WB.x));                 // A - i W B
      if (km != k)
        stg(out, (unsigned)(((km >> 2) * ny + y) * kColBlock + (km & 3)),
            make_float2(A.x - WB.y, -A.y - WB.x));              // conj A - i conj(W B)
    } else {
      // zero padding: frequencies M + 1 .. 4 nblk - 1 of every row
      const int j = i - npair;
      const int k = M + 1 + j / kRows, y = y0 + j % kRows;
      if (y < ny) stg(out, (unsigned)(((k >> 2) * ny + y) * kColBlock + (k & 3)), make_float2(0.f, 0.f));
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Row pass over K lines per workgroup, one after the other (the problem's lines in groups of K,
// the last group may be short).  The lines of a row block share its thickness stencil: after
// the first line it comes from the workgroup's own L1 instead of being fetched again by
// another workgroup.  The transform buffer is reused line by line.  K is a compile-time
// constant: the line bodies are laid out one after the other, which keeps the register
// allocation of one line (a run-time loop over lines spills).
// ---------------------------------------------------------------------------------------------
template <int NT, bool XDEP, int K, int I = 0>
__device__ __forceinline__ void rowfft_group_lines(const ProbDesc& p, int base, int n, int mode) {
  if constexpr (I < K) {
    if (I < n) {
      if (I > 0) __syncthreads();  // the previous line's split has read the buffer and table
      rowfft_body<NT, XDEP>(p, base + I, mode);
      rowfft_group_lines<NT, XDEP, K, I + 1>(p, base, n, mode);
    }
  }
}

template <int NT, bool XDEP, int K>
__device__ __forceinline__ void rowfft_group_body(const ProbDesc& p, int local, int mode) {
  const int L = p.lp.n;
  const int ng = (L + K - 1) / K;
  const int rb = local / ng;
  const int g0 = (local - rb * ng) * K;
  rowfft_group_lines<NT, XDEP, K>(p, rb * L + g0, min(K, L - g0), mode);
}


template <bool B, int NT, int K>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(EPR_ROWFFT_WAVES))) void k_rowfft(KArgs a, const ProbDesc* __restrict__ table) {
  EPR_DISPATCH(B, a, table, xcd_remap(blockIdx.x, gridDim.x), (rowfft_group_body<NT, false, K>), a.mode);
}
// x-dependent spectrum
template <bool B, int NT, int K>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(EPR_ROWFFT_WAVES))) void k_rowfft_x(KArgs a, const ProbDesc* __restrict__ table) {
  EPR_DISPATCH(B, a, table, xcd_remap(blockIdx.x, gridDim.x), (rowfft_group_body<NT, true, K>), a.mode);
}

// the row-pass instances by lines per workgroup, as two-parameter templates for EPR_LAUNCH_SC
template <bool B, int NT> constexpr auto k_rowfft1 = k_rowfft<B, NT, 1>;
template <bool B, int NT> constexpr auto k_rowfft2 = k_rowfft<B, NT, 2>;
template <bool B, int NT> constexpr auto k_rowfft4 = k_rowfft<B, NT, 4>;
template <bool B, int NT> constexpr auto k_rowfft_x1 = k_rowfft_x<B, NT, 1>;
template <bool B, int NT> constexpr auto k_rowfft_x2 = k_rowfft_x<B, NT, 2>;
template <bool B, int NT> constexpr auto k_rowfft_x4 = k_rowfft_x<B, NT, 4>;

hipError_t launch_rowfft(const KArgs& a, int total_blocks, size_t lds, hipStream_t s, int nt) {
  const bool x = a.table ? a.xdep != 0 : a.p.xcol != nullptr;
  const int k = a.table ? a.rl : row_lines(a.p);
  if (x && a.mode != kRowCopyFft) {
    switch (k) {
      case 4: EPR_LAUNCH_SC(k_rowfft_x4, a, total_blocks, nt, lds, s); break;
      case 2: EPR_LAUNCH_SC(k_rowfft_x2, a, total_blocks, nt, lds, s); break;
      default: EPR_LAUNCH_SC(k_rowfft_x1, a, total_blocks, nt, lds, s); break;
    }
  } else {
    switch (k) {
      case 4: EPR_LAUNCH_SC(k_rowfft4, a, total_blocks, nt, lds, s); break;
      case 2: EPR_LAUNCH_SC(k_rowfft2, a, total_blocks, nt, lds, s); break;
      default: EPR_LAUNCH_SC(k_rowfft1, a, total_blocks, nt, lds, s); break;
    }
  }
  return hipGetLastError();
}

hipError_t set_rowfft_attributes() {
  const void* const fns[] = {EPR_SC_FNS(k_rowfft1), EPR_SC_FNS(k_rowfft2), EPR_SC_FNS(k_rowfft4),
                             EPR_SC_FNS(k_rowfft_x1), EPR_SC_FNS(k_rowfft_x2), EPR_SC_FNS(k_rowfft_x4)};
  return allow_dynamic_lds(fns);
}

}  // namespace epr
