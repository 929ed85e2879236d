// Column pass: column FFT, the fused Paganin-type filter (Section 2), inverse column FFT.
#include <hip/hip_runtime.h>

#include "spectral.h"

namespace epr {

// ---------------------------------------------------------------------------------------------
// Column pass: per (line s, block of kColBlock frequencies) forward FFT along y, multiply by
// scale / (1 + h_s (fx^2 + fy^2)), inverse FFT along y (via conjugation), in place.  The block
// is one contiguous run of ny * kColBlock complex values.
// ---------------------------------------------------------------------------------------------
// EMAX: complex values of the largest column block the instance transforms (lengths up to
// EMAX / kColBlock are compiled in).
template <int NT, int EMAX = SizeClass<NT>::kColEmax>
__device__ __forceinline__ void colfft_body(const ProbDesc& p, int local, int) {
  constexpr int kColF4 = (EMAX / 2 + NT - 1) / NT;  // float4 per thread, column block
  extern __shared__ float2 buf[];
  const int ny = p.ny, nx = p.nx;
  const int s = local / p.nblk;
  const int blk = local - s * p.nblk;
  gptr<float2> g = G(p.spec) + ((size_t)s * p.nblk + blk) * ny * kColBlock;
  // output: in place, or the spectra of one preconditioner block (block-wise preconditioner)
  gptr<float2> go = G(p.spec_out ? p.spec_out : p.spec) + ((size_t)s * p.nblk + blk) * ny * kColBlock;
  const int n4 = ny * kColBlock / 2;
  const int tid = threadIdx.x;
  const TwTable tw = load_twiddles(kColBlock * lds_rows(ny), p.col, tid, NT);
  {
    // the block is one contiguous run: copy it to LDS with direct global->LDS loads, 16 bytes
    // per lane, one 1 KiB chunk (32 rows) per wave and instruction (no registers involved);
    // each chunk lands after its padding row
    gptr<const float4> g4 = (gptr<const float4>)g;
    float4* b4 = reinterpret_cast<float4*>(buf);
    const int lane = tid & 63, wave = tid >> 6;
    for (int base = wave * 64; base < n4; base += NT) {
      if (base + lane < n4)
        __builtin_amdgcn_global_load_lds((const gvoid_t*)((gptr<const char>)g4 + (unsigned)((base + lane) * 16)),
                                         (lvoid_t*)(b4 + base + 2 * (base >> 6)), 16, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(0);  // all loads of this wave have landed in LDS
  }
  __syncthreads();
  ColumnFilter filt;
  filt.h = p.lp.h[s];
  filt.scale = p.lp.spec_scale;
  filt.inv_ny = 1.f / (float)ny;
  filt.inv_nx = 1.f / (float)nx;
  filt.ny = ny;
  filt.col0 = blk * kColBlock;
  // compile-time lengths store the result from their last stage; the others from LDS here
  if (!fft_filter_ifft_lds<kColBlock, NT, EMAX, 2>(0, p.col, tw, filt, go)) {
    gptr<float4> g4 = (gptr<float4>)go;
    const float4* b4 = reinterpret_cast<const float4*>(buf);
#pragma unroll
    for (int k = 0; k < kColF4; ++k) {
      const int i = tid + k * NT;
      if (i < n4) {
        const float4 v = b4[i + 2 * (i >> 6)];  // float4 i = complex 2i, 2i+1 of row i/2
        stg(g4, (unsigned)i, make_float4(v.x, -v.y, v.z, -v.w));
      }
    }
  }
}

template <bool B, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_colfft(KArgs a, const ProbDesc* __restrict__ table) {
  EPR_DISPATCH(B, a, table, xcd_remap(blockIdx.x, gridDim.x), colfft_body<NT>, 0);
}

// The 1024-thread column pass for columns of at most kColMidMax rows (the 2160 x 2560 problems):
// without the 4096-point transforms it needs 64 VGPRs, so eight waves per SIMD, and two
// workgroups share a CU where their LDS fits (ny <= 2213), against one for the full instance.
template <bool B>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8))) void k_colfft_mid(KArgs a, const ProbDesc* __restrict__ table) {
  EPR_DISPATCH(B, a, table, xcd_remap(blockIdx.x, gridDim.x), (colfft_body<1024, kColBlock * kColMidMax>), 0);
}

hipError_t launch_colfft(const KArgs& a, int total_blocks, size_t lds, hipStream_t s, int nt) {
  const int ny_max = a.table ? a.ny_max : a.p.ny;
  if (nt == 1024 && ny_max > 0 && ny_max <= kColMidMax) {
    if (a.table)
      hipLaunchKernelGGL(k_colfft_mid<true>, dim3(total_blocks), dim3(1024), lds, s, a, a.table);
    else
      hipLaunchKernelGGL(k_colfft_mid<false>, dim3(total_blocks), dim3(1024), lds, s, a, a.table);
    return hipGetLastError();
  }
  EPR_LAUNCH_SC(k_colfft, a, total_blocks, nt, lds, s);
  return hipGetLastError();
}

hipError_t set_colfft_attributes() {
  const void* const fns[] = {EPR_SC_FNS(k_colfft), (const void*)k_colfft_mid<false>, (const void*)k_colfft_mid<true>};
  return allow_dynamic_lds(fns);
}

}  // namespace epr
