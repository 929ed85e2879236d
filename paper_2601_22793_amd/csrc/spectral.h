// Shared by the spectral kernels: the row pass (back-transport + row real FFT, k_rowfft.hip), the
// column FFT with the fused Paganin-type filter (Section 2, k_colfft.hip), and the row inverse
// real FFT with the fused update and single-thickness projection (Methods 4.4, Eq. 7,
// k_rowinv.hip).
//
// Real transforms of length nx use the half-length complex trick: z[m] = r[2m] + i r[2m+1],
// Z = FFT_{nx/2}(z), X[k] = (Z[k] + conj Z[M-k])/2 - i W^k (Z[k] - conj Z[M-k])/2 with
// W = exp(-2 pi i / nx), and the mirror relation for the inverse.  All transforms are
// unnormalised; the product of their gains (ny * nx/2) is removed by the filter's scale.
//
// Every kernel is instantiated for two size classes, NT = 512 threads (nx, ny <= 2048) and
// NT = 1024 threads (<= 4096), so that each thread holds at most 8 (rows) or 16 (columns)
// complex values per FFT stage and 16 pixels of a row block.  The row inverse of small single
// images also runs groups of NT = 128 or 256 threads, one line each (k_rowinv_g).  Global memory phases issue all
// of a thread's loads before using any of them.
#pragma once

#include <hip/hip_runtime.h>

#include "dev_common.h"
#include "epr_internal.h"
#include "fft_lds.h"

namespace epr {

typedef __attribute__((address_space(1))) void gvoid_t;  // global memory
typedef __attribute__((address_space(3))) void lvoid_t;  // LDS

template <int NT>
struct SizeClass {
  static constexpr int kMaxNx = 4 * NT;                     // 2048 or 4096
  static constexpr int kRowEmax = kRows * (kMaxNx / 2);     // complex values of a row block
  static constexpr int kColEmax = kColBlock * kMaxNx;       // complex values of a column block
  static constexpr int kPix = kRows * kMaxNx / NT;          // pixels of a row block per thread
  static constexpr int kSpecPerThread = (kRows * (kMaxNx / 2 + kColBlock) + NT - 1) / NT;
  static constexpr int kColF4 = kColEmax / 2 / NT;          // float4 per thread, column block
};

// Float offset, in a row-transform buffer (kRows rows, padded), of the thread's pixel in row r
// and column x = tid + j NT: sample x is the real (even x) or imaginary (odd x) part of complex
// element x / 2.  NT / 2 is a multiple of 32, so the offset is a per-thread base plus a
// compile-time constant and the LDS accesses take immediate offsets.
// CNT sequences interleaved (kRows rows of one line, or of several lines one after another).
template <int NT, int CNT = kRows>
struct RowPix {
  static_assert((NT / 2) % (1 << kLdsPadShift) == 0, "row pixel layout");
  static constexpr int kJ = 2 * CNT * (NT / 2 + ((NT / 2) >> kLdsPadShift));
  int base;
  __device__ __forceinline__ explicit RowPix(int tid)
      : base(2 * CNT * ((tid >> 1) + (tid >> (kLdsPadShift + 1))) + (tid & 1)) {}
  __device__ __forceinline__ int at(int r, int j) const { return base + j * kJ + 2 * r; }
};

// W_nx^k (0 <= k <= nx/2) of the real-transform split from the table of the half-length
// transform, W_M^j with M = nx/2: W_nx^(2j) = W_M^j and W_nx^(2j+1) = W_M^j W_nx^1.
__device__ __forceinline__ float2 half_tw(const TwTable& tw, float2 w1, int k) {
  const float2 w = tw(k >> 1);
  return (k & 1) ? cmul(w, w1) : w;
}

// launch K<batched, threads> for a launch of nt-thread kernels
#define EPR_LAUNCH_SC(K, a, grid, nt, lds, s)                                                \
  do {                                                                                       \
    if (nt == 512) {                                                                         \
      if ((a).table)                                                                         \
        hipLaunchKernelGGL((K<true, 512>), dim3(grid), dim3(512), lds, s, a, a.table);               \
      else                                                                                   \
        hipLaunchKernelGGL((K<false, 512>), dim3(grid), dim3(512), lds, s, a, a.table);              \
    } else {                                                                                 \
      if ((a).table)                                                                         \
        hipLaunchKernelGGL((K<true, 1024>), dim3(grid), dim3(1024), lds, s, a, a.table);             \
      else                                                                                   \
        hipLaunchKernelGGL((K<false, 1024>), dim3(grid), dim3(1024), lds, s, a, a.table);            \
    }                                                                                        \
  } while (0)

// the instances of K<batched, threads>, as entries of a function list
#define EPR_SC_FNS(K)                                    \
  (const void*)K<false, 512>, (const void*)K<true, 512>, \
      (const void*)K<false, 1024>, (const void*)K<true, 1024>

// allow each kernel of the list its dynamic LDS (up to the CU's 160 KB)
template <int N>
inline hipError_t allow_dynamic_lds(const void* const (&fns)[N]) {
  for (const void* f : fns) {
    const hipError_t e =
        hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 64);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace epr
