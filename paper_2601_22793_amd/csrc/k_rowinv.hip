// Row inverse pass: inverse row real FFT with the fused update and single-thickness projection
// (Methods 4.4, Eq. 7).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "spectral.h"

namespace epr {

// ---------------------------------------------------------------------------------------------
// Row inverse pass: per block of kRows rows, for every line: inverse real FFT of the filtered
// half spectrum -> dI_s; then either write dI_s (precondition mode) or accumulate the
// projection of I_s + omega dI_s onto one thickness (solve mode) and write tau.
//   * The block's 4 x 4 tiles of a line are copied verbatim to LDS by direct global->LDS loads;
//     the next line's copy streams in while the current line is transformed (the transform
//     reads its twiddles from LDS, so no other global load waits behind the copy).
//   * The thread's pixels, their thickness and their projection sums stay in registers.
// ---------------------------------------------------------------------------------------------
template <int NT>
__device__ __forceinline__ void fetch_row_tiles(gptr<const float2> sp, float2* dst, int nblk,
                                                int ny, int y0) {
  // 16-byte chunk q of the block: tile blk = q / 8, row r = (q / 2) % 4, columns 2 (q % 2) + {0,1}
  const int nq = nblk * 8;
  const int tid = group_thread<NT>(), lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  float4* d4 = reinterpret_cast<float4*>(dst);
  for (int base = wave * 64; base < nq; base += NT) {
    const int q = base + lane;
    if (q < nq) {
      const int blk = q >> 3, r = (q >> 1) & 3;
      const int y = min(y0 + r, ny - 1);  // rows past the image repeat the last row
      gptr<const char> src = (gptr<const char>)sp + (unsigned)(((blk * ny + y) * 2 + (q & 1)) * 16);
      __builtin_amdgcn_global_load_lds((const gvoid_t*)src, (lvoid_t*)(d4 + base), 16, 0, 0);
    }
  }
}

constexpr float kThick = 8.f;  // largest a_s tau of the update's difference form

// GR: lines transformed at once, by groups of NT threads (GR NT threads a workgroup).
// XDEP: x-dependent spectrum, the update and projection constants are read per column.
// BLK (with XDEP): block-wise preconditioner.  Each line has p.nbp filtered spectra, one per
// preconditioner block b (block 0 at p.spec, block b >= 1 in p.spec_blk); the row
// inverse transforms each of them and blends them per column with the interpolation weights
// lambda_b(x) (p.xblk[x] = {b0, t}: lambda_b0 = 1 - t, lambda_(b0+1) = t, 0 otherwise) before
// the update.
template <int NT, int GR, bool SOLVE, bool XDEP, bool BLK = false>
__device__ __forceinline__ void rowinv_body(const ProbDesc& p, int local, int) {
  using SC = SizeClass<NT>;
  extern __shared__ float2 buf[];
  const int nx = p.nx, ny = p.ny, M = nx >> 1;
  const int y0 = local * kRows;
  const int L = p.lp.n;
  const int tid = group_thread<NT>();
  const int grp = GR > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / NT) : 0;
  const int nin = p.nblk * kColBlock * kRows;  // complex values of one line's tiles
  const size_t line_elems = (size_t)p.nblk * ny * kColBlock;
  const int region = nin + kRows * lds_rows(M);  // LDS of one group
  float2* raw = buf + grp * region;  // the line's tiles as copied: [block][row][column]
  float2* F = raw + nin;             // transform buffer
  const TwTable tw = load_twiddles(GR * region, p.row, threadIdx.x, NT * GR);
  const float2 w1 = G(p.row_tw)[1];
  gptr<const float2> spec = G((const float2*)p.spec);
  fetch_row_tiles<NT>(spec + min(grp, L - 1) * line_elems, raw, p.nblk, ny, y0);

  // the thread's pixels: row r, column x = tid + j NT (k = r * kPerRow + j)
  constexpr int kPerRow = SC::kMaxNx / NT;
  // live[j]: the wave has columns of chunk j inside the row (wave-uniform; narrow images in a
  // size class leave whole chunks empty, which are then skipped)
  bool live[kPerRow];
#pragma unroll
  for (int j = 0; j < kPerRow; ++j)
    live[j] = __builtin_amdgcn_readfirstlane((tid & ~63) + j * NT) < nx;
  float tv[SC::kPix], acc[SC::kPix];
#pragma unroll
  for (int k = 0; k < SC::kPix; ++k) {
    const int r = k / kPerRow, x = min(tid + (k % kPerRow) * NT, nx - 1);
    const int y = min(y0 + r, ny - 1);
    tv[k] = 0.f;
    if constexpr (SOLVE)
      if (live[k % kPerRow]) tv[k] = ldg(G((const float*)p.tau), (unsigned)(__mul24(y, nx) + x));
    acc[k] = 0.f;
  }
  // A pixel is thick if some a_s tau of it leaves the range of the update's difference form (a NaN
  // does not: that form carries it on).  any_thick: the wave has such a pixel.
  float amax = 0.f;
  bool any_thick = false;
  if constexpr (SOLVE) {
    float tmax = 0.f;
    for (int s = 0; s < L; ++s) amax = fmaxf(amax, p.lp.a_hi[s]);
    amax = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(amax)));
#pragma unroll
    for (int k = 0; k < SC::kPix; ++k) tmax = fmaxf(tmax, tv[k]);
    any_thick = __any(amax * tmax > kThick);
  }
  const float odd_sign = (tid & 1) ? -1.f : 1.f;  // NT is even: x has the parity of tid
  const RowPix<NT> pix(tid);
  // sum of every update the thread applies: finite exactly when each of them is (the floor
  // of the update would otherwise hide a NaN)
  float chk = 0.f;
  // transform units: one per line, or one per (line, preconditioner block), block fastest
  const int nb = BLK ? p.nbp : 1;
  const int nunit = L * nb;
  float dacc[BLK ? SC::kPix : 1];
#pragma unroll
  for (int k = 0; k < (BLK ? SC::kPix : 1); ++k) dacc[k] = 0.f;

  // (a group without a line in the last round transforms line L - 1 again, for nothing)
  for (int u0 = 0; u0 < nunit; u0 += GR) {
    const int un = u0 + grp;
    const int s = BLK ? un / nb : min(un, L - 1);
    const int bk = BLK ? un - s * nb : 0;
    __builtin_amdgcn_s_waitcnt(0);  // this wave's copies of unit un have landed
    __syncthreads();                // ... and everyone's; unit un-1 is no longer read
    // Z[k] = E_k + i O_k, E_k = (X_k + conj X_{M-k})/2, O_k = (X_k - conj X_{M-k})/2 W^-k;
    // store conj(Z) so that a forward FFT followed by conjugation inverts it.
    // W_nx^(M-k) = -conj(W_nx^k).
    const int half = M >> 1;
    for (int i = tid; i < (half + 1) * kRows; i += NT) {
      const int k = i / kRows, r = i - k * kRows;
      // tile position of frequency k in row r: (k / 4) * 16 + r * 4 + k % 4
      const float2 xk = raw[((k >> 2) << 4) | (r << 2) | (k & 3)];
      const float2 xm = raw[(((M - k) >> 2) << 4) | (r << 2) | ((M - k) & 3)];
      const float2 wk = half_tw(tw, w1, k);
      {
        const float2 xmc = cconj(xm);
        const float2 E = make_float2(0.5f * (xk.x + xmc.x), 0.5f * (xk.y + xmc.y));
        const float2 D = make_float2(0.5f * (xk.x - xmc.x), 0.5f * (xk.y - xmc.y));
        const float2 O = cmul(D, cconj(wk));
        const float2 Z = make_float2(E.x - O.y, E.y + O.x);
        F[lds_index<kRows>(k, r)] = cconj(Z);
      }
      if (k != 0 && 2 * k != M) {
        const float2 xkc = cconj(xk);
        const float2 E = make_float2(0.5f * (xm.x + xkc.x), 0.5f * (xm.y + xkc.y));
        const float2 D = make_float2(0.5f * (xm.x - xkc.x), 0.5f * (xm.y - xkc.y));
        const float2 O = cmul(D, make_float2(-wk.x, -wk.y));  // conj(W^(M-k)) = -W^k
        const float2 Z = make_float2(E.x - O.y, E.y + O.x);
        F[lds_index<kRows>(M - k, r)] = cconj(Z);
      }
    }
    __syncthreads();  // the tiles are consumed: unit un+1 streams in during the transform
    if (u0 + GR < nunit) {
      const int s1 = BLK ? (un + 1) / nb : min(un + GR, L - 1), b1 = BLK ? (un + 1) - s1 * nb : 0;
      gptr<const float2> sb = b1 == 0 ? spec : G((const float2*)p.spec_blk) + (size_t)(b1 - 1) * p.spec_set;
      fetch_row_tiles<NT>(sb + (size_t)s1 * line_elems, raw, p.nblk, ny, y0);
    }
    fft_lds<kRows, NT, SC::kRowEmax, SOLVE ? (BLK ? 5 : 3) : 4>(grp * region + nin, p.row, tw);
    if (GR > 1 && un >= nunit) continue;

    const float* fb = reinterpret_cast<const float*>(F);
    if constexpr (BLK) {
      // blend this block's output into the line's update; the update follows the last block
#pragma unroll
      for (int k = 0; k < SC::kPix; ++k) {
        const int r = k / kPerRow, x = tid + (k % kPerRow) * NT;
        if (live[k % kPerRow] && x < nx) {
          const float2 bt = ldg(G(p.xblk), (unsigned)x);
          const int b0 = (int)bt.x;
          const float lam = bk == b0 ? 1.f - bt.y : (bk == b0 + 1 ? bt.y : 0.f);
          dacc[k] = fmaf(lam, odd_sign * fb[pix.at(r, k % kPerRow)], dacc[k]);
        }
      }
      if (bk + 1 < nb) continue;
    }
    if constexpr (SOLVE) {
      // The projection sums w_s mu_s ln(max(I_s + omega dI_s, 1e-6 w_s) / w_s).  With
      // E = exp(a_s tau) and z = (omega / w_s) dI_s that logarithm is
      //   -a_s tau + ln(max(1 + z E, 1e-6 E)),
      // and since sum_s w_s mu_s a_s = 1 / inv_den, tau itself leaves the sum: the new thickness is
      // tau - inv_den sum_s w_s mu_s ln(max(1 + z E, 1e-6 E)).  Near convergence the logarithm is
      // small, so its rounding and that of E count for little, where exp(-a_s tau) and the
      // logarithm of it, rounded, would give tau back to a few 1e-7 only in every iteration
      // (errors of whole solves: halved for multi-pixel shifts, a fifth for the local closure).
      // exp and ln through the hardware base-2 transcendentals (v_exp_f32 / v_log_f32, about one
      // ulp).  Pixels with a_s tau > 8 (transmission below 3e-4, where a new thickness far from tau
      // would cancel) take -ln(max(exp(-a_s tau) + z, 1e-6)) as it stands: each pixel by its own
      // thickness, so its rounding does not depend on the pixels that share its wave; only waves
      // that hold such a pixel form both.
      const float la2 = p.lp.a[s] * 1.4426950408889634f;
      const float mws_ln2 = p.lp.mw[s] * 0.69314718055994531f;
      const float om = p.relax, om_w = p.relax * p.lp.inv_w[s];
      auto update = [&](auto mixed) {
        // (opaque to the optimiser, which would keep the comparisons of the mixed form as 16 lane
        // masks through the loop over the lines and spill scalar registers)
        float am = amax;
        if constexpr (decltype(mixed)::value) asm volatile("" : "+s"(am));
#pragma unroll
        for (int j = 0; j < kPerRow; ++j) {
          const int x = tid + j * NT;
          if (!live[j] || x >= nx) continue;
          // conj of the transform output: the odd (imaginary) samples change sign
          float c_a2 = la2, c_z = om_w * odd_sign, c_mw = mws_ln2;
          if constexpr (XDEP) {  // the column's constants, once for its kRows pixels
            const float4 c = xcol_at(p, x, s), q = xproj_at(p, x, s);
            c_a2 = c.y * 1.4426950408889634f;
            c_z = BLK ? om * q.y : om * q.y * odd_sign;
            c_mw = q.x * 0.69314718055994531f;
          }
#pragma unroll
          for (int r = 0; r < kRows; ++r) {
            const int k = r * kPerRow + j;
            float v;
            if constexpr (BLK) {
              v = dacc[k];
              dacc[k] = 0.f;
            } else {
              v = fb[pix.at(r, j)];
            }
            chk += v;
            const float t2 = c_a2 * tv[k], z = c_z * v;
            const float E = __builtin_amdgcn_exp2f(t2);
            const float u = fmaf(z, E, 1.f);
            // what the rounding of 1 + z E dropped, as far as it matters: the logarithm needs
            // du / u, which is du for u near 1 and, bounded so, below its rounding elsewhere
            const float du = __builtin_amdgcn_fmed3f(fmaf(z, E, 1.f - u), -1.2e-7f, 1.2e-7f);
            float l = fmaf(du, 1.4426950408889634f, __builtin_amdgcn_logf(fmaxf(u, 1e-6f * E)));
            if constexpr (decltype(mixed)::value) {
              const float r = fmaxf(z + __builtin_amdgcn_exp2f(-t2), 1e-6f);
              l = am * tv[k] > kThick ? __builtin_amdgcn_logf(r) : l;
            }
            acc[k] = fmaf(c_mw, l, acc[k]);
          }
        }
      };
      if (__builtin_expect(any_thick, 0))
        update(std::true_type{});
      else
        update(std::false_type{});
    } else {
      gptr<float> o = G(p.out) + (size_t)s * nx * ny;
#pragma unroll
      for (int k = 0; k < SC::kPix; ++k) {
        const int r = k / kPerRow, x = tid + (k % kPerRow) * NT, y = y0 + r;
        if (live[k % kPerRow] && x < nx && y < ny)
          stg(o, (unsigned)(__mul24(y, nx) + x), odd_sign * fb[pix.at(r, k % kPerRow)]);
      }
    }
  }

  if constexpr (SOLVE) {
    const float inv_den = p.lp.inv_den, pc = p.lp.phase_coef;
    bool bad = !(fabsf(chk) <= 3.40282347e38f);
    if constexpr (GR > 1) {
      // the groups' projection sums meet in LDS (each in its own region, [row][column]), in the
      // order of the groups; group g finishes the rows r with r mod GR = g
      __syncthreads();
#pragma unroll
      for (int k = 0; k < SC::kPix; ++k) {
        const int r = k / kPerRow, x = tid + (k % kPerRow) * NT;
        if (live[k % kPerRow] && x < nx) reinterpret_cast<float*>(raw)[r * nx + x] = acc[k];
      }
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < SC::kPix; ++k) {
      const int r = k / kPerRow, x = tid + (k % kPerRow) * NT, y = y0 + r;
      if (GR > 1 && r % GR != grp) continue;
      if (live[k % kPerRow] && x < nx && y < ny) {
        float sum = acc[k];
        if constexpr (GR > 1) {
          sum = 0.f;
#pragma unroll
          for (int g = 0; g < GR; ++g)
            sum += reinterpret_cast<const float*>(buf + g * region)[r * nx + x];
        }
        float id = inv_den;
        if constexpr (XDEP) id = ldg(G(p.xden), (unsigned)x);
        const float t = fmaf(-sum, id, amax * tv[k] > kThick ? 0.f : tv[k]);
        bad = bad || !(fabsf(t) <= 3.40282347e38f);
        stg(G(p.tau), (unsigned)(__mul24(y, nx) + x), t);
        if (p.phase_out) stg(G(p.phase_out), (unsigned)(__mul24(y, nx) + x), pc * t);
      }
    }
    // one vector store per wave that met a non-finite value (every writer stores 1)
    if (__any(bad) && (tid & 63) == 0 && p.status != nullptr) G(p.status)[0] = 1u;
  }
}

// solve and precondition modes are separate kernels: each is register-allocated for its own path
template <bool B, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_rowinv(
    KArgs a, const ProbDesc* __restrict__ table) {
  EPR_DISPATCH(B, a, table, xcd_remap(blockIdx.x, gridDim.x), (rowinv_body<NT, 1, true, false>), 0);
}
template <bool B, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_rowinv_x(
    KArgs a, const ProbDesc* __restrict__ table) {
  EPR_DISPATCH(B, a, table, xcd_remap(blockIdx.x, gridDim.x), (rowinv_body<NT, 1, true, true>), 0);
}
// x-dependent spectrum with the block-wise preconditioner
template <int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_rowinv_xb(
    KArgs a, const ProbDesc* __restrict__ table) {
  EPR_DISPATCH(false, a, table, xcd_remap(blockIdx.x, gridDim.x),
               (rowinv_body<NT, 1, true, true, true>), 0);
}
template <bool B, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_rowinv_pre(
    KArgs a, const ProbDesc* __restrict__ table) {
  EPR_DISPATCH(B, a, table, xcd_remap(blockIdx.x, gridDim.x), (rowinv_body<NT, 1, false, false>), 0);
}

// GR lines of a row block at once (single problems): GR groups of NT threads, each with its own
// LDS buffers, take the lines in turn.  A row block's lines are a serial chain of LDS transforms
// and barriers, and a small image has few row blocks: 64 workgroups on 256 CUs at 256 rows.  (The
// plans' radices fit any NT >= nx / 4: kRows (nx / 2) / 12 <= nx / 4.)
template <int NT, int GR, bool SOLVE, bool XDEP>
__global__ __launch_bounds__(NT * GR) __attribute__((amdgpu_waves_per_eu(4))) void k_rowinv_g(
    KArgs a, const ProbDesc* __restrict__ table) {
  EPR_DISPATCH(false, a, table, xcd_remap(blockIdx.x, gridDim.x),
               (rowinv_body<NT, GR, SOLVE, XDEP>), 0);
}

template <int NT, int GR>
void launch_rowinv_g(const KArgs& a, int total_blocks, hipStream_t s) {
  const size_t lds = lds_rowinv_groups(a.p, GR);
  const dim3 grid(total_blocks), block(NT * GR);
  if (a.mode != kRowInvSolve)
    hipLaunchKernelGGL((k_rowinv_g<NT, GR, false, false>), grid, block, lds, s, a, a.table);
  else if (a.p.xcol)
    hipLaunchKernelGGL((k_rowinv_g<NT, GR, true, true>), grid, block, lds, s, a, a.table);
  else
    hipLaunchKernelGGL((k_rowinv_g<NT, GR, true, false>), grid, block, lds, s, a, a.table);
}

// single-problem kernels (the block-wise row inverse)
#define EPR_LAUNCH_X(K, a, grid, nt, lds, s)                                                  \
  do {                                                                                       \
    if (nt == 512)                                                                           \
      hipLaunchKernelGGL((K<512>), dim3(grid), dim3(512), lds, s, a, a.table);              \
    else                                                                                     \
      hipLaunchKernelGGL((K<1024>), dim3(grid), dim3(1024), lds, s, a, a.table);            \
  } while (0)

hipError_t launch_rowinv(const KArgs& a, int total_blocks, size_t lds, hipStream_t s, int nt) {
  const bool x = a.table ? a.xdep != 0 : a.p.xcol != nullptr;
  // Several lines at once for a single problem of at most one row block per CU (a workgroup of
  // groups fills one).  256 x 256, 10 lines: 30 -> 17 us; 1024 x 1024, 8 lines, x-dependent:
  // 36 -> 27 us; 90 x 96, 4 lines, preconditioner: 13 -> 7 us.  With more row blocks, or two groups
  // of 512 threads for wider rows, the CUs that hold two blocks run them one after the other and
  // the pass gets slower (1215 x 1500, 4 lines: 34 -> 46 us).
  if (!a.table && a.p.nbp == 0 && a.p.nx <= 1024 && a.p.lp.n > 1 && total_blocks <= kRowGroupBlocks) {
    if (a.p.nx <= 512 && a.p.lp.n > 4)
      launch_rowinv_g<128, 8>(a, total_blocks, s);
    else if (a.p.lp.n > 2)
      launch_rowinv_g<256, 4>(a, total_blocks, s);
    else
      launch_rowinv_g<256, 2>(a, total_blocks, s);
    return hipGetLastError();
  }
  if (a.mode == kRowInvSolve && !a.table && a.p.xcol && a.p.nbp > 0)
    EPR_LAUNCH_X(k_rowinv_xb, a, total_blocks, nt, lds, s);
  else if (a.mode == kRowInvSolve && x)
    EPR_LAUNCH_SC(k_rowinv_x, a, total_blocks, nt, lds, s);
  else if (a.mode == kRowInvSolve)
    EPR_LAUNCH_SC(k_rowinv, a, total_blocks, nt, lds, s);
  else
    EPR_LAUNCH_SC(k_rowinv_pre, a, total_blocks, nt, lds, s);
  return hipGetLastError();
}


hipError_t set_rowinv_attributes() {
  const void* const fns[] = {EPR_SC_FNS(k_rowinv), EPR_SC_FNS(k_rowinv_pre), EPR_SC_FNS(k_rowinv_x),
                             (const void*)k_rowinv_xb<512>, (const void*)k_rowinv_xb<1024>,
#define EPR_G_FNS(NT, GR)                                   \
  (const void*)k_rowinv_g<NT, GR, true, false>,             \
      (const void*)k_rowinv_g<NT, GR, true, true>,          \
      (const void*)k_rowinv_g<NT, GR, false, false>
                             EPR_G_FNS(128, 8), EPR_G_FNS(256, 4), EPR_G_FNS(256, 2)};
#undef EPR_G_FNS
  return allow_dynamic_lds(fns);
}

}  // namespace epr
