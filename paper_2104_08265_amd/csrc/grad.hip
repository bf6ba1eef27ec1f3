// Per-row gradient gather for the differentiable mode.
//
// Given H = dL/dS (the convolution's adjoint applied to dL/dM), the raster
// S = sum_j Q_j A_j (x) B_j gives, for row j with window cells (b, k),
//   g_Q       = sum H A_b B_k
//   g_t       = Q sum H A_b dB_k/dt          g_sigma_t = Q sum H A_b dB_k/dsigma_t
//   g_p       = Q I sum H dA_b/du B_k       g_sigma_p = Q I sum H dA_b/dsigma_u B_k
// with u = I p, sigma_u = I sigma_p.  For a cell with edges e_lo = max(k, lo),
// e_hi = min(k+1, hi) and z = (e - mu) / sigma, the clipped integral
// w = Phi(z_hi) - Phi(z_lo) has
//   dw/dmu    = -(phi(z_hi) [hi edge free] - phi(z_lo) [lo edge free]) / sigma
//   dw/dsigma = -(z_hi phi(z_hi) [free] - z_lo phi(z_lo) [free]) / sigma,
// an edge clipped to the truncation window (mu +- nsigma sigma) being fixed in z.
//
// One wave per row.  The five sums factor over an impact row b: with the tick sums
// r0, r1, r2 of H B, H dB/dmu, H dB/dsigma they gain A r0, A r1, A r2, dA/dmu r0 and
// dA/dsigma r0.  So a lane keeps the factors of up to three ticks in registers and walks
// down the impact rows (8 or 16 lanes side by side on consecutive ticks, as wastes fewer on the
// window's width), three multiply-adds per cell where the direct sums take ten with two LDS
// reads of three doubles each; the edges' erf and exponential are evaluated once per edge
// instead of twice per cell.  Bound by the latency of H's short rows (49% of the vector issue
// slots, four waves per SIMD; five or more spill and are slower): 1.5e5 rows of 1400 cells
// took 816 us, now 540 us.  Consecutive rows share an XCD's L2.  Sums in FP64, reduced across the wave.
#include "convcommon.hpp"
#include "erfpoly.hpp"
#include "kernels.hpp"

namespace wct {

namespace {

struct AxisD {
  double w, dmu, dsig;
};

constexpr int kGradRows = 128;  // impact rows whose factors wait in LDS at a time
constexpr int kGradTicks = 3;   // ticks per lane at a time
constexpr int kGradAhead = 4;   // impact rows per lane loaded at a time

// (out of line: inlined, its registers cost the kernel a wave per SIMD)
__device__ __attribute__((noinline)) double erf_call(double x) { return erf(x); }

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// The factors of cells c0 .. c0 + n - 1 of an axis.  A lane evaluates one edge and takes the
// upper one of its cell from the next lane, 63 cells a pass.  Edges outside the window are
// clipped to it (their z is then fixed, so they carry no derivative).
template <typename T>
__device__ __forceinline__ void axis_factors(int c0, int n, double mu, double sigma, double lo, double hi,
                                             AxisD* __restrict__ out, int lane) {
  constexpr double inv_sqrt2pi = 0.39894228040143267794, sqrt_half = 0.70710678118654752440;
  const double rs = 1.0 / sigma;
  for (int base = 0; base < n; base += 63) {
    const int x = min(base + lane, n);
    const double kf = (double)(c0 + x);
    const bool below = kf < lo, above = kf > hi;
    const double d = (below ? lo : above ? hi : kf) - mu;
    double z = d * rs;
    // beyond the polynomial (wide windows, or widths next to the rounding of the position)
    const bool wide = !(fabs(z) * sqrt_half <= kErfPolyEdge);
    double e;
    if (sizeof(T) == 8 || __ballot(wide)) {  // FP64 plans: the polynomial's error would show
      z = d / sigma;
      e = erf_call(z * sqrt_half);
    } else {
      e = erf_poly(z * sqrt_half);
    }
    const double phi = below || above ? 0.0 : inv_sqrt2pi * exp(-0.5 * z * z);
    const double zphi = z * phi;
    const double e1 = __shfl_down(e, 1), phi1 = __shfl_down(phi, 1), zphi1 = __shfl_down(zphi, 1);
    if (lane < 63 && base + lane < n) {
      AxisD a;
      a.w = 0.5 * (e1 - e);
      a.dmu = -(phi1 - phi) / sigma;
      a.dsig = -(zphi1 - zphi) / sigma;
      out[base + lane] = a;
    }
  }
}

__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace

template <typename T>
__global__ void __launch_bounds__(256, 4) k_grad_gather(DepoView<T> d, RasterGeom g, double nsigma,
                                                     const T* __restrict__ H, T* __restrict__ gq, T* __restrict__ gt,
                                                     T* __restrict__ gp, T* __restrict__ gst,
                                                     T* __restrict__ gsp) {
  __shared__ AxisD s_a[4][kGradRows];
  __shared__ AxisD s_b[4][16 * kGradTicks];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t j = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * 4 + wv;
  if (j >= d.n) return;
  const int pl_i = d.plane ? d.plane[j] : 0;
  const int ev_id = d.event ? d.event[j] : 0;
  const int ev = ev_id - g.event_base;
  double s0 = 0, s1 = 0, s2 = 0, s3 = 0, s4 = 0;
  double q = 0;
  int I = 1;
  bool ok = pl_i >= 0 && pl_i < g.n_planes && ev_id >= 0 && ev >= 0 && ev < g.n_events;
  if (ok) {
    const PlaneGeom& pl = g.pl[pl_i];
    I = pl.I;
    q = (double)d.q[j];
    const double t = (double)d.t[j], p = (double)d.p[j];
    const double st = (double)d.st[j], sp = (double)d.sp[j];
    ok = q >= 0.0 && st > 0.0 && sp > 0.0 && isfinite(q) && isfinite(t) && isfinite(p) && isfinite(st) &&
         isfinite(sp);
    if (ok) {
      const double u = (double)pl.I * p, su = (double)pl.I * sp;
      const double hu = nsigma * su, ht = nsigma * st;
      const double ulo = u - hu, uhi = u + hu, tlo = t - ht, thi = t + ht;
      const int b0 = (int)fmax(floor(ulo), 0.0), b1 = (int)fmin(ceil(uhi), (double)pl.nb);
      const int k0 = (int)fmax(floor(tlo), 0.0), k1 = (int)fmin(ceil(thi), (double)pl.nt);
      const T* h = H + (int64_t)ev * g.grid_ev_stride + pl.grid_off;
      const int nk = k1 - k0;
      // lanes per impact row: 8 when that covers the window's ticks with less to spare
      const int width = (nk + 7) / 8 * 8 < (nk + 15) / 16 * 16 ? 8 : 16, rows = 64 / width;
      const int lt = lane & (width - 1), lr = lane / width;
      for (int cb = b0; cb < b1; cb += kGradRows) {
        const int nbr = min(kGradRows, b1 - cb);
        axis_factors<T>(cb, nbr, u, su, ulo, uhi, s_a[wv], lane);
        for (int ck = k0; ck < k1; ck += width * kGradTicks) {
          const int nkr = min(width * kGradTicks, k1 - ck);
          axis_factors<T>(ck, nkr, t, st, tlo, thi, s_b[wv], lane);
          wave_fence();
          AxisD B[kGradTicks];
          bool in[kGradTicks];
#pragma unroll
          for (int e = 0; e < kGradTicks; ++e) {
            in[e] = lt + e * width < nkr;
            B[e] = s_b[wv][in[e] ? lt + e * width : 0];
          }
          // kGradAhead rows' values are requested together (one at a time: 650 us)
          for (int b = lr; b < nbr; b += kGradAhead * rows) {
            T hv[kGradAhead][kGradTicks];
#pragma unroll
            for (int a = 0; a < kGradAhead; ++a) {
              const T* hr = h + (int64_t)(cb + min(b + a * rows, nbr - 1)) * pl.nt + ck + lt;
#pragma unroll
              for (int e = 0; e < kGradTicks; ++e) hv[a][e] = in[e] ? hr[e * width] : T(0);
            }
#pragma unroll
            for (int a = 0; a < kGradAhead; ++a) {
              double r0 = 0, r1 = 0, r2 = 0;
#pragma unroll
              for (int e = 0; e < kGradTicks; ++e) {
                const double v = (double)hv[a][e];
                r0 = fma(v, B[e].w, r0);
                r1 = fma(v, B[e].dmu, r1);
                r2 = fma(v, B[e].dsig, r2);
              }
              if (b + a * rows < nbr) {
                const AxisD A = s_a[wv][b + a * rows];
                s0 = fma(A.w, r0, s0);
                s1 = fma(A.w, r1, s1);
                s2 = fma(A.w, r2, s2);
                s3 = fma(A.dmu, r0, s3);
                s4 = fma(A.dsig, r0, s4);
              }
            }
          }
          wave_fence();
        }
      }
    }
  }
  s0 = wave_sum(s0);
  s1 = wave_sum(s1);
  s2 = wave_sum(s2);
  s3 = wave_sum(s3);
  s4 = wave_sum(s4);
  if (lane == 0) {
    gq[j] = (T)s0;
    gt[j] = (T)(q * s1);
    gst[j] = (T)(q * s2);
    gp[j] = (T)(q * I * s3);
    gsp[j] = (T)(q * I * s4);
  }
}

template <typename T>
hipError_t launch_grad_gather(const DepoView<T>& d, const RasterGeom& g, double nsigma, const T* H, T* gq, T* gt,
                              T* gp, T* gst, T* gsp, hipStream_t st) {
  if (d.n <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)((d.n + 3) / 4);
  hipLaunchKernelGGL((k_grad_gather<T>), dim3(blocks), dim3(256), 0, st, d, g, nsigma, H, gq, gt, gp, gst, gsp);
  return hipGetLastError();
}

template hipError_t launch_grad_gather<float>(const DepoView<float>&, const RasterGeom&, double, const float*, float*,
                                              float*, float*, float*, float*, hipStream_t);
template hipError_t launch_grad_gather<double>(const DepoView<double>&, const RasterGeom&, double, const double*,
                                               double*, double*, double*, double*, double*, hipStream_t);

}  // namespace wct
