// The mean raster's tile kernel (arXiv:2104.08265 Sec. 2.1.1): the charge of a tile is a
// sum of outer products over the rows that reach it,
//     S[b, k] = sum_j (Q_j A_j[b]) B_j[k],
// a contraction over j, so it runs on the matrix cores: a work item's rows are taken 16 at
// a time, their weights are laid into LDS ([row][impact row], [row][tick], zero outside
// the window), and each group of four rows is one FP64 16x16x4 product per 16 x 16 block
// of the tile that any of the four windows reaches.  The tile is summed in registers and
// written from there.
//
// Before, every cell of every window was an LDS atomic add, and those adds were the bound
// (4.3e8 of them at 71% of the LDS atomic peak: 2.87 ms on the three-plane event of 1e5
// depositions, now 0.76 ms, 4.2 TB/s over the 3.17 GB grid).  The products take the whole
// 16 x 16 blocks (about twice the cells), yet only 0.03 ms of matrix time for that event
// (1.0e6 products of 64 cycles); what is left is the weights and the write of the grid.  FP64
// products because the weights are FP64: a cell's sum is rounded once, to the grid's type (relative L2 error of that
// grid 2.7e-8, with FP32 adds 1.2e-7).
#include "erfpoly.hpp"
#include "rasterwin.hpp"

namespace wct {

namespace {

constexpr int kMeanRows = 16;  // rows staged at a time: four per wave
typedef double d4 __attribute__((ext_vector_type(4)));

// LDS stride (doubles) of a staged row of n weights: n rounded so that the strides are an
// odd multiple of 16 doubles (128 bytes): the two rows that half a wave reads lie in the two
// halves of the 64 banks.
constexpr int mean_stride(int n) { return n % 32 == 0 ? n + 16 : n; }

// Blocks per CU: as many as the accumulators (8 registers per 16 x 16 block and wave) leave
// registers for without spilling.
constexpr int mean_blocks(int th, int tw) { return th * tw > 6144 ? 2 : (th * tw > 4096 ? 3 : 4); }

// A group of four rows' weights, one row per sixteen lanes, into LDS: the 16-blocks
// [a0, a1] along rows (into da, times q), then [b0, b1] along ticks (into db).  A weight is
// half the difference of its two edges' values, each edge evaluated once: a lane takes its
// upper edge from the next lane, the last one from the next block's first.  Edges are
// clipped to the window, so they coincide outside it and the weights there are 0.  Both
// axes go through one loop, with one erf in it: its coefficients are then live once.
// Edges beyond the polynomial (windows past 4.2 sigma, or widths next to the rounding of the
// position, whose edges round to several sigma) take the library's erf of the quotient, and
// so do all edges of FP64 grids: a few 1e-16 of an erf are 1e-15 of the weights, which an FP64
// cell shows (relative L2 error 2e-15 against 1e-16) and an FP32 cell does not.
struct AxisWin {
  double lo, hi, mu, s2, inv;  // window, centre, sqrt 2 sigma, 1 / (sqrt 2 sigma)
};
__device__ __attribute__((noinline)) double erf_call(double x) { return erf(x); }
template <typename T>
__device__ __forceinline__ void stage_group(double* __restrict__ da, double* __restrict__ db, int a0, int a1, int b0,
                                            int b1, int ca, int cb, AxisWin u, AxisWin t, double q, int l16) {
  const int na = a1 - a0 + 2, n = na + (b1 - b0 + 2);  // blocks of edges: one more than blocks of cells
  double e = 0.0;
  for (int i = 0; i < n; ++i) {
    const bool second = i >= na;  // uniform
    const int blk = second ? b0 + (i - na) : a0 + i;
    const double c = (double)((second ? cb : ca) + 16 * blk + l16);
    const double d = fmin(fmax(c, second ? t.lo : u.lo), second ? t.hi : u.hi) - (second ? t.mu : u.mu);
    const double x = d * (second ? t.inv : u.inv);
    double v;
    if (sizeof(T) == 8 || wave_any(!(fabs(x) <= kErfPolyEdge)))
      v = erf_call(d / (second ? t.s2 : u.s2));
    else
      v = erf_poly(x);
    const double up = __shfl(l16 == 0 ? v : e, (l16 + 1) & 15, 16);  // lane 15 reads lane 0's next block
    if (i != 0 && i != na) (second ? db : da)[16 * (blk - 1) + l16] = (second ? 0.5 : q * 0.5) * (up - e);
    e = v;
  }
}

}  // namespace

// A block takes work items and clearing groups in step, as the fluctuated tile kernel
// does.  Wave v owns the tile's 16-row blocks v, v + 4, ... (interleaved, so that a window
// of 61 rows occupies all four waves) over all its 16-tick blocks.
template <typename T, int TH, int TW>
__global__ void __launch_bounds__(256, mean_blocks(TH, TW)) k_tile_mean(DepoView<T> d, RasterGeom g, double nsigma, T* __restrict__ grid,
                                                      const int32_t* __restrict__ list,
                                                      const int32_t* __restrict__ offs,
                                                      const int32_t* __restrict__ items,
                                                      const int32_t* __restrict__ item_off,
                                                      const int32_t* __restrict__ counts, int64_t ntiles, int item_shift,
                                                      int32_t* __restrict__ ctrl, const int2* __restrict__ hull) {
  constexpr int R = kMeanRows, RB = TH / 64, CB = TW / 16;
  constexpr int SA = mean_stride(TH), SB = mean_stride(TW);
  static_assert(TH % 64 == 0 && TW % 16 == 0, "a wave takes whole 16 x 16 blocks");
  __shared__ double s_a[R * SA];
  __shared__ double s_b[R * SB];
  __shared__ int4 s_rng[R / 4];  // per group of four rows: first and last 16-blocks along rows and ticks
  __shared__ int s_item;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, l16 = lane & 15, sub = lane >> 4;
  const int zgroup = zero_group(ntiles), nzero = (int)((ntiles + zgroup - 1) / zgroup);
  const int nitems = ctrl[kCtrlNItems];
  bool more_items = true;  // block-uniform
  for (int step = 0;; ++step) {
    if (threadIdx.x == 0) s_item = more_items ? next_item(ctrl, step == 0) : INT_MAX;
    __syncthreads();
    const int item = __builtin_amdgcn_readfirstlane(s_item);
    const int zg = (int)blockIdx.x + step * (int)gridDim.x;  // clearing groups are dealt out evenly
    more_items = item < nitems;
    const bool more_zero = zg < nzero;
    if (!more_items && !more_zero) break;
    __syncthreads();  // every thread has read s_item
    if (more_items) {
      const TileItem w = tile_item<TH, TW>(g, item, items, item_off, offs, counts, item_shift);
      const PlaneGeom& pl = g.pl[w.plane];
      d4 acc[RB][CB];
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int c = 0; c < CB; ++c) acc[i][c] = d4{0.0, 0.0, 0.0, 0.0};
      for (int rc = w.r0; rc < w.r1; rc += R) {
        // wave v stages the group of rows rc + 4 v .. + 3, sixteen lanes per row
        const int slot = 4 * wv + sub, r = rc + slot;
        double q = 0.0;
        AxisWin u{0.0, 0.0, 0.0, 1.0, 1.0}, t{0.0, 0.0, 0.0, 1.0, 1.0};
        int a0 = TH / 16, a1 = -1, b0 = TW / 16, b1 = -1;
        if (r < w.r1) {
          const RowWin rw = row_window(d, (int64_t)list[r], g, nsigma);
          const int bb0 = max(rw.b0, w.tb0), bb1 = min(rw.b1, w.tb0 + w.th);
          const int kk0 = max(rw.k0, w.tk0), kk1 = min(rw.k1, w.tk0 + w.tw);
          if (rw.ok && bb0 < bb1 && kk0 < kk1) {
            q = rw.q;
            u = AxisWin{rw.ulo, rw.uhi, rw.u, rw.su * kSqrt2, 1.0 / (rw.su * kSqrt2)};
            t = AxisWin{rw.tlo, rw.thi, rw.t, rw.st * kSqrt2, 1.0 / (rw.st * kSqrt2)};
            a0 = (bb0 - w.tb0) >> 4;
            a1 = (bb1 - 1 - w.tb0) >> 4;
            b0 = (kk0 - w.tk0) >> 4;
            b1 = (kk1 - 1 - w.tk0) >> 4;
          }
        }
#pragma unroll
        for (int o = 16; o < 64; o <<= 1) {  // the group's blocks: the hull over its four rows
          a0 = min(a0, __shfl_xor(a0, o, 64));
          a1 = max(a1, __shfl_xor(a1, o, 64));
          b0 = min(b0, __shfl_xor(b0, o, 64));
          b1 = max(b1, __shfl_xor(b1, o, 64));
        }
        a0 = __builtin_amdgcn_readfirstlane(a0);
        a1 = __builtin_amdgcn_readfirstlane(a1);
        b0 = __builtin_amdgcn_readfirstlane(b0);
        b1 = __builtin_amdgcn_readfirstlane(b1);
        if (a0 <= a1)
          stage_group<T>(s_a + slot * SA, s_b + slot * SB, a0, a1, b0, b1, w.tb0, w.tk0, u, t, q, l16);
        if (lane == 0) s_rng[wv] = make_int4(a0, a1, b0, b1);
        __syncthreads();
#pragma unroll
        for (int gr = 0; gr < R / 4; ++gr) {
          const int4 rg = s_rng[gr];
          const int ga0 = __builtin_amdgcn_readfirstlane(rg.x), ga1 = __builtin_amdgcn_readfirstlane(rg.y);
          const int gb0 = __builtin_amdgcn_readfirstlane(rg.z), gb1 = __builtin_amdgcn_readfirstlane(rg.w);
          // operand layout of the FP64 16x16x4 product: lane l holds A[l & 15][l >> 4] and
          // B[l >> 4][l & 15]
          double bf[CB];
#pragma unroll
          for (int c = 0; c < CB; ++c)
            if (c >= gb0 && c <= gb1) bf[c] = s_b[(4 * gr + sub) * SB + 16 * c + l16];
#pragma unroll
          for (int i = 0; i < RB; ++i) {
            const int rb = wv + 4 * i;
            if (rb < ga0 || rb > ga1) continue;
            const double af = s_a[(4 * gr + sub) * SA + 16 * rb + l16];
#pragma unroll
            for (int c = 0; c < CB; ++c)
              if (c >= gb0 && c <= gb1) acc[i][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(af, bf[c], acc[i][c], 0, 0, 0);
          }
        }
        __syncthreads();
      }
      // element e of a block's result is row 4 e + (lane >> 4), tick lane & 15
      T* gp = grid + (int64_t)w.ev * g.grid_ev_stride + pl.grid_off;
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int c = 0; c < CB; ++c) {
          const int k = 16 * c + l16;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int b = 16 * (wv + 4 * i) + 4 * e + sub;
            if (b < w.th && k < w.tw) {
              T* dst = gp + (int64_t)(w.tb0 + b) * pl.nt + w.tk0 + k;
              const T v = (T)acc[i][c][e];
              if (w.owned)
                *dst = v;
              else if (v != T(0))
                atomicAdd(dst, v);
            }
          }
        }
    }
    if (more_zero) clear_group<T, TH, TW>(g, zg, zgroup, ntiles, counts, hull, grid);
  }
}

template <typename T, int TH, int TW>
hipError_t launch_tile_mean(const DepoView<T>& d, const RasterGeom& g, double nsigma, T* grid, const RasterWs& ws,
                            int n_cu, hipStream_t st) {
  const dim3 blocks((unsigned)(n_cu * mean_blocks(TH, TW)));
  hipLaunchKernelGGL((k_tile_mean<T, TH, TW>), blocks, dim3(256), 0, st, d, g, nsigma, grid, ws.list, ws.offs, ws.items,
                     ws.item_off, ws.counts, ws.ntiles, ws.item_shift, ws.ctrl, ws.hull);
  return hipGetLastError();
}

#define WCT_MEAN_INST(TT, TH_, TW_, OCC)                                                                              \
  template hipError_t launch_tile_mean<TT, TH_, TW_>(const DepoView<TT>&, const RasterGeom&, double, TT*,             \
                                                     const RasterWs&, int, hipStream_t);
WCT_TILE_VARIANTS(WCT_MEAN_INST)
#undef WCT_MEAN_INST

}  // namespace wct
