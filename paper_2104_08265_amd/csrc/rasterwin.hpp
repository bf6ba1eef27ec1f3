// Device code shared by the raster kernels (raster.hip, rastermean.hip): a row's window,
// the tile of an index, and the clearing of tiles no row touches.  Window bounds are
// formed in FP64 exactly as the oracle forms them: files that include this are compiled
// with contraction off.
#pragma once

#include "kernels.hpp"

namespace wct {

struct RowWin {
  double q, u, su, t, st;
  double ulo, uhi, tlo, thi;
  int b0, b1, k0, k1;  // cell ranges clipped to the grid, [b0, b1) x [k0, k1)
  int plane, event;  // event: slot in this call's grids (id - event_base)
  int key_event;     // event id (fluctuation counter word 2)
  bool ok;
};

__device__ __forceinline__ int clamp_idx(double v) {
  v = fmin(fmax(v, -1.0e9), 1.0e9);
  return (int)v;
}

template <typename T>
__device__ __forceinline__ RowWin row_window(const DepoView<T>& d, int64_t j, const RasterGeom& g, double nsigma) {
  RowWin w;
  w.plane = d.plane ? d.plane[j] : 0;
  w.key_event = d.event ? d.event[j] : 0;
  w.event = w.key_event - g.event_base;
  w.ok = w.plane >= 0 && w.plane < g.n_planes && w.key_event >= 0 && w.event >= 0 && w.event < g.n_events;
  if (!w.ok) return w;
  const PlaneGeom& pl = g.pl[w.plane];
  w.q = (double)d.q[j];
  const double p = (double)d.p[j];
  const double sp = (double)d.sp[j];
  w.t = (double)d.t[j];
  w.st = (double)d.st[j];
  w.ok = (w.q >= 0.0) && (w.st > 0.0) && (sp > 0.0) && isfinite(w.q) && isfinite(w.t) && isfinite(p) &&
         isfinite(w.st) && isfinite(sp);
  if (!w.ok) return w;
  w.u = (double)pl.I * p;
  w.su = (double)pl.I * sp;
  const double hu = nsigma * w.su;
  w.ulo = w.u - hu;
  w.uhi = w.u + hu;
  const double ht = nsigma * w.st;
  w.tlo = w.t - ht;
  w.thi = w.t + ht;
  w.b0 = max(clamp_idx(floor(w.ulo)), 0);
  w.b1 = min(clamp_idx(ceil(w.uhi)), pl.nb);
  w.k0 = max(clamp_idx(floor(w.tlo)), 0);
  w.k1 = min(clamp_idx(ceil(w.thi)), pl.nt);
  w.ok = w.b0 < w.b1 && w.k0 < w.k1;
  return w;
}

__device__ __forceinline__ int find_plane(const RasterGeom& g, int tin) {
  int p = 0;
  for (int k = 1; k < g.n_planes; ++k)
    if (tin >= g.pl[k].tile_off) p = k;
  return p;
}

// Writes zeros over tile t of the grid with the block's threads: 16-byte stores when the
// tile's rows start on 16-byte boundaries, element stores otherwise.
template <typename T, int TH, int TW>
__device__ __forceinline__ void zero_tile(const RasterGeom& g, int64_t t, T* __restrict__ grid) {
  constexpr int V = 16 / (int)sizeof(T);
  static_assert(TW % V == 0, "tile width must be a whole number of 16-byte vectors");
  const int ev = (int)(t / g.ntiles_ev);
  const int tin = (int)(t - (int64_t)ev * g.ntiles_ev);
  const PlaneGeom& pl = g.pl[find_plane(g, tin)];
  const int tl = tin - pl.tile_off;
  const int tr = tl / pl.ntc, tc = tl - (tl / pl.ntc) * pl.ntc;
  const int tb0 = tr * TH, tk0 = tc * TW;
  const int th = min(TH, pl.nb - tb0), tw = min(TW, pl.nt - tk0);
  T* gp = grid + (int64_t)ev * g.grid_ev_stride + pl.grid_off + (int64_t)tb0 * pl.nt + tk0;
  if (tw == TW && pl.nt % V == 0 && (reinterpret_cast<uintptr_t>(gp) & 15) == 0) {
    constexpr int VR = TW / V;  // vectors per tile row
    const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int x = threadIdx.x; x < th * VR; x += blockDim.x) {
      const int r = x / VR, c = x - (x / VR) * VR;
      *reinterpret_cast<float4*>(gp + (int64_t)r * pl.nt + c * V) = z;
    }
  } else {
    for (int x = threadIdx.x; x < th * TW; x += blockDim.x) {
      const int r = x / TW, c = x - (x / TW) * TW;
      if (c < tw) gp[(int64_t)r * pl.nt + c] = T(0);
    }
  }
}

// The block's next work item (thread 0 asks): its first one is its own index, the later
// ones come from the queue of its stripe (blocks, like the items of a stripe, go round the
// kQueues queues).  Atomics on one address are served one after the other, 11.5 ns apart
// on MI355X: 1024 blocks popping one shared head took 12 us a round, striped over eight
// lines 1.8 us.  The stripes hold every eighth item, so they end together.
__device__ __forceinline__ int next_item(int32_t* __restrict__ ctrl, bool first) {
  const int x = blockIdx.x % kQueues;
  if (first) return (int)blockIdx.x;
  return (int)gridDim.x + kQueues * atomicAdd(&ctrl[kCtrlHeads + kQueueStride * x], 1) + x;
}

// Tiles per clearing group: kZeroGroup, fewer on small grids so that every block has some.
__device__ __forceinline__ int zero_group(int64_t ntiles) {
  const int64_t each = ntiles / gridDim.x;
  return each < 1 ? 1 : (each < kZeroGroup ? (int)each : kZeroGroup);
}

// Clears the tiles no row touches of group zg (`zgroup` consecutive tiles), empty tiles
// next to each other together.  With band hulls (wct_simulate), an empty tile outside its
// band's hull is left as it is: the row transform reads only inside the hulls.
template <typename T, int TH, int TW>
__device__ __forceinline__ void clear_group(const RasterGeom& g, int zg, int zgroup, int64_t ntiles,
                                            const int32_t* __restrict__ counts, const int2* __restrict__ hull,
                                            T* __restrict__ grid) {
  constexpr int V = 16 / (int)sizeof(T);
  static_assert(TW % V == 0, "tile width must be a whole number of 16-byte vectors");
  static_assert(kZeroGroup < 32, "a group's tiles are the bits of a word");
  const int64_t t0 = (int64_t)zg * zgroup;
  const int n = (int)(ntiles - t0 < zgroup ? ntiles - t0 : zgroup);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nwv = blockDim.x >> 6;
  // every wave looks at the whole group, one tile per lane
  uint32_t empty = (uint32_t)__ballot(lane < n && counts[t0 + (lane < n ? lane : 0)] == 0);
  int x = 0;  // tiles of the group dealt with
  while (empty >> x) {
    // tile x of the group: its band (a tile row of a plane) and column
    const int ev = (int)((t0 + x) / g.ntiles_ev);
    const int tin = (int)(t0 + x - (int64_t)ev * g.ntiles_ev);
    const int p = find_plane(g, tin);
    const PlaneGeom& pl = g.pl[p];
    const int tl = tin - (int)pl.tile_off, tr = tl / pl.ntc, tc = tl - tr * pl.ntc;
    const int in_band = min(n - x, pl.ntc - tc);  // the group's tiles in this band from here on
    uint32_t m = (empty >> x) & ((1u << in_band) - 1u);
    if (hull) {
      const int2 h = hull[(int64_t)ev * bands_before(g, g.n_planes) + bands_before(g, p) + tr];
      const int lo = max(kSpanBase - h.x - tc, 0), hi = min(h.y - tc, in_band);
      m = h.y > 0 && lo < hi ? m & ((1u << hi) - 1u) & ~((1u << lo) - 1u) : 0u;
    }
    while (m) {  // runs of empty tiles
      const int c0 = __builtin_ctz(m);
      const int run = __builtin_ctz(~(m >> c0));
      m &= ~(((1u << run) - 1u) << c0);
      const int tb0 = tr * TH, tk0 = (tc + c0) * TW;
      const int th = min(TH, pl.nb - tb0), tw = min(run * TW, pl.nt - tk0);
      T* gp = grid + (int64_t)ev * g.grid_ev_stride + pl.grid_off + (int64_t)tb0 * pl.nt + tk0;
      if (tw == run * TW && pl.nt % V == 0 && (reinterpret_cast<uintptr_t>(gp) & 15) == 0) {
        const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int r = wv; r < th; r += nwv)
          for (int c = lane; c < tw / V; c += 64) *reinterpret_cast<float4*>(gp + (int64_t)r * pl.nt + c * V) = z;
      } else {
        for (int r = wv; r < th; r += nwv)
          for (int c = lane; c < tw; c += 64) gp[(int64_t)r * pl.nt + c] = T(0);
      }
    }
    x += in_band;
    if (x >= n) break;
  }
}

// One work item of the tile kernels: rows [r0, r1) of the row list on tile t.
struct TileItem {
  int t, ev, plane, tb0, tk0, th, tw;  // tile, its event slot and plane, its cells [tb0, tb0 + th) x [tk0, tk0 + tw)
  int r0, r1;
  bool owned;  // the tile's only item: plain stores, else atomic adds onto the cleared tile
};
template <int TH, int TW>
__device__ __forceinline__ TileItem tile_item(const RasterGeom& g, int item, const int32_t* __restrict__ items,
                                              const int32_t* __restrict__ item_off,
                                              const int32_t* __restrict__ offs,
                                              const int32_t* __restrict__ counts, int item_shift) {
  TileItem w;
  w.t = items[item];
  const int chunk = item - item_off[w.t], rows = counts[w.t];
  w.owned = rows <= 1 << item_shift;
  w.ev = w.t / g.ntiles_ev;
  const int tin = w.t - w.ev * g.ntiles_ev;
  w.plane = find_plane(g, tin);
  const PlaneGeom& pl = g.pl[w.plane];
  const int tl = tin - pl.tile_off;
  const int tr = tl / pl.ntc, tc = tl - (tl / pl.ntc) * pl.ntc;
  w.tb0 = tr * TH;
  w.tk0 = tc * TW;
  w.th = min(TH, pl.nb - w.tb0);
  w.tw = min(TW, pl.nt - w.tk0);
  w.r0 = offs[w.t] + (chunk << item_shift);
  w.r1 = w.r0 + min(1 << item_shift, rows - (chunk << item_shift));
  return w;
}

}  // namespace wct
