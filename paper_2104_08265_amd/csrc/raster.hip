// Rasterisation and scatter adding of depositions (arXiv:2104.08265 Sec. 2.1.1):
// every depo-plane row becomes a patch of clipped Gaussian bin integrals Q*A_b*B_k
// (or binomial electron counts, Sec. 4.3.1) that is added into its plane's grid.
//
// Scatter adding goes through LDS-privatised tiles of TH x TW cells:
//  1. k_count    - each row counts the tiles its window overlaps (<= 4; wider rows go
//                  to a separate list handled in 64 x 64 chunks with global atomics, k_big)
//                  and keeps the value each increment returns, its slot in that tile's
//                  row list; optionally it marks the impact rows its window reaches;
//  2. k_plan     - each touched tile gets its slice of a row list and a number of work items
//                  (of up to 2^item_shift rows); optionally the rows' tick spans;
//  3. k_fill     - rows are written into their tiles' slices at their slots (plain stores);
//                  tiles of several work items are cleared;
//  4. the tile kernel (rastermean.hip for the mean, rasterdraw.hip for drawn counts) - persistent
//                  blocks take work items from striped queues (next_item) and, in step, groups
//                  of consecutive tiles to clear; a work item accumulates its rows' in-tile
//                  sub-patches and then writes the tile: plain stores when the tile has one
//                  item, global atomic adds when a crowded tile was split across items (those
//                  tiles are cleared first by k_fill); a group's tiles that no row touches
//                  are cleared with plain stores, so the grid needs no separate clearing.
// Window bounds are formed in FP64 exactly as the oracle forms them, so both sides
// agree on which cells a row touches; fluctuated counts use the deterministic
// Philox + binomial chain of fluct.hpp (this file is compiled with contraction off).
#include <type_traits>

#include "rasterwin.hpp"

namespace wct {

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Erf at the cell edges of [k0, k1) for a window (lo, hi) around mu: edge 0 = max(k0, lo),
// edge n = min(k1, hi), interior edges the integers between.  A cell's weight (the
// Gaussian's integral over its part inside the window) is then 0.5 (e[x+1] - e[x]),
// computed from the same doubles the oracle uses, with one erf per edge.
// Both axes of a patch share one pass over the lanes: the impact edges [b0, b1] first,
// then the tick edges [k0, k1] (a short tick window would leave most lanes idle in a
// pass of its own).
template <int MODE>
__device__ __forceinline__ void edge_fill2(double* __restrict__ ea, int b0, int b1, double mua, double siga,
                                           double loa, double hia, double* __restrict__ eb, int k0, int k1,
                                           double mub, double sigb, double lob, double hib, int lane) {
  const int na = b1 - b0, nb = k1 - k0;
  const double s2a = siga * kSqrt2, s2b = sigb * kSqrt2;
  for (int x = lane; x <= na + 1 + nb; x += 64) {
    const bool a = x <= na;
    const int i = a ? x : x - (na + 1), n = a ? na : nb, c0 = a ? b0 : k0, c1 = a ? b1 : k1;
    const double lo = a ? loa : lob, hi = a ? hia : hib, mu = a ? mua : mub, s2 = a ? s2a : s2b;
    const double edge = i == 0 ? fmax((double)c0, lo) : (i == n ? fmin((double)c1, hi) : (double)(c0 + i));
    const double v = MODE != kModeMean ? det_erf((edge - mu) / s2) : erf((edge - mu) / s2);
    (a ? ea : eb)[i] = v;
  }
}
__device__ __forceinline__ double edge_weight(const double* e, int x) { return 0.5 * (e[x + 1] - e[x]); }

// x / d for 0 <= x < 2^22 without an integer divide (float reciprocal, then corrected).
__device__ __forceinline__ int div_small(int x, int d, float rd) {
  int q = (int)((float)x * rd);
  if (q * d > x) --q;
  else if ((q + 1) * d <= x) ++q;
  return q;
}

// Cells whose count needs the full sampler wait in per-wave queues, one per regime of the
// sampler (inversion, chop-down), so that a batch of 64 runs one regime's code with all
// lanes instead of every wave diverging over both.  Cells whose count follows from the
// cheap tests (p = 0, p = 1, or the exact zero bound) never enter them.
//
// A queue lives in registers: position e (< 128) is held by lane e & 63 in slot e >> 6.
// A push moves each new entry to its lane with one ds_permute per 32-bit word; a run
// takes slot 0 (positions 0..63) and slot 1 moves down.  The queues are emptied at the
// end of every chunk of a row, so a batch shares the row's electron count N (a
// wave-uniform value: the sampler's power loop then runs under scalar control).

__device__ __forceinline__ int lanes_below(uint64_t mask, int lane) {
  return __popcll(mask & ((1ull << lane) - 1ull));
}

__device__ __forceinline__ uint32_t lo32(double v) { return (uint32_t)__double_as_longlong(v); }
__device__ __forceinline__ uint32_t hi32(double v) { return (uint32_t)((uint64_t)__double_as_longlong(v) >> 32); }
__device__ __forceinline__ double mkd(uint32_t lo, uint32_t hi) {
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ uint32_t permute_to(int lane_dst, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_ds_permute(lane_dst << 2, (int)v);
}

struct RegQueue {
  double p0, u0, p1, u1;  // probability and uniform of the entries in slot 0 / slot 1
  uint32_t d0, d1;        // their tile offsets
  int n;                  // entries (wave-uniform)
};

__device__ __forceinline__ void rq_push(RegQueue& q, bool need, double p, double u, uint32_t dst, int lane) {
  const uint64_t mask = __ballot(need);
  const int cnt = __popcll(mask);
  if (cnt == 0) return;
  // new entries go to positions n .. n+cnt-1; the other lanes fill the rest of the
  // rotation so that every lane sends and receives exactly one value
  const int below = lanes_below(mask, lane);
  const int t = need ? below : cnt + (lane - below);
  const int to = (q.n + t) & 63;
  const double rp = mkd(permute_to(to, lo32(p)), permute_to(to, hi32(p)));
  const double ru = mkd(permute_to(to, lo32(u)), permute_to(to, hi32(u)));
  const uint32_t rd = permute_to(to, dst);
  const int off = (lane - q.n) & 63;
  if (off < cnt) {
    if (((q.n + off) >> 6) == 0) {
      q.p0 = rp;
      q.u0 = ru;
      q.d0 = rd;
    } else {
      q.p1 = rp;
      q.u1 = ru;
      q.d1 = rd;
    }
  }
  q.n += cnt;
}

// Samples slot 0 (lanes below `take`) with regime REGIME, then moves slot 1 down.
template <typename T, int REGIME, typename Add>
__device__ __forceinline__ void rq_run(RegQueue& q, int take, int N, double lfN, int lane, const DetTablesSmall& tb,
                                       const double* __restrict__ lf, Add add) {
  if (lane < take) {
    const int k = binom_regime_draw<REGIME>(N, lfN, q.p0, q.u0, tb, lf);
    if (k) add(q.d0, (T)k);
  }
  q.p0 = q.p1;
  q.u0 = q.u1;
  q.d0 = q.d1;
  q.n -= take;
}

// A cell's outcome of the cheap tests: added at once, queued for its regime, or nothing.
template <typename T, typename Add>
__device__ __forceinline__ void cell_route(RegQueue& qi, RegQueue& qc, int quick, double p, double u, int N,
                                           double lfN, uint32_t dst, int lane, const DetTablesSmall& tb,
                                           const double* __restrict__ lf, Add add) {
  if (quick > 0) add(dst, (T)quick);
  rq_push(qi, quick == -1, p, u, dst, lane);
  if (qi.n >= 64) rq_run<T, 0>(qi, 64, N, lfN, lane, tb, lf, add);
  rq_push(qc, quick == -2, p, u, dst, lane);
  if (qc.n >= 64) rq_run<T, 1>(qc, 64, N, lfN, lane, tb, lf, add);
}

// One wave rasterises the cells [b0, b1) x [k0, k1) of a row; `dst(b, k)` names a cell and
// `add(dst, value)` accumulates a nonzero contribution.  Fluctuated cells are drawn in
// tick pairs: cells (b, 2m), (b, 2m+1) share one Philox4x32-10 block (counter
// b*ceil(N_t/2) + m), words 0-1 for the even tick and 2-3 for the odd one.
template <typename T, int MODE, typename Dst, typename Add>
__device__ __forceinline__ void patch_cells(const RowWin& w, int b0, int b1, int k0, int k1, int nt, uint32_t did,
                                            uint32_t ev, uint32_t plane, uint32_t key0, uint32_t key1,
                                            double* __restrict__ ea, double* __restrict__ eb,
                                            const DetTablesSmall& tb, const double* __restrict__ lf, int lane, Dst dst,
                                            Add add) {
  const int nbr = b1 - b0, nkr = k1 - k0;
  edge_fill2<MODE>(ea, b0, b1, w.u, w.su, w.ulo, w.uhi, eb, k0, k1, w.t, w.st, w.tlo, w.thi, lane);
  wave_sync();
  if (MODE == kModeNormal) {
    // each cell's count from its own normal: no search, no queue
    const int N = __builtin_amdgcn_readfirstlane((int)floor(fmin(w.q + 0.5, 2147483647.0)));
    if (N > 0) {
      const int j0 = k0 >> 1, np = ((k1 - 1) >> 1) - j0 + 1;
      const uint32_t half_nt = (uint32_t)((nt + 1) >> 1);
      const float rd = 1.0f / (float)np;
      for (int x = lane; x < nbr * np; x += 64) {
        const int bi = div_small(x, np, rd), pj = x - bi * np;
        const int b = b0 + bi, m = j0 + pj;
        const Philox4 ph = philox4x32_10((uint32_t)b * half_nt + (uint32_t)m, did, ev, plane << 24, key0, key1);
        double ze, zo;
        box_muller_pair(ph, &ze, &zo);
        const double a = edge_weight(ea, bi);
        const int ke = 2 * m, ko = 2 * m + 1;
        if (ke >= k0) {
          const int n = normal_count(N, a * edge_weight(eb, ke - k0), ze);
          if (n > 0) add(dst(b, ke), (T)n);
        }
        if (ko < k1) {
          const int n = normal_count(N, a * edge_weight(eb, ko - k0), zo);
          if (n > 0) add(dst(b, ko), (T)n);
        }
      }
    }
  } else if (MODE == kModeMean) {
    const float rd = 1.0f / (float)nkr;
    for (int x = lane; x < nbr * nkr; x += 64) {
      const int bi = div_small(x, nkr, rd), ki = x - bi * nkr;
      add(dst(b0 + bi, k0 + ki), (T)(w.q * (edge_weight(ea, bi) * edge_weight(eb, ki))));
    }
  } else {
    // the row's electron count, wave-uniform (counts are 32-bit: charges from 2^31 - 1
    // electrons up draw as 2^31 - 1)
    const int N = __builtin_amdgcn_readfirstlane((int)floor(fmin(w.q + 0.5, 2147483647.0)));
    if (N > 0) {
      const double lfN = lfact_of(N, lf, tb);
      RegQueue qi, qc;
      qi.n = 0;
      qc.n = 0;
      const int j0 = k0 >> 1, np = ((k1 - 1) >> 1) - j0 + 1;
      const uint32_t half_nt = (uint32_t)((nt + 1) >> 1);
      const float rd = 1.0f / (float)np;
      const int total = nbr * np;
      for (int base = 0; base < total; base += 64) {
        const int x = base + lane;
        int quick_e = 0, quick_o = 0;
        double pe = 0.0, po = 0.0, ue = 0.0, uo = 0.0;
        uint32_t de = 0, dodd = 0;
        if (x < total) {
          const int bi = div_small(x, np, rd), pj = x - bi * np;
          const int b = b0 + bi, m = j0 + pj;
          const Philox4 ph = philox4x32_10((uint32_t)b * half_nt + (uint32_t)m, did, ev, plane << 24, key0, key1);
          const double a = edge_weight(ea, bi);
          const int ke = 2 * m, ko = 2 * m + 1;
          if (ke >= k0) {
            pe = a * edge_weight(eb, ke - k0);
            ue = uniform53(ph.w0, ph.w1);
            de = dst(b, ke);
            quick_e = binom_quick(N, pe, ue);
          }
          if (ko < k1) {
            po = a * edge_weight(eb, ko - k0);
            uo = uniform53(ph.w2, ph.w3);
            dodd = dst(b, ko);
            quick_o = binom_quick(N, po, uo);
          }
        }
        cell_route<T>(qi, qc, quick_e, pe, ue, N, lfN, de, lane, tb, lf, add);
        cell_route<T>(qi, qc, quick_o, po, uo, N, lfN, dodd, lane, tb, lf, add);
      }
      if (qi.n > 0) rq_run<T, 0>(qi, qi.n, N, lfN, lane, tb, lf, add);
      if (qc.n > 0) rq_run<T, 1>(qc, qc.n, N, lfN, lane, tb, lf, add);
    }
  }
  wave_sync();
}

// Up to three ranges cleared in one launch.
__global__ void k_clear3(int32_t* a, int64_t na, int32_t* b, int64_t nb, int32_t* c, int64_t nc) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < na + nb + nc; i += (int64_t)gridDim.x * blockDim.x)
    *(i < na ? a + i : i < na + nb ? b + (i - na) : c + (i - na - nb)) = 0;
}

__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// 1. tiles per row ---------------------------------------------------------
// A row's slot in a tile's row list is the tile counter's value before its increment,
// kept in rank[4 j + n] (n-th tile of row j, rows of tiles outer), so the list fill
// needs no second pass of atomics.  The block first counts its rows per tile in an LDS
// table (open addressing: 2048 slots for at most 4 x 256 tiles, so every probe sequence
// ends at a free or matching slot) and then makes one global atomic add per distinct
// tile: rows of a shower or a track that share tiles no longer queue on one counter.
constexpr int kCountBlock = 256;
constexpr int kCountSlots = 2048;
// Row flags: the rows of a block mostly belong to one plane and overlap, so they mark a copy
// of its words in LDS (planes of up to 65536 impact rows), which is merged at the end.
// Marking device memory directly, 64 lanes met in the same words (three-plane event
// 117 us, with LDS 19 us).
constexpr int kCountWords = 2048;
template <typename T, int TH, int TW>
__global__ void __launch_bounds__(kCountBlock) k_count(DepoView<T> d, RasterGeom g, double nsigma,
                                                       int32_t* __restrict__ counts, int32_t* __restrict__ rank,
                                                       int32_t* __restrict__ list, int32_t* __restrict__ ctrl,
                                                       uint32_t* __restrict__ bits, int2* __restrict__ hull) {
  static_assert(kCountSlots > 4 * kCountBlock && (kCountSlots & (kCountSlots - 1)) == 0, "count table size");
  __shared__ int32_t s_key[kCountSlots];  // tile index, -1 = free
  __shared__ int32_t s_cnt[kCountSlots];  // rows of this block in the tile, then their first slot
  __shared__ int32_t s_pack[4 * kCountBlock];  // per (thread, n): table slot | (rank in the block) << 11
  __shared__ uint32_t s_bits[kCountWords];
  __shared__ unsigned long long s_plane;  // event * kMaxPlanes + plane of the rows marked in LDS
  constexpr unsigned long long kNone = ~0ull;
  for (int e = threadIdx.x; e < kCountSlots; e += kCountBlock) {
    s_key[e] = -1;
    s_cnt[e] = 0;
  }
  if (bits)
    for (int e = threadIdx.x; e < kCountWords; e += kCountBlock) s_bits[e] = 0;
  if (threadIdx.x == 0) s_plane = kNone;
  __syncthreads();
  const int64_t j = blockIdx.x * (int64_t)kCountBlock + threadIdx.x;
  int nt = 0;
  RowWin w;
  w.ok = false;
  if (j < d.n) w = row_window(d, j, g, nsigma);
  const unsigned long long in_plane = w.ok ? (unsigned long long)w.event * kMaxPlanes + w.plane : kNone;
  if (bits) {
    unsigned long long first = in_plane;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) first = min(first, __shfl_xor(first, o, 64));
    if ((threadIdx.x & 63) == 0 && first != kNone) atomicMin(&s_plane, first);
    __syncthreads();
  }
  if (w.ok) {
    const PlaneGeom& pl = g.pl[w.plane];
    const int tr0 = w.b0 / TH, tr1 = (w.b1 - 1) / TH, tc0 = w.k0 / TW, tc1 = (w.k1 - 1) / TW;
    const bool wide = (tr1 - tr0 + 1) * (tc1 - tc0 + 1) > 4;
    if (bits) {
      // The impact rows this window reaches are marked, 32 to a word.  Test first, so that
      // rows outside the block's plane do not contend.  A wide row, which no tile counts,
      // widens the hulls of its bands itself (these rows are few).
      uint32_t* f = bits + (int64_t)w.event * g.bits_ev + g.bit_off[w.plane];
      for (int wd = w.b0 >> 5; wd <= (w.b1 - 1) >> 5; ++wd) {
        uint32_t m = ~0u;
        if (wd == w.b0 >> 5) m &= ~0u << (w.b0 & 31);
        if (wd == (w.b1 - 1) >> 5) m &= ~0u >> (31 - ((w.b1 - 1) & 31));
        if (in_plane == s_plane && wd < kCountWords)
          atomicOr(&s_bits[wd], m);
        else if ((f[wd] & m) != m)
          atomicOr(&f[wd], m);
      }
      if (wide) {
        int bands_ev = 0;
        for (int q = 0; q < g.n_planes; ++q) bands_ev += g.pl[q].ntr;
        int2* h = hull + (int64_t)w.event * bands_ev + bands_before(g, w.plane);
        for (int tr = tr0; tr <= tr1; ++tr) {
          atomicMax(&h[tr].x, kSpanBase - tc0);
          atomicMax(&h[tr].y, tc1 + 1);
        }
      }
    }
    if (wide) {
      list[4 * d.n - 1 - atomicAdd(&ctrl[kCtrlNBig], 1)] = (int32_t)j;
    } else {
      const int64_t base = (int64_t)w.event * g.ntiles_ev + pl.tile_off;
      for (int tr = tr0; tr <= tr1; ++tr)
        for (int tc = tc0; tc <= tc1; ++tc) {
          const int32_t key = (int32_t)(base + (int64_t)tr * pl.ntc + tc);
          uint32_t h = ((uint32_t)key * 2654435761u) >> 21;  // 11 bits
          for (int probe = 0; probe < kCountSlots; ++probe) {
            const int32_t old = atomicCAS(&s_key[h], -1, key);
            if (old == -1 || old == key) break;
            h = (h + 1) & (kCountSlots - 1);
          }
          const int loc = atomicAdd(&s_cnt[h], 1);
          s_pack[4 * threadIdx.x + nt++] = (int32_t)h | (loc << 11);
        }
    }
  }
  __syncthreads();
  if (bits && s_plane != kNone) {
    uint32_t* f = bits + (int64_t)(s_plane / kMaxPlanes) * g.bits_ev + g.bit_off[s_plane % kMaxPlanes];
    for (int e = threadIdx.x; e < kCountWords; e += kCountBlock) {
      const uint32_t m = s_bits[e];
      if (m && (f[e] & m) != m) atomicOr(&f[e], m);
    }
  }
  for (int e = threadIdx.x; e < kCountSlots; e += kCountBlock) {
    const int c = s_cnt[e];
    if (c > 0) s_cnt[e] = atomicAdd(&counts[s_key[e]], c);
  }
  __syncthreads();
  for (int n = 0; n < nt; ++n) {
    const int32_t pk = s_pack[4 * threadIdx.x + n];
    rank[4 * j + n] = s_cnt[pk & (kCountSlots - 1)] + (pk >> 11);
  }
}

// 2. what the tiles' counts decide, in one launch ------------------------------------
// Blocks [0, tile_blocks): kPlanTiles tiles each.  A touched tile gets a slice of the row
// list and its work items (of up to 2^shift rows).  The slices' order does not matter, so a
// block takes its share of the list and of the items with one atomic add each, where three
// scan launches and one for the items kept tile order (18 us on the three-plane detector).
// The blocks after them, one per band of TH impact rows (one tile row of a plane), with
// spans: the band's tiles that some row reaches (a tile row's count, or a wide row's window)
// form the hull of tile columns [lo, hi]; ticks [TW lo, TW (hi + 1)) hold every nonzero cell
// of the band, so the band's marked rows take that span and its other rows {0, 0}.  The hull
// is kept ({2^30 - lo, hi + 1}) for the tile kernel, which clears only the empty tiles
// inside it: the row transform reads nothing else.
constexpr int kPlanTiles = 1024;

__device__ __forceinline__ int items_of(int c, int shift) { return (c + (1 << shift) - 1) >> shift; }

__device__ __forceinline__ void plan_tiles(int64_t base, const int32_t* __restrict__ counts, int64_t ntiles, int shift,
                                           int32_t* __restrict__ offs, int32_t* __restrict__ item_off,
                                           int32_t* __restrict__ items, int32_t* __restrict__ ctrl) {
  __shared__ int2 s_wave[4];
  __shared__ int2 s_base;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int c[4];
  int2 v = make_int2(0, 0);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int64_t t = base + 4 * threadIdx.x + e;
    c[e] = t < ntiles ? counts[t] : 0;
    v.x += c[e];
    v.y += items_of(c[e], shift);
  }
  int2 incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int ax = __shfl_up(incl.x, o, 64), ay = __shfl_up(incl.y, o, 64);
    if (lane >= o) {
      incl.x += ax;
      incl.y += ay;
    }
  }
  if (lane == 63) s_wave[wv] = incl;
  __syncthreads();
  int2 before = make_int2(incl.x - v.x, incl.y - v.y), all = make_int2(0, 0);
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if (w < wv) {
      before.x += s_wave[w].x;
      before.y += s_wave[w].y;
    }
    all.x += s_wave[w].x;
    all.y += s_wave[w].y;
  }
  if (threadIdx.x == 0 && all.x > 0)
    s_base = make_int2(atomicAdd(&ctrl[kCtrlTotal], all.x), atomicAdd(&ctrl[kCtrlNItems], all.y));
  __syncthreads();
  if (all.x == 0) return;
  int row = s_base.x + before.x, item = s_base.y + before.y;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (c[e] == 0) continue;
    const int64_t t = base + 4 * threadIdx.x + e;
    offs[t] = row;
    item_off[t] = item;
    row += c[e];
    for (const int end = item + items_of(c[e], shift); item < end; ++item) items[item] = (int32_t)t;
  }
}

template <int TH, int TW>
__device__ __forceinline__ void band_spans(const RasterGeom& g, int band, const int32_t* __restrict__ counts,
                                           int bands_ev, const uint32_t* __restrict__ bits, int2* __restrict__ span,
                                           int2* __restrict__ hull) {
  __shared__ int s_lo[4], s_hi[4];
  const int ev = band / bands_ev;
  int tr = band - ev * bands_ev;
  int p = 0;
  while (p + 1 < g.n_planes && tr >= g.pl[p].ntr) tr -= g.pl[p++].ntr;
  const PlaneGeom& pl = g.pl[p];
  const int32_t* cnt = counts + (int64_t)ev * g.ntiles_ev + pl.tile_off + (int64_t)tr * pl.ntc;
  int lo = INT_MAX, hi = -1;
  for (int tc = threadIdx.x; tc < pl.ntc; tc += 256)
    if (cnt[tc] > 0) {
      lo = min(lo, tc);
      hi = max(hi, tc);
    }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = min(lo, __shfl_xor(lo, o, 64));
    hi = max(hi, __shfl_xor(hi, o, 64));
  }
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    s_lo[wv] = lo;
    s_hi[wv] = hi;
  }
  __syncthreads();
  lo = min(min(s_lo[0], s_lo[1]), min(s_lo[2], s_lo[3]));
  hi = max(max(s_hi[0], s_hi[1]), max(s_hi[2], s_hi[3]));
  int2* hb = hull + band;  // [event][band]
  const int2 wide = *hb;   // the wide rows' tile columns, {2^30 - lo, hi + 1} or {0, 0}
  if (wide.y > 0) {
    lo = min(lo, kSpanBase - wide.x);
    hi = max(hi, wide.y - 1);
  }
  __syncthreads();  // every thread has read the wide rows' hull
  if (threadIdx.x == 0) *hb = hi >= 0 ? make_int2(kSpanBase - lo, hi + 1) : make_int2(0, 0);
  const int klo = hi >= 0 ? lo * TW : 0, khi = hi >= 0 ? min((hi + 1) * TW, pl.nt) : 0;
  int2* f = span + (int64_t)ev * g.rows_ev + pl.row_off;
  const uint32_t* fb = bits + (int64_t)ev * g.bits_ev + g.bit_off[p];
  const int b1 = min((tr + 1) * TH, pl.nb);
  for (int b = tr * TH + threadIdx.x; b < b1; b += 256)
    f[b] = (fb[b >> 5] >> (b & 31)) & 1u ? make_int2(kSpanBase - klo, khi) : make_int2(0, 0);
}

template <int TH, int TW>
__global__ void __launch_bounds__(256) k_plan(RasterGeom g, const int32_t* __restrict__ counts, int64_t ntiles,
                                              int shift, int tile_blocks, int32_t* __restrict__ offs,
                                              int32_t* __restrict__ item_off, int32_t* __restrict__ items,
                                              int32_t* __restrict__ ctrl, int bands_ev,
                                              const uint32_t* __restrict__ bits, int2* __restrict__ span,
                                              int2* __restrict__ hull) {
  if ((int)blockIdx.x < tile_blocks)
    plan_tiles((int64_t)blockIdx.x * kPlanTiles, counts, ntiles, shift, offs, item_off, items, ctrl);
  else
    band_spans<TH, TW>(g, (int)blockIdx.x - tile_blocks, counts, bands_ev, bits, span, hull);
}

// 3. rows into tile slices (the first fill_blocks blocks); the others clear the tiles that
// several work items accumulate into, a block's tiles gridDim apart (crowded tiles are
// neighbours) ------------------------------------------------------------------------
constexpr int kSplitBlocks = 1024;
template <typename T, int TH, int TW>
__global__ void __launch_bounds__(256) k_fill(DepoView<T> d, RasterGeom g, double nsigma, int fill_blocks,
                                              const int32_t* __restrict__ offs, const int32_t* __restrict__ rank,
                                              int32_t* __restrict__ list, const int32_t* __restrict__ counts,
                                              int64_t ntiles, int shift, T* __restrict__ grid) {
  if ((int)blockIdx.x >= fill_blocks) {
    __shared__ int s_n;
    __shared__ int64_t s_t[256];
    for (int64_t t0 = (int)blockIdx.x - fill_blocks; t0 < ntiles; t0 += (int64_t)256 * kSplitBlocks) {
      if (threadIdx.x == 0) s_n = 0;
      __syncthreads();
      const int64_t t = t0 + (int64_t)threadIdx.x * kSplitBlocks;
      if (t < ntiles && counts[t] > (1 << shift)) s_t[atomicAdd(&s_n, 1)] = t;
      __syncthreads();
      for (int i = 0; i < s_n; ++i) zero_tile<T, TH, TW>(g, s_t[i], grid);
      __syncthreads();
    }
    return;
  }
  const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (j >= d.n) return;
  const RowWin w = row_window(d, j, g, nsigma);
  if (!w.ok) return;
  const PlaneGeom& pl = g.pl[w.plane];
  const int tr0 = w.b0 / TH, tr1 = (w.b1 - 1) / TH, tc0 = w.k0 / TW, tc1 = (w.k1 - 1) / TW;
  if ((tr1 - tr0 + 1) * (tc1 - tc0 + 1) > 4) return;
  const int64_t base = (int64_t)w.event * g.ntiles_ev + pl.tile_off;
  int n = 0;
  for (int tr = tr0; tr <= tr1; ++tr)
    for (int tc = tc0; tc <= tc1; ++tc) {
      const int64_t t = base + (int64_t)tr * pl.ntc + tc;
      list[offs[t] + rank[4 * j + n++]] = (int32_t)j;
    }
}

// 5. rows wider than 4 tiles: 64 x 64 chunks per wave, straight to global atomics ------
template <typename T, int MODE>
__global__ void __launch_bounds__(256, 3) k_big(DepoView<T> d, RasterGeom g, double nsigma, uint64_t seed,
                                             T* __restrict__ grid, const int32_t* __restrict__ list,
                                             const int32_t* __restrict__ ctrl, const DetTables* __restrict__ tables,
                                             const double* __restrict__ lf) {
  constexpr int NWAVE = 4, CB = 64, CK = 64;
  __shared__ double s_ea[NWAVE][CB + 1];
  __shared__ double s_eb[NWAVE][CK + 1];
  __shared__ DetTablesSmall s_tb;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (MODE == kModeBinomial) {
    for (int x = threadIdx.x; x < 129; x += blockDim.x) s_tb.inv[x] = tables->inv[x];
    for (int x = threadIdx.x; x < 19; x += blockDim.x) s_tb.fact[x] = tables->fact[x];
    __syncthreads();
  }
  const int nbig = ctrl[kCtrlNBig];
  const uint32_t key0 = (uint32_t)seed, key1 = (uint32_t)(seed >> 32);
  for (int r = blockIdx.x; r < nbig; r += gridDim.x) {
    const int64_t j = __builtin_amdgcn_readfirstlane(list[4 * d.n - 1 - r]);
    const RowWin w = row_window(d, j, g, nsigma);
    if (!w.ok) continue;
    const PlaneGeom& pl = g.pl[w.plane];
    T* gp = grid + (int64_t)w.event * g.grid_ev_stride + pl.grid_off;
    const uint32_t did = d.depo_id ? (uint32_t)d.depo_id[j] : (uint32_t)j;
    const int kstart = w.k0 & ~1;  // chunks start on even ticks: a Philox pair never straddles two
    const int ncb = (w.b1 - w.b0 + CB - 1) / CB, nck = (w.k1 - kstart + CK - 1) / CK;
    const int nt = pl.nt;
    auto dst = [&](int b, int k) { return (uint32_t)((int64_t)b * nt + k); };
    auto add = [&](uint32_t o, T v) { atomicAdd(gp + o, v); };
    for (int c = wv; c < ncb * nck; c += NWAVE) {
      const int cb = c / nck, ck = c - (c / nck) * nck;
      const int b0 = w.b0 + cb * CB, b1 = min(b0 + CB, w.b1);
      const int k0 = max(kstart + ck * CK, w.k0), k1 = min(kstart + (ck + 1) * CK, w.k1);
      patch_cells<T, MODE>(w, b0, b1, k0, k1, pl.nt, did, (uint32_t)w.key_event, (uint32_t)w.plane, key0, key1,
                           s_ea[wv], s_eb[wv], s_tb, lf, lane, dst, add);
    }
  }
}

// ---------------------------------------------------------------------------
hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)blocks), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

#define WCT_CHECK_LAUNCH()                  \
  do {                                      \
    hipError_t e_ = hipGetLastError();      \
    if (e_ != hipSuccess) return e_;        \
  } while (0)

// Rows per work item.  An item's time grows with its rows, and the call ends with its last
// block: of items of 256 rows the track event (3e5 rows, 6.5e5 row visits of tiles) has
// 7220 for 1024 blocks and would end 1.47 times later than with the work dealt out evenly
// (items of 64 rows 1.22), an event of 6000 rows on one track 95 items, 23 times (16 rows:
// 2.5).  Smaller items cost more tile writes by atomics.  So: about the rows a CU has in
// 1/64 of the call, between 16 and 256; of the mean raster, whose rows cost a tenth beside the
// same writes, in 1/8 (in 1/64 the track event's mean raster took 1100 us instead of 840).
// n counts all rows of a call: wct_simulate over several sub-batches (more events than
// max_events) rasters only a sub-batch's events at a time, whose rows the host does not know, so
// their items are larger than such events alone would get, and never larger than 256 rows.
static int item_shift(int64_t n, int mode, int n_cu) {
  int s = kItemShiftMin;
  while (s < kItemShiftMax && ((int64_t)(mode == kModeMean ? 8 : 64) * n_cu << s) < n) ++s;
  return s;
}

template <typename T, int TH, int TW>
hipError_t launch_raster_tiles(const DepoView<T>& d, const RasterGeom& g, double nsigma, int mode, uint64_t seed,
                               T* grid, RasterWs ws, const DetTables* tables, const double* lfact, int n_cu,
                               hipStream_t st, ProfHook* prof) {
  const int64_t nt = ws.ntiles;
  if (nt >= INT32_MAX) return hipErrorInvalidValue;  // tile indices and list offsets are int32
  ws.item_shift = item_shift(d.n, mode, n_cu);
  if (prof) prof->begin("raster_bin", st);
  const int bands_ev = bands_before(g, g.n_planes);
  if (ws.span && (!ws.hull || !ws.bits)) return hipErrorInvalidValue;  // spans come with hulls and row flags
  // control words and counts are contiguous
  const int64_t n_clear = kCtrlWords + nt, n_hull = ws.span ? 2 * (int64_t)g.n_events * bands_ev : 0;
  const int64_t n_bits = ws.span ? (int64_t)g.n_events * g.bits_ev : 0;
  const int64_t clear_blocks = (n_clear + n_hull + n_bits + 255) / 256;
  hipLaunchKernelGGL(k_clear3, dim3((unsigned)(clear_blocks < 4096 ? clear_blocks : 4096)), dim3(256), 0, st, ws.ctrl,
                     n_clear, reinterpret_cast<int32_t*>(ws.hull), n_hull, reinterpret_cast<int32_t*>(ws.bits), n_bits);
  WCT_CHECK_LAUNCH();
  if (d.n > 0) {
    hipLaunchKernelGGL((k_count<T, TH, TW>), dim3((unsigned)((d.n + kCountBlock - 1) / kCountBlock)),
                       dim3(kCountBlock), 0, st, d, g, nsigma, ws.counts, ws.rank, ws.list, ws.ctrl,
                       ws.span ? ws.bits : nullptr, ws.hull);
    WCT_CHECK_LAUNCH();
  }
  const int tile_blocks = (int)((nt + kPlanTiles - 1) / kPlanTiles);
  hipLaunchKernelGGL((k_plan<TH, TW>), dim3((unsigned)(tile_blocks + (ws.span ? g.n_events * bands_ev : 0))), dim3(256),
                     0, st, g, ws.counts, nt, ws.item_shift, tile_blocks, ws.offs, ws.item_off, ws.items, ws.ctrl,
                     bands_ev, ws.bits, ws.span, ws.hull);
  WCT_CHECK_LAUNCH();
  if (d.n > 0) {
    const int fill_blocks = (int)((d.n + 255) / 256);
    const int64_t split_blocks = nt < kSplitBlocks ? nt : kSplitBlocks;
    hipLaunchKernelGGL((k_fill<T, TH, TW>), dim3((unsigned)(fill_blocks + split_blocks)), dim3(256), 0, st, d, g, nsigma,
                       fill_blocks, ws.offs, ws.rank, ws.list, ws.counts, nt, ws.item_shift, grid);
    WCT_CHECK_LAUNCH();
  }
  hipError_t e = hipSuccess;
  if (prof) prof->end(st);
  static const char* const kTileName[3] = {"raster_tile_mean", "raster_tile_fluct", "raster_tile_normal"};
  if (prof) prof->begin(kTileName[mode], st);
  if (mode == kModeMean)
    e = launch_tile_mean<T, TH, TW>(d, g, nsigma, grid, ws, n_cu, st);
  else
    e = launch_tile_draw<T, TH, TW>(d, g, nsigma, mode, seed, grid, ws, tables, lfact, n_cu, st);
  if (e != hipSuccess) return e;
  if (prof) prof->end(st);
  if (prof) prof->begin("raster_wide_rows", st);
#define WCT_BIG_LAUNCH(M)                                                                                      \
  hipLaunchKernelGGL((k_big<T, M>), dim3(256), dim3(256), 0, st, d, g, nsigma, seed, grid, ws.list, ws.ctrl, tables, \
                     lfact)
  if (mode == kModeBinomial)
    WCT_BIG_LAUNCH(kModeBinomial);
  else if (mode == kModeNormal)
    WCT_BIG_LAUNCH(kModeNormal);
  else
    WCT_BIG_LAUNCH(kModeMean);
#undef WCT_BIG_LAUNCH
  WCT_CHECK_LAUNCH();
  if (prof) prof->end(st);
  return hipSuccess;
}

template <typename T>
hipError_t launch_raster(const DepoView<T>& d, const RasterGeom& g, double nsigma, int mode, uint64_t seed,
                         T* grid, const RasterWs& ws, const DetTables* tables, const double* lfact, int n_cu,
                         hipStream_t st, ProfHook* prof, int tile) {
  if (mode < kModeMean || mode > kModeNormal) return hipErrorInvalidValue;
  int id = 0;  // index among the variants of type T
  hipError_t e = hipErrorInvalidValue;
#define WCT_TILE_CASE(TT, TH_, TW_, OCC)                                                                    \
  if constexpr (std::is_same<T, TT>::value) {                                                              \
    if (id++ == tile)                                                                                      \
      e = launch_raster_tiles<T, TH_, TW_>(d, g, nsigma, mode, seed, grid, ws, tables, lfact, n_cu,      \
                                                st, prof);                                                  \
  }
  WCT_TILE_VARIANTS(WCT_TILE_CASE)
#undef WCT_TILE_CASE
  return e;
}

template hipError_t launch_raster<float>(const DepoView<float>&, const RasterGeom&, double, int, uint64_t, float*,
                                         const RasterWs&, const DetTables*, const double*, int, hipStream_t,
                                         ProfHook*, int);
template hipError_t launch_raster<double>(const DepoView<double>&, const RasterGeom&, double, int, uint64_t, double*,
                                          const RasterWs&, const DetTables*, const double*, int, hipStream_t,
                                          ProfHook*, int);

// ln(n!) table for the chop-down sampler, filled with the sampler's own det_lfact.
__global__ void k_lfact_table(double* __restrict__ out, int n, const DetTables* __restrict__ tables) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = det_lfact((int64_t)i, *tables);
}
hipError_t launch_lfact_table(double* out, int n, const DetTables* tables, hipStream_t st) {
  hipLaunchKernelGGL(k_lfact_table, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, out, n, tables);
  return hipGetLastError();
}

}  // namespace wct
