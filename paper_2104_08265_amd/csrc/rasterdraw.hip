// The tile kernel of drawn counts (arXiv:2104.08265 Sec. 4.3.1): binomial electron counts, or
// the binomial's normal approximation.  fluct.hpp defines every count as an FP64 computation
// on the cell's probability and its Philox words.  The kernel takes FP32 estimates of the
// same quantities first (fastdraw.hpp); they decide all but a few cells in a thousand, and the
// defining computation runs for those, 64 at a time.  The counts are the defining ones.
//
// What bounds it: vector instructions (Philox's products, the searches' steps).  Before, every
// cell ran the FP64 searches and the weights the FP64 erf series, and the counts were added
// with floating-point LDS atomics, which MI355X serves at 194 cycles per wave instruction
// where 32-bit integer ones take 5.4 (measured, 256-thread blocks, any address pattern).  A
// tile is therefore summed in 32-bit integers and converted when it is written; an item
// whose electrons could overflow them adds to the grid directly.  Together: three-plane
// event of 1e5 depositions 6.3 -> 2.7 ms (87% of the vector issue slots), two-face showers of 1e6 depositions 37 -> 21 ms
// (93%).
#include "erfpoly.hpp"
#include "fastdraw.hpp"
#include "rasterwin.hpp"

namespace wct {

namespace {

constexpr int kItemRows = 1 << kItemShiftMax;
static_assert(kItemRows - 1 <= (int)kEntryRow, "an entry holds the row's index in the item");
// Cells waiting for a batch of 64, per wave: inversion entries from the bottom, mode-search
// entries from the top (each below 64 before a tick pair's push of at most 128 in all).
constexpr int kWait = 256;
// Cells left undecided: below 64 before a batch adds 64 (binomial) or a tick pair 128 (normal).
// They are kept across items (undecided_entry).
constexpr int kUndecidedBinomial = 128, kUndecidedNormal = 192;
// Electrons of an item up to which its 32-bit tile cannot overflow (the sum is rounded).
constexpr float kTileElectrons = 4.0e9f;

// Waves per block (they share a tile), and blocks per CU: what LDS holds (160 KB), at most
// four (128 vector registers; five waves per SIMD or more spill: 7.6 to 9.4 ms for the
// event that took 6.6).
constexpr int kDrawWaves = 4, kDrawThreads = 64 * kDrawWaves;
template <int MODE, int TH, int TW>
constexpr int draw_blocks() {
  constexpr int wave = 4 * (TH + TW) + (MODE == kModeBinomial ? 8 * kUndecidedBinomial + 8 * kWait : 8 * kUndecidedNormal);
  constexpr int lds = 4 * TH * TW + 4 * kItemRows + kDrawWaves * wave + 128;
  constexpr int n = 163840 / lds;
  return n > 4 ? 4 : n;
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// Everything the kernel takes.  The out-of-line functions below get its address (the kernel
// argument segment), so that calling them costs the kernel no registers.
template <typename T>
struct DrawArgs {
  DepoView<T> d;
  RasterGeom g;
  double nsigma;
  uint32_t key0, key1;
  T* grid;
  const int32_t *list, *offs, *items, *item_off, *counts;
  int64_t ntiles;
  int item_shift;
  int32_t* ctrl;
  const DetTables* tables;
  const double* lf;
  const int2* hull;
};

// x ^ y ^ z, one instruction
__device__ __forceinline__ uint32_t xor3(uint32_t x, uint32_t y, uint32_t z) {
  return __builtin_amdgcn_bitop3_b32(x, y, z, 0x96);
}

// philox4x32_10 (fluct.hpp) with the round keys made by scalar adds where they are used
// (kept across the loop over cells, the compiler spills the 20 of them).
__device__ __forceinline__ Philox4 philox_cell(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                               uint32_t k1) {
  __asm__ volatile("" : "+s"(k0), "+s"(k1));
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
    c0 = xor3((uint32_t)(p1 >> 32), c1, k0);
    c1 = (uint32_t)p1;
    c2 = xor3((uint32_t)(p0 >> 32), c3, k1);
    c3 = (uint32_t)p0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return Philox4{c0, c1, c2, c3};
}

__device__ __forceinline__ float electrons_of(double q) { return (float)floor(fmin(q + 0.5, 2147483647.0)); }

// An undecided cell: the row, and the cell's offset in its tile below the tile's row and
// column modulo 8 (a row of the tile path reaches at most four tiles).
__device__ __forceinline__ uint32_t undecided_tile(int tr, int tc) {
  return ((uint32_t)tr & 7u) << kEntryDstBits | ((uint32_t)tc & 7u) << (kEntryDstBits + 3);
}

// The defining computation of one cell's count (lanes may hold cells of different rows); the
// cell's index in the grid goes to *at.
// Out of line, like the erf series: inlined, the FP64 constants of both cost the loop over
// cells about 470 spilled scalar registers.
template <typename T, int MODE, int TH, int TW>
__device__ __attribute__((noinline)) int exact_count(const DrawArgs<T>* args, uint2 cell, int64_t* at) {
  const DepoView<T>& d = args->d;
  const RasterGeom& g = args->g;
  const DetTables& tb = *args->tables;
  const double* __restrict__ lf = args->lf;
  const int64_t j = cell.x;
  const RowWin w = row_window(d, j, g, args->nsigma);
  const int off = (int)(cell.y & kEntryDst), tr0 = w.b0 / TH, tc0 = w.k0 / TW;
  const int tr = tr0 + (((int)(cell.y >> kEntryDstBits) - tr0) & 7);
  const int tc = tc0 + (((int)(cell.y >> (kEntryDstBits + 3)) - tc0) & 7);
  const int b = tr * TH + off / TW, k = tc * TW + off % TW;
  if (!w.ok || b < w.b0 || b >= w.b1 || k < w.k0 || k >= w.k1) {  // the tick beside a window's end
    *at = 0;
    return 0;
  }
  const PlaneGeom& pl = g.pl[w.plane];
  *at = (int64_t)w.event * g.grid_ev_stride + pl.grid_off + (int64_t)b * pl.nt + k;
  const double s2a = w.su * kSqrt2, s2b = w.st * kSqrt2;
  double e[4];
#pragma unroll 1
  for (int i = 0; i < 4; ++i) {  // one erf in the code
    const double at = (i < 2 ? (double)b : (double)k) + (double)(i & 1);
    const double edge = i == 0 ? fmax(at, w.ulo) : i == 1 ? fmin(at, w.uhi) : i == 2 ? fmax(at, w.tlo) : fmin(at, w.thi);
    const double v = det_erf((edge - (i < 2 ? w.u : w.t)) / (i < 2 ? s2a : s2b));
    e[0] = i == 0 ? v : e[0];
    e[1] = i == 1 ? v : e[1];
    e[2] = i == 2 ? v : e[2];
    e[3] = i == 3 ? v : e[3];
  }
  const double p = (0.5 * (e[1] - e[0])) * (0.5 * (e[3] - e[2]));
  const int N = (int)floor(fmin(w.q + 0.5, 2147483647.0));
  const uint32_t did = d.depo_id ? (uint32_t)d.depo_id[j] : (uint32_t)j;
  const uint32_t half_nt = (uint32_t)((pl.nt + 1) >> 1);
  const Philox4 ph = philox4x32_10((uint32_t)b * half_nt + (uint32_t)(k >> 1), did, (uint32_t)w.key_event,
                                   (uint32_t)w.plane << 24, args->key0, args->key1);
  if (MODE == kModeNormal) {
    double ze, zo;
    box_muller_pair(ph, &ze, &zo);
    return N > 0 ? normal_count(N, p, (k & 1) ? zo : ze) : 0;
  }
  const double u = (k & 1) ? uniform53(ph.w2, ph.w3) : uniform53(ph.w0, ph.w1);
  const int quick = binom_quick(N, p, u);
  if (quick >= 0) return quick;
  return quick == -1 ? binom_regime_draw<0>(N, 0.0, p, u, tb, lf)
                     : binom_regime_draw<1>(N, lfact_of(N, lf, tb), p, u, tb, lf);
}

__device__ __attribute__((noinline)) double det_erf_call(double x) { return det_erf(x); }

// A row's weights on the tile's cells [b0, b1) x [k0, k1) into LDS: impact weights times
// `scale`, tick weights from slot k0 & 1 on (slots of a tick pair side by side, ticks
// outside the window 0).  A lane holds one edge of either axis and takes the upper edge of
// its cell from the next lane, 63 cells a pass.  Edges beyond the polynomial's range (wide
// windows, or widths next to the rounding of the position) take the series.
__device__ __forceinline__ void row_weights(const RowWin& w, int b0, int b1, int k0, int k1, float scale,
                                            float* __restrict__ wa, float* __restrict__ wb, int lane) {
  const int na = b1 - b0, nb = k1 - k0, odd = k0 & 1;
  const double s2a = w.su * kSqrt2, s2b = w.st * kSqrt2, ra = 1.0 / s2a, rb = 1.0 / s2b;
  if (lane == 0) {
    wb[0] = 0.0f;
    wb[(odd + nb - 1) | 1] = 0.0f;
  }
  wave_sync();
  for (int base = 0; base < na + 1 + nb; base += 63) {
    const int x = base + lane;
    const bool a = x <= na;
    const int i = min(a ? x : x - (na + 1), a ? na : nb);
    const double at = (double)((a ? b0 : k0) + i);
    const double edge = fmin(fmax(at, a ? w.ulo : w.tlo), a ? w.uhi : w.thi);
    const double dx = edge - (a ? w.u : w.t), z = dx * (a ? ra : rb);
    double v;
    if (wave_any(!(fabs(z) <= kErfPolyEdge)))
      v = det_erf_call(dx / (a ? s2a : s2b));
    else
      v = erf_poly(z);
    const double up = __shfl_down(v, 1);
    const float wt = (float)(0.5 * (up - v));
    if (lane < 63 && i < (a ? na : nb)) {
      if (a)
        wa[i] = wt * scale;
      else
        wb[odd + i] = wt;
    }
  }
  wave_sync();
}

}  // namespace

// Persistent blocks take work items from striped queues and, in step, a group of tiles to
// clear, whose stores drain while the rows are drawn.  The waves of a block claim the
// item's rows one at a time.  A wave draws a row's cells in tick pairs (cells (b, 2m) and
// (b, 2m + 1) share a Philox block); binomial cells that are not surely 0 wait in LDS until 64
// of one regime are together, whatever their rows, so a batch fills all lanes.
#define WCT_DRAW_ARGS (const DrawArgs<T>*)(const void*)__builtin_amdgcn_kernarg_segment_ptr()
template <typename T, int MODE, int TH, int TW>
__global__ void __launch_bounds__(kDrawThreads, (draw_blocks<MODE, TH, TW>())) k_tile(DrawArgs<T> args) {
  const DepoView<T>& d = args.d;
  const RasterGeom& g = args.g;
  const int32_t* __restrict__ list = args.list;
  const int32_t* __restrict__ counts = args.counts;
  const int64_t ntiles = args.ntiles;
  int32_t* __restrict__ ctrl = args.ctrl;
  T* __restrict__ grid = args.grid;
  constexpr bool BINOM = MODE == kModeBinomial;
  constexpr int NW = kDrawWaves, WAIT = BINOM ? kWait : 1, UND = BINOM ? kUndecidedBinomial : kUndecidedNormal;
  static_assert(TH * TW - 1 <= (int)kEntryDst, "an entry holds the cell's tile offset");
  static_assert(TW % 2 == 0, "tick pairs do not straddle tiles");
  __shared__ uint32_t tile[TH * TW];
  __shared__ float s_a[NW][TH];
  __shared__ alignas(8) float s_b[NW][TW];
  __shared__ uint2 s_wait[NW][WAIT];  // wait_entry
  __shared__ uint2 s_und[NW][UND];
  __shared__ float s_n[kItemRows];
  __shared__ float s_sum[NW];
  __shared__ int s_item, s_row;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint2* const wait = s_wait[wv];
  const int zgroup = zero_group(ntiles), nzero = (int)((ntiles + zgroup - 1) / zgroup);
  const int nitems = ctrl[kCtrlNItems];
  bool more_items = true;  // block-uniform
  int nx = 0;              // undecided cells of this wave, kept across items
  for (int step = 0;; ++step) {
    if (threadIdx.x == 0) s_item = more_items ? next_item(ctrl, step == 0) : INT_MAX;
    __syncthreads();
    const int item = __builtin_amdgcn_readfirstlane(s_item);  // block-uniform: keep it scalar
    const int zg = (int)blockIdx.x + step * (int)gridDim.x;  // clearing groups are dealt out evenly
    more_items = item < nitems;
    const bool more_zero = zg < nzero;
    if (!more_items && !more_zero) break;
    __syncthreads();  // every thread has read s_item
    if (more_items) {
      const TileItem w_ = tile_item<TH, TW>(g, item, args.items, args.item_off, args.offs, counts, args.item_shift);
      const int tb0 = w_.tb0, tk0 = w_.tk0, th = w_.th, tw = w_.tw, r0 = w_.r0, r1 = w_.r1;
      const PlaneGeom& pl = g.pl[w_.plane];
      T* gp = grid + (int64_t)w_.ev * g.grid_ev_stride + pl.grid_off + (int64_t)tb0 * pl.nt + tk0;
      for (int x = threadIdx.x; x < TH * TW; x += kDrawThreads) tile[x] = 0;
      // the rows' electron counts and their sum
      float n = 0.0f;
      for (int x = threadIdx.x; x < r1 - r0; x += kDrawThreads) n += (s_n[x] = electrons_of((double)d.q[list[r0 + x]]));
  #pragma unroll
      for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
      if (lane == 0) s_sum[wv] = n;
      if (threadIdx.x == 0) s_row = r0;
      __syncthreads();
      float sum = 0.0f;
#pragma unroll
      for (int v = 0; v < NW; ++v) sum += s_sum[v];
      const bool direct = sum > kTileElectrons;  // block-uniform
      if (direct && w_.owned) {  // (a split tile is clear already)
        for (int x = threadIdx.x; x < th * TW; x += kDrawThreads)
          if (x % TW < tw) gp[(int64_t)(x / TW) * pl.nt + x % TW] = T(0);
        __threadfence();
        __syncthreads();
      }
      auto add = [&](uint32_t o, int k) {
        if (k <= 0) return;
        if (direct)
          atomicAdd(gp + (int64_t)(o / TW) * pl.nt + o % TW, (T)k);
        else
          atomicAdd(&tile[o], (uint32_t)k);
      };
      // waiting cells of this wave (wave-uniform counts); the undecided ones below `old` are of
      // earlier items, whose tiles are written
      int ni = 0, nc = 0, old = nx;
      const uint32_t tile_bits = undecided_tile(tb0 / TH, tk0 / TW);
      auto leave = [&](bool undecided, uint32_t row, uint32_t dst) {
        const uint64_t mask = __builtin_amdgcn_ballot_w64(undecided);
        if (undecided) s_und[wv][nx + lanes_below(mask)] = make_uint2((uint32_t)list[r0 + (int)row], tile_bits | dst);
        nx += __popcll(mask);
      };
      // runs the regimes that hold at least `least` cells, and undecided ones by 64 before that
      // (they are then below 64 before a batch adds to them)
      auto run = [&](int least) {
        for (;;) {
          if (nx >= 64) {
            nx -= 64;
            wave_sync();
            const uint2 cell = s_und[wv][nx + lane];
            int64_t at;
            const int k = exact_count<T, MODE, TH, TW>(WCT_DRAW_ARGS, cell, &at);
            wave_sync();
            if (nx + lane >= old)
              add(cell.y & kEntryDst, k);
            else if (k > 0)
              atomicAdd(grid + at, (T)k);
            old = min(old, nx);
          } else if (BINOM && ni >= least) {
            const int take = min(ni, 64);
            ni -= take;
            wave_sync();
            const int at = ni + min(lane, take - 1);
            const uint2 q = wait[at];
            int k;
            const bool sure = fast_inversion(s_n[q.x & kEntryRow], entry_p(q.x), entry_u(q.y), &k);
            wave_sync();
            if (lane < take && sure) add(q.y & kEntryDst, k);
            leave(lane < take && !sure, q.x & kEntryRow, q.y & kEntryDst);
          } else if (BINOM && nc >= least) {
            const int take = min(nc, 64);
            wave_sync();
            const int at = WAIT - nc + min(lane, take - 1);
            nc -= take;
            const uint2 q = wait[at];
            int k;
            const bool sure = fast_chopdown(s_n[q.x & kEntryRow], entry_p(q.x), entry_u(q.y), &k);
            wave_sync();
            if (lane < take && sure) add(q.y & kEntryDst, k);
            leave(lane < take && !sure, q.x & kEntryRow, q.y & kEntryDst);
          } else {
            break;
          }
        }
      };
      // the waves claim rows one at a time, so that they finish the item together
      auto claim = [&]() {
        int r = 0;
        if (lane == 0) r = atomicAdd(&s_row, 1);
        return __builtin_amdgcn_readfirstlane(r);
      };
      for (int r = claim(); r < r1; r = claim()) {
        // the row is wave-uniform: a scalar index makes its parameters scalar loads and registers
        const int64_t j = __builtin_amdgcn_readfirstlane(list[r]);
        const RowWin w = row_window(d, j, g, args.nsigma);
        const int b0 = max(w.b0, tb0), b1 = min(w.b1, tb0 + th);
        const int k0 = max(w.k0, tk0), k1 = min(w.k1, tk0 + tw);
        if (!w.ok || b0 >= b1 || k0 >= k1) continue;
        const float N = electrons_of(w.q);
        if (!(N > 0.0f)) continue;
        const uint32_t did = d.depo_id ? (uint32_t)d.depo_id[j] : (uint32_t)j;
        row_weights(w, b0, b1, k0, k1, N, s_a[wv], s_b[wv], lane);
        const float* wa = s_a[wv];
        const float2* wb = reinterpret_cast<const float2*>(s_b[wv]);
        const float rN = 1.0f / N, zero_limit = fast_zero_limit(N);
        const uint32_t ev = (uint32_t)w.key_event, pc = (uint32_t)w_.plane << 24;
        // pairs (bi, pj) of the window, 64 a pass: the position, the Philox counter and the tile
        // offset advance by 64 pairs without a division
        const int m0 = k0 >> 1, np = ((k1 - 1) >> 1) - m0 + 1, total = (b1 - b0) * np;
        const int dq = 64 / np, dr = 64 - dq * np;
        const uint32_t half_nt = (uint32_t)((pl.nt + 1) >> 1);
        int bi = lane / np, pj = lane - bi * np;
        uint32_t ctr = (uint32_t)(b0 + bi) * half_nt + (uint32_t)(m0 + pj);
        uint32_t dst = (uint32_t)((b0 - tb0 + bi) * TW + 2 * (m0 + pj) - tk0);
        const uint32_t row = (uint32_t)(r - r0);
        const uint32_t ctr_step = (uint32_t)dq * half_nt + (uint32_t)dr, ctr_wrap = half_nt - (uint32_t)np;
        const uint32_t dst_step = (uint32_t)(dq * TW + 2 * dr), dst_wrap = (uint32_t)(TW - 2 * np);
        for (int base = 0; base < total; base += 64) {
          const bool in = base + lane < total;
          const Philox4 ph = philox_cell(ctr, did, ev, pc, args.key0, args.key1);
          float a = 0.0f;
          float2 bw = make_float2(0.0f, 0.0f);
          if (in) {
            a = wa[bi];
            bw = wb[pj];
          }
          if constexpr (BINOM) {
            const float mu[2] = {a * bw.x, a * bw.y};
            const uint32_t w[2] = {ph.w0, ph.w2};
            const int left = total - base;  // lanes that hold a pair
            const uint64_t all = left >= 64 ? ~0ull : (1ull << left) - 1ull;
            uint64_t need[2], top[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              need[h] = __builtin_amdgcn_ballot_w64(!(fmaf((float)w[h], 0x1p-32f, mu[h]) < zero_limit)) & all;
              top[h] = __builtin_amdgcn_ballot_w64(mu[h] >= (float)kMuSwitch) & need[h];
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              if (need[h] == 0) continue;
              const uint64_t low = need[h] & ~top[h];
              int at = ni + lanes_below(low);
              if (top[h]) {
                const int up = WAIT - 1 - nc - lanes_below(top[h]);
                at = __builtin_amdgcn_inverse_ballot_w64(top[h]) ? up : at;
              }
              if (__builtin_amdgcn_inverse_ballot_w64(need[h]))
                wait[at] = make_uint2(entry_x(mu[h] * rN, row), entry_y(w[h], dst + h));
              ni += __popcll(low);
              nc += __popcll(top[h]);
            }
            run(64);
          } else {
            float ze, zo;
            const bool ok = fast_normal_pair(ph.w0, ph.w1, ph.w2, &ze, &zo);
            const float mue = a * bw.x, muo = a * bw.y;
            int ke, ko;
            const bool se = fast_normal_count(N, mue, mue * rN, ze, &ke) && ok;
            const bool so = fast_normal_count(N, muo, muo * rN, zo, &ko) && ok;
            if (in && se) add(dst, ke);
            if (in && so) add(dst + 1, ko);
            leave(in && !se, row, dst);
            leave(in && !so, row, dst + 1);
            run(64);
          }
          const bool wrap = pj + dr >= np;
          pj += wrap ? dr - np : dr;
          bi += wrap ? dq + 1 : dq;
          ctr += wrap ? ctr_step + ctr_wrap : ctr_step;
          dst += wrap ? dst_step + dst_wrap : dst_step;
        }
      }
      run(1);
      __syncthreads();
      if (!direct) {
        constexpr int V = 16 / (int)sizeof(T);
        if (w_.owned && tw == TW && pl.nt % V == 0 && (reinterpret_cast<uintptr_t>(gp) & 15) == 0) {
          constexpr int VR = TW / V;  // 16-byte vectors per tile row
          for (int x = threadIdx.x; x < th * VR; x += kDrawThreads) {
            const int rr = x / VR, c = x - (x / VR) * VR;
            const uint32_t* src = &tile[rr * TW + c * V];
            T v[V];
  #pragma unroll
            for (int e = 0; e < V; ++e) v[e] = (T)src[e];
            *reinterpret_cast<float4*>(gp + (int64_t)rr * pl.nt + c * V) = *reinterpret_cast<const float4*>(v);
          }
        } else {
          for (int x = threadIdx.x; x < th * TW; x += kDrawThreads) {
            const int rr = x / TW, c = x - (x / TW) * TW;
            if (c < tw) {
              T* dst = gp + (int64_t)rr * pl.nt + c;
              if (w_.owned)
                *dst = (T)tile[x];
              else if (tile[x] != 0)
                atomicAdd(dst, (T)tile[x]);
            }
          }
        }
      }
      // the tile's stores have been served before another wave adds an undecided cell to it
      __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
    }
    if (more_zero) clear_group<T, TH, TW>(g, zg, zgroup, ntiles, counts, args.hull, grid);
  }
  if (lane < nx) {
    int64_t at;
    const int k = exact_count<T, MODE, TH, TW>(WCT_DRAW_ARGS, s_und[wv][lane], &at);
    if (k > 0) atomicAdd(grid + at, (T)k);
  }
}
#undef WCT_DRAW_ARGS

template <typename T, int TH, int TW>
hipError_t launch_tile_draw(const DepoView<T>& d, const RasterGeom& g, double nsigma, int mode, uint64_t seed, T* grid,
                            const RasterWs& ws, const DetTables* tables, const double* lfact, int n_cu,
                            hipStream_t st) {
  DrawArgs<T> a{};
  a.d = d;
  a.g = g;
  a.nsigma = nsigma;
  a.key0 = (uint32_t)seed;
  a.key1 = (uint32_t)(seed >> 32);
  a.grid = grid;
  a.list = ws.list;
  a.offs = ws.offs;
  a.items = ws.items;
  a.item_off = ws.item_off;
  a.counts = ws.counts;
  a.ntiles = ws.ntiles;
  a.item_shift = ws.item_shift;
  a.ctrl = ws.ctrl;
  a.tables = tables;
  a.lf = lfact;
  a.hull = ws.hull;
#define WCT_DRAW_LAUNCH(M) \
  hipLaunchKernelGGL((k_tile<T, M, TH, TW>), dim3((unsigned)(n_cu * draw_blocks<M, TH, TW>())), dim3(kDrawThreads), 0, st, a)
  if (mode == kModeBinomial)
    WCT_DRAW_LAUNCH(kModeBinomial);
  else
    WCT_DRAW_LAUNCH(kModeNormal);
#undef WCT_DRAW_LAUNCH
  return hipGetLastError();
}

#define WCT_DRAW_INST(TT, TH_, TW_, OCC)                                                                            \
  static_assert(draw_blocks<kModeBinomial, TH_, TW_>() == OCC, "blocks per CU of a tile variant");                   \
  template hipError_t launch_tile_draw<TT, TH_, TW_>(const DepoView<TT>&, const RasterGeom&, double, int, uint64_t, \
                                                     TT*, const RasterWs&, const DetTables*, const double*, int,    \
                                                     hipStream_t);
WCT_TILE_VARIANTS(WCT_DRAW_INST)
#undef WCT_DRAW_INST

}  // namespace wct
