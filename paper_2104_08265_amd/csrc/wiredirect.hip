// Pass B as direct sums along wires, an alternative to the wire transforms of conv.hip /
// conv_ct.hip for responses 2K+1 = 21 wires wide (arXiv:2104.08265 Eq. 1; Eq. 2 with the
// tick axis transformed only).  With the response's tick spectrum R^_t[k][i](w_t) (plan
// data, scaled by 1/L_t for the inverse tick transform of pass C),
//
//   M^(w, w_t) = sum_{k=-K..K} sum_{i<I} R^_t[k][i](w_t) S^(I (w + k) + i, w_t),
//
// rows outside the grid being zero: along wires the signal is a correlation with 2K+1
// taps per phase, which the column transforms evaluate through a length-L_w transform
// pair and a product with the full 2D spectrum R~; here it is summed as it stands.
// Work per output: (2K+1) I complex products (FP32: 840 FMAs), against the transforms'
// 10 forward and one inverse transform per (frequency, wire column) plus the read of R~
// (10 complex per output); the direct sum reads only S^ and 21 I coefficients per
// frequency.
#include "convcommon.hpp"

namespace wct {

namespace {

constexpr int kDirectK = kDirectHalfWires;  // response half-width the kernel is compiled for
// WL output wires per lane, 64 WL per block: eight, or four on small launches (direct_lanes).
// A block's ten phases run one after the other, so a launch that cannot fill the chip takes
// a block's time, and halving the block's wires halves it; eight read fewer staged values per
// multiply-add.
template <int WL>
struct DirectTile {
  static constexpr int WT = 64 * WL;                      // output wires per block
  static constexpr int SUBS = WT / kDirectTileWires;      // tiles of the flags per block
  static constexpr int SUB_LANES = 64 / SUBS;
  static constexpr int SUB_SPAN = kDirectTileWires + 2 * kDirectK;  // S^ wires staged per phase and tile
  // LDS stride of one frequency's staged wires of a tile, and of a block's contiguous wires: one
  // pad element every WL wires, so that lanes reading wires WL apart hit distinct banks
  static constexpr int SUB_PSTR = SUB_SPAN + SUB_SPAN / WL + 1;
  static constexpr int SPAN = WT + 2 * kDirectK;
  static constexpr int PSTR = SPAN + SPAN / WL + 1;
};

}  // namespace

// One block: kChunk tick frequencies (one per wave, so a wave's coefficients are
// uniform: scalar loads) x two tiles of kDirectTileWires wires of one (chunk, event).  Phases
// are staged through LDS in two buffers: the next phase's global loads are in flight while
// the current one is summed.  With tile flags the blocks take the tiles that some row
// reaches, two by two, whatever lies between them, and the last blocks the others: bound by
// its multiply-adds, the pass costs what the reached tiles do (16 sparse events, 41% of the
// 256-wire tiles reached: 10.6 -> 7.8 ms; in whole 512-wire blocks, 51%).  A tile no row
// reaches never reads S^, of which pass A writes only what the reached tiles read: beside a
// reached one in a block it is summed over zeros, so that its M^ is exactly 0.
template <typename T, int WL>
__global__ void __launch_bounds__(64 * kChunk) k_colpass_direct(const cx<T>* __restrict__ shat, int64_t shat_ev_stride,
                                                               const cx<T>* __restrict__ rtick, cx<T>* __restrict__ mhat,
                                                               int64_t mhat_ev_stride, int nw, int nphase, int nchunk,
                                                               int ntile, int n_events, WireTiles wt) {
  using D = DirectTile<WL>;
  constexpr int K = kDirectK, NK = 2 * K + 1, SUBS = D::SUBS, SW = kDirectTileWires;
  constexpr int SPAN = D::SUB_SPAN, SUB_PSTR = D::SUB_PSTR, SUB_LANES = D::SUB_LANES, PSTR = SUBS * SUB_PSTR, C = kChunk;
  constexpr int CPV = 16 / (int)sizeof(cx<T>);  // complex values per 16-byte load
  constexpr int VPW = C / CPV;                  // 16-byte loads per staged wire
  constexpr int NE = SUBS * SPAN * VPW, NPT = (NE + 64 * C - 1) / (64 * C);
  using V = typename Vec16<T>::type;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem_raw);  // [2][C][PSTR]
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  const int tile = L % ntile, rest = L / ntile;
  const int ev = rest % n_events, ch = rest / n_events;
  const int tid = (int)threadIdx.x, lane = tid & 63;
  const int f = __builtin_amdgcn_readfirstlane(tid >> 6);  // this wave's frequency in the chunk
  // the block's tiles: the reached ones come first, then the others, each in order
  const int nsub = (nw + SW - 1) / SW;
  int sub[SUBS];
  bool dead = false, last = true;  // no row reaches the tiles; some row reaches the last of them
#pragma unroll
  for (int b = 0; b < SUBS; ++b) sub[b] = SUBS * tile + b;
  if (wt.live) {  // one flag per lane (at most 64 tiles: the launcher checks)
    const bool live = lane < nsub && wt.live[ev * wt.ev_stride + lane];
    const uint64_t m = __ballot(live), below = (1ull << lane) - 1ull;
    const int nlive = __popcll(m);
    dead = SUBS * tile >= nlive;
    last = SUBS * tile + SUBS - 1 < nlive;
    const int place = lane >= nsub ? -1 : live ? __popcll(m & below) : nlive + lane - __popcll(m & below);
#pragma unroll
    for (int b = 0; b < SUBS; ++b) {
      const uint64_t who = __ballot(place == SUBS * tile + b);
      sub[b] = who ? __builtin_ctzll(who) : nsub;
    }
  }
  // first wire of each tile (past the grid, halo included, where there is none)
  int w0s[SUBS];
#pragma unroll
  for (int b = 0; b < SUBS; ++b) w0s[b] = sub[b] < nsub ? sub[b] * SW : nw + K;
  const int lsub = lane / SUB_LANES, w_lane = (lsub == 0 ? w0s[0] : w0s[SUBS - 1]) + WL * (lane % SUB_LANES);
  static_assert(SUBS <= 2, "a lane's tile is the first or the last");
  if (dead) {  // no row reaches the tiles: M^ = 0
    if (wt.skip_dead) return;
    cx<T>* dst = mhat + ev * mhat_ev_stride;
    for (int o = 0; o < WL; ++o) {
      const int w = w_lane + o;
      if (w < nw) dst[(int64_t)w * (nchunk * C) + ch * C + f] = mk(T(0), T(0));
    }
    return;
  }
  const cx<T>* src = shat + ev * shat_ev_stride + (int64_t)ch * nphase * nw * C;
  // the row flags of the staged wires (rows of wires w0 - K .. w0 + SW + K), one bit each
  constexpr int kBitWords = (SPAN * 10 + 31) / 32 + 2;  // up to 10 phases
  __shared__ uint32_t s_bits[SUBS * kBitWords];
  const bool bits = wt.rowbits != nullptr && nphase <= 10;
  auto first_word = [&](int b) { return max(0, w0s[b] - K) * nphase >> 5; };
  if (bits) {
#pragma unroll
    for (int b = 0; b < SUBS; ++b) {
      const int wd0 = first_word(b), wd1 = (min(nw, w0s[b] + SW + K) * nphase + 31) >> 5;
      for (int x = tid; x < wd1 - wd0; x += 64 * C) s_bits[b * kBitWords + x] = wt.rowbits[ev * wt.bits_ev + wd0 + x];
    }
    __syncthreads();
  }
  auto row_live = [&](int b, int w, int i) {
    if (!bits) return b < SUBS - 1 || last;  // (the flags know an unreached tile's rows)
    const int r = w * nphase + i;
    return ((s_bits[b * kBitWords + (r >> 5) - (b == 0 ? first_word(0) : first_word(SUBS - 1))] >> (r & 31)) & 1u) != 0;
  };

  V stage[NPT];
  auto load = [&](int i) {
    const cx<T>* s = src + (int64_t)i * nw * C;
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      const int e = tid + u * 64 * C;
      const int b = e / (SPAN * VPW), w = (b == 0 ? w0s[0] : w0s[SUBS - 1]) - K + e / VPW - b * SPAN;
      V v = {};
      if (e < NE && w >= 0 && w < nw && row_live(b, w, i)) v = *reinterpret_cast<const V*>(s + (int64_t)w * C + (e % VPW) * CPV);
      stage[u] = v;
    }
  };
  auto store = [&](int b) {
    cx<T>* d = lds + b * C * PSTR;
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      const int e = tid + u * 64 * C;
      if (e < NE) {
        const int b = e / (SPAN * VPW), x = e / VPW - b * SPAN, f0 = (e % VPW) * CPV;
#pragma unroll
        for (int q = 0; q < CPV; ++q)
          d[(f0 + q) * PSTR + b * SUB_PSTR + x + x / WL] = mk(stage[u][2 * q], stage[u][2 * q + 1]);
      }
    }
  };

  T ax[WL], ay[WL];
#pragma unroll
  for (int o = 0; o < WL; ++o) ax[o] = ay[o] = T(0);
  load(0);
  store(0);
  __syncthreads();
  for (int i = 0; i < nphase; ++i) {
    if (i + 1 < nphase) load(i + 1);
    const cx<T>* coef = rtick + ((int64_t)(ch * C + f) * nphase + i) * NK;  // uniform: scalar loads
    cx<T> r[NK];
#pragma unroll
    for (int k = 0; k < NK; ++k) r[k] = coef[k];
    // a tile's staged wire x = WL l + j (lane l of the tile, j < WL + 2K) sits at (WL + 1) l + j + j / WL
    const cx<T>* s = lds + (i & 1) * C * PSTR + f * PSTR + lsub * SUB_PSTR + (WL + 1) * (lane % SUB_LANES);
#pragma unroll
    for (int j = 0; j < WL + 2 * K; ++j) {
      const cx<T> v = s[j + j / WL];
#pragma unroll
      for (int o = 0; o < WL; ++o) {
        if (j - o < 0 || j - o > 2 * K) continue;  // output wire w_lane + o, tap k = j - o - K
        const cx<T> c = r[j - o];
        ax[o] = fma(c.x, v.x, ax[o]);
        ax[o] = fma(-c.y, v.y, ax[o]);
        ay[o] = fma(c.x, v.y, ay[o]);
        ay[o] = fma(c.y, v.x, ay[o]);
      }
    }
    if (i + 1 < nphase) store((i + 1) & 1);
    __syncthreads();
  }
  cx<T>* dst = mhat + ev * mhat_ev_stride;
  const int fpad = nchunk * C;
#pragma unroll
  for (int o = 0; o < WL; ++o) {
    const int w = w_lane + o;
    if (w < nw) dst[(int64_t)w * fpad + ch * C + f] = mk(ax[o], ay[o]);  // [w][fpad]
  }
}

// Adjoint of the direct pass: H^(I c + i, w_t) = sum_k conj(R^_t[k][i](w_t)) G^(c - k, w_t)
// (the correlation's transpose; G^ rows outside the wires are zero).  One staged window
// of G^ serves all I phases: each lane keeps its 8 + 2K values in registers and runs the
// 21 taps once per phase with that phase's coefficients.
template <typename T, int WL>
__global__ void __launch_bounds__(64 * kChunk) k_colpass_adj_direct(const cx<T>* __restrict__ ghat,
                                                                   int64_t ghat_ev_stride,
                                                                   const cx<T>* __restrict__ rtick,
                                                                   cx<T>* __restrict__ hhat, int64_t hhat_ev_stride,
                                                                   int nw, int nphase, int nchunk, int ntile,
                                                                   int n_events) {
  using D = DirectTile<WL>;
  constexpr int K = kDirectK, NK = 2 * K + 1, WT = D::WT, SPAN = D::SPAN, PSTR = D::PSTR, C = kChunk;
  constexpr int CPV = 16 / (int)sizeof(cx<T>);
  constexpr int VPW = C / CPV;
  constexpr int NE = SPAN * VPW;
  using V = typename Vec16<T>::type;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem_raw);  // [C][PSTR]
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  const int tile = L % ntile, rest = L / ntile;
  const int ev = rest % n_events, ch = rest / n_events;
  const int w0 = tile * WT;
  const int tid = (int)threadIdx.x, lane = tid & 63;
  const int f = __builtin_amdgcn_readfirstlane(tid >> 6);
  const cx<T>* src = ghat + ev * ghat_ev_stride + (int64_t)ch * nw * C;  // [chunk][wire][C]
  for (int e = tid; e < NE; e += 64 * C) {
    const int w = w0 - K + e / VPW;
    V v = {};
    if (w >= 0 && w < nw) v = *reinterpret_cast<const V*>(src + (int64_t)w * C + (e % VPW) * CPV);
    const int x = e / VPW, f0 = (e % VPW) * CPV;
#pragma unroll
    for (int q = 0; q < CPV; ++q) lds[(f0 + q) * PSTR + x + x / WL] = mk(v[2 * q], v[2 * q + 1]);
  }
  __syncthreads();
  // G^ of wires w0 + WL lane - K + j, j < WL + 2K
  cx<T> g[WL + 2 * K];
  const cx<T>* s = lds + f * PSTR + (WL + 1) * lane;
#pragma unroll
  for (int j = 0; j < WL + 2 * K; ++j) g[j] = s[j + j / WL];
  cx<T>* dst = hhat + ev * hhat_ev_stride + (int64_t)ch * nphase * nw * C;  // [chunk][i][wire][C]
  for (int i = 0; i < nphase; ++i) {
    const cx<T>* coef = rtick + ((int64_t)(ch * C + f) * nphase + i) * NK;  // uniform: scalar loads
    cx<T> r[NK];
#pragma unroll
    for (int k = 0; k < NK; ++k) r[k] = coef[k];
#pragma unroll
    for (int o = 0; o < WL; ++o) {
      // output wire c = w0 + WL lane + o takes G^(c - k) = g[o + K - k], k = -K..K
      T ax = T(0), ay = T(0);
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) {
        const cx<T> c = r[kk], v = g[o + 2 * K - kk];  // conj(c) * v
        ax = fma(c.x, v.x, ax);
        ax = fma(c.y, v.y, ax);
        ay = fma(c.x, v.y, ay);
        ay = fma(-c.y, v.x, ay);
      }
      const int w = w0 + WL * lane + o;
      if (w < nw) dst[((int64_t)i * nw + w) * C + f] = mk(ax, ay);
    }
  }
}

// Output wires per lane of a launch: four below eight blocks of eight per CU (the adjoint,
// whose block stages once, below four).  Blocks of eight against four, us a plane (dense, FP32,
// n events of a plane): forward, 256 wires 1256 blocks 73 and 44, 2512 140 and 81; 600 wires
// 676 52 and 37, 2028 119 and 91, 2704 159 and 119; 800 wires 1564 106 and 99, 3128 187 and 183,
// 4692 268 and 266, 6256 351 and 351; 2400 wires 6255 355 and 354.  With the flags of a sparse
// event eight are ahead on large launches (three planes, 6255 to 9000 blocks, whole call 5825
// against 5870 us).  Adjoint, 256 wires 1256 blocks 69 and 65, 2512 128 and 123; 600 wires 676
// 54 and 46, 1352 98 and 82, 2028 133 and 123; 800 wires 1564 136 and 151, 3128 264 and 293;
// 1000 wires 676 69 and 73, 2028 185 and 194; 2400 wires 560 and 584.  The lines are not where
// every dense plane would put them: a plane whose last 512 wires are at most half there (256,
// 600 wires) pays 1.2 to 1.8 times past them for the lanes it pads, the others at most 6% on
// either side.
static int direct_lanes(int nw, int nchunk, int n_events, int n_cu, int per_cu) {
  const int64_t blocks = (int64_t)nchunk * n_events * ((nw + DirectTile<8>::WT - 1) / DirectTile<8>::WT);
  return blocks < (int64_t)per_cu * n_cu ? 4 : 8;
}

bool colpass_direct_fits(int K) { return K == kDirectK; }

// Dynamic LDS above the default 64 KB for the direct kernels (on the current device).
void wiredirect_init_kernels() {
  const int lim = 160 * 1024 - 1024;
  auto raise = [&](const void* f) { (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lim); };
  raise((const void*)k_colpass_direct<float, 8>);
  raise((const void*)k_colpass_direct<double, 8>);
  raise((const void*)k_colpass_direct<float, 4>);
  raise((const void*)k_colpass_direct<double, 4>);
  raise((const void*)k_colpass_adj_direct<float, 8>);
  raise((const void*)k_colpass_adj_direct<double, 8>);
  raise((const void*)k_colpass_adj_direct<float, 4>);
  raise((const void*)k_colpass_adj_direct<double, 4>);
}

template <typename T>
hipError_t launch_colpass_direct(const cx<T>* shat, int64_t shat_ev_stride, const cx<T>* rtick, cx<T>* mhat,
                                 int64_t mhat_ev_stride, int nw, int nphase, int nchunk, int n_events, int n_cu,
                                 hipStream_t st, const WireTiles& wt) {
  static_assert(kChunk == 4, "one wave per frequency of a chunk");
  if (wt.live && nw > 64 * kDirectTileWires) return hipErrorInvalidValue;  // (plans end at 5120 wires)
  hipError_t e = hipSuccess;
  auto run = [&](auto wl) {
    constexpr int WL = decltype(wl)::value;
    using D = DirectTile<WL>;
    const int ntile = (nw + D::WT - 1) / D::WT;  // blocks per (chunk, event): one or two tiles of the flags each
    const int64_t nblk = (int64_t)nchunk * n_events * ntile;
    if (nblk <= 0) return;
    if (nblk > 0x7fffffff) {
      e = hipErrorInvalidValue;
      return;
    }
    const size_t lds = sizeof(cx<T>) * 2 * kChunk * D::SUBS * D::SUB_PSTR;  // FP64: above 64 KB (wiredirect_init_kernels)
    hipLaunchKernelGGL((k_colpass_direct<T, WL>), dim3((unsigned)nblk), dim3(64 * kChunk), lds, st, shat,
                       shat_ev_stride, rtick, mhat, mhat_ev_stride, nw, nphase, nchunk, ntile, n_events, wt);
    e = hipGetLastError();
  };
  if (direct_lanes(nw, nchunk, n_events, n_cu, 8) == 4)
    run(std::integral_constant<int, 4>());
  else
    run(std::integral_constant<int, 8>());
  return e;
}

// Whether rows [lo, hi) of a plane's row flags hold a set bit, over the range's words first,
// first + step, ...
__device__ __forceinline__ bool any_row(const uint32_t* __restrict__ bits, int lo, int hi, int first, int step) {
  for (int wd = (lo >> 5) + first; wd <= (hi - 1) >> 5; wd += step) {
    uint32_t v = bits[wd];
    if (wd == lo >> 5) v &= ~0u << (lo & 31);
    if (wd == (hi - 1) >> 5) v &= ~0u >> (31 - ((hi - 1) & 31));
    if (v) return true;
  }
  return false;
}

// Latency: a few dependent loads per thread (from the row spans and in three launches, 44 us
// on the three-plane detector).  The first n_events * tiles_ev blocks: one tile of the
// direct pass each; the others: one (event, wire) per thread.
__global__ void __launch_bounds__(256) k_reach(WireTileGeom g, int ntiles, int64_t nwires,
                                               const uint32_t* __restrict__ bits, uint8_t* __restrict__ tiles,
                                               uint8_t* __restrict__ wires) {
  if ((int)blockIdx.x < ntiles) {
    const int ev = blockIdx.x / g.tiles_ev;
    int t = blockIdx.x - ev * g.tiles_ev;
    int p = 0;
    while (p + 1 < g.n_planes && t >= g.tile_off[p + 1]) ++p;
    t -= g.tile_off[p];
    const int wlo = max(0, t * kDirectTileWires - kDirectK);
    const int whi = min(g.nw[p], (t + 1) * kDirectTileWires + kDirectK);
    const bool any = any_row(bits + (int64_t)ev * g.bits_ev + g.bit_off[p], wlo * g.I[p], whi * g.I[p], threadIdx.x, 256);
    const bool live = __syncthreads_or(any) != 0;
    if (threadIdx.x == 0) tiles[blockIdx.x] = live;
    return;
  }
  const int64_t x = ((int64_t)blockIdx.x - ntiles) * 256 + threadIdx.x;
  if (x >= nwires) return;
  const int ev = (int)(x / g.wires_ev);
  int w = (int)(x - (int64_t)ev * g.wires_ev);
  int p = 0;
  while (p + 1 < g.n_planes && w >= g.wire_off[p + 1]) ++p;
  w -= g.wire_off[p];
  const int wlo = max(0, w - g.K[p]), whi = min(g.nw[p], w + g.K[p] + 1);
  wires[x] = any_row(bits + (int64_t)ev * g.bits_ev + g.bit_off[p], wlo * g.I[p], whi * g.I[p], 0, 1);
}

hipError_t launch_reach(const WireTileGeom& g, int n_events, const uint32_t* bits, uint8_t* tiles, uint8_t* wires,
                        hipStream_t st) {
  const int64_t ntiles = (int64_t)n_events * g.tiles_ev, nwires = (int64_t)n_events * g.wires_ev;
  const int64_t blocks = ntiles + (nwires + 255) / 256;
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_reach, dim3((unsigned)blocks), dim3(256), 0, st, g, (int)ntiles, nwires, bits, tiles, wires);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_colpass_adj_direct(const cx<T>* ghat, int64_t ghat_ev_stride, const cx<T>* rtick, cx<T>* hhat,
                                     int64_t hhat_ev_stride, int nw, int nphase, int nchunk, int n_events, int n_cu,
                                     hipStream_t st) {
  hipError_t e = hipSuccess;
  auto run = [&](auto wl) {
    constexpr int WL = decltype(wl)::value;
    using D = DirectTile<WL>;
    const int ntile = (nw + D::WT - 1) / D::WT;
    const int64_t nblk = (int64_t)nchunk * n_events * ntile;
    if (nblk <= 0) return;
    if (nblk > 0x7fffffff) {
      e = hipErrorInvalidValue;
      return;
    }
    hipLaunchKernelGGL((k_colpass_adj_direct<T, WL>), dim3((unsigned)nblk), dim3(64 * kChunk),
                       sizeof(cx<T>) * kChunk * D::PSTR, st, ghat, ghat_ev_stride, rtick, hhat, hhat_ev_stride, nw,
                       nphase, nchunk, ntile, n_events);
    e = hipGetLastError();
  };
  if (direct_lanes(nw, nchunk, n_events, n_cu, 4) == 4)
    run(std::integral_constant<int, 4>());
  else
    run(std::integral_constant<int, 8>());
  return e;
}

#define WCT_DIRECT_INST(T)                                                                                          \
  template hipError_t launch_colpass_adj_direct<T>(const cx<T>*, int64_t, const cx<T>*, cx<T>*, int64_t, int, int,  \
                                                   int, int, int, hipStream_t);                                     \
  template hipError_t launch_colpass_direct<T>(const cx<T>*, int64_t, const cx<T>*, cx<T>*, int64_t, int, int, int, \
                                               int, int, hipStream_t, const WireTiles&);
WCT_DIRECT_INST(float)
WCT_DIRECT_INST(double)
#undef WCT_DIRECT_INST

}  // namespace wct
