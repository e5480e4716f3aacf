// K2: neighbour finder -- step C2 of the tracker definition.
//
// One wave per tile of up to 64 consecutive hits of one row (so every lane
// owns one hit, whatever the row size).  Rows are sorted z-line-major, so the
// candidates any hit of the tile can reach in an adjacent row lie in one
// contiguous run of that row's z-lines: the z-lines covering the tile's
// [z_min - w_z, z_max + w_z] (the same padded window and float32 bin rule the
// per-hit search uses, so every per-hit range is inside the staged run).  The
// run's hits and bin starts are staged in LDS with coalesced loads; a lane
// collects the hits in its two windows as short lists (a byte per hit, its
// place in the run) and then tests the pairs of the two lists.  Tiles whose run
// is larger than the stage, or with more candidates than a list holds, are left
// to a second kernel with a larger stage (a wave takes 20 KB of LDS there), and
// what fits neither searches the rows in global memory.
//
// Bound: vector instruction issue.  A wave runs as long as its longest lane,
// so what counts is that the pair test (20 instructions) runs for the largest
// list of the wave and not for every candidate that any lane passes, and that
// a passing candidate costs one byte store and not a predicated write to each
// of 4 or 8 register slots.  With such slots, loads that could be of either
// memory, and every tile beyond the stage searched in global memory, the pass
// took 2262 us on the 512 uneven chunks (1100 now), 365 us on the 32-orbit
// frame (258), 106 us on the central event (60) and 245 us on one sector of
// 210k clusters (70).
//
// All window tests and the pair deviation use float32 with contraction off, in
// the order the definition writes them, so the argmin is bit-identical to any
// other evaluation of the definition.
#include <algorithm>
#include <type_traits>

#include "device_common.h"

namespace tpc {
namespace {

constexpr int kThreads = 64;             // one wave; one hit per lane
// What a wave stages per adjacent row (hits, bins), the length of its lists and the waves per SIMD it is held to.
// Two sizes (the tuning knob TPC_KNOB_LINK_SLOTS: 4 and 8 for sparse and dense rows), and a third for the tiles that
// fit neither.
template <uint32_t kHits_, uint32_t kBins_, int kLen_, int kWaves_, class Place_>
struct Shape {
  static constexpr uint32_t kHits = kHits_, kBins = kBins_;
  static constexpr int kLen = kLen_, kWaves = kWaves_;
  using Place = Place_;   // a hit's place in the stage
};
using Sparse = Shape<256, 128, 8, 7, uint8_t>;      // 5.7 KB of LDS
using Dense = Shape<256, 256, 12, 6, uint8_t>;      // 6.8 KB
using Large = Shape<640, 512, 32, 1, uint16_t>;     // 20.6 KB

constexpr int kGroup = 6;       // candidates tested at a time (4: +3% on the 32-orbit frame)
constexpr int kRunBins = 3;     // z-lines of at most this many bins are searched as one run (see K5's search)

// The grid of an adjacent row.
struct Grid {
  int ny, nz;
  float y_lo, inv_wy, z_lo, inv_wz;
};

// Bins of a window around (y, z): z-lines iz0..iz1, bins iy0..iy1 of each.
struct Window {
  int iy0, iy1, iz0, iz1;
};
__device__ __forceinline__ Window window_of(const Grid& g, float y, float z, float wy, float wz) {
#pragma clang fp contract(off)
  const float py = wy + kWinPad, pz = wz + kWinPad;
  return Window{bin1(y - py, g.y_lo, g.inv_wy, g.ny), bin1(y + py, g.y_lo, g.inv_wy, g.ny),
                bin1(z - pz, g.z_lo, g.inv_wz, g.nz), bin1(z + pz, g.z_lo, g.inv_wz, g.nz)};
}

// The deviation of hit h from the line through pd and pu.
__device__ __forceinline__ float deviation(float2 h, float2 pd, float2 pu, float t, float rho) {
#pragma clang fp contract(off)
  const float yp = pd.x + t * (pu.x - pd.x);
  const float zp = pd.y + t * (pu.y - pd.y);
  const float ey = h.x - yp, ez = h.y - zp;
  return ey * ey + rho * (ez * ez);
}

// The best pair so far: smallest (deviation, up, down), starting from the largest deviation allowed.
struct Best {
  float dev;
  uint32_t u, d;
};
constexpr uint32_t kNone = 0xFFFFFFFFu;

// ---- staged rows ----
template <class Sh>
struct Stage {
  // the last group of a run reads up to kGroup - 1 entries past it
  float2 yz[2][Sh::kHits + kGroup];
  uint16_t bs[2][Sh::kBins + 2];
  typename Sh::Place list[2][Sh::kLen][kThreads];
};

struct Slice {
  Grid g;
  uint32_t off;     // global sorted position of the first staged hit
  int bofs;         // first staged bin
  bool staged;
};

// The z-lines of adjacent row sr reachable from z in [zmin, zmax] with window half-width wz, staged when they fit.
template <class Sh>
__device__ __forceinline__ Slice stage_row(const DevPtrs& d, uint32_t sr, float zmin, float zmax, float wz, bool stage,
                                           float2* yz, uint16_t* lbs) {
#pragma clang fp contract(off)
  const uint32_t R = d.R;
  const RowConst rc = d.rows[sr % R];
  const SectorConst sc = d.secs[sr / R];
  const uint2 meta = d.row_meta[sr];
  Slice v;
  v.g = Grid{(int)(meta.y & 0xFFFFu), (int)(meta.y >> 16), rc.y_lo, rc.inv_wy, sc.z_lo, sc.inv_wz};
  const uint32_t* bs = d.bin_start + meta.x;
  const float pz = wz + kWinPad;
  const int iz0 = bin1(zmin - pz, v.g.z_lo, v.g.inv_wz, v.g.nz), iz1 = bin1(zmax + pz, v.g.z_lo, v.g.inv_wz, v.g.nz);
  const uint32_t b0 = (uint32_t)(iz0 * v.g.ny), b1 = (uint32_t)((iz1 + 1) * v.g.ny);   // bins [b0, b1), starts [b0, b1]
  const uint32_t s0 = bs[b0], s1 = bs[b1];
  v.off = s0;
  v.bofs = (int)b0;
  v.staged = stage && s1 - s0 <= Sh::kHits && b1 - b0 + 1 <= Sh::kBins;
  if (v.staged) {
    for (uint32_t j = threadIdx.x; j < s1 - s0; j += kThreads) yz[j] = d.syz[s0 + j];
    for (uint32_t j = threadIdx.x; j <= b1 - b0; j += kThreads) lbs[j] = (uint16_t)(bs[b0 + j] - s0);
  }
  return v;
}

// Places of the staged hits within the window of h, ascending, to the lane's
// list; their number (the list holds the first kLen).
template <class Sh>
__device__ __forceinline__ int collect(const Slice& v, const float2* yz, const uint16_t* bs, float2 h, float wy, float wz,
                                       typename Sh::Place (*list)[kThreads]) {
#pragma clang fp contract(off)
  const uint32_t lane = threadIdx.x;
  const Window w = window_of(v.g, h.x, h.y, wy, wz);
  const int ny = v.g.ny;
  int b0 = w.iz0 * ny + w.iy0 - v.bofs;
  const int e = w.iz1 * ny + w.iy1 - v.bofs;
  int b1 = ny <= kRunBins ? e : b0 + (w.iy1 - w.iy0);
  uint32_t q = bs[b0], hi = bs[b1 + 1];
  int n = 0;
  for (;;) {
    while (q >= hi && b1 < e) {
      b0 += ny;
      b1 += ny;
      q = bs[b0];
      hi = bs[b1 + 1];
    }
    if (q >= hi) break;
    float2 c[kGroup];
#pragma unroll
    for (int j = 0; j < kGroup; ++j) c[j] = yz[q + j];
    const uint32_t left = hi - q;
#pragma unroll
    for (int j = 0; j < kGroup; ++j) {
      const bool pass = (uint32_t)j < left & fabsf(c[j].x - h.x) <= wy & fabsf(c[j].y - h.y) <= wz;
      if (pass & n < Sh::kLen) list[n][lane] = (typename Sh::Place)(q + j);
      n += pass ? 1 : 0;
    }
    q += kGroup;
  }
  return n;
}

// ---- rows in global memory ----
struct RowView {
  Grid g;
  const float2* yz;        // the row's hits
  const uint32_t* bs;      // its bin starts (global positions)
  uint32_t off;            // global sorted position of yz[0]
};
__device__ __forceinline__ RowView row_view(const DevPtrs& d, uint32_t sr) {
  const RowConst& rc = d.rows[sr % d.R];
  const SectorConst& sc = d.secs[sr / d.R];
  const uint2 meta = d.row_meta[sr];
  return RowView{Grid{(int)(meta.y & 0xFFFFu), (int)(meta.y >> 16), rc.y_lo, rc.inv_wy, sc.z_lo, sc.inv_wz},
                 d.syz + d.row_off[sr], d.bin_start + meta.x, d.row_off[sr]};
}

// fn(q, (y, z)) for every hit q (relative to v.off) of the bins covering a window around h, ascending.
template <class Fn>
__device__ __forceinline__ void for_window(const RowView& v, float2 h, float wy, float wz, Fn fn) {
  const Window w = window_of(v.g, h.x, h.y, wy, wz);
  for (int iz = w.iz0; iz <= w.iz1; ++iz) {
    const uint32_t hi = v.bs[iz * v.g.ny + w.iy1 + 1] - v.off;
    for (uint32_t q = v.bs[iz * v.g.ny + w.iy0] - v.off; q < hi; ++q) {
      const float2 c = v.yz[q];
      if (fabsf(c.x - h.x) <= wy && fabsf(c.y - h.y) <= wz) fn(q, c);
    }
  }
}

// Links of the hit at sorted position p of row sr, any number of candidates.
__device__ __forceinline__ void link_global(const DevPtrs& d, uint32_t p, uint32_t sr, float rho) {
  const RowConst& rc = d.rows[sr % d.R];
  const RowView dn = row_view(d, sr - 1), up = row_view(d, sr + 1);
  const float2 h = d.syz[p];
  int32_t bu = -1, bd = -1;
  float best = rc.dmax;
  for_window(dn, h, rc.wy_dn, rc.wz_dn, [&](uint32_t qd, float2 pd) {
    for_window(up, h, rc.wy_up, rc.wz_up, [&](uint32_t qu, float2 pu) {
      const float dev = deviation(h, pd, pu, rc.t, rho);
      const int32_t gu = (int32_t)(up.off + qu);
      if (dev < best || (dev == best && (bu < 0 || gu < bu))) {   // down positions ascend
        best = dev;
        bu = gu;
        bd = (int32_t)(dn.off + qd);
      }
    });
  });
  d.up0[p] = bu;
  d.down0[p] = bd;
}

// Minimum over the wave (NaN ignored).
__device__ __forceinline__ float wave_minf(float v) {
  auto step = [&](auto ctrl) {
    const int o = __builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), decltype(ctrl)::value, 0xF, 0xF, false);
    v = fminf(v, __int_as_float(o));
  };
  step(std::integral_constant<int, 0x121>());   // rotations by 1, 2, 4 and 8 lanes in each row of 16
  step(std::integral_constant<int, 0x122>());
  step(std::integral_constant<int, 0x124>());
  step(std::integral_constant<int, 0x128>());
  auto lane = [&](int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
  return fminf(fminf(lane(0), lane(16)), fminf(lane(32), lane(48)));
}

// Links of one tile.  Tiles that do not fit the shape (a run larger than the
// stage, a list longer than its lanes hold) search in global memory, or with
// kRetry are left: false, and nothing is written.
template <class Sh, bool kRetry>
__device__ __forceinline__ bool link_tile(const DevPtrs& d, uint32_t tile, float rho, Stage<Sh>& S) {
  const uint32_t sr = d.tile_sr[tile], R = d.R, row = sr % R;
  const uint32_t a = d.row_off[sr] + (tile - d.tile_off[sr]) * kThreads;
  const uint32_t cnt = min((uint32_t)kThreads, d.row_off[sr + 1] - a);
  const uint32_t lane = threadIdx.x;
  const bool mine = lane < cnt;
  const uint32_t p = a + lane;
  if (row == 0 || row + 1 >= R) {
    if (mine) {
      d.up0[p] = -1;
      d.down0[p] = -1;
    }
    return true;
  }
  const float2 h = mine ? d.syz[p] : make_float2(0.0f, 0.0f);
  const float zmin = wave_minf(mine ? h.y : INFINITY), zmax = -wave_minf(mine ? -h.y : INFINITY);
  // a non-finite or out-of-range z (flagged by K1) has no place in the z-line
  // order: such a tile searches the adjacent rows in global memory
  const bool stage = !__any(mine && !(fabsf(h.y) <= kMaxCoord));
  const RowConst rc = d.rows[row];
  const Slice dn = stage_row<Sh>(d, sr - 1, zmin, zmax, rc.wz_dn, stage, S.yz[0], S.bs[0]);
  const Slice up = stage_row<Sh>(d, sr + 1, zmin, zmax, rc.wz_up, stage, S.yz[1], S.bs[1]);
  __syncthreads();
  bool global = mine;
  Best best{rc.dmax, kNone, kNone};
  if (dn.staged && up.staged) {   // wave-uniform
    const int nu = mine ? collect<Sh>(up, S.yz[1], S.bs[1], h, rc.wy_up, rc.wz_up, S.list[1]) : 0;
    const int nd = nu > 0 ? collect<Sh>(dn, S.yz[0], S.bs[0], h, rc.wy_dn, rc.wz_dn, S.list[0]) : 0;
    global = nu > Sh::kLen || nd > Sh::kLen;
    // four of the upper hits at a time in registers against every lower one
    constexpr int kUp = 4;
    const int pairs_u = global ? 0 : nu, pairs_d = global ? 0 : nd;
    for (int u0 = 0; __any(u0 < pairs_u && pairs_d > 0); u0 += kUp) {
      uint32_t qu[kUp];
      float2 pu[kUp];
#pragma unroll
      for (int k = 0; k < kUp; ++k) {
        const uint32_t q = S.list[1][u0 + k][lane];
        qu[k] = u0 + k < pairs_u ? q : 0u;
      }
#pragma unroll
      for (int k = 0; k < kUp; ++k) pu[k] = S.yz[1][qu[k]];
      for (int kd = 0; __any(kd < pairs_d && u0 < pairs_u); ++kd) {
        const uint32_t q = S.list[0][kd][lane], qd = kd < pairs_d ? q : 0u;
        const float2 pd = S.yz[0][qd];
#pragma unroll
        for (int k = 0; k < kUp; ++k) {
          const float dev = deviation(h, pd, pu[k], rc.t, rho);
          // lower hits ascend, so of two pairs with the same upper hit the first has the smaller lower one
          const bool take = kd < pairs_d & u0 + k < pairs_u & (dev < best.dev | (dev == best.dev & qu[k] < best.u));
          best.dev = take ? dev : best.dev;
          best.u = take ? qu[k] : best.u;
          best.d = take ? qd : best.d;
        }
      }
    }
  }
  if (kRetry && __any(global)) return false;
  if (global) {
    link_global(d, p, sr, rho);
  } else if (mine) {
    d.up0[p] = best.u == kNone ? -1 : (int32_t)(up.off + best.u);
    d.down0[p] = best.u == kNone ? -1 : (int32_t)(dn.off + best.d);
  }
  return true;
}

template <class Sh, bool kRetry>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(Sh::kWaves)))
k_links(DevPtrs d, float rho, uint32_t G) {
  __shared__ Stage<Sh> S;
  // Tiles go to the XCDs (block b runs on XCD b % kXcds) in groups of G
  // consecutive tiles, group g on XCD g % kXcds: the adjacent-row runs that
  // tiles of rows r - 1 and r + 1 both stage are then read through one L2
  // (G = 1: consecutive tiles on consecutive XCDs).
  const uint32_t l = blockIdx.x / kXcds;
  const uint32_t tile = G <= 1 ? blockIdx.x : ((l / G) * kXcds + blockIdx.x % kXcds) * G + l % G;
  if (tile >= d.n_link_tiles) return;
  if (!link_tile<Sh, kRetry>(d, tile, rho, S) && threadIdx.x == 0)
    d.link_retry[atomicAdd(&d.hdr->link_retries, 1u)] = tile;
}

// The tiles that k_links left, with the large stage: dense rows (a chunk of
// 200k clusters has 1300 hits a row, most of them in the third of the drift
// range that its particles reach at the inner rows).
__global__ void __launch_bounds__(kThreads) k_links_large(DevPtrs d, float rho) {
  __shared__ Stage<Large> S;
  const uint32_t n = d.hdr->link_retries;
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    link_tile<Large, false>(d, d.link_retry[i], rho, S);
    __syncthreads();   // the stage is read to the end before the next tile fills it
  }
}

}  // namespace

void launch_links(const DevPtrs& d, uint32_t max_row_hits, hipStream_t s) {
  if (d.n_link_tiles == 0) return;
  // group size: as set, or one contiguous eighth of the tiles per XCD
  const uint32_t n = d.n_link_tiles;
  const uint32_t G = d.k2_group == kLinkGroupEighth ? (n + kXcds - 1) / kXcds : std::max<uint32_t>(1u, d.k2_group);
  const uint64_t groups = (n + (uint64_t)G - 1) / G;
  const uint32_t blocks = G == 1 ? n : (uint32_t)((groups + kXcds - 1) / kXcds * kXcds * G);   // every group slot
  // rows of at most the staged hits always fit, so a tile is left only for a list that overflows: no second launch
  if (max_row_hits <= Dense::kHits) {
    if (d.k2_slots == 4) hipLaunchKernelGGL((k_links<Sparse, false>), dim3(blocks), dim3(kThreads), 0, s, d, d.rho, G);
    else hipLaunchKernelGGL((k_links<Dense, false>), dim3(blocks), dim3(kThreads), 0, s, d, d.rho, G);
    return;
  }
  if (d.k2_slots == 4) hipLaunchKernelGGL((k_links<Sparse, true>), dim3(blocks), dim3(kThreads), 0, s, d, d.rho, G);
  else hipLaunchKernelGGL((k_links<Dense, true>), dim3(blocks), dim3(kThreads), 0, s, d, d.rho, G);
  hipLaunchKernelGGL(k_links_large, dim3(std::min(n, 2048u)), dim3(kThreads), 0, s, d, d.rho);
}

}  // namespace tpc
