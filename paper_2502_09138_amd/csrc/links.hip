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
// to a second kernel with a larger stage (a wave takes 20 KB of LDS there) and
// longer lists, which it fills as often as it takes; a run that is larger than
// that stage too is walked in global memory, with the same lists.
//
// Bound: vector instruction issue.  A wave runs as long as its longest lane,
// so what counts is that the pair test (20 instructions) runs for the largest
// list of the wave and not for every candidate that any lane passes, and that
// a passing candidate costs one byte store and not a predicated write to each
// of 4 or 8 register slots.  With such slots, loads that could be of either
// memory, and every tile beyond the small stage searched in global memory, the
// pass took 2300 us on 512 chunks of 1k to 200k clusters (19M in all; 1140
// now), 373 us on the 32-orbit frame (261), 107 us on the central event (63)
// and 245 us on one sector of 210k clusters (69).
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
// What a wave stages per adjacent row (hits, bins), the length of its lists, the upper hits that it tests together and the
// waves per SIMD it is held to.  Two sizes (the tuning knob TPC_KNOB_LINK_SLOTS: 4 and 8 for sparse and dense rows), and a
// third for the tiles that fit neither.
template <uint32_t kHits_, uint32_t kBins_, int kLen_, int kUp_, int kWaves_, class Place_>
struct Shape {
  static constexpr uint32_t kHits = kHits_, kBins = kBins_;
  static constexpr int kLen = kLen_, kUp = kUp_, kWaves = kWaves_;
  static_assert(kLen % kUp == 0, "the upper list is read in whole groups");
  using Place = Place_;   // a hit's place in the stage, or in its row
};
using Sparse = Shape<256, 128, 8, 4, 7, uint8_t>;      // 5.7 KB of LDS
using Dense = Shape<256, 256, 12, 4, 6, uint8_t>;      // 6.8 KB
using Large = Shape<640, 512, 32, 8, 1, uint16_t>;     // 20.6 KB

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

// Where an adjacent row is read: hits by place, starts of its bins as places.
struct Staged {
  const float2* yz;
  const uint16_t* bs;
  int bofs;         // first staged bin
  __device__ __forceinline__ uint32_t start(int b) const { return bs[b - bofs]; }
};
struct InRow {      // the whole row, in global memory
  const float2* yz;
  const uint32_t* bs;
  uint32_t off;     // global sorted position of yz[0]
  __device__ __forceinline__ uint32_t start(int b) const { return bs[b] - off; }
};

// A lane's walk over the hits of the bins that cover the window of h, in ascending place.
struct Walk {
  uint32_t q, hi;   // of the run of bins [b0, b1]
  int b0, b1, e;    // e: the window's last bin
};
template <class Row>
__device__ __forceinline__ Walk walk_of(const Row& row, const Grid& g, float2 h, float wy, float wz) {
  const Window w = window_of(g, h.x, h.y, wy, wz);
  Walk k;
  k.b0 = w.iz0 * g.ny + w.iy0;
  k.e = w.iz1 * g.ny + w.iy1;
  k.b1 = g.ny <= kRunBins ? k.e : k.b0 + (w.iy1 - w.iy0);
  k.q = row.start(k.b0);
  k.hi = row.start(k.b1 + 1);
  return k;
}
// The next group of hits of the walk: fn(place, pass, hit).  false at its end.
template <class Row, class Fn>
__device__ __forceinline__ bool next_group(Walk& k, const Row& row, int ny, float2 h, float wy, float wz, Fn fn) {
#pragma clang fp contract(off)
  while (k.q >= k.hi && k.b1 < k.e) {
    k.b0 += ny;
    k.b1 += ny;
    k.q = row.start(k.b0);
    k.hi = row.start(k.b1 + 1);
  }
  if (k.q >= k.hi) return false;
  float2 c[kGroup];   // past the run's end: the stage's slack, or the arrays after the hits in the workspace
#pragma unroll
  for (int j = 0; j < kGroup; ++j) c[j] = row.yz[k.q + j];
  const uint32_t left = k.hi - k.q;
#pragma unroll
  for (int j = 0; j < kGroup; ++j) fn(k.q + j, (uint32_t)j < left & fabsf(c[j].x - h.x) <= wy & fabsf(c[j].y - h.y) <= wz);
  k.q += kGroup;
  return true;
}

// The hits within the window of h to the lane's list; their number (the list holds the first kLen).
template <class Sh>
__device__ __forceinline__ int collect(const Staged& row, const Grid& g, float2 h, float wy, float wz,
                                       typename Sh::Place (*list)[kThreads]) {
  const uint32_t lane = threadIdx.x;
  Walk k = walk_of(row, g, h, wy, wz);
  int n = 0;
  while (next_group(k, row, g.ny, h, wy, wz, [&](uint32_t q, bool pass) {
    if (pass & (n < Sh::kLen)) list[n][lane] = (typename Sh::Place)q;
    n += pass ? 1 : 0;
  })) {
  }
  return n;
}
// The next of them, while a whole group still fits the list.
template <class Sh, class Row>
__device__ __forceinline__ int collect_some(Walk& k, const Row& row, const Grid& g, float2 h, float wy, float wz,
                                            typename Sh::Place (*list)[kThreads]) {
  const uint32_t lane = threadIdx.x;
  int n = 0;
  while (n <= Sh::kLen - kGroup && next_group(k, row, g.ny, h, wy, wz, [&](uint32_t q, bool pass) {
    if (pass) list[n][lane] = (typename Sh::Place)q;
    n += pass ? 1 : 0;
  })) {
  }
  return n;
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

// Every pair of the first nd of the lower list and the first nu of the upper one, kUp of the upper hits at a time in
// registers against every lower one.  Called by the whole wave.
template <class Sh, class Row>
__device__ __forceinline__ void test_pairs(const Stage<Sh>& S, const Row& dn, const Row& up, int nd, int nu, float2 h, float t,
                                           float rho, Best& best) {
  constexpr int kUp = Sh::kUp;
  const uint32_t lane = threadIdx.x;
  for (int u0 = 0; __any(u0 < nu && nd > 0); u0 += kUp) {
    uint32_t qu[kUp];
    float2 pu[kUp];
#pragma unroll
    for (int k = 0; k < kUp; ++k) {
      const uint32_t q = S.list[1][u0 + k][lane];
      qu[k] = u0 + k < nu ? q : 0u;
    }
#pragma unroll
    for (int k = 0; k < kUp; ++k) pu[k] = up.yz[qu[k]];
    for (int kd = 0; __any(kd < nd && u0 < nu); ++kd) {
      const uint32_t q = S.list[0][kd][lane], qd = kd < nd ? q : 0u;
      const float2 pd = dn.yz[qd];
#pragma unroll
      for (int k = 0; k < kUp; ++k) {
        const float dev = deviation(h, pd, pu[k], t, rho);
        // lower hits ascend, so of two pairs with the same upper hit the first has the smaller lower one
        const bool take = (kd < nd) & (u0 + k < nu) & ((dev < best.dev) | ((dev == best.dev) & (qu[k] < best.u)));
        best.dev = take ? dev : best.dev;
        best.u = take ? qu[k] : best.u;
        best.d = take ? qd : best.d;
      }
    }
  }
}

// The best pair of the two windows, however many hits they hold: a list of upper hits after the other, and against each
// of them the lower hits a list at a time.  Called by the whole wave.
template <class Sh, class Row>
__device__ __forceinline__ void test_windows(Stage<Sh>& S, const Row& dn, const Row& up, const Grid& gd, const Grid& gu,
                                             bool mine, float2 h, const RowConst& rc, float rho, Best& best) {
  Walk wu{0u, 0u, 0, 0, 0};
  if (mine) wu = walk_of(up, gu, h, rc.wy_up, rc.wz_up);
  for (;;) {
    const int nu = mine ? collect_some<Sh>(wu, up, gu, h, rc.wy_up, rc.wz_up, S.list[1]) : 0;
    if (!__any(nu > 0)) break;   // a walk ends its list early only at its own end
    Walk wd{0u, 0u, 0, 0, 0};
    if (nu > 0) wd = walk_of(dn, gd, h, rc.wy_dn, rc.wz_dn);
    for (;;) {
      const int nd = nu > 0 ? collect_some<Sh>(wd, dn, gd, h, rc.wy_dn, rc.wz_dn, S.list[0]) : 0;
      if (!__any(nd > 0)) break;
      test_pairs(S, dn, up, nd, nu, h, rc.t, rho, best);
    }
  }
}

// A tile: its row, the row's constants and the lane's hit.
struct Tile {
  uint32_t sr, p;   // (sector, row), the lane's sorted position
  bool mine, edge;  // the lane has a hit; the row is the first or the last
};
__device__ __forceinline__ Tile tile_of(const DevPtrs& d, uint32_t tile) {
  Tile t;
  t.sr = d.tile_sr[tile];
  const uint32_t R = d.R, row = t.sr % R;
  const uint32_t a = d.row_off[t.sr] + (tile - d.tile_off[t.sr]) * kThreads;
  t.mine = threadIdx.x < min((uint32_t)kThreads, d.row_off[t.sr + 1] - a);
  t.p = a + threadIdx.x;
  t.edge = row == 0 || row + 1 >= R;
  return t;
}

__device__ __forceinline__ void write_links(const DevPtrs& d, const Tile& t, const Best& best, uint32_t off_up, uint32_t off_dn) {
  if (!t.mine) return;
  d.up0[t.p] = best.u == kNone ? -1 : (int32_t)(off_up + best.u);
  d.down0[t.p] = best.u == kNone ? -1 : (int32_t)(off_dn + best.d);
}

// The two adjacent rows' slices of a tile.
template <class Sh>
__device__ __forceinline__ void stage_tile(const DevPtrs& d, const Tile& t, const RowConst& rc, float2 h, Stage<Sh>& S, Slice& dn,
                                           Slice& up) {
  const float zmin = wave_minf(t.mine ? h.y : INFINITY), zmax = -wave_minf(t.mine ? -h.y : INFINITY);
  // a non-finite or out-of-range z (flagged by K1) has no place in the z-line
  // order: such a tile searches the adjacent rows in global memory
  const bool stage = !__any(t.mine && !(fabsf(h.y) <= kMaxCoord));
  dn = stage_row<Sh>(d, t.sr - 1, zmin, zmax, rc.wz_dn, stage, S.yz[0], S.bs[0]);
  up = stage_row<Sh>(d, t.sr + 1, zmin, zmax, rc.wz_up, stage, S.yz[1], S.bs[1]);
  __syncthreads();
}

// Links of one tile; false, and nothing written, where a run is larger than the stage or a list longer than its lanes hold.
template <class Sh>
__device__ __forceinline__ bool link_tile(const DevPtrs& d, uint32_t tile, float rho, Stage<Sh>& S) {
  const Tile t = tile_of(d, tile);
  Best best{0.0f, kNone, kNone};
  if (t.edge) {
    write_links(d, t, best, 0u, 0u);
    return true;
  }
  const float2 h = t.mine ? d.syz[t.p] : make_float2(0.0f, 0.0f);
  const RowConst rc = d.rows[t.sr % d.R];
  Slice dn, up;
  stage_tile(d, t, rc, h, S, dn, up);
  if (!(dn.staged && up.staged)) return false;   // wave-uniform
  const Staged rd{S.yz[0], S.bs[0], dn.bofs}, ru{S.yz[1], S.bs[1], up.bofs};
  const int nu = t.mine ? collect<Sh>(ru, up.g, h, rc.wy_up, rc.wz_up, S.list[1]) : 0;
  const int nd = nu > 0 ? collect<Sh>(rd, dn.g, h, rc.wy_dn, rc.wz_dn, S.list[0]) : 0;
  if (__any(nu > Sh::kLen || nd > Sh::kLen)) return false;
  best.dev = rc.dmax;
  test_pairs(S, rd, ru, nd, nu, h, rc.t, rho, best);
  write_links(d, t, best, up.off, dn.off);
  return true;
}

template <class Sh>
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
  if (!link_tile<Sh>(d, tile, rho, S) && threadIdx.x == 0)
    d.link_retry[atomicAdd(&d.hdr->link_retries, 1u)] = tile;
}

// The tiles that k_links left: dense rows (a chunk of 200k clusters has 1300
// hits a row, most of them in the third of the drift range that its particles
// reach at the inner rows) and crowded or wide windows.  The pass takes 481 us
// on one sector of 483k clusters (3400 hits a row, some 20 in a window), 2312
// on one of 969k, and 1058 on two sectors of rows of 600 hits in a patch of 20
// by 25 cm.  Walking the upper window in global memory for every lower hit of
// such a tile took 2238, 15093 and 22932.  Where no tile was left the launch
// costs 2 us.
__global__ void __launch_bounds__(kThreads) k_links_large(DevPtrs d, float rho) {
  __shared__ Stage<Large> S;
  const uint32_t n = d.hdr->link_retries;
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const Tile t = tile_of(d, d.link_retry[i]);   // never of the first or the last row
    const float2 h = t.mine ? d.syz[t.p] : make_float2(0.0f, 0.0f);
    const RowConst rc = d.rows[t.sr % d.R];
    Slice dn, up;
    stage_tile(d, t, rc, h, S, dn, up);
    Best best{rc.dmax, kNone, kNone};
    if (dn.staged && up.staged) {
      test_windows(S, Staged{S.yz[0], S.bs[0], dn.bofs}, Staged{S.yz[1], S.bs[1], up.bofs}, dn.g, up.g, t.mine, h, rc, rho, best);
    } else {
      dn.off = d.row_off[t.sr - 1];
      up.off = d.row_off[t.sr + 1];
      test_windows(S, InRow{d.syz + dn.off, d.bin_start + d.row_meta[t.sr - 1].x, dn.off},
                   InRow{d.syz + up.off, d.bin_start + d.row_meta[t.sr + 1].x, up.off}, dn.g, up.g, t.mine, h, rc, rho, best);
    }
    write_links(d, t, best, up.off, dn.off);
    __syncthreads();   // the stage is read to the end before the next tile fills it
  }
}

}  // namespace

void launch_links(const DevPtrs& d, hipStream_t s) {
  if (d.n_link_tiles == 0) return;
  // group size: as set, or one contiguous eighth of the tiles per XCD
  const uint32_t n = d.n_link_tiles;
  const uint32_t G = d.k2_group == kLinkGroupEighth ? (n + kXcds - 1) / kXcds : std::max<uint32_t>(1u, d.k2_group);
  const uint64_t groups = (n + (uint64_t)G - 1) / G;
  const uint32_t blocks = G == 1 ? n : (uint32_t)((groups + kXcds - 1) / kXcds * kXcds * G);   // every group slot
  if (d.k2_slots == 4) hipLaunchKernelGGL(k_links<Sparse>, dim3(blocks), dim3(kThreads), 0, s, d, d.rho, G);
  else hipLaunchKernelGGL(k_links<Dense>, dim3(blocks), dim3(kThreads), 0, s, d, d.rho, G);
  // any tile may be left (a list can overflow whatever the row's size)
  hipLaunchKernelGGL(k_links_large, dim3(std::min(n, 2048u)), dim3(kThreads), 0, s, d, d.rho);
}

}  // namespace tpc
