// K5: tracklet constructor -- step C5 of the tracker definition.
//
// Each tracklet (chain start) walks its chain (dependent up1 gathers), seeds
// from three chain hits, fits the chain, extends outward through the row
// grids and refits inward with a fresh covariance, filling gaps and extending
// below the chain.  Two schedules compute it: the row-synchronous kernel
// (k_tracklets_rs, a wave sweeps the rows of one sector in lockstep with each
// row staged in LDS where it fits; for frames whose waves are all resident, and
// k_tracklets_res where whole sectors fit in LDS) and the lane-per-tracklet
// pipeline (k_seed, k_up, k_sort, k_down, k_guard; larger frames).  The helix state p[5] and packed covariance C[15] are accumulated in
// double registers (see par_t / cov_t); the per-step increments and the
// Jacobian are float32.  The transport exploits the sparsity of the Jacobian
// (6 non-trivial entries).
//
// Latency is the bound (each row step is a dependent chain: propagate ->
// grid lookup -> candidate loads -> update), so the per-row constants are
// staged in LDS, a row's grid is located with one 8-byte load, and the
// float32 step arithmetic uses the hardware reciprocal / square root (its
// rounding is relative to one row step; the results are checked against the
// FP64 definition to 1e-4 relative, not bit-exact).
//
// The per-tracklet row -> hit column lives in global memory (row-major over
// tracklets, so lanes at the same row write one coalesced segment); the
// downward pass rewrites every row in [x_ref row, outermost row] with its
// final value, which is the only range the selector reads.
//
// z precision: in a continuous-readout frame the drift coordinate reaches
// several thousand cm, where one float32 ulp is ~5e-4 cm; summed over ~150
// steps that shifts tan(lambda) by ~1e-4 relative.  Each lane therefore keeps
// the state's z relative to its start hit (zref); z_m - zref is exact in
// float32 for the hits of one track (Sterbenz), and zref is added back only
// when the result is stored.
#include <algorithm>

#include "device_common.h"

namespace tpc {
namespace {

constexpr int kThreads = 64;

// tracklets of the lane-per-tracklet pipeline: all, or none where the device has left them to the row-by-row sweeps
__device__ __forceinline__ uint32_t pipe_n(const DevPtrs& d) { return min(*d.pipe_n, d.tcap); }

__device__ __forceinline__ int tri(int i, int j) { return i * (i + 1) / 2 + j; }   // i >= j

// Arithmetic types of the Kalman state p and of its covariance C.  Both are
// accumulated in double: a track's covariance shrinks by up to seven orders
// of magnitude under strongly correlated updates (y, sin phi and q/pT move
// together), so a float32 recursion loses about 1e-2 of its relative
// precision, and a float32 state rounds every row's increment of sin phi and
// y into values hundreds of times larger, which shifts the fitted q/pT by
// more than 1e-4.  Everything evaluated per row step from the state (the
// increments, the Jacobian, the search window) stays in float32, where its
// rounding is relative to the step itself.
using par_t = double;
using cov_t = double;

__device__ __forceinline__ float frcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float fsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ float frsqrt(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ float fabs_(float x) { return fabsf(x); }
// double reciprocal: the float32 hardware estimate refined by one Newton step (relative error ~1e-14)
__device__ __forceinline__ double frcp(double x) {
  const double r = __builtin_amdgcn_rcpf(float(x));
  return r * (2.0 - x * r);
}
__device__ __forceinline__ double fabs_(double x) { return fabs(x); }

// native vector types: arrays of them stay in registers
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct Trk {
  par_t p[5];
  cov_t c[15];
};

// The state at the innermost hit of the inward pass, in the float32 the result is stored in.
struct Snap {
  float p[5];
  float c[15];
};
__device__ __forceinline__ Snap snap_of(const Trk& t) {
  Snap s;
#pragma unroll
  for (int q = 0; q < 5; ++q) s.p[q] = float(t.p[q]);
#pragma unroll
  for (int q = 0; q < 15; ++q) s.c[q] = float(t.c[q]);
  return s;
}

// Per-row constants used in the tracklet loop: x, half-width, y_lo, 1/(2Y).
struct RowK {
  float x, half_y, y_lo, inv_wy;
};

// asin(u)/u and d/du of it; |u| is below 0.02 for row-to-row steps.
__device__ __forceinline__ float asin_over(float u) {
  const float u2 = u * u;
  if (fabsf(u) < 0.05f) return 1.0f + u2 * (1.0f / 6.0f + u2 * (3.0f / 40.0f + u2 * (5.0f / 112.0f)));
  return asinf(u) / u;
}
__device__ __forceinline__ float asin_over_prime(float u) {
  const float u2 = u * u;
  if (fabsf(u) < 0.1f)
    return u * (1.0f / 3.0f + u2 * (3.0f / 10.0f + u2 * (15.0f / 56.0f + u2 * (35.0f / 144.0f))));
  return (u * frsqrt(1.0f - u2) - asinf(u)) / u2;
}
// Helix transport from x to x + dx with covariance; false on |sin phi| >= s_max or |u| >= 1.
// The failure tests do not branch (a branch costs every lane of the wave); on
// false the state holds meaningless values, and every caller stops the
// tracklet without reading it again.
//
// The increments of one row step (dy, dz, kappa*dx) and the Jacobian are
// evaluated in float32: their rounding is relative to the step, far below the
// tolerance.  They are accumulated into the state in par_t, and the covariance
// is transported in cov_t.
__device__ __forceinline__ bool propagate(Trk& t, float dx, const KfConst& k) {
  using V = cov_t;
  const float s1 = float(t.p[2]), tl = float(t.p[3]), qp = float(t.p[4]);
  const float kap = k.bk * qp;
  const par_t s2p = t.p[2] + par_t(kap * dx);
  const float s2 = float(s2p);
  const float c1 = fsqrt((1.0f - s1) * (1.0f + s1));
  const float c2 = fsqrt((1.0f - s2) * (1.0f + s2));
  const float ic = frcp(c1 + c2);
  const float dy = dx * ((s1 + s2) * ic);
  const float L = fsqrt(dx * dx + dy * dy);
  const float u = 0.5f * kap * L;
  const bool ok = fabsf(s1) < k.s_max && fabsf(s2) < k.s_max && fabsf(u) < 1.0f;
  const float sgn = dx >= 0.0f ? 1.0f : -1.0f;
  const float S = sgn * L * asin_over(u);
  // Jacobian entries (exact derivative of the map above)
  const float ic1 = frcp(c1), ic2 = frcp(c2);
  const float D = (1.0f + c1 * c2 + s1 * s2) * (ic * ic);
  const float ddy_ds1 = dx * D * (ic1 + ic2);
  const float ddy_dk = dx * dx * (D * ic2) * k.bk;
  const float dS_dL = sgn * frsqrt(1.0f - u * u);
  const float dS_dkap = sgn * 0.5f * L * L * asin_over_prime(u);
  const float dL_ddy = L > 0.0f ? dy * frcp(L) : 0.0f;
  const V A = ddy_ds1;                                  // F02
  const V B = ddy_dk;                                   // F04
  const V Cc = tl * dS_dL * dL_ddy * ddy_ds1;           // F12
  const V Dd = S;                                       // F13
  const V E = tl * (dS_dL * dL_ddy * ddy_dk + dS_dkap * k.bk);  // F14
  const V Fk = k.bk * dx;                               // F24
  t.p[0] += par_t(dy);
  t.p[1] += par_t(tl * S);
  t.p[2] = s2p;
  // C' = F C F^T with F = I + {02:A, 04:B, 12:Cc, 13:Dd, 14:E, 24:Fk}
  V* c = t.c;
  V M[5][5];
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = 0; j < 5; ++j) M[i][j] = i >= j ? c[tri(i, j)] : c[tri(j, i)];
  V G[5][5];   // G = F C
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    G[0][j] = M[0][j] + A * M[2][j] + B * M[4][j];
    G[1][j] = M[1][j] + Cc * M[2][j] + Dd * M[3][j] + E * M[4][j];
    G[2][j] = M[2][j] + Fk * M[4][j];
    G[3][j] = M[3][j];
    G[4][j] = M[4][j];
  }
#pragma unroll
  for (int i = 0; i < 5; ++i) {   // C'_ij = sum_k G_ik F_jk
    const V g0 = G[i][0], g1 = G[i][1], g2 = G[i][2], g3 = G[i][3], g4 = G[i][4];
    const V r0 = g0 + A * g2 + B * g4;
    const V r1 = g1 + Cc * g2 + Dd * g3 + E * g4;
    const V r2 = g2 + Fk * g4;
    const V rr[5] = {r0, r1, r2, g3, g4};
#pragma unroll
    for (int j = 0; j <= i; ++j) c[tri(i, j)] = rr[j];
  }
  return ok;
}

// Kalman update with a measurement of (y, z).  The covariance update is the
// plain C' = C - K H C: in double it keeps far more precision than the
// parameters need (the Joseph form, which guards the positive definiteness of
// a float32 recursion, costs 40 more double operations per step).  Each
// element takes two fused multiply-adds (the sum of the two products and its
// subtraction would be three operations).
__device__ __forceinline__ void update(Trk& t, float ym, float zm, const KfConst& k, float& chi2) {
  using P = par_t;
  using V = cov_t;
  V* c = t.c;
  const V vy = k.vyd, vz = k.vzd;
  const V r0 = V(P(ym) - t.p[0]), r1 = V(P(zm) - t.p[1]);
  const V S00 = c[0] + vy, S01 = c[1], S11 = c[2] + vz;
  const V id = frcp(S00 * S11 - S01 * S01);
  const V I00 = S11 * id, I01 = -S01 * id, I11 = S00 * id;
  V c0[5], c1[5];   // columns 0 and 1 of C (C_i0, C_i1)
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    c0[i] = c[tri(i, 0)];
    c1[i] = i >= 1 ? c[tri(i, 1)] : c[tri(1, 0)];
  }
  V K0[5], K1[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    K0[i] = c0[i] * I00 + c1[i] * I01;
    K1[i] = c0[i] * I01 + c1[i] * I11;
    t.p[i] = fma(K0[i], r0, fma(K1[i], r1, t.p[i]));
  }
#pragma unroll
  for (int i = 4; i >= 0; --i)   // downwards, so that each element is overwritten after its last use (fewer moves: -1%)
#pragma unroll
    for (int j = i; j >= 0; --j) c[tri(i, j)] = fma(-K0[i], c0[j], fma(-K1[i], c1[j], c[tri(i, j)]));
  chi2 += float(r0 * (I00 * r0 + I01 * r1) + r1 * (I01 * r0 + I11 * r1));
}

__device__ __forceinline__ void set_c0(Trk& t, const KfConst& k) {
#pragma unroll
  for (int i = 0; i < 15; ++i) t.c[i] = cov_t(0);
  t.c[tri(0, 0)] = k.vyd;
  t.c[tri(1, 1)] = k.vzd;
  t.c[tri(2, 2)] = k.c0_sinphi;
  t.c[tri(3, 3)] = k.c0_tanl;
  t.c[tri(4, 4)] = k.c0_qpt;
}

// Grid search in row sr for the candidate closest to the prediction; -1 if
// none, else its position, with its (y, z) in hv.  The hits of the bins that
// the window touches are tested in ascending position, kGroup of them at a
// time (their loads are contiguous and issued together).  Where a z-line has
// few bins, its bins and those of the next lines are taken as one run: the
// hits between them are outside the window and fail its test, and a lane
// whose window straddles two lines does not cost its wave a second group.
constexpr int kGroup = 6;   // measured on the 32-orbit frame: 4 -> 6 is -3.7% in K5, 8 and above slower
constexpr int kGroupLds = 4;   // most candidates that a lane of the LDS searches reads together
constexpr int kRunBins = 3;    // z-lines of at most this many bins are searched as one run

// two consecutive hits with one 16-byte load (hits are 8-byte aligned)
typedef f32x4 f32x4_at8 __attribute__((aligned(8)));

__device__ __forceinline__ int32_t search_m(const DevPtrs& d, uint2 meta, const RowK& rk, const SectorConst& sc,
                                            const Trk& t, const KfConst& k, float zref, float2& hv) {
  const float sy2 = float(t.c[0] + k.vyd), sz2 = float(t.c[2] + k.vzd);
  const float wy = fminf(k.gate * fsqrt(sy2), k.cap), wz = fminf(k.gate * fsqrt(sz2), k.cap);
  const float isy = frcp(sy2), isz = frcp(sz2);
  const float yp = float(t.p[0]), zp = float(t.p[1]);          // zp relative to zref
  const float za = zref + zp;                     // absolute, for the bin range only
  const int ny = (int)(meta.y & 0xFFFFu), nz = (int)(meta.y >> 16);
  const int iy0 = bin1((yp - wy) - kWinPad, rk.y_lo, rk.inv_wy, ny);
  const int iy1 = bin1((yp + wy) + kWinPad, rk.y_lo, rk.inv_wy, ny);
  const int iz0 = bin1((za - wz) - kWinPad, sc.z_lo, sc.inv_wz, nz);
  const int iz1 = bin1((za + wz) + kWinPad, sc.z_lo, sc.inv_wz, nz);
  // bins [b0, b1] of the first run, which ends in the z-line of bin b1; e: the last bin of the window
  uint32_t b0 = meta.x + (uint32_t)(iz0 * ny + iy0);
  const uint32_t e = meta.x + (uint32_t)(iz1 * ny + iy1);
  uint32_t b1 = ny <= kRunBins ? e : b0 + (uint32_t)(iy1 - iy0);
  uint32_t q = d.bin_start[b0], hi = d.bin_start[b1 + 1];
  int32_t best = -1;
  float bd = INFINITY;
  for (;;) {
    while (q >= hi && b1 < e) {
      b0 += (uint32_t)ny;
      b1 += (uint32_t)ny;
      q = d.bin_start[b0];
      hi = d.bin_start[b1 + 1];
    }
    if (q >= hi) break;
    // up to kGroup - 1 entries past the run's end are read (the array is followed by others in the workspace)
    // and not used
    float2 h[kGroup];
    const f32x4_at8* src = reinterpret_cast<const f32x4_at8*>(d.syz + q);
#pragma unroll
    for (int j = 0; j < kGroup / 2; ++j) {
      const f32x4 v = src[j];
      h[2 * j] = make_float2(v.x, v.y);
      h[2 * j + 1] = make_float2(v.z, v.w);
    }
    const uint32_t n = hi - q;
#pragma unroll
    for (int j = 0; j < kGroup; ++j) {
      const float dy = h[j].x - yp, dz = (h[j].y - zref) - zp;
      const float dd = __builtin_fmaf(dy * dy, isy, (dz * dz) * isz);
      const bool take = (uint32_t)j < n & fabsf(dy) <= wy & fabsf(dz) <= wz & dd < bd;
      best = take ? (int32_t)(q + j) : best;
      bd = take ? dd : bd;
      hv.x = take ? h[j].x : hv.x;
      hv.y = take ? h[j].y : hv.y;
    }
    q += kGroup;
  }
  return best;
}

__device__ __forceinline__ int32_t search(const DevPtrs& d, uint32_t sr, const RowK& rk, const SectorConst& sc,
                                          const Trk& t, const KfConst& k, float zref, float2& hv) {
  return search_m(d, d.row_meta[sr], rk, sc, t, k, zref, hv);
}

// The same search for the lanes of a wave together: the candidates of all searching lanes are cut into items of kItem,
// and the items are dealt out to all 64 lanes, whichever lane they belong to.  Called by the whole wave, converged.
//
// Bound: vector instructions (the passes that search issue one in 92% of their cycles).  On the 32-orbit frame a search
// has 5.2 candidates on average and 28 of a wave's 64 lanes search in a step, but the lane with the most takes 2.9 groups
// of 6: tested lane by lane (search_m), 13% of the tests do work, and they are half of the instructions.  Dealt out, a
// step's 49 items take one round (the average; chunks 63, some two).  An item's owner is found by a scan over the items'
// starts, its window is read with lane permutes, and the winner comes from an LDS minimum over (deviation, position): the
// smallest deviation, ties to the smaller position, which is what the ascending scan of search_m takes.
// k_up and k_down: 32-orbit frame 2151 -> 1843 us, 512 uneven chunks 5466 -> 5010, 8 heavy-ion orbits 924 -> 833.  Items of 2:
// +4%, of 6: +2%.  A window of more than two runs (a narrow grid under a wide cap) is left to search_m, and the wave's other
// windows with it: shared after it, they made a central event with a gate of 40 sigma and a cap of 15 cm 2215 us instead of
// 1815 (2040 lane by lane throughout).
constexpr int kItem = 4;
struct WaveSearch {
  unsigned long long key[kThreads];   // per lane: (deviation, position) of its best candidate
  float2 hv[kThreads];                // (y, z) of it
  uint32_t map[kThreads];             // slot -> lane + 1 at the slot of a lane's first item, else 0
};
static_assert(kItem % 2 == 0 && kItem <= kGroup, "items are loaded in pairs; the arrays' slack covers a group");

template <int kCtrl, int kRows, class Op>
__device__ __forceinline__ uint32_t dpp_step(uint32_t v, Op op) {
  return op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, kRows, 0xF, false));
}
// inclusive scan over the wave, op's identity 0
template <class Op>
__device__ __forceinline__ uint32_t dpp_scan(uint32_t v, Op op) {
  v = dpp_step<0x111, 0xF>(v, op);   // row_shr 1, 2, 4, 8
  v = dpp_step<0x112, 0xF>(v, op);
  v = dpp_step<0x114, 0xF>(v, op);
  v = dpp_step<0x118, 0xF>(v, op);
  v = dpp_step<0x142, 0xA>(v, op);   // row_bcast 15 into rows 1 and 3
  v = dpp_step<0x143, 0xC>(v, op);   // row_bcast 31 into rows 2 and 3
  return v;
}

// where the hits and bin starts are read: the frame's arrays, or a row staged in LDS (hits from position first, bins from
// the row's first)
struct InFrame {
  const float2* yz;
  const uint32_t* bs;
  __device__ __forceinline__ uint32_t start(uint32_t b) const { return bs[b]; }
  __device__ __forceinline__ const float2* at(uint32_t q) const { return yz + q; }
};
struct InStage {
  const float2* yz;
  const uint32_t* bs;
  uint32_t first, bins;
  __device__ __forceinline__ uint32_t start(uint32_t b) const { return bs[b - bins]; }
  __device__ __forceinline__ const float2* at(uint32_t q) const { return yz + (q - first); }
};
template <class Row>
__device__ __forceinline__ int32_t search_wave(const DevPtrs& d, const Row& row, WaveSearch& l, bool want, uint2 meta, const RowK& rk,
                                               const SectorConst& sc, const Trk& t, const KfConst& k, float zref,
                                               float2& hv) {
  if (!__any(want)) return -1;
  const uint32_t lane = threadIdx.x;
  const float sy2 = float(t.c[0] + k.vyd), sz2 = float(t.c[2] + k.vzd);
  const float wy = fminf(k.gate * fsqrt(sy2), k.cap), wz = fminf(k.gate * fsqrt(sz2), k.cap);
  const float isy = frcp(sy2), isz = frcp(sz2);
  const float yp = float(t.p[0]), zp = float(t.p[1]);
  uint32_t b0 = 0, b1 = 0, e = 0, ny = 0;
  if (want) {
    const float za = zref + zp;
    ny = meta.y & 0xFFFFu;
    const int nz = (int)(meta.y >> 16);
    const int iy0 = bin1((yp - wy) - kWinPad, rk.y_lo, rk.inv_wy, (int)ny);
    const int iy1 = bin1((yp + wy) + kWinPad, rk.y_lo, rk.inv_wy, (int)ny);
    const int iz0 = bin1((za - wz) - kWinPad, sc.z_lo, sc.inv_wz, nz);
    const int iz1 = bin1((za + wz) + kWinPad, sc.z_lo, sc.inv_wz, nz);
    b0 = meta.x + (uint32_t)iz0 * ny + (uint32_t)iy0;
    e = meta.x + (uint32_t)iz1 * ny + (uint32_t)iy1;
    b1 = ny <= (uint32_t)kRunBins ? e : b0 + (uint32_t)(iy1 - iy0);
  }
  // some lane has more than two runs: it would search alone, so all do, beside it
  if (__any(want && b1 + ny < e)) return want ? search_m(d, meta, rk, sc, t, k, zref, hv) : -1;
  l.key[lane] = ~0ull;
  // up to two runs per lane: [q0, h0) and [q1, h1)
  uint32_t q0 = 0, h0 = 0, q1 = 0, h1 = 0;
  if (want) {
    q0 = row.start(b0);
    h0 = row.start(b1 + 1);
    if (b1 < e) {
      q1 = row.start(b0 + ny);
      h1 = row.start(b1 + ny + 1);
    }
  }
  const uint32_t n0 = (h0 - q0 + kItem - 1) / kItem, n = n0 + (h1 - q1 + kItem - 1) / kItem;
  const uint32_t end = dpp_scan(n, [](uint32_t a, uint32_t b) { return a + b; });
  const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)end, kWave - 1);
  const uint32_t start = end - n, split = start + n0;
  const bool two = __any(h1 > q1);
  for (uint32_t base = 0; base < total; base += kWave) {
    l.map[lane] = 0;
    wave_lds_order();
    if (n > 0 && end > base && start < base + kWave) l.map[max(start, base) - base] = lane + 1;
    wave_lds_order();
    const uint32_t own = dpp_scan(l.map[lane], [](uint32_t a, uint32_t b) { return max(a, b); }) - 1;
    const int at = (int)(own * 4);
    auto from = [&](uint32_t v) { return (uint32_t)__builtin_amdgcn_ds_bpermute(at, (int)v); };
    auto fromf = [&](float v) { return __int_as_float(__builtin_amdgcn_ds_bpermute(at, __float_as_int(v))); };
    const uint32_t slot = base + lane;
    uint32_t q = from(q0 - start * kItem), lim = from(h0);
    if (two) {
      const uint32_t s1 = from(split), qb = from(q1 - split * kItem), hb = from(h1);
      if (slot >= s1) {
        q = qb;
        lim = hb;
      }
    }
    q += slot * kItem;
    const float oyp = fromf(yp), owy = fromf(wy), oisy = fromf(isy);
    const float ozr = fromf(zref), ozp = fromf(zp), owz = fromf(wz), oisz = fromf(isz);
    float bd = INFINITY;
    uint32_t bq = 0;
    float2 bh = make_float2(0.0f, 0.0f);
    if (slot < total) {
      float2 h[kItem];
      const f32x4_at8* src = reinterpret_cast<const f32x4_at8*>(row.at(q));
#pragma unroll
      for (int j = 0; j < kItem / 2; ++j) {
        const f32x4 v = src[j];
        h[2 * j] = make_float2(v.x, v.y);
        h[2 * j + 1] = make_float2(v.z, v.w);
      }
      const uint32_t m = lim - q;
#pragma unroll
      for (int j = 0; j < kItem; ++j) {
        const float dy = h[j].x - oyp, dz = (h[j].y - ozr) - ozp;
        const float dd = __builtin_fmaf(dy * dy, oisy, (dz * dz) * oisz);
        const bool take = (uint32_t)j < m & fabsf(dy) <= owy & fabsf(dz) <= owz & dd < bd;
        bq = take ? q + j : bq;
        bd = take ? dd : bd;
        bh.x = take ? h[j].x : bh.x;
        bh.y = take ? h[j].y : bh.y;
      }
    }
    const bool found = bd < INFINITY;
    unsigned long long mine = 0;
    wave_lds_order();
    if (found) {
      const uint32_t b = (uint32_t)__float_as_int(bd + 0.0f);
      mine = ((unsigned long long)(b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u)) << 32) | bq;
      __hip_atomic_fetch_min(&l.key[own], mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
    wave_lds_order();
    if (found && l.key[own] == mine) l.hv[own] = bh;
  }
  wave_lds_order();
  const unsigned long long best = l.key[lane];
  if (best == ~0ull) return -1;
  hv = l.hv[lane];
  return (int32_t)(uint32_t)best;
}

// Value of another lane of the kL lanes of a tracklet: a DPP move inside rows of 16.
template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_min(uint32_t v) {
  return min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, kCtrl, 0xF, 0xF, false));
}
template <int kL>
__device__ __forceinline__ uint32_t group_min(uint32_t v) {
  if (kL >= 2) v = dpp_min<0xB1>(v);    // quad_perm 1,0,3,2
  if (kL >= 4) v = dpp_min<0x4E>(v);    // quad_perm 2,3,0,1
  if (kL >= 8) v = dpp_min<0x141>(v);   // row_half_mirror
  if (kL >= 16) v = dpp_min<0x140>(v);  // row_mirror
  return v;
}

// The same search over a row staged in LDS: (y, z) of the row's hits at
// yz[q - first] and its bin starts (global positions) in bs[].  It is run by the
// kL lanes that carry the same tracklet: on every pair of z-lines they take kU
// candidates in turn, walking the two lines as one flat sequence, and then
// exchange their best candidates (DPP moves inside the tracklet's lanes, no LDS
// round trip).  A turn is read whole: its entries past the z-line's end (at
// most kGroupLds - 1, inside the stage's slack) are masked out.
// The result -- smallest deviation, ties to the smaller position -- is the same
// as a single ascending scan.
template <int kL>
__device__ __forceinline__ int32_t search_lds(const float2* yz, const uint32_t* bs, uint32_t first, uint2 meta,
                                              const RowK& rk, const SectorConst& sc, const Trk& t, const KfConst& k,
                                              float zref, uint32_t sub) {
  constexpr int kU = kL == 2 ? 4 : 2;
  const float sy2 = float(t.c[0] + k.vyd), sz2 = float(t.c[2] + k.vzd);
  const float wy = fminf(k.gate * fsqrt(sy2), k.cap), wz = fminf(k.gate * fsqrt(sz2), k.cap);
  const float isy = frcp(sy2), isz = frcp(sz2);
  const float yp = float(t.p[0]), zp = float(t.p[1]);
  const float za = zref + zp;
  const int ny = (int)(meta.y & 0xFFFFu), nz = (int)(meta.y >> 16);
  const int iy0 = bin1((yp - wy) - kWinPad, rk.y_lo, rk.inv_wy, ny);
  const int iy1 = bin1((yp + wy) + kWinPad, rk.y_lo, rk.inv_wy, ny);
  const int iz0 = bin1((za - wz) - kWinPad, sc.z_lo, sc.inv_wz, nz);
  const int iz1 = bin1((za + wz) + kWinPad, sc.z_lo, sc.inv_wz, nz);
  uint32_t best = 0xFFFFFFFFu;
  float bd = INFINITY;
  // z-lines are taken two at a time (a window almost never spans more): the
  // candidates of the pair of lines form one flat sequence -- line iz, then
  // line iz + 1, so positions ascend -- and the lanes of a tracklet take kU of
  // it in turn
  for (int iz = iz0; iz <= iz1; iz += 2) {
    const int izb = iz + 1 <= iz1 ? iz + 1 : iz;
    const uint32_t lo0 = bs[iz * ny + iy0], hi0 = bs[iz * ny + iy1 + 1];
    const uint32_t lo1 = bs[izb * ny + iy0], hi1 = bs[izb * ny + iy1 + 1];
    const uint32_t n0 = hi0 - lo0, tot = n0 + (izb > iz ? hi1 - lo1 : 0u);
    for (uint32_t g0 = sub * kU; g0 < tot; g0 += kL * kU) {
      uint32_t pos[kU];
      float2 h[kU];
#pragma unroll
      for (int j = 0; j < kU; ++j) {
        const uint32_t f = g0 + j;   // past the end: at most kU - 1 entries beyond a line, masked below
        pos[j] = f < n0 ? lo0 + f : lo1 + (f - n0);
        h[j] = yz[pos[j] - first];
      }
#pragma unroll
      for (int j = 0; j < kU; ++j) {
        const float dy = h[j].x - yp, dz = (h[j].y - zref) - zp;
        if (g0 + j < tot && fabsf(dy) <= wy && fabsf(dz) <= wz) {
          const float dd = __builtin_fmaf(dy * dy, isy, (dz * dz) * isz);
          if (dd < bd) {
            best = pos[j];
            bd = dd;
          }
        }
      }
    }
  }
  // the lanes' candidates: smallest deviation (not negative, so its bits order as it does), ties to the smaller position
  const uint32_t mine = (uint32_t)__float_as_int(bd), least = group_min<kL>(mine);
  return (int32_t)group_min<kL>(mine == least ? best : 0xFFFFFFFFu);
}

// Three-point seed; false on failure.
__device__ __forceinline__ bool seed3(float x0, float2 h0, float xm, float2 hm, float xl, float2 hl, const KfConst& k,
                                      Trk& t) {
  const float ax = xm - x0, ay = hm.x - h0.x, bx = xl - xm, by = hl.x - hm.x, cx = xl - x0, cy = hl.x - h0.x;
  const float cross = ax * by - ay * bx;
  const float la = sqrtf(ax * ax + ay * ay), lb = sqrtf(bx * bx + by * by), lc = sqrtf(cx * cx + cy * cy);
  if (!(la > 0.0f && lb > 0.0f && lc > 0.0f)) return false;
  const float kap = 2.0f * cross / (la * lb * lc);
  const float u = 0.5f * kap * lc;
  if (!(fabsf(u) < 1.0f)) return false;
  const float phi0 = atan2f(cy, cx) - asinf(u);
  const float s0l = lc * asin_over(u);
  float qpt = k.bk != 0.0f ? kap / k.bk : 0.0f;
  qpt = fminf(k.qpt_max, fmaxf(-k.qpt_max, qpt));
  float sp, cp;
  sincosf(phi0, &sp, &cp);
  t.p[0] = h0.x;
  t.p[1] = 0.0f;             // z relative to the start hit
  t.p[2] = sp;
  t.p[3] = (hl.y - h0.y) / s0l;
  t.p[4] = qpt;
  return cp > 0.0f && fabsf(sp) < k.s_max;
}

__device__ __forceinline__ void load_rows(const DevPtrs& d, RowK* lrows) {
  for (uint32_t r = threadIdx.x; r < d.R; r += blockDim.x) {
    const RowConst rc = d.rows[r];
    lrows[r] = RowK{rc.x, rc.half_y, rc.y_lo, rc.inv_wy};
  }
  __syncthreads();
}

// SPD guard for the stored covariance.  Near-singular fits (a short, strongly
// curved arc can correlate sin phi and q/pT at 0.99) sit within float32
// rounding of the positive-definite boundary; LDL^T with every pivot floored
// at kPivotFloor * C_kk returns them to a nearby positive-definite matrix and
// leaves every other covariance untouched (no rebuild when no pivot is low).
constexpr float kPivotFloor = 1e-5f;

__device__ __forceinline__ void spd_guard(float* c) {
  float L[5][5], D[5];
  bool fixed = false;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    float dk = c[tri(k, k)];
#pragma unroll
    for (int j = 0; j < k; ++j) dk -= L[k][j] * L[k][j] * D[j];
    const float floor_k = kPivotFloor * c[tri(k, k)];
    if (!(dk > floor_k)) {
      dk = floor_k;
      fixed = true;
    }
    D[k] = dk;
    const float idk = 1.0f / dk;
#pragma unroll
    for (int i = k + 1; i < 5; ++i) {
      float v = c[tri(i, k)];
#pragma unroll
      for (int j = 0; j < k; ++j) v -= L[i][j] * L[k][j] * D[j];
      L[i][k] = v * idk;
    }
  }
  if (!fixed) return;
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = 0; j <= i; ++j) {
      float v = (i == j ? 1.0f : L[i][j]) * D[j];
#pragma unroll
      for (int q = 0; q < j; ++q) v += L[i][q] * L[j][q] * D[q];
      c[tri(i, j)] = v;
    }
}

template <bool kGuard>
__device__ __forceinline__ void store_tracklet(const DevPtrs& d, uint32_t i, int nh, uint32_t rin, uint32_t rout,
                                               uint32_t r0, const Snap& snap, float chi2, float zref) {
  const uint32_t T = d.tcap;
  d.tk_info[i] = nh;
  d.tk_info[T + i] = (int32_t)rin;
  d.tk_info[2 * T + i] = (int32_t)rout;
  d.tk_info[3 * T + i] = (int32_t)r0;
#pragma unroll
  for (int q = 0; q < 5; ++q) d.tk_param[(size_t)q * T + i] = q == 1 ? snap.p[q] + zref : snap.p[q];
  float c[15];
#pragma unroll
  for (int q = 0; q < 15; ++q) c[q] = snap.c[q];
  if (kGuard) spd_guard(c);
#pragma unroll
  for (int q = 0; q < 15; ++q) d.tk_cov[(size_t)q * T + i] = c[q];
  d.tk_chi2[i] = chi2;
}

// The covariance guard over every stored tracklet, one lane each (for k_down,
// whose lanes store as they finish: there the guard would cost the whole wave
// once for every group of lanes that finish together).  When the refit ran in
// bucket order its results wait in slot order (one contiguous record per
// tracklet, see kRec*), so that the refit's lanes write whole lines; the
// guard gathers each tracklet's record through the bucket slot of tracklet i
// and writes the result arrays in tracklet order.
enum : int { kRecInfo = 0, kRecParam = 4, kRecCov = 9, kRecChi2 = 24, kRecWords = 25 };

__global__ void __launch_bounds__(256) k_guard(DevPtrs d) {
  const uint32_t nt = pipe_n(d), T = d.tcap;
  const bool staged = d.k5_refit_order == 0;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nt; i += gridDim.x * blockDim.x) {
    if (staged) {
      if (d.tk_info[i] < 0) continue;   // no seed, or the chain fit failed: no refit record
      const uint32_t* rec = d.k5_rec + (size_t)d.k5_inv[i] * kRecWords;
      uint32_t w[kRecWords];
#pragma unroll
      for (int q = 0; q < kRecWords; ++q) w[q] = rec[q];
#pragma unroll
      for (int q = 0; q < 4; ++q) d.tk_info[(size_t)q * T + i] = (int32_t)w[kRecInfo + q];
#pragma unroll
      for (int q = 0; q < 5; ++q) d.tk_param[(size_t)q * T + i] = __int_as_float((int)w[kRecParam + q]);
      float c[15];
#pragma unroll
      for (int q = 0; q < 15; ++q) c[q] = __int_as_float((int)w[kRecCov + q]);
      spd_guard(c);
#pragma unroll
      for (int q = 0; q < 15; ++q) d.tk_cov[(size_t)q * T + i] = c[q];
      d.tk_chi2[i] = __int_as_float((int)w[kRecChi2]);
    } else {
      if (d.tk_info[i] < 1) continue;
      float c[15];
#pragma unroll
      for (int q = 0; q < 15; ++q) c[q] = d.tk_cov[(size_t)q * T + i];
      spd_guard(c);
#pragma unroll
      for (int q = 0; q < 15; ++q) d.tk_cov[(size_t)q * T + i] = c[q];
    }
  }
}

// ---------------------------------------------------------------------------
// Lane-per-tracklet schedule: k_seed, k_up, k_sort, k_down, k_guard.
//
// A wave steps as long as its longest lane.  With one loop per pass (chain
// fit, outward extension, inward refit) a wave steps through its longest
// chain fit, then its longest extension, then its longest refit, and on a
// 32-orbit frame only about 56% of the lane steps do work.  Here the chain
// fit and the outward extension run as one loop (both move outward one row
// per step, so the lanes of a wave, which hold consecutive tracklets of one
// sector and start rows close together, stay on the same rows), and the
// inward refits are regrouped by (sector, outermost row) before they run: a
// wave's lanes then start the refit on the same row and walk the same rows in
// step, and most of them stop within a few rows of each other.
//
// k_seed: one lane per tracklet walks its chain (dependent up1 gathers that
// fill the chain's rows of the row -> hit column) and builds the three-point
// seed.  It leaves the seed in tk_param, the chain's last row in
// tk_info[2T + i] and 0 (seeded) or -1 (no seed) in tk_info[i].
// k_up: chain fit and outward extension, one lane per tracklet; it hands the
// refit its start (below) and counts the tracklet in its (sector, outermost
// row) bucket.
// k_sort: bucket offsets (an exclusive scan) and a scatter of the tracklet
// indices into bucket order (the order inside a bucket does not matter: every
// tracklet's refit is independent of the others).
// k_down: the inward refit, one lane per tracklet in bucket order; stores the
// tracklet.
// k_guard: the covariance guard over every stored tracklet.
//
// Workgroups are dispatched round-robin over the 8 XCDs (block b -> XCD b % 8),
// each with its own L2.  Tracklets (and buckets) are ordered by sector, so each
// XCD is given one contiguous eighth of them: its lanes then search the row
// grids of a few sectors only, which stay resident in that XCD's L2.
__global__ void __launch_bounds__(kThreads) k_seed(DevPtrs d, KfConst k) {
  __shared__ float lx[kMaxRows];
  const uint32_t nt = pipe_n(d);
  const uint32_t R = d.R, T = d.tcap;
  // the bucket counts of k_up start at zero (the C4 row counts are not used after C4)
  for (uint32_t q = blockIdx.x * blockDim.x + threadIdx.x; q < d.SR; q += gridDim.x * blockDim.x) d.row_nstart[q] = 0;
  const XcdSched sch = xcd_sched(nt);
  if (sch.first >= sch.end) return;   // the grid is sized for the tracklet capacity
  for (uint32_t r = threadIdx.x; r < R; r += blockDim.x) lx[r] = d.rows[r].x;
  __syncthreads();
  for (uint32_t vb = sch.first; vb < sch.end; vb += sch.stride) {
    const uint32_t i = vb * kThreads + threadIdx.x;
    if (i >= nt) continue;
    const uint32_t r0 = d.start_sr[i] % R;
    int32_t* H = d.tk_rowhit + i;     // row r at H[r * T]
    const int32_t p0 = (int32_t)d.start_pos[i];
    int32_t p = p0, plast = p0;
    uint32_t n = 0;
    while (p >= 0 && r0 + n < R) {   // links step one row outward, so a chain ends before row R
      H[(size_t)(r0 + n) * T] = p;
      plast = p;
      ++n;
      p = d.up1[p];
    }
    const uint32_t m = (n - 1) / 2, rl = r0 + n - 1;
    const int32_t pm = H[(size_t)(r0 + m) * T];
    Trk t;
    const bool ok = seed3(lx[r0], d.syz[p0], lx[r0 + m], d.syz[pm], lx[rl], d.syz[plast], k, t);
    if (ok) {
#pragma unroll
      for (int q = 0; q < 5; ++q) d.tk_param[(size_t)q * T + i] = float(t.p[q]);   // seed3 works in float32
    }
    d.tk_info[2 * T + i] = (int32_t)rl;
    d.tk_info[i] = ok ? 0 : -1;
  }
}

// atomicAdd(&ctr[key], 1) for every lane with `on`, one atomic per distinct
// key in the wave (many tracklets share a bucket, and the atomics of one
// address serialize); returns the lane's slot (the counter before its add).
// Called by all lanes of the wave.
__device__ __forceinline__ uint32_t wave_claim(uint32_t* ctr, uint32_t key, bool on) {
  const uint32_t lane = threadIdx.x % kWave;
  uint32_t slot = 0;
  unsigned long long todo = __ballot(on);
  while (todo) {
    const int leader = __ffsll((long long)todo) - 1;
    const uint32_t lk = (uint32_t)__shfl((int)key, leader, kWave);
    const unsigned long long grp = __ballot(on && key == lk) & todo;
    uint32_t base = 0;
    if ((int)lane == leader) base = atomicAdd(&ctr[lk], (uint32_t)__popcll(grp));
    base = (uint32_t)__shfl((int)base, leader, kWave);
    if ((grp >> lane) & 1ull) slot = base + (uint32_t)__popcll(grp & ((1ull << lane) - 1ull));
    todo &= ~grp;
  }
  return slot;
}

// Hand-off from k_up to k_down, per tracklet i, in the rows of tk_cov (free
// until the tracklet is stored, by the lane that has read its hand-off), as
// 32-bit words at word w * T + i: 0-5 sin phi, tan lambda and q/pT at the
// outermost hit (double, low word first), 6-7 that hit's (y, z), 8 the
// outermost row, 9 the start row r0, 10 z_ref, 11 the sector.
enum : int { kHoPout = 0, kHoHit = 6, kHoRout = 8, kHoR0 = 9, kHoZref = 10, kHoSec = 11 };

__device__ __forceinline__ void put_word(const DevPtrs& d, int w, uint32_t i, uint32_t v) {
  reinterpret_cast<uint32_t*>(d.tk_cov)[(size_t)w * d.tcap + i] = v;
}
__device__ __forceinline__ uint32_t get_word(const DevPtrs& d, int w, uint32_t i) {
  return reinterpret_cast<const uint32_t*>(d.tk_cov)[(size_t)w * d.tcap + i];
}

__device__ __forceinline__ void set_priority(uint32_t rows_left, uint32_t& level) {
  const uint32_t want = (rows_left >= 75) + (rows_left >= 150) + (rows_left >= 225);
  if (want == level) return;
  level = want;
  if (want == 3) __builtin_amdgcn_s_setprio(3);
  else if (want == 2) __builtin_amdgcn_s_setprio(2);
  else if (want == 1) __builtin_amdgcn_s_setprio(1);
  else __builtin_amdgcn_s_setprio(0);
}

// The order in which an XCD's waves (64 consecutive tracklets or bucket slots
// each) are started: most row steps first, by the start row (k_up) or the
// outermost row (k_down) of the wave's ends.  An XCD holds 512 of them (four
// per SIMD), and those started last run on with its SIMDs emptying; in plain
// order they are as long as any, and on the 32-orbit frame (970 per XCD) 2.5
// (k_up) and 2.9 (k_down) waves per SIMD were resident on average.  Ordered,
// k_up took 911 us instead of 1155 and k_down 1257 instead of 1348 (before their searches were shared by the wave).
// Only the last kOrdered waves are ordered: earlier ones are never among those
// that run on, and the ordered waves of many sectors run side by side, which
// the L2 pays for.  k_down, which reads more of each sector, is left in plain
// order altogether where there are more (512 uneven chunks, 2048 per XCD: k_up
// gains 165 us from ordering the last 1024, k_down would lose 140).
// One workgroup per XCD, one thread per ordered wave: a sort of (rows / 4, wave).
constexpr int kOrderThreads = 1024;
constexpr uint32_t kOrdered = kOrderThreads;
template <bool kDown>
__global__ void __launch_bounds__(kOrderThreads) k_order(DevPtrs d) {
  __shared__ uint32_t v[kOrderThreads];
  const uint32_t n = kDown ? d.k5_off[d.SR] : pipe_n(d), R = d.R;
  const uint32_t need = (n + kThreads - 1) / kThreads, per = (need + kXcds - 1) / kXcds;
  const uint32_t first = min(need, blockIdx.x * per), b1 = min(need, first + per);
  const uint32_t b0 = kDown && b1 - first > kOrdered ? b1 : b1 - min(b1 - first, kOrdered), tid = threadIdx.x;
  for (uint32_t b = first + tid; b < b0; b += kOrderThreads) d.k5_order[b] = b;
  if (b0 == b1) return;   // none to sort
  uint32_t x = 0xFFFFFFFFu;
  if (b0 + tid < b1) {
    const uint32_t j0 = (b0 + tid) * kThreads, j1 = min(n, j0 + kThreads) - 1;
    // rows that the wave does not step through
    const uint32_t key = kDown ? R - 1 - max(get_word(d, kHoRout, d.k5_perm[j0]), get_word(d, kHoRout, d.k5_perm[j1]))
                               : min(d.start_sr[j0] % R, d.start_sr[j1] % R);
    x = ((key / 4) << 16) | tid;
  }
  v[tid] = x;
  __syncthreads();
  for (uint32_t k = 2; k <= (uint32_t)kOrderThreads; k *= 2)   // bitonic, ascending
    for (uint32_t j = k / 2; j > 0; j /= 2) {
      const uint32_t o = tid ^ j;
      if (o > tid) {
        const uint32_t a = v[tid], c = v[o];
        if ((a > c) == ((tid & k) == 0)) {
          v[tid] = c;
          v[o] = a;
        }
      }
      __syncthreads();
    }
  if (b0 + tid < b1) d.k5_order[b0 + tid] = b0 + (v[tid] & 0xFFFFu);
}

__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) k_up(DevPtrs d, KfConst k) {
  extern __shared__ RowK lrows[];   // of the R rows
  __shared__ WaveSearch ws;
  // the state at each lane's outermost hit so far (in LDS rather than registers)
  __shared__ par_t out_p[3][kThreads];
  __shared__ float2 out_hit[kThreads];
  __shared__ uint32_t out_row[kThreads];
  const uint32_t lane = threadIdx.x;
  const uint32_t nt = pipe_n(d);
  const XcdSched sch = xcd_sched(nt);
  if (sch.first >= sch.end) return;   // the grid is sized for the tracklet capacity
  load_rows(d, lrows);
  const uint32_t R = d.R, T = d.tcap;
  uint32_t steps = 0, prio = 0;
  for (uint32_t vb = sch.first; vb < sch.end; vb += sch.stride) {
    const uint32_t i = d.k5_order[vb] * kThreads + threadIdx.x;
    bool on = i < nt && d.tk_info[i] >= 0;   // the lane's tracklet is still stepped
    const bool mine = on;
    const uint32_t sr0 = on ? d.start_sr[i] : 0;
    const uint32_t sec = sr0 / R, srb = sec * R, r0 = sr0 - srb;
    const SectorConst sc = d.secs[sec];
    const uint32_t rl = on ? (uint32_t)d.tk_info[2 * T + i] : 0;
    int32_t* H = d.tk_rowhit + i;     // row r at H[r * T]
    const float2 h0 = on ? d.syz[d.start_pos[i]] : make_float2(0.0f, 0.0f);
    const float zref = h0.y;
    Trk t;
#pragma unroll
    for (int q = 0; q < 5; ++q) t.p[q] = on ? par_t(d.tk_param[(size_t)q * T + i]) : par_t(0);
    set_c0(t, k);
    float chi2 = 0.0f, xprev = lrows[r0].x;
    auto save = [&](float2 h, uint32_t r) {
#pragma unroll
      for (int q = 0; q < 3; ++q) out_p[q][lane] = t.p[2 + q];
      out_hit[lane] = h;
      out_row[lane] = r;
    };
    save(h0, rl);
    int miss = 0;
    bool failed = false;
    // chain fit and outward extension, one row per iteration; while a row is
    // stepped, the chain hits' coordinates are loaded two rows ahead (their
    // indices three) and the next row's grid word one row ahead
    const int32_t hk1 = r0 + 1 <= rl ? H[(size_t)(r0 + 1) * T] : -1;
    float2 hnx = hk1 >= 0 ? d.syz[hk1] : make_float2(0.0f, 0.0f);
    int32_t hk2 = r0 + 2 <= rl ? H[(size_t)(r0 + 2) * T] : -1;
    float2 hn2 = hk2 >= 0 ? d.syz[hk2] : make_float2(0.0f, 0.0f);
    int32_t hk3 = r0 + 3 <= rl ? H[(size_t)(r0 + 3) * T] : -1;
    uint2 mnx = on && r0 + 1 < R && r0 + 1 > rl ? d.row_meta[srb + r0 + 1] : make_uint2(0u, 0u);
    uint32_t r = r0 + 1;
    on = on && r < R;
    // the whole wave steps until its last lane ends: all lanes take part in the search (those that have ended keep
    // their last values)
    float2 hm = make_float2(0.0f, 0.0f);
    uint2 meta = make_uint2(0u, 0u);
    RowK rk{};
    while (__any(on)) {
      bool want = false;
      if (on) {
        // issue priority by the rows still ahead (outward, then about as many inward): a wave far from its
        // end goes first, so fewer waves are left running alone at the end (-1.6% on the 32-orbit frame)
        set_priority(2 * (R - __builtin_amdgcn_readfirstlane(r)), prio);
        const bool chain = r <= rl;
        hm = hnx;
        meta = mnx;
        hnx = hn2;
        hn2 = hk3 >= 0 ? d.syz[hk3] : make_float2(0.0f, 0.0f);
        hk3 = r + 3 <= rl ? H[(size_t)(r + 3) * T] : -1;
        if (r + 1 < R && r + 1 > rl) mnx = d.row_meta[srb + r + 1];
        ++steps;
        rk = lrows[r];
        const bool pok = propagate(t, rk.x - xprev, k);
        xprev = rk.x;
        failed = chain && !pok;
        on = pok && (chain || !(fabs_(t.p[0]) > rk.half_y + k.margin));
        want = on && !chain;
      }
      int32_t h = search_wave(d, InFrame{d.syz, d.bin_start}, ws, want, meta, rk, sc, t, k, zref, hm);
      if (on) {
        if (want) H[(size_t)r * T] = h;
        else h = 0;   // chain rows hold a hit
        if (h >= 0) {
          update(t, hm.x, hm.y - zref, k, chi2);
          if (r >= rl) {
            save(hm, r);
            miss = 0;
          }
        } else if (++miss > k.max_miss) {
          on = false;
        }
        on = on && ++r < R;
      }
    }
    uint32_t key = 0;
    if (mine && failed) d.tk_info[i] = -2;   // the chain fit failed: no tracklet
    on = mine && !failed;
    if (on) {
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const unsigned long long b = (unsigned long long)__double_as_longlong(out_p[q][lane]);
        put_word(d, kHoPout + 2 * q, i, (uint32_t)b);
        put_word(d, kHoPout + 2 * q + 1, i, (uint32_t)(b >> 32));
      }
      const float2 ho = out_hit[lane];
      const uint32_t rout = out_row[lane];
      put_word(d, kHoHit, i, (uint32_t)__float_as_int(ho.x));
      put_word(d, kHoHit + 1, i, (uint32_t)__float_as_int(ho.y));
      put_word(d, kHoRout, i, rout);
      put_word(d, kHoR0, i, r0);
      put_word(d, kHoZref, i, (uint32_t)__float_as_int(zref));
      put_word(d, kHoSec, i, sec);
      key = srb + rout;
    }
    (void)wave_claim(d.row_nstart, key, on);   // count the tracklet in its refit bucket
  }
  uint32_t sum = steps;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) sum += (uint32_t)__shfl_xor((int)sum, off, kWave);
  if (threadIdx.x == 0 && sum) atomicAdd(&d.hdr->n_steps, (unsigned long long)sum);
}

// Scatter of the refit tracklets into (sector, outermost row) order; k5_off
// holds the exclusive scan of the bucket counts (total at [SR]) and serves as
// the buckets' fill cursors.
__global__ void __launch_bounds__(256) k_sort(DevPtrs d) {
  const uint32_t nt = pipe_n(d), R = d.R;
  for (uint32_t b = blockIdx.x * blockDim.x; b < nt; b += gridDim.x * blockDim.x) {   // wave-uniform bounds
    const uint32_t i = b + threadIdx.x;
    const bool on = i < nt && d.tk_info[i] >= 0;
    const uint32_t key = on ? get_word(d, kHoSec, i) * R + get_word(d, kHoRout, i) : 0u;
    const uint32_t slot = wave_claim(d.k5_off, key, on);
    if (on) {
      d.k5_perm[slot] = i;
      d.k5_inv[i] = slot;
    }
  }
}

__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) k_down(DevPtrs d, KfConst k) {
  extern __shared__ RowK lrows[];   // of the R rows
  // the state at each lane's innermost hit so far, in the float32 it is stored
  // in (in LDS rather than registers: four waves per SIMD instead of three)
  __shared__ f32x4 snap_s[5][kThreads];
  __shared__ uint32_t nh_s[kThreads], rin_s[kThreads];
  __shared__ WaveSearch ws;
  const uint32_t lane = threadIdx.x;
  auto save = [&](const Trk& t) {
    const Snap v = snap_of(t);
    snap_s[0][lane] = f32x4{v.p[0], v.p[1], v.p[2], v.p[3]};
#pragma unroll
    for (int q = 0; q < 4; ++q) snap_s[1 + q][lane] = f32x4{q == 0 ? v.p[4] : v.c[4 * q - 1], v.c[4 * q], v.c[4 * q + 1], v.c[4 * q + 2]};
  };
  // bucket order: the refit tracklets (the scan total; the scatter moves only
  // [0, SR)); tracklet order: every tracklet, those without a hand-off skipped
  const bool sorted = d.k5_refit_order == 0;
  const uint32_t nv = sorted ? d.k5_off[d.SR] : pipe_n(d);
  const uint32_t R = d.R, T = d.tcap;
  const XcdSched sch = xcd_sched(nv);
  if (sch.first >= sch.end) return;   // the grid is sized for the tracklet capacity
  load_rows(d, lrows);
  uint32_t steps = 0, prio = 0;
  for (uint32_t vb = sch.first; vb < sch.end; vb += sch.stride) {
    const uint32_t j = (sorted ? d.k5_order[vb] : vb) * kThreads + threadIdx.x;
    const bool mine = j < nv && (sorted || d.tk_info[j] >= 0);
    const uint32_t i = !mine ? 0 : sorted ? d.k5_perm[j] : j;
    Trk t;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const unsigned long long b = (unsigned long long)get_word(d, kHoPout + 2 * q, i) |
                                   ((unsigned long long)get_word(d, kHoPout + 2 * q + 1, i) << 32);
      t.p[2 + q] = __longlong_as_double((long long)b);
    }
    const float hy = __int_as_float((int)get_word(d, kHoHit, i)), hz = __int_as_float((int)get_word(d, kHoHit + 1, i));
    const uint32_t rout = mine ? get_word(d, kHoRout, i) : 0, r0 = mine ? get_word(d, kHoR0, i) : 0;
    const float zref = __int_as_float((int)get_word(d, kHoZref, i));
    const uint32_t sec = mine ? get_word(d, kHoSec, i) : 0, srb = sec * R;
    const SectorConst sc = d.secs[sec];
    int32_t* H = d.tk_rowhit + i;     // row r at H[r * T]
    // inward refit from the outermost hit, fresh covariance
    t.p[0] = hy;
    t.p[1] = hz - zref;
    set_c0(t, k);
    float chi2 = 0.0f;
    nh_s[lane] = 1;
    save(t);
    rin_s[lane] = rout;
    float xprev = lrows[rout].x;
    int miss = 0;
    // the outward pass's row -> hit entries are loaded three rows ahead and
    // their coordinates two rows ahead, the next row's grid word one row ahead
    auto known = [&](int r) { return r >= (int)r0 && r >= 0 ? H[(size_t)r * T] : -1; };
    int32_t hA = known((int)rout - 1), hB = known((int)rout - 2), hC = known((int)rout - 3);
    float2 vA = hA >= 0 ? d.syz[hA] : make_float2(0.0f, 0.0f);
    float2 vB = hB >= 0 ? d.syz[hB] : make_float2(0.0f, 0.0f);
    uint2 mA = rout >= 1 ? d.row_meta[srb + rout - 1] : make_uint2(0u, 0u);
    int r = (int)rout - 1;
    bool on = mine && r >= 0;
    float2 hm = make_float2(0.0f, 0.0f);
    uint2 meta = make_uint2(0u, 0u);
    RowK rk{};
    int32_t h = -1;
    while (__any(on)) {   // the whole wave, as in the outward pass
      bool want = false, below = false;
      if (on) {
        set_priority(2 * (uint32_t)__builtin_amdgcn_readfirstlane(r), prio);
        h = hA;
        hm = vA;
        meta = mA;
        hA = hB;
        vA = vB;
        hB = hC;
        vB = hC >= 0 ? d.syz[hC] : make_float2(0.0f, 0.0f);
        hC = known(r - 3);
        if (r >= 1) mA = d.row_meta[srb + (uint32_t)r - 1];
        rk = lrows[r];
        ++steps;
        const bool pok = propagate(t, rk.x - xprev, k);
        xprev = rk.x;
        below = (uint32_t)r < r0;
        on = pok && !(below && fabs_(t.p[0]) > rk.half_y + k.margin);
        want = on && h < 0;
      }
      const int32_t hs = search_wave(d, InFrame{d.syz, d.bin_start}, ws, want, meta, rk, sc, t, k, zref, hm);
      if (on) {
        if (want) h = hs;
        // the row's entry changes only where the refit searched: below the start
        // row (never written before) or in a gap the outward pass left
        if (want && (below || h >= 0)) H[(size_t)r * T] = h;
        if (h >= 0) {
          update(t, hm.x, hm.y - zref, k, chi2);
          __hip_atomic_fetch_add(&nh_s[lane], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
          save(t);
          rin_s[lane] = (uint32_t)r;
          if (below) miss = 0;
        } else if (below && ++miss > k.max_miss) {
          on = false;
        }
        on = on && --r >= 0;
      }
    }
    if (!mine) continue;
    const int nh = (int)nh_s[lane];
    const uint32_t rin = rin_s[lane];
    Snap snap;
    const f32x4 w0 = snap_s[0][lane];
    snap.p[0] = w0.x;
    snap.p[1] = w0.y;
    snap.p[2] = w0.z;
    snap.p[3] = w0.w;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 w = snap_s[1 + q][lane];
      if (q == 0) snap.p[4] = w.x;
      else snap.c[4 * q - 1] = w.x;
      snap.c[4 * q] = w.y;
      snap.c[4 * q + 1] = w.z;
      snap.c[4 * q + 2] = w.w;
    }
    if (sorted) {   // the record at the tracklet's bucket slot: consecutive lanes, consecutive records
      uint32_t* rec = d.k5_rec + (size_t)j * kRecWords;
      rec[kRecInfo] = (uint32_t)nh;
      rec[kRecInfo + 1] = rin;
      rec[kRecInfo + 2] = rout;
      rec[kRecInfo + 3] = r0;
#pragma unroll
      for (int q = 0; q < 5; ++q) rec[kRecParam + q] = (uint32_t)__float_as_int(q == 1 ? snap.p[q] + zref : snap.p[q]);
#pragma unroll
      for (int q = 0; q < 15; ++q) rec[kRecCov + q] = (uint32_t)__float_as_int(snap.c[q]);
      rec[kRecChi2] = (uint32_t)__float_as_int(chi2);
    } else {
      store_tracklet<false>(d, i, nh, rin, rout, r0, snap, chi2, zref);
    }
  }
  uint32_t sum = steps;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) sum += (uint32_t)__shfl_xor((int)sum, off, kWave);
  if (threadIdx.x == 0 && sum) atomicAdd(&d.hdr->n_steps, (unsigned long long)sum);
}

// ---------------------------------------------------------------------------
// Row-synchronous schedule ("coalesced row-grid reads").  A wave takes up to
// 64 / kL tracklets of ONE sector, kL lanes per tracklet: they split each
// candidate search and run the rest of the step redundantly (kL = 1: the whole
// wave shares its searches, search_wave).  After each tracklet's lanes have
// walked its chain and built its seed, the wave sweeps the rows
// in lockstep -- outward, then inward --
// and at every row stages that row's (y, z) and bin starts in LDS with one
// coalesced load shared by all lanes; the loads for the next row are issued
// before the current row's Kalman step and land in registers while it runs.
// Every search and every measurement read then hits LDS, which takes the
// dependent global-memory round trips out of the per-row critical path.  Rows
// larger than the stage fall back to global-memory search for that row.
//
// The stage is filled with 16-byte loads that every lane issues
// unconditionally: the (y, z) pairs from the even index at or below the row's
// first hit, the bin starts from the multiple of four at or below the row's
// first bin (both arrays carry padding at their ends, so reads past a row stay
// inside the allocation).  A load whose slot lies past the row re-reads the
// first one; the stage entries it fills are never used.
constexpr int kStageHits = 320;
constexpr int kStageBins = kStageHits + 2;                       // nBins + 1 <= N_r + 1
constexpr int kPreYz = 3;   // float4 loads per lane: 2 hits each
constexpr int kPreBs = 2;   // uint4 loads per lane: 4 bin starts each
// alignment slack (1), whole-group reads past a z-line (kGroupLds - 1)
static_assert(kPreYz * kThreads * 2 >= kStageHits + 1 + kGroupLds - 1, "yz stage too small");
static_assert(kPreBs * kThreads * 4 >= kStageBins + 3, "bin stage too small");

struct Stage {
  uint32_t first;   // global index of stage entry 0 (even, <= the row's first hit)
  uint32_t boff;    // stage index of the row's bin 0
  uint2 meta;
  RowK rk;
  bool fits;
};


struct Prefetch {
  f32x4 yz[kPreYz];
  u32x4 bs[kPreBs];
  Stage st;
};

__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = min(v, (uint32_t)__shfl_xor((int)v, off, kWave));
  return v;
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, off, kWave));
  return v;
}

// Issue the loads of sector row r (wave-uniform) into registers.  The row's
// offsets and grid word come from the wave's LDS copy of the sector's row
// table, so no load here waits on another; only the 64-entry chunks the row
// needs are loaded (a scalar decision), each lane from an index clamped into
// the row, so the loads need no per-lane predication.
// Issue priority of a wave from the rows it still has to step through (a
// longest-remaining-first order for the waves that share a SIMD); `level`
// holds the wave's current setting, so the instruction is issued on changes only.
__device__ __forceinline__ float uniform_f(float v) {
  return __int_as_float((int)__builtin_amdgcn_readfirstlane((uint32_t)__float_as_int(v)));
}
template <bool kAllFit>
__device__ __forceinline__ void prefetch_row(const DevPtrs& d, const RowK* lrows, const uint32_t* roff_s,
                                             const uint2* meta_s, uint32_t r, Prefetch& pf) {
  const uint32_t lane = threadIdx.x;
  const uint32_t a = __builtin_amdgcn_readfirstlane(roff_s[r]);
  const uint32_t n = __builtin_amdgcn_readfirstlane(roff_s[r + 1]) - a;
  const uint2 meta = meta_s[r];
  pf.st.meta = make_uint2(__builtin_amdgcn_readfirstlane(meta.x), __builtin_amdgcn_readfirstlane(meta.y));
  const RowK rk = lrows[r];   // the row's constants, for the step that uses the stage
  pf.st.rk = RowK{uniform_f(rk.x), uniform_f(rk.half_y), uniform_f(rk.y_lo), uniform_f(rk.inv_wy)};
  pf.st.fits = kAllFit || n <= (uint32_t)kStageHits;
  const uint32_t ybase = a & ~1u, ycnt = a + n - ybase;
  pf.st.first = ybase;
  const uint32_t bbase = pf.st.meta.x & ~3u;
  pf.st.boff = pf.st.meta.x - bbase;
  if (!pf.st.fits) return;
  const f32x4* ysrc = reinterpret_cast<const f32x4*>(d.syz + ybase);
#pragma unroll
  for (int m = 0; m < kPreYz; ++m) {
    const uint32_t q = lane + m * kThreads;   // pair q holds entries 2q, 2q + 1
    pf.yz[m] = ysrc[2 * q < ycnt ? q : 0];
  }
  const uint32_t bcnt = pf.st.boff + (pf.st.meta.y & 0xFFFFu) * (pf.st.meta.y >> 16) + 1;   // every row has a grid
  const u32x4* bsrc = reinterpret_cast<const u32x4*>(d.bin_start + bbase);
#pragma unroll
  for (int m = 0; m < kPreBs; ++m) {
    const uint32_t q = lane + m * kThreads;   // quad q holds entries 4q .. 4q + 3
    pf.bs[m] = bsrc[4 * q < bcnt ? q : 0];
  }
}

// Write prefetched registers to the LDS stage (call between two barriers).
__device__ __forceinline__ void commit_row(const Prefetch& pf, f32x4* yz4_s, u32x4* bs4_s, Stage& st) {
  const uint32_t lane = threadIdx.x;
  st = pf.st;
  if (!st.fits) return;
#pragma unroll
  for (int m = 0; m < kPreYz; ++m) yz4_s[lane + m * kThreads] = pf.yz[m];
#pragma unroll
  for (int m = 0; m < kPreBs; ++m) bs4_s[lane + m * kThreads] = pf.bs[m];
}

// Bound: the longest wave's chain of some 300 row steps, each a stream of about
// 500 vector instructions that one wave issues at one in 5 cycles (of 4400
// cycles a step on a sector of 22k hits, 3200 are the step, 600 the next row's
// loads and 260 the wait for them).  More lanes per tracklet shorten the step's
// search, as long as the waves stay alone, or two together, on their SIMDs:
// fewer lanes where there are more tracklets (row_lanes).  Registers: three
// waves per SIMD at two lanes (a central event has 2400 waves; 24 values
// spilled, and still faster than two waves per SIMD), two at one lane, any
// number above, where nothing spills.
template <bool kAllFit, int kL>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(kL == 2 ? 3 : kL == 1 ? 2 : 1)))
k_tracklets_rs(DevPtrs d, KfConst k) {
  __shared__ RowK lrows[kMaxRows];
  __shared__ f32x4 yz4_s[kPreYz * kThreads];   // the staged row: (y, z) pairs
  __shared__ u32x4 bs4_s[kPreBs * kThreads];   // and its bin starts
  const float2* yz_s = reinterpret_cast<const float2*>(yz4_s);
  const uint32_t* bs_s = reinterpret_cast<const uint32_t*>(bs4_s);
  __shared__ uint32_t roff_s[kMaxRows + 1];   // the current sector's row offsets
  __shared__ uint2 meta_s[kMaxRows];          // and grid words
  __shared__ WaveSearch ws;                    // kL = 1
  const uint32_t R = d.R, T = d.tcap, S = d.S;
  const uint32_t lane = threadIdx.x;
  const uint32_t W = d.wave_off[S];
  // XCD-contiguous ranges of waves (one wave per block, waves ordered by sector)
  const uint32_t per = (W + kXcds - 1) / kXcds;
  const uint32_t xcd = blockIdx.x % kXcds;
  const uint32_t vend = min(W, (xcd + 1) * per);
  // the grid is sized for the tracklet capacity; blocks without a wave leave at once
  if (xcd * per + blockIdx.x / kXcds >= vend) return;
  load_rows(d, lrows);
  unsigned long long my_steps = 0;
  uint32_t prio = 0;   // s_setprio level of this wave (waves start at 0)
  for (uint32_t v = xcd * per + blockIdx.x / kXcds; v < vend; v += gridDim.x / kXcds) {
    // sector of wave v: last s with wave_off[s] <= v
    uint32_t lo = 0, hi = S;
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) / 2;
      if (d.wave_off[mid] <= v) lo = mid; else hi = mid;
    }
    const uint32_t sec = lo, srb = sec * R;
    const uint32_t ts = min(d.row_start_off[srb], T), te = min(d.row_start_off[srb + R], T);
    const uint32_t sub = lane % kL;   // the lanes of a tracklet compute the same and store identical values
    const uint32_t i = ts + (v - d.wave_off[sec]) * (kThreads / kL) + lane / kL;
    const SectorConst sc = d.secs[sec];
    int32_t* H = d.tk_rowhit + i;
    __syncthreads();   // the previous wave's last reads of the row table are done
    for (uint32_t q = lane; q <= R; q += kThreads) {
      roff_s[q] = d.row_off[srb + q];
      if (q < R) meta_s[q] = d.row_meta[srb + q];
    }
    __syncthreads();
    // ---- per lane: chain walk and seed ----
    bool ok = i < te;
    uint32_t r0 = 0, rl = 0, n = 0;
    float zref = 0.0f, chi2 = 0.0f, xprev = 0.0f;
    Trk t;
    if (ok) {
      const uint32_t sr0 = d.start_sr[i];
      r0 = sr0 % R;
      int32_t p = (int32_t)d.start_pos[i];
      int32_t plast = p;
      while (p >= 0 && r0 + n < R) {
        H[(size_t)(r0 + n) * T] = p;
        plast = p;
        ++n;
        p = d.up1[p];
      }
      const uint32_t m = (n - 1) / 2;
      rl = r0 + n - 1;
      const int32_t pm = H[(size_t)(r0 + m) * T];
      const float2 h0 = d.syz[d.start_pos[i]];
      zref = h0.y;
      if (seed3(lrows[r0].x, h0, lrows[r0 + m].x, d.syz[pm], lrows[rl].x, d.syz[plast], k, t)) {
        set_c0(t, k);
        xprev = lrows[r0].x;
      } else {
        d.tk_info[i] = -1;
        ok = false;
      }
    }
    uint32_t steps = ok ? n - 1 : 0;
    // ---- outward sweep ----
    bool up = ok, failed = false;
    par_t pout[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) pout[q] = t.p[q];
    uint32_t rout = rl;
    int miss = 0;
    Stage st;
    Prefetch pf;
    // the staged row's search: one lane's, or the wave's (called converged, for the lanes that want one)
    auto find = [&](uint32_t sr, float2& hm) {
      if (!(kAllFit || st.fits)) return search(d, sr, st.rk, sc, t, k, zref, hm);
      const int32_t h = search_lds<kL>(yz_s, bs_s + st.boff, st.first, st.meta, st.rk, sc, t, k, zref, sub);
      if (h >= 0) hm = yz_s[(uint32_t)h - st.first];
      return h;
    };
    auto find_all = [&](bool want, float2& hm) {
      return kAllFit || st.fits
                 ? search_wave(d, InStage{yz_s, bs_s + st.boff, st.first, st.meta.x}, ws, want, st.meta, st.rk, sc, t, k, zref, hm)
                 : search_wave(d, InFrame{d.syz, d.bin_start}, ws, want, st.meta, st.rk, sc, t, k, zref, hm);
    };
    auto hit = [&](int32_t h) { return (kAllFit || st.fits) ? yz_s[(uint32_t)h - st.first] : d.syz[h]; };
    uint32_t r = __builtin_amdgcn_readfirstlane(wave_min(up ? r0 + 1 : R));   // wave-uniform from here on
    if (r < R) {
      prefetch_row<kAllFit>(d, lrows, roff_s, meta_s, r, pf);
      commit_row(pf, yz4_s, bs4_s, st);
      __syncthreads();
    }
    int32_t hnext = (up && r <= rl && r > r0) ? H[(size_t)r * T] : -1;
    // Drain every load issued so far (the sector constants, the first row, the
    // chain hit) before the loop: the compiler's wait counters are tracked per
    // register across the back edge, and a value still pending from before the
    // loop would otherwise make every iteration wait for all its loads --
    // including the prefetch of the next row, which should overlap the step.
    __builtin_amdgcn_s_waitcnt(0);
    while (r < R && __any(up)) {
      set_priority(2 * R - r, prio);   // the rest of this sweep, then (about) the whole inward sweep
      if (r + 1 < R) prefetch_row<kAllFit>(d, lrows, roff_s, meta_s, r + 1, pf);
      const int32_t hchain = hnext;
      hnext = (up && r + 1 <= rl && r + 1 > r0) ? H[(size_t)(r + 1) * T] : -1;
      // flags instead of nested branches: a lane that stops here keeps nothing of this step (its state is not read again)
      const bool chain = r <= rl;
      bool go = false;
      int32_t h = hchain;
      float2 hm;
      auto finish = [&] {
        if (go && !chain) H[(size_t)r * T] = h;
        if (go && h >= 0) {
          if (chain) hm = hit(h);
          update(t, hm.x, hm.y - zref, k, chi2);
          if (r >= rl) {
#pragma unroll
            for (int q = 0; q < 5; ++q) pout[q] = t.p[q];
            rout = r;
            miss = 0;
          }
        }
        const bool missed = go && h < 0;
        miss += missed ? 1 : 0;
        up = up && !(missed && miss > k.max_miss);
      };
      if (up && r > r0) {
        const RowK rk = st.rk;
        steps += chain ? 0u : 1u;
        const bool pok = propagate(t, rk.x - xprev, k);
        xprev = rk.x;
        failed = failed || (!pok && chain);
        go = pok && (chain || fabs_(t.p[0]) <= rk.half_y + k.margin);
        up = go;
        if constexpr (kL > 1) {
          if (go && !chain) h = find(srb + r, hm);
          finish();
        }
      }
      if constexpr (kL == 1) {
        const int32_t hs = find_all(go && !chain, hm);
        if (go && !chain) h = hs;
        if (go) finish();
      }
      __syncthreads();
      if (r + 1 < R) commit_row(pf, yz4_s, bs4_s, st);
      __syncthreads();
      ++r;
    }
    if (failed) {
      d.tk_info[i] = -2;
      ok = false;
    }
    // ---- inward sweep from each lane's outermost hit, fresh covariance ----
    bool down = ok;
    int nh = 1;
    Snap snap;
    uint32_t rin = rout;
    if (down) {
      const float2 ho = d.syz[H[(size_t)rout * T]];
#pragma unroll
      for (int q = 2; q < 5; ++q) t.p[q] = pout[q];
      t.p[0] = ho.x;
      t.p[1] = ho.y - zref;
      set_c0(t, k);
      chi2 = 0.0f;
      snap = snap_of(t);
      xprev = lrows[rout].x;
      miss = 0;
    }
    int32_t rr = (int32_t)__builtin_amdgcn_readfirstlane(wave_max(down ? rout : 0)) - 1;
    if (rr >= 0) {
      prefetch_row<kAllFit>(d, lrows, roff_s, meta_s, (uint32_t)rr, pf);
      commit_row(pf, yz4_s, bs4_s, st);
      __syncthreads();
    }
    hnext = (down && rr >= (int32_t)r0 && rr < (int32_t)rout) ? H[(size_t)rr * T] : -1;
    __builtin_amdgcn_s_waitcnt(0);   // as before the outward sweep
    while (rr >= 0 && __any(down)) {
      set_priority((uint32_t)rr, prio);
      if (rr > 0) prefetch_row<kAllFit>(d, lrows, roff_s, meta_s, (uint32_t)rr - 1, pf);
      const int32_t hrow = hnext;
      hnext = (down && rr - 1 >= (int32_t)r0 && rr - 1 < (int32_t)rout) ? H[(size_t)(rr - 1) * T] : -1;
      const bool below = (uint32_t)rr < r0;
      bool go = false;
      int32_t h = below ? -1 : hrow;
      float2 hm;
      auto finish = [&] {
        if (go && (below || h != hrow)) H[(size_t)rr * T] = h;   // changed only where the refit searched
        if (go && h >= 0) {
          if (!below && h == hrow) hm = hit(h);
          update(t, hm.x, hm.y - zref, k, chi2);
          ++nh;
          snap = snap_of(t);
          rin = (uint32_t)rr;
          if (below) miss = 0;
        }
        const bool missed = go && below && h < 0;
        miss += missed ? 1 : 0;
        down = down && !(missed && miss > k.max_miss);
      };
      if (down && rr < (int32_t)rout) {   // flags, as in the outward sweep
        const RowK rk = st.rk;
        ++steps;
        const bool pok = propagate(t, rk.x - xprev, k);
        xprev = rk.x;
        go = pok && !(below && fabs_(t.p[0]) > rk.half_y + k.margin);
        down = go;
        if constexpr (kL > 1) {
          if (go && h < 0) h = find(srb + (uint32_t)rr, hm);
          finish();
        }
      }
      if constexpr (kL == 1) {
        const int32_t hs = find_all(go && h < 0, hm);
        if (go && h < 0) h = hs;
        if (go) finish();
      }
      __syncthreads();
      if (rr > 0) commit_row(pf, yz4_s, bs4_s, st);
      __syncthreads();
      --rr;
    }
    if (ok) {
      store_tracklet<true>(d, i, nh, rin, rout, r0, snap, chi2, zref);
      if (sub == 0) my_steps += steps;
    }
  }
  if (my_steps) atomicAdd(&d.hdr->n_steps, my_steps);
}

// ---------------------------------------------------------------------------
// Row-synchronous schedule on resident sectors.  Where a whole sector fits in
// the LDS of a compute unit (hits, bin starts, chain links and the row -> hit
// columns of its workgroup's tracklets), a workgroup loads it once and its
// waves sweep the rows without touching global memory and without barriers.
// In k_tracklets_rs the next row's staging took about half of a row step: of
// 4360 cycles on a pp frame 800 went into issuing its loads and 1400 into
// waiting for them (a sector's few waves read each row first in their XCD, at
// the latency of the last-level cache).
//
// Few tracklets leave the card idle, and the time is one wave's chain of
// dependent steps, so kL lanes share a tracklet (2 .. 16: as many as keep every
// wave alone on its SIMD): they test the candidates of a search side by side,
// which makes each step shorter, and run the rest redundantly.
//
// Against k_tracklets_rs: a pp frame of one orbit 504 -> 334 us, of four orbits
// 578 -> 413 us, one chunk of 5k hits 540 -> 330 us.
constexpr int kResThreads = 256;
constexpr uint32_t kResLdsBytes = 160u << 10;
constexpr uint32_t kResPer = kResThreads / 2;   // tracklets of a workgroup, at two lanes each
constexpr uint32_t kResRowHits = 254;  // a column holds a hit's place in its row in a byte
constexpr uint32_t kNoHit = 255;
constexpr uint32_t kNoLink = 0xFFFFu;
constexpr uint32_t kRowTable = 32;     // bytes of a row in the row table: RowK, then a RowInfo

// LDS of a sector of up to cap hits, its positions relative to the sector's first (16-bit): hits, row table, bin starts,
// the columns of kResPer tracklets, and the links where there is room for them.
struct ResLds {
  uint32_t rows, bs, col, up, total;   // byte offsets; hits at 0; up 0: no links; total 0: the sector does not fit
};
inline ResLds res_lds(uint32_t cap, uint32_t max_row, uint32_t R, uint32_t hits_per_bin) {
  auto up16 = [](uint32_t v) { return (v + 15u) & ~15u; };
  ResLds l{};
  if (cap >= kNoLink || max_row > kResRowHits) return l;
  l.rows = up16(8 * cap);
  l.bs = up16(l.rows + kRowTable * R);
  l.col = up16(l.bs + 2 * (cap / hits_per_bin + 2 * R));
  const uint32_t end = up16(l.col + R * kResPer), with_up = up16(end + 2 * cap);
  if (end > kResLdsBytes) return l;
  l.up = with_up <= kResLdsBytes ? end : 0u;
  l.total = l.up ? with_up : end;
  return l;
}

// A row in the row table; hits are named by their place, the sorted position less the sector's first.
struct RowInfo {
  uint32_t first, n, bins, dims;   // place of the first hit, hits, place of bin 0 among the bin starts, ny | nz << 16
};
struct RowEntry {
  f32x4 k;
  u32x4 i;
};

// The search of C5 in a resident row: the place of the candidate closest to
// the prediction, -1 if none.  Rows of few hits are tested whole; otherwise the
// bins of the window, two z-lines at a time as one flat sequence (few-bin lines
// all at once, see search_m).  The lanes of a tracklet take kU candidates in
// turn; then the smallest deviation wins, ties to the smaller place.
template <int kL>
__device__ __forceinline__ int32_t search_row(const float2* yz, const uint16_t* bsec, const RowInfo& rr, const RowK& rk,
                                              const SectorConst& sc, const Trk& t, const KfConst& k, float zref,
                                              uint32_t sub) {
  constexpr uint32_t kU = kL >= 8 ? 1 : kL == 4 ? 2 : 4;
  const float sy2 = float(t.c[0] + k.vyd), sz2 = float(t.c[2] + k.vzd);
  const float wy = fminf(k.gate * fsqrt(sy2), k.cap), wz = fminf(k.gate * fsqrt(sz2), k.cap);
  const float isy = frcp(sy2), isz = frcp(sz2);
  const float yp = float(t.p[0]), zp = float(t.p[1]);
  uint32_t best = 0xFFFFFFFFu;
  float bd = INFINITY;
  // candidates lo0 .. lo0 + n0 - 1, then lo1 .., tot in all
  auto test = [&](uint32_t lo0, uint32_t n0, uint32_t lo1, uint32_t tot) {
    for (uint32_t f0 = sub * kU; f0 < tot; f0 += kL * kU) {
      uint32_t pos[kU];
      float2 h[kU];
#pragma unroll
      for (uint32_t j = 0; j < kU; ++j) {
        const uint32_t f = min(f0 + j, tot - 1);
        pos[j] = f < n0 ? lo0 + f : lo1 + (f - n0);
        h[j] = yz[pos[j]];
      }
#pragma unroll
      for (uint32_t j = 0; j < kU; ++j) {   // a clamped place is tested twice, which changes nothing
        const float dy = h[j].x - yp, dz = (h[j].y - zref) - zp;
        const float dd = __builtin_fmaf(dy * dy, isy, (dz * dz) * isz);
        const bool take = fabsf(dy) <= wy & fabsf(dz) <= wz & dd < bd;
        best = take ? pos[j] : best;
        bd = take ? dd : bd;
      }
    }
  };
  if (rr.n <= 2 * kL * kU) {   // wave-uniform
    if (rr.n) test(rr.first, rr.n, 0u, rr.n);
  } else {
    const float za = zref + zp;
    const int ny = (int)(rr.dims & 0xFFFFu), nz = (int)(rr.dims >> 16);
    const int iy0 = bin1((yp - wy) - kWinPad, rk.y_lo, rk.inv_wy, ny);
    const int iy1 = bin1((yp + wy) + kWinPad, rk.y_lo, rk.inv_wy, ny);
    const int iz0 = bin1((za - wz) - kWinPad, sc.z_lo, sc.inv_wz, nz);
    const int iz1 = bin1((za + wz) + kWinPad, sc.z_lo, sc.inv_wz, nz);
    const uint16_t* bs = bsec + rr.bins;
    if (ny <= kRunBins) {
      const uint32_t lo = bs[iz0 * ny + iy0], n = bs[iz1 * ny + iy1 + 1] - lo;
      test(lo, n, 0u, n);
    } else {
      for (int iz = iz0; iz <= iz1; iz += 2) {
        const int izb = iz + 1 <= iz1 ? iz + 1 : iz;
        const uint32_t lo0 = bs[iz * ny + iy0], n0 = bs[iz * ny + iy1 + 1] - lo0;
        const uint32_t lo1 = bs[izb * ny + iy0], n1 = bs[izb * ny + iy1 + 1] - lo1;
        test(lo0, n0, lo1, n0 + (izb > iz ? n1 : 0u));
      }
    }
  }
  // deviations are not negative, so their bits order as they do
  const uint32_t mine = (uint32_t)__float_as_int(bd), least = group_min<kL>(mine);
  return (int32_t)group_min<kL>(mine == least ? best : 0xFFFFFFFFu);
}

__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane(v); }

// A sector in LDS.
struct Resident {
  const float2* yz;
  const f32x4* rows;         // the row table
  const uint16_t *bs, *up;   // bin starts; links (nullptr: not resident)
  uint32_t a0;               // the sector's first sorted position

  // A row is the same for the whole wave; its entry is read a step before it is needed (into vector registers, no wait)
  // and moved to scalar registers then.  Scalar loads would not do: they share a counter with LDS reads but return out of
  // order, so the step's first LDS read would wait for them.
  __device__ __forceinline__ RowEntry entry(uint32_t r) const {
    return RowEntry{rows[2 * r], *reinterpret_cast<const u32x4*>(rows + 2 * r + 1)};
  }
  __device__ __forceinline__ float x(uint32_t r) const { return reinterpret_cast<const float*>(rows + 2 * r)[0]; }
  __device__ __forceinline__ uint32_t first(uint32_t r) const {
    return reinterpret_cast<const uint32_t*>(rows + 2 * r + 1)[0];
  }
  // the place after p in its chain, kNoLink at its end
  __device__ __forceinline__ uint32_t next(const DevPtrs& d, uint32_t p) const {
    if (up) return up[p];
    const int32_t u = d.up1[a0 + p];
    return u >= 0 ? (uint32_t)u - a0 : kNoLink;
  }
};
__device__ __forceinline__ RowK row_k(const RowEntry& e) {
  return RowK{uniform_f(e.k.x), uniform_f(e.k.y), uniform_f(e.k.z), uniform_f(e.k.w)};
}
__device__ __forceinline__ RowInfo row_info(const RowEntry& e) {
  return RowInfo{uniform(e.i.x), uniform(e.i.y), uniform(e.i.z), uniform(e.i.w)};
}

// Chain, seed and both sweeps of tracklet i, kL lanes; returns its row steps on
// the lane that writes.  col[r * kPer] is the hit in row r, as its place in the
// row: one lane of the tracklet writes it and all of them read it, so every
// point between the two is ordered (no instruction: a wave's LDS accesses
// complete in order).
template <int kL, uint32_t kPer>
__device__ __forceinline__ uint32_t sweep(const DevPtrs& d, const KfConst& k, const Resident& S, uint8_t* col, uint32_t sec,
                                          uint32_t i, uint32_t te) {
  const uint32_t R = d.R, T = d.tcap, sub = threadIdx.x % kL;
  const bool writes = sub == 0;   // of the lanes of a tracklet, which hold the same
  const SectorConst sc = d.secs[sec];
  bool ok = i < te;
  uint32_t r0 = 0, rl = 0, n = 0;
  float zref = 0.0f, chi2 = 0.0f, xprev = 0.0f;
  Trk t;
  wave_lds_order();   // the lanes' last reads of the previous tracklet's column
  if (ok) {
    r0 = d.start_sr[i] - sec * R;
    const uint32_t p0 = d.start_pos[i] - S.a0;
    // chain walk: its rows of the column and, following at half the speed, its middle hit
    uint32_t p = p0, last = p0, mid = p0;
    while (p != kNoLink && r0 + n < R) {
      last = p;
      if (writes) col[(r0 + n) * kPer] = (uint8_t)(p - S.first(r0 + n));
      if (n && n % 2 == 0) mid = S.next(d, mid);
      p = S.next(d, p);
      ++n;
    }
    rl = r0 + n - 1;
    const float2 h0 = S.yz[p0];
    zref = h0.y;
    if (seed3(S.x(r0), h0, S.x(r0 + (n - 1) / 2), S.yz[mid], S.x(rl), S.yz[last], k, t)) {
      set_c0(t, k);
      xprev = S.x(r0);
    } else {
      if (writes) d.tk_info[i] = -1;
      ok = false;
    }
  }
  uint32_t steps = ok ? n - 1 : 0;
  // ---- outward sweep ----
  bool up = ok, failed = false;
  par_t pout[3] = {t.p[2], t.p[3], t.p[4]};
  uint32_t rout = rl;
  int miss = 0;
  wave_lds_order();   // the chain's rows of the column
  uint32_t r = uniform(wave_min(up ? r0 + 1 : R));
  RowEntry next = S.entry(r < R ? r : 0);
  uint32_t hnext = r < R ? col[r * kPer] : kNoHit;   // used only in chain rows
  for (; r < R && __any(up); ++r) {
    const RowInfo row = row_info(next);
    const RowK rk = row_k(next);
    const uint32_t hchain = hnext, rn = r + 1 < R ? r + 1 : r;
    next = S.entry(rn);
    hnext = col[rn * kPer];
    if (up && r > r0) {
      const bool chain = r <= rl;
      steps += chain ? 0u : 1u;
      const bool pok = propagate(t, rk.x - xprev, k);
      xprev = rk.x;
      failed = failed || (!pok && chain);
      const bool go = pok && (chain || fabs_(t.p[0]) <= rk.half_y + k.margin);
      up = go;
      int32_t h = chain ? (int32_t)(row.first + hchain) : -1;
      if (go && !chain) {
        h = search_row<kL>(S.yz, S.bs, row, rk, sc, t, k, zref, sub);
        if (writes) col[r * kPer] = (uint8_t)(h >= 0 ? (uint32_t)h - row.first : kNoHit);
      }
      if (go && h >= 0) {
        const float2 hm = S.yz[h];
        update(t, hm.x, hm.y - zref, k, chi2);
        if (r >= rl) {
#pragma unroll
          for (int q = 0; q < 3; ++q) pout[q] = t.p[2 + q];
          rout = r;
          miss = 0;
        }
      }
      const bool missed = go && h < 0;
      miss += missed ? 1 : 0;
      up = up && !(missed && miss > k.max_miss);
    }
    wave_lds_order();   // the row's column entry
  }
  if (failed) {
    if (writes) d.tk_info[i] = -2;
    ok = false;
  }
  // ---- inward sweep from each lane's outermost hit, fresh covariance ----
  bool down = ok;
  int nh = 1;
  Snap snap;
  uint32_t rin = rout;
  if (down) {
    const float2 ho = S.yz[S.first(rout) + col[rout * kPer]];
#pragma unroll
    for (int q = 0; q < 3; ++q) t.p[2 + q] = pout[q];
    t.p[0] = ho.x;
    t.p[1] = ho.y - zref;
    set_c0(t, k);
    chi2 = 0.0f;
    snap = snap_of(t);
    xprev = S.x(rout);
    miss = 0;
  }
  int32_t q = (int32_t)uniform(wave_max(down ? rout : 0)) - 1;
  next = S.entry(q >= 0 ? (uint32_t)q : 0);
  hnext = q >= 0 ? col[(uint32_t)q * kPer] : kNoHit;   // used only in [r0, rout)
  for (; q >= 0 && __any(down); --q) {
    const RowInfo row = row_info(next);
    const RowK rk = row_k(next);
    const uint32_t hrow = hnext, qn = q > 0 ? (uint32_t)q - 1 : 0;
    next = S.entry(qn);
    hnext = col[qn * kPer];
    if (down && q < (int32_t)rout) {
      ++steps;
      const bool pok = propagate(t, rk.x - xprev, k);
      xprev = rk.x;
      const bool below = (uint32_t)q < r0;
      const bool go = pok && !(below && fabs_(t.p[0]) > rk.half_y + k.margin);
      down = go;
      int32_t h = below || hrow == kNoHit ? -1 : (int32_t)(row.first + hrow);
      if (go && h < 0) {
        h = search_row<kL>(S.yz, S.bs, row, rk, sc, t, k, zref, sub);
        if (writes) col[(uint32_t)q * kPer] = (uint8_t)(h >= 0 ? (uint32_t)h - row.first : kNoHit);
      }
      if (go && h >= 0) {
        const float2 hm = S.yz[h];
        update(t, hm.x, hm.y - zref, k, chi2);
        ++nh;
        snap = snap_of(t);
        rin = (uint32_t)q;
        if (below) miss = 0;
      }
      const bool missed = go && below && h < 0;
      miss += missed ? 1 : 0;
      down = down && !(missed && miss > k.max_miss);
    }
    wave_lds_order();   // the row's column entry
  }
  if (!ok) return 0;
  int32_t* H = d.tk_rowhit + i;     // the column's rows that the selector reads
  for (uint32_t w = rin + sub; w <= rout; w += kL) {
    const uint32_t h = col[w * kPer];
    H[(size_t)w * T] = h == kNoHit ? -1 : (int32_t)(S.a0 + S.first(w) + h);
  }
  if (!writes) return 0;
  store_tracklet<true>(d, i, nh, rin, rout, r0, snap, chi2, zref);
  return steps;
}

template <int kL>
__device__ __forceinline__ void resident_sector(const DevPtrs& d, const KfConst& k, const ResLds& l, unsigned char* lds,
                                                uint32_t sec, uint32_t part, uint32_t parts) {
  constexpr uint32_t kPer = kResThreads / kL;   // tracklets per workgroup
  const uint32_t R = d.R, T = d.tcap, tid = threadIdx.x, srb = sec * R;
  const uint32_t ts = min(d.row_start_off[srb], T), te = min(d.row_start_off[srb + R], T);
  if (ts + part * kPer >= te) return;   // the grid is sized without the number of tracklets
  float2* yz = reinterpret_cast<float2*>(lds);
  f32x4* rows = reinterpret_cast<f32x4*>(lds + l.rows);
  uint16_t* bs = reinterpret_cast<uint16_t*>(lds + l.bs);
  uint16_t* up = l.up ? reinterpret_cast<uint16_t*>(lds + l.up) : nullptr;
  const uint32_t a0 = d.row_off[srb], n_hits = d.row_off[srb + R] - a0;
  // in batches whose loads are all out before the first is written to LDS
  constexpr uint32_t kU = 8;
  for (uint32_t q0 = tid; q0 < n_hits; q0 += kU * kResThreads) {
    float2 h[kU];
    int32_t u[kU];
#pragma unroll
    for (uint32_t j = 0; j < kU; ++j) {
      const uint32_t q = a0 + min(q0 + j * kResThreads, n_hits - 1);
      h[j] = d.syz[q];
      u[j] = up ? d.up1[q] : -1;
    }
#pragma unroll
    for (uint32_t j = 0; j < kU; ++j) {
      const uint32_t q = q0 + j * kResThreads;
      if (q >= n_hits) break;
      yz[q] = h[j];
      if (up) up[q] = (uint16_t)(u[j] >= 0 ? (uint32_t)u[j] - a0 : kNoLink);
    }
  }
  // row table and bin starts, 16 lanes a row; a row's n / K bins and their end fit between first / K + 2 r of this row
  // and of the next
  for (uint32_t r = tid / 16; r < R; r += kResThreads / 16) {
    const RowConst rc = d.rows[r];
    const uint32_t o = d.row_off[srb + r], n = d.row_off[srb + r + 1] - o, lane = tid % 16;
    const uint2 m = d.row_meta[srb + r];
    const uint32_t at = (o - a0) / (uint32_t)d.grid_k + 2 * r, nb = (m.y & 0xFFFFu) * (m.y >> 16);
    if (lane == 0) {
      rows[2 * r] = f32x4{rc.x, rc.half_y, rc.y_lo, rc.inv_wy};
      *reinterpret_cast<u32x4*>(rows + 2 * r + 1) = u32x4{o - a0, n, at, m.y};
    }
    for (uint32_t b0 = lane; b0 <= nb; b0 += 16 * kU) {
      uint32_t v[kU];
#pragma unroll
      for (uint32_t j = 0; j < kU; ++j) v[j] = d.bin_start[m.x + min(b0 + 16 * j, nb)];
#pragma unroll
      for (uint32_t j = 0; j < kU; ++j)
        if (b0 + 16 * j <= nb) bs[at + b0 + 16 * j] = (uint16_t)(v[j] - a0);
    }
  }
  __syncthreads();
  const Resident S{yz, rows, bs, up, a0};
  uint32_t steps = 0;   // of all its tracklets: at most 2^23 of 510 steps over the frame
  for (uint32_t i0 = ts + part * kPer; i0 < te; i0 += parts * kPer)   // workgroup-uniform
    steps += sweep<kL, kPer>(d, k, S, lds + l.col + tid / kL, sec, i0 + tid / kL, te);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) steps += (uint32_t)__shfl_xor((int)steps, off, kWave);
  if (tid % kWave == 0 && steps) atomicAdd(&d.hdr->n_steps, (unsigned long long)steps);
}

// Lanes for a wave on each of the 1024 SIMDs; a quarter goes to workgroups that are not full.
constexpr uint32_t kLanesAlone = 1024u * kWave * 3 / 4;

__global__ void __launch_bounds__(kResThreads) __attribute__((amdgpu_waves_per_eu(3)))
k_tracklets_res(DevPtrs d, KfConst k, ResLds l, uint32_t parts) {
  extern __shared__ __align__(16) unsigned char res_s[];
  // the first part of every sector, then the second and so on: the workgroups without tracklets come last, and the others
  // spread over the XCDs and CUs
  const uint32_t sec = blockIdx.x % d.S, part = blockIdx.x / d.S;
  const uint32_t n = min(d.hdr->n_starts, d.tcap);
  const uint32_t own = min(d.row_start_off[(sec + 1) * d.R], d.tcap) - min(d.row_start_off[sec * d.R], d.tcap);
  // the most lanes that leave every wave alone on its SIMD, and the sector's parts room for its tracklets at once: a second
  // round takes as long as the first (one sector of 13k hits among 399 without hits 1832 us a call at 16 lanes, 745 at two)
  auto lanes = [&](uint32_t kL) { return n * kL <= kLanesAlone && own * kL <= parts * kResThreads; };
  if (lanes(16)) resident_sector<16>(d, k, l, res_s, sec, part, parts);
  else if (lanes(8)) resident_sector<8>(d, k, l, res_s, sec, part, parts);
  else if (lanes(4)) resident_sector<4>(d, k, l, res_s, sec, part, parts);
  else resident_sector<2>(d, k, l, res_s, sec, part, parts);
}

constexpr uint32_t kSparse = 128;   // see launch_tracklets

// Waves of the row-synchronous schedule: ceil(tracklets of sector s / per_wave)
// per sector, prefix-summed (one block).  More than most of them, or (most
// given) more than kSparse hits a tracklet: none, and the tracklets are left to
// the pipeline.
__global__ void __launch_bounds__(1024) k_waves(DevPtrs d, uint32_t per_wave, uint32_t most) {
  __shared__ uint32_t wsum[1024 / kWave];
  const uint32_t S = d.S, R = d.R, T = d.tcap;
  const uint32_t per = (S + blockDim.x - 1) / blockDim.x;
  const uint32_t s0 = min(S, threadIdx.x * per), s1 = min(S, s0 + per);
  uint32_t sum = 0;
  for (uint32_t s = s0; s < s1; ++s) {
    const uint32_t a = min(d.row_start_off[s * R], T), b = min(d.row_start_off[(s + 1) * R], T);
    sum += (b - a + per_wave - 1) / per_wave;
  }
  uint32_t total;
  uint32_t run = block_exclusive_scan<uint32_t>(sum, wsum, &total);
  for (uint32_t s = s0; s < s1; ++s) {
    d.wave_off[s] = run;
    const uint32_t a = min(d.row_start_off[s * R], T), b = min(d.row_start_off[(s + 1) * R], T);
    run += (b - a + per_wave - 1) / per_wave;
  }
  if (threadIdx.x == 0) {
    const bool rows = most == ~0u || (total <= most && (uint64_t)d.hdr->n_starts * kSparse >= d.N);
    d.wave_off[S] = rows ? total : 0;
    d.hdr->pipe_starts = rows ? 0 : d.hdr->n_starts;
  }
}

}  // namespace

// Once per device: the resident kernel takes more dynamic LDS than the default limit.
hipError_t init_tracklets() {
  return hipFuncSetAttribute((const void*)k_tracklets_res, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kResLdsBytes);
}

// Frames of up to kRowSyncHits hits are swept row by row: at 12 hits a tracklet (12 to 24 were seen) the waves of one lane
// per tracklet are all resident, two on a SIMD.  Up to kRowSyncMaybe they may be, and the device decides on the number of
// tracklets: both schedules are launched, and one finds nothing to do (8 launches, 20 to 35 us, or 2 launches, 8 us).  Larger
// frames go through the pipeline.  us of a call, pipeline / row by row: 4 dense sectors, 0.92M hits 1420 / 1230; 40 chunks
// of up to 200k, 1.45M 1380 / 1260; 8 heavy-ion orbits, 2.6M, 2008 waves 1228 / 1083 (1130 here); with more waves than are resident, 8
// dense sectors, 1.86M 1690 / 2090; 9 heavy-ion orbits, 2.9M 1268 / 1530.
// The device also decides where rows are too large to stage and the frame may hold few tracklets for its hits (kSparse):
// the row sweeps pass every row between a wave's first and last, and tracklets of noise are short and far apart, while
// the pipeline's lanes end with their tracklet.  us of K5 on hits without particles, pipeline / row by row (hits a
// tracklet): 6 sectors of 52k 203 / 625 (2000), 30 of 52k 237 / 631 (2100) and, over less drift, 275 / 346 (148), 36 of 61k 273 / 436
// (272), 10 of 106k 284 / 308 (238), 8 of 182k 294 / 306 (71); with particles one sector of 142k 792 / 657 (12), of 969k
// 916 / 795 (65).  Up to kRowSyncHits, frames whose rows are all staged are swept row by row whatever they hold.
constexpr uint32_t kResidentWaves = 2048;
constexpr uint32_t kRowSyncHits = kResidentWaves * kWave * 12;
constexpr uint32_t kRowSyncMaybe = kResidentWaves * kWave * 24;
// Lanes per tracklet, by the frame's hits (us at 8 / 4 / 2 / 1 lanes): 22k 607 / 629 / 700 / 828; 144k 636 / 622 / 672 / 774;
// 324k 1041 / 719 / 714 / 829; 646k 1484 / 1093 / 812 / 907; 1.28M 2470 / 1615 / 968 / 981.  Two lanes only where all rows
// are staged: their searches of a larger row are in global memory, each lane for itself (921k, rows of 1600: 1398 at two
// lanes, 1229 at one).
inline uint32_t row_lanes(uint32_t hits, bool staged) {
  return hits <= (1u << 17) ? 8 : hits <= (1u << 18) ? 4 : staged && hits <= kRowSyncHits ? 2 : 1;
}

void launch_tracklets(const DevPtrs& frame, const KfConst& k, uint32_t max_row_hits, hipStream_t s) {
  if (frame.tcap == 0) return;
  DevPtrs d = frame;
  const bool staged = max_row_hits <= (uint32_t)kStageHits;   // every row: the kernel carries no search in global memory
  const bool maybe = d.k5_mode == 0 && d.N <= kRowSyncMaybe && (d.N > kRowSyncHits || !staged);
  const bool rowsync = maybe || d.k5_mode == 2 || (d.k5_mode == 0 && d.N <= kRowSyncHits);
  d.pipe_n = maybe ? &d.hdr->pipe_starts : &d.hdr->n_starts;
  // the pipeline of such a frame has few waves, or none: without the sort's three launches, which are 7 us where it has none
  if (maybe && d.N <= kRowSyncHits) d.k5_refit_order = 1;
  // Resident sectors while their workgroups run side by side (three on a CU at most, by registers; about a tracklet per 16
  // hits): 60 chunks of up to 13k hits run 7% faster than row by row, 500 of up to 3k as fast, and 400 of up to 13k, one
  // workgroup on a CU at a time, 2.3 times as long.  Every sector has as many parts as the fullest one needs at two lanes
  // a tracklet: no more than 1024 in all, of which most have nothing to do where one sector is full and the others are not
  // (us of a call, row by row / resident: one of 13k hits among 99 of 700 661 / 618, two among 198 of 600 785 / 914).
  const ResLds l = res_lds(std::max(1u, d.max_sector_hits), max_row_hits, d.R, (uint32_t)d.grid_k);
  const uint32_t full = (d.max_sector_hits / 16 + kResPer - 1) / kResPer;
  if (d.k5_mode != 1 && l.total && d.res_blocks <= 256u * std::min(3u, kResLdsBytes / l.total) && (uint64_t)d.S * full <= 1024u) {
    // a sector with more tracklets than its parts hold loops
    const uint32_t parts = std::max((768u + d.S - 1) / d.S, full);
    hipLaunchKernelGGL(k_tracklets_res, dim3(d.S * parts), dim3(kResThreads), l.total, s, d, k, l, parts);
    return;
  }
  if (rowsync) {
    const uint32_t lanes = row_lanes(d.N, staged), per_wave = kThreads / lanes;
    hipLaunchKernelGGL(k_waves, dim3(1), dim3(1024), 0, s, d, per_wave, maybe ? kResidentWaves : ~0u);
    uint32_t blocks = (d.tcap + per_wave - 1) / per_wave + d.S;
    if (blocks > 16384) blocks = 16384;
    auto kern = lanes == 8   ? (staged ? k_tracklets_rs<true, 8> : k_tracklets_rs<false, 8>)
                : lanes == 4 ? (staged ? k_tracklets_rs<true, 4> : k_tracklets_rs<false, 4>)
                : lanes == 2 ? k_tracklets_rs<true, 2>
                             : k_tracklets_rs<false, 1>;
    hipLaunchKernelGGL(kern, dim3(xcd_grid(blocks)), dim3(kThreads), 0, s, d, k);
    if (!maybe) return;
  }
  uint32_t blocks = (d.tcap + kThreads - 1) / kThreads;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(k_seed, dim3(xcd_grid(blocks)), dim3(kThreads), 0, s, d, k);
  hipLaunchKernelGGL(k_order<false>, dim3(kXcds), dim3(kOrderThreads), 0, s, d);
  hipLaunchKernelGGL(k_up, dim3(xcd_grid(blocks)), dim3(kThreads), d.R * sizeof(RowK), s, d, k);
  const uint32_t sort_blocks = std::min<uint32_t>((d.tcap + 255) / 256, 4096);
  if (d.k5_refit_order == 0) {
    launch_scan_u32(d.row_nstart, d.k5_off, d.SR, d.scan_blocks, s);
    hipLaunchKernelGGL(k_sort, dim3(sort_blocks), dim3(256), 0, s, d);
    hipLaunchKernelGGL(k_order<true>, dim3(kXcds), dim3(kOrderThreads), 0, s, d);
  }
  hipLaunchKernelGGL(k_down, dim3(xcd_grid(blocks)), dim3(kThreads), d.R * sizeof(RowK), s, d, k);
  hipLaunchKernelGGL(k_guard, dim3(sort_blocks), dim3(256), 0, s, d);
}

}  // namespace tpc
