// K7-K9: sector merger and merged-chain refit -- steps C8 and C9 of the
// tracker definition, on the C7 tracks of a completed request.
//
// A particle that crosses a sector edge leaves one track segment per sector.
// C8 links a segment a to a segment b of the neighbouring sector on the same
// side when a's state, rotated into b's frame and propagated to b's x_ref,
// lands within fixed windows of b's state, b starting at a larger radius;
// each segment keeps its best successor (smallest position score) and each
// its best predecessor, and a link needs both.  C9 refits every chain of two
// or more segments with one inward Kalman pass over all its clusters.
//
//   k_merge_prep    per sector: first track (tracks are in sector order),
//                   neighbours, tracks sorted by tan(lambda) bin
//   k_merge_match   one wave per segment a: the tracks of the two
//                   neighbouring sectors; tan(lambda) and q/pT are invariants
//                   of the rotation and the propagation, so their windows are
//                   tested first; survivors are propagated in double.  Best
//                   successor kept in the wave; best predecessor by a 64-bit
//                   atomicMin of (score as float bits, a).
//   k_merge_link    mutual best -> next[a]; predecessor flags
//   k_merge_count   per chain head: clusters (scans follow)
//   k_merge_heads   per chain head: record, segment offsets, list of refits
//   k_merge_copy    merged cluster lists
//   k_merge_refit   the refit of the chains of several segments (state and
//                   covariance in double)
#include "device_common.h"

namespace tpc {
namespace {

constexpr int kThreads = 256;
constexpr int kSide = 18;

__device__ __forceinline__ int tri(int i, int j) { return i * (i + 1) / 2 + j; }

struct MTrack {
  uint32_t sector;
  int32_t phys;
  double x, p[5];
  double r_in;
};

__device__ __forceinline__ MTrack load_track(const DevPtrs& d, const MergeArgs& m, uint32_t t) {
  MTrack a;
  a.sector = d.out_sector[t];
  a.phys = m.phys[a.sector];
  a.x = d.out_xref[t];
#pragma unroll
  for (int q = 0; q < 5; ++q) a.p[q] = d.out_param[(size_t)t * 5 + q];
  a.r_in = sqrt(a.x * a.x + a.p[0] * a.p[0]);
  return a;
}

// Helix transport of the state only (the map of C5), in double.
__device__ __forceinline__ double asin_over_d(double u) {
  const double u2 = u * u;
  if (fabs(u) < 1e-2) return 1.0 + u2 * (1.0 / 6.0 + u2 * (3.0 / 40.0 + u2 * (5.0 / 112.0 + u2 * (35.0 / 1152.0))));
  return asin(u) / u;
}
__device__ __forceinline__ double asin_over_prime_d(double u) {
  const double u2 = u * u;
  if (fabs(u) < 1e-2) return u * (1.0 / 3.0 + u2 * (3.0 / 10.0 + u2 * (15.0 / 56.0 + u2 * (35.0 / 144.0))));
  return (u / sqrt(1.0 - u2) - asin(u)) / u2;
}

// x1 -> x2 with the exact Jacobian F (sparse entries A..Fk) when cov is given.
__device__ bool prop_d(double* p, double x1, double x2, double bk, double smax, double* c) {
  const double dx = x2 - x1;
  const double s1 = p[2], tl = p[3], kap = bk * p[4];
  if (!(fabs(s1) < smax)) return false;
  const double s2 = s1 + kap * dx;
  if (!(fabs(s2) < smax)) return false;
  const double c1 = sqrt((1.0 - s1) * (1.0 + s1)), c2 = sqrt((1.0 - s2) * (1.0 + s2));
  const double dy = dx * ((s1 + s2) / (c1 + c2));
  const double L = sqrt(dx * dx + dy * dy);
  const double u = 0.5 * kap * L;
  if (!(fabs(u) < 1.0)) return false;
  const double sgn = dx >= 0.0 ? 1.0 : -1.0;
  const double S = sgn * L * asin_over_d(u);
  if (c) {
    const double D = (1.0 + c1 * c2 + s1 * s2) / ((c1 + c2) * (c1 + c2));
    const double A = dx * D * (1.0 / c1 + 1.0 / c2);
    const double B = dx * (D / c2) * bk * dx;
    const double dS_dL = sgn / sqrt(1.0 - u * u);
    const double dS_dkap = sgn * 0.5 * L * L * asin_over_prime_d(u);
    const double dL_ddy = L > 0.0 ? dy / L : 0.0;
    const double Cc = tl * dS_dL * dL_ddy * A;
    const double Dd = S;
    const double E = tl * (dS_dL * dL_ddy * B + dS_dkap * bk);
    const double Fk = bk * dx;
    double M[5][5], G[3][5];
    for (int i = 0; i < 5; ++i)
      for (int j = 0; j < 5; ++j) M[i][j] = i >= j ? c[tri(i, j)] : c[tri(j, i)];
    for (int j = 0; j < 5; ++j) {
      G[0][j] = M[0][j] + A * M[2][j] + B * M[4][j];
      G[1][j] = M[1][j] + Cc * M[2][j] + Dd * M[3][j] + E * M[4][j];
      G[2][j] = M[2][j] + Fk * M[4][j];
    }
    // C' = G F^T on the lower triangle (rows 3, 4 of F are those of the identity)
    for (int i = 0; i < 5; ++i) {
      const double g0 = i < 3 ? G[i][0] : M[i][0], g1 = i < 3 ? G[i][1] : M[i][1], g2 = i < 3 ? G[i][2] : M[i][2];
      const double g3 = i < 3 ? G[i][3] : M[i][3], g4 = i < 3 ? G[i][4] : M[i][4];
      const double rr[5] = {g0 + A * g2 + B * g4, g1 + Cc * g2 + Dd * g3 + E * g4, g2 + Fk * g4, g3, g4};
      for (int j = 0; j <= i; ++j) c[tri(i, j)] = rr[j];
    }
  }
  p[0] += dy;
  p[1] += tl * S;
  p[2] = s2;
  return true;
}

// Rotation into the frame turned by the angle with cosine cd and sine sd, at
// the same point in space; first-order covariance onto the new plane x' = const.
__device__ bool rotate_d(double& x, double* p, double cd, double sd, double bk, double* c) {
  const double s = p[2], cs = sqrt((1.0 - s) * (1.0 + s));
  const double s2 = s * cd - cs * sd, c2 = cs * cd + s * sd;
  if (!(c2 > 0.0)) return false;
  const double x2 = x * cd + p[0] * sd;
  const double y2 = -x * sd + p[0] * cd;
  if (c) {
    // J = I except J00 = cs/c2, J10 = -tanl sd/c2, J20 = -bk qpt sd, J22 = c2/cs
    const double j00 = cs / c2, j10 = -p[3] * sd / c2, j20 = -bk * p[4] * sd, j22 = c2 / cs;
    double M[5][5];
    for (int i = 0; i < 5; ++i)
      for (int j = 0; j < 5; ++j) M[i][j] = i >= j ? c[tri(i, j)] : c[tri(j, i)];
    double G[5][5];   // G = J M
    for (int j = 0; j < 5; ++j) {
      G[0][j] = j00 * M[0][j];
      G[1][j] = j10 * M[0][j] + M[1][j];
      G[2][j] = j20 * M[0][j] + j22 * M[2][j];
      G[3][j] = M[3][j];
      G[4][j] = M[4][j];
    }
    for (int i = 0; i < 5; ++i) {   // C' = G J^T
      const double rr[5] = {G[i][0] * j00, G[i][0] * j10 + G[i][1], G[i][0] * j20 + G[i][2] * j22, G[i][3], G[i][4]};
      for (int j = 0; j <= i; ++j) c[tri(i, j)] = rr[j];
    }
  }
  x = x2;
  p[0] = y2;
  p[2] = s2;
  return true;
}

// Kalman update of (y, z), Joseph form, in double.
__device__ void update_d(double* p, double* c, double ym, double zm, double vy, double vz, double& chi2) {
  const double r0 = ym - p[0], r1 = zm - p[1];
  const double S00 = c[0] + vy, S01 = c[1], S11 = c[2] + vz;
  const double det = S00 * S11 - S01 * S01;
  const double I00 = S11 / det, I01 = -S01 / det, I11 = S00 / det;
  double c0[5], c1[5], K0[5], K1[5];
  for (int i = 0; i < 5; ++i) {
    c0[i] = c[tri(i, 0)];
    c1[i] = i >= 1 ? c[tri(i, 1)] : c[1];
  }
  for (int i = 0; i < 5; ++i) {
    K0[i] = c0[i] * I00 + c1[i] * I01;
    K1[i] = c0[i] * I01 + c1[i] * I11;
    p[i] += K0[i] * r0 + K1[i] * r1;
  }
  double P[5][5];
  for (int i = 0; i < 5; ++i)
    for (int j = 0; j < 5; ++j) P[i][j] = (i >= j ? c[tri(i, j)] : c[tri(j, i)]) - K0[i] * c0[j] - K1[i] * c1[j];
  for (int i = 0; i < 5; ++i)
    for (int j = 0; j <= i; ++j)
      c[tri(i, j)] = P[i][j] + (K0[i] * vy - P[i][0]) * K0[j] + (K1[i] * vz - P[i][1]) * K1[j];
  chi2 += r0 * (I00 * r0 + I01 * r1) + r1 * (I01 * r0 + I11 * r1);
}

__device__ __forceinline__ uint32_t n_tracks(const DevPtrs& d) { return min(d.hdr->n_tracks, d.max_tracks); }

// Neighbour of physical sector ph one step (+1 / -1) along its side's ring.
__device__ __forceinline__ int32_t neighbour(int32_t ph, int step) {
  const int32_t side = ph / kSide, i = ph % kSide;
  return side * kSide + (i + step + kSide) % kSide;
}

// Tracks of a sector in ascending tan(lambda) bin (any order inside a bin), for the matching: (tan(lambda),
// q/pT, z, track) per slot, slot range = the sector's track range.
constexpr int kPrepThreads = 1024;
constexpr int kTanBins = 256;
// Bin of a tan(lambda): monotone, so the tracks within a window lie between the bins of its ends.
__device__ __forceinline__ int tan_bin(double tl) {
  const double u = (tl + 2.0) * 64.0;
  return u > 0.0 ? (u < kTanBins - 1 ? (int)u : kTanBins - 1) : 0;
}

// One workgroup per sector: its track range, its neighbours in the frame, the
// cleared per-track words and the sector's slots of the sorted list (a
// counting sort with the bins in LDS).
__global__ void __launch_bounds__(kPrepThreads) k_merge_prep(DevPtrs d, MergeArgs m) {
  __shared__ uint32_t hist[kTanBins + 1], wsum[kPrepThreads / kWave], range[2];
  __shared__ int32_t nb[2];
  const uint32_t s = blockIdx.x, tid = threadIdx.x;
  for (uint32_t b = tid; b < (uint32_t)kTanBins; b += kPrepThreads) hist[b] = 0u;
  if (tid < 2) {
    // first track of sector s and of sector s + 1: lower bounds in the sorted track sectors
    uint32_t lo = 0, hi = n_tracks(d);
    while (lo < hi) {
      const uint32_t mid = (lo + hi) / 2;
      if (d.out_sector[mid] < s + tid) lo = mid + 1; else hi = mid;
    }
    range[tid] = lo;
    nb[tid] = INT32_MAX;
  }
  __syncthreads();
  const uint32_t t0 = range[0], t1 = range[1];
  const int32_t ph = m.phys[s];
  if (ph >= 0) {
    // the frame's first sector that holds each physical neighbour
    const int32_t dn = neighbour(ph, -1), up = neighbour(ph, 1);
    for (uint32_t q = tid; q < d.S; q += kPrepThreads) {
      const int32_t v = m.phys[q];
      if (v == dn) atomicMin(&nb[0], (int32_t)q);
      if (v == up) atomicMin(&nb[1], (int32_t)q);
    }
  }
  for (uint32_t t = t0 + tid; t < t1; t += kPrepThreads) {
    m.pred_key[t] = ~0ull;
    m.has_pred[t] = 0u;
    if (ph >= 0) atomicAdd(&hist[tan_bin(d.out_param[(size_t)t * 5 + 3])], 1u);
  }
  __syncthreads();
  if (tid < 2) m.nbr[2 * s + tid] = nb[tid] == INT32_MAX ? -1 : nb[tid];
  if (tid == 0) {
    m.sec_first[s] = t0;
    if (s + 1 == d.S) m.sec_first[d.S] = t1;
    if (s == 0) d.hdr->merge_refits = 0u;
  }
  if (ph < 0) return;
  block_scan_array(hist, kTanBins, wsum);
  for (uint32_t t = t0 + tid; t < t1; t += kPrepThreads) {
    const float* p = d.out_param + (size_t)t * 5;
    const uint32_t at = t0 + atomicAdd(&hist[tan_bin(p[3])], 1u);
    m.sorted[at] = make_float4(p[3], p[4], p[1], __uint_as_float(t));
  }
}

// Path length S(x) of track state (s1, kap) over dx, with sin phi held at +-smax beyond it: monotone in
// dx, so its values at the innermost and outermost row bound the path to any row the track reaches.
__device__ __forceinline__ double path_bound(double s1, double kap, double dx, double smax) {
  const double s2 = fmin(smax, fmax(-smax, s1 + kap * dx));
  if (s2 != s1 + kap * dx) dx = (s2 - s1) / kap;   // clamped, so kap != 0
  const double c1 = sqrt((1.0 - s1) * (1.0 + s1)), c2 = sqrt((1.0 - s2) * (1.0 + s2));
  const double dy = dx * ((s1 + s2) / (c1 + c2));
  const double L = sqrt(dx * dx + dy * dy), u = fmin(1.0, fabs(0.5 * kap * L));
  return (dx >= 0.0 ? L : -L) * asin_over_d(u);
}

// One wave per track a: its lanes test the tracks of the two neighbouring
// sectors whose tan(lambda) bin can match.  Cheap float32 windows with slack
// (tan(lambda), q/pT, and the z that a's path can reach) leave a few
// candidates, which are tested exactly in double.  Bound: instruction issue.
// One thread per track, walking every track of both sectors, made nearly
// every one of a wave's iterations run the double part for a lane or two:
// 787 us for 31k tracks and 3485 us for 126k, against 87 us and 468 us here.
constexpr int kMatchWaves = 4;
__global__ void __launch_bounds__(kMatchWaves * kWave) k_merge_match(DevPtrs d, MergeArgs m) {
  const uint32_t nt = n_tracks(d), lane = threadIdx.x % kWave;
  const uint32_t a = blockIdx.x * kMatchWaves + threadIdx.x / kWave;
  if (a >= nt) return;
  const MTrack ta = load_track(d, m, a);
  int32_t best = -1;
  double best_s = 0.0;
  const float tla = (float)ta.p[3], qa = (float)ta.p[4];
  const float wt = (float)m.dtanl * 1.001f + 1e-6f, wq = (float)m.dqpt * 1.001f + 1e-5f;
  for (int side = 0; ta.phys >= 0 && side < 2; ++side) {
    const int32_t nb = m.nbr[2 * ta.sector + side];
    if (nb < 0) continue;
    // the rotation into the neighbour's frame is the same for every b
    const int step = side == 0 ? -1 : 1;
    double x = ta.x, q[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) q[i] = ta.p[i];
    if (!rotate_d(x, q, m.cos20, step * m.sin20, m.bk, nullptr)) continue;
    if (!(fabs(q[2]) < m.s_max)) continue;   // no propagation starts there
    // z within reach (lane 0: to the innermost row, lane 1: to the outermost)
    const double end = d.rows[lane & 1u ? d.R - 1 : 0].x;
    const double ze = q[1] + q[3] * path_bound(q[2], m.bk * q[4], end - x, m.s_max);
    const double z0 = __shfl(ze, 0, kWave), z1 = __shfl(ze, 1, kWave);
    const double slack = m.dz * 1.001 + 0.01 + 1e-4 * fabs(z1 - z0) + 1e-6 * fabs(q[1]);
    const float zlo = (float)(fmin(z0, z1) - slack), zhi = (float)(fmax(z0, z1) + slack);
    const uint32_t b0 = m.sec_first[nb], b1 = m.sec_first[nb + 1];
    // first slot whose bin reaches the window, 64 probes at a time
    const int klo = tan_bin(ta.p[3] - m.dtanl), khi = tan_bin(ta.p[3] + m.dtanl);
    uint32_t lo = b0, hi = b1;
    while (hi - lo > (uint32_t)kWave) {
      const uint32_t st = (hi - lo + kWave - 1) / kWave, p = lo + lane * st;
      const uint32_t below = (uint32_t)__popcll(__ballot(p < hi && tan_bin(m.sorted[p < hi ? p : lo].x) < klo));
      hi = min(hi, lo + below * st);
      if (below) lo += (below - 1) * st + 1;
    }
    {
      const uint32_t p = lo + lane;
      lo += (uint32_t)__popcll(__ballot(p < hi && tan_bin(m.sorted[p < hi ? p : b0].x) < klo));
    }
    for (uint32_t base = lo; base < b1; base += kWave) {
      const bool in = base + lane < b1;
      const float4 v = in ? m.sorted[base + lane] : make_float4(INFINITY, 0.0f, 0.0f, 0.0f);
      if (tan_bin(__shfl(v.x, 0, kWave)) > khi) break;   // bins ascend
      if (!(in && fabsf(tla - v.x) <= wt && fabsf(qa - v.y) <= wq && v.z >= zlo && v.z <= zhi)) continue;
      const uint32_t b = __float_as_uint(v.w);
      const MTrack tb = load_track(d, m, b);
      if (!(fabs(ta.p[3] - tb.p[3]) <= m.dtanl && fabs(ta.p[4] - tb.p[4]) <= m.dqpt)) continue;
      if (!(tb.r_in > ta.r_in)) continue;
      double qb[5];
#pragma unroll
      for (int i = 0; i < 5; ++i) qb[i] = q[i];
      if (!prop_d(qb, x, tb.x, m.bk, m.s_max, nullptr)) continue;
      const double dy = qb[0] - tb.p[0], dz = qb[1] - tb.p[1];
      if (!(fabs(dy) <= m.dy && fabs(dz) <= m.dz && fabs(qb[2] - tb.p[2]) <= m.dsinphi)) continue;
      const double cyy = d.out_cov[(size_t)b * 15 + 0], czz = d.out_cov[(size_t)b * 15 + 2];
      const double sc = dy * dy / (cyy + m.vy) + dz * dz / (czz + m.vz);
      if (best < 0 || sc < best_s || (sc == best_s && (int32_t)b < best)) {
        best = (int32_t)b;
        best_s = sc;
      }
      const unsigned long long key = ((unsigned long long)__float_as_uint((float)sc) << 32) | a;
      atomicMin(&m.pred_key[b], key);
    }
  }
  if (__any(best >= 0)) {   // the lanes' best: smallest score, ties to the smaller index
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      const int32_t ob = __shfl_xor(best, off, kWave);
      const double os = __shfl_xor(best_s, off, kWave);
      if (ob >= 0 && (best < 0 || os < best_s || (os == best_s && ob < best))) {
        best = ob;
        best_s = os;
      }
    }
  }
  if (lane == 0) m.succ[a] = best;
}

__global__ void __launch_bounds__(kThreads) k_merge_link(DevPtrs d, MergeArgs m) {
  const uint32_t nt = n_tracks(d);
  const uint32_t a = blockIdx.x * kThreads + threadIdx.x;
  if (a >= nt) return;
  const int32_t b = m.succ[a];
  const bool link = b >= 0 && (uint32_t)(m.pred_key[b] & 0xFFFFFFFFull) == a;
  m.next[a] = link ? b : -1;
  if (link) m.has_pred[b] = 1u;
}

// Per track: 1 if it heads a chain (for the scan of chain indices), and at
// each head the chain's cluster count (for the scan of cluster offsets).
__global__ void __launch_bounds__(kThreads) k_merge_count(DevPtrs d, MergeArgs m) {
  const uint32_t nt = n_tracks(d);
  const uint32_t a = blockIdx.x * kThreads + threadIdx.x;
  if (a >= nt) return;
  const bool head = m.has_pred[a] == 0u;
  m.head_flag[a] = head ? 1u : 0u;
  uint32_t n = 0;
  if (head)
    for (int32_t t = (int32_t)a; t >= 0; t = m.next[t]) n += d.out_first[t + 1] - d.out_first[t];
  m.chain_clusters[a] = n;
}

// Row of input cluster id inside sector s (upper bound in the sector's row offsets).
__device__ __forceinline__ uint32_t row_of(const DevPtrs& d, uint32_t s, uint32_t id) {
  uint32_t lo = 0, hi = d.R;   // first row r with row_off[s*R + r + 1] > id
  while (lo < hi) {
    const uint32_t mid = (lo + hi) / 2;
    if (d.row_off[s * d.R + mid + 1] <= id) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// Per chain head: the chain's record, the cluster offset of each of its
// segments, and its place in the list of chains to refit if it has several.
__global__ void __launch_bounds__(kThreads) k_merge_heads(DevPtrs d, MergeArgs m) {
  const uint32_t nt = n_tracks(d);
  const uint32_t a = blockIdx.x * kThreads + threadIdx.x;
  const bool head = a < nt && m.head_flag[a] != 0u;
  int32_t nseg = 0;
  if (head) {
    const uint32_t c = m.head_scan[a];   // chain index
    uint32_t o = m.cl_scan[a];
    m.heads[c] = a;
    m.first[c] = o;
    for (int32_t t = (int32_t)a; t >= 0; t = m.next[t]) {
      m.seg_off[t] = o;
      o += d.out_first[t + 1] - d.out_first[t];
      m.head_of[t] = a;
      ++nseg;
    }
    if (c + 1 == m.head_scan[nt]) m.first[c + 1] = o;
    m.nseg[c] = nseg;
    m.chi2[c] = d.out_chi2[a];
    m.ndf[c] = 2 * (int32_t)(o - m.cl_scan[a]) - 5;
#pragma unroll
    for (int q = 0; q < 5; ++q) m.param[(size_t)c * 5 + q] = d.out_param[(size_t)a * 5 + q];
#pragma unroll
    for (int q = 0; q < 15; ++q) m.cov[(size_t)c * 15 + q] = d.out_cov[(size_t)a * 15 + q];
  }
  // one atomic per wave; the order of the refits does not matter
  const unsigned long long multi = __ballot(nseg > 1);
  const uint32_t lane = threadIdx.x % kWave;
  uint32_t base = 0;
  if (lane == 0 && multi) base = atomicAdd(&d.hdr->merge_refits, (uint32_t)__popcll(multi));
  base = (uint32_t)__shfl((int)base, 0, kWave);
  if (nseg > 1) m.refit[base + (uint32_t)__popcll(multi & ((1ull << lane) - 1ull))] = a;
}

// Per track, one wave: its clusters to their place in the chain's list and,
// where the chain is refitted, each cluster's row.
__global__ void __launch_bounds__(kThreads) k_merge_copy(DevPtrs d, MergeArgs m) {
  const uint32_t nt = n_tracks(d), lane = threadIdx.x % kWave;
  const uint32_t t = blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave;
  if (t >= nt) return;
  const uint32_t j0 = d.out_first[t], n = d.out_first[t + 1] - j0, o = m.seg_off[t], s = d.out_sector[t];
  const bool rows = m.next[t] >= 0 || m.has_pred[t] != 0u;
  for (uint32_t j = lane; j < n; j += kWave) {
    const uint32_t id = d.out_clusters[j0 + j];
    m.clusters[o + j] = id;
    if (rows) m.cl_row[o + j] = (uint8_t)row_of(d, s, id);
  }
}

// Per chain of several segments, one lane: the inward pass over the chain's
// clusters, from the outermost one of the last segment, in double.  Bound:
// the latency of the dependent steps (few chains, no more than a wave or two
// per SIMD), so the next clusters' ids and coordinates are loaded ahead and
// their rows come from k_merge_copy (270 us for 31k tracks, 427 us for 126k,
// and 22 and 73 us in k_merge_copy); with the rows searched and every load on
// the chain, in the thread that also copied the clusters, it was 609 and
// 829 us.
__global__ void __launch_bounds__(kWave) k_merge_refit(DevPtrs d, MergeArgs m) {
  const uint32_t k = blockIdx.x * kWave + threadIdx.x;
  if (k >= d.hdr->merge_refits) return;
  const uint32_t a = m.refit[k], c = m.head_scan[a];
  const int32_t o0 = (int32_t)m.first[c];
  int32_t seg = (int32_t)a;
  while (m.next[seg] >= 0) seg = m.next[seg];
  int32_t o = (int32_t)(m.seg_off[seg] + (d.out_first[seg + 1] - d.out_first[seg])) - 1;
  uint32_t sec = d.out_sector[seg];
  int32_t seg0 = (int32_t)m.seg_off[seg];   // first merged cluster of the current segment
  // cluster o is in hand; o - 1's coordinates and o - 2's id are on their way
  auto id_at = [&](int32_t q) { return m.clusters[q > o0 ? q : o0]; };
  uint32_t row = m.cl_row[o], row1 = m.cl_row[o > o0 ? o - 1 : o0];
  const uint32_t id0 = id_at(o), id1 = id_at(o - 1);
  uint32_t id2 = id_at(o - 2);
  const float y0 = d.y[id0], z0 = d.z[id0];
  float y1 = d.y[id1], z1 = d.z[id1];
  double p[5], cv[15];
  double x = d.out_xref[seg];
#pragma unroll
  for (int q = 0; q < 5; ++q) p[q] = d.out_param[(size_t)seg * 5 + q];
  double ch = 0.0;
  bool ok = prop_d(p, x, d.rows[row].x, m.bk, m.s_max, nullptr);
  if (ok) {
    x = d.rows[row].x;
    p[0] = y0;
    p[1] = z0;
#pragma unroll
    for (int q = 0; q < 15; ++q) cv[q] = 0.0;
    cv[0] = m.vy;
    cv[2] = m.vz;
    cv[5] = m.c0_sinphi;
    cv[9] = m.c0_tanl;
    cv[14] = m.c0_qpt;
    while (o > o0) {
      if (o == seg0) {
        // previous segment in the chain: the one whose next is seg
        int32_t pv = (int32_t)a;
        while (m.next[pv] != seg) pv = m.next[pv];
        const int step = (m.phys[d.out_sector[pv]] % kSide - m.phys[sec] % kSide + kSide) % kSide == 1 ? 1 : -1;
        if (!rotate_d(x, p, m.cos20, step * m.sin20, m.bk, cv)) { ok = false; break; }
        seg = pv;
        sec = d.out_sector[seg];
        seg0 = (int32_t)m.seg_off[seg];
      }
      --o;
      row = row1;
      const float ym = y1, zm = z1;
      y1 = d.y[id2];
      z1 = d.z[id2];
      id2 = id_at(o - 2);
      row1 = m.cl_row[o > o0 ? o - 1 : o0];
      const double xr = d.rows[row].x;
      if (!prop_d(p, x, xr, m.bk, m.s_max, cv)) { ok = false; break; }
      x = xr;
      update_d(p, cv, ym, zm, m.vy, m.vz, ch);
    }
  }
  if (!ok) {
    m.ndf[c] = -1;   // the chain keeps its first segment's result
    return;
  }
#pragma unroll
  for (int q = 0; q < 5; ++q) m.param[(size_t)c * 5 + q] = (float)p[q];
#pragma unroll
  for (int q = 0; q < 15; ++q) m.cov[(size_t)c * 15 + q] = (float)cv[q];
  m.chi2[c] = (float)ch;
}

}  // namespace

void launch_merge(const DevPtrs& d, const MergeArgs& m, uint32_t nt, hipStream_t s) {
  if (nt == 0) return;
  hipLaunchKernelGGL(k_merge_prep, dim3(d.S), dim3(kPrepThreads), 0, s, d, m);
  const uint32_t g = (nt + kThreads - 1) / kThreads;
  const uint32_t waves = kThreads / kWave;
  hipLaunchKernelGGL(k_merge_match, dim3((nt + kMatchWaves - 1) / kMatchWaves), dim3(kMatchWaves * kWave), 0, s, d, m);
  hipLaunchKernelGGL(k_merge_link, dim3(g), dim3(kThreads), 0, s, d, m);
  hipLaunchKernelGGL(k_merge_count, dim3(g), dim3(kThreads), 0, s, d, m);
  launch_scan_u32(m.head_flag, m.head_scan, nt, d.scan_blocks, s);
  launch_scan_u32(m.chain_clusters, m.cl_scan, nt, d.scan_blocks, s);
  hipLaunchKernelGGL(k_merge_heads, dim3(g), dim3(kThreads), 0, s, d, m);
  hipLaunchKernelGGL(k_merge_copy, dim3((nt + waves - 1) / waves), dim3(kThreads), 0, s, d, m);
  // a chain to refit has at least two tracks
  hipLaunchKernelGGL(k_merge_refit, dim3((nt / 2 + kWave - 1) / kWave + 1), dim3(kWave), 0, s, d, m);
}

}  // namespace tpc
