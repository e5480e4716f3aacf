// C10/C11: track-model compression of the clusters of a completed request,
// and its decoding.
//
// Encoding writes, per track, the model (x_ref and six coefficients of the
// second-order expansion of the fitted helix around x_ref) and, per track
// cluster, its row and the quantised residuals (k_y, k_z) to that model; the
// clusters on no track are listed raw, in input order.  Decoding rebuilds the
// clusters from the stream.  Every float32 step is written out in the order the
// definition gives, with contraction off, so the codes are the same bits as
// any other evaluation of the definition; the coefficients are computed in
// double (IEEE division and square root) and rounded once.
//
// Encoding runs in two launches around a scan of the row counts:
//   k_codec_models  the models, one lane per track; and per (sector, row) the
//                   clusters on no track as a bit per input cluster.  A
//                   cluster is on a track when the tracklet that owns it (C6)
//                   was accepted, so no pass over the tracks has to mark them.
//   k_codec_stream  the codes of kChunk consecutive track clusters per
//                   workgroup, and per (sector, row) the raw list.
// A workgroup's clusters belong to a few dozen tracks, nearly always of one
// sector: the track boundaries and the sector's row offsets are staged in LDS,
// and both searches of a cluster (its track, its row) run there.  Decoding has
// the same shape, with the models staged too.  Bound: HBM traffic (25 B per
// track cluster encoding, 14 B decoding) and the gather of the input
// coordinates by cluster id, whose lines stay in an XCD's L2 because each XCD
// takes one contiguous eighth of the track clusters (tracks are in sector
// order).
#include <algorithm>

#include "device_common.h"

namespace tpc {
namespace {

constexpr int kThreads = 256;
constexpr int16_t kEscape = -32768;
constexpr int kPer = 8;                           // track clusters per lane
constexpr uint32_t kChunk = kPer * kThreads;      // and per workgroup
constexpr uint32_t kTrackCap = 512;               // track boundaries staged per workgroup

// Last index k with a[k] <= v in the ascending array a[0..n] (a[0] <= v).
__device__ __forceinline__ uint32_t last_le(const uint32_t* a, uint32_t n, uint32_t v) {
  uint32_t lo = 0, hi = n;   // a[lo] <= v < a[hi] (a[n] treated as +inf)
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) / 2;
    if (a[mid] <= v) lo = mid;
    else hi = mid;
  }
  return lo;
}

// The same by a whole wave, 64 probes at a time.
__device__ __forceinline__ uint32_t wave_last_le(const uint32_t* a, uint32_t n, uint32_t v) {
  uint32_t lo = 0, hi = n;
  while (hi - lo > 1) {
    const uint32_t st = (hi - lo + kWave - 1) / kWave, p = lo + (threadIdx.x % kWave + 1) * st;
    const uint32_t le = (uint32_t)__popcll(__ballot(p < hi && a[p < hi ? p : lo] <= v));
    lo += le * st;
    hi = min(hi, lo + st);
  }
  return lo;
}

// The tracks of a workgroup's clusters [j0, j1): the first of them and the
// starts of the others, staged in LDS when there are at most kTrackCap.
struct TrackWindow {
  uint32_t t0, n;          // tracks t0 .. t0 + n
  const uint32_t* starts;  // [n] first cluster of track t0 + 1 + k
  bool staged;
};
__device__ __forceinline__ TrackWindow track_window(const uint32_t* first, uint32_t n_tracks, uint32_t j0, uint32_t j1,
                                                    uint32_t* lds, uint32_t* ends) {
  const uint32_t w = threadIdx.x / kWave;
  if (w < 2) {
    const uint32_t t = wave_last_le(first, n_tracks, w == 0 ? j0 : j1 - 1);
    if (threadIdx.x % kWave == 0) ends[w] = t;
  }
  __syncthreads();
  TrackWindow tw;
  tw.t0 = ends[0];
  tw.n = ends[1] >= ends[0] ? ends[1] - ends[0] : 0u;   // first[] ascends, so ends[1] >= ends[0]
  tw.starts = lds;
  tw.staged = tw.n <= kTrackCap;
  if (tw.staged)
    for (uint32_t k = threadIdx.x; k < tw.n; k += kThreads) lds[k] = first[tw.t0 + 1 + k];
  return tw;
}
// Track of cluster j of the window, as an offset from t0 (staged windows).
__device__ __forceinline__ uint32_t track_in(const TrackWindow& tw, uint32_t j) {
  uint32_t lo = 0, hi = tw.n;   // number of starts <= j
  while (lo < hi) {
    const uint32_t mid = (lo + hi) / 2;
    if (tw.starts[mid] <= j) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// c0 + u * (c1 + u * c2), u = xr - x_ref, float32, no fused multiply-add.
__device__ __forceinline__ float predict(float xr, float x_ref, float c0, float c1, float c2) {
#pragma clang fp contract(off)
  const float u = xr - x_ref;
  const float inner = c1 + u * c2;
  const float outer = u * inner;
  return c0 + outer;
}

// The model of track t.
__device__ __forceinline__ void write_model(const CodecArgs& a, uint32_t t) {
  const float* p = a.param + 5 * (size_t)t;
  float* c = a.coef + 6 * (size_t)t;
  const double s = p[2], T = p[3], qpt = p[4];
  if (fabs(s) < 1.0) {
    const double kappa = a.bk * qpt;
    const double cc = sqrt(1.0 - s * s);
    const double ic = 1.0 / cc;
    const double ic3 = ic * ic * ic;
    c[0] = p[0];
    c[1] = (float)(s * ic);
    c[2] = (float)(0.5 * kappa * ic3);
    c[3] = p[1];
    c[4] = (float)(T * ic);
    c[5] = (float)(((0.5 * T) * s) * kappa * ic3);
  } else {
    for (int q = 0; q < 6; ++q) c[q] = 0.0f;   // no model: every cluster of the track is escaped
  }
  a.x_ref[t] = a.xref_in[t];
  a.first[t] = a.first_in[t];
  if (t + 1 == a.n_tracks) a.first[t + 1] = a.first_in[t + 1];
}

// Workgroups [0, SR): the clusters of row sr on no track, a bit per input
// cluster, and their number.  The others: the models.
__global__ void __launch_bounds__(kThreads) k_codec_models(CodecArgs a) {
  __shared__ uint32_t bits[65536 / 32], wsum[kThreads / kWave];
  if (blockIdx.x >= a.SR) {
    const uint32_t t0 = (blockIdx.x - a.SR) * kThreads + threadIdx.x;
    if (t0 == 0) {
      *a.n_escaped = 0;
      if (a.n_tracks == 0) a.first[0] = 0;
    }
    if (t0 < a.n_tracks) write_model(a, t0);
    return;
  }
  const uint32_t sr = blockIdx.x;
  const uint32_t b = a.row_off[sr], n = a.row_off[sr + 1] - b, words = (n + 31) / 32;
  if (n <= (uint32_t)kWave) {   // by its first wave, without barriers (see emit_row)
    const uint32_t p = threadIdx.x;
    if (p >= (uint32_t)kWave) return;
    const uint32_t key = p < n ? a.W[b + p] : 0u, id = p < n ? a.sid[b + p] - b : 0u;
    const bool un = p < n && !(key && (a.tk_pack[0x7FFFFFu - (key & 0x7FFFFFu)] & 1ull));
    if (p < 2) bits[p] = 0u;
    wave_lds_order();
    if (un) atomicOr(&bits[id / 32], 1u << (id % 32));
    wave_lds_order();
    if (p < (n + 7) / 8) a.un_bits[b + p] = (uint8_t)(bits[p / 4] >> (8 * (p % 4)));
    const uint32_t total = (uint32_t)__popcll(__ballot(un));
    if (p == 0) a.row_cnt[sr] = total;
    return;
  }
  for (uint32_t w = threadIdx.x; w < words; w += kThreads) bits[w] = 0u;
  __syncthreads();
  constexpr int kU = 4;
  for (uint32_t p0 = threadIdx.x; p0 < n; p0 += kU * kThreads) {
    uint32_t key[kU], id[kU];
    unsigned long long acc[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const uint32_t p = p0 + u * kThreads;
      key[u] = p < n ? a.W[b + p] : 0u;
      id[u] = p < n ? a.sid[b + p] - b : 0u;
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) acc[u] = key[u] ? a.tk_pack[0x7FFFFFu - (key[u] & 0x7FFFFFu)] : 0ull;
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (p0 + u * kThreads < n && !(acc[u] & 1ull)) atomicOr(&bits[id[u] / 32], 1u << (id[u] % 32));
  }
  __syncthreads();
  uint32_t c = 0;
  for (uint32_t w = threadIdx.x; w < words; w += kThreads) c += (uint32_t)__popc(bits[w]);
  for (uint32_t w = threadIdx.x; w < (n + 7) / 8; w += kThreads)
    a.un_bits[b + w] = (uint8_t)(bits[w / 4] >> (8 * (w % 4)));
  uint32_t total;
  (void)block_exclusive_scan<uint32_t>(c, wsum, &total);
  if (threadIdx.x == 0) a.row_cnt[sr] = total;
}

// The raw list of row sr, in input order.  Rows of up to 64 clusters are listed by one wave (and marked by one, above): a
// // request of many small sectors is bound by its rows, of which a CU then holds two to three times as many (2000 sectors of 700
// clusters, 304k rows: the call 660 -> 365 us, 540 when the tracks' clusters were marked in a word per cluster).
__device__ __forceinline__ void emit_row(const CodecArgs& a, uint32_t sr, uint32_t* wsum) {
  const uint32_t b = a.row_off[sr], n = a.row_off[sr + 1] - b, bytes = (n + 7) / 8;
  uint32_t base = a.row_pos[sr];
  if (n <= (uint32_t)kWave) {
    const uint32_t p = threadIdx.x;
    if (p >= (uint32_t)kWave) return;
    const bool un = p < n && (a.un_bits[b + p / 8] >> (p % 8) & 1u);
    const uint32_t k = base + (uint32_t)__popcll(__ballot(un) & ((1ull << p) - 1ull));
    if (un) {
      a.un_row[k] = (uint8_t)(sr % a.R);
      reinterpret_cast<float2*>(a.un_yz)[k] = make_float2(a.y[b + p], a.z[b + p]);
    }
    return;
  }
  for (uint32_t w0 = 0; w0 < bytes; w0 += kThreads) {   // block-uniform chunks
    const uint32_t w = w0 + threadIdx.x;
    uint32_t v = w < bytes ? a.un_bits[b + w] : 0u, total;
    uint32_t k = base + block_exclusive_scan<uint32_t>((uint32_t)__popc(v), wsum, &total);
    for (; v; v &= v - 1, ++k) {
      const uint32_t i = b + w * 8 + (uint32_t)__ffs((int)v) - 1;
      a.un_row[k] = (uint8_t)(sr % a.R);
      reinterpret_cast<float2*>(a.un_yz)[k] = make_float2(a.y[i], a.z[i]);
    }
    base += total;
  }
}

// Workgroups [0, row_blocks): the raw lists.  The others: the codes of kChunk
// track clusters.  On the 32-orbit frame (9.3M track clusters) the encoder's
// kernels take 219 us (this one 161 us, about half of it the gather of y and z);
// 455 us when every cluster searched its track and its row in global memory
// from any XCD and the tracks' clusters were marked in a word per cluster.
__global__ void __launch_bounds__(kThreads) k_codec_stream(CodecArgs a, uint32_t row_blocks, uint32_t per) {
#pragma clang fp contract(off)
  __shared__ uint32_t starts[kTrackCap], ro[kMaxRows + 1], wsum[kThreads / kWave], ends[2];
  if (blockIdx.x < row_blocks) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.n_unassigned = a.row_pos[a.SR];
    if (blockIdx.x < a.SR) emit_row(a, blockIdx.x, wsum);
    return;
  }
  const uint32_t blk = blockIdx.x - row_blocks;   // row_blocks is a multiple of kXcds
  const uint64_t j0w = (uint64_t)((blk % kXcds) * per + blk / kXcds) * kChunk;
  if (j0w >= a.n_cl) return;
  const uint32_t j0 = (uint32_t)j0w, j1 = (uint32_t)min((uint64_t)j0 + kChunk, a.n_cl);
  uint32_t id[kPer];
  float ym[kPer], zm[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) id[u] = a.clusters[min(j0 + u * kThreads + threadIdx.x, j1 - 1)];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    ym[u] = a.y[id[u]];
    zm[u] = a.z[id[u]];
  }
  const TrackWindow tw = track_window(a.first_in, a.n_tracks, j0, j1, starts, ends);
  const uint32_t s0 = a.sector[tw.t0];
  for (uint32_t r = threadIdx.x; r <= a.R; r += kThreads) ro[r] = a.row_off[s0 * a.R + r];
  __syncthreads();
  uint32_t esc = 0;
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const uint32_t j = j0 + u * kThreads + threadIdx.x;
    if (j >= j1) break;
    const uint32_t t = tw.staged ? tw.t0 + track_in(tw, j) : last_le(a.first_in, a.n_tracks, j);
    // the row: in the staged offsets unless the window's later tracks are of another sector
    const bool here = id[u] < ro[a.R];
    uint32_t r;
    if (here) r = last_le(ro, a.R, id[u]);
    else r = last_le(a.row_off, a.SR, id[u]) % a.R;
    const float* c = a.coef + 6 * (size_t)t;
    const float xr = a.rows[r].x, xref = a.xref_in[t];
    const float py = predict(xr, xref, c[0], c[1], c[2]);
    const float pz = predict(xr, xref, c[3], c[4], c[5]);
    const float vy = (ym[u] - py) * a.inv_qy;
    const float vz = (zm[u] - pz) * a.inv_qz;
    const bool model = fabsf(a.param[5 * (size_t)t + 2]) < 1.0f;
    short2 k;
    float2 raw = make_float2(0.0f, 0.0f);
    if (model && fabsf(vy) <= 32767.0f && fabsf(vz) <= 32767.0f) {
      k = make_short2((short)(int)rintf(vy), (short)(int)rintf(vz));
    } else {
      k = make_short2(kEscape, 0);
      raw = make_float2(ym[u], zm[u]);
      ++esc;
    }
    a.row[j] = (uint8_t)r;
    reinterpret_cast<short2*>(a.code)[j] = k;
    reinterpret_cast<float2*>(a.raw)[j] = raw;
  }
  // escaped clusters: one atomic per wave
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) esc += (uint32_t)__shfl_xor((int)esc, off, kWave);
  if (threadIdx.x % kWave == 0 && esc) atomicAdd(a.n_escaped, esc);
}

// A decoded coordinate pair.
__device__ __forceinline__ float2 decode_one(const float* c, float xref, float xr, short2 k, float q_y, float q_z) {
#pragma clang fp contract(off)
  const float py = predict(xr, xref, c[0], c[1], c[2]);
  const float pz = predict(xr, xref, c[3], c[4], c[5]);
  const float dy = (float)k.x * q_y;
  const float dz = (float)k.y * q_z;
  return make_float2(py + dy, pz + dz);
}

// The window's models are staged when it has at most kModelCap tracks.  A lane
// takes kPer / kVec groups of kVec consecutive clusters: with kVec = 4 codes,
// rows and results move in 16- and 4-byte units, for arrays aligned to them
// (what an allocator returns); kVec = 1 takes any alignment.  30 us for 9.3M
// track clusters (146 MB, 4.9 TB/s); 110 us when a lane took single clusters
// and read every model from global memory.
constexpr uint32_t kModelCap = 256;
template <int kVec>
__global__ void __launch_bounds__(kThreads) k_codec_decode(DecodeArgs a, uint32_t chunks) {
  __shared__ uint32_t starts[kTrackCap], ends[2];
  __shared__ float model[kModelCap + 1][7], lx[256];
  if (blockIdx.x >= chunks) {   // the clusters on no track
    for (uint64_t k = (uint64_t)(blockIdx.x - chunks) * kThreads + threadIdx.x; k < a.n_un;
         k += (uint64_t)(gridDim.x - chunks) * kThreads) {
      const float2 v = reinterpret_cast<const float2*>(a.un_yz)[k];
      a.y_out[a.n_cl + k] = v.x;
      a.z_out[a.n_cl + k] = v.y;
      a.row_out[a.n_cl + k] = a.un_row[k];
    }
    return;
  }
  // the chunk's clusters, from here on by their place in it
  const uint64_t at = (uint64_t)blockIdx.x * kChunk;
  const uint32_t j0 = (uint32_t)at, n = (uint32_t)min((uint64_t)kChunk, a.n_cl - at);
  const short2* codes = reinterpret_cast<const short2*>(a.code) + at;
  const uint8_t* rows = a.row + at;
  const float2* raw = reinterpret_cast<const float2*>(a.raw) + at;
  float *y_out = a.y_out + at, *z_out = a.z_out + at;
  uint8_t* row_out = a.row_out + at;
  for (uint32_t r = threadIdx.x; r < 256u; r += kThreads) lx[r] = r < a.R ? a.rows[r].x : 0.0f;
  const TrackWindow tw = track_window(a.first, a.n_tracks, j0, j0 + n, starts, ends);
  const bool models = tw.n <= kModelCap;
  if (models)
    for (uint32_t k = threadIdx.x; k < 7 * (tw.n + 1); k += kThreads) {
      const uint32_t t = tw.t0 + k / 7, q = k % 7;
      model[k / 7][q] = q < 6 ? a.coef[6 * (size_t)t + q] : a.x_ref[t];
    }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kPer / kVec; ++u) {
    const uint32_t jb = (u * kThreads + threadIdx.x) * kVec;
    if (jb >= n) break;
    short2 code[kVec];
    uint8_t row[kVec];
    float y[kVec], z[kVec];
    const bool whole = kVec > 1 && jb + kVec <= n;
    if (whole) {
      const int4 cw = *reinterpret_cast<const int4*>(codes + jb);
      const uint32_t rw = *reinterpret_cast<const uint32_t*>(rows + jb);
      const int w4[4] = {cw.x, cw.y, cw.z, cw.w};
#pragma unroll
      for (int v = 0; v < kVec; ++v) {
        code[v] = make_short2((short)w4[v & 3], (short)(w4[v & 3] >> 16));
        row[v] = (uint8_t)(rw >> (8 * v));
      }
    } else {
#pragma unroll
      for (int v = 0; v < kVec; ++v) {
        const uint32_t j = min(jb + v, n - 1);
        code[v] = codes[j];
        row[v] = rows[j];
      }
    }
    uint32_t tl = tw.staged ? track_in(tw, j0 + jb) : 0u;
#pragma unroll
    for (int v = 0; v < kVec; ++v) {
      const uint32_t j = min(jb + v, n - 1);
      if (tw.staged)
        while (tl < tw.n && starts[tl] <= j0 + j) ++tl;
      float2 o;
      if (code[v].x == kEscape) {
        o = raw[j];
      } else {
        const uint32_t t = tw.staged ? tw.t0 + tl : last_le(a.first, a.n_tracks, j0 + j);
        const float xr = row[v] < a.R ? lx[row[v]] : a.rows[row[v]].x;
        if (models) o = decode_one(model[tl], model[tl][6], xr, code[v], a.q_y, a.q_z);
        else o = decode_one(a.coef + 6 * (size_t)t, a.x_ref[t], xr, code[v], a.q_y, a.q_z);
      }
      y[v] = o.x;
      z[v] = o.y;
    }
    if (whole) {
      const int q = kVec > 1 ? 1 : 0;   // indexes inside the arrays for kVec = 1, where this is not reached
      *reinterpret_cast<float4*>(y_out + jb) = make_float4(y[0], y[q], y[2 * q], y[3 * q]);
      *reinterpret_cast<float4*>(z_out + jb) = make_float4(z[0], z[q], z[2 * q], z[3 * q]);
      *reinterpret_cast<uint32_t*>(row_out + jb) = (uint32_t)row[0] | ((uint32_t)row[q] << 8) |
                                                     ((uint32_t)row[2 * q] << 16) | ((uint32_t)row[3 * q] << 24);
    } else {
#pragma unroll
      for (int v = 0; v < kVec; ++v)
        if (jb + v < n) {
          y_out[jb + v] = y[v];
          z_out[jb + v] = z[v];
          row_out[jb + v] = row[v];
        }
    }
  }
}

}  // namespace

void launch_codec_encode(const CodecArgs& a, unsigned long long* scan_blocks, hipStream_t s) {
  const uint32_t model_blocks = std::max(1u, (a.n_tracks + kThreads - 1) / kThreads);
  hipLaunchKernelGGL(k_codec_models, dim3(a.SR + model_blocks), dim3(kThreads), 0, s, a);
  launch_scan_u32(a.row_cnt, a.row_pos, a.SR, scan_blocks, s);
  const uint32_t chunks = (uint32_t)((a.n_cl + kChunk - 1) / kChunk), per = (chunks + kXcds - 1) / kXcds;
  const uint32_t row_blocks = xcd_grid(std::max(1u, a.SR));
  hipLaunchKernelGGL(k_codec_stream, dim3(row_blocks + per * kXcds), dim3(kThreads), 0, s, a, row_blocks, per);
}

void launch_codec_decode(const DecodeArgs& a, hipStream_t s) {
  const uint32_t chunks = (uint32_t)((a.n_cl + kChunk - 1) / kChunk);
  const uint32_t un = (uint32_t)std::min<uint64_t>((a.n_un + kThreads - 1) / kThreads, 2048);
  const bool wide = ((uintptr_t)a.code % 16 | (uintptr_t)a.row % 4 | (uintptr_t)a.y_out % 16 | (uintptr_t)a.z_out % 16 |
                     (uintptr_t)a.row_out % 4) == 0;
  if (wide) hipLaunchKernelGGL(k_codec_decode<4>, dim3(chunks + un), dim3(kThreads), 0, s, a, chunks);
  else hipLaunchKernelGGL(k_codec_decode<1>, dim3(chunks + un), dim3(kThreads), 0, s, a, chunks);
}

}  // namespace tpc
