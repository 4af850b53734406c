// The seed-scan kernels for gfx950 (Yeo et al., CTD/WIT 2019, section 2.2, Eq. 1).
//
// Work decomposition (one MI355X):
//   * one lane per seed; a wave scans chunks of up to 64 seeds of one window. The
//     persistent grid (sized to the resident capacity) shares the chunks event by event
//     (plan_kernel): a workgroup stands in one event at a time, its waves taking the
//     event's chunks one by one with the other workgroups there. With a field map, the
//     65x129 (B_r, B_z) nodes are staged in LDS once per workgroup and shared by all its
//     waves;
//   * the event's hits are staged in LDS, ordered by layer and, within a layer, by
//     the twisted azimuth psi = phi - s_l z of the wire centre; a 1 mm radial table
//     maps a radius range to the layers whose band (widened by the largest drift +
//     sqrt(lambda) + 1 mm) it can meet, and a layer x psi-sector table gives the
//     circular run of a layer's hits that a block in that sector can reach;
//   * each lane runs B RKN steps in registers and writes the B+1 points to an LDS
//     column; it then walks the runs of its block's layers and sector (records
//     gathered from LDS), tests each hit with a sphere bound (all B chords lie within
//     B h / 2 of the block's middle point) and the wave appends the survivors to an
//     LDS work list (ballot + mbcnt compaction);
//   * the list is processed densely (one item per lane, the tail spread over lane
//     groups): exact chord/wire distance of the B chords, the minimum folded into the
//     seed's running minimum (a per-workgroup slab [hit][lane] in HBM, updated with an
//     integer atomic min on the non-negative float bit pattern: order-free and
//     deterministic); a per-wave LDS bitmap marks the (wave, hit) rows that received
//     a minimum in the current tile;
//   * after the last block each lane forms E = sum min((D - d)^2, lambda) in FP64,
//     reading only the marked rows (the others still hold +inf) and resetting them to
//     +inf, so a wave writes its slab columns once and afterwards only where a chunk
//     touched them.
// Every filter is exact: a pair it drops can only have a distance above
// d + sqrt(lambda), where the term is lambda whatever the distance is.
#include <type_traits>

#include <algorithm>

#include "internal.hpp"

namespace rkn {

constexpr int kCap = 176;          // work-list entries per wave
constexpr int kTabBins = 1024;     // 1 mm radial bins, the last one open-ended
constexpr float kBandMargin = 1.0f;   // radial band table
constexpr float kCullMargin = 0.05f;  // sphere test: covers FP32 rounding of the test (~1e-2 mm)
constexpr int kSectors = 256;         // twisted-azimuth sectors of the candidate table (finer
                                      // sectors stage fewer pairs; 256 fill the workgroup's LDS)
// A sector entry: the run's first hit (bits 0-8) and length (bits 9-15); kSectAll
// stands for the whole layer (a run longer than 127 hits, or a reach past pi).
constexpr uint32_t kSectAll = 0xffffu;
constexpr int kPipeWaves = 12;  // waves per workgroup of pipe_kernel at most
constexpr int kTraceFold = 8;   // rkn_trace: steps between folds of the block-relative sums
constexpr float kPi = 3.14159265358979f;

// How scan_kernel divides a launch's chunks. len > 0: tiles of at most len chunks of one
// event, one for each workgroup (n_tiles of them). len = 0: each event's chunks are taken
// from its own counter. Behind it in memory, per event [n_events + 1]: its first tile, or
// the chunks taken.
struct ScanPlan {
  int64_t chunk0, chunk_end;  // the launch's chunks
  int32_t len, n_tiles, n_events;
};
constexpr size_t kPlanHead = 64;

struct ScanArgs {
  FieldDev field;
  const HitRec<float>* hits32;
  const HitRec<double>* hits64;
  const int32_t* ev_off;
  const int32_t* layer_off;   // [n_events][n_layers+1]
  const float2* layer_r;      // (rmin, rmax) per layer
  const float* ev_maxdrift;
  const float* hits_phi;      // twisted azimuth psi of each layer-ordered hit's wire centre
  const float2* layer_twist;  // [n_events][n_layers] (dphi/dz of the layer's wires, psi deviation)
  float wire_zmin, wire_zmax; // z extent of all wires
  float b_max;                // |B| is nowhere larger
  int n_layers;
  int sect_bytes;             // LDS bytes reserved for the layer x sector table
  int hits_bytes;             // LDS bytes reserved for hit records
  int field_bytes;            // LDS bytes reserved for the field map (0: uniform)
  int touch_words;            // 32-bit words of a wave's row bitmap (>= max hits / 32)
  int n_pairs, n_con, pair_bytes;   // pipe_kernel: pairs per workgroup, consumers and LDS bytes of one
  const Seg* segs;            // [n_seg + 1]: windows (or explicit seeds' events) and their chunks
  int n_seg;
  const int32_t* n_seg_dev;   // if set, the segment count is read here (captured launches)
  const int64_t* ev_chunk;    // first chunk of each event [n_events + 1]
  int n_events;
  int walk;                   // 1: windows walked in scan order, lanes out of reach in z not culled; -1: not decided
  int64_t chunk0, n_chunks;   // the chunks to scan: [chunk0, chunk0 + n_chunks)
  const int64_t* n_chunks_dev;   // if set, n_chunks is read here
  const WindowDev* windows;
  const double* seeds5;       // explicit seeds [n][5] in scan order (NULL: windows)
  const int64_t* perm;        // scan order -> caller index (explicit seeds)
  ScanPlan* plan;             // scan_kernel's division of the chunks (plan_kernel writes it)
  void* mscratch;
  int64_t slab_stride;        // elements per workgroup slab
  double R0, charge, h, lambda;
  int n_steps;
  int turn_stop;              // 1: a lane's track ends with the first step inside r < R0
  double* score;
  int32_t* nin;
  ArgminPart* parts;          // per chunk, [chunk - chunk0]
  // refinement forward mode (MODE 1): per output slot = scan position
  const int32_t* hits_orig;   // original index (within its event) of each layer-ordered hit
  const int64_t* base_of;     // scan position -> refinement seed whose inlier set applies
  uint8_t* mask;              // [n_base][max_hits] inlier flags (original hit order)
  int define_mask;            // 1: set mask from (D - d)^2 < lambda, 0: read it
  float* resid;               // [n_pos][max_hits] residual D - d of inliers, NaN otherwise
  int32_t* argmin_step;       // [n_pos][max_hits] chord index of the minimum (inliers), -1 otherwise
  double* phi;                // [n_pos] sum of squared inlier residuals
  float* tape;                // [n_ckpt][13][n_pos] FP32 states every ckpt steps (NULL: none)
  int ckpt, n_ckpt;
  int64_t n_pos;
  int max_hits;
  // adaptive step size (scan_kernel variant 2): path length, error bound, step range
  double path_len;
  float tol, h_min, h_max;
  // work counters of the counting instance (COUNT): seed-steps taken, sphere tests
  // made, chord/wire distances evaluated
  unsigned long long* work;
};

// ---------------------------------------------------------------------------------
// Upload-time preparation: per event, order the hits by layer and, within a layer,
// by the twisted azimuth psi = phi(m) - s_l m_z of the wire centre m (ties by upload
// order), where s_l = dphi/dz of the layer's stereo wires (taken from the layer's
// first hit). Along a wire, phi - s_l z stays within dev_l of psi; the kernel uses
// (s_l, dev_l) per layer to turn a block's middle point into a psi window. Also
// builds the FP32/FP64 hit records, the per-layer offsets and the event's largest
// drift.
// Azimuth for the sector lookup: octant reduction and an odd degree-7 polynomial
// for atan on [0, 1] (our least-squares fit; |error| < 1e-4 rad, far inside the
// table's 2e-3 rad margin).
__device__ __forceinline__ float sector_atan2(float y, float x) {
  const float ax = fabsf(x), ay = fabsf(y);
  const float hi = fmaxf(ax, ay), lo = fminf(ax, ay);
  const float t = hi > 0.0f ? lo * __builtin_amdgcn_rcpf(hi) : 0.0f;
  const float u = t * t;
  float r = t * fmaf(fmaf(fmaf(-0.03898633f, u, 0.14626420f), u, -0.32117486f), u, 0.99921381f);
  r = ay > ax ? 0.5f * kPi - r : r;
  r = x < 0.0f ? kPi - r : r;
  return y < 0.0f ? -r : r;
}

__device__ __forceinline__ float wrap_pi(float d) {
  return d >= kPi ? d - 2.0f * kPi : (d < -kPi ? d + 2.0f * kPi : d);
}

__global__ void __launch_bounds__(256)
prep_hits_kernel(const int32_t* __restrict__ ev_off, const int32_t* __restrict__ wire_id,
                 const float* __restrict__ drift, const HitRec<float>* __restrict__ wire32,
                 const HitRec<double>* __restrict__ wire64, const int32_t* __restrict__ wire_layer,
                 int n_layers, HitRec<float>* __restrict__ out32, HitRec<double>* __restrict__ out64,
                 int32_t* __restrict__ layer_off, float* __restrict__ ev_maxdrift, int32_t* __restrict__ orig,
                 float* __restrict__ out_psi, float2* __restrict__ layer_twist) {
  __shared__ int s_layer[RKN_MAX_HITS_PER_EVENT];
  __shared__ float s_psi[RKN_MAX_HITS_PER_EVENT];
  __shared__ int s_count[RKN_MAX_LAYERS + 1];
  __shared__ int s_first[RKN_MAX_LAYERS];
  __shared__ unsigned int s_dev[RKN_MAX_LAYERS];
  __shared__ float s_slope[RKN_MAX_LAYERS];
  __shared__ unsigned int s_max;
  const int e = blockIdx.x, tid = threadIdx.x;
  const int base = ev_off[e], n = ev_off[e + 1] - base;
  for (int l = tid; l <= n_layers; l += blockDim.x) s_count[l] = 0;
  for (int l = tid; l < n_layers; l += blockDim.x) {
    s_dev[l] = 0u;
    s_first[l] = 0x7fffffff;
  }
  if (tid == 0) s_max = 0u;
  __syncthreads();
  unsigned int mymax = 0u;
  for (int i = tid; i < n; i += blockDim.x) {
    const int l = wire_layer[wire_id[base + i]];
    s_layer[i] = l;
    atomicAdd(&s_count[l], 1);
    atomicMin(&s_first[l], i);
    const unsigned int bits = __float_as_uint(drift[base + i]);
    mymax = bits > mymax ? bits : mymax;
  }
  atomicMax(&s_max, mymax);
  __syncthreads();
  for (int l = tid; l < n_layers; l += blockDim.x) {
    float sl = 0.0f;
    if (s_first[l] < n) {
      const HitRec<float> r = wire32[wire_id[base + s_first[l]]];
      const float r2 = r.mx * r.mx + r.my * r.my;
      sl = (fabsf(r.uz) > 1e-6f && r2 > 0.0f) ? (r.mx * r.uy - r.my * r.ux) / (r2 * r.uz) : 0.0f;
    }
    s_slope[l] = sl;
  }
  __syncthreads();
  for (int i = tid; i < n; i += blockDim.x) {
    const int l = s_layer[i];
    const float sl = s_slope[l];
    const HitRec<float> r = wire32[wire_id[base + i]];
    const float phi = atan2f(r.my, r.mx);
    s_psi[i] = wrap_pi(phi - sl * r.mz);
    float dev = 0.0f;
    for (int q = -2; q <= 2; ++q) {
      if (q == 0) continue;
      const float t = 0.5f * (float)q * r.L;
      const float d = wrap_pi(atan2f(r.my + t * r.uy, r.mx + t * r.ux) - phi) - sl * r.uz * t;
      dev = fmaxf(dev, fabsf(d));
    }
    atomicMax(&s_dev[l], __float_as_uint(dev));
  }
  __syncthreads();
  if (tid == 0) {
    int acc = 0;
    for (int l = 0; l < n_layers; ++l) {
      const int c = s_count[l];
      s_count[l] = acc;
      acc += c;
    }
    s_count[n_layers] = acc;
    for (int l = 0; l <= n_layers; ++l) layer_off[(size_t)e * (n_layers + 1) + l] = s_count[l];
    // the deviation is sampled at t = +-L/2, +-L; its curvature term is bounded by
    // doubling the sampled maximum
    for (int l = 0; l < n_layers; ++l)
      layer_twist[(size_t)e * n_layers + l] = make_float2(s_slope[l], 2.0f * __uint_as_float(s_dev[l]));
    ev_maxdrift[e] = __uint_as_float(s_max);
  }
  __syncthreads();
  for (int i = tid; i < n; i += blockDim.x) {
    const int l = s_layer[i];
    const float psi = s_psi[i];
    int rank = s_count[l];
    for (int j = 0; j < n; ++j)
      rank += (s_layer[j] == l) && (s_psi[j] < psi || (s_psi[j] == psi && j < i));
    const int w = wire_id[base + i];
    HitRec<float> r32 = wire32[w];
    HitRec<double> r64 = wire64[w];
    r32.drift = drift[base + i];
    r64.drift = (double)drift[base + i];
    out32[base + rank] = r32;
    out64[base + rank] = r64;
    orig[base + rank] = i;
    out_psi[base + rank] = psi;
  }
}

hipError_t launch_prep_hits(rkn_ctx* c, const int32_t* d_wire_id, const float* d_drift) {
  if (c->n_events == 0) return hipSuccess;
  hipLaunchKernelGGL(prep_hits_kernel, dim3(c->n_events), dim3(256), 0, c->stream,
                     c->ev_off.as<int32_t>(), d_wire_id, d_drift, c->wire32.as<HitRec<float>>(),
                     c->wire64.as<HitRec<double>>(), c->wire_layer.as<int32_t>(), c->n_layers,
                     c->hits32.as<HitRec<float>>(), c->hits64.as<HitRec<double>>(),
                     c->layer_off.as<int32_t>(), c->ev_maxdrift.as<float>(), c->hits_orig.as<int32_t>(),
                     c->hits_phi.as<float>(), c->layer_ext.as<float2>());
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
__device__ __forceinline__ unsigned long long* plan_events(ScanPlan* p) {
  return reinterpret_cast<unsigned long long*>(reinterpret_cast<unsigned char*>(p) + kPlanHead);
}

// The chunks of event e that belong to the launch: [first, returned end).
__device__ __forceinline__ int64_t event_chunks(const ScanPlan* p, const int64_t* ev_chunk, int e, int64_t* first) {
  *first = max(ev_chunk[e], p->chunk0);
  return max(min(ev_chunk[e + 1], p->chunk_end), *first);
}

constexpr int kPlanThreads = 1024;
constexpr int kMaxWaves = 16;    // waves of a scan_kernel workgroup at most

// One workgroup: the division of a launch's n chunks over `grid` workgroups of `waves`
// waves, on n_cu CUs (see ScanPlan). A workgroup stages one event at a time, so a share of
// chunks that lies in two events costs it two rounds.
//  * At most one chunk per wave: the shortest tiles that end with their event and give each
//    workgroup at most one, in as few workgroups per CU as can be (200 events of 4 chunks:
//    1.75 ms in equal shares, 0.79 ms in tiles).
//  * More, or more events than workgroups: every workgroup starts at its place in the
//    chunks and takes its event's chunks one by one with the other workgroups there, then
//    those of the events up to the next workgroup's place, then helps where chunks are
//    left. (One run of 7/8 of its share per workgroup and a queue of runs for the rest,
//    cut without regard to events: 64 events of 64 chunks 2.9 ms, 4000 events of one chunk
//    20 ms; this way 2.0 and 13.)
__global__ void __launch_bounds__(kPlanThreads) plan_kernel(ScanArgs a, int grid, int waves, int n_cu) {
  __shared__ int s_tiles[kMaxWaves + 1];
  __shared__ int s_sum[kPlanThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t n = a.n_chunks_dev ? *a.n_chunks_dev : a.n_chunks;
  ScanPlan plan{a.chunk0, a.chunk0 + n, 0, 0, a.n_events};
  unsigned long long* per_event = plan_events(a.plan);
  auto chunks_of = [&](int e) {
    int64_t first;
    return event_chunks(&plan, a.ev_chunk, e, &first) - first;
  };
  if (n <= (int64_t)grid * waves) {
    // tiles of every length 1 .. waves; summed in the wave first (200 lanes adding to one
    // counter each: 35 us)
    for (int l = tid; l <= kMaxWaves; l += kPlanThreads) s_tiles[l] = 0;
    __syncthreads();
    int t[kMaxWaves + 1] = {0};
    for (int e = tid; e < a.n_events; e += kPlanThreads) {
      const int c = (int)chunks_of(e);
#pragma unroll
      for (int l = 1; l <= kMaxWaves; ++l) t[l] += (c + l - 1) / l;
    }
#pragma unroll
    for (int l = 1; l <= kMaxWaves; ++l) {
      for (int o = 32; o >= 1; o >>= 1) t[l] += __shfl_xor(t[l], o, 64);
      if (lane == 0 && t[l]) atomicAdd(&s_tiles[l], t[l]);
    }
    __syncthreads();
    const int per_cu = (int)((n + (int64_t)n_cu * waves - 1) / ((int64_t)n_cu * waves));
    for (int g = min(max(per_cu, 1) * n_cu, grid);; g = min(g + n_cu, grid)) {
      int l = 1;
      while (l <= waves && s_tiles[l] > g) ++l;
      if (l <= waves) {
        plan.len = l;
        plan.n_tiles = s_tiles[l];
      }
      if (plan.len > 0 || g >= grid) break;
    }
  }
  if (plan.len == 0) {
    for (int e = tid; e < a.n_events; e += kPlanThreads) per_event[e] = 0;
  } else {
    // the events' first tiles: a running sum over the events
    int total = 0;
    for (int e0 = 0; e0 < a.n_events; e0 += kPlanThreads) {
      const int e = e0 + tid;
      const int t = e < a.n_events ? ((int)chunks_of(e) + plan.len - 1) / plan.len : 0;
      int incl = t;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(incl, o, 64);
        if (lane >= o) incl += x;
      }
      __syncthreads();   // the sums of the round before have been read
      if (lane == 63) s_sum[wave] = incl;
      __syncthreads();
      int base = total;
      for (int w = 0; w < kPlanThreads / 64; ++w) {
        if (w < wave) base += s_sum[w];
        total += s_sum[w];
      }
      if (e < a.n_events) per_event[e] = (unsigned long long)(base + incl - t);
    }
  }
  if (tid == 0) *a.plan = plan;
}

template <typename R>
__device__ __forceinline__ const HitRec<R>* hits_of(const ScanArgs& a);
template <>
__device__ __forceinline__ const HitRec<float>* hits_of<float>(const ScanArgs& a) { return a.hits32; }
template <>
__device__ __forceinline__ const HitRec<double>* hits_of<double>(const ScanArgs& a) { return a.hits64; }

template <typename R>
__device__ __forceinline__ void atomic_min_nonneg(R* p, R v) {
  if constexpr (sizeof(R) == 4) {
    atomicMin(reinterpret_cast<unsigned int*>(p), __float_as_uint(v));
  } else {
    atomicMin(reinterpret_cast<unsigned long long*>(p), (unsigned long long)__double_as_longlong(v));
  }
}

template <typename R>
__device__ __forceinline__ R load_coherent(const R* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Fold one item's block minimum into the seed's running minimum for the hit. In
// the scan, a block whose minimum is not below (d + sqrt(lambda))^2 cannot change
// the hit's term (it stays lambda unless another block comes closer), so it is not
// written. The refinement pass writes every block (its inlier set is fixed).
// The wave's row of the hit is marked in its LDS bitmap.
template <typename R, int TILE, int MODE, typename S>
__device__ __forceinline__ void fold_min(S* slab, uint32_t* touch, int hh, int s, R d2, int chord, R lim2) {
  if constexpr (MODE == 0) {
    if (!(d2 < lim2)) return;
    atomic_min_nonneg(slab + (size_t)hh * TILE + s, d2);
  } else {
    // (distance bits, chord index): the minimum distance, then the lowest chord
    const unsigned long long key =
        ((unsigned long long)__float_as_uint((float)d2) << 32) | (unsigned long long)(unsigned)chord;
    atomicMin(reinterpret_cast<unsigned long long*>(slab + (size_t)hh * TILE + s), key);
  }
  atomicOr(touch + (hh >> 5), 1u << (hh & 31));
}

// Dense pass over a wave's work list: item = (lane << 16) | hit. Full groups of 64
// items take one item per lane and all chords of the block; the remaining n < 64
// items take G lanes each (G = 8, 4 or 2 with G n <= 64), the chords of an item
// strided over its lanes, so the tail pass costs about B / G chords instead of B.
// The fold is an atomic minimum of (distance[, chord]) and so order-free: lanes of an
// item may fold separately and the seed's running minimum ends as after a full
// reduction over the G lanes. In the scan, adjacent lanes first merge their minima
// with one row shift (half the atomics, and half their L2 write-backs, for three
// instructions); the refinement pass folds every lane's (distance, chord) key.
template <typename R, int B, int TILE, int COLS, int MODE, bool Y_FIRST, typename S>
__device__ __forceinline__ void flush_items(const uint32_t* items, int n_items, const R* pts,
                                            const HitRec<R>* s_hits, S* slab, uint32_t* touch, int lane,
                                            int nb, int step0, R sqrt_lam) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  int done = 0;
  for (; n_items - done >= 64; done += 64) {
    const uint32_t it = items[done + lane];
    const int s = (int)(it >> 16), hh = (int)(it & 0xffffu);
    const HitRec<R> w = s_hits[hh];
    R px = pts[0 * COLS + s], py = pts[1 * COLS + s], pz = pts[2 * COLS + s];
    R dmin = (R)INFINITY;
    int jmin = 0;
#pragma unroll
    for (int j = 1; j <= B; ++j) {
      if (j <= nb) {
        const R qx = pts[(j * 3 + 0) * COLS + s], qy = pts[(j * 3 + 1) * COLS + s],
                qz = pts[(j * 3 + 2) * COLS + s];
        const R d2 = j > 1 && !Y_FIRST
                         ? seg_wire_d2<R, true>(px, py, pz, qx, qy, qz, w.mx, w.my, w.mz, w.ux, w.uy, w.uz, w.L)
                         : seg_wire_d2<R>(px, py, pz, qx, qy, qz, w.mx, w.my, w.mz, w.ux, w.uy, w.uz, w.L);
        if (d2 < dmin) {
          dmin = d2;
          jmin = j - 1;
        }
        px = qx;
        py = qy;
        pz = qz;
      }
    }
    const R lim = w.drift + sqrt_lam;
    fold_min<R, TILE, MODE>(slab, touch, hh, s, dmin, step0 + jmin, lim * lim);
  }
  const int n_rem = n_items - done;
  if (n_rem > 0) {
    const int G = n_rem <= 8 ? 8 : (n_rem <= 16 ? 4 : (n_rem <= 32 ? 2 : 1));
    const int k = lane / G, sub = lane - k * G;
    const bool act = k < n_rem;
    const uint32_t it = items[done + (act ? k : 0)];
    const int s = (int)(it >> 16), hh = (int)(it & 0xffffu);
    const HitRec<R> w = s_hits[hh];
    R dmin = (R)INFINITY;
    int jmin = 0;
    for (int j = sub; j < nb; j += G) {
      const R d2 = seg_wire_d2<R>(pts[(j * 3 + 0) * COLS + s], pts[(j * 3 + 1) * COLS + s], pts[(j * 3 + 2) * COLS + s],
                                  pts[(j * 3 + 3) * COLS + s], pts[(j * 3 + 4) * COLS + s], pts[(j * 3 + 5) * COLS + s],
                                  w.mx, w.my, w.mz, w.ux, w.uy, w.uz, w.L);
      if (d2 < dmin) {   // the lane's chords in increasing order: keeps the lowest on ties
        dmin = d2;
        jmin = j;
      }
    }
    bool folds = act && sub < nb;
    if constexpr (MODE == 0 && sizeof(R) == 4) {
      if (G > 1) {
        // pairs of an item's lanes (aligned inside rows of 16) merge their minima first:
        // non-negative floats order as their bit patterns
        const unsigned bits = __float_as_uint(dmin);
        const unsigned o = (unsigned)__builtin_amdgcn_update_dpp((int)bits, (int)bits, 0x101, 0xf, 0xf, false);
        dmin = __uint_as_float(o < bits ? o : bits);
        folds = folds && (sub & 1) == 0;
      }
    }
    if (folds) {
      const R lim = w.drift + sqrt_lam;
      fold_min<R, TILE, MODE>(slab, touch, hh, s, dmin, step0 + jmin, lim * lim);
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS writes of the wave's lanes visible to all its lanes (list handoffs within a wave).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Dense sphere test of the staged candidates items[lo, hi) (item = (lane << 16) | hit),
// one per lane: the wire's line against the sphere of radius Kcull + d around the
// middle point of the owner lane's block (column jc of its points). Survivors are
// compacted in place from items[lo] on (every lane reads its chunk before any lane
// writes, and survivors never pass the chunk being read); returns their end.
template <typename R, int COLS, bool COUNT>
__device__ __forceinline__ int test_staged(uint32_t* items, int lo, int hi, const R* pts, const HitRec<R>* s_hits,
                                           int jc, R Kcull, int lane, int nb, unsigned long long& w_tests,
                                           unsigned long long& w_chords) {
  wave_sync();
  int out = lo;
  for (int base = lo; base < hi; base += 64) {
    const bool act = base + lane < hi;
    const uint32_t it = items[act ? base + lane : lo];
    wave_sync();
    const int s = (int)(it >> 16), hh = (int)(it & 0xffffu);
    const HitRec<R> w = s_hits[hh];
    const R cx = pts[(jc * 3 + 0) * COLS + s], cy = pts[(jc * 3 + 1) * COLS + s], cz = pts[(jc * 3 + 2) * COLS + s];
    const R rx = cx - w.mx, ry = cy - w.my, rz = cz - w.mz;
    const R tt = rx * w.ux + ry * w.uy + rz * w.uz;
    const R d2 = rx * rx + ry * ry + rz * rz - tt * tt;
    const R thr = Kcull + w.drift;
    const bool pass = act & (d2 <= thr * thr);   // every lane's loads are in bounds
    if constexpr (COUNT) {
      w_tests += act ? 1 : 0;
      w_chords += pass ? nb : 0;
    }
    const uint64_t m = __ballot(pass);
    if (pass) items[out + lane_rank(m)] = it;
    out += (int)__popcll(m);
    wave_sync();
  }
  return out;
}

// The staged event: its hits and the tables the cull walks (LDS).
template <typename R>
struct EventLds {
  HitRec<R>* hits;
  uint16_t* ltab;    // 1 mm radial bin -> layers [l0, l1p), l0 | l1p << 8
  uint16_t* sect;    // layer x twisted-azimuth sector -> run of the layer's hits
  int* loff;         // first hit of each layer
  float* slope;      // dphi/dz of each layer's wires
};

// Stage event ev with nthreads threads (the caller's barriers order it).
template <typename R>
__device__ __forceinline__ void stage_event(const ScanArgs& a, const EventLds<R>& L, int ev, int tid, int nthreads,
                                            double block_len) {
  const int hbase = a.ev_off[ev];
  const int nh = a.ev_off[ev + 1] - hbase;
  const HitRec<R>* ghits = hits_of<R>(a) + hbase;
  for (int i = tid; i < nh; i += nthreads) L.hits[i] = ghits[i];
  const int32_t* loff = a.layer_off + (size_t)ev * (a.n_layers + 1);
  for (int l = tid; l <= a.n_layers; l += nthreads) L.loff[l] = loff[l];
  // radial bins: the layers whose band, widened by the event's largest drift +
  // sqrt(lambda) + 1 mm, meets the bin: [l0, l1p) packed as l0 | l1p << 8
  const float D = a.ev_maxdrift[ev] + (float)sqrt(a.lambda) + kBandMargin;
  for (int b = tid; b < kTabBins; b += nthreads) {
    const float lo_r = (float)b, hi_r = b == kTabBins - 1 ? INFINITY : (float)(b + 1);
    int l0 = 0;
    while (l0 < a.n_layers && a.layer_r[l0].y + D < lo_r) ++l0;
    int l1 = a.n_layers - 1;
    while (l1 >= 0 && a.layer_r[l1].x - D > hi_r) --l1;
    L.ltab[b] = (uint16_t)(l0 | ((l1 + 1) << 8));
  }
  // layer x twisted-azimuth sector: the circular run of a layer's hits (sorted by
  // psi) that a block whose middle point c has psi_c = phi_c - s_l z_c in the
  // sector can reach. A kept pair needs a wire point w within
  // rho = d + sqrt(lambda) + margin + B h / 2 of c; then |phi_w - phi_c| <=
  // 2 asin(rho / (2 (r_l - rho))) (radii >= r_l - rho and r_l),
  // |z_w - z_c| <= rho, and phi_w - s_l z_w is within dev_l of the hit's psi.
  const float rho = a.ev_maxdrift[ev] + (float)sqrt(a.lambda) + kCullMargin + 0.5f * (float)block_len;
  const float* gpsi = a.hits_phi + hbase;
  for (int l = tid; l < a.n_layers; l += nthreads) L.slope[l] = a.layer_twist[(size_t)ev * a.n_layers + l].x;
  for (int q = tid; q < a.n_layers * kSectors; q += nthreads) {
    const int l = q / kSectors, k = q - l * kSectors;
    const int lb = loff[l], nl = loff[l + 1] - lb;
    uint32_t ent = 0u;
    if (nl > 0) {
      const float2 tw = a.layer_twist[(size_t)ev * a.n_layers + l];
      const float rl = a.layer_r[l].x - rho;
      const float ratio = rl > 0.0f ? rho / (2.0f * rl) : 2.0f;
      const float dphi = ratio < 1.0f ? 2.0f * asinf(ratio) : kPi;
      const float W = dphi + fabsf(tw.x) * rho + tw.y + 2e-3f;
      if (W >= kPi) {
        ent = kSectAll;
      } else {
        const float a0 = -kPi + (2.0f * kPi / kSectors) * k, a1 = a0 + 2.0f * kPi / kSectors;
        auto inside = [&](int j) {
          const float ps = gpsi[lb + j];
          if (ps >= a0 && ps <= a1) return true;
          float d1 = a0 - ps, d2 = ps - a1;
          d1 -= 2.0f * kPi * floorf(d1 / (2.0f * kPi));
          d2 -= 2.0f * kPi * floorf(d2 / (2.0f * kPi));
          return fminf(d1, d2) <= W;
        };
        int cnt = 0, start = -1;
        bool prev = inside(nl - 1);
        for (int j = 0; j < nl; ++j) {
          const bool in = inside(j);
          cnt += in;
          if (in && !prev && start < 0) start = j;
          prev = in;
        }
        if (cnt == nl) start = 0;
        ent = cnt > 127 ? kSectAll : (cnt > 0 ? ((uint32_t)start | ((uint32_t)cnt << 9)) : 0u);
      }
    }
    L.sect[q] = (uint16_t)ent;
  }
}

// One lane's place in a chunk: whether it has a seed, and the seed's output index.
struct LaneSlot {
  bool in_tile;
  int64_t gidx;
};

// A chunk's lanes; with v not NULL also their seeds (lanes without one repeat the first).
__device__ __forceinline__ LaneSlot lane_slot(const ScanArgs& a, int seg, int64_t ch, int lane, double* v) {
  const Seg sg = a.segs[seg];
  const int64_t first = (ch - sg.chunk0) * kChunk;
  LaneSlot q;
  q.in_tile = lane < sg.size - first;
  const int64_t local = first + (q.in_tile ? lane : 0);
  q.gidx = sg.gbase + local;
  if (a.seeds5) {
    if (v) {
#pragma unroll
      for (int d = 0; d < 5; ++d) v[d] = a.seeds5[q.gidx * 5 + d];
    }
    q.gidx = a.perm[q.gidx];
  } else if (a.walk) {
    q.gidx = sg.gbase + window_scan_seed(a.windows[seg], local, v);
  } else if (v) {
    window_seed(a.windows[seg], local, v);
  }
  return q;
}

// The starting state of a chunk's lanes; valid: the lane's seed has a momentum.
template <typename R>
__device__ __forceinline__ LaneSlot load_seed(const ScanArgs& a, int seg, int64_t ch, int lane, State<R>& st,
                                              bool& valid) {
  double v[5];
  const LaneSlot q = lane_slot(a, seg, ch, lane, v);
  const double pm = sqrt(v[2] * v[2] + v[3] * v[3] + v[4] * v[4]);
  valid = q.in_tile && (pm >= 1e-3);
  const double ipm = valid ? 1.0 / pm : 0.0;
  st.x = (R)(a.R0 * cos(v[0]));
  st.y = (R)(a.R0 * sin(v[0]));
  st.z = (R)v[1];
  st.tx = valid ? (R)(v[2] * ipm) : (R)1;
  st.ty = valid ? (R)(v[3] * ipm) : (R)0;
  st.tz = valid ? (R)(v[4] * ipm) : (R)0;
  st.lam = valid ? (R)(kKappa * a.charge * ipm) : (R)0;
  st.cx = st.cy = st.cz = (R)0;
  st.ctx = st.cty = st.ctz = (R)0;
  return q;
}

// The checkpoint of a lane at one of the refinement pass's checkpoint steps.
template <typename R>
__device__ __forceinline__ void write_tape(const ScanArgs& a, int step, int64_t gidx, const State<R>& st) {
  float* tp = a.tape + (size_t)(step / a.ckpt) * 13 * a.n_pos + gidx;
  const float v13[13] = {(float)st.x,   (float)st.y,   (float)st.z,   (float)st.cx, (float)st.cy, (float)st.cz,
                         (float)st.tx,  (float)st.ty,  (float)st.tz,  (float)st.ctx, (float)st.cty, (float)st.ctz,
                         (float)st.lam};
#pragma unroll
  for (int q = 0; q < 13; ++q) tp[(size_t)q * a.n_pos] = v13[q];
}

// Segment holding chunk ch: segs[s].chunk0 <= ch < segs[s + 1].chunk0.
__device__ __forceinline__ int find_seg(const Seg* segs, int n_seg, int64_t ch) {
  int lo = 0, hi = n_seg;
  while (hi - lo > 1) {
    const int mid = (lo + hi) / 2;
    if (segs[mid].chunk0 <= ch)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// The same from segment lo on, which starts at or before ch: by doubling steps, since the
// chunk lies in the same or the next segment where an event has few windows, and anywhere in
// the event where it has many (10^5 one-point windows).
__device__ __forceinline__ int find_seg_from(const Seg* segs, int n_seg, int lo, int64_t ch) {
  int step = 1;
  while (lo + step < n_seg && segs[lo + step].chunk0 <= ch) {
    lo += step;
    step *= 2;
  }
  return lo + find_seg(segs + lo, min(step, n_seg - lo), ch);
}

// One block of fixed steps of a wave's lanes: the points into the lanes' columns, the
// radial range of the block (r2min, r2max), and the block's increments into the origin
// (the folded position, within an ulp of the last one, ends the block's last chord and
// starts the next block). VAR 1: a lane whose track ended keeps its state.
//
// Where no lane can come back inside r < R0 within the block (steady lanes move at most
// 1.1 h per step), the live lanes step without a test in between, and the scheduler can
// overlap their steps. Tested after every step, a step took half as long again: 24 events'
// turn loop, 308 -> 292 ms.
template <typename R, int FIELD, int B, int COLS, int VAR>
__device__ __forceinline__ void take_block(const ScanArgs& a, const float2* nodes, State<R>& st, Prop<R, FIELD>& pr,
                                           R* pts, int lane, int nb, R h, R r0sq, R far2, bool steady, bool& live,
                                           R& r2min, R& r2max) {
  const bool live0 = live;
  pts[0 * COLS + lane] = st.x;
  pts[1 * COLS + lane] = st.y;
  pts[2 * COLS + lane] = st.z;
  r2min = r2max = pr.r2;
  auto take = [&](int j, bool go) {
    if (go) pr.step(st, a.field, nodes, h);
    pts[(j * 3 + 0) * COLS + lane] = pr.px;
    pts[(j * 3 + 1) * COLS + lane] = pr.py;
    pts[(j * 3 + 2) * COLS + lane] = pr.pz;
    r2min = vmin(r2min, pr.r2);
    r2max = vmax(r2max, pr.r2);
  };
  if constexpr (VAR == 1) {
    if (nb == B && __ballot(live && (!steady || pr.r2 < far2)) == 0) {
      if (live) {
#pragma unroll
        for (int j = 1; j <= B; ++j) take(j, true);
      }
    } else if (nb == B) {
#pragma unroll
      for (int j = 1; j <= B; ++j) {
        take(j, live);
        live = live && !inside_r0(pr.px, pr.py, r0sq);
      }
    } else {
      for (int j = 1; j <= B; ++j) {
        take(j, j <= nb && live);
        live = live && !inside_r0(pr.px, pr.py, r0sq);
      }
    }
  } else if (nb == B) {   // every block but a short last one: straight-line steps
#pragma unroll
    for (int j = 1; j <= B; ++j) take(j, true);
  } else {
    for (int j = 1; j <= B; ++j) take(j, j <= nb);
  }
  if (VAR == 0 || live0) {
    pr.fold(st);
    pts[(nb * 3 + 0) * COLS + lane] = pr.px;
    pts[(nb * 3 + 1) * COLS + lane] = pr.py;
    pts[(nb * 3 + 2) * COLS + lane] = pr.pz;
    r2min = vmin(r2min, pr.r2);
    r2max = vmax(r2max, pr.r2);
  }
}

// take_block for a seed on four lanes (see QuadProp): the wave's 16 seeds from column sd.
template <int B, int COLS, int VAR>
__device__ __forceinline__ void take_block_quad(const ScanArgs& a, const float* nodes, QuadProp& pr, float* pts, int sd,
                                                int comp, int nb, float h, float r0sq, float far2, bool steady,
                                                bool& live, float& r2min, float& r2max) {
  const bool live0 = live;
  float* col = pts + comp * COLS + sd;
  col[0] = pr.s;
  r2min = r2max = pr.r2;
  auto take = [&](int j, bool go) {
    if (go) pr.step(a.field, nodes, h);
    col[j * 3 * COLS] = pr.p;
    r2min = fminf(r2min, pr.r2);
    r2max = fmaxf(r2max, pr.r2);
  };
  if (nb == B && (VAR == 0 || __ballot(live && (!steady || pr.r2 < far2)) == 0)) {
    if (VAR == 0 || live) {
#pragma unroll
      for (int j = 1; j <= B; ++j) take(j, true);
    }
  } else {
    for (int j = 1; j <= B; ++j) {
      take(j, j <= nb && (VAR == 0 || live));
      if constexpr (VAR == 1) live = live && !inside_r0(quad_perm<0x00>(pr.p), quad_perm<0x55>(pr.p), r0sq);
    }
  }
  if (VAR == 0 || live0) {
    pr.fold();
    col[nb * 3 * COLS] = pr.p;
    r2min = fminf(r2min, pr.r2);
    r2max = fmaxf(r2max, pr.r2);
  }
}

// Whether a lane's steps keep |T| near 1 over the whole path (the integrator's drift per
// step is of order (h |lam B|)^5), so that none is longer than 1.1 h.
template <typename R>
__device__ __forceinline__ bool steady_lane(const ScanArgs& a, R lam) {
  return a.n_steps <= 100000 && fabsf((float)lam) * (float)a.h * a.b_max < 0.02f;
}

// Wire candidates of one block for the wave's 64 lanes, and the chord distances of the
// kept pairs. Per lane: whether its block is to be culled (on), the radial range of its
// points (r2min, r2max) and its points in column `lane` of pts (COLS columns; lanes past
// them have no block).
//
// With z_skip, a block whose middle point lies outside [z_lo, z_hi] is out of every wire's
// reach along z and has no candidates (it would hold 16 % of the 512-event batch's
// distances). Only the scan drops it: the refinement's inliers count wherever they are, and
// the counting instance counts the pairs of the radial and sphere rules.
//
// Per layer whose band meets the block's radial range, the candidates are the run of
// hits that can reach the azimuth sector of the block's middle point. Each lane walks
// its own runs and stages (lane, hit) pairs in the wave's list (cheap steps, as many as
// the longest run in the wave); the staged pairs are then sphere-tested densely, one
// per lane, and the survivors kept at the list's front for the distance pass.
template <typename R, int B, int TILE, int COLS, int MODE, bool Y_FIRST, bool COUNT, typename S>
__device__ __forceinline__ void cull_block(const EventLds<R>& L, const R* pts, uint32_t* items, S* slab,
                                           uint32_t* touch, int lane, bool on, int nb, int step0, R r2min, R r2max,
                                           float half_h, bool z_skip, float z_lo, float z_hi, R Kcull, R sqrt_lam,
                                           unsigned long long& w_tests, unsigned long long& w_chords) {
  const int jc = nb / 2;
  // the block's middle point, from this lane's own column
  const R cx = pts[(jc * 3 + 0) * COLS + lane], cy = pts[(jc * 3 + 1) * COLS + lane],
          cz = pts[(jc * 3 + 2) * COLS + lane];
  // radial range of the block's chords (a chord point is within hmax/2 of an endpoint)
  const float rmin = fmaxf((float)fsqrt(r2min) - half_h, 0.0f);
  const float rmax = (float)fsqrt(r2max);
  // clamp in float first: fminf/fmaxf map NaN to the bound, so the index is in range
  const int b_lo = (int)fminf(fmaxf(rmin, 0.0f), (float)(kTabBins - 1));
  const int b_hi = (int)fminf(fmaxf(rmax, 0.0f), (float)(kTabBins - 1));
  const int L0 = L.ltab[b_lo] & 0xff, L1p = L.ltab[b_hi] >> 8;
  const bool z_in = MODE != 0 || COUNT || !z_skip || !((float)cz > z_hi || (float)cz < z_lo);
  const int n_lay = on && z_in ? max(L1p - L0, 0) : 0;
  const float phic = sector_atan2((float)cy, (float)cx);
  int n_items = 0;   // survivors: items[0, n_items)
  int n_stage = 0;   // staged candidates: items[n_items, n_items + n_stage)
  for (int dl = 0; __ballot(dl < n_lay) != 0; ++dl) {
    const bool has = dl < n_lay;
    const int l = has ? L0 + dl : 0;
    const float psic = wrap_pi(phic - L.slope[l] * (float)cz);
    int sect = (int)((psic + kPi) * (kSectors / (2.0f * kPi)));
    sect = sect < 0 ? 0 : (sect > kSectors - 1 ? kSectors - 1 : sect);
    const uint32_t ent = has ? (uint32_t)L.sect[l * kSectors + sect] : 0u;
    const int lb = L.loff[l], nl = L.loff[l + 1] - lb;
    const bool all = ent == kSectAll;
    const int start = all ? 0 : (int)(ent & 511u), cnt = all ? nl : (int)(ent >> 9);
    // the run's first item and the step at which it wraps to the layer's first hit,
    // formed before the loop (so the loop waits on none of the table reads)
    const uint32_t first = ((uint32_t)lane << 16) | (uint32_t)(lb + start);
    const int wrap = nl - start;
    for (int k = 0;; ++k) {
      const bool act = k < cnt;
      const uint64_t m = __ballot(act);
      if (m == 0) break;
      const int off = k < wrap ? k : k - nl;
      if (act) items[n_items + n_stage + lane_rank(m)] = first + (uint32_t)off;
      n_stage += (int)__popcll(m);
      if (n_items + n_stage > kCap - 64) {
        n_items = test_staged<R, COLS, COUNT>(items, n_items, n_items + n_stage, pts, L.hits, jc, Kcull, lane, nb,
                                              w_tests, w_chords);
        n_stage = 0;
        if (n_items > kCap - 64) {
          flush_items<R, B, TILE, COLS, MODE, Y_FIRST>(items, n_items, pts, L.hits, slab, touch, lane, nb, step0,
                                                       sqrt_lam);
          n_items = 0;
        }
      }
    }
  }
  if (n_stage)
    n_items = test_staged<R, COLS, COUNT>(items, n_items, n_items + n_stage, pts, L.hits, jc, Kcull, lane, nb, w_tests,
                                          w_chords);
  if (n_items)
    flush_items<R, B, TILE, COLS, MODE, Y_FIRST>(items, n_items, pts, L.hits, slab, touch, lane, nb, step0, sqrt_lam);
}

// Results of a chunk's lanes from their slab column, read and reset at the marked rows.
// Rows are read U at a time: 1 where other waves hide the reads' latency (and unmarked
// rows are then not read at all), more where the wave is alone.
// MODE 0: score (Eq. 1, FP64), n_in and the chunk's argmin (E, then index).
template <typename R, int TILE, int U, typename S>
__device__ __forceinline__ void finish_scan(const ScanArgs& a, const EventLds<R>& L, S* slab, const uint32_t* touch,
                                            int lane, int nh, int seg, int64_t ch, bool valid) {
  const LaneSlot q = lane_slot(a, seg, ch, lane, nullptr);
  double E = 0.0;
  int cnt = 0;
  for (int i0 = 0; i0 < nh; i0 += U) {
    R m2[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u;
      m2[u] = (R)INFINITY;
      // rows without a mark were not written in this chunk: +inf, nothing to reset
      if (i < nh && (U > 1 || ((touch[i >> 5] >> (i & 31)) & 1u)))
        m2[u] = load_coherent(slab + (size_t)i * TILE + lane);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u;
      if (i >= nh) break;
      if ((touch[i >> 5] >> (i & 31)) & 1u) slab[(size_t)i * TILE + lane] = (R)INFINITY;
      if (valid) {
        const double r = sqrt((double)m2[u]) - (double)L.hits[i].drift;
        const double tq = r * r;
        if (tq < a.lambda) {
          E += tq;
          ++cnt;
        } else {
          E += a.lambda;
        }
      }
    }
  }
  if (!valid) E = INFINITY;
  __threadfence_block();   // the resets land before the next chunk's minima
  long long idx = q.in_tile ? (long long)q.gidx : (long long)0x7fffffffffffffffLL;
  if (q.in_tile) {
    if (a.score) a.score[q.gidx] = E;
    if (a.nin) a.nin[q.gidx] = cnt;
  }
  double be = q.in_tile ? E : INFINITY;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const double oe = __shfl_xor(be, o, 64);
    const long long oi = __shfl_xor(idx, o, 64);
    if (oe < be || (oe == be && oi < idx)) {
      be = oe;
      idx = oi;
    }
  }
  if (lane == 0) {
    a.parts[ch - a.chunk0].e = be;
    a.parts[ch - a.chunk0].idx = idx;
  }
}

// sum + r^2 with the square rounded first, whatever the code around it: Phi of a seed then
// does not depend on the kernel that ran it, and Gauss-Newton compares the Phi of its trials
// with one that another launch may have formed.
__device__ __forceinline__ double add_square(double sum, double r) {
#pragma clang fp contract(off)
  return sum + r * r;
}

// MODE 1: inlier residuals (original hit order) and argmin chords.
template <typename R, int TILE, int U, typename S>
__device__ __forceinline__ void finish_refine(const ScanArgs& a, const EventLds<R>& L, S* slab, const uint32_t* touch,
                                              int lane, int hbase, int nh, int seg, int64_t ch, bool valid) {
  const LaneSlot q = lane_slot(a, seg, ch, lane, nullptr);
  if (q.in_tile) {
    const int64_t base = a.base_of ? a.base_of[q.gidx] : q.gidx;
    uint8_t* mrow = a.mask + (size_t)base * a.max_hits;
    float* rrow = a.resid + (size_t)q.gidx * a.max_hits;
    int32_t* arow = a.argmin_step + (size_t)q.gidx * a.max_hits;
    double ph = 0.0;
    for (int i0 = 0; i0 < nh; i0 += U) {
      unsigned long long key[U];
      int o[U];
      uint8_t set[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u;
        key[u] = 0xffffffffffffffffULL;
        if (i >= nh) continue;
        if (U > 1 || ((touch[i >> 5] >> (i & 31)) & 1u)) key[u] = load_coherent(slab + (size_t)i * TILE + lane);
        o[u] = a.hits_orig[hbase + i];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (i0 + u < nh && !a.define_mask) set[u] = mrow[o[u]];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u;
        if (i >= nh) break;
        if ((touch[i >> 5] >> (i & 31)) & 1u) slab[(size_t)i * TILE + lane] = 0xffffffffffffffffULL;
        // no block came within the cull reach: the distance is beyond it (+inf here)
        const float d2 = key[u] == 0xffffffffffffffffULL ? INFINITY : __uint_as_float((unsigned)(key[u] >> 32));
        const double r = sqrt((double)d2) - (double)L.hits[i].drift;
        bool in;
        if (a.define_mask) {
          in = valid && (r * r < a.lambda);
          mrow[o[u]] = in ? 1 : 0;
        } else {
          in = valid && set[u] != 0;
        }
        rrow[o[u]] = in ? (float)r : NAN;
        arow[o[u]] = (in && key[u] != 0xffffffffffffffffULL) ? (int32_t)(unsigned)(key[u] & 0xffffffffu) : -1;
        if (in) ph = add_square(ph, r);
      }
    }
    for (int i = nh; i < a.max_hits; ++i) {
      if (a.define_mask) mrow[i] = 0;   // the whole row is defined, unused columns 0
      rrow[i] = NAN;
      arow[i] = -1;
    }
    a.phi[q.gidx] = valid ? ph : INFINITY;
  } else {
    for (int i = 0; i < nh; ++i)
      if ((touch[i >> 5] >> (i & 31)) & 1u) slab[(size_t)i * TILE + lane] = 0xffffffffffffffffULL;
  }
  __threadfence_block();
}

// What a workgroup works on (LDS, not registers held across a chunk): a part of event
// `event`, whose chunks end at ge. Its size counts: in the 12- and 16-wave shapes the last
// bytes of LDS decide how many hits an event may have.
struct Work {
  int64_t ge;
  int64_t pos, own_end;      // the workgroup's own place in the chunks: [pos, own_end) is left
  unsigned long long best;   // where chunks are left, while it searches
  int seg, event, hbase, nh;
  bool stage, done, search;
};
// With each wave's chunk and segment: what the shapes' limits leave for it (18 layers: 12
// waves up to 314 hits; 128 bytes more cost four of them).
static_assert(sizeof(Work) + 12 * (sizeof(int64_t) + sizeof(int)) <= 256, "12-wave shape");
static_assert(sizeof(Work) + 16 * (sizeof(int64_t) + sizeof(int)) <= 272, "16-wave shape");

// The last event whose first chunk is at most ch.
__device__ __forceinline__ int find_event(const int64_t* ev_chunk, int n_events, int64_t ch) {
  int lo = 0, hi = n_events;
  while (hi - lo > 1) {
    const int mid = (lo + hi) / 2;
    if (ev_chunk[mid] <= ch)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// Makes chunks [g0, end) of event ev the workgroup's part, one for each wave by its number,
// so that those of a part of few chunks run on different SIMDs; ge: the event's end.
template <int WAVES>
__device__ __forceinline__ void set_part(const ScanArgs& a, Work& sh, int64_t* first, int ev, int64_t g0, int64_t end,
                                         int64_t ge) {
  for (int w = 0; w < WAVES; ++w) first[w] = g0 + w < end ? g0 + w : -1;
  sh.ge = ge;
  sh.seg = find_seg(a.segs, a.n_seg_dev ? *a.n_seg_dev : a.n_seg, g0);
  sh.stage = ev != sh.event;
  sh.event = ev;
  sh.hbase = a.ev_off[ev];
  sh.nh = a.ev_off[ev + 1] - sh.hbase;
  sh.search = sh.done = false;
}

// Takes up to a chunk per wave of event ev; false if none is left.
template <int WAVES>
__device__ __forceinline__ bool take_part(const ScanArgs& a, Work& sh, int64_t* first, int ev) {
  int64_t g0;
  const int64_t ge = event_chunks(a.plan, a.ev_chunk, ev, &g0);
  g0 += (int64_t)atomicAdd(plan_events(a.plan) + ev, (unsigned long long)WAVES);
  if (g0 >= ge) return false;
  set_part<WAVES>(a, sh, first, ev, g0, min(g0 + WAVES, ge), ge);
  return true;
}

// The workgroup's place (thread 0).
__device__ __forceinline__ void start_work(ScanPlan* p, Work& sh) {
  const int64_t n = p->chunk_end - p->chunk0, grid = gridDim.x, b = blockIdx.x;
  sh.event = -1;
  sh.pos = p->len > 0 ? b : p->chunk0 + n * b / grid;
  sh.own_end = p->len > 0 ? min(b + 1, (int64_t)p->n_tiles) : p->chunk0 + n * (b + 1) / grid;
}

// The workgroup's next part of its own (thread 0, between barriers): its tile, or chunks of
// the events from its place on; sh.search if there is none left and it may help elsewhere.
template <int WAVES>
__device__ __forceinline__ void next_part(const ScanArgs& a, Work& sh, int64_t* first) {
  ScanPlan* p = a.plan;
  if (p->len > 0) {
    const int64_t t = sh.pos;
    sh.search = false;
    sh.done = t >= sh.own_end;
    if (sh.done) return;
    sh.pos = sh.own_end;
    const int64_t* tile0 = reinterpret_cast<const int64_t*>(plan_events(p));
    const int ev = find_event(tile0, p->n_events, t);
    int64_t g0;
    const int64_t ge = event_chunks(p, a.ev_chunk, ev, &g0);
    g0 += (t - tile0[ev]) * p->len;
    set_part<WAVES>(a, sh, first, ev, g0, min(g0 + p->len, ge), 0);
    return;
  }
  for (int64_t pos = sh.pos; pos < sh.own_end;) {
    const int ev = find_event(a.ev_chunk, p->n_events, pos);
    pos = a.ev_chunk[ev + 1];
    sh.pos = pos;
    if (take_part<WAVES>(a, sh, first, ev)) return;
  }
  sh.best = 0;
  sh.search = true;
  sh.done = false;
}

// An event with chunks left, by all threads: the most of them, weighted so that workgroups
// that search at the same time do not all go to the same one.
__device__ __forceinline__ void search_events(const ScanArgs& a, Work& sh, int tid, int nthreads) {
  for (int e = tid; e < a.plan->n_events; e += nthreads) {
    int64_t g0;
    const int64_t ge = event_chunks(a.plan, a.ev_chunk, e, &g0);
    const int64_t left = ge - g0 - (int64_t)__hip_atomic_load(plan_events(a.plan) + e, __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_AGENT);
    if (left <= 0) continue;
    const uint32_t weight = 64 + ((blockIdx.x * 37u + (uint32_t)e * 11u) & 63u);
    const uint64_t key = min((uint64_t)left * weight, (uint64_t)0xffffffff);
    atomicMax(&sh.best, key << 32 | (uint32_t)e);
  }
}

// A wave's next chunk (one lane): of the workgroup's event, whose chunks all workgroups
// there share, so that none of their waves waits for another; -1: none is left.
__device__ __forceinline__ int64_t next_chunk(const ScanArgs& a, const Work& sh) {
  if (sh.ge == 0) return -1;   // a tile has no more chunks than waves
  const int64_t ch = max(a.ev_chunk[sh.event], a.plan->chunk0) +
                     (int64_t)atomicAdd(plan_events(a.plan) + sh.event, 1ULL);
  return ch < sh.ge ? ch : -1;
}

// The slab entry that means "no minimum yet".
template <typename S>
__device__ __forceinline__ S slab_empty() {
  if constexpr (std::is_same<S, unsigned long long>::value) {
    return 0xffffffffffffffffULL;
  } else {
    return (S)INFINITY;
  }
}

// Waves per SIMD that scan_kernel's registers must leave room for. The FP32 instances in the
// uniform field come out at 125 to 130 registers; 128 hold a fourth workgroup on a CU
// wherever the LDS does (8 layers, 40 hits, 12^5 seeds: 1.30 ms past 128, 1.16 within;
// adaptive steps, 18 layers, 300 events of 5^5 seeds: 2.63 and 2.21 ms). The others: what a
// workgroup needs.
template <typename R, int FIELD, int B, int WAVES, int MODE, int VAR, bool COUNT>
constexpr int waves_per_simd() {
  const bool four = sizeof(R) == 4 && FIELD == 0 && MODE == 0 && !COUNT && (VAR != 2 || B == 4);
  return four ? 4 : (WAVES + 3) / 4;
}

// VAR 0: fixed steps over the whole path; 1: fixed steps, the track ends with its
// turn partition; 2: adaptive step size (scan mode only), turn_stop as given.
// COUNT: the instance that also counts its work (seed-steps, sphere tests, chord
// distances) into a.work; the timed instances leave it out.
template <typename R, int FIELD, int B, int WAVES, int MODE, int VAR, bool COUNT = false>
__global__ void __launch_bounds__(64 * WAVES, (waves_per_simd<R, FIELD, B, WAVES, MODE, VAR, COUNT>()))
scan_kernel(ScanArgs a) {
  constexpr int TILE = 64 * WAVES;
  // MODE 0: the scan (score E). MODE 1: the refinement forward pass (FP32 only):
  // argmin chords, checkpoints and inlier residuals.
  using Slab = typename std::conditional<MODE == 0, R, unsigned long long>::type;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float2* s_field = reinterpret_cast<float2*>(smem);
  EventLds<R> L;
  L.hits = reinterpret_cast<HitRec<R>*>(smem + a.field_bytes);
  L.ltab = reinterpret_cast<uint16_t*>(smem + a.field_bytes + a.hits_bytes);
  L.sect = reinterpret_cast<uint16_t*>(smem + a.field_bytes + a.hits_bytes + kTabBins * 2);
  R* s_pts = reinterpret_cast<R*>(smem + a.field_bytes + a.hits_bytes + kTabBins * 2 + a.sect_bytes);
  uint32_t* s_items = reinterpret_cast<uint32_t*>(s_pts + WAVES * (B + 1) * 3 * 64);
  // small tables sized by the uploaded event set: layer offsets and twist slopes of
  // the current event, the per-wave row bitmaps
  L.loff = reinterpret_cast<int*>(s_items + WAVES * kCap);
  L.slope = reinterpret_cast<float*>(L.loff + a.n_layers + 1);
  uint32_t* s_touch = reinterpret_cast<uint32_t*>(L.slope + a.n_layers);
  __shared__ Work sh;
  __shared__ int64_t s_chunk[WAVES];
  __shared__ int s_seg[WAVES];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // longest chord: every point of a block's chords lies within B hmax / 2 of its
  // middle point, and every point of a chord within hmax / 2 of one of its ends
  const double hmax = VAR == 2 ? (double)a.h_max : a.h;
  R* pts = s_pts + wave * (B + 1) * 3 * 64;
  uint32_t* items = s_items + wave * kCap;
  Slab* slab = reinterpret_cast<Slab*>(a.mscratch) + (size_t)blockIdx.x * a.slab_stride + wave * 64;
  uint32_t* touch = s_touch + wave * a.touch_words;
  unsigned long long w_steps = 0, w_tests = 0, w_chords = 0;   // COUNT only
  bool filled = false;   // the wave's slab columns hold "no minimum yet" (between chunks)
  const R h = (R)a.h;
  const double lam = a.lambda;
  const float2* nodes = nullptr;
  if constexpr (FIELD == 1) {
    const int nn = (int)padded_field_nodes(a.field.nr, a.field.nz);
    for (int i = tid; i < nn; i += TILE) s_field[i] = a.field.nodes[i];
    nodes = s_field;   // made visible by the barriers before the first chunk
  }

  if (tid == 0) start_work(a.plan, sh);
  for (;;) {
    __syncthreads();   // every wave is done with the part and its tables
    if (tid == 0) next_part<WAVES>(a, sh, s_chunk);
    __syncthreads();
    while (sh.search) {
      search_events(a, sh, tid, TILE);
      __syncthreads();
      if (tid == 0) {
        const unsigned long long best = sh.best;
        sh.best = 0;
        if (best == 0) {
          sh.done = true;
          sh.search = false;
        } else {
          take_part<WAVES>(a, sh, s_chunk, (int)(uint32_t)best);
        }
      }
      __syncthreads();
    }
    if (sh.done) break;
    if (sh.stage) {
      stage_event<R>(a, L, sh.event, tid, TILE, B * hmax);
      __syncthreads();
    }
    for (;;) {
      if (lane == 0 && s_chunk[wave] >= 0)
        s_seg[wave] = find_seg_from(a.segs, a.n_seg_dev ? *a.n_seg_dev : a.n_seg, sh.seg, s_chunk[wave]);
      wave_sync();
      if (s_chunk[wave] < 0) break;
      if (!filled) {
        const int rows = (int)(a.slab_stride / TILE);
        for (int i = 0; i < rows; ++i) slab[(size_t)i * TILE + lane] = slab_empty<Slab>();
        filled = true;
      }
      State<R> st;
      bool valid;
      [[maybe_unused]] LaneSlot q = load_seed<R>(a, s_seg[wave], s_chunk[wave], lane, st, valid);
      Prop<R, FIELD> pr;   // fixed steps: current point and the block's increments
      pr.start(st);
      pr.init_field(st, a.field, nodes);
      for (int i = lane; i < a.touch_words; i += 64) touch[i] = 0u;
      __threadfence_block();
      wave_sync();

      constexpr bool STOP = VAR != 0;    // lanes can end before the last block
      constexpr bool ADAPT = VAR == 2;
      // adaptive: at most 4 L / h_min + 8 trial steps per lane (every rejection at
      // least shortens the step, and h_min steps are always taken)
      const int nblocks = ADAPT ? (int)((4.0 * a.path_len / a.h_min + 8.0 + B - 1) / B) : (a.n_steps + B - 1) / B;
      const R Kcull = (R)(0.5 * B * hmax + sqrt(lam) + (double)kCullMargin);
      const R sqrt_lam = (R)sqrt(lam);
      // beyond these the middle point of a block is out of every wire's reach
      const float z_pad = (float)Kcull + a.ev_maxdrift[sh.event];
      const float z_lo = a.wire_zmin - z_pad, z_hi = a.wire_zmax + z_pad;
      // STOP (a lane's track can end early: at the end of its turn partition, the first
      // step inside r < R0, or with adaptive steps at the end of the path): from then on
      // the lane's state is frozen, so its later chords have zero length at that end
      // point and cannot lower any distance; a block that starts frozen is not culled at
      // all, and a wave whose lanes are all frozen leaves the loop (after writing the
      // frozen state into the checkpoints still ahead, when a tape is recorded)
      const R r0sq = (R)(a.R0 * a.R0);
      const bool stop_turn = VAR == 1 || (ADAPT && a.turn_stop);
      bool live = valid;                          // lanes without a seed have no track to end
      const R far2 = (R)((a.R0 + 1.1 * B * a.h + 1.0) * (a.R0 + 1.1 * B * a.h + 1.0));
      const bool steady = VAR == 1 && steady_lane(a, st.lam);
      R hl = (R)a.h_max, arc = (R)0;              // adaptive: next step and path so far
      const R path = (R)a.path_len;
      for (int blk = 0; blk < nblocks; ++blk) {
        if constexpr (FIELD == 0 && MODE == 0 && VAR == 0 && !COUNT) {
          // in the uniform field T_z is constant: a lane past the chamber and flying on
          // has seen its last wire (0.1 mm: the FP32 rounding of z over a path)
          const bool gone = !valid || ((float)st.z > z_hi + 0.1f && st.tz >= (R)0) ||
                            ((float)st.z < z_lo - 0.1f && st.tz <= (R)0);
          if (__ballot(!gone) == 0) break;
        }
        if constexpr (STOP) {
          if (__ballot(live) == 0) {
            if constexpr (MODE == 1) {
              // the remaining checkpoints hold the frozen state (as if stepped on)
              if (a.tape && q.in_tile)
                for (int step = blk * B; step < a.n_steps; step += B)
                  if (step % a.ckpt == 0) write_tape<R>(a, step, q.gidx, st);
            }
            break;
          }
        }
        const bool live0 = live;
        const int nb = ADAPT ? B : min(B, a.n_steps - blk * B);
        if constexpr (MODE == 1) {
          const int step = blk * B;
          // a checkpoint restarts the adjoint's recompute: the field there is evaluated
          // at the stored state, as the recompute does
          if (a.ckpt > 0 && step % a.ckpt == 0) pr.init_field(st, a.field, nodes);
          if (a.tape && q.in_tile && step % a.ckpt == 0) write_tape<R>(a, step, q.gidx, st);
        }
        R r2min, r2max;
        if constexpr (ADAPT) {
          pts[0 * 64 + lane] = st.x;
          pts[1 * 64 + lane] = st.y;
          pts[2 * 64 + lane] = st.z;
          r2min = r2max = radius2(st.x, st.y);
#pragma unroll
          for (int j = 1; j <= B; ++j) {
            // one trial step; accepted when its error estimate is within the bound
            // (or it is the smallest step), else the lane stays and retries shorter
            if (live) {
              const R hs = hl < path - arc ? hl : path - arc;
              State<R> tr = st;
              R err;
              rkn_step_err<R, FIELD>(tr, a.field, nodes, hs, err);
              const bool acc = err <= (R)a.tol || hs <= (R)a.h_min;
              R g = err > (R)0 ? (R)0.9 * fsqrt(fsqrt((R)a.tol / err)) : (R)4;
              g = g > (R)4 ? (R)4 : (g < (R)0.25 ? (R)0.25 : g);
              if (acc) {
                st = tr;
                arc += hs;
                if (hs == hl) hl *= g;   // a cut last step leaves the step size
                live = arc < path && !(stop_turn && inside_r0(st.x, st.y, r0sq));
              } else {
                hl = hs * (g < (R)1 ? g : (R)1);
              }
              hl = hl > (R)a.h_max ? (R)a.h_max : (hl < (R)a.h_min ? (R)a.h_min : hl);
            }
            pts[(j * 3 + 0) * 64 + lane] = st.x;
            pts[(j * 3 + 1) * 64 + lane] = st.y;
            pts[(j * 3 + 2) * 64 + lane] = st.z;
            const R r2 = radius2(st.x, st.y);
            r2min = vmin(r2min, r2);
            r2max = vmax(r2max, r2);
          }
        } else {
          take_block<R, FIELD, B, 64, VAR>(a, nodes, st, pr, pts, lane, nb, h, r0sq, far2, steady, live, r2min, r2max);
        }
        cull_block<R, B, TILE, 64, MODE, VAR == 2, COUNT>(L, pts, items, slab, touch, lane,
                                                          valid && (!STOP || live0), nb, blk * B, r2min, r2max,
                                                          0.5f * (float)hmax, a.walk, z_lo, z_hi, Kcull, sqrt_lam,
                                                          w_tests, w_chords);
        if constexpr (COUNT) w_steps += (valid && (!STOP || live0)) ? nb : 0;
      }
      // The minima of a seed were folded by lanes of its own wave, and the slab is this
      // workgroup's alone: a workgroup-scope release/acquire (the atomics complete at L2;
      // the reads below bypass L1) orders them before the reads. An agent-scope fence
      // here would write the whole L2's dirty lines back to memory at every chunk.
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
      if constexpr (MODE == 1)
        finish_refine<R, TILE, 1>(a, L, slab, touch, lane, sh.hbase, sh.nh, s_seg[wave], s_chunk[wave], valid);
      else
        finish_scan<R, TILE, 1>(a, L, slab, touch, lane, sh.nh, s_seg[wave], s_chunk[wave], valid);
      if (lane == 0) s_chunk[wave] = next_chunk(a, sh);
    }
  }
  if constexpr (COUNT) {
    atomicAdd(a.work + 0, w_steps);
    atomicAdd(a.work + 1, w_tests);
    atomicAdd(a.work + 2, w_chords);
  }
}

// The same scan for launches of few chunks, where a chunk's 6000 dependent steps and not
// the chip's rate set the time: propagation and culling run side by side. A pair is one
// chunk's producer waves, which only step its seeds and write the points of C blocks per
// phase into one of two LDS buffers, and C consumer waves, which cull and compare one
// block each of the phase before. A workgroup holds a.n_pairs pairs (chunks of any events)
// that share the field map; the producers come first, so that they sit on different SIMDs.
// COLS: columns of the points (seeds of a chunk at most). QUAD: a seed on four lanes, 16
// to a producer (QuadProp).
// Same blocks, lists and arithmetic per chunk as scan_kernel: the same results for a chunk
// of the same seeds (seeds together in other chunks: the last bits, see seg_wire_d2).
//
// What bounds it is the producers' instruction stream: a wave alone on its SIMD issues a
// VALU instruction every 5.6 to 8 cycles. A map step is 138 of them and took 930 cycles on
// one lane per seed, 90 and 650 on four; one wave stepping and culling took 1800. 96 seeds
// of 6000 steps: 4.5 -> 2.3 (7 consumers; 3.7 with 1) -> 1.8 ms on quads; 6^5 FP64 seeds in
// the uniform field 1.07 -> 0.37 ms; the refinement's forward pass over 512 events of 8
// seeds 6.7 -> 3.0 -> 2.2 ms (two pairs per CU, one round instead of two).
template <typename R, int FIELD, int B, int COLS, int MODE, int VAR, bool QUAD>
__global__ void __launch_bounds__(64 * kPipeWaves) pipe_kernel(ScanArgs a) {
  using Slab = typename std::conditional<MODE == 0, R, unsigned long long>::type;
  constexpr int kPts = (B + 1) * 3 * COLS;   // points of one block
  constexpr int NP = QUAD ? COLS / 16 : 1;   // producers of a pair
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ int s_blocks[2][kPipeWaves];    // blocks written in a phase, per producer
  const int C = a.n_con;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_pairs = a.n_pairs, n_prod = n_pairs * NP;
  const bool producer = wave < n_prod;
  const int pair = producer ? wave / NP : (wave - n_prod) / C;
  const int con = producer ? 0 : (wave - n_prod) % C;
  const int sub = producer ? wave % NP : NP + con;   // the wave's number within its pair
  float2* s_field = reinterpret_cast<float2*>(smem);
  unsigned char* mine = smem + a.field_bytes + (size_t)pair * a.pair_bytes;
  EventLds<R> L;
  L.hits = reinterpret_cast<HitRec<R>*>(mine);
  R* s_pts = reinterpret_cast<R*>(mine + a.hits_bytes);
  R* s_r2 = s_pts + 2 * C * kPts;          // per block: r2min (-1: not to be culled), r2max
  L.sect = reinterpret_cast<uint16_t*>(s_r2 + 2 * C * 128);
  L.ltab = reinterpret_cast<uint16_t*>(reinterpret_cast<unsigned char*>(L.sect) + a.sect_bytes);
  uint32_t* items = reinterpret_cast<uint32_t*>(L.ltab + kTabBins) + con * kCap;
  uint32_t* touch = reinterpret_cast<uint32_t*>(L.ltab + kTabBins) + C * kCap;
  L.loff = reinterpret_cast<int*>(touch + a.touch_words);
  L.slope = reinterpret_cast<float*>(L.loff + a.n_layers + 1);
  Slab* slab = reinterpret_cast<Slab*>(a.mscratch) + ((size_t)blockIdx.x * n_pairs + pair) * a.slab_stride;
  const float2* nodes = nullptr;
  if constexpr (FIELD == 1) {
    const int nn = (int)padded_field_nodes(a.field.nr, a.field.nz);
    for (int i = tid; i < nn; i += blockDim.x) s_field[i] = a.field.nodes[i];
    nodes = s_field;   // made visible by the barriers before the first chunk
  }
  const int rows = (int)(a.slab_stride / 64);
  for (int i = sub; i < rows; i += NP + C) slab[(size_t)i * 64 + lane] = slab_empty<Slab>();
  __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): in L2 before another wave's atomics
  const int n_seg = a.n_seg_dev ? *a.n_seg_dev : a.n_seg;
  const int64_t n_chunks = a.n_chunks_dev ? *a.n_chunks_dev : a.n_chunks;
  const R h = (R)a.h;
  const double lam = a.lambda;
  const R Kcull = (R)(0.5 * B * a.h + sqrt(lam) + (double)kCullMargin);
  const R sqrt_lam = (R)sqrt(lam);
  const R r0sq = (R)(a.R0 * a.R0);
  const R far2 = (R)((a.R0 + 1.1 * B * a.h + 1.0) * (a.R0 + 1.1 * B * a.h + 1.0));
  const int nblocks = (a.n_steps + B - 1) / B;
  constexpr bool STOP = VAR != 0;
  int cur_event = -1;
  for (int64_t g = blockIdx.x; g * n_pairs < n_chunks; g += gridDim.x) {
    const bool has = g * n_pairs + pair < n_chunks;
    const int64_t ch = a.chunk0 + min(g * n_pairs + pair, n_chunks - 1);
    const int seg = __builtin_amdgcn_readfirstlane(find_seg(a.segs, n_seg, ch));
    const int ev = a.segs[seg].event;
    const int hbase = a.ev_off[ev];
    const int nh = a.ev_off[ev + 1] - hbase;
    __syncthreads();   // the pair is done with its last chunk's tables
    if (ev != cur_event) stage_event<R>(a, L, ev, sub * 64 + lane, 64 * (NP + C), B * a.h);
    cur_event = ev;
    if (sub == 0)
      for (int i = lane; i < a.touch_words; i += 64) touch[i] = 0u;
    __syncthreads();
    const float z_pad = (float)Kcull + a.ev_maxdrift[ev];
    const float z_lo = a.wire_zmin - z_pad, z_hi = a.wire_zmax + z_pad;
    // blocks written in phase ph, by a producer of this pair or of any; after the barrier
    auto blocks_of_pair = [&](int ph) {
      int m = 0;
      for (int k = 0; k < NP; ++k) m = max(m, s_blocks[ph & 1][pair * NP + k]);
      return __builtin_amdgcn_readfirstlane(m);
    };
    auto any_block = [&](int ph) {
      int m = 0;
      for (int k = 0; k < n_prod; ++k) m |= s_blocks[ph & 1][k];
      return __builtin_amdgcn_readfirstlane(m) != 0;
    };
    if (producer) {
      // the lane's seed (column of the points) and, on quads, its component
      const int sd = QUAD ? sub * 16 + (lane >> 2) : lane;
      const int comp = QUAD ? min(lane & 3, 2) : 0;
      State<R> st;
      bool valid;
      const LaneSlot q = load_seed<R>(a, seg, ch, sd, st, valid);
      valid = valid && has;
      Prop<R, FIELD> pr;
      QuadProp qp;
      const float* qnodes = nullptr;
      if constexpr (QUAD) {
        qp.s = comp == 0 ? st.x : (comp == 1 ? st.y : st.z);
        qp.st = comp == 0 ? st.tx : (comp == 1 ? st.ty : st.tz);
        qp.cs = qp.cst = 0.0f;
        qp.lam = st.lam;
        qp.is_z = comp == 2;
        qnodes = reinterpret_cast<const float*>(nodes) + (comp == 2 ? 1 : 0);
        qp.start();
        qp.init_field(a.field, qnodes);
      } else {
        pr.start(st);
        pr.init_field(st, a.field, nodes);
      }
      bool live = valid;   // as in scan_kernel
      const bool steady = VAR == 1 && steady_lane(a, st.lam);
      [[maybe_unused]] auto tape = [&](int step) {
        if constexpr (QUAD) {
          float* tp = a.tape + (size_t)(step / a.ckpt) * 13 * a.n_pos + q.gidx;
          tp[(size_t)comp * a.n_pos] = qp.s;
          tp[(size_t)(3 + comp) * a.n_pos] = qp.cs;
          tp[(size_t)(6 + comp) * a.n_pos] = qp.st;
          tp[(size_t)(9 + comp) * a.n_pos] = qp.cst;
          if (comp == 0) tp[(size_t)12 * a.n_pos] = qp.lam;
        } else {
          write_tape<R>(a, step, q.gidx, st);
        }
      };
      int blk = 0;
      bool ended = !has;   // the wave's seeds have no block left
      for (int ph = 0;; ++ph) {
        int made = 0;
        for (int c = 0; c < C && blk < nblocks; ++c, ++blk) {
          R* r2 = s_r2 + ((ph & 1) * C + c) * 128;
          if constexpr (STOP) {
            if (!ended && __ballot(live) == 0) {
              ended = true;
              if constexpr (MODE == 1) {
                if (a.tape && q.in_tile)
                  for (int step = blk * B; step < a.n_steps; step += B)
                    if (step % a.ckpt == 0) tape(step);
              }
            }
          }
          if constexpr (FIELD == 0 && MODE == 0 && VAR == 0) {
            const bool gone = !valid || ((float)st.z > z_hi + 0.1f && st.tz >= (R)0) ||
                              ((float)st.z < z_lo - 0.1f && st.tz <= (R)0);
            ended = ended || __ballot(!gone) == 0;
          }
          if (ended) {
            if (NP == 1) {
              blk = nblocks;
              break;
            }
            // another producer of the pair may go on: no block of these seeds there
            r2[sd] = (R)-1;
            continue;
          }
          const bool live0 = live;
          const int nb = min(B, a.n_steps - blk * B);
          if constexpr (MODE == 1) {
            const int step = blk * B;
            if (a.ckpt > 0 && step % a.ckpt == 0) {
              if constexpr (QUAD)
                qp.init_field(a.field, qnodes);
              else
                pr.init_field(st, a.field, nodes);
            }
            if (a.tape && q.in_tile && step % a.ckpt == 0) tape(step);
          }
          R* pts = s_pts + ((ph & 1) * C + c) * kPts;
          R r2min = (R)-1, r2max = (R)-1;
          if constexpr (QUAD) {
            take_block_quad<B, COLS, VAR>(a, qnodes, qp, pts, sd, comp, nb, h, r0sq, far2, steady, live, r2min, r2max);
          } else {
            if (COLS == 64 || lane < COLS)
              take_block<R, FIELD, B, COLS, VAR>(a, nodes, st, pr, pts, lane, nb, h, r0sq, far2, steady, live, r2min,
                                                 r2max);
          }
          r2[sd] = valid && (!STOP || live0) ? r2min : (R)-1;
          r2[64 + sd] = r2max;
          made = c + 1;
        }
        if (lane == 0) s_blocks[ph & 1][wave] = made;
        __syncthreads();
        if (!any_block(ph)) break;
      }
    } else {
      for (int ph = 0;; ++ph) {
        const int prev = (ph & 1) ^ 1;
        if (ph > 0 && con < blocks_of_pair(ph - 1)) {
          const int blk = (ph - 1) * C + con;
          const R* r2 = s_r2 + (prev * C + con) * 128;
          unsigned long long w_tests = 0, w_chords = 0;
          const bool on = (COLS == 64 || lane < COLS) && !(r2[lane] < (R)0);
          cull_block<R, B, 64, COLS, MODE, false, false>(L, s_pts + (prev * C + con) * kPts, items, slab, touch, lane,
                                                         on, min(B, a.n_steps - blk * B), blk * B, r2[lane],
                                                         r2[64 + lane], 0.5f * (float)a.h, a.walk, z_lo, z_hi, Kcull,
                                                         sqrt_lam, w_tests, w_chords);
        }
        __syncthreads();
        if (!any_block(ph)) break;
      }
      __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): the minima are in L2
    }
    __syncthreads();
    if (sub == 0 && has) {
      bool valid;
      {
        State<R> st;
        load_seed<R>(a, seg, ch, lane, st, valid);
      }
      if constexpr (MODE == 1)
        finish_refine<R, 64, 8>(a, L, slab, touch, lane, hbase, nh, seg, ch, valid);
      else
        finish_scan<R, 64, 8>(a, L, slab, touch, lane, nh, seg, ch, valid);
      __builtin_amdgcn_s_waitcnt(0x0f70);   // the resets, before the next chunk's minima
    }
  }
}

__global__ void __launch_bounds__(256)
event_argmin_kernel(const ArgminPart* __restrict__ parts, const int64_t* __restrict__ ev_chunk, int64_t c0, int64_t c1,
                    int64_t* best_i, double* best_e) {
  const int e = blockIdx.x, tid = threadIdx.x;
  const int64_t t0 = max(ev_chunk[e], c0), t1 = min(ev_chunk[e + 1], c1);
  double be = INFINITY;
  long long bi = 0x7fffffffffffffffLL;
  for (int64_t t = t0 + tid; t < t1; t += 256) {
    const ArgminPart p = parts[t - c0];
    if (p.e < be || (p.e == be && p.idx < bi)) {
      be = p.e;
      bi = p.idx;
    }
  }
  __shared__ double se[256];
  __shared__ long long si[256];
  se[tid] = be;
  si[tid] = bi;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (tid < s) {
      const double oe = se[tid + s];
      const long long oi = si[tid + s];
      if (oe < se[tid] || (oe == se[tid] && oi < si[tid])) {
        se[tid] = oe;
        si[tid] = oi;
      }
    }
    __syncthreads();
  }
  if (tid == 0) {
    // the first range of chunks defines the event's best, later ones lower it
    const bool none = t1 <= t0;
    if (c0 == 0 || (!none && (best_i[e] < 0 || se[0] < best_e[e] || (se[0] == best_e[e] && si[0] < best_i[e])))) {
      best_i[e] = none ? -1 : si[0];
      best_e[e] = none ? INFINITY : se[0];
    }
  }
}

// LDS bytes of the layer x sector candidate table (uint16 entries, 256-byte rounded).
static size_t align64(size_t n) { return (n + 63) & ~(size_t)63; }

static size_t sect_table_bytes(const rkn_ctx* c) {
  return align64((size_t)std::max(c->n_layers, 1) * kSectors * sizeof(uint16_t));
}

static int touch_words(const rkn_ctx* c) { return std::max((c->max_hits_event + 31) / 32, 1); }

// LDS regions of one workgroup of scan_kernel<R, FIELD, B, WAVES, ...>, in order:
// field map, hit records, radial table, sector table, points, work lists, layer
// offsets and slopes, row bitmaps.
static size_t field_lds_bytes(const rkn_ctx* c, int field) {
  return field == 1 ? align64(padded_field_nodes(c->nr, c->nz) * sizeof(float2)) : 0;
}
static size_t hits_lds_bytes(const rkn_ctx* c, size_t rsize) {
  return align64((size_t)c->max_hits_event * (rsize == 4 ? sizeof(HitRec<float>) : sizeof(HitRec<double>)));
}
static size_t scan_lds_bytes(const rkn_ctx* c, size_t rsize, int field, int B, int waves) {
  return field_lds_bytes(c, field) + hits_lds_bytes(c, rsize) + kTabBins * 2 + sect_table_bytes(c) +
         (size_t)waves * (B + 1) * 3 * 64 * rsize + (size_t)waves * kCap * 4 +
         (size_t)(2 * std::max(c->n_layers, 1) + 1) * 4 + (size_t)waves * touch_words(c) * 4;
}

// Steps per block; 0 picks the default: 6 for the FP32 field-map path (12-wave
// workgroups, the fastest shape measured on the 512-event batch), else 8.
int resolve_block_steps(const rkn_ctx* c, const rkn_scan_params* p) {
  if (p->block_steps != 0) return p->block_steps;
  return (p->precision == 32 && c->field_kind == 1) ? 6 : 8;
}

// Workgroups of a kernel that one CU holds, from the kernel's register and LDS
// needs (code-object metadata) and the CU's resources on gfx950: 4 SIMDs of 512
// VGPRs per lane (allocated in granules of 8) and at most 8 waves each, and the
// LDS of the device. (This does not use the runtime's occupancy query, whose
// answer for wide workgroups differs between HIP runtime versions.)
static int resident_per_cu(const rkn_ctx* c, const void* kern, int threads, size_t smem) {
  hipFuncAttributes at{};
  if (hipFuncGetAttributes(&at, kern) != hipSuccess) return 0;
  const int waves = (threads + 63) / 64;
  const size_t lds = smem + at.sharedSizeBytes;
  if (lds > (size_t)c->max_lds_block) return 0;
  const int by_lds = lds > 0 ? (int)((size_t)c->max_lds_block / lds) : 32;
  const int regs = at.numRegs > 0 ? ((at.numRegs + 7) / 8) * 8 : 8;
  const int per_simd = std::min(512 / regs, 8);
  const int by_regs = (4 * per_simd) / waves;
  return std::min(by_lds, by_regs);
}

template <typename R, int FIELD, int B, int WAVES>
static bool shape_fits(const rkn_ctx* c) {
  const size_t smem = scan_lds_bytes(c, sizeof(R), FIELD, B, WAVES);
  if (smem + 256 > (size_t)c->max_lds_block) return false;
  // every variant (fixed steps, turn-partition stop, adaptive) must fit the shape
  bool ok = resident_per_cu(c, (const void*)scan_kernel<R, FIELD, B, WAVES, 0, 0>, 64 * WAVES, smem) >= 1 &&
            resident_per_cu(c, (const void*)scan_kernel<R, FIELD, B, WAVES, 0, 1>, 64 * WAVES, smem) >= 1;
  if constexpr (std::is_same<R, float>::value)
    ok = ok && resident_per_cu(c, (const void*)scan_kernel<R, FIELD, B, WAVES, 0, 2>, 64 * WAVES, smem) >= 1;
  return ok;
}

// Waves per workgroup. The FP32 field-map path stages the map in LDS once per
// workgroup, so it uses the widest workgroup that fits: 16 waves with 4-step
// blocks, 12 with 6-step blocks, 8 with 8-step blocks (falling back to 8 waves when
// an event has too many hits, or the runtime reserves too much LDS, for the wider
// shape). Tiles are built for the shape chosen here, and the launch uses the same.
static int scan_waves(const rkn_ctx* c, int precision, int B) {
  if (precision == 64 || c->field_kind == 0) return 4;
  if (B == 4 && shape_fits<float, 1, 4, 16>(c)) return 16;
  if (B == 6 && shape_fits<float, 1, 6, 12>(c)) return 12;
  return 8;
}

// Whether a launch walks its windows in scan order and skips lanes past the wires' z range
// (long: more than one chunk per wave). A launch of one window that fits the chip at once
// gains nothing from either (10 windows of 8^5..12^5 seeds: 0.97-1.02) and keeps the
// grid's order, in which the wave's lists, and with them the rounding of each distance,
// are those of the seeds' own neighbours; so do explicit seeds, whose order is the
// caller's. Decided once for a scan: the parts of one that runs in several launches share
// the windows' chunks, which mean other seeds in the other order.
static int walks(const ScanArgs& a, bool longer) {
  return longer || (!a.seeds5 && (a.n_seg_dev || a.n_seg > 1)) ? 1 : 0;
}

template <typename R, int FIELD, int B, int WAVES, int MODE = 0>
static hipError_t launch_scan_t(rkn_ctx* c, ScanArgs& a, int64_t max_chunks, bool alloc_only, DevBuf* slab_buf,
                                void* raw_slab = nullptr, size_t raw_bytes = 0) {
  constexpr int TILE = 64 * WAVES;
  a.hits_bytes = (int)hits_lds_bytes(c, sizeof(R));
  a.field_bytes = (int)field_lds_bytes(c, FIELD);
  a.sect_bytes = (int)sect_table_bytes(c);
  a.touch_words = touch_words(c);
  const size_t smem = scan_lds_bytes(c, sizeof(R), FIELD, B, WAVES);
  if (smem + 256 > (size_t)c->max_lds_block) return hipErrorInvalidConfiguration;
  auto kern = a.turn_stop ? scan_kernel<R, FIELD, B, WAVES, MODE, 1> : scan_kernel<R, FIELD, B, WAVES, MODE, 0>;
  if constexpr (MODE == 0) {
    if (a.h_max > 0) kern = scan_kernel<R, FIELD, B, WAVES, MODE, 2>;
    if (a.work) kern = scan_kernel<R, FIELD, B, WAVES, MODE, 0, true>;   // fixed steps only (checked by the caller)
  }
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  const int per_cu = resident_per_cu(c, (const void*)kern, TILE, smem);
  if (per_cu < 1) return hipErrorInvalidConfiguration;
  int64_t grid = (int64_t)per_cu * c->n_cu;
  if (a.walk < 0) a.walk = walks(a, max_chunks > grid * WAVES);
  if (grid > max_chunks) grid = max_chunks;
  if (grid < 1) grid = 1;
  a.slab_stride = (int64_t)(c->max_hits_event > 0 ? c->max_hits_event : 1) * TILE;
  const size_t per_wg = (size_t)a.slab_stride * (MODE == 0 ? sizeof(R) : sizeof(unsigned long long));
  if (raw_slab) {
    // caller-provided memory: the persistent grid shrinks to the slabs that fit
    const int64_t fit = (int64_t)(raw_bytes / per_wg);
    if (fit < 1) return hipErrorInvalidValue;
    if (grid > fit) grid = fit;
    a.mscratch = raw_slab;
  } else {
    e = slab_buf->ensure((size_t)grid * per_wg);
    if (e != hipSuccess) return e;
    a.mscratch = slab_buf->p;
  }
  if (alloc_only) return hipSuccess;
  hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(kPlanThreads), 0, c->stream, a, (int)grid, WAVES, c->n_cu);
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(TILE), smem, c->stream, a);
  return hipGetLastError();
}

// LDS of one pair of pipe_kernel<R, ., B, cols, ...> with C consumers.
static size_t pair_lds_bytes(const rkn_ctx* c, size_t rsize, int B, int cols, int C) {
  return align64(hits_lds_bytes(c, rsize) + 2 * (size_t)C * ((size_t)(B + 1) * 3 * cols + 128) * rsize +
                 sect_table_bytes(c) + kTabBins * 2 + (size_t)C * kCap * 4 + (size_t)touch_words(c) * 4 +
                 (size_t)(2 * std::max(c->n_layers, 1) + 1) * 4);
}

// Launches pipe_kernel if the launch suits it (false otherwise): fixed steps, and chunks
// few enough that each CU gets at most as many pairs as its LDS holds; then each pair has
// as many consumers as fit. QUAD: seeds on four lanes, while each producer gets a SIMD of
// its own (two producers on one share its issue slots: 17 000 seeds of one event 2.68 ms
// on one lane each, 2.81 on four). Past that scan_kernel's waves fill the chip and are the faster
// (768 chunks of 64 trials in the field map, two rounds of pairs: Gauss-Newton 43 ms
// against 37), except where an event has at most 16 seeds: its one wave per workgroup
// takes two rounds as well (1000 events of 8 seeds: 10.3 ms against 16.7). No more than four
// pairs of 64 seeds on a CU, so that each producer has a SIMD to itself (70 000 FP64 seeds
// of one event, 40 hits, uniform field, five pairs: 2.79 ms, against 2.56 in scan_kernel).
template <typename R, int FIELD, int B, int COLS, int MODE, bool QUAD = false>
static bool launch_pipe_t(rkn_ctx* c, ScanArgs& a, int64_t max_chunks, bool alloc_only, DevBuf* slab_buf,
                          void* raw_slab, size_t raw_bytes, hipError_t* err) {
  if (a.work || a.h_max > 0 || max_chunks < 1) return false;
  // what scan_kernel's narrowest shape has no room for is refused for any number of seeds
  if (scan_lds_bytes(c, sizeof(R), FIELD, B, sizeof(R) == 8 || FIELD == 0 ? 4 : 8) + 256 > (size_t)c->max_lds_block)
    return false;
  auto kern =
      a.turn_stop ? pipe_kernel<R, FIELD, B, COLS, MODE, 1, QUAD> : pipe_kernel<R, FIELD, B, COLS, MODE, 0, QUAD>;
  constexpr int prod = QUAD ? COLS / 16 : 1;   // producers of a pair
  const size_t field = field_lds_bytes(c, FIELD), room = (size_t)c->max_lds_block - 512;
  auto fits = [&](int64_t pairs, int con) {   // that many pairs of con consumers on one CU
    const size_t pair = pair_lds_bytes(c, sizeof(R), B, COLS, con);
    return FIELD == 1 ? pairs * (prod + con) <= kPipeWaves && field + pairs * pair <= room
                      : prod + con <= kPipeWaves && pairs * (pair + 512) <= room && pairs * (prod + con) <= 16;
  };
  int64_t per_cu = (max_chunks + c->n_cu - 1) / c->n_cu;
  if ((QUAD || COLS == 64) && per_cu * prod > 4) return false;   // a SIMD for each producer
  if (!fits(per_cu, 1)) {
    if (COLS > 16) return false;
    int64_t most = kPipeWaves;
    while (most > 0 && !fits(most, 1)) --most;
    if (per_cu > 2 * most) return false;
    per_cu = most;
  }
  const int n = FIELD == 1 ? (int)per_cu : 1;
  int con = 7, threads = 0, resident = 0;
  size_t pair = 0, smem = 0;
  for (; con >= 1; --con) {
    if (!fits(per_cu, con)) continue;
    pair = pair_lds_bytes(c, sizeof(R), B, COLS, con);
    smem = field + n * pair;
    threads = 64 * n * (prod + con);
    resident = resident_per_cu(c, (const void*)kern, threads, smem);
    if ((int64_t)resident * n >= per_cu) break;
  }
  if (con < 1) return false;
  *err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (*err != hipSuccess) return true;
  const int64_t groups = (max_chunks + n - 1) / n;
  const int64_t grid = std::min(groups, (int64_t)resident * c->n_cu);
  a.field_bytes = (int)field;
  a.hits_bytes = (int)hits_lds_bytes(c, sizeof(R));
  a.sect_bytes = (int)sect_table_bytes(c);
  a.touch_words = touch_words(c);
  a.n_pairs = n;
  a.n_con = con;
  a.pair_bytes = (int)pair;
  a.slab_stride = (int64_t)(c->max_hits_event > 0 ? c->max_hits_event : 1) * 64;
  const size_t bytes = (size_t)grid * n * a.slab_stride * (MODE == 0 ? sizeof(R) : sizeof(unsigned long long));
  if (raw_slab) {
    if (bytes > raw_bytes) return false;
    a.mscratch = raw_slab;
  } else {
    if ((*err = slab_buf->ensure(bytes)) != hipSuccess) return true;
    a.mscratch = slab_buf->p;
  }
  if (a.walk < 0) a.walk = walks(a, false);
  if (alloc_only) return true;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(threads), smem, c->stream, a);
  *err = hipGetLastError();
  return true;
}

int scan_tile(const rkn_ctx* c, const rkn_scan_params* p) {
  return 64 * scan_waves(c, p->precision, p->precision == 64 ? 4 : resolve_block_steps(c, p));
}

static hipError_t dispatch_scan(rkn_ctx* c, const rkn_scan_params* p, ScanArgs& a, int64_t max_chunks,
                                bool alloc_only, DevBuf* slab, void* raw_slab = nullptr, size_t raw_bytes = 0) {
  const int B = resolve_block_steps(c, p);
  hipError_t e = hipSuccess;
  auto pipe = [&](auto launch) { return launch(c, a, max_chunks, alloc_only, slab, raw_slab, raw_bytes, &e); };
  bool done;
  if (p->precision == 64)
    done = c->field_kind == 0 ? pipe(launch_pipe_t<double, 0, 4, 64, 0>) : pipe(launch_pipe_t<double, 1, 4, 64, 0>);
  else if (c->field_kind == 0)
    done = B == 4 ? pipe(launch_pipe_t<float, 0, 4, 64, 0>)
                  : (B == 6 ? pipe(launch_pipe_t<float, 0, 6, 64, 0>) : pipe(launch_pipe_t<float, 0, 8, 64, 0>));
  else
    done = B == 4   ? pipe(launch_pipe_t<float, 1, 4, 64, 0, true>) || pipe(launch_pipe_t<float, 1, 4, 64, 0>)
           : B == 6 ? pipe(launch_pipe_t<float, 1, 6, 64, 0, true>) || pipe(launch_pipe_t<float, 1, 6, 64, 0>)
                    : pipe(launch_pipe_t<float, 1, 8, 64, 0, true>) || pipe(launch_pipe_t<float, 1, 8, 64, 0>);
  if (done) return e;
  if (p->precision == 64)
    return c->field_kind == 0 ? launch_scan_t<double, 0, 4, 4>(c, a, max_chunks, alloc_only, slab, raw_slab, raw_bytes)
                              : launch_scan_t<double, 1, 4, 4>(c, a, max_chunks, alloc_only, slab, raw_slab, raw_bytes);
  if (c->field_kind == 0) {
    if (B == 4) return launch_scan_t<float, 0, 4, 4>(c, a, max_chunks, alloc_only, slab, raw_slab, raw_bytes);
    if (B == 6) return launch_scan_t<float, 0, 6, 4>(c, a, max_chunks, alloc_only, slab, raw_slab, raw_bytes);
    return launch_scan_t<float, 0, 8, 4>(c, a, max_chunks, alloc_only, slab, raw_slab, raw_bytes);
  }
  const int W = scan_waves(c, 32, B);
  if (B == 4)
    return W == 16 ? launch_scan_t<float, 1, 4, 16>(c, a, max_chunks, alloc_only, slab, raw_slab, raw_bytes)
                   : launch_scan_t<float, 1, 4, 8>(c, a, max_chunks, alloc_only, slab, raw_slab, raw_bytes);
  if (B == 6)
    return W == 12 ? launch_scan_t<float, 1, 6, 12>(c, a, max_chunks, alloc_only, slab, raw_slab, raw_bytes)
                   : launch_scan_t<float, 1, 6, 8>(c, a, max_chunks, alloc_only, slab, raw_slab, raw_bytes);
  return launch_scan_t<float, 1, 8, 8>(c, a, max_chunks, alloc_only, slab, raw_slab, raw_bytes);
}

FieldDev field_dev(const rkn_ctx* c) {
  FieldDev f{};
  f.bz = c->bz;
  if (c->field_kind == 1) {
    f.nodes = c->field_nodes.as<float2>();
    f.nr = c->nr;
    f.nz = c->nz;
    f.stride = c->nr + 1;
    f.r0 = c->r0;
    f.z0 = c->z0;
    f.inv_dr = (double)(c->nr - 1) / (c->r1 - c->r0);
    f.inv_dz = (double)(c->nz - 1) / (c->z1 - c->z0);
  }
  return f;
}

// What every scan reads: the field, the prepared hits and the propagation parameters.
static ScanArgs base_args(rkn_ctx* c, const rkn_scan_params* p, const ScanSegs& w) {
  ScanArgs a{};
  a.field = field_dev(c);
  a.hits32 = c->hits32.as<HitRec<float>>();
  a.hits64 = c->hits64.as<HitRec<double>>();
  a.ev_off = c->ev_off.as<int32_t>();
  a.layer_off = c->layer_off.as<int32_t>();
  a.layer_r = c->layer_r.as<float2>();
  a.ev_maxdrift = c->ev_maxdrift.as<float>();
  a.hits_phi = c->hits_phi.as<float>();
  a.layer_twist = c->layer_ext.as<float2>();
  a.n_layers = c->n_layers;
  a.wire_zmin = c->wire_zmin;
  a.wire_zmax = c->wire_zmax;
  a.b_max = c->b_max;
  a.segs = w.segs;
  a.n_seg = w.n_seg;
  a.n_seg_dev = w.n_seg_dev;
  a.ev_chunk = w.ev_chunk;
  a.n_events = c->n_events;
  a.chunk0 = w.chunk0;
  a.n_chunks = w.n_chunks;
  a.n_chunks_dev = w.n_chunks_dev;
  a.walk = -1;
  a.windows = w.windows;
  a.seeds5 = w.seeds5;
  a.perm = w.perm;
  a.R0 = p->R0;
  a.charge = p->charge;
  a.h = p->step_mm;
  a.lambda = p->lambda_mm2;
  a.n_steps = p->n_steps;
  a.turn_stop = p->turn_stop;
  return a;
}

// Refinement forward pass over explicit seeds (FP32, block of 8 steps).
hipError_t launch_refine_fwd(rkn_ctx* c, const rkn_scan_params* p, const ScanSegs& w, const int64_t* d_base_of,
                             uint8_t* d_mask, int define_mask, float* d_resid, int32_t* d_argmin, double* d_phi,
                             float* d_tape, int ckpt, int n_ckpt, int64_t n_pos) {
  hipError_t e = c->r_counter.ensure(scan_plan_bytes(c));
  if (e != hipSuccess) return e;
  ScanArgs a = base_args(c, p, w);
  a.plan = c->r_counter.as<ScanPlan>();
  a.hits_orig = c->hits_orig.as<int32_t>();
  a.base_of = d_base_of;
  a.mask = d_mask;
  a.define_mask = define_mask;
  a.resid = d_resid;
  a.argmin_step = d_argmin;
  a.phi = d_phi;
  a.tape = d_tape;
  a.ckpt = ckpt;
  a.n_ckpt = n_ckpt;
  a.n_pos = n_pos;
  a.max_hits = c->max_hits_event > 0 ? c->max_hits_event : 1;
  if (w.n_chunks == 0) return hipSuccess;
  static_assert(kRefineBlock == 8, "the refinement pass runs 8-step blocks");
  auto pipe = [&](auto launch) { return launch(c, a, w.n_chunks, false, &c->r_slab, nullptr, (size_t)0, &e); };
  // few seeds per event (trials: 6 per seed): narrower points leave LDS for more pairs
  bool done;
  if (c->field_kind == 0)
    done = pipe(launch_pipe_t<float, 0, 8, 64, 1>);
  else if (w.max_lanes <= 16)
    done = pipe(launch_pipe_t<float, 1, 8, 16, 1, true>) || pipe(launch_pipe_t<float, 1, 8, 16, 1>);
  else if (w.max_lanes <= 48)
    done = pipe(launch_pipe_t<float, 1, 8, 48, 1, true>) || pipe(launch_pipe_t<float, 1, 8, 48, 1>);
  else
    done = pipe(launch_pipe_t<float, 1, 8, 64, 1, true>) || pipe(launch_pipe_t<float, 1, 8, 64, 1>);
  if (done) return e;
  return c->field_kind == 0 ? launch_scan_t<float, 0, 8, 4, 1>(c, a, w.n_chunks, false, &c->r_slab)
                            : launch_scan_t<float, 1, 8, 8, 1>(c, a, w.n_chunks, false, &c->r_slab);
}

static ScanArgs scan_args(rkn_ctx* c, const rkn_scan_params* p, const ScanSegs& w, double* d_score, int32_t* d_nin,
                          ArgminPart* parts, void* plan) {
  ScanArgs a = base_args(c, p, w);
  a.plan = static_cast<ScanPlan*>(plan);
  a.score = d_score;
  if (c->adapt) {   // set only for the adaptive scan entry point's call
    a.path_len = p->n_steps * p->step_mm;
    a.tol = (float)c->adapt->tol_mm;
    a.h_min = (float)c->adapt->h_min_mm;
    a.h_max = (float)c->adapt->h_max_mm;
  }
  a.nin = d_nin;
  a.parts = parts;
  a.work = c->count_work;
  return a;
}

static hipError_t launch_event_argmin(rkn_ctx* c, const ScanSegs& w, const ArgminPart* parts, int64_t c0, int64_t c1,
                                      int64_t* d_best_i, double* d_best_e) {
  if (c->n_events > 0)
    hipLaunchKernelGGL(event_argmin_kernel, dim3(c->n_events), dim3(256), 0, c->stream, parts, w.ev_chunk, c0, c1,
                       d_best_i, d_best_e);
  return hipGetLastError();
}

hipError_t launch_scan(rkn_ctx* c, const rkn_scan_params* p, const ScanSegs& w, double* d_score, int32_t* d_nin,
                       int64_t* d_best_i, double* d_best_e) {
  hipError_t e = c->parts.ensure(sizeof(ArgminPart) * (size_t)(w.n_chunks > 0 ? w.n_chunks : 1));
  if (e != hipSuccess) return e;
  e = c->counter.ensure(scan_plan_bytes(c));
  if (e != hipSuccess) return e;
  ScanArgs a = scan_args(c, p, w, d_score, d_nin, c->parts.as<ArgminPart>(), c->counter.p);
  if (w.n_chunks > 0) {
    e = dispatch_scan(c, p, a, w.n_chunks, false, &c->mscratch);
    if (e != hipSuccess) return e;
  }
  return launch_event_argmin(c, w, c->parts.as<ArgminPart>(), 0, w.n_chunks, d_best_i, d_best_e);
}

hipError_t launch_scan_dev(rkn_ctx* c, const rkn_scan_params* p, const ScanSegs& w, double* d_score, int32_t* d_nin,
                           int64_t* d_best_i, double* d_best_e, bool alloc_only, const ScanScratch* scratch) {
  const ScanScratch own{&c->b_parts, &c->b_counter, &c->b_slab};
  const ScanScratch& s = scratch ? *scratch : own;
  hipError_t e = s.parts->ensure(sizeof(ArgminPart) * (size_t)(w.n_chunks > 0 ? w.n_chunks : 1));
  if (e != hipSuccess) return e;
  e = s.counter->ensure(scan_plan_bytes(c));
  if (e != hipSuccess) return e;
  ScanArgs a = scan_args(c, p, w, d_score, d_nin, s.parts->as<ArgminPart>(), s.counter->p);
  e = dispatch_scan(c, p, a, w.n_chunks, alloc_only, s.slab);
  if (e != hipSuccess || alloc_only) return e;
  return launch_event_argmin(c, w, s.parts->as<ArgminPart>(), 0, w.n_chunks, d_best_i, d_best_e);
}

hipError_t launch_scan_raw(rkn_ctx* c, const rkn_scan_params* p, const ScanSegs& w, double* d_score, int32_t* d_nin,
                           int64_t* d_best_i, double* d_best_e, ArgminPart* d_parts, int64_t max_parts,
                           void* d_plan, void* d_slab, size_t slab_bytes) {
  // as many launches as the argmin partials need; each lowers the events' best, and all
  // walk the windows as one launch of the whole scan would
  int walk = -1;
  if (w.n_chunks > max_parts) {
    ScanArgs whole = scan_args(c, p, w, d_score, d_nin, d_parts, d_plan);
    const hipError_t e = dispatch_scan(c, p, whole, w.n_chunks, true, nullptr, d_slab, slab_bytes);
    if (e != hipSuccess) return e;
    walk = whole.walk;
  }
  for (int64_t c0 = 0; c0 < w.n_chunks || c0 == 0; c0 += max_parts) {
    ScanSegs part = w;
    part.chunk0 = c0;
    part.n_chunks = std::min(max_parts, w.n_chunks - c0);
    ScanArgs a = scan_args(c, p, part, d_score, d_nin, d_parts, d_plan);
    a.walk = walk;
    if (part.n_chunks > 0) {
      const hipError_t e = dispatch_scan(c, p, a, part.n_chunks, false, nullptr, d_slab, slab_bytes);
      if (e != hipSuccess) return e;
    }
    const hipError_t e = launch_event_argmin(c, w, d_parts, c0, c0 + part.n_chunks, d_best_i, d_best_e);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

size_t scan_plan_bytes(const rkn_ctx* c) {
  return kPlanHead + sizeof(int64_t) * ((size_t)c->n_events + 1);
}

size_t scan_slab_bytes_per_workgroup(const rkn_ctx* c, const rkn_scan_params* p) {
  const size_t elem = p->precision == 64 ? sizeof(double) : sizeof(float);
  return (size_t)(c->max_hits_event > 0 ? c->max_hits_event : 1) * (size_t)scan_tile(c, p) * elem;
}

// ---------------------------------------------------------------------------------
template <typename R, int FIELD>
__global__ void __launch_bounds__(256)
trace_kernel(FieldDev f, double R0, double charge, double hstep, int turn_stop, int64_t n_seeds,
             const double* __restrict__ seeds, int n_sel, const int32_t* __restrict__ steps,
             double* __restrict__ out) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n_seeds) return;
  const double* v = seeds + 5 * s;
  const double pm = sqrt(v[2] * v[2] + v[3] * v[3] + v[4] * v[4]);
  double* o = out + (size_t)s * n_sel * 6;
  if (!(pm >= 1e-3)) {
    for (int k = 0; k < 6 * n_sel; ++k) o[k] = NAN;
    return;
  }
  State<R> st;
  st.x = (R)(R0 * cos(v[0]));
  st.y = (R)(R0 * sin(v[0]));
  st.z = (R)v[1];
  st.tx = (R)(v[2] / pm);
  st.ty = (R)(v[3] / pm);
  st.tz = (R)(v[4] / pm);
  st.lam = (R)(kKappa * charge / pm);
  st.cx = st.cy = st.cz = (R)0;
  st.ctx = st.cty = st.ctz = (R)0;
  const R h = (R)hstep;
  const R r0sq = (R)(R0 * R0);
  int n = 0;
  bool live = true;   // with turn_stop, states after the end of the turn partition stay
  Prop<R, FIELD> pr;  // the scan's propagation, folded every kTraceFold steps
  pr.start(st);
  pr.init_field(st, f, f.nodes);
  for (int k = 0; k < n_sel; ++k) {
    const int target = steps[k];
    for (; n < target && live; ++n) {
      pr.step(st, f, f.nodes, h);
      live = !(turn_stop && inside_r0(pr.px, pr.py, r0sq));
      if ((n + 1) % kTraceFold == 0) pr.fold(st);
    }
    o[6 * k + 0] = (double)pr.px;
    o[6 * k + 1] = (double)pr.py;
    o[6 * k + 2] = (double)pr.pz;
    o[6 * k + 3] = (double)pr.tx;
    o[6 * k + 4] = (double)pr.ty;
    o[6 * k + 5] = (double)pr.tz;
  }
}

hipError_t launch_trace(rkn_ctx* c, const rkn_scan_params* p, int64_t n_seeds, const double* d_seeds,
                        int32_t n_sel, const int32_t* d_steps, double* d_states) {
  const FieldDev f = field_dev(c);
  const dim3 grid((unsigned)((n_seeds + 255) / 256)), block(256);
  if (n_seeds == 0) return hipSuccess;
  if (p->precision == 64) {
    if (c->field_kind == 0)
      hipLaunchKernelGGL((trace_kernel<double, 0>), grid, block, 0, c->stream, f, p->R0, p->charge,
                         p->step_mm, p->turn_stop, n_seeds, d_seeds, n_sel, d_steps, d_states);
    else
      hipLaunchKernelGGL((trace_kernel<double, 1>), grid, block, 0, c->stream, f, p->R0, p->charge,
                         p->step_mm, p->turn_stop, n_seeds, d_seeds, n_sel, d_steps, d_states);
  } else {
    if (c->field_kind == 0)
      hipLaunchKernelGGL((trace_kernel<float, 0>), grid, block, 0, c->stream, f, p->R0, p->charge,
                         p->step_mm, p->turn_stop, n_seeds, d_seeds, n_sel, d_steps, d_states);
    else
      hipLaunchKernelGGL((trace_kernel<float, 1>), grid, block, 0, c->stream, f, p->R0, p->charge,
                         p->step_mm, p->turn_stop, n_seeds, d_seeds, n_sel, d_steps, d_states);
  }
  return hipGetLastError();
}

}  // namespace rkn
