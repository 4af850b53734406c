// Circle Hough transform over the hit wires and the seed window of each peak
// (Yeo et al., CTD/WIT 2019, section 2.1 and Fig. 4), for gfx950.
//
//  vote:   one lane per centre cell, 256 cells per workgroup; the event's hits
//          (wire waists quantised to 2^-8 mm) sit in LDS; the radius bin is an FP32
//          estimate, decided by exact edge comparisons (FP64 on integers < 2^53) where
//          it lies within its own error of an edge; counts go to 16-bit LDS counters
//          (an event has at most 512 hits) and out as planes [radius][cell], and the
//          workgroup's maximum is kept and folded into the event maximum with an
//          integer atomic max (order-free).
//  peaks:  one workgroup per 256 cells, which ends at once if their maximum lies below
//          max(min_votes, ceil(max/2)); bins at or above that test their 26 neighbours
//          and survivors are appended to a per-event list (4096 entries; an event with
//          more peaks is resolved by the select stage).
//  select: one workgroup per event keeps the max_cand best (count desc, flat asc)
//          and turns each into a window (FP64 geometry, integer counts); when the
//          list overflowed it walks the whole accumulator with the peak rule, so the
//          choice never depends on the order of the list's appends.
#include <math.h>

#include <algorithm>
#include <string>
#include <vector>

#include "internal.hpp"

namespace rkn {

constexpr int kHoughCells = 256;
constexpr int kMaxNr = 64;
constexpr int kCandCap = 4096;
constexpr int kEventChunk = 64;   // 540 MB of 256 x 256 x 64 bins; 16 or 32 leave the selection more often alone

// One event's counts: planes [n_r][cell_stride], the stride a multiple of 8 bins, then
// the maximum of each vote workgroup.
__host__ __device__ inline long long cell_stride(const HoughDev& hp) {
  return ((long long)hp.n_xy * hp.n_xy + 7) / 8 * 8;
}
__host__ __device__ inline int vote_blocks(const HoughDev& hp) {
  return (hp.n_xy * hp.n_xy + kHoughCells - 1) / kHoughCells;
}
__host__ __device__ inline long long event_stride(const HoughDev& hp) {
  return hp.n_r * cell_stride(hp) + (vote_blocks(hp) + 7) / 8 * 8;
}
__device__ __forceinline__ long long bin_at(const HoughDev& hp, int a, int b, int k) {
  return k * cell_stride(hp) + (long long)a * hp.n_xy + b;
}
// The order of bins in all outputs: flat = (a n_xy + b) n_r + k.
__device__ __forceinline__ long long flat_of(const HoughDev& hp, int a, int b, int k) {
  return ((long long)a * hp.n_xy + b) * hp.n_r + k;
}

// Bound by VALU: about 16 operations per (cell, hit), 630 M of them for 64 events of 150
// hits on 256 x 256 cells. Bins are found as k = floor((rho - r_min) / w), rho from FP32
// squares. Its operands are exact (integers < 2^24; a hit further than that, 32 m, lies
// outside every radius either way), so that the bin's real-valued coordinate carries at most
// delta = 2^-21 r_max / w + 2^-22 n_r of rounding; within delta of an edge the exact
// squares decide. 64 events: 370 us. (FP64 squares for every hit and 16-bit counters read
// and written back by their lane, counts out as 32 bits [cell][radius]: 950 us.)
// A counter word holds cells t and t + 128, so the lanes of a wave hit different banks.
__global__ void __launch_bounds__(kHoughCells)
hough_vote_kernel(HoughDev hp, int max_hits, const int32_t* __restrict__ ev_off, const int32_t* __restrict__ wire_id,
                  const double* __restrict__ wx, const double* __restrict__ wy, int ev0,
                  unsigned short* __restrict__ acc, uint32_t* __restrict__ ev_max) {
  constexpr int kHalf = kHoughCells / 2;
  extern __shared__ float2 s_hit[];                                            // [max_hits, even]
  uint32_t* s_cnt = reinterpret_cast<uint32_t*>(s_hit + ((max_hits + 1) & ~1));   // [n_r][kHalf]
  __shared__ double s_edge[kMaxNr + 1];
  __shared__ unsigned int s_max;
  const int e = ev0 + blockIdx.y, tid = threadIdx.x;
  const int base = ev_off[e], nh = ev_off[e + 1] - base;
  for (int i = tid; i < nh; i += kHoughCells) {
    const int w = wire_id[base + i];
    s_hit[i] = make_float2((float)(2.0 * rint(wx[w] * 256.0)), (float)(2.0 * rint(wy[w] * 256.0)));   // half to even
  }
  for (int k = tid; k <= hp.n_r; k += kHoughCells) {
    const double rk = (double)hp.rmin_q + (double)hp.wr_q * k;
    s_edge[k] = 4.0 * rk * rk;
  }
  for (int i = tid; i < hp.n_r * kHalf; i += kHoughCells) s_cnt[i] = 0u;
  if (tid == 0) s_max = 0u;
  __syncthreads();
  const int ncell = hp.n_xy * hp.n_xy;
  const int cell0 = (int)blockIdx.x * kHoughCells, cell = cell0 + tid;
  if (cell < ncell) {
    const int a = cell / hp.n_xy, b = cell - a * hp.n_xy;
    const float xc2 = (float)(-2 * hp.half_q + hp.wxy_q * (2 * a + 1));   // twice the centre, exact
    const float yc2 = (float)(-2 * hp.half_q + hp.wxy_q * (2 * b + 1));
    const float inv2w = 1.0f / (2.0f * (float)hp.wr_q);
    const float k_off = -2.0f * (float)hp.rmin_q * inv2w;
    const float delta = 0x1p-21f * ((float)hp.n_r - k_off) + 0x1p-22f * (float)hp.n_r;
    const float mid = 0.5f - delta;
    const unsigned one = tid < kHalf ? 1u : 0x10000u;
    uint32_t* col = s_cnt + (tid & (kHalf - 1));
#pragma unroll 4
    for (int i = 0; i < nh; ++i) {
      const float2 h = s_hit[i];
      const float dx = h.x - xc2, dy = h.y - yc2;
      const float kf = __builtin_fmaf(__builtin_amdgcn_sqrtf(__builtin_fmaf(dx, dx, dy * dy)), inv2w, k_off);
      const float kl = floorf(kf);
      int k = (int)kl;
      if (fabsf((kf - kl) - 0.5f) > mid) {
        const double ex = (double)dx, ey = (double)dy, rho2 = ex * ex + ey * ey;   // 4 rho^2, exact
        if (rho2 < s_edge[0] || rho2 >= s_edge[hp.n_r]) continue;
        k = k < 0 ? 0 : (k > hp.n_r - 1 ? hp.n_r - 1 : k);
        while (k > 0 && rho2 < s_edge[k]) --k;
        while (k < hp.n_r - 1 && rho2 >= s_edge[k + 1]) ++k;
      }
      if ((unsigned)k < (unsigned)hp.n_r) atomicAdd(col + k * kHalf, one);
    }
  }
  __syncthreads();
  // planes out, two cells a thread: words 2 j and 2 j + 1 hold the pair in their low
  // halves (cells below 128) or high halves
  const long long cs = cell_stride(hp);
  unsigned short* A = acc + (size_t)blockIdx.y * event_stride(hp);
  unsigned short* out = A + cell0;
  const int j = tid & (kHalf / 2 - 1), hi = (tid >> 6) & 1;
  const int c = hi * kHalf + 2 * j;
  unsigned mymax = 0u;
  for (int k = tid >> 7; k < hp.n_r; k += 2) {
    const uint2 w = *reinterpret_cast<const uint2*>(s_cnt + k * kHalf + 2 * j);
    const unsigned v0 = hi ? w.x >> 16 : w.x & 0xffffu, v1 = hi ? w.y >> 16 : w.y & 0xffffu;
    if (cell0 + c < cs) *reinterpret_cast<uint32_t*>(out + k * cs + c) = v0 | v1 << 16;   // cs is even
    mymax = max(mymax, max(v0, v1));
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) mymax = max(mymax, (unsigned)__shfl_xor((int)mymax, o, 64));
  if ((tid & 63) == 0) atomicMax(&s_max, mymax);
  __syncthreads();
  if (tid == 0) {
    A[hp.n_r * cs + blockIdx.x] = (unsigned short)s_max;
    atomicMax(ev_max + e, s_max);
  }
}

// Event maxima and candidate counts of n events to zero.
__global__ void hough_zero_kernel(uint32_t* p, uint32_t* q, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = q[i] = 0u;
}

// One event's counts in the order of the outputs: 32 bits, [cell][radius]. Bound by memory:
// planes in and bins out, both in whole lines by way of LDS. 2048^2 x 64 bins: 2.3 ms with
// each bin read from its plane by itself, now 0.73 (with the vote).
__global__ void __launch_bounds__(kHoughCells)
hough_unpack_kernel(HoughDev hp, const unsigned short* __restrict__ acc, uint32_t* __restrict__ out) {
  __shared__ unsigned short s_plane[kMaxNr][kHoughCells + 2];
  const int tid = threadIdx.x, cell0 = (int)blockIdx.x * kHoughCells;
  const int n = min(kHoughCells, hp.n_xy * hp.n_xy - cell0);
  if (tid < n) {
#pragma unroll 8
    for (int k = 0; k < hp.n_r; ++k) s_plane[k][tid] = acc[k * cell_stride(hp) + cell0 + tid];
  }
  __syncthreads();
  uint32_t* o = out + (size_t)cell0 * hp.n_r;
  for (int i = tid; i < n * hp.n_r; i += kHoughCells) o[i] = s_plane[i % hp.n_r][i / hp.n_r];
}

// Peak rule: the bin's count reaches the event's threshold, is >= all 26
// neighbours and > the neighbours with a smaller flat index.
__device__ __forceinline__ uint32_t peak_threshold(const HoughDev& hp, uint32_t ev_max) {
  uint32_t thr = (ev_max + 1u) / 2u;
  if (thr < (uint32_t)hp.min_votes) thr = (uint32_t)hp.min_votes;
  return thr < 1u ? 1u : thr;
}

__device__ __forceinline__ bool beats_neighbours(const HoughDev& hp, const unsigned short* A, int a, int b, int k,
                                                 uint32_t c) {
  const long long v = flat_of(hp, a, b, k);
  bool ok = true;   // no early exit: the 26 loads are in flight together
#pragma unroll
  for (int da = -1; da <= 1; ++da)
#pragma unroll
    for (int db = -1; db <= 1; ++db)
#pragma unroll
      for (int dk = -1; dk <= 1; ++dk) {
        if (!da && !db && !dk) continue;
        const int aa = a + da, bb = b + db, kk = k + dk;
        const bool in = aa >= 0 && bb >= 0 && kk >= 0 && aa < hp.n_xy && bb < hp.n_xy && kk < hp.n_r;
        const uint32_t o = A[in ? bin_at(hp, aa, bb, kk) : bin_at(hp, a, b, k)];
        ok &= !(in && (o > c || (o == c && flat_of(hp, aa, bb, kk) < v)));
      }
  return ok;
}

// Bound by latency: few of an event's workgroups hold a bin that reaches the threshold.
// Those read their 32 KB of counts, 16 bytes a lane, list the bins that reach it, and test
// one bin a lane: 106 us for 64 events. (32-bit counts, every bin read by a lane: 510 us;
// 16-bit ones, 8 a lane: 229; the bins of the few workgroups tested where they lie: 170.)
__global__ void __launch_bounds__(256)
hough_peaks_kernel(HoughDev hp, const unsigned short* __restrict__ acc, const uint32_t* __restrict__ ev_max,
                   int ev0, uint32_t* __restrict__ cand_n, uint2* __restrict__ cand) {
  __shared__ unsigned short s_bin[kMaxNr * kHoughCells];   // k * 256 + cell in the workgroup
  __shared__ int s_n;
  const int e = ev0 + blockIdx.y, tid = threadIdx.x;
  const long long cs = cell_stride(hp);
  const unsigned short* A = acc + (size_t)blockIdx.y * event_stride(hp);
  const uint32_t top_here = A[hp.n_r * cs + blockIdx.x], thr = peak_threshold(hp, ev_max[e]);
  if (top_here < thr) return;   // thr >= 1: padding cells never pass below either
  if (tid == 0) s_n = 0;
  __syncthreads();
  const int cell0 = (int)blockIdx.x * kHoughCells, own = (tid & 31) * 8;
  if (cell0 + own < cs) {
#pragma unroll 8
    for (int k = tid >> 5; k < hp.n_r; k += 8) {
      const uint4 q = *reinterpret_cast<const uint4*>(A + k * cs + cell0 + own);
      const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if ((i & 1 ? w[i / 2] >> 16 : w[i / 2] & 0xffffu) >= thr)
          s_bin[atomicAdd(&s_n, 1)] = (unsigned short)(k * kHoughCells + own + i);
    }
  }
  __syncthreads();
  for (int i = tid; i < s_n; i += 256) {
    const int k = s_bin[i] / kHoughCells, cell = cell0 + s_bin[i] % kHoughCells;
    const int a = cell / hp.n_xy, b = cell - a * hp.n_xy;
    const uint32_t c = A[bin_at(hp, a, b, k)];
    if (!beats_neighbours(hp, A, a, b, k, c)) continue;
    const uint32_t slot = atomicAdd(cand_n + e, 1u);
    if (slot < (uint32_t)kCandCap) cand[(size_t)e * kCandCap + slot] = make_uint2(c, (uint32_t)flat_of(hp, a, b, k));
  }
}

__device__ int half_max_extent(const HoughDev& hp, const unsigned short* A, int a, int b, int k, int axis) {
  const uint32_t c = A[bin_at(hp, a, b, k)];
  const int lim = axis == 2 ? hp.n_r : hp.n_xy;
  int n = 1;
  for (int dir = -1; dir <= 1; dir += 2) {
    for (int step = 1;; ++step) {
      int aa = a, bb = b, kk = k;
      if (axis == 0) aa += dir * step;
      if (axis == 1) bb += dir * step;
      if (axis == 2) kk += dir * step;
      const int pos = axis == 0 ? aa : (axis == 1 ? bb : kk);
      if (pos < 0 || pos >= lim) break;
      if (2u * A[bin_at(hp, aa, bb, kk)] < c) break;
      ++n;
    }
  }
  return n;
}

__global__ void __launch_bounds__(256)
hough_select_kernel(HoughDev hp, const unsigned short* __restrict__ acc, const uint32_t* __restrict__ ev_max, int ev0,
                    const uint32_t* __restrict__ cand_n, const uint2* __restrict__ cand,
                    WinSlot* __restrict__ slots, int32_t* __restrict__ n_valid) {
  __shared__ uint2 s_best[kMaxCand];
  __shared__ uint2 s_red[2][4];
  __shared__ int s_nsel;
  const int e = ev0 + blockIdx.x, tid = threadIdx.x;
  const unsigned short* A = acc + (size_t)blockIdx.x * event_stride(hp);
  // More peaks than the list holds: which ones the list kept depends on the order
  // of the appends, so the selection then walks the whole accumulator with the
  // peak rule instead (slower, same result as an unbounded list).
  const bool overflow = cand_n[e] > (uint32_t)kCandCap;
  const uint32_t thr = peak_threshold(hp, ev_max[e]);
  const int n = (int)min(cand_n[e], (uint32_t)kCandCap);
  const uint2* L = cand + (size_t)e * kCandCap;
  // repeated selection of the best remaining (count desc, flat asc)
  uint2 prev = make_uint2(0xffffffffu, 0u);   // strictly "worse than" this bound
  int nsel = 0;
  for (int j = 0; j < hp.max_cand && (overflow || j < n); ++j) {
    uint2 best = make_uint2(0u, 0xffffffffu);
    bool have = false;
    if (!overflow) {
      for (int i = tid; i < n; i += 256) {
        const uint2 x = L[i];
        const bool after_prev = x.x < prev.x || (x.x == prev.x && x.y > prev.y);
        if (!after_prev) continue;
        if (!have || x.x > best.x || (x.x == best.x && x.y < best.y)) {
          best = x;
          have = true;
        }
      }
    } else {
      const long long nbins = (long long)hp.n_xy * hp.n_xy * hp.n_r;
      for (long long v = tid; v < nbins; v += 256) {
        const int k = (int)(v / ((long long)hp.n_xy * hp.n_xy)), cell = (int)(v % ((long long)hp.n_xy * hp.n_xy));
        const int a = cell / hp.n_xy, b = cell - a * hp.n_xy;
        const uint32_t cnt = A[bin_at(hp, a, b, k)];
        if (cnt < thr) continue;
        const uint2 x = make_uint2(cnt, (uint32_t)flat_of(hp, a, b, k));
        const bool after_prev = x.x < prev.x || (x.x == prev.x && x.y > prev.y);
        if (!after_prev) continue;
        if (have && !(x.x > best.x || (x.x == best.x && x.y < best.y))) continue;
        if (!beats_neighbours(hp, A, a, b, k, cnt)) continue;
        best = x;
        have = true;
      }
    }
    auto better = [](uint2 o, uint2 m) { return o.x > m.x || (o.x == m.x && o.y < m.y); };
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
      const uint2 o = make_uint2((uint32_t)__shfl_xor((int)best.x, s, 64), (uint32_t)__shfl_xor((int)best.y, s, 64));
      if (better(o, best)) best = o;
    }
    if ((tid & 63) == 0) s_red[j & 1][tid >> 6] = best;
    __syncthreads();
    uint2 w = s_red[j & 1][0];
    for (int q = 1; q < 4; ++q)
      if (better(s_red[j & 1][q], w)) w = s_red[j & 1][q];
    if (w.y == 0xffffffffu && w.x == 0u) break;
    if (tid == 0) s_best[nsel] = w;
    prev = w;
    ++nsel;
  }
  if (tid == 0) s_nsel = nsel;
  __syncthreads();
  nsel = s_nsel;
  if (tid < nsel) {
    const long long flat = s_best[tid].y;
    const int a = (int)(flat / ((long long)hp.n_xy * hp.n_r));
    const int b = (int)((flat / hp.n_r) % hp.n_xy);
    const int k = (int)(flat % hp.n_r);
    const double xc = -hp.xy_half + hp.wxy * (a + 0.5), yc = -hp.xy_half + hp.wxy * (b + 0.5);
    const double R = hp.r_min + hp.wr * (k + 0.5);
    const double d = sqrt(xc * xc + yc * yc), R0 = hp.R0;
    WinSlot out{};
    out.valid = 0;
    if (d > 0.0 && d <= R + R0 && d >= fabs(R - R0)) {
      const double al = (R0 * R0 - R * R + d * d) / (2.0 * d);
      double hh = R0 * R0 - al * al;
      hh = hh > 0.0 ? sqrt(hh) : 0.0;
      const double cx = xc / d, cy = yc / d;
      const double P[2][2] = {{al * cx - hh * cy, al * cy + hh * cx}, {al * cx + hh * cy, al * cy - hh * cx}};
      const double pt = kKappa * hp.b_ref * R;
      double best_dot = 0.0;
      int pick = -1;
      for (int j = 0; j < 2; ++j) {
        double vx = -(P[j][1] - yc) / R, vy = (P[j][0] - xc) / R;
        if (hp.charge > 0.0) {
          vx = -vx;
          vy = -vy;
        }
        const double dot = vx * P[j][0] + vy * P[j][1];
        if (dot > best_dot) {
          best_dot = dot;
          pick = j;
          out.w.center[2] = pt * vx;
          out.w.center[3] = pt * vy;
        }
      }
      if (pick >= 0) {
        out.valid = 1;
        out.w.center[0] = atan2(P[pick][1], P[pick][0]);
        out.w.center[1] = hp.center_z;
        out.w.center[4] = hp.center_pz;
        const int e1 = half_max_extent(hp, A, a, b, k, 0);
        const int e2 = half_max_extent(hp, A, a, b, k, 1);
        const int e3 = half_max_extent(hp, A, a, b, k, 2);
        int s = e1 > e2 ? e1 : e2;
        s = e3 > s ? e3 : s;
        for (int q = 0; q < 5; ++q) {
          int nn = hp.count[q] + hp.grow[q] * (s - 1);
          nn = nn > hp.count_max ? hp.count_max : nn;
          nn = nn < 1 ? 1 : nn;
          out.w.count[q] = nn;
        }
        for (;;) {
          const long long prod = (long long)out.w.count[0] * out.w.count[1] * out.w.count[2] *
                                 out.w.count[3] * out.w.count[4];
          if (prod <= hp.max_seeds) break;
          int big = 0;
          for (int q = 1; q < 5; ++q)
            if (out.w.count[q] > out.w.count[big]) big = q;
          if (out.w.count[big] <= 1) break;
          out.w.count[big] -= 1;
        }
        for (int q = 0; q < 5; ++q) out.w.half_width[q] = hp.gran[q] * 0.5 * (double)(out.w.count[q] - 1);
        out.w.event = e;
      }
    }
    slots[(size_t)e * hp.max_cand + tid] = out;
  }
  if (tid == 0) n_valid[e] = nsel;
}

}  // namespace rkn

namespace rkn {

static rkn_status herr(rkn_ctx* c, hipError_t e, const char* where) {
  c->err = std::string(where) + ": " + hipGetErrorString(e);
  return e == hipErrorOutOfMemory ? RKN_E_NOMEM : RKN_E_DEVICE;
}

static bool dyadic(double v) { return std::isfinite(v) && v * 256.0 == std::floor(v * 256.0) && std::fabs(v) < 1e6; }

rkn_status make_hough_dev(rkn_ctx* c, const rkn_hough_params* p, HoughDev& h) {
  if (!p) {
    c->err = "hough params is NULL";
    return RKN_E_ARG;
  }
  const double wxy = 2.0 * p->xy_half / (p->n_xy > 0 ? p->n_xy : 1);
  const double wr = (p->r_max - p->r_min) / (p->n_r > 0 ? p->n_r : 1);
  if (p->n_xy < 1 || p->n_xy > 2048 || p->n_r < 1 || p->n_r > kMaxNr) {
    c->err = "hough: n_xy must be in [1, 2048] and n_r in [1, 64]";
    return RKN_E_ARG;
  }
  if (!(p->xy_half > 0) || !(p->r_max > p->r_min) || !(p->r_min >= 0) || !dyadic(p->xy_half) ||
      !dyadic(wxy) || !dyadic(p->r_min) || !dyadic(wr) || p->r_max > 4096.0 || p->xy_half > 4096.0) {
    c->err = "hough: xy_half, 2 xy_half/n_xy, r_min and (r_max-r_min)/n_r must be positive multiples of 2^-8 mm (<= 4096 mm)";
    return RKN_E_ARG;
  }
  if (p->max_cand < 1 || p->max_cand > kMaxCand || p->min_votes < 0 || p->count_max < 1 || p->max_seeds_window < 1) {
    c->err = "hough: max_cand in [1, 64], min_votes >= 0, count_max >= 1, max_seeds_window >= 1";
    return RKN_E_ARG;
  }
  if (!std::isfinite(p->R0) || p->R0 <= 0 || !std::isfinite(p->charge) || p->charge == 0 ||
      !std::isfinite(p->b_ref) || p->b_ref == 0 || !std::isfinite(p->center_z) || !std::isfinite(p->center_pz)) {
    c->err = "hough: R0 > 0, charge != 0, b_ref != 0, finite centres";
    return RKN_E_ARG;
  }
  for (int q = 0; q < 5; ++q) {
    if (!std::isfinite(p->gran[q]) || p->gran[q] < 0 || p->count[q] < 1 || p->grow[q] < 0) {
      c->err = "hough: gran >= 0, count >= 1, grow >= 0";
      return RKN_E_ARG;
    }
  }
  h.n_xy = p->n_xy;
  h.n_r = p->n_r;
  h.half_q = (int)std::llround(p->xy_half * 256.0);
  h.wxy_q = (int)std::llround(wxy * 256.0);
  h.rmin_q = (int)std::llround(p->r_min * 256.0);
  h.wr_q = (int)std::llround(wr * 256.0);
  h.min_votes = p->min_votes;
  h.max_cand = p->max_cand;
  h.R0 = p->R0;
  h.charge = p->charge;
  h.b_ref = p->b_ref;
  h.xy_half = p->xy_half;
  h.r_min = p->r_min;
  h.wxy = wxy;
  h.wr = wr;
  for (int q = 0; q < 5; ++q) {
    h.gran[q] = p->gran[q];
    h.count[q] = p->count[q];
    h.grow[q] = p->grow[q];
  }
  h.center_z = p->center_z;
  h.center_pz = p->center_pz;
  h.count_max = p->count_max;
  h.max_seeds = p->max_seeds_window;
  return RKN_OK;
}

static hipError_t zero_counts(rkn_ctx* c, int ev0, int n) {
  hipLaunchKernelGGL(hough_zero_kernel, dim3((n + 255) / 256), dim3(256), 0, c->stream,
                     c->hough_max.as<uint32_t>() + ev0, c->hough_cand_n.as<uint32_t>() + ev0, n);
  return hipGetLastError();
}

// Accumulate, find peaks and build windows for events [ev0, ev0+n); device slots.
static hipError_t run_hough_chunk(rkn_ctx* c, const HoughDev& h, int ev0, int n, bool windows) {
  hipError_t e;
  DevBuf& acc = c->hough_acc;
  // at most 4 + 32 KB of the workgroup's 64
  const size_t smem = sizeof(float2) * ((c->max_hits_event + 1) & ~1) + sizeof(uint32_t) * h.n_r * (kHoughCells / 2);
  hipLaunchKernelGGL(hough_vote_kernel, dim3(vote_blocks(h), n),
                     dim3(kHoughCells), smem, c->stream, h, c->max_hits_event, c->ev_off.as<int32_t>(),
                     c->hits_wire.as<int32_t>(), c->wire_wx.as<double>(), c->wire_wy.as<double>(), ev0,
                     acc.as<unsigned short>(), c->hough_max.as<uint32_t>());
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (!windows) return hipSuccess;
  hipLaunchKernelGGL(hough_peaks_kernel, dim3(vote_blocks(h), n), dim3(256), 0,
                     c->stream, h, acc.as<unsigned short>(), c->hough_max.as<uint32_t>(), ev0,
                     c->hough_cand_n.as<uint32_t>(),
                     c->hough_cand.as<uint2>());
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(hough_select_kernel, dim3(n), dim3(256), 0, c->stream, h, acc.as<unsigned short>(),
                     c->hough_max.as<uint32_t>(), ev0,
                     c->hough_cand_n.as<uint32_t>(), c->hough_cand.as<uint2>(), c->hough_slots.as<WinSlot>(),
                     c->hough_nsel.as<int32_t>());
  return hipGetLastError();
}

hipError_t ensure_hough_buffers(rkn_ctx* c, const HoughDev& h) {
  hipError_t e;
  const int ne = c->n_events;
  const size_t nb = (size_t)event_stride(h);
  if ((e = c->hough_acc.ensure(sizeof(unsigned short) * nb * std::min(kEventChunk, std::max(ne, 1)))) != hipSuccess)
    return e;
  if ((e = c->hough_max.ensure(sizeof(uint32_t) * ne)) != hipSuccess) return e;
  if ((e = c->hough_cand_n.ensure(sizeof(uint32_t) * ne)) != hipSuccess) return e;
  if ((e = c->hough_cand.ensure(sizeof(uint2) * (size_t)kCandCap * ne)) != hipSuccess) return e;
  if ((e = c->hough_slots.ensure(sizeof(WinSlot) * (size_t)kMaxCand * ne)) != hipSuccess) return e;
  if ((e = c->hough_nsel.ensure(sizeof(int32_t) * ne)) != hipSuccess) return e;
  return hipSuccess;
}

hipError_t queue_hough_all(rkn_ctx* c, const HoughDev& h) {
  if (c->n_events == 0) return hipSuccess;
  const hipError_t ez = zero_counts(c, 0, c->n_events);
  if (ez != hipSuccess) return ez;
  for (int ev0 = 0; ev0 < c->n_events; ev0 += kEventChunk) {
    const int n = std::min(kEventChunk, c->n_events - ev0);
    hipError_t e = run_hough_chunk(c, h, ev0, n, true);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace rkn

using namespace rkn;

extern "C" {

rkn_status rkn_hough_accumulator(rkn_ctx* c, const rkn_hough_params* hp, int32_t event, int32_t ptr_flags,
                                 uint32_t* acc) {
  if (!c) return RKN_E_ARG;
  HoughDev h;
  rkn_status st = make_hough_dev(c, hp, h);
  if (st != RKN_OK) return st;
  if (c->h_ev_off.empty()) {
    c->err = "no hits uploaded";
    return RKN_E_STATE;
  }
  if (event < 0 || event >= c->n_events || !acc || (ptr_flags & ~RKN_PTR_DEVICE)) {
    c->err = "bad event, output pointer or flags";
    return RKN_E_ARG;
  }
  hipError_t e;
  if ((e = hipSetDevice(c->device)) != hipSuccess) return herr(c, e, "hipSetDevice");
  if ((e = ensure_hough_buffers(c, h)) != hipSuccess) return herr(c, e, "hough alloc");
  const size_t nb = (size_t)h.n_xy * h.n_xy * h.n_r;
  const bool dev = (ptr_flags & RKN_PTR_DEVICE) != 0;
  if (!dev && (e = c->hough_public.ensure(nb * sizeof(uint32_t))) != hipSuccess) return herr(c, e, "hough alloc");
  if ((e = zero_counts(c, event, 1)) != hipSuccess) return herr(c, e, "hough clear");
  if ((e = run_hough_chunk(c, h, event, 1, false)) != hipSuccess) return herr(c, e, "hough vote");
  hipLaunchKernelGGL(hough_unpack_kernel, dim3(vote_blocks(h)), dim3(kHoughCells), 0, c->stream, h,
                     c->hough_acc.as<unsigned short>(), dev ? acc : c->hough_public.as<uint32_t>());
  e = hipGetLastError();
  if (e == hipSuccess && !dev) e = hipMemcpyAsync(acc, c->hough_public.p, nb * sizeof(uint32_t), hipMemcpyDeviceToHost,
                                                  c->stream);
  if (e == hipSuccess && !dev) e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return herr(c, e, "hough copy");
  return RKN_OK;
}

rkn_status rkn_hough_seed_windows(rkn_ctx* c, const rkn_hough_params* hp, int32_t max_windows, rkn_window* out,
                                  int32_t* n_out) {
  if (!c) return RKN_E_ARG;
  HoughDev h;
  rkn_status st = make_hough_dev(c, hp, h);
  if (st != RKN_OK) return st;
  if (c->h_ev_off.empty()) {
    c->err = "no hits uploaded";
    return RKN_E_STATE;
  }
  if (max_windows < 0 || (max_windows > 0 && !out) || !n_out) {
    c->err = "bad output arrays";
    return RKN_E_ARG;
  }
  hipError_t e;
  if ((e = hipSetDevice(c->device)) != hipSuccess) return herr(c, e, "hipSetDevice");
  if ((e = ensure_hough_buffers(c, h)) != hipSuccess) return herr(c, e, "hough alloc");
  const int ne = c->n_events;
  std::vector<WinSlot> slots((size_t)h.max_cand * ne);
  std::vector<int32_t> nsel(ne);
  if ((e = queue_hough_all(c, h)) != hipSuccess) return herr(c, e, "hough");
  e = hipMemcpyAsync(slots.data(), c->hough_slots.p, sizeof(WinSlot) * slots.size(), hipMemcpyDeviceToHost,
                     c->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(nsel.data(), c->hough_nsel.p, sizeof(int32_t) * ne, hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return herr(c, e, "hough copy");
  int32_t n = 0;
  for (int ev = 0; ev < ne; ++ev) {
    int cand = 0;
    for (int j = 0; j < nsel[ev]; ++j) {
      const WinSlot& s = slots[(size_t)ev * h.max_cand + j];
      if (!s.valid) continue;
      if (n < max_windows) {
        rkn_window& w = out[n];
        w.event = ev;
        w.candidate = cand;
        for (int q = 0; q < 5; ++q) {
          w.center[q] = s.w.center[q];
          w.half_width[q] = s.w.half_width[q];
          w.count[q] = s.w.count[q];
        }
        w.pad = 0;
      }
      ++cand;
      ++n;
    }
  }
  *n_out = n;
  if (n > max_windows) {
    c->err = "hough: " + std::to_string(n) + " windows do not fit in max_windows";
    return RKN_E_CAPACITY;
  }
  return RKN_OK;
}

}  // extern "C"
