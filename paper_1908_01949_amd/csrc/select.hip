// Selection of the k lowest-score seeds of every event, on the device: the host step
// of the paper's coarse-to-fine refinement that picks the best seeds of a scan
// before finer seed sets are built around them (section 2.2), and the input of the
// derivative-based refinement (the best seeds per event of a batched scan).
#include <algorithm>
#include <string>
#include <vector>

#include "internal.hpp"

namespace rkn {

constexpr int kTopMax = 16;

__device__ __forceinline__ bool key_less(double a, long long ia, double b, long long ib) {
  return a < b || (a == b && ia < ib);
}

// The k lowest (score, index) pairs of a workgroup's candidates, ascending; NaN scores are
// never selected. `get(j, s, i)` reads candidate j of n. Each thread keeps a sorted list
// of its kTopMax best over a strided pass; k rounds of a workgroup argmin over the list
// heads then merge them into s_sc, s_sel (index -1 and infinity past the last candidate).
template <class GET>
__device__ __forceinline__ void block_topk(long long n, int k, double* s_sc, long long* s_sel, const GET& get) {
  __shared__ double s_e[4];
  __shared__ long long s_i[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double bs[kTopMax];
  long long bi[kTopMax];
#pragma unroll
  for (int j = 0; j < kTopMax; ++j) {
    bs[j] = INFINITY;
    bi[j] = 0x7fffffffffffffffLL;
  }
  for (long long g = tid; g < n; g += 256) {
    double s;
    long long i;
    get(g, s, i);
    if (!(s == s) || i < 0) continue;
#pragma unroll
    for (int j = 0; j < kTopMax; ++j) {
      const bool lt = key_less(s, i, bs[j], bi[j]);
      const double ts = lt ? bs[j] : s;
      const long long ti = lt ? bi[j] : i;
      bs[j] = lt ? s : bs[j];
      bi[j] = lt ? i : bi[j];
      s = ts;
      i = ti;
    }
  }
  for (int r = 0; r < k; ++r) {
    double be = bs[0];
    long long bx = bi[0];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      const double oe = __shfl_xor(be, o, 64);
      const long long ox = __shfl_xor(bx, o, 64);
      if (key_less(oe, ox, be, bx)) {
        be = oe;
        bx = ox;
      }
    }
    if (lane == 0) {
      s_e[wave] = be;
      s_i[wave] = bx;
    }
    __syncthreads();
    be = s_e[0];
    bx = s_i[0];
    for (int w = 1; w < 4; ++w)
      if (key_less(s_e[w], s_i[w], be, bx)) {
        be = s_e[w];
        bx = s_i[w];
      }
    const bool none = bx == 0x7fffffffffffffffLL;
    if (tid == 0) {
      s_sel[r] = none ? -1 : bx;
      s_sc[r] = none ? INFINITY : be;
    }
    // the owner of the winning head (indices are unique) pops it
    if (!none && bi[0] == bx) {
#pragma unroll
      for (int j = 0; j + 1 < kTopMax; ++j) {
        bs[j] = bs[j + 1];
        bi[j] = bi[j + 1];
      }
      bs[kTopMax - 1] = INFINITY;
      bi[kTopMax - 1] = 0x7fffffffffffffffLL;
    }
    __syncthreads();
  }
}

// Candidates of one slice of an event's seeds: its k lowest to part_s, part_i. An event
// whose seeds one workgroup reads alone is bound by that CU's loads and its 16 compares a
// seed (16^5 seeds: 3.7 ms); see topk_slices for the split.
__global__ void __launch_bounds__(256)
topk_slice_kernel(const double* __restrict__ score, const long long* __restrict__ seg_off, int k,
                  double* __restrict__ part_s, long long* __restrict__ part_i) {
  __shared__ long long s_sel[kTopMax];
  __shared__ double s_sc[kTopMax];
  const int e = blockIdx.y, n_sl = gridDim.x;
  const long long n = seg_off[e + 1] - seg_off[e], per = (n + n_sl - 1) / n_sl;
  const long long j0 = min(n, per * blockIdx.x), j1 = min(n, j0 + per), lo = seg_off[e] + j0;
  block_topk(j1 - j0, k, s_sc, s_sel, [&](long long j, double& s, long long& i) {
    i = lo + j;
    s = score[i];
  });
  if ((int)threadIdx.x < k) {
    const size_t o = ((size_t)e * n_sl + blockIdx.x) * k + threadIdx.x;
    part_s[o] = s_sc[threadIdx.x];
    part_i[o] = s_sel[threadIdx.x];
  }
}

// One workgroup per event: the k lowest of its scores (n_sl = 1) or of its slices'
// candidates. Seeds are decoded from the event's windows, whose seeds are contiguous from
// seg_off[e] in window order.
__global__ void __launch_bounds__(256)
topk_kernel(const double* __restrict__ score, const long long* __restrict__ seg_off,
            const double* __restrict__ part_s, const long long* __restrict__ part_i, int n_sl,
            const WindowDev* __restrict__ windows, const int32_t* __restrict__ win_off, int n_seg,
            const int32_t* __restrict__ win_total, int k, int64_t* __restrict__ out_idx,
            double* __restrict__ out_score, double* __restrict__ out_seed, double* __restrict__ out_step) {
  __shared__ long long s_sel[kTopMax];
  __shared__ double s_sc[kTopMax];
  const int e = blockIdx.x, tid = threadIdx.x;
  const long long lo = seg_off[e], hi = seg_off[e + 1];
  if (n_sl > 1) {
    const size_t o = (size_t)e * n_sl * k;
    block_topk((long long)n_sl * k, k, s_sc, s_sel, [&](long long j, double& s, long long& i) {
      s = part_s[o + j];
      i = part_i[o + j];
    });
  } else {
    block_topk(hi - lo, k, s_sc, s_sel, [&](long long j, double& s, long long& i) {
      i = lo + j;
      s = score[i];
    });
  }
  if (tid < k) {
    const long long g = s_sel[tid];
    const size_t o = (size_t)e * k + tid;
    out_idx[o] = g;
    out_score[o] = s_sc[tid];
    double v[5] = {NAN, NAN, NAN, NAN, NAN}, st[5] = {NAN, NAN, NAN, NAN, NAN};
    if (g >= 0 && (out_seed || out_step)) {
      const int w0 = win_off[e];
      const int w1 = e + 1 < n_seg ? win_off[e + 1] : *win_total;
      long long local = g - lo;
      for (int w = w0; w < w1; ++w) {
        long long size = 1;
        for (int d = 0; d < 5; ++d) size *= windows[w].count[d];
        if (local < size) {
          window_seed(windows[w], local, v);
          // the step of the grid the seed came from (0 where the window has one point)
          for (int d = 0; d < 5; ++d)
            st[d] = windows[w].count[d] > 1 ? 2.0 * windows[w].half_width[d] / (double)(windows[w].count[d] - 1)
                                            : 0.0;
          break;
        }
        local -= size;
      }
    }
    if (out_seed)
      for (int d = 0; d < 5; ++d) out_seed[o * 5 + d] = v[d];
    if (out_step)
      for (int d = 0; d < 5; ++d) out_step[o * 5 + d] = st[d];
  }
}

// Slices per event: enough workgroups for two on each of 256 CUs, at most 256 (their
// candidates are merged by one workgroup). The rule knows the events only, the seeds of a
// batch are counted on the device. One event of 16^5 seeds: 3.73 ms -> 47 us in 256
// slices; 64 events of 4 x 10^4 seeds in 8: 77 us; 3 x 8 windows: 40 us.
static int topk_slices(int n_events) { return std::min(256, (512 + n_events - 1) / n_events); }

static size_t topk_part_rows(int n_events) { return (size_t)topk_slices(n_events) * n_events * kTopMax; }

size_t topk_scratch_bytes(int n_events) {
  return n_events > 0 ? topk_part_rows(n_events) * (sizeof(double) + sizeof(long long)) : 0;
}

hipError_t launch_topk(rkn_ctx* c, const double* d_score, const long long* d_seg_off, const WindowDev* d_windows,
                       const int32_t* d_win_off, int n_seg, const int32_t* d_win_total, int k, int64_t* d_idx,
                       double* d_sc, double* d_seed, double* d_step) {
  if (n_seg <= 0) return hipSuccess;
  if (k < 1 || k > kTopMax) return hipErrorInvalidValue;
  const int n_sl = topk_slices(n_seg);
  double* part_s = c->sel_parts.as<double>();
  long long* part_i = (long long*)(part_s + topk_part_rows(n_seg));
  if (n_sl > 1)
    hipLaunchKernelGGL(topk_slice_kernel, dim3(n_sl, n_seg), dim3(256), 0, c->stream, d_score, d_seg_off, k, part_s,
                       part_i);
  hipLaunchKernelGGL(topk_kernel, dim3(n_seg), dim3(256), 0, c->stream, d_score, d_seg_off, part_s, part_i, n_sl,
                     d_windows, d_win_off, n_seg, d_win_total, k, d_idx, d_sc, d_seed, d_step);
  return hipGetLastError();
}

}  // namespace rkn
