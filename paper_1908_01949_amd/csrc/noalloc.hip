// rkn_scan_windows_noalloc: the window scan of rkn_scan_windows for callers that
// cannot allocate device memory (code under stream capture, tight serving loops,
// harnesses that forbid hipMalloc). Its work memory -- the device windows, their
// segments, the per-event chunk offsets, the division of the chunks, the argmin partials
// and the slab of running minima -- lives in one file-scope device array per GPU, held
// from the library's load until the process ends. Nothing in the call allocates.
//
// Host code never passes the array's name to a kernel or a copy: `scratch` in host
// code is a stand-in symbol, not a device address. Its address on each device is
// looked up once (noalloc_init, from rkn_create with that device current) and kept
// in g_ptr; every use goes through it.
#include <mutex>
#include <string>
#include <vector>

#include "internal.hpp"

namespace rkn {

constexpr size_t kScratchBytes = size_t(256) << 20;   // per GPU

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

constexpr int kMaxDevices = 64;

std::mutex g_mu;
bool g_done[kMaxDevices] = {};
hipError_t g_err[kMaxDevices] = {};
unsigned char* g_ptr[kMaxDevices] = {};

size_t align256(size_t n) { return (n + 255) & ~size_t(255); }

}  // namespace

hipError_t noalloc_init(int device) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_mu);
  if (!g_done[device]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    g_err[device] = e;
    g_ptr[device] = e == hipSuccess ? static_cast<unsigned char*>(ptr) : nullptr;
    g_done[device] = true;
  }
  return g_err[device];
}

}  // namespace rkn

using namespace rkn;

extern "C" {

rkn_status rkn_scan_windows_noalloc(rkn_ctx* c, const rkn_scan_params* p, int32_t n_windows, const rkn_window* w,
                                    double* score, int32_t* n_in, int64_t* best_index, double* best_score) {
  if (!c) return RKN_E_ARG;
  rkn_status st = validate_scan(c, p);
  if (st != RKN_OK) return st;
  if (!(p->ptr_flags & RKN_PTR_DEVICE) || !best_index || !best_score) {
    c->err = "scan (no allocation): outputs must be device pointers (ptr_flags RKN_PTR_DEVICE); best_index "
             "and best_score must not be NULL";
    return RKN_E_ARG;
  }
  hipError_t e;
  if ((e = hipSetDevice(c->device)) != hipSuccess) {
    c->err = std::string("hipSetDevice: ") + hipGetErrorString(e);
    return RKN_E_DEVICE;
  }
  if (c->device >= kMaxDevices || !g_done[c->device] || !g_ptr[c->device]) {
    c->err = std::string("scan (no allocation): no work array on this device: ") +
             (c->device < kMaxDevices && g_done[c->device] ? hipGetErrorString(g_err[c->device])
                                                          : "not initialised");
    return RKN_E_DEVICE;
  }
  std::vector<WindowDev> wins;
  SegList list(c->n_events);
  if ((st = prepare_scan_windows(c, n_windows, w, wins, list)) != RKN_OK) return st;
  rkn_scan_params q = *p;
  q.block_steps = resolve_block_steps(c, &q);
  // layout of the work array for this call; the argmin partials take at most half of
  // what is left (a scan of more chunks runs in several launches), the slab the rest
  const size_t n_seg = list.segs.size();
  const size_t o_win = 0;
  const size_t o_segs = o_win + align256(sizeof(WindowDev) * wins.size());
  const size_t o_evc = o_segs + align256(sizeof(Seg) * n_seg);
  const size_t o_plan = o_evc + align256(sizeof(int64_t) * list.ev_chunk.size());
  const size_t o_parts = o_plan + align256(scan_plan_bytes(c));
  const size_t per_wg = scan_slab_bytes_per_workgroup(c, &q);
  // The limit that rknscan.h states: 48 bytes for every workgroup's worth of seeds beside
  // the windows, 4 bytes an event and one workgroup's minima. It is a contract, not the
  // layout below, which needs less but for very many events: what was refused stays
  // refused when the layout changes.
  const size_t T = (size_t)scan_tile(c, &q);
  size_t need = o_win + align256(sizeof(WindowDev) * wins.size()) + align256(sizeof(int32_t) * list.ev_chunk.size()) +
                256 + per_wg;
  for (size_t k = 0; k + 1 < n_seg; ++k) need += 48 * (((size_t)list.segs[k].size + T - 1) / T);
  if (need > kScratchBytes || o_parts + 256 + per_wg > kScratchBytes) {
    c->err = "scan (no allocation): " + std::to_string(n_windows) + " windows, their " + std::to_string(list.seeds) +
             " seeds and the running minima of one workgroup need " + std::to_string(need) +
             " bytes, more than the " + std::to_string(kScratchBytes) + "-byte work array";
    return RKN_E_CAPACITY;
  }
  const size_t room = kScratchBytes - o_parts - per_wg;
  const int64_t max_parts =
      std::max<int64_t>(std::min<int64_t>(list.chunks, (int64_t)(room / 2 / sizeof(ArgminPart))), 1);
  const size_t o_slab = o_parts + align256(sizeof(ArgminPart) * (size_t)max_parts);
  unsigned char* base = g_ptr[c->device];
  if ((e = hipMemcpyAsync(base + o_win, wins.data(), sizeof(WindowDev) * wins.size(), hipMemcpyHostToDevice,
                          c->stream)) != hipSuccess ||
      (e = hipMemcpyAsync(base + o_segs, list.segs.data(), sizeof(Seg) * n_seg, hipMemcpyHostToDevice, c->stream)) !=
          hipSuccess ||
      (e = hipMemcpyAsync(base + o_evc, list.ev_chunk.data(), sizeof(int64_t) * list.ev_chunk.size(),
                          hipMemcpyHostToDevice, c->stream)) != hipSuccess) {
    c->err = std::string("scan (no allocation) upload: ") + hipGetErrorString(e);
    return RKN_E_DEVICE;
  }
  ScanSegs segs;
  segs.segs = reinterpret_cast<const Seg*>(base + o_segs);
  segs.n_seg = (int)n_seg - 1;
  segs.ev_chunk = reinterpret_cast<const int64_t*>(base + o_evc);
  segs.n_chunks = list.chunks;
  segs.windows = reinterpret_cast<const WindowDev*>(base + o_win);
  e = launch_scan_raw(c, &q, segs, score, n_in, best_index, best_score,
                      reinterpret_cast<ArgminPart*>(base + o_parts), max_parts,
                      base + o_plan, base + o_slab, kScratchBytes - o_slab);
  if (e == hipErrorInvalidConfiguration) {
    c->err = "scan configuration does not fit the device (LDS per workgroup); use FP32 or fewer hits per event";
    return RKN_E_UNSUPPORTED;
  }
  if (e != hipSuccess) {
    c->err = std::string("scan (no allocation) launch: ") + hipGetErrorString(e);
    return RKN_E_DEVICE;
  }
  return RKN_OK;
}

}  // extern "C"
