// C ABI of libhfreshard (declarations and contracts: include/hfreshard.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <string>

#include "hfreshard.h"
#include "kernels.hpp"
#include "plan.hpp"

// the Python binding mirrors these layouts field by field
static_assert(sizeof(hf_desc) == 88 && sizeof(hf_tile) == 48 && sizeof(hf_tensor_info) == 32, "ABI struct layout");
static_assert(sizeof(hf_model_desc) == 36 && sizeof(hf_gen_layout) == 32 && sizeof(hf_train_layout) == 12, "ABI struct layout");

struct hf_plan {
  hf::Plan p;
};

// Work-list staging area of hf_reshard_execute_static: device memory that exists from the
// moment the library is loaded, so that the entry point never has to allocate.  In host code
// this name is only a handle for hipGetSymbolAddress; the address the kernels get is looked
// up once per device (scratch_of).
static __device__ __align__(256) unsigned char scratch[hf::kStaticRoom];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};       // device address of `scratch` on each device
uint64_t g_scratch_serial[kMaxDevices] = {}; // Plan::serial of the work list staged there
std::atomic<uint64_t> g_next_serial{1};

thread_local std::string g_err;

int fail(int code, const std::string &msg) {
  g_err = msg;
  return code;
}

template <typename T> void release(T *&ptr) {
  if (ptr) (void)hipFree(ptr);
  ptr = nullptr;
}

void free_device(hf::Plan &p) {
  for (hf::DevList *l : {&p.dev_fwd, &p.dev_auto, &p.dev_own, &p.dev_back, &p.dev_offload, &p.dev_reload}) l->d = nullptr;
  p.d_mc_dst = p.d_auto_dst = nullptr;
  p.d_gather_out = nullptr;
  release(p.d_forward);
  release(p.d_others);
}

// Uploads arrays into one allocation, in the place of what `block` held: an allocation and a copy each cost a small plan more
// than its bytes do (building and uploading the tiny decoder's plan 0.16 ms with an allocation per array, 0.105 with two).  The device pointer of an empty array is null, and all are when it fails.
struct Upload {
  char *&block;
  struct Part {
    const void *v;
    size_t bytes, at;
    void *d; // the pointer to the device copy, for `set`
    void (*set)(void *d, char *at);
  };
  Part parts[8];
  size_t n = 0, total = 0;

  explicit Upload(char *&into) : block(into) {}
  template <typename T> void add(const std::vector<T> &v, T **d) {
    *d = nullptr;
    if (v.empty()) return;
    parts[n++] = {v.data(), v.size() * sizeof(T), total, d, [](void *to, char *at) { *static_cast<T **>(to) = reinterpret_cast<T *>(at); }};
    total += (v.size() * sizeof(T) + 255) / 256 * 256;
  }
  void add(hf::DevList &l) { add(l.tiles, &l.d); }

  int run() {
    release(block);
    if (total == 0) return HF_OK;
    hipError_t e = hipMalloc(reinterpret_cast<void **>(&block), total);
    if (e != hipSuccess) {
      block = nullptr;
      return fail(e == hipErrorOutOfMemory ? HF_ENOMEM : HF_EHIP, std::string("hipMalloc: ") + hipGetErrorString(e));
    }
    const std::unique_ptr<char[]> packed(total <= (256u << 10) ? new (std::nothrow) char[total]() : nullptr);
    for (size_t i = 0; i < n && e == hipSuccess; ++i) {
      if (packed) std::memcpy(packed.get() + parts[i].at, parts[i].v, parts[i].bytes);
      else e = hipMemcpy(block + parts[i].at, parts[i].v, parts[i].bytes, hipMemcpyHostToDevice);
    }
    if (packed) e = hipMemcpy(block, packed.get(), total, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
      release(block); // nobody runs what was not copied
      return fail(HF_EHIP, std::string("hipMemcpy: ") + hipGetErrorString(e));
    }
    for (size_t i = 0; i < n; ++i) parts[i].set(parts[i].d, block + parts[i].at);
    return HF_OK;
  }
};

// Makes the train->gen work list of the current multicast mode resident, in the place of another mode's.  Called
// at plan time and from hf_plan_set_param, never from an execution entry point.
int upload_forward_list(hf::Plan &p) {
  Upload up(p.d_forward);
  up.add(p.dev_fwd);
  p.d_mc_dst = nullptr;
  if (p.active_fwd_uses_mc_dst()) up.add(p.mc_dst, &p.d_mc_dst);
  return up.run();
}

// The library's own list stays resident beside the mode's (5 MB at the Llama-7B shape): which of
// the two hf_reshard_execute runs is then a matter of parameters alone, and a captured graph keeps the one it holds.
int upload(hf::Plan &p) {
  free_device(p);
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(HF_EHIP, std::string("no HIP device: ") + hipGetErrorString(e));
  p.device = dev;
  int rc = upload_forward_list(p);
  if (rc == HF_OK) {
    Upload up(p.d_others);
    for (hf::DevList *l : {&p.dev_auto, &p.dev_own, &p.dev_back, &p.dev_offload, &p.dev_reload}) up.add(*l);
    up.add(p.auto_dst, &p.d_auto_dst);
    up.add(p.gather_out, &p.d_gather_out);
    rc = up.run();
  }
  if (rc != HF_OK) free_device(p);
  return rc;
}

// Gives `field`, a parameter that the lists depend on, another value, rebuilds and re-uploads them.  A
// value that is refused, or one whose lists find no host memory, leaves the plan as it was.
int retile(hf::Plan &p, int64_t &field, int64_t value) {
  const int64_t old_value = field;
  hf::WorkLists old = std::move(static_cast<hf::WorkLists &>(p));
  static_cast<hf::WorkLists &>(p) = hf::WorkLists();
  p.multicast = old.multicast;
  field = value;
  std::string err;
  int rc;
  try {
    rc = hf::build_tiles(p, err);
  } catch (const std::bad_alloc &) {
    rc = HF_ENOMEM;
    err = "out of host memory while tiling";
  }
  if (rc != HF_OK) {
    field = old_value;
    static_cast<hf::WorkLists &>(p) = std::move(old);
    return fail(rc, err);
  }
  p.serial = g_next_serial++;
  if (!(p.flags & HF_PLAN_HOST_ONLY)) return upload(p);
  return HF_OK;
}

// Makes another device current while it exists (-1: none).
struct OnDevice {
  int before = -1;
  hipError_t e = hipSuccess;
  explicit OnDevice(int device) {
    if (device < 0) return;
    int now = -1;
    if ((e = hipGetDevice(&now)) != hipSuccess || now == device) return;
    if ((e = hipSetDevice(device)) == hipSuccess) before = now;
  }
  ~OnDevice() {
    if (before >= 0) (void)hipSetDevice(before);
  }
  OnDevice(const OnDevice &) = delete;
  OnDevice &operator=(const OnDevice &) = delete;
};

// the lists of another multicast mode; without host memory for them the plan stays as it was
int set_multicast(hf::Plan &p, int64_t value) {
  const bool old_auto = p.multicast_auto;
  const int64_t old_mode = p.multicast;
  hf::DevList dev = std::move(p.dev_fwd);
  std::vector<hf_tile> cb = std::move(p.tiles_fwd_cb), pf = std::move(p.tiles_fwd_pf);
  hf::DevList dev_static = std::move(p.dev_static);
  std::vector<uint64_t> static_dst = std::move(p.static_dst);
  const uint64_t static_bytes = p.static_bytes;
  p.dev_fwd = hf::DevList();
  p.dev_fwd.d = dev.d;
  p.multicast_auto = value == HF_MULTICAST_AUTO;
  p.multicast = p.multicast_auto ? hf::default_multicast(p) : value;
  try {
    hf::build_forward_lists(p);
  } catch (const std::bad_alloc &) {
    p.multicast_auto = old_auto;
    p.multicast = old_mode;
    p.dev_fwd = std::move(dev);
    p.tiles_fwd_cb = std::move(cb);
    p.tiles_fwd_pf = std::move(pf);
    p.dev_static = std::move(dev_static);
    p.static_dst = std::move(static_dst);
    p.static_bytes = static_bytes;
    return fail(HF_ENOMEM, "out of host memory while building the work list");
  }
  return HF_OK;
}

// train_optional: the call does not read or write train_buf (it may then be null)
int check_buffers(const hf::Plan &p, const void *train_buf, const void *gen_buf, bool train_optional) {
  if (!gen_buf || (!train_buf && !train_optional)) return fail(HF_EINVAL, "null plan or buffer");
  if ((reinterpret_cast<uintptr_t>(train_buf) | reinterpret_cast<uintptr_t>(gen_buf)) % 256)
    return fail(HF_EINVAL, "train_buf and gen_buf must be 256-byte aligned");
  const char *t0 = static_cast<const char *>(train_buf), *g0 = static_cast<const char *>(gen_buf);
  if (t0 && t0 < g0 + p.gen_bytes && g0 < t0 + p.train_bytes) return fail(HF_EINVAL, "train_buf and gen_buf overlap");
  return HF_OK;
}

int check_exec(const hf_plan *plan, const void *train_buf, const void *gen_buf, bool train_optional = false) {
  if (!plan) return fail(HF_EINVAL, "null plan or buffer");
  if (int rc = check_buffers(plan->p, train_buf, gen_buf, train_optional)) return rc;
  if (plan->p.flags & HF_PLAN_HOST_ONLY) return fail(HF_EINVAL, "plan was built with HF_PLAN_HOST_ONLY: it has no device copy");
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev != plan->p.device)
    return fail(HF_EINVAL, "the current HIP device is not the one the plan was built on");
  return HF_OK;
}

// temporal_loads: the work list counts on re-reads being served by L2
enum { kListTransition = 0, kListFullRefresh = 1, kListOther = 2 }; // names the list in the kernel's name

// How a list wants to be run when the plan leaves the choice to the library.
enum ListShape {
  kShapeStreaming = 0,  // every byte is read once from HBM
  kShapeCacheBlocked,   // later passes re-read from L2: plain loads, 8 KiB workgroups
  kShapePrefetched      // copy workgroups find their source in L2: plain loads, one wavefront per KiB
};

// One-to-one lists that the memory-side cache can help: plain loads (below), and the parts of a record on one XCD (place_of), so that a line which
// two parts share leaves L2 once.  What L2 fetches, of the payload, on all XCDs / on one: rows of 690 bytes 1.102 / 1.055, of 324 1.341 / 1.191, of 260 1.051 / 1.007,
// whole lines 1.012 / 1.004 (the records themselves); what it writes is the same.  us, three sets of buffers in turn: back, hidden 512 in rows of 690 bytes, 89 MB
// 14.82 / 14.53, execute 33 MB 6.49 / 6.23, 78 MB 12.25 / 11.92, install 87 MB 14.91 / 14.47, rows of 324 bytes 76 MB 15.34 / 14.78, refresh 116 MB 17.82 / 17.37, 174 MB 25.19 / 24.89.
// On one against all, 48 lists of 26 to 199 MB: rows of calls 0.975 (0.93-1.01); one call that is waited for, 16 to 60 us with the host's part, on the same buffers 0.991, source
// cold after 1 GiB of reads 1.008, after an optimizer step over the source 1.013 (at most 1.056), after 1 GiB of other writes 1.024 (at most 1.075): where the lines of a source come from
// memory, eight records at a time are, as it seems, too wide a window already.  No size of list between these is better or worse off.  Longer lists want the narrow window of
// addresses throughout: 344 MB 52.5 / 53.4, 590 MB 89.7 / 91.9, Llama-7B back 4180 / 4320; two, four or eight KiB in turn to an XCD instead: 1-4 % behind at all sizes.
// Shared pieces under HF_MULTICAST_OFF, which are read again for each destination, stay on all XCDs: 29 MB 7.37 / 7.95, 56 MB 12.1 / 12.9, 80 MB 16.6 / 18.1, 91 MB 17.7 / 19.2.
constexpr uint64_t kCachedList = 192ull << 20;

// Cache policy when the caller leaves it to the library.  TB/s (read once + written), 3 sets of buffers in
// turn, hidden 1024 and 512; records whose rows share lines are loaded plainly under every policy:
//   one-to-one: plain loads find what the memory-side cache (256 MiB) still holds of a short list's source, 51
//     MB 6.6 against 5.4 with non-temporal ones, 154 MB 7.9 / 6.3, 206 MB level, 411 MB 6.4 / 6.7, 2 GB 6.5 / 6.8;
//   registers (about two destinations): plain loads throughout, 231 MB 8.4 / 6.2, 3.9 GB 6.6 / 6.1; stores
//     compiler non-temporal up to 231 MB (odd rows 8.2 against 7.8 system-scope, even ones level),
//     system-scope above (3.9 GB 6.62 / 6.25, odd rows 6.54 / 6.30);
//   prefetched: plain loads (the block waits in L2); compiler non-temporal stores at three
//     and four destinations (system-scope level for whole lines, odd rows 2-9 % behind at three), system-scope
//     ones at seven and eight (hidden 1024 and 2048 5.42 / 5.23 and 5.86 / 5.71, odd rows 5.02 / 4.78, Llama-7B layers
//     5.68 / 5.48; not everywhere: hidden 5120 6.77 / 6.81, 8192 6.24 / 6.22, a merge of eight stages 6.72 / 6.80);
//   cache-blocked: plain loads, non-temporal stores (system-scope ones disturb the block, 8 % behind).
// The state of the memory-side cache before the call matters more than where the source is.  us, plain /
// non-temporal loads, one-to-one 168 MB (whole halves of lines; odd rows 145 MB): three sets in turn 26.8 /
// 29.0 (26.2 / 27.2); source cold, after 1 GiB of reads 26.7 / 28.8 (26.2 / 26.9); source just written, after 1
// GiB of writes 32.3 / 32.6 (29.7 / 30.0); source cold after 1 GiB of writes 35.0 / 30.8 (32.9 / 31.5): only then
// plain loads are behind, because they push out lines that somebody has yet to write to memory.  Registers at
// 168 MB, plain / non-temporal loads with non-temporal stores: 32.3 / 35.3, 31.7 / 35.0, 32.4 / 38.0 and 39.2 / 36.8.
int automatic_policy(const hf::Plan &p, const hf::DevList &list, bool registers, ListShape shape, bool short_list) {
  if (short_list && hf::non_temporal_when_short(list)) return 5;
  if (shape == kShapeCacheBlocked) return 5;
  if (shape == kShapePrefetched) return p.moved_bytes[0] >= 6 * p.unique_bytes[0] ? 1 : 5;
  if (registers) return list.bytes <= (256ull << 20) ? 5 : 1;
  return list.bytes <= kCachedList ? 1 : 0;
}

// One-to-one lists whose bytes the chip moves about as fast as workgroups of one wavefront are handed out (4.7 per ns): workgroups of
// 256 lanes with two slots each, half as many wavefronts and an eighth as many workgroups.  Against one wavefront, 189 lists of 8 to 25 MB, up to
// 16 MiB | above: rows of calls (a replayed graph of 60, three sets of buffers in turn) 0.85 (0.74-0.96) | 0.90 (0.78-1.05); one call that is waited for, 14 to 20 us with the
// host's part, on the same buffers 0.98 | 0.95, after an optimizer step over the source 0.97 | 0.94, source cold after 1 GiB of reads 1.00 | 1.01, after 1 GiB
// of other writes 1.01 | 1.02 (at most 1.06; the kernel alone 1.00-1.04 | 1.07).  Rows of calls, us: the tiny decoder (8 MB) 3.37 / 2.82, back, hidden 512, 15 MB 3.41 / 2.71, rows of 324 bytes 22 MB
// 5.16 / 5.41.  Above, single wavefronts are level or ahead: 34 MB 6.32 / 6.21 and 6.77 / 6.80, rows of 324 bytes 28 MB 6.71 / 6.65 (cold 9.44 / 9.68, after writes 11.1 /
// 12.5), 60 MB cold 14.1 / 14.9.
constexpr uint64_t kShortList = 24ull << 20;

int not_resident() { return fail(HF_EHIP, "the work list is not on the device (an earlier upload failed)"); }

// `at`: where the list's records are on the device
int launch(const hf::Plan &p, const hf::DevList &list, const hf::DevTile *at, const uint64_t *extra_dst, const void *src, void *dst,
           void *stream, int list_tag, ListShape shape = kShapeStreaming) {
  if (!at && !list.tiles.empty()) return not_resident();
  const bool temporal_loads = shape == kShapeCacheBlocked;
  const bool own_choice = shape == kShapeStreaming && !extra_dst && p.variant == HF_VARIANT_PARTS && !p.wg_threads && !p.part_bytes;
  const bool short_list = own_choice && list.bytes <= kShortList;
  const int variant = own_choice && list.one_to_one && list.bytes <= kCachedList ? hf::kVariantPartsTogether : (int)p.variant;
  const int policy = p.cache_policy >= 0 ? (int)p.cache_policy : automatic_policy(p, list, extra_dst != nullptr, shape, short_list);
  // Automatic launch shape, measured on the Llama-7B / 34B transitions: lists whose later
  // passes hit L2 run best with 256 lanes x 2 vectors (8 KiB per workgroup); plain streaming
  // lists with one wavefront x 1 vector (1 KiB per workgroup), unless they are short.
  const bool large = temporal_loads || short_list;
  const int threads = p.wg_threads ? (int)p.wg_threads : large ? 256 : 64;
  uint32_t part = p.part_bytes ? (uint32_t)p.part_bytes : (large ? 8192u : threads == 64 ? 1024u : 4096u);
  part = threads == 64 ? std::min(part, 8192u) : std::max(part, 4096u);
  const int e = hf::launch_tiles(at, list.tiles.size(), extra_dst, src, dst, variant, (int)p.grid_wgs, policy,
                                 list.unit_bytes, part,
                                 (uint32_t)(p.max_wgs_per_launch * (256 / threads)), threads, list_tag, stream);
  if (e != 0) return fail(HF_EHIP, std::string("kernel launch: ") + hipGetErrorString(static_cast<hipError_t>(e)));
  return HF_OK;
}

int forward_tag(const hf::Plan &p) { return (p.flags & HF_COPY_OWN) ? kListFullRefresh : kListTransition; }
ListShape forward_shape(const hf::Plan &p) {
  switch (p.effective_multicast()) {
  case HF_MULTICAST_CACHE_BLOCKED: return kShapeCacheBlocked;
  case HF_MULTICAST_PREFETCHED: return kShapePrefetched;
  default: return kShapeStreaming;
  }
}

// What hf_reshard_execute runs while every choice is the library's (Plan::dev_auto, auto_launch)
int launch_auto(const hf::Plan &p, const void *src, void *dst, void *stream) {
  if (!p.dev_auto.d) return not_resident();
  const hf::AutoLaunch a = hf::auto_launch(p);
  const int threads = a.short_list ? hf::kAutoShortThreads : 64;
  const int e = hf::launch_tiles(p.dev_auto.d, p.dev_auto.tiles.size(), p.d_auto_dst, src, dst, a.paced ? hf::kVariantAutoPaced : hf::kVariantAuto,
                                 a.wgs_per_cu, a.policy, p.dev_auto.unit_bytes, (uint32_t)threads * 16, (uint32_t)(p.max_wgs_per_launch * 256 / threads), threads,
                                 forward_tag(p), stream);
  if (e != 0) return fail(HF_EHIP, std::string("kernel launch: ") + hipGetErrorString(static_cast<hipError_t>(e)));
  return HF_OK;
}

} // namespace

extern "C" {

int hf_reshard_plan(const hf_model_desc *model, const hf_train_layout *train, const hf_gen_layout *gen, hf_plan **out) {
  if (out) *out = nullptr;
  if (!model || !train || !gen || !out) return fail(HF_EINVAL, "null argument");
  hf_plan *pl = new (std::nothrow) hf_plan();
  if (!pl) return fail(HF_ENOMEM, "out of host memory");
  std::string err;
  int rc;
  try {
    rc = hf::build_plan(*model, *train, *gen, pl->p, err);
  } catch (const std::bad_alloc &) {
    rc = HF_ENOMEM;
    err = "out of host memory while building the plan";
  }
  pl->p.serial = g_next_serial++;
  if (rc == HF_OK && !(gen->flags & HF_PLAN_HOST_ONLY)) {
    rc = upload(pl->p);
    if (rc != HF_OK) err = g_err;
  }
  if (rc != HF_OK) {
    delete pl;
    return fail(rc, err);
  }
  *out = pl;
  return HF_OK;
}

void hf_plan_destroy(hf_plan *plan) {
  if (!plan) return;
  free_device(plan->p);
  delete plan;
}

int hf_reshard_execute(const hf_plan *plan, const void *train_buf, void *gen_buf, void *hip_stream) {
  // gathering out of the generation buffers: gen_buf is source and destination (disjoint
  // pieces), train_buf is not used and need not exist
  const bool from_gen = plan && (plan->p.flags & HF_GATHER_FROM_GEN);
  if (int rc = check_exec(plan, train_buf, gen_buf, from_gen)) return rc;
  if (from_gen) train_buf = gen_buf;
  const hf::Plan &p = plan->p;
  if (p.runs_auto()) return launch_auto(p, train_buf, gen_buf, hip_stream);
  return launch(p, p.dev_fwd, p.dev_fwd.d, p.d_mc_dst, train_buf, gen_buf, hip_stream, forward_tag(p), forward_shape(p));
}

int hf_reshard_execute_static(const hf_plan *plan, const void *train_buf, void *gen_buf, void *hip_stream) {
  if (!plan) return fail(HF_EINVAL, "null plan or buffer");
  const hf::Plan &p = plan->p;
  const bool from_gen = (p.flags & HF_GATHER_FROM_GEN) != 0;
  if (int rc = check_buffers(p, train_buf, gen_buf, from_gen)) return rc;
  if (from_gen) train_buf = gen_buf; // source and destination are disjoint pieces of gen_buf
  if (p.static_bytes > HF_STATIC_SCRATCH_BYTES)
    return fail(HF_ERANGE, "work list of " + std::to_string(p.static_bytes) + " bytes or more does not fit the static scratch of " +
                               std::to_string((size_t)HF_STATIC_SCRATCH_BYTES) + " bytes: raise HF_PARAM_TILE_BYTES or use hf_reshard_execute");
  // the work list of the mode in force, from the plan's host copy, or the form of it that fits
  const bool own_form = !p.dev_static.tiles.empty();
  const hf::DevList &list = own_form ? p.dev_static : p.dev_fwd;
  const std::vector<uint64_t> &dst = own_form ? p.static_dst : p.mc_dst;
  const size_t n = list.tiles.size(), tile_bytes = n * sizeof(hf::DevTile), extra_at = (tile_bytes + 255) / 256 * 256;
  const size_t extra_bytes = p.active_fwd_uses_mc_dst() ? dst.size() * sizeof(uint64_t) : 0;
  if (n == 0) return HF_OK;
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(HF_EHIP, std::string("no HIP device: ") + hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return fail(HF_ERANGE, "device index beyond the library's table");
  if (p.device >= 0 && dev != p.device) return fail(HF_EINVAL, "the current HIP device is not the one the plan was built on");
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  char *base = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) { // once per device, with that device current
      void *ptr = nullptr;
      e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
      if (e != hipSuccess || !ptr) return fail(HF_EHIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
      g_scratch_ptr[dev] = ptr;
    }
    base = static_cast<char *>(g_scratch_ptr[dev]);
    if (g_scratch_serial[dev] != p.serial) { // another plan's list (or none) is staged: replace it, in stream order
      g_scratch_serial[dev] = 0;
      e = hipMemcpyAsync(base, list.tiles.data(), tile_bytes, hipMemcpyHostToDevice, st);
      if (e == hipSuccess && extra_bytes) e = hipMemcpyAsync(base + extra_at, dst.data(), extra_bytes, hipMemcpyHostToDevice, st);
      if (e != hipSuccess) return fail(HF_EHIP, std::string("staging the work list: ") + hipGetErrorString(e));
      g_scratch_serial[dev] = p.serial;
    }
  }
  // (the form that fits has no load-only records)
  const ListShape shape = own_form && forward_shape(p) == kShapePrefetched ? kShapeStreaming : forward_shape(p);
  return launch(p, list, reinterpret_cast<const hf::DevTile *>(base), extra_bytes ? reinterpret_cast<const uint64_t *>(base + extra_at) : nullptr,
                train_buf, gen_buf, hip_stream, forward_tag(p), shape);
}

// host_buf must be pinned host memory; returns the address the device uses for it
static int device_view_of_pinned(const void *host_buf, size_t bytes, void **out) {
  hipPointerAttribute_t at;
  std::memset(&at, 0, sizeof at);
  if (hipPointerGetAttributes(&at, host_buf) != hipSuccess) {
    (void)hipGetLastError(); // an unknown pointer leaves a sticky error behind
    return fail(HF_EINVAL, "host_buf is not known to the HIP runtime: it must be pinned host memory (hipHostMalloc)");
  }
  if (at.type != hipMemoryTypeHost || !at.devicePointer)
    return fail(HF_EINVAL, "host_buf must be pinned host memory that the device can address (hipHostMalloc)");
  void *base = nullptr;
  size_t size = 0;
  if (hipMemGetAddressRange(reinterpret_cast<hipDeviceptr_t *>(&base), &size, at.devicePointer) == hipSuccess && base) {
    const char *lo = static_cast<const char *>(base), *p0 = static_cast<const char *>(at.devicePointer);
    if (p0 < lo || p0 + bytes > lo + size) return fail(HF_EINVAL, "host_buf is shorter than hf_plan_remote_bytes");
  } else {
    (void)hipGetLastError();
  }
  *out = at.devicePointer;
  return HF_OK;
}

static int offload_common(const hf_plan *plan, const void *gen_buf, const void *host_buf, void **host_dev) {
  if (!plan || !gen_buf || !host_buf) return fail(HF_EINVAL, "null plan or buffer");
  const hf::Plan &p = plan->p;
  if (p.flags & HF_PLAN_HOST_ONLY) return fail(HF_EINVAL, "plan was built with HF_PLAN_HOST_ONLY: it has no device copy");
  if (!(p.flags & HF_PLAN_OFFLOAD)) return fail(HF_EINVAL, "plan was built without HF_PLAN_OFFLOAD");
  if (p.kind_mask != 0x1F) return fail(HF_EINVAL, "plan is restricted to some descriptor kinds");
  if ((reinterpret_cast<uintptr_t>(gen_buf) | reinterpret_cast<uintptr_t>(host_buf)) % 256)
    return fail(HF_EINVAL, "gen_buf and host_buf must be 256-byte aligned");
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev != p.device)
    return fail(HF_EINVAL, "the current HIP device is not the one the plan was built on");
  return device_view_of_pinned(host_buf, p.remote_bytes, host_dev);
}

// The host link, not HBM, bounds these two: a handful of persistent workgroups (each lane
// with eight 16-byte accesses in flight) keeps it full.  More would only queue host-bound
// writes in the memory fabric ahead of the HBM traffic of kernels on other streams.
// A workgroup that loads the next record while it stores one (reshard_link) gains where a record is over before its loads
// have come back: into the generation buffer, GB/s, pieces of 2 to 8 KiB 35 / 47, records of 16 KiB 47 / 56; with 32 KiB
// (compile_list) the other one is 1 % ahead (57.0 / 56.6).  Outwards it is level or up to 3 % ahead throughout.
static int launch_link(const hf::Plan &p, const hf::DevList &list, const void *src, void *dst, bool outwards, void *stream) {
  if (!list.d && !list.tiles.empty()) return not_resident();
  const int policy = p.cache_policy >= 0 ? (int)p.cache_policy : 0;
  const bool ahead = !list.short_rows && (outwards || list.bytes / 2 < list.tiles.size() * (24ull << 10));
  const int e = hf::launch_tiles(list.d, list.tiles.size(), nullptr, src, dst, ahead ? hf::kVariantLink : (int)HF_VARIANT_PERSISTENT, (int)p.offload_wgs, policy,
                                 list.unit_bytes, 4096u, (uint32_t)p.max_wgs_per_launch, 256, kListOther, stream);
  if (e != 0) return fail(HF_EHIP, std::string("kernel launch: ") + hipGetErrorString(static_cast<hipError_t>(e)));
  return HF_OK;
}

int hf_offload_remote(const hf_plan *plan, const void *gen_buf, void *host_buf, void *hip_stream) {
  void *hd = nullptr;
  if (int rc = offload_common(plan, gen_buf, host_buf, &hd)) return rc;
  return launch_link(plan->p, plan->p.dev_offload, gen_buf, hd, true, hip_stream);
}

int hf_reload_remote(const hf_plan *plan, const void *host_buf, void *gen_buf, void *hip_stream) {
  void *hd = nullptr;
  if (int rc = offload_common(plan, gen_buf, host_buf, &hd)) return rc;
  return launch_link(plan->p, plan->p.dev_reload, hd, gen_buf, false, hip_stream);
}

size_t hf_plan_remote_bytes(const hf_plan *plan) { return plan ? plan->p.remote_bytes : 0; }
size_t hf_plan_remote_rank_offset(const hf_plan *plan, int rank) {
  if (!plan || rank < 0 || rank >= plan->p.N || plan->p.mat_pos[rank] < 0) return (size_t)-1;
  return plan->p.remote_rank_off[plan->p.mat_pos[rank]];
}

int hf_plan_check_buffers(const hf_plan *plan, const void *train_buf, size_t train_len, const void *gen_buf, size_t gen_len) {
  if (!plan) return fail(HF_EINVAL, "null plan or buffer");
  const hf::Plan &p = plan->p;
  // a plan that gathers out of the generation buffers never touches train_buf
  if (int rc = check_buffers(p, train_buf, gen_buf, (p.flags & HF_GATHER_FROM_GEN) != 0)) return rc;
  if (train_buf && train_len < p.train_bytes) return fail(HF_EINVAL, "train_buf is shorter than hf_plan_train_bytes");
  if (gen_len < p.gen_bytes) return fail(HF_EINVAL, "gen_buf is shorter than hf_plan_gen_bytes");
  if (p.flags & HF_PLAN_HOST_ONLY) return HF_OK;
  struct { const char *ptr; size_t need; const char *name; } bufs[] = {{static_cast<const char *>(train_buf), p.train_bytes, "train_buf"},
                                                                        {static_cast<const char *>(gen_buf), p.gen_bytes, "gen_buf"}};
  for (auto &b : bufs) {
    if (!b.ptr) continue;
    void *base = nullptr;
    size_t size = 0;
    if (hipMemGetAddressRange(reinterpret_cast<hipDeviceptr_t *>(&base), &size, const_cast<char *>(b.ptr)) != hipSuccess || !base) {
      (void)hipGetLastError();
      return fail(HF_ERANGE, std::string(b.name) + " is not inside a device allocation of the HIP runtime");
    }
    if (b.ptr + b.need > static_cast<const char *>(base) + size)
      return fail(HF_ERANGE, std::string(b.name) + ": the device allocation ends before the bytes the plan needs");
  }
  return HF_OK;
}

int hf_reshard_install_own(const hf_plan *plan, const void *train_buf, void *gen_buf, void *hip_stream) {
  if (int rc = check_exec(plan, train_buf, gen_buf)) return rc;
  const hf::Plan &p = plan->p;
  return launch(p, p.dev_own, p.dev_own.d, nullptr, train_buf, gen_buf, hip_stream, kListOther);
}

int hf_reshard_back(const hf_plan *plan, void *train_buf, const void *gen_buf, void *hip_stream) {
  if (int rc = check_exec(plan, train_buf, gen_buf)) return rc;
  const hf::Plan &p = plan->p;
  if (p.flags & HF_GROUPING_VANILLA)
    return fail(HF_EINVAL, "vanilla grouping keeps the training shard besides the generation buffer: nothing to re-partition");
  return launch(p, p.dev_back, p.dev_back.d, nullptr, gen_buf, train_buf, hip_stream, kListOther);
}

int hf_gather_responses(const hf_plan *plan, const void *resp_in, void *resp_out, size_t slot_bytes, void *hip_stream) {
  if (!plan || !resp_in || !resp_out) return fail(HF_EINVAL, "null plan or buffer");
  const hf::Plan &p = plan->p;
  if (p.flags & HF_PLAN_HOST_ONLY) return fail(HF_EINVAL, "plan was built with HF_PLAN_HOST_ONLY: it has no device copy");
  if (slot_bytes == 0 || slot_bytes % 4) return fail(HF_EINVAL, "slot_bytes must be a positive multiple of 4");
  if ((reinterpret_cast<uintptr_t>(resp_in) | reinterpret_cast<uintptr_t>(resp_out)) % 256)
    return fail(HF_EINVAL, "resp_in and resp_out must be 256-byte aligned");
  const char *a = static_cast<const char *>(resp_in), *b = static_cast<const char *>(resp_out);
  const size_t in_bytes = (size_t)p.N * slot_bytes, out_bytes = in_bytes * p.dg;
  if (a < b + out_bytes && b < a + in_bytes) return fail(HF_EINVAL, "resp_in and resp_out overlap");
  if (!p.d_gather_out) return not_resident();
  const int e = hf::launch_gather_slots(p.d_gather_out, (uint32_t)p.N, (uint32_t)p.dg, resp_in, resp_out, slot_bytes, hip_stream);
  if (e == (int)hipErrorInvalidValue) return fail(HF_ERANGE, "slots too large for one launch");
  if (e != 0) return fail(HF_EHIP, std::string("kernel launch: ") + hipGetErrorString(static_cast<hipError_t>(e)));
  return HF_OK;
}

int hf_plan_micro_dp_peer(const hf_plan *plan, int rank, int j) {
  if (!plan || rank < 0 || rank >= plan->p.N || j < 0 || j >= plan->p.dg) return -1;
  return plan->p.micro_peers[(size_t)rank * plan->p.dg + j];
}

int hf_plan_set_param(hf_plan *plan, int param, int64_t value) {
  if (!plan) return fail(HF_EINVAL, "null plan");
  hf::Plan &p = plan->p;
  switch (param) {
  case HF_PARAM_TILE_BYTES:
    return retile(p, p.tile_bytes, value);
  case HF_PARAM_GRID_WGS:
    if (value < 1 || value > 65536) return fail(HF_EINVAL, "grid workgroups must be in [1, 65536]");
    p.grid_wgs = value;
    return HF_OK;
  case HF_PARAM_VARIANT:
    if (value < HF_VARIANT_PERSISTENT || value > HF_VARIANT_PARTS) return fail(HF_EINVAL, "unknown kernel variant");
    p.variant = value;
    return HF_OK;
  case HF_PARAM_MULTICAST: {
    if (value < HF_MULTICAST_AUTO || value > HF_MULTICAST_PREFETCHED) return fail(HF_EINVAL, "unknown multicast mode");
    const OnDevice there(p.device); // the plan's other lists are on it
    if (there.e != hipSuccess) return fail(HF_EHIP, std::string("the plan's device: ") + hipGetErrorString(there.e));
    if (int rc = set_multicast(p, value)) return rc;
    p.serial = g_next_serial++;
    if (!(p.flags & HF_PLAN_HOST_ONLY)) return upload_forward_list(p);
    return HF_OK;
  }
  case HF_PARAM_OFFLOAD_WGS:
    if (value < 1 || value > 4096) return fail(HF_EINVAL, "offload workgroups must be in [1, 4096]");
    p.offload_wgs = value;
    return HF_OK;
  case HF_PARAM_PREFETCH_BLOCK_BYTES:
    if (value < (1 << 20) || value > (64 << 20)) return fail(HF_EINVAL, "prefetch block must be in [1 MiB, 64 MiB]");
    return retile(p, p.prefetch_block_bytes, value);
  case HF_PARAM_PREFETCH_MERGE:
    if (value < 0 || value > HF_MAX_PREFETCH_CHUNKS) return fail(HF_EINVAL, "prefetch merge must be in [0, 8]");
    return retile(p, p.prefetch_merge, value);
  case HF_PARAM_ROW_INTERLEAVE:
    if (value != 0 && value != 1) return fail(HF_EINVAL, "row interleave must be 0 or 1");
    return retile(p, p.row_interleave, value);
  case HF_PARAM_MC_BLOCK_BYTES:
    if (value < (1 << 20) || value > (1ll << 30)) return fail(HF_EINVAL, "multicast block must be in [1 MiB, 1 GiB]");
    return retile(p, p.mc_block_bytes, value);
  case HF_PARAM_MAX_WGS_PER_LAUNCH:
    if (value < 1024 || value > 0xFFFFFFFFll / 256) return fail(HF_EINVAL, "workgroups per launch must be in [1024, 16777215]");
    p.max_wgs_per_launch = value;
    return HF_OK;
  case HF_PARAM_WG_THREADS:
    if (value != 0 && value != 64 && value != 256) return fail(HF_EINVAL, "workgroup size must be 0 (automatic), 64 or 256");
    p.wg_threads = value;
    return HF_OK;
  case HF_PARAM_CACHE_POLICY:
    if (value < -1 || value > 5) return fail(HF_EINVAL, "cache policy must be in [-1, 5]");
    p.cache_policy = value;
    return HF_OK;
  case HF_PARAM_PART_BYTES:
    if (value != 0 && value != 1024 && value != 2048 && value != 4096 && value != 8192 && value != 16384 && value != 32768)
      return fail(HF_EINVAL, "part bytes must be 0 (automatic) or a power of two from 1024 to 32768");
    p.part_bytes = value;
    return HF_OK;
  }
  return fail(HF_EINVAL, "unknown parameter");
}

int hf_debug_restrict_kinds(hf_plan *plan, int kind_mask) {
  if (!plan) return fail(HF_EINVAL, "null plan");
  if (kind_mask < 1 || kind_mask > 0x1F) return fail(HF_EINVAL, "kind mask must be in [1, 31]");
  return retile(plan->p, plan->p.kind_mask, kind_mask);
}

int64_t hf_plan_get_param(const hf_plan *plan, int param) {
  if (!plan) return -1;
  switch (param) {
  case HF_PARAM_TILE_BYTES: return plan->p.tile_bytes;
  case HF_PARAM_GRID_WGS: return plan->p.grid_wgs;
  case HF_PARAM_VARIANT: return plan->p.variant;
  case HF_PARAM_MULTICAST: return plan->p.effective_multicast();
  case HF_PARAM_MC_BLOCK_BYTES: return plan->p.mc_block_bytes;
  case HF_PARAM_OFFLOAD_WGS: return plan->p.offload_wgs;
  case HF_PARAM_ROW_INTERLEAVE: return plan->p.row_interleave;
  case HF_PARAM_PREFETCH_BLOCK_BYTES: return plan->p.prefetch_block_bytes;
  case HF_PARAM_PREFETCH_MERGE: return plan->p.effective_prefetch_merge();
  case HF_PARAM_WG_THREADS: return plan->p.wg_threads;
  case HF_PARAM_MAX_WGS_PER_LAUNCH: return plan->p.max_wgs_per_launch;
  case HF_PARAM_CACHE_POLICY: return plan->p.cache_policy;
  case HF_PARAM_PART_BYTES: return plan->p.part_bytes;
  case HF_PARAM_AUTOMATIC_LIST: return plan->p.runs_auto() ? (int64_t)plan->p.dev_auto.tiles.size() : 0;
  }
  return -1;
}

size_t hf_plan_train_bytes(const hf_plan *plan) { return plan ? plan->p.train_bytes : 0; }
size_t hf_plan_gen_bytes(const hf_plan *plan) { return plan ? plan->p.gen_bytes : 0; }
int hf_plan_num_ranks(const hf_plan *plan) { return plan ? plan->p.N : 0; }
int hf_plan_num_mat(const hf_plan *plan) { return plan ? (int)plan->p.mat.size() : 0; }
int hf_plan_mat_rank(const hf_plan *plan, int i) {
  return (plan && i >= 0 && i < (int)plan->p.mat.size()) ? plan->p.mat[i] : -1;
}
int hf_plan_micro_dp_size(const hf_plan *plan) { return plan ? plan->p.dg : 0; }

size_t hf_plan_rank_train_offset(const hf_plan *plan, int rank) {
  if (!plan || rank < 0 || rank >= plan->p.N) return (size_t)-1;
  return plan->p.train_tab[rank].base;
}

size_t hf_plan_rank_gen_offset(const hf_plan *plan, int rank) {
  if (!plan || rank < 0 || rank >= plan->p.N || plan->p.mat_pos[rank] < 0) return (size_t)-1;
  return plan->p.gen_tab[rank].base;
}

int hf_plan_rank_coords(const hf_plan *plan, int rank, int32_t out[6]) {
  if (!plan || !out) return fail(HF_EINVAL, "null argument");
  if (rank < 0 || rank >= plan->p.N) return fail(HF_ERANGE, "rank out of range");
  const hf::Coords &c = plan->p.coords[rank];
  out[0] = c.dp; out[1] = c.pp; out[2] = c.tp; out[3] = c.gpp; out[4] = c.gtp; out[5] = c.micro;
  return HF_OK;
}

size_t hf_plan_num_tensors(const hf_plan *plan, int which_buf, int rank) {
  if (!plan || rank < 0 || rank >= plan->p.N) return 0;
  if (which_buf == HF_BUF_TRAIN) return plan->p.train_tab[rank].tensors.size();
  if (which_buf == HF_BUF_GEN && plan->p.mat_pos[rank] >= 0) return plan->p.gen_tab[rank].tensors.size();
  return 0;
}

int hf_plan_get_tensor(const hf_plan *plan, int which_buf, int rank, size_t i, hf_tensor_info *out) {
  if (!plan || !out) return fail(HF_EINVAL, "null argument");
  if (which_buf != HF_BUF_TRAIN && which_buf != HF_BUF_GEN) return fail(HF_EINVAL, "which_buf must be HF_BUF_TRAIN or HF_BUF_GEN");
  if (rank < 0 || rank >= plan->p.N) return fail(HF_ERANGE, "rank out of range");
  if (which_buf == HF_BUF_GEN && plan->p.mat_pos[rank] < 0) return fail(HF_ERANGE, "rank has no generation buffer");
  const hf::RankTable &tab = which_buf == HF_BUF_TRAIN ? plan->p.train_tab[rank] : plan->p.gen_tab[rank];
  if (i >= tab.tensors.size()) return fail(HF_ERANGE, "tensor index past the end");
  const hf::TensorRec &t = tab.tensors[i];
  const hf::Coords &c = plan->p.coords[rank];
  const bool repl = t.id == HF_T_LN1 || t.id == HF_T_LN2 || t.id == HF_T_LNF || t.id == HF_G_LN1 || t.id == HF_G_LN2 || t.id == HF_G_LNF;
  out->tensor_id = t.id;
  out->layer = t.layer;
  out->rows = t.rows;
  out->cols = t.cols;
  out->offset = tab.base + t.off;
  out->tp_index = repl ? 0 : (which_buf == HF_BUF_TRAIN ? c.tp : c.gtp);
  out->replicated = repl ? 1 : 0;
  return HF_OK;
}

static const hf_desc *desc_at(const hf::Plan &p, int direction, size_t i) {
  if (direction == HF_DIR_TRAIN_TO_GEN) {
    if (i < p.fwd_peer.size()) return &p.fwd_peer[i];
    i -= p.fwd_peer.size();
    if ((p.flags & HF_COPY_OWN) && i < p.fwd_own.size()) return &p.fwd_own[i];
    return nullptr;
  }
  if (direction == HF_DIR_GEN_TO_TRAIN && i < p.back.size()) return &p.back[i];
  if ((direction == HF_DIR_OFFLOAD || direction == HF_DIR_RELOAD) && i < p.remote.size()) return &p.remote[i];
  return nullptr;
}

size_t hf_plan_num_desc(const hf_plan *plan, int direction) {
  if (!plan) return 0;
  const hf::Plan &p = plan->p;
  if (direction == HF_DIR_TRAIN_TO_GEN) return p.fwd_peer.size() + ((p.flags & HF_COPY_OWN) ? p.fwd_own.size() : 0);
  if (direction == HF_DIR_GEN_TO_TRAIN) return p.back.size();
  if (direction == HF_DIR_OFFLOAD || direction == HF_DIR_RELOAD) return p.remote.size();
  return 0;
}

int hf_plan_get_desc(const hf_plan *plan, int direction, size_t i, hf_desc *out) {
  if (!plan || !out) return fail(HF_EINVAL, "null argument");
  const hf_desc *d = desc_at(plan->p, direction, i);
  if (!d) return fail(HF_ERANGE, "no such descriptor");
  *out = *d;
  if (direction == HF_DIR_RELOAD) {
    std::swap(out->src_off, out->dst_off);
    std::swap(out->src_block_stride, out->dst_block_stride);
    std::swap(out->src_row_stride, out->dst_row_stride);
  }
  return HF_OK;
}

// totals are cached when the work lists are built
size_t hf_plan_bytes_moved(const hf_plan *plan, int direction) {
  if (!plan) return 0;
  if (direction == HF_DIR_TRAIN_TO_GEN || direction == HF_DIR_GEN_TO_TRAIN) return plan->p.moved_bytes[direction];
  if (direction == HF_DIR_OFFLOAD || direction == HF_DIR_RELOAD) {
    size_t total = 0;
    for (const hf_desc &d : plan->p.remote) total += hf::desc_bytes(d);
    return total;
  }
  return 0;
}

size_t hf_plan_unique_src_bytes(const hf_plan *plan, int direction) {
  if (!plan) return 0;
  if (direction == HF_DIR_TRAIN_TO_GEN || direction == HF_DIR_GEN_TO_TRAIN) return plan->p.unique_bytes[direction];
  return hf_plan_bytes_moved(plan, direction); // the image holds every remote piece once
}

size_t hf_plan_num_own_view(const hf_plan *plan, int rank) {
  if (!plan || rank < 0 || rank >= plan->p.N) return 0;
  size_t n = 0;
  for (const hf_desc &d : plan->p.fwd_own) n += d.dst_rank == rank;
  return n;
}

int hf_plan_get_own_view(const hf_plan *plan, int rank, size_t i, hf_desc *out) {
  if (!plan || !out) return fail(HF_EINVAL, "null argument");
  if (rank < 0 || rank >= plan->p.N) return fail(HF_ERANGE, "rank out of range");
  for (const hf_desc &d : plan->p.fwd_own)
    if (d.dst_rank == rank && i-- == 0) {
      *out = d;
      return HF_OK;
    }
  return fail(HF_ERANGE, "no such own-view entry");
}

size_t hf_plan_num_tiles(const hf_plan *plan, int direction) {
  if (!plan) return 0;
  const hf::Plan &p = plan->p;
  if (direction == HF_DIR_TRAIN_TO_GEN) return p.active_fwd_count();
  if (direction == HF_DIR_GEN_TO_TRAIN) return p.tiles_back.size();
  if (direction == HF_DIR_OFFLOAD) return p.tiles_offload.size();
  if (direction == HF_DIR_RELOAD) return p.tiles_reload.size();
  return 0;
}

int hf_plan_get_tile(const hf_plan *plan, int direction, size_t i, hf_tile *out) {
  if (!plan || !out) return fail(HF_EINVAL, "null argument");
  if (i >= hf_plan_num_tiles(plan, direction)) return fail(HF_ERANGE, "no such tile");
  const hf::Plan &p = plan->p;
  *out = direction == HF_DIR_GEN_TO_TRAIN                    ? p.tiles_back[i]
         : direction == HF_DIR_OFFLOAD                           ? p.tiles_offload[i]
         : direction == HF_DIR_RELOAD                            ? p.tiles_reload[i]
                                                                 : p.active_fwd()[i];
  return HF_OK;
}

int hf_plan_get_tile_dst(const hf_plan *plan, int direction, size_t i, uint32_t k, uint64_t *out) {
  hf_tile tl;
  if (!out) return fail(HF_EINVAL, "null argument");
  if (int rc = hf_plan_get_tile(plan, direction, i, &tl)) return rc;
  if (k >= tl.n_dst) return fail(HF_ERANGE, "no such destination");
  *out = k == 0 ? tl.dst_off : plan->p.mc_dst[tl.dst_list + k - 1];
  return HF_OK;
}

int hf_calib_copy(const void *src, void *dst, size_t bytes, void *hip_stream) {
  if (!src && !dst) return fail(HF_EINVAL, "null buffers");
  if (bytes % 16 || (reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) % 16)
    return fail(HF_EINVAL, "calibration copy needs 16-byte aligned pointers and size");
  const char *s = static_cast<const char *>(src), *d = static_cast<const char *>(dst);
  if (s && d && s < d + bytes && d < s + bytes) return fail(HF_EINVAL, "calibration copy: buffers overlap");
  const int e = hf::launch_calib_copy(src, dst, bytes, hip_stream);
  if (e != 0) return fail(HF_EHIP, std::string("kernel launch: ") + hipGetErrorString(static_cast<hipError_t>(e)));
  return HF_OK;
}

int hf_calib_fanout(const void *src, void *dst, size_t bytes, int n_dst, size_t dst_stride, int method, size_t block_bytes,
                    int wg_bytes, void *hip_stream) {
  if (!src && !dst) return fail(HF_EINVAL, "null buffers");
  if (method < HF_FANOUT_REGISTERS || method > HF_FANOUT_PREFETCHED) return fail(HF_EINVAL, "unknown fan-out method");
  if ((!src || !dst) && method != HF_FANOUT_REGISTERS) return fail(HF_EINVAL, "fan-out copy: blocks need both a source and destinations");
  if (method != HF_FANOUT_REGISTERS && block_bytes == 0) return fail(HF_EINVAL, "fan-out copy: this method needs a block size");
  if (n_dst < 1 || n_dst > 8) return fail(HF_EINVAL, "n_dst must be in [1, 8]");
  if (wg_bytes != 1024 && wg_bytes != 4096 && wg_bytes != 8192) return fail(HF_EINVAL, "wg_bytes must be 1024, 4096 or 8192");
  if (bytes == 0 || bytes % 8192 || dst_stride % 256 || dst_stride < bytes || block_bytes % 65536 ||
      (reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) % 256)
    return fail(HF_EINVAL, "fan-out copy: sizes or alignment out of contract");
  const char *s0 = static_cast<const char *>(src), *d0 = static_cast<const char *>(dst);
  const size_t span = (size_t)(n_dst - 1) * dst_stride + bytes;
  if (s0 && d0 && s0 < d0 + span && d0 < s0 + bytes) return fail(HF_EINVAL, "fan-out copy: buffers overlap");
  const int e = hf::launch_calib_fanout(src, dst, bytes, n_dst, dst_stride, method, block_bytes, wg_bytes, hip_stream);
  if (e == (int)hipErrorInvalidValue) return fail(HF_ERANGE, "fan-out copy: too many workgroups for one launch");
  if (e != 0) return fail(HF_EHIP, std::string("kernel launch: ") + hipGetErrorString(static_cast<hipError_t>(e)));
  return HF_OK;
}

int hf_plan_validate(const hf_plan *plan) {
  if (!plan) return fail(HF_EINVAL, "null plan");
  std::string err;
  int rc;
  try {
    rc = hf::validate_plan(plan->p, err);
  } catch (const std::bad_alloc &) {
    rc = HF_ENOMEM;
    err = "out of host memory while validating";
  }
  return rc == HF_OK ? HF_OK : fail(rc, err);
}

const char *hf_last_error(void) { return g_err.c_str(); }
const char *hf_version(void) { return "hfreshard 0.1 (gfx950)"; }

} // extern "C"
