// Host-only driver: the ABI's own code (abi.hip, compiled as plain C++) over a stand-in for the HIP
// runtime that can refuse an allocation or a copy, over host memory that can run out, and launch entry points that launch nothing but
// look at what they are given.
#define HIP_SYMBOL(x) (x)
#define __align__(n) __attribute__((aligned(n)))
#include <cstdio>
#include <cstdlib>
#include <map>

#include "abi.hip"

namespace {

int g_device_calls_left = -1; // allocations and uploads until one fails; -1 = none fails
long g_host_allocations_left = -1; // the same for operator new
std::map<const char *, size_t> g_device; // what hipMalloc has handed out
int g_current = 0;                       // device of the calls
std::map<const char *, int> g_device_of; // the device of an allocation
int g_device_calls = 0;            // made so far: allocations, uploads and frees
int g_launches = 0, g_bad_launches = 0;
const void *g_last_list = nullptr;

bool refuse() { ++g_device_calls; return g_device_calls_left >= 0 && g_device_calls_left-- == 0; }
bool on_device(const void *p, size_t bytes) {
  auto it = g_device.upper_bound(static_cast<const char *>(p));
  return it != g_device.begin() && (--it, static_cast<const char *>(p) + bytes <= it->first + it->second);
}

#define REQUIRE(c)                                                                              \
  do {                                                                                          \
    if (!(c)) { std::printf("line %d: %s (%s)\n", __LINE__, #c, hf_last_error()); return false; } \
  } while (0)

} // namespace

// the linker puts this in the place of operator new (--wrap)
extern "C" void *__real__Znwm(size_t n);
extern "C" void *__wrap__Znwm(size_t n) {
  if (g_host_allocations_left >= 0 && g_host_allocations_left-- == 0) throw std::bad_alloc();
  return __real__Znwm(n);
}

extern "C" {
hipError_t hipGetDevice(int *d) { *d = g_current; return hipSuccess; }
hipError_t hipSetDevice(int d) { g_current = d; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) {
  if (refuse()) return hipErrorOutOfMemory;
  *p = std::malloc(n);
  const long left = g_host_allocations_left; // what is noted here is not the library's
  g_host_allocations_left = -1;
  g_device[static_cast<char *>(*p)] = n;
  g_device_of[static_cast<char *>(*p)] = g_current;
  g_host_allocations_left = left;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  ++g_device_calls;
  g_device.erase(static_cast<char *>(p));
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void *dst, const void *src, size_t n, hipMemcpyKind) {
  if (refuse()) return hipErrorUnknown;
  std::memcpy(dst, src, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(dst, src, n);
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *symbol) {
  *p = const_cast<void *>(symbol);
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *at, const void *p) {
  at->type = hipMemoryTypeHost;
  at->devicePointer = const_cast<void *>(p);
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t *, size_t *, hipDeviceptr_t) { return hipErrorNotFound; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in"; }
}

namespace hf {
int launch_tiles(const DevTile *tiles, size_t n, const uint64_t *extra_dst, const void *, void *, int, int, int, uint32_t, uint32_t, uint32_t, int,
                 int, void *) {
  ++g_launches;
  g_last_list = tiles;
  bool staged = reinterpret_cast<const unsigned char *>(tiles) >= scratch && reinterpret_cast<const unsigned char *>(tiles + n) <= scratch + sizeof scratch;
  bool ok = n == 0 || staged || on_device(tiles, n * sizeof *tiles);
  for (size_t i = 0; ok && i < n; ++i)
    if (!(tiles[i].n_dst & kLoadOnly) && tiles[i].n_dst > 1) ok = extra_dst && (staged || on_device(extra_dst + tiles[i].dst_list, (tiles[i].n_dst - 1) * 8));
  g_bad_launches += !ok;
  return 0;
}
int launch_gather_slots(const uint32_t *out_slots, uint32_t n_slots, uint32_t n_dst, const void *, void *, size_t, void *) {
  ++g_launches;
  g_bad_launches += !on_device(out_slots, (size_t)n_slots * n_dst * 4);
  return 0;
}
int launch_calib_copy(const void *, void *, size_t, void *) { return 0; }
int launch_calib_fanout(const void *, void *, size_t, int, size_t, int, size_t, int, void *) { return 0; }
} // namespace hf

namespace {

char *const kTrain = reinterpret_cast<char *>(1ull << 40), *const kGen = reinterpret_cast<char *>(2ull << 40); // never read

// every execution call of the plan; true = none was launched on a list that is not there
bool run_all(hf_plan *pl, int &refused) {
  refused = 0;
  const int launched = g_launches;
  for (int rc : {hf_reshard_execute(pl, kTrain, kGen, nullptr), hf_reshard_install_own(pl, kTrain, kGen, nullptr),
                 hf_reshard_back(pl, kTrain, kGen, nullptr), hf_offload_remote(pl, kGen, kTrain, nullptr),
                 hf_reload_remote(pl, kTrain, kGen, nullptr), hf_gather_responses(pl, kTrain, kGen, 4096, nullptr)}) {
    REQUIRE(rc == HF_OK || rc == HF_EHIP);
    refused += rc != HF_OK;
  }
  REQUIRE(g_bad_launches == 0 && g_launches - launched == 6 - refused);
  return true;
}

// A parameter change whose upload fails at any point leaves calls that are refused, not launches on lists
// that are not there; the next change that succeeds makes them run again.
bool failed_uploads() {
  const hf_model_desc m{2, 256, 4, 4, 64, 688, 1024, 2, 0};
  const hf_gen_layout gl{1, 1, HF_PLAN_OFFLOAD, nullptr, 0};
  const hf_train_layout tl{1, 4, 1};
  for (int mode = HF_MULTICAST_OFF; mode <= HF_MULTICAST_PREFETCHED; ++mode)
    for (int change = 0; change < 2; ++change) {
      hf_plan *pl = nullptr;
      REQUIRE(hf_reshard_plan(&m, &tl, &gl, &pl) == HF_OK);
      int refused, failures = 0;
      REQUIRE(run_all(pl, refused) && refused == 0);
      for (int at = 0;; ++at) {
        g_device_calls_left = at;
        const int rc = change ? hf_plan_set_param(pl, HF_PARAM_TILE_BYTES, 8192) : hf_plan_set_param(pl, HF_PARAM_MULTICAST, mode);
        g_device_calls_left = -1;
        REQUIRE(run_all(pl, refused) && (refused > 0) == (rc != HF_OK));
        if (rc == HF_OK) break;
        ++failures;
        REQUIRE(hf_plan_set_param(pl, HF_PARAM_TILE_BYTES, 65536) == HF_OK && hf_plan_set_param(pl, HF_PARAM_MULTICAST, mode) == HF_OK);
        REQUIRE(run_all(pl, refused) && refused == 0);
      }
      REQUIRE(failures >= 2);
      hf_plan_destroy(pl);
      REQUIRE(g_device.empty());
    }
  return true;
}

// Variant, workgroup size, part size and cache policy choose which list hf_reshard_execute runs, and are fields of the plan: they
// touch no device memory, so that none can fail, and a captured graph keeps the list that it holds.
bool launch_parameters() {
  const hf_model_desc m{2, 256, 4, 4, 64, 688, 1024, 2, 0};
  const hf_gen_layout gl{1, 1, HF_PLAN_OFFLOAD, nullptr, 0};
  const hf_train_layout tl{1, 4, 1};
  const struct { int param; int64_t named, automatic; } params[] = {{HF_PARAM_VARIANT, HF_VARIANT_PERSISTENT, HF_VARIANT_PARTS},
                                                                    {HF_PARAM_WG_THREADS, 64, 0}, {HF_PARAM_PART_BYTES, 2048, 0},
                                                                    {HF_PARAM_CACHE_POLICY, 3, -1}};
  hf_plan *pl = nullptr;
  REQUIRE(hf_reshard_plan(&m, &tl, &gl, &pl) == HF_OK);
  REQUIRE(hf_reshard_execute(pl, kTrain, kGen, nullptr) == HF_OK && g_bad_launches == 0);
  const void *automatic = g_last_list, *named = nullptr;
  const size_t bytes = pl->p.dev_auto.tiles.size() * sizeof(hf::DevTile);
  int refused;
  for (const auto &c : params) {
    const int calls = g_device_calls;
    g_device_calls_left = 0;
    const int there = hf_plan_set_param(pl, c.param, c.named);
    REQUIRE(hf_reshard_execute(pl, kTrain, kGen, nullptr) == HF_OK && g_bad_launches == 0 && g_last_list != automatic);
    REQUIRE(!named || g_last_list == named);
    named = g_last_list;
    const bool kept = on_device(automatic, bytes);
    const int back = hf_plan_set_param(pl, c.param, c.automatic);
    REQUIRE(hf_reshard_execute(pl, kTrain, kGen, nullptr) == HF_OK && g_bad_launches == 0 && g_last_list == automatic);
    g_device_calls_left = -1;
    REQUIRE(there == HF_OK && back == HF_OK && kept && g_device_calls == calls);
    REQUIRE(run_all(pl, refused) && refused == 0);
  }
  hf_plan_destroy(pl);
  REQUIRE(g_device.empty());
  return true;
}

// A plan stays on the device that it was built on when a mode is named while another device is current.
bool another_device_current() {
  const hf_model_desc m{2, 256, 4, 4, 64, 688, 1024, 2, 0};
  const hf_gen_layout gl{1, 1, 0, nullptr, 0};
  const hf_train_layout tl{1, 4, 1};
  hf_plan *pl = nullptr;
  g_current = 1;
  REQUIRE(hf_reshard_plan(&m, &tl, &gl, &pl) == HF_OK);
  for (int mode = HF_MULTICAST_AUTO; mode <= HF_MULTICAST_PREFETCHED; ++mode) {
    g_current = 0;
    REQUIRE(hf_plan_set_param(pl, HF_PARAM_MULTICAST, mode) == HF_OK && g_current == 0);
    REQUIRE(hf_reshard_execute(pl, kTrain, kGen, nullptr) == HF_EINVAL);
    for (const auto &a : g_device) REQUIRE(g_device_of.at(a.first) == 1);
    g_current = 1;
    REQUIRE(hf_reshard_execute(pl, kTrain, kGen, nullptr) == HF_OK && g_bad_launches == 0);
  }
  hf_plan_destroy(pl);
  g_current = 0;
  REQUIRE(g_device.empty());
  return true;
}

// What the plan says of itself: every parameter, and every tile of every list with its destinations.
std::string state_of(const hf_plan *pl) {
  std::string s;
  for (int k = 0; k <= HF_PARAM_PREFETCH_MERGE; ++k) s += std::to_string(hf_plan_get_param(pl, k)) + " ";
  for (int dir = 0; dir < 4; ++dir)
    for (size_t i = 0; i < hf_plan_num_tiles(pl, dir); ++i) {
      hf_tile t;
      uint64_t at = 0;
      hf_plan_get_tile(pl, dir, i, &t);
      s.append(reinterpret_cast<const char *>(&t), sizeof t);
      for (uint32_t k = 0; k < t.n_dst; ++k) {
        hf_plan_get_tile_dst(pl, dir, i, k, &at);
        s.append(reinterpret_cast<const char *>(&at), sizeof at);
      }
    }
  return s + std::to_string(hf_plan_bytes_moved(pl, 0)) + " " + std::to_string(hf_plan_unique_src_bytes(pl, 0));
}

// A parameter change that finds no host memory, or whose value is refused, leaves the plan as it was.
bool failed_changes() {
  const hf_model_desc m{2, 256, 4, 4, 64, 688, 1024, 2, 0};
  const hf_gen_layout gl{1, 1, HF_PLAN_OFFLOAD, nullptr, 0};
  const hf_train_layout tl{1, 4, 1};
  hf_plan *pl = nullptr;
  REQUIRE(hf_reshard_plan(&m, &tl, &gl, &pl) == HF_OK);
  const std::string before = state_of(pl);
  const struct { int param; int64_t value; } changes[] = {{HF_PARAM_TILE_BYTES, 65536}, {HF_PARAM_MC_BLOCK_BYTES, 4 << 20},
                                                          {HF_PARAM_PREFETCH_BLOCK_BYTES, 1 << 20}, {HF_PARAM_PREFETCH_MERGE, 4},
                                                          {HF_PARAM_ROW_INTERLEAVE, 0}, {HF_PARAM_MULTICAST, HF_MULTICAST_CACHE_BLOCKED}, {-1, 3}};
  int refused, failures = 0;
  for (const auto &c : changes)
    for (long at = 0;; at += 1 + at / 8) {
      g_host_allocations_left = at;
      const int rc = c.param < 0 ? hf_debug_restrict_kinds(pl, (int)c.value) : hf_plan_set_param(pl, c.param, c.value);
      const bool ran_out = g_host_allocations_left < 0;
      g_host_allocations_left = -1;
      REQUIRE(ran_out == (rc == HF_ENOMEM) && (ran_out || rc == HF_OK));
      if (!ran_out) { // back again
        hf_plan_destroy(pl);
        REQUIRE(hf_reshard_plan(&m, &tl, &gl, &pl) == HF_OK);
        break;
      }
      ++failures;
      REQUIRE(state_of(pl) == before && run_all(pl, refused) && refused == 0);
    }
  REQUIRE(failures > 50);
  REQUIRE(hf_plan_set_param(pl, HF_PARAM_TILE_BYTES, 4095) == HF_EINVAL && state_of(pl) == before);
  REQUIRE(run_all(pl, refused) && refused == 0);
  hf_plan_destroy(pl);
  return true;
}

// The limit of hf_reshard_execute_static counts payload.  Lists of odd rows that it admits run, whatever
// their records come to; what is staged stays inside the array (the sanitizer watches its end).
bool static_limit() {
  struct { hf_model_desc m; hf_train_layout tl; hf_gen_layout gl; int64_t mode, tile; int kinds; uint64_t counted; bool own_form; } cases[] = {
      // rows of 1260 bytes: 18.0 MB of tiles as the lists have them, 16.3 by payload
      {{24, 768, 32, 16, 80, 2520, 11004, 2, 0}, {4, 4, 1}, {1, 2, HF_PLAN_HOST_ONLY, nullptr, 0}, HF_MULTICAST_PREFETCHED, 4096, 0x1F, 16272960, false},
      {{24, 768, 32, 16, 80, 2520, 11004, 2, 0}, {4, 4, 1}, {1, 2, HF_PLAN_HOST_ONLY | HF_COPY_OWN, nullptr, 0}, HF_MULTICAST_REGISTERS, 4096, 0x1F, 15509344, false},
      // rows just below the tile size, two records each: 27 MB of records
      {{60, 1024, 4, 4, 8, 4 * 2045, 4, 2, 0}, {1, 4, 1}, {1, 1, HF_PLAN_HOST_ONLY, nullptr, 0}, HF_MULTICAST_REGISTERS, 4096, 1 << HF_ROW, 0, true},
      // and over the limit
      {{64, 1024, 4, 4, 8, 4 * 2045, 4, 2, 0}, {1, 4, 1}, {1, 1, HF_PLAN_HOST_ONLY, nullptr, 0}, HF_MULTICAST_REGISTERS, 4096, 1 << HF_ROW, ~0ull, false}};
  for (const auto &c : cases) {
    hf_plan *pl = nullptr;
    REQUIRE(hf_reshard_plan(&c.m, &c.tl, &c.gl, &pl) == HF_OK);
    REQUIRE(hf_debug_restrict_kinds(pl, c.kinds) == HF_OK && hf_plan_set_param(pl, HF_PARAM_TILE_BYTES, c.tile) == HF_OK);
    REQUIRE(hf_plan_set_param(pl, HF_PARAM_MULTICAST, c.mode) == HF_OK && hf_plan_set_param(pl, HF_PARAM_PREFETCH_MERGE, 8) == HF_OK);
    const hf::DevList &list = c.own_form ? pl->p.dev_static : pl->p.dev_fwd;
    const int rc = hf_reshard_execute_static(pl, kTrain, kGen, nullptr);
    if (c.counted == ~0ull) {
      REQUIRE(rc == HF_ERANGE && pl->p.static_bytes > HF_STATIC_SCRATCH_BYTES);
    } else {
      REQUIRE(rc == HF_OK && g_bad_launches == 0 && g_last_list == scratch);
      REQUIRE(c.own_form == !pl->p.dev_static.tiles.empty() && (!c.counted || pl->p.static_bytes == c.counted));
      REQUIRE(!std::memcmp(scratch, list.tiles.data(), list.tiles.size() * sizeof(hf::DevTile)));
    }
    hf_plan_destroy(pl);
  }
  return true;
}

} // namespace

int main() {
  if (!static_limit() || !failed_uploads() || !launch_parameters() || !another_device_current() || !failed_changes()) return 1;
  std::printf("ok\n");
  return 0;
}
