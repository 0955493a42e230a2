// gfx950 copy kernels that execute a reshard plan's tile list.
//
// The work is pure data movement (HybridFlow Section 5.2 steps 1 and 4 re-arrange
// parameters, they compute nothing), so the kernels are shaped for HBM bandwidth and use
// no MFMA and, in the default path, no LDS.  Every lane moves slots of 16 bytes, whatever the
// alignment of the rows (slots.hpp), so a wavefront touches 1 KiB of consecutive bytes per
// instruction.  Measured against accesses of 8, 4 or 2 bytes for rows that are no more aligned
// (Llama-like shape, hidden 768, rows of 1026 bytes in a quarter of the bytes, 1.4 GB moved):
// 252 against 357 us for the whole transition; in the other direction on a small shape with rows of
// 690 bytes (89 MB) 16.7 against 28.2 us, together with records cut to fit (below).
//
// Where pieces are shared and every choice is the library's, reshard_auto runs a list of its own (below).
// Otherwise, and for the lists with one destination per piece, reshard_parts: the list's records (up to 128 KiB each) are cut into parts
// of 1 to 8 KiB and every part gets its own short-lived workgroup of 64 or 256 lanes,
// which loads its one or two slots per lane, stores them and exits.  The hardware
// dispatcher hands out workgroups in index order, so the chip works on one narrow window
// of source and destination addresses that moves through the list, and a slow CU simply
// takes fewer workgroups.  One training piece wanted by several ranks of a micro-DP group
// (Section 5.3) is served by records that name several destinations (loaded once, stored to
// each), by default with load-only records in front of every block of the list that bring the
// block into the L2 of the XCD that will copy it (prefetched list), or by listing its tiles
// once per destination in an order that lets L2 serve the re-reads (cache-blocked list).
//
// Kept beside it, selectable per plan, for measurements: persistent workgroups that stride
// over the tile list, the same with one wavefront per stride (wavefront-level dispatch),
// the same staged through LDS, and one workgroup per tile.  The persistent kernel and
// reshard_link also carry the offload / reload of the remote pieces, where the host link is the
// bound and few workgroups are wanted.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "hfreshard.h"
#include "kernels.hpp"

namespace hf {

namespace {

constexpr int kWG = 256;    // threads per workgroup = 4 wavefronts of 64
constexpr int kWave = 64;

constexpr int kMaxUnroll = 8;  // independent accesses in flight per lane (persistent kernels)

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_any __attribute__((aligned(2))); // the same 16 bytes at any even address

// Cache policy of the streaming accesses: bit 0 = plain (temporal) loads instead of
// non-temporal ones; bit 1 = plain stores; bit 2 = non-temporal stores through the
// compiler builtin (`nt`) instead of the default `sc0 sc1 nt` (system-scope, streaming)
// 16-byte store.  Every byte is touched once, so nothing is worth keeping in L2 except the
// source block of the cache-blocked multicast list (plain loads there).  Measured on a
// one-shot 1:1 copy of 8 GiB: stores `sc0 sc1 nt` 6.74 TB/s vs `nt` 6.66 TB/s with 64-lane
// workgroups, 6.66 vs 6.42 TB/s with 256-lane workgroups; plain stores 6.55 / 6.37 TB/s.
// The addresses need not be aligned (slots at either end of an odd row are not).
template <int kPolicy> __device__ __forceinline__ u32x4 load_stream(const char *p) {
  if constexpr (kPolicy & 1) return *reinterpret_cast<const u32x4_any *>(p);
  else return __builtin_nontemporal_load(reinterpret_cast<const u32x4_any *>(p));
}
template <int kPolicy> __device__ __forceinline__ void store_stream(char *p, u32x4 v) {
  if constexpr (kPolicy & 2) {
    *reinterpret_cast<u32x4_any *>(p) = v;
  } else if constexpr (!(kPolicy & 4)) {
    // a vector store like any other to the hardware; the compiler's own wait counts stay
    // correct because an extra outstanding store can only make its vmcnt waits longer.  The
    // compiler does not see a memory instruction here, so the wait state gfx9 wants between
    // a store of more than 64 bits and a vector instruction that overwrites its data
    // registers is supplied by hand.
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1 nt\n\ts_nop 0" : : "v"(p), "v"(v) : "memory");
  } else {
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4_any *>(p));
  }
}

// a loaded value is "used" without any store: an empty instruction sequence that takes
// its registers as inputs keeps the load from being optimised away
__device__ __forceinline__ void keep_alive(const u32x4 &v) { asm volatile("" : : "v"(v.x), "v"(v.y), "v"(v.z), "v"(v.w)); }
// around the loads in one of two branches that load the same addresses in different ways: the compiler
// would make one load of the two, of the plain kind
__device__ __forceinline__ void keep_apart() { asm volatile(""); }

// Rows of less than 16 bytes: one slot per row.  The row's first and last V's bytes, which overlap in rows
// that are not one or two V long.  Bound by the number of accesses to partial lines.  8 layers, hidden
// 2048, the row-parallel tensors with TP 4 -> 1, us, this / 2 bytes at a time / vectors as wide as the
// row's alignment: rows of 14 bytes 9.0 / 12.0 / 13.3, cache-blocked list 9.1 / 19.9 / 12.6; 12 bytes 8.9 / 10.7 /
// 12.1 and 8.4 / 15.9 / 10.9; 4 bytes 8.6 / 8.7 / 11.3 and 5.6 / 6.2 / 9.4.
template <typename V, int kGroup>
__device__ __forceinline__ void copy_short_rows_by(const DevTile &tl, const uint64_t *__restrict__ extra_dst, const char *__restrict__ src,
                                                   char *__restrict__ dst_base, uint32_t lane, uint32_t begin, uint32_t end) {
  typedef V Any __attribute__((aligned(2)));
  const uint32_t last = tl.row_bytes - (uint32_t)sizeof(V);
  for (uint32_t row = begin + lane; row < end; row += kGroup) {
    const char *__restrict__ s = src + (size_t)row * tl.src_row_stride;
    const V v0 = *reinterpret_cast<const Any *>(s), v1 = *reinterpret_cast<const Any *>(s + last);
    for (uint32_t j = 0; j < tl.n_dst; ++j) { // uniform trip count
      char *__restrict__ d = dst_base + (j == 0 ? tl.dst_off : extra_dst[tl.dst_list + j - 1]) + (size_t)row * tl.dst_row_stride;
      *reinterpret_cast<Any *>(d) = v0;
      if (last) *reinterpret_cast<Any *>(d + last) = v1; // uniform
    }
  }
}
template <int kGroup>
__device__ __forceinline__ void copy_short_rows(const DevTile &tl, const uint64_t *__restrict__ extra_dst, const char *__restrict__ src,
                                                char *__restrict__ dst_base, uint32_t lane, uint32_t begin, uint32_t end) {
  // uniform branches
  if (tl.row_bytes >= 8) copy_short_rows_by<uint64_t, kGroup>(tl, extra_dst, src, dst_base, lane, begin, end);
  else if (tl.row_bytes >= 4) copy_short_rows_by<uint32_t, kGroup>(tl, extra_dst, src, dst_base, lane, begin, end);
  else copy_short_rows_by<uint16_t, kGroup>(tl, extra_dst, src, dst_base, lane, begin, end);
}

// Slots begin + lane + k * kGroup (k < kUnroll) below `end` of a record, between their loads and their
// stores; `lane` is the index inside a group of kGroup consecutive lanes.
template <int kGroup, int kPolicy, int kUnroll> struct SlotBatch {
  u32x4 v[kUnroll];
  uint32_t doff[kUnroll];
  bool live[kUnroll];

  __device__ __forceinline__ void load(const DevTile &tl, const char *__restrict__ src, uint32_t lane, uint32_t begin, uint32_t end) {
    // no branch between the loads, so that all are in flight: a slot with nothing to do loads the
    // record's first 16 bytes
    const uint32_t per_row = slots_per_row(tl);
    uint32_t soff[kUnroll];
    if (per_row == 0) { // uniform
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) {
        const uint32_t i = begin + lane + k * kGroup;
        live[k] = slot_offsets(tl, 0, i, soff[k], doff[k]) & (i < end);
      }
    } else {
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) {
        const uint32_t i = begin + lane + k * kGroup, row = i / per_row;
        live[k] = slot_offsets(tl, row, i - row * per_row, soff[k], doff[k]) & (i < end);
      }
    }
    if (shares_lines(tl)) { // uniform
      keep_apart();
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) v[k] = load_stream<kPolicy | 1>(src + (live[k] ? soff[k] : 0u));
      keep_apart();
    } else {
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) v[k] = load_stream<kPolicy>(src + (live[k] ? soff[k] : 0u));
    }
  }

  __device__ __forceinline__ void store(const DevTile &tl, const uint64_t *__restrict__ extra_dst, char *__restrict__ dst_base) const {
    // All loads are waited for here, before the first store: the compiler does not count the
    // stores of policy 0, so a wait for load k between them would wait for stores as well
    // (offload over the host link: 13.8 against 12.4 ms for 348 MB each way).
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) keep_alive(v[k]);
    for (uint32_t j = 0; j < tl.n_dst; ++j) { // uniform trip count
      char *__restrict__ dst = dst_base + (j == 0 ? tl.dst_off : extra_dst[tl.dst_list + j - 1]);
#pragma unroll
      for (int k = 0; k < kUnroll; ++k)
        if (live[k]) store_stream<kPolicy>(dst + doff[k], v[k]);
    }
  }
};

// Copies slots begin + lane + k * kGroup (k < kUnroll) below `end` of a record to its n_dst
// destinations; `lane` is the index inside a group of kGroup consecutive lanes (a workgroup or
// one wavefront), so the lanes of a wavefront walk consecutive bytes of a row and spill into
// the next row at its end.  All kUnroll slots are loaded before the first of them is stored.
template <int kGroup, int kPolicy, int kUnroll>
__device__ __forceinline__ void copy_slots(const DevTile &tl, const uint64_t *__restrict__ extra_dst,
                                           const char *__restrict__ src_base, char *__restrict__ dst_base, uint32_t lane,
                                           uint32_t begin, uint32_t end) {
  const char *__restrict__ src = src_base + tl.src_off;
  if constexpr (kUnroll == 1) {
    const uint32_t i = begin + lane;
    uint32_t soff, doff;
    if (i >= end || !slot_offsets(tl, i, soff, doff)) return;
    u32x4 v;
    if (shares_lines(tl)) { // uniform
      keep_apart();
      v = load_stream<kPolicy | 1>(src + soff);
      keep_apart();
    } else {
      v = load_stream<kPolicy>(src + soff);
    }
    for (uint32_t j = 0; j < tl.n_dst; ++j) // uniform trip count
      store_stream<kPolicy>(dst_base + (j == 0 ? tl.dst_off : extra_dst[tl.dst_list + j - 1]) + doff, v);
  } else if (begin < end) { // uniform
    SlotBatch<kGroup, kPolicy, kUnroll> b;
    b.load(tl, src, lane, begin, end);
    b.store(tl, extra_dst, dst_base);
  }
}

// n <= kChunks loads of 16 bytes, `stride` apart, all in flight together (beyond n the last one again)
template <int kChunks> __device__ __forceinline__ void load_chunks(const char *p, uint32_t n, uint32_t stride) {
  u32x4 v[kChunks];
#pragma unroll
  for (uint32_t j = 0; j < kChunks; ++j) v[j] = load_stream<1>(p + (size_t)min(j, n - 1) * stride);
#pragma unroll
  for (uint32_t j = 0; j < kChunks; ++j) keep_alive(v[j]);
}

// Loads the slots of the sources of a load-only record (rows of at least 16 bytes) and stores nothing.  The copy records of
// the chunks follow later in the list with the same number of workgroups each; where that is a multiple of
// eight, the workgroup that copies part k of a chunk runs on the XCD (workgroup index mod 8) whose L2 the
// group with part number k has filled.
template <int kGroup, int kUnroll>
__device__ __forceinline__ void load_slots(const DevTile &tl, const char *__restrict__ src_base, uint32_t lane, uint32_t begin,
                                           uint32_t end) {
  const uint32_t n = tl.n_dst & ~kLoadOnly, stride = tl.dst_list;
  const char *__restrict__ src = src_base + tl.src_off;
  // Enough slots to keep in flight: source by source, no branch between the loads.  Prefetched list under the
  // persistent wavefronts, 4 layers of Llama-7B, TP 8 -> 2: 1846 us, slot by slot 1984.
  if constexpr (kUnroll == kMaxUnroll) {
    if (begin >= end) return; // uniform
    uint32_t soff[kUnroll], doff;
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) slot_offsets(tl, min(begin + lane + k * kGroup, end - 1), soff[k], doff); // inside the row in any case
    for (uint32_t j = 0; j < n; ++j) { // uniform
      u32x4 v[kUnroll];
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) v[k] = load_stream<1>(src + (size_t)j * stride + soff[k]);
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) keep_alive(v[k]);
    }
    return;
  }
#pragma unroll
  for (int k = 0; k < kUnroll; ++k) {
    uint32_t soff, doff;
    const uint32_t i = begin + lane + k * kGroup;
    if (i >= end || !slot_offsets(tl, i, soff, doff)) continue;
    const char *p = src + soff;
    if (n == 2) load_chunks<2>(p, n, stride); // uniform
    else if (n == 1) load_chunks<1>(p, n, stride);
    else if (n <= 4) load_chunks<4>(p, n, stride);
    else load_chunks<HF_MAX_PREFETCH_CHUNKS>(p, n, stride);
  }
}

// slots [begin, end) of a record, begin + kUnroll * kGroup at most
template <int kGroup, int kPolicy, int kUnroll>
__device__ __forceinline__ void run_slots(const DevTile &tl, const uint64_t *__restrict__ extra_dst, const char *__restrict__ src,
                                          char *__restrict__ dst, uint32_t lane, uint32_t begin, uint32_t end) {
  // uniform branches
  if (tl.n_dst & kLoadOnly) load_slots<kGroup, kUnroll>(tl, src, lane, begin, end);
  else if (tl.row_bytes < kSlot) copy_short_rows<kGroup>(tl, extra_dst, src + tl.src_off, dst, lane, begin, end);
  else copy_slots<kGroup, kPolicy, kUnroll>(tl, extra_dst, src, dst, lane, begin, end);
}

// A whole record.  The next batch of loads is under way while a batch is stored: the persistent
// workgroups are few (offload and reload: 8), so what a lane has in flight is what the link sees.
// The second batch takes registers (157 in all, three wavefronts a SIMD; 61 and eight with one batch), and
// costs the lists on HBM nothing for it: 4 layers of Llama-7B, TP 8 -> 2, us, two batches / one: persistent
// workgroups one-to-one 2471 / 2496, cache-blocked 1673 / 1687, back 830 / 846; one workgroup per record 2407 / 2459.
template <int kGroup, int kPolicy>
__device__ __forceinline__ void run_tile(const DevTile &tl, const uint64_t *__restrict__ extra_dst,
                                         const char *__restrict__ src, char *__restrict__ dst, uint32_t lane) {
  constexpr uint32_t step = kMaxUnroll * kGroup;
  uint32_t i = tl.first;
  if ((tl.n_dst & kLoadOnly) || tl.row_bytes < kSlot) { // uniform
    for (; i < tl.end; i += step) run_slots<kGroup, kPolicy, kMaxUnroll>(tl, extra_dst, src, dst, lane, i, min(i + step, tl.end));
    return;
  }
  src += tl.src_off;
  SlotBatch<kGroup, kPolicy, kMaxUnroll> a, b;
  a.load(tl, src, lane, i, tl.end);
  for (;;) { // no load under a condition between a batch's loads and its stores: the waits count what is in flight
    if (i + step >= tl.end) return a.store(tl, extra_dst, dst);
    b.load(tl, src, lane, i += step, tl.end);
    a.store(tl, extra_dst, dst);
    if (i + step >= tl.end) return b.store(tl, extra_dst, dst);
    a.load(tl, src, lane, i += step, tl.end);
    b.store(tl, extra_dst, dst);
  }
}

// Persistent workgroups: workgroup w copies tiles w, w+grid, w+2*grid, ...  Every
// workgroup leaves the loop after at most ceil(n/grid) rounds; there is no waiting on
// other workgroups anywhere.
template <int kPolicy>
__global__ __launch_bounds__(kWG) void reshard_persistent(const DevTile *__restrict__ tiles, uint32_t n_tiles,
                                                          const uint64_t *__restrict__ extra_dst,
                                                          const char *__restrict__ src, char *__restrict__ dst) {
  for (uint32_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
    const DevTile tl = tiles[t];
    run_tile<kWG, kPolicy>(tl, extra_dst, src, dst, threadIdx.x);
  }
}

// Offload and reload: as reshard_persistent, but the next batch of loads is under way also where it is another
// record's, and the record after it is already there.  Bound: what eight workgroups have under way on the link.  Rows of 16
// bytes or more, one destination.  Figures at launch_link.
template <int kPolicy>
__global__ __launch_bounds__(kWG) void reshard_link(const DevTile *__restrict__ tiles, uint32_t n_tiles, const char *__restrict__ src,
                                                    char *__restrict__ dst) {
  constexpr uint32_t step = kMaxUnroll * kWG;
  SlotBatch<kWG, kPolicy, kMaxUnroll> a, b;
  uint32_t t = blockIdx.x;
  if (t >= n_tiles) return;
  DevTile at = tiles[t], bt, next = tiles[min(t + gridDim.x, n_tiles - 1)];
  uint32_t i = at.first;
  a.load(at, src + at.src_off, threadIdx.x, i, at.end);
  // the place after (tile, i): in the record, or in the workgroup's next; false: there is none
  const auto advance = [&](const DevTile &from, DevTile &to) {
    to = from;
    i += step;
    if (i < from.end) return true;
    t += gridDim.x;
    to = next;
    i = to.first;
    next = tiles[min(t + gridDim.x, n_tiles - 1)];
    return t < n_tiles;
  };
  for (;;) { // every round ends a batch; no load under a condition between a batch's loads and its stores
    if (!advance(at, bt)) return a.store(at, nullptr, dst);
    b.load(bt, src + bt.src_off, threadIdx.x, i, bt.end);
    a.store(at, nullptr, dst);
    if (!advance(bt, at)) return b.store(bt, nullptr, dst);
    a.load(at, src + at.src_off, threadIdx.x, i, at.end);
    b.store(bt, nullptr, dst);
  }
}

// Same, but every wavefront walks the list on its own: wavefront g of G copies tiles
// g, g+G, ...  (wavefront-level dispatch; pair it with tiles of a few KiB to 32 KiB).
template <int kPolicy>
__global__ __launch_bounds__(kWG) void reshard_wave_persistent(const DevTile *__restrict__ tiles, uint32_t n_tiles,
                                                               const uint64_t *__restrict__ extra_dst,
                                                               const char *__restrict__ src, char *__restrict__ dst) {
  const uint32_t waves_per_wg = kWG / kWave;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave); // uniform -> scalar tile loads
  const uint32_t g = blockIdx.x * waves_per_wg + wave, G = gridDim.x * waves_per_wg;
  for (uint32_t t = g; t < n_tiles; t += G) {
    const DevTile tl = tiles[t];
    run_tile<kWave, kPolicy>(tl, extra_dst, src, dst, threadIdx.x % kWave);
  }
}

template <int kPolicy>
__global__ __launch_bounds__(kWG) void reshard_one_tile(const DevTile *__restrict__ tiles, uint32_t n_tiles,
                                                        const uint64_t *__restrict__ extra_dst,
                                                        const char *__restrict__ src, char *__restrict__ dst) {
  const uint32_t t = blockIdx.x;
  if (t < n_tiles) {
    const DevTile tl = tiles[t];
    run_tile<kWG, kPolicy>(tl, extra_dst, src, dst, threadIdx.x);
  }
}

// One short-lived workgroup per kUnroll * kThreads slots: workgroup b copies part b % parts
// of record b / parts (or as place_of says) and exits (parts = ceil(unit bytes / part bytes), the same for every
// record; parts beyond the end of a short record are empty, and the planner cuts records so that few
// are).  The hardware dispatcher hands
// out workgroups in index order, so at any moment the chip works on one narrow, moving
// window of source and destination addresses, and a slow CU simply takes fewer
// workgroups.  All kUnroll slots of a lane are loaded before the
// first store.  kList does not change the code: it names the work list in the kernel's
// name, so that a profiler's per-kernel statistics keep apart what one process launches
// over different lists (0 = train->gen without own pieces, 1 = train->gen with own
// pieces, 2 = any other list: reverse, own pieces alone).
template <int kPolicy, int kUnroll, int kThreads, int kList>
__global__ __launch_bounds__(kThreads) void reshard_parts(const DevTile *__restrict__ tiles, uint32_t n_tiles, uint32_t parts, uint32_t inverse, uint32_t group,
                                                          const uint64_t *__restrict__ extra_dst,
                                                          const char *__restrict__ src, char *__restrict__ dst) {
  const Place p = place_of(blockIdx.x, parts, inverse, n_tiles, group);
  if (p.record < n_tiles) {
    const DevTile tl = tiles[p.record];
    const uint32_t begin = tl.first + p.part * (kUnroll * kThreads), end = min(begin + kUnroll * kThreads, tl.end);
    run_slots<kThreads, kPolicy, kUnroll>(tl, extra_dst, src, dst, threadIdx.x, begin, end);
  }
}

// 16 bytes that begin with the last n of `head` and go on with the first of `tail` (0 < n < 16)
__device__ __forceinline__ u32x4 join(const u32x4 &head, const u32x4 &tail, uint32_t n) {
  const uint64_t h0 = (uint64_t)head.y << 32 | head.x, h1 = (uint64_t)head.w << 32 | head.z;
  const uint64_t t0 = (uint64_t)tail.y << 32 | tail.x, t1 = (uint64_t)tail.w << 32 | tail.z;
  const uint32_t up = 8 * n, down = 128 - up; // tail << up | head >> down
  const bool wide = up >= 64;
  const uint32_t u = up & 63, d = down & 63;
  const uint64_t tu0 = t0 << u, tu1 = t1 << u | (t0 >> 1) >> (63 - u);
  const uint64_t hd0 = h0 >> d | (h1 << 1) << (63 - d), hd1 = h1 >> d;
  // up < 64: down > 64 (or both are 64: wide); tail moves by less than a half, head by more than one
  const uint64_t lo = wide ? (down == 64 ? h1 : hd0) : tu0 | h1 >> d;
  const uint64_t hi = wide ? (down == 64 ? t0 : t0 << u | hd1) : tu1;
  return u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
}

// A wavefront that stores its KiB to several destinations issues a store only when the one before has been
// acknowledged.  What bounds a launch with several destinations is how many stores are under way: without the
// wait the write streams pile up in front of the memory channels.  Plain streams of 640 MiB (records as here), TB/s read
// once + written, with the wait / without: 3 destinations 6.57 / 6.46, 4 6.69 / 6.12, 7 6.75 / 5.55, 8 6.49 / 5.61, each
// with at most 25 wavefronts on a CU; with as many as fit (32) 6.49 / 6.54, 6.27 / 6.06, 5.92 / 5.48, 5.75 / 5.58; with 21
// 6.19, 6.39, 6.59, 6.43.  One store left under way: between the two.  Two destinations: level (6.61 / 6.55).
__device__ __forceinline__ void wait_for_stores() { asm volatile("s_waitcnt vmcnt(0)" : : : "memory"); }

// Calls store(distance) for the first destination (distance 0) and the n - 1 listed ones.
template <bool kPaced, typename F> __device__ __forceinline__ void each_destination(const uint64_t *__restrict__ distances, uint32_t n, F store) {
  uint64_t next = distances[0]; // the list is never empty and ends with an entry of its own
  store(uint64_t(0));
  for (uint32_t j = 1; j < n; ++j) { // uniform
    const uint64_t d = next;
    next = distances[j]; // under way while the store is waited for
    if constexpr (kPaced) wait_for_stores();
    store(d);
  }
}

// A row of less than 16 bytes, as in copy_short_rows_by.
template <typename V> __device__ __forceinline__ void copy_short_row_by(const char *__restrict__ s, char *__restrict__ d, uint32_t last,
                                                                        const uint64_t *__restrict__ distances, uint32_t n) {
  typedef V Any __attribute__((aligned(2)));
  const V v0 = *reinterpret_cast<const Any *>(s), v1 = *reinterpret_cast<const Any *>(s + last);
  for (uint32_t j = 0; j < n; ++j) { // uniform
    char *__restrict__ to = d + (j ? distances[j - 1] : 0);
    *reinterpret_cast<Any *>(to) = v0;
    if (last) *reinterpret_cast<Any *>(to + last) = v1; // uniform
  }
}
__device__ __forceinline__ void copy_short_row(const DevTile &tl, const uint64_t *__restrict__ distances, const char *__restrict__ src,
                                               char *__restrict__ dst, uint32_t row) {
  src += tl.src_off + (size_t)row * tl.src_row_stride;
  dst += tl.dst_off + (size_t)row * tl.dst_row_stride;
  // uniform branches
  if (tl.row_bytes >= 8) copy_short_row_by<uint64_t>(src, dst, tl.row_bytes - 8, distances, tl.n_dst);
  else if (tl.row_bytes >= 4) copy_short_row_by<uint32_t>(src, dst, tl.row_bytes - 4, distances, tl.n_dst);
  else copy_short_row_by<uint16_t>(src, dst, tl.row_bytes - 2, distances, tl.n_dst);
}

// One slot per lane of a band (slots.hpp).  Bound by the stores, as above; what the form is for is that no line is
// written in two parts by two wavefronts, which memory takes five times as long for as for a whole line: row-parallel tensors alone,
// TB/s, 4 destinations and one read, plain streams: stripes of 2752 bytes 5.68 by stripes / 6.07 by rows, 1040
// bytes 4.47 / 6.36, 1024 5.76 / 6.11; with the own stripe left out (3 destinations, lines at its edges remain in
// parts) 2752 5.27 / 5.65, 1040 4.60 / 5.92, 1024 5.85 / 6.40, 6912 (two stripes) 6.22 / 6.12.  The second load
// of a joined slot is under way with the first.
template <int kPolicy, bool kPaced>
__device__ __forceinline__ void copy_band(const DevTile &tl, const uint64_t *__restrict__ distances, const char *__restrict__ src,
                                          char *__restrict__ dst, uint32_t i) {
  const BandSlot b = band_slot(tl, i);
  const uint32_t left = tl.row_bytes - b.at; // of the stripe's row
  const bool joined = left < kSlot;          // the slot's last bytes are the next stripe's
  const u32x4 head = load_stream<kPolicy>(src + band_source(tl, b.row, b.stripe) + (joined ? tl.row_bytes - kSlot : b.at));
  u32x4 tail = head, both = head;
  uint32_t next = b.stripe;
  if (joined) {
    const bool wraps = (b.stripe + 1) * tl.row_bytes == tl.dst_row_stride;
    next = wraps ? 0 : b.stripe + 1;
    tail = load_stream<kPolicy>(src + band_source(tl, b.row + wraps, next));
    both = join(head, tail, left);
  }
  dst += tl.dst_off + (uint64_t)i * kSlot;
  const uint32_t n = band_members(tl);
  uint64_t entry = distances[0];
  for (uint32_t j = 0; j < n; ++j) { // uniform
    const uint32_t skip = (uint32_t)(entry >> 56);
    char *__restrict__ d = dst + (entry & kBandDistance);
    entry = distances[j + 1]; // the list ends with an entry of its own
    const bool first = skip != b.stripe + 1, second = skip != next + 1;
    u32x4 v = both;
    if (first != second) { // one of the two stripes: a whole slot inside it
      v = first ? head : tail;
      d += first ? (int32_t)(left - kSlot) : (int32_t)left;
    }
    if (kPaced && j) wait_for_stores();
    if (first | second) store_stream<kPolicy>(d, v);
  }
}

// The list that runs while every choice is the library's: one wavefront per KiB of a record (kThreads lanes, where the list is
// short: eight of them), as reshard_parts, but on whole KiB of the destination, and without load-only records.  Plain streams to 8 destinations that start 256, 512 or 768
// bytes into a KiB run at 6.25, 6.06 and 6.26 TB/s, on the KiB at 6.68 (3 destinations 6.60, 6.59, 6.61 and 6.66).
// Fetching the records of the next 8 MiB into L2 ahead of their wavefronts: 1-2 % slower.  Whole calls against the
// prefetched list (us, before / now): Llama-7B TP 8 -> 2 8640 / 8187, with own pieces 10560 / 10050-10170, 13B layers 2829
// / 2721, gathered out of the generation buffers 1701 / 1621, rows of 1026 bytes 245 / 228.
template <int kPolicy, bool kPaced, int kThreads, int kList>
__global__ __launch_bounds__(kThreads) void reshard_auto(const DevTile *__restrict__ tiles, uint32_t n_tiles, uint32_t parts, uint32_t inverse,
                                                      const uint64_t *__restrict__ distances,
                                                      const char *__restrict__ src, char *__restrict__ dst) {
  const uint32_t t = record_of(blockIdx.x, parts, inverse);
  const uint32_t part = blockIdx.x - t * parts;
  if (t >= n_tiles) return;
  const DevTile tl = tiles[t];
  const uint32_t i = tl.first - slots_into_kib(tl) + part * kThreads + threadIdx.x;
  if (i >= tl.end || (int32_t)(i - tl.first) < 0) return;
  distances += tl.dst_list;
  // uniform branches
  if ((tl.n_dst & kBand) == kBand) {
    if (tl.n_dst & kBandParts) copy_band<5, kPaced>(tl, distances, src, dst, i);
    else copy_band<kPolicy, kPaced>(tl, distances, src, dst, i);
  } else if (tl.row_bytes < kSlot) {
    copy_short_row(tl, distances, src, dst, i);
  } else {
    uint32_t soff, doff;
    if (!slot_offsets(tl, i, soff, doff)) return;
    const u32x4 v = load_stream<kPolicy>(src + tl.src_off + soff);
    dst += tl.dst_off + doff;
    each_destination<kPaced>(distances, tl.n_dst, [&](uint64_t d) { store_stream<kPolicy>(dst + d, v); });
  }
}

// Tile staged through LDS in 16 KiB slabs: global -> registers -> LDS, barrier,
// LDS -> registers -> global.  Exists to measure whether staging buys anything for the
// block-level permutations of this path (it moves the same HBM bytes).
constexpr uint32_t kSlab = 16 * 1024;
__device__ __forceinline__ void copy_slots_lds(const DevTile &tl, const uint64_t *__restrict__ extra_dst,
                                               const char *__restrict__ src_base, char *__restrict__ dst_base, u32x4 *stage) {
  const char *__restrict__ src = src_base + tl.src_off;
  constexpr uint32_t per_slab = kSlab / kSlot;
  for (uint32_t base = tl.first; base < tl.end; base += per_slab) {
    const uint32_t n = min(per_slab, tl.end - base);
    uint32_t soff, doff;
    for (uint32_t j = threadIdx.x; j < n; j += kWG)
      if (slot_offsets(tl, base + j, soff, doff)) stage[j] = load_stream<0>(src + soff);
    __syncthreads();
    for (uint32_t d = 0; d < tl.n_dst; ++d) {
      char *__restrict__ dst = dst_base + (d == 0 ? tl.dst_off : extra_dst[tl.dst_list + d - 1]);
      for (uint32_t j = threadIdx.x; j < n; j += kWG)
        if (slot_offsets(tl, base + j, soff, doff)) store_stream<0>(dst + doff, stage[j]);
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(kWG) void reshard_persistent_lds(const DevTile *__restrict__ tiles, uint32_t n_tiles,
                                                              const uint64_t *__restrict__ extra_dst,
                                                              const char *__restrict__ src, char *__restrict__ dst) {
  __shared__ u32x4 stage[kSlab / kSlot];
  for (uint32_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
    const DevTile tl = tiles[t];
    // uniform branches; few slots at a time, for the registers: 48, which leaves room for eight wavefronts a
    // SIMD (69 and seven with run_tile here: 4 layers of Llama-7B 2655 against 2549 us, back 894 / 859)
    if (tl.n_dst & kLoadOnly)
      for (uint32_t i = tl.first; i < tl.end; i += 4 * kWG) load_slots<kWG, 4>(tl, src, threadIdx.x, i, min(i + 4 * kWG, tl.end));
    else if (tl.row_bytes < kSlot) copy_short_rows<kWG>(tl, extra_dst, src + tl.src_off, dst, threadIdx.x, tl.first, tl.end);
    else copy_slots_lds(tl, extra_dst, src, dst, stage);
  }
}

__global__ __launch_bounds__(kWG) void calib_copy(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst, size_t n_vec) {
  const size_t stride = (size_t)gridDim.x * kWG;
  for (size_t i = (size_t)blockIdx.x * kWG + threadIdx.x; i < n_vec; i += stride) dst[i] = src[i];
}

// All-gather of per-rank result slots inside micro-DP groups (HybridFlow Section 5.2
// step 3): every input slot goes to n_dst output slots, out_slots[in * n_dst ...].  A workgroup
// takes one part of an input slot to all of them (or to dst_per_wg of them).  kForm 2: slots of
// whole 128-byte lines; the part is loaded once.  kForm 1: any slot of at least 16 bytes; a lane
// loads for every output slot the 16 bytes that fill an aligned vector there (from L1 / L2 after
// the first), and the vectors at either end are moved inside the slot.  kForm 0: 4 bytes at a time.
// Bound: HBM, one read and n_dst writes.  Measured against one workgroup per (output slot, 4 KiB)
// that reads the input slot again for each, us: 8 ranks in groups of four, 16 MiB slots 150-164
// -> 110 (6.1 TB/s), 16 MiB - 12 bytes (4-byte accesses then) 275 -> 108; groups of eight 297 -> 209
// and 729 -> 207, 201428 bytes 7.1 -> 4.3.  Single wavefronts with system-scope stores are best
// for whole lines (110; 256 lanes and non-temporal stores 137), 512 lanes with non-temporal stores
// for odd slots below 1 MiB (4.9 against 5.8 for 201428 bytes), level with the others above.
// Odd slots loaded once and stored unaligned: 140-165 instead of 108.
// kForm 2: as in reshard_auto a wavefront's stores wait for one another.  Of a long gather a CU holds 25 (kForm 2) or 16
// (kForm 1) wavefronts only (launch_gather_slots).
constexpr int gather_lanes(int form) { return form == 2 ? kWave : form == 1 ? 512 : kWG; }
template <int kForm>
__global__ __launch_bounds__(gather_lanes(kForm)) void gather_slots(const uint32_t *__restrict__ out_slots, uint32_t n_dst, uint32_t chunks,
                                                          uint32_t dst_per_wg, uint64_t slot_bytes, const char *__restrict__ in, char *__restrict__ out) {
  const uint32_t slot = blockIdx.x / chunks, chunk = blockIdx.x - slot * chunks;
  const uint64_t i = (uint64_t)chunk * gather_lanes(kForm) + threadIdx.x;
  const uint32_t j0 = blockIdx.y * dst_per_wg, j1 = min(j0 + dst_per_wg, n_dst);
  const uint32_t *__restrict__ list = out_slots + (size_t)slot * n_dst;
  in += slot * slot_bytes;
  if constexpr (kForm == 2) {
    if (i * kSlot >= slot_bytes) return;
    const u32x4 v = load_stream<1>(in + i * kSlot);
    for (uint32_t j = j0; j < j1; ++j) { // uniform
      const uint64_t to = list[j] * slot_bytes;
      if (j != j0) wait_for_stores();
      store_stream<1>(out + to + i * kSlot, v);
    }
  } else if constexpr (kForm == 1) {
    for (uint32_t j = j0; j < j1; ++j) { // uniform
      const uint64_t to = list[j] * slot_bytes;
      const int64_t at = (int64_t)(i * kSlot) - (int64_t)(to & 127);
      if (at > -(int64_t)kSlot && at < (int64_t)slot_bytes) {
        const uint64_t b = at < 0 ? 0 : min((uint64_t)at, slot_bytes - kSlot);
        store_stream<5>(out + to + b, load_stream<1>(in + b));
      }
    }
  } else {
    if (i * 4 >= slot_bytes) return;
    const uint32_t v = *reinterpret_cast<const uint32_t *>(in + i * 4);
    for (uint32_t j = j0; j < j1; ++j) *reinterpret_cast<uint32_t *>(out + list[j] * slot_bytes + i * 4) = v;
  }
}

// read-only and write-only counterparts of calib_copy (ceilings of one direction)
__global__ __launch_bounds__(kWG) void calib_read(const u32x4 *__restrict__ src, size_t n_vec) {
  const size_t stride = (size_t)gridDim.x * kWG;
  u32x4 acc = {0, 0, 0, 0};
  for (size_t i = (size_t)blockIdx.x * kWG + threadIdx.x; i < n_vec; i += stride) acc ^= __builtin_nontemporal_load(src + i);
  keep_alive(acc);
}
__global__ __launch_bounds__(kWG) void calib_write(u32x4 *__restrict__ dst, size_t n_vec) {
  const size_t stride = (size_t)gridDim.x * kWG;
  const u32x4 v = {0x5A5A5A5Au, 0x5A5A5A5Au, 0x5A5A5A5Au, 0x5A5A5A5Au};
  for (size_t i = (size_t)blockIdx.x * kWG + threadIdx.x; i < n_vec; i += stride) __builtin_nontemporal_store(v, dst + i);
}

// One read, n_dst writes (hf_calib_fanout); src == null: writes only, dst == null: the
// read only.  A workgroup handles kUnroll vectors per lane.  method 0 (registers): every
// workgroup stores its vectors to all n_dst places.  method 1 (cache-blocked): the grid is
// (blocks x n_dst passes x workgroups per block) and a workgroup stores to the place of its
// pass, so that passes 2.. re-read what pass 1 brought into L2.  method 2 (prefetched): the
// grid is (blocks x 2 passes x workgroups per block); pass 0 only loads the block, pass 1
// loads it again (from L2) and stores it to all n_dst places.
template <int kThreads, int kUnroll>
__global__ __launch_bounds__(kThreads) void calib_fanout(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst, size_t n_vec,
                                                         uint32_t n_dst, size_t stride_vec, uint32_t block_vecs, int method) {
  constexpr uint32_t per_wg = kThreads * kUnroll;
  size_t first;
  uint32_t pass = 0;
  if (method == 0) {
    first = (size_t)blockIdx.x * per_wg;
  } else {
    const uint32_t wpb = block_vecs / per_wg; // workgroups per block pass
    const uint32_t passes = method == 1 ? n_dst : 2;
    const uint32_t block = blockIdx.x / (wpb * passes), rest = blockIdx.x - block * (wpb * passes);
    pass = rest / wpb;
    first = (size_t)block * block_vecs + (size_t)(rest - pass * wpb) * per_wg;
  }
  u32x4 v[kUnroll];
#pragma unroll
  for (int k = 0; k < kUnroll; ++k) {
    const size_t i = first + (size_t)k * kThreads + threadIdx.x;
    v[k] = u32x4{0x5A5A5A5Au, 0x5A5A5A5Au, 0x5A5A5A5Au, 0x5A5A5A5Au};
    if (src && i < n_vec) v[k] = method ? src[i] : __builtin_nontemporal_load(src + i);
  }
  if (!dst || (method == 2 && pass == 0)) { // read only
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) keep_alive(v[k]);
    return;
  }
  const uint32_t j0 = method == 1 ? pass : 0, j1 = method == 1 ? pass + 1 : n_dst;
  for (uint32_t j = j0; j < j1; ++j)
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) {
      const size_t i = first + (size_t)k * kThreads + threadIdx.x;
      if (i < n_vec) __builtin_nontemporal_store(v[k], dst + (size_t)j * stride_vec + i);
    }
}

// Launches and returns what the launch itself returned.  A call that is over in 2 to 3 us waits for the host: without the
// launch configuration's way through the runtime (<<< >>>) and a question for the last error 2.42 us per call from native code, 2.67 with
// them; from Python 3.09 and 3.34.
template <typename... P, typename... A>
hipError_t enqueue(void (*kernel)(P...), dim3 grid, int threads, uint32_t lds, hipStream_t st, A... args) {
  const auto go = [&](P... p) {
    void *list[] = {const_cast<void *>(static_cast<const void *>(&p))...};
    return hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, dim3(threads), list, lds, st);
  };
  const hipError_t e = go(args...);
  if (e != hipSuccess) (void)hipGetLastError(); // it is reported here, not to whoever asks next
  return e;
}

template <int kPolicy, int kList>
hipError_t launch_parts(const DevTile *d_tiles, uint32_t n, const uint64_t *extra_dst, const char *s, char *d, uint32_t unit_bytes,
                  uint32_t part_bytes, int wg_threads, uint32_t group, hipStream_t st) {
  const uint32_t parts = (unit_bytes + part_bytes - 1) / part_bytes, inverse = inverse_of(parts);
  const dim3 g(n * parts);
  if (wg_threads == kWave) { // one wavefront per workgroup: part_bytes = U * 1 KiB
    switch (part_bytes / 1024) {
    case 1: return enqueue((reshard_parts<kPolicy, 1, kWave, kList>), g, kWave, 0, st, d_tiles, n, parts, inverse, group, extra_dst, s, d);
    case 2: return enqueue((reshard_parts<kPolicy, 2, kWave, kList>), g, kWave, 0, st, d_tiles, n, parts, inverse, group, extra_dst, s, d);
    case 4: return enqueue((reshard_parts<kPolicy, 4, kWave, kList>), g, kWave, 0, st, d_tiles, n, parts, inverse, group, extra_dst, s, d);
    default: return enqueue((reshard_parts<kPolicy, 8, kWave, kList>), g, kWave, 0, st, d_tiles, n, parts, inverse, group, extra_dst, s, d);
    }
  } else {
    switch (part_bytes / 4096) {
    case 1: return enqueue((reshard_parts<kPolicy, 1, kWG, kList>), g, kWG, 0, st, d_tiles, n, parts, inverse, group, extra_dst, s, d);
    case 2: return enqueue((reshard_parts<kPolicy, 2, kWG, kList>), g, kWG, 0, st, d_tiles, n, parts, inverse, group, extra_dst, s, d);
    case 4: return enqueue((reshard_parts<kPolicy, 4, kWG, kList>), g, kWG, 0, st, d_tiles, n, parts, inverse, group, extra_dst, s, d);
    default: return enqueue((reshard_parts<kPolicy, 8, kWG, kList>), g, kWG, 0, st, d_tiles, n, parts, inverse, group, extra_dst, s, d);
    }
  }
}

template <int kPolicy, bool kPaced, int kThreads>
hipError_t launch_auto(const DevTile *d_tiles, uint32_t n, const uint64_t *distances, const char *s, char *d, uint32_t parts, uint32_t wgs_per_cu,
                 int list_tag, hipStream_t st) {
  // LDS that nothing uses keeps further workgroups off the CU: 160 KB of it, given out in 1280 bytes
  const uint32_t lds = wgs_per_cu ? 160 * 1024 / wgs_per_cu / 1280 * 1280 : 0, inverse = inverse_of(parts);
  const dim3 g(n * parts);
  if (list_tag == 0) return enqueue((reshard_auto<kPolicy, kPaced, kThreads, 0>), g, kThreads, lds, st, d_tiles, n, parts, inverse, distances, s, d);
  return enqueue((reshard_auto<kPolicy, kPaced, kThreads, 1>), g, kThreads, lds, st, d_tiles, n, parts, inverse, distances, s, d);
}

template <int kPolicy>
hipError_t launch_policy(const DevTile *d_tiles, uint32_t n, uint32_t grid, const uint64_t *extra_dst, const char *s, char *d,
                   int variant, uint32_t unit_bytes, uint32_t part_bytes, int wg_threads, int list_tag, hipStream_t st) {
  const uint32_t group = variant == kVariantPartsTogether ? 3 : 0;
  switch (variant) {
  case HF_VARIANT_PARTS:
  case kVariantPartsTogether:
    switch (list_tag) {
    case 0: return launch_parts<kPolicy, 0>(d_tiles, n, extra_dst, s, d, unit_bytes, part_bytes, wg_threads, group, st);
    case 1: return launch_parts<kPolicy, 1>(d_tiles, n, extra_dst, s, d, unit_bytes, part_bytes, wg_threads, group, st);
    default: return launch_parts<kPolicy, 2>(d_tiles, n, extra_dst, s, d, unit_bytes, part_bytes, wg_threads, group, st);
    }
  case kVariantLink:
    return enqueue(reshard_link<kPolicy>, dim3(grid), kWG, 0, st, d_tiles, n, s, d);
  case HF_VARIANT_ONE_WG_PER_TILE:
    return enqueue(reshard_one_tile<kPolicy>, dim3(n), kWG, 0, st, d_tiles, n, extra_dst, s, d);
  case HF_VARIANT_WAVE_PERSISTENT:
    return enqueue(reshard_wave_persistent<kPolicy>, dim3(grid), kWG, 0, st, d_tiles, n, extra_dst, s, d);
  default:
    return enqueue(reshard_persistent<kPolicy>, dim3(grid), kWG, 0, st, d_tiles, n, extra_dst, s, d);
  }
}

} // namespace

int launch_tiles(const DevTile *d_tiles, size_t n_tiles, const uint64_t *extra_dst, const void *src, void *dst,
                 int variant, int grid_wgs, int cache_policy, uint32_t unit_bytes, uint32_t part_bytes,
                 uint32_t max_wgs_per_launch, int wg_threads, int list_tag, void *stream) {
  if (n_tiles == 0) return 0;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const char *s = static_cast<const char *>(src);
  char *d = static_cast<char *>(dst);
  // A HIP grid holds fewer than 2^32 threads per dimension (a larger one is not refused,
  // its size wraps), so the kernels that take one workgroup per tile or per part go out
  // in several launches of at most max_wgs_per_launch workgroups, in list order.
  size_t tiles_per_launch = n_tiles;
  const bool automatic = variant == kVariantAuto || variant == kVariantAutoPaced;
  const uint32_t parts = (unit_bytes + part_bytes - 1) / part_bytes;
  if (variant == HF_VARIANT_PARTS || variant == kVariantPartsTogether || automatic) {
    if (parts > max_wgs_per_launch) return (int)hipErrorInvalidValue;
    tiles_per_launch = max_wgs_per_launch / parts;
  } else if (variant == HF_VARIANT_ONE_WG_PER_TILE) {
    tiles_per_launch = max_wgs_per_launch;
  }
  for (size_t first = 0; first < n_tiles; first += tiles_per_launch) {
    const uint32_t n = (uint32_t)std::min(tiles_per_launch, n_tiles - first);
    const uint32_t grid = (uint32_t)std::min<size_t>(n, (size_t)grid_wgs);
    const DevTile *t = d_tiles + first;
    hipError_t e;
    if (automatic) {
      const auto go = [&](auto launch) { e = launch(t, n, extra_dst, s, d, parts, (uint32_t)grid_wgs, list_tag, st); };
      if (variant == kVariantAutoPaced) go(cache_policy == 1 ? launch_auto<1, true, kWave> : launch_auto<5, true, kWave>);
      else if (wg_threads == kWave) go(launch_auto<1, false, kWave>);
      else go(cache_policy == 1 ? launch_auto<1, false, kAutoShortThreads> : launch_auto<5, false, kAutoShortThreads>);
    } else if (variant == HF_VARIANT_LDS_STAGED) {
      e = enqueue(reshard_persistent_lds, dim3(grid), kWG, 0, st, t, n, extra_dst, s, d);
    } else {
      switch (cache_policy) {
      case 1: e = launch_policy<1>(t, n, grid, extra_dst, s, d, variant, unit_bytes, part_bytes, wg_threads, list_tag, st); break;
      case 2: e = launch_policy<2>(t, n, grid, extra_dst, s, d, variant, unit_bytes, part_bytes, wg_threads, list_tag, st); break;
      case 3: e = launch_policy<3>(t, n, grid, extra_dst, s, d, variant, unit_bytes, part_bytes, wg_threads, list_tag, st); break;
      case 4: e = launch_policy<4>(t, n, grid, extra_dst, s, d, variant, unit_bytes, part_bytes, wg_threads, list_tag, st); break;
      case 5: e = launch_policy<5>(t, n, grid, extra_dst, s, d, variant, unit_bytes, part_bytes, wg_threads, list_tag, st); break;
      default: e = launch_policy<0>(t, n, grid, extra_dst, s, d, variant, unit_bytes, part_bytes, wg_threads, list_tag, st); break;
      }
    }
    if (e != hipSuccess) return (int)e;
  }
  return 0;
}

int launch_gather_slots(const uint32_t *d_out_slots, uint32_t n_slots, uint32_t n_dst, const void *in, void *out, size_t slot_bytes,
                        void *stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  // output vectors stay below what one HIP grid holds, whatever a workgroup covers
  const uint64_t limit = (slot_bytes / (slot_bytes % kSlot ? 4 : kSlot) + kWG - 1) / kWG;
  if (limit * n_slots * n_dst > 0xFFFFFFFFull / kWG) return (int)hipErrorInvalidValue;
  const char *s = static_cast<const char *>(in);
  char *d = static_cast<char *>(out);
  const int form = slot_bytes % 128 == 0 ? 2 : slot_bytes >= kSlot ? 1 : 0;
  const uint64_t per_wg = (form ? kSlot : 4) * gather_lanes(form);
  const uint64_t chunks = (slot_bytes + (form == 1 ? 124 : 0) + per_wg - 1) / per_wg; // a slot begins up to 124 bytes into a line
  // Few parts: the output slots are spread over workgroups too, until there are 8192 wavefronts (the
  // chip holds that many), or 16384 while a workgroup keeps four output slots.  us for 8 ranks x 8:
  // slots of 65548 bytes 4.0 unsplit, 3.5 split, 201428 bytes 4.9 / 4.3, 1 MiB 11.4 / 10.9; with two
  // output slots per input slot of 1 MiB splitting costs 30 % (3.9 / 5.1).
  const uint64_t waves = chunks * n_slots * (gather_lanes(form) / kWave);
  const uint32_t split = (uint32_t)std::min<uint64_t>(n_dst, std::max<uint64_t>({1, 8192 / waves, std::min<uint64_t>(16384 / waves, n_dst / 4)}));
  const uint32_t per = (n_dst + split - 1) / split;
  const dim3 grid((uint32_t)(chunks * n_slots), (n_dst + per - 1) / per);
  // LDS that nothing uses keeps further workgroups off the CU once the chip is filled four times over: 25 wavefronts of whole lines,
  // 16 of odd slots.  us, all that fit / 25 (24) / 21 (16): groups of four, 16 MiB 110.2 101.3 104.8, odd
  // 109.6 112.7 108.9; of eight, 16 MiB 208 187 189, 4 MiB 196 183 178, odd 200 200 189; of two, 16 MiB 62.7 60.4 61.9, odd 68.1
  // 66.2 66.9.  Short ones lose: of eight, 128 KiB 3.55 3.74, 201428 bytes 4.17 4.31 4.57.
  const uint32_t lds = waves < 4 * 8192 ? 0 : form == 2 ? 6400 : form == 1 ? 61440 : 0;
  switch (form) {
  case 2: return (int)enqueue(gather_slots<2>, grid, gather_lanes(2), lds, st, d_out_slots, n_dst, (uint32_t)chunks, per, slot_bytes, s, d);
  case 1: return (int)enqueue(gather_slots<1>, grid, gather_lanes(1), lds, st, d_out_slots, n_dst, (uint32_t)chunks, per, slot_bytes, s, d);
  default: return (int)enqueue(gather_slots<0>, grid, gather_lanes(0), 0, st, d_out_slots, n_dst, (uint32_t)chunks, per, slot_bytes, s, d);
  }
}

int launch_calib_fanout(const void *src, void *dst, size_t bytes, int n_dst, size_t dst_stride, int method, size_t block_bytes,
                        int wg_bytes, void *stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  const size_t n_vec = bytes / 16, stride_vec = dst_stride / 16;
  const size_t wgs_one_pass = (bytes + wg_bytes - 1) / wg_bytes;
  size_t grid = wgs_one_pass;
  if (method) {
    const size_t blocks = (bytes + block_bytes - 1) / block_bytes;
    grid = blocks * (size_t)(method == 1 ? n_dst : 2) * (block_bytes / wg_bytes);
  }
  const int threads = wg_bytes == 1024 ? kWave : kWG;
  if (grid == 0 || grid > 0xFFFFFFFFull / threads) return (int)hipErrorInvalidValue; // beyond one HIP grid
  const dim3 g((uint32_t)grid);
  const u32x4 *s = static_cast<const u32x4 *>(src);
  u32x4 *d = static_cast<u32x4 *>(dst);
  const uint32_t bv = (uint32_t)(block_bytes / 16);
  if (wg_bytes == 1024) hipLaunchKernelGGL((calib_fanout<kWave, 1>), g, dim3(kWave), 0, st, s, d, n_vec, (uint32_t)n_dst, stride_vec, bv, method);
  else if (wg_bytes == 4096) hipLaunchKernelGGL((calib_fanout<kWG, 1>), g, dim3(kWG), 0, st, s, d, n_vec, (uint32_t)n_dst, stride_vec, bv, method);
  else hipLaunchKernelGGL((calib_fanout<kWG, 2>), g, dim3(kWG), 0, st, s, d, n_vec, (uint32_t)n_dst, stride_vec, bv, method);
  return (int)hipGetLastError();
}

int launch_calib_copy(const void *src, void *dst, size_t bytes, void *stream) {
  if (bytes == 0) return 0;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (src && dst)
    hipLaunchKernelGGL(calib_copy, dim3(4096), dim3(kWG), 0, st, static_cast<const u32x4 *>(src), static_cast<u32x4 *>(dst), bytes / 16);
  else if (src) // read only
    hipLaunchKernelGGL(calib_read, dim3(4096), dim3(kWG), 0, st, static_cast<const u32x4 *>(src), bytes / 16);
  else
    hipLaunchKernelGGL(calib_write, dim3(4096), dim3(kWG), 0, st, static_cast<u32x4 *>(dst), bytes / 16);
  return (int)hipGetLastError();
}

} // namespace hf
