// Internal representation of a reshard plan (host side).  Not part of the ABI.
#pragma once

#include <cstdint>
#include <map>
#include <string>
#include <utility>
#include <vector>

#include "hfreshard.h"
#include "slots.hpp"

namespace hf {

// Position of a rank in the training grid and in the generation grid
// (HybridFlow Section 5.1 for the sizes, Section 5.3 for the grouping rules).
struct Coords {
  int dp, pp, tp;      // training: r = dp*p*t + pp*t + tp
  int gpp, gtp, micro; // generation stage, generation TP index, index in the micro-DP group
};

struct TensorRec {
  int id;        // HF_T_* or HF_G_*
  int layer;     // global layer, -1 for embed / lnf / head
  uint32_t rows, cols;
  uint64_t off;  // bytes from the start of the rank region
};

struct RankTable {
  std::vector<TensorRec> tensors;
  std::map<std::pair<int, int>, int> index; // (id, layer) -> position in `tensors`
  uint64_t size = 0;                        // region bytes (multiple of 4096)
  uint64_t base = 0;                        // bytes from the buffer base
  const TensorRec &at(int id, int layer) const { return tensors[index.at({id, layer})]; }
};

// A work list as the kernels walk it (see slots.hpp): the tiles of a host list, cut into records of at most unit_bytes / 16
// slots; one-to-one lists of up to 64 Ki tiles are first joined into pieces where they go on from one another.
struct DevList {
  std::vector<DevTile> tiles;
  uint32_t unit_bytes = 0;
  uint64_t bytes = 0;   // read once and written
  bool one_to_one = false; // every piece is read once and goes to one place (compile_list only)
  bool short_rows = false; // below 16 bytes (likewise)
  bool parts_of_lines = false; // more than one destination line in 16 is written in part (likewise)
  DevTile *d = nullptr; // device copy
};

// the array of hf_reshard_execute_static: 20 MiB
constexpr uint64_t kStaticRoom = HF_STATIC_SCRATCH_BYTES + (4u << 20);

// tiles of a multicast list measured by payload: all, those with several destinations, destinations 2..n
struct PayloadCount {
  uint64_t tiles = 0, shared = 0, extra = 0;
  void add(uint64_t n, uint64_t n_dst) {
    tiles += n;
    shared += n_dst > 1 ? n : 0;
    extra += n * (n_dst - 1);
  }
};

// What build_tiles makes of the descriptors.
struct WorkLists {
  // tiles_fwd = [peer tiles | own tiles], one destination per tile
  std::vector<hf_tile> tiles_fwd, tiles_back;
  size_t n_tiles_fwd_peer = 0;
  // multicast work list for execute: descriptors that read the same training piece are
  // tiled once; destinations 2..n of every tile are in mc_dst
  std::vector<hf_tile> tiles_fwd_mc;
  std::vector<uint64_t> mc_dst;
  // (in the mode that runs it) the same work, one destination per tile, in cache-blocked order
  std::vector<hf_tile> tiles_fwd_cb;
  // (likewise) the multicast list with a prefetch tile (n_dst == 0: loaded, stored nowhere) for every
  // tile, block-wise in front of the tiles themselves
  std::vector<hf_tile> tiles_fwd_pf;
  // offload / reload work lists (only with HF_PLAN_OFFLOAD): gen_buf -> image and back
  std::vector<hf_tile> tiles_offload, tiles_reload;
  bool has_sharing = false; // some training piece has more than one destination
  // totals of the descriptors that take part, per direction
  uint64_t moved_bytes[2] = {0, 0}, unique_bytes[2] = {0, 0};
  int64_t multicast = HF_MULTICAST_CACHE_BLOCKED; // build_tiles chooses it where the caller has not
  // The lists the kernels walk: train->gen in the current multicast mode (with or without the
  // own pieces, see active_fwd), own pieces alone, reverse, offload, reload.
  DevList dev_fwd, dev_own, dev_back, dev_offload, dev_reload;
  // What hf_reshard_execute runs while every choice is the library's (see build_auto_list), and its destinations
  // 2..n of a record (bands: all), as distances from the first.  Empty where it would be dev_fwd.
  DevList dev_auto;
  std::vector<uint64_t> auto_dst;
  bool auto_joins = false; // some of its slots are joined from two stripes
  // hf_reshard_execute_static: the train->gen list as its limit counts it (at least that many bytes where it
  // is over the limit), and what it stages in the place of dev_fwd and mc_dst (no records = those)
  PayloadCount payload_mc;
  uint64_t static_bytes = 0;
  DevList dev_static;
  std::vector<uint64_t> static_dst;
};

struct Plan : WorkLists {
  hf_model_desc m{};
  int p = 0, t = 0, d = 0, pg = 0, tg = 0;
  uint32_t flags = 0;
  int a = 0, b = 0, dg = 0, N = 0;
  int lps = 0, lpgs = 0; // layers per training / generation stage
  std::vector<int> mat;     // materialised ranks in buffer order
  std::vector<int> mat_pos; // rank -> position in `mat`, -1 if absent
  std::vector<Coords> coords;
  std::vector<int32_t> micro_peers; // [rank * dg + j] = rank with micro-DP index j in rank's micro-DP group
  std::vector<uint32_t> gather_out; // [rank * dg + j] = output slot of the j-th member of rank's group that takes rank's responses
  std::vector<RankTable> train_tab, gen_tab; // per rank (gen_tab[r].base valid only if materialised)
  uint64_t train_bytes = 0, gen_bytes = 0;

  // step 1 (train -> gen): pieces from micro-DP peers, and pieces from the rank's own shard
  std::vector<hf_desc> fwd_peer, fwd_own;
  // step 4 (gen -> train): inverse of the own pieces
  std::vector<hf_desc> back;
  // offload image (host side of hf_offload_remote / hf_reload_remote): one descriptor per
  // peer descriptor, src_off = where the piece sits in gen_buf, dst_off = where it sits in
  // the packed host image; remote_rank_off[i] = start of the i-th materialised rank's part
  std::vector<hf_desc> remote;
  std::vector<uint64_t> remote_rank_off;
  uint64_t remote_bytes = 0;

  // multicast mode that execute really uses: without sharing the multicast lists are the
  // one-destination work in another order, and the plain list with streaming loads is faster
  int64_t effective_prefetch_merge() const;
  int64_t effective_multicast() const { return has_sharing ? multicast : (int64_t)HF_MULTICAST_OFF; }
  // host copy of the current mode's work list (what hf_reshard_execute runs unless runs_auto, and what
  // hf_reshard_execute_static stages), and its length
  const std::vector<hf_tile> &active_fwd() const {
    switch (effective_multicast()) {
    case HF_MULTICAST_REGISTERS: return tiles_fwd_mc;
    case HF_MULTICAST_CACHE_BLOCKED: return tiles_fwd_cb;
    case HF_MULTICAST_PREFETCHED: return tiles_fwd_pf;
    default: return tiles_fwd;
    }
  }
  size_t active_fwd_count() const {
    return effective_multicast() == HF_MULTICAST_OFF && !(flags & HF_COPY_OWN) ? n_tiles_fwd_peer : active_fwd().size();
  }
  bool active_fwd_uses_mc_dst() const {
    return effective_multicast() == HF_MULTICAST_REGISTERS || effective_multicast() == HF_MULTICAST_PREFETCHED;
  }

  // bytes written per distinct byte read, train -> gen
  double fan_out() const { return unique_bytes[0] ? (double)moved_bytes[0] / (double)unique_bytes[0] : 0; }
  // hf_reshard_execute runs dev_auto
  bool runs_auto() const {
    return multicast_auto && variant == HF_VARIANT_PARTS && !wg_threads && !part_bytes && cache_policy < 0 && !dev_auto.tiles.empty();
  }

  int64_t tile_bytes = 128 * 1024;
  int64_t grid_wgs = 2048;
  int64_t variant = HF_VARIANT_PARTS;
  bool multicast_auto = true; // the mode follows the list's fan-out until the caller names one
  int64_t mc_block_bytes = 2 << 20;
  int64_t prefetch_block_bytes = 6 << 20; // measured over identical buffer placements: 6 MiB is 0.5-2.6 % ahead of 8 MiB on the 7B and 13B
                                          // shapes at 3 to 7 destinations per piece and level on the 34B shape; 4 MiB and 10+ MiB are behind
  int64_t prefetch_merge = 0; // copy tiles per chunked load-only tile; 0 = chosen from the fan-out
  int64_t cache_policy = -1; // auto
  int64_t part_bytes = 0; // 0 = chosen per launch
  int64_t max_wgs_per_launch = 0xFFFFFFFFll / 256; // a grid holds fewer than 2^32 threads
  int64_t wg_threads = 0; // 0 = chosen per launch
  int64_t kind_mask = 0x1F; // bit k: descriptors of kind k take part (hf_debug_restrict_kinds)
  int64_t offload_wgs = 8; // persistent workgroups of the offload / reload kernels
  int64_t row_interleave = 1; // tiles of the column stripes of one row-parallel tensor go out round-robin

  // changes whenever the work lists change: tells hf_reshard_execute_static whether the list
  // it staged for this plan is still the current one
  uint64_t serial = 0;

  // device copy (null for HF_PLAN_HOST_ONLY): the lists above (of train->gen the current mode's and dev_auto), the extra
  // destinations where their records have several, and the output slots of every rank's responses.  All lie in two
  // allocations: what a multicast mode replaces, and the rest
  int device = -1;
  char *d_forward = nullptr, *d_others = nullptr;
  uint64_t *d_mc_dst = nullptr;
  uint64_t *d_auto_dst = nullptr;
  uint32_t *d_gather_out = nullptr;
};

// Builds everything except the device copy.  Returns HF_OK or an error, with `err` set.
int build_plan(const hf_model_desc &m, const hf_train_layout &tl, const hf_gen_layout &gl, Plan &out, std::string &err);
// (Re)creates the tile lists from the descriptors with out.tile_bytes.
int build_tiles(Plan &pl, std::string &err);
// Decides what hf_reshard_execute_static runs (static_bytes, dev_static, static_dst).
void build_static_list(Plan &pl, uint64_t limit, uint64_t room);
// (Re)creates what the current multicast mode runs: its host list, dev_fwd and the static list.
void build_forward_lists(Plan &pl);
int64_t default_multicast(const Plan &pl); // needs the byte totals build_tiles sets
int64_t default_prefetch_merge(const Plan &pl); // likewise
inline int64_t Plan::effective_prefetch_merge() const { return prefetch_merge ? prefetch_merge : default_prefetch_merge(*this); }
// How Plan::dev_auto is launched.
struct AutoLaunch {
  bool short_list; // eight wavefronts to a workgroup
  bool paced;      // a wavefront's stores wait for one another
  int policy;      // 1 = system-scope stores, 5 = non-temporal ones
  int wgs_per_cu;  // at most; 0 = as many as fit
};
AutoLaunch auto_launch(const Plan &pl);
// Stores of a short list with one destination per piece, see there.
bool non_temporal_when_short(const DevList &list);
// Host-side consistency check (see hf_plan_validate).
int validate_plan(const Plan &pl, std::string &err);
uint64_t desc_bytes(const hf_desc &d);
uint64_t unique_src_bytes(const std::vector<const hf_desc *> &descs);

} // namespace hf
