// Host-only driver: the device lists (records and slots, slots.hpp) against the tile lists they are
// made from, byte by byte, on random small plans and in every multicast mode.
#include <cstdio>
#include <cstring>
#include <set>
#include <string>
#include <tuple>
#include <vector>

#include "plan.hpp"

namespace {

uint64_t g_state = 12345;
uint32_t rnd(uint32_t n) { // 0 .. n-1
  g_state = g_state * 6364136223846793005ull + 1442695040888963407ull;
  return (uint32_t)((g_state >> 33) % n);
}
template <typename T, size_t N> T pick(const T (&v)[N]) { return v[rnd(N)]; }

#define REQUIRE(c)                                                                              \
  do {                                                                                          \
    if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return false; }                     \
  } while (0)

// where every destination byte comes from (~0 = not written), and which source bytes are read
struct Bytes {
  std::vector<uint64_t> from;
  std::vector<char> read;
};

void expand(const std::vector<hf_tile> &tiles, size_t n, const std::vector<uint64_t> &mc_dst, Bytes &b) {
  for (size_t i = 0; i < n; ++i)
    for (uint32_t r = 0; r < tiles[i].rows; ++r)
      for (uint32_t k = 0; k < tiles[i].row_bytes; ++k) {
        const hf_tile &t = tiles[i];
        const uint64_t s = t.src_off + (uint64_t)r * t.src_row_stride + k;
        if (t.n_dst) b.read[s] = 1;
        for (uint32_t j = 0; j < t.n_dst; ++j)
          b.from[(j ? mc_dst[t.dst_list + j - 1] : t.dst_off) + (uint64_t)r * t.dst_row_stride + k] = s;
      }
}

bool check_list(const hf::DevList &l, const std::vector<uint64_t> &mc_dst, const Bytes &want, int64_t tile_bytes, bool prefetched = false,
                bool whole_tiles = false) {
  std::vector<char> done(want.from.size(), 0);
  typedef std::tuple<uint64_t, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t> Key;
  std::multiset<Key> loads, shared;
  bool copying = false;
  REQUIRE(whole_tiles || l.unit_bytes == tile_bytes || (l.unit_bytes < tile_bytes && l.unit_bytes % 8192 == 0));
  for (const hf::DevTile &t : l.tiles) {
    REQUIRE(t.first < t.end && (t.end - t.first) * hf::kSlot <= l.unit_bytes);
    const bool load_only = t.n_dst & hf::kLoadOnly;
    if (load_only && copying) { // a new block
      REQUIRE(loads == shared);
      loads.clear();
      shared.clear();
    }
    copying = !load_only;
    const uint32_t chunks = load_only ? t.n_dst & ~hf::kLoadOnly : 1;
    REQUIRE(chunks >= 1 && chunks <= HF_MAX_PREFETCH_CHUNKS);
    for (uint32_t c = 0; c < chunks; ++c) {
      const uint64_t src_off = t.src_off + (uint64_t)c * (load_only ? t.dst_list : 0);
      const Key key{src_off, t.first, t.end, t.row_bytes, t.src_row_stride, t.slots & ~hf::kSharesLines};
      if (load_only) loads.insert(key);
      else if (t.n_dst > 1 && t.row_bytes >= hf::kSlot) shared.insert(key); // shorter rows are not loaded ahead
      for (uint32_t i = t.first; i < t.end; ++i) {
        uint32_t s, d, n = hf::kSlot;
        if (load_only) { // 16 bytes whatever the row's length
          if (!hf::slot_offsets(t, i, s, d)) continue;
          const uint32_t in_row = s - (hf::slots_per_row(t) ? i / hf::slots_per_row(t) : 0) * t.src_row_stride;
          REQUIRE(in_row + n <= t.row_bytes);
        } else if (t.row_bytes < hf::kSlot) {
          s = i * t.src_row_stride;
          d = i * t.dst_row_stride;
          n = t.row_bytes;
        } else if (!hf::slot_offsets(t, i, s, d)) {
          continue;
        }
        for (uint32_t k = 0; k < n; ++k) {
          REQUIRE(src_off + s + k < want.read.size() && want.read[src_off + s + k]); // loads stay inside the sources
          if (load_only) continue;
          for (uint32_t j = 0; j < t.n_dst; ++j) {
            const uint64_t at = (j ? mc_dst[t.dst_list + j - 1] : t.dst_off) + d + k;
            REQUIRE(at < want.from.size() && want.from[at] == src_off + s + k);
            done[at] = 1;
          }
        }
      }
    }
  }
  if (prefetched) REQUIRE(loads == shared);
  else REQUIRE(loads.empty());
  for (size_t i = 0; i < done.size(); ++i) REQUIRE(done[i] == (want.from[i] != ~0ull));
  return true;
}

bool check_plan(hf::Plan &pl) {
  const size_t image = pl.remote_bytes, train = pl.train_bytes, gen = pl.gen_bytes;
  const bool from_gen = pl.flags & HF_GATHER_FROM_GEN;
  auto one = [&](const hf::DevList &l, const std::vector<hf_tile> &tiles, size_t first, size_t n, size_t src, size_t dst, bool prefetched = false) {
    Bytes b{std::vector<uint64_t>(dst, ~0ull), std::vector<char>(src, 0)};
    std::vector<hf_tile> part(tiles.begin() + first, tiles.begin() + first + n);
    expand(part, n, pl.mc_dst, b);
    return check_list(l, pl.mc_dst, b, pl.tile_bytes, prefetched);
  };
  REQUIRE(one(pl.dev_fwd, pl.active_fwd(), 0, pl.active_fwd_count(), from_gen ? gen : train, gen,
              pl.effective_multicast() == HF_MULTICAST_PREFETCHED));
  REQUIRE(one(pl.dev_own, pl.tiles_fwd, pl.n_tiles_fwd_peer, pl.tiles_fwd.size() - pl.n_tiles_fwd_peer, train, gen));
  REQUIRE(one(pl.dev_back, pl.tiles_back, 0, pl.tiles_back.size(), gen, train));
  REQUIRE(one(pl.dev_offload, pl.tiles_offload, 0, pl.tiles_offload.size(), gen, image));
  REQUIRE(one(pl.dev_reload, pl.tiles_reload, 0, pl.tiles_reload.size(), image, gen));
  // the form that hf_reshard_execute_static stages where the records do not fit (here: never do)
  static int calls = 0;
  if (calls++ % 5 == 0) {
    hf::build_static_list(pl, 1ull << 40, 0);
    Bytes b{std::vector<uint64_t>(gen, ~0ull), std::vector<char>(from_gen ? gen : train, 0)};
    std::vector<hf_tile> part(pl.active_fwd().begin(), pl.active_fwd().begin() + pl.active_fwd_count());
    expand(part, part.size(), pl.mc_dst, b);
    REQUIRE(check_list(pl.dev_static, pl.static_dst, b, pl.tile_bytes, false, true));
    for (const hf::DevTile &t : pl.dev_static.tiles) REQUIRE(t.first == 0 && !(t.n_dst & hf::kLoadOnly));
    const uint64_t bytes = (pl.dev_static.tiles.size() * sizeof(hf_tile) + 255) / 256 * 256 + pl.static_dst.size() * sizeof(uint64_t);
    // no larger than what the limit counts; the same where it counts no load-only tiles
    REQUIRE(pl.effective_multicast() == HF_MULTICAST_PREFETCHED ? bytes <= pl.static_bytes : bytes == pl.static_bytes);
    hf::build_static_list(pl, pl.static_bytes, 1ull << 40); // at the limit, and the records fit
    REQUIRE(pl.dev_static.tiles.empty() && pl.static_dst.empty());
    const uint64_t counted = pl.static_bytes;
    if (counted) {
      hf::build_static_list(pl, counted - 1, 0); // beyond it
      REQUIRE(pl.static_bytes > counted - 1 && pl.dev_static.tiles.empty());
    }
    hf::build_static_list(pl, HF_STATIC_SCRATCH_BYTES, hf::kStaticRoom);
  }
  if (pl.dev_fwd.unit_bytes == pl.tile_bytes) // the records of a list do not outgrow its tiles
    REQUIRE(pl.dev_fwd.tiles.size() <= pl.active_fwd_count() + pl.active_fwd_count() / 8 + 8);
  return true;
}

bool check_modes(hf::Plan &pl) {
  for (int mode = HF_MULTICAST_OFF; mode <= HF_MULTICAST_PREFETCHED; ++mode) {
    pl.multicast_auto = false;
    pl.multicast = mode;
    hf::build_forward_lists(pl);
    if (!check_plan(pl)) {
      const hf_model_desc &m = pl.m;
      std::printf("L %d h %d q %d kv %d hd %d F %d V %d  p %d t %d pg %d tg %d flags %x tile %lld mode %d\n", m.n_layers, m.hidden, m.n_q_heads,
                  m.n_kv_heads, m.head_dim, m.ffn, m.vocab, pl.p, pl.t, pl.pg, pl.tg, (unsigned)pl.flags, (long long)pl.tile_bytes, mode);
      return false;
    }
  }
  return true;
}

// The plan's own check (hf_plan_validate) looks at the records: it passes, and finds any one record changed.
bool check_validation(hf::Plan &pl) {
  std::string err;
  REQUIRE(hf::validate_plan(pl, err) == HF_OK);
  for (hf::DevList *l : {&pl.dev_fwd, &pl.dev_own, &pl.dev_back, &pl.dev_offload, &pl.dev_reload}) {
    if (l->tiles.empty()) continue;
    for (int change = 0; change < 9; ++change) {
      const size_t i = rnd((uint32_t)l->tiles.size());
      const std::vector<hf::DevTile> keep = l->tiles;
      hf::DevTile &t = l->tiles[i];
      const bool load_only = t.n_dst & hf::kLoadOnly;
      // (slots that stand for no byte may come or go without effect: whole rows come and go here)
      switch (change) {
      case 0: t.src_off += 2; break;
      case 1: if (load_only) continue; t.dst_off += 2; break;
      case 2: t.src_row_stride += 2; if (!hf::slots_per_row(t) || t.end <= hf::slots_per_row(t)) { t = keep[i]; continue; } break;
      case 3: if (!hf::slots_per_row(t)) continue; t.end += 1 + hf::slots_per_row(t); break;
      case 4: if (t.end - t.first < 24 || hf::slots_per_row(t) > 8) continue; t.end -= 16; break;
      case 5: if (load_only || t.n_dst < 2) continue; --t.n_dst; break;
      case 6: l->tiles.erase(l->tiles.begin() + i); break;
      case 7: if (!load_only || (t.n_dst & ~hf::kLoadOnly) < 2) continue; --t.n_dst; break;
      default: t.end = t.first; break;
      }
      const int rc = hf::validate_plan(pl, err);
      if (rc == HF_OK) std::printf("change %d of record %zu passes\n", change, i);
      l->tiles = keep;
      REQUIRE(rc != HF_OK);
    }
  }
  return true;
}

// Row-parallel stripes of 2 to 16 bytes as the last bytes of the buffer that is read: gathered out of the
// generation buffers, the last of which is that of a first-stage rank (it ends with a down projection).
bool check_short_rows_at_the_end() {
  const int32_t ranks[] = {4, 5, 6, 7, 0, 1, 2, 3};
  for (int per_rank : {1, 3, 6, 7, 8}) {
    const hf_model_desc m{2, per_rank % 2 ? 1024 : 2048, 4, 4, 2, 4 * per_rank, 4, 2, 0};
    const hf_gen_layout gl{2, 1, HF_PLAN_HOST_ONLY | HF_GATHER_FROM_GEN, ranks, 8};
    hf::Plan pl;
    std::string err;
    REQUIRE(hf::build_plan(m, {2, 4, 1}, gl, pl, err) == HF_OK);
    REQUIRE(pl.effective_multicast() == HF_MULTICAST_PREFETCHED); // the library's own choice
    if (!check_modes(pl)) return false;
  }
  return true;
}

} // namespace

int main() {
  if (!check_short_rows_at_the_end()) return 1;
  const int hiddens[] = {1, 2, 4, 6, 8, 24, 64, 129, 136, 260}, heads[] = {1, 2, 3, 4, 8, 33}, ones[] = {1, 1, 2}, tps[] = {1, 2, 4};
  const long long tile_sizes[] = {4096, 8192, 12288, 32768, 131072};
  const unsigned flag_sets[] = {0, HF_COPY_OWN, HF_PLAN_OFFLOAD, HF_GATHER_FROM_GEN};
  for (int n = 0; n < 80; ++n) {
    const int tg = pick(tps), a = pick(tps), pg = pick(ones), b = pick(ones), t = tg * a, p = pg * b, kv = t * pick(ones);
    const hf_model_desc m{p * pick(ones), pick(hiddens), kv * pick(ones), kv, pick(heads), t * (1 + (int)rnd(70)), t * (1 + (int)rnd(9)), 2, 0};
    hf_model_desc q = m;
    q.n_q_heads = kv * (1 + (int)rnd(3));
    const hf_gen_layout gl{pg, tg, HF_PLAN_HOST_ONLY | pick(flag_sets), nullptr, 0};
    hf::Plan pl;
    pl.tile_bytes = pick(tile_sizes);
    pl.prefetch_block_bytes = 1 << (12 + rnd(6));
    pl.prefetch_merge = rnd(9);
    pl.mc_block_bytes = 1 << (12 + rnd(6));
    pl.row_interleave = rnd(4) != 0;
    std::string err;
    if (hf::build_plan(q, {p, t, 1}, gl, pl, err) != HF_OK) { std::printf("plan: %s\n", err.c_str()); return 1; }
    if (!check_modes(pl)) return 1;
    if (n % 16 == 0 && !check_validation(pl)) return 1;
  }
  std::printf("ok\n");
  return 0;
}
