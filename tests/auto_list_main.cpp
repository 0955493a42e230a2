// Host-only driver: the list that hf_reshard_execute runs while every choice is the library's (Plan::dev_auto: records,
// and bands of whole destination rows), against the tile list of the mode in force, byte by byte, on random small plans.
#include <cstdio>
#include <cstring>
#include <vector>

#include "plan.hpp"

namespace {

uint64_t g_state = 777;
uint32_t rnd(uint32_t n) { // 0 .. n-1
  g_state = g_state * 6364136223846793005ull + 1442695040888963407ull;
  return (uint32_t)((g_state >> 33) % n);
}
template <typename T, size_t N> T pick(const T (&v)[N]) { return v[rnd(N)]; }

#define REQUIRE(c)                                                                              \
  do {                                                                                          \
    if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return false; }                     \
  } while (0)

int g_bands = 0, g_joined = 0, g_kept_apart = 0, g_plans = 0;

bool check(const hf::Plan &pl) {
  const bool from_gen = pl.flags & HF_GATHER_FROM_GEN;
  const size_t n_src = from_gen ? pl.gen_bytes : pl.train_bytes;
  std::vector<uint64_t> want(pl.gen_bytes, ~0ull), got(pl.gen_bytes, ~0ull); // where every destination byte comes from
  std::vector<char> read(n_src, 0);
  for (const hf_tile &t : pl.tiles_fwd_mc)
    for (uint32_t r = 0; r < t.rows; ++r)
      for (uint32_t k = 0; k < t.row_bytes; ++k) {
        const uint64_t s = t.src_off + (uint64_t)r * t.src_row_stride + k;
        read[s] = 1;
        for (uint32_t j = 0; j < t.n_dst; ++j)
          want[(j ? pl.mc_dst[t.dst_list + j - 1] : t.dst_off) + (uint64_t)r * t.dst_row_stride + k] = s;
      }
  if (pl.dev_auto.tiles.empty()) {
    REQUIRE(!pl.has_sharing || pl.tiles_fwd_mc.empty());
    return true;
  }
  ++g_plans;
  // a load of n bytes stays inside the sources; a store writes what belongs there (again, where slots overlap)
  const auto move = [&](uint64_t from, uint64_t to, uint32_t n) {
    for (uint32_t k = 0; k < n; ++k) {
      if (from + k >= n_src || !read[from + k] || to + k >= want.size() || want[to + k] != from + k) return false;
      got[to + k] = from + k;
    }
    return true;
  };
  for (const hf::DevTile &t : pl.dev_auto.tiles) {
    REQUIRE(t.first < t.end && (t.end - t.first + hf::slots_into_kib(t)) * hf::kSlot <= pl.dev_auto.unit_bytes);
    REQUIRE(t.dst_list < pl.auto_dst.size()); // one entry is looked at in any case
    if ((t.n_dst & hf::kBand) == hf::kBand) {
      ++g_bands;
      const uint32_t n = hf::band_members(t), a = t.dst_row_stride / t.row_bytes;
      REQUIRE(n >= 1 && t.dst_list + n < pl.auto_dst.size() && t.dst_off % 128 == 0);
      for (uint32_t i = t.first; i < t.end; ++i) {
        const hf::BandSlot b = hf::band_slot(t, i);
        // the slot's bytes, one by one, by the definition of a row
        const uint64_t at = (uint64_t)i * hf::kSlot;
        REQUIRE(b.row == at / t.dst_row_stride && b.stripe == at % t.dst_row_stride / t.row_bytes && b.at == at % t.dst_row_stride % t.row_bytes);
        const uint32_t left = t.row_bytes - b.at;
        const bool joined = left < hf::kSlot;
        const uint32_t next = joined && b.stripe + 1 == a ? 0 : b.stripe + 1, next_row = b.row + (joined && b.stripe + 1 == a);
        const uint64_t s = t.src_off + hf::band_source(t, b.row, b.stripe) - t.src_off, s2 = hf::band_source(t, next_row, next);
        g_joined += joined;
        for (uint32_t j = 0; j < n; ++j) {
          const uint64_t entry = pl.auto_dst[t.dst_list + j], d = t.dst_off + (entry & hf::kBandDistance) + at;
          const uint32_t skip = (uint32_t)(entry >> 56);
          if (!joined) {
            if (skip != b.stripe + 1) REQUIRE(move(s + b.at, d, hf::kSlot));
          } else if (skip == next + 1) {
            ++g_kept_apart;
            REQUIRE(move(s + t.row_bytes - hf::kSlot, d + left - hf::kSlot, hf::kSlot));
          } else if (skip == b.stripe + 1) {
            ++g_kept_apart;
            REQUIRE(move(s2, d + left, hf::kSlot));
          } else {
            REQUIRE(move(s + b.at, d, left) && move(s2, d + left, hf::kSlot - left));
            // the two loads are of whole slots
            for (uint32_t k = 0; k < hf::kSlot; ++k) REQUIRE(read[s + t.row_bytes - hf::kSlot + k] && read[s2 + k]);
          }
        }
      }
      continue;
    }
    REQUIRE(!(t.n_dst & hf::kLoadOnly) && t.n_dst >= 1 && (t.n_dst == 1 || t.dst_list + t.n_dst - 1 <= pl.auto_dst.size()));
    for (uint32_t i = t.first; i < t.end; ++i) {
      uint32_t s, d, n = hf::kSlot;
      if (t.row_bytes < hf::kSlot) {
        s = i * t.src_row_stride;
        d = i * t.dst_row_stride;
        n = t.row_bytes;
      } else if (!hf::slot_offsets(t, i, s, d)) {
        continue;
      }
      for (uint32_t j = 0; j < t.n_dst; ++j) REQUIRE(move(t.src_off + s, t.dst_off + (j ? pl.auto_dst[t.dst_list + j - 1] : 0) + d, n));
    }
  }
  REQUIRE(got == want);
  return true;
}

bool check_plan(const hf_model_desc &m, int p, int t, int pg, int tg, int d, uint32_t flags, const std::vector<int32_t> &mat, int64_t tile, bool validate,
                bool interleave = true) {
  const hf_gen_layout gl{pg, tg, HF_PLAN_HOST_ONLY | flags, mat.empty() ? nullptr : mat.data(), (int)mat.size()};
  hf::Plan pl;
  pl.tile_bytes = tile;
  pl.row_interleave = interleave;
  std::string err;
  REQUIRE(hf::build_plan(m, {p, t, d}, gl, pl, err) == HF_OK);
  if (pl.gen_bytes > 6 << 20) return true; // it is expanded byte by byte
  bool ok = check(pl);
  if (ok && validate) {
    ok = hf::validate_plan(pl, err) == HF_OK;
    if (!ok) std::printf("validate: %s\n", err.c_str());
    // and it finds any one record changed
    for (int change = 0; ok && change < 5 && !pl.dev_auto.tiles.empty(); ++change) {
      const std::vector<hf::DevTile> keep = pl.dev_auto.tiles;
      const size_t i = rnd((uint32_t)keep.size());
      hf::DevTile &r = pl.dev_auto.tiles[i];
      switch (change) {
      case 0: r.src_off += 2; break;
      case 1: r.dst_off += 2; break;
      case 2: if ((r.n_dst & 0xFFFF) < 2) continue; --r.n_dst; break;
      case 3: pl.dev_auto.tiles.erase(pl.dev_auto.tiles.begin() + i); break;
      default: r.end = r.first; break;
      }
      if (hf::validate_plan(pl, err) == HF_OK) { std::printf("change %d of record %zu passes\n", change, i); ok = false; }
      pl.dev_auto.tiles = keep;
    }
  }
  if (!ok)
    std::printf("L %d h %d q %d kv %d hd %d F %d V %d  p %d t %d pg %d tg %d d %d flags %x mat %zu tile %lld\n", m.n_layers, m.hidden, m.n_q_heads,
                m.n_kv_heads, m.head_dim, m.ffn, m.vocab, p, t, pg, tg, d, flags, mat.size(), (long long)tile);
  return ok;
}

// Records are cut until at most one wavefront's place in nine is empty, those in front of a piece that begins inside a KiB among
// them, or until they are too small for it.
bool few_empty(const hf_model_desc &m, int p, int t, int pg, int tg, uint32_t flags) {
  hf::Plan pl;
  std::string err;
  REQUIRE(hf::build_plan(m, {p, t, 1}, {pg, tg, HF_PLAN_HOST_ONLY | flags, nullptr, 0}, pl, err) == HF_OK && !pl.dev_auto.tiles.empty());
  uint64_t slots = 0;
  for (const hf::DevTile &t : pl.dev_auto.tiles) slots += t.end - t.first;
  REQUIRE(pl.dev_auto.unit_bytes % 16384 || pl.dev_auto.tiles.size() * (pl.dev_auto.unit_bytes / hf::kSlot) <= slots + slots / 8);
  return true;
}

// Row-parallel pieces whose rows are longer than one record can hold (2^24 slots a row), stripe after stripe: every byte has its
// slot.  Such a plan is too large to expand; what is counted are the slots of rows that lie on 128-byte boundaries.
bool long_rows(int ffn) {
  const hf_model_desc m{1, 2, 4, 4, 1, ffn, 4, 2, 0};
  hf::Plan pl;
  pl.row_interleave = 0;
  std::string err;
  REQUIRE(hf::build_plan(m, {1, 4, 1}, {1, 1, HF_PLAN_HOST_ONLY | HF_COPY_OWN, nullptr, 0}, pl, err) == HF_OK);
  uint64_t want = 0, slots = 0;
  for (const auto *descs : {&pl.fwd_peer, &pl.fwd_own})
    for (const hf_desc &d : *descs)
      if (d.tensor_id == HF_G_DOWN) want += (uint64_t)d.rows * d.row_bytes;
  const auto down = pl.gen_tab[0].at(HF_G_DOWN, 0);
  const uint64_t bytes = (uint64_t)down.rows * down.cols * 2;
  for (const hf::DevTile &t : pl.dev_auto.tiles) {
    bool in = false;
    for (int r = 0; r < 4; ++r) in = in || t.dst_off - (pl.gen_tab[r].base + down.off) < bytes;
    if (!in) continue;
    REQUIRE((t.n_dst & hf::kBand) != hf::kBand && t.row_bytes % 128 == 0 && hf::boundary_mask(t) == 0);
    REQUIRE(hf::slots_per_row(t) ? hf::slots_per_row(t) == t.row_bytes / hf::kSlot : (uint64_t)t.end * hf::kSlot <= t.row_bytes);
    slots += (uint64_t)(t.end - t.first) * t.n_dst;
  }
  REQUIRE(want == 4 * bytes && slots * hf::kSlot == want);
  return true;
}

} // namespace

int main() {
  const int hiddens[] = {8, 24, 64, 72, 129, 136, 260}, heads[] = {1, 4, 8, 33, 65}, ones[] = {1, 1, 2}, tps[] = {1, 2, 4}, as[] = {2, 2, 4, 4, 8};
  const long long tile_sizes[] = {4096, 8192, 12288, 32768, 131072};
  const unsigned flag_sets[] = {0, 0, HF_COPY_OWN, HF_GATHER_FROM_GEN, HF_GROUPING_VANILLA};
  for (int n = 0; n < 120; ++n) {
    const int tg = pick(tps), a = pick(as), pg = pick(ones), b = pick(ones), t = tg * a, p = pg * b, kv = t * pick(ones), d = pick(ones);
    hf_model_desc m{p * pick(ones), pick(hiddens), kv * (1 + (int)rnd(3)), kv, pick(heads), t * (1 + (int)rnd(90)), t * (1 + (int)rnd(9)), 2, 0};
    const unsigned flags = pick(flag_sets);
    // some of the ranks, in any order
    std::vector<int32_t> mat;
    if (flags != HF_GATHER_FROM_GEN && rnd(3) == 0) {
      for (int r = 0; r < p * t * d; ++r)
        if (rnd(3)) mat.insert(mat.begin() + rnd((uint32_t)mat.size() + 1), r);
    }
    if (!check_plan(m, p, t, pg, tg, d, flags, mat, pick(tile_sizes), n % 7 == 0)) return 1;
  }
  // rows long enough for every phase of a slot against a line, several records per tensor
  for (int cols : {8, 9, 15, 63, 64, 65, 171, 513})
    if (!check_plan({1, 64, 4, 4, cols, 4 * cols, 4, 2, 0}, 1, 4, 1, 1, 1, cols % 2 ? 0u : (uint32_t)HF_COPY_OWN, {}, 8192, false)) return 1;
  // pieces a little shorter than a power of two, hidden 128 to 1024
  for (int h = 128; h <= 1024; h *= 2)
    for (uint32_t flags : {0u, (uint32_t)HF_COPY_OWN, (uint32_t)HF_GATHER_FROM_GEN})
      for (int tg : {1, 2})
        if (!few_empty({4, h, h / 16, 8, 16, h * 3 / 8 * 8, 3200, 2, 0}, 1, 8, 1, tg, flags) ||
            !few_empty({4, h, h / 16, 8, 16, h * 15 / 8, 3200, 2, 0}, 2, 4, 1, tg, flags)) return 1;
  for (int ffn : {1 << 27, 1 << 28, 1 << 29})
    if (!long_rows(ffn)) {
      std::printf("rows of %d elements\n", ffn);
      return 1;
    }
  // shards' regions in an order that no step describes: no bands, the same bytes; in their own order there are bands
  for (const std::vector<int32_t> &order : {std::vector<int32_t>{2, 0, 3, 1}, std::vector<int32_t>{0, 1, 2, 3}}) {
    const int before = g_bands;
    if (!check_plan({2, 64, 4, 4, 16, 256, 8, 2, 0}, 1, 4, 1, 1, 1, HF_GATHER_FROM_GEN, order, 4096, true)) return 1;
    if ((g_bands == before) != (order[0] == 2)) {
      std::printf("%d bands with rank %d first\n", g_bands - before, order[0]);
      return 1;
    }
  }
  // stripe after stripe: the same bytes without bands
  const int bands = g_bands;
  for (uint32_t flags : {0u, (uint32_t)HF_COPY_OWN, (uint32_t)HF_GATHER_FROM_GEN}) {
    if (!check_plan({2, 64, 4, 4, 16, 512, 8, 2, 0}, 1, 4, 1, 1, 1, flags, {}, 4096, true, false)) return 1;
    if (g_bands != bands) {
      std::printf("%d bands without row interleave\n", g_bands - bands);
      return 1;
    }
    if (!check_plan({2, 64, 4, 4, 16, 512, 8, 2, 0}, 1, 4, 1, 1, 1, flags, {}, 4096, true)) return 1;
    if (g_bands == bands) {
      std::printf("no bands with row interleave\n");
      return 1;
    }
    g_bands = bands;
  }
  if (g_bands < 300 || g_joined < 500 || g_kept_apart < 100 || g_plans < 40) {
    std::printf("bands %d joined %d kept apart %d plans %d\n", g_bands, g_joined, g_kept_apart, g_plans);
    return 1;
  }
  std::printf("ok\n");
  return 0;
}
