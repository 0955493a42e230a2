// Host-only driver: how the kernels that give every record the same number of workgroups find a workgroup's record and part, how
// many of them the lists leave empty, and how the automatic list is launched.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "plan.hpp"

#define REQUIRE(c)                                                                              \
  do {                                                                                          \
    if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return false; }                     \
  } while (0)

namespace {

// exact up to the largest grid (2^26 workgroups) and beyond
bool division() {
  for (uint32_t parts = 1; parts <= 4096; ++parts) {
    const uint32_t inverse = hf::inverse_of(parts);
    for (uint64_t q : {0ull, 1ull, 2ull, 12345ull, (1ull << 26) / parts, 0x7FFFFFFFull / parts})
      for (int64_t rest : {-1ll, 0ll, 1ll, (long long)parts / 2, (long long)parts - 1, (long long)parts}) {
        const int64_t b = (int64_t)(q * parts) + rest;
        if (b >= 0 && b <= 0x7FFFFFFF) REQUIRE(hf::record_of((uint32_t)b, parts, inverse) == (uint32_t)b / parts);
      }
  }
  return true;
}

// every part of every record once; eight whole records at a time, each with all its parts on one XCD
bool places() {
  for (uint32_t group : {0u, 3u})
    for (uint32_t parts : {1u, 3u, 8u, 13u, 16u, 104u, 128u})
      for (uint32_t n : {1u, 7u, 8u, 9u, 16u, 31u}) {
        std::vector<int> seen(n * parts, 0), xcd(n, -1);
        for (uint32_t b = 0; b < n * parts; ++b) {
          const hf::Place p = hf::place_of(b, parts, hf::inverse_of(parts), n, group);
          REQUIRE(p.record < n && p.part < parts);
          ++seen[p.record * parts + p.part];
          if (group == 0) REQUIRE(p.record == b / parts && p.part == b % parts);
          if (group == 3 && p.record < n / 8 * 8) {
            if (xcd[p.record] < 0) xcd[p.record] = (int)(b % 8);
            REQUIRE(xcd[p.record] == (int)(b % 8));
          }
        }
        for (int s : seen) REQUIRE(s == 1);
      }
  return true;
}

// Pieces that are a little longer than a power of two or than a tile: one remainder each, few workgroups empty, records that
// begin where the one before ends.
bool lists(int hidden, int ffn, int64_t tile) {
  hf::Plan pl;
  std::string err;
  pl.tile_bytes = tile;
  REQUIRE(hf::build_plan({4, hidden, 8, 8, hidden / 8, ffn, 3208, 2, 0}, {1, 4, 1}, {1, 2, HF_PLAN_HOST_ONLY, nullptr, 0}, pl, err) == HF_OK);
  for (const hf::DevList *l : {&pl.dev_fwd, &pl.dev_own, &pl.dev_back}) {
    REQUIRE(!l->tiles.empty() && l->unit_bytes <= (uint64_t)tile && (l->unit_bytes == (uint64_t)tile || l->unit_bytes % 8192 == 0));
    uint64_t slots = 0, remainders = 0, pieces = 0;
    for (const hf::DevTile &t : l->tiles) {
      REQUIRE(t.first < t.end && (t.end - t.first) * hf::kSlot <= l->unit_bytes);
      REQUIRE(t.first == 0 || (&t)[-1].end == t.first);
      slots += t.end - t.first;
      pieces += t.first == 0;
      remainders += (t.end - t.first) * hf::kSlot < l->unit_bytes;
    }
    REQUIRE(remainders <= pieces);
    REQUIRE(l->unit_bytes <= 8192 || l->tiles.size() * (l->unit_bytes / hf::kSlot) <= slots + slots / 8);
  }
  REQUIRE(hf::validate_plan(pl, err) == HF_OK);
  return true;
}

// The automatic list, hidden 768 with rows of 1026 bytes: the largest half of the tile size whose records leave at most one workgroup in nine empty, no
// finer one (a quarter of it leaves fewer empty, and moves the bytes no faster).
bool automatic(int64_t tile) {
  hf::Plan pl;
  std::string err;
  pl.tile_bytes = tile;
  REQUIRE(hf::build_plan({24, 768, 12, 12, 64, 2052, 5004, 2, 0}, {1, 4, 1}, {1, 1, HF_PLAN_HOST_ONLY, nullptr, 0}, pl, err) == HF_OK && pl.runs_auto());
  const auto records = [&](uint64_t unit) {
    uint64_t n = 0, piece = 0;
    for (const hf::DevTile &t : pl.dev_auto.tiles) {
      if (t.first == 0) {
        n += (piece + unit / hf::kSlot - 1) / (unit / hf::kSlot);
        piece = hf::slots_into_kib(t);
      }
      piece += t.end - t.first;
    }
    return n + (piece + unit / hf::kSlot - 1) / (unit / hf::kSlot);
  };
  uint64_t slots = 0, unit = (uint64_t)tile;
  for (const hf::DevTile &t : pl.dev_auto.tiles) slots += t.end - t.first;
  while (unit % 16384 == 0 && records(unit) * (unit / hf::kSlot) > slots + slots / 8) unit /= 2;
  REQUIRE(pl.dev_auto.unit_bytes == unit && pl.dev_auto.tiles.size() == records(unit));
  return true;
}

// How automatic lists are launched, on both sides of the lines.
struct Choice { int hidden, heads, ffn, layers, tp, gen_tp; uint32_t flags; bool short_list, paced; int policy, wgs_per_cu; };
bool launches() {
  const uint32_t own = HF_COPY_OWN, gen = HF_GATHER_FROM_GEN;
  for (const Choice &c : {
           Choice{256, 4, 704, 2, 4, 1, 0, true, false, 5, 0}, Choice{256, 4, 704, 5, 4, 1, 0, false, true, 5, 25}, // three destinations
           Choice{256, 8, 712, 2, 8, 1, 0, true, false, 5, 0}, Choice{256, 8, 712, 6, 8, 1, 0, false, true, 1, 25}, // seven
           Choice{256, 4, 704, 2, 2, 1, own, true, false, 1, 0}, Choice{512, 8, 1412, 4, 2, 1, own, false, false, 1, 0}, // two
           // three destinations: a CU is not filled up, whatever the records (all that fit: 10, 9 and 3 % slower), unless slots are joined
           Choice{320, 8, 960, 96, 8, 2, 0, false, true, 5, 25}, Choice{192, 4, 544, 96, 4, 1, gen, false, true, 5, 25}, Choice{320, 4, 832, 96, 4, 1, 0, false, true, 5, 25},
           Choice{768, 12, 2052, 24, 4, 1, 0, false, true, 5, 0},
           // four, records of 8 KiB: below the line non-temporal stores are 2 % slower, above it 4 % faster
           Choice{256, 4, 640, 40, 4, 1, own, false, true, 1, 25}, Choice{288, 4, 768, 40, 4, 1, own, false, true, 1, 25}, Choice{256, 4, 640, 96, 4, 1, own, false, true, 5, 25},
           Choice{1024, 8, 2688, 12, 4, 1, own, false, true, 1, 25}, Choice{768, 12, 2052, 12, 4, 1, own, false, true, 5, 25}}) {
    hf::Plan pl;
    std::string err;
    REQUIRE(hf::build_plan({c.layers, c.hidden, c.heads, c.heads, c.hidden / c.heads, c.ffn, 4096, 2, 0}, {1, c.tp, 1},
                           {1, c.gen_tp, c.flags | HF_PLAN_HOST_ONLY, nullptr, 0}, pl, err) == HF_OK && pl.runs_auto());
    const hf::AutoLaunch a = hf::auto_launch(pl);
    if (a.short_list != c.short_list || a.paced != c.paced || a.policy != c.policy || a.wgs_per_cu != c.wgs_per_cu) {
      std::printf("hidden %d layers %d TP %d -> %d, %.0f MB: short %d paced %d policy %d per CU %d\n", c.hidden, c.layers, c.tp, c.gen_tp, pl.dev_auto.bytes / 1e6,
                  a.short_list, a.paced, a.policy, a.wgs_per_cu);
      return false;
    }
  }
  return true;
}

// Short one-to-one lists take non-temporal stores where many lines are written in part and the list is 12 MiB or longer: below, a call alone
// is 4 % slower with them.
struct Stores { int hidden, ffn, layers, tp, gen_tp; bool in_part, non_temporal; };
bool stores_of_short_lists() {
  for (const Stores &c : {Stores{256, 688, 2, 4, 2, true, false}, Stores{256, 688, 3, 4, 2, true, false}, Stores{256, 688, 4, 4, 2, true, true}, // 8.4, 11.6 and 14.7 MB
                          Stores{512, 1408, 1, 2, 1, false, false}}) { // 17 MB of whole lines
    hf::Plan pl;
    std::string err;
    REQUIRE(hf::build_plan({c.layers, c.hidden, 4, 4, c.hidden / 4, c.ffn, 1024, 2, 0}, {1, c.tp, 1}, {1, c.gen_tp, HF_PLAN_HOST_ONLY, nullptr, 0}, pl, err) == HF_OK);
    REQUIRE(pl.dev_fwd.one_to_one && pl.dev_fwd.bytes <= 24u << 20 && pl.dev_fwd.parts_of_lines == c.in_part);
    if (hf::non_temporal_when_short(pl.dev_fwd) != c.non_temporal) {
      std::printf("hidden %d layers %d, %.1f MB\n", c.hidden, c.layers, pl.dev_fwd.bytes / 1e6);
      return false;
    }
  }
  return true;
}

// Lists that read a piece again for each destination are no one-to-one lists, and keep the records of their tiles.
bool one_to_one() {
  const int32_t alone[] = {0};
  for (int ranks : {0, 1}) { // all; one, whose pieces nobody else wants
    hf::Plan pl;
    std::string err;
    REQUIRE(hf::build_plan({3, 512, 8, 8, 64, 1416, 1116, 2, 0}, {1, 4, 1}, {1, 1, HF_PLAN_HOST_ONLY, ranks ? alone : nullptr, ranks}, pl, err) == HF_OK);
    pl.multicast_auto = false;
    pl.multicast = HF_MULTICAST_OFF;
    hf::build_forward_lists(pl);
    REQUIRE(pl.effective_multicast() == HF_MULTICAST_OFF && pl.has_sharing == !ranks && pl.dev_fwd.one_to_one == !pl.has_sharing);
    REQUIRE(pl.dev_own.one_to_one && pl.dev_back.one_to_one);
    if (!pl.has_sharing) continue;
    size_t pieces = 0;
    for (const hf::DevTile &t : pl.dev_fwd.tiles) pieces += t.first == 0;
    REQUIRE(pieces == pl.n_tiles_fwd_peer); // not joined
  }
  return true;
}

} // namespace

int main() {
  if (!division() || !places() || !launches() || !stores_of_short_lists() || !one_to_one()) return 1;
  for (int64_t tile : {65536ll, 131072ll, 1ll << 20})
    if (!automatic(tile)) return 1;
  for (int hidden : {64, 136, 520, 1032})
    for (int ffn : {260, 1036, 2060})
      for (int64_t tile : {4096ll, 8192ll, 20480ll, 131072ll, 1ll << 20})
        if (!lists(hidden, ffn, tile)) {
          std::printf("hidden %d ffn %d tile %lld\n", hidden, ffn, (long long)tile);
          return 1;
        }
  std::printf("ok\n");
  return 0;
}
