// The device's view of a work list: records that the kernels walk, and the arithmetic that
// maps a position in a record ("slot") to bytes.  Shared by the planner (host), the kernels
// and a host test.  Not part of the ABI.
//
// A slot is what one lane moves at a time: 16 bytes.  The rows of a tile are cut into slots on
// the DESTINATION's grid, not from the row's first byte on: slot c of a row covers the bytes
// [16 c - lead, 16 c - lead + 16) of it, where lead is the distance of the row's first byte
// from the boundary before it.  Slots that stick out at either end of the row are moved inside
// (they then overlap their neighbour and write the same bytes again), so that rows of any even
// length >= 16 at any even address are copied with 16-byte accesses only; gfx950 takes them at any
// alignment.  Rows below 16 bytes are one slot each, copied as their first and last 8, 4 or 2 bytes.
#pragma once
#include <cstdint>

#include "hfreshard.h"

#if defined(__HIP__)
#define HF_HD __attribute__((host, device)) inline
#else
#define HF_HD inline
#endif

namespace hf {

constexpr uint32_t kSlot = 16;
constexpr uint32_t kLoadOnly = 0x80000000u; // DevTile::n_dst: kLoadOnly | number of chunks
constexpr uint32_t kBand = 0xC0000000u;     // DevTile::n_dst: kBand | number of destinations (see band_slot)
constexpr uint32_t kBandApart = 0x20000000u; // and: the source's rows are whole rows too
constexpr uint32_t kBandParts = 0x10000000u; // and: lines are written in part (at the edges of stripes left out)

struct DevTile {
  uint64_t src_off, dst_off;
  uint32_t first, end; // slots [first, end) of the geometry below
  uint32_t row_bytes, src_row_stride, dst_row_stride;
  uint32_t slots;      // bits 0..23: slots per row, 0 = one row; bits 24..30: boundary - 1 (127 or 15), or
                       // 0 = every row starts on a boundary and is a whole number of slots; bit 31: see shares_lines
  uint32_t n_dst;      // copies: destinations.  kLoadOnly | c: the slots of c sources, dst_list bytes
                       // apart, are loaded and stored nowhere (they are brought into L2); the rows
                       // of such a record have 16 bytes or more
  uint32_t dst_list;   // copies: position of destinations 2..n_dst in the list of extra offsets
};
static_assert(sizeof(DevTile) == 48, "one record of the device list");

HF_HD uint32_t slots_per_row(const DevTile &t) { return t.slots & 0xFFFFFFu; }
HF_HD uint32_t boundary_mask(const DevTile &t) { return t.slots >> 24 & 127; }
// Two wavefronts want parts of the same 64-byte half of a line of the source.  Such a record is loaded with
// plain loads.  What leaves L2 is the same under either kind (every XCD that wants a part of a line fetches it:
// 1.27 times the payload for rows of 1026 bytes), but the second fetch is served sooner, by the memory-side cache
// as it seems, where non-temporal loads leave nothing.  Row-parallel tensors alone, one to one, 4
// GB, TB/s: rows of 1026 bytes 4.4 -> 5.4, 1040 4.6 -> 5.7, 2050 5.0 -> 6.1, 4098 5.65 -> 6.3; whole model with
// rows of 1410 bytes 6.5 -> 6.9.  Rows of whole halves (2752) gain alone (6.0 -> 6.35) but not in whole
// models (6.77 either way, 6.74 with hidden 2048), so the line lies at 64 bytes.
constexpr uint32_t kSharesLines = 0x80000000u;
HF_HD bool shares_lines(const DevTile &t) { return t.slots & kSharesLines; }

// Offsets of slot `col` of row `row` on either side; false: nothing to do in this slot.  Needs
// row_bytes >= 16.
HF_HD bool slot_offsets(const DevTile &t, uint32_t row, uint32_t col, uint32_t &src, uint32_t &dst) {
  src = row * t.src_row_stride;
  dst = row * t.dst_row_stride;
  const int32_t q = (int32_t)(col * kSlot) - (int32_t)(((uint32_t)t.dst_off + dst) & boundary_mask(t));
  const uint32_t last = t.row_bytes - kSlot, at = q < 0 ? 0u : (uint32_t)q < last ? (uint32_t)q : last;
  src += at;
  dst += at;
  return q > -(int32_t)kSlot && q < (int32_t)t.row_bytes;
}

// The same for slot i of the record.
HF_HD bool slot_offsets(const DevTile &t, uint32_t i, uint32_t &src, uint32_t &dst) {
  const uint32_t per_row = slots_per_row(t);
  uint32_t row = 0;
  if (per_row) row = i / per_row; // uniform over the record
  const uint32_t col = i - row * per_row;
  if (boundary_mask(t)) return slot_offsets(t, row, col, src, dst); // uniform
  src = row * t.src_row_stride + col * kSlot;
  dst = row * t.dst_row_stride + col * kSlot;
  return true;
}

// A band: a run of whole destination rows of a row-parallel tensor, put together from the column stripes of its
// a training shards (Section 5.3: the shards inside one generation shard).  Slots lie on the destination, whose rows
// follow one another without a gap, so that every line is written whole by one wavefront, also where two stripes meet in
// it.  In a DevTile: src_off = stripe 0 of row 0, stripe k src_row_stride pages of 4 KiB further on; row_bytes = a
// stripe's row (16 bytes or more), and the distance of its rows (kBandApart: the stripes lie in whole rows of
// their own, as in the destination); dst_off = row 0 of the first
// destination, dst_row_stride = a whole row; slots [first, end) counted from row 0; slots = the row in which slot
// `first` begins.  Destination j is listed at dst_list + j: the distance from the first one and, in the
// uppermost byte, 1 + the stripe that is not copied there (its own, resident piece), or 0.
struct BandSlot {
  uint32_t row, stripe, at; // where the slot's first byte comes from; `at` is counted from the stripe's row
};
// n / d and what is left, for n < 2^24 and 16 <= d; inv = 1 / d to 22 bits
HF_HD uint32_t divide_by(uint32_t n, uint32_t d, float inv, uint32_t &rest) {
  uint32_t q = (uint32_t)((float)n * inv);
  rest = n - q * d;
  if ((int32_t)rest < 0) { --q; rest += d; }
  if (rest >= d) { ++q; rest -= d; }
  return q;
}
HF_HD float reciprocal(uint32_t d) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_rcpf((float)d);
#else
  return 1.0f / (float)d;
#endif
}
// slot i of a band, first <= i < end
HF_HD BandSlot band_slot(const DevTile &t, uint32_t i) {
  BandSlot b;
  uint32_t col;
  b.row = t.slots + divide_by(i * kSlot - t.slots * t.dst_row_stride, t.dst_row_stride, reciprocal(t.dst_row_stride), col);
  b.stripe = divide_by(col, t.row_bytes, reciprocal(t.row_bytes), b.at);
  return b;
}
HF_HD uint64_t band_source(const DevTile &t, uint32_t row, uint32_t stripe) { // the first byte of a stripe's row
  const uint32_t in_shard = t.n_dst & kBandApart ? row * t.dst_row_stride + stripe * t.row_bytes : row * t.row_bytes;
  return t.src_off + ((uint64_t)t.src_row_stride << 12) * stripe + in_shard;
}
HF_HD uint32_t band_members(const DevTile &t) { return t.n_dst & 0xFFFFu; }
constexpr uint64_t kBandDistance = (1ull << 56) - 1; // the rest of an entry of the destination list is the stripe
constexpr uint32_t kBandLargest = 1u << 22;          // record and row together stay below 2^24 bytes

// Records of Plan::dev_auto: slots between the KiB of the destination that slot `first` lies in and that slot, where the record
// is a band or one row (the KiB of all destinations lie alike).
HF_HD uint32_t slots_into_kib(const DevTile &t) {
  const bool band = (t.n_dst & kBand) == kBand;
  if (!band && slots_per_row(t)) return 0;
  return (((uint32_t)t.dst_off & ~(band ? 0u : boundary_mask(t))) / kSlot + t.first) & 63;
}

// b / parts, for the kernels that give every record `parts` workgroups.  The division stands in front of everything else a
// workgroup does, so the host brings 2^(32 + k) / parts, rounded up, where k is log2 of parts, rounded down (below 2^32 but for
// powers of two).  Exact for b < 2^31: rounding up adds less than b / 2^(32 + k) < 1 / 2^(k + 1) < 1 / parts to the quotient.
HF_HD uint32_t log2_of(uint32_t parts) { return 31 - (uint32_t)__builtin_clz(parts); }
HF_HD uint32_t record_of(uint32_t b, uint32_t parts, uint32_t inverse) {
  const uint32_t q = parts & (parts - 1) ? (uint32_t)((uint64_t)b * inverse >> 32) : b; // uniform
  return q >> log2_of(parts);
}
inline uint32_t inverse_of(uint32_t parts) { return parts & (parts - 1) ? (uint32_t)(((1ull << (32 + log2_of(parts))) + parts - 1) / parts) : 0; }

// What workgroup b copies.  Workgroups go to the XCDs in turn.  group 0: the parts of a record follow one another and
// fall to all XCDs.  group 3: of every eight whole records each XCD has one (where there are no eight left, as group 0), so that
// a record, and a line of the source that two parts of it share, is fetched into one L2 and not into several.
struct Place {
  uint32_t record, part;
};
HF_HD Place place_of(uint32_t b, uint32_t parts, uint32_t inverse, uint32_t n_records, uint32_t group) {
  Place p;
  p.record = record_of(b, parts, inverse);
  p.part = b - p.record * parts;
  const uint32_t others = (1u << group) - 1, first = p.record & ~others;
  if (first + others < n_records) { // uniform
    const uint32_t i = b - first * parts;
    p.record = first + (i & others);
    p.part = i >> group;
  }
  return p;
}

// Slot geometry of rows that start at dst_off, dst_off + dst_row_stride, ... (rows of them):
// fills `slots`, returns the number of slots in all.
//
// 128-byte boundaries (the cache line) are taken where they keep a line from being written by two
// wavefronts and cost at most one slot in eight: a wavefront's 64 slots then are whole lines.
// Measured against 16-byte boundaries everywhere: rows of 2752 bytes (Llama-7B down projection, 22
// lines for 21.5) 8.43 against 8.50 ms for the whole transition, 10.48 against 10.59 with own pieces;
// rows of 1026 bytes (72 slots for 65, just inside the limit) 257 against 266 us.  Tried as a limit
// of one slot in 32 too: the same as none for the 1026-byte rows.  lines = false: 16-byte boundaries
// only (reload reads the host image, whose lines matter more there than the destination's).
inline uint32_t slot_geometry(uint64_t dst_off, uint32_t rows, uint32_t row_bytes, uint32_t dst_row_stride, uint32_t vec_bytes,
                              uint32_t &slots, bool lines = true) {
  if (row_bytes < kSlot) {
    slots = 1;
    return rows;
  }
  const auto lead_of = [&](uint32_t boundary) -> uint32_t { // largest over the rows (even addresses)
    if (rows == 1 || dst_row_stride % boundary == 0) return (uint32_t)dst_off % boundary;
    return boundary - vec_bytes;
  };
  const uint32_t lead16 = lead_of(16), lead128 = lines ? lead_of(128) : 0; // lead16 is 0 where vec_bytes is 16
  const uint32_t n16 = (lead16 + row_bytes + kSlot - 1) / kSlot;
  if (rows == 1) {
    slots = lead128 ? 127u << 24 : vec_bytes == kSlot ? 0 : 15u << 24;
    return ((lead128 ? lead128 : lead16) + row_bytes + kSlot - 1) / kSlot;
  }
  const uint32_t n128 = (lead128 + row_bytes + 127) / 128 * 8;
  const bool lines_whole = vec_bytes == kSlot && (dst_row_stride == row_bytes || (lead128 == 0 && row_bytes % 128 == 0));
  const bool on_lines = lines && !lines_whole && n128 <= n16 + n16 / 8;
  slots = on_lines ? n128 | 127u << 24 : vec_bytes == kSlot ? n16 : n16 | 15u << 24;
  return rows * (slots & 0xFFFFFFu);
}

// kSharesLines or 0, for the geometry that slot_geometry has put into `slots`
inline uint32_t source_lines(uint64_t src_off, uint64_t dst_off, uint32_t rows, uint32_t row_bytes, uint32_t src_row_stride, uint32_t slots) {
  if (rows == 1) return (src_off - (slots >> 24 == 127 ? dst_off % 128 : 0)) % 64 ? kSharesLines : 0;
  return src_off % 64 || src_row_stride % 64 || row_bytes % 64 ? kSharesLines : 0;
}

} // namespace hf
