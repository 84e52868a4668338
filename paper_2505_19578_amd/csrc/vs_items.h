// Items of the token-level rows: what the kernels that make them and the one that walks them agree on.  Plain C++, so that a
// test can compile it for the CPU.
#ifndef SP_VS_ITEMS_H
#define SP_VS_ITEMS_H
#include <cstddef>
#include <cstdint>

// One item of a row's work list: 64 keys, a packed K image followed by the V image.  code: the 64-key tile of the sequence,
// or with VS_GATHERED the gathered image; v: keys of the item that every query of the row may attend to, whatever its
// offsets (kept keys of a tile; of a gathered image those that no band holds; all of the sink and, forced, the diagonal).
struct alignas(16) VsItem {
  uint32_t code, unused;
  uint64_t v;
};
constexpr uint32_t VS_GATHERED = 1u << 31;

// How many tiles an item lies below a row's first tile: 1 and more below the row, 0 and -1 on the diagonal.  For a gathered
// image it means nothing (no offset is read), but the mask is computed from it all the same.
constexpr int vs_tiles_below(int first_tile, uint32_t code) { return first_tile - (int)(code & ~VS_GATHERED); }

// The room for the items: what the vertical-slash search keeps for its statistics, which is done by then (the sizes that callers
// have been told: every logit of a query block and two numbers per query), less the bitmaps of the bands, any / all.
constexpr size_t vs_round_up(size_t x) { return (x + 255) / 256 * 256; }
constexpr size_t vs_statistics_bytes(size_t maps, size_t seq, size_t block) {
  return vs_round_up(maps * block * seq * sizeof(float)) + vs_round_up(maps * block * 2 * sizeof(float));
}
constexpr size_t vs_band_bytes(size_t maps, size_t seq) {
  return vs_round_up(maps * 2 * ((seq / 64 + 63) / 64) * sizeof(uint64_t));
}
// in items of one head
constexpr int64_t vs_item_room(size_t maps, size_t seq, size_t block) {
  return (int64_t)((vs_statistics_bytes(maps, seq, block) - vs_band_bytes(maps, seq)) / sizeof(VsItem) / maps);
}
// Items before those of row i, where rows row0, .. each have a place for every tile they reach, spb (r + 1) of row r.
constexpr int64_t vs_items_before(int64_t i, int64_t row0, int64_t spb) { return (i * (i + 1) - row0 * (row0 + 1)) / 2 * spb; }
// First row of the launch that ends before row1: as many rows as have room; row1 if not even one has.
constexpr int vs_first_row(int row1, int64_t room, int64_t spb) {
  int row0 = row1;
  while (row0 > 0 && vs_items_before(row1, row0 - 1, spb) <= room) --row0;
  return row0;
}

#endif
