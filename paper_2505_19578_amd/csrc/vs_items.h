// Items of the token-level rows: what the kernels that make them and the one that walks them agree on.  Plain C++, so that a
// test can compile it for the CPU.
#ifndef SP_VS_ITEMS_H
#define SP_VS_ITEMS_H
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

#endif
