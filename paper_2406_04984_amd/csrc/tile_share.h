// The deal of a list of tiles that every XCD holds whole.  Plain C++ but for the function attributes, so that a host program
// can check it.
#pragma once
#include "tile_div.h"

namespace meft {

// First of the tiles 0 .. all - 1 that are part x of 8 (the part ends where x + 1 begins): consecutive ones, so that the tiles of a
// group, and those of a column, which share its rows of B, are as few parts' as can be.  No two parts differ by more than one tile.
// all < 2^28.
MEFT_HOST_DEVICE int tile_share_first(int all, int x) { return (int)((uint32_t)all * (uint32_t)x >> 3); }

}  // namespace meft
