// Layout of the tile table that the expert GEMMs take their work from (int32 words):
//   tiles[0] = number of row tiles; tiles[1] = number of reduction segments (a multiple of 8);
//   tiles[2 .. 2+64) = the tile counters of up to eight persistent launches (8 XCDs each, zeroed with the table);
//   tiles[kTileSeg ..)  = reduction segments (expert, row0, row1, slot), longest first, dealt out evenly to
//     the 8 XCD shares of a tile list;
//   tiles[kTileHot ..)  = number of split experts, then (expert, first slot, slots) for each;
//   tiles[kTileX .. +9) = where each XCD's share of the row tiles starts (and where the last one ends);
//   tiles[kTileHdr ..)  = row tiles as (expert, row0) pairs, experts ascending, rows ascending (tiles
//     that share a weight panel are neighbours and meet in one L2); XCD x's share is the eighth
//     [tiles[kTileX + x], tiles[kTileX + x + 1]) of them, which its work-groups take from a counter.
#pragma once
#include "r3_common.h"

namespace r3 {

constexpr int kRowTile = 256;       // rows per row tile
constexpr int kRowTokensPad = 64;   // zeros after the row->token list
constexpr int kMaxSplitSlots = 32;
constexpr int kMaxSegs = kMaxE + kMaxSplitSlots + 8;
constexpr int kTileX = 2 + 64;               // 9 ints: first row tile of every XCD's share, and the end
constexpr int kTileSeg = kTileX + 16;
constexpr int kTileHot = kTileSeg + 4 * kMaxSegs;
constexpr int kTileHdr = kTileHot + 1 + 3 * kMaxSplitSlots + 3;

}  // namespace r3
