// Where the lanes of a 16 x 16 MFMA find their share of a K-step in LDS, for operand rows that lie there as the formats have them.  On the host as well, so that it
// can be looked at without a GPU.
//
// Lane 16 q + c has row c and a quarter of the K-step.  Which quarter is q's is free, as long as both operands have it alike, and it decides about the banks: a
// 16-byte read takes the lanes of half a wave in two goes, 0 - 3 with 12 - 15 and 20 - 27, then the others, so that what must not meet are rows 0 - 3 and 12 - 15 of an even q and
// rows 4 - 11 of the odd one behind it.  LDS cycles that are conflicts, with quarter q as q's own / as here: int8 codes with resident weights 48 / 0 % (the LDS active 35 / 18 % of
// a launch), E2M3 38 / 24 %, in 256 x 256 tiles 41 / 28 %: the 8-byte reads of E2M3 meet instead, which take half a wave at once (2 cycles of 8, where it was 4 of 10).
#pragma once

namespace qvggt {

// int8 blocks: four 16-byte chunks a row of 64 bytes, whose places are swizzled with bits 2 and 3 of the row
constexpr int i8_quarter(int q) { return q ^ ((q & 1) << 1); }
constexpr int i8_place(int row, int q) { return row * 64 + ((i8_quarter(q) ^ (row >> 2 & 3)) << 4); }

// E2M3: two K-tiles, each with two blobs a row of 48 bytes: 16 bytes of a blob here, its other 8 e2m3_rest() behind them
constexpr int e2m3_tile(int q) { return q & 1; }
constexpr int e2m3_blob(int q) { return q >> 1; }
constexpr int e2m3_place(int row, int q, int tile_bytes) { return e2m3_tile(q) * tile_bytes + row * 48 + e2m3_blob(q) * 16; }
constexpr int e2m3_rest(int q) { return 32 - 8 * e2m3_blob(q); }

}  // namespace qvggt
