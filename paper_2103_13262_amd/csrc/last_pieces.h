// Which workgroups take the tiles of the experts' last pieces in a launch of whole tiles that another product follows (internal;
// compiled for the host as well).
#pragma once

namespace moe {

// The big tiles go round the W workgroups of each of the 8 XCDs from the first on; the number of the first one that gets no tile
// of the last round.
constexpr int first_free_workgroup(long big_tiles, int W) { return (int)((big_tiles + 7) / 8 % W); }

// The last pieces, in tiles of their own behind that round: up to this many stay with each of the workgroups that it left
// free, more go round all workgroups from the first free one on.  A big tile moves 4/3 of what a last piece's tile moves, so one
// or two of them end with the big tiles' last round or soon after; a third makes the launch longer.  dXs with dW1 of 40
// drawn loads (9 to 123 experts, 3696 to 19220 tokens, top-1 and top-2, Zipf 0 to 1.3, h 2048 to 5984): with 2 to 4 per free
// workgroup, going round all takes 12 % less on average (up to 30 %: N 4493, d 1632, h 5760, 10 experts, 581 -> 404 us) than staying;
// with 1 to 2 staying takes 2.3 % less (up to 13 %: N 12696, d 992, h 4320, 47 experts, 696 -> 606 us).
constexpr int kLastPiecesEach = 2;

// tiles: the last pieces' tiles as they are computed (pieces times column tiles of that width).
constexpr bool last_pieces_stay(long tiles, int first_free, int W) { return tiles <= 8L * kLastPiecesEach * (W - first_free); }

}  // namespace moe
