// The reach of a traceback walk's fetch (sw16.hip), in plain C++ so that a host
// program can check it.
#pragma once

namespace pastis {

// Lane slots (of RP rows each) and columns that a fetch of W lanes holds: at
// least 16 rows where a strip has one piece.
constexpr int walk_slots(int RP, bool multi) { return multi || RP > 8 ? 1 : (15 + RP) / RP; }
constexpr int walk_cols(int W) { return W < 16 ? 16 : W; }
// Row of the fetch's first slot, where its last one holds row block blk (below 0
// near the top of a).
constexpr int walk_first_row(int blk, int RP, int slots) { return (blk - (slots - 1)) * RP; }
// Does the fetch fill row r (counted from its first row r0) of a's la residues?
constexpr bool walk_holds_row(int r0, int r, int la) { return r0 + r >= 0 && r0 + r < la; }
// May a lane look at row r and column c of the fetch, which holds cend columns?
// Rows above a's first are in the fetch's LDS but never filled: their residues
// would index the score table anywhere.
constexpr bool walk_reads(int r0, int r, int c, int cend) {
    return r >= 0 && r0 + r >= 0 && c < cend;
}

}  // namespace pastis
