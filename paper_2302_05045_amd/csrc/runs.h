// Which entries of idx a tile row's run holds: the arithmetic of the weight gradient's epilogue by itself, so that it can be
// checked on the host over widths and counts that no test allocates.  constexpr functions serve device and host alike.
#pragma once

namespace samo {
namespace runs {

constexpr unsigned kNone = ~0u;              // the position of an entry that is not there

// First position in the tile of row `row` of a tile (or part of one) that starts at row first_row, column col0.  The positions of a layer
// fit 31 bits.  It is for the layer's own rows: (first_row + row) * in passes 2^32 behind the last of a wide one.
constexpr unsigned row_key(int first_row, int row, int in, int col0)
{
    return (unsigned)(first_row + row) * (unsigned)in + (unsigned)col0;
}

// The same of row pair + half for the entries of a pair of rows, pair even.  rows: how many of the tile's rows from first_row on the layer has, not
// positive if none; it is even, as a layer's sides are multiples of 8.  A pair behind them has no entries, only kNone, and is given the
// layer's last pair of rows: whatever its key, kNone is a column of no tile (taken as it is, the key of row 255 of the last tile behind
// 8 x 2^24 is 2^32 - 256, and kNone would be its column 255).
constexpr unsigned pair_key(int first_row, int pair, int half, int rows, int in, int col0)
{
    return (unsigned)half * (unsigned)in + row_key(first_row, pair < rows ? pair : rows - 2, in, col0);
}

// Column in the tile of an entry at position pos; not below the tile's columns if the entry is not in the row's run.
constexpr unsigned column_of(unsigned pos, unsigned key) { return pos - key; }

}  // namespace runs
}  // namespace samo
