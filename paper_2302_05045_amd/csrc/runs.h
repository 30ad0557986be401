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

// How many entries idx has: a buffer may be longer (an index rebuilt with fewer elements kept in the place of another), and what is behind
// the ones seg_ptr counts is no index.  counted: the last value of seg_ptr.
constexpr int entries_of(int nnz, int counted) { return counted < nnz ? counted : nnz; }

// The entries between which a row's run begins: the first one whose position is not below the row's key is at lo at least, at hi at most.
struct Range {
    int lo, hi;
};

// A look reads kLook entries at once.  The first one is put where the run begins if the segment's entries are spread evenly over it; offset:
// the key's place in the segment.  It may reach beyond the range, never beyond the index (entries >= kLook).
constexpr int kLook = 32;
constexpr int first_look(Range r, int offset, int entries)
{
    const int at = r.lo + (((r.hi - r.lo) * offset) >> 10) - kLook / 2, from = at > r.lo ? at : r.lo;
    return from < entries - kLook ? from : entries - kLook;
}

// The second one beside the first, which began at `seen`, on the side that it points to.
constexpr int second_look(Range r, int seen, int entries)
{
    const int beside = r.lo == seen + kLook ? r.lo : r.hi - kLook, from = beside > 0 ? beside : 0;
    return from < entries - kLook ? from : entries - kLook;
}

// What is left of a range after a look at `at` that found `below` entries below the key.
constexpr Range after_look(Range r, int at, int below)
{
    const int first = at + below, lo = below > 0 && first > r.lo ? first : r.lo, hi = below < kLook && first < r.hi ? first : r.hi;
    return {lo, hi > lo ? hi : lo};
}

// The entry in the middle of a range: entries go up to 2^31, their sum does not fit.
constexpr int middle(Range r) { return r.lo + ((r.hi - r.lo) >> 1); }

// Column in the tile of an entry at position pos; not below the tile's columns if the entry is not in the row's run.
constexpr unsigned column_of(unsigned pos, unsigned key) { return pos - key; }

}  // namespace runs
}  // namespace samo
