// Which entries of idx a tile row's run holds: the arithmetic of the weight gradient's epilogue by itself, so that it can be
// checked on the host over widths and counts that no test allocates.  constexpr functions serve device and host alike.
#pragma once

namespace samo {
namespace runs {

// First position in the tile of row `row` of a tile (or part of one) that starts at row first_row, column col0.  The positions of a layer
// fit 31 bits, those of the rows of its last tile behind it 32: 256 rows of 2^24, or less than twice the layer's.
constexpr unsigned row_key(int first_row, int row, int in, int col0)
{
    return (unsigned)(first_row + row) * (unsigned)in + (unsigned)col0;
}

// The position of an entry that is not there, in a tile column: left of the first row's first position, so that it is the furthest from
// every row, those behind the layer's last too, whose entries are all of this kind (2^32 - 1 in its place would be column 255 of
// row 255 in the last tile of an 8 x 2^24 layer).
constexpr unsigned no_position(int col0) { return (unsigned)col0 - 1u; }

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

// Where both looks missed (rows of very different density in one segment): eight entries that part what is left in nine, one to each lane.
// Entries go up to 2^31, so no two of them are added.
constexpr int kProbes = 8;
constexpr int probe(Range r, int j) { return r.lo + (int)((unsigned)(j + 1) * (unsigned)(r.hi - r.lo) / (kProbes + 1)); }
// What is left when `below` of them are below the key.
constexpr Range after_probes(Range r, int below)
{
    return {below > 0 ? probe(r, below - 1) + 1 : r.lo, below < kProbes ? probe(r, below) : r.hi};
}

// Column in the tile of an entry at position pos; not below the tile's columns if the entry is not in the row's run.
constexpr unsigned column_of(unsigned pos, unsigned key) { return pos - key; }

}  // namespace runs
}  // namespace samo
