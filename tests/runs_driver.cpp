// Host checks of the weight gradient's run arithmetic (csrc/runs.h), over sides that no GPU test allocates.
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

#include "runs.h"

namespace runs = samo::runs;

namespace {

long failures = 0;

void expect(bool ok, const char *what, long a, long b, long c, long d)
{
    if (ok) return;
    if (++failures <= 20) std::printf("FAILED %s: %ld %ld %ld %ld\n", what, a, b, c, d);
}

// Every row of a part of the last tile row, the ones behind the layer among them, in the first and the last two tile columns: the run takes the
// row's own positions, no other row's, and nothing that is not an entry.
void rows_of_tiles(long out, long in, long part0, int tile_rows, int tile_cols)
{
    const long tiles = (in + tile_cols - 1) / tile_cols;
    const long n = out * in;
    std::vector<long> at;
    for (long t : {0l, 1l, tiles - 2, tiles - 1})
        if (t >= 0 && t < tiles && std::find(at.begin(), at.end(), t) == at.end()) at.push_back(t);
    for (long t : at) {
        const int col0 = (int)(t * tile_cols), cols = (int)std::min<long>(tile_cols, in - col0);
        for (int row = 0; row < tile_rows; ++row) {
            const unsigned key = runs::row_key((int)part0, row, (int)in, col0);
            expect(runs::column_of(runs::no_position(col0), key) >= (unsigned)cols, "no entry", out, in, part0 + row, col0);
            if (part0 + row >= out) continue;
            const long first = (part0 + row) * in + col0;
            for (long p : {first - 1, first, first + cols - 1, first + cols, n - 1, 0l})
                if (p >= first - 1 && p < n && p >= 0)
                    expect((runs::column_of((unsigned)p, key) < (unsigned)cols) == (p >= first && p < first + cols), "entry", out, in, part0 + row, p);
        }
    }
}

// A layer's index as the epilogue reads it: idx of nnz entries, of which seg_ptr counts fewer where the buffer is that of an older, longer index.
struct Layer {
    int out, in, nnz;
    std::vector<int> idx, seg_ptr;
};

Layer layer_of(int out, int in, const std::vector<char> &mask, const std::vector<int> &tail)
{
    Layer l = {out, in, 0, {}, {0}};
    for (int p = 0; p < out * in; ++p) {
        if (mask[p]) l.idx.push_back(p);
        if (p % 1024 == 1023 || p + 1 == out * in) l.seg_ptr.push_back((int)l.idx.size());
    }
    l.idx.insert(l.idx.end(), tail.begin(), tail.end());
    l.nnz = (int)l.idx.size();
    return l;
}

// Where the run of a row begins that has that key, as the kernel looks for it.
int begin_of(const Layer &l, int entries, int key)
{
    runs::Range r = {l.seg_ptr[key / 1024], l.seg_ptr[key / 1024 + 1]};
    auto look = [&](int at) {
        int below = 0;
        for (int e = 0; e < runs::kLook; ++e) below += l.idx.at(at + e) < key;
        r = runs::after_look(r, at, below);
    };
    if (r.lo < r.hi && entries >= runs::kLook) {
        const int seen = runs::first_look(r, key & 1023, entries);
        look(seen);
        if (r.lo < r.hi) look(runs::second_look(r, seen, entries));
    }
    for (int steps = 0; r.lo < r.hi; ++steps) {
        expect(steps < 4, "steps", steps, r.lo, r.hi, key);
        int below = 0;
        for (int j = 0; j < runs::kProbes; ++j) below += l.idx.at(runs::probe(r, j)) < key;
        r = runs::after_probes(r, below);
    }
    return r.lo;
}

// Every row of every tile against the index itself: all its entries, in their places, and none of the tail behind the index.
void runs_of_layer(const Layer &l, int tile_cols, const char *what)
{
    const int entries = runs::entries_of(l.nnz, l.seg_ptr.back()), count = l.seg_ptr.back();
    for (int row = 0; row < l.out; ++row)
        for (int col0 = 0; col0 < l.in; col0 += tile_cols) {
            const int cols = std::min(tile_cols, l.in - col0), key = (int)runs::row_key(0, row, l.in, col0);
            const int first = (int)(std::lower_bound(l.idx.begin(), l.idx.begin() + count, key) - l.idx.begin());
            const int last = (int)(std::lower_bound(l.idx.begin(), l.idx.begin() + count, key + cols) - l.idx.begin());
            int k = begin_of(l, entries, key);
            expect(k == first, what, row, col0, k, first);
            while (k < entries && runs::column_of((unsigned)l.idx[k], (unsigned)key) < (unsigned)cols) ++k;
            expect(k == last, what, row, col0, k, last);
        }
}

void runs_of_masks()
{
    std::mt19937 rng(11);
    auto uniform = [&] { return std::uniform_real_distribution<double>(0, 1)(rng); };
    const int sides[][2] = {{8, 8}, {16, 136}, {64, 520}, {40, 1032}, {520, 64}, {24, 2560}};
    for (auto &side : sides)
        for (int kind = 0; kind < 8; ++kind) {
            const int out = side[0], in = side[1], n = out * in;
            const double keep[] = {0.0, 0.002, 0.05, 0.1, 0.5, 1.0, 0.1, 0.1};
            std::vector<char> mask(n);
            for (int p = 0; p < n; ++p) {
                double k = keep[kind];
                if (kind == 6) k = p / in % 10 == 3 ? 0.6 : 0.05;                  // rows of very different density
                if (kind == 7) k = p % 1024 >= 824 ? 1.0 : 0.0;                    // a segment's last elements alone
                mask[p] = uniform() < k;
            }
            std::vector<int> tail;                                                // the end of an older index
            for (int p = n - n / 5; p < n; ++p)
                if (uniform() < 0.5) tail.push_back(p);
            for (int cols : {128, 160, 256}) {
                runs_of_layer(layer_of(out, in, mask, {}), cols, "run");
                runs_of_layer(layer_of(out, in, mask, tail), cols, "run with a tail behind the index");
                std::vector<int> zeros(50, 0);
                runs_of_layer(layer_of(out, in, mask, zeros), cols, "run with zeros behind the index");
            }
        }
}

// The probes of what two looks left, at the ends of the range of entries: in order, never further from the beginning.
void probes_of_ranges()
{
    const int top = 2147483647;
    for (int lo : {0, 1, 1 << 30, (1 << 30) + 1, top - 1024, top - 9, top - 1})
        for (int length = 1; length <= 1024 && length <= top - lo; ++length) {
            const runs::Range r = {lo, lo + length};
            for (int j = 0; j < runs::kProbes; ++j) {
                const int k = runs::probe(r, j);
                expect(k >= lo && k < r.hi && (j == 0 || k >= runs::probe(r, j - 1)), "probe", lo, length, j, k);
            }
            for (int at = 0; at <= length; ++at) {
                int below = 0;
                for (int j = 0; j < runs::kProbes; ++j) below += runs::probe(r, j) - lo < at;
                const runs::Range is = runs::after_probes(r, below);
                expect(is.lo - lo <= at && at <= is.hi - lo && is.hi - is.lo < length, "left", lo, length, at, is.hi - is.lo);
            }
            for (int below = 0; below <= runs::kProbes; ++below) {                // whatever idx holds, the search ends
                const runs::Range is = runs::after_probes(r, below);
                expect(is.lo >= r.lo && is.hi <= r.hi && is.hi - is.lo < length, "shorter", lo, length, below, is.hi - is.lo);
            }
        }
}

}  // namespace

int main()
{
    runs_of_masks();
    probes_of_ranges();
    const long most = 2147483647, side = 1 << 24;
    for (int rows : {128, 256})
        for (int cols : {128, 160, 192, 256})
            for (long out : {8l, 16l, 64l, 120l, 127l / 8 * 8, 128l, 136l, 248l, 256l, 264l, 512l, 1000l, 1l << 20, 1l << 24})
                for (long in : {side, side - 8, side / 2, side / 2 + 8, most / out / 8 * 8, most / out / 8 * 8 - 8, 8l, 136l, 520l}) {
                    if (in > side || out * in > most) continue;
                    for (int part : {16, 32}) {                                // rows of a wave
                        for (long at = (out - 1) / rows * rows, end = at + rows; at < end; at += part) rows_of_tiles(out, in, at, part, cols);
                        for (long at = (in - 1) / rows * rows, end = at + rows; at < end; at += part) rows_of_tiles(in, out, at, part, cols);
                    }
                }
    std::printf("%ld failures\n", failures);
    return failures ? 1 : 0;
}
