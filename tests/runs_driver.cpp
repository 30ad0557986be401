// Host checks of the weight gradient's run arithmetic (csrc/runs.h), over sides that no GPU test allocates.
#include <algorithm>
#include <cstdio>
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
        const int rows = (int)std::min<long>(tile_rows, out - part0);
        for (int row = 0; row < tile_rows; ++row) {
            const unsigned key = runs::pair_key((int)part0, row & ~1, row & 1, rows, (int)in, col0);
            expect(runs::column_of(runs::kNone, key) >= (unsigned)cols, "no entry", out, in, part0 + row, col0);
            if (part0 + row >= out) continue;
            const long first = (part0 + row) * in + col0;
            for (long p : {first - 1, first, first + cols - 1, first + cols, n - 1, 0l})
                if (p >= first - 1 && p < n && p >= 0)
                    expect((runs::column_of((unsigned)p, key) < (unsigned)cols) == (p >= first && p < first + cols), "entry", out, in, part0 + row, p);
        }
    }
}

}  // namespace

int main()
{
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
