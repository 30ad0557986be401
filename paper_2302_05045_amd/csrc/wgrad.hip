// Weight gradient of a fully connected layer written straight into the compressed gradient
// (Section III-C compresses each layer's dense fp16 gradient as soon as the backward pass has
// produced it; Section VI-C, on the compute overhead of that compression, names fusing that
// compression into the backward kernels as the way to remove it).  dW = dY^T X is a dense
// contraction over the tokens: fp16 MFMA with fp32 accumulation, operands staged through
// LDS; the epilogue rounds each accumulator once to fp16 — the value the dense gradient tensor
// would have held — and stores only the entries the layer's index keeps.  The dense gradient is
// never written to or read back from HBM.
//
// How the operands travel.  They arrive tokens-outer (dY is tokens x out, X is tokens x in) and go
// global -> LDS without passing registers (global_load_lds_dwordx4: each lane names 16 bytes of
// global memory, the wave's 1 KiB lands contiguously in LDS at a base held in M0), in the layout
// they have in memory — per token, a run of features.  An MFMA lane wants 8 tokens of one feature;
// the transposing LDS read ds_read_b64_tr_b16 forms that: within each group of 16 lanes, lanes
// 4r .. 4r+3 name the 16 features of token r (r = 0..3), and lane i receives feature i of those four
// tokens.  Which tokens a lane gets does not matter as long as both operands agree.  No transposes on
// the vector ALU and no registers for bytes in flight: a ring of four stages, three on their way
// while the fourth is multiplied.  The compiler cannot know which LDS reads alias a copy in flight
// and would wait for all of them before every read, so the copies are issued from inline assembly
// and the kernels count their outstanding copies themselves: every stage is exactly 4 copies per
// wave, the partial last stage included (rows past the last token are copied from a row of zeros).
//
// Tile shapes, all 8 waves with two waves per SIMD, in two groups of four (waves 0-3, 4-7: one
// of each group per SIMD):
//   256 x 256, 32 tokens per stage, 64 (out) x 128 (in) per wave, 128 accumulators;
//   256 rows x 128, 160 or 192 columns for calls that large tiles would not fill a round with;
//   128 x 128 for smaller calls, and for what is left of a call after whole rounds of large tiles where
//   that is at most half a round: each group covers the whole tile with 64 x 64 per wave (64
//   accumulators) and multiplies half of the tokens of every 64-token stage; group 1 hands its sums to
//   group 0 through LDS at the end;
//   128 x 128 by four waves, four workgroups to a compute unit, for short calls of more tiles than compute units
//   (wgrad_resident_kernel: a kernel of its own; what is said here of rings and groups is of the others).
// Calls of few tiles may have their tokens split over several workgroups per tile (plan_split).
// Short calls go through the stages with all waves in step (loop_apart).
//
// What bounds the large tile: power, and the overlap of its parts.  Per 32-token stage of a
// 256 x 256 tile (all compute units, ordinary fp16 values), in cycles: the matrix instructions
// alone 1054, the copies alone 760, the LDS reads alone 515 — but copies and multiplications
// issued by all waves in step take 2240 (1760 interleaved), because a wave whose copies queue up
// issues no matrix instructions and its partner on the SIMD queues up at the same moment.  So the two
// groups run half a stage apart: while one multiplies, the other reads its fragments and issues its
// copies, and they change places at a barrier: 1230 cycles.  From registers alone the chip sustains
// 1655 TFLOP/s (1.70 GHz) with the 32x32x16 instruction and 1930 (1.97 GHz) with 16x16x32, which
// touches half as many accumulators per flop: the clock gives way under the matrix units' power.
// 16x16x32, and an order in which consecutive instructions share an operand (1.5 % over row order).
// A 4096 x 4096 layer, before (32x32x16, all waves in step) and after: 8192 tokens 0.273 -> 0.207 ms
// (1007 -> 1329 TFLOP/s), 2048 tokens 0.083 -> 0.066 ms.  The 128 x 128 tile on a 1024 x 4096 layer: 8192
// tokens 0.087 -> 0.072 ms, 2048 tokens 0.0279 -> 0.0248.
#include <atomic>
#include <cstdlib>
#include <type_traits>

#include "common.h"
#include "runs.h"

namespace samo {
namespace {

#define LDS_AS __attribute__((address_space(3)))
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));

constexpr int kWgThreads = 512;
constexpr int kRowPitch = 1024 + 32;                 // an LDS row is one copy instruction's 1 KiB; with the pad eight consecutive
                                                     // rows, 32 bytes of each, cover the 64 banks once
constexpr int kStageRows = 32;
constexpr int kStageBytes = kStageRows * kRowPitch;  // 33792
constexpr int kStages = 4;
constexpr int kLdsBytes = kStages * kStageBytes;     // 135168: one workgroup per CU
constexpr int kBigTile = 256, kSmallTile = 128;
constexpr int kGroupDepth = 4;                       // tile rows of a group of tiles that share operand panels
// Tokens of one operand in an LDS row, and in a stage (16 rows of each operand).
constexpr int row_tokens(int tile) { return 512 / tile; }
constexpr int stage_tokens(int tile) { return 16 * row_tokens(tile); }       // 32, 64

// What a workgroup knows of the layer its tile belongs to.
struct WgradArgs {
    const _Float16 *dy;      // tokens x out
    const _Float16 *x;       // tokens x in
    int64_t tokens;
    int out, in;
    const int32_t *idx;
    const int32_t *seg_ptr;
    int64_t nnz;
    void *gc;                // fp32 or fp16, by the kernel's OUT
    float inv_scale;
    int accumulate;
};

// A launch: the 256 x 256 tiles of up to kWgradMaxJobs layers in one list, layer after layer
// (layer j owns tiles first_tile[j] .. first_tile[j+1] - 1, tiles_out[j] x tiles_in[j] of them);
// the launch's workgroups take tiles first .. first + tiles - 1 of that list, or, with quadrants
// set, four workgroups take the 128 x 128 quarters of each.
struct WgradBatch {
    WgradJob job[kWgradMaxJobs];
    int tiles_out[kWgradMaxJobs], tiles_in[kWgradMaxJobs];
    uint32_t per_group[kWgradMaxJobs];       // 2^32 / (tile rows of a group * tiles_in), rounded up
    int first_tile[kWgradMaxJobs + 1];       // 32 bits: a layer of less than 2^31 elements, sides up to 2^24, has less than 2^18 tiles of 128 x 128
                                             // (131072 of 8 x 2^24, 246000 of 136 x 15.7 M), a call less than 2^21; tile_origin's reciprocal takes up to 2^32
    int jobs;
    float inv_scale;
    int accumulate;
    int quadrants;
    int first, tiles;
    int tile_cols;                           // columns of a tile that is not quartered: 256, or 128, 160 or 192; 128 of the resident shape
    // splits > 1: that many workgroups share a tile, each multiplies split_tokens[j] tokens and leaves its fp32
    // sums at the kept positions in partial[j] + split * partial_stride[j]; wgrad_sum_kernel adds them up.
    int splits;
    int64_t split_tokens[kWgradMaxJobs];
    float *partial[kWgradMaxJobs];
    int64_t partial_stride[kWgradMaxJobs];
};
constexpr int kOutPartial = 3;
constexpr int kResidentShape = 512;         // SAMO_KNOB_WGRAD_TILE: 128 x 128 tiles, four workgroups to a compute unit
constexpr int kMaxSplits = 64;              // what SAMO_KNOB_WGRAD_SPLIT may ask for; the rule takes up to 16

__device__ __attribute__((aligned(16))) const unsigned char wgrad_zero_row[16] = {0};

// One copy instruction: the wave's 64 x 16 bytes from the lanes' global addresses to LDS at
// lds_byte_addr + 16 * lane.  It writes M0, a register the compiler reserves and does not let an
// asm statement declare as clobbered; nothing else in these kernels makes the compiler use M0 (no
// register arrays indexed at run time, no other LDS-direct or GWS operation).
__device__ __forceinline__ void dma16(const void *g, unsigned lds_byte_addr)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(lds_byte_addr) : "memory");
}

// The same with the global addresses as a scalar base plus a 32-bit offset per lane.  A scalar
// register that a vector instruction has written (the compiler may have parked the base in one) must
// not be read by a memory instruction for five cycles: the wait states in front cover that.
__device__ __forceinline__ void dma16_from(const void *base, unsigned lane_offset, unsigned lds_byte_addr)
{
    asm volatile("s_nop 3\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_offset), "s"(base), "s"(lds_byte_addr)
                 : "memory");
}

// 8 tokens of one feature for an MFMA lane: two transposing reads of one token of four LDS rows each,
// the rows' tokens `step` bytes apart.
__device__ __forceinline__ half8 read_fragment(const unsigned char *p, int step)
{
    const short4v a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS short4v *)(LDS_AS unsigned char *)p);
    const short4v b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS short4v *)(LDS_AS unsigned char *)(p + step));
    const short8v q = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    return __builtin_bit_cast(half8, q);
}

// Workgroups are dealt round-robin to the 8 XCDs: each XCD gets a contiguous run of tiles so
// that the tiles sharing operand panels, and neighbouring runs of idx, meet in one L2.  Within
// the run, tiles go down groups of 4 tile rows before they go across: the 32 tiles an XCD works on
// at a time then share about 4 + 8 operand panels rather than 1 + 32.
// Returns false for a workgroup with nothing to do: the surplus of the last round, or a quarter
// that lies outside the matrix.
// JOB_FIRST: the job's descriptor is requested with the launch's fields.  The list's tiles have TILE_ROWS rows.
template <bool JOB_FIRST, int TILE_ROWS = kBigTile>
__device__ __forceinline__ bool tile_origin(const WgradBatch &B, WgradArgs &A, int &row0, int &col0)
{
    // The workgroup's first copies wait for this function, and what it reads comes from the kernel arguments by way of
    // cold caches: a single job's descriptor is read at fixed places, and everything at once (left alone, the compiler loads each
    // value in front of its use, one trip more: the kernel of 1003 tokens, 4096 x 1024, 15.8 -> 15.4 us, 200 tokens, 2560 x 7680,
    // 27.8 -> 27.0; FC1 of the 2.7B model 101.0 -> 100.4).  Launches of few workgroups (kFewBlocks) take the descriptor after the
    // launch's fields: 512 x 512, 20 / 100 / 300 tokens, left alone, everything at once, so: 6.23, 7.01, 8.97 us; 6.49, 7.26, 9.20;
    // 6.10, 6.88, 8.86.  Only a list of several jobs is searched.
    const int quadrants = B.quadrants, tiles = B.tiles, splits = B.splits, jobs = B.jobs, first_listed = B.first, tile_cols = B.tile_cols;
    const float inv_scale = B.inv_scale;
    const int accumulate = B.accumulate;
    WgradJob J = B.job[0];
    int j = 0, first = 0, tiles_out = B.tiles_out[0], tiles_in = B.tiles_in[0];
    uint32_t per_group = B.per_group[0];
    if (JOB_FIRST)
        asm volatile("" ::"s"(quadrants), "s"(tiles), "s"(splits), "s"(jobs), "s"(first_listed), "s"(tile_cols), "s"(inv_scale), "s"(accumulate),
                     "s"(J.dy), "s"(J.x), "s"(J.tokens), "s"(J.out), "s"(J.in), "s"(J.idx), "s"(J.seg_ptr), "s"(J.nnz), "s"(J.gc), "s"(tiles_out),
                     "s"(tiles_in), "s"(per_group));
    else
        asm volatile("" ::"s"(quadrants), "s"(tiles), "s"(splits), "s"(jobs), "s"(first_listed), "s"(tile_cols), "s"(inv_scale), "s"(accumulate),
                     "s"(tiles_out), "s"(tiles_in), "s"(per_group));
    const int shares = quadrants ? tiles * 4 : tiles;            // workgroups of one split
    const int blocks = shares * splits;
    const int per_xcd = (blocks + 7) / 8;
    int local = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (local >= blocks) return false;
    const int split = splits > 1 ? local / shares : 0;           // the tiles of one split stay together
    local -= split * shares;
    const int listed = first_listed + (quadrants ? local >> 2 : local);
    if (jobs > 1) {
        while (j + 1 < jobs && listed >= B.first_tile[j + 1]) ++j;
        J = B.job[j];
        first = B.first_tile[j]; tiles_out = B.tiles_out[j]; tiles_in = B.tiles_in[j];
        per_group = B.per_group[j];
    }
    A.dy = J.dy; A.x = J.x; A.tokens = J.tokens; A.out = J.out; A.in = J.in;
    A.idx = J.idx; A.seg_ptr = J.seg_ptr; A.nnz = J.nnz; A.gc = J.gc;
    A.inv_scale = inv_scale; A.accumulate = accumulate;
    if (splits > 1) {
        const int64_t begin = split * B.split_tokens[j], left = J.tokens - begin;
        A.tokens = left < B.split_tokens[j] ? (left > 0 ? left : 0) : B.split_tokens[j];
        if (left > 0) {
            A.dy += begin * J.out;
            A.x += begin * J.in;
        }
        A.gc = B.partial[j] + split * B.partial_stride[j];
    }
    const int tile = listed - first;
    // tile / (kGroupDepth * tiles_in) by the reciprocal the host prepared (2^32 over it, rounded up: one too many at most)
    int group = (int)(((uint64_t)(uint32_t)tile * per_group) >> 32);
    if (group * kGroupDepth * tiles_in > tile) --group;
    const int in_group = tile - group * kGroupDepth * tiles_in;
    const int group_rows = tiles_out - group * kGroupDepth < kGroupDepth ? tiles_out - group * kGroupDepth : kGroupDepth;
    const int across = group_rows == kGroupDepth ? in_group / kGroupDepth : in_group / group_rows;
    row0 = (group * kGroupDepth + in_group - across * group_rows) * TILE_ROWS;   // first row of dW (feature of dY)
    col0 = across * tile_cols;                             // first column of dW (feature of X)
    if (quadrants) {
        row0 += (local & 1) * kSmallTile;
        col0 += ((local >> 1) & 1) * kSmallTile;
    }
    return row0 < A.out && col0 < A.in;
}

// Epilogue of one wave over ROWS rows of a tile held as an image in LDS (fp16; fp32 sums for kOutPartial).  The kept entries
// of a row in the tile are a run of idx: from its first entry at or after the row's first column to the last one before
// the tile's end.  Each half-wave takes every other row, all of them at once, 32 entries of every row a step:
// idx is read and the compressed gradient written coalesced, the values are picked from the image.
//
// Where a run begins is searched in steps with the tile's other work between them.  open() reads the segment's range from seg_ptr;
// look() reads 32 entries around the place where interpolation inside the segment puts the beginning; settle() decides.
// Eight lanes, 16 bytes each, look for one row together, so that an instruction reads eight pieces of 128 bytes, and the
// entries below the row's first column are counted across them.  (What it replaces: a lane by itself read 32 entries for a bound
// of its own, two bounds to a row, 64 places with every instruction: 3 to 5 us of a workgroup's time where all of a launch's
// search together.)  Kept elements spread evenly over a segment of k put the beginning within sqrt(k (1 - k / 1024)) / 2
// of the guess in the mean square (5 entries at 10 % kept, 8 at 50 %).  A look of 32 misses one row in hundreds, but one
// in most tiles at 20 % kept; a miss is a near one on masks without structure, so a second look beside the first comes before any
// other search (2376 x 7080, 20 % kept, 235 tokens 29.4 -> 27.9 us with it; left out where more than two groups of lanes missed, layers of no
// round width lose 3 to 7 % at 20 % kept, and gain nothing on rows of different density).  Rows of very different density that share a
// segment miss it too: the eight lanes part what is left in nine at a time (1000 x 520, 300 tokens, 20 % kept, a tenth of the rows ten times
// denser 12.1 us by bisection, 11.4 so; 7856 x 4632, 106 tokens 45.4 and 44.0).  Where a run ends shows when it is read.
// begin() requests the first AHEAD steps' idx, which travels while the image is written, and the values that are added to:
// with EARLY at once, else when their positions are known and the image is written (the 128 x 128 tile of the longer calls, 4096 x 1024, 1003
// tokens, accumulating 15.6 against 15.85 us; FC1 of the 2.7B model 102.9 against 102.1 the other way, four workgroups to a compute unit
// 3 to 5 %).  Before and now, 10 % kept unless said, us: 512 x 512, 100 tokens 6.75 and
// 6.17; 4096 x 1024, 1003 tokens 15.2 and 14.3; 4096 x 4096, 500 tokens 22.6 and 20.0; 7856 x 4632, 106 tokens, 20 % 50.3 and 43.7;
// FC1 of the 2.7B model 98.7 and 96.1 (20 %: 105.3 and 102.1).  Rows of very different density (a tenth of
// them ten times denser): 7856 x 4632 63.7 and 42.0, FC1 113 and 111, 512 x 520, 100 tokens 9.1 and 9.2.
typedef int Look __attribute__((ext_vector_type(4), aligned(4)));

// The sum over aligned groups of eight lanes, in every lane.
__device__ __forceinline__ int sum_of_eight(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);        // quad_perm 1 0 3 2
    v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);        // quad_perm 2 3 0 1
    return v + __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true); // row_half_mirror
}

template <int OUT, int ROWS, int AHEAD, bool EARLY = true>
struct RunPass {
    static constexpr int kLooks = ROWS / 8, kRows = ROWS / 2, kLook = runs::kLook;
    int first_row, rows, col0, cols;
    int counted, entries;                    // the last value of seg_ptr; the entries of idx that may be looked at, from look() on
    int lo[kLooks], hi[kLooks];              // row 8 i + lane / 8: the entries between which its run begins; from settle() on lo is where
    int seen_at[kLooks];                     // -1: nothing was looked at
    Look seen[kLooks];
    unsigned from[kRows];                    // row 2 it + half-wave: the step's first entry; unsigned: may pass 2^31 behind a layer's last
    unsigned pos[AHEAD][kRows];
    _Float16 old[AHEAD][kRows];

    __device__ __forceinline__ unsigned key(const WgradArgs &A, int row) const { return runs::row_key(first_row, row, A.in, col0); }
    __device__ __forceinline__ int look_row(int i) const { return 8 * i + (int)((threadIdx.x & 63) >> 3); }

    __device__ __forceinline__ void open(const WgradArgs &A, int row0, int column0, int tile_cols)
    {
        first_row = row0;
        col0 = column0;
        rows = A.out - row0 < ROWS ? A.out - row0 : ROWS;            // not positive: none
        cols = A.in - col0 < tile_cols ? A.in - col0 : tile_cols;
        // by a scalar load without a branch, which travels with the first copies (await): a vector load of a uniform value, and a load behind a
        // branch, are waited for at once (7856 x 4632, 106 tokens, 20 % kept 28.9 -> 29.7 us)
        const int32_t *last = A.idx ? A.seg_ptr + ((unsigned)A.out * (unsigned)A.in + (kSeg - 1)) / kSeg : reinterpret_cast<const int32_t *>(wgrad_zero_row);
        counted = *(const __attribute__((address_space(4))) int32_t *)last;
#pragma unroll
        for (int i = 0; i < kLooks; ++i) {
            lo[i] = hi[i] = (int)A.nnz;                              // no such row: an empty run
            if (look_row(i) >= rows) continue;
            const int p = (int)key(A, look_row(i));
            lo[i] = hi[i] = p;                                       // nothing pruned: position = entry
            if (A.idx) {
                lo[i] = A.seg_ptr[p / kSeg];
                hi[i] = A.seg_ptr[p / kSeg + 1];
            }
        }
    }
    // Behind the first copies.  The compiler, which does not know of the waits in asm, has to see the scalar load used before the main loop:
    // it would wait for all of a stage's LDS reads at once otherwise, as those and a scalar load return in any order.
    __device__ __forceinline__ void await() const { asm volatile("" ::"s"(counted)); }
    __device__ __forceinline__ void look(const WgradArgs &A)
    {
        entries = A.idx ? runs::entries_of((int)A.nnz, counted) : (int)A.nnz;
#pragma unroll
        for (int i = 0; i < kLooks; ++i) {
            seen[i] = Look{0, 0, 0, 0};
            seen_at[i] = -1;
            if (hi[i] > lo[i] && entries >= kLook) {
                seen_at[i] = runs::first_look({lo[i], hi[i]}, (int)(key(A, look_row(i)) & (kSeg - 1)), entries);
                seen[i] = *reinterpret_cast<const Look *>(A.idx + seen_at[i] + 4 * (threadIdx.x & 7));
            }
        }
    }
    // What the look of a row's eight lanes leaves of the range, if there was one.  (Both ends are written whatever the case: stores to
    // either of two arrays keep them in memory.)
    __device__ __forceinline__ void narrow(const WgradArgs &A, int i, bool looked)
    {
        const int want = (int)key(A, look_row(i));
        int below = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) below += seen[i][e] < want ? 1 : 0;
        below = sum_of_eight(below);
        const runs::Range was = {lo[i], hi[i]}, is = runs::after_look(was, seen_at[i], below);
        lo[i] = looked ? is.lo : was.lo;
        hi[i] = looked ? is.hi : was.hi;
    }
    __device__ __forceinline__ void settle(const WgradArgs &A)
    {
#pragma unroll
        for (int i = 0; i < kLooks; ++i) narrow(A, i, seen_at[i] >= 0);
        bool left = false;
#pragma unroll
        for (int i = 0; i < kLooks; ++i) left |= lo[i] < hi[i];
        if (!__ballot(left)) return;
        // A miss on a mask without structure is a near one: the 32 entries beside the look, on the side it points to.
        left = false;
#pragma unroll
        for (int i = 0; i < kLooks; ++i) {
            if (lo[i] < hi[i] && entries >= kLook) {
                seen_at[i] = runs::second_look({lo[i], hi[i]}, seen_at[i], entries);
                seen[i] = *reinterpret_cast<const Look *>(A.idx + seen_at[i] + 4 * (threadIdx.x & 7));
            }
        }
#pragma unroll
        for (int i = 0; i < kLooks; ++i) {
            narrow(A, i, lo[i] < hi[i] && seen_at[i] >= 0);
            left |= lo[i] < hi[i];
        }
        while (__ballot(left)) {                                     // all the searches a step at a time
            int there[kLooks];
#pragma unroll
            for (int i = 0; i < kLooks; ++i) there[i] = lo[i] < hi[i] ? A.idx[runs::probe({lo[i], hi[i]}, threadIdx.x & 7)] : 0;
            left = false;
#pragma unroll
            for (int i = 0; i < kLooks; ++i) {
                const runs::Range was = {lo[i], hi[i]}, is = runs::after_probes(was, sum_of_eight(there[i] < (int)key(A, look_row(i)) ? 1 : 0));
                const bool open = was.lo < was.hi;
                lo[i] = open ? is.lo : was.lo;
                hi[i] = open ? is.hi : was.hi;
                left |= lo[i] < hi[i];
            }
        }
    }
    // A step's positions; with EARLY also the values that are added to.
    __device__ __forceinline__ void request(const WgradArgs &A)
    {
        const unsigned l32 = threadIdx.x & 31, end = (unsigned)entries;
#pragma unroll
        for (int a = 0; a < AHEAD; ++a)
#pragma unroll
            for (int it = 0; it < kRows; ++it) {
                const unsigned k = from[it] + a * 32 + l32;
                pos[a][it] = k < end ? (A.idx ? (unsigned)A.idx[k] : k) : runs::no_position(col0);
            }
        if (EARLY) request_old(A);
    }
    // The values that are added to.  Those of entries behind the run belong to other tiles, whose workgroups may be writing
    // them: they are read to have all of them on their way at once, and not used.
    __device__ __forceinline__ void request_old(const WgradArgs &A)
    {
        if (OUT != kOutF16 || !A.accumulate) return;
        if (!EARLY) asm volatile("" ::: "memory");                   // not before the image is written
        const unsigned l32 = threadIdx.x & 31, end = (unsigned)entries;
#pragma unroll
        for (int a = 0; a < AHEAD; ++a) {
            if (!EARLY && !wanted(A, a)) break;
#pragma unroll
            for (int it = 0; it < kRows; ++it) {
                const unsigned k = from[it] + a * 32 + l32;
                const bool there = EARLY ? k < end : column(A, a, it) < (unsigned)cols;
                old[a][it] = there ? reinterpret_cast<const _Float16 *>(A.gc)[k] : (_Float16)0.f;
            }
        }
    }
    // Column in the tile of the lane's entry of row 2 it + half-wave; not below cols: it isn't in the row's run.
    // (The pair's key in scalar registers: the halves' keys of all rows by themselves were kept in vector registers, of which there are no more.)
    __device__ __forceinline__ unsigned column(const WgradArgs &A, int a, int it) const
    {
        return runs::column_of(pos[a][it], ((threadIdx.x & 63) >> 5) * (unsigned)A.in + key(A, 2 * it));
    }
    // Whether any row of the wave has entries in step a of those requested (of the first, some row is taken to have).
    __device__ __forceinline__ bool wanted(const WgradArgs &A, int a) const
    {
        if (a == 0) return true;
        bool in = false;
#pragma unroll
        for (int it = 0; it < kRows; ++it) in |= column(A, a, it) < (unsigned)cols;
        return __ballot(in) != 0;
    }
    __device__ __forceinline__ void begin(const WgradArgs &A)
    {
        const int h = (threadIdx.x & 63) >> 5;
#pragma unroll
        for (int it = 0; it < kRows; ++it) from[it] = (unsigned)__shfl(lo[it / 4], 8 * ((2 * it & 7) + h), 64);
        request(A);
    }
    // The entries requested; returns, in lanes 31 and 63, whether a row's run may go on behind the last of them.
    // img: the image's row of the pass's first row.
    template <typename Pixel>
    __device__ __forceinline__ bool step(const WgradArgs &A, const Pixel *img, int pitch)
    {
        const int h = (threadIdx.x & 63) >> 5;
        bool on = false;
#pragma unroll
        for (int a = 0; a < AHEAD; ++a) {
            if (!wanted(A, a)) return false;
#pragma unroll
            for (int it = 0; it < kRows; ++it) {
                const unsigned at = column(A, a, it), k = from[it] + a * 32 + (threadIdx.x & 31);
                const bool in = at < (unsigned)cols;
                if (a == AHEAD - 1) on |= at < (unsigned)cols - 1;
                const Pixel v = img[(2 * it + h) * pitch + (in ? at : 0)];        // all rows' reads in flight together
                if (!in) continue;
                if (OUT == kOutPartial) reinterpret_cast<float *>(A.gc)[k] = (float)v;
                else if (OUT == kOutF32) reinterpret_cast<float *>(A.gc)[k] = (float)v * A.inv_scale;
                else reinterpret_cast<_Float16 *>(A.gc)[k] = A.accumulate ? (_Float16)(old[a][it] + v) : v;
            }
        }
        return on;
    }
    template <typename Pixel>
    __device__ __forceinline__ void finish(const WgradArgs &A, const Pixel *img, int pitch)
    {
        while (__ballot(step(A, img, pitch)) & 0x8000000080000000ull) {
#pragma unroll
            for (int it = 0; it < kRows; ++it) from[it] += 32 * AHEAD;
            request(A);
            if (!EARLY) request_old(A);
        }
    }
};

// The two passes of a wave over a tile whose sums are held in LDS half of the rows at a time.
template <typename Pass>
struct TwoPasses {
    Pass half[2];
    __device__ __forceinline__ void await() const { half[0].await(); half[1].await(); }
    __device__ __forceinline__ void look(const WgradArgs &A) { half[0].look(A); half[1].look(A); }
    __device__ __forceinline__ void settle(const WgradArgs &A) { half[0].settle(A); half[1].settle(A); }
};

// Waits until at most `younger` stages' copies of this wave are outstanding (and every LDS read has returned).
__device__ __forceinline__ void wait_copies(int64_t younger)
{
    if (younger >= 2) asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" ::: "memory");
    else if (younger == 1) asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}

// A bare workgroup barrier: what has to be complete before it is waited for explicitly.
__device__ __forceinline__ void meet()
{
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The main loop: acc += the wave's OB x IB blocks of 16 x 16 of a tile of COLS <= TILE columns.  A stage is 32
// LDS rows, row j < 16 row_tokens(TILE) consecutive tokens of X (room for TILE features each), row 16 + j
// the same tokens of dY.
// Waves 0-3 (group 0) copy X, waves 4-7 (group 1) dY.  x_at / y_at: byte offset, within a row, of the
// wave's first feature of the first of the two tokens it multiplies per row.  The epilogue's look
// and its outcome come with the last stages; the ring is free after the next __syncthreads.
//
// The groups' half stages, b(i) the barriers all eight waves meet at:
//   group 0:  b(0) fetch 0  b(1) multiply 0  b(2) fetch 1  b(3) multiply 1 ...
//   group 1:  b(0)          b(1) fetch 0     b(2) multiply 0  b(3) fetch 1 ...
// fetch s reads the stage's fragments into registers and issues the copies of stage s + 3 into the ring
// slot of stage s - 1: group 1, the later one, has finished reading that slot before b(2s).  Stage
// s + 1 is read from b(2s + 2) on, so every wave waits for its own copies of it before that barrier —
// group 0 at the end of multiply s, group 1 at the end of fetch s — when the copies of stages s + 2
// and s + 3 are the only younger ones.  The loads of run.open are older than every copy.  Those of
// run.look are requested when the last full stage is on its way: the wait for run.open's results
// is a wait for every copy in flight, once, where only one or two stages are; after it they can only make
// the waits of the last stages longer than needed, never shorter.
//
// Not APART, all waves take a stage together, one barrier each: fetch s and multiply s are one step, the copies of stage
// s + 3 go into the slot of stage s - 1, which every wave has finished reading before the barrier of step s.  That
// saves the half stage at either end and the second barrier, and is quicker where a call has few stages
// (loop_apart).  run.look comes first in the small tile, whose registers allow it, and travels under the whole
// loop; the large tile requests it where the other loop does.  Its wait for every copy in flight is
// made explicit and remembered.
template <int TILE, int COLS, bool APART, typename Run, int OB, int IB>
__device__ __forceinline__ void multiply_tile(const WgradArgs &A, int row0, int col0, int x_at, int y_at, unsigned char *lds,
                                                Run &run, f32x4 (&acc)[OB][IB])
{
    constexpr int kRowTokens = row_tokens(TILE), kTokens = stage_tokens(TILE), kTokenLanes = 64 / kRowTokens;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int group = wave >> 2;
    // Copy role: one instruction of a wave moves one row, kTokenLanes lanes per token.  Wave w owns rows 4w .. 4w+3.
    const int features = group ? A.out : A.in;
    const int f0 = group ? row0 : col0;
    const int64_t row_bytes = (int64_t)features * 2;
    const int f = lane % kTokenLanes * 8;
    const bool wanted = f0 + f < features && (COLS == TILE || group || f < COLS);   // else: the first feature again
    const unsigned f_bytes = (unsigned)(wanted ? f : 0) * 2;
    const int sub = lane / kTokenLanes;
    const unsigned lane_offset = (unsigned)sub * (unsigned)row_bytes + f_bytes;      // below 2^27: a row has at most 2^24 features
    const unsigned char *gbase = reinterpret_cast<const unsigned char *>(group ? A.dy : A.x) + (int64_t)f0 * 2;
    const unsigned lds_rows = (unsigned)(size_t)(LDS_AS unsigned char *)lds + (unsigned)(wave * 4) * kRowPitch;
    const int64_t stages = (A.tokens + kTokens - 1) / kTokens;
    const int64_t full = A.tokens / kTokens;                 // stages without rows past the last token
    const int first_token = (wave & 3) * 4 * kRowTokens;     // of the wave's rows in a stage
    auto issue_stage = [&](int64_t s) {
        const unsigned dst = lds_rows + (unsigned)(s % kStages) * kStageBytes;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t token = s * kTokens + first_token + kRowTokens * i + sub;
            dma16(token < A.tokens ? gbase + token * row_bytes + f_bytes : wgrad_zero_row, dst + i * kRowPitch);
        }
    };
#pragma unroll
    for (int bo = 0; bo < OB; ++bo)
#pragma unroll
        for (int bi = 0; bi < IB; ++bi)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[bo][bi][r] = 0.f;
    // 16 lanes read four rows, 16 features: the lane groups take rows 0-3, 4-7, 8-11, 12-15
    const int lane_read = (lane >> 2) * kRowPitch + (lane & 3) * 8;
    const int x_off = lane_read + x_at, y_off = lane_read + 16 * kRowPitch + y_at;

    for (int64_t s = 0; s < 3 && s < stages; ++s) issue_stage(s);
    run.await();
    unsigned slot = 0;                                       // LDS offset of the stage being read
    const unsigned char *gnext = gbase + (3 * kTokens + first_token) * row_bytes;    // the wave's rows three stages ahead
    auto multiply = [&](const half8 (&xa)[IB], const half8 (&yb)[OB]) {
#pragma unroll
        for (int q = 0; q < OB * IB; ++q) {
            const int bi = q / OB, bo = (bi & 1) ? OB - 1 - q % OB : q % OB;
            acc[bo][bi] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[bi], yb[bo], acc[bo][bi], 0, 0, 0);
        }
    };
    auto advance = [&]() {
        gnext += kTokens * row_bytes;
        slot = slot == (kStages - 1) * kStageBytes ? 0 : slot + kStageBytes;
    };
    if constexpr (!APART) {
        const int64_t look = TILE == kSmallTile || full <= 3 ? 0 : full - 3;
        int64_t arrived = 0;                                 // stages whose copies are known to be there
        for (int64_t s = 0; s < stages; ++s) {
            if (s == look) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                run.look(A);
                arrived = s + 3;
            }
            if (s < arrived) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            else wait_copies(stages - 1 - s);
            meet();
            const unsigned char *cur = lds + slot;
            const unsigned dst = lds_rows + (slot >= kStageBytes ? slot - kStageBytes : slot + 3 * kStageBytes);
            if (s + 3 < full) {
#pragma unroll
                for (int i = 0; i < 4; ++i) dma16_from(gnext + kRowTokens * i * row_bytes, lane_offset, dst + i * kRowPitch);
            } else if (s + 3 < stages) issue_stage(s + 3);
            half8 xa[IB], yb[OB];
#pragma unroll
            for (int bo = 0; bo < OB; ++bo) yb[bo] = read_fragment(cur + y_off + bo * 32, TILE * 2);
#pragma unroll
            for (int bi = 0; bi < IB; ++bi) xa[bi] = read_fragment(cur + x_off + bi * 32, TILE * 2);
            multiply(xa, yb);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            advance();
        }
        if (stages == 0) run.look(A);
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        run.settle(A);
        return;
    }
    wait_copies(stages - 1);
    meet();                                                  // b(0)
    if (group == 1) meet();                                  // half a stage behind from here on

    auto stage = [&](int64_t s, auto steady_loop) {
        constexpr bool kSteady = decltype(steady_loop)::value;      // stage s + 3 exists and is full
        const unsigned char *cur = lds + slot;
        const unsigned dst = lds_rows + (slot >= kStageBytes ? slot - kStageBytes : slot + 3 * kStageBytes);
        auto copy = [&](int i) {
            __builtin_amdgcn_sched_barrier(0);               // the copies stay spread between the LDS reads
            if (kSteady) dma16_from(gnext + kRowTokens * i * row_bytes, lane_offset, dst + i * kRowPitch);
            __builtin_amdgcn_sched_barrier(0);
        };
        half8 xa[IB], yb[OB];
#pragma unroll
        for (int bo = 0; bo < OB; ++bo) yb[bo] = read_fragment(cur + y_off + bo * 32, TILE * 2);
        copy(0);
#pragma unroll
        for (int bi = 0; bi < IB; ++bi) {
            xa[bi] = read_fragment(cur + x_off + bi * 32, TILE * 2);
            if (bi == IB / 3) copy(1);
            if (bi == 2 * IB / 3) copy(2);
        }
        copy(3);
        if (!kSteady && s + 3 < stages) issue_stage(s + 3);
        if (group == 0) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        else wait_copies(kSteady ? 2 : stages - 2 - s);
        __builtin_amdgcn_sched_barrier(0);
        meet();
        __builtin_amdgcn_s_setprio(1);                       // the multiplying wave first: the other one's reads fit in between
        __builtin_amdgcn_sched_barrier(0);
        multiply(xa, yb);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
        if (group == 0) wait_copies(kSteady ? 2 : stages - 2 - s);
        meet();
        advance();
    };
    int64_t s = 0;
    for (; s + 3 < full; ++s) stage(s, std::true_type{});
    run.look(A);
    for (; s < stages; ++s) stage(s, std::false_type{});
    if (group == 0) meet();
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    run.settle(A);
}

// 256 x (32 IB) tile, IB = 8 or fewer for calls of less than a round: 64 (out) x 16 IB (in) per wave, waves as 4 x 2;
// both groups multiply every token.
template <int OUT, int IB, bool APART>
__global__ void __launch_bounds__(kWgThreads, 2) wgrad_big_kernel(const WgradBatch B)
{
    constexpr int kTile = kBigTile, kCols = 32 * IB, kEpiPitch = kCols + 8;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    WgradArgs A;
    int row0, col0;
    if (!tile_origin<true>(B, A, row0, col0)) return;

    const int t = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int wo = wave & 3, wi = wave >> 2;
    f32x4 acc[4][IB];
    if constexpr (OUT == kOutPartial) {                      // fp32 sums: the ring holds half of the rows at a time
        constexpr int kHalf = kTile / 2, kSumPitch = kCols + 4, kRows = kHalf / 8;
        static_assert(kHalf * kSumPitch * 4 <= kLdsBytes, "half of the tile's sums fit in the stages");
        TwoPasses<RunPass<OUT, kRows, 2>> run;               // of each half wave w gathers rows 16 w ..
        for (int half = 0; half < 2; ++half) run.half[half].open(A, row0 + half * kHalf + wave * kRows, col0, kCols);
        multiply_tile<kTile, kCols, APART>(A, row0, col0, wi * (kCols / 2) * 2, wo * 64 * 2, lds, run, acc);
        float *sums = reinterpret_cast<float *>(lds);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            __syncthreads();
            run.half[half].begin(A);
            if (wo >> 1 == half) {
#pragma unroll
                for (int bo = 0; bo < 4; ++bo)
#pragma unroll
                    for (int bi = 0; bi < IB; ++bi) {
                        const int col = wi * (kCols / 2) + bi * 16 + (lane >> 4) * 4;
                        *reinterpret_cast<f32x4 *>(sums + ((wo & 1) * 64 + bo * 16 + (lane & 15)) * kSumPitch + col) = acc[bo][bi];
                    }
            }
            __syncthreads();
            run.half[half].finish(A, sums + wave * kRows * kSumPitch, kSumPitch);
        }
        return;
    }
    RunPass<OUT, kTile / 8, 2> run;                          // wave w gathers rows 32 w ..
    run.open(A, row0 + wave * 32, col0, kCols);
    multiply_tile<kTile, kCols, APART>(A, row0, col0, wi * (kCols / 2) * 2, wo * 64 * 2, lds, run, acc);
    __syncthreads();
    run.begin(A);

    // accumulator layout: lane l holds dW[.. + (l & 15)][.. + 4 * (l >> 4) + r], r = 0..3
    _Float16 *img = reinterpret_cast<_Float16 *>(lds);
    static_assert(kTile * kEpiPitch * 2 <= kLdsBytes, "the whole tile's image fits in the stages");
#pragma unroll
    for (int bo = 0; bo < 4; ++bo)
#pragma unroll
        for (int bi = 0; bi < IB; ++bi) {
            half4 h;
#pragma unroll
            for (int e = 0; e < 4; ++e) h[e] = (_Float16)acc[bo][bi][e];           // round to nearest even
            const int col = wi * (kCols / 2) + bi * 16 + (lane >> 4) * 4;
            *reinterpret_cast<half4 *>(img + (wo * 64 + bo * 16 + (lane & 15)) * kEpiPitch + col) = h;
        }
    __syncthreads();
    run.finish(A, img + wave * 32 * kEpiPitch, kEpiPitch);
}

// 128 x 128 tile: 64 x 64 per wave, the waves of a group as 2 x 2; group g multiplies tokens 2g and 2g + 1 of every row.
// FEW: for launches of fewer than kFewBlocks workgroups (768 x 768, 36 of them, 300 tokens: 9.22 us without and 8.93 with; 1024 x 1024, 64, 200
// tokens 8.30 and 8.32; 4096 x 1024, 256, 700 tokens 12.73 and 12.84).
constexpr unsigned kFewBlocks = 64;
template <int OUT, bool APART, bool FEW>
__global__ void __launch_bounds__(kWgThreads, 2) wgrad_small_kernel(const WgradBatch B)
{
    constexpr int kTile = kSmallTile, kEpiPitch = kTile + 8, kSumPitch = kTile + 4;
    static_assert(kTile * kSumPitch * 4 + kTile * kEpiPitch * 2 <= kLdsBytes, "group 1's sums and the image reuse the stages");
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    WgradArgs A;
    int row0, col0;
    if (!tile_origin<!FEW>(B, A, row0, col0)) return;

    const int t = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    RunPass<OUT, kTile / 8, 2, !APART> run;                  // wave w gathers rows 16 w ..
    run.open(A, row0 + wave * 16, col0, kTile);
    const int half = wave >> 2;
    const int wo = wave & 1, wi = (wave >> 1) & 1;
    f32x4 acc[4][4];
    const int tokens_at = half * 2 * kTile * 2;
    multiply_tile<kTile, kTile, APART>(A, row0, col0, tokens_at + wi * 64 * 2, tokens_at + wo * 64 * 2, lds, run, acc);
    __syncthreads();
    run.begin(A);

    // group 1's sums -> LDS as fp32; group 0 adds them to its own, rounds once to fp16 and writes
    // the image behind them
    float *sums = reinterpret_cast<float *>(lds);
    _Float16 *img = reinterpret_cast<_Float16 *>(lds + kTile * kSumPitch * 4);
    if (half == 1) {
#pragma unroll
        for (int bo = 0; bo < 4; ++bo)
#pragma unroll
            for (int bi = 0; bi < 4; ++bi) {
                const int col = wi * 64 + bi * 16 + (lane >> 4) * 4;
                *reinterpret_cast<f32x4 *>(sums + (wo * 64 + bo * 16 + (lane & 15)) * kSumPitch + col) = acc[bo][bi];
            }
    }
    __syncthreads();
    if (half == 0) {
#pragma unroll
        for (int bo = 0; bo < 4; ++bo)
#pragma unroll
            for (int bi = 0; bi < 4; ++bi) {
                const int col = wi * 64 + bi * 16 + (lane >> 4) * 4;
                f32x4 *at = reinterpret_cast<f32x4 *>(sums + (wo * 64 + bo * 16 + (lane & 15)) * kSumPitch + col);
                const f32x4 o = *at;
                if (OUT == kOutPartial) {
                    f32x4 sum;
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[e] = acc[bo][bi][e] + o[e];
                    *at = sum;
                    continue;
                }
                half4 h;
#pragma unroll
                for (int e = 0; e < 4; ++e) h[e] = (_Float16)(acc[bo][bi][e] + o[e]);   // round to nearest even
                *reinterpret_cast<half4 *>(img + (wo * 64 + bo * 16 + (lane & 15)) * kEpiPitch + col) = h;
            }
    }
    if (APART) run.request_old(A);
    __syncthreads();
    if constexpr (OUT == kOutPartial) run.finish(A, sums + wave * 16 * kSumPitch, kSumPitch);
    else run.finish(A, img + wave * 16 * kEpiPitch, kEpiPitch);
}

// 128 x 128 tile by a workgroup of four waves, of which a compute unit holds four (128 registers, 34 KB of LDS): 64 x 64 per wave,
// the waves as 2 x 2, a ring of two 32-token stages of 16 LDS rows (8 of X, 8 of dY).  For calls whose time is not the main loop but what
// is around it: with one workgroup to a compute unit the start of a tile (arguments, first copies), the search for its runs, the image and
// the gather are waited for one after the other, 7 us and more a round; here other tiles' steps run meanwhile.  Nothing in a workgroup
// overlaps anything else, which is why the code is plain: all waves take a stage together, its look comes after the loop.
// Rings of three and four stages (three and two workgroups to a unit) are slower (7856 x 4632, 106 tokens, 20 % kept 32.5 us and more
// against 29.3; one workgroup of 256 x 256: 43.5), and so are 128 x 256 tiles, two to a unit, by 0 to 15 % where this shape is the best.
// The copies set the pace of the loop, twice the bytes per flop of the large tile, so long calls are not for it (plan_tiles).
constexpr int kResidentThreads = 256, kResidentRows = 16, kResidentStage = kResidentRows * kRowPitch, kResidentPitch = kSmallTile + 8;
constexpr int kResidentLds = kSmallTile * kResidentPitch * 2;
static_assert(2 * kResidentStage <= kResidentLds, "the ring of two stages fits in the image's place");
static_assert(4 * (kResidentLds + 1024) <= 160 * 1024, "four workgroups to a compute unit");

// A pointer all lanes of a wave agree on, told to the compiler.
__device__ __forceinline__ const unsigned char *uniform(const unsigned char *p)
{
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    return reinterpret_cast<const unsigned char *>((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a) |
                                                   (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)) << 32);
}

template <int OUT>
__global__ void __launch_bounds__(kResidentThreads, 4) wgrad_resident_kernel(const WgradBatch B)
{
    constexpr int kTokens = 32, kRowTokens = row_tokens(kSmallTile);
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    WgradArgs A;
    int row0, col0;
    if (!tile_origin<true, kSmallTile>(B, A, row0, col0)) return;
    const int t = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int wo = wave & 1, wi = wave >> 1;

    // Copies: wave w owns rows 2w, 2w + 1 of either operand, a row holds four tokens: 4 row + lane / 16.
    const int64_t x_bytes = (int64_t)A.in * 2, y_bytes = (int64_t)A.out * 2;
    const int sub = lane >> 4, f = (lane & 15) * 8;
    const unsigned xf = (unsigned)(col0 + f < A.in ? f : 0) * 2, yf = (unsigned)(row0 + f < A.out ? f : 0) * 2;    // else: the first feature again
    const unsigned x_lane = (unsigned)sub * (unsigned)x_bytes + xf, y_lane = (unsigned)sub * (unsigned)y_bytes + yf;   // below 2^27
    const unsigned char *xbase = reinterpret_cast<const unsigned char *>(A.x) + (int64_t)col0 * 2;
    const unsigned char *ybase = reinterpret_cast<const unsigned char *>(A.dy) + (int64_t)row0 * 2;
    const int first_token = 2 * kRowTokens * wave;
    const unsigned x_rows = (unsigned)(size_t)(LDS_AS unsigned char *)lds + (unsigned)(wave * 2) * kRowPitch;
    const unsigned y_rows = x_rows + kResidentRows / 2 * kRowPitch;
    const int stages = (int)((A.tokens + kTokens - 1) / kTokens), full = (int)(A.tokens / kTokens);   // tokens fit 31 bits
    const unsigned char *xnext = xbase + first_token * x_bytes, *ynext = ybase + first_token * y_bytes;
    auto issue = [&](int s) {                                // stages in order, from 0
        const unsigned slot = (s & 1) * kResidentStage;
        if (s < full) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                dma16_from(uniform(xnext + kRowTokens * i * x_bytes), x_lane, x_rows + slot + i * kRowPitch);
                dma16_from(uniform(ynext + kRowTokens * i * y_bytes), y_lane, y_rows + slot + i * kRowPitch);
            }
            xnext += kTokens * x_bytes;
            ynext += kTokens * y_bytes;
            return;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int64_t token = (int64_t)s * kTokens + first_token + kRowTokens * i + sub;
            const bool there = token < A.tokens;
            dma16(there ? xbase + token * x_bytes + xf : wgrad_zero_row, x_rows + slot + i * kRowPitch);
            dma16(there ? ybase + token * y_bytes + yf : wgrad_zero_row, y_rows + slot + i * kRowPitch);
        }
    };
    // Wave w gathers rows 32 w .. 32 w + 31; in two parts where old values take registers too.
    constexpr int kParts = OUT == kOutF16 ? 2 : 1, kPartRows = kSmallTile / 4 / kParts;
    RunPass<OUT, kPartRows, 1> run[kParts];
#pragma unroll
    for (int i = 0; i < kParts; ++i) run[i].open(A, row0 + wave * 32 + i * kPartRows, col0, kSmallTile);
    if (stages > 0) issue(0);
#pragma unroll
    for (int i = 0; i < kParts; ++i) run[i].await();
    f32x4 acc[4][4];
#pragma unroll
    for (int bo = 0; bo < 4; ++bo)
#pragma unroll
        for (int bi = 0; bi < 4; ++bi)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[bo][bi][r] = 0.f;
    // 16 lanes read four rows, 16 features: the lane groups take rows 0-3 and 4-7, tokens 0 and 1, then 2 and 3 of each
    const int lane_read = ((lane >> 2) & 7) * kRowPitch + (lane >> 5) * 2 * kSmallTile * 2 + (lane & 3) * 8;
    const int x_off = lane_read + wi * 64 * 2, y_off = lane_read + kResidentRows / 2 * kRowPitch + wo * 64 * 2;
    for (int s = 0; s < stages; ++s) {
        // stage s is there, and every wave has read stage s - 1, whose place the next copies take
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        meet();
        if (s + 1 < stages) issue(s + 1);
        const unsigned char *cur = lds + (s & 1) * kResidentStage;
        half8 xa[4], yb[4];
#pragma unroll
        for (int bo = 0; bo < 4; ++bo) yb[bo] = read_fragment(cur + y_off + bo * 32, kSmallTile * 2);
#pragma unroll
        for (int bi = 0; bi < 4; ++bi) xa[bi] = read_fragment(cur + x_off + bi * 32, kSmallTile * 2);
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int bi = q / 4, bo = (bi & 1) ? 3 - q % 4 : q % 4;
            acc[bo][bi] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[bi], yb[bo], acc[bo][bi], 0, 0, 0);
        }
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kParts; ++i) run[i].look(A);
#pragma unroll
    for (int i = 0; i < kParts; ++i) run[i].settle(A);
    run[0].begin(A);
    _Float16 *img = reinterpret_cast<_Float16 *>(lds);
#pragma unroll
    for (int bo = 0; bo < 4; ++bo)
#pragma unroll
        for (int bi = 0; bi < 4; ++bi) {
            half4 h;
#pragma unroll
            for (int e = 0; e < 4; ++e) h[e] = (_Float16)acc[bo][bi][e];           // round to nearest even
            const int col = wi * 64 + bi * 16 + (lane >> 4) * 4;
            *reinterpret_cast<half4 *>(img + (wo * 64 + bo * 16 + (lane & 15)) * kResidentPitch + col) = h;
        }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kParts; ++i) {
        if (i + 1 < kParts) run[i + 1].begin(A);
        run[i].finish(A, img + (wave * 32 + i * kPartRows) * kResidentPitch, kResidentPitch);
    }
}

// Adds the splits' sums of every kept element in split order, rounds once to fp16 and stores as the
// unsplit kernels do.  One workgroup row (blockIdx.y) per job.
constexpr int kSumThreads = 256;

template <int OUT>
__global__ void __launch_bounds__(kSumThreads) wgrad_sum_kernel(const WgradBatch B)
{
    const int j = blockIdx.y;
    const int64_t nnz = B.job[j].nnz, stride = B.partial_stride[j];
    const float *__restrict__ part = B.partial[j];
    for (int64_t k = (int64_t)blockIdx.x * kSumThreads + threadIdx.x; k < nnz; k += (int64_t)gridDim.x * kSumThreads) {
        float sum = part[k];
        for (int s = 1; s < B.splits; ++s) sum += part[s * stride + k];
        const _Float16 h = (_Float16)sum;                        // round to nearest even
        if (OUT == kOutF32) reinterpret_cast<float *>(B.job[j].gc)[k] = (float)h * B.inv_scale;
        else {
            _Float16 *dst = reinterpret_cast<_Float16 *>(B.job[j].gc) + k;
            *dst = B.accumulate ? (_Float16)(*dst + h) : h;
        }
    }
}

// What the matrix units sustain with nothing to fetch: every wave issues sixteen independent 16x16x32 fp16 MFMAs per
// iteration from registers, 4 x 4 blocks in the order of the kernels above, two waves to a SIMD as there.  The operands are
// ordinary fp16 values (a few set mantissa and exponent bits, varying by lane and block), because the clock
// the chip holds under this load, and with it the rate, depends on how many bits toggle.  Each workgroup
// leaves one float.
__global__ void __launch_bounds__(kWgThreads, 2) mfma_rate_kernel(int64_t iters, float *__restrict__ sink)
{
    f32x4 acc[4][4];
    half8 xa[4], yb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            xa[b][i] = (_Float16)(0.37f * (float)((int)((threadIdx.x + 3 * b) % 7) + i) - 1.f);
            yb[b][i] = (_Float16)(0.011f * (float)((int)((threadIdx.x + 2 * b) % 5) + 2 * i) - 0.03f);
        }
    for (int64_t it = 0; it < iters; ++it) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int bi = q / 4, bo = (bi & 1) ? 3 - q % 4 : q % 4;
            acc[bo][bi] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[bi], yb[bo], acc[bo][bi], 0, 0, 0);
        }
    }
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) sum += acc[i][j][r];
    sum += __shfl_xor(sum, 32, 64);
    if (threadIdx.x == 0) sink[blockIdx.x] = sum;
}

// Whether the two wave groups of a launch run half a stage apart (multiply_tile).  In step a short call is over
// earlier, apart a long one is faster per stage.  In us, in step and apart: 128 x 128 tiles, 1024 x 1024, 100 / 300 / 500 /
// 700 / 1003 / 1500 tokens 7.8 / 9.5 / 10.9 / 12.3 / 15.5 / 19.7 and 8.4 / 10.3 / 11.5 / 12.8 / 15.0 / 18.3; 256 x 256 tiles,
// 4096 x 4096, 64 / 100 / 160 / 200 / 300 tokens 11.4 / 13.2 / 14.2 / 16.3 / 18.8 and 12.4 / 14.1 / 14.6 / 16.2 / 17.9.  Tiles
// of 128 to 192 columns and the splits of a call have the one loop only.
bool loop_apart(int64_t tokens, bool small) { return tokens > (small ? 11 * stage_tokens(kSmallTile) : 6 * stage_tokens(kBigTile)); }

// The kernel of a tile shape: 32 * blocks columns of a 256-row tile, or the small one.
typedef void (*TileKernel)(const WgradBatch);
template <int OUT>
TileKernel tile_kernel_of(bool small, int blocks, bool apart, bool few)
{
    if (small && apart) return &wgrad_small_kernel<OUT, true, false>;         // long enough for the difference not to show
    if (small) return few ? &wgrad_small_kernel<OUT, false, true> : &wgrad_small_kernel<OUT, false, false>;
    switch (blocks) {
    case 4: return &wgrad_big_kernel<OUT, 4, true>;
    case 5: return &wgrad_big_kernel<OUT, 5, true>;
    case 6: return &wgrad_big_kernel<OUT, 6, true>;
    default: return apart ? &wgrad_big_kernel<OUT, 8, true> : &wgrad_big_kernel<OUT, 8, false>;
    }
}
TileKernel tile_kernel(int out, bool small, int blocks, bool apart, bool few)
{
    if (out == kOutPartial) return small ? &wgrad_small_kernel<kOutPartial, true, false> : &wgrad_big_kernel<kOutPartial, 8, true>;
    return out == kOutF32 ? tile_kernel_of<kOutF32>(small, blocks, apart, few) : tile_kernel_of<kOutF16>(small, blocks, apart, few);
}

// The LDS size above 64 KiB is a per-device attribute of a kernel: set once per device, where the
// device's number of compute units is read too.
hipError_t configure_once(int *cus)
{
    static std::atomic<uint64_t> configured{0};
    static int cus_of[64];
    int device = 0;
    if (hipError_t e = hipGetDevice(&device)) return e;
    const uint64_t bit = 1ull << (device & 63);
    if (!(configured.load(std::memory_order_acquire) & bit)) {
        for (int out : {(int)kOutF32, (int)kOutF16, kOutPartial})
            for (int shape = 3; shape <= 8; ++shape)                             // 3: the small tile
                for (bool apart : {false, true})
                    for (bool few : {false, true}) {
                        const void *k = reinterpret_cast<const void *>(tile_kernel(out, shape == 3, shape, apart, few));
                        if (hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes)) return e;
                    }
        int n = 0;
        if (hipError_t e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, device)) return e;
        cus_of[device & 63] = n;
        configured.fetch_or(bit, std::memory_order_release);
    }
    *cus = cus_of[device & 63];
    return hipSuccess;
}

}  // namespace

hipError_t wgrad_configure(int *cus) { return configure_once(cus); }

hipError_t launch_mfma_rate(int64_t iters, float *sink, int workgroups, hipStream_t s)
{
    if (workgroups > 0) mfma_rate_kernel<<<dim3((unsigned)workgroups), dim3(kWgThreads), 0, s>>>(iters, sink);
    return hipGetLastError();
}

namespace {

uint32_t per_group_of(int tiles_in) { return (uint32_t)((1ull << 32) / ((uint32_t)kGroupDepth * (uint32_t)tiles_in) + 1u); }

// The jobs' tiles of a shape, layer after layer.
void cut_tiles(WgradBatch *b, int rows, int cols)
{
    b->tile_cols = cols;
    b->first_tile[0] = 0;
    for (int k = 0; k < b->jobs; ++k) {
        b->tiles_out[k] = (int)ceil_div(b->job[k].out, rows);
        b->tiles_in[k] = (int)ceil_div(b->job[k].in, cols);
        b->first_tile[k + 1] = b->first_tile[k] + b->tiles_out[k] * b->tiles_in[k];
        b->per_group[k] = per_group_of(b->tiles_in[k]);
    }
}

// The call's job list with its large tiles; false if there is nothing to write.
bool list_tiles(const WgradJob *jobs, int count, float inv_scale, int accumulate, WgradBatch *out)
{
    WgradBatch &b = *out;
    b.jobs = 0; b.inv_scale = inv_scale; b.accumulate = accumulate; b.splits = 1;
    for (int j = 0; j < count && b.jobs < kWgradMaxJobs; ++j) {
        if (jobs[j].out <= 0 || jobs[j].in <= 0 || jobs[j].nnz <= 0) continue;     // nothing to write
        const int k = b.jobs++;
        b.job[k] = jobs[j];
    }
    if (b.jobs == 0) return false;
    cut_tiles(&b, kBigTile, kBigTile);
    for (int k = b.jobs; k < kWgradMaxJobs; ++k) {
        b.job[k] = b.job[0]; b.tiles_out[k] = b.tiles_in[k] = 1; b.first_tile[k + 1] = b.first_tile[b.jobs];
        b.per_group[k] = per_group_of(1);
    }
    return true;
}

void launch_tiles(int out_kind, const WgradBatch &b, bool small, unsigned blocks, hipStream_t s)
{
    const dim3 grid((blocks + 7) / 8 * 8), threads(kWgThreads);  // whole rounds of the 8 XCDs; the surplus exits at once
    int64_t tokens = 0;
    for (int j = 0; j < b.jobs; ++j) tokens = b.job[j].tokens > tokens ? b.job[j].tokens : tokens;
    tile_kernel(out_kind, small, b.tile_cols / 32, loop_apart(tokens, small), blocks < kFewBlocks)<<<grid, threads, kLdsBytes, s>>>(b);
}

void launch_resident(int out_kind, WgradBatch &b, hipStream_t s)
{
    b.quadrants = 0; b.first = 0; b.tiles = b.first_tile[b.jobs];
    const dim3 grid((unsigned)((b.tiles + 7) / 8 * 8)), threads(kResidentThreads);
    if (out_kind == kOutF32) wgrad_resident_kernel<kOutF32><<<grid, threads, kResidentLds, s>>>(b);
    else wgrad_resident_kernel<kOutF16><<<grid, threads, kResidentLds, s>>>(b);
}

// What the tile rules price: the longest job's 32-token stages and the kept fraction of all jobs together.
struct CallSize {
    int stages;
    double keep, nnz;
};
CallSize size_of(const WgradBatch &b)
{
    CallSize c = {0, 0.0, 0.0};
    double elements = 0.0;
    for (int j = 0; j < b.jobs; ++j) {
        const int s = (int)ceil_div(b.job[j].tokens, (int64_t)stage_tokens(kBigTile));       // tokens fit 31 bits
        c.stages = s > c.stages ? s : c.stages;
        c.nnz += (double)b.job[j].nnz;
        elements += (double)b.job[j].out * b.job[j].in;
    }
    c.keep = c.nnz / elements;
    return c;
}

// Tiles of all jobs in a shape: less than 2^21 (8 layers of less than 2^31 elements, sides up to 2^24, of 128 x 128 at least).
int count_tiles(const WgradBatch &b, int rows, int cols)
{
    int n = 0;
    for (int j = 0; j < b.jobs; ++j) n += ((b.job[j].out + rows - 1) / rows) * ((b.job[j].in + cols - 1) / cols);
    return n;
}

// Time in us of a launch of that many workgroups of one shape (columns of a 256-row tile, or 128 x 128 with `small`), each
// of them `stages` stages long: what is around a tile's loop, the loop, and the gather of what the tile keeps, per
// round of the compute units.  A stage costs less while part of the chip is idle (the clock is higher and the memory
// less busy): 256 columns 0.545 us up to half of the compute units, 0.73 with all of them.  Fitted to 1000 calls (sides 512 ..
// 12000, 100 .. 8192 tokens, 3 to 25 % kept) in every shape: 2 to 3.5 % rms in the tiles of 256 rows, 10 % in 128 x 128 up to four rounds.
double launch_us(bool small, int cols, int workgroups, int stages, double keep, int cus)
{
    const double rounds = (workgroups + cus - 1) / cus, full = workgroups / (rounds * cus);
    const double busy = full < 0.5 ? 0.0 : full > 0.9 ? 1.0 : (full - 0.5) / 0.4;
    double around = 6.0, stage = 0.73, idle_stage = 0.545, gather = 0.36e-3, area = 256.0 * cols;
    if (small) around = 4.2, stage = 0.26, idle_stage = 0.231, gather = 0.34e-3, area = 128.0 * 128.0;
    else if (cols == 128) around = 5.9, stage = 0.473, idle_stage = 0.43, gather = 0.235e-3;
    else if (cols == 160) stage = 0.538, idle_stage = 0.448, gather = 0.24e-3;
    else if (cols == 192) around = 5.9, stage = 0.615, idle_stage = 0.49, gather = 0.30e-3;
    return 1.5 + rounds * (around + (idle_stage + busy * (stage - idle_stage)) * stages + gather * keep * area);
}

// The same of the resident shape: whole rounds of four workgroups to every compute unit, and a last one with `most` of them on the
// busiest.  Fitted to 411 calls of up to 2048 tokens: 6 % rms.
double resident_us(int workgroups, int stages, double keep, int cus)
{
    const int rounds = workgroups / (4 * cus), most = (workgroups - rounds * 4 * cus + cus - 1) / cus;
    const double kept = keep * 16.384;                         // thousand entries a tile
    double us = 1.4 + rounds * (3.85 + 0.986 * stages + 0.98 * kept);
    if (most > 0) us += 3.2 + (0.1 + 0.2 * most) * stages + 0.444 * kept * most;
    return us;
}

// How the tiles of an unsplit call are launched: `wide` of the list, in tiles of 32 * blocks columns, and the
// last `quarters` large tiles of the list as small ones (blocks is 8 then); blocks == 0: all in the resident shape.  us: what
// it takes by the prices above.
struct TilePlan {
    int wide, quarters, blocks;
    double us;
};

// Short calls of more tiles than compute units go to four workgroups to a unit.  Us, as the rules below would run it and so, 10 % kept
// unless said: 2320 x 2624, 112 tokens, 5 % 9.8 and 7.2; 4096 x 4096, 200 and 300 tokens 14.4 and 13.1, 16.9 and 16.8; 2376 x 7080, 235
// tokens, 5 % 22.8 and 19.1; 7856 x 4632, 106 tokens, 20 % 43.3 and 28.6; 10760 x 5200, 408 tokens, 12 % 65.8 and 62.8; past about 600
// tokens the copies of the smaller tiles cost more than is gained (4096 x 4096, 500 tokens 20.1 and 21.3, 1000 33.3 and 37.5), and with a
// tile to a compute unit or less there is nothing to share one.  2 % below the other price, because that of this shape is the rougher one.
TilePlan resident_if_quicker(const TilePlan &plan, int small_tiles, const CallSize &c, int cus)
{
    if (small_tiles <= cus) return plan;
    const double us = resident_us(small_tiles, c.stages, c.keep, cus);
    return us * 1.02 < plan.us ? TilePlan{0, small_tiles, 0, us} : plan;
}

// Large tiles in whole rounds of the compute units; what is left over after the last whole
// round goes to the small shape when that is the quicker way to finish it: up to half a round
// of large tiles is at most two rounds of small ones, and a small round takes 0.4 of a large.
// A call of less than a round leaves compute units idle: it takes the shape that is priced lowest.  3072 x 3072 (144 large
// tiles, 228 of 160 columns): 2048 tokens 47.5 -> 43.8 us, 512 tokens 21.5 -> 18.9; 2560 x 2560 without a workspace (100, or
// 200 of 128 columns) 42.1 -> 38.4.  (224 columns are not built: they would be the best shape where 192 columns
// overflow the round and 224 do not, by these prices for at most 6 %.)  Behind whole rounds the same (the last columns of the
// largest layer in narrower tiles that make one full round) gains nothing: with all compute units busy the
// chip is at its power limit, and idle ones let the others run faster (400 tiles 107.1 -> 103.6 us, but 102.4 -> 106.1
// for the transposed layer and 104.1 -> 110.0 for 432 tiles).
TilePlan plan_tiles(const WgradBatch &b, int cus, bool round_forced)
{
    const int tiles = b.first_tile[b.jobs];
    const int shape = knob(SAMO_KNOB_WGRAD_TILE, 0);           // tuning and test aid: 128, 256 or 512 (the resident shape)
    if (shape == kSmallTile) return {0, tiles, 8, 0.0};
    if (shape == kResidentShape) return {0, tiles, 0, 0.0};
    if (shape == kBigTile || cus <= 0) return {tiles, 0, 8, 0.0};
    const int forced_cols = knob(SAMO_KNOB_WGRAD_COLS, 0);     // test aid: narrow tiles whatever they cost
    const CallSize c = size_of(b);
    TilePlan plan = {tiles, 0, 8, launch_us(false, 256, tiles, c.stages, c.keep, cus)};
    const int quarters = count_tiles(b, kSmallTile, kSmallTile);
    if (forced_cols == 0 && (tiles >= cus || round_forced)) {
        const int left = tiles % cus;
        if (left != 0 && left <= cus / 2)
            plan = {tiles - left, left, 8,
                    launch_us(false, 256, tiles - left, c.stages, c.keep, cus) + launch_us(true, 128, left * 4, c.stages, c.keep, cus)};
        return round_forced ? plan : resident_if_quicker(plan, quarters, c, cus);
    }
    const double small_us = launch_us(true, 128, quarters, c.stages, c.keep, cus);
    if (small_us < plan.us) plan = {0, tiles, 8, small_us};
    if (forced_cols) plan.us = 1e30;
    for (int blocks = 4; blocks <= 6; ++blocks) {
        if (forced_cols && forced_cols != 32 * blocks) continue;
        const int narrow = count_tiles(b, kBigTile, 32 * blocks);
        const double us = launch_us(false, 32 * blocks, narrow, c.stages, c.keep, cus);
        if (us < plan.us) plan = {narrow, 0, blocks, us};
    }
    return forced_cols ? plan : resident_if_quicker(plan, quarters, c, cus);
}

// Whether, and how, the tiles of a call are shared by several workgroups each: `splits` workgroups per tile
// of the shape `small` says; splits == 1: not at all.
struct SplitPlan {
    int splits;
    bool small;
};

// A call whose large tiles would fill less than half of the compute units may have its tokens split over workgroups.
// The splits' sums are written and read at 6.5 TB/s (in part in the caches) by one more launch (2.8 us and 0.2 per split).  A split is taken where
// it is priced below the call as plan_tiles would run it.  Unsplit and split, 10 % kept, us: 512 x 512,
// 2048 tokens 21.5 -> 14.6, 8192 tokens 62.6 -> 17.6; 1024 x 1024, 8192 tokens 59.7 -> 27.5; 2560 x 2560, 2048 tokens
// 38.4 -> 36.1, but 1024 tokens 24.4 and 26.1, 300 tokens 13.9 and 17.5: not split.
SplitPlan plan_split(const WgradBatch &b, int cus)
{
    SplitPlan best = {1, true};
    const int tiles = b.first_tile[b.jobs];
    if (tiles * 2 > cus) return best;
    const int forced = knob(SAMO_KNOB_WGRAD_SPLIT, 0), shape = knob(SAMO_KNOB_WGRAD_TILE, 0);
    const CallSize c = size_of(b);
    if (forced > 1) {                                          // bounded: the workgroups of a launch are counted in 32 bits
        const int most = c.stages < kMaxSplits ? c.stages : kMaxSplits;
        return {forced < most ? forced : most > 0 ? most : 1, shape != kBigTile};
    }
    if (forced == 1 || shape != 0 || knob(SAMO_KNOB_WGRAD_ROUND, 0) > 0 || knob(SAMO_KNOB_WGRAD_COLS, 0) > 0 || c.stages < 8)
        return best;
    const int quarters = count_tiles(b, kSmallTile, kSmallTile);
    double least = plan_tiles(b, cus, false).us;
    for (int s = 2; s <= 16 && s * 4 <= c.stages; ++s)
        for (int small = 0; small <= 1; ++small) {
            const double us = launch_us(small != 0, kBigTile, (small ? quarters : tiles) * s, (c.stages + s - 1) / s, c.keep, cus) +
                              2.8 + 0.2 * s + 8.0 * s * c.nnz / 6.5e6;
            if (us < least) {
                least = us;
                best = {s, small != 0};
            }
        }
    return best;
}

// Places the splits' sums in the workspace (or only adds up its size, with ws == NULL); returns the bytes.
size_t place_partials(WgradBatch *b, const SplitPlan &plan, unsigned char *ws)
{
    const int64_t unit = stage_tokens(plan.small ? kSmallTile : kBigTile);
    size_t at = 0;
    b->splits = plan.splits;
    for (int j = 0; j < kWgradMaxJobs; ++j) {
        const int64_t stages = ceil_div(b->job[j].tokens, unit);
        b->split_tokens[j] = ceil_div(stages, (int64_t)plan.splits) * unit;
        b->partial_stride[j] = ceil_div(b->job[j].nnz, (int64_t)64) * 64;
        b->partial[j] = reinterpret_cast<float *>(ws + at);
        if (j < b->jobs) at += (size_t)b->partial_stride[j] * plan.splits * sizeof(float);
    }
    return at;
}

}  // namespace

// Bytes launch_wgrad can use to split these jobs' tokens over workgroups (0: it would not split them).
hipError_t wgrad_workspace(const WgradJob *jobs, int count, size_t *bytes)
{
    *bytes = 0;
    WgradBatch b;
    if (!list_tiles(jobs, count, 1.f, 0, &b)) return hipSuccess;
    int cus = 0;
    if (hipError_t e = configure_once(&cus)) return e;
    const SplitPlan plan = plan_split(b, cus);
    if (plan.splits > 1) *bytes = place_partials(&b, plan, nullptr);
    return hipSuccess;
}

hipError_t launch_wgrad(int out_kind, const WgradJob *jobs, int count, float inv_scale, int accumulate, void *ws,
                        size_t ws_bytes, hipStream_t s)
{
    WgradBatch b;
    if (!list_tiles(jobs, count, inv_scale, accumulate, &b)) return hipSuccess;
    int cus = 0;
    if (hipError_t e = configure_once(&cus)) return e;
    const int big_tiles = b.first_tile[b.jobs];
    if (ws) {
        const SplitPlan plan = plan_split(b, cus);
        if (plan.splits > 1 && place_partials(&b, plan, static_cast<unsigned char *>(ws)) <= ws_bytes) {
            b.quadrants = plan.small ? 1 : 0; b.first = 0; b.tiles = big_tiles;
            launch_tiles(kOutPartial, b, plan.small, (unsigned)(big_tiles * plan.splits * (plan.small ? 4 : 1)), s);
            int64_t most = 0;
            for (int j = 0; j < b.jobs; ++j) most = b.job[j].nnz > most ? b.job[j].nnz : most;
            const int64_t wgs = ceil_div(most, (int64_t)kSumThreads);
            const dim3 grid((unsigned)(wgs < 4096 ? wgs : 4096), (unsigned)b.jobs);
            if (out_kind == kOutF32) wgrad_sum_kernel<kOutF32><<<grid, dim3(kSumThreads), 0, s>>>(b);
            else wgrad_sum_kernel<kOutF16><<<grid, dim3(kSumThreads), 0, s>>>(b);
            return hipGetLastError();
        }
        b.splits = 1;
    }
    const int round = knob(SAMO_KNOB_WGRAD_ROUND, 0);          // test aid: tiles per round in place of the CU count
    const TilePlan plan = plan_tiles(b, round > 0 ? round : cus, round > 0);
    if (plan.blocks == 0) {
        cut_tiles(&b, kSmallTile, kSmallTile);
        launch_resident(out_kind, b, s);
        return hipGetLastError();
    }
    if (plan.wide > 0) {
        b.quadrants = 0; b.first = 0; b.tiles = plan.wide;
        if (plan.blocks != 8) cut_tiles(&b, kBigTile, 32 * plan.blocks);
        launch_tiles(out_kind, b, false, (unsigned)plan.wide, s);
    }
    if (plan.quarters > 0) {
        b.quadrants = 1; b.first = plan.wide; b.tiles = plan.quarters;
        launch_tiles(out_kind, b, true, (unsigned)(plan.quarters * 4), s);
    }
    return hipGetLastError();
}

}  // namespace samo
