// Mask -> index construction (the paper's ind_i, Section III and III-B) for gfx950.
//
// The pruner's output arrives as a byte mask over the flattened layer.  The mask is read ONCE.
// A workgroup of eight wavefronts owns a block of 64, 128 or 256 consecutive segments of
// SAMO_SEG_ELEMS = 1024 mask bytes, taken in passes of 64; in a pass a wavefront takes eight of
// them, every lane loading 16 bytes of each, so a segment is one coalesced 1 KiB access and eight
// are in flight per lane.  The kept bytes are counted per lane (popcount of a 16-bit flag word)
// and scanned across the wave, which gives the segments their totals; the number of kept elements in
// front of the workgroup then comes from a chained scan across workgroups (each publishes its own count
// at once and the running total as soon as it knows it; a successor sums the counts back to the nearest
// running total); finally
// the ascending int32 positions are produced from the flag bits still held in registers,
// collected per pair of segments in LDS and stored as contiguous runs.  All integer work: one read of the
// mask plus the write of the index.
//
// A caller that has to know the count before it can allocate the index makes two calls.  Counting needs no chain: the
// counts within blocks of 64 segments and the blocks' offsets are two launches, neither of which waits for anything
// (count_kernel, offsets_kernel).  The second call need not read the mask again: the first can leave its flag words (an eighth of the
// mask's size) in a buffer of the caller, and fill_kernel makes the positions from those and from seg_ptr.  Seven layers of
// the 2.7B shape (550 M mask bytes, 10 % kept): 101 + 6.5 us and 56 us.  (The chained kernel counted them in 125 + 3 us: a workgroup
// that waits for its predecessors reads nothing meanwhile.)
//
// The chain lives in seg_ptr itself: seg_ptr[e], e the end of a workgroup's block of segments, is
// the number of kept elements up to there — exactly the running total the next workgroup needs.
// While unknown it holds kEmpty, then -1 - (own count), then the final value.  Workgroups take
// their blocks in the order of a ticket drawn at start, so every predecessor of a running
// workgroup is itself running or done and the wait for it ends; the wait is bounded all the same,
// and a workgroup that gives up marks its block kPoison, which its successors pass on and the
// last block of the job reports as *nnz = -1.
#include "common.h"

namespace samo {
namespace {

constexpr int kIndexThreads = 512;        // index_kernel: eight wavefronts per workgroup
constexpr int kWavesPerWg = kIndexThreads / 64;

// bit (8*b + 7) set for every non-zero byte b of x
__device__ __forceinline__ uint32_t nonzero_byte_flags(uint32_t x)
{
    return (((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) & 0x80808080u;
}

// 16 flag bits for 16 mask bytes; bytes at or beyond n read as 0.
__device__ __forceinline__ uint32_t lane_flags(const uint8_t *__restrict__ mask, int64_t n, int64_t first)
{
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    if (first + 16 <= n) {
        typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
        const u32x4 q = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(mask + first));   // read once
        w[0] = q.x; w[1] = q.y; w[2] = q.z; w[3] = q.w;
    } else {
        for (int b = 0; b < 16; ++b)
            if (first + b < n) w[b >> 2] |= (uint32_t)mask[first + b] << (8 * (b & 3));
    }
    // Every non-zero byte is now 0x80: a dot product of the four bytes of a word with the weights
    // 1, 2, 4, 8 (16 .. 128 for the next word, accumulated) is 128 times their flag bits in order.
    uint32_t lo = __builtin_amdgcn_udot4(nonzero_byte_flags(w[0]), 0x08040201u, 0u, false);
    lo = __builtin_amdgcn_udot4(nonzero_byte_flags(w[1]), 0x80402010u, lo, false);
    uint32_t hi = __builtin_amdgcn_udot4(nonzero_byte_flags(w[2]), 0x08040201u, 0u, false);
    hi = __builtin_amdgcn_udot4(nonzero_byte_flags(w[3]), 0x80402010u, hi, false);
    return (lo >> 7) | (hi << 1);
}

__device__ __forceinline__ int wave_sum(int x)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
    return x;
}

// Inclusive scan over the 64 lanes with data-parallel primitives: a shifted add within each row of
// 16 lanes (four steps), then lane 15 of a row added to the whole next row and lane 31 to the upper
// half — the operands move inside the vector ALU, no trip through the LDS crossbar.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_add(int x)
{
    // lanes the pattern does not feed read 0 (bound_ctrl); rows outside ROW_MASK add 0
    return x + __builtin_amdgcn_update_dpp(0, x, CTRL, ROW_MASK, 0xf, true);
}

__device__ __forceinline__ int wave_inclusive_scan(int x, int lane)
{
    (void)lane;
    x = dpp_add<0x111, 0xf>(x);               // row_shr:1
    x = dpp_add<0x112, 0xf>(x);               // row_shr:2
    x = dpp_add<0x114, 0xf>(x);               // row_shr:4
    x = dpp_add<0x118, 0xf>(x);               // row_shr:8
    x = dpp_add<0x142, 0xa>(x);               // row_bcast:15 into rows 1 and 3
    x = dpp_add<0x143, 0xc>(x);               // row_bcast:31 into rows 2 and 3
    return x;
}

// Workgroup -> job lookup for the batched launches: the job table travels in the kernel
// argument segment (scalar loads, no device table to allocate or copy), wg_start is the
// exclusive prefix of the jobs' workgroup counts.
// The first job's entries are requested with `num`, all at once: the caches are cold when a launch begins, and every line of
// the table that is read one after the other is a trip of its own (a mask of 42 MB, whole build, with the fill's loads side by side as well: 38.7 -> 37.5 us).
__device__ __forceinline__ int find_job(const IndexBatch &batch, int wg)
{
    asm volatile("" ::"s"(batch.num), "s"(batch.wg_start[0]), "s"(batch.mask[0]), "s"(batch.n[0]), "s"(batch.idx[0]), "s"(batch.cap[0]),
                 "s"(batch.seg_ptr[0]), "s"(batch.nnz[0]), "s"(batch.flags[0]));
    int lo = 0, hi = batch.num;                 // invariant: wg_start[lo] <= wg < wg_start[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (batch.wg_start[mid] <= wg) lo = mid; else hi = mid;
    }
    return lo;
}

// A workgroup takes its block in PASSES passes of 64 KiB: in a pass every wave loads eight
// consecutive segments — all eight 16-byte loads of a lane in flight before anything is reduced —
// and keeps only their flag bits (two segments to a register) for the fill.  The per-lane counts travel
// through the wave scans packed two to a register: a count is at most 1024, a 16-bit field is
// enough.  What a workgroup pays once whatever its block's size — drawing the ticket, waiting for
// its predecessors in the chain — is a dozen microseconds, against less than two for a pass, so a
// launch with enough mask to keep the compute units busy takes four passes per workgroup (256 KiB
// blocks), smaller ones two or one.
// The fill takes the segments in pairs, 32 consecutive elements to a lane: a pair's positions are one
// contiguous run of idx, and the loop that turns a lane's flag word into positions runs as often as the
// fullest lane of the wave has kept elements, about 8 times for a pair at 10 % kept, where two words of 16
// took 5 to 6 each.
constexpr int kSegsPerPass = 8;           // per wave
constexpr int kPairs = kSegsPerPass / 2;
static_assert(kFlagGroupSegs == kSegsPerPass && kPairs == 4, "a lane's flag words of a pass are one 16-byte vector");
constexpr int kMaxPasses = 4;
__host__ __device__ constexpr int segs_per_wg(int passes) { return kSegsPerPass * kWavesPerWg * passes; }

// States of a chain entry other than a final running total (which is >= 0).
constexpr int kEmpty = INT32_MIN;         // nothing published yet
constexpr int kPoison = INT32_MIN + 1;    // a predecessor gave up
__device__ __forceinline__ int encode_count(int c) { return -1 - c; }
__device__ __forceinline__ int decode_count(int v) { return -1 - v; }

__device__ __forceinline__ int chain_load(const int32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void chain_store(int32_t *p, int v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// seg_ptr position of the chain entry of block b (blocks of `block_segs` segments): the end of its segments.
__device__ __forceinline__ int64_t chain_slot(int64_t b, int64_t nseg, int block_segs)
{
    const int64_t e = (b + 1) * block_segs;
    return e < nseg ? e : nseg;
}

// Prepares a batch: every job's seg_ptr[0] = 0 and *nnz = 0 (the ticket counter is one of these),
// every block's chain entry = kEmpty.
__global__ void __launch_bounds__(kThreads)
index_init_kernel(const IndexBatch batch)
{
    const int t = blockIdx.x * kThreads + threadIdx.x;
    if (t < batch.num) {
        batch.seg_ptr[t][0] = 0;
        *batch.nnz[t] = 0;
    }
    if (t < batch.wg_start[batch.num]) {
        const int job = find_job(batch, t);
        const int64_t nseg = (batch.n[job] + kSeg - 1) / kSeg;
        batch.seg_ptr[job][chain_slot(t - batch.wg_start[job], nseg, segs_per_wg(batch.passes))] = kEmpty;
    }
}

// Number of kept elements in front of block `blk` of a job (wave 0 of the workgroup, all lanes):
// sums the published counts of the predecessors back to the nearest running total, 64 chain
// entries per look (more per look did not pay: measured).  Returns kPoison if a predecessor gave
// up or never shows.
__device__ __forceinline__ int kept_before_block(const int32_t *seg_ptr, int64_t nseg, int block_segs, int blk, int lane,
                                                 int spin_limit)
{
    int prefix = 0;
    int back = blk - 1;                       // nearest predecessor not yet accounted for
    int spins = 0;
    while (back >= 0) {
        const int b = back - lane;            // lane i looks at block back - i
        int v = kEmpty;
        if (b >= 0) v = chain_load(seg_ptr + chain_slot(b, nseg, block_segs));
        const unsigned long long m_total = __ballot(b >= 0 && v >= 0);
        const int first_total = m_total ? __ffsll((long long)m_total) - 1 : 64;
        // the lanes in front of the first running total must all hold counts
        const bool wanted = lane <= first_total && b >= 0;
        if (__any(wanted && v == kPoison)) return kPoison;
        if (__any(wanted && v == kEmpty)) {
            if (++spins > spin_limit) return kPoison;
            __builtin_amdgcn_s_sleep(2);
            continue;
        }
        int part = 0;
        if (wanted) part = (lane == first_total) ? v : decode_count(v);
        prefix += wave_sum(part);
        if (first_total < 64) break;
        back -= 64;
    }
    return prefix;
}

// Between one lane's LDS stores and another lane's loads, both of one wave: they execute in order, this keeps the
// compiler to it (a fence of wavefront scope is no instruction).
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Views of the wave's LDS area, an array of int32_t, that may alias it.
typedef uint16_t __attribute__((may_alias)) AliasU16;
typedef uint32_t __attribute__((ext_vector_type(4), may_alias)) AliasU32x4;

// From 16 elements of either segment of every pair (as the mask is loaded: 1 KiB of one segment per
// instruction; lanes that load 32 bytes apart read 17 % slower) to 32 consecutive elements of the pair, by
// way of the wave's LDS area.
__device__ __forceinline__ void pair_words(const uint32_t (&halves)[kPairs], uint32_t (&word)[kPairs], int32_t *stage, int lane)
{
    AliasU16 *to = reinterpret_cast<AliasU16 *>(stage) + (lane >> 1) * 2 * kPairs + (lane & 1);
#pragma unroll
    for (int j = 0; j < kPairs; ++j) {
        to[2 * j] = (uint16_t)halves[j];                                 // word (lane / 2) of the pair's first segment
        to[32 * 2 * kPairs + 2 * j] = (uint16_t)(halves[j] >> 16);       // ... of its second
    }
    wave_lds_order();
    const AliasU32x4 w = reinterpret_cast<const AliasU32x4 *>(stage)[lane];
    word[0] = w.x; word[1] = w.y; word[2] = w.z; word[3] = w.w;
    wave_lds_order();
}

// The other way round: 16 elements of either segment of every pair from 32 consecutive ones.
__device__ __forceinline__ void word_halves(const uint32_t (&word)[kPairs], uint32_t (&halves)[kPairs], int32_t *stage, int lane)
{
    reinterpret_cast<AliasU32x4 *>(stage)[lane] = (AliasU32x4){word[0], word[1], word[2], word[3]};
    wave_lds_order();
    const AliasU16 *from = reinterpret_cast<const AliasU16 *>(stage) + (lane >> 1) * 2 * kPairs + (lane & 1);
#pragma unroll
    for (int j = 0; j < kPairs; ++j) halves[j] = from[2 * j] | ((uint32_t)from[32 * 2 * kPairs + 2 * j] << 16);
    wave_lds_order();
}

// A lane's flag words of a group of eight segments, one vector, past the caches.
__device__ __forceinline__ void store_flags(uint4 *to, const uint32_t (&word)[kPairs])
{
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store((u32x4){word[0], word[1], word[2], word[3]}, reinterpret_cast<u32x4 *>(to));
}

// Writes the positions of one pair of segments, base the pair's first element; idx[out0 ..] takes them in order,
// nothing at or beyond cap.  The positions go to LDS (the wave's own kSeg ints: no workgroup barrier), then leave as
// contiguous 256-byte stores.  Lane l holds the flag word of elements base + 32 l .. base + 32 l + 31 in `word`; a pair with
// more than kSeg of them is written segment by segment, from `half`: the flag bits of elements 16 l .. 16 l + 15 of
// the first segment, and of the second in the upper 16 bits.  Two full segments would not fit the LDS area, and
// the fuller the lanes, the more of their positions share a bank: a full lane's run starts 32 words after the
// run of the lane before it, 16 segment by segment (an 8000 x 8000 layer of which everything is kept, whole build: 94 us, and 155 with
// two halves of 32 elements a lane; the line lies where the pair stops fitting: 640, 768 and 896 are slower or the same).
__device__ __forceinline__ void emit_pair(uint32_t word, uint32_t half, int base, int64_t out0, int64_t cap,
                                          int32_t *__restrict__ idx, int32_t *stage, int lane)
{
    const int cnt = __popc(word);
    const int incl = wave_inclusive_scan(cnt, lane);
    const int total = __builtin_amdgcn_readlane(incl, 63);
    auto write = [&](uint32_t bits, int first, int at, int count) {
        int32_t *to = stage + at;
        while (bits) {
            *to++ = first + __builtin_ctz(bits);
            bits &= bits - 1;
        }
        wave_lds_order();
        count = storable(cap, out0, count);
        int32_t *__restrict__ out = idx + out0;
        for (int o = lane; o < count; o += 64) out[o] = stage[o];
        wave_lds_order();
    };
    if (total <= kSeg) {
        write(word, base + lane * 32, incl - cnt, total);
        return;
    }
    const int c = __popc(half & 0xffffu) | (__popc(half >> 16) << 16);        // a segment's count fits 16 bits
    const int before = wave_inclusive_scan(c, lane) - c;
    const int first_total = __builtin_amdgcn_readlane(before + c, 63) & 0xffff;
    write(half & 0xffffu, base + lane * 16, before & 0xffff, first_total);
    out0 += first_total;
    write(half >> 16, base + kSeg + lane * 16, before >> 16, total - first_total);
}

template <int PASSES>
__global__ void __launch_bounds__(kIndexThreads)
index_kernel(const IndexBatch batch)
{
    constexpr int kSegsPerWave = kSegsPerPass * PASSES;
    constexpr int kSegsPerWg = segs_per_wg(PASSES);
    constexpr int kPerLane = kSegsPerWg / 64;     // segment counts a lane of wave 0 takes in the block's scan
    __shared__ int sh_ticket;
    __shared__ int sh_seg[kSegsPerWg];        // kept elements per segment, then in front of it within the block
    __shared__ int sh_base;                   // kept elements in front of the block, or kPoison
    __shared__ __attribute__((aligned(16))) int32_t sh_stage[kWavesPerWg][kSeg];   // positions of a pair per wave, on their way out
    if (threadIdx.x == 0) sh_ticket = (int)atomicAdd(reinterpret_cast<unsigned long long *>(batch.ticket), 1ull);
    __syncthreads();
    const int ticket = __builtin_amdgcn_readfirstlane(sh_ticket);
    const int job = find_job(batch, ticket);
    const int blk = ticket - batch.wg_start[job];
    const int64_t n = batch.n[job];
    const int64_t nseg = (n + kSeg - 1) / kSeg;
    int32_t *__restrict__ seg_ptr = batch.seg_ptr[job];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t seg0 = ((int64_t)blk * kWavesPerWg + wave) * kSegsPerWave;     // segments beyond nseg read as empty

    uint32_t fp[PASSES][kPairs];              // flag bits of segments 2j (low half) and 2j + 1 (high half) of a pass
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        uint32_t f[2 * kPairs];
#pragma unroll
        for (int q = 0; q < 2 * kPairs; ++q)
            f[q] = lane_flags(batch.mask[job], n, (seg0 + p * kSegsPerPass + q) * kSeg + lane * 16);
#pragma unroll
        for (int j = 0; j < kPairs; ++j) {
            const int incl = wave_inclusive_scan(__popc(f[2 * j]) | (__popc(f[2 * j + 1]) << 16), lane);
            if (lane == 63) {                  // the last lane's inclusive prefixes are the segment totals
                int *dst = sh_seg + wave * kSegsPerWave + p * kSegsPerPass + 2 * j;
                dst[0] = incl & 0xffff;
                dst[1] = incl >> 16;
            }
            fp[p][j] = f[2 * j] | (f[2 * j + 1] << 16);
        }
        asm volatile("" ::: "memory");        // the next pass's loads are requested after this pass's flag words exist
    }
    __syncthreads();

    const int64_t slot = chain_slot(blk, nseg, kSegsPerWg);
    const bool last_block = (blk + 1 == batch.wg_start[job + 1] - batch.wg_start[job]);
    if (wave == 0) {
        int c[kPerLane], mine = 0;
#pragma unroll
        for (int i = 0; i < kPerLane; ++i) {
            c[i] = sh_seg[kPerLane * lane + i];
            mine += c[i];
        }
        const int incl = wave_inclusive_scan(mine, lane);
        const int total = __shfl(incl, 63, 64);
        if (blk > 0 && lane == 0) chain_store(seg_ptr + slot, encode_count(total));
        const int before = kept_before_block(seg_ptr, nseg, kSegsPerWg, blk, lane, batch.spin_limit);
        if (lane == 0) {
            chain_store(seg_ptr + slot, before == kPoison ? kPoison : before + total);
            sh_base = before;
            if (last_block) *batch.nnz[job] = (before == kPoison) ? -1 : (int64_t)before + total;
        }
        int run = incl - mine;
#pragma unroll
        for (int i = 0; i < kPerLane; ++i) {
            sh_seg[kPerLane * lane + i] = run;
            run += c[i];
        }
    }
    __syncthreads();
    const int base = __builtin_amdgcn_readfirstlane(sh_base);
    if (base == kPoison) return;

    // seg_ptr entries strictly inside the block (its first is the predecessor's chain entry)
    const int64_t first_seg = (int64_t)blk * kSegsPerWg;
    for (int t = threadIdx.x; t < kSegsPerWg; t += kIndexThreads)
        if (t >= 1 && first_seg + t < slot) seg_ptr[first_seg + t] = base + sh_seg[t];

    const int64_t cap = batch.cap[job];
    if (cap <= 0 || seg0 >= nseg) return;      // no room: this job only counts
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        uint32_t word[kPairs];
        pair_words(fp[p], word, sh_stage[wave], lane);
#pragma unroll
        for (int j = 0; j < kPairs; ++j) {
            const int sq = p * kSegsPerPass + 2 * j;
            emit_pair(word[j], fp[p][j], (int)((seg0 + sq) * kSeg),             // a layer's flat size fits int32
                      (int64_t)base + __builtin_amdgcn_readfirstlane(sh_seg[wave * kSegsPerWave + sq]), cap, batch.idx[job], sh_stage[wave], lane);
        }
    }
}

// Counting without a chain, in two launches.  count_kernel streams the mask: a wave takes a group of eight segments, a
// workgroup a block of kCountWaves groups, and leaves in seg_ptr the number of kept elements from the block's start to the
// end of each of its segments; the block's own total, in its last entry, is encoded as in the chain.  No workgroup waits for another.
// offsets_kernel adds what lies in front of each block: a workgroup sums the totals of all the blocks before its own (back to one
// that another workgroup has already replaced by the running total), so nothing waits there either.
// What bounds it: the mask read at HBM rate, and the flag words written beside it, an eighth of that: 550 MB of mask in one launch 101 us,
// 6.1 TB/s read and written, in the two that the binding makes of so many 54 and 49; a kernel that only reads them takes 82.  Blocks of 16 or 32 segments (two or four waves) count as fast
// but leave offsets_kernel two or four times the totals to sum (8.5 us instead of 6.5 with 32).
constexpr int kCountWaves = 8;
constexpr int kBlockSegs = kCountWaves * kSegsPerPass;
constexpr int kOffsetBlocks = 32;          // blocks of a workgroup of offsets_kernel
static_assert(kBlockSegs <= 64 && kOffsetBlocks <= 64, "a wave scans a block's segments, and a workgroup's blocks");
// LDS a counting workgroup asks for beside its own 8 KB, so that two and not four share a compute unit's 160 KB, and the number
// of workgroups from which on it does: a long launch reads faster with 16 waves in flight per compute unit, a short one is over sooner
// with all it can hold (us without and with, masks of 64 / 128 / 192 / 256 / 400 MB: 19.9 / 34.3 / 46.0 / 59.1 / 89.5 and
// 20.9 / 34.4 / 44.9 / 57.7 / 84.1).
constexpr int kCountLdsPad = 48000;
constexpr int64_t kCountPadFrom = 2048;

template <bool FLAGS>
__global__ void __launch_bounds__(kCountWaves * 64)
count_kernel(const IndexBatch batch)
{
    __shared__ __attribute__((aligned(16))) int32_t sh_stage[FLAGS ? kCountWaves : 1][kPairs * 64];
    __shared__ int sh_seg[kBlockSegs];
    const int job = find_job(batch, (int)blockIdx.x);
    const int64_t n = batch.n[job];
    const int64_t nseg = (n + kSeg - 1) / kSeg;
    const int64_t block = (int)blockIdx.x - batch.wg_start[job];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t group = block * kCountWaves + wave, seg0 = group * kSegsPerPass;
    if (seg0 < nseg) {
        uint32_t f[2 * kPairs], half[kPairs];
        const uint8_t *__restrict__ mask = batch.mask[job];
#pragma unroll
        for (int q = 0; q < 2 * kPairs; ++q) f[q] = lane_flags(mask, n, (seg0 + q) * kSeg + lane * 16);
#pragma unroll
        for (int j = 0; j < kPairs; ++j) {
            const int incl = wave_inclusive_scan(__popc(f[2 * j]) | (__popc(f[2 * j + 1]) << 16), lane);
            if (lane == 63) {                  // the last lane's inclusive prefixes are the segment totals
                sh_seg[wave * kSegsPerPass + 2 * j] = incl & 0xffff;
                sh_seg[wave * kSegsPerPass + 2 * j + 1] = incl >> 16;
            }
            half[j] = f[2 * j] | (f[2 * j + 1] << 16);
        }
        if (FLAGS) {
            uint32_t word[kPairs];
            pair_words(half, word, sh_stage[wave], lane);
            store_flags(batch.flags[job] + group * 64 + lane, word);
        }
    } else if (lane < kSegsPerPass) {
        sh_seg[wave * kSegsPerPass + lane] = 0;
    }
    __syncthreads();
    if (wave == 0) {
        const int incl = wave_inclusive_scan(lane < kBlockSegs ? sh_seg[lane] : 0, lane);
        const int64_t at = block * kBlockSegs + lane + 1, end = chain_slot(block, nseg, kBlockSegs);
        if (at <= end) batch.seg_ptr[job][at] = at == end ? encode_count(incl) : incl;
    }
}

// An entry that another workgroup may be replacing: a reader takes the old or the new value, whichever its caches hold.
__device__ __forceinline__ int either_load(const int32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
__device__ __forceinline__ void either_store(int32_t *p, int v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }

// The sum of the totals of the blocks in front of `block0` (all threads of the workgroup; every thread gets it).  A look takes
// kLooks entries per thread, the nearest first; entries that another workgroup replaces meanwhile read as either value.
__device__ __forceinline__ int kept_before(const int32_t *seg_ptr, int64_t nseg, int64_t block0, int *sh_nearest, int *sh_sum)
{
    constexpr int kLooks = 4;
    const int tid = threadIdx.x;
    int before = 0;
    for (int64_t back = block0 - 1; back >= 0; back -= kLooks * kThreads) {
        int v[kLooks];
#pragma unroll
        for (int k = 0; k < kLooks; ++k) {
            const int64_t b = back - (k * kThreads + tid);
            v[k] = b >= 0 ? either_load(seg_ptr + chain_slot(b, nseg, kBlockSegs)) : 0;      // in front of the first block: a total of 0
        }
        int nearest = kLooks * kThreads;
#pragma unroll
        for (int k = kLooks - 1; k >= 0; --k) {
            const unsigned long long totals = __ballot(v[k] >= 0);
            if (totals) nearest = k * kThreads + (tid & ~63) + __ffsll((long long)totals) - 1;
        }
        if ((tid & 63) == 0) sh_nearest[tid >> 6] = nearest;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) nearest = sh_nearest[w] < nearest ? sh_nearest[w] : nearest;
        int part = 0;
#pragma unroll
        for (int k = 0; k < kLooks; ++k) {
            const int i = k * kThreads + tid;
            part += i < nearest ? decode_count(v[k]) : i == nearest ? v[k] : 0;
        }
        part = wave_sum(part);
        if ((tid & 63) == 0) sh_sum[tid >> 6] = part;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) before += sh_sum[w];
        if (nearest < kLooks * kThreads) break;
    }
    return before;
}

__global__ void __launch_bounds__(kThreads)
offsets_kernel(const IndexBatch batch)
{
    __shared__ int sh_base[kOffsetBlocks], sh_nearest[kThreads / 64], sh_sum[kThreads / 64];
    const int job = find_job(batch, (int)blockIdx.x);
    const int64_t nseg = (batch.n[job] + kSeg - 1) / kSeg;
    const int64_t blocks = (nseg + kBlockSegs - 1) / kBlockSegs;
    const int wg = (int)blockIdx.x - batch.wg_start[job];
    const int64_t block0 = (int64_t)wg * kOffsetBlocks;
    int32_t *seg_ptr = batch.seg_ptr[job];
    const int tid = threadIdx.x;
    constexpr int kEach = kOffsetBlocks * kBlockSegs / kThreads;
    const int64_t first = block0 * kBlockSegs + 1;
    int in_block[kEach], own = 0;
#pragma unroll
    for (int i = 0; i < kEach; ++i) {
        const int64_t at = first + i * kThreads + tid;
        in_block[i] = at <= nseg ? seg_ptr[at] : 0;
    }
    if (tid < kOffsetBlocks && block0 + tid < blocks) own = decode_count(seg_ptr[chain_slot(block0 + tid, nseg, kBlockSegs)]);
    const int before = kept_before(seg_ptr, nseg, block0, sh_nearest, sh_sum);
    if (tid < 64) {
        const int incl = wave_inclusive_scan(own, tid);
        if (tid < kOffsetBlocks) sh_base[tid] = before + incl - own;
        if (tid == 0 && wg == 0) seg_ptr[0] = 0;
        if (tid == 63 && block0 + kOffsetBlocks >= blocks) {
            *batch.nnz[job] = (int64_t)before + incl;
            // past the caches: a host that polls it has the count before the launch has ended
            if (batch.mirror) __hip_atomic_store(batch.mirror + job, (int64_t)before + incl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kEach; ++i) {
        const int slot = i * kThreads + tid;
        const int64_t at = first + slot;
        if (at > nseg) continue;
        const bool end = slot % kBlockSegs == kBlockSegs - 1 || at == nseg;
        either_store(seg_ptr + at, sh_base[slot / kBlockSegs] + (end ? decode_count(in_block[i]) : in_block[i]));
    }
}


// The positions from the flag words and the seg_ptr a counting call left: a wave takes a group of eight
// segments (1 KiB of flag words in one load, where the mask is 8 KiB) and nothing waits for anything.
// A negative *nnz is no count: a build in one call leaves it, with a seg_ptr that is no table of offsets, where it gave up.  Nothing
// is stored then, and whatever seg_ptr holds no store leaves idx[0 .. cap) (storable).
// A lane holds 32 consecutive elements of each of the group's four pairs of segments.  Where a group keeps at most kStage
// elements its four pairs go through the loop over kept elements side by side (about 9 trips at 10 % kept, which share the
// loop's overhead, where one pair after the other took 8 each) and leave as one run; up to twice that, two pairs at a time.
// What bounds it: HBM, with the vector ALU close behind: 69 MB of flag words and 220 MB of idx in 56 us, 5.2 TB/s; 69 us with one
// pair at a time, 4-byte stores and idx through the caches.  A larger stage costs more in occupancy than it saves (58 us with 1280
// positions, 74 with 2048).
constexpr int kFillWaves = 4;
constexpr int kStage = kSeg;               // positions a wave collects before they leave

// Writes the positions of K pairs of segments that hold `total` <= kStage kept elements together.  word[k]: the lane's 32 elements
// of pair k; at[k]: how many of these pairs' kept elements come before them; base: the first pair's first element.
// The stage is shifted so that its 16-byte vectors are those of idx: whole ones leave as such, past the caches, and the
// ends, shared with the neighbouring runs, element by element.
template <int K>
__device__ __forceinline__ void emit_pairs(const uint32_t *word, const int *at, int total, int base, int64_t out0, int64_t cap,
                                           int32_t *__restrict__ idx, int32_t *stage, int lane)
{
    const int shift = (int)(out0 & 3);
    uint32_t bits[K];
    int to[K], first[K];
    uint32_t left = 0u;
    constexpr int kTrips = 2;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        bits[k] = word[k];
        to[k] = shift + at[k];
        first[k] = base + 2 * kSeg * k + 32 * lane;
        left |= bits[k];
    }
    while (__any(left != 0u)) {
        left = 0u;
#pragma unroll
        for (int k = 0; k < K; ++k) {
#pragma unroll
            for (int u = 0; u < kTrips; ++u) {
                if (bits[k] != 0u) stage[to[k] + u] = first[k] + __builtin_ctz(bits[k]);
                bits[k] &= bits[k] - 1u;
            }
            to[k] += kTrips;
            left |= bits[k];
        }
    }
    wave_lds_order();
    const int end = shift + storable(cap, out0, total);
    int32_t *__restrict__ out = idx + (out0 - shift);
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    for (int e = 4 * lane; e < end; e += 256) {
        const i32x4 q = *reinterpret_cast<const i32x4 *>(stage + e);
        if (e >= shift && e + 4 <= end) {
            __builtin_nontemporal_store(q, reinterpret_cast<i32x4 *>(out + e));
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (e + u >= shift && e + u < end) out[e + u] = q[u];
        }
    }
    wave_lds_order();
}

__global__ void __launch_bounds__(kFillWaves * 64)
fill_kernel(const IndexBatch batch)
{
    __shared__ __attribute__((aligned(16))) int32_t sh_stage[kFillWaves][kStage + 4];
    const int job = find_job(batch, (int)blockIdx.x);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t nseg = (batch.n[job] + kSeg - 1) / kSeg;
    const int64_t group = (int64_t)((int)blockIdx.x - batch.wg_start[job]) * kFillWaves + wave;
    const int64_t seg0 = group * kFlagGroupSegs;
    if (seg0 >= nseg) return;                 // whole waves leave; nothing below is a workgroup barrier
    // neither is written by this launch: scalar loads
    const int64_t counted = *(const __attribute__((address_space(4))) int64_t *)batch.nnz[job];
    const int64_t out0 = *(const __attribute__((address_space(4))) int32_t *)(batch.seg_ptr[job] + seg0);
    const uint4 w = batch.flags[job][group * 64 + lane];
    asm volatile("" ::"s"(counted), "s"(out0), "v"(w.x), "v"(w.y), "v"(w.z), "v"(w.w));       // one trip for the three, not one after the other
    if (counted < 0) return;
    const uint32_t word[kPairs] = {w.x, w.y, w.z, w.w};
    const int64_t cap = batch.cap[job];
    int32_t *__restrict__ idx = batch.idx[job];
    int32_t *stage = sh_stage[wave];
    const int base = (int)(seg0 * kSeg);
    int at[kPairs], total[kPairs];
#pragma unroll
    for (int j = 0; j < kPairs; j += 2) {     // a pair's count fits 16 bits
        const int c = __popc(word[j]) | (__popc(word[j + 1]) << 16);
        const int incl = wave_inclusive_scan(c, lane);
        const int all = __builtin_amdgcn_readlane(incl, 63);
        const int before = incl - c;
        at[j] = before & 0xffff;
        at[j + 1] = before >> 16;
        total[j] = all & 0xffff;
        total[j + 1] = all >> 16;
    }
    const int half = total[0] + total[1];
    // One pair alone, the end of a mask: three empty ones beside it would quadruple the trips' work (a mask of 1000 elements, count
    // and fill, 10 / 50 / 100 % kept: 10.3, 12.1 and 12.9 us with them, 9.6, 10.2 and 10.6 without).
    if (total[1] + total[2] + total[3] == 0 && half <= kStage) {
        emit_pairs<1>(word, at, half, base, out0, cap, idx, stage, lane);
        return;
    }
    if (half + total[2] + total[3] <= kStage) {
        at[1] += total[0];
        at[2] += half;
        at[3] += half + total[2];
        emit_pairs<4>(word, at, half + total[2] + total[3], base, out0, cap, idx, stage, lane);
        return;
    }
    if (half <= kStage && total[2] + total[3] <= kStage) {
        at[1] += total[0];
        at[3] += total[2];
        emit_pairs<2>(word, at, half, base, out0, cap, idx, stage, lane);
        emit_pairs<2>(word + 2, at + 2, total[2] + total[3], base + 4 * kSeg, out0 + half, cap, idx, stage, lane);
        return;
    }
    uint32_t halves[kPairs];
    word_halves(word, halves, stage, lane);
    int64_t out = out0;
#pragma unroll
    for (int j = 0; j < kPairs; ++j) {
        emit_pair(word[j], halves[j], base + 2 * kSeg * j, out, cap, idx, stage, lane);
        out += total[j];
    }
}

__global__ void __launch_bounds__(kThreads)
seg_ptr_from_idx_kernel(const int32_t *__restrict__ idx, int64_t nnz, int64_t nseg, int32_t *__restrict__ seg_ptr)
{
    const int64_t s = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (s > nseg) return;
    const int64_t key = s * kSeg;          // first i with idx[i] >= key
    int64_t lo = 0, hi = nnz;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)idx[mid] < key) lo = mid + 1; else hi = mid;
    }
    seg_ptr[s] = (int32_t)lo;
}

__global__ void set_flag_kernel(int32_t *flag, int32_t value) { *flag = value; }

__global__ void __launch_bounds__(kThreads)
validate_kernel(const int32_t *__restrict__ idx, int64_t nnz, int64_t n, int64_t nseg,
                const int32_t *__restrict__ seg_ptr, int32_t *__restrict__ ok)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    bool bad = false;
    if (i < nnz) {
        const int64_t j = idx[i];
        if (j < 0 || j >= n) bad = true;
        else if (i > 0 && (int64_t)idx[i - 1] >= j) bad = true;
        else if (seg_ptr) {
            const int64_t s = j / kSeg;
            if (!((int64_t)seg_ptr[s] <= i && i < (int64_t)seg_ptr[s + 1])) bad = true;
        }
    }
    if (seg_ptr && i <= nseg) {
        if (i == 0 && seg_ptr[0] != 0) bad = true;
        if (i == nseg && (int64_t)seg_ptr[nseg] != nnz) bad = true;
        if (i < nseg && seg_ptr[i] > seg_ptr[i + 1]) bad = true;
    }
    if (bad) *ok = 0;
}

}  // namespace

hipError_t launch_index_batch(const IndexBatch &batch, hipStream_t s)
{
    if (batch.num <= 0) return hipSuccess;
    const int wgs = batch.wg_start[batch.num];
    const int init_threads = wgs > batch.num ? wgs : batch.num;
    index_init_kernel<<<dim3((unsigned)ceil_div(init_threads, kThreads)), dim3(kThreads), 0, s>>>(batch);
    if (wgs > 0) {
        const dim3 grid((unsigned)wgs), block(kIndexThreads);
        if (batch.passes == 4) index_kernel<4><<<grid, block, 0, s>>>(batch);
        else if (batch.passes == 2) index_kernel<2><<<grid, block, 0, s>>>(batch);
        else index_kernel<1><<<grid, block, 0, s>>>(batch);
    }
    return hipGetLastError();
}

hipError_t launch_index_count(IndexBatch &batch, bool flags, hipStream_t s)
{
    if (batch.num <= 0) return hipSuccess;
    int64_t wgs = 0;
    for (int j = 0; j < batch.num; ++j) {
        batch.wg_start[j] = (int)wgs;
        wgs += ceil_div(ceil_div(batch.n[j], kSeg), kBlockSegs);
    }
    batch.wg_start[batch.num] = (int)wgs;
    if (wgs > 0) {
        const dim3 grid((unsigned)wgs), block(kCountWaves * 64);
        const int pad = wgs >= kCountPadFrom ? kCountLdsPad : 0;
        if (flags) count_kernel<true><<<grid, block, pad, s>>>(batch);
        else count_kernel<false><<<grid, block, pad, s>>>(batch);
    }
    wgs = 0;
    for (int j = 0; j < batch.num; ++j) {
        batch.wg_start[j] = (int)wgs;
        const int64_t w = ceil_div(ceil_div(batch.n[j], kSeg), kBlockSegs * kOffsetBlocks);
        wgs += w > 0 ? w : 1;                 // an empty job has a seg_ptr and a count as well
    }
    batch.wg_start[batch.num] = (int)wgs;
    offsets_kernel<<<dim3((unsigned)wgs), dim3(kThreads), 0, s>>>(batch);
    return hipGetLastError();
}

hipError_t launch_index_fill(const IndexBatch &batch, hipStream_t s)
{
    const int wgs = batch.num > 0 ? batch.wg_start[batch.num] : 0;
    if (wgs > 0) fill_kernel<<<dim3((unsigned)wgs), dim3(kFillWaves * 64), 0, s>>>(batch);
    return hipGetLastError();
}

int64_t index_fill_workgroups(int64_t n) { return ceil_div(ceil_div(n, kSeg), kFlagGroupSegs * kFillWaves); }

int64_t index_job_workgroups(int64_t n, int passes) { return ceil_div(ceil_div(n, kSeg), segs_per_wg(passes)); }

// Passes per workgroup for a chained launch over `mask_bytes` bytes of mask: the most for which the launch still has a dozen
// blocks per compute unit.  With 1, 2 and 4 passes, 10 % kept, us: 7 layers of the 2.7B shape (550 MB of mask: 33, 16
// and 8 blocks per compute unit) 174, 160, 163; 32 layers 794, 753, 751.
int index_passes_for(int64_t mask_bytes, int compute_units)
{
    const int64_t wanted = (int64_t)compute_units * 12;
    for (int passes = kMaxPasses; passes > 1; passes /= 2)
        if (mask_bytes / ((int64_t)segs_per_wg(passes) * kSeg) >= wanted) return passes;
    return 1;
}

hipError_t launch_seg_ptr_from_idx(const int32_t *idx, int64_t nnz, int64_t n, int32_t *seg_ptr, hipStream_t s)
{
    const int64_t nseg = ceil_div(n, kSeg);
    seg_ptr_from_idx_kernel<<<dim3((unsigned)ceil_div(nseg + 1, kThreads)), dim3(kThreads), 0, s>>>(idx, nnz, nseg,
                                                                                                   seg_ptr);
    return hipGetLastError();
}

hipError_t launch_validate(const int32_t *idx, int64_t nnz, int64_t n, const int32_t *seg_ptr, int32_t *ok,
                           hipStream_t s)
{
    const int64_t nseg = ceil_div(n, kSeg);
    set_flag_kernel<<<dim3(1), dim3(1), 0, s>>>(ok, 1);
    const int64_t work = nnz > nseg + 1 ? nnz : nseg + 1;
    validate_kernel<<<dim3((unsigned)ceil_div(work, kThreads)), dim3(kThreads), 0, s>>>(idx, nnz, n, nseg, seg_ptr,
                                                                                       ok);
    return hipGetLastError();
}

}  // namespace samo
