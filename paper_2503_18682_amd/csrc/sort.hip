// Binning: device-wide exclusive scan, instance emission, a stable LSD radix
// sort of (key, value) pairs and the per-tile ranges of the sorted instances.
//
// Ordering strategy.  The per-pixel order is ascending (depth, Gaussian id)
// (eq. 1 of the paper orders primitives by the depth of their centres; ties
// are broken by id).  Instead of sorting one 64-bit (tile | depth) key per
// Gaussian-tile instance, the Gaussian-views are sorted once by their 32-bit
// depth key (stable, so equal depths keep id order), instances are emitted in
// that order, and a stable radix sort on the tile id alone (13-20 bits) groups
// them by tile without disturbing the depth order inside a tile.
#include <algorithm>

#include "internal.h"

namespace rgs {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
// Binning scan: items per thread (4 or 8) chosen from the item count, as for
// the radix passes below.
constexpr int kScanItemsMin = 4;
constexpr int scan_tile(int items) { return kThreads * items; }
constexpr int kScanSelfPrefixBlocks = 1024;
// Radix sort: digits of up to 11 bits, so that a 32-bit key takes 3 passes and a tile id one or two.
constexpr int kMaxDigitBits = 11;
constexpr int kMaxBins = 1 << kMaxDigitBits;
constexpr int kHistWordsLog = 12;  // counters of a histogram block (all copies of all bins)
constexpr int kHistWords = 1 << kHistWordsLog;
constexpr int kEmitThreads = 512;  // 8 waves (emit_plan)
constexpr int kLargeTile = 4096;   // items of a block of a large sort: its workgroups take several blocks

// Element count of a device-sized array: a frame whose instance count
// overflowed the capacity is treated as empty downstream (its status reports
// the overflow), so no kernel ever reads entries that were not written.
__device__ __forceinline__ int64_t clamp_count(const int64_t *n_dev, int64_t n_max)
{
    if (!n_dev) return n_max;
    const int64_t n = *n_dev;
    return n <= n_max ? n : 0;
}

// Emission plan: the tile rows of all binning boxes, in depth order, are dealt
// to blocks of 8 waves (the blocks of the tile sort's first pass) in runs of
// `rows` rows, about a tile of box instances (a block may have any number).
// The runs are as long as needed for no more blocks than the sort has.  A wave
// takes `step` rows of its block at a time, one per lane.
struct EmitPlan {
    int64_t total, rows_all;  // box instances (0 when they exceed the capacity) and tile rows
    int blocks, rows, step;   // rows = 8 step with step 8, 16 or 32 (wide rows), or a multiple of 512 with step 64
};

__device__ __forceinline__ EmitPlan emit_plan(const int64_t *counters, int64_t capacity, int tile_shift)
{
    EmitPlan P;
    P.total = clamp_count(counters, capacity);
    P.rows_all = P.total ? counters[2] : 0;
    const int64_t most = ((capacity - 1) >> tile_shift) + 1;
    // rows of a tile of box instances (in single precision: any choice is valid)
    const float fit = (float)P.rows_all / (float)max(P.total, (int64_t)1) * (float)(1 << tile_shift);
    int rows = 64;
    while (rows < 512 && ((float)(2 * rows) <= fit || most * rows < P.rows_all)) rows *= 2;
    if (rows == 512) {
        rows = 512 * max(1, (int)(fit * (1.0f / 512.0f)));
        while (most * rows < P.rows_all) rows += 512;
    }
    P.rows = rows;
    P.step = min(rows / 8, 64);
    P.blocks = (int)((P.rows_all + rows - 1) / rows);
    return P;
}

// Orders the LDS accesses of a wave's lanes (which run in step).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Inclusive scan across a wave (all lanes active): row shifts inside the
// 16-lane rows, then each row's last lane broadcast to the rows behind it.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x)
{
#define RGS_DPP(CTRL, ROWS) (uint32_t) __builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false)
    x += RGS_DPP(0x111, 0xf);  // row_shr:1, 2, 4, 8
    x += RGS_DPP(0x112, 0xf);
    x += RGS_DPP(0x114, 0xf);
    x += RGS_DPP(0x118, 0xf);
    x += RGS_DPP(0x142, 0xa);  // row_bcast:15 into rows 1 and 3
    x += RGS_DPP(0x143, 0xc);  // row_bcast:31 into rows 2 and 3
#undef RGS_DPP
    return x;
}

// Inclusive scan across a block of WAVES waves; returns the inclusive
// prefix and writes the block total to *total.
template <int WAVES>
__device__ __forceinline__ uint32_t block_inclusive_scan(uint32_t x, uint32_t *smem /*[WAVES]*/, uint32_t *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t v = wave_inclusive_scan(x);
    if (lane == 63) smem[wave] = v;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const uint32_t t = smem[w];
        if (w < wave) before += t;
        all += t;
    }
    __syncthreads();
    *total = all;
    return before + v;
}

// ---------------------------------------------------------------- radix sort
// Digit of one pass: `bits` sorted bits of key - base, spread evenly over the
// passes.  With kmax (the largest key, on the device, known after the first
// pass's histogram) the first pass takes kFirstBits bits and the other two share what
// is left of the bits that key - base can have.
struct RadixPass {
    const uint32_t *kmax;  // device, may be null: then `bits` bits are sorted
    uint32_t base;
    int bits, pass, passes;
};
constexpr int kFirstBits = 9;

struct Digit {
    uint32_t base, mask;
    int shift, bits;
    __device__ __forceinline__ uint32_t of(uint32_t key) const { return ((key - base) >> shift) & mask; }
};

__device__ __forceinline__ Digit pass_digit(const RadixPass &P)
{
    int shift = 0, bits = 0, total = P.bits, p = 0;
    if (P.kmax) {
        bits = kFirstBits;
        p = 1;
        if (P.pass > 0) {
            const uint32_t top = *P.kmax;
            total = top > P.base ? 32 - __builtin_clz(top - P.base) : 0;
            total = max(total, kFirstBits);
        }
    }
    for (; p <= P.pass; ++p) {
        shift += bits;
        bits = (total - shift + (P.passes - p) - 1) / (P.passes - p);
    }
    return Digit{P.base, (1u << bits) - 1u, shift, bits};
}

// Block of items of this workgroup, of nb: workgroups are dealt to the 8 XCDs
// in turn, and each XCD takes runs of neighbouring blocks.  The blocks in
// flight on one XCD then write next to each other in every digit's range, and
// their short runs merge into whole lines in that XCD's L2 (blocks dealt in
// order leave every line shared by several XCDs, each writing its part to
// memory).  At least 8 runs per XCD even out blocks of different work: the first in
// depth order have the widest tile rows.  Returns nb or more when there is none.
// A launch of a large sort has at most kMaxGrid workgroups, a multiple of 8, and each takes every grid-th place
// `at`: blocks are as many as the capacity can need, and a workgroup that finds none costs as much as the wait for
// the count.  20000 Gaussians at 640x480 in a workspace for 80M instances took 269 us with a workgroup for each
// possible block and take 174 us; full sorts lose up to 1 % (with 3072 workgroups 167 us, and 3 %).  The emission's
// blocks are of unequal work, and rounds of them even out worse: twice as many workgroups.
__device__ __forceinline__ int xcd_run(int nb)  // log2 of the run: nb / 64, up to 64
{
    return nb >= 4096 ? 6 : nb >= 64 ? 25 - __builtin_clz((unsigned)nb) : 0;
}

__device__ __forceinline__ int xcd_block(int nb, int at)
{
    const int lrun = xcd_run(nb), k = at >> 3, xcd = at & 7;
    return ((((k >> lrun) << 3) + xcd) << lrun) + (k & ((1 << lrun) - 1));
}

// Places that hold the nb blocks (the last round of runs may be partly empty).
__device__ __forceinline__ int xcd_places(int nb)
{
    const int round = 8 << xcd_run(nb);
    return (nb + round - 1) & -round;
}

// Entries of a block's histogram row in the block-major layout: 16-bit counts
// (a block has fewer items than that), whole uint4 of them.
__device__ __forceinline__ int hist_row(int bins) { return max(bins, 8); }

// Writes digit d's count of a block's histogram.
template <bool SELF>
__device__ __forceinline__ void put_count(uint32_t *hist, int bins, int nblocks, int block, int d, uint32_t count)
{
    if (SELF)
        reinterpret_cast<uint16_t *>(hist)[(size_t)block * hist_row(bins) + d] = (uint16_t)count;
    else
        hist[(size_t)d * nblocks + block] = count;
}

// Digit histogram of one block's items; with `drop`, keys equal to drop_key
// are left out (they leave the sort in this pass).  Blocks past the
// device-side count write nothing.  All keys of a thread are loaded before the
// first is counted.  Up to 8 interleaved copies of each counter (by lane)
// keep equal digits of a wave off one LDS address.
template <int THREADS, int ITEMS, bool SELF>
__global__ __launch_bounds__(THREADS) void k_radix_hist(const uint32_t *__restrict__ keys, int64_t n_max,
                                                        const int64_t *__restrict__ n_dev, RadixPass pass, bool drop,
                                                        uint32_t drop_key, uint32_t *__restrict__ hist, int nblocks,
                                                        int grid, const uint32_t *__restrict__ part_max, int n_parts,
                                                        uint32_t *__restrict__ kmax_out)
{
    constexpr int TILE = THREADS * ITEMS;
    __shared__ uint32_t cnt[kHistWords];
    const int tid = threadIdx.x;
    if (kmax_out && blockIdx.x == gridDim.x - 1) {  // the extra workgroup: largest key
        uint32_t top = 0u;
        constexpr int kStep = 16;
        for (int i = tid; i < n_parts; i += THREADS * kStep) {
            uint32_t x[kStep];
#pragma unroll
            for (int j = 0; j < kStep; ++j) x[j] = part_max[min(i + j * THREADS, n_parts - 1)];
#pragma unroll
            for (int j = 0; j < kStep; ++j) top = max(top, x[j]);
        }
        if (tid == 0) cnt[0] = 0u;
        __syncthreads();
        atomicMax(&cnt[0], top);
        __syncthreads();
        if (tid == 0) *kmax_out = cnt[0];
        return;
    }
    uint32_t key[ITEMS];
    auto load = [&](int64_t base, int left) {
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) key[j] = (keys + base)[(uint32_t)min(j * THREADS + tid, left - 1)];
    };
    if constexpr (SELF) {  // loads by the launch's bounds do not wait for the count
        const int64_t base = (int64_t)blockIdx.x * TILE;
        if (base >= n_max) return;
        load(base, (int)min(n_max - base, (int64_t)TILE));
    }
    const int64_t n = clamp_count(n_dev, n_max);
    constexpr bool ROUNDS = TILE == kLargeTile;
    const int nb = (int)((n + TILE - 1) / TILE), end = SELF ? nb : xcd_places(nb);
    for (int at = (int)blockIdx.x; at < end; at += grid) {
        const int block = SELF ? at : xcd_block(nb, at);
        if (block >= nb) {  // uniform per block
            if constexpr (!ROUNDS) return;
            continue;
        }
        const int64_t base = (int64_t)block * TILE;
        const int left = (int)min(n - base, (int64_t)TILE);
        if constexpr (!SELF) load(base, left);
        const Digit D = pass_digit(pass);
        const int bins = 1 << D.bits;
        const int cshift = min(3, kHistWordsLog - D.bits);  // log2 of the copies
        for (int i = tid; i < bins << cshift; i += THREADS) cnt[i] = 0u;
        __syncthreads();
        const uint32_t copy = tid & ((1u << cshift) - 1u);
#pragma unroll
        for (int j = 0; j < ITEMS; ++j)
            if (j * THREADS + tid < left && !(drop && key[j] == drop_key))
                atomicAdd(&cnt[(D.of(key[j]) << cshift) + copy], 1u);
        __syncthreads();
        const int row = SELF ? hist_row(bins) : bins;
        for (int d = tid; d < row; d += THREADS) {
            uint32_t x = 0;
            if (d < bins)
                for (int c = 0; c < 1 << cshift; ++c) x += cnt[(d << cshift) + c];
            put_count<SELF>(hist, bins, nblocks, block, d, x);
        }
        if constexpr (!ROUNDS) return;
        __syncthreads();
    }
}

// Exclusive scan of each digit's row hist[d][0..nb) (one block per digit)
// over the nb = ceil(n / tile) blocks that hold items (tile = keys per block),
// or over the emission's blocks.
__global__ __launch_bounds__(kThreads) void k_radix_scan_rows(uint32_t *__restrict__ hist, int nblocks,
                                                              int64_t n_max, const int64_t *__restrict__ n_dev,
                                                              RadixPass pass, int tile, bool segments,
                                                              uint32_t *__restrict__ row_total)
{
    __shared__ uint32_t smem[kWaves];
    if (blockIdx.x >> pass_digit(pass).bits) return;  // no such digit in this pass
    const int64_t n = clamp_count(n_dev, n_max);
    const int nb = segments ? emit_plan(n_dev, n_max, __builtin_ctz((unsigned)tile)).blocks
                            : (int)std::min<int64_t>((n + tile - 1) / tile, nblocks);
    uint32_t *row = hist + (size_t)blockIdx.x * nblocks;
    constexpr int kPer = 8;  // entries per thread and step: a contiguous run, scanned in registers
    uint32_t carry = 0;
    for (int base = 0; base < nb; base += kThreads * kPer) {
        uint32_t x[kPer], sum = 0;
        const int i0 = base + threadIdx.x * kPer;
#pragma unroll
        for (int j = 0; j < kPer; ++j) x[j] = i0 + j < nb ? row[i0 + j] : 0u;
#pragma unroll
        for (int j = 0; j < kPer; ++j) sum += x[j];
        uint32_t tot;
        uint32_t run = carry + block_inclusive_scan<kWaves>(sum, smem, &tot) - sum;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            if (i0 + j < nb) row[i0 + j] = run;
            run += x[j];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) row_total[blockIdx.x] = carry;
}

// Stable scatter of one block's items by digit.  A thread's keys and values
// are all loaded first, with no branch around the loads, so that a wave waits
// for memory once and not once per round; the digits' output positions are
// summed up while they are in flight.  Each wave then ranks ITEMS rounds of 64
// consecutive items: lanes holding the same digit are found with one ballot
// per digit bit, ranked by popcount of the lower peers, and a per-wave LDS
// counter per digit carries the rank across rounds.  Items are staged in
// LDS in block-local sorted order and written out in runs of equal digits.
// With `drop`, keys equal to drop_key are not written; the first block
// stores the number of items kept (the sum of the digit totals) in *kept_out (may be null).
// SELF: hist is block-major and unscanned (rows of hist_row(bins) entries); each
// block sums the rows before its own (and all of them for the digit bases)
// itself, so the pass needs no scan launch.  Otherwise hist is digit-major and
// scanned, with row_total.
// With `ranges` (SEG, a sort of one pass) the digits are the tiles, and the first block
// writes the range of each one that has items: no k_tile_ranges launch (4 us).
// SEG: the items are the emission's: those of block b are the
// seg[b].y from seg[b].x on, any number of them, taken a tile at a time; the
// number of items sorted goes to *kept_out.  Where a window of 16 blocks is less than half
// full, neighbouring blocks whose items fit one tile are taken by one workgroup: a 5120x3840
// frame of needles lists a tenth of its box instances, and its pass took 286 us
// with a workgroup for each block and takes 210 us; a frame that lists three quarters
// would lose (59 -> 63 us).
template <int THREADS, int ITEMS, bool SELF, bool SEG>
__global__ __launch_bounds__(THREADS, SELF || SEG ? 4 : 6) void k_radix_scatter(
    const uint32_t *__restrict__ keys_in, const uint32_t *__restrict__ vals_in, uint32_t *__restrict__ keys_out,
    uint32_t *__restrict__ vals_out, int64_t n_max, const int64_t *__restrict__ n_dev, RadixPass pass, bool drop,
    uint32_t drop_key, int64_t *__restrict__ kept_out, const uint32_t *__restrict__ hist,
    const uint32_t *__restrict__ row_total, int nblocks, const uint2 *__restrict__ seg, uint2 *__restrict__ ranges)
{
    constexpr int TILE = THREADS * ITEMS, WAVES = THREADS / 64;
    constexpr int kCntWords = WAVES * kMaxBins / 2, kSumWords = SELF ? 16 * THREADS : 0;
    constexpr int kMemA = 2 * TILE > kCntWords ? 2 * TILE : kCntWords;
    // partial sums of the histogram, per-wave digit counters (16 bits each) and
    // staged items take turns
    __shared__ uint4 s_mem4[(kMemA > kSumWords ? kMemA : kSumWords) / 4];
    __shared__ uint32_t s_base[kMaxBins];   // digit: output position of its first item, later minus s_start
    __shared__ uint16_t s_start[kMaxBins];  // digit: block-local position of its first item
    __shared__ uint32_t smem[WAVES];
    uint32_t *const s_mem = reinterpret_cast<uint32_t *>(s_mem4);
    uint16_t *const wave_cnt = reinterpret_cast<uint16_t *>(s_mem);
    uint32_t *const s_keys = s_mem, *const s_vals = s_mem + TILE;

    int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, at0 = wave * (TILE / WAVES) + lane;
    uint32_t key[ITEMS], val[ITEMS];
    auto load = [&](int64_t base, int left) {
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) key[r] = (keys_in + base)[(uint32_t)min(at0 + r * 64, max(left - 1, 0))];
        if (vals_in) {
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) val[r] = (vals_in + base)[(uint32_t)min(at0 + r * 64, max(left - 1, 0))];
        } else {
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) val[r] = (uint32_t)(base + at0 + r * 64);
        }
    };
    // small sorts load at once, by the launch's bounds; large ones know their block first
    constexpr bool kEarly = SELF && !SEG;
    if constexpr (kEarly) {
        const int64_t base = (int64_t)blockIdx.x * TILE;
        if (base >= n_max) return;
        load(base, (int)min(n_max - base, (int64_t)TILE));
    }
    const int64_t n = clamp_count(n_dev, n_max);
    const Digit D = pass_digit(pass);
    const int nb = SEG ? emit_plan(n_dev, n_max, __builtin_ctz(TILE)).blocks : (int)((n + TILE - 1) / TILE);
    if (kept_out && nb == 0 && blockIdx.x == 0 && tid == 0) *kept_out = 0;
    constexpr bool ROUNDS = TILE == kLargeTile;
    const int end = SELF ? nb : xcd_places(nb);
    for (int place = (int)blockIdx.x; place < end; place += (int)gridDim.x) {
        if constexpr (ROUNDS) {  // (nothing of one round is kept in registers for the next)
            asm volatile("" : "+v"(tid));
            lane = tid & 63, wave = tid >> 6, at0 = wave * (TILE / WAVES) + lane;
        }
        int block = SELF ? place : xcd_block(nb, place);
        if (block >= nb) {  // uniform per block
            if constexpr (!ROUNDS) return;
            continue;
        }
        int64_t base = (int64_t)block * TILE;
        int todo = (int)min(n - base, (int64_t)TILE);  // items of the block
        // (SEG) the workgroup's segments, from `block` on, `segs` of them: lane s
        // holds segment s of the window of kWindow that `block` lies in
        constexpr int kWindow = 16;
        uint2 part = make_uint2(0u, 0u);
        int seg0 = 0, segs = 1;
        if constexpr (SEG) {
            const int first = block & ~(kWindow - 1), here = min(nb - first, kWindow);
            if (lane < here) part = seg[first + lane];
            seg0 = block - first;
            todo = (int)__builtin_amdgcn_readlane(part.y, seg0);
            const int all = (int)__builtin_amdgcn_readlane(wave_inclusive_scan(part.y), kWindow - 1);
            if (2 * (int64_t)all <= (int64_t)here * TILE) {
                int group = -1, held = 0;
                const int want = seg0;
                segs = todo = 0;
                for (int s = 0; s < here; ++s) {
                    const int c = (int)__builtin_amdgcn_readlane(part.y, s);
                    if (s == 0 || held + c > TILE) {
                        ++group;
                        held = 0;
                    }
                    held += c;
                    if (group == want) {
                        if (segs == 0) seg0 = s;
                        ++segs;
                        todo = held;
                    }
                }
                if (segs == 0) {  // uniform per block
                    if constexpr (!ROUNDS) return;
                    continue;
                }
                block = first + seg0;
            }
            base = (int64_t)(uint32_t)__builtin_amdgcn_readlane(part.x, seg0);
        }
        // items [from, from + TILE) of the workgroup's
        auto load_items = [&](int from) {
            const int left = min(todo - from, TILE);
            if (!SEG || segs == 1) {
                load(base + from, left);
                return;
            }
            uint32_t src[ITEMS];
            uint32_t start = 0;  // items before the segment
            for (int s = seg0; s < seg0 + segs; ++s) {
                const uint32_t delta = (uint32_t)__builtin_amdgcn_readlane(part.x, s) - start;
#pragma unroll
                for (int r = 0; r < ITEMS; ++r) {
                    const uint32_t i = (uint32_t)(from + min(at0 + r * 64, max(left - 1, 0)));
                    if (s == seg0 || i >= start) src[r] = i + delta;
                }
                start += (uint32_t)__builtin_amdgcn_readlane(part.y, s);
            }
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) key[r] = keys_in[src[r]];
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) val[r] = vals_in[src[r]];
        };
        int from = 0;
        if constexpr (!kEarly) load_items(0);
        const int bins = 1 << D.bits;

        // output position of each digit's first item of this block
        if constexpr (SELF) {
            // each thread sums eight neighbouring digits over every groups-th row
            const int row = hist_row(bins), octs = row >> 3;
            const int oct = tid & (octs - 1), group = tid / octs, groups = THREADS / octs;
            uint32_t all[8] = {}, pre[8] = {};
            constexpr int kStep = 8;
            const uint4 *src = reinterpret_cast<const uint4 *>(hist) + oct;
            for (int r0 = group; r0 < nb; r0 += groups * kStep) {
                uint4 x[kStep];
#pragma unroll
                for (int j = 0; j < kStep; ++j) x[j] = src[(size_t)(min(r0 + j * groups, nb - 1) * octs)];
#pragma unroll
                for (int j = 0; j < kStep; ++j) {
                    const int r = r0 + j * groups;
                    const uint32_t in = r < nb ? ~0u : 0u, before = r < block ? ~0u : 0u;
                    const uint32_t w[4] = {x[j].x & in, x[j].y & in, x[j].z & in, x[j].w & in};
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t lo = w[q] & 0xffffu, hi = w[q] >> 16;
                        all[2 * q] += lo;
                        all[2 * q + 1] += hi;
                        pre[2 * q] += lo & before;
                        pre[2 * q + 1] += hi & before;
                    }
                }
            }
            // partial sums [group][digit], all of them and then those before the block
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                s_mem4[2 * tid + q] = make_uint4(all[4 * q], all[4 * q + 1], all[4 * q + 2], all[4 * q + 3]);
                s_mem4[2 * THREADS + 2 * tid + q] = make_uint4(pre[4 * q], pre[4 * q + 1], pre[4 * q + 2], pre[4 * q + 3]);
            }
            __syncthreads();
        }
        uint32_t dig_carry = 0;
#pragma unroll 1
        for (int d0 = 0; d0 < bins; d0 += THREADS) {
            const int d = d0 + tid;
            uint32_t pre = 0, all = 0;
            if (d < bins) {
                if constexpr (SELF) {
                    const int row = hist_row(bins), groups = 8 * THREADS / row;
                    for (int g = 0; g < groups; ++g) {
                        all += s_mem[g * row + d];
                        pre += s_mem[8 * THREADS + g * row + d];
                    }
                } else {
                    all = row_total[d];
                    pre = hist[(size_t)d * nblocks + block];
                }
            }
            uint32_t dig_tot;
            const uint32_t dig_base = dig_carry + block_inclusive_scan<WAVES>(all, smem, &dig_tot) - all;
            dig_carry += dig_tot;
            if (d < bins) s_base[d] = dig_base + pre;
            if (SEG && ranges && block == 0 && d < bins && all != 0u) ranges[d] = make_uint2(dig_base, dig_base + all);
        }
        if (kept_out && block == 0 && tid == 0) *kept_out = (int64_t)dig_carry;
        const uint32_t n32 = (uint32_t)n;
        for (;;) {
            const int left = min(todo - from, TILE);
            __syncthreads();
            for (int i = tid; i < WAVES * bins / 2; i += THREADS) s_mem[i] = 0u;
            __syncthreads();

            // position of each item among the items of its digit in its wave
            uint16_t *const cnt = wave_cnt + wave * bins;
            uint32_t rank[ITEMS];
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) {
                const bool valid = at0 + r * 64 < left && !(drop && key[r] == drop_key);
                const uint32_t d = D.of(key[r]);
                const uint64_t some = __ballot(valid);
                uint32_t lo = (uint32_t)some, hi = (uint32_t)(some >> 32);  // lanes of the same digit
                for (int b = 0; b < D.bits; ++b) {
                    const int32_t bit = (int32_t)(d << (31 - b)) >> 31;  // 0 or all ones
                    const uint64_t m = __ballot(bit != 0);
                    lo &= ~((uint32_t)m ^ (uint32_t)bit);
                    hi &= ~((uint32_t)(m >> 32) ^ (uint32_t)bit);
                }
                const uint32_t below = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
                const uint32_t prior = cnt[d];
                wave_sync();
                if (valid && below == 0) cnt[d] = (uint16_t)(prior + (uint32_t)(__popc(lo) + __popc(hi)));
                wave_sync();
                rank[r] = valid ? prior + below : 0xffffffffu;
            }
            __syncthreads();

            // per digit: prefix over the waves, block-local start
            uint32_t carry = 0;
#pragma unroll 1
            for (int d0 = 0; d0 < bins; d0 += THREADS) {
                const int d = d0 + tid;
                uint32_t run = 0;
                if (d < bins)
#pragma unroll
                    for (int w = 0; w < WAVES; ++w) {
                        const uint32_t c = wave_cnt[w * bins + d];
                        wave_cnt[w * bins + d] = (uint16_t)run;
                        run += c;
                    }
                uint32_t tot;
                const uint32_t start = carry + block_inclusive_scan<WAVES>(run, smem, &tot) - run;
                carry += tot;
                if (d < bins) {
                    s_start[d] = (uint16_t)start;
                    s_base[d] -= start;
                }
            }
            const int count = (int)carry;  // items of this tile that stay in the sort
            __syncthreads();
#pragma unroll
            for (int r = 0; r < ITEMS; ++r)
                if (rank[r] != 0xffffffffu) {
                    const uint32_t d = D.of(key[r]);
                    rank[r] += (uint32_t)s_start[d] + cnt[d];
                }
            __syncthreads();  // the counters give way to the staged items
#pragma unroll
            for (int r = 0; r < ITEMS; ++r)
                if (rank[r] != 0xffffffffu) {
                    s_keys[rank[r]] = key[r];
                    s_vals[rank[r]] = val[r];
                }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) {
                const int p = r * THREADS + tid;
                if (p < count) {
                    const uint32_t k = s_keys[p];
                    const uint32_t dst = s_base[D.of(k)] + (uint32_t)p;
                    if (dst < n32) {
                        keys_out[dst] = k;
                        vals_out[dst] = s_vals[p];
                    }
                }
            }
            from += TILE;
            if (!SEG || from >= todo) break;  // uniform per block
            load_items(from);
            // the digits' next positions: past this tile's items
            __syncthreads();
            for (int d = tid; d < bins; d += THREADS)
                s_base[d] += d + 1 < bins ? (uint32_t)s_start[d + 1] : (uint32_t)count;
        }
        if constexpr (!ROUNDS) return;
        __syncthreads();
    }
}

// ---------------------------------------------------------------------- scan
// Binning scan over the depth-sorted Gaussian-views: each item carries two
// counts, the tiles of its binning box (instances) and the tile rows of that
// box; both are scanned at once (block sums hold the pair as two uint64).
// A culled view (sorted key 0xffffffff, all at the end) counts nothing and
// costs no gather; a kept one reads its box.
__device__ __forceinline__ void scan_item(const uint32_t *__restrict__ keys, const uint2 *__restrict__ boxes,
                                          const uint32_t *__restrict__ order, int64_t idx, int TW, int TH,
                                          uint32_t &tiles, uint32_t &rows, uint2 &box)
{
    tiles = rows = 0u;
    box = make_uint2(0u, 0u);
    if (keys[idx] != 0xffffffffu) {
        box = boxes[order[idx]];
        const PixelBox pb = unpack_box(box);
        rows = (uint32_t)(pb.y1 / TH - pb.y0 / TH + 1);
        tiles = rows * (uint32_t)(pb.x1 / TW - pb.x0 / TW + 1);
    }
}

// Gathers each sorted item's two counts once (the tiles into `tiles`, read back
// by k_scan_apply, which scans them in place) and reduces them per block.
// The gathered binning box is also stored in depth order (`sorted_boxes`), so
// the emission kernel reads it coalesced instead of gathering it again.
template <int ITEMS>
__global__ __launch_bounds__(kThreads) void k_scan_reduce(const uint32_t *__restrict__ keys,
                                                          const uint2 *__restrict__ boxes,
                                                          const uint32_t *__restrict__ order, int64_t n_max,
                                                          const int64_t *__restrict__ n_dev, int TW, int TH,
                                                          uint32_t *__restrict__ tiles,
                                                          uint2 *__restrict__ sorted_boxes,
                                                          unsigned long long *__restrict__ block_sums)
{
    const int64_t n = clamp_count(n_dev, n_max);
    __shared__ unsigned long long part[2][kWaves];
    const int64_t base = (int64_t)blockIdx.x * scan_tile(ITEMS);
    unsigned long long at = 0, ar = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int64_t idx = base + (int64_t)j * kThreads + threadIdx.x;
        if (idx < n) {
            uint32_t t, r;
            uint2 box;
            scan_item(keys, boxes, order, idx, TW, TH, t, r, box);
            tiles[idx] = t;
            sorted_boxes[idx] = box;
            at += t;
            ar += r;
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        at += __shfl_xor(at, d, 64);
        ar += __shfl_xor(ar, d, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        part[0][threadIdx.x >> 6] = at;
        part[1][threadIdx.x >> 6] = ar;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const unsigned long long *p = part[threadIdx.x];
        block_sums[2 * blockIdx.x + threadIdx.x] = p[0] + p[1] + p[2] + p[3];
    }
}

// Single-block exclusive scan of the block-sum pairs; writes the two totals
// to counters[0] (instances) and counters[2] (tile rows).
__global__ __launch_bounds__(1024) void k_scan_top(unsigned long long *__restrict__ block_sums, int nb,
                                                   int64_t *__restrict__ counters)
{
    __shared__ unsigned long long wsum[2][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long carry[2] = {0, 0};
    for (int base = 0; base < nb; base += 1024) {
        const int i = base + threadIdx.x;
        unsigned long long x[2], v[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            x[c] = i < nb ? block_sums[2 * i + c] : 0ull;
            v[c] = x[c];
        }
        for (int d = 1; d < 64; d <<= 1) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const unsigned long long y = __shfl_up(v[c], d, 64);
                if (lane >= d) v[c] += y;
            }
        }
        if (lane == 63) {
            wsum[0][wave] = v[0];
            wsum[1][wave] = v[1];
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            unsigned long long before = 0, all = 0;
            for (int w = 0; w < 16; ++w) {
                if (w < wave) before += wsum[c][w];
                all += wsum[c][w];
            }
            if (i < nb) block_sums[2 * i + c] = carry[c] + before + v[c] - x[c];
            carry[c] += all;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        counters[0] = (int64_t)carry[0];
        counters[2] = (int64_t)carry[1];
    }
}

// Sums of the (tiles, rows) block-sum pairs of the blocks before `block`
// (pre) and of all nb blocks (all), the same in every thread.
__device__ void block_prefix_pairs(const unsigned long long *__restrict__ block_sums, int nb, int block,
                                   unsigned long long (&pre)[2], unsigned long long (&all)[2])
{
    __shared__ unsigned long long part[4][kWaves];
    unsigned long long v[4] = {0, 0, 0, 0};
    for (int i = threadIdx.x; i < nb; i += kThreads) {
        const unsigned long long t = block_sums[2 * i], r = block_sums[2 * i + 1];
        v[2] += t;
        v[3] += r;
        if (i < block) {
            v[0] += t;
            v[1] += r;
        }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
        for (int d = 32; d >= 1; d >>= 1) v[c] += __shfl_xor(v[c], d, 64);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int c = 0; c < 4; ++c) part[c][threadIdx.x >> 6] = v[c];
    __syncthreads();
    pre[0] = part[0][0] + part[0][1] + part[0][2] + part[0][3];
    pre[1] = part[1][0] + part[1][1] + part[1][2] + part[1][3];
    all[0] = part[2][0] + part[2][1] + part[2][2] + part[2][3];
    all[1] = part[3][0] + part[3][1] + part[3][2] + part[3][3];
}

// Offsets of every sorted item, scanned in place over the counts k_scan_reduce
// left in `offsets` (box tiles), and, when the instances fit, where each
// step of the emission starts: steps[m] = (item, row of its box) of tile row
// m plan.step.
// With `self_prefix` (few blocks), block_sums still holds every block's raw
// pair: each block sums the pairs before its own and all of them, block 0
// writes the totals to counters[0] and counters[2], and k_scan_top is not
// launched.  Otherwise k_scan_top has turned block_sums into exclusive
// prefixes and written the totals.
template <int ITEMS>
__global__ __launch_bounds__(kThreads) void k_scan_apply(int64_t n_max, const int64_t *__restrict__ n_dev,
                                                         int64_t capacity, int tile_w, int tile_h,
                                                         const uint2 *__restrict__ sorted_boxes,
                                                         const unsigned long long *__restrict__ block_sums,
                                                         int64_t *__restrict__ counters, bool self_prefix,
                                                         int tile_shift, uint32_t *__restrict__ offsets,
                                                         uint2 *__restrict__ steps)
{
    static_assert(ITEMS % 4 == 0, "whole 16-byte loads per thread");
    __shared__ uint32_t smem[kWaves];
    const int64_t n = clamp_count(n_dev, n_max);
    // blocked arrangement: thread t owns items base + t*ITEMS .. (aligned 16-byte groups)
    const int64_t base = (int64_t)blockIdx.x * scan_tile(ITEMS) + (int64_t)threadIdx.x * ITEMS;
    uint32_t c[ITEMS], r[ITEMS];
    const int hshift = __builtin_ctz(tile_h);
    if (base + ITEMS <= n) {
        const uint4 *pc = reinterpret_cast<const uint4 *>(offsets + base);
        const uint4 *pb = reinterpret_cast<const uint4 *>(sorted_boxes + base);
#pragma unroll
        for (int v = 0; v < ITEMS / 4; ++v) {
            const uint4 cv = pc[v], b0 = pb[2 * v], b1 = pb[2 * v + 1];
            c[4 * v] = cv.x; c[4 * v + 1] = cv.y; c[4 * v + 2] = cv.z; c[4 * v + 3] = cv.w;
            r[4 * v] = b0.y; r[4 * v + 1] = b0.w; r[4 * v + 2] = b1.y; r[4 * v + 3] = b1.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const bool in = base + j < n;
            c[j] = in ? offsets[base + j] : 0u;
            r[j] = in ? sorted_boxes[base + j].y : 0u;
        }
    }
    uint32_t lt = 0, lr = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        r[j] = c[j] ? (r[j] >> 16 >> hshift) - ((r[j] & 0xffffu) >> hshift) + 1u : 0u;
        lt += c[j];
        lr += r[j];
    }
    uint32_t tot;
    const uint32_t bt = block_inclusive_scan<kWaves>(lt, smem, &tot) - lt;
    const uint32_t br = block_inclusive_scan<kWaves>(lr, smem, &tot) - lr;
    unsigned long long pre[2], all[2];
    if (self_prefix) {
        block_prefix_pairs(block_sums, (int)gridDim.x, (int)blockIdx.x, pre, all);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            counters[0] = (int64_t)all[0];
            counters[2] = (int64_t)all[1];
        }
    } else {
        pre[0] = block_sums[2 * blockIdx.x];
        pre[1] = block_sums[2 * blockIdx.x + 1];
        all[0] = (unsigned long long)counters[0];
        all[1] = (unsigned long long)counters[2];
    }
    const int64_t totals[3] = {(int64_t)all[0], 0, (int64_t)all[1]};
    const EmitPlan P = emit_plan(totals, capacity, tile_shift);
    const int sshift = __builtin_ctz((unsigned)P.step);
    const bool fits = all[0] <= (unsigned long long)capacity;
    unsigned long long rt = pre[0] + bt;
    uint32_t rr = (uint32_t)(pre[1] + br);  // below the instances, so 32 bits where they fit
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int64_t idx = base + j;
        if (idx < n) {
            offsets[idx] = rt > 0xffffffffull ? 0xffffffffu : (uint32_t)rt;
            if (fits && c[j])
                for (uint32_t m = (rr + (uint32_t)P.step - 1u) >> sshift; m << sshift < rr + r[j]; ++m)
                    steps[m] = make_uint2((uint32_t)idx, (m << sshift) - rr);
        }
        rt += c[j];
        rr += r[j];
    }
}

// Depth order and binning scan of at most kSmallViews Gaussian-views by one
// workgroup, in place of six sort and two scan launches of 4 to 8 us each.  A least
// significant digit sort in LDS: each wave ranks its ROUNDS * 64 items in order
// by the lanes of equal digit, and the digits are the bits between the
// near plane's key and the largest one, spread over as few passes as 8 bits a pass allow.
// Then the boxes are gathered and both counts scanned, as k_scan_reduce and k_scan_apply do.
// Whole frames at 128x128 by the number of Gaussians, general path -> this: 64 73 -> 48
// us, 1000 95 -> 73 us, 2000 119 -> 104 us, 4000 148 -> 136 us; 8000 155 -> 165 us, so the line is at 4096.
// Bound by the latency of a pass (about 2.5 us).
constexpr int kSmallDigitBits = 8;
constexpr int64_t kSmallViews = 4096;

template <int THREADS, int ROUNDS>
__global__ __launch_bounds__(THREADS) void k_order_small(
    const uint32_t *__restrict__ keys, const uint2 *__restrict__ boxes, int n, uint32_t near_key, int wshift,
    int hshift, int64_t capacity, int tile_shift, uint32_t *__restrict__ keys_out, uint32_t *__restrict__ order,
    uint32_t *__restrict__ offsets, uint2 *__restrict__ steps, uint2 *__restrict__ sorted_boxes,
    int64_t *__restrict__ counters)
{
    constexpr int kBins = 1 << kSmallDigitBits, WAVES = THREADS / 64;
    static_assert(THREADS >= kBins, "a thread per digit");
    __shared__ uint32_t s_key[ROUNDS * THREADS];
    __shared__ uint16_t s_id[ROUNDS * THREADS];
    __shared__ uint32_t s_cnt_words[WAVES * kBins / 2];  // digit counts of each wave, 16 bits each, cleared by words
    __shared__ uint32_t s_wave[WAVES];
    __shared__ unsigned long long s_sum[2][WAVES];
    uint16_t(*const s_cnt)[kBins] = reinterpret_cast<uint16_t(*)[kBins]>(s_cnt_words);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int at0 = wave * ROUNDS * 64 + lane;  // item r of the thread is at0 + 64 r
    uint32_t key[ROUNDS], id[ROUNDS];
    uint32_t top = 0u;  // largest kept key
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        id[r] = (uint32_t)(at0 + 64 * r);
        key[r] = keys[min(at0 + 64 * r, n - 1)];
        if (at0 + 64 * r >= n) key[r] = 0xffffffffu;
        if (key[r] != 0xffffffffu) top = max(top, key[r]);
    }
    if (tid == 0) s_wave[0] = 0u;
    __syncthreads();
    if (top) atomicMax(&s_wave[0], top);
    __syncthreads();
    top = s_wave[0];
    const int bits = top > near_key ? 32 - __clz((int)(top - near_key)) : 1;
    const int passes = (bits + kSmallDigitBits - 1) / kSmallDigitBits, width = (bits + passes - 1) / passes;
    const uint32_t mask = (1u << width) - 1u;
    int count = n;  // items, after the first pass the kept ones
    for (int p = 0; p < passes; ++p) {
        __syncthreads();
        for (int i = tid; i < WAVES * kBins / 2; i += THREADS) s_cnt_words[i] = 0u;
        __syncthreads();
        const int shift = p * width;
        uint32_t digit[ROUNDS], rank[ROUNDS];
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const bool valid = p == 0 ? key[r] != 0xffffffffu : at0 + 64 * r < count;
            const uint32_t d = ((key[r] - near_key) >> shift) & mask;
            uint64_t same = __ballot(valid);  // lanes of the same digit
            for (int b = 0; b < width; ++b) {
                const bool one = (d >> b) & 1u;
                const uint64_t m = __ballot(one);
                same &= one ? m : ~m;
            }
            const uint32_t below =
                __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
            const uint32_t prior = s_cnt[wave][d];
            wave_sync();
            if (valid && below == 0) s_cnt[wave][d] = (uint16_t)(prior + (uint32_t)__popcll(same));
            wave_sync();
            digit[r] = d;
            rank[r] = valid ? prior + below : 0xffffffffu;
        }
        __syncthreads();
        uint32_t before[WAVES] = {}, run = 0;
        if (tid <= (int)mask)
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                before[w] = run;
                run += s_cnt[w][tid];
            }
        uint32_t tot;
        const uint32_t start = block_inclusive_scan<WAVES>(run, s_wave, &tot) - run;
        if (tid <= (int)mask)
#pragma unroll
            for (int w = 0; w < WAVES; ++w) s_cnt[w][tid] = (uint16_t)(start + before[w]);
        count = (int)tot;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r)
            if (rank[r] != 0xffffffffu) {
                const uint32_t to = s_cnt[wave][digit[r]] + rank[r];
                s_key[to] = key[r];
                s_id[to] = (uint16_t)id[r];
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r)
            if (at0 + 64 * r < count) {
                key[r] = s_key[at0 + 64 * r];
                id[r] = s_id[at0 + 64 * r];
            }
    }
    // thread t scans positions t ROUNDS .. t ROUNDS + ROUNDS - 1
    uint32_t c[ROUNDS], rows[ROUNDS];
    uint2 box[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int at = tid * ROUNDS + r;
        box[r] = make_uint2(0u, 0u);
        if (at < count) {
            id[r] = s_id[at];
            box[r] = boxes[id[r]];
            keys_out[at] = s_key[at];
            order[at] = id[r];
        }
    }
    unsigned long long lt = 0, lr = 0;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int at = tid * ROUNDS + r;
        const PixelBox pb = unpack_box(box[r]);
        rows[r] = at < count ? (uint32_t)((pb.y1 >> hshift) - (pb.y0 >> hshift) + 1) : 0u;
        c[r] = rows[r] * (uint32_t)((pb.x1 >> wshift) - (pb.x0 >> wshift) + 1);
        if (at < count) sorted_boxes[at] = box[r];
        lt += c[r];
        lr += rows[r];
    }
    unsigned long long it = lt, ir = lr;  // inclusive over the wave
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long a = __shfl_up(it, d, 64), b = __shfl_up(ir, d, 64);
        if (lane >= d) {
            it += a;
            ir += b;
        }
    }
    if (lane == 63) {
        s_sum[0][wave] = it;
        s_sum[1][wave] = ir;
    }
    __syncthreads();
    unsigned long long pre[2] = {0, 0}, all[2] = {0, 0};
#pragma unroll
    for (int w = 0; w < WAVES; ++w)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (w < wave) pre[q] += s_sum[q][w];
            all[q] += s_sum[q][w];
        }
    if (tid == 0) {
        counters[0] = (int64_t)all[0];
        counters[2] = (int64_t)all[1];
        counters[4] = count;
        *reinterpret_cast<uint32_t *>(counters + 6) = top;
    }
    const int64_t totals[3] = {(int64_t)all[0], 0, (int64_t)all[1]};
    const EmitPlan P = emit_plan(totals, capacity, tile_shift);
    const int sshift = __builtin_ctz((unsigned)P.step);
    const bool fits = all[0] <= (unsigned long long)capacity;
    unsigned long long rt = pre[0] + it - lt;
    uint32_t rr = (uint32_t)(pre[1] + ir - lr);
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int at = tid * ROUNDS + r;
        if (at < count) {
            offsets[at] = rt > 0xffffffffull ? 0xffffffffu : (uint32_t)rt;
            if (fits && c[r])
                for (uint32_t m = (rr + (uint32_t)P.step - 1u) >> sshift; m << sshift < rr + rows[r]; ++m)
                    steps[m] = make_uint2((uint32_t)at, (m << sshift) - rr);
        }
        rt += c[r];
        rr += rows[r];
    }
}

// ---------------------------------------------------------------- emission
// The listed tiles of the depth-sorted Gaussian-views' boxes, in three levels,
// each spread over the lanes of a wave:
//   Gaussian-view: its rows in the wave's step;
//   tile row: the conic is gathered (one 64-byte line), the support's x-extent
//     over the row and over its rows of pixel slots gives the interval of listed
//     tiles, and of slot columns, in the row;
//   listed tile: (tile id, id | slot bits), written next to each other.
// (A lane that wrote every tile of its row took 105 us of a 1280x960 frame close
// to a wall, whose rows are up to 160 tiles wide, and 0.90 ms of a 5120x3840 frame
// of needles whose boxes are nine tenths empty, and with the histogram launch 1.05 ms
// of 8 views; this takes 45 us, 0.25 ms and 0.85 ms.  A wave for every 512 box
// instances balances the blocks, but leaves most lanes idle in wide rows and
// computes steps of few rows in narrow ones: 1.7 ms for the 8 views.)
// Box tiles that are not listed are never written: a block's instances lie from
// its first row's box offset on, seg[block] = (offset, number).  `hist` counts
// them by the tile sort's first digit, so that pass needs no histogram launch.
// Instances stay grouped by Gaussian-view in depth order, so a stable sort on the tile id
// alone leaves every tile's list in depth order.  The kernel also clears the
// tile ranges and the compositing scheduling words for the stages after the
// tile sort (clear_a_words uint32 at `clear_a`, then `clear_b`).
// Instantiated per tile shape, so the slot layout of the culling bits is
// constant.

// Pixels of the box columns [bx0, bx1] whose centres lie in the extent
// [xl, xr] of offsets from u0, as [pa, pb]; a rectangle of pixel centres
// [sx0, sx1] inside the box meets the extent iff sx1 >= pa and sx0 <= pb.
// The estimates are at most one pixel off; the comparisons decide.  pa > pb
// when either bound is not a number (no comparison holds then).
__device__ __forceinline__ void pixel_extent(double xl, double xr, double u0, int bx0, int bx1, int &pa, int &pb)
{
#pragma clang fp contract(off)
    const double lo = (double)bx0, hi = (double)bx1;
    double a = ceil(xl + u0 - 0.5), b = floor(xr + u0 - 0.5);
    if (!(a + 0.5 - u0 >= xl))
        a += 1.0;
    else if ((a - 1.0) + 0.5 - u0 >= xl)
        a -= 1.0;
    if (!(b + 0.5 - u0 <= xr))
        b -= 1.0;
    else if ((b + 1.0) + 0.5 - u0 <= xr)
        b += 1.0;
    pa = (int)fmin(fmax(a, lo), hi + 1.0);
    pb = (int)fmax(fmin(b, hi), lo - 1.0);
    if (__builtin_isunordered(xl, xr)) pa = bx1 + 1, pb = bx0 - 1;
}

// Spreads counted work over a wave: lane l owns `count` units from `start` on
// (the exclusive scan of the counts), and the lane holding unit at0 + lane gets
// the owner's lane.  `before` is the owner of unit at0 - 1, used where no owner
// starts in the window up to this lane; slots are 64 LDS words of the wave.
__device__ __forceinline__ int unit_owner(uint32_t start, uint32_t count, uint32_t at0, int before, uint32_t *slots)
{
    const int lane = threadIdx.x & 63;
    slots[lane] = 64u;
    wave_sync();
    if (count != 0u && start - at0 < 64u) slots[start - at0] = (uint32_t)lane;
    wave_sync();
    const uint32_t mine = slots[lane];
    const uint64_t starts = __ballot(mine != 64u) & (~0ull >> (63 - lane));
    const int from = starts ? 63 - __builtin_clzll(starts) : 0;
    const int owner = __shfl((int)mine, from, 64);
    wave_sync();
    return starts ? owner : before;
}

template <int TW, int TH, int TILE, bool SELF>
__global__ __launch_bounds__(kEmitThreads) void k_emit(
    const uint32_t *__restrict__ order, const uint32_t *__restrict__ offsets, const uint2 *__restrict__ steps,
    const uint2 *__restrict__ sorted_boxes, const Conic *__restrict__ conics, const DevView *__restrict__ views,
    int64_t n, const int64_t *__restrict__ counters, int64_t capacity, RadixPass pass,
    uint32_t *__restrict__ inst_tiles, uint32_t *__restrict__ inst_ids, uint2 *__restrict__ seg,
    uint32_t *__restrict__ hist, int nblocks, uint32_t *__restrict__ clear_a, int64_t clear_a_words,
    uint32_t *__restrict__ clear_b, int64_t clear_b_words)
{
    constexpr SlotLayout SL = slot_layout(TW, TH);
    constexpr int NR = SL.bits ? SL.slots / SL.bx : 0;  // slot rows whose columns travel with the instance
    constexpr int BX = SL.bits ? SL.bx : 1, CW = SL.bits ? SL.cw : TW;
    constexpr int LW = TW == 8 ? 3 : TW == 16 ? 4 : 5, LH = TH == 8 ? 3 : TH == 16 ? 4 : 5;
    constexpr int LC = CW == 8 ? 3 : CW == 16 ? 4 : 5;
    constexpr int WAVES = kEmitThreads / 64;
    constexpr int kGRow = 4, kRRow = 2 + NR;
    __shared__ uint32_t cnt[kMaxBins];
    __shared__ uint32_t s_g[WAVES][kGRow][64], s_r[WAVES][kRRow][64], s_slots[WAVES][64], s_listed[2][WAVES];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    {
        const int64_t stride = (int64_t)gridDim.x * kEmitThreads, at = (int64_t)blockIdx.x * kEmitThreads + tid;
        for (int64_t i = at; i < clear_a_words; i += stride) clear_a[i] = 0u;
        for (int64_t i = at; i < clear_b_words; i += stride) clear_b[i] = 0u;
    }
    const EmitPlan P = emit_plan(counters, capacity, __builtin_ctz(TILE));
    constexpr bool ROUNDS = TILE == kLargeTile;
    const int end = SELF ? P.blocks : xcd_places(P.blocks);
    for (int place = (int)blockIdx.x; place < end; place += (int)gridDim.x) {
        const int block = SELF ? place : xcd_block(P.blocks, place);
        if (block >= P.blocks) {  // uniform per block
            if constexpr (!ROUNDS) return;
            continue;
        }
        const Digit D = pass_digit(pass);
        const int bins = 1 << D.bits;
        for (int i = tid; i < bins; i += kEmitThreads) cnt[i] = 0u;
        const uint32_t kept = (uint32_t)counters[4];
        const uint32_t row_first = (uint32_t)block * (uint32_t)P.rows;
        const uint32_t row_end = (uint32_t)min((int64_t)row_first + P.rows, P.rows_all);
        const int sshift = __builtin_ctz((unsigned)P.step);
        // box offset of the block's first row
        const uint2 start = steps[row_first >> sshift];
        const uint2 start_box = sorted_boxes[start.x];
        const uint32_t base =
            offsets[start.x] + start.y * ((start_box.x >> 16 >> LW) - ((start_box.x & 0xffffu) >> LW) + 1u);
        __syncthreads();
        uint32_t(*const G)[64] = s_g[wave];
        uint32_t(*const Rw)[64] = s_r[wave];
        uint32_t *const slots = s_slots[wave];
        uint32_t out = 0u;
        int turn = 0;
        for (uint32_t r0 = row_first; r0 < row_end; r0 += WAVES * P.step, turn ^= 1) {
            const uint32_t mine = r0 + (uint32_t)(wave * P.step);  // first row of the wave's step
            const int n_rows = mine < row_end ? min(P.step, (int)(row_end - mine)) : 0;
            uint32_t listed = 0u;
            if (n_rows) {
                // the Gaussian-views of the step's rows, from the one that its first row belongs to
                const uint2 first = steps[mine >> sshift];
                const uint32_t k = min(first.x + (uint32_t)lane, kept - 1u);
                const uint32_t id = order[k];
                const uint2 box = sorted_boxes[k];
                const uint32_t skip = lane == 0 ? first.y : 0u;
                const uint32_t rows = first.x + lane < kept ? (box.y >> 16 >> LH) - ((box.y & 0xffffu) >> LH) + 1u - skip : 0u;
                const uint32_t g_start = wave_inclusive_scan(rows) - rows;
                G[0][lane] = id;
                G[1][lane] = box.x;
                G[2][lane] = box.y;
                G[3][lane] = skip - g_start;  // row of the box = row of the step + this
                const int g = unit_owner(g_start, rows, 0u, 0, slots);
                if (lane < n_rows) {
                    const uint32_t gid = G[0][g];
                    const Conic C = conics[gid];
                    const PixelBox pb = unpack_box(make_uint2(G[1][g], G[2][g]));
                    const int ty = (pb.y0 >> LH) + (int)(lane + G[3][g]);
                    const DevView &V = views[gid / (uint32_t)n];
                    const uint32_t tile0 = (uint32_t)V.tile_base + (uint32_t)(ty * V.tiles_x);
                    const ConicFrame F = conic_frame(C);
                    BandRanges B;
                    band_ranges(C, F, pb, ty, TW, TH, B);
                    int pa, pe;
                    pixel_extent(B.row_xl, B.row_xr, C.u0, pb.x0, pb.x1, pa, pe);
                    const int ta = max(pb.x0, pa) >> LW, tb = min(pb.x1, pe) >> LW;
                    if (B.row_valid && pa <= pb.x1 && pe >= pb.x0 && ta <= tb) {
                        listed = (uint32_t)(tb - ta + 1);
                        Rw[0][lane] = tile0 + (uint32_t)ta;
                        Rw[1][lane] = gid;
#pragma unroll
                        for (int q = 0; q < NR; ++q) {
                            // slot columns [lo, hi) from tile ta's first on
                            uint32_t cols = 0u;
                            if ((B.valid >> q) & 1u) {
                                int qa = pa, qe = pe;
                                if (NR > 1) pixel_extent(B.xl[q], B.xr[q], C.u0, pb.x0, pb.x1, qa, qe);
                                if (qa <= pb.x1 && qe >= pb.x0) {
                                    const int c0 = max(max(pb.x0, qa) >> LC, ta * BX);
                                    const int c1 = min(min(pb.x1, qe) >> LC, tb * BX + BX - 1);
                                    if (c0 <= c1) cols = (uint32_t)(c0 - ta * BX) | (uint32_t)(c1 + 1 - ta * BX) << 16;
                                }
                            }
                            Rw[2 + q][lane] = cols;
                        }
                    }
                }
            }
            const uint32_t r_end = wave_inclusive_scan(listed), r_start = r_end - listed;
            const uint32_t n_listed = __builtin_amdgcn_readlane(r_end, 63);
            if (lane == 0) s_listed[turn][wave] = n_listed;
            __syncthreads();
            uint32_t at = base + out;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                const uint32_t x = s_listed[turn][w];
                at += w < wave ? x : 0u;
                out += x;
            }
            int r_before = 0;
            for (uint32_t ebase = 0; ebase < n_listed; ebase += 64u) {
                const int r = unit_owner(r_start, listed, ebase, r_before, slots);
                r_before = __builtin_amdgcn_readlane(r, 63);
                const uint32_t e = ebase + lane;
                const uint32_t j = e - (uint32_t)__shfl((int)r_start, r, 64);
                if (e < n_listed) {
                    const uint32_t tile = Rw[0][r] + j;
                    uint32_t bands = 0u;
#pragma unroll
                    for (int q = 0; q < NR; ++q) {
                        const uint32_t cols = Rw[2 + q][r], lo = cols & 0xffffu, hi = cols >> 16;
#pragma unroll
                        for (int c = 0; c < BX; ++c) {
                            const uint32_t col = j * BX + c;
                            if (col >= lo && col < hi) bands |= 1u << (q * BX + c);
                        }
                    }
                    inst_tiles[at + e] = tile;
                    inst_ids[at + e] = Rw[1][r] | (SL.bits ? bands << kIdBits : 0u);
                    atomicAdd(&cnt[D.of(tile)], 1u);
                }
            }
        }
        __syncthreads();
        if (tid == 0) seg[block] = make_uint2(base, out);
        const int row = SELF ? hist_row(bins) : bins;
        for (int d = tid; d < row; d += kEmitThreads)
            put_count<SELF>(hist, bins, nblocks, block, d, d < bins ? cnt[d] : 0u);
        if constexpr (!ROUNDS) return;
        __syncthreads();
    }
}

// ------------------------------------------------------------ tile ranges
__global__ __launch_bounds__(kThreads) void k_fill_u32(uint32_t *__restrict__ p, uint32_t value, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) p[i] = value;
}

__global__ void k_copy_i64(const int64_t *__restrict__ src, int64_t *__restrict__ dst)
{
    if (threadIdx.x == 0) *dst = *src;
}

// Each thread takes four consecutive positions per step (one 16-byte load and
// the two neighbours), so the grid-stride loop keeps four times as many loads
// in flight per step as one position per thread would.
__global__ __launch_bounds__(kThreads) void k_tile_ranges(const uint32_t *__restrict__ inst_tiles,
                                                          const int64_t *__restrict__ counters, int64_t capacity,
                                                          int64_t total_tiles, uint2 *__restrict__ ranges)
{
    const int64_t m = clamp_count(counters, capacity);
    const int64_t groups = (m + 3) / 4;
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    constexpr uint32_t kNone = 0xffffffffu;  // no neighbour (never a tile id)
    for (int64_t g = (int64_t)blockIdx.x * kThreads + threadIdx.x; g < groups; g += stride) {
        const int64_t p0 = 4 * g;
        uint32_t t[6];  // tiles at positions p0 - 1 .. p0 + 4
        if (p0 + 4 <= m) {
            const uint4 v = *reinterpret_cast<const uint4 *>(inst_tiles + p0);
            t[1] = v.x;
            t[2] = v.y;
            t[3] = v.z;
            t[4] = v.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) t[1 + j] = p0 + j < m ? inst_tiles[p0 + j] : kNone;
        }
        t[0] = p0 > 0 ? inst_tiles[p0 - 1] : kNone;
        t[5] = p0 + 4 < m ? inst_tiles[p0 + 4] : kNone;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t tj = t[1 + j];
            if (tj >= total_tiles) continue;  // also past the end (kNone)
            if (t[j] != tj) ranges[tj].x = (uint32_t)(p0 + j);
            if (t[j + 2] != tj) ranges[tj].y = (uint32_t)(p0 + j + 1);
        }
    }
}

// -------------------------------------------------------- tile scheduling
// Work order of the compositing kernels: work items sorted by decreasing list
// length (coarse buckets, order inside a bucket arbitrary), so
// the longest lists start first and the persistent grid drains evenly.  A
// tile whose list is longer than the average work of a compositing wave
// (listed instances / waves, at least split_min; split_min 0: never split)
// becomes two items, each compositing half of the tile's pixel rows against
// the whole list, which halves the longest chains of dependent work; split tiles
// come before all others, so that k_blend_team finds them by their number.  Item
// value = tile << 2 | part (0 whole tile, 1 first half, 2 second half).
constexpr int kSchedBuckets = 256;
constexpr int kSplitBuckets = 64;  // the buckets of split tiles, above those of all others
constexpr int64_t kRangeBlocks = 4096;

// Lists of whole tiles: steps of 4 entries up to 512, then of 32 up to 2560.  In dense frames only lists above the
// average work of a wave are split, and with one bucket for all whole tiles above 764 entries the longest came in
// any order: six views of up to 2209x2179, lists of up to 2826 entries, 2600 us of compositing, 2030 us with these.
__device__ __forceinline__ uint32_t work_bucket(uint32_t len, uint32_t parts)
{
    if (parts == 2u)
        return (uint32_t)(kSchedBuckets - kSplitBuckets) + min(len >> 5, (uint32_t)(kSplitBuckets - 1));
    return len < 512u ? len >> 2 : min(128u + ((len - 512u) >> 5), (uint32_t)(kSchedBuckets - kSplitBuckets - 1));
}

// average work of a wave
__device__ __forceinline__ uint32_t wave_share(const int64_t *listed, uint32_t waves)
{
    return (uint32_t)((*listed + waves - 1) / waves);
}

__device__ __forceinline__ uint32_t split_length(const int64_t *listed, uint32_t split_min, uint32_t waves)
{
    return split_min == 0u ? 0u : max(split_min, wave_share(listed, waves));
}

__device__ __forceinline__ uint32_t work_parts(uint32_t len, uint32_t split_len)
{
    return (split_len != 0u && len >= split_len) ? 2u : 1u;
}

// The entries of all items' lists and the longest list of a workgroup's tiles, for n_items[2..4] (all zero before).
// One pair of atomics per workgroup: atomics on one address take about 13 ns each, one after the other, and a pair
// per wave was 9 us of six views of 2452x2465.
struct ListSums {
    unsigned long long entries;
    uint32_t longest;

    // all lanes of a wave, after the words were cleared
    __device__ __forceinline__ void count(uint32_t len, uint32_t parts)
    {
        unsigned long long sum = (unsigned long long)len * parts;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            sum += __shfl_xor(sum, d, 64);
            len = max(len, (uint32_t)__shfl_xor((int)len, d, 64));
        }
        if ((threadIdx.x & 63) == 0 && len != 0u) {
            atomicAdd(&entries, sum);
            atomicMax(&longest, len);
        }
    }
    // one thread, after all have counted
    __device__ __forceinline__ void add_to(uint32_t *n_items) const
    {
        if (longest == 0u) return;
        atomicAdd(reinterpret_cast<unsigned long long *>(n_items + 2), entries);
        atomicMax(n_items + 4, longest);
    }
};

__global__ __launch_bounds__(kThreads) void k_sched_hist(const uint2 *__restrict__ ranges, int64_t total_tiles,
                                                         const int64_t *__restrict__ listed, uint32_t split_min,
                                                         uint32_t waves, uint32_t *__restrict__ hist,
                                                         uint32_t *__restrict__ sums)
{
    const uint32_t split_len = split_length(listed, split_min, waves);
    __shared__ uint32_t cnt[kSchedBuckets];
    __shared__ ListSums all;
    cnt[threadIdx.x] = 0;
    if (threadIdx.x == 0) all = {0ull, 0u};
    __syncthreads();
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    uint32_t len = 0u, parts = 0u;
    if (t < total_tiles) {
        const uint2 r = ranges[t];
        len = r.y - r.x;
        parts = work_parts(len, split_len);
        atomicAdd(&cnt[work_bucket(len, parts)], parts);
    }
    if (sums) all.count(len, parts);
    __syncthreads();
    if (cnt[threadIdx.x]) atomicAdd(&hist[threadIdx.x], cnt[threadIdx.x]);
    if (sums && threadIdx.x == 0) all.add_to(sums);
}

__global__ __launch_bounds__(kThreads) void k_sched_scatter(const uint2 *__restrict__ ranges, int64_t total_tiles,
                                                            const int64_t *__restrict__ listed, uint32_t split_min,
                                                            uint32_t waves, const uint32_t *__restrict__ hist,
                                                            uint32_t *__restrict__ cursor,
                                                            uint32_t *__restrict__ n_items,
                                                            uint32_t *__restrict__ work_order)
{
    __shared__ uint32_t smem[kWaves];
    __shared__ uint32_t base[kSchedBuckets];
    __shared__ uint32_t cnt[kSchedBuckets];
    const uint32_t split_len = split_length(listed, split_min, waves);
    // buckets in decreasing order: bucket b starts after all items of buckets > b
    const uint32_t hb = hist[kSchedBuckets - 1 - threadIdx.x];
    uint32_t tot;
    const uint32_t before = block_inclusive_scan<kWaves>(hb, smem, &tot) - hb;
    base[kSchedBuckets - 1 - threadIdx.x] = before;
    cnt[threadIdx.x] = 0;
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) n_items[0] = tot;
        if (threadIdx.x == kSplitBuckets - 1) n_items[1] = before + hb;  // those of split tiles
    }
    __syncthreads();
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    uint32_t b = 0, rank = 0, parts = 0;
    if (t < total_tiles) {
        const uint2 r = ranges[t];
        parts = work_parts(r.y - r.x, split_len);
        b = work_bucket(r.y - r.x, parts);
        rank = atomicAdd(&cnt[b], parts);
    }
    __syncthreads();
    if (cnt[threadIdx.x]) base[threadIdx.x] += atomicAdd(&cursor[threadIdx.x], cnt[threadIdx.x]);
    __syncthreads();
    if (parts == 1u) work_order[base[b] + rank] = (uint32_t)t << 2;
    if (parts == 2u) {
        work_order[base[b] + rank] = (uint32_t)t << 2 | 1u;
        work_order[base[b] + rank + 1] = (uint32_t)t << 2 | 2u;
    }
}

// The same for at most kSmallTiles tiles in one launch of one workgroup: 2.7 us
// instead of 5.5 for 560 tiles.
constexpr int kSmallTiles = 1024;

__global__ __launch_bounds__(kSmallTiles) void k_sched_small(const uint2 *__restrict__ ranges, int total_tiles,
                                                             const int64_t *__restrict__ listed, uint32_t split_min,
                                                             uint32_t waves, uint32_t *__restrict__ n_items,
                                                             uint32_t *__restrict__ work_order, bool sums)
{
    __shared__ uint32_t base[kSchedBuckets];
    __shared__ uint32_t smem[kSmallTiles / 64];
    const int t = threadIdx.x;
    __shared__ ListSums all;
    if (t < kSchedBuckets) base[t] = 0u;
    if (t == 0) all = {0ull, 0u};
    uint2 r = make_uint2(0u, 0u);
    if (t < total_tiles) r = ranges[t];
    __syncthreads();
    const uint32_t split_len = split_length(listed, split_min, waves);
    const uint32_t len = r.y - r.x, parts = t < total_tiles ? work_parts(len, split_len) : 0u;
    const uint32_t b = work_bucket(len, parts);
    const uint32_t rank = parts ? atomicAdd(&base[b], parts) : 0u;
    if (sums) all.count(len, parts);
    __syncthreads();
    // buckets in decreasing order, as in k_sched_scatter
    const uint32_t hb = t < kSchedBuckets ? base[kSchedBuckets - 1 - t] : 0u;
    uint32_t tot;
    const uint32_t before = block_inclusive_scan<kSmallTiles / 64>(hb, smem, &tot) - hb;
    if (t < kSchedBuckets) base[kSchedBuckets - 1 - t] = before;
    if (t == 0) n_items[0] = tot;
    if (sums && t == 0) all.add_to(n_items);
    if (t == kSplitBuckets - 1) n_items[1] = before + hb;  // those of split tiles
    __syncthreads();
    if (parts == 1u) work_order[base[b] + rank] = (uint32_t)t << 2;
    if (parts == 2u) {
        work_order[base[b] + rank] = (uint32_t)t << 2 | 1u;
        work_order[base[b] + rank + 1] = (uint32_t)t << 2 | 2u;
    }
}

}  // namespace

int radix_passes(int bits) { return bits <= 0 ? 0 : (bits + kMaxDigitBits - 1) / kMaxDigitBits; }

namespace {
// Workgroup shapes by the sort's size.  Up to kSelfMax items a pass is two
// launches, the scatter summing the histogram rows itself: at 0.5M keys, a third of
// them kept, three passes took 44 us and with a scan launch 50 us; at 0.6M
// kept it is 73 against 58 us, as every block reads the rows of all.  Up to
// kMidMax blocks stay small, so that there are enough of them (1.5M tile ids: 42
// us, 49 us at twice the items); above, larger blocks write longer runs (22.5M depth keys
// and 66M tile ids: 1.44 ms, 1.66 ms at half the items).
constexpr int kSortThreads = 512, kSmallItems = 4, kLargeItems = kLargeTile / kSortThreads;
constexpr int64_t kSelfMax = int64_t(1) << 19, kMidMax = int64_t(1) << 23;

int block_items(int64_t n_max) { return kSortThreads * (n_max <= kMidMax ? kSmallItems : kLargeItems); }

// log2 of the items of a block of a sort of up to n_max items
int tile_shift(int64_t n_max) { return __builtin_ctz((unsigned)block_items(n_max)); }
}  // namespace

namespace {
// Places that reach every block of xcd_block for any nb up to nblocks: its
// last round of runs may be partly empty (8 runs of at most 64 or nb / 64 blocks).
int xcd_grid(int nblocks) { return (nblocks + std::min(512, nblocks / 8) + 15) & ~7; }
constexpr int kMaxGrid = 4096, kMaxEmitGrid = 8192;  // of a large sort

// The widest digit of any pass of a sort on `bits` bits; with a key range the
// first pass has kFirstBits bits and the others up to the widest.
int widest_digit(int bits, bool ranged, int pass)
{
    if (ranged) return pass == 0 ? kFirstBits : kMaxDigitBits;
    const int passes = radix_passes(bits);
    return passes == 0 ? 0 : (bits + passes - 1) / passes;
}
}  // namespace

// Histogram rows of every block, and the digit totals where they are scanned
// in a launch of their own.
size_t radix_scratch_words(int64_t n_max, int bits, bool ranged)
{
    const bool self = n_max <= kSelfMax;
    const int64_t tile = block_items(n_max);
    const size_t bins = (size_t)1 << widest_digit(bits, ranged, 1);
    const size_t blocks = (size_t)((n_max + tile - 1) / tile);
    return self ? std::max(bins, (size_t)8) / 2 * blocks : bins * blocks + bins;
}

namespace {
template <int TH, int IT, bool SELF>
void radix_pass(const uint32_t *ki, const uint32_t *vi, uint32_t *ko, uint32_t *vo, int64_t n_max, const int64_t *pn,
                const RadixPass &pass, int wide, bool drop, uint32_t drop_key, int64_t *kept_out,
                const RadixRange *top, const uint2 *seg, uint2 *ranges, uint32_t *scratch, hipStream_t stream)
{
    constexpr int tile = TH * IT;
    const int nblocks = (int)((n_max + tile - 1) / tile), all = xcd_grid(nblocks);
    const int grid = tile == kLargeTile ? std::min(all, kMaxGrid) : all;
    uint32_t *const hist = scratch, *const row_total = scratch + (size_t)wide * nblocks;
    // the first histogram launch also finds the largest key, in one more
    // workgroup; the emission has made the histogram of its segments
    if (!seg)
        k_radix_hist<TH, IT, SELF><<<grid + (top ? 1 : 0), TH, 0, stream>>>(
            ki, n_max, pn, pass, drop, drop_key, hist, nblocks, grid, top ? top->part_max : nullptr,
            top ? top->n_parts : 0, top ? top->kmax : nullptr);
    if (!SELF) k_radix_scan_rows<<<wide, kThreads, 0, stream>>>(hist, nblocks, n_max, pn, pass, tile, seg != nullptr,
                                                               row_total);
    const auto scatter = seg ? &k_radix_scatter<TH, IT, SELF, true> : &k_radix_scatter<TH, IT, SELF, false>;
    scatter<<<grid, TH, 0, stream>>>(ki, vi, ko, vo, n_max, pn, pass, drop, drop_key, kept_out, hist, row_total, nblocks,
                                     seg, ranges);
}

hipError_t sort_passes(uint32_t *keys, uint32_t *vals, uint32_t *keys_alt, uint32_t *vals_alt, int64_t n_max,
                       const int64_t *n_dev, int bits, const RadixRange *range, bool drop, uint32_t drop_key,
                       int64_t *kept_out, bool iota, const uint2 *seg, uint2 *ranges, uint32_t *scratch,
                       hipStream_t stream)
{
    const int passes = radix_passes(bits);
    const bool fewer = drop || seg;  // items leave the sort in the first pass
    uint32_t *ki = keys, *vi = vals, *ko = keys_alt, *vo = vals_alt;
    for (int p = 0; p < passes; ++p) {
        const bool first = p == 0;
        const RadixPass pass{range ? range->kmax : nullptr, range ? range->base : 0u, bits, p, passes};
        const int wide = 1 << widest_digit(bits, range != nullptr, p);
        const auto run = n_max <= kSelfMax  ? &radix_pass<kSortThreads, kSmallItems, true>
                         : n_max <= kMidMax ? &radix_pass<kSortThreads, kSmallItems, false>
                                            : &radix_pass<kSortThreads, kLargeItems, false>;
        run(ki, iota && first ? nullptr : vi, ko, vo, n_max, fewer && !first ? kept_out : n_dev, pass, wide,
            drop && first, drop_key, fewer && first ? kept_out : nullptr, first ? range : nullptr,
            first ? seg : nullptr, passes == 1 ? ranges : nullptr, scratch, stream);
        std::swap(ki, ko);
        std::swap(vi, vo);
    }
    return hipGetLastError();
}
}  // namespace

hipError_t radix_sort(uint32_t *keys, uint32_t *vals, uint32_t *keys_alt, uint32_t *vals_alt, int64_t n_max,
                      const int64_t *n_dev, int bits, const RadixRange *range, bool drop, uint32_t drop_key,
                      int64_t *kept_out, uint32_t *scratch, hipStream_t stream, bool iota)
{
    if (n_max <= 0 || radix_passes(bits) == 0) {
        if (drop) k_fill_u32<<<1, kThreads, 0, stream>>>(reinterpret_cast<uint32_t *>(kept_out), 0u, 2);
        return hipGetLastError();
    }
    return sort_passes(keys, vals, keys_alt, vals_alt, n_max, n_dev, bits, range, drop, drop_key, kept_out, iota,
                       nullptr, nullptr, scratch, stream);
}

// sized for the smallest tile, so either choice of items per thread fits
size_t scan_block_entries(int64_t n)
{
    const int64_t tile = scan_tile(kScanItemsMin);
    return 2 * (size_t)((n + tile - 1) / tile + 1);
}

namespace {
template <int ITEMS>
void scan_launch(const uint32_t *keys, const uint2 *boxes, const uint32_t *order, int64_t n, const int64_t *n_dev,
                 int tile_w, int tile_h, int64_t capacity, uint32_t *offsets, uint2 *steps, uint2 *sorted_boxes,
                 unsigned long long *block_sums, int64_t *counters, hipStream_t stream)
{
    const int nb = (int)((n + scan_tile(ITEMS) - 1) / scan_tile(ITEMS));
    k_scan_reduce<ITEMS><<<nb, kThreads, 0, stream>>>(keys, boxes, order, n, n_dev, tile_w, tile_h, offsets,
                                                      sorted_boxes, block_sums);
    // up to kScanSelfPrefixBlocks blocks, each apply block sums the block
    // pairs before it (at most that many loads) instead of a separate scan
    const bool self_prefix = nb <= kScanSelfPrefixBlocks;
    if (!self_prefix) k_scan_top<<<1, 1024, 0, stream>>>(block_sums, nb, counters);
    k_scan_apply<ITEMS><<<nb, kThreads, 0, stream>>>(n, n_dev, capacity, tile_w, tile_h, sorted_boxes, block_sums,
                                                     counters, self_prefix, tile_shift(capacity), offsets, steps);
}

// The binning's scratch: the emission's steps (at least 64 rows each, or 8 of
// a block), its blocks' segments (no more than the tile sort has blocks) and the tile sort's histograms.
int64_t emit_blocks(int64_t capacity) { return ((capacity - 1) >> tile_shift(capacity)) + 1; }
size_t step_words(int64_t capacity)
{
    return 4 * (size_t)(std::max(capacity / 64 + 1, 8 * emit_blocks(capacity)) / 2 + 1);
}
size_t seg_words(int64_t capacity) { return 4 * (size_t)(emit_blocks(capacity) / 2 + 1); }
}  // namespace

hipError_t binning_scan(const uint32_t *keys, const uint2 *boxes, const uint32_t *order, int64_t n,
                        const int64_t *n_dev, int tile_w, int tile_h, int64_t capacity, uint32_t *offsets,
                        uint32_t *bin_scratch, uint2 *sorted_boxes, unsigned long long *block_sums,
                        int64_t *counters, hipStream_t stream)
{
    if (n <= 0) {
        // counters[0] and counters[2] (int64) = 0, counters[1] (capacity) kept
        k_fill_u32<<<1, kThreads, 0, stream>>>(reinterpret_cast<uint32_t *>(counters), 0u, 2);
        k_fill_u32<<<1, kThreads, 0, stream>>>(reinterpret_cast<uint32_t *>(counters + 2), 0u, 2);
        return hipGetLastError();
    }
    if (n <= (int64_t(1) << 20))
        scan_launch<4>(keys, boxes, order, n, n_dev, tile_w, tile_h, capacity, offsets,
                       reinterpret_cast<uint2 *>(bin_scratch), sorted_boxes, block_sums, counters, stream);
    else
        scan_launch<8>(keys, boxes, order, n, n_dev, tile_w, tile_h, capacity, offsets,
                       reinterpret_cast<uint2 *>(bin_scratch), sorted_boxes, block_sums, counters, stream);
    return hipGetLastError();
}

bool order_small(int64_t n) { return n > 0 && n <= kSmallViews; }

hipError_t launch_order_small(const uint32_t *keys, const uint2 *boxes, int64_t n, uint32_t near_key, int tile_w,
                              int tile_h, int64_t capacity, uint32_t *keys_out, uint32_t *order, uint32_t *offsets,
                              uint32_t *bin_scratch, uint2 *sorted_boxes, int64_t *counters, hipStream_t stream)
{
#define RGS_SMALL(THREADS, ROUNDS)                                                                                   \
    k_order_small<THREADS, ROUNDS><<<1, THREADS, 0, stream>>>(                                                       \
        keys, boxes, (int)n, near_key, __builtin_ctz((unsigned)tile_w), __builtin_ctz((unsigned)tile_h), capacity,   \
        tile_shift(capacity), keys_out, order, offsets, reinterpret_cast<uint2 *>(bin_scratch), sorted_boxes, counters)
    if (n <= 256)
        RGS_SMALL(256, 1);
    else if (n <= 1024)
        RGS_SMALL(512, 2);
    else if (n <= 2048)
        RGS_SMALL(1024, 2);
    else
        RGS_SMALL(1024, 4);
#undef RGS_SMALL
    return hipGetLastError();
}

size_t bin_scratch_words(int64_t capacity, int tile_bits)
{
    return step_words(capacity) + seg_words(capacity) + radix_scratch_words(capacity, tile_bits, false);
}

hipError_t emit_and_sort(const uint32_t *order, const uint32_t *offsets, uint32_t *bin_scratch,
                         const uint2 *sorted_boxes, const Conic *conics, const DevView *views, int64_t n,
                         const int64_t *counters, int64_t capacity, int tile_w, int tile_h, int tile_bits,
                         uint32_t *tiles, uint32_t *ids, uint32_t *tiles_alt, uint32_t *ids_alt, int64_t *listed,
                         uint2 *ranges, int64_t total_tiles, uint32_t *sched, hipStream_t stream, bool emit)
{
    const uint2 *const steps = reinterpret_cast<const uint2 *>(bin_scratch);
    uint2 *const seg = reinterpret_cast<uint2 *>(bin_scratch + step_words(capacity));
    uint32_t *const hist = bin_scratch + step_words(capacity) + seg_words(capacity);
    if (!emit)
        return sort_passes(tiles, ids, tiles_alt, ids_alt, capacity, counters, tile_bits, nullptr, false, 0u, listed,
                           false, seg, ranges, hist, stream);
    const int nblocks = (int)emit_blocks(capacity), all = xcd_grid(nblocks);
    const int grid = capacity > kMidMax ? std::min(all, kMaxEmitGrid) : all;
    const RadixPass pass{nullptr, 0u, tile_bits, 0, radix_passes(tile_bits)};
    // runs even with no Gaussian: it clears the ranges and scheduling words
#define RGS_EMIT_SEG(W, H, SEG, SELF)                                                                                 \
    k_emit<W, H, SEG, SELF><<<grid, kEmitThreads, 0, stream>>>(order, offsets, steps, sorted_boxes, conics, views,     \
                                                           n > 0 ? n : 1, counters, capacity, pass, tiles, ids, seg, \
                                                           hist, nblocks,                                             \
                                                           reinterpret_cast<uint32_t *>(ranges), 2 * total_tiles,     \
                                                           sched, (int64_t)sched_words())
#define RGS_EMIT(W, H)                                                                 \
    if (tile_w == W && tile_h == H) {                                                  \
        if (capacity <= kSelfMax)                                                      \
            RGS_EMIT_SEG(W, H, kSortThreads * kSmallItems, true);                      \
        else if (capacity <= kMidMax)                                                  \
            RGS_EMIT_SEG(W, H, kSortThreads * kSmallItems, false);                     \
        else                                                                           \
            RGS_EMIT_SEG(W, H, kSortThreads * kLargeItems, false);                     \
        return hipGetLastError();                                                      \
    }
    RGS_EMIT(8, 8)
    RGS_EMIT(8, 16)
    RGS_EMIT(8, 32)
    RGS_EMIT(16, 8)
    RGS_EMIT(16, 16)
    RGS_EMIT(16, 32)
    RGS_EMIT(32, 8)
    RGS_EMIT(32, 16)
    RGS_EMIT(32, 32)
#undef RGS_EMIT
#undef RGS_EMIT_SEG
    return hipErrorInvalidValue;
}

hipError_t launch_fill_u32(uint32_t *p, uint32_t value, int64_t n, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    k_fill_u32<<<(unsigned)((n + kThreads - 1) / kThreads), kThreads, 0, stream>>>(p, value, n);
    return hipGetLastError();
}

hipError_t launch_copy_i64(const int64_t *src, int64_t *dst, hipStream_t stream)
{
    k_copy_i64<<<1, 64, 0, stream>>>(src, dst);
    return hipGetLastError();
}

size_t sched_backward_heads() { return (size_t)kQueues * kQueueStride; }
size_t sched_item_count() { return 2 * sched_backward_heads() + 2 * kSchedBuckets; }
size_t sched_words() { return sched_item_count() + 6; }

hipError_t launch_tile_ranges(const uint32_t *inst_tiles, const int64_t *counters, int64_t capacity,
                              int64_t total_tiles, int tile_bits, uint32_t split_min, uint32_t waves, bool sums,
                              uint2 *ranges, uint32_t *sched, uint32_t *work_order, hipStream_t stream)
{
    uint32_t *const n_items = sched + sched_item_count();
    // the ranges, queue heads and scheduling histograms were cleared by k_emit; a tile sort
    // of one pass has written the ranges
    // a grid-stride loop over the listed instances (a grid sized for the whole
    // capacity would mostly launch idle workgroups)
    if (capacity > 0 && radix_passes(tile_bits) > 1) {
        const unsigned grid = (unsigned)std::min<int64_t>((capacity + 4 * kThreads - 1) / (4 * kThreads), kRangeBlocks);
        k_tile_ranges<<<grid, kThreads, 0, stream>>>(inst_tiles, counters, capacity, total_tiles, ranges);
    }
    if (total_tiles <= kSmallTiles) {
        k_sched_small<<<1, kSmallTiles, 0, stream>>>(ranges, (int)total_tiles, counters, split_min, waves, n_items,
                                                     work_order, sums);
        return hipGetLastError();
    }
    const unsigned nb = (unsigned)((total_tiles + kThreads - 1) / kThreads);
    uint32_t *hist = sched + 2 * sched_backward_heads(), *cursor = hist + kSchedBuckets;
    k_sched_hist<<<nb, kThreads, 0, stream>>>(ranges, total_tiles, counters, split_min, waves, hist,
                                              sums ? n_items : nullptr);
    k_sched_scatter<<<nb, kThreads, 0, stream>>>(ranges, total_tiles, counters, split_min, waves, hist, cursor,
                                                 n_items, work_order);
    return hipGetLastError();
}

}  // namespace rgs
