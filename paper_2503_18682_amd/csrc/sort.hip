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
// Scans of at least this many blocks write the row owner map in row order.
constexpr int kScanRowOrderBlocks = 4096;
// Radix sort: digits of up to 11 bits, so that a 32-bit key takes 3 passes and a tile id one or two.
constexpr int kMaxDigitBits = 11;
constexpr int kMaxBins = 1 << kMaxDigitBits;
constexpr int kHistWordsLog = 12;  // counters of a histogram block (all copies of all bins)
constexpr int kHistWords = 1 << kHistWordsLog;

// Element count of a device-sized array: a frame whose instance count
// overflowed the capacity is treated as empty downstream (its status reports
// the overflow), so no kernel ever reads entries that were not written.
__device__ __forceinline__ int64_t clamp_count(const int64_t *n_dev, int64_t n_max)
{
    if (!n_dev) return n_max;
    const int64_t n = *n_dev;
    return n <= n_max ? n : 0;
}

// Inclusive scan across a block of WAVES waves; returns the inclusive
// prefix and writes the block total to *total.
template <int WAVES>
__device__ __forceinline__ uint32_t block_inclusive_scan(uint32_t x, uint32_t *smem /*[WAVES]*/, uint32_t *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t v = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(v, d, 64);
        if (lane >= d) v += y;
    }
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

// Block of items of this workgroup: workgroups are dealt to the 8 XCDs in
// turn, and each XCD takes a contiguous run of the nb blocks.  The blocks in
// flight on one XCD then write next to each other in every digit's range, and
// their short runs merge into whole lines in that XCD's L2 (blocks dealt in
// order leave every line shared by several XCDs, each writing its part to
// memory).  Returns nb or more when there is none.
__device__ __forceinline__ int xcd_block(int nb)
{
    const int share = (nb + 7) >> 3, k = (int)(blockIdx.x >> 3);
    return k < share ? (int)(blockIdx.x & 7u) * share + k : nb;
}

// Words of a block's histogram row in the block-major layout (whole uint4).
__device__ __forceinline__ int hist_row(int bins) { return max(bins, 4); }

// Digit histogram of one block's items; with `drop`, keys equal to drop_key
// are left out (they leave the sort in this pass).  Blocks past the
// device-side count write nothing.  All keys of a thread are loaded before the
// first is counted.  Up to 8 interleaved copies of each counter (by lane)
// keep equal digits of a wave off one LDS address.
template <int THREADS, int ITEMS, bool SELF>
__global__ __launch_bounds__(THREADS) void k_radix_hist(const uint32_t *__restrict__ keys, int64_t n_max,
                                                        const int64_t *__restrict__ n_dev, RadixPass pass, bool drop,
                                                        uint32_t drop_key, uint32_t *__restrict__ hist, int nblocks,
                                                        const uint32_t *__restrict__ part_max, int n_parts,
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
    const int nb = (int)((n + TILE - 1) / TILE), block = SELF ? (int)blockIdx.x : xcd_block(nb);
    if (block >= nb) return;  // uniform per block
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
        hist[SELF ? (size_t)block * row + d : (size_t)d * nblocks + block] = x;
    }
}

// Exclusive scan of each digit's row hist[d][0..nb) (one block per digit)
// over the nb = ceil(n / tile) blocks that hold items (tile = keys per block).
__global__ __launch_bounds__(kThreads) void k_radix_scan_rows(uint32_t *__restrict__ hist, int nblocks,
                                                              int64_t n_max, const int64_t *__restrict__ n_dev,
                                                              RadixPass pass, int tile,
                                                              uint32_t *__restrict__ row_total)
{
    __shared__ uint32_t smem[kWaves];
    if (blockIdx.x >> pass_digit(pass).bits) return;  // no such digit in this pass
    const int64_t n = clamp_count(n_dev, n_max);
    const int nb = (int)std::min<int64_t>((n + tile - 1) / tile, nblocks);
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
// With `drop`, keys equal to drop_key are not written, and the first block
// stores the number of items kept (the sum of the digit totals) in *kept_out.
// SELF: hist is block-major and unscanned (rows of hist_row(bins) words); each
// block sums the rows before its own (and all of them for the digit bases)
// itself, so the pass needs no scan launch.  Otherwise hist is digit-major and
// scanned, with row_total.
template <int THREADS, int ITEMS, bool SELF>
__global__ __launch_bounds__(THREADS, SELF ? 4 : 5) void k_radix_scatter(
    const uint32_t *__restrict__ keys_in, const uint32_t *__restrict__ vals_in, uint32_t *__restrict__ keys_out,
    uint32_t *__restrict__ vals_out, int64_t n_max, const int64_t *__restrict__ n_dev, RadixPass pass, bool drop,
    uint32_t drop_key, int64_t *__restrict__ kept_out, const uint32_t *__restrict__ hist,
    const uint32_t *__restrict__ row_total, int nblocks)
{
    constexpr int TILE = THREADS * ITEMS, WAVES = THREADS / 64;
    constexpr int kCntWords = WAVES * kMaxBins / 2, kSumWords = SELF ? 8 * THREADS : 0;
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

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int at0 = wave * (TILE / WAVES) + lane;
    uint32_t key[ITEMS], val[ITEMS];
    // small sorts load at once, by the launch's bounds; large ones know their block first
    auto load = [&](int64_t base, int left) {
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) key[r] = (keys_in + base)[(uint32_t)min(at0 + r * 64, left - 1)];
        if (vals_in) {
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) val[r] = (vals_in + base)[(uint32_t)min(at0 + r * 64, left - 1)];
        } else {
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) val[r] = (uint32_t)(base + at0 + r * 64);
        }
    };
    if constexpr (SELF) {
        const int64_t base = (int64_t)blockIdx.x * TILE;
        if (base >= n_max) return;
        load(base, (int)min(n_max - base, (int64_t)TILE));
    }
    const int64_t n = clamp_count(n_dev, n_max);
    const Digit D = pass_digit(pass);
    const int nb = (int)((n + TILE - 1) / TILE), block = SELF ? (int)blockIdx.x : xcd_block(nb);
    if (block >= nb) {  // uniform per block
        if (drop && nb == 0 && blockIdx.x == 0 && tid == 0) *kept_out = 0;
        return;
    }
    const int64_t base = (int64_t)block * TILE;
    const int left = (int)min(n - base, (int64_t)TILE);
    if constexpr (!SELF) load(base, left);
    const int bins = 1 << D.bits;

    // output position of each digit's first item of this block
    if constexpr (SELF) {
        // each thread sums four neighbouring digits over every groups-th row
        const int row = hist_row(bins), quads = row >> 2;
        const int quad = tid & (quads - 1), group = tid / quads, groups = THREADS / quads;
        uint4 all = make_uint4(0u, 0u, 0u, 0u), pre = all;
        constexpr int kStep = 16;
        const uint4 *src = reinterpret_cast<const uint4 *>(hist) + quad;
        for (int r0 = group; r0 < nb; r0 += groups * kStep) {
            uint4 x[kStep];
#pragma unroll
            for (int j = 0; j < kStep; ++j) x[j] = src[(size_t)(min(r0 + j * groups, nb - 1) * quads)];
#pragma unroll
            for (int j = 0; j < kStep; ++j) {
                const int r = r0 + j * groups;
                const uint32_t in = r < nb ? ~0u : 0u, before = r < block ? ~0u : 0u;
                all.x += x[j].x & in; all.y += x[j].y & in; all.z += x[j].z & in; all.w += x[j].w & in;
                pre.x += x[j].x & before; pre.y += x[j].y & before; pre.z += x[j].z & before; pre.w += x[j].w & before;
            }
        }
        s_mem4[tid] = all;
        s_mem4[THREADS + tid] = pre;
        __syncthreads();
    }
    uint32_t dig_carry = 0;
#pragma unroll 1
    for (int d0 = 0; d0 < bins; d0 += THREADS) {
        const int d = d0 + tid;
        uint32_t pre = 0, all = 0;
        if (d < bins) {
            if constexpr (SELF) {
                const int row = hist_row(bins), groups = 4 * THREADS / row;
                for (int g = 0; g < groups; ++g) {
                    all += s_mem[g * row + d];
                    pre += s_mem[4 * THREADS + g * row + d];
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
    }
    if (drop && block == 0 && tid == 0) *kept_out = (int64_t)dig_carry;
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
        __builtin_amdgcn_wave_barrier();
        if (valid && below == 0) cnt[d] = (uint16_t)(prior + (uint32_t)(__popc(lo) + __popc(hi)));
        __builtin_amdgcn_wave_barrier();
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
    const int count = (int)carry;  // items of this block that stay in the sort
    const uint32_t n32 = (uint32_t)n;
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

// Gathers each sorted item's two counts once (into `tiles` and `rows`, read
// back by k_scan_apply, which scans them in place) and reduces them per block.
// The gathered binning box is also stored in depth order (`sorted_boxes`), so
// the emission kernel reads it coalesced instead of gathering it again.
template <int ITEMS>
__global__ __launch_bounds__(kThreads) void k_scan_reduce(const uint32_t *__restrict__ keys,
                                                          const uint2 *__restrict__ boxes,
                                                          const uint32_t *__restrict__ order, int64_t n_max,
                                                          const int64_t *__restrict__ n_dev, int TW, int TH,
                                                          uint32_t *__restrict__ tiles, uint32_t *__restrict__ rows,
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
            rows[idx] = r;
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
// left in `offsets` (box tiles) and `row_offsets` (tile rows), plus the owner
// map of the tile rows (row_owner[r] = sorted position owning row r) when the
// instances fit.  The map is written per item (each thread the rows of its
// own items) or, with `rows_in_order`, in row order by consecutive threads,
// each looking its row's owner up in the block's item table.  Row order
// coalesces the stores, which pays off at tens of millions of items; with a
// few hundred blocks the lookups' latency is exposed and per item is faster.
// With `self_prefix` (few blocks), block_sums still holds every block's raw
// pair: each block sums the pairs before its own and all of them, block 0
// writes the totals to counters[0] and counters[2], and k_scan_top is not
// launched.  Otherwise k_scan_top has turned block_sums into exclusive
// prefixes and written the totals.
template <int ITEMS>
__global__ __launch_bounds__(kThreads) void k_scan_apply(int64_t n_max, const int64_t *__restrict__ n_dev,
                                                         int64_t capacity,
                                                         const unsigned long long *__restrict__ block_sums,
                                                         int64_t *__restrict__ counters, bool self_prefix,
                                                         bool rows_in_order, uint32_t *__restrict__ offsets,
                                                         uint32_t *__restrict__ row_offsets,
                                                         uint32_t *__restrict__ row_owner)
{
    static_assert(ITEMS % 4 == 0, "whole 16-byte loads per thread");
    __shared__ uint32_t smem[kWaves];
    const int64_t n = clamp_count(n_dev, n_max);
    // blocked arrangement: thread t owns items base + t*ITEMS .. (aligned 16-byte groups)
    const int64_t base = (int64_t)blockIdx.x * scan_tile(ITEMS) + (int64_t)threadIdx.x * ITEMS;
    uint32_t c[ITEMS], r[ITEMS];
    if (base + ITEMS <= n) {
        const uint4 *pc = reinterpret_cast<const uint4 *>(offsets + base);
        const uint4 *pr = reinterpret_cast<const uint4 *>(row_offsets + base);
#pragma unroll
        for (int v = 0; v < ITEMS / 4; ++v) {
            const uint4 cv = pc[v], rv = pr[v];
            c[4 * v] = cv.x; c[4 * v + 1] = cv.y; c[4 * v + 2] = cv.z; c[4 * v + 3] = cv.w;
            r[4 * v] = rv.x; r[4 * v + 1] = rv.y; r[4 * v + 2] = rv.z; r[4 * v + 3] = rv.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const bool in = base + j < n;
            c[j] = in ? offsets[base + j] : 0u;
            r[j] = in ? row_offsets[base + j] : 0u;
        }
    }
    uint32_t lt = 0, lr = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
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
    }
    const uint32_t block_rows = tot;  // tile rows of the block's items
    const bool fits = all[0] <= (unsigned long long)capacity;
    unsigned long long rt = pre[0] + bt;
    unsigned long long rr = pre[1] + br;
    // first row of each of the block's items, relative to the block's first row
    __shared__ uint32_t row_start[scan_tile(ITEMS)];
    uint32_t lr0 = br;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int64_t idx = base + j;
        if (idx < n) {
            offsets[idx] = rt > 0xffffffffull ? 0xffffffffu : (uint32_t)rt;
            row_offsets[idx] = rr > 0xffffffffull ? 0xffffffffu : (uint32_t)rr;
            // rows <= instances, so every row index lies below capacity
            if (fits && !rows_in_order)
                for (uint32_t q = 0; q < r[j]; ++q) row_owner[rr + q] = (uint32_t)idx;
        }
        row_start[threadIdx.x * ITEMS + j] = lr0;
        rt += c[j];
        rr += r[j];
        lr0 += r[j];
    }
    if (!fits || !rows_in_order) return;  // uniform over the grid
    __syncthreads();
    // owner map of the block's rows, written in row order by consecutive
    // threads: the owner of row q is the last item whose first row is <= q
    // (items without rows share the first row of the next item)
    const int64_t block_base = (int64_t)blockIdx.x * scan_tile(ITEMS);
    const int nvalid = (int)min((int64_t)scan_tile(ITEMS), n - block_base);
    const unsigned long long row0 = pre[1];
    for (uint32_t q = threadIdx.x; q < block_rows; q += kThreads) {
        int lo = 0, hi = nvalid;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (row_start[mid] <= q)
                lo = mid;
            else
                hi = mid;
        }
        // rows <= instances, so every row index lies below capacity
        row_owner[row0 + q] = (uint32_t)(block_base + lo);
    }
}

// ---------------------------------------------------------------- emission
// One lane per tile row of the sorted Gaussian-views (a grid-stride loop
// over the row count the scan produced): the lane computes the support's
// x-extent over the row and over its rows of pixel slots and writes every
// tile of the box row at its scanned position, as (tile id, id | slot bits)
// when the tile's pixel-centre rectangle meets the support and as the empty
// marker `empty_tile` otherwise.  Instances end up
// grouped by Gaussian-view in depth order, so a stable sort on the tile id
// alone leaves every tile's list in depth order.  The kernel also clears the
// tile ranges and the compositing scheduling words for the stages after the
// tile sort (`clear` holds clear_words uint32 at `clear_a`, then `clear_b`).
// Instantiated per tile shape, so the slot layout of the culling bits is
// constant.
template <int TW, int TH>
__global__ __launch_bounds__(kThreads) void k_emit(const uint32_t *__restrict__ order,
                                                   const uint32_t *__restrict__ offsets,
                                                   const uint32_t *__restrict__ row_offsets,
                                                   const uint32_t *__restrict__ row_owner,
                                                   const uint2 *__restrict__ sorted_boxes,
                                                   const Conic *__restrict__ conics,
                                                   const DevView *__restrict__ views, int64_t n,
                                                   const int64_t *__restrict__ counters, int64_t capacity,
                                                   uint32_t empty_tile, uint32_t *__restrict__ inst_tiles,
                                                   uint32_t *__restrict__ inst_ids, uint32_t *__restrict__ clear_a,
                                                   int64_t clear_a_words, uint32_t *__restrict__ clear_b,
                                                   int64_t clear_b_words)
{
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    const int64_t tid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    for (int64_t i = tid; i < clear_a_words; i += stride) clear_a[i] = 0u;
    for (int64_t i = tid; i < clear_b_words; i += stride) clear_b[i] = 0u;
    if (counters[0] > capacity) return;  // overflow: the instance total reports it
    const int64_t rows = counters[2];
    for (int64_t r = tid; r < rows; r += stride) {
        const uint32_t k = row_owner[r];
        const uint32_t id = order[k];
        const PixelBox pb = unpack_box(sorted_boxes[k]);
        const int v = (int)(id / (uint32_t)n);
        const int row = (int)(r - row_offsets[k]);
        const int ty = pb.y0 / TH + row;
        const int tx0 = pb.x0 / TW, tx1 = pb.x1 / TW;
        int64_t pos = (int64_t)offsets[k] + (int64_t)row * (tx1 - tx0 + 1);
        const Conic C = conics[id];
        const ConicFrame F = conic_frame(C);
        BandRanges B;
        band_ranges(C, F, pb, ty, TW, TH, B);
        const uint32_t row_base = (uint32_t)views[v].tile_base + (uint32_t)(ty * views[v].tiles_x);
        for (int tx = tx0; tx <= tx1; ++tx, ++pos) {
            uint32_t bands;
            const bool listed = tile_listed(C, B, pb, tx, TW, TH, bands);
            inst_tiles[pos] = listed ? row_base + (uint32_t)tx : empty_tile;
            inst_ids[pos] = pack_instance(id, bands, TW, TH);
        }
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
// length (coarse buckets of 4 entries, order inside a bucket arbitrary), so
// the longest lists start first and the persistent grid drains evenly.  A
// tile whose list is longer than the average work of a compositing wave
// (listed instances / waves, at least split_min; split_min 0: never split)
// becomes two items, each compositing half of the tile's pixel rows against
// the whole list, which halves the longest chains of dependent work.  Item
// value = tile << 2 | part (0 whole tile, 1 first half, 2 second half).
constexpr int kSchedBuckets = 256;
constexpr int64_t kRangeBlocks = 4096;

__device__ __forceinline__ uint32_t work_bucket(uint32_t len)
{
    return min(len >> 2, (uint32_t)(kSchedBuckets - 1));
}

__device__ __forceinline__ uint32_t split_length(const int64_t *listed, uint32_t split_min, uint32_t waves)
{
    if (split_min == 0u) return 0u;
    const int64_t share = (*listed + waves - 1) / waves;
    return (uint32_t)max((int64_t)split_min, share);
}

__device__ __forceinline__ uint32_t work_parts(uint32_t len, uint32_t split_len)
{
    return (split_len != 0u && len >= split_len) ? 2u : 1u;
}

__global__ __launch_bounds__(kThreads) void k_sched_hist(const uint2 *__restrict__ ranges, int64_t total_tiles,
                                                         const int64_t *__restrict__ listed, uint32_t split_min,
                                                         uint32_t waves, uint32_t *__restrict__ hist)
{
    const uint32_t split_len = split_length(listed, split_min, waves);
    __shared__ uint32_t cnt[kSchedBuckets];
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (t < total_tiles) {
        const uint2 r = ranges[t];
        atomicAdd(&cnt[work_bucket(r.y - r.x)], work_parts(r.y - r.x, split_len));
    }
    __syncthreads();
    if (cnt[threadIdx.x]) atomicAdd(&hist[threadIdx.x], cnt[threadIdx.x]);
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
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_items = tot;
    __syncthreads();
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    uint32_t b = 0, rank = 0, parts = 0;
    if (t < total_tiles) {
        const uint2 r = ranges[t];
        b = work_bucket(r.y - r.x);
        parts = work_parts(r.y - r.x, split_len);
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

}  // namespace

int radix_passes(int bits) { return bits <= 0 ? 0 : (bits + kMaxDigitBits - 1) / kMaxDigitBits; }

namespace {
// Workgroup shapes, from timings of whole sorts (rocprofv3; graph replays).
// Up to kSelfMax items a pass is two launches, and the shortest chain in a
// workgroup wins: three passes over 0.5M depth keys took 34 us of scatter at
// 512 x 4 and 37 at 1024 x 4 or 512 x 8.  Above it a pass has a scan launch of its
// own and 512 x 8 is best: a sort of 22.5M depth keys and one of 66M tile ids (8 views)
// took 0.93 ms of scatter and histograms of it, 1.10 ms at 256 x 16, 0.99 ms at 512 x 16.
constexpr int kSelfThreads = 512, kSelfItems = 4;
constexpr int kScanThreads = 512, kScanItems = 8;
constexpr int64_t kSelfMax = int64_t(1) << 20;
}  // namespace

namespace {
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
    const int64_t tile = self ? kSelfThreads * kSelfItems : kScanThreads * kScanItems;
    const size_t row = std::max((size_t)1 << widest_digit(bits, ranged, 1), (size_t)4);
    return row * (size_t)((n_max + tile - 1) / tile) + (self ? 0 : row);
}

hipError_t radix_sort(uint32_t *keys, uint32_t *vals, uint32_t *keys_alt, uint32_t *vals_alt, int64_t n_max,
                      const int64_t *n_dev, int bits, const RadixRange *range, bool drop, uint32_t drop_key,
                      int64_t *kept_out, uint32_t *scratch, hipStream_t stream, bool iota)
{
    const int passes = radix_passes(bits);
    if (n_max <= 0 || passes == 0) {
        if (drop) k_fill_u32<<<1, kThreads, 0, stream>>>(reinterpret_cast<uint32_t *>(kept_out), 0u, 2);
        return hipGetLastError();
    }
    uint32_t *ki = keys, *vi = vals, *ko = keys_alt, *vo = vals_alt;
    for (int p = 0; p < passes; ++p) {
        const int wide = 1 << widest_digit(bits, range != nullptr, p);
        uint32_t *const hist = scratch;
        // the first pass drops, the later ones sort the kept items
        const bool pdrop = drop && p == 0;
        const int64_t *pn = drop && p > 0 ? kept_out : n_dev;
        const uint32_t *pvi = iota && p == 0 ? nullptr : vi;
        const RadixPass pass{range ? range->kmax : nullptr, range ? range->base : 0u, bits, p, passes};
        // the first histogram launch also finds the largest key, in one more workgroup
        const bool top = range && p == 0;
        const uint32_t *parts = top ? range->part_max : nullptr;
        const int n_parts = top ? range->n_parts : 0;
        uint32_t *kmax_out = top ? range->kmax : nullptr;
        if (n_max <= kSelfMax) {
            constexpr int TH = kSelfThreads, IT = kSelfItems, tile = TH * IT;
            const int nblocks = (int)((n_max + tile - 1) / tile), grid = (nblocks + 7) & ~7;
            k_radix_hist<TH, IT, true><<<grid + top, TH, 0, stream>>>(ki, n_max, pn, pass, pdrop, drop_key, hist,
                                                                      nblocks, parts, n_parts, kmax_out);
            k_radix_scatter<TH, IT, true><<<grid, TH, 0, stream>>>(ki, pvi, ko, vo, n_max, pn, pass, pdrop, drop_key,
                                                                   kept_out, hist, nullptr, nblocks);
        } else {
            constexpr int TH = kScanThreads, IT = kScanItems, tile = TH * IT;
            const int nblocks = (int)((n_max + tile - 1) / tile), grid = (nblocks + 7) & ~7;
            uint32_t *const row_total = scratch + (size_t)wide * nblocks;
            k_radix_hist<TH, IT, false><<<grid + top, TH, 0, stream>>>(ki, n_max, pn, pass, pdrop, drop_key, hist,
                                                                       nblocks, parts, n_parts, kmax_out);
            k_radix_scan_rows<<<wide, kThreads, 0, stream>>>(hist, nblocks, n_max, pn, pass, tile, row_total);
            k_radix_scatter<TH, IT, false><<<grid, TH, 0, stream>>>(ki, pvi, ko, vo, n_max, pn, pass, pdrop, drop_key,
                                                                    kept_out, hist, row_total, nblocks);
        }
        uint32_t *t;
        t = ki; ki = ko; ko = t;
        t = vi; vi = vo; vo = t;
    }
    return hipGetLastError();
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
                 int tile_w, int tile_h, int64_t capacity, uint32_t *offsets, uint32_t *row_offsets,
                 uint32_t *row_owner, uint2 *sorted_boxes, unsigned long long *block_sums, int64_t *counters,
                 hipStream_t stream)
{
    const int nb = (int)((n + scan_tile(ITEMS) - 1) / scan_tile(ITEMS));
    k_scan_reduce<ITEMS><<<nb, kThreads, 0, stream>>>(keys, boxes, order, n, n_dev, tile_w, tile_h, offsets,
                                                      row_offsets, sorted_boxes, block_sums);
    // up to kScanSelfPrefixBlocks blocks, each apply block sums the block
    // pairs before it (at most that many loads) instead of a separate scan
    const bool self_prefix = nb <= kScanSelfPrefixBlocks;
    if (!self_prefix) k_scan_top<<<1, 1024, 0, stream>>>(block_sums, nb, counters);
    k_scan_apply<ITEMS><<<nb, kThreads, 0, stream>>>(n, n_dev, capacity, block_sums, counters, self_prefix,
                                                     nb >= kScanRowOrderBlocks, offsets, row_offsets, row_owner);
}
}  // namespace

hipError_t binning_scan(const uint32_t *keys, const uint2 *boxes, const uint32_t *order, int64_t n,
                        const int64_t *n_dev, int tile_w, int tile_h, int64_t capacity, uint32_t *offsets,
                        uint32_t *row_offsets, uint32_t *row_owner, uint2 *sorted_boxes,
                        unsigned long long *block_sums, int64_t *counters, hipStream_t stream)
{
    if (n <= 0) {
        // counters[0] and counters[2] (int64) = 0, counters[1] (capacity) kept
        k_fill_u32<<<1, kThreads, 0, stream>>>(reinterpret_cast<uint32_t *>(counters), 0u, 2);
        k_fill_u32<<<1, kThreads, 0, stream>>>(reinterpret_cast<uint32_t *>(counters + 2), 0u, 2);
        return hipGetLastError();
    }
    if (n <= (int64_t(1) << 20))
        scan_launch<4>(keys, boxes, order, n, n_dev, tile_w, tile_h, capacity, offsets, row_offsets, row_owner,
                       sorted_boxes, block_sums, counters, stream);
    else
        scan_launch<8>(keys, boxes, order, n, n_dev, tile_w, tile_h, capacity, offsets, row_offsets, row_owner,
                       sorted_boxes, block_sums, counters, stream);
    return hipGetLastError();
}

int emit_grid(int num_cus) { return 8 * num_cus; }

hipError_t launch_emit(const uint32_t *order, const uint32_t *offsets, const uint32_t *row_offsets,
                       const uint32_t *row_owner, const uint2 *sorted_boxes, const Conic *conics, const DevView *views,
                       int64_t n, int n_views, const int64_t *counters, int64_t capacity, int tile_w, int tile_h,
                       uint32_t empty_tile, uint32_t *inst_tiles, uint32_t *inst_ids, uint2 *ranges,
                       int64_t total_tiles, uint32_t *sched, int grid, hipStream_t stream)
{
    // runs even with no Gaussian: it clears the ranges and scheduling words
#define RGS_EMIT(W, H)                                                                                               \
    if (tile_w == W && tile_h == H) {                                                                                \
        k_emit<W, H><<<grid, kThreads, 0, stream>>>(order, offsets, row_offsets, row_owner, sorted_boxes, conics,     \
                                                    views, n > 0 ? n : 1, counters, capacity, empty_tile, inst_tiles, \
                                                    inst_ids, reinterpret_cast<uint32_t *>(ranges), 2 * total_tiles,  \
                                                    sched, (int64_t)sched_words());                                   \
        return hipGetLastError();                                                                                    \
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
    (void)n_views;
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
size_t sched_words() { return sched_item_count() + 4; }

hipError_t launch_tile_ranges(const uint32_t *inst_tiles, const int64_t *counters, int64_t capacity,
                              int64_t total_tiles, uint32_t split_min, uint32_t waves, uint2 *ranges,
                              uint32_t *sched, uint32_t *work_order, hipStream_t stream)
{
    // the ranges, queue heads and scheduling histograms were cleared by k_emit
    // a grid-stride loop over the listed instances (a grid sized for the whole
    // capacity would mostly launch idle workgroups)
    if (capacity > 0) {
        const unsigned grid = (unsigned)std::min<int64_t>((capacity + 4 * kThreads - 1) / (4 * kThreads), kRangeBlocks);
        k_tile_ranges<<<grid, kThreads, 0, stream>>>(inst_tiles, counters, capacity, total_tiles, ranges);
    }
    const unsigned nb = (unsigned)((total_tiles + kThreads - 1) / kThreads);
    uint32_t *hist = sched + 2 * sched_backward_heads(), *cursor = hist + kSchedBuckets;
    k_sched_hist<<<nb, kThreads, 0, stream>>>(ranges, total_tiles, counters, split_min, waves, hist);
    k_sched_scatter<<<nb, kThreads, 0, stream>>>(ranges, total_tiles, counters, split_min, waves, hist, cursor,
                                                 sched + sched_item_count(), work_order);
    return hipGetLastError();
}

}  // namespace rgs
