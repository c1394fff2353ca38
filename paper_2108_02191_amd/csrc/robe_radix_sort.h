// Stable LSD radix sort of (key, value) pairs of 32-bit words on a range of key bits, for the token
// sort of the backward pass (S2 in robe_backward_dedup.h).
//
// Eight bits per pass, three kernels per pass, no kernel ever waits for another workgroup:
//
//   count    a workgroup takes a tile of kSortTile pairs, counts the digits of its keys in LDS and
//            writes the counts to tile_count[digit][tile].
//   offsets  one workgroup per digit: an exclusive prefix over that digit's row of tile counts -
//            how many pairs of the digit the tiles before hold - and the digit's total.
//   scatter  a workgroup takes its tile again, finds where every digit starts (an exclusive scan of
//            the 256 totals), ranks every pair among the tile's pairs of the same digit in input
//            order (so the sort is stable), puts the tile into LDS in digit order and writes it out
//            from there, a digit's pairs to consecutive slots.
//            Up to kFewTiles tiles there is no such kernel: the counts lie tile by tile, and every
//            workgroup of the scatter adds the rows of the other tiles up itself, a digit per thread,
//            64 KB out of the L2 at the most (33 tiles: 8.1 us instead of 7.3, and no offsets kernel of 4.7).
//
// Inside a tile, wavefront w of the scatter kernel owns pairs [w * 512, (w + 1) * 512) and walks
// them 64 at a time, so the input order is (wavefront, round, lane): a pair's rank is what earlier rounds of its wavefront
// counted for the digit, plus the lanes below it in its own round with the same digit (found with one
// ballot per digit bit), plus what the wavefronts before it hold.
//
// It records nothing but kernels on the stream (no fill operations), and for the sizes met here
// (10^5 .. 10^7 pairs) it is shorter on launches than the device library's sort.  Up to 2^21 pairs the backward
// mostly needs less than a sort: see the grouping at the end of this file.
#pragma once
#include "robe_backward_dedup.h"

namespace robe {

constexpr int kSortBlock = 256;                       // count and offsets kernels: 4 wavefronts
constexpr int kSortRounds = 16;                       // count kernel: keys per thread
constexpr uint32_t kSortTile = kSortBlock * kSortRounds;   // 4096 pairs
constexpr uint32_t kDigits = 256;
constexpr uint32_t kFewTiles = 64;
static_assert(kSortBlock == (int)kDigits, "one thread per digit in the per-digit steps");

struct SortPass {
    uint32_t shift;      // first key bit of this pass's digit
    uint32_t mask;       // (1 << bits) - 1, bits <= 8
    uint32_t n;          // pairs
    uint32_t tiles;      // ceil(n / kSortTile)
    uint32_t few;        // 1: at most kFewTiles tiles, no offsets kernel
    uint32_t *tile_count;   // [kDigits][tiles]: counts, then the digit's pairs in the tiles before; few: [tiles][kDigits], counts
    uint32_t *totals;       // [kDigits]: pairs of each digit
};

// RUNS: equal keys sit side by side (every pass after the first: the pairs are sorted by the lower
// digits), and the copies of a frequent token would put dozens of LDS atomics of a wavefront on one
// word.  Then each run of equal digits among the 64 consecutive keys of a wavefront adds once, its
// length (31 -> 12 us on 8.5 M keys in runs of 37; 10 -> 12 us on keys without runs, hence not in
// the first pass).
template <bool RUNS>
__global__ __launch_bounds__(kSortBlock) void sort_count_kernel(SortPass s, const uint32_t *__restrict__ keys)
{
    __shared__ uint32_t h[kDigits];
    h[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t tile = blockIdx.x;
    const uint64_t base = (uint64_t)tile * kSortTile;
    uint32_t k[kSortRounds];
#pragma unroll
    for (int i = 0; i < kSortRounds; ++i) {
        const uint64_t at = base + (uint32_t)i * kSortBlock + threadIdx.x;
        k[i] = at < s.n ? keys[at] : 0u;
    }
    const uint32_t lane = threadIdx.x & 63u;
#pragma unroll
    for (int i = 0; i < kSortRounds; ++i) {
        const uint64_t at = base + (uint32_t)i * kSortBlock + threadIdx.x;
        const bool have = at < s.n;
        const uint32_t digit = have ? ((k[i] >> s.shift) & s.mask) : 0xFFFFFFFFu;   // no key: a run of its own, never added
        if constexpr (RUNS) {
            const uint32_t prev = __shfl_up(digit, 1);
            const bool head = lane == 0 || digit != prev;
            const uint64_t heads = __ballot(head);
            if (head && have) {
                const uint64_t above = heads & ~((2ull << lane) - 1ull);            // heads in the lanes after this one
                const uint32_t next = above ? (uint32_t)__builtin_ctzll(above) : 64u;
                atomicAdd(&h[digit], next - lane);
            }
        } else {
            if (have) atomicAdd(&h[digit], 1u);
        }
    }
    __syncthreads();
    s.tile_count[s.few ? (uint64_t)tile * kDigits + threadIdx.x : (uint64_t)threadIdx.x * s.tiles + tile] = h[threadIdx.x];
}

// Exclusive prefix of one value per thread over the workgroup's BLOCK threads.  `wave_total` is LDS
// for BLOCK / 64 words; the call ends with a barrier, so it may be reused right after.
template <int BLOCK>
__device__ __forceinline__ uint32_t exclusive_scan_block(uint32_t v, uint32_t *wave_total, uint32_t &total)
{
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (uint32_t off = 1; off < 64u; off <<= 1) {
        const uint32_t up = __shfl_up(incl, off);
        if (lane >= off) incl += up;
    }
    if (lane == 63u) wave_total[wave] = incl;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
#pragma unroll
    for (uint32_t w = 0; w < (uint32_t)BLOCK / 64u; ++w) {
        const uint32_t x = wave_total[w];
        before += w < wave ? x : 0u;
        total += x;
    }
    __syncthreads();
    return before + incl - v;
}

// One workgroup per digit.
constexpr int kOffsetItems = 8;   // tile counts per thread and step

__global__ __launch_bounds__(kSortBlock) void sort_offsets_kernel(SortPass s)
{
    __shared__ uint32_t wave_total[4];
    const uint32_t digit = blockIdx.x, t = threadIdx.x;
    uint32_t carry = 0;           // the same in every thread
    uint32_t *row = s.tile_count + (uint64_t)digit * s.tiles;
    for (uint32_t t0 = 0; t0 < s.tiles; t0 += kSortBlock * kOffsetItems) {     // same trip count for the whole workgroup
        uint32_t c[kOffsetItems], sum = 0;
#pragma unroll
        for (int k = 0; k < kOffsetItems; ++k) {
            const uint32_t i = t0 + t * kOffsetItems + (uint32_t)k;
            c[k] = i < s.tiles ? row[i] : 0u;
            sum += c[k];
        }
        uint32_t total;
        uint32_t a = carry + exclusive_scan_block<kSortBlock>(sum, wave_total, total);
#pragma unroll
        for (int k = 0; k < kOffsetItems; ++k) {
            const uint32_t i = t0 + t * kOffsetItems + (uint32_t)k;
            if (i < s.tiles) row[i] = a;
            a += c[k];
        }
        carry += total;
    }
    if (t == 0) s.totals[digit] = carry;
}

// Rank of this lane's digit (below 2^BITS) among those that the wavefront has met so far, in order of rounds
// and lanes; count: the wavefront's counters in LDS, which the call moves on.  Lanes that hold nothing
// (`have` false) are not counted.  The lanes of equal digit are found with one ballot per bit: lane masks as
// two words that lose, bit by bit, the lanes that differ (one three-operand instruction per word; written with
// 64-bit selects and populations under a mask a tile of 1.7 M pairs took 15.4 us a pass, now 14.2).
template <int BITS>
__device__ __forceinline__ uint32_t rank_in_tile(uint32_t digit, bool have, uint32_t *count)
{
    const uint64_t live = __ballot(have);
    uint32_t lo = (uint32_t)live, hi = (uint32_t)(live >> 32);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const uint32_t mine = 0u - ((digit >> b) & 1u);
        const uint64_t bit = __ballot(mine != 0u);
        lo &= ~((uint32_t)bit ^ mine);
        hi &= ~((uint32_t)(bit >> 32) ^ mine);
    }
    const uint32_t below = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
    const uint32_t so_far = count[digit];                   // every lane reads before the first lane of a set adds
    __builtin_amdgcn_wave_barrier();
    if (have && below == 0) count[digit] = so_far + (uint32_t)(__popc(lo) + __popc(hi));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return so_far + below;
}

// Which tile a scattering workgroup takes: every XCD an eighth of the tiles, in order, so that what neighbouring
// tiles write of a digit meets in one L2 instead of leaving eight of them in halves of a line.  Launched with
// tile_blocks() workgroups; those past the last tile end at once.  The radix sort gains by it from some
// 3 M pairs on and loses below (why was not looked into).  24 bits, us, in turn / by eighths: 852 K pairs
// 57.2 / 58.4, 1.7 M 66.5 / 72.5, 2.5 M 77.4 / 79.4, 3.5 M 101.0 / 94.6, 8.5 M 188 / 160.  (The grouping below, 852 K
// tokens with their atomics: 71.3 / 70.2.)
constexpr uint32_t kSpreadTiles = 700;
__host__ __device__ inline uint32_t tile_blocks(uint32_t tiles) { return (tiles + 7u) / 8u * 8u; }
__device__ __forceinline__ uint32_t tile_of_block(uint32_t tiles)
{
    return (blockIdx.x & 7u) * ((tiles + 7u) / 8u) + (blockIdx.x >> 3);
}

// BLOCK threads take a tile of kSortTile pairs, kSortTile / BLOCK rounds of 64 per wavefront.
// Measured on 8.5 M pairs: 512 threads (74 registers, six wavefronts per SIMD) 2 us per pass faster
// than 256 (128 registers, four per SIMD); 1024 slower again.
constexpr int kScatterBlock = 512;

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void sort_scatter_kernel(SortPass s, const uint32_t *__restrict__ keys_in,
                                                             const uint32_t *__restrict__ vals_in,
                                                             uint32_t *__restrict__ keys_out,
                                                             uint32_t *__restrict__ vals_out)
{
    constexpr int ROUNDS = (int)kSortTile / BLOCK, WAVES = BLOCK / 64;
    static_assert(BLOCK >= (int)kDigits && BLOCK * ROUNDS == (int)kSortTile, "a thread per digit, whole rounds");
    __shared__ uint32_t wave_count[WAVES][kDigits];   // per wavefront: pairs of each digit so far; later: its base in the tile
    __shared__ uint32_t digit_slot[kDigits];          // first output slot of this tile's pairs of each digit; later: minus the digit's first tile-local slot
    __shared__ uint2 staged[kSortTile];               // the tile in digit order
    __shared__ uint32_t wave_total[WAVES];
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint32_t tile = s.tiles < kSpreadTiles ? blockIdx.x : tile_of_block(s.tiles);
    if (tile >= s.tiles) return;
    const uint64_t base = (uint64_t)tile * kSortTile + (uint64_t)wave * (ROUNDS * 64u);
    for (uint32_t d = t; d < (uint32_t)WAVES * kDigits; d += BLOCK) (&wave_count[0][0])[d] = 0;
    {   // a digit's pairs start after all pairs of the smaller digits, then after the digit's pairs in the tiles before
        uint32_t all, before_tiles = 0, digit_total = 0;
        if (s.few) {
            // threads t and t + 256 share digit t: the tiles with even and with odd numbers
            static_assert(BLOCK == 2 * (int)kDigits, "two threads per digit");
            uint32_t *half = reinterpret_cast<uint32_t *>(staged);         // (free until the tile is put in order)
            const uint32_t digit = t & (kDigits - 1u);
#pragma unroll 8
            for (uint32_t k = t / kDigits; k < s.tiles; k += 2u) {
                const uint32_t c = s.tile_count[(uint64_t)k * kDigits + digit];
                before_tiles += k < tile ? c : 0u;
                digit_total += c;
            }
            if (t >= kDigits) {
                half[digit] = before_tiles;
                half[kDigits + digit] = digit_total;
            }
            __syncthreads();
            if (t < kDigits) {
                before_tiles += half[t];
                digit_total += half[kDigits + t];
            }
        } else if (t < kDigits) {
            before_tiles = s.tile_count[(uint64_t)t * s.tiles + tile];
            digit_total = s.totals[t];
        }
        const uint32_t before_digits = exclusive_scan_block<BLOCK>(t < kDigits ? digit_total : 0u, wave_total, all);
        if (t < kDigits) digit_slot[t] = before_digits + before_tiles;
    }
    __syncthreads();

    uint32_t key[ROUNDS], val[ROUNDS], rank[ROUNDS];
#pragma unroll
    for (int i = 0; i < ROUNDS; ++i) {
        const uint64_t at = base + (uint32_t)i * 64u + lane;
        key[i] = at < s.n ? keys_in[at] : 0xFFFFFFFFu;
        val[i] = at < s.n ? vals_in[at] : 0u;
    }
#pragma unroll
    for (int i = 0; i < ROUNDS; ++i)
        rank[i] = rank_in_tile<8>((key[i] >> s.shift) & s.mask, base + (uint32_t)i * 64u + lane < s.n, wave_count[wave]);
    __syncthreads();
    // per digit: the tile's count, every wavefront's base inside the digit, the digit's first slot
    uint32_t in_digit = 0;
    if (t < kDigits) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const uint32_t c = wave_count[w][t];
            wave_count[w][t] = in_digit;
            in_digit += c;
        }
    }
    {   // exclusive scan of the 256 digit counts: where each digit starts in the tile.  Folded into the
        // two tables the loops below look up once per pair: a wavefront's first tile-local slot of a
        // digit, and the distance from a digit's tile-local slots to its output slots.
        uint32_t all;
        const uint32_t start = exclusive_scan_block<BLOCK>(in_digit, wave_total, all);
        if (t < kDigits) {
#pragma unroll
            for (int w = 0; w < WAVES; ++w) wave_count[w][t] += start;
            digit_slot[t] -= start;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ROUNDS; ++i) {
        const uint64_t at = base + (uint32_t)i * 64u + lane;
        if (at < s.n) {
            const uint32_t digit = (key[i] >> s.shift) & s.mask;
            staged[wave_count[wave][digit] + rank[i]] = make_uint2(key[i], val[i]);
        }
    }
    __syncthreads();
    const uint64_t tile_base = (uint64_t)tile * kSortTile;
    const uint32_t in_tile = s.n - tile_base < kSortTile ? (uint32_t)(s.n - tile_base) : kSortTile;
#pragma unroll
    for (int i = 0; i < ROUNDS; ++i) {
        const uint32_t j = (uint32_t)i * BLOCK + t;
        if (j < in_tile) {
            const uint2 kv = staged[j];
            const uint32_t digit = (kv.x >> s.shift) & s.mask;
            const uint32_t slot = digit_slot[digit] + j;      // wraps like the subtraction above: the sum is the slot
            keys_out[slot] = kv.x;
            vals_out[slot] = kv.y;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Grouping: equal keys side by side, or nearly so, for up to 2^21 pairs.
//
// The kernels that sum runs of equal keys put the positions they look at in order of 26 key bits
// themselves (Geom::window_sort), so that all they need is that the copies of a key are close together.  Two
// radix passes of 8 bits gave them that, six kernels of 5 to 10 us that a small input cannot fill.
// Here one pass places the pairs by their top GroupPlan::bits key bits, and then every tile of kSortTile
// places, which holds a bucket or a few, is ordered by the next eight bits inside LDS, with no counts of other tiles:
// a key's copies are split where a tile ends.  Runs, of 1704 K Zipf tokens (294 K distinct): 322 K after 16
// sorted bits, 333 K here with 10 bits (375 K with 8); of 118 K tokens (23.0 K) 24.5 K, and 24.9 K with 8 bits.  (What more runs
// and their order cost the atomics: see combine_scatter_kernel.)
// The keys of single-hot lookups, and of bags of many tokens, are hashed where they are needed: no kernel writes them
// first, and their array has room for counts of 10 bits.
//   count    as above, the counts tile by tile
//   offsets  one wavefront per 64 digits and sixteenth of the tiles (left out up to kFewTiles tiles)
//   scatter  as above, writing (key, value) words
//   local    a tile by the next bits
// Keys and sort, us: 1704 K lookups 61 -> 41, 852 K 46 -> 29; bags, 118 K tokens 33 -> 24.  Tiles of 8192: 1 to
// 3 us longer for as many runs less.  Ordered by the whole span of their keys instead of the bits below the
// bucket's: the same for the atomics, and the regions' kernel 10 us longer (neighbours then write the same
// regions at a time).  Every step is stable.
// ---------------------------------------------------------------------------------------------
struct GroupPlan {
    uint32_t n, tiles, few;      // as in SortPass (few: with 256 digits only)
    uint32_t shift;              // first key bit of the digit; it has log2(DIG) bits, the topmost that matter
    uint32_t local_shift, local_mask;
    uint32_t *tile_count;        // [tiles][DIG]
    uint32_t *totals;            // [DIG]
    uint32_t F, F_recip;         // tables
    uint32_t row_values;         // 1: the values are the tokens' rows, 0: their positions
};

constexpr int kGroupBlock = 512;
constexpr uint32_t kGroupMostTiles = 512;     // 2^21 pairs
constexpr int kGroupOffsetsBlock = 1024;
constexpr int kGroupOffsetsRows = (int)kGroupMostTiles / (kGroupOffsetsBlock / 64);

// Where a kernel has its pairs from: single-hot ids (the row is the position), ids and their rows, two arrays, or
// (the local step) the words that the step before wrote.
enum GroupSource { GROUP_LOOKUPS, GROUP_BAGS, GROUP_PAIRS, GROUP_LOCAL };

// The keys of a thread's ROUNDS tokens base, base + step, .. and, unless they come from an array, their rows.
template <GroupSource FROM, int ROUNDS>
__device__ __forceinline__ void group_keys(const GroupPlan &s, const Params &p, const int64_t *__restrict__ indices,
                                           const uint32_t *__restrict__ bag_rows, const uint32_t *__restrict__ keys, uint32_t base, uint32_t step,
                                           uint32_t (&key)[ROUNDS], uint32_t (&row)[ROUNDS])
{
    if constexpr (FROM == GROUP_PAIRS) {
#pragma unroll
        for (int i = 0; i < ROUNDS; ++i) key[i] = base + (uint32_t)i * step < s.n ? keys[base + (uint32_t)i * step] : 0u;
    } else {
        int64_t x[ROUNDS];
#pragma unroll
        for (int i = 0; i < ROUNDS; ++i) {
            const uint32_t at = base + (uint32_t)i * step;
            x[i] = at < s.n ? indices[at] : 0;
            row[i] = FROM == GROUP_LOOKUPS ? at : (at < s.n ? bag_rows[at] : 0u);
        }
#pragma unroll
        for (int i = 0; i < ROUNDS; ++i) key[i] = sort_key(p, x[i], mod_m(row[i], s.F, s.F_recip));
    }
}

template <int DIG, GroupSource FROM>
__global__ __launch_bounds__(kGroupBlock) void group_count_kernel(GroupPlan s, Params p, const int64_t *__restrict__ indices,
                                                                  const uint32_t *__restrict__ bag_rows, const uint32_t *keys,
                                                                  TableArgs tab, uint32_t n_tab, uint2 *__restrict__ tables,
                                                                  Clear clear)
{
    constexpr int ROUNDS = (int)kSortTile / kGroupBlock;
    __shared__ uint32_t h[DIG];
    if (FROM == GROUP_LOOKUPS && blockIdx.x >= clear.work) {
        fill_u32<kGroupBlock>(clear.dst, clear.n, 0u, blockIdx.x - clear.work);
        return;
    }
    if (FROM == GROUP_LOOKUPS && blockIdx.x == 0 && threadIdx.x < n_tab) tables[threadIdx.x] = make_uint2(tab.col[threadIdx.x], tab.dim[threadIdx.x]);
    for (uint32_t d = threadIdx.x; d < (uint32_t)DIG; d += kGroupBlock) h[d] = 0;
    __syncthreads();
    const uint32_t base = blockIdx.x * kSortTile;              // (at most 2^21)
    uint32_t k[ROUNDS], row[ROUNDS];
    group_keys<FROM, ROUNDS>(s, p, indices, bag_rows, keys, base + threadIdx.x, kGroupBlock, k, row);
#pragma unroll
    for (int i = 0; i < ROUNDS; ++i)
        if (base + (uint32_t)i * kGroupBlock + threadIdx.x < s.n) atomicAdd(&h[(k[i] >> s.shift) & (DIG - 1u)], 1u);
    __syncthreads();
    for (uint32_t d = threadIdx.x; d < (uint32_t)DIG; d += kGroupBlock) s.tile_count[(uint64_t)blockIdx.x * DIG + d] = h[d];
}

// counts -> the digit's pairs in the tiles before; the digit's total.  Launched with DIG / 64 workgroups.
template <int DIG>
__global__ __launch_bounds__(kGroupOffsetsBlock) void group_offsets_kernel(GroupPlan s)
{
    constexpr uint32_t WAVES = kGroupOffsetsBlock / 64;
    __shared__ uint32_t part[WAVES][64];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, digit = blockIdx.x * 64u + lane;
    const uint32_t rows = (s.tiles + WAVES - 1u) / WAVES, first = wave * rows;        // rows <= kGroupOffsetsRows
    uint32_t c[kGroupOffsetsRows], sum = 0;
#pragma unroll
    for (uint32_t k = 0; k < (uint32_t)kGroupOffsetsRows; ++k) {
        c[k] = k < rows && first + k < s.tiles ? s.tile_count[(uint64_t)(first + k) * DIG + digit] : 0u;
        sum += c[k];
    }
    part[wave][lane] = sum;
    __syncthreads();
    uint32_t at = 0;
#pragma unroll
    for (uint32_t w = 0; w < WAVES; ++w) at += w < wave ? part[w][lane] : 0u;
    if (wave == WAVES - 1u) s.totals[digit] = at + sum;
#pragma unroll
    for (uint32_t k = 0; k < (uint32_t)kGroupOffsetsRows; ++k) {
        if (k < rows && first + k < s.tiles) s.tile_count[(uint64_t)(first + k) * DIG + digit] = at;
        at += c[k];
    }
}

// The local step: the tile stays where it is, by the bits below; pairs come as words and leave in two arrays.
// Otherwise they leave as words.
template <int DIG, GroupSource FROM>
__global__ __launch_bounds__(kGroupBlock) void group_scatter_kernel(GroupPlan s, Params p, const int64_t *__restrict__ indices,
                                                                    const uint32_t *__restrict__ bag_rows,
                                                                    uint32_t *__restrict__ keys, uint32_t *__restrict__ vals,
                                                                    uint2 *__restrict__ words)
{
    constexpr bool LOCAL = FROM == GROUP_LOCAL;
    constexpr int BLOCK = kGroupBlock, ROUNDS = (int)kSortTile / BLOCK, WAVES = BLOCK / 64;
    constexpr int BITS = DIG == 256 ? 8 : 10;
    static_assert(DIG == 256 || DIG == 1024, "digits of 8 or 10 bits");
    static_assert(!LOCAL || DIG == 256, "the local step has one form");
    constexpr uint32_t PER = (DIG + BLOCK - 1) / BLOCK;         // digits per thread (threads past DIG have none)
    __shared__ uint32_t wave_count[WAVES][DIG];
    __shared__ uint32_t digit_slot[LOCAL ? 1 : DIG];
    __shared__ uint2 staged[kSortTile];
    __shared__ uint32_t wave_total[WAVES];
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint32_t tile = LOCAL ? blockIdx.x : tile_of_block(s.tiles);
    if (tile >= s.tiles) return;
    const uint32_t base = tile * kSortTile + wave * (ROUNDS * 64u);
    const uint32_t shift = LOCAL ? s.local_shift : s.shift, mask = LOCAL ? s.local_mask : DIG - 1u;

    uint32_t key[ROUNDS], val[ROUNDS], rank[ROUNDS];
    if constexpr (LOCAL) {
#pragma unroll
        for (int i = 0; i < ROUNDS; ++i) {
            const uint32_t at = base + (uint32_t)i * 64u + lane;
            const uint2 w = at < s.n ? words[at] : make_uint2(0u, 0u);
            key[i] = w.x;
            val[i] = w.y;
        }
    } else {
        group_keys<FROM, ROUNDS>(s, p, indices, bag_rows, keys, base + lane, 64u, key, val);
#pragma unroll
        for (int i = 0; i < ROUNDS; ++i) {
            const uint32_t at = base + (uint32_t)i * 64u + lane;
            if constexpr (FROM == GROUP_PAIRS) val[i] = at < s.n ? vals[at] : 0u;
            else if (FROM == GROUP_BAGS && !s.row_values) val[i] = at;
        }
    }
    for (uint32_t d = t; d < (uint32_t)(WAVES * DIG); d += BLOCK) (&wave_count[0][0])[d] = 0;
    if constexpr (!LOCAL) {   // a digit's pairs start after all pairs of the smaller digits, then after the digit's pairs in the tiles before
        uint32_t before_tiles[PER], digit_total[PER], all, sum = 0;
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) before_tiles[q] = digit_total[q] = 0;
        if (DIG == 256 && s.few) {
            static_assert(BLOCK == 512, "two threads per digit of eight bits");
            uint32_t *half = reinterpret_cast<uint32_t *>(staged);             // (free until the tile is put in order)
            const uint32_t digit = t & 255u;
#pragma unroll 8
            for (uint32_t k = t >> 8; k < s.tiles; k += 2u) {
                const uint32_t c = s.tile_count[(uint64_t)k * DIG + digit];
                before_tiles[0] += k < tile ? c : 0u;
                digit_total[0] += c;
            }
            if (t >= 256u) {
                half[digit] = before_tiles[0];
                half[256u + digit] = digit_total[0];
            }
            __syncthreads();
            if (t < 256u) {
                before_tiles[0] += half[t];
                digit_total[0] += half[256u + t];
            }
        } else if (t * PER < (uint32_t)DIG) {
#pragma unroll
            for (uint32_t q = 0; q < PER; ++q) {
                before_tiles[q] = s.tile_count[(uint64_t)tile * DIG + t * PER + q];
                digit_total[q] = s.totals[t * PER + q];
            }
        }
        if (t * PER < (uint32_t)DIG) {
#pragma unroll
            for (uint32_t q = 0; q < PER; ++q) sum += digit_total[q];
        }
        uint32_t at = exclusive_scan_block<BLOCK>(sum, wave_total, all);
        if (t * PER < (uint32_t)DIG) {
#pragma unroll
            for (uint32_t q = 0; q < PER; ++q) {
                digit_slot[t * PER + q] = at + before_tiles[q];
                at += digit_total[q];
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ROUNDS; ++i)
        rank[i] = rank_in_tile<BITS>((key[i] >> shift) & mask, base + (uint32_t)i * 64u + lane < s.n, wave_count[wave]);
    __syncthreads();
    // as in sort_scatter_kernel: every wavefront's first tile-local slot of a digit, and the distance from a
    // digit's tile-local slots to its output slots
    uint32_t in_digit[PER], sum = 0, all;
    if (t * PER < (uint32_t)DIG) {
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) {
            in_digit[q] = 0;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                const uint32_t c = wave_count[w][t * PER + q];
                wave_count[w][t * PER + q] = in_digit[q];
                in_digit[q] += c;
            }
            sum += in_digit[q];
        }
    }
    uint32_t start = exclusive_scan_block<BLOCK>(sum, wave_total, all);
    if (t * PER < (uint32_t)DIG) {
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) {
#pragma unroll
            for (int w = 0; w < WAVES; ++w) wave_count[w][t * PER + q] += start;
            if constexpr (!LOCAL) digit_slot[t * PER + q] -= start;
            start += in_digit[q];
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ROUNDS; ++i)
        if (base + (uint32_t)i * 64u + lane < s.n)
            staged[wave_count[wave][(key[i] >> shift) & mask] + rank[i]] = make_uint2(key[i], val[i]);
    __syncthreads();
    const uint32_t tile_base = tile * kSortTile;
    const uint32_t in_tile = s.n - tile_base < kSortTile ? s.n - tile_base : kSortTile;
#pragma unroll
    for (int i = 0; i < ROUNDS; ++i) {
        const uint32_t j = (uint32_t)i * BLOCK + t;
        if (j < in_tile) {
            const uint2 kv = staged[j];
            if constexpr (LOCAL) {
                keys[tile_base + j] = kv.x;
                vals[tile_base + j] = kv.y;
            } else {
                words[digit_slot[(kv.x >> shift) & mask] + j] = kv;      // wraps like the subtraction above: the sum is the slot
            }
        }
    }
}

}  // namespace robe
