// Single-hot forward of small blocks (Eq. 4 of the paper), every distinct token gathered once.
//
// With blocks of one or two floats a lookup reads d / Z lines of 128 bytes for a row of 4d: 852 K lookups of
// 128 single floats fetch 5.7 GB through the fabric, 1116 us, though most of them repeat a token that another
// lookup has.  Rows of equal tokens are equal bits, so one lookup of every token gathers and the others copy
// its row out of the output, four lines instead of 128:
//
//   D1 find    lookups table by table, a tile of kDistinctTile per workgroup: equal tokens of a tile are found by
//              a hash table in LDS; the first of each enters a hash table in memory, or finds there who
//              came first in another tile (where the tile has repeats enough).  rep[position]: the row that
//              gathers for it.
//   D2 gather  the rows that gather for themselves, as single_hot_kernel does.
//   D3 copy    the others.
//   D4         the last samples' rows, plainly: rep lies there until now.
//
// The forward call has no workspace, but `out` is its own to write: the hash table lies at its front until D2,
// rep at its end until D4, whose rows no other lookup copies from.  Tokens are the same when the token part of h
// is (and of g, with the sign on): then every offset and every sign is.
//
// 852 K Zipf lookups over 26 tables, d = 128, 100 MB array: Z = 1 1092 -> 574 us (gather 433, 2.9 GB of lines read
// and 0.1 GB written at 6.9 TB/s; copy 98, find 23, the last samples 14, clearing the table 6), Z = 2 543 -> 373.
// Ids that never repeat pay D1 and the empty D3: Z = 1 1976 -> 2007, Z = 2 1060 -> 1086 (2054 and 1130 with every token
// entered in memory, see distinct_least_repeats).  Tiles of 2048 lookups: of 4096
// 208 K lookups take 212 us instead of 203, of 1024 852 K 576 instead of 570.
#pragma once
#include "robe_kernels.h"

namespace robe {

constexpr uint32_t kDistinctBlock = 512;
constexpr uint32_t kDistinctPer = 4;
constexpr uint32_t kDistinctTile = kDistinctBlock * kDistinctPer;
constexpr uint32_t kDistinctSlots = 2u * kDistinctTile;      // of the table in LDS: half of them stay free
constexpr uint32_t kDistinctProbes = 64;                     // places looked at in the table in memory; then the lookup gathers for itself
constexpr uint32_t kDistinctRows = 32;                       // positions of a wavefront in D2 and D3

struct DistinctPlan {
    uint32_t n;                // positions = F * batch, table by table: f * batch + b (the samples before those of D4)
    uint32_t batch, batch_recip, F;
    uint64_t *table;           // (th + 1) << 32 | row; 0: free
    uint32_t mask;             // its places - 1, a power of two and at least 2n places
    uint32_t *rep;             // [n]
    uint32_t least_repeats;    // see distinct_least_repeats
};

// A tile with fewer repeated lookups than this stays out of the table in memory, whose atomics are most of what the
// lists cost where hardly any id repeats (D1 of 852 K lookups that differ 58 us).  If the pairs of a whole table are
// equal as often as those of a tile, the share of its lookups that repeat is repeats * batch / kDistinctTile^2: a
// quarter, below which they gain nothing, Z = 4 least of all.  Up to tiles a quarter of whose own lookups repeat.
__host__ __device__ inline uint32_t distinct_least_repeats(uint64_t batch)
{
    const uint64_t least = (uint64_t)kDistinctTile * kDistinctTile / 4u / batch;
    return least < 1u ? 1u : (least < kDistinctTile / 4u ? (uint32_t)least : kDistinctTile / 4u);
}

// The lists of robe_forward_places.h, which D1 begins.
struct PlacePlan {
    uint32_t buckets, bucket_shift;      // of r = th mod m; bucket_shift: log2 of the slots of one
    uint32_t *counts, *starts;           // [buckets], [buckets + 1]: entries of a bucket, entries before it
    uint32_t most;                       // entries there is room for, a multiple of 64
    uint32_t least;                      // fewer entries are gathered
    uint32_t *entries;                   // [most + kPlacePad] the entries by bucket, see place_entry
    uint32_t r_bits, r_mask;             // bits of r; 2^r_bits - 1
    uint32_t *row;                       // [most] their rows of out
    uint32_t segments, segment_shift;    // the free rows lie in so many lists (a power of two), by D1's workgroups in turn; tile t has the
    uint32_t segment_rows;               // next 64 of list t mod segments.  Room of each list, a multiple of 64
    uint32_t *free_count;                // [segments] rows of each list
    uint32_t *total;                     // lookups that gather for themselves
    uint32_t *pages;                     // [tiles][64] the free rows, as multiples of 64 floats: row * page_elems
    uint32_t out_bytes;
    uint32_t page_elems, page_recip;     // d / 64; ceil(2^16 / page_elems): i / page_elems = i * page_recip >> 16 for i < 512
    uint32_t *used;                      // entries that have room and whose tiles find free rows; the others' rows are gathered.  Behind it: whether there are others
    uint32_t tail, ends;                 // rows from n on that have a word in tail_rep; the rows after those, which hold the words
    uint32_t *tail_rep;                  // [ends][d], 2^tail_shift words of each: see place_last_kernel
    uint32_t tail_shift;
};
constexpr uint32_t kLastMost = 32;             // most words of such a row, 1 << tail_shift
constexpr uint32_t kPlacePad = 256;            // words past the end of the lists that F3 may read
constexpr uint32_t kPlaceSelf = 0x80000000u;   // in rep: the row gathers for itself, and the lower bits say which of its bucket it is

// The row b * F + f of a position, and its table.
__device__ __forceinline__ uint32_t distinct_row(const DistinctPlan &s, uint32_t q, uint32_t &f)
{
    f = div_m(q, s.batch, s.batch_recip);
    return (q - f * s.batch) * s.F + f;
}

// Where a token's walk through the table in memory starts (modulo its places).
__device__ __forceinline__ uint32_t table_place(uint32_t h, uint32_t g) { return ((h ^ (g << 7)) * 0x85EBCA6Bu) ^ (h >> 13); }

template <bool SIGN, bool PLACES>
__global__ __launch_bounds__(kDistinctBlock) void distinct_find_kernel(Params p, DistinctPlan s, PlacePlan lists, const int64_t *__restrict__ indices)
{
    __shared__ uint32_t place[kDistinctSlots];               // tile-local lookup + 1; 0: free
    __shared__ uint32_t th[kDistinctTile], rep[kDistinctTile];
    __shared__ uint32_t tg[SIGN ? kDistinctTile : 1];
    __shared__ uint32_t repeats;                             // lookups of the tile whose token another one of it has
    const uint32_t t = threadIdx.x, base = blockIdx.x * kDistinctTile;
    if (t == 0) repeats = 0;
    for (uint32_t i = t; i < kDistinctSlots; i += kDistinctBlock) place[i] = 0;
    uint32_t row[kDistinctPer], f[kDistinctPer];
    int64_t x[kDistinctPer];
#pragma unroll
    for (uint32_t i = 0; i < kDistinctPer; ++i) {
        const uint32_t q = base + i * kDistinctBlock + t;
        row[i] = f[i] = 0;
        x[i] = 0;
        if (q < s.n) {
            row[i] = distinct_row(s, q, f[i]);
            x[i] = indices[row[i]];
        }
    }
    uint32_t h[kDistinctPer], g[kDistinctPer], lead[kDistinctPer];
#pragma unroll
    for (uint32_t i = 0; i < kDistinctPer; ++i) {
        const uint32_t j = i * kDistinctBlock + t;
        h[i] = staged_h(p, x[i], f[i]);
        g[i] = SIGN ? staged_g(p, x[i], f[i]) : 0u;
        th[j] = h[i];
        if constexpr (SIGN) tg[j] = g[i];
    }
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < kDistinctPer; ++i) {
        const uint32_t j = i * kDistinctBlock + t;
        lead[i] = j;
        if (base + j < s.n) {
            // (kDistinctTile entries at most in twice as many places: the walk ends)
            for (uint32_t at = ((h[i] ^ g[i]) * 0x9E3779B1u) % kDistinctSlots;; at = (at + 1u) % kDistinctSlots) {
                uint32_t there = __hip_atomic_load(&place[at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (there == 0) there = atomicCAS(&place[at], 0u, j + 1u);
                if (there == 0) break;
                if (th[there - 1u] == h[i] && (!SIGN || tg[there - 1u] == g[i])) {
                    lead[i] = there - 1u;
                    break;
                }
            }
        }
        const uint64_t again = __ballot(lead[i] != j);
        if ((t & 63u) == 0) atomicAdd(&repeats, (uint32_t)__popcll(again));
    }
    __syncthreads();
    const bool enter = repeats >= s.least_repeats;          // uniform over the workgroup
#pragma unroll
    for (uint32_t i = 0; i < kDistinctPer; ++i) {
        const uint32_t j = i * kDistinctBlock + t;
        if (base + j >= s.n || lead[i] != j) continue;
        uint32_t mine = row[i];
        if (!enter) {
            rep[j] = mine;
            continue;
        }
        const uint64_t entry = ((uint64_t)(h[i] + 1u) << 32) | row[i];
        uint32_t at = table_place(h[i], g[i]);
        for (uint32_t tries = 0; tries < kDistinctProbes; ++tries, ++at) {
            uint64_t *slot = s.table + (at & s.mask);
            uint64_t there = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // (on failure `there` becomes what the place holds)
            if (there == 0 && __hip_atomic_compare_exchange_strong(slot, &there, entry, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
            if ((uint32_t)(there >> 32) != h[i] + 1u) continue;
            const uint32_t first = (uint32_t)there;
            if constexpr (SIGN) {
                if (staged_g(p, indices[first], first % s.F) != g[i]) continue;
            }
            mine = first;
            break;
        }
        rep[j] = mine;
    }
    __syncthreads();
    if constexpr (!PLACES) {
#pragma unroll
        for (uint32_t i = 0; i < kDistinctPer; ++i) {
            const uint32_t q = base + i * kDistinctBlock + t;
            if (q < s.n) s.rep[q] = rep[lead[i]];
        }
    } else {
        __shared__ uint32_t free_n[kDistinctPer * kDistinctBlock / 64u], free_first;
        const uint32_t lane = t & 63u, wave = t >> 6;
        bool free[kDistinctPer];
        uint32_t before[kDistinctPer];
#pragma unroll
        for (uint32_t i = 0; i < kDistinctPer; ++i) {
            const uint32_t q = base + i * kDistinctBlock + t;
            free[i] = false;
            if (q < s.n) {
                uint32_t w = rep[lead[i]];
                free[i] = w != row[i];
                if (!free[i]) w = kPlaceSelf | atomicAdd(&lists.counts[mod_m(h[i], p.m, p.m_recip) >> lists.bucket_shift], 1u);
                s.rep[q] = w;
            }
            const uint64_t mask = __ballot(free[i]);
            before[i] = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (lane == 0) free_n[i * (kDistinctBlock / 64u) + wave] = (uint32_t)__popcll(mask);
        }
        __syncthreads();
        const uint32_t seg = blockIdx.x & (lists.segments - 1u);
        uint32_t all = 0, mine[kDistinctPer];
#pragma unroll
        for (uint32_t k = 0; k < kDistinctPer * kDistinctBlock / 64u; ++k) {
#pragma unroll
            for (uint32_t i = 0; i < kDistinctPer; ++i)
                if (k == i * (kDistinctBlock / 64u) + wave) mine[i] = all;
            all += free_n[k];
        }
        if (t == 0) {
            free_first = atomicAdd(&lists.free_count[seg], all);
            atomicAdd(lists.total, min(kDistinctTile, s.n - base) - all);
        }
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < kDistinctPer; ++i) {
            const uint32_t k = free_first + mine[i] + before[i];
            if (free[i] && k < lists.segment_rows) lists.pages[(((k >> 6) << lists.segment_shift) + seg) * 64u + (k & 63u)] = row[i] * lists.page_elems;
        }
    }
}

// Bring the values of the lanes with `yes` to the front, in order; how many there are.
__device__ __forceinline__ uint32_t to_front(bool yes, uint64_t mask, uint32_t &a, uint32_t &b, uint32_t &c)
{
    const uint32_t lo = (uint32_t)mask, hi = (uint32_t)(mask >> 32);
    const uint32_t count = (uint32_t)__popcll(mask), before = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
    const uint32_t lane = threadIdx.x & 63u;
    const int to = (int)((yes ? before : count + lane - before) << 2);      // the other lanes fill the places behind
    a = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)a);
    b = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)b);
    c = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)c);
    return count;
}

// The rows of the lanes with `self` (mask: their ballot).
template <int V, bool CONSEC, bool SIGN, typename AT>
__device__ __forceinline__ void gather_rows(const Params &p, const Geom &q, bool self, uint64_t mask, uint32_t row, uint32_t th, uint32_t tg,
                                            const AT *__restrict__ array, float *__restrict__ out)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t n = to_front(self, mask, row, th, tg);
    const uint32_t grp = lane & (q.G - 1u), sub = lane >> q.g_shift, step = 64u >> q.g_shift;
    Lane<V, CONSEC, SIGN> L;
    L.init(p, q, grp);
    for (uint32_t r = 0; r < n; r += step * kUnroll) {         // trip count uniform over the wavefront
        uint32_t k[kUnroll];
        bool live[kUnroll];
        float v[kUnroll][V];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const uint32_t from = r + (uint32_t)u * step + sub;
            live[u] = from < n;
            const int src = (int)(live[u] ? from : 0u);
            k[u] = __shfl(row, src);
            L.gather(p, array, __shfl(th, src), SIGN ? __shfl(tg, src) : 0u, v[u]);      // the first stands in for dead slots
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
            if (live[u]) store_row<V, CONSEC>(out + (uint64_t)k[u] * p.d, q, grp, v[u]);
    }
}

template <int V, bool CONSEC, bool SIGN, typename AT>
__global__ __launch_bounds__(kRowBlock) void distinct_gather_kernel(Params p, Geom q, DistinctPlan s, const AT *__restrict__ array,
                                                                    const int64_t *__restrict__ indices, float *__restrict__ out)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t at = blockIdx.x * kDistinctRows + lane;
    uint32_t f = 0, row = 0, th = 0, tg = 0;
    bool self = false;
    if (lane < kDistinctRows && at < s.n) {
        row = distinct_row(s, at, f);
        self = s.rep[at] == row;
        if (self) {
            const int64_t x = indices[row];
            th = staged_h(p, x, f);
            if constexpr (SIGN) tg = staged_g(p, x, f);
        }
    }
    gather_rows<V, CONSEC, SIGN>(p, q, self, __ballot(self), row, th, tg, array, out);
}

// The lanes with `copy`: row `from` of out to row `row`.  W: floats per lane and access (4 where rows are aligned for it).  A row
// is G lanes' work, in several steps if longer.
template <int W>
__device__ __forceinline__ void copy_rows(bool copy, uint32_t row, uint32_t from, uint32_t d, uint32_t g_shift, float *__restrict__ out)
{
    typedef typename Vec<W>::A T;
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t unused = 0;
    const uint32_t n = to_front(copy, __ballot(copy), row, from, unused);
    const uint32_t G = 1u << g_shift, grp = lane & (G - 1u), sub = lane >> g_shift, step = 64u >> g_shift;
    for (uint32_t r = 0; r < n; r += step * kUnroll) {         // trip count uniform over the wavefront
        uint32_t to[kUnroll], src[kUnroll];
        bool live[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const uint32_t j = r + (uint32_t)u * step + sub;
            live[u] = j < n;
            to[u] = __shfl(row, (int)(live[u] ? j : 0u));
            src[u] = __shfl(from, (int)(live[u] ? j : 0u));
        }
        for (uint32_t i = grp * W; i < d; i += G * W) {
            T v[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) v[u] = *reinterpret_cast<const T *>(out + (uint64_t)src[u] * d + i);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                if (live[u]) __builtin_nontemporal_store(v[u], reinterpret_cast<T *>(out + (uint64_t)to[u] * d + i));
        }
    }
}

template <int W>
__global__ __launch_bounds__(kRowBlock) void distinct_copy_kernel(DistinctPlan s, uint32_t d, uint32_t g_shift, uint32_t per_xcd, float *__restrict__ out)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t block = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;      // an eighth of the tables' order per XCD, see RowWalk
    const uint64_t at = (uint64_t)block * kDistinctRows + lane;
    uint32_t f = 0, row = 0, from = 0;
    bool copy = false;
    if (lane < kDistinctRows && at < s.n) {
        row = distinct_row(s, (uint32_t)at, f);
        from = s.rep[at];
        copy = from != row && from < s.n;                      // (rows of these samples are below n)
    }
    copy_rows<W>(copy, row, from, d, g_shift, out);
}

}  // namespace robe
