// Single-hot forward of blocks of one or two floats on arrays that no L2 holds (Eq. 4 of the paper): the distinct
// tokens in the order of the places they read.
//
// Gathered token by token, every element of a distinct token is a line of 128 bytes (robe_forward_distinct.h): 178 K
// distinct tokens of 128 single floats read 2.9 GB out of an array of 100 MB, each of its lines 29 times.  But block
// c of a token with key th starts at ((th + Ch c mod P) mod P) mod m: with r = th mod m that is r + Ch c, or
// r + Ch c - P where the sum passed P, modulo m.  So the tokens whose block c lies in a region of the array have r in
// one window, or in a second one a fixed distance away, and if the tokens lie by r, a region's workgroup reads its
// part of the array once, finds for every chunk the tokens of two windows, and serves them out of LDS:
//
//   D1 find     as in robe_forward_distinct.h; a lookup that gathers for itself also counts in a bucket of r (an
//               integer atomic, which says how many were there before), the others' rows are listed as free.
//   F1 scan     first entry of every bucket, if there are entries enough.  Beside it the tokens of the last samples, which hold the
//               lists, are looked up in D1's table.
//   F2 place    the lookups that gather for themselves enter their key and row in the list.
//   F3 regions  a workgroup per 2^14 slots.  What it finds leaves in tiles of 64 entries, element by element
//               (consecutive lanes write consecutive words).  A tile lies in 64 of the free rows, which no one else
//               needs before D3.
//   F4 rows     a workgroup per tile turns it round and writes the tokens' rows.
//   D3 copy     as there.
//   D4 last     the last samples' rows: copied where F1 found the token, else gathered.
//
// The lists (two and a half words a lookup) lie in the last samples' rows until D4.  What has no room - ids that hardly
// repeat leave few rows free - is gathered by F2 as D2 does there, and so are all where there are too few entries (PlacePlan::least):
// such a call costs what F1, F3 and F4 take to start and D1's counts, 10 to 15 us more than one without lists (up to 33 at 250 M slots).  It was a
// quarter of the call and more while F2 gathered 64 rows a wavefront and D4 all of its rows: uniform ids, d = 128, gathered / by
// place: Z = 1, 413 K lookups of 31 K distinct tokens, 53 M slots 192 / 274 us then, 189 / 202 now; Z = 2, 858 K of 62 K, 55 M 244 / 356,
// 245 / 260; Z = 1, 780 K of 31 K, 100 M 228 / 344, 229 / 240.
//
// 852 K Zipf lookups over 26 tables (178 K distinct tokens), d = 128, 100 MB array, Z = 1: 588 -> some 262 us (D1 30 instead
// of 24, F1 8, F2 10, F3 84, F4 34, D3 72 instead of 99, D4 17 instead of 15 (29 with all of its rows gathered), clearing 6, where
// the gather took 440).  F3 has three parts that hardly overlap: its region's load 35, the walk 32, the stores 28 (161 MB, as a line's
// elements come from two windows).  Forms tried beside an F3 of 95: a hash and a page of its own for every entry instead of keys that
// compare packed and one page a tile 112; every workgroup three regions, the next loaded during the walk 100 (the walk's loads then wait
// for it).  Beside one of 78 (the same lookups, the array in the last-level cache): regions of 2^13 floats 123; of 2^15, one workgroup
// per CU, 81.  With short windows (d = 512, Z = 1, 78 K lookups) those take 348 and 127 us against 185.
#pragma once
#include "robe_backward_regions.h"
#include "robe_forward_distinct.h"

namespace robe {

constexpr uint32_t kPlaceShift = 14;          // floats of a region: 64 KB of LDS, two workgroups per CU
constexpr uint32_t kPlaceBlock = 1024;
constexpr uint32_t kPlaceAhead = 3;           // tiles whose loads are requested together
constexpr uint32_t kPlaceMostSegments = 32;
constexpr uint32_t kPlaceTurn = 64;           // elements of a tile turned round at a time (128, more LDS for fewer steps: 38 us instead of 33)
constexpr uint32_t kPlaceMostD = 512;
constexpr uint32_t kLastRows = 2;             // rows of a wavefront of D4: most are copied, all at once

constexpr size_t kPlaceLds = ((size_t)4 << kPlaceShift) + 16;       // of F3: the region, and a float past it for blocks of two

// The entry of a key th = q m + r: q above the bits of r.  Entries compare as their keys do.
__device__ __forceinline__ uint32_t place_entry(const Params &p, const PlacePlan &s, uint32_t th, uint32_t r)
{
    return (div_m(th, p.m, p.m_recip) << s.r_bits) | r;
}

// For threads t < 1024 of a workgroup: the entries in use, see PlacePlan::used.
__device__ __forceinline__ uint32_t places_used(const PlacePlan &s, uint32_t total, uint32_t lane)
{
    uint32_t tiles = lane < s.segments ? min(s.free_count[lane], s.segment_rows) / 64u : 0xFFFFFFFFu;
#pragma unroll
    for (int x = 1; x < 64; x <<= 1) tiles = min(tiles, (uint32_t)__shfl_xor((int)tiles, x));
    const uint32_t room = 64u * s.segments * tiles;                       // <= most + 64 * segments
    const uint32_t used = min(min(total, s.most), room);
    return used >= s.least ? used : 0u;
}

// The word of row n + i, i < tail: the row that has its token, or kPlaceSelf.
__device__ __forceinline__ uint32_t *tail_word(const PlacePlan &s, uint32_t d, uint32_t i)
{
    return s.tail_rep + (uint64_t)(i >> s.tail_shift) * d + (i & ((1u << s.tail_shift) - 1u));
}

// Workgroup 0 scans, the others look the last samples' tokens up: the table is whole now, and still there.
template <bool SIGN>
__global__ __launch_bounds__(kScanThreads) void place_scan_kernel(Params p, DistinctPlan d, PlacePlan s, uint32_t F_recip, const int64_t *__restrict__ indices)
{
    __shared__ uint32_t wave_sum[kScanThreads / 64u];
    if (blockIdx.x == 0) {
        const uint32_t total = *s.total, used = places_used(s, total, threadIdx.x & 63u);
        if (threadIdx.x == 0) {
            s.used[0] = used;
            s.used[1] = used < total;
        }
        uint32_t c[kScanPer];
        if (used != 0) scan_counts(s.counts, s.starts, s.buckets, c, wave_sum);
        return;
    }
    const uint32_t i = (blockIdx.x - 1u) * kScanThreads + threadIdx.x;
    if (i >= s.tail) return;
    const uint32_t row = d.n + i, f = mod_m(row, d.F, F_recip);
    const int64_t x = indices[row];
    const uint32_t th = staged_h(p, x, f), tg = SIGN ? staged_g(p, x, f) : 0u;
    uint32_t found = kPlaceSelf, at = table_place(th, tg);
    for (uint32_t tries = 0; tries < kDistinctProbes; ++tries, ++at) {
        const uint64_t there = d.table[at & d.mask];
        if (there == 0) break;
        if ((uint32_t)(there >> 32) != th + 1u) continue;
        const uint32_t first = (uint32_t)there;
        if constexpr (SIGN) {
            if (staged_g(p, indices[first], mod_m(first, d.F, F_recip)) != tg) continue;
        }
        found = first;
        break;
    }
    *tail_word(s, p.d, i) = found;
}

template <int V, bool CONSEC, bool SIGN, typename AT>
__global__ __launch_bounds__(kRowBlock) void place_tokens_kernel(Params p, Geom q, DistinctPlan d, PlacePlan s, const AT *__restrict__ array,
                                                                 const int64_t *__restrict__ indices, float *__restrict__ out)
{
    const uint32_t lane = threadIdx.x & 63u, used = *s.used;
    // nothing to gather: 64 positions a wavefront, and half the wavefronts have none; else as D2 of robe_forward_distinct.h
    const uint32_t per = s.used[1] == 0 ? kRowBlock : kDistinctRows;
    const uint64_t at = (uint64_t)blockIdx.x * per + lane;
    uint32_t f = 0, row = 0, th = 0, tg = 0;
    bool self = false;
    if (lane < per && at < d.n) {
        row = distinct_row(d, (uint32_t)at, f);
        const uint32_t w = d.rep[at];
        self = (w & kPlaceSelf) != 0;
        if (self) {
            const int64_t x = indices[row];
            th = staged_h(p, x, f);
            const uint32_t r = mod_m(th, p.m, p.m_recip), k = used ? s.starts[r >> s.bucket_shift] + (w & ~kPlaceSelf) : 0u;
            if (k < used) {
                s.entries[k] = place_entry(p, s, th, r);
                s.row[k] = row;
                self = false;
            } else if constexpr (SIGN) {
                tg = staged_g(p, x, f);
            }
        }
    }
    const uint64_t plain = __ballot(self);
    if (plain) gather_rows<V, CONSEC, SIGN>(p, q, self, plain, row, th, tg, array, out);
}

// Up to kPlaceAhead tiles of a window: meant are the entries e with 4 * (r + the window's delta) below four times the region's
// length and e - base below width (per tile: 0 for one that is not the window's).
template <int Z>
struct PlaceBatch {
    uint32_t entry[kPlaceAhead];
    uint32_t page[Z];                            // of tile u in lane u: see PlacePlan::pages, of the chunk's element j
    uint32_t delta, base, width[kPlaceAhead], in_page[Z];
};

// What a lane holds of its window: the tiles of the entries whose block of one chunk starts in the region, of the keys whose
// sum with the chunk's term stays below P or of those that pass it: [first, first + count), whose r goes from lo on, and
// the first `over` tiles, where the window wraps.  delta: -4 lo.
struct PlaceWindow {
    uint32_t first, count, delta, over;
};

__device__ __forceinline__ PlaceWindow place_window(const Params &p, const PlacePlan &s, uint32_t used, uint32_t r0, uint32_t len, uint32_t shift, bool live)
{
    // r in [r0 - shift, r0 - shift + len) modulo m, in whole buckets
    const uint32_t lo = wrap(r0 + p.m - shift, p.m), end = min(lo + len, p.m), over = lo + len - end;
    uint32_t a = s.starts[lo >> s.bucket_shift], b = s.starts[((end - 1u) >> s.bucket_shift) + 1u];
    uint32_t c = s.starts[((over ? over - 1u : 0u) >> s.bucket_shift) + 1u];
    a = min(a, used);
    b = live ? min(b, used) : 0u;
    c = live && over ? min(c, used) : 0u;
    PlaceWindow w;
    w.first = a >> 6;
    w.count = b > a ? ((b + 63u) >> 6) - w.first : 0u;
    w.over = (c + 63u) >> 6;
    w.delta = 0u - 4u * lo;
    return w;
}

// (all loads in one branch: one that every lane asked for itself waited for each)
template <typename AT>
__device__ __forceinline__ void load_region(const Params &p, const AT *__restrict__ array, uint32_t r0, uint32_t len, float4 *to)
{
    constexpr uint32_t kVecs = (1u << kPlaceShift) / 4u / kPlaceBlock;
    float v[kVecs][4];
    if (len == 1u << kPlaceShift) {
#pragma unroll
        for (uint32_t u = 0; u < kVecs; ++u) load_span<4>(array, r0 + 4u * (u * kPlaceBlock + threadIdx.x), v[u]);
    } else {
#pragma unroll
        for (uint32_t u = 0; u < kVecs; ++u) {
#pragma unroll
            for (uint32_t k = 0; k < 4u; ++k) v[u][k] = widen(array[r0 + min(4u * (u * kPlaceBlock + threadIdx.x) + k, len - 1u)]);
        }
    }
#pragma unroll
    for (uint32_t u = 0; u < kVecs; ++u) to[u * kPlaceBlock + threadIdx.x] = make_float4(v[u][0], v[u][1], v[u][2], v[u][3]);
}

template <int Z, typename AT>
__global__ __launch_bounds__(kPlaceBlock, 8) void place_regions_kernel(Params p, PlacePlan s, const AT *__restrict__ array, const uint32_t *__restrict__ entries,
                                                                       const uint32_t *__restrict__ pages, float *__restrict__ out)
{
    extern __shared__ float4 place_lds[];
    float *slots = reinterpret_cast<float *>(place_lds);
    const uint32_t used = *s.used;
    if (used == 0) return;
    const uint32_t t = threadIdx.x, lane = t & 63u;
    auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
    auto of_lane = [](uint32_t v, uint32_t l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l); };
    // A lane's window, in every region: chunk and class (0: the sum stays below P), lane after lane
    const uint32_t my_w = uniform(t >> 6) + lane * (kPlaceBlock / 64u), my_c = my_w >> 1;
    const bool my_live = my_w < 2u * p.C;
    const uint32_t my_cc = mul_p(p.Ch, my_live ? my_c : 0u);
    // (keys compare as their entries do)
    const uint32_t least = place_entry(p, s, kP - my_cc, mod_m(kP - my_cc, p.m, p.m_recip));      // of those that pass P, above 0
    const uint32_t my_base = my_w & 1u ? least : 0u, my_width = my_w & 1u ? 0u - least : least;
    uint32_t my_shift = mod_m(my_cc, p.m, p.m_recip);
    if (my_w & 1u) my_shift = wrap(my_shift + p.m - mod_m(kP, p.m, p.m_recip), p.m);
    uint32_t my_page[Z], my_in_page[Z];
#pragma unroll
    for (int j = 0; j < Z; ++j) {                                // (element i lies in page i / page_elems of its tile)
        const uint32_t i = my_c * Z + j;
        my_page[j] = (i * s.page_recip) >> 16;
        my_in_page[j] = i - my_page[j] * s.page_elems;
    }
    // A lane that has nothing to store points past the end of the buffer: every store is issued, so that the compiler knows
    // how many are in flight and lets a wait for loads leave the stores before them alone.
    const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(out, 0, (int)s.out_bytes, 0x00027000);

    const uint32_t r0 = blockIdx.x << kPlaceShift, len = min(1u << kPlaceShift, p.m - r0), len4 = 4u * len;
    const PlaceWindow my = place_window(p, s, used, r0, len, my_shift, my_live);
    load_region(p, array, r0, len, place_lds);
    __syncthreads();
    if (Z > 1) {                                                 // and the float after the region
        if (t == 0) slots[len] = widen(array[wrap(r0 + len, p.m)]);
        __syncthreads();
    }
    // tiles [first, first + count) of window w
    auto load = [&](PlaceBatch<Z> &b, uint32_t w, uint32_t first, uint32_t count, uint32_t delta) {
        const uint32_t width = of_lane(my_width, w);
        b.delta = delta;
        b.base = of_lane(my_base, w);
#pragma unroll
        for (int j = 0; j < Z; ++j) {
            b.in_page[j] = of_lane(my_in_page[j], w) << 8;
            b.page[j] = pages[(first + min(lane, kPlaceAhead - 1u)) * 64u + of_lane(my_page[j], w)];      // (both lists go on for some words)
        }
#pragma unroll
        for (uint32_t u = 0; u < kPlaceAhead; ++u) {
            b.width[u] = u < count ? width : 0u;
            b.entry[u] = entries[(first + u) * 64u + lane];
        }
    };
    auto serve = [&](const PlaceBatch<Z> &b) {
        bool on[kPlaceAhead];
        float x[kPlaceAhead][Z];
#pragma unroll
        for (uint32_t u = 0; u < kPlaceAhead; ++u) {
            const uint32_t rel = ((b.entry[u] & s.r_mask) << 2) + b.delta;
            on[u] = (rel < len4) & (b.entry[u] - b.base < b.width[u]);
            const float *from = reinterpret_cast<const float *>(reinterpret_cast<const char *>(place_lds) + min(rel, len4 - 4u));
#pragma unroll
            for (int j = 0; j < Z; ++j) x[u][j] = from[j];
        }
#pragma unroll
        for (uint32_t u = 0; u < kPlaceAhead; ++u) {
            const int at = on[u] ? (int)(lane * 4u) : -4;
#pragma unroll
            for (int j = 0; j < Z; ++j)
                __builtin_amdgcn_raw_buffer_store_b32((int)__float_as_uint(x[u][j]), rows, at, (int)((of_lane(b.page[j], u) << 8) + b.in_page[j]), 0);
        }
    };
    // the walk: window w of the wavefront, from its tile n on; todo: windows to come
    uint64_t todo = __ballot(my.count != 0);
    uint32_t w = 0, n = 0, first = 0, count = 0;
    auto fetch = [&](PlaceBatch<Z> &b) {                         // past the last window: a batch of nothing
        if (n >= count && todo != 0) {
            w = (uint32_t)__builtin_ctzll(todo);
            todo &= todo - 1ull;
            n = 0;
            first = of_lane(my.first, w);
            count = of_lane(my.count, w);
        }
        const uint32_t left = n < count ? count - n : 0u;
        load(b, w, first + (left ? n : 0u), left, of_lane(my.delta, w));
        n += kPlaceAhead;
        return left != 0;
    };
    // Loads and stores of a wavefront complete in the order they were issued, so that a wait for loads waits for all
    // stores before them too: a batch's loads are requested before the stores of the batch before it (three
    // or four batches on their way: level).  (Each batch in registers
    // of its own: a copy would wait for its loads.  No way out of the loop between a batch's loads and its use, or they would move there.)
    PlaceBatch<Z> even, odd;
    for (bool more = todo != 0 && fetch(even); more;) {
        fetch(odd);
        serve(even);
        more = fetch(even);
        serve(odd);
    }
    for (uint64_t wrapped = __ballot(my.over != 0); wrapped != 0; wrapped &= wrapped - 1ull) {      // a few windows of the launch
        const uint32_t l = (uint32_t)__builtin_ctzll(wrapped), end = of_lane(my.over, l);
        for (n = 0; n < end; n += kPlaceAhead) {
            load(even, l, n, end - n, of_lane(my.delta, l) + 4u * p.m);
            serve(even);
        }
    }
}

template <bool SIGN>
__global__ __launch_bounds__(256) void place_rows_kernel(Params p, PlacePlan s, uint32_t F, uint32_t F_recip, const int64_t *__restrict__ indices, float *out)
{
    __shared__ float turn[kPlaceTurn][65];
    __shared__ uint32_t page[64], row[64], tg[SIGN ? 64 : 1];
    const uint32_t used = *s.used, tile = blockIdx.x, t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    if (tile * 64u >= used) return;
    const uint32_t count = min(64u, used - tile * 64u);
    if (t < 64u) {
        page[t] = s.pages[tile * 64u + t];
        const uint32_t r = t < count ? s.row[tile * 64u + t] : 0u;
        row[t] = r;
        if constexpr (SIGN) tg[t] = t < count ? staged_g(p, indices[r], mod_m(r, F, F_recip)) : 0u;
    }
    __syncthreads();
    for (uint32_t i0 = 0; i0 < p.d; i0 += kPlaceTurn) {
        const uint32_t elems = min(kPlaceTurn, p.d - i0);
        constexpr uint32_t kAhead = 8;
        for (uint32_t e0 = wave; e0 < elems; e0 += 4u * kAhead) {
            float v[kAhead];
#pragma unroll
            for (uint32_t u = 0; u < kAhead; ++u) {
                const uint32_t i = i0 + min(e0 + 4u * u, elems - 1u), pg = (i * s.page_recip) >> 16;
                v[u] = out[(uint64_t)(page[pg] + i - pg * s.page_elems) * 64u + lane];
            }
#pragma unroll
            for (uint32_t u = 0; u < kAhead; ++u)
                if (e0 + 4u * u < elems) turn[e0 + 4u * u][lane] = v[u];
        }
        __syncthreads();
        for (uint32_t k = wave; k < count; k += 4u) {
            float *to = out + (uint64_t)row[k] * p.d + i0;
            for (uint32_t e = lane; e < elems; e += 64u) {
                float v = turn[e][k];
                if constexpr (SIGN) v = apply_sign(v, sign_mask(add_p(tg[k], mul_p(p.Cg, i0 + e))));
                to[e] = v;
            }
        }
        __syncthreads();
    }
}

// The rows past n, when all others are final: copied where F1 found who has the token, else gathered.  A workgroup's words lie in
// one of the last rows, which it writes when all its wavefronts have read them.
template <int V, bool CONSEC, bool SIGN, typename AT>
__global__ __launch_bounds__(kLastMost * 64 / kLastRows) void place_last_kernel(Params p, Geom q, DistinctPlan d, PlacePlan s, uint32_t F_recip, uint32_t g_shift,
                                                                                const AT *__restrict__ array, const int64_t *__restrict__ indices, float *__restrict__ out)
{
    __shared__ uint32_t words[kLastMost];
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6, first = blockIdx.x << s.tail_shift;
    const uint32_t live = min(1u << s.tail_shift, s.tail > first ? s.tail - first : 0u);
    if (t < live) words[t] = *tail_word(s, p.d, first + t);
    __syncthreads();
    const uint32_t i = wave * kLastRows + lane;
    uint32_t row = d.n + first + i, from = kPlaceSelf, th = 0, tg = 0;
    bool self = false, copy = false;
    if (lane < kLastRows && i < live) {
        from = words[i];
        self = from == kPlaceSelf;
        copy = !self;
    } else if (wave == 0 && lane == kLastRows) {
        row = d.n + s.tail + blockIdx.x;
        self = true;
    }
    if (self) {
        const uint32_t f = mod_m(row, d.F, F_recip);
        const int64_t x = indices[row];
        th = staged_h(p, x, f);
        if constexpr (SIGN) tg = staged_g(p, x, f);
    }
    copy_rows<4>(copy, row, from, p.d, g_shift, out);
    const uint64_t plain = __ballot(self);
    if (plain) gather_rows<V, CONSEC, SIGN>(p, q, self, plain, row, th, tg, array, out);
}

}  // namespace robe
