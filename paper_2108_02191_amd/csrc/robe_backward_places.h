// Backward scatter-add (Eq. 3 of the paper) and the fused update for small blocks: the runs in the order of the places
// they write, as robe_forward_places.h takes the tokens in the order of those they read.
//
// With blocks of one or two floats a run leaves d / Z records, and region_reduce_kernel fetches a line of 128 bytes for every
// one of them to read four or eight (514 us for 19.6 M records at Z = 1), while the float atomics of the other route
// cost a 64-byte request each (1178 us).  Sorting every element's (place, value) pair by region writes and reads eight bytes an
// element in pieces of 64 (22.7 M pairs: 35 us to count, 178 to write, 76 to add).  But where a run writes follows from its
// key: with the runs by r = th mod m, the elements that land in a region of the array are those of two windows of runs
// per element of a row (robe_forward_places.h has the arithmetic).  So only the rows are moved, once, and the region's workgroup
// finds the rest.  After R1 of robe_backward_regions.h:
//
//   S1 count    every run counts in a bucket of r.
//   R3 scan     first entry of every bucket.
//   S2 place    entry (see place_entry) and source row of every run.  Runs past the room for their rows (how many there will be
//               is not known on the host) are added to the gradient array by float atomics here.
//   S3 turn     tiles of 64 runs, element by element.
//   S4 reduce   a workgroup per region of up to 2^14 slots (RunPlan::shift): for every element and window, tile by tile, the entries' places, and the values of
//               those that lie in the region, added to an LDS copy; then the rule applied to it.  ds_add_f32 runs at 0.33
//               lanes per clock and CU on this GPU, a compare-and-swap at 2.2 (random places) to 4.7 (neighbours), but only one
//               lane of those at a place gets through, so the few that do not try once more and then take the slow one.
//
// Backward of 852 K Zipf lookups, d = 128, Z = 1, 100 MB array: 405 -> 286 us (S1 9, R3 8, S2 8, S3 47, S4 106 instead of
// the pairs' 294); with ids of 10 M a table, for whose pairs there was no room, 1182 -> 346.  S4 without its additions takes
// 45 us less, without the write-back 43 (each measured in a copy); double words and their 64-bit additions, at half the
// region or one workgroup per CU, 13 and 20 more; every compare-and-swap waited for by itself, 6 more.
// The order of the additions is not fixed (the reproducible option keeps region_reduce_kernel).
#pragma once
#include "robe_forward_places.h"

namespace robe {

constexpr uint32_t kRunBlock = 256;
constexpr uint32_t kRunWb = 4;             // vectors per thread in flight in the write-back
constexpr uint32_t kRunTurn = 64;           // elements of a tile turned round at a time
constexpr uint32_t kRunSlots = (1u << kPlaceShift) + 64u;      // of S4 in LDS: the region, a word per lane
constexpr uint32_t kRunShort = 96;           // entries a window on average up to which S4 takes one tile at a time
constexpr uint32_t kRunAhead = 3;            // tiles whose loads are requested together

struct RunPlan {
    PlacePlan place;       // buckets, bucket_shift, r_bits, r_mask, counts, starts, entries, row (source block), most
    uint32_t *rank;        // [n] at run starts: which of its bucket the run is
    uint32_t *tg;          // [most] token part of the sign hash (sign on only)
    float *tiles;          // [most / 64][d][64]
    uint32_t shift;        // log2 of the slots of a region of S4
};

__device__ __forceinline__ uint32_t runs_used(const PlacePlan &s) { return min(s.starts[s.buckets], s.most); }

// A run starts wherever a walk of R1 does, so a frequent token leaves one in walk after walk, and additions to one word go one by one
// (26 tokens in 852 K lookups: 60 us): the positions where walks start go to workgroups of their own, the first `starts`
// of the launch, where neighbours of the same bucket are added as one.
__global__ __launch_bounds__(kRunBlock) void run_count_kernel(Params p, RegionPlan s, RunPlan l, uint32_t walk, uint32_t starts)
{
    const uint32_t lane = threadIdx.x & 63u;
    const bool first = blockIdx.x < starts;
    const uint64_t i = first ? ((uint64_t)blockIdx.x * kRunBlock + threadIdx.x) * walk : (uint64_t)(blockIdx.x - starts) * kRunBlock + threadIdx.x;
    bool head = false;
    uint32_t bucket = 0;
    if (i < s.n && (first || (uint32_t)i % walk != 0)) {
        const uint32_t th = s.keys[i];
        head = s.head[i] != 0;
        bucket = mod_m(th, p.m, p.m_recip) >> l.place.bucket_shift;
    }
    if (!first) {
        if (head) l.rank[i] = atomicAdd(&l.place.counts[bucket], 1u);
        return;
    }
    const uint32_t before = __shfl_up(bucket, 1);
    const uint64_t heads = __ballot(head), leads = __ballot(head && (lane == 0 || !((heads >> (lane - 1u)) & 1ull) || before != bucket));
    const uint64_t below = leads & ((2ull << lane) - 1ull);        // (lane 63: 2 << 63 is 0, and all are below)
    const uint32_t lead = below ? 63u - (uint32_t)__builtin_clzll(below) : 0u;
    const uint64_t ends = (leads | ~heads) & ~((2ull << lane) - 1ull);
    uint32_t base = 0;
    if (head && lead == lane) base = atomicAdd(&l.place.counts[bucket], (ends ? (uint32_t)__builtin_ctzll(ends) : 64u) - lane);
    base = __shfl(base, (int)lead);
    if (head) l.rank[i] = base + lane - lead;
}

// The first float of a source block's row.
__device__ __forceinline__ const float *source_row(const Params &p, const RegionPlan &s, const float *grad_out, uint32_t src)
{
    return src < s.src_own ? grad_out + (uint64_t)src * p.Z : s.P + (uint64_t)(src - s.src_own) * p.Z;
}

template <bool SIGN>
__global__ __launch_bounds__(kRunBlock) void run_place_kernel(Params p, RegionPlan s, RunPlan l, const float *__restrict__ grad_out, float *__restrict__ spill)
{
    const uint32_t i = blockIdx.x * kRunBlock + threadIdx.x, lane = threadIdx.x & 63u;
    uint32_t th = 0, src = 0, tg = 0;
    bool over = false;
    if (i < s.n && s.head[i]) {
        th = s.keys[i];
        src = s.src_row[i];
        if constexpr (SIGN) tg = s.run_tg[i];
        const uint32_t r = mod_m(th, p.m, p.m_recip), k = l.place.starts[r >> l.place.bucket_shift] + l.rank[i];
        over = k >= l.place.most;
        if (!over) {
            l.place.entries[k] = place_entry(p, l.place, th, r);
            l.place.row[k] = src;
            if constexpr (SIGN) l.tg[k] = tg;
        }
    }
    if (spill == nullptr) return;                               // there is room for all
    for (uint64_t todo = __ballot(over); todo != 0; todo &= todo - 1ull) {
        const int from = __builtin_ctzll(todo);
        const uint32_t h = __shfl(th, from), g = __shfl(tg, from);
        const float *row = source_row(p, s, grad_out, __shfl(src, from));
        for (uint32_t e = lane; e < p.d; e += 64u) {
            const uint32_t c = chunk_of(p, e);
            float v = row[e];
            if constexpr (SIGN) v = apply_sign(v, sign_mask(add_p(g, mul_p(p.Cg, e))));
            __hip_atomic_fetch_add(spill + wrap(offset_of(p, h, mul_p(p.Ch, c)) + e - c * p.Z, p.m), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

template <bool SIGN>
__global__ __launch_bounds__(kRunBlock) void run_turn_kernel(Params p, RegionPlan s, RunPlan l, const float *__restrict__ grad_out)
{
    __shared__ float turn[kRunTurn][65];
    __shared__ uint32_t src[64], tg[SIGN ? 64 : 1];
    const uint32_t used = runs_used(l.place), tile = blockIdx.x, t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    constexpr uint32_t kWaves = kRunBlock / 64u, kAhead = 16;
    static_assert(64u % (kWaves * kAhead) == 0, "every step takes runs of the tile alone");
    if (tile * 64u >= used) return;
    const uint32_t count = min(64u, used - tile * 64u);
    if (t < 64u) {                                               // past the last run: its row, for the values 0
        src[t] = l.place.row[tile * 64u + min(t, count - 1u)];
        if constexpr (SIGN) tg[t] = l.tg[tile * 64u + min(t, count - 1u)];
    }
    __syncthreads();
    float *to = l.tiles + (uint64_t)tile * 64u * p.d;
    for (uint32_t i0 = 0; i0 < p.d; i0 += kRunTurn) {
        const uint32_t elems = min(kRunTurn, p.d - i0);
        for (uint32_t e = lane; e < elems; e += 64u) {
            const uint32_t cg = SIGN ? mul_p(p.Cg, i0 + e) : 0u;
            for (uint32_t k0 = wave; k0 < 64u; k0 += kWaves * kAhead) {
                float v[kAhead];
#pragma unroll
                for (uint32_t u = 0; u < kAhead; ++u) v[u] = source_row(p, s, grad_out, src[k0 + u * kWaves])[i0 + e];
#pragma unroll
                for (uint32_t u = 0; u < kAhead; ++u) {
                    const uint32_t k = k0 + u * kWaves;
                    if constexpr (SIGN) v[u] = apply_sign(v[u], sign_mask(add_p(tg[k], cg)));
                    turn[e][k] = k < count ? v[u] : 0.0f;
                }
            }
        }
        __syncthreads();
        for (uint32_t e = wave; e < elems; e += kWaves) to[(i0 + e) * 64u + lane] = turn[e][lane];
        __syncthreads();
    }
}

// Up to A tiles of a window, see PlaceBatch.
template <uint32_t A>
struct RunBatch {
    uint32_t entry[A];
    float v[A];
    uint32_t delta, base, width[A];
};

// What S4's walk needs of its region and wavefront: see run_reduce_kernel.
struct RunWalk {
    PlaceWindow my;
    uint32_t my_base, my_width, wave, len4, last_tile, r_mask;
};

// A: tiles whose loads are requested together.
template <uint32_t A>
__device__ __forceinline__ void run_walk(const Params &p, const RunWalk &k, const uint32_t *__restrict__ entries, const float *__restrict__ tiles, float *acc)
{
    const uint32_t lane = threadIdx.x & 63u, len4 = k.len4;
    auto of_lane = [](uint32_t v, uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)x); };
    // tiles [first, first + count) of window w
    auto load = [&](RunBatch<A> &b, uint32_t w, uint32_t first, uint32_t count, uint32_t delta) {
        const uint32_t width = of_lane(k.my_width, w), i = (k.wave + w * (kPlaceBlock / 64u)) >> 1;
        b.delta = delta;
        b.base = of_lane(k.my_base, w);
#pragma unroll
        for (uint32_t u = 0; u < A; ++u) {
            const uint32_t tile = min(first + u, k.last_tile);
            b.width[u] = u < count ? width : 0u;
            b.entry[u] = entries[tile * 64u + lane];
            b.v[u] = tiles[(uint64_t)(tile * p.d + i) * 64u + lane];
        }
    };
    uint32_t *bits = reinterpret_cast<uint32_t *>(acc);
    // One compare-and-swap per value, all on their way together; a lane that has nothing to add tries a word of its own.  The
    // few that find another value in between go on alone.
    auto serve = [&](const RunBatch<A> &b) {
        uint32_t at[A], old[A], got[A];
        bool on[A], again = false;
#pragma unroll
        for (uint32_t u = 0; u < A; ++u) {
            const uint32_t rel = ((b.entry[u] & k.r_mask) << 2) + b.delta;
            on[u] = (rel < len4) & (b.entry[u] - b.base < b.width[u]);
            at[u] = on[u] ? rel >> 2 : (1u << kPlaceShift) + lane;
            old[u] = bits[at[u]];
        }
#pragma unroll
        for (uint32_t u = 0; u < A; ++u) got[u] = atomicCAS(&bits[at[u]], old[u], __float_as_uint(__uint_as_float(old[u]) + b.v[u]));
#pragma unroll
        for (uint32_t u = 0; u < A; ++u) again |= on[u] && got[u] != old[u];
        if (!__any(again)) return;
#pragma unroll
        for (uint32_t u = 0; u < A; ++u) {
            if (!on[u] || got[u] == old[u]) continue;
            if (!__hip_atomic_compare_exchange_strong(&bits[at[u]], &got[u], __float_as_uint(__uint_as_float(got[u]) + b.v[u]), __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_WORKGROUP))
                __hip_atomic_fetch_add(&acc[at[u]], b.v[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    };
    uint64_t todo = __ballot(k.my.count != 0);                      // windows to come
    uint32_t w = 0, n = 0, first = 0, count = 0;
    auto fetch = [&](RunBatch<A> &b) {                              // past the last window: a batch of nothing
        if (n >= count && todo != 0) {
            w = (uint32_t)__builtin_ctzll(todo);
            todo &= todo - 1ull;
            n = 0;
            first = of_lane(k.my.first, w);
            count = of_lane(k.my.count, w);
        }
        const uint32_t left = n < count ? count - n : 0u;
        load(b, w, first + (left ? n : 0u), left, of_lane(k.my.delta, w));
        n += A;
        return left != 0;
    };
    RunBatch<A> even, odd;
    for (bool more = todo != 0 && fetch(even); more;) {
        fetch(odd);
        serve(even);
        more = fetch(even);
        serve(odd);
    }
    for (uint64_t wrapped = __ballot(k.my.over != 0); wrapped != 0; wrapped &= wrapped - 1ull) {
        const uint32_t x = (uint32_t)__builtin_ctzll(wrapped), end = of_lane(k.my.over, x);
        for (n = 0; n < end; n += A) {
            load(even, x, n, end - n, of_lane(k.my.delta, x) + 4u * p.m);
            serve(even);
        }
    }
}

// The rule applied to region_len slots from r0 on, acc their gradient; kPlaceBlock threads.
template <int RULE>
__device__ __forceinline__ void run_write_back(const RegionPlan &s, const float *acc, uint32_t r0, uint32_t region_len, float *__restrict__ dst,
                                                   float *__restrict__ state, float lr, float eps, int vec_ok)
{
    typedef Vec<4>::A V4;
    const uint32_t nvec = vec_ok ? region_len / 4u : 0u, lane = threadIdx.x & 63u;
    for (uint32_t it0 = 0; it0 < nvec; it0 += kPlaceBlock * kRunWb) {   // same trip count for the whole workgroup
        V4 g[kRunWb], w[kRunWb], st[kRunWb];
        bool touch[kRunWb];
#pragma unroll
        for (uint32_t u = 0; u < kRunWb; ++u) {
            const uint32_t it = it0 + u * kPlaceBlock + threadIdx.x;
#pragma unroll
            for (int k = 0; k < 4; ++k) g[u][k] = 0.0f;
            if (it < nvec) g[u] = *reinterpret_cast<const V4 *>(&acc[4u * it]);
            const bool any = g[u][0] != 0.0f || g[u][1] != 0.0f || g[u][2] != 0.0f || g[u][3] != 0.0f;
            touch[u] = ((__ballot(any) >> (lane & ~3u)) & 0xFull) != 0 && it < nvec;      // whole 64-byte granules, or nothing of them
            if (touch[u]) {
                const uint32_t at = r0 + 4u * it;
                w[u] = s.keep_array ? *reinterpret_cast<const V4 *>(dst + at) : __builtin_nontemporal_load(reinterpret_cast<const V4 *>(dst + at));
                if constexpr (RULE == 1) st[u] = __builtin_nontemporal_load(reinterpret_cast<const V4 *>(state + at));
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < kRunWb; ++u) {
            if (!touch[u]) continue;
            const uint32_t at = r0 + 4u * (it0 + u * kPlaceBlock + threadIdx.x);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float wk = w[u][k], sk = RULE == 1 ? st[u][k] : 0.0f;
                small_rule<RULE>(wk, sk, g[u][k], lr, eps);
                w[u][k] = wk;
                if constexpr (RULE == 1) st[u][k] = sk;
            }
            if (s.keep_array) *reinterpret_cast<V4 *>(dst + at) = w[u];
            else __builtin_nontemporal_store(w[u], reinterpret_cast<V4 *>(dst + at));
            if constexpr (RULE == 1) __builtin_nontemporal_store(st[u], reinterpret_cast<V4 *>(state + at));
        }
    }
    for (uint32_t i = 4u * nvec + threadIdx.x; i < region_len; i += kPlaceBlock) {          // tail, or unaligned buffers
        float w = dst[r0 + i], st = RULE == 1 ? state[r0 + i] : 0.0f;
        if (acc[i] == 0.0f) continue;
        small_rule<RULE>(w, st, acc[i], lr, eps);
        dst[r0 + i] = w;
        if constexpr (RULE == 1) state[r0 + i] = st;
    }
}

// RULE as in region_reduce_kernel.
template <int RULE>
__global__ __launch_bounds__(kPlaceBlock, 8) void run_reduce_kernel(Params p, RegionPlan s, RunPlan l, const uint32_t *__restrict__ entries, const float *__restrict__ tiles,
                                                                    float *__restrict__ dst, float *__restrict__ state, float lr, float eps, int vec_ok)
{
    extern __shared__ float acc[];
    const uint32_t used = runs_used(l.place);
    if (used == 0) return;
    const uint32_t t = threadIdx.x, lane = t & 63u, last_tile = (used - 1u) >> 6;
    constexpr uint32_t kWaves = kPlaceBlock / 64u;
    auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
    for (uint32_t i = t; i < 1u << l.shift; i += kPlaceBlock) acc[i] = 0.0f;      // (the lanes' own words may hold anything)
    // a lane's window: element and class (see place_regions_kernel; every element has windows of its own, since a block may end in the next region)
    const uint32_t wave = uniform(t >> 6), my_w = wave + lane * kWaves, my_i = my_w >> 1;
    const bool my_live = my_w < 2u * p.d;
    const uint32_t my_c = my_live ? chunk_of(p, my_i) : 0u, my_cc = mul_p(p.Ch, my_c);
    const uint32_t least = place_entry(p, l.place, kP - my_cc, mod_m(kP - my_cc, p.m, p.m_recip));
    const uint32_t my_base = my_w & 1u ? least : 0u, my_width = my_w & 1u ? 0u - least : least;
    uint32_t my_shift = wrap(mod_m(my_cc, p.m, p.m_recip) + (my_live ? my_i - my_c * p.Z : 0u), p.m);
    if (my_w & 1u) my_shift = wrap(my_shift + p.m - mod_m(kP, p.m, p.m_recip), p.m);
    const uint32_t r0 = blockIdx.x << l.shift, len = min(1u << l.shift, p.m - r0);
    const PlaceWindow my = place_window(p, l.place, used, r0, len, my_shift, my_live);
    if (!__syncthreads_or((int)(my.count | my.over))) return;     // nothing lands here
    RunWalk k;
    k.my = my;
    k.my_base = my_base;
    k.my_width = my_width;
    k.wave = wave;
    k.len4 = 4u * len;
    k.last_tile = last_tile;
    k.r_mask = l.place.r_mask;
    // (short windows: the tiles after the first would mostly be requested in vain, and the walk is bound by what it issues.  208 K
    // lookups, d = 128, tables of up to 100 K ids, 50 M slots, whole backward: Z = 1 204 -> 176 us, Z = 2 193 -> 169; 117 entries
    // a window, 852 K lookups: 275, one at a time 278)
    if (((uint64_t)used << l.shift) <= (uint64_t)kRunShort * p.m) run_walk<1>(p, k, entries, tiles, acc);
    else run_walk<kRunAhead>(p, k, entries, tiles, acc);
    __syncthreads();
    run_write_back<RULE>(s, acc, r0, len, dst, state, lr, eps, vec_ok);
}

}  // namespace robe
