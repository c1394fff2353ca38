// Backward scatter-add (Eq. 3 of the paper) and the fused update for small blocks: the values themselves
// are sorted by destination region.
//
// With blocks of one or two floats a run leaves d / Z records, and region_reduce_kernel fetches a line of
// 128 bytes for every one of them to read four or eight (514 us for 19.6 M records at Z = 1), while the
// float atomics of the other route cost a 64-byte request each (1178 us).  Here the kernel that bins the
// runs reads every summed row once, whole, and writes (place, value) pairs, so that what the region's
// workgroup reads is the stream of its own pairs.  After R1 of robe_backward_regions.h:
//
//   E1 count     every run's d elements are hashed to their places and counted per region in LDS.
//   R3 scan      first slot of every region.
//   E2 scatter   the same walk, a tile of kElemTile elements at a time: hashed, ranked inside their
//                region by LDS counters, put into LDS in region order and written from there, so that
//                consecutive lanes write consecutive pairs (region_bin_kernel, which writes its eight-byte
//                records one by one, takes 246 us for as many and reads no rows; E2 170, E1 34).
//                Pairs past the room for them (RegionPlan::rec_cap: the runs are not known on the host, and
//                room for every gradient element was seventy times the rest of the workspace) are added
//                to the gradient array with float atomics, as the other route adds all of them.
//   E3 reduce    one workgroup per region of 2^14 slots adds its pairs into an LDS copy and applies the
//                rule to it.  ds_add_f32 runs at 0.33 lanes per clock and CU on this GPU, a compare-and-swap
//                at 2.2 (random places) to 4.7 (neighbours), but only one lane of those at a place gets
//                through a round, and the runs of a frequent token leave their pairs side by side: two
//                rounds of the one, the other for the lanes that are left (74 us; compare-and-swap
//                until it succeeds 147, one round 78).
//
// The order of the additions is not fixed (the reproducible option keeps region_reduce_kernel).
#pragma once
#include "robe_backward_regions.h"

namespace robe {

constexpr uint32_t kElemShift = 14;           // regions of 2^14 slots: 64 KB of LDS, two workgroups per CU in E3
constexpr uint32_t kElemBlock = 1024;
constexpr uint32_t kElemBlocks = 256;         // grid of E1 and E2: E2 fills a CU's LDS
constexpr uint32_t kElemPer = 12;             // elements per thread and tile in E2
constexpr uint32_t kElemTile = kElemBlock * kElemPer;
constexpr uint32_t kElemRuns = 256;           // runs of a tile, at most
constexpr uint32_t kElemMaxRegions = 3600;

// LDS of E2: the tile, three words per region, the run list (a tile's runs and one more step of positions)
__host__ __device__ constexpr size_t elem_lds_bytes(uint32_t NR, bool sign)
{
    return (size_t)kElemTile * 8 + (size_t)NR * 12 + (size_t)(kElemRuns + kElemBlock) * (sign ? 12u : 8u) + 64 * 4;
}
static_assert(elem_lds_bytes(kElemMaxRegions, true) <= 160 * 1024, "E2: one workgroup per CU");

// How a tile's elements are dealt out: 2^row_shift threads per run (d rounded up to a power of two), so
// that a thread has the same element of every run it meets and its part of the hash is a constant.  (With
// the elements of a tile side by side, two divisions and a product modulo P per element made E1 alone 84 us.)
struct ElemLanes {
    uint32_t i, c, j, cc, cg;   // element, its chunk, its place in the chunk; (Ch * c) mod P, (Cg * i) mod P
    uint32_t k0, step;          // this thread's first run of a tile, runs between its runs
    uint32_t runs;              // runs of a tile
    bool live;                  // the element exists
};

__device__ __forceinline__ ElemLanes elem_lanes(const Params &p, uint32_t row_shift)
{
    ElemLanes l;
    l.i = threadIdx.x & ((1u << row_shift) - 1u);
    l.live = l.i < p.d;
    l.c = l.i / p.Z;
    l.j = l.i - l.c * p.Z;
    l.cc = mod_p((uint64_t)p.Ch * l.c);
    l.cg = mod_p((uint64_t)p.Cg * l.i);
    l.k0 = threadIdx.x >> row_shift;
    l.step = kElemBlock >> row_shift;
    l.runs = l.step * kElemPer < kElemRuns ? l.step * kElemPer : kElemRuns;
    return l;
}

// Walk this workgroup's sorted positions; call f(first, count) for every tile of runs, which lie in
// run_th / run_src [/ run_tg] [0, count).  All threads of the workgroup take part; f may use barriers.
template <bool SIGN, typename F>
__device__ __forceinline__ void for_each_tile(const RegionPlan &s, uint32_t tile_runs, uint32_t *run_th, uint32_t *run_src,
                                              uint32_t *run_tg, uint32_t *wave_n, F f)
{
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint64_t b = (uint64_t)blockIdx.x * s.pos_per_block;
    uint64_t e = b + s.pos_per_block;
    if (e > s.n) e = s.n;
    uint32_t held = 0;                                          // runs in the list, the same in every thread
    for (uint64_t p0 = b; p0 < e; p0 += kElemBlock) {
        const uint64_t i = p0 + t;
        const bool in = i < e;
        const uint64_t at = in ? i : p0;
        const bool head = in && s.head[at] != 0;
        const uint32_t th = s.keys[at], src = s.src_row[at], tg = SIGN ? s.run_tg[at] : 0u;
        const uint64_t heads = __ballot(head);
        if (lane == 0) wave_n[wave] = (uint32_t)__popcll(heads);
        __syncthreads();
        uint32_t to = held;
#pragma unroll
        for (uint32_t w = 0; w < kElemBlock / 64u; ++w) {
            const uint32_t c = wave_n[w];
            to += w < wave ? c : 0u;
            held += c;
        }
        if (head) {
            const uint32_t k = to + (uint32_t)__popcll(heads & ((1ull << lane) - 1ull));   // < tile_runs + kElemBlock
            run_th[k] = th;
            run_src[k] = src;
            if constexpr (SIGN) run_tg[k] = tg;
        }
        __syncthreads();
        uint32_t done = 0;
        const bool last = p0 + kElemBlock >= e;
        while (held - done >= tile_runs || (last && held > done)) {
            const uint32_t count = held - done < tile_runs ? held - done : tile_runs;
            f(done, count);
            done += count;
        }
        // what is left moves to the front (fewer than tile_runs <= kElemRuns runs)
        const uint32_t left = held - done;
        uint32_t mv_th = 0, mv_src = 0, mv_tg = 0;
        if (t < left) {
            mv_th = run_th[done + t];
            mv_src = run_src[done + t];
            if constexpr (SIGN) mv_tg = run_tg[done + t];
        }
        __syncthreads();
        if (t < left) {
            run_th[t] = mv_th;
            run_src[t] = mv_src;
            if constexpr (SIGN) run_tg[t] = mv_tg;
        }
        held = left;
        // (the barrier after the next step's counts orders these writes before the list is read)
    }
}

__global__ __launch_bounds__(kElemBlock) void element_count_kernel(Params p, RegionPlan s, uint32_t row_shift)
{
    extern __shared__ uint32_t elem_lds[];
    uint32_t *hist = elem_lds;                                   // NR
    uint32_t *run_th = hist + s.NR, *run_src = run_th + kElemRuns + kElemBlock, *wave_n = run_src + kElemRuns + kElemBlock;
    for (uint32_t r = threadIdx.x; r < s.NR; r += kElemBlock) hist[r] = 0;
    __syncthreads();
    const ElemLanes l = elem_lanes(p, row_shift);
    for_each_tile<false>(s, l.runs, run_th, run_src, nullptr, wave_n, [&](uint32_t first, uint32_t count) {
#pragma unroll
        for (uint32_t u = 0; u < kElemPer; ++u) {
            const uint32_t k = l.k0 + u * l.step;
            if (l.live && k < count) atomicAdd(&hist[wrap(offset_of(p, run_th[first + k], l.cc) + l.j, p.m) >> kElemShift], 1u);
        }
        __syncthreads();
    });
    __syncthreads();
    uint32_t *mine = s.wg_first + (uint64_t)blockIdx.x * s.NR;   // see region_bin_kernel
    for (uint32_t r = threadIdx.x; r < s.NR; r += kElemBlock) {
        const uint32_t c = hist[r];
        if (c) mine[r] = atomicAdd(&s.counts[r], c);
    }
}

template <bool SIGN>
__global__ __launch_bounds__(kElemBlock) void element_scatter_kernel(Params p, RegionPlan s, uint32_t row_shift,
                                                                     const float *__restrict__ grad_out,
                                                                     float *__restrict__ spill)   // where pairs past rec_cap go; NULL: there are none
{
    extern __shared__ uint32_t elem_lds[];
    uint2 *staged = reinterpret_cast<uint2 *>(elem_lds);          // kElemTile pairs in region order
    uint32_t *cnt = elem_lds + 2u * kElemTile;                    // pairs of each region in the tile; then where they start in it
    uint32_t *slot = cnt + s.NR;                                  // next output slot of each region, minus the region's start in the tile
    uint32_t *next = slot + s.NR;                                 // next output slot of each region
    uint32_t *run_th = next + s.NR, *run_src = run_th + kElemRuns + kElemBlock;
    uint32_t *run_tg = run_src + kElemRuns + kElemBlock;
    uint32_t *wave_n = run_tg + (SIGN ? kElemRuns + kElemBlock : 0u);
    uint32_t *wave_sum = wave_n + 16;
    uint32_t *spills = wave_sum + 16;                             // 1: pairs of the tile lie past rec_cap
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint32_t *mine = s.wg_first + (uint64_t)blockIdx.x * s.NR;
    for (uint32_t r = t; r < s.NR; r += kElemBlock) next[r] = s.starts[r] + mine[r];   // (regions without pairs of this workgroup: never used)
    __syncthreads();
    const ElemLanes l = elem_lanes(p, row_shift);
    for_each_tile<SIGN>(s, l.runs, run_th, run_src, run_tg, wave_n, [&](uint32_t first, uint32_t count) {
        const uint32_t items = count * p.d;
        for (uint32_t r = t; r < s.NR; r += kElemBlock) cnt[r] = 0;
        if (t == 0) *spills = 0;
        __syncthreads();
        uint32_t at[kElemPer], rank[kElemPer];
        float v[kElemPer];
#pragma unroll
        for (uint32_t u = 0; u < kElemPer; ++u) {
            const uint32_t k = l.k0 + u * l.step;
            v[u] = 0.0f;
            if (l.live && k < count) {
                const uint32_t src = run_src[first + k];
                const float *row = src < s.src_own ? grad_out + (uint64_t)src * p.Z : s.P + (uint64_t)(src - s.src_own) * p.Z;
                v[u] = row[l.i];
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < kElemPer; ++u) {
            const uint32_t k = l.k0 + u * l.step;
            at[u] = rank[u] = 0;
            if (l.live && k < count) {
                at[u] = wrap(offset_of(p, run_th[first + k], l.cc) + l.j, p.m);
                rank[u] = atomicAdd(&cnt[at[u] >> kElemShift], 1u);
            }
        }
        __syncthreads();
        // exclusive scan of the counts, four regions per thread
        constexpr uint32_t kPer = (kElemMaxRegions + kElemBlock - 1u) / kElemBlock;
        uint32_t c[kPer], sum = 0;
#pragma unroll
        for (uint32_t q = 0; q < kPer; ++q) {
            const uint32_t r = t * kPer + q;
            c[q] = r < s.NR ? cnt[r] : 0u;
            sum += c[q];
        }
        uint32_t incl = sum;
#pragma unroll
        for (uint32_t off = 1; off < 64u; off <<= 1) {
            const uint32_t up = __shfl_up(incl, off);
            if (lane >= off) incl += up;
        }
        if (lane == 63u) wave_sum[wave] = incl;
        __syncthreads();
        uint32_t a = incl - sum;
#pragma unroll
        for (uint32_t w = 0; w < kElemBlock / 64u; ++w) a += w < wave ? wave_sum[w] : 0u;
#pragma unroll
        for (uint32_t q = 0; q < kPer; ++q) {
            const uint32_t r = t * kPer + q;
            if (r < s.NR) {
                const uint32_t out = next[r];
                cnt[r] = a;
                slot[r] = out - a;                                 // (wraps; the sum below is the slot)
                next[r] = out + c[q];
                if (c[q] && out + c[q] > s.rec_cap) *spills = 1;
            }
            a += c[q];
        }
        __syncthreads();
#pragma unroll
        for (uint32_t u = 0; u < kElemPer; ++u)
            if (l.live && l.k0 + u * l.step < count) {
                if constexpr (SIGN) v[u] = apply_sign(v[u], sign_mask(add_p(run_tg[first + l.k0 + u * l.step], l.cg)));
                staged[cnt[at[u] >> kElemShift] + rank[u]] = make_uint2(at[u], __float_as_uint(v[u]));
            }
        __syncthreads();
        if (*spills == 0) {                                       // (its own loop: the check inside it cost 6 us of 170)
#pragma unroll
            for (uint32_t u = 0; u < kElemPer; ++u) {
                const uint32_t j = t + u * kElemBlock;
                if (j < items) {
                    const uint2 x = staged[j];
                    s.rec[slot[x.x >> kElemShift] + j] = x;
                }
            }
        } else {
            for (uint32_t j = t; j < items; j += kElemBlock) {
                const uint2 x = staged[j];
                const uint32_t to = slot[x.x >> kElemShift] + j;
                if (to < s.rec_cap) s.rec[to] = x;
                else if (spill != nullptr) __hip_atomic_fetch_add(spill + x.x, __uint_as_float(x.y), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __syncthreads();
    });
}

// E3.  RULE as in region_reduce_kernel.
constexpr uint32_t kElemNone = 0xFFFFFFFFu;
constexpr int kElemTries = 2;       // compare-and-swap rounds before the slow atomic (see above)
constexpr int kElemAhead = 8;       // pairs per thread whose loads are in flight together
constexpr uint32_t kElemWb = 4;     // vectors per thread in flight in the write-back

template <int RULE>
__global__ __launch_bounds__(kElemBlock) void element_reduce_kernel(Params p, RegionPlan s, float *__restrict__ dst,
                                                                    float *__restrict__ state, float lr, float eps, int vec_ok)
{
    extern __shared__ float elem_acc[];
    const uint32_t r = blockIdx.x;
    const uint32_t rb = s.starts[r], end = s.starts[r + 1u], re = end < s.rec_cap ? end : s.rec_cap;
    if (rb >= re) return;                                          // nothing lands in this region, or all of it past the room
    const uint32_t r0 = r << kElemShift;
    const uint32_t region_len = (p.m - r0) < (1u << kElemShift) ? (p.m - r0) : (1u << kElemShift);
    uint32_t *bits = reinterpret_cast<uint32_t *>(elem_acc);
    for (uint32_t i = threadIdx.x; i < region_len; i += kElemBlock) elem_acc[i] = 0.0f;
    __syncthreads();
    for (uint32_t k0 = rb + threadIdx.x; k0 < re; k0 += kElemBlock * kElemAhead) {
        uint2 x[kElemAhead];
#pragma unroll
        for (int u = 0; u < kElemAhead; ++u) {
            const uint32_t k = k0 + (uint32_t)u * kElemBlock;
            x[u] = make_uint2(0xFFFFFFFFu, 0u);
            if (k < re) {
                const uint64_t w = __builtin_nontemporal_load(reinterpret_cast<const uint64_t *>(s.rec + k));
                x[u] = make_uint2((uint32_t)w, (uint32_t)(w >> 32));
            }
        }
        uint32_t a[kElemAhead], old[kElemAhead];
#pragma unroll
        for (int u = 0; u < kElemAhead; ++u) {
            a[u] = x[u].x < p.m && x[u].x - r0 < region_len ? x[u].x - r0 : kElemNone;
            old[u] = a[u] != kElemNone ? bits[a[u]] : 0u;
        }
#pragma unroll
        for (int u = 0; u < kElemAhead; ++u) {
            if (a[u] == kElemNone) continue;
            const float v = __uint_as_float(x[u].y);
            bool done = false;
#pragma unroll
            for (int tries = 0; tries < kElemTries; ++tries)
                if (!done)
                    done = __hip_atomic_compare_exchange_strong(&bits[a[u]], &old[u], __float_as_uint(__uint_as_float(old[u]) + v),
                                                                __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (!done) __hip_atomic_fetch_add(&elem_acc[a[u]], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    __syncthreads();
    typedef Vec<4>::A V4;
    const uint32_t nvec = vec_ok ? region_len / 4u : 0u, lane = threadIdx.x & 63u;
    for (uint32_t it0 = 0; it0 < nvec; it0 += kElemBlock * kElemWb) {   // same trip count for the whole workgroup
        V4 g[kElemWb], w[kElemWb], st[kElemWb];
        bool touch[kElemWb];
#pragma unroll
        for (uint32_t u = 0; u < kElemWb; ++u) {
            const uint32_t it = it0 + u * kElemBlock + threadIdx.x;
#pragma unroll
            for (int k = 0; k < 4; ++k) g[u][k] = 0.0f;
            if (it < nvec) g[u] = *reinterpret_cast<const V4 *>(&elem_acc[4u * it]);
            const bool any = g[u][0] != 0.0f || g[u][1] != 0.0f || g[u][2] != 0.0f || g[u][3] != 0.0f;
            touch[u] = ((__ballot(any) >> (lane & ~3u)) & 0xFull) != 0 && it < nvec;      // whole 64-byte granules, or nothing of them
            if (touch[u]) {
                const uint32_t at = r0 + 4u * it;
                w[u] = s.keep_array ? *reinterpret_cast<const V4 *>(dst + at) : __builtin_nontemporal_load(reinterpret_cast<const V4 *>(dst + at));
                if constexpr (RULE == 1) st[u] = __builtin_nontemporal_load(reinterpret_cast<const V4 *>(state + at));
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < kElemWb; ++u) {
            if (!touch[u]) continue;
            const uint32_t at = r0 + 4u * (it0 + u * kElemBlock + threadIdx.x);
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
    for (uint32_t i = 4u * nvec + threadIdx.x; i < region_len; i += kElemBlock) {          // tail, or unaligned buffers
        float w = dst[r0 + i], st = RULE == 1 ? state[r0 + i] : 0.0f;
        if (elem_acc[i] == 0.0f) continue;
        small_rule<RULE>(w, st, elem_acc[i], lr, eps);
        dst[r0 + i] = w;
        if constexpr (RULE == 1) state[r0 + i] = st;
    }
}

}  // namespace robe
