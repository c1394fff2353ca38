// HIP kernels of the ROBE-Z path for gfx950 (wave64).
//
// Work decomposition shared by the forward gather and the backward scatter:
//
//   * A wavefront owns a tile of rows (single-hot: TL consecutive lookups;
//     bags: 64/G consecutive bags).  In a first pass every lane hashes ONE
//     token of the tile - the part of h and g that depends on the token and on
//     the table id, (B*x + A*e + D) mod P - so the 64-bit modular work is done
//     once per token instead of once per lane that touches the token.
//   * In a second pass a group of G = d/V lanes walks the tile's tokens.  A
//     lane fetches the staged token term from the lane that hashed it
//     (wavefront shuffle), adds its own chunk term (C*c) mod P, which is a
//     per-lane constant, and finishes with one reciprocal-multiply `mod m`.
//   * A lane owns V elements of a row.  CONSEC layout: V consecutive elements
//     of one chunk (one hash, one unaligned 4V-byte load).  STRIDED layout:
//     elements grp + k*G, k < V (lanes of a group touch consecutive addresses,
//     which is what coalesces float atomics, and what Z < V needs).
//
// The integer maps are those of Eq. 5 (h, idx) and Eq. 2 (g) of the paper; the
// gather is Eq. 4, the scatter Eq. 3.
#pragma once
#include "robe_device.h"

namespace robe {

constexpr int kBlock = 256;           // 4 wavefronts
// The kernels that walk rows: every wavefront its own workgroup, so that a slot is free again as soon as its
// wavefront has ended.  Blocks of 512, 256, 128, 64 threads, us: bags on the bfloat16 copy of the 1 GB array
// 637 / 592 / 588 / 570, single-hot forward of 1.7 M lookups in a step 687 / 675 / 673 / 668.
constexpr int kRowBlock = 64;
constexpr int kRowWaves = kRowBlock / 64;
constexpr int kUnroll = 4;            // tokens in flight per lane group

// Launch geometry, filled on the host.
struct Geom {
    uint32_t F;        // number of tables (features)
    uint32_t G;        // lanes per row, power of two, <= 64; G * V >= d
    uint32_t d;        // elements per row; in the strided layout lane slots grp + k * G past it stay idle
    uint32_t g_shift;  // log2(G)
    uint32_t TL;       // rows per wavefront tile (single-hot kernels), multiple of 64/G, <= 64 (0: unused)
    uint32_t bpx;      // workgroups per XCD when rows are walked table by table (0: walk rows in memory order)
    int64_t batch;     // rows = batch * F
    // Where the F tables of this launch sit in the caller's buffers.  A plain call covers all of a
    // sample's tables (F_in = F, e0 = 0, row_floats = F * d, col0 = 0); a call for tables of mixed
    // dimensions launches once per run of consecutive tables of one dimension.
    uint32_t F_in;       // tables per sample in indices / offsets
    uint32_t e0;         // table id of this launch's first table = its place in a sample's input row
    int64_t row_floats;  // floats per sample in out / grad_out
    int64_t col0;        // first float of this launch's first table inside a sample
    // The walk's divisions and addresses (a 64-bit division is some 150 instructions and stood before the
    // first load of every wavefront; a call of 64 samples spent a quarter of its time there).
    uint32_t F_recip, batch_recip;   // min(floor(2^32 / x), 2^32 - 1), see mod_m
    uint32_t z_shift, c_shift;       // log2 of Z and of d / Z where these are powers of two (single_hot_block_kernel)
    uint32_t narrow;     // 1: rows below 2^31, and 64 rows apart is less than 2^30 floats or ids, in either order
    uint32_t plain;      // 1: the trivial view above, rows follow each other in memory
    // Sorted backward over tables of different dimensions (one launch for all of them): per table its
    // first float inside a sample (.x) and its dimension (.y); d above is then the largest dimension.
    // NULL: every table has dimension d and row k starts at float k * d.
    const uint2 *tables;
    // Sorted backward: 1 when the sort looked at few key bits, so that tokens whose keys agree in those
    // bits sit interleaved; the combine kernels then sort the positions they look at together (with
    // float atomics a wavefront's 64, without a lane group's G) by 26 bits of the key (window_key) before they
    // look for runs.
    uint32_t window_sort;
};

// One row of a launch: where its id (or bag bounds) and its d floats live, and its table id.
struct RowRef {
    int64_t in_row;    // index into indices (single-hot) or offsets (bags)
    int64_t out_off;   // first float in out / grad_out
    uint32_t e;
};

// Which rows a wavefront works on.
//
// Row k = b*F + f of the [batch][F] layout belongs to table f.  Workgroups are handed to the 8 XCDs
// round-robin, and every XCD has its own L2.  Walking the rows in memory order shows every L2 the
// frequent tokens of all F tables; walking them table by table (position q = f*batch + b) and giving
// XCD x the x-th eighth of that order shows each L2 the frequent tokens of about F/8 tables only, so
// far more of them stay resident.  With bpx == 0 the order is the memory order.
constexpr uint32_t kXcds = 8;

struct RowWalk {
    int64_t q0;    // first position of this wavefront in walk order
    int64_t b0;    // its sample
    uint32_t f0;   // its table
};

__device__ __forceinline__ bool start_walk(const Geom &q, int64_t rows, int64_t rows_per_wave, RowWalk &w)
{
    uint32_t block = blockIdx.x;
    if (q.bpx) {
        const uint32_t x = block % kXcds, j = block / kXcds;
        block = x * q.bpx + j;
    }
    w.q0 = ((int64_t)block * kRowWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * rows_per_wave;
    if (w.q0 >= rows) return false;
    if (q.narrow) {
        const uint32_t q0 = (uint32_t)w.q0;
        if (q.bpx) {
            w.f0 = div_m(q0, (uint32_t)q.batch, q.batch_recip);
            w.b0 = q0 - w.f0 * (uint32_t)q.batch;
        } else {
            w.b0 = div_m(q0, q.F, q.F_recip);
            w.f0 = q0 - (uint32_t)w.b0 * q.F;
        }
    } else if (q.bpx) {
        w.f0 = (uint32_t)(w.q0 / q.batch);
        w.b0 = w.q0 - (int64_t)w.f0 * q.batch;
    } else {
        w.b0 = w.q0 / (int64_t)q.F;
        w.f0 = (uint32_t)(w.q0 - w.b0 * (int64_t)q.F);
    }
    return true;
}

// The wavefront's next n <= 64 rows where they are evenly spaced: row `ahead` has its id at in0 + ahead * in_step
// and its floats from out0 + ahead * out_step on, 32-bit distances from a base that is the same for all lanes.
struct RowLine {
    bool on;           // (uniform) false: walk_row finds every row on its own
    int64_t in0, out0;
    uint32_t in_step, out_step;
};

__device__ __forceinline__ RowLine line_of(const Geom &q, const RowWalk &w, uint32_t n, uint32_t d)
{
    RowLine l;
    l.on = q.narrow && (q.bpx ? w.b0 + (int64_t)n <= q.batch : q.plain != 0);
    if (q.bpx) {
        l.in0 = w.b0 * (int64_t)q.F_in + q.e0 + w.f0;
        l.out0 = w.b0 * q.row_floats + q.col0 + (int64_t)w.f0 * d;
        l.in_step = q.F_in;
        l.out_step = (uint32_t)q.row_floats;
    } else {
        l.in0 = w.q0;
        l.out0 = w.q0 * d;
        l.in_step = 1;
        l.out_step = d;
    }
    return l;
}

// The table id of the row `ahead` steps after the wavefront's first one, for rows on a line.
__device__ __forceinline__ uint32_t line_table(const Geom &q, const RowWalk &w, uint32_t ahead)
{
    return q.e0 + (q.bpx ? w.f0 : mod_m(w.f0 + ahead, q.F, q.F_recip));       // f0 + ahead < F + 64
}

// The row `ahead` steps after the wavefront's first one (ahead < 64).
__device__ __forceinline__ RowRef walk_row(const Geom &q, const RowWalk &w, uint32_t ahead, uint32_t d)
{
    int64_t b;
    uint32_t f;
    if (q.bpx) {
        b = w.b0 + ahead;
        f = w.f0;
        while (b >= q.batch) {   // crosses into the next table(s); at most `ahead` rounds
            b -= q.batch;
            ++f;
        }
    } else {
        const uint32_t t = w.f0 + ahead;  // < F + 64
        const uint32_t over = div_m(t, q.F, q.F_recip);
        f = t - over * q.F;
        b = w.b0 + over;
    }
    RowRef r;
    r.in_row = b * (int64_t)q.F_in + q.e0 + f;
    r.out_off = b * q.row_floats + q.col0 + (int64_t)f * d;
    r.e = q.e0 + f;
    return r;
}

template <int V>
struct Vec {
    typedef float A __attribute__((ext_vector_type(V)));  // V floats at natural vector alignment
    typedef A U __attribute__((aligned(4)));              // the same at 4-byte alignment
    typedef uint16_t HA __attribute__((ext_vector_type(V)));  // V bfloat16 bit patterns
    typedef HA HU __attribute__((aligned(2)));                 // ... at 2-byte alignment
};

// An array element as float32.  The array is float32, or bfloat16 bit patterns (uint16_t): the upper
// half of the float32 pattern, widened exactly by appending 16 zero bits.
__device__ __forceinline__ float widen(float v) { return v; }
__device__ __forceinline__ float widen(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// float32 -> bfloat16 bit pattern: round to nearest, ties to even; NaN stays NaN.
__device__ __forceinline__ uint16_t narrow_bf16(float v)
{
    const uint32_t u = __float_as_uint(v);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu) != 0u) return (uint16_t)((u >> 16) | 0x0040u);
    const uint32_t keep = u >> 16, drop = u & 0xFFFFu;
    return (uint16_t)(keep + ((drop > 0x8000u || (drop == 0x8000u && (keep & 1u))) ? 1u : 0u));
}

// V consecutive array elements from `pos` on, all inside the array, as float32.
template <int V, typename AT>
__device__ __forceinline__ void load_span(const AT *__restrict__ array, uint32_t pos, float (&v)[V])
{
    if constexpr (sizeof(AT) == 4) {
        const typename Vec<V>::A u = *reinterpret_cast<const typename Vec<V>::U *>(array + pos);
#pragma unroll
        for (int k = 0; k < V; ++k) v[k] = u[k];
    } else {
        const typename Vec<V>::HA u = *reinterpret_cast<const typename Vec<V>::HU *>(array + pos);
#pragma unroll
        for (int k = 0; k < V; ++k) v[k] = widen((uint16_t)u[k]);
    }
}

// N spans at once, each lane's own; a span may cross the end of the circular array.  That is asked once
// for all of them and the whole wavefront, so that the usual case is N loads in a row.  Only the spans
// that `want` names are read.
template <int V, int N, typename AT>
__device__ __forceinline__ void load_spans(const Params &p, const AT *__restrict__ array, const uint32_t (&pos)[N],
                                           const bool (&want)[N], float (&v)[N][V])
{
    bool cross = false;
#pragma unroll
    for (int u = 0; u < N; ++u) cross |= V > 1 && pos[u] + V > p.m;
#pragma unroll
    for (int u = 0; u < N; ++u) {
#pragma unroll
        for (int k = 0; k < V; ++k) v[u][k] = 0.0f;
    }
    if (!__any(cross)) {
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (want[u]) load_span<V>(array, pos[u], v[u]);
    } else {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            if (want[u]) {
#pragma unroll
                for (int k = 0; k < V; ++k) v[u][k] = widen(array[wrap(pos[u] + k, p.m)]);
            }
        }
    }
}

// Per-lane constants: which elements this lane owns and their chunk terms.
template <int V, bool CONSEC, bool SIGN>
struct Lane {
    static constexpr int NH = CONSEC ? 1 : V;   // distinct (chunk, position) pairs
    uint32_t cc[NH];                             // (Ch * c) mod P
    uint32_t jj[NH];                             // position inside the chunk
    uint32_t cg[SIGN ? V : 1];                   // (Cg * i) mod P per owned element, plus 1 (see sign_mask_of_sum)
    uint32_t live;                               // bit k: owned element k exists (strided layout with G * V > d)

    __device__ __forceinline__ bool has(int k) const { return CONSEC || ((live >> k) & 1u) != 0u; }

    __device__ __forceinline__ void init(const Params &p, const Geom &q, uint32_t grp)
    {
        live = 0;
#pragma unroll
        for (int k = 0; k < NH; ++k) {
            uint32_t i = CONSEC ? grp * V : grp + (uint32_t)k * q.G;
            if (!CONSEC) {
                if (i < q.d) live |= 1u << k;
                else i = 0;       // an idle slot: it reads element 0's array slot (in bounds) and writes nothing
            }
            const uint32_t c = chunk_of(p, i);
            jj[k] = i - c * p.Z;
            cc[k] = mul_p(p.Ch, c);
        }
        if constexpr (SIGN) {
            const uint32_t step = CONSEC ? p.Cg : mul_p(p.Cg, q.G);
            cg[0] = mul_p(p.Cg, CONSEC ? grp * V : grp);
#pragma unroll
            for (int k = 1; k < V; ++k) cg[k] = add_p(cg[k - 1], step);
#pragma unroll
            for (int k = 0; k < V; ++k) ++cg[k];
        }
    }

    // Array position of pair k for a token whose staged term is th.  `place` is 0 unless blocks are
    // larger than embeddings (Z > d): then it is where the token's embedding starts inside its chunk,
    // place + jj < Z <= m, so one wrap still does.
    __device__ __forceinline__ uint32_t position(const Params &p, uint32_t th, int k, uint32_t place = 0) const
    {
        return wrap(offset_of(p, th, cc[k]) + jj[k] + place, p.m);
    }

    __device__ __forceinline__ uint32_t mask(uint32_t tg, int k) const
    {
        return SIGN ? sign_mask_of_sum(tg, cg[k]) : 0u;
    }

    // v[k] = g * M[idx] for the V owned elements of one token.
    template <typename AT>
    __device__ __forceinline__ void gather(const Params &p, const AT *__restrict__ array,
                                           uint32_t th, uint32_t tg, float (&v)[V], uint32_t place = 0) const
    {
        if constexpr (CONSEC) {
            const uint32_t pos = position(p, th, 0, place);
            if (V == 1 || pos + V <= p.m) {
                load_span<V>(array, pos, v);
            } else {  // the lane's own span crosses the end of the circular array
#pragma unroll
                for (int k = 0; k < V; ++k) v[k] = widen(array[wrap(pos + k, p.m)]);
            }
        } else {
#pragma unroll
            for (int k = 0; k < V; ++k) v[k] = widen(array[position(p, th, k, place)]);   // idle slots read some valid slot
        }
        if constexpr (SIGN) {
#pragma unroll
            for (int k = 0; k < V; ++k) v[k] = apply_sign(v[k], mask(tg, k));
        }
    }

    // grad_array[idx] += g * v[k] for the V owned elements of one token.
    // own: the lane's first element (grp in the strided layout); dlim: elements at or past it do not
    // exist in this row (tables of mixed dimensions; the lane constants are those of the largest).
    __device__ __forceinline__ void scatter(const Params &p, float *__restrict__ grad_array,
                                            uint32_t th, uint32_t tg, const float (&v)[V], uint32_t place = 0,
                                            uint32_t own = 0, uint32_t stride = 0, uint32_t dlim = 0xFFFFFFFFu) const
    {
        const uint32_t pos0 = CONSEC ? position(p, th, 0, place) : 0u;
#pragma unroll
        for (int k = 0; k < V; ++k) {
            // CONSEC: every element wraps on its own
            if (!has(k) || own + (uint32_t)k * stride >= dlim) continue;
            const uint32_t pos = CONSEC ? wrap(pos0 + (uint32_t)k, p.m) : position(p, th, k, place);
            const float val = SIGN ? apply_sign(v[k], mask(tg, k)) : v[k];
            __hip_atomic_fetch_add(grad_array + pos, val, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
};

// The value of lane `lane ^ J`.  Inside rows of 16 lanes by DPP moves, which cost no trip through LDS.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xF, 0xF, false);
}
template <int J>
__device__ __forceinline__ uint32_t xor_lane(uint32_t v)
{
    if constexpr (J == 1) return dpp_move<0xB1>(v);                       // quad_perm [1,0,3,2]
    else if constexpr (J == 2) return dpp_move<0x4E>(v);                  // quad_perm [2,3,0,1]
    else if constexpr (J == 3) return dpp_move<0x1B>(v);                  // quad_perm [3,2,1,0]
    else if constexpr (J == 4) return dpp_move<0x1B>(dpp_move<0x141>(v));
    else if constexpr (J == 7) return dpp_move<0x141>(v);                 // row_half_mirror
    else if constexpr (J == 8) return dpp_move<0x128>(v);                 // row_ror:8
    else if constexpr (J == 15) return dpp_move<0x140>(v);                // row_mirror
    else if constexpr (J == 16) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x401F);
    else if constexpr (J == 31) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x7C1F);
    else return (uint32_t)__shfl_xor((int)v, J);
}

template <int J, int HALF>
__device__ __forceinline__ uint32_t keep_ordered(uint32_t key, uint32_t lane)
{
    const uint32_t other = xor_lane<J>(key), low = min(key, other), high = max(key, other);
    return (lane & HALF) == 0u ? low : high;
}

// The keys of G = 1, 2, 4 .. 64 lanes in ascending order (every group of G lanes on its own; all lanes take part): a bitonic network whose
// stages begin with a comparison against the mirrored lane, so that all go upwards.  18 of its 21 exchanges are
// DPP moves.  The sort of a window was 42 exchanges through LDS with 37-bit keys.  Direct scatter of 53 K lookups of
// d = 16 16.4 -> 15.5 us; combining 117 K tokens 31.2 -> 29.8, 133 K 13.1 -> 12.4, 852 K lookups 92 -> 87.
__device__ __forceinline__ uint32_t sort_lanes(uint32_t key, uint32_t G)
{
    const uint32_t lane = threadIdx.x & 63u;
    if (G >= 2u) key = keep_ordered<1, 1>(key, lane);
    if (G >= 4u) {
        key = keep_ordered<3, 2>(key, lane);
        key = keep_ordered<1, 1>(key, lane);
    }
    if (G >= 8u) {
        key = keep_ordered<7, 4>(key, lane);
        key = keep_ordered<2, 2>(key, lane);
        key = keep_ordered<1, 1>(key, lane);
    }
    if (G >= 16u) {
        key = keep_ordered<15, 8>(key, lane);
        key = keep_ordered<4, 4>(key, lane);
        key = keep_ordered<2, 2>(key, lane);
        key = keep_ordered<1, 1>(key, lane);
    }
    if (G >= 32u) {
        key = keep_ordered<31, 16>(key, lane);
        key = keep_ordered<8, 8>(key, lane);
        key = keep_ordered<4, 4>(key, lane);
        key = keep_ordered<2, 2>(key, lane);
        key = keep_ordered<1, 1>(key, lane);
    }
    if (G >= 64u) {
        key = keep_ordered<63, 32>(key, lane);
        key = keep_ordered<16, 16>(key, lane);
        key = keep_ordered<8, 8>(key, lane);
        key = keep_ordered<4, 4>(key, lane);
        key = keep_ordered<2, 2>(key, lane);
        key = keep_ordered<1, 1>(key, lane);
    }
    return key;
}

// What a window is ordered by: 26 bits of the token's key and the lane it came from; positions without a token last.
// Tokens that differ in the other bits alone may interleave: runs are found by the whole key, so that only cuts some.
__device__ __forceinline__ uint32_t window_key(bool ok, uint32_t key, uint32_t lane)
{
    return ((ok ? min(key & 0x3FFFFFFu, 0x3FFFFFEu) : 0x3FFFFFFu) << 6) | lane;
}
__device__ __forceinline__ bool window_key_ok(uint32_t k) { return k < 0xFFFFFFC0u; }

// Load / store the V owned elements of one output row.
template <int V, bool CONSEC>
__device__ __forceinline__ void store_row(float *__restrict__ row, const Geom &q, uint32_t grp, const float (&v)[V])
{
    if constexpr (CONSEC) {
        typename Vec<V>::A a;
#pragma unroll
        for (int k = 0; k < V; ++k) a[k] = v[k];
        __builtin_nontemporal_store(a, reinterpret_cast<typename Vec<V>::A *>(row + grp * V));
    } else {
#pragma unroll
        for (int k = 0; k < V; ++k)
            if (grp + (uint32_t)k * q.G < q.d) __builtin_nontemporal_store(v[k], row + grp + (uint32_t)k * q.G);
    }
}

// KEEP: the row will be read again soon (the tokens of a bag all read the bag's row), so it is loaded
// with the default cache policy; otherwise it is streamed past the caches' resident lines.
// (strided layout) the same for a row of d elements, d <= q.d
template <int V, bool KEEP>
__device__ __forceinline__ void load_row_of(const float *__restrict__ row, uint32_t G, uint32_t d, uint32_t grp, float (&v)[V])
{
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const uint32_t i = grp + (uint32_t)k * G;
        const float *at = row + (i < d ? i : 0u);           // idle slots read element 0; nobody stores their value
        v[k] = KEEP ? *at : __builtin_nontemporal_load(at);
    }
}

template <int V, bool CONSEC, bool KEEP = false>
__device__ __forceinline__ void load_row(const float *__restrict__ row, const Geom &q, uint32_t grp, float (&v)[V])
{
    if constexpr (CONSEC) {
        const typename Vec<V>::A *at = reinterpret_cast<const typename Vec<V>::A *>(row + grp * V);
        const typename Vec<V>::A a = KEEP ? *at : __builtin_nontemporal_load(at);
#pragma unroll
        for (int k = 0; k < V; ++k) v[k] = a[k];
    } else {
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const uint32_t i = grp + (uint32_t)k * q.G;
            const float *at = row + (i < q.d ? i : 0u);       // idle slots read element 0; nobody stores their value
            v[k] = KEEP ? *at : __builtin_nontemporal_load(at);
        }
    }
}

// Blocks larger than embeddings (Z > d, Section 3.3): r = Z / d consecutive tokens of a table share
// a chunk.  The chunk id x div r takes the token's seat in h, and the embedding starts
// (x mod r) * d places into the chunk.  Otherwise the key is the token and the place is 0.
__device__ __forceinline__ int64_t block_key(const Params &p, int64_t x, uint32_t &place)
{
    place = 0;
    if (p.r == 0) return x;
    place = (uint32_t)((uint64_t)x % p.r) * p.d;
    return (int64_t)((uint64_t)x / p.r);
}

// Token-and-table part of h (and of g) for one token.
__device__ __forceinline__ uint32_t staged_h(const Params &p, int64_t x, uint32_t e)
{
    return mul_add_p(p.Bh, fold_p((uint64_t)x), mul_add_p(p.Ah, e, p.Dh));     // e <= 2^31 - 2 < P
}
__device__ __forceinline__ uint32_t staged_g(const Params &p, int64_t x, uint32_t e)
{
    return mul_add_p(p.Bg, fold_p((uint64_t)x), mul_add_p(p.Ag, e, p.Dg));
}

// ---------------------------------------------------------------------------
// Single-hot forward / backward: one wavefront per tile of TL lookups.
// ---------------------------------------------------------------------------
template <int V, bool CONSEC, bool SIGN, bool BWD, typename AT = float>
__global__ __launch_bounds__(kRowBlock) void single_hot_kernel(Params p, Geom q,
                                                            const AT *__restrict__ src,      // fwd: array; bwd: grad_out
                                                            const int64_t *__restrict__ indices,
                                                            int64_t rows,
                                                            float *__restrict__ dst)         // fwd: out; bwd: grad_array
{
    const uint32_t lane = threadIdx.x & 63u;
    RowWalk w;
    if (!start_walk(q, rows, (int64_t)q.TL, w)) return;  // uniform over the wavefront
    const uint32_t n = (uint32_t)((rows - w.q0) < (int64_t)q.TL ? (rows - w.q0) : (int64_t)q.TL);

    // pass 1: lane l hashes the l-th lookup of the tile
    uint32_t th = 0, tg = 0, pl = 0;
    if (lane < n) {
        const RowRef k = walk_row(q, w, lane, p.d);
        const int64_t x = indices[k.in_row];
        th = staged_h(p, block_key(p, x, pl), k.e);
        if constexpr (SIGN) tg = staged_g(p, x, k.e);
    }

    // pass 2: groups of G lanes walk the tile, 64/G rows per step
    const uint32_t grp = lane & (q.G - 1u);
    const uint32_t sub = lane >> q.g_shift;
    const uint32_t step = 64u >> q.g_shift;
    Lane<V, CONSEC, SIGN> L;
    L.init(p, q, grp);

    for (uint32_t r = 0; r < n; r += step * kUnroll) {  // trip count uniform over the wavefront
        uint32_t rl[kUnroll], thr[kUnroll], tgr[kUnroll], plr[kUnroll];
        bool live[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            rl[u] = r + (uint32_t)u * step + sub;
            live[u] = rl[u] < n;
            const uint32_t srcl = live[u] ? rl[u] : 0u;
            thr[u] = __shfl(th, (int)srcl);
            tgr[u] = SIGN ? __shfl(tg, (int)srcl) : 0u;
            plr[u] = p.r ? __shfl(pl, (int)srcl) : 0u;
        }
        if constexpr (!BWD) {
            float v[kUnroll][V];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) L.gather(p, src, thr[u], tgr[u], v[u], plr[u]);  // lookup 0 stands in for dead slots
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                if (live[u]) store_row<V, CONSEC>(dst + walk_row(q, w, rl[u], p.d).out_off, q, grp, v[u]);
        } else {
            float v[kUnroll][V];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const uint32_t safe = live[u] ? rl[u] : 0u;
                load_row<V, CONSEC>(src + walk_row(q, w, safe, p.d).out_off, q, grp, v[u]);
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                if (live[u]) L.scatter(p, dst, thr[u], tgr[u], v[u], plr[u]);
        }
    }
}

// ---------------------------------------------------------------------------
// Single-hot forward for blocks of at least four lanes' elements (Z >= 4V, or Z > d), consecutive layout.
//
// The kernel above hashes a block's offset in every lane that reads a part of it.  Here a lane hashes
// one (lookup, chunk) pair - the 64 / G * kUnroll lookups of a pass have at most 64 of them - and the
// lanes that read the block fetch its offset.  Vector instructions per wavefront of eight lookups
// (d = 128, Z = 32): 510 -> 260 with the sign, 343 -> 179 without.
// 852 K lookups with the sign 147 -> 142 us.  More lookups in flight per wavefront or several passes in
// its life do not help (143 against 145 ... 150), fewer neither (two 143, one 156).
// ---------------------------------------------------------------------------
template <int V, bool SIGN, typename AT>
__global__ __launch_bounds__(kRowBlock) void single_hot_block_kernel(Params p, Geom q,
                                                                  const AT *__restrict__ array,
                                                                  const int64_t *__restrict__ indices,
                                                                  int64_t rows,
                                                                  float *__restrict__ out)
{
    const uint32_t lane = threadIdx.x & 63u;
    RowWalk w;
    if (!start_walk(q, rows, (int64_t)q.TL, w)) return;  // uniform over the wavefront
    const uint32_t n = (uint32_t)((rows - w.q0) < (int64_t)q.TL ? (rows - w.q0) : (int64_t)q.TL);
    const RowLine line = line_of(q, w, n, p.d);
    const uint32_t c_shift = q.c_shift, C = 1u << c_shift;       // chunks of an embedding
    const uint32_t mine = lane >> c_shift;                       // which lookup of a pass this lane hashes a chunk of
    const uint32_t sub = lane >> q.g_shift, step = 64u >> q.g_shift;
    const uint32_t pass = step * kUnroll;

    for (uint32_t r = 0; r < n; r += pass) {              // trip count uniform over the wavefront
        const uint32_t end = r + pass < n ? r + pass : n;
        const bool have = r + mine < end;
        int64_t x = 0;
        uint32_t e = 0;
        if (line.on) {
            if (have) x = indices[line.in0 + (int64_t)((r + mine) * line.in_step)];
            e = line_table(q, w, r + mine);
        } else if (have) {
            const RowRef k = walk_row(q, w, r + mine, p.d);
            x = indices[k.in_row];
            e = k.e;
        }
        // (what does not need the id, while it is on its way)
        const uint32_t grp = lane & (q.G - 1u);
        const uint32_t i0 = grp * V, c = p.C == 1u ? 0u : i0 >> q.z_shift, jj = i0 - (c << q.z_shift);
        const uint32_t cc = mul_p(p.Ch, lane & (C - 1u));
        uint32_t cg[V];
        if constexpr (SIGN) {
            cg[0] = mul_p(p.Cg, i0);
#pragma unroll
            for (int k = 1; k < V; ++k) cg[k] = add_p(cg[k - 1], p.Cg);
        }
        uint32_t o = 0, tg = 0, place;
        const int64_t key = block_key(p, x, place);
        o = wrap(offset_of(p, staged_h(p, key, e), cc) + place, p.m);
        if constexpr (SIGN) tg = staged_g(p, x, e) + 1u;
        const uint32_t from = (sub << c_shift) + c;           // the lane that hashed this lane's block, of the first lookups

        uint32_t pos[kUnroll], tgr[kUnroll];
        bool live[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int at = (int)(from + ((uint32_t)u * step << c_shift));
            live[u] = r + (uint32_t)u * step + sub < end;
            pos[u] = wrap(__shfl(o, at) + jj, p.m);
            tgr[u] = SIGN ? __shfl(tg, at) : 0u;
        }
        float v[kUnroll][V];
        load_spans<V, kUnroll>(p, array, pos, live, v);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            if (!live[u]) continue;
            if constexpr (SIGN) {
#pragma unroll
                for (int k = 0; k < V; ++k) v[u][k] = apply_sign(v[u][k], sign_mask_of_sum(cg[k], tgr[u]));
            }
            const uint32_t row = r + (uint32_t)u * step + sub;
            if (line.on) store_row<V, true>(out + line.out0 + row * line.out_step, q, grp, v[u]);
            else store_row<V, true>(out + walk_row(q, w, row, p.d).out_off, q, grp, v[u]);
        }
    }
}

// ---------------------------------------------------------------------------
// Single-hot backward for the direct scatter, with the duplicates of a tile combined first.
//
// Float atomics on one address serialise (tens of nanoseconds each), and a table with a handful of
// distinct tokens sends thousands of lookups of a batch to the same d addresses.  A wavefront takes
// a tile of 64 lookups - with the table-by-table row walk, 64 consecutive samples of one table -
// finds the distinct tokens among them (ballots over the staged hash terms), and every lane group
// sums the gradient rows of one distinct token at a time and scatters the sum once.  Strided lane
// layout (lanes of a group on consecutive addresses), as in the plain scatter.
// ---------------------------------------------------------------------------
template <int V, bool SIGN>
__global__ __launch_bounds__(kRowBlock) void single_hot_backward_tile_kernel(Params p, Geom q,
                                                                          const float *__restrict__ grad_out,
                                                                          const int64_t *__restrict__ indices,
                                                                          int64_t rows,
                                                                          float *__restrict__ grad_array)
{
    const uint32_t lane = threadIdx.x & 63u;
    RowWalk w;
    if (!start_walk(q, rows, 64, w)) return;             // uniform over the wavefront
    const uint32_t n = (uint32_t)((rows - w.q0) < 64 ? (rows - w.q0) : 64);

    // lane l hashes the l-th lookup of the tile
    uint32_t th = 0, tg = 0, pl = 0;
    const bool have = lane < n;
    if (have) {
        const RowRef k = walk_row(q, w, lane, p.d);
        const int64_t x = indices[k.in_row];
        th = staged_h(p, block_key(p, x, pl), k.e);
        if constexpr (SIGN) tg = staged_g(p, x, k.e);
    }
    // Distinct tokens: the lowest lane of every set of equal (th, place, tg) leads it and keeps the
    // set.  (Equal th and place mean equal offsets; with the sign on, equal tg as well means equal signs.)
    uint64_t remaining = __ballot(have), members = 0;
    while (remaining) {                                   // one round per distinct token; uniform
        const int lead = __ffsll((unsigned long long)remaining) - 1;
        const uint32_t lth = __shfl(th, lead), ltg = SIGN ? __shfl(tg, lead) : 0u, lpl = __shfl(pl, lead);
        const uint64_t same = __ballot(have && th == lth && pl == lpl && (!SIGN || tg == ltg));
        if ((int)lane == lead) members = same;
        remaining &= ~same;
    }
    const uint32_t mem_lo = (uint32_t)members, mem_hi = (uint32_t)(members >> 32);

    const uint32_t grp = lane & (q.G - 1u);
    const uint32_t sub = lane >> q.g_shift;
    const uint32_t step = 64u >> q.g_shift;               // lane groups per wavefront
    Lane<V, false, SIGN> L;
    L.init(p, q, grp);

    // Group `sub` takes the leaders among lanes sub, sub + step, ..., kUnroll of them at a time: the
    // first row of each is requested at once (distinct tokens keep kUnroll rows in flight, as in the
    // plain scatter), the further rows of a set follow, and every set is scattered once.
    for (uint32_t l0 = 0; l0 < 64u; l0 += step * kUnroll) {        // same trip count for every lane
        uint64_t todo[kUnroll];
        uint32_t lth[kUnroll], ltg[kUnroll], lpl[kUnroll];
        bool any_rows[kUnroll];
        float acc[kUnroll][V];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const uint32_t lead = l0 + (uint32_t)u * step + sub;
            const bool in = lead < 64u;
            const int from = (int)(in ? lead : 0u);
            todo[u] = ((uint64_t)__shfl(mem_hi, from) << 32) | __shfl(mem_lo, from);
            if (!in) todo[u] = 0;
            lth[u] = __shfl(th, from);
            ltg[u] = SIGN ? __shfl(tg, from) : 0u;
            lpl[u] = p.r ? __shfl(pl, from) : 0u;
            any_rows[u] = todo[u] != 0;
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {                         // first row of every set
            const uint32_t j = any_rows[u] ? (uint32_t)(__ffsll((unsigned long long)todo[u]) - 1) : 0u;
            todo[u] &= todo[u] - 1u;                               // (0 stays 0)
            load_row<V, false>(grad_out + walk_row(q, w, j, p.d).out_off, q, grp, acc[u]);   // lookup 0 stands in
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {                         // the other rows of the set
            while (__any(todo[u] != 0)) {
                float v[kUnroll][V];
                bool live[kUnroll];
#pragma unroll
                for (int t = 0; t < kUnroll; ++t) {
                    live[t] = todo[u] != 0;
                    const uint32_t j = live[t] ? (uint32_t)(__ffsll((unsigned long long)todo[u]) - 1) : 0u;
                    todo[u] &= todo[u] - 1u;
                    load_row<V, false>(grad_out + walk_row(q, w, j, p.d).out_off, q, grp, v[t]);
                }
#pragma unroll
                for (int t = 0; t < kUnroll; ++t) {
                    if (live[t]) {
#pragma unroll
                        for (int k = 0; k < V; ++k) acc[u][k] += v[t][k];
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
            if (any_rows[u]) L.scatter(p, grad_array, lth[u], ltg[u], acc[u], lpl[u]);
    }
}

// ---------------------------------------------------------------------------
// The same for rows of several lane groups to a wavefront (G <= 32; taken for rows of up to 48 floats).
//
// At the sizes that come here (some ten thousand lookups) a SIMD holds one wavefront and the kernel is a
// chain of latencies.  The one above finds the distinct tokens one by one, 64 rounds of dependent lane
// exchanges where most tokens differ, and its groups then meet unequal sets.  Here the wavefront sorts
// its 64 lookups by token (sort_lanes); every group walks the G lookups
// that its own lanes hold and adds runs in registers; a run that goes on in the next group is handed
// over, so that a token still costs one row of atomics per tile.  53248 lookups, d = 16, Z = 4: 20.9 us
// before, 16.7 now; with one group per wavefront (d = 128) the walk is 64 rows long and loses
// (52000 lookups: 74 against 94 us with the forward), so those keep the kernel above.
// ---------------------------------------------------------------------------
constexpr int kWindowRows = 8;          // gradient rows a lane group requests before it adds them

template <int V, bool SIGN>
__global__ __launch_bounds__(kRowBlock) void single_hot_backward_window_kernel(Params p, Geom q,
                                                                          const float *__restrict__ grad_out,
                                                                          const int64_t *__restrict__ indices,
                                                                          int64_t rows,
                                                                          float *__restrict__ grad_array)
{
    const uint32_t lane = threadIdx.x & 63u;
    RowWalk w;
    if (!start_walk(q, rows, 64, w)) return;             // uniform over the wavefront
    const uint32_t n = (uint32_t)((rows - w.q0) < 64 ? (rows - w.q0) : 64);

    // lane l hashes the l-th lookup of the tile
    uint32_t th = 0, tg = 0, pl = 0;
    uint64_t at = 0;                                      // first float of its gradient row
    if (lane < n) {
        const RowRef k = walk_row(q, w, lane, p.d);
        const int64_t x = indices[k.in_row];
        th = staged_h(p, block_key(p, x, pl), k.e);
        if constexpr (SIGN) tg = staged_g(p, x, k.e);
        at = (uint64_t)k.out_off;
    }
    const uint32_t grp = lane & (q.G - 1u);
    const uint32_t base_lane = lane - grp;
    Lane<V, false, SIGN> L;
    L.init(p, q, grp);                                    // (while the ids are on their way)

    // Equal (th, place, tg) mean equal offsets and signs.  They are brought side by side by a mix of the
    // three; what a run is, is decided on all three below.
    {
        const uint32_t mix = th + pl * 0x9E3779B1u + (SIGN ? tg * 0x85EBCA6Bu : 0u);
        const uint32_t sk = sort_lanes(window_key(lane < n, mix, lane), 64u);
        const int from = (int)(sk & 63u);                 // (lookups past the end sort last: n of them stay in front)
        th = __shfl(th, from);
        if (p.r) pl = __shfl(pl, from);
        if constexpr (SIGN) tg = __shfl(tg, from);
        const uint32_t lo = __shfl((uint32_t)at, from), hi = __shfl((uint32_t)(at >> 32), from);
        at = ((uint64_t)hi << 32) | lo;
    }
    // is this token another than the one before?
    const int prev = (int)(lane ? lane - 1u : 0u);
    const uint32_t p_th = __shfl(th, prev), p_pl = p.r ? __shfl(pl, prev) : 0u, p_tg = SIGN ? __shfl(tg, prev) : 0u;
    const bool head = lane == 0 || p_th != th || (p.r && p_pl != pl) || (SIGN && p_tg != tg);
    const uint64_t heads = __ballot(head && lane < n);
    const uint64_t mine = (heads >> base_lane) & ((1ull << q.G) - 1ull);    // of this group's lookups (G <= 32)
    const bool joins = base_lane < n && (mine & 1ull) == 0;                 // the first run began in the group before

    float acc[V], first[V];                               // the open run; the group's first run, if it joins the group before
#pragma unroll
    for (int k = 0; k < V; ++k) acc[k] = first[k] = 0.0f;
    uint32_t run_th = 0, run_tg = 0, run_pl = 0, first_th = 0, first_tg = 0, first_pl = 0;
    bool open = false, joining = joins;
    for (uint32_t k0 = 0; k0 < q.G; k0 += kWindowRows) {    // same trip count for every lane
        uint32_t rth[kWindowRows], rtg[kWindowRows], rpl[kWindowRows];
        bool ok[kWindowRows], rhead[kWindowRows];
        float v[kWindowRows][V];
#pragma unroll
        for (int u = 0; u < kWindowRows; ++u) {
            const uint32_t of = base_lane + ((k0 + u) & (q.G - 1u));
            ok[u] = k0 + u < q.G && of < n;
            rth[u] = __shfl(th, (int)of);
            rtg[u] = SIGN ? __shfl(tg, (int)of) : 0u;
            rpl[u] = p.r ? __shfl(pl, (int)of) : 0u;
            rhead[u] = __shfl((int)head, (int)of) != 0;
            const uint32_t lo = __shfl((uint32_t)at, (int)of), hi = __shfl((uint32_t)(at >> 32), (int)of);
            if (ok[u]) load_row<V, false>(grad_out + (((uint64_t)hi << 32) | lo), q, grp, v[u]);
        }
#pragma unroll
        for (int u = 0; u < kWindowRows; ++u) {
            if (!ok[u]) continue;
            if (rhead[u] && open) {
                if (joining) {                            // handed over by the group before: it waits for what that one has
#pragma unroll
                    for (int k = 0; k < V; ++k) first[k] = acc[k];
                    first_th = run_th;
                    first_tg = run_tg;
                    first_pl = run_pl;
                    joining = false;
                } else {
                    L.scatter(p, grad_array, run_th, run_tg, acc, run_pl);
                }
#pragma unroll
                for (int k = 0; k < V; ++k) acc[k] = 0.0f;
            }
#pragma unroll
            for (int k = 0; k < V; ++k) acc[k] += v[u][k];
            run_th = rth[u];
            run_tg = rtg[u];
            run_pl = rpl[u];
            open = true;
        }
    }
    // Hand the open runs over, group by group: a group whose lookups are one run adds what it gets to its
    // own and passes it on, any other finishes its first run with it.
    const uint32_t sub = lane >> q.g_shift, groups = 64u >> q.g_shift;
    const bool one_run = joins && (mine == 0);
    for (uint32_t s = 1; s < groups; ++s) {               // uniform
        float got[V];
#pragma unroll
        for (int k = 0; k < V; ++k) got[k] = __shfl(acc[k], (int)(lane >= q.G ? lane - q.G : lane));
        if (sub != s || !joins) continue;
#pragma unroll
        for (int k = 0; k < V; ++k) {
            if (one_run) acc[k] += got[k];
            else first[k] += got[k];
        }
    }
    if (joins && !one_run) L.scatter(p, grad_array, first_th, first_tg, first, first_pl);
    const uint32_t after = base_lane + q.G;               // the next group's first lookup
    const bool handed = after < n && after < 64u && ((heads >> (after & 63u)) & 1ull) == 0;
    if (open && !handed) L.scatter(p, grad_array, run_th, run_tg, acc, run_pl);
}

// ---------------------------------------------------------------------------
// Bag-sum forward / bag backward: one group of G lanes per bag, 64/G bags per
// wavefront.  A group stages up to G of its bag's tokens at a time.
// ---------------------------------------------------------------------------
template <int V, bool CONSEC, bool SIGN, bool BWD, typename AT = float>
__global__ __launch_bounds__(kRowBlock) void bag_kernel(Params p, Geom q,
                                                     const AT *__restrict__ src,         // fwd: array; bwd: grad_out
                                                     const int64_t *__restrict__ indices,
                                                     const int64_t *__restrict__ offsets,
                                                     int64_t rows, int64_t n_indices,
                                                     float *__restrict__ dst)            // fwd: out; bwd: grad_array
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t step = 64u >> q.g_shift;                 // bags per wavefront
    RowWalk w;
    if (!start_walk(q, rows, (int64_t)step, w)) return;     // uniform over the wavefront
    const uint32_t grp = lane & (q.G - 1u);
    const uint32_t sub = lane >> q.g_shift;
    const uint32_t base_lane = lane - grp;                  // first lane of this group
    const bool have_bag = w.q0 + sub < rows;
    const RowRef bag = walk_row(q, w, have_bag ? sub : 0u, p.d);
    const uint32_t e = bag.e;

    int64_t t0 = 0, t1 = 0;
    if (have_bag) {
        t0 = offsets[bag.in_row];
        t1 = offsets[bag.in_row + 1];
        t0 = t0 < 0 ? 0 : (t0 > n_indices ? n_indices : t0);
        t1 = t1 < t0 ? t0 : (t1 > n_indices ? n_indices : t1);
    }

    Lane<V, CONSEC, SIGN> L;
    L.init(p, q, grp);

    float acc[V];
#pragma unroll
    for (int k = 0; k < V; ++k) acc[k] = 0.0f;
    if constexpr (BWD) {
        if (have_bag) load_row<V, CONSEC>(src + bag.out_off, q, grp, acc);
    }

    for (int64_t tb = t0; __any(tb < t1); tb += q.G) {
        // stage: lane `grp` of the group hashes token tb + grp
        const int64_t left = t1 - tb;                       // <= 0 once this group is done
        const uint32_t cnt = left <= 0 ? 0u : (left < (int64_t)q.G ? (uint32_t)left : q.G);
        uint32_t th = 0, tg = 0, pl = 0;
        if (grp < cnt) {
            const int64_t x = indices[tb + grp];
            th = staged_h(p, block_key(p, x, pl), e);
            if constexpr (SIGN) tg = staged_g(p, x, e);
        }
        for (uint32_t u0 = 0; __any(u0 < cnt); u0 += kUnroll) {
            uint32_t thr[kUnroll], tgr[kUnroll], plr[kUnroll];
            bool live[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                live[u] = u0 + u < cnt;
                const uint32_t srcl = base_lane + (live[u] ? u0 + u : 0u);
                thr[u] = __shfl(th, (int)srcl);
                tgr[u] = SIGN ? __shfl(tg, (int)srcl) : 0u;
                plr[u] = p.r ? __shfl(pl, (int)srcl) : 0u;
            }
            if constexpr (!BWD) {
                float v[kUnroll][V];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) L.gather(p, src, thr[u], tgr[u], v[u], plr[u]);
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    if (live[u]) {
#pragma unroll
                        for (int k = 0; k < V; ++k) acc[k] += v[u][k];
                    }
                }
            } else {
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
                    if (live[u]) L.scatter(p, dst, thr[u], tgr[u], acc, plr[u]);
            }
        }
    }
    if constexpr (!BWD) {
        if (have_bag) store_row<V, CONSEC>(dst + bag.out_off, q, grp, acc);
    }
}

// ---------------------------------------------------------------------------
// Bag-sum forward for blocks of at least four lanes' elements, consecutive layout: as bag_kernel, but the
// offset of a (token, chunk) pair is hashed by one lane (see single_hot_block_kernel).  A lane group hashes the
// chunks of Z / V tokens at a time, and slots past the end of a bag read nothing.  426 K bags of 20, 1 GB array
// (bfloat16 copy): 570 -> 555 us; float array, with its backward 2412 -> 2377.
// ---------------------------------------------------------------------------
template <int V, bool SIGN, typename AT>
__global__ __launch_bounds__(kRowBlock) void bag_block_kernel(Params p, Geom q,
                                                              const AT *__restrict__ array,
                                                              const int64_t *__restrict__ indices,
                                                              const int64_t *__restrict__ offsets,
                                                              int64_t rows, int64_t n_indices,
                                                              float *__restrict__ out)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t step = 64u >> q.g_shift;                 // bags per wavefront
    RowWalk w;
    if (!start_walk(q, rows, (int64_t)step, w)) return;     // uniform over the wavefront
    const uint32_t grp = lane & (q.G - 1u);
    const uint32_t sub = lane >> q.g_shift;
    const uint32_t base_lane = lane - grp;                  // first lane of this group
    const bool have_bag = w.q0 + sub < rows;
    const RowRef bag = walk_row(q, w, have_bag ? sub : 0u, p.d);

    int64_t t0 = 0, t1 = 0;
    if (have_bag) {
        t0 = offsets[bag.in_row];
        t1 = offsets[bag.in_row + 1];
        t0 = t0 < 0 ? 0 : (t0 > n_indices ? n_indices : t0);
        t1 = t1 < t0 ? t0 : (t1 > n_indices ? n_indices : t1);
    }

    // chunk and place in it of this lane's elements; the pair this lane hashes: token grp >> c_shift, chunk
    // grp & (C - 1) of every round of `round` tokens
    const uint32_t C = 1u << q.c_shift, i0 = grp * V;
    const uint32_t c = p.C == 1u ? 0u : i0 >> q.z_shift, jj = i0 - (c << q.z_shift);
    const uint32_t cc = mul_p(p.Ch, grp & (C - 1u));
    const uint32_t round = q.G >> q.c_shift, my_token = grp >> q.c_shift;
    uint32_t cg[V];
    if constexpr (SIGN) {
        cg[0] = mul_p(p.Cg, i0);
#pragma unroll
        for (int k = 1; k < V; ++k) cg[k] = add_p(cg[k - 1], p.Cg);
    }
    // the parts of h and g that all tokens of the bag share
    const uint32_t th0 = mul_add_p(p.Ah, bag.e, p.Dh), tg0 = SIGN ? mul_add_p(p.Ag, bag.e, p.Dg) : 0u;

    float acc[V];
#pragma unroll
    for (int k = 0; k < V; ++k) acc[k] = 0.0f;

    for (int64_t tb = t0; __any(tb < t1); tb += q.G) {
        // lane `grp` of the group hashes token tb + grp
        const int64_t left = t1 - tb;                       // <= 0 once this group is done
        const uint32_t cnt = left <= 0 ? 0u : (left < (int64_t)q.G ? (uint32_t)left : q.G);
        uint32_t th = 0, tg = 0, pl = 0;
        if (grp < cnt) {
            const int64_t x = indices[tb + grp];
            th = mul_add_p(p.Bh, fold_p((uint64_t)block_key(p, x, pl)), th0);
            if constexpr (SIGN) tg = mul_add_p(p.Bg, fold_p((uint64_t)x), tg0) + 1u;
        }
        for (uint32_t r0 = 0; __any(r0 < cnt); r0 += round) {
            const int of = (int)(base_lane + r0 + my_token);             // r0 + my_token < G
            uint32_t o = offset_of(p, __shfl(th, of), cc);
            if (p.r) o = wrap(o + __shfl(pl, of), p.m);
            for (uint32_t u0 = 0; u0 < round && __any(r0 + u0 < cnt); u0 += kUnroll) {
                uint32_t pos[kUnroll], tgr[kUnroll];
                bool live[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    live[u] = r0 + u0 + u < cnt;
                    pos[u] = wrap(__shfl(o, (int)(base_lane + ((u0 + (uint32_t)u) << q.c_shift) + c)) + jj, p.m);
                    tgr[u] = SIGN ? __shfl(tg, (int)(base_lane + r0 + u0 + u)) : 0u;
                }
                float v[kUnroll][V];
                load_spans<V, kUnroll>(p, array, pos, live, v);
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    if (!live[u]) continue;
#pragma unroll
                    for (int k = 0; k < V; ++k)
                        acc[k] += SIGN ? apply_sign(v[u][k], sign_mask_of_sum(cg[k], tgr[u])) : v[u][k];
                }
            }
        }
    }
    if (have_bag) store_row<V, true>(out + bag.out_off, q, grp, acc);
}

// ---------------------------------------------------------------------------
// Bag-sum forward for short bags: a lane group takes kShortBags bags at a time.
//
// A bag of a few tokens is four dependent trips to memory (bounds, ids, array, and the store's way out)
// around almost no work, and a wavefront that did one per lane group and left spent its life in them.
// The bounds of all its bags are requested together, then their tokens' ids (a lane per token, whatever
// bag it belongs to), and the array is read kUnroll tokens at a time across the bags' ends.  Tokens are
// added in their order, so the sums are those of bag_kernel bit for bit.
// 39013 bags of 3 on average, d = 100, Z = 10, signs: 31.0 us with one bag per group, 24.0 with four.
// ---------------------------------------------------------------------------
constexpr uint32_t kShortBags = 4;

template <int V, bool CONSEC, bool SIGN, typename AT>
__global__ __launch_bounds__(kRowBlock) void short_bag_kernel(Params p, Geom q,
                                                           const AT *__restrict__ array,
                                                           const int64_t *__restrict__ indices,
                                                           const int64_t *__restrict__ offsets,
                                                           int64_t rows, int64_t n_indices,
                                                           float *__restrict__ out)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t step = 64u >> q.g_shift;                 // lane groups per wavefront
    RowWalk w;
    if (!start_walk(q, rows, (int64_t)(step * kShortBags), w)) return;     // uniform over the wavefront
    const uint32_t grp = lane & (q.G - 1u);
    const uint32_t first = (lane >> q.g_shift) * kShortBags;               // this group's first row of the wavefront's
    const uint32_t base_lane = lane - grp;
    const int64_t left = rows - w.q0 - (int64_t)first;
    const uint32_t bags = left <= 0 ? 0u : (left < (int64_t)kShortBags ? (uint32_t)left : kShortBags);

    // bounds of the bags; cum[k]: tokens in the bags before bag k
    int64_t t0[kShortBags], to[kShortBags];
    uint32_t e[kShortBags], cum[kShortBags + 1];
    {
        int64_t t1[kShortBags];
#pragma unroll
        for (uint32_t k = 0; k < kShortBags; ++k) {
            const RowRef r = walk_row(q, w, k < bags ? first + k : 0u, p.d);
            e[k] = r.e;
            to[k] = r.out_off;
            t0[k] = offsets[r.in_row];
            t1[k] = offsets[r.in_row + 1];
        }
        cum[0] = 0;
#pragma unroll
        for (uint32_t k = 0; k < kShortBags; ++k) {
            t0[k] = t0[k] < 0 ? 0 : (t0[k] > n_indices ? n_indices : t0[k]);
            t1[k] = t1[k] < t0[k] ? t0[k] : (t1[k] > n_indices ? n_indices : t1[k]);
            const uint64_t c = k < bags ? (uint64_t)(t1[k] - t0[k]) : 0u;
            cum[k + 1] = cum[k] + (uint32_t)c;              // (below 2^31: the host takes this kernel below 2^29 tokens)
        }
    }
    const uint32_t total = cum[kShortBags];

    Lane<V, CONSEC, SIGN> L;
    L.init(p, q, grp);

    float acc[V];
#pragma unroll
    for (int k = 0; k < V; ++k) acc[k] = 0.0f;
    uint32_t cur = 0;                                        // the bag that acc belongs to
    // write the bags up to (not including) `next`: the one being summed, then empty ones
    auto finish = [&](uint32_t next) {
#pragma unroll
        for (uint32_t k = 0; k < kShortBags; ++k) {
            if (k >= cur && k < next) {
                store_row<V, CONSEC>(out + to[k], q, grp, acc);
#pragma unroll
                for (int i = 0; i < V; ++i) acc[i] = 0.0f;
            }
        }
        cur = next;
    };
    for (uint32_t tb = 0; __any(tb < total); tb += q.G) {
        const uint32_t cnt = tb >= total ? 0u : (total - tb < q.G ? total - tb : q.G);
        uint32_t th = 0, tg = 0, pl = 0;
        if (grp < cnt) {
            const uint32_t j = tb + grp;
            int64_t at = t0[0];
            uint32_t ek = e[0], before = 0;
#pragma unroll
            for (uint32_t k = 1; k < kShortBags; ++k) {
                if (j >= cum[k]) {
                    at = t0[k];
                    ek = e[k];
                    before = cum[k];
                }
            }
            const int64_t x = indices[at + (int64_t)(j - before)];
            th = staged_h(p, block_key(p, x, pl), ek);
            if constexpr (SIGN) tg = staged_g(p, x, ek);
        }
        for (uint32_t u0 = 0; __any(u0 < cnt); u0 += kUnroll) {
            uint32_t thr[kUnroll], tgr[kUnroll], plr[kUnroll];
            bool live[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                live[u] = u0 + u < cnt;
                const uint32_t srcl = base_lane + (live[u] ? u0 + u : 0u);
                thr[u] = __shfl(th, (int)srcl);
                tgr[u] = SIGN ? __shfl(tg, (int)srcl) : 0u;
                plr[u] = p.r ? __shfl(pl, (int)srcl) : 0u;
            }
            float v[kUnroll][V];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) L.gather(p, array, thr[u], tgr[u], v[u], plr[u]);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                if (live[u]) {
                    const uint32_t j = tb + u0 + (uint32_t)u;
                    uint32_t bag = 0;                        // the last one that starts at or before token j
#pragma unroll
                    for (uint32_t k = 1; k < kShortBags; ++k) bag += j >= cum[k] ? 1u : 0u;
                    if (bag != cur) finish(bag);
#pragma unroll
                    for (int k = 0; k < V; ++k) acc[k] += v[u][k];
                }
            }
        }
    }
    finish(bags);
}

// ---------------------------------------------------------------------------
// Shape-generic fallback (any d, Z with Z | d): one thread per (row, element),
// every hash evaluated in full by the thread that needs it.
// ---------------------------------------------------------------------------
template <bool SIGN, bool BWD, typename AT = float>
__global__ __launch_bounds__(kBlock) void generic_kernel(Params p, Geom q, uint32_t rows_per_block,
                                                         const AT *__restrict__ src,
                                                         const int64_t *__restrict__ indices,
                                                         const int64_t *__restrict__ offsets,  // NULL: single-hot
                                                         int64_t rows, int64_t n_indices,
                                                         float *__restrict__ dst)
{
    const int64_t row_base = (int64_t)blockIdx.x * rows_per_block;
    const uint64_t items = (uint64_t)rows_per_block * p.d;
    for (uint64_t local = threadIdx.x; local < items; local += kBlock) {
        const uint32_t rl = (uint32_t)(local / p.d);
        const uint32_t i = (uint32_t)(local - (uint64_t)rl * p.d);
        const int64_t row = row_base + rl;
        if (row >= rows) break;
        const int64_t b = row / (int64_t)q.F;
        const uint32_t f = (uint32_t)(row - b * (int64_t)q.F);
        const uint32_t e = q.e0 + f;
        const int64_t in_row = b * (int64_t)q.F_in + e;
        const int64_t at = b * q.row_floats + q.col0 + (int64_t)f * p.d + i;   // this element in out / grad_out
        const uint32_t c = i / p.Z, j = i - c * p.Z;
        const uint32_t cc = mod_p((uint64_t)p.Ch * c);
        const uint32_t cg = SIGN ? mod_p((uint64_t)p.Cg * i) : 0u;
        int64_t t0 = in_row, t1 = in_row + 1;
        if (offsets != nullptr) {
            t0 = offsets[in_row];
            t1 = offsets[in_row + 1];
            t0 = t0 < 0 ? 0 : (t0 > n_indices ? n_indices : t0);
            t1 = t1 < t0 ? t0 : (t1 > n_indices ? n_indices : t1);
        }
        float acc = 0.0f;
        if constexpr (BWD) acc = src[at];
        for (int64_t t = t0; t < t1; ++t) {
            const int64_t x = indices[t];
            // Z > d (Section 3.3): r = Z/d embeddings share a chunk; the chunk id x / r takes the
            // token's seat in h and the embedding starts (x mod r) * d places into the chunk
            const int64_t key = p.r ? (int64_t)((uint64_t)x / p.r) : x;
            const uint32_t place = p.r ? (uint32_t)((uint64_t)x % p.r) * p.d : 0u;
            const uint32_t pos = wrap(offset_of(p, staged_h(p, key, e), cc) + j + place, p.m);
            const uint32_t msk = SIGN ? sign_mask(add_p(staged_g(p, x, e), cg)) : 0u;
            if constexpr (BWD) {
                __hip_atomic_fetch_add(dst + pos, apply_sign(acc, msk), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                const float v = apply_sign(widen(src[pos]), msk);
                acc = (offsets == nullptr) ? v : acc + v;   // single-hot keeps the sign of zero
            }
        }
        if constexpr (!BWD) dst[at] = acc;
    }
}

// ---------------------------------------------------------------------------
// float32 array -> bfloat16 array (post-hoc quantisation of a trained array).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void to_bf16_kernel(const float *__restrict__ src, uint16_t *__restrict__ dst,
                                                         uint64_t n, int vec_ok)
{
    const uint64_t tid = (uint64_t)blockIdx.x * kBlock + threadIdx.x, stride = (uint64_t)gridDim.x * kBlock;
    const uint64_t nvec = vec_ok ? n / 4u : 0u;
    for (uint64_t i = tid; i < nvec; i += stride) {
        const Vec<4>::A a = __builtin_nontemporal_load(reinterpret_cast<const Vec<4>::A *>(src) + i);
        Vec<4>::HA h;
#pragma unroll
        for (int k = 0; k < 4; ++k) h[k] = narrow_bf16(a[k]);
        __builtin_nontemporal_store(h, reinterpret_cast<Vec<4>::HA *>(dst) + i);
    }
    for (uint64_t i = 4u * nvec + tid; i < n; i += stride) dst[i] = narrow_bf16(src[i]);
}

// ---------------------------------------------------------------------------
// Integer maps alone (testing aid): one thread per (lookup, chunk) / (lookup, element).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void offsets_kernel(Params p, uint32_t F, const int64_t *__restrict__ indices,
                                                         int64_t n, int64_t *__restrict__ out)
{
    const int64_t total = n * (int64_t)p.C;
    for (int64_t it = (int64_t)blockIdx.x * kBlock + threadIdx.x; it < total; it += (int64_t)gridDim.x * kBlock) {
        const int64_t k = it / p.C;
        const uint32_t c = (uint32_t)(it - k * p.C);
        const uint32_t e = (uint32_t)(k % (int64_t)F);
        const int64_t x = indices[k];
        if (p.r) {  // Z > d: one entry per lookup, the place of element 0
            const uint32_t place = (uint32_t)((uint64_t)x % p.r) * p.d;
            out[it] = (int64_t)wrap(offset_of(p, staged_h(p, (int64_t)((uint64_t)x / p.r), e), 0u) + place, p.m);
        } else {
            out[it] = (int64_t)offset_of(p, staged_h(p, x, e), mod_p((uint64_t)p.Ch * c));
        }
    }
}

__global__ __launch_bounds__(kBlock) void signs_kernel(Params p, uint32_t F, uint32_t use_sign,
                                                       const int64_t *__restrict__ indices, int64_t n,
                                                       int8_t *__restrict__ out)
{
    const int64_t total = n * (int64_t)p.d;
    for (int64_t it = (int64_t)blockIdx.x * kBlock + threadIdx.x; it < total; it += (int64_t)gridDim.x * kBlock) {
        const int64_t k = it / p.d;
        const uint32_t i = (uint32_t)(it - k * p.d);
        const uint32_t e = (uint32_t)(k % (int64_t)F);
        const uint32_t res = add_p(staged_g(p, indices[k], e), mod_p((uint64_t)p.Cg * i));
        out[it] = (!use_sign || (res & 1u)) ? (int8_t)1 : (int8_t)-1;
    }
}

// ---------------------------------------------------------------------------
// Optimizer steps on touched slots (Adagrad, SGD).  Explicitly rounded float32 steps (no contraction).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void adagrad_one(float &w, float &s, float g, float lr, float eps)
{
    s = __fadd_rn(s, __fmul_rn(g, g));
    w = __fsub_rn(w, __fdiv_rn(__fmul_rn(lr, g), __fadd_rn(__fsqrt_rn(s), eps)));
}

// One thread per vector of V slots, no loop: measured fastest on MI355X (deeper per-thread
// unrolling lost to register pressure); streaming loads and stores keep the three arrays from
// displacing each other in the caches.  keep_array: the array is small enough to stay in the
// last-level cache until the next forward pass reads it, so it alone is read and written with
// the default cache policy.  The skip decision is taken per aligned group of kLineLanes
// lanes (64 bytes when V = 4, the granule that measured best among 16..256 bytes): a granule is
// either rewritten whole or not touched at all, because partially written granules cost the
// memory system far more than the bytes they save.
constexpr uint32_t kLineLanes = 4;

// RULE 0: Adagrad (array, state, grad).  RULE 1: SGD (array, grad; `state` and `eps` unused).
template <int V, int RULE>
__global__ __launch_bounds__(kBlock) void update_kernel(float *__restrict__ array, float *__restrict__ state,
                                                        float *__restrict__ grad, uint64_t m, float lr, float eps,
                                                        bool keep_array, bool clear_grad)
{
    typedef typename Vec<V>::A VT;
    const uint64_t nvec = m / V;
    const uint64_t it = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    const bool in_range = it < nvec;
    VT g;
#pragma unroll
    for (int k = 0; k < V; ++k) g[k] = 0.0f;
    if (in_range) g = __builtin_nontemporal_load(reinterpret_cast<const VT *>(grad + it * V));
    bool any = false;
#pragma unroll
    for (int k = 0; k < V; ++k) any |= (g[k] != 0.0f);
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t line_any = (__ballot(any) >> (lane & ~(kLineLanes - 1u))) & ((1ull << kLineLanes) - 1ull);
    if (in_range && line_any != 0) {  // an untouched granule: nothing read beyond the gradient, nothing written
        VT w;
        if (keep_array) w = *reinterpret_cast<const VT *>(array + it * V);
        else w = __builtin_nontemporal_load(reinterpret_cast<const VT *>(array + it * V));
        VT s;
        if constexpr (RULE == 0) s = __builtin_nontemporal_load(reinterpret_cast<const VT *>(state + it * V));
#pragma unroll
        for (int k = 0; k < V; ++k) {
            if (g[k] != 0.0f) {      // slots with a zero gradient are rewritten with the bits they had
                if constexpr (RULE == 0) {
                    float wk = w[k], sk = s[k];
                    adagrad_one(wk, sk, g[k], lr, eps);
                    w[k] = wk;
                    s[k] = sk;
                } else {
                    w[k] = __fsub_rn(w[k], __fmul_rn(lr, g[k]));
                }
            }
            g[k] = 0.0f;
        }
        if (keep_array) *reinterpret_cast<VT *>(array + it * V) = w;
        else __builtin_nontemporal_store(w, reinterpret_cast<VT *>(array + it * V));
        if constexpr (RULE == 0) __builtin_nontemporal_store(s, reinterpret_cast<VT *>(state + it * V));
        if (clear_grad) __builtin_nontemporal_store(g, reinterpret_cast<VT *>(grad + it * V));
    }
    // tail (m not a multiple of V): first threads of block 0
    if (V > 1 && blockIdx.x == 0) {
        const uint64_t j = nvec * V + threadIdx.x;
        if (threadIdx.x < V && j < m) {
            const float gj = grad[j];
            if (gj != 0.0f) {
                if constexpr (RULE == 0) {
                    float wj = array[j], sj = state[j];
                    adagrad_one(wj, sj, gj, lr, eps);
                    array[j] = wj;
                    state[j] = sj;
                } else {
                    array[j] = __fsub_rn(array[j], __fmul_rn(lr, gj));
                }
                grad[j] = 0.0f;
            }
        }
    }
}

// Whole vectors of four words by a thread each, what is left in front of and behind them by single threads.
// 100 MB: one word a thread and step 20.9 us, so 14.3.  `block`: which of the workgroups of BLOCK threads.
constexpr uint32_t kFillVecs = 4;      // vectors per thread
__host__ __device__ inline uint32_t fill_blocks(uint64_t n, uint32_t block)      // n < 2^33
{
    return (uint32_t)((n + 4ull * block * kFillVecs - 1) / (4ull * block * kFillVecs));
}

template <uint32_t BLOCK>
__device__ __forceinline__ void fill_u32(uint32_t *__restrict__ dst, uint64_t n, uint32_t v, uint32_t block)
{
    const uint64_t skip = (4u - (((uintptr_t)dst >> 2) & 3u)) & 3u, head = skip < n ? skip : n, vecs = (n - head) / 4u;
    typedef uint32_t V4 __attribute__((ext_vector_type(4)));
    V4 *at = reinterpret_cast<V4 *>(dst + head);
    const V4 v4 = {v, v, v, v};
    const uint64_t first = (uint64_t)block * (BLOCK * kFillVecs) + threadIdx.x;
#pragma unroll
    for (uint32_t k = 0; k < kFillVecs; ++k)
        if (first + k * BLOCK < vecs) at[first + k * BLOCK] = v4;
    if (block == 0) {
        if (threadIdx.x < head) dst[threadIdx.x] = v;
        const uint64_t tail = head + 4u * vecs + threadIdx.x;
        if (threadIdx.x < 4u && tail < n) dst[tail] = v;
    }
}

__global__ __launch_bounds__(kBlock) void fill_u32_kernel(uint32_t *__restrict__ dst, uint64_t n, uint32_t v)
{
    fill_u32<kBlock>(dst, n, v, blockIdx.x);
}

// A gradient array to be cleared before the scatter, by workgroups that the first kernel of the sort gets on top of
// its own `work` ones: that kernel keeps a few hundred workgroups waiting for memory, and a launch is saved.
// 25 M slots: 14.4 + 5.9 us in two launches, 15.4 in one; 6 M: 6.5 + 5.5, 7.8.
struct Clear {
    uint32_t *dst;
    uint64_t n;          // words; 0: nothing to clear
    uint32_t work;
};

}  // namespace robe
