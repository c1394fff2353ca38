// Device-side integer maps of ROBE-Z for gfx950: h (Eq. 5), g (Eq. 2), idx (Eq. 5)
// of arXiv 2108.02191, evaluated in registers with 32/64-bit arithmetic only.
//
// Every shortcut below is exact over the integers:
//   * P = 2^31 - 1 is a Mersenne prime, so t mod P folds: 2^31 == 1 (mod P).
//   * a sum of residues is reduced again before it can reach 2^64.
//   * r mod m for r < 2^31 uses a 32-bit reciprocal estimate that is low by at
//     most one, corrected by a single conditional subtraction.
//   * s in [0, 2P) is reduced by min(s, s - P): below P the subtraction wraps to more than s.
// The kernels that gather are bound by instruction issue as much as by memory (quarter-rate integer
// multiplies above all), so these are written for the fewest instructions.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace robe {

constexpr uint32_t kP = 2147483647u;

// Kernel-argument form of a ROBE-Z instance (host fills it from robe_hash_t).
struct Params {
    uint32_t m;        // array length, 1 <= m <= 2^31 - 1
    uint32_t m_recip;  // min(floor(2^32 / m), 2^32 - 1)
    uint32_t d, Z, C;  // C = d / Z chunks per embedding (1 when Z > d)
    uint32_t z_recip;  // ceil(2^32 / Z): floor(i / Z) = mulhi(i, z_recip) for i < 2^16; 0 where C = 1; Z = 1: see chunk_of
    uint32_t r;        // Z / d embeddings per chunk when Z > d, else 0
    uint32_t Ah, Bh, Ch, Dh;
    uint32_t Ag, Bg, Cg, Dg;
};

// t mod P for any 64-bit t, result in [0, P).
__device__ __forceinline__ uint32_t mod_p(uint64_t t)
{
    uint64_t s = (t & kP) + (t >> 31);              // < 2^33 + 2^31, congruent to t
    uint32_t r = (uint32_t)(s & kP) + (uint32_t)(s >> 31);  // < 2^31 + 5
    return r >= kP ? r - kP : r;
}

// (a + b) mod P for a, b in [0, P).
__device__ __forceinline__ uint32_t add_p(uint32_t a, uint32_t b)
{
    const uint32_t s = a + b;                        // < 2^32 - 2
    return min(s, s - kP);
}

// (a * b + c) mod P for a, c < P and b <= P: the sum is at most P^2 - 1 < 2^62, so its upper part is
// at most P - 1 and the two parts add up to less than 2P.
__device__ __forceinline__ uint32_t mul_add_p(uint32_t a, uint32_t b, uint32_t c)
{
    const uint64_t t = (uint64_t)a * b + c;
    const uint32_t s = ((uint32_t)t & kP) + (uint32_t)(t >> 31);
    return min(s, s - kP);
}

// (a * b) mod P for a < P, b <= P.
__device__ __forceinline__ uint32_t mul_p(uint32_t a, uint32_t b) { return mul_add_p(a, b, 0u); }

// x mod P, possibly P itself for 0 (a factor of mul_p), for any 64-bit x: its three parts of 31, 31 and
// 2 bits added up.
__device__ __forceinline__ uint32_t fold_p(uint64_t x)
{
    uint32_t s = ((uint32_t)x & kP) + ((uint32_t)(x >> 31) & kP);     // <= 2P
    s = min(s, s - kP) + (uint32_t)(x >> 62);                         // <= P + 3
    return min(s, s - kP);
}

// r mod m for r < 2^31.  q = floor(r * recip / 2^32) is floor(r/m) or one less.
__device__ __forceinline__ uint32_t mod_m(uint32_t r, uint32_t m, uint32_t recip)
{
    const uint32_t rem = r - __umulhi(r, recip) * m; // in [0, 2m), fits since m < 2^31
    return min(rem, rem - m);
}

// floor(r / m) by the same reciprocal, for r < 2^31.
__device__ __forceinline__ uint32_t div_m(uint32_t r, uint32_t m, uint32_t recip)
{
    const uint32_t q = __umulhi(r, recip);
    return q + (r - q * m >= m ? 1u : 0u);
}

// The chunk of element i < d <= 2^16 of an embedding.
__device__ __forceinline__ uint32_t chunk_of(const Params &p, uint32_t i)
{
    return p.Z == 1u ? i : __umulhi(i, p.z_recip);
}

// Token part of a hash: (B * x) mod P with x read as an unsigned 64-bit integer.
__device__ __forceinline__ uint32_t token_term(uint32_t B, int64_t x)
{
    return mul_p(B, fold_p((uint64_t)x));
}

// h(e,x,c) from the two parts.
__device__ __forceinline__ uint32_t offset_of(const Params &p, uint32_t tok_h, uint32_t stat_h)
{
    return mod_m(add_p(tok_h, stat_h), p.m, p.m_recip);
}

// (o + j) mod m for o < m, j < Z <= m.
__device__ __forceinline__ uint32_t wrap(uint32_t pos, uint32_t m)
{
    return min(pos, pos - m);                        // (pos < 2m < 2^32; below m the subtraction wraps past pos)
}

// Sign bit mask of g: 0x80000000 when g == -1 (hash residue even), else 0.
__device__ __forceinline__ uint32_t sign_mask(uint32_t residue)
{
    return ((residue & 1u) ^ 1u) << 31;
}

// The same for the residue (a + b) mod P, given a and b + 1 (a, b < P).  With s = a + b + 1 < 2^32: a + b reaches P
// exactly where s has bit 31, and taking the odd P off changes the parity, so the residue is even
// where bit 0 and bit 31 of s differ.
__device__ __forceinline__ uint32_t sign_mask_of_sum(uint32_t a, uint32_t b_plus_1)
{
    const uint32_t s = a + b_plus_1;
    return ((s << 31) ^ s) & 0x80000000u;
}

__device__ __forceinline__ float apply_sign(float v, uint32_t mask)
{
    return __uint_as_float(__float_as_uint(v) ^ mask);
}

}  // namespace robe
