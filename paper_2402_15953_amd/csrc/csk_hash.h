// Device-side polynomial hashing over the Mersenne prime field p = 2^61 - 1.
//
// The sign hashes are degree-3 polynomials (a 4-wise independent family) and the bin
// hashes degree-1 polynomials (2-wise independent), as the initialization paragraph
// of Sec. 3.2 requires; Sec. 4 evaluates them over a Mersenne prime field.  Keys are
// 32-bit, so one Horner step v*x + a multiplies a 61-bit value by a 32-bit key: two
// 32x32->64 multiplies, then the Mersenne fold 2^61 = 1 (mod p).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "csk_internal.h"

namespace csk {

constexpr uint64_t kHashP = (1ull << 61) - 1;

// One Horner step: returns r = v * x + a (mod p) in redundant form.
// Invariant: v < 2^63 and a < 2^61 give r < 2^61 + 2^34 + 8 + 2^61 < 2^63, so steps
// chain without an intermediate fold; hcanon() reduces the final value.
__device__ __forceinline__ uint64_t hstep(uint64_t v, uint32_t x, uint64_t a)
{
    const uint64_t lo = (uint64_t)(uint32_t)v * (uint64_t)x;  // < 2^64
    // v * x = t * 2^32 + (lo mod 2^32) with t = (v >> 32) * x + (lo >> 32) < 2^63 + 2^32
    const uint64_t t = (uint64_t)(uint32_t)(v >> 32) * (uint64_t)x + (lo >> 32);
    // (v * x mod 2^61) + (v * x >> 61) + a, using 2^61 = 1 (mod p): the low 61 bits are
    // the word pair (lo mod 2^32, t mod 2^29), built in the high half of lo's register
    // pair, so the sum is one 64-bit add (seven instructions a step).  The add is
    // written as the instruction itself: left to the compiler, it reassociates the three
    // terms into zero-extended 64-bit adds.
    const uint64_t low61 = ((uint64_t)((uint32_t)t & 0x1FFFFFFFu) << 32) | (uint32_t)lo;
    const uint64_t s = (t >> 29) + a;
    uint64_t r;
    asm("v_lshl_add_u64 %0, %1, 0, %2" : "=v"(r) : "v"(low61), "v"(s));
    return r;
}

// v * x + a (mod p) for a leading-bits evaluation: v < 2^63, a < 2^61 (wave-uniform).  With
// 2^64 = 8 (mod p) the product's third word folds in one multiply-add, and the sum may
// wrap past 2^64 once: the result is then short of the value by 8 modulo p.
__device__ __forceinline__ uint64_t hstep_wrap(uint64_t v, uint32_t x, uint64_t a)
{
    const uint64_t lo = (uint64_t)(uint32_t)v * (uint64_t)x;
    const uint64_t t = (uint64_t)(uint32_t)(v >> 32) * (uint64_t)x + (lo >> 32);
    const uint64_t low64 = ((uint64_t)(uint32_t)t << 32) | (uint32_t)lo;
    // both written as the instructions themselves, as in hstep
    uint64_t s, r;
    asm("v_mad_u64_u32 %0, vcc, %1, 8, %2" : "=v"(s) : "v"((uint32_t)(t >> 32)), "s"(a) : "vcc");
    asm("v_lshl_add_u64 %0, %1, 0, %2" : "=v"(r) : "v"(low64), "v"(s));
    return r;
}

// Canonical residue in [0, p) of a redundant value r < 2^63.
__device__ __forceinline__ uint64_t hcanon(uint64_t r)
{
    r = (r & kHashP) + (r >> 61);  // < 2^61 + 4
    return r >= kHashP ? r - kHashP : r;
}

// b0 + b1 x mod p (canonical)
__device__ __forceinline__ uint64_t hash_deg1(const uint64_t *b, uint32_t x)
{
    return hcanon(hstep(b[1], x, b[0]));
}

// a0 + a1 x + a2 x^2 + a3 x^3 mod p (canonical)
__device__ __forceinline__ uint64_t hash_deg3(const uint64_t *a, uint32_t x)
{
    return hcanon(hstep(hstep(hstep(a[3], x, a[2]), x, a[1]), x, a[0]));
}

// Bucket of a tuple: j = (sum of its columns' canonical bin values) mod m (the sum is
// below 8 * 2^61 < 2^64).  A power-of-two m keeps the low bits; any other m uses a
// Barrett reduction with mdiv = floor((2^64 - 1) / m), whose quotient estimate is at most
// two below the true one.
struct BinMod {
    uint32_t m;
    uint32_t pow2;
    uint64_t mdiv;
    __device__ __forceinline__ uint32_t reduce(uint64_t s) const
    {
        if (pow2) return (uint32_t)s & (m - 1);
        uint64_t r = s - __umul64hi(s, mdiv) * (uint64_t)m;
        if (r >= m) r -= m;
        if (r >= m) r -= m;
        return (uint32_t)r;
    }
};

// Per-relation hashing plan as the kernels read it: joins at each key column and the
// bucket reduction.
struct DevPlan {
    int32_t n_edges[kMaxCols];
    BinMod bm;
};

template <int NC>
__device__ __forceinline__ void load_keys(const uint32_t *__restrict__ keys, uint64_t i, bool vec2,
                                          uint32_t (&x)[NC])
{
    if constexpr (NC == 2) {
        if (vec2) {
            const uint2 v = reinterpret_cast<const uint2 *>(keys)[i];
            x[0] = v.x;
            x[1] = v.y;
            return;
        }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) x[c] = keys[i * NC + c];
}

// Hash one tuple for one repetition; `cf` points at that repetition's coefficients
// (per column: b0, b1, then a0..a3 per join).  Returns the bucket j in [0, m) and the
// sign bit (1 = negative).
template <int NC>
__device__ __forceinline__ void hash_rep(const uint64_t *__restrict__ cf, const DevPlan &plan,
                                         const uint32_t (&x)[NC], uint32_t &j, uint32_t &neg)
{
    uint64_t js = 0;
    neg = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        js += hash_deg1(cf, x[c]);
        cf += 2;
        const int ne = plan.n_edges[c];
        for (int e = 0; e < ne; ++e) {
            neg ^= (uint32_t)hash_deg3(cf, x[c]) & 1u;
            cf += 4;
        }
    }
    j = plan.bm.reduce(js);
}

// Bucket only (for segments holding a bucket range, where signs are needed only for
// tuples inside the range).
template <int NC>
__device__ __forceinline__ uint32_t hash_bin(const uint64_t *__restrict__ cf, const DevPlan &plan,
                                             const uint32_t (&x)[NC])
{
    uint64_t js = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        js += hash_deg1(cf, x[c]);
        cf += 2 + 4 * plan.n_edges[c];
    }
    return plan.bm.reduce(js);
}

template <int NC>
__device__ __forceinline__ uint32_t hash_neg(const uint64_t *__restrict__ cf, const DevPlan &plan,
                                             const uint32_t (&x)[NC])
{
    uint32_t neg = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        cf += 2;
        for (int e = 0; e < plan.n_edges[c]; ++e) {
            neg ^= (uint32_t)hash_deg3(cf, x[c]) & 1u;
            cf += 4;
        }
    }
    return neg;
}

// (tuple chunk, segment) of a two-dimensional launch's workgroup.  Workgroups go to the 8 XCDs
// round-robin by linear id; the ids one XCD receives are given a contiguous run of the
// chunk-major order, so the segments of one tuple chunk run on one XCD (two at a run's
// ends) and that XCD's L2 fetches the chunk's keys once.
struct SegTile {
    uint32_t chunk, seg;
};
__device__ __forceinline__ SegTile seg_tile()
{
    const uint32_t G = gridDim.x * gridDim.y;
    const uint32_t L = blockIdx.x + blockIdx.y * gridDim.x;
    const uint32_t xcd = L & 7u, w = L >> 3;
    const uint32_t P = xcd * (G >> 3) + min(xcd, G & 7u) + w;  // a bijection of [0, G)
    return {P / gridDim.y, P % gridDim.y};
}

__host__ __device__ inline BinMod make_binmod(uint32_t m)
{
    BinMod b;
    b.m = m;
    b.pow2 = (m & (m - 1)) == 0 ? 1u : 0u;
    b.mdiv = ~0ull / m;
    return b;
}

// a / 2^k mod p for a < p, k < 61: powers of two rotate the field's 61 bits.
__device__ __forceinline__ uint64_t rotr61(uint64_t a, uint32_t k)
{
    return (a >> k) | ((a << (61 - k)) & kHashP);
}

// What the hashes of a group of tuples came closest to their rounding limits by (the
// larger, the closer); see CoefE1::bin_neg_fast.
struct HashFlag {
    uint32_t bin = 0, sign = 0;
    __device__ __forceinline__ void merge(const HashFlag &o)
    {
        bin = max(bin, o.bin);
        sign = max(sign, o.sign);
    }
};

// Coefficients of one repetition for relations whose every key column takes part in
// exactly one join (chains, stars), m = 2^k: b0, b1, a0..a3 per column, held in registers.
//
// Only k bits of a bin value and one bit of a sign value reach the sketch.  Dividing the
// polynomials by 2^k (bins) and by 2 (signs) modulo p rotates those bits to the top: for
// h < p, h / 2^k mod p = (h >> k) + (h mod 2^k) 2^(61-k).  The hash is then the leading
// bits of the divided polynomial's residue, which need neither the exact low bits nor the
// canonical reduction of its last step: a bin takes three instructions instead of nine, a
// sign's last step three instead of nine (the update kernels are bound by instructions).
// 10^7 tuples, m = 2^16, d = 9: the two-column update kernel 212 -> 158 us (82 -> 53 vector
// instructions per tuple and repetition), the one-column one 125 -> 100 us.
template <int NC>
struct CoefE1 {
    uint64_t b0[NC], b1[NC], a[NC][4];  // divided by 2^k (bins) and by 2 (signs)
    uint64_t B[NC];                     // floor(b1 2^64 / p)
    uint64_t C[NC];                     // floor(b0 2^(32+k) / 2^61)
    uint32_t m, sh;                     // 2^k, 61 - k
    template <typename P>  // a generic, global or constant address-space pointer
    __device__ __forceinline__ void load(P cf, uint32_t m_)
    {
        m = m_;
        const uint32_t k = 31u - (uint32_t)__builtin_clz(m_);
        sh = 61u - k;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            b0[c] = rotr61(cf[6 * c], k);
            b1[c] = rotr61(cf[6 * c + 1], k);
#pragma unroll
            for (int i = 0; i < 4; ++i) a[c][i] = rotr61(cf[6 * c + 2 + i], 1);
            // b1 2^64 / p = 8 b1 + 8 b1 / p, and 8 b1 = q p + (8 b1 mod 2^61) + q, q = b1 >> 58
            const uint64_t q = b1[c] >> 58;
            B[c] = 8 * b1[c] + q + (((8 * b1[c]) & kHashP) + q >= kHashP ? 1u : 0u);
            C[c] = b0[c] >> (29u - k);
        }
    }
    // Sum of the columns' bin values (the caller masks it with m - 1) and sign bit, exact.
    __device__ __forceinline__ uint32_t bin(const uint32_t (&x)[NC]) const
    {
        uint32_t j = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c) j += (uint32_t)(hcanon(hstep(b1[c], x[c], b0[c])) >> sh);
        return j;
    }
    __device__ __forceinline__ uint32_t neg(const uint32_t (&x)[NC]) const
    {
        uint32_t s = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c)
            s ^= (uint32_t)(hcanon(hstep(hstep(hstep(a[c][3], x[c], a[c][2]), x[c], a[c][1]), x[c], a[c][0])) >> 60);
        return s;
    }
    // The same from the leading bits.  With F = (b0 + b1 x mod p) / p the bin value is
    // floor(2^k F) (no multiple of p / 2^k lies between the residue over p and over 2^61).
    // t = floor(x B / 2^32) mod 2^32 is short of b1 x / p in 2^-32 units by less than 2
    // (the dropped half unit of x B, and x times B's rounding), so t 2^k + C is short of
    // 2^(32+k) F by less than 2^(k+1) + 2: its bits 32 and up are the bin value unless its
    // low word is within that of 2^32.  The word is the flag (one hash in 2^(31-k) is taken
    // again exactly).
    __device__ __forceinline__ uint32_t bin_fast(const uint32_t (&x)[NC], HashFlag &flag) const
    {
        uint32_t j = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint32_t t = __umulhi(x[c], (uint32_t)B[c]) + x[c] * (uint32_t)(B[c] >> 32);
            const uint64_t r = (uint64_t)t * m + C[c];
            j += (uint32_t)(r >> 32);
            flag.bin = max(flag.bin, (uint32_t)r);
        }
        return j;
    }
    // The sign is bit 60 of V mod p, V = v x + a0, v the second Horner step's value, v < 2^64
    // and short of it by 8 when its sum wrapped (8 x < 2^35).  V mod p = (V mod 2^61) +
    // (V >> 61), minus p at most once, and V >> 61 < 2^35 + 1: bit 60 of V decides unless V mod
    // 2^60 is within 2^36 + 1 of 2^60.  In 2^32 units, V is hi(v) x + floor(lo(v) x / 2^32) +
    // hi(a0) and at most one carry: bit 28 of that word unless its low 28 bits are within
    // 24 of 2^28 (16, two carries, rounded up).  The flag is those bits times 16.
    __device__ __forceinline__ uint32_t neg_fast(const uint32_t (&x)[NC], HashFlag &flag) const
    {
        uint32_t s = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint64_t v = hstep_wrap(hstep(a[c][3], x[c], a[c][2]), x[c], a[c][1]);
            const uint32_t t = __umulhi((uint32_t)v, x[c]) + (uint32_t)(v >> 32) * x[c] + (uint32_t)(a[c][0] >> 32);
            s ^= t;
            flag.sign = max(flag.sign, t << 4);
        }
        return (s >> 28) & 1u;
    }
    __device__ __forceinline__ void bin_neg_fast(const uint32_t (&x)[NC], uint32_t &j, uint32_t &neg,
                                                 HashFlag &flag) const
    {
        j = bin_fast(x, flag);
        neg = neg_fast(x, flag);
    }
    // Whether a bin (a sign) of the group has to be taken again with bin() (neg()); `canon`
    // (0xFFFFFFFF outside tests) lowers the limits.
    __device__ __forceinline__ bool bin_near(const HashFlag &f, uint32_t canon) const { return bin_near(f, m, canon); }
    static __device__ __forceinline__ bool bin_near(const HashFlag &f, uint32_t m, uint32_t canon)
    {
        return f.bin >= min(canon, 0u - 2u * m - 2u);
    }
    static __device__ __forceinline__ bool sign_near(const HashFlag &f, uint32_t canon)
    {
        return f.sign >= min(canon, 0u - 16u * 24u);
    }
};

}  // namespace csk
