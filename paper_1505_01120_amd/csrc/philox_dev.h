// Philox4x32-10 and the quarter-disc hit test of the Monte-Carlo partition
// kernel (MapCLPartition, the SparkCLPi demo of paper sec. 3.2.1), as device
// functions.  The library's Monte-Carlo tiles and the VALU-ceiling probe
// (a register-only loop of the same instruction mix) both use them.
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

namespace sparkcl {

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).
// The key words are wave-uniform and stay in scalar registers; each round is
// two 32x32->64 products and two three-way xors per lane.
struct U4 {
    uint32_t x, y, z, w;
};

// Three-way xor as one gfx950 v_bitop3_b32 (truth table 0x96 = a ^ b ^ c).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ U4 philox10(U4 c, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c.x;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
        U4 n;
        n.x = xor3((uint32_t)(p1 >> 32), c.y, k0);
        n.y = (uint32_t)p1;
        n.z = xor3((uint32_t)(p0 >> 32), c.w, k1);
        n.w = (uint32_t)p0;
        c = n;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

// Point (a, b) * 2^-24 from the top 24 bits of two words; a hit iff
// a^2 + b^2 <= 2^48, decided exactly in 64-bit integers (two 32x32->64
// multiply-adds).
__device__ __forceinline__ uint32_t disc_hit(uint32_t wa, uint32_t wb)
{
    const uint32_t a = wa >> 8, b = wb >> 8;
    const uint64_t r2 = (uint64_t)a * a + (uint64_t)b * b;
    return r2 <= (1ull << 48) ? 1u : 0u;
}

// The same test for a whole wave at once, as the mask of lanes whose point
// lies outside.  With a and b left in the words' top 24 bits a^2 + b^2 is
// scaled by 2^16, and a miss is a sum of 2^64 or more: the second
// multiply-add's carry, which arrives in a scalar register for the scalar
// unit to count.  (a^2 + b^2 = 2^48 itself has no solution with
// a, b < 2^24: 2^48 is a sum of two squares only as (2^24)^2 + 0.)
//
// kWhole: the words' low 8 bits are left in, which adds less than 2^42 to the
// scaled sum.  A sum without a carry is then still a hit and one of
// 2^64 + 2^42 or more still a miss; in between (`high`, the sum's upper word,
// below kDiscBand; about 2^-22 of the points) the caller has to ask again
// without kWhole.  Two vector instructions per sample, plus a share of the
// band test, against 7.5 for the comparison and the add.
constexpr uint32_t kDiscBand = 1u << 10;
template <bool kWhole>
__device__ __forceinline__ uint64_t disc_miss_mask(uint32_t wa, uint32_t wb, uint32_t &high)
{
    const uint32_t a = kWhole ? wa : wa & 0xFFFFFF00u, b = kWhole ? wb : wb & 0xFFFFFF00u;
    const uint64_t aa = (uint64_t)a * a;
    uint64_t sum, carry;
    __asm__("v_mad_u64_u32 %0, %1, %2, %2, %3" : "=v"(sum), "=s"(carry) : "v"(b), "v"(aa));
    high = (uint32_t)(sum >> 32);
    return carry & __builtin_amdgcn_read_exec();
}

// Philox4x32-10 on counters (lo, hi, pid, 0) that differ in `lo` only: the
// first three rounds' products and xors of the other words are the same for
// all of them and are made once per tile, in scalar registers.  37 vector
// instructions per block instead of 40 and the 64-bit counter add.
struct PhiloxTile {
    uint32_t k1, x2, m1, z2, z3, k0_3; // round constants, see block()

    __device__ __forceinline__ PhiloxTile(uint32_t hi, uint32_t pid, uint32_t key0, uint32_t key1)
    {
        const uint64_t q0 = (uint64_t)0xCD9E8D57u * pid; // round 1, second product
        const uint32_t x1 = (uint32_t)(q0 >> 32) ^ hi ^ key0;
        const uint64_t q1 = (uint64_t)0xD2511F53u * x1;  // round 2, first product
        k1 = __builtin_amdgcn_readfirstlane(key1);
        x2 = __builtin_amdgcn_readfirstlane((uint32_t)q0 ^ (key0 + 0x9E3779B9u));
        z2 = __builtin_amdgcn_readfirstlane((uint32_t)(q1 >> 32) ^ (key1 + 0xBB67AE85u));
        k0_3 = __builtin_amdgcn_readfirstlane(key0 + 2 * 0x9E3779B9u);
        m1 = __builtin_amdgcn_readfirstlane(key1 + 2 * 0xBB67AE85u);
        z3 = __builtin_amdgcn_readfirstlane((uint32_t)q1 ^ m1);
    }

    __device__ __forceinline__ U4 block(uint32_t lo) const
    {
        const uint64_t a1 = (uint64_t)0xD2511F53u * lo;
        const uint64_t b2 = (uint64_t)0xCD9E8D57u * ((uint32_t)(a1 >> 32) ^ k1);
        const uint64_t a3 = (uint64_t)0xD2511F53u * ((uint32_t)(b2 >> 32) ^ x2);
        const uint64_t b3 = (uint64_t)0xCD9E8D57u * ((uint32_t)a1 ^ z2);
        U4 c{xor3((uint32_t)(b3 >> 32), (uint32_t)b2, k0_3), (uint32_t)b3,
             (uint32_t)(a3 >> 32) ^ z3, (uint32_t)a3};
        uint32_t k0 = k0_3, kk1 = m1;
#pragma unroll
        for (int r = 3; r < 10; ++r) {
            k0 += 0x9E3779B9u;
            kk1 += 0xBB67AE85u;
            const uint64_t p0 = (uint64_t)0xD2511F53u * c.x;
            const uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
            c = U4{xor3((uint32_t)(p1 >> 32), c.y, k0), (uint32_t)p1,
                   xor3((uint32_t)(p0 >> 32), c.w, kk1), (uint32_t)p0};
        }
        return c;
    }
};

// One iteration of the Monte-Carlo-only executor's loop, and of the probe that
// measures its ceiling: the samples outside the quarter disc among the pairs of
// kMcPairs blocks per lane, at lo, lo + step, ..., counted for the whole wave,
// all lanes active.  Independent blocks keep the multiplies' latency covered
// at the executor's waves per SIMD.
constexpr int kMcPairs = 2;
__device__ __forceinline__ uint32_t wave_misses(const PhiloxTile &ph, uint32_t lo, uint32_t step)
{
    U4 r[kMcPairs];
#pragma unroll
    for (int u = 0; u < kMcPairs; ++u)
        r[u] = ph.block(lo + u * step);
    uint32_t misses = 0, low = ~0u, h0, h1;
#pragma unroll
    for (int u = 0; u < kMcPairs; ++u) {
        misses += (uint32_t)__popcll(disc_miss_mask<true>(r[u].x, r[u].y, h0)) +
                  (uint32_t)__popcll(disc_miss_mask<true>(r[u].z, r[u].w, h1));
        low = min(low, min(h0, h1));
    }
    if (__ballot(low < kDiscBand) != 0) { // a point near the arc: all again, exactly
        misses = 0;
#pragma unroll
        for (int u = 0; u < kMcPairs; ++u)
            misses += (uint32_t)__popcll(disc_miss_mask<false>(r[u].x, r[u].y, h0)) +
                      (uint32_t)__popcll(disc_miss_mask<false>(r[u].z, r[u].w, h1));
    }
    return misses;
}

} // namespace sparkcl
