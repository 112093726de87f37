// Philox4x32-10 counter-based generator for the device (Salmon, Moraes,
// Dror, Shaw, "Parallel random numbers: as easy as 1, 2, 3", SC'11).
//
// A round multiplies counter words 0 and 2 by two odd 32-bit constants,
// keeps both halves of each 64-bit product, and permutes them with the
// remaining words and the round key; the key advances by two Weyl constants
// between rounds.  The key here is the run seed (wave-uniform), so the key
// schedule lives in scalar registers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mcmie {

struct Block4 {
    uint32_t r0, r1, r2, r3;
};

constexpr uint32_t kPhiloxMulA = 0xD2511F53u, kPhiloxMulB = 0xCD9E8D57u;
constexpr uint32_t kPhiloxWeylA = 0x9E3779B9u, kPhiloxWeylB = 0xBB67AE85u;

__device__ __forceinline__ Block4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t pa = (uint64_t)kPhiloxMulA * c0;
        const uint64_t pb = (uint64_t)kPhiloxMulB * c2;
        // Three-input XOR in one gfx950 instruction (truth table 0x96).
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(pb >> 32), c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(pa >> 32), c3, k1, 0x96);
        c1 = (uint32_t)pb;
        c3 = (uint32_t)pa;
        c0 = n0;
        c2 = n2;
        k0 += kPhiloxWeylA;
        k1 += kPhiloxWeylB;
    }
    return Block4{c0, c1, c2, c3};
}

// The generator at the counters (step, instance, id_lo, id_hi) of one photon:
// the parts of its first three rounds that do not depend on the step, kept per
// photon (key words folded in).  philox_step finishes the block: 18 of the 20
// products, and three of the remaining 19 three-input XORs become plain ones,
// which issue at twice their rate.
struct PhotonKey {
    uint32_t x1, x2, x3, x4;
};

__device__ __forceinline__ PhotonKey photon_key(uint32_t instance, uint64_t id, uint32_t k0, uint32_t k1)
{
    const uint64_t pb = (uint64_t)kPhiloxMulB * (uint32_t)id;                                 // round 1
    const uint64_t pa = (uint64_t)kPhiloxMulA * ((uint32_t)(pb >> 32) ^ instance ^ k0);       // round 2
    return PhotonKey{(uint32_t)(id >> 32) ^ k1, (uint32_t)pb ^ (k0 + kPhiloxWeylA),
                     (uint32_t)(pa >> 32) ^ (k1 + kPhiloxWeylB), (uint32_t)pa ^ (k1 + 2u * kPhiloxWeylB)};
}

__device__ __forceinline__ Block4 philox_step(const PhotonKey &p, uint32_t step, uint32_t k0, uint32_t k1)
{
    uint64_t pa = (uint64_t)kPhiloxMulA * step;                       // round 1
    uint32_t c3 = (uint32_t)pa;
    uint64_t pb = (uint64_t)kPhiloxMulB * ((uint32_t)(pa >> 32) ^ p.x1);   // round 2
    uint32_t c0 = (uint32_t)(pb >> 32) ^ p.x2, c1 = (uint32_t)pb, c2 = p.x3 ^ c3;
    k0 += 2u * kPhiloxWeylA;
    k1 += 2u * kPhiloxWeylB;
#pragma unroll
    for (int round = 2; round < 10; ++round) {
        pa = (uint64_t)kPhiloxMulA * c0;
        pb = (uint64_t)kPhiloxMulB * c2;
        c0 = __builtin_amdgcn_bitop3_b32((uint32_t)(pb >> 32), c1, k0, 0x96);
        c2 = round == 2 ? (uint32_t)(pa >> 32) ^ p.x4
                        : __builtin_amdgcn_bitop3_b32((uint32_t)(pa >> 32), c3, k1, 0x96);
        c1 = (uint32_t)pb;
        c3 = (uint32_t)pa;
        k0 += kPhiloxWeylA;
        k1 += kPhiloxWeylB;
    }
    return Block4{c0, c1, c2, c3};
}

// Uniform in (0, 1) from one 32-bit word: (2 floor(r / 2^9) + 1) / 2^24,
// exact in FP32 (23 random bits at the centre of their cell).
// Built without a conversion: the 23 bits under the exponent field of 1.0
// give 1 + k 2^-23, and subtracting 1 - 2^-24 is exact (both lie in [1/2, 2]).
__device__ __forceinline__ float uniform01(uint32_t r)
{
    return __uint_as_float(__builtin_amdgcn_alignbit(0x7Fu, r, 9u)) - 0x1.fffffep-1f;
}

}  // namespace mcmie
