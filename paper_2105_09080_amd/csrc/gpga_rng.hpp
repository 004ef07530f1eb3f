// Counter RNG shared by the gradient kernels: Philox4x32-10 and Box-Muller, addressed by
// (column quad, a, b, tag) under the problem's seed.
#pragma once

#include "gpga_internal.hpp"

constexpr uint32_t kPhiloxM0 = 0xD2511F53u;
constexpr uint32_t kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u;
constexpr uint32_t kPhiloxW1 = 0xBB67AE85u;

constexpr uint32_t TAG_GRAD = 1u;
constexpr uint32_t TAG_FEAT = 2u;
constexpr uint32_t TAG_MU = 3u;

struct u32x4 {
    uint32_t a, b, c, d;
};

// Philox4x32 with 10 rounds (Salmon et al., SC'11): two 32x32->64 multiplies per
// round, outputs permuted and xor-ed with the round key; key += Weyl constants.
__device__ __forceinline__ u32x4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                               uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)kPhiloxM0 * c0, p1 = (uint64_t)kPhiloxM1 * c2;
        const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
        const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
        // three-input xor in one instruction (v_bitop3_b32, truth table 0x96 = a ^ b ^ c)
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32(hi1, c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32(hi0, c3, k1, 0x96);
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
        k0 += kPhiloxW0;
        k1 += kPhiloxW1;
    }
    return {c0, c1, c2, c3};
}

// 32 random bits -> uniform in (0,1), exactly representable in fp32: u = ((r >> 9) + 0.5) * 2^-23.
// Built without an integer-to-float conversion: the 23 bits become the mantissa of a float in
// [1, 2) (one funnel shift puts the exponent 0x7F above them), and subtracting 1 - 2^-24 leaves
// (k + 0.5) * 2^-23 exactly (it has at most 24 significant bits, so the subtraction does not round).
__device__ __forceinline__ float uniform23(uint32_t r) {
    const uint32_t bits = __builtin_amdgcn_alignbit(0x7Fu, r, 9u);  // ({0x7F, r} >> 9) = 0x3F800000 | (r >> 9)
    return __uint_as_float(bits) - 0x1.fffffep-1f;
}

// Four standard normals for one column quad: Box-Muller on (u0,u1) and (u2,u3).
// The transcendental part uses the hardware units directly: v_log_f32 (log2),
// v_sqrt_f32, and v_sin_f32 / v_cos_f32, whose argument is in revolutions, so
// sin(2 pi u) is one instruction on u itself with no range reduction.  Measured
// over all 2^23 possible u: |sin|, |cos| error <= 1.3e-7, ln relative error
// <= 1.7e-7, radius error <= 4.9e-7 (radius <= 5.7).
// kScaled: times `scale`, a factor of the radii, with every product rounded.
template <bool kScaled>
__device__ __forceinline__ v4f box_muller4_of(const u32x4& r, float scale) {
    constexpr float kMinus2Ln2 = -1.3862943611198906f;  // -2 ln u = (-2 ln 2) log2 u
    float ra = __builtin_amdgcn_sqrtf(kMinus2Ln2 * __builtin_amdgcn_logf(uniform23(r.a)));
    float rb = __builtin_amdgcn_sqrtf(kMinus2Ln2 * __builtin_amdgcn_logf(uniform23(r.c)));
    const float ub = uniform23(r.b), ud = uniform23(r.d);
    v4f z;
    if (kScaled) {
#pragma clang fp contract(off)
        ra *= scale;
        rb *= scale;
        z.x = ra * __builtin_amdgcn_cosf(ub);
        z.y = ra * __builtin_amdgcn_sinf(ub);
        z.z = rb * __builtin_amdgcn_cosf(ud);
        z.w = rb * __builtin_amdgcn_sinf(ud);
        return z;
    }
    z.x = ra * __builtin_amdgcn_cosf(ub);
    z.y = ra * __builtin_amdgcn_sinf(ub);
    z.z = rb * __builtin_amdgcn_cosf(ud);
    z.w = rb * __builtin_amdgcn_sinf(ud);
    return z;
}
__device__ __forceinline__ v4f box_muller4(const u32x4& r) { return box_muller4_of<false>(r, 1.f); }
__device__ __forceinline__ v4f normals4(uint32_t c4, uint32_t a, uint32_t b, uint32_t tag,
                                        uint32_t k0, uint32_t k1) {
    return box_muller4(philox4x32_10(c4, a, b, tag, k0, k1));
}

// The same generator taken apart for many draws per column quad.  Counter words (c4, a, b, tag): the first two rounds
// leave words that depend on the quad alone (PhiloxQuad) and words that depend on (a, b) alone (PhiloxPair), and
// what is left of them per draw is two xors.  A PhiloxPair of uniform a, b stays in scalar registers: the xors are
// written plainly, since the three-input instruction exists for vectors only (with it the second round's product of
// scalars took two quarter-rate vector multiplies a draw).
struct PhiloxQuad {
    uint32_t lo0, hi1, lo1;
    __device__ __forceinline__ PhiloxQuad(uint32_t c4, uint32_t tag, uint32_t k1) {
        const uint64_t p0 = (uint64_t)kPhiloxM0 * c4;
        lo0 = (uint32_t)p0;
        const uint64_t p1 = (uint64_t)kPhiloxM1 * ((uint32_t)(p0 >> 32) ^ tag ^ k1);
        hi1 = (uint32_t)(p1 >> 32);
        lo1 = (uint32_t)p1;
    }
};
struct PhiloxPair {
    uint32_t x0, x2, x3;
    __device__ __forceinline__ PhiloxPair(uint32_t a, uint32_t b, uint32_t k0, uint32_t k1) {
        const uint64_t p1 = (uint64_t)kPhiloxM1 * b;
        const uint64_t p0 = (uint64_t)kPhiloxM0 * ((uint32_t)(p1 >> 32) ^ a ^ k0);
        x0 = (uint32_t)p1 ^ (k0 + kPhiloxW0);
        x2 = (uint32_t)(p0 >> 32) ^ (k1 + kPhiloxW1);
        x3 = (uint32_t)p0 ^ (k1 + 2u * kPhiloxW1);
    }
};
__device__ __forceinline__ u32x4 philox_rounds(const PhiloxQuad& q, const PhiloxPair& r, uint32_t k0, uint32_t k1) {
    uint32_t c0 = q.hi1 ^ r.x0, c1 = q.lo1, c2 = q.lo0 ^ r.x2, c3 = 0u;  // after two rounds; c3 ^ key comes as r.x3
#pragma unroll
    for (int n = 2; n < 10; ++n) {
        const uint32_t key0 = k0 + (uint32_t)n * kPhiloxW0, key1 = k1 + (uint32_t)n * kPhiloxW1;
        const uint64_t p0 = (uint64_t)kPhiloxM0 * c0, p1 = (uint64_t)kPhiloxM1 * c2;
        c0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, key0, 0x96);
        c2 = n == 2 ? (uint32_t)(p0 >> 32) ^ r.x3 : __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, key1, 0x96);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
    }
    return {c0, c1, c2, c3};
}

// The synthetic gradient of four columns: sigma * N(seed, TAG_GRAD, i, k, c), with sigma in the two radii.  The products are
// rounded here, as a stored gradient is: no fused multiply-add of a later use takes them in.
__device__ __forceinline__ v4f synth_quad(uint32_t c4, uint32_t i, uint32_t kiter, uint32_t k0, uint32_t k1, float sigma) {
    return box_muller4_of<true>(philox4x32_10(c4, i, kiter, TAG_GRAD, k0, k1), sigma);
}

// The same for many rows and iterations of one column quad: words of the first two rounds that depend on the quad alone are
// kept, those of the iteration (uniform) are scalar, and four vector instructions are left of the eight.
struct SynthQuad {
    uint32_t lo0, hi1, lo1;
    __device__ __forceinline__ SynthQuad(uint32_t c4, uint32_t k1) {
        const uint64_t p0 = (uint64_t)kPhiloxM0 * c4;
        lo0 = (uint32_t)p0;
        const uint64_t p1 = (uint64_t)kPhiloxM1 * ((uint32_t)(p0 >> 32) ^ TAG_GRAD ^ k1);
        hi1 = (uint32_t)(p1 >> 32);
        lo1 = (uint32_t)p1;
    }
    __device__ __forceinline__ v4f gradient(uint32_t i, uint32_t kiter, uint32_t k0, uint32_t k1, float sigma) const {
        const uint64_t pk = (uint64_t)kPhiloxM1 * kiter;
        const uint64_t pi = (uint64_t)kPhiloxM0 * (i ^ ((uint32_t)(pk >> 32) ^ k0));
        uint32_t c0 = hi1 ^ ((uint32_t)pk ^ (k0 + kPhiloxW0)), c1 = lo1;
        uint32_t c2 = __builtin_amdgcn_bitop3_b32((uint32_t)(pi >> 32), lo0, k1 + kPhiloxW1, 0x96), c3 = (uint32_t)pi;
#pragma unroll
        for (int n = 2; n < 10; ++n) {
            const uint32_t key0 = k0 + (uint32_t)n * kPhiloxW0, key1 = k1 + (uint32_t)n * kPhiloxW1;
            const uint64_t p0 = (uint64_t)kPhiloxM0 * c0, p1 = (uint64_t)kPhiloxM1 * c2;
            c0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, key0, 0x96);
            c2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, key1, 0x96);
            c1 = (uint32_t)p1;
            c3 = (uint32_t)p0;
        }
        return box_muller4_of<true>({c0, c1, c2, c3}, sigma);
    }
};

// Feature quad h_{i,m} of four columns = mu_i + zeta_{i,m}, rounded to fp32 like a stored feature would be.
__device__ __forceinline__ v4f virtual_quad(const v4f& mu, const PhiloxQuad& quad, uint32_t i, uint32_t m, uint32_t k0, uint32_t k1) {
    return mu + box_muller4(philox_rounds(quad, PhiloxPair(i, m, k0, k1), k0, k1));
}
