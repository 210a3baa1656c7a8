// thermal_noise.h -- the random vector of Brown's thermal field for one cell
// and step (section "Thermal fluctuations"), shared by the field-buffer
// kernel and the fused local Heun pass.
//
// Philox4x32-10 (Salmon, Moraes, Dror and Shaw, SC 2011) at counter
// (cell, step mod 2^32, step div 2^32, 0) and key (seed mod 2^32, seed div
// 2^32); 32-bit outputs x -> u = (floor(x / 2^8) + 1/2) / 2^24; Box-Muller:
// eta_x, eta_y = sqrt(-2 ln u0) (cos, sin)(2 pi u1), eta_z = sqrt(-2 ln u2) cos(2 pi u3).
#pragma once

#include <hip/hip_runtime.h>

namespace mm {

struct PhiloxU4 {
    unsigned int x, y, z, w;
};

// The generator's cost is its instructions (an uncoupled Heun step has no memory
// traffic).  Both halves of a product come from one 64-bit multiply-add (an addend
// the compiler cannot see to be 0 keeps it from splitting it in two), the three
// terms of a word from one three-input operation.
__device__ inline unsigned int philox_xor3(unsigned int a, unsigned int b, unsigned int c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ inline PhiloxU4 philox4x32_10(PhiloxU4 c, unsigned int k0, unsigned int k1) {
    // round multipliers and the key increments (Weyl sequence)
    constexpr unsigned int MA = 0xD2511F53u, MB = 0xCD9E8D57u;
    constexpr unsigned int WA = 0x9E3779B9u, WB = 0xBB67AE85u;
    unsigned long long zero = 0;
    asm("" : "+s"(zero));
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const unsigned long long p0 = (unsigned long long)MA * c.x + zero;
        const unsigned long long p1 = (unsigned long long)MB * c.z + zero;
        c = PhiloxU4{philox_xor3((unsigned int)(p1 >> 32), c.y, k0), (unsigned int)p1,
                     philox_xor3((unsigned int)(p0 >> 32), c.w, k1), (unsigned int)p0};
        k0 += WA;
        k1 += WB;
    }
    return c;
}

__device__ inline float philox_unit24(unsigned int x) { return ((float)(x >> 8) + 0.5f) * 0x1p-24f; }

// sqrt(-2 ln u) for u in [2^-25, 1]: the base-2 logarithm times -2 ln 2 in two
// parts, and the root from the reciprocal root by one correction step (its
// argument is never subnormal, infinite or, by the bound, 0).
__device__ inline float boxmuller_radius(float u) {
    const float l = __builtin_amdgcn_logf(u);
    const float x = fmaxf(__builtin_fmaf(l, -0x1.62e43p+0f, l * 0x1.05c61p-28f), 0x1p-126f);
    const float y = __builtin_amdgcn_rsqf(x);
    const float r = x * y;
    return __builtin_fmaf(__builtin_fmaf(-r, r, x), 0.5f * y, r);
}

// sin and cos of 2 pi u for u in [0, 1]: u = n/4 + f exactly, |f| <= 1/8; minimax
// polynomials in f^2, 2 pi in two parts.  With the coefficients rounded to FP32 they
// are within 1.9e-9 (sine) and 1.1e-8 (cosine) of the value.
__device__ inline void sincos_turns(float u, float& sn, float& cs) {
    const float n = __builtin_rintf(4.f * u);
    const float f = __builtin_fmaf(n, -0.25f, u), z = f * f;
    float p = __builtin_fmaf(z, 0x1.4be09ep+5f, -0x1.32cb0ep+6f);
    p = __builtin_fmaf(z, p, 0x1.466bbcp+6f);
    p = __builtin_fmaf(z, p, -0x1.4abbcep+5f);
    const float s = __builtin_fmaf(f, 0x1.921fb6p+2f, f * __builtin_fmaf(z, p, -0x1.777a5cp-23f));
    float q = __builtin_fmaf(z, 0x1.d9d57ep+5f, -0x1.55c5ep+6f);
    q = __builtin_fmaf(z, q, 0x1.03c1dep+6f);
    q = __builtin_fmaf(z, q, -0x1.3bd3ccp+4f);
    const float c = __builtin_fmaf(z, q, 1.f);
    const unsigned int k = (unsigned int)n;
    const unsigned int neg = (k & 2u) << 30;
    const bool odd = k & 1u;
    sn = __uint_as_float(__float_as_uint(odd ? c : s) ^ neg);
    cs = __uint_as_float(__float_as_uint(odd ? -s : c) ^ neg);
}

// sc * eta for cell i at generator step `step`.  RMS error of eta against 64 bits over
// 15.7 million values: 5.24e-8 (5.42e-8 with the library's functions).
__device__ inline float3 thermal_eta(long long i, unsigned long long step, unsigned long long seed, float sc) {
    const PhiloxU4 o = philox4x32_10(PhiloxU4{(unsigned int)i, (unsigned int)step, (unsigned int)(step >> 32), 0u},
                                     (unsigned int)seed, (unsigned int)(seed >> 32));
    const float r0 = sc * boxmuller_radius(philox_unit24(o.x));
    const float r2 = sc * boxmuller_radius(philox_unit24(o.z));
    float s1, c1, s3, c3;
    sincos_turns(philox_unit24(o.y), s1, c1);
    sincos_turns(philox_unit24(o.w), s3, c3);
    return make_float3(r0 * c1, r0 * s1, r2 * c3);
}

}  // namespace mm
