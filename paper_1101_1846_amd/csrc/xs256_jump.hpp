// xs256_jump.hpp -- XS256 start states of a wave's 64 lanes at equal distances
// 2^lgc from one common state, without a chain of table products per lane.
//
// A jump is linear in the state, and also in the state's own future: with
// x^k = sum c_i x^i (mod the characteristic polynomial of the step, i < 256),
// the state after k steps is the XOR of the states after i steps over the set
// bits c_i.  The states after 0 .. 255 steps are windows of 8 in 263
// consecutive numbers, so one expansion of the wave's state gives a 4-bit
// lookup table of that sum, and each lane then takes a single product with the
// coefficients of its own distance (64 times 32 bytes for each 2^lgc, built by
// the host once).  What bounds it is latency: the radix-16 tree it replaces
// chained 4 products per level over up to 5 levels and 3 launches (24 to 90
// us); this takes about 8.
#pragma once
#include "rng_device.hpp"

namespace rngx {

// The XOR of r over all 64 lanes (uniform); all lanes active.
__device__ __forceinline__ uint32_t xor_over_64(uint32_t r)
{
    r ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)r, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
    r ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)r, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
    r ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)r, 0x141, 0xF, 0xF, false);  // row_half_mirror
    r ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)r, 0x140, 0xF, 0xF, false);  // row_mirror
    return (uint32_t)__builtin_amdgcn_readlane((int)r, 0) ^ (uint32_t)__builtin_amdgcn_readlane((int)r, 16) ^
           (uint32_t)__builtin_amdgcn_readlane((int)r, 32) ^ (uint32_t)__builtin_amdgcn_readlane((int)r, 48);
}

// Nibble `lane` of the uniform vector x.  (The words are read out of the
// compiler's sight: it turns the selects into an index, and the vector into an
// array in LDS.)
__device__ __forceinline__ uint32_t lane_nibble(const uint32_t (&x)[8], int lane)
{
    uint32_t w = x[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) {
        uint32_t xi = x[i];
        asm("" : "+v"(xi));
        w = lane >> 3 == i ? xi : w;
    }
    return (w >> (4 * (lane & 7))) & 15u;
}

// x <- M x by a whole wave for uniform x: lane p looks up nibble p in the
// 4-bit table T (global) and the 64 entries are XORed across the lanes.
__device__ __forceinline__ void xs256_wave_product(const uint4 *T, uint32_t (&x)[8], int lane)
{
    const uint32_t n = lane_nibble(x, lane);
    const uint4 a = T[2 * lane * 16 + n], b = T[(2 * lane + 1) * 16 + n];
    x[0] = xor_over_64(a.x);
    x[1] = xor_over_64(a.y);
    x[2] = xor_over_64(a.z);
    x[3] = xor_over_64(a.w);
    x[4] = xor_over_64(b.x);
    x[5] = xor_over_64(b.y);
    x[6] = xor_over_64(b.z);
    x[7] = xor_over_64(b.w);
}

// Uniform x moved k steps on: a product per nonzero hexadecimal digit of k.
__device__ __forceinline__ void xs256_wave_jump(uint32_t (&x)[8], uint64_t k, int lane, const DevTables &tab)
{
    for (int j = 0; j < 16 && (k >> (4 * j)); ++j) {
        const uint32_t d = (uint32_t)(k >> (4 * j)) & 15u;
        if (d) xs256_wave_product(tab.xs256_t4w + ((size_t)j * 15 + (d - 1)) * 2048, x, lane);
    }
}

constexpr int kXs256PolyMin = 5, kXs256PolyMax = 12;  // log2 of the distances with a coefficient table
constexpr int kXs256Window = 264;                     // words of s_w below

// The state of lane l: x (uniform, v_0 .. v_7) moved l 2^lgc steps on.
// t4: 2048 quads of LDS, s_w: kXs256Window words, both the wave's own.
__device__ __forceinline__ void xs256_lane_starts(uint32_t (&x)[8], uint32_t lgc, uint4 *t4, uint32_t *s_w, int lane,
                                                  const DevTables &tab)
{
    // numbers 0 .. 262 from v_0 on: 16 lanes each from every 64th state (with 8
    // from every 32nd the gathers took more than the steps saved)
    const uint32_t n = lane_nibble(x, lane);
    GenXS256 g;
    uint4 a[4], b[4];
#pragma unroll
    for (int d = 1; d < 4; ++d) {
        const uint4 *T = tab.xs256_t4w + ((size_t)15 + 4 * d - 1) * 2048;  // M^(64 d)
        a[d] = T[2 * lane * 16 + n];
        b[d] = T[(2 * lane + 1) * 16 + n];
    }
    const uint4 *poly = tab.xs256_poly + ((size_t)(lgc - kXs256PolyMin) * 64 + lane) * 2;
    const uint4 c0 = poly[0], c1 = poly[1];
#pragma unroll
    for (int i = 0; i < 8; ++i) g.v[i] = x[i];
#pragma unroll
    for (int d = 1; d < 4; ++d) {
        const uint32_t y[8] = {xor_over_64(a[d].x), xor_over_64(a[d].y), xor_over_64(a[d].z), xor_over_64(a[d].w),
                               xor_over_64(b[d].x), xor_over_64(b[d].y), xor_over_64(b[d].z), xor_over_64(b[d].w)};
#pragma unroll
        for (int i = 0; i < 8; ++i) g.v[i] = lane >> 4 == d ? y[i] : g.v[i];
    }
    // a wave's LDS instructions execute in order: compiler fences are enough
    asm volatile("" ::: "memory");
    uint32_t *w = s_w + 64 * (lane >> 4);  // the 16 lanes write the same words
    if (lane < 16)
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = g.v[i];
#pragma unroll 1
    for (int i = 0; i < 64; i += 8)
#pragma unroll
        for (int k = 0; k < 8; ++k) w[8 + i + k] = g.next();  // up to word 263
    asm volatile("" ::: "memory");
    // quad (2p + h) * 16 + v, p = lane: words 4h .. 4h+3 of the XOR of the
    // states after 4p + k steps over the set bits k of v, in Gray-code order
    uint32_t m[11], e[8];
#pragma unroll
    for (int i = 0; i < 11; ++i) m[i] = s_w[4 * lane + i];
#pragma unroll
    for (int i = 0; i < 8; ++i) e[i] = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int v = i ^ (i >> 1);
        if (i) {
            const int k = __builtin_ctz(i);
#pragma unroll
            for (int j = 0; j < 8; ++j) e[j] ^= m[k + j];
        }
        t4[2 * lane * 16 + v] = make_uint4(e[0], e[1], e[2], e[3]);
        t4[(2 * lane + 1) * 16 + v] = make_uint4(e[4], e[5], e[6], e[7]);
    }
    asm volatile("" ::: "memory");
    x[0] = c0.x;
    x[1] = c0.y;
    x[2] = c0.z;
    x[3] = c0.w;
    x[4] = c1.x;
    x[5] = c1.y;
    x[6] = c1.z;
    x[7] = c1.w;
    gf2_apply256_t4_loop(t4, x);
    asm volatile("" ::: "memory");
}

}  // namespace rngx
