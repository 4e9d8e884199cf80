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
constexpr int kXs256Window = 264;                     // words of the expansion below
constexpr int kXs256Lds = 2048 + kXs256Window;        // words of LDS for xs256_lane_starts

// The state of lane l: x (uniform, v_0 .. v_7) moved l 2^lgc steps on.  lds:
// kXs256Lds words of the wave's own, 16-byte aligned.  The 4-bit table is built
// and used a quarter at a time (16 of the 64 nibbles, 8 KiB).
__device__ __forceinline__ void xs256_lane_starts(uint32_t (&x)[8], uint32_t lgc, uint32_t *lds, int lane,
                                                  const DevTables &tab)
{
    uint4 *t4 = (uint4 *)lds;
    uint32_t *s_w = lds + 2048;
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
    // Quarter i: quad (2p + h) * 16 + v holds words 4h .. 4h+3 of the XOR of the
    // states after 4 (16 i + p) + k steps over the set bits k of v; lane 4p + j
    // writes entries 4j .. 4j+3 of nibble p.  Then 16 nibbles of the
    // coefficients look theirs up.  (A loop: straight-line code costs its first
    // fetch, 9000 against 4000 clocks for the look-ups.)
    uint32_t c[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w}, r[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const uint32_t on2 = 0u - (uint32_t)(lane & 1), on3 = 0u - (uint32_t)((lane >> 1) & 1);
    uint4 *const mine = t4 + (lane >> 2) * 32 + 4 * (lane & 3);
#pragma unroll 1
    for (int i = 0; i < 4; ++i) {
        uint32_t m[11], e[8];
#pragma unroll
        for (int k = 0; k < 11; ++k) m[k] = s_w[64 * i + 4 * (lane >> 2) + k];
        asm volatile("" ::: "memory");
#pragma unroll
        for (int k = 0; k < 8; ++k) e[k] = (m[2 + k] & on2) ^ (m[3 + k] & on3);
#pragma unroll
        for (int n = 0; n < 4; ++n) {  // entries 0, 1, 3, 2
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (n) e[k] ^= m[(n & 1 ? 0 : 1) + k];
            mine[n ^ (n >> 1)] = make_uint4(e[0], e[1], e[2], e[3]);
            mine[16 + (n ^ (n >> 1))] = make_uint4(e[4], e[5], e[6], e[7]);
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int p = 0; p < 16; p += 2) {
            const uint32_t w = p < 8 ? c[0] : c[1];
            const uint32_t n0 = (w >> (4 * (p & 7))) & 15u, n1 = (w >> (4 * (p & 7) + 4)) & 15u;
            const uint4 a0 = t4[(2 * p) * 16 + n0], a1 = t4[(2 * p + 1) * 16 + n0];
            const uint4 b0 = t4[(2 * p + 2) * 16 + n1], b1 = t4[(2 * p + 3) * 16 + n1];
            r[0] = xor3(r[0], a0.x, b0.x);
            r[1] = xor3(r[1], a0.y, b0.y);
            r[2] = xor3(r[2], a0.z, b0.z);
            r[3] = xor3(r[3], a0.w, b0.w);
            r[4] = xor3(r[4], a1.x, b1.x);
            r[5] = xor3(r[5], a1.y, b1.y);
            r[6] = xor3(r[6], a1.z, b1.z);
            r[7] = xor3(r[7], a1.w, b1.w);
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int k = 0; k < 6; ++k) c[k] = c[k + 2];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = r[i];
}

}  // namespace rngx
