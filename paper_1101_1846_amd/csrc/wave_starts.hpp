// wave_starts.hpp -- start states of a wave's 64 lanes from one state that they
// share: lane l moves k + l 2^lgc steps on, k any distance.  Latency bounds it,
// so what the lanes share is done once for the wave: powers are squared up in
// registers or read in one load, and a product of the shared state with a GF(2)
// matrix is an XOR across the lanes (about 3 us for KISS, 8 for XS256).
#pragma once
#include "xs256_jump.hpp"

namespace rngx {

constexpr int kWaveStartLds = kXs256Lds;  // words of LDS of the wave's own

template <class G>
__device__ __forceinline__ void wave_starts(G &g, uint64_t k, uint32_t lgc, uint32_t *lds, int lane,
                                            const DevTables &tab)
{
    constexpr bool kMwc16 = G::kId == G_MWC1616 || G::kId == G_KISS;
    constexpr bool kXs32 = G::kId == G_XS32 || G::kId == G_KISS;
    if constexpr (G::kId == G_XS256) {
        xs256_wave_jump(g.v, k, lane, tab);
        xs256_lane_starts(g.v, lgc, lds, lane, tab);
    }
    if constexpr (G::kId == G_MWC32) {
        const uint64_t mine = tab.mwc32_pow[lane];
        auto power = [&](int b) {
            return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(mine >> 32), b) << 32 |
                   (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine, b);
        };
        uint64_t z = (uint64_t)g.c << 32 | g.x;
        for (int b = 0; b < 64 && (k >> b); ++b)
            if ((k >> b) & 1) z = mwc32_mulmod(z, power(b), tab.mwc32_a, tab.mwc32_m);
        for (int b = 0; b < 6; ++b) {
            const uint64_t r = mwc32_mulmod(z, power((int)lgc + b), tab.mwc32_a, tab.mwc32_m);
            z = (lane >> b) & 1 ? r : z;
        }
        g.x = (uint32_t)z;
        g.c = (uint32_t)(z >> 32);
    }
    if constexpr (kXs32) {
        uint32_t *word;
        if constexpr (G::kId == G_KISS) word = &g.jsr;
        else word = &g.y;
        uint32_t y = (uint32_t)__builtin_amdgcn_readfirstlane((int)*word);
        for (int b0 = 0; b0 < 64 && (k >> b0); b0 += 16) {
            uint32_t col[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) col[i] = tab.xs32_pow[(b0 + i) * 32 + (lane & 31)];
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if ((k >> (b0 + i)) & 1) y = xor_over_32(col[i] & (0u - ((y >> (lane & 31)) & 1u)));
        }
#pragma unroll 2
        for (int b = 0; b < 6; ++b) {
            const uint32_t r = gf2_apply32(tab.xs32_pow + (lgc + b) * 32, y);
            y = (lane >> b) & 1 ? r : y;
        }
        *word = y;
    }
    if constexpr (kMwc16) {
        // lanes below 32 carry the powers of the first word, the others of the second
        const uint32_t ai = lane < 32 ? g.a1 : g.a2, m = ai * 65536u - 1u;
        uint32_t c = (0u - m) % m, u = 0;  // one step is a; a 2^48 = 2^32 (mod a 2^16 - 1)
        uint32_t a = 69069u, d = 1234567u, ua = 1, ud = 0;
        for (uint32_t b = 0; b < lgc + 6 || (b < 64 && (k >> b)); ++b) {
            if ((k >> b) & 1) {
                u = u ? mwc16_mulmod(u, c, ai) : c;
                ud = a * ud + d;
                ua *= a;
            }
            if (b >= lgc && b < lgc + 6) {
                const bool on = (lane >> (b - lgc)) & 1;
                const uint32_t z = mwc16_mulmod(g.z, (uint32_t)__builtin_amdgcn_readlane((int)c, 0), g.a1);
                const uint32_t w = mwc16_mulmod(g.w, (uint32_t)__builtin_amdgcn_readlane((int)c, 32), g.a2);
                g.z = on ? z : g.z;
                g.w = on ? w : g.w;
                if constexpr (G::kId == G_KISS) g.jcong = on ? a * g.jcong + d : g.jcong;
            }
            c = mwc16_mulmod(c, c, ai);
            d = a * d + d;
            a *= a;
        }
        if (k) {
            g.z = mwc16_mulmod(g.z, (uint32_t)__builtin_amdgcn_readlane((int)u, 0), g.a1);
            g.w = mwc16_mulmod(g.w, (uint32_t)__builtin_amdgcn_readlane((int)u, 32), g.a2);
            if constexpr (G::kId == G_KISS) g.jcong = ua * g.jcong + ud;
        }
    }
}

// Each lane's own state moved its own k steps on (k below 2^nb, nb <= 24,
// uniform); not for XS256.  A chain of nb products, so no load is in it: the
// MWC16 powers are squared up in registers (their table would take a search for
// the multiplier too), the MWC32 ones lie one per lane, and the xorshift32
// columns are copied to lds (kLaneJumpLds words of the wave's own) at once.
constexpr int kLaneJumpLds = 24 * 32;

template <class G>
__device__ __forceinline__ void lane_jump(G &g, uint32_t k, int nb, uint32_t *lds, int lane, const DevTables &tab)
{
    static_assert(G::kId != G_XS256);
    constexpr bool kMwc16 = G::kId == G_MWC1616 || G::kId == G_KISS;
    constexpr bool kXs32 = G::kId == G_XS32 || G::kId == G_KISS;
    uint32_t cz = 0, cw = 0, a = 69069u, d = 1234567u;
    uint64_t power = 0;
    if constexpr (G::kId == G_MWC32) power = tab.mwc32_pow[lane];
    if constexpr (kXs32) {
        asm volatile("" ::: "memory");
        uint32_t v[kLaneJumpLds / 64];
#pragma unroll
        for (int i = 0; i < kLaneJumpLds / 64; ++i) v[i] = tab.xs32_pow[64 * i + lane];
#pragma unroll
        for (int i = 0; i < kLaneJumpLds / 64; ++i) lds[64 * i + lane] = v[i];
        asm volatile("" ::: "memory");
    }
    if constexpr (kMwc16) {  // one step is a; a 2^48 = 2^32 (mod a 2^16 - 1)
        const uint32_t m1 = g.a1 * 65536u - 1u, m2 = g.a2 * 65536u - 1u;
        cz = (0u - m1) % m1;
        cw = (0u - m2) % m2;
    }
#pragma unroll 1
    for (int b = 0; b < nb; ++b) {
        const bool on = (k >> b) & 1;
        if (__ballot(on)) {  // uniform
            if constexpr (G::kId == G_MWC32) {
                const uint64_t c = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(power >> 32), b) << 32 |
                                   (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)power, b);
                const uint64_t r = mwc32_mulmod((uint64_t)g.c << 32 | g.x, c, tab.mwc32_a, tab.mwc32_m);
                g.x = on ? (uint32_t)r : g.x;
                g.c = on ? (uint32_t)(r >> 32) : g.c;
            }
            if constexpr (kXs32) {
                uint32_t y;
                if constexpr (G::kId == G_KISS) y = g.jsr;
                else y = g.y;
                const uint4 *m = (const uint4 *)(lds + 32 * b);
                uint32_t r = 0;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint4 c = m[i];
                    r ^= c.x & (uint32_t)__builtin_amdgcn_sbfe((int)y, 4 * i, 1);
                    r ^= c.y & (uint32_t)__builtin_amdgcn_sbfe((int)y, 4 * i + 1, 1);
                    r ^= c.z & (uint32_t)__builtin_amdgcn_sbfe((int)y, 4 * i + 2, 1);
                    r ^= c.w & (uint32_t)__builtin_amdgcn_sbfe((int)y, 4 * i + 3, 1);
                }
                y = on ? r : y;
                if constexpr (G::kId == G_KISS) g.jsr = y;
                else g.y = y;
            }
            if constexpr (kMwc16) {
                const uint32_t z = mwc16_mulmod(g.z, cz, g.a1), w = mwc16_mulmod(g.w, cw, g.a2);
                g.z = on ? z : g.z;
                g.w = on ? w : g.w;
            }
            if constexpr (G::kId == G_KISS) g.jcong = on ? a * g.jcong + d : g.jcong;
        }
        if constexpr (kMwc16) {
            cz = mwc16_mulmod(cz, cz, g.a1);
            cw = mwc16_mulmod(cw, cw, g.a2);
        }
        d = a * d + d;
        a *= a;
    }
    asm volatile("" ::: "memory");
}

}  // namespace rngx
