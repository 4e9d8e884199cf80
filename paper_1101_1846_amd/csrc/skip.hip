// skip.hip -- jump-ahead of many states by one distance k (Sec. II.A.4: the
// MWC congruence z <- a^k z mod m that follows from eqs. (2)-(3), the k-th power of the GF(2)
// step matrix of eqs. (5) and (6), and the affine LCG map).  Every state moves
// by the same k, so the k-step map is built once -- on the host for the
// constants that do not depend on the state, once per workgroup in LDS for
// the rest -- and each state then pays a single application:
//   MWC32    one fold-domain multiply by a^k                (host constant)
//   MWC16    one multiply per word by a_i^k of its multiplier (392 constants, LDS)
//   XS32     M^k y by four byte lookups                     (host columns, LDS tables)
//   XS256    M^k v by 64 nibble lookups                     (LDS table of M^k)
//   LCG      X <- A_k X + C_k                               (host constants)
// The XS256 table is built per workgroup from the columns of M^k, each the sum of
// up to 256 steps of a unit state weighted by x^k mod the step's characteristic
// polynomial, whose coefficients the host works out (a few hundred ns per
// nonzero hexadecimal digit of k).  With a chain of table products, one per
// digit, in its place, the launch took 37 us for 2^20 states and a k of four
// digits, now 34 (its look-ups take the rest), and 33 for 2^16 states and a k of
// ten digits, now 16.  A k of one digit (a table in memory) or two (one product per
// column) needs no such sum: 65536 states 14.7 and 14.8 us with it, 6.5 and 12.2
// without, 2^20 29.9 and 29.6, 21.9 and 26.9.  Below kXs256TableMin states each
// takes its own products, one per nonzero digit, by the lane or, for few, by a
// whole wave; below kXs256ChainMax too if there are at most two (10^4 states, us,
// products / sums: 7.1 / 14.5 and 11.7 / 14.6, but 16.4 / 14.4 for three).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "host_math.hpp"
#include "rng.h"
#include "rng_abi_internal.hpp"
#include "xs256_jump.hpp"

namespace rngx {

namespace {

constexpr int kSkipWG = 256;
// XS256 workgroups take 1024 lanes: four to a column of M^k while the table is
// built, and 16 waves per CU share the LDS reads when they apply it.  (Splitting
// a product's nibbles over the four lanes of a quad reads four table rows at
// once, whose entries share LDS banks; products on the matrix cores, as parities
// of FP4 sums, take longer over packing the bits than the look-ups alone: 25
// against 16 us per 2^20 states; with the states' 64 MB and the launch a k of one
// digit, which builds nothing, takes 22.)
constexpr int kSkipXs256WG = 1024;
template <class G>
constexpr int skip_wg()
{
    return G::kId == G_XS256 ? kSkipXs256WG : kSkipWG;
}
constexpr uint64_t kXs256TableMin = (uint64_t)1 << 13, kXs256ChainMax = (uint64_t)1 << 16;

struct SkipArgs {
    uint32_t *st;           // [W][ld]
    uint64_t ld, S, k;
    uint64_t mwc32_f;       // a^k * 2^64 mod m (fold domain)
    uint32_t lcg_a, lcg_c;  // k steps of the LCG
    uint32_t xs32[32];      // columns of M^k, xorshift32
    uint64_t poly[4];       // x^k mod the characteristic polynomial of the XS256 step
    uint32_t digits;        // nonzero hexadecimal digits of k
    uint32_t t4w[2];        // the tables of the first two
    DevTables tab;
};

__device__ __forceinline__ uint32_t xs32_by_bytes(const uint32_t *t8, uint32_t y)
{
    return xor3(t8[y & 255], t8[256 + ((y >> 8) & 255)], t8[512 + ((y >> 16) & 255)]) ^ t8[768 + (y >> 24)];
}

__device__ __forceinline__ uint32_t lds_t392_index(const uint16_t *t, uint32_t a)
{
    uint32_t lo = 0, hi = kMwc16Count;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (t[mid] <= a) lo = mid;
        else hi = mid;
    }
    return lo;
}

// kFew: XS256 and a k of one or two nonzero hexadecimal digits.
template <class G, bool kFew = false>
__global__ __launch_bounds__(skip_wg<G>()) void k_skip_by(SkipArgs a)
{
    constexpr int WG = skip_wg<G>();
    constexpr bool kMwc16 = G::kId == G_MWC1616 || G::kId == G_KISS;
    constexpr bool kXs32 = G::kId == G_XS32 || G::kId == G_KISS;
    constexpr bool kXs256 = G::kId == G_XS256;
    __shared__ uint16_t s_t392[kMwc16 ? kMwc16Count : 1];
    __shared__ uint32_t s_c16[kMwc16 ? kMwc16Count : 1];  // a_i^k * 2^48 mod m_i
    __shared__ uint32_t s_t8[kXs32 ? 1024 : 1];           // byte tables of the xorshift32 M^k
    __shared__ uint4 s_t4[kXs256 ? 2048 : 1];              // partial columns, then the table of M^k
    __shared__ uint32_t s_col[kXs256 ? 256 * 8 : 1];       // columns of M^k
    const uint32_t tid = threadIdx.x;
    if constexpr (kMwc16) {
        for (uint32_t i = tid; i < (uint32_t)kMwc16Count; i += WG) {
            const uint32_t ai = a.tab.t392[i];
            const uint32_t *p = a.tab.mwc16_pow + (size_t)i * 64;
            uint32_t c = (uint32_t)(((uint64_t)1 << 48) % (ai * 65536u - 1u));  // fold image of 1
            for (int b = 0; b < 64 && (a.k >> b); ++b)
                if ((a.k >> b) & 1) c = mwc16_mulmod(c, p[b], ai);
            s_t392[i] = (uint16_t)ai;
            s_c16[i] = c;
        }
    }
    if constexpr (kXs32) {
        // entry p * 256 + v: XOR of columns 8p + j over the set bits j of v
        for (uint32_t e = tid; e < 1024; e += WG) {
            const uint32_t p = e >> 8, v = e & 255;
            uint32_t r = 0;
            for (int j = 0; j < 8; ++j)
                if ((v >> j) & 1) r ^= a.xs32[8 * p + j];
            s_t8[e] = r;
        }
    }
    if constexpr (kXs256) {
        // Column c of M^k is the XOR of M^i e_c over the set bits i of x^k mod
        // the characteristic polynomial: threads c, 256 + c, ... take 64 of the
        // 256 steps each, from the columns of M^64, M^128 and M^192 (entries of
        // single bits in those tables).  For k of two hexadecimal digits it is the
        // second one's map of column c of the first one's, a quarter of its 64
        // nibbles per thread; a single digit's table is the one in memory.
        const uint32_t c = tid & 255, seg = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 8);
        auto column = [&](uint32_t table, uint32_t (&v)[8]) {
            const uint4 *T = a.tab.xs256_t4w + (size_t)table * 2048 + (c >> 2) * 32 + (1u << (c & 3));
            const uint4 lo = T[0], hi = T[16];
            v[0] = lo.x;
            v[1] = lo.y;
            v[2] = lo.z;
            v[3] = lo.w;
            v[4] = hi.x;
            v[5] = hi.y;
            v[6] = hi.z;
            v[7] = hi.w;
        };
        uint32_t col[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        if constexpr (kFew) {
            if (a.digits == 1) {
                const uint4 *T = a.tab.xs256_t4w + (size_t)a.t4w[0] * 2048;
                const uint4 q0 = T[tid], q1 = T[kSkipXs256WG + tid];
                s_t4[tid] = q0;
                s_t4[kSkipXs256WG + tid] = q1;
            } else {
                uint32_t v[8];
                column(a.t4w[0], v);
                const uint4 *T = a.tab.xs256_t4w + (size_t)a.t4w[1] * 2048 + seg * 512;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    uint32_t w = v[h];
#pragma unroll
                    for (int i = 1; i < 4; ++i) w = seg == (uint32_t)i ? v[2 * i + h] : w;
#pragma unroll
                    for (int p = 0; p < 8; ++p) {
                        const uint32_t n = (w >> (4 * p)) & 15u;
                        const uint4 lo = T[(8 * h + p) * 32 + n], hi = T[(8 * h + p) * 32 + 16 + n];
                        col[0] ^= lo.x;
                        col[1] ^= lo.y;
                        col[2] ^= lo.z;
                        col[3] ^= lo.w;
                        col[4] ^= hi.x;
                        col[5] ^= hi.y;
                        col[6] ^= hi.z;
                        col[7] ^= hi.w;
                    }
                }
            }
        } else {
            GenXS256 g;
#pragma unroll
            for (int i = 0; i < 8; ++i) g.v[i] = (uint32_t)(c / 32 == (uint32_t)i) << (c % 32);
            if (seg) column(15 + 4 * seg - 1, g.v);
            uint64_t bits = a.poly[seg];  // uniform
#pragma unroll 1
            for (int i = 0; i < 64; i += 8, bits >>= 8)
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    if ((bits >> b) & 1)
#pragma unroll
                        for (int k = 0; k < 8; ++k) col[k] ^= g.v[k];
                    g.next();
                }
        }
        if (!kFew || a.digits != 1) {
            uint32_t *part = (uint32_t *)s_t4;  // [4][8][256]
#pragma unroll
            for (int i = 0; i < 8; ++i) part[(seg * 8 + i) * 256 + c] = col[i];
            __syncthreads();
            for (uint32_t e = tid; e < 2048; e += WG)  // word e / 256 of column e % 256
                s_col[(e & 255) * 8 + (e >> 8)] = xor3(part[e], part[2048 + e], part[4096 + e]) ^ part[6144 + e];
            __syncthreads();
            // quad q = (2p + h) * 16 + v: words 4h .. 4h+3 of the XOR of columns 4p + j over the set bits j of v
            for (uint32_t q = tid; q < 2048; q += WG) {
                const uint32_t p = q >> 5, h = (q >> 4) & 1, v = q & 15;
                uint32_t r[4] = {0, 0, 0, 0};
                for (int j = 0; j < 4; ++j)
                    if ((v >> j) & 1)
                        for (int w = 0; w < 4; ++w) r[w] ^= s_col[(4 * p + j) * 8 + 4 * h + w];
                s_t4[q] = make_uint4(r[0], r[1], r[2], r[3]);
            }
        }
    }
    if constexpr (kMwc16 || kXs32 || kXs256) __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * WG;
    for (uint64_t s = (uint64_t)blockIdx.x * WG + tid; s < a.S; s += stride) {
        G g;
        g.load(a.st, a.ld, s, a.tab);
        if constexpr (G::kId == G_MWC32) {
            const uint64_t z = mwc32_mulmod((uint64_t)g.c << 32 | g.x, a.mwc32_f, a.tab.mwc32_a, a.tab.mwc32_m);
            g.x = (uint32_t)z;
            g.c = (uint32_t)(z >> 32);
        } else if constexpr (kXs256) {
            gf2_apply256_t4(s_t4, g.v);
        } else if constexpr (G::kId == G_XS32) {
            g.y = xs32_by_bytes(s_t8, g.y);
        } else {  // MWC1616, KISS
            g.z = mwc16_mulmod(g.z, s_c16[lds_t392_index(s_t392, g.a1)], g.a1);
            g.w = mwc16_mulmod(g.w, s_c16[lds_t392_index(s_t392, g.a2)], g.a2);
            if constexpr (G::kId == G_KISS) {
                g.jsr = xs32_by_bytes(s_t8, g.jsr);
                g.jcong = a.lcg_a * g.jcong + a.lcg_c;
            }
        }
        g.store(a.st, a.ld, s);
    }
}

// Each state jumps by k on its own (the generator's own jump).
template <class G>
__global__ __launch_bounds__(kSkipWG) void k_skip_each(SkipArgs a)
{
    const uint64_t s = (uint64_t)blockIdx.x * kSkipWG + threadIdx.x;
    if (s >= a.S) return;
    G g;
    g.load(a.st, a.ld, s, a.tab);
    g.jump(a.k, a.tab);
    g.store(a.st, a.ld, s);
}

// A wave per state, for few states: the k-step map is built from the step's own
// constants in registers, so that nothing is prepared in LDS or on the host (a
// table of 392 MWC16 constants per workgroup took the launch to 15 us for one
// KISS state).  Lanes below 32 carry the first MWC16 word, the others the
// second; lane c of 32 holds column c of each xorshift32 power, read 16 powers
// ahead, and a product is an XOR over those lanes.
constexpr uint64_t kSkipWaveMax = 4096;

template <class G>
__global__ __launch_bounds__(64) void k_skip_wave(SkipArgs a)
{
    constexpr bool kMwc16 = G::kId == G_MWC1616 || G::kId == G_KISS;
    constexpr bool kXs32 = G::kId == G_XS32 || G::kId == G_KISS;
    const int lane = threadIdx.x;
    G g;
    load_uniform(g, a.st, a.ld, blockIdx.x);
    const int nb = 64 - __builtin_clzll(a.k);  // k > 0
    uint32_t y = 0;
    if constexpr (G::kId == G_XS32) y = g.y;
    if constexpr (G::kId == G_KISS) y = g.jsr;
    if constexpr (kXs32) {
        y = (uint32_t)__builtin_amdgcn_readfirstlane((int)y);
        for (int b0 = 0; b0 < nb; b0 += 16) {
            uint32_t col[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) col[i] = a.tab.xs32_pow[(b0 + i) * 32 + (lane & 31)];  // 64 powers
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if ((a.k >> (b0 + i)) & 1) y = xor_over_32(col[i] & (0u - ((y >> (lane & 31)) & 1u)));
        }
    }
    if constexpr (G::kId == G_XS256) xs256_wave_jump(g.v, a.k, lane, a.tab);
    if constexpr (G::kId == G_XS32) g.y = y;
    if constexpr (kMwc16) {
        const uint32_t ai = lane < 32 ? g.a1 : g.a2, m = ai * 65536u - 1u;
        uint32_t z = lane < 32 ? g.z : g.w, c = (0u - m) % m;  // one step is a; a 2^48 = 2^32 (mod m)
        uint32_t la = 69069u, lc = 1234567u;
        for (int b = 0; b < nb; ++b) {
            if ((a.k >> b) & 1) {
                z = mwc16_mulmod(z, c, ai);
                if constexpr (G::kId == G_KISS) g.jcong = la * g.jcong + lc;
            }
            c = mwc16_mulmod(c, c, ai);
            lc = la * lc + lc;
            la *= la;
        }
        g.z = (uint32_t)__builtin_amdgcn_readlane((int)z, 0);
        g.w = (uint32_t)__builtin_amdgcn_readlane((int)z, 32);
        if constexpr (G::kId == G_KISS) g.jsr = y;
    }
    if (lane == 0) g.store(a.st, a.ld, blockIdx.x);
}

template <class G>
int launch_skip_by(const SkipArgs &a, hipStream_t stream)
{
    if constexpr (G::kId != G_MWC32) {
        if (a.S <= kSkipWaveMax) {
            hipLaunchKernelGGL(k_skip_wave<G>, dim3((unsigned)a.S), dim3(64), 0, stream, a);
            return hipGetLastError() == hipSuccess ? 0 : -1;
        }
    }
    if (G::kId == G_XS256 && (a.S < kXs256TableMin || (a.S < kXs256ChainMax && a.digits <= 2))) {  // see the file comment
        hipLaunchKernelGGL(k_skip_each<G>, dim3((unsigned)((a.S + kSkipWG - 1) / kSkipWG)), dim3(kSkipWG), 0, stream,
                           a);
        return hipGetLastError() == hipSuccess ? 0 : -1;
    }
    // workgroups that build LDS tables stride over the states: one per CU
    // for XS256, two for MWC16
    constexpr int WG = skip_wg<G>();
    const uint64_t cap = G::kId == G_XS256 ? 256 : (G::kId == G_MWC1616 || G::kId == G_KISS) ? 512 : 4096;
    const uint64_t need = (a.S + WG - 1) / WG;
    const unsigned blocks = (unsigned)(need < cap ? need : cap);
    if constexpr (G::kId == G_XS256) {
        if (a.digits <= 2) {
            hipLaunchKernelGGL((k_skip_by<G, true>), dim3(blocks), dim3(WG), 0, stream, a);
            return hipGetLastError() == hipSuccess ? 0 : -1;
        }
    }
    hipLaunchKernelGGL(k_skip_by<G>, dim3(blocks), dim3(WG), 0, stream, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace

int dispatch_skip(int g, uint32_t *st, uint64_t ld, uint64_t S, uint64_t k, const DevTables &tab, hipStream_t s)
{
    if (S == 0 || k == 0) return 0;
    SkipArgs a{};
    a.st = st;
    a.ld = ld;
    a.S = S;
    a.k = k;
    a.tab = tab;
    if (g == RNG_MWC32) a.mwc32_f = mwc32_fold_const(k);
    if (g == RNG_XS256 && S > kSkipWaveMax) {
        for (uint32_t j = 0; j < 16; ++j)
            if (const uint32_t d = (uint32_t)(k >> (4 * j)) & 15u) {
                if (a.digits < 2) a.t4w[a.digits] = j * 15 + d - 1;
                ++a.digits;
            }
        if (S >= kXs256TableMin && a.digits > 2) xs256_jump_poly(k, (uint32_t *)a.poly);
    }
    if ((g == RNG_XS32 || g == RNG_KISS) && S > kSkipWaveMax) xs32_lcg_jump(k, a.xs32, &a.lcg_a, &a.lcg_c);
    switch (g) {
    case RNG_MWC32: return launch_skip_by<GenMWC32>(a, s);
    case RNG_XS256: return launch_skip_by<GenXS256>(a, s);
    case RNG_XS32: return launch_skip_by<GenXS32>(a, s);
    case RNG_KISS: return launch_skip_by<GenKISS>(a, s);
    case RNG_MWC1616: return launch_skip_by<GenMWC1616>(a, s);
    }
    return -2;
}

}  // namespace rngx
