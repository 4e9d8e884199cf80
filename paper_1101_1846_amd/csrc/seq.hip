// seq.hip -- long sequences of few streams for the generators whose jump is a
// handful of instructions (MWC32, XS32, KISS, MWC1616): sequence splitting and
// leapfrogging (Sec. II.A.4) of one stream, and bulk generation of few.
//
// The two are joined: the sequence is cut into blocks of K numbers, 64
// consecutive blocks make a window, and wave p of the Wp waves of a stream
// takes windows p, p + Wp, p + 2 Wp, ...  Lane l starts at its block of the
// first window (a jump built in registers), and from one window to the next
// it leaps L = 64 K Wp numbers with one application of the L-step map.  What
// bounds it is the write rate: a window is 64 K consecutive numbers, so a wave
// writes 32 KiB runs (K = 128) that start on whole 128-byte lines for any
// length, thread count and output alignment, and no start state passes through
// memory.  A split into rows, by contrast, has row lengths that divide nothing
// evenly, whose partial lines halve the write rate, and a leap for every
// number costs a GF(2) or modular product per 4 bytes.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "host_math.hpp"
#include "rng.h"
#include "rng_abi_internal.hpp"

namespace rngx {

namespace {

struct SeqArgs {
    const uint32_t *state;  // [W][ld]
    uint64_t ld, S, N;      // word stride, streams, numbers per stream
    uint32_t *out;          // [S][N]
    uint32_t *final_state;  // [W][1] of the only stream, or null
    uint32_t wp;            // waves per stream
    DevTables tab;
};

typedef __attribute__((address_space(1))) uint32_t gu32;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) u32x4 gu32x4;

constexpr int kSeqLineWords = 32;  // 128-byte lines

template <int DT>
__device__ __forceinline__ uint32_t seq_bits(uint32_t u)
{
    if constexpr (DT == RNG_DT_F32) return __float_as_uint(to_unit_f32(u));
    else return u;
}

__device__ __forceinline__ uint32_t xs32_apply_bytes(const uint32_t *t8, uint32_t y)
{
    return xor3(t8[y & 255], t8[256 + ((y >> 8) & 255)], t8[512 + ((y >> 16) & 255)]) ^ t8[768 + (y >> 24)];
}

// The jump from the first block of a stream to block 64 p + lane, K = 2^LGK
// numbers each, and the map of the leap by 64 wp blocks.  Both are built from
// the powers M^(K 2^b), bit by bit; what bounds this is a serial chain of
// dependent instructions and loads, so everything that a wave shares is done
// once for it:
//  - MWC16 powers are squared up in registers from the step's own constant (a
//    table look-up per bit costs its memory latency, and the multiplier a
//    search first), lanes below 32 on the first word, the others on the second;
//  - MWC32 powers are read at once, one per lane;
//  - an xorshift32 product of the whole wave's state is an XOR over 32 lanes
//    that hold a column each, read for all bits at once.  Only the 6 bits of
//    the lane's own block take 64 instructions each.
// (With every lane jumping through all bits on its own, and the loads in the
// chain, k_seq took 11 us for 2^18 KISS numbers, most of it here.)
template <class G, int LGK>
struct SeqJump {
    static constexpr bool kMwc16 = G::kId == G_MWC1616 || G::kId == G_KISS;
    static constexpr bool kXs32 = G::kId == G_XS32 || G::kId == G_KISS;
    static constexpr int kMaxBits = 13;  // of p and wp (waves per stream, at most 4 kSeqWaves)
    uint64_t l32 = 0;              // the leap: MWC32 constant
    uint32_t lz = 0, lw = 0;       // MWC16 constants
    uint32_t la = 1, lc = 0;       // LCG map
    const uint32_t *t8 = nullptr;  // xorshift32 byte tables

    __device__ __forceinline__ void start(G &g, uint32_t p, uint32_t wp, uint32_t *s_t8, int lane, const DevTables &tab)
    {
        const int nb = 32 - __builtin_clz(wp);  // p < wp: bits of both
        if constexpr (G::kId == G_MWC32) {
            const uint64_t mine = tab.mwc32_pow[lane];
            auto power = [&](int b) {
                return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(mine >> 32), b) << 32 |
                       (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine, b);
            };
            uint64_t z = (uint64_t)g.c << 32 | g.x;
            for (int b = 0; b < nb; ++b) {
                const uint64_t c = power(LGK + 6 + b);
                if ((p >> b) & 1) z = mwc32_mulmod(z, c, tab.mwc32_a, tab.mwc32_m);
                if ((wp >> b) & 1) l32 = l32 ? mwc32_mulmod(l32, c, tab.mwc32_a, tab.mwc32_m) : c;
            }
#pragma unroll
            for (int b = 0; b < 6; ++b) {
                const uint64_t r = mwc32_mulmod(z, power(LGK + b), tab.mwc32_a, tab.mwc32_m);
                z = (lane >> b) & 1 ? r : z;
            }
            g.x = (uint32_t)z;
            g.c = (uint32_t)(z >> 32);
        }
        uint32_t col = 1u << (lane & 31);  // column of the leap
        if constexpr (kXs32) {
            const uint32_t *m = tab.xs32_pow + LGK * 32;
            uint32_t &word = xs32_word(g), cols[kMaxBits];
#pragma unroll
            for (int b = 0; b < kMaxBits; ++b) cols[b] = m[(6 + b) * 32 + (lane & 31)];
            uint32_t y = (uint32_t)__builtin_amdgcn_readfirstlane((int)word);
#pragma unroll
            for (int b = 0; b < kMaxBits; ++b)
                if ((p >> b) & 1) y = xor_over_32(cols[b] & (0u - ((y >> (lane & 31)) & 1u)));
            word = y;
#pragma unroll
            for (int b = 0; b < 6; ++b) {
                const uint32_t r = gf2_apply32(m + b * 32, word);
                word = (lane >> b) & 1 ? r : word;
            }
            for (int b = 0; b < nb; ++b)
                if ((wp >> b) & 1) col = gf2_apply32(m + (6 + b) * 32, col);
        }
        if constexpr (kMwc16) {
            const uint32_t ai = lane < 32 ? g.a1 : g.a2, m = ai * 65536u - 1u;
            uint32_t c = (0u - m) % m;  // one step is a; a 2^48 = 2^32 (mod a 2^16 - 1)
            uint32_t zi = lane < 32 ? g.z : g.w, li = 0, a = 69069u, d = 1234567u;
            auto square = [&] {
                c = mwc16_mulmod(c, c, ai);
                d = a * d + d;
                a *= a;
            };
            uint32_t cz[6], cw[6], ca[6], cd[6];
#pragma unroll
            for (int b = 0; b < LGK; ++b) square();
#pragma unroll
            for (int b = 0; b < 6; ++b) {
                cz[b] = (uint32_t)__builtin_amdgcn_readlane((int)c, 0);
                cw[b] = (uint32_t)__builtin_amdgcn_readlane((int)c, 32);
                ca[b] = a;
                cd[b] = d;
                square();
            }
            for (int b = 0; b < nb; ++b) {
                if ((p >> b) & 1) {
                    zi = mwc16_mulmod(zi, c, ai);
                    if constexpr (G::kId == G_KISS) g.jcong = a * g.jcong + d;
                }
                if ((wp >> b) & 1) {
                    li = li ? mwc16_mulmod(li, c, ai) : c;
                    lc = a * lc + d;
                    la *= a;
                }
                square();
            }
            lz = (uint32_t)__builtin_amdgcn_readlane((int)li, 0);
            lw = (uint32_t)__builtin_amdgcn_readlane((int)li, 32);
            g.z = (uint32_t)__builtin_amdgcn_readlane((int)zi, 0);
            g.w = (uint32_t)__builtin_amdgcn_readlane((int)zi, 32);
#pragma unroll
            for (int b = 0; b < 6; ++b) {
                const bool on = (lane >> b) & 1;
                g.z = on ? mwc16_mulmod(g.z, cz[b], g.a1) : g.z;
                g.w = on ? mwc16_mulmod(g.w, cw[b], g.a2) : g.w;
                if constexpr (G::kId == G_KISS) g.jcong = on ? ca[b] * g.jcong + cd[b] : g.jcong;
            }
        }
        if constexpr (kXs32) {
            // entry q * 256 + v: XOR of columns 8q + i over the set bits i of v
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const uint32_t v = (uint32_t)(e & 3) * 64 + lane;
                uint32_t r = 0;
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    r ^= (uint32_t)__builtin_amdgcn_readlane((int)col, 8 * (e >> 2) + i) & (0u - ((v >> i) & 1u));
                s_t8[e * 64 + lane] = r;
            }
            t8 = s_t8;
        }
    }
    static __device__ __forceinline__ uint32_t &xs32_word(G &g)
    {
        if constexpr (G::kId == G_KISS) return g.jsr;
        else return g.y;
    }
    __device__ __forceinline__ void leap(G &g, const DevTables &tab) const
    {
        if constexpr (G::kId == G_MWC32) {
            const uint64_t r = mwc32_mulmod((uint64_t)g.c << 32 | g.x, l32, tab.mwc32_a, tab.mwc32_m);
            g.x = (uint32_t)r;
            g.c = (uint32_t)(r >> 32);
        }
        if constexpr (kMwc16) {
            g.z = mwc16_mulmod(g.z, lz, g.a1);
            g.w = mwc16_mulmod(g.w, lw, g.a2);
        }
        if constexpr (kXs32) xs32_word(g) = xs32_apply_bytes(t8, xs32_word(g));
        if constexpr (G::kId == G_KISS) g.jcong = la * g.jcong + lc;
    }
};

// One wave per workgroup: nothing is shared between waves, and a wave that
// ends makes room for the next at once (4 per CU with K = 128).  The pipelined
// stores are those of the bulk kernel: the transposed quads of a window wait
// in registers and go out while the next window is generated.
template <class G, int DT, int K>
__global__ __launch_bounds__(64) void k_seq(SeqArgs a)
{
    constexpr int U = 8, LD = K + 4, QPR = K / 4, RPI = 64 / QPR, LGK = __builtin_ctz(K);
    constexpr bool kBytes = G::kId == G_XS32 || G::kId == G_KISS;
    __shared__ __attribute__((aligned(16))) uint32_t tile[64 * LD];
    __shared__ uint32_t s_t8[kBytes ? 1024 : 1];
    const int lane = threadIdx.x;
    const uint32_t s = blockIdx.x / a.wp, p = blockIdx.x - s * a.wp;
    // numbers before the first whole line of the stream's output
    gu32 *out = (gu32 *)a.out + (uint64_t)s * a.N;
    const uint32_t mis = (uint32_t)((uintptr_t)out >> 2) & (kSeqLineWords - 1);
    const uint32_t head = (uint32_t)min<uint64_t>(mis ? kSeqLineWords - mis : 0, a.N);
    const uint64_t body = a.N - head, nwin = (body + 64 * K - 1) / (64 * K);
    if (p >= nwin && p) return;
    G g;
    load_uniform(g, a.state, a.ld, s);
    for (uint32_t k = 0; k < head; ++k) {
        const uint32_t u = seq_bits<DT>(g.next());
        if (p == 0 && lane == 0) out[k] = u;
    }
    if (body == 0) {
        if (a.final_state && lane == 0) g.store(a.final_state, 1, 0);
        return;
    }
    out += head;
    SeqJump<G, LGK> j;
    j.start(g, p, a.wp, s_t8, lane, a.tab);
    uint32_t *row = tile + lane * LD;
    const int r0 = lane / QPR, q = lane % QPR;
    const uint32_t *src = tile + r0 * LD + 4 * q;
    const uint64_t stride = a.wp, full = body / (64 * K);
    uint64_t t = p;
    G g0 = g;  // the state at the start of the lane's block
    u32x4 P[QPR];
    auto eight = [&](int k) {
        uint32_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = seq_bits<DT>(g.next());
#pragma unroll
        for (int u = 0; u < U; u += 4) *(uint4 *)&row[k + u] = make_uint4(v[u], v[u + 1], v[u + 2], v[u + 3]);
    };
    // LDS instructions of a wave execute in issue order: compiler fences are enough
    auto transpose = [&]() {
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < QPR; ++i) P[i] = *(const u32x4 *)(src + i * RPI * LD);
        asm volatile("" ::: "memory");
    };
    if (t < full) {
#pragma unroll
        for (int k = 0; k < K; k += U) eight(k);
        transpose();
        gu32 *dst = out + t * (64 * K) + r0 * K + 4 * q;
        for (t += stride; t < full; t += stride) {
            j.leap(g0, a.tab);
            g = g0;
#pragma unroll
            for (int k = 0; k < K; k += U) {
                eight(k);
#pragma unroll
                for (int i = k * QPR / K; i < (k + U) * QPR / K; ++i) *(gu32x4 *)(dst + i * RPI * K) = P[i];
                __builtin_amdgcn_sched_barrier(0);
            }
            transpose();
            dst = out + t * (64 * K) + r0 * K + 4 * q;
        }
#pragma unroll
        for (int i = 0; i < QPR; ++i) *(gu32x4 *)(dst + i * RPI * K) = P[i];
        if (t - stride == nwin - 1) {  // the sequence ends with this window
            if (a.final_state && lane == 63) g.store(a.final_state, 1, 0);
            return;
        }
        if (t >= nwin) return;
        j.leap(g0, a.tab);
        g = g0;
    }
    if (t != nwin - 1) return;
    // the last window, not full: each lane stops at the end of the sequence
    const uint64_t w0 = t * (64 * K);
    const uint32_t left = (uint32_t)(body - w0), at = (uint32_t)lane * K;
    const uint32_t len = left > at ? min(left - at, (uint32_t)K) : 0;
    uint32_t k = 0;
    for (; k + U <= len; k += U) eight((int)k);
    for (; k < len; ++k) row[k] = seq_bits<DT>(g.next());
    if (a.final_state && len && at + len == left) g.store(a.final_state, 1, 0);
    asm volatile("" ::: "memory");
    gu32 *dst = out + w0;
    for (int i = 0; i < QPR; ++i) {
        const uint32_t c = (uint32_t)(r0 + i * RPI) * K + 4 * q;
        const uint32_t *from = src + i * RPI * LD;
        if (c + 4 <= left) {
            *(gu32x4 *)(dst + c) = *(const u32x4 *)from;
        } else if (c < left) {
            for (uint32_t e = 0; e < left - c; ++e) dst[c + e] = from[e];
        }
    }
}

template <class G, int DT>
int launch_seq_k(const SeqArgs &a, int k, hipStream_t st)
{
    const dim3 grid((unsigned)(a.S * a.wp)), block(64);
    switch (k) {
    case 32: hipLaunchKernelGGL((k_seq<G, DT, 32>), grid, block, 0, st, a); break;
    case 64: hipLaunchKernelGGL((k_seq<G, DT, 64>), grid, block, 0, st, a); break;
    default: hipLaunchKernelGGL((k_seq<G, DT, 128>), grid, block, 0, st, a); break;
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <class G>
int launch_seq_t(int dt, const SeqArgs &a, int k, hipStream_t st)
{
    return dt == RNG_DT_F32 ? launch_seq_k<G, RNG_DT_F32>(a, k, st) : launch_seq_k<G, RNG_DT_U32>(a, k, st);
}

// Block length and waves per stream.  Blocks of 128 numbers run 4 waves per CU
// (LDS), of 64 eight, of 32 sixteen: the longest that leave a window for about
// every wave.  A stream takes its share of those waves, or fewer if as many
// rounds of windows need no more.
void seq_shape(uint64_t S, uint64_t N, int *k, uint32_t *wp)
{
    const uint64_t total = S * N;
    *k = total >= ((uint64_t)1 << 23) ? 128 : total >= ((uint64_t)1 << 21) ? 64 : 32;
    const uint64_t win = (N + 64 * *k - 1) / (64 * *k), slots = kSeqWaves * (uint64_t)(128 / *k);
    const uint64_t share = slots > S ? slots / S : 1, rounds = (win + share - 1) / share;
    *wp = (uint32_t)((win + rounds - 1) / rounds);
}

}  // namespace

int launch_seq(int g, int dt, const uint32_t *state, uint64_t ld, uint64_t S, uint64_t N, void *out,
               uint32_t *final_state, const DevTables &tab, hipStream_t st)
{
    SeqArgs a{};
    a.state = state;
    a.ld = ld;
    a.S = S;
    a.N = N;
    a.out = (uint32_t *)out;
    a.final_state = final_state;
    a.tab = tab;
    int k;
    seq_shape(S, N, &k, &a.wp);
    switch (g) {
    case RNG_MWC32: return launch_seq_t<GenMWC32>(dt, a, k, st);
    case RNG_XS256: return launch_seq_xs256(dt, state, ld, S, N, out, final_state, tab, st);
    case RNG_XS32: return launch_seq_t<GenXS32>(dt, a, k, st);
    case RNG_KISS: return launch_seq_t<GenKISS>(dt, a, k, st);
    case RNG_MWC1616: return launch_seq_t<GenMWC1616>(dt, a, k, st);
    }
    return -2;
}

// The start state is read, and the final one written, by any wave while others
// store their numbers, so neither may lie in memory that the sequence writes: a
// start state that the output or the final state overlaps is copied to ws first,
// and a final state that the output or the start state in use overlaps is worked
// out in ws (the start state moved by `total`) and copied to its place last.
int seq_run(int g, const uint32_t *state_one, uint64_t total, int t, void *out, uint32_t *final_state, uint32_t *ws,
            const DevTables &tab, hipStream_t st)
{
    const uint64_t words = (uint64_t)gen_words(g);
    auto overlap = [](const void *p, uint64_t np, const void *q, uint64_t nq) {
        return (uintptr_t)p < (uintptr_t)q + 4 * nq && (uintptr_t)q < (uintptr_t)p + 4 * np;
    };
    const uint32_t *start = state_one;
    const bool late = overlap(final_state, words, out, total);
    if (late || overlap(state_one, words, out, total) || overlap(state_one, words, final_state, words)) start = ws;
    const bool by_ws = late || (start == ws && overlap(final_state, words, ws, words));
    if (start != state_one)
        if (int rc = check_launch(dispatch_state_copy(g, state_one, 1, 0, ws, 1, 0, st), "sequence: start state"))
            return rc;
    if (int rc = check_launch(launch_seq(g, t, start, 1, 1, total, out, by_ws ? nullptr : final_state, tab, st), "sequence"))
        return rc;
    if (!by_ws) return RNG_OK;
    if (int rc = check_launch(dispatch_skip(g, ws, 1, 1, total, tab, st), "sequence: final state")) return rc;
    return check_launch(dispatch_state_copy(g, ws, 1, 0, final_state, 1, 0, st), "sequence: final state");
}

}  // namespace rngx
