// seq_xs256.hip -- long XS256 sequences of few streams (sequence splitting,
// leapfrogging, bulk generation of few; Sec. II.A.4).  As in seq.hip a stream
// is cut into windows of 64 blocks, one block per lane, and wave p of Wp takes
// windows p, p + Wp, ...; but a lane's leap would be a 256x256 GF(2) product,
// so a block is long, a row of C = 2^lgc numbers that the wave stores tile by
// tile, and a wave has few windows.  Only the wave's own state moves from one
// to the next, a product per nonzero hexadecimal digit of 64 C Wp, and the
// lanes start from it each time (xs256_jump.hpp), about 8 us against 185 for a
// window of 4096-number rows: no start states in memory and one launch.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "rng.h"
#include "rng_abi_internal.hpp"
#include "xs256_jump.hpp"

namespace rngx {

namespace {

struct SeqXsArgs {
    const uint32_t *state;  // [8][ld]
    uint64_t ld, S, N;      // word stride, streams, numbers per stream
    uint32_t *out;          // [S][N]
    uint32_t *final_state;  // [8][1] of the only stream, or null
    uint32_t lgc, wp;       // log2 of the numbers per row, waves per stream
    DevTables tab;
};

typedef __attribute__((address_space(1))) uint32_t gu32;
typedef __attribute__((address_space(1))) char gchar;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) u32x4 gu32x4;

template <int DT>
__device__ __forceinline__ uint32_t xs_bits(uint32_t u)
{
    if constexpr (DT == RNG_DT_F32) return __float_as_uint(to_unit_f32(u));
    else return u;
}

// One wave per workgroup, four per CU.  K: tile depth, at most C.
template <int DT, int K>
__global__ __launch_bounds__(64) void k_seq_xs256(SeqXsArgs a)
{
    constexpr int U = 8, LD = K + 4, QPR = K / 4, RPI = 64 / QPR;
    __shared__ __attribute__((aligned(16))) uint32_t tile[64 * LD > kXs256Lds ? 64 * LD : kXs256Lds];
    const int lane = threadIdx.x;
    const uint32_t s = blockIdx.x / a.wp, p = blockIdx.x - s * a.wp;
    gu32 *out = (gu32 *)a.out + (uint64_t)s * a.N;
    const uint32_t mis = (uint32_t)((uintptr_t)out >> 2) & 31;
    const uint32_t head = (uint32_t)min<uint64_t>(mis ? 32 - mis : 0, a.N);
    const uint32_t lgwin = a.lgc + 6, C = 1u << a.lgc;
    const uint64_t body = a.N - head, nwin = (body + ((uint64_t)1 << lgwin) - 1) >> lgwin;
    if (p >= nwin && p) return;
    GenXS256 g;
    load_uniform(g, a.state, a.ld, s);
    // numbers before the first whole line of the stream's output
    for (uint32_t k = 0; k < head; ++k) {
        const uint32_t u = xs_bits<DT>(g.next());
        if (p == 0 && lane == 0) out[k] = u;
    }
    if (body == 0) {
        if (a.final_state && lane == 0) g.store(a.final_state, 1, 0);
        return;
    }
    out += head;
    GenXS256 base = g;  // the state at the start of the window (uniform)
    xs256_wave_jump(base.v, (uint64_t)p << lgwin, lane, a.tab);

    uint32_t *row = tile + lane * LD;
    const int r0 = lane / QPR, q = lane % QPR;
    const uint32_t *src = tile + r0 * LD + 4 * q;
    uint32_t off[QPR];  // bytes from a window's tile to this lane's quads
#pragma unroll
    for (int i = 0; i < QPR; ++i) off[i] = (((uint32_t)(r0 + i * RPI) << a.lgc) + 4 * q) * 4;
    auto eight = [&](int k) {
        uint32_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = xs_bits<DT>(g.next());
#pragma unroll
        for (int u = 0; u < U; u += 4) *(uint4 *)&row[k + u] = make_uint4(v[u], v[u + 1], v[u + 2], v[u + 3]);
    };
    u32x4 P[QPR];
    auto transpose = [&] {
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < QPR; ++i) P[i] = *(const u32x4 *)(src + i * RPI * LD);
        asm volatile("" ::: "memory");
    };
    const uint32_t T = C / K;
    const uint64_t full = body >> lgwin;
#pragma unroll 1
    for (uint64_t t = p; t < nwin; t += a.wp) {
        if (t != p) xs256_wave_jump(base.v, (uint64_t)a.wp << lgwin, lane, a.tab);
        g = base;
        asm volatile("" ::: "memory");  // the last tile is in registers
        xs256_lane_starts(g.v, a.lgc, tile, lane, a.tab);
        gchar *dst = (gchar *)(out + (t << lgwin));
        if (t < full) {
#pragma unroll
            for (int k = 0; k < K; k += U) eight(k);
            transpose();
            for (uint32_t i = 1; i < T; ++i) {
#pragma unroll
                for (int k = 0; k < K; k += U) {
                    eight(k);
#pragma unroll
                    for (int i = k * QPR / K; i < (k + U) * QPR / K; ++i) *(gu32x4 *)(dst + off[i]) = P[i];
                    __builtin_amdgcn_sched_barrier(0);
                }
                transpose();
                dst += 4 * K;
            }
#pragma unroll
            for (int i = 0; i < QPR; ++i) *(gu32x4 *)(dst + off[i]) = P[i];
            if (a.final_state && lane == 63 && t == nwin - 1 && full == nwin) g.store(a.final_state, 1, 0);
            continue;
        }
        // The last window, not full: whole rows, then one that ends inside, then
        // none.  The same tiles without the overlap; the row that ends is cut
        // in the tile where it does, and its lane goes on for nothing.
        const uint32_t left = (uint32_t)(body - (t << lgwin)), end = left & (C - 1);
        const bool cut = (uint32_t)lane == left >> a.lgc;
        const uint32_t ntiles = left < C ? (left + K - 1) / K : T;
        for (uint32_t i = 0; i < ntiles; ++i, dst += 4 * K) {
            const uint32_t k0 = i * K;
            if (end > k0 && end - k0 <= K) {  // uniform
                const uint32_t cnt = cut ? end - k0 : (uint32_t)K;
                uint32_t k = 0;
                for (; k + U <= cnt; k += U) eight((int)k);
                for (; k < cnt; ++k) row[k] = xs_bits<DT>(g.next());
                if (cut) {
                    if (a.final_state) g.store(a.final_state, 1, 0);
                    gu32 *to = out + (t << lgwin) + left;  // the numbers after the last whole quad
                    for (uint32_t e = left & 3; e; --e) to[-(int)e] = row[cnt - e];
                }
            } else {
#pragma unroll
                for (int k = 0; k < K; k += U) eight(k);
            }
            transpose();
#pragma unroll
            for (int j = 0; j < QPR; ++j)
                if (off[j] / 4 + k0 + 4 <= left) *(gu32x4 *)(dst + off[j]) = P[j];
        }
        if (a.final_state && end == 0 && (uint32_t)lane + 1 == left >> a.lgc) g.store(a.final_state, 1, 0);
    }
}

template <int DT>
int launch_seq_xs(const SeqXsArgs &a, hipStream_t st)
{
    const dim3 grid((unsigned)(a.S * a.wp)), block(64);
    if (a.lgc >= 7) hipLaunchKernelGGL((k_seq_xs256<DT, 128>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((k_seq_xs256<DT, 32>), grid, block, 0, st, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Row length and waves per stream by what they cost, in ns: a number per lane
// 44 (by its instructions, and by its store when every wave writes), the start
// of a window 8000.
void seq_xs_shape(uint64_t S, uint64_t N, uint32_t *lgc, uint32_t *wp)
{
    double best = 1e300;
    for (uint32_t c : {12u, 11u, 10u, 9u, 8u, 7u, 5u}) {
        const uint64_t nwin = (N + ((uint64_t)64 << c) - 1) >> (c + 6);
        const uint64_t share = std::max<uint64_t>(1, std::min(nwin, kSeqWaves / S));
        for (uint64_t more = 0; more < 2; ++more) {  // one pass of waves, or a wave per window
            const uint64_t most = more ? std::min<uint64_t>(nwin, 8 * share) : share, rounds = (nwin + most - 1) / most;
            const uint64_t w = (nwin + rounds - 1) / rounds;
            const double waves = (double)(S * w), passes = std::ceil(waves / kSeqWaves);
            const double t = passes * (double)rounds * (8000 + (double)(1u << c) * 44);
            if (t < best) {
                best = t;
                *lgc = c;
                *wp = (uint32_t)w;
            }
        }
    }
}

}  // namespace

int launch_seq_xs256(int dt, const uint32_t *state, uint64_t ld, uint64_t S, uint64_t N, void *out,
                     uint32_t *final_state, const DevTables &tab, hipStream_t st)
{
    SeqXsArgs a{};
    a.state = state;
    a.ld = ld;
    a.S = S;
    a.N = N;
    a.out = (uint32_t *)out;
    a.final_state = final_state;
    a.tab = tab;
    seq_xs_shape(S, N, &a.lgc, &a.wp);
    return dt == RNG_DT_F32 ? launch_seq_xs<RNG_DT_F32>(a, st) : launch_seq_xs<RNG_DT_U32>(a, st);
}

}  // namespace rngx
