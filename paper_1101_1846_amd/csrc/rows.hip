// rows.hip -- stream-major rows of any length, count and alignment, one row
// per lane.  What bounds rows that are no whole number of 128-byte lines is
// partial lines: written from row starts in tiles of 128 numbers, every tile
// of a row of 1000 ends inside a line that the next tile completes some
// microseconds later, after the first half has left the L2 (XS256, 300007 x
// 1000: 3.0 TB/s, against 4.9 for rows of 896 or 992).  Here a lane first
// steps to the next line boundary and keeps those up to 31 numbers in
// registers; its tiles are whole lines from there on, and behind its last
// number it writes the first ones of the next lane's row, which complete the
// line that the two rows share.  Only a group of 64 rows begins and ends with
// a partial line.
//
// Too few streams for that are cut into P chunks each, P a power of two up to
// 64, and a lane's row is a chunk: chunk v mod P of stream v / P, which follows
// the row before it in memory like any other.  All chunks of a stream are lanes
// of one wave, so every lane has read its start state before the last chunk's
// writes the stream's back, and one launch does it.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "rng.h"
#include "rng_abi_internal.hpp"
#include "wave_starts.hpp"

namespace rngx {

namespace {

struct RowArgs {
    uint32_t *state;  // [W][ld]
    uint64_t ld, S;   // word stride, streams
    uint64_t N;       // numbers per stream
    uint32_t lgp, C;  // log2 of the chunks per stream, numbers per chunk (the last one N - (P - 1) C)
    uint32_t *out;    // [S][N]
    DevTables tab;
};

typedef __attribute__((address_space(1))) uint32_t gu32;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) u32x4 gu32x4;

template <int DT>
__device__ __forceinline__ uint32_t row_bits(uint32_t u)
{
    if constexpr (DT == RNG_DT_F32) return __float_as_uint(to_unit_f32(u));
    else return u;
}

// Groups whose states a wave reads before its first store (a wait for a load
// waits for the stores before it too), as far as the registers go: 512 for 4
// waves per CU with tiles of 128, 256 for 8 with tiles of 64.  Chunks make one
// group per wave.
template <class G>
constexpr int row_groups(int K, bool chunks)
{
    return chunks ? 1 : K >= 128 ? 16 : G::W > 6 ? 4 : 8;
}

// Rows below this take 64-number tiles, 8 waves per CU: most of a short row is
// its head and its last tile, which do not overlap their own stores.
constexpr uint64_t kRowShort = 512;

// kChunks: more than one chunk per stream.
template <class G, int DT, int K, bool kChunks>
__global__ __launch_bounds__(64) void k_rows(RowArgs a)
{
    constexpr int U = 8, LD = K + 4, QPR = K / 4, RPI = 64 / QPR, MG = row_groups<G>(K, kChunks);
    __shared__ __attribute__((aligned(16))) uint32_t tile[64 * LD];
    __shared__ uint32_t s_ext[64];  // numbers from a row's first whole line to the next row's
    const int lane = threadIdx.x;
    const uint64_t wave = blockIdx.x, nwaves = gridDim.x, R = kChunks ? a.S << a.lgp : a.S, groups = (R + 63) / 64;
    const uint32_t ng = (uint32_t)((groups - wave + nwaves - 1) / nwaves);  // the launcher keeps it within MG
    const uint32_t N = (uint32_t)a.N, lgp = kChunks ? a.lgp : 0, lastj = (1u << lgp) - 1, tail = N - lastj * a.C;
    // row r of a group from the group's first number on
    auto begin = [&](uint32_t r) { return kChunks ? (r >> lgp) * N + (r & lastj) * a.C : r * N; };
    uint32_t *row = tile + lane * LD;
    const int r0 = lane / QPR, q = lane % QPR;
    const uint32_t *src = tile + r0 * LD + 4 * q;
    G gs[MG];
#pragma unroll
    for (int i = 0; i < MG; ++i)
        if ((uint32_t)i < ng)
            gs[i].load(a.state, a.ld, min((wave + (uint64_t)i * nwaves) * 64 + lane, R - 1) >> lgp, a.tab);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): every state is in before the first store
    G g;
    u32x4 P[QPR];
    auto eight = [&](int k) {
        uint32_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = row_bits<DT>(g.next());
#pragma unroll
        for (int u = 0; u < U; u += 4) *(uint4 *)&row[k + u] = make_uint4(v[u], v[u + 1], v[u + 2], v[u + 3]);
    };
    auto fence = [] { asm volatile("" ::: "memory"); };  // a wave's LDS instructions execute in order
    auto transpose = [&] {
        fence();
#pragma unroll
        for (int i = 0; i < QPR; ++i) P[i] = *(const u32x4 *)(src + i * RPI * LD);
        fence();
    };
    for (uint32_t gi = 0; gi < ng; ++gi) {
        const uint64_t sb = wave + (uint64_t)gi * nwaves, s0 = sb * 64;
        g = gs[0];
#pragma unroll
        for (int i = 0; i + 1 < MG; ++i) gs[i] = gs[i + 1];
        const uint32_t rows = (uint32_t)min<uint64_t>(64, R - s0);
        // words relative to the line in which the group starts
        gu32 *base = (gu32 *)a.out + (s0 >> lgp) * a.N;
        const uint32_t e = (uint32_t)((uintptr_t)base >> 2) & 31;
        base -= e;
        // lanes past the last row repeat it, numbers and stores alike
        const uint32_t rl = min((uint32_t)lane, rows - 1), j = rl & lastj, rel = e + begin(rl);
        const bool mine = (uint32_t)lane < rows;
        const uint32_t len = !kChunks ? N : j == lastj ? tail : a.C;
        if constexpr (kChunks) lane_jump(g, j * a.C, 32 - __builtin_clz(lastj * a.C), tile, lane, a.tab);
        const uint32_t h = min((0u - rel) & 31u, len);
        uint32_t maxh = 0;
#pragma unroll
        for (int b = 16; b; b >>= 1)
            if (__ballot(h >= maxh + b)) maxh += b;
        uint32_t hv[31];
        if (maxh) {
#pragma unroll
            for (int k = 0; k < 31; ++k) {
                hv[k] = 0;
                if ((uint32_t)k < maxh) {
                    G n = g;
                    hv[k] = row_bits<DT>(n.next());
                    if ((uint32_t)k < h) g = n;
                }
            }
            if (e) {  // the first row's share of the line that the previous group ends in
                fence();
#pragma unroll
                for (int k = 0; k < 31; ++k)
                    if (lane == 0) tile[k] = hv[k];
                fence();
                const uint32_t h0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)h);
                if ((uint32_t)lane < h0) base[e + lane] = tile[lane];
                fence();
            }
        }
        uint32_t hn = (uint32_t)__shfl_down((int)h, 1, 64);  // every lane active
        hn = (uint32_t)lane + 1 < rows ? hn : 0;
        const uint32_t L = len - h;
        const uint32_t ext = L + hn, prevL = (uint32_t)__shfl_up((int)L, 1, 64);
        s_ext[lane] = ext;
        uint32_t off[QPR];  // bytes: this lane's quad of the rows that it stores
#pragma unroll
        for (int i = 0; i < QPR; ++i) off[i] = ((e + begin(min((uint32_t)(r0 + i * RPI), rows - 1)) + 31) & ~31u) * 4 + 16 * q;
        uint32_t minL = L, maxE = ext;
#pragma unroll
        for (int o = 32; o; o >>= 1) {
            minL = min(minL, (uint32_t)__shfl_xor((int)minL, o, 64));
            maxE = max(maxE, (uint32_t)__shfl_xor((int)maxE, o, 64));
        }
        minL = (uint32_t)__builtin_amdgcn_readfirstlane((int)minL);
        maxE = (uint32_t)__builtin_amdgcn_readfirstlane((int)maxE);
        const uint32_t Tf = minL / K;  // whole tiles of every row

        __attribute__((address_space(1))) char *dst = (__attribute__((address_space(1))) char *)base;
        if (Tf) {
#pragma unroll
            for (int k = 0; k < K; k += U) eight(k);
            transpose();
            for (uint32_t t = 1; t < Tf; ++t) {
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
            dst += 4 * K;
        }
        for (uint32_t k0 = Tf * K; k0 < maxE; k0 += K, dst += 4 * K) {
            const uint32_t cnt = L > k0 ? min(L - k0, (uint32_t)K) : 0;
            uint32_t k = 0;
            for (; k + U <= cnt; k += U) eight((int)k);
            for (; k < cnt; ++k) row[k] = row_bits<DT>(g.next());
            if (maxh && lane && mine) {  // the previous row's line ends with the first numbers of this one
                const uint32_t at = prevL - k0;  // wraps below k0: never < K then, up to at + 31
#pragma unroll
                for (int i = 0; i < 31; ++i)
                    if ((uint32_t)i < h && at + i < (uint32_t)K) row[(int)(at + i) - LD] = hv[i];
            }
            fence();
#pragma unroll 4
            for (int i = 0; i < QPR; ++i) {
                const uint32_t n = s_ext[r0 + i * RPI], c = k0 + 4 * q;
                const uint32_t *from = src + i * RPI * LD;
                const uint32_t r = min((uint32_t)(r0 + i * RPI), rows - 1);
                gu32 *to = (gu32 *)(dst + (((e + begin(r) + 31) & ~31u) * 4 + 16 * q));
                if (c + 4 <= n) {
                    *(gu32x4 *)to = *(const u32x4 *)from;
                } else if (c < n) {
                    for (uint32_t w = 0; w < n - c; ++w) to[w] = from[w];
                }
            }
            fence();
        }
        if (mine && j == lastj) g.store(a.state, a.ld, (s0 + lane) >> lgp);
    }
}

template <class G, int DT, int K>
int launch_rows_k(const RowArgs &a, hipStream_t st)
{
    const uint64_t groups = ((a.S << a.lgp) + 63) / 64, waves = 1024 * (128 / K);
    const uint64_t per = std::min<uint64_t>((groups + waves - 1) / waves, row_groups<G>(K, a.lgp > 0));
    const dim3 grid((unsigned)((groups + per - 1) / per)), block(64);
    if constexpr (G::kId != G_XS256) {
        if (a.lgp) {
            hipLaunchKernelGGL((k_rows<G, DT, K, true>), grid, block, 0, st, a);
            return hipGetLastError() == hipSuccess ? 0 : -1;
        }
    }
    hipLaunchKernelGGL((k_rows<G, DT, K, false>), grid, block, 0, st, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <class G>
int launch_rows_t(int dt, const RowArgs &a, hipStream_t st)
{
    if (a.C < kRowShort)
        return dt == RNG_DT_F32 ? launch_rows_k<G, RNG_DT_F32, 64>(a, st) : launch_rows_k<G, RNG_DT_U32, 64>(a, st);
    return dt == RNG_DT_F32 ? launch_rows_k<G, RNG_DT_F32, 128>(a, st) : launch_rows_k<G, RNG_DT_U32, 128>(a, st);
}

}  // namespace

// Chunks of S streams of N numbers: as many as give every wave slot a group of
// 64 (four waves per CU; eight with chunks below kRowShort of the generators whose
// numbers cost most: MWC1616 13810 x 2500 +21 %, but XS32 -17 %), of 64 numbers or
// more.  They are whole lines
// if that makes the last one, which takes the rest, at most an eighth longer.  (A
// last chunk that is shorter would take its whole group off the overlapped tiles.)
bool row_chunks(int g, uint64_t S, uint64_t N, uint32_t *lgp, uint32_t *C)
{
    uint32_t lg = 0;
    if (g == RNG_XS256 || S > 65536) return false;
    while (lg < 6) {
        const uint64_t c = N >> (lg + 1), lanes = S << (lg + 1);
        const bool two = (g == RNG_KISS || g == RNG_MWC1616) && c < kRowShort;
        if (c < 64 || lanes > (two ? 2 : 1) * (uint64_t)65536) break;
        ++lg;
    }
    if (lg == 0) return false;
    const uint64_t c = N >> lg, whole = c & ~(uint64_t)31;
    *lgp = lg;
    *C = (uint32_t)(8 * (N - (whole << lg)) <= whole ? whole : c);
    return true;
}

int launch_rows(int g, int dt, uint32_t *state, uint64_t ld, uint64_t S, uint64_t N, uint32_t lgp, uint32_t C, void *out,
                const DevTables &tab, hipStream_t st)
{
    RowArgs a{};
    a.state = state;
    a.ld = ld;
    a.S = S;
    a.N = N;
    a.lgp = lgp;
    a.C = C;
    a.out = (uint32_t *)out;
    a.tab = tab;
    switch (g) {
    case RNG_MWC32: return launch_rows_t<GenMWC32>(dt, a, st);
    case RNG_XS256: return launch_rows_t<GenXS256>(dt, a, st);
    case RNG_XS32: return launch_rows_t<GenXS32>(dt, a, st);
    case RNG_KISS: return launch_rows_t<GenKISS>(dt, a, st);
    case RNG_MWC1616: return launch_rows_t<GenMWC1616>(dt, a, st);
    }
    return -2;
}

}  // namespace rngx
