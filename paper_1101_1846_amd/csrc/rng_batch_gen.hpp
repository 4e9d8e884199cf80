// rng_batch_gen.hpp -- the persistent generation kernel of the batched path,
// included by one translation unit per workgroup size (batch_gen_*.hip) so
// that its 25 (workgroup, unroll) shapes compile in parallel.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rng_batch_internal.hpp"
#include "rng_device.hpp"
#include "rng_internal.hpp"
#include "wave_starts.hpp"

namespace rngx {

#define RNGX_COMPILER_FENCE() asm volatile("" ::: "memory")
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Pointers read from the request table are generic to the compiler, which
// would address through FLAT instructions; FLAT accesses also count as LDS
// traffic and serialise with the tile's LDS reads.  These buffers are device
// global memory: say so, so that loads and stores are global_*.
typedef __attribute__((address_space(1))) uint32_t gu32;
typedef __attribute__((address_space(1))) u32x4 gu32x4;

__device__ __forceinline__ gu32 *global_ptr(uint32_t *p) { return (gu32 *)p; }

// LDS tile depth of the generation kernel: kBatchTile samples per row, or 32
// for 1024-lane workgroups, whose 16 tiles of 64 rows would not fit in the
// 160 KiB of LDS at 64.
constexpr int batch_tile_depth(int wg) { return wg >= 1024 ? 32 : kBatchTile; }

template <int DT>
__device__ __forceinline__ uint32_t bits_of(uint32_t u)
{
    if constexpr (DT == RNG_DT_F32) return __float_as_uint(to_unit_f32(u));
    else return u;
}

// cnt numbers of the lane's own into its row of the LDS tile.  Lanes with a whole
// block left take the unrolled path together; a lane whose numbers end inside it
// stops exactly there.
template <class G, int DT, int U>
__device__ __forceinline__ void batch_numbers(G &g, uint32_t *row, uint32_t cnt)
{
    uint32_t k = 0;
#pragma unroll 1
    for (; k + U <= cnt; k += U) {
        uint32_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = bits_of<DT>(g.next());
        if constexpr (U % 4 == 0) {
#pragma unroll
            for (int u = 0; u < U; u += 4) *(uint4 *)&row[k + u] = make_uint4(v[u], v[u + 1], v[u + 2], v[u + 3]);
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) row[k + u] = v[u];
        }
    }
    for (; k < cnt; ++k) row[k] = bits_of<DT>(g.next());
}

// The rows of one tile, lane l's states in g: c = 2^lgc samples of lane l from
// l c on, up to `left` (the samples from the tile's start to the request's end,
// at most 64 c).  K samples at a time go through the LDS tile and are stored
// with consecutive lanes on consecutive quads of a row.
template <class G, int DT, int U, int K>
__device__ __forceinline__ void batch_rows(G &g, gu32 *out, uint32_t left, uint32_t lgc, uint32_t *tile, int lane)
{
    static_assert(K % U == 0 && K % 4 == 0, "tile depth");
    constexpr int LD = K + 4, QPR = K / 4, RPI = 64 / QPR;
    const uint32_t c = 1u << lgc, at = (uint32_t)lane << lgc;
    // With 8 rows or fewer the other lanes step too, for nothing (their numbers stay in
    // LDS): a wave with so few lanes at work runs at less than half the rate beside
    // others (16 XS256 requests of 64 samples 9.9 us, so 8.6).
    const uint32_t longest = min(left, c), idle = left <= 8 * c ? longest : 0;
    const uint32_t len = left > at ? min(left - at, c) : idle;
    const bool aligned = ((uintptr_t)out & 15) == 0;
    uint32_t *row = tile + lane * LD;
    for (uint32_t k0 = 0; k0 < longest; k0 += K) {
        batch_numbers<G, DT, U>(g, row, len > k0 ? min(len - k0, (uint32_t)K) : 0);
        RNGX_COMPILER_FENCE();
        if (aligned && k0 + K <= c && left == 64u << lgc) {  // uniform: every quad is whole
            const int r0 = lane / QPR, q = lane % QPR;
            u32x4 P[QPR];
#pragma unroll
            for (int i = 0; i < QPR; ++i) P[i] = *(const u32x4 *)(tile + (r0 + i * RPI) * LD + 4 * q);
#pragma unroll
            for (int i = 0; i < QPR; ++i) *(gu32x4 *)(out + (((uint32_t)(r0 + i * RPI) << lgc) + k0 + 4 * q)) = P[i];
        } else if (aligned) {
            const int r0 = lane / QPR, q = lane % QPR;
#pragma unroll 4
            for (int i = 0; i < QPR; ++i) {
                const uint32_t col = k0 + 4 * q, pos = ((uint32_t)(r0 + i * RPI) << lgc) + col;
                const uint32_t *s = tile + (r0 + i * RPI) * LD + 4 * q;
                if (col < c && pos + 4 <= left) {
                    *(gu32x4 *)(out + pos) = *(const u32x4 *)s;
                } else if (col < c && pos < left) {
                    for (uint32_t e = 0; e < left - pos; ++e) out[pos + e] = s[e];
                }
            }
        } else {
            constexpr int RPW = 64 / K;
            const int r0 = lane / K, w = lane % K;
#pragma unroll 4
            for (int i = 0; i < K; ++i) {
                const uint32_t col = k0 + w, pos = ((uint32_t)(r0 + i * RPW) << lgc) + col;
                if (col < c && pos < left) out[pos] = tile[(r0 + i * RPW) * LD + w];
            }
        }
        RNGX_COMPILER_FENCE();
    }
}

// One tile: the wave starts its lanes from the request's state, and the lane
// that produces the request's last sample writes the state back.
template <class G, int U, int K>
__device__ __forceinline__ void batch_tile(const BatchArgs &a, const BatchReq &q, uint32_t r, uint32_t i, uint32_t dtype,
                                           uint32_t *tile, int lane)
{
    const uint64_t first = (uint64_t)i << (q.lgc + 6), rest = q.length - first;
    const uint32_t left = (uint32_t)min(rest, (uint64_t)64 << q.lgc);
    G g;
    load_uniform(g, a.ws + (uint64_t)8 * r, 1, 0);
    const uint64_t k = (batch_moved(q) ? 0 : q.offset) + first;
    if (k || left > 1u << q.lgc) wave_starts(g, k, q.lgc, tile, lane, a.tab);  // else one row, from the state itself
    gu32 *out = global_ptr(q.out) + first;
    if (dtype == RNG_DT_F32) batch_rows<G, RNG_DT_F32, U, K>(g, out, left, q.lgc, tile, lane);
    else batch_rows<G, RNG_DT_U32, U, K>(g, out, left, q.lgc, tile, lane);
    if (i + 1 == q.ntiles && (uint32_t)lane == (left - 1) >> q.lgc) g.store(q.state, q.stride, 0);
}

// A packed tile: lane l steps request r + l, `count` requests of one group, from its
// own state to its end; the rows, which begin anywhere, go out one by one.
template <class G, int DT, int U, int K>
__device__ __forceinline__ void batch_pack_rows(G &g, const BatchReq &mine, uint32_t count, uint32_t *tile, int lane)
{
    constexpr int LD = K + 4;
    constexpr uint32_t R = 8;  // divides the tile's 64 rows
    const uint32_t len = (uint32_t)lane < count ? (uint32_t)mine.length : 0;
    const uint64_t out = (uint64_t)mine.out;
    for (uint32_t k0 = 0; __ballot(len > k0); k0 += K) {
        batch_numbers<G, DT, U>(g, tile + lane * LD, len > k0 ? min(len - k0, (uint32_t)K) : 0);
        RNGX_COMPILER_FENCE();
        const uint32_t at = k0 + (uint32_t)lane;
        // R rows at once, so that their LDS reads overlap (10^4 XS256 requests of 256
        // samples 31 us, so 25); rows past `count` have no length
        for (uint32_t i = 0; i < count; i += R) {
            uint32_t v[R];
#pragma unroll
            for (uint32_t j = 0; j < R; ++j) v[j] = tile[(i + j) * LD + min(lane, K - 1)];
#pragma unroll
            for (uint32_t j = 0; j < R; ++j) {
                const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)len, (int)(i + j));
                const uint64_t to = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(out >> 32), (int)(i + j)) << 32 |
                                    (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)out, (int)(i + j));
                if (lane < K && at < n) global_ptr((uint32_t *)to)[at] = v[j];
            }
        }
        RNGX_COMPILER_FENCE();
    }
}

template <class G, int U, int K>
__device__ __forceinline__ void batch_pack(const BatchArgs &a, const BatchReq *reqs, uint32_t r, uint32_t count,
                                           uint32_t dtype, uint32_t *tile, int lane)
{
    const uint32_t m = r + min((uint32_t)lane, count - 1);
    const BatchReq mine = reqs[m];
    G g;
    g.load(a.ws + (uint64_t)8 * m, 1, 0);
    if (dtype == RNG_DT_F32) batch_pack_rows<G, RNG_DT_F32, U, K>(g, mine, count, tile, lane);
    else batch_pack_rows<G, RNG_DT_U32, U, K>(g, mine, count, tile, lane);
    if ((uint32_t)lane < count) g.store(mine.state, mine.stride, 0);
}

// Persistent generation.  Wave w of the grid's W waves takes tile w first;
// the tiles from W on are pulled from atomic counters (reset by the root
// kernel), so a batch with fewer tiles than waves issues no atomics and the
// waves without a tile leave at once.  Of 2^c counters, number i hands out tiles
// W + i, W + i + 2^c, ... to the waves w = i mod 2^c.
template <int WG, int U>
__global__ __launch_bounds__(WG) void k_batch_gen(BatchArgs a)
{
    constexpr int K = batch_tile_depth(WG), NW = WG / 64, LD = K + 4;
    constexpr int kTileWords = 64 * LD > kWaveStartLds ? 64 * LD : kWaveStartLds;
    static_assert(kTileWords % 4 == 0, "16-byte aligned tiles");
    __shared__ __attribute__((aligned(16))) uint32_t lds[NW * kTileWords];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t nwaves = gridDim.x * NW, n_tiles = uniform_read(&a.hdr->n_tiles);
    const BatchReq *reqs = plan_at<const BatchReq>(a.hdr, uniform_read(&a.hdr->off_reqs));
    uint32_t *tile = &lds[wv * kTileWords];
    uint32_t t = blockIdx.x * NW + wv;
    while (t < n_tiles) {
        const uint32_t r = uniform_read(a.tile_req + t);
        const BatchReq q = uniform_read(reqs + r);
        const BatchGroup gr = uniform_read(a.hdr->groups + q.group);
        const uint32_t i = t - q.tile_base;
        if (__builtin_expect(q.lgc >= kBatchPacked, 0)) {  // its code behind the others' (small plans gain 0.3 us)
            const uint32_t count = q.lgc - kBatchPacked + 1;
            switch (gr.gen) {
            case G_MWC32: batch_pack<GenMWC32, U, K>(a, reqs, r, count, gr.dtype, tile, lane); break;
            case G_XS256: batch_pack<GenXS256, U, K>(a, reqs, r, count, gr.dtype, tile, lane); break;
            case G_XS32: batch_pack<GenXS32, U, K>(a, reqs, r, count, gr.dtype, tile, lane); break;
            case G_KISS: batch_pack<GenKISS, U, K>(a, reqs, r, count, gr.dtype, tile, lane); break;
            case G_MWC1616: batch_pack<GenMWC1616, U, K>(a, reqs, r, count, gr.dtype, tile, lane); break;
            }
        } else {
            switch (gr.gen) {
            case G_MWC32: batch_tile<GenMWC32, U, K>(a, q, r, i, gr.dtype, tile, lane); break;
            case G_XS256: batch_tile<GenXS256, U, K>(a, q, r, i, gr.dtype, tile, lane); break;
            case G_XS32: batch_tile<GenXS32, U, K>(a, q, r, i, gr.dtype, tile, lane); break;
            case G_KISS: batch_tile<GenKISS, U, K>(a, q, r, i, gr.dtype, tile, lane); break;
            case G_MWC1616: batch_tile<GenMWC1616, U, K>(a, q, r, i, gr.dtype, tile, lane); break;
            }
        }
        if (nwaves >= n_tiles) break;  // every tile was handed out statically
        const uint32_t lgc = uniform_read(&a.hdr->lg_counters), mine = (blockIdx.x * NW + wv) & ((1u << lgc) - 1);
        uint32_t next = 0;
        if (lane == 0) next = atomicAdd(a.counter + mine * kBatchCounterWords, 1u);
        t = nwaves + mine + ((uint32_t)__builtin_amdgcn_readfirstlane((int)next) << lgc);
    }
}

template <int WG, int U>
static int gen_t(const BatchArgs &a, unsigned grid, hipStream_t s)
{
    hipLaunchKernelGGL((k_batch_gen<WG, U>), dim3(grid), dim3(WG), 0, s, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int WG, int U>
static int occ_t(int *blocks)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_batch_gen<WG, U>, WG, 0) == hipSuccess ? 0 : -1;
}

// Launch (occupancy query with grid == 0 and blocks != nullptr) for one
// workgroup size and any unroll in {1, 2, 4, 8, 16}; -2 for other unrolls.
template <int WG>
int batch_gen_wg(const BatchArgs &a, int unroll, unsigned grid, hipStream_t s, int *blocks)
{
    switch (unroll) {
#define RNGX_U(U) case U: return blocks ? occ_t<WG, U>(blocks) : gen_t<WG, U>(a, grid, s);
    RNGX_U(1) RNGX_U(2) RNGX_U(4) RNGX_U(8) RNGX_U(16)
#undef RNGX_U
    }
    return -2;
}

#define RNGX_BATCH_GEN_INSTANTIATE(WG) \
    template int batch_gen_wg<WG>(const BatchArgs &, int, unsigned, hipStream_t, int *);

}  // namespace rngx
