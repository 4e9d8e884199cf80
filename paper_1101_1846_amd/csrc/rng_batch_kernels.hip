// rng_batch_kernels.hip -- the first kernel of the batched path (start states,
// tile map, empty requests), and the dispatch to the persistent generation
// kernel (rng_batch_gen.hpp, built per workgroup size in batch_gen_*.hip), whose
// wavefronts pull tiles from an atomic counter until the batch is done.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "rng_batch_internal.hpp"
#include "rng_device.hpp"
#include "rng_internal.hpp"
#include "wave_starts.hpp"

namespace rngx {

// Calls F.template operator()<Generator>() for the generator id g.
template <class F>
__device__ __forceinline__ void with_gen(uint32_t g, F &&f)
{
    switch (g) {
    case G_MWC32: f.template operator()<GenMWC32>(); break;
    case G_XS256: f.template operator()<GenXS256>(); break;
    case G_XS32: f.template operator()<GenXS32>(); break;
    case G_KISS: f.template operator()<GenKISS>(); break;
    case G_MWC1616: f.template operator()<GenMWC1616>(); break;
    }
}

constexpr int kRootWG = 256;

// Moves the state of an empty request, or the copy of one that batch_moved names, by
// its offset.  The whole wave; q uniform.
template <class G>
__device__ __forceinline__ void root_move(const BatchArgs &a, const BatchReq &q, uint32_t r, uint32_t *lds, int lane)
{
    const bool moved = batch_moved(q);
    G g;
    g.load(q.state, q.stride, 0);
    const uint64_t k = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(q.offset >> 32)) << 32 |
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)q.offset);
    wave_starts(g, k, kBatchLgMin, lds, lane, a.tab);
    if (lane == 0) g.store(moved ? a.ws + (uint64_t)8 * r : q.state, moved ? 1 : q.stride, 0);
}

__device__ __forceinline__ bool root_moves(const BatchReq &q)
{
    return batch_moved(q) || (q.length == 0 && q.offset);
}

// Copies the start state of each request (the wave that ends a request writes the
// state while others may not have read it yet), writes the request of each of its
// tiles, and moves the states of root_moves.  Also clears the generation kernel's tile
// counters.
// One wave per request; kMany: `each` <= 8 requests per wave at once, a lane for each
// word, as a request is mostly the latency of its reads (us, one by one / at once: 5000
// requests 5.4 / 4.4, 10^4 6.8 / 4.6, 10^5 33 / 9).
template <bool kMany>
__global__ __launch_bounds__(kRootWG) void k_batch_root(BatchArgs a, PlanInline pin, uint32_t each)
{
    __shared__ __attribute__((aligned(16))) uint32_t s_lds[kRootWG / 64][kWaveStartLds];
    const BatchHeader *hp = pin.bytes ? (const BatchHeader *)pin.q : a.hdr;
    if (pin.bytes && blockIdx.x == 0)  // the plan for the generation kernel
        for (uint32_t i = threadIdx.x; i * 16 < pin.bytes; i += kRootWG) ((uint4 *)a.hdr)[i] = pin.q[i];
    const BatchReq *reqs = plan_at<const BatchReq>(hp, hp->off_reqs);
    if (blockIdx.x == 0 && threadIdx.x < 1u << kBatchLgCounters) a.counter[threadIdx.x * kBatchCounterWords] = 0;
    const int lane = threadIdx.x & 63;
    const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = hp->n;
    constexpr uint32_t kWords = GenMWC32::W << 4 * G_MWC32 | GenXS256::W << 4 * G_XS256 | GenXS32::W << 4 * G_XS32 |
                                GenKISS::W << 4 * G_KISS | GenMWC1616::W << 4 * G_MWC1616;
    const uint32_t wave = blockIdx.x * (kRootWG / 64) + wv, waves = gridDim.x * (kRootWG / 64);
    if constexpr (kMany) {
        const uint32_t word = (uint32_t)lane & 7;
        for (uint64_t r0 = (uint64_t)wave * each; r0 < n; r0 += (uint64_t)waves * each) {
            const uint32_t sub = (uint32_t)lane >> 3, r = (uint32_t)r0 + sub;
            const bool here = sub < each && r < n;
            const BatchReq q = reqs[here ? r : n - 1];
            const uint32_t words = kWords >> 4 * hp->groups[q.group].gen & 15;
            const bool moves = here && root_moves(q);
            if (here && !moves && word < words) a.ws[(uint64_t)8 * r + word] = q.state[(uint64_t)word * q.stride];
            if (here && q.ntiles <= 64)
                for (uint32_t i = word; i < q.ntiles; i += 8) a.tile_req[q.tile_base + i] = r;
            for (uint64_t left = __ballot(word == 0 && here && (moves || q.ntiles > 64)); left; left &= left - 1) {
                const uint32_t t = (uint32_t)r0 + ((uint32_t)__builtin_ctzll(left) >> 3);
                const BatchReq u = reqs[t];
                if (root_moves(u))
                    with_gen(hp->groups[u.group].gen, [&]<class G>() { root_move<G>(a, u, t, s_lds[wv], lane); });
                if (u.ntiles > 64)
                    for (uint32_t i = lane; i < u.ntiles; i += 64) a.tile_req[u.tile_base + i] = t;
            }
        }
    } else {
        for (uint32_t r = wave; r < n; r += waves) {
            const BatchReq q = reqs[r];
            const uint32_t gen = hp->groups[q.group].gen;
            uint32_t state = 0;  // on its way while the tiles are written
            if ((uint32_t)lane < (kWords >> 4 * gen & 15)) state = q.state[(uint64_t)lane * q.stride];
            for (uint32_t i = lane; i < q.ntiles; i += 64) a.tile_req[q.tile_base + i] = r;
            if (root_moves(q)) with_gen(gen, [&]<class G>() { root_move<G>(a, q, r, s_lds[wv], lane); });
            else if ((uint32_t)lane < (kWords >> 4 * gen & 15)) a.ws[(uint64_t)8 * r + lane] = state;
        }
    }
}

// ------------------------------------------------------------------ launchers
int launch_batch_root(const BatchArgs &a, const PlanInline &pin, uint32_t requests, uint32_t moves, hipStream_t s)
{
    // No more requests per wave than the 4096 waves at once need, as states move one by
    // one, and one where most move (10^4 XS256 requests with an offset 112 us, so 102).
    const uint64_t each = moves > requests / 2 ? 1 : std::max<uint64_t>(std::min<uint64_t>(((uint64_t)requests + 4095) / 4096, 8), 1);
    const uint64_t per = each * (kRootWG / 64);
    const unsigned grid = (unsigned)std::min<uint64_t>(((uint64_t)requests + per - 1) / per, 1024);
    if (each > 1) hipLaunchKernelGGL(k_batch_root<true>, dim3(grid), dim3(kRootWG), 0, s, a, pin, (uint32_t)each);
    else hipLaunchKernelGGL(k_batch_root<false>, dim3(grid ? grid : 1), dim3(kRootWG), 0, s, a, pin, 1u);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int WG>
int batch_gen_wg(const BatchArgs &a, int unroll, unsigned grid, hipStream_t s, int *blocks);

static int batch_gen_dispatch(const BatchArgs &a, int wg, int unroll, unsigned grid, hipStream_t s, int *blocks)
{
    switch (wg) {
    case 64: return batch_gen_wg<64>(a, unroll, grid, s, blocks);
    case 128: return batch_gen_wg<128>(a, unroll, grid, s, blocks);
    case 256: return batch_gen_wg<256>(a, unroll, grid, s, blocks);
    case 512: return batch_gen_wg<512>(a, unroll, grid, s, blocks);
    case 1024: return batch_gen_wg<1024>(a, unroll, grid, s, blocks);
    }
    return -2;
}

int launch_batch_gen(const BatchArgs &a, int wg, int unroll, unsigned grid, hipStream_t s)
{
    return batch_gen_dispatch(a, wg, unroll, grid, s, nullptr);
}

int batch_gen_occupancy(int wg, int unroll, int *blocks_per_cu)
{
    if (!blocks_per_cu) return -1;
    return batch_gen_dispatch(BatchArgs{}, wg, unroll, 0, nullptr, blocks_per_cu);
}

}  // namespace rngx
