// rng_aux_kernels.hpp -- the kernels around generation: seeding and a state
// copy, with their launchers (instantiated per generator together with the
// generation kernels of rng_kernels.hpp).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rng_device.hpp"
#include "rng_internal.hpp"

namespace rngx {

inline unsigned grid_for(uint64_t lanes, int wg) { return (unsigned)((lanes + wg - 1) / wg); }

// ------------------------------------------------------------------ seeding
template <class G>
__global__ __launch_bounds__(256) void k_seed(uint32_t *__restrict__ st, uint64_t S, uint64_t seed,
                                              uint64_t first, DevTables tab)
{
    uint64_t s = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (s >= S) return;
    uint64_t d[4];
#pragma unroll
    for (int j = 0; j < G::D; ++j) d[j] = splitmix64_at(seed, (first + s) * G::D + j);
    G g;
    g.seed(d, tab);
    g.store(st, S, s);
}

// ------------------------------------------------------------------ helpers
// Copy one stream's state between a [W] contiguous buffer and slot `idx` of
// a [W][T] structure-of-arrays buffer.
template <int W>
__global__ void k_state_copy(const uint32_t *__restrict__ src, uint64_t src_stride, uint64_t src_idx,
                             uint32_t *__restrict__ dst, uint64_t dst_stride, uint64_t dst_idx)
{
    int w = threadIdx.x;
    if (w < W) dst[w * dst_stride + dst_idx] = src[w * src_stride + src_idx];
}

// ------------------------------------------------------------------ launchers

template <class G>
int launch_seed_t(uint64_t seed, uint64_t first, uint64_t S, uint32_t *st, const DevTables &tab,
                  hipStream_t stream)
{
    hipLaunchKernelGGL(k_seed<G>, dim3(grid_for(S, 256)), dim3(256), 0, stream, st, S, seed, first, tab);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <class G>
int launch_state_copy_t(const uint32_t *src, uint64_t ss, uint64_t si, uint32_t *dst, uint64_t ds,
                        uint64_t di, hipStream_t stream)
{
    hipLaunchKernelGGL(k_state_copy<G::W>, dim3(1), dim3(64), 0, stream, src, ss, si, dst, ds, di);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace rngx
