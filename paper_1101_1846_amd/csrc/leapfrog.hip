// leapfrog.hip -- leapfrog parallelisation of one sequence (Sec. II.A.4), the
// entry point.  A lane that emits R_j, R_{j+T}, R_{j+2T}, ... pays a T-step map
// for every number, a 256x256 GF(2) product for XS256 (15 ms for 2^30 numbers,
// bound by its LDS look-ups); the lanes here leap over blocks of numbers
// instead, as split sequences do (seq.hip, seq_xs256.hip: 0.71 ms).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rng.h"
#include "rng_abi_internal.hpp"

using namespace rngx;

extern "C" {

int rng_leapfrog_workspace_bytes(int g, uint64_t n_threads, uint64_t *bytes)
{
    if (check_gen(g)) return RNG_EINVAL;
    if (!bytes) return fail(RNG_EINVAL, "bytes is NULL");
    if (n_threads > ((uint64_t)1 << 36)) return fail(RNG_ERANGE, "n_threads above 2^36");
    // One copy of a state is used of it.  The size, a state per thread and the
    // tables of a leap by n_threads steps, is the one that callers have been given.
    const uint64_t states = (n_threads * gen_words(g) * 4 + 255) & ~(uint64_t)255;
    *bytes = states + 256 + (g == RNG_XS256 ? 40960 : g == RNG_XS32 || g == RNG_KISS ? 4096 : 0);
    return RNG_OK;
}

int rng_generate_leapfrog(int g, const uint32_t *d_state_one, uint64_t total, uint64_t n_threads, int t,
                          void *d_out, uint32_t *d_final_state, void *d_workspace, uint64_t workspace_bytes,
                          void *stream)
{
    if (check_gen(g)) return RNG_EINVAL;
    if (t != RNG_U32 && t != RNG_F32) return fail(RNG_EINVAL, "unknown dtype %d", t);
    if (!d_state_one || !d_final_state) return fail(RNG_EINVAL, "NULL state");
    hipStream_t st = (hipStream_t)stream;
    if (total == 0) {
        if (d_final_state == d_state_one) return RNG_OK;
        hipError_t e = hipMemcpyAsync(d_final_state, d_state_one, gen_words(g) * 4, hipMemcpyDeviceToDevice, st);
        return e == hipSuccess ? RNG_OK : hip_fail(e, "hipMemcpyAsync");
    }
    if (!d_out || !d_workspace) return fail(RNG_EINVAL, "NULL output or workspace");
    if (n_threads == 0) return fail(RNG_EINVAL, "n_threads is 0");
    if (((uintptr_t)d_out & 3) || ((uintptr_t)d_workspace & 255) || ((uintptr_t)d_state_one & 3) ||
        ((uintptr_t)d_final_state & 3))
        return fail(RNG_EINVAL, "misaligned pointer");
    if (int rc = check_sizes(1, total, 1)) return rc;
    const uint64_t T = n_threads < total ? n_threads : total;
    uint64_t need = 0;
    if (int rc = rng_leapfrog_workspace_bytes(g, T, &need)) return rc;
    if (workspace_bytes < need)
        return fail(RNG_ENOMEM, "workspace %llu bytes < %llu", (unsigned long long)workspace_bytes,
                    (unsigned long long)need);
    DevTables tab;
    if (int rc = device_tables(&tab)) return rc;
    return seq_run(g, d_state_one, total, t, d_out, d_final_state, (uint32_t *)d_workspace, tab, st);
}

}  // extern "C"
