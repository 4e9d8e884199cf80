// leapfrog.hip -- leapfrog parallelisation of one sequence (Sec. II.A.4).  For
// the generators with a cheap jump the lanes leap over blocks (seq.hip).  For
// XS256, thread j of T emits R_j, R_{j+T}, R_{j+2T}, ..., so that number i of
// the sequence lands at out[i] and every wave stores 64 consecutive numbers:
// it starts at state_j (a radix-16 tree of jumps, as for sequence splitting),
// steps once, and then leaps T steps per number by v <- M^T v, a 256x256 GF(2)
// product through a 4-bit table in LDS that is built on the device.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rng.h"
#include "rng_abi_internal.hpp"

namespace rngx {

namespace {

constexpr uint64_t kConstBytes = 256;
constexpr uint64_t kColBytes = 256 * 8 * 4;
constexpr uint64_t kTableBytes = 2048 * 16;
constexpr uint64_t kByteTableBytes = 4 * 256 * 4;

uint64_t align256(uint64_t x) { return (x + 255) & ~(uint64_t)255; }

struct LeapArgs {
    const uint32_t *ws;     // [8][T] thread start states (state_j)
    const uint4 *t4;        // 4-bit table of M^T
    uint64_t T, total;
    uint32_t *out;          // [total]
    uint32_t *final_state;  // [8]
    DevTables tab;
};

template <int DT>
__device__ __forceinline__ uint32_t bits(uint32_t u)
{
    if constexpr (DT == RNG_DT_F32) return __float_as_uint(to_unit_f32(u));
    else return u;
}

// Column c of M^T for the r = 8 XorShift: the unit state e_c jumped by T.
__global__ __launch_bounds__(256) void k_leap_xs256_cols(uint64_t T, uint32_t *cols, DevTables tab)
{
    const uint32_t c = threadIdx.x;
    GenXS256 g;
#pragma unroll
    for (int i = 0; i < 8; ++i) g.v[i] = (uint32_t)(c / 32 == (uint32_t)i) << (c % 32);
    g.jump(T, tab);
#pragma unroll
    for (int i = 0; i < 8; ++i) cols[c * 8 + i] = g.v[i];
}

// Quad q = (2p + h) * 16 + v of the 4-bit table: words 4h .. 4h+3 of the XOR
// of columns 4p + k over the set bits k of v.
__global__ __launch_bounds__(256) void k_leap_xs256_table(const uint32_t *cols, uint4 *t4)
{
    const uint32_t q = blockIdx.x * 256 + threadIdx.x;
    const uint32_t p = q >> 5, h = (q >> 4) & 1, v = q & 15;
    uint32_t r[4] = {0, 0, 0, 0};
    for (int k = 0; k < 4; ++k)
        if ((v >> k) & 1)
            for (int w = 0; w < 4; ++w) r[w] ^= cols[(4 * p + k) * 8 + 4 * h + w];
    t4[q] = make_uint4(r[0], r[1], r[2], r[3]);
}

// Thread j: state_j -> one step (R_j) -> leaps of T steps (R_{j+T}, ...).
// The thread that emits R_{total-1} writes the final state.
template <int DT>
__global__ __launch_bounds__(256) void k_leapfrog(LeapArgs a)
{
    __shared__ uint4 s_t4[2048];
    stage_quads<256, 2048>(s_t4, a.t4);
    __syncthreads();
    const uint64_t j = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= a.T) return;
    GenXS256 g;
    g.load(a.ws, a.T, j);
    uint32_t u = g.next();
    for (uint64_t pos = j;;) {
        a.out[pos] = bits<DT>(u);
        if (pos == a.total - 1) g.store(a.final_state, 1, 0);
        pos += a.T;
        if (pos >= a.total) break;
        gf2_apply256_t4(s_t4, g.v);
        u = g.last();
    }
}

}  // namespace

}  // namespace rngx

using namespace rngx;

extern "C" {

int rng_leapfrog_workspace_bytes(int g, uint64_t n_threads, uint64_t *bytes)
{
    if (check_gen(g)) return RNG_EINVAL;
    if (!bytes) return fail(RNG_EINVAL, "bytes is NULL");
    if (n_threads > ((uint64_t)1 << 36)) return fail(RNG_ERANGE, "n_threads above 2^36");
    const bool bytes_t = g == RNG_XS32 || g == RNG_KISS;
    *bytes = align256(n_threads * gen_words(g) * 4) + kConstBytes + (g == RNG_XS256 ? kColBytes + kTableBytes : 0) +
             (bytes_t ? kByteTableBytes : 0);
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
    uint32_t *ws = (uint32_t *)d_workspace;
    if (seq_gen(g)) return seq_run(g, d_state_one, total, t, d_out, d_final_state, ws, tab, st);
    uint32_t *cols = (uint32_t *)((char *)d_workspace + align256(T * gen_words(g) * 4) + kConstBytes);
    uint4 *t4 = (uint4 *)((char *)cols + kColBytes);
    // thread j starts at state_j: a radix-16 tree, its first three levels (with
    // the copy of state_0) in one launch
    int rc = check_launch(dispatch_tree_head(g, d_state_one, ws, T, 1, tab, st), "leapfrog: tree head");
    for (uint32_t shift = kTreeHeadShift; !rc && ((uint64_t)1 << shift) < T; shift += 4)
        rc = check_launch(dispatch_tree_level(g, ws, T, shift, 1, tab, st), "leapfrog: tree level");
    if (rc) return rc;
    hipLaunchKernelGGL(k_leap_xs256_cols, dim3(1), dim3(256), 0, st, T, cols, tab);
    hipLaunchKernelGGL(k_leap_xs256_table, dim3(8), dim3(256), 0, st, (const uint32_t *)cols, t4);
    if (hipGetLastError() != hipSuccess) return fail(RNG_EHIP, "leapfrog: XS256 table");
    LeapArgs a{};
    a.ws = ws;
    a.t4 = t4;
    a.T = T;
    a.total = total;
    a.out = (uint32_t *)d_out;
    a.final_state = d_final_state;
    a.tab = tab;
    const dim3 grid((unsigned)((T + 255) / 256)), block(256);
    if (t == RNG_F32) hipLaunchKernelGGL((k_leapfrog<RNG_DT_F32>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((k_leapfrog<RNG_DT_U32>), grid, block, 0, st, a);
    return check_launch(hipGetLastError() == hipSuccess ? 0 : -1, "rng_generate_leapfrog");
}

}  // extern "C"
