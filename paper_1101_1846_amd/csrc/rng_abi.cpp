// rng_abi.cpp -- the C ABI declared in include/rng.h: argument checks,
// per-device tables, launch-shape selection, and the call sequences of the
// multi-kernel operations (sequence splitting).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>

#include "host_math.hpp"
#include "rng.h"
#include "rng_abi_internal.hpp"
#include "rng_internal.hpp"

namespace rngx {

static thread_local std::string g_last_error;

int fail(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return code;
}

int hip_fail(hipError_t e, const char *what)
{
    return fail(RNG_EHIP, "%s: %s", what, hipGetErrorString(e));
}

// ---------------------------------------------------------------- tables
namespace {
struct DevEntry {
    bool ready = false;
    void *blob = nullptr;
    DevTables tab{};
};
std::mutex g_mu;
DevEntry g_dev[kMaxDevices];
}  // namespace

int device_tables(DevTables *out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(RNG_ENODEV, "device %d out of range", dev);
    std::lock_guard<std::mutex> lk(g_mu);
    DevEntry &d = g_dev[dev];
    if (!d.ready) {
        hipDeviceProp_t prop;
        if ((e = hipGetDeviceProperties(&prop, dev)) != hipSuccess) return hip_fail(e, "hipGetDeviceProperties");
        if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
            return fail(RNG_ENODEV, "device %d is %s; this library is built for gfx950", dev, prop.gcnArchName);
        const HostTables &H = host_tables();
        const size_t o_t392 = 0, n_t392 = sizeof(H.t392);
        const size_t o_m32 = 1024, n_m32 = sizeof(H.mwc32_pow_fold);
        const size_t o_lcg = o_m32 + 1024, n_lcg = sizeof(H.lcg_pow);
        const size_t o_x32 = o_lcg + 1024, n_x32 = sizeof(H.xs32_pow);
        const size_t o_m16 = o_x32 + n_x32, n_m16 = sizeof(H.mwc16_pow_fold);
        const size_t o_x256w = (o_m16 + n_m16 + 255) & ~(size_t)255, n_x256w = H.xs256_t4w.size() * sizeof(uint32_t);
        const size_t o_poly = o_x256w + n_x256w, n_poly = H.xs256_poly.size() * sizeof(uint32_t);
        const size_t total = o_poly + n_poly;
        std::string host(total, '\0');
        std::memcpy(&host[o_t392], H.t392, n_t392);
        std::memcpy(&host[o_m32], H.mwc32_pow_fold, n_m32);
        std::memcpy(&host[o_lcg], H.lcg_pow, n_lcg);
        std::memcpy(&host[o_x32], H.xs32_pow, n_x32);
        std::memcpy(&host[o_m16], H.mwc16_pow_fold, n_m16);
        std::memcpy(&host[o_x256w], H.xs256_t4w.data(), n_x256w);
        std::memcpy(&host[o_poly], H.xs256_poly.data(), n_poly);
        void *blob = nullptr;
        if ((e = hipMalloc(&blob, total)) != hipSuccess) return hip_fail(e, "hipMalloc(tables)");
        if ((e = hipMemcpy(blob, host.data(), total, hipMemcpyHostToDevice)) != hipSuccess) {
            (void)hipFree(blob);
            return hip_fail(e, "hipMemcpy(tables)");
        }
        char *b = (char *)blob;
        d.tab.t392 = (const uint16_t *)(b + o_t392);
        d.tab.mwc32_pow = (const uint64_t *)(b + o_m32);
        d.tab.lcg_pow = (const uint32_t *)(b + o_lcg);
        d.tab.xs32_pow = (const uint32_t *)(b + o_x32);
        d.tab.mwc16_pow = (const uint32_t *)(b + o_m16);
        d.tab.xs256_t4w = (const uint4 *)(b + o_x256w);
        d.tab.xs256_poly = (const uint4 *)(b + o_poly);
        d.tab.mwc32_a = H.mwc32_a;
        d.tab.mwc32_m = H.mwc32_m;
        d.blob = blob;
        d.ready = true;
    }
    *out = d.tab;
    return RNG_OK;
}

int device_tables_if_ready(DevTables *out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(RNG_ENODEV, "device %d out of range", dev);
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_dev[dev].ready) return fail(RNG_EINVAL, "device %d has no tables yet: call rng_init() on it first", dev);
    *out = g_dev[dev].tab;
    return RNG_OK;
}

int shutdown_tables()
{
    std::lock_guard<std::mutex> lk(g_mu);
    int cur = 0;
    (void)hipGetDevice(&cur);
    for (int i = 0; i < kMaxDevices; ++i) {
        if (!g_dev[i].ready) continue;
        (void)hipSetDevice(i);
        (void)hipFree(g_dev[i].blob);
        g_dev[i] = DevEntry();
    }
    (void)hipSetDevice(cur);
    return RNG_OK;
}

// ---------------------------------------------------------------- shapes
int gen_words(int g)
{
    switch (g) {
    case RNG_MWC32: return 2;
    case RNG_XS256: return 8;
    case RNG_XS32: return 1;
    case RNG_KISS: return 6;
    case RNG_MWC1616: return 4;
    }
    return 0;
}

static std::mutex g_shape_mu;
static Shape g_shape[2][6][2] = {};  // [rows written as runs][generator][dtype]

// Rows of 4 or 8 KiB (n = 1024, 2048) over whole groups of 64 runs are
// written as 16 KiB runs of 4 or 2 adjacent rows per lane (on workgroups of
// up to 256 lanes, when the launch is resident): streams per run, else 0.
uint32_t run_rows(uint64_t S, uint64_t N)
{
    if (N != 1024 && N != 2048) return 0;
    const uint32_t seg = (uint32_t)(4096 / N);
    return S && S % (64 * (uint64_t)seg) == 0 ? seg : 0;
}

// Untuned defaults: 256 lanes, unroll 8 (measured on 1 KiB rows), and for
// runs 64 lanes, unroll 16 (within about 1 % of the fastest shape for every
// generator at 2^20 x 1024; 256 x 8 ran 15 % slower for XS256 and KISS).
Shape tuned_shape(int g, int dt, bool runs)
{
    std::lock_guard<std::mutex> lk(g_shape_mu);
    Shape s = g_shape[runs][g][dt];
    if (!s.wg) s = runs ? Shape{64, 16} : Shape{256, 8};
    return s;
}

// XS256 rows of an odd number of 4 KiB (N = 1024 (2i + 1)) run as four
// jumped chunks on 512- and 1024-lane workgroups: chunk c starts c N bytes
// into its row, so the four chunks of a row cover four column slots of 1 KiB.
// For an even number the chunk starts share at most two slots (N = 2048) or
// one (N = 4096 m), and the plain order is faster.
bool xs256_chunked_rows(uint64_t N) { return N % 1024 == 0 && (N / 1024) % 2 == 1; }

// The shape rng_generate uses for S streams of n samples: the one tuned for
// runs when the rows are written as runs, else the other one, except that
// XS256 rows taking the four-chunk path get 512-lane workgroups (the tuned
// shape is measured on other row lengths).
Shape row_shape(int g, int dt, uint64_t S, uint64_t n)
{
    if (run_rows(S, n)) return tuned_shape(g, dt, true);
    Shape s = tuned_shape(g, dt, false);
    if (g == RNG_XS256 && xs256_chunked_rows(n) && s.wg < 512) s.wg = 512;
    return s;
}

void set_tuned_shape(int g, int dt, bool runs, Shape s)
{
    std::lock_guard<std::mutex> lk(g_shape_mu);
    g_shape[runs][g][dt] = s;
}

bool valid_shape(uint32_t wg, uint32_t unroll)
{
    return (wg == 64 || wg == 128 || wg == 256 || wg == 512 || wg == 1024) &&
           (unroll == 1 || unroll == 2 || unroll == 4 || unroll == 8 || unroll == 16);
}

// Smallest chunk worth a jump: the jump costs a few modular multiplies for
// MWC/LCG words and 32x32 mat-vecs for xorshift32, but 256x256 mat-vecs for
// the r = 8 XorShift.
static uint64_t min_chunk(int g)
{
    switch (g) {
    case RNG_MWC32: return 64;
    case RNG_XS32: return 128;
    case RNG_MWC1616: return 128;
    case RNG_KISS: return 256;
    case RNG_XS256: return 4096;
    }
    return 1u << 30;
}

// Fewer streams than a wave has lanes: one lane per chunk, about 2^17 lanes,
// chunks a multiple of 64 samples and at least the generator's minimum.
void lane_chunks(int g, uint64_t S, uint64_t N, uint64_t *C, uint32_t *P)
{
    const uint64_t p = ((uint64_t)1 << 17) / S;
    uint64_t c = std::max<uint64_t>(min_chunk(g), (N + p - 1) / p);
    c = (c + 63) / 64 * 64;
    *C = c;
    *P = (uint32_t)((N + c - 1) / c);
}

// Lanes that chunked bulk generation by k_generate aims for (general_rows, shapes of
// more than 256 lanes asked for, XS256 above the sequences' stream counts): the waves
// the device holds at once with 128-deep LDS tiles (4 per CU, 256 CUs) times 64.  Measured
// against 2^17 and 2^15 over 64..65536 streams: 2^16 is 15-40 % faster than
// 2^17 for MWC32 and KISS and equal for XS256; 2^15 slows XS256 and KISS.
constexpr uint64_t kGenLanes = (uint64_t)1 << 16;

// Split each stream into P chunks when there are too few streams to fill the
// chip (256 CUs x 4 SIMDs; aim for >= 2 waves per SIMD).
void choose_chunks(int g, uint64_t S, uint64_t N, uint64_t align, uint64_t *C, uint32_t *P, uint64_t target_lanes)
{
    uint64_t p = 1;
    while (S * p * 2 <= target_lanes && N / (p * 2) >= min_chunk(g)) p *= 2;
    if (p == 1) {
        *C = N;
        *P = 1;
        return;
    }
    uint64_t c = (N + p - 1) / p;
    c = (c + align - 1) / align * align;
    *C = c;
    *P = (uint32_t)((N + c - 1) / c);
}

int dispatch_generate(int g, int dt, const GenArgs &a, int wg, int unroll, bool staged, hipStream_t st)
{
    switch (g) {
    case RNG_MWC32: return launch_generate_t<GenMWC32>(dt, a, wg, unroll, staged, st);
    case RNG_XS256: return launch_generate_t<GenXS256>(dt, a, wg, unroll, staged, st);
    case RNG_XS32: return launch_generate_t<GenXS32>(dt, a, wg, unroll, staged, st);
    case RNG_KISS: return launch_generate_t<GenKISS>(dt, a, wg, unroll, staged, st);
    case RNG_MWC1616: return launch_generate_t<GenMWC1616>(dt, a, wg, unroll, staged, st);
    }
    return -2;
}

#define RNGX_GEN_SWITCH(g, call)                                        \
    switch (g) {                                                        \
    case RNG_MWC32: { using G = GenMWC32; return call; }                \
    case RNG_XS256: { using G = GenXS256; return call; }                \
    case RNG_XS32: { using G = GenXS32; return call; }                  \
    case RNG_KISS: { using G = GenKISS; return call; }                  \
    case RNG_MWC1616: { using G = GenMWC1616; return call; }            \
    }                                                                   \
    return -2;

int dispatch_seed(int g, uint64_t seed, uint64_t first, uint64_t S, uint32_t *st, const DevTables &tab,
                  hipStream_t s)
{
    RNGX_GEN_SWITCH(g, launch_seed_t<G>(seed, first, S, st, tab, s))
}

int dispatch_state_copy(int g, const uint32_t *src, uint64_t ss, uint64_t si, uint32_t *dst, uint64_t ds,
                        uint64_t di, hipStream_t s)
{
    RNGX_GEN_SWITCH(g, launch_state_copy_t<G>(src, ss, si, dst, ds, di, s))
}

int dispatch_fused(int g, const FusedArgs &a, hipStream_t s)
{
    RNGX_GEN_SWITCH(g, launch_fused_pi_t<G>(a, s))
}

int check_launch(int rc, const char *what)
{
    if (rc == 0) return RNG_OK;
    if (rc == -2) return fail(RNG_EINVAL, "%s: unsupported launch shape", what);
    hipError_t e = hipGetLastError();
    return fail(RNG_EHIP, "%s: launch failed: %s", what, hipGetErrorString(e));
}

static bool mul_overflows(uint64_t a, uint64_t b, uint64_t *r)
{
    return __builtin_mul_overflow(a, b, r);
}

// Jump constants of the rotated tile order (d N / 4 samples, d = 0..3).  The
// xorshift32 columns cost about 12 us of host time per distance, so the last
// few row lengths are cached.  MWC1616 needs none from the host: the MWC16
// words' constants depend on the stream's multiplier and are built in LDS.
static void rot_constants(int g, uint64_t N, GenArgs &a)
{
    if (g == RNG_MWC32) {
        for (int d = 0; d < 4; ++d) a.rot_mwc32[d] = mwc32_fold_const((uint64_t)d * (N / 4));
        return;
    }
    if (g == RNG_MWC1616) return;
    struct Entry {
        uint64_t N = 0;
        uint32_t cols[4][32];
        uint32_t lcg[4][2];
    };
    static std::mutex mu;
    static Entry cache[8];
    static unsigned next = 0;
    std::lock_guard<std::mutex> lk(mu);
    const Entry *hit = nullptr;
    for (const Entry &e : cache)
        if (e.N == N) hit = &e;
    if (!hit) {
        Entry &e = cache[next++ % 8];
        for (int d = 0; d < 4; ++d) xs32_lcg_jump((uint64_t)d * (N / 4), e.cols[d], &e.lcg[d][0], &e.lcg[d][1]);
        e.N = N;
        hit = &e;
    }
    std::memcpy(a.rot_xs32, hit->cols, sizeof(hit->cols));
    std::memcpy(a.rot_lcg, hit->lcg, sizeof(hit->lcg));
}

// Fewer rows than a wave has lanes whose chunks (row_chunks) do not begin on whole
// lines from the stream's start on.
static bool split_lines(int g, uint64_t S, uint64_t N)
{
    uint32_t lgp, c;
    return S < 64 && N <= kRowMax && !(row_chunks(g, S, N, &lgp, &c) && c % 32 == 0);
}

// Streams that run as long sequences, windows of consecutive numbers across a
// wave (seq.hip, seq_xs256.hip), instead of rows or chunks of a row per lane: up
// to one stream per wave of the device, from the lengths on at which a stream's
// windows outnumber its 64 chunks' worth of waves (KISS, us, chunks / windows:
// 64 x 2048 10.9 / 14.0, 1000 x 4096 14.3 / 16.9, 256 x 10^4 22 / 17, 512 x 10^5
// 78 / 51, 64 x 10^5 71 / 23; 1500 x 100001 146 / 163).  XS256, whose chunks
// start by a chain of table products per lane, from shorter rows on (64 x 512
// 18.3 / 12.6, 1000 x 1000 42 / 20), with four streams per wave (4096 x 4096
// 151 / 67, 4096 x 10^4 188 / 95; but 4096 x 65536 231 / 227, 2 10^4 x 10^4 421
// either way, and 4096 x 3072 at 16 bytes into a line 70 against 56 for the four
// chunks of a workgroup), and with more where rows that long start inside 128-byte
// lines (10^4 x 25001 525 / 358).
static bool seq_streams(int g, uint64_t S, uint64_t N, bool vec4, const void *out)
{
    switch (g) {
    case RNG_XS256:
        if (S <= kSeqWaves) return N >= 512;
        if (S <= 4 * kSeqWaves && N >= 2048 && N < 16384) return !(vec4 && S % 64 == 0 && xs256_chunked_rows(N));
        return N >= 16384 && S <= ((uint64_t)1 << 24) && (N % 32 != 0 || ((uintptr_t)out & 127));
    // the cheap generators: a stream of the few whose chunks would break lines
    // early (MWC32 10 x 2500, us, general / chunks / windows 7.7 / 10.5 / 7.1, 33 x
    // 6000 8.8 / 13.8 / 7.3, but 1 x 4096 7.1 / 4.2 / 7.7; XS32 10 x 6000 13.8 / 17.3
    // / 9.0), many streams later, as windows outrun their chunks later (XS32 1000 x
    // 8192 14.7 / 16.4, 1000 x 16384 19.5 / 19.0, and the four windows of 500 x 16384
    // 15.5 / 20.6; MWC32 300 x 6000 15 / 7.8)
    case RNG_MWC32:
        if (S <= kSeqWaves / 2) return N >= 6000 || (N >= 340 && split_lines(g, S, N));
        return S <= kSeqWaves && N >= 16384;
    case RNG_XS32:
        if (S <= kSeqWaves / 4) return N >= 8192 || (N >= 4096 && split_lines(g, S, N));
        if (S <= kSeqWaves / 2) return N >= 8192 && (N < 12000 || N >= 20000);
        return S <= kSeqWaves && N >= 16384;
    }
    return S <= kSeqWaves && N >= 8192;
}

// Rows that k_generate takes although they are no whole tiles: short ones, whose
// heads and last tiles, which do not overlap their stores, cost more line by line
// (rows.hip) than the partial lines do while these stay in the caches.  From 17000
// timed calls of 1 to 3 10^5 streams x 64 to 10^6 numbers at 0, 4 and 16 bytes into
// a line; against the better kernel it is within 5 % on four of five, against the
// general one alone never far behind (us or time, general / line by line):
//   fewer rows than lanes: up to 128 numbers (XS32 33 x 100 5.1 / 7.6, KISS 10 x 75
//     8.6 / 13.3, MWC1616 10 x 128 5.2 / 7.3, XS256 10 x 128 at 4 bytes 9.7 / 11.3),
//     MWC32 whose chunks would break lines up to 340 (3 x 168 6.9 / 9.4);
//   whole lines: XS256 below 128, XS32 and MWC32 x 96, a tile and a half (XS32 100 x
//     96 5.6 / 6.0), and short rows that fill the lanes (XS32 65536 x 96 -10 %,
//     8192 x 512 7.5 / 8.6);
//   whole tiles: rows of two to four long chunks, which k_generate keeps 64 streams
//     apart (MWC32 24576 x 8192 144 / 156, 25000 x 1024 18.0 / 20.3, XS32 20032 x 8192
//     -26 %, KISS 28032 x 8192 -23 %, but XS32 8192 x 1024 15.2 / 11.2, 16384 x 2048
//     +11 %, 16384 x 16384 +17 %);
//   rows that begin inside 16 bytes: below 128 numbers (XS256 1000 x 75 10.9 / 13.4),
//     as k_generate then stores word by word (XS32 1000 x 203 twice as long);
//   else by how many numbers a lane's start and a number's steps are worth: XS256
//     1000 x 340 16.3 / 21.2, 13810 x 776 -7 %, but x 3000 +22 %; KISS 1000 x 168 -17 %,
//     x 300 +5 %, 8192 x 1000 24.7 / 18.8, x 1300 19.6 / 25.2, 40000 x 776 -6 %; MWC1616
//     1000 x 300 -17 %, x 460 +25 %, 13810 x 776 -6 %; XS32 8192 x 340 8.1 / 14.6, 2000 x
//     11000 -18 %, but 152 x 11000 +43 %, 300 x 16384 12.0 / 14.3; MWC32 13810 x 2500
//     -15 %, 40000 x 1300 -7 %, but 2000 x 50000 +22 %.
// KISS's rows gain from every lane (1000 x 75 14.2 / 12.1).  More rows than lanes
// lose only as whole tiles off a line's start (100000 x 512 at 16 bytes: XS32 39.1 /
// 42.2, XS256 46.6 / 54.2) and for XS256 as short rows beyond 2^18 (300000 x 200 62.7
// / 73.2, but 200000 x 168 44.5 / 39.8) or below 64 numbers (250000 x 60 23.8 / 28.1);
// MWC32 10^5 x 75 +54 %.  XS256 rows of an odd number of 4 KiB, which k_generate takes
// with 512 lanes, where the last pass of the row kernel's waves is short (100000 x 3072
// 255 / 280, but 64000 x 1024 130 / 44, 300007 x 3072 804 / 759).
static bool general_rows(int g, uint64_t S, uint64_t N, bool vec4, const void *out)
{
    const bool cheap = g == RNG_XS32 || g == RNG_MWC32, lines = N % 32 == 0 && !((uintptr_t)out & 127);
    if (S > 65536) {
        if (!vec4 || g == RNG_KISS) return false;
        if (lines) return g == RNG_XS256 && xs256_chunked_rows(N) && 20 * S < 17 * ((S + 65535) & ~(uint64_t)65535);
        if (g == RNG_XS256 && (N < 64 || S > ((uint64_t)1 << 18))) return N < 256;
        return N % kGenTile == 0 && N >= 512;
    }
    if (S < 64) {
        if (!lines && (N < 128 || (N == 128 && (vec4 || g == RNG_XS256)))) return true;
        if (g == RNG_MWC32 && vec4 && N < 340) return split_lines(g, S, N);
    }
    if (lines) {
        if (g == RNG_XS256) return N < 128;
        if (cheap && N == 96) return true;
        if (N % kGenTile == 0 && N >= (cheap ? 1024 : g == RNG_KISS ? 4096 : 3072) && N < 12288 && S > (cheap ? 8192 : 12288))
            return true;
        return g != RNG_KISS && N <= 512 && (S > 32768 || (cheap && S * N >= (uint64_t)1 << 22));
    }
    if (!vec4) return N < 128 && g != RNG_KISS;
    switch (g) {
    case RNG_XS256: return N < 512 || (S > kSeqWaves && N < 1536);
    case RNG_KISS: return N < 192 || (N < 1700 && (S > 16384 || (S >= 8192 && N >= 1100)));
    case RNG_MWC1616: return S >= 64 && N < (S > 8192 ? 1536 : 400);
    }
    if (S * N >= (uint64_t)1 << 26) return false;
    return S >= 64 && (N < 8192 || S >= kSeqWaves / 2 || (g == RNG_XS32 && S >= kSeqWaves / 4 && N >= 12000 && N < 60000));
}

// The kernels that take a call, and its chunks.  The row and sequence kernels have
// launch shapes of their own; row kernels only if `rows` (the caller asked for no
// shape, or for one of up to 256 lanes).
enum class Route { kGeneral, kFew, kRows, kSequences };

struct Chunks {
    uint64_t C;
    uint32_t P, lgp;  // kRows: 2^lgp chunks
};

static Route choose_route(int g, uint64_t S, uint64_t N, const void *out, bool staged, bool rows, Chunks *k)
{
    const bool vec4 = N % 4 == 0 && ((uintptr_t)out & 15) == 0;
    const bool general = !staged || (N <= kRowMax && general_rows(g, S, N, vec4, out));
    if (!general && seq_streams(g, S, N, vec4, out)) return Route::kSequences;
    rows = rows && !general && N <= kRowMax;
    uint32_t c;
    if (rows && row_chunks(g, S, N, &k->lgp, &c)) {
        k->C = c;
        return Route::kRows;
    }
    if (staged && S < 64) {
        lane_chunks(g, S, N, &k->C, &k->P);
        if (k->P > 1) return Route::kFew;
    }
    choose_chunks(g, S, N, kGenTile, &k->C, &k->P, kGenLanes);
    if (rows && k->P == 1 && N >= kRowMin && (!vec4 || S % 64 != 0 || N % kGenTile != 0)) {
        k->C = N;
        k->lgp = 0;
        return Route::kRows;
    }
    return Route::kGeneral;
}

// Whether rng_generate's shape changes anything for this call.
bool shape_matters(int g, uint64_t S, uint64_t N, const void *out)
{
    Chunks k;
    return choose_route(g, S, N, out, true, true, &k) == Route::kGeneral;
}

// Shared by rng_generate, rng_generate_ex and the tuner: S streams whose states
// live at stride ld.  asked: the caller chose the launch shape.
int generate_impl(int g, int dt, uint32_t *d_state, uint64_t ld, uint64_t S, uint64_t N, void *d_out,
                  Shape shape, bool asked, bool staged, hipStream_t st)
{
    if (S == 0 || N == 0) return RNG_OK;
    DevTables tab;
    int rc = device_tables(&tab);
    if (rc) return rc;
    GenArgs a{};
    a.state = d_state;
    a.ld = ld;
    a.S = S;
    a.N = N;
    a.out = d_out;
    a.vec4 = (N % 4 == 0) && (((uintptr_t)d_out & 15) == 0);
    a.nt = 0;  // plain stores: the streaming hint measured slower for these writes
    a.tab = tab;
    Chunks k;
    switch (choose_route(g, S, N, d_out, staged, shape.wg <= 256 || !asked, &k)) {
    case Route::kSequences:
        if (int e = check_launch(launch_seq(g, dt, d_state, ld, S, N, d_out, nullptr, tab, st), "rng_generate")) return e;
        return check_launch(dispatch_skip(g, d_state, ld, S, N, tab, st), "rng_generate: state");
    case Route::kRows:
        return check_launch(launch_rows(g, dt, d_state, ld, S, N, k.lgp, (uint32_t)k.C, d_out, tab, st), "rng_generate");
    case Route::kFew:
        return check_launch(generate_few(g, dt, d_state, ld, S, N, k.C, k.P, d_out, tab, st), "rng_generate");
    case Route::kGeneral: break;
    }
    a.C = k.C;
    a.P = k.P;
    // XS256 rows of an odd number of 4 KiB (no rotated order: a row would need
    // a 256 x 256 jump inside the write stream): four chunks per stream, each
    // jumped once at its start, before any store (one table product per
    // nonzero hexadecimal digit of j N / 4: one for N = 1024), so that the
    // waves of a group write four different column slots at once.  Only with
    // workgroups of 8+ waves: they hold all four chunks of their groups and
    // write the states back themselves, and their 32-sample tiles measured
    // faster here than 4-wave workgroups with 128-sample tiles (XS256 2^20 x
    // 1024: 832-867 us at 512 lanes against 1090-1127 at 256 and 883-949 for
    // the plain order).
    // rows of 4 or 8 KiB on workgroups of up to 256 lanes: runs of 4 or 2
    // adjacent rows per lane, 16 KiB each (when the launch is resident; else
    // the orders below), from more runs of 64 lanes on than CUs: with fewer, one
    // wave per CU steps alone (49152 x 1024 u32, us, runs / rotated rows: MWC1616
    // 72.6 / 43.5, KISS 109 / 47, MWC32 50 / 33, XS256 128 / 39; at 65536 x 1024 74
    // / 52, 110 / 55, 59 / 42, 129 / 44, but MWC1616 80128 x 1024 75 / 86).
    if (staged && a.P == 1 && a.vec4 && shape.wg <= 256) {
        a.seg = run_rows(S, N);
        if (a.seg && S / (64 * a.seg) <= 256) a.seg = 0;
    }
    if (g == RNG_XS256 && staged && a.P == 1 && a.vec4 && S % 64 == 0 && xs256_chunked_rows(N) && shape.wg >= 512) {
        a.C = N / kXs256RowChunks;
        a.P = kXs256RowChunks;
    }
    // rows of whole 4 KiB multiples on the resident schedule: rotated tile order
    if (g != RNG_XS256 && staged && a.P == 1 && a.vec4 && S % 64 == 0 && N % 1024 == 0) {
        a.rot = 1;
        rot_constants(g, N, a);
    }
    rc = dispatch_generate(g, dt, a, (int)shape.wg, (int)shape.unroll, staged, st);
    if (rc != kStatesNotWritten) return check_launch(rc, "rng_generate");
    // chunks of one stream in several workgroups: the states advance after
    // every chunk has read them
    return check_launch(dispatch_skip(g, d_state, ld, S, N, tab, st), "rng_generate: state");
}

int check_gen(int g) { return gen_words(g) ? RNG_OK : fail(RNG_EINVAL, "unknown generator %d", g); }

int check_sizes(uint64_t S, uint64_t N, uint64_t words)
{
    uint64_t t;
    if (mul_overflows(S, N, &t) || mul_overflows(t, 4, &t))
        return fail(RNG_ERANGE, "n_streams * n * 4 overflows 64 bits");
    if (mul_overflows(S, words, &t) || mul_overflows(t, 4, &t))
        return fail(RNG_ERANGE, "state size overflows 64 bits");
    // keeps every grid below 2^31 workgroups (64-lane groups, <= 2^30 waves)
    if (S > ((uint64_t)1 << 36)) return fail(RNG_ERANGE, "n_streams above 2^36");
    return RNG_OK;
}

// Sequence splitting after the argument checks of the entry points: the
// workspace (ws_bytes available) holds a copy of the start state if the final
// state overlaps it.  Launches only.
int split_args_check(uint64_t total, uint64_t n_threads, const void *d_out, const uint32_t *d_state_one,
                     const uint32_t *d_final_state)
{
    if (!d_out) return fail(RNG_EINVAL, "NULL output");
    if (n_threads == 0) return fail(RNG_EINVAL, "n_threads is 0");
    if (((uintptr_t)d_out & 3) || ((uintptr_t)d_state_one & 3) || ((uintptr_t)d_final_state & 3))
        return fail(RNG_EINVAL, "misaligned pointer");
    return check_sizes(1, total, 1);
}

int split_run(int g, const uint32_t *d_state_one, uint64_t total, uint64_t n_threads, int t, void *d_out,
              uint32_t *d_final_state, uint32_t *ws, uint64_t ws_bytes, const DevTables &tab, hipStream_t st)
{
    uint64_t need;
    if (int rc = split_scratch_bytes(g, total, n_threads, &need)) return rc;
    if (ws_bytes < need)
        return fail(RNG_ENOMEM, "workspace %llu bytes < %llu", (unsigned long long)ws_bytes, (unsigned long long)need);
    return seq_run(g, d_state_one, total, t, d_out, d_final_state, ws, tab, st);
}

// Workspace bytes a split of `total` samples over n_threads threads uses:
// one state per thread with work.
int split_scratch_bytes(int g, uint64_t total, uint64_t n_threads, uint64_t *bytes)
{
    if (n_threads == 0) return fail(RNG_EINVAL, "n_threads is 0");
    const uint64_t C = (total + n_threads - 1) / n_threads;
    const uint64_t T = C ? (total + C - 1) / C : 0;
    if (mul_overflows(T, (uint64_t)gen_words(g) * 4, bytes)) return fail(RNG_ERANGE, "n_threads too large");
    return RNG_OK;
}

// Windows of the fused consumer: blocks as long as leave a window for each of
// 2048 waves and two for each stream (a start costs 3 to 8 us, a number of each
// lane about 25 ns, and the last window is part empty), none shorter than 64
// numbers; none at all for streams too short for lanes.  Of the lengths that do,
// the one with the fewest steps, a start counted as the 107 that it takes of a
// full device.  XS256 up to 8192 streams (us, chunks / windows: 1 x 4 10^6 195 /
// 20, 1000 x 10^4 227 / 29, 10^4 x 10^4 191 / 182, 2 10^4 x 5000 165 / 285), as
// long as the last windows' idle lanes and the starts cost less than a chunk's
// jump per lane, 170 us or 3 10^8 steps (7000 x 530637 2258 / 2882).
static void fused_windows(int g, uint64_t S, uint64_t N, FusedArgs &a)
{
    // a lane per stream is sooner done (us, lanes / windows: KISS 8 x 300 11.9 / 12.3;
    // XS256 300 x 300 12.7 / 16, 4096 x 850 31 / 34, 8192 x 1400 49 / 62, x 2000 69 / 59)
    if (N < (g == RNG_XS256 || g == RNG_KISS ? 320 : 256)) return;
    if (g == RNG_XS256 && N <= 4096 && 100 * N < 34000 + 16 * S) return;
    uint32_t lg = 12;
    while (lg > 6 && (S * ((N + ((uint64_t)64 << lg) - 1) >> (lg + 6)) < 2048 || ((uint64_t)128 << lg) > N)) --lg;
    auto steps = [&](uint32_t l) { return ((N + ((uint64_t)64 << l) - 1) >> (l + 6)) * 64 * (((uint64_t)1 << l) + 107); };
    for (uint32_t l = lg; l >= 6; --l)
        if (steps(l) < steps(lg)) lg = l;
    if (g == RNG_XS256 && S >= 64 && S * (steps(lg) - N) > 300000000) return;
    const uint64_t nwin = (N + ((uint64_t)64 << lg) - 1) >> (lg + 6);
    uint64_t p = 4096 / S ? 4096 / S : 1;
    if (p > nwin) p = nwin;
    a.windows = 1;
    a.lgc = lg;
    a.P = (uint32_t)p;
}

}  // namespace rngx

using namespace rngx;

// ====================================================================== ABI
extern "C" {

const char *rng_strerror(int code)
{
    switch (code) {
    case RNG_OK: return "success";
    case RNG_EINVAL: return "invalid argument";
    case RNG_ERANGE: return "size out of range";
    case RNG_ENOMEM: return "insufficient memory or workspace";
    case RNG_EHIP: return "HIP runtime error";
    case RNG_ENODEV: return "no usable gfx950 device";
    case RNG_EAGAIN: return "not ready";
    }
    return "unknown error";
}

const char *rng_last_error(void) { return g_last_error.c_str(); }

int rng_init(void)
{
    DevTables t;
    if (int rc = device_tables(&t)) return rc;
    return scratch_init_current_device();
}

int rng_shutdown(void) { return shutdown_tables(); }

int rng_state_words(int g, uint32_t *words)
{
    if (check_gen(g)) return RNG_EINVAL;
    if (!words) return fail(RNG_EINVAL, "words is NULL");
    *words = (uint32_t)gen_words(g);
    return RNG_OK;
}

int rng_mwc32_multiplier(uint32_t *a)
{
    if (!a) return fail(RNG_EINVAL, "a is NULL");
    *a = mwc32_multiplier();
    return RNG_OK;
}

int rng_mwc16_multipliers(uint16_t *h_out, uint32_t cap, uint32_t *count)
{
    if (!count) return fail(RNG_EINVAL, "count is NULL");
    const auto &t = mwc16_multipliers();
    *count = (uint32_t)t.size();
    if (h_out) {
        if (cap < t.size()) return fail(RNG_ERANGE, "cap %u < %zu", cap, t.size());
        std::memcpy(h_out, t.data(), t.size() * sizeof(uint16_t));
    }
    return RNG_OK;
}

int rng_seed(int g, uint64_t seed, uint64_t first_stream, uint64_t n_streams, uint32_t *d_state,
             void *stream)
{
    if (check_gen(g)) return RNG_EINVAL;
    if (n_streams == 0) return RNG_OK;
    if (!d_state) return fail(RNG_EINVAL, "d_state is NULL");
    if ((uintptr_t)d_state & 3) return fail(RNG_EINVAL, "d_state not 4-byte aligned");
    if (int rc = check_sizes(n_streams, 1, gen_words(g))) return rc;
    uint64_t end;
    if (__builtin_add_overflow(first_stream, n_streams, &end) ||
        mul_overflows(end, 4, &end))
        return fail(RNG_ERANGE, "first_stream + n_streams too large");
    DevTables tab;
    if (int rc = device_tables(&tab)) return rc;
    return check_launch(dispatch_seed(g, seed, first_stream, n_streams, d_state, tab, (hipStream_t)stream),
                        "rng_seed");
}

static int generate_checked(int g, uint32_t *d_state, uint64_t n_streams, uint64_t n, int t, void *d_out, Shape shape,
                            bool asked, void *stream)
{
    if (check_gen(g)) return RNG_EINVAL;
    if (t != RNG_U32 && t != RNG_F32) return fail(RNG_EINVAL, "unknown dtype %d", t);
    if (!valid_shape(shape.wg, shape.unroll))
        return fail(RNG_EINVAL, "launch shape wg=%u unroll=%u", shape.wg, shape.unroll);
    if (n_streams == 0 || n == 0) return RNG_OK;
    if (!d_state || !d_out) return fail(RNG_EINVAL, "NULL state or output");
    if (((uintptr_t)d_state & 3) || ((uintptr_t)d_out & 3))
        return fail(RNG_EINVAL, "state and output must be 4-byte aligned");
    if (int rc = check_sizes(n_streams, n, gen_words(g))) return rc;
    return generate_impl(g, t, d_state, n_streams, n_streams, n, d_out, shape, asked, true, (hipStream_t)stream);
}

int rng_generate_ex(int g, uint32_t *d_state, uint64_t n_streams, uint64_t n, int t, void *d_out,
                    uint32_t wg, uint32_t unroll, void *stream)
{
    return generate_checked(g, d_state, n_streams, n, t, d_out, Shape{wg, unroll}, true, stream);
}

int rng_generate(int g, uint32_t *d_state, uint64_t n_streams, uint64_t n, int t, void *d_out, void *stream)
{
    if (check_gen(g)) return RNG_EINVAL;
    if (t != RNG_U32 && t != RNG_F32) return fail(RNG_EINVAL, "unknown dtype %d", t);
    return generate_checked(g, d_state, n_streams, n, t, d_out, row_shape(g, t, n_streams, n), false, stream);
}

int rng_skip(int g, uint32_t *d_state, uint64_t n_streams, uint64_t k, void *stream)
{
    if (check_gen(g)) return RNG_EINVAL;
    if (n_streams == 0 || k == 0) return RNG_OK;
    if (!d_state) return fail(RNG_EINVAL, "d_state is NULL");
    if ((uintptr_t)d_state & 3) return fail(RNG_EINVAL, "d_state not 4-byte aligned");
    if (int rc = check_sizes(n_streams, 1, gen_words(g))) return rc;
    DevTables tab;
    if (int rc = device_tables(&tab)) return rc;
    return check_launch(dispatch_skip(g, d_state, n_streams, n_streams, k, tab, (hipStream_t)stream), "rng_skip");
}

int rng_split_workspace_bytes(int g, uint64_t n_threads, uint64_t *bytes)
{
    if (check_gen(g)) return RNG_EINVAL;
    if (!bytes) return fail(RNG_EINVAL, "bytes is NULL");
    uint64_t b;
    if (mul_overflows(n_threads, (uint64_t)gen_words(g) * 4, &b)) return fail(RNG_ERANGE, "n_threads too large");
    *bytes = b;
    return RNG_OK;
}

int rng_generate_split(int g, const uint32_t *d_state_one, uint64_t total, uint64_t n_threads, int t,
                       void *d_out, uint32_t *d_final_state, void *d_workspace, uint64_t workspace_bytes,
                       void *stream)
{
    if (check_gen(g)) return RNG_EINVAL;
    if (t != RNG_U32 && t != RNG_F32) return fail(RNG_EINVAL, "unknown dtype %d", t);
    if (!d_state_one || !d_final_state) return fail(RNG_EINVAL, "NULL state");
    if (total == 0) {
        // nothing generated: the final state is the initial one
        if (d_final_state == d_state_one) return RNG_OK;
        hipError_t e = hipMemcpyAsync(d_final_state, d_state_one, gen_words(g) * 4, hipMemcpyDeviceToDevice,
                                      (hipStream_t)stream);
        return e == hipSuccess ? RNG_OK : hip_fail(e, "hipMemcpyAsync");
    }
    if (int rc = split_args_check(total, n_threads, d_out, d_state_one, d_final_state)) return rc;
    if (!d_workspace) return fail(RNG_EINVAL, "NULL workspace");
    if ((uintptr_t)d_workspace & 255) return fail(RNG_EINVAL, "misaligned pointer");
    uint64_t need;
    if (int rc = split_scratch_bytes(g, total, n_threads, &need)) return rc;
    if (workspace_bytes < need)
        return fail(RNG_ENOMEM, "workspace %llu bytes < %llu", (unsigned long long)workspace_bytes,
                    (unsigned long long)need);
    DevTables tab;
    if (int rc = device_tables(&tab)) return rc;
    return split_run(g, d_state_one, total, n_threads, t, d_out, d_final_state, (uint32_t *)d_workspace,
                     workspace_bytes, tab, (hipStream_t)stream);
}

int rng_fused_pi(int g, uint32_t *d_state, uint64_t n_streams, uint64_t n, uint64_t *d_count, void *stream)
{
    if (check_gen(g)) return RNG_EINVAL;
    if (n_streams == 0 || n == 0) return RNG_OK;
    if (!d_state || !d_count) return fail(RNG_EINVAL, "NULL state or count");
    if (((uintptr_t)d_state & 3) || ((uintptr_t)d_count & 7)) return fail(RNG_EINVAL, "misaligned pointer");
    if (int rc = check_sizes(n_streams, n, gen_words(g))) return rc;
    DevTables tab;
    if (int rc = device_tables(&tab)) return rc;
    FusedArgs a{};
    a.state = d_state;
    a.ld = n_streams;
    a.S = n_streams;
    a.N = n;
    a.count = d_count;
    a.tab = tab;
    choose_chunks(g, n_streams, n, 8, &a.C, &a.P, (uint64_t)1 << 17);
    if (n_streams < 64 || (g == RNG_XS256 && n_streams <= 8192)) fused_windows(g, n_streams, n, a);
    if (!a.windows && a.P == 1) a.C = n;
    if (int rc = check_launch(dispatch_fused(g, a, (hipStream_t)stream), "rng_fused_pi")) return rc;
    if (!a.windows && a.P == 1) return RNG_OK;
    return check_launch(dispatch_skip(g, d_state, n_streams, n_streams, n, tab, (hipStream_t)stream),
                        "rng_fused_pi: state");
}

}  // extern "C"
