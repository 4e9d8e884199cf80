// rng_batch.cpp -- the batched path of the C ABI: plans a batch of
// independent requests (row lengths, grouping by generator and dtype), ships
// the plan through pinned host memory or in the first kernel's arguments, and
// launches two kernels, directly or as one captured HIP graph per shape: root
// (start states, tile map, tile counter) and persistent generation.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "rng.h"
#include "rng_abi_internal.hpp"
#include "rng_batch_internal.hpp"

namespace rngx {
int launch_batch_root(const BatchArgs &a, const PlanInline &pin, uint32_t requests, uint32_t moves, hipStream_t s);
int launch_batch_gen(const BatchArgs &a, int wg, int unroll, unsigned grid, hipStream_t s);
int batch_gen_occupancy(int wg, int unroll, int *blocks_per_cu);
}  // namespace rngx

using namespace rngx;

struct rng_batch {
    std::mutex mu;
    int device = 0;
    uint32_t max_requests = 0;
    uint64_t max_samples = 0;
    uint64_t C = 1024;
    bool chunk_auto = false;  // C chosen per plan (RNG_BATCH_CHUNK_AUTO)
    uint32_t wg = 256, unroll = 8;
    bool wg_asked = false;  // wg is the caller's (or the tuner's) choice
    uint64_t map_cap = 0;  // tiles the map holds
    char *d_plan = nullptr, *h_plan = nullptr;  // packed plan (BatchHeader first), device and pinned staging
    uint32_t *d_ws = nullptr, *d_counter = nullptr, *d_map = nullptr;
    hipEvent_t copied = nullptr;
    hipStream_t capture = nullptr;  // private stream the graphs are recorded on
    bool copy_pending = false;
    bool planned = false;
    struct Graph {
        uint32_t wg, unroll;
        hipGraph_t graph;
        hipGraphExec_t exec;
    };
    std::vector<Graph> graphs;
    bool use_graph = false;               // replay a captured graph instead of launching directly
    uint32_t occ_wg = 0, occ_unroll = 0;  // shape of the cached occupancy
    unsigned gen_full = 0;                // generation workgroups resident at once for that shape
    int num_cu = 256;
    uint32_t moves = 0;               // requests of the plan whose state the root kernel moves
    std::vector<rng_request_t> last;  // last planned table, re-planned on a chunk change
    std::vector<uint16_t> codes;      // [max_requests] group and row bits, while a plan is made
    BatchHeader &hdr() { return *(BatchHeader *)h_plan; }
};

// Rows are at most as long as the chunk length allows, the power of two at most
// C (in automatic mode 4096); a request of up to 64 rows takes the shortest that
// fit it in one tile.
static uint64_t longest_row(const rng_batch *h)
{
    uint64_t c = (uint64_t)1 << kBatchLgMax;
    while (!h->chunk_auto && c > h->C) c /= 2;
    return c;
}

// log2 of the row length of a batch of n requests, `total` samples, by what it
// costs, in ns: a tile's start 16000, a sample of each row 94 with all waves
// writing (5.6 TB/s over 2048), 70 in the last tiles, which run out alone.
// (16 requests, 10^6 samples: rows of 32, 19 us against 70 with rows of 1024;
// 100, 10^7: 36 with 128, 80 with 32; 890, 8.4 10^7: 108 with 512, 132 with
// 1024, 162 with 128; from about 3 10^8 samples on the longest.)
static uint32_t row_bits(uint64_t n, uint64_t total, uint32_t longest)
{
    uint32_t best = longest;
    double least = 1e300;
    for (uint32_t lg = longest; lg >= (uint32_t)kBatchLgMin; --lg) {
        const double tiles = (double)n + (double)(total >> (lg + 6));
        const double t = (tiles * 16000 + (double)(total >> 6) * 94) / 2048 + 16000 + 70.0 * (double)(1u << lg);
        if (t < least) {
            least = t;
            best = lg;
        }
    }
    return best;
}

// Tiles of any plan: rows below the longest are chosen only while they make
// fewer than 18 tiles per sample of a row, 18 2^11, beside one per request.
static uint64_t tile_capacity(const rng_batch *h)
{
    const uint64_t per = 64 * longest_row(h);
    return std::max((h->max_samples + per - 1) / per, (uint64_t)1 << 16) + h->max_requests;
}

static uint64_t align16(uint64_t x) { return (x + 15) & ~(uint64_t)15; }

// Packed plan: header, requests (16-byte aligned each).
static uint64_t plan_capacity(const rng_batch *h)
{
    return align16(sizeof(BatchHeader)) + align16(sizeof(BatchReq) * (uint64_t)h->max_requests);
}

// Sizes the tile map, and at first the plan and the start states.  Growing the
// map drops the captured graphs, which hold the old address.
static int alloc_ws(rng_batch *h)
{
    const uint64_t tiles = tile_capacity(h), plan_bytes = plan_capacity(h);
    if (plan_bytes >= ((uint64_t)1 << 32)) return fail(RNG_ENOMEM, "batch plan above 4 GiB");
    if (tiles >= ((uint64_t)1 << 32) || (!h->chunk_auto && h->max_samples / h->C >= ((uint64_t)1 << 32)))
        return fail(RNG_ENOMEM, "more than 2^32 chunks of %llu samples", (unsigned long long)h->C);
    if (tiles <= h->map_cap) return RNG_OK;
    for (auto &g : h->graphs) {
        (void)hipGraphExecDestroy(g.exec);
        (void)hipGraphDestroy(g.graph);
    }
    h->graphs.clear();
    (void)hipDeviceSynchronize();  // no launch may still use the old buffers
    if (h->d_map) (void)hipFree(h->d_map);
    h->d_map = nullptr;
    h->map_cap = 0;
    h->planned = false;
    hipError_t e;
    if (!h->d_ws && (e = hipMalloc((void **)&h->d_ws, (uint64_t)h->max_requests * 32)) != hipSuccess)
        return hip_fail(e, "hipMalloc(batch states)");
    if (!h->d_plan && (e = hipMalloc((void **)&h->d_plan, plan_bytes)) != hipSuccess)
        return hip_fail(e, "hipMalloc(batch plan)");
    if (!h->h_plan) {
        if ((e = hipHostMalloc((void **)&h->h_plan, plan_bytes, hipHostMallocDefault)) != hipSuccess)
            return hip_fail(e, "hipHostMalloc(batch plan)");
        std::memset(h->h_plan, 0, sizeof(BatchHeader));
    }
    if ((e = hipMalloc((void **)&h->d_map, tiles * 4)) != hipSuccess) return hip_fail(e, "hipMalloc(tile map)");
    h->map_cap = tiles;
    return RNG_OK;
}

static void free_batch(rng_batch *h)
{
    for (auto &g : h->graphs) {
        (void)hipGraphExecDestroy(g.exec);
        (void)hipGraphDestroy(g.graph);
    }
    if (h->copied) (void)hipEventDestroy(h->copied);
    if (h->capture) (void)hipStreamDestroy(h->capture);
    if (h->d_plan) (void)hipFree(h->d_plan);
    if (h->d_map) (void)hipFree(h->d_map);
    if (h->d_ws) (void)hipFree(h->d_ws);
    if (h->d_counter) (void)hipFree(h->d_counter);
    if (h->h_plan) (void)hipHostFree(h->h_plan);
    delete h;
}

static bool shape_ok(uint32_t wg, uint32_t unroll)
{
    int b = 0;
    return batch_gen_occupancy((int)wg, (int)unroll, &b) == 0;
}

static BatchArgs make_args(rng_batch *h, const DevTables &tab)
{
    BatchArgs a{};
    a.hdr = (const BatchHeader *)h->d_plan;
    a.tile_req = h->d_map;
    a.ws = h->d_ws;
    a.counter = h->d_counter;
    a.tab = tab;
    return a;
}

static int plan(rng_batch_t *h, const rng_request_t *reqs, uint32_t n);

extern "C" {

int rng_batch_create(uint32_t max_requests, uint64_t max_samples, rng_batch_t **out)
{
    if (!out) return fail(RNG_EINVAL, "NULL handle pointer");
    if (max_requests == 0) return fail(RNG_EINVAL, "max_requests is 0");
    if (max_samples > ((uint64_t)1 << 40)) return fail(RNG_ERANGE, "max_samples above 2^40");
    DevTables tab;
    if (int rc = device_tables(&tab)) return rc;
    auto *h = new rng_batch();
    h->max_requests = max_requests;
    h->max_samples = max_samples;
    (void)hipGetDevice(&h->device);
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, h->device) == hipSuccess) h->num_cu = prop.multiProcessorCount;
    hipError_t e = hipSuccess;
    int rc = RNG_OK;
    if ((e = hipMalloc((void **)&h->d_counter, kBatchCounterWords << (kBatchLgCounters + 2))) != hipSuccess ||
        (e = hipEventCreateWithFlags(&h->copied, hipEventDisableTiming)) != hipSuccess ||
        (e = hipStreamCreateWithFlags(&h->capture, hipStreamNonBlocking)) != hipSuccess)
        rc = hip_fail(e, "rng_batch_create");
    if (!rc) rc = alloc_ws(h);
    if (!rc) {
        try {
            h->codes.resize(max_requests);
        } catch (const std::bad_alloc &) {
            rc = fail(RNG_ENOMEM, "no host memory for %u requests", max_requests);
        }
    }
    if (rc) {
        free_batch(h);
        return rc;
    }
    *out = h;
    return RNG_OK;
}

int rng_batch_destroy(rng_batch_t *h)
{
    if (!h) return RNG_OK;
    {
        std::lock_guard<std::mutex> lk(h->mu);
        if (h->copy_pending) (void)hipEventSynchronize(h->copied);
    }
    free_batch(h);
    return RNG_OK;
}

int rng_batch_set_shape(rng_batch_t *h, uint32_t wg, uint32_t unroll, uint32_t chunk)
{
    if (!h) return fail(RNG_EINVAL, "NULL handle");
    std::lock_guard<std::mutex> lk(h->mu);
    uint32_t w = wg ? wg : h->wg, u = unroll ? unroll : h->unroll;
    if (!shape_ok(w, u)) return fail(RNG_EINVAL, "batch launch shape wg=%u unroll=%u not available", w, u);
    if (chunk) {
        const bool autoc = chunk == RNG_BATCH_CHUNK_AUTO;
        if (!autoc && chunk % kBatchTile)
            return fail(RNG_EINVAL, "chunk %u is not a multiple of %d", chunk, kBatchTile);
        if (h->copy_pending) (void)hipEventSynchronize(h->copied);
        const uint64_t old_c = h->C;
        const bool old_auto = h->chunk_auto;
        h->chunk_auto = autoc;
        if (!autoc) h->C = chunk;
        if (int rc = alloc_ws(h)) {
            h->C = old_c;
            h->chunk_auto = old_auto;
            return rc;
        }
        h->planned = false;  // the plan depends on the chunk length
        if (!h->last.empty()) {
            std::vector<rng_request_t> t = h->last;
            if (int rc = plan(h, t.data(), (uint32_t)t.size())) return rc;
        }
    }
    h->wg = w;
    h->unroll = u;
    if (wg) h->wg_asked = true;
    return RNG_OK;
}

int rng_batch_set_graph(rng_batch_t *h, int use_graph)
{
    if (!h) return fail(RNG_EINVAL, "NULL handle");
    if (use_graph != 0 && use_graph != 1) return fail(RNG_EINVAL, "use_graph must be 0 or 1");
    std::lock_guard<std::mutex> lk(h->mu);
    h->use_graph = use_graph == 1;
    return RNG_OK;
}

int rng_batch_get_shape(rng_batch_t *h, uint32_t *wg, uint32_t *unroll, uint32_t *chunk)
{
    if (!h || !wg || !unroll || !chunk) return fail(RNG_EINVAL, "NULL argument");
    std::lock_guard<std::mutex> lk(h->mu);
    *wg = h->wg;
    *unroll = h->unroll;
    *chunk = h->chunk_auto ? RNG_BATCH_CHUNK_AUTO : (uint32_t)h->C;
    return RNG_OK;
}

int rng_batch_set(rng_batch_t *h, const rng_request_t *reqs, uint32_t n)
{
    if (!h) return fail(RNG_EINVAL, "NULL handle");
    if (n && !reqs) return fail(RNG_EINVAL, "NULL request table");
    if (n > h->max_requests) return fail(RNG_ENOMEM, "%u requests > capacity %u", n, h->max_requests);
    if (n > 1) {
        // two requests on one state would race on its write-back: an open
        // hash table of at least twice the pointers (null ones fail the plan)
        uint32_t bits = 4;
        while (((uint64_t)1 << bits) < 2 * (uint64_t)n) ++bits;
        std::vector<uintptr_t> seen((uint64_t)1 << bits, 0);
        const uint64_t mask = seen.size() - 1;
        for (uint32_t i = 0; i < n; ++i) {
            const uintptr_t p = (uintptr_t)reqs[i].d_state;
            uint64_t at = (p * 0x9E3779B97F4A7C15ull) >> (64 - bits);
            while (seen[at] && seen[at] != p) at = (at + 1) & mask;
            if (p && seen[at] == p) return fail(RNG_EINVAL, "two requests share one d_state");
            seen[at] = p;
        }
    }
    return batch_set_distinct(h, reqs, n);
}

}  // extern "C"

// rng_batch_set for callers that already keep one request per state (the
// server's batches).
int rngx::batch_set_distinct(rng_batch_t *h, const rng_request_t *reqs, uint32_t n)
{
    if (!h) return fail(RNG_EINVAL, "NULL handle");
    if (n && !reqs) return fail(RNG_EINVAL, "NULL request table");
    std::lock_guard<std::mutex> lk(h->mu);
    int rc = plan(h, reqs, n);
    if (rc == RNG_OK) h->last.assign(reqs, reqs + n);
    return rc;
}

extern "C" {

// Lengths from which on each generator's requests keep a tile of their own, from the
// counts of those up to kBatchPackMax by generator and length: the shared tiles take
// as long as their longest request, a step in common each, the others the sum of their
// starts, both at once, so the limits lie where the two meet.  Times in 0.1 ns, measured
// on 2500 to 100000 requests of 16 to 4000 samples; a step takes longer the more shared
// tiles there are.
constexpr uint32_t kPackBin = 64, kPackBins = kBatchPackMax / kPackBin;
static void packed_lengths(const uint32_t (&count)[6][kPackBins], uint64_t (&packs)[6])
{
    static const uint64_t kOwnTile[6] = {0, 17, 62, 27, 38, 24}, kStep[6] = {1, 540, 740, 630, 700, 550};
    uint64_t upto[6][kPackBins + 1], shorts = 0, packed = 0;  // upto[g][b]: requests in the first b bins
    for (uint32_t g = 1; g < 6; ++g) {
        upto[g][0] = 0;
        for (uint32_t b = 0; b < kPackBins; ++b) upto[g][b + 1] = upto[g][b] + count[g][b];
        shorts += upto[g][kPackBins];
    }
    if (shorts < kBatchPackMin) return;
    for (uint64_t x = kPackBin * 540;; x += kPackBin * 540) {
        uint64_t own = 0, in = 0, least = kPackBins;
        for (uint32_t g = 1; g < 6; ++g) {
            const uint64_t bins = std::min<uint64_t>(x * 131072 / (kPackBin * kStep[g] * (131072 + packed)), kPackBins);
            packs[g] = bins * kPackBin;
            in += upto[g][bins];
            own += (upto[g][kPackBins] - upto[g][bins]) * kOwnTile[g];
            least = std::min(least, bins);
        }
        packed = in;
        if (own <= x || least == kPackBins) return;
    }
}

static int plan(rng_batch_t *h, const rng_request_t *reqs, uint32_t n)
{
    if (n > h->max_requests) return fail(RNG_ENOMEM, "%u requests > capacity %u", n, h->max_requests);
    uint64_t total_samples = 0;
    uint32_t short_of[6][kPackBins];
    const bool many = n >= kBatchPackMin;
    if (many) std::memset(short_of, 0, sizeof(short_of));
    for (uint32_t i = 0; i < n; ++i) {
        const rng_request_t &r = reqs[i];
        if (check_gen(r.gen)) return fail(RNG_EINVAL, "request %u: unknown generator %d", i, r.gen);
        if (r.dtype != RNG_U32 && r.dtype != RNG_F32) return fail(RNG_EINVAL, "request %u: dtype %d", i, r.dtype);
        if (!r.d_state || ((uintptr_t)r.d_state & 3)) return fail(RNG_EINVAL, "request %u: bad state pointer", i);
        if (r.state_stride == 0) return fail(RNG_EINVAL, "request %u: state_stride is 0", i);
        if (r.length && (!r.d_out || ((uintptr_t)r.d_out & 3))) return fail(RNG_EINVAL, "request %u: bad output", i);
        if (__builtin_add_overflow(total_samples, r.length, &total_samples))
            return fail(RNG_ERANGE, "total length overflows");
        if (many && r.length - 1 < kBatchPackMax) ++short_of[r.gen][(r.length - 1) / kPackBin];
    }
    if (total_samples > h->max_samples)
        return fail(RNG_ENOMEM, "batch of %llu samples > capacity %llu", (unsigned long long)total_samples,
                    (unsigned long long)h->max_samples);
    // The pinned staging buffers are about to be rewritten: wait for the
    // previous launch's copies to leave them.
    if (h->copy_pending) {
        hipError_t e = hipEventSynchronize(h->copied);
        if (e != hipSuccess) return hip_fail(e, "hipEventSynchronize");
        h->copy_pending = false;
    }
    h->planned = false;  // until this plan is complete: a failure below leaves nothing to launch
    const uint32_t longest = (uint32_t)__builtin_ctzll(longest_row(h)), cap = row_bits(n, total_samples, longest);
    uint64_t packs[6] = {0};
    if (many) packed_lengths(short_of, packs);
    // A request that one lane steps through sooner than the lanes' starts take stays
    // one row (16 requests, us, more rows / one: XS256 of 64 samples 14.3 / 9.5, of 100
    // 14.7 / 12.2, KISS of 64 11.6 / 9.3).
    static const uint64_t kOneRow[6] = {0, 32, 128, 32, 64, 32};
    auto tile_bits = [cap, longest](const rng_request_t &r) {
        const bool one = r.offset == 0 && r.length <= kOneRow[r.gen];
        const uint32_t bits = r.length > 1 ? 64 - (uint32_t)__builtin_clzll(r.length - 1) : 0;  // 2^bits >= length
        const uint32_t lg = std::max<uint32_t>(kBatchLgMin, one ? bits : bits < 6 ? 0 : bits - 6);
        return std::min(lg, one ? longest : cap);
    };
    auto tiles_of = [](uint64_t length, uint32_t lg) { return (length + ((uint64_t)64 << lg) - 1) >> (lg + 6); };
    // per request: key = 16 (a tile of its own) + 2 generator + dtype, and its row bits
    uint64_t tiles = 0;
    uint32_t moves = 0;
    uint32_t count[32] = {0}, group[32] = {0}, begin[32] = {0};
    for (uint32_t i = 0; i < n; ++i) {
        const rng_request_t &r = reqs[i];
        const bool packed = r.length - 1 < packs[r.gen];  // no empty one
        const uint32_t key = (packed ? 0 : 16) + (uint32_t)r.gen * 2 + (uint32_t)r.dtype;
        const uint32_t lg = packed ? kBatchPacked : tile_bits(r);
        h->codes[i] = (uint16_t)(key << 8 | lg);
        moves += r.offset && (packed || r.length == 0);
        ++count[key];
        tiles += packed ? 0 : tiles_of(r.length, lg);
    }
    for (uint32_t k = 0; k < 16; ++k) tiles += (count[k] + 63) / 64;
    if (tiles > h->map_cap)
        return fail(RNG_ENOMEM, "batch needs %llu tiles > %llu", (unsigned long long)tiles, (unsigned long long)h->map_cap);
    // requests by (generator, dtype), in table order within each; all that share tiles
    // come first, as these take longest
    BatchHeader &H = h->hdr();
    std::memset(&H, 0, sizeof(H));
    H.n = n;
    H.off_reqs = (uint32_t)align16(sizeof(BatchHeader));
    BatchReq *Q = plan_at<BatchReq>(&H, H.off_reqs);
    uint32_t at = 0;
    for (uint32_t k = 0; k < 32; ++k) {
        begin[k] = at;
        at += count[k];
    }
    for (uint32_t k = 0; k < 16; ++k)
        if (count[k] || count[16 + k]) {
            group[k] = group[16 + k] = H.ngroups;
            H.groups[H.ngroups++] = BatchGroup{k / 2, k % 2};
        }
    for (uint32_t i = 0; i < n; ++i) {
        const rng_request_t &r = reqs[i];
        const uint32_t k = h->codes[i] >> 8, lg = h->codes[i] & 255;
        Q[begin[k]++] = BatchReq{r.d_state, r.state_stride, r.offset, r.length, (uint32_t *)r.d_out,
                                 0, lg == kBatchPacked ? 0 : (uint32_t)tiles_of(r.length, lg), group[k], lg};
    }
    for (uint32_t k = 0; k < 16; ++k)  // begin[k] is their end now
        for (uint32_t i = 0; i < count[k]; i += 64) {
            BatchReq &first = Q[begin[k] - count[k] + i];
            first.ntiles = 1;
            first.lgc = kBatchPacked + std::min(count[k] - i, 64u) - 1;
        }
    uint32_t base = 0;
    for (uint32_t i = 0; i < n; ++i) {
        Q[i].tile_base = base;
        base += Q[i].ntiles;
    }
    H.n_tiles = base;
    h->moves = moves;
    // (every counter needs a wave: a grid that leaves tiles over has one per CU at least)
    H.lg_counters = total_samples < (uint64_t)base * 8192 && h->num_cu >= 1 << kBatchLgCounters ? kBatchLgCounters : 0;
    H.plan_bytes = (uint32_t)align16(H.off_reqs + sizeof(BatchReq) * (uint64_t)n);
    h->planned = true;
    return RNG_OK;
}

int rng_batch_launch(rng_batch_t *h, void *stream)
{
    if (!h) return fail(RNG_EINVAL, "NULL handle");
    std::lock_guard<std::mutex> lk(h->mu);
    if (!h->planned) return fail(RNG_EINVAL, "rng_batch_set has not been called since the last shape change");
    int dev = 0;
    (void)hipGetDevice(&dev);
    if (dev != h->device) return fail(RNG_EINVAL, "batch created on device %d, current device %d", h->device, dev);
    DevTables tab;
    if (int rc = device_tables(&tab)) return rc;
    hipStream_t st = (hipStream_t)stream;
    const BatchHeader &H = h->hdr();
    hipError_t e;
    // a small plan in the root kernel's arguments (direct launches), else the
    // whole plan in one copy
    static thread_local PlanInline pin;
    pin.bytes = 0;
    if (!h->use_graph && H.plan_bytes <= kInlinePlanBytes) {
        pin.bytes = H.plan_bytes;
        std::memcpy(pin.q, h->h_plan, H.plan_bytes);
    } else {
        if ((e = hipMemcpyAsync(h->d_plan, h->h_plan, H.plan_bytes, hipMemcpyHostToDevice, st)) != hipSuccess)
            return hip_fail(e, "rng_batch_launch: upload");
        if ((e = hipEventRecord(h->copied, st)) != hipSuccess) return hip_fail(e, "hipEventRecord");
        h->copy_pending = true;
    }

    if (h->occ_wg != h->wg || h->occ_unroll != h->unroll) {
        int per_cu = 0;
        if (batch_gen_occupancy((int)h->wg, (int)h->unroll, &per_cu) || per_cu <= 0) per_cu = 1;
        h->gen_full = (unsigned)(h->num_cu * per_cu);
        h->occ_wg = h->wg;
        h->occ_unroll = h->unroll;
    }
    const unsigned gen_grid = h->gen_full;
    if (!h->use_graph) {
        const BatchArgs a = make_args(h, tab);
        int rc = launch_batch_root(a, pin, H.n, h->moves, st);
        if (!rc && H.n_tiles) {
            // Up to a tile per CU goes out as workgroups of one wave, a CU each, if it
            // is long: four waves that share one slow each other down (16 XS256 requests
            // of 64 samples 15.3 us in workgroups of 256 lanes, 10.7 of 64, 100 of them
            // 22.4 and 16.8; no difference from 300 on; but 16 MWC32 requests of 1000
            // 7.7 and 8.5, and one XS256 request of two tiles 13.1 and 14.9).  So many
            // requests in so few tiles share them, which is long too.
            bool slow = H.n >= kBatchPackMin;
            for (uint32_t i = 0; i < H.ngroups; ++i) slow |= H.groups[i].gen == G_XS256 || H.groups[i].gen == G_KISS;
            const bool alone = !h->wg_asked && slow && H.n_tiles > h->wg / 64 && H.n_tiles <= (uint32_t)h->num_cu;
            const uint32_t wg = alone ? 64 : h->wg;
            const unsigned need = (unsigned)std::min<uint64_t>(gen_grid, (H.n_tiles + wg / 64 - 1) / (wg / 64));
            rc = launch_batch_gen(a, (int)wg, (int)h->unroll, need, st);
        }
        return check_launch(rc, "rng_batch_launch");
    }
    rng_batch::Graph *gp = nullptr;
    for (auto &g : h->graphs)
        if (g.wg == h->wg && g.unroll == h->unroll) gp = &g;
    if (!gp) {
        const BatchArgs a = make_args(h, tab);
        rng_batch::Graph g{h->wg, h->unroll, nullptr, nullptr};
        // Recorded on the handle's own stream (the caller's may be the null
        // stream, which cannot capture); nothing runs while recording.
        hipStream_t cs = h->capture;
        if ((e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal)) != hipSuccess)
            return hip_fail(e, "hipStreamBeginCapture");
        pin.bytes = 0;  // the graph's root kernel reads the uploaded plan
        int rc = launch_batch_root(a, pin, h->max_requests, 0, cs);
        if (!rc) rc = launch_batch_gen(a, (int)h->wg, (int)h->unroll, gen_grid, cs);
        e = hipStreamEndCapture(cs, &g.graph);
        if (rc) {
            if (g.graph) (void)hipGraphDestroy(g.graph);
            return check_launch(rc, "rng_batch_launch: capture");
        }
        if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture");
        if ((e = hipGraphInstantiate(&g.exec, g.graph, nullptr, nullptr, 0)) != hipSuccess) {
            (void)hipGraphDestroy(g.graph);
            return hip_fail(e, "hipGraphInstantiate");
        }
        h->graphs.push_back(g);
        gp = &h->graphs.back();
    }
    if ((e = hipGraphLaunch(gp->exec, st)) != hipSuccess) return hip_fail(e, "hipGraphLaunch");
    return RNG_OK;
}

int rng_batch_autotune(rng_batch_t *h, uint32_t reps, uint32_t *best_wg, uint32_t *best_unroll,
                       uint32_t *best_chunk, float *best_us, void *stream)
{
    if (!h || !best_wg || !best_unroll || !best_chunk) return fail(RNG_EINVAL, "NULL argument");
    if (reps == 0) return fail(RNG_EINVAL, "reps is 0");
    uint64_t n, total = 0;
    {
        std::lock_guard<std::mutex> lk(h->mu);
        if (h->last.empty()) return fail(RNG_EINVAL, "no planned batch to tune on");
        n = h->last.size();
        for (const rng_request_t &r : h->last) total += r.length;
    }
    // every built shape: workgroups of 64..1024 lanes x unroll 1..16 (the
    // paper chose its block size by occupancy and unrolled its main loop)
    static const uint32_t wgs[] = {64, 128, 256, 512, 1024}, unrolls[] = {1, 2, 4, 8, 16};
    uint32_t shapes[25][2];
    for (int i = 0; i < 25; ++i) {
        shapes[i][0] = wgs[i / 5];
        shapes[i][1] = unrolls[i % 5];
    }
    // Longest first, and none that plans the same rows as one before it: between
    // those, timing noise would store a limit for later, larger batches.
    static const uint32_t chunks[] = {4096, 2048, 1024, 512};
    uint32_t planned_bits = ~0u;
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t e0, e1;
    hipError_t e;
    if ((e = hipEventCreate(&e0)) != hipSuccess) return hip_fail(e, "hipEventCreate");
    if ((e = hipEventCreate(&e1)) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return hip_fail(e, "hipEventCreate");
    }
    float best = 1e30f;
    uint32_t bw = h->wg, bu = h->unroll, bc = (uint32_t)h->C;
    int rc = RNG_OK;
    for (uint32_t c : chunks) {
        const uint32_t bits = row_bits(n, total, (uint32_t)__builtin_ctz(c));
        if (bits == planned_bits) continue;
        planned_bits = bits;
        for (auto &sh : shapes) {
            if ((rc = rng_batch_set_shape(h, sh[0], sh[1], c))) break;
            if ((rc = rng_batch_launch(h, stream))) break;  // warm-up (and graph capture)
            (void)hipEventRecord(e0, st);
            for (uint32_t r = 0; r < reps && !rc; ++r) rc = rng_batch_launch(h, stream);
            (void)hipEventRecord(e1, st);
            if (rc) break;
            if ((e = hipEventSynchronize(e1)) != hipSuccess) {
                rc = hip_fail(e, "hipEventSynchronize");
                break;
            }
            float ms = 0;
            (void)hipEventElapsedTime(&ms, e0, e1);
            float us = ms * 1000.0f / reps;
            if (us < best) {
                best = us;
                bw = sh[0];
                bu = sh[1];
                bc = c;
            }
        }
        if (rc) break;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) return rc;
    if ((rc = rng_batch_set_shape(h, bw, bu, bc))) return rc;
    *best_wg = bw;
    *best_unroll = bu;
    *best_chunk = bc;
    if (best_us) *best_us = best;
    return RNG_OK;
}

}  // extern "C"
