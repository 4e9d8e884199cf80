// rng_batch_internal.hpp -- device-side layout of a batch of independent
// generation requests (shared by the host planner and the batch kernels).
//
// Every request is cut into tiles of 64 rows of 2^lgc consecutive samples, one
// row per lane of the wave that takes the tile, the last row and the last tile
// shorter.  The wave moves its lanes from the request's start state to their
// rows by itself (wave_starts.hpp), so no chunk states pass through memory.
// Requests are grouped by (generator, dtype) and their tiles numbered
// consecutively.  Of many short requests, up to 64 of a group share a tile instead,
// one per lane.
#pragma once
#include <stdint.h>

#include "rng_device.hpp"

namespace rngx {

constexpr int kBatchMaxGroups = 10;  // 5 generators x 2 dtypes
constexpr int kBatchTile = 64;       // LDS tile depth of the batch kernel
constexpr int kBatchLgMin = 5, kBatchLgMax = 12;  // rows of 32 to 4096 samples

// Tiles beyond the waves of the grid are pulled from 2^lg_counters counters, a
// 128-byte line each, of which wave w uses number w mod 2^lg_counters.  Atomics on
// one address follow each other in about 13 ns: tiles of fewer than 8192 samples
// end sooner than that over 2048 waves (10^4 requests of 16 samples: 155 us from one
// counter, 52 from 32).  Longer ones share one, which balances them best.
constexpr uint32_t kBatchLgCounters = 5, kBatchCounterWords = 32;

// kBatchPacked + c - 1 in lgc: the first of c requests that share one tile (the
// others have none), a request per lane.  From kBatchPackMin requests of at most
// kBatchPackMax samples on, about as many as the device holds waves: a tile of its
// own costs each some 9 us of a wave, 8 more for XS256, a step in common 54 to 74 ns
// (10^4 requests, us of the launch, own tiles / shared: XS256 x 100 74 / 13, x 320 77
// / 30, x 700 80 / 62, KISS x 320 49 / 29, XS32 x 256 35 / 21, MWC32 x 256 23.5 / 18.9,
// x 320 23.5 / 23.5; 30000: XS256 x 1000 211 / 90).
constexpr uint32_t kBatchPacked = 64, kBatchPackMin = 2048, kBatchPackMax = 4096;

struct BatchReq {
    uint32_t *state;     // word 0 of the stream's state
    uint64_t stride;     // word stride of that state
    uint64_t offset;     // samples skipped before the first output
    uint64_t length;     // samples produced
    uint32_t *out;       // [length]
    uint32_t tile_base;  // its first tile
    uint32_t ntiles;     // ceil(length / 64 2^lgc)
    uint32_t group;
    uint32_t lgc;        // log2 of the row length, or kBatchPacked and more
};

// Requests whose start state the root kernel moves by the offset, so that the
// tiles count from there: a slice that ends beyond position 2^64 of its stream (a
// tile's position, the offset and the samples before the tile, would not fit 64
// bits), and one that shares its tile.
__device__ __forceinline__ bool batch_moved(const BatchReq &q)
{
    return q.offset + q.length < q.offset || (q.lgc >= kBatchPacked && q.offset);
}

struct BatchGroup {
    uint32_t gen, dtype;
};

// Heads the packed plan that one copy uploads: the header, then the requests,
// sorted by group, at byte off_reqs.
struct BatchHeader {
    uint32_t n;  // requests
    uint32_t ngroups;
    uint32_t n_tiles;
    uint32_t off_reqs;
    uint32_t plan_bytes;
    uint32_t lg_counters;
    uint32_t pad[2];
    BatchGroup groups[kBatchMaxGroups];
};

// Plans of at most kInlinePlanBytes travel in the root kernel's arguments
// instead of an upload (direct launches only: a captured graph keeps the
// arguments it was recorded with).  The root kernel reads the plan there, and
// its first workgroup writes it to the device plan buffer for the generation
// kernel.  This saves the copy and the wait for it.
constexpr uint32_t kInlinePlanBytes = 2048;

struct PlanInline {
    uint32_t bytes;  // 0: the plan was uploaded to BatchArgs::hdr
    uint32_t pad[3];
    uint4 q[kInlinePlanBytes / 16];
};

struct BatchArgs {
    const BatchHeader *hdr;  // the packed plan
    uint32_t *tile_req;      // [n_tiles] request of every tile
    uint32_t *ws;            // [n][8] start states of the requests
    uint32_t *counter;       // tile counters of the persistent kernel
    DevTables tab;
};

template <class T>
__host__ __device__ inline T *plan_at(const BatchHeader *p, uint32_t off)
{
    return (T *)((const char *)p + off);
}

}  // namespace rngx
