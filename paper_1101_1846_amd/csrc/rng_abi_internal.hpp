// rng_abi_internal.hpp -- helpers shared by the C ABI translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rng.h"
#include "rng_internal.hpp"

namespace rngx {

struct Shape {
    uint32_t wg, unroll;
};

int fail(int code, const char *fmt, ...);
int hip_fail(hipError_t e, const char *what);
int check_launch(int rc, const char *what);
int check_gen(int g);
int check_sizes(uint64_t S, uint64_t N, uint64_t words);
int device_tables(DevTables *out);
int gen_words(int g);
bool valid_shape(uint32_t wg, uint32_t unroll);
uint32_t run_rows(uint64_t S, uint64_t N);
Shape tuned_shape(int g, int dt, bool runs);
Shape row_shape(int g, int dt, uint64_t S, uint64_t n);
void set_tuned_shape(int g, int dt, bool runs, Shape s);
bool shape_matters(int g, uint64_t S, uint64_t N, const void *out);
// Chunks per stream: the largest power of two p with S p <= target_lanes and
// chunks of at least the generator's minimum length.
void choose_chunks(int g, uint64_t S, uint64_t N, uint64_t align, uint64_t *C, uint32_t *P, uint64_t target_lanes);
// Chunks for one lane per chunk (fewer streams than a wave has lanes).
void lane_chunks(int g, uint64_t S, uint64_t N, uint64_t *C, uint32_t *P);
int generate_impl(int g, int dt, uint32_t *d_state, uint64_t ld, uint64_t S, uint64_t N, void *d_out,
                  Shape shape, bool asked, bool staged, hipStream_t st);
int dispatch_generate(int g, int dt, const GenArgs &a, int wg, int unroll, bool staged, hipStream_t st);
int dispatch_skip(int g, uint32_t *st, uint64_t ld, uint64_t S, uint64_t k, const DevTables &tab, hipStream_t s);
int dispatch_state_copy(int g, const uint32_t *src, uint64_t ss, uint64_t si, uint32_t *dst, uint64_t ds,
                        uint64_t di, hipStream_t s);

// Fewer streams than a wave has lanes: lane v takes chunk v mod P of stream
// v / P (chunks of C samples), then the states advance by N (few.hip).
int generate_few(int g, int dt, uint32_t *d_state, uint64_t ld, uint64_t S, uint64_t N, uint64_t C, uint64_t P,
                 void *d_out, const DevTables &tab, hipStream_t st);

// Long sequences of few streams without start states in memory (seq.hip, and
// seq_xs256.hip for XS256): S streams of N numbers from states at word stride
// ld into out [S][N].  With S = 1 the state after the last number goes to
// final_state if that is not null (it must not overlap the start state); the
// start states are not written.
constexpr uint64_t kSeqWaves = 1024;  // 4 per CU
int launch_seq(int g, int dt, const uint32_t *state, uint64_t ld, uint64_t S, uint64_t N, void *out,
               uint32_t *final_state, const DevTables &tab, hipStream_t st);
int launch_seq_xs256(int dt, const uint32_t *state, uint64_t ld, uint64_t S, uint64_t N, void *out,
                     uint32_t *final_state, const DevTables &tab, hipStream_t st);
// One sequence of `total` numbers through launch_seq; start and final states may lie
// anywhere: those that overlap each other or the output go through ws (one state).
int seq_run(int g, const uint32_t *state_one, uint64_t total, int t, void *out, uint32_t *final_state, uint32_t *ws,
            const DevTables &tab, hipStream_t st);

// Rows of any length (32 <= N < 2^24), count and alignment, one per lane, or
// 2^lgp chunks of C numbers per stream, one per lane (rows.hip; row_chunks gives
// them, false if there is none to gain).  The states are rewritten.
constexpr uint64_t kRowMin = 32, kRowMax = ((uint64_t)1 << 24) - 1;
bool row_chunks(int g, uint64_t S, uint64_t N, uint32_t *lgp, uint32_t *C);
int launch_rows(int g, int dt, uint32_t *state, uint64_t ld, uint64_t S, uint64_t N, uint32_t lgp, uint32_t C, void *out,
                const DevTables &tab, hipStream_t st);

// Tables of the current device only if they exist already (never allocates).
int device_tables_if_ready(DevTables *out);
// Looks up, once per device, the address of the allocation-free entry
// point's scratch array on the current device (called by rng_init).
int scratch_init_current_device();
// Sequence splitting: argument checks, the workspace that a caller has to bring (a
// state per thread; one is used), and the launches themselves (seq_run).
int split_args_check(uint64_t total, uint64_t n_threads, const void *d_out, const uint32_t *d_state_one,
                     const uint32_t *d_final_state);
int split_scratch_bytes(int g, uint64_t total, uint64_t n_threads, uint64_t *bytes);
int split_run(int g, const uint32_t *d_state_one, uint64_t total, uint64_t n_threads, int t, void *d_out,
              uint32_t *d_final_state, uint32_t *ws, uint64_t ws_bytes, const DevTables &tab, hipStream_t st);

// rng_batch_set without the check that no two requests share a state (for
// callers that keep one request per state).
int batch_set_distinct(rng_batch_t *h, const rng_request_t *reqs, uint32_t n);
}  // namespace rngx
