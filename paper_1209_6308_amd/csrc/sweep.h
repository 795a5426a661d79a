// The triangle-listing form of the census sweep (sweep.hip). Internal; not
// part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "triad_internal.h"

namespace triad {

// Device counters of one sweep (64-bit words, zeroed by its first kernel):
// acc[0..15] the 16 classes as signed sums (triangle classes exact, the open
// and dyadic classes before the triangles' share is taken out; see sums.h), then
constexpr int SW_ABOVE = 17;  // entries above their row's own id
constexpr int SW_WORDS = 32;
constexpr int SW_COPIES = 64;
// labelled: the 64 states, then the entries above
constexpr int SW_LAB_ABOVE = 64, SW_LAB_WORDS = 80;
// err[0]: raised by the row checks, err[1]: by the entry checks, err[2]: by the
// symmetry check and k_sw_pack
constexpr int SW_ERRS = 4;

constexpr int SW_CLK = 66, SW_STATUS = SW_CLK + 5;

struct SweepIn {
  int64_t n, nnz;
  const int64_t* off;
  const int32_t* nbr;
  const uint8_t* flg;
};

// Enqueues the whole sweep of one graph on s: validation, orientation,
// triangle counts and per-row sums. *acc (SW_COPIES copies of SW_WORDS words, to be summed; labelled: SW_LAB_WORDS) and *err (SW_ERRS
// words) are its counters, in scratch memory. validate: also check symmetry.
// status (device, SW_STATUS words): from word SW_CLK on, the device clock at
// the start, after the orientation, after the sorting and listing, after the
// counting, at the end (a stage that did not run leaves its word).
int sweep_census(const SweepIn& in, bool validate, bool labelled, unsigned long long** acc, uint32_t** err, Scratch& scratch,
                 uint64_t* status, hipStream_t s);
// Labelled: the 64 states (n below SW_LAB_MAX_N).
constexpr int64_t SW_LAB_MAX_N = (int64_t)1 << 29;
// The 16 counts and the high word of 003 (labelled: 64 states and the high word
// of state 0) into d_out unless an error is set; status gets the same words and
// then the error bits.
void sweep_finish(const unsigned long long* acc, uint32_t* err, bool labelled, int64_t nnz, int64_t n, uint64_t* d_out,
                  uint64_t* status, hipStream_t s);

// A batch (the concatenated CSR of in, nv rows, the largest member nmax
// vertices): enqueues the whole batched census; d_out [graphs][16] is written
// unless an error is found, *err (one word, in scratch memory) has its bits
// afterwards. Its scratch is sweep_batch_bytes from an arena. Launch shape:
// wavefronts per workgroup (1, 2, 4), workgroups, entries per wavefront and
// turn (a multiple of 64; 0: chosen here). Capturable.
size_t sweep_batch_bytes(int32_t graphs, int64_t nv, int64_t nnz);
int sweep_batch_groups(int waves);  // default workgroups
int sweep_batch(int32_t graphs, int64_t nv, const SweepIn& in, const int64_t* vbase, int64_t nmax, int waves,
                int groups, int64_t range, uint64_t* d_out, uint32_t** err, Scratch& scratch, hipStream_t s);

}  // namespace triad
