// hb_ragged.hpp -- packed batches in tiles (hb_ragged.hip), for callers with workspace.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hb {

// What k_long_pick decides.
struct LongMeta {
    uint32_t max_key;   // largest sort key seen
    uint32_t from[3];   // per algorithm: messages of at least this key are long
    uint32_t count[3];  // their number
    uint32_t pos[3];    // first position in `sorted`
    uint32_t group[4];  // first group of SM3, SHA-1, MD5, and the end
};

// Device workspace of launch_ragged_long.
struct LongWs {
    uint32_t *hist, *cursor, *start;  // 3 * kBins each
    uint32_t *sorted;                 // n message indices at most
    LongMeta *meta;
    uint32_t min_key;                 // no message of fewer blocks is long
};

// Whether launch_ragged's workgroups for n messages fill the chip at most once: every
// message then starts at once, and picking out the long ones gains nothing.
bool ragged_in_one_round(uint64_t n, bool mixed);

// As launch_ragged, the batch's longest messages picked out and started first.
hipError_t launch_ragged_long(const LongWs &w, const uint8_t *algos, int algo, const uint8_t *msgs, const uint64_t *offs,
                              const uint64_t *lens, uint64_t n, uint8_t *out, uint32_t stride, hipStream_t stream);

}  // namespace hb
