// The retrieval pool behind the opaque laser_pool handle, and its construction on the device (pool_index.hip).
#pragma once

#include <vector>

#include "common.h"

namespace laser {

struct Pool {
    int32_t* P = nullptr;
    uint32_t* seq_end = nullptr;
    uint32_t* sa = nullptr;
    IndexEntry* table = nullptr;
    uint64_t cap_mask = 0;
    int64_t n_tokens = 0, n_keys = 0, n_entries = 0, n_sa = 0, device_bytes = 0;
    int n_max = 0;
};

// The regrouped pool's sequences in their final order, empty ones left out.
struct PoolLayout {
    std::vector<uint32_t> dst_off;      // [n + 1] where they begin in P
    std::vector<uint32_t> src_off;      // [n] where they begin in the caller's token array
    std::vector<uint32_t> sub;          // [n] their sub-pool
    std::vector<int64_t> sub_key;       // keys of the sub-pools, ascending
    uint32_t token_bits = 0;            // all tokens or-ed together
};

// Fills p (arrays and counts; nothing is kept on failure). *no_memory: the device could not hold the pool and the working
// arrays, or they exceed mem_limit bytes (< 0: no limit).
int build_index_device(const int32_t* tokens, const PoolLayout& lay, int n_max, int64_t mem_limit, hipStream_t stream, Pool* p, bool* no_memory);

}  // namespace laser
