// What a launch of the search kernels works on.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ann {

struct SearchParams {
    const uint8_t* vectors;
    int64_t n;
    int64_t row_stride;
    int32_t row_bytes;
    const int32_t* graph;
    int32_t degree;
    uint32_t degree_inv;  // ceil(2^20 / degree): s / degree == (s * degree_inv) >> 20 for s < 1024
    const uint8_t* queries;
    int64_t nq;
    int64_t q_base, q_count;  // this launch serves queries [q_base, q_base + q_count)
    int32_t k, itopk, width, max_iters;
    int32_t n_entry, entry_mode;
    uint64_t seed;
    const int32_t* route;            // nq * route_c nearest clusters (routed mode)
    const int64_t* cluster_offsets;  // routed mode
    int32_t route_c;
    int32_t n_clusters;   // routed mode: a route id outside [0, n_clusters) names no cluster (no window, no entries)
    int32_t hash_bits;    // visited hash has 1 << hash_bits slots
    int32_t window_bits;  // bits of the visited bitmap (multiple of 32; 0 = none)
    int32_t cap;        // most candidates one round can produce, multiple of 64
    int32_t* out_ids;
    uint32_t* out_dists;
    int32_t* out_counters;  // nq * 4 or null
    const int32_t* order;   // execution order: the launch's i-th query is order[q_base + i]; null = identity
    int64_t q_per_xcd;      // queries of this launch handed to each of the 8 XCDs
    const uint32_t* table;  // ordered keys of the launch's i-th query against its first window, i * table_stride on; or null
    int32_t table_stride;   // keys per query
    int32_t rank_rows;      // clusters of up to this many rows are searched by rank (rank_search.h); 0: none
    int32_t rank_places;    // ranks that are settled, a multiple of kRankTiles * kRankTile
    int32_t* again;         // positions that the search by rank has left to another: how many, then which; or null
};

__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t counter) {
    uint64_t z = seed + (counter + 1) * 0x9E3779B97F4A7C15ull;
    z ^= z >> 30;
    z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27;
    z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z;
}

}  // namespace ann
