// Keys of many queries against every row of their cluster, ahead of the search.
//
// A query that is routed to one cluster scores a third to nearly all of the cluster's rows, and the queries of one
// cluster gather the same rows again and again.  Here every row is read once for Q queries at a time, and the
// ordered keys go to a table that the search then reads four bytes at a time.  A key has the bits that the search's
// own gather would give it: the sums run over the same pieces in the same lanes and meet in the same tree.
//
// Float rows only.  A uint8 row of 128 bytes costs the search so little that the table, which is written to memory and
// read again, was no gain: 500 000 queries over clusters of 1 950 such rows took 10.3 ms with it (on the matrix
// cores), 10.0 ms without.
//
// The execution order has put the queries of a cluster next to each other.  A workgroup takes Q consecutive
// positions - runs of one cluster, one after the other - and one slice of the clusters' rows, shared out to its
// four wavefronts.  Neighbouring positions run on one XCD, whose L2 then serves the re-reads of a cluster's rows.
#pragma once

#include "row_ops.h"

namespace ann {

struct KeyTableParams {
    const uint8_t* vectors;
    int64_t n;
    int64_t row_stride;
    int32_t row_bytes;
    const uint8_t* queries;
    const int32_t* order;            // position -> query
    const int32_t* route;            // query -> cluster
    int64_t q_base, q_count;         // positions [q_base, q_base + q_count); table row i belongs to position q_base + i
    const int64_t* cluster_offsets;
    int32_t n_clusters;
    int32_t stride;                  // keys per query, a multiple of 32: rows beyond it are left to the search
    int32_t slices, slice_rows;      // slices of a cluster's rows, slice_rows (a multiple of 64) rows each
    uint32_t* table;
    int32_t* none;                   // a counter that is set to zero, or null
};

template <int Q>
unsigned key_table_grid(const KeyTableParams& p) {
    return (unsigned)(64 * ((p.q_count + Q * 64 - 1) / (Q * 64)) * p.slices);
}

// The runs a workgroup works on, all values uniform.
template <int Q>
struct KeyTableRuns {
    static_assert(Q <= 64, "a position per lane");
    int64_t pos;       // first position of the run, relative to q_base
    int m;             // its queries
    int64_t lo;        // its cluster's first row
    int r0, r1;        // rows lo + [r0, r1)
    int slice, left;   // positions from pos on, this run's included
    int32_t query, cluster;  // of position pos + lane, for lanes below left

    __device__ __forceinline__ void begin(const KeyTableParams& p, int lane) {
        // on each XCD eight neighbouring position sets go through a slice side by side, then through the next slice
        const int64_t per_xcd = ((p.q_count + Q * 64 - 1) / (Q * 64)) * 8;
        const int at = blockIdx.x >> 3;
        const int of_eight = at / (8 * p.slices), in_eight = at - of_eight * (8 * p.slices);
        slice = in_eight >> 3;
        pos = ((int64_t)(blockIdx.x & 7) * per_xcd + of_eight * 8 + (in_eight & 7)) * Q;
        left = p.q_count - pos < Q ? (p.q_count > pos ? (int)(p.q_count - pos) : 0) : Q;
        m = 0;
        query = lane < left ? p.order[p.q_base + pos + lane] : 0;
        cluster = lane < left ? p.route[query] : -1;
    }
    // The next run with rows in this slice.
    __device__ __forceinline__ bool next(const KeyTableParams& p, int lane) {
        for (;;) {
            pos += m;
            left -= m;
            if (left <= 0) return false;
            if (m > 0) {
                query = __shfl(query, lane + m);
                cluster = __shfl(cluster, lane + m);
            }
            const int32_t c = __builtin_amdgcn_readfirstlane(cluster);
            const uint64_t other = __ballot(lane >= left || cluster != c);
            m = other ? __builtin_ctzll(other) : 64;
            if ((uint32_t)c >= (uint32_t)p.n_clusters) continue;
            lo = p.cluster_offsets[c];
            const int64_t size = p.cluster_offsets[c + 1] - lo;
            const int cols = size < (int64_t)p.stride ? (int)size : p.stride;
            r0 = slice * p.slice_rows;
            r1 = r0 + p.slice_rows < cols ? r0 + p.slice_rows : cols;
            if (r0 < r1) return true;
        }
    }
};

// Float rows as the search variant (dtype, metric, g, nch) reads them (key_table.hip), and the positions per workgroup.
hipError_t launch_key_table(int dtype, int metric, int g, int nch, const KeyTableParams& p, hipStream_t stream);
constexpr int key_table_set(int nch) { return nch <= 3 ? 8 : nch <= 6 ? 4 : 2; }

}  // namespace ann
