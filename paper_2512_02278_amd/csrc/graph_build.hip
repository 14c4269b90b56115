// kNN graph -> fixed-degree search graph.
//
// The paper searches "the CAGRA index" (Fantasy Sec. 3.2, stage 3) and leaves its construction
// to that index's own publication; the steps here are that publication's graph optimisation,
// with ranks standing in for distances:
//   1. detour count of an edge x -> y of rank j: the number of earlier neighbours z of x (rank
//      below j) that list y at a rank below j;
//   2. a row keeps its d_out edges of smallest (count, rank);
//   3. reverse edges: node y collects the sources x of its in-edges, ordered by (position of y
//      in x's pruned row, x), at most d_out of them;
//   4. merged row: the first d_out - d_out/2 forward edges, then up to d_out/2 reverse edges not
//      among those, then the remaining forward edges that are not in the row yet.
// An id outside [0, n) or equal to the row's own node is absent everywhere.
//
// One wavefront works on a run of consecutive nodes.  Step 1 is the expensive one: d_in graph
// rows of d_in ids are read per node (16 KB at d_in = 64), a random gather like the search's
// own, but with rows that mostly sit in the node's own cluster: runs of consecutive nodes stay
// on one XCD so that its L2 serves the re-reads.  The ids of x's row go into a small LDS table
// (id -> rank); the ids of every neighbour's row are looked up there and bump an LDS counter.
// Step 3 is a counting sort by target (histogram, scan, scatter of (position, source) words) followed by a selection per node, so that the result does not
// depend on the order in which the atomics land.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "graph_build.h"
#include "wave.h"

namespace ann {
namespace {

constexpr int kNodesPerWave = 32;
// Nodes per workgroup of in_edges_kernel (at most 256).  Small on purpose: the fewer nodes an XCD has in
// flight, the fewer target lists are half-written in its L2 at a time, and the more of their words of 4 bytes (8 where position and
// source do not fit) merge into whole lines before they are written back (25M nodes of 32 edges: 21.8 ms with 256, 9.3 with 32, 8.3 with 8).
constexpr int kChunkNodes = 8;
constexpr int kScanChunk = 4096;  // elements per workgroup of the scan kernels: 256 threads x 16

__device__ __forceinline__ void wave_lds_sync() { __syncthreads(); }  // one wavefront per workgroup

__device__ __forceinline__ bool is_present(int32_t y, int64_t n, int64_t x) { return y >= 0 && (int64_t)y < n && (int64_t)y != x; }

__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
    v = min(v, row_xor<1>(v));
    v = min(v, row_xor<2>(v));
    v = min(v, row_xor<7>(v));   // the other four of eight
    v = min(v, row_xor<15>(v));  // the other eight of sixteen
    auto s = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = min(s[0], s[1]);
    s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)min(s[0], s[1]));
}

// Node run of workgroup b: runs are dealt to the 8 XCDs (workgroup b runs on XCD b % 8) so that
// each XCD walks one contiguous eighth of the ids.
__device__ __forceinline__ int64_t first_node_of(int64_t b, int64_t runs_per_xcd) {
    return ((b & 7) * runs_per_xcd + (b >> 3)) * kNodesPerWave;
}

// ------------------------------------------------------------------------------------- steps 1 + 2
// id -> rank table of one row: a byte per slot, rank + 1 or 0 where no id of the row falls.
//
// Where the row's ids lie within kSlots consecutive ones, as they do in a cluster, id y has slot y - (smallest id of the
// row), and a lookup is that one byte: ids outside the range, and absent ones, read slot kSlots, which stays 0.
//
// Otherwise slots are addressed by hash(id) = (id ^ (id >> shift)) mod kSlots, and a lookup is one byte read and one
// comparison with the id that holds the rank; it never walks.  For that no two ids of a row may share a slot: the row
// tries up to kTries shifts.  64 ids drawn at random fit at a try with probability 0.6, 128 with 0.14.  Ids that still
// find their slot taken (after the last try; 1 row in 40 of 64 random ids, and about one id per row of 128) are
// compared one by one.
constexpr int kSlots = 4096, kTries = 8;
constexpr int kNever = 1 << 20;  // a rank above all others
constexpr int kAhead = 64;       // ranks beyond the last that are asked for by loads in flight

__device__ __forceinline__ uint32_t slot_of(uint32_t id, int shift) { return (id ^ (id >> shift)) & (kSlots - 1); }

// R registers per lane: rank j of a row lives in lane j % 64, register j / 64 (d_in <= 64 * R).
//
// An entry y of rank rr in the row of the neighbour of rank i is a detour of the edge x -> y of rank j if y is in x's row
// and j is above both i and rr: eight table reads are in flight per lane (and where the ids do not lie close together, eight
// reads of the ids at those ranks).  What the entry is needs no test: an absent one equals no id of x's row, and a rank of d_in - 1
// is below no other.  1M nodes 64 -> 32: 1.2 to 1.3 ms from machine to machine (1.48 ms with the second read everywhere), 524 vector and 145 LDS instructions per
// node (590, 211); 250 000 nodes 128 -> 64: 1.3 to 1.4 ms (1.63), 1 969 and 555 (2 261, 815).  Bound by LDS: its units are 0.85 and 0.77 busy, half of
// that with bank conflicts of random byte reads; the vector ALUs 0.72 and 0.62.
template <int R, bool VEC>
__global__ void __launch_bounds__(64) graph_prune_kernel(const int32_t* __restrict__ knn, int64_t n, int d_in, int d_out,
                                                         int32_t* __restrict__ pruned, int64_t runs_per_xcd) {
    __shared__ __align__(16) uint8_t table[kSlots + 16];
    __shared__ uint32_t cnt[64 * R + 1];            // detour count per rank + 1
    __shared__ int32_t at_rank[64 * R + 1];         // id per rank + 1 of x's row, -1 where absent
    __shared__ int32_t nbr[64 * R + kAhead];        // x's row, -1 where absent and beyond d_in
    __shared__ int32_t orow[64];
    __shared__ uint8_t extra[64 * R];               // rank + 1 of the ids that have no slot
    const int lane = lane_id();
    const int64_t x0 = first_node_of(blockIdx.x, runs_per_xcd);
    const int64_t x1 = x0 + kNodesPerWave < n ? x0 + kNodesPerWave : n;
    for (int i = lane; i <= kSlots / 16; i += 64) reinterpret_cast<uint4*>(table)[i] = make_uint4(0, 0, 0, 0);
    if (lane == 0) at_rank[0] = -1;
    for (int i = lane; i < kAhead; i += 64) nbr[64 * R + i] = -1;

    // the next node's row is read while this one is worked on
    int32_t coming[R];
    auto row_of = [&](int64_t x) {
#pragma unroll
        for (int r = 0; r < R; ++r) coming[r] = x < x1 && lane + 64 * r < d_in ? knn[x * d_in + lane + 64 * r] : -1;
    };
    row_of(x0);
    for (int64_t x = x0; x < x1; ++x) {
        int32_t mine[R];
        bool have[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int j = lane + 64 * r;
            mine[r] = coming[r];
            have[r] = is_present(mine[r], n, x);
            nbr[j] = at_rank[j + 1] = have[r] ? mine[r] : -1;
            cnt[j + 1] = 0u;
        }
        row_of(x + 1);
        wave_lds_sync();
        uint32_t least = 0x7fffffffu;
#pragma unroll
        for (int r = 0; r < R; ++r) least = have[r] ? min(least, (uint32_t)mine[r]) : least;
        least = wave_min(least);
        bool apart = false;
#pragma unroll
        for (int r = 0; r < R; ++r) apart |= have[r] && (uint32_t)mine[r] - least >= (uint32_t)kSlots;
        const bool near = !__any(apart);  // wave-uniform
        int shift = 31, n_extra = 0;      // wave-uniform
        if (near) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (have[r]) table[(uint32_t)mine[r] - least] = (uint8_t)(lane + 64 * r + 1);
        } else {
            for (int attempt = 0;; ++attempt) {
                // 31: the id itself (ids are below 2^31); then the low bits stirred with others
                shift = attempt == 0 ? 31 : attempt == 1 ? 12 : attempt == 2 ? 5 : attempt == 3 ? 8 : attempt == 4 ? 3 : attempt == 5 ? 10 : attempt == 6 ? 7 : 14;
    #pragma unroll
                for (int r = 0; r < R; ++r)
                    if (have[r]) table[slot_of((uint32_t)mine[r], shift)] = (uint8_t)(lane + 64 * r + 1);
                wave_lds_sync();
                bool lost[R], any = false;
    #pragma unroll
                for (int r = 0; r < R; ++r) {
                    lost[r] = have[r] && table[slot_of((uint32_t)mine[r], shift)] != (uint8_t)(lane + 64 * r + 1);
                    any |= lost[r];
                }
                if (!__any(any)) break;
                if (attempt == kTries - 1) {
    #pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const uint64_t m = __ballot(lost[r]);
                        if (lost[r]) extra[rank_below(m, n_extra)] = (uint8_t)(lane + 64 * r + 1);
                        n_extra += __builtin_popcountll(m);
                    }
                    break;
                }
                wave_lds_sync();
    #pragma unroll
                for (int r = 0; r < R; ++r)
                    if (have[r]) table[slot_of((uint32_t)mine[r], shift)] = 0;
                wave_lds_sync();
            }
        }
        wave_lds_sync();

        // N entries per lane: y[e] is an entry of rank rr in the row of the neighbour of rank i, later[e] = max(i, rr) + 1;
        // both hops must rank below the edge itself.  kNever as a rank: not an entry.
        auto count = [&](auto is_near, const auto& y, const auto& later) {
            constexpr int N = sizeof(y) / sizeof(y[0]);
            uint32_t at[N];
            if constexpr (decltype(is_near)::value) {
#pragma unroll
                for (int e = 0; e < N; ++e) at[e] = table[min((uint32_t)y[e] - least, (uint32_t)kSlots)];
#pragma unroll
                for (int e = 0; e < N; ++e)
                    if ((int)at[e] > later[e]) atomicAdd(&cnt[at[e]], 1u);
                return;
            }
            int32_t id[N];
#pragma unroll
            for (int e = 0; e < N; ++e) at[e] = table[slot_of((uint32_t)y[e], shift)];
#pragma unroll
            for (int e = 0; e < N; ++e) id[e] = at_rank[at[e]];
#pragma unroll
            for (int e = 0; e < N; ++e)
                if (id[e] == y[e] && (int)at[e] > later[e]) atomicAdd(&cnt[at[e]], 1u);
            for (int o = 0; o < n_extra; ++o) {
                const int j = extra[o];
                const int32_t want = at_rank[j];
#pragma unroll
                for (int e = 0; e < N; ++e)
                    if (y[e] == want && j > later[e]) atomicAdd(&cnt[j], 1u);
            }
        };
        // rows of the neighbours at ranks 0 .. d_in-2 (the last one has no edge after it)
        auto walk = [&](auto is_near) {
            if constexpr (VEC) {
                // rows of d_in % 4 == 0 ids, 16-byte aligned: a lane reads four consecutive ranks, 16 * R lanes cover a row,
                // so one load instruction fetches 4 / R rows; the next UV loads are in flight while UV are looked up
                constexpr int kLanesPerRow = 16 * R, kRowsPerLoad = 64 / kLanesPerRow, UV = 2, kStep = UV * kRowsPerLoad;
                const int quad = lane % kLanesPerRow, sub = lane / kLanesPerRow;
                const int column = min(4 * quad, d_in - 4), rank1 = 4 * quad < d_in ? 4 * quad + 1 : kNever;
                int4 v[2][UV];
                int hop1[2][UV];  // rank of the neighbour, + 1
                auto fetch = [&](int buf, int i0) {
    #pragma unroll
                    for (int u = 0; u < UV; ++u) {
                        const int i = i0 + u * kRowsPerLoad + sub;
                        const int32_t z = nbr[i];
                        hop1[buf][u] = z >= 0 ? i + 1 : kNever;  // an absent neighbour: row 0 is read for nothing
                        v[buf][u] = *reinterpret_cast<const int4*>(knn + (uint64_t)(uint32_t)max(z, 0) * (uint32_t)d_in + column);
                    }
                };
                auto look_up = [&](int buf) {
                    int32_t y[4 * UV];
                    int later[4 * UV];
    #pragma unroll
                    for (int u = 0; u < UV; ++u) {
                        y[4 * u] = v[buf][u].x;
                        y[4 * u + 1] = v[buf][u].y;
                        y[4 * u + 2] = v[buf][u].z;
                        y[4 * u + 3] = v[buf][u].w;
    #pragma unroll
                        for (int c = 0; c < 4; ++c) later[4 * u + c] = max(hop1[buf][u], rank1 + c);
                    }
                    count(is_near, y, later);
                };
                fetch(0, 0);
                for (int i0 = 0; i0 < d_in - 1; i0 += 2 * kStep) {
                    fetch(1, i0 + kStep);
                    look_up(0);
                    fetch(0, i0 + 2 * kStep);
                    look_up(1);
                }
            } else {
                // any d_in: a lane reads rank lane (+ 64) of one row per load, U rows in flight
                constexpr int U = 8;
                for (int i0 = 0; i0 < d_in - 1; i0 += U) {
                    int32_t y[U * R];
                    int later[U * R];
    #pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int i = i0 + u;
                        const int32_t z = i < d_in - 1 ? __builtin_amdgcn_readfirstlane(nbr[i]) : -1;
    #pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const int rr = lane + 64 * r;
                            y[u * R + r] = (z >= 0 && rr < d_in - 1) ? knn[(int64_t)z * d_in + rr] : -1;
                            later[u * R + r] = max(i, rr) + 1;
                        }
                    }
                    count(is_near, y, later);
                }
            }
        };
        if (near) walk(std::true_type());
        else walk(std::false_type());
        wave_lds_sync();
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (have[r]) table[near ? (uint32_t)mine[r] - least : slot_of((uint32_t)mine[r], shift)] = 0;

        // position of every present edge in ascending (count, rank): the edges whose count is lower, bit by bit from the
        // top - among the edges that agree with this one so far, those with a 0 where it has a 1 - and of the rest those
        // of lower rank.  About 55 instructions for 64 edges; comparing every pair of them took 128 and 16 LDS reads.
        uint32_t same[R][2 * R];  // the edges (a bit each, 32 to a word) that agree with this lane's edge of register r
        int c[R], pos[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const uint64_t m = __ballot(have[q]);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                same[r][2 * q] = (uint32_t)m;
                same[r][2 * q + 1] = (uint32_t)(m >> 32);
            }
            c[q] = (int)cnt[lane + 64 * q + 1];
            pos[q] = 0;
        }
        // counts are below 64 R: there are fewer ranks than that below an edge's
#pragma unroll
        for (int bit = R == 1 ? 5 : 6; bit >= 0; --bit) {
            uint64_t ones[R], any = 0;
#pragma unroll
            for (int q = 0; q < R; ++q) {
                ones[q] = __ballot((c[q] >> bit) & 1);
                any |= ones[q];
            }
            if (any) {  // uniform
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const uint32_t set = (uint32_t)(-((c[r] >> bit) & 1));
#pragma unroll
                    for (int h = 0; h < 2 * R; ++h) {
                        const uint32_t o = (uint32_t)(ones[h / 2] >> (32 * (h % 2)));
                        pos[r] += __builtin_popcount(__builtin_amdgcn_bitop3_b32(same[r][h], o, set, 0x20));  // same & ~o & set
                        same[r][h] = __builtin_amdgcn_bitop3_b32(same[r][h], o, set, 0x90);                   // same & ~(o ^ set)
                    }
                }
            }
        }
        const uint64_t below = (1ull << lane) - 1;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int h = 0; h <= 2 * r + 1; ++h)
                pos[r] += __builtin_popcount(same[r][h] & (h / 2 < r ? ~0u : (uint32_t)(below >> (32 * (h % 2)))));
        orow[lane] = -1;
        wave_lds_sync();
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (have[r] && pos[r] < d_out) orow[pos[r]] = mine[r];
        wave_lds_sync();
        if (lane < d_out) pruned[x * d_out + lane] = orow[lane];  // a present id or -1
        wave_lds_sync();
    }
}

// ------------------------------------------------------------------------------------- step 3
__global__ void __launch_bounds__(256) fill_zero_u32_kernel(uint32_t* p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = 0u;
}

// indeg[y] <- number of edges into y of the pruned graph, slot[e] <- a place of its own for edge e among those into its target.
//
// One returning atomic on device memory per edge is memory-side work of a 32-byte transaction each: 0.3 ms for 1M nodes of 32 edges
// inside the pruning kernel, whose loads waited for them.  The edges of neighbouring nodes point into the same few clusters, so a
// workgroup counts those of kCountNodes nodes in LDS, in a window of kCountWindow ids around them, and adds every counter to its
// node's total once; the total before that is where its edges' places begin.  Targets outside the window are counted directly.
constexpr int kCountNodes = 1024, kCountWindow = 16384;
__global__ void __launch_bounds__(1024) count_in_edges_kernel(const int32_t* __restrict__ g, int64_t n, int d, int nodes,
                                                              uint32_t* indeg, uint32_t* slot, int64_t groups_per_xcd) {
    __shared__ uint32_t count[kCountWindow];
    constexpr int U = 8;  // edges in flight per thread
    const int64_t x0 = ((blockIdx.x & 7) * groups_per_xcd + (blockIdx.x >> 3)) * nodes;
    if (x0 >= n) return;  // the whole workgroup
    const int64_t first = x0 * d, edges = (n - x0 < nodes ? n - x0 : nodes) * d;
    const int64_t w0 = x0 + nodes / 2 - kCountWindow / 2;  // may lie below 0
    for (int i = threadIdx.x; i < kCountWindow; i += 1024) count[i] = 0u;
    __syncthreads();
    // (an entry of the pruned graph is a present id or -1)
    for (int64_t t0 = threadIdx.x; t0 < edges; t0 += 1024 * U) {
        int32_t y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) y[u] = t0 + u * 1024 < edges ? g[first + t0 + u * 1024] : -1;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (y[u] < 0) continue;
            const uint64_t at = (uint64_t)(y[u] - w0);
            slot[first + t0 + u * 1024] = at < (uint64_t)kCountWindow ? atomicAdd(&count[at], 1u) : atomicAdd(&indeg[y[u]], 1u);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kCountWindow; i += 1024)
        if (count[i]) count[i] = atomicAdd(&indeg[w0 + i], count[i]);
    __syncthreads();
    for (int64_t t0 = threadIdx.x; t0 < edges; t0 += 1024 * U) {
        int32_t y[U];
        uint32_t at[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            y[u] = t0 + u * 1024 < edges ? g[first + t0 + u * 1024] : -1;
            at[u] = y[u] >= 0 ? slot[first + t0 + u * 1024] : 0u;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t i = (uint64_t)(y[u] - w0);
            if (y[u] >= 0 && i < (uint64_t)kCountWindow) slot[first + t0 + u * 1024] = at[u] + count[i];
        }
    }
}

// Exclusive scan of indeg[0..n) into off[0..n] (64-bit), in three launches: per-chunk sums, a scan of
// those by one workgroup, then every chunk scans itself on top of its prefix.
__global__ void __launch_bounds__(256) chunk_sums_kernel(const uint32_t* __restrict__ deg, int64_t n, int64_t* sums) {
    __shared__ int64_t part[256];
    const int t = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * kScanChunk + t * 16;
    int64_t s = 0;
    for (int i = 0; i < 16; ++i)
        if (base + i < n) s += deg[base + i];
    part[t] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w) part[t] += part[t + w];
        __syncthreads();
    }
    if (t == 0) sums[blockIdx.x] = part[0];
}

__global__ void __launch_bounds__(1024) scan_sums_kernel(int64_t* sums, int64_t count) {
    __shared__ int64_t part[1024];
    const int t = threadIdx.x;
    const int64_t per = (count + 1023) / 1024;
    const int64_t lo = t * per, hi = lo + per < count ? lo + per : count;
    int64_t s = 0;
    for (int64_t i = lo; i < hi; ++i) s += sums[i];
    part[t] = s;
    __syncthreads();
    for (int w = 1; w < 1024; w <<= 1) {  // Hillis-Steele inclusive scan of the per-thread sums
        const int64_t v = t >= w ? part[t - w] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    int64_t run = part[t] - s;
    for (int64_t i = lo; i < hi; ++i) {
        const int64_t c = sums[i];
        sums[i] = run;
        run += c;
    }
}

__global__ void __launch_bounds__(256) offsets_kernel(const uint32_t* __restrict__ deg, int64_t n,
                                                      const int64_t* __restrict__ sums, int64_t* off) {
    __shared__ int64_t part[256];
    const int t = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * kScanChunk + t * 16;
    int64_t s = 0;
    for (int i = 0; i < 16; ++i)
        if (base + i < n) s += deg[base + i];
    part[t] = s;
    __syncthreads();
    for (int w = 1; w < 256; w <<= 1) {
        const int64_t v = t >= w ? part[t - w] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    int64_t run = sums[blockIdx.x] + part[t] - s;
    for (int i = 0; i < 16; ++i) {
        if (base + i < n) {
            off[base + i] = run;
            run += deg[base + i];
            if (base + i == n - 1) off[n] = run;
        }
    }
}

// A word of an in-edge orders by (position in the source's row, source): 32 bits where both fit, else 64.
template <class Word>
__device__ __forceinline__ Word edge_word(int position, int64_t source, int source_bits) {
    return sizeof(Word) == 8 ? (Word)(((uint64_t)(uint32_t)position << 32) | (uint32_t)source) : (Word)((uint32_t)position << source_bits | (uint32_t)source);
}

// Chunk of kChunkNodes nodes a workgroup of the edge kernel works on: like the node runs above, the chunks
// are dealt so that an XCD walks a contiguous eighth of the ids; the edges of neighbouring nodes point
// into the same few clusters, and their words then meet in one L2 before they are written back.
__device__ __forceinline__ int64_t chunk_of(int64_t b, int64_t chunks_per_xcd) { return (b & 7) * chunks_per_xcd + (b >> 3); }

// pairs[off[y] + slot[e]] <- the word of every edge e into y
//
// Chunk c covers the kChunkNodes nodes from kChunkNodes * c on: element t of their rows is node
// kChunkNodes * c + t / d, position t % d, with t / d == (t * d_inv) >> 22 for t < 256 * d, d <= 64
// (d_inv = ceil(2^22 / d)).
template <class Word>
__global__ void __launch_bounds__(256) in_edges_kernel(const int32_t* __restrict__ g, int64_t n, int d, uint32_t d_inv,
                                                       const int64_t* __restrict__ off, const uint32_t* __restrict__ slot,
                                                       Word* __restrict__ pairs, int64_t chunks_per_xcd, int source_bits) {
    const int64_t xb = chunk_of(blockIdx.x, chunks_per_xcd) * kChunkNodes;
    const int rows = n - xb < kChunkNodes ? (n > xb ? (int)(n - xb) : 0) : kChunkNodes;
    for (int t = threadIdx.x; t < rows * d; t += 256) {
        const int xl = (int)(((uint32_t)t * d_inv) >> 22);
        const int64_t x = xb + xl;
        const int32_t y = g[xb * d + t];
        if (is_present(y, n, x)) pairs[off[y] + slot[xb * d + t]] = edge_word<Word>(t - xl * d, x, source_bits);
    }
}

// ------------------------------------------------------------------------------------- steps 3 (selection) + 4
// The 64 smallest words of a node's in-edges, ascending: one per lane, all ones where there are fewer.  first: the first 64 of them.
__device__ __forceinline__ uint64_t smallest_in_edges(const uint64_t* __restrict__ pairs, uint64_t first, int64_t lo, int64_t hi, int lane) {
    uint64_t best[1] = {kInfKey};
    for (int64_t c0 = lo; c0 < hi; c0 += 64) {
        uint64_t v[1] = {c0 == lo ? first : c0 + lane < hi ? pairs[c0 + lane] : kInfKey};
        bitonic_sort<1>(v, lane);
        if (c0 == lo) {  // the first chunk (the only one for most nodes) is the best so far as it is
            best[0] = v[0];
            continue;
        }
        // element e of the best so far against element 63 - e of the sorted chunk keeps the 64 smallest of both, as one
        // bitonic run
        const uint64_t o = xor_lane64<63>(v[0], lane);
        best[0] = o < best[0] ? o : best[0];
        bitonic_merge<1>(best, lane);
    }
    return best[0];
}
__device__ __forceinline__ uint32_t smallest_in_edges(const uint32_t* __restrict__ pairs, uint32_t first, int64_t lo, int64_t hi, int lane) {
    const LaneBits bits(lane);
    uint32_t best = hi - lo <= 32 ? bits.sort<32>(first) : bits.sort<64>(first);  // uniform; lanes from 32 on hold nothing
    for (int64_t c0 = lo + 64; c0 < hi; c0 += 64) {
        const uint32_t v = c0 + lane < hi ? pairs[c0 + lane] : 0xffffffffu;
        best = bits.clean<5>(min(best, ~bits.sort<64>(~v)));  // against a descending chunk
    }
    return best;
}

template <class Word>
__global__ void __launch_bounds__(64) graph_merge_kernel(const int32_t* __restrict__ pruned, int64_t n, int d,
                                                         const int64_t* __restrict__ off,
                                                         const Word* __restrict__ pairs, int32_t* __restrict__ out,
                                                         int64_t runs_per_xcd, int source_bits) {
    __shared__ int32_t fwd[64];
    __shared__ int32_t row[64];
    const int lane = lane_id();
    const int h = d / 2, nh = d - h;
    const int64_t x0 = first_node_of(blockIdx.x, runs_per_xcd);
    const int64_t x1 = x0 + kNodesPerWave < n ? x0 + kNodesPerWave : n;
    // two nodes ahead the bounds of the in-edges, one node ahead the first of them and the pruned row
    auto bound = [&](int64_t x) { return off[x < x1 ? x : x1]; };
    auto first = [&](int64_t lo, int64_t hi) { return lo + lane < hi ? pairs[lo + lane] : (Word)~(Word)0; };
    auto row_of = [&](int64_t x) { return x < x1 && lane < d ? pruned[x * d + lane] : -1; };
    int64_t lo = x0 < x1 ? bound(x0) : 0, hi = x0 < x1 ? bound(x0 + 1) : 0, after = x0 < x1 ? bound(x0 + 2) : 0;
    Word next_words = first(lo, hi);
    int32_t next_row = row_of(x0);
    for (int64_t x = x0; x < x1; ++x) {
        const Word words = next_words;
        const int32_t f = next_row;
        const int64_t from = lo, to = hi;
        lo = hi;
        hi = after;
        next_words = first(lo, hi);
        next_row = row_of(x + 1);
        after = bound(x + 3);
        const Word word = smallest_in_edges(pairs, words, from, to, lane);
        const int32_t source = (int32_t)(sizeof(Word) == 8 ? (uint32_t)word : (uint32_t)word & ((1u << source_bits) - 1u));
        const int32_t rv = (lane < d && word != (Word)~(Word)0) ? source : -1;
        const bool fok = is_present(f, n, x);
        fwd[lane] = fok ? f : -1;
        const bool head = fok && lane < nh;
        const uint64_t bh = __ballot(head);
        const int n_head = __builtin_popcountll(bh);
        if (head) row[rank_below(bh)] = f;
        wave_lds_sync();
        bool member = false;
        for (int t = 0; t < nh; ++t) member |= fwd[t] == rv;
        const bool fresh = rv >= 0 && !member;
        const uint64_t bf = __ballot(fresh);
        const int rk = rank_below(bf);
        const int n_fresh = __builtin_popcountll(bf);
        const int n_take = n_fresh < h ? n_fresh : h;
        if (fresh && rk < h) row[n_head + rk] = rv;
        wave_lds_sync();
        bool dup = false;
        for (int t = 0; t < n_take; ++t) dup |= row[n_head + t] == f;
        const bool tail = fok && lane >= nh && !dup;
        const uint64_t bt = __ballot(tail);
        const int pos = n_head + n_take + rank_below(bt);
        if (tail && pos < d) row[pos] = f;
        const int all = n_head + n_take + __builtin_popcountll(bt);
        const int len = all < d ? all : d;
        wave_lds_sync();
        if (lane < d) out[x * d + lane] = lane < len ? row[lane] : -1;
        wave_lds_sync();
    }
}

unsigned blocks_for(int64_t items) {
    const int64_t b = (items + 255) / 256;
    return (unsigned)(b < 65536 ? (b > 0 ? b : 1) : 65536);
}

int64_t align256(int64_t b) { return (b + 255) & ~(int64_t)255; }

int64_t runs_per_xcd_of(int64_t n) {
    const int64_t runs = (n + kNodesPerWave - 1) / kNodesPerWave;
    return (runs + 7) / 8;
}

}  // namespace

namespace {

template <int R>
void launch_prune_rows(bool vec, dim3 grid, hipStream_t stream, const int32_t* knn, int64_t n, int d_in, int d_out, int32_t* pruned, int64_t rpx) {
    if (vec) hipLaunchKernelGGL((graph_prune_kernel<R, true>), grid, dim3(64), 0, stream, knn, n, d_in, d_out, pruned, rpx);
    else hipLaunchKernelGGL((graph_prune_kernel<R, false>), grid, dim3(64), 0, stream, knn, n, d_in, d_out, pruned, rpx);
}

}  // namespace

hipError_t launch_graph_prune(const int32_t* knn, int64_t n, int d_in, int d_out, int32_t* pruned, hipStream_t stream) {
    const int64_t rpx = runs_per_xcd_of(n);
    const dim3 grid((unsigned)(8 * rpx));
    // rows that start on 16-byte boundaries are read four ids per lane
    const bool vec = d_in % 4 == 0 && (reinterpret_cast<uintptr_t>(knn) & 15u) == 0;
    if (d_in <= 64) launch_prune_rows<1>(vec, grid, stream, knn, n, d_in, d_out, pruned, rpx);
    else launch_prune_rows<2>(vec, grid, stream, knn, n, d_in, d_out, pruned, rpx);
    return hipGetLastError();
}

// scratch layout: pruned (n * d i32) | indeg (n u32) | off (n + 1 i64) | chunk sums (i64) | in-edge words (n * d u64 or u32)
int64_t graph_optimize_scratch_bytes(int64_t n, int d) {
    const int64_t chunks = (n + kScanChunk - 1) / kScanChunk;
    return align256(n * d * 4) + align256(n * 4) + align256((n + 1) * 8) + align256(chunks * 8) + align256(n * d * 8);
}

hipError_t launch_graph_optimize(const int32_t* knn, int64_t n, int d_in, int d, int32_t* out, void* scratch,
                                 hipStream_t stream) {
    const int64_t chunks = (n + kScanChunk - 1) / kScanChunk;
    char* base = static_cast<char*>(scratch);
    int32_t* pruned = reinterpret_cast<int32_t*>(base);
    base += align256(n * d * 4);
    uint32_t* indeg = reinterpret_cast<uint32_t*>(base);
    base += align256(n * 4);
    int64_t* off = reinterpret_cast<int64_t*>(base);
    base += align256((n + 1) * 8);
    int64_t* sums = reinterpret_cast<int64_t*>(base);
    base += align256(chunks * 8);
    // until the last kernel writes it, `out` holds the slot of every edge within its target's list
    uint32_t* slot = reinterpret_cast<uint32_t*>(out);
    const uint32_t d_inv = (uint32_t)(((1u << 22) + d - 1) / d);
    const int64_t chunks_per_xcd = ((n + kChunkNodes - 1) / kChunkNodes + 7) / 8;
    const unsigned node_blocks = (unsigned)(8 * chunks_per_xcd);
    hipLaunchKernelGGL(fill_zero_u32_kernel, dim3(blocks_for(n)), dim3(256), 0, stream, indeg, n);
    const hipError_t e = launch_graph_prune(knn, n, d_in, d, pruned, stream);
    if (e != hipSuccess) return e;
    const int nodes = n >= 256 * kCountNodes ? kCountNodes : 256;  // fewer where the chip would be left idle
    const int64_t groups_per_xcd = ((n + nodes - 1) / nodes + 7) / 8;
    hipLaunchKernelGGL(count_in_edges_kernel, dim3((unsigned)(8 * groups_per_xcd)), dim3(1024), 0, stream, pruned, n, d, nodes, indeg, slot,
                       groups_per_xcd);
    hipLaunchKernelGGL(chunk_sums_kernel, dim3((unsigned)chunks), dim3(256), 0, stream, indeg, n, sums);
    hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(1024), 0, stream, sums, chunks);
    hipLaunchKernelGGL(offsets_kernel, dim3((unsigned)chunks), dim3(256), 0, stream, indeg, n, sums, off);
    const int64_t rpx = runs_per_xcd_of(n);
    int source_bits = 1;
    while ((int64_t)1 << source_bits < n) ++source_bits;
    // a word of all ones stands for "none"
    const bool narrow = source_bits < 32 && ((uint64_t)(d - 1) << source_bits | (uint64_t)(n - 1)) < 0xffffffffu;
    auto finish = [&](auto* words) {
        typedef std::remove_reference_t<decltype(*words)> Word;
        hipLaunchKernelGGL(in_edges_kernel<Word>, dim3(node_blocks), dim3(256), 0, stream, pruned, n, d, d_inv, off, slot, words, chunks_per_xcd, source_bits);
        hipLaunchKernelGGL(graph_merge_kernel<Word>, dim3((unsigned)(8 * rpx)), dim3(64), 0, stream, pruned, n, d, off, words, out, rpx, source_bits);
    };
    if (narrow) finish(reinterpret_cast<uint32_t*>(base));
    else finish(reinterpret_cast<uint64_t*>(base));
    return hipGetLastError();
}

}  // namespace ann
