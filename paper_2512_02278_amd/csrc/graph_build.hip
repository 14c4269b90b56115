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
// Step 3 is a counting sort by target (histogram - counted by the pruning kernel itself -, scan,
// scatter of (position, source) words) followed by a selection per node, so that the result does not
// depend on the order in which the atomics land.
#include <hip/hip_runtime.h>

#include "graph_build.h"
#include "wave.h"

namespace ann {
namespace {

constexpr int kNodesPerWave = 32;
// Nodes per workgroup of in_edges_kernel (at most 256).  Small on purpose: the fewer nodes an XCD has in
// flight, the fewer target lists are half-written in its L2 at a time, and the more of their 8-byte words
// merge into whole lines before they are written back (22.5 ms per 25M nodes with 256, 9.5 ms with 8).
constexpr int kChunkNodes = 8;
constexpr int kScanChunk = 4096;  // elements per workgroup of the scan kernels: 256 threads x 16

__device__ __forceinline__ void wave_lds_sync() { __syncthreads(); }  // one wavefront per workgroup

__device__ __forceinline__ bool is_present(int32_t y, int64_t n, int64_t x) { return y >= 0 && (int64_t)y < n && (int64_t)y != x; }

// Node run of workgroup b: runs are dealt to the 8 XCDs (workgroup b runs on XCD b % 8) so that
// each XCD walks one contiguous eighth of the ids.
__device__ __forceinline__ int64_t first_node_of(int64_t b, int64_t runs_per_xcd) {
    return ((b & 7) * runs_per_xcd + (b >> 3)) * kNodesPerWave;
}

// ------------------------------------------------------------------------------------- steps 1 + 2
// id -> rank table of one row: a byte per slot, rank + 1 or 0 where no id of the row falls, addressed directly by
// hash(id) = (id ^ (id >> shift)) mod kSlots.  A lookup is one byte read and one comparison with the id that holds the
// rank; it never walks.  For that no two ids of a row may share a slot: the row tries up to kTries shifts.  The first
// leaves the low bits of the id, which are distinct whenever the row's neighbours lie within kSlots consecutive ids, as
// they do in a cluster; 64 ids drawn at random fit at a try with probability 0.6, 128 with 0.14.  Ids that still find
// their slot taken (after the last try; 1 row in 40 of 64 random ids, and about one id per row of 128) are compared
// one by one.
constexpr int kSlots = 4096, kTries = 8;
constexpr int kNever = 1 << 20;  // a rank above all others
constexpr int kAhead = 64;       // ranks beyond the last that are asked for by loads in flight

__device__ __forceinline__ uint32_t slot_of(uint32_t id, int shift) { return (id ^ (id >> shift)) & (kSlots - 1); }

// R registers per lane: rank j of a row lives in lane j % 64, register j / 64 (d_in <= 64 * R).
//
// An entry y of rank rr in the row of the neighbour of rank i is a detour of the edge x -> y of rank j if y is in x's row
// and j is above both i and rr: sixteen table reads are in flight per lane, then sixteen reads of the ids at those ranks.
// What the entry is needs no test: an absent one equals no id of x's row, and a rank of d_in - 1 is below no other.
// About 7 vector instructions per 64 lookups (25 with a Bloom filter, a queue and a bucketed table).  1M nodes 64 -> 32:
// 1.70 ms (3.13 ms before), 590 vector and 211 LDS instructions per node; 250 000 nodes 128 -> 64: 1.79 ms (4.71 ms), 2 261 and 815.
// Bound by LDS: its units are 0.84 and 0.80 busy, nearly half of that with bank conflicts of random byte reads; the vector ALUs
// 0.63 and 0.56.
//
// COUNT: the kernel also counts the in-edges of the pruned graph (step 3's histogram) - one returning
// atomic per pruned edge, whose result is the edge's slot in its target's list.  The atomics are
// memory-side work that overlaps this kernel's instruction-bound lookups, instead of a pass of its own.
template <int R, bool COUNT, bool VEC>
__global__ void __launch_bounds__(64) graph_prune_kernel(const int32_t* __restrict__ knn, int64_t n, int d_in, int d_out,
                                                         int32_t* __restrict__ pruned, int64_t runs_per_xcd,
                                                         uint32_t* indeg, uint32_t* __restrict__ slot) {
    __shared__ __align__(16) uint8_t table[kSlots];
    __shared__ uint32_t cnt[64 * R + 1];            // detour count per rank + 1
    __shared__ int32_t at_rank[64 * R + 1];         // id per rank + 1 of x's row, -1 where absent
    __shared__ int32_t nbr[64 * R + kAhead];        // x's row, -1 where absent and beyond d_in
    __shared__ int32_t orow[64];
    __shared__ uint8_t extra[64 * R];               // rank + 1 of the ids that have no slot
    const int lane = lane_id();
    const int64_t x0 = first_node_of(blockIdx.x, runs_per_xcd);
    const int64_t x1 = x0 + kNodesPerWave < n ? x0 + kNodesPerWave : n;
    for (int i = lane; i < kSlots / 16; i += 64) reinterpret_cast<uint4*>(table)[i] = make_uint4(0, 0, 0, 0);
    if (lane == 0) at_rank[0] = -1;
    for (int i = lane; i < kAhead; i += 64) nbr[64 * R + i] = -1;

    // the next node's row is read while this one is worked on, and the slot of an edge is stored a node later, when the
    // atomic that counts it has long returned
    int32_t coming[R];
    auto row_of = [&](int64_t x) {
#pragma unroll
        for (int r = 0; r < R; ++r) coming[r] = x < x1 && lane + 64 * r < d_in ? knn[x * d_in + lane + 64 * r] : -1;
    };
    bool counted = false;
    uint32_t counted_slot = 0;
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
        int shift = 31, n_extra = 0;  // wave-uniform
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
        wave_lds_sync();

        // N entries per lane: y[e] is an entry of rank rr in the row of the neighbour of rank i, later[e] = max(i, rr) + 1;
        // both hops must rank below the edge itself.  kNever as a rank: not an entry.
        auto count = [&](const auto& y, const auto& later) {
            constexpr int N = sizeof(y) / sizeof(y[0]);
            uint32_t at[N];
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
                count(y, later);
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
                count(y, later);
            }
        }
        wave_lds_sync();
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (have[r]) table[slot_of((uint32_t)mine[r], shift)] = 0;

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
        if constexpr (COUNT) {
            if (counted) slot[(x - 1) * d_out + lane] = counted_slot;
        }
        counted = false;
        if (lane < d_out) {
            const int32_t y = orow[lane];  // a present id or -1
            pruned[x * d_out + lane] = y;
            counted = y >= 0;
            if (COUNT && counted) counted_slot = atomicAdd(&indeg[y], 1u);
        }
        wave_lds_sync();
    }
    if constexpr (COUNT) {
        if (counted) slot[(x1 - 1) * d_out + lane] = counted_slot;
    }
}

// ------------------------------------------------------------------------------------- step 3
__global__ void __launch_bounds__(256) fill_zero_u32_kernel(uint32_t* p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = 0u;
}

// Chunk of kChunkNodes nodes a workgroup of the edge kernel works on: like the node runs above, the chunks
// are dealt so that an XCD walks a contiguous eighth of the ids; the edges of neighbouring nodes point
// into the same few clusters, and their 8-byte words then meet in one L2 before they are written back.
__device__ __forceinline__ int64_t chunk_of(int64_t b, int64_t chunks_per_xcd) { return (b & 7) * chunks_per_xcd + (b >> 3); }

// Chunk c covers the kChunkNodes nodes from kChunkNodes * c on: element t of their rows is node
// kChunkNodes * c + t / d, position t % d, with t / d == (t * d_inv) >> 22 for t < 256 * d, d <= 64
// (d_inv = ceil(2^22 / d)).
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

// pairs[off[y] + slot[e]] <- (position << 32) | source of every edge e into y
__global__ void __launch_bounds__(256) in_edges_kernel(const int32_t* __restrict__ g, int64_t n, int d, uint32_t d_inv,
                                                       const int64_t* __restrict__ off, const uint32_t* __restrict__ slot,
                                                       uint64_t* __restrict__ pairs, int64_t chunks_per_xcd) {
    const int64_t xb = chunk_of(blockIdx.x, chunks_per_xcd) * kChunkNodes;
    const int rows = n - xb < kChunkNodes ? (n > xb ? (int)(n - xb) : 0) : kChunkNodes;
    for (int t = threadIdx.x; t < rows * d; t += 256) {
        const int xl = (int)(((uint32_t)t * d_inv) >> 22);
        const int64_t x = xb + xl;
        const int32_t y = g[xb * d + t];
        if (is_present(y, n, x)) pairs[off[y] + slot[xb * d + t]] = ((uint64_t)(uint32_t)(t - xl * d) << 32) | (uint32_t)x;
    }
}

// ------------------------------------------------------------------------------------- steps 3 (selection) + 4
__global__ void __launch_bounds__(64) graph_merge_kernel(const int32_t* __restrict__ pruned, int64_t n, int d,
                                                         const int64_t* __restrict__ off,
                                                         const uint64_t* __restrict__ pairs, int32_t* __restrict__ out,
                                                         int64_t runs_per_xcd) {
    __shared__ int32_t fwd[64];
    __shared__ int32_t row[64];
    const int lane = lane_id();
    const int h = d / 2, nh = d - h;
    const int64_t x0 = first_node_of(blockIdx.x, runs_per_xcd);
    const int64_t x1 = x0 + kNodesPerWave < n ? x0 + kNodesPerWave : n;
    for (int64_t x = x0; x < x1; ++x) {
        // the 64 smallest (position, source) words of x's in-edges, ascending: one word per lane
        uint64_t best[1] = {kInfKey};
        const int64_t lo = off[x], hi = off[x + 1];
        for (int64_t c0 = lo; c0 < hi; c0 += 64) {
            uint64_t v[1] = {c0 + lane < hi ? pairs[c0 + lane] : kInfKey};
            bitonic_sort<1>(v, lane);
            if (c0 == lo) {  // the first chunk (the only one for most nodes) is the best so far as it is
                best[0] = v[0];
                continue;
            }
            // element e of the best so far against element 63 - e of the sorted chunk keeps the 64
            // smallest of both, as one bitonic run
            const uint64_t o = xor_lane64<63>(v[0], lane);
            best[0] = o < best[0] ? o : best[0];
            bitonic_merge<1>(best, lane);
        }
        const int32_t rv = (lane < d && best[0] != kInfKey) ? (int32_t)(uint32_t)best[0] : -1;
        const int32_t f = lane < d ? pruned[x * d + lane] : -1;
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

template <int R, bool COUNT>
void launch_prune_rc(bool vec, dim3 grid, hipStream_t stream, const int32_t* knn, int64_t n, int d_in, int d_out,
                     int32_t* pruned, int64_t rpx, uint32_t* indeg, uint32_t* slot) {
    if (vec)
        hipLaunchKernelGGL((graph_prune_kernel<R, COUNT, true>), grid, dim3(64), 0, stream, knn, n, d_in, d_out, pruned, rpx, indeg, slot);
    else
        hipLaunchKernelGGL((graph_prune_kernel<R, COUNT, false>), grid, dim3(64), 0, stream, knn, n, d_in, d_out, pruned, rpx, indeg, slot);
}

hipError_t launch_prune(const int32_t* knn, int64_t n, int d_in, int d_out, int32_t* pruned, uint32_t* indeg,
                        uint32_t* slot, hipStream_t stream) {
    const int64_t rpx = runs_per_xcd_of(n);
    const dim3 grid((unsigned)(8 * rpx));
    // rows that start on 16-byte boundaries are read four ids per lane
    const bool vec = d_in % 4 == 0 && (reinterpret_cast<uintptr_t>(knn) & 15u) == 0;
    if (d_in <= 64 && indeg) launch_prune_rc<1, true>(vec, grid, stream, knn, n, d_in, d_out, pruned, rpx, indeg, slot);
    else if (d_in <= 64) launch_prune_rc<1, false>(vec, grid, stream, knn, n, d_in, d_out, pruned, rpx, indeg, slot);
    else if (indeg) launch_prune_rc<2, true>(vec, grid, stream, knn, n, d_in, d_out, pruned, rpx, indeg, slot);
    else launch_prune_rc<2, false>(vec, grid, stream, knn, n, d_in, d_out, pruned, rpx, indeg, slot);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_graph_prune(const int32_t* knn, int64_t n, int d_in, int d_out, int32_t* pruned, hipStream_t stream) {
    return launch_prune(knn, n, d_in, d_out, pruned, nullptr, nullptr, stream);
}

// scratch layout: pruned (n * d i32) | indeg (n u32) | off (n + 1 i64) | chunk sums (i64) | pairs (n * d u64)
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
    uint64_t* pairs = reinterpret_cast<uint64_t*>(base);
    // until the last kernel writes it, `out` holds the slot of every edge within its target's list
    uint32_t* slot = reinterpret_cast<uint32_t*>(out);
    const uint32_t d_inv = (uint32_t)(((1u << 22) + d - 1) / d);
    const int64_t chunks_per_xcd = ((n + kChunkNodes - 1) / kChunkNodes + 7) / 8;
    const unsigned node_blocks = (unsigned)(8 * chunks_per_xcd);
    hipLaunchKernelGGL(fill_zero_u32_kernel, dim3(blocks_for(n)), dim3(256), 0, stream, indeg, n);
    const hipError_t e = launch_prune(knn, n, d_in, d, pruned, indeg, slot, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(chunk_sums_kernel, dim3((unsigned)chunks), dim3(256), 0, stream, indeg, n, sums);
    hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(1024), 0, stream, sums, chunks);
    hipLaunchKernelGGL(offsets_kernel, dim3((unsigned)chunks), dim3(256), 0, stream, indeg, n, sums, off);
    hipLaunchKernelGGL(in_edges_kernel, dim3(node_blocks), dim3(256), 0, stream, pruned, n, d, d_inv, off, slot, pairs, chunks_per_xcd);
    const int64_t rpx = runs_per_xcd_of(n);
    hipLaunchKernelGGL(graph_merge_kernel, dim3((unsigned)(8 * rpx)), dim3(64), 0, stream, pruned, n, d, off, pairs, out, rpx);
    return hipGetLastError();
}

}  // namespace ann
