// Search of uint8 rows by whole clusters: the keys of a query against every row of its cluster come off the matrix cores
// into LDS, and the search then never reads a vector.
//
// A workgroup takes up to eight queries that stand next to each other in the execution order (most of them routed to one
// cluster).  Its wavefronts share the cluster's rows out among them, sixteen rows and eight queries per
// v_mfma_i32_16x16x64_i8, and leave a word per (query, row) in LDS; after one or two barriers every query is searched by a
// wavefront of its own.
//
// A word holds everything the search needs of a row: (key - smallest key of the cluster) << sh | row in the cluster << 1,
// bit 0 being the list's "expanded" mark.  A 32-bit compare of two words is the order by (key, id), and a list entry is one
// register per lane: a compare-exchange of the sorting networks is one lane move and one v_med3_u32, and a new word is
// inserted into the sorted list by one lane shift and one v_med3_u32 per register.  Taking a neighbour's word out of the
// table (one ds_wrxchg) leaves the mark "scored" behind: that one instruction is the visited test, the duplicate test
// and the key.
//
// What a word cannot hold ends the search of that query here: a graph edge that leaves the cluster (or the part of it that
// the table covers), and a key too far from the cluster's smallest that would have to enter a list that is not full.  The
// wavefront then searches the query anew with BeamSearch, which gathers rows.  ann_index_load counts how often that is to be
// expected (sample_clusters_kernel), and a call of which too many queries would is searched by gathering.
//
// Everything is exact integer arithmetic: ids, keys, rounds and counters are those of the gathering search.
//
// Measured (before: beam_search_kernel): 500 000 queries, clusters of 1 953 rows of 128 bytes, list of 184: 7.1 ms (9.35), 5 080 vector
// instructions a query (11 400); 10 000 queries, clusters of 1 000: 100 to 116 us (187); 100 queries, clusters of 100: 25 us (43).  What bounds it
// now: sixteen wavefronts of a compute unit find room in LDS with clusters of two thousand rows, and a round is a chain of two LDS round trips,
// one graph row from L2 and some 65 vector and 60 scalar instructions; the vector ALUs are 0.6 busy.  The making of the keys is 28 % of
// a wavefront's time (three or four tiles of rows in flight instead of two change nothing), waiting for the slowest of eight queries 10 %.  Tables of 16 bits per row
// (twice the wavefronts) need a second pass over the cluster for the smallest key, which cost what they saved (7.9 ms); loads of the
// rows in the order of the matrix operand, without the stage, kept the address units busy with 16 bytes at a time (1.7 ms for the
// making of the keys, 2.5 without).
#pragma once

#include "beam_search_kernel.h"

namespace ann {

struct ClusterParams {
    SearchParams s;
    int32_t group;         // queries per workgroup, 1 .. 4 * per_lane
    int32_t per_lane;      // queries whose keys a lane holds: 1 or 2
    int32_t cap;           // rows of a cluster that the table covers
    int32_t region_words;  // LDS words per query
    int32_t graph_words;   // LDS words for the cluster's graph rows (a workgroup of one query), or 0
};

constexpr int kMaxClusterGroup = 8;       // queries, and wavefronts, of a workgroup
constexpr int kClusterHeaderWords = 16;  // smallest key of each query's cluster
constexpr int kStageWords = 256;         // sixteen pieces of 64 bytes, on their way to the matrix instruction

// LDS words of a query in front of its table: compacted words and parents; while the keys are made, a wavefront's stage.
constexpr int cluster_table_at(int batch) { return batch + 64 > kStageWords ? batch + 64 : kStageWords; }
constexpr int kMaxClusterRows = 8192;

template <class Row, int LPL, int CPL>
struct ClusterSearch {
    static constexpr uint32_t kNone = 0xffffffffu;    // no entry; a row that has been scored
    static constexpr int kInsertMax = 9;              // at most this many new words are inserted one by one
    static constexpr int kTableAt = cluster_table_at(64 * CPL);

    const ClusterParams& cp;
    const SearchParams& p;
    const int lane;
    const LaneBits bits;
    uint32_t* const found;
    uint32_t* const parents;
    uint32_t* const table;
    const uint16_t* const graph;  // LDS: neighbours as rows of the cluster, or null
    int64_t lo;                   // the cluster's first row
    uint32_t size;                // rows in the table
    uint32_t base;                // smallest key
    int sh;                       // where the key starts in a word
    uint32_t L[LPL];
    uint32_t worst;  // list entry number itopk - 1, or `far` while the list is not full
    uint32_t far;    // words from here on are rows whose key is too far from the smallest (kNone aside)
    int n_parents = 0;

    __device__ __forceinline__ ClusterSearch(const ClusterParams& cp_, uint32_t* region, const uint16_t* graph_, int lane_)
        : cp(cp_), p(cp_.s), lane(lane_), bits(lane_), found(region), parents(region + 64 * CPL), table(region + kTableAt), graph(graph_) {}

    __device__ __forceinline__ static void lds_order() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    // Entries beyond itopk are left where they are: they never come back, and nobody looks at them.
    __device__ __forceinline__ void find_worst() {
        const int e = p.itopk - 1;
        uint32_t last = kNone;
#pragma unroll
        for (int r = 0; r < LPL; ++r) {
            const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)L[r], e & 63);
            if ((e >> 6) == r) last = w;
        }
        worst = min(last, far);
    }

    // Up to 64 words, one per lane from lane 64 - K on (kNone elsewhere), into the list.
    template <int K>
    __device__ __forceinline__ void merge(uint32_t w) {
        // descending, and the smallest last: entry e of the last register against word 63 - e leaves one run that rises and falls
        w = ~bits.template sort<K>(~w);
        L[LPL - 1] = min(L[LPL - 1], w);
        constexpr int P = LPL <= 1 ? 1 : LPL <= 2 ? 2 : LPL <= 4 ? 4 : 8;
        register_stages<P, P / 2>();
#pragma unroll
        for (int r = 0; r < LPL; ++r) L[r] = bits.template clean<5>(L[r]);
    }
    template <int P, int D>
    __device__ __forceinline__ void register_stages() {
        if constexpr (D >= 1) {
            constexpr int pad = P - LPL;
#pragma unroll
            for (int i = 0; i < P; ++i)
                if ((i & D) == 0 && i >= pad) {
                    const uint32_t a = L[i - pad], b = L[i + D - pad];
                    L[i - pad] = min(a, b);
                    L[i + D - pad] = max(a, b);
                }
            register_stages<P, D / 2>();
        }
    }
    // w uniform.  Every entry becomes the middle one of its predecessor, w and itself.
    __device__ __forceinline__ void insert(uint32_t w) {
        uint32_t wrapped = 0;
#pragma unroll
        for (int r = 0; r < LPL; ++r) {
            uint32_t below;
            if (r == 0) below = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)L[r], 0x138, 0xf, 0xf, true);  // wave_shr:1, 0 into lane 0
            else below = (uint32_t)__builtin_amdgcn_update_dpp((int)wrapped, (int)L[r], 0x138, 0xf, 0xf, false);
            if (r + 1 < LPL) wrapped = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)L[r], 0x13c, 0xf, 0xf, true);  // wave_ror:1
            L[r] = med3(below, w, L[r]);
        }
    }

    // Takes the words of the rows rel (one per lane and register; no row: any number that is none) out of the table and
    // brings those that can enter the list into it.  `foreign`: lanes whose graph edge leaves the table.  False: this query
    // needs the gathering search.
    __device__ __forceinline__ bool score(const uint32_t (&rel)[CPL], uint64_t foreign) {
        uint32_t w[CPL];
#pragma unroll
        for (int t = 0; t < CPL; ++t) {
            w[t] = kNone;
            if (rel[t] < size) w[t] = __hip_atomic_exchange(&table[rel[t]], kNone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        uint64_t keep[CPL];
        int m = 0;
#pragma unroll
        for (int t = 0; t < CPL; ++t) {
            keep[t] = __ballot(w[t] < worst);
            m += __builtin_popcountll(keep[t]);
        }
        if (worst == far) {  // uniform; a far row is of no account once the list is full
#pragma unroll
            for (int t = 0; t < CPL; ++t) foreign |= __ballot(w[t] - far < kNone - far);
        }
        if (foreign) return false;
        if (m <= kInsertMax) {
#pragma unroll
            for (int t = 0; t < CPL; ++t)
                for (uint64_t b = keep[t]; b;) {
                    const int j = __builtin_ctzll(b);
                    asm("s_bitset0_b64 %0, %1" : "+s"(b) : "s"(j));
                    insert((uint32_t)__builtin_amdgcn_readlane((int)w[t], j));
                }
        } else if (CPL == 1) {
            merge<64>(w[0] < worst ? w[0] : kNone);
        } else {
            int at = 0;
#pragma unroll
            for (int t = 0; t < CPL; ++t) {
                if (w[t] < worst) found[rank_below(keep[t], at)] = w[t];
                at += __builtin_popcountll(keep[t]);
            }
            lds_order();
            int from = 0;
            for (; m - from > 32; from += 64) merge<64>(from + lane < m ? found[from + lane] : kNone);
            const int at32 = from + lane - 32, at16 = from + lane - 48;
            if (m - from > 16) merge<32>(at32 >= from && at32 < m ? found[at32] : kNone);
            else if (m - from > 0) merge<16>(at16 >= from && at16 < m ? found[at16] : kNone);
            lds_order();
        }
        find_worst();
        return true;
    }

    // False: this query needs the gathering search.
    __device__ __forceinline__ bool run(int64_t qi) {
#pragma unroll
        for (int r = 0; r < LPL; ++r) L[r] = kNone;
        far = 0xffffffffu >> sh << sh;
        worst = far;
        parents[lane] = 0;
        uint32_t rel[CPL];
        {
            const int32_t c = p.route[qi];
            const bool known = (uint32_t)c < (uint32_t)p.n_clusters;
            const int64_t first = known ? p.cluster_offsets[c] : 0, end = known ? p.cluster_offsets[c + 1] : 0;
            uint64_t foreign = 0;
#pragma unroll
            for (int t = 0; t < CPL; ++t) {
                const int j = t * 64 + lane;
                rel[t] = kNone;
                bool out = false;
                if (j < p.n_entry && end > first) {
                    const uint64_t z = splitmix64_at(p.seed, (uint64_t)qi * (uint64_t)p.n_entry + (uint64_t)j);
                    const int32_t e = (int32_t)(first + (int64_t)(z % (uint64_t)(end - first)));
                    if ((uint32_t)e < (uint32_t)p.n) {
                        rel[t] = (uint32_t)e - (uint32_t)lo;
                        out = rel[t] >= size;
                    }
                }
                foreign |= __ballot(out);
            }
            if (!score(rel, foreign)) return false;
        }

        // lane s of register t reads neighbour (64 t + s) % degree of parent (64 t + s) / degree
        uint32_t parent_at[CPL], column[CPL];
#pragma unroll
        for (int t = 0; t < CPL; ++t) {
            const int s = t * 64 + lane;
            const int i = (int)(((uint32_t)s * p.degree_inv) >> 20);
            parent_at[t] = (uint32_t)(i < p.width ? i : p.width - 1);
            column[t] = (uint32_t)(s - i * p.degree);
        }
        uint64_t listed[LPL];  // lanes of entries below itopk
#pragma unroll
        for (int r = 0; r < LPL; ++r) listed[r] = __ballot(r * 64 + lane < p.itopk);
        const char* const rows = reinterpret_cast<const char*>(p.graph + lo * p.degree);
        const uint32_t row_mask = (1u << (sh - 1)) - 1u;
        int iters = 0;
        for (; iters < p.max_iters; ++iters) {
            int total = 0;
#pragma unroll
            for (int r = 0; r < LPL; ++r) {
                if (r == 0 || total < p.width) {  // uniform
                    const uint64_t b = __ballot((L[r] & 1u) == 0u) & listed[r];
                    const int rank = rank_below(b, total);
                    const bool take = __builtin_amdgcn_inverse_ballot_w64(__ballot(rank < p.width) & b);
                    if (take) parents[rank] = (L[r] >> 1) & row_mask;
                    L[r] |= take ? 1u : 0u;
                    total += __builtin_popcountll(b);
                }
            }
            if (total == 0) break;
            const int np = total < p.width ? total : p.width;
            n_parents += np;
            lds_order();
            // Lanes without a parent read for one that has been expanded before, whose neighbours' words are gone: from the second round
            // on that is what the places of `parents` beyond np hold.
            if (iters == 0) {
                const uint32_t first = parents[0];
                if (lane >= np) parents[lane] = first;
                lds_order();
            }
            uint64_t foreign = 0;
            uint32_t at[CPL];
#pragma unroll
            for (int t = 0; t < CPL; ++t) at[t] = (uint32_t)__umul24(parents[parent_at[t]], (uint32_t)p.degree) + column[t];
            if (graph) {
#pragma unroll
                for (int t = 0; t < CPL; ++t) rel[t] = graph[at[t]];
#pragma unroll
                for (int t = 0; t < CPL; ++t) foreign |= __ballot(rel[t] == 0xfffeu);
            } else {
                uint32_t most = 0;
#pragma unroll
                for (int t = 0; t < CPL; ++t) rel[t] = *reinterpret_cast<const uint32_t*>(rows + at[t] * 4u);
#pragma unroll
                for (int t = 0; t < CPL; ++t) {
                    rel[t] -= (uint32_t)lo;
                    most = max(most, rel[t]);
                }
                if (__any(most >= size)) {
#pragma unroll
                    for (int t = 0; t < CPL; ++t) foreign |= __ballot(rel[t] >= size) & __ballot(rel[t] + (uint32_t)lo < (uint32_t)p.n);
                }
            }
            if (!score(rel, foreign)) return false;
        }

        // first k entries
        const int64_t at = qi * p.k;
#pragma unroll
        for (int r = 0; r < LPL; ++r) {
            const int e = r * 64 + lane;
            if (e < p.k) {
                const bool have = L[r] != kNone;
                p.out_ids[at + e] = have ? (int32_t)((uint32_t)lo + ((L[r] >> 1) & row_mask)) : -1;
                p.out_dists[at + e] = have ? Row::key_to_output(base + (L[r] >> sh)) : Row::pad_output();
            }
        }
        if (p.out_counters) {
            int n_dist = 0;
            for (uint32_t i = (uint32_t)lane; i < size; i += 64) n_dist += table[i] == kNone ? 1 : 0;
            n_dist = group_sum<64>(n_dist, lane);
            if (lane == 0) {
                int32_t* c = p.out_counters + qi * 4;
                c[0] = iters;
                c[1] = n_dist;
                c[2] = n_parents;
                c[3] = 0;
            }
        }
        return true;
    }
};

typedef int cluster_v4i __attribute__((ext_vector_type(4)));

// The keys of the workgroup's queries [first, last) against the rows lo .. lo + size - 1, as they are, to their tables, and
// the smallest of each to head[].  KC: pieces of 64 bytes per row.  W: queries per lane (ClusterParams::per_lane).
//
// Bytes are shifted into int8, v = q ^ 0x80 and w = x ^ 0x80; bytes beyond the row's end count as shifted zeros.
//     L2:  sum (q - x)^2 = sum v^2 + sum w^2 - 2 sum v w
//     IP:  -q.x = -(sum v w + 128 (sum v + sum w) + 128^2 d)
// Lane l of the matrix instruction holds 16 bytes of operand row l % 16 and gets results for vector l % 16 and the operand
// rows 4 (l / 16) .. + 3 of the queries.  Query g W + r stands in operand row 4 g + r, so that with few queries all lanes still
// have results that count.
template <int KC, int W, bool L2, bool FULL>
__device__ __forceinline__ void cluster_keys(const ClusterParams& cp, uint32_t* head, uint32_t* tables, uint32_t* stage, int32_t query, int first, int last,
                                             int64_t lo, int size, int lane, int wave, int waves) {
    typedef cluster_v4i v4i;
    const SearchParams& p = cp.s;
    asm volatile("" : "+v"(lane));  // or the lane-dependent values of all instances would be kept in registers across the loop over runs
    const int col = lane & 15, grp = lane >> 4;
    const v4i zero = {(int)0x80808080, (int)0x80808080, (int)0x80808080, (int)0x80808080};
    auto term = [&](const v4i& w, int acc) {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_sdot4(w[i], L2 ? w[i] : 0x01010101, acc, false);
        return acc;
    };
    // sum over the four lanes that hold pieces of one row
    auto over_pieces = [&](int v) {
        auto s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        v = (int)s[0] + (int)s[1];
        s = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return (int)s[0] + (int)s[1];
    };
    v4i a[KC];
    int qterm = 0;
    {
        const int at = (col >> 2) * W + (col & 3);
        const int32_t q = __shfl(query, at < last ? at : last - 1);
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            const int off = c * 64 + grp * 16;
            a[c] = zero;
            if (FULL || c < KC - 1 || off < p.row_bytes) a[c] = *reinterpret_cast<const v4i*>(p.queries + (int64_t)q * p.row_bytes + off);
            a[c] ^= (int)0x80808080;
            qterm = term(a[c], qterm);
        }
        qterm = over_pieces(qterm);
        if (!L2) qterm = -128 * qterm - 16384 * p.row_bytes;
    }
    int add[W];  // what the key of the lane's query number r needs beyond the row's part and the product
    uint32_t least[W];
    uint32_t* out[W];
    bool wanted[W];
#pragma unroll
    for (int r = 0; r < W; ++r) {
        add[r] = __shfl(qterm, 4 * grp + r) ^ (L2 ? 0 : (int)0x80000000);
        least[r] = 0xffffffffu;
        wanted[r] = grp * W + r >= first && grp * W + r < last;
        out[r] = tables + (size_t)(grp * W + r) * cp.region_words;
    }
    // A lane loads piece lane % 4 of row lane / 4, so that a row's 64 bytes are one access, and the wavefront's stage in LDS
    // hands every lane the piece lane / 16 of row lane % 16 (piece i of row r in unit 4 r + (i ^ r / 4): the eight lanes that
    // read at a time then meet all banks).
    const uint8_t* const row0 = p.vectors + lo * p.row_stride;
    const uint32_t stride = (uint32_t)p.row_stride;
    const int tiles = (size + 15) >> 4;
    const int from_row = lane >> 2, from_piece = lane & 3;
    v4i* const put = reinterpret_cast<v4i*>(stage) + (from_row * 4 + (from_piece ^ (from_row >> 2)));
    const v4i* const get = reinterpret_cast<const v4i*>(stage) + (col * 4 + (grp ^ (col >> 2)));
    auto load = [&](v4i (&x)[KC], int tile) {
        const int row = tile * 16 + from_row;
        const uint8_t* const at = row0 + (uint64_t)(uint32_t)(row < size ? row : size - 1) * stride + from_piece * 16;
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            x[c] = zero;
            if (FULL || c < KC - 1 || c * 64 + from_piece * 16 < p.row_bytes) x[c] = *reinterpret_cast<const v4i*>(at + c * 64);
        }
    };
    auto keys = [&](const v4i (&x)[KC], int tile) {
        v4i w[KC];
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            *put = x[c] ^ (int)0x80808080;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            w[c] = *get;
            __builtin_amdgcn_wave_barrier();
        }
        v4i dot = {0, 0, 0, 0};
        int part = 0;
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            dot = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[c], w[c], dot, 0, 0, 0);
            part = term(w[c], part);
        }
        part = over_pieces(part);
        if (!L2) part = -128 * part;
        const int row = tile * 16 + col;
#pragma unroll
        for (int r = 0; r < W; ++r) {
            const uint32_t key = (uint32_t)(part + add[r]) - (uint32_t)dot[r] * (L2 ? 2u : 1u);
            if (wanted[r] && row < size) {
                out[r][row] = key;
                least[r] = min(least[r], key);
            }
        }
    };
    // D tiles of a wavefront in flight; beyond the last tile the cluster's last row is read again
    constexpr int D = 2;
    v4i x[D][KC];
#pragma unroll
    for (int u = 0; u < D; ++u) load(x[u], wave + u * waves);
    for (int tile = wave; tile < tiles; tile += D * waves) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            if (tile + u * waves < tiles) keys(x[u], tile + u * waves);
            load(x[u], tile + (u + D) * waves);
        }
    }
#pragma unroll
    for (int r = 0; r < W; ++r) {
        least[r] = min(least[r], row_xor<1>(least[r]));
        least[r] = min(least[r], row_xor<2>(least[r]));
        least[r] = min(least[r], row_xor<4>(least[r]));
        least[r] = min(least[r], row_xor<8>(least[r]));
        if (wanted[r] && col == 0) atomicMin(&head[grp * W + r], least[r]);
    }
}

template <int NCH, int W, bool L2>
__device__ __forceinline__ void cluster_keys_of(const ClusterParams& cp, uint32_t* head, uint32_t* tables, uint32_t* stage, int32_t query, int first, int last,
                                                int64_t lo, int size, int lane, int wave, int waves) {
    // rows of NCH pieces of 64 bytes, or fewer
#define ANN_KEYS(KC, FULL) cluster_keys<KC, W, L2, FULL>(cp, head, tables, stage, query, first, last, lo, size, lane, wave, waves)
    if (cp.s.row_bytes == NCH * 64) ANN_KEYS(NCH, true);
    else if (cp.s.row_bytes > (NCH - 1) * 64) ANN_KEYS(NCH, false);
    else ANN_KEYS(NCH - 1, false);
#undef ANN_KEYS
}

// Wavefronts per SIMD that the registers are to allow: for short clusters LDS allows more than four.
template <class Row>
constexpr int cluster_wavefronts(int lpl, int cpl) {
    return lpl == 8 ? 3 : Row::G * Row::NCH > 8 || cpl > 2 ? 4 : lpl == 4 ? 5 : 6;
}

template <class Row, int LPL, int CPL>
__global__ void __launch_bounds__(64 * kMaxClusterGroup, cluster_wavefronts<Row>(LPL, CPL)) cluster_search_kernel(const ClusterParams cp) {
    extern __shared__ uint32_t lds[];
    const SearchParams& p = cp.s;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), waves = (int)(blockDim.x >> 6);
    const int64_t b = blockIdx.x;
    const int64_t pos = ((b & 7) * p.q_per_xcd + (b >> 3)) * cp.group;  // q_per_xcd: workgroups per XCD
    if (pos >= p.q_count) return;                                        // the whole workgroup
    const int m = p.q_count - pos < cp.group ? (int)(p.q_count - pos) : cp.group;
    uint32_t* const head = lds;
    uint32_t* const regions = lds + kClusterHeaderWords;
    // behind the regions: stages of wavefronts that have no query of their own, the cluster's graph rows
    uint32_t* const stages = regions + cp.group * cp.region_words;
    uint32_t* const stage = wave < cp.group ? regions + wave * cp.region_words : stages + (wave - cp.group) * kStageWords;
    uint16_t* const graph = cp.graph_words ? reinterpret_cast<uint16_t*>(stages + (waves - cp.group) * kStageWords) : nullptr;
    int32_t query = 0, cluster = -1;
    if (lane < m) {
        query = p.order ? p.order[p.q_base + pos + lane] : (int32_t)(p.q_base + pos + lane);
        cluster = p.route[query];
    }
    if (threadIdx.x < kClusterHeaderWords) head[threadIdx.x] = 0xffffffffu;
    __syncthreads();

    typedef ClusterSearch<Row, LPL, CPL> Search;
    int64_t my_lo = 0;
    uint32_t my_size = 0;
    // the runs of queries of one cluster
    for (int first = 0; first < m;) {
        const int32_t c = __builtin_amdgcn_readlane(cluster, first);
        const uint64_t other = __ballot(lane >= first && lane < m && cluster != c);
        const int last = other ? __builtin_ctzll(other) : m;
        int64_t lo = 0, hi = 0;
        if ((uint32_t)c < (uint32_t)p.n_clusters) {
            lo = p.cluster_offsets[c];
            hi = p.cluster_offsets[c + 1];
        }
        lo = lo < 0 ? 0 : lo;
        hi = hi > p.n ? p.n : hi;
        const int size = hi <= lo ? 0 : hi - lo < cp.cap ? (int)(hi - lo) : cp.cap;
        const int w = cp.group == 1 ? 0 : wave;  // a workgroup of one query: all wavefronts work for it
        if (w >= first && w < last) {
            my_lo = lo;
            my_size = (uint32_t)size;
        }
        if (size > 0) {
            constexpr bool L2 = Row::kMetric == kL2;
            constexpr int NCH = Row::G * Row::NCH / 4;
            uint32_t* const tables = regions + Search::kTableAt;
            if (cp.per_lane == 1) cluster_keys_of<NCH, 1, L2>(cp, head, tables, stage, query, first, last, lo, size, lane, wave, waves);
            else cluster_keys_of<NCH, 2, L2>(cp, head, tables, stage, query, first, last, lo, size, lane, wave, waves);
            if (graph) {
                const int total = size * p.degree;
                for (int i = (int)threadIdx.x; i < total; i += (int)blockDim.x) {
                    const uint32_t id = (uint32_t)p.graph[lo * p.degree + i], rel = id - (uint32_t)lo;
                    graph[i] = rel < (uint32_t)size ? (uint16_t)rel : id < (uint32_t)p.n ? (uint16_t)0xfffe : (uint16_t)0xffff;
                }
            }
        }
        first = last;
    }
    __syncthreads();

    // keys into words
    const int mine = cp.group == 1 ? 0 : wave;
    Search s(cp, regions + (mine < m ? mine : 0) * cp.region_words, graph, lane);
    s.lo = my_lo;
    s.size = my_size;
    s.base = mine < m ? head[mine] : 0u;
    s.sh = 1 + (s.size > 1 ? 32 - __builtin_clz(s.size - 1) : 1);
    if (mine < m) {
        const uint32_t most = 0xffffffffu >> s.sh;
        const uint32_t step = 4 * (cp.group == 1 ? blockDim.x : 64u);
        for (uint32_t i = 4 * (cp.group == 1 ? threadIdx.x : (uint32_t)lane); i < s.size; i += step) {
            uint4* const at = reinterpret_cast<uint4*>(s.table + i);  // up to three words beyond the cluster's
            uint4 k = *at;
            k.x = min(k.x - s.base, most) << s.sh | i << 1;
            k.y = min(k.y - s.base, most) << s.sh | (i << 1) + 2;
            k.z = min(k.z - s.base, most) << s.sh | (i << 1) + 4;
            k.w = min(k.w - s.base, most) << s.sh | (i << 1) + 6;
            *at = k;
        }
    }
    if (cp.group == 1) __syncthreads();
    else Search::lds_order();
    if (wave >= m) return;
    const int64_t qi = __builtin_amdgcn_readlane(query, wave);
    if (!s.run(qi)) {
        int again = lane;
        asm volatile("" : "+v"(again));  // as in cluster_keys
        BeamSearch<Row, LPL, CPL, 0, false> g(p, regions + wave * cp.region_words, again, 0);
        g.run(qi);
    }
}

template <int METRIC, int G, int NCH>
hipError_t launch_cluster_search(const ClusterParams& p, int list_variant, unsigned grid, unsigned threads, size_t lds_bytes, hipStream_t stream);

#define ANN_CLUSTER_LIST(N, LPL, CPL)                                                                                           \
    case N:                                                                                                                     \
        hipLaunchKernelGGL((cluster_search_kernel<Row, LPL, CPL>), dim3(grid), dim3(threads), lds_bytes, stream, p);           \
        break;

#define ANN_DEFINE_CLUSTER_SEARCH(METRIC, G, NCH)                                                                               \
    template <>                                                                                                                 \
    hipError_t launch_cluster_search<METRIC, G, NCH>(const ClusterParams& p, int list_variant, unsigned grid, unsigned threads, \
                                                     size_t lds_bytes, hipStream_t stream) {                                    \
        using Row = RowOps<kU8, METRIC, G, NCH>;                                                                                \
        switch (list_variant) {                                                                                                 \
            ANN_CLUSTER_LIST(0, 1, 1)                                                                                           \
            ANN_CLUSTER_LIST(1, 2, 2)                                                                                           \
            ANN_CLUSTER_LIST(2, 3, 2)                                                                                           \
            ANN_CLUSTER_LIST(3, 4, 2)                                                                                           \
            ANN_CLUSTER_LIST(4, 4, 4)                                                                                           \
            ANN_CLUSTER_LIST(5, 4, 8)                                                                                           \
            ANN_CLUSTER_LIST(6, 8, 8)                                                                                           \
            default: return hipErrorInvalidValue;                                                                               \
        }                                                                                                                       \
        return hipGetLastError();                                                                                               \
    }

}  // namespace ann
