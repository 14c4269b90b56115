// Search by rank (see rank_search.h).
#include "rank_search.h"
#include "wave.h"

namespace ann {
namespace {

template <int CPL>
struct RankSearch {
    static constexpr int kHalo = kRankHalo, kTile = kRankTile;
    static constexpr uint32_t kNobody = 128u << 7;
    // A row on its way to its place is tagged with the last bits of its bucket.  Neighbours with one tag are of one bucket, or their
    // buckets are sixteen or more apart: then their keys are in order, and nothing comes of taking them for one.
    static constexpr int kTag = 12;
    static constexpr uint32_t kTagged = (1u << kTag) - 1u;
    static constexpr uint32_t kMostCrowded = kRankBitWords + 64 - 1;  // what the words of bits and parents hold
    static_assert(kMaxRankRows <= 1 << kTag, "a row and a place fit in front of the tag");
    static_assert(kRankBitWords + 64 + rank_row_words(kRankTiles * kRankTile) >= 2 * kRankCells, "room for `begins` in front of the buckets");

    const SearchParams& p;
    const uint32_t* const keys;  // of rows lo .. lo + size - 1
    const int lane;
    uint32_t* const bits;        // a bit per rank
    uint32_t* const parents;     // twice their ranks
    float2* const begins;        // where bits, parents and the first of by_rank are later: a cell's first bucket, and how many it has
    uint32_t* const list;        // where bits and parents are later: how many buckets are crowded, then (first place << 8 | rows) of each
    uint16_t* const by_rank;     // row of a rank below `near`
    uint16_t* const code_of;     // rank of a row, as (rank / 32) << 7 | rank % 32
    uint8_t* const buckets;      // where code_of is later
    int64_t lo;
    int size;
    int near;                    // ranks from here on are in the order of the buckets only
    float least, scale;          // the smallest key; cells of the range of the keys

    __device__ __forceinline__ RankSearch(const SearchParams& p_, uint32_t* lds, const uint32_t* keys_, int lane_)
        : p(p_), keys(keys_), lane(lane_), bits(lds), parents(lds + kRankBitWords), begins(reinterpret_cast<float2*>(lds)), list(lds),
          by_rank(reinterpret_cast<uint16_t*>(parents + 64)), code_of(by_rank + 2 * rank_row_words(p_.rank_places)), buckets(reinterpret_cast<uint8_t*>(code_of)) {}

    __device__ __forceinline__ static void lds_order() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // A key's cell and, behind the point, its place in it: 0 up to and without kRankCells.
    __device__ __forceinline__ float cell_of(float key) const {
        return __builtin_amdgcn_fmed3f((key - least) * scale, 0.0f, (float)kRankCells - 0x1p-17f);
    }
    // Every step rounds once, and the last one of a cell ends at most where the next cell's buckets begin: monotonous.
    __device__ __forceinline__ uint32_t bucket_at(float cell) const {
        const float2 at = begins[(uint32_t)cell];
        return (uint32_t)__builtin_fmaf(__builtin_amdgcn_fractf(cell), at.y, at.x);
    }
    // Chunks of 512 rows, a register of 64 each; `work(first register, lane)` for those that there are.  (With a copy of the lane number
    // that the compiler cannot see through: it would keep the 48 row numbers in registers from chunk to chunk.)
    static constexpr int kChunk = 8, kChunks = kMaxRankRows / (64 * kChunk);
    template <class Work>
    __device__ __forceinline__ void each_chunk(Work work) const {
#pragma unroll
        for (int c = 0; c < kChunks; ++c)
            if (c * 64 * kChunk < size) {  // uniform
                int at = lane;
                asm volatile("" : "+v"(at));
                work(c * kChunk, at);
            }
    }

    // Buckets of more rows than the tiles settle (kHalo + 1: a row of such a bucket passes kHalo others at most).  `words`: in a byte each, where a lane's buckets begin among its rows.
    __device__ __forceinline__ void list_crowded(const uint32_t* words, uint32_t first, uint32_t rows, uint32_t stored) {
#pragma unroll 1
        for (int i = 0; i < 16; ++i) {
            uint32_t from = words[lane * 16 + i];
            const uint32_t after = i < 15 ? words[lane * 16 + i + 1] : rows;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t start = from & 0xffu, end = (j < 3 ? from >> 8 : after) & 0xffu;
                if (end - start > (uint32_t)(kHalo + 1) && first + start < stored) {
                    const uint32_t at = __hip_atomic_fetch_add(list, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (at < kMostCrowded) list[1 + at] = (first + start) << 8 | (end - start);
                }
                from >>= 8;
            }
        }
    }
    // Puts their rows in order, each by counting those below it, before the tiles are gone through.
    __device__ __forceinline__ void settle_crowded(int stored) {
        const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)list[0]);
        for (uint32_t i = 0; i < n; ++i) {
            const uint32_t which = (uint32_t)__builtin_amdgcn_readfirstlane((int)list[1 + i]);
            const int start = (int)(which >> 8), rows = (int)(which & 0xffu);
            if (start + rows > stored) {  // the last one, which not all places are kept of
                near = start;
                continue;
            }
            uint32_t row[4];
            uint64_t at[4];
            int below[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                row[c] = by_rank[start + min(c * 64 + lane, rows - 1)];
                below[c] = 0;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c * 64 < rows) at[c] = (uint64_t)keys[row[c] & kTagged] << 32 | row[c];
            if (rows <= 64) {
                // copies of one row mostly are in order
                const uint64_t next = (uint64_t)next_lane((uint32_t)(at[0] >> 32), 0xffffffffu) << 32 | next_lane((uint32_t)at[0], 0xffffffffu);
                if (!__any(lane < rows - 1 && next < at[0])) continue;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll 1
                for (int l = 0; l < min(rows - c * 64, 64); ++l) {
                    const uint64_t other = lane_word(at[c], l);
#pragma unroll
                    for (int o = 0; o < 4; ++o)
                        if (o * 64 < rows) below[o] += other < at[o] ? 1 : 0;
                }
            lds_order();
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c * 64 + lane < rows) {
                    by_rank[start + below[c]] = (uint16_t)row[c];
                    code_of[row[c] & kTagged] = code(start + below[c]);  // `near` may come to lie among them
                }
            lds_order();
        }
    }

    __device__ __forceinline__ bool rank() {
        uint32_t key[kChunk * kChunks];  // of row 64 t + lane
        each_chunk([&](int t0, int lane) {
#pragma unroll
            for (int t = t0; t < t0 + kChunk; ++t)
                if (t * 64 < size) key[t] = keys[t * 64 + lane];  // a query's row of the table is whole 64s
        });
        // the range of the keys, in cells
        const uint32_t some = (uint32_t)__builtin_amdgcn_readfirstlane((int)key[0]);
        uint32_t lowest = some, highest = some;
        each_chunk([&](int t0, int lane) {
            if ((t0 + kChunk) * 64 > size) {  // uniform
#pragma unroll
                for (int t = t0; t < t0 + kChunk; ++t) key[t] = lane < size - t * 64 ? key[t] : some;
            }
#pragma unroll
            for (int t = t0; t < t0 + kChunk; ++t) {
                lowest = min(lowest, key[t]);
                highest = max(highest, key[t]);
            }
        });
        least = ordered_to_float(~wave_max(~lowest));
        const float range = ordered_to_float(wave_max(highest)) - least;
        scale = (float)kRankCells / range;
        // (also keys that are no numbers, or all the same)
        if (!(range < 1e30f && scale < 1e30f)) return false;
        uint32_t* const counts = bits;
        reinterpret_cast<uint2*>(counts)[lane] = make_uint2(0u, 0u);
        lds_order();
        each_chunk([&](int t0, int lane) {
#pragma unroll
            for (int t = t0; t < t0 + kChunk; ++t) {
                const float cell = cell_of(ordered_to_float(key[t]));
                key[t] = __builtin_bit_cast(uint32_t, cell);
                if (lane < size - t * 64) __hip_atomic_fetch_add(&counts[(uint32_t)cell], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        });
        lds_order();
        {
            const uint2 held = reinterpret_cast<const uint2*>(counts)[lane];
            const uint32_t upto = wave_inclusive_sum(held.x + held.y);
            const float each = (float)(kRankBuckets - 1) / (float)size;
            const float first = (float)(upto - held.y - held.x) * each, second = (float)(upto - held.y) * each, end = (float)upto * each;
            reinterpret_cast<float4*>(begins)[lane] = make_float4(first, second - first, second, end - second);
        }
        lds_order();

        // how many rows every bucket holds; the cell gives way to the bucket
#pragma unroll
        for (int i = 0; i < kRankBuckets / 1024; ++i) reinterpret_cast<uint4*>(buckets)[i * 64 + lane] = make_uint4(0, 0, 0, 0);
        lds_order();
        uint32_t* const words = reinterpret_cast<uint32_t*>(buckets);
        each_chunk([&](int t0, int lane) {
#pragma unroll
            for (int t = t0; t < t0 + kChunk; ++t) {
                key[t] = bucket_at(__builtin_bit_cast(float, key[t]));
                if (lane < size - t * 64)
                    __hip_atomic_fetch_add(&words[key[t] >> 2], 1u << (8u * key[t] & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        });
        lds_order();
        // a lane's 64 buckets: where each begins among the lane's rows
        uint32_t w[16];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 v = reinterpret_cast<const uint4*>(buckets)[lane * 4 + i];
            w[4 * i] = v.x;
            w[4 * i + 1] = v.y;
            w[4 * i + 2] = v.z;
            w[4 * i + 3] = v.w;
        }
        uint32_t crowded = 0;  // the high bit of a byte of more than kHalo + 1 rows (and now and then of the one above it)
#pragma unroll
        for (int i = 0; i < 16; ++i) crowded |= w[i] | (w[i] + 0x01010101u * (127u - (kHalo + 1)));
        const bool any_crowded = __any((crowded & 0x80808080u) != 0u);
        if (any_crowded && lane == 0) list[0] = 0u;
        uint32_t before = 0, rows = 0;  // the rows so far, in every byte; their number
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const uint32_t pairs = w[i] + (w[i] << 8), upto = pairs + (pairs << 16);  // sums of up to four bytes, exact where they fit one
            rows = __builtin_amdgcn_sad_u8(w[i], 0u, rows);
            w[i] = (upto << 8) + before;
            before = __builtin_amdgcn_perm(0u, rows, 0u);  // the lowest byte four times
        }
        // more than 255 rows in one bucket show as a wrong total, more in a lane's as such
        const uint32_t upto = wave_inclusive_sum(rows);
        if (__ballot(rows > 255u) || __builtin_amdgcn_readlane((int)upto, 63) != size) return false;
        const uint32_t first = upto - rows;
        const int stored = min(size, p.rank_places + kHalo);
#pragma unroll
        for (int i = 0; i < 4; ++i) reinterpret_cast<uint4*>(buckets)[lane * 4 + i] = make_uint4(w[4 * i], w[4 * i + 1], w[4 * i + 2], w[4 * i + 3]);
        lds_order();
        if (any_crowded) {
            list_crowded(words, first, rows, (uint32_t)stored);
            lds_order();
            if ((uint32_t)__builtin_amdgcn_readfirstlane((int)list[0]) > kMostCrowded) return false;
        }
        // rows in the order of their buckets; the bucket gives way to the place, and a tag
        each_chunk([&](int t0, int lane) {
            constexpr int U = 4;
#pragma unroll
            for (int t1 = t0; t1 < t0 + kChunk; t1 += U) {
                uint32_t old[U], base[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t b = key[t1 + u];
                    old[u] = 0;
                    if (lane < size - (t1 + u) * 64)
                        old[u] = __hip_atomic_fetch_add(&words[b >> 2], 1u << (8u * b & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    base[u] = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(b >> 4 & 0xfcu), (int)first);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t b = key[t1 + u];
                    key[t1 + u] = b << kTag | (base[u] + __builtin_amdgcn_ubfe(old[u], 8u * b & 31u, 8));
                    asm volatile("" : "+v"(key[t1 + u]));  // here, not at its use: there it would keep three registers
                }
            }
        });
        lds_order();
        each_chunk([&](int t0, int lane) {
#pragma unroll
            for (int t = t0; t < t0 + kChunk; ++t) {
                if (lane < size - t * 64) {
                    const uint32_t row = (uint32_t)(t * 64 + lane), at = key[t] & kTagged;
                    code_of[row] = code((int)at);
                    if ((int)at < stored) by_rank[at] = (uint16_t)((key[t] & ~kTagged) | row);
                }
            }
        });
        if (lane == 0) code_of[size] = (uint16_t)kNobody;
        lds_order();
        near = size;
        if (any_crowded) settle_crowded(stored);
        // Tiles of places.  The middle lanes of a tile see all places that a row may have to pass.  Tiles are read before those in front
        // of them are written.
        constexpr int N = kRankTiles;
        uint32_t next_row[N], next_key[N];
        auto read = [&](int t0) {
#pragma unroll
            for (int u = 0; u < N; ++u) next_row[u] = by_rank[min(max((t0 + u) * kTile - kHalo + lane, 0), stored - 1)];
#pragma unroll
            for (int u = 0; u < N; ++u) next_key[u] = keys[next_row[u] & kTagged];
        };
        read(0);
        const int places = min(size, p.rank_places);
        for (int t0 = 0; t0 * kTile < places; t0 += N) {
            uint32_t row[N], at_key[N], other[N];
            uint64_t same[N], run[N], more = 0;
            int move[N];
#pragma unroll
            for (int u = 0; u < N; ++u) {
                row[u] = next_row[u];
                at_key[u] = other[u] = next_key[u];
            }
            if ((t0 + N) * kTile < places) read(t0 + N);
            lds_order();
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int at = (t0 + u) * kTile - kHalo + lane;
                const uint32_t b = at >= 0 && at < stored ? row[u] >> kTag : 0x80000000u + (uint32_t)lane;
                same[u] = run[u] = __ballot(b == next_lane(b, 0xffffffffu));  // as the next lane's
                more |= run[u];
                move[u] = 0;
            }
            for (int d = 1; more; ++d) {  // uniform
                if (d > kHalo) break;  // a crowded bucket, which is in order
                uint64_t swap[N], equal[N], ties = 0;
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    other[u] = next_lane(other[u], 0u);
                    swap[u] = __ballot(other[u] < at_key[u]) & run[u];
                    equal[u] = __ballot(other[u] == at_key[u]) & run[u];
                    ties |= equal[u];
                }
                if (ties) {  // uniform
#pragma unroll
                    for (int u = 0; u < N; ++u) {
                        const uint32_t other_row = (uint32_t)__builtin_amdgcn_ds_bpermute((lane + d) << 2, (int)row[u]);
                        swap[u] |= equal[u] & __ballot(other_row < row[u]);
                    }
                }
                more = 0;
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    move[u] += __builtin_amdgcn_inverse_ballot_w64(swap[u]) ? 1 : 0;
                    move[u] -= __builtin_amdgcn_inverse_ballot_w64(swap[u] << d) ? 1 : 0;
                    run[u] &= same[u] >> d;
                    more |= run[u];
                }
            }
            if (size > places && (t0 + N) * kTile >= places) {
                // the last tile ends where a bucket does
                const uint64_t begins = ~(same[N - 1] << 1) & ((1ull << (64 - kHalo)) - 1ull);
                near = min(near, (t0 + N - 1) * kTile - kHalo + 63 - __builtin_clzll(begins));
            }
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int at = (t0 + u) * kTile - kHalo + lane;
                if (lane >= kHalo && lane < 64 - kHalo && at < near) by_rank[at + move[u]] = (uint16_t)(row[u] & kTagged);
            }
        }
        lds_order();
        for (int r0 = 0; r0 < near; r0 += 64 * kChunk) {
            uint32_t row[kChunk];
#pragma unroll
            for (int u = 0; u < kChunk; ++u) row[u] = by_rank[min(r0 + u * 64 + lane, near - 1)];
#pragma unroll
            for (int u = 0; u < kChunk; ++u)
                if (r0 + u * 64 + lane < near) code_of[row[u]] = code(r0 + u * 64 + lane);
        }
        lds_order();
        return true;
    }
    static __device__ __forceinline__ uint16_t code(int rank) { return (uint16_t)((uint32_t)(rank >> 5) << 7 | (uint32_t)(rank & 31)); }

    // The rows rel are scored; a number from `size` on is no row.
    __device__ __forceinline__ void mark(const uint32_t (&rel)[CPL]) {
        uint32_t code[CPL];
#pragma unroll
        for (int t = 0; t < CPL; ++t) code[t] = code_of[min(rel[t], (uint32_t)size)];
#pragma unroll
        for (int t = 0; t < CPL; ++t) {
            uint32_t* const word = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(bits) + (code[t] >> 5));
            __hip_atomic_fetch_or(word, 1u << (code[t] & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        lds_order();
    }
    static __device__ __forceinline__ uint64_t lane_word(uint64_t v, int from) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, from);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), from);
        return (uint64_t)hi << 32 | lo;
    }

    // False: this query needs BeamSearch.
    __device__ __forceinline__ bool run(int64_t qi) {
        const int32_t c = p.route[qi];
        if ((uint32_t)c >= (uint32_t)p.n_clusters) return false;
        lo = p.cluster_offsets[c];
        const int64_t end = p.cluster_offsets[c + 1];
        if (lo < 0 || end > p.n || end <= lo || end - lo > p.rank_rows) return false;
        size = (int)(end - lo);
        if (!rank()) return false;

        for (int i = lane; i < kRankBitWords; i += 64) bits[i] = 0u;
        lds_order();
        uint32_t rel[CPL];
#pragma unroll
        for (int t = 0; t < CPL; ++t) {
            const int j = t * 64 + lane;
            rel[t] = 0xffffffffu;
            if (j < p.n_entry) rel[t] = (uint32_t)(splitmix64_at(p.seed, (uint64_t)qi * (uint64_t)p.n_entry + (uint64_t)j) % (uint64_t)size);
        }
        mark(rel);

        // lane s of register t reads neighbour (64 t + s) % degree of parent (64 t + s) / degree
        uint32_t parent_at[CPL], column[CPL];
#pragma unroll
        for (int t = 0; t < CPL; ++t) {
            const int s = t * 64 + lane;
            const int i = (int)(((uint32_t)s * p.degree_inv) >> 20);
            parent_at[t] = (uint32_t)(i < p.width ? i : p.width - 1);
            column[t] = 4u * (uint32_t)(s - i * p.degree);
        }
        const uint32_t row_bytes = 4u * (uint32_t)p.degree;
        const char* const rows = reinterpret_cast<const char*>(p.graph + lo * p.degree);
        uint64_t done = 0;  // this lane's ranks that have been expanded
        int iters = 0, n_parents = 0;
        for (; iters < p.max_iters; ++iters) {
            const uint64_t scored = *reinterpret_cast<const uint64_t*>(bits + 2 * lane);
            const uint64_t open = scored & ~done;
            const uint64_t any_open = __ballot(open != 0);
            // The first `width` open entries.  A rank below itopk is in the list whatever has been scored; where the last one taken
            // lies beyond, the list's end is looked for and they are taken again.
            bool again = false;
            int np, last, edge = 64;  // the list ends with the bits in_edge of lane `edge`
            uint64_t in_edge = ~0ull, closed;
            for (;;) {  // uniform, twice at most
                uint64_t lanes = edge < 64 ? any_open & (2ull * (1ull << edge) - 1ull) : any_open;
                np = last = 0;
                closed = done;
                while (lanes) {
                    const int l = __builtin_ctzll(lanes);
                    lanes &= lanes - 1;
                    const uint64_t word = lane_word(open, l) & (l == edge ? in_edge : ~0ull);
                    const int at = rank_below(word, np);
                    const uint64_t taken = __ballot(at < p.width) & word;
                    if (__builtin_amdgcn_inverse_ballot_w64(taken)) parents[at] = (uint32_t)(2 * (l * 64 + lane));
                    if (taken) last = l * 64 + 63 - __builtin_clzll(taken);
                    closed |= lane == l ? taken : 0ull;
                    np += __builtin_popcountll(taken);
                    if (np >= p.width) break;
                }
                if (last < p.itopk || edge < 64) break;
                const int count = __builtin_popcountll(scored);
                const int upto = (int)wave_inclusive_sum((uint32_t)count);
                const uint64_t beyond = __ballot(upto >= p.itopk);
                if (!beyond) break;
                edge = __builtin_ctzll(beyond);
                const int left = p.itopk - (__builtin_amdgcn_readlane(upto, edge) - __builtin_amdgcn_readlane(count, edge));
                const uint64_t word = lane_word(scored, edge);
                const uint64_t cut = __ballot(rank_below(word) == left - 1) & word;  // one bit
                in_edge = cut | (cut - 1);
                if (last <= edge * 64 + __builtin_ctzll(cut)) break;
                again = true;
            }
            done = closed;
            if (np == 0) break;
            if (last >= near) return false;
            n_parents += np;
            lds_order();
            if (iters == 0 || again) {
                // Lanes without a parent read for one that is expanded anyhow, which marks nothing new: their places hold those of earlier
                // rounds, unless there was none or more had been taken at first.
                const uint32_t first = parents[0];
                if (lane >= np) parents[lane] = first;
                lds_order();
            }
            uint32_t at[CPL];
#pragma unroll
            for (int t = 0; t < CPL; ++t) at[t] = parents[parent_at[t]];
#pragma unroll
            for (int t = 0; t < CPL; ++t) {
                const uint32_t row = *reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(by_rank) + at[t]);
                at[t] = (uint32_t)__umul24(row, row_bytes) + column[t];
            }
#pragma unroll
            for (int t = 0; t < CPL; ++t) rel[t] = *reinterpret_cast<const uint32_t*>(rows + at[t]);
            uint32_t most = 0;
#pragma unroll
            for (int t = 0; t < CPL; ++t) {
                rel[t] -= (uint32_t)lo;
                most = max(most, rel[t]);
            }
            if (__any(most >= (uint32_t)size)) {
                bool foreign = false;
#pragma unroll
                for (int t = 0; t < CPL; ++t) foreign |= rel[t] >= (uint32_t)size && rel[t] + (uint32_t)lo < (uint32_t)p.n;
                if (__any(foreign)) return false;
            }
            mark(rel);
        }

        // first k entries
        const uint64_t scored = *reinterpret_cast<const uint64_t*>(bits + 2 * lane);
        const int total = __builtin_amdgcn_readlane((int)wave_inclusive_sum((uint32_t)__builtin_popcountll(scored)), 63);
        int32_t* const out_ids = p.out_ids + qi * p.k;
        uint32_t* const out_dists = p.out_dists + qi * p.k;
        uint64_t lanes = __ballot(scored != 0);
        for (int done_k = 0; lanes && done_k < p.k;) {  // uniform
            const int l = __builtin_ctzll(lanes);
            lanes &= lanes - 1;
            const uint64_t word = lane_word(scored, l);
            const int at = rank_below(word, done_k);
            const bool take = __builtin_amdgcn_inverse_ballot_w64(word) && at < p.k;
            if (l * 64 + 63 - __builtin_clzll(__ballot(take) | 1ull) >= near) return false;
            if (take) {
                const uint32_t row = by_rank[l * 64 + lane];
                out_ids[at] = (int32_t)((uint32_t)lo + row);
                out_dists[at] = __builtin_bit_cast(uint32_t, ordered_to_float(keys[row]));
            }
            done_k += __builtin_popcountll(word);
        }
        for (int e = total + lane; e < p.k; e += 64) {
            out_ids[e] = -1;
            out_dists[e] = 0x7f800000u;
        }
        if (p.out_counters && lane == 0) {
            int32_t* const counters = p.out_counters + qi * 4;
            counters[0] = iters;
            counters[1] = total;
            counters[2] = n_parents;
            counters[3] = 0;
        }
        return true;
    }
};

template <int CPL>
__global__ void __launch_bounds__(64, 5) rank_search_kernel(const SearchParams p) {
    extern __shared__ uint32_t lds[];
    const int64_t b = blockIdx.x;
    const int64_t local = (b & 7) * p.q_per_xcd + (b >> 3);
    if (local >= p.q_count) return;  // the whole workgroup
    RankSearch<CPL> s(p, lds, p.table + local * p.table_stride, lane_id());
    if (!s.run(p.order[p.q_base + local]) && s.lane == 0) p.again[1 + atomicAdd(p.again, 1)] = (int32_t)local;
}

}  // namespace

hipError_t launch_rank_search(const SearchParams& p, int cpl, unsigned grid, size_t lds_bytes, hipStream_t stream) {
#define ANN_RANK(CPL) \
    if (cpl == CPL) hipLaunchKernelGGL((rank_search_kernel<CPL>), dim3(grid), dim3(64), lds_bytes, stream, p);
    ANN_RANK(2) ANN_RANK(4) ANN_RANK(8)
#undef ANN_RANK
    return hipGetLastError();
}

}  // namespace ann
