// Routing: for each query the route_c nearest centroids under (key, cluster index).
// Single-GPU form of Fantasy's stage 1 ("K-means as classifier", Sec. 3.1): it only
// decides in which clusters a query's entry nodes are drawn.
//
// One wavefront per query.  Centroid rows are scored exactly like vector rows
// (same RowOps), each lane group walking its own stride of centroids and keeping
// its route_c best in registers; the groups' lists are then sorted together.
//
// Float rows that are an odd multiple of 16 bytes: the matrix cores have listed the few best centroids of every query by
// score (route_mfma.hip), |c|^2 - 2 q.c for L2, which rounds larger sums than the key here does.  Where the listed scores are
// further apart than that rounding, they are the answer; else the listed rows are scored here, and should even the
// last listed one be too near, all rows are, so the result is always this kernel's own.
// Nearest two of 1 000 centroids, 30 000 fp16 rows of 400 bytes: 83 us, with all rows scored here 851 us.
#pragma once

#include "row_ops.h"

namespace ann {

constexpr int kMaxRouteC = 8;

struct RouteParams {
    const uint8_t* centroids;  // n_clusters dense rows of row_bytes
    int32_t n_clusters;
    int32_t row_bytes;
    const uint8_t* queries;
    int64_t nq;
    int32_t route_c;
    int32_t* out;  // nq * route_c
    const uint64_t* words;  // [query][slice][route_c + route_spare_words] (ordered score << 32 | cluster), ascending per slice; or null
    int32_t slices;
    const float* largest;   // the largest |c|^2 (with words); fp32: in front of it a word that is not 0 if there are extreme centroids
};

// Listed beyond the route_c that are wanted.  If even the last one is too near, the query's wavefront walks all centroids, and a few such
// walks are the launch: with two spare words one of some thousand queries did (6 400 fp16 rows of 1 008 bytes, 400 centroids, nearest
// four: 129 us, with three 59), and scores of long fp32 rows have to be further apart (settle_route).
constexpr int kMaxSpareWords = 4;
__host__ __device__ constexpr int route_spare_words(bool f32, int row_bytes, int route_c) { return f32 && row_bytes > 512 && route_c > 2 ? 4 : 3; }
constexpr int kMaxRouteSlices = 64;

// What the listed words leave to do: nothing (the first route_c are in list[]), score the listed centroids, or all.
enum RouteRest { kRouteDone, kRouteListed, kRouteAll };

template <class Row>
__device__ __forceinline__ RouteRest settle_route(const RouteParams& p, const Row& row, int64_t qi, int lane, uint32_t* list) {
    const int each = p.route_c + route_spare_words(Row::kDtype == kF32, p.row_bytes, p.route_c), total = p.slices * each;
    constexpr int kWords = (kMaxRouteSlices * (kMaxRouteC + kMaxSpareWords) + 63) / 64;
    uint64_t w[kWords];
#pragma unroll
    for (int i = 0; i < kWords; ++i) w[i] = i * 64 + lane < total ? p.words[qi * total + i * 64 + lane] : ~0ull;
    float sum = 0.0f;
#pragma unroll
    for (int c = 0; c < Row::NCH; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (Row::kDtype == kF16) {
                const half2_t h = __builtin_bit_cast(half2_t, (uint32_t)row.q[c][i]);
                sum = __builtin_fmaf((float)h.x, (float)h.x, __builtin_fmaf((float)h.y, (float)h.y, sum));
            } else {
                const uint32_t bits = row.q[c][i];
                const float f = __builtin_bit_cast(float, bits);
                sum = __builtin_fmaf(f, f, sum);
            }
        }
    // How far apart two scores have to be for the keys to be in their order (u = 2^-24, a rounding to nearest; S = |q|^2 + |c|^2, at
    // least twice the sum of all |q_i c_i|, and half of |q - c|^2):
    //   * q.c on the matrix cores.  An instruction takes its sixteen products in two groups of eight: it lines a group up with its
    //     largest, cuts the others off at 2^-24 of that, and adds the group to the sum with one rounding (so it was found; in 50 million
    //     trials no instruction was off by more than 5.8 u of its products' and the sum's magnitudes).  The cuts are at most 7 u of all
    //     products; a rounding is counted as 2 u of the sum of magnitudes, two of them per 16 elements of fp16, twelve of fp32, whose parts'
    //     products add up to at most 1.02 of theirs and leave u out.  Twice that in the score:
    //         fp16 u S (0.25 dim + 11), fp32 u S (1.55 dim + 33)
    //     (where extreme values are left to the fp32 instruction: at most two roundings of 2 u per element, fp32 u S 4 dim)
    //   * |c|^2, summed in a chain, and the score's own rounding:                             u S (dim + 2)
    //   * the key: differences, squares, a lane's chain and five levels of the group's sum:   2 u S (elements per lane + 8)
    // Each of the two scores and of the two keys may be off that way.  1.01 is for products of roundings, and for those of S.
    // (A bound on ordinary sums, (dim + 64) u S, let rows whose squares all round the same way change places: (1, 0.999 * 2^-12, ..)
    // and (1, 1.0001 * 2^-12, .., 0, ..) seen from zero, 252 fp32 elements.)
    const float scale = group_sum<Row::G>(sum, lane) + *p.largest;
    constexpr bool kHalf = Row::kDtype == kF16;
    constexpr int kSize = kHalf ? 2 : 4, kPerLane = Row::NCH * 16 / kSize;
    const float dim = (float)(p.row_bytes / kSize);
    bool extreme = false;  // (of queries only large ones count: next to |c|^2 the products of tiny ones are nothing)
    if constexpr (!kHalf) extreme = scale >= 0x1p113f || __builtin_bit_cast(uint32_t, p.largest[-1]) != 0u;
    const float apart = 1.01f * scale * (2.0f * ((kHalf ? 1.25f : extreme ? 5.0f : 2.55f) * dim + (kHalf ? 14.0f : 36.0f) + 2.0f * (kPerLane + 8)) * 0x1p-24f);
    // (not a number: all; so large that a key may be infinite, where every score is finite: all)
    RouteRest rest = scale >= 0x1p-60f && scale <= 0x1p125f ? kRouteDone : kRouteAll;
    float before = 0.0f, wanted = 0.0f;
    for (int r = 0; r < each; ++r) {
        uint64_t least = ~0ull;
#pragma unroll
        for (int i = 0; i < kWords; ++i) least = w[i] < least ? w[i] : least;
        for (int d = 1; d < 64; d <<= 1) {
            const uint64_t o = __shfl_xor((unsigned long long)least, d);
            least = o < least ? o : least;
        }
#pragma unroll
        for (int i = 0; i < kWords; ++i) w[i] = w[i] == least ? ~0ull : w[i];
        const uint32_t c = (uint32_t)least;
        if (lane == 0) list[r] = c;
        if (c >= (uint32_t)p.n_clusters) {  // no centroid: fine if there is none left, else a score without order is missing
            if (r < p.n_clusters) rest = kRouteAll;
            continue;
        }
        const float score = ordered_to_float((uint32_t)(least >> 32));
        if (r >= 1 && r <= p.route_c && !(score - before > apart) && rest == kRouteDone) rest = kRouteListed;
        before = score;
        if (r == p.route_c - 1) wanted = score;
        // a centroid that is not listed scores no less than the last one that is
        if (r == each - 1 && !(score - wanted > apart)) rest = kRouteAll;
    }
    return rest;
}

template <class Row>
__global__ void __launch_bounds__(64) route_kernel(const RouteParams p) {
    constexpr int PR = (64 / Row::G * kMaxRouteC + 63) / 64;  // registers per lane of the final sort
    __shared__ uint64_t pool[64 * PR];
    __shared__ uint32_t list[kMaxRouteC + kMaxSpareWords];
    const int lane = lane_id();
    const int64_t qi = blockIdx.x;
    if (qi >= p.nq) return;
    Row row;
    row.load_query(p.queries + qi * (int64_t)p.row_bytes, p.row_bytes, lane);
    constexpr int G = Row::G, NCH = Row::NCH, RPS = 64 / G;
    const int grp = lane / G;

    bool listed = false;
    if constexpr (Row::kDtype != kU8) {
        if (p.words) {
            const RouteRest rest = settle_route(p, row, qi, lane, list);
            __syncthreads();
            if (rest == kRouteDone) {
                if (lane < p.route_c) p.out[qi * p.route_c + lane] = (int32_t)list[lane];
                return;
            }
            listed = rest == kRouteListed;
        }
    }

    uint64_t best[kMaxRouteC];
#pragma unroll
    for (int i = 0; i < kMaxRouteC; ++i) best[i] = kInfKey;

    const int rows = listed ? p.route_c + route_spare_words(Row::kDtype == kF32, p.row_bytes, p.route_c) : p.n_clusters;
    for (int c0 = 0; c0 < rows; c0 += RPS) {
        const int at = c0 + grp;
        const int c = !listed || at >= rows ? at : (int)list[at];
        const bool live = at < rows && (uint32_t)c < (uint32_t)p.n_clusters;
        u32x4 x[NCH];
        row.load_row(x, row.lane_piece(p.centroids + (int64_t)(live ? c : 0) * p.row_bytes), live);
        const uint32_t okey = row.key(x, lane);
        uint64_t cand = live ? (((uint64_t)okey << 32) | (uint32_t)c) : kInfKey;
        if (__any(cand < best[kMaxRouteC - 1])) {
#pragma unroll
            for (int i = 0; i < kMaxRouteC; ++i) {  // insertion into the ascending list
                const uint64_t lo = cand < best[i] ? cand : best[i];
                cand = cand < best[i] ? best[i] : cand;
                best[i] = lo;
            }
        }
    }
    // RPS groups x kMaxRouteC entries: sort them in one go
#pragma unroll
    for (int r = 0; r < PR; ++r) pool[r * 64 + lane] = kInfKey;
    __syncthreads();
    if (row.lg == 0) {
#pragma unroll
        for (int i = 0; i < kMaxRouteC; ++i) pool[grp * kMaxRouteC + i] = best[i];
    }
    __syncthreads();
    uint64_t v[PR];
#pragma unroll
    for (int r = 0; r < PR; ++r) v[r] = pool[lane * PR + r];
    bitonic_sort<PR>(v, lane);
#pragma unroll
    for (int r = 0; r < PR; ++r)
        if (lane * PR + r < p.route_c) p.out[qi * p.route_c + lane * PR + r] = (int32_t)(uint32_t)v[r];
}

}  // namespace ann
