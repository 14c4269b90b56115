// Routing for uint8 vectors of 128 dimensions on the matrix cores.
//
// Stage 1 of Fantasy (Sec. 3.2, "Local K-means Assignment") is the one dense
// contraction on the path: Q (b x d) against the centroids C (d x C), then the
// nearest clusters per query.  Here both operands are shifted into int8 and the query
// is negated on the way, u = 127 - q (byte-wise q ^ 0x7f) and w = c - 128 (c ^ 0x80),
// multiplied on v_mfma_i32_32x32x32_i8 with exact int32 accumulation (dot = u.w), and
// ranked by the key without its per-query terms:
//     L2:  sum (q - c)^2 = sum ((w + 1) + u)^2   ->   bias_c + 2 dot,  bias_c = sum (c - 127)^2
//     IP:  -q.c = -(127 - u).(w + 128)           ->   bias_c +   dot,  bias_c = -127 sum w
// which orders a query's centroids exactly as (key, cluster index) does.  Negating the
// query makes the score a sum, so one shift-add per result forms the packed word below.
//
// Tiling.  A = 32 centroids x 32 bytes, B = 32 queries x 32 bytes per instruction;
// a wavefront keeps 64 queries (two B sets) in registers for the whole kernel and
// walks all centroids, 32 at a time.  The four wavefronts of a workgroup (256 queries)
// share each centroid tile: it is fetched from L2 once (one 16-byte piece per thread,
// shifted to int8 on the way), double-buffered in LDS in the order the matrix
// instruction consumes it, and read back conflict-free.  Without the sharing the kernel
// is bound by L2 bandwidth.  In the 32x32 result a lane holds 16 centroids
// of ONE query (column = lane % 32), so the running best list of a query lives in
// two lanes' registers and needs no exchange until the end.  Rows are visited in
// ascending cluster order, so a strict "<" keeps the lower index among equal keys.
//
// Selection is the expensive part (16 results per lane and tile against 4 matrix
// instructions), so it works on packed words: the bias array holds bias*16 + v, v being
// the result slot of that row inside a lane, and one multiply-add gives score*16 + v.  A
// tree of v_min3 finds a tile's best (score, row) in a lane, and only a tile whose best
// beats the worst kept score is looked at value by value.
#include <hip/hip_runtime.h>

#include "route_mfma.h"
#include "route_mfma_u8.h"

namespace ann {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kMinNearestTiles = 128;  // see launch_rc
constexpr int kPadScore = 0x03ffffff;  // score of the padding rows: above every real one, and score*16 fits

template <int METRIC>
__global__ void __launch_bounds__(256) centroid_bias_kernel(const uint8_t* centroids, int n_clusters, int padded,
                                                            int32_t* bias) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= padded) return;
    // result slot of a row inside a lane: tile row 8 (v / 4) + 4 half + v % 4  <->  v
    const int slot = 4 * ((c & 31) >> 3) + (c & 3);
    if (c >= n_clusters) {
        bias[c] = kPadScore * 16 + slot;
        return;
    }
    const uint32_t* row = reinterpret_cast<const uint32_t*>(centroids + (int64_t)c * 128);
    int32_t acc = 0;
    for (int i = 0; i < 32; ++i) {
        if (METRIC == 0) {
            // (c - 127) as int8 is c ^ 0x7f with the sign flipped: its square is the same
            const uint32_t w1 = row[i] ^ 0x7f7f7f7fu;
            acc = __builtin_amdgcn_sdot4((int)w1, (int)w1, acc, false);
        } else {
            const uint32_t w = row[i] ^ 0x80808080u;
            acc = __builtin_amdgcn_sdot4((int)w, 0x01010101, acc, false);
        }
    }
    bias[c] = (METRIC == 0 ? acc : -127 * acc) * 16 + slot;
}

template <int METRIC, int RC>
__global__ void __launch_bounds__(256) route_mfma_u8_kernel(const uint8_t* __restrict__ centroids,
                                                            const int32_t* __restrict__ bias, int n_clusters,
                                                            const uint8_t* __restrict__ queries, int64_t nq,
                                                            int32_t* __restrict__ out, uint64_t* __restrict__ partial,
                                                            int tiles_per_slice) {
    // blockIdx.y = slice of the centroid tiles this workgroup walks.  With one slice the final
    // clusters go to `out`; with several, each slice writes its best (score, cluster) words to
    // partial[q][slice][RC] and route_merge_kernel picks the overall best.
    constexpr int NQS = 2;  // query sets of 32 per wavefront
    __shared__ uint64_t pool[4][NQS * 32][2][RC];
    __shared__ v4i atile[2][8 * 32];  // [piece 0..7][row 0..31] 16-byte units of one centroid tile
    __shared__ v4i btile[2][8];       // the tile's 32 bias words
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 31, half = lane >> 5;
    const int64_t q0 = ((int64_t)blockIdx.x * 4 + wave) * (NQS * 32);  // may lie beyond nq: such wavefronts only help loading

    // B: lane holds, for query (q0 + 32 s + col), the 16 bytes number 2 t + half of the row
    v4i b[NQS][4];
#pragma unroll
    for (int s = 0; s < NQS; ++s) {
        int64_t q = q0 + s * 32 + col;
        if (q >= nq) q = nq - 1;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            b[s][t] = *reinterpret_cast<const v4i*>(queries + q * 128 + (2 * t + half) * 16);
            b[s][t] ^= (int)0x7f7f7f7f;  // u = 127 - q
        }
    }
    int32_t best_s[NQS][RC], best_i[NQS][RC];
#pragma unroll
    for (int s = 0; s < NQS; ++s)
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            best_s[s][r] = 0x7fffffff;
            best_i[s][r] = 0x7fffffff;
        }

    // thread x fetches piece x % 8 of tile row x / 8 (eight threads read one 128-byte row)
    const int ld_row = threadIdx.x >> 3, ld_piece = threadIdx.x & 7;
    const int all_tiles = (n_clusters + 31) / 32;
    const int tile0 = blockIdx.y * tiles_per_slice;
    const int n_tiles = min(all_tiles, tile0 + tiles_per_slice);
    auto fetch = [&](int ct) {
        int r = ct * 32 + ld_row;
        if (r >= n_clusters) r = n_clusters - 1;
        return *reinterpret_cast<const v4i*>(centroids + (int64_t)r * 128 + ld_piece * 16) ^ (int)0x80808080;
    };
    const v4i* bias4 = reinterpret_cast<const v4i*>(bias);
    atile[tile0 & 1][ld_piece * 32 + ld_row] = fetch(tile0);
    if (threadIdx.x < 8) btile[tile0 & 1][threadIdx.x] = bias4[tile0 * 8 + threadIdx.x];
    __syncthreads();
    for (int ct = tile0; ct < n_tiles; ++ct) {
        v4i next, next_bias;
        if (ct + 1 < n_tiles) {
            next = fetch(ct + 1);
            if (threadIdx.x < 8) next_bias = bias4[(ct + 1) * 8 + threadIdx.x];
        }
        v4i a[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) a[t] = atile[ct & 1][(2 * t + half) * 32 + col];
        // result element v of a lane is row 8 (v / 4) + 4 half + v % 4 of the tile
        v4i bs[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) bs[g] = btile[ct & 1][2 * g + half];
        // both query sets are multiplied before either is looked at: the matrix core works on
        // the second while the vector ALU selects from the first
        v16i accs[NQS];
#pragma unroll
        for (int s = 0; s < NQS; ++s) {
            accs[s] = v16i{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int t = 0; t < 4; ++t) accs[s] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[t], b[s][t], accs[s], 0, 0, 0);
        }
#pragma unroll
        for (int s = 0; s < NQS; ++s) {
            const v16i acc = accs[s];
            // packed[v] = score * 16 + v
            int32_t packed[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) packed[v] = bs[v / 4][v % 4] + (acc[v] << (METRIC == 0 ? 5 : 4));
            int32_t m01 = min(min(packed[0], packed[1]), packed[2]);
            int32_t m02 = min(min(packed[3], packed[4]), packed[5]);
            int32_t m03 = min(min(packed[6], packed[7]), packed[8]);
            int32_t m04 = min(min(packed[9], packed[10]), packed[11]);
            int32_t m05 = min(min(packed[12], packed[13]), packed[14]);
            const int32_t tile_best = min(min(min(m01, m02), min(m03, m04)), min(m05, packed[15]));
            const int32_t tile_score = tile_best >> 4;
            if constexpr (RC == 1) {
                // strict "<" on the score alone: among equal scores the earlier tile stays
                const bool better = tile_score < best_s[s][0];
                best_s[s][0] = better ? tile_score : best_s[s][0];
                best_i[s][0] = better ? ct * 32 + 8 * ((tile_best & 15) >> 2) + 4 * half + (tile_best & 3) : best_i[s][0];
            } else if (__any(tile_score < best_s[s][RC - 1])) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int32_t score = packed[v] >> 4;
                    const int32_t idx = ct * 32 + 8 * (v / 4) + 4 * half + (v % 4);
                    if (score < best_s[s][RC - 1]) {
                        // insertion; equal scores stay behind the earlier (smaller) index
                        int32_t cs = score, ci = idx;
#pragma unroll
                        for (int r = 0; r < RC; ++r) {
                            const bool first = cs < best_s[s][r];
                            const int32_t ts = best_s[s][r], ti = best_i[s][r];
                            best_s[s][r] = first ? cs : ts;
                            best_i[s][r] = first ? ci : ti;
                            cs = first ? ts : cs;
                            ci = first ? ti : ci;
                        }
                    }
                }
            }
        }
        if (ct + 1 < n_tiles) {
            atile[(ct + 1) & 1][ld_piece * 32 + ld_row] = next;
            if (threadIdx.x < 8) btile[(ct + 1) & 1][threadIdx.x] = next_bias;
        }
        __syncthreads();
    }

    // the two lanes of a query merge their ascending lists through LDS
#pragma unroll
    for (int s = 0; s < NQS; ++s)
#pragma unroll
        for (int r = 0; r < RC; ++r)
            pool[wave][s * 32 + col][half][r] =
                ((uint64_t)((uint32_t)best_s[s][r] ^ 0x80000000u) << 32) | (uint32_t)best_i[s][r];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // lane -> query (q0 + lane): every lane merges one query
    const int64_t q = q0 + lane;
    if (q < nq) {
        int ia = 0, ib = 0;
        for (int r = 0; r < RC; ++r) {
            const uint64_t x = ia < RC ? pool[wave][lane][0][ia] : ~0ull;
            const uint64_t y = ib < RC ? pool[wave][lane][1][ib] : ~0ull;
            const bool take_x = x < y;
            if (gridDim.y == 1)
                out[q * RC + r] = (int32_t)(uint32_t)(take_x ? x : y);
            else
                partial[(q * gridDim.y + blockIdx.y) * RC + r] = take_x ? x : y;
            ia += take_x ? 1 : 0;
            ib += take_x ? 0 : 1;
        }
    }
}

// Where a centroid goes among the tiles (see RouteU8Block): one workgroup.
template <int METRIC>
__global__ void __launch_bounds__(1024) route_u8_order_kernel(const int32_t* bias, int n_clusters, int max_tiles, int32_t* shape,
                                                              int32_t* half, int32_t* map) {
    __shared__ int32_t wave_even[16];
    const int t = threadIdx.x, wave = t >> 6;
    for (int i = t; i < max_tiles * 32; i += 1024) {
        half[i] = 0x1fffffff;  // padding never wins
        map[i] = 0x7fffffff;
    }
    auto even_at = [&](int c) { return c < n_clusters && (METRIC != 0 || ((bias[c] >> 4) & 1) == 0); };
    // even centroids in front of this wavefront's, and in the whole block of 1024
    auto count = [&](bool even, int* before) {
        const uint64_t m = __ballot(even);
        if ((t & 63) == 0) wave_even[wave] = __builtin_popcountll(m);
        __syncthreads();
        int all = 0;
        *before = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        for (int w = 0; w < 16; ++w) {
            if (w < wave) *before += wave_even[w];
            all += wave_even[w];
        }
        __syncthreads();
        return all;
    };
    int total = 0, before;
    for (int c0 = 0; c0 < n_clusters; c0 += 1024) total += count(even_at(c0 + t), &before);
    const int even_tiles = (total + 31) / 32, odd_tiles = (n_clusters - total + 31) / 32;
    if (t == 0) {
        shape[0] = even_tiles;
        shape[1] = even_tiles + odd_tiles;
    }
    int even_run = 0;
    for (int c0 = 0; c0 < n_clusters; c0 += 1024) {
        const int c = c0 + t;
        const bool even = even_at(c);
        const int all = count(even, &before);
        if (c < n_clusters) {
            const int at = even ? even_run + before : even_tiles * 32 + (c0 - even_run) + (t - before);
            half[at] = METRIC == 0 ? bias[c] >> 5 : bias[c] >> 4;
            map[at] = c;
        }
        even_run += all;
    }
}

// One thread per 16-byte unit of the tiles.
__global__ void __launch_bounds__(256) route_u8_rows_kernel(const uint8_t* centroids, int n_clusters, int64_t units, const int32_t* map, v4i* rows) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= units) return;
    const int tile = (int)(i >> 8), piece = (int)(i >> 5) & 7, row = (int)i & 31;
    const int c = map[tile * 32 + row];
    rows[i] = (uint32_t)c < (uint32_t)n_clusters ? *reinterpret_cast<const v4i*>(centroids + (int64_t)c * 128 + piece * 16) ^ (int)0x80808080
                                                 : v4i{0, 0, 0, 0};
}

// The nearest cluster of each query (route_c = 1), for many centroids.
//
// As route_mfma_u8_kernel, but nothing is packed: the accumulators start at half the bias, so a result is the score
// itself (IP) or half of it without its lowest bit (L2), which is the same for all rows of a tile; a tile costs a lane
// eight three-way minima and four instructions for the running best and its tile.  Which row of the tile it was is found
// once, at the end: the wavefront computes the 32 scores of each query's best tile again and looks for the equal one.
// Among equal scores the lowest cluster wins: they lie in one class of tiles, whose order is that of the clusters, and a
// lane keeps the first; the two lanes of a query meet in the final search.
// 500 000 queries x 16 384 centroids: 0.93 to 1.00 ms from box to box, where route_mfma_u8_kernel takes 1.16 to 1.24 ms on the
// same ones.
template <int METRIC, int kTiles>
__global__ void __launch_bounds__(256) route_nearest_u8_kernel(const v4i* __restrict__ rows, const int32_t* __restrict__ half_bias,
                                                               const int32_t* __restrict__ map, const int32_t* __restrict__ shape,
                                                               const uint8_t* __restrict__ queries, int64_t nq,
                                                               int32_t* __restrict__ out, uint64_t* __restrict__ partial,
                                                               int tiles_per_slice) {
    constexpr int NQS = 2;  // query sets of 32 per wavefront
    __shared__ v4i atile[2][kTiles * 256];  // [tile][piece][row] 16-byte units; in the end 16 queries of each wavefront
    __shared__ v4i btile[2][kTiles * 8];    // the tiles' half biases
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 31, half = lane >> 5;
    const int64_t q0 = ((int64_t)blockIdx.x * 4 + wave) * (NQS * 32);  // may lie beyond nq: such wavefronts only help loading
    const int even_tiles = shape[0];
    const int tile0 = blockIdx.y * tiles_per_slice;
    const int n_tiles = min(shape[1], tile0 + tiles_per_slice);
    if (tile0 >= n_tiles) {  // the whole workgroup; only the last slice can be empty (a tile more or less of padding)
        const int64_t q = q0 + lane;
        if (q < nq) partial[q * gridDim.y + blockIdx.y] = ~0ull;
        return;
    }

    v4i b[NQS][4];
#pragma unroll
    for (int s = 0; s < NQS; ++s) {
        int64_t q = q0 + s * 32 + col;
        if (q >= nq) q = nq - 1;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            b[s][t] = *reinterpret_cast<const v4i*>(queries + q * 128 + (2 * t + half) * 16) ^ (int)0x7f7f7f7f;  // u = 127 - q
        }
    }
    int32_t best[NQS], best_tile[NQS];
#pragma unroll
    for (int s = 0; s < NQS; ++s) {
        best[s] = 0x7fffffff;
        best_tile[s] = tile0;
    }
    const v4i* bias4 = reinterpret_cast<const v4i*>(half_bias);
    // a step is kTiles tiles: one barrier for all of them (the arrays hold whole steps beyond the last tile)
    v4i next[kTiles], next_bias;
    auto fetch = [&](int ct) {
#pragma unroll
        for (int i = 0; i < kTiles; ++i) next[i] = rows[(int64_t)(ct + i) * 256 + threadIdx.x];
        if (threadIdx.x < 8 * kTiles) next_bias = bias4[(int64_t)ct * 8 + threadIdx.x];
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int i = 0; i < kTiles; ++i) atile[buf][i * 256 + threadIdx.x] = next[i];
        if (threadIdx.x < 8 * kTiles) btile[buf][threadIdx.x] = next_bias;
    };
    fetch(tile0);
    stage(0);
    __syncthreads();
    int buf = 0;
    for (int ct0 = tile0; ct0 < n_tiles; ct0 += kTiles, buf ^= 1) {
        if (ct0 + kTiles < n_tiles) fetch(ct0 + kTiles);
#pragma unroll
        for (int i = 0; i < kTiles; ++i) {
            const int ct = ct0 + i;
            if (ct >= n_tiles) break;
            v4i a[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) a[t] = atile[buf][i * 256 + (2 * t + half) * 32 + col];
            v16i c;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const v4i bs = btile[buf][i * 8 + 2 * g + half];
#pragma unroll
                for (int k = 0; k < 4; ++k) c[4 * g + k] = bs[k];
            }
            const int odd = METRIC == 0 && ct >= even_tiles ? 1 : 0;
            v16i accs[NQS];
#pragma unroll
            for (int s = 0; s < NQS; ++s) {
                accs[s] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[0], b[s][0], c, 0, 0, 0);
#pragma unroll
                for (int t = 1; t < 4; ++t) accs[s] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[t], b[s][t], accs[s], 0, 0, 0);
            }
#pragma unroll
            for (int s = 0; s < NQS; ++s) {
                const v16i v = accs[s];
                const int32_t m0 = min(min(v[0], v[1]), v[2]), m1 = min(min(v[3], v[4]), v[5]), m2 = min(min(v[6], v[7]), v[8]);
                const int32_t m3 = min(min(v[9], v[10]), v[11]), m4 = min(min(v[12], v[13]), v[14]);
                const int32_t m = min(min(min(m0, m1), min(m2, m3)), min(m4, v[15]));
                const int32_t score = METRIC == 0 ? (m << 1) | odd : m;
                best_tile[s] = score < best[s] ? ct : best_tile[s];
                best[s] = min(best[s], score);
            }
        }
        if (ct0 + kTiles < n_tiles) stage(buf ^ 1);
        __syncthreads();
    }

    // The 16 rows of the better half's tile, four lanes (32 bytes each) per row; both halves' if their scores are equal.
    const int row16 = lane >> 2, part = lane & 3;
    int32_t cluster = 0, score_of = 0;
    v4i* const uq = &atile[0][0] + wave * 128;
#pragma unroll
    for (int s = 0; s < NQS; ++s) {
        for (int c0 = 0; c0 < 32; c0 += 4) {
            if ((c0 & 15) == 0) {  // this wavefront's next 16 queries
                __builtin_amdgcn_wave_barrier();
                if ((col & 16) == c0) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) uq[(col & 15) * 8 + 2 * t + half] = b[s][t];
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
            int32_t best2[4][2], tile2[4][2];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    best2[u][h] = __builtin_amdgcn_readlane(best[s], c0 + u + 32 * h);
                    tile2[u][h] = __builtin_amdgcn_readlane(best_tile[s], c0 + u + 32 * h);
                }
            v4i x[4][2];
            int32_t hb[4], id[4];
            auto load = [&](int u, int h) {
                const int32_t tile = h ? tile2[u][1] : tile2[u][0];
                const int row = 8 * (row16 >> 2) + 4 * h + (row16 & 3);
#pragma unroll
                for (int k = 0; k < 2; ++k) x[u][k] = rows[(int64_t)tile * 256 + (part * 2 + k) * 32 + row];
                hb[u] = half_bias[tile * 32 + row];
                id[u] = map[tile * 32 + row];
            };
            // lowest cluster whose score is `want`
            auto find = [&](int u, int32_t want, int tile) {
                int32_t dot = 0;
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const v4i q = uq[((c0 & 15) + u) * 8 + part * 2 + k];
#pragma unroll
                    for (int i = 0; i < 4; ++i) dot = __builtin_amdgcn_sdot4(q[i], x[u][k][i], dot, false);
                }
                dot += __builtin_amdgcn_update_dpp(0, dot, 0xB1, 0xf, 0xf, true);  // quad_perm [1,0,3,2]
                dot += __builtin_amdgcn_update_dpp(0, dot, 0x4E, 0xf, 0xf, true);  // quad_perm [2,3,0,1]
                const int32_t m = hb[u] + dot;
                uint64_t hit = __ballot((METRIC == 0 ? 2 * m + (tile >= even_tiles ? 1 : 0) : m) == want);
                int32_t found = 0x7fffffff;
                while (hit) {  // one row, but for equal scores
                    const int l = __builtin_ctzll(hit);
                    found = min(found, __builtin_amdgcn_readlane(id[u], l));
                    hit &= ~(0xfull << (l & ~3));
                }
                return found;
            };
            int pick[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {  // four queries' rows in flight
                pick[u] = best2[u][1] < best2[u][0] ? 1 : 0;
                load(u, pick[u]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int32_t want = pick[u] ? best2[u][1] : best2[u][0];
                int32_t found = find(u, want, pick[u] ? tile2[u][1] : tile2[u][0]);
                if (best2[u][0] == best2[u][1]) {  // uniform
                    load(u, 1);
                    found = min(found, find(u, want, tile2[u][1]));
                }
                const bool my = lane == s * 32 + c0 + u;
                cluster = my ? found : cluster;
                score_of = my ? want : score_of;
            }
        }
    }
    const int64_t q = q0 + lane;
    if (q < nq) {
        if (gridDim.y == 1) out[q] = cluster;
        else partial[q * gridDim.y + blockIdx.y] = ((uint64_t)((uint32_t)score_of ^ 0x80000000u) << 32) | (uint32_t)cluster;
    }
}

template <int METRIC>
static hipError_t launch_rc(int rc, const uint8_t* centroids, const char* block, int n_clusters,
                            const uint8_t* queries, int64_t nq, int32_t* out, uint64_t* partial, int slices,
                            hipStream_t stream) {
    const RouteU8Block at(n_clusters);
    const int32_t* bias = reinterpret_cast<const int32_t*>(block + at.bias);
    const int all_tiles = (n_clusters + 31) / 32;
    const int tiles_per_slice = (all_tiles + slices - 1) / slices;
    // the final search of route_nearest_u8_kernel takes as long as some eighty tiles: 500 000 queries x 16 384 / 8 192 / 4 096
    // centroids in 1.00 / 0.54 / 0.31 ms, the other kernel's 1.24 / 0.62 / 0.32 ms (100 000: 255 / 143 / 91 and 346 / 175 / 89 us)
    if (rc == 1 && tiles_per_slice >= kMinNearestTiles) {
        // with both classes padded there may be a tile more than that
        const int per = (all_tiles + slices) / slices;
        slices = (all_tiles + per) / per;
        hipLaunchKernelGGL((route_nearest_u8_kernel<METRIC, kRouteU8StepTiles>), dim3((unsigned)((nq + 255) / 256), (unsigned)slices), dim3(256), 0, stream,
                           reinterpret_cast<const v4i*>(block + at.rows), reinterpret_cast<const int32_t*>(block + at.half),
                           reinterpret_cast<const int32_t*>(block + at.map), reinterpret_cast<const int32_t*>(block + at.shape),
                           queries, nq, out, partial, per);
        if (slices > 1) return launch_route_merge(rc, partial, slices, nq, out, stream);
        return hipGetLastError();
    }
    slices = (all_tiles + tiles_per_slice - 1) / tiles_per_slice;  // no slice may start beyond the last tile
    const dim3 grid((unsigned)((nq + 255) / 256), (unsigned)slices), threads(256);
    switch (rc) {
        case 1:
            hipLaunchKernelGGL((route_mfma_u8_kernel<METRIC, 1>), grid, threads, 0, stream, centroids, bias, n_clusters, queries, nq, out, partial, tiles_per_slice);
            break;
        case 2:
            hipLaunchKernelGGL((route_mfma_u8_kernel<METRIC, 2>), grid, threads, 0, stream, centroids, bias, n_clusters, queries, nq, out, partial, tiles_per_slice);
            break;
        case 3:
            hipLaunchKernelGGL((route_mfma_u8_kernel<METRIC, 3>), grid, threads, 0, stream, centroids, bias, n_clusters, queries, nq, out, partial, tiles_per_slice);
            break;
        case 4:
            hipLaunchKernelGGL((route_mfma_u8_kernel<METRIC, 4>), grid, threads, 0, stream, centroids, bias, n_clusters, queries, nq, out, partial, tiles_per_slice);
            break;
        case 5:
            hipLaunchKernelGGL((route_mfma_u8_kernel<METRIC, 5>), grid, threads, 0, stream, centroids, bias, n_clusters, queries, nq, out, partial, tiles_per_slice);
            break;
        case 6:
            hipLaunchKernelGGL((route_mfma_u8_kernel<METRIC, 6>), grid, threads, 0, stream, centroids, bias, n_clusters, queries, nq, out, partial, tiles_per_slice);
            break;
        case 7:
            hipLaunchKernelGGL((route_mfma_u8_kernel<METRIC, 7>), grid, threads, 0, stream, centroids, bias, n_clusters, queries, nq, out, partial, tiles_per_slice);
            break;
        case 8:
            hipLaunchKernelGGL((route_mfma_u8_kernel<METRIC, 8>), grid, threads, 0, stream, centroids, bias, n_clusters, queries, nq, out, partial, tiles_per_slice);
            break;
        default: return hipErrorInvalidValue;
    }
    if (slices > 1) return launch_route_merge(rc, partial, slices, nq, out, stream);
    return hipGetLastError();
}

template <int METRIC>
static hipError_t fill_block(const uint8_t* centroids, int n_clusters, char* block, hipStream_t stream) {
    const RouteU8Block at(n_clusters);
    const int padded = route_mfma_u8_padded(n_clusters), max_tiles = padded / 32 + kRouteU8StepTiles;
    int32_t* const bias = reinterpret_cast<int32_t*>(block + at.bias);
    int32_t* const map = reinterpret_cast<int32_t*>(block + at.map);
    hipLaunchKernelGGL((centroid_bias_kernel<METRIC>), dim3((unsigned)((padded + 255) / 256)), dim3(256), 0, stream, centroids, n_clusters,
                       padded, bias);
    hipLaunchKernelGGL((route_u8_order_kernel<METRIC>), dim3(1), dim3(1024), 0, stream, bias, n_clusters, max_tiles,
                       reinterpret_cast<int32_t*>(block + at.shape), reinterpret_cast<int32_t*>(block + at.half), map);
    hipLaunchKernelGGL(route_u8_rows_kernel, dim3((unsigned)max_tiles), dim3(256), 0, stream, centroids, n_clusters, (int64_t)max_tiles * 256, map,
                       reinterpret_cast<v4i*>(block + at.rows));
    return hipGetLastError();
}

hipError_t launch_route_u8_block(int metric, const uint8_t* centroids, int n_clusters, void* block, hipStream_t stream) {
    char* const to = static_cast<char*>(block);
    return metric == 0 ? fill_block<0>(centroids, n_clusters, to, stream) : fill_block<1>(centroids, n_clusters, to, stream);
}

int route_mfma_u8_slices(int n_clusters, int64_t nq) { return route_slices((n_clusters + 31) / 32, 8, nq); }

hipError_t launch_route_mfma_u8(int metric, int route_c, const uint8_t* centroids, const void* block, int n_clusters,
                                const uint8_t* queries, int64_t nq, int32_t* out, uint64_t* partial, int slices,
                                hipStream_t stream) {
    const char* const from = static_cast<const char*>(block);
    return metric == 0 ? launch_rc<0>(route_c, centroids, from, n_clusters, queries, nq, out, partial, slices, stream)
                       : launch_rc<1>(route_c, centroids, from, n_clusters, queries, nq, out, partial, slices, stream);
}

}  // namespace ann
