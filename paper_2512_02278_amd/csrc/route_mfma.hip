// Routing on the matrix cores for any element type and any row length (a multiple of 16 bytes): nearest route_c centroids
// per query under (score, cluster index).
//
// Stage 1 of Fantasy (Sec. 3.2, "Local K-means Assignment") is a dense contraction,
// Q (b x d) against C (d x C), followed by a per-query selection.  The score that is ranked is
// the key without its per-query constant:
//     L2:  |c|^2 - 2 q.c          IP:  -q.c
// uint8 operands are shifted by -128 into int8 (exact int32 sums; for the inner product the shift
// adds -128*sum(c') per centroid, which goes into the bias); fp16 / fp32 operands accumulate in
// fp32 on v_mfma_f32_32x32x16_f16 / v_mfma_f32_32x32x16_bf16 (three parts per fp32 value).
//
// A wavefront owns a 64 x 64 block of scores (two operand sets of 32 rows on either side): four 32x32
// accumulator tiles, and per 16-byte piece of the rows two reads of each operand feed four matrix
// instructions.  Operand chunks are staged in LDS by the workgroup (see the kernel); the rows can be of any
// length.  In a 32x32 result a lane holds 16 centroids of one query, so a query's best candidates live in a few
// lanes' registers and are merged once at the end.  A lane visits its rows in ascending cluster order, so a
// strict "<" keeps the lower index among equal scores, and the final merge compares (score, index) words.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "route_mfma.h"

namespace ann {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

template <int DT>
struct Mma;

template <>
struct Mma<0> {  // uint8 -> int8, int32 sums
    typedef v16i acc_t;
    typedef int32_t score_t;
    static constexpr int kParts = 1;
    static __device__ __forceinline__ v4i prep(v4i x) { return x ^ (int)0x80808080; }
    static __device__ __forceinline__ acc_t mma(acc_t c, v4i a, v4i b) {
        return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ score_t score(score_t bias, int32_t dot, bool l2) {
        return bias - (l2 ? 2 : 1) * dot;
    }
    static __device__ __forceinline__ uint32_t ordered(score_t s) { return (uint32_t)s ^ 0x80000000u; }
    static constexpr score_t kWorst = 0x7fffffff;
};
template <>
struct Mma<1> {  // fp16, fp32 sums
    typedef v16f acc_t;
    typedef float score_t;
    static constexpr int kParts = 1;
    static __device__ __forceinline__ v4i prep(v4i x) { return x; }
    static __device__ __forceinline__ acc_t mma(acc_t c, v4i a, v4i b) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
    }
    static __device__ __forceinline__ score_t score(score_t bias, float dot, bool l2) {
        return l2 ? __builtin_fmaf(-2.0f, dot, bias) : bias - dot;  // bias is 0 for real rows of an IP index
    }
    static __device__ __forceinline__ uint32_t ordered(score_t s) {
        s = s + 0.0f;
        const uint32_t u = __builtin_bit_cast(uint32_t, s);
        return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    }
    static constexpr score_t kWorst = __builtin_inff();
};
// fp32: every value is the sum of three bf16 values (its 24 bits are theirs, 8 each, rounded to nearest, so that the
// second and third are at most 2^-8 and 2^-17 of it), and of the nine products of two sums the six largest run on
// v_mfma_f32_32x32x16_bf16, the smallest first.  What is left out is at most 2^-24 of a product, as much as one rounding of
// an fp32 product may be off (two factors of 1.00388), and 2^-27 on average.  Six such instructions take 3/8 of the time of
// the eight v_mfma_f32_32x32x2_f32 that 16 elements take otherwise, and they round six sums where those round sixteen.
// Against 64 bits, what the key of the chosen centroid exceeds the nearest one's by, fp32 instructions / parts, in units of
// |q|^2 + |c|^2 or |q||c|; mean and worst of 100 000 queries to 1 024 centroids:
//   half way between two Gaussian centroids, L2: 8 elements 1.7e-10 and 5e-8 / 1.7e-10 and 4e-8, 32 1.7e-9 and 3e-8 / 1.7e-9
//     and 3e-8, 96 1.35e-9 and 2.0e-8 / 1.35e-9 and 1.6e-8, 256 8.4e-10 and 1e-8 / 8.5e-10 and 1e-8;
//   all mantissas within 2^-16 of the worst one, all products of one sign (inner product): 8 elements 1.0e-8 and 1.5e-7 / 0, 32
//     4.2e-9 and 3.0e-7 / 8.6e-11 and 3.7e-9, 96 7.1e-8 and 7.8e-7 / 5.9e-8 and 1.1e-7, 256 1.5e-7 and 9.4e-7 / 5.4e-8 and
//     1.3e-7; every second centroid with any mantissas instead: 32 2.7e-8 and 3.5e-7 / 3.7e-8 and 5.6e-8, 96 9.2e-8 and 7.4e-7 /
//     8.2e-8 and 9.5e-8, 256 1.8e-7 and 9.9e-7 / 2.1e-8 and 4.8e-7.
//
// A sum of parts is what the fp32 instruction gives only while no product of two parts overflows (the parts of a large
// value differ in sign: infinity minus infinity) and none that counts underflows.  Rows whose largest magnitude lies
// outside [2^-40, 2^57) are therefore ranked by the fp32 instruction (Mma<3>): within it a sum of 1 536 products stays
// below 2^126, and of the largest product of two rows (2^-80 at least) 46 bits lie above the smallest normal value.
template <>
struct Mma<2> : Mma<1> {
    static constexpr int kParts = 3;
    // whether the row whose largest magnitude has these bits (0: a row of zeros) is not for this instruction
    static __device__ __forceinline__ bool apart(uint32_t peak) {
        return peak != 0u && (peak < __builtin_bit_cast(uint32_t, 0x1p-40f) || peak >= __builtin_bit_cast(uint32_t, 0x1p57f));
    }
    static __device__ __forceinline__ uint32_t magnitude(uint32_t bits) { return bits & 0x7fffffffu; }
    // parts of four floats: part[p] holds four bf16
    static __device__ __forceinline__ void split(v4i x, uint2 (&part)[kParts]) {
        const v4f f = __builtin_bit_cast(v4f, x);
        v2f lo = {f.x, f.y}, hi = {f.z, f.w};
#pragma unroll
        for (int p = 0; p < kParts; ++p) {
            part[p].x = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, v2bf));
            part[p].y = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, v2bf));
            lo.x -= __builtin_bit_cast(float, part[p].x << 16);
            lo.y -= __builtin_bit_cast(float, part[p].x & 0xffff0000u);
            hi.x -= __builtin_bit_cast(float, part[p].y << 16);
            hi.y -= __builtin_bit_cast(float, part[p].y & 0xffff0000u);
        }
    }
    static __device__ __forceinline__ acc_t mma(acc_t c, v4i a, v4i b) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
    }
};
template <>
struct Mma<3> : Mma<1> {  // fp32, the values as they are: four K = 2 instructions per 16-byte piece
    static __device__ __forceinline__ acc_t mma(acc_t c, v4i a, v4i b) {
        const v4f x = __builtin_bit_cast(v4f, a), y = __builtin_bit_cast(v4f, b);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(x.x, y.x, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(x.y, y.y, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(x.z, y.z, c, 0, 0, 0);
        return __builtin_amdgcn_mfma_f32_32x32x2f32(x.w, y.w, c, 0, 0, 0);
    }
};

__global__ void route_clear_words_kernel(uint32_t* words) { words[threadIdx.x] = 0u; }

// bias[c]: the per-centroid term of the score; rows beyond n_clusters (padding up to a multiple
// of 128) get a value that never wins.  Float types: of the three words behind them the first becomes 1 if any centroid is not for the
// bf16 parts (fp32), the second the largest |c|^2 (not a number: something larger than any), the third the sum of all.
template <int DT, int METRIC>
__global__ void __launch_bounds__(256) route_bias_kernel(const uint8_t* centroids, int n_clusters, int padded,
                                                         int row_bytes, void* bias_out) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= padded) return;
    const uint8_t* row = centroids + (int64_t)c * row_bytes;
    if constexpr (DT == 0) {
        int32_t* bias = static_cast<int32_t*>(bias_out);
        if (c >= n_clusters) {
            bias[c] = 0x3fffffff;
            return;
        }
        int32_t acc = 0;
        for (int i = 0; i < row_bytes / 4; ++i) {
            const uint32_t w = reinterpret_cast<const uint32_t*>(row)[i] ^ 0x80808080u;
            acc = METRIC == 0 ? __builtin_amdgcn_sdot4((int)w, (int)w, acc, false)
                              : __builtin_amdgcn_sdot4((int)w, 0x01010101, acc, false);
        }
        bias[c] = METRIC == 0 ? acc : -128 * acc;
    } else {
        float* bias = static_cast<float*>(bias_out);
        float acc = 0.0f;
        uint32_t peak = 0u;
        const int n = c < n_clusters ? row_bytes / (DT == 1 ? 2 : 4) : 0;
        for (int i = 0; i < n; ++i) {
            const float v = DT == 1 ? (float)reinterpret_cast<const _Float16*>(row)[i]
                                    : reinterpret_cast<const float*>(row)[i];
            acc = __builtin_fmaf(v, v, acc);
            if (DT == 2) peak = max(peak, Mma<2>::magnitude(__builtin_bit_cast(uint32_t, v)));
        }
        bias[c] = c >= n_clusters ? 1.0e38f : METRIC == 0 ? acc : 0.0f;
        uint32_t* const words = reinterpret_cast<uint32_t*>(bias) + padded;
        if (DT == 2 && Mma<2>::apart(peak)) words[0] = 1u;
        uint32_t largest = __builtin_bit_cast(uint32_t, acc) & 0x7fffffffu;
        for (int d = 1; d < 64; d <<= 1) largest = max(largest, (uint32_t)__shfl_xor((int)largest, d));
        for (int d = 1; d < 64; d <<= 1) acc += __shfl_xor(acc, d);
        if ((threadIdx.x & 63) == 0) {
            atomicMax(&words[1], largest);
            atomicAdd(reinterpret_cast<float*>(&words[2]), acc);
        }
    }
}

// One workgroup: 128 queries against 128 centroids at a time, four wavefronts in a 2 x 2 arrangement, each
// owning a 64 x 64 block of scores (2 x 2 result tiles of 32 x 32).  The rows are walked in chunks of 64 or 128
// bytes (route_mfma_chunk); a chunk of both operands is staged in LDS once per workgroup, piece-major
// ([16-byte piece][row], one unit of padding per piece so that the staging writes spread over the banks),
// which is the order the matrix instruction consumes: lane (row % 32, half) reads consecutive 16-byte units.
// The next chunk travels from L2 to registers while the current one is multiplied; two LDS buffers, one
// barrier per chunk.  (Streaming the operands straight from L1/L2 in the instruction's layout - 32 rows x 32
// bytes per load - left this kernel at a twelfth of the fp16 matrix rate.)
template <int I, int CHUNK>
constexpr int route_operand_units() {  // 16-byte units of one operand chunk in LDS
    return (Mma<I>::kParts == 1 ? CHUNK / 16 : 2 * Mma<I>::kParts) * (128 + 1);
}

template <int I, int CHUNK, int RC>
constexpr int route_smem_units() {  // two buffers of both operands; the pool of best lists reuses them
    const int staging = 4 * route_operand_units<I, CHUNK>(), pool = 128 * 4 * RC / 2;
    return staging > pool ? staging : pool;
}

// I: how the products are taken (Mma<I>).  The bits of apart[] (fp32 only, else null) are the rows of the workgroup's 128
// queries that the bf16 parts are not for: Mma<2> sets them and leaves those rows out, Mma<3> writes them only.
template <int I, int CHUNK, int METRIC, int RC>
__device__ __forceinline__ void route_queries(v4i* smem, typename Mma<I>::score_t* bias_lds, uint32_t* apart, const uint8_t* __restrict__ centroids,
                                              const void* __restrict__ bias_in, int n_clusters, int row_bytes,
                                              const uint8_t* __restrict__ queries, int64_t nq, int32_t* __restrict__ out,
                                              uint64_t* __restrict__ partial, int tiles_per_slice) {
    // blockIdx.y = slice of the 128-centroid tiles this workgroup walks; with several slices the best words
    // of a slice go to partial[q][slice][RC] and route_merge_kernel finishes the job
    typedef Mma<I> M;
    typedef typename M::acc_t acc_t;
    typedef typename M::score_t score_t;
    // bytes of a row per chunk, and its 16-byte pieces as they are staged: all of them, or two of each bf16 part
    constexpr int kChunk = CHUNK;
    constexpr int kRows = 128, kPieces = M::kParts == 1 ? kChunk / 16 : 2 * M::kParts, kPieceStride = kRows + 1;
    constexpr int kOperand = route_operand_units<I, CHUNK>();
    static_assert(route_smem_units<I, CHUNK, RC>() >= 4 * kOperand, "two buffers of both operands");
    const score_t* bias = static_cast<const score_t*>(bias_in);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wq = wave >> 1, wc = wave & 1;  // which 64 queries / which 64 centroids of the tile
    const int col = lane & 31, half = lane >> 5;
    const int64_t q0 = (int64_t)blockIdx.x * kRows;

    // staging: thread x moves piece x % kMoved of rows x / kMoved + i * kStageRows (the threads of a row read contiguous bytes)
    constexpr int kMoved = kChunk / 16, kStageRows = 256 / kMoved, kStage = kRows / kStageRows;
    const int st_piece = threadIdx.x % kMoved, st_row = threadIdx.x / kMoved;
    const uint8_t* const qbase = queries + q0 * row_bytes + st_piece * 16;
    int qoff[kStage];
#pragma unroll
    for (int i = 0; i < kStage; ++i) {
        const int64_t left = nq - 1 - q0;  // the last query again beyond the batch's end
        const int r = st_row + kStageRows * i;
        qoff[i] = (r < left ? r : (int)left) * row_bytes;
    }
    uint32_t peak[kStage];  // of this thread's share of its rows
#pragma unroll
    for (int i = 0; i < kStage; ++i) peak[i] = 0u;
    score_t best_s[2][RC];
    int32_t best_i[2][RC];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            best_s[s][r] = M::kWorst;
            best_i[s][r] = 0x7fffffff;
        }

    const int chunks = (row_bytes + kChunk - 1) / kChunk;
    const int all_tiles = (n_clusters + kRows - 1) / kRows;
    const int tile_end = min(all_tiles, (int)(blockIdx.y + 1) * tiles_per_slice);
    const v4i zero = v4i{0, 0, 0, 0};
    const int tile0 = blockIdx.y * tiles_per_slice;
    // The scores of 16 rows (base + 8 (v / 4) + v % 4) into a lane's list.  A score counts if it is below the RC-th best of the
    // query's two lists, this lane's and the other half's: all of their rows come before these, so an equal score loses.
    // Nearly every single score is such a one for some of the 64 lanes, but a lane has few of them, so the lanes go through
    // their own: 25 000 fp16 rows of 1536 bytes x 8 192, nearest four: 534 -> 467 us; 100 000 of 256 bytes x 4 000, nearest
    // eight: 887 -> 372 us (with the next tile's chunk on its way meanwhile and the biases in LDS, which alone give 2 to 8 %).
    auto take_best = [&](score_t (&list_s)[RC], int32_t (&list_i)[RC], const acc_t& dot, const score_t (&bs)[16], int base) {
        score_t low[RC], high[RC];
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            const uint32_t w = __builtin_bit_cast(uint32_t, list_s[r]);
            const auto both = __builtin_amdgcn_permlane32_swap(w, w, false, false);
            const uint32_t in_low = both[0], in_high = both[1];  // (a bit cast of a vector's element takes element 0)
            low[r] = __builtin_bit_cast(score_t, in_low);
            high[r] = __builtin_bit_cast(score_t, in_high);
        }
        score_t limit = min(low[RC - 1], high[RC - 1]);
#pragma unroll
        for (int r = 0; r + 1 < RC; ++r) limit = min(limit, max(low[r], high[RC - 2 - r]));
        score_t score[16];
        uint32_t open = 0;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            score[v] = M::score(bs[v], dot[v], METRIC == 0);
            open |= score[v] < limit ? 1u << v : 0u;
        }
        if (__any(__builtin_popcount(open) > (RC <= 4 ? RC + 1 : 8))) {
            // mostly the first rows of all: one after the other costs less than finding them (3 000 fp16 rows of 256 bytes x 300,
            // nearest eight: 38.7 -> 32.1 us)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (score[v] < list_s[RC - 1]) insert_nearest<RC>(list_s, list_i, score[v], base + 8 * (v / 4) + (v % 4));
            return;
        }
        while (open) {
            const int v = __builtin_ctz(open);
            open &= open - 1;
            score_t pick[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) pick[j] = score[j];
#pragma unroll
            for (int d = 0; d < 4; ++d)
#pragma unroll
                for (int j = 0; j < 16 >> (d + 1); ++j) pick[j] = (v >> d & 1) ? pick[2 * j + 1] : pick[2 * j];
            insert_nearest<RC>(list_s, list_i, pick[0], base + v + (v & ~3));  // 8 (v / 4) + v % 4
        }
    };
    const uint8_t* cbase;
    int coff[kStage];
    v4i ra[kStage], rb[kStage];
    score_t tile_bias;  // of centroid threadIdx.x of the tile
    auto aim = [&](int ct) {
        cbase = centroids + (int64_t)ct * kRows * row_bytes + st_piece * 16;
#pragma unroll
        for (int i = 0; i < kStage; ++i) {
            const int r = st_row + kStageRows * i, last = n_clusters - 1 - ct * kRows;
            coff[i] = (r < last ? r : last) * row_bytes;  // beyond the last: its bias never wins
        }
        tile_bias = bias[ct * kRows + (threadIdx.x & (kRows - 1))];
    };
    auto fetch = [&](int ch) {
        const int off = ch * kChunk;
        const bool ok = off + st_piece * 16 < row_bytes;  // the last chunk may be partly empty
#pragma unroll
        for (int i = 0; i < kStage; ++i) {
            ra[i] = ok ? M::prep(*reinterpret_cast<const v4i*>(cbase + coff[i] + off)) : zero;
            rb[i] = ok ? M::prep(*reinterpret_cast<const v4i*>(qbase + qoff[i] + off)) : zero;
        }
    };
    if (tile0 < tile_end) {  // (a slice beyond the last tile: no launch has one)
        aim(tile0);
        fetch(0);
    }
    for (int ct = tile0; ct < tile_end; ++ct) {
        auto stage = [&](int buf) {
            v4i* a = smem + buf * 2 * kOperand;
            v4i* b = a + kOperand;
            if constexpr (I == 2) {
                if (ct == tile0) {
#pragma unroll
                    for (int i = 0; i < kStage; ++i)
#pragma unroll
                        for (int e = 0; e < 4; ++e) peak[i] = max(peak[i], M::magnitude((uint32_t)rb[i][e]));
                }
            }
#pragma unroll
            for (int i = 0; i < kStage; ++i) {
                if constexpr (M::kParts == 1) {
                    a[st_piece * kPieceStride + st_row + kStageRows * i] = ra[i];
                    b[st_piece * kPieceStride + st_row + kStageRows * i] = rb[i];
                } else {
                    uint2 pa[M::kParts], pb[M::kParts];
                    M::split(ra[i], pa);
                    M::split(rb[i], pb);
#pragma unroll
                    for (int p = 0; p < M::kParts; ++p) {
                        const int unit = (2 * p + (st_piece >> 1)) * kPieceStride + st_row + kStageRows * i;
                        reinterpret_cast<uint2*>(a + unit)[st_piece & 1] = pa[p];
                        reinterpret_cast<uint2*>(b + unit)[st_piece & 1] = pb[p];
                    }
                }
            }
        };
        acc_t acc[2][2];
        // the products of chunk ch; the first chunk's start from zero
        auto multiply = [&](int ch, auto first) {
            const v4i* a_chunk = smem + (ch & 1) * 2 * kOperand;
            const v4i* b_chunk = a_chunk + kOperand;
            acc_t none;
#pragma unroll
            for (int v = 0; v < 16; ++v) none[v] = 0;
            if constexpr (M::kParts == 1) {
#pragma unroll
                for (int t = 0; t < kPieces / 2; ++t) {
                    v4i a[2], b[2];
#pragma unroll
                    for (int i = 0; i < 2; ++i) a[i] = a_chunk[(2 * t + half) * kPieceStride + wc * 64 + i * 32 + col];
#pragma unroll
                    for (int s = 0; s < 2; ++s) b[s] = b_chunk[(2 * t + half) * kPieceStride + wq * 64 + s * 32 + col];
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int s = 0; s < 2; ++s) acc[i][s] = M::mma(decltype(first)::value && t == 0 ? none : acc[i][s], a[i], b[s]);
                }
            } else {
                v4i a[2][M::kParts], b[2][M::kParts];
#pragma unroll
                for (int p = 0; p < M::kParts; ++p) {
#pragma unroll
                    for (int i = 0; i < 2; ++i) a[i][p] = a_chunk[(2 * p + half) * kPieceStride + wc * 64 + i * 32 + col];
#pragma unroll
                    for (int s = 0; s < 2; ++s) b[s][p] = b_chunk[(2 * p + half) * kPieceStride + wq * 64 + s * 32 + col];
                }
                constexpr int pa[6] = {1, 0, 2, 0, 1, 0}, pb[6] = {1, 2, 0, 1, 0, 0};
#pragma unroll
                for (int k = 0; k < 6; ++k)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int s = 0; s < 2; ++s) acc[i][s] = M::mma(decltype(first)::value && k == 0 ? none : acc[i][s], a[i][pa[k]], b[s][pb[k]]);
            }
        };
        // two buffers: a wavefront that is a tile ahead has passed a barrier that the last reader of this buffer had to reach
        score_t* const bias_now = bias_lds + (ct & 1) * kRows;
        if (threadIdx.x < kRows) bias_now[threadIdx.x] = tile_bias;
        stage(0);
        __syncthreads();
        if (chunks > 1) fetch(1);
        multiply(0, std::true_type());
        if (chunks > 1) stage(1);
        __syncthreads();
        for (int ch = 1; ch < chunks; ++ch) {
            if (ch + 1 < chunks) fetch(ch + 1);
            multiply(ch, std::false_type());
            if (ch + 1 < chunks) stage((ch + 1) & 1);
            __syncthreads();
        }
        // the next tile's first chunk is on its way while this one's scores are looked at
        if (ct + 1 < tile_end) {
            aim(ct + 1);
            fetch(0);
        }
        // result element v of a lane is row 8 (v / 4) + 4 half + v % 4 of its 32-row tile
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int base = ct * kRows + wc * 64 + i * 32 + 4 * half;
            score_t bs[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) bs[v] = bias_now[wc * 64 + i * 32 + 4 * half + 8 * (v / 4) + (v % 4)];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                if constexpr (RC <= 2) {  // an insertion is a few instructions
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        insert_nearest<RC>(best_s[s], best_i[s], M::score(bs[v], acc[i][s][v], METRIC == 0), base + 8 * (v / 4) + (v % 4));
                } else {
                    take_best(best_s[s], best_i[s], acc[i][s], bs, base);
                }
            }
        }
    }

    if constexpr (I == 2) {
        // the kMoved threads of a row are neighbours; the barrier below is before the bits are read
        static_assert(kMoved == 4, "a quad of lanes per row");
#pragma unroll
        for (int i = 0; i < kStage; ++i) {
            uint32_t top = peak[i];
            top = max(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0xB1, 0xf, 0xf, true));  // quad_perm [1,0,3,2]
            top = max(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x4E, 0xf, 0xf, true));  // quad_perm [2,3,0,1]
            const int r = st_row + kStageRows * i;
            if (st_piece == 0 && M::apart(top)) atomicOr(&apart[r >> 5], 1u << (r & 31));
        }
    }

    // A query's candidates sit in four ascending lists: two lanes (halves) in each of the two wavefronts that
    // hold its row of the tile.  They meet in LDS (the staging buffers are free now) and one thread per
    // query merges them.
    uint64_t* pool = reinterpret_cast<uint64_t*>(smem);  // [query 0..127][list 0..3][RC]
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int r = 0; r < RC; ++r)
            pool[((wq * 64 + s * 32 + col) * 4 + wc * 2 + half) * RC + r] =
                ((uint64_t)M::ordered(best_s[s][r]) << 32) | (uint32_t)best_i[s][r];
    __syncthreads();
    const int64_t q = q0 + threadIdx.x;
    bool wanted = threadIdx.x < kRows && q < nq;
    if constexpr (I >= 2) wanted = wanted && (apart[(threadIdx.x >> 5) & 3] >> (threadIdx.x & 31) & 1u) == (I == 3 ? 1u : 0u);
    if (wanted) {
        const uint64_t* mine = pool + threadIdx.x * 4 * RC;
        int at[4] = {0, 0, 0, 0};
        for (int r = 0; r < RC; ++r) {
            uint64_t best = ~0ull;
            int from = 0;
#pragma unroll
            for (int l = 0; l < 4; ++l) {
                const uint64_t x = at[l] < RC ? mine[l * RC + at[l]] : ~0ull;
                if (x < best) {
                    best = x;
                    from = l;
                }
            }
#pragma unroll
            for (int l = 0; l < 4; ++l) at[l] += from == l ? 1 : 0;
            if (out)
                out[q * RC + r] = (int32_t)(uint32_t)best;
            else
                partial[(q * gridDim.y + blockIdx.y) * RC + r] = best;
        }
    }
}

template <int DT, int CHUNK, int METRIC, int RC>
__global__ void __launch_bounds__(256) route_mfma_kernel(const uint8_t* __restrict__ centroids,
                                                         const void* __restrict__ bias, int n_clusters,
                                                         int row_bytes, const uint8_t* __restrict__ queries,
                                                         int64_t nq, int32_t* __restrict__ out,
                                                         uint64_t* __restrict__ partial, int tiles_per_slice) {
    // [buffer 0 / 1][centroids, queries]; afterwards the pool of best lists
    __shared__ v4i smem[route_smem_units<DT, CHUNK, RC>()];
    __shared__ typename Mma<DT>::score_t bias_lds[2 * 128];
    static_assert(DT != 2 || route_operand_units<3, CHUNK>() <= route_operand_units<2, CHUNK>(), "the fp32 instruction's operands fit");
    if constexpr (DT != 2) {
        route_queries<DT, CHUNK, METRIC, RC>(smem, bias_lds, nullptr, centroids, bias, n_clusters, row_bytes, queries, nq, out, partial, tiles_per_slice);
    } else {
        // an extreme centroid counts for every query, an extreme query for itself: which queries share a workgroup
        // changes no result
        __shared__ uint32_t apart[4];
        const bool all = static_cast<const uint32_t*>(bias)[route_mfma_padded(n_clusters)] != 0u;
        if (threadIdx.x < 4) apart[threadIdx.x] = all ? ~0u : 0u;
        if (!all) route_queries<2, CHUNK, METRIC, RC>(smem, bias_lds, apart, centroids, bias, n_clusters, row_bytes, queries, nq, out, partial, tiles_per_slice);
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane((int)(apart[0] | apart[1] | apart[2] | apart[3])))
            route_queries<3, CHUNK, METRIC, RC>(smem, bias_lds, apart, centroids, bias, n_clusters, row_bytes, queries, nq, out, partial, tiles_per_slice);
    }
}

// One thread per query: the RC smallest of its slices' words.
template <int RC>
__global__ void __launch_bounds__(256) route_merge_kernel(const uint64_t* __restrict__ partial, int slices, int64_t nq,
                                                          int32_t* __restrict__ out) {
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= nq) return;
    uint64_t best[RC];
#pragma unroll
    for (int r = 0; r < RC; ++r) best[r] = ~0ull;
    for (int i = 0; i < slices * RC; ++i) {
        uint64_t c = partial[q * slices * RC + i];
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            const uint64_t lo = c < best[r] ? c : best[r];
            c = c < best[r] ? best[r] : c;
            best[r] = lo;
        }
    }
#pragma unroll
    for (int r = 0; r < RC; ++r) out[q * RC + r] = (int32_t)(uint32_t)best[r];
}

hipError_t launch_route_merge(int route_c, const uint64_t* partial, int slices, int64_t nq, int32_t* out,
                              hipStream_t stream) {
    const dim3 grid((unsigned)((nq + 255) / 256)), block(256);
#define ANN_RC(N) \
    case N: hipLaunchKernelGGL((route_merge_kernel<N>), grid, block, 0, stream, partial, slices, nq, out); break;
    switch (route_c) {
        ANN_RC(1) ANN_RC(2) ANN_RC(3) ANN_RC(4) ANN_RC(5) ANN_RC(6) ANN_RC(7) ANN_RC(8)
        default: return hipErrorInvalidValue;
    }
#undef ANN_RC
    return hipGetLastError();
}

// Slices of the centroid range (grid.y).  512 workgroups are resident (two per compute unit, for their registers); the
// slices are chosen so that the last round of workgroups is as full as can be: a workgroup costs its tiles, in chunks of
// their rows, and about two chunks besides.  25 000 queries x 8 192 centroids of 1536 bytes in five slices: 0.51 ms, in two
// (as many as fill the chip at all) 0.54 ms.
// At most 64, at least two tiles each, and partial results of at most 8 MB beyond nq * slices = 131 072.
// Bytes of a row per chunk.  128 halve the barriers and the rounds to L2, which counts where there are no more workgroups than
// places (65 536 queries); 64 pad rows less and halve the LDS, which counts in long batches, most for uint8, whose products take
// half the time.  64 / 128, us: 200 000 queries x 500 centroids, uint8 rows of 192 bytes 55 / 72, 512 124 / 157, 1 536 401 / 567, fp16
// rows of 192 40 / 51, 448 85 / 88, 704 122 / 126, 1 024 160 / 156, 1 536 282 / 244; 107 837 x 3 687 fp16 128 115 / 122, 256 168 / 181, 352
// 268 / 238, 480 367 / 318; 400 000 x 117, 32 bytes: uint8 17 / 25, fp16 13 / 19;
// 20 000 x 8 000 (nearest four) uint8 192 149 / 157, 448 296 / 278, 704 459 / 423, 1 536 722 / 821, fp16 192 194 / 198, 448 266 / 234, 1 536
// 508 / 449; 60 000 x 1 000 fp16 96 20.1 / 18.8, 256 31.6 / 29.7.
static int route_mfma_chunk(int dtype, int row_bytes, int64_t nq) {
    if (dtype == 2) return 64;
    const int rest = row_bytes % 128;
    const bool half_empty = rest > 0 && rest <= 64;  // the last chunk of 128
    if (nq > 65536) return dtype == 0 || row_bytes <= 256 || half_empty ? 64 : 128;
    return (half_empty && row_bytes < 448) || (dtype == 0 && row_bytes >= 768) ? 64 : 128;
}

int route_mfma_slices(int dtype, int n_clusters, int row_bytes, int route_c, int64_t nq) {
    const int64_t groups = (nq + 127) / 128;
    const int tiles = (n_clusters + 127) / 128, chunk = route_mfma_chunk(dtype, row_bytes, nq), chunks = (row_bytes + chunk - 1) / chunk;
    int best = 1;
    int64_t best_cost = 0;
    for (int s = 1; s <= 64 && s <= (tiles > 1 ? tiles / 2 : 1); ++s) {
        if (s > 1 && nq * s > 131072 && nq * s * route_c * 8 > (8 << 20)) break;
        const int64_t cost = (groups * s + 511) / 512 * ((int64_t)((tiles + s - 1) / s) * chunks + 2);
        if (s == 1 || cost < best_cost) {
            best = s;
            best_cost = cost;
        }
    }
    return best;
}

template <int DT, int CHUNK, int METRIC>
static hipError_t launch_rc(int rc, const uint8_t* centroids, const void* bias, int n_clusters, int row_bytes,
                            const uint8_t* queries, int64_t nq, int32_t* out, uint64_t* partial, int slices,
                            hipStream_t stream) {
    const int all_tiles = (n_clusters + 127) / 128;
    const int tiles_per_slice = (all_tiles + slices - 1) / slices;
    slices = route_mfma_used_slices(n_clusters, slices);
    const dim3 grid((unsigned)((nq + 127) / 128), (unsigned)slices), block(256);
#define ANN_RC(N)                                                                                                 \
    case N:                                                                                                       \
        hipLaunchKernelGGL((route_mfma_kernel<DT, CHUNK, METRIC, N>), grid, block, 0, stream, centroids, bias, n_clusters, \
                           row_bytes, queries, nq, slices > 1 ? nullptr : out, partial, tiles_per_slice);         \
        break;
    switch (rc) {
        ANN_RC(1) ANN_RC(2) ANN_RC(3) ANN_RC(4) ANN_RC(5) ANN_RC(6) ANN_RC(7) ANN_RC(8)
        default:
            if constexpr (DT != 0) {  // lists with spare words
                switch (rc) {
                    ANN_RC(9) ANN_RC(10) ANN_RC(11)
                    default:
                        if constexpr (DT == 2) {
                            switch (rc) {
                                ANN_RC(12)
                                default: return hipErrorInvalidValue;
                            }
                            break;
                        }
                        return hipErrorInvalidValue;
                }
                break;
            }
            return hipErrorInvalidValue;
    }
#undef ANN_RC
    if (slices > 1 && out) return launch_route_merge(rc, partial, slices, nq, out, stream);
    return hipGetLastError();
}

template <int DT, int METRIC>
static hipError_t launch_bias(const uint8_t* centroids, int n_clusters, int row_bytes, void* bias, hipStream_t stream) {
    const int padded = route_mfma_padded(n_clusters);
    if (DT != 0) hipLaunchKernelGGL(route_clear_words_kernel, dim3(1), dim3(3), 0, stream, static_cast<uint32_t*>(bias) + padded);
    hipLaunchKernelGGL((route_bias_kernel<DT, METRIC>), dim3((unsigned)((padded + 255) / 256)), dim3(256), 0, stream,
                       centroids, n_clusters, padded, row_bytes, bias);
    return hipGetLastError();
}

#define ANN_DISPATCH(CALL)                                     \
    switch (dtype * 2 + metric) {                              \
        case 0: return CALL(0, 0);                             \
        case 1: return CALL(0, 1);                             \
        case 2: return CALL(1, 0);                             \
        case 3: return CALL(1, 1);                             \
        case 4: return CALL(2, 0);                             \
        case 5: return CALL(2, 1);                             \
        default: return hipErrorInvalidValue;                  \
    }

hipError_t launch_route_bias(int dtype, int metric, const uint8_t* centroids, int n_clusters, int row_bytes, void* bias,
                             hipStream_t stream) {
#define ANN_CALL(D, M) launch_bias<D, M>(centroids, n_clusters, row_bytes, bias, stream)
    ANN_DISPATCH(ANN_CALL)
#undef ANN_CALL
}

hipError_t launch_route_mfma(int dtype, int metric, int route_c, const uint8_t* centroids, const void* bias,
                             int n_clusters, int row_bytes, const uint8_t* queries, int64_t nq, int32_t* out,
                             uint64_t* partial, int slices, hipStream_t stream) {
    if ((slices > 1 || !out) && !partial) return hipErrorInvalidValue;
    const bool half = route_mfma_chunk(dtype, row_bytes, nq) == 64;
#define ANN_CALL(D, M)                                                                                                          \
    (D == 2 || half ? launch_rc<D, 64, M>(route_c, centroids, bias, n_clusters, row_bytes, queries, nq, out, partial, slices, stream) \
                    : launch_rc<D, D == 2 ? 64 : 128, M>(route_c, centroids, bias, n_clusters, row_bytes, queries, nq, out, partial, slices, stream))
    ANN_DISPATCH(ANN_CALL)
#undef ANN_CALL
}

}  // namespace ann
