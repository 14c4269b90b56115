// The local half of Fantasy's stage 4 ("Combine vector candidate results", Sec. 3.1): a rank
// returns the vectors of its top-k, not only their ids, and the origin merges the k*c
// candidates it receives for a query into the final top-k.
//
//   gather_rows_kernel   out[i] = vectors[ids[i]] (zeros for id < 0); G lanes move one row in
//                        16-byte pieces, so a 128-byte row is one full-line load and store.
//   merge_runs_kernel, merge_topk_kernel    the c lists of k (key, id) pairs are loaded as packed
//                        64-bit words, put in order by register bitonic networks and the first k
//                        written back.  Order: (key, id) ascending, padding (id < 0) last.
#include <hip/hip_runtime.h>

#include "combine.h"
#include "row_ops.h"

namespace ann {

__global__ void __launch_bounds__(256) gather_rows_kernel(const uint8_t* __restrict__ vectors, int64_t n,
                                                          int64_t row_stride, int row_bytes, uint64_t pieces_inv,
                                                          const int32_t* __restrict__ ids, int64_t count,
                                                          uint8_t* __restrict__ out) {
    const int pieces = row_bytes >> 4;
    const int64_t total = count * pieces;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        // i / pieces as the high half of i * ceil(2^64 / pieces): exact while i * pieces^2 < 2^64 (pieces <= 384)
        const int64_t r = pieces_inv ? (int64_t)__umul64hi((uint64_t)i, pieces_inv) : i / pieces;
        const int p = (int)(i - r * pieces);
        const int32_t id = ids[r];
        u32x4 v = {0, 0, 0, 0};
        if (id >= 0 && (int64_t)id < n)
            v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(vectors + (int64_t)id * row_stride + p * 16));
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(out + r * row_bytes + p * 16));
    }
}

// keys are int32 (uint8 data) or float; both are turned into order-preserving uint32
template <bool FLOAT_KEYS>
__device__ __forceinline__ uint64_t pack_candidate(int32_t id, uint32_t raw) {
    const uint32_t okey = FLOAT_KEYS ? float_to_ordered(__builtin_bit_cast(float, raw)) : (raw ^ 0x80000000u);
    return id >= 0 ? ((uint64_t)okey << 32) | (uint32_t)id : kInfKey;
}
template <bool FLOAT_KEYS>
__device__ __forceinline__ void write_candidate(uint64_t v, int32_t* id, uint32_t* key) {
    const bool have = v != kInfKey;
    const uint32_t okey = (uint32_t)(v >> 32);
    *id = have ? (int32_t)(uint32_t)v : -1;
    *key = !have ? (FLOAT_KEYS ? 0x7f800000u : 0x7fffffffu)
                 : (FLOAT_KEYS ? __builtin_bit_cast(uint32_t, ordered_to_float(okey)) : (okey ^ 0x80000000u));
}

// k <= 64: P lanes per query, R candidates per lane.  Only the K smallest are wanted (K >= k, a power of two, at most P): every
// run of K lanes is sorted by itself, and two runs are merged by keeping the smaller of an element of one and of its mirror
// image in the other, which leaves the K smallest of both as one bitonic run.  Bound by the vector ALU: 10 of 80 candidates
// take a quarter of the instructions that sorting 128 places takes.  100 000 queries:
// 24 us where the whole sort took 49 us.
template <bool FLOAT_KEYS, int P, int R, int K>
__global__ void __launch_bounds__(256) merge_runs_kernel(const int32_t* __restrict__ ids, const uint32_t* __restrict__ keys,
                                                         int64_t nq, int per_query, int k,
                                                         int32_t* __restrict__ out_ids, uint32_t* __restrict__ out_keys) {
    const int lane = lane_id(), sub = lane % P;
    const int64_t q = (int64_t)blockIdx.x * (256 / P) + threadIdx.x / P;
    uint64_t v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = r * P + sub;
        v[r] = kInfKey;
        if (q < nq && e < per_query) v[r] = pack_candidate<FLOAT_KEYS>(ids[q * per_query + e], keys[q * per_query + e]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint64_t one[1] = {v[r]};
        bitonic_sort_runs<1, K>(one, lane);
        v[r] = one[0];
    }
    auto keep = [&](uint64_t a, uint64_t mirrored) {
        uint64_t one[1] = {mirrored < a ? mirrored : a};
        bitonic_clean<1, K / 2>(one, lane);
        return one[0];
    };
#pragma unroll
    for (int r = 1; r < R; ++r) v[0] = keep(v[0], xor_lane64<K - 1>(v[r], lane));
    if constexpr (K < 32 && P > 16) v[0] = keep(v[0], xor_lane64<31>(v[0], lane));
    if constexpr (K < 64 && P > 32) v[0] = keep(v[0], xor_lane64<63>(v[0], lane));
    if (q < nq && sub < k) write_candidate<FLOAT_KEYS>(v[0], out_ids + q * k + sub, out_keys + q * k + sub);
}

// k > 64: one wavefront sorts all of a query's candidates.
template <bool FLOAT_KEYS, int R>
__global__ void __launch_bounds__(64) merge_topk_kernel(const int32_t* __restrict__ ids, const uint32_t* __restrict__ keys,
                                                        int64_t nq, int per_query, int k,
                                                        int32_t* __restrict__ out_ids, uint32_t* __restrict__ out_keys) {
    const int lane = lane_id();
    const int64_t q = blockIdx.x;
    if (q >= nq) return;
    uint64_t v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = lane * R + r;
        v[r] = kInfKey;
        if (e < per_query) v[r] = pack_candidate<FLOAT_KEYS>(ids[q * per_query + e], keys[q * per_query + e]);
    }
    bitonic_sort<R>(v, lane);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = lane * R + r;
        if (e < k) write_candidate<FLOAT_KEYS>(v[r], out_ids + q * k + e, out_keys + q * k + e);
    }
}

hipError_t launch_gather_rows(const uint8_t* vectors, int64_t n, int64_t row_stride, int row_bytes, const int32_t* ids,
                              int64_t count, uint8_t* out, hipStream_t stream) {
    const int64_t total = count * (row_bytes >> 4);
    const unsigned blocks = (unsigned)((total + 255) / 256 < 65536 ? (total + 255) / 256 : 65536);
    const int pieces = row_bytes >> 4;
    const uint64_t inv = pieces > 1 && total < (int64_t)1 << 46 ? ~0ull / (uint64_t)pieces + 1 : 0;
    hipLaunchKernelGGL(gather_rows_kernel, dim3(blocks), dim3(256), 0, stream, vectors, n, row_stride, row_bytes, inv, ids,
                       count, out);
    return hipGetLastError();
}

template <bool F, int K>
static void launch_runs(const int32_t* ids, const uint32_t* keys, int64_t nq, int per_query, int k, int32_t* out_ids,
                        uint32_t* out_keys, hipStream_t stream) {
#define ANN_RUNS(P, R)                                                                                               \
    hipLaunchKernelGGL((merge_runs_kernel<F, P, R, K>), dim3((unsigned)((nq + 256 / P - 1) / (256 / P))), dim3(256), 0, stream, ids, \
                       keys, nq, per_query, k, out_ids, out_keys)
    // as few lanes per query as hold a run, while that is at most eight registers: a wavefront then has several queries, no
    // lanes are left over and no runs of different lanes have to be merged
    if constexpr (K < 64) {
        switch ((per_query + K - 1) / K) {
            case 1: ANN_RUNS(K, 1); return;
            case 2: ANN_RUNS(K, 2); return;
            case 3: ANN_RUNS(K, 3); return;
            case 4: ANN_RUNS(K, 4); return;
            case 5: ANN_RUNS(K, 5); return;
            case 6: ANN_RUNS(K, 6); return;
            case 7: case 8: ANN_RUNS(K, 8); return;
            default: break;
        }
    }
    if (per_query <= 64) ANN_RUNS(64, 1);
    else if (per_query <= 128) ANN_RUNS(64, 2);
    else if (per_query <= 256) ANN_RUNS(64, 4);
    else ANN_RUNS(64, 8);
#undef ANN_RUNS
}

template <bool F>
static hipError_t launch_merge(const int32_t* ids, const uint32_t* keys, int64_t nq, int per_query, int k, int32_t* out_ids,
                               uint32_t* out_keys, hipStream_t stream) {
    if (k <= 16) launch_runs<F, 16>(ids, keys, nq, per_query, k, out_ids, out_keys, stream);
    else if (k <= 32) launch_runs<F, 32>(ids, keys, nq, per_query, k, out_ids, out_keys, stream);
    else if (k <= 64) launch_runs<F, 64>(ids, keys, nq, per_query, k, out_ids, out_keys, stream);
    else {
        const dim3 grid((unsigned)nq), block(64);
        if (per_query <= 128) hipLaunchKernelGGL((merge_topk_kernel<F, 2>), grid, block, 0, stream, ids, keys, nq, per_query, k, out_ids, out_keys);
        else if (per_query <= 256) hipLaunchKernelGGL((merge_topk_kernel<F, 4>), grid, block, 0, stream, ids, keys, nq, per_query, k, out_ids, out_keys);
        else hipLaunchKernelGGL((merge_topk_kernel<F, 8>), grid, block, 0, stream, ids, keys, nq, per_query, k, out_ids, out_keys);
    }
    return hipGetLastError();
}

hipError_t launch_merge_topk(bool float_keys, const int32_t* ids, const void* keys, int64_t nq, int per_query, int k,
                             int32_t* out_ids, void* out_keys, hipStream_t stream) {
    const uint32_t* const in = static_cast<const uint32_t*>(keys);
    uint32_t* const out = static_cast<uint32_t*>(out_keys);
    return float_keys ? launch_merge<true>(ids, in, nq, per_query, k, out_ids, out, stream)
                      : launch_merge<false>(ids, in, nq, per_query, k, out_ids, out, stream);
}

}  // namespace ann
