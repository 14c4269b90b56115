// Matrix-core routing for any element type and row length (route_mfma.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ann {

// Entries of the per-centroid bias array: n_clusters rounded up to whole tiles of 128 rows.
constexpr int route_mfma_padded(int n_clusters) { return (n_clusters + 127) / 128 * 128; }

// Bytes of what launch_route_bias fills: the array, and for float types three words behind it.
inline size_t route_mfma_bias_bytes(int n_clusters) { return 4 * ((size_t)route_mfma_padded(n_clusters) + 3); }

// bias (4 bytes per entry: int32 for uint8 data, float otherwise): the per-centroid term of the
// score; padding entries get a value that never wins.  Float types: the first word behind the array is 0 unless a centroid of
// fp32 is out of the range of the bf16 parts (route_mfma.hip), the second the largest |c|^2, the third the sum of all.
hipError_t launch_route_bias(int dtype, int metric, const uint8_t* centroids, int n_clusters, int row_bytes, void* bias,
                             hipStream_t stream);

// Small batches leave most CUs idle when every workgroup walks all centroids, so the centroid
// range is cut into slices (grid.y): about 512 workgroups, each slice at least `min_steps`
// steps long, at most 64 slices.  `steps` = steps of the centroid loop (tiles or tile pairs).
inline int route_slices(int steps, int min_steps, int64_t nq) {
    const int64_t groups = (nq + 255) / 256;
    int64_t s = 512 / groups;
    if (s > steps / min_steps) s = steps / min_steps;
    if (s > 64) s = 64;
    return s < 1 ? 1 : (int)s;
}
// Of `slices` asked for, as many as leave none empty.
inline int route_mfma_used_slices(int n_clusters, int slices) {
    const int tiles = route_mfma_padded(n_clusters) / 128, each = (tiles + slices - 1) / slices;
    return (tiles + each - 1) / each;
}
int route_mfma_slices(int dtype, int n_clusters, int row_bytes, int route_c, int64_t nq);

// Each slice leaves its best (ordered score << 32 | cluster) words in partial[q][slice][route_c],
// ascending; this picks the route_c smallest per query.
hipError_t launch_route_merge(int route_c, const uint64_t* partial, int slices, int64_t nq, int32_t* out,
                              hipStream_t stream);

// out[q][0..route_c): the nearest clusters of query q under (score, cluster index), ascending.
// slices > 1 needs `partial`: DEVICE scratch of nq * slices * route_c uint64.  Without `out` the slices' words are all that is
// wanted, of any number of slices; route_c may then be up to 11 (fp16) or 12 (fp32).
hipError_t launch_route_mfma(int dtype, int metric, int route_c, const uint8_t* centroids, const void* bias,
                             int n_clusters, int row_bytes, const uint8_t* queries, int64_t nq, int32_t* out,
                             uint64_t* partial, int slices, hipStream_t stream);

// A score and its cluster into an ascending list: behind all scores that are no larger, and what is larger moves on.  (What moves on
// must not be compared again: it would end behind its equals, or be lost to them.)
template <int RC, class S>
__device__ __forceinline__ void insert_nearest(S (&list_s)[RC], int32_t (&list_i)[RC], S score, int32_t cluster) {
    bool here = score < list_s[RC - 1];
#pragma unroll
    for (int r = RC - 1; r >= 1; --r) {
        const bool moves = score < list_s[r - 1];
        list_s[r] = moves ? list_s[r - 1] : here ? score : list_s[r];
        list_i[r] = moves ? list_i[r - 1] : here ? cluster : list_i[r];
        here = moves;
    }
    list_s[0] = here ? score : list_s[0];
    list_i[0] = here ? cluster : list_i[0];
}

}  // namespace ann
