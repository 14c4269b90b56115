// Matrix-core routing for uint8 vectors of 128 dimensions (route_mfma_u8.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ann {

// Length of the per-centroid bias array: n_clusters rounded up to whole tiles of 32.
inline int route_mfma_u8_padded(int n_clusters) { return (n_clusters + 31) / 32 * 32; }

// Tiles that route_nearest_u8_kernel reads at a time.
constexpr int kRouteU8StepTiles = 2;

// What the routing keeps per index, in one block of DEVICE memory (offsets in bytes):
//   bias   the per-centroid term of the score, packed with the result slot of the row inside a lane
//   shape  {tiles of centroids with an even bias, tiles}
//   half   bias / 2, rounded down, and `map`, the cluster, of every row of the tiles
//   rows   the tiles: centroids shifted into int8, in the order the matrix instruction reads them
// The tiles hold the centroids whose bias is even first, then the others, each class in ascending order and padded to
// whole tiles of 32 rows.  (Inner product: all are in the first class and `half` is the bias itself.)
struct RouteU8Block {
    size_t bias, shape, half, map, rows, bytes;
    explicit RouteU8Block(int n_clusters) {
        const size_t padded = (size_t)route_mfma_u8_padded(n_clusters), tiles = padded / 32 + kRouteU8StepTiles;
        auto up = [](size_t v) { return (v + 255) / 256 * 256; };
        bias = 0;
        shape = up(4 * padded);
        half = shape + 256;
        map = half + up(128 * tiles);
        rows = map + up(128 * tiles);
        bytes = rows + 4096 * tiles;
    }
};

// Fills the block.
hipError_t launch_route_u8_block(int metric, const uint8_t* centroids, int n_clusters, void* block, hipStream_t stream);

// Slices to cut the centroid range into for a batch of nq queries (1 for large batches).
int route_mfma_u8_slices(int n_clusters, int64_t nq);

// out[q][0..route_c): the nearest clusters of query q under (key, cluster index), ascending.
// slices > 1 needs `partial`: DEVICE scratch of nq * slices * route_c uint64.
hipError_t launch_route_mfma_u8(int metric, int route_c, const uint8_t* centroids, const void* block, int n_clusters,
                                const uint8_t* queries, int64_t nq, int32_t* out, uint64_t* partial, int slices,
                                hipStream_t stream);

}  // namespace ann
