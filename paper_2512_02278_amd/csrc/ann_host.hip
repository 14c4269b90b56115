// Host side of libann: argument checks, choice of kernel variant, launches.
// Declarations and the meaning of every argument: include/ann.h.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>

#include "ann.h"
#include "cluster_search.h"
#include "combine.h"
#include "graph_build.h"
#include "key_table.h"
#include "rank_search.h"
#include "route_mfma.h"
#include "route_mfma_u8.h"
#include "schedule.h"
#include "variants.h"

namespace ann {

// explicit specialisations live in the inst_*.hip files
#define ANN_DECLARE(DT, METRIC, G, NCH)                                                                           \
    template <>                                                                                                  \
    hipError_t launch_search<DT, METRIC, G, NCH>(const SearchParams&, int, int, unsigned, size_t, hipStream_t);   \
    template <>                                                                                                  \
    hipError_t launch_route<DT, METRIC, G, NCH>(const RouteParams&, hipStream_t);
ANN_ROW_VARIANTS(ANN_DECLARE)
#undef ANN_DECLARE

struct RowVariant {
    int dtype, metric, g, nch;
    hipError_t (*search)(const SearchParams&, int, int, unsigned, size_t, hipStream_t);
    hipError_t (*route)(const RouteParams&, hipStream_t);
};

#define ANN_ENTRY(DT, METRIC, G, NCH) {DT, METRIC, G, NCH, &launch_search<DT, METRIC, G, NCH>, &launch_route<DT, METRIC, G, NCH>},
static const RowVariant kRowVariants[] = {ANN_ROW_VARIANTS(ANN_ENTRY)};
#undef ANN_ENTRY

template <>
hipError_t launch_cluster_search<kL2, 4, 2>(const ClusterParams&, int, unsigned, unsigned, size_t, hipStream_t);
template <>
hipError_t launch_cluster_search<kL2, 8, 2>(const ClusterParams&, int, unsigned, unsigned, size_t, hipStream_t);
template <>
hipError_t launch_cluster_search<kIP, 4, 2>(const ClusterParams&, int, unsigned, unsigned, size_t, hipStream_t);
template <>
hipError_t launch_cluster_search<kIP, 8, 2>(const ClusterParams&, int, unsigned, unsigned, size_t, hipStream_t);

static thread_local char g_error[512] = "";

static int fail(int code, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_error, sizeof(g_error), fmt, ap);
    va_end(ap);
    return code;
}

static int elem_size(int dtype) { return dtype == ANN_U8 ? 1 : dtype == ANN_F16 ? 2 : 4; }

constexpr uint32_t kMagic = 0x414e4e31u;  // "ANN1"
constexpr int kMaxItopk = 512, kMaxBatch = 512, kMaxWidth = 64;
constexpr int64_t kMaxQueriesPerLaunch = 1 << 22;
// Visited bitmap over the routed clusters: 8192 ids cover a cluster of the 100M / 16384
// partition (about 6100 ids) with room to spare; ids beyond it use the hash.
constexpr int kDefaultWindowBits = 8192, kMaxWindowBits = 1 << 17;
// From this batch size on, a routed batch is executed grouped by cluster (schedule.hip).
constexpr int64_t kMinQueriesForClusterOrder = 16384;
constexpr int64_t kTableBytes = 1ll << 30;
constexpr int64_t kMinQueriesToLeaveSome = 20000;  // see rank_rows

}  // namespace ann

namespace ann {

// Lets the calling thread allocate and query events while another thread captures a stream: that neither fails nor
// invalidates the other's capture (this call's own stream is not being captured, or it would not be here).
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

// Device memory for the key tables of a handle's calls, kept from call to call: allocated and released per call, even
// from a pool that stays mapped, 300 MB held the calling thread for 0.5 ms.  At most kMost blocks of at most kTableBytes,
// one for each call in flight; given back with the handle.  Any number of threads and streams: a block belongs to one call
// from take() to give_back(), and then to the stream of that call until its work has ended.  A block that is too small is
// replaced, in the order of the call's stream: nothing waits for the device.  A call that finds no block for itself searches
// without a table: it never waits for another stream's work, and no thread waits for another one's allocation.
struct TableBlocks {
    static constexpr int kMost = 4;
    struct Block {
        void* memory = nullptr;
        size_t bytes = 0;
        hipEvent_t done = nullptr;     // after the last user's work
        hipStream_t stream = nullptr;  // of the last user
        bool taken = false;
    };
    std::mutex mutex;
    Block blocks[kMost];

    // A block of at least `bytes` for a call on `stream`, or null.
    Block* take(size_t bytes, hipStream_t stream) {
        RelaxedCapture relaxed;
        Block *fits = nullptr, *small = nullptr, *empty = nullptr;
        Block* b;
        {
            std::lock_guard<std::mutex> lock(mutex);
            for (Block& c : blocks) {
                if (c.taken) continue;
                if (!c.memory) empty = &c;
                else if (c.stream == stream || idle(c)) (c.bytes >= bytes ? fits : small) = &c;
            }
            b = fits ? fits : small ? small : empty;
            if (!b) return nullptr;
            b->taken = true;
        }
        // what the stream does from here on comes after the last user's work (which is of this stream, unless this is a new
        // stream at a destroyed one's address, or has ended)
        bool ready = !b->memory || hipStreamWaitEvent(stream, b->done, 0) == hipSuccess;
        if (ready && b->bytes < bytes) {
            drop(b, stream);
            ready = allocate(b, bytes, stream);
            if (!ready) {
                std::lock_guard<std::mutex> lock(mutex);
                for (Block& c : blocks)
                    if (!c.taken && c.memory && idle(c)) drop(&c, stream);
                ready = allocate(b, bytes, stream);
            }
        }
        if (ready) return b;
        (void)hipGetLastError();
        std::lock_guard<std::mutex> lock(mutex);
        b->taken = false;
        return nullptr;
    }

    // The call's work on the block has been enqueued on `stream`.
    void give_back(Block* b, hipStream_t stream) {
        std::lock_guard<std::mutex> lock(mutex);
        b->stream = stream;
        // without the event nobody could tell when the work has ended: the block is not handed out again
        b->taken = hipEventRecord(b->done, stream) != hipSuccess;
    }

    void release() {
        for (Block& b : blocks) {
            if (b.memory) (void)(b.taken ? hipDeviceSynchronize() : hipEventSynchronize(b.done));  // searches still running
            if (b.memory) (void)hipFree(b.memory);
            if (b.done) (void)hipEventDestroy(b.done);
            b = Block();
        }
    }

   private:
    static bool idle(const Block& b) {
        const bool ended = hipEventQuery(b.done) == hipSuccess;
        if (!ended) (void)hipGetLastError();  // "not ready" is no error
        return ended;
    }
    static void drop(Block* b, hipStream_t stream) {
        if (b->memory) (void)hipFreeAsync(b->memory, stream);
        b->memory = nullptr;
        b->bytes = 0;
    }
    static bool allocate(Block* b, size_t bytes, hipStream_t stream) {
        const size_t step = size_t(32) << 20, rounded = (bytes + step - 1) / step * step;
        if (!b->done && hipEventCreateWithFlags(&b->done, hipEventDisableTiming) != hipSuccess) b->done = nullptr;
        if (!b->done || hipMallocAsync(&b->memory, rounded, stream) != hipSuccess) {
            b->memory = nullptr;
            (void)hipGetLastError();
            return false;
        }
        b->bytes = rounded;
        return true;
    }
};

}  // namespace ann

struct ann_index {
    uint32_t magic;
    ann_index_desc_t d;
    int row_bytes;
    const ann::RowVariant* variant;
    // set by ann_index_set_option:
    int hash_bits_bias;       // extra (or fewer) bits for the visited hash
    int window_bits;          // size of the visited bitmap over the routed clusters' ids
    int64_t cluster_order_min;  // batches of at least this many queries run grouped by cluster; < 0: never
    int team;                   // wavefronts per query; 0: chosen per call from the batch size and the row length
    bool matrix_core_routing;
    void* centroid_bias;     // DEVICE, owned: RouteU8Block of the uint8 d=128 matrix-core routing, or null
    void* route_bias;        // DEVICE, owned: the same for the general matrix-core routing, or null
    ann::TableBlocks tables;  // DEVICE, owned: memory for key tables
    int64_t longest_cluster;  // rows of the longest cluster, or a bound on it
    bool by_clusters;         // whether searches by whole clusters (cluster_search.h) were looked at and fit
    double leaving, far;      // shares of graph edges that leave their cluster, and of keys that are too far, if so
    double in_long, copied;   // shares of the rows in clusters too long for the search by rank, and of rows of which there are many copies
};

using namespace ann;

// The smallest variant that covers the row; among equals the one with fewer lanes per row (more rows
// per instruction).  lanes != 0 restricts the choice to variants with that many lanes per row.
static const RowVariant* pick_variant(int dtype, int metric, int64_t row_bytes, int lanes) {
    const RowVariant* best = nullptr;
    for (const RowVariant& v : kRowVariants)
        if (v.dtype == dtype && v.metric == metric && (int64_t)v.g * v.nch * 16 >= row_bytes && (lanes == 0 || v.g == lanes) &&
            (!best || v.g * v.nch < best->g * best->nch || (v.g * v.nch == best->g * best->nch && v.g < best->g)))
            best = &v;
    return best;
}

constexpr int kMaxClusterRowBytes = 256, kFarRows = 1024, kCopiedRows = 128, kManyCopies = 12;
constexpr int64_t kSampledEdges = 1ll << 24;
constexpr float kMostNormRatio = 8.0f;  // largest |c|^2 to their mean

// What ann_index_load finds out about an index whose clusters may be searched whole (DEVICE, behind what the routing keeps).
struct ClusterSample {
    unsigned long long longest;  // rows of the longest cluster
    uint32_t leaving;            // sampled graph edges that leave the cluster
    uint32_t far;                // uint8: sampled keys that are too far above the smallest for a word of cluster_search.h
    uint32_t copied;             // others: sampled rows of which a cluster holds kManyCopies or more
    unsigned long long in_long;  // rows in clusters that are too long for the search by rank
};

// One workgroup: the longest cluster, the rows in those of more than `most_ranked`, and zeros for what sample_clusters_kernel adds up.
static __global__ void __launch_bounds__(1024) longest_cluster_kernel(const int64_t* off, int n_clusters, ClusterSample* out, int64_t most_ranked) {
    __shared__ unsigned long long longest, in_long;
    if (threadIdx.x == 0) longest = in_long = 0;
    __syncthreads();
    int64_t most = 0, rows = 0;
    for (int c = (int)threadIdx.x; c < n_clusters; c += 1024) {
        const int64_t size = off[c + 1] - off[c];
        most = max(most, size);
        rows += size > most_ranked ? size : 0;
    }
    atomicMax(&longest, (unsigned long long)most);
    if (rows) atomicAdd(&in_long, (unsigned long long)rows);
    __syncthreads();
    if (threadIdx.x == 0) *out = ClusterSample{longest, 0u, 0u, 0u, in_long};
}

// A workgroup takes runs of 64 rows, `step` rows from start to start, and counts the graph edges that leave their cluster.  The first
// kFarRows workgroups also look at the keys of 64 rows of a cluster as seen from another of its rows (uint8).
static __global__ void __launch_bounds__(64) sample_clusters_kernel(ann_index_desc_t d, int row_bytes, int64_t runs, int64_t step, ClusterSample* sample) {
    const int lane = lane_id();
    const int64_t* const off = static_cast<const int64_t*>(d.cluster_offsets);
    const unsigned long long longest = sample->longest;
    if (d.dtype == ANN_U8 && longest > (unsigned long long)kMaxClusterRows) return;  // not searched by whole clusters whatever is found
    uint32_t leaving = 0;
    for (int64_t run = blockIdx.x; run < runs; run += gridDim.x) {
        const int64_t row = run * step + lane;
        int at = 0, end = d.n_clusters;  // the last cluster that starts at or before the row
        while (end - at > 1) {
            const int mid = at + (end - at) / 2;
            if (off[mid] <= row) at = mid;
            else end = mid;
        }
        // the bounds of the row's cluster (a row of none: all ids)
        int lo = 0, hi = (int)d.n;
        if (row < d.n && off[at] <= row && row < off[at + 1] && off[at + 1] <= d.n) {
            lo = off[at] < 0 ? 0 : (int)off[at];
            hi = (int)off[at + 1];
        }
        const int32_t* const edges = d.graph + run * step * d.degree;
        const int rows = d.n - run * step < 64 ? (int)(d.n - run * step) : 64;
        int r = lane / d.degree, c = lane % d.degree;
        const int over_r = 64 / d.degree, over_c = 64 % d.degree;
        for (int i0 = 0; i0 < d.degree; i0 += 8) {
            int32_t id[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int at_edge = (i0 + u) * 64 + lane;
                id[u] = at_edge < rows * d.degree ? edges[at_edge] : -1;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int from = __shfl(lo, r), to = __shfl(hi, r);  // (r is beyond 63 only past the last edge)
                leaving += id[u] >= 0 && (int64_t)id[u] < d.n && (id[u] < from || id[u] >= to) ? 1u : 0u;
                r += over_r;
                c += over_c;
                if (c >= d.degree) {
                    c -= d.degree;
                    ++r;
                }
            }
        }
        if (run >= kFarRows || d.dtype != ANN_U8) continue;
        lo = __builtin_amdgcn_readfirstlane(lo);
        const int size = __builtin_amdgcn_readfirstlane(hi) - lo;
        if (size > kMaxClusterRows) continue;  // a row of none
        const int64_t other = lo + (int64_t)size * lane / 64;
        const uint8_t* const vectors = static_cast<const uint8_t*>(d.vectors);
        const uint32_t* const x = reinterpret_cast<const uint32_t*>(vectors + run * step * d.row_stride_bytes);
        const uint32_t* const y = reinterpret_cast<const uint32_t*>(vectors + other * d.row_stride_bytes);
        uint32_t xx = 0, xy = 0, yy = 0;
        for (int i = 0; i < row_bytes / 4; ++i) {
            xx = __builtin_amdgcn_udot4(x[i], x[i], xx, false);
            xy = __builtin_amdgcn_udot4(x[i], y[i], xy, false);
            yy = __builtin_amdgcn_udot4(y[i], y[i], yy, false);
        }
        const uint32_t key = d.metric == ANN_L2 ? xx + yy - 2u * xy : 0x80000000u - xy;
        uint32_t least = other == run * step ? 0xffffffffu : key;
        for (int s = 1; s < 64; s <<= 1) least = min(least, (uint32_t)__shfl_xor(least, s));
        const int sh = 1 + (longest > 1 ? 32 - __builtin_clz((uint32_t)longest - 1u) : 1);
        const uint64_t far = __ballot(key > least && key - least >= (0xffffffffu >> sh));
        if (far && lane == 0) atomicAdd(&sample->far, (uint32_t)__builtin_popcountll(far));
    }
    for (int s = 1; s < 64; s <<= 1) leaving += __shfl_xor(leaving, s);
    if (leaving && lane == 0) atomicAdd(&sample->leaving, leaving);
}

// A workgroup looks for the copies of a row in its cluster (by the first 16 bytes, 16 in the middle and the last 16), kCopiedRows of them spread
// over all.
static __global__ void __launch_bounds__(512) copied_rows_kernel(ann_index_desc_t d, int row_bytes, ClusterSample* sample) {
    constexpr int U = 6;  // rows of a thread, all loads in flight: 3 072 of a workgroup
    static_assert(512 * U >= kMaxRankRows, "a workgroup holds a cluster that is ranked");
    __shared__ int copies;
    const int64_t* const off = static_cast<const int64_t*>(d.cluster_offsets);
    const char* const vectors = static_cast<const char*>(d.vectors);
    const auto piece = [&](int64_t r, int at) { return *reinterpret_cast<const uint4*>(vectors + r * d.row_stride_bytes + at); };
    const auto equal = [](const uint4& a, const uint4& b) { return a.x == b.x && a.y == b.y && a.z == b.z && a.w == b.w; };
    const int64_t row = d.n * blockIdx.x / gridDim.x;
    int at = 0, end = d.n_clusters;  // the last cluster that starts at or before the row
    while (end - at > 1) {
        const int mid = at + (end - at) / 2;
        if (off[mid] <= row) at = mid;
        else end = mid;
    }
    const int64_t lo = off[at], size = off[at + 1] - lo;
    if (lo < 0 || lo > row || size < 1 || lo + size > d.n || lo + size <= row || size > kMaxRankRows) return;  // (the whole workgroup)
    if (threadIdx.x == 0) copies = 0;
    __syncthreads();
    const int middle = row_bytes / 32 * 16, last = row_bytes - 16;
    uint4 y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) y[u] = piece(lo + min(u * 512 + (int)threadIdx.x, (int)size - 1), 0);
    const uint4 x0 = piece(row, 0), x1 = piece(row, middle), x2 = piece(row, last);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int r = u * 512 + (int)threadIdx.x;
        if (r < size && equal(y[u], x0) && equal(piece(lo + r, middle), x1) && equal(piece(lo + r, last), x2)) atomicAdd(&copies, 1);
    }
    __syncthreads();
    if (threadIdx.x == 0 && copies >= kManyCopies) atomicAdd(&sample->copied, 1u);
}

// Whether HIP knows these bytes as device memory; clears the error if it does not.
static bool on_device(const void* p, size_t bytes) {
    hipPointerAttribute_t a;
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipPointerGetAttributes(&a, p) == hipSuccess && a.type == hipMemoryTypeDevice &&
        hipMemGetAddressRange(&base, &size, const_cast<void*>(p)) == hipSuccess)
        return bytes <= size && (size_t)(static_cast<const char*>(p) - static_cast<const char*>(base)) <= size - bytes;
    (void)hipGetLastError();
    return false;
}

static size_t padded256(size_t n) { return (n + 255) / 256 * 256; }

// Where a handle's ClusterSample is: behind the routing's block of `bytes`.
static ClusterSample* sample_behind(void* block, size_t bytes) {
    return reinterpret_cast<ClusterSample*>(static_cast<char*>(block) + padded256(bytes));
}

// A captured call keeps to what it would have allocated for a search that gathers rows.  (Nor does the default stream, asked for as
// null, take work while another stream that waits for it is being captured.)
static bool may_allocate_more(hipStream_t stream) {
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &capture) == hipSuccess) return capture == hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return false;
}

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

extern "C" const char* ann_last_error(void) { return g_error; }

namespace {

// Keys per query of a key table, unless the visited bitmap is shorter: half as long again as the mean cluster; rows beyond are gathered.
int64_t table_rows(const ann_index_t* h) {
    const int64_t mean = h->d.n / h->d.n_clusters;
    return (mean + mean / 2 + 127) / 64 * 64;
}
// Rows of the longest cluster that a search with such a table ranks.
int64_t most_ranked(const ann_index_t* h) { return table_rows(h) < kMaxRankRows ? table_rows(h) : kMaxRankRows; }

// Whether any call on the handle can search with a key table (table_stride).
bool may_use_table(const ann_index_t* h) {
    return h->d.entry_mode == ANN_ENTRY_ROUTED && h->d.route_c == 1 && h->d.dtype != ANN_U8 && h->row_bytes >= 256 && h->d.n / h->d.n_clusters >= 256;
}

// The visited bitmap of a search with a key table need not be longer than the longest cluster: of 11 to 12 KB of LDS per query
// with 512 neighbours a round it takes one.  46 239 queries over 512-byte rows, clusters of 450: 477 us, with the whole bitmap 494;
// 5 000 over 1 536-byte rows 649 and 656; 3 410 over 400-byte rows, all resident at once or not, 166 and 218.
// Without memory or an answer from the device the bitmap keeps its length.
void find_longest_cluster(ann_index_t* h) {
    RelaxedCapture relaxed;
    const size_t count = (size_t)h->d.n_clusters + 1;
    int64_t* const off = new (std::nothrow) int64_t[count];
    if (!off) return;
    if (hipMemcpy(off, h->d.cluster_offsets, count * sizeof(int64_t), hipMemcpyDeviceToHost) == hipSuccess) {
        h->longest_cluster = 0;
        for (size_t c = 0; c + 1 < count; ++c)
            if (off[c + 1] - off[c] > h->longest_cluster) h->longest_cluster = off[c + 1] - off[c];
    } else {
        (void)hipGetLastError();
    }
    delete[] off;
}

// Whether the matrix cores only list centroids and the plain kernel settles which are nearest (route_kernel.h): float rows that
// are an odd multiple of 16 bytes, whose nearest centroids have always been those of the plain kernel's keys.
bool settled_routing(const ann_index_t* h) { return h->route_bias && h->d.dtype != ANN_U8 && h->row_bytes % 32 != 0; }

// How far apart listed scores have to be grows with the largest |c|^2 of all: where that stands out, most queries would be settled by
// the plain kernel after all, and the lists be made for nothing.  Waits for the default stream.
hipError_t norms_allow_listing(const ann_index_t* h, bool* allow) {
    float norms[2];
    const hipError_t e = hipMemcpy(norms, static_cast<const float*>(h->route_bias) + route_mfma_padded(h->d.n_clusters) + 1, sizeof(norms), hipMemcpyDeviceToHost);
    *allow = e == hipSuccess && std::isfinite(norms[0]) && norms[0] <= kMostNormRatio * (norms[1] / (float)h->d.n_clusters);
    return e;
}

// The longest cluster, and how often searches by whole clusters cannot end in them.  `sample`: DEVICE memory of the handle.  Waits for
// the default stream.
hipError_t look_at_clusters(ann_index_t* h, ClusterSample* sample) {
    const int64_t most = kSampledEdges / (64 * (int64_t)h->d.degree), all = (h->d.n + 63) / 64;
    const int64_t runs = all <= most ? all : most, step = all <= most ? 64 : h->d.n / runs;
    hipLaunchKernelGGL(longest_cluster_kernel, dim3(1), dim3(1024), 0, nullptr, static_cast<const int64_t*>(h->d.cluster_offsets), h->d.n_clusters, sample, most_ranked(h));
    hipLaunchKernelGGL(sample_clusters_kernel, dim3((unsigned)(runs < 8192 ? runs : 8192)), dim3(64), 0, nullptr, h->d, h->row_bytes, runs, step, sample);
    if (h->d.dtype != ANN_U8) hipLaunchKernelGGL(copied_rows_kernel, dim3(kCopiedRows), dim3(512), 0, nullptr, h->d, h->row_bytes, sample);
    ClusterSample got;
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpy(&got, sample, sizeof(got), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return e;
    h->longest_cluster = (int64_t)got.longest;
    h->by_clusters = h->d.dtype == ANN_U8 && got.longest <= (unsigned long long)kMaxClusterRows;
    h->leaving = got.leaving / (64.0 * (double)runs * h->d.degree);
    h->far = got.far / (64.0 * (double)(runs < kFarRows ? runs : kFarRows));
    h->copied = got.copied / (double)kCopiedRows;
    h->in_long = (double)got.in_long / (double)h->d.n;
    return hipSuccess;
}

}  // namespace

extern "C" int ann_index_load(const ann_index_desc_t* desc, ann_index_t** out_handle) {
    if (!desc || !out_handle) return fail(ANN_EINVAL, "ann_index_load: null argument");
    *out_handle = nullptr;
    const ann_index_desc_t& d = *desc;
    if (!d.vectors || !d.graph) return fail(ANN_EINVAL, "ann_index_load: vectors and graph must not be null");
    if (d.n < 1 || d.n > 2147483647ll) return fail(ANN_EINVAL, "ann_index_load: n = %lld outside 1..2^31-1", (long long)d.n);
    if (d.dtype != ANN_U8 && d.dtype != ANN_F16 && d.dtype != ANN_F32)
        return fail(ANN_EINVAL, "ann_index_load: unknown dtype %d", d.dtype);
    if (d.metric != ANN_L2 && d.metric != ANN_IP) return fail(ANN_EINVAL, "ann_index_load: unknown metric %d", d.metric);
    if (d.dim < 1) return fail(ANN_EINVAL, "ann_index_load: dim = %d", d.dim);
    const int64_t row_bytes = (int64_t)d.dim * elem_size(d.dtype);
    if (row_bytes % 16 != 0)
        return fail(ANN_EINVAL, "ann_index_load: a row of %lld bytes is not a multiple of 16", (long long)row_bytes);
    if (d.row_stride_bytes < row_bytes || d.row_stride_bytes % 16 != 0 || d.row_stride_bytes > INT32_MAX)
        return fail(ANN_EINVAL,
                    "ann_index_load: row_stride_bytes = %lld (rows are %lld bytes; must be a multiple of 16 below 2^31)",
                    (long long)d.row_stride_bytes, (long long)row_bytes);
    if (!aligned16(d.vectors)) return fail(ANN_EINVAL, "ann_index_load: vectors not 16-byte aligned");
    if (d.degree < 1 || d.degree > kMaxBatch) return fail(ANN_EINVAL, "ann_index_load: degree = %d outside 1..%d", d.degree, kMaxBatch);
    if (d.n_entry < 1 || d.n_entry > kMaxBatch)
        return fail(ANN_EINVAL, "ann_index_load: n_entry = %d outside 1..%d", d.n_entry, kMaxBatch);
    if (d.entry_mode != ANN_ENTRY_UNIFORM && d.entry_mode != ANN_ENTRY_ROUTED)
        return fail(ANN_EINVAL, "ann_index_load: unknown entry_mode %d", d.entry_mode);
    if (d.entry_mode == ANN_ENTRY_ROUTED) {
        if (!d.centroids || !d.cluster_offsets) return fail(ANN_EINVAL, "ann_index_load: routed entries need centroids and cluster_offsets");
        if (!aligned16(d.centroids)) return fail(ANN_EINVAL, "ann_index_load: centroids not 16-byte aligned");
        if (d.n_clusters < 1) return fail(ANN_EINVAL, "ann_index_load: n_clusters = %d", d.n_clusters);
        if (d.route_c < 1 || d.route_c > d.n_clusters || d.route_c > kMaxRouteC)
            return fail(ANN_EINVAL, "ann_index_load: route_c = %d outside 1..min(n_clusters, %d)", d.route_c, kMaxRouteC);
    }
    const RowVariant* best = pick_variant(d.dtype, d.metric, row_bytes, 0);
    if (!best) return fail(ANN_EUNSUPPORTED, "ann_index_load: no kernel variant for rows of %lld bytes of this dtype", (long long)row_bytes);
    ann_index* h = new (std::nothrow) ann_index;
    if (!h) return fail(ANN_ENOMEM, "ann_index_load: out of host memory");
    h->magic = kMagic;
    h->d = d;
    h->row_bytes = (int)row_bytes;
    h->variant = best;
    h->hash_bits_bias = 0;
    h->window_bits = d.entry_mode == ANN_ENTRY_ROUTED ? kDefaultWindowBits : 0;
    h->cluster_order_min = kMinQueriesForClusterOrder;
    h->team = 0;
    h->matrix_core_routing = true;
    h->centroid_bias = nullptr;
    h->route_bias = nullptr;
    h->longest_cluster = d.n;
    h->by_clusters = false;
    h->leaving = 1.0;
    h->far = h->in_long = h->copied = 0.0;
    const bool mfma_route = d.entry_mode == ANN_ENTRY_ROUTED;
    // A search by whole clusters is a choice: arrays that are not known to be in place on a device (a handle that only routes may have
    // stand-ins) are not looked at, and are searched by gathering.  Loading an index of 10 000 rows takes 40 us with that look, 22
    // without; with the offsets read back, an allocation of its own and two more copies it took 79.  A million float rows with 64 edges: 107, 44 without.
    const bool look = mfma_route && ((d.route_c == 1 && d.dtype == ANN_U8 && row_bytes <= kMaxClusterRowBytes) || may_use_table(h)) &&
                      on_device(d.vectors, (size_t)(d.n - 1) * d.row_stride_bytes + row_bytes) &&
                      on_device(d.graph, (size_t)d.n * d.degree * sizeof(int32_t)) &&
                      on_device(d.cluster_offsets, ((size_t)d.n_clusters + 1) * sizeof(int64_t)) && may_allocate_more(nullptr);
    // Rows of an odd multiple of 16 bytes can do without (matrix_routing): no memory, centroids that are not known to be on a
    // device, or a default stream that takes no work because of another one's capture, are no reason to refuse them, and nothing
    // is read then.
    const bool needed = row_bytes % 32 == 0;
    RelaxedCapture relaxed;
    if (mfma_route && !(d.dtype == ANN_U8 && d.dim == 128) &&
        (needed || (on_device(d.centroids, (size_t)d.n_clusters * row_bytes) && may_allocate_more(nullptr)))) {
        hipError_t e = hipMalloc(&h->route_bias, padded256(route_mfma_bias_bytes(d.n_clusters)) + sizeof(ClusterSample));
        if (e == hipSuccess)
            e = launch_route_bias(d.dtype, d.metric, static_cast<const uint8_t*>(d.centroids), d.n_clusters,
                                  (int)row_bytes, h->route_bias, nullptr);
        bool listing = true;
        if (e == hipSuccess && look) e = look_at_clusters(h, sample_behind(h->route_bias, route_mfma_bias_bytes(d.n_clusters)));
        if (e == hipSuccess && settled_routing(h)) e = norms_allow_listing(h, &listing);
        else if (e == hipSuccess && !look) e = hipStreamSynchronize(nullptr);
        if (e != hipSuccess || !listing) {
            if (h->route_bias) (void)hipFree(h->route_bias);
            h->route_bias = nullptr;
            if (needed) {
                delete h;
                return fail(e == hipErrorOutOfMemory ? ANN_ENOMEM : ANN_EHIP, "ann_index_load: preparing the routing failed: %s",
                            hipGetErrorString(e));
            }
            (void)hipGetLastError();
        }
    }
    if (mfma_route && d.dtype == ANN_U8 && d.dim == 128) {
        // routing runs on the matrix cores; what it reads of the centroids is laid out once, here
        hipError_t e = hipMalloc(&h->centroid_bias, padded256(RouteU8Block(d.n_clusters).bytes) + sizeof(ClusterSample));
        if (e == hipSuccess)
            e = launch_route_u8_block(d.metric, static_cast<const uint8_t*>(d.centroids), d.n_clusters, h->centroid_bias, nullptr);
        if (e == hipSuccess) e = look ? look_at_clusters(h, sample_behind(h->centroid_bias, RouteU8Block(d.n_clusters).bytes)) : hipStreamSynchronize(nullptr);
        if (e != hipSuccess) {
            if (h->centroid_bias) (void)hipFree(h->centroid_bias);
            delete h;
            return fail(e == hipErrorOutOfMemory ? ANN_ENOMEM : ANN_EHIP, "ann_index_load: preparing the routing failed: %s",
                        hipGetErrorString(e));
        }
    }
    if (may_use_table(h) && h->longest_cluster == d.n) find_longest_cluster(h);  // not looked at
    *out_handle = h;
    return ANN_OK;
}

extern "C" int ann_free(ann_index_t* h) {
    if (!h) return ANN_OK;
    if (h->magic != kMagic) return fail(ANN_EINVAL, "ann_free: not a live handle");
    h->magic = 0;
    if (h->centroid_bias) (void)hipFree(h->centroid_bias);
    if (h->route_bias) (void)hipFree(h->route_bias);
    h->tables.release();
    delete h;
    return ANN_OK;
}

namespace {

struct Plan {
    int list_variant, cap, hash_bits;
    size_t lds_bytes;
};

int make_plan(const ann_index* h, int itopk, int width, Plan* plan, const char* who) {
    if (itopk < 1 || itopk > kMaxItopk) return fail(ANN_EUNSUPPORTED, "%s: itopk = %d outside 1..%d", who, itopk, kMaxItopk);
    if (width < 1 || width > kMaxWidth) return fail(ANN_EUNSUPPORTED, "%s: width = %d outside 1..%d", who, width, kMaxWidth);
    const int64_t batch = (int64_t)width * h->d.degree;
    if (batch > kMaxBatch) return fail(ANN_EUNSUPPORTED, "%s: width*degree = %lld above %d", who, (long long)batch, kMaxBatch);
    const int need = (int)(batch > h->d.n_entry ? batch : h->d.n_entry);
    int lv = -1;
    for (int i = 0; i < kNumListVariants; ++i)
        if (64 * kListVariants[i][0] >= itopk && 64 * kListVariants[i][1] >= need) {
            lv = i;
            break;
        }
    if (lv < 0) return fail(ANN_EUNSUPPORTED, "%s: no list variant for itopk = %d, batch = %d", who, itopk, need);
    plan->list_variant = lv;
    plan->cap = 64 * kListVariants[lv][1];
    // the table is emptied once 3/4 full; right after that it holds <= itopk ids and one
    // round adds <= need, so 3/4 of its size must cover itopk + need
    int bits = 6;
    while (((3 << bits) >> 2) < itopk + need) ++bits;
    bits += (h->window_bits ? 0 : 1) + h->hash_bits_bias;  // without a bitmap: one more bit, so that resets are rarer
    while (((3 << bits) >> 2) < itopk + need) ++bits;
    if (bits > 13) bits = 13;
    plan->hash_bits = bits;
    // words: round scratch (keys + ids, or a copy of the list), parents, window table, bitmap, hash
    const size_t scratch = 3 * (size_t)plan->cap > 128 * (size_t)kListVariants[lv][0] ? 3 * (size_t)plan->cap
                                                                                   : 128 * (size_t)kListVariants[lv][0];
    plan->lds_bytes = sizeof(uint32_t) * (scratch + 64 + 32 + 8 + (size_t)hash_at(h->window_bits) + (size_t(1) << bits));
    return ANN_OK;
}

}  // namespace

extern "C" int64_t ann_lds_bytes(ann_index_t* h, int itopk, int width) {
    if (!h || h->magic != kMagic) return fail(ANN_EINVAL, "ann_lds_bytes: not a live handle");
    Plan plan;
    const int rc = make_plan(h, itopk, width, &plan, "ann_lds_bytes");
    return rc != ANN_OK ? rc : (int64_t)plan.lds_bytes;
}

extern "C" int ann_index_set_option(ann_index_t* h, int option, int64_t value) {
    if (!h || h->magic != kMagic) return fail(ANN_EINVAL, "ann_index_set_option: not a live handle");
    switch (option) {
        case ANN_OPT_CLUSTER_ORDER_MIN_QUERIES:
            h->cluster_order_min = value;
            return ANN_OK;
        case ANN_OPT_VISITED_WINDOW_BITS:
            if (value < 0 || value > kMaxWindowBits)
                return fail(ANN_EINVAL, "ann_index_set_option: visited window of %lld bits outside 0..%d", (long long)value, kMaxWindowBits);
            h->window_bits = h->d.entry_mode == ANN_ENTRY_ROUTED ? (int)((value + 31) / 32 * 32) : 0;
            return ANN_OK;
        case ANN_OPT_VISITED_HASH_BITS_BIAS:
            if (value < -4 || value > 4) return fail(ANN_EINVAL, "ann_index_set_option: hash bits bias %lld outside -4..4", (long long)value);
            h->hash_bits_bias = (int)value;
            return ANN_OK;
        case ANN_OPT_MATRIX_CORE_ROUTING:
            h->matrix_core_routing = value != 0;
            return ANN_OK;
        case ANN_OPT_WAVEFRONTS_PER_QUERY:
            if (value != 0 && value != 1 && value != 2 && value != 4)
                return fail(ANN_EUNSUPPORTED, "ann_index_set_option: %lld wavefronts per query (0, 1, 2 or 4)", (long long)value);
            h->team = (int)value;
            return ANN_OK;
        case ANN_OPT_LANES_PER_ROW: {
            const RowVariant* v = value < 0 || value > 64 ? nullptr : pick_variant(h->d.dtype, h->d.metric, h->row_bytes, (int)value);
            if (!v)
                return fail(ANN_EUNSUPPORTED, "ann_index_set_option: no kernel variant with %lld lanes per row for this index", (long long)value);
            h->variant = v;
            return ANN_OK;
        }
        default:
            return fail(ANN_EINVAL, "ann_index_set_option: unknown option %d", option);
    }
}

namespace {

// Where a call's temporaries come from: consecutive 256-byte aligned pieces of one block, which is either
// given (the static scratch) or one stream-ordered allocation of `reserve` bytes, made when the first piece
// is asked for and released on the same stream once the call has enqueued its work.  One allocation per
// call, not one per temporary: on the host an allocate/release pair costs as much as several kernel launches
// (with two pairs per call, small batches in flight on four streams reached 11.9 M queries/s, with one 14.8 M).  Where `reserve`
// bytes are not to be had, the block holds `least`, what the call cannot do without.
struct Workspace {
    hipStream_t stream;
    char* base = nullptr;
    size_t bytes = 0, used = 0;
    size_t reserve = 0, least = 0;  // reserve > 0: the block is this call's own allocation (made on first use)
    bool owned = false;
    size_t routing_room = SIZE_MAX;  // bytes of it that the routing's own temporaries may take

    Workspace(hipStream_t s, size_t reserve_bytes, size_t least_bytes) : stream(s), reserve(reserve_bytes), least(least_bytes) {}
    Workspace(hipStream_t s, void* buffer, size_t buffer_bytes) : stream(s), base(static_cast<char*>(buffer)), bytes(buffer_bytes) {}
    Workspace(const Workspace&) = delete;

    // DEVICE memory of `n` bytes, 256-byte aligned, or null (the reason in *err).
    void* take(size_t n, hipError_t* err) {
        *err = hipSuccess;
        if (!base && reserve > 0) {
            void* p = nullptr;
            *err = hipMallocAsync(&p, reserve, stream);
            if (*err != hipSuccess && least > 0 && least < reserve) {
                (void)hipGetLastError();
                reserve = least;
                routing_room = 0;
                *err = hipMallocAsync(&p, reserve, stream);
            }
            if (*err != hipSuccess) {
                (void)hipGetLastError();
                reserve = 0;  // later pieces are not had either
                return nullptr;
            }
            base = static_cast<char*>(p);
            bytes = reserve;
            owned = true;
        }
        const size_t at = (used + 255) / 256 * 256;
        if (!base || at + n > bytes) {
            *err = hipErrorOutOfMemory;
            return nullptr;
        }
        used = at + n;
        return base + at;
    }
    ~Workspace() {
        if (owned) (void)hipFreeAsync(base, stream);
    }
};

// Slices of the centroid range the matrix-core routing of nq queries is cut into, with partial results of at most `room` bytes.
int routing_slices(const ann_index_t* h, int64_t nq, size_t room) {
    const int slices = h->centroid_bias ? route_mfma_u8_slices(h->d.n_clusters, nq)
                                        : route_mfma_slices(h->d.dtype, h->d.n_clusters, h->row_bytes, h->d.route_c, nq);
    if (slices <= 1) return 1;
    const size_t most = room / (sizeof(uint64_t) * (size_t)nq * h->d.route_c);
    return most >= (size_t)slices ? slices : most > 1 ? (int)most : 1;
}

// Whether nq queries are routed on the matrix cores.  Rows of a multiple of 32 bytes always are.  For the others that takes
// a second launch and memory (float) or leaves half a chunk empty, while the plain kernel's time goes with the steps it walks the centroids
// in, and from some thousand queries on with their number.  Plain / matrix, us, nearest one and eight:
//   100 queries: fp16 48-byte rows, 400 centroids (50 steps) 26 / 33, 27 / 44, 1 600 81 / 30, 80 / 51; 400-byte, 100 (50 steps) 24 / 34, 24 / 37,
//   400 71 / 31, 72 / 48; fp32 1 008-byte 400 77 / 50, 77 / 69; uint8 48-byte 400 13 / 33, 13 / 34, 1 600 38 / 33, 38 / 43; 144-byte 1 600 68 / 31, 69 / 47.
//   6 400 queries: fp16 400-byte, 100 centroids 50 / 32, 50 / 48, 400 141 / 36, 140 / 64; uint8 144-byte, 400 68 / 28, 68 / 37.
// 200 000 queries over fp16 rows of 272 bytes, 4 000 centroids: 20.05 / 0.80 ms.
bool matrix_routing(const ann_index_t* h, int64_t nq, hipStream_t stream) {
    if (!h->matrix_core_routing || !(h->centroid_bias || h->route_bias)) return false;
    if (h->row_bytes % 32 == 0) return true;
    const double steps = (double)h->d.n_clusters * h->variant->g / 64;
    return steps * (nq > 4000 ? nq / 4000.0 : 1.0) >= 64 + 16 * h->d.route_c && may_allocate_more(stream);
}
constexpr int64_t kListedQueries = 65536;  // per launch: lists of 12 are 6.3 MB then
int listed_words(const ann_index_t* h) { return h->d.route_c + route_spare_words(h->d.dtype == ANN_F32, h->row_bytes, h->d.route_c); }
int listed_slices(const ann_index_t* h, int64_t nq) {
    const int slices = route_mfma_slices(h->d.dtype, h->d.n_clusters, h->row_bytes, listed_words(h), nq < kListedQueries ? nq : kListedQueries);
    return route_mfma_used_slices(h->d.n_clusters, slices);
}
size_t listed_bytes(const ann_index_t* h, int64_t nq) {
    return sizeof(uint64_t) * (size_t)(nq < kListedQueries ? nq : kListedQueries) * listed_slices(h, nq) * listed_words(h);
}

// Bytes of temporaries the routing of nq queries takes.
size_t route_scratch_bytes(const ann_index_t* h, int64_t nq, hipStream_t stream) {
    if (nq <= 0 || !matrix_routing(h, nq, stream)) return 0;
    if (settled_routing(h)) return padded256(listed_bytes(h, nq));
    const int slices = routing_slices(h, nq, SIZE_MAX);
    return slices > 1 ? padded256(sizeof(uint64_t) * (size_t)nq * slices * h->d.route_c) : 0;
}

// How a call searches: rows gathered (all zero), with a table of keys (key_table.h) or by whole clusters (cluster_search.h).
struct Way {
    int table_stride = 0;   // keys per query
    int group = 0;          // queries per workgroup
    int waves = 0;          // wavefronts per workgroup
    int graph_words = 0;    // see ClusterParams
};

bool grouped_order(const ann_index_t* h, int64_t nq, const Way& way) {
    return h->d.entry_mode == ANN_ENTRY_ROUTED && h->cluster_order_min >= 0 &&
           (nq >= h->cluster_order_min || way.table_stride > 0 || way.group > 1) && nq <= 2147483647ll;
}

// Bytes of temporaries a whole search call of nq queries takes (what Workspace::take hands out): the routes and
// the routing's own temporaries unless the caller brings the routes, and the execution order of a large batch.
size_t search_scratch_bytes(const ann_index_t* h, int64_t nq, bool routes_given, const Way& way, hipStream_t stream) {
    if (h->d.entry_mode != ANN_ENTRY_ROUTED || nq <= 0) return 0;
    size_t need = 0;
    if (!routes_given) need += padded256(sizeof(int32_t) * (size_t)nq * h->d.route_c) + route_scratch_bytes(h, nq, stream);
    if (grouped_order(h, nq, way)) need += padded256(sizeof(int32_t) * ((size_t)nq + h->d.n_clusters));
    return need;
}

// Of those, what the call cannot do without: the routes, and the order that a large batch runs in whichever way it is searched.
size_t search_scratch_needed(const ann_index_t* h, int64_t nq, bool routes_given) {
    if (h->d.entry_mode != ANN_ENTRY_ROUTED || nq <= 0) return 0;
    return (routes_given ? 0 : padded256(sizeof(int32_t) * (size_t)nq * h->d.route_c)) +
           (grouped_order(h, nq, Way()) ? padded256(sizeof(int32_t) * ((size_t)nq + h->d.n_clusters)) : 0);
}

int route_impl(ann_index_t* h, const void* queries, int64_t nq, int32_t* out_clusters, Workspace& ws) {
    hipStream_t st = ws.stream;
    const bool matrix = matrix_routing(h, nq, st);
    if (matrix && !settled_routing(h)) {
        // matrix-core routing; small batches cut the centroid range into slices and merge them, if there is room for that
        int slices = routing_slices(h, nq, ws.routing_room);
        uint64_t* partial = nullptr;
        if (slices > 1) {
            hipError_t e;
            partial = static_cast<uint64_t*>(ws.take(sizeof(uint64_t) * (size_t)nq * slices * h->d.route_c, &e));
            if (!partial) slices = 1;
        }
        const uint8_t* cen = static_cast<const uint8_t*>(h->d.centroids);
        const uint8_t* qs = static_cast<const uint8_t*>(queries);
        const hipError_t e =
            h->centroid_bias ? launch_route_mfma_u8(h->d.metric, h->d.route_c, cen, h->centroid_bias, h->d.n_clusters, qs, nq,
                                                    out_clusters, partial, slices, st)
                             : launch_route_mfma(h->d.dtype, h->d.metric, h->d.route_c, cen, h->route_bias, h->d.n_clusters,
                                                 h->row_bytes, qs, nq, out_clusters, partial, slices, st);
        if (e != hipSuccess) return fail(ANN_EHIP, "ann_route: launch failed: %s", hipGetErrorString(e));
        return ANN_OK;
    }
    // without room for the lists the plain kernel looks at every centroid
    uint64_t* words = nullptr;
    if (matrix && settled_routing(h) && listed_bytes(h, nq) <= ws.routing_room) {
        hipError_t e;
        words = static_cast<uint64_t*>(ws.take(listed_bytes(h, nq), &e));
    }
    const int64_t most = words ? kListedQueries : kMaxQueriesPerLaunch;
    for (int64_t q0 = 0; q0 < nq; q0 += most) {
        RouteParams rp;
        rp.centroids = static_cast<const uint8_t*>(h->d.centroids);
        rp.n_clusters = h->d.n_clusters;
        rp.row_bytes = h->row_bytes;
        rp.queries = static_cast<const uint8_t*>(queries) + q0 * h->row_bytes;
        rp.nq = nq - q0 < most ? nq - q0 : most;
        rp.route_c = h->d.route_c;
        rp.out = out_clusters + q0 * h->d.route_c;
        rp.words = words;
        rp.slices = 1;
        rp.largest = nullptr;
        hipError_t e = hipSuccess;
        if (words) {
            rp.slices = listed_slices(h, nq);
            rp.largest = static_cast<const float*>(h->route_bias) + route_mfma_padded(h->d.n_clusters) + 1;
            e = launch_route_mfma(h->d.dtype, h->d.metric, listed_words(h), rp.centroids, h->route_bias, rp.n_clusters, rp.row_bytes,
                                  rp.queries, rp.nq, nullptr, words, rp.slices, st);
        }
        if (e == hipSuccess) e = h->variant->route(rp, st);
        if (e != hipSuccess) return fail(ANN_EHIP, "ann_route: launch failed: %s", hipGetErrorString(e));
    }
    return ANN_OK;
}

}  // namespace

extern "C" int ann_route(ann_index_t* h, const void* queries, int64_t nq, int32_t* out_clusters, void* stream) {
    if (!h || h->magic != kMagic) return fail(ANN_EINVAL, "ann_route: not a live handle");
    if (h->d.entry_mode != ANN_ENTRY_ROUTED) return fail(ANN_EINVAL, "ann_route: the index has no centroids");
    if (nq < 0) return fail(ANN_EINVAL, "ann_route: nq = %lld", (long long)nq);
    if (nq == 0) return ANN_OK;
    if (!queries || !out_clusters) return fail(ANN_EINVAL, "ann_route: null argument");
    if (!aligned16(queries)) return fail(ANN_EINVAL, "ann_route: queries not 16-byte aligned");
    Workspace ws(static_cast<hipStream_t>(stream), route_scratch_bytes(h, nq, static_cast<hipStream_t>(stream)), 0);
    return route_impl(h, queries, nq, out_clusters, ws);
}

namespace {

// Wavefronts per query when the caller has not fixed them.  A team pays where a round's gathers are the long pole (rows of 256
// bytes and more: a wavefront covers few of them per instruction and has a bounded number of loads in flight) and the chip is
// not full anyway: up to 1 024 queries its 1 024 SIMDs hold all wavefronts of teams of four at once.
// 1 / 2 / 4 wavefronts per query, us, uniform entries, list of 100, 81 neighbours a round, 200 000 fp16 rows in clusters of 1 000:
//     queries     50             1 000             1 500             3 001             6 000
//   256 bytes   122/120/116    166/157/150       167/158/151       184/173/253       267/335/521
//   384         175/147/128    231/201/181       231/201/251       248/285/364       454/496/699
//   400         145/126/112    216/197/181       226/204/254       259/325/393       536/517/699
//   512         143/121/108    190/166/153       200/180/249       239/295/362       527/511/681
//   768         251/186/145    293/220/187       339/270/227       443/364/349       718/704/738
//   1 024       244/189/153    304/238/199       303/249/221       429/408/413       946/910/856
//   1 536       254/187/145    301/245/216       346/314/358       615/609/576     1 313/1 260/1 208
// In a routed search most neighbours have been seen, and a round has fewer rows to gather.  List of 128, 128 neighbours a
// round, 1 000 and 1 500 queries: 384 bytes 105/107/105 and 111/115/174, 400 bytes 167/155/147 and 174/167/222, 768 bytes
// 168/142/130 and 178/160/155, 1 536 bytes 210/196/195 and 261/267/309 (6 000: 914/910/903).  List of 64, 32 neighbours: 256
// bytes 115/126/126, 384 bytes 119/132/131, 400 bytes 180/178/175, 1 536 bytes 196/189/186 (6 000: 762/765/819).  256 neighbours, 4 400
// queries: 1 024 bytes 521/517/539, 1 536 bytes 781/764/751; 512 neighbours, 3 465 queries: 1 024 bytes 728/-/653.
// Rounds of few neighbours leave a team little to share: 16 neighbours, uniform entries, 1 000 queries: 256 bytes 181/200/201, 512
// bytes 203/213/210, 768 bytes 258/231/220; 32 neighbours, 6 000 queries, 1 024 bytes 491/491/691 (17 MB of rows) and 674/683/803
// (200 MB).  Teams that are not all resident wait for each other's places: 384 neighbours, 1 400 and 2 400 queries: 256 bytes
// 256/224/316 and 369/426/515, 400 bytes 384/299/362 and 685/643/651, 768 bytes 614/422/470 and 1 034/948/880.
// Large batches of long rows are bound by bytes in flight again: 50 000 queries over 1 536 bytes 9 665 / - / 9 187.
int default_team(const ann_index_t* h, int64_t nq, int width) {
    const int bytes = h->row_bytes;
    const int64_t round = (int64_t)width * h->d.degree;
    if (bytes < 256 || (bytes <= 512 && round < 32)) return 1;
    if (h->d.entry_mode != ANN_ENTRY_UNIFORM) {
        if (h->variant->g == 32 ? nq <= (round > 256 ? 1024 : 1280) : nq <= 1024 && round >= 256) return 4;
        return (bytes >= 1024 && (nq >= 6000 || round >= 512)) || (bytes >= 1536 && nq >= 4096 && round >= 128) ? 4 : 1;
    }
    if (nq <= 1024) return 4;
    if (bytes >= 1024) return round >= 64 ? 4 : nq <= 2560 || nq >= 6000 ? 2 : 1;
    // as long as teams of two are all resident
    return nq <= (round > 256 || (h->variant->g == 32 && bytes <= 512) ? 2048 : 2560) ? 2 : 1;
}

// Share of a cluster's rows that a search is expected to score: a parent brings 3 + degree / 4 new rows, at most 15, and
// fewer the more of the cluster has been seen.  Measured / expected: list 64, degree 16, clusters of 2 441 rows 0.23 / 0.24, of 800
// 0.47 / 0.48; 112, 24, 800 0.68 / 0.70; 64, 32, 2 441 0.35 / 0.33; 128, 32, 800 0.76 / 0.78; 184, 64, 2 441 0.71 / 0.67; 256, 64, 1 600 0.85 / 0.85.
double scored_share(const ann_index_t* h, int64_t parents, int64_t mean) {
    const double fresh = h->d.degree < 48 ? 3.0 + h->d.degree / 4.0 : 15.0;
    return 1.0 - std::exp(-std::pow((double)parents * fresh / (double)mean, 0.75));
}

// Share from which a table of keys pays.  Time without / with, share expected in brackets; the lines lie between what gained and
// what lost of 1 930 pairs over 100 to 460 MB of rows:
//   * A batch long enough to run grouped by cluster gathers from the caches as it is, and the table pays for most of a cluster only:
//     256 bytes L2 0.92 [0.78], 1.04 [0.92], products 0.96 [0.60] (with 64 rounds 1.10), 1.07 [0.67]; 384 bytes 0.88 [0.48], 1.05 [0.60],
//     1.07 [0.67]; 400 bytes L2 0.88 [0.60], 1.04 [0.67]; 512 bytes fp16 0.95 [0.48], 1.1 [0.60], fp32 0.83 [0.32], 1.05 [0.48]; 768 bytes
//     L2 0.89 [0.78], 1.06 [0.96], with 512 neighbours a round 1.05 [0.67], 1.12 [0.78]; 1 536 bytes L2 0.82 [0.48], 1.35 [0.67], products
//     0.88 [0.24], 1.1 [0.32].
//   * A short batch pays for the table kernel's own length: 2 000 to 4 000 queries over 256 bytes 0.82 [0.24], 1.1 [0.40] (L2 0.97 at
//     [0.78]), 384 to 768 bytes 0.75 [0.24], 0.92 [0.33], 1.02 [0.40]; 1 000 to 1 500 queries over 1 536 bytes 0.73 [0.24], 1.20 [0.48].
double table_share(const ann_index_t* h, int64_t nq, int64_t parents, int width) {
    const int bytes = h->row_bytes;
    const bool f32 = h->d.dtype == ANN_F32, f16_l2 = !f32 && h->d.metric == ANN_L2;  // f16_l2: the most instructions per byte
    if (nq >= h->cluster_order_min) {
        if (bytes >= 1024) return f16_l2 ? 0.5 : 0.3;
        if (bytes >= 512) return f16_l2 ? ((int64_t)width * h->d.degree >= 512 ? 0.66 : 0.96) : f32 ? 0.45 : 0.49;
        if (bytes > 256) return f32 ? 0.59 : 0.65;
        return f16_l2 ? 0.86 : parents >= 48 * (int64_t)width ? 0.59 : 0.65;
    }
    if (bytes >= 1024) return nq < 1536 ? 0.38 : 0.0;
    if (nq >= 4096) return 0.0;
    return bytes > 256 ? 0.36 : f16_l2 ? 0.93 : 0.4;
}

// Keys per query of the key table (key_table.h) this call searches with, 0 for a search that gathers every row.
//
// The table costs a product of every query with every row of its cluster; it saves the rows the search would gather.
// Measured over rows of 256 to 1536 bytes, clusters of 300 to 2 441 rows and lists of 64 to 256 entries, time without / with,
// batches that are not grouped otherwise:
//   * with 16 queries per cluster (8 for rows of 1 KB), about eight rows per parent x row bytes >= 0.8 x vector instructions of the
//     products, and the shares above: 0.97 .. 1.4 at 256 bytes, 1.0 .. 2.0 at 384 bytes, 1.0 .. 4.2 above;
//   * with 4 queries per cluster 0.8 .. 1.1, and where few rows of large clusters are gathered (768-byte L2 rows, list of
//     64, clusters of 2 441) 0.6 .. 0.8 at any batch size.
// Rows below 256 bytes and clusters below 256 rows were not measured.
int table_stride(const ann_index_t* h, int64_t nq, int itopk, int width, int max_iters, hipStream_t stream) {
    if (!may_use_table(h)) return 0;
    // a fixed team, an order that is never grouped and a hash without bitmap ask for the search they describe
    if (h->team != 0 || h->cluster_order_min < 0 || h->window_bits == 0) return 0;
    const int64_t mean = h->d.n / h->d.n_clusters;
    if (nq > 2147483647ll || nq / h->d.n_clusters < (h->row_bytes >= 1024 ? 8 : 16)) return 0;
    const int64_t parents = (int64_t)width * max_iters < itopk ? (int64_t)width * max_iters : itopk;
    const int64_t gathered = 8 * parents < mean ? 8 * parents : mean;
    const int64_t twice_products = (int64_t)h->d.dim * (h->d.dtype == ANN_F16 && h->d.metric == ANN_IP ? 1 : 4);
    if (10 * gathered * h->row_bytes < 4 * twice_products * mean || scored_share(h, parents, mean) < table_share(h, nq, parents, width)) return 0;
    int64_t stride = table_rows(h);
    if (stride > h->window_bits) stride = h->window_bits;
    return may_allocate_more(stream) ? (int)stride : 0;
}

// Whether a search with a key table ranks the clusters' rows (rank_search.h): those of the longest cluster, and the ranks that it settles.
//
// Of 50 calls over 8 to 400 clusters (300 to 2 900 rows of 200 to 1 536 bytes, lists of 32 to 256, 16 to 512 neighbours a round) the whole call
// without / with ranks, and [rounds x (64 x registers of the list + 2 x neighbours - 200) over the rows of a cluster]: 0.92 [2.1], 0.95 [3.4], 0.96 [3.1],
// 0.97 [2.9], 0.98 [3.5], 0.94 [below 0: a list and a round of 64 at most], 1.09 [5.0], 1.07 [6.0], 1.18 [6.5], 1.07 [7.7], 1.10 [14], 1.19 [28], 1.25 [36]; with few
// queries, where a round's latency counts, up to 1.45.
void rank_rows(const ann_index_t* h, int64_t nq, int itopk, int width, int max_iters, int stride, SearchParams* p) {
    const int64_t parents = (int64_t)width * max_iters < itopk ? (int64_t)width * max_iters : itopk;
    // Queries that are left to another search: those that meet an edge that leaves their cluster, after they have been ranked, and those in long
    // clusters.  That search comes after this one, and a query alone takes as long as a small batch: 8 000 queries of 96 fp32 elements 407 us
    // with none in long clusters, 626 [share of the queries 0.016], 633 [0.05], 631 [0.35], without ranks 545 to 608; 5 000 of 768 fp16 elements
    // 493, 689, 705, 744, without 587 to 696.  In a large batch they may be many: 20 000 queries 780, 1 100 [0.016], 1 118 [0.05], 1 148 [0.15], 1 202 [0.35], without
    // 1 103, 1 105, 1 174, 1 198, 1 181; 768 elements 1 269, 1 531, 1 621, 1 936, 2 084, without 1 575, 1 622, 1 788, 2 246, 2 052.  Between them 18 000
    // queries with one long cluster in four hundred: 1 037, without 1 014.
    const double anew = h->leaving * (double)(parents * h->d.degree);
    if (anew > 1.0 / 128 || h->in_long > 0.2 || (nq < kMinQueriesToLeaveSome && (anew + h->in_long) * (double)nq > 0.5)) return;
    const int64_t mean = h->d.n / h->d.n_clusters, longest = h->longest_cluster < stride ? h->longest_cluster : stride;
    // (an option may cut the visited bitmap, and with it the table's rows: a query's keys are read 64 at a time, and how many clusters are too long
    // then has not been looked at)
    if (mean > kMaxRankRows || stride % 64 != 0 || (stride < table_rows(h) && stride < h->longest_cluster)) return;
    // Copies of a row meet in one bucket, whose rows are put in order one by one: where all rows have two copies 0.77 of the time without ranks, eight 1.02,
    // twenty 1.32, fifty 1.46.
    if (h->copied > 0.5) return;
    // Ranking costs as much as there are rows; it saves, a round, what the list and the neighbours cost beyond the search for
    // bits that are set.
    const int64_t rounds = (parents + width - 1) / width;
    if (2 * rounds * (64 * ((itopk + 63) / 64) + 2 * width * h->d.degree - 200) < 9 * mean) return;
    p->rank_rows = (int)(longest < kMaxRankRows ? longest : kMaxRankRows);
    // The search expands what its list holds at the end, and at first the best of its entries.  Of n entries drawn at random fewer than
    // `width` are among the nearest share f of the rows with the probability summed up here: in one of fifty calls for some query.
    const double n = h->d.n_entry, rare = 0.02 / (double)nq;
    double f = 0.0, fewer = 1.0;
    while (fewer > rare && f < 0.99) {
        f += 0.02;
        double term = std::pow(1.0 - f, n);
        fewer = 0.0;
        for (int i = 0; i < width; ++i) {
            fewer += term;
            term *= (n - i) / (i + 1) * f / (1.0 - f);
        }
    }
    if (f >= 0.99) f = 1.0;
    const int group = kRankTiles * kRankTile, most = (p->rank_rows + group - 1) / group * group;
    const double want = std::fmax(f * (double)longest, 2.0 * itopk + 64.0) + kRankHalo;
    p->rank_places = want >= most ? most : ((int)want + group - 1) / group * group;
}

constexpr size_t kLdsBytes = 160 * 1024;  // of a compute unit; one workgroup may have all of it

// LDS words per query of a search by whole clusters: the table, or the gathering search that may follow.
int cluster_region_words(const ann_index_t* h, const Plan& plan) {
    const int table = cluster_table_at(plan.cap) + (int)((h->longest_cluster + 15) / 16 * 16);
    const int gather = (int)(plan.lds_bytes / sizeof(uint32_t));
    return ((table > gather ? table : gather) + 3) / 4 * 4;
}

// Whether a call searches by whole clusters (cluster_search.h), and in which workgroups.  Time in us of the gathering search,
// then of workgroups of one query (four or eight wavefronts) / four queries / eight; d bytes per row, clusters of m rows, a list
// of l, w parents a round:
//   * Few queries: one to a workgroup, whose wavefronts share the making of the keys.  Nothing is shared between queries, so no
//     execution order is needed either.  133 queries, d 96, m 1107, l 160, w 6: 78 | 42 / 65 / 66; 436, d 256, m 1107, l 112, w 1: 194 |
//     120 / 137 / 152; 1 581, d 96, m 991, l 64, w 1: 116 | 77 / 87 / 85; with a dozen queries per cluster sharing pays earlier:
//     1 009, d 144, m 1085, l 160, w 1: 260 | 150 / 142 / 150; 1 876, d 256, m 530: 209 | 141 / 121 / 119; 3 764, d 128, m 859: 83 | 77 / 55 / 52.
//     Eight wavefronts are better up to a few hundred queries (182, d 96, m 997: four 51, eight 48; 652, d 128, m 653: 40, 43).
//     The making of the keys has to be worth the rounds that get shorter: d 256, m 3707, l 32, w 2: 67 | 72; d 128, m 7674, l 64, w 8: 43 | 43,
//     against d 128, m 7542, l 100, w 4: 101 | 74 and d 128, m 7720, l 256, w 4: 145 | 96.  Workgroups have to be resident all at once (2 387,
//     d 128, m 7486: 197 | 392).
//     Every query streams its whole cluster, where one that gathers reads part of it: up to 100 MB, and 4 MB more per round, for the whole
//     call.  d 128, m 6103 (781 KB), 3.2 GB, l 184 and 100, w 4: 300 queries 155 | 122 and 106 | 99, 600 160 | 151 and 109 | 127, 1 000 165 | 193 and
//     113 | 170, on four streams at once 51 | 124 and 36 | 120; m 2000, 2.1 GB: 1 000 145 | 112 and 99 | 90, on four streams 40 | 44 and 29 | 41,
//     2 000 156 | 155 and 107 | 130, 56 | 85 and 56 | 80; m 6103 in the caches (31 MB), l 184: 600 129 | 89, on four streams 35 | 51, 1 000 132 | 107, 39 | 86.
//   * More queries: four or eight to a workgroup, grouped by cluster.  Eight make the keys for less, four wait less for the
//     slowest of them: 44 027, d 144, m 748, l 160, w 2: 1 221 | - / 812 / 884; 9 180, d 256, m 753, l 160, w 1: 448 | - / 273 / 334; 16 893, d 128,
//     m 931, l 64, w 2: 192 | - / 122 / 125; 40 653, d 128, m 1054, l 64, w 2: 506 | - / 315 / 306; 34 070, d 144, m 1877, l 112, w 4: 671 | - / 480 / 450;
//     28 938, d 96, m 1839, l 64, w 8: 353 | - / 352 / 326; but 2 298, d 256, m 1646, l 64, w 6: 107 | - / 62 / 83.
//     What decides against gathering is [clusters read per query, over the share of its cluster that a query is expected to score].  Of 3 185
//     calls over 60 indices (rows of 64 to 256 bytes, 100 to 6 000 a cluster, 1 MB to 2 GB) those below 0.76 took 0.6 to 0.85 of the gathering
//     search's time, those above up to 2.2 times: d 128, m 2000, 2.1 GB, l 184, w 4: 5 000 199 | 330 [1.57], 10 000 368 | 469 [1.30], 20 000 606 | 667 [0.98],
//     40 000 1 044 | 1 011 [0.71], 80 000 1 864 | 1 628 [0.36]; m 1000: 10 000 340 | 370 [1.22], 20 000 588 | 557 [1.01], 40 000 983 | 798 [0.76], 80 000 1 828 |
//     1 320 [0.55]; m 129, 75 000 clusters, 3 967: 243 | 362 [1.0].  Twelve wavefronts of a compute unit have to find room in LDS (7 382, d 128, m 4745,
//     eight: 307 | - / 429), and where no more do, the line is 0.45: d 128, l 256, w 4: 22 717, m 2972 831 | 1 072 [0.46], 18 332, m 2335 0.79 of the
//     time [0.37]; l 184: 38 412, m 2780 888 | 932 [0.49].  Rows of 64 edges take their time to read in either search, 0.66: m 1948 0.55 of
//     the time [0.57], m 2336 0.75 [0.65], m 2967 1.55 times [1.19].
//   * Where edges leave the clusters, some queries are searched anew.  Few queries all wait for one of them, large batches hide up to one
//     in a hundred: time with none | [share of the queries] and number expected, d 128, l 184, w 4: 1 000 queries, m 1000: 115 | 76 none, 90 [0.0006] 0.6,
//     150 [0.006] 6, 165 [0.6] 600; 100: 106 | 59 none, 75 [0.006] 0.6, 105 [0.018] 1.8, 130 [0.6] 60; 100 000, m 2000: 2 037 | 1 626 none, 1 740 [0.006],
//     1 858 [0.018], 2 178 [0.06], 3 520 [0.6]; 40 000, m 1000: 742 | 438 none, 509 [0.006], 521 [0.018], 576 [0.06], 861 [0.6]; 10 000, m 2000: 333 | 307 none,
//     375 [0.006].
void search_by_clusters(const ann_index_t* h, int64_t nq, int itopk, int width, int max_iters, Way* way) {
    if (!h->by_clusters || nq < 1 || nq > 2147483647ll) return;
    // options that ask for a search of another kind
    if (h->team != 0 || h->cluster_order_min < 0 || h->window_bits == 0 || h->hash_bits_bias != 0 ||
        h->variant != pick_variant(h->d.dtype, h->d.metric, h->row_bytes, 0))
        return;
    Plan plan;
    if (make_plan(h, itopk, width, &plan, "ann_search") != ANN_OK) return;
    const size_t head = sizeof(uint32_t) * kClusterHeaderWords, region = sizeof(uint32_t) * (size_t)cluster_region_words(h, plan);
    const size_t stages = sizeof(uint32_t) * (kMaxClusterGroup - 1) * kStageWords;
    const int64_t rounds = ((int64_t)width * max_iters < itopk ? max_iters : (itopk + width - 1) / width);
    // queries that will have to be searched anew, which costs both searches: an edge that leaves the cluster counts at any time, a key that is too
    // far until the list is full
    const int64_t parents = (int64_t)width * max_iters < itopk ? (int64_t)width * max_iters : itopk;
    const double anew = h->leaving * (double)(parents * h->d.degree) + h->far * (double)(itopk + width * h->d.degree);
    const double cluster_bytes = (double)(h->d.n / h->d.n_clusters) * h->row_bytes;
    // matrix instructions that the keys of up to sixteen queries take
    const int64_t products = (h->d.n / h->d.n_clusters + 15) / 16 * ((h->row_bytes + 63) / 64), per_cluster = nq / h->d.n_clusters;
    if (nq < 1000 || (nq < 3000 && per_cluster < 5)) {
        const size_t graph = ((size_t)h->longest_cluster * h->d.degree + 1) / 2 * sizeof(uint32_t), each = head + region + stages;
        if (products > 50 * rounds || each * (size_t)((nq + 255) / 256) > kLdsBytes || anew * (double)nq > 0.5) return;
        if ((double)nq * cluster_bytes > 1e6 * (100.0 + 4.0 * (double)rounds)) return;
        way->group = 1;
        way->waves = nq <= 384 ? kMaxClusterGroup : 4;
        // a small cluster's graph rows fit beside the table (100 queries, m 100, degree 32: 33.7 without, 31.1 with; 40 KB and more
        // take longer than they save)
        if (nq <= 256 && graph <= 16 * 1024 && each + graph <= kLdsBytes) way->graph_words = (int)(graph / sizeof(uint32_t));
        return;
    }
    if (anew > 1.0 / 128 || products > 45 * rounds * (per_cluster < 1 ? 1 : per_cluster < 4 ? per_cluster : 4)) return;
    const size_t fours = 4 * (kLdsBytes / (head + 4 * region)), eights = 8 * (kLdsBytes / (head + 8 * region));
    if (fours < 12) return;
    const int group = products > 4 * rounds && nq >= 4096 && per_cluster >= 8 && eights >= fours ? 8 : 4;
    // clusters that the workgroups read in all: each of those that have queries once, and one more wherever a workgroup begins
    const double met = h->d.n_clusters * (1.0 - std::exp(-(double)nq / h->d.n_clusters)), runs = met + (double)nq / group;
    double most = fours > 12 ? 0.8 : h->d.degree < 48 ? 0.45 : 0.66;
    if (anew * (double)nq > 0.5) most *= 0.6;  // the searches that some queries need afterwards
    if (runs > most * scored_share(h, parents, h->d.n / h->d.n_clusters) * (double)nq) return;
    way->group = way->waves = group;
}

// Entries drawn over the whole index: everything that a search scores is remembered in the hash, which has LDS to spare where registers
// or the batch bound the queries in flight (a compute unit holds 16 to 20 wavefronts over float rows, 28 over short uint8 rows).  Twice
// the ids that may come, so that it need not be emptied - rows are scored again after that - and insertions seldom meet.  With single words in place of buckets
// (hash_insert) and the smallest hash / now, us, 100, 1 000, 2 000, 4 000 queries, indices of 200 000 rows in clusters of 1 000 with a third of their edges anywhere:
// 400-byte fp16 rows, list of 100, 81 neighbours a round 349/245, 478/365, 593/469, 936/745; 1 536 bytes (100 000 rows), 128, 256 504/360, 1 219/823, 2 345/1 703, 4 642/4 642;
// 512-byte fp32 rows, 192, 192 445/354, 588/459, 945/745, 1 982/1 963; 128-byte uint8 rows, 64, 32 344/233, 439/374, 437/401, 492/408.  Single words in the
// larger hash were slower than in the small one here and there (384 bytes, 256, 256, 1 000 queries 616/663).
// Batches on other streams share the compute units: of short rows four find room.  us a batch with the small hash / with all of the LDS for one batch / now,
// one, four and eight streams: 128-byte uint8 rows, 128, 128: 1 000 queries 344/286/345, 94/144/90, 93/139/85, 2 000 367/313/351, 115/171/108, 107/167/101; 64, 32: 1 000
// 439/318/374, 125/171/98, 121/158/99; 96 bytes, 192, 256: 500 508/458/446, 148/187/139, 145/180/133, 1 000 514/466/494, 177/367/163, 171/354/157; 384 bytes, 128, 128: 4 000
// 970/862/959, 575/609/573, 607/619/605.  Of float rows fewer are in flight, and they may have all of it but where a thousand would take 40 KB each: 384 bytes, 64, 64
// 274/198/225, 106/115/86, 125/122/105; 256 bytes, 256, 256 575/495/518, 405/413/340, 397/405/336; 400 bytes, 100, 81 478/340/365, 198/169/147, 193/165/143.  Of longer rows
// all: 512 bytes, 192, 192, 1 000 588/459, 430/315, 415/299; 1 536 bytes, 128, 256 1 219/822, 1 133/729, 1 141/741; 768 bytes of uint8, 128, 128 520/424, 272/242, 267/231.
// Searches of few rounds visit few ids, and a large hash takes time to clear: three rounds, 100 queries of 384 bytes 15.6 us, with a hash for the
// whole list 17.2, 1 000 on four streams 12.0 and 18.1.
void enlarge_hash(const ann_index_t* h, int64_t nq, int itopk, int width, int max_iters, Plan* plan) {
    if (h->d.entry_mode != ANN_ENTRY_UNIFORM || h->hash_bits_bias != 0) return;
    const int64_t parents = (int64_t)width * max_iters < itopk ? (int64_t)width * max_iters : itopk;
    const int64_t visits = parents * h->d.degree + h->d.n_entry, resident = (nq + 255) / 256;
    size_t room = kLdsBytes / (size_t)resident;
    if (h->d.dtype == ANN_U8 && h->row_bytes < 512) room /= 4;
    else if (h->row_bytes < 512 && resident > 2 && room > 32 * 1024) room = 32 * 1024;
    const size_t least = h->d.dtype == ANN_U8 ? 5800 : 8192;
    if (room < least) room = least;
    while (plan->hash_bits < 13 && (int64_t(1) << plan->hash_bits) < 2 * visits) {
        const size_t more = sizeof(uint32_t) << plan->hash_bits;
        if (plan->lds_bytes + more > room) break;
        plan->lds_bytes += more;
        ++plan->hash_bits;
    }
}

// Checks the arguments of a search and launches it; `route` is null for uniform entries.
int search_impl(ann_index_t* h, const void* queries, int64_t nq, const int32_t* route, bool route_given, int k,
                int itopk, int width, int max_iters, int32_t* out_ids, void* out_dists, int32_t* out_counters,
                Workspace& ws, Way way) {
    hipStream_t stream = ws.stream;
    if (nq < 0) return fail(ANN_EINVAL, "ann_search: nq = %lld", (long long)nq);
    if (k < 1 || k > itopk) return fail(ANN_EINVAL, "ann_search: k = %d outside 1..itopk (%d)", k, itopk);
    if (max_iters < 0) return fail(ANN_EINVAL, "ann_search: max_iters = %d", max_iters);
    if (route_given && h->d.entry_mode != ANN_ENTRY_ROUTED)
        return fail(ANN_EINVAL, "ann_search_routed: the index does not use routed entries");
    Plan plan;
    const int rc = make_plan(h, itopk, width, &plan, "ann_search");
    if (rc != ANN_OK) return rc;
    if (nq == 0) return ANN_OK;
    enlarge_hash(h, nq, itopk, width, max_iters, &plan);
    if (!queries || !out_ids || !out_dists || (route_given && !route)) return fail(ANN_EINVAL, "ann_search: null argument");
    if (!aligned16(queries)) return fail(ANN_EINVAL, "ann_search: queries not 16-byte aligned");

    if (h->d.entry_mode == ANN_ENTRY_ROUTED && !route_given) {
        hipError_t e;
        int32_t* routes = static_cast<int32_t*>(ws.take(sizeof(int32_t) * (size_t)nq * h->d.route_c, &e));
        if (!routes) return fail(ANN_ENOMEM, "ann_search: no scratch memory for the routes: %s", hipGetErrorString(e));
        const int r = route_impl(h, queries, nq, routes, ws);
        if (r != ANN_OK) return r;
        route = routes;
    }
    // routed batches that are large enough run grouped by cluster, for cache reuse
    int32_t* order = nullptr;
    if (grouped_order(h, nq, way)) {
        hipError_t e;
        order = static_cast<int32_t*>(ws.take(sizeof(int32_t) * ((size_t)nq + h->d.n_clusters), &e));
        if (order) {
            e = launch_cluster_order(route, h->d.route_c, nq, h->d.n_clusters, order + nq, order, stream);
            if (e != hipSuccess) return fail(ANN_EHIP, "ann_search: launching the execution-order kernels failed: %s", hipGetErrorString(e));
        } else if (grouped_order(h, nq, Way())) {
            return fail(ANN_ENOMEM, "ann_search: no scratch memory for the execution order: %s", hipGetErrorString(e));
        } else {
            way = Way();  // which alone wanted the order: gather
        }
    }
    const int stride = way.table_stride;
    int64_t per_launch = kMaxQueriesPerLaunch;
    TableBlocks::Block* block = nullptr;
    if (stride > 0 && order) {
        // a query's keys, and its place in the list of those that the search by rank leaves
        int64_t most = (kTableBytes - 4) / (4 * ((int64_t)stride + 1));
        if (most > 512) most = most / 512 * 512;
        const int64_t launches = (nq + most - 1) / most, even = (nq + launches - 1) / launches;
        per_launch = (even + 511) / 512 * 512;
        if (per_launch > most) per_launch = most;
        if (per_launch > nq) per_launch = nq;
        block = h->tables.take(4 * ((size_t)stride + 1) * (size_t)per_launch + 4, stream);
        if (!block) per_launch = kMaxQueriesPerLaunch;  // no memory: gather every row
    }
    uint32_t* const table = block ? static_cast<uint32_t*>(block->memory) : nullptr;
    const int team = h->team ? h->team : default_team(h, nq, width);
    hipError_t e = hipSuccess;
    for (int64_t q0 = 0; q0 < nq && e == hipSuccess; q0 += per_launch) {
        const int64_t cnt = nq - q0 < per_launch ? nq - q0 : per_launch;
        SearchParams p;
        p.vectors = static_cast<const uint8_t*>(h->d.vectors);
        p.n = h->d.n;
        p.row_stride = h->d.row_stride_bytes;
        p.row_bytes = h->row_bytes;
        p.graph = h->d.graph;
        p.degree = h->d.degree;
        p.degree_inv = ((1u << 20) + (uint32_t)h->d.degree - 1) / (uint32_t)h->d.degree;
        p.queries = static_cast<const uint8_t*>(queries);
        p.nq = nq;
        p.q_base = q0;
        p.q_count = cnt;
        p.q_per_xcd = (cnt + 7) / 8;
        p.k = k;
        p.itopk = itopk;
        p.width = width;
        p.max_iters = max_iters;
        p.n_entry = h->d.n_entry;
        p.entry_mode = h->d.entry_mode;
        p.seed = h->d.seed;
        p.route = route;
        p.cluster_offsets = h->d.cluster_offsets;
        p.route_c = h->d.route_c;
        p.n_clusters = h->d.n_clusters;
        p.hash_bits = plan.hash_bits;
        p.window_bits = h->window_bits;
        p.cap = plan.cap;
        p.out_ids = out_ids;
        p.out_dists = static_cast<uint32_t*>(out_dists);
        p.out_counters = out_counters;
        p.order = order;
        p.table = table;
        p.table_stride = table ? stride : 0;
        p.rank_rows = p.rank_places = 0;
        p.again = nullptr;
        if (table) rank_rows(h, nq, itopk, width, max_iters, stride, &p);
        if (p.rank_rows > 0) p.again = reinterpret_cast<int32_t*>(table + (size_t)stride * (size_t)per_launch);
        size_t lds_bytes = plan.lds_bytes;
        if (way.group > 0) {
            ClusterParams c;
            c.group = way.group;
            c.per_lane = way.group <= 4 ? 1 : 2;
            c.cap = (int)h->longest_cluster;
            c.region_words = cluster_region_words(h, plan);
            c.graph_words = way.graph_words;
            p.q_per_xcd = ((cnt + way.group - 1) / way.group + 7) / 8;  // workgroups
            c.s = p;
            lds_bytes = sizeof(uint32_t) * ((size_t)kClusterHeaderWords + (size_t)way.group * c.region_words + (size_t)(way.waves - way.group) * kStageWords + way.graph_words);
            const unsigned grid = (unsigned)(8 * p.q_per_xcd), threads = (unsigned)(64 * way.waves);
            const bool l2 = h->d.metric == ANN_L2, small = h->row_bytes <= 128;
            e = l2 ? (small ? launch_cluster_search<kL2, 4, 2>(c, plan.list_variant, grid, threads, lds_bytes, stream)
                            : launch_cluster_search<kL2, 8, 2>(c, plan.list_variant, grid, threads, lds_bytes, stream))
                   : (small ? launch_cluster_search<kIP, 4, 2>(c, plan.list_variant, grid, threads, lds_bytes, stream)
                            : launch_cluster_search<kIP, 8, 2>(c, plan.list_variant, grid, threads, lds_bytes, stream));
            continue;
        }
        if (table) {
            KeyTableParams t;
            t.vectors = p.vectors;
            t.n = p.n;
            t.row_stride = p.row_stride;
            t.row_bytes = p.row_bytes;
            t.queries = p.queries;
            t.order = order;
            t.q_base = q0;
            t.q_count = cnt;
            t.route = route;
            t.cluster_offsets = p.cluster_offsets;
            t.n_clusters = p.n_clusters;
            t.stride = stride;
            // several workgroups for every place on the chip, of at least 128 rows each
            const int64_t mean = h->d.n / h->d.n_clusters + 1, set = key_table_set(h->variant->nch), sets = (cnt + set - 1) / set;
            const int64_t want = (4096 + sets - 1) / sets;
            t.slice_rows = (int)((mean + mean / 16 + want - 1) / want + 63) / 64 * 64;
            if (t.slice_rows < 128) t.slice_rows = 128;
            t.slices = (stride + t.slice_rows - 1) / t.slice_rows;
            t.table = table;
            t.none = p.again;
            e = launch_key_table(h->d.dtype, h->d.metric, h->variant->g, h->variant->nch, t, stream);
            if (e != hipSuccess) break;
            const int64_t longest = (h->longest_cluster + 127) / 128 * 128;
            if (longest < p.window_bits) {
                lds_bytes -= sizeof(uint32_t) * (size_t)(hash_at(p.window_bits) - hash_at((int)longest));
                p.window_bits = (int)longest;
            }
        }
        unsigned grid = (unsigned)(8 * p.q_per_xcd);
        if (p.again) {
            e = launch_rank_search(p, kListVariants[plan.list_variant][1], grid, (size_t)rank_lds_bytes(p.rank_rows, p.rank_places), stream);
            if (e != hipSuccess) break;
            // (2 048 workgroups, eight of the twelve to twenty-eight that a compute unit holds, where 0.15 and 0.35 of the queries were left:
            // 1 300 and 1 439 us instead of 1 148 and 1 202, 20 000 queries; without any 4 us in either case)
            const size_t resident = 256 * (kLdsBytes / lds_bytes < 20 ? kLdsBytes / lds_bytes : 20);
            if (grid > resident) grid = (unsigned)resident;
        }
        e = h->variant->search(p, plan.list_variant, team, grid, lds_bytes, stream);
    }
    if (block) h->tables.give_back(block, stream);
    if (e != hipSuccess) return fail(ANN_EHIP, "ann_search: launch failed: %s", hipGetErrorString(e));
    return ANN_OK;
}

Way choose_way(ann_index_t* h, int64_t nq, int itopk, int width, int max_iters, hipStream_t stream) {
    Way way;
    way.table_stride = table_stride(h, nq, itopk, width, max_iters, stream);
    if (way.table_stride == 0) search_by_clusters(h, nq, itopk, width, max_iters, &way);
    if (way.group > 1 && nq < h->cluster_order_min && !may_allocate_more(stream)) way = Way();  // no scratch for the order
    return way;
}

}  // namespace

extern "C" int ann_search_counters(ann_index_t* h, const void* queries, int64_t nq, int k, int itopk, int width,
                                   int max_iters, int32_t* out_ids, void* out_dists, int32_t* out_counters,
                                   void* stream) {
    if (!h || h->magic != kMagic) return fail(ANN_EINVAL, "ann_search: not a live handle");
    const Way way = choose_way(h, nq, itopk, width, max_iters, static_cast<hipStream_t>(stream));
    Workspace ws(static_cast<hipStream_t>(stream), search_scratch_bytes(h, nq, false, way, static_cast<hipStream_t>(stream)),
                 search_scratch_needed(h, nq, false));
    return search_impl(h, queries, nq, nullptr, false, k, itopk, width, max_iters, out_ids, out_dists, out_counters, ws, way);
}

extern "C" int ann_search_routed(ann_index_t* h, const void* queries, int64_t nq, const int32_t* routes, int k,
                                 int itopk, int width, int max_iters, int32_t* out_ids, void* out_dists,
                                 int32_t* out_counters, void* stream) {
    if (!h || h->magic != kMagic) return fail(ANN_EINVAL, "ann_search_routed: not a live handle");
    const Way way = choose_way(h, nq, itopk, width, max_iters, static_cast<hipStream_t>(stream));
    Workspace ws(static_cast<hipStream_t>(stream), search_scratch_bytes(h, nq, true, way, static_cast<hipStream_t>(stream)),
                 search_scratch_needed(h, nq, true));
    return search_impl(h, queries, nq, routes, true, k, itopk, width, max_iters, out_ids, out_dists, out_counters, ws, way);
}

extern "C" int ann_search(ann_index_t* h, const void* queries, int64_t nq, int k, int itopk, int width, int max_iters,
                          int32_t* out_ids, void* out_dists, void* stream) {
    return ann_search_counters(h, queries, nq, k, itopk, width, max_iters, out_ids, out_dists, nullptr, stream);
}

// ---------------------------------------------------------------------------------------------
// ann_search_static: the same search with its temporaries in a device array that is part of the
// library's code object, for callers that cannot allocate.
namespace {

constexpr size_t kStaticScratchBytes = (size_t)ANN_STATIC_SCRATCH_BYTES;
// Host code must not use this name as an address: it is a host-side stand-in.  The device address is
// asked for once per device (static_scratch_of_current_device) and that pointer is what kernels get.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_static_mutex;
void* g_static_ptr[kMaxDevices];  // per device: where that device holds its copy of `scratch`

int static_scratch_of_current_device(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(ANN_EHIP, "ann_search_static: hipGetDevice failed: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(ANN_EUNSUPPORTED, "ann_search_static: device %d outside 0..%d", dev, kMaxDevices - 1);
    std::lock_guard<std::mutex> lock(g_static_mutex);
    if (!g_static_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return fail(ANN_EHIP, "ann_search_static: hipGetSymbolAddress failed: %s", hipGetErrorString(e));
        g_static_ptr[dev] = ptr;
    }
    *out = g_static_ptr[dev];
    return ANN_OK;
}

}  // namespace

extern "C" int ann_search_static(ann_index_t* h, const void* queries, int64_t nq, int k, int itopk, int width, int max_iters,
                                 int32_t* out_ids, void* out_dists, void* stream) {
    if (!h || h->magic != kMagic) return fail(ANN_EINVAL, "ann_search_static: not a live handle");
    // routes and execution order have to fit; the routing cuts the centroids into as many slices as there is room for
    const bool routed = h->d.entry_mode == ANN_ENTRY_ROUTED && nq > 0;
    Way way;
    search_by_clusters(h, nq, itopk, width, max_iters, &way);
    auto bytes = [&] { return routed ? padded256(sizeof(int32_t) * (size_t)nq * h->d.route_c) + search_scratch_bytes(h, nq, true, way, static_cast<hipStream_t>(stream)) : 0; };
    if (bytes() > kStaticScratchBytes) way = Way();
    const size_t need = bytes();
    if (need > kStaticScratchBytes)
        return fail(ANN_EUNSUPPORTED,
                    "ann_search_static: %lld queries need %zu bytes of temporaries, the static scratch holds %zu; split the batch",
                    (long long)nq, need, kStaticScratchBytes);
    void* base = nullptr;
    if (need > 0) {
        const int rc = static_scratch_of_current_device(&base);
        if (rc != ANN_OK) return rc;
    }
    Workspace ws(static_cast<hipStream_t>(stream), base, need > 0 ? kStaticScratchBytes : 0);
    ws.routing_room = kStaticScratchBytes - need;
    return search_impl(h, queries, nq, nullptr, false, k, itopk, width, max_iters, out_ids, out_dists, nullptr, ws, way);
}

extern "C" int ann_gather_vectors(ann_index_t* h, const int32_t* ids, int64_t count, void* out_vectors, void* stream) {
    if (!h || h->magic != kMagic) return fail(ANN_EINVAL, "ann_gather_vectors: not a live handle");
    if (count < 0) return fail(ANN_EINVAL, "ann_gather_vectors: count = %lld", (long long)count);
    if (count == 0) return ANN_OK;
    if (!ids || !out_vectors) return fail(ANN_EINVAL, "ann_gather_vectors: null argument");
    if (!aligned16(out_vectors)) return fail(ANN_EINVAL, "ann_gather_vectors: out_vectors not 16-byte aligned");
    const hipError_t e = launch_gather_rows(static_cast<const uint8_t*>(h->d.vectors), h->d.n, h->d.row_stride_bytes,
                                            h->row_bytes, ids, count, static_cast<uint8_t*>(out_vectors),
                                            static_cast<hipStream_t>(stream));
    return e == hipSuccess ? ANN_OK : fail(ANN_EHIP, "ann_gather_vectors: launch failed: %s", hipGetErrorString(e));
}

extern "C" int ann_merge_topk(int key_dtype, const int32_t* ids, const void* keys, int64_t nq, int per_query, int k,
                              int32_t* out_ids, void* out_keys, void* stream) {
    if (key_dtype != ANN_U8 && key_dtype != ANN_F16 && key_dtype != ANN_F32)
        return fail(ANN_EINVAL, "ann_merge_topk: unknown key_dtype %d", key_dtype);
    if (nq < 0) return fail(ANN_EINVAL, "ann_merge_topk: nq = %lld", (long long)nq);
    if (per_query < 1 || per_query > kMaxItopk) return fail(ANN_EUNSUPPORTED, "ann_merge_topk: per_query = %d outside 1..%d", per_query, kMaxItopk);
    if (k < 1 || k > per_query) return fail(ANN_EINVAL, "ann_merge_topk: k = %d outside 1..per_query (%d)", k, per_query);
    if (nq == 0) return ANN_OK;
    if (!ids || !keys || !out_ids || !out_keys) return fail(ANN_EINVAL, "ann_merge_topk: null argument");
    for (int64_t q0 = 0; q0 < nq; q0 += kMaxQueriesPerLaunch) {
        const int64_t cnt = nq - q0 < kMaxQueriesPerLaunch ? nq - q0 : kMaxQueriesPerLaunch;
        const hipError_t e = launch_merge_topk(key_dtype != ANN_U8, ids + q0 * per_query,
                                               static_cast<const uint32_t*>(keys) + q0 * per_query, cnt, per_query, k,
                                               out_ids + q0 * k, static_cast<uint32_t*>(out_keys) + q0 * k,
                                               static_cast<hipStream_t>(stream));
        if (e != hipSuccess) return fail(ANN_EHIP, "ann_merge_topk: launch failed: %s", hipGetErrorString(e));
    }
    return ANN_OK;
}

namespace {

int check_graph_shape(const char* who, int64_t n, int d_in, int d_out) {
    if (n < 1 || n > 0x7fffffffLL) return fail(ANN_EINVAL, "%s: n = %lld outside 1..2^31-1", who, (long long)n);
    if (d_in < 1 || d_out < 1 || d_out > d_in) return fail(ANN_EINVAL, "%s: need 1 <= d_out <= d_in (got %d, %d)", who, d_out, d_in);
    if (d_in > kMaxKnnDegree || d_out > kMaxGraphDegree)
        return fail(ANN_EUNSUPPORTED, "%s: d_in = %d above %d or d_out = %d above %d", who, d_in, kMaxKnnDegree, d_out, kMaxGraphDegree);
    return ANN_OK;
}

}  // namespace

extern "C" int ann_graph_prune(const int32_t* knn, int64_t n, int d_in, int d_out, int32_t* pruned, void* stream) {
    if (const int rc = check_graph_shape("ann_graph_prune", n, d_in, d_out)) return rc;
    if (!knn || !pruned) return fail(ANN_EINVAL, "ann_graph_prune: null argument");
    const hipError_t e = launch_graph_prune(knn, n, d_in, d_out, pruned, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? ANN_OK : fail(ANN_EHIP, "ann_graph_prune: launch failed: %s", hipGetErrorString(e));
}

extern "C" int64_t ann_graph_optimize_workspace_bytes(int64_t n, int d_in, int d_out) {
    if (const int rc = check_graph_shape("ann_graph_optimize_workspace_bytes", n, d_in, d_out)) return rc;
    return graph_optimize_scratch_bytes(n, d_out);
}

extern "C" int ann_graph_optimize(const int32_t* knn, int64_t n, int d_in, int d_out, int32_t* out_graph, void* workspace,
                                  int64_t workspace_bytes, void* stream) {
    if (const int rc = check_graph_shape("ann_graph_optimize", n, d_in, d_out)) return rc;
    if (!knn || !out_graph || !workspace) return fail(ANN_EINVAL, "ann_graph_optimize: null argument");
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return fail(ANN_EINVAL, "ann_graph_optimize: workspace not 256-byte aligned");
    const int64_t need = ann_graph_optimize_workspace_bytes(n, d_in, d_out);
    if (workspace_bytes < need)
        return fail(ANN_EINVAL, "ann_graph_optimize: workspace of %lld bytes, %lld needed", (long long)workspace_bytes, (long long)need);
    const hipError_t e = launch_graph_optimize(knn, n, d_in, d_out, out_graph, workspace, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? ANN_OK : fail(ANN_EHIP, "ann_graph_optimize: launch failed: %s", hipGetErrorString(e));
}

namespace ann {
__global__ void __launch_bounds__(256) ann_calibration_copy_kernel(uint4* __restrict__ dst, const uint4* __restrict__ src,
                                                                   int64_t n16) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (int64_t)gridDim.x * 256) dst[i] = src[i];
}
}  // namespace ann

namespace ann {
// Piece p (16 bytes) is piece p % pieces of row p / pieces.  A workgroup takes 8 * 256 consecutive pieces at a
// time (256 whole rows of 128 bytes) and every thread has its eight loads in flight before it uses one.
__global__ void __launch_bounds__(256) ann_calibration_gather_kernel(const uint8_t* __restrict__ vectors, int64_t n,
                                                                     int64_t row_stride, int pieces, uint64_t pieces_inv,
                                                                     const int32_t* __restrict__ ids, int64_t count,
                                                                     uint32_t* sink) {
    __shared__ uint32_t part[256];
    const int64_t total = count * pieces;
    uint32_t acc = 0;
    // the ids of the next chunk are fetched while the rows of the current one are in flight
    // p / pieces as the high half of p * ceil(2^64 / pieces): exact for p < 2^41, pieces <= 128
    auto row_of = [&](int64_t p) -> int64_t { return pieces == 1 ? p : (int64_t)__umul64hi((uint64_t)p, pieces_inv); };
    auto id_of = [&](int64_t p) -> int32_t { return p < total ? ids[row_of(p)] : -1; };
    const int64_t step = (int64_t)gridDim.x * 2048;
    int64_t base = (int64_t)blockIdx.x * 2048;
    int32_t id[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) id[u] = id_of(base + u * 256 + threadIdx.x);
    for (; base < total; base += step) {
        typedef uint32_t word4 __attribute__((ext_vector_type(4)));
        word4 x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t p = base + u * 256 + threadIdx.x;
            x[u] = word4{0u, 0u, 0u, 0u};
            if (id[u] >= 0 && (int64_t)id[u] < n) {
                const int64_t r = row_of(p);
                // no row is read twice: non-temporal loads keep them from displacing each other in L2
                x[u] = __builtin_nontemporal_load(
                    reinterpret_cast<const word4*>(vectors + (int64_t)id[u] * row_stride + (p - r * pieces) * 16));
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) id[u] = id_of(base + step + u * 256 + threadIdx.x);
#pragma unroll
        for (int u = 0; u < 8; ++u) acc ^= x[u].x ^ x[u].y ^ x[u].z ^ x[u].w;
    }
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] ^= part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) atomicXor(sink, part[0]);
}
}  // namespace ann

extern "C" int ann_calibration_gather(ann_index_t* h, const int32_t* ids, int64_t count, uint32_t* sink, void* stream) {
    if (!h || h->magic != kMagic) return fail(ANN_EINVAL, "ann_calibration_gather: not a live handle");
    if (count < 0) return fail(ANN_EINVAL, "ann_calibration_gather: count = %lld", (long long)count);
    if (count == 0) return ANN_OK;
    if (!ids || !sink) return fail(ANN_EINVAL, "ann_calibration_gather: null argument");
    const int pieces = h->row_bytes / 16;  // at most 128 (2048-byte rows)
    if (count > (int64_t)1 << 33) return fail(ANN_EUNSUPPORTED, "ann_calibration_gather: count above 2^33");
    const uint64_t pieces_inv = pieces == 1 ? 0 : (~0ull) / (uint64_t)pieces + 1;  // ceil(2^64 / pieces)
    const int64_t want = (count * pieces + 2047) / 2048;  // eight pieces per thread
    const unsigned blocks = (unsigned)(want < 1 ? 1 : want > 2048 ? 2048 : want);  // 8 workgroups of 4 wavefronts per compute unit
    hipLaunchKernelGGL(ann::ann_calibration_gather_kernel, dim3(blocks), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<const uint8_t*>(h->d.vectors), h->d.n, h->d.row_stride_bytes, pieces, pieces_inv, ids, count,
                       sink);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? ANN_OK : fail(ANN_EHIP, "ann_calibration_gather: launch failed: %s", hipGetErrorString(e));
}

extern "C" int ann_calibration_copy(void* dst, const void* src, int64_t bytes, void* stream) {
    if (!dst || !src || bytes < 0 || bytes % 16 != 0 || !aligned16(dst) || !aligned16(src))
        return fail(ANN_EINVAL, "ann_calibration_copy: pointers must be non-null and 16-byte aligned, bytes a multiple of 16");
    if (bytes == 0) return ANN_OK;
    hipLaunchKernelGGL(ann::ann_calibration_copy_kernel, dim3(256 * 16), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<uint4*>(dst), static_cast<const uint4*>(src), bytes / 16);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? ANN_OK : fail(ANN_EHIP, "ann_calibration_copy: launch failed: %s", hipGetErrorString(e));
}
