/* Which kernels libann launches, and on what memory, without a GPU: the HIP functions that it calls are defined here (the program's
 * symbols come before those of the HIP runtime).  Kernels do not run; their names are noted.  Device memory is host memory whose
 * ranges are remembered.  argv[1] names the scenario. */
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

#include "ann.h"

/* ---- the runtime ---- */
#define MAX 4096
static struct { const void* host; const char* name; } kernels[MAX];
static int n_kernels;
static struct { char* at; size_t bytes; } ranges[MAX];
static int n_ranges;
static size_t async_limit = (size_t)1 << 40; /* hipMallocAsync refuses more */
static char launched[1 << 16];
static int host_reads; /* copies from memory that is no device memory */
static struct { dim3 grid, block; size_t lds; hipStream_t stream; } config;
static uint32_t sample_result[3]; /* what the kernel that looks at a sample of an index finds: edges that leave, keys too far, rows with many copies */
static unsigned threads; /* of the last launch's workgroups */
static unsigned blocks;  /* how many */
static size_t most_async; /* largest hipMallocAsync */
static size_t lds_used;  /* by the last launch's workgroups */
static int sampled, default_stream_free = 1;

static int find(const void* p) {
    for (int i = 0; i < n_ranges; ++i)
        if ((const char*)p >= ranges[i].at && (const char*)p < ranges[i].at + ranges[i].bytes) return i;
    return -1;
}
static void* device(size_t bytes) { /* zeros; large ones take no memory until they are touched */
    void* p = mmap(NULL, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (p == MAP_FAILED) exit(3);
    ranges[n_ranges].at = p;
    ranges[n_ranges++].bytes = bytes;
    return p;
}
static void release(void* p) {
    const int i = find(p);
    if (i < 0) return;
    munmap(ranges[i].at, ranges[i].bytes);
    ranges[i] = ranges[--n_ranges];
}

void** __hipRegisterFatBinary(const void* d) { (void)d; static void* m; return &m; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned limit, void* t, void* b, dim3* bd, dim3* gd, int* w) {
    (void)m, (void)dev, (void)limit, (void)t, (void)b, (void)bd, (void)gd, (void)w;
    kernels[n_kernels].host = host;
    kernels[n_kernels++].name = name;
}
void __hipRegisterVar(void** m, void* var, char* h, char* d, int ext, size_t size, int c, int g) {
    (void)m, (void)var, (void)h, (void)d, (void)ext, (void)size, (void)c, (void)g;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
    config.grid = grid, config.block = block, config.lds = lds, config.stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
    *grid = config.grid, *block = config.block, *lds = config.lds, *s = config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t s) {
    (void)s;
    threads = block.x, blocks = grid.x, lds_used = lds;
    for (int i = 0; i < n_kernels; ++i) {
        if (kernels[i].host != f) continue;
        strcat(launched, kernels[i].name);
        strcat(launched, " ");
        if (strstr(kernels[i].name, "longest_cluster_kernel")) {
            const int64_t* off = *(const int64_t**)args[0];
            uint64_t longest = 0, in_long = 0;
            for (int c = 0; c < *(int*)args[1]; ++c) {
                if ((uint64_t)(off[c + 1] - off[c]) > longest) longest = off[c + 1] - off[c];
                if (off[c + 1] - off[c] > *(int64_t*)args[3]) in_long += off[c + 1] - off[c];
            }
            memcpy(*(char**)args[2], &longest, sizeof(longest));
            memcpy(*(char**)args[2] + 24, &in_long, sizeof(in_long));
        }
        if (strstr(kernels[i].name, "sample_clusters_kernel")) {
            sampled = 1;
            char* sample = *(char**)args[4]; /* rows of the longest cluster (8 bytes), then the counts */
            memcpy(sample + 8, sample_result, sizeof(sample_result));
        }
    }
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t bytes) { *p = device(bytes); return hipSuccess; }
hipError_t hipFree(void* p) { release(p); return hipSuccess; }
hipError_t hipMallocAsync(void** p, size_t bytes, hipStream_t s) {
    (void)s;
    *p = NULL;
    if (bytes > async_limit) return hipErrorOutOfMemory;
    if (bytes > most_async) most_async = bytes;
    *p = device(bytes);
    return hipSuccess;
}
hipError_t hipFreeAsync(void* p, hipStream_t s) { (void)s; release(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t bytes, hipMemcpyKind k) {
    if (k == hipMemcpyDeviceToHost && find(s) < 0) {
        ++host_reads;
        return hipErrorInvalidValue;
    }
    memcpy(d, s, bytes);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
    memset(a, 0, sizeof(*a));
    a->type = find(p) >= 0 ? hipMemoryTypeDevice : hipMemoryTypeUnregistered;
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
    const int i = find(p);
    if (i < 0) return hipErrorInvalidValue;
    *base = ranges[i].at, *size = ranges[i].bytes;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* c) {
    *c = hipStreamCaptureStatusNone;
    return s || default_stream_free ? hipSuccess : hipErrorStreamCaptureImplicit;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) { (void)m; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { (void)s; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t e) { (void)e; return "an error"; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { (void)s; static void* at; if (!at) at = device(ANN_STATIC_SCRATCH_BYTES); *p = at; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned f) { (void)f; *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { (void)e, (void)s; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned f) { (void)s, (void)e, (void)f; return hipSuccess; }

/* ---- scenarios ---- */
#define CHECK(x) do { if (!(x)) { printf("line %d: %s (%s) after: %s\n", __LINE__, #x, ann_last_error(), launched); exit(1); } } while (0)
static int ran(const char* name) { return strstr(launched, name) != NULL; }

/* An index of n_clusters clusters of `mean` rows over device memory. */
static ann_index_desc_t index_of(int dtype, int dim, int mean, int n_clusters, int degree, int route_c) {
    const int size = dtype == ANN_U8 ? 1 : dtype == ANN_F16 ? 2 : 4;
    ann_index_desc_t d;
    memset(&d, 0, sizeof(d));
    d.n = (int64_t)mean * n_clusters;
    d.dim = dim, d.dtype = dtype, d.row_stride_bytes = (int64_t)dim * size, d.metric = ANN_L2;
    d.vectors = device((size_t)d.n * d.row_stride_bytes);
    d.graph = device((size_t)d.n * degree * 4);
    d.degree = degree, d.n_entry = 32, d.entry_mode = ANN_ENTRY_ROUTED, d.seed = 1;
    d.centroids = device((size_t)n_clusters * dim * size);
    int64_t* off = device(((size_t)n_clusters + 1) * 8);
    for (int c = 0; c <= n_clusters; ++c) off[c] = (int64_t)c * mean;
    d.cluster_offsets = off, d.n_clusters = n_clusters, d.route_c = route_c;
    return d;
}
static ann_index_t* load(const ann_index_desc_t* d) {
    ann_index_t* h = NULL;
    CHECK(ann_index_load(d, &h) == ANN_OK && h);
    return h;
}

/* What a way of searching or routing wants of scratch memory, and the call can do without, is no reason to refuse the call. */
static void scratch(void) {
    ann_index_desc_t d = index_of(ANN_U8, 128, 500, 100, 32, 1);
    ann_index_t* h = load(&d);
    const int nq = 2000;
    void* q = device(nq * 128);
    int32_t *routes = device(nq * 4), *ids = device(nq * 40), *keys = device(nq * 40);
    launched[0] = 0;
    CHECK(ann_search_routed(h, q, nq, routes, 10, 184, 4, 100, ids, keys, NULL, NULL) == ANN_OK && ran("cluster_search_kernel") && ran("cluster_order_kernel"));
    async_limit = 0;
    launched[0] = 0;
    CHECK(ann_search_routed(h, q, nq, routes, 10, 184, 4, 100, ids, keys, NULL, NULL) == ANN_OK && ran("beam_search_kernel") && !ran("cluster_"));
    CHECK(ann_route(h, q, nq, routes, NULL) == ANN_OK);
    CHECK(ann_search(h, q, nq, 10, 184, 4, 100, ids, keys, NULL) == ANN_ENOMEM); /* no room for the routes */
    async_limit = nq * 4 + 255;                                                 /* room for the routes */
    launched[0] = 0;
    CHECK(ann_search(h, q, nq, 10, 184, 4, 100, ids, keys, NULL) == ANN_OK && ran("beam_search_kernel") && !ran("cluster_"));
    ann_free(h);
    /* rows of an odd multiple of 16 bytes: slices (uint8) and lists (float) */
    const int types[3] = {ANN_U8, ANN_F16, ANN_F32}, dims[3] = {144, 200, 100};
    for (int t = 0; t < 3; ++t) {
        d = index_of(types[t], dims[t], 50, 2000, 16, 2);
        h = load(&d);
        void* x = device((size_t)nq * 400);
        for (int room = 0; room < 2; ++room) {
            async_limit = room ? nq * 8 + 255 : 0;
            CHECK(ann_route(h, x, nq, routes = device(nq * 8), NULL) == ANN_OK);
            CHECK(ann_search(h, x, nq, 10, 64, 2, 100, ids, keys, NULL) == (room ? ANN_OK : ANN_ENOMEM));
        }
        ann_free(h);
    }
}

/* A handle of routed uint8 rows is loaded over arrays that are not, or not whole, in device memory; nothing of them is read. */
static void stand_ins(void) {
    const int dims[2] = {128, 144};
    for (int t = 0; t < 2; ++t) {
        for (int which = 0; which < 6; ++which) {
            ann_index_desc_t d = index_of(ANN_U8, dims[t], 500, 100, 32, 1);
            if (which == 0) d.vectors = aligned_alloc(256, 1 << 20);
            if (which == 1) d.graph = aligned_alloc(256, 1 << 20);
            if (which == 2) d.cluster_offsets = aligned_alloc(256, 1 << 20);
            if (which == 3) d.vectors = device((size_t)d.n * dims[t] - 256);
            if (which == 4) d.graph = device((size_t)d.n * 32 * 4 - 256);
            if (which == 5) default_stream_free = 0; /* another stream is being captured */
            sampled = host_reads = 0;
            ann_index_t* h = load(&d);
            CHECK(!sampled && !host_reads);
            default_stream_free = 1;
            ann_free(h);
        }
        ann_index_desc_t d = index_of(ANN_U8, dims[t], 500, 100, 32, 1);
        sampled = 0;
        ann_free(load(&d));
        CHECK(sampled);
    }
    ann_index_desc_t d = index_of(ANN_F32, 100, 500, 100, 32, 1);
    default_stream_free = 0;
    launched[0] = 0;
    ann_free(load(&d));
    CHECK(!launched[0]);
}

/* A search by whole clusters is for indices whose queries will end in it: not one in a small batch, few in a large one. */
static void searched_anew(void) {
    const struct { int nq; uint32_t leaving, far; int whole; } calls[] = {
        /* 16 777 216 edges, 184 * 32 of them a query; 65 536 keys, 184 + 128 of them before the list is full */
        {100, 0, 0, 1}, {100, 1, 0, 1}, {100, 40, 0, 0}, {100, 0, 1, 1}, {100, 0, 2, 0}, {900, 0, 0, 1}, {900, 1, 0, 1}, {900, 4, 0, 0}, {900, 0, 1, 0},
        {40000, 0, 0, 1}, {40000, 20, 0, 1}, {40000, 25, 0, 0}, {40000, 0, 1, 1}, {40000, 0, 2, 0}, {40000, 31250, 0, 0}};
    ann_index_desc_t d = index_of(ANN_U8, 128, 1000, 1000, 32, 1);
    void* q = device(40000 * 128);
    int32_t *routes = device(40000 * 4), *ids = device(40000 * 40), *keys = device(40000 * 40);
    for (unsigned i = 0; i < sizeof(calls) / sizeof(calls[0]); ++i) {
        sample_result[0] = calls[i].leaving, sample_result[1] = calls[i].far, sample_result[2] = 0;
        ann_index_t* h = load(&d);
        launched[0] = 0;
        CHECK(ann_search_routed(h, q, calls[i].nq, routes, 10, 184, 4, 200, ids, keys, NULL, NULL) == ANN_OK);
        if (ran("cluster_search_kernel") != calls[i].whole) printf("call %u\n", i);
        CHECK(ran("cluster_search_kernel") == calls[i].whole);
        ann_free(h);
    }
}

/* Whole clusters are read where that costs no more than the rows that a query would gather. */
static void bytes_read(void) {
    const struct { int dim, mean, clusters, degree, nq, itopk, width, group; } calls[] = {
        {128, 6103, 16384, 32, 1000, 184, 4, 0}, {128, 6103, 16384, 32, 100, 184, 4, 1}, {128, 6103, 40, 32, 999, 184, 4, 0}, {128, 100, 100, 32, 100, 64, 1, 1},
        {128, 1000, 1000, 32, 1000, 184, 4, 1}, {128, 2000, 8192, 32, 2000, 184, 4, 0}, {256, 2500, 2048, 32, 2000, 100, 4, 0},
        {128, 2000, 8192, 32, 5000, 184, 4, 0}, {128, 2000, 8192, 32, 20000, 184, 4, 0}, {128, 2000, 8192, 32, 500000, 184, 4, 8},
        {128, 1000, 16384, 32, 10000, 100, 4, 0}, {128, 1000, 16384, 32, 100000, 184, 4, 4}, {128, 1000, 1000, 32, 10000, 128, 4, 4}, {96, 2500, 8192, 32, 80000, 64, 1, 0},
        {128, 1000, 1000, 32, 4000, 184, 4, 4}, {96, 129, 74596, 64, 3967, 128, 2, 0}, {128, 2972, 736, 32, 22717, 256, 4, 0}, {128, 2300, 60, 64, 9000, 256, 4, 4}};
    int32_t *routes = device(500000 * 4), *ids = device(500000 * 4), *keys = device(500000 * 4);
    void* q = device((size_t)500000 * 256);
    for (unsigned i = 0; i < sizeof(calls) / sizeof(calls[0]); ++i) {
        ann_index_desc_t d = index_of(ANN_U8, calls[i].dim, calls[i].mean, calls[i].clusters, calls[i].degree, 1);
        ann_index_t* h = load(&d);
        launched[0] = 0;
        CHECK(ann_search_routed(h, q, calls[i].nq, routes, 1, calls[i].itopk, calls[i].width, 200, ids, keys, NULL, NULL) == ANN_OK);
        const int whole = ran("cluster_search_kernel"), group = !whole ? 0 : !ran("cluster_order_kernel") && !ran("cluster_scatter_kernel") ? 1 : (int)threads / 64;
        if (group != calls[i].group) printf("call %u: %d\n", i, group);
        CHECK(group == calls[i].group);
        ann_free(h);
        release((void*)d.vectors), release((void*)d.graph);
    }
}

/* Rows are ranked where few queries will have to be searched otherwise: of a small batch none. */
static void ranked(void) {
    const struct { int nq; uint32_t leaving; int long_clusters, window_bits, width, ranks; uint32_t copied; } calls[] = {
        /* 16 777 216 edges, 256 * 64 of them a query */
        {8000, 0, 0, 0, 4, 1}, {8000, 1, 0, 0, 4, 0}, {20000, 0, 0, 0, 4, 1}, {20000, 8, 0, 0, 4, 1}, {20000, 9, 0, 0, 4, 0},
        {20000, 1u << 24, 0, 0, 4, 0},
        /* clusters of 3 300 rows among 400 of 2 000 */
        {8000, 0, 1, 0, 4, 0}, {19999, 0, 1, 0, 4, 0}, {20000, 0, 1, 0, 4, 1}, {20000, 0, 40, 0, 4, 1}, {20000, 0, 60, 0, 4, 0}, {20000, 9, 1, 0, 4, 0},
        /* a visited bitmap that cuts the rows of the table: the longest cluster fits, does so in rows that are not whole 64s, does not fit */
        {8000, 0, 0, 2048, 4, 1}, {8000, 0, 0, 2016, 4, 0}, {8000, 0, 0, 1024, 4, 0}, {20000, 0, 1, 3200, 4, 1}, {20000, 0, 1, 3008, 4, 0},
        /* 128 rows, of some of which there are copies */
        {8000, 0, 0, 0, 4, 1, 64}, {8000, 0, 0, 0, 4, 0, 65}, {20000, 0, 0, 0, 4, 0, 128},
        /* rounds of few neighbours */
        {20000, 0, 0, 0, 1, 1}, {20000, 0, 0, 0, 8, 1}};
    void* q = device((size_t)20000 * 384);
    int32_t *routes = device(20000 * 4), *ids = device(20000 * 40), *keys = device(20000 * 40);
    ann_index_desc_t d = index_of(ANN_F32, 96, 2000, 400, 64, 1);
    for (unsigned i = 0; i < sizeof(calls) / sizeof(calls[0]); ++i) {
        int64_t* off = (int64_t*)d.cluster_offsets;
        for (int c = 0; c < 400; ++c) off[c + 1] = off[c] + (c < calls[i].long_clusters ? 3300 : c < 2 * calls[i].long_clusters ? 700 : 2000);
        sample_result[0] = calls[i].leaving, sample_result[1] = 0, sample_result[2] = calls[i].copied;
        ann_index_t* h = load(&d);
        if (calls[i].window_bits) CHECK(ann_index_set_option(h, ANN_OPT_VISITED_WINDOW_BITS, calls[i].window_bits) == ANN_OK);
        launched[0] = 0, most_async = 0;
        CHECK(ann_search_routed(h, q, calls[i].nq, routes, 10, 256, calls[i].width, 200, ids, keys, NULL, NULL) == ANN_OK);
        if (ran("rank_search_kernel") != calls[i].ranks) printf("call %u\n", i);
        CHECK(ran("key_table_kernel") && ran("rank_search_kernel") == calls[i].ranks && ran("left_over_search_kernel") == calls[i].ranks);
        const size_t stride = calls[i].window_bits && calls[i].window_bits < 3072 ? (size_t)calls[i].window_bits : 3072;
        CHECK(most_async >= 4 * (stride + 1) * (size_t)calls[i].nq + 4); /* keys, and the list of those that are left */
        if (calls[i].ranks) CHECK(blocks >= 256 * 12 && blocks <= 256 * 28); /* as many as a chip holds */
        ann_free(h);
    }
}

/* With entries drawn over the whole index the visited hash has room for twice what a search will visit. */
static void hash(void) {
    const struct { int dtype, dim, nq, itopk, width, rounds; size_t more; } calls[] = {
        /* bytes of LDS beyond those of the smallest hash, 512 and 256 words */
        {ANN_F16, 200, 100, 100, 3, 200, 4 * (8192 - 512)}, {ANN_F16, 200, 100, 100, 3, 10, 4 * (2048 - 512)},
        {ANN_F16, 200, 100, 100, 3, 3, 4 * (1024 - 512)}, {ANN_F16, 200, 100, 100, 3, 0, 0},
        {ANN_U8, 128, 100, 64, 1, 200, 4 * (8192 - 256)}, {ANN_U8, 128, 100, 64, 1, 16, 4 * (2048 - 256)}, {ANN_U8, 128, 100, 64, 1, 2, 0},
        /* a thousand queries: what leaves room for other batches */
        {ANN_U8, 128, 1000, 64, 1, 200, 4 * (2048 - 256)}, {ANN_F16, 200, 1000, 100, 3, 200, 4 * (4096 - 512)}, {ANN_F16, 256, 1000, 100, 3, 200, 4 * (8192 - 512)}};
    void* q = device((size_t)1000 * 512);
    int32_t *ids = device(1000 * 40), *keys = device(1000 * 40);
    for (unsigned i = 0; i < sizeof(calls) / sizeof(calls[0]); ++i) {
        ann_index_desc_t d = index_of(calls[i].dtype, calls[i].dim, 1000, 100, calls[i].dtype == ANN_U8 ? 32 : 27, 1);
        d.entry_mode = ANN_ENTRY_UNIFORM;
        ann_index_t* h = load(&d);
        CHECK(ann_search(h, q, calls[i].nq, 10, calls[i].itopk, calls[i].width, calls[i].rounds, ids, keys, NULL) == ANN_OK);
        const size_t more = lds_used - (size_t)ann_lds_bytes(h, calls[i].itopk, calls[i].width);
        if (more != calls[i].more) printf("call %u: %zu\n", i, more);
        CHECK(more == calls[i].more);
        ann_free(h);
    }
}

int main(int argc, char** argv) {
    const char* what = argc > 1 ? argv[1] : "";
    if (!strcmp(what, "scratch")) scratch();
    else if (!strcmp(what, "stand_ins")) stand_ins();
    else if (!strcmp(what, "searched_anew")) searched_anew();
    else if (!strcmp(what, "bytes_read")) bytes_read();
    else if (!strcmp(what, "ranked")) ranked();
    else if (!strcmp(what, "hash")) hash();
    else return 2;
    printf("%s ok\n", what);
    return 0;
}
