// Key tables of float vectors (see key_table.h).
#include "key_table.h"
#include "row_variants.h"

namespace ann {

// The queries' pieces in registers, two rows per lane group in flight.  Bound by the vector ALU (0.93 of its issue slots
// for fp32 rows, 0.59 for fp16 products; the products of a key cost what they cost the search) and the three wavefronts per
// SIMD that 150 registers allow: 20 000 queries x 2 441 rows of 96 floats in 0.37 ms, 5 000 x 2 441 rows of 768 fp16 products
// in 0.37 ms.
// N: queries computed, the run's m of them real; without tests between them their chains of dependent products
// interleave.  FULL: see RowOps::load_full_row.
template <class Row, bool FULL, int N>
__device__ __forceinline__ void key_table_rows(const KeyTableParams& p, const KeyTableRuns<key_table_set(Row::NCH)>& run, const Row& row,
                                               const u32x4 (&q)[key_table_set(Row::NCH)][Row::NCH], int lane, int wave) {
    constexpr int G = Row::G, NCH = Row::NCH, RPS = 64 / G;
    const uint8_t* const piece0 = row.lane_piece(p.vectors);
    const uint32_t stride = (uint32_t)p.row_stride;
    u32x4 x[2][NCH];
    auto load = [&](int u, int j) {
        // a row beyond the last is the last one again; an id that is no row (offsets beyond n) reads row 0
        const uint64_t id = (uint64_t)(run.lo + (j < run.r1 ? j : run.r1 - 1));
        const uint8_t* const piece = piece0 + (uint64_t)(id < (uint64_t)p.n ? (uint32_t)id : 0u) * stride;
        if constexpr (FULL) row.load_full_row(x[u], piece, true);
        else row.load_row(x[u], piece, true);
    };
    uint32_t* const out = p.table + (run.pos + (row.lg & (N - 1))) * p.stride;
    const bool mine = row.lg < run.m;  // lanes N .. G-1 of a group hold copies
    int j = run.r0 + wave * (2 * RPS) + lane / G;
    load(0, j);
    load(1, j + RPS);
    for (int base = run.r0 + wave * (2 * RPS); base < run.r1; base += 8 * RPS, j += 8 * RPS) {
        float v[2][N];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int t = 0; t < N; ++t) v[u][t] = 0.0f;
            // RowOps::partial of N queries side by side
#pragma unroll
            for (int c = 0; c < NCH; ++c)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int t = 0; t < N; ++t) v[u][t] = Row::step(v[u][t], q[t][c][i], x[u][c][i]);
            // the sums are wanted here: moved down to their use, past the loads, they would keep every difference of
            // an L2 key in a register
#pragma unroll
            for (int t = 0; t < N; ++t) asm volatile("" : "+v"(v[u][t]));
            load(u, j + u * RPS + 8 * RPS);
        }
        const uint32_t k0 = Row::ordered(group_sums<G>(v[0], lane)), k1 = Row::ordered(group_sums<G>(v[1], lane));
        if (mine && j < run.r1) out[j] = k0;
        if (mine && j + RPS < run.r1) out[j + RPS] = k1;
    }
}

template <class Row>
__global__ void __launch_bounds__(256) key_table_kernel(const KeyTableParams p) {
    constexpr int NCH = Row::NCH, Q = key_table_set(Row::NCH);
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (p.none && blockIdx.x == 0 && threadIdx.x == 0) *p.none = 0;
    KeyTableRuns<Q> run;
    run.begin(p, lane);
    while (run.next(p, lane)) {
        Row row;
        u32x4 q[Q][NCH];
#pragma unroll
        for (int t = 0; t < Q; ++t) {
            // beyond the last: the last query again; its keys are not stored
            const int64_t qi = __builtin_amdgcn_readlane(run.query, t < run.m ? t : run.m - 1);
            row.load_query(p.queries + qi * p.row_bytes, p.row_bytes, lane);
#pragma unroll
            for (int i = 0; i < NCH; ++i) q[t][i] = row.q[i];
        }
        if (row.full) {
            if (run.m > Q / 2) key_table_rows<Row, true, Q>(p, run, row, q, lane, wave);
            else key_table_rows<Row, true, Q / 2>(p, run, row, q, lane, wave);
        } else {
            if (run.m > Q / 2) key_table_rows<Row, false, Q>(p, run, row, q, lane, wave);
            else key_table_rows<Row, false, Q / 2>(p, run, row, q, lane, wave);
        }
    }
}

hipError_t launch_key_table(int dtype, int metric, int g, int nch, const KeyTableParams& p, hipStream_t stream) {
#define ANN_TABLE(DT, METRIC, G, NCH)                                                                                   \
    if constexpr (DT != kU8)                                                                                            \
        if (dtype == DT && metric == METRIC && g == G && nch == NCH) {                                                  \
            hipLaunchKernelGGL((key_table_kernel<RowOps<DT, METRIC, G, NCH>>), dim3(key_table_grid<key_table_set(NCH)>(p)), \
                               dim3(256), 0, stream, p);                                                                \
            return hipGetLastError();                                                                                   \
        }
    ANN_ROW_VARIANTS(ANN_TABLE)
#undef ANN_TABLE
    return hipErrorInvalidValue;
}

}  // namespace ann
