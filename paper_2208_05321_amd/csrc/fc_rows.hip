// Row movement: one row-group of lanes per embedding row, 16-byte accesses where dim allows.
// Used for the evict gather, the host-table store of evicted rows, the miss fill and the flush
// (paper Section 4.3, "data transmitter": rows scattered in one memory become a block in the other).
#include "rows_device.h"

#include <algorithm>

namespace fc {

// dst[dst_idx ? dst_idx[j] : j] = src[src_idx ? src_idx[j] : j] for j in [0, rows); row length D floats.
// lpr (power of two, <= 64) consecutive lanes own one row; a lane moves VEC floats per access.
// KIND only names the instantiation (profilers then tell the three uses apart): 0 evicted-row gather (HBM -> HBM
// block), 1 evicted-row store (block -> host table), 2 miss fill (host table -> cache slots, or block -> slots).
template <int VEC, int KIND>
__global__ __launch_bounds__(256) void k_copy_rows(float* __restrict__ dst, const int32_t* __restrict__ dst_idx,
                                                   unsigned dst_rows, const float* __restrict__ src,
                                                   const int32_t* __restrict__ src_idx, unsigned src_rows, int rows,
                                                   int D, int lpr_shift, int32_t* __restrict__ tag_out,
                                                   const int32_t* __restrict__ tags, float* __restrict__ twin, int32_t* __restrict__ tag_twin) {
    using V = typename Vec<VEC>::T;
    const int lpr = 1 << lpr_shift;
    const int gpb = blockDim.x >> lpr_shift;
    const int gl = threadIdx.x >> lpr_shift, lane = threadIdx.x & (lpr - 1);
    const int nv = D / VEC;
    for (int j = blockIdx.x * gpb + gl; j < rows; j += gridDim.x * gpb) {
        const int di = dst_idx ? dst_idx[j] : j;
        const int si = src_idx ? src_idx[j] : j;
        if (KIND == 0 && tag_out && lane == 0) {
            const int32_t tag = tags[j];
            tag_out[j] = tag;
            if (tag_twin) tag_twin[j] = tag;
        }
        if ((unsigned)di >= dst_rows || (unsigned)si >= src_rows) continue;   // never true for lists this library builds
        const V* __restrict__ s = reinterpret_cast<const V*>(src + (size_t)si * D);
        V* __restrict__ d = reinterpret_cast<V*>(dst + (size_t)di * D);
        // the evicted rows and the rows of an arrival block are read for the last time here: non-temporal loads keep them
        // from displacing the cached rows in the memory-side cache
        for (int cidx = lane; cidx < nv; cidx += lpr) {
            const V v = KIND == 1 ? s[cidx] : nt_load_row(&s[cidx]);
            d[cidx] = v;
            if (KIND == 0 && twin) reinterpret_cast<V*>(twin + (size_t)j * D)[cidx] = v;
        }
    }
}

template <int VEC>
__global__ __launch_bounds__(256) void k_swap_rows(RowArgs a) { swap_rows<VEC>(a, blockIdx.x, gridDim.x); }

// Flush: every resident slot's row (with a dirty array: every dirty one) goes to its place in the host table.
template <int VEC>
__global__ __launch_bounds__(256) void k_flush_rows(float* __restrict__ host, const float* __restrict__ cache,
                                                    const int32_t* __restrict__ slot_rank, int C, int D, int lpr_shift,
                                                    const uint8_t* __restrict__ dirty) {
    using V = typename Vec<VEC>::T;
    const int lpr = 1 << lpr_shift;
    const int gpb = blockDim.x >> lpr_shift;
    const int gl = threadIdx.x >> lpr_shift, lane = threadIdx.x & (lpr - 1);
    const int nv = D / VEC;
    for (int s = blockIdx.x * gpb + gl; s < C; s += gridDim.x * gpb) {
        const int r = slot_rank[s];
        if (r < 0) continue;
        if (dirty && !dirty[s]) continue;
        const V* __restrict__ src = reinterpret_cast<const V*>(cache + (size_t)s * D);
        V* __restrict__ d = reinterpret_cast<V*>(host + (size_t)r * D);
        for (int cidx = lane; cidx < nv; cidx += lpr) d[cidx] = src[cidx];
    }
}

template <int VEC>
__global__ __launch_bounds__(256) void k_fill_rows(RowArgs a) { fill_rows<VEC>(a, blockIdx.x, gridDim.x); }

int launch_copy_rows(fc_cache* c, hipStream_t s, int prof_item, float* dst, const int32_t* dst_idx, int64_t dst_rows,
                     const float* src, const int32_t* src_idx, int64_t src_rows, int64_t rows, int max_blocks, int32_t* tag_out,
                     const int32_t* tags, float* twin, int32_t* tag_twin) {
    if (rows <= 0) return FC_OK;
    const int sh = shift_of(c->lpr);
    const int gpb = 256 >> sh;
    int64_t blocks = cdiv(rows, gpb);
    if (blocks > max_blocks) blocks = max_blocks;
    ProfScope ps(c, prof_item, s);
#define FC_LAUNCH_ROWS(V, K) \
    k_copy_rows<V, K><<<(unsigned)blocks, 256, 0, s>>>(dst, dst_idx, (unsigned)dst_rows, src, src_idx, (unsigned)src_rows, (int)rows, c->D, sh, tag_out, tags, twin, tag_twin)
#define FC_LAUNCH_ROWS_V(K) \
    switch (c->vec) { case 4: FC_LAUNCH_ROWS(4, K); break; case 2: FC_LAUNCH_ROWS(2, K); break; default: FC_LAUNCH_ROWS(1, K); break; }
    if (prof_item == P_EVICT_GATHER) { FC_LAUNCH_ROWS_V(0) }
    else if (prof_item == P_EVICT_STORE) { FC_LAUNCH_ROWS_V(1) }
    else { FC_LAUNCH_ROWS_V(2) }
#undef FC_LAUNCH_ROWS_V
#undef FC_LAUNCH_ROWS
    FC_HIP(hipGetLastError());
    return FC_OK;
}

// A sort to go along runs in the first workgroup of the launch (launch_rows_and_sort).
int launch_fill_rows(fc_cache* c, hipStream_t s, int64_t rows, float* dst, int64_t dst_rows, int max_blocks, bool only_transit,
                     const int32_t* plan, SortJob* along) {
    if (rows <= 0) return FC_OK;
    const int sh = shift_of(c->lpr);
    if (max_blocks <= 0) max_blocks = c->fill_blocks;
    const RowArgs a{dst ? dst : c->cache, dst ? nullptr : c->fill_slots, (unsigned)(dst ? dst_rows : c->C), c->host_dev, c->miss_ranks, (unsigned)c->N,
                    c->fill_src, c->stage_dev, (unsigned)(DMA_BLOCKS * c->staging_rows), (int)rows, c->D, sh, only_transit ? 1 : 0, plan};
    if (along) return launch_rows_and_sort(c, s, false, a, max_blocks, along);
    const unsigned blocks = (unsigned)std::min<int64_t>(cdiv(rows, 256 >> sh), max_blocks);
    ProfScope ps(c, P_MISS_FILL, s);
    switch (c->vec) {
        case 4: k_fill_rows<4><<<blocks, 256, 0, s>>>(a); break;
        case 2: k_fill_rows<2><<<blocks, 256, 0, s>>>(a); break;
        default: k_fill_rows<1><<<blocks, 256, 0, s>>>(a); break;
    }
    FC_HIP(hipGetLastError());
    return FC_OK;
}

int launch_swap_rows(fc_cache* c, hipStream_t s, int64_t rows, SortJob* along) {
    if (rows <= 0) return FC_OK;
    const int sh = shift_of(c->lpr);
    const RowArgs a{c->cache, c->fill_slots, (unsigned)c->C, c->host_dev, c->miss_ranks, (unsigned)c->N, c->fill_src, nullptr, 0, (int)rows, c->D, sh, 0, nullptr};
    if (along) return launch_rows_and_sort(c, s, true, a, c->swap_blocks, along);
    const unsigned blocks = (unsigned)std::min<int64_t>(cdiv(rows, 256 >> sh), c->swap_blocks);
    ProfScope ps(c, P_MISS_FILL, s);
    switch (c->vec) {
        case 4: k_swap_rows<4><<<blocks, 256, 0, s>>>(a); break;
        case 2: k_swap_rows<2><<<blocks, 256, 0, s>>>(a); break;
        default: k_swap_rows<1><<<blocks, 256, 0, s>>>(a); break;
    }
    FC_HIP(hipGetLastError());
    return FC_OK;
}

int launch_flush_rows(fc_cache* c, hipStream_t s) {
    const int sh = shift_of(c->lpr);
    const int gpb = 256 >> sh;
    int64_t blocks = cdiv(c->C, gpb);
    if (blocks > 8192) blocks = 8192;
    ProfScope ps(c, P_FLUSH_ROWS, s);
    switch (c->vec) {
        case 4: k_flush_rows<4><<<(unsigned)blocks, 256, 0, s>>>(c->host_dev, c->cache, c->slot_rank, (int)c->C, c->D, sh, c->dirty); break;
        case 2: k_flush_rows<2><<<(unsigned)blocks, 256, 0, s>>>(c->host_dev, c->cache, c->slot_rank, (int)c->C, c->D, sh, c->dirty); break;
        default: k_flush_rows<1><<<(unsigned)blocks, 256, 0, s>>>(c->host_dev, c->cache, c->slot_rank, (int)c->C, c->D, sh, c->dirty); break;
    }
    FC_HIP(hipGetLastError());
    return FC_OK;
}

}  // namespace fc
