// Row movement: one row-group of lanes per embedding row, 16-byte accesses where dim allows.
// Used for the evict gather, the host-table store of evicted rows, the miss fill and the flush
// (paper Section 4.3, "data transmitter": rows scattered in one memory become a block in the other).
#include "fc_internal.h"

namespace fc {

template <int VEC> struct Vec;
template <> struct Vec<1> { using T = float; };
template <> struct Vec<2> { using T = float2; };
template <> struct Vec<4> { using T = float4; };
__device__ __forceinline__ float nt_load_row(const float* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ float2 nt_load_row(const float2* p) { return make_float2(__builtin_nontemporal_load(&p->x), __builtin_nontemporal_load(&p->y)); }
__device__ __forceinline__ float4 nt_load_row(const float4* p) {
    typedef float v4f __attribute__((ext_vector_type(4)));
    const v4f t = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p));
    return make_float4(t.x, t.y, t.z, t.w);
}

// dst[dst_idx ? dst_idx[j] : j] = src[src_idx ? src_idx[j] : j] for j in [0, rows); row length D floats.
// lpr (power of two, <= 64) consecutive lanes own one row; a lane moves VEC floats per access.
// KIND only names the instantiation (profilers then tell the three uses apart): 0 evicted-row gather (HBM -> HBM
// block), 1 evicted-row store (block -> host table), 2 miss fill (host table -> cache slots, or block -> slots).
template <int VEC, int KIND>
__global__ __launch_bounds__(256) void k_copy_rows(float* __restrict__ dst, const int32_t* __restrict__ dst_idx,
                                                   unsigned dst_rows, const float* __restrict__ src,
                                                   const int32_t* __restrict__ src_idx, unsigned src_rows, int rows,
                                                   int D, int lpr_shift, int32_t* __restrict__ tag_out,
                                                   const int32_t* __restrict__ tags) {
    using V = typename Vec<VEC>::T;
    const int lpr = 1 << lpr_shift;
    const int gpb = blockDim.x >> lpr_shift;
    const int gl = threadIdx.x >> lpr_shift, lane = threadIdx.x & (lpr - 1);
    const int nv = D / VEC;
    for (int j = blockIdx.x * gpb + gl; j < rows; j += gridDim.x * gpb) {
        const int di = dst_idx ? dst_idx[j] : j;
        const int si = src_idx ? src_idx[j] : j;
        if (KIND == 0 && tag_out && lane == 0) tag_out[j] = tags[j];
        if ((unsigned)di >= dst_rows || (unsigned)si >= src_rows) continue;   // never true for lists this library builds
        const V* __restrict__ s = reinterpret_cast<const V*>(src + (size_t)si * D);
        V* __restrict__ d = reinterpret_cast<V*>(dst + (size_t)di * D);
        // the evicted rows and the rows of an arrival block are read for the last time here: non-temporal loads keep them
        // from displacing the cached rows in the memory-side cache
        for (int cidx = lane; cidx < nv; cidx += lpr) d[cidx] = KIND == 1 ? s[cidx] : nt_load_row(&s[cidx]);
    }
}

// Rows change places (default transmitter): slot fill_slots[j] gives its row to the host table (row old_rank[j]; -1: the slot
// was empty) and gets row miss_ranks[j] from there.  Every slot and every host row occurs once, so no row waits for another
// and no block in between is needed.  Bound by the host link; what it replaces moved each evicted row through HBM twice more,
// and needed a second stream with two waits of 10 us each.
template <int VEC>
__global__ __launch_bounds__(256) void k_swap_rows(float* __restrict__ cache, const int32_t* __restrict__ fill_slots, unsigned C,
                                                   float* host, const int32_t* __restrict__ miss_ranks,
                                                   const int32_t* __restrict__ old_rank, unsigned N, int rows, int D, int lpr_shift) {
    using V = typename Vec<VEC>::T;
    const int lpr = 1 << lpr_shift;
    const int gpb = blockDim.x >> lpr_shift;
    const int gl = threadIdx.x >> lpr_shift, lane = threadIdx.x & (lpr - 1);
    const int nv = D / VEC;
    const int stride = gridDim.x * gpb;
    int j = blockIdx.x * gpb + gl;
    int s = 0, r = 0, o = -1;                // the list entries of the next row are requested before this row's data
    if (j < rows) { s = fill_slots[j]; r = miss_ranks[j]; o = old_rank[j]; }
    while (j < rows) {
        const int jn = j + stride;
        int sn = 0, rn = 0, on = -1;
        if (jn < rows) { sn = fill_slots[jn]; rn = miss_ranks[jn]; on = old_rank[jn]; }
        if ((unsigned)s < C && (unsigned)r < N) {            // never false for lists this library builds
            V* row = reinterpret_cast<V*>(cache + (size_t)s * D);
            const V* in = reinterpret_cast<const V*>(host + (size_t)r * D);
            V* out = reinterpret_cast<V*>(host + (size_t)o * D);
            const bool leaves = (unsigned)o < N;
            for (int cidx = lane; cidx < nv; cidx += lpr) {
                const V v = in[cidx];
                if (leaves) out[cidx] = nt_load_row(&row[cidx]);
                row[cidx] = v;
            }
        }
        j = jn; s = sn; r = rn; o = on;
    }
}

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

// Miss fill of the DMA evict transmitter: row j goes to slot fill_slots[j] (to row j if there is no such list); it
// comes from the host table, or, if its newest copy is still in transit (fill_src[j] <= -2), from the evicted-row
// block that holds it.
template <int VEC>
__global__ __launch_bounds__(256) void k_fill_rows(float* __restrict__ cache, const int32_t* __restrict__ fill_slots,
                                                   unsigned C, const float* __restrict__ host,
                                                   const int32_t* __restrict__ miss_ranks, unsigned N,
                                                   const float* __restrict__ blocks, const int32_t* __restrict__ fill_src,
                                                   unsigned block_rows, int rows, int D, int lpr_shift, int only_transit,
                                                   const int32_t* __restrict__ plan) {
    if (plan) rows = plan[PL_STATUS] == FC_OK && plan[PL_MISS] <= rows ? plan[PL_MISS] : 0;
    using V = typename Vec<VEC>::T;
    const int lpr = 1 << lpr_shift;
    const int gpb = blockDim.x >> lpr_shift;
    const int gl = threadIdx.x >> lpr_shift, lane = threadIdx.x & (lpr - 1);
    const int nv = D / VEC;
    // The three list entries of the NEXT row are requested before this row's data: each is a dependent access of a
    // microsecond or so, and a row-group that waits for them has no host read in flight.
    const int stride = gridDim.x * gpb;
    int j = blockIdx.x * gpb + gl;
    int di = 0, code = -1, r = 0;
    if (j < rows) { di = fill_slots ? fill_slots[j] : j; code = fill_src[j]; r = miss_ranks[j]; }
    while (j < rows) {
        const int jn = j + stride;
        int din = 0, coden = -1, rn = 0;
        if (jn < rows) { din = fill_slots ? fill_slots[jn] : jn; coden = fill_src[jn]; rn = miss_ranks[jn]; }
        const float* srow = nullptr;
        if (code <= -2) {
            const unsigned k = (unsigned)(-2 - code);
            if (k < block_rows) srow = blocks + (size_t)k * D;
        } else if (!only_transit && (unsigned)r < N) {
            srow = host + (size_t)r * D;
        }
        if (srow && (unsigned)di < C) {          // never false for lists this library builds
            const V* __restrict__ sv = reinterpret_cast<const V*>(srow);
            V* __restrict__ d = reinterpret_cast<V*>(cache + (size_t)di * D);
            for (int cidx = lane; cidx < nv; cidx += lpr) d[cidx] = sv[cidx];
        }
        j = jn; di = din; code = coden; r = rn;
    }
}

static inline int shift_of(int lpr) { int s = 0; while ((1 << s) < lpr) ++s; return s; }

int launch_copy_rows(fc_cache* c, hipStream_t s, int prof_item, float* dst, const int32_t* dst_idx, int64_t dst_rows,
                     const float* src, const int32_t* src_idx, int64_t src_rows, int64_t rows, int max_blocks, int32_t* tag_out,
                     const int32_t* tags) {
    if (rows <= 0) return FC_OK;
    const int sh = shift_of(c->lpr);
    const int gpb = 256 >> sh;
    int64_t blocks = cdiv(rows, gpb);
    if (blocks > max_blocks) blocks = max_blocks;
    ProfScope ps(c, prof_item, s);
#define FC_LAUNCH_ROWS(V, K) \
    k_copy_rows<V, K><<<(unsigned)blocks, 256, 0, s>>>(dst, dst_idx, (unsigned)dst_rows, src, src_idx, (unsigned)src_rows, (int)rows, c->D, sh, tag_out, tags)
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

int launch_fill_rows(fc_cache* c, hipStream_t s, int64_t rows, float* dst, int64_t dst_rows, int max_blocks, bool only_transit,
                     const int32_t* plan) {
    if (rows <= 0) return FC_OK;
    const int sh = shift_of(c->lpr);
    const int gpb = 256 >> sh;
    int64_t blocks = cdiv(rows, gpb);
    if (max_blocks <= 0) max_blocks = c->fill_blocks;
    if (blocks > max_blocks) blocks = max_blocks;
    ProfScope ps(c, P_MISS_FILL, s);
#define FC_FILL(V) \
    k_fill_rows<V><<<(unsigned)blocks, 256, 0, s>>>(dst ? dst : c->cache, dst ? nullptr : c->fill_slots, (unsigned)(dst ? dst_rows : c->C), \
                                                    c->host_dev, c->miss_ranks, (unsigned)c->N, \
                                                    c->stage_dev, c->fill_src, (unsigned)(DMA_BLOCKS * c->staging_rows), (int)rows, c->D, sh, only_transit ? 1 : 0, plan)
    switch (c->vec) { case 4: FC_FILL(4); break; case 2: FC_FILL(2); break; default: FC_FILL(1); break; }
#undef FC_FILL
    FC_HIP(hipGetLastError());
    return FC_OK;
}

int launch_swap_rows(fc_cache* c, hipStream_t s, int64_t rows) {
    if (rows <= 0) return FC_OK;
    const int sh = shift_of(c->lpr);
    int64_t blocks = cdiv(rows, 256 >> sh);
    if (blocks > c->fill_blocks) blocks = c->fill_blocks;
    ProfScope ps(c, P_MISS_FILL, s);
#define FC_SWAP(V) \
    k_swap_rows<V><<<(unsigned)blocks, 256, 0, s>>>(c->cache, c->fill_slots, (unsigned)c->C, c->host_dev, c->miss_ranks, c->fill_src, (unsigned)c->N, (int)rows, c->D, sh)
    switch (c->vec) { case 4: FC_SWAP(4); break; case 2: FC_SWAP(2); break; default: FC_SWAP(1); break; }
#undef FC_SWAP
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
