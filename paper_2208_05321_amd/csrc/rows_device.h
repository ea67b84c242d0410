// Rows between the cache slots and the mapped host table, as device code: the kernels of fc_rows.hip, and the kernel of fc_small.hip
// that sorts in its first workgroup and moves rows in the others, are made of it.
#pragma once

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

// Where rows come from and go to; workgroup `wg` of `wgs` takes every wgs-th stretch of rows, a row-group of 1 << lpr_shift lanes one row.
struct RowArgs {
    float* cache; const int32_t* slots; unsigned slot_rows;      // destination rows (slots == nullptr: row j)
    float* host; const int32_t* miss_ranks; unsigned N;
    const int32_t* src;                                          // per row: the rank that leaves (swap), or where the newest copy is (fill)
    const float* blocks; unsigned block_rows;                    // fill: evicted-row blocks
    int rows, D, lpr_shift, only_transit;
    const int32_t* plan;                                         // fill, may be null: rows = the missing rows it states, if at most `rows`
};

// Rows change places (default transmitter): slot slots[j] gives its row to the host table (row src[j]; -1: the slot
// was empty) and gets row miss_ranks[j] from there.  Every slot and every host row occurs once, so no row waits for another
// and no block in between is needed.  Bound by the host link; what it replaces moved each evicted row through HBM twice more,
// and needed a second stream with two waits of 10 us each.
template <int VEC>
__device__ __forceinline__ void swap_rows(const RowArgs& a, int wg, int wgs) {
    using V = typename Vec<VEC>::T;
    const int lpr = 1 << a.lpr_shift;
    const int gpb = blockDim.x >> a.lpr_shift;
    const int gl = threadIdx.x >> a.lpr_shift, lane = threadIdx.x & (lpr - 1);
    const int nv = a.D / VEC;
    const int stride = wgs * gpb;
    int j = wg * gpb + gl;
    int s = 0, r = 0, o = -1;                // the list entries of the next row are requested before this row's data
    if (j < a.rows) { s = a.slots[j]; r = a.miss_ranks[j]; o = a.src[j]; }
    while (j < a.rows) {
        const int jn = j + stride;
        int sn = 0, rn = 0, on = -1;
        if (jn < a.rows) { sn = a.slots[jn]; rn = a.miss_ranks[jn]; on = a.src[jn]; }
        if ((unsigned)s < a.slot_rows && (unsigned)r < a.N) {            // never false for lists this library builds
            V* row = reinterpret_cast<V*>(a.cache + (size_t)s * a.D);
            const V* in = reinterpret_cast<const V*>(a.host + (size_t)r * a.D);
            V* out = reinterpret_cast<V*>(a.host + (size_t)o * a.D);
            const bool leaves = (unsigned)o < a.N;
            for (int cidx = lane; cidx < nv; cidx += lpr) {
                const V v = in[cidx];
                if (leaves) out[cidx] = nt_load_row(&row[cidx]);
                row[cidx] = v;
            }
        }
        j = jn; s = sn; r = rn; o = on;
    }
}

// Miss fill of the DMA evict transmitter: row j goes to slot slots[j] (to row j if there is no such list); it
// comes from the host table, or, if its newest copy is still in transit (src[j] <= -2), from the evicted-row
// block that holds it.
template <int VEC>
__device__ __forceinline__ void fill_rows(const RowArgs& a, int wg, int wgs) {
    int rows = a.rows;
    if (a.plan) rows = a.plan[PL_STATUS] == FC_OK && a.plan[PL_MISS] <= rows ? a.plan[PL_MISS] : 0;
    using V = typename Vec<VEC>::T;
    const int lpr = 1 << a.lpr_shift;
    const int gpb = blockDim.x >> a.lpr_shift;
    const int gl = threadIdx.x >> a.lpr_shift, lane = threadIdx.x & (lpr - 1);
    const int nv = a.D / VEC;
    // The three list entries of the NEXT row are requested before this row's data: each is a dependent access of a
    // microsecond or so, and a row-group that waits for them has no host read in flight.
    const int stride = wgs * gpb;
    int j = wg * gpb + gl;
    int di = 0, code = -1, r = 0;
    if (j < rows) { di = a.slots ? a.slots[j] : j; code = a.src[j]; r = a.miss_ranks[j]; }
    while (j < rows) {
        const int jn = j + stride;
        int din = 0, coden = -1, rn = 0;
        if (jn < rows) { din = a.slots ? a.slots[jn] : jn; coden = a.src[jn]; rn = a.miss_ranks[jn]; }
        const float* srow = nullptr;
        if (code <= -2) {
            const unsigned k = (unsigned)(-2 - code);
            if (k < a.block_rows) srow = a.blocks + (size_t)k * a.D;
        } else if (!a.only_transit && (unsigned)r < a.N) {
            srow = a.host + (size_t)r * a.D;
        }
        if (srow && (unsigned)di < a.slot_rows) {          // never false for lists this library builds
            const V* __restrict__ sv = reinterpret_cast<const V*>(srow);
            V* __restrict__ d = reinterpret_cast<V*>(a.cache + (size_t)di * a.D);
            for (int cidx = lane; cidx < nv; cidx += lpr) d[cidx] = sv[cidx];
        }
        j = jn; di = din; code = coden; r = rn;
    }
}

static inline int shift_of(int lpr) { int s = 0; while ((1 << s) < lpr) ++s; return s; }

}  // namespace fc
