// cache_prepare: Algorithm 1 of the paper (PrepareCache + PrepareCPURowIdxOnGPU, Section 4.3) as a short
// chain of gfx950 kernels.
//
// The paper's prototype strings together framework calls (unique, isin, nonzero, index_fill, argsort,
// index_copy).  Here the same decisions come out of two rank-space bitmaps and popcount scans, with no sort:
//   ubits  rows used by this batch        -> unique() is "which bits are set", ascending for free
//   rbits  rows resident in HBM           -> missing = ubits & ~rbits, evictable = rbits & ~ubits
// and the empty slots are read off the slot->rank map: the i-th missing rank takes the i-th empty slot.
// The victims of Section 4.3 (LFU by static frequency rank: of the rows the batch does not use, the evict_num with
// the largest cpu_row_idx) are the top evict_num set bits of (rbits & ~ubits): a suffix count over bitmap tiles finds the threshold tile.
#include "fc_internal.h"

#include <omp.h>
#include <string.h>

#include <algorithm>
#include <utility>

namespace fc {

// ---------------------------------------------------------------------------------------------------------
// K1  ids -> frequency rank (idx_map lookup), mark the rank, count access-level hits, check offsets.
//
// A mark is a byte per rank, set by a plain store (every writer stores the same 1, and the L2s merge bytes): no atomics to queue up
// on popular rows, nothing in LDS to clear and merge, and small workgroups that find room beside the previous batch's forward and
// backward kernels.  Frequent ids are by construction the LOW ranks, so below `dense` ranks K2a reads every byte; above, marks
// are few, and a second byte says which MARK_CHUNK ranks hold any, so that K2a reads those alone (and a batch whose popular
// rows have moved to high ranks costs no more than the reads).  Bound by the latency of two random reads per id.
// Measured (us, a bitmap set by atomics, popular ranks in LDS first, and its count -> these two): 426 k ids, 10 M rows 25.6 + 6.3 ->
// 8.8 + 6.4; 53 k ids, 4 M rows 14.0 + 3.7 -> 7.0 + 5.2; 1.7 M ids, 100 M rows, beside backward 66-74 + 5.8 -> 41-46 + 13.  `dense` at
// 2 / 4 / 8 / 32 ranks per id, K2a alone: 12.7 / 13.1 / 12.8 / 17.2 at 100 M rows, 5.5 / 5.9 / 5.7 / 6.3 at 10 M; without the chunks (all of the
// 100 M bytes read) 26.
// ---------------------------------------------------------------------------------------------------------
constexpr int MARK_THREADS = 256, MARK_ITEMS = 4;
constexpr int MARK_CHUNK = 256;

__global__ __launch_bounds__(MARK_THREADS) void k_remap_mark(const int64_t* __restrict__ ids, int n,
                                                               const int64_t* __restrict__ offsets, int num_bags,
                                                               const int32_t* __restrict__ freq_rank, int64_t N,
                                                               uint8_t* __restrict__ ubytes, uint8_t* __restrict__ uchunks, int dense,
                                                               const uint32_t* __restrict__ rbits,
                                                               int32_t* __restrict__ rbuf, uint32_t* err, int32_t* __restrict__ hitpart,
                                                               int4* __restrict__ gsum, int groups) {
    __shared__ int red[MARK_THREADS / 64];
    const int tid = threadIdx.x;
    for (int g = blockIdx.x * MARK_THREADS + tid; g < groups; g += gridDim.x * MARK_THREADS) gsum[g] = make_int4(0, 0, 0, 0);      // for K2a
    const int64_t work = n > num_bags + 1 ? n : num_bags + 1;
    int hits = 0;
    uint32_t flags = 0;
    for (int64_t i0 = (int64_t)blockIdx.x * (MARK_ITEMS * MARK_THREADS) + tid; i0 < work; i0 += (int64_t)gridDim.x * (MARK_ITEMS * MARK_THREADS)) {
        int64_t id[MARK_ITEMS], o0[MARK_ITEMS], o1[MARK_ITEMS];
        int r[MARK_ITEMS];
        uint32_t rb[MARK_ITEMS];
#pragma unroll
        for (int k = 0; k < MARK_ITEMS; ++k) {
            const int64_t i = i0 + k * MARK_THREADS;
            id[k] = i < n ? ids[i] : 0;
            o0[k] = i <= num_bags ? offsets[i] : 0;
            o1[k] = i < num_bags ? offsets[i + 1] : o0[k];
        }
#pragma unroll
        for (int k = 0; k < MARK_ITEMS; ++k) {
            const bool ok = (uint64_t)id[k] < (uint64_t)N;
            if (!ok) flags |= EF_ID_RANGE;
            r[k] = ok ? freq_rank[id[k]] : -1;
        }
#pragma unroll
        for (int k = 0; k < MARK_ITEMS; ++k) rb[k] = r[k] >= 0 ? rbits[(uint32_t)r[k] >> 5] : 0u;
#pragma unroll
        for (int k = 0; k < MARK_ITEMS; ++k) {
            const int64_t i = i0 + k * MARK_THREADS;
            if (i < n) {
                if (r[k] >= 0) {
                    ubytes[r[k]] = 1;
                    if (r[k] >= dense) uchunks[r[k] / MARK_CHUNK] = 1;
                    hits += (rb[k] >> (r[k] & 31)) & 1u;
                }
                rbuf[i] = r[k];
            }
            if (i <= num_bags) {
                if (o0[k] != i) flags |= EF_NOT_ONE_PER_BAG;
                if ((i == 0 && o0[k] != 0) || (i == num_bags && o0[k] != (int64_t)n) || o1[k] < o0[k]) flags |= EF_BAD_OFFSETS;
            }
        }
    }
    hits = wave_sum(hits);
    if ((tid & 63) == 0) red[tid >> 6] = hits;
    __syncthreads();
    if (tid == 0) {
        int s = 0;
#pragma unroll
        for (int k = 0; k < MARK_THREADS / 64; ++k) s += red[k];
        hitpart[blockIdx.x] = s;
    }
    if (flags) atomicOr(err, flags);
}

// ---------------------------------------------------------------------------------------------------------
// K1 where device memory has no room for the bytes: marks are bits of ubits, cleared before.  Device-scope atomics on one address
// serialise at the memory side (~100 ns each on this part), so the low end of rank space, the popular rows, is first marked in a
// per-workgroup LDS bitmap and merged into the global one once per workgroup; only the long tail of rare ranks goes to global
// atomics directly.  At most BITS_MAX_BLOCKS workgroups run, so a hot word sees at most that many global atomics.
// us, beside forward and backward, bytes / this / global atomics alone: 53 k ids, 4 M rows 10 / 16 / 49; 426 k ids, 10 M rows 24 / 38 / 209; 1.7 M ids,
// 100 M rows 38 / 66 / 498.
// ---------------------------------------------------------------------------------------------------------
constexpr int BITS_THREADS = 1024, BITS_ITEMS = 2;
constexpr int BITS_LDS_WORDS = 12288;      // 48 KB: ranks below 393,216
constexpr int BITS_MAX_BLOCKS = 256;

__global__ __launch_bounds__(BITS_THREADS) void k_remap_bits(const int64_t* __restrict__ ids, int n,
                                                             const int64_t* __restrict__ offsets, int num_bags,
                                                             const int32_t* __restrict__ freq_rank, int64_t N,
                                                             uint32_t* ubits, const uint32_t* __restrict__ rbits,
                                                             int32_t* __restrict__ rbuf, uint32_t* err,
                                                             int32_t* __restrict__ hitpart, int per_block,
                                                             int lds_words, int4* __restrict__ gsum, int groups) {
    __shared__ uint32_t low[BITS_LDS_WORDS];
    __shared__ int red[BITS_THREADS / 64];
    const int tid = threadIdx.x;
    for (int g = blockIdx.x * BITS_THREADS + tid; g < groups; g += gridDim.x * BITS_THREADS) gsum[g] = make_int4(0, 0, 0, 0);      // for K2a
    for (int w = tid; w < lds_words; w += BITS_THREADS) low[w] = 0;
    __syncthreads();
    const int64_t work = n > num_bags + 1 ? n : num_bags + 1;
    const int64_t begin = (int64_t)blockIdx.x * per_block;
    const int64_t end = begin + per_block < work ? begin + per_block : work;
    int hits = 0;
    uint32_t flags = 0;
    // four ids per thread and round: all loads of a stage are issued before any of them is waited for
    for (int64_t i0 = begin + tid; i0 < end; i0 += 4 * BITS_THREADS) {
        int64_t id[4];
        int r[4];
        uint32_t rb[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t i = i0 + (int64_t)k * BITS_THREADS;
            id[k] = (i < end && i < n) ? ids[i] : 0;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t i = i0 + (int64_t)k * BITS_THREADS;
            r[k] = -1;
            if (i < end && i < n) {
                if (id[k] < 0 || id[k] >= N) flags |= EF_ID_RANGE;
                else r[k] = freq_rank[id[k]];
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) rb[k] = r[k] >= 0 ? rbits[(uint32_t)r[k] >> 5] : 0u;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t i = i0 + (int64_t)k * BITS_THREADS;
            if (i < end && i < n) {
                if (r[k] >= 0) {
                    const uint32_t w = (uint32_t)r[k] >> 5, bit = 1u << (r[k] & 31);
                    if (w < (uint32_t)lds_words) atomicOr(&low[w], bit);
                    // rare ranks: bits are only ever set during this kernel, so a read that sees the bit is final
                    else if (!(ubits[w] & bit)) atomicOr(&ubits[w], bit);
                    hits += (rb[k] & bit) != 0;
                }
                rbuf[i] = r[k];
            }
            if (i < end && i <= num_bags) {
                const int64_t o = offsets[i];
                if (o != i) flags |= EF_NOT_ONE_PER_BAG;
                if (i == 0 && o != 0) flags |= EF_BAD_OFFSETS;
                if (i == num_bags && o != (int64_t)n) flags |= EF_BAD_OFFSETS;
                if (i < num_bags && offsets[i + 1] < o) flags |= EF_BAD_OFFSETS;
            }
        }
    }
    __syncthreads();
    // Merge into the global bitmap: LDS words first, then all global reads at once, then the atomics still needed.
    // Every workgroup holds the hottest words, so each starts at a different word: by the time most of them reach a
    // hot word its bits are already set and the (coherent) read spares the atomic.
    const int rot = (int)(((int64_t)blockIdx.x * lds_words) / gridDim.x);
    constexpr int FL = BITS_LDS_WORDS / BITS_THREADS;
    uint32_t v[FL], g[FL];
    int wi[FL];
#pragma unroll
    for (int k = 0; k < FL; ++k) {
        int w = k * BITS_THREADS + tid;
        v[k] = 0;
        if (w < lds_words) {
            w += rot;
            if (w >= lds_words) w -= lds_words;
            v[k] = low[w];
        }
        wi[k] = w;
    }
#pragma unroll
    for (int k = 0; k < FL; ++k)
        g[k] = v[k] ? __hip_atomic_load(&ubits[wi[k]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0xFFFFFFFFu;
#pragma unroll
    for (int k = 0; k < FL; ++k)
        if (v[k] & ~g[k]) atomicOr(&ubits[wi[k]], v[k]);
    hits = wave_sum(hits);
    if ((tid & 63) == 0) red[tid >> 6] = hits;
    __syncthreads();
    if (tid == 0) {
        int s = 0;
#pragma unroll
        for (int k = 0; k < BITS_THREADS / 64; ++k) s += red[k];
        hitpart[blockIdx.x] = s;
    }
    if (flags) atomicOr(err, flags);
}

// ---------------------------------------------------------------------------------------------------------
// K2a  per rank-space tile: rows used, rows missing, rows evictable.  The tile's 32768 marks become its bitmap words (all of
//      them written) and the set ones are cleared.  A lane turns 16 bytes into 16 bits with four 4-byte dot products.
//      On the way (DMA evict transmitter): the block that this batch's victims will go to has reached the host table, so
//      rows still marked as in transit in it become plain "not resident" (what k_clear_transit does; folded in here
//      because nothing before K2c reads rank_slot, and a launch of its own lengthened the index chain).
// ---------------------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t bits_of(uint4 v) {
    const uint32_t lo = __builtin_amdgcn_udot4(v.y, 0x80402010u, __builtin_amdgcn_udot4(v.x, 0x08040201u, 0u, false), false);
    const uint32_t hi = __builtin_amdgcn_udot4(v.w, 0x80402010u, __builtin_amdgcn_udot4(v.z, 0x08040201u, 0u, false), false);
    return lo | hi << 8;
}

// A wavefront counts SUB_TILES / 4 sub-tiles of 4096 ranks, a lane 64 neighbouring ranks of each: four lanes share a chunk.
constexpr int WAVE_SUBS = SUB_TILES / (RT_THREADS / 64);

template <bool BYTES>
__global__ __launch_bounds__(RT_THREADS) void k_rank_count(uint4* ubytes16, uint8_t* uchunks, int dense_tiles, uint2* __restrict__ ubits64,
                                                           const uint2* __restrict__ rbits64, const uint2* __restrict__ pbits64, int protect_prev,
                                                           uint32_t* __restrict__ bsum, uint32_t* __restrict__ ssum, int4* gsum,
                                                           const int32_t* __restrict__ landed_ranks, int landed, int landed_base,
                                                           int32_t* rank_slot, uint32_t* next_err) {
    static_assert(SUB_TILES * 64 * 64 == RT_WORDS * 32 && MARK_CHUNK == 4 * 64, "");
    __shared__ int part[SUB_TILES], upart[RT_THREADS / 64];
    for (int j = blockIdx.x * RT_THREADS + threadIdx.x; j < landed; j += gridDim.x * RT_THREADS) {
        const int r = landed_ranks[j];
        if (rank_slot[r] == -2 - (landed_base + j)) rank_slot[r] = -1;
    }
    const bool dense = (int)blockIdx.x < dense_tiles;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const size_t p0 = (size_t)blockIdx.x * (RT_WORDS / 2) + w * (WAVE_SUBS * 64) + lane;      // 64-rank pieces
    uint4 v[WAVE_SUBS][4];
    uint2 q[WAVE_SUBS], pv[WAVE_SUBS];
    uint32_t any[WAVE_SUBS];
#pragma unroll
    for (int k = 0; k < WAVE_SUBS; ++k) any[k] = !BYTES ? 0u : dense ? 1u : uchunks[(p0 + k * 64) / 4];
#pragma unroll
    for (int k = 0; k < WAVE_SUBS; ++k) q[k] = rbits64[p0 + k * 64];
#pragma unroll
    for (int k = 0; k < WAVE_SUBS; ++k) pv[k] = protect_prev ? pbits64[p0 + k * 64] : make_uint2(0, 0);
#pragma unroll
    for (int k = 0; k < WAVE_SUBS; ++k) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[k][j] = make_uint4(0, 0, 0, 0);
        if (any[k]) {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[k][j] = ubytes16[(p0 + k * 64) * 4 + j];
        }
    }
    int cu = 0;
#pragma unroll
    for (int k = 0; k < WAVE_SUBS; ++k) {
        uint2 uu;
        if (BYTES) {
            uint32_t u[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                u[j] = bits_of(v[k][j]);
                if (u[j]) ubytes16[(p0 + k * 64) * 4 + j] = make_uint4(0, 0, 0, 0);
            }
            if (!dense && any[k] && (lane & 3) == 0) uchunks[(p0 + k * 64) / 4] = 0;       // its four lanes have read it, in one instruction
            uu = make_uint2(u[0] | u[1] << 16, u[2] | u[3] << 16);
            ubits64[p0 + k * 64] = uu;
        } else uu = ubits64[p0 + k * 64];
        cu += __popc(uu.x) + __popc(uu.y);
        // look-ahead: rows of the previously prepared batch are not evictable either
        const int miss = __popc(uu.x & ~q[k].x) + __popc(uu.y & ~q[k].y);
        const int evictable = __popc(q[k].x & ~pv[k].x & ~uu.x) + __popc(q[k].y & ~pv[k].y & ~uu.y);
        const int c = wave_sum(miss | evictable << 16);
        if (lane == 0) part[w * WAVE_SUBS + k] = c;
    }
    cu = wave_sum(cu);
    if (lane == 0) upart[w] = cu;
    __syncthreads();
    if (threadIdx.x < SUB_TILES) ssum[(size_t)blockIdx.x * SUB_TILES + threadIdx.x] = (uint32_t)part[threadIdx.x];
    if (threadIdx.x == 0) {
        uint32_t t = 0;                        // 32768 at most in either half
        int used = 0;
#pragma unroll
        for (int k = 0; k < SUB_TILES; ++k) t += (uint32_t)part[k];
#pragma unroll
        for (int k = 0; k < RT_THREADS / 64; ++k) used += upart[k];
        bsum[blockIdx.x] = t;
        // (cleared by K1; most tiles of a large table have nothing to add)
        int* g = reinterpret_cast<int*>(&gsum[blockIdx.x / GROUP_TILES]);
        if (t & 0xffff) atomicAdd(&g[0], (int)(t & 0xffff));
        if (t >> 16) atomicAdd(&g[1], (int)(t >> 16));
        if (protect_prev && used) atomicAdd(&g[2], used);
        if (blockIdx.x == 0) *next_err = 0;    // the next call's error word
    }
}

// ---------------------------------------------------------------------------------------------------------
// K2b  totals, the call's status, evict_num = numel(miss) - empty slots, and for a tile: where its missing ranks go in the
//      list, how many victims it gives up (from the top rank down) and where those go.
//
//      All of it is a sum over the tiles' counts.  K2a adds those of GROUP_TILES neighbours up (its atomics meet at most that often
//      on a word), so every workgroup of K2c works it out for its own tile from the sums of the groups and the counts of its own
//      group, and the first one reports to the host before it starts on its tile; a kernel of one workgroup in between took 6 us at
//      306 tiles and 11-16 at 3052, and a launch (3052 tiles, planning + emitting: 15.7 + 12.6 -> 20).
//      (Tried: letting the last workgroup of K2a to finish do this, found by an atomic ticket.  One ticket per tile on
//      one address costs about 100 ns each on this part, 300 us at 3052 tiles: slower than the launch it saves.)
// ---------------------------------------------------------------------------------------------------------
struct PlanArgs {
    const uint32_t *bsum, *ssum; const int4* gsum;       // K2a's counts: per tile, sub-tile and group of tiles
    const uint32_t* err; const uint32_t* async_flags;
    const int32_t* hitpart; HostCtl* hctl;
    int32_t* plan;                                   // status, victims, missing rows: the decision for kernels enqueued behind
    int NB, C, nfree, nmark, ticket, protect_prev;
};
struct PlanTotals { int status, used, miss, need; };

__device__ __forceinline__ PlanTotals plan_totals(const PlanArgs& a, int used, int miss, int evictable) {
    // without the look-ahead's second protected set, resident rows are either used or evictable
    if (!a.protect_prev) used = miss + (a.C - a.nfree) - evictable;
    const uint32_t ef = *a.err;
    PlanTotals t{FC_OK, used, miss, miss - a.nfree};
    if (ef & EF_BAD_OFFSETS) t.status = FC_ERR_BAD_OFFSETS;
    else if (ef & EF_ID_RANGE) t.status = FC_ERR_ID_OUT_OF_RANGE;
    else if (used > a.C) t.status = FC_ERR_BATCH_EXCEEDS_CACHE;
    if (t.need < 0) t.need = 0;
    // enough evictable rows?  (always, unless the look-ahead protects the previous batch as well)
    if (t.status == FC_OK && t.need > evictable) t.status = FC_ERR_BATCH_EXCEEDS_CACHE;
    if (t.status != FC_OK) t.need = 0;
    return t;
}

// K sums at once
template <int NT, int K>
__device__ __forceinline__ void block_sums(int (&v)[K], int* lds /* K * NT / 64 ints */) {
#pragma unroll
    for (int j = 0; j < K; ++j) {
        v[j] = wave_sum(v[j]);
        if ((threadIdx.x & 63) == 0) lds[j * (NT / 64) + (threadIdx.x >> 6)] = v[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < K; ++j) {
        v[j] = 0;
#pragma unroll
        for (int k = 0; k < NT / 64; ++k) v[j] += lds[j * (NT / 64) + k];
    }
    __syncthreads();
}

template <int NT>
__device__ __forceinline__ void plan_report(const PlanArgs& a, const PlanTotals& t, int* lds) {
    int sum[1] = {0};
    for (int k = threadIdx.x; k < a.nmark; k += NT) sum[0] += a.hitpart[k];
    block_sums<NT, 1>(sum, lds);
    const int hits = sum[0];
    if (threadIdx.x == 0) { a.plan[PL_STATUS] = t.status; a.plan[PL_NEED] = t.need; a.plan[PL_MISS] = t.miss; }
    if (threadIdx.x < HOST_REC_WORDS)
        report_to_host(a.hctl, a.ticket, t.status, t.used, t.miss, t.need, hits, t.status == FC_OK ? a.nfree + t.need - t.miss : a.nfree,
                       (int)*a.async_flags, (int)(*a.err & EF_NOT_ONE_PER_BAG), threadIdx.x);
}

constexpr int FREE_TILE = 1024;

// ---------------------------------------------------------------------------------------------------------
// K2c  write the missing ranks (ascending), pick and retire the victims, update rbits.
//      A thread lists its set bits in LDS; what touches memory per rank (a random read and two or three writes) is then done
//      by all threads side by side, all random reads of a thread before the first is waited for.
//      SPLIT workgroups share a tile.  Popularity falls off as a power, so the tiles just beyond the cached ranks hold ten
//      times the average number of missing and evicted ranks (13,000 of each in one tile at 142 k slots of 9.4 M rows), and
//      with a tile to a workgroup, one of those was the kernel's duration: 8 to a tile up to SPLIT_TILES tiles (33 M rows);
//      beyond, tiles are many and ranks spread thinner, and 8 times the workgroups take longer than the fullest tile.
//      Measured (us by events, k_rank_plan + one workgroup per tile with the bits handled one by one -> this): 852 k ids, 9.4 M rows
//      8.2 + 32 -> 16; 426 k ids, 10 M rows 7.5 + 20 -> 15 (plain), 10 + 29 -> 18 (pipelined).
// ---------------------------------------------------------------------------------------------------------
constexpr int EMIT_LIST = 4096;                // ranks of either kind listed at a time
constexpr int EMIT_SPLIT = SUB_TILES;

template <int WORDS> struct Bits { uint32_t w[WORDS]; };          // the bits of a thread: 16 of one word, or four words
__device__ __forceinline__ Bits<1> load_bits(const uint32_t* p, size_t i, Bits<1>) {
    return Bits<1>{{reinterpret_cast<const uint16_t*>(p)[i]}};
}
__device__ __forceinline__ Bits<4> load_bits(const uint32_t* p, size_t i, Bits<4>) {
    const uint4 v = reinterpret_cast<const uint4*>(p)[i];
    return Bits<4>{{v.x, v.y, v.z, v.w}};
}
__device__ __forceinline__ void store_bits(uint32_t* p, size_t i, const Bits<1>& b) { reinterpret_cast<uint16_t*>(p)[i] = (uint16_t)b.w[0]; }
__device__ __forceinline__ void store_bits(uint32_t* p, size_t i, const Bits<4>& b) {
    reinterpret_cast<uint4*>(p)[i] = make_uint4(b.w[0], b.w[1], b.w[2], b.w[3]);
}

template <int SPLIT>
__global__ __launch_bounds__(RT_THREADS) void k_rank_emit(const uint32_t* __restrict__ ubits, uint32_t* rbits, const uint32_t* __restrict__ pbits, PlanArgs a,
                                                          int32_t* __restrict__ miss_ranks, int32_t* __restrict__ vrank,
                                                          int32_t* __restrict__ vslot, int32_t* rank_slot,
                                                          int32_t* slot_rank, int transit_base,
                                                          int transit_rows, int32_t* __restrict__ fill_src) {
    // (ubits is rewritten by a later K2a in full and becomes pbits by a swap of pointers)
    static_assert(SPLIT == 1 || (SPLIT == 8 && RT_WORDS == 4 * RT_THREADS), "a thread holds 16 bits or four words");
    constexpr int WORDS = SPLIT == 1 ? 4 : 1;
    constexpr int RANKS = SPLIT == 1 ? 128 : 16;           // per thread
    using B = Bits<WORDS>;
    __shared__ int lds[7 * RT_THREADS / 64];
    __shared__ uint16_t mlist[EMIT_LIST], vlist[EMIT_LIST];
    const int tid = threadIdx.x, me = blockIdx.x / SPLIT, sub = blockIdx.x % SPLIT;
    const size_t idx = (size_t)blockIdx.x * RT_THREADS + tid;
    const B u = load_bits(ubits, idx, B()), r = load_bits(rbits, idx, B());
    B p{};
    if (a.protect_prev) p = load_bits(pbits, idx, B());
    // missing, evictable, used in all; missing before and evictable above this tile; both before this workgroup in the tile; bits here
    int sum[7] = {0, 0, 0, 0, 0, 0, 0};
    const int groups = (a.NB + GROUP_TILES - 1) / GROUP_TILES, mine = me / GROUP_TILES;
    for (int g = tid; g < groups; g += RT_THREADS) {
        const int4 v = a.gsum[g];
        sum[0] += v.x; sum[1] += v.y; sum[2] += v.z;
        if (g < mine) sum[3] += v.x;
        if (g > mine) sum[4] += v.y;
    }
    const int nb = mine * GROUP_TILES + tid;
    if (tid < GROUP_TILES && nb < a.NB) {
        const uint32_t v = a.bsum[nb];
        if (nb < me) sum[3] += (int)(v & 0xffff);
        if (nb > me) sum[4] += (int)(v >> 16);
    }
    if (SPLIT > 1 && tid >= 64 && tid < 64 + sub) {
        const uint32_t v = a.ssum[me * SPLIT + tid - 64];
        sum[3] += (int)(v & 0xffff);
        sum[5] = (int)(v >> 16);
    }
#pragma unroll
    for (int k = 0; k < WORDS; ++k) sum[6] |= (u.w[k] | r.w[k]) != 0;
    block_sums<RT_THREADS, 7>(sum, lds);
    const PlanTotals totals = plan_totals(a, sum[2], sum[0], sum[1]);
    if (blockIdx.x == 0) plan_report<RT_THREADS>(a, totals, lds);
    const int status = totals.status, need = totals.need, mbase = sum[3], above = sum[4];
    if (status != FC_OK) return;           // failed call: K2a has cleared the marks, nothing else is touched
    if (!sum[6]) return;                   // neither used nor resident rows here
    B mw, cw, vw{};
    int cm = 0, cc = 0;
#pragma unroll
    for (int k = 0; k < WORDS; ++k) {
        mw.w[k] = u.w[k] & ~r.w[k];
        cw.w[k] = r.w[k] & ~u.w[k] & ~p.w[k];
        cm += __popc(mw.w[k]);
        cc += __popc(cw.w[k]);
    }
    // victims of this tile: all but its `skip` lowest evictable ranks, the tiles above it having given theirs
    const int mine_c = (int)(a.bsum[me] >> 16);
    const int take = max(0, min(mine_c, need - above)), v0 = need - above - take;
    const int skip = mine_c - take - sum[5];   // counted from this workgroup's first evictable rank
    int both;
    const uint32_t pre = (uint32_t)block_excl_scan<RT_THREADS>((int)((uint32_t)cm | (uint32_t)cc << 16), both, lds);
    const int pm = (int)(pre & 0xffff), totm = (int)((uint32_t)both & 0xffff), totc = (int)((uint32_t)both >> 16);
    const int pv = (int)(pre >> 16) - max(skip, 0);        // place among this workgroup's victims; negative: stays
    const int vbase = v0 + max(-skip, 0), totv = max(0, totc - max(skip, 0));
    const bool transit = transit_base >= 0 && need <= transit_rows;
    const int rank0 = blockIdx.x * (RT_THREADS * RANKS);
    for (int w0 = 0; w0 < totm || w0 < totv; w0 += EMIT_LIST) {        // (one round if SPLIT > 1)
        if (cm && pm < w0 + EMIT_LIST && pm + cm > w0) {
            int q = pm - w0;
#pragma unroll
            for (int k = 0; k < WORDS; ++k)
                for (uint32_t word = mw.w[k]; word; word &= word - 1, ++q)
                    if ((unsigned)q < (unsigned)EMIT_LIST) mlist[q] = (uint16_t)(tid * RANKS + k * 32 + __ffs(word) - 1);
        }
        if (cc && pv < w0 + EMIT_LIST && pv + cc > w0) {
            int q = pv - w0;
#pragma unroll
            for (int k = 0; k < WORDS; ++k)
                for (uint32_t word = cw.w[k]; word; word &= word - 1, ++q)
                    if ((unsigned)q < (unsigned)EMIT_LIST) {
                        vlist[q] = (uint16_t)(tid * RANKS + k * 32 + __ffs(word) - 1);
                        vw.w[k] |= word & (0u - word);
                    }
        }
        __syncthreads();
        for (int t0 = tid; t0 < EMIT_LIST && (w0 + t0 - tid < totm || w0 + t0 - tid < totv); t0 += 4 * RT_THREADS) {
            int mr[4], ms[4], vr[4], vs[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int t = t0 + k * RT_THREADS;
                mr[k] = t < EMIT_LIST && w0 + t < totm ? rank0 + mlist[t] : -1;
                vr[k] = t < EMIT_LIST && w0 + t < totv ? rank0 + vlist[t] : -1;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                ms[k] = fill_src && mr[k] >= 0 ? rank_slot[mr[k]] : -1;
                vs[k] = vr[k] >= 0 ? rank_slot[vr[k]] : -1;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int t = w0 + t0 + k * RT_THREADS;
                if (mr[k] >= 0) {
                    miss_ranks[mbase + t] = mr[k];
                    // where the row's newest copy is: -1 the host table, <= -2 an evicted-row block (in transit)
                    if (fill_src) fill_src[mbase + t] = ms[k];
                }
                if (vr[k] >= 0) {
                    const int j = vbase + t;
                    vrank[j] = vr[k];
                    vslot[j] = vs[k];
                    // not resident any more; with the DMA evict transmitter the newest copy of the row is
                    // "in transit" in row j of an evicted-row block until the host threads have stored it
                    rank_slot[vr[k]] = transit ? -2 - (transit_base + j) : -1;
                    // empty, and whose row it still holds (every such slot is refilled below); the test is always true
                    if ((unsigned)vs[k] < (unsigned)a.C) slot_rank[vs[k]] = -2 - vr[k];
                }
            }
        }
        __syncthreads();
    }
    if (cm || totv > 0) {
        uint32_t changed = 0;
        B out;
#pragma unroll
        for (int k = 0; k < WORDS; ++k) { out.w[k] = (r.w[k] & ~vw.w[k]) | mw.w[k]; changed |= mw.w[k] | vw.w[k]; }
        if (changed) store_bits(rbits, idx, out);
    }
}

// ---------------------------------------------------------------------------------------------------------
// K6  the i-th missing rank takes the i-th lowest empty slot; both index maps are updated.
//     a) empty slots per tile of FREE_TILE slots;  b) each tile ranks its empty slots after the tiles below it.
// ---------------------------------------------------------------------------------------------------------
// 256 threads with 4 consecutive slots each: a workgroup this small finds room on a compute unit at once, also while
// the forward / backward kernels of the previous batch fill the chip (cache_plan_next)
constexpr int FREE_THREADS = 256;
constexpr int FREE_PER = FREE_TILE / FREE_THREADS;

// bit k set: slot s0 + k is empty
__device__ __forceinline__ unsigned empty_mask(const int32_t* __restrict__ slot_rank, int s0, int C) {
    unsigned m = 0;
    if (s0 + FREE_PER <= C) {
        const int4 v = *reinterpret_cast<const int4*>(slot_rank + s0);
        m = (v.x < 0 ? 1u : 0u) | (v.y < 0 ? 2u : 0u) | (v.z < 0 ? 4u : 0u) | (v.w < 0 ? 8u : 0u);
    } else {
        for (int k = 0; k < FREE_PER; ++k) if (s0 + k < C && slot_rank[s0 + k] < 0) m |= 1u << k;
    }
    return m;
}

__global__ __launch_bounds__(FREE_THREADS) void k_free_count(const int32_t* __restrict__ slot_rank, int C,
                                                             int32_t* __restrict__ tcount) {
    static_assert(FREE_PER == 4, "empty_mask reads four slots at a time");
    __shared__ int red[FREE_THREADS / 64];
    const int s0 = blockIdx.x * FREE_TILE + threadIdx.x * FREE_PER;
    const int e = __popc(empty_mask(slot_rank, s0, C));
    const int w = wave_sum(e);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = w;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
#pragma unroll
        for (int k = 0; k < FREE_THREADS / 64; ++k) t += red[k];
        tcount[blockIdx.x] = t;
    }
}

// LIST: no slot was empty before, so the empty ones are the victims', and each tile picks its own, and counts those of the tiles below it, from the
// list of victims: no kernel that counts them comes before.
constexpr int LIST_LOADS = 8;
template <bool LIST>
__global__ __launch_bounds__(FREE_THREADS) void k_free_assign(int32_t* slot_rank, int C, const int32_t* __restrict__ tcount, const int32_t* __restrict__ vslot,
                                                              int M, const int32_t* __restrict__ miss_ranks,
                                                              int32_t* __restrict__ fill_slots, int32_t* rank_slot,
                                                              int32_t* __restrict__ old_rank, const int32_t* __restrict__ plan,
                                                              uint8_t* dirty, uint64_t* __restrict__ dirty_words, int ticket) {
    // dirty: a row that leaves without having been updated is dropped (old_rank -1); this tile's updated ones are counted
    // plan: the number of missing rows as the device knows it (the host has not seen it yet)
    if (plan) M = plan[PL_STATUS] == FC_OK ? plan[PL_MISS] : 0;
    __shared__ int lds[FREE_THREADS / 64];
    __shared__ uint32_t bits[LIST ? FREE_TILE / 32 : 1];
    int part = 0;
    if (LIST) {
        if (threadIdx.x < FREE_TILE / 32) bits[threadIdx.x] = 0;
        __syncthreads();
        const int tile0 = blockIdx.x * FREE_TILE;
        auto look = [&](int s) {
            if (s < tile0) ++part;
            else if (s < tile0 + FREE_TILE) atomicOr(&bits[(s - tile0) >> 5], 1u << (s & 31));
        };
        // (a list much longer than the guess it was chosen by is bound by the latency of its loads: several on their way at once; 80 k victims of 100 k
        // slots 33 -> 18 us)
        int v = threadIdx.x * 4;
        for (; v - (int)threadIdx.x * 4 + LIST_LOADS * FREE_THREADS * 4 <= M; v += LIST_LOADS * FREE_THREADS * 4) {
            int4 q[LIST_LOADS];
#pragma unroll
            for (int k = 0; k < LIST_LOADS; ++k) q[k] = *reinterpret_cast<const int4*>(vslot + v + k * FREE_THREADS * 4);
#pragma unroll
            for (int k = 0; k < LIST_LOADS; ++k) { look(q[k].x); look(q[k].y); look(q[k].z); look(q[k].w); }
        }
        for (; v < M; v += FREE_THREADS * 4) {
            if (v + 4 <= M) {
                const int4 q = *reinterpret_cast<const int4*>(vslot + v);
                look(q.x); look(q.y); look(q.z); look(q.w);
            } else for (int u = v; u < M; ++u) look(vslot[u]);
        }
    } else for (int g = threadIdx.x; g < (int)blockIdx.x; g += FREE_THREADS) part += tcount[g];
    int base;
    (void)block_excl_scan<FREE_THREADS>(part, base, lds);
    if (base >= M) {                                         // all missing rows were placed in lower tiles
        if (dirty && threadIdx.x == 0) post_count(dirty_words + blockIdx.x, 0, ticket);
        return;
    }
    const int s0 = blockIdx.x * FREE_TILE + threadIdx.x * FREE_PER;
    static_assert(FREE_TILE % 32 == 0 && FREE_PER == 4, "a thread's four bits lie in one word");
    const unsigned m = LIST ? (bits[(threadIdx.x * FREE_PER) >> 5] >> ((threadIdx.x * FREE_PER) & 31)) & 15u : empty_mask(slot_rank, s0, C);
    int tot;
    int j = base + block_excl_scan<FREE_THREADS>(__popc(m), tot, lds), written = 0;
    for (int k = 0; k < FREE_PER; ++k) {
        if (!((m >> k) & 1u)) continue;
        if (j >= M) break;
        const int s = s0 + k;
        const int r = miss_ranks[j];
        fill_slots[j] = s;
        int leaves = -2 - min(slot_rank[s], -1);                    // rank of the row that leaves (-1: the slot was empty)
        if (dirty && leaves >= 0) {
            if (dirty[s]) { dirty[s] = 0; ++written; }
            else leaves = -1;
        }
        if (old_rank) old_rank[j] = leaves;
        slot_rank[s] = r;
        rank_slot[r] = s;
        ++j;
    }
    if (dirty) {
        (void)block_excl_scan<FREE_THREADS>(written, tot, lds);
        if (threadIdx.x == 0) post_count(dirty_words + blockIdx.x, tot, ticket);
    }
}

// ---------------------------------------------------------------------------------------------------------
// FC_DIRTY_TRACK: of the victims (vrank[j], vslot[j]), j < need, keep those whose slot is dirty, in order.
//     a) dirty victims per tile of DIRTY_TILE victims;  b) each tile writes its dirty victims after those of the
//     tiles before it, clears the dirty flags of all its victims, and (DMA evict transmitter) marks the kept rows as
//     in transit at their place in the block; the last tile reports the total to the host.
// ---------------------------------------------------------------------------------------------------------
constexpr int DIRTY_TILE = 1024;
constexpr int DIRTY_THREADS = 256;
constexpr int DIRTY_PER = DIRTY_TILE / DIRTY_THREADS;

__global__ __launch_bounds__(DIRTY_THREADS) void k_dirty_count(const int32_t* __restrict__ vslot, int need, int C,
                                                              const uint8_t* __restrict__ dirty, int32_t* __restrict__ dcount) {
    __shared__ int red[DIRTY_THREADS / 64];
    const int j0 = blockIdx.x * DIRTY_TILE + threadIdx.x * DIRTY_PER;
    int e = 0;
    for (int k = 0; k < DIRTY_PER; ++k) {
        const int j = j0 + k;
        if (j < need) { const int s = vslot[j]; if ((unsigned)s < (unsigned)C && dirty[s]) ++e; }
    }
    const int w = wave_sum(e);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = w;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
#pragma unroll
        for (int k = 0; k < DIRTY_THREADS / 64; ++k) t += red[k];
        dcount[blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(DIRTY_THREADS) void k_dirty_keep(const int32_t* __restrict__ vrank, const int32_t* __restrict__ vslot,
                                                             int need, int C, uint8_t* dirty, const int32_t* __restrict__ dcount,
                                                             int32_t* __restrict__ out_rank, int32_t* __restrict__ out_slot,
                                                             int32_t* rank_slot, int transit_base, int32_t* dctl, int ticket) {
    __shared__ int lds[DIRTY_THREADS / 64];
    int part = 0;
    for (int g = threadIdx.x; g < (int)blockIdx.x; g += DIRTY_THREADS) part += dcount[g];
    int base;
    (void)block_excl_scan<DIRTY_THREADS>(part, base, lds);
    const int j0 = blockIdx.x * DIRTY_TILE + threadIdx.x * DIRTY_PER;
    unsigned m = 0;
    int sl[DIRTY_PER];
    for (int k = 0; k < DIRTY_PER; ++k) {
        const int j = j0 + k;
        sl[k] = -1;
        if (j < need) {
            const int s = vslot[j];
            if ((unsigned)s < (unsigned)C) { sl[k] = s; if (dirty[s]) m |= 1u << k; }
        }
    }
    int tot;
    int o = base + block_excl_scan<DIRTY_THREADS>(__popc(m), tot, lds);
    for (int k = 0; k < DIRTY_PER; ++k) {
        if (sl[k] < 0) continue;
        if ((m >> k) & 1u) {
            const int r = vrank[j0 + k];
            out_rank[o] = r;
            out_slot[o] = sl[k];
            if (transit_base >= 0) rank_slot[r] = -2 - (transit_base + o);
            ++o;
        }
        dirty[sl[k]] = 0;                  // the slot is empty now; whatever is loaded next equals its host copy
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        dctl[0] = base + tot;
        __threadfence_system();
        *reinterpret_cast<volatile int32_t*>(&dctl[1]) = ticket;   // the count first, then the ticket the host polls for
    }
}

// DMA evict transmitter: the host threads have stored block `base / staging_rows`; rows still marked as in transit
// in that block are plain "not resident" again (a row re-fetched or re-evicted meanwhile carries another value).
__global__ __launch_bounds__(256) void k_clear_transit(const int32_t* __restrict__ ranks, int count, int base,
                                                       int32_t* rank_slot) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < count) {
        const int r = ranks[j];
        if (rank_slot[r] == -2 - (base + j)) rank_slot[r] = -1;
    }
}

// K8  gpu_row_idx of every input id.
__global__ __launch_bounds__(256) void k_slots_out(const int32_t* __restrict__ rbuf,
                                                   const int32_t* __restrict__ rank_slot, int32_t* __restrict__ slots,
                                                   int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) slots[i] = rank_slot[rbuf[i]];
}

// ---------------------------------------------------------------------------------------------------------
int ensure_rbuf(fc_cache* c, int64_t n) {
    if (n <= c->n_cap) return FC_OK;
    FC_HIP(hipDeviceSynchronize());
    if (c->rbuf) FC_HIP(hipFree(c->rbuf));
    c->rbuf = nullptr; c->n_cap = 0;
    const int64_t cap = n + n / 4 + 1024;
    FC_HIP(hipMalloc((void**)&c->rbuf, (size_t)cap * 4));
    c->n_cap = cap;
    return FC_OK;
}

__global__ __launch_bounds__(256) void k_zero_words(uint4* p) { p[(size_t)blockIdx.x * 256 + threadIdx.x] = make_uint4(0, 0, 0, 0); }

// The mark bytes and, in the same allocation, those of the chunks (zero between calls), with the first batch that needs them.  Where
// there is no room for them (num_rows bytes) marks are bits, until a cache_reserve finds room.
bool mark_bytes(fc_cache* c) {
    if (c->ubytes || c->no_mark_bytes) return c->ubytes != nullptr;
    const size_t ranks = (size_t)c->NB * RT_WORDS * 32, bytes = ranks + ranks / MARK_CHUNK;
    uint8_t* p = nullptr;
    if (hipMalloc((void**)&p, bytes) != hipSuccess || hipMemset(p, 0, bytes) != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
        (void)hipGetLastError();
        if (p) (void)hipFree(p);
        c->no_mark_bytes = true;
        return false;
    }
    c->ubytes = p;
    c->uchunks = p + ranks;
    return true;
}

// Evicted rows stored by kernel: gather into a device block on the caller's stream (so the slots can be refilled at once); the block
// is stored into the mapped host table by a kernel on the side stream.  This is how victims leave where the exchange of
// k_swap_rows does not apply: default transmitter with missing rows that were fetched ahead of time, or prepared ahead with FC_DIRTY_TRACK, and
// FC_EVICT_DMA with more victims than a block holds.
// Measured on MI355X: zero-copy stores that saturate the host link stall the other memory operations of the
// compute units they run on and starve reads in the other direction, so such a store must not run under small
// latency-bound kernels (they wait for it to end) nor under the forward / backward kernels (they slow down
// several-fold).  Default schedule (evict_early == 2): the store starts together with the miss fill, once all
// index kernels are done, and the caller's stream waits for it right after the fill; the two then share the
// link (the store finishes first, the fill catches up) and everything after runs undisturbed.
// Blocks before the last are stored at once because the one block buffer must be free again for the next gather.
static int store_block(fc_cache* c, int64_t off, int64_t rows) {
    FC_HIP(hipEventRecord(c->ev_gather_done, c->pst));
    FC_HIP(hipStreamWaitEvent(c->side, c->ev_gather_done, 0));
    FC_TRY(launch_copy_rows(c, c->side, P_EVICT_STORE, c->host_dev, c->out_rank + off, c->N, c->stage_dev, nullptr, c->staging_rows, rows, c->evict_blocks));
    FC_HIP(hipEventRecord(c->ev_evict_done, c->side));
    c->evict_pending = true;
    return FC_OK;
}

static int evict_direct(fc_cache* c, int64_t need, int64_t* last_off, int64_t* last_rows) {
    const int64_t S = c->staging_rows;
    for (int64_t off = 0; off < need; off += S) {
        const int64_t rows = need - off < S ? need - off : S;
        if (off > 0) FC_HIP(hipStreamWaitEvent(c->pst, c->ev_evict_done, 0));   // block buffer is being read
        FC_TRY(launch_copy_rows(c, c->pst, P_EVICT_GATHER, c->stage_dev, nullptr, c->staging_rows, c->cache, c->out_slot + off, c->C, rows, 1 << 20));
        if (off + rows >= need && c->evict_early != 1) { *last_off = off; *last_rows = rows; break; }
        FC_TRY(store_block(c, off, rows));
    }
    return FC_OK;
}

// Every handed-over block is in the host table: no row is in transit any more.
static int drop_transit_marks(fc_cache* c, hipStream_t st) {
    for (int b = 0; b < DMA_BLOCKS; ++b) {
        if (c->blk_rows[b] > 0) {
            k_clear_transit<<<(unsigned)cdiv(c->blk_rows[b], 256), 256, 0, st>>>(c->vrank_buf[b], (int)c->blk_rows[b],
                                                                                       (int)(b * c->staging_rows), c->rank_slot);
            c->blk_rows[b] = 0;
        }
    }
    FC_HIP(hipGetLastError());
    return FC_OK;
}

// DMA evict transmitter: wait until every handed-over block is in the host table and drop all transit marks
// (afterwards the host table alone is current for every non-resident row, and all blocks are free).
int dma_quiesce(fc_cache* c, hipStream_t st) {
    if (!c->dma_evict) return FC_OK;
    pool_wait(c, pool_published(c));
    FC_TRY(drop_transit_marks(c, st));
    // the index kernels of a later batch read and write the same map entries, possibly on another stream
    FC_HIP(hipEventRecord(c->ev_quiesce, st));
    c->quiesce_stream = st;
    return FC_OK;
}

// DMA evict transmitter: gather into block `buf` ...
static bool ranks_travel_along(const fc_cache* c, int64_t need) { return need * (int64_t)(c->D + 1) <= c->staging_rows * (int64_t)c->D; }
// A small block: the gather writes its rows (and ranks) into the pinned landing block as well, and there is no copy to hand over.  The copy
// costs the host 20-25 us (the side stream's wait for a gather that has just been enqueued 16, the copy and its events 5), the stores the
// caller's stream what they take on the link.  On a planned step that hides behind what the host does, so the limit is where the
// rows of the step stop being few (INLINE_BYTES); a plain one is in the way of the sort.
// us a step, copy / this: planned, 2.6 k lookups of 32 columns (31 KB) 107 / 70, 53 k of 64 columns (1.4 MB) 121 / 107 and the first pass 205 / 175 (both with the rows
// fetched on the index stream), of 96 columns (2.1 MB) 107 / 114, of 128 columns (2.7 MB) 124 / 132; plain, 1024 lookups of 16 columns 60 / 46, 10 k of 32 columns (134 KB)
// 83 / 79, 18 k of 64 columns (470 KB) 82 / 85.
static bool lands_directly(const fc_cache* c, int64_t need, bool ahead) {
    if (c->prof_on) return false;      // a span stands for the gather, or for the block's way over the link
    return ranks_travel_along(c, need) && need * (int64_t)c->D * 4 <= (ahead ? INLINE_BYTES : LAND_BYTES);
}
static int gather_block(fc_cache* c, int64_t need, int buf, bool ahead) {
    float* blk = c->stage_dev + (size_t)buf * c->staging_rows * c->D;
    // the ranks travel behind the rows, in one copy, where the block has room for both (a copy of their own costs the host as
    // much as four launches)
    const bool along = ranks_travel_along(c, need), direct = lands_directly(c, need, ahead);
    float* land = direct ? c->blk_pin[buf] : nullptr;
    FC_TRY(launch_copy_rows(c, c->pst, P_EVICT_GATHER, blk, nullptr, c->staging_rows, c->cache, c->out_slot, c->C, need, 1 << 20,
                            along ? reinterpret_cast<int32_t*>(blk + (size_t)need * c->D) : nullptr, c->out_rank, land,
                            direct ? reinterpret_cast<int32_t*>(land + (size_t)need * c->D) : nullptr));
    FC_HIP(hipEventRecord(c->ev_gather_done, c->pst));
    if (direct) FC_HIP(hipEventRecord(c->ev_d2h[buf], c->pst));
    return FC_OK;
}
// ... and hand the block and its rank list to the DMA engine on the side stream, and let the host threads scatter it once it has
// landed.  Nothing on the caller's stream waits for it.
// The host waits while this handle's last block is still on its way, if that was handed over a while ago (the rows that come in are
// enqueued by now, and the GPU is busy with them).  With several handles in turn nothing else holds it back until each has DMA_BLOCKS
// blocks in flight, and a dozen copies at once beside the fills take three times as long as one after the other and never catch up.
// us a step, three handles in turn, plain schedule, without / with this: 294 k lookups of 128 columns, 22 k rows each way 715 / 262,
// 781 k of 256 columns, 32 k rows 1645 / 616, 635 k of 107 columns, 9 k rows 485 / 484.  (`ahead_now`, as in wait_if_far_ahead: HBM binds.)
static int send_block(fc_cache* c, int64_t need, int buf, bool ahead) {
    const float* blk = c->stage_dev + (size_t)buf * c->staging_rows * c->D;
    const bool together = ranks_travel_along(c, need);
    if (lands_directly(c, need, ahead)) {                // its rows are on their way, or there
        c->vrank_at[buf] = reinterpret_cast<const int32_t*>(c->blk_pin[buf] + (size_t)need * c->D);
        c->copy_timed[buf] = false;
        c->blk_rows[buf] = need;
        c->copy_seq[buf] = pool_publish(c, buf, need);
        return FC_OK;
    }
    if (c->last_copy_buf >= 0 && c->copy_timed[c->last_copy_buf] && !(ahead && c->ahead_now)) {
        const float ago = std::chrono::duration<float, std::micro>(std::chrono::steady_clock::now() - c->copy_at).count();
        if (ago > FAR_AHEAD_US) FC_HIP(hipEventSynchronize(c->ev_d2h[c->last_copy_buf]));
    }
    FC_HIP(hipStreamWaitEvent(c->side, c->ev_gather_done, 0));
    {
        ProfScope ps(c, P_D2H_BLOCK, c->side);
        if (c->ev_copy_a[buf]) FC_HIP(hipEventRecord(c->ev_copy_a[buf], c->side));
        if (!together) FC_HIP(hipMemcpyAsync(c->vrank_pin[buf], c->out_rank, (size_t)need * 4, hipMemcpyDeviceToHost, c->side));
        FC_HIP(hipMemcpyAsync(c->blk_pin[buf], blk, (size_t)need * (c->D + (together ? 1 : 0)) * 4, hipMemcpyDeviceToHost, c->side));
    }
    FC_HIP(hipEventRecord(c->ev_d2h[buf], c->side));
    c->vrank_at[buf] = together ? reinterpret_cast<const int32_t*>(c->blk_pin[buf] + (size_t)need * c->D) : c->vrank_pin[buf];
    if (c->ev_copy_a[buf]) { c->copy_timed[buf] = true; c->last_copy_buf = buf; }
    c->blk_rows[buf] = need;
    c->copy_at = std::chrono::steady_clock::now();
    c->copy_seq[buf] = pool_publish(c, buf, need);
    return FC_OK;
}

// The paper's transmitter: block on the source side -> one bulk copy -> scatter on the target side.
static int evict_staged(fc_cache* c, int64_t need, const int32_t* vrank_host) {
    const int64_t S = c->staging_rows;
    const size_t rowb = (size_t)c->D * 4;
    for (int64_t off = 0; off < need; off += S) {
        const int64_t rows = need - off < S ? need - off : S;
        FC_TRY(launch_copy_rows(c, c->pst, P_EVICT_GATHER, c->stage_dev, nullptr, c->staging_rows, c->cache, c->out_slot + off, c->C, rows, 1 << 20));
        {
            ProfScope ps(c, P_D2H_BLOCK, c->pst);
            FC_HIP(hipMemcpyAsync(c->stage_pin, c->stage_dev, rows * rowb, hipMemcpyDeviceToHost, c->pst));
        }
        FC_HIP(hipStreamSynchronize(c->pst));
        float* host = c->host; const float* blk = c->stage_pin; const int32_t* vr = vrank_host + off;
#pragma omp parallel for schedule(static)
        for (int64_t j = 0; j < rows; ++j) memcpy(host + (size_t)vr[j] * c->D, blk + (size_t)j * c->D, rowb);
    }
    return FC_OK;
}

static int fill_staged(fc_cache* c, int64_t M, const int32_t* miss_host) {
    const int64_t S = c->staging_rows;
    const size_t rowb = (size_t)c->D * 4;
    for (int64_t off = 0; off < M; off += S) {
        const int64_t rows = M - off < S ? M - off : S;
        const float* host = c->host; float* blk = c->stage_pin; const int32_t* mr = miss_host + off;
#pragma omp parallel for schedule(static)
        for (int64_t j = 0; j < rows; ++j) memcpy(blk + (size_t)j * c->D, host + (size_t)mr[j] * c->D, rowb);
        {
            ProfScope ps(c, P_H2D_BLOCK, c->pst);
            FC_HIP(hipMemcpyAsync(c->stage_dev2, c->stage_pin, rows * rowb, hipMemcpyHostToDevice, c->pst));
        }
        FC_TRY(launch_copy_rows(c, c->pst, P_MISS_FILL, c->cache, c->fill_slots + off, c->C, c->stage_dev2, nullptr, c->staging_rows, rows, 1 << 20));
        FC_HIP(hipStreamSynchronize(c->pst));   // the pinned block is reused by the next round
    }
    return FC_OK;
}

// A kernel writes a small record into pinned host memory and, last, a ticket; the host polls for the ticket (cheaper
// than an event round trip, and the kernels enqueued behind it keep the GPU busy meanwhile).  Falls back to the
// stream's status so that a failed launch cannot hang the caller.
static int wait_for_ticket(const volatile int32_t* ticket_word, int32_t ticket, hipStream_t st) {
    uint64_t spins = 0;
    while (*ticket_word != ticket) {
        __builtin_ia32_pause();
        if ((++spins & 0x3FFF) == 0) {
            const hipError_t q = hipStreamQuery(st);
            if (q == hipSuccess) break;                          // stream drained: the record is there
            if (q != hipErrorNotReady) { (void)hipGetLastError(); return FC_ERR_HIP; }
        }
    }
    __atomic_thread_fence(__ATOMIC_ACQUIRE);
    return *ticket_word == ticket ? FC_OK : FC_ERR_HIP;
}

// The planning record, word by word (see HostCtl); usually all eight words are there once the last one is.
static int wait_for_record(const HostCtl* rec, int32_t ticket, hipStream_t st, int32_t* out) {
    for (int k = HOST_REC_WORDS - 1; k >= 0; --k) {
        const volatile uint64_t* word = &rec->word[k];
        FC_TRY(wait_for_ticket(reinterpret_cast<const volatile int32_t*>(word) + 1, ticket, st));
        out[k] = (int32_t)(uint32_t)*word;
    }
    return FC_OK;
}

// FC_DIRTY_TRACK: see fc_cache::dirty_words
int dirty_total(fc_cache* c) {
    int64_t rows = 0;
    for (int k = 0; k < c->dirty_parts; ++k) {
        const volatile uint64_t* word = c->dirty_words + k;
        FC_TRY(wait_for_ticket(reinterpret_cast<const volatile int32_t*>(word) + 1, c->dirty_ticket, c->stream));
        rows += (int64_t)(uint32_t)*word;
    }
    if (c->dirty_parts) { c->last.bytes_d2h = rows * (int64_t)c->D * 4; c->dirty_seen = rows; }
    c->dirty_parts = 0;
    return FC_OK;
}

// Whether a plain call's rows change places, the clean ones among the victims being dropped (FC_DIRTY_TRACK).  With FC_EVICT_DMA only while
// victims come out clean (serving) and no block is on its way: then there is nothing for the block and the host threads to do, and a row that
// does turn out dirty may be stored in its place at once, because no older copy of it is still to arrive there.  (Marks of blocks that have
// arrived are dropped here: the ring of blocks, which drops them otherwise, comes to a halt with the last dirty victim.  Serving after some training with
// the marks left in place / this: 30 k lookups of 128 columns 58 / 52.5 us a step, 3.3 k of 64 40 / 30, 664 of 32 34 / 24.5.)
// us a step, victims sorted out by two kernels and the host waiting for their number / this: 426 k lookups of 128 columns 478 / 462, 63 k of 128 133 / 121,
// 6.6 k of 128 55 / 44, 664 of 32 36 / 23; with FC_EVICT_DMA 30 k of 128 73 / 67, 135 of 10
// 32 / 20, 1.6 M of 16 203 / 192.
static bool drops_clean(fc_cache* c, hipStream_t st) {
    if (!c->dirty_words || st != c->stream) return false;
    if (!c->dma_evict) return true;
    bool there = true;               // the latest call's counts (nearly always: its kernels were enqueued a call ago)
    for (int k = 0; k < c->dirty_parts && there; ++k) there = (int32_t)(*(const volatile uint64_t*)(c->dirty_words + k) >> 32) == c->dirty_ticket;
    if (there && c->dirty_parts && dirty_total(c) != FC_OK) return false;
    if (c->dirty_seen != 0) return false;
    bool marked = false;
    for (int64_t rows : c->blk_rows) marked |= rows > 0;
    return !marked || (pool_completed(c) == pool_published(c) && drop_transit_marks(c, st) == FC_OK);
}

// Index half of Algorithm 1: every decision (unique rows, misses, victims, slot assignment, both maps, the slots
// of the batch) and no row movement.  Fills *mv with what prepare_move has to do.
int launch_slots_out(fc_cache* c, hipStream_t st, int32_t* slots, int64_t n) {
    if (n > 0) {
        ProfScope ps(c, P_SLOTS_OUT, st);
        k_slots_out<<<(unsigned)cdiv(n, 256), 256, 0, st>>>(c->rbuf, c->rank_slot, slots, (int)n);
    }
    FC_HIP(hipGetLastError());
    return FC_OK;
}

// Everything up to the decisions (the emitting kernel), enqueued.  write_slots: a small batch's one kernel writes them, too.
int index_launch(fc_cache* c, hipStream_t st, bool lookahead, const int64_t* ids, int64_t n, const int64_t* offsets,
                 int64_t num_bags, int32_t* slots, bool write_slots, IndexRun* run, bool mark_emitted) {
    const int64_t LIM = ((int64_t)1 << 31) - 65536;
    if (!c || n < 0 || num_bags < 0 || n >= LIM || num_bags >= LIM || !offsets || (n > 0 && (!ids || !slots)))
        return FC_ERR_INVALID_ARG;
    FC_HIP(hipSetDevice(c->device));
    // what can run out of memory comes before any state changes: list set, error word and evicted-row block in turn, rows in transit
    const bool small = !lookahead && prepare_small_fits(c, n, num_bags);
    FC_TRY(ensure_rbuf(c, n));
    const bool bytes = !small && mark_bytes(c);
    c->pst = st;
    // the list set this call rewrites (missing ranks, victims, fill slots) was last read by the row movement two
    // batches back, possibly on another stream
    use_list_set(c, c->lset ^ 1);
    c->have_lists = false;
    if (c->move_stream[c->lset] != no_stream() && c->move_stream[c->lset] != st) FC_HIP(hipStreamWaitEvent(st, c->ev_move_done[c->lset], 0));
    if (c->last_index_stream != no_stream() && c->last_index_stream != st)      // (what ran on `pre` ended with ev_pre_done)
        FC_HIP(hipStreamWaitEvent(st, c->last_index_stream == c->pre ? c->ev_pre_done : c->ev_index_done, 0));
    if (c->quiesce_stream != no_stream() && c->quiesce_stream != st) FC_HIP(hipStreamWaitEvent(st, c->ev_quiesce, 0));
    c->quiesce_stream = no_stream();
    const int32_t ticket = c->ticket = (c->ticket + 1) & 0x7fffffff;
    const int protect_prev = lookahead ? 1 : 0;
    int transit_base = -1, buf = 0;
    int64_t landed = 0;
    if (c->dma_evict) {
        // the block this call may fill was handed over DMA_BLOCKS blocks ago: its rows must be in the host table by now
        const uint64_t seq = pool_published(c) + 1;
        buf = (int)(seq % DMA_BLOCKS);
        if (seq > DMA_BLOCKS) pool_wait(c, seq - DMA_BLOCKS);
        landed = c->blk_rows[buf];            // cleared by k_rank_count below, before anything reads rank_slot or rewrites the list
        c->blk_rows[buf] = 0;
        if (!c->dirty_track) c->vrank = c->vrank_buf[buf];
        // after more victims than a block holds no block was handed over, so this is the list that movement reads
        if (c->vrank_kept && c->move_stream[c->lset ^ 1] != st) FC_HIP(hipStreamWaitEvent(st, c->ev_move_done[c->lset ^ 1], 0));
        transit_base = (int)(buf * c->staging_rows);
    }
    const bool small_slots = small && write_slots;
    const int transit = c->dirty_track ? -1 : transit_base;
    const int32_t* landed_ranks = c->dma_evict ? c->vrank_buf[buf] : nullptr;
    if (small) {
        if (c->evict_pending) {        // as below
            FC_HIP(hipStreamWaitEvent(st, c->ev_evict_done, 0));
            c->evict_pending = false;
        }
        FC_TRY(launch_prepare_small(c, st, ids, n, offsets, num_bags, small_slots ? slots : nullptr, ticket, landed_ranks, landed,
                                    buf * c->staging_rows, transit, run->drop_clean = drops_clean(c, st)));
    } else {
        const int64_t work = n > num_bags + 1 ? n : num_bags + 1;
        int64_t nmark;
        // two error words in turn: a call's K2a clears the next call's
        uint32_t *err = &c->ctl->err[c->err_set], *next_err = &c->ctl->err[c->err_set ^ 1];
        c->err_set ^= 1;
        const int groups = (int)cdiv(c->NB, GROUP_TILES);
        const int64_t dense_tiles = std::min(c->NB, cdiv(n * c->mark_dense, RT_WORDS * 32));
        if (bytes) {
            nmark = std::min<int64_t>(cdiv(work, MARK_ITEMS * MARK_THREADS), MARK_HIT_PARTS);
            ProfScope ps(c, P_REMAP_MARK, st);
            k_remap_mark<<<(unsigned)nmark, MARK_THREADS, 0, st>>>(ids, (int)n, offsets, (int)num_bags, c->freq_rank, c->N, c->ubytes, c->uchunks,
                                                                  (int)std::min(dense_tiles * RT_WORDS * 32, c->N), c->rbits, c->rbuf, err, c->hitpart, c->gsum, groups);
        } else {
            const int64_t per_block = cdiv(cdiv(work, std::min<int64_t>(cdiv(work, BITS_ITEMS * BITS_THREADS), BITS_MAX_BLOCKS)), BITS_THREADS) * BITS_THREADS;
            const int64_t words = c->NB * RT_WORDS;
            nmark = cdiv(work, per_block);
            k_zero_words<<<(unsigned)(words / 1024), 256, 0, st>>>((uint4*)c->ubits);
            ProfScope ps(c, P_REMAP_MARK, st);
            k_remap_bits<<<(unsigned)nmark, BITS_THREADS, 0, st>>>(ids, (int)n, offsets, (int)num_bags, c->freq_rank, c->N, c->ubits, c->rbits, c->rbuf, err,
                                                                  c->hitpart, (int)per_block, (int)std::min<int64_t>(words, BITS_LDS_WORDS), c->gsum, groups);
        }
        {
            ProfScope ps(c, P_RANK_COUNT, st);
#define FC_COUNT(B) \
            k_rank_count<B><<<(unsigned)c->NB, RT_THREADS, 0, st>>>((uint4*)c->ubytes, c->uchunks, (int)dense_tiles, (uint2*)c->ubits, (const uint2*)c->rbits, \
                                                                   (const uint2*)c->pbits, protect_prev, c->bsum, c->ssum, c->gsum, \
                                                                   landed_ranks, (int)landed, (int)(buf * c->staging_rows), c->rank_slot, next_err)
            if (bytes) FC_COUNT(true); else FC_COUNT(false);
#undef FC_COUNT
        }
        const PlanArgs pa{c->bsum, c->ssum, c->gsum, err, &c->ctl->async_flags, c->hitpart, c->hctl, c->plan[c->lset], (int)c->NB, (int)c->C, (int)c->nfree, (int)nmark, ticket,
                          protect_prev};
        // Last batch's evicted rows must have reached the host table before the victim lists and the block buffer
        // are reused and before any of those rows could be fetched again; the kernels above do not care.
        if (c->evict_pending) {
            FC_HIP(hipStreamWaitEvent(st, c->ev_evict_done, 0));
            c->evict_pending = false;
        }
        ProfScope ps(c, P_RANK_EMIT, st);
#define FC_EMIT(S) \
        k_rank_emit<S><<<(unsigned)(c->NB * S), RT_THREADS, 0, st>>>(c->ubits, c->rbits, c->pbits, pa, \
                                                                       c->miss_ranks, c->vrank, c->vslot, c->rank_slot, c->slot_rank, \
                                                                       transit, (int)c->staging_rows, \
                                                                       c->dma_evict ? c->fill_src : nullptr)
        if (c->NB <= c->split_tiles) FC_EMIT(EMIT_SPLIT); else FC_EMIT(1);
#undef FC_EMIT
    }
    const bool plain = st == c->stream;         // nothing on another stream waits for the events below, until a call says so
    if (!plain && mark_emitted) FC_HIP(hipEventRecord(c->ev_emit_done, st));
    FC_HIP(hipGetLastError());
    // whatever the decision is: the host hears of a refusal while workgroups of the emitting kernel still read the bitmap, the counts (of
    // tiles, groups and hits) and the error word, which the next batch's first kernels write
    if (plain) c->due |= DUE_INDEX; else c->due &= ~DUE_INDEX;
    c->last_index_stream = st;
    run->ticket = ticket; run->nfree = c->nfree; run->n = n; run->num_bags = num_bags;
    run->small = small; run->small_slots = small_slots; run->buf = buf; run->transit_base = transit_base;
    return FC_OK;
}

// j-th missing rank -> j-th empty slot.  M < 0: the host does not know yet how many there are.
int index_assign(fc_cache* c, hipStream_t st, const IndexRun& run, int64_t M, bool drop_clean) {
    if (M == 0 || run.small) return FC_OK;
    int32_t* old_rank = c->dma_evict && !drop_clean ? nullptr : c->fill_src;
    const unsigned tiles = (unsigned)cdiv(c->C, FREE_TILE);
    // From the list of victims while reading it costs each tile less than the kernel that it saves, and the host its launch (M < 0: as many as last
    // time, most likely).  us, counting and assigning / assigning from the list: 11 victims of 935 k slots 6.9 / 4.3, 2.3 k of 5.7 k 6.2 / 5.4, 5.5 k of 60 k
    // 6.8 / 7.3, 4 k of 6 M 16 / 10, 4 k of 20 M 73 / 29.
    // Every tile reads the whole list, so where the number is a guess what a wrong one could cost is bounded: 9 k victims of 935 k slots 9.5 / 9, 80 k of
    // 100 k (7.8 M words) 10 / 18, 170 k of 180 k (30 M) 10 / 36, and beyond the limit 150 k of 1.5 M (220 M) 11 / 57.
    const int64_t most = M < 0 ? std::min(run.n, c->C) : M;
    const bool list = run.nfree == 0 && (M < 0 ? c->last.n_miss : M) <= ASSIGN_LIST_MOST &&
                      (most <= 2 * ASSIGN_LIST_MOST || most * tiles <= ASSIGN_LIST_WORDS);
    if (!list) {
        ProfScope ps(c, P_FREE_COUNT, st);
        k_free_count<<<tiles, FREE_THREADS, 0, st>>>(c->slot_rank, (int)c->C, c->tcount);
    }
    ProfScope ps(c, P_FREE_PICK, st);
#define FC_ASSIGN(L) \
    k_free_assign<L><<<tiles, FREE_THREADS, 0, st>>>(c->slot_rank, (int)c->C, c->tcount, c->vslot, (int)M, c->miss_ranks, c->fill_slots, \
                                                     c->rank_slot, old_rank, M < 0 ? c->plan[c->lset] : nullptr, \
                                                     drop_clean ? c->dirty : nullptr, c->dirty_words, run.ticket)
    if (list) FC_ASSIGN(true); else FC_ASSIGN(false);
#undef FC_ASSIGN
    FC_HIP(hipGetLastError());
    return FC_OK;
}

// Wait for the decisions (status, counts) ...
static int wait_index(fc_cache* c, hipStream_t st, const IndexRun& run) {
    int32_t h[HOST_REC_WORDS];
    return wait_for_record(c->hctl, run.ticket, st, h);
}
// ... and take them over.
int index_result(fc_cache* c, hipStream_t st, const IndexRun& run, MovePlan* mv) {
    int32_t h[HOST_REC_WORDS];
    FC_TRY(wait_for_record(c->hctl, run.ticket, st, h));
    if (h[HW_STATUS] != FC_OK) return h[HW_STATUS];
    c->nfree = h[HW_NFREE];
    if (!run.small) std::swap(c->ubits, c->pbits);        // this batch is the "previous" one next time
    c->last_one_per_bag = run.n == run.num_bags && !(h[HW_BATCH_FLAGS] & (int32_t)EF_NOT_ONE_PER_BAG);
    const int64_t M = h[HW_MISS], need = h[HW_NEED];
    mv->valid = true; mv->M = M; mv->need = need; mv->buf = run.buf; mv->transit_base = run.transit_base;
    c->dirty_parts = 0;
    c->last.n_ids = run.n;
    c->last.n_unique = h[HW_UNIQUE];
    c->last.n_hit_unique = h[HW_UNIQUE] - M;
    c->last.n_hit_ids = h[HW_HITS];
    c->last.n_miss = M;
    c->last.n_evict = need;
    c->last.bytes_h2d = M * (int64_t)c->D * 4;
    c->last.bytes_d2h = need * (int64_t)c->D * 4;
    c->have_lists = true;
    return FC_OK;
}

// before_slots: an event the slot write-out (the first kernel that writes the caller's buffer) has to wait for.
// defer_slots: leave the slot write-out to the caller (who folds it into the sort).
int prepare_index(fc_cache* c, hipStream_t st, bool lookahead, const int64_t* ids, int64_t n, const int64_t* offsets,
                  int64_t num_bags, int32_t* slots, MovePlan* mv, hipEvent_t before_slots, bool defer_slots) {
    IndexRun run;
    const bool plain = st == c->stream;
    FC_TRY(index_launch(c, st, lookahead, ids, n, offsets, num_bags, slots, !defer_slots && !before_slots, &run));
    // (a larger batch's by now: the emitting kernel has reported, and the latest call's counts come before it)
    if (c->dirty_words && plain && !run.small) FC_TRY(wait_index(c, st, run));
    const bool drop_clean = run.small ? run.drop_clean : drops_clean(c, st);
    FC_TRY(index_result(c, st, run, mv));
    FC_TRY(index_assign(c, st, run, mv->M, drop_clean));
    if (drop_clean) {
        mv->clean_out = true;
        c->dirty_parts = mv->M == 0 ? 0 : run.small ? 1 : (int)cdiv(c->C, FREE_TILE);
        c->dirty_ticket = run.ticket;
    }
    if (!plain) { FC_HIP(hipEventRecord(c->ev_assign_done, st)); c->decided = c->ev_assign_done; }
    // every row of the batch has its slot now: write the slots out
    if (before_slots) FC_HIP(hipStreamWaitEvent(st, before_slots, 0));
    if (!defer_slots) {
        if (!run.small_slots) FC_TRY(launch_slots_out(c, st, slots, n));
    }
    c->aux = (st == c->pre && !lookahead) ? c->pre : c->pf;
    return FC_OK;
}

static int move_done(fc_cache* c, hipStream_t st, bool ahead) {
    if (st == c->stream && !ahead && !c->plans_ahead) c->due |= DUE_MOVE << c->lset;
    else {
        FC_HIP(hipEventRecord(c->ev_move_done[c->lset], st));
        c->due &= ~(DUE_MOVE << c->lset);
    }
    c->move_stream[c->lset] = st;
    return FC_OK;
}

// Row-movement half: evicted rows out (gather, then DMA block / kernel store / staged copy), missing rows in.
// ahead: the batch was prepared ahead of time, so the next one's index half will wait for this on a library stream.
// send_rows: the evicted block is not handed over here but by the caller (send_block), once it has enqueued what else it has; its rows.
// along: a sort to launch with the missing rows, where a kernel brings them over the link (SortJob::launched says so).
int prepare_move(fc_cache* c, hipStream_t st, const MovePlan& mv, bool ahead, int64_t* send_rows, SortJob* along) {
    c->pst = st;
    // the lists this half reads are complete once the last decision is taken; the slot write-out (and, folded into it,
    // the sort) is waited for by whoever hands the batch to the caller
    if (c->last_index_stream != st) FC_HIP(hipStreamWaitEvent(st, c->decided, 0));
    const int64_t M = mv.M;
    int64_t need = mv.need;                    // victims to write back
    const bool staged = (c->flags & FC_TRANSMIT_STAGED) != 0;
    c->out_rank = c->vrank; c->out_slot = c->vslot;
    if (c->dirty_track && !mv.clean_out && need > 0) {
        // keep the dirty victims only; their number decides the size of the copies below, so the host waits for it
        const bool dma_block = c->dma_evict && need <= c->staging_rows;
        int32_t* orank = dma_block ? c->vrank_buf[mv.buf] : c->lists[c->lset][5];
        int32_t* oslot = c->lists[c->lset][6];
        const unsigned tiles = (unsigned)cdiv(need, DIRTY_TILE);
        const int32_t ticket = c->dticket = (c->dticket + 1) & 0x7fffffff;
        k_dirty_count<<<tiles, DIRTY_THREADS, 0, st>>>(c->vslot, (int)need, (int)c->C, c->dirty, c->dcount);
        k_dirty_keep<<<tiles, DIRTY_THREADS, 0, st>>>(c->vrank, c->vslot, (int)need, (int)c->C, c->dirty, c->dcount, orank, oslot,
                                                     c->rank_slot, dma_block ? mv.transit_base : -1, c->dctl, ticket);
        FC_HIP(hipGetLastError());
        const volatile int32_t* dv = reinterpret_cast<const volatile int32_t*>(c->dctl);
        FC_TRY(wait_for_ticket(dv + 1, ticket, st));
        need = c->dirty_seen = dv[0];
        c->out_rank = orank; c->out_slot = oslot;
        c->last.bytes_d2h = need * (int64_t)c->D * 4;
    }
    if (staged && (M > 0 || need > 0)) {
        if (M > 0) FC_HIP(hipMemcpyAsync(c->list_pin, c->miss_ranks, (size_t)M * 4, hipMemcpyDeviceToHost, st));
        if (need > 0) FC_HIP(hipMemcpyAsync(c->list_pin + c->C, c->out_rank, (size_t)need * 4, hipMemcpyDeviceToHost, st));
        FC_HIP(hipStreamSynchronize(st));
    }
    // Default transmitter, rows straight from the host table: they change places with the victims in one kernel.
    if (mv.clean_out || (!staged && !c->dma_evict && !c->dirty_track && !mv.arrived)) {
        FC_TRY(launch_swap_rows(c, st, M, along));                        // every victim's slot is among those that are filled
        FC_TRY(move_done(c, st, ahead));
        c->pf_dep = c->ev_move_done[c->lset];
        return FC_OK;
    }
    int64_t last_off = 0, last_rows = 0;
    // Rows fetched ahead of time (cache_plan_next) were read from the host table and from evicted-row blocks other
    // than the one this batch's victims go to (its marks were dropped before this batch was indexed), so the
    // victims need not wait for them; a kernel-store evict reuses the block buffer from its start and has to.
    bool arrival_waited = !mv.arrived || c->arrived_by[c->lset] == c->decided;
    bool dma_path = false, send = false;
    // DMA miss path: ev_arrive of this list set is recorded by a gather thread once it has handed the last chunk to the
    // DMA engine; the host waits here until that has happened (the GPU meanwhile works through the current batch)
    const bool via_dma = mv.arrived && c->gather_pending;
    if (via_dma) { FC_TRY(gather_wait(c)); c->gather_pending = false; }
    if (need > 0) {
        if (staged) FC_TRY(evict_staged(c, need, c->list_pin + c->C));
        else if (c->dma_evict && mv.need <= c->staging_rows) { FC_TRY(gather_block(c, need, mv.buf, ahead)); dma_path = send = true; }
        else {
            // more victims than one block holds (or no DMA transmitter): store by kernel, block by block; the
            // block buffer is reused from its start, so nothing may be in transit in it any more: every missing row, also one
            // that was in transit when the batch was indexed, comes from the host table below
            if (!arrival_waited) { FC_HIP(hipStreamWaitEvent(st, c->arrived_by[c->lset], 0)); arrival_waited = true; }
            FC_TRY(dma_quiesce(c, st));
            FC_TRY(evict_direct(c, need, &last_off, &last_rows));
        }
    } else if (c->dma_evict) dma_path = true;
    if (M > 0) {
        if (last_rows > 0 && c->evict_early == 2) {       // store and fill share the link, then the link falls silent
            FC_TRY(store_block(c, last_off, last_rows));
            last_rows = -1;
        }
        if (!arrival_waited) FC_HIP(hipStreamWaitEvent(st, c->arrived_by[c->lset], 0));
        if (staged) FC_TRY(fill_staged(c, M, c->list_pin));
        else if (mv.arrived) {
            FC_TRY(launch_copy_rows(c, st, P_ROWS_IN, c->cache, c->fill_slots, c->C, c->arrive[c->lset], nullptr, c->staging_rows, M, 1 << 20));
            // DMA miss path: rows in transit did not come over the link; their newest copies are in evicted-row blocks
            // gathered by earlier batches (this stream has run those gathers)
            if (via_dma && c->dma_evict) FC_TRY(launch_fill_rows(c, st, M, nullptr, 0, 0, true));
        }
        else if (dma_path) FC_TRY(launch_fill_rows(c, st, M, nullptr, 0, 0, false, nullptr, along));
        else FC_TRY(launch_copy_rows(c, st, P_MISS_FILL, c->cache, c->fill_slots, c->C, c->host_dev, c->miss_ranks, c->N, M, c->fill_blocks));
    }
    if (last_rows > 0) FC_TRY(store_block(c, last_off, last_rows));
    if (last_rows < 0) { FC_HIP(hipStreamWaitEvent(st, c->ev_evict_done, 0)); c->evict_pending = false; }
    FC_HIP(hipGetLastError());
    FC_TRY(move_done(c, st, ahead));
    // (after the rows that come in: by then the gather may be through, and the side stream's wait for it costs the host next to nothing)
    if (send && send_rows) *send_rows = need;
    else if (send) FC_TRY(send_block(c, need, mv.buf, ahead));
    c->vrank_kept = c->dma_evict && !c->dirty_track && !dma_path;
    // The next early fetch reads evicted-row blocks gathered up to now and host rows stored up to now: with the DMA
    // transmitter the gather just enqueued is the last thing it needs (host rows still on their way carry transit
    // marks); after a kernel store it has to wait for the whole movement.
    if (!dma_path) c->pf_dep = c->ev_move_done[c->lset];
    else if (need > 0) c->pf_dep = c->ev_gather_done;
    return FC_OK;
}

int prepare_impl(fc_cache* c, hipStream_t st, bool lookahead, const int64_t* ids, int64_t n, const int64_t* offsets,
                 int64_t num_bags, int32_t* slots) {
    MovePlan mv;
    // the slot write-out is folded into the first kernel of the sort, unless the index kernel of a small batch has them in registers
    const bool beside = !lookahead && sorts_beside_rows(c, n);
    const bool fold = !lookahead && !beside && c->presort && n > 0 && num_bags > 0 && !prepare_small_fits(c, n, num_bags);
    FC_TRY(prepare_index(c, st, lookahead, ids, n, offsets, num_bags, slots, &mv, nullptr, fold));
    if (lookahead) {
        if (n > 0) (void)presort_impl(c, slots, n, offsets, num_bags);   // on failure the backward pass sorts (and reports) itself
        // Rows about to be evicted or overwritten may still be in use by work the caller enqueued before this call (the backward
        // pass of the batch before the current one); the index decisions did not care.
        FC_HIP(hipStreamWaitEvent(st, c->ev_s_now, 0));
        return prepare_move(c, st, mv, true);
    }
    // The rows first: while they cross the link the host gets ahead of the GPU.  A sort for one workgroup goes along with them, one on
    // another stream is under way before them.
    SortJob along;
    int64_t send_rows = 0;
    const bool before = n <= SMALL_SORT_IDS || beside;
    int rs = FC_OK;
    if (n > 0 && before) rs = presort_impl(c, slots, n, offsets, num_bags, fold ? slots : nullptr, &along);
    FC_TRY(prepare_move(c, st, mv, false, &send_rows, along.n > 0 ? &along : nullptr));
    if (n > 0 && !before) rs = presort_impl(c, slots, n, offsets, num_bags, fold ? slots : nullptr);
    if (along.n > 0 && !along.launched) {
        const int32_t *keys, *vals;
        rs = sort_small(along, st, &keys, &vals);
        if (rs != FC_OK) for (PresortRec& r : c->rec) r.valid = r.valid && r.ticket != c->ticket;
    }
    const int rw = fold && rs != FC_OK ? launch_slots_out(c, st, slots, n) : FC_OK;
    if (send_rows > 0) FC_TRY(send_block(c, send_rows, mv.buf, false));      // whatever else failed: its rows are marked as in transit
    FC_TRY(rw);
    if (c->plans_ahead) {              // the sort's first kernel reads what the next index half writes
        FC_HIP(hipEventRecord(c->ev_index_done, st));
        c->due &= ~DUE_INDEX;
    }
    return FC_OK;
}

}  // namespace fc
