// Small batches: the whole index half of cache_prepare (Algorithm 1) in one workgroup, and the (slot, bag) sort of the
// backward pass in another.
//
// A small batch is bound by the chain of launches, not by bytes: seven index kernels and three to nine sort kernels of 2-10 us
// each, with 4 us between them, for a few kilobytes of work.  One workgroup of 16 wavefronts keeps the batch's bitmap over
// rank space in LDS (160 KB per compute unit on gfx950), so that the phases are separated by workgroup barriers instead of
// kernel boundaries.  The decisions are those of the kernels in fc_prepare.hip and fc_sort.hip, element for element.
// Measured: 1024 ids, 100 k rows: index 33 us of kernels in 7 launches -> 13 us in one, sort 17 us in 3 -> 7.6 us in one, a
// training step 144 -> 118 us; 3328 ids, 1 M rows: 37 us in 7 -> 27 us in one, an inference step 101 -> 85 us (since then: below).
// The limit of 4096 ids: a single compute unit resolves about one random line per nanosecond and issues one instruction
// per cycle, and at 10 k ids it takes as long (40 + 32 us) as the kernels that use all of them (37 + 33 us and 11 launches,
// whose launching the host overlaps).  The limits on rows and slots are what fits LDS.
#include "rows_device.h"

#include <algorithm>

namespace fc {

constexpr int SM_THREADS = 1024;
constexpr int SM_WAVES = SM_THREADS / 64;
constexpr int SM_ITEMS = 8;                                       // slots of a thread in flight together
constexpr int SM_IDS = SMALL_MAX_IDS / SM_THREADS;                // ids of a thread
constexpr int SM_R8 = SMALL_MAX_WORDS / (SM_WAVES * 64 * 8);      // pairs of 16-byte pieces of the bitmap per lane, at most

struct SmallArgs {
    const int64_t* ids; const int64_t* offsets; const int32_t* freq_rank;
    uint4 *rbits4, *pbits4;
    int32_t *rank_slot, *slot_rank;
    int32_t *miss_ranks, *vrank, *vslot, *fill_slots, *fill_src;
    int32_t* ranks;                    // rank of every id
    int32_t* slots_out;                // slot of every id; null: left to the caller (folded into the sort)
    const int32_t* landed_ranks;       // see k_rank_count
    const Ctl* ctl; HostCtl* hctl; int32_t* plan;
    int64_t N;
    int n, num_bags, C, words, landed, landed_base, transit_base, transit_rows, ticket, nfree;
    bool dma;
    uint8_t* dirty; uint64_t* dirty_words;      // see k_free_assign; null: rows leave whether updated or not
};

// Words of a bitmap over one pair of 16-byte pieces (256 ranks).
__device__ __forceinline__ int popc8(uint4 a, uint4 b) {
    return __popc(a.x) + __popc(a.y) + __popc(a.z) + __popc(a.w) + __popc(b.x) + __popc(b.y) + __popc(b.z) + __popc(b.w);
}
__device__ __forceinline__ uint4 and_not(uint4 x, uint4 y) { return make_uint4(x.x & ~y.x, x.y & ~y.y, x.z & ~y.z, x.w & ~y.w); }
__device__ __forceinline__ bool differ(uint4 x, uint4 y) { return ((x.x ^ y.x) | (x.y ^ y.y) | (x.z ^ y.z) | (x.w ^ y.w)) != 0; }
// bits of the 32-rank word starting at rank `at` that lie below rank r
__device__ __forceinline__ uint32_t word_below(int at, int r) { return r <= at ? 0u : r >= at + 32 ? 0xFFFFFFFFu : (1u << (r - at)) - 1u; }
__device__ __forceinline__ uint4 below(uint4 v, int at, int r) {
    return make_uint4(v.x & word_below(at, r), v.y & word_below(at + 32, r), v.z & word_below(at + 64, r), v.w & word_below(at + 96, r));
}

// lanes of m before this one, and whether this one is among them
__device__ __forceinline__ int lanes_before(uint64_t m) { return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0)); }
__device__ __forceinline__ bool has_lane(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Dynamic LDS: rank bitmap [words], prefix counts [words / 8], slot masks [slot chunks], a queue [ids].
//
// Every decision that has an order (the j-th missing rank, the j-th victim, the j-th empty slot) is a prefix count: counts
// per 256 ranks are scanned once, and whoever meets an element (an id with a missing rank, a slot with a victim) works out
// its place from that and a popcount, all elements side by side; loops over the bits of a word, one lane each, took four
// times as long here.  The code is kept short: a workgroup that runs once fetches its instructions from memory, too.
// What bounds it is the chain of dependent reads, a microsecond each, so a thread keeps its ids' ranks and slots in registers, what
// other threads need goes through LDS wherever it fits, and what a later phase reads is requested before the phase in between.  1024 ids, 100 k rows, 1500 slots: 16.7 -> 10.9 us; 3328 ids,
// 1 M rows, 15 k slots: 31.4 -> 21.6 on one batch again and again, 24.0 in a serving loop (of the 21.6: init 2.6, ids to marks 3.6, prefix counts 1.9, threshold 0.7, missing 1.0, slots 3.9, victims and empty
// slots 2.4, slots out 1.1, bitmaps 2.4).  A unit runs 16 wavefronts on four SIMDs, so 100 instructions for all are 0.7 us.
__global__ __launch_bounds__(SM_THREADS) void k_prepare_small(SmallArgs a) {
    extern __shared__ __align__(16) uint32_t lds_bits[];
    __shared__ int part[SM_WAVES][2], before[SM_WAVES][2], holes[SM_WAVES];
    __shared__ uint32_t s_cand[8];
    __shared__ int s_hits, s_used, s_threshold, s_queue, s_queue2, s_dirty;
    __shared__ uint32_t s_flags;
    uint32_t* ub = lds_bits;                                                   // rows of this batch
    uint32_t* pre = ub + a.words;                                              // missing and (high half) evictable rows before
                                                                               // a pair of pieces, in its wavefront's stretch
    uint64_t* fmask = reinterpret_cast<uint64_t*>(pre + a.words / 8);          // slots to fill, 64 a word
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int per_wave = a.words / SM_WAVES / 8;                               // pairs of pieces per wavefront
    const int chunks_wave = (a.C + 64 * SM_WAVES - 1) / (64 * SM_WAVES);       // 64-slot chunks per wavefront, at most 64
    uint16_t* queue = reinterpret_cast<uint16_t*>(fmask + chunks_wave * SM_WAVES);
    const int nfree = a.nfree;
    // ids and offsets, and the resident bits this thread will look at
    int64_t id[SM_IDS], o0[SM_IDS], o1[SM_IDS];
#pragma unroll
    for (int k = 0; k < SM_IDS; ++k) {
        const int i = tid + k * SM_THREADS;
        id[k] = i < a.n ? a.ids[i] : 0;
        o0[k] = i <= a.num_bags ? a.offsets[i] : i;
        o1[k] = i < a.num_bags ? a.offsets[i + 1] : o0[k];
    }
    uint4 q0[SM_R8], q1[SM_R8];
#pragma unroll
    for (int k = 0; k < SM_R8; ++k) {
        const int p = w * per_wave + k * 64 + lane;
        const bool live = k * 64 + lane < per_wave;
        q0[k] = live ? a.rbits4[2 * p] : make_uint4(0, 0, 0, 0);
        q1[k] = live ? a.rbits4[2 * p + 1] : make_uint4(0, 0, 0, 0);
    }
    const uint32_t async_flags = a.ctl->async_flags;
    for (int j = tid; j < a.words / 4; j += SM_THREADS) reinterpret_cast<uint4*>(ub)[j] = make_uint4(0, 0, 0, 0);
    if (tid == 0) { s_hits = s_used = s_queue = s_queue2 = s_dirty = 0; s_flags = 0; s_threshold = 0x7fffffff; }
    // rows of the block that has reached the host table (fill_src below reads what this leaves; who else reads it meanwhile asks
    // only whether it is negative)
    for (int j = tid; j < a.landed; j += SM_THREADS) {
        const int r = a.landed_ranks[j];
        if (a.rank_slot[r] == -2 - (a.landed_base + j)) a.rank_slot[r] = -1;
    }
    __syncthreads();
    // ids -> ranks, marked in LDS; access-level hits; offsets
    uint32_t flags = 0;
    int r[SM_IDS], s[SM_IDS];
#pragma unroll
    for (int k = 0; k < SM_IDS; ++k) {
        const bool ok = (uint64_t)id[k] < (uint64_t)a.N;
        if (!ok) flags |= EF_ID_RANGE;
        r[k] = ok && tid + k * SM_THREADS < a.n ? a.freq_rank[id[k]] : -1;
    }
#pragma unroll
    for (int k = 0; k < SM_IDS; ++k) s[k] = r[k] >= 0 ? a.rank_slot[r[k]] : -1;
    int row[SM_ITEMS];                                     // rows of this lane's first slots
#pragma unroll
    for (int k = 0; k < SM_ITEMS; ++k) {
        const int slot = (w * chunks_wave + k) * 64 + lane;
        row[k] = k < chunks_wave && slot < a.C ? a.slot_rank[slot] : 0x7fffffff;
    }
#pragma unroll
    for (int k = 0; k < SM_IDS; ++k) {
        const int i = tid + k * SM_THREADS;
        if (i > a.num_bags) continue;
        if (o0[k] != i) flags |= EF_NOT_ONE_PER_BAG;
        if ((i == 0 && o0[k] != 0) || (i == a.num_bags && o0[k] != (int64_t)a.n) || o1[k] < o0[k]) flags |= EF_BAD_OFFSETS;
    }
#pragma unroll 1
    for (int i = tid + SM_IDS * SM_THREADS; i <= a.num_bags; i += SM_THREADS) {        // more bags than ids
        const int64_t o = a.offsets[i];
        if (o != i) flags |= EF_NOT_ONE_PER_BAG;
        if (i == a.num_bags && o != (int64_t)a.n) flags |= EF_BAD_OFFSETS;
        if (i < a.num_bags && a.offsets[i + 1] < o) flags |= EF_BAD_OFFSETS;
    }
    int hits = 0, used = 0;
    uint64_t missing[SM_IDS];                              // lanes whose id k is the first of its row, and the row is missing
    int misses = 0;
#pragma unroll
    for (int k = 0; k < SM_IDS; ++k) {
        bool first = false;
        if (r[k] >= 0) {
            const uint32_t bit = 1u << (r[k] & 31);
            uint32_t* word = &ub[(uint32_t)r[k] >> 5];
            // (popular rows: a plain read is one broadcast, atomics on one word queue up)
            first = !(*reinterpret_cast<volatile uint32_t*>(word) & bit) && !(atomicOr(word, bit) & bit);
            used += first;
            hits += s[k] >= 0;
        }
        missing[k] = __ballot(first && s[k] < 0);
        misses += __popcll(missing[k]);
        if (tid + k * SM_THREADS < a.n) a.ranks[tid + k * SM_THREADS] = r[k];
    }
    if (misses) {                                          // their positions in the batch are queued
        int at = 0;
        if (lane == 0) at = atomicAdd(&s_queue, misses);
        at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
        for (int k = 0; k < SM_IDS; ++k) {
            if (has_lane(missing[k])) queue[at + lanes_before(missing[k])] = (uint16_t)(tid + k * SM_THREADS);
            at += __popcll(missing[k]);
        }
    }
    hits = wave_sum(hits);
    used = wave_sum(used);
    if (lane == 0) { atomicAdd(&s_hits, hits); atomicAdd(&s_used, used); }
    if (flags) atomicOr(&s_flags, flags);
    __syncthreads();
    // missing and evictable rows before each pair of pieces
    const uint4* ub4 = reinterpret_cast<const uint4*>(ub);
    int cm = 0, cc = 0;
#pragma unroll
    for (int k = 0; k < SM_R8; ++k) {
        if (k * 64 >= per_wave) break;
        const bool live = k * 64 + lane < per_wave;
        const int p = w * per_wave + k * 64 + lane;
        int nm = 0, nc = 0;
        if (live) {
            const uint4 u0 = ub4[2 * p], u1 = ub4[2 * p + 1];
            nm = popc8(and_not(u0, q0[k]), and_not(u1, q1[k]));
            nc = popc8(and_not(q0[k], u0), and_not(q1[k], u1));
        }
        int x = wave_scan(nm | nc << 16);                  // 64 pairs hold 16384 ranks: no carry between the halves
        // (a stretch holds at most 65536 ranks, and what precedes a pair in it at most 65280: 16 bits each)
        if (live) pre[p] = (uint32_t)(cm + (x & 0xffff) - nm) | (uint32_t)(cc + (x >> 16) - nc) << 16;
        x = __builtin_amdgcn_readlane(x, 63);
        cm += x & 0xffff;
        cc += x >> 16;
    }
    if (lane == 0) { part[w][0] = cm; part[w][1] = cc; }
    __syncthreads();
    // totals, and what precedes this wavefront's stretch
    const int pm = lane < SM_WAVES ? part[lane][0] : 0, pc = lane < SM_WAVES ? part[lane][1] : 0;
    const int sm = wave_scan(pm), sc = wave_scan(pc);
    const int M = __builtin_amdgcn_readlane(sm, 63), totC = __builtin_amdgcn_readlane(sc, 63);
    const int c0 = __builtin_amdgcn_readlane(sc - pc, __builtin_amdgcn_readfirstlane(w));
    if (w == 0 && lane < SM_WAVES) { before[lane][0] = sm - pm; before[lane][1] = sc - pc; }
    const uint32_t ef = s_flags;
    const int totU = s_used;
    int status = FC_OK;
    if (ef & EF_BAD_OFFSETS) status = FC_ERR_BAD_OFFSETS;
    else if (ef & EF_ID_RANGE) status = FC_ERR_ID_OUT_OF_RANGE;
    else if (totU > a.C) status = FC_ERR_BATCH_EXCEEDS_CACHE;
    int need = M - nfree;
    if (need < 0 || status != FC_OK) need = 0;
    if (w == SM_WAVES - 1) {
        if (lane == 0) { a.plan[PL_STATUS] = status; a.plan[PL_NEED] = need; a.plan[PL_MISS] = M; }
        const int nf = status == FC_OK ? nfree + need - M : nfree;
        report_to_host(a.hctl, a.ticket, status, totU, M, need, s_hits, nf, (int)async_flags, (int)(ef & EF_NOT_ONE_PER_BAG), lane);
    }
    if (status != FC_OK) return;
    // the victims are the evictable ranks from the threshold up: the one with `skip` evictable ranks below it
    const int skip = totC - need;
    if (need > 0 && skip >= c0 && skip < c0 + cc) {        // it lies in this wavefront's stretch
#pragma unroll
        for (int k = 0; k < SM_R8; ++k) {
            if (k * 64 >= per_wave) break;
            const int p = w * per_wave + k * 64 + lane;
            if (k * 64 + lane < per_wave) {
                const uint4 e0 = and_not(q0[k], ub4[2 * p]), e1 = and_not(q1[k], ub4[2 * p + 1]);
                const int left = skip - c0 - (int)(pre[p] >> 16);
                if (left >= 0 && left < popc8(e0, e1)) {   // one lane of one wavefront
                    s_cand[0] = e0.x; s_cand[1] = e0.y; s_cand[2] = e0.z; s_cand[3] = e0.w;
                    s_cand[4] = e1.x; s_cand[5] = e1.y; s_cand[6] = e1.z; s_cand[7] = e1.w;
                    s_threshold = p << 9 | left;           // resolved below
                }
            }
        }
    }
    __syncthreads();
    int threshold = 0x7fffffff;
    if (need > 0) {                                        // every thread for itself
        int left = s_threshold & 511, j = 0;
        uint32_t m = s_cand[0];
        while (left >= __popc(m)) { left -= __popc(m); m = s_cand[++j]; }      // ends: fewer than the pair's count
        const bool here = lane < 32 && ((m >> lane) & 1u) && __popc(m & ((1u << lane) - 1u)) == left;
        threshold = (s_threshold >> 9) * 256 + j * 32 + __ffsll((unsigned long long)__ballot(here)) - 1;
    }
    // each missing rank goes to its place
#pragma unroll 1
    for (int q = tid; q < M; q += SM_THREADS) {
        const int rank = a.ranks[queue[q]], p = rank >> 8;
        const uint4 b0 = below(and_not(ub4[2 * p], a.rbits4[2 * p]), p * 256, rank),
                    b1 = below(and_not(ub4[2 * p + 1], a.rbits4[2 * p + 1]), p * 256 + 128, rank);
        a.miss_ranks[before[p / per_wave][0] + (int)(pre[p] & 0xffff) + popc8(b0, b1)] = rank;
    }
    __syncthreads();
    // slots whose row is a victim, and those that were empty, are the ones to fill
    int cf = 0;
    if (M > 0) {
#pragma unroll 1
        for (int k0 = 0; k0 < chunks_wave; k0 += SM_ITEMS) {
            int next[SM_ITEMS];
#pragma unroll
            for (int k = 0; k < SM_ITEMS; ++k) {
                const int c = k0 + SM_ITEMS + k, slot = (w * chunks_wave + c) * 64 + lane;
                next[k] = c < chunks_wave && slot < a.C ? a.slot_rank[slot] : 0x7fffffff;
            }
            uint64_t vm[SM_ITEMS];
            int victims = 0;
#pragma unroll
            for (int k = 0; k < SM_ITEMS; ++k) {
                const int x = row[k];
                if (k0 + k >= chunks_wave) { vm[k] = 0; continue; }
                const bool victim = (unsigned)x - (unsigned)threshold < 0x7fffffffu - (unsigned)threshold &&       // neither empty nor past the last slot
                                    !((ub[x >> 5] >> (x & 31)) & 1u);
                vm[k] = __ballot(victim);
                victims += __popcll(vm[k]);
                const uint64_t m = vm[k] | __ballot(x < 0);
                if (lane == 0) fmask[w * chunks_wave + k0 + k] = m;
                cf += __popcll(m);
            }
            if (victims) {
                int at = 0;
                if (lane == 0) at = atomicAdd(&s_queue2, victims);
                at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
                for (int k = 0; k < SM_ITEMS; ++k) {
                    if (has_lane(vm[k])) queue[at + lanes_before(vm[k])] = (uint16_t)((w * chunks_wave + k0 + k) * 64 + lane);
                    at += __popcll(vm[k]);
                }
            }
#pragma unroll
            for (int k = 0; k < SM_ITEMS; ++k) row[k] = next[k];
        }
    }
    if (lane == 0) holes[w] = cf;
    __syncthreads();
    const bool transit = a.transit_base >= 0 && need <= a.transit_rows;
#pragma unroll 1
    for (int q = tid; q < need; q += SM_THREADS) {         // each victim goes to its place
        const int slot = queue[q], rank = a.slot_rank[slot], p = rank >> 8;
        const uint4 b0 = below(and_not(a.rbits4[2 * p], ub4[2 * p]), p * 256, rank),
                    b1 = below(and_not(a.rbits4[2 * p + 1], ub4[2 * p + 1]), p * 256 + 128, rank);
        const int j = before[p / per_wave][1] + (int)(pre[p] >> 16) + popc8(b0, b1) - skip;
        a.vrank[j] = rank;
        a.vslot[j] = slot;
        a.rank_slot[rank] = transit ? -2 - (a.transit_base + j) : -1;
    }
    // the j-th lowest empty slot is the j-th missing rank's
    {
        const uint64_t m = lane < chunks_wave && M > 0 ? fmask[w * chunks_wave + lane] : 0;
        int j0 = wave_sum(lane < w ? holes[lane] : 0);     // (w < 16)
#pragma unroll 1
        for (int k = 0; k < chunks_wave && j0 < M; ++k) {
            const uint64_t mk = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(m >> 32), k) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)m, k);
            const int j = j0 + lanes_before(mk);
            if (has_lane(mk) && j < M) a.fill_slots[j] = (w * chunks_wave + k) * 64 + lane;
            j0 += __popcll(mk);
        }
    }
    __syncthreads();
#pragma unroll 1
    for (int j = tid; j < M; j += SM_THREADS) {
        const int slot = a.fill_slots[j], rank = a.miss_ranks[j];
        // FC_EVICT_DMA: where the row's newest copy is (-1 the host table, <= -2 in transit); else the row that leaves the slot
        int src = a.dma && !a.dirty ? a.rank_slot[rank] : a.slot_rank[slot];
        if (a.dirty && src >= 0) {
            if (a.dirty[slot]) { a.dirty[slot] = 0; atomicAdd(&s_dirty, 1); }
            else src = -1;
        }
        a.fill_src[j] = src;
        a.slot_rank[slot] = rank;
        a.rank_slot[rank] = slot;
    }
    if (a.dirty) {
        __syncthreads();
        if (tid == 0) post_count(a.dirty_words, s_dirty, a.ticket);
    }
    if (a.slots_out) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < SM_IDS; ++k) if (s[k] < 0 && r[k] >= 0) s[k] = a.rank_slot[r[k]];
#pragma unroll
        for (int k = 0; k < SM_IDS; ++k) if (tid + k * SM_THREADS < a.n) a.slots_out[tid + k * SM_THREADS] = s[k];
    }
    // the bitmaps change hands: resident = without the victims, with the missing; previous batch = this one
#pragma unroll
    for (int k = 0; k < SM_R8; ++k) {
        if (k * 64 >= per_wave) break;
        const int p = w * per_wave + k * 64 + lane, at = p * 256;
        if (k * 64 + lane < per_wave) {
            const uint4 u0 = ub4[2 * p], u1 = ub4[2 * p + 1];
            uint4 k0 = and_not(q0[k], u0), k1 = and_not(q1[k], u1);            // evictable: stay if below the threshold
            if (at >= threshold) k0 = k1 = make_uint4(0, 0, 0, 0);
            else if (at + 256 > threshold) { k0 = below(k0, at, threshold); k1 = below(k1, at + 128, threshold); }
            const uint4 r0 = make_uint4(u0.x | k0.x, u0.y | k0.y, u0.z | k0.z, u0.w | k0.w),
                        r1 = make_uint4(u1.x | k1.x, u1.y | k1.y, u1.z | k1.z, u1.w | k1.w);
            if (differ(r0, q0[k]) || differ(r1, q1[k])) { a.rbits4[2 * p] = r0; a.rbits4[2 * p + 1] = r1; }
            a.pbits4[2 * p] = u0;
            a.pbits4[2 * p + 1] = u1;
        }
    }
}

static size_t prepare_small_lds(const fc_cache* c, int64_t n) {
    const size_t words = (size_t)c->NB * RT_WORDS;
    return (words + words / 8) * 4 + (size_t)cdiv(c->C, 64 * SM_WAVES) * SM_WAVES * 8 + (size_t)cdiv(n, 8) * 16;
}

bool prepare_small_fits(const fc_cache* c, int64_t n, int64_t num_bags) {
    return c->small_index && n <= SMALL_MAX_IDS && num_bags <= 4 * SMALL_MAX_IDS && c->NB * RT_WORDS <= SMALL_MAX_WORDS && c->C <= SMALL_MAX_SLOTS &&
           prepare_small_lds(c, n) <= SMALL_MAX_LDS;
}

int launch_prepare_small(fc_cache* c, hipStream_t st, const int64_t* ids, int64_t n, const int64_t* offsets, int64_t num_bags,
                         int32_t* slots, int32_t ticket, const int32_t* landed_ranks, int64_t landed, int64_t landed_base,
                         int transit_base, bool drop_clean) {
    SmallArgs a;
    a.ids = ids; a.offsets = offsets; a.freq_rank = c->freq_rank;
    a.rbits4 = (uint4*)c->rbits; a.pbits4 = (uint4*)c->pbits;
    a.rank_slot = c->rank_slot; a.slot_rank = c->slot_rank;
    a.miss_ranks = c->miss_ranks; a.vrank = c->vrank; a.vslot = c->vslot; a.fill_slots = c->fill_slots;
    a.fill_src = c->fill_src; a.dma = c->dma_evict; a.nfree = (int)c->nfree;
    a.ranks = c->rbuf; a.slots_out = slots;
    a.landed_ranks = landed_ranks; a.landed = (int)landed; a.landed_base = (int)landed_base;
    a.ctl = c->ctl; a.hctl = c->hctl; a.plan = c->plan[c->lset]; a.N = c->N;
    a.n = (int)n; a.num_bags = (int)num_bags; a.C = (int)c->C; a.words = (int)(c->NB * RT_WORDS);
    a.dirty = drop_clean ? c->dirty : nullptr; a.dirty_words = c->dirty_words;
    a.transit_base = transit_base; a.transit_rows = (int)c->staging_rows; a.ticket = ticket;
    const size_t lds = prepare_small_lds(c, n);
    ProfScope ps(c, P_REMAP_MARK, st);
    k_prepare_small<<<1, SM_THREADS, lds, st>>>(a);
    FC_HIP(hipGetLastError());
    return FC_OK;
}

// ---------------------------------------------------------------------------------------------------------
// Stable sort of up to SMALL_SORT_IDS (slot, bag) pairs by slot in one workgroup: LSD passes of at most 8 bits on words that
// hold key and lookup number together (see pos_bits), exchanged
// through LDS; the lookup number becomes its bag at the end.
// Against the kernels of fc_sort.hip (us, rows of 64 columns; those kernels / this).  Beside the missing rows (k_rows_and_sort), a training step, plain: 15 k slots
// (two passes) 3 k lookups 59 / 45, 7 k 76 / 58, 10.1 k 86 / 67, 13.3 k 99 / 79; 200 k slots (three) 3 k 59 / 50, 7 k 65 / 61, 8.5 k 67 / 66, 10.1 k 69 / 70,
// 13.3 k 73 / 79: the limit is where the two meet with three passes.  Planned ahead: 15 k slots 5.2 k 82-104 / 73-91, 10.1 k 85-114 / 83-84, 13.3 k 104-119 / 95; 200 k slots 5.2 k
// 93-97 / 73-87, 10.1 k 98-101 / 77-83, 13.3 k 101-105 / 81-87.  A sort inside the backward call, that call alone: 15 k slots 3 k 26 / 19,
// 7 k 27 / 24.6, 8.5 k 27.4 / 27, 10.1 k 27.7 / 28.6, 13.3 k 29 / 33; 200 k slots 3 k 27 / 21, 5.2 k 27.4 / 26.9, 7 k 28 / 29.5, 10.1 k 28.4 / 35.3, so that between
// 9 k lookups (two passes) or 5.5 k (three) and the limit, which is the same for all, a backward call that sorts takes up to 7 us more than it could.
// ---------------------------------------------------------------------------------------------------------
struct SmallSort {
    const int32_t *keys_in, *rank_slot; int32_t* slots_out; const int64_t* offsets; const int32_t* status; uint32_t* flags;
    int32_t *keys_out, *vals_out;
    int num_bags, one_per_bag, n, limit, passes, radix_bits, pos_bits;
};

__device__ __forceinline__ void sort_in_workgroup(const SmallSort& a) {
    const int32_t* __restrict__ keys_in = a.keys_in;
    const int32_t* __restrict__ rank_slot = a.rank_slot;
    const int64_t* __restrict__ offsets = a.offsets;
    int32_t* __restrict__ slots_out = a.slots_out;
    int32_t* __restrict__ keys_out = a.keys_out;
    int32_t* __restrict__ vals_out = a.vals_out;
    const int num_bags = a.num_bags, one_per_bag = a.one_per_bag, n = a.n, limit = a.limit, passes = a.passes, radix_bits = a.radix_bits, pos_bits = a.pos_bits;
    // two arrays of rounds * SM_THREADS words, the digit counts, and each element's place within its wavefront and digit
    extern __shared__ __align__(16) uint32_t sm_words[];
    const int rounds = (n + SM_THREADS - 1) / SM_THREADS;  // elements per thread
    const int radix = 1 << radix_bits, mask = radix - 1;
    uint32_t* from = sm_words;
    uint32_t* to = sm_words + rounds * SM_THREADS;
    int* wc = reinterpret_cast<int*>(sm_words + 2 * rounds * SM_THREADS);      // [SM_WAVES][radix]
    uint16_t* place = reinterpret_cast<uint16_t*>(wc + SM_WAVES * radix);
    __shared__ int scan[SM_WAVES];
    __shared__ int s_other;                                // some bag does not hold just its own lookup
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    bool bad = false, other = false;
    const bool refused = a.status && *a.status != FC_OK;       // neither slots nor offsets are touched then
    // with as many lookups as bags, most likely bag i holds lookup i: seen here, in order, rather than looked up in sorted order below
    const bool check = !one_per_bag && !refused && n == num_bags;
    if (tid == 0) s_other = check ? offsets[n] != (int64_t)n : !one_per_bag;
    constexpr int BATCH = 5;                               // elements of a thread in flight together
#pragma unroll 1
    for (int i0 = tid; i0 - tid < n; i0 += BATCH * SM_THREADS) {
        int key[BATCH];
        int64_t off[BATCH];
#pragma unroll
        for (int k = 0; k < BATCH; ++k) key[k] = keys_in[min(i0 + k * SM_THREADS, n - 1)];
#pragma unroll
        for (int k = 0; k < BATCH; ++k) off[k] = check ? offsets[min(i0 + k * SM_THREADS, n - 1)] : 0;
        if (rank_slot) {
#pragma unroll
            for (int k = 0; k < BATCH; ++k) key[k] = key[k] >= 0 ? rank_slot[key[k]] : -1;     // (-1: an id out of range, the call is refused)
        }
#pragma unroll
        for (int k = 0; k < BATCH; ++k) {
            const int i = i0 + k * SM_THREADS;
            if (i >= n) break;
            if (rank_slot && !refused) slots_out[i] = key[k];
            if ((unsigned)key[k] >= (unsigned)limit) { bad = true; key[k] = limit; }
            other |= check && off[k] != i;
            from[i] = ((uint32_t)key[k] << pos_bits) | (uint32_t)i;
        }
    }
    if (refused) return;
    if (bad && a.flags) atomicOr(a.flags, EF_BAD_SLOT);
    const uint64_t lt = (1ull << lane) - 1ull;
    const int e0 = w * 64 * rounds + lane;                 // this wavefront's elements: e0 + 64 * k
    int* mine = wc + w * radix;
#pragma unroll 1
    for (int p = 0; p < passes; ++p) {
        const int shift = pos_bits + p * radix_bits;
        for (int d = tid; d < SM_WAVES * radix; d += SM_THREADS) wc[d] = 0;
        __syncthreads();
        if (p == 0 && other) s_other = 1;
#pragma unroll 1
        for (int k = 0; k < rounds; ++k) {
            const int e = e0 + 64 * k;
            const bool valid = e < n;
            const int d = ((valid ? from[e] : 0) >> shift) & mask;
            const uint64_t peers = same_digit<8>(d, radix_bits, __ballot(valid));
            const int before = __popcll(peers & lt);
            if (valid) {
                const int at = mine[d];
                if (before == 0) mine[d] = at + __popcll(peers);
                place[e] = (uint16_t)(at + before);
            }
        }
        __syncthreads();
        // wc[w][d] becomes where wavefront w's first element of digit d goes
        int run = 0;
        if (tid < radix) {
#pragma unroll
            for (int k = 0; k < SM_WAVES; ++k) { const int c = wc[k * radix + tid]; wc[k * radix + tid] = run; run += c; }
        }
        int tot;
        const int base = block_excl_scan<SM_THREADS>(run, tot, scan);
        if (tid < radix) {
#pragma unroll
            for (int k = 0; k < SM_WAVES; ++k) wc[k * radix + tid] += base;
        }
        __syncthreads();
#pragma unroll 2
        for (int k = 0; k < rounds; ++k) {
            const int e = e0 + 64 * k;
            if (e < n) {
                const uint32_t x = from[e];
                to[mine[(x >> shift) & mask] + place[e]] = x;
            }
        }
        __syncthreads();
        uint32_t* t = from; from = to; to = t;
    }
    const bool opb = s_other == 0;
#pragma unroll 4
    for (int e = tid; e < n; e += SM_THREADS) {
        const uint32_t x = from[e];
        const int i = (int)(x & ((1u << pos_bits) - 1));
        keys_out[e] = (int)(x >> pos_bits);
        vals_out[e] = opb ? i : bag_of_lookup(offsets, num_bags, i);
    }
}

__global__ __launch_bounds__(SM_THREADS) void k_sort_small(SmallSort a) { sort_in_workgroup(a); }

// The sort in the first workgroup, rows on their way in the others: neither needs the other, the sort keeps one compute unit busy and the
// rows the link.  (Every workgroup is given the sort's LDS, beyond some 7000 lookups more than half of a compute unit's; the rows take 64 workgroups at most.)
// us a step, one launch after the other / this: 1024 lookups of 16 columns 36.5 / 32.5, 1157 of 128 columns 41.8 / 35.5, 163 of 226 columns 59 / 54.
template <int VEC, bool SWAP>
__global__ __launch_bounds__(SM_THREADS) void k_rows_and_sort(RowArgs r, SmallSort a) {
    if (blockIdx.x == 0) sort_in_workgroup(a);
    else if (SWAP) swap_rows<VEC>(r, blockIdx.x - 1, gridDim.x - 1);
    else fill_rows<VEC>(r, blockIdx.x - 1, gridDim.x - 1);
}

// A word holds key and lookup number: 18 bits of key at the limit of 10240 lookups, 20 at 4096, 22 at 1024.  (At a fixed split of 18 and 14, a small
// batch with 2^18 or more slots took the general sort, six launches: us a step, 1444 lookups of 32 columns, 935 k slots 58 / 47.)
static int pos_bits(int n) {
    int b = 0;
    while ((1 << b) < n) ++b;
    return b;
}

bool sort_small_fits(const SortJob& j) {
    return (j.src == SORT_SRC_SLOTS || j.src == SORT_SRC_RANKS) && j.n <= SMALL_SORT_IDS && j.bits + pos_bits(j.n) <= 32 && !j.max_bits && !j.no_fuse;
}

static SmallSort small_sort(const SortJob& j, size_t* lds) {
    const int passes = (j.bits + 7) / 8, rb = (j.bits + passes - 1) / passes;
    *lds = 4 * (2 * (size_t)cdiv(j.n, SM_THREADS) * SM_THREADS + ((size_t)SM_WAVES << rb) + (size_t)cdiv(j.n, 2));
    return SmallSort{j.keys_in, j.src == SORT_SRC_RANKS ? j.rank_slot : nullptr, j.slots_out, j.offsets, j.status, j.flags, j.keysA, j.valsA,
                     j.num_bags, j.one_per_bag && j.n == j.num_bags, j.n, j.limit, passes, rb, pos_bits(j.n)};
}

int sort_small(const SortJob& j, hipStream_t st, const int32_t** kres, const int32_t** vres) {
    ProfScope ps(j.prof, P_SORT_SCATTER, st);
    size_t lds;
    const SmallSort a = small_sort(j, &lds);
    k_sort_small<<<1, SM_THREADS, lds, st>>>(a);
    FC_HIP(hipGetLastError());
    *kres = j.keysA; *vres = j.valsA;
    if (j.last_stream) *j.last_stream = st;
    return FC_OK;
}

int launch_rows_and_sort(fc_cache* c, hipStream_t st, bool swap, const RowArgs& r, int max_blocks, SortJob* j) {
    size_t lds;
    const SmallSort a = small_sort(*j, &lds);
    // (blocks are counted in workgroups of 256 elsewhere)
    const unsigned blocks = 1 + (unsigned)std::min<int64_t>(cdiv(r.rows, SM_THREADS >> r.lpr_shift), cdiv(max_blocks, SM_THREADS / 256));
    ProfScope ps(c, P_MISS_FILL, st);
#define FC_BOTH(V) \
    if (swap) k_rows_and_sort<V, true><<<blocks, SM_THREADS, lds, st>>>(r, a); else k_rows_and_sort<V, false><<<blocks, SM_THREADS, lds, st>>>(r, a)
    switch (c->vec) { case 4: FC_BOTH(4); break; case 2: FC_BOTH(2); break; default: FC_BOTH(1); break; }
#undef FC_BOTH
    FC_HIP(hipGetLastError());
    j->launched = true;
    return FC_OK;
}

}  // namespace fc
