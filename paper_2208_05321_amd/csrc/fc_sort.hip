// Stable LSD radix sort of (key, value) int32 pairs, 64-wide wavefronts, tiles of RS_TILE keys per workgroup.
// With SortJob::status the first pass of a refused batch does nothing; the later ones then order whatever the scratch holds (a
// pass is in bounds for any keys, and by the time those on the side stream run, the word may belong to a later batch).
// Used by the backward pass and the slot-order forward (sort lookups by slot, value = bag) and by the static-module
// build (sort ids by descending count).  Keys come from one of four sources, see SortSrc.  A pass is either
// count -> scan -> scatter (up to RS_MAX_BITS bits per digit) or, for batch-sized jobs, count -> scatter: the scatter kernel adds the
// tiles' counts up itself, beyond SS_TILES tiles with the help of per-supertile sums (see radix_sort for which is chosen when).
#include "fc_internal.h"

#include <stdlib.h>

namespace fc {

// Jobs of up to FUSE_MAX_TILES tiles run without a scan kernel: beyond SS_TILES tiles k_sort_hist also adds the counts of SS_TILES neighbouring
// tiles up, and k_sort_scatter derives its offsets from those sums (digits of at most FUSE_MAX_BITS bits).
constexpr int SS_TILES = 32, FUSE_MAX_TILES = 2048, FUSE_MAX_BITS = 9;

// First-pass key of lookup i: its slot, or the sentinel C if the slot is out of range.
__device__ __forceinline__ int first_key(const int32_t* __restrict__ slots, int i, int C, bool& bad) {
    const int k = slots[i];
    if ((unsigned)k >= (unsigned)C) { bad = true; return C; }
    return k;
}

// key of element i by source (SORT_SRC_RANKS is turned into slots by k_sort_hist first)
template <int SRC>
__device__ __forceinline__ int load_key(const int32_t* __restrict__ keys_in, int i, int limit, bool& bad) {
    if (SRC == SORT_SRC_SLOTS) return first_key(keys_in, i, limit, bad);
    if (SRC == SORT_SRC_COUNTS) return limit - keys_in[i];      // limit = largest count: descending counts ascend
    return keys_in[i];
}

// ALIKE: most keys of a tile have the same digit (occurrence counts: most ids never occur, and the upper digits are alike).  Atomics on one
// LDS counter queue up, so the lanes that share the first lane's digit are added up first (10 M keys: 37 -> 10 us).
template <int SRC, bool ALIKE>
__global__ __launch_bounds__(RS_THREADS) void k_sort_hist(const int32_t* __restrict__ keys_in, int n, int limit, int shift,
                                                          int radix_bits, int nblk, int32_t* __restrict__ ghist,
                                                          int32_t* __restrict__ stot,
                                                          uint32_t* flags, const int32_t* __restrict__ rank_slot,
                                                          int32_t* __restrict__ slots_out,
                                                          int32_t* __restrict__ zero_ptr, int zero_words,
                                                          const int32_t* __restrict__ status) {
    constexpr int ITEMS = RS_ITEMS;
    __shared__ int h[1 << RS_MAX_BITS];
    if (zero_ptr) {     // what the previous sort left in the other set of supertile tables, a slice per workgroup
        const int per = (zero_words + (int)gridDim.x - 1) / (int)gridDim.x;
        const int z1 = min(zero_words, ((int)blockIdx.x + 1) * per);
        for (int i = (int)blockIdx.x * per + (int)threadIdx.x; i < z1; i += RS_THREADS) zero_ptr[i] = 0;
    }
    const int radix = 1 << radix_bits, mask = radix - 1;
    const int tile0 = blockIdx.x * (RS_THREADS * ITEMS);
    // all of the tile's keys are requested before anything waits for one (a lane beyond n rereads the last key)
    int key[ITEMS];
    bool bad = false;
    if (SRC == SORT_SRC_RANKS) {
        // gpu_row_idx of every input id (Algorithm 1's last index_select), written out on the way to becoming sort keys
        int r[ITEMS];
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) r[it] = keys_in[min(tile0 + it * RS_THREADS + (int)threadIdx.x, n - 1)];
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) key[it] = r[it] >= 0 ? rank_slot[r[it]] : -1;     // (-1: an id out of range, the call is refused)
        if (status && *status != FC_OK) return;    // refused: the caller's buffer is his own again
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int i = tile0 + it * RS_THREADS + (int)threadIdx.x;
            if (i < n) slots_out[i] = key[it];
            if ((unsigned)key[it] >= (unsigned)limit) { bad = true; key[it] = limit; }
        }
    } else
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
        key[it] = load_key<SRC>(keys_in, min(tile0 + it * RS_THREADS + (int)threadIdx.x, n - 1), limit, bad);
    for (int d = threadIdx.x; d < radix; d += RS_THREADS) h[d] = 0;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const bool valid = tile0 + it * RS_THREADS + (int)threadIdx.x < n;
        const int d = (key[it] >> shift) & mask;
        if (ALIKE) {
            const int d0 = __builtin_amdgcn_readfirstlane(d);
            const int same = __popcll(__ballot(valid && d == d0));
            if (valid && d != d0) atomicAdd(&h[d], 1);
            if ((threadIdx.x & 63) == 0) atomicAdd(&h[d0], same);
        } else if (valid) atomicAdd(&h[d], 1);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < radix; d += RS_THREADS) {
        const int cnt = h[d];
        ghist[(size_t)blockIdx.x * radix + d] = cnt;   // tile-major: one contiguous run per tile
        // counts of SS_TILES neighbouring tiles added up (the table starts at zero): the scatter kernel builds its
        // offsets from these and from the counts of the few tiles before it, and no scan kernel runs in between
        if (stot && cnt) atomicAdd(&stot[(size_t)(blockIdx.x / SS_TILES) * radix + d], cnt);
    }
    if (bad && flags) atomicOr(flags, EF_BAD_SLOT);
}

// Exclusive scan, per digit, of the per-tile counts over the tiles, in place; the digit totals go to dtot.
// The table is tile-major (ghist[tile * radix + digit]): a tile writes its counts, and reads its offsets back, as one
// contiguous run (digit-major, every one of those accesses touched a sector of its own: at 2048 digits x 832 tiles the
// two kernels around this one moved ten times the table).  Here a workgroup takes SC_DIG neighbouring digits, so that
// its reads and writes of one tile's entries are a contiguous 64 bytes, and SC_GROUPS ranges of tiles side by side:
// sums per range first, then each range again with its starting value.
constexpr int SC_DIG = 16, SC_GROUPS = 32, SC_PF = 8;
__global__ __launch_bounds__(SC_DIG * SC_GROUPS) void k_sort_scan(int32_t* ghist, int nblk, int radix, int32_t* __restrict__ dtot) {
    __shared__ int part[SC_GROUPS][SC_DIG];
    const int dl = threadIdx.x % SC_DIG, q = threadIdx.x / SC_DIG;
    const int d = blockIdx.x * SC_DIG + dl;
    const bool live = d < radix;
    const int per = (nblk + SC_GROUPS - 1) / SC_GROUPS;
    const int t0 = q * per, t1 = min(nblk, t0 + per);
    int sum = 0;
    if (live) {
        for (int t = t0; t < t1; t += SC_PF) {
            int v[SC_PF];
#pragma unroll
            for (int k = 0; k < SC_PF; ++k) v[k] = t + k < t1 ? ghist[(size_t)(t + k) * radix + d] : 0;
#pragma unroll
            for (int k = 0; k < SC_PF; ++k) sum += v[k];
        }
    }
    part[q][dl] = sum;
    __syncthreads();
    int run = 0, tot = 0;
#pragma unroll
    for (int g = 0; g < SC_GROUPS; ++g) {
        const int s = part[g][dl];
        if (g < q) run += s;
        tot += s;
    }
    if (live) {
        for (int t = t0; t < t1; t += SC_PF) {
            int v[SC_PF];
#pragma unroll
            for (int k = 0; k < SC_PF; ++k) v[k] = t + k < t1 ? ghist[(size_t)(t + k) * radix + d] : 0;
#pragma unroll
            for (int k = 0; k < SC_PF; ++k) {
                if (t + k < t1) ghist[(size_t)(t + k) * radix + d] = run;
                run += v[k];
            }
        }
        if (q == 0) dtot[d] = tot;
    }
}

// FUSED: `dtot` holds the per-supertile digit counts written by k_sort_hist instead of the digit totals, and `ghist` the
// raw per-tile counts (no scan kernel has run).  OPB (SORT_SRC_SLOTS only): bag b holds exactly lookup b, as checked by
// the caller, so the value of lookup i is i and the offsets are not read.
// MAXB = 9: digits of at most 9 bits; the tile is put in order in LDS first and then written run by run, so that neighbouring
// lanes write neighbouring words (straight from the registers, every lane of a store touched a line of its own, and the
// requests to L2 alone took 9 us at 1.7 M pairs).  MAXB = 11 (the static module's long jobs, experiments): runs of one or two
// keys, nothing to gain, and no LDS to spare.
// A batch has one tile for a compute unit or a few, so a tile's time is that of its wavefronts' instruction chains, not of its
// bytes: NT = 512 threads of four pairs each rather than 256 of eight, a digit to a thread, addresses of the count rows by a
// shift, matches of a digit in four instructions a bit.
// us a launch, 256 threads of eight pairs and a loop over the bits -> this: 53 k pairs, 8-bit digits 11.4 -> 7.0; 426 k, 9 bits 16.1 and
// 13.8 -> 12.7 and 10.6; 1.7 M, 7 bits 18.3 -> 13.6.
template <int SRC, int NT, bool FUSED, bool OPB, int MAXB>
__global__ __launch_bounds__(NT) void k_sort_scatter(const int32_t* __restrict__ keys_in,
                                                     const int32_t* __restrict__ vals_in,
                                                     const int64_t* __restrict__ offsets, int num_bags, int n,
                                                     int limit, int shift, int radix_bits, int nblk,
                                                     const int32_t* __restrict__ ghist,
                                                     const int32_t* __restrict__ dtot,
                                                     int32_t* __restrict__ keys_out,
                                                     int32_t* __restrict__ vals_out, const int32_t* __restrict__ status) {
    if (SRC == SORT_SRC_SLOTS && status && *status != FC_OK) return;      // refused: neither slots nor offsets may be read any more
    constexpr int NW = NT / 64, TILE = RS_TILE, ITEMS = TILE / NT;
    constexpr bool STAGE = MAXB <= 9;
    __shared__ int base[1 << MAXB];            // where this tile's run of each digit starts in the output
    __shared__ int wc[NW][1 << MAXB];          // per-wavefront digit counts, then exclusive offsets
    __shared__ int lds[NW];
    __shared__ int2 stage[STAGE ? TILE : 1];
    const int radix = 1 << radix_bits, mask = radix - 1;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int tile0 = blockIdx.x * TILE + w * (64 * ITEMS);
    // The tile's keys and values are requested first, all together, so that their latency runs beside the digit
    // bases below.  A lane beyond n rereads element n-1 and is masked out later.
    int key[ITEMS], val[ITEMS];
    int64_t o0[ITEMS], o1[ITEMS];
    bool bad = false;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int i = min(tile0 + it * 64 + lane, n - 1);
        key[it] = load_key<SRC>(keys_in, i, limit, bad);
        if (SRC == SORT_SRC_SLOTS && OPB) val[it] = i;
        else if (SRC == SORT_SRC_SLOTS) {      // bag of lookup i, first guess: one lookup per bag
            const int g = min(i, num_bags - 1);
            o0[it] = offsets[g];
            o1[it] = offsets[g + 1];
        } else if (SRC == SORT_SRC_COUNTS) val[it] = i;
        else val[it] = vals_in[i];
    }
    if constexpr (FUSED) {
        // digit totals = sum over the supertiles; this tile's offset within a digit = the supertiles before its own plus
        // the tiles before it inside its own.  A digit belongs to NT / radix threads, which take the rows in turn; a thread
        // requests FUSE_ROWS rows of either kind together (rows past the last reread it, unused).
        static_assert((1 << MAXB) <= NT, "a thread holds one digit");
        constexpr int FUSE_ROWS = 8;
        const int nsup = (nblk + SS_TILES - 1) / SS_TILES, mysup = blockIdx.x / SS_TILES, before = blockIdx.x - mysup * SS_TILES;
        const int parts = NT >> radix_bits, part = tid >> radix_bits, d = tid & mask;
        const int32_t* __restrict__ mine = ghist + ((size_t)mysup * SS_TILES << radix_bits);
        int tot = 0, bef = 0;
        if (nblk <= SS_TILES) {                // one supertile, and no sums of it: every tile's counts
            for (int r0 = part; r0 < nblk; r0 += FUSE_ROWS * parts) {
                int v[FUSE_ROWS];
#pragma unroll
                for (int k = 0; k < FUSE_ROWS; ++k) v[k] = ghist[((unsigned)min(r0 + k * parts, nblk - 1) << radix_bits) + d];
#pragma unroll
                for (int k = 0; k < FUSE_ROWS; ++k) {
                    const int r = r0 + k * parts;
                    tot += r < nblk ? v[k] : 0;
                    bef += r < (int)blockIdx.x ? v[k] : 0;
                }
            }
        } else
        for (int r0 = part; r0 < nsup || r0 < before; r0 += FUSE_ROWS * parts) {
            int v0[FUSE_ROWS], v1[FUSE_ROWS];
#pragma unroll
            for (int k = 0; k < FUSE_ROWS; ++k) {
                const int r = r0 + k * parts;
                v0[k] = dtot[((unsigned)min(r, nsup - 1) << radix_bits) + d];
                v1[k] = mine[((unsigned)min(r, before) << radix_bits) + d];
            }
#pragma unroll
            for (int k = 0; k < FUSE_ROWS; ++k) {
                const int r = r0 + k * parts;
                tot += r < nsup ? v0[k] : 0;
                bef += (r < mysup ? v0[k] : 0) + (r < before ? v1[k] : 0);
            }
        }
        if (parts > 1) {                       // join the parts (wc serves as scratch)
            int* scr = &wc[0][0];
            static_assert((NW << MAXB) >= 2 * NT, "");
            scr[tid] = tot; scr[NT + tid] = bef;
            __syncthreads();
            tot = bef = 0;
            if (tid < radix)
                for (int k = 0; k < parts; ++k) { tot += scr[(k << radix_bits) + tid]; bef += scr[NT + (k << radix_bits) + tid]; }
            __syncthreads();
        }
        int total;
        const int run = block_excl_scan<NT>(tot, total, lds);
        if (part == 0) base[d] = run + bef;
    } else {   // digit bases: exclusive scan of the digit totals, plus this tile's offset within the digit
        const int per = (radix + NT - 1) / NT;
        const int d0 = tid * per;
        int local = 0;
        for (int k = 0; k < per; ++k) if (d0 + k < radix) local += dtot[d0 + k];
        int tot;
        int run = block_excl_scan<NT>(local, tot, lds);
        for (int k = 0; k < per; ++k) {
            const int d = d0 + k;
            if (d < radix) {
                base[d] = run + ghist[(size_t)blockIdx.x * radix + d];
                run += dtot[d];
            }
        }
    }
    for (int d = tid; d < radix; d += NT) {
#pragma unroll
        for (int k = 0; k < NW; ++k) wc[k][d] = 0;
    }
    __syncthreads();
    if (SRC == SORT_SRC_SLOTS && !OPB) {
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int i = min(tile0 + it * 64 + lane, n - 1);
            const int g = min(i, num_bags - 1);
            val[it] = (o0[it] <= i && i < o1[it]) ? g : bag_of(offsets, num_bags, i);
        }
    }
    const uint64_t lt = (1ull << lane) - 1ull;
    uint64_t peers[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
        peers[it] = same_digit<MAXB>((key[it] >> shift) & mask, radix_bits, __ballot(tile0 + it * 64 + lane < n));
    int lrank[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const bool valid = tile0 + it * 64 + lane < n;
        const int d = (key[it] >> shift) & mask;
        const int before = __popcll(peers[it] & lt);
        int old = 0;
        if (valid) old = wc[w][d];
        if (valid && before == 0) wc[w][d] = old + __popcll(peers[it]);
        lrank[it] = old + before;
    }
    __syncthreads();
    if (STAGE) {
        // wc[k][d]: where wavefront k's first pair of digit d goes within the tile; base[d]: what that place lacks to the output's
        static_assert(!STAGE || (1 << MAXB) <= NT, "a thread holds one digit");
        int cnt = 0;
        if (tid < radix)
#pragma unroll
            for (int k = 0; k < NW; ++k) cnt += wc[k][tid];
        int total;
        int run = block_excl_scan<NT>(cnt, total, lds);
        if (tid < radix) {
            base[tid] -= run;
#pragma unroll
            for (int k = 0; k < NW; ++k) { const int c = wc[k][tid]; wc[k][tid] = run; run += c; }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it)
            if (tile0 + it * 64 + lane < n) stage[wc[w][(key[it] >> shift) & mask] + lrank[it]] = make_int2(key[it], val[it]);
        __syncthreads();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int j = it * NT + tid;
            if (j < total) {
                const int2 kv = stage[j];
                const int dest = j + base[(kv.x >> shift) & mask];
                keys_out[dest] = kv.x;
                vals_out[dest] = kv.y;
            }
        }
        return;
    }
    for (int d = tid; d < radix; d += NT) {
        int run = 0;
#pragma unroll
        for (int k = 0; k < NW; ++k) { const int cnt = wc[k][d]; wc[k][d] = run; run += cnt; }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        if (tile0 + it * 64 + lane < n) {
            const int d = (key[it] >> shift) & mask;
            const int dest = base[d] + wc[w][d] + lrank[it];
            keys_out[dest] = key[it];
            vals_out[dest] = val[it];
        }
    }
}


template <int SRC, bool FUSED, bool OPB>
static void launch_pass(const SortJob& j, hipStream_t st, const int32_t* kin, const int32_t* vin, int32_t* kout, int32_t* vout,
                        int shift, int rb, int32_t* stot) {
    const int radix = 1 << rb;
    const int nblk = (int)cdiv(j.n, RS_TILE);
    {
        ProfScope ps(j.prof, P_SORT_HIST, st);
        const bool first = shift == 0 && j.stot_other && j.other_dirty > 0;
#define FC_HIST(A) \
        k_sort_hist<SRC, A><<<(unsigned)nblk, RS_THREADS, 0, st>>>(kin, j.n, j.limit, shift, rb, nblk, j.ghist, FUSED ? stot : nullptr, \
                                                                   j.flags, j.rank_slot, j.slots_out, \
                                                                   first ? j.stot_other : nullptr, first ? (int)j.other_dirty : 0, j.status)
        if constexpr (!FUSED && (SRC == SORT_SRC_COUNTS || SRC == SORT_SRC_PAIRS)) { if (j.src == SORT_SRC_COUNTS) FC_HIST(true); else FC_HIST(false); }
        else FC_HIST(false);
#undef FC_HIST
    }
    if (!FUSED) {
        ProfScope ps(j.prof, P_SORT_SCAN, st);
        k_sort_scan<<<(unsigned)cdiv(radix, SC_DIG), SC_DIG * SC_GROUPS, 0, st>>>(j.ghist, nblk, radix, j.dtot);
    }
    // SORT_SRC_RANKS: the slots are written now, the rest of the pass reads them
    constexpr int SSRC = SRC == SORT_SRC_RANKS ? SORT_SRC_SLOTS : SRC;
    ProfScope ps(j.prof, P_SORT_SCATTER, st);
#define FC_SCATTER(NT, F, B) \
    k_sort_scatter<SSRC, NT, F, OPB, B><<<(unsigned)nblk, NT, 0, st>>>(SRC == SORT_SRC_RANKS ? j.slots_out : kin, vin, j.offsets, j.num_bags, \
                                                                                     j.n, j.limit, shift, rb, nblk, j.ghist, FUSED ? stot : j.dtot, kout, vout, SRC == SORT_SRC_RANKS ? j.status : nullptr)
    if (FUSED || rb <= 9) FC_SCATTER(512, FUSED, 9);
    else FC_SCATTER(256, false, 11);
#undef FC_SCATTER
}

template <bool FUSED>
static void first_pass(const SortJob& j, hipStream_t st, int32_t* kout, int32_t* vout, int rb, int32_t* stot) {
    const bool opb = j.one_per_bag && j.n == j.num_bags;
    if (j.src == SORT_SRC_PAIRS) launch_pass<SORT_SRC_PAIRS, FUSED, false>(j, st, j.keys_in, j.vals_in, kout, vout, 0, rb, stot);
    else if (j.src == SORT_SRC_COUNTS) launch_pass<SORT_SRC_COUNTS, FUSED, false>(j, st, j.keys_in, j.vals_in, kout, vout, 0, rb, stot);
    else if (j.src == SORT_SRC_SLOTS) {
        if (opb) launch_pass<SORT_SRC_SLOTS, FUSED, true>(j, st, j.keys_in, j.vals_in, kout, vout, 0, rb, stot);
        else launch_pass<SORT_SRC_SLOTS, FUSED, false>(j, st, j.keys_in, j.vals_in, kout, vout, 0, rb, stot);
    } else {
        if (opb) launch_pass<SORT_SRC_RANKS, FUSED, true>(j, st, j.keys_in, j.vals_in, kout, vout, 0, rb, stot);
        else launch_pass<SORT_SRC_RANKS, FUSED, false>(j, st, j.keys_in, j.vals_in, kout, vout, 0, rb, stot);
    }
}

template <bool FUSED>
static int run_passes(const SortJob& j, hipStream_t st, int passes, int rb, int32_t* stot, size_t stot_pass,
                      const int32_t** kres, const int32_t** vres) {
    const int32_t* kin = j.keys_in; const int32_t* vin = j.vals_in;
    int32_t* kout = j.keysA; int32_t* vout = j.valsA;
    for (int p = 0; p < passes; ++p) {
        int32_t* sp = FUSED && stot ? stot + stot_pass * p : nullptr;
        if (p == 1 && j.tail_stream && j.tail_event && j.tail_stream != st) {
            FC_HIP(hipEventRecord(j.tail_event, st));
            FC_HIP(hipStreamWaitEvent(j.tail_stream, j.tail_event, 0));
            st = j.tail_stream;
        }
        if (p == 0) first_pass<FUSED>(j, st, kout, vout, rb, sp);
        else launch_pass<SORT_SRC_PAIRS, FUSED, false>(j, st, kin, vin, kout, vout, p * rb, rb, sp);
        kin = kout; vin = vout;
        if (kout == j.keysA) { kout = j.keysB; vout = j.valsB; } else { kout = j.keysA; vout = j.valsA; }
    }
    *kres = kin; *vres = vin;
    if (j.last_stream) *j.last_stream = st;
    return FC_OK;
}

// passes with a scan kernel
static int scan_passes(int bits, int two) { return bits <= 2 * two ? (bits + two - 1) / two : (bits + 7) / 8; }
size_t sort_table_ints(int64_t n, int bits) {
    const int passes = scan_passes(bits, RS_TWO_PASS_BITS);
    return (size_t)cdiv(n, RS_TILE) << ((bits + passes - 1) / passes);
}

int radix_sort(const SortJob& j, hipStream_t st, const int32_t** kres, const int32_t** vres) {
    // Every pass is a chain of short launches bound by latency rather than by bytes.  Batches of up to FUSE_MAX_TILES
    // tiles take passes of at most 9 bits, each two launches (counts, then offsets and scatter in one kernel; the per-supertile
    // counts make the scan in between unnecessary; the caller supplies their table).  Up to 18 key bits that is two passes,
    // beyond three of 7 bits, which leave runs of 16 keys per digit and tile.  (Up to 18 bits a scan kernel per pass was kept
    // while a tile's 256 threads added its rows up 8 at a time; with 16 rows together, or with 8 of either kind by 512 threads as now,
    // the two launches it costs decide: 53 k pairs 143 -> 138 us a step, 852 k 1207 -> 1196, 426 k the same.)  Larger jobs (the static module's ranking) and, beyond
    // SS_TILES tiles, callers without a table keep the scan kernel: two passes up to 22 key bits, beyond that passes of at most 8 bits.
    // (j.max_bits / j.no_fuse, from FC_SORT_BITS / FC_SORT_FUSED at cache_create, override this for experiments.)
    const int env_bits = (j.max_bits >= 4 && j.max_bits <= RS_TWO_PASS_BITS) ? j.max_bits : 0;
    const bool env_fused = !j.no_fuse;
    const int64_t nblk = cdiv(j.n, RS_TILE);
    int passes, rb;
    // (Up to SS_TILES tiles the scatter kernel adds all tiles' counts up itself: no atomics on a table that all tiles share, and callers without
    // one need no scan kernels either.  us a launch, 26 tiles, counts with the table / without: 4.5 and 3.6 / 4.1 and 3.4; the backward pass
    // that allocates nothing, us a step: 18 k lookups of 128 columns 100 / 93, 38 k of 128 118 / 110.)
    const bool table = nblk > SS_TILES;
    bool fused = env_fused && (j.stot || !table) && nblk <= FUSE_MAX_TILES;
    size_t stot_pass = 0;
    if (fused) {
        const int lim = env_bits ? (env_bits < FUSE_MAX_BITS ? env_bits : FUSE_MAX_BITS) : FUSE_MAX_BITS;
        passes = (j.bits + lim - 1) / lim;
        rb = (j.bits + passes - 1) / passes;
        stot_pass = table ? (size_t)cdiv(nblk, SS_TILES) << rb : 0;
        if ((int64_t)(stot_pass * passes) > j.stot_cap) fused = false;
        // Counts of 10 and 11 bits are ranked in one pass with a scan kernel, not two without: most have the same digit, and a pass over
        // those costs more than two launches.  us a build, two passes / one, 20 k ids counted: 1000 rows 119 / 101, 10 k 129 / 100, 65 k 160 / 128.
        if (j.src == SORT_SRC_COUNTS && scan_passes(j.bits, env_bits ? env_bits : RS_TWO_PASS_BITS) < passes) fused = false;
    }
    if (!fused) {
        passes = scan_passes(j.bits, env_bits ? env_bits : RS_TWO_PASS_BITS);
        rb = (j.bits + passes - 1) / passes;
    }
    int32_t* stot = fused && table ? j.stot : nullptr;
    if (j.dirtied) *j.dirtied = fused ? (int64_t)(stot_pass * passes) : 0;
    if (fused) FC_TRY((run_passes<true>(j, st, passes, rb, stot, stot_pass, kres, vres)));
    else FC_TRY((run_passes<false>(j, st, passes, rb, stot, stot_pass, kres, vres)));
    FC_HIP(hipGetLastError());
    return FC_OK;
}

}  // namespace fc
