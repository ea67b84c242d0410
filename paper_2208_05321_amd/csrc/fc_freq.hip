// Static module of the cache (paper Section 4.2), built on the GPU: count how often every id occurs in (a sample
// of) the dataset, order the rows by descending count (ties: lower id first) -> idx_map ("freq_rank"), and
// re-order the embedding table accordingly.
#include "fc_internal.h"

#include <limits.h>
#include <omp.h>
#include <string.h>

#include <algorithm>
#include <memory>
#include <new>
#include <vector>

struct fc_freq {
    int64_t N = 0;
    int device = 0;
    hipStream_t stream = nullptr;
    int32_t* counts = nullptr;     // [N]
    int64_t total = 0;             // ids counted so far: no single counter can exceed it
    uint32_t* flags = nullptr;     // EF_ID_RANGE
    int32_t* maxc = nullptr;
};

namespace fc {

// counts[id] += occurrences.  Popular ids repeat thousands of times and device atomics on one address, or one cache line (the ids of a
// small column are neighbours), queue up, so each workgroup first aggregates its ids in an LDS hash table and sends one atomic per distinct id.
template <int NT, int ITEMS>
__global__ __launch_bounds__(NT) void k_freq_count(const int64_t* __restrict__ ids, int64_t n, int64_t N,
                                                   int32_t* counts, uint32_t* flags) {
    constexpr int HASH = 2 * NT * ITEMS;           // twice the ids of a workgroup: open addressing always finds a free entry
    constexpr int BITS = __builtin_ctz(HASH);
    __shared__ int hkey[HASH];
    __shared__ int hcnt[HASH];
    const int64_t base = (int64_t)blockIdx.x * NT * ITEMS;
    int64_t id[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int64_t i = base + k * NT + threadIdx.x;
        id[k] = i < n ? ids[i] : INT64_MAX;
    }
    for (int e = threadIdx.x; e < HASH; e += NT) { hkey[e] = -1; hcnt[e] = 0; }
    __syncthreads();
    bool bad = false;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        if ((uint64_t)id[it] >= (uint64_t)N) { bad |= base + it * NT + threadIdx.x < n; continue; }
        const int k = (int)id[it];
        unsigned h = ((unsigned)k * 2654435761u) >> (32 - BITS);
        for (;;) {
            const int prev = atomicCAS(&hkey[h], -1, k);
            if (prev == -1 || prev == k) { atomicAdd(&hcnt[h], 1); break; }
            h = (h + 1) & (HASH - 1);
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < HASH; e += NT)
        if (hkey[e] >= 0) atomicAdd(&counts[hkey[e]], hcnt[e]);
    if (bad) atomicOr(flags, EF_ID_RANGE);
}

// 16 bytes a lane, and few workgroups: each ends with an atomic on one address (10 M counters: 23 -> 9.5 us).
__global__ __launch_bounds__(1024) void k_max_i32(const int32_t* __restrict__ x, int64_t n, int32_t* out) {
    __shared__ int red[16];
    int m = 0;
    const int64_t n4 = n / 4, stride = (int64_t)gridDim.x * 1024, t = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    for (int64_t i = t; i < n4; i += stride) {
        const int4 v = reinterpret_cast<const int4*>(x)[i];
        m = max(max(m, max(v.x, v.y)), max(v.z, v.w));
    }
    if (t < n - 4 * n4) m = max(m, x[4 * n4 + t]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_down(m, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < 16; ++k) m = max(m, red[k]);
        atomicMax(out, m);
    }
}

// sorted position r holds id inv[r]; the id's rank is r
__global__ __launch_bounds__(256) void k_rank_of(const int32_t* __restrict__ inv, int64_t n, int32_t* __restrict__ rank) {
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r < n) rank[inv[r]] = (int32_t)r;
}

// dst[r, :] = src[inv[r], :]; both tables may be mapped host memory
__global__ __launch_bounds__(256) void k_reorder_rows(float* __restrict__ dst, const float* __restrict__ src,
                                                      const int32_t* __restrict__ inv, int64_t rows, int D, int vec4) {
    const int lane = threadIdx.x & 63;
    const int64_t w0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6, nw = ((int64_t)gridDim.x * 256) >> 6;
    for (int64_t r = w0; r < rows; r += nw) {
        const float* s = src + (size_t)inv[r] * D;
        float* d = dst + (size_t)r * D;
        if (vec4) { for (int c = lane; c < D / 4; c += 64) reinterpret_cast<float4*>(d)[c] = reinterpret_cast<const float4*>(s)[c]; }
        else { for (int c = lane; c < D; c += 64) d[c] = s[c]; }
    }
}

static void freq_free(fc_freq* f) {
    if (!f) return;
    (void)hipSetDevice(f->device);
    if (f->counts) (void)hipFree(f->counts);
    if (f->flags) (void)hipFree(f->flags);
    if (f->maxc) (void)hipFree(f->maxc);
    delete f;
}

static int freq_init(fc_freq* f, int64_t N, void* stream) {
    FC_HIP(hipGetDevice(&f->device));
    f->N = N; f->stream = (hipStream_t)stream;
    FC_HIP(hipMalloc((void**)&f->counts, (size_t)N * 4));
    FC_HIP(hipMalloc((void**)&f->flags, 4));
    FC_HIP(hipMalloc((void**)&f->maxc, 4));
    FC_HIP(hipMemsetAsync(f->counts, 0, (size_t)N * 4, f->stream));
    FC_HIP(hipMemsetAsync(f->flags, 0, 4, f->stream));
    FC_HIP(hipStreamSynchronize(f->stream));
    return FC_OK;
}

// Result arrays on their way to the caller's ordinary memory.  The runtime's own copy into such memory moves it through a
// staging buffer with one thread, which also takes the page faults of arrays nobody has touched yet (10 M ints: 3.9 ms, 2.4 of
// them the copy); here chunks land in two pinned buffers in turn and several threads carry them on, faults included, while
// the next chunk crosses the link.  The threads are the bottleneck (40 MB: 0.9 ms of faults and 0.5 of copying, 0.7 on the link), so they
// take faults while the GPU still counts and sorts.  10 M rows, counted, ranked and copied out: 6.7 -> 4.5 ms, 4 M 3.1 -> 1.85, 20 M 11.6 -> 8.0.
struct CopyOut {
    static constexpr size_t CHUNK = 8u << 20;
    struct Piece { char* dst; const char* src; size_t len; };
    char* pin[2] = {nullptr, nullptr};
    hipEvent_t ev[2] = {nullptr, nullptr};
    int32_t* dst[3] = {};                      // the arrays, `bytes` long each, one after the other; sources are known later
    const int32_t* src[3] = {};
    size_t bytes = 0, arrays = 0, touched = 0;      // touched: bytes, all arrays in a row
    int threads = 1;
    bool ok = false;

    CopyOut() {
        threads = omp_get_max_threads();
        if (threads > 16) threads = 16;
        ok = true;
        for (int k = 0; k < 2 && ok; ++k)
            ok = hipHostMalloc((void**)&pin[k], CHUNK, hipHostMallocDefault) == hipSuccess &&
                 hipEventCreateWithFlags(&ev[k], hipEventDisableTiming) == hipSuccess;
        if (!ok) (void)hipGetLastError();
    }
    ~CopyOut() {
        for (int k = 0; k < 2; ++k) {
            if (ev[k]) (void)hipEventDestroy(ev[k]);
            if (pin[k]) (void)hipHostFree(pin[k]);
        }
    }
    CopyOut(const CopyOut&) = delete;
    CopyOut& operator=(const CopyOut&) = delete;

    size_t pieces() const { return arrays * cdiv(bytes, CHUNK); }
    Piece piece(size_t i) const {
        const size_t per = cdiv(bytes, CHUNK), a = i / per, off = i % per * CHUNK;
        return {(char*)dst[a] + off, (const char*)src[a] + off, std::min(CHUNK, bytes - off)};
    }

    // Faults the next pages in, a block of 2 MB to a thread: where pages are that large, threads that met in one would each clear it.  One
    // instruction reads a byte and writes it back, so that the first access is a write: a read would map the zero page, and the write after it
    // fault again (arrays of 8 to 80 MB: 10 ms more).
    void touch_some() {
        constexpr size_t BLOCK = 2u << 20;
        const size_t a = touched / bytes, off = touched % bytes;
        char* const from = (char*)dst[a] + off;
        char* const first = (char*)((uintptr_t)from & ~(uintptr_t)(BLOCK - 1));
        char* const to = std::min((char*)dst[a] + bytes, first + threads * BLOCK);
#pragma omp parallel for schedule(static, 1) num_threads(threads)
        for (int t = 0; t < threads; ++t)
            for (char* q = std::max(from, first + t * BLOCK); q < std::min(to, first + (t + 1) * BLOCK); q = (char*)(((uintptr_t)q & ~(uintptr_t)4095) + 4096))
                __asm__ volatile("orb $0, %0" : "+m"(*q) : : "cc");
        touched += to - from;
    }

    // Until what has been enqueued on st is done, pages are faulted in.
    int wait_touching(hipStream_t st) {
        FC_HIP(hipEventRecord(ev[0], st));
        while (touched < arrays * bytes) {
            const hipError_t q = hipEventQuery(ev[0]);
            if (q == hipSuccess) return FC_OK;
            (void)hipGetLastError();
            if (q != hipErrorNotReady) return FC_ERR_HIP;
            touch_some();
        }
        FC_HIP(hipEventSynchronize(ev[0]));
        return FC_OK;
    }

    // Returns once every piece is where it belongs.
    int run(hipStream_t st) {
        for (size_t i = 0; i <= pieces(); ++i) {
            if (i < pieces()) {
                const Piece q = piece(i);
                FC_HIP(hipMemcpyAsync(pin[i & 1], q.src, q.len, hipMemcpyDeviceToHost, st));
                FC_HIP(hipEventRecord(ev[i & 1], st));
            }
            if (i > 0) {
                const Piece q = piece(i - 1);
                const size_t per = cdiv(bytes, CHUNK), end = (i - 1) / per * bytes + (i - 1) % per * CHUNK + q.len;
                while (touched < end) touch_some();
                FC_HIP(hipEventSynchronize(ev[(i - 1) & 1]));
                const char* p = pin[(i - 1) & 1];
#pragma omp parallel for schedule(static) num_threads(threads)
                for (int t = 0; t < threads; ++t) {
                    const size_t a = q.len * t / threads, b = q.len * (t + 1) / threads;
                    memcpy(q.dst + a, p + a, b - a);
                }
            }
        }
        return FC_OK;
    }
};
constexpr size_t ONE_BY_ONE_MOST = 2u << 20;   // bytes of an array: see freq_build_impl
constexpr size_t COPY_OUT_MIN = 8u << 20;      // 2 M rows: 2.2 -> 1.9 ms; below, setting the buffers up costs what they save

static int freq_build_impl(fc_freq* f, int32_t* freq_rank_host, int32_t* inv_rank_host, int32_t* counts_host) {
    const int64_t N = f->N;
    const size_t bytes = (size_t)N * 4;
    hipStream_t st = f->stream;
    std::unique_ptr<CopyOut> out;
    if (bytes >= COPY_OUT_MIN) {                   // set up beside the counting
        out.reset(new (std::nothrow) CopyOut());
        if (out && !out->ok) out.reset();
    }
    uint32_t flags = 0;
    FC_HIP(hipMemsetAsync(f->maxc, 0, 4, st));
    k_max_i32<<<(unsigned)std::min<int64_t>(256, cdiv(N, 4096)), 1024, 0, st>>>(f->counts, N, f->maxc);
    FC_HIP(hipGetLastError());
    int32_t maxc = 0;
    // (into pinned memory the copies do not hold the host up)
    int32_t* word = out ? reinterpret_cast<int32_t*>(out->pin[1]) : nullptr;
    FC_HIP(hipMemcpyAsync(word ? word : &maxc, f->maxc, 4, hipMemcpyDeviceToHost, st));
    FC_HIP(hipMemcpyAsync(word ? (void*)(word + 1) : (void*)&flags, f->flags, 4, hipMemcpyDeviceToHost, st));
    // One allocation: giving back a large one costs 0.25 ms, whatever its size (10 M rows, seven of them: 1.7 ms of 6.7).  Small ones come
    // out of a block that the runtime keeps, and are cheaper one by one, up to 2 MB each (0.3 M rows 325 us in one, 290 one by one; 0.4 M 373 and 367; 0.53 M 485 and 615).  The
    // digit table is not known yet, so it is laid out for the most digits that a count of all ids so far could take.
    int most = 1;
    while (((int64_t)1 << most) <= f->total) ++most;
    size_t table = 0;
    for (int b = 1; b <= most; ++b) table = std::max(table, sort_table_ints(N, b));
    const size_t part = (bytes + 255) & ~(size_t)255;
    const bool one = part > ONE_BY_ONE_MOST;
    char* mem[5] = {};
    auto body = [&]() -> int {
        const size_t tables = (table + (1 << RS_MAX_BITS)) * 4;
        if (one) {
            FC_HIP(hipMalloc((void**)&mem[0], 4 * part + tables));
        } else
            for (int k = 0; k < 5; ++k) FC_HIP(hipMalloc((void**)&mem[k], k < 4 ? part : tables));
        int32_t* buf[5];
        for (int k = 0; k < 5; ++k) buf[k] = reinterpret_cast<int32_t*>(one ? mem[0] + k * part : mem[k]);
        int32_t* const wanted[3] = {counts_host, inv_rank_host, freq_rank_host};
        if (out) {
            out->bytes = bytes;
            for (int32_t* p : wanted) if (p) out->dst[out->arrays++] = p;
            FC_TRY(out->wait_touching(st));
            maxc = word[0]; flags = (uint32_t)word[1];
        } else FC_HIP(hipStreamSynchronize(st));
        if (flags & EF_ID_RANGE) return FC_ERR_ID_OUT_OF_RANGE;
        int bits = 1;
        while (((int64_t)1 << bits) <= maxc) ++bits;
        SortJob j;
        j.src = SORT_SRC_COUNTS; j.keys_in = f->counts; j.n = (int)N; j.limit = maxc; j.bits = bits;
        j.keysA = buf[0]; j.valsA = buf[1]; j.keysB = buf[2]; j.valsB = buf[3];
        j.ghist = buf[4]; j.dtot = j.ghist + table;
        const int32_t *ks, *vs;
        FC_TRY(radix_sort(j, st, &ks, &vs));       // stable: equal counts keep ascending id order
        int32_t* rank = const_cast<int32_t*>(ks);  // the sorted keys have served
        k_rank_of<<<(unsigned)cdiv(N, 256), 256, 0, st>>>(vs, N, rank);
        FC_HIP(hipGetLastError());
        if (out) {
            const int32_t* const from[3] = {f->counts, vs, rank};
            for (int k = 0, a = 0; k < 3; ++k) if (wanted[k]) out->src[a++] = from[k];
            FC_TRY(out->wait_touching(st));
            return out->run(st);
        }
        if (freq_rank_host) FC_HIP(hipMemcpyAsync(freq_rank_host, rank, bytes, hipMemcpyDeviceToHost, st));
        if (inv_rank_host) FC_HIP(hipMemcpyAsync(inv_rank_host, vs, bytes, hipMemcpyDeviceToHost, st));
        if (counts_host) FC_HIP(hipMemcpyAsync(counts_host, f->counts, bytes, hipMemcpyDeviceToHost, st));
        FC_HIP(hipStreamSynchronize(st));
        return FC_OK;
    };
    const int rc = body();
    if (rc != FC_OK) (void)hipStreamSynchronize(st);       // nothing enqueued may still use what is given back
    for (char* p : mem) if (p) (void)hipFree(p);
    return rc;
}

static bool pinned_dev_ptr(const void* host, void** dev) {
    hipPointerAttribute_t attr;
    if (hipPointerGetAttributes(&attr, host) != hipSuccess || attr.type != hipMemoryTypeHost) { (void)hipGetLastError(); return false; }
    if (hipHostGetDevicePointer(dev, const_cast<void*>(host), 0) != hipSuccess) { (void)hipGetLastError(); return false; }
    return true;
}

}  // namespace fc

using namespace fc;

extern "C" {

int freq_create(int64_t num_rows, void* hip_stream, fc_freq** out) {
    const int64_t LIM = ((int64_t)1 << 31) - 65536;
    if (!out) return FC_ERR_INVALID_ARG;
    *out = nullptr;
    if (num_rows <= 0 || num_rows >= LIM) return FC_ERR_INVALID_ARG;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) { (void)hipGetLastError(); return FC_ERR_HIP; }
    fc_freq* f = new (std::nothrow) fc_freq();
    if (!f) return FC_ERR_INVALID_ARG;
    const int rc = freq_init(f, num_rows, hip_stream);
    if (rc != FC_OK) { freq_free(f); return rc; }
    *out = f;
    return FC_OK;
}

int freq_add(fc_freq* f, const int64_t* ids_dev, int64_t n) {
    if (!f || n < 0 || (n > 0 && !ids_dev)) return FC_ERR_INVALID_ARG;
    if (n == 0) return FC_OK;
    // counters are 32 bits wide: an id that occurred more than 2^31 - 1 times would wrap around unnoticed, so the
    // accumulator takes at most that many ids in all (larger datasets are sampled, as Section 4.2 suggests)
    if (f->total + n > (int64_t)INT32_MAX) return FC_ERR_COUNT_OVERFLOW;
    f->total += n;
    FC_HIP(hipSetDevice(f->device));
    // us a call, 2048 ids a workgroup / 4096 / 8192: 21 k ids 7.9 / 7.2 / 11.3, 65 k 14.0 / 9.7 / 12.8, 130 k 23 / 15 / 14, 426 k 65 / 40 / 28,
    // 1.7 M 236 / 147 / 93: what grows is the number of workgroups that meet on the popular ids.
    if (n <= 1 << 17) k_freq_count<1024, 4><<<(unsigned)cdiv(n, 4096), 1024, 0, f->stream>>>(ids_dev, n, f->N, f->counts, f->flags);
    else k_freq_count<1024, 8><<<(unsigned)cdiv(n, 8192), 1024, 0, f->stream>>>(ids_dev, n, f->N, f->counts, f->flags);
    FC_HIP(hipGetLastError());
    return FC_OK;
}

int freq_build(fc_freq* f, int32_t* freq_rank_host, int32_t* inv_rank_host, int32_t* counts_host) {
    if (!f) return FC_ERR_INVALID_ARG;
    FC_HIP(hipSetDevice(f->device));
    return freq_build_impl(f, freq_rank_host, inv_rank_host, counts_host);
}

int freq_destroy(fc_freq* f) {
    if (!f) return FC_ERR_INVALID_ARG;
    (void)hipSetDevice(f->device);
    (void)hipStreamSynchronize(f->stream);
    freq_free(f);
    return FC_OK;
}

int table_reorder(const float* src_pinned, float* dst_pinned, const int32_t* inv_rank_host, int64_t num_rows, int32_t dim,
                  void* hip_stream) {
    const int64_t LIM = ((int64_t)1 << 31) - 65536;
    if (!src_pinned || !dst_pinned || !inv_rank_host || num_rows <= 0 || num_rows >= LIM || dim <= 0 || src_pinned == dst_pinned)
        return FC_ERR_INVALID_ARG;
    for (int64_t r = 0; r < num_rows; ++r) if (inv_rank_host[r] < 0 || inv_rank_host[r] >= num_rows) return FC_ERR_NOT_PERMUTATION;
    void *sd = nullptr, *dd = nullptr;
    if (!pinned_dev_ptr(src_pinned, &sd) || !pinned_dev_ptr(dst_pinned, &dd)) return FC_ERR_NOT_PINNED;
    hipStream_t st = (hipStream_t)hip_stream;
    int32_t* inv = nullptr;
    FC_HIP(hipMalloc((void**)&inv, (size_t)num_rows * 4));
    int rc = FC_OK;
    auto body = [&]() -> int {
        FC_HIP(hipMemcpyAsync(inv, inv_rank_host, (size_t)num_rows * 4, hipMemcpyHostToDevice, st));
        k_reorder_rows<<<4096, 256, 0, st>>>((float*)dd, (const float*)sd, inv, num_rows, dim, dim % 4 == 0);
        FC_HIP(hipGetLastError());
        FC_HIP(hipStreamSynchronize(st));
        return FC_OK;
    };
    rc = body();
    (void)hipFree(inv);
    return rc;
}

}  // extern "C"
