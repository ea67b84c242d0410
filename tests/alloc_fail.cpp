// A program of its own around libfreqcache.so whose device allocations can be made to fail: hipMalloc and hipFree of this executable
// come before the runtime's.  A handle with FC_EVICT_DMA takes small batches (indexed by one workgroup) until the ring of evicted-row
// blocks has been round, then batches that need the mark map, for which there is no room: they take place all the same, and every
// row of every later batch is its own.  Row r of the table holds r.
#include <hip/hip_runtime_api.h>

#include <dlfcn.h>
#include <stdio.h>
#include <stdlib.h>

#include <set>
#include <vector>

#include "freqcache.h"

static size_t fail_from = 0;             // allocations of at least this many bytes fail; 0: none
static int failed = 0;
static std::set<void*> live;

extern "C" hipError_t hipMalloc(void** p, size_t bytes) {
    static const auto real = reinterpret_cast<hipError_t (*)(void**, size_t)>(dlsym(RTLD_NEXT, "hipMalloc"));
    if (fail_from && bytes >= fail_from) { ++failed; return hipErrorOutOfMemory; }
    const hipError_t e = real(p, bytes);
    if (e == hipSuccess) live.insert(*p);
    return e;
}

extern "C" hipError_t hipFree(void* p) {
    static const auto real = reinterpret_cast<hipError_t (*)(void*)>(dlsym(RTLD_NEXT, "hipFree"));
    live.erase(p);
    return real(p);
}

static void need(bool ok, const char* what) {
    if (!ok) { printf("FAILED: %s\n", what); fflush(stdout); exit(1); }
}

constexpr int64_t N = 1000000, C = 6000, SMALL = 3000, BIG = 5000;
constexpr int D = 4;

static int step(fc_cache* c, int64_t first, int64_t n) {
    static int64_t *ids = nullptr, *off = nullptr;
    static int32_t* slots = nullptr;
    static float* out = nullptr;
    if (!ids) {
        need(hipMalloc((void**)&ids, BIG * 8) == hipSuccess && hipMalloc((void**)&off, (BIG + 1) * 8) == hipSuccess &&
             hipMalloc((void**)&slots, BIG * 4) == hipSuccess && hipMalloc((void**)&out, BIG * D * 4) == hipSuccess, "buffers");
    }
    std::vector<int64_t> h(n), o(n + 1);
    for (int64_t i = 0; i < n; ++i) h[i] = first + (i * 7) % n;          // 7 and n have no common factor
    for (int64_t i = 0; i <= n; ++i) o[i] = i;
    need(hipMemcpy(ids, h.data(), n * 8, hipMemcpyHostToDevice) == hipSuccess, "ids");
    need(hipMemcpy(off, o.data(), (n + 1) * 8, hipMemcpyHostToDevice) == hipSuccess, "offsets");
    const int rc = cache_prepare(c, ids, n, off, n, slots);
    if (rc != FC_OK) return rc;
    need(embedding_bag_fwd(c, slots, n, off, n, out) == FC_OK, "forward");
    std::vector<float> r(n * D);
    need(hipMemcpy(r.data(), out, n * D * 4, hipMemcpyDeviceToHost) == hipSuccess, "rows");
    int64_t wrong = 0;
    for (int64_t i = 0; i < n * D; ++i) wrong += r[i] != (float)h[i / D];
    if (wrong) printf("batch at %ld: %ld of %ld values are another row's\n", (long)first, (long)wrong, (long)(n * D));
    need(wrong == 0, "rows of the batch");
    return FC_OK;
}

int main() {
    std::vector<int32_t> rank(N);
    for (int64_t i = 0; i < N; ++i) rank[i] = (int32_t)i;
    fc_cache* c = nullptr;
    need(cache_create(N, D, C, rank.data(), nullptr, 0, FC_EVICT_DMA, nullptr, &c) == FC_OK, "create");
    float* host = cache_host_weight(c);
    for (int64_t i = 0; i < N * D; ++i) host[i] = (float)(i / D);
    for (int k = 0; k < 8; ++k) need(step(c, k * SMALL, SMALL) == FC_OK, "small batch");      // from the third on, 3000 rows leave with each
    fail_from = N;                       // the mark map (num_rows bytes), not the smaller buffers of a batch
    for (int k = 0; k < 2; ++k) {
        need(step(c, (100 + 2 * k) * SMALL, BIG) == FC_OK, "large batch without room");
        need(cache_reserve(c, BIG, 0) == FC_OK, "reserve without room");
    }
    need(failed > 0, "an allocation that failed");
    printf("allocations that failed: %d\n", failed);
    fail_from = 0;
    need(step(c, 104 * SMALL, BIG) == FC_OK, "large batch");
    need(cache_reserve(c, BIG, 0) == FC_OK, "reserve");
    need(step(c, 106 * SMALL, BIG) == FC_OK, "large batch");
    for (int k = 0; k < 8; ++k) need(step(c, k * SMALL, SMALL) == FC_OK, "small batch after it");
    need(cache_check(c) == FC_OK, "check");          // (not before: it drops the marks of rows in transit)
    const size_t mine = 4;               // buffers of step()
    need(cache_destroy(c) == FC_OK, "destroy");
    printf("allocations left: %ld\n", (long)(live.size() - mine));
    need(live.size() == mine, "everything is given back");
    printf("ok\n");
    return 0;
}
