// Host-only checks of the one-shot batched call's choices and of its scratch (built and
// run by tests/test_batch_host.py): batch.cpp with the runtime calls that it makes on
// the way and the kernels' launchers replaced by stand-ins that keep books.
#include <cstdio>
#include <cstdlib>
#include <set>
#include <vector>

#include "batch.cpp"

static int served = 0;          // workgroups of a server's kernel
static int fail_at = 0;         // the allocation of this number fails (1: the first); 0: none
static size_t fail_above = ~size_t(0);  // allocations larger than this fail
static int allocations = 0;
static std::set<void*> held;    // scratch not yet given back
static int failures = 0;

struct Launch {
    std::vector<BatchItem> items;
    std::vector<BatchPart> parts;
    int nwg = 0;
};
static Launch last;

#define CHECK(c)                                                        \
    do {                                                                \
        if (!(c)) {                                                     \
            std::fprintf(stderr, "FAILED line %d: %s\n", __LINE__, #c); \
            ++failures;                                                 \
        }                                                               \
    } while (0)

extern "C" {
hipError_t hipMallocAsync(void** p, size_t bytes, hipStream_t) {
    if (++allocations == fail_at || bytes > fail_above) return hipErrorOutOfMemory;
    *p = std::malloc(bytes);
    held.insert(*p);
    return hipSuccess;
}
hipError_t hipFreeAsync(void* p, hipStream_t) {
    CHECK(held.erase(p) == 1);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t bytes, hipMemcpyKind, hipStream_t) {
    memcpy(d, s, bytes);
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) {
    *st = hipStreamCaptureStatusNone;
    return hipSuccess;
}
int sssp_dense_solve_ex(const int32_t*, int64_t, int32_t, int32_t, int32_t*, int32_t*, uint32_t, const sssp_tuning*,
                        void*) { return SSSP_OK; }
int sssp_last_status(void*, int32_t*, int64_t*) { return SSSP_OK; }
}

namespace sssp {
int set_error(int code, const char*) { return code; }
const char* last_error_text() { return ""; }
int stream_ctl(hipStream_t, Ctl** c, int* cus, long long* khz) {
    *c = nullptr;
    *cus = 256;
    *khz = 100000;
    return SSSP_OK;
}
int check_instance(const sssp_instance&, int) { return SSSP_OK; }
int served_workgroups(int) { return served; }
int batch_occupancy(int* per_cu) { return *per_cu = 1, 0; }
int max_batch_single_n() { return 16384; }
int max_batch_slice() { return 16384; }
size_t ctl_size() { return 64; }
hipError_t zero_fill(void*, size_t, hipStream_t) { return hipSuccess; }
hipError_t weight_range(const int32_t*, int64_t, int32_t, int32_t*, hipStream_t) { return hipSuccess; }
hipError_t compact_copy(const int32_t*, int64_t, int32_t, void*, int64_t, int, hipStream_t) { return hipSuccess; }
hipError_t launch_batch(const BatchItem* items, const BatchPart* parts, int32_t nparts, Bar*, char*, uint32_t,
                        long long, Ctl*, int nwg, hipStream_t) {
    last.parts.assign(parts, parts + nparts);
    int32_t k = 0;
    for (const BatchPart& p : last.parts) k = std::max(k, p.item + 1);
    last.items.assign(items, items + k);
    last.nwg = nwg;
    return hipSuccess;
}
}  // namespace sssp

static int solve(const std::vector<int32_t>& sizes, const sssp_tuning* t = nullptr) {
    std::vector<sssp_instance> inst;
    static int32_t word;
    for (size_t i = 0; i < sizes.size(); ++i)
        inst.push_back(sssp_instance{&word + i, sizes[i], sizes[i], 0, &word, &word});
    last = Launch();
    allocations = 0;
    return sssp_dense_solve_batched(inst.data(), (int32_t)inst.size(), 0, t, nullptr);
}

static int max_parts() {
    int m = 0;
    for (const BatchItem& it : last.items) m = std::max(m, it.parts);
    return m;
}

static void beside_a_server() {
    for (int held_by_it : {1, 128, 192, 248, 256}) {
        served = held_by_it;
        for (const auto& sizes : {std::vector<int32_t>{70}, {6000, 3000, 500}, {16384, 16384, 2}, {1000, 1000}}) {
            CHECK(solve(sizes) == SSSP_OK);
            CHECK(max_parts() == 1 && last.parts.size() == sizes.size());
        }
    }
    served = 0;
    CHECK(solve({6000, 3000, 500}) == SSSP_OK);
    CHECK(max_parts() > 1);
    CHECK(held.empty());
}

// Small graphs are solved by one workgroup, and so are those of which the others' slices
// would make a gang of two; all workgroups of a split launch run at once.
static void sizes_that_are_split() {
    for (int n : {1, 64, 65, 700, 768}) {
        CHECK(solve({n}) == SSSP_OK && max_parts() == 1);
        CHECK(solve({n, n, 6000}) == SSSP_OK && max_parts() > 1);
        for (const BatchItem& it : last.items) CHECK((it.n == n) == (it.parts == 1));
    }
    for (int n : {769, 2049, 4097, 6001, 16384}) CHECK(solve({n}) == SSSP_OK && max_parts() > 1);
    for (int count = 1; count <= 300; ++count)
        for (int n : {769, 1500, 2048, 2049, 4000, 4100, 6000, 9000}) {
            CHECK(solve(std::vector<int32_t>(count, n)) == SSSP_OK);
            CHECK(max_parts() == 1 || (max_parts() >= (n > 4096 ? 2 : 3) && last.parts.size() <= 256));
            CHECK(max_parts() == 1 || last.items[0].S * (max_parts() - 1) < n);
        }
    for (int workgroups = 1; workgroups <= 12; ++workgroups) {
        sssp_tuning t{};
        t.workgroups = workgroups;
        CHECK(solve({6000}, &t) == SSSP_OK && max_parts() != 2 && (max_parts() > 1) == (workgroups >= 6));
    }
    // 64 instances of three members; of the rest, the largest have the workgroups left over
    std::vector<int32_t> mixed(64, 5500);
    for (int n : {4000, 3000, 1000, 769, 768, 200}) mixed.push_back(n);
    CHECK(solve(mixed) == SSSP_OK && last.parts.size() <= 256);
    for (const BatchItem& it : last.items)
        CHECK(it.parts == (it.n == 5500 ? 3 : it.n <= 768 ? 1 : (it.n + 255) / 256));
    // more of them: wider slices, so that it does for all, then for the largest
    mixed.insert(mixed.end(), 4, 4000);
    CHECK(solve(mixed) == SSSP_OK && last.parts.size() <= 256);
    for (const BatchItem& it : last.items)
        CHECK(it.parts == (it.n == 5500 ? 3 : it.n > 1024 ? (it.n + 511) / 512 : 1));
    mixed.insert(mixed.end(), 14, 4000);
    CHECK(solve(mixed) == SSSP_OK && last.parts.size() <= 256);
    for (const BatchItem& it : last.items) CHECK(it.n != 4000 || it.parts == 4 || it.parts == 1);
    CHECK(solve(std::vector<int32_t>(96, 2000)) == SSSP_OK && max_parts() == 1);
    CHECK(solve(std::vector<int32_t>(48, 2000)) == SSSP_OK && max_parts() > 1);
    CHECK(held.empty());
}

// Every allocation of the call fails in turn: what was taken before is given back.  Where
// there is no room for the gangs' exchange memory, the call solves without gangs.
static void short_of_memory() {
    const std::vector<int32_t> sizes = {6000, 3000, 500};
    CHECK(solve(sizes) == SSSP_OK && held.empty());
    const int all = allocations;
    CHECK(all == 4);
    for (fail_at = 1; fail_at <= all; ++fail_at) {
        const int rc = solve(sizes);
        CHECK(rc == (fail_at == 1 ? SSSP_OK : SSSP_ENOMEM));
        CHECK(held.empty());
    }
    fail_at = 0;
    fail_above = 4096;
    CHECK(solve(sizes) == SSSP_OK && max_parts() == 1);
    CHECK(held.empty());
    fail_above = 0;
    CHECK(solve(sizes) == SSSP_ENOMEM && held.empty());
    fail_above = ~size_t(0);
}

int main() {
    beside_a_server();
    sizes_that_are_split();
    short_of_memory();
    if (failures) return 1;
    std::printf("batch host ok\n");
    return 0;
}
