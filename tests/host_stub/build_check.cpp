// Builds that fail halfway, on a runtime of which nothing is real: "device" memory is host memory, kernels do nothing, one value
// read back from the device is 3, longer reads give what is there (zeros).  This program's definitions take the place of the
// runtime's in the library.  From the call that `fail_from` counts down to on, everything that can fail does.  Prints one line
// per check that fails, returns how many did.
#include "fm.h"

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <vector>

static long fail_from = -1, launches = 0, failed = 0;
static std::map<void*, size_t> live;
static int last = 0;

static int can_fail()
{
    if (fail_from < 0 || --fail_from >= 0) return last = 0;
    fail_from = 0;  // and every call from here on
    ++failed;
    return last = 2;
}

struct Dim3 {
    uint32_t x, y, z;
};
extern "C" {
int hipGetDevice(int* d) { return *d = 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { const int e = last; last = 0; return e; }
const char* hipGetErrorString(int) { return "as the test wants"; }
int hipMalloc(void** p, size_t n)
{
    if (can_fail()) return 2;
    *p = calloc(n, 1);
    live[*p] = n;
    return 0;
}
int hipFree(void* p)
{
    if (live.erase(p) != 1) printf("freed twice\n"), abort();
    free(p);
    return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) { return (*p = calloc(n, 1)) == nullptr; }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void*)
{
    if (can_fail()) return 2;
    const int64_t three = 3;
    memcpy(d, kind == 2 && n == 8 ? (const void*)&three : s, n);
    return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void*)
{
    if (can_fail()) return 2;
    memset(d, v, n);
    return 0;
}
int hipDeviceSynchronize() { return 0; }
int hipStreamSynchronize(void*) { return can_fail(); }
int hipStreamIsCapturing(void*, int* s) { return *s = 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetSymbolAddress(void** p, const void*)
{
    static char block[1 << 16];
    *p = block;
    return 0;
}
int __hipPushCallConfiguration(Dim3, Dim3, size_t, void*) { return 0; }
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* s, void** st)
{
    *g = *b = Dim3{1, 1, 1};
    *s = 0;
    *st = nullptr;
    return 0;
}
int hipLaunchKernel(const void*, Dim3, Dim3, void**, size_t, void*)
{
    if (can_fail()) return 2;
    ++launches;
    return 0;
}
}

static size_t live_bytes()
{
    (void)fm_trim();
    size_t t = 0;
    for (const auto& b : live) t += b.second;
    return t;
}

int main()
{
    int bad = 0;
    const int64_t N = (1 << 21) + 3, D = 300, nnz = 4096;
    std::vector<int64_t> rowptr(N + 1, nnz);
    std::vector<int32_t> col(nnz);
    std::vector<float> val(nnz, 1.f);
    for (int64_t i = 0; i < nnz; ++i) rowptr[i] = i, col[i] = (int32_t)(i % D);
    alignas(16) static float some[64];
    fm_params p = {};
    p.K = 16;  // whose tiles are another shape than those that are built before K is known
    auto forward = [&](fm_matrix* m) { return fm_forward(m, &p, nullptr, some, some, some, some, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr); };
    auto csc = [](fm_matrix* m) { return fm_build_csc(m, nullptr); };
    auto strata = [](fm_matrix* m) { return fm_partition(m, 3, nullptr); };
    auto batches = [](fm_matrix* m) { return fm_partition_batches(m, 3, nullptr); };
    auto begin = [&](fm_matrix* m) { return fm_stratified_begin(m, &p, some, some, some, some, nullptr); };
    auto epoch = [&](fm_matrix* m) { return fm_minibatch_epoch(m, &p, some, some, some, some, nullptr, nullptr); };
    using Call = std::function<int(fm_matrix*)>;
    struct {
        const char* what;
        std::vector<Call> before;
        Call call;
        Call refused;  // FM_ESTATE as long as the call has not succeeded; may be empty
    } const cases[] = {{"fm_build_csc", {}, csc, strata},
                       {"fm_partition", {csc}, strata, begin},
                       {"fm_partition_batches", {csc}, batches, epoch},
                       {"the index for another K", {csc}, forward, Call()}};
    for (const auto& c : cases) {
        auto open = [&] {
            (void)fm_trim();  // fresh pinned memory: the check of the rows reads from it that they are sound
            fm_matrix* m = nullptr;
            if (fm_build_csr(N, D, nnz, rowptr.data(), col.data(), val.data(), nullptr, &m) != FM_OK) printf("no handle: %s\n", fm_last_error(nullptr)), exit(1);
            for (const Call& b : c.before)
                if (b(m) != FM_OK) printf("%s: no start\n", c.what), exit(1);
            return m;
        };
        fm_matrix* m = open();
        long n = launches;
        if (c.call(m) != FM_OK) ++bad, printf("%s failed\n", c.what);
        const long whole = launches - n;
        fm_destroy(m);
        long at = 0, kept = 0;
        for (;; ++at) {
            m = open();
            const size_t held = live_bytes();
            fail_from = at;
            failed = 0;
            const int rc = c.call(m);
            fail_from = -1;
            if (failed == 0) break;
            if (rc == FM_OK || rc == FM_ESTATE) ++bad, printf("%s, call %ld fails: returned %d\n", c.what, at, rc);
            // an index that is built anew was given up; what hangs on the columns of a handle stays (a flag and a mark per column)
            const size_t rest = live_bytes();
            if (c.refused && rest > held + 2 * (size_t)D * 4) ++bad, printf("%s, call %ld fails: %zu bytes left\n", c.what, at, rest - held);
            if (c.refused && c.refused(m) != FM_ESTATE) ++bad, printf("%s, call %ld fails: taken for done\n", c.what, at);
            n = launches;
            if (c.call(m) != FM_OK) ++bad, printf("%s, call %ld fails: not to be had again\n", c.what, at);
            // once the index is there, the three blocks of the workspace and the pass itself may fail and leave it
            if (!c.refused && launches - n == 1 && ++kept <= 4)
                ;
            else if (launches - n < whole - (c.refused ? 1 : 0))  // the flags per column are not cleared again
                ++bad, printf("%s, call %ld fails: then %ld launches of %ld\n", c.what, at, launches - n, whole);
            fm_destroy(m);
        }
        if (at < 10) ++bad, printf("%s: %ld calls that can fail\n", c.what, at);
        fm_destroy(m);
    }
    if (live_bytes() != 0) ++bad, printf("%zu bytes never freed\n", live_bytes());
    return bad;
}
