// Builds that fail halfway, on the stub of the runtime.  Prints one line per check that fails, returns how many did.
#include "library_stub.h"

#include <functional>
#include <vector>

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
