// When stratified epochs are captured and replayed, on the stub of the runtime.  Prints one line per check that fails, returns how
// many did.
#include "library_stub.h"

#include <vector>

int main()
{
    int bad = 0;
    const int64_t N = 40, D = 30;
    std::vector<int64_t> rowptr(N + 1);
    std::vector<int32_t> col(N);
    std::vector<float> val(N, 1.f);
    for (int64_t i = 0; i <= N; ++i) rowptr[i] = i;
    for (int64_t i = 0; i < N; ++i) col[i] = (int32_t)(i % D);
    alignas(16) static float one[64], two[64];
    fm_params p = {};
    p.K = 16;
    fm_matrix* m = nullptr;
    if (fm_build_csr(N, D, N, rowptr.data(), col.data(), val.data(), nullptr, &m) != FM_OK || fm_build_csc(m, nullptr) != FM_OK ||
        fm_partition(m, 3, nullptr) != FM_OK)
        return printf("no start: %s\n", fm_last_error(m)), 1;
    const auto epoch = [&](const char* what, float* w, long want_captures, long want_replays, bool direct) {
        const long c = captures, r = replays, n = launches;
        if (fm_stratified_epoch(m, &p, one, one, w, one, nullptr, nullptr) != FM_OK) ++bad, printf("%s: %s\n", what, fm_last_error(m));
        if (captures - c != want_captures || replays - r != want_replays)
            ++bad, printf("%s: %ld captures, %ld replays\n", what, captures - c, replays - r);
        if ((launches - n > 0) != direct) ++bad, printf("%s: %ld launches\n", what, launches - n);
    };
    epoch("by default", one, 0, 0, true);
    if (fm_set_option(m, FM_OPT_GRAPH, 2) != FM_OK) ++bad, printf("option refused\n");
    epoch("first", one, 1, 1, true);  // its launches are those that are recorded
    epoch("again", one, 0, 1, false);
    epoch("other arrays", two, 1, 1, true);
    epoch("these again", two, 0, 1, false);
    p.eta = 0.5f;
    epoch("other parameters", two, 1, 1, true);
    capture_fails = true;
    epoch("no graph to be had", one, 1, 0, true);
    capture_fails = false;
    epoch("one to be had again", one, 1, 1, true);
    if (fm_set_option(m, FM_OPT_GRAPH, 1) != FM_OK) ++bad, printf("option refused\n");
    epoch("by default again", one, 0, 0, true);
    fm_destroy(m);
    return bad;
}
