// fm_panel_rows over heights of matrices: prints one line per rule that is broken, returns how many were.
#include "fm_panels.h"

#include <algorithm>
#include <cstdio>

int main()
{
    int bad = 0;
    const auto check = [&](int64_t N, int64_t limit) {
        const int64_t rows = fm_panel_rows(N, limit), panels = (N + rows - 1) / rows;
        int64_t list[FM_XCDS] = {};
        for (int64_t b = 0; b < panels; ++b) list[b % FM_XCDS] += std::min(rows, N - b * rows);
        const int64_t longest = *std::max_element(list, list + FM_XCDS);
        if (rows < 1 || rows > limit) ++bad, printf("%lld rows: panels of %lld, more than %lld\n", (long long)N, (long long)rows, (long long)limit);
        if (N >= 64513 && panels < FM_XCDS * FM_XCD_PANELS) ++bad, printf("%lld rows: %lld panels\n", (long long)N, (long long)panels);
        // all panels have `rows` rows but the last ones, which lack less than one row for each panel together
        if (FM_XCDS * longest > N + FM_XCDS * (panels / FM_XCDS + 1)) ++bad, printf("%lld rows: a list of %lld\n", (long long)N, (long long)longest);
    };
    for (int64_t limit : {int64_t(32768), int64_t(1000)})
        for (int64_t N : {64513, 65535, 65536, 100000, 120000, 131073, 200000, 200001, 400001, 450000, 600000, 786431, 786432, 786433, 800000, 1048577, 10000000, 2147483647})
            for (int64_t d = -30; d <= 30; d += 3)
                if (N + d >= 64513) check(N + d, limit);
    if (fm_panel_rows(0, 32768) < 1 || fm_panel_rows(1, 32768) != 1) ++bad, printf("small matrices\n");
    return bad;
}
