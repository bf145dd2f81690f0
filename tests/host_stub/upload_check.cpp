// fm_ring_upload on the stub runtime: prints one line per check that fails, returns how many did.
#include "fm_upload.h"

#include <cstdint>
#include <cstdio>
#include <vector>

int main()
{
    int bad = 0;
    const size_t MB = size_t(1) << 20;
    const size_t sizes[][3] = {{1, 0, 5}, {4 * MB, 4 * MB, 4 * MB}, {9 * MB + 3, 40 * MB + 1, 21 * MB}, {0, 33 * MB, 0}};
    for (hipStream_t st : {hipStream_t(nullptr), hipStreamPerThread})
        for (int round = 0; round < 2; ++round)  // the second takes the blocks that the first left
            for (const auto& size : sizes) {
                std::vector<std::vector<uint8_t>> host, dev;
                std::vector<FmUploadPart> parts;
                for (int p = 0; p < 3; ++p) {
                    host.emplace_back(size[p]);
                    dev.emplace_back(size[p], 0xEE);
                    for (size_t i = 0; i < size[p]; ++i) host[p][i] = (uint8_t)((i * 2654435761u >> 13) + p + round);
                }
                for (int p = 0; p < 3; ++p) parts.push_back({dev[p].data(), host[p].data(), size[p]});
                FmUploadRing* r = fm_ring_take(0);
                if (r == nullptr || !fm_ring_upload(r, parts.data(), 3, st)) ++bad, printf("upload refused\n");
                (void)hipStreamSynchronize(st);  // all that follows on the caller's stream comes after the copies
                for (int p = 0; p < 3; ++p)
                    if (host[p] != dev[p]) ++bad, printf("stream %p, round %d, %zu bytes: not there\n", (void*)st, round, size[p]);
                fm_ring_give(r);
            }
    // given back before the copies have run: the next upload through the ring may not overwrite its blocks
    {
        std::vector<uint8_t> a(10 * MB, 1), b(10 * MB, 2), da(a.size()), db(b.size());
        for (int k = 0; k < 2; ++k) {
            FmUploadRing* r = fm_ring_take(0);
            const FmUploadPart part = {(k ? db : da).data(), (k ? b : a).data(), a.size()};
            if (!fm_ring_upload(r, &part, 1, k ? hipStreamPerThread : nullptr)) ++bad, printf("upload refused\n");
            fm_ring_give(r);
        }
        (void)hipStreamSynchronize(nullptr);
        (void)hipStreamSynchronize(hipStreamPerThread);
        if (a != da || b != db) ++bad, printf("blocks given back too early\n");
    }
    // a copy that is refused ends the upload, and every thread of it
    for (int k : {0, 1, 7, 8, 11}) {
        std::vector<uint8_t> a(50 * MB), d(a.size());
        const FmUploadPart part = {d.data(), a.data(), a.size()};
        FmUploadRing* r = fm_ring_take(0);
        stub_fail_copy = k;
        if (fm_ring_upload(r, &part, 1, nullptr)) ++bad, printf("refused copy %d not reported\n", k);
        stub_fail_copy = -1;
        (void)hipStreamSynchronize(nullptr);
        fm_ring_give(r);
    }
    fm_ring_trim();
    return bad;
}
