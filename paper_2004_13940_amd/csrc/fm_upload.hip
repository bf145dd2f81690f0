#include "fm_upload.h"

#include <string.h>

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

// A few threads copy into the blocks while the blocks before are on their way.  The runtime's own path for pageable memory
// moved 4e8 bytes at 30 GB/s, pinned memory moves them at 57, and four threads copy at 65.  A ring belongs to one upload at a
// time; up to RING_POOL of them are kept for the next, and fm_trim gives them back.
namespace {
constexpr size_t RING_BLOCK = size_t(4) << 20;
constexpr int RING_THREADS = 4;
constexpr int RING_SLOTS = 2 * RING_THREADS;
constexpr size_t RING_POOL = 2;
}  // namespace

struct FmUploadRing {
    int device = 0;
    char* block = nullptr;  // RING_SLOTS blocks of RING_BLOCK bytes
    hipEvent_t done[RING_SLOTS] = {};
    bool busy[RING_SLOTS] = {};
};

namespace {
std::mutex g_ring_lock;
std::vector<FmUploadRing*> g_rings;

void ring_destroy(FmUploadRing* r)
{
    if (r == nullptr) return;
    for (hipEvent_t e : r->done)
        if (e != nullptr) (void)hipEventDestroy(e);
    if (r->block != nullptr) (void)hipHostFree(r->block);
    delete r;
}
}  // namespace

FmUploadRing* fm_ring_take(int device)
{
    {
        std::lock_guard<std::mutex> g(g_ring_lock);
        for (size_t i = g_rings.size(); i-- > 0;)
            if (g_rings[i]->device == device) {
                FmUploadRing* r = g_rings[i];
                g_rings.erase(g_rings.begin() + (ptrdiff_t)i);
                return r;
            }
    }
    FmUploadRing* r = new (std::nothrow) FmUploadRing();
    if (r == nullptr) return nullptr;
    r->device = device;
    bool ok = hipHostMalloc((void**)&r->block, RING_SLOTS * RING_BLOCK) == hipSuccess;
    for (hipEvent_t& e : r->done) ok = ok && hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess;
    if (ok) return r;
    (void)hipGetLastError();
    ring_destroy(r);
    return nullptr;
}

void fm_ring_give(FmUploadRing* r)
{
    if (r == nullptr) return;
    for (int slot = 0; slot < RING_SLOTS; ++slot) {
        if (r->busy[slot]) (void)hipEventSynchronize(r->done[slot]);
        r->busy[slot] = false;
    }
    {
        std::lock_guard<std::mutex> g(g_ring_lock);
        if (g_rings.size() < RING_POOL) {
            try {
                g_rings.push_back(r);
                return;
            } catch (...) {
            }
        }
    }
    ring_destroy(r);
}

void fm_ring_trim()
{
    std::vector<FmUploadRing*> rings;
    {
        std::lock_guard<std::mutex> g(g_ring_lock);
        rings.swap(g_rings);
    }
    for (FmUploadRing* r : rings) ring_destroy(r);
}

// The calling thread enqueues every copy: a stream handle may name another stream in another thread (hipStreamPerThread).
bool fm_ring_upload(FmUploadRing* r, const FmUploadPart* parts, int nparts, hipStream_t st)
{
    struct Chunk {
        char* dev;
        const char* host;
        size_t bytes;
    };
    std::vector<Chunk> chunks;
    std::vector<std::thread> threads;
    try {
        for (int p = 0; p < nparts; ++p)
            for (size_t o = 0; o < parts[p].bytes; o += RING_BLOCK)
                chunks.push_back({(char*)parts[p].dev + o, (const char*)parts[p].host + o, std::min(RING_BLOCK, parts[p].bytes - o)});
        threads.reserve(RING_THREADS);
    } catch (...) {
        return false;
    }
    // Chunk i goes through block i % RING_SLOTS.  Under the lock: how many chunks have been handed to threads, how many are
    // enqueued, which block holds a chunk that is not, and whether something failed.
    std::mutex lock;
    std::condition_variable moved;
    size_t handed = 0, enqueued = 0;
    bool full[RING_SLOTS] = {}, failed = false;
    auto block_of = [&](size_t i) { return r->block + i % RING_SLOTS * RING_BLOCK; };
    // Waits until the copy that read the block last has arrived, and fills it.
    auto fill = [&](size_t i) {
        const int slot = (int)(i % RING_SLOTS);
        if (r->busy[slot] && hipEventSynchronize(r->done[slot]) != hipSuccess) return false;
        memcpy(block_of(i), chunks[i].host, chunks[i].bytes);
        return true;
    };
    auto helper = [&] {
        const bool device = hipSetDevice(r->device) == hipSuccess;
        std::unique_lock<std::mutex> g(lock);
        failed = failed || !device;
        while (!failed && handed < chunks.size()) {
            const size_t i = handed++;
            moved.wait(g, [&] { return failed || i < enqueued + RING_SLOTS; });
            if (failed) break;
            g.unlock();
            const bool good = fill(i);
            g.lock();
            full[i % RING_SLOTS] = good;
            failed = failed || !good;
            moved.notify_all();
        }
        if (failed) moved.notify_all();
    };
    try {
        for (int t = 0; t < RING_THREADS; ++t) threads.emplace_back(helper);
    } catch (...) {  // no more threads to be had: those that run do the work, or the calling one
    }
    for (size_t i = 0; i < chunks.size(); ++i) {
        const int slot = (int)(i % RING_SLOTS);
        bool good = true;
        if (threads.empty()) {
            good = fill(i);
        } else {
            std::unique_lock<std::mutex> g(lock);
            moved.wait(g, [&] { return failed || full[slot]; });
            good = !failed;
        }
        if (good) {
            r->busy[slot] = true;
            good = hipMemcpyAsync(chunks[i].dev, block_of(i), chunks[i].bytes, hipMemcpyHostToDevice, st) == hipSuccess &&
                   hipEventRecord(r->done[slot], st) == hipSuccess;
        }
        std::lock_guard<std::mutex> g(lock);
        full[slot] = false;
        enqueued = i + 1;
        failed = failed || !good;
        moved.notify_all();
        if (failed) break;
    }
    for (std::thread& t : threads) t.join();
    if (failed) (void)hipGetLastError();
    return !failed;
}
