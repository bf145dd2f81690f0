// Upload of large arrays from pageable host memory through a ring of pinned blocks.  Host code on the HIP runtime and the
// standard library alone.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

struct FmUploadRing;

struct FmUploadPart {
    void* dev;
    const void* host;
    size_t bytes;
};

// From so many bytes on: 6.4e7 bytes take 2.2 ms on the runtime's path; below, starting the threads and filling the ring for
// the first blocks is no longer small beside what is gained.
constexpr size_t FM_RING_MIN = size_t(64) << 20;

FmUploadRing* fm_ring_take(int device);  // nullptr: none to be had
// Waits for the copies that still read its blocks.
void fm_ring_give(FmUploadRing* r);
void fm_ring_trim();
// Enqueues all copies on st; the host arrays have been read when it returns.  False: something failed, nothing is known
// about the destination.
bool fm_ring_upload(FmUploadRing* r, const FmUploadPart* parts, int nparts, hipStream_t st);
