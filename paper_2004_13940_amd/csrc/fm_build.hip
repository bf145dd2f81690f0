// Integer-only builders: exclusive scan, stable LSD radix sort with values, CSR->CSC transpose,
// the per-stratum matrices of the double partition, and the work-item lists for long
// columns.  Everything here is deterministic (integer atomics are only used for
// counts, whose totals do not depend on the order of the additions).
#include "fm_device.h"
#include "fm_internal.h"

namespace {

// ------------------------------------------------------------------ scan ----
constexpr int SCAN_T = 256;
constexpr int SCAN_E = 8;
constexpr int SCAN_TILE = SCAN_T * SCAN_E;

// exclusive prefix of one int64 per thread across the 256 threads of a block
__device__ __forceinline__ int64_t block_exclusive_256(int64_t v, int64_t (*sh)[SCAN_T], int64_t* total)
{
    const int t = threadIdx.x;
    sh[0][t] = v;
    __syncthreads();
    int cur = 0;
    for (int o = 1; o < SCAN_T; o <<= 1) {
        int64_t x = sh[cur][t];
        if (t >= o) x += sh[cur][t - o];
        sh[cur ^ 1][t] = x;
        __syncthreads();
        cur ^= 1;
    }
    const int64_t incl = sh[cur][t];
    if (total != nullptr) *total = sh[cur][SCAN_T - 1];
    __syncthreads();
    return incl - v;
}

__global__ __launch_bounds__(SCAN_T) void k_scan_sums(const int64_t* __restrict__ d, int64_t n,
                                                      int64_t* __restrict__ sums)
{
    __shared__ int64_t sh[2][SCAN_T];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
    int64_t v = 0;
    for (int u = 0; u < SCAN_E; ++u) {
        const int64_t i = base + (int64_t)u * SCAN_T + threadIdx.x;
        if (i < n) v += d[i];
    }
    int64_t total;
    block_exclusive_256(v, sh, &total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(SCAN_T) void k_scan_apply(int64_t* __restrict__ d, int64_t n,
                                                       const int64_t* __restrict__ offs)
{
    __shared__ int64_t sh[2][SCAN_T];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_E;
    int64_t x[SCAN_E];
    int64_t tot = 0;
#pragma unroll
    for (int u = 0; u < SCAN_E; ++u) {
        x[u] = (base + u < n) ? d[base + u] : 0;
        tot += x[u];
    }
    int64_t run = block_exclusive_256(tot, sh, nullptr) + (offs != nullptr ? offs[blockIdx.x] : 0);
#pragma unroll
    for (int u = 0; u < SCAN_E; ++u) {
        if (base + u < n) d[base + u] = run;
        run += x[u];
    }
}

// Eight consecutive values of an array of n from e, a multiple of eight, on: 16 bytes at a time where all are there.
constexpr int OWN_E = 8;
template <class T>
__device__ __forceinline__ void load_eight(const T* __restrict__ p, int64_t e, int64_t n, uint32_t (&v)[OWN_E])
{
    static_assert(sizeof(T) == 4, "words");
    if (e + OWN_E <= n) {
        const uint4 a = *reinterpret_cast<const uint4*>(p + e), b = *reinterpret_cast<const uint4*>(p + e + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else {
#pragma unroll
        for (int i = 0; i < OWN_E; ++i) v[i] = e + i < n ? (uint32_t)p[e + i] : 0u;
    }
}
__device__ __forceinline__ void store_eight(uint32_t* __restrict__ p, int64_t e, int64_t n, const uint32_t (&v)[OWN_E])
{
    if (e + OWN_E <= n) {
        *reinterpret_cast<uint4*>(p + e) = make_uint4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<uint4*>(p + e + 4) = make_uint4(v[4], v[5], v[6], v[7]);
    } else {
#pragma unroll
        for (int i = 0; i < OWN_E; ++i)
            if (e + i < n) p[e + i] = v[i];
    }
}

// ------------------------------------------------------------ radix sort ----
constexpr int RS_T = 512;
constexpr int RS_W = RS_T / FM_WAVE;
constexpr int RS_ROUNDS = 16;
constexpr int RS_TILE = RS_T * RS_ROUNDS;
constexpr int RS_VALUES = 3;  // arrays that can travel with the keys

struct SortIn {
    const uint32_t* key;
    const uint32_t* v[RS_VALUES];
};
struct SortOut {
    uint32_t* key;
    uint32_t* v[RS_VALUES];
};

// The digits of a tile, counted.  A thread takes RS_ROUNDS consecutive keys and adds a run of equal digits at once: in a key
// that earlier passes have sorted, and in the strata of a column's entries, the digits of a wavefront are few, and one by one
// their additions to the same counter stood in line (4.9e7 keys by 16 strata 141 us, by the top four bits of a sorted column
// 153).  A counter per wavefront and digit; one addition where all lanes hold one digit.  Bound: one read of the keys, which
// for the strata's the kernel that makes them has in hand.  Counts of opening 4.9e7 entries in 16 strata: 589 -> 203 us (eight launches).
struct DigitCount {
    uint32_t h[RS_W][256];
};
__device__ __forceinline__ void count_digits_begin(DigitCount& c)
{
    for (int k = threadIdx.x; k < RS_W * 256; k += RS_T) (&c.h[0][0])[k] = 0;
    __syncthreads();
}
// d: the digits of OWN_E consecutive keys, the first `count` of them (0 to OWN_E)
__device__ __forceinline__ void count_digits(DigitCount& c, const uint32_t (&d)[OWN_E], int count)
{
    uint32_t* h = c.h[threadIdx.x / FM_WAVE];
    const uint32_t lead = (uint32_t)__builtin_amdgcn_readfirstlane((int)d[0]);
    bool one = count == OWN_E;
#pragma unroll
    for (int u = 0; u < OWN_E; ++u) one = one && d[u] == lead;
    if (__all(one)) {
        if (threadIdx.x % FM_WAVE == 0) atomicAdd(&h[lead], (uint32_t)(OWN_E * FM_WAVE));
        return;
    }
    uint32_t run = 0;
#pragma unroll
    for (int u = 0; u < OWN_E; ++u) {
        run += u < count ? 1u : 0u;
        if (run > 0 && (u == OWN_E - 1 || d[u + 1 < OWN_E ? u + 1 : u] != d[u] || u + 1 >= count)) {
            atomicAdd(&h[d[u]], run);
            run = 0;
        }
        if (u + 1 >= count) run = 0;
    }
}
__device__ __forceinline__ void count_digits_end(const DigitCount& c, int nbins, int64_t* __restrict__ hist, int64_t nblocks)
{
    __syncthreads();
    if ((int)threadIdx.x < nbins) {
        uint32_t t = 0;
#pragma unroll
        for (int w = 0; w < RS_W; ++w) t += c.h[w][threadIdx.x];
        hist[(int64_t)threadIdx.x * nblocks + blockIdx.x] = (int64_t)t;
    }
}

__global__ __launch_bounds__(RS_T) void k_radix_hist(const uint32_t* __restrict__ keys, int64_t n, int shift, int nbins,
                                                     int64_t* __restrict__ hist, int64_t nblocks)
{
    __shared__ DigitCount c;
    count_digits_begin(c);
#pragma unroll
    for (int r = 0; r < RS_ROUNDS / OWN_E; ++r) {
        const int64_t e = (int64_t)blockIdx.x * RS_TILE + ((int64_t)r * RS_T + threadIdx.x) * OWN_E;
        uint32_t d[OWN_E] = {};
        if (e < n) load_eight(keys, e, n, d);
#pragma unroll
        for (int u = 0; u < OWN_E; ++u) d[u] = (d[u] >> shift) & 255u;
        count_digits(c, d, e >= n ? 0 : n - e < OWN_E ? (int)(n - e) : OWN_E);
    }
    count_digits_end(c, nbins, hist, nblocks);
}

// One stable pass: a workgroup orders its tile by the digit in LDS and writes it out from there, so that the elements of a
// digit leave as one run (32 of them on average at 256 digits) instead of one by one.  A wavefront takes 1,024 consecutive
// elements, 64 a round; an element's place is the number of equal digits before it in the wavefront (a counter per digit
// and the lanes below), plus those of the wavefronts before.  The values travel with the keys: fetching them afterwards by
// a sorted index was a random line per entry and array, and a search for its row besides (2.4 ms for 4.9e7 entries).  A
// pass over 4.9e7 entries with two values takes 0.33 ms.  Kernels of opening that data set, its 16 strata and one epoch:
// 18.6 -> 9.6 ms.
template <int NV>
__global__ __launch_bounds__(RS_T) void k_radix_scatter(const SortIn in, const SortOut out, int64_t n, int shift, int nbins,
                                                        const int64_t* __restrict__ hist, int64_t nblocks)
{
    __shared__ uint32_t data[RS_TILE];
    __shared__ uint32_t cnt[RS_W][256];
    __shared__ uint32_t scan[2][256];
    __shared__ uint32_t from[256];  // where the run of a digit goes, minus where it starts in the tile (modulo 2^32)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int k = tid; k < RS_W * 256; k += RS_T) (&cnt[0][0])[k] = 0;
    __syncthreads();
    const int64_t tile = (int64_t)blockIdx.x * RS_TILE;
    const int m = (int)((n - tile) < RS_TILE ? (n - tile) : RS_TILE);
    const int first = wave * (RS_TILE / RS_W) + lane;
    uint32_t key[RS_ROUNDS], pos[RS_ROUNDS];
#pragma unroll
    for (int u = 0; u < RS_ROUNDS; ++u) key[u] = first + u * 64 < m ? in.key[tile + first + u * 64] : 0u;
    volatile uint32_t* mine = cnt[wave];
#pragma unroll
    for (int u = 0; u < RS_ROUNDS; ++u) {
        const bool valid = first + u * 64 < m;
        const uint32_t dg = (key[u] >> shift) & 255u;
        unsigned long long mask = __ballot(valid);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const bool bb = (dg >> bit) & 1u;
            const unsigned long long bal = __ballot(bb);
            mask &= bb ? bal : ~bal;
        }
        const uint32_t rank = (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
        const uint32_t before = mine[dg];
        pos[u] = before + rank;
        __builtin_amdgcn_wave_barrier();
        if (valid && rank == 0) mine[dg] = before + (uint32_t)__popcll(mask);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    uint32_t total = 0;
    if (tid < 256) {
        for (int w = 0; w < RS_W; ++w) {
            const uint32_t c = cnt[w][tid];
            cnt[w][tid] = total;
            total += c;
        }
        scan[0][tid] = total;
    }
    __syncthreads();
    int cur = 0;
    for (int o = 1; o < 256; o <<= 1) {
        if (tid < 256) scan[cur ^ 1][tid] = scan[cur][tid] + (tid >= o ? scan[cur][tid - o] : 0u);
        __syncthreads();
        cur ^= 1;
    }
    if (tid < 256) {
        const uint32_t start = scan[cur][tid] - total;
        for (int w = 0; w < RS_W; ++w) cnt[w][tid] += start;
        from[tid] = tid < nbins ? (uint32_t)hist[(int64_t)tid * nblocks + blockIdx.x] - start : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < RS_ROUNDS; ++u) {
        pos[u] += cnt[wave][(key[u] >> shift) & 255u];
        if (first + u * 64 < m) data[pos[u]] = key[u];
    }
    __syncthreads();
    uint32_t dst[RS_ROUNDS];
#pragma unroll
    for (int u = 0; u < RS_ROUNDS; ++u) {
        const int i = tid + u * RS_T;
        const uint32_t k = i < m ? data[i] : 0u;
        dst[u] = from[(k >> shift) & 255u] + (uint32_t)i;
        if (i < m && out.key != nullptr) out.key[dst[u]] = k;
    }
#pragma unroll
    for (int a = 0; a < NV; ++a) {
        uint32_t x[RS_ROUNDS];
#pragma unroll
        for (int u = 0; u < RS_ROUNDS; ++u) x[u] = first + u * 64 < m ? in.v[a][tile + first + u * 64] : 0u;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < RS_ROUNDS; ++u)
            if (first + u * 64 < m) data[pos[u]] = x[u];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < RS_ROUNDS; ++u) {
            const int i = tid + u * RS_T;
            if (i < m) out.v[a][dst[u]] = data[i];
        }
    }
}

// ------------------------------------------------------------- CSR check ----
// Sum over the 256 threads of a workgroup, valid in thread 0.
__device__ __forceinline__ int64_t block_sum_256(int64_t v, int64_t* sh)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    const int64_t t = sh[0] + sh[1] + sh[2] + sh[3];
    __syncthreads();
    return t;
}

// The rules of fm_build_csr, one pass over the uploaded arrays.  Columns ascend inside every row exactly when every
// entry whose column is not above its predecessor's opens a row, so the entries with a descent are counted once over
// the entries and once over the starts of the non-empty rows, and the two counts must agree (no search for the row of
// an entry).  A matrix with rowptr[i] = i D whose columns ascend in [0, D) stores every column in every row.
// One result per workgroup in pinned host memory: no counter to clear, nothing to copy back.  Bound: one read of
// the pointers and columns; 4.9e7 entries take 0.06 ms where the loop on the host took 20 ms.
__global__ __launch_bounds__(256) void k_check_csr(const int64_t* __restrict__ rowptr, const int32_t* __restrict__ col,
                                                   int64_t N, int64_t D, int64_t nnz, FmCheck* __restrict__ out)
{
    __shared__ int64_t sh[4];
    const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    int64_t bad = 0, descents = 0, not_dense = 0;
    for (int64_t i = first; i < N; i += step) {
        const int64_t b = rowptr[i], e = rowptr[i + 1];
        if (b < 0 || e < b || e > nnz)
            bad = 1;
        else if (b > 0 && e > b && col[b - 1] >= col[b])
            --descents;
        if (b != i * D) not_dense = 1;
    }
    for (int64_t t = first * OWN_E; t < nnz; t += step * OWN_E) {
        uint32_t c[OWN_E];
        int32_t before = t > 0 ? col[t - 1] : -1;
        load_eight(col, t, nnz, c);
#pragma unroll
        for (int u = 0; u < OWN_E; ++u) {
            if (t + u >= nnz) continue;
            const int32_t x = (int32_t)c[u];
            if (x < 0 || x >= D) bad = 1;
            if (t + u > 0 && before >= x) ++descents;
            before = x;
        }
    }
    bad = block_sum_256(bad, sh);
    descents = block_sum_256(descents, sh);
    not_dense = block_sum_256(not_dense, sh);
    if (threadIdx.x == 0) out[blockIdx.x] = FmCheck{bad, descents, not_dense};
}

// ------------------------------------------------------------- transpose ----
// owner of entry e in a pointer array ptr[0..n]: the k with ptr[k] <= e < ptr[k+1]
__device__ __forceinline__ int64_t owner_of(const int64_t* __restrict__ ptr, int64_t n, int64_t e)
{
    int64_t lo = 0, hi = n;
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (ptr[mid] <= e) lo = mid; else hi = mid;
    }
    return lo;
}

// The owners of the entries e .. e + OWN_E - 1 below n, e < n: one search, then a few steps from one to the next (a long run
// of empty owners is searched again).  The lanes of a wavefront hold consecutive stretches: it looks for the owner of its
// first entry and for a bound of its last one's together, and a lane searches the few owners in between.  On their own the
// lanes' lookups of twenty steps filled the L1 (4.9e7 entries in rows of 39: 160 -> 122 us, with their strata 231 -> 191).
__device__ __forceinline__ void owners_of(const int64_t* __restrict__ ptr, int64_t nown, int64_t e, int64_t n,
                                          uint32_t (&own)[OWN_E])
{
    const int64_t first = (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)e >> 32)) << 32 |
                                    (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uint64_t)e));
    const int64_t last = first + FM_WAVE * OWN_E < n ? first + FM_WAVE * OWN_E - 1 : n - 1;
    int64_t k = owner_of(ptr, nown, first), above = k + 1;
    for (int64_t step = 1; above < nown && ptr[above] <= last; step *= 2) above = above + step < nown ? above + step : nown;
    while (above - k > 1) {
        const int64_t mid = (k + above) >> 1;
        if (ptr[mid] <= e) k = mid; else above = mid;
    }
    int64_t next = ptr[k + 1];
#pragma unroll
    for (int i = 0; i < OWN_E; ++i) {
        for (int step = 0; e + i < n && next <= e + i; ++step) {
            k = step < 4 ? k + 1 : owner_of(ptr, nown, e + i);
            next = ptr[k + 1];
        }
        own[i] = (uint32_t)k;
    }
}

__global__ __launch_bounds__(256) void k_owners(const int64_t* __restrict__ ptr, int64_t nown, int64_t n,
                                                uint32_t* __restrict__ out)
{
    const int64_t e = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * OWN_E;
    if (e >= n) return;
    uint32_t own[OWN_E];
    owners_of(ptr, nown, e, n, own);
    store_eight(out, e, n, own);
}

// ptr[j] = number of sorted keys smaller than j, j = 0..ncols
__global__ void k_ptr_from_sorted(const uint32_t* __restrict__ keys, int64_t n, int64_t ncols,
                                  int64_t* __restrict__ ptr)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j > ncols) return;
    int64_t lo = 0, hi = n;  // first position with key >= j
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)keys[mid] < j) lo = mid + 1; else hi = mid;
    }
    ptr[j] = lo;
}

// -------------------------------------------------------------- partition ----
// Stratum and major index (row of a CSR entry, column of a CSC entry) of every stored entry; `major` is the pointer array
// of the orientation being processed (rowptr for CSR, colptr for CSC) and `minor` its index array.  A workgroup takes a tile of
// the sort and leaves the counts of its first digit as well.
__global__ __launch_bounds__(RS_T) void k_stratum_keys(const int64_t* __restrict__ major, int64_t nmajor,
                                                       const int32_t* __restrict__ minor, int64_t n, int64_t N, int64_t D,
                                                       int32_t P, int by_rows, const int32_t* __restrict__ place,
                                                       uint32_t* __restrict__ keys, uint32_t* __restrict__ maj, int nbins,
                                                       int64_t* __restrict__ hist, int64_t nblocks)
{
    __shared__ DigitCount c;
    count_digits_begin(c);
    for (int r = 0; r < RS_ROUNDS / OWN_E; ++r) {
        const int64_t e = (int64_t)blockIdx.x * RS_TILE + ((int64_t)r * RS_T + threadIdx.x) * OWN_E;
        uint32_t key[OWN_E] = {};
        if (e < n) {
            uint32_t own[OWN_E], mn[OWN_E];
            load_eight(minor, e, n, mn);
            owners_of(major, nmajor, e, n, own);
#pragma unroll
            for (int u = 0; u < OWN_E; ++u) {
                if (e + u >= n) continue;
                const int64_t i = by_rows == 1 ? own[u] : mn[u];
                const int64_t j = by_rows == 1 ? mn[u] : own[u];
                const int32_t p = fm_block_of(i, N, P);
                int32_t s = p;  // row batches: the key is the row block alone
                if (by_rows != 2) {
                    s = (place != nullptr ? place[j] : fm_block_of(j, D, P)) - p;
                    if (s < 0) s += P;
                }
                key[u] = (uint32_t)s;
            }
            store_eight(keys, e, n, key);
            store_eight(maj, e, n, own);
        }
#pragma unroll
        for (int u = 0; u < OWN_E; ++u) key[u] &= 255u;
        count_digits(c, key, e >= n ? 0 : n - e < OWN_E ? (int)(n - e) : OWN_E);
    }
    count_digits_end(c, nbins, hist, nblocks);
}

// The (stratum, major) pairs of the entries in stratum order are runs: entry i opens one where it differs from the entry
// before.  Pass 0 counts a tile's runs, pass 1 lists them (tile_cnt then scanned): major index and first entry.
constexpr int HD_E = OWN_E;
constexpr int HD_TILE = 256 * HD_E;
__global__ __launch_bounds__(256) void k_heads(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ maj, int64_t n,
                                               int pass, int64_t* __restrict__ tile_cnt, int32_t* __restrict__ nz_major,
                                               int64_t* __restrict__ nz_beg)
{
    __shared__ int64_t sh[2][SCAN_T];
    const int64_t base = (int64_t)blockIdx.x * HD_TILE + (int64_t)threadIdx.x * HD_E;
    uint32_t mj[HD_E], ky[HD_E];
    unsigned heads = 0;
    if (base < n) {
        uint32_t pk = base > 0 ? keys[base - 1] : 0u, pm = base > 0 ? maj[base - 1] : 0u;
        load_eight(keys, base, n, ky);
        load_eight(maj, base, n, mj);
#pragma unroll
        for (int u = 0; u < HD_E; ++u) {
            if (base + u < n && (base + u == 0 || ky[u] != pk || mj[u] != pm)) heads |= 1u << u;
            pk = ky[u];
            pm = mj[u];
        }
    }
    int64_t total;
    int64_t pos = block_exclusive_256(__popc(heads), sh, &total);
    if (!pass) {
        if (threadIdx.x == 0) tile_cnt[blockIdx.x] = total;
        return;
    }
    pos += tile_cnt[blockIdx.x];
#pragma unroll
    for (int u = 0; u < HD_E; ++u)
        if (heads >> u & 1u) {
            nz_major[pos] = (int32_t)mj[u];
            nz_beg[pos] = base + u;
            ++pos;
        }
}

// out[t] = number of elements of the ascending array a[0..n) that are smaller than bound[t]
__global__ void k_lower_bounds(const int64_t* __restrict__ a, int64_t n, const int64_t* __restrict__ bound, int64_t nb,
                               int64_t* __restrict__ out)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nb) return;
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (a[mid] < bound[t]) lo = mid + 1; else hi = mid;
    }
    out[t] = lo;
}

// first list position in [lo, hi) whose row is >= bound
__device__ __forceinline__ int64_t first_listed_row(const int32_t* __restrict__ rows, int64_t lo, int64_t hi, int64_t bound)
{
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)rows[mid] < bound) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// cell[p*P + c] = entries of row block p in the columns of block c (or placed at worker c): exactly those of the rows
// of block p in stratum (c - p) mod P, whose rows are listed in ascending order with the offset of their entries.
// Two searches per cell; counting entry by entry with atomics on the P x P table took 67 ms for 4.9e7 entries at
// P = 16 (a handful of cells takes most of the additions), this takes microseconds.
__global__ void k_cell_table(const int32_t* __restrict__ touched, const int64_t* __restrict__ touched_beg,
                             const int64_t* __restrict__ list_off, const int64_t* __restrict__ row_bounds, int32_t P,
                             int64_t* __restrict__ cell)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)P * P) return;
    const int32_t p = (int32_t)(t / P), c = (int32_t)(t % P);
    const int32_t s = c >= p ? c - p : c - p + P;
    const int64_t lo = first_listed_row(touched, list_off[s], list_off[s + 1], row_bounds[p]);
    const int64_t hi = first_listed_row(touched, lo, list_off[s + 1], row_bounds[p + 1]);
    cell[t] = touched_beg[hi] - touched_beg[lo];
}

// ------------------------------------------------------------ long index ----
constexpr int LI_T = 256;
constexpr int LI_E = 4;
constexpr int LI_TILE = LI_T * LI_E;

__global__ __launch_bounds__(LI_T) void k_long_count(const int64_t* __restrict__ ptr, int64_t ncols, int seg,
                                                     int64_t* __restrict__ tile_long, int64_t* __restrict__ tile_items)
{
    __shared__ int64_t sh[2][SCAN_T];
    const int64_t base = (int64_t)blockIdx.x * LI_TILE + (int64_t)threadIdx.x * LI_E;
    int64_t nl = 0, ni = 0;
    for (int u = 0; u < LI_E; ++u) {
        const int64_t c = base + u;
        if (c < ncols) {
            const int64_t len = ptr[c + 1] - ptr[c];
            if (len > seg) {
                nl += 1;
                ni += (len + seg - 1) / seg;
            }
        }
    }
    int64_t t0, t1;
    block_exclusive_256(nl, sh, &t0);
    block_exclusive_256(ni, sh, &t1);
    if (threadIdx.x == 0) {
        tile_long[blockIdx.x] = t0;
        tile_items[blockIdx.x] = t1;
    }
}

__global__ __launch_bounds__(LI_T) void k_long_fill(const int64_t* __restrict__ ptr, int64_t ncols,
                                                    const int32_t* __restrict__ ids, int seg,
                                                    const int64_t* __restrict__ tile_long,
                                                    const int64_t* __restrict__ tile_items,
                                                    int32_t* __restrict__ long_col, int64_t* __restrict__ long_vcol,
                                                    int64_t* __restrict__ long_first)
{
    __shared__ int64_t sh[2][SCAN_T];
    const int64_t base = (int64_t)blockIdx.x * LI_TILE + (int64_t)threadIdx.x * LI_E;
    int64_t nl = 0, ni = 0;
    for (int u = 0; u < LI_E; ++u) {
        const int64_t c = base + u;
        if (c < ncols) {
            const int64_t len = ptr[c + 1] - ptr[c];
            if (len > seg) {
                nl += 1;
                ni += (len + seg - 1) / seg;
            }
        }
    }
    int64_t lpos = block_exclusive_256(nl, sh, nullptr) + tile_long[blockIdx.x];
    int64_t ipos = block_exclusive_256(ni, sh, nullptr) + tile_items[blockIdx.x];
    for (int u = 0; u < LI_E; ++u) {
        const int64_t c = base + u;
        if (c >= ncols) break;
        const int64_t len = ptr[c + 1] - ptr[c];
        if (len <= seg) continue;
        const int32_t j = ids != nullptr ? ids[c] : (int32_t)c;
        long_col[lpos] = j;
        long_vcol[lpos] = c;
        if (long_first != nullptr) long_first[lpos] = ipos;
        ++lpos;
        ipos += (len + seg - 1) / seg;
    }
}

// Items of every long column, consecutive segments of `seg` entries; one wavefront per column.
__global__ __launch_bounds__(256) void k_items(const int64_t* __restrict__ ptr, const int32_t* __restrict__ long_col,
                                               const int64_t* __restrict__ long_vcol, const int64_t* __restrict__ long_first,
                                               int64_t nlong, int seg, int32_t* __restrict__ item_col,
                                               int64_t* __restrict__ item_beg, int32_t* __restrict__ item_len,
                                               int64_t* __restrict__ long_beg, int32_t* __restrict__ long_len)
{
    const int64_t lc = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
    if (lc >= nlong) return;
    const int64_t c = long_vcol[lc], b = ptr[c], len = ptr[c + 1] - b;
    const int64_t first = long_first[lc], n = long_first[lc + 1] - first;
    const int32_t j = long_col[lc];
    if (long_beg != nullptr && threadIdx.x % 64 == 0) {
        long_beg[lc] = b;
        long_len[lc] = (int32_t)len;
    }
    for (int64_t k = threadIdx.x % 64; k < n; k += 64) {
        const int64_t left = len - k * seg;
        item_col[first + k] = j;
        item_beg[first + k] = b + k * seg;
        item_len[first + k] = (int32_t)(left < seg ? left : seg);
    }
}


// -------------------------------------------- short non-empty columns ----
// Columns with 1..seg entries, in (virtual) column order: k_cols works through this list;
// empty columns only feel the regulariser and are handled by an elementwise kernel.
__global__ __launch_bounds__(LI_T) void k_short_list(const int64_t* __restrict__ ptr, int64_t ncols,
                                                     const int32_t* __restrict__ ids, int seg,
                                                     int pass, int64_t* __restrict__ tile_cnt,
                                                     int32_t* __restrict__ short_col, int64_t* __restrict__ short_vcol,
                                                     int64_t* __restrict__ short_beg, int32_t* __restrict__ short_len)
{
    __shared__ int64_t sh[2][SCAN_T];
    const int64_t base = (int64_t)blockIdx.x * LI_TILE + (int64_t)threadIdx.x * LI_E;
    int64_t ns = 0;
    for (int u = 0; u < LI_E; ++u) {
        const int64_t c = base + u;
        if (c < ncols) {
            const int64_t len = ptr[c + 1] - ptr[c];
            if (len > 0 && len <= seg) ns += 1;
        }
    }
    int64_t total;
    int64_t pos = block_exclusive_256(ns, sh, &total);
    if (!pass) {
        if (threadIdx.x == 0) tile_cnt[blockIdx.x] = total;
        return;
    }
    pos += tile_cnt[blockIdx.x];
    for (int u = 0; u < LI_E; ++u) {
        const int64_t c = base + u;
        if (c >= ncols) break;
        const int64_t len = ptr[c + 1] - ptr[c];
        if (len > 0 && len <= seg) {
            short_col[pos] = ids != nullptr ? ids[c] : (int32_t)c;
            short_vcol[pos] = c;
            short_beg[pos] = ptr[c];
            short_len[pos] = (int32_t)len;
            ++pos;
        }
    }
}

// off[s] = number of list entries whose position in the column list is < bounds[s], s = 0..nstrata
__global__ void k_stratum_offsets(const int64_t* __restrict__ vcol, int64_t n, const int64_t* __restrict__ bounds,
                                  int32_t nstrata, int64_t* __restrict__ off)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s > nstrata) return;
    const int64_t bound = bounds[s];
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (vcol[mid] < bound) lo = mid + 1; else hi = mid;
    }
    off[s] = lo;
}


// ---------------------------------------------------- full-matrix items ----
// first position in rows[beg,end) (ascending) whose row is >= bound
__device__ __forceinline__ int64_t first_row_at_least(const int32_t* __restrict__ rows, int64_t beg, int64_t end,
                                                      int64_t bound)
{
    int64_t lo = beg, hi = end;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)rows[mid] < bound) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Items of every long column of the full matrix.  A column with fewer than heavy_min
// entries is cut into consecutive segments of `seg` entries.  A heavy column is first
// cut at the boundaries of the row panels [b*panel, (b+1)*panel) and every piece then
// into segments of `seg`; its items carry the key (b % FM_XCDS, b / FM_XCDS) so that the
// stable sort by key hands panel b to XCD b % FM_XCDS in ascending panel order.  Other
// items get the last position of the list (slot % FM_XCDS) and run after the panels.
// A column with at least tile_min entries ("dense-ish") is instead cut at the boundaries of
// row tiles of `tile` rows and into segments of `tseg`; its items get the key
// FM_XCDS*(maxpos+1) + tile id, i.e. they sort behind the eight lists, tile by tile, and are
// processed by the kernel that stages a tile of aggregate rows in LDS.
// One workgroup per long column; pass 0 counts, pass 1 fills.
__global__ __launch_bounds__(256) void k_full_items(const int64_t* __restrict__ colptr, const int32_t* __restrict__ crow,
                                                    const int32_t* __restrict__ long_col, int64_t N, int seg,
                                                    int64_t panel, int64_t heavy_min, int64_t maxpos, int64_t tile,
                                                    int64_t tile_min, int tseg, int pass,
                                                    int64_t* __restrict__ nitems, const int64_t* __restrict__ long_first,
                                                    int32_t* __restrict__ item_col, int64_t* __restrict__ item_beg,
                                                    int32_t* __restrict__ item_len, uint32_t* __restrict__ item_key)
{
    __shared__ int64_t sh[2][SCAN_T];
    const int64_t lc = blockIdx.x;
    const int32_t j = long_col[lc];
    const int64_t beg = colptr[j], end = colptr[j + 1], cnt = end - beg;
    const int64_t first = pass ? long_first[lc] : 0;
    const bool tiled = cnt >= tile_min;
    if (!tiled && cnt < heavy_min) {
        const int64_t nit = (cnt + seg - 1) / seg;
        if (!pass) {
            if (threadIdx.x == 0) nitems[lc] = nit;
            return;
        }
        for (int64_t k = threadIdx.x; k < nit; k += blockDim.x) {
            const int64_t slot = first + k;
            item_col[slot] = j;
            item_beg[slot] = beg + k * seg;
            item_len[slot] = (int32_t)((cnt - k * seg) < seg ? (cnt - k * seg) : seg);
            item_key[slot] = (uint32_t)((slot % FM_XCDS) * (maxpos + 1) + maxpos);
        }
        return;
    }
    const int64_t piece = tiled ? tile : panel;  // rows per piece
    const int64_t sg = tiled ? tseg : seg;       // entries per item inside a piece
    const int64_t npieces = (N + piece - 1) / piece;
    int64_t running = 0;
    // a search per piece: where the next one starts is the next thread's answer
    __shared__ int64_t starts[256];
    for (int64_t b0 = 0; b0 < npieces; b0 += blockDim.x - 1) {
        const int64_t b = b0 + threadIdx.x;
        int64_t lo = end;
        if (b < npieces) {  // the rows are distinct: at most `row` of them lie before, and at most N - row from there on
            const int64_t row = b * piece;
            lo = first_row_at_least(crow, end - (N - row) > beg ? end - (N - row) : beg, beg + row < end ? beg + row : end, row);
        }
        starts[threadIdx.x] = lo;
        __syncthreads();
        const bool mine = b < npieces && threadIdx.x + 1 < blockDim.x;
        const int64_t hi = mine ? starts[threadIdx.x + 1] : lo;
        const int64_t nb = (hi - lo + sg - 1) / sg;
        int64_t total;
        const int64_t off = block_exclusive_256(nb, sh, &total);
        if (pass) {
            const uint32_t key = tiled ? (uint32_t)(FM_XCDS * (maxpos + 1) + b)
                                       : (uint32_t)((b % FM_XCDS) * (maxpos + 1) + b / FM_XCDS);
            for (int64_t k = 0; k < nb; ++k) {
                const int64_t slot = first + running + off + k;
                item_col[slot] = j;
                item_beg[slot] = lo + k * sg;
                item_len[slot] = (int32_t)((hi - lo - k * sg) < sg ? (hi - lo - k * sg) : sg);
                item_key[slot] = key;
            }
        }
        running += total;
    }
    if (!pass && threadIdx.x == 0) nitems[lc] = running;
}

// tile_ptr[t] = number of sorted keys smaller than base + t, t = 0..ntiles
__global__ void k_tile_ptr(const uint32_t* __restrict__ keys, int64_t n, int64_t base, int64_t ntiles,
                           int64_t* __restrict__ tile_ptr)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t > ntiles) return;
    const int64_t bound = base + t;
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)keys[mid] < bound) lo = mid + 1; else hi = mid;
    }
    tile_ptr[t] = lo;
}

// item records copied into processing order, so that the column kernel streams them
__global__ void k_order_items(const uint32_t* __restrict__ order, int64_t n, const int64_t* __restrict__ item_beg,
                              const int32_t* __restrict__ item_len, int64_t* __restrict__ ord_beg,
                              int32_t* __restrict__ ord_len)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        const uint32_t it = order[i];
        ord_beg[i] = item_beg[it];
        ord_len[i] = item_len[it];
    }
}

__global__ void k_iota_u32(uint32_t* __restrict__ x, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = (uint32_t)i;
}

// Key of item i of strata 0..nstrata-1 (item_off[s] is the first item of stratum s): its stratum, then its first row in
// units of 2^shift rows.
__global__ void k_row_keys(const int64_t* __restrict__ item_beg, int64_t n, const int32_t* __restrict__ row,
                           const int64_t* __restrict__ item_off, int32_t nstrata, int shift, int row_bits,
                           uint32_t* __restrict__ keys, uint32_t* __restrict__ idx)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int32_t lo = 0, hi = nstrata - 1;  // last stratum that starts at or before i
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (item_off[mid] <= i) lo = mid; else hi = mid - 1;
    }
    keys[i] = ((uint32_t)lo << row_bits) | ((uint32_t)row[item_beg[i]] >> shift);
    idx[i] = (uint32_t)i;
}

// list_off[x] = number of sorted keys smaller than x * (maxpos+1), x = 0..FM_XCDS
// and list_off[FM_XCDS+1+x] = number of keys smaller than x*(maxpos+1)+maxpos (first non-panel item)
__global__ void k_list_offsets(const uint32_t* __restrict__ keys, int64_t n, int64_t maxpos,
                               int64_t* __restrict__ list_off)
{
    const int x = threadIdx.x;
    if (x > 2 * FM_XCDS) return;
    const int64_t bound = x <= FM_XCDS ? (int64_t)x * (maxpos + 1)
                                       : (int64_t)(x - FM_XCDS - 1) * (maxpos + 1) + maxpos;
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)keys[mid] < bound) lo = mid + 1; else hi = mid;
    }
    list_off[x] = lo;
}

inline unsigned blocks_for(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

// ---------------------------------------------------------------- hosts ----

static int bits_for(int64_t maxval)
{
    int b = 0;
    while (b < 32 && ((int64_t)1 << b) <= maxval) ++b;
    return b;
}

int fm_check_csr(fm_matrix* m, hipStream_t st, bool* valid)
{
    *valid = false;
    FmCheck* res = reinterpret_cast<FmCheck*>(m->h_scal + 8);
    // few entries per thread while the grid is small (latency), at most two workgroups per compute unit (bandwidth)
    const int64_t work = std::max<int64_t>(std::max(m->nnz, m->N), 1);
    const unsigned grid = (unsigned)std::min<int64_t>(FM_CHECK_BLOCKS, (work + 4 * 256 - 1) / (4 * 256));
    hipLaunchKernelGGL(k_check_csr, dim3(grid), dim3(256), 0, st, (const int64_t*)m->rowptr, (const int32_t*)m->col, m->N,
                       m->D, m->nnz, res);
    FM_HIP(m, hipGetLastError());
    FM_HIP(m, hipStreamSynchronize(st));
    FmCheck sum = {0, 0, 0};
    for (unsigned b = 0; b < grid; ++b) {
        sum.bad += res[b].bad;
        sum.descents += res[b].descents;
        sum.not_dense += res[b].not_dense;
    }
    *valid = sum.bad == 0 && sum.descents == 0;
    m->is_dense = *valid && sum.not_dense == 0 && m->N > 0 && m->D > 0 && m->nnz == m->N * m->D;
    return FM_OK;
}

int fm_scan_exclusive_i64(fm_matrix* m, int64_t* d, int64_t n, hipStream_t st)
{
    if (n <= 0) return FM_OK;
    const int64_t ntiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    if (ntiles == 1) {
        hipLaunchKernelGGL(k_scan_apply, dim3(1), dim3(SCAN_T), 0, st, d, n, (const int64_t*)nullptr);
        FM_HIP(m, hipGetLastError());
        return FM_OK;
    }
    int64_t* sums = nullptr;
    FM_TRY(fm_dev_alloc(m, (void**)&sums, (size_t)ntiles * sizeof(int64_t)));
    hipLaunchKernelGGL(k_scan_sums, dim3((unsigned)ntiles), dim3(SCAN_T), 0, st, (const int64_t*)d, n, sums);
    FM_HIP(m, hipGetLastError());
    int rc = fm_scan_exclusive_i64(m, sums, ntiles, st);
    if (rc == FM_OK) {
        hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)ntiles), dim3(SCAN_T), 0, st, d, n, (const int64_t*)sums);
        if (hipGetLastError() != hipSuccess) rc = fm_fail(m, FM_EHIP, "scan apply launch failed");
    }
    fm_spend(m, {sums});
    return rc;
}

// Stable sort of n keys by their low `bits`, with NV arrays of values beside them, from `in` (left as it is) into `out`.
// tmp: a second set of arrays where bits > 8.  out.key may be null if nobody reads the sorted keys and bits <= 8.
// counted: null, or room for 256 counts a tile (sort_hist) that holds those of the first digit.
static int64_t sort_tiles(int64_t n) { return (n + RS_TILE - 1) / RS_TILE; }
static int sort_bins(int bits) { return bits > 8 ? 256 : 1 << bits; }  // of the first digit
static int sort_hist(fm_matrix* m, int64_t n, int64_t** hist)
{
    return fm_dev_alloc(m, (void**)hist, (size_t)(256 * sort_tiles(n)) * sizeof(int64_t));
}
template <int NV>
static int sort_pairs(fm_matrix* m, const SortIn& in, const SortOut& out, const SortOut& tmp, int64_t n, int bits, hipStream_t st,
                      int64_t* counted = nullptr)
{
    if (n <= 0) return FM_OK;
    const int passes = std::max(1, (bits + 7) / 8);
    const int64_t nblocks = sort_tiles(n);
    int64_t* hist = counted;
    if (hist == nullptr) FM_TRY(sort_hist(m, n, &hist));
    int rc = FM_OK;
    SortIn from = in;
    for (int k = 0; k < passes && rc == FM_OK; ++k) {
        const SortOut& to = (passes - 1 - k) % 2 == 0 ? out : tmp;
        const int shift = 8 * k, nbins = k < passes - 1 ? 256 : 1 << std::max(bits - shift, 0);
        if (k > 0 || counted == nullptr) {
            hipLaunchKernelGGL(k_radix_hist, dim3((unsigned)nblocks), dim3(RS_T), 0, st, from.key, n, shift, nbins, hist, nblocks);
            if (hipGetLastError() != hipSuccess) { rc = fm_fail(m, FM_EHIP, "radix hist launch failed"); break; }
        }
        rc = fm_scan_exclusive_i64(m, hist, nbins * nblocks, st);
        if (rc != FM_OK) break;
        hipLaunchKernelGGL(k_radix_scatter<NV>, dim3((unsigned)nblocks), dim3(RS_T), 0, st, from, to, n, shift, nbins,
                           (const int64_t*)hist, nblocks);
        if (hipGetLastError() != hipSuccess) { rc = fm_fail(m, FM_EHIP, "radix scatter launch failed"); break; }
        from.key = to.key;
        for (int a = 0; a < RS_VALUES; ++a) from.v[a] = to.v[a];
    }
    fm_spend(m, {hist});
    return rc;
}

int fm_sort_by_key_u32(fm_matrix* m, uint32_t* keys, uint32_t* idx, uint32_t* keys_alt, uint32_t* idx_alt, int64_t n, int bits,
                       hipStream_t st, bool* result_in_alt)
{
    // the last pass ends in `out`; the first reads keys and idx, which the second may overwrite
    const bool odd = std::max(1, (bits + 7) / 8) % 2 == 1;
    const SortOut a = {keys, {idx, nullptr, nullptr}}, b = {keys_alt, {idx_alt, nullptr, nullptr}};
    *result_in_alt = odd && n > 0;
    return sort_pairs<1>(m, SortIn{keys, {idx, nullptr, nullptr}}, odd ? b : a, odd ? a : b, n, bits, st);
}


// List of the non-empty columns with at most `seg` entries.  ptr[c], ptr[c+1] bound the entries of list
// position c, ids[c] is its column (nullptr: c itself); per stratum when nstrata > 1: h_bounds[s] is the
// first position of stratum s and h_short_off[s] where it starts in the short list.  Every listed column comes with its
// first entry and its length, so that a kernel asks for all three at once.  Two steps: the count, which arrives in out->nshort
// with the next fm_settle, and the list; h_short_off arrives with the one behind it.
static int count_short_list(fm_matrix* m, const int64_t* ptr, const int32_t* ids, int64_t ncols_total, int32_t nstrata, int seg,
                            LongIndex* out, int64_t** tc, hipStream_t st)
{
    out->nshort = 0;
    out->h_short_off.assign(nstrata + 1, 0);
    *tc = nullptr;
    if (ncols_total <= 0) return FM_OK;
    const int64_t ntiles = (ncols_total + LI_TILE - 1) / LI_TILE;
    FM_TRY(fm_dev_alloc(m, (void**)tc, (size_t)(ntiles + 1) * sizeof(int64_t)));
    FM_HIP(m, hipMemsetAsync(*tc, 0, (size_t)(ntiles + 1) * sizeof(int64_t), st));
    hipLaunchKernelGGL(k_short_list, dim3((unsigned)ntiles), dim3(LI_T), 0, st, ptr, ncols_total, ids, seg, 0, *tc,
                       (int32_t*)nullptr, (int64_t*)nullptr, (int64_t*)nullptr, (int32_t*)nullptr);
    FM_HIP(m, hipGetLastError());
    FM_TRY(fm_scan_exclusive_i64(m, *tc, ntiles + 1, st));
    return fm_read_later(m, &out->nshort, *tc + ntiles, sizeof(int64_t), st);
}

static int fill_short_list(fm_matrix* m, const int64_t* ptr, const int32_t* ids, int64_t ncols_total,
                           const std::vector<int64_t>& h_bounds, int32_t nstrata, int seg, LongIndex* out, int64_t* tc, hipStream_t st)
{
    const int64_t n = out->nshort;
    if (n > 0) {
        const int64_t ntiles = (ncols_total + LI_TILE - 1) / LI_TILE;
        int64_t *vcol = nullptr, *d_off = nullptr, *d_bounds = nullptr;
        FM_TRY(fm_dev_alloc(m, (void**)&out->short_col, (size_t)n * sizeof(int32_t)));
        FM_TRY(fm_dev_alloc(m, (void**)&out->short_beg, (size_t)n * sizeof(int64_t)));
        FM_TRY(fm_dev_alloc(m, (void**)&out->short_len, (size_t)n * sizeof(int32_t)));
        FM_TRY(fm_dev_alloc(m, (void**)&vcol, (size_t)n * sizeof(int64_t)));
        FM_TRY(fm_dev_alloc(m, (void**)&d_off, (size_t)(nstrata + 1) * sizeof(int64_t)));
        FM_TRY(fm_dev_alloc(m, (void**)&d_bounds, (size_t)(nstrata + 1) * sizeof(int64_t)));
        FM_TRY(fm_send(m, d_bounds, h_bounds.data(), (size_t)(nstrata + 1) * sizeof(int64_t), st));
        hipLaunchKernelGGL(k_short_list, dim3((unsigned)ntiles), dim3(LI_T), 0, st, ptr, ncols_total, ids, seg, 1, tc,
                           out->short_col, vcol, out->short_beg, out->short_len);
        FM_HIP(m, hipGetLastError());
        hipLaunchKernelGGL(k_stratum_offsets, dim3(blocks_for(nstrata + 1, 256)), dim3(256), 0, st, (const int64_t*)vcol,
                           n, (const int64_t*)d_bounds, nstrata, d_off);
        FM_HIP(m, hipGetLastError());
        FM_TRY(fm_read_later(m, out->h_short_off.data(), d_off, (size_t)(nstrata + 1) * sizeof(int64_t), st));
        fm_spend(m, {vcol, d_off, d_bounds});
    }
    fm_spend(m, {tc});
    return FM_OK;
}

// Columns with very many items get a workgroup each in the finish step: their list, stratum by stratum.
static int build_vlong_list(fm_matrix* m, const std::vector<int64_t>& h_first, LongIndex* out, hipStream_t st)
{
    std::vector<int32_t> h_vlong;
    out->h_vlong_off.assign(out->h_long_off.size(), 0);
    for (size_t s = 0; s + 1 < out->h_long_off.size(); ++s) {
        for (int64_t lc = out->h_long_off[s]; lc < out->h_long_off[s + 1]; ++lc)
            if (h_first[(size_t)lc + 1] - h_first[(size_t)lc] > m->tune.vlong) h_vlong.push_back((int32_t)lc);
        out->h_vlong_off[s + 1] = (int64_t)h_vlong.size();
    }
    out->nvlong = (int64_t)h_vlong.size();
    if (out->nvlong == 0) return FM_OK;
    FM_TRY(fm_dev_alloc(m, (void**)&out->vlong, h_vlong.size() * sizeof(int32_t)));
    return fm_send(m, out->vlong, h_vlong.data(), h_vlong.size() * sizeof(int32_t), st);
}

// The long columns that a workgroup sums whole, stratum by stratum.
static int build_big_list(fm_matrix* m, const std::vector<int32_t>& h_len, LongIndex* out, hipStream_t st)
{
    std::vector<int32_t> h_big;
    out->h_big_off.assign(out->h_long_off.size(), 0);
    for (size_t s = 0; s + 1 < out->h_long_off.size(); ++s) {
        for (int64_t lc = out->h_long_off[s]; lc < out->h_long_off[s + 1]; ++lc)
            if (h_len[(size_t)lc] > FM_WHOLE_WAVE) h_big.push_back((int32_t)lc);
        out->h_big_off[s + 1] = (int64_t)h_big.size();
    }
    if (h_big.empty()) return FM_OK;
    FM_TRY(fm_dev_alloc(m, (void**)&out->big, h_big.size() * sizeof(int32_t)));
    return fm_send(m, out->big, h_big.data(), h_big.size() * sizeof(int32_t), st);
}

// Processing order of the items of a stratum or batch: by first row, so that the items of different columns that gather
// the same rows are worked on at the same time by one workgroup.  In column order they lay a column of items apart, and
// whether they met in the L2 of one XCD hung on that number of items: a table of 64 columns, K=32, 16 strata took 2.32 ms
// at 1e6 rows with items of 256 entries, 3.10 with items of 64, 3.60 and 3.52 at 1.2e6 rows; by row it takes 2.17 and 2.45.
// Mini-batch epoch of the click-style workload (2.5e6 rows): 4.17 -> 3.60 ms.  Below 2^16 rows the aggregates are found in
// a cache in any order (text-like workload, 5e4 rows, 32 strata: 847 us both ways; table of 1e5 rows, K=32: 276 -> 250 us)
// and a partition is spared the sort.
constexpr int64_t FM_ROW_ORDER_MIN = 1 << 16;
static int order_by_row(fm_matrix* m, const int32_t* row, int32_t nstrata, LongIndex* out, hipStream_t st)
{
    if (m->N < FM_ROW_ORDER_MIN) return FM_OK;
    const int64_t n = out->nitems;
    const int strat_bits = bits_for(nstrata - 1);  // at most 20
    const int row_bits_all = bits_for(m->N - 1);
    // coarser rows where the key would need a fourth pass of the sort
    const int row_bits = std::min(row_bits_all, std::max(24 - strat_bits, 8));
    uint32_t *k0 = nullptr, *i0 = nullptr, *k1 = nullptr, *i1 = nullptr;
    int64_t* d_off = nullptr;
    FM_TRY(fm_dev_alloc(m, (void**)&k0, (size_t)n * 4));
    FM_TRY(fm_dev_alloc(m, (void**)&i0, (size_t)n * 4));
    FM_TRY(fm_dev_alloc(m, (void**)&k1, (size_t)n * 4));
    FM_TRY(fm_dev_alloc(m, (void**)&i1, (size_t)n * 4));
    FM_TRY(fm_dev_alloc(m, (void**)&d_off, (size_t)(nstrata + 1) * sizeof(int64_t)));
    FM_TRY(fm_dev_alloc(m, (void**)&out->ord_beg, (size_t)n * sizeof(int64_t)));
    FM_TRY(fm_dev_alloc(m, (void**)&out->ord_len, (size_t)n * sizeof(int32_t)));
    FM_TRY(fm_send(m, d_off, out->h_item_off.data(), (size_t)(nstrata + 1) * sizeof(int64_t), st));
    hipLaunchKernelGGL(k_row_keys, dim3(blocks_for(n, 256)), dim3(256), 0, st, (const int64_t*)out->item_beg, n, row,
                       (const int64_t*)d_off, nstrata, row_bits_all - row_bits, row_bits, k0, i0);
    FM_HIP(m, hipGetLastError());
    bool alt = false;
    FM_TRY(fm_sort_by_key_u32(m, k0, i0, k1, i1, n, strat_bits + row_bits, st, &alt));
    out->order = alt ? i1 : i0;
    hipLaunchKernelGGL(k_order_items, dim3(blocks_for(n, 256)), dim3(256), 0, st, (const uint32_t*)out->order, n,
                       (const int64_t*)out->item_beg, (const int32_t*)out->item_len, out->ord_beg, out->ord_len);
    FM_HIP(m, hipGetLastError());
    fm_spend(m, {k0, k1, alt ? i0 : i1, d_off, out->item_beg, out->item_len});
    out->item_beg = nullptr;
    out->item_len = nullptr;
    return FM_OK;
}

int fm_build_long_index(fm_matrix* m, const int64_t* ptr, const int32_t* ids, const int32_t* row, int64_t ncols_total,
                        const std::vector<int64_t>& h_bounds, int32_t nstrata, LongIndex* out, hipStream_t st)
{
    out->nshort = 0;
    out->h_short_off.assign(nstrata + 1, 0);
    out->nlong = out->nitems = 0;
    out->h_long_off.assign(nstrata + 1, 0);
    out->h_item_off.assign(nstrata + 1, 0);
    // Not for one block (or batch), whose steps have the bits of the full-gradient epoch's; who sets an item length gets items.
    out->whole = nstrata > 1 && m->tune.seg <= 0 && (m->N + nstrata - 1) / nstrata <= FM_WHOLE_ROWS;
    if (ncols_total <= 0) return FM_OK;
    const int64_t ntiles = (ncols_total + LI_TILE - 1) / LI_TILE;
    int64_t *tl = nullptr, *ti = nullptr;
    FM_TRY(fm_dev_alloc(m, (void**)&tl, (size_t)(ntiles + 1) * sizeof(int64_t)));
    FM_TRY(fm_dev_alloc(m, (void**)&ti, (size_t)(ntiles + 1) * sizeof(int64_t)));
    const int seg = m->tune.seg > 0 ? m->tune.seg : fm_item_length(m->nnz / nstrata, nstrata > 1);
    int64_t* tc = nullptr;
    FM_TRY(count_short_list(m, ptr, ids, ncols_total, nstrata, seg, out, &tc, st));
    FM_HIP(m, hipMemsetAsync(tl, 0, (size_t)(ntiles + 1) * sizeof(int64_t), st));
    FM_HIP(m, hipMemsetAsync(ti, 0, (size_t)(ntiles + 1) * sizeof(int64_t), st));
    hipLaunchKernelGGL(k_long_count, dim3((unsigned)ntiles), dim3(LI_T), 0, st, ptr, ncols_total, seg, tl, ti);
    FM_HIP(m, hipGetLastError());
    FM_TRY(fm_scan_exclusive_i64(m, tl, ntiles + 1, st));
    FM_TRY(fm_scan_exclusive_i64(m, ti, ntiles + 1, st));
    int64_t nlong = 0, nitems = 0;
    FM_TRY(fm_read_later(m, &nlong, tl + ntiles, sizeof(int64_t), st));
    FM_TRY(fm_read_later(m, &nitems, ti + ntiles, sizeof(int64_t), st));
    FM_TRY(fm_settle(m, st));
    FM_TRY(fill_short_list(m, ptr, ids, ncols_total, h_bounds, nstrata, seg, out, tc, st));
    out->nlong = nlong;
    out->nitems = nitems;
    if (nlong > 0) {
        int64_t* vcol = nullptr;
        FM_TRY(fm_dev_alloc(m, (void**)&out->long_col, (size_t)nlong * sizeof(int32_t)));
        FM_TRY(fm_dev_alloc(m, (void**)&out->long_first, (size_t)(nlong + 1) * sizeof(int64_t)));
        FM_TRY(fm_dev_alloc(m, (void**)&out->item_col, (size_t)nitems * sizeof(int32_t)));
        FM_TRY(fm_dev_alloc(m, (void**)&out->item_beg, (size_t)nitems * sizeof(int64_t)));
        FM_TRY(fm_dev_alloc(m, (void**)&out->item_len, (size_t)nitems * sizeof(int32_t)));
        FM_TRY(fm_dev_alloc(m, (void**)&vcol, (size_t)nlong * sizeof(int64_t)));
        if (out->whole) {
            FM_TRY(fm_dev_alloc(m, (void**)&out->long_beg, (size_t)nlong * sizeof(int64_t)));
            FM_TRY(fm_dev_alloc(m, (void**)&out->long_len, (size_t)nlong * sizeof(int32_t)));
        }
        hipLaunchKernelGGL(k_long_fill, dim3((unsigned)ntiles), dim3(LI_T), 0, st, ptr, ncols_total, ids, seg,
                           (const int64_t*)tl, (const int64_t*)ti, out->long_col, vcol, out->long_first);
        FM_HIP(m, hipGetLastError());
        FM_TRY(fm_send(m, out->long_first + nlong, &nitems, sizeof(int64_t), st));
        hipLaunchKernelGGL(k_items, dim3(blocks_for(nlong, 4)), dim3(256), 0, st, ptr, (const int32_t*)out->long_col,
                           (const int64_t*)vcol, (const int64_t*)out->long_first, nlong, seg, out->item_col, out->item_beg,
                           out->item_len, out->long_beg, out->long_len);
        FM_HIP(m, hipGetLastError());
        std::vector<int64_t> h_vcol((size_t)nlong), h_first((size_t)nlong + 1);
        std::vector<int32_t> h_len(out->whole ? (size_t)nlong : 0);
        FM_TRY(fm_read_later(m, h_vcol.data(), vcol, (size_t)nlong * sizeof(int64_t), st));
        FM_TRY(fm_read_later(m, h_first.data(), out->long_first, (size_t)(nlong + 1) * sizeof(int64_t), st));
        FM_TRY(fm_read_later(m, h_len.data(), out->long_len, h_len.size() * sizeof(int32_t), st));
        FM_TRY(fm_settle(m, st));
        // per-stratum ranges of the concatenated lists
        int64_t k = 0;
        for (int32_t s = 0; s <= nstrata; ++s) {
            while (k < nlong && h_vcol[(size_t)k] < h_bounds[(size_t)s]) ++k;
            out->h_long_off[s] = k;
            out->h_item_off[s] = h_first[(size_t)k];
        }
        fm_spend(m, {vcol});
        FM_TRY(build_vlong_list(m, h_first, out, st));
        if (out->whole) FM_TRY(build_big_list(m, h_len, out, st));
        FM_TRY(order_by_row(m, row, nstrata, out, st));
    }
    fm_spend(m, {tl, ti});
    return FM_OK;
}

// What a build allocates belongs to the handle once the build has settled; of one that fails (no memory, a launch refused)
// nothing stays, and the handle is as it was before.
struct BuildScope {
    fm_matrix* m;
    std::vector<FmAlloc> before;
    bool done = false;
    explicit BuildScope(fm_matrix* m_) : m(m_), before(m_->allocs) {}
    ~BuildScope()
    {
        if (done) return;
        (void)hipDeviceSynchronize();
        fm_unsettled(m);
        for (size_t i = m->allocs.size(); i-- > 0;) {
            void* p = m->allocs[i].p;
            const bool older = std::any_of(before.begin(), before.end(), [p](const FmAlloc& a) { return a.p == p; });
            if (!older) fm_dev_free(m, p);
        }
    }
};

// Frees the device arrays of an index and resets it.
static void free_long_index(fm_matrix* m, LongIndex* li)
{
    for (void* p : {(void*)li->long_col, (void*)li->long_first, (void*)li->item_col, (void*)li->item_beg,
                    (void*)li->item_len, (void*)li->short_col, (void*)li->short_beg, (void*)li->short_len, (void*)li->order, (void*)li->ord_beg,
                    (void*)li->ord_len, (void*)li->tile_ptr, (void*)li->vlong, (void*)li->long_beg, (void*)li->long_len, (void*)li->big})
        if (p != nullptr) fm_dev_free(m, p);
    *li = LongIndex();
}

// Entries per item when nobody has set it: a run is a serial chain of rounds of 16 entries, so items are as short as
// still fills the chip (8 groups of 8 lanes per wavefront, 16 wavefronts on each of 256 compute units) once over; below
// 32 the partial sums (one row per item) would cost as much as the entries, above 256 nothing is gained, and 256 only by
// launches that fill the chip twice over (gradients of 256 / 128: text-like 1.2e7 entries, K = 16 157 / 151 us, K = 64 307 / 299;
// click-style 1e7, K = 16 141 / 134; 3.9e7 511 / 513; hashed 3.2e7, K = 64 1403 / 1411).
// A stratum or batch (part of the matrix) has no panels: its items are worked on by their first rows, and the shorter they are
// the fewer rows are in flight and the more of their lines are shared (click-style, K = 16, items of 128 or 256 / 64 / 48 /
// 32: strata of 6.1e6 entries 27.3 / 26.9 / 26.6 / 26.6 ms, batches of 6.1e6 2568 / 2489 / 2468 / 2498 us, of 3e6, K = 8
// - / 1236 / 1221 / 1261, strata of 1.2e7 4596 / 4365 / - / -; hashed batches of 2e6, K = 64 1573 / 1580 / 1596 / 1613).
int fm_item_length(int64_t entries, bool part)
{
    constexpr int64_t FILL = 8 * 16 * 256;
    if (part) return entries / 64 >= FILL ? 48 : 32;
    int seg = 32;
    while (seg < 256 && entries / (2 * seg) >= (seg < 128 ? FILL : 2 * FILL)) seg *= 2;
    return seg;
}

// Shape of the LDS tiles for N rows and latent size K (K = 0: not known yet).  Explicit settings win; else two tiles must fit
// the LDS of a compute unit (1024 rows only while [G | r] of a row is at most 17 floats).  Larger tiles mean fewer items, hence
// fewer partial sums to write and read back.
void fm_tile_shape(const fm_matrix* m, int32_t K, int* tile_rows, int* tile_min, int* tile_seg)
{
    const FmTune& T = m->tune;
    const int64_t N = m->N;
    // One workgroup works on one tile: tall matrices take big tiles (fewer items, hence fewer partial sums), and shorter ones
    // none: their panels hold the rows in the L2 as well, and one launch over longer items beats three kernels on three
    // streams.  Gradients in us, with tiles of 512 (below 2^18 rows 256) and without: text-like rows, K = 16 1.4e5 197 / 145, 2e5
    // 180 / 158, 4e5 300 / 342, 1e6 516 / 568, K = 32 2e5 196 / 189, 4e5 354 / 398; click-style, K = 16 1.8e5 130 / 103, 2.6e5
    // 164 / 142, 3e5 167 / 162, 4.2e5 229 / 235, 1e6 513 / 560, K = 32 3e5 196 / 194, 4.2e5 262 / 288, 7e5 472 / 518.
    int rows = 512, dense = 8, seg = 256;
    if (K > 0 && K % 4 == 0 && K <= 16 && N >= (int64_t(1) << 21)) {
        rows = 1024, dense = 12, seg = 512;
    } else if (N < 360000) {
        dense = 0;
    }
    *tile_rows = T.tile > 0 ? (T.tile < 64 ? 64 : T.tile) : rows;
    *tile_min = T.tile_min >= 0 ? T.tile_min : dense;
    *tile_seg = T.tile_seg > 0 ? T.tile_seg : seg;
}

static int build_full_index(fm_matrix* m, const FmTune& T, LongIndex* out, hipStream_t st);

int fm_build_full_index(fm_matrix* m, int32_t K, hipStream_t st)
{
    free_long_index(m, &m->lfull);
    m->lfull_shape[0] = 0;  // no index has tiles of no rows: who finds it so builds one
    FmTune T = m->tune;
    if (T.seg <= 0) T.seg = fm_item_length(m->nnz, false);
    fm_tile_shape(m, K, &T.tile, &T.tile_min, &T.tile_seg);
    BuildScope scope(m);
    LongIndex built;
    FM_TRY(build_full_index(m, T, &built, st));
    FM_TRY(fm_settle(m, st));
    m->lfull = built;
    m->lfull_shape[0] = T.tile;
    m->lfull_shape[1] = T.tile_min;
    m->lfull_shape[2] = T.tile_seg;
    scope.done = true;
    return FM_OK;
}

static int build_full_index(fm_matrix* m, const FmTune& T, LongIndex* out, hipStream_t st)
{
    int64_t* tc = nullptr;
    FM_TRY(count_short_list(m, m->colptr, nullptr, m->D, 1, T.seg, out, &tc, st));
    out->nlong = out->nitems = 0;
    out->h_long_off.assign(2, 0);
    out->h_item_off.assign(2, 0);
    const int64_t D = m->D;
    if (D <= 0 || m->nnz == 0) {
        fm_spend(m, {tc});  // no columns with entries: none short
        return FM_OK;
    }
    // 1. the long columns, in column order
    const int64_t ntiles = (D + LI_TILE - 1) / LI_TILE;
    int64_t *tl = nullptr, *ti = nullptr, *vcol = nullptr;
    FM_TRY(fm_dev_alloc(m, (void**)&tl, (size_t)(ntiles + 1) * sizeof(int64_t)));
    FM_TRY(fm_dev_alloc(m, (void**)&ti, (size_t)(ntiles + 1) * sizeof(int64_t)));
    FM_HIP(m, hipMemsetAsync(tl, 0, (size_t)(ntiles + 1) * sizeof(int64_t), st));
    FM_HIP(m, hipMemsetAsync(ti, 0, (size_t)(ntiles + 1) * sizeof(int64_t), st));
    hipLaunchKernelGGL(k_long_count, dim3((unsigned)ntiles), dim3(LI_T), 0, st, (const int64_t*)m->colptr, D, T.seg, tl, ti);
    FM_HIP(m, hipGetLastError());
    FM_TRY(fm_scan_exclusive_i64(m, tl, ntiles + 1, st));
    int64_t nlong = 0;
    FM_TRY(fm_read_later(m, &nlong, tl + ntiles, sizeof(int64_t), st));
    FM_TRY(fm_settle(m, st));
    fm_spend(m, {tl, ti});
    FM_TRY(fill_short_list(m, m->colptr, nullptr, m->D, {0, m->D}, 1, T.seg, out, tc, st));
    if (nlong == 0) return FM_OK;
    if (nlong > 0x7fffffffLL) return fm_fail(m, FM_ERANGE, "too many long columns");
    FM_TRY(fm_dev_alloc(m, (void**)&out->long_col, (size_t)nlong * sizeof(int32_t)));
    FM_TRY(fm_dev_alloc(m, (void**)&out->long_first, (size_t)(nlong + 1) * sizeof(int64_t)));
    FM_TRY(fm_dev_alloc(m, (void**)&vcol, (size_t)nlong * sizeof(int64_t)));
    hipLaunchKernelGGL(k_long_fill, dim3((unsigned)ntiles), dim3(LI_T), 0, st, (const int64_t*)m->colptr, D,
                       (const int32_t*)nullptr, T.seg, (const int64_t*)tl, (const int64_t*)ti, out->long_col, vcol,
                       (int64_t*)nullptr);
    FM_HIP(m, hipGetLastError());
    // 2. items per long column, then their first ids
    // With a number of panels asked for, they shrink (down to 1024 rows) until there are as many.
    int64_t panel = T.panel;
    if (T.min_panels > 0)
        while (panel > 1024 && (m->N + panel - 1) / panel < T.min_panels) panel /= 2;
    else
        panel = fm_panel_rows(m->N, T.panel);
    const int64_t npanels = (m->N + panel - 1) / panel;
    const bool in_panels = T.min_panels > 0 ? npanels >= T.min_panels : m->N >= FM_PANEL_ROWS;
    out->in_panels = in_panels;
    // the density that makes a column heavy does not depend on how tall the panels are
    const double heavy_density = (double)T.heavy_per_panel / (double)T.panel;
    const int64_t heavy_min =
        in_panels ? std::max<int64_t>((int64_t)(heavy_density * (double)m->N) + 1, (int64_t)T.seg + 1) : INT64_MAX;
    const int64_t maxpos = (npanels + FM_XCDS - 1) / FM_XCDS;
    // dense-ish columns (at least tile_min entries per row tile on average) go to the LDS-staged kernel
    const int64_t tile = T.tile;
    const int64_t nrtiles = (m->N + tile - 1) / tile;
    const int64_t tile_min = (T.tile_min > 0 && nrtiles >= 2)
                                 ? std::max<int64_t>((int64_t)T.tile_min * nrtiles, (int64_t)T.seg + 1)
                                 : INT64_MAX;
    const int64_t key_tiles = (int64_t)FM_XCDS * (maxpos + 1);
    if (key_tiles + nrtiles >= (1LL << 32)) return fm_fail(m, FM_ERANGE, "too many row tiles");
    FM_HIP(m, hipMemsetAsync(out->long_first, 0, (size_t)(nlong + 1) * sizeof(int64_t), st));
    hipLaunchKernelGGL(k_full_items, dim3((unsigned)nlong), dim3(256), 0, st, (const int64_t*)m->colptr,
                       (const int32_t*)m->crow, (const int32_t*)out->long_col, m->N, T.seg, panel, heavy_min,
                       maxpos, tile, tile_min, T.tile_seg, 0, out->long_first, (const int64_t*)nullptr, (int32_t*)nullptr, (int64_t*)nullptr,
                       (int32_t*)nullptr, (uint32_t*)nullptr);
    FM_HIP(m, hipGetLastError());
    FM_TRY(fm_scan_exclusive_i64(m, out->long_first, nlong + 1, st));
    std::vector<int64_t> h_first((size_t)nlong + 1);
    FM_TRY(fm_read_later(m, h_first.data(), out->long_first, (size_t)(nlong + 1) * sizeof(int64_t), st));
    FM_TRY(fm_settle(m, st));
    const int64_t nitems = h_first[(size_t)nlong];
    if (nitems >= (1LL << 32)) return fm_fail(m, FM_ERANGE, "too many column items");
    FM_TRY(fm_dev_alloc(m, (void**)&out->item_col, (size_t)nitems * sizeof(int32_t)));
    FM_TRY(fm_dev_alloc(m, (void**)&out->item_beg, (size_t)nitems * sizeof(int64_t)));
    FM_TRY(fm_dev_alloc(m, (void**)&out->item_len, (size_t)nitems * sizeof(int32_t)));
    uint32_t *k0 = nullptr, *i0 = nullptr, *k1 = nullptr, *i1 = nullptr;
    FM_TRY(fm_dev_alloc(m, (void**)&k0, (size_t)nitems * 4));
    FM_TRY(fm_dev_alloc(m, (void**)&i0, (size_t)nitems * 4));
    FM_TRY(fm_dev_alloc(m, (void**)&k1, (size_t)nitems * 4));
    FM_TRY(fm_dev_alloc(m, (void**)&i1, (size_t)nitems * 4));
    hipLaunchKernelGGL(k_full_items, dim3((unsigned)nlong), dim3(256), 0, st, (const int64_t*)m->colptr,
                       (const int32_t*)m->crow, (const int32_t*)out->long_col, m->N, T.seg, panel, heavy_min,
                       maxpos, tile, tile_min, T.tile_seg, 1, (int64_t*)nullptr, (const int64_t*)out->long_first, out->item_col, out->item_beg,
                       out->item_len, k0);
    FM_HIP(m, hipGetLastError());
    // 3. processing order: stable sort of the item ids by (XCD list, panel position)
    hipLaunchKernelGGL(k_iota_u32, dim3(blocks_for(nitems, 256)), dim3(256), 0, st, i0, nitems);
    FM_HIP(m, hipGetLastError());
    bool alt = false;
    FM_TRY(fm_sort_by_key_u32(m, k0, i0, k1, i1, nitems, bits_for(key_tiles + nrtiles), st, &alt));
    int64_t* d_off = nullptr;
    FM_TRY(fm_dev_alloc(m, (void**)&d_off, (2 * FM_XCDS + 1) * sizeof(int64_t)));
    hipLaunchKernelGGL(k_list_offsets, dim3(1), dim3(64), 0, st, (const uint32_t*)(alt ? k1 : k0), nitems, maxpos, d_off);
    FM_HIP(m, hipGetLastError());
    int64_t h_off[2 * FM_XCDS + 1];
    FM_TRY(fm_read_later(m, h_off, d_off, sizeof(h_off), st));
    FM_TRY(fm_settle(m, st));
    for (int x = 0; x <= FM_XCDS; ++x) out->list_off[x] = h_off[x];
    for (int x = 0; x < FM_XCDS; ++x) out->list_mid[x] = h_off[FM_XCDS + 1 + x];
    out->tile_rows = tile;
    out->ntiles = 0;
    if (out->list_off[FM_XCDS] < nitems) {  // there are tile items
        out->ntiles = nrtiles;
        FM_TRY(fm_dev_alloc(m, (void**)&out->tile_ptr, (size_t)(nrtiles + 1) * sizeof(int64_t)));
        hipLaunchKernelGGL(k_tile_ptr, dim3(blocks_for(nrtiles + 1, 256)), dim3(256), 0, st,
                           (const uint32_t*)(alt ? k1 : k0), nitems, key_tiles, nrtiles, out->tile_ptr);
        FM_HIP(m, hipGetLastError());
    }
    out->order = alt ? i1 : i0;
    fm_spend(m, {alt ? i0 : i1});
    FM_TRY(fm_dev_alloc(m, (void**)&out->ord_beg, (size_t)nitems * sizeof(int64_t)));
    FM_TRY(fm_dev_alloc(m, (void**)&out->ord_len, (size_t)nitems * sizeof(int32_t)));
    hipLaunchKernelGGL(k_order_items, dim3(blocks_for(nitems, 256)), dim3(256), 0, st, (const uint32_t*)out->order,
                       nitems, (const int64_t*)out->item_beg, (const int32_t*)out->item_len, out->ord_beg,
                       out->ord_len);
    FM_HIP(m, hipGetLastError());
    fm_spend(m, {k0, k1, d_off, vcol});
    out->nlong = nlong;
    out->nitems = nitems;
    out->h_long_off[1] = nlong;
    out->h_item_off[1] = nitems;
    return build_vlong_list(m, h_first, out, st);
}

extern "C" int fm_build_csc(fm_matrix* m, void* hip_stream)
{
    if (m == nullptr) return FM_EINVAL;
    hipStream_t st = (hipStream_t)hip_stream;
    if (m->has_csc) return FM_OK;
    BuildScope scope(m);
    const int64_t n = m->nnz;
    FM_TRY(fm_dev_alloc(m, (void**)&m->colptr, (size_t)(m->D + 1) * sizeof(int64_t)));  // not read before has_csc is set
    FM_TRY(fm_dev_alloc(m, (void**)&m->crow, (size_t)(n + FM_ENTRY_PAD) * sizeof(int32_t)));
    FM_TRY(fm_dev_alloc(m, (void**)&m->cval, (size_t)(n + FM_ENTRY_PAD) * sizeof(float)));
    if (n == 0) {
        FM_HIP(m, hipMemsetAsync(m->colptr, 0, (size_t)(m->D + 1) * sizeof(int64_t), st));
    } else {
        // the columns with the row and the value of every entry, sorted by column
        const int bits = bits_for(m->D - 1);
        uint32_t *row = nullptr, *key = nullptr, *t[3] = {nullptr, nullptr, nullptr};
        FM_TRY(fm_dev_alloc(m, (void**)&row, (size_t)n * 4));
        FM_TRY(fm_dev_alloc(m, (void**)&key, (size_t)n * 4));
        if (bits > 8)
            for (uint32_t*& x : t) FM_TRY(fm_dev_alloc(m, (void**)&x, (size_t)n * 4));
        hipLaunchKernelGGL(k_owners, dim3(blocks_for(n, 256 * OWN_E)), dim3(256), 0, st, (const int64_t*)m->rowptr, m->N, n, row);
        FM_HIP(m, hipGetLastError());
        const SortIn in = {reinterpret_cast<const uint32_t*>(m->col), {row, reinterpret_cast<const uint32_t*>(m->val), nullptr}};
        const SortOut out = {key, {reinterpret_cast<uint32_t*>(m->crow), reinterpret_cast<uint32_t*>(m->cval), nullptr}};
        FM_TRY(sort_pairs<2>(m, in, out, SortOut{t[0], {t[1], t[2], nullptr}}, n, bits, st));
        hipLaunchKernelGGL(k_ptr_from_sorted, dim3(blocks_for(m->D + 1, 256)), dim3(256), 0, st, (const uint32_t*)key, n, m->D,
                           m->colptr);
        FM_HIP(m, hipGetLastError());
        fm_spend(m, {row, key, t[0], t[1], t[2]});
    }
    FM_TRY(fm_build_full_index(m, 0, st));
    scope.done = true;
    m->has_csc = true;
    fm_drop_workspace(m);
    return FM_OK;
}

static int partition_impl(fm_matrix* m, int32_t P, const int32_t* place, hipStream_t st);
static int ensure_marks(fm_matrix* m, hipStream_t st);

// One orientation of the per-stratum matrices: the entries in (stratum, major, minor) order, the list
// of the (stratum, major) pairs that hold an entry with the offset of their first one, and where every
// stratum starts in the entries (h_ent_off) and in that list (h_list_off).
// (batches: the column orientation keyed by row block alone, P = number of batches)
struct StrataSide {
    int32_t* ind = nullptr;
    float* val = nullptr;
    int32_t* nz_major = nullptr;
    int64_t* nz_beg = nullptr;  // [count + 1]
    int64_t count = 0;
    std::vector<int64_t> h_ent_off, h_list_off;  // [P + 1]
};

static int build_strata_side(fm_matrix* m, bool by_rows, const int32_t* place, hipStream_t st, StrataSide* out, int32_t P,
                             bool batches = false)
{
    const int64_t n = m->nnz;
    const int64_t nmajor = by_rows ? m->N : m->D;
    const int64_t* major = by_rows ? m->rowptr : m->colptr;
    const int32_t* minor = by_rows ? m->col : m->crow;
    const float* val = by_rows ? m->val : m->cval;
    out->h_ent_off.assign(P + 1, 0);
    out->h_list_off.assign(P + 1, 0);
    FM_TRY(fm_dev_alloc(m, (void**)&out->ind, (size_t)(n + FM_ENTRY_PAD) * sizeof(int32_t)));
    FM_TRY(fm_dev_alloc(m, (void**)&out->val, (size_t)(n + FM_ENTRY_PAD) * sizeof(float)));
    if (n == 0) {
        FM_TRY(fm_dev_alloc(m, (void**)&out->nz_major, sizeof(int32_t)));
        FM_TRY(fm_dev_alloc(m, (void**)&out->nz_beg, sizeof(int64_t)));
        FM_HIP(m, hipMemsetAsync(out->nz_beg, 0, sizeof(int64_t), st));
        return FM_OK;
    }
    const int bits = bits_for(P - 1);
    uint32_t *k0 = nullptr, *j0 = nullptr, *keys = nullptr, *maj = nullptr, *t[4] = {nullptr, nullptr, nullptr, nullptr};
    for (uint32_t** x : {&k0, &j0, &keys, &maj}) FM_TRY(fm_dev_alloc(m, (void**)x, (size_t)n * 4));
    if (bits > 8)
        for (uint32_t*& x : t) FM_TRY(fm_dev_alloc(m, (void**)&x, (size_t)n * 4));
    int64_t* hist = nullptr;
    FM_TRY(sort_hist(m, n, &hist));
    hipLaunchKernelGGL(k_stratum_keys, dim3((unsigned)sort_tiles(n)), dim3(RS_T), 0, st, major, nmajor, minor, n, m->N, m->D, P,
                       batches ? 2 : (by_rows ? 1 : 0), place, k0, j0, sort_bins(bits), hist,
                       sort_tiles(n));
    FM_HIP(m, hipGetLastError());
    const SortIn in = {k0, {reinterpret_cast<const uint32_t*>(minor), reinterpret_cast<const uint32_t*>(val), j0}};
    const SortOut sorted = {keys, {reinterpret_cast<uint32_t*>(out->ind), reinterpret_cast<uint32_t*>(out->val), maj}};
    FM_TRY(sort_pairs<3>(m, in, sorted, SortOut{t[0], {t[1], t[2], t[3]}}, n, bits, st, hist));
    // the stable sort keeps the entries of a stratum in the order of the source (by major index): the
    // (stratum, major) pairs are runs, found by comparing neighbours
    const int64_t htiles = (n + HD_TILE - 1) / HD_TILE;
    int64_t* pos = nullptr;
    FM_TRY(fm_dev_alloc(m, (void**)&pos, (size_t)(htiles + 1) * sizeof(int64_t)));
    FM_HIP(m, hipMemsetAsync(pos + htiles, 0, sizeof(int64_t), st));
    hipLaunchKernelGGL(k_heads, dim3((unsigned)htiles), dim3(256), 0, st, (const uint32_t*)keys, (const uint32_t*)maj, n, 0, pos,
                       (int32_t*)nullptr, (int64_t*)nullptr);
    FM_HIP(m, hipGetLastError());
    FM_TRY(fm_scan_exclusive_i64(m, pos, htiles + 1, st));
    int64_t count = 0;
    FM_TRY(fm_read_later(m, &count, pos + htiles, sizeof(int64_t), st));
    FM_TRY(fm_settle(m, st));
    out->count = count;
    FM_TRY(fm_dev_alloc(m, (void**)&out->nz_major, (size_t)count * sizeof(int32_t)));
    FM_TRY(fm_dev_alloc(m, (void**)&out->nz_beg, (size_t)(count + 1) * sizeof(int64_t)));
    hipLaunchKernelGGL(k_heads, dim3((unsigned)htiles), dim3(256), 0, st, (const uint32_t*)keys, (const uint32_t*)maj, n, 1, pos,
                       out->nz_major, out->nz_beg);
    FM_HIP(m, hipGetLastError());
    FM_TRY(fm_send(m, out->nz_beg + count, &n, sizeof(int64_t), st));
    // where every stratum starts: in the entries (keys smaller than s), then in the list of pairs
    int64_t *d_ent = nullptr, *d_list = nullptr;
    FM_TRY(fm_dev_alloc(m, (void**)&d_ent, (size_t)(P + 1) * sizeof(int64_t)));
    FM_TRY(fm_dev_alloc(m, (void**)&d_list, (size_t)(P + 1) * sizeof(int64_t)));
    hipLaunchKernelGGL(k_ptr_from_sorted, dim3(blocks_for(P + 1, 256)), dim3(256), 0, st, (const uint32_t*)keys, n, (int64_t)P, d_ent);
    FM_HIP(m, hipGetLastError());
    hipLaunchKernelGGL(k_lower_bounds, dim3(blocks_for(P + 1, 256)), dim3(256), 0, st, (const int64_t*)out->nz_beg, count,
                       (const int64_t*)d_ent, (int64_t)(P + 1), d_list);
    FM_HIP(m, hipGetLastError());
    FM_TRY(fm_read_later(m, out->h_ent_off.data(), d_ent, (size_t)(P + 1) * sizeof(int64_t), st));
    FM_TRY(fm_read_later(m, out->h_list_off.data(), d_list, (size_t)(P + 1) * sizeof(int64_t), st));
    fm_spend(m, {k0, j0, keys, maj, t[0], t[1], t[2], t[3], pos, d_ent, d_list});
    return FM_OK;
}

extern "C" int fm_partition(fm_matrix* m, int32_t P, void* hip_stream)
{
    if (m == nullptr) return FM_EINVAL;
    return partition_impl(m, P, nullptr, (hipStream_t)hip_stream);
}

extern "C" int fm_partition_placed(fm_matrix* m, int32_t P, const int32_t* place, void* hip_stream)
{
    if (m == nullptr) return FM_EINVAL;
    if (place == nullptr) return fm_fail(m, FM_EINVAL, "place is NULL");
    for (int64_t j = 0; j < m->D; ++j)
        if (place[j] < 0 || place[j] >= P)
            return fm_fail(m, FM_ERANGE, "place[%lld] = %d outside [0,%d)", (long long)j, place[j], P);
    return partition_impl(m, P, place, (hipStream_t)hip_stream);
}

static int partition_impl(fm_matrix* m, int32_t P, const int32_t* place, hipStream_t st)
{
    if (!m->has_csc) return fm_fail(m, FM_ESTATE, "fm_partition needs fm_build_csc first");
    if (P < 1 || P > FM_MAXP) return fm_fail(m, FM_EINVAL, "P=%d outside 1..%d", P, FM_MAXP);
    if (m->P != 0) return fm_fail(m, FM_ESTATE, "matrix is already partitioned (P=%d)", m->P);
    if (m->N < 1 || m->D < 1) return fm_fail(m, FM_EINVAL, "cannot partition an empty matrix");
    FM_TRY(fm_ensure_lazy(m, st));
    FM_TRY(ensure_marks(m, st));
    BuildScope scope(m);
    std::vector<int64_t> h_rb((size_t)P + 1), h_cb((size_t)P + 1), h_cell_nnz;
    for (int32_t b = 0; b <= P; ++b) {
        h_rb[b] = (int64_t)(((__int128)b * (__int128)m->N) / (__int128)P);
        h_cb[b] = (int64_t)(((__int128)b * (__int128)m->D) / (__int128)P);
    }
    std::vector<float> h_rho((size_t)P);
    for (int32_t b = 0; b < P; ++b) h_rho[b] = (float)((double)(h_rb[b + 1] - h_rb[b]) / (double)m->N);
    float* d_rho = nullptr;
    int64_t* d_rb = nullptr;
    int32_t* d_place = nullptr;
    FM_TRY(fm_dev_alloc(m, (void**)&d_rho, (size_t)P * sizeof(float)));
    FM_TRY(fm_send(m, d_rho, h_rho.data(), (size_t)P * sizeof(float), st));
    FM_TRY(fm_dev_alloc(m, (void**)&d_rb, (size_t)(P + 1) * sizeof(int64_t)));
    FM_TRY(fm_send(m, d_rb, h_rb.data(), (size_t)(P + 1) * sizeof(int64_t), st));
    if (place != nullptr) {
        FM_TRY(fm_dev_alloc(m, (void**)&d_place, (size_t)m->D * sizeof(int32_t)));
        FM_TRY(fm_send(m, d_place, place, (size_t)m->D * sizeof(int32_t), st));
    }

    StrataSide rows, cols;
    FM_TRY(build_strata_side(m, true, d_place, st, &rows, P));
    FM_TRY(fm_settle(m, st));  // its scratch serves the other side
    FM_TRY(build_strata_side(m, false, d_place, st, &cols, P));
    FM_TRY(fm_settle(m, st));

    // cell table (row block, column block or worker the column started at)
    if (P <= FM_MAXP_CELLS) {
        h_cell_nnz.assign((size_t)P * P, 0);
        if (m->nnz > 0) {
            int64_t *d_cell = nullptr, *d_off = nullptr;
            FM_TRY(fm_dev_alloc(m, (void**)&d_cell, (size_t)P * P * sizeof(int64_t)));
            FM_TRY(fm_dev_alloc(m, (void**)&d_off, (size_t)(P + 1) * sizeof(int64_t)));
            FM_TRY(fm_send(m, d_off, rows.h_list_off.data(), (size_t)(P + 1) * sizeof(int64_t), st));
            hipLaunchKernelGGL(k_cell_table, dim3(blocks_for((int64_t)P * P, 256)), dim3(256), 0, st,
                               (const int32_t*)rows.nz_major, (const int64_t*)rows.nz_beg, (const int64_t*)d_off,
                               (const int64_t*)d_rb, P, d_cell);
            FM_HIP(m, hipGetLastError());
            FM_TRY(fm_read_later(m, h_cell_nnz.data(), d_cell, (size_t)P * P * sizeof(int64_t), st));
            fm_spend(m, {d_cell, d_off});
        }
    }
    LongIndex strata;
    FM_TRY(fm_build_long_index(m, cols.nz_beg, cols.nz_major, cols.ind, cols.count, cols.h_list_off, P, &strata, st));
    FM_TRY(fm_settle(m, st));
    scope.done = true;
    m->P = P;
    m->h_rb = h_rb;
    m->h_cb = h_cb;
    m->d_rho = d_rho;
    m->d_rb = d_rb;
    m->d_place = d_place;
    m->s_col = rows.ind;
    m->s_val = rows.val;
    // the rows that have an entry in stratum s: its refresh visits only these (a row's entries end
    // where those of the next listed row begin)
    m->s_touched = rows.nz_major;
    m->s_touched_beg = rows.nz_beg;
    m->ntouched = rows.count;
    m->h_touch_off = rows.h_list_off;
    m->s_row = cols.ind;
    m->s_cval = cols.val;
    m->s_ncol = cols.nz_major;
    m->s_ncol_beg = cols.nz_beg;
    m->nncol = cols.count;
    m->h_ncol_off = cols.h_list_off;
    m->h_strat_nnz_off = cols.h_ent_off;
    m->h_cell_nnz = std::move(h_cell_nnz);
    m->lstrat = strata;
    fm_drop_workspace(m);
    return FM_OK;
}

int fm_ensure_lazy(fm_matrix* m, hipStream_t st)
{
    if (m->lazy_last != nullptr) return FM_OK;
    FM_TRY(fm_dev_alloc(m, (void**)&m->lazy_last, (size_t)std::max<int64_t>(m->D, 1) * sizeof(int32_t)));
    FM_TRY(fm_fill_i32(m, m->lazy_last, m->D, 0, st));  // the callers wait for the stream
    m->lazy_clear = true;
    return FM_OK;
}

static int ensure_marks(fm_matrix* m, hipStream_t st)
{
    if (m->col_mark != nullptr) return FM_OK;
    int32_t* marks = nullptr;
    FM_TRY(fm_dev_alloc(m, (void**)&marks, (size_t)m->D * sizeof(int32_t)));
    FM_HIP(m, hipMemsetAsync(marks, 0, (size_t)m->D * sizeof(int32_t), st));  // the callers wait for the stream
    m->col_mark = marks;
    return FM_OK;
}

extern "C" int fm_partition_batches(fm_matrix* m, int32_t B, void* hip_stream)
{
    if (m == nullptr) return FM_EINVAL;
    hipStream_t st = (hipStream_t)hip_stream;
    if (!m->has_csc) return fm_fail(m, FM_ESTATE, "fm_partition_batches needs fm_build_csc first");
    if (B < 1 || B > FM_MAXP) return fm_fail(m, FM_EINVAL, "B=%d outside 1..%d", B, FM_MAXP);
    if (m->B != 0) return fm_fail(m, FM_ESTATE, "row batches are already built (B=%d)", m->B);
    if (m->N < 1 || m->D < 1) return fm_fail(m, FM_EINVAL, "cannot split an empty matrix");
    FM_TRY(fm_ensure_lazy(m, st));
    FM_TRY(ensure_marks(m, st));
    BuildScope scope(m);
    std::vector<int64_t> h_bb((size_t)B + 1);
    std::vector<float> h_rho((size_t)B);
    for (int32_t b = 0; b <= B; ++b) h_bb[b] = (int64_t)(((__int128)b * (__int128)m->N) / (__int128)B);
    for (int32_t b = 0; b < B; ++b) h_rho[b] = (float)((double)(h_bb[b + 1] - h_bb[b]) / (double)m->N);
    float* d_rho = nullptr;
    int64_t* d_bb = nullptr;
    FM_TRY(fm_dev_alloc(m, (void**)&d_rho, (size_t)B * sizeof(float)));
    FM_TRY(fm_send(m, d_rho, h_rho.data(), (size_t)B * sizeof(float), st));
    FM_TRY(fm_dev_alloc(m, (void**)&d_bb, (size_t)(B + 1) * sizeof(int64_t)));
    FM_TRY(fm_send(m, d_bb, h_bb.data(), (size_t)(B + 1) * sizeof(int64_t), st));
    StrataSide cols;
    FM_TRY(build_strata_side(m, false, nullptr, st, &cols, B, true));
    FM_TRY(fm_settle(m, st));
    LongIndex batches;
    FM_TRY(fm_build_long_index(m, cols.nz_beg, cols.nz_major, cols.ind, cols.count, cols.h_list_off, B, &batches, st));
    FM_TRY(fm_settle(m, st));
    scope.done = true;
    m->B = B;
    m->h_bb = h_bb;
    m->d_brho = d_rho;
    m->d_bb = d_bb;
    m->b_row = cols.ind;
    m->b_cval = cols.val;
    m->b_ncol = cols.nz_major;
    m->b_ncol_beg = cols.nz_beg;
    m->nbcol = cols.count;
    m->h_bcol_off = cols.h_list_off;
    m->h_batch_nnz_off = cols.h_ent_off;
    m->lbatch = batches;
    fm_drop_workspace(m);
    return FM_OK;
}
