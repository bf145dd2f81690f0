// C-ABI entry points and the epoch drivers.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <utility>

#include "fm_internal.h"
#include "fm_upload.h"

static thread_local std::string g_build_error;

int fm_fail(fm_matrix* m, int code, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    if (m != nullptr) m->err = buf; else g_build_error = buf;
    return code;
}

// Device blocks that handles have given back, kept for the next handle.  A scoring service makes and destroys a handle
// per batch of requests and a build makes and frees gigabytes of scratch: mapping and unmapping that memory cost 8 ms
// of the 60 ms that opening a data set of 4.9e7 entries took.  Blocks come back idle (see fm_dev_free), so any thread
// and stream may take them.  Bounded to POOL_CAP per process; all of it goes back to the driver when an allocation
// fails or the program calls fm_trim.  Requests up to POOL_MIN are left to the runtime, which hands them out of its own chunks in under a microsecond.
namespace {
constexpr size_t POOL_MIN = size_t(1) << 20;
constexpr size_t POOL_CAP = size_t(4) << 30;
constexpr size_t POOL_PINNED_CAP = 32;  // pinned scalar blocks

struct PoolBlock {
    void* p;
    size_t bytes;
    int device;
};
std::mutex g_pool_lock;
std::vector<PoolBlock> g_pool;  // oldest first
size_t g_pool_bytes = 0;
std::vector<std::pair<int, void*>> g_pinned;

// Sizes are rounded so that a block fits the next request of about the same size: to 1/16 of the power of two below.
size_t pool_round(size_t bytes)
{
    size_t unit = size_t(1) << 16;
    while (unit * 32 <= bytes) unit <<= 1;
    return (bytes + unit - 1) / unit * unit;
}

void pool_drain()
{
    std::vector<PoolBlock> all;
    {
        std::lock_guard<std::mutex> g(g_pool_lock);
        all.swap(g_pool);
        g_pool_bytes = 0;
    }
    for (const PoolBlock& b : all) (void)hipFree(b.p);
}

void* pool_take(size_t bytes, int device)
{
    std::lock_guard<std::mutex> g(g_pool_lock);
    for (size_t i = g_pool.size(); i-- > 0;)
        if (g_pool[i].bytes == bytes && g_pool[i].device == device) {
            void* p = g_pool[i].p;
            g_pool.erase(g_pool.begin() + (ptrdiff_t)i);
            g_pool_bytes -= bytes;
            return p;
        }
    return nullptr;
}

void pool_give(void* p, size_t bytes, int device)
{
    std::vector<void*> evicted;
    {
        std::lock_guard<std::mutex> g(g_pool_lock);
        if (bytes > POOL_CAP) {
            evicted.push_back(p);
        } else {
            while (g_pool_bytes + bytes > POOL_CAP) {
                evicted.push_back(g_pool.front().p);
                g_pool_bytes -= g_pool.front().bytes;
                g_pool.erase(g_pool.begin());
            }
            g_pool.push_back({p, bytes, device});
            g_pool_bytes += bytes;
        }
    }
    for (void* q : evicted) (void)hipFree(q);
}
}  // namespace

// On the device the handle was created on, which need not be the current one: a block returns to that device's list.
int fm_dev_alloc(fm_matrix* m, void** p, size_t bytes)
{
    *p = nullptr;
    if (bytes == 0) bytes = 16;
    const bool pooled = bytes > POOL_MIN;
    const size_t want = pooled ? pool_round(bytes) : bytes;
    if (pooled) *p = pool_take(want, m->device);
    if (*p == nullptr) {
        int current = m->device;
        const bool elsewhere = hipGetDevice(&current) == hipSuccess && current != m->device;
        if (elsewhere) (void)hipSetDevice(m->device);
        hipError_t e = hipMalloc(p, want);
        if (e != hipSuccess) {  // what the pool holds may be what is missing
            (void)hipGetLastError();
            pool_drain();
            e = hipMalloc(p, want);
        }
        if (elsewhere) (void)hipSetDevice(current);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return fm_fail(m, FM_ENOMEM, "hipMalloc of %zu bytes failed: %s", bytes, hipGetErrorString(e));
        }
    }
    m->allocs.push_back({*p, pooled ? want : 0});
    return FM_OK;
}

// No work that uses the block may be in flight on any stream: it may be handed to another handle at once.
void fm_dev_free(fm_matrix* m, void* p)
{
    if (p == nullptr) return;
    size_t bytes = 0;
    for (size_t i = m->allocs.size(); i-- > 0;)
        if (m->allocs[i].p == p) {
            bytes = m->allocs[i].pool_bytes;
            m->allocs.erase(m->allocs.begin() + (ptrdiff_t)i);
            break;
        }
    if (bytes > 0)
        pool_give(p, bytes, m->device);
    else
        (void)hipFree(p);
}

void fm_spend(fm_matrix* m, std::initializer_list<void*> scratch)
{
    for (void* p : scratch)
        if (p != nullptr) m->spent.push_back(p);
}

// Room in the pinned block for so many bytes, or nullptr.
static char* pinned_room(fm_matrix* m, size_t bytes)
{
    if (m->pin_used + bytes > (FM_PINNED_DOUBLES - 8) * sizeof(double)) return nullptr;
    char* p = reinterpret_cast<char*>(m->h_scal + 8) + m->pin_used;
    m->pin_used += (bytes + 7) / 8 * 8;
    return p;
}

// Through pinned memory: the runtime's way to and from pageable memory takes 15 us and more whatever the size.
int fm_read_later(fm_matrix* m, void* dst, const void* src, size_t bytes, hipStream_t st)
{
    if (bytes == 0) return FM_OK;
    char* pin = pinned_room(m, bytes);
    FM_HIP(m, hipMemcpyAsync(pin != nullptr ? pin : dst, src, bytes, hipMemcpyDeviceToHost, st));
    if (pin != nullptr) m->reads.push_back({dst, (size_t)(pin - reinterpret_cast<char*>(m->h_scal + 8)), bytes});
    return FM_OK;
}

int fm_send(fm_matrix* m, void* dst, const void* src, size_t bytes, hipStream_t st)
{
    if (bytes == 0) return FM_OK;
    char* pin = pinned_room(m, bytes);
    if (pin != nullptr) memcpy(pin, src, bytes);
    FM_HIP(m, hipMemcpyAsync(dst, pin != nullptr ? pin : src, bytes, hipMemcpyHostToDevice, st));
    if (pin == nullptr) FM_HIP(m, hipStreamSynchronize(st));  // src is the caller's
    return FM_OK;
}

void fm_unsettled(fm_matrix* m)
{
    if (m->reads.empty() && m->spent.empty() && m->pin_used == 0) return;
    (void)hipDeviceSynchronize();
    m->reads.clear();
    m->pin_used = 0;
    for (void* p : m->spent) fm_dev_free(m, p);
    m->spent.clear();
}

int fm_settle(fm_matrix* m, hipStream_t st)
{
    const hipError_t e = hipStreamSynchronize(st);
    if (e == hipSuccess)
        for (const FmRead& r : m->reads) memcpy(r.dst, reinterpret_cast<char*>(m->h_scal + 8) + r.at, r.bytes);
    m->reads.clear();
    m->pin_used = 0;
    if (e != hipSuccess) return fm_fail(m, FM_EHIP, "building failed: %s", hipGetErrorString(e));
    for (void* p : m->spent) fm_dev_free(m, p);
    m->spent.clear();
    return FM_OK;
}

extern "C" int fm_trim(void)
{
    pool_drain();
    std::vector<std::pair<int, void*>> pinned;
    {
        std::lock_guard<std::mutex> g(g_pool_lock);
        pinned.swap(g_pinned);
    }
    for (const auto& b : pinned) (void)hipHostFree(b.second);
    fm_ring_trim();
    return FM_OK;
}

static int pinned_alloc(fm_matrix* m)
{
    {
        std::lock_guard<std::mutex> g(g_pool_lock);
        for (size_t i = g_pinned.size(); i-- > 0;)
            if (g_pinned[i].first == m->device) {
                m->h_scal = (double*)g_pinned[i].second;
                g_pinned.erase(g_pinned.begin() + (ptrdiff_t)i);
                return FM_OK;
            }
    }
    if (hipHostMalloc((void**)&m->h_scal, FM_PINNED_DOUBLES * sizeof(double)) == hipSuccess) return FM_OK;
    (void)hipGetLastError();
    m->h_scal = nullptr;
    return fm_fail(m, FM_ENOMEM, "pinned allocation failed");
}

static void pinned_free(fm_matrix* m)
{
    if (m->h_scal == nullptr) return;
    {
        std::lock_guard<std::mutex> g(g_pool_lock);
        if (g_pinned.size() < POOL_PINNED_CAP) {
            g_pinned.push_back({m->device, m->h_scal});
            return;
        }
    }
    (void)hipHostFree(m->h_scal);
}

ProfScope::ProfScope(fm_matrix* m_, hipStream_t st_, int id_) : m(m_), st(st_), id(id_)
{
    if (!m->prof) return;
    for (hipEvent_t* ev : {&a, &b}) {
        if (!m->prof_pool.empty()) {
            *ev = m->prof_pool.back();
            m->prof_pool.pop_back();
        } else if (hipEventCreate(ev) != hipSuccess) {
            *ev = nullptr;
        }
    }
    if (a != nullptr) (void)hipEventRecord(a, st);
}

ProfScope::~ProfScope()
{
    if (!m->prof || a == nullptr || b == nullptr) return;
    (void)hipEventRecord(b, st);
    m->prof_recs.push_back({id, a, b});
}

static const char* const kKernelNames[FMK_COUNT] = {
    "rows_forward", "rows_refresh", "cols", "cols_long", "cols_tile", "cols_finish", "reduce", "bias"};

extern "C" int fm_profile_enable(fm_matrix* m, int32_t on)
{
    if (m == nullptr) return FM_EINVAL;
    m->prof = on != 0;
    return FM_OK;
}
extern "C" int fm_profile_kernels(void) { return FMK_COUNT; }
extern "C" const char* fm_profile_kernel_name(int32_t k) { return (k >= 0 && k < FMK_COUNT) ? kKernelNames[k] : ""; }

extern "C" int fm_profile_read(fm_matrix* m, int64_t* launches, double* total_ms)
{
    if (m == nullptr || launches == nullptr || total_ms == nullptr) return FM_EINVAL;
    FM_HIP(m, hipDeviceSynchronize());
    for (const ProfRec& r : m->prof_recs) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, r.a, r.b) == hipSuccess) {
            m->prof_launches[r.id] += 1;
            m->prof_ms[r.id] += (double)ms;
        }
        m->prof_pool.push_back(r.a);
        m->prof_pool.push_back(r.b);
    }
    m->prof_recs.clear();
    for (int k = 0; k < FMK_COUNT; ++k) {
        launches[k] = m->prof_launches[k];
        total_ms[k] = m->prof_ms[k];
        m->prof_launches[k] = 0;
        m->prof_ms[k] = 0.0;
    }
    return FM_OK;
}

extern "C" const char* fm_last_error(const fm_matrix* m) { return m != nullptr ? m->err.c_str() : g_build_error.c_str(); }

extern "C" int fm_destroy(fm_matrix* m)
{
    if (m == nullptr) return FM_OK;
    int current = -1;  // the blocks go back idle: wait for the device they are on
    const bool elsewhere = hipGetDevice(&current) == hipSuccess && current != m->device;
    if (elsewhere) (void)hipSetDevice(m->device);
    (void)hipDeviceSynchronize();
    fm_drop_graph(m);
    if (m->gstream != nullptr) (void)hipStreamDestroy(m->gstream);
    if (m->g_in != nullptr) (void)hipEventDestroy(m->g_in);
    if (m->g_out != nullptr) (void)hipEventDestroy(m->g_out);
    for (const FmAlloc& a : m->allocs)
        if (a.pool_bytes > 0)
            pool_give(a.p, a.pool_bytes, m->device);
        else
            (void)hipFree(a.p);
    pinned_free(m);
    if (m->side1 != nullptr) (void)hipStreamDestroy(m->side1);
    if (m->side2 != nullptr) (void)hipStreamDestroy(m->side2);
    for (hipEvent_t e : {m->ev_fork, m->ev_join1, m->ev_join2})
        if (e != nullptr) (void)hipEventDestroy(e);
    for (const ProfRec& r : m->prof_recs) {
        (void)hipEventDestroy(r.a);
        (void)hipEventDestroy(r.b);
    }
    for (hipEvent_t e : m->prof_pool) (void)hipEventDestroy(e);
    if (elsewhere) (void)hipSetDevice(current);
    delete m;
    return FM_OK;
}

// The first violation of the CSR rules in row order, for the message (the check itself runs on the device).
static int first_csr_error(int64_t N, int64_t D, int64_t nnz, const int64_t* rowptr, const int32_t* col)
{
    for (int64_t i = 0; i < N; ++i) {
        const int64_t b = rowptr[i], e = rowptr[i + 1];
        if (e < b || e > nnz) return fm_fail(nullptr, FM_EUNSORTED, "rowptr not monotone at row %lld", (long long)i);
        for (int64_t t = b; t < e; ++t) {
            const int64_t c = col[t];
            if (c < 0 || c >= D)
                return fm_fail(nullptr, FM_ERANGE, "column %lld of row %lld outside [0,%lld)", (long long)c,
                               (long long)i, (long long)D);
            if (t > b && col[t - 1] >= c)
                return fm_fail(nullptr, FM_EUNSORTED, "columns of row %lld not strictly ascending", (long long)i);
        }
    }
    return FM_OK;
}

extern "C" int fm_build_csr(int64_t N, int64_t D, int64_t nnz, const int64_t* rowptr, const int32_t* col,
                            const float* val, void* hip_stream, fm_matrix** out)
{
    if (out == nullptr) return fm_fail(nullptr, FM_EINVAL, "out is NULL");
    *out = nullptr;
    if (N < 0 || D < 0 || nnz < 0 || rowptr == nullptr || (nnz > 0 && (col == nullptr || val == nullptr)))
        return fm_fail(nullptr, FM_EINVAL, "bad sizes or NULL arrays");
    if (N >= (1LL << 31) || D >= (1LL << 31) || nnz >= (1LL << 32))
        return fm_fail(nullptr, FM_ERANGE, "N, D must be < 2^31 and nnz < 2^32");
    if (rowptr[0] != 0 || rowptr[N] != nnz) return fm_fail(nullptr, FM_EUNSORTED, "rowptr[0] != 0 or rowptr[N] != nnz");
    hipStream_t st = (hipStream_t)hip_stream;
    fm_matrix* m = new (std::nothrow) fm_matrix();
    if (m == nullptr) return fm_fail(nullptr, FM_ENOMEM, "out of host memory");
    m->N = N;
    m->D = D;
    m->nnz = nnz;
    int rc = hipGetDevice(&m->device) == hipSuccess ? FM_OK : fm_fail(m, FM_EHIP, "no current device");
    const size_t pointers = (size_t)(N + 1) * sizeof(int64_t), entries = (size_t)nnz * sizeof(int32_t);
    const size_t pad = FM_ENTRY_PAD * sizeof(int32_t);
    static_assert(sizeof(int32_t) == sizeof(float), "indices and values of one size");
    if (rc == FM_OK) rc = fm_dev_alloc(m, (void**)&m->rowptr, pointers);
    if (rc == FM_OK) rc = fm_dev_alloc(m, (void**)&m->col, entries + pad);
    if (rc == FM_OK) rc = fm_dev_alloc(m, (void**)&m->val, entries + pad);
    const FmUploadPart parts[3] = {{m->rowptr, rowptr, pointers}, {m->col, col, entries}, {m->val, val, entries}};
    FmUploadRing* ring = rc == FM_OK && pointers + 2 * entries >= FM_RING_MIN ? fm_ring_take(m->device) : nullptr;
    if (rc == FM_OK && !(ring != nullptr && fm_ring_upload(ring, parts, 3, st))) {
        auto copy = [&](const FmUploadPart& p) -> int {
            if (p.bytes > 0) FM_HIP(m, hipMemcpyAsync(p.dev, p.host, p.bytes, hipMemcpyHostToDevice, st));
            return FM_OK;
        };
        for (const FmUploadPart& p : parts)
            if (rc == FM_OK) rc = copy(p);
    }
    if (rc == FM_OK) rc = fm_dev_alloc(m, (void**)&m->scal, (8 + FM_REDUCE_TMP + 1) * sizeof(double));
    if (rc == FM_OK) m->aux_rows = reinterpret_cast<int32_t*>(m->scal + 8 + FM_REDUCE_TMP);
    if (rc == FM_OK) rc = pinned_alloc(m);
    bool valid = false;
    if (rc == FM_OK) rc = fm_check_csr(m, st, &valid);  // waits for the uploads
    if (ring != nullptr) {
        if (rc != FM_OK) (void)hipStreamSynchronize(st);
        fm_ring_give(ring);
    }
    if (!valid) {  // also where a step failed: what is wrong with the matrix itself is reported first
        const int bad = first_csr_error(N, D, nnz, rowptr, col);
        if (bad != FM_OK) {
            fm_destroy(m);  // g_build_error holds the message
            return bad;
        }
        if (rc == FM_OK) rc = fm_fail(m, FM_EHIP, "the matrix changed while it was uploaded");
    }
    if (rc == FM_OK) rc = fm_noalloc_init_device(m);  // set-up for fm_forward_noalloc on this device
    if (rc != FM_OK) {
        g_build_error = m->err;
        fm_destroy(m);
        return rc;
    }
    *out = m;
    return FM_OK;
}

extern "C" int fm_get_csc(const fm_matrix* m, int64_t* colptr, int32_t* row, float* val)
{
    if (m == nullptr) return FM_EINVAL;
    fm_matrix* mm = const_cast<fm_matrix*>(m);
    if (!m->has_csc) return fm_fail(mm, FM_ESTATE, "CSC not built");
    FM_HIP(mm, hipDeviceSynchronize());
    if (colptr) FM_HIP(mm, hipMemcpy(colptr, m->colptr, (size_t)(m->D + 1) * sizeof(int64_t), hipMemcpyDeviceToHost));
    if (row && m->nnz) FM_HIP(mm, hipMemcpy(row, m->crow, (size_t)m->nnz * sizeof(int32_t), hipMemcpyDeviceToHost));
    if (val && m->nnz) FM_HIP(mm, hipMemcpy(val, m->cval, (size_t)m->nnz * sizeof(float), hipMemcpyDeviceToHost));
    return FM_OK;
}

extern "C" int fm_get_block_index(const fm_matrix* m, int64_t* row_bounds, int64_t* col_bounds, int64_t* cell_nnz)
{
    if (m == nullptr) return FM_EINVAL;
    fm_matrix* mm = const_cast<fm_matrix*>(m);
    if (m->P == 0) return fm_fail(mm, FM_ESTATE, "matrix not partitioned");
    if (col_bounds != nullptr && m->d_place != nullptr)
        return fm_fail(mm, FM_ESTATE, "the columns were placed one by one (fm_partition_placed): there are no column blocks");
    if (row_bounds) memcpy(row_bounds, m->h_rb.data(), (size_t)(m->P + 1) * sizeof(int64_t));
    if (col_bounds) memcpy(col_bounds, m->h_cb.data(), (size_t)(m->P + 1) * sizeof(int64_t));
    if (cell_nnz) {
        if (m->h_cell_nnz.empty()) return fm_fail(mm, FM_ESTATE, "the cell table is only kept for P <= %d", FM_MAXP_CELLS);
        memcpy(cell_nnz, m->h_cell_nnz.data(), (size_t)m->P * m->P * sizeof(int64_t));
    }
    return FM_OK;
}

extern "C" int fm_get_stratum_nnz(const fm_matrix* m, int32_t s, int64_t* nnz_out)
{
    if (m == nullptr || nnz_out == nullptr) return FM_EINVAL;
    fm_matrix* mm = const_cast<fm_matrix*>(m);
    if (m->P == 0) return fm_fail(mm, FM_ESTATE, "matrix not partitioned");
    if (s < 0 || s >= m->P) return fm_fail(mm, FM_EINVAL, "stratum %d outside [0,%d)", s, m->P);
    *nnz_out = m->h_strat_nnz_off[s + 1] - m->h_strat_nnz_off[s];
    return FM_OK;
}

// Pointer array over all nmaj rows (or columns) of one stratum or batch, expanded on the host from the list
// of the rows (columns) that have entries there: list positions [l0, l1), entries from ent0 on.
static int expand_ptr(fm_matrix* mm, const int32_t* nz_major, const int64_t* nz_beg, int64_t l0, int64_t l1,
                      int64_t ent0, int64_t ent1, int64_t nmaj, int64_t* ptr)
{
    const size_t cnt = (size_t)(l1 - l0);
    std::vector<int32_t> idx(cnt);
    std::vector<int64_t> beg(cnt);
    if (cnt > 0) {
        FM_HIP(mm, hipMemcpy(idx.data(), nz_major + l0, cnt * sizeof(int32_t), hipMemcpyDeviceToHost));
        FM_HIP(mm, hipMemcpy(beg.data(), nz_beg + l0, cnt * sizeof(int64_t), hipMemcpyDeviceToHost));
    }
    int64_t k = 0;
    for (size_t t = 0; t < cnt; ++t) {
        for (; k <= idx[t]; ++k) ptr[k] = beg[t] - ent0;  // rows up to and including this one start here
    }
    for (; k <= nmaj; ++k) ptr[k] = ent1 - ent0;
    return FM_OK;
}

static int get_stratum(const fm_matrix* m, int32_t s, bool by_rows, int64_t* ptr, int32_t* ind, float* val)
{
    if (m == nullptr) return FM_EINVAL;
    fm_matrix* mm = const_cast<fm_matrix*>(m);
    if (m->P == 0) return fm_fail(mm, FM_ESTATE, "matrix not partitioned");
    if (s < 0 || s >= m->P) return fm_fail(mm, FM_EINVAL, "stratum %d outside [0,%d)", s, m->P);
    FM_HIP(mm, hipDeviceSynchronize());
    const int64_t nmaj = by_rows ? m->N : m->D;
    const int64_t off = m->h_strat_nnz_off[s], cnt = m->h_strat_nnz_off[s + 1] - off;
    if (ptr) {
        const std::vector<int64_t>& lo = by_rows ? m->h_touch_off : m->h_ncol_off;
        FM_TRY(expand_ptr(mm, by_rows ? m->s_touched : m->s_ncol, by_rows ? m->s_touched_beg : m->s_ncol_beg, lo[s],
                          lo[s + 1], off, off + cnt, nmaj, ptr));
    }
    if (ind && cnt)
        FM_HIP(mm, hipMemcpy(ind, (by_rows ? m->s_col : m->s_row) + off, (size_t)cnt * sizeof(int32_t),
                             hipMemcpyDeviceToHost));
    if (val && cnt)
        FM_HIP(mm, hipMemcpy(val, (by_rows ? m->s_val : m->s_cval) + off, (size_t)cnt * sizeof(float),
                             hipMemcpyDeviceToHost));
    return FM_OK;
}

extern "C" int fm_get_stratum_csr(const fm_matrix* m, int32_t s, int64_t* rowptr, int32_t* col, float* val)
{
    return get_stratum(m, s, true, rowptr, col, val);
}
extern "C" int fm_get_stratum_csc(const fm_matrix* m, int32_t s, int64_t* colptr, int32_t* row, float* val)
{
    return get_stratum(m, s, false, colptr, row, val);
}

extern "C" int fm_get_batch_csc(const fm_matrix* m, int32_t b, int64_t* colptr, int32_t* row, float* val)
{
    if (m == nullptr) return FM_EINVAL;
    fm_matrix* mm = const_cast<fm_matrix*>(m);
    if (m->B == 0) return fm_fail(mm, FM_ESTATE, "row batches not built");
    if (b < 0 || b >= m->B) return fm_fail(mm, FM_EINVAL, "batch %d outside [0,%d)", b, m->B);
    FM_HIP(mm, hipDeviceSynchronize());
    const int64_t off = m->h_batch_nnz_off[b], cnt = m->h_batch_nnz_off[b + 1] - off;
    if (colptr)
        FM_TRY(expand_ptr(mm, m->b_ncol, m->b_ncol_beg, m->h_bcol_off[b], m->h_bcol_off[b + 1], off, off + cnt, m->D, colptr));
    if (row && cnt) FM_HIP(mm, hipMemcpy(row, m->b_row + off, (size_t)cnt * sizeof(int32_t), hipMemcpyDeviceToHost));
    if (val && cnt) FM_HIP(mm, hipMemcpy(val, m->b_cval + off, (size_t)cnt * sizeof(float), hipMemcpyDeviceToHost));
    return FM_OK;
}

// ------------------------------------------------------------ workspace ----

static int check_params(fm_matrix* m, const fm_params* p)
{
    if (p == nullptr) return fm_fail(m, FM_EINVAL, "params is NULL");
    int vec, lanes;
    if (!fm_shape_for_K(p->K, &vec, &lanes))
        return fm_fail(m, FM_EINVAL, "K=%d unsupported (1..64, or a multiple of 4 up to 256)", p->K);
    if (p->loss != FM_LOSS_SQUARED && p->loss != FM_LOSS_LOGISTIC) return fm_fail(m, FM_EINVAL, "unknown loss %d", p->loss);
    if (p->half_gather && p->K % 4 != 0) return fm_fail(m, FM_EINVAL, "half_gather needs K to be a multiple of 4");
    return FM_OK;
}

// stratified calls keep fp32 gathers: their incremental refresh adds fp32 changes to aggregates that
// would have been formed from rounded factors
static int no_half(fm_matrix* m, const fm_params* p)
{
    if (p->half_gather) return fm_fail(m, FM_EINVAL, "half_gather applies to fm_forward, fm_evaluate, fm_sgd_epoch and fm_minibatch_epoch");
    return FM_OK;
}

// Packed rows exist when [G | r] of a row fits one 128-byte line (a whole number of float4, K <= 28): a column-side gather
// is then a single request.  For larger K a row of G is one or more whole lines by itself.
static bool packed_exists(const fm_matrix* m, int32_t K) { return m->opt.aux != 1 && K % 4 == 0 && K + 1 <= 32; }

// Which layout a pass takes whose columns gather from so many rows (all of the matrix, a batch).  At K = 16 a row of G is half a
// line and a packed row a whole one: planar moves half the bytes, and as long as the multipliers of the rows (4 bytes each) stay
// in an XCD's L2 beside them, the second request for r is a cheap one.  Planar over packed, times, K = 16:
//   full epochs  text-like 1e5 rows 0.93, 2e5 0.92, 3e5 0.90, 4e5 1.06; hashed 1e5 0.88, 2e5 0.92, 4e5 0.98; click-style 1e5 1.02, 1.5e5 0.96,
//                1.8e5 0.99, 2e5 1.00, 2.2e5 1.06, 2.5e5 1.02, 3e5 1.00, 3.6e5 1.03, 6e5 1.09, 1e7 1.17
//   batches      click-style 75,000 rows 0.89, 156,250 0.83, 312,500 0.97, 4e5 1.00, 5e5 1.01, 6.7e5 1.04, 1e6 1.05, 2.5e6 1.06; text-like 5e5 1.00, 1e6 1.01
//   strata       the refresh, which reads and writes rows, gains by it too: click-style 4,700 rows to a block 0.86, 75,000 0.76, 156,250
//                0.81, 1e6 0.97, 1.5e6 0.94 to 0.97, 3e6 0.98, 4e6 0.99, 5e6 0.99, text-like 1.5e6 0.96: on either side of any line.  A single
//                block is like a batch: click-style 1.5e5 rows 0.93, 3e5 0.98, 6e5 1.05, 1e6 1.05, 3e6 1.07, text-like 1e5 0.93, 3e5 0.97
// Other K mostly pack better: a packed row up to K = 12 is half a line itself, and from K = 20 on a planar row straddles lines
// (click-style, full epochs of 6e5 rows, K = 8 1.18, 12 1.20, 20 1.14, 28 1.21; 16 strata of 1e5 and 6e5 rows and 4 of 2e6, K = 8 1.06, 0.99, 1.06,
// K = 12 1.07, 1.06, 1.13, K = 20 1.02, 0.95, 1.05, K = 28 1.05, 1.09, 1.17; text-like 2e5 rows, 16 strata, K = 8 1.04, K = 20 0.97).  Where every
// row stores every column the rows are gathered one after the other, whole lines in any layout, and planar ones are the
// shorter (tables of 40 columns, 8 strata of 1e6 rows, K = 8 0.82, K = 20 0.80, of 2e5 0.97, K = 28 1.01, K = 4 0.99 to 1.05).
constexpr int64_t FM_PLANAR_ROWS = 200000;        // full epochs, gradients
constexpr int64_t FM_PLANAR_ROWS_BATCH = 400000;  // batches, a single block of strata: their items are worked on in row order
static bool take_packed(const fm_matrix* m, int32_t K, int64_t rows, int64_t planar_rows)
{
    if (!packed_exists(m, K)) return false;
    if (m->opt.aux == 2) return true;
    return m->is_dense && K >= 8 ? false : K != 16 || rows > planar_rows;
}

// Both layouts may come up on this handle: a forward pass then leaves the one it took in the word that fm_get_aux reads.  Options
// that change the answer, and another K, drop the aggregates with it.
static bool packed_possible(const fm_matrix* m, int32_t K) { return take_packed(m, K, 1, 0); }
static int32_t* layout_word(const fm_matrix* m, int32_t K) { return packed_possible(m, K) ? m->aux_rows : nullptr; }

static int64_t packed_stride(int32_t K) { return ((int64_t)K + 3 + 15) / 16 * 16; }

static int64_t whole_lines(int64_t floats) { return (floats + 31) / 32 * 32; }

int64_t fm_aux_floats(const fm_matrix* m, int32_t K, bool packed)
{
    if (packed) return m->N * packed_stride(K);
    return whole_lines(m->N * (int64_t)K) + whole_lines(m->N * 2) + m->N;
}

FmAux fm_aux_layout(const fm_matrix* m, int32_t K, bool packed)
{
    FmAux x;
    if (packed) {
        x.gs = x.ss = x.as = packed_stride(K);
        x.G = m->aux;
        x.r = m->aux + K;
        x.a = m->aux + K + 1;
        x.q = m->aux + K + 2;
    } else {
        x.gs = K;
        x.ss = 1;
        x.as = 2;
        x.G = m->aux;
        x.a = m->aux + whole_lines(m->N * (int64_t)K);
        x.q = x.a + 1;
        x.r = x.a + whole_lines(m->N * 2);
    }
    return x;
}

bool fm_side_streams(fm_matrix* m)
{
    if (!m->opt.side_streams) return false;
    if (m->side_state == 0) {
        m->side_state = -1;
        if (hipStreamCreateWithFlags(&m->side1, hipStreamNonBlocking) == hipSuccess &&
            hipStreamCreateWithFlags(&m->side2, hipStreamNonBlocking) == hipSuccess &&
            hipEventCreateWithFlags(&m->ev_fork, hipEventDisableTiming) == hipSuccess &&
            hipEventCreateWithFlags(&m->ev_join1, hipEventDisableTiming) == hipSuccess &&
            hipEventCreateWithFlags(&m->ev_join2, hipEventDisableTiming) == hipSuccess)
            m->side_state = 1;
        else
            (void)hipGetLastError();
    }
    return m->side_state == 1;
}

void fm_drop_graph(fm_matrix* m)
{
    if (m->gexec != nullptr) {
        (void)hipGraphExecDestroy(m->gexec);
        m->gexec = nullptr;
    }
}

void fm_drop_workspace(fm_matrix* m)
{
    fm_drop_graph(m);
    if (m->wsK != 0) (void)hipDeviceSynchronize();  // the blocks go back idle
    for (void* p : {(void*)m->aux, (void*)m->dV, (void*)m->dwn, (void*)m->part, (void*)m->row_part})
        fm_dev_free(m, p);
    m->aux = m->dV = m->part = m->row_part = nullptr;
    m->dwn = nullptr;
    m->wsK = 0;
    m->aux_full = false;
    m->aux_held = false;
}

// (re)allocate the per-K workspace
static int ensure_ws(fm_matrix* m, int32_t K)
{
    if (m->wsK == K) return FM_OK;
    fm_drop_workspace(m);
    if (m->has_csc) {  // the LDS tiles of the dense-ish columns are shaped for K
        int shape[3];
        fm_tile_shape(m, K, &shape[0], &shape[1], &shape[2]);
        if (memcmp(shape, m->lfull_shape, sizeof(shape)) != 0) {
            FM_HIP(m, hipDeviceSynchronize());
            FM_TRY(fm_build_full_index(m, K, nullptr));
        }
    }
    const size_t D = (size_t)m->D;
    // fm_evaluate leaves three doubles per row block there: more than the aggregates of a single row with K <= 2 take
    // either layout: which one a call takes is its own matter
    const int64_t rows = packed_exists(m, K) ? fm_aux_floats(m, K, true) : 0;
    FM_TRY(fm_dev_alloc(m, (void**)&m->aux,
                        (size_t)std::max<int64_t>(std::max<int64_t>(rows, fm_aux_floats(m, K, false)), 6) * sizeof(float)));
    // the dense kernels may be switched on and off: room for both paths
    const int64_t chunks = fm_dense_fits(m, K) ? fm_dense_chunks(m->N, m->D, K) : 0;
    const int64_t dense_items = chunks * 2;  // a batch of few rows has two to a column and workgroup
    int64_t items = std::max<int64_t>(m->lfull.nitems, m->D * dense_items);
    for (const LongIndex* li : {&m->lstrat, &m->lbatch})
        for (size_t s = 0; s + 1 < li->h_item_off.size(); ++s) items = std::max(items, li->h_item_off[s + 1] - li->h_item_off[s]);
    FM_TRY(fm_dev_alloc(m, (void**)&m->part,
                        (size_t)std::max<int64_t>(items, 1) * (size_t)fm_part_stride(K) * sizeof(float)));
    FM_TRY(fm_dev_alloc(m, (void**)&m->row_part, (size_t)std::max<int64_t>(std::max<int64_t>(fm_rows_max_grid(m, m->N, K), chunks), 1) * 2 * sizeof(float)));
    if (m->P > 0) {
        FM_TRY(fm_dev_alloc(m, (void**)&m->dV, D * K * sizeof(float)));
        FM_TRY(fm_dev_alloc(m, (void**)&m->dwn, D * sizeof(float2)));
    }
    m->wsK = K;
    return FM_OK;
}

static int ensure_strat_ws(fm_matrix* m, int32_t K)
{
    return ensure_ws(m, K);  // fm_partition dropped any older workspace, so dV/dwn are there
}

static void fill_long(const fm_matrix* m, ColArgs& A, const LongIndex& li, int32_t s, bool strat)
{
    const int64_t l0 = strat ? li.h_long_off[s] : 0, l1 = strat ? li.h_long_off[s + 1] : li.nlong;
    const int64_t i0 = strat ? li.h_item_off[s] : 0, i1 = strat ? li.h_item_off[s + 1] : li.nitems;
    A.nlong = l1 - l0;
    A.nitems = i1 - i0;
    A.part = m->part - i0 * A.ps;  // this launch's items have the first rows: one stratum or batch is in flight at a time
    A.long_base = l0;
    A.item_base = i0;
    A.long_col = li.long_col;
    A.long_first = li.long_first;
    A.item_col = li.item_col;
    A.item_beg = li.item_beg;
    A.item_len = li.item_len;
    A.order = li.order != nullptr ? li.order + i0 : nullptr;  // a stratum or batch: one sequence, list_off is zero
    A.ord_beg = li.ord_beg != nullptr ? li.ord_beg + i0 : nullptr;
    A.ord_len = li.ord_len != nullptr ? li.ord_len + i0 : nullptr;
    for (int x = 0; x <= FM_XCDS; ++x) A.list_off[x] = li.list_off[x];
    for (int x = 0; x < FM_XCDS; ++x) A.list_mid[x] = li.list_mid[x];
    // a single block or batch steps with the bits of the whole matrix
    A.long_runs = m->lfull.in_panels && (!strat || A.P == 1) ? 1 : 0;
    A.tile_rows = li.tile_rows;
    A.ntiles = strat ? 0 : li.ntiles;
    A.tile_ptr = li.tile_ptr;
    const int64_t v0 = strat && !li.h_vlong_off.empty() ? li.h_vlong_off[s] : 0;
    const int64_t v1 = strat ? (li.h_vlong_off.empty() ? 0 : li.h_vlong_off[s + 1]) : li.nvlong;
    A.vlong = li.vlong != nullptr ? li.vlong + v0 : nullptr;
    A.nvlong = v1 - v0;
    A.vlong_items = m->tune.vlong;
    if (strat && li.whole) {
        A.whole = 1;
        A.long_beg = li.long_beg;
        A.long_len = li.long_len;
        A.nbig = li.h_big_off.empty() ? 0 : li.h_big_off[s + 1] - li.h_big_off[s];
        A.big_cols = A.nbig > 0 ? li.big + li.h_big_off[s] : nullptr;
    }
    const int64_t s0 = strat ? li.h_short_off[s] : 0, s1 = strat ? li.h_short_off[s + 1] : li.nshort;
    A.short_col = li.short_col != nullptr ? li.short_col + s0 : nullptr;
    A.short_beg = li.short_beg != nullptr ? li.short_beg + s0 : nullptr;
    A.short_len = li.short_len != nullptr ? li.short_len + s0 : nullptr;
    A.nshort = s1 - s0;
}

// RowArgs outputs pointing into the handle's aggregates, for a pass that keeps them packed or planar
static void aux_outputs(fm_matrix* m, int32_t K, RowArgs& A, bool with_aq, bool packed)
{
    const FmAux x = fm_aux_layout(m, K, packed);
    A.whole_rows = packed ? 1 : 0;  // never leave a line partly written
    A.aux_rows = layout_word(m, K);
    A.G = x.G;
    A.gs = x.gs;
    A.ss = x.ss;
    A.as = x.as;
    A.r = x.r;
    A.a = with_aq ? x.a : nullptr;
    A.q = with_aq ? x.q : nullptr;
}

// ---------------------------------------------------------------- forward ----

// With half_gather: refresh the handle's half-precision copy of V (one streaming pass) and hand it to the row kernel.
static int half_copy(fm_matrix* m, const fm_params* p, const float* V, const _Float16** out, hipStream_t st)
{
    *out = nullptr;
    if (!p->half_gather) return FM_OK;
    const int64_t n = m->D * (int64_t)p->K;
    if (m->Vh == nullptr || m->VhK != p->K) {
        if (m->Vh != nullptr) {
            FM_HIP(m, hipDeviceSynchronize());
            fm_dev_free(m, m->Vh);
            m->Vh = nullptr;
        }
        FM_TRY(fm_dev_alloc(m, (void**)&m->Vh, (size_t)std::max<int64_t>(n, 1) * sizeof(_Float16)));
        m->VhK = p->K;
    }
    FM_TRY(fm_to_half(m, V, m->Vh, n, st));
    *out = m->Vh;
    return FM_OK;
}

// (loss, multiplier) pairs that a forward pass over all rows leaves (what: see forward_args): one per workgroup
static int64_t forward_pairs(const fm_matrix* m, const fm_params* p, int what = FM_DENSE_FORWARD)
{
    return fm_dense_takes(m, p, m->N, what) ? fm_dense_chunks(m->N, m->D, p->K) : fm_rows_grid(m, m->N, p->K);
}

// The sums over n pairs (or, single, n multipliers `stride` floats apart) as an epilogue.
static void set_epilogue(fm_matrix* m, FmEpilogue& E, const float* x, int64_t n, int64_t stride, bool single)
{
    memset(&E, 0, sizeof(E));
    E.on = 1;
    E.x = x;
    E.n = n;
    E.stride = stride;
    E.single = single ? 1 : 0;
    E.nsums = fm_epi_nsums(n);
    E.sums = m->scal + 8;
    E.scal = m->scal;
}

// After the last kernel of a call with an objective: its two terms from the figures in pinned memory.
static int read_objective(fm_matrix* m, const fm_params* p, double* objective, hipStream_t st)
{
    FM_HIP(m, hipStreamSynchronize(st));
    objective[0] = (double)p->loss_scale * m->h_scal[0];
    objective[1] = 0.5 * (double)p->lambda_w * m->h_scal[2] + 0.5 * (double)p->lambda_v * m->h_scal[3];
    return FM_OK;
}

// mode 0: caller arrays (dense); 1: handle's aggregates, G and r; 2: handle's, G r a q; packed: their layout
static int forward_args(fm_matrix* m, const fm_params* p, const float* y, const float* w0, const float* w,
                        const float* V, float* yhat, float* a, float* G, float* q, float* r, int mode, bool packed,
                        bool want_sums, int what, RowArgs& A, hipStream_t st)
{
    memset(&A, 0, sizeof(A));
    A.N = m->N;
    A.K = p->K;
    A.rowptr = m->rowptr;
    A.col = m->col;
    A.val = m->val;
    A.w0 = w0;
    A.w = w;
    A.V = V;
    A.big = fm_rows_big(m, p->K);
    A.y = y;
    A.yhat = yhat;
    if (mode == 0) {
        A.a = a;
        A.G = G;
        A.q = q;
        A.r = r;
        A.gs = p->K;
        A.ss = A.as = 1;
    } else {
        aux_outputs(m, p->K, A, mode == 2, packed);
        m->aux_held = true;
    }
    A.row_part = (want_sums && y != nullptr) ? m->row_part : nullptr;
    A.loss = p->loss;
    A.s = p->loss_scale;
    if (fm_dense_takes(m, p, m->N, what)) {
        A.dense_D = (int32_t)m->D;
        A.dense_half = p->half_gather;
    } else {
        FM_TRY(half_copy(m, p, V, &A.Vh, st));
    }
    return FM_OK;
}

static int run_forward(fm_matrix* m, const fm_params* p, const float* y, const float* w0, const float* w,
                       const float* V, float* yhat, float* a, float* G, float* q, float* r, int mode, bool packed,
                       bool want_sums, hipStream_t st)
{
    RowArgs A;
    FM_TRY(forward_args(m, p, y, w0, w, V, yhat, a, G, q, r, mode, packed, want_sums, FM_DENSE_FORWARD, A, st));
    return fm_launch_rows(m, A, false, st);  // the pairs stay in m->row_part
}

// Forward at the parameters as they stand, the sums and the objective: what the epochs with several steps report.
static int objective_pass(fm_matrix* m, const fm_params* p, const float* y, const float* w0, const float* w, const float* V,
                          int mode, bool packed, double* objective, hipStream_t st)
{
    FM_TRY(run_forward(m, p, y, w0, w, V, nullptr, nullptr, nullptr, nullptr, nullptr, mode, packed, true, st));
    FmEpilogue E;
    set_epilogue(m, E, m->row_part, forward_pairs(m, p), 0, false);
    if (m->D * ((int64_t)p->K + 1) <= FM_EPI_REG) {
        E.reg_w = w;
        E.reg_V = V;
        E.reg_nw = m->D;
        E.reg_nV = m->D * (int64_t)p->K;
    } else {
        FM_TRY(fm_reg_partials(m, w, m->D, V, m->D * (int64_t)p->K, &E.regs, &E.nregs, st));
    }
    E.host = m->h_scal;
    FM_TRY(fm_run_epilogue(m, E, st));
    return read_objective(m, p, objective, st);
}

extern "C" int fm_forward(fm_matrix* m, const fm_params* p, const float* y, const float* w0, const float* w,
                          const float* V, float* yhat, float* a, float* G, float* q, float* r, double* loss_sum,
                          void* hip_stream)
{
    if (m == nullptr) return FM_EINVAL;
    FM_TRY(check_params(m, p));
    if (w0 == nullptr || w == nullptr || V == nullptr) return fm_fail(m, FM_EINVAL, "w0, w, V must not be NULL");
    if ((r != nullptr || loss_sum != nullptr) && y == nullptr) return fm_fail(m, FM_EINVAL, "r and loss_sum need y");
    FM_TRY(fm_check_vec_aligned(m, {V, G}));
    hipStream_t st = (hipStream_t)hip_stream;
    FM_TRY(ensure_ws(m, p->K));
    if (m->N == 0) {
        if (loss_sum) *loss_sum = 0.0;
        return FM_OK;
    }
    FM_TRY(run_forward(m, p, y, w0, w, V, yhat, a, G, q, r, 0, false, loss_sum != nullptr, st));
    if (loss_sum != nullptr) {
        FM_TRY(fm_reduce_pairs(m, m->row_part, forward_pairs(m, p), m->h_scal, st));
        FM_HIP(m, hipStreamSynchronize(st));
        *loss_sum = m->h_scal[0];
    }
    return FM_OK;
}

extern "C" int fm_evaluate(fm_matrix* m, const fm_params* p, const float* y, const float* w0, const float* w,
                           const float* V, double* metrics, void* hip_stream)
{
    if (m == nullptr) return FM_EINVAL;
    FM_TRY(check_params(m, p));
    if (y == nullptr || w0 == nullptr || w == nullptr || V == nullptr || metrics == nullptr)
        return fm_fail(m, FM_EINVAL, "y, w0, w, V, metrics must not be NULL");
    FM_TRY(fm_check_vec_aligned(m, {V}));
    hipStream_t st = (hipStream_t)hip_stream;
    FM_TRY(ensure_ws(m, p->K));
    metrics[0] = metrics[1] = metrics[2] = 0.0;
    if (m->N == 0) return FM_OK;
    // The sums per row block go to the start of the aggregate storage, which holds nothing afterwards; those of few blocks
    // straight to pinned memory, where they are added up without another launch (49,990 x 22, K=4: 24.9 -> 23.4 us).
    m->aux_held = false;
    m->aux_full = false;
    const int64_t blocks = forward_pairs(m, p);
    const bool direct = blocks <= FM_CHECK_BLOCKS;
    static_assert(sizeof(FmCheck) == 3 * sizeof(double), "the block results of the CSR check leave room for as many triples");
    RowArgs A;
    memset(&A, 0, sizeof(A));
    A.N = m->N;
    A.K = p->K;
    A.rowptr = m->rowptr;
    A.col = m->col;
    A.val = m->val;
    A.w0 = w0;
    A.w = w;
    A.V = V;
    A.big = fm_rows_big(m, p->K);
    A.y = y;
    A.gs = p->K;
    A.ss = A.as = 1;
    A.eval_part = direct ? m->h_scal + 8 : reinterpret_cast<double*>(m->aux);
    A.loss = p->loss;
    A.s = 1.f;
    if (fm_dense_takes(m, p, m->N, FM_DENSE_FORWARD)) {
        A.dense_D = (int32_t)m->D;
        A.dense_half = p->half_gather;
    } else {
        FM_TRY(half_copy(m, p, V, &A.Vh, st));
    }
    FM_TRY(fm_launch_rows(m, A, false, st));
    if (!direct) FM_TRY(fm_reduce_eval(m, A.eval_part, blocks, m->h_scal, m->scal + 8, st));
    FM_HIP(m, hipStreamSynchronize(st));
    if (direct) {
        for (int c = 0; c < 3; ++c) m->h_scal[c] = 0.0;
        for (int64_t b = 0; b < blocks; ++b)
            for (int c = 0; c < 3; ++c) m->h_scal[c] += A.eval_part[3 * b + c];
    }
    const double n = (double)m->N;
    metrics[0] = m->h_scal[0] / n;
    metrics[1] = sqrt(m->h_scal[1] / n);
    metrics[2] = m->h_scal[2] / n;
    return FM_OK;
}

// --------------------------------------------------------------- gradient ----

// The column pass behind the dense one X: only the finish, of all columns.
static void dense_long(const fm_matrix* m, const DenseArgs& X, ColArgs& A)
{
    A.ndense = X.nchunks * X.nparts;
    A.nlong = m->D;
    A.nvlong = A.ndense > m->tune.vlong ? m->D : 0;  // a workgroup per column, or a wavefront
    A.vlong_items = m->tune.vlong;
}

// The data sums of all columns of a dense matrix from r and G of A, and A.epi's sums beside them.
static int dense_sums(fm_matrix* m, ColArgs& A, hipStream_t st)
{
    DenseArgs X;
    memset(&X, 0, sizeof(X));
    X.N = m->N;
    X.D = m->D;
    X.K = A.K;
    X.nchunks = fm_dense_chunks(m->N, m->D, A.K);
    X.X = m->val;
    X.G = const_cast<float*>(A.G);
    X.r = const_cast<float*>(A.r);
    X.gs = A.gs;
    X.ss = A.rs;
    X.part = A.part;
    X.ps = A.ps;
    X.nparts = fm_dense_parts(X.N, X.D, X.K);
    X.epi = A.epi;
    FM_TRY(fm_launch_dense(m, X, FM_DENSE_GRADIENT, st));
    dense_long(m, X, A);
    return FM_OK;
}

static void base_col_args(fm_matrix* m, const fm_params* p, bool packed, ColArgs& A)
{
    memset(&A, 0, sizeof(A));
    A.D = m->D;
    A.K = p->K;
    A.lambda_w = p->lambda_w;
    A.lambda_v = p->lambda_v;
    A.eta = p->eta;
    A.N = m->N;
    A.part = m->part;
    A.ps = fm_part_stride(p->K);
    // Aggregates that do not fit the memory-side cache: rows that are gathered once do not push others out of the L2.
    const int64_t aux_bytes = fm_aux_floats(m, p->K, packed) * (int64_t)sizeof(float);
    A.packed = packed ? FM_PACKED_LANE : FM_PLANAR;
    A.nt = aux_bytes > (int64_t(256) << 20) ? 1 : 0;
    A.big = aux_bytes > FM_BUF_BYTES || m->opt.wide_addresses ? 1 : 0;
}

extern "C" int fm_gradient(fm_matrix* m, const fm_params* p, const float* r, const float* G, const float* w,
                           const float* V, float* grad_w0, float* grad_w, float* grad_V, void* hip_stream)
{
    if (m == nullptr) return FM_EINVAL;
    FM_TRY(check_params(m, p));
    if (!m->has_csc) return fm_fail(m, FM_ESTATE, "fm_gradient needs fm_build_csc first");
    if (r == nullptr || G == nullptr || w == nullptr || V == nullptr)
        return fm_fail(m, FM_EINVAL, "r, G, w, V must not be NULL");
    FM_TRY(fm_check_vec_aligned(m, {G, V, grad_V}));
    hipStream_t st = (hipStream_t)hip_stream;
    FM_TRY(ensure_ws(m, p->K));
    FmEpilogue E;
    set_epilogue(m, E, r, m->N, 1, true);
    E.grad_w0 = grad_w0;
    if (m->D == 0 || (grad_w == nullptr && grad_V == nullptr))
        return grad_w0 != nullptr ? fm_run_epilogue(m, E, st) : FM_OK;
    const bool dense = fm_dense_takes(m, p, m->N, FM_DENSE_GRADIENT);
    const bool packed = !dense && take_packed(m, p->K, m->N, FM_PLANAR_ROWS);
    if (packed_exists(m, p->K)) {
        // Where packed rows exist the handle holds r and G of the call afterwards, for fm_get_aux.  Packed, one streaming pass
        // makes every gather of the columns one request (and dense-ish columns can be staged through LDS); planar, the columns
        // and the dense kernels read the caller's arrays as they are.
        FM_TRY(fm_keep_aux(m, packed, r, G, st));
        m->aux_held = true;
        m->aux_full = false;
    }
    ColArgs A;
    base_col_args(m, p, packed, A);
    if (grad_w0 != nullptr) A.epi = E;
    A.ptr = m->colptr;
    A.row = m->crow;
    A.val = m->cval;
    if (packed) {
        const FmAux x = fm_aux_layout(m, p->K, true);
        A.r = x.r;
        A.G = x.G;
        A.gs = x.gs;
        A.rs = x.ss;
    } else {
        A.r = r;
        A.G = G;
        A.gs = p->K;
        A.rs = 1;
    }
    A.w = const_cast<float*>(w);
    A.V = const_cast<float*>(V);
    A.grad_w = grad_w;
    A.grad_V = grad_V;
    if (dense)
        FM_TRY(dense_sums(m, A, st));
    else
        fill_long(m, A, m->lfull, 0, false);
    return fm_launch_cols(m, A, false, st);
}

// ------------------------------------------------------------ full epoch ----

// Forward and data sums of a dense pass over the rows of R in one kernel; A then has only the finish left.
static int dense_step(fm_matrix* m, const RowArgs& R, bool regs, ColArgs& A, hipStream_t st)
{
    DenseArgs X;
    fm_dense_rows(R, &X);
    X.part = A.part;
    X.ps = A.ps;
    X.nparts = fm_dense_parts(X.N, X.D, X.K);
    X.regs = regs ? fm_reg_scratch(m) : nullptr;
    FM_TRY(fm_launch_dense(m, X, FM_DENSE_FORWARD | FM_DENSE_GRADIENT, st));
    dense_long(m, X, A);
    return FM_OK;
}

extern "C" int fm_sgd_epoch(fm_matrix* m, const fm_params* p, const float* y, float* w0, float* w, float* V,
                            double* objective, void* hip_stream)
{
    if (m == nullptr) return FM_EINVAL;
    FM_TRY(check_params(m, p));
    if (!m->has_csc) return fm_fail(m, FM_ESTATE, "fm_sgd_epoch needs fm_build_csc first");
    if (y == nullptr || w0 == nullptr || w == nullptr || V == nullptr)
        return fm_fail(m, FM_EINVAL, "y, w0, w, V must not be NULL");
    FM_TRY(fm_check_vec_aligned(m, {V}));
    hipStream_t st = (hipStream_t)hip_stream;
    FM_TRY(ensure_ws(m, p->K));
    if (m->N == 0 || m->D == 0) {
        if (objective) objective[0] = objective[1] = 0.0;
        return FM_OK;
    }
    // steps 1-3: G, r, loss and sum r
    const bool packed = take_packed(m, p->K, m->N, FM_PLANAR_ROWS);
    RowArgs R;
    FM_TRY(forward_args(m, p, y, w0, w, V, nullptr, nullptr, nullptr, nullptr, nullptr, 1, packed, true,
                        FM_DENSE_FORWARD | FM_DENSE_GRADIENT, R, st));
    m->aux_full = false;
    const bool dense = R.dense_D > 0;  // then the data sums of step 4 come with them
    if (!dense) FM_TRY(fm_launch_rows(m, R, false, st));
    // steps 4-5 fused: gradient of every column and the step on w, V
    ColArgs A;
    base_col_args(m, p, packed, A);
    A.ptr = m->colptr;
    A.row = m->crow;
    A.val = m->cval;
    const FmAux x = fm_aux_layout(m, p->K, packed);
    A.r = x.r;
    A.G = x.G;
    A.gs = x.gs;
    A.rs = x.ss;
    A.w = w;
    A.V = V;
    if (!dense) fill_long(m, A, m->lfull, 0, false);
    if (p->update_w0 || objective != nullptr) {
        set_epilogue(m, A.epi, m->row_part, forward_pairs(m, p, FM_DENSE_FORWARD | FM_DENSE_GRADIENT), 0, false);
        if (dense) A.epi.nsums = 0;  // the pairs of this very launch: the finish adds them
        if (p->update_w0) A.epi.w0 = w0;
        A.epi.eta = p->eta;
        if (objective != nullptr) {  // regulariser at the parameters the epoch starts from
            if (dense) {
                A.epi.regs = fm_reg_scratch(m);
                A.epi.nregs = 1;
            } else {
                FM_TRY(fm_reg_partials(m, w, m->D, V, m->D * (int64_t)p->K, &A.epi.regs, &A.epi.nregs, st));
            }
            A.epi.host = m->h_scal;
        }
    }
    if (dense) FM_TRY(dense_step(m, R, objective != nullptr, A, st));
    FM_TRY(fm_launch_cols(m, A, true, st));
    return objective != nullptr ? read_objective(m, p, objective, st) : FM_OK;
}

// ------------------------------------------------------- stratified epoch ----

// All of the strata's calls ask for the layout here: a step goes on from aggregates that fm_stratified_begin left, now or in a
// graph.
static bool strata_packed(const fm_matrix* m, int32_t K)
{
    return take_packed(m, K, m->N, m->P == 1 ? FM_PLANAR_ROWS_BATCH : INT64_MAX);
}

extern "C" int fm_stratified_begin(fm_matrix* m, const fm_params* p, const float* y, const float* w0,
                                   const float* w, const float* V, void* hip_stream)
{
    if (m == nullptr) return FM_EINVAL;
    FM_TRY(check_params(m, p));
    FM_TRY(no_half(m, p));
    if (m->P == 0) return fm_fail(m, FM_ESTATE, "stratified calls need fm_partition first");
    if (y == nullptr || w0 == nullptr || w == nullptr || V == nullptr)
        return fm_fail(m, FM_EINVAL, "y, w0, w, V must not be NULL");
    FM_TRY(fm_check_vec_aligned(m, {V}));
    hipStream_t st = (hipStream_t)hip_stream;
    FM_TRY(ensure_strat_ws(m, p->K));
    FM_TRY(run_forward(m, p, y, w0, w, V, nullptr, nullptr, nullptr, nullptr, nullptr, 2, strata_packed(m, p->K), false, st));
    m->aux_full = true;
    return FM_OK;
}

// Regulariser shares of P floor-split row blocks: the table, the bounds, and the two values it holds.
static void set_shares(ColArgs& A, const float* rho, const int64_t* bounds, int64_t N, int32_t P)
{
    A.rho = rho;
    A.rb = bounds;
    const int64_t base = N / P;
    A.rho_small = (float)((double)base / (double)N);
    A.rho_big = (float)((double)(base + 1) / (double)N);
}

// Column-side arguments of stratum s (s == P: the flush after the last stratum).
static void strat_col_args(fm_matrix* m, const fm_params* p, int32_t s, float* w, float* V, bool lazy, ColArgs& A)
{
    base_col_args(m, p, strata_packed(m, p->K), A);
    A.w = w;
    A.V = V;
    A.P = m->P;
    A.s = s;
    if (!p->reg_full_per_cell) set_shares(A, m->d_rho, m->d_rb, m->N, m->P);
    A.place = m->d_place;
    if (lazy) A.lazy_last = m->lazy_last;
}

// One stratum.  lazy: columns that are empty in their cell postpone their regulariser-only step
// (the caller starts the epoch with lazy_last = 0 and flushes after the last stratum).
static int stratified_step(fm_matrix* m, const fm_params* p, int32_t s, const float* y, const float* w0, float* w,
                           float* V, bool lazy, hipStream_t st)
{
    // phase A: block gradients of the stratum's P cells and the step on every column block
    ColArgs A;
    strat_col_args(m, p, s, w, V, lazy, A);
    A.ptr = nullptr;  // no pointer array per stratum: short columns carry their extent, long ones their items
    A.mark = lazy ? nullptr : m->col_mark;
    A.row = m->s_row;
    A.val = m->s_cval;
    const FmAux x = fm_aux_layout(m, p->K, strata_packed(m, p->K));
    A.r = x.r;
    A.G = x.G;
    A.gs = x.gs;
    A.rs = x.ss;
    if (!p->stale_aux) {  // the changes are only recorded for the refresh
        A.dV = m->dV;
        A.dwn = m->dwn;
    }
    fill_long(m, A, m->lstrat, s, true);
    A.xcd_runs = A.order != nullptr ? 1 : 0;
    FM_TRY(fm_launch_cols(m, A, true, st));
    if (p->stale_aux) return FM_OK;  // Algorithm 1: the aggregates wait for the re-computation
    // phase B: incremental refresh of the aggregates and multipliers
    RowArgs R;
    memset(&R, 0, sizeof(R));
    R.N = m->N;
    R.K = p->K;
    if (p->refresh_all_rows) {
        R.rowptr = m->rowptr;
        R.col = m->col;
        R.val = m->val;
    } else {
        R.col = m->s_col;
        R.val = m->s_val;
        // only the rows that have an entry in this stratum
        R.rows = m->s_touched + m->h_touch_off[s];
        R.rowptr = m->s_touched_beg + m->h_touch_off[s];
        R.N = m->h_touch_off[s + 1] - m->h_touch_off[s];
    }
    R.w0 = w0;
    R.V = m->dV;
    R.big = fm_rows_big(m, p->K);
    R.dwn = m->dwn;
    R.y = y;
    aux_outputs(m, p->K, R, true, strata_packed(m, p->K));
    // An XCD keeps to one run of rows where the aggregates fit half of the chip's L2s (4 MB each) and row blocks are small: up
    // to FM_WHOLE_ROWS rows.  The block that meets a popular column block has most of a stratum's entries, and its XCD most of
    // the work when it fills the XCD's run.  Epochs with runs / without, us: text-like 5e4 rows, K=16, 32 strata 577 / 599;
    // click-style K=16, 64 strata, 6e4 rows 953 / 1001, 1.2e5 1225 / 1298; hashed K=32, 64 strata, 2e4 rows 1510 / 1607,
    // 5e4 1790 / 1868; with planar rows at K=16, half the bytes: text-like 6e4 rows, 32 strata 468 / 506, 2e5, 128 strata 1918 /
    // 2071, click-style 1.2e5, 64 strata 930 / 1044, 2.5e5, 128 strata 2045 / 2237, hashed 2e5, 128 strata 4200 / 4345.  Outside:
    // hashed K=32, 16 strata, 5e4 rows 785 / 753, 2e5, 32 strata 3165 / 2500; K=64, 64 strata, 1.2e5 rows (31 MB) 3635 / 3420;
    // click-style 2.5e5 rows, 16 strata 776 / 708.
    const int64_t aggregates = m->N * R.gs * (int64_t)sizeof(float);
    R.xcd_runs = aggregates <= int64_t(FM_XCDS) << 21 && m->N <= FM_WHOLE_ROWS * m->P ? 1 : 0;
    R.loss = p->loss;
    R.s = p->loss_scale;
    return fm_launch_rows(m, R, true, st);
}

extern "C" int fm_stratified_step(fm_matrix* m, const fm_params* p, int32_t s, const float* y, const float* w0,
                                  float* w, float* V, void* hip_stream)
{
    if (m == nullptr) return FM_EINVAL;
    FM_TRY(check_params(m, p));
    FM_TRY(no_half(m, p));
    if (m->P == 0) return fm_fail(m, FM_ESTATE, "stratified calls need fm_partition first");
    if (s < 0 || s >= m->P) return fm_fail(m, FM_EINVAL, "stratum %d outside [0,%d)", s, m->P);
    if (y == nullptr || w0 == nullptr || w == nullptr || V == nullptr)
        return fm_fail(m, FM_EINVAL, "y, w0, w, V must not be NULL");
    FM_TRY(fm_check_vec_aligned(m, {V}));
    if (m->wsK != p->K || !m->aux_full) return fm_fail(m, FM_ESTATE, "call fm_stratified_begin first");
    return stratified_step(m, p, s, y, w0, w, V, false, (hipStream_t)hip_stream);
}

// The bias step from the multipliers as they stand in the aggregate rows.
static void set_bias_step(fm_matrix* m, const fm_params* p, float* w0, FmEpilogue& E)
{
    const FmAux x = fm_aux_layout(m, p->K, strata_packed(m, p->K));
    set_epilogue(m, E, x.r, m->N, x.ss, true);
    E.w0 = w0;
    E.eta = p->eta;
}

static int stratified_bias_step(fm_matrix* m, const fm_params* p, float* w0, hipStream_t st)
{
    FmEpilogue E;
    set_bias_step(m, p, w0, E);
    return fm_run_epilogue(m, E, st);
}

// lazy_last is zero when an epoch starts: it is made so with the structures, and the flush of an epoch leaves it so.  Only
// what follows an epoch that could not be enqueued to its end clears it, and an epoch that a caller captures: its graph may
// be replayed after such a one.  `sound`, for lazy_clear once the epoch is enqueued: a captured epoch has not run yet.
static int clear_lazy(fm_matrix* m, hipStream_t st, bool* sound)
{
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    const bool known = hipStreamIsCapturing(st, &capture) == hipSuccess;
    if (!known) (void)hipGetLastError();
    const bool captured = !known || capture != hipStreamCaptureStatusNone;
    *sound = !captured || m->lazy_clear;
    if (captured || !m->lazy_clear) FM_TRY(fm_fill_i32(m, m->lazy_last, m->D, 0, st));
    m->lazy_clear = false;
    return FM_OK;
}

extern "C" int fm_stratified_end(fm_matrix* m, const fm_params* p, float* w0, void* hip_stream)
{
    if (m == nullptr) return FM_EINVAL;
    FM_TRY(check_params(m, p));
    if (m->wsK != p->K || !m->aux_full) return fm_fail(m, FM_ESTATE, "call fm_stratified_begin first");
    if (w0 == nullptr) return fm_fail(m, FM_EINVAL, "w0 must not be NULL");
    hipStream_t st = (hipStream_t)hip_stream;
    if (p->update_w0) {
        FM_TRY(stratified_bias_step(m, p, w0, st));
    }
    return FM_OK;
}

// Everything one stratified epoch enqueues (no allocation, no host transfer, no wait).
static int enqueue_stratified_epoch(fm_matrix* m, const fm_params* p, const float* y, float* w0, float* w, float* V,
                                    bool lazy, hipStream_t st)
{
    FM_TRY(run_forward(m, p, y, w0, w, V, nullptr, nullptr, nullptr, nullptr, nullptr, 2, strata_packed(m, p->K), false, st));
    for (int32_t s = 0; s < m->P; ++s) FM_TRY(stratified_step(m, p, s, y, w0, w, V, lazy, st));
    if (lazy) {  // the sums of the bias step beside it
        ColArgs F;
        strat_col_args(m, p, m->P, w, V, true, F);
        if (p->update_w0) set_bias_step(m, p, w0, F.epi);
        FM_TRY(fm_launch_cols_flush(m, F, st));
        if (F.epi.nsums > 0) FM_TRY(fm_run_epilogue_final(m, F.epi, st));
    } else if (p->update_w0) {
        FM_TRY(stratified_bias_step(m, p, w0, st));
    }
    return FM_OK;
}

static bool graph_ready(fm_matrix* m)
{
    if (m->graph_state == 0) {
        m->graph_state = -1;
        if (hipStreamCreateWithFlags(&m->gstream, hipStreamNonBlocking) == hipSuccess &&
            hipEventCreateWithFlags(&m->g_in, hipEventDisableTiming) == hipSuccess &&
            hipEventCreateWithFlags(&m->g_out, hipEventDisableTiming) == hipSuccess)
            m->graph_state = 1;
        else
            (void)hipGetLastError();
    }
    return m->graph_state == 1;
}

// Capture the epoch on the internal stream (or reuse the capture made for the same arguments) and
// replay it between two events on the caller's stream.  Returns FM_ESTATE if no graph could be
// built: the caller then enqueues the epoch directly.
static int replay_stratified_epoch(fm_matrix* m, const fm_params* p, const float* y, float* w0, float* w, float* V,
                                   bool lazy, hipStream_t st)
{
    const void* key[4] = {y, w0, w, V};
    const bool same = m->gexec != nullptr && memcmp(&m->gkey_p, p, sizeof(fm_params)) == 0 &&
                      memcmp(m->gkey_ptr, key, sizeof(key)) == 0 && m->gkey_lazy == lazy;
    if (!same) {
        fm_drop_graph(m);
        (void)fm_side_streams(m);  // created outside the capture
        if (hipStreamBeginCapture(m->gstream, hipStreamCaptureModeThreadLocal) != hipSuccess) {
            (void)hipGetLastError();
            return FM_ESTATE;
        }
        const int rc = enqueue_stratified_epoch(m, p, y, w0, w, V, lazy, m->gstream);
        hipGraph_t graph = nullptr;
        const hipError_t e = hipStreamEndCapture(m->gstream, &graph);
        if (rc != FM_OK || e != hipSuccess || graph == nullptr) {
            (void)hipGetLastError();
            if (graph != nullptr) (void)hipGraphDestroy(graph);
            return FM_ESTATE;
        }
        const hipError_t ei = hipGraphInstantiate(&m->gexec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (ei != hipSuccess) {
            (void)hipGetLastError();
            m->gexec = nullptr;
            return FM_ESTATE;
        }
        m->gkey_p = *p;
        memcpy(m->gkey_ptr, key, sizeof(key));
        m->gkey_lazy = lazy;
    }
    FM_HIP(m, hipEventRecord(m->g_in, st));
    FM_HIP(m, hipStreamWaitEvent(m->gstream, m->g_in, 0));
    FM_HIP(m, hipGraphLaunch(m->gexec, m->gstream));
    FM_HIP(m, hipEventRecord(m->g_out, m->gstream));
    FM_HIP(m, hipStreamWaitEvent(st, m->g_out, 0));
    return FM_OK;
}

extern "C" int fm_stratified_epoch(fm_matrix* m, const fm_params* p, const float* y, float* w0, float* w, float* V,
                                   double* objective, void* hip_stream)
{
    if (m == nullptr) return FM_EINVAL;
    FM_TRY(check_params(m, p));
    FM_TRY(no_half(m, p));
    if (m->P == 0) return fm_fail(m, FM_ESTATE, "stratified calls need fm_partition first");
    if (y == nullptr || w0 == nullptr || w == nullptr || V == nullptr)
        return fm_fail(m, FM_EINVAL, "y, w0, w, V must not be NULL");
    FM_TRY(fm_check_vec_aligned(m, {V}));
    hipStream_t st = (hipStream_t)hip_stream;
    FM_TRY(ensure_strat_ws(m, p->K));
    // The refresh of a stratum reads the change of a column only where the column has entries in
    // its cell, so the regulariser-only steps of the other columns can wait (not when every row
    // is refreshed from every column's change).
    const bool lazy = (!p->refresh_all_rows || p->stale_aux) && m->lazy_last != nullptr && m->opt.lazy_reg;
    // Replay from a graph costs two events, the graph's launch and, first of all, its making (390 us for 16 strata of 5e4 rows),
    // and a kernel in it starts no sooner behind the one before than a kernel on the stream, which the host enqueues three
    // times as fast as the smallest strata run.  Epochs direct / replayed, us: text-like 5e4 rows, 32 strata 441 / 493, 3e3 rows, 32
    // strata 303 / 372; click-style 1e7 rows, 64 strata 26280 / 26340, 5e4 rows, 64 strata 768 / 880; hashed 4e5 rows, K = 64, 64
    // strata 7410 / 7490; uniform 2e3 rows, 4 strata 67 / 94.  It is for callers whose host thread has other things to do.
    bool done = false;
    bool sound = true;
    if (lazy) FM_TRY(clear_lazy(m, st, &sound));
    if (!m->prof && m->opt.graph == 2 && graph_ready(m)) {
        const int rc = replay_stratified_epoch(m, p, y, w0, w, V, lazy, st);
        if (rc == FM_OK)
            done = true;
        else if (rc != FM_ESTATE)
            return rc;
    }
    if (!done) FM_TRY(enqueue_stratified_epoch(m, p, y, w0, w, V, lazy, st));
    if (lazy) m->lazy_clear = sound;
    m->aux_full = true;
    m->aux_held = true;
    return objective != nullptr ? objective_pass(m, p, y, w0, w, V, 2, strata_packed(m, p->K), objective, st) : FM_OK;
}

// ------------------------------------------------------- mini-batch epoch ----

extern "C" int fm_minibatch_epoch(fm_matrix* m, const fm_params* p, const float* y, float* w0, float* w, float* V,
                                  double* objective, void* hip_stream)
{
    if (m == nullptr) return FM_EINVAL;
    FM_TRY(check_params(m, p));
    if (m->B == 0) return fm_fail(m, FM_ESTATE, "fm_minibatch_epoch needs fm_partition_batches first");
    if (y == nullptr || w0 == nullptr || w == nullptr || V == nullptr)
        return fm_fail(m, FM_EINVAL, "y, w0, w, V must not be NULL");
    FM_TRY(fm_check_vec_aligned(m, {V}));
    hipStream_t st = (hipStream_t)hip_stream;
    FM_TRY(ensure_ws(m, p->K));
    m->aux_full = false;
    m->aux_held = true;
    const bool packed = take_packed(m, p->K, m->N / m->B, FM_PLANAR_ROWS_BATCH);
    const FmAux x = fm_aux_layout(m, p->K, packed);
    // a column without entries in a batch only takes the regulariser's step there: postponed
    // until the column next has entries, or the epoch ends
    const bool lazy = m->opt.lazy_reg;
    bool sound = true;
    if (lazy) FM_TRY(clear_lazy(m, st, &sound));
    auto col_args = [&](int32_t b, ColArgs& A) {
        base_col_args(m, p, packed, A);
        A.w = w;
        A.V = V;
        A.P = m->B;
        A.s = b;
        A.batch = 1;
        if (!p->reg_full_per_cell) set_shares(A, m->d_brho, m->d_bb, m->N, m->B);
        if (lazy) A.lazy_last = m->lazy_last;
    };
    int vec = 0, lanes = 0;
    (void)fm_shape_for_K(p->K, &vec, &lanes);  // checked with the parameters
    int32_t* word = layout_word(m, p->K);        // the first pass writes it for all
    for (int32_t b = 0; b < m->B; ++b) {
        const int64_t r0 = m->h_bb[b], nb = m->h_bb[b + 1] - r0;
        RowArgs R;
        bool dense = false;
        if (nb > 0) {  // steps 1-3 on the rows of the batch, at the parameters as they stand
            memset(&R, 0, sizeof(R));
            R.N = nb;
            R.K = p->K;
            R.rowptr = m->rowptr + r0;
            R.col = m->col;
            R.val = m->val;
            R.w0 = w0;
            R.w = w;
            R.V = V;
            R.big = fm_rows_big(m, p->K);
            R.y = y + r0;
            R.G = x.G + r0 * x.gs;
            R.gs = x.gs;
            R.ss = x.ss;
            R.as = x.as;
            R.r = x.r + r0 * x.ss;
            R.whole_rows = packed ? 1 : 0;
            R.aux_rows = word;
            word = nullptr;
            R.row_part = p->update_w0 ? m->row_part : nullptr;
            R.loss = p->loss;
            R.s = p->loss_scale;
            // Batches of few rows whose columns are summed whole (groups of up to eight lanes) are the sparse kernels', us for
            // six batches dense / sparse: 64 columns, K=32 1,000 rows each 108 / 71, 2,000 111 / 89, 4,000 (not whole) 109 / 114;
            // 22 columns, K=8 80 / 59, 82 / 66, 87 / 101.
            dense = fm_dense_takes(m, p, nb, FM_DENSE_FORWARD | FM_DENSE_GRADIENT) &&
                    !(m->lbatch.whole && lanes <= 8 && m->opt.dense_rows != 1 && !p->half_gather);
            if (dense) {
                R.dense_D = (int32_t)m->D;
                R.dense_half = p->half_gather;
                R.val = m->val + r0 * m->D;
            } else {
                FM_TRY(half_copy(m, p, V, &R.Vh, st));  // the factors as they stand
                FM_TRY(fm_launch_rows(m, R, false, st));
            }
        }
        // steps 4-5 over the batch's rows: gradient and step of every column that has entries there
        ColArgs A;
        col_args(b, A);
        A.ptr = nullptr;
        A.mark = lazy ? nullptr : m->col_mark;
        A.row = m->b_row;
        A.val = m->b_cval;
        A.r = x.r;
        A.G = x.G;
        A.gs = x.gs;
        A.rs = x.ss;
        if (!dense) fill_long(m, A, m->lbatch, b, true);
        A.xcd_runs = A.order != nullptr ? 1 : 0;
        if (p->update_w0 && nb > 0) {
            set_epilogue(m, A.epi, m->row_part, dense ? fm_dense_chunks(nb, m->D, p->K) : fm_rows_grid(m, nb, p->K), 0, false);
            if (dense) A.epi.nsums = 0;
            A.epi.w0 = w0;
            A.epi.eta = p->eta;
        }
        if (dense) FM_TRY(dense_step(m, R, false, A, st));
        FM_TRY(fm_launch_cols(m, A, true, st));
    }
    if (lazy) {
        ColArgs F;
        col_args(m->B, F);
        FM_TRY(fm_launch_cols_flush(m, F, st));
        m->lazy_clear = sound;
    }
    return objective != nullptr ? objective_pass(m, p, y, w0, w, V, 1, packed, objective, st) : FM_OK;
}

extern "C" int fm_get_aux(const fm_matrix* m, float* a, float* G, float* q, float* r, void* hip_stream)
{
    if (m == nullptr) return FM_EINVAL;
    fm_matrix* mm = const_cast<fm_matrix*>(m);
    if (m->wsK == 0 || !m->aux_held) return fm_fail(mm, FM_ESTATE, "no aggregates held");
    if ((a != nullptr || q != nullptr) && !m->aux_full)
        return fm_fail(mm, FM_ESTATE, "a and q are only held after a stratified call");
    hipStream_t st = (hipStream_t)hip_stream;
    FM_TRY(fm_unpack_aux(mm, packed_possible(m, m->wsK), a, G, q, r, st));
    return FM_OK;
}


// ------------------------------------------------------------- settings ----

extern "C" int fm_set_option(fm_matrix* m, int32_t option, int32_t value)
{
    if (m == nullptr) return FM_EINVAL;
    switch (option) {
        case FM_OPT_AUX_PLANAR:
            if (m->opt.aux != (value == 0 || value == 2 ? value : 1)) {
                FM_HIP(m, hipDeviceSynchronize());
                fm_drop_workspace(m);  // the aggregates change layout
                m->opt.aux = value == 0 || value == 2 ? value : 1;
            }
            return FM_OK;
        case FM_OPT_SIDE_STREAMS:
            m->opt.side_streams = value != 0;
            fm_drop_graph(m);
            return FM_OK;
        case FM_OPT_LAZY_REG:
            m->opt.lazy_reg = value != 0;
            return FM_OK;
        case FM_OPT_DENSE_ROWS:
            m->opt.dense_rows = value == 0 || value == 2 ? value : 1;
            return FM_OK;
        case FM_OPT_WIDE_ADDRESSES:
            m->opt.wide_addresses = value != 0;
            fm_drop_graph(m);
            return FM_OK;
        case FM_OPT_GRAPH:
            if (value < 0 || value > 2) return fm_fail(m, FM_EINVAL, "graph mode %d outside 0..2", value);
            m->opt.graph = value;
            return FM_OK;
    }
    return fm_fail(m, FM_EINVAL, "unknown option %d", option);
}

extern "C" int fm_set_tuning(fm_matrix* m, int32_t seg, int32_t panel, int32_t heavy_per_panel, int32_t vlong,
                             int32_t min_panels)
{
    if (m == nullptr) return FM_EINVAL;
    if (m->has_csc) return fm_fail(m, FM_ESTATE, "fm_set_tuning must come before fm_build_csc");
    FmTune& t = m->tune;
    if (seg > 0) t.seg = seg < 16 ? 16 : seg;
    if (panel > 0) t.panel = panel < 64 ? 64 : panel;
    if (heavy_per_panel > 0) t.heavy_per_panel = heavy_per_panel;
    if (vlong > 0) t.vlong = vlong;
    if (min_panels > 0) t.min_panels = min_panels;
    return FM_OK;
}

extern "C" int fm_set_tile_tuning(fm_matrix* m, int32_t tile_rows, int32_t min_per_tile, int32_t tile_seg)
{
    if (m == nullptr) return FM_EINVAL;
    if (m->has_csc) return fm_fail(m, FM_ESTATE, "fm_set_tile_tuning must come before fm_build_csc");
    FmTune& t = m->tune;
    if (tile_rows > 0) t.tile = tile_rows < 64 ? 64 : tile_rows;
    if (min_per_tile >= 0) t.tile_min = min_per_tile;
    if (tile_seg > 0) t.tile_seg = tile_seg < 16 ? 16 : tile_seg;
    return FM_OK;
}
