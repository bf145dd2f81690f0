// Internal declarations shared by the translation units of libfm_mi355x.so.
// gfx950 only: 64-lane wavefronts are assumed throughout.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <initializer_list>
#include <string>
#include <vector>

#include "fm.h"
#include "fm_panels.h"

constexpr int FM_WAVE = 64;
constexpr int FM_BLOCK = 256;             // threads per workgroup of the pass kernels
constexpr int FM_WAVES = FM_BLOCK / FM_WAVE;
constexpr int FM_MAXP = 1 << 20;       // row blocks / batches
constexpr int FM_MAXP_CELLS = 4096;     // the P x P table of entries per cell is only kept up to this P
constexpr int64_t FM_ENTRY_PAD = 16;      // entries by which the arrays of entries (index, value) are longer than they need be
// Panels are for matrices of so many rows; below, the aggregate rows of up to 128 bytes stay in the caches in any order (7e4 text-like rows, in panels / without, K = 8
// 61 / 53, K = 64 108 / 121; 5e4 rows, K = 16 44 / 35, K = 64 72 / 82; 1e5 rows, K = 16 56 / 59, K = 64 95 / 118).
constexpr int64_t FM_PANEL_ROWS = 63 * 1024 + 1;

// Tunables of the column-side work decomposition, per handle (fm_set_tuning, fm_set_tile_tuning;
// tile, tile_min < 0, tile_seg: 0 or negative = chosen per latent size, see fm_tile_shape).
struct FmTune {
    int seg = 0;               // entries per work item of a long column; 0: by the number of entries, fm_item_length
    int panel = 32768;         // rows per panel of the L2-blocked traversal of heavy columns
    int heavy_per_panel = 16;  // a column is heavy if it averages at least this many entries per panel
    int vlong = 128;           // columns with more items than this are finished by a whole workgroup (128 against 512,
                               // items of 128: mini-batch click epoch K=32 1.63 and 1.67 ms, stratified table K=64 934
                               // and 959 us, hashed epoch K=64 2.50 and 2.48 ms)
    int min_panels = 0;        // set: panels are halved until there are so many, and matrices with fewer have none; 0: see
                               // fm_panel_rows, from FM_PANEL_ROWS rows on
    int tile = 0;              // rows per LDS tile of the kernel for dense-ish columns
    int tile_min = -1;         // a column is dense-ish if it averages this many entries per tile (0: none)
    int tile_seg = 0;          // entries per item inside a tile
};

// Per-handle switches between code paths that compute the same thing (fm_set_option).
struct FmOptions {
    int aux = 0;               // layout of the aggregates: 0 as take_packed chooses, 1 planar, 2 packed where that exists
    bool side_streams = true;  // column kernels that touch disjoint columns overlap on internal side streams
    bool lazy_reg = true;      // regulariser-only steps of a stratified or mini-batch epoch are postponed
    int graph = 1;             // stratified epoch from a captured graph: 2; directly: 0, 1
    int dense_rows = 2;        // matrices that store every column in every row take the dense (MFMA) kernels: 0 never, 1 always,
                               // 2 where fm_dense_takes says that they are the faster ones
    bool wide_addresses = false;  // gathers take 64-bit addresses at any size
};

// Where the handle keeps the aggregates.  Packed (exists when [G | r] fits one 128-byte line: K % 4 == 0,
// K <= 28): one row [G_0..G_{K-1}, r, a, q, pad] per example with a stride that is a multiple of
// 16 floats.  Planar: G dense [N x K], pairs (a, q), and r as a dense vector.
struct FmAux {
    float *G, *r, *a, *q;
    int64_t gs, ss, as;  // floats between rows of G, of r, of a and q
};
// floats per row of partial sums [acc_0..acc_{K-1} | gw | s2 | pad]: a multiple of 32 (128 bytes)
inline int64_t fm_part_stride(int32_t K) { return ((int64_t)K + 2 + 31) / 32 * 32; }
// Arrays up to this size are gathered through a buffer descriptor with offsets of 32 bits (see fm_walk; wide groups use
// 64-bit addresses at any size)
constexpr int64_t FM_BUF_BYTES = 0xFFFFF000LL;
// How the column kernels read the aggregate rows (ColArgs::packed).
enum { FM_PLANAR = 0, FM_PACKED_LANE = 1 };
int64_t fm_aux_floats(const fm_matrix* m, int32_t K, bool packed);
FmAux fm_aux_layout(const fm_matrix* m, int32_t K, bool packed);

enum fm_kernel_id {
    FMK_ROWS_FORWARD = 0,
    FMK_ROWS_REFRESH,
    FMK_COLS,
    FMK_COLS_LONG,  // dense matrices only: items of long columns are part of FMK_COLS
    FMK_COLS_TILE,
    FMK_COLS_FINISH,
    FMK_REDUCE,
    FMK_BIAS,  // no launch of its own any more; the name stays in the list that callers read
    FMK_COUNT
};

// What one workgroup of the CSR check found, written straight to pinned host memory.
struct FmCheck {
    int64_t bad;        // pointers not monotone or outside [0, nnz], or a column outside [0, D)
    int64_t descents;   // entries whose column is not above that of the entry before, minus those that open a row
    int64_t not_dense;  // row i does not start at i * D
};
constexpr int FM_CHECK_BLOCKS = 512;
constexpr size_t FM_PINNED_DOUBLES = 8192;  // of a handle: 8 scalars, then the block results or what a build moves
static_assert(8 + FM_CHECK_BLOCKS * sizeof(FmCheck) / sizeof(double) <= FM_PINNED_DOUBLES, "room for the CSR check");

// Columns of a stratum or batch hold at most as many entries as a row block (or batch) has rows.  Up to FM_WHOLE_ROWS a
// column is summed at once, by a wavefront, or by a workgroup from FM_WHOLE_WAVE entries on.  Epochs of 8 and 32 strata or
// batches of text-like, click-style and hashed rows and tables, K 4 to 32, whole against in items: 1,100 rows 1.13 to 1.40
// times as fast, 2,000 rows 1.12 to 1.39; 2,300 rows 0.99 to 1.34, 4,000 rows 1.15 to 1.27 at K = 4 but 0.90 (table, K=16;
// text-like, K=32) to 1.14 above.  A wavefront for up to 128 or 512 entries: 0.985 to 1.016 and 0.98 to 1.08 times the time.
constexpr int64_t FM_WHOLE_ROWS = 2048;
constexpr int32_t FM_WHOLE_WAVE = 256;

// Work items for columns longer than `seg` entries (of one matrix, or of all strata
// concatenated).  Offsets in item_beg are global offsets into the entry arrays.  Items of
// a column are numbered consecutively (long_first); partial sums live at the item id, counted from the launch's first item.
struct LongIndex {
    int64_t nlong = 0, nitems = 0;
    int32_t* long_col = nullptr;    // [nlong] column id
    int64_t* long_first = nullptr;  // [nlong+1] first item of each long column
    int32_t* item_col = nullptr;    // [nitems]
    int64_t* item_beg = nullptr;    // [nitems]
    int32_t* item_len = nullptr;    // [nitems]
    std::vector<int64_t> h_long_off, h_item_off;  // per-stratum ranges (size P+1), or {0,nlong}
    // non-empty columns with at most `seg` entries, in column order (per stratum: h_short_off)
    int64_t nshort = 0;
    int32_t* short_col = nullptr;
    int64_t* short_beg = nullptr;   // first entry and number of entries of every listed column
    int32_t* short_len = nullptr;
    std::vector<int64_t> h_short_off;
    // processing order of the full matrix: FM_XCDS lists of item ids, list x walked by the
    // workgroups that run on XCD x, heavy columns panel by panel; of strata and batches: by first row inside each
    // (then all list offsets are 0 and item_beg, item_len are given back); order == nullptr: id order
    uint32_t* order = nullptr;      // [nitems]
    int64_t* ord_beg = nullptr;     // [nitems] item_beg / item_len in processing order
    int32_t* ord_len = nullptr;
    int64_t list_off[FM_XCDS + 1] = {0};
    int64_t list_mid[FM_XCDS] = {0};  // in list x, positions from list_mid[x] on are not panel items
    bool in_panels = false;         // the full matrix: heavy columns are cut at row panels
    // items of dense-ish columns: positions list_off[FM_XCDS]..nitems of `order`, sorted by row tile
    int64_t tile_rows = 0, ntiles = 0;
    int64_t* tile_ptr = nullptr;    // [ntiles+1] positions in `order`
    int32_t* vlong = nullptr;       // [nvlong] indices into long_col of columns with > vlong items
    int64_t nvlong = 0;
    std::vector<int64_t> h_vlong_off;  // per stratum: where its part of vlong starts (the full matrix: all of it)
    // strata and batches of at most FM_WHOLE_ROWS rows: the long columns as they are, for k_cols_whole
    bool whole = false;
    int64_t* long_beg = nullptr;    // [nlong] first entry
    int32_t* long_len = nullptr;    // [nlong] number of entries
    int32_t* big = nullptr;         // indices into long_col of columns with more than FM_WHOLE_WAVE entries
    std::vector<int64_t> h_big_off;  // per stratum
};

struct ProfRec {
    int id;
    hipEvent_t a, b;
};

struct FmAlloc {
    void* p;
    size_t pool_bytes;  // size of a block that goes back to the pool; 0: to the runtime
};

// A value on its way to the host, see fm_read_later.
struct FmRead {
    void* dst;
    size_t at, bytes;  // in the pinned block
};

struct fm_matrix {
    int64_t N = 0, D = 0, nnz = 0;
    FmTune tune;
    FmOptions opt;
    unsigned tile_attr_set = 0;  // bit log2(L): k_cols_tile<L> has been given its dynamic-LDS limit
    // CSR
    int64_t* rowptr = nullptr;
    int32_t* col = nullptr;
    float* val = nullptr;
    // CSC
    bool has_csc = false;
    int64_t* colptr = nullptr;
    int32_t* crow = nullptr;
    float* cval = nullptr;
    LongIndex lfull;
    int lfull_shape[3] = {0, 0, 0};  // tile rows, entries per tile that make a column dense-ish, item length in a tile
    // double partition and per-stratum matrices
    int32_t P = 0;
    std::vector<int64_t> h_rb, h_cb, h_cell_nnz, h_strat_nnz_off;  // bounds, P*P table, P+1 offsets
    int32_t* d_place = nullptr;    // [D] worker every column starts at (fm_partition_placed), nullptr: its column block
    float* d_rho = nullptr;        // [P] share |I_p|/N of the regulariser that a step on row block p applies
    int64_t* d_rb = nullptr;       // [P+1] row block bounds
    int64_t* d_bb = nullptr;       // [B+1] batch bounds
    int32_t* lazy_last = nullptr;  // [D] see ColArgs::lazy_last
    bool lazy_clear = false;       // it is zero when the next epoch starts: the flush of the last one left it so
    // Per-stratum matrices: the entries of X ordered by (stratum, row, column) in s_col/s_val and by
    // (stratum, column, row) in s_row/s_cval.  No pointer array over all P*N rows or P*D columns: only
    // the rows (columns) that have an entry in a stratum are listed, with the offset of their entries.
    int32_t* s_col = nullptr;
    float* s_val = nullptr;
    int32_t* s_row = nullptr;
    float* s_cval = nullptr;
    LongIndex lstrat;
    int32_t* s_touched = nullptr;  // per stratum: the rows with at least one entry there, ascending
    int64_t* s_touched_beg = nullptr;  // [ntouched+1] where the entries of each listed row begin
    int64_t ntouched = 0;
    std::vector<int64_t> h_touch_off;  // [P+1] offsets into s_touched
    int32_t* s_ncol = nullptr;      // the same for the columns of every stratum
    int64_t* s_ncol_beg = nullptr;  // [nncol+1]
    int64_t nncol = 0;
    std::vector<int64_t> h_ncol_off;  // [P+1]
    int32_t* col_mark = nullptr;    // [D] zero between launches; see ColArgs::mark
    // row batches of the mini-batch epoch: per batch the CSC of the matrix restricted to its rows
    int32_t B = 0;
    std::vector<int64_t> h_bb, h_batch_nnz_off;  // [B+1] row bounds, [B+1] offsets into b_row/b_cval
    int32_t* b_row = nullptr;     // entries ordered by (batch, column, row)
    float* b_cval = nullptr;
    int32_t* b_ncol = nullptr;      // the columns with an entry in every batch, and where their entries begin
    int64_t* b_ncol_beg = nullptr;  // [nbcol+1]
    int64_t nbcol = 0;
    std::vector<int64_t> h_bcol_off;  // [B+1]
    LongIndex lbatch;
    float* d_brho = nullptr;  // [B] share |I_b|/N
    // workspace, sized for wsK
    int32_t wsK = 0;
    float* aux = nullptr;   // aggregates, see fm_aux_layout
    _Float16* Vh = nullptr; // [D*K] half-precision copy of V for passes with half_gather (allocated on first use)
    int32_t VhK = 0;        // the K it was sized for
    // Every row stores all D columns in order (col[e] == e % D): `val` is then a dense row-major N x D
    // matrix and passes over all of it or over a batch of rows can run as dense contractions.
    bool is_dense = false;
    float* dV = nullptr;    // [D*K] last step's change of V
    float2* dwn = nullptr;  // [D] (change of w_j, change of |v_j|^2)
    float* part = nullptr;      // [items of the largest launch * part_stride(K)] partial sums, see fm_part_stride
    float* row_part = nullptr;  // [2 * row blocks]: loss, sum r
    double* scal = nullptr;     // device scalars: 0 loss, 1 sum r, 2 |w|^2, 3 |V|^2
    double* h_scal = nullptr;   // pinned: 8 doubles that mirror scal, then one FmCheck per workgroup of k_check_csr, what
                                // fm_evaluate's workgroups leave, or what a build moves (fm_read_later, fm_send)
    bool aux_full = false;      // a, q valid (not only G, r)
    bool aux_held = false;      // the aggregate rows hold the result of a pass (fm_get_aux may read them)
    int32_t* aux_rows = nullptr;  // device, behind scal: 1 where they are packed rows, 0 where planar; see layout_word
    // side streams so that the LDS-bound and the memory-bound column kernels overlap
    hipStream_t side1 = nullptr, side2 = nullptr;
    hipEvent_t ev_fork = nullptr, ev_join1 = nullptr, ev_join2 = nullptr;
    int side_state = 0;  // 0 not tried, 1 ready, -1 unavailable or disabled
    // the stratified epoch as a captured graph (for callers that ask for it), replayed while the
    // caller passes the same parameters and arrays; built on an internal stream
    hipStream_t gstream = nullptr;
    hipEvent_t g_in = nullptr, g_out = nullptr;
    hipGraphExec_t gexec = nullptr;
    fm_params gkey_p = {};
    const void* gkey_ptr[4] = {nullptr, nullptr, nullptr, nullptr};
    bool gkey_lazy = false;
    int graph_state = 0;  // 0 not tried, 1 stream and events ready, -1 unavailable
    // profiling
    bool prof = false;
    std::vector<ProfRec> prof_recs;
    std::vector<hipEvent_t> prof_pool;
    int64_t prof_launches[FMK_COUNT] = {0};
    double prof_ms[FMK_COUNT] = {0};
    // bookkeeping
    int device = 0;  // the device the handle was created on
    std::vector<FmAlloc> allocs;
    // what a build has enqueued and not waited for yet (fm_settle)
    std::vector<void*> spent;
    std::vector<FmRead> reads;
    size_t pin_used = 0;  // bytes of the pinned block behind its scalars
    std::string err;
};

// ---- helpers (fm_api.hip) ----
int fm_fail(fm_matrix* m, int code, const char* fmt, ...);
// the kernels read and write the arrays that hold K floats per row four floats at a time
inline int fm_check_vec_aligned(fm_matrix* m, std::initializer_list<const void*> arrays)
{
    for (const void* a : arrays)
        if ((reinterpret_cast<uintptr_t>(a) & 15u) != 0)
            return fm_fail(m, FM_EINVAL, "device arrays with K floats per row (V, G, grad_V) must be 16-byte aligned");
    return FM_OK;
}
int fm_dev_alloc(fm_matrix* m, void** p, size_t bytes);
void fm_dev_free(fm_matrix* m, void* p);
// Builds enqueue on one stream and wait as rarely as they can: scratch is given up with fm_spend, values are read with
// fm_read_later (dst must live until then) and written with fm_send, and fm_settle waits, delivers the values and gives the
// scratch back.
void fm_spend(fm_matrix* m, std::initializer_list<void*> scratch);
int fm_read_later(fm_matrix* m, void* dst, const void* src, size_t bytes, hipStream_t st);
int fm_send(fm_matrix* m, void* dst, const void* src, size_t bytes, hipStream_t st);
int fm_settle(fm_matrix* m, hipStream_t st);
void fm_unsettled(fm_matrix* m);  // forgets what a build that failed left behind
void fm_drop_workspace(fm_matrix* m);  // forces reallocation after the structures changed
void fm_drop_graph(fm_matrix* m);      // a captured epoch holds pointers into the workspace and the structures
bool fm_side_streams(fm_matrix* m);    // creates them on first use; false if switched off or unavailable

#define FM_HIP(m, expr)                                                                  \
    do {                                                                                 \
        hipError_t e__ = (expr);                                                         \
        if (e__ != hipSuccess)                                                           \
            return fm_fail((m), FM_EHIP, "%s failed: %s", #expr, hipGetErrorString(e__)); \
    } while (0)

#define FM_TRY(expr)          \
    do {                      \
        int rc__ = (expr);    \
        if (rc__ != FM_OK) return rc__; \
    } while (0)

struct ProfScope {
    fm_matrix* m;
    hipStream_t st;
    int id;
    hipEvent_t a = nullptr, b = nullptr;
    ProfScope(fm_matrix* m_, hipStream_t st_, int id_);
    ~ProfScope();
};

// ---- build (fm_build.hip) ----
// Checks the uploaded CSR arrays on the device and sets is_dense; waits for the stream.
int fm_check_csr(fm_matrix* m, hipStream_t st, bool* valid);
int fm_scan_exclusive_i64(fm_matrix* m, int64_t* d, int64_t n, hipStream_t st);
int fm_sort_by_key_u32(fm_matrix* m, uint32_t* keys, uint32_t* idx, uint32_t* keys_alt, uint32_t* idx_alt,
                       int64_t n, int bits, hipStream_t st, bool* result_in_alt);
// ptr[c], ptr[c+1] bound the entries of list position c = 0..ncols_total-1; ids[c] is its column;
// h_bounds[s] (nstrata+1 values) is the first list position of stratum s
int fm_build_long_index(fm_matrix* m, const int64_t* ptr, const int32_t* ids, const int32_t* row, int64_t ncols_total,
                        const std::vector<int64_t>& h_bounds, int32_t nstrata, LongIndex* out, hipStream_t st);
// lfull, with the panel order of heavy columns and the LDS tiles shaped for latent size K (0: unknown)
int fm_build_full_index(fm_matrix* m, int32_t K, hipStream_t st);
void fm_tile_shape(const fm_matrix* m, int32_t K, int* tile_rows, int* tile_min, int* tile_seg);
int fm_item_length(int64_t entries, bool part);  // of a launch over so many entries, all of the matrix or part of it
int fm_ensure_lazy(fm_matrix* m, hipStream_t st);  // allocates and clears lazy_last on first use

// ---- pass kernels (fm_rows.hip / fm_cols.hip / fm_reduce.hip) ----
struct RowArgs {
    int64_t N;
    int32_t K;
    const int64_t* rowptr;
    const int32_t* col;
    const float* val;
    const float* w0;    // device scalar
    const float* w;     // forward: weights
    const float* V;     // forward: factors ; refresh: dV
    const _Float16* Vh; // forward, nullable: gather the rows of V from this half-precision copy instead
    const float2* dwn;  // refresh: (dw_j, dn_j)
    const float* y;     // nullable
    float *yhat, *a, *G, *q, *r;  // forward: nullable outputs ; refresh: in/out aggregates
    int64_t gs;         // floats between consecutive rows of G
    int64_t ss;         // floats between consecutive rows of r (1, or the aggregate row stride)
    int64_t as;         // ... of a and q (2: they are pairs and move as one float2)
    int32_t whole_rows; // packed aggregate rows: r, a, q move as one float4 (forward: and the padding is written with them)
    int32_t* aux_rows;  // forward into the handle's aggregates: takes whole_rows; nullable
    float* row_part;    // nullable: [2*gridDim] loss and sum r per block
    double* eval_part;  // nullable: [3*gridDim] sums of losses, squared errors and correct signs per block
    int32_t big;          // what is gathered (V, its half copy or dV, dwn) is larger than FM_BUF_BYTES
    int32_t dense_D;      // forward: > 0 when `val` is a dense row-major N x dense_D matrix (col is then not read)
    int32_t dense_half;   // ... whose scores take V rounded to half precision (the kernel rounds it: no copy)
    int32_t xcd_runs;     // refresh: the rows in FM_XCDS runs, one per XCD, and not dealt out one workgroup after the other
    const int32_t* rows;  // nullable: the launch covers rows[0..N) instead of rows 0..N-1, and
                          // rowptr[k], rowptr[k+1] bound the entries of rows[k]
    int32_t loss;
    float s;
};
// RowArgs::big of a row kernel that gathers K floats per column, and up to two more beside them
inline int32_t fm_rows_big(const fm_matrix* m, int32_t K)
{
    return m->D * std::max<int64_t>(K, 2) * (int64_t)sizeof(float) > FM_BUF_BYTES || m->opt.wide_addresses ? 1 : 0;
}
int fm_launch_rows(fm_matrix* m, const RowArgs& A, bool refresh, hipStream_t st);
struct DenseArgs;
void fm_dense_rows(const RowArgs& A, DenseArgs* E);  // the forward pass A as a dense one
constexpr int64_t FM_SPLIT_LANES = 1 << 21;  // see fm_rows_split
int fm_rows_split(const fm_matrix* m, int64_t N, int32_t K, int lanes);
int64_t fm_rows_grid(const fm_matrix* m, int64_t N, int32_t K);      // workgroups of a forward pass over N rows
int64_t fm_rows_max_grid(const fm_matrix* m, int64_t N, int32_t K);  // ... and the most of one over a block of them
// once per device, with that device current: resolves the address of the static scratch array of
// fm_forward_noalloc (fm_noalloc.hip); called when a handle is created
int fm_noalloc_init_device(fm_matrix* m);
int fm_keep_aux(fm_matrix* m, bool packed, const float* r, const float* G, hipStream_t st);  // the caller's; K a multiple of 4
int fm_to_half(fm_matrix* m, const float* x, _Float16* out, int64_t n, hipStream_t st);  // round to nearest even
// dense matrices (fm_dense.hip)
bool fm_dense_fits(const fm_matrix* m, int32_t K);           // the dense kernels exist for this matrix and K
int64_t fm_dense_chunks(int64_t N, int64_t D, int32_t K);    // workgroups of a pass over N rows; never fewer for more rows
int fm_dense_parts(int64_t N, int64_t D, int32_t K);         // items that one of them leaves for a column
enum { FM_DENSE_FORWARD = 1, FM_DENSE_GRADIENT = 2 };
// ... and take such a pass over so many rows
bool fm_dense_takes(const fm_matrix* m, const fm_params* p, int64_t rows, int what);
int fm_launch_dense(fm_matrix* m, const DenseArgs& A, int what, hipStream_t st);  // gradient: partial sums; the finish follows
int fm_unpack_aux(fm_matrix* m, bool rows_exist, float* a, float* G, float* q, float* r, hipStream_t st);

// What is left of an epoch when the columns have stepped: the sums over the examples, the bias step and the figures of
// the objective.  One workgroup, which rides along with the last column kernel.
struct FmEpilogue {
    int32_t on;
    const float* x;        // raw values, one pair (loss, multiplier) per row block or, with single, one multiplier per row
    int64_t n, stride;
    int32_t single;
    double* sums;          // [2 * nsums] partial pairs of x, written by the kernel before (nsums == 0: x is read as it is)
    int32_t nsums;
    const double* regs;    // nullable: [2 * nregs] partial pairs (|w|^2, |V|^2)
    int32_t nregs;
    const float *reg_w, *reg_V;  // nullable: the parameters themselves instead, while nothing else of the launch steps them
    int64_t reg_nw, reg_nV;
    float* w0;             // nullable: takes the bias step
    float eta;
    float* grad_w0;        // nullable
    double* scal;          // device: loss, sum of the multipliers
    double* host;          // nullable, pinned: loss, sum of the multipliers, |w|^2, |V|^2
};
constexpr int FM_EPI_DIRECT = 2048;  // values the epilogue sums itself; above, workgroups of the kernel before do
constexpr int64_t FM_EPI_REG = 1 << 15;  // parameters whose squares the epilogue adds up itself
constexpr int FM_EPI_CHUNK = 4096;   // ... one for so many values
inline int fm_epi_nsums(int64_t n)
{
    if (n <= FM_EPI_DIRECT) return 0;
    const int64_t nb = (n + FM_EPI_CHUNK - 1) / FM_EPI_CHUNK;
    return (int)(nb < 512 ? nb : 512);
}

// Workgroups of k_cols that work on consecutive items of a stratum or batch on one XCD.  Epochs with 1 / 4 / 8 / 16 / 64, us:
// strata, K = 16: click-style 1e7 rows, 64 strata 26345 / 26244 / 26214 / 26292 / 30400, 1.25e6 rows, 16 strata 2779 / 2714 /
// 2693 / 2682 / 3020, text-like 2e5 rows 774 / 764 / 762 / 766 / -, hashed 4e5 rows, K = 32 4289 / 4290 / 4288 / 4296 / -;
// batches: click-style 156,250 rows, K = 16 - / 2413 / 2398 / 2390 / - (an eighth of the batch to an XCD: 2479), 312,500
// rows, K = 8 - / 984 / 969 / 965 / - (990), text-like 25,000 rows - / 364 / 367 / 366 / - (372).  Longer runs are uneven.
constexpr int FM_RUN_BLOCKS = 8;

struct ColArgs {
    int64_t D;
    int32_t K;
    const int64_t* ptr;  // [D+1] global offsets of the full matrix (which columns are empty); nullptr for a stratum or batch
    const int32_t* row;
    const float* val;
    const float* r;
    const float* G;
    int64_t gs, rs;  // row strides of G and r in floats
    // > 0: a dense pass has left the partial sums of all columns, those of column j at the items
    // j * ndense .. (j + 1) * ndense - 1; only the finish is left
    int64_t ndense;
    int32_t packed;  // FM_PLANAR, or FM_PACKED_LANE: G rows are packed aggregate rows [G | r | a | q | pad]
    float* w;        // updated in place when update
    float* V;
    float* grad_w;   // !update: outputs (nullable)
    float* grad_V;
    float* dV;       // delta outputs (nullable)
    float2* dwn;
    const int32_t* short_col;  // list of the short non-empty columns of this launch
    const int64_t* short_beg;  // first entry and number of entries of every listed column
    const int32_t* short_len;
    int64_t nshort;
    // nullable, with ptr == nullptr and steps taken at once: every column that takes its step from data sets
    // mark[j] = 1, and the kernel of the columns without entries skips the marked ones and clears the mark
    int32_t* mark;
    float lambda_w, lambda_v, eta;
    // regulariser share: rho = 1 when rho == nullptr, else rho[p] = |I_p|/N with p = (c(j) - s) mod P, where
    // c(j) = place[j], or the column block of j when place == nullptr
    const int32_t* place;
    const float* rho;
    const int64_t* rb;           // with rho: [P+1] bounds of the row blocks (strata) or batches
    float rho_small, rho_big;    // with rho: the shares of a block of floor(N/P) rows and of one more
    int64_t N;
    int32_t P, s;
    int32_t batch;  // 1: steps are row batches, step t acts on row block t (else on (colblock - t) mod P)
    // nullable, update only: lazy_last[j] = number of strata of this epoch whose step column j has
    // taken.  A column that is empty in a cell only feels the regulariser there; with this array
    // those steps are postponed until the column next has entries (or the epoch ends) and then
    // taken as one multiplication, so no pass over the columns that are empty in a stratum is needed.
    int32_t* lazy_last;
    // long-column items
    const int32_t* long_col;
    const int64_t* long_first;
    const int32_t* item_col;
    const int64_t* item_beg;
    const int32_t* item_len;
    int64_t nlong, nitems;        // counts of this launch
    int64_t long_base, item_base;  // first long column / first item of this launch (absolute ids)
    const uint32_t* order;         // nullable: item ids in processing order, FM_XCDS lists and what follows them
    const int64_t* ord_beg;        // with order: item_beg / item_len in processing order
    const int32_t* ord_len;
    int64_t list_off[FM_XCDS + 1];
    int64_t list_mid[FM_XCDS];
    int64_t tile_rows, ntiles;     // dense-ish columns: items sorted by row tile, after the lists
    const int64_t* tile_ptr;
    int64_t lin_base, lin_count;   // positions of `order` that are taken in sequence (tile items that are not staged; all of a stratum or batch)
    int32_t xcd_runs;              // the lin items in runs of FM_RUN_BLOCKS workgroups to an XCD, not dealt out one after the other
    int32_t long_runs;             // runs are added up in fp64 but for a few entries, see FM_LONG_RUNS
    int64_t blk_lists, blk_lin, blk_short;  // workgroups of k_cols per role, in this order; then epi.nsums for the sums
    int32_t nt;                    // gathers of rows that are not used again soon carry the non-temporal hint
    int32_t big;                   // the gathered array is larger than FM_BUF_BYTES
    FmEpilogue epi;
    // strata and batches of few rows: long columns summed whole (k_cols_whole)
    int32_t whole;
    const int64_t* long_beg;
    const int32_t* long_len;
    const int32_t* big_cols;       // the nbig of them that a workgroup sums
    int64_t nbig;
    const int32_t* vlong;          // nullable: long columns finished by a whole workgroup
    int64_t nvlong;
    int32_t vlong_items;           // threshold that defines vlong
    float* part;                    // rows [acc | gw | s2 | pad] of ps floats, indexed by absolute item id: the rows from item_base on are there
    int64_t ps;
};
int fm_launch_cols(fm_matrix* m, const ColArgs& A, bool update, hipStream_t st);
// takes the postponed regulariser steps of every column up to stratum A.s (exclusive)
int fm_launch_cols_flush(fm_matrix* m, const ColArgs& A, hipStream_t st);

// A pass over rows of a dense matrix (fm_dense.hip).
struct DenseArgs {
    int64_t N, D;
    int32_t K;
    int64_t nchunks;
    const float* X;  // row-major N x D
    const float *w0, *w, *V, *y;  // forward; y nullable
    int32_t half;                 // forward: V rounded to half precision
    float *yhat, *a, *G, *q, *r;  // forward: nullable outputs; gradient alone: G and r are read
    int64_t gs, ss, as;           // floats between rows of G, of r, of a and q
    int32_t whole_rows;           // forward: packed aggregate rows [G | r | a | q | pad] go out whole
    int32_t loss;
    int32_t* aux_rows;            // forward into the handle's aggregates: takes whole_rows; nullable
    float s;
    float* row_part;    // forward, nullable: [2 * nchunks] loss and sum of r per workgroup
    double* eval_part;  // forward alone, nullable: [3 * nchunks] sums of losses, squared errors and correct signs
    float* part;        // gradient: partial sums, rows of ps floats, nparts items to a column and workgroup
    int64_t ps;
    int32_t nparts;
    FmEpilogue epi;     // gradient alone: on = the sums over the examples ride along
    double* regs;       // nullable, without epi: one more workgroup leaves |w|^2 and |V|^2 there
};

constexpr int FM_REG_PAIRS = 512;      // partial pairs of fm_reg_partials
constexpr int FM_REDUCE_TMP = 2048;  // doubles of stage-1 scratch a reduction may use
// tmp: FM_REDUCE_TMP doubles of device scratch, or nullptr for the handle's own
int fm_reduce_pairs(fm_matrix* m, const float* part, int64_t nblocks, double* out2, hipStream_t st,
                    double* tmp = nullptr);
double* fm_reg_scratch(fm_matrix* m);  // 2 * FM_REG_PAIRS doubles in the handle's scratch
// |w|^2 and |V|^2 as nregs partial pairs of doubles in the handle's scratch
int fm_reg_partials(fm_matrix* m, const float* w, int64_t nw, const float* V, int64_t nV, const double** regs, int32_t* nregs,
                    hipStream_t st);
int fm_reduce_eval(fm_matrix* m, const double* part, int64_t n, double* out3, double* tmp, hipStream_t st);
int fm_run_epilogue(fm_matrix* m, const FmEpilogue& E, hipStream_t st);  // as kernels of its own
int fm_run_epilogue_final(fm_matrix* m, const FmEpilogue& E, hipStream_t st);  // ... where another launch left the partial sums
int fm_fill_i32(fm_matrix* m, int32_t* x, int64_t n, int32_t v, hipStream_t st);

// lanes per row/column group and floats per lane for a given K; false if K unsupported
bool fm_shape_for_K(int32_t K, int* vec, int* lanes);
