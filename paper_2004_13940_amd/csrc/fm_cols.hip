// Column-side kernels: the atomic-free transposed product for the gradient
// (eqs. updates_w, updates_v) over a CSC copy, with the parameter step fused in.
//
//   gw_j   = sum_i x_ij r_i
//   s2_j   = sum_i x_ij^2 r_i
//   gV_jk  = sum_i x_ij r_i G_ik
//   grad_w_j  = gw_j + rho lambda_w w_j
//   grad_V_jk = gV_jk - s2_j v_jk + rho lambda_v v_jk
//
// A group of L lanes owns one column (lane `sub` holds VEC latent dimensions).
// Columns longer than `seg` entries are cut into items: k_cols finishes the shorter ones and
// writes one partial sum per item, and k_cols_finish adds the partials of a column in a
// fixed order, so results are bit-reproducible from run to run.  Items of heavy
// columns are cut at row-panel boundaries and handed out panel by panel, one panel at a
// time per XCD, so that the gathered rows of G stay in that XCD's L2.
#include "fm_device.h"
#include "fm_epilogue.h"
#include "fm_internal.h"

namespace {

// The multiplier of an entry of planar aggregates: x r, with r an array of its own.
template <class SUM>
struct OwnMultiplier {
    struct T {
        float r[1];
    };
    FmOwnArray<1> r;
    SUM gw, s2;            // this lane's entries
    float round_w, round_2;  // in fp64: those of the round
    template <int ADDR>
    __device__ __forceinline__ T load(int i) const
    {
        T t;
        r.template get<ADDR>(i, t.r);
        return t;
    }
    __device__ __forceinline__ float use(T t, float x)
    {
        const float xr = x * t.r[0];
        if constexpr (std::is_same_v<SUM, double>) {
            round_w += xr;
            round_2 += x * xr;
        } else {
            gw += xr;
            s2 += x * xr;
        }
        return xr;
    }
    __device__ __forceinline__ void end_round()
    {
        if constexpr (std::is_same_v<SUM, double>) {
            gw += (double)round_w;
            s2 += (double)round_2;
            round_w = round_2 = 0.f;
        }
    }
};

// How a run is added up.  Where columns are cut at panels a run is up to 256 entries long, and one chain of fp32 additions rounds
// each at the size of all before it: a few entries (eight; 16 of packed rows, for the registers; four in wide groups) are added
// in fp32, these sums in fp64, and the run is rounded once.  Sums of one sign over columns of 2e5 rows, 0.5 % and 5 % dense, items
// of 128: share of results that are not the nearest float, one chain 0.27 and 0.14, fp32 sums of 16 0.14 and 0.05, now 0.08
// and 0.02 (packed 0.13 and 0.04).  Costs 0 to 2 % of an epoch (text-like 2e5 rows, K = 16 181 -> 183 us; hashed 4e5 rows, K = 64 2210
// -> 2240; click-style 1e7 rows nothing).  Elsewhere runs keep to fp32: those of strata and batches are of up to 48 entries unless
// the caller sets their length (click-style 1.5e6 rows, K = 20, 32 strata 5802, with fp64 5932; 3e5 rows, K = 16 782, 796), those
// of short matrices as long as the entries leave work for all compute units (2e4 text-like rows, K = 20 39.9, 41.0).
enum { FM_LONG_RUNS = 0, FM_SHORT_RUNS = 1 };

// Sums of the run of `len` entries from beg on: acc, this lane's latent slice; gw, s2 on every lane of the group.  All
// groups of the wavefront call it together.
template <int VEC, int L, int PACKED, int ADDR, int RUNS>
__device__ __forceinline__ void walk_column(const ColArgs& A, int64_t beg, int len, int sub, int kbase, bool kact,
                                            float (&acc)[VEC], float& gw, float& s2)
{
    using Sum = std::conditional_t<RUNS == FM_SHORT_RUNS, float, double>;
    Sum sum[VEC] = {}, sum_w = 0, sum_2 = 0;
    if constexpr (PACKED == FM_PACKED_LANE) {
        // lanes past the latent ones, at least the last of the group, read the scalars [r | a | q | pad]
        fm_walk<VEC, L, FM_WALK_PACKED, ADDR>(A.row, A.val, beg, len, A.G, A.gs, sub, kact ? kbase : A.K, sum, sum_w, sum_2,
                                              FmOwnNone());
        gw = (float)sum_w;
        s2 = (float)sum_2;
    } else if constexpr (L >= FM_WIDE_GROUP) {
        const float* __restrict__ r = A.r;
        const int64_t rs = A.rs;
        float g = 0.f, s = 0.f;
        fm_walk_wide<VEC, L>(A.row, A.val, beg, beg + len, A.G, A.gs, sub, kact ? kbase : 0, sum, [&](int i, float x) {
            const float xr = x * r[(int64_t)i * rs];
            g += xr;
            s += x * xr;
            return xr;
        });
        gw = fm_group_sum<L>(g);
        s2 = fm_group_sum<L>(s);
    } else {
        OwnMultiplier<Sum> own{FmOwnArray<1>(A.r, A.rs), 0, 0, 0.f, 0.f};
        fm_walk<VEC, L, FM_WALK_SUM, ADDR>(A.row, A.val, beg, len, A.G, A.gs, sub, kact ? kbase : 0, sum, sum_w, sum_2, own);
        gw = fm_group_sum<L>((float)own.gw);
        s2 = fm_group_sum<L>((float)own.s2);
    }
#pragma unroll
    for (int z = 0; z < VEC; ++z) acc[z] = (float)sum[z];
}

// once: the gathered rows are not used again soon
template <int VEC, int L, int PACKED, int RUNS>
__device__ __forceinline__ void accumulate_entries(const ColArgs& A, bool once, int64_t beg, int len, int sub, int kbase,
                                                   bool kact, float (&acc)[VEC], float& gw, float& s2)
{
    if (L >= FM_WIDE_GROUP || A.big)
        walk_column<VEC, L, PACKED, FM_ADDR_PTR, RUNS>(A, beg, len, sub, kbase, kact, acc, gw, s2);
    else if (once && A.nt)
        walk_column<VEC, L, PACKED, FM_ADDR_BUF_NT, RUNS>(A, beg, len, sub, kbase, kact, acc, gw, s2);
    else
        walk_column<VEC, L, PACKED, FM_ADDR_BUF, RUNS>(A, beg, len, sub, kbase, kact, acc, gw, s2);
}

// The class of column j that decides which row block it meets in which stratum: its column block in
// the ring of Section 4.2, or the worker it was placed at when columns travel one by one (Section 4.3).
__device__ __forceinline__ int32_t column_class(const ColArgs& A, int64_t j)
{
    if (A.rho == nullptr || A.batch) return 0;
    return A.place != nullptr ? A.place[j] : fm_block_of(j, A.D, A.P);
}

// Share of the regulariser that the step of stratum t applies to a column of class qb.
__device__ __forceinline__ float reg_share(const ColArgs& A, int32_t qb, int32_t t)
{
    if (A.rho == nullptr) return 1.f;
    if (A.batch) return A.rho[t];
    int32_t p = (qb - t) % A.P;
    if (p < 0) p += A.P;
    return A.rho[p];
}

// A column with no entries in its cell only feels the regulariser: x <- x - eta rho lambda x,
// taken as one rounded multiplication by c = 1 - eta (rho lambda).
__device__ __forceinline__ float step_factor(float rho, float lambda, float eta)
{
    return __fsub_rn(1.f, __fmul_rn(eta, __fmul_rn(rho, lambda)));
}

__device__ __forceinline__ double pow_int(double c, uint32_t n)
{
    double r = 1.0;
    while (n != 0) {
        if (n & 1u) r *= c;
        c *= c;
        n >>= 1;
    }
    return r;
}

// Postponed regulariser-only steps t0 .. t1-1 of a column of column block qb, as one factor each
// for v_j and w_j.  The floor split makes row blocks of two sizes only, so the steps have two
// factors only, and the run is  c_small^(n - n_big) * c_big^(n_big)  with n_big read off the block
// bounds; the product is formed in fp64 and rounded once, which is closer to the exact product than
// the n rounded multiplications of steps taken one by one (a single step gives its factor exactly).
__device__ __forceinline__ void catch_up_factors(const ColArgs& A, int32_t qb, int32_t t0, int32_t t1, float& fv,
                                                 float& fw)
{
    fv = fw = 1.f;
    const int32_t n = t1 - t0;
    if (n <= 0) return;
    if (A.rho == nullptr) {  // every step applies the whole regulariser
        fv = (float)pow_int((double)step_factor(1.f, A.lambda_v, A.eta), (uint32_t)n);
        fw = (float)pow_int((double)step_factor(1.f, A.lambda_w, A.eta), (uint32_t)n);
        return;
    }
    int64_t rows;  // rows of the row blocks that the steps t0 .. t1-1 act on
    if (A.batch) {
        rows = A.rb[t1] - A.rb[t0];
    } else {  // blocks p0, p0-1, ..., cyclically
        int32_t p0 = (qb - t0) % A.P;
        if (p0 < 0) p0 += A.P;
        const int32_t lo = p0 - n + 1;
        rows = lo >= 0 ? A.rb[p0 + 1] - A.rb[lo] : (A.rb[p0 + 1] - A.rb[0]) + (A.rb[A.P] - A.rb[A.P + lo]);
    }
    const int64_t base = A.N / A.P;  // rows of a small block; a big one has one more
    const uint32_t n_big = (uint32_t)(rows - (int64_t)n * base);
    const uint32_t n_small = (uint32_t)n - n_big;
    fv = (float)(pow_int((double)step_factor(A.rho_small, A.lambda_v, A.eta), n_small) *
                 pow_int((double)step_factor(A.rho_big, A.lambda_v, A.eta), n_big));
    fw = (float)(pow_int((double)step_factor(A.rho_small, A.lambda_w, A.eta), n_small) *
                 pow_int((double)step_factor(A.rho_big, A.lambda_w, A.eta), n_big));
}

// What the step of column j needs besides the data sums; asked for early, so that it overlaps the gathers.  Every lane
// loads (an inactive slice: the first), no branch: nothing has to be waited for before the entries are asked for.
template <int VEC>
struct ColState {
    float v[VEC];
    float w;
    float rho;   // share of the regulariser
    int32_t qb;  // class of the column
    int32_t t0;  // first stratum whose step the column has not taken yet
};

template <int VEC, bool UPDATE>
__device__ __forceinline__ ColState<VEC> load_column(const ColArgs& A, int64_t j, int kbase, bool kact)
{
    ColState<VEC> c;
    fm_load_vec<VEC>(A.V + j * A.K + (kact ? kbase : 0), c.v);
    c.w = A.w[j];
    c.t0 = A.s;
    if constexpr (UPDATE) {
        if (A.lazy_last != nullptr) c.t0 = A.lazy_last[j];
    }
    c.qb = column_class(A, j);
    c.rho = reg_share(A, c.qb, A.s);
    return c;
}

// Turn the data sums of column j into the gradient, and either store it or take the
// step (optionally recording the change for the incremental refresh).
template <int VEC, int L, bool UPDATE>
__device__ __forceinline__ void finish_column(const ColArgs& A, int64_t j, int sub, int kbase, bool kact,
                                              const float (&acc)[VEC], float gw, float s2, ColState<VEC> c)
{
    const int K = A.K;
    const float rho = c.rho;
    float fv = 1.f, fw = 1.f;
    if (c.t0 < A.s) catch_up_factors(A, c.qb, c.t0, A.s, fv, fw);  // postponed regulariser-only steps
    float dn = 0.f;
    if (kact) {
        float g[VEC];
        if (c.t0 < A.s) {
#pragma unroll
            for (int z = 0; z < VEC; ++z) c.v[z] = __fmul_rn(c.v[z], fv);
        }
        const float rl = __fmul_rn(rho, A.lambda_v);
#pragma unroll
        for (int z = 0; z < VEC; ++z) g[z] = __fmaf_rn(rl, c.v[z], __fmaf_rn(-s2, c.v[z], acc[z]));
        if constexpr (UPDATE) {
            float d[VEC], vn[VEC];
#pragma unroll
            for (int z = 0; z < VEC; ++z) {
                d[z] = __fmul_rn(-A.eta, g[z]);
                vn[z] = __fadd_rn(c.v[z], d[z]);
                dn += d[z] * (2.f * c.v[z] + d[z]);  // |v+d|^2 - |v|^2 without cancellation
            }
            fm_store_vec<VEC>(A.V + j * K + kbase, vn);
            if (A.dV != nullptr) fm_store_vec<VEC>(A.dV + j * K + kbase, d);
        } else {
            if (A.grad_V != nullptr) fm_store_vec<VEC>(A.grad_V + j * K + kbase, g);
        }
    }
    if constexpr (UPDATE) {
        if (A.dwn != nullptr) dn = fm_group_sum<L>(dn);
    }
    if (sub == 0) {
        float wj = c.w;
        if (c.t0 < A.s) wj = __fmul_rn(wj, fw);
        const float g = __fmaf_rn(__fmul_rn(rho, A.lambda_w), wj, gw);
        if constexpr (UPDATE) {
            const float d = __fmul_rn(-A.eta, g);
            A.w[j] = __fadd_rn(wj, d);
            if (A.dwn != nullptr) A.dwn[j] = make_float2(d, dn);
            if (A.lazy_last != nullptr) A.lazy_last[j] = A.s + 1;
            if (A.mark != nullptr) A.mark[j] = 1;  // this column has taken its step from data
        } else {
            if (A.grad_w != nullptr) A.grad_w[j] = g;
        }
    }
}

// Partial sums of item `it`: one row [acc_0..acc_{K-1} | gw | s2 | pad] of A.ps floats, a whole
// number of 128-byte lines.  Items are written in processing order and read in column order, so
// the rows are scattered: with float4 lanes the group writes the whole row, padding included, so
// that no line is left partly written.
template <int VEC, int L>
__device__ __forceinline__ void store_partial(const ColArgs& A, int64_t it, int sub, int kbase, bool kact,
                                              const float (&acc)[VEC], float gw, float s2)
{
    float* __restrict__ row = A.part + it * A.ps;
    if constexpr (VEC == 4) {
        for (int o = sub * 4; o < A.ps; o += L * 4) {
            float z[4] = {0.f, 0.f, 0.f, 0.f};
            if (o < A.K) {
#pragma unroll
                for (int t = 0; t < 4; ++t) z[t] = acc[t];  // first pass only: o == kbase
            } else if (o == A.K) {
                z[0] = gw;
                z[1] = s2;
            }
            fm_store_vec<4>(row + o, z);
        }
    } else {
        if (kact) fm_store_vec<VEC>(row + kbase, acc);
        if (sub == 0) {
            row[A.K] = gw;
            row[A.K + 1] = s2;
        }
    }
}

// The columns without an LDS tile, one launch: a workgroup is either one of blk_lists / blk_lin workgroups that take the
// items of long columns (one group per item, a partial sum each), one of blk_short that take the short columns (1..seg
// entries; one group per column, which finishes it), or one of the epilogue's that add up the examples.  The kinds touch
// disjoint data; as launches of their own they needed a fork and a join of streams, which cost a stratum of the text-like
// workload as much as its columns did.  Items come first: they are the longest runs.
// With an order array, workgroup b takes its items from list b % FM_XCDS (the XCD it runs on).  Items of strata and batches are
// in row order; with xcd_runs every XCD takes FM_RUN_BLOCKS workgroups of that order in a run, and the rows and multipliers
// that the items of a run share are asked for by one L2.
template <int VEC, int L, bool UPDATE, int PACKED, int RUNS>
__device__ __forceinline__ void cols_block(const ColArgs& A)
{
    constexpr int R = FM_WAVE / L;
    const int lane = threadIdx.x & (FM_WAVE - 1);
    const int wave = threadIdx.x / FM_WAVE;
    const int sub = lane & (L - 1);
    const int slot = wave * R + lane / L;
    const int kbase = sub * VEC;
    const bool kact = kbase < A.K;
    int64_t b = blockIdx.x;
    const int64_t blk_items = A.blk_lists + A.blk_lin;
    if (b >= blk_items + A.blk_short) {
        __shared__ double sh[FM_WAVES];
        fm_epi_partial<FM_BLOCK>(A.epi, (int)(b - blk_items - A.blk_short), sh);
        return;
    }
    const bool items = b < blk_items;
    float acc[VEC];
#pragma unroll
    for (int z = 0; z < VEC; ++z) acc[z] = 0.f;
    float gw = 0.f, s2 = 0.f;
    int64_t id = -1, beg = 0;  // item or column
    int len = 0;
    bool once = true;
    ColState<VEC> c = {};
    if (items) {
        if (b >= A.blk_lists) {
            int64_t lb = b - A.blk_lists;
            if (A.xcd_runs) {
                const int64_t k = lb / FM_XCDS;
                lb = (k / FM_RUN_BLOCKS * FM_XCDS + lb % FM_XCDS) * FM_RUN_BLOCKS + k % FM_RUN_BLOCKS;
            }
            const int64_t rel = lb * (FM_WAVES * R) + slot;
            once = false;
            if (rel < A.lin_count) {
                const int64_t pos = A.lin_base + rel;
                id = A.order[pos];
                beg = A.ord_beg[pos];
                len = A.ord_len[pos];
            }
        } else if (A.order != nullptr) {
            const int x = (int)(b % FM_XCDS);
            const int64_t first = A.list_off[x] + (b / FM_XCDS) * (FM_WAVES * R);
            once = first >= A.list_mid[x];  // not an item of a heavy column inside a panel: those gather their rows again soon
            if (first + slot < A.list_off[x + 1]) {
                id = A.order[first + slot];
                beg = A.ord_beg[first + slot];
                len = A.ord_len[first + slot];
            }
        } else {
            const int64_t pos = b * (FM_WAVES * R) + slot;
            if (pos < A.nitems) {
                id = A.item_base + pos;
                beg = A.item_beg[id];
                len = A.item_len[id];
            }
        }
    } else {
        const int64_t pos = (b - blk_items) * (FM_WAVES * R) + slot;
        const int64_t p = pos < A.nshort ? pos : A.nshort - 1;
        const int64_t j = A.short_col[p];
        beg = A.short_beg[p];
        len = A.short_len[p];
        c = load_column<VEC, UPDATE>(A, j, kbase, kact);
        if (pos < A.nshort)
            id = j;
        else
            len = 0;
    }
    accumulate_entries<VEC, L, PACKED, RUNS>(A, once, beg, len, sub, kbase, kact, acc, gw, s2);
    if (id < 0) return;
    if (items)
        store_partial<VEC, L>(A, id, sub, kbase, kact, acc, gw, s2);
    else
        finish_column<VEC, L, UPDATE>(A, id, sub, kbase, kact, acc, gw, s2, c);
}

// Wavefronts to a SIMD that the compiler must leave room for, where it would not by itself with the sums in fp64 and does
// without spilling.
constexpr int cols_waves(int vec, int l, int packed, bool update, bool few)
{
    if (l >= FM_WIDE_GROUP) return 8;
    return vec == 4 && !few && ((packed == FM_PLANAR && l == 4) || (packed == FM_PACKED_LANE && l == 8 && update)) ? 5 : 1;
}

// FEW: four wavefronts to a SIMD and not the five that its registers leave room for, by naming a register that nothing uses
// (LDS, the other means, is what k_cols_tile beside it lives on).  The items in panel order then have fewer panels' rows in
// flight and find more of them in the L2: see few_wavefronts.
template <int VEC, int L, bool UPDATE, int PACKED, bool FEW = false>
__global__ __launch_bounds__(FM_BLOCK, cols_waves(VEC, L, PACKED, UPDATE, FEW)) void k_cols(const ColArgs A)
{
    if constexpr (FEW) asm volatile("" ::: "v103");
    cols_block<VEC, L, UPDATE, PACKED, FM_LONG_RUNS>(A);
}

// Strata, batches and matrices without panels.
template <int VEC, int L, bool UPDATE, int PACKED>
__global__ __launch_bounds__(FM_BLOCK, L >= FM_WIDE_GROUP ? 8 : 1) void k_cols_part(const ColArgs A)
{
    cols_block<VEC, L, UPDATE, PACKED, FM_SHORT_RUNS>(A);
}

// Columns with nothing stored (in this matrix or stratum) only feel the regulariser; one group
// of LE = K/VEC lanes per column over all D columns, consecutive groups on consecutive columns
// so that V is streamed.  The gradient is finish_column with zero data sums; the step is the
// multiplication by the step factor.  A group takes FM_EMPTY_U columns, one from each of as many
// consecutive slabs of columns: the tests for emptiness are all issued before the first row of V
// is asked for, and all rows before the first is written, so that the kernel is not one memory
// round trip after the other per column.
constexpr int FM_EMPTY_U = 4;
template <int VEC, int LE, bool UPDATE>
__global__ __launch_bounds__(FM_BLOCK) void k_cols_empty(const ColArgs A)
{
    constexpr int R = FM_WAVE / LE;
    constexpr int U = FM_EMPTY_U;
    const int lane = threadIdx.x & (FM_WAVE - 1);
    const int wave = threadIdx.x / FM_WAVE;
    const int sub = lane & (LE - 1);
    const int grp = lane / LE;
    const int kbase = sub * VEC;
    const bool kact = kbase < A.K;
    int64_t j[U];
    bool todo[U];  // uniform inside a group
#pragma unroll
    for (int u = 0; u < U; ++u) {
        j[u] = ((int64_t)blockIdx.x * U + u) * (FM_WAVES * R) + wave * R + grp;
        todo[u] = j[u] < A.D;
        if (todo[u]) {
            if (A.ptr != nullptr) {
                todo[u] = A.ptr[j[u] + 1] == A.ptr[j[u]];
            } else {  // a stratum or batch: the columns with entries marked themselves; the marks are left clear
                const bool marked = A.mark[j[u]] != 0;
                if (marked && sub == 0) A.mark[j[u]] = 0;
                todo[u] = !marked;
            }
        }
    }
    if constexpr (!UPDATE) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!todo[u]) continue;
            float acc[VEC];
#pragma unroll
            for (int z = 0; z < VEC; ++z) acc[z] = 0.f;
            finish_column<VEC, LE, false>(A, j[u], sub, kbase, kact, acc, 0.f, 0.f,
                                          load_column<VEC, false>(A, j[u], kbase, kact));
        }
    } else {
        float v[U][VEC];
        float wj[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int z = 0; z < VEC; ++z) v[u][z] = 0.f;
            wj[u] = 0.f;
            if (todo[u] && kact) fm_load_vec<VEC>(A.V + j[u] * A.K + kbase, v[u]);
            if (todo[u] && sub == 0) wj[u] = A.w[j[u]];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!todo[u]) continue;
            const int32_t qb = column_class(A, j[u]);
            const float rho = reg_share(A, qb, A.s);
            float dn = 0.f;
            if (kact) {
                const float f = step_factor(rho, A.lambda_v, A.eta);
                float vn[VEC], d[VEC];
#pragma unroll
                for (int z = 0; z < VEC; ++z) {
                    vn[z] = __fmul_rn(v[u][z], f);
                    d[z] = vn[z] - v[u][z];
                    dn += d[z] * (2.f * v[u][z] + d[z]);
                }
                fm_store_vec<VEC>(A.V + j[u] * A.K + kbase, vn);
                if (A.dV != nullptr) fm_store_vec<VEC>(A.dV + j[u] * A.K + kbase, d);
            }
            if (A.dwn != nullptr) dn = fm_group_sum<LE>(dn);
            if (sub == 0) {
                const float wn = __fmul_rn(wj[u], step_factor(rho, A.lambda_w, A.eta));
                A.w[j[u]] = wn;
                if (A.dwn != nullptr) A.dwn[j[u]] = make_float2(wn - wj[u], dn);
            }
        }
    }
}

// The postponed regulariser steps of every column, strata lazy_last[j] .. A.s-1; one group of LE
// lanes per column, consecutive columns in consecutive groups.  Leaves lazy_last at zero for the next epoch.  The
// workgroups behind the columns: the epilogue's.
template <int VEC, int LE>
__global__ __launch_bounds__(FM_BLOCK) void k_cols_flush(const ColArgs A)
{
    constexpr int R = FM_WAVE / LE;
    const int lane = threadIdx.x & (FM_WAVE - 1);
    const int wave = threadIdx.x / FM_WAVE;
    const int sub = lane & (LE - 1);
    const int grp = lane / LE;
    const int64_t cols = (A.D + FM_WAVES * R - 1) / (FM_WAVES * R);
    if (blockIdx.x >= cols) {
        __shared__ double sh[FM_WAVES];
        if (A.epi.nsums > 0)
            fm_epi_partial<FM_BLOCK>(A.epi, (int)(blockIdx.x - cols), sh);
        else
            fm_epi_final<FM_BLOCK>(A.epi, sh);
        return;
    }
    const int64_t j = (int64_t)blockIdx.x * (FM_WAVES * R) + wave * R + grp;
    if (j >= A.D) return;  // whole groups leave together
    const int32_t t0 = A.lazy_last[j];
    if (sub == 0) A.lazy_last[j] = 0;
    if (t0 >= A.s) return;
    const int32_t qb = column_class(A, j);
    float fv, fw;
    catch_up_factors(A, qb, t0, A.s, fv, fw);
    const int kbase = sub * VEC;
    if (kbase < A.K) {
        float v[VEC];
        fm_load_vec<VEC>(A.V + j * A.K + kbase, v);
#pragma unroll
        for (int z = 0; z < VEC; ++z) v[z] = __fmul_rn(v[z], fv);
        fm_store_vec<VEC>(A.V + j * A.K + kbase, v);
    }
    if (sub == 0) A.w[j] = __fmul_rn(A.w[j], fw);
}

// Dense-ish columns, LDS-staged: workgroup t copies G and r of the tile_rows rows of row tile t
// (packed or planar aggregates) into LDS once, then its groups walk the tile's items
// (pieces of dense-ish columns whose rows lie inside the tile) and gather G and r from LDS.
// One partial sum per item, as in k_cols.  L lanes of VEC=4 latent dimensions per group.
template <int L>
__global__ __launch_bounds__(FM_BLOCK) void k_cols_tile(const ColArgs A)
{
    constexpr int VEC = 4;
    constexpr int NG = FM_BLOCK / L;
    // Beside k_cols, which waits for memory most of the time: its wavefronts go first where both could issue (click-style
    // gradient, 1e7 rows 4585 -> 4538 us, 6e6 rows, K=12 2524 -> 2490; text-like, 1e6 rows 796 -> 795).
    __builtin_amdgcn_s_setprio(3);
    extern __shared__ float tile[];  // G part: tile_rows x K floats, then r: tile_rows floats
    const int K = A.K;
    const int S = K;
    float* __restrict__ tile_r = tile + A.tile_rows * K;
    const int chunks = K / VEC;  // float4 chunks of G per row
    const int64_t t = blockIdx.x;
    const int64_t row0 = t * A.tile_rows;
    const int64_t nrows = (A.N - row0) < A.tile_rows ? (A.N - row0) : A.tile_rows;
    {   // copy in batches of eight float4 per thread: all loads of a batch are issued before the first store
        const int total = (int)nrows * chunks;
        const float* __restrict__ src = A.G + row0 * A.gs;
        const float* __restrict__ rsrc = A.r + row0 * A.rs;
        constexpr int U = 8;
        for (int c0 = threadIdx.x; c0 < total; c0 += U * FM_BLOCK) {
            float4 v[U];
            int dst[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = c0 + u * FM_BLOCK;
                const int cc = c < total ? c : total - 1;
                const int rr = cc / chunks, ch = cc - rr * chunks;
                dst[u] = c < total ? (rr << 8) | ch : -1;  // chunks <= 64 for every K of this path
                v[u] = *reinterpret_cast<const float4*>(src + (int64_t)rr * A.gs + ch * VEC);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (dst[u] < 0) continue;
                const int rr = dst[u] >> 8, ch = dst[u] & 255;
                *reinterpret_cast<float4*>(tile + rr * S + ch * VEC) = v[u];
            }
        }
        // r of the rows (a loop of its own: no branch between the loads of a batch above)
        for (int rr = threadIdx.x; rr < (int)nrows; rr += FM_BLOCK) tile_r[rr] = rsrc[(int64_t)rr * A.rs];
    }
    __syncthreads();

    const int sub = threadIdx.x & (L - 1);
    const int grp = threadIdx.x / L;
    const int kbase = sub * VEC;
    const bool kact = kbase < K;
    const int kb = kact ? kbase : 0;
    const int64_t pend = A.tile_ptr[t + 1];
    for (int64_t pos = A.tile_ptr[t] + grp; pos < pend; pos += NG) {
        const int64_t it = A.order[pos];
        const int64_t beg = A.ord_beg[pos];
        const int64_t end = beg + A.ord_len[pos];
        float acc[VEC] = {0.f, 0.f, 0.f, 0.f};
        float gw = 0.f, s2 = 0.f;
        constexpr int CH = L < 16 ? 16 / L : 1;  // entry slots per lane and iteration
        for (int64_t e = beg; e < end; e += L * CH) {
            int il[CH];
            float xr[CH];
#pragma unroll
            for (int u = 0; u < CH; ++u) {  // own entries: index and value from global memory
                const int64_t my = e + u * L + sub;
                const bool has = my < end;
                const int64_t mc = has ? my : end - 1;
                il[u] = (int)((int64_t)A.row[mc] - row0);
                xr[u] = has ? A.val[mc] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < CH; ++u) {  // r of the own entry from LDS
                const float x = xr[u];
                xr[u] = x * tile_r[il[u]];
                gw += xr[u];
                s2 += x * xr[u];
            }
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                fm_static_for<0, L>([&](auto tc) {
                    constexpr int T = decltype(tc)::value;
                    const int ir = fm_bcast_i<L, T>(il[u]);
                    const float mt = fm_bcast_f<L, T>(xr[u]);
                    const float4 g = *reinterpret_cast<const float4*>(tile + ir * S + kb);
                    acc[0] += mt * g.x;
                    acc[1] += mt * g.y;
                    acc[2] += mt * g.z;
                    acc[3] += mt * g.w;
                });
            }
        }
        gw = fm_group_sum<L>(gw);
        s2 = fm_group_sum<L>(s2);
        store_partial<4, L>(A, it, sub, kbase, kact, acc, gw, s2);
    }
}

// Sum of the partials first, first+step, ... < last of one column, in fp64 and in that
// order; eight loads are issued before the first add so that the loop is not one memory
// round trip per item.
template <int VEC>
__device__ __forceinline__ void add_partials(const ColArgs& A, int64_t first, int64_t last, int64_t step, int kbase,
                                             bool kact, double (&acc)[VEC], double& gw, double& s2)
{
    constexpr int U = 8;
    const int kb = kact ? kbase : 0;
    int64_t it = first;
    for (; it + (U - 1) * step < last; it += U * step) {
        float p[U][VEC];
        float g0[U], g1[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float* __restrict__ row = A.part + (it + u * step) * A.ps;
            fm_load_vec<VEC>(row + kb, p[u]);
            g0[u] = row[A.K];
            g1[u] = row[A.K + 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int z = 0; z < VEC; ++z) acc[z] += (double)p[u][z];
            gw += (double)g0[u];
            s2 += (double)g1[u];
        }
    }
    for (; it < last; it += step) {
        const float* __restrict__ row = A.part + it * A.ps;
        float p[VEC];
        fm_load_vec<VEC>(row + kb, p);
#pragma unroll
        for (int z = 0; z < VEC; ++z) acc[z] += (double)p[z];
        gw += (double)row[A.K];
        s2 += (double)row[A.K + 1];
    }
}

// Sum over the wavefront's groups; lanes with equal `sub` hold the same latent slice.  Fixed butterfly order.
template <int VEC, int L>
__device__ __forceinline__ void add_groups(double (&acc)[VEC], double& gw, double& s2)
{
    if constexpr (L < FM_WAVE) {
#pragma unroll
        for (int z = 0; z < VEC; ++z) acc[z] += fm_xor_lane<L>(acc[z]);
        gw += fm_xor_lane<L>(gw);
        s2 += fm_xor_lane<L>(s2);
        add_groups<VEC, 2 * L>(acc, gw, s2);
    }
}

// The long columns from their partial sums, one launch.  Workgroups 0..nvlong-1: one column of more than vlong_items
// items each (group g of the workgroup adds items g, g+NG, ... in fp64, every wavefront adds its groups by the butterfly,
// and the first group adds the wavefronts and finishes the column).  The workgroups after them: one wavefront per long
// column, the listed ones left out.  The last workgroup, if epi.on: the sums over the examples and the bias step.
// What bounds it is the serial chain of loads of a column, not registers: the same 108 for every lane count.  One group
// adding all NG group totals from LDS, unrolled, spilled below 8 lanes (epoch of 49,990 x 22, K=4: 109.6 us, now 34.5).
template <int VEC, int L, bool UPDATE>
__global__ __launch_bounds__(FM_BLOCK) void k_cols_finish(const ColArgs A)
{
    constexpr int R = FM_WAVE / L;
    constexpr int NG = FM_BLOCK / L;  // groups per workgroup
    constexpr int S = L * VEC + 2;    // doubles per wavefront
    __shared__ double sh[FM_WAVES * S];
    const int lane = threadIdx.x & (FM_WAVE - 1);
    const int wave = threadIdx.x / FM_WAVE;
    const int sub = threadIdx.x & (L - 1);
    const int kbase = sub * VEC;
    const bool kact = kbase < A.K;
    double acc[VEC];
#pragma unroll
    for (int z = 0; z < VEC; ++z) acc[z] = 0.0;
    double gw = 0.0, s2 = 0.0;
    const int64_t b = blockIdx.x;
    if (A.epi.on && b == (int64_t)gridDim.x - 1) {
        fm_epi_final<FM_BLOCK>(A.epi, sh);
        return;
    }
    int64_t lc, j;
    ColState<VEC> c;  // asked for ahead of the partial sums
    const bool dense = A.ndense > 0;  // every column has the same number of items
    if (b < A.nvlong) {
        lc = dense ? b : A.vlong[b];
        const int64_t first = dense ? lc * A.ndense : A.long_first[lc];
        const int64_t last = dense ? first + A.ndense : A.long_first[lc + 1];
        j = dense ? lc : A.long_col[lc];
        c = load_column<VEC, UPDATE>(A, j, kbase, kact);
        add_partials<VEC>(A, first + threadIdx.x / L, last, NG, kbase, kact, acc, gw, s2);
        add_groups<VEC, L>(acc, gw, s2);
        double* mine = sh + wave * S;
        if (lane < L) {
#pragma unroll
            for (int z = 0; z < VEC; ++z) mine[kbase + z] = acc[z];
            if (sub == 0) {
                mine[L * VEC] = gw;
                mine[L * VEC + 1] = s2;
            }
        }
        __syncthreads();
        if (threadIdx.x >= L) return;
#pragma unroll
        for (int w = 1; w < FM_WAVES; ++w) {  // wavefront 0 is the one that adds
#pragma unroll
            for (int z = 0; z < VEC; ++z) acc[z] += sh[w * S + kbase + z];
            gw += sh[w * S + L * VEC];
            s2 += sh[w * S + L * VEC + 1];
        }
    } else {
        const int64_t rel = (b - A.nvlong) * FM_WAVES + wave;
        if (rel >= A.nlong) return;  // whole wavefront leaves together
        lc = A.long_base + rel;
        const int64_t first = dense ? lc * A.ndense : A.long_first[lc];
        const int64_t last = dense ? first + A.ndense : A.long_first[lc + 1];
        if (A.nvlong > 0 && last - first > A.vlong_items) return;
        j = dense ? lc : A.long_col[lc];
        c = load_column<VEC, UPDATE>(A, j, kbase, kact);
        add_partials<VEC>(A, first + lane / L, last, R, kbase, kact, acc, gw, s2);
        add_groups<VEC, L>(acc, gw, s2);
        if (lane >= L) return;
    }
    float accf[VEC];
#pragma unroll
    for (int z = 0; z < VEC; ++z) accf[z] = (float)acc[z];
    finish_column<VEC, L, UPDATE>(A, j, sub, kbase, kact, accf, (float)gw, (float)s2, c);
}

// A stratum or batch of few rows (FM_WHOLE_ROWS), groups of up to eight lanes: every column is summed where it is finished,
// no partial sums and no second launch.  Workgroups: one per column of more than FM_WHOLE_WAVE entries (its groups take
// consecutive slices, added in fp64 as k_cols_finish does), then one wavefront per other long column, one group per short
// column, the sums over the examples, and, where nobody has to add those up first, the bias step.  Bound: latency, list ->
// entries -> gathers -> step; what goes is a launch and the round trip of the partial sums (stratum of the text-like
// workload, 5e4 rows, 32 strata: columns and finish 14.0 us, now 9.2).
template <int VEC, int L, int PACKED>
__global__ __launch_bounds__(FM_BLOCK) void k_cols_whole(const ColArgs A)
{
    constexpr int R = FM_WAVE / L;
    constexpr int NG = FM_BLOCK / L;
    constexpr int S = L * VEC + 2;
    constexpr int ROUND = 16;  // entries of a round of the walk
    __shared__ double sh[FM_WAVES * S];
    const int lane = threadIdx.x & (FM_WAVE - 1);
    const int wave = threadIdx.x / FM_WAVE;
    const int sub = lane & (L - 1);
    const int kbase = sub * VEC;
    const bool kact = kbase < A.K;
    const int64_t b = blockIdx.x;
    const int64_t waves_end = A.nbig + A.blk_lin;
    if (b >= waves_end + A.blk_short) {
        if (A.epi.nsums > 0)
            fm_epi_partial<FM_BLOCK>(A.epi, (int)(b - waves_end - A.blk_short), sh);
        else
            fm_epi_final<FM_BLOCK>(A.epi, sh);
        return;
    }
    const bool big = b < A.nbig, whole = b < waves_end;  // uniform
    int64_t j, beg;
    int len;
    bool valid = true;
    if (whole) {
        const int64_t rel = big ? 0 : (b - A.nbig) * FM_WAVES + wave;
        valid = big || rel < A.nlong;
        const int64_t lc = big ? A.big_cols[b] : A.long_base + (valid ? rel : 0);
        j = A.long_col[lc];
        beg = A.long_beg[lc];
        const int n = A.long_len[lc];
        valid = valid && (big || n <= FM_WHOLE_WAVE);
        const int groups = big ? NG : R, group = big ? (int)threadIdx.x / L : lane / L;
        const int slice = ((n + groups - 1) / groups + ROUND - 1) / ROUND * ROUND;
        const int at = group * slice;
        len = !valid || at >= n ? 0 : n - at < slice ? n - at : slice;
        beg += at;
    } else {
        const int64_t pos = (b - waves_end) * (FM_WAVES * R) + wave * R + lane / L;
        valid = pos < A.nshort;
        const int64_t p = valid ? pos : A.nshort - 1;
        j = A.short_col[p];
        beg = A.short_beg[p];
        len = valid ? A.short_len[p] : 0;
    }
    const ColState<VEC> c = load_column<VEC, true>(A, j, kbase, kact);
    float acc[VEC];
#pragma unroll
    for (int z = 0; z < VEC; ++z) acc[z] = 0.f;
    float gw = 0.f, s2 = 0.f;
    accumulate_entries<VEC, L, PACKED, FM_SHORT_RUNS>(A, false, beg, len, sub, kbase, kact, acc, gw, s2);
    if (whole) {
        double accd[VEC];
#pragma unroll
        for (int z = 0; z < VEC; ++z) accd[z] = (double)acc[z];
        double gwd = (double)gw, s2d = (double)s2;
        add_groups<VEC, L>(accd, gwd, s2d);
        if (big) {
            double* mine = sh + wave * S;
            if (lane < L) {
#pragma unroll
                for (int z = 0; z < VEC; ++z) mine[kbase + z] = accd[z];
                if (sub == 0) {
                    mine[L * VEC] = gwd;
                    mine[L * VEC + 1] = s2d;
                }
            }
            __syncthreads();
            valid = wave == 0;
#pragma unroll
            for (int w = 1; w < FM_WAVES; ++w) {  // wavefront 0 is the one that adds
#pragma unroll
                for (int z = 0; z < VEC; ++z) accd[z] += sh[w * S + kbase + z];
                gwd += sh[w * S + L * VEC];
                s2d += sh[w * S + L * VEC + 1];
            }
        }
        valid = valid && lane < L;
#pragma unroll
        for (int z = 0; z < VEC; ++z) acc[z] = (float)accd[z];
        gw = (float)gwd;
        s2 = (float)s2d;
    }
    if (valid) finish_column<VEC, L, true>(A, j, sub, kbase, kact, acc, gw, s2, c);
}

// LDS-staged kernel for the tile items; false if the tile does not fit in LDS for this K
// (the caller then runs the items through k_cols).
template <int L>
bool launch_tile_l(fm_matrix* m, const ColArgs& A, size_t lds, hipStream_t st)
{
    constexpr unsigned bit = 1u << __builtin_ctz((unsigned)L);
    if (!(m->tile_attr_set & bit)) {  // opt in once per handle to more than the default 64 KB of dynamic LDS
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_cols_tile<L>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 256) != hipSuccess) {
            (void)hipGetLastError();
            if (lds > 64 * 1024) return false;
        }
        m->tile_attr_set |= bit;
    }
    hipLaunchKernelGGL((k_cols_tile<L>), dim3((unsigned)A.ntiles), dim3(FM_BLOCK), lds, st, A);
    return true;
}

inline size_t tile_lds(const ColArgs& A) { return (size_t)A.tile_rows * (size_t)(A.K + 1) * sizeof(float); }

// at least two workgroups per compute unit, or the copy of one tile cannot overlap the work on another
inline bool tile_fits(const ColArgs& A)
{
    return A.ntiles > 0 && A.ntiles <= 0x7fffffffLL && A.K % 4 == 0 && tile_lds(A) <= 72 * 1024;
}

inline bool launch_tile(fm_matrix* m, const ColArgs& A, hipStream_t st)
{
    const size_t lds = tile_lds(A);
    int need = A.K / 4, l = 1;
    while (l < need) l <<= 1;
    switch (l) {
        case 1: return launch_tile_l<1>(m, A, lds, st);
        case 2: return launch_tile_l<2>(m, A, lds, st);
        case 4: return launch_tile_l<4>(m, A, lds, st);
        case 8: return launch_tile_l<8>(m, A, lds, st);
        case 16: return launch_tile_l<16>(m, A, lds, st);
        case 32: return launch_tile_l<32>(m, A, lds, st);
        case 64: return launch_tile_l<64>(m, A, lds, st);
    }
    return false;
}

// k_cols_empty with LE = smallest power of two >= K/VEC lanes per column
template <int VEC, int LE>
int launch_empty_l(fm_matrix* m, const ColArgs& A, bool update, hipStream_t st)
{
    const int64_t per = (int64_t)FM_WAVES * (FM_WAVE / LE) * FM_EMPTY_U;
    const int64_t grid = (A.D + per - 1) / per;
    if (grid > 0x7fffffffLL) return fm_fail(m, FM_ERANGE, "column grid too large");
    if (update)
        hipLaunchKernelGGL((k_cols_empty<VEC, LE, true>), dim3((unsigned)grid), dim3(FM_BLOCK), 0, st, A);
    else
        hipLaunchKernelGGL((k_cols_empty<VEC, LE, false>), dim3((unsigned)grid), dim3(FM_BLOCK), 0, st, A);
    FM_HIP(m, hipGetLastError());
    return FM_OK;
}

template <int VEC>
int launch_empty(fm_matrix* m, const ColArgs& A, bool update, hipStream_t st)
{
    int need = A.K / VEC, l = 1;
    while (l < need) l <<= 1;
    switch (l) {
        case 1: return launch_empty_l<VEC, 1>(m, A, update, st);
        case 2: return launch_empty_l<VEC, 2>(m, A, update, st);
        case 4: return launch_empty_l<VEC, 4>(m, A, update, st);
        case 8: return launch_empty_l<VEC, 8>(m, A, update, st);
        case 16: return launch_empty_l<VEC, 16>(m, A, update, st);
        case 32: return launch_empty_l<VEC, 32>(m, A, update, st);
        case 64: return launch_empty_l<VEC, 64>(m, A, update, st);
    }
    return fm_fail(m, FM_EINVAL, "unsupported K=%d", A.K);
}

template <int VEC, int LE>
int launch_flush_l(fm_matrix* m, const ColArgs& A, hipStream_t st)
{
    const int64_t per = (int64_t)FM_WAVES * (FM_WAVE / LE);
    const int64_t grid = (A.D + per - 1) / per + (A.epi.on ? std::max<int64_t>(A.epi.nsums, 1) : 0);
    if (grid > 0x7fffffffLL) return fm_fail(m, FM_ERANGE, "column grid too large");
    ProfScope ps(m, st, FMK_COLS);
    hipLaunchKernelGGL((k_cols_flush<VEC, LE>), dim3((unsigned)grid), dim3(FM_BLOCK), 0, st, A);
    FM_HIP(m, hipGetLastError());
    return FM_OK;
}

template <int VEC>
int launch_flush(fm_matrix* m, const ColArgs& A, hipStream_t st)
{
    int need = A.K / VEC, l = 1;
    while (l < need) l <<= 1;
    switch (l) {
        case 1: return launch_flush_l<VEC, 1>(m, A, st);
        case 2: return launch_flush_l<VEC, 2>(m, A, st);
        case 4: return launch_flush_l<VEC, 4>(m, A, st);
        case 8: return launch_flush_l<VEC, 8>(m, A, st);
        case 16: return launch_flush_l<VEC, 16>(m, A, st);
        case 32: return launch_flush_l<VEC, 32>(m, A, st);
        case 64: return launch_flush_l<VEC, 64>(m, A, st);
    }
    return fm_fail(m, FM_EINVAL, "unsupported K=%d", A.K);
}

// From so many floats of V on the empty columns run beside the others, which are bound by latency while those stream
// (gradient of 4e5 hashed rows, D = 4e6, K=64: 2525 -> 2480 us; of 2e6 rows, D = 2e7: 14.27 -> 14.11 ms).  Below, the fork
// and the join cost more than they give (1e5 rows, D = 1e6: 603 -> 607 us), and so does a third kernel beside the LDS-staged one
// (click-style epoch, 1e7 rows: 7.31 -> 7.98 ms).
constexpr int64_t FM_EMPTY_BESIDE = int64_t(1) << 27;

// Columns of a matrix whose aggregate rows do not fit the memory-side cache (256 MB): what the L2 does not hold comes from
// HBM.  Click-style gradient, K=16, five wavefronts / four, us: 1e7 rows 4538 / 4495, 5e6 rows 2316 / 2267, 2.5e6 rows (320
// MB) 1246 / 1244; epoch 7139 / 7131, 3607 / 3570, 1895 / 1890.  Below it the fifth hides latency: text-like, 1e6 rows (128
// MB) 795 / 844.
inline bool few_wavefronts(const ColArgs& A)
{
    return A.ptr != nullptr && A.N * A.gs * (int64_t)sizeof(float) > int64_t(256) << 20;
}

template <int VEC, int L, int PACKED>
int launch_cols_t(fm_matrix* m, const ColArgs& A, bool update, hipStream_t st)
{
    constexpr int R = FM_WAVE / L;
    const int64_t per = FM_WAVES * R;
    if (A.nlong > 0x7fffffffLL) return fm_fail(m, FM_ERANGE, "column grid too large");
    int64_t ntile_items = A.order != nullptr ? A.nitems - A.list_off[FM_XCDS] : 0;
    // columns without entries only feel the regulariser (skipped when there is none and nothing records the
    // change, or when such steps are postponed)
    const bool need_empty =
        (A.lambda_w != 0.f || A.lambda_v != 0.f || !update || A.dV != nullptr) && A.lazy_last == nullptr;
    ColArgs Am = A;
    if (!need_empty || A.ptr != nullptr) Am.mark = nullptr;  // marks are only set when a kernel will clear them
    if constexpr (L < FM_WIDE_GROUP) {
        if (A.whole && A.ndense == 0 && update) {
            Am.blk_lin = (A.nlong + FM_WAVES - 1) / FM_WAVES;
            Am.blk_short = (A.nshort + per - 1) / per;
            const int64_t sums = A.epi.on ? std::max<int64_t>(A.epi.nsums, 1) : 0;
            const int64_t grid = A.nbig + Am.blk_lin + Am.blk_short + sums;
            if (grid > 0x7fffffffLL) return fm_fail(m, FM_ERANGE, "column grid too large");
            if (grid > 0) {
                ProfScope ps(m, st, FMK_COLS);
                hipLaunchKernelGGL((k_cols_whole<VEC, L, PACKED>), dim3((unsigned)grid), dim3(FM_BLOCK), 0, st, Am);
                FM_HIP(m, hipGetLastError());
            }
            if (A.epi.on && A.epi.nsums > 0) {  // added up by now
                Am.nlong = Am.nvlong = 0;
                ProfScope ps(m, st, FMK_COLS_FINISH);
                hipLaunchKernelGGL((k_cols_finish<VEC, L, true>), dim3(1), dim3(FM_BLOCK), 0, st, Am);
                FM_HIP(m, hipGetLastError());
            }
            if (need_empty && A.ptr == nullptr && A.D > 0) {
                ProfScope ps(m, st, FMK_COLS);
                FM_TRY((launch_empty<VEC>(m, Am, true, st)));
            }
            return FM_OK;
        }
    }
    if (A.ndense == 0) {  // else a dense pass has left the partial sums of every column
        // LDS-staged items go to a side stream, so that the LDS-bound kernel overlaps the memory-bound one (not while
        // per-kernel timing is on: each kernel is then timed alone on the launch stream)
        hipStream_t s_tile = st;
        bool staged = false, side = false;
        if constexpr (VEC == 4) {
            if (ntile_items > 0 && tile_fits(A)) {
                side = !m->prof && fm_side_streams(m);
                if (side) {
                    FM_HIP(m, hipEventRecord(m->ev_fork, st));
                    FM_HIP(m, hipStreamWaitEvent(m->side1, m->ev_fork, 0));
                    s_tile = m->side1;
                }
                ProfScope ps(m, s_tile, FMK_COLS_TILE);
                staged = launch_tile(m, A, s_tile);
                FM_HIP(m, hipGetLastError());
            }
        }
        if (A.nitems > 0) {
            if (A.order != nullptr) {
                int64_t longest = 0;
                for (int x = 0; x < FM_XCDS; ++x)
                    longest = std::max<int64_t>(longest, A.list_off[x + 1] - A.list_off[x]);
                Am.blk_lists = FM_XCDS * ((longest + per - 1) / per);
                if (!staged) {  // the tile items through global memory
                    Am.lin_base = A.list_off[FM_XCDS];
                    Am.lin_count = ntile_items;
                    Am.blk_lin = (ntile_items + per - 1) / per;
                    if (A.xcd_runs) {
                        constexpr int64_t all = FM_XCDS * FM_RUN_BLOCKS;
                        Am.blk_lin = (Am.blk_lin + all - 1) / all * all;
                    }
                }
            } else {
                Am.blk_lists = (A.nitems + per - 1) / per;
            }
        }
        Am.blk_short = (A.nshort + per - 1) / per;
        // empty columns of the full matrix: regulariser only (a stratum's wait for the marks, below); nothing to launch
        // when every column of the matrix is listed as short or long
        const bool empty = need_empty && A.ptr != nullptr && A.D > 0 && A.nshort + A.nlong < A.D;
        const bool beside = empty && !side && A.D * (int64_t)A.K >= FM_EMPTY_BESIDE && !m->prof && fm_side_streams(m);
        if (beside) {
            FM_HIP(m, hipEventRecord(m->ev_fork, st));
            FM_HIP(m, hipStreamWaitEvent(m->side2, m->ev_fork, 0));
        }
        auto launch = [&](const ColArgs& B, hipStream_t q) -> int {
            const int64_t grid = B.blk_lists + B.blk_lin + B.blk_short + (B.epi.on ? B.epi.nsums : 0);
            if (grid > 0x7fffffffLL) return fm_fail(m, FM_ERANGE, "column grid too large");
            if (grid <= 0) return FM_OK;
            ProfScope ps(m, q, FMK_COLS);
            auto go = [&](auto few) {
                constexpr bool F = decltype(few)::value;
                auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(FM_BLOCK), 0, q, B); };
                if (F || B.long_runs) {
                    if (update) run(&k_cols<VEC, L, true, PACKED, F>); else run(&k_cols<VEC, L, false, PACKED, F>);
                } else {
                    if (update) run(&k_cols_part<VEC, L, true, PACKED>); else run(&k_cols_part<VEC, L, false, PACKED>);
                }
            };
            if constexpr (VEC == 4 && L == 8) {
                if (few_wavefronts(B))
                    go(std::true_type());
                else
                    go(std::false_type());
            } else {
                go(std::false_type());
            }
            FM_HIP(m, hipGetLastError());
            return FM_OK;
        };
        if (side && Am.blk_lists > 0 && Am.blk_short > 0) {
            // a matrix tall enough for LDS tiles forks anyway: the short columns then run beside the items from the start
            // (click-style workload, 1e7 rows: 7.40 against 7.55 ms per epoch in one launch)
            ColArgs B = Am;
            B.blk_lists = B.blk_lin = 0;
            B.epi.on = 0;
            FM_HIP(m, hipStreamWaitEvent(m->side2, m->ev_fork, 0));
            FM_TRY(launch(B, m->side2));
            FM_HIP(m, hipEventRecord(m->ev_join2, m->side2));
            B = Am;
            B.blk_short = 0;
            FM_TRY(launch(B, st));
            FM_HIP(m, hipStreamWaitEvent(st, m->ev_join2, 0));
        } else {
            FM_TRY(launch(Am, st));
        }
        if (empty) FM_TRY((launch_empty<VEC>(m, A, update, beside ? m->side2 : st)));
        if (beside) {
            FM_HIP(m, hipEventRecord(m->ev_join2, m->side2));
            FM_HIP(m, hipStreamWaitEvent(st, m->ev_join2, 0));
        }
        if (side) {
            FM_HIP(m, hipEventRecord(m->ev_join1, m->side1));
            FM_HIP(m, hipStreamWaitEvent(st, m->ev_join1, 0));
        }
    }
    // nothing left for single wavefronts when every long column is on the list of the very long ones
    const int64_t by_wave = A.nvlong == A.nlong ? 0 : (A.nlong + FM_WAVES - 1) / FM_WAVES;
    const int64_t g3 = A.nvlong + by_wave + (A.epi.on ? 1 : 0);
    if (g3 > 0) {
        ProfScope ps(m, st, FMK_COLS_FINISH);
        if (update)
            hipLaunchKernelGGL((k_cols_finish<VEC, L, true>), dim3((unsigned)g3), dim3(FM_BLOCK), 0, st, Am);
        else
            hipLaunchKernelGGL((k_cols_finish<VEC, L, false>), dim3((unsigned)g3), dim3(FM_BLOCK), 0, st, Am);
        FM_HIP(m, hipGetLastError());
    }
    // a stratum or batch whose steps are taken at once: every column that had entries has marked itself by now
    if (need_empty && A.ptr == nullptr && A.D > 0) {
        ProfScope ps(m, st, FMK_COLS);
        FM_TRY((launch_empty<VEC>(m, Am, update, st)));
    }
    return FM_OK;
}

template <int VEC, int PACKED>
int launch_cols_v(fm_matrix* m, int lanes, const ColArgs& A, bool update, hipStream_t st)
{
    if constexpr (PACKED == FM_PLANAR) {  // a packed row, K <= 28, takes two to eight lanes
        switch (lanes) {
            case 1: return launch_cols_t<VEC, 1, PACKED>(m, A, update, st);
            case 16: return launch_cols_t<VEC, 16, PACKED>(m, A, update, st);
            case 32: return launch_cols_t<VEC, 32, PACKED>(m, A, update, st);
            case 64: return launch_cols_t<VEC, 64, PACKED>(m, A, update, st);
        }
    }
    switch (lanes) {
        case 2: return launch_cols_t<VEC, 2, PACKED>(m, A, update, st);
        case 4: return launch_cols_t<VEC, 4, PACKED>(m, A, update, st);
        case 8: return launch_cols_t<VEC, 8, PACKED>(m, A, update, st);
    }
    return fm_fail(m, FM_EINVAL, "unsupported lane count %d", lanes);
}

}  // namespace

// lanes per column group: K/VEC latent lanes, plus one lane for the scalars of a packed row
// when the row [G | r] lies inside one 128-byte line
static bool cols_shape(int32_t K, int packed, int* vec, int* lanes)
{
    if (!fm_shape_for_K(K, vec, lanes)) return false;
    if (packed == FM_PACKED_LANE) {
        int need = K / 4 + 1, l = 1;
        while (l < need) l <<= 1;
        *lanes = l;
    }
    return true;
}

int fm_launch_cols(fm_matrix* m, const ColArgs& A, bool update, hipStream_t st)
{
    int vec, lanes;
    if (!cols_shape(A.K, A.packed, &vec, &lanes)) return fm_fail(m, FM_EINVAL, "unsupported K=%d", A.K);
    if (A.packed == FM_PACKED_LANE) return launch_cols_v<4, FM_PACKED_LANE>(m, lanes, A, update, st);
    switch (vec) {
        case 4: return launch_cols_v<4, FM_PLANAR>(m, lanes, A, update, st);
        case 2: return launch_cols_v<2, FM_PLANAR>(m, lanes, A, update, st);
        default: return launch_cols_v<1, FM_PLANAR>(m, lanes, A, update, st);
    }
}

int fm_launch_cols_flush(fm_matrix* m, const ColArgs& A, hipStream_t st)
{
    int vec, lanes;
    if (!fm_shape_for_K(A.K, &vec, &lanes)) return fm_fail(m, FM_EINVAL, "unsupported K=%d", A.K);
    if (A.lazy_last == nullptr || A.D <= 0) return FM_OK;
    switch (vec) {
        case 4: return launch_flush<4>(m, A, st);
        case 2: return launch_flush<2>(m, A, st);
        default: return launch_flush<1>(m, A, st);
    }
}
