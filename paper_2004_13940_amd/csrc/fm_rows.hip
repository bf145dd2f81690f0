// Row-side kernels: the fused forward pass (aggregates, prediction, loss, multiplier)
// and the incremental refresh of the aggregates of a stratified step.
//
// Layout: a wavefront is split into groups of L lanes; one group owns one row, lane
// `sub` of the group owns VEC consecutive latent dimensions [sub*VEC, sub*VEC+VEC).
// A group reads its row's (column, value) pairs (coalesced, each lane the ones it holds), broadcasts each pair inside the
// group and gathers the V row of that column as one contiguous 4*K-byte request.
#include <string.h>

#include "fm_device.h"
#include "fm_internal.h"

namespace {

// FORWARD_HALF: V rows from the half-precision copy, _SMALL: in a small launch; *_BIG: what is gathered is larger than FM_BUF_BYTES (groups of fewer
// than FM_WIDE_GROUP lanes; wider ones use 64-bit addresses throughout)
enum {
    MODE_FORWARD = 0,
    MODE_REFRESH = 1,
    MODE_FORWARD_HALF = 2,
    MODE_REFRESH_BIG = 3,
    MODE_FORWARD_BIG = 4,
    MODE_FORWARD_HALF_BIG = 5,
    MODE_FORWARD_HALF_SMALL = 6
};
constexpr bool is_refresh(int mode) { return mode == MODE_REFRESH || mode == MODE_REFRESH_BIG; }
constexpr bool is_half(int mode)
{
    return mode == MODE_FORWARD_HALF || mode == MODE_FORWARD_HALF_BIG || mode == MODE_FORWARD_HALF_SMALL;
}
constexpr int addr_of(int mode)
{
    return mode == MODE_FORWARD || mode == MODE_FORWARD_HALF || mode == MODE_FORWARD_HALF_SMALL || mode == MODE_REFRESH
               ? FM_ADDR_BUF
               : FM_ADDR_PTR;
}

// Per-entry work of a score: w_j x_ij.
struct OwnScore {
    struct T {
        float w[1];
    };
    FmOwnArray<1> w;
    float a;
    template <int ADDR>
    __device__ __forceinline__ T load(int c) const
    {
        T t;
        w.template get<ADDR>(c, t.w);
        return t;
    }
    __device__ __forceinline__ float use(T t, float x)
    {
        a += t.w[0] * x;
        return x;
    }
    __device__ __forceinline__ void end_round() const {}
};

// Per-entry work of a refresh: the changes of w_j and of |v_j|^2.
struct OwnRefresh {
    struct T {
        float d[2];
    };
    FmOwnArray<2> dwn;
    float a, q;
    template <int ADDR>
    __device__ __forceinline__ T load(int c) const
    {
        T t;
        dwn.template get<ADDR>(c, t.d);
        return t;
    }
    __device__ __forceinline__ float use(T t, float x)
    {
        a += t.d[0] * x;
        q += t.d[1] * (x * x);
        return x;
    }
    __device__ __forceinline__ void end_round() const {}
};

// Sum over the groups of L lanes that share a row of LS lanes, on every lane.
template <int VEC, int L, int LS>
__device__ __forceinline__ void add_parts(float (&acc)[VEC])
{
    if constexpr (L < LS) {
#pragma unroll
        for (int z = 0; z < VEC; ++z) acc[z] += fm_xor_lane<L>(acc[z]);
        add_parts<VEC, 2 * L, LS>(acc);
    }
}

// SP > 1 (forward, up to eight lanes): SP groups of L lanes share a row and add up what each has of it.
template <int VEC, int L, int MODE, int SP = 1>
__global__ __launch_bounds__(FM_BLOCK, L >= FM_WIDE_GROUP && is_refresh(MODE) ? 8 : 1) void k_rows(const RowArgs A)
{
    constexpr int LS = L * SP;       // lanes per row
    constexpr int R = FM_WAVE / LS;  // rows per wavefront
    const int lane = threadIdx.x & (FM_WAVE - 1);
    const int wave = threadIdx.x / FM_WAVE;
    const int sub = lane & (L - 1);
    const int grp = lane / LS;
    const int part = lane / L % SP;
    int64_t blk = blockIdx.x;
    if constexpr (is_refresh(MODE)) {
        if (A.xcd_runs) blk = blk % FM_XCDS * (gridDim.x / FM_XCDS) + blk / FM_XCDS;
    }
    const int64_t slot = blk * (FM_WAVES * R) + wave * R + grp;
    const bool valid = slot < A.N;
    // Every lane loads, of the last row where its own is past the end: without branches the loads of a stage are all on
    // their way before the first is waited for.
    const int64_t at = valid ? slot : A.N - 1;
    const int64_t beg = A.rowptr[at], end = A.rowptr[at + 1];
    int64_t row = at;
    if constexpr (is_refresh(MODE)) {  // listed rows: pointers are indexed by list position
        const int32_t* __restrict__ list = A.rows != nullptr ? A.rows + at : reinterpret_cast<const int32_t*>(A.rowptr);
        const int32_t listed = *list;
        if (A.rows != nullptr) row = listed;
    }
    const int len = valid ? (int)(end - beg) : 0;
    const int K = A.K;
    const int kbase = sub * VEC;
    const bool kact = kbase < K;  // K is a multiple of VEC, so the whole slice is in range
    const int kb = kact ? kbase : 0;
    const uint64_t grow = (uint64_t)(uint32_t)row * (uint32_t)A.gs;  // row < 2^31, strides < 2^31
    const uint64_t srow = (uint64_t)(uint32_t)row * (uint32_t)A.ss;
    const uint64_t arow = (uint64_t)(uint32_t)row * (uint32_t)A.as;

    float acc[VEC];
#pragma unroll
    for (int u = 0; u < VEC; ++u) acc[u] = 0.f;
    float a_acc = 0.f, q_acc = 0.f;
    [[maybe_unused]] bool touched = false;
    [[maybe_unused]] float g_old[VEC] = {};
    [[maybe_unused]] float a_old = 0.f, q_old = 0.f;
    const float y_i = *(A.y != nullptr ? A.y + row : A.w0);  // not used without labels
    if constexpr (!is_refresh(MODE)) {
        if constexpr (L < FM_WIDE_GROUP) {
            OwnScore own{FmOwnArray<1>(A.w, 1), 0.f};
            float unused = 0.f;
            if constexpr (is_half(MODE))
                fm_walk<VEC, L, FM_WALK_SCORE, addr_of(MODE), 16, 8, SP, MODE == MODE_FORWARD_HALF_SMALL>(
                    A.col, A.val, beg, len, A.Vh, K, sub, kb, acc, unused, q_acc, own, part);
            else
                fm_walk<VEC, L, FM_WALK_SCORE, addr_of(MODE), 16, 8, SP>(A.col, A.val, beg, len, A.V, K, sub, kb, acc, unused,
                                                                         q_acc, own, part);
            a_acc = own.a;
            add_parts<VEC, L, LS>(acc);
        } else {
            const float* __restrict__ w = A.w;
            auto own = [&](int c, float x) {
                a_acc += w[c] * x;
                return x;
            };
            if constexpr (is_half(MODE))
                fm_gather_accumulate<VEC, L>(A.col, A.val, beg, beg + len, A.Vh, K, sub, kb, acc, q_acc, own);
            else
                fm_gather_accumulate<VEC, L>(A.col, A.val, beg, beg + len, A.V, K, sub, kb, acc, q_acc, own);
        }
    } else {
        // rows that have no entry in this stratum keep their aggregates untouched
        touched = len > 0;  // uniform inside a group
        fm_load_vec<VEC>(A.G + grow + kb, g_old);
        if (L < FM_WIDE_GROUP && VEC == 4 && A.whole_rows) {  // [r | a | q | pad] of a packed row
            float z[4];
            fm_load_vec<4>(A.G + grow + K, z);
            a_old = z[1];
            q_old = z[2];
        } else {  // (a, q) of a planar row
            float z[2];
            fm_load_vec<2>(A.a + arow, z);
            a_old = z[0];
            q_old = z[1];
        }
        // A row has few entries inside one stratum (1 to 4 where it has any): rounds as short as the group allows, four
        // gathers at a time, so that few registers are in use and many rows in flight; for groups of up to eight lanes a
        // slot without an entry is no request (BUF addressing).  Missing entries used to repeat the last one: three of
        // four requests of a row with one entry (stratified epoch of the click-style workload, 1e7 rows, 64 strata:
        // 39.0 -> 38.5 ms).
        if constexpr (L >= FM_WIDE_GROUP) {
            const float2* __restrict__ dwn = A.dwn;
            fm_walk_wide<VEC, L>(A.col, A.val, beg, beg + len, A.V, K, sub, kb, acc, [&](int c, float x) {
                const float2 d = dwn[c];
                a_acc += d.x * x;
                q_acc += d.y * (x * x);
                return x;
            });
        } else {
            OwnRefresh own{FmOwnArray<2>(reinterpret_cast<const float*>(A.dwn), 2), 0.f, 0.f};
            float unused = 0.f;
            fm_walk<VEC, L, FM_WALK_SUM, addr_of(MODE), L < 4 ? 4 : L, 4>(A.col, A.val, beg, len, A.V, K, sub, kb, acc, unused,
                                                                          unused, own);
            a_acc = own.a;
            q_acc = own.q;
        }
    }
    if (!kact) {  // idle lanes of a group wider than K/VEC worked on a valid but foreign slice
#pragma unroll
        for (int u = 0; u < VEC; ++u) acc[u] = 0.f;
        if constexpr (!is_refresh(MODE)) q_acc = 0.f;
    }

    float l_i = 0.f, r_i = 0.f;
    [[maybe_unused]] float yh_i = 0.f;
    const bool want = A.row_part != nullptr || A.eval_part != nullptr;
    if constexpr (!is_refresh(MODE)) {
        float pair = 0.f;
#pragma unroll
        for (int z = 0; z < VEC; ++z) pair += acc[z] * acc[z];
        const float a_i = fm_group_sum<LS>(a_acc);
        const float q_i = fm_group_sum<LS>(q_acc);
        pair = fm_group_sum<L>(pair);
        const float yh = A.w0[0] + a_i + 0.5f * (pair - q_i);
        if (valid && part == 0) {
            if (sub == 0) {
                if (A.yhat != nullptr) A.yhat[row] = yh;
                if (A.y != nullptr) {
                    yh_i = yh;
                    loss_and_multiplier(A.loss, A.s, yh, y_i, want, l_i, r_i);
                }
            }
            if (A.G != nullptr && kact) fm_store_vec<VEC>(A.G + grow + kbase, acc);
            if (A.whole_rows) {
                // packed aggregate rows: [r | a | q] and the padding behind G go out as float4 too, so
                // that every 128-byte line of the row is written whole
                if constexpr (VEC == 4) {
                    const int tail4 = (int)(A.gs - K) / 4;
                    for (int t = sub; t < tail4; t += L) {
                        float z[4] = {0.f, 0.f, 0.f, 0.f};
                        if (t == 0) {
                            z[0] = r_i;
                            z[1] = a_i;
                            z[2] = q_i;
                        }
                        fm_store_vec<4>(A.G + grow + K + 4 * t, z);
                    }
                }
            } else if (sub == 0) {
                if (A.a != nullptr) A.a[arow] = a_i;
                if (A.q != nullptr) A.q[arow] = q_i;
                if (A.y != nullptr && A.r != nullptr) A.r[srow] = r_i;
            }
        }
    } else {
        const float da = fm_group_sum<L>(a_acc);
        const float dq = fm_group_sum<L>(q_acc);
        float pair = 0.f;
        float g[VEC];
#pragma unroll
        for (int z = 0; z < VEC; ++z) {
            g[z] = g_old[z] + acc[z];
            pair += g[z] * g[z];
        }
        if (!(touched && kact)) pair = 0.f;
        pair = fm_group_sum<L>(pair);
        float a_i = 0.f, q_i = 0.f;
        if (touched && sub == 0) {
            a_i = a_old + da;
            q_i = q_old + dq;
            const float yh = A.w0[0] + a_i + 0.5f * (pair - q_i);
            if (A.yhat != nullptr) A.yhat[row] = yh;
            loss_and_multiplier(A.loss, A.s, yh, y_i, want, l_i, r_i);
        }
        // All stores of a row together, so that its line is written back once.  The kernel is bound by its requests in
        // flight, so r, a, q of a packed row go out (and come in) as one float4 and not one by one: a stratum of the
        // click-style workload (1e7 rows, 64 strata) 311 -> 252 us, of the text-like one (5e4 rows, 32 strata) 8.9 -> 7.2.
        // The rest of the padding stays as the forward pass wrote it: the line was read and is in the L2 (with it 254 and
        // 9.1 us, with non-temporal stores 270 us).
        if (touched && kact) fm_store_vec<VEC>(A.G + grow + kbase, g);
        if (L < FM_WIDE_GROUP && VEC == 4 && A.whole_rows) {
            if (touched && sub == 0) {
                const float z[4] = {r_i, a_i, q_i, 0.f};
                fm_store_vec<4>(A.G + grow + K, z);
            }
        } else if (touched && sub == 0) {
            const float z[2] = {a_i, q_i};
            fm_store_vec<2>(A.a + arow, z);
            A.r[srow] = r_i;
        }
    }

    if constexpr (!is_refresh(MODE)) {
        if (A.aux_rows != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *A.aux_rows = A.whole_rows;
    }
    if (A.row_part != nullptr) {
        // l_i, r_i are non-zero only in lane 0 of a group: fixed-order block sums
        __shared__ float sh[2 * FM_WAVES];
        const float ls = fm_wave_sum(l_i);
        const float rs = fm_wave_sum(r_i);
        if (lane == 0) {
            sh[wave] = ls;
            sh[FM_WAVES + wave] = rs;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            float t0 = 0.f, t1 = 0.f;
#pragma unroll
            for (int wv = 0; wv < FM_WAVES; ++wv) {
                t0 += sh[wv];
                t1 += sh[FM_WAVES + wv];
            }
            A.row_part[2 * (int64_t)blockIdx.x] = t0;
            A.row_part[2 * (int64_t)blockIdx.x + 1] = t1;
        }
    }
    if constexpr (!is_refresh(MODE)) {
        if (A.eval_part != nullptr) {  // sums of losses, squared errors and correct signs of the block's rows
            __shared__ double she[3 * FM_WAVES];
            fm_eval_wave(valid && sub == 0 && part == 0, yh_i, y_i, l_i, lane, she + 3 * wave);
            __syncthreads();
            if (threadIdx.x < 3) {
                double t = 0.0;
#pragma unroll
                for (int wv = 0; wv < FM_WAVES; ++wv) t += she[3 * wv + threadIdx.x];
                A.eval_part[3 * (int64_t)blockIdx.x + threadIdx.x] = t;
            }
        }
    }
}

template <int VEC, int L>
int launch_rows_t(fm_matrix* m, const RowArgs& A, bool refresh, hipStream_t st)
{
    const int split = refresh ? 1 : fm_rows_split(m, A.N, A.K, L);
    const int64_t per = FM_WAVES * (FM_WAVE / (L * split));
    int64_t grid = (A.N + per - 1) / per;
    if (grid <= 0) return FM_OK;
    if (refresh && A.xcd_runs) grid = (grid + FM_XCDS - 1) / FM_XCDS * FM_XCDS;
    if (grid > 0x7fffffffLL) return fm_fail(m, FM_ERANGE, "row grid too large");
    ProfScope ps(m, st, refresh ? FMK_ROWS_REFRESH : FMK_ROWS_FORWARD);
    constexpr bool W = L >= FM_WIDE_GROUP;  // wide groups use 64-bit addresses throughout: one variant
    auto launch = [&](auto mode) {
        constexpr int M = decltype(mode)::value;
        if constexpr (!W && (M == MODE_FORWARD || M == MODE_FORWARD_HALF || M == MODE_FORWARD_HALF_SMALL)) {
            if (split == 2) {
                hipLaunchKernelGGL((k_rows<VEC, L, M, 2>), dim3((unsigned)grid), dim3(FM_BLOCK), 0, st, A);
                return;
            }
            if (split == 4) {
                hipLaunchKernelGGL((k_rows<VEC, L, M, 4>), dim3((unsigned)grid), dim3(FM_BLOCK), 0, st, A);
                return;
            }
        }
        // A forward pass of many rounds of workgroups: three of them to a compute unit (by LDS that nobody uses), so that the
        // entries of their rows stay in its L1 until they are used up (click-style scores, 2.5e6 rows, K=16: 722 -> 702 us;
        // a small launch needs the fourth: text-like epoch of 5e4 rows 59.2 -> 60.5 us).  With and without for fewer lanes: K=8,
        // 2e6 click-style rows 490 and 501 us, 9e5 text-like 332 and 346; K=2 408 and 415; K=4 441 and 441; K=1 409 and 413.
        // Groups of eight lanes hold half as many rows and want every workgroup that fits (K=32, 5.4e5 rows: 193 us with three,
        // 175 without; half-precision V, 1e6 rows: 507 and 379), unless V is far beyond the L1: four of the six for which there
        // are registers then find more of it in the L2 (K=32, 8e5 rows of 50 uniform columns: 8,000 columns, 1 MB, 351 -> 313 us,
        // 25,000 453 -> 424; 2e6 click-style rows 687 -> 675; but 1.5e6 rows of 12 of 1,200 columns 176 -> 189, 8e5 rows of 50 of
        // 80 203 -> 215; and half-precision V, whose rows are half as long, 2e6 click-style rows 664 -> 732).
        const bool many = grid >= 4 * 3 * 256;
        const bool beyond_l1 = m->D * (int64_t)A.K * (int64_t)sizeof(float) > 512 * 1024;
        const size_t lds = L < 8 && !is_refresh(M) && many ? 52 * 1024 : L == 8 && M == MODE_FORWARD && many && beyond_l1 ? 36 * 1024 : 0;
        hipLaunchKernelGGL((k_rows<VEC, L, M>), dim3((unsigned)grid), dim3(FM_BLOCK), lds, st, A);
    };
    if (refresh) {
        if (A.big)
            launch(std::integral_constant<int, W ? MODE_REFRESH : MODE_REFRESH_BIG>());
        else
            launch(std::integral_constant<int, MODE_REFRESH>());
    } else if (A.Vh != nullptr) {
        if constexpr (VEC == 4) {
            // Groups of eight lanes, small launches: each batch of requests whole before it is converted (scores of 3,000 text-like
            // rows, K=32 19.6 -> 15.5 us, 6e4 rows 50.4 -> 47.6).  Large ones are bound by the lines they ask for, and fewer
            // requests in flight find more of them in the caches (click-style rows, K=32: 5e5 184 -> 189 us, 2e6 670 -> 701).
            constexpr int SMALL = L == 8 ? MODE_FORWARD_HALF_SMALL : MODE_FORWARD_HALF;
            if (A.big)
                launch(std::integral_constant<int, W ? MODE_FORWARD_HALF : MODE_FORWARD_HALF_BIG>());
            else if (A.N * L <= FM_SPLIT_LANES)
                launch(std::integral_constant<int, SMALL>());
            else
                launch(std::integral_constant<int, MODE_FORWARD_HALF>());
        } else {
            return fm_fail(m, FM_EINVAL, "half_gather needs K to be a multiple of 4");
        }
    } else if (A.big) {
        launch(std::integral_constant<int, W ? MODE_FORWARD : MODE_FORWARD_BIG>());
    } else {
        launch(std::integral_constant<int, MODE_FORWARD>());
    }
    FM_HIP(m, hipGetLastError());
    return FM_OK;
}

template <int VEC>
int launch_rows_v(fm_matrix* m, int lanes, const RowArgs& A, bool refresh, hipStream_t st)
{
    switch (lanes) {
        case 1: return launch_rows_t<VEC, 1>(m, A, refresh, st);
        case 2: return launch_rows_t<VEC, 2>(m, A, refresh, st);
        case 4: return launch_rows_t<VEC, 4>(m, A, refresh, st);
        case 8: return launch_rows_t<VEC, 8>(m, A, refresh, st);
        case 16: return launch_rows_t<VEC, 16>(m, A, refresh, st);
        case 32: return launch_rows_t<VEC, 32>(m, A, refresh, st);
        case 64: return launch_rows_t<VEC, 64>(m, A, refresh, st);
    }
    return fm_fail(m, FM_EINVAL, "unsupported lane count %d", lanes);
}

}  // namespace

namespace {
__global__ void k_unpack_aux(const FmAux planar, const FmAux rows, const int32_t* __restrict__ aux_rows, int64_t N, int32_t K,
                             float* a, float* G, float* q, float* r)
{
    const FmAux x = *aux_rows != 0 ? rows : planar;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t per = K + 3;
    if (t >= N * per) return;
    const int64_t i = t / per;
    const int c = (int)(t % per);
    if (c < K) {
        if (G != nullptr) G[i * K + c] = x.G[i * x.gs + c];
    } else if (c == K) {
        if (r != nullptr) r[i] = x.r[i * x.ss];
    } else if (c == K + 1) {
        if (a != nullptr) a[i] = x.a[i * x.as];
    } else {
        if (q != nullptr) q[i] = x.q[i * x.as];
    }
}
}  // namespace

namespace {
// Caller-side dense r[N], G[N x K] into the aggregates, one float4 per thread: packed rows [G | r | 0 | 0 | pad], written
// whole, or planar ones, as they come.
__global__ void k_keep_aux(const FmAux x, int packed, int32_t* __restrict__ aux_rows, int64_t N, int32_t K, const float* __restrict__ r,
                           const float* __restrict__ G)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t == 0) *aux_rows = packed;
    const int64_t per = x.gs / 4;  // float4 per row
    if (t >= N * per) return;
    const int64_t i = t / per;
    const int o = (int)(t % per) * 4;
    float z[4] = {0.f, 0.f, 0.f, 0.f};
    if (o < K)
        fm_load_vec<4>(G + i * K + o, z);
    else if (o == K)
        z[0] = r[i];
    fm_store_vec<4>(x.G + i * x.gs + o, z);
    if (!packed && o == 0) x.r[i] = r[i];
}
}  // namespace

namespace {
__global__ void k_to_half(const float4* __restrict__ x, fm_h4* __restrict__ out, int64_t n4)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n4) return;
    const float4 v = x[i];
    fm_h4 h;
    h.x = (_Float16)v.x;
    h.y = (_Float16)v.y;
    h.z = (_Float16)v.z;
    h.w = (_Float16)v.w;
    out[i] = h;
}
}  // namespace

// n a multiple of 4; conversion rounds to nearest even (subnormal halves kept)
int fm_to_half(fm_matrix* m, const float* x, _Float16* out, int64_t n, hipStream_t st)
{
    const int64_t n4 = n / 4;
    if (n4 <= 0) return FM_OK;
    const int64_t grid = (n4 + 255) / 256;
    if (grid > 0x7fffffffLL) return fm_fail(m, FM_ERANGE, "conversion too large");
    hipLaunchKernelGGL(k_to_half, dim3((unsigned)grid), dim3(256), 0, st, reinterpret_cast<const float4*>(x),
                       reinterpret_cast<fm_h4*>(out), n4);
    FM_HIP(m, hipGetLastError());
    return FM_OK;
}

int fm_keep_aux(fm_matrix* m, bool packed, const float* r, const float* G, hipStream_t st)
{
    const FmAux x = fm_aux_layout(m, m->wsK, packed);
    const int64_t total = m->N * (x.gs / 4);
    if (total <= 0) return FM_OK;
    const int64_t grid = (total + 255) / 256;
    if (grid > 0x7fffffffLL) return fm_fail(m, FM_ERANGE, "aggregate copy too large");
    hipLaunchKernelGGL(k_keep_aux, dim3((unsigned)grid), dim3(256), 0, st, x, packed ? 1 : 0, m->aux_rows, m->N, m->wsK, r, G);
    FM_HIP(m, hipGetLastError());
    return FM_OK;
}

// Each pass chooses its layout, and passes may run when a caller's graph is launched, in any order and long after they were
// enqueued: which one the aggregates have is known where they are, in the word that a pass leaves beside them.
int fm_unpack_aux(fm_matrix* m, bool rows_exist, float* a, float* G, float* q, float* r, hipStream_t st)
{
    const int64_t total = m->N * (int64_t)(m->wsK + 3);
    if (total <= 0) return FM_OK;
    const int64_t grid = (total + 255) / 256;
    if (grid > 0x7fffffffLL) return fm_fail(m, FM_ERANGE, "aggregate copy too large");
    hipLaunchKernelGGL(k_unpack_aux, dim3((unsigned)grid), dim3(256), 0, st, fm_aux_layout(m, m->wsK, false),
                       fm_aux_layout(m, m->wsK, rows_exist), (const int32_t*)m->aux_rows, m->N, m->wsK, a, G, q, r);
    FM_HIP(m, hipGetLastError());
    return FM_OK;
}

bool fm_shape_for_K(int32_t K, int* vec, int* lanes)
{
    if (K < 1) return false;
    const int v = (K % 4 == 0) ? 4 : (K % 2 == 0) ? 2 : 1;
    int need = K / v, l = 1;
    while (l < need) l <<= 1;
    if (l > 64) return false;
    if (!(K <= 64 || (K % 4 == 0 && K <= 256))) return false;
    *vec = v;
    *lanes = l;
    return true;
}

// Lane groups that share a row of a forward pass over N rows.  A row is a chain of rounds of 16 entries, which more groups
// shorten; that pays while the launch stays small (up to 2^21 lanes, four times what the chip holds at once)
// and as long as it halves the rounds: evaluation of text-like rows of 60 entries, 2e5 rows, K=16 117 us
// alone, 107 in two groups; 1e5 rows, K=8 64.4 and 55.7; click-style rows of 39 entries (3 rounds or 2), 6e4 rows, K=16 34.7
// and 37.5.
int fm_rows_split(const fm_matrix* m, int64_t N, int32_t K, int lanes)
{
    if (lanes >= FM_WIDE_GROUP || m->N <= 0 || fm_rows_big(m, K) != 0) return 1;
    const int64_t row = m->nnz / m->N;  // entries of a row on average
    int sp = 1;
    auto rounds = [&](int s) { return (row + 16 * s - 1) / (16 * s); };
    while (sp < 4 && N * lanes * 2 * sp <= FM_SPLIT_LANES && 2 * rounds(2 * sp) <= rounds(sp)) sp *= 2;
    return sp;
}

int64_t fm_rows_grid(const fm_matrix* m, int64_t N, int32_t K)
{
    int vec, lanes;
    if (!fm_shape_for_K(K, &vec, &lanes)) return 0;
    const int64_t per = (int64_t)FM_WAVES * (FM_WAVE / (lanes * fm_rows_split(m, N, K, lanes)));
    return (N + per - 1) / per;
}

int64_t fm_rows_max_grid(const fm_matrix* m, int64_t N, int32_t K)
{
    return std::max<int64_t>(fm_rows_grid(m, N, K), FM_SPLIT_LANES / FM_BLOCK + 1);
}

void fm_dense_rows(const RowArgs& A, DenseArgs* E)
{
    memset(E, 0, sizeof(*E));
    E->N = A.N;
    E->D = A.dense_D;
    E->K = A.K;
    E->nchunks = fm_dense_chunks(A.N, A.dense_D, A.K);
    E->X = A.val;
    E->w0 = A.w0;
    E->w = A.w;
    E->V = A.V;
    E->half = A.dense_half;
    E->y = A.y;
    E->yhat = A.yhat;
    E->a = A.a;
    E->G = A.G;
    E->q = A.q;
    E->r = A.r;
    E->gs = A.gs;
    E->ss = A.ss;
    E->as = A.as;
    E->whole_rows = A.whole_rows;
    E->aux_rows = A.aux_rows;
    E->loss = A.loss;
    E->s = A.s;
    E->row_part = A.row_part;
    E->eval_part = A.eval_part;
}

int fm_launch_rows(fm_matrix* m, const RowArgs& A, bool refresh, hipStream_t st)
{
    if (!refresh && A.dense_D > 0) {
        DenseArgs E;
        fm_dense_rows(A, &E);
        return A.N > 0 ? fm_launch_dense(m, E, FM_DENSE_FORWARD, st) : FM_OK;
    }
    int vec, lanes;
    if (!fm_shape_for_K(A.K, &vec, &lanes)) return fm_fail(m, FM_EINVAL, "unsupported K=%d", A.K);
    switch (vec) {
        case 4: return launch_rows_v<4>(m, lanes, A, refresh, st);
        case 2: return launch_rows_v<2>(m, lanes, A, refresh, st);
        default: return launch_rows_v<1>(m, lanes, A, refresh, st);
    }
}
