// Dense matrices: when every row stores all D columns in order, the CSR values are a dense row-major
// N x D matrix X, and the two sparse products of the pass are dense contractions:
//   G = X V                (eq. compute_a_jk for all rows at once),
//   X^T (r . G)            (the sum over the examples in eq. updates_v),
// which run on the fp32 matrix cores (v_mfma_f32_32x32x2_f32: full fp32 products and sums).  The
// column indices are never read.  Everything else (predictions, loss, multipliers, the fixed-order
// fp64 finish of the partial sums, the fused step) is shared with the sparse path.
//
// Operand layout of the 32x32x2 tile C[32 x 32] += A[32 x 2] B[2 x 32] over the 64 lanes of a wavefront:
//   A: lane l holds A[l % 32][l / 32];   B: lane l holds B[l / 32][l % 32];
//   C: register v of lane l holds C[8 * (v / 4) + 4 * (l / 32) + v % 4][l % 32].
#include <float.h>

#include "fm_device.h"
#include "fm_epilogue.h"
#include "fm_internal.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int DT = 32;  // rows, columns and latent dimensions per tile
constexpr int FM_DENSE_MAX = 2 * DT;    // largest D and K of these kernels
constexpr int FM_DENSE_TILES = 8;   // 32-row tiles to a sum in fp32 at most; a wavefront has two such sums
constexpr int FM_DENSE_CUS = 256;   // compute units
// Workgroups that a compute unit holds: by registers, and by LDS where D and K take two tiles.
constexpr int dense_per_cu(int db, int kb) { return db + kb > 3 ? 2 : db + kb > 2 ? 3 : 4; }
__device__ __forceinline__ int c_row(int v, int half) { return 8 * (v / 4) + 4 * half + (v % 4); }

// What a lane of the wavefront wrote to LDS is there for its other lanes: the LDS takes a wavefront's accesses in order,
// the compiler has to keep them so.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// s[v] of lane l: a term of row c_row(v, l / 32).  Returns the sum over the 32 lanes of a half for row
// c_row(l % 32 / 2, l / 32): every exchange halves the registers a lane answers for.
__device__ __forceinline__ float row_sums(float (&s)[16], int lo)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const bool up = lo & 16;
        const float keep = up ? s[i + 8] : s[i], send = up ? s[i] : s[i + 8];
        s[i] = keep + fm_xor_lane<16>(send);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool up = lo & 8;
        const float keep = up ? s[i + 4] : s[i], send = up ? s[i] : s[i + 4];
        s[i] = keep + fm_xor_lane<8>(send);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const bool up = lo & 4;
        const float keep = up ? s[i + 2] : s[i], send = up ? s[i] : s[i + 2];
        s[i] = keep + fm_xor_lane<4>(send);
    }
    const bool up = lo & 2;
    const float keep = up ? s[1] : s[0], send = up ? s[0] : s[1];
    const float t = keep + fm_xor_lane<2>(send);
    return t + fm_xor_lane<1>(t);
}

// One pass over the rows of X.  DB, KB: tiles that D and K take (what is missing to a whole tile is zero).
//   FM_DENSE_FORWARD   aggregates, prediction, loss and multiplier of every row
//   FM_DENSE_GRADIENT  per workgroup and column the partial sums acc = sum_i x_ij r_i G_ik, gw = sum_i x_ij r_i,
//                      s2 = sum_i x_ij^2 r_i (eqs. updates_w, updates_v), as the rows [acc | gw | s2 | pad] of the
//                      items that the workgroup has for the column, which the finish kernel adds
//                      in fp64 in item order
//   both               an epoch: X is read once, and the tile of G goes from one product into the other in registers
// A wavefront takes up to 2 * FM_DENSE_TILES tiles of 32 consecutive rows, a workgroup four times as many.  Sums in fp32 end
// with half of a wavefront's tiles, 256 rows at most; from there on, across wavefronts and workgroups, they are fp64.  A tile
// of X is staged in LDS with an odd row stride, read by columns for the first product (A operand: 32 rows, two columns a step) and
// by rows for the second (A operand: 32 columns, two rows a step).  The rows of a step of the second product are paired
// as the result registers of the first hold them (rows c_row(v, 0) and c_row(v, 1)), so that register v, times r, is its
// B operand as it stands.  Bound: 1e6 rows, D = 64, K = 32 are 392 MB of X, G, y and r (71 us at the rate of a copy) and
// 52 us of matrix instructions (47 % of the time by their counter), with vector instructions for another quarter of the issue
// slots; the epoch takes 120 us, 6 of them the finish, where a forward and a column kernel that each read X took 204.  D = 45,
// K = 8: 118 us, 500 through the sparse kernels.  X by float4 although they meet banks of the LDS four to one on the way in:
// when the kernel was new, 137 us, float by float 149.  The operands from V are read from LDS: in registers they cost the
// third wavefront of a SIMD.
// LDS of a wavefront: its tile of X, then r, a, q of the tile's rows and as many zeros.
template <int DB>
struct DenseLds {
    static constexpr int S = DB * DT + 1;  // odd row stride: columns of the tile spread over the banks
    static constexpr int R = DT * S, A = R + DT, Q = A + DT, Z = Q + DT, FLOATS = Z + DT;
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t fm_rsrc(const float* p, int64_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, (int)bytes, 0x20000);
}

// Byte offsets from the start of a tile of G (gs floats to a row) of value k of the rows that a lane's result registers hold.
// All of it is in the offset that is compared with the range of the descriptor, so that a row past the end is out of range by
// its own number (the scalar offset of a buffer access is not part of what the compiler promises to check).
struct RowOffsets {
    uint32_t base, row;  // a lane that takes no part: FM_BUF_NONE throughout, a sum past it could wrap
    __device__ __forceinline__ RowOffsets(bool takes_part, int half, int k, int gs)
        : base(takes_part ? (uint32_t)(4 * half * gs + k) * 4u : FM_BUF_NONE), row(takes_part ? (uint32_t)gs * 4u : 0u)
    {
    }
    __device__ __forceinline__ int operator()(int v) const { return (int)(base + __umul24((uint32_t)c_row(v, 0), row)); }
};

template <int DB, int KB, int WHAT>
__global__ __launch_bounds__(FM_BLOCK, dense_per_cu(DB, KB)) void k_dense(const DenseArgs A)
{
    constexpr bool FORWARD = WHAT & FM_DENSE_FORWARD, GRADIENT = WHAT & FM_DENSE_GRADIENT;
    constexpr int DP = DB * DT, KP = KB * DT;
    using Lds = DenseLds<DB>;
    constexpr int S = Lds::S;
    extern __shared__ float lds[];
    __shared__ double sh[FM_WAVES * 4];
    const int64_t b = blockIdx.x;
    if (b >= A.nchunks) {  // the workgroups behind the chunks: sums that depend on nothing here
        if (A.epi.on)
            fm_epi_partial<FM_BLOCK>(A.epi, (int)(b - A.nchunks), sh);
        else
            fm_reg_pair<FM_BLOCK>(A.w, A.D, A.V, A.D * (int64_t)A.K, A.regs, sh);
        return;
    }
    const int D = (int)A.D, K = A.K, gs = (int)A.gs;
    const int lane = threadIdx.x & (FM_WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / FM_WAVE);  // uniform, and so is all that follows from it
    const int half = lane / 32, lo = lane % 32;
    const int64_t tiles = (A.N + DT - 1) / DT, parts = A.nchunks * FM_WAVES, part = b * FM_WAVES + wave;
    const int64_t t0 = part * tiles / parts, t1 = (part + 1) * tiles / parts;
    // A tile's rows are contiguous in memory.  Whole float4 up to its last value: the entries are padded for the rest of the
    // last one.  Loaded a tile ahead.
    constexpr int NC = DT * DP / 4 / FM_WAVE;
    float x[NC][4];
    float row_in = 0.f;                     // label, or multiplier, of row lo of the tile
    [[maybe_unused]] float g_in[KB][16];    // gradient alone: its tile of G
    const float* __restrict__ row_src = FORWARD ? A.y : A.r;
    const int64_t row_stride = FORWARD ? 1 : A.ss;
    auto load_tile = [&](int64_t t, int ln) {
        const int64_t left = (A.N - t * DT) * D;
        const __amdgpu_buffer_rsrc_t xs = t < t1 ? fm_rsrc(A.X + t * DT * D, ((left < DT * D ? left : DT * D) + 3) / 4 * 16) : fm_rsrc(A.X, 0);
#pragma unroll
        for (int i = 0; i < NC; ++i) fm_buf_load<4, false>(xs, (uint32_t)(ln + i * FM_WAVE) * 16u, x[i]);
        const int64_t row = t * DT + ln % DT;
        if (row_src != nullptr) row_in = row < A.N ? row_src[row * row_stride] : 0.f;
        if constexpr (!FORWARD) {
            const int64_t rest = (A.N - t * DT) * A.gs;
            const __amdgpu_buffer_rsrc_t gr =
                t < t1 ? fm_rsrc(A.G + t * DT * A.gs, (rest < DT * A.gs ? rest : DT * A.gs) * 4) : fm_rsrc(A.G, 0);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                const int k = kb * DT + ln % DT;
                const RowOffsets at(k < A.K, ln / DT, k, (int)A.gs);
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    g_in[kb][v] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(gr, at(v), 0, 0));
            }
        }
    };
    load_tile(t0, lane);
    float2* wn = reinterpret_cast<float2*>(lds);  // [DP] (w_j, |v_j|^2)
    float* vl = lds + 2 * DP;                     // [DP x KP] V, padded with zeros
    float* area = lds + (FORWARD ? 2 * DP + DP * KP : 0);
    float* tile = area + wave * Lds::FLOATS;
    if constexpr (FORWARD) {
        for (int e = threadIdx.x; e < DP * KP; e += FM_BLOCK) {
            const int j = e / KP, k = e % KP;
            // half_gather: rounded here, no copy of V (evaluation of 1e6 x 64, K = 32: 387 us by the sparse kernel, 83 by this)
            const float v = j < D && k < K ? A.V[j * K + k] : 0.f;
            vl[e] = A.half ? (float)(_Float16)v : v;
        }
        __syncthreads();
        static_assert(FM_BLOCK / DP >= 4, "four threads to a column");
        const int j = threadIdx.x / 4, p = threadIdx.x % 4;
        float n2 = 0.f;
        if (j < DP)
            for (int k = p; k < KP; k += 4) n2 += vl[j * KP + k] * vl[j * KP + k];
        n2 = fm_group_sum<4>(n2);
        if (p == 0 && j < DP) wn[j] = make_float2(j < D ? A.w[j] : 0.f, n2);
        __syncthreads();
    }
    for (int j = D + half; j < DP; j += 2) tile[lo * S + j] = 0.f;  // the columns past D stay zero
    if (half == 0) tile[Lds::Z + lo] = 0.f;
    // where this lane finds what it stores behind G in a packed row [G | r | a | q | pad]
    [[maybe_unused]] const float* behind = tile + (lo == K ? Lds::R : lo == K + 1 ? Lds::A : lo == K + 2 ? Lds::Q : Lds::Z);
    // Sums of the tiles from t_half on, and of those before: neither stands for more than FM_DENSE_TILES tiles, and they are
    // not added in fp32 (`first` is zero when it takes the sum).
    const int t_half = t0 + (t1 - t0 + 1) / 2;
    [[maybe_unused]] f32x16 acc[DB][KB], first[DB][KB];
    [[maybe_unused]] float gw[DB], s2[DB], first_gw[DB], first_s2[DB];
    auto next_sum = [&](bool clear) {
#pragma unroll
        for (int jb = 0; jb < DB; ++jb) {
            first_gw[jb] = clear ? 0.f : first_gw[jb] + gw[jb];
            first_s2[jb] = clear ? 0.f : first_s2[jb] + s2[jb];
            gw[jb] = s2[jb] = 0.f;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    first[jb][kb][v] = clear ? 0.f : first[jb][kb][v] + acc[jb][kb][v];
                    acc[jb][kb][v] = 0.f;
                }
        }
    };
    if constexpr (GRADIENT) next_sum(true);
    [[maybe_unused]] double sum_lr = 0.0, sum_es = 0.0;  // lower half: loss, squared error; upper: r, correct signs
    const float w0 = FORWARD ? A.w0[0] : 0.f;
    const bool want = A.row_part != nullptr || (!GRADIENT && A.eval_part != nullptr);
    const uint32_t magic = ((1u << 20) + (uint32_t)D - 1) / (uint32_t)D;  // e / D = e magic >> 20 for e < 2^12, D <= 64
#pragma unroll 1
    for (int64_t tid = t0; tid < t1; ++tid) {
        if (GRADIENT && tid == t_half) next_sum(false);
        const int64_t row0 = tid * DT;
        const int nrows = (int)((A.N - row0) < DT ? (A.N - row0) : DT);
        // The lane's number as a value of this turn of the loop: what is derived from it (addresses in LDS, w and |v|^2 read
        // from there) is formed anew and not kept in a hundred registers for the next turn.
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int half_t = ln / 32;
        wave_sync();  // the tile before has been read
        if (nrows < DT) {
#pragma unroll
            for (int i = 0; i < NC; ++i)
#pragma unroll
                for (int z = 0; z < 4; ++z)
                    if ((ln + i * FM_WAVE) * 4 + z >= nrows * D) x[i][z] = 0.f;
        }
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const uint32_t e = (uint32_t)(ln + i * FM_WAVE) * 4;
            if (D == DP) {
                float* d = tile + e / DP * S + e % DP;
#pragma unroll
                for (int z = 0; z < 4; ++z) d[z] = x[i][z];
            } else {
#pragma unroll
                for (int z = 0; z < 4; ++z) {
                    const uint32_t row = ((e + z) * magic) >> 20;
                    if (e < (uint32_t)(DT * D)) tile[e + z + row * (uint32_t)(S - D)] = x[i][z];
                }
            }
            __builtin_amdgcn_sched_barrier(0);  // few addresses at a time: registers
        }
        const float r_in = row_in;
        [[maybe_unused]] float g_now[KB][16];
        if constexpr (!FORWARD) {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int v = 0; v < 16; ++v) g_now[kb][v] = g_in[kb][v];
        }
        load_tile(tid + 1, ln);
        f32x16 g[KB];
        if constexpr (FORWARD) {
            const __amdgpu_buffer_rsrc_t rows =
                fm_rsrc(A.G != nullptr ? A.G + row0 * gs : A.X, A.G != nullptr ? (int64_t)nrows * gs * 4 : 0);
            const int64_t mine = row0 + (lo < nrows ? lo : 0);
            const float y_i = r_in;
            wave_sync();
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int v = 0; v < 16; ++v) g[kb][v] = 0.f;
            float a_i = 0.f, q_i = 0.f;  // this lane: row lo, columns of parity `half`
#pragma unroll
            for (int t = 0; t < DP / 2; ++t) {
                const float xt = tile[lo * S + 2 * t + half];
                const float2 c = wn[2 * t + half_t];
                const float* v = vl + (2 * t + half_t) * KP + lo;  // B operand: V[2t + half][kb * 32 + lo]
                a_i += xt * c.x;
                q_i += (xt * xt) * c.y;
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) g[kb] = __builtin_amdgcn_mfma_f32_32x32x2f32(xt, v[kb * DT], g[kb], 0, 0, 0);
                if (t % 8 == 7) {  // what was read so far is used up here, or it would be kept for the end of the loop
                    asm volatile("" : "+v"(a_i), "+v"(q_i));
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            float s[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                s[v] = 0.f;
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) s[v] += g[kb][v] * g[kb][v];
            }
            const float pair = row_sums(s, lo);
            if ((lo & 1) == 0) tile[Lds::A + c_row(lo / 2, half)] = pair;
            a_i += fm_xor_lane<32>(a_i);
            q_i += fm_xor_lane<32>(q_i);
            wave_sync();
            const float yh = w0 + a_i + 0.5f * (tile[Lds::A + lo] - q_i);
            wave_sync();
            float l_i = 0.f, r_i = 0.f;
            if (A.y != nullptr) loss_and_multiplier(A.loss, A.s, yh, y_i, want, l_i, r_i);
            if (lo >= nrows) l_i = r_i = 0.f;
            sum_lr += (double)(half == 0 ? l_i : r_i);
            if (!GRADIENT && A.eval_part != nullptr && lo < nrows) {
                const double d = (double)yh - (double)y_i;
                sum_es += half == 0 ? d * d : (yh >= 0.f ? 1.f : -1.f) == y_i ? 1.0 : 0.0;
            }
            if (half == 0) {
                tile[Lds::R + lo] = r_i;
                tile[Lds::A + lo] = a_i;
                tile[Lds::Q + lo] = q_i;
                if (lo < nrows) {
                    if (!GRADIENT && A.yhat != nullptr) A.yhat[mine] = yh;
                    if (!A.whole_rows) {
                        if (!GRADIENT && A.a != nullptr) A.a[mine * A.as] = a_i;
                        if (!GRADIENT && A.q != nullptr) A.q[mine * A.as] = q_i;
                        if (A.y != nullptr && A.r != nullptr) A.r[mine * A.ss] = r_i;
                    }
                }
            }
            wave_sync();
            // rows past the end are out of the descriptor's range: not stored
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                const int k = kb * DT + ln % DT;
                const RowOffsets at(k < (A.whole_rows ? gs : K), half_t, k, gs);
                if (A.whole_rows) {  // packed aggregate rows go out whole
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const float z = behind[c_row(v, half)];
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(k < K ? g[kb][v] : z), rows, at(v), 0, 0);
                    }
                } else {
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(g[kb][v]), rows, at(v), 0, 0);
                }
            }
        } else {
            if (half == 0) tile[Lds::R + lo] = r_in;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int v = 0; v < 16; ++v) g[kb][v] = g_now[kb][v];
            wave_sync();
        }
        if constexpr (GRADIENT) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float r = tile[Lds::R + c_row(v, half)];
                float gr[KB];
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) gr[kb] = g[kb][v] * r;
#pragma unroll
                for (int jb = 0; jb < DB; ++jb) {
                    const float xt = tile[c_row(v, half) * S + jb * DT + lo];
                    const float xr = xt * r;
                    gw[jb] += xr;
                    s2[jb] += xt * xr;
#pragma unroll
                    for (int kb = 0; kb < KB; ++kb)
                        acc[jb][kb] = __builtin_amdgcn_mfma_f32_32x32x2f32(xt, gr[kb], acc[jb][kb], 0, 0, 0);
                }
                if (v % 4 == 3) {
#pragma unroll
                    for (int jb = 0; jb < DB; ++jb) asm volatile("" : "+v"(gw[jb]), "+v"(s2[jb]));
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }  // tiles of this wavefront
    int thread = threadIdx.x;  // formed anew, not kept over the loop: registers
    asm volatile("" : "+v"(thread));
    const int half_e = thread % FM_WAVE / 32, lo_e = thread % 32;
    if constexpr (GRADIENT) {
        // The wavefronts are added in fp64 in one block of LDS, each at another quarter of the rows c_row(v, .) at a time (one after
        // the other, the pass over 262,000 x 64, K=64 took 6 us longer); the order of the terms is fixed.  From there they go out
        // as whole rows of the partial sums, see fm_dense_parts.
        constexpr int SP = KP + 2;
        double* sum = reinterpret_cast<double*>(area);
        static_assert(DP * SP * sizeof(double) <= FM_WAVES * Lds::FLOATS * sizeof(float), "the sums fit where the tiles were");
        static_assert((2 * DP + DP * KP) % 2 == 0, "aligned doubles");
        static_assert(FM_WAVES == 4, "a quarter to a wavefront");
#pragma unroll 1
        for (int step = 0; step < FM_WAVES; ++step) {
            __syncthreads();
            auto add = [&](double* p, double x) { *p = step == 0 ? x : *p + x; };
            const int mine = (wave + step) % FM_WAVES;
#pragma unroll
            for (int part = 0; part < FM_WAVES; ++part) {
                if (part != mine) continue;
#pragma unroll
                for (int jb = 0; jb < DB; ++jb) {
#pragma unroll
                    for (int v = 4 * part; v < 4 * part + 4; ++v)
#pragma unroll
                        for (int kb = 0; kb < KB; ++kb)
                            add(sum + (jb * DT + c_row(v, half_e)) * SP + kb * DT + lo_e,
                                (double)first[jb][kb][v] + (double)acc[jb][kb][v]);
                    if (part != jb) continue;
                    const double gd = (double)first_gw[jb] + (double)gw[jb], sd = (double)first_s2[jb] + (double)s2[jb];
                    const double gt = gd + fm_xor_lane<32>(gd), st = sd + fm_xor_lane<32>(sd);
                    if (half_e == 0) {
                        add(sum + (jb * DT + lo_e) * SP + KP, gt);
                        add(sum + (jb * DT + lo_e) * SP + KP + 1, st);
                    }
                }
            }
        }
        __syncthreads();
        const int ps4 = (int)A.ps / 4;
        for (int e = threadIdx.x; e < D * ps4; e += FM_BLOCK) {
            const int j = e / ps4, o = (e - j * ps4) * 4;
            float z[4], left[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int k = o + i;
                const double t = k < K ? sum[j * SP + k] : k < K + 2 ? sum[j * SP + KP + k - K] : 0.0;
                z[i] = (float)t;
                // nothing is left of a sum that is no finite float: infinity minus itself would make it NaN
                left[i] = fabsf(z[i]) <= FLT_MAX ? (float)(t - (double)z[i]) : 0.f;
            }
            float* out = A.part + ((int64_t)j * A.nchunks + b) * A.nparts * A.ps + o;
            fm_store_vec<4>(out, z);
            if (A.nparts == 2) fm_store_vec<4>(out + A.ps, left);
        }
    }
    if constexpr (FORWARD) {
        if (b == 0 && threadIdx.x == 0 && A.aux_rows != nullptr) *A.aux_rows = A.whole_rows;
        if (want) {
            sum_lr = fm_group_sum<32>(sum_lr);
            if constexpr (!GRADIENT) sum_es = fm_group_sum<32>(sum_es);
            if (lo_e == 0) {
                sh[wave * 4 + half_e] = sum_lr;
                if constexpr (!GRADIENT) sh[wave * 4 + 2 + half_e] = sum_es;
            }
            __syncthreads();
            if (threadIdx.x < (GRADIENT ? 2 : 4)) {
                const int c = threadIdx.x;
                double t = 0.0;
#pragma unroll
                for (int w = 0; w < FM_WAVES; ++w) t += sh[w * 4 + c];
                if (A.row_part != nullptr && c < 2) A.row_part[2 * b + c] = (float)t;
                if (!GRADIENT && A.eval_part != nullptr && c != 1) A.eval_part[3 * b + (c == 0 ? 0 : c - 1)] = t;
            }
        }
    }
}

template <int DB, int KB, int WHAT>
int launch_dense_t(fm_matrix* m, const DenseArgs& A, hipStream_t st)
{
    constexpr size_t LDS = ((WHAT & FM_DENSE_FORWARD ? (2 + KB * DT) * DB * DT : 0) + FM_WAVES * DenseLds<DB>::FLOATS) * sizeof(float);
    static_assert(LDS <= 64 * 1024, "no opt-in to more LDS needed");
    const int64_t grid = A.nchunks + (A.epi.on ? A.epi.nsums : A.regs != nullptr ? 1 : 0);
    if (grid > 0x7fffffffLL) return fm_fail(m, FM_ERANGE, "chunk grid too large");
    ProfScope ps(m, st, WHAT & FM_DENSE_GRADIENT ? FMK_COLS_LONG : FMK_ROWS_FORWARD);
    hipLaunchKernelGGL((k_dense<DB, KB, WHAT>), dim3((unsigned)grid), dim3(FM_BLOCK), LDS, st, A);
    FM_HIP(m, hipGetLastError());
    return FM_OK;
}

template <int WHAT>
int launch_dense(fm_matrix* m, const DenseArgs& A, hipStream_t st)
{
    const bool d2 = A.D > DT, k2 = A.K > DT;
    if (d2 && k2) return launch_dense_t<2, 2, WHAT>(m, A, st);
    if (d2) return launch_dense_t<2, 1, WHAT>(m, A, st);
    if (k2) return launch_dense_t<1, 2, WHAT>(m, A, st);
    return launch_dense_t<1, 1, WHAT>(m, A, st);
}

}  // namespace

// Up to two tiles each way: the accumulators stay in registers.
bool fm_dense_fits(const fm_matrix* m, int32_t K) { return m->is_dense && m->D <= FM_DENSE_MAX && K <= FM_DENSE_MAX; }

// A launch of few rows spends its time in one chain, from V or G through LDS and the products to the sums, the longer the more
// tiles D and K take.  The sparse kernels spread such a launch over more wavefronts.  Dense / sparse, us:
//   gradient  60 columns, K=64  1,000 rows 16.7 / 11.0  4,000 17.1 / 14.8  8,000 21.3 / 16.9  16,000 21.2 / 23.5
//             64 columns, K=32               12.4 / 10.9        12.3 / 12.2        15.3 / 13.2         15.5 / 18.2
//             22 columns, K=8                14.0 / 14.6        12.1 / 13.7        14.0 / 12.4         12.7 / 14.4
//   evaluate  60 columns, K=64               24.6 / 22.1        24.6 / 22.5        24.8 / 23.7         25.0 / 28.2
//             20 columns, K=64               21.4 / 19.0        21.6 / 19.4        21.7 / 20.3         21.9 / 23.2
//             64 columns, K=32               21.3 / 18.3        21.3 / 19.7        21.6 / 23.3         21.7 / 26.8
//   epoch     60 columns, K=64               25.3 / 22.7  2,000 25.0 / 25.5  4,000 25.9 / 27.3         30.4 / 38.4
//             64 columns, K=32               17.6 / 17.4        18.0 / 17.3        18.0 / 18.7         21.2 / 29.4
// Half-precision factors are always the dense kernels': they need no copy of V, which is a launch of its own and memory.
bool fm_dense_takes(const fm_matrix* m, const fm_params* p, int64_t rows, int what)
{
    const int32_t K = p->K;
    if (m->opt.dense_rows == 0 || rows < 1 || !fm_dense_fits(m, K)) return false;
    if (m->opt.dense_rows == 1 || p->half_gather) return true;
    const bool both = m->D > DT && K > DT, either = m->D > DT || K > DT;
    if (what == FM_DENSE_GRADIENT) return !either || rows > 8192;
    if (what == FM_DENSE_FORWARD) return !either || rows > (K > DT ? 8192 : 4096);
    return !both || rows > 2048;
}

// Workgroups of a pass over N rows: one tile to a wavefront while the chip is not full, then as many as it holds at once,
// in as few rounds as leave no wavefront more than 16 tiles (1e6 x 64, K=32: 977 workgroups of 8 tiles a wavefront took 129
// us, the last 209 of them alone).
int64_t fm_dense_chunks(int64_t N, int64_t D, int32_t K)
{
    const int64_t tiles = (N + DT - 1) / DT;
    const int64_t slots = FM_DENSE_CUS * dense_per_cu(D > DT ? 2 : 1, K > DT ? 2 : 1);
    if (tiles <= FM_WAVES * slots) return (tiles + FM_WAVES - 1) / FM_WAVES;
    const int64_t most = FM_WAVES * slots * 2 * FM_DENSE_TILES;
    return slots * ((tiles + most - 1) / most);
}

// Items that a workgroup leaves for a column: the sum rounded to fp32 and, second, what rounding left.  Rounding once more
// shows where the sums in fp32 are short (one tile to a wavefront) or a workgroup stands for few of them (D and K of two
// tiles each): 262,144 x 64, K=64, sums of terms of one sign, error relative to the sum of their magnitudes 1.7e-9 with the
// second item, as with an fp32 sum to every 64 rows that are all added in fp64.  Elsewhere one item is no worse than that
// and costs half the memory (gradient of 1e6 x 32, K=32 52.1 us, with two items 56.6).
int fm_dense_parts(int64_t N, int64_t D, int32_t K)
{
    const int64_t slots = FM_DENSE_CUS * dense_per_cu(D > DT ? 2 : 1, K > DT ? 2 : 1);
    return (D > DT && K > DT) || (N + DT - 1) / DT <= FM_WAVES * slots ? 2 : 1;
}

int fm_launch_dense(fm_matrix* m, const DenseArgs& A, int what, hipStream_t st)
{
    if (A.D < 1 || A.D > FM_DENSE_MAX || A.K < 1 || A.K > FM_DENSE_MAX || A.N < 1 || A.nchunks < 1 || A.X == nullptr)
        return fm_fail(m, FM_EINVAL, "bad arguments of the dense pass");
    const bool outputs = A.yhat != nullptr || A.eval_part != nullptr || (!A.whole_rows && (A.a != nullptr || A.q != nullptr));
    if (what == (FM_DENSE_FORWARD | FM_DENSE_GRADIENT) && outputs) return fm_fail(m, FM_EINVAL, "an epoch leaves G and r only");
    switch (what) {
        case FM_DENSE_FORWARD: return launch_dense<FM_DENSE_FORWARD>(m, A, st);
        case FM_DENSE_GRADIENT: return launch_dense<FM_DENSE_GRADIENT>(m, A, st);
        case FM_DENSE_FORWARD | FM_DENSE_GRADIENT: return launch_dense<FM_DENSE_FORWARD | FM_DENSE_GRADIENT>(m, A, st);
    }
    return fm_fail(m, FM_EINVAL, "unknown dense pass %d", what);
}
