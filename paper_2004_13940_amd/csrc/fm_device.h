// Device-side helpers shared by the row and column kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fm_internal.h"

#include <type_traits>

template <int VEC>
__device__ __forceinline__ void fm_load_vec(const float* __restrict__ p, float (&v)[VEC])
{
    if constexpr (VEC == 4) {
        const float4 t = *reinterpret_cast<const float4*>(p);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else if constexpr (VEC == 2) {
        const float2 t = *reinterpret_cast<const float2*>(p);
        v[0] = t.x; v[1] = t.y;
    } else {
        v[0] = *p;
    }
}

// The same from a row stored as IEEE half precision (the internal copy of V that a pass with
// fm_params.half_gather reads): half the bytes per gathered row, widened to fp32 on arrival.
typedef _Float16 fm_h4 __attribute__((ext_vector_type(4)));
typedef _Float16 fm_h2 __attribute__((ext_vector_type(2)));
template <int VEC>
__device__ __forceinline__ void fm_load_vec(const _Float16* __restrict__ p, float (&v)[VEC])
{
    if constexpr (VEC == 4) {
        const fm_h4 t = *reinterpret_cast<const fm_h4*>(p);
        v[0] = (float)t.x; v[1] = (float)t.y; v[2] = (float)t.z; v[3] = (float)t.w;
    } else if constexpr (VEC == 2) {
        const fm_h2 t = *reinterpret_cast<const fm_h2*>(p);
        v[0] = (float)t.x; v[1] = (float)t.y;
    } else {
        v[0] = (float)*p;
    }
}

template <int VEC>
__device__ __forceinline__ void fm_store_vec(float* __restrict__ p, const float (&v)[VEC])
{
    if constexpr (VEC == 4) {
        *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
    } else if constexpr (VEC == 2) {
        *reinterpret_cast<float2*>(p) = make_float2(v[0], v[1]);
    } else {
        *p = v[0];
    }
}

// Value held by the lane whose number differs in bit X (a power of two below 64).  Inside 16 lanes by DPP, which has
// neither the address arithmetic of ds_bpermute nor a wait on the LDS crossbar behind it.
template <int X>
__device__ __forceinline__ int fm_xor_lane(int v)
{
    if constexpr (X == 1) {
        return __builtin_amdgcn_mov_dpp(v, 0xB1 /* quad_perm [1,0,3,2] */, 0xf, 0xf, true);
    } else if constexpr (X == 2) {
        return __builtin_amdgcn_mov_dpp(v, 0x4E /* quad_perm [2,3,0,1] */, 0xf, 0xf, true);
    } else if constexpr (X == 4) {
        // quads 0 and 2 of a row of 16 take the quad after them, then quads 1 and 3 the one before them
        const int x = __builtin_amdgcn_update_dpp(v, v, 0x104 /* row_shl:4 */, 0xf, 0x5, false);
        return __builtin_amdgcn_update_dpp(x, v, 0x114 /* row_shr:4 */, 0xf, 0xa, false);
    } else if constexpr (X == 8) {
        return __builtin_amdgcn_mov_dpp(v, 0x128 /* row_ror:8 */, 0xf, 0xf, true);
    } else if constexpr (X == 16) {
        return __builtin_amdgcn_ds_swizzle(v, (16 << 10) | 0x1f);
    } else {
        return __shfl_xor(v, X, 64);
    }
}
template <int X>
__device__ __forceinline__ float fm_xor_lane(float v)
{
    return __int_as_float(fm_xor_lane<X>(__float_as_int(v)));
}
template <int X>
__device__ __forceinline__ double fm_xor_lane(double v)
{
    return __hiloint2double(fm_xor_lane<X>(__double2hiint(v)), fm_xor_lane<X>(__double2loint(v)));
}

// Sum over the L lanes of a group (L a power of two, groups aligned to L lanes);
// every lane of the group receives the total.  Fixed butterfly order.
template <int L, typename T>
__device__ __forceinline__ T fm_group_sum(T v)
{
    if constexpr (L > 1) {
        v += fm_xor_lane<L / 2>(v);
        return fm_group_sum<L / 2>(v);
    }
    return v;
}

// Sum over all 64 lanes of the wave, fixed butterfly order.
template <typename T>
__device__ __forceinline__ T fm_wave_sum(T v)
{
    return fm_group_sum<FM_WAVE>(v);
}

// Largest of the values of a wavefront's groups (the L lanes of a group hold the same one), as a wave-uniform number (a
// scalar register: branches on it do not diverge).
template <int L>
__device__ __forceinline__ int fm_wave_max(int v)
{
    auto take = [&](int t) { v = t > v ? t : v; };
    if constexpr (L <= 1) take(fm_xor_lane<1>(v));
    if constexpr (L <= 2) take(fm_xor_lane<2>(v));
    if constexpr (L <= 4) take(__builtin_amdgcn_mov_dpp(v, 0x141 /* row_half_mirror */, 0xf, 0xf, true));
    if constexpr (L <= 8) take(__builtin_amdgcn_mov_dpp(v, 0x140 /* row_mirror */, 0xf, 0xf, true));
    const int a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
    const int c = __builtin_amdgcn_readlane(v, 32), d = __builtin_amdgcn_readlane(v, 48);
    const int ab = a > b ? a : b, cd = c > d ? c : d;
    return ab > cd ? ab : cd;
}

// Multiplier of one example, and its loss where `want` (uniform) says that somebody reads it: the logarithm is most of
// the instructions (cases after eq. updates_v; the loss constants make the printed multiplier the exact derivative).
// expf only ever sees a non-positive argument.
__device__ __forceinline__ void loss_and_multiplier(int32_t loss, float s, float yh, float y, bool want, float& l, float& r)
{
    l = 0.f;
    if (loss == FM_LOSS_SQUARED) {
        const float d = yh - y;
        if (want) l = 0.5f * d * d;
        r = s * d;
    } else {
        const float mg = y * yh;
        const float e = expf(mg > 0.f ? -mg : mg);
        const float sy = -s * y;
        r = (mg > 0.f ? sy * e : sy) / (1.f + e);
        if (want) l = (mg > 0.f ? 0.f : -mg) + log1pf(e);
    }
}

// What fm_evaluate counts, over the lanes with `has`: sum of losses, of squared errors, number of correct signs
// (a score of 0 counts as +1).  Written to out[0..2] by lane 0.
__device__ __forceinline__ void fm_eval_wave(bool has, float yh, float y, float l, int lane, double* out)
{
    const double d = has ? (double)yh - (double)y : 0.0;
    const float ls = fm_wave_sum(has ? l : 0.f);
    const double sq = fm_wave_sum(d * d);
    const int ok = __popcll(__ballot(has && (yh >= 0.f ? 1.f : -1.f) == y));
    if (lane == 0) {
        out[0] = (double)ls;
        out[1] = sq;
        out[2] = (double)ok;
    }
}

// Block b of the floor split of n items into P blocks that holds index i:
// b = floor(((i+1) P - 1) / n)   (inverse of the bound floor(b n / P)).
// The quotient in fp64, at most one off (both terms below 2^51), and put right: a division of 64-bit integers is a hundred
// instructions.
__device__ __forceinline__ int32_t fm_block_of(int64_t i, int64_t n, int32_t P)
{
    const int64_t x = (i + 1) * (int64_t)P - 1;
    int32_t b = (int32_t)((double)x * (1.0 / (double)n));
    const int64_t rest = x - (int64_t)b * n;
    if (rest < 0)
        --b;
    else if (rest >= n)
        ++b;
    return b;
}

template <bool FIRST, class A, class B>
__device__ __forceinline__ auto& fm_pick(A& a, B& b)
{
    if constexpr (FIRST) return a; else return b;
}

// Compile-time loop: f(std::integral_constant<int, I>) for I = 0..N-1.
template <int I, int N, class F>
__device__ __forceinline__ void fm_static_for(F&& f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        fm_static_for<I + 1, N>(f);
    }
}

// Value of `v` held by lane T of the caller's L-lane group, T known at compile time:
// a DPP quad permute for groups of up to four lanes (no LDS traffic), the LDS crossbar
// (ds_bpermute) for wider groups.
template <int L, int T>
__device__ __forceinline__ int fm_bcast_i(int v)
{
    if constexpr (L == 1) {
        return v;
    } else if constexpr (L == 2) {
        return __builtin_amdgcn_mov_dpp(v, T == 0 ? 0xA0 : 0xF5, 0xf, 0xf, true);
    } else if constexpr (L == 4) {
        return __builtin_amdgcn_mov_dpp(v, T * 0x55, 0xf, 0xf, true);
    } else if constexpr (L == 8) {
        // two DPP moves instead of a trip through the LDS crossbar: every quad broadcasts its lane
        // T % 4, then the quad that does not hold lane T takes the other quad's value (a row shift by
        // four lanes, written only to the banks of those quads)
        const int x = __builtin_amdgcn_mov_dpp(v, (T % 4) * 0x55, 0xf, 0xf, true);
        if constexpr (T < 4)
            return __builtin_amdgcn_update_dpp(x, x, 0x114 /* row_shr:4 */, 0xf, 0xa, false);
        else
            return __builtin_amdgcn_update_dpp(x, x, 0x104 /* row_shl:4 */, 0xf, 0x5, false);
    } else {
        return __shfl(v, T, L);
    }
}
template <int L, int T>
__device__ __forceinline__ float fm_bcast_f(float v)
{
    return __int_as_float(fm_bcast_i<L, T>(__float_as_int(v)));
}

// The score of a row by a wide group of L lanes: it walks the entries [beg,end), idx[e] names a row of `src` (`stride` floats
// apart) and val[e] its coefficient.  Lane `sub` of the group
//   * loads entry e+sub of every L entries (coalesced) and calls
//       m = own(index, value)      -- per-entry work of that lane, linear in the value;
//                                     returns the multiplier of the gathered row
//   * receives every entry's (index, m) by broadcast, four gathers at a time, and accumulates
//       acc[z] += m * src[index*stride + kb + z]     and     sq += m^2 * src[..]^2.
// Few registers, so that more rows are in flight.  `kb` must be a valid offset for every lane (idle lanes pass 0 and discard
// acc).
template <int VEC, int L, class Own, class SRC>
__device__ __forceinline__ void fm_gather_accumulate(const int32_t* __restrict__ idx, const float* __restrict__ val,
                                                     int64_t beg, int64_t end, const SRC* __restrict__ src,
                                                     int64_t stride, int sub, int kb, float (&acc)[VEC], float& sq,
                                                     Own&& own)
{
    for (int64_t e = beg; e < end; e += L) {
        const int64_t want = e + sub;
        const bool has = want < end;
        const int64_t my = has ? want : end - 1;
        const int ix = idx[my];
        const float mu = own(ix, has ? val[my] : 0.f);
        const int nv = (int)((end - e) < L ? (end - e) : L);  // only the entries that exist
        for (int t0 = 0; t0 < nv; t0 += 4) {
            float g[4][VEC];
            float mt[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = t0 + u < nv ? t0 + u : nv - 1;
                const int it = __shfl(ix, t, L);
                const float mm = __shfl(mu, t, L);
                mt[u] = t0 + u < nv ? mm : 0.f;
                fm_load_vec<VEC>(src + (int64_t)it * stride + kb, g[u]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
#pragma unroll
                for (int z = 0; z < VEC; ++z) {
                    acc[z] += mt[u] * g[u][z];
                    sq += (mt[u] * mt[u]) * (g[u][z] * g[u][z]);
                }
            }
        }
    }
}

// From this many lanes on a group walks alone (fm_walk_wide), below it in step with its wavefront's other groups
// (fm_walk).  Rounds in step for 16 lanes and more kept one to four runs per wavefront apart at the price of 78 to 102
// registers, six or four wavefronts per SIMD where eight fit: 2e6 hashed rows over 2e7 permuted columns, K=64, gradient
// 11.53 ms in step, 10.10 alone; stratified epoch over 128 strata 76.4 and 64.2 ms; text-like
// workload with K=64 stratified 1.10 and 1.08, K=22 1.11 and 1.04, epochs 135.8 and 134.7 us, 96.7 and 93.2 us.
constexpr int FM_WIDE_GROUP = 16;

// The inner loop of the column kernels and of the refresh for wide groups (K > 32, or K > 16 where it is not a multiple of
// four, or odd from 9 on).  A group walks its run [beg,end) L entries to a round, four gathers at a time, at most 64
// registers in all.  Latency-bound: the indices of the next round are on their way during this one, and the gathers of a
// round are issued before the multipliers (own's own loads) are waited for.
template <int VEC, int L, class Own, class SUM>
__device__ __forceinline__ void fm_walk_wide(const int32_t* __restrict__ idx, const float* __restrict__ val, int64_t beg,
                                             int64_t end, const float* __restrict__ src, int64_t stride, int sub, int kb,
                                             SUM (&acc)[VEC], Own&& own)
{
    const int len = (int)(end - beg);
    if (len <= 0) return;
    const int32_t* __restrict__ ip = idx + beg;
    const float* __restrict__ vp = val + beg;
    const float* __restrict__ sp = src + kb;
    int ix = ip[sub < len ? sub : len - 1];
    float mu = sub < len ? vp[sub] : 0.f;
    for (int at = 0;;) {
        const int nv = len - at < L ? len - at : L;
        const int i = ix;
        float x = mu;
        at += L;
        const int t = at + sub < len ? at + sub : len - 1;
        if (at < len) {  // the next round's indices are on their way during this one
            ix = ip[t];
            mu = at + sub < len ? vp[t] : 0.f;
        }
        x = own(i, x);
        for (int t0 = 0; t0 < nv; t0 += 4) {
            float g[4][VEC];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int it = __shfl(i, t0 + u < nv ? t0 + u : nv - 1, L);
                fm_load_vec<VEC>(sp + (int64_t)it * stride, g[u]);
            }
            constexpr bool APART = std::is_same_v<SUM, double>;  // four entries in fp32, these sums in fp64
            float sum[VEC];
#pragma unroll
            for (int z = 0; z < VEC; ++z) sum[z] = APART ? 0.f : (float)acc[z];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float m = __shfl(x, t0 + u, L);  // 0 where the run is over
#pragma unroll
                for (int z = 0; z < VEC; ++z) sum[z] += m * g[u][z];
            }
#pragma unroll
            for (int z = 0; z < VEC; ++z) acc[z] = APART ? acc[z] + (SUM)sum[z] : (SUM)sum[z];
        }
        if (at >= len) break;
    }
}

// How a walk addresses the rows it gathers.  BUF, BUF_NT: byte offsets of 32 bits from one buffer descriptor (arrays of
// up to FM_BUF_BYTES): one address register per gather instead of two, and an offset of FM_BUF_NONE is out of range,
// which reads zero without a request to memory, so slots without an entry cost nothing.  PTR: 64-bit addresses for
// larger arrays; slots without an entry repeat the run's last one.
enum { FM_ADDR_BUF = 0, FM_ADDR_BUF_NT = 1, FM_ADDR_PTR = 2 };
constexpr uint32_t FM_BUF_NONE = (uint32_t)FM_BUF_BYTES;  // + the offset inside a row (at most 1 KB) does not wrap

template <int VEC, bool NT>
__device__ __forceinline__ void fm_buf_load(__amdgpu_buffer_rsrc_t rs, uint32_t off, float (&v)[VEC])
{
    constexpr int AUX = NT ? 2 : 0;
    typedef int i4 __attribute__((ext_vector_type(4)));
    typedef int i2 __attribute__((ext_vector_type(2)));
    if constexpr (VEC == 4) {
        const i4 t = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, AUX);
        v[0] = __int_as_float(t.x); v[1] = __int_as_float(t.y); v[2] = __int_as_float(t.z); v[3] = __int_as_float(t.w);
    } else if constexpr (VEC == 2) {
        const i2 t = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)off, 0, AUX);
        v[0] = __int_as_float(t.x); v[1] = __int_as_float(t.y);
    } else {
        v[0] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, 0, AUX));
    }
}

// What a walk adds up per entry with value x and gathered row g:
//   SUM     acc += m g with the multiplier m that `own` makes of x
//   PACKED  rows are [G | r | ..] and the last lane of a group holds r in its first float; acc += x r G on the latent
//           lanes, gw += x r and s2 += x^2 r on every lane
//   SCORE   acc += x g, s2 += x^2 g^2
enum { FM_WALK_SUM = 0, FM_WALK_PACKED = 1, FM_WALK_SCORE = 2 };

// Per-entry work of the lane that holds the entry, besides the gathered row: load() asks for what the entry's index names
// (a slot without an entry, index < 0, gets zeros), use() takes it and returns the multiplier.  Two steps, so that what it
// asks for and the gathers of the round are on their way together.  end_round() after the entries that a lane holds of a round.
struct FmOwnNone {
    struct T {};
    template <int ADDR>
    __device__ __forceinline__ T load(int) const { return T(); }
    __device__ __forceinline__ float use(T, float x) const { return x; }
    __device__ __forceinline__ void end_round() const {}
};

// An array of W floats per index, read by load(): through a buffer descriptor, or with 64-bit addresses.
template <int W>
struct FmOwnArray {
    const float* p;
    uint32_t stride;  // floats
    __amdgpu_buffer_rsrc_t rs;
    __device__ __forceinline__ FmOwnArray(const float* p_, int64_t stride_)
        : p(p_), stride((uint32_t)stride_),
          rs(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p_), 0, (int)FM_BUF_NONE, 0x20000))
    {
    }
    template <int ADDR>
    __device__ __forceinline__ void get(int i, float (&v)[W]) const
    {
        if constexpr (ADDR == FM_ADDR_PTR) {
#pragma unroll
            for (int z = 0; z < W; ++z) v[z] = 0.f;
            if (i >= 0) fm_load_vec<W>(p + (int64_t)i * stride, v);
        } else {
            fm_buf_load<W, false>(rs, i >= 0 ? (uint32_t)i * (stride * (uint32_t)sizeof(float)) : FM_BUF_NONE, v);
        }
    }
};

// N consecutive entries at once; the arrays of entries are padded by FM_ENTRY_PAD, so that a load that begins inside a run
// stays inside its array.  Entries lie at any multiple of four bytes.
template <int N, typename T>
__device__ __forceinline__ void fm_load_entries(const T* __restrict__ p, T (&v)[N])
{
    static_assert(N - 1 <= FM_ENTRY_PAD, "loads past the end of a run");
    if constexpr (N >= 4) {
        typedef T t4 __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
        for (int i = 0; i < N; i += 4) {
            const t4 t = *reinterpret_cast<const t4*>(p + i);
            v[i] = t.x; v[i + 1] = t.y; v[i + 2] = t.z; v[i + 3] = t.w;
        }
    } else if constexpr (N == 2) {
        typedef T t2 __attribute__((ext_vector_type(2), aligned(4)));
        const t2 t = *reinterpret_cast<const t2*>(p);
        v[0] = t.x; v[1] = t.y;
    } else {
        v[0] = *p;
    }
}

// S slots of a round from slot S0 on (a lane holds U consecutive ones): the gathers ...
template <int VEC, int L, int ADDR, int S, int S0, bool FIRST, int U, class SRC>
__device__ __forceinline__ void fm_slot_loads(const int (&ix)[U], __amdgpu_buffer_rsrc_t rs, const SRC* __restrict__ src,
                                              int64_t stride, int kb, float (&g)[S][VEC])
{
    auto load_all = [&](auto&& load) {
        fm_static_for<0, S>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            constexpr int u = (S0 + s) % U, T = (S0 + s) / U;
            load(s, fm_bcast_i<L, T>(ix[u]));
        });
    };
    if constexpr (sizeof(SRC) == 2) {
        // FIRST: all requests before the first conversion.  Left to itself the compiler converts what two loads of eight lanes
        // have brought before it asks for more.
        static_assert(VEC == 4, "half rows come four at a time");
        typedef int i2 __attribute__((ext_vector_type(2)));
        i2 raw[S];
        load_all([&](int s, int it) {
            if constexpr (ADDR == FM_ADDR_PTR)
                raw[s] = *reinterpret_cast<const i2*>(src + (int64_t)it * stride + kb);
            else
                raw[s] = __builtin_amdgcn_raw_buffer_load_b64(rs, it + kb * (int)sizeof(SRC), 0, ADDR == FM_ADDR_BUF_NT ? 2 : 0);
        });
        if constexpr (FIRST) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const fm_h4 h = __builtin_bit_cast(fm_h4, raw[s]);
            g[s][0] = (float)h.x; g[s][1] = (float)h.y; g[s][2] = (float)h.z; g[s][3] = (float)h.w;
        }
    } else {
        load_all([&](int s, int it) {
            if constexpr (ADDR == FM_ADDR_PTR)
                fm_load_vec<VEC>(src + (int64_t)it * stride + kb, g[s]);
            else
                fm_buf_load<VEC, ADDR == FM_ADDR_BUF_NT>(rs, (uint32_t)it + (uint32_t)(kb * (int)sizeof(SRC)), g[s]);
        });
    }
}

// ... and the sums in entry order.
template <int VEC, int L, int KIND, int S, int S0, int U>
__device__ __forceinline__ void fm_slot_sums(const float (&mu)[U], const float (&g)[S][VEC], float (&acc)[VEC], float& gw, float& s2)
{
    fm_static_for<0, S>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        constexpr int u = (S0 + s) % U, T = (S0 + s) / U;
        const float x = fm_bcast_f<L, T>(mu[u]);
        if constexpr (KIND == FM_WALK_PACKED) {
            const float m = x * fm_bcast_f<L, L - 1>(g[s][0]);
#pragma unroll
            for (int z = 0; z < VEC; ++z) acc[z] += m * g[s][z];
            gw += m;
            s2 += x * m;
        } else {
#pragma unroll
            for (int z = 0; z < VEC; ++z) {
                acc[z] += x * g[s][z];
                if constexpr (KIND == FM_WALK_SCORE) s2 += (x * x) * (g[s][z] * g[s][z]);
            }
        }
    });
}

// Sums of the run in fp64: those of the batch in fp32, from zero, then added.
template <int VEC, int L, int KIND, int S, int S0, int U>
__device__ __forceinline__ void fm_slot_sums(const float (&mu)[U], const float (&g)[S][VEC], double (&acc)[VEC], double&, double&)
{
    static_assert(KIND == FM_WALK_SUM);
    float a[VEC] = {}, b = 0.f, c = 0.f;
    fm_slot_sums<VEC, L, KIND, S, S0>(mu, g, a, b, c);
#pragma unroll
    for (int z = 0; z < VEC; ++z) acc[z] += (double)a[z];
}

// The inner loop of the kernels for groups of up to eight lanes.  Every group of L lanes walks
// its own run [beg,end) of one row or column, all groups of the wavefront in step: a round takes the next C entries of
// every run, in batches of SMAX or four slots by the longest run left, so the choice is a scalar branch, and a group whose
// run is over sits the round out.  The indices of the next round are loaded while the gathers of this one are on their way,
// and so is what the holder of an entry asks for (own): a round costs one memory latency, not three.  Columns of a few
// entries are what a stratum or a batch consists of; with a
// slot loop and a four-at-a-time tail per group a column of 15 entries took six round trips, here it takes two.
// A lane loads the U = C / L entries of a round that it holds at once: the L1 stalls on every further request for a line
// that is still on its way, and entry by entry a round of four lanes made four of them (click-style scores, 2.5e6 rows,
// K=16: 806 -> 721 us with this change alone; 1e5 text-like rows, K=8: 79.9 -> 64.9).  Against the row kernel's own loop,
// without rounds in step, index prefetch or wide loads: 775 -> 721 and 78.6 -> 64.9 us.
// SMAX = 8 rather than 16: few registers, more wavefronts (mini-batch epoch of the click-style workload, 2.5e6 rows:
// 4.53 -> 4.20 ms).
// The refresh of a stratum, whose runs are mostly shorter than a round, takes rounds of four or eight in fours.
// kb: offset of the lane's slice in a row, valid for every lane.
// FIRST: see fm_slot_loads.
// SUM: float, or double for long runs (see FM_SHORT_RUNS).
// SP > 1: SP groups share a run, group `part` of them takes every SP-th stretch of C entries.
template <int VEC, int L, int KIND, int ADDR, int C = 16, int SMAX = 8, int SP = 1, bool FIRST = false, class Own, class SRC, class SUM>
__device__ __forceinline__ void fm_walk(const int32_t* __restrict__ idx, const float* __restrict__ val, int64_t beg,
                                        int len, const SRC* __restrict__ src, int64_t stride, int sub, int kb,
                                        SUM (&acc)[VEC], SUM& gw, SUM& s2, Own&& own, int part = 0)
{
    constexpr int U = C / L;
    constexpr bool APART = std::is_same_v<SUM, double> && KIND == FM_WALK_PACKED;
    static_assert(L < FM_WIDE_GROUP && C % L == 0 && ((SMAX == 8 && C == 16) || (SMAX == 4 && (C == 4 || C == 8))),
                  "rounds of whole batches");
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<SRC*>(src), 0, (int)FM_BUF_NONE, 0x20000);
    const uint32_t row_bytes = (uint32_t)stride * (uint32_t)sizeof(SRC);
    const int32_t* __restrict__ ip = idx + beg;
    const float* __restrict__ vp = val + beg;
    int raw[U];
    float mu[U];
    auto fetch = [&](int at, int (&i)[U], float (&x)[U]) {
        const int t = at + part * C + sub * U;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            i[u] = -1;
            x[u] = 0.f;
        }
        if (t < len) {
            fm_load_entries<U>(ip + t, i);
            fm_load_entries<U>(vp + t, x);
        }
#pragma unroll
        for (int u = 1; u < U; ++u) {
            i[u] = t + u < len ? i[u] : -1;
            x[u] = t + u < len ? x[u] : 0.f;
        }
    };
    fetch(0, raw, mu);
    int left = fm_wave_max<L * SP>(len);
    if (left <= 0) return;
    for (int at = 0;; at += C * SP, left -= C * SP) {
        int in[U];
        float mn[U];
        const bool more = left > C * SP;
        if (more) fetch(at + C * SP, in, mn);
        int ix[U];
        typename std::decay_t<Own>::T pre[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            pre[u] = own.template load<ADDR>(raw[u]);
            if constexpr (ADDR == FM_ADDR_PTR) {
                // a slot without an entry repeats an entry of its own run: of this lane's, or of the run's first lane,
                // which holds one as long as the run is not over
                const int first = fm_bcast_i<L, 0>(raw[0]);
                ix[u] = raw[u] >= 0 ? raw[u] : first >= 0 ? first : 0;
            } else {
                ix[u] = raw[u] >= 0 ? (int)((uint32_t)raw[u] * row_bytes) : (int)FM_BUF_NONE;
            }
        }
        auto multipliers = [&] {
#pragma unroll
            for (int u = 0; u < U; ++u) mu[u] = own.use(pre[u], mu[u]);
            own.end_round();
        };
        if (at + part * C < len) {
            [[maybe_unused]] float a[VEC] = {}, a_w = 0.f, a_2 = 0.f;  // packed rows: of the round
            auto& to = fm_pick<APART>(a, acc);
            auto& to_w = fm_pick<APART>(a_w, gw);
            auto& to_2 = fm_pick<APART>(a_2, s2);
            bool done = false;
            if constexpr (SMAX == 8) {
                if (left > 4) {
                    done = true;
                    float g[8][VEC];
                    fm_slot_loads<VEC, L, ADDR, 8, 0, FIRST>(ix, rs, src, stride, kb, g);
                    multipliers();
                    fm_slot_sums<VEC, L, KIND, 8, 0>(mu, g, to, to_w, to_2);
                    if (left > 8) {
                        fm_slot_loads<VEC, L, ADDR, 8, 8, FIRST>(ix, rs, src, stride, kb, g);
                        fm_slot_sums<VEC, L, KIND, 8, 8>(mu, g, to, to_w, to_2);
                    }
                }
            }
            if (!done) {
                float g[4][VEC];
                fm_slot_loads<VEC, L, ADDR, 4, 0, FIRST>(ix, rs, src, stride, kb, g);
                multipliers();
                fm_slot_sums<VEC, L, KIND, 4, 0>(mu, g, to, to_w, to_2);
                if constexpr (SMAX == 4 && C == 8) {
                    if (left > 4) {
                        fm_slot_loads<VEC, L, ADDR, 4, 4, FIRST>(ix, rs, src, stride, kb, g);
                        fm_slot_sums<VEC, L, KIND, 4, 4>(mu, g, to, to_w, to_2);
                    }
                }
            }
            if constexpr (APART) {
#pragma unroll
                for (int z = 0; z < VEC; ++z) acc[z] += (double)a[z];
                gw += (double)a_w;
                s2 += (double)a_2;
            }
        }
        if (!more) break;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            raw[u] = in[u];
            mu[u] = mn[u];
        }
    }
}
