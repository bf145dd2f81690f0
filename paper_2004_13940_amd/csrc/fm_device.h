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

// Sum over the L lanes of a group (L a power of two, groups aligned to L lanes);
// every lane of the group receives the total.  Fixed butterfly order.
template <int L, typename T>
__device__ __forceinline__ T fm_group_sum(T v)
{
#pragma unroll
    for (int o = L / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, L);
    return v;
}

// Sum over all 64 lanes of the wave, fixed butterfly order.
template <typename T>
__device__ __forceinline__ T fm_wave_sum(T v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Loss value and multiplier for one example (cases after eq. updates_v; the loss
// constants make the printed multiplier the exact derivative).  expf only ever sees
// a non-positive argument.
__device__ __forceinline__ void loss_and_multiplier(int32_t loss, float s, float yh, float y, float& l, float& r)
{
    if (loss == FM_LOSS_SQUARED) {
        const float d = yh - y;
        l = 0.5f * d * d;
        r = s * d;
    } else {
        const float mg = y * yh;
        if (mg > 0.f) {
            const float e = expf(-mg);
            l = log1pf(e);
            r = -s * y * e / (1.f + e);
        } else {
            const float e = expf(mg);
            l = -mg + log1pf(e);
            r = -s * y / (1.f + e);
        }
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
__device__ __forceinline__ int32_t fm_block_of(int64_t i, int64_t n, int32_t P)
{
    return (int32_t)(((i + 1) * (int64_t)P - 1) / n);
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

// Entry slots per lane and iteration so that a group keeps 16 row gathers in flight.
template <int L>
struct FmChunk {
    static constexpr int CH = (16 / L) > 0 ? (16 / L) : 1;
};

// S entry slots (slot s = entry s%L of lane-slot s/L): broadcast each entry's index and
// multiplier inside the group, gather the rows with at most 16 loads in flight, then
// accumulate.
template <int VEC, int L, bool SQ, int S, class IX, class MU, class SRC>
__device__ __forceinline__ void fm_gather_slots(const IX& ix, const MU& mu, const SRC* __restrict__ src,
                                                int64_t stride, int kb, float (&acc)[VEC], float& sq)
{
    constexpr int B = S < 16 ? S : 16;
    fm_static_for<0, S / B>([&](auto bc) {
        constexpr int B0 = decltype(bc)::value * B;
        float g[B][VEC];
        float mt[B];
        fm_static_for<0, B>([&](auto sc) {
            constexpr int s = B0 + decltype(sc)::value;
            constexpr int u = s / L, T = s % L;
            const int raw = fm_bcast_i<L, T>(ix[u]);
            mt[s - B0] = fm_bcast_f<L, T>(mu[u]);
            fm_load_vec<VEC>(src + (int64_t)raw * stride + kb, g[s - B0]);
        });
#pragma unroll
        for (int s = 0; s < B; ++s) {
#pragma unroll
            for (int z = 0; z < VEC; ++z) {
                acc[z] += mt[s] * g[s][z];
                if constexpr (SQ) sq += (mt[s] * mt[s]) * (g[s][z] * g[s][z]);
            }
        }
    });
}

// The inner loop of the row kernels.  A group of L lanes walks the entries [beg,end) of one sparse row: idx[e] names a row of `src`
// (`stride` floats apart) and val[e] its coefficient.  Lane `sub` of the group
//   * loads entry e+sub of every L-entry slot (coalesced) and calls
//       m = own(index, value)      -- per-entry work of that lane, linear in the value;
//                                     returns the multiplier of the gathered row
//   * receives every entry's (index, m) by broadcast and accumulates
//       acc[z] += m * src[index*stride + kb + z]     (and, if SQ, sq += m^2 * src[..]^2).
// Full chunks of L*CH entries run without masking; the tail runs in L-entry slots whose
// missing entries repeat the last entry with value 0.  `kb` must be a valid offset for
// every lane (idle lanes pass 0 and discard acc).
template <int VEC, int L, bool SQ, int CH = FmChunk<L>::CH, class Own, class SRC = float>
__device__ __forceinline__ void fm_gather_accumulate(const int32_t* __restrict__ idx, const float* __restrict__ val,
                                                     int64_t beg, int64_t end, const SRC* __restrict__ src,
                                                     int64_t stride, int sub, int kb, float (&acc)[VEC], float& sq,
                                                     Own&& own)
{
    int64_t e = beg;
    // the lean form (CH == 1) of wide groups takes every entry through the four-at-a-time loop below:
    // few registers, so that more rows or columns are in flight
    constexpr bool CHUNKS = !(CH == 1 && L >= 16);
    for (; CHUNKS && e + L * CH <= end; e += L * CH) {
        int ix[CH];
        float mu[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int64_t my = e + u * L + sub;
            ix[u] = idx[my];
            mu[u] = val[my];
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) mu[u] = own(ix[u], mu[u]);
        fm_gather_slots<VEC, L, SQ, CH * L>(ix, mu, src, stride, kb, acc, sq);
    }
    for (; e < end; e += L) {
        const int64_t want = e + sub;
        const bool has = want < end;
        const int64_t my = has ? want : end - 1;
        int ix[1];
        float mu[1];
        ix[0] = idx[my];
        mu[0] = own(ix[0], has ? val[my] : 0.f);
        if constexpr (L <= 4) {
            fm_gather_slots<VEC, L, SQ, L>(ix, mu, src, stride, kb, acc, sq);
        } else {
            // wide groups: only the entries that exist, four gathers at a time
            const int nv = (int)((end - e) < L ? (end - e) : L);
            for (int t0 = 0; t0 < nv; t0 += 4) {
                float g[4][VEC];
                float mt[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int t = t0 + u < nv ? t0 + u : nv - 1;
                    const int it = __shfl(ix[0], t, L);
                    const float mm = __shfl(mu[0], t, L);
                    mt[u] = t0 + u < nv ? mm : 0.f;
                    fm_load_vec<VEC>(src + (int64_t)it * stride + kb, g[u]);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
#pragma unroll
                    for (int z = 0; z < VEC; ++z) {
                        acc[z] += mt[u] * g[u][z];
                        if constexpr (SQ) sq += (mt[u] * mt[u]) * (g[u][z] * g[u][z]);
                    }
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
template <int VEC, int L, class Own>
__device__ __forceinline__ void fm_walk_wide(const int32_t* __restrict__ idx, const float* __restrict__ val, int64_t beg,
                                             int64_t end, const float* __restrict__ src, int64_t stride, int sub, int kb,
                                             float (&acc)[VEC], Own&& own)
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
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float m = __shfl(x, t0 + u, L);  // 0 where the run is over
#pragma unroll
                for (int z = 0; z < VEC; ++z) acc[z] += m * g[u][z];
            }
        }
        if (at >= len) break;
    }
}

// Largest value over the 64 lanes, as a wave-uniform number (a scalar register: branches on it do not diverge).
__device__ __forceinline__ int fm_wave_max(int v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const int t = __shfl_xor(v, o, 64);
        v = t > v ? t : v;
    }
    return __builtin_amdgcn_readfirstlane(v);
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

// What a walk adds up per entry with multiplier m and gathered row g:
//   SUM     acc += m g
//   PACKED  rows are [G | r | ..], lane rl holds r in its first float; acc += x r G on the latent lanes,
//           gw += x r and s2 += x^2 r on lane rl
enum { FM_WALK_SUM = 0, FM_WALK_PACKED = 1 };

// S slots of a round from slot S0 on: all loads, then all sums in entry order.
template <int VEC, int L, int KIND, int ADDR, int S, int S0, class IX, class MU>
__device__ __forceinline__ void fm_slots(const IX& ix, const MU& mu, __amdgpu_buffer_rsrc_t rs, const float* __restrict__ src,
                                         int64_t stride, int kb, int rl, bool scalar_lane, float (&acc)[VEC], float& gw,
                                         float& s2)
{
    float g[S][VEC];
    float xt[S];
    fm_static_for<0, S>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        constexpr int u = (S0 + s) / L, T = (S0 + s) % L;
        const int it = fm_bcast_i<L, T>(ix[u]);
        xt[s] = fm_bcast_f<L, T>(mu[u]);
        if constexpr (ADDR == FM_ADDR_PTR)
            fm_load_vec<VEC>(src + (int64_t)it * stride + kb, g[s]);
        else
            fm_buf_load<VEC, ADDR == FM_ADDR_BUF_NT>(rs, (uint32_t)it + (uint32_t)(kb * (int)sizeof(float)), g[s]);
    });
#pragma unroll
    for (int s = 0; s < S; ++s) {
        if constexpr (KIND == FM_WALK_PACKED) {
            const float m = xt[s] * __shfl(g[s][0], rl, L);
#pragma unroll
            for (int z = 0; z < VEC; ++z) acc[z] += m * g[s][z];
            if (scalar_lane) {
                gw += m;
                s2 += xt[s] * m;
            }
        } else {
#pragma unroll
            for (int z = 0; z < VEC; ++z) acc[z] += xt[s] * g[s][z];
        }
    }
}

// The inner loop of the column kernels and of the refresh for groups of up to eight lanes.  Every group of L lanes walks
// its own run [beg,end) of one column, all groups of the wavefront in step: a round takes the next C entries of every run,
// in batches of SMAX or four slots by the longest run left, so the choice is a scalar branch, and a group whose run is
// over sits the round out.  The indices of the next round are loaded while the gathers of this one are on their way: a
// round costs one memory latency, not two.  Columns of a few entries are what a stratum or a batch consists of; with a
// slot loop and a four-at-a-time tail per group a column of 15 entries took six round trips, here it takes two.
// SMAX = 8 rather than 16 in the columns: 103 registers instead of 146 at eight lanes of a packed row, four wavefronts per
// SIMD instead of three (mini-batch epoch of the click-style workload, 2.5e6 rows: 4.53 -> 4.20 ms).
// The refresh of a stratum, whose runs are mostly shorter than a round, takes rounds of four or eight in fours.
//   own(index, value) -> multiplier: the work of the lane that holds the entry
template <int VEC, int L, int KIND, int ADDR, int C = 16, int SMAX = 8, class Own>
__device__ __forceinline__ void fm_walk(const int32_t* __restrict__ idx, const float* __restrict__ val, int64_t beg,
                                        int64_t end, const float* __restrict__ src, int64_t stride, int sub, int kb, int rl,
                                        float (&acc)[VEC], float& gw, float& s2, Own&& own)
{
    constexpr int U = C / L;
    static_assert(L < FM_WIDE_GROUP && C % L == 0 && ((SMAX == 8 && C == 16) || (SMAX == 4 && (C == 4 || C == 8))),
                  "rounds of whole batches");
    const int len = (int)(end - beg);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(src), 0, (int)FM_BUF_NONE, 0x20000);
    const uint32_t row_bytes = (uint32_t)stride * (uint32_t)sizeof(float);
    const bool scalar_lane = sub == rl;
    const int32_t* __restrict__ ip = idx + beg;
    const float* __restrict__ vp = val + beg;
    int ix[U], raw[U];
    float mu[U];
    auto fetch = [&](int at, int (&i)[U], float (&x)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = at + u * L + sub;
            i[u] = -1;
            x[u] = 0.f;
            if (t < len) {
                i[u] = ip[t];
                x[u] = vp[t];
            } else if (ADDR == FM_ADDR_PTR && len > 0) {
                i[u] = ip[len - 1];
            }
        }
    };
    // Short rounds: the first indices are on their way while the longest run is found, six steps across the wavefront.
    // Not for the columns: mini-batch click epoch 4.23 -> 3.96 ms, but full click epoch 7.37 -> 7.59 ms.
    constexpr bool EARLY = C < 16;
    if constexpr (EARLY) fetch(0, raw, mu);
    int left = fm_wave_max(len);
    if (left <= 0) return;
    if constexpr (!EARLY) fetch(0, raw, mu);
    for (int at = 0;; at += C, left -= C) {
        int in[U];
        float mn[U];
        const bool more = left > C;
        if (more) fetch(at + C, in, mn);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (ADDR == FM_ADDR_PTR) {
                ix[u] = raw[u] < 0 ? 0 : raw[u];  // only where the run is empty: its group sits the round out
                if (at + u * L + sub < len) mu[u] = own(raw[u], mu[u]);
            } else {
                ix[u] = (int)FM_BUF_NONE;
                if (raw[u] >= 0) {
                    mu[u] = own(raw[u], mu[u]);
                    ix[u] = (int)((uint32_t)raw[u] * row_bytes);
                }
            }
        }
        if (at < len) {
            bool done = false;
            if constexpr (SMAX == 8) {
                if (left > 4) {
                    done = true;
                    fm_slots<VEC, L, KIND, ADDR, 8, 0>(ix, mu, rs, src, stride, kb, rl, scalar_lane, acc, gw, s2);
                    if (left > 8)
                        fm_slots<VEC, L, KIND, ADDR, 8, 8>(ix, mu, rs, src, stride, kb, rl, scalar_lane, acc, gw, s2);
                }
            }
            if (!done) {
                fm_slots<VEC, L, KIND, ADDR, 4, 0>(ix, mu, rs, src, stride, kb, rl, scalar_lane, acc, gw, s2);
                if constexpr (SMAX == 4 && C == 8) {
                    if (left > 4)
                        fm_slots<VEC, L, KIND, ADDR, 4, 4>(ix, mu, rs, src, stride, kb, rl, scalar_lane, acc, gw, s2);
                }
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
