// Sums over the examples and the bias step as roles of workgroups inside other launches: an epoch of a small matrix is
// bound by its launches, and the sums depend on nothing but the row kernel.  Fixed order, fp64 accumulation.
#pragma once

#include "fm_device.h"
#include "fm_internal.h"

// Sum over the workgroup (T threads), valid in thread 0.  sh: T / 64 doubles.
template <int T>
__device__ __forceinline__ double fm_block_sum(double v, double* sh)
{
    v = fm_wave_sum(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < T / 64; ++i) t += sh[i];
    __syncthreads();
    return t;
}

template <int T>
__device__ __forceinline__ void fm_epi_load(const FmEpilogue& E, int64_t lo, int64_t hi, double& s0, double& s1)
{
    if (E.single) {
        for (int64_t i = lo + threadIdx.x; i < hi; i += T) s1 += (double)E.x[i * E.stride];
    } else {
        const float2* __restrict__ p = reinterpret_cast<const float2*>(E.x);
        for (int64_t i = lo + threadIdx.x; i < hi; i += T) {
            const float2 v = p[i];
            s0 += (double)v.x;
            s1 += (double)v.y;
        }
    }
}

// Workgroup b of E.nsums: its contiguous share of the values.  sh: T / 64 doubles.
template <int T>
__device__ __forceinline__ void fm_epi_partial(const FmEpilogue& E, int b, double* sh)
{
    const int64_t chunk = (E.n + E.nsums - 1) / E.nsums;
    const int64_t lo = (int64_t)b * chunk;
    const int64_t hi = lo + chunk < E.n ? lo + chunk : E.n;
    double s0 = 0.0, s1 = 0.0;
    fm_epi_load<T>(E, lo, hi, s0, s1);
    const double t0 = fm_block_sum<T>(s0, sh);
    const double t1 = fm_block_sum<T>(s1, sh);
    if (threadIdx.x == 0) {
        E.sums[2 * b] = t0;
        E.sums[2 * b + 1] = t1;
    }
}

// |w|^2 and |V|^2 by one workgroup, into out[0..1].
template <int T>
__device__ __forceinline__ void fm_reg_pair(const float* __restrict__ w, int64_t nw, const float* __restrict__ V, int64_t nV,
                                            double* out, double* sh)
{
    double a = 0.0, b = 0.0;
    for (int64_t i = threadIdx.x; i < nw; i += T) a += (double)w[i] * (double)w[i];
    for (int64_t i = threadIdx.x; i < nV; i += T) b += (double)V[i] * (double)V[i];
    a = fm_block_sum<T>(a, sh);
    b = fm_block_sum<T>(b, sh);
    if (threadIdx.x == 0) {
        out[0] = a;
        out[1] = b;
    }
}

template <int T>
__device__ __forceinline__ void fm_epi_final(const FmEpilogue& E, double* sh)
{
    double s0 = 0.0, s1 = 0.0, q0 = 0.0, q1 = 0.0;
    if (E.nsums > 0) {
        for (int i = threadIdx.x; i < E.nsums; i += T) {
            s0 += E.sums[2 * i];
            s1 += E.sums[2 * i + 1];
        }
    } else {
        fm_epi_load<T>(E, 0, E.n, s0, s1);
    }
    if (E.regs != nullptr)
        for (int i = threadIdx.x; i < E.nregs; i += T) {
            q0 += E.regs[2 * i];
            q1 += E.regs[2 * i + 1];
        }
    if (E.reg_w != nullptr) {
        for (int64_t i = threadIdx.x; i < E.reg_nw; i += T) q0 += (double)E.reg_w[i] * (double)E.reg_w[i];
        for (int64_t i = threadIdx.x; i < E.reg_nV; i += T) q1 += (double)E.reg_V[i] * (double)E.reg_V[i];
    }
    const double loss = fm_block_sum<T>(s0, sh);
    const double rsum = fm_block_sum<T>(s1, sh);
    if (E.regs != nullptr || E.reg_w != nullptr) {
        q0 = fm_block_sum<T>(q0, sh);
        q1 = fm_block_sum<T>(q1, sh);
    }
    if (threadIdx.x == 0) {
        E.scal[0] = loss;
        E.scal[1] = rsum;
        const float g = (float)rsum;
        if (E.grad_w0 != nullptr) E.grad_w0[0] = g;
        if (E.w0 != nullptr) E.w0[0] = E.w0[0] - E.eta * g;
        if (E.host != nullptr) {
            E.host[0] = loss;
            E.host[1] = rsum;
            E.host[2] = q0;
            E.host[3] = q1;
        }
    }
}
