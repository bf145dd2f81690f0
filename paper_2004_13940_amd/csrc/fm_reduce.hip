// Deterministic reductions (fixed order, fp64 accumulation) and the bias step.
#include "fm_device.h"
#include "fm_epilogue.h"
#include "fm_internal.h"

namespace {

constexpr int RED_THREADS = 1024;
constexpr int RED_BLOCKS = FM_REDUCE_TMP;

__device__ __forceinline__ double block_sum_1024(double v, double* sh)
{
    v = fm_wave_sum(v);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) sh[wave] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < RED_THREADS / 64; ++i) t += sh[i];
    __syncthreads();
    return t;  // valid in thread 0
}

// part holds n interleaved pairs (x0,x1).  Stage 1: workgroup b sums its contiguous share of the
// pairs into tmp[2b], tmp[2b+1]; stage 2: one workgroup adds the nb partial pairs into out2.
__global__ __launch_bounds__(RED_THREADS) void k_reduce_pairs(const float* __restrict__ part, int64_t n,
                                                              double* __restrict__ tmp)
{
    __shared__ double sh[RED_THREADS / 64];
    const int64_t chunk = (n + gridDim.x - 1) / gridDim.x;
    const int64_t lo = (int64_t)blockIdx.x * chunk;
    const int64_t hi = lo + chunk < n ? lo + chunk : n;
    double s0 = 0.0, s1 = 0.0;
    const float2* p2 = reinterpret_cast<const float2*>(part);
    for (int64_t i = lo + threadIdx.x; i < hi; i += RED_THREADS) {
        const float2 v = p2[i];
        s0 += (double)v.x;
        s1 += (double)v.y;
    }
    const double t0 = block_sum_1024(s0, sh);
    const double t1 = block_sum_1024(s1, sh);
    if (threadIdx.x == 0) {
        tmp[2 * blockIdx.x] = t0;
        tmp[2 * blockIdx.x + 1] = t1;
    }
}

__global__ __launch_bounds__(RED_THREADS) void k_reduce_pairs_final(const double* __restrict__ tmp, int nb,
                                                                    double* __restrict__ out2)
{
    __shared__ double sh[RED_THREADS / 64];
    double s0 = 0.0, s1 = 0.0;
    for (int i = threadIdx.x; i < nb; i += RED_THREADS) {
        s0 += tmp[2 * i];
        s1 += tmp[2 * i + 1];
    }
    const double t0 = block_sum_1024(s0, sh);
    const double t1 = block_sum_1024(s1, sh);
    if (threadIdx.x == 0) {
        out2[0] = t0;
        out2[1] = t1;
    }
}

// one workgroup straight over the pairs, for as many as it reads in a few rounds
__global__ __launch_bounds__(RED_THREADS) void k_reduce_pairs_small(const float* __restrict__ part, int64_t n,
                                                                    double* __restrict__ out2)
{
    __shared__ double sh[RED_THREADS / 64];
    double s0 = 0.0, s1 = 0.0;
    const float2* p2 = reinterpret_cast<const float2*>(part);
    for (int64_t i = threadIdx.x; i < n; i += RED_THREADS) {
        const float2 v = p2[i];
        s0 += (double)v.x;
        s1 += (double)v.y;
    }
    const double t0 = block_sum_1024(s0, sh);
    const double t1 = block_sum_1024(s1, sh);
    if (threadIdx.x == 0) {
        out2[0] = t0;
        out2[1] = t1;
    }
}

// |w|^2 and |V|^2: workgroup b writes the pair of its shares of both arrays
__global__ __launch_bounds__(RED_THREADS) void k_reg_partials(const float* __restrict__ w, int64_t nw,
                                                              const float* __restrict__ V, int64_t nV,
                                                              double* __restrict__ out)
{
    __shared__ double sh[RED_THREADS / 64];
    auto share = [&](const float* __restrict__ x, int64_t n) {
        const int64_t chunk = (n + gridDim.x - 1) / gridDim.x;
        const int64_t lo = (int64_t)blockIdx.x * chunk;
        const int64_t hi = lo + chunk < n ? lo + chunk : n;
        double s = 0.0;
        for (int64_t i = lo + threadIdx.x; i < hi; i += RED_THREADS) {
            const double v = (double)x[i];
            s += v * v;
        }
        return block_sum_1024(s, sh);
    };
    const double a = share(w, nw);
    const double b = share(V, nV);
    if (threadIdx.x == 0) {
        out[2 * blockIdx.x] = a;
        out[2 * blockIdx.x + 1] = b;
    }
}

__global__ __launch_bounds__(FM_BLOCK) void k_epi_sums(const FmEpilogue E)
{
    __shared__ double sh[FM_WAVES];
    fm_epi_partial<FM_BLOCK>(E, blockIdx.x, sh);
}

__global__ __launch_bounds__(RED_THREADS) void k_epi_final(const FmEpilogue E)
{
    __shared__ double sh[RED_THREADS / 64];
    fm_epi_final<RED_THREADS>(E, sh);
}

// part: n triples (loss, squared error, correct signs); workgroup b sums its contiguous share into out[3b..3b+2]
__global__ __launch_bounds__(RED_THREADS) void k_eval_sums(const double* __restrict__ part, int64_t n,
                                                           double* __restrict__ out)
{
    __shared__ double sh[RED_THREADS / 64];
    const int64_t chunk = (n + gridDim.x - 1) / gridDim.x;
    const int64_t lo = (int64_t)blockIdx.x * chunk;
    const int64_t hi = lo + chunk < n ? lo + chunk : n;
    double s[3] = {0.0, 0.0, 0.0};
    for (int64_t i = lo + threadIdx.x; i < hi; i += RED_THREADS)
#pragma unroll
        for (int c = 0; c < 3; ++c) s[c] += part[3 * i + c];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double t = block_sum_1024(s[c], sh);
        if (threadIdx.x == 0) out[3 * blockIdx.x + c] = t;
    }
}

__global__ void k_fill_i32(int32_t* __restrict__ x, int64_t n, int32_t v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = v;
}

}  // namespace

int fm_reduce_pairs(fm_matrix* m, const float* part, int64_t nblocks, double* out2, hipStream_t st, double* tmp)
{
    // stage-1 scratch of FM_REDUCE_TMP doubles (pairs: at most RED_BLOCKS / 2 workgroups); by default
    // scal[8..8+RED_BLOCKS)
    if (tmp == nullptr) tmp = m->scal + 8;
    int nb = (int)((nblocks + 4 * RED_THREADS - 1) / (4 * RED_THREADS));
    if (nb < 1) nb = 1;
    if (nb > RED_BLOCKS / 2) nb = RED_BLOCKS / 2;
    ProfScope ps(m, st, FMK_REDUCE);
    if (nb == 1) {
        hipLaunchKernelGGL(k_reduce_pairs_small, dim3(1), dim3(RED_THREADS), 0, st, part, nblocks, out2);
        FM_HIP(m, hipGetLastError());
        return FM_OK;
    }
    hipLaunchKernelGGL(k_reduce_pairs, dim3(nb), dim3(RED_THREADS), 0, st, part, nblocks, tmp);
    FM_HIP(m, hipGetLastError());
    hipLaunchKernelGGL(k_reduce_pairs_final, dim3(1), dim3(RED_THREADS), 0, st, (const double*)tmp, nb, out2);
    FM_HIP(m, hipGetLastError());
    return FM_OK;
}

double* fm_reg_scratch(fm_matrix* m)
{
    // behind the partial pairs of the epilogue (2 * 512 doubles) in the handle's scratch
    static_assert(FM_REDUCE_TMP >= 2 * 512 + 2 * FM_REG_PAIRS, "scratch of the reductions");
    return m->scal + 8 + 2 * 512;
}

int fm_reg_partials(fm_matrix* m, const float* w, int64_t nw, const float* V, int64_t nV, const double** regs, int32_t* nregs,
                    hipStream_t st)
{
    double* out = fm_reg_scratch(m);
    int64_t nb = (std::max(nw, nV) + 16 * RED_THREADS - 1) / (16 * RED_THREADS);
    nb = std::min<int64_t>(std::max<int64_t>(nb, 1), FM_REG_PAIRS);
    ProfScope ps(m, st, FMK_REDUCE);
    hipLaunchKernelGGL(k_reg_partials, dim3((unsigned)nb), dim3(RED_THREADS), 0, st, w, nw, V, nV, out);
    FM_HIP(m, hipGetLastError());
    *regs = out;
    *nregs = (int32_t)nb;
    return FM_OK;
}

int fm_run_epilogue(fm_matrix* m, const FmEpilogue& E, hipStream_t st)
{
    ProfScope ps(m, st, FMK_REDUCE);
    if (E.nsums > 0) {
        hipLaunchKernelGGL(k_epi_sums, dim3((unsigned)E.nsums), dim3(FM_BLOCK), 0, st, E);
        FM_HIP(m, hipGetLastError());
    }
    return fm_run_epilogue_final(m, E, st);
}

int fm_run_epilogue_final(fm_matrix* m, const FmEpilogue& E, hipStream_t st)
{
    hipLaunchKernelGGL(k_epi_final, dim3(1), dim3(RED_THREADS), 0, st, E);
    FM_HIP(m, hipGetLastError());
    return FM_OK;
}

// n triples per row block into out3; tmp: 3 * 256 doubles
int fm_reduce_eval(fm_matrix* m, const double* part, int64_t n, double* out3, double* tmp, hipStream_t st)
{
    ProfScope ps(m, st, FMK_REDUCE);
    if (n > 4 * RED_THREADS) {
        const int nb = (int)std::min<int64_t>(256, (n + RED_THREADS - 1) / RED_THREADS);
        hipLaunchKernelGGL(k_eval_sums, dim3(nb), dim3(RED_THREADS), 0, st, part, n, tmp);
        FM_HIP(m, hipGetLastError());
        part = tmp;
        n = nb;
    }
    hipLaunchKernelGGL(k_eval_sums, dim3(1), dim3(RED_THREADS), 0, st, part, n, out3);
    FM_HIP(m, hipGetLastError());
    return FM_OK;
}

// A fill by a kernel (not a memset node), so that a caller may capture the epoch into a graph.
int fm_fill_i32(fm_matrix* m, int32_t* x, int64_t n, int32_t v, hipStream_t st)
{
    if (n <= 0) return FM_OK;
    const int64_t grid = (n + 255) / 256;
    if (grid > 0x7fffffffLL) return fm_fail(m, FM_ERANGE, "fill too large");
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)grid), dim3(256), 0, st, x, n, v);
    FM_HIP(m, hipGetLastError());
    return FM_OK;
}
