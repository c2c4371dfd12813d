// Elementwise kernels (initial state, stand-alone cost layer), the <C>/norm
// readout, and the fixed-order reduction of per-workgroup FP64 partial sums.
//
// <C> (arXiv:2604.26423, eq. 5 with exact probabilities): sum |a_x|^2 C(x)
// over the normalised state.  Partial sums are FP64, combined in a fixed
// order (no atomics), so the result is identical from run to run.
#include <algorithm>

#include "device.h"

namespace qs {

namespace {

constexpr int kElemThreads = 256;
constexpr int64_t kElemMaxBlocks = 16384;
constexpr int kReduceChunk = 1024;

int64_t elem_grid(int64_t dim)
{
    int64_t g = (dim + kElemThreads - 1) / kElemThreads;
    return g < kElemMaxBlocks ? g : kElemMaxBlocks;
}

template <typename V>
__global__ void __launch_bounds__(kElemThreads) init_plus_kernel(V *psi, int64_t dim, double amp0)
{
    using R = typename Real<V>::T;
    const V a{(R)amp0, (R)0};
    for (int64_t x = (int64_t)blockIdx.x * kElemThreads + threadIdx.x; x < dim;
         x += (int64_t)gridDim.x * kElemThreads)
        psi[x] = a;
}

// exp(-i theta (W - 2C)/20), per element from an FP64 argument reduced mod 2 pi.
template <typename V>
__global__ void __launch_bounds__(kElemThreads) cost_layer_kernel(V *psi, const int32_t *diag,
                                                                  int64_t dim, int64_t W, double theta)
{
    for (int64_t x = (int64_t)blockIdx.x * kElemThreads + threadIdx.x; x < dim;
         x += (int64_t)gridDim.x * kElemThreads)
        psi[x] = cmul(psi[x], expi<V>(theta * (double)(2 * (int64_t)diag[x] - W) / 20.0));
}

// Bound by the read of the state and the diagonal (12 B per complex64
// amplitude): 16-byte streaming loads from a contiguous range per workgroup, four
// strides in flight (strides of the whole grid instead: 275 us), and
// no more workgroups than fill the chip, so that one reduction chunk takes
// their sums (one amplitude per load and 16384 workgroups: 283 us + 16 us of
// reductions at n = 27, now 230 + 5).
constexpr int kExpectThreads = 512;
constexpr int64_t kExpectMaxBlocks = 512;
template <typename V>
__global__ void __launch_bounds__(kExpectThreads) expect_kernel(const V *psi, const int32_t *diag, int64_t dim,
                                                                double *partials)
{
    using Wd = WideLoad<V>;
    constexpr int K = Wd::K, U = 4;
    __shared__ double red[2 * (kExpectThreads / 64)];
    double acc[2] = {0.0, 0.0};
    auto add = [&](const V (&a)[K], const int32_t (&c)[K]) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double pr = (double)a[k].x * (double)a[k].x + (double)a[k].y * (double)a[k].y;
            acc[0] += pr;
            acc[1] += pr * (double)c[k];
        }
    };
    // a contiguous range per workgroup (dim and the grid are powers of two, dim
    // at least 2)
    const int64_t S = kExpectThreads * K, per = dim / gridDim.x, lo = blockIdx.x * per, hi = lo + per;
    int64_t x = lo + (int64_t)threadIdx.x * K;
    for (; x + (U - 1) * S < hi; x += U * S) {
        V a[U][K];
        int32_t c[U][K];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            Wd::load(psi, x + u * S, a[u]);
            Wd::load_c(diag, x + u * S, c[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) add(a[u], c[u]);
    }
    for (; x < hi; x += S) {
        V a[K];
        int32_t c[K];
        Wd::load(psi, x, a);
        Wd::load_c(diag, x, c);
        add(a, c);
    }
    block_sum(acc, red, threadIdx.x, kExpectThreads);
    if (threadIdx.x == 0) {
        partials[blockIdx.x * kSlots + 0] = acc[0];
        partials[blockIdx.x * kSlots + 1] = acc[1];
        partials[blockIdx.x * kSlots + 2] = 0.0;
        partials[blockIdx.x * kSlots + 3] = 0.0;
    }
}

// The rows of a job are summed in chunks of kReduceChunk, one workgroup each,
// and the chunks' sums by one workgroup per job: a fixed order.  A workgroup
// reads four rows per thread, so that a job of one chunk (up to 2^10 tiles)
// costs one launch and the time of a few loads.
__device__ __forceinline__ void sum_rows(const double *in, int64_t lo, int64_t hi, double *red, double *out)
{
    double acc[kSlots] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
#pragma unroll
        for (int k = 0; k < kSlots; ++k) acc[k] += in[i * kSlots + k];
    }
    block_sum(acc, red, threadIdx.x, 256);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < kSlots; ++k) out[k] = acc[k];
    }
}

__host__ __device__ __forceinline__ int64_t reduce_chunks(int64_t rows)
{
    return (rows + kReduceChunk - 1) / kReduceChunk;
}

// Workgroup (b, j): chunk b of job j.
__global__ void __launch_bounds__(256) reduce_chunks_kernel(const double *in, ReduceJobs jobs, int64_t stride,
                                                            double *tmp)
{
    __shared__ double red[kSlots * 4];
    const int j = blockIdx.y;
    const int64_t rows = jobs.rows[j], lo = (int64_t)blockIdx.x * kReduceChunk;
    if (lo >= rows) return;
    const int64_t hi = lo + kReduceChunk < rows ? lo + kReduceChunk : rows;
    sum_rows(in + jobs.off[j] * kSlots, lo, hi, red, tmp + (j * stride + blockIdx.x) * kSlots);
}

// Workgroup j: job j, from its rows (stride 0) or from its chunks' sums.
__global__ void __launch_bounds__(256) reduce_jobs_kernel(const double *in, ReduceJobs jobs, int64_t stride,
                                                          double *out)
{
    __shared__ double red[kSlots * 4];
    const int j = blockIdx.x;
    if (stride) sum_rows(in + j * stride * kSlots, 0, reduce_chunks(jobs.rows[j]), red, out + j * kSlots);
    else sum_rows(in + jobs.off[j] * kSlots, 0, jobs.rows[j], red, out + j * kSlots);
}

}  // namespace

namespace {
// Copies between index order and the swizzled state layout (internal.h).
template <typename V>
__global__ void __launch_bounds__(kElemThreads) gather_kernel(const V *psi, int64_t first, int64_t count, V *dst)
{
    for (int64_t i = (int64_t)blockIdx.x * kElemThreads + threadIdx.x; i < count; i += (int64_t)gridDim.x * kElemThreads)
        dst[i] = psi[swz(first + i)];
}

template <typename V>
__global__ void __launch_bounds__(kElemThreads) scatter_kernel(V *psi, int64_t first, int64_t count, const V *src)
{
    for (int64_t i = (int64_t)blockIdx.x * kElemThreads + threadIdx.x; i < count; i += (int64_t)gridDim.x * kElemThreads)
        psi[swz(first + i)] = src[i];
}
}  // namespace

hipError_t launch_copy_amplitudes(int prec, void *psi, int64_t first, int64_t count, void *buf, int to_state,
                                  hipStream_t st)
{
    if (count <= 0) return hipSuccess;
    const dim3 g((unsigned)elem_grid(count)), b(kElemThreads);
    if (prec == 0) {
        if (to_state) hipLaunchKernelGGL(scatter_kernel<float2>, g, b, 0, st, (float2 *)psi, first, count, (const float2 *)buf);
        else hipLaunchKernelGGL(gather_kernel<float2>, g, b, 0, st, (const float2 *)psi, first, count, (float2 *)buf);
    } else {
        if (to_state) hipLaunchKernelGGL(scatter_kernel<double2>, g, b, 0, st, (double2 *)psi, first, count, (const double2 *)buf);
        else hipLaunchKernelGGL(gather_kernel<double2>, g, b, 0, st, (const double2 *)psi, first, count, (double2 *)buf);
    }
    return hipGetLastError();
}

hipError_t launch_init_plus(int prec, void *psi, int n, int nq, hipStream_t st)
{
    const int64_t dim = (int64_t)1 << n;
    const double amp0 = sqrt(ldexp(1.0, -nq));
    if (prec == 0)
        hipLaunchKernelGGL(init_plus_kernel<float2>, dim3((unsigned)elem_grid(dim)), dim3(kElemThreads), 0, st,
                           (float2 *)psi, dim, amp0);
    else
        hipLaunchKernelGGL(init_plus_kernel<double2>, dim3((unsigned)elem_grid(dim)), dim3(kElemThreads), 0, st,
                           (double2 *)psi, dim, amp0);
    return hipGetLastError();
}

hipError_t launch_cost_layer(int prec, void *psi, const int32_t *diag, int n, int64_t W, double theta,
                             hipStream_t st)
{
    const int64_t dim = (int64_t)1 << n;
    if (prec == 0)
        hipLaunchKernelGGL(cost_layer_kernel<float2>, dim3((unsigned)elem_grid(dim)), dim3(kElemThreads), 0, st,
                           (float2 *)psi, diag, dim, W, theta);
    else
        hipLaunchKernelGGL(cost_layer_kernel<double2>, dim3((unsigned)elem_grid(dim)), dim3(kElemThreads), 0,
                           st, (double2 *)psi, diag, dim, W, theta);
    return hipGetLastError();
}

int64_t expect_grid(int64_t dim)
{
    const int64_t g = (dim + 2 * kExpectThreads - 1) / (2 * kExpectThreads);
    return g < kExpectMaxBlocks ? g : kExpectMaxBlocks;
}

hipError_t launch_expect(int prec, const void *psi, const int32_t *diag, int n, double *partials, hipStream_t st)
{
    const int64_t dim = (int64_t)1 << n;
    const dim3 g((unsigned)expect_grid(dim)), b(kExpectThreads);
    if (prec == 0) hipLaunchKernelGGL(expect_kernel<float2>, g, b, 0, st, (const float2 *)psi, diag, dim, partials);
    else hipLaunchKernelGGL(expect_kernel<double2>, g, b, 0, st, (const double2 *)psi, diag, dim, partials);
    return hipGetLastError();
}

int64_t reduce_tmp_doubles(int64_t rows)
{
    // every job has at most kReduceJobs times the chunks of the longest
    return kReduceJobs * (reduce_chunks(rows) + 1) * kSlots;
}

hipError_t launch_reduce_jobs(const double *partials, const ReduceJobs &jobs, double *tmp, double *out,
                              hipStream_t st)
{
    if (jobs.count < 1 || jobs.count > kReduceJobs) return hipErrorInvalidValue;
    int64_t chunks = 0;
    for (int j = 0; j < jobs.count; ++j) chunks = std::max(chunks, reduce_chunks(jobs.rows[j]));
    const int64_t stride = chunks > 1 ? chunks : 0;
    if (stride) {
        hipLaunchKernelGGL(reduce_chunks_kernel, dim3((unsigned)chunks, (unsigned)jobs.count), dim3(256), 0, st,
                           partials, jobs, stride, tmp);
        if (hipError_t e = hipGetLastError()) return e;
    }
    hipLaunchKernelGGL(reduce_jobs_kernel, dim3((unsigned)jobs.count), dim3(256), 0, st, stride ? tmp : partials, jobs,
                       stride, out);
    return hipGetLastError();
}

}  // namespace qs
