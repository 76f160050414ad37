// Estimators from the root counts R (Algorithm 1's last loop and the farness
// identity of Section 4.2):
//   diag[v]      = R[v] / tau                      estimates Omega_vv
//   farness[v]   = (n R[v] + S) / tau - 2          n Omega_vv + tr(Omega) - 2
//   closeness[v] = n / farness[v]
// with S = sum_w R[w] an exact 64-bit integer, so every output is one or two
// correctly rounded binary64 operations and is bit-reproducible.
#include "fc_kernels.hpp"

#pragma clang fp contract(off)

namespace fc {

namespace {

// HBM streaming; the blocks are few and each adds once to the total (an atomic
// per wave of 2048 blocks was 8192 atomics on one address, 40 us for 200 K
// counts and 101 us for 10^6; now 5.7 us and 6.1 us).
constexpr uint32_t kSumThreads = 256, kSumBlocks = 256;

__global__ __launch_bounds__(kSumThreads) void sum_u32_kernel(const uint32_t *__restrict__ x,
                                                              int32_t n, unsigned long long *sum) {
    __shared__ unsigned long long s_sum[kSumThreads / 64u];
    unsigned long long acc = 0;
    const int64_t step = static_cast<int64_t>(gridDim.x) * kSumThreads;
    int64_t i = static_cast<int64_t>(blockIdx.x) * kSumThreads + threadIdx.x;
    for (; i + 7 * step < n; i += 8 * step) {  // eight loads in flight
        uint32_t r[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) r[q] = x[i + q * step];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc += r[q];
    }
    for (; i < n; i += step) acc += x[i];
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    if ((threadIdx.x & 63u) == 0) s_sum[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (uint32_t w = 1; w < kSumThreads / 64u; ++w) acc += s_sum[w];
    if (acc) atomicAdd(sum, acc);
}

__global__ __launch_bounds__(256) void estimate_kernel(const uint32_t *__restrict__ R, int32_t n,
                                                       uint32_t tau, int literal,
                                                       const unsigned long long *__restrict__ sum,
                                                       double *__restrict__ diag,
                                                       double *__restrict__ farness,
                                                       double *__restrict__ closeness) {
    const int32_t v = static_cast<int32_t>(blockIdx.x * blockDim.x + threadIdx.x);
    if (v >= n) return;
    const double dt = static_cast<double>(tau);
    const uint32_t r = R[v];
    if (diag) {
        double d = static_cast<double>(r) / dt;
        if (literal) {
            // minimum-norm solution of L* x = e_{u*} - 1/(n+1) 1 gives
            // - x(u*) + 2 x(v) = -(n+2)/(n+1)^2
            const double n1 = static_cast<double>(static_cast<int64_t>(n) + 1);
            const double shift = static_cast<double>(static_cast<int64_t>(n) + 2) / (n1 * n1);
            d = d - shift;
        }
        diag[v] = d;
    }
    if (farness || closeness) {
        const unsigned long long num =
            static_cast<unsigned long long>(n) * r + *sum;
        const double f = static_cast<double>(num) / dt - 2.0;
        if (farness) farness[v] = f;
        if (closeness) closeness[v] = static_cast<double>(n) / f;
    }
}

// Plain fills (used instead of memset nodes inside captured HIP graphs).
__global__ void fill_u64_kernel(unsigned long long *__restrict__ p, size_t count,
                                unsigned long long value) {
    for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < count;
         i += static_cast<size_t>(gridDim.x) * blockDim.x)
        p[i] = value;
}

}  // namespace

hipError_t launch_fill_u64(unsigned long long *p, size_t count, unsigned long long value,
                           hipStream_t stream) {
    if (count == 0) return hipSuccess;
    size_t blocks = (count + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    fill_u64_kernel<<<static_cast<unsigned int>(blocks), 256, 0, stream>>>(p, count, value);
    return hipGetLastError();
}

hipError_t launch_sum_u32(const uint32_t *x, int32_t n, unsigned long long *sum,
                          hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const uint32_t blocks = (static_cast<uint32_t>(n) + kSumThreads - 1u) / kSumThreads;
    sum_u32_kernel<<<blocks < kSumBlocks ? blocks : kSumBlocks, kSumThreads, 0, stream>>>(x, n, sum);
    return hipGetLastError();
}

hipError_t launch_estimate(const uint32_t *R, int32_t n, uint32_t tau, int literal,
                           const unsigned long long *sum, double *diag, double *farness,
                           double *closeness, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    estimate_kernel<<<(n + 255) / 256, 256, 0, stream>>>(R, n, tau, literal, sum, diag, farness,
                                                         closeness);
    return hipGetLastError();
}

}  // namespace fc
