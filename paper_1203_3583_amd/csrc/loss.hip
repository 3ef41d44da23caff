// The phase-hologram loss around the transforms (include/asf.h): the phase-only source
// field, the intensity mismatch and the two ends of its gradient, each one pass over its
// arrays, and between them one workgroup that adds the mismatch's partial sums.  The four
// passes are bound by memory: one thread per element and step, neighbouring lanes on
// neighbouring elements, every array read or written once.  (At 1024^2 points and pixels
// they move 88 MB with FP32 phases and an FP64 target, 96 MB with FP64 phases; as separate
// elementwise operations the same arithmetic took 30 launches and 1.0 GB around the same
// forward and adjoint.)
#include <hip/hip_runtime.h>

#include "asf_internal.h"

namespace asf {
namespace {

constexpr int kThreads = 256;
constexpr int64_t kMaxBlocks = 2048;   // eight workgroups per CU

// u1 = amp exp(i theta), theta rounded to FP32
template <class T>
__global__ void __launch_bounds__(kThreads) phase_field_kernel(int64_t n, const float *__restrict__ amp,
                                                               const T *__restrict__ theta,
                                                               float2 *__restrict__ u1) {
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
        float s, c;
        sincosf((float)theta[i], &s, &c);
        u1[i] = make_float2(amp[i] * c, amp[i] * s);
    }
}

// Sum of v over the workgroup, in thread 0 (a fixed order: the same sum every time).
__device__ inline double block_sum(double v, double *scratch) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s += scratch[i];
    return s;
}

// diff = |u2|^2 - target in FP64; per workgroup the sums of diff^2 and target^2
template <class T>
__global__ void __launch_bounds__(kThreads) loss_kernel(int64_t m, const float2 *__restrict__ u2,
                                                        const T *__restrict__ target, double *__restrict__ diff,
                                                        double *__restrict__ partial) {
    __shared__ double scratch[kThreads / 64];
    double num = 0.0, den = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < m; i += (int64_t)gridDim.x * kThreads) {
        const float2 u = u2[i];
        const double t = (double)target[i];
        const double d = ((double)u.x * (double)u.x + (double)u.y * (double)u.y) - t;
        diff[i] = d;
        num += d * d;
        den += t * t;
    }
    num = block_sum(num, scratch);
    den = block_sum(den, scratch);
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = num;
        partial[2 * blockIdx.x + 1] = den;
    }
}

// sums[0] = sum of target^2, loss[0] = sum of diff^2 over it
__global__ void __launch_bounds__(1024) loss_finish_kernel(int blocks, const double *__restrict__ partial,
                                                           double *__restrict__ den_out, double *__restrict__ loss) {
    __shared__ double scratch[16];
    double num = 0.0, den = 0.0;
    for (int i = threadIdx.x; i < blocks; i += 1024) {
        num += partial[2 * i];
        den += partial[2 * i + 1];
    }
    num = block_sum(num, scratch);
    den = block_sum(den, scratch);
    if (threadIdx.x == 0) {
        den_out[0] = den;
        loss[0] = num / den;
    }
}

// g2 = 4 grad / den diff u2 (the gradient of u2, real and imaginary parts), formed in
// FP64 and rounded once
__global__ void __launch_bounds__(kThreads) loss_backward_kernel(int64_t m, const float2 *__restrict__ u2,
                                                                 const double *__restrict__ diff,
                                                                 const double *__restrict__ den,
                                                                 const double *__restrict__ grad,
                                                                 float2 *__restrict__ g2) {
    const double k = 4.0 * (grad[0] / den[0]);
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < m; i += (int64_t)gridDim.x * kThreads) {
        const float2 u = u2[i];
        const double d = k * diff[i];
        g2[i] = make_float2((float)(d * (double)u.x), (float)(d * (double)u.y));
    }
}

// dtheta = Re(conj(g1) i u1) = g1.y u1.x - g1.x u1.y
template <class T>
__global__ void __launch_bounds__(kThreads) phase_backward_kernel(int64_t n, const float2 *__restrict__ u1,
                                                                  const float2 *__restrict__ g1,
                                                                  T *__restrict__ dtheta) {
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
        const float2 u = u1[i], g = g1[i];
        dtheta[i] = (T)(g.y * u.x - g.x * u.y);
    }
}

unsigned blocks_for(int64_t n) {
    const int64_t b = (n + kThreads - 1) / kThreads;
    return (unsigned)(b < kMaxBlocks ? b : kMaxBlocks);
}

}  // namespace

hipError_t launch_phase_field(int64_t n, const float *amp, const void *theta, bool f64, float2 *u1, hipStream_t s) {
    if (f64)
        hipLaunchKernelGGL(phase_field_kernel<double>, dim3(blocks_for(n)), dim3(kThreads), 0, s, n, amp,
                           static_cast<const double *>(theta), u1);
    else
        hipLaunchKernelGGL(phase_field_kernel<float>, dim3(blocks_for(n)), dim3(kThreads), 0, s, n, amp,
                           static_cast<const float *>(theta), u1);
    return hipGetLastError();
}

hipError_t launch_intensity_loss(int64_t m, const float2 *u2, const void *target, bool f64, double *diff,
                                 double *sums, double *loss, hipStream_t s) {
    static_assert(ASF_LOSS_SUMS >= 2 * kMaxBlocks + 1, "a pair per workgroup, and the denominator");
    const unsigned blocks = blocks_for(m);
    if (f64)
        hipLaunchKernelGGL(loss_kernel<double>, dim3(blocks), dim3(kThreads), 0, s, m, u2,
                           static_cast<const double *>(target), diff, sums + 1);
    else
        hipLaunchKernelGGL(loss_kernel<float>, dim3(blocks), dim3(kThreads), 0, s, m, u2,
                           static_cast<const float *>(target), diff, sums + 1);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(loss_finish_kernel, dim3(1), dim3(1024), 0, s, (int)blocks, sums + 1, sums, loss);
    return hipGetLastError();
}

hipError_t launch_intensity_loss_backward(int64_t m, const float2 *u2, const double *diff, const double *sums,
                                          const double *grad, float2 *g2, hipStream_t s) {
    hipLaunchKernelGGL(loss_backward_kernel, dim3(blocks_for(m)), dim3(kThreads), 0, s, m, u2, diff, sums, grad, g2);
    return hipGetLastError();
}

hipError_t launch_phase_backward(int64_t n, const float2 *u1, const float2 *g1, void *dtheta, bool f64,
                                 hipStream_t s) {
    if (f64)
        hipLaunchKernelGGL(phase_backward_kernel<double>, dim3(blocks_for(n)), dim3(kThreads), 0, s, n, u1, g1,
                           static_cast<double *>(dtheta));
    else
        hipLaunchKernelGGL(phase_backward_kernel<float>, dim3(blocks_for(n)), dim3(kThreads), 0, s, n, u1, g1,
                           static_cast<float *>(dtheta));
    return hipGetLastError();
}

}  // namespace asf
