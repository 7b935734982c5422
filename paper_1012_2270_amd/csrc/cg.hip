// The vector kernels of a conjugate-gradient iteration.
//
// A short solve is bound by launches and by the waits between them, a long one
// by the vectors' bytes.  One workgroup of 1,024 threads per CU reads 16 bytes
// per load; each kernel first adds the partial sums of the one before it (in a
// fixed order, the same in every workgroup), so no kernel of one workgroup
// stands between them: three launches an iteration beside the SpMV instead of
// five, two where the SpMV leaves the parts of p.q.  27-point 96^3 (884,736
// rows), BF16, 136 iterations: 20.7 us an iteration before, 13.7 as three
// kernels (3.5 to 17.7 MB each, held by the Infinity Cache: bound by launch and
// by the wait for the first loads), 10.9 and 0.9 more in the SpMV as two; the
// gap every fourth iteration, where the host decides, is filled by the next
// product; the solve 6.85 -> 4.64 ms.  Sums are FP64 and in a fixed order, so a
// solve gives the same bits every time.
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace rg {

constexpr int kCgThreads = 1024;

// Sum of v over the workgroup, in every thread.
__device__ __forceinline__ double cg_block_sum(double v) {
    __shared__ double sh[kCgThreads / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < kCgThreads / 64; i++) t += sh[i];
    __syncthreads();
    return t;
}

__device__ __forceinline__ double cg_finish(const double *part, int n) {
    double v = 0.0;
    for (int i = threadIdx.x; i < n; i += kCgThreads) v += part[i];
    return cg_block_sum(v);
}

// 16 bytes of a vector that starts at any element
template <class VT> struct CgVec {
    static constexpr int W = 16 / (int)sizeof(VT);
    typedef VT type __attribute__((ext_vector_type(W)));
    typedef type at __attribute__((aligned(sizeof(VT))));
};

// f(first element, count) over [0, n): W elements per thread and pass, the
// rest by single elements
template <class VT, class F> __device__ __forceinline__ void cg_loop(int64_t n, F f) {
    constexpr int W = CgVec<VT>::W;
    const int64_t nv = n / W, stride = (int64_t)gridDim.x * kCgThreads;
    const int64_t t = (int64_t)blockIdx.x * kCgThreads + threadIdx.x;
    int64_t i = t;
    for (; i + stride < nv; i += 2 * stride) f(i * W, (i + stride) * W);
    if (i < nv) f(i * W, (int64_t)-1);
}

template <class VT>
__global__ __launch_bounds__(kCgThreads) void cg_dot_k(int64_t n, const VT *p, const VT *q, double *part) {
    using VA = typename CgVec<VT>::at;
    constexpr int W = CgVec<VT>::W;
    double acc = 0.0;
    auto one = [&](const typename CgVec<VT>::type &a, const typename CgVec<VT>::type &b) {
#pragma unroll
        for (int j = 0; j < W; j++) acc += (double)a[j] * (double)b[j];
    };
    cg_loop<VT>(n, [&](int64_t i, int64_t k) {
        const typename CgVec<VT>::type a = *(const VA *)(p + i), b = *(const VA *)(q + i);
        if (k >= 0) {
            const typename CgVec<VT>::type c = *(const VA *)(p + k), d = *(const VA *)(q + k);
            one(a, b);
            one(c, d);
        } else {
            one(a, b);
        }
    });
    if (blockIdx.x == 0 && threadIdx.x < n % W) {
        const int64_t i = n / W * W + threadIdx.x;
        acc += (double)p[i] * (double)q[i];
    }
    const double t = cg_block_sum(acc);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
}

template <class VT>
__global__ __launch_bounds__(kCgThreads) void cg_step_k(int64_t n, VT *x, VT *r, const VT *p, const VT *q,
                                                        const double *rr, const double *part_pq, int n_pq,
                                                        double *part_rr) {
    using VV = typename CgVec<VT>::type;
    using VA = typename CgVec<VT>::at;
    constexpr int W = CgVec<VT>::W;
    const VT alpha = (VT)(*rr / cg_finish(part_pq, n_pq));
    double acc = 0.0;
    auto one = [&](int64_t i, VV xv, VV rv, const VV &pv, const VV &qv) {
#pragma unroll
        for (int j = 0; j < W; j++) {
            xv[j] += alpha * pv[j];
            rv[j] = rv[j] - alpha * qv[j];
            acc += (double)rv[j] * (double)rv[j];
        }
        *(VA *)(x + i) = xv;
        *(VA *)(r + i) = rv;
    };
    cg_loop<VT>(n, [&](int64_t i, int64_t k) {
        const VV x0 = *(const VA *)(x + i), r0 = *(const VA *)(r + i), p0 = *(const VA *)(p + i),
                 q0 = *(const VA *)(q + i);
        if (k >= 0) {
            const VV x1 = *(const VA *)(x + k), r1 = *(const VA *)(r + k), p1 = *(const VA *)(p + k),
                     q1 = *(const VA *)(q + k);
            one(i, x0, r0, p0, q0);
            one(k, x1, r1, p1, q1);
        } else {
            one(i, x0, r0, p0, q0);
        }
    });
    if (blockIdx.x == 0 && threadIdx.x < n % W) {
        const int64_t i = n / W * W + threadIdx.x;
        x[i] += alpha * p[i];
        const VT ri = r[i] - alpha * q[i];
        r[i] = ri;
        acc += (double)ri * (double)ri;
    }
    const double t = cg_block_sum(acc);
    if (threadIdx.x == 0) part_rr[blockIdx.x] = t;
}

template <class VT>
__global__ __launch_bounds__(kCgThreads) void cg_dir_k(int64_t n, VT *p, const VT *r, const double *rr_old,
                                                       double *rr_new, const double *rr0, const double *part_rr,
                                                       CgHost *host, unsigned long long seq) {
    using VV = typename CgVec<VT>::type;
    using VA = typename CgVec<VT>::at;
    constexpr int W = CgVec<VT>::W;
    const double s = cg_finish(part_rr, (int)gridDim.x);
    const VT beta = (VT)(s / *rr_old);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *rr_new = s;
        if (host) {
            host->rr = s;
            host->rr0 = *rr0;
            __hip_atomic_store(&host->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    cg_loop<VT>(n, [&](int64_t i, int64_t k) {
        const VV r0 = *(const VA *)(r + i);
        VV p0 = *(const VA *)(p + i);
        if (k >= 0) {
            const VV r1 = *(const VA *)(r + k);
            VV p1 = *(const VA *)(p + k);
#pragma unroll
            for (int j = 0; j < W; j++) p1[j] = r1[j] + beta * p1[j];
            *(VA *)(p + k) = p1;
        }
#pragma unroll
        for (int j = 0; j < W; j++) p0[j] = r0[j] + beta * p0[j];
        *(VA *)(p + i) = p0;
    });
    if (blockIdx.x == 0 && threadIdx.x < n % W) {
        const int64_t i = n / W * W + threadIdx.x;
        p[i] = r[i] + beta * p[i];
    }
}

hipError_t launch_cg_dot(int64_t n, const void *p, const void *q, int f64, double *part_pq, hipStream_t st) {
    const dim3 g(cg_blocks(n)), b(kCgThreads);
    if (f64) hipLaunchKernelGGL(cg_dot_k<double>, g, b, 0, st, n, (const double *)p, (const double *)q, part_pq);
    else hipLaunchKernelGGL(cg_dot_k<float>, g, b, 0, st, n, (const float *)p, (const float *)q, part_pq);
    return hipGetLastError();
}

// r.r before iteration it (kScalRRInit writes the first)
static int rr_slot(int it) { return it % 2 ? kRR : kRROdd; }

hipError_t launch_cg_step(int64_t n, void *x, void *r, const void *p, const void *q, int f64, const double *scal,
                          int it, const double *part_pq, int n_pq, double *part_rr, hipStream_t st) {
    const dim3 g(cg_blocks(n)), b(kCgThreads);
    const double *rr = scal + rr_slot(it);
    if (f64)
        hipLaunchKernelGGL(cg_step_k<double>, g, b, 0, st, n, (double *)x, (double *)r, (const double *)p,
                           (const double *)q, rr, part_pq, n_pq, part_rr);
    else
        hipLaunchKernelGGL(cg_step_k<float>, g, b, 0, st, n, (float *)x, (float *)r, (const float *)p,
                           (const float *)q, rr, part_pq, n_pq, part_rr);
    return hipGetLastError();
}

hipError_t launch_cg_dir(int64_t n, void *p, const void *r, int f64, double *scal, int it, const double *part_rr,
                         CgHost *host, unsigned long long seq, hipStream_t st) {
    const dim3 g(cg_blocks(n)), b(kCgThreads);
    const double *old = scal + rr_slot(it);
    double *now = scal + rr_slot(it + 1);
    if (f64)
        hipLaunchKernelGGL(cg_dir_k<double>, g, b, 0, st, n, (double *)p, (const double *)r, old, now, scal + kRR0,
                           part_rr, host, seq);
    else
        hipLaunchKernelGGL(cg_dir_k<float>, g, b, 0, st, n, (float *)p, (const float *)r, old, now, scal + kRR0,
                           part_rr, host, seq);
    return hipGetLastError();
}

}  // namespace rg
