// Shared pieces of the two-level preconditioned CG (cg_coarse.hip): the
// device scalars of one inner solve, the ordered sums of partials that every
// workgroup forms for itself, and the barycentric weights that tie an
// element's N nodes to its four corners.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace stdg {

// Slots of the scalar record of a solve.  Kernels of iteration `it` return at
// once when DONE holds an iteration number <= it (0: not done); the kernel
// that sets it writes it + 1, so its own late workgroups still run.
enum { TL_RZ = 0 /* two slots, by parity */, TL_ALPHA = 2, TL_DONE = 3, TL_RR = 4, TL_ITERS = 5, TL_COUNT = 6 };

__device__ inline bool tl_done(const double* scal, int it) {
    const double d = scal[TL_DONE];
    return d != 0.0 && d <= (double)it;
}

// sum of part[stride i], i < n, in a fixed order by a workgroup of T threads;
// every thread gets it (sh: T / 64 doubles)
template <int T> __device__ inline double tl_sum(const double* __restrict__ part, int n, int stride, double* sh) {
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += T) s += part[(int64_t)stride * i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < T / 64; ++w) t += sh[w];
    return t;
}

// sum of v over a workgroup of T threads in a fixed order, valid in thread 0
template <int T> __device__ inline double tl_reduce(double v, double* sh) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < T / 64; ++w) t += sh[w];
    return t;
}

// alpha = (r.z) / (p.q) of iteration `it` (0 at the start and on a breakdown)
__device__ inline double tl_alpha(const double* scal, double pq, int it) {
    const double rz = scal[TL_RZ + ((it - 1) & 1)];
    return it > 0 && pq > 0.0 && rz > 0.0 ? rz / pq : 0.0;
}

// The scalars of the direction update of iteration `it`: every workgroup
// forms them from the same partials, workgroup 0 records them.
struct TlStep {
    double alpha, beta;
    bool stop;      // converged or broken down: x is updated, p is not
};
template <int T>
__device__ inline TlStep tl_step(double* scal, int it, const double* __restrict__ part_up, int n_up,
                                 const double* __restrict__ part_c, int n_c, double cdot_scale, double tol2,
                                 double* sh) {
    TlStep s;
    const double rr = tl_sum<T>(part_up, n_up, 2, sh);
    const double rz = tl_sum<T>(part_up + 1, n_up, 2, sh) + cdot_scale * tl_sum<T>(part_c, n_c, 1, sh);
    s.alpha = scal[TL_ALPHA];
    const double prev = it > 0 ? scal[TL_RZ + ((it - 1) & 1)] : 0.0;
    s.beta = prev > 0.0 ? rz / prev : 0.0;
    s.stop = !(rr > tol2) || (it > 0 && s.alpha == 0.0) || !(rz > 0.0);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        scal[TL_RZ + (it & 1)] = rz;
        scal[TL_RR] = rr;
        scal[TL_ITERS] = (double)it;
        if (s.stop) scal[TL_DONE] = (double)(it + 1);
    }
    return s;
}

// Barycentric coordinates of the nodes (j1, j2, j3)/p, j1 fastest: the values
// of the four corner functions at node r are w[r][0..3].
template <int N> struct Bary {
    float w[N][4];
    constexpr Bary() : w() {
        const int p = N == 4 ? 1 : (N == 10 ? 2 : (N == 20 ? 3 : 4));
        int r = 0;
        for (int c = 0; c <= p; ++c)
            for (int b = 0; b <= p - c; ++b)
                for (int a = 0; a <= p - c - b; ++a, ++r) {
                    w[r][0] = (float)(p - a - b - c) / (float)p;
                    w[r][1] = (float)a / (float)p;
                    w[r][2] = (float)b / (float)p;
                    w[r][3] = (float)c / (float)p;
                }
    }
};

}  // namespace stdg
