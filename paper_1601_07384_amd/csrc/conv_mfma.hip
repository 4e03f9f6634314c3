// Space-time DG convection with the Rusanov flux (eq. convdg) on the FP64
// matrix cores, for meshes whose groups of one geometry class fill.
//
// Evaluating the velocity at the quadrature points and testing the fluxes
// against the basis are contractions with tables that a class (the volume
// tables: every element) shares, and they chain without moving data: the
// points of a group of four come out of the first product with point hi of a
// column in lane group hi (mfma64.hpp), so the lane forms that point's fluxes
// from its three components, and the fluxes are the contraction operand
// (over the points) of the second product as they stand.
//
// One workgroup per group and component-wise 16 elements per wavefront; the
// time points run inside, their sums weighted into the G output rows in
// registers.  The tables pass through LDS in chunks of QC points: one copy
// [point][N padded] serves both products.  663,552 elements, p = 3: 60 matrix
// instructions of 256 FMAs per four volume points and 45 per four face points,
// 0.9 ms of the matrix cores in all; measured 7,204 us for the kernel with a
// lane per element and scalar tables, 1,803 us here (196,608 elements, p = 2,
// p_gamma = 1: 785 -> 473 us; 24,576, p = 3, p_gamma = 2: 1,876 -> 550; 3,072,
// p = 4, p_gamma = 1: 1,304 -> 499).

#include "internal.hpp"
#include "kernels.hpp"
#include "mfma64.hpp"

namespace stdg {
namespace {

constexpr int CT = 256;
constexpr int QC = 36;      // points per chunk: a face of p = 3 whole, its 125 volume points in four

// n points' rows of N doubles, `stride` apart, from src into LDS [QC][NP], zero
// where point or column is padding
template <int N> __device__ inline void stage_points(const double* __restrict__ src, int n, int stride, double* L) {
    constexpr int NP = M64<N>::NP;
    for (int t = threadIdx.x; t < QC * NP; t += CT) {
        const int k = t % NP, q = t / NP;
        L[t] = q < n && k < N ? src[(int64_t)q * stride + k] : 0.0;
    }
}

// v[c] += values of the columns' coefficients x[c] at points 4 g + lane row:
// lane (hi, column) ends up with point 4 g + hi
template <int N>
__device__ __forceinline__ void eval_points(const double* L, int g, int lo, int hi, const double (&x)[3][M64<N>::NQ],
                                            double (&v)[3]) {
    constexpr int NQ = M64<N>::NQ, NP = M64<N>::NP;
    v[0] = v[1] = v[2] = 0.0;
#pragma unroll
    for (int t = 0; t < NQ; ++t) {
        const double a = L[(4 * g + lo) * NP + m64_col<N>(t, hi)];
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, x[c][t], v[c], 0, 0, 0);
    }
}

// o[rg][c] += sum over the four points of a group of table(point, row) f[c]
template <int N>
__device__ __forceinline__ void test_points(const double* L, int g, int lo, int hi, const double (&f)[3],
                                            double (&o)[M64<N>::NQ][3]) {
    constexpr int NQ = M64<N>::NQ, NP = M64<N>::NP;
#pragma unroll
    for (int rg = 0; rg < NQ; ++rg) {
        const double a = L[(4 * g + hi) * NP + 4 * rg + lo];
#pragma unroll
        for (int c = 0; c < 3; ++c) o[rg][c] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, f[c], o[rg][c], 0, 0, 0);
    }
}

template <int N, int G>
__global__ void __launch_bounds__(CT) kc_convection(
    const double* __restrict__ vbar, const double* __restrict__ vbc, const m64_i4* __restrict__ segs,
    const int32_t* __restrict__ nbr, const int64_t* __restrict__ tet_face, const double* __restrict__ cJinv,
    const double* __restrict__ cdet, const double* __restrict__ cnrm, const double* __restrict__ PHf,
    const double* __restrict__ PHn, const double* __restrict__ FW, const double* __restrict__ PHv,
    const double* __restrict__ dPHv, const double* __restrict__ wv, const double* __restrict__ tw,
    const double* __restrict__ gq, int nqv, int nqf, int qt, double dt, double* __restrict__ ups, int64_t E, int64_t F,
    uint32_t n_segs) {
    constexpr int NQ = M64<N>::NQ, NP = M64<N>::NP;
    // volume: values and the three gradient components; faces: own and neighbour's values
    constexpr int LD = 4 * QC * NP > 64 * G * N ? 4 * QC * NP : 64 * G * N;
    __shared__ double L[LD];
    __shared__ double Wq[QC];
    const uint32_t group = m64_group(gridDim.x);
    if (group >= n_segs) return;
    const m64_i4 sg = segs[group];
    const int cl = sg.z;
    const int64_t e0 = sg.x, e1 = e0 + sg.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hi = lane >> 4, lo = lane & 3;
    const int64_t e = e0 + 16 * wave + (lane & 15);
    const bool valid = e < e1;
    const int64_t cs = E * G * N;
    // coefficients at a time point of the element row at `base` of a vector
    // with component stride `str`
    auto coeffs = [&](const double* src, int64_t rows, int64_t row, bool ok, const double (&gt)[G],
                      double (&x)[3][NQ]) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const __amdgpu_buffer_rsrc_t r = m64_rsrc(src + c * rows * G * N, (uint32_t)(8 * rows * G * N));
#pragma unroll
            for (int t = 0; t < NQ; ++t) x[c][t] = 0.0;
#pragma unroll
            for (int b = 0; b < G; ++b) {
                double v[NQ];
                m64_load<N>(r, ok ? (uint32_t)((row * G + b) * N * 8) : M64_OOB, hi, v);
#pragma unroll
                for (int t = 0; t < NQ; ++t) x[c][t] += gt[b] * v[t];
            }
        }
    };
    double J[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) J[i] = cJinv[(int64_t)cl * 9 + i];
    const double det = cdet[cl];
    double acc[G][NQ][3];
#pragma unroll
    for (int a = 0; a < G; ++a)
#pragma unroll
        for (int rg = 0; rg < NQ; ++rg)
#pragma unroll
            for (int c = 0; c < 3; ++c) acc[a][rg][c] = 0.0;
#pragma unroll 1
    for (int tp = 0; tp < qt; ++tp) {
        double gt[G];
#pragma unroll
        for (int b = 0; b < G; ++b) gt[b] = gq[tp * G + b];
        const double wt = tw[tp];
        double x[3][NQ];
        coeffs(vbar, E, e, valid, gt, x);
        double o[NQ][3];
#pragma unroll
        for (int rg = 0; rg < NQ; ++rg)
#pragma unroll
            for (int c = 0; c < 3; ++c) o[rg][c] = 0.0;
        // volume points: -F_cd = -v_c v_d pulled back by J^-T, tested with grad phi
#pragma unroll 1
        for (int q0 = 0; q0 < nqv; q0 += QC) {
            const int n = nqv - q0 < QC ? nqv - q0 : QC;
            __syncthreads();
            stage_points<N>(PHv + (int64_t)q0 * N, n, N, L);
            for (int t = tid; t < 3 * QC * NP; t += CT) {
                const int k = t % NP, q = t / NP % QC, d = t / (NP * QC);
                L[QC * NP + t] = q < n && k < N ? dPHv[((int64_t)(q0 + q) * N + k) * 3 + d] : 0.0;
            }
            if (tid < QC) Wq[tid] = tid < n ? wv[q0 + tid] : 0.0;
            __syncthreads();
#pragma unroll 1
            for (int g = 0; 4 * g < n; ++g) {
                double v[3];
                eval_points<N>(L, g, lo, hi, x, v);
                const double w = -wt * Wq[4 * g + hi] * det;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const double s = w * (J[d * 3] * v[0] + J[d * 3 + 1] * v[1] + J[d * 3 + 2] * v[2]);
                    const double f[3] = {s * v[0], s * v[1], s * v[2]};
                    test_points<N>(L + (1 + d) * QC * NP, g, lo, hi, f, o);
                }
            }
        }
        // faces: own trace against the neighbour's (or the boundary data)
#pragma unroll 1
        for (int f = 0; f < 4; ++f) {
            const int64_t k = valid ? nbr[4 * e + f] : -1;
            double xn[3][NQ];
            // (the elements of a class have the same boundary faces)
            if (nbr[4 * e0 + f] >= 0) coeffs(vbar, E, k, valid, gt, xn);
            else coeffs(vbc, F, valid ? tet_face[4 * e + f] : -1, valid, gt, xn);
            const double* nr = cnrm + (int64_t)cl * 12 + f * 3;
            const double n0 = nr[0], n1 = nr[1], n2 = nr[2];
#pragma unroll 1
            for (int q0 = 0; q0 < nqf; q0 += QC) {
                const int n = nqf - q0 < QC ? nqf - q0 : QC;
                const int64_t off = ((int64_t)cl * 4 + f) * nqf + q0;
                __syncthreads();
                stage_points<N>(PHf + off * N, n, N, L);
                stage_points<N>(PHn + off * N, n, N, L + QC * NP);
                if (tid < QC) Wq[tid] = tid < n ? FW[off + tid] : 0.0;
                __syncthreads();
#pragma unroll 1
                for (int g = 0; 4 * g < n; ++g) {
                    double vm[3], vp[3];
                    eval_points<N>(L, g, lo, hi, x, vm);
                    eval_points<N>(L + QC * NP, g, lo, hi, xn, vp);
                    const double unm = vm[0] * n0 + vm[1] * n1 + vm[2] * n2;
                    const double unp = vp[0] * n0 + vp[1] * n1 + vp[2] * n2;
                    const double am = vm[0] * vm[0] + vm[1] * vm[1] + vm[2] * vm[2];
                    const double ap = vp[0] * vp[0] + vp[1] * vp[1] + vp[2] * vp[2];
                    const double smax = 2.0 * sqrt(am > ap ? am : ap);
                    const double w = wt * Wq[4 * g + hi];
                    double fc[3];
#pragma unroll
                    for (int c = 0; c < 3; ++c)
                        fc[c] = w * (0.5 * (vp[c] * unp + vm[c] * unm) - 0.5 * smax * (vp[c] - vm[c]));
                    test_points<N>(L, g, lo, hi, fc, o);
                }
            }
        }
#pragma unroll
        for (int a = 0; a < G; ++a)
#pragma unroll
            for (int rg = 0; rg < NQ; ++rg)
#pragma unroll
                for (int c = 0; c < 3; ++c) acc[a][rg][c] += gt[a] * o[rg][c];
    }
    __syncthreads();
    const int64_t first = e0 + 16 * wave, left = e1 - first;
    if (left <= 0) return;
    const int count = (int)(left < 16 ? left : 16) * G * N;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        double* dst = ups + c * cs + first * G * N;
        m64_flush<N, G>(L + wave * 16 * G * N, lane, hi, count, [&](int rg, int a) { return dt * acc[a][rg][c]; },
                        [&](int i, m64_d2u v) { m64_put(dst, i, count, v); });
    }
}

template <int N, int G>
hipError_t launch_conv(const stdg_mesh* m, const double* vbar, const double* vbc, double* ups, hipStream_t s) {
    const PicardTables& t = m->pt;
    const PicardDevice& d = m->pd;
    hipLaunchKernelGGL((kc_convection<N, G>), dim3(m64_blocks(m->d.n_segs)), dim3(CT), 0, s, vbar, vbc, (const m64_i4*)m->d.segs,
                       m->d.nbr, d.tet_face, d.cJinv, d.cdet, d.cnrm, d.PHf, d.PHn, d.FW, d.PHv, d.dPHv, d.wv, d.tw,
                       d.gq, t.nqv, t.nqf, t.qt, m->cfg.dt, ups, m->E, (int64_t)m->faces.size(), (uint32_t)m->d.n_segs);
    return hipGetLastError();
}

}  // namespace

// groups that pay, the sums of all time nodes in registers (N G up to 80),
// and buffer offsets below 2 GiB
hipError_t conv_mfma(const stdg_mesh* m, const double* vbar, const double* vbc, double* ups, hipStream_t s) {
    if (!groups_pay(m, GroupKernel::CONVECTION) || 8 * (int64_t)m->faces.size() * m->Nst >= ((int64_t)1 << 31)) return hipErrorNotSupported;
#define STDG_CV(n, g) \
    if (m->N == n && m->G == g) return launch_conv<n, g>(m, vbar, vbc, ups, s);
    STDG_CV(4, 1) STDG_CV(4, 2) STDG_CV(4, 3) STDG_CV(4, 4) STDG_CV(4, 5)
    STDG_CV(10, 1) STDG_CV(10, 2) STDG_CV(10, 3) STDG_CV(10, 4) STDG_CV(10, 5)
    STDG_CV(20, 1) STDG_CV(20, 2) STDG_CV(20, 3) STDG_CV(20, 4) STDG_CV(35, 1) STDG_CV(35, 2)
#undef STDG_CV
    return hipErrorNotSupported;
}

}  // namespace stdg
