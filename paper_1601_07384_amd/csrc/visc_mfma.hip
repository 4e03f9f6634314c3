// Viscous operator (eq. A1_mod) and its block-Jacobi step on the FP64 matrix
// cores, for meshes whose groups of one geometry class fill:
//   y_i = D^-1 [ (MI (x) T) x_i + nu dt sum_k (SV_k (x) W) x_nb(k) ]   (PRE)
// or the bracket alone, all three velocity components at once, with the dot
// products BiCGStab needs of the result.
//
// One workgroup per group: the class's six N x N blocks (five couplings, mass)
// and, with PRE, its NG x NG inverse diagonal block are staged in LDS; a
// wavefront takes 16 elements with 3 G columns each (component, time node),
// so an operand read from LDS feeds 3 G matrix instructions.  The bracket's
// rows are the contraction operand of the D^-1 product in place (mfma64.hpp),
// so the intermediate vector is neither stored nor read.  What bounds it is
// the row traffic (x of five elements per element through the caches) beside
// 14 N^2 flops a column.  663,552 elements, p = 3, p_gamma = 0: 1,005 us for
// the operator, the block-Jacobi and the dot kernel with one thread per row,
// 317 us here (385 with the dot against a third vector); 196,608, p = 2,
// p_gamma = 1: 281 -> 97 (117) us; 24,576, p = 3, p_gamma = 2 (N G = 60, one
// wavefront per SIMD): 320 -> 78 (83); 3,072, p = 4, p_gamma = 1: 178 -> 57 (64).

#include "internal.hpp"
#include "kernels.hpp"
#include "mfma64.hpp"
#include "two_level.hpp"

namespace stdg {
namespace {

constexpr int VT = 256;     // threads: four wavefronts of 16 elements

// DOTS: 0 none, 1 the workgroup's share of w.y, 2 those of x.y and y.y
// (part[blk] and part[gridDim.x + blk])
template <int N, int G, bool PRE, int DOTS>
__global__ void __launch_bounds__(VT) k_visc_mfma(const double* __restrict__ SVt, const double* __restrict__ MIt,
                                                  const double* __restrict__ DV, const m64_i4* __restrict__ segs,
                                                  const int32_t* __restrict__ nbr, const double* __restrict__ Tm,
                                                  const double* __restrict__ W, double nu_dt, const double* x,
                                                  double* __restrict__ y, const double* w, double* __restrict__ part,
                                                  int64_t E, uint32_t n_segs, uint32_t xbytes) {
    constexpr int NQ = M64<N>::NQ, NP = M64<N>::NP, NC = 3 * G;
    __shared__ double A[6 * N * NP > 64 * G * N ? 6 * N * NP : 64 * G * N];
    __shared__ double Dl[PRE ? G * NP * G * NP : 1];
    __shared__ double red[VT / 64];
    const uint32_t group = m64_group(gridDim.x);
    double d0 = 0.0, d1 = 0.0;
    if (group < n_segs) {                               // uniform over the workgroup
        const m64_i4 sg = segs[group];
        const int c = sg.z;
        const int64_t e1 = (int64_t)sg.x + sg.y;
        m64_stage<N, VT>(SVt + (int64_t)c * 5 * N * N, A, 5);
        m64_stage<N, VT>(MIt + (int64_t)c * N * N, A + 5 * N * NP, 1);
        if (PRE) {
            // [b][column][a][row], zero where either is padding
            const double* D = DV + (int64_t)c * (N * G) * (N * G);
            for (int t = threadIdx.x; t < G * NP * G * NP; t += VT) {
                const int r = t % NP, a = t / NP % G, col = t / (NP * G) % NP, b = t / (NP * G * NP);
                Dl[t] = r < N && col < N ? D[(b * N + col) * (N * G) + a * N + r] : 0.0;
            }
        }
        __syncthreads();
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, hi = lane >> 4, lo = lane & 3;
        const int64_t e = (int64_t)sg.x + 16 * wave + (lane & 15);
        const bool valid = e < e1;
        int nb[5];
        nb[0] = valid ? (int)e : -1;
#pragma unroll
        for (int f = 0; f < 4; ++f) nb[f + 1] = valid ? nbr[4 * e + f] : -1;
        const int64_t cs = E * G * N;
        __amdgpu_buffer_rsrc_t rx[3];
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) rx[cc] = m64_rsrc(x + cc * cs, xbytes);
        double acc[NQ][NC];
#pragma unroll
        for (int rg = 0; rg < NQ; ++rg)
#pragma unroll
            for (int q = 0; q < NC; ++q) acc[rg][q] = 0.0;
        double wa[G];
#pragma unroll
        for (int a = 0; a < G; ++a) wa[a] = nu_dt * W[a];
        auto couple = [&](int k) {
            const uint32_t base = nb[k] >= 0 ? (uint32_t)nb[k] * (uint32_t)(G * N * 8) : M64_OOB;
            double b[NC][NQ];
#pragma unroll
            for (int cc = 0; cc < 3; ++cc)
#pragma unroll
                for (int a = 0; a < G; ++a)
                    m64_load<N>(rx[cc], base == M64_OOB ? M64_OOB : base + (uint32_t)(a * N * 8), hi, b[cc * G + a]);
            if (k == 0) {
                // the mass block against the time-mixed own columns first
                double bt[NC][NQ];
#pragma unroll
                for (int cc = 0; cc < 3; ++cc)
#pragma unroll
                    for (int a = 0; a < G; ++a)
#pragma unroll
                        for (int t = 0; t < NQ; ++t) {
                            double s = 0.0;
#pragma unroll
                            for (int bb = 0; bb < G; ++bb) s += Tm[a * G + bb] * b[cc * G + bb][t];
                            bt[cc * G + a][t] = s;
                        }
                m64_block<N, NC>(A + 5 * N * NP, bt, lo, hi, acc);
            }
#pragma unroll
            for (int q = 0; q < NC; ++q)
#pragma unroll
                for (int t = 0; t < NQ; ++t) b[q][t] *= wa[q % G];
            m64_block<N, NC>(A + k * N * NP, b, lo, hi, acc);
        };
        couple(0);
        couple(1);
        couple(2);
        couple(3);
        couple(4);
        double z[NQ][NC];
        if constexpr (PRE) {
#pragma unroll
            for (int rg = 0; rg < NQ; ++rg)
#pragma unroll
                for (int q = 0; q < NC; ++q) z[rg][q] = 0.0;
#pragma unroll
            for (int b = 0; b < G; ++b)
#pragma unroll
                for (int t = 0; t < NQ; ++t) {
                    const double* col = Dl + ((b * NP + 4 * t + hi) * G) * NP + lo;
#pragma unroll
                    for (int a = 0; a < G; ++a)
#pragma unroll
                        for (int rg = 0; rg < NQ; ++rg) {
                            const double av = col[a * NP + 4 * rg];
#pragma unroll
                            for (int cc = 0; cc < 3; ++cc)
                                z[rg][cc * G + a] = __builtin_amdgcn_mfma_f64_4x4x4f64(av, acc[t][cc * G + b],
                                                                                      z[rg][cc * G + a], 0, 0, 0);
                        }
                }
        }
        // out through the blocks' LDS, the dots beside the stores
        __syncthreads();
        const int64_t first = (int64_t)sg.x + 16 * wave, left = e1 - first;
        const int count = left <= 0 ? 0 : (int)(left < 16 ? left : 16) * G * N;
        if (count > 0)
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                const int64_t at = cc * cs + first * G * N;
                m64_flush<N, G>(
                    A + wave * 16 * G * N, lane, hi, count,
                    [&](int rg, int a) { return PRE ? z[rg][cc * G + a] : acc[rg][cc * G + a]; },
                    [&](int i, m64_d2u v) {
                        m64_put(y + at, i, count, v);
                        if (DOTS >= 1) {
                            const double* from = (DOTS == 1 ? w : x) + at + i;
                            m64_d2u u;
                            if ((N * G) % 2 == 0 || i + 1 < count) {
                                u = *reinterpret_cast<const m64_d2u*>(from);
                            } else {                    // the last of an odd number of values
                                u.x = *from;
                                u.y = 0.0;
                                v.y = 0.0;
                            }
                            d0 += u.x * v.x + u.y * v.y;
                            if (DOTS == 2) d1 += v.x * v.x + v.y * v.y;
                        }
                    });
            }
    }
    if (DOTS >= 1) {
        const double s = tl_reduce<VT>(d0, red);
        if (threadIdx.x == 0) part[blockIdx.x] = s;
    }
    if (DOTS == 2) {
        const double s = tl_reduce<VT>(d1, red);
        if (threadIdx.x == 0) part[gridDim.x + blockIdx.x] = s;
    }
}

// y = D^-1 x alone (the preconditioned right-hand side): D from LDS against
// the rows as they are loaded.  Bound: HBM; 663,552 elements, p = 3, a thread
// per row before: 389 us -> 100.
template <int N, int G>
__global__ void __launch_bounds__(VT) k_prec_mfma(const double* __restrict__ DV, const m64_i4* __restrict__ segs,
                                                  const double* __restrict__ x, double* __restrict__ y, int64_t E,
                                                  uint32_t n_segs, uint32_t xbytes) {
    constexpr int NQ = M64<N>::NQ, NP = M64<N>::NP;
    constexpr int ND = G * NP * G * NP;
    __shared__ double Dl[ND > 64 * G * N ? ND : 64 * G * N];
    const uint32_t group = m64_group(gridDim.x);
    if (group >= n_segs) return;
    const m64_i4 sg = segs[group];
    const double* D = DV + (int64_t)sg.z * (N * G) * (N * G);
    for (int t = threadIdx.x; t < ND; t += VT) {
        const int r = t % NP, a = t / NP % G, col = t / (NP * G) % NP, b = t / (NP * G * NP);
        Dl[t] = r < N && col < N ? D[(b * N + col) * (N * G) + a * N + r] : 0.0;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, hi = lane >> 4, lo = lane & 3;
    const int64_t e = (int64_t)sg.x + 16 * wave + (lane & 15), e1 = (int64_t)sg.x + sg.y;
    const int64_t cs = E * G * N;
    double z[3][NQ][G];
    double b[3][G][NQ];
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
        const __amdgpu_buffer_rsrc_t rx = m64_rsrc(x + cc * cs, xbytes);
#pragma unroll
        for (int a = 0; a < G; ++a) {
            m64_load<N>(rx, e < e1 ? (uint32_t)((e * G + a) * N * 8) : M64_OOB, hi, b[cc][a]);
#pragma unroll
            for (int rg = 0; rg < NQ; ++rg) z[cc][rg][a] = 0.0;
        }
    }
    __syncthreads();
#pragma unroll
    for (int bb = 0; bb < G; ++bb)
#pragma unroll
        for (int t = 0; t < NQ; ++t) {
            const double* col = Dl + ((bb * NP + m64_col<N>(t, hi)) * G) * NP + lo;
#pragma unroll
            for (int a = 0; a < G; ++a)
#pragma unroll
                for (int rg = 0; rg < NQ; ++rg) {
                    const double av = col[a * NP + 4 * rg];
#pragma unroll
                    for (int cc = 0; cc < 3; ++cc)
                        z[cc][rg][a] = __builtin_amdgcn_mfma_f64_4x4x4f64(av, b[cc][bb][t], z[cc][rg][a], 0, 0, 0);
                }
        }
    __syncthreads();
    const int64_t first = (int64_t)sg.x + 16 * wave, left = e1 - first;
    if (left <= 0) return;
    const int count = (int)(left < 16 ? left : 16) * G * N;
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
        double* dst = y + cc * cs + first * G * N;
        m64_flush<N, G>(Dl + wave * 16 * G * N, lane, hi, count, [&](int rg, int a) { return z[cc][rg][a]; },
                        [&](int i, m64_d2u v) { m64_put(dst, i, count, v); });
    }
}

template <int N, int G, bool PRE, int DOTS>
hipError_t launch_visc(const stdg_mesh* m, const double* x, double* y, const double* w, double* part, hipStream_t s) {
    const PicardDevice& d = m->pd;
    hipLaunchKernelGGL((k_visc_mfma<N, G, PRE, DOTS>), dim3((unsigned)visc_mfma_blocks(m)), dim3(VT), 0, s, d.SVt, d.MIt,
                       d.DV, (const m64_i4*)m->d.segs, m->d.nbr, d.Tm, d.W, m->cfg.nu * m->cfg.dt, x, y, w, part, m->E,
                       (uint32_t)m->d.n_segs, (uint32_t)(8 * m->E * m->Nst));
    return hipGetLastError();
}

}  // namespace

int64_t visc_mfma_blocks(const stdg_mesh* m) { return m64_blocks(m->d.n_segs); }

// N G up to 80 (the inverse diagonal block in LDS), groups that pay, and
// offsets within a component below 2 GiB
bool visc_mfma_supported(const stdg_mesh* m) {
    return (m->N == 4 || m->N == 10 || m->N == 20 || m->N == 35) && m->G <= 5 && m->Nst <= 80 &&
           8 * m->E * m->Nst < ((int64_t)1 << 31) && groups_pay(m, GroupKernel::VISCOUS);
}

#define STDG_VISC_NG                                                              \
    STDG_NG(4, 1) STDG_NG(4, 2) STDG_NG(4, 3) STDG_NG(4, 4) STDG_NG(4, 5)         \
    STDG_NG(10, 1) STDG_NG(10, 2) STDG_NG(10, 3) STDG_NG(10, 4) STDG_NG(10, 5)    \
    STDG_NG(20, 1) STDG_NG(20, 2) STDG_NG(20, 3) STDG_NG(20, 4) STDG_NG(35, 1) STDG_NG(35, 2)

hipError_t prec_mfma(const stdg_mesh* m, const double* x, double* y, hipStream_t s) {
#define STDG_NG(n, g)                                                                                              \
    if (m->N == n && m->G == g) {                                                                                  \
        hipLaunchKernelGGL((k_prec_mfma<n, g>), dim3((unsigned)visc_mfma_blocks(m)), dim3(VT), 0, s, m->pd.DV,      \
                           (const m64_i4*)m->d.segs, x, y, m->E, (uint32_t)m->d.n_segs, (uint32_t)(8 * m->E * m->Nst)); \
        return hipGetLastError();                                                                                  \
    }
    STDG_VISC_NG
#undef STDG_NG
    return hipErrorInvalidValue;
}

hipError_t visc_mfma(const stdg_mesh* m, bool pre, int dots, const double* x, double* y, const double* w, double* part,
                     hipStream_t s) {
#define STDG_NG(n, g)                                                                  \
    if (m->N == n && m->G == g) {                                                      \
        if (!pre) return launch_visc<n, g, false, 0>(m, x, y, w, part, s);                  \
        if (dots == 0) return launch_visc<n, g, true, 0>(m, x, y, w, part, s);              \
        return dots == 1 ? launch_visc<n, g, true, 1>(m, x, y, w, part, s)                  \
                         : launch_visc<n, g, true, 2>(m, x, y, w, part, s);                 \
    }
    STDG_VISC_NG
#undef STDG_NG
    return hipErrorInvalidValue;
}

}  // namespace stdg
