// Matrix-free pressure Schur operator y = S x (eq. CS_19, negated; Sec. 2.4).
//
// S = dt^2 S^sp (x) C: for element i with neighbours k_f across its local
// faces f,
//   Y_i = sum_{k in {i, k_0..k_3}} B_{c(i),k} (X_k C^T)
// where X_k is the N x G coefficient matrix of element k ([G][N] in memory),
// B_{c,0..4} the class-deduplicated dt^2-scaled spatial blocks and C the G x G
// time factor.
//
// FP64 (p <= 4, p_gamma <= 4): groups of up to 64 elements of one class on the
// FP64 matrix cores, meshes without such groups with a thread per (coupling,
// row) (schur_apply_list); meshes whose elements carry their own blocks stream them
// (cg_elem.hip), and at p = 1 large meshes take an element per lane
// (schur_apply_run).  FP32 vectors and other degrees: one thread per (element,
// time node), the neighbour column x'_m = sum_b C_ab x_k[b][m] formed on the
// fly, N outputs in registers; a wavefront of one class reads its blocks
// through scalar loads (stored transposed, BT[c][k][m][r], so that a column is
// contiguous), others per lane.
#include "internal.hpp"
#include "kernels.hpp"
#include "mfma64.hpp"
#include "two_level.hpp"

namespace stdg {

template <int N, int G, typename T>
__device__ __forceinline__ void accumulate_block(const T* __restrict__ Bk, const T* __restrict__ xt,
                                                 const T (&Ca)[G], T (&acc)[N]) {
#pragma unroll
    for (int m = 0; m < N; ++m) {
        T xp = T(0);
#pragma unroll
        for (int b = 0; b < G; ++b) xp += Ca[b] * xt[b * N + m];
        const T* col = Bk + m * N;
#pragma unroll
        for (int r = 0; r < N; ++r) acc[r] += col[r] * xp;
    }
}

template <int N, int G, typename T>
__global__ void __launch_bounds__(256) schur_apply_tn(
    const T* __restrict__ BT, const int32_t* __restrict__ cls, const int32_t* __restrict__ nbr,
    const T* __restrict__ C, const T* __restrict__ x, T* __restrict__ y, int64_t E) {
    const int a = (int)(blockIdx.x % G);
    const int64_t i = (int64_t)(blockIdx.x / G) * 256 + threadIdx.x;
    const bool valid = i < E;
    const int64_t ii = valid ? i : E - 1;          // inactive lanes mirror a valid element
    const int c = cls[ii];
    const int c0 = __builtin_amdgcn_readfirstlane(c);
    const bool uniform = __all(c == c0);
    T Ca[G];
#pragma unroll
    for (int b = 0; b < G; ++b) Ca[b] = C[a * G + b];
    T acc[N];
#pragma unroll
    for (int r = 0; r < N; ++r) acc[r] = T(0);
    int nb[5];
    nb[0] = (int)ii;
#pragma unroll
    for (int f = 0; f < 4; ++f) nb[f + 1] = nbr[4 * ii + f];
    if (uniform) {
        const T* Bc = BT + (int64_t)c0 * 5 * N * N;
        for (int k = 0; k < 5; ++k) {
            const int t = nb[k];
            // a uniform class has the same boundary faces on every lane
            if (__builtin_amdgcn_readfirstlane(t) < 0) continue;
            accumulate_block<N, G, T>(Bc + k * N * N, x + (int64_t)t * G * N, Ca, acc);
        }
    } else {
        const T* Bc = BT + (int64_t)c * 5 * N * N;
        for (int k = 0; k < 5; ++k) {
            const int t = nb[k];
            if (t < 0) continue;
            accumulate_block<N, G, T>(Bc + k * N * N, x + (int64_t)t * G * N, Ca, acc);
        }
    }
    if (valid) {
        T* yi = y + (i * G + a) * N;
#pragma unroll
        for (int r = 0; r < N; ++r) yi[r] = acc[r];
    }
}

// Any (N, G): one thread per (element, spatial row), all time nodes.
template <int G, typename T>
__global__ void __launch_bounds__(256) schur_apply_rows(
    const T* __restrict__ BT, const int32_t* __restrict__ cls, const int32_t* __restrict__ nbr,
    const T* __restrict__ C, const T* __restrict__ x, T* __restrict__ y, int64_t E, int N) {
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = gid / N;
    const int n = (int)(gid - i * N);
    if (i >= E) return;
    const T* Bc = BT + (int64_t)cls[i] * 5 * N * N;
    T acc[G];
#pragma unroll
    for (int b = 0; b < G; ++b) acc[b] = T(0);
    for (int k = 0; k < 5; ++k) {
        const int64_t t = (k == 0) ? i : (int64_t)nbr[4 * i + (k - 1)];
        if (t < 0) continue;
        const T* xt = x + t * G * N;
        for (int m = 0; m < N; ++m) {
            const T bv = Bc[((int64_t)k * N + m) * N + n];
#pragma unroll
            for (int b = 0; b < G; ++b) acc[b] += bv * xt[b * N + m];
        }
    }
    T* yi = y + i * G * N;
#pragma unroll
    for (int a = 0; a < G; ++a) {
        T s = T(0);
#pragma unroll
        for (int b = 0; b < G; ++b) s += C[a * G + b] * acc[b];
        yi[a * N + n] = s;
    }
}

// FP64 y = S x.  A workgroup takes a group of up to 64 elements of one class:
// the class's five blocks staged in LDS, a wavefront on 16 CW elements with G
// columns each (mfma64.hpp: rows read 16 bytes a lane, an operand from LDS
// serving CW G matrix instructions, results in place for the G x G time factor
// and written in whole lines).  Bound: HBM at p <= 2, the matrix cores and the
// operand reads at p = 3, 4, the launch (7.8 us in a loop from the host)
// below 10^4 elements.  MI355X, kernels per entry on the vector units before
// -> this one, us: 663,552 elements, p = 3, G = 1: 92.5 -> 77.3 in a row of 50
// launches (2.7 TB/s of x and y; 105 -> 81 one by one); 196,608, p = 2: G = 1
// 19.9 -> 14.8, G = 2 29.7 -> 24.5; 82,944, p = 3, G = 2: 33.0 -> 24.9; 48,000,
// p = 2, G = 3: 41 -> 11.5; with walls 10,368, p = 4, G = 5: 50 -> 34 and 1,296,
// p = 3: 35 -> 7.7; no two neighbours of one class (schur_apply_list), 82,944,
// p = 3, G = 2: 391 -> 198.  The sums' rounding is half as large.
// With DOT the workgroup's share of x.y goes to part[blockIdx.x].
// EN: elements whose rows pass through LDS at a time.  At p = 4 with four and
// five time nodes the rows of 16 take more LDS than the blocks (72 and 90 KB
// against 50), which leaves two and one workgroups per CU instead of three and
// two; m64_narrow() says where 8 pay.
template <int N, int G, int CW, bool DOT, int EN>
__global__ void __launch_bounds__(256 / CW) schur_apply_m64(const double* __restrict__ BT,
                                                           const m64_i4* __restrict__ segs,
                                                           const int32_t* __restrict__ nbr,
                                                           const double* __restrict__ C, const double* x,
                                                           double* __restrict__ y, int64_t E, uint32_t n_segs,
                                                           double* __restrict__ part) {
    constexpr int NT = 256 / CW, NQ = M64<N>::NQ, NP = M64<N>::NP, NC = CW * G;
    constexpr int OUT = 4 * EN * G * N;
    constexpr int LD = 5 * N * NP > OUT ? 5 * N * NP : OUT;
    __shared__ double A[LD];
    __shared__ double red[NT / 64];
    double d = 0.0;
    const uint32_t group = m64_group(gridDim.x);
    if (group < n_segs) {
        const m64_i4 sg = segs[group];
        const int c = sg.z;
        const int64_t e0 = sg.x, e1 = e0 + sg.y;
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, hi = lane >> 4, lo = lane & 3;
        int nb[5][CW];
#pragma unroll
        for (int q = 0; q < CW; ++q) {
            const int64_t e = e0 + 16 * (CW * w + q) + (lane & 15);
            const bool valid = e < e1;
            nb[0][q] = valid ? (int)e : -1;
#pragma unroll
            for (int f = 0; f < 4; ++f) nb[f + 1][q] = valid ? nbr[4 * e + f] : -1;
        }
        m64_stage<N, NT>(BT + (int64_t)c * 5 * N * N, A, 5);
        const __amdgpu_buffer_rsrc_t rx = m64_rsrc(x, (uint32_t)(8 * E * G * N));
        double acc[NQ][NC];
#pragma unroll
        for (int rg = 0; rg < NQ; ++rg)
#pragma unroll
            for (int q = 0; q < NC; ++q) acc[rg][q] = 0.0;
        __syncthreads();
        auto couple = [&](int k) {
            double b[NC][NQ];
#pragma unroll
            for (int q = 0; q < CW; ++q) {
                const int s = k == 0 ? nb[0][q] : (k == 1 ? nb[1][q] : (k == 2 ? nb[2][q] : (k == 3 ? nb[3][q] : nb[4][q])));
#pragma unroll
                for (int a = 0; a < G; ++a)
                    m64_load<N>(rx, s >= 0 ? (uint32_t)((s * G + a) * N) * 8u : M64_OOB, hi, b[q * G + a]);
            }
            m64_block<N, NC>(A + k * N * NP, b, lo, hi, acc);
        };
        // large blocks (p = 4) one coupling at a time, so that the rows of
        // the next are not all held at once
        if constexpr (NQ * NC > 16) {
#pragma unroll 1
            for (int k = 0; k < 5; ++k) couple(k);
        } else {
#pragma unroll
            for (int k = 0; k < 5; ++k) couple(k);
        }
        double Cm[G][G];
#pragma unroll
        for (int a = 0; a < G; ++a)
#pragma unroll
            for (int b = 0; b < G; ++b) Cm[a][b] = C[a * G + b];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < CW; ++q) {
            const int64_t first = e0 + 16 * (CW * w + q), left = e1 - first;
            if (left <= 0) continue;
            const int count = (int)(left < 16 ? left : 16) * G * N;
            const int64_t at = first * G * N;
            m64_flush<N, G, EN>(
                A + w * EN * G * N, lane, hi, count,
                [&](int rg, int a) {
                    double s = 0.0;
#pragma unroll
                    for (int b = 0; b < G; ++b) s += Cm[a][b] * acc[rg][q * G + b];
                    return s;
                },
                [&](int i, m64_d2u v) {
                    m64_put(y + at, i, count, v);
                    if (DOT) {
                        d += x[at + i] * v.x;
                        if (i + 1 < count) d += x[at + i + 1] * v.y;
                    }
                });
        }
    }
    if (DOT) {
        const double s = tl_reduce<NT>(d, red);
        if (threadIdx.x == 0) part[blockIdx.x] = s;
    }
}

// y = S x at p = 1 with one or two time nodes on large meshes of whole runs (64
// elements of one class): a wavefront per run, lane l = element 64 run + l.  For
// each coupling the wavefront moves the 64 rows it needs (contiguous in
// memory) into its LDS with 16-byte loads that walk them in order, then every
// lane reads its own row back and applies the class block column by column
// through scalar loads.  The G x G time factor is applied to the result, which
// leaves through LDS the same way.  Row pieces sit at an odd stride of 16-byte
// units, so that the 16 lanes of each pass of a 16-byte read hit distinct banks.
// Bound: HBM.  A row is 4 doubles here, so schur_apply_m64's 64 elements are one
// 16-byte load per lane and coupling beside staging and two barriers.  us, groups /
// this: G = 1 48,000 elements 4.5 / 7.5, 384,000 15.1 / 9.0, 663,552 23.7 / 14.9; G = 2
// 48,000 5.9 / 9.2, 131,712 10.8 / 8.2, 663,552 40.2 / 28.1; G = 3, p = 2 the groups
// at every size (p = 2, 663,552 39.5 / 47.4).
template <int N, int G>
__global__ void __launch_bounds__(64) schur_apply_run(const double* __restrict__ BT, const int32_t* __restrict__ cls,
                                                      const int32_t* __restrict__ nbr, const double* __restrict__ C,
                                                      const double* __restrict__ x, double* __restrict__ y,
                                                      int64_t E, uint32_t n_runs) {
    typedef double d2 __attribute__((ext_vector_type(2)));
    constexpr int R = N * G, NP = R / 2, STR = NP % 2 == 0 ? NP + 1 : NP;
    static_assert(R % 2 == 0, "rows of whole 16-byte pieces");
    __shared__ d2 L[64 * STR];
    const int lane = threadIdx.x;
    const uint32_t run = m64_group(gridDim.x);
    if (run >= n_runs) return;
    const int64_t e0 = (int64_t)run * 64, e = e0 + lane;
    const bool valid = e < E;
    const int c = __builtin_amdgcn_readfirstlane(cls[e0]);
    int nbk[4] = {-1, -1, -1, -1};
    if (valid) {
#pragma unroll
        for (int f = 0; f < 4; ++f) nbk[f] = nbr[4 * e + f];
    }
    double z[G][N];
#pragma unroll
    for (int b = 0; b < G; ++b)
#pragma unroll
        for (int r = 0; r < N; ++r) z[b][r] = 0.0;
    for (int k = 0; k < 5; ++k) {
        const int src = k == 0 ? (valid ? (int)e : -1) : nbk[k - 1];
        if (__builtin_amdgcn_readfirstlane(__ballot(src >= 0) != 0 ? 1 : 0) == 0) continue;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int pc = i * 64 + lane, row = pc / NP, piece = pc - row * NP;
            const int s = __shfl(src, row, 64);
            const m64_d2u v = s >= 0 ? reinterpret_cast<const m64_d2u*>(x + (int64_t)s * R)[piece] : m64_d2u{0.0, 0.0};
            L[row * STR + piece] = d2{v.x, v.y};
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        double xr[R];
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const d2 t = L[lane * STR + j];
            xr[2 * j] = t.x;
            xr[2 * j + 1] = t.y;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const double* Bk = BT + ((int64_t)c * 5 + k) * N * N;
#pragma unroll
        for (int m = 0; m < N; ++m) {
            const double* col = Bk + m * N;
#pragma unroll
            for (int r = 0; r < N; ++r) {
                const double a = col[r];
#pragma unroll
                for (int b = 0; b < G; ++b) z[b][r] += a * xr[b * N + m];
            }
        }
    }
    double yr[R];
#pragma unroll
    for (int a = 0; a < G; ++a)
#pragma unroll
        for (int r = 0; r < N; ++r) {
            double s = 0.0;
#pragma unroll
            for (int b = 0; b < G; ++b) s += C[a * G + b] * z[b][r];
            yr[a * N + r] = s;
        }
#pragma unroll
    for (int j = 0; j < NP; ++j) L[lane * STR + j] = d2{yr[2 * j], yr[2 * j + 1]};
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int pc = i * 64 + lane, row = pc / NP, piece = pc - row * NP;
        const d2 v = L[row * STR + piece];
        if (e0 + row < E) reinterpret_cast<m64_d2u*>(y + (e0 + row) * R)[piece] = m64_d2u{v.x, v.y};
    }
}

// y = S x element by element: a thread per coupling and row, EPB elements per
// workgroup of LT threads, the five couplings in parallel and summed through
// LDS.  Bound: the blocks, 5 N^2 values per element through L2.
// With DOT (FP64) the workgroup's share of x.y goes to part[blockIdx.x].
constexpr int LT = 256;
template <int N> constexpr int list_epb() { return LT / (5 * N) > 0 ? LT / (5 * N) : 1; }
template <int N, int G, typename T, bool DOT>
__global__ void __launch_bounds__(LT) schur_apply_list(const T* __restrict__ BT, const int32_t* __restrict__ cls,
                                                       const int32_t* __restrict__ nbr, const T* __restrict__ C,
                                                       const T* x, T* __restrict__ y, int64_t E,
                                                       double* __restrict__ part) {
    constexpr int EPB = list_epb<N>();
    static_assert(5 * N <= LT, "a thread per coupling and row");
    __shared__ T A[EPB * 5 * G * N];
    __shared__ double red[LT / 64];
    double d = 0.0;
    const int t = threadIdx.x, el = t / (5 * N), kr = t - el * (5 * N), k = kr / N, r = kr - k * N;
    const int64_t i = (int64_t)blockIdx.x * EPB + el;
    const bool on = el < EPB && i < E;
    const int64_t s = !on ? -1 : (k == 0 ? i : (int64_t)nbr[4 * i + (k - 1)]);
    T acc[G];
#pragma unroll
    for (int b = 0; b < G; ++b) acc[b] = T(0);
    if (s >= 0) {
        const T* Bk = BT + ((int64_t)cls[i] * 5 + k) * N * N + r;
        const T* xt = x + s * G * N;
#pragma unroll 10
        for (int mm = 0; mm < N; ++mm) {
            const T bv = Bk[mm * N];
#pragma unroll
            for (int b = 0; b < G; ++b) acc[b] += bv * xt[b * N + mm];
        }
    }
    if (el < EPB)
#pragma unroll
        for (int b = 0; b < G; ++b) A[((el * 5 + k) * G + b) * N + r] = acc[b];
    __syncthreads();
    if (on && k == 0) {
        T z[G];
#pragma unroll
        for (int b = 0; b < G; ++b) {
            z[b] = T(0);
#pragma unroll
            for (int kk = 0; kk < 5; ++kk) z[b] += A[((el * 5 + kk) * G + b) * N + r];
        }
#pragma unroll
        for (int a = 0; a < G; ++a) {
            T v = T(0);
#pragma unroll
            for (int b = 0; b < G; ++b) v += C[a * G + b] * z[b];
            y[(i * G + a) * N + r] = v;
            if (DOT) d += (double)x[(i * G + a) * N + r] * (double)v;
        }
    }
    if (DOT) {
        const double p = tl_reduce<LT>(d, red);
        if (t == 0) part[blockIdx.x] = p;
    }
}

// Workgroups of the FP64 operator: groups where they fill (segs_fill), small
// meshes too (us, groups / one by one: 2,058 elements, p = 3, G = 2 6.5 / 8.5;
// 48,000, p = 1, G = 2 5.5 / 8.0; 3,072, p = 4, G = 2 14.1 / 25.0; equal at 750 and
// 1,296, p = 3).
template <int N> static unsigned apply64_blocks(const stdg_mesh* m) {
    return segs_fill(m) ? m64_blocks(m->d.n_segs) : (unsigned)((m->E + list_epb<N>() - 1) / list_epb<N>());
}

// Rows leave schur_apply_m64 eight elements at a time (p = 4, G = 4, 5): where
// there are more groups than CUs.  Up to one group per CU the second pass
// through LDS is all that the smaller slices bring; at G = 5 three rounds of one
// workgroup per CU are faster than one and a half of two.  16 / 8 (the kernel
// before both, which staged x), us: G = 4 192 groups 29.4 / 33.0 (30.5), 384 46.5 /
// 46.2 (48.0), 528 70.1 / 71.2 (70.8), 720 84.7 / 72.7 (78.5), 1,248 122 / 111 (128);
// G = 5 192 groups 34.5 / 34.9 (35.0), 264 60.5 / 52.6 (57.9), 504 69.8 / 59.9
// (67.2), 576 93.9 / 84.1 (88.0), 624 94.7 / 97.5 (88.1), 768 101 / 104 (94), 792 126 /
// 105 (115), 1,536 200 / 163 (175).  G = 3 no difference.
template <int N, int G> static bool m64_narrow(int64_t groups) {
    constexpr int CUS = 256;
    if (N != 35 || G < 4 || groups <= CUS) return false;
    return G < 5 || groups <= 600 || groups > 3 * CUS;
}

template <int N, int G, int CW, bool DOT>
static hipError_t launch_m64(const stdg_mesh* m, const double* C, const double* x, double* y, double* part,
                             hipStream_t s) {
    constexpr int NARROW = N == 35 && G >= 4 ? 8 : 16;
    const dim3 grid(apply64_blocks<N>(m));
    if (segs_fill(m)) {
        const auto kernel = m64_narrow<N, G>(m->d.n_segs) ? schur_apply_m64<N, G, CW, DOT, NARROW>
                                                          : schur_apply_m64<N, G, CW, DOT, 16>;
        hipLaunchKernelGGL(kernel, grid, dim3(256 / CW), 0, s, m->d.blocks, (const m64_i4*)m->d.segs, m->d.nbr, C, x,
                           y, m->E, (uint32_t)m->d.n_segs, part);
    } else
        hipLaunchKernelGGL((schur_apply_list<N, G, double, DOT>), grid, dim3(LT), 0, s, m->d.blocks, m->d.cls,
                           m->d.nbr, C, x, y, m->E, part);
    return hipGetLastError();
}

// p = 1, one or two time nodes, 100,000 elements and more in whole runs
static bool run64(const stdg_mesh* m) {
    return m->N == 4 && m->G <= 2 && m->E >= 100000 && m->d.n_segs == (m->E + 63) / 64;
}

template <int N, int G>
static hipError_t launch_run(const stdg_mesh* m, const double* C, const double* x, double* y, hipStream_t s) {
    const uint32_t runs = (uint32_t)m->d.n_segs;
    hipLaunchKernelGGL((schur_apply_run<N, G>), dim3(m64_blocks(runs)), dim3(64), 0, s, m->d.blocks, m->d.cls,
                       m->d.nbr, C, x, y, m->E, runs);
    return hipGetLastError();
}

template <int N, int G, typename T>
static hipError_t launch_tn(const stdg_mesh* m, const T* BT, const T* C, const T* x, T* y, hipStream_t s) {
    const int64_t blocks = (m->E + 255) / 256 * G;
    hipLaunchKernelGGL((schur_apply_tn<N, G, T>), dim3((unsigned)blocks), dim3(256), 0, s, BT,
                       m->d.cls, m->d.nbr, C, x, y, m->E);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_rows(const stdg_mesh* m, const T* BT, const T* C, const T* x, T* y,
                              hipStream_t s) {
    const int64_t work = m->E * m->N;
    const int threads = 256;
    const int64_t blocks = (work + threads - 1) / threads;
    switch (m->G) {
#define STDG_G(g)                                                                              \
    case g:                                                                                    \
        hipLaunchKernelGGL((schur_apply_rows<g, T>), dim3(blocks), dim3(threads), 0, s, BT,   \
                           m->d.cls, m->d.nbr, C, x, y, m->E, m->N);                          \
        break;
        STDG_G(1) STDG_G(2) STDG_G(3) STDG_G(4) STDG_G(5) STDG_G(6) STDG_G(7)
#undef STDG_G
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// column groups per wavefront: two where an element has one column
template <int N, int G> constexpr int m64_cw() { return N == 20 && G == 1 ? 2 : 1; }

static bool m64_supported(const stdg_mesh* m) {
    return (m->N == 4 || m->N == 10 || m->N == 20 || m->N == 35) && m->G <= 5 &&
           8 * m->E * m->G * m->N <= (int64_t)M64_OOB;
}

#define STDG_ALL_NG                                                       \
    STDG_NG(4, 1) STDG_NG(4, 2) STDG_NG(4, 3) STDG_NG(4, 4) STDG_NG(4, 5) \
    STDG_NG(10, 1) STDG_NG(10, 2) STDG_NG(10, 3) STDG_NG(10, 4) STDG_NG(10, 5) \
    STDG_NG(20, 1) STDG_NG(20, 2) STDG_NG(20, 3) STDG_NG(20, 4) STDG_NG(20, 5) \
    STDG_NG(35, 1) STDG_NG(35, 2) STDG_NG(35, 3) STDG_NG(35, 4) STDG_NG(35, 5)

static hipError_t apply_m64(const stdg_mesh* m, const double* C, const double* x, double* y, double* part,
                            hipStream_t s) {
#define STDG_NG(n, g) \
    if (m->N == n && m->G == g)                                                       \
        return part ? launch_m64<n, g, m64_cw<n, g>(), true>(m, C, x, y, part, s)     \
                    : launch_m64<n, g, m64_cw<n, g>(), false>(m, C, x, y, part, s);
    STDG_ALL_NG
#undef STDG_NG
    return hipErrorInvalidValue;
}

// FP32 by schur_apply_list: the thread of schur_apply_tn runs through 5 N^2
// block values in series, whose latency alone is 15 us at p = 3 and 32 (one
// class per wavefront) to 115 us (several) at p = 4; the list grows with the
// elements.  us, thread per element / list: p = 3 1,296 elements with walls,
// G = 2 21.2 / 8.7, 6,000 15.0 / 8.2, 16,464 17.8 / 15.6, 82,944 16.6 / 70; p = 4
// with walls 750 115 / 9.4, 10,368 112 / 28.6, periodic 3,072 32.3 / 10.3; p = 2
// 16,464, G = 2 8.0 / 9.0.
static bool list32(const stdg_mesh* m) { return m->N >= 20 && m->E <= 12000; }

template <typename T>
static hipError_t launch_apply(const stdg_mesh* m, const T* BT, const T* C, const T* x, T* y,
                               hipStream_t s) {
    if constexpr (sizeof(T) == 8) {
        // meshes whose elements carry their own blocks: the per-element FP64 tables
        if (elem_apply64_supported(m)) return elem_apply_f64(m, C, x, y, s);
        if (run64(m)) return m->G == 1 ? launch_run<4, 1>(m, C, x, y, s) : launch_run<4, 2>(m, C, x, y, s);
        if (m64_supported(m)) return apply_m64(m, C, x, y, nullptr, s);
    } else if (list32(m)) {
#define STDG_NG(n, g)                                                                                       \
    if constexpr (n >= 20) if (m->N == n && m->G == g) {                                                    \
        hipLaunchKernelGGL((schur_apply_list<n, g, float, false>),                                          \
                           dim3((unsigned)((m->E + list_epb<n>() - 1) / list_epb<n>())), dim3(LT), 0, s, BT, \
                           m->d.cls, m->d.nbr, C, x, y, m->E, (double*)nullptr);                            \
        return hipGetLastError();                                                                           \
    }
        STDG_ALL_NG
#undef STDG_NG
    }
#define STDG_NG(n, g) \
    if (m->N == n && m->G == g) return launch_tn<n, g, T>(m, BT, C, x, y, s);
    STDG_ALL_NG
#undef STDG_NG
    return launch_rows<T>(m, BT, C, x, y, s);
}

// workgroups of launch_apply_dot_f64 (0: no such kernel for this mesh)
int64_t apply_dot_blocks(const stdg_mesh* m) {
    if (elem_apply64_supported(m) || !m64_supported(m)) return 0;
#define STDG_NG(n, g) \
    if (m->N == n && m->G == g) return apply64_blocks<n>(m);
    STDG_ALL_NG
#undef STDG_NG
    return 0;
}

// y = (B (x) C) x and the workgroups' shares of x.y
hipError_t launch_apply_dot_f64(const stdg_mesh* m, const double* C, const double* x, double* y, double* part,
                                hipStream_t s) {
    return apply_m64(m, C, x, y, part, s);
}

hipError_t launch_apply_f64_c(const stdg_mesh* m, const double* C, const double* x, double* y,
                              hipStream_t s) {
    return launch_apply<double>(m, m->d.blocks, C, x, y, s);
}

hipError_t launch_apply_f32_c(const stdg_mesh* m, const float* C, const float* x, float* y, hipStream_t s) {
    return launch_apply<float>(m, m->d.blocks32, C, x, y, s);
}

// y[e][a][n] = sum_b M[a][b] x[e][b][n]  (time mixing)
template <typename T>
__global__ void k_tmix(const T* __restrict__ x, T* __restrict__ y, const T* __restrict__ M, int64_t E,
                       int G, int N) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= E * N) return;
    const int64_t e = t / N;
    const int n = (int)(t - e * N);
    T v[8];
    for (int b = 0; b < G; ++b) v[b] = x[(e * G + b) * N + n];
    for (int a = 0; a < G; ++a) {
        T s = T(0);
        for (int b = 0; b < G; ++b) s += M[a * G + b] * v[b];
        y[(e * G + a) * N + n] = s;
    }
}

hipError_t time_mix_f64(const stdg_mesh* m, const double* M, const double* x, double* y, hipStream_t s) {
    hipLaunchKernelGGL(k_tmix<double>, dim3((unsigned)((m->E * m->N + 255) / 256)), dim3(256), 0, s, x, y, M,
                       m->E, m->G, m->N);
    return hipGetLastError();
}

hipError_t time_mix_f32(const stdg_mesh* m, const float* M, const float* x, float* y, hipStream_t s) {
    hipLaunchKernelGGL(k_tmix<float>, dim3((unsigned)((m->E * m->N + 255) / 256)), dim3(256), 0, s, x, y, M,
                       m->E, m->G, m->N);
    return hipGetLastError();
}

hipError_t launch_apply_f64(const stdg_mesh* m, const double* x, double* y, hipStream_t s) {
    return launch_apply<double>(m, m->d.blocks, m->d.C, x, y, s);
}

hipError_t launch_apply_f32(const stdg_mesh* m, const float* x, float* y, hipStream_t s) {
    return launch_apply<float>(m, m->d.blocks32, m->d.C32, x, y, s);
}

__global__ void cvt_d2f(const double* __restrict__ a, float* __restrict__ b, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = (float)a[i];
}
__global__ void cvt_f2d(const float* __restrict__ a, double* __restrict__ b, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = (double)a[i];
}

hipError_t convert_d2f(const double* a, float* b, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(cvt_d2f, dim3((n + 255) / 256), dim3(256), 0, s, a, b, n);
    return hipGetLastError();
}
hipError_t convert_f2d(const float* a, double* b, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(cvt_f2d, dim3((n + 255) / 256), dim3(256), 0, s, a, b, n);
    return hipGetLastError();
}

}  // namespace stdg
