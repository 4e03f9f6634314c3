// Block-row kernels of the Picard step on the FP64 matrix cores (Sec. 2.6,
// steps 1, 3, 4, 5, 6; eqs. average, goback, prevpress / A3_mod, A1_mod,
// A2_mod): every output row of N coefficients is a sum of small N x N blocks
// times gathered rows, the blocks shared by a geometry class (and local face).
//
// One workgroup takes a group of up to 64 consecutive entities that share
// their blocks (elements of one class, or faces, which are sorted by the
// classes and local faces of their two sides).  The blocks are staged in LDS
// and four wavefronts take 16 entities each, their components and time nodes
// as further columns, so an operand read from LDS feeds several matrix
// instructions and a row is read with 16-byte loads (mfma64.hpp).  They
// replace, where the groups fill, kernels with one output row per thread,
// which read every row with a stride of N doubles between lanes.
// What bounds them is the row traffic, on small meshes the latency of one
// group.  82,944 elements, p = 3, p_gamma = 1: average 275 -> 76 us, goback 383
// -> 170, right-hand side 266 -> 67; 663,552 elements, p_gamma = 0: average 976
// -> 291 us (0.96 GB), goback 1,437 -> 357, gradient 912 -> 299, right-hand side
// 1,068 -> 273; the three transfers of 1,296 elements with walls, p = 3,
// p_gamma = 1: 162 -> 37.

#include <algorithm>

#include "internal.hpp"
#include "kernels.hpp"
#include "mfma64.hpp"

namespace stdg {
namespace {

constexpr int RT = 256;

// wavefronts per SIMD to leave registers for: the kernels wait on rows, so
// four where the accumulators allow it (663,552 elements, p = 3: goback 441 ->
// 357 us, gradient 417 -> 299 together with the group records below; average,
// whose four row sets fill more registers, 291 -> 309: it keeps two)
template <int N, int G> constexpr int waves() {
    return M64<N>::NQ * 3 * G <= 18 ? 4 : (M64<N>::NQ * G <= 25 ? 2 : 1);
}

// components (or directions) of one workgroup: all three while their
// accumulators leave room for two wavefronts per SIMD
template <int N, int G> constexpr int comps() { return M64<N>::NQ * 3 * G <= 48 ? 3 : 1; }

template <int R, int C> __device__ inline void zero(double (&a)[R][C]) {
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < C; ++j) a[i][j] = 0.0;
}

// doubles of LDS: the staged blocks, and afterwards the four wavefronts'
// output rows
template <int N, int G, int BLOCKS> constexpr int lds_size() {
    return BLOCKS * N * M64<N>::NP > 4 * 16 * G * N ? BLOCKS * N * M64<N>::NP : 4 * 16 * G * N;
}

// acc[rg][col0 + a] of the wavefront's entities first .. (those below end) to
// the rows of y ([entity][G][N]) times scale(a); all wavefronts have passed a
// barrier since they last read the blocks in `lds`
template <int N, int G, int NC, typename S>
__device__ __forceinline__ void put_rows(double* lds, int wave, int lane, int hi, double* __restrict__ y, int64_t first,
                                         int64_t end, const double (&acc)[M64<N>::NQ][NC], int col0, S&& scale) {
    const int64_t left = end - first;
    if (left <= 0) return;
    const int count = (int)(left < 16 ? left : 16) * G * N;
    double* dst = y + first * G * N;
    m64_flush<N, G>(lds + wave * 16 * G * N, lane, hi, count,
                    [&](int rg, int a) { return scale(a) * acc[rg][col0 + a]; },
                    [&](int i, m64_d2u v) { m64_put(dst, i, count, v); });
}

struct Lane {
    int lane, wave, hi, lo;
    __device__ Lane() {
        lane = threadIdx.x & 63;
        wave = threadIdx.x >> 6;
        hi = lane >> 4;
        lo = lane & 3;
    }
};

// eq. average: vbar[c][i][a] = sum_f A_{i,f} vhat[c][face(i,f)][a]
template <int N, int G>
__global__ void __launch_bounds__(RT) kr_average(const double* __restrict__ At, const m64_i4* __restrict__ segs,
                                                 const int64_t* __restrict__ tet_face, const double* __restrict__ vhat,
                                                 double* __restrict__ vbar, int64_t E, int64_t F, uint32_t n_groups) {
    constexpr int NQ = M64<N>::NQ, NP = M64<N>::NP, CP = comps<N, G>();
    __shared__ double A[lds_size<N, G, 4>()];
    const uint32_t gi = m64_group(gridDim.x);
    if (gi >= n_groups) return;
    const m64_i4 g = segs[gi];
    const int c0 = blockIdx.y * CP, c = g.z;
    const int64_t e0 = g.x, e1 = e0 + g.y;
    m64_stage<N, RT>(At + (int64_t)c * 4 * N * N, A, 4);
    __syncthreads();
    const Lane l;
    const int64_t i = e0 + 16 * l.wave + (l.lane & 15);
    const bool valid = i < e1;
    __amdgpu_buffer_rsrc_t rv[CP];
#pragma unroll
    for (int k = 0; k < CP; ++k) rv[k] = m64_rsrc(vhat + (c0 + k) * F * G * N, (uint32_t)(8 * F * G * N));
    double acc[NQ][CP * G];
    zero(acc);
    int64_t face[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) face[f] = valid ? tet_face[4 * i + f] : -1;
#pragma unroll
    for (int f = 0; f < 4; ++f) {
        double b[CP * G][NQ];
#pragma unroll
        for (int k = 0; k < CP; ++k)
#pragma unroll
            for (int a = 0; a < G; ++a)
                m64_load<N>(rv[k], valid ? (uint32_t)((face[f] * G + a) * N * 8) : M64_OOB, l.hi, b[k * G + a]);
        m64_block<N, CP * G>(A + f * N * NP, b, l.lo, l.hi, acc);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < CP; ++k)
        put_rows<N, G>(A, l.wave, l.lane, l.hi, vbar + (c0 + k) * E * G * N, e0 + 16 * l.wave, e1, acc, k * G,
                       [](int) { return 1.0; });
}

// eq. goback on faces f0 .. f1: out[c][j][a] = GB_l vbar_l[a] + GB_r vbar_r[a]
// (boundary faces: one side, from vbdry)
template <int N, int G>
__global__ void __launch_bounds__(RT, (waves<N, G>())) kr_goback(const double* __restrict__ GBt, const int64_t* __restrict__ fl,
                                                const int64_t* __restrict__ fr,
                                                const double* __restrict__ vbar, const double* __restrict__ vbdry,
                                                double* __restrict__ out, int64_t f0, int64_t f1, int64_t F, int64_t E,
                                                const m64_i4* __restrict__ grp, uint32_t n_groups) {
    constexpr int NQ = M64<N>::NQ, NP = M64<N>::NP, CP = comps<N, G>();
    __shared__ double A[lds_size<N, G, 2>()];
    const uint32_t gi = m64_group(gridDim.x);
    if (gi >= n_groups) return;
    const m64_i4 g = grp[gi];
    const int c0 = blockIdx.y * CP;
    const int64_t j0 = g.x, j1 = j0 + g.y;
    if (j0 < f0 || j0 >= f1) return;      // (f0 and f1 lie between groups)
    const bool inner = g.w >= 0;
    const Lane l;
    const int64_t j = j0 + 16 * l.wave + (l.lane & 15);
    const bool valid = j < j1;
    const double* src = inner ? vbar : vbdry;
    double acc[NQ][CP * G];
    zero(acc);
    // the left rows are in flight while the blocks are staged
    const int64_t side[2] = {valid ? fl[j] : -1, valid && inner ? fr[j] : -1};
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (q == 1 && !inner) break;
        double b[CP * G][NQ];
#pragma unroll
        for (int k = 0; k < CP; ++k) {
            const __amdgpu_buffer_rsrc_t rv = m64_rsrc(src + (c0 + k) * E * G * N, (uint32_t)(8 * E * G * N));
#pragma unroll
            for (int a = 0; a < G; ++a)
                m64_load<N>(rv, side[q] >= 0 ? (uint32_t)((side[q] * G + a) * N * 8) : M64_OOB, l.hi, b[k * G + a]);
        }
        if (q == 0) {
            m64_stage<N, RT>(GBt + (int64_t)g.z * N * N, A, 1);
            if (inner) m64_stage<N, RT>(GBt + (int64_t)g.w * N * N, A + N * NP, 1);
            __syncthreads();
        }
        m64_block<N, CP * G>(A + q * N * NP, b, l.lo, l.hi, acc);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < CP; ++k)
        put_rows<N, G>(A, l.wave, l.lane, l.hi, out + (c0 + k) * F * G * N, j0 + 16 * l.wave, j1, acc, k * G,
                       [](int) { return 1.0; });
}

// dual-grid pressure gradient: w[d][j][a] = dt sum_b TW[a][b] (US_{l,d} p_l[b] + UN_{l,d} p_r[b])
template <int N, int G>
__global__ void __launch_bounds__(RT, (waves<N, G>())) kr_dualgrad(const double* __restrict__ USt, const double* __restrict__ UNt,
                                                  const int64_t* __restrict__ fl, const int64_t* __restrict__ fr,
                                                  const double* __restrict__ TW,
                                                  const double* __restrict__ p, double dt, double* __restrict__ w,
                                                  int64_t F, int64_t E, const m64_i4* __restrict__ grp,
                                                  uint32_t n_groups) {
    constexpr int NQ = M64<N>::NQ, NP = M64<N>::NP, CP = comps<N, G>();
    __shared__ double A[lds_size<N, G, 2 * CP>()];
    const uint32_t gi = m64_group(gridDim.x);
    if (gi >= n_groups) return;
    const m64_i4 g = grp[gi];
    const int d0 = blockIdx.y * CP;
    const int64_t j0 = g.x, j1 = j0 + g.y;
    const bool inner = g.w >= 0;
    const int64_t key = (int64_t)g.z * 3 + d0;
    const Lane l;
    const int64_t j = j0 + 16 * l.wave + (l.lane & 15);
    const bool valid = j < j1;
    const __amdgpu_buffer_rsrc_t rp = m64_rsrc(p, (uint32_t)(8 * E * G * N));
    // both sides' rows in flight while the blocks are staged
    const int64_t side[2] = {valid ? fl[j] : -1, valid && inner ? fr[j] : -1};
    double b[2][G][NQ];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int a = 0; a < G; ++a)
            m64_load<N>(rp, side[q] >= 0 ? (uint32_t)((side[q] * G + a) * N * 8) : M64_OOB, l.hi, b[q][a]);
    m64_stage<N, RT>(USt + key * N * N, A, CP);
    if (inner) m64_stage<N, RT>(UNt + key * N * N, A + CP * N * NP, CP);
    double acc[CP][NQ][G];
#pragma unroll
    for (int d = 0; d < CP; ++d) zero(acc[d]);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (q == 1 && !inner) break;
        double bt[G][NQ];
#pragma unroll
        for (int a = 0; a < G; ++a)
#pragma unroll
            for (int t = 0; t < NQ; ++t) {
                double s = 0.0;
#pragma unroll
                for (int bb = 0; bb < G; ++bb) s += TW[a * G + bb] * b[q][bb][t];
                bt[a][t] = s;
            }
#pragma unroll
        for (int d = 0; d < CP; ++d) m64_block<N, G>(A + (q * CP + d) * N * NP, bt, l.lo, l.hi, acc[d]);
    }
    __syncthreads();
#pragma unroll
    for (int d = 0; d < CP; ++d)
        put_rows<N, G>(A, l.wave, l.lane, l.hi, w + (d0 + d) * F * G * N, j0 + 16 * l.wave, j1, acc[d], 0,
                       [dt](int) { return dt; });
}

// pressure right-hand side: b[i][a] = dt W_a sum_{f,d} Q^T_{i,f,d} Fv[d][face][a]
template <int N, int G>
__global__ void __launch_bounds__(RT, (waves<N, G>())) kr_rhs(const double* __restrict__ QTt, const m64_i4* __restrict__ segs,
                                             const int64_t* __restrict__ tet_face,
                                             const double* __restrict__ W, const double* __restrict__ Fv, double dt,
                                             double* __restrict__ out, int64_t E, int64_t F, uint32_t n_groups) {
    constexpr int NQ = M64<N>::NQ, NP = M64<N>::NP;
    __shared__ double A[lds_size<N, G, 3>()];
    const uint32_t gi = m64_group(gridDim.x);
    if (gi >= n_groups) return;
    const m64_i4 g = segs[gi];
    const int c = g.z;
    const int64_t e0 = g.x, e1 = e0 + g.y;
    const Lane l;
    const int64_t i = e0 + 16 * l.wave + (l.lane & 15);
    const bool valid = i < e1;
    __amdgpu_buffer_rsrc_t rv[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) rv[d] = m64_rsrc(Fv + d * F * G * N, (uint32_t)(8 * F * G * N));
    double acc[NQ][G];
    zero(acc);
#pragma unroll 1
    for (int f = 0; f < 4; ++f) {
        double b[3][G][NQ];
        const int64_t j = valid ? tet_face[4 * i + f] : -1;
#pragma unroll
        for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int a = 0; a < G; ++a)
                m64_load<N>(rv[d], valid ? (uint32_t)((j * G + a) * N * 8) : M64_OOB, l.hi, b[d][a]);
        __syncthreads();
        m64_stage<N, RT>(QTt + ((int64_t)c * 4 + f) * 3 * N * N, A, 3);
        __syncthreads();
#pragma unroll
        for (int d = 0; d < 3; ++d) m64_block<N, G>(A + d * N * NP, b[d], l.lo, l.hi, acc);
    }
    __syncthreads();
    put_rows<N, G>(A, l.wave, l.lane, l.hi, out, e0 + 16 * l.wave, e1, acc, 0, [&](int a) { return dt * W[a]; });
}

// components per workgroup of the viscous right-hand side: beside the sums it
// holds as many mixed columns, so all three only at p = 1 with one or two time
// nodes.
// One against three, us: 3,072 elements, p = 2, p_gamma = 4 26.5 -> 8.8 (14.6 on
// the vector units), p = 3, p_gamma = 2 26.1 -> 9.9; 48,000, p = 2, p_gamma = 4
// 104 -> 61 (94; three spilled 64 registers), p_gamma = 1 23.2 -> 23.1.
template <int N, int G> constexpr int rhs_comps() { return N == 4 && G <= 2 ? 3 : 1; }

// viscous right-hand side: M (sum_b g0g1[a][b] vprev_b - T[a][b] lam_b) - ups_a - nu dt W_a sum_{bdry f} BB_f vbc
template <int N, int G>
__global__ void __launch_bounds__(RT, (waves<N, G>())) kr_visc_rhs(const double* __restrict__ MIt, const double* __restrict__ BBt,
                                                  const m64_i4* __restrict__ segs,
                                                  const int32_t* __restrict__ nbr, const int64_t* __restrict__ tet_face,
                                                  const double* __restrict__ g0g1, const double* __restrict__ Tm,
                                                  const double* __restrict__ W, const double* __restrict__ vprev,
                                                  const double* __restrict__ ups, const double* __restrict__ lam,
                                                  const double* __restrict__ vbc, double nu_dt,
                                                  double* __restrict__ rhs, int64_t E, int64_t F, uint32_t n_groups) {
    constexpr int NQ = M64<N>::NQ, CP = rhs_comps<N, G>();
    __shared__ double A[lds_size<N, G, 1>()];
    const uint32_t gi = m64_group(gridDim.x);
    if (gi >= n_groups) return;
    const m64_i4 g = segs[gi];
    const int c0 = blockIdx.y * CP, c = g.z;
    const int64_t e0 = g.x, e1 = e0 + g.y;
    m64_stage<N, RT>(MIt + (int64_t)c * N * N, A, 1);
    const Lane l;
    const int64_t i = e0 + 16 * l.wave + (l.lane & 15);
    const bool valid = i < e1;
    double acc[NQ][CP * G];
    // start from -ups in the rows this lane will store
#pragma unroll
    for (int rg = 0; rg < NQ; ++rg)
#pragma unroll
        for (int k = 0; k < CP; ++k)
#pragma unroll
            for (int a = 0; a < G; ++a)
                acc[rg][k * G + a] = valid && 4 * rg + l.hi < N
                                         ? -ups[(((c0 + k) * E + i) * G + a) * N + 4 * rg + l.hi] : 0.0;
    double bt[CP * G][NQ];
#pragma unroll
    for (int k = 0; k < CP; ++k) {
        const __amdgpu_buffer_rsrc_t rp = m64_rsrc(vprev + (c0 + k) * E * G * N, (uint32_t)(8 * E * G * N));
        const __amdgpu_buffer_rsrc_t rl = m64_rsrc(lam + (c0 + k) * E * G * N, (uint32_t)(8 * E * G * N));
#pragma unroll
        for (int a = 0; a < G; ++a)
#pragma unroll
            for (int t = 0; t < NQ; ++t) bt[k * G + a][t] = 0.0;
#pragma unroll
        for (int b = 0; b < G; ++b) {
            double v[NQ], u[NQ];
            const uint32_t off = valid ? (uint32_t)((i * G + b) * N * 8) : M64_OOB;
            m64_load<N>(rp, off, l.hi, v);
            m64_load<N>(rl, off, l.hi, u);
#pragma unroll
            for (int a = 0; a < G; ++a)
#pragma unroll
                for (int t = 0; t < NQ; ++t) bt[k * G + a][t] += g0g1[a * G + b] * v[t] - Tm[a * G + b] * u[t];
        }
    }
    __syncthreads();
    m64_block<N, CP * G>(A, bt, l.lo, l.hi, acc);
    // boundary faces (the same ones on every element of a class)
    for (int f = 0; f < 4; ++f) {
        if (nbr[4 * e0 + f] >= 0) continue;
        __syncthreads();
        m64_stage<N, RT>(BBt + ((int64_t)c * 4 + f) * N * N, A, 1);
        const int64_t j = valid ? tet_face[4 * i + f] : -1;
        double b[CP * G][NQ];
#pragma unroll
        for (int k = 0; k < CP; ++k) {
            const __amdgpu_buffer_rsrc_t rb = m64_rsrc(vbc + (c0 + k) * F * G * N, (uint32_t)(8 * F * G * N));
#pragma unroll
            for (int a = 0; a < G; ++a) {
                m64_load<N>(rb, valid ? (uint32_t)((j * G + a) * N * 8) : M64_OOB, l.hi, b[k * G + a]);
#pragma unroll
                for (int t = 0; t < NQ; ++t) b[k * G + a][t] *= -nu_dt * W[a];
            }
        }
        __syncthreads();
        m64_block<N, CP * G>(A, b, l.lo, l.hi, acc);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < CP; ++k)
        put_rows<N, G>(A, l.wave, l.lane, l.hi, rhs + (c0 + k) * E * G * N, e0 + 16 * l.wave, e1, acc, k * G,
                       [](int) { return 1.0; });
}

}  // namespace

// A group kernel costs a time per group (blocks staged, one workgroup's chain),
// the kernels on the vector units one per element beside a floor that grows
// with p.  So groups are used while their number stays below
//   base + elements / slope,
// four and more elements each on average: `base` groups take as long as the
// other kernel's floor, and from `slope` elements per group on the groups are
// as fast on any mesh.  Fitted to 7 meshes of 4 to 40 elements per group for
// each of 486, 1,536 and 3,456 groups; us, groups / vector units:
//   average, p = 2, p_gamma = 1: 486 groups of 4 9 / 14, 1,536 of 4 19 / 17, of
//   16 22 / 27, 3,456 of 8 38 / 31, of 24 46 / 82;
//   goback, p = 2, p_gamma = 1: 1,536 of 4 22 / 13, of 16 25 / 28, 3,456 of 8 44 / 33;
//   p = 1: 1,536 of 8 10 / 7, of 40 16 / 16; p = 3: 1,536 of 4 48 / 47, of 16 52 / 100;
//   pressure right-hand side, p = 1, p_gamma = 2: 3,456 of 24 26 / 24, of 40 31 / 37;
//   p >= 2 ahead at every number;
//   viscous right-hand side, p = 2, p_gamma = 1: 1,536 of 4 14 / 11, of 12 15 / 16;
//   viscous operator (with D^-1 and the dots, per BiCGStab iteration), p = 1,
//   p_gamma = 1: 1,536 of 4 27 / 25, 3,456 of 12 56 / 45, of 24 62 / 67;
//   convection, p = 2, p_gamma = 1: 486 of 4 77 / 124, 1,536 of 8 219 / 141, of 40
//   243 / 365, 3,456 of 8 510 / 220.
// Convection of 4, 5 time nodes has a longer chain (p = 1 78 us, p = 2 180) than
// the lane-per-element kernel on small meshes of whole runs or many classes (51,
// 140); where runs mix few classes that kernel takes 170 to 800.
bool groups_pay(const stdg_mesh* m, GroupKernel k) {
    const bool faces = k == GroupKernel::FACES;
    const int64_t n = faces ? (int64_t)m->faces.size() : m->E;
    const int64_t groups = faces ? m->pd.n_face_groups : m->d.n_segs;
    if (4 * groups > n) return false;
    // by kernel, p - 1 and time nodes 1, 2, 3, more
    constexpr int ANY = 1 << 30;
    static const int base[6][4][4] = {
        {{500, 64, 64, 64}, {2000, 900, 800, 300}, {1600, 1600, 800, 800}, {1000, 1000, 1000, 1000}},
        {{1000, 128, 128, 128}, {1000, 660, 660, 400}, {3200, 2400, 1600, 1000}, {2000, 2000, 2000, 500}},
        {{3500, 1700, 1400, 600}, {ANY, ANY, ANY, ANY}, {ANY, ANY, ANY, ANY}, {ANY, ANY, ANY, ANY}},
        {{1600, 300, 600, 100}, {1700, 1000, 1000, 400}, {2000, 1150, 1000, 300}, {1000, 1000, 300, 0}},
        {{3500, 1300, 1000, 900}, {3500, 3200, 2400, 1500}, {2500, 2500, 2500, 2500}, {2500, 2500, 2500, 2500}},
        {{2100, 650, 420, 50}, {2400, 650, 450, 50}, {3000, 1400, 550, 480}, {400, 450, 0, 0}}};
    const int deg = m->N == 4 ? 0 : (m->N == 10 ? 1 : (m->N == 20 ? 2 : 3));
    const bool rows = k != GroupKernel::VISCOUS && k != GroupKernel::CONVECTION;
    const int slope = rows && deg == 0 ? 48 : (faces ? 20 : 32);
    if (k == GroupKernel::CONVECTION && deg < 2 && m->G > 3 && m->E < 12000 &&
        (64 * (int64_t)m->n_classes > m->E || 64 * groups < n + 64))
        return false;
    return groups <= base[(int)k][deg][std::min(m->G, 4) - 1] + n / slope;
}

// every component within the 2 GiB of a buffer offset
bool rows_mfma_supported(const stdg_mesh* m, GroupKernel k) {
    return (m->N == 4 || m->N == 10 || m->N == 20 || m->N == 35) && m->G <= 5 && groups_pay(m, k) &&
           8 * (int64_t)m->faces.size() * m->Nst < ((int64_t)1 << 31);
}

#define STDG_ROWS(CALL)                                                                     \
    STDG_NG(CALL, 4, 1) STDG_NG(CALL, 4, 2) STDG_NG(CALL, 4, 3) STDG_NG(CALL, 4, 4)          \
    STDG_NG(CALL, 4, 5) STDG_NG(CALL, 10, 1) STDG_NG(CALL, 10, 2) STDG_NG(CALL, 10, 3)       \
    STDG_NG(CALL, 10, 4) STDG_NG(CALL, 10, 5) STDG_NG(CALL, 20, 1) STDG_NG(CALL, 20, 2)      \
    STDG_NG(CALL, 20, 3) STDG_NG(CALL, 20, 4) STDG_NG(CALL, 20, 5) STDG_NG(CALL, 35, 1)      \
    STDG_NG(CALL, 35, 2) STDG_NG(CALL, 35, 3) STDG_NG(CALL, 35, 4) STDG_NG(CALL, 35, 5)      \
    return hipErrorInvalidValue;
#define STDG_NG(CALL, n, g)           \
    if (m->N == n && m->G == g) {     \
        CALL(n, g);                   \
        return hipGetLastError();     \
    }

hipError_t rows_average(const stdg_mesh* m, const double* vhat, double* vbar, hipStream_t s) {
    const int64_t E = m->E, F = (int64_t)m->faces.size();
#define STDG_CALL(n, g)                                                                                           \
    hipLaunchKernelGGL((kr_average<n, g>), dim3(m64_blocks(m->d.n_segs), 3 / comps<n, g>()), dim3(RT), 0, s, m->pd.At, \
                       (const m64_i4*)m->d.segs, m->pd.tet_face, vhat, vbar, E, F, (uint32_t)m->d.n_segs)
    STDG_ROWS(STDG_CALL)
#undef STDG_CALL
}

hipError_t rows_goback(const stdg_mesh* m, const double* vbar, const double* vbdry, double* out, int64_t f0, int64_t f1,
                       hipStream_t s) {
    if (f1 <= f0) return hipSuccess;
    const PicardDevice& d = m->pd;
    const int64_t F = (int64_t)m->faces.size();
#define STDG_CALL(n, g)                                                                                               \
    hipLaunchKernelGGL((kr_goback<n, g>), dim3(m64_blocks(d.n_face_groups), 3 / comps<n, g>()), dim3(RT), 0, s, d.GBt, d.fl,       \
                       d.fr, vbar, vbdry, out, f0, f1, F, m->E, (const m64_i4*)d.face_groups, (uint32_t)d.n_face_groups)
    STDG_ROWS(STDG_CALL)
#undef STDG_CALL
}

hipError_t rows_dualgrad(const stdg_mesh* m, const double* p, double dt, double* w, hipStream_t s) {
    const PicardDevice& d = m->pd;
    const int64_t F = (int64_t)m->faces.size();
#define STDG_CALL(n, g)                                                                                             \
    hipLaunchKernelGGL((kr_dualgrad<n, g>), dim3(m64_blocks(d.n_face_groups), 3 / comps<n, g>()), dim3(RT), 0, s, d.USt, d.UNt,        \
                       d.fl, d.fr, d.TW, p, dt, w, F, m->E, (const m64_i4*)d.face_groups, (uint32_t)d.n_face_groups)
    STDG_ROWS(STDG_CALL)
#undef STDG_CALL
}

hipError_t rows_rhs_pressure(const stdg_mesh* m, const double* Fv, double dt, double* b, hipStream_t s) {
    const int64_t E = m->E, F = (int64_t)m->faces.size();
#define STDG_CALL(n, g)                                                                                          \
    hipLaunchKernelGGL((kr_rhs<n, g>), dim3(m64_blocks(m->d.n_segs)), dim3(RT), 0, s, m->pd.QTt, (const m64_i4*)m->d.segs,     \
                       m->pd.tet_face, m->pd.W, Fv, dt, b, E, F, (uint32_t)m->d.n_segs)
    STDG_ROWS(STDG_CALL)
#undef STDG_CALL
}

hipError_t rows_visc_rhs(const stdg_mesh* m, const double* vprev, const double* ups, const double* lam,
                         const double* vbc, double* rhs, hipStream_t s) {
    const PicardDevice& d = m->pd;
    const int64_t E = m->E, F = (int64_t)m->faces.size();
#define STDG_CALL(n, g)                                                                                            \
    hipLaunchKernelGGL((kr_visc_rhs<n, g>), dim3(m64_blocks(m->d.n_segs), 3 / rhs_comps<n, g>()), dim3(RT), 0, s, d.MIt, d.BBt,       \
                       (const m64_i4*)m->d.segs, m->d.nbr, d.tet_face, d.g0g1, d.Tm, d.W, vprev, ups, lam, vbc,      \
                       m->cfg.nu * m->cfg.dt, rhs, E, F, (uint32_t)m->d.n_segs)
    STDG_ROWS(STDG_CALL)
#undef STDG_CALL
}

}  // namespace stdg
