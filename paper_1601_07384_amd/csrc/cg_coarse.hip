// Two-level preconditioner of the FP32 inner CG on B (x) I (eq. CS_19 on every
// time node).  With the block-Jacobi step alone the iterations grow with the
// number of elements across the domain: nothing carries the smooth part of
// the error further than one element per iteration.  The second level does,
// in one additive step:
//   M^-1 r = c^-1 (B_e^-1 r + P K P^T r),
// P the continuous piecewise linear functions on a tensor grid of vertices,
// sampled at the element nodes (corner values by `corner` or `tri`, node
// values by the barycentric weights), K the inverse of dt^2 times the
// Laplacian of that grid (linear elements, lumped mass, its constant mode
// left out), which is spectrally equivalent to P^T B P: on structured cubes
// 34..38 iterations per 1e-5 at p = 2, 3 whatever the size, as many as with
// the exact P^T B P, against 103 (8^3), 150 (12^3) and about 420 (48^3) with
// block Jacobi alone (CPU emulation; solve times at tl_min_elements in
// cg_fused.hip and at limits below).
//
// K is applied exactly, by fast diagonalisation: with the generalised
// eigenvectors V_d of the one-dimensional stiffness and lumped mass matrices
// K = (V_z (x) V_y (x) V_x) (l_x + l_y + l_z)^-1 (V_z (x) V_y (x) V_x)^T,
// six small matrix products (48 x 48 per plane at 48^3) on
// v_mfma_f32_16x16x4f32 in three kernels: the planes forward, the columns
// there and back around the division, the planes backward.  What bounds them
// is latency (48 workgroups per time node at 48^3, 64 MFLOP in all), so the
// work per launch is one whole plane or column tile held in LDS.
//
// The grid: the vertices' own coordinate lines when the vertices are a tensor
// grid (then a corner is a grid node), otherwise uniform lines with as many
// cells as hexahedra of six elements fill the box, corners interpolated
// trilinearly.  It needs a mesh that fills its bounding box (the elements'
// volumes add up to it), elements a few cells wide and spacings within bounds
// (limits); other meshes keep the block-Jacobi step.

#include <algorithm>
#include <cmath>
#include <map>
#include <numeric>
#include <vector>

#include "internal.hpp"
#include "kernels.hpp"
#include "two_level.hpp"

namespace stdg {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int MAXN = 80;        // grid lines per direction (two padded planes in 64 KB of LDS)
constexpr int CC = 32;          // columns per workgroup of the column kernel
// lanes per grid node of the restriction: a node of a tensor grid is reached
// by about 24 corners, one of a grid between scattered vertices by about 190
// (4,374 scattered elements: 14.6 us with 8 lanes per node, 5.0 with 64)
constexpr int RL1 = 8, RLW = 64;
// Where the second level does not earn its launches and passes (an iteration
// takes 1.4 to 3 times that of block Jacobi alone) block Jacobi stays alone: on
// elements many cells wide, which alias the grid functions, and on lines of
// very different spacing, where the FP32 rounding of the smooth part reaches
// the rough one.  Periodic meshes need half the iterations of block Jacobi, so
// small ones earn less.  Solve to 1e-8, time of two-level / block Jacobi, 384 to
// 7,986 elements, p = 1, 2, 3; spacings graded by the given factor:
//   scattered, walls, elements 2.8 cells wide (graded 10 in all directions) 0.53
//   to 0.90, 3.5 (30) 0.90 to 2.5, more (100) 1.3 to 6.1; periodic 2.0 (4) 0.50
//   to 1.01, 2.8 (10) 0.72 to 1.18, 3.1 (15) 0.85 to 1.22, and 24,576 elements
//   2.8 0.77;
//   tensor grid, walls, 100 or 127 0.35 to 0.97, once 1.21 (127), 1,000 0.48 to
//   1.60, 10^4 0.46 to 1.02 at p = 1, 2 and not converged at p = 3; periodic,
//   common blocks, 8 0.53 to 0.97, 16 0.76 to 1.23, 100 0.90 to 1.31, from 24,576
//   elements 100 0.80 to 0.96; periodic, blocks per element, 384 and 1,296
//   elements 10 0.72 to 0.92, 100 0.85 to 1.35, from 3,072 100 0.73 to 1.03.
struct Limits {
    double width;       // cells an element spans in any direction
    double grading;     // widest spacing / narrowest, all directions together
};
Limits limits(const stdg_mesh* m) {
    const bool small = m->cfg.periodic && m->N != 35 && m->E < 16384;
    return Limits{small ? 2.25 : 3.25, small && (!elem_supported(m) || m->E < 3000) ? 8.0 : 100.5};
}

inline int pad16(int n) { return (n + 15) / 16 * 16; }

// g[a][node] = sum over the corners that reach the node, RL lanes per node, in a
// fixed order.  A node of a tensor grid has K entries (padded with slot -1),
// one between scattered vertices the entries row[node] .. row[node + 1]: there
// the fullest node has many times the mean (graded meshes, 3,072 elements, 14 to
// 47 times), and padded rows would be mostly padding, read in every iteration.
template <bool HASW>
__global__ void __launch_bounds__(256) k_restrict(const int32_t* __restrict__ slot, const float* __restrict__ w,
                                                  const int64_t* __restrict__ row, int K,
                                                  const float* __restrict__ e4, int64_t estr, float* __restrict__ g,
                                                  int nodes, const double* __restrict__ scal, int it) {
    constexpr int RL = HASW ? RLW : RL1;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t j = t / RL;
    const int a = blockIdx.y, l = (int)(t % RL);
    float s = 0.0f;
    if (j < nodes) {
        const float* ea = e4 + a * estr;
        if (HASW) {
            const int64_t end = row[j + 1];
            for (int64_t k = row[j] + l; k < end; k += RL) s += w[k] * ea[slot[k]];
        } else {
            for (int k = l; k < K; k += RL) {
                const int c = slot[j * K + k];
                s += c >= 0 ? ea[c] : 0.0f;
            }
        }
    }
#pragma unroll
    for (int o = RL / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, RL);
    if (l == 0 && j < nodes && !tl_done(scal, it)) g[(int64_t)a * nodes + j] = s;
}

// threads of the plane and column kernels on grids padded to 16 T lines: a
// wavefront per 16 x 16 tile of a result while a workgroup holds as many
template <int T> constexpr int plane_threads() { return T * T < 4 ? 256 : (T * T > 16 ? 1024 : 64 * T * T); }
template <int T> constexpr int column_threads() { return T < 2 ? 256 : 128 * T; }

// One plane z = const: out = My^T in Mx, in and out [ny][nx] (Mx, My padded
// to multiples of 16 with zeros; V forward, V^T backward; the larger pad is
// 16 T).  The wavefront's operands of both products are under way before the
// plane is staged: loaded inside the products they cost a cache latency per
// 16 lines (24^3, two time nodes: 4.4 -> 3.7 us; the column kernel 5.6 -> 4.4).
template <int T>
__global__ void __launch_bounds__(plane_threads<T>()) k_plane(const float* __restrict__ in, float* __restrict__ out,
                                                              const float* __restrict__ Mx,
                                                              const float* __restrict__ My, int nx, int ny,
                                                              const double* __restrict__ scal, int it) {
    constexpr int P = 16 * T, S = P + 1, NT = plane_threads<T>(), NW = NT / 64;
    __shared__ float X[P * S], U[P * S];
    const int px = (nx + 15) / 16 * 16, py = (ny + 15) / 16 * 16;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lo = lane & 15, hi = lane >> 4;
    float bx[4 * T], ay[4 * T];
    auto column = [&](const float* __restrict__ M, int pad, int c, float (&v)[4 * T]) {
#pragma unroll
        for (int k = 0; k < 4 * T; ++k) v[k] = 4 * k < pad && c < pad ? M[(4 * k + hi) * pad + c] : 0.0f;
    };
    if (wave < T * T) {
        column(Mx, px, wave % T * 16 + lo, bx);
        column(My, py, wave / T * 16 + lo, ay);
    }
    const float* src = in + (int64_t)blockIdx.x * nx * ny;
#pragma unroll
    for (int t = tid; t < P * P; t += NT) {
        const int i = t / P, j = t % P;
        X[i * S + j] = (i < ny && j < nx) ? src[i * nx + j] : 0.0f;
    }
    if (tl_done(scal, it)) return;
    __syncthreads();
#pragma unroll
    for (int t0 = 0; t0 < T * T; t0 += NW) {
        const int t = t0 + wave, r0 = t / T * 16, c0 = t % T * 16;
        if (t >= T * T) break;
        if (t0 > 0) column(Mx, px, c0 + lo, bx);
        f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < 4 * T; ++k)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(X[(r0 + lo) * S + 4 * k + hi], bx[k], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) U[(r0 + 4 * hi + r) * S + c0 + lo] = acc[r];
    }
    __syncthreads();
    float* dst = out + (int64_t)blockIdx.x * nx * ny;
#pragma unroll
    for (int t0 = 0; t0 < T * T; t0 += NW) {
        const int t = t0 + wave, r0 = t / T * 16, c0 = t % T * 16;
        if (t >= T * T) break;
        if (t0 > 0) column(My, py, r0 + lo, ay);
        f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < 4 * T; ++k)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ay[k], U[(4 * k + hi) * S + c0 + lo], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (r0 + 4 * hi + r < ny && c0 + lo < nx) dst[(r0 + 4 * hi + r) * nx + c0 + lo] = acc[r];
    }
}

// CC columns of one time node: forward in z, times scale / (l_x + l_y + l_z)
// (0 for the constant mode), backward in z, in place; the workgroup's share
// of the sum of (transformed value)^2 times that factor, i.e. of (P^T r) . K (P^T r).
// pz = 16 T; operands under way first, as in k_plane.
template <int T>
__global__ void __launch_bounds__(column_threads<T>()) k_columns(float* __restrict__ t, const float* __restrict__ Vz,
                                                                 const float* __restrict__ VzT,
                                                                 const float* __restrict__ lam, int nx, int ny, int nz,
                                                                 float scale, float cut, double* __restrict__ part,
                                                                 const double* __restrict__ scal, int it) {
    constexpr int P = 16 * T, S = CC + 1, NT = column_threads<T>(), CT = CC / 16;
    __shared__ float X[P * S], U[P * S];
    __shared__ double red[NT / 64];
    const int cols = nx * ny;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lo = lane & 15, hi = lane >> 4;
    const int c0 = blockIdx.x * CC, r0 = wave / CT * 16, b0 = wave % CT * 16;
    const bool tile = wave < T * CT;
    float* ta = t + (int64_t)blockIdx.y * nz * cols;
    const int col = c0 + b0 + lo;
    float af[4 * T], ab[4 * T], lxy = 0.0f, lz[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (tile) {
#pragma unroll
        for (int k = 0; k < 4 * T; ++k) {
            af[k] = Vz[(4 * k + hi) * P + r0 + lo];
            ab[k] = VzT[(4 * k + hi) * P + r0 + lo];
        }
        if (col < cols) lxy = lam[col % nx] + lam[nx + col / nx];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (r0 + 4 * hi + r < nz) lz[r] = lam[nx + ny + r0 + 4 * hi + r];
    }
#pragma unroll
    for (int q = tid; q < P * CC; q += NT) {
        const int i = q / CC, j = q % CC;
        X[i * S + j] = (i < nz && c0 + j < cols) ? ta[(int64_t)i * cols + c0 + j] : 0.0f;
    }
    if (tl_done(scal, it)) return;
    __syncthreads();
    double d = 0.0;
    if (tile) {
        f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < 4 * T; ++k)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(af[k], X[(4 * k + hi) * S + b0 + lo], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int kz = r0 + 4 * hi + r;
            const float l = kz < nz && col < cols ? lxy + lz[r] : 0.0f;
            const float f = l > cut ? scale / l : 0.0f;
            d += (double)acc[r] * (double)acc[r] * (double)f;
            U[kz * S + b0 + lo] = f * acc[r];
        }
    }
    __syncthreads();
    if (tile) {
        f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < 4 * T; ++k)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ab[k], U[(4 * k + hi) * S + b0 + lo], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int iz = r0 + 4 * hi + r;
            if (iz < nz && col < cols) ta[(int64_t)iz * cols + col] = acc[r];
        }
    }
    const double s = tl_reduce<NT>(d, red);
    if (tid == 0) part[blockIdx.y * gridDim.x + blockIdx.x] = s;
}

// A whole grid of at most SMALL_NODES nodes and SMALL_LINES lines in each
// direction in one workgroup per time node, in place of the restriction (with
// GATHER), the two plane kernels and the column kernel:
// bound by its eight barriers and the gather (a lane's 24 scattered corners
// take one CU's address unit 10 us at 1,000 nodes, hence SMALL_GATHER; the
// restriction on its own 3.2 us).  7^3 nodes: four kernels 13.2 us -> 6.5; 9^3,
// two time nodes: three kernels 10.7 -> 5.3.
constexpr int SMALL_NODES = 1024, SMALL_LINES = 16, SMALL_GATHER = 384;
template <bool GATHER, int NT>
__global__ void __launch_bounds__(NT) k_small(const int32_t* __restrict__ slot, int K,
                                                       const float* __restrict__ e4, int64_t estr,
                                                       float* __restrict__ g, const float* __restrict__ V0,
                                                       const float* __restrict__ V1, const float* __restrict__ V2,
                                                       const float* __restrict__ lam, int nx, int ny, int nz,
                                                       float scale, float cut, double* __restrict__ part,
                                                       const double* __restrict__ scal, int it) {
    constexpr int L = SMALL_LINES, S = L + 1;
    __shared__ float a[NT], b[NT], V[3][L * S];
    __shared__ double red[NT / 64];
    const int t = threadIdx.x, nodes = nx * ny * nz;
    for (int k = t; k < 3 * L * L; k += NT) {
        const int d = k / (L * L), q = k % (L * L);
        V[d][q / L * S + q % L] = (d == 0 ? V0 : (d == 1 ? V1 : V2))[q];
    }
    const bool on = t < nodes;
    float v = 0.0f;
    if (on) {
        if (GATHER) {
            typedef int i4 __attribute__((ext_vector_type(4)));
            const float* ea = e4 + blockIdx.x * estr;
            const i4* row = reinterpret_cast<const i4*>(slot + (int64_t)t * K);
#pragma unroll 6
            for (int k = 0; k < K / 4; ++k) {
                const i4 c = row[k];
#pragma unroll
                for (int u = 0; u < 4; ++u) v += c[u] >= 0 ? ea[c[u]] : 0.0f;
            }
        } else {
            v = g[(int64_t)blockIdx.x * nodes + t];
        }
        a[t] = v;
    }
    const int x = t % nx, y = t / nx % ny, z = t / (nx * ny);
    const float l = on ? lam[x] + lam[nx + y] + lam[nx + ny + z] : 0.0f;
    if (tl_done(scal, it)) return;
    // sum over a line of `src` through this node (first entry at, step, n
    // entries) times column c of V (forward) or its row (backward)
    auto line = [&](const float* src, int at, int step, int n, const float* Vd, int c, bool fwd) {
        // two sums, so that an LDS latency covers several terms
        float s[2] = {0.0f, 0.0f};
        int i = 0;
        for (; i + 4 <= n; i += 4)
#pragma unroll
            for (int u = 0; u < 4; ++u) s[u & 1] += src[at + (i + u) * step] * Vd[fwd ? (i + u) * S + c : c * S + i + u];
#pragma unroll
        for (int u = 0; u < 3; ++u)
            if (i + u < n) s[u & 1] += src[at + (i + u) * step] * Vd[fwd ? (i + u) * S + c : c * S + i + u];
        return s[0] + s[1];
    };
    __syncthreads();
    if (on) b[t] = line(a, t - x, 1, nx, V[0], x, true);
    __syncthreads();
    if (on) a[t] = line(b, t - y * nx, nx, ny, V[1], y, true);
    __syncthreads();
    double d = 0.0;
    if (on) {
        v = line(a, t - z * nx * ny, nx * ny, nz, V[2], z, true);
        const float f = l > cut ? scale / l : 0.0f;
        d = (double)v * (double)v * (double)f;
        b[t] = f * v;
    }
    __syncthreads();
    if (on) a[t] = line(b, t - z * nx * ny, nx * ny, nz, V[2], z, false);
    __syncthreads();
    if (on) b[t] = line(a, t - y * nx, nx, ny, V[1], y, false);
    __syncthreads();
    if (on) g[(int64_t)blockIdx.x * nodes + t] = line(b, t - x, 1, nx, V[0], x, false);
    const double s = tl_reduce<NT>(d, red);
    if (t == 0) part[blockIdx.x] = s;
}

// corner values of every element by trilinear interpolation (grids that do
// not pass through the vertices): tri = cell indices packed 10 bits each and
// the three fractions
struct TriCorner { int32_t cell; float f[3]; };
__global__ void __launch_bounds__(256) k_corners(const TriCorner* __restrict__ tri, const float* __restrict__ y,
                                                 float* __restrict__ yc, int64_t n, int64_t estr, int nx, int ny,
                                                 int nz, int wrap, const double* __restrict__ scal, int it) {
    if (tl_done(scal, it)) return;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= n) return;
    const TriCorner c = tri[t];
    const float* ya = y + (int64_t)blockIdx.y * nx * ny * nz;
    const int i0 = c.cell & 1023, j0 = (c.cell >> 10) & 1023, k0 = c.cell >> 20;
    const int i1 = wrap && i0 + 1 == nx ? 0 : i0 + 1, j1 = wrap && j0 + 1 == ny ? 0 : j0 + 1,
              k1 = wrap && k0 + 1 == nz ? 0 : k0 + 1;
    auto at = [&](int i, int j, int k) { return ya[((int64_t)k * ny + j) * nx + i]; };
    auto line = [&](int j, int k) { return (1.0f - c.f[0]) * at(i0, j, k) + c.f[0] * at(i1, j, k); };
    auto face = [&](int k) { return (1.0f - c.f[1]) * line(j0, k) + c.f[1] * line(j1, k); };
    yc[blockIdx.y * estr + t] = (1.0f - c.f[2]) * face(k0) + c.f[2] * face(k1);
}

// ------------------------------------------------------------ host tables
// One-dimensional problem on the lines x (periodic with period L): eigenvalues
// l and M-orthonormal eigenvectors V [n][n] of the linear-element stiffness
// against the lumped mass, by cyclic Jacobi rotations.
void line_eigen(const std::vector<double>& x, bool periodic, double L, std::vector<double>& l,
                std::vector<double>& V) {
    const int n = (int)x.size();
    std::vector<double> A((size_t)n * n, 0.0), M(n, 0.0);
    const int cells = periodic ? n : n - 1;
    for (int i = 0; i < cells; ++i) {
        const int j = (i + 1) % n;
        const double h = i + 1 < n ? x[i + 1] - x[i] : x[0] + L - x[i];
        M[i] += 0.5 * h;
        M[j] += 0.5 * h;
        A[i * n + i] += 1.0 / h;
        A[j * n + j] += 1.0 / h;
        A[i * n + j] -= 1.0 / h;
        A[j * n + i] -= 1.0 / h;
    }
    for (int i = 0; i < n; ++i)
        for (int j = 0; j < n; ++j) A[i * n + j] /= std::sqrt(M[i] * M[j]);
    V.assign((size_t)n * n, 0.0);     // rows are eigenvectors while rotating
    for (int i = 0; i < n; ++i) V[i * n + i] = 1.0;
    for (int sweep = 0; sweep < 30; ++sweep) {
        double off = 0.0, diag = 0.0;
        for (int i = 0; i < n; ++i)
            for (int j = 0; j < n; ++j) (i == j ? diag : off) += A[i * n + j] * A[i * n + j];
        if (off <= 1e-24 * (diag + off)) break;
        for (int p = 0; p < n; ++p)
            for (int q = p + 1; q < n; ++q) {
                const double apq = A[p * n + q];
                if (apq == 0.0) continue;
                const double th = (A[q * n + q] - A[p * n + p]) / (2.0 * apq);
                const double t = (th >= 0.0 ? 1.0 : -1.0) / (std::fabs(th) + std::sqrt(th * th + 1.0));
                const double c = 1.0 / std::sqrt(t * t + 1.0), s = t * c;
                for (int k = 0; k < n; ++k) {
                    const double u = A[p * n + k], v = A[q * n + k];
                    A[p * n + k] = c * u - s * v;
                    A[q * n + k] = s * u + c * v;
                }
                for (int k = 0; k < n; ++k) {
                    const double u = A[k * n + p], v = A[k * n + q];
                    A[k * n + p] = c * u - s * v;
                    A[k * n + q] = s * u + c * v;
                }
                for (int k = 0; k < n; ++k) {
                    const double u = V[p * n + k], v = V[q * n + k];
                    V[p * n + k] = c * u - s * v;
                    V[q * n + k] = s * u + c * v;
                }
            }
    }
    l.resize(n);
    std::vector<double> W((size_t)n * n);
    for (int k = 0; k < n; ++k) {
        l[k] = std::max(A[k * n + k], 0.0);
        for (int i = 0; i < n; ++i) W[i * n + k] = V[k * n + i] / std::sqrt(M[i]);
    }
    V.swap(W);
}

// A line of vertices in one direction: the values from lo to hi, no gap
// between neighbouring ones above tol.  A value joins every line within tol of
// it, so the outcome is the same in any order of the values, every value lies
// in its line, and the index found by line_of is that of a line whatever the
// coordinates' noise.
struct Line { double lo, hi; };
void join(std::vector<Line>& l, Line v, double tol) {
    const auto a = std::lower_bound(l.begin(), l.end(), v.lo - tol, [](const Line& q, double at) { return q.hi < at; });
    auto b = a;
    for (; b != l.end() && b->lo <= v.hi + tol; ++b) v = Line{std::min(v.lo, b->lo), std::max(v.hi, b->hi)};
    if (a == b) {
        l.insert(a, v);
    } else {
        *a = v;
        l.erase(a + 1, b);
    }
}
int line_of(const std::vector<Line>& l, double v) {
    const auto a = std::upper_bound(l.begin(), l.end(), v, [](double at, const Line& q) { return at < q.lo; });
    return std::max((int)(a - l.begin()) - 1, 0);
}

// the lines of coordinate d of the element corners (with a period, hi is
// identified with lo), empty past MAXN of them
std::vector<Line> lines_of(const stdg_mesh* m, int d, double lo, double hi, bool periodic, double tol) {
    std::vector<Line> x;
    bool many = false;
#pragma omp parallel
    {
        std::vector<Line> own;
#pragma omp for schedule(static)
        for (int64_t t = 0; t < m->E; ++t)
            for (int k = 0; k < 4 && (int)own.size() <= MAXN; ++k) {
                double v = (double)m->vert[t][k][d];
                if (periodic && std::fabs(v - hi) < tol) v = lo;
                join(own, Line{v, v}, tol);
            }
#pragma omp critical
        {
            many = many || (int)own.size() > MAXN;
            for (size_t i = 0; i < own.size() && !many; ++i) {
                join(x, own[i], tol);
                many = (int)x.size() > MAXN;
            }
        }
    }
    if (many) x.clear();
    return x;
}

// the host tables packed into one buffer, so that a mesh makes one
// allocation and one copy for them (pieces at 256-byte boundaries)
struct Pack {
    std::vector<char> host;
    template <typename T> size_t add(const std::vector<T>& v) {
        const size_t at = reserve(v.size() * sizeof(T));
        std::copy((const char*)v.data(), (const char*)(v.data() + v.size()), host.begin() + at);
        return at;
    }
    size_t reserve(size_t bytes) {
        const size_t at = host.size();
        host.resize(at + (bytes + 255) / 256 * 256);
        return at;
    }
};

}  // namespace

bool coarse_supported(const stdg_mesh* m) { return m->d.coarse.nodes > 0; }

// Grid, eigenvectors and the transfer tables of the second level (see the
// head of this file); nothing is built where the rule does not hold.
int upload_coarse(stdg_mesh* m) {
    CoarseTables& c = m->d.coarse;
    const int64_t E = m->E;
    double lo[3], hi[3], vol = 0.0;
    for (int d = 0; d < 3; ++d) { lo[d] = 1e300; hi[d] = -1e300; }
#pragma omp parallel for schedule(static) reduction(+ : vol) reduction(min : lo[:3]) reduction(max : hi[:3])
    for (int64_t t = 0; t < E; ++t) {
        const auto& v = m->vert[t];
        for (int k = 0; k < 4; ++k)
            for (int d = 0; d < 3; ++d) {
                lo[d] = std::min(lo[d], (double)v[k][d]);
                hi[d] = std::max(hi[d], (double)v[k][d]);
            }
        vol += std::fabs((double)det3(sub(v[1], v[0]), sub(v[2], v[0]), sub(v[3], v[0]))) / 6.0;
    }
    double L[3], box = 1.0;
    for (int d = 0; d < 3; ++d) box *= L[d] = hi[d] - lo[d];
    if (!(std::fabs(vol - box) <= 1e-9 * box)) return STDG_OK;
    const bool per = m->cfg.periodic != 0;
    const double h = std::cbrt(6.0 * vol / (double)E);
    std::vector<double> x[3];
    std::vector<Line> line[3];
    double tol[3];
    bool tensor = true;
    size_t nodes = 1;
    for (int d = 0; d < 3; ++d) {
        tol[d] = 1e-6 * std::min(h, L[d]);
        if (tensor) line[d] = lines_of(m, d, lo[d], hi[d], per, tol[d]);
        for (const Line& v : line[d]) x[d].push_back(v.lo + 0.5 * (v.hi - v.lo));
        tensor = tensor && !x[d].empty();
        nodes *= x[d].size();
    }
    // a tensor grid of vertices holds about one node per six elements; far
    // more lines than that belong to scattered vertices
    if (tensor && nodes > (size_t)E) tensor = false;
    for (int d = 0; d < 3; ++d) {
        if (!tensor) {
            const int cells = std::min(std::max(1, (int)std::llround(L[d] / h)), MAXN - 1);
            x[d].resize(per ? cells : cells + 1);
            for (size_t i = 0; i < x[d].size(); ++i) x[d][i] = lo[d] + L[d] * (double)i / cells;
        }
        if (x[d].size() < 2) return STDG_OK;
    }
    double narrow = 1e300, spread = 0.0;
    for (int d = 0; d < 3; ++d)
        for (size_t i = 0; i + 1 < x[d].size() + (per ? 1 : 0); ++i) {
            const double w = i + 1 < x[d].size() ? x[d][i + 1] - x[d][i] : x[d][0] + L[d] - x[d][i];
            narrow = std::min(narrow, w);
            spread = std::max(spread, w);
        }
    const Limits lim = limits(m);
    if (tensor && spread > lim.grading * narrow) return STDG_OK;
    const int n[3] = {(int)x[0].size(), (int)x[1].size(), (int)x[2].size()};
    const int G = m->G;
    const int64_t epad = (E + 63) / 64 * 64;
    // position of every corner
    std::vector<int32_t> corner(tensor ? 4 * epad : 0, 0);
    std::vector<TriCorner> tri(tensor ? 0 : 4 * epad);
    const int N3 = n[0] * n[1] * n[2];
    std::vector<int32_t> count(N3, 0);
    auto node = [&](int i, int j, int k) { return (k * n[1] + j) * n[0] + i; };
    auto visit = [&](int64_t c4, auto&& f) {
        if (tensor) { f(corner[c4], 1.0f); return; }
        const TriCorner& q = tri[c4];
        const int i0[3] = {q.cell & 1023, (q.cell >> 10) & 1023, q.cell >> 20};
        for (int s = 0; s < 8; ++s) {
            float w = 1.0f;
            int i[3];
            for (int d = 0; d < 3; ++d) {
                const int up1 = (s >> d) & 1;
                w *= up1 ? q.f[d] : 1.0f - q.f[d];
                i[d] = i0[d] + up1;
                if (per && i[d] == n[d]) i[d] = 0;
            }
            if (w != 0.0f) f(node(i[0], i[1], i[2]), w);
        }
    };
    double wide = 0.0;
#pragma omp parallel for schedule(static) reduction(max : wide)
    for (int64_t t = 0; t < E; ++t) {
        double first[3], last[3];
        for (int k = 0; k < 4; ++k) {
            int i0[3];
            float f[3];
            double pos[3];      // in cells, a period not wrapped
            for (int d = 0; d < 3; ++d) {
                const double v = (double)m->vert[t][k][d];
                if (tensor) {
                    const bool up = per && std::fabs(v - hi[d]) < tol[d];
                    i0[d] = up ? 0 : line_of(line[d], v);
                    pos[d] = up ? n[d] : i0[d];
                } else {
                    const int cells = per ? n[d] : n[d] - 1;
                    const double s = (v - lo[d]) / L[d] * cells;
                    i0[d] = std::min(std::max((int)std::floor(s), 0), cells - 1);
                    f[d] = (float)std::min(std::max(s - i0[d], 0.0), 1.0);
                    pos[d] = s;
                }
                first[d] = k > 0 ? std::min(first[d], pos[d]) : pos[d];
                last[d] = k > 0 ? std::max(last[d], pos[d]) : pos[d];
            }
            if (tensor) corner[4 * t + k] = node(i0[0], i0[1], i0[2]);
            else tri[4 * t + k] = TriCorner{i0[0] | (i0[1] << 10) | (i0[2] << 20), {f[0], f[1], f[2]}};
        }
        for (int d = 0; d < 3; ++d) wide = std::max(wide, last[d] - first[d]);
    }
    if (wide > lim.width) return STDG_OK;
    for (int64_t c4 = 0; c4 < 4 * E; ++c4) visit(c4, [&](int j, float) { ++count[j]; });
    std::vector<int64_t> row(tensor ? 0 : N3 + 1, 0);
    int K = 0;
    size_t entries = 0;
    if (tensor) {
        K = (*std::max_element(count.begin(), count.end()) + RL1 - 1) / RL1 * RL1;
        entries = (size_t)K * N3;
        // a node that many more corners reach than others (2 on a cube of 4^3
        // hexahedra with walls)
        if (entries > 8 * (size_t)(4 * E)) return STDG_OK;
    } else {
        for (int j = 0; j < N3; ++j) row[j + 1] = row[j] + count[j];
        entries = (size_t)row[N3];
    }
    std::vector<int32_t> slot(entries, -1);
    std::vector<float> wgt(tensor ? 0 : entries, 0.0f);
    std::fill(count.begin(), count.end(), 0);
    for (int64_t c4 = 0; c4 < 4 * E; ++c4)
        visit(c4, [&](int j, float w) {
            const size_t at = (tensor ? (size_t)j * K : (size_t)row[j]) + count[j];
            slot[at] = (int32_t)c4;
            if (!tensor) wgt[at] = w;
            ++count[j];
        });
    // one-dimensional eigenproblems (equal lines share one)
    std::vector<double> l[3], V[3];
    std::vector<float> lam, mats[3], matsT[3];
    double top = 0.0;
    for (int d = 0; d < 3; ++d) {
        int same = -1;
        for (int o = 0; o < d; ++o) {
            bool eq = n[o] == n[d];
            for (int i = 0; eq && i < n[d]; ++i) eq = std::fabs((x[d][i] - lo[d]) - (x[o][i] - lo[o])) <= tol[d];
            if (eq && std::fabs(L[o] - L[d]) <= tol[d]) same = o;
        }
        if (same >= 0) { l[d] = l[same]; V[d] = V[same]; }
        else line_eigen(x[d], per, L[d], l[d], V[d]);
        const int pd = pad16(n[d]);
        mats[d].assign((size_t)pd * pd, 0.0f);
        matsT[d].assign((size_t)pd * pd, 0.0f);
        for (int i = 0; i < n[d]; ++i)
            for (int k = 0; k < n[d]; ++k) {
                mats[d][i * pd + k] = (float)V[d][i * n[d] + k];
                matsT[d][k * pd + i] = (float)V[d][i * n[d] + k];
            }
        double mx = 0.0;
        for (double v : l[d]) { lam.push_back((float)v); mx = std::max(mx, v); }
        top += mx;
    }
    double low = top;       // smallest non-zero eigenvalue; half of it separates the constant mode
    for (int d = 0; d < 3; ++d)
        for (double v : l[d])
            if (v > 1e-8 * top) low = std::min(low, v);
    c.cut = (float)(0.5 * low);
    c.scale = (float)(1.0 / (m->cfg.dt * m->cfg.dt));
    c.n[0] = n[0]; c.n[1] = n[1]; c.n[2] = n[2];
    c.per = per ? 1 : 0;
    c.K = K;
    c.epad = epad;
    Pack pk;
    size_t at[15];
    for (int d = 0; d < 3; ++d) {
        at[d] = pk.add(mats[d]);
        at[3 + d] = pk.add(matsT[d]);
    }
    at[6] = pk.add(lam);
    at[7] = pk.add(slot);
    at[8] = tensor ? pk.add(corner) : pk.add(tri);
    at[9] = tensor ? 0 : pk.add(wgt);
    at[14] = tensor ? 0 : pk.add(row);
    const size_t copied = pk.host.size();
    // work vectors after the tables
    size_t end = copied;
    auto room = [&](size_t bytes) {
        const size_t o = end;
        end += (bytes + 255) / 256 * 256;
        return o;
    };
    at[10] = room(sizeof(float) * 4 * epad * G);
    at[11] = room(sizeof(float) * (size_t)N3 * G);
    at[12] = room(sizeof(float) * (size_t)N3 * G);
    at[13] = room(sizeof(double) * (size_t)((n[0] * n[1] + CC - 1) / CC) * G);
    const size_t yc = room(tensor ? 0 : sizeof(float) * 4 * epad * G);
    STDG_HIP(hipMalloc(&c.base, end));
    STDG_HIP(hipMemcpy(c.base, pk.host.data(), copied, hipMemcpyHostToDevice));
    char* base = (char*)c.base;
    for (int d = 0; d < 3; ++d) {
        c.V[d] = (float*)(base + at[d]);
        c.VT[d] = (float*)(base + at[3 + d]);
    }
    c.lam = (float*)(base + at[6]);
    c.slot = (int32_t*)(base + at[7]);
    if (tensor) {
        c.corner = (int32_t*)(base + at[8]);
    } else {
        c.tri = base + at[8];
        c.wgt = (float*)(base + at[9]);
        c.row = (int64_t*)(base + at[14]);
        c.yc = (float*)(base + yc);
    }
    c.e4 = (float*)(base + at[10]);
    c.g = (float*)(base + at[11]);
    c.t = (float*)(base + at[12]);
    c.part = (double*)(base + at[13]);
    c.nodes = N3;
    return STDG_OK;
}

void free_coarse(stdg_mesh* m) {
    CoarseTables& c = m->d.coarse;
    if (c.base) (void)hipFree(c.base);
    c = CoarseTables();
}

namespace {
bool small_grid(const CoarseTables& c) {
    return c.nodes <= SMALL_NODES && std::max({c.n[0], c.n[1], c.n[2]}) <= SMALL_LINES;
}

template <int T> void plane(const CoarseTables& c, int G, bool fwd, const double* scal, int it, hipStream_t s) {
    float* const* V = fwd ? c.V : c.VT;
    hipLaunchKernelGGL(k_plane<T>, dim3(c.n[2] * G), dim3(plane_threads<T>()), 0, s, fwd ? c.g : c.t, fwd ? c.t : c.g,
                       V[0], V[1], c.n[0], c.n[1], scal, it);
}
template <int T> void columns(const CoarseTables& c, int G, const double* scal, int it, hipStream_t s) {
    hipLaunchKernelGGL(k_columns<T>, dim3((c.n[0] * c.n[1] + CC - 1) / CC, G), dim3(column_threads<T>()), 0, s, c.t,
                       c.V[2], c.VT[2], c.lam, c.n[0], c.n[1], c.n[2], c.scale, c.cut, c.part, scal, it);
}
// f of the number of 16-line pads of n lines (up to MAXN)
#define STDG_PADS(n, f, ...)                   \
    switch (((n) + 15) / 16) {                 \
        case 1: f<1>(__VA_ARGS__); break;      \
        case 2: f<2>(__VA_ARGS__); break;      \
        case 3: f<3>(__VA_ARGS__); break;      \
        case 4: f<4>(__VA_ARGS__); break;      \
        default: f<5>(__VA_ARGS__); break;     \
    }
}  // namespace

int coarse_partials(const stdg_mesh* m) {
    const CoarseTables& c = m->d.coarse;
    return small_grid(c) ? m->G : (c.n[0] * c.n[1] + CC - 1) / CC * m->G;
}

// corner sums c.e4 -> K P^T r on the grid (c.g) and, off the grid, at the
// corners (c.yc); the dot (P^T r) . K (P^T r) in c.part
hipError_t coarse_solve(const stdg_mesh* m, const double* scal, int it, hipStream_t s) {
    const CoarseTables& c = m->d.coarse;
    const int G = m->G, nx = c.n[0], ny = c.n[1], nz = c.n[2];
    const int64_t estr = 4 * c.epad;
    const bool small = small_grid(c), gather = small && !c.wgt && c.nodes <= SMALL_GATHER;
    const dim3 rgrid((unsigned)(((int64_t)c.nodes * (c.wgt ? RLW : RL1) + 255) / 256), G);
    if (c.wgt)
        hipLaunchKernelGGL(k_restrict<true>, rgrid, dim3(256), 0, s, c.slot, c.wgt, c.row, c.K, c.e4, estr, c.g, c.nodes,
                           scal, it);
    else if (!gather)
        hipLaunchKernelGGL(k_restrict<false>, rgrid, dim3(256), 0, s, c.slot, c.wgt, c.row, c.K, c.e4, estr, c.g, c.nodes,
                           scal, it);
    if (small) {
        // (a thread per node)
        const bool few = c.nodes <= SMALL_GATHER;
        hipLaunchKernelGGL((gather ? k_small<true, SMALL_GATHER>
                                   : (few ? k_small<false, SMALL_GATHER> : k_small<false, SMALL_NODES>)),
                           dim3(G), dim3(few ? SMALL_GATHER : SMALL_NODES), 0, s, c.slot, c.K, c.e4, estr, c.g,
                           c.V[0], c.V[1], c.V[2], c.lam, nx, ny, nz, c.scale, c.cut, c.part, scal, it);
    } else {
        STDG_PADS(std::max(nx, ny), plane, c, G, true, scal, it, s)
        STDG_PADS(nz, columns, c, G, scal, it, s)
        STDG_PADS(std::max(nx, ny), plane, c, G, false, scal, it, s)
    }
    if (c.tri)
        hipLaunchKernelGGL(k_corners, dim3((unsigned)((4 * m->E + 255) / 256), G), dim3(256), 0, s,
                           (const TriCorner*)c.tri, c.g, c.yc, 4 * m->E, estr, nx, ny, nz, c.per, scal, it);
    return hipGetLastError();
}

}  // namespace stdg
