// Small dense blocks on the FP64 matrix cores: v_mfma_f64_4x4x4f64 runs four
// independent 4 x 4 x 4 products (blocks b = 0..3); lane 16 k + 4 b + i holds
// A_b[i][k], lane 16 k + 4 b + j holds B_b[k][j], and D_b[i][j] lands in lane
// 16 i + 4 b + j.  A wavefront takes 16 columns (entities), column 4 b + j in
// lanes 16 k + 4 b + j for every k; the A operand is the same in the four
// blocks.  A column's N values are contracted in NQ steps of four; which four
// is free, and the even-odd pairs of m64_col let a lane load two neighbouring
// values with one 16-byte load (four lanes of a column 64 contiguous bytes)
// where one value per step would take two 8-byte ones.  A result row 4 rg +
// hi (hi = lane / 16) of a column sits in the lane that holds contraction
// index hi of that column, so a result is the B operand of a further product
// as it stands (its steps then take the rows in natural order).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace stdg {

typedef double m64_d2 __attribute__((ext_vector_type(2)));

// byte offset past every buffer (loads give 0) that a row's length does not wrap
constexpr uint32_t M64_OOB = 0xFFFF0000u;

// A group of entities that share their blocks (Mesh tables `segs`,
// `face_groups`): x the first, y their number (up to 64), z (and w) the blocks.
typedef int m64_i4 __attribute__((ext_vector_type(4)));

// workgroup -> group, consecutive ones on one XCD (grids are multiples of 8)
__device__ inline uint32_t m64_group(uint32_t blocks) { return (blockIdx.x % 8) * (blocks / 8) + blockIdx.x / 8; }
inline unsigned m64_blocks(int64_t groups) { return (unsigned)((groups + 7) / 8 * 8); }

template <int N> struct M64 {
    static constexpr int NQ = (N + 3) / 4;      // contraction steps and row groups
    static constexpr int NP = 4 * NQ;           // padded rows
    static constexpr int S8 = N / 8;            // pairs of steps loaded 16 bytes at a time
};

__device__ inline __amdgpu_buffer_rsrc_t m64_rsrc(const double* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(p), (short)0, (int)bytes, 0x00020000);
}

// column of the block that step t of lane group hi multiplies (clamped where
// the step is padding: the B value there is zero)
template <int N> __device__ inline int m64_col(int t, int hi) {
    constexpr int S8 = M64<N>::S8;
    const int c = t < 2 * S8 ? 8 * (t / 2) + 2 * hi + (t & 1) : 8 * S8 + 4 * (t - 2 * S8) + hi;
    return c < N ? c : N - 1;
}

// the lane's share of the row of N values at byte offset `off` (M64_OOB: zeros)
template <int N> __device__ inline void m64_load(__amdgpu_buffer_rsrc_t r, uint32_t off, int hi, double (&b)[M64<N>::NQ]) {
    constexpr int S8 = M64<N>::S8, NQ = M64<N>::NQ;
#pragma unroll
    for (int s = 0; s < S8; ++s) {
        const m64_d2 v = __builtin_bit_cast(
            m64_d2, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(off + 16u * (uint32_t)hi), 64 * s, 0));
        b[2 * s] = v.x;
        b[2 * s + 1] = v.y;
    }
#pragma unroll
    for (int t = 2 * S8; t < NQ; ++t) {
        const int c = 8 * S8 + 4 * (t - 2 * S8) + hi;
        b[t] = __builtin_bit_cast(
            double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)(c < N ? off + 8u * (uint32_t)c : M64_OOB), 0, 0));
    }
}

// acc[rg][c] += block times column c: the block in LDS, [column][NP rows]
template <int N, int NC>
__device__ __forceinline__ void m64_block(const double* A, const double (&b)[NC][M64<N>::NQ], int lo, int hi,
                                          double (&acc)[M64<N>::NQ][NC]) {
    constexpr int NQ = M64<N>::NQ, NP = M64<N>::NP;
#pragma unroll
    for (int t = 0; t < NQ; ++t) {
        const double* col = A + m64_col<N>(t, hi) * NP + lo;
#pragma unroll
        for (int rg = 0; rg < NQ; ++rg) {
            const double av = col[4 * rg];
#pragma unroll
            for (int c = 0; c < NC; ++c) acc[rg][c] = __builtin_amdgcn_mfma_f64_4x4x4f64(av, b[c][t], acc[rg][c], 0, 0, 0);
        }
    }
}

// nb blocks [N columns][N rows] of src into LDS [N][NP], padded rows zero, by
// a workgroup of T threads
template <int N, int T> __device__ inline void m64_stage(const double* __restrict__ src, double* A, int nb) {
    constexpr int NP = M64<N>::NP;
    for (int t = threadIdx.x; t < nb * N * NP; t += T) {
        const int r = t % NP, c = t / NP;
        A[t] = r < N ? src[c * N + r] : 0.0;
    }
}

// Results of 16 consecutive entities (columns) back to memory: the wavefront's
// rows [entity][time node][N] of one component are contiguous, so they pass
// through its own LDS slice `buf` (16 G N doubles) and leave as 16-byte
// stores of consecutive lanes; straight from the accumulators every store
// instruction would touch 16 rows, 32 bytes each (goback, 663,552 elements,
// p = 3: 465 -> 445 us, the preconditioned viscous operator 340 -> 317).  value(rg, a) is the lane's result row 4 rg + hi at
// time node a; out(i, v) takes the two values at offset i of the component
// (relative to the first entity), of which those below `count` exist.  EN
// entities pass at a time (buf: EN G N doubles).
typedef double m64_d2u __attribute__((ext_vector_type(2), aligned(8)));   // rows start at any multiple of 8 bytes
template <int N, int G, int EN = 16, typename V, typename O>
__device__ __forceinline__ void m64_flush(double* buf, int lane, int hi, int count, V&& value, O&& out) {
    constexpr int NQ = M64<N>::NQ, TOT = EN * G * N;
    static_assert(EN == 16 || TOT % 2 == 0, "pairs within a part");
    // (lanes of absent entities write too; their values are not read)
    double* row = buf + (lane & (EN - 1)) * (G * N);
#pragma unroll
    for (int part = 0; part < 16 / EN; ++part) {
        if (EN == 16 || (lane & 15) / EN == part)
#pragma unroll
            for (int a = 0; a < G; ++a)
#pragma unroll
                for (int rg = 0; rg < NQ; ++rg)
                    if (4 * rg + hi < N) row[a * N + 4 * rg + hi] = value(rg, a);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int left = count - part * TOT;
#pragma unroll
        for (int i0 = 0; i0 < TOT; i0 += 128) {
            const int i = i0 + 2 * lane;
            if (i < left && i < TOT) out(part * TOT + i, m64_d2u{buf[i], buf[i + 1 < TOT ? i + 1 : i]});
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// store of m64_flush's pair at y + i
__device__ __forceinline__ void m64_put(double* y, int i, int count, m64_d2u v) {
    if (i + 1 < count) *reinterpret_cast<m64_d2u*>(y + i) = v;
    else y[i] = v.x;
}

}  // namespace stdg
