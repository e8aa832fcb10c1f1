// Device helpers shared by the HIP sources of the library (internal).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace bddc {
namespace dev {

// Cross-lane moves without LDS: DPP within rows of 16 lanes, and the gfx950
// row-swap permutes across rows.  Every lane of the wave must be active.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
constexpr int DPP_XOR1 = 0xB1;      // quad_perm [1,0,3,2]
constexpr int DPP_XOR2 = 0x4E;      // quad_perm [2,3,0,1]
constexpr int DPP_HALF_MIRROR = 0x141;  // lane i <-> i ^ 7 within 8 lanes
constexpr int DPP_ROR4 = 0x124;     // row_ror:4 within 16 lanes
constexpr int DPP_ROR8 = 0x128;     // lane i <-> i ^ 8 within 16 lanes

// v + v[l ^ 16], v + v[l ^ 32]
__device__ __forceinline__ float add_xor16(float v) {
    auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
__device__ __forceinline__ float add_xor32(float v) {
    auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
__device__ __forceinline__ double add_xor16(double v) {
    auto l = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    auto h = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
}
__device__ __forceinline__ double add_xor32(double v) {
    auto l = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
}

// Sum over the 16 lanes of a row in the order of an xor butterfly 8, 4, 2, 1
// (after the first step lanes l and l ^ 8 hold the same value, so the rotation
// by 4 is the exchange with l ^ 4).  An LDS permute a step (__shfl_xor) costs a
// round trip through LDS each; these stay in the vector pipe and take fewer
// registers (64^3: float64 Neumann product 50.2 -> 45.8 us, update 7.1 -> 6.3,
// direction update 11.5 -> 10.6; 16^3 sequence of 10: 4.92 -> 4.42 ms).
template <typename T>
__device__ __forceinline__ T row16_sum(T v) {
    v += dpp<DPP_ROR8>(v);
    v += dpp<DPP_ROR4>(v);
    v += dpp<DPP_XOR2>(v);
    v += dpp<DPP_XOR1>(v);
    return v;
}

// Sum over the wave in the order of an xor butterfly 32, 16, ..., 1.
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
    return row16_sum(add_xor16(add_xor32(v)));
}

// Sum over the block (every thread gets the result); sh holds >= 16 doubles.
__device__ __forceinline__ double block_sum(double v, double *sh) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, nw = blockDim.x >> 6;
    __syncthreads();
    if (l == 0) sh[w] = v;
    __syncthreads();
    double t = 0.0;
    for (int i = 0; i < nw; ++i) t += sh[i];
    __syncthreads();
    return t;
}

// Per-thread part of a contiguous sum: element i goes to thread i % nthr,
// four independent accumulators so that the loads are issued together.
__device__ __forceinline__ double strided_part(const double *p, int n, int t, int nthr) {
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int i = t;
    for (; i + 3 * nthr < n; i += 4 * nthr) {
        s0 += p[i];
        s1 += p[i + nthr];
        s2 += p[i + 2 * nthr];
        s3 += p[i + 3 * nthr];
    }
    for (; i < n; i += nthr) s0 += p[i];
    return (s0 + s1) + (s2 + s3);
}

// Sum of p[0..n) by one wave in a fixed order: every wave that calls it gets
// the same value.
__device__ __forceinline__ double wave_sum_contig(const double *p, int n) {
    return wave_sum(strided_part(p, n, threadIdx.x & 63, 64));
}

// Sum of p[0..n) by the whole block in a fixed order (every thread gets it).
__device__ __forceinline__ double block_sum_contig(const double *p, int n, double *sh) {
    return block_sum(strided_part(p, n, threadIdx.x, blockDim.x), sh);
}

// Block-wide sums of the per-thread values acc[0..ncol) (ncol <= NC, a block
// of exactly 256 threads): 16 columns at a time are transposed through LDS
// (lds: 16 * 256 doubles), thread (u, j) adds the entries j, j + 16, ... of
// column u (consecutive lanes read consecutive words) and a sum over 16 lanes
// finishes; res[q] (LDS, NC doubles) receives column q.  Fixed
// order; every thread may read res after the call.
template <int NC>
__device__ __forceinline__ void block_sum_cols(const double (&acc)[NC], int ncol, double *lds, double *res) {
    const int t = threadIdx.x, u = t >> 4, j = t & 15;
#pragma unroll
    for (int q0 = 0; q0 < NC; q0 += 16) {
        if (q0 < ncol) {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (q0 + v < NC) lds[v * 256 + t] = acc[q0 + v < NC ? q0 + v : 0];
            __syncthreads();
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < 16; ++i) s += lds[u * 256 + i * 16 + j];
            s = row16_sum(s);
            if (j == 0 && q0 + u < ncol) res[q0 + u] = s;
            __syncthreads();
        }
    }
}

__device__ __forceinline__ float bf16_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

// Q1 reference stiffness on the unit cube: 1/3 on the diagonal, 0 between
// vertices differing in one coordinate, -1/12 otherwise.
__device__ __forceinline__ double kref_entry(int v, int w) {
    const int nd = __popc(v ^ w);
    return nd == 0 ? (1.0 / 3.0) : (nd == 1 ? 0.0 : (-1.0 / 12.0));
}

}  // namespace dev
}  // namespace bddc
