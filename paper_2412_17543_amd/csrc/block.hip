// Block products of the block adjoint and of grouped condensation (several
// right-hand sides at once): the batched symmetric products y_i = S_i x_i
// (Schur), u_i = D N_i D g_i (Neumann, eq. localCorr, with the coarse
// restriction (D Phi_i)^T g_i of eq. coarse_problem) or K_II^{-1} b_i
// (interior), 16 columns at a time, on the matrix cores, and the assembly of
// the per-subdomain results.
//
// k_symm: one block of 8 waves per (subdomain, 16-column chunk).  Wave w owns
// the tile columns J = w, w + 8, ... (NJ of them) and keeps their results Y_J
// in MFMA registers; the block walks the packed upper-triangle tiles one tile
// row I at a time, each wave its own columns J >= I:
//   column part Y_J += T^T X_I, J > I  (in the wave's registers: with k-slot g
//               of step s standing for row 4 g + s, the tile's storage layout,
//               tile_index, is the operand as loaded)
//   row part    Y_I += T X_J           (the tile transposed through the wave's
//               LDS slot; the waves' sums are added in wave order by the wave
//               that owns column I)
// so every entry is summed in a fixed order (the product is reproducible bit
// by bit) and LDS carries one write and one read of a tile, X (staged in
// operand order) and 8 partial tiles a row.  Each column's next tile, one row
// down, is requested as soon as the current one is used: NJ tiles in flight a
// wave, in registers (but NJ = 4, of the 128 registers that two blocks leave a
// lane, passes one column's tile through scratch in the first 8 tile rows; NJ = 3
// keeps an index or two there, NJ = 5 has registers enough).  One variant serves
// all subdomains of a launch, the one that the largest needs.  A short ragged
// tail stored as a strip after the tiles (uses_strip) follows as one more tile
// row.
// What bounds it: the matrix cores, 8 v_mfma_f64_16x16x4f64 a tile and chunk
// (about 70 cycles each: 0.21 ms for the 0.46 M tiles of 96^3 and two chunks;
// the tiles' bytes take 0.15 ms).  Two blocks a compute unit (at most 80 KB of
// LDS, 128 registers) cover each other's row ends.  Measured at 96^3, 20 columns:
// 0.83 -> 0.42 ms a product in two chunks, against 4 waves, X and Y in 126 KB of
// LDS and both parts read back through it (block adjoint 65.0 -> 47.1 ms); 0.32
// with the last four columns beside the first 16 (X4).
// v_mfma_f64_16x16x4f64 takes A[i][k] and B[k][j] in lane i (j) + 16 k and
// returns (i, j) in lane j + 16 (i % 4), register i / 4.
#include <hip/hip_runtime.h>

#include "internal.h"
#include "kernels.h"

namespace bddc {

namespace {

typedef double dvec4 __attribute__((ext_vector_type(4)));
typedef double dvec2 __attribute__((ext_vector_type(2)));

constexpr int NW = 8;               // waves of a block

// Workgroup barrier that orders LDS only: the tile loads in flight are not
// waited for (a plain __syncthreads() would drain them at every row end).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

typedef unsigned int uvec4 __attribute__((ext_vector_type(4)));

// Raw buffer over `bytes` bytes from p: loads at or past the end return zero
// without a memory access.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_rsrc(const void *p, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)min(bytes, (int64_t)INT32_MAX), 0x00020000);
}

// Two blocks per compute unit (4 waves per SIMD) up to NJ = 4.
// X4: 16 + 4 columns in one block, for 17 to 20 columns.  The tile, its transpose
// and its row end then serve all of them, and the four go through
// v_mfma_f64_4x4x4f64 (four blocks of 4 rows; A as above, B[k][j] in lane
// j + 16 k of every block's lanes, (i, j) of block m returned in lane
// 4 m + j + 16 i): 9 ns a step and SIMD against 28, where a second chunk would
// take 28 for 16 columns of which 12 are none.  96^3, 20 columns: 0.42 -> 0.32 ms
// a product, block adjoint 34.5 -> 30.2 ms.  It covers 17 to 20 columns only: a
// product takes 0.25 ms for 1 to 16, 0.32 to 20, then 0.44 (21) to 0.45 (32) in two
// chunks.
__device__ __forceinline__ double mfma4(double a, double b, double c) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

template <int NJ, bool X4>
__global__ void __launch_bounds__(NW * 64, NJ <= 4 ? 4 : 2) k_symm(BlockSymvArgs a, int nsub) {
    extern __shared__ __align__(16) double sm[];
    // the column chunks of one subdomain are 8 blocks apart: the same XCD takes
    // them at the same time, so the second reads the tiles from its L2
    constexpr int W = X4 ? 20 : 16;                    // columns of a block
    const int nch = X4 ? 1 : (a.ncols + 15) / 16;
    int sub, chunk;
    {
        const int b = blockIdx.x, grp = b / (8 * nch), q = b - grp * 8 * nch, m = min(8, nsub - 8 * grp);
        sub = 8 * grp + q % m;
        chunk = q / m;
    }
    const BlockItem it = a.items[sub];
    const int c0 = 16 * chunk;
    const int n = it.n;
    const int nt = tile_rows(n), npad = 16 * ((n + 15) / 16);   // nt: tile rows (without a strip's rows)
    const int64_t total = full_tiles(n);
    double *xs = sm;                                   // X in operand order: [tile][s][lane]
    double *ts = xs + (size_t)npad * 16;               // per wave one 16 x 16 tile
    double *x4 = ts + NW * 256;                        // the last four columns: [tile][s][k][column]
    const int tid = threadIdx.x, L = tid & 63, li = L & 15, lk = L >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t *gb = a.gB + it.xoff;
    // the wave's tiles of row 0, requested before anything else; tile (I, J)
    // is number S(I) + J of the packed sequence, S(I + 1) = S(I) + nt - I - 1
    const __amdgpu_buffer_rsrc_t rs = raw_rsrc(a.tiles + it.tile * 256, total * 2048);
    const int end = (int)total * 2048;
    uvec4 fa[NJ], fb[NJ];
    auto request = [&](int jj, int I, int S) {         // (past the triangle: zeros, no access)
        const int J = jj * NW + w;
        const int off = (J < nt && J >= I ? (S + J) * 2048 : end) + L * 16;
        fa[jj] = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
        fb[jj] = __builtin_amdgcn_raw_buffer_load_b128(rs, off + 1024, 0, 0);
    };
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) request(jj, 0, 0);
    // X_i: 8 entries per thread at a time, all index loads before the gathers
    for (int e0 = tid; e0 < W * npad; e0 += NW * 64 * 8) {
        int gi[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = e0 + NW * 64 * u, cc = e / npad, k = e - cc * npad;
            gi[u] = (e < W * npad && k < n && c0 + cc < a.ncols) ? gb[k] : -1;
        }
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = e0 + NW * 64 * u, cc = e / npad;
            v[u] = gi[u] >= 0 ? a.X[(int64_t)(c0 + cc) * a.ldx + gi[u]] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = e0 + NW * 64 * u, cc = e / npad, k = e - cc * npad;
            if (X4 && cc >= 16) {
                if (e < W * npad) x4[(k >> 4) * 64 + (k & 3) * 16 + 4 * ((k & 15) >> 2) + cc - 16] = v[u];
            } else if (e < W * npad) {
                xs[(k >> 4) * 256 + (k & 3) * 64 + cc + 16 * ((k & 15) >> 2)] = v[u];
            }
        }
    }
    __syncthreads();
    double *tw = ts + w * 256;
    // entry (r, c) of the transposed tile at 16 p(r) + (c ^ (r & 11)), p swapping
    // bits 0 and 2: both the writes (lanes c, rows 4 lk + s) and the reads
    // (lanes r, columns 4 lk + s) touch every bank once
    const int wb = 16 * (((lk & 2) << 2) | (lk & 1)) + (li ^ ((lk & 2) << 2));
    const int rb = 16 * ((li & 10) | ((li & 1) << 2) | ((li >> 2) & 1)) + ((4 * lk) ^ (li & 11));
    auto transpose = [&](const double (&t)[4], double (&u)[4]) {
        wave_sync();                                   // the previous tile is read
#pragma unroll
        for (int s = 0; s < 4; ++s) tw[(wb ^ s) + 16 * ((s & 2) | ((s & 1) << 2))] = t[s];
        wave_sync();
#pragma unroll
        for (int s = 0; s < 4; ++s) u[s] = tw[rb ^ s];
    };
    const dvec4 zero = {0.0, 0.0, 0.0, 0.0};
    const int x4l = 4 * lk + (li & 3);                 // the lane's entry of a step's four columns
    const int r4 = 4 * (li >> 2) + lk;                 // row of the lane's result
    // Coarse restriction c_i = (D Phi_i)^T X_i from the staged X, 16 coarse DOFs
    // at a time: wave w takes the 16-row tiles w, w + 8, ..., U of them
    // requested together (four consecutive entries of a DOF's row a lane, the
    // steps' operands as loaded), the waves' sums added in wave order.
    if (a.phir) {
        constexpr int U = 4;
        const int nci = a.nc[sub], ldp = phi_ld(n), tt = npad / 16, pend = nci * ldp * 8;
        const __amdgpu_buffer_rsrc_t pr = raw_rsrc(a.phir + a.phr_off[sub], pend);
        for (int q0 = 0; q0 < nci; q0 += 16) {
            dvec4 acc = zero;
            double acc4 = 0.0;
            for (int t0 = w; t0 < tt; t0 += NW * U) {
                uvec4 pa[U], pb[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int t = t0 + NW * u, k = 16 * t + 4 * lk;
                    const int off = t < tt && k < ldp && q0 + li < nci ? ((q0 + li) * ldp + k) * 8 : pend;
                    pa[u] = __builtin_amdgcn_raw_buffer_load_b128(pr, off, 0, 0);
                    pb[u] = __builtin_amdgcn_raw_buffer_load_b128(pr, off + 16, 0, 0);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int t = t0 + NW * u;
                    if (t < tt) {                      // (wave-uniform)
                        const double v[4] = {__hiloint2double(pa[u].y, pa[u].x), __hiloint2double(pa[u].w, pa[u].z),
                                             __hiloint2double(pb[u].y, pb[u].x), __hiloint2double(pb[u].w, pb[u].z)};
#pragma unroll
                        for (int s = 0; s < 4; ++s) {
                            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(v[s], xs[t * 256 + s * 64 + L], acc, 0, 0, 0);
                            if constexpr (X4) acc4 = mfma4(v[s], x4[t * 64 + s * 16 + x4l], acc4);
                        }
                    }
                }
                // (a tile past the last: its zero read is not left outstanding)
#pragma unroll
                for (int u = 0; u < U; ++u) asm volatile("" ::"v"(pa[u]), "v"(pb[u]));
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) tw[r * 64 + L] = acc[r];
            lds_barrier();
            if (tid < 256) {
                double v = ts[tid];
#pragma unroll
                for (int q = 1; q < NW; ++q) v += ts[q * 256 + tid];
                const int q = q0 + lk + 4 * w, col = c0 + li;      // (w = tid / 64 < 4: register of the result)
                if (q < nci && col < a.ncols) a.cpart[(int64_t)col * a.cs + a.c_off[sub] + q] = v;
            }
            lds_barrier();
            if constexpr (X4) {
                tw[L] = acc4;
                lds_barrier();
                if (tid < 64) {
                    double v = ts[tid];
#pragma unroll
                    for (int q = 1; q < NW; ++q) v += ts[q * 256 + tid];
                    const int q = q0 + r4, col = c0 + 16 + (li & 3);
                    if (q < nci && col < a.ncols) a.cpart[(int64_t)col * a.cs + a.c_off[sub] + q] = v;
                }
                lds_barrier();
            }
        }
    }
    dvec4 yacc[NJ], racc = zero;
    double yacc4[NJ], racc4 = 0.0;
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) { yacc[jj] = zero; yacc4[jj] = 0.0; }
    // the waves' row parts, in wave order, in the registers of wave `owner`
    auto row_sum = [&](int owner, dvec4 &y, double &y4) {
        wave_sync();
#pragma unroll
        for (int r = 0; r < 4; ++r) tw[r * 64 + L] = racc[r];
        lds_barrier();
        if (w == owner) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double v = ts[r * 64 + L];
#pragma unroll
                for (int q = 1; q < NW; ++q) v += ts[q * 256 + r * 64 + L];
                y[r] += v;
            }
        }
        lds_barrier();
        racc = zero;
        if constexpr (X4) {
            tw[L] = racc4;
            lds_barrier();
            if (w == owner) {
                double v = ts[L];
#pragma unroll
                for (int q = 1; q < NW; ++q) v += ts[q * 256 + L];
                y4 += v;
            }
            lds_barrier();
            racc4 = 0.0;
        }
    };
    int S = 0;
#pragma unroll
    for (int ib = 0; ib < NJ; ++ib) {
        for (int wi = 0; wi < NW; ++wi) {
            const int I = ib * NW + wi;
            if (I >= nt) break;
            double xi[4], xi4[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                xi[s] = xs[I * 256 + s * 64 + L];
                xi4[s] = X4 ? x4[I * 64 + s * 16 + x4l] : 0.0;
            }
            const int Sn = S + nt - I - 1;
#pragma unroll
            for (int jj = ib; jj < NJ; ++jj) {
                const int J = jj * NW + w;
                const bool live = J < nt && J >= I;    // (wave-uniform)
                double t[4] = {__hiloint2double(fa[jj].y, fa[jj].x), __hiloint2double(fa[jj].w, fa[jj].z),
                               __hiloint2double(fb[jj].y, fb[jj].x), __hiloint2double(fb[jj].w, fb[jj].z)};
                double u[4];
                if (live) {
                    transpose(t, u);
                    if (J > I) {
#pragma unroll
                        for (int s = 0; s < 4; ++s) {
                            yacc[jj] = __builtin_amdgcn_mfma_f64_16x16x4f64(t[s], xi[s], yacc[jj], 0, 0, 0);
                            if constexpr (X4) yacc4[jj] = mfma4(t[s], xi4[s], yacc4[jj]);
                        }
                    }
                }
                // on every path, so that the number of loads in flight is known
                request(jj, I + 1, Sn);
                if (live) {
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        racc = __builtin_amdgcn_mfma_f64_16x16x4f64(u[s], xs[J * 256 + s * 64 + L], racc, 0, 0, 0);
                        if constexpr (X4) racc4 = mfma4(u[s], x4[J * 64 + s * 16 + x4l], racc4);
                    }
                }
            }
            row_sum(wi, yacc[ib], yacc4[ib]);
            S = Sn;
        }
    }
    // loads issued past the wave's last tile read nothing; make sure none is
    // outstanding at exit
#pragma unroll
    for (int d = 0; d < NJ; ++d) asm volatile("" ::"v"(fa[d]), "v"(fb[d]));
    // The ragged tail rows n0 + r, r < rem, stored whole as a row-major strip
    // after the tiles: one more tile row, whose 16-column chunks are the
    // chunks q < nt (row part and column part, as for a tile, by the wave that
    // owns column q) and the corner (the full rem x rem block: row part only,
    // wave nt % 8).
    const int rem = uses_strip(n) ? n % 16 : 0;
    dvec4 yrag = zero;
    double yrag4 = 0.0;
    if (rem > 0) {
        const int n0 = 16 * nt;
        const double *sp = a.tiles + (it.tile + total) * 256;
        constexpr int G = 2;        // chunks whose entries are requested together
        double xr[4], xr4[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            xr[s] = xs[nt * 256 + s * 64 + L];
            xr4[s] = X4 ? x4[nt * 64 + s * 16 + x4l] : 0.0;
        }
#pragma unroll
        for (int j0 = 0; j0 <= NJ; j0 += G) {
            double v[G][4], u[4];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int jj = j0 + g, q = jj < NJ ? jj * NW + w : nt;
                const int cv = jj < NJ ? (q < nt ? 16 : 0) : jj == NJ && w == nt % NW ? rem : 0;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int r = 4 * lk + s;
                    v[g][s] = (r < rem && li < cv) ? sp[(int64_t)r * n + 16 * q + li] : 0.0;
                }
            }
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int jj = j0 + g, q = jj < NJ ? jj * NW + w : nt;
                if (jj < NJ ? q < nt : jj == NJ && w == nt % NW) {     // (wave-uniform)
                    transpose(v[g], u);
                    if (jj < NJ) {
#pragma unroll
                        for (int s = 0; s < 4; ++s) {
                            yacc[jj < NJ ? jj : 0] =
                                __builtin_amdgcn_mfma_f64_16x16x4f64(v[g][s], xr[s], yacc[jj < NJ ? jj : 0], 0, 0, 0);
                            if constexpr (X4) yacc4[jj < NJ ? jj : 0] = mfma4(v[g][s], xr4[s], yacc4[jj < NJ ? jj : 0]);
                        }
                    }
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        racc = __builtin_amdgcn_mfma_f64_16x16x4f64(u[s], xs[q * 256 + s * 64 + L], racc, 0, 0, 0);
                        if constexpr (X4) racc4 = mfma4(u[s], x4[q * 64 + s * 16 + x4l], racc4);
                    }
                }
            }
        }
        row_sum(0, yrag, yrag4);
    }
    // Y through LDS ([column][row], odd stride, over X and the tiles' slots),
    // so that it is written in whole lines
    __syncthreads();
    const int ldy = npad + 1;
    auto put = [&](int J, const dvec4 &y, double y4) {
#pragma unroll
        for (int r = 0; r < 4; ++r) sm[li * ldy + 16 * J + 4 * r + lk] = y[r];
        if constexpr (X4) sm[(16 + (li & 3)) * ldy + 16 * J + r4] = y4;
    };
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj)
        if (jj * NW + w < nt) put(jj * NW + w, yacc[jj], yacc4[jj]);
    if (rem > 0 && w == 0) put(nt, yrag, yrag4);
    __syncthreads();
    for (int e = tid; e < W * n; e += NW * 64) {
        const int cc = e / n, k = e - cc * n, col = c0 + cc;
        if (col < a.ncols) a.ypart[(int64_t)col * a.ylen + it.xoff + k] = sm[cc * ldy + k];
    }
}

// out[g + col ldo] = sum of part[col plen + idx[e]], e in [ptr[g], ptr[g+1])
__global__ void __launch_bounds__(256) k_gather_block(int n, const int32_t *ptr, const int32_t *idx,
                                                      const double *part, int64_t plen, double *out, int64_t ldo,
                                                      int ncols) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    const int e0 = ptr[g], e1 = ptr[g + 1];
    for (int col = blockIdx.y; col < ncols; col += gridDim.y) {
        const double *p = part + (int64_t)col * plen;
        double s = 0.0;
        for (int e = e0; e < e1; ++e) s += p[idx[e]];
        out[g + (int64_t)col * ldo] = s;
    }
}

}  // namespace

static size_t symm_smem(int max_n, int cols = 16) {
    return sizeof(double) * ((size_t)cols * 16 * ((max_n + 15) / 16) + NW * 256);
}
constexpr size_t SYMM_HALF = 80 * 1024;     // two blocks a compute unit

int set_symm_smem_limit() {
    const void *f[4] = {(const void *)k_symm<3, false>, (const void *)k_symm<4, false>, (const void *)k_symm<5, false>,
                        (const void *)k_symm<3, true>};
    for (const void *p : f)
        if (hipFuncSetAttribute(p, hipFuncAttributeMaxDynamicSharedMemorySize, (int)symm_smem(SYMM_MAX_N)) != hipSuccess)
            return 1;
    return 0;
}

// max_n: the largest subdomain size, max_nt: the most tile rows of one
void launch_symm(const BlockSymvArgs &a, int nsub, int max_n, int max_nt, hipStream_t s) {
    if (nsub <= 0 || a.ncols <= 0) return;
    const dim3 grid(nsub * ((a.ncols + 15) / 16)), block(NW * 64);
    const size_t smem = symm_smem(max_n), smem4 = symm_smem(max_n, 20);
    // 17 to 20 columns, while two blocks still fit a compute unit (subdomains
    // of up to 8^3 elements); above them two chunks
    if (a.ncols > 16 && a.ncols <= 20 && max_nt <= 3 * NW && smem4 <= SYMM_HALF)
        hipLaunchKernelGGL((k_symm<3, true>), dim3(nsub), block, smem4, s, a, nsub);
    else if (max_nt <= 3 * NW) hipLaunchKernelGGL((k_symm<3, false>), grid, block, smem, s, a, nsub);
    else if (max_nt <= 4 * NW) hipLaunchKernelGGL((k_symm<4, false>), grid, block, smem, s, a, nsub);
    else hipLaunchKernelGGL((k_symm<5, false>), grid, block, smem, s, a, nsub);
}

void launch_gather_block(int n, const int32_t *ptr, const int32_t *idx, const double *part, int64_t plen, double *out,
                         int64_t ldo, int ncols, hipStream_t s) {
    if (n <= 0 || ncols <= 0) return;
    hipLaunchKernelGGL(k_gather_block, dim3((n + 255) / 256, std::min(ncols, 8)), dim3(256), 0, s, n, ptr, idx, part,
                       plen, out, ldo, ncols);
}

}  // namespace bddc
