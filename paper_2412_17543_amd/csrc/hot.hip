// gfx950 kernels of one deflated-PCG iteration (Algorithm 1) preconditioned
// by two- or three-level BDDC (Section 3.2), on the interface problem of
// Section 3.1.
//
// One iteration is a fixed chain of kernels that can be captured once as a
// graph and replayed:
//   k_symv (S)   q_i = S_i p_i                      Alg. 1 line 9 (A p)
//   k_update     alpha, x += alpha p, r -= alpha q  lines 9-11
//   k_symv (N)   stopping test (Section 5); u_i = D N_i D r_i and the
//                coarse residual partials c_i = (D Phi_i)^T r_i
//   coarse       k_coarse_dense (two levels, or three levels in explicit form);
//                three levels as a chain: k_l2_a, k_l2_b, level 3 by the
//                dense product, k_l2_c, k_l2_d
//   k_prolong    w_i = u_i + D Phi_i u_C            eq. averaging_subdomain_solves
//   k_zasm       z = sum_i R_i^T w_i, r^T z, (AW)^T z   line 13
//   k_pupd       beta, mu, p = z + beta p - W mu    lines 14-16
// A converged or failed solve sets ctl->done; every later kernel returns at
// once, so replaying more iterations than needed is harmless.
//
// Reductions never cross blocks inside a kernel: a producer writes one
// partial per block (or per work item), column by column, and every block of
// the consuming kernel sums them in index order, so all blocks see bitwise
// the same scalars and every run gives the same result.
#include <hip/hip_runtime.h>

#include "devutil.h"
#include "internal.h"
#include "kernels.h"

namespace bddc {

using dev::block_sum;
using dev::block_sum_cols;
using dev::block_sum_contig;
using dev::wave_sum;
using dev::wave_sum_contig;

namespace {

template <typename T>
struct Acc {
    using type = double;
};
template <>
struct Acc<float> {
    using type = float;
};
template <>
struct Acc<uint16_t> {
    using type = float;
};

typedef unsigned int uvec2 __attribute__((ext_vector_type(2)));

typedef unsigned int uvec4 __attribute__((ext_vector_type(4)));

// Buffer resource over `bytes` bytes from p (raw, unswizzled): loads past the
// end return zero without a memory access.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const void *p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000);
}
constexpr int LOAD_NT = 2;          // non-temporal: each tile is read once per product

// Element i of a float64 array through a buffer resource of `n` elements:
// zero past the end, without a memory access.  A fixed-count loop of such
// loads needs no per-element condition, so the loads are all issued before
// the first wait.  Byte offsets below 2^31.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t vec_rsrc(const double *p, int64_t n) {
    return tile_rsrc(p, (int)(n * 8));
}
__device__ __forceinline__ double ld_rc(__amdgpu_buffer_rsrc_t r, int64_t i) {
    const uvec2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)(i * 8), 0, 0);
    return __hiloint2double(v.y, v.x);
}

// The four values lane l holds of a 16x16 tile: rows 4*(l/16)+i, column l%16
// (element order of tile_index); tile t of the resource (the whole offset is
// in the vector operand, which is what the range check sees).  settle() waits for
// a fragment that is not going to be used (a loop exit), so that no path
// reaches the loop head with its load outstanding.
template <typename T>
struct Frag;
template <>
struct Frag<double> {
    uvec4 a, b;
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int t, int l) {
        a = __builtin_amdgcn_raw_buffer_load_b128(r, t * 2048 + l * 16, 0, LOAD_NT);
        b = __builtin_amdgcn_raw_buffer_load_b128(r, t * 2048 + 1024 + l * 16, 0, LOAD_NT);
    }
    __device__ __forceinline__ void settle() const { asm volatile("" ::"v"(a), "v"(b)); }
    __device__ __forceinline__ void get(double v[4]) const {
        v[0] = __hiloint2double(a.y, a.x); v[1] = __hiloint2double(a.w, a.z);
        v[2] = __hiloint2double(b.y, b.x); v[3] = __hiloint2double(b.w, b.z);
    }
};
template <>
struct Frag<float> {
    uvec4 a;
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int t, int l) {
        a = __builtin_amdgcn_raw_buffer_load_b128(r, t * 1024 + l * 16, 0, LOAD_NT);
    }
    __device__ __forceinline__ void settle() const { asm volatile("" ::"v"(a)); }
    __device__ __forceinline__ void get(float v[4]) const {
        v[0] = __uint_as_float(a.x); v[1] = __uint_as_float(a.y);
        v[2] = __uint_as_float(a.z); v[3] = __uint_as_float(a.w);
    }
};
template <>
struct Frag<uint16_t> {
    uvec2 a;
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int t, int l) {
        a = __builtin_amdgcn_raw_buffer_load_b64(r, t * 512 + l * 8, 0, LOAD_NT);
    }
    __device__ __forceinline__ void settle() const { asm volatile("" ::"v"(a)); }
    __device__ __forceinline__ void get(float v[4]) const {
        v[0] = dev::bf16_to_f32(a.x & 0xffffu);
        v[1] = dev::bf16_to_f32(a.x >> 16);
        v[2] = dev::bf16_to_f32(a.y & 0xffffu);
        v[3] = dev::bf16_to_f32(a.y >> 16);
    }
};

using dev::DPP_HALF_MIRROR;
using dev::DPP_ROR4;
using dev::DPP_ROR8;
using dev::DPP_XOR1;
using dev::DPP_XOR2;
using dev::dpp;

// the sum over the four lanes l % 16 + 16 g
template <typename T>
__device__ __forceinline__ T col_sum4(T v) { return dev::add_xor32(dev::add_xor16(v)); }

// Sums of ra[0..3] over the 16 lanes of a row of the wave, by exchange:
// lanes with bit 3 set keep rows 2, 3 and pass rows 0, 1 to lane ^ 8 (and
// the converse), then bit 2 halves again against the mirrored lane, and two
// quad swaps finish.  Returns, in every lane, the full sum of ra[cl >> 2].
template <typename A>
__device__ __forceinline__ A row_sum4(const A (&ra)[4], int cl) {
    const bool b3 = (cl & 8) != 0, b2 = (cl & 4) != 0;
    A k0 = b3 ? ra[2] : ra[0], k1 = b3 ? ra[3] : ra[1];
    const A s0 = b3 ? ra[0] : ra[2], s1 = b3 ? ra[1] : ra[3];
    k0 += dpp<DPP_ROR8>(s0);
    k1 += dpp<DPP_ROR8>(s1);
    A m = b2 ? k1 : k0;
    const A sd = b2 ? k0 : k1;
    m += dpp<DPP_HALF_MIRROR>(sd);
    m += dpp<DPP_XOR1>(m);
    m += dpp<DPP_XOR2>(m);
    return m;
}

__device__ __forceinline__ double to_d(double v) { return v; }
__device__ __forceinline__ double to_d(float v) { return (double)v; }
__device__ __forceinline__ double to_d(uint16_t v) { return (double)dev::bf16_to_f32(v); }

// s plus, in list order, the partial products part[idx[e]], e in [e0, e1): the
// first four together (most nodes have two to four entries: pointer, index
// and value latencies once each), the rest L at a time.  A subdomain cut into
// many segments gives lists of up to dozens of entries, which one by one cost
// two latencies each (residual update: 16^3, 12 to 48 entries a node, 11.2 ->
// 6.6 us; holed 64^3 16.1 -> 9.0 us).
template <int L>
__device__ __forceinline__ double gather_range(const int32_t *idx, const double *part, int e, int e1, double s) {
    if constexpr (L > 4) {
        while (e < e1) {                    // (past the list: its last entry again, not added)
            int id[L];
            double v[L];
#pragma unroll
            for (int u = 0; u < L; ++u) id[u] = idx[min(e + u, e1 - 1)];
#pragma unroll
            for (int u = 0; u < L; ++u) v[u] = part[id[u]];
#pragma unroll
            for (int u = 0; u < L; ++u)
                if (e + u < e1) s += v[u];
            e += L;
        }
    } else {
        for (; e < e1; e += L) {
            int id[L];
            double v[L];
#pragma unroll
            for (int u = 0; u < L; ++u) id[u] = e + u < e1 ? idx[e + u] : -1;
#pragma unroll
            for (int u = 0; u < L; ++u) v[u] = id[u] >= 0 ? part[id[u]] : 0.0;
#pragma unroll
            for (int u = 0; u < L; ++u)
                if (id[u] >= 0) s += v[u];
        }
    }
    return s;
}

// Sum of the partial products listed for assembled entry t (fixed order).
// LONG: lists of product segments, else lists of subdomains (at most 8 or so).
template <bool LONG = false>
__device__ __forceinline__ double gather_sum(const Gather &G, int64_t t) {
    const int e0 = G.ptr[t], e1 = G.ptr[t + 1];
    if constexpr (!LONG) return gather_range<4>(G.idx, G.part, e0, e1, 0.0);
    const double s = gather_range<4>(G.idx, G.part, e0, min(e0 + 4, e1), 0.0);
    return gather_range<16>(G.idx, G.part, e0 + 4, e1, s);
}

// Stopping test of Section 5 (eq. stopping_rhs, or eq. stopping_residual with
// stop_rule 1) on the residual whose per-block ||r||^2 partials are in
// rr_part.  first: the first test of a solve, on r_0 (zero iterations
// allowed); otherwise after the residual update, `iter` loop passes done.
// Every block evaluates it identically; block 0 records the outcome.
__device__ bool stop_eval(Ctl *c, const double *rr_part, int rr_n, const double *bb_part, int bb_n, bool first,
                          int stop_rule, int max_it, int iter, double *res_hist, int hist_cap) {
    __shared__ int s_stop;
    if (threadIdx.x < 64) {
        const double rr = wave_sum_contig(rr_part, rr_n);
        double bb = 0.0, denom2;
        if (first) {
            bb = wave_sum_contig(bb_part, bb_n);
            denom2 = stop_rule == 0 ? bb : rr;
        } else {
            denom2 = c->denom2;
        }
        const bool conv = (first && bb == 0.0) || rr < c->rtol2 * denom2;
        const bool bad = !isfinite(rr);
        const bool maxed = !first && iter >= max_it;
        const bool run_end = !first && iter >= c->iter_stop;   // restart_every: end of a run
        const bool stop = conv || bad || maxed || run_end;
        if (threadIdx.x == 0) {
            s_stop = stop ? 1 : 0;
            if (blockIdx.x == 0) {
                c->rr = rr;
                if (first) {
                    c->bb = bb;
                    c->r0r0 = rr;
                    c->denom2 = denom2;
                    if (bb == 0.0) c->zero_rhs = 1;
                } else {
                    c->iter = iter;
                }
                if (res_hist && iter < hist_cap) res_hist[iter] = rr;
                if (c->hprog) {
                    volatile double *hp = c->hprog;
                    hp[0] = rr;
                    hp[1] = denom2;
                    hp[2] = (double)iter;
                }
                if (bad) c->status = BDDC_EBREAKDOWN;
                else if (!conv && maxed) c->status = BDDC_ENOTCONV;
                if (stop) ctl_finish(c);
            }
        }
    }
    __syncthreads();
    return s_stop != 0;
}

// The test at the start of the preconditioner's product (direction j not yet
// advanced).  While the basis is recording and `defer` is set, the test is
// left to k_pupd instead, so that the last pass also produces z = M^{-1} r,
// which the harmonic-Ritz matrices need (Section 4.2).
__device__ bool stop_test(const SymvArgs &a) {
    Ctl *c = a.ctl;
    const bool first = a.test == 2;
    return stop_eval(c, a.rr_part, a.rr_n, a.bb_part, a.bb_n, first, a.stop_rule, a.max_it, first ? 0 : c->j + 1,
                     a.res_hist, a.hist_cap);
}

// ctl->done read once per block (a block of the kernel that sets it may be
// running meanwhile): every thread gets the same answer.
__device__ bool block_done(const Ctl *c) {
    __shared__ int s_done;
    if (threadIdx.x == 0) s_done = c->done;
    __syncthreads();
    return s_done != 0;
}

// y = M x with M (k x k row-major), x and y in LDS, k <= RMAX, by a block of
// 256 threads: 16 lanes a row, lane c taking the columns c, c + 16, ... (one
// thread a row is a chain of k LDS reads and adds, 20 of them 1 us).  No
// barrier at the end.
__device__ __forceinline__ void small_matvec(const double *M, int k, const double *x, double *y) {
    const int c = threadIdx.x & 15;
    for (int r0 = 0; r0 < k; r0 += 16) {               // (block-uniform: every lane takes part in the sum)
        const int r = r0 + (threadIdx.x >> 4);
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < RMAX / 16; ++u) {
            const int q = c + 16 * u;
            if (r < k && q < k) s += M[r * k + q] * x[q];
        }
        s = dev::row16_sum(s);
        if (c == 0 && r < k) y[r] = s;
    }
}

// y_r = sum_{q < ncol} M[q * ldm + r] x[q] for r in [r0, r1) (M read column
// by column, i.e. the transposed access of a row-major symmetric matrix, so
// consecutive lanes read consecutive addresses).  Lanes take 64 rows; the NW
// waves take as many row blocks as there are (up to NW) and split the columns
// of each among the waves left over (these are chains of loads: more waves,
// fewer round trips); partial sums are added in wave order by the first wave
// of a row block, which calls store(r, y_r).  x is in LDS.
template <int NW, typename F>
__device__ __forceinline__ void cm_matvec(const double *M, int64_t ldm, int r0, int r1, int ncol, const double *x,
                                          double (*part)[64], F store) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    const int nrb = (r1 - r0 + 63) / 64, G = max(1, min(nrb, NW)), P = NW / G, g = w / P, pt = w - g * P;
    const int q0 = (int)((int64_t)ncol * pt / P), q1 = (int)((int64_t)ncol * (pt + 1) / P);
    for (int b0 = 0; b0 < nrb; b0 += G) {
        const int r = r0 + 64 * (b0 + g) + l;
        const bool live = g < G && r < r1;
        double s = 0.0;
        if (live) {
#pragma unroll 8
            for (int q = q0; q < q1; ++q) s += M[(int64_t)q * ldm + r] * x[q];
        }
        part[w][l] = s;
        __syncthreads();
        if (live && pt == 0) {
            double t = 0.0;
            for (int q = 0; q < P; ++q) t += part[w + q][l];
            store(r, t);
        }
        __syncthreads();
    }
}

}  // namespace

// registers for at least 6 waves per SIMD (4 with four float64 tiles in flight)
// A segment record, read through the constant address space: the index is
// block-uniform, so these become scalar loads.
__device__ __forceinline__ SymvItem load_item(const SymvItem *items, int i) {
    typedef const __attribute__((address_space(4))) int32_t CInt;
    CInt *q = (CInt *)(items + i);
    return SymvItem{q[0], q[1], q[2], q[3], q[4], q[5], q[6], q[7], q[8], q[9], q[10], q[11]};
}

template <typename T, int U>
constexpr int symv_waves_per_simd() { return (sizeof(T) == 8 && U == 4) ? 4 : 6; }

// Dot product, in float64 and entry order, of the V = 16 / sizeof(T) entries
// of one 16-byte vector with V consecutive values of x.
template <typename T, typename X>
__device__ __forceinline__ double dot16(const uvec4 &v, const X *x) {
    if constexpr (sizeof(T) == 8) {
        return __hiloint2double(v.y, v.x) * (double)x[0] + __hiloint2double(v.w, v.z) * (double)x[1];
    } else if constexpr (sizeof(T) == 4) {
        return (((double)__uint_as_float(v.x) * (double)x[0] + (double)__uint_as_float(v.y) * (double)x[1]) +
                (double)__uint_as_float(v.z) * (double)x[2]) +
               (double)__uint_as_float(v.w) * (double)x[3];
    } else {
        const unsigned int u[4] = {v.x, v.y, v.z, v.w};
        double s = 0.0;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            s += (double)dev::bf16_to_f32((uint16_t)(u[h] & 0xffffu)) * (double)x[2 * h];
            s += (double)dev::bf16_to_f32((uint16_t)(u[h] >> 16)) * (double)x[2 * h + 1];
        }
        return s;
    }
}

// Coarse restriction c_i = (D Phi_i)^T x_i of subdomain `sub` (n rows), with
// x_i staged in LDS (zero past n to a multiple of 16), for the DOFs q = c,
// c + C, ... of segment c of the subdomain's C (so that a split subdomain
// shares the work): wave w takes the w-th, (w + NW)-th, ... of those DOFs,
// QB of them at a time; a lane dots the 16-byte
// pieces V l, V l + 64 V, ... of each DOF's column-major row with x, JM
// pieces per round trip, and the wave's sum (fixed order) is the partial.
// Pieces of DOFs past nc_i read as zero through the range check (t past
// the segment's count gives q >= nc_i).
template <typename T, int NW, typename X>
__device__ __forceinline__ void coarse_tail(const SymvArgs &a, int sub, int c, int n, const X *xs, int wu, int l) {
    constexpr int V = 16 / (int)sizeof(T), W = 64 * V, QB = sizeof(T) == 2 ? 1 : 2, JM = 2;
    const int C = a.op.nchunk[sub], nci = a.nc[sub], ld = phi_ld(n);
    const int nq = nci > c ? (nci - c + C - 1) / C : 0;   // this segment's DOFs
    const __amdgpu_buffer_rsrc_t pr =
        tile_rsrc(reinterpret_cast<const T *>(a.phir) + a.phr_off[sub], nci * ld * (int)sizeof(T));
    double *cp = a.cpart + a.c_off[sub];
    for (int t0 = wu; t0 < nq; t0 += NW * QB) {
        double acc[QB];
#pragma unroll
        for (int qi = 0; qi < QB; ++qi) acc[qi] = 0.0;
        for (int p0 = V * l; p0 < ld; p0 += JM * W) {
            uvec4 f[QB][JM];
#pragma unroll
            for (int qi = 0; qi < QB; ++qi)
#pragma unroll
                for (int jj = 0; jj < JM; ++jj)
                    f[qi][jj] = p0 + jj * W < ld ? __builtin_amdgcn_raw_buffer_load_b128(
                                                       pr, ((c + C * (t0 + NW * qi)) * ld + p0 + jj * W) * (int)sizeof(T),
                                                       0, 0)
                                                 : uvec4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int qi = 0; qi < QB; ++qi)
#pragma unroll
                for (int jj = 0; jj < JM; ++jj)
                    if (p0 + jj * W < ld) acc[qi] += dot16<T>(f[qi][jj], xs + p0 + jj * W);
        }
#pragma unroll
        for (int qi = 0; qi < QB; ++qi) {
            const double s = wave_sum(acc[qi]);
            const int t = t0 + NW * qi;
            if (l == 0 && t < nq) cp[c + C * t] = s;
        }
    }
}

// Name tags of the three operator batches (the kernel is the same; only the
// Neumann batch makes the stopping test and the coarse restriction).
struct OpSchur { static constexpr bool neumann = false; };
struct OpNeumann { static constexpr bool neumann = true; };
struct OpInterior { static constexpr bool neumann = false; };

template <typename T, int NW, int U, typename OP>
__global__ void __launch_bounds__(NW * 64, (symv_waves_per_simd<T, U>())) k_symv(SymvArgs a) {
    using ACC = typename Acc<T>::type;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double red[16];
    constexpr int NT = NW * 64;
    constexpr int GATHER_PER_THREAD = NT >= 512 ? 1 : 512 / NT;
    constexpr int SR = 4;           // strip rows per pass (registers)
    // the first pass requested with the gathered values where registers allow
    // (not beside the stopping test's registers in the float64 Neumann batch)
    constexpr bool STRIP_EARLY = sizeof(T) == 2 || (sizeof(T) == 4 && U == 2) || (sizeof(T) == 8 && U == 4 && !OP::neumann);
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, g4 = 4 * (l >> 4), cl = l & 15;
    const int wu = __builtin_amdgcn_readfirstlane(w);     // wave-uniform control flow
    // Segment records are block-uniform: read through the constant address
    // space (scalar loads).  The first one is in flight during the control
    // check; the gather indices and first tile stage of a segment are issued
    // as soon as its record is there (before the stopping test for the first
    // segment), then gathered values, then the second stage, in this order,
    // so that waiting for the values never waits for the second stage (loads
    // complete in issue order).  Three round trips before the first tile is
    // used.
    SymvItem it = load_item(a.op.items, blockIdx.x);
    if (a.gated && block_done(a.ctl)) return;
    const bool test_here = OP::neumann && a.test && !(a.defer && a.ctl->record);

    // Tiles past w1 read as zero without a memory access (resource over tiles
    // [t, w1) for the stage starting at tile t), so the loads of the next U
    // tiles are issued unconditionally while the current U are used; two
    // register sets in turn, so that no copy waits for a load.
    double dot = 0.0;
    // the block's segments (consecutive pieces of the global tile sequence,
    // each inside one subdomain), one after the other
    for (bool first = true;; first = false) {
        const int n = it.n;
        const T *tb = reinterpret_cast<const T *>(a.op.tiles) + (int64_t)it.tile * 256;
        const int32_t *gb = a.op.gB + it.x_off;
        const int ntf = it.ntf;     // tile rows
        const int ntl = it.ntl;     // the tiles; a strip's slots follow
        // the waves split the segment's tiles; the segment holding slot ntl
        // also takes the ragged tail's strip (after its tiles)
        const int span = max(min(it.t1, ntl) - it.t0, 0);
        const bool strip_here = it.strip && it.t0 <= ntl && ntl < it.t1;
        const int w0 = it.t0 + (int)((int64_t)span * wu / NW);
        const int w1 = it.t0 + (int)((int64_t)span * (wu + 1) / NW);
        auto stage = [&](int t) {
            return tile_rsrc(tb + (int64_t)t * 256, max(w1 - t, 0) * 256 * (int)sizeof(T));
        };
        int gi[GATHER_PER_THREAD];
    #pragma unroll
        for (int j = 0; j < GATHER_PER_THREAD; ++j) gi[j] = gb[min(tid + j * NT, max(n - 1, 0))];
        asm volatile("" ::: "memory");                        // (keeps those loads first)
        Frag<T> fa[U], fb[U];
    #pragma unroll
        for (int u = 0; u < U; ++u) fa[u].load(stage(w0), u, l);
        if (first && test_here && stop_test(a)) return;
        const int npad = ((n + TILE - 1) / TILE) * TILE;
        ACC *xs = reinterpret_cast<ACC *>(smem_raw);
        ACC *yw = xs + npad;
        double xv[GATHER_PER_THREAD];
    #pragma unroll
        for (int j = 0; j < GATHER_PER_THREAD; ++j) xv[j] = a.x[gi[j]];
        asm volatile("" ::: "memory");                        // (the gathered values before fb)
        // the strip segment: its first SR rows at column tid, requested before
        // the second tile stage and applied right after the staging below
        const int rem = n % TILE, n0 = n - rem;
        const T *sp = tb + (int64_t)ntl * 256;
        T sv[SR];
        if (STRIP_EARLY && strip_here) {
    #pragma unroll
            for (int r = 0; r < SR; ++r) sv[r] = (r < rem && tid < n) ? sp[(int64_t)r * n + tid] : (T)0;
        }
        asm volatile("" ::: "memory");
    #pragma unroll
        for (int u = 0; u < U; ++u) fb[u].load(stage(w0 + U), u, l);
    #pragma unroll
        for (int j = 0; j < GATHER_PER_THREAD; ++j) {
            const int k = tid + j * NT;
            if (k < npad) xs[k] = k < n ? (ACC)xv[j] : (ACC)0;
        }
        if (npad > GATHER_PER_THREAD * NT) {   // long interfaces: indices through 32-bit offsets
            const __amdgpu_buffer_rsrc_t gr = tile_rsrc(gb, n * 4);
            for (int k = tid + GATHER_PER_THREAD * NT; k < npad; k += NT)
                xs[k] = k < n ? (ACC)a.x[(int)__builtin_amdgcn_raw_buffer_load_b32(gr, k * 4, 0, 0)] : (ACC)0;
        }
        for (int k = tid; k < NW * npad; k += NT) yw[k] = (ACC)0;
        __syncthreads();

        ACC *myy = yw + wu * npad;
        // Ragged tail rows n0 + r (r < n % 16), stored whole: rows r0..r0+SR-1 at
        // column k = k0 + tid (entries v, zero past the strip).  The thread
        // adds S[n0+r][k] x[n0+r] into y_k (columns below n0); the products
        // S[n0+r][k] x_k are summed over the wave and added into y_(n0+r).
        // Every addition goes into the thread's own wave's partials, in a
        // fixed order.
        auto strip_rows = [&](int k0, int r0, const T (&v)[SR]) {
            const int k = k0 + tid;
            const ACC xk = k < n ? xs[k] : (ACC)0;
            ACC t = (ACC)0;
    #pragma unroll
            for (int r = 0; r < SR; ++r) {
                if (r0 + r < rem) {
                    const ACC vr = (ACC)to_d(v[r]);
                    t += vr * xs[n0 + r0 + r];
                    const ACC sr = wave_sum(vr * xk);
                    if (l == 0) myy[n0 + r0 + r] += sr;
                }
            }
            if (k < n0) myy[k] += t;
        };
        if (STRIP_EARLY && strip_here) strip_rows(0, 0, sv);
        if (w0 >= w1) {
    #pragma unroll
            for (int u = 0; u < U; ++u) { fa[u].settle(); fb[u].settle(); }
        } else {
            int I = 0, rs = 0;
            while (rs + (ntf - I) <= w0) { rs += ntf - I; ++I; }
            int J = I + (w0 - rs);
            ACC xi[4], ra[4];
    #pragma unroll
            for (int q = 0; q < 4; ++q) { xi[q] = xs[I * TILE + g4 + q]; ra[q] = (ACC)0; }
            // Every fragment is used arithmetically on every path (a tile past
            // w1 reads as zero and only its bookkeeping is skipped), so no path
            // leaves a load outstanding when its registers are loaded again.
            auto use = [&](const Frag<T> (&f)[U], int t) {
    #pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool live = t + u < w1;
                    ACC v[4];
                    f[u].get(v);
                    // no direct part past the range (J < ntf holds for a live
                    // tile; the test keeps the float64 Schur variants free of spills)
                    const ACC xj = (live && J < ntf) ? xs[J * TILE + cl] : (ACC)0;
    #pragma unroll
                    for (int q = 0; q < 4; ++q) ra[q] += v[q] * xj;
                    const ACC s = col_sum4(v[0] * xi[0] + v[1] * xi[1] + v[2] * xi[2] + v[3] * xi[3]);
                    if (!live) continue;
                    if (J != I && l < 16) myy[J * TILE + cl] += s;
                    if (++J == ntf) {
                        const ACC m = row_sum4(ra, cl);
                        if ((cl & 3) == 0) myy[I * TILE + g4 + (cl >> 2)] += m;
    #pragma unroll
                        for (int q = 0; q < 4; ++q) ra[q] = (ACC)0;
                        ++I;
                        J = I;
                        if (I < ntf) {
    #pragma unroll
                            for (int q = 0; q < 4; ++q) xi[q] = xs[I * TILE + g4 + q];
                        }
                    }
                }
            };
            // fa holds tiles [t, t + U), fb the next U (both issued above)
            for (int t = w0;;) {
                use(fa, t);
                t += U;
                if (t >= w1) {
    #pragma unroll
                    for (int u = 0; u < U; ++u) fb[u].settle();
                    break;
                }
    #pragma unroll
                for (int u = 0; u < U; ++u) fa[u].load(stage(t + U), u, l);
                use(fb, t);
                t += U;
                if (t >= w1) {
    #pragma unroll
                    for (int u = 0; u < U; ++u) fa[u].settle();
                    break;
                }
    #pragma unroll
                for (int u = 0; u < U; ++u) fb[u].load(stage(t + U), u, l);
            }
            if (J != I) {   // flush a partly processed tile row
                const ACC m = row_sum4(ra, cl);
                if ((cl & 3) == 0) myy[I * TILE + g4 + (cl >> 2)] += m;
            }
        }
        if (strip_here) {   // the rest of the strip (more than SR rows, or columns past NT)
            for (int k0 = 0; k0 < n; k0 += NT) {
                for (int r0 = 0; r0 < rem; r0 += SR) {
                    if (STRIP_EARLY && k0 == 0 && r0 == 0) continue;
                    T v[SR];
    #pragma unroll
                    for (int r = 0; r < SR; ++r)
                        v[r] = (r0 + r < rem && k0 + tid < n) ? sp[(int64_t)(r0 + r) * n + k0 + tid] : (T)0;
                    strip_rows(k0, r0, v);
                }
            }
        }
        __syncthreads();

        double *yp = a.ypart + it.yoff;
        for (int k = tid; k < n; k += NW * 64) {
            ACC s = (ACC)0;
    #pragma unroll
            for (int q = 0; q < NW; ++q) s += yw[q * npad + k];
            const double y = (double)s;
            yp[k] = y;
            dot += (double)xs[k] * y;
        }
        if constexpr (OP::neumann) {   // this segment's share of the coarse restriction
            if (a.cpart) coarse_tail<T, NW>(a, it.sub, it.chunk, n, xs, wu, l);
        }
        __syncthreads();   // LDS is reused by the next segment
        if (it.next < 0) break;
        it = load_item(a.op.items, it.next);
    }
    if (a.dot) {
        dot = block_sum(dot, red);
        if (threadIdx.x == 0) a.dot[blockIdx.x] = dot;
    }
}

// ---------------------------------------------------------------------------
// Alg. 1 lines 9-11: alpha = rho_j / p^T A p (every block sums the per-item
// partials of the Schur product), q = sum_i R_i^T q_i, x += alpha p,
// r -= alpha q; per-block ||r||^2; the product is kept as AP_j for recycling.
// ---------------------------------------------------------------------------
// Operands of nodes gb, gb + stride, ..., UN of them: q from its partial
// products (in list order, as gather_sum adds them), x, p, r.  The pointer,
// index and partial loads of all UN nodes are issued together (three round
// trips for the group instead of three per node).
constexpr int UPD_SLOTS = 8;        // partials per node fetched in the first pass
template <int UPD_UN>
__device__ __forceinline__ void upd_load(const UpdArgs &a, int64_t gb, int64_t stride, double (&q)[UPD_UN],
                                         double (&xv)[UPD_UN], double (&pv)[UPD_UN], double (&rv)[UPD_UN]) {
    int e0[UPD_UN], e1[UPD_UN];
#pragma unroll
    for (int u = 0; u < UPD_UN; ++u) {
        const int64_t g = gb + u * stride;
        const bool ok = g < a.n;
        e0[u] = ok ? a.q.ptr[g] : 0;
        e1[u] = ok ? a.q.ptr[g + 1] : 0;
        xv[u] = ok ? a.x[g] : 0.0;
        pv[u] = ok ? a.p[g] : 0.0;
        rv[u] = ok ? a.r[g] : 0.0;
    }
    int id[UPD_UN][UPD_SLOTS];
#pragma unroll
    for (int u = 0; u < UPD_UN; ++u)
#pragma unroll
        for (int m = 0; m < UPD_SLOTS; ++m) id[u][m] = e0[u] + m < e1[u] ? a.q.idx[e0[u] + m] : -1;
#pragma unroll
    for (int u = 0; u < UPD_UN; ++u) {
        double v[UPD_SLOTS];
#pragma unroll
        for (int m = 0; m < UPD_SLOTS; ++m) v[m] = id[u][m] >= 0 ? a.q.part[id[u][m]] : 0.0;
        double sum = 0.0;
#pragma unroll
        for (int m = 0; m < UPD_SLOTS; ++m)
            if (id[u][m] >= 0) sum += v[m];
        q[u] = gather_range<16>(a.q.idx, a.q.part, e0[u] + UPD_SLOTS, e1[u], sum);
    }
}

// UPD_UN nodes per pass: 4 when every thread has several nodes, else 1
template <int UPD_UN>
__global__ void __launch_bounds__(256) k_update(UpdArgs a) {
    __shared__ double red[16];
    Ctl *c = a.ctl;
    if (c->done) return;
    const int j = c->j;
    const int64_t g0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    // the operands of this thread's first nodes do not depend on alpha: their
    // loads are issued before the reduction
    double q[UPD_UN], xv[UPD_UN], pv[UPD_UN], rv[UPD_UN];
    upd_load<UPD_UN>(a, g0, stride, q, xv, pv, rv);
    const double pAp = block_sum_contig(a.dot, a.dot_n, red);
    const double alpha = (j < a.hist_cap ? a.rho_hist[j] : 0.0) / pAp;
    const bool bad = !(pAp > 0.0) || !isfinite(alpha) || j >= a.hist_cap;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        c->pAp = pAp;
        c->alpha = alpha;
        if (j < a.hist_cap) { a.d_hist[j] = pAp; a.a_hist[j] = alpha; }
        if (bad) { c->status = BDDC_EBREAKDOWN; ctl_finish(c); }
    }
    if (bad) return;
    const bool rec = a.AP && c->record && j < a.cap;
    double rr = 0.0;
    for (int64_t gb = g0; gb < a.n; gb += UPD_UN * stride) {
        if (gb != g0) upd_load<UPD_UN>(a, gb, stride, q, xv, pv, rv);
#pragma unroll
        for (int u = 0; u < UPD_UN; ++u) {
            const int64_t g = gb + u * stride;
            if (g < a.n) {
                const double xi = xv[u] + alpha * pv[u];
                const double ri = rv[u] - alpha * q[u];
                a.x[g] = xi;
                a.r[g] = ri;
                rr += ri * ri;
                if (rec) a.AP[(int64_t)j * a.ld + g] = q[u];
            }
        }
    }
    rr = block_sum(rr, red);
    if (threadIdx.x == 0) a.rr_part[blockIdx.x] = rr;
}

// ---------------------------------------------------------------------------
// Coarse prolongation (eq. averaging_subdomain_solves), one block per
// subdomain: w_i = u_i + (D Phi_i) u_C|_i, u_i summed from the partial
// products of the Neumann operator's work items.
// ---------------------------------------------------------------------------
// Element i of a T array through a buffer resource (zero past its end).
template <typename T>
__device__ __forceinline__ double ld_rc_as(__amdgpu_buffer_rsrc_t r, int i);
template <>
__device__ __forceinline__ double ld_rc_as<double>(__amdgpu_buffer_rsrc_t r, int i) { return ld_rc(r, i); }
template <>
__device__ __forceinline__ double ld_rc_as<float>(__amdgpu_buffer_rsrc_t r, int i) {
    return (double)__uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, i * 4, 0, 0));
}
template <>
__device__ __forceinline__ double ld_rc_as<uint16_t>(__amdgpu_buffer_rsrc_t r, int i) {
    return (double)dev::bf16_to_f32(__builtin_amdgcn_raw_buffer_load_b16(r, i * 2, 0, 0));
}

// Sums of up to NE rows' parts at once, 32 lanes a row (every lane of the wave
// active; rows < 0: no access, zero), in the same order for every reader.
template <int NE>
__device__ __forceinline__ void symblk_rows(__amdgpu_buffer_rsrc_t pr, int nb, const int (&row)[NE], double (&s)[NE]) {
    const int l = threadIdx.x & 31, nbp = symblk_ld(nb), np = 64 * nb * nbp;
#pragma unroll
    for (int e = 0; e < NE; ++e) s[e] = 0.0;
    for (int k0 = 0; k0 < nb; k0 += 64) {
        double v[NE][2];
#pragma unroll
        for (int e = 0; e < NE; ++e)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int k = k0 + 32 * u + l;
                v[e][u] = ld_rc(pr, row[e] >= 0 && k < nb ? row[e] * nbp + k : np);
            }
#pragma unroll
        for (int e = 0; e < NE; ++e) s[e] += v[e][0] + v[e][1];
    }
#pragma unroll
    for (int e = 0; e < NE; ++e) s[e] = dev::row16_sum(dev::add_xor16(s[e]));
}

enum { UC_VEC, UC_SOLVE, UC_PARTS };

// u_C is read (UC_VEC), added from the parts of the product in blocks
// (UC_PARTS), or solved for.
// UC_SOLVE (dense coarse operators of up to FUSED_MAX_NC rows, one column): the
// block computes the entries of u_C that its subdomain needs from the coarse
// partials, a wave per entry with the operands of four entries requested
// before r_C is gathered, in the summation order of
// k_coarse_dense, whose launch it replaces.  One preconditioner application
// against that launch and one for r_C before it: 18 coarse DOFs (16^3) 19.8 ->
// 16.1 us, 82 24.1 -> 20.0, 216 (32^3) 28.0 -> 23.8, 444 37.8 -> 33.9.  Above,
// every block's rows of M (nc_i nC entries) cost what the launches do: with room
// for 2,048 columns 790 DOFs take 45.8 us either way, 1,932 45.9 against 31.7.
template <typename T, int UC>
__global__ void __launch_bounds__(256) k_prolong(ProlArgs a) {
    extern __shared__ double uCl[];
    constexpr int PF = 16, CF = 4;      // basis entries / partials of a row requested early
    if (a.gated && a.ctl->done) return;
    // 512 rows of one subdomain per block (large subdomains take several)
    const int i = a.ch_sub[blockIdx.x], r0 = a.ch_row[blockIdx.x];
    const int n = a.nB[i], C = a.nchunk[i];
    const int nci = UC != UC_VEC || a.uC ? a.nc[i] : 0, ld = phi_ld(n);
    const int32_t *ci = a.cidx + a.c_off[i];
    const T *ph = reinterpret_cast<const T *>(a.phir) + a.phr_off[i];   // column-major, rows of ld
    const double *up = a.upart + a.pb[i];
    double *wl = a.wloc + a.b_off[i];
    // The first CF partial sums and PF basis entries of this thread's first
    // two rows do not depend on u_C: they are requested before its gather,
    // through range-checked loads (no conditions; entries past the
    // subdomain's arrays read as zero, other rows' entries are not used).
    // Consecutive threads read consecutive entries of each basis column.
    const __amdgpu_buffer_rsrc_t ur = vec_rsrc(up, (int64_t)C * n);
    const __amdgpu_buffer_rsrc_t pr = tile_rsrc(ph, nci * ld * (int)sizeof(T));
    const int k0 = r0 + threadIdx.x, k1 = r0 + threadIdx.x + 256;
    double u0[CF], u1[CF], pr0[PF], pr1[PF];
#pragma unroll
    for (int cc = 0; cc < CF; ++cc) {
        u0[cc] = ld_rc(ur, cc * n + k0);
        u1[cc] = ld_rc(ur, cc * n + k1);
    }
#pragma unroll
    for (int q = 0; q < PF; ++q) {
        pr0[q] = ld_rc_as<T>(pr, q * ld + k0);
        pr1[q] = ld_rc_as<T>(pr, q * ld + k1);
    }
    if constexpr (UC == UC_SOLVE) {
        constexpr int EG = 4;
        __shared__ double rs[FUSED_MAX_NC];
        const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, ldm = (int)a.ldm;
        const __amdgpu_buffer_rsrc_t mr = tile_rsrc(a.M, a.nC * ldm * 8);
        uvec4 m[EG][4];
        auto request = [&](int q0) {                   // entries q0, q0 + 4, ... (past the last: zeros, no access)
#pragma unroll
            for (int j = 0; j < EG; ++j) {
                const int q = q0 + 4 * j, row = q < nci ? ci[q] : a.nC;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int col = 2 * l + 128 * u;
                    m[j][u] = __builtin_amdgcn_raw_buffer_load_b128(mr, (col < ldm ? row * ldm + col : a.nC * ldm) * 8, 0, 0);
                }
            }
        };
        request(wv);
        for (int q = threadIdx.x; q < FUSED_MAX_NC; q += 256) rs[q] = q < a.nC ? gather_sum(a.rc, q) : 0.0;
        __syncthreads();
        for (int q0 = wv; q0 < nci; q0 += 4 * EG) {
            if (q0 != wv) request(q0);
#pragma unroll
            for (int j = 0; j < EG; ++j) {
                double s[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int col = 2 * l + 128 * u;
                    s[u] = __hiloint2double(m[j][u].y, m[j][u].x) * rs[col] + __hiloint2double(m[j][u].w, m[j][u].z) * rs[col + 1];
                }
                const double t = wave_sum((s[0] + s[1]) + (s[2] + s[3]));
                if (l == 0 && q0 + 4 * j < nci) uCl[q0 + 4 * j] = a.sign * t;
            }
        }
        // (a wave without entries leaves its first requests unused: none outstanding at exit)
#pragma unroll
        for (int j = 0; j < EG; ++j)
#pragma unroll
            for (int u = 0; u < 4; ++u) asm volatile("" ::"v"(m[j][u]));
    } else if constexpr (UC == UC_PARTS) {
        // the parts of four entries a round, 32 lanes each
        const __amdgpu_buffer_rsrc_t sr = vec_rsrc(a.upC, (int64_t)64 * a.nbC * symblk_ld(a.nbC));
        const int g = threadIdx.x >> 5;
        for (int qb = 0; qb < nci; qb += 32) {
            int rw[4];
            double s[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) rw[j] = qb + g + 8 * j < nci ? ci[qb + g + 8 * j] : -1;
            symblk_rows(sr, a.nbC, rw, s);
            if ((threadIdx.x & 31) == 0) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (qb + g + 8 * j < nci) uCl[qb + g + 8 * j] = s[j];
            }
        }
    } else {
        for (int q = threadIdx.x; q < nci; q += blockDim.x) uCl[q] = a.uC[ci[q]];
    }
    __syncthreads();
    // w = sum of the partials, then the basis terms, in column order; both rows
    // advance together, so that a subdomain cut into many segments or with
    // many coarse DOFs waits once for both (holed 64^3: 19.5 -> 16.1 us)
    double w0 = 0.0, w1 = 0.0;
#pragma unroll
    for (int cc = 0; cc < CF; ++cc)
        if (cc < C) { w0 += u0[cc]; w1 += u1[cc]; }
    for (int cc = CF; cc < C; cc += CF) {
        double v0[CF], v1[CF];
#pragma unroll
        for (int m = 0; m < CF; ++m) {
            v0[m] = ld_rc(ur, (cc + m) * n + k0);
            v1[m] = ld_rc(ur, (cc + m) * n + k1);
        }
#pragma unroll
        for (int m = 0; m < CF; ++m)
            if (cc + m < C) { w0 += v0[m]; w1 += v1[m]; }
    }
#pragma unroll
    for (int q = 0; q < PF; ++q)
        if (q < nci) { w0 += pr0[q] * uCl[q]; w1 += pr1[q] * uCl[q]; }
    constexpr int QF = 16;
    for (int qb = PF; qb < nci; qb += QF) {
        double v0[QF], v1[QF];
#pragma unroll
        for (int m = 0; m < QF; ++m) {
            v0[m] = ld_rc_as<T>(pr, (qb + m) * ld + k0);
            v1[m] = ld_rc_as<T>(pr, (qb + m) * ld + k1);
        }
#pragma unroll
        for (int m = 0; m < QF; ++m)
            if (qb + m < nci) { w0 += v0[m] * uCl[qb + m]; w1 += v1[m] * uCl[qb + m]; }
    }
    if (k0 < n) wl[k0] = w0;
    if (k1 < n) wl[k1] = w1;
}

// Block products: PCOLS columns a block, one partial product per subdomain.
// Every basis entry read serves all of them (a grid row per column read the
// bases 20 times, from the memory-side cache at best: 210 -> 70 us at 96^3, 20
// columns).  The columns' u_C pass through LDS UCH entries at a
// time; summation order as in k_prolong.
constexpr int PCOLS = 8, UCH = 128;
template <int UC>
__global__ void __launch_bounds__(256) k_prolong_cols(ProlArgs a, int ncols) {
    __shared__ double uCl[UCH * PCOLS];
    constexpr int QF = 8;
    const int ng = (ncols + PCOLS - 1) / PCOLS, b = blockIdx.x / ng, c0 = (blockIdx.x - b * ng) * PCOLS;
    const int nc = min(PCOLS, ncols - c0), t = threadIdx.x;
    const int i = a.ch_sub[b], r0 = a.ch_row[b];
    const int n = a.nB[i], nci = UC != UC_VEC || a.uC ? a.nc[i] : 0, ld = phi_ld(n);
    const int32_t *ci = a.cidx + a.c_off[i];
    const __amdgpu_buffer_rsrc_t pr =
        tile_rsrc(reinterpret_cast<const double *>(a.phir) + a.phr_off[i], nci * ld * (int)sizeof(double));
    const int k0 = r0 + t, k1 = r0 + t + 256;
    double w0[PCOLS], w1[PCOLS];
#pragma unroll
    for (int c = 0; c < PCOLS; ++c) {
        const double *up = a.upart + (int64_t)(c0 + c) * a.cs_u + a.pb[i];
        w0[c] = c < nc && k0 < n ? up[k0] : 0.0;
        w1[c] = c < nc && k1 < n ? up[k1] : 0.0;
    }
    for (int q0 = 0; q0 < nci; q0 += UCH) {
        const int cnt = min(UCH, nci - q0);
        if (q0) __syncthreads();
        for (int e = cnt * PCOLS + t; e < ((cnt + QF - 1) / QF) * QF * PCOLS; e += 256) uCl[e] = 0.0;
        if constexpr (UC == UC_PARTS) {
            for (int c = 0; c < nc; ++c) {
                const __amdgpu_buffer_rsrc_t sr =
                    vec_rsrc(a.upC + (int64_t)(c0 + c) * a.cs_uC, (int64_t)64 * a.nbC * symblk_ld(a.nbC));
                for (int qb = 0; qb < cnt; qb += 32) {
                    int rw[4];
                    double s[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int q = qb + (t >> 5) + 8 * j;
                        rw[j] = q < cnt ? ci[q0 + q] : -1;
                    }
                    symblk_rows(sr, a.nbC, rw, s);
                    if ((t & 31) == 0) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const int q = qb + (t >> 5) + 8 * j;
                            if (q < cnt) uCl[q * PCOLS + c] = s[j];
                        }
                    }
                }
            }
            for (int e = t; e < cnt * PCOLS; e += 256)
                if (e % PCOLS >= nc) uCl[e] = 0.0;
        } else {
            for (int e = t; e < cnt * PCOLS; e += 256) {
                const int c = e % PCOLS;
                uCl[e] = c < nc ? a.uC[(int64_t)(c0 + c) * a.cs_uC + ci[q0 + e / PCOLS]] : 0.0;
            }
        }
        __syncthreads();
        for (int q = 0; q < cnt; q += QF) {
            double v0[QF], v1[QF];
#pragma unroll
            for (int m = 0; m < QF; ++m) {
                v0[m] = ld_rc(pr, (q0 + q + m) * ld + k0);
                v1[m] = ld_rc(pr, (q0 + q + m) * ld + k1);
            }
#pragma unroll
            for (int m = 0; m < QF; ++m)
#pragma unroll
                for (int c = 0; c < PCOLS; ++c) {
                    const double u = uCl[(q + m) * PCOLS + c];
                    w0[c] += v0[m] * u;
                    w1[c] += v1[m] * u;
                }
        }
    }
#pragma unroll
    for (int c = 0; c < PCOLS; ++c) {
        double *wl = a.wloc + (int64_t)(c0 + c) * a.cs_w + a.b_off[i];
        if (c < nc && k0 < n) wl[k0] = w0[c];
        if (c < nc && k1 < n) wl[k1] = w1[c];
    }
}

// ---------------------------------------------------------------------------
// Alg. 1 line 13, assembly: z = sum_i R_i^T w_i (weights folded into the
// stored operators).  Per-block partials of r^T z and (AW)^T z (line 15),
// column-major.  With `advance`, block 0 moves the direction index to j + 1
// (no block of this kernel reads it).
// ---------------------------------------------------------------------------
template <int KM>
__global__ void __launch_bounds__(256) k_zasm(ZasmArgs a) {
    __shared__ double lds[16 * 256];
    __shared__ double res[KM + 1];
    Ctl *c = a.ctl;
    if (a.gated && c->done) return;
    if (a.advance && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) c->j = c->j + 1;
    {
        const int64_t col = blockIdx.y;  // one column per grid row (block products; no partials)
        a.w.part += col * a.cs_w;
        a.r += col * a.cs_r;
        a.z += col * a.cs_z;
    }
    const int k = a.part ? c->k : 0;
    double acc[KM + 1];
#pragma unroll
    for (int q = 0; q <= KM; ++q) acc[q] = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const __amdgpu_buffer_rsrc_t awr = vec_rsrc(a.AW, (int64_t)k * a.ld);
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < a.n; g += stride) {
        // the node's (AW) and r entries are requested with its gather, not
        // after the store of z (which the compiler may not move them past)
        double aw[KM > 0 ? KM : 1], rg = 0.0;
        if (a.part) {
            rg = a.r[g];
#pragma unroll
            for (int q = 0; q < KM; ++q) aw[q] = ld_rc(awr, (int64_t)q * a.ld + g);
        }
        const double z = gather_sum(a.w, g);
        a.z[g] = z;
        if (a.part) {
            acc[0] += rg * z;
#pragma unroll
            for (int q = 0; q < KM; ++q) acc[1 + q] += aw[q] * z;
        }
    }
    if (!a.part) return;
    block_sum_cols<KM + 1>(acc, k + 1, lds, res);
    if (threadIdx.x <= k) a.part[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = res[threadIdx.x];
}

// ---------------------------------------------------------------------------
// Alg. 1 lines 14-16 (line 7 when `first`): every block sums the k_zasm
// partials into rho = r^T z and t = (AW)^T z, mu = (W^T A W)^{-1} t,
// beta = rho / rho_prev; p = z + beta p - W mu.  Block 0 records rho, beta,
// mu for the recycling step.  `hist_only` records without updating p (the
// extra preconditioner application after convergence).
// ---------------------------------------------------------------------------
// The partials (at most VGRID = 2 x 256 a column) and the operands of the
// thread's first UN nodes are all requested before the first wait (90^3, 20
// columns: 17.6 -> 15.9 us; two nodes a pass gained nothing in the assembly).
template <int KM, int UN>
__global__ void __launch_bounds__(256) k_pupd(PupdArgs a) {
    __shared__ double lds[16 * 256];
    __shared__ double tv[KM + 1];
    __shared__ double mu[RMAX];
    __shared__ double wawi[KM > 0 ? KM * KM : 1];
    Ctl *c = a.ctl;
    if (a.gated && c->done) return;
    const int k = c->k, j = c->j;
    // the stopping test deferred from the preconditioner's product (while
    // recording): on a stop, record rho and mu of this z and leave p alone
    bool hist_only = a.hist_only;
    if (a.test && c->record) {
        const bool first = a.test == 2;
        if (stop_eval(c, a.rr_part, a.rr_n, a.bb_part, a.bb_n, first, a.stop_rule, a.max_it, first ? 0 : j,
                      a.res_hist, a.hist_cap))
            hist_only = true;
    }
    const int64_t g0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    static_assert(VGRID <= 512, "two partials a thread and column");
    double z0[UN], p0[UN], w0[UN][KM > 0 ? KM : 1];
    // columns q >= k and nodes past n read as zero through the range check, so
    // every load is unconditional
    const __amdgpu_buffer_rsrc_t wr = vec_rsrc(a.W, (int64_t)k * a.ld);
    auto fetch = [&](int64_t gb) {
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int64_t g = gb + u * stride;
            const bool ok = g < a.n;
            z0[u] = ok ? a.z[g] : 0.0;
            p0[u] = ok ? a.p[g] : 0.0;
#pragma unroll
            for (int q = 0; q < KM; ++q) w0[u][q] = ld_rc(wr, ok ? (int64_t)q * a.ld + g : (int64_t)k * a.ld);
        }
    };
    {
        double acc[KM + 1], ac2[KM + 1];
        const int64_t zend = (int64_t)(k + 1) * a.zpart_n;
        const __amdgpu_buffer_rsrc_t zr = vec_rsrc(a.zpart, zend);
        const int b0 = threadIdx.x, b1 = threadIdx.x + 256;
#pragma unroll
        for (int q = 0; q <= KM; ++q) acc[q] = ld_rc(zr, b0 < a.zpart_n ? (int64_t)q * a.zpart_n + b0 : zend);
        if (a.zpart_n > 256) {
#pragma unroll
            for (int q = 0; q <= KM; ++q) ac2[q] = ld_rc(zr, b1 < a.zpart_n ? (int64_t)q * a.zpart_n + b1 : zend);
#pragma unroll
            for (int q = 0; q <= KM; ++q) acc[q] += ac2[q];
        }
        // the operands of this thread's first nodes do not depend on beta and
        // mu: their loads overlap the reductions
        if (!hist_only) fetch(g0);
        for (int e = threadIdx.x; e < k * k; e += blockDim.x) wawi[e] = a.WAWinv[e];
        block_sum_cols<KM + 1>(acc, k + 1, lds, tv);
    }
    // (block_sum_cols ends with a barrier: wawi is complete)
    small_matvec(wawi, k, tv + 1, mu);
    __syncthreads();
    const double rho = tv[0];
    const double beta = a.first ? 0.0 : rho / a.rho_hist[j - 1];
    const bool bad = !(rho > 0.0) || !isfinite(rho) || !isfinite(beta);
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) {
            if (j < a.hist_cap) a.rho_hist[j] = rho;
            if (!a.first && j >= 1 && j - 1 < a.hist_cap) a.b_hist[j - 1] = beta;
            if (bad && !hist_only) { c->status = BDDC_EBREAKDOWN; ctl_finish(c); }
        }
        if (threadIdx.x < k && j < a.hist_cap) a.mu_hist[(int64_t)j * RMAX + threadIdx.x] = mu[threadIdx.x];
    }
    if (hist_only || bad) return;
    const bool rec = a.P && c->record && j < a.cap;
    // all loads of a pass issued at once; summation in column order
    for (int64_t gb = g0; gb < a.n; gb += UN * stride) {
        if (gb != g0) fetch(gb);
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int64_t g = gb + u * stride;
            double p = z0[u] + beta * p0[u];
#pragma unroll
            for (int q = 0; q < KM; ++q)
                if (q < k) p -= w0[u][q] * mu[q];
            if (g < a.n) {
                a.p[g] = p;
                if (rec) a.P[(int64_t)j * a.ld + g] = p;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// out = b - sum_i R_i^T q_i (initial or true residual; out = the assembled
// product when b is null); per-block partials (column-major) of ||out||^2
// and, with want_wtr, of W^T out (Alg. 1 line 3).
// ---------------------------------------------------------------------------
template <int KM>
__global__ void __launch_bounds__(256) k_resid(ResidArgs a) {
    __shared__ double lds[16 * 256];
    __shared__ double res[KM + 1];
    const int k = a.want_wtr ? a.ctl->k : 0;
    double acc[KM + 1];
#pragma unroll
    for (int q = 0; q <= KM; ++q) acc[q] = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < a.n; g += stride) {
        const double q = gather_sum<true>(a.q, g);
        const double r = a.b ? a.b[g] - q : q;
        a.out[g] = r;
        acc[0] += r * r;
        const __amdgpu_buffer_rsrc_t wr = vec_rsrc(a.W, (int64_t)k * a.ld);
#pragma unroll
        for (int q2 = 0; q2 < KM; ++q2) acc[1 + q2] += ld_rc(wr, (int64_t)q2 * a.ld + g) * r;
    }
    block_sum_cols<KM + 1>(acc, k + 1, lds, res);
    if (threadIdx.x <= k) a.part[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = res[threadIdx.x];
}

// Alg. 1 lines 3-4: gamma = (W^T A W)^{-1} W^T r (every block, from the
// k_resid partials); x += W gamma; r -= AW gamma (= b - A x_0); ||r||^2.
template <int KM>
__global__ void __launch_bounds__(256) k_defl_init(DeflArgs a) {
    __shared__ double lds[16 * 256];
    __shared__ double tv[KM + 1];
    __shared__ double gam[RMAX];
    __shared__ double red[16];
    const int k = a.ctl->k;
    {
        double acc[KM + 1];
#pragma unroll
        for (int q = 0; q <= KM; ++q) acc[q] = 0.0;
        const __amdgpu_buffer_rsrc_t wr = vec_rsrc(a.wpart, (int64_t)(k + 1) * a.wpart_n);
        for (int b = threadIdx.x; b < a.wpart_n; b += blockDim.x) {
#pragma unroll
            for (int q = 0; q <= KM; ++q) acc[q] += ld_rc(wr, (int64_t)q * a.wpart_n + b);
        }
        block_sum_cols<KM + 1>(acc, k + 1, lds, tv);
    }
    for (int e = threadIdx.x; e < k * k; e += blockDim.x) lds[e] = a.WAWinv[e];
    __syncthreads();
    small_matvec(lds, k, tv + 1, gam);
    __syncthreads();
    double rr = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < a.n; g += stride) {
        double x = a.x[g], r = a.r[g];
        for (int q = 0; q < k; ++q) {
            x += a.W[(int64_t)q * a.ld + g] * gam[q];
            r -= a.AW[(int64_t)q * a.ld + g] * gam[q];
        }
        a.x[g] = x;
        a.r[g] = r;
        rr += r * r;
    }
    rr = block_sum(rr, red);
    if (threadIdx.x == 0) a.rr_part[blockIdx.x] = rr;
}

// out[c] = sum_b part[c * n + b] (column-major partials), one block per column
// Re-orthogonalisation (Alg. 1, optional line after the residual update):
// k_wtr writes per-block W^T r partials; k_reorth sums them in every block
// (fixed order), gamma = (W^T W)^{-1} W^T r, r -= W gamma and per-block
// ||r||^2 partials that replace the update's for the stopping test.
template <int KM>
__global__ void __launch_bounds__(256) k_wtr(ReorthArgs a) {
    __shared__ double lds[16 * 256];
    __shared__ double res[KM > 0 ? KM : 1];
    if (a.ctl->done) return;
    const int k = a.ctl->k;
    if (k == 0) return;
    double acc[KM > 0 ? KM : 1];
#pragma unroll
    for (int q = 0; q < KM; ++q) acc[q] = 0.0;
    const __amdgpu_buffer_rsrc_t wr = vec_rsrc(a.W, (int64_t)k * a.ld);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < a.n; g += stride) {
        const double r = a.r[g];
#pragma unroll
        for (int q = 0; q < KM; ++q) acc[q] += ld_rc(wr, (int64_t)q * a.ld + g) * r;
    }
    block_sum_cols<KM>(acc, k, lds, res);
    if (threadIdx.x < k) a.part[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = res[threadIdx.x];
}

template <int KM>
__global__ void __launch_bounds__(256) k_reorth(ReorthArgs a) {
    __shared__ double lds[16 * 256];
    __shared__ double tv[KM > 0 ? KM : 1], gam[KM > 0 ? KM : 1];
    __shared__ double red[16];
    if (a.ctl->done) return;
    const int k = a.ctl->k;
    if (k == 0) return;
    {
        double acc[KM > 0 ? KM : 1];
#pragma unroll
        for (int q = 0; q < KM; ++q) acc[q] = 0.0;
        const __amdgpu_buffer_rsrc_t pr = vec_rsrc(a.part, (int64_t)k * gridDim.x);
        for (int b = threadIdx.x; b < (int)gridDim.x; b += blockDim.x) {
#pragma unroll
            for (int q = 0; q < KM; ++q) acc[q] += ld_rc(pr, (int64_t)q * gridDim.x + b);
        }
        block_sum_cols<KM>(acc, k, lds, tv);
    }
    if (threadIdx.x < k) {
        double s = 0.0;
        for (int q = 0; q < k; ++q) s += a.WWinv[threadIdx.x * k + q] * tv[q];
        gam[threadIdx.x] = s;
    }
    __syncthreads();
    double rr = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < a.n; g += stride) {
        double r = a.r[g];
        for (int q = 0; q < k; ++q) r -= a.W[(int64_t)q * a.ld + g] * gam[q];
        a.r[g] = r;
        rr += r * r;
    }
    rr = block_sum(rr, red);
    if (threadIdx.x == 0) a.rr_part[blockIdx.x] = rr;
}

__global__ void __launch_bounds__(256) k_reduce(ReduceArgs a) {
    __shared__ double red[16];
    const int c = blockIdx.x;
    const double s = block_sum_contig(a.part + (int64_t)c * a.n, a.n, red);
    if (threadIdx.x == 0) a.out[c] = s;
}

// ---------------------------------------------------------------------------
// coarse problem (eq. coarse_problem); three levels: the multilevel paragraph
// of Section 3.2, subdomains acting as the elements of subregions.  Every
// matrix here is symmetric and row-major; products read it column by column.
// ---------------------------------------------------------------------------
// Dense product u = sign * M r of up to FUSED_MAX_NC rows (row-major M, rows
// padded with zeros to the even length ldm): a wave per row, four rows a
// block.  Latency alone: the row (512 columns in four 16-byte loads a lane,
// zero past the row through the range check) is requested before the block
// gathers r into LDS.  (A launch of its own for r: 4.6 us before 4.6 us at 460
// rows; with the gather in every block 4.7 us.)
constexpr int CD_ROWS = 4;
__global__ void __launch_bounds__(CD_ROWS * 64) k_coarse_dense(CoarseDenseArgs a) {
    __shared__ double rs[FUSED_MAX_NC];
    if (a.ctl->done) return;
    a.rc.part += blockIdx.y * a.cs_rc;  // one column per grid row (block products)
    a.u += blockIdx.y * a.cs_u;
    const int n = a.n, ldm = (int)a.ldm;
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int row = blockIdx.x * CD_ROWS + w;
    const bool live = row < n;
    const __amdgpu_buffer_rsrc_t mr = tile_rsrc(a.M + (int64_t)(live ? row : 0) * ldm, live ? ldm * 8 : 0);
    uvec4 m[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) m[u] = __builtin_amdgcn_raw_buffer_load_b128(mr, (2 * l + 128 * u) * 8, 0, 0);
    for (int q = threadIdx.x; q < FUSED_MAX_NC; q += CD_ROWS * 64) rs[q] = q < n ? gather_sum(a.rc, q) : 0.0;
    __syncthreads();
    double s[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int col = 2 * l + 128 * u;
        s[u] = __hiloint2double(m[u].y, m[u].x) * rs[col] + __hiloint2double(m[u].w, m[u].z) * rs[col + 1];
    }
    const double t = wave_sum((s[0] + s[1]) + (s[2] + s[3]));
    if (live && l == 0) a.u[row] = a.sign * t;
}

// Larger symmetric coarse operators: the upper triangle in 64 x 64 blocks,
// half the bytes of the full matrix.  One block of threads per matrix block
// (I, J); thread 16 i + j holds the 4 x 4 patch (i, j), stored in the order the
// threads read it and requested before r is gathered on the panels I and J.
// Its four row sums are added over the 16 lanes of the row of patches, for
// J > I its four column sums over the 4 lanes of the wave in that column, then
// over the waves in order.  (Sixteen entries of one row a thread: sixteen
// column sums over 64 lanes, take 16.7 us a launch at 3,595 rows and 7.3 at
// 1,932; the patches 13.6 and 6.6, of which the gather and the start of a launch
// are about 4.  The full matrix by rows, with a launch for r before it: 20.7 and
// 11.6 us.)
// A row's parts are stored side by side, for readers of single rows.
__device__ __forceinline__ int symblk_start(int I, int nb) { return I * nb - I * (I - 1) / 2; }

__global__ void __launch_bounds__(256) k_symblk(SymBlkArgs a) {
    __shared__ double colw[4][64];
    __shared__ double xsh[128];     // r_J, then r_I
    if (a.ctl->done) return;
    const int b = blockIdx.x / a.ncols, col = blockIdx.x - b * a.ncols;
    const int t = threadIdx.x, i = t >> 4, j = t & 15, w = t >> 6;
    const double2 *bp = reinterpret_cast<const double2 *>(a.B + (int64_t)b * 4096) + t;
    double2 v[4][2];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int h = 0; h < 2; ++h) v[r][h] = bp[(2 * r + h) * 256];
    const int I = a.bI[b], J = I + (b - symblk_start(I, a.nb)), nbp = symblk_ld(a.nb);
    double *part = a.part + col * a.cs_part;
    a.rc.part += col * a.cs_rc;
    if (t < 128) {
        const int g = t < 64 ? 64 * J + t : 64 * I + t - 64;
        xsh[t] = g < a.n ? gather_sum(a.rc, g) : 0.0;
    }
    __syncthreads();
    double xj[4], xi[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        xj[c] = xsh[4 * j + c];
        xi[c] = xsh[64 + 4 * i + c];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const double s = dev::row16_sum((v[r][0].x * xj[0] + v[r][0].y * xj[1]) + (v[r][1].x * xj[2] + v[r][1].y * xj[3]));
        if (j == r) part[(int64_t)(64 * I + 4 * i + r) * nbp + J] = s;
    }
    if (J == I) return;             // (block-uniform) a diagonal block holds both triangles
    double cs[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        double u = 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) u += (c & 1 ? v[r][c >> 1].y : v[r][c >> 1].x) * xi[r];
        cs[c] = col_sum4(u);
    }
    if ((t & 63) < 16) {
#pragma unroll
        for (int c = 0; c < 4; ++c) colw[w][4 * j + c] = cs[c];
    }
    __syncthreads();
    if (t < 64) part[(int64_t)(64 * J + t) * nbp + I] = ((colw[0][t] + colw[1][t]) + colw[2][t]) + colw[3][t];
}

__global__ void __launch_bounds__(256) k_symblk_sum(SymBlkArgs a) {
    if (a.ctl->done) return;
    const __amdgpu_buffer_rsrc_t pr =
        vec_rsrc(a.part + blockIdx.y * a.cs_part, (int64_t)64 * a.nb * symblk_ld(a.nb));
    const int r = blockIdx.x * 8 + (threadIdx.x >> 5);
    const int row[1] = {r < a.n ? r : -1};
    double s[1];
    symblk_rows(pr, a.nb, row, s);
    if ((threadIdx.x & 31) == 0 && r < a.n) a.u[blockIdx.y * a.cs_u + r] = s[0];
}

__device__ __forceinline__ void l2_cols(L2Args &a) {
    const int64_t col = blockIdx.y;     // one column per grid row (block products)
    a.rc.part += col * a.cs_rc;
    a.vI2 += col * a.cs_vI2;
    a.t2 += col * a.cs_t2;
    a.rB2 += col * a.cs_rB2;
    a.u2 += col * a.cs_u2;
    a.c3loc += col * a.cs_c3loc;
    a.u3 += col * a.cs_u3;
    a.uC += col * a.cs_uC;
}

// Waves of a level-2 block: 16 where one block per compute unit takes all
// (a launch then lasts as long as one block's chain of loads: 125 subregions,
// a 9.0 -> 7.9, b 10.9 -> 9.4 us), 4 where the blocks queue (1,728 subregions: b
// 19 us with 4 waves, 62 with 16).
constexpr int L2_ONE_ROUND = 256;

// Level 2, phase A (one block per subregion): the subregion's coarse
// residual r_L, interior pre-solve v_I = K_II^{-1} r_I and its interface
// coupling t = K_BI K_II^{-1} r_I (from the swept subregion matrix).
template <int NW>
__global__ void __launch_bounds__(NW * 64) k_l2_a(L2Args a) {
    extern __shared__ double rL[];
    __shared__ double part[NW][64];
    if (a.ctl->done) return;
    l2_cols(a);
    const int j = blockIdx.x;
    const int nL = a.nL[j], nI = a.nI2[j];
    const int loff = a.L_off[j];
    for (int q = threadIdx.x; q < nL; q += blockDim.x) rL[q] = gather_sum(a.rc, a.L[loff + q]);
    __syncthreads();
    double *vI2 = a.vI2 + a.I2_off[j], *t2 = a.t2 + a.B2_off[j], *rB2 = a.rB2 + a.B2_off[j];
    cm_matvec<NW>(a.K2 + a.K2_off[j], nL, 0, nL, nI, rL, part, [&](int q, double y) {
        if (q < nI) vI2[q] = -y;
        else { t2[q - nI] = y; rB2[q - nI] = rL[q]; }
    });
}

// Level 2, phase B (one block per subregion): level-2 interface residual
// g = r_G - sum_j R_j^T t_j, then u = (D N D) g and c3 = (D Phi)^T g.
template <int NW>
__global__ void __launch_bounds__(NW * 64) k_l2_b(L2Args a) {
    extern __shared__ double gs[];
    __shared__ double part[NW][64];
    if (a.ctl->done) return;
    l2_cols(a);
    const int j = blockIdx.x;
    const int nB = a.nL[j] - a.nI2[j];
    const int b2 = a.B2_off[j];
    for (int k = threadIdx.x; k < nB; k += blockDim.x) {
        const int gi = a.g2[b2 + k];
        const double r = a.rB2[b2 + k];
        gs[k] = r - gather_range<4>(a.asm2_idx, a.t2, a.asm2_ptr[gi], a.asm2_ptr[gi + 1], 0.0);
    }
    __syncthreads();
    double *u2 = a.u2 + b2, *c3 = a.c3loc + a.C3_off[j];
    cm_matvec<NW>(a.N2 + a.N2_off[j], nB, 0, nB, nB, gs, part, [&](int k, double y) { u2[k] = y; });
    cm_matvec<NW>(a.Phi2 + a.P2_off[j], a.nc3[j], 0, a.nc3[j], nB, gs, part, [&](int q, double y) { c3[q] = y; });
}

// Level 2, phase C: u_j + (D Phi_j) u3 at every interface position of every
// subregion, 16 lanes a position (each position once: phase D needs it in
// every subregion that shares the DOF, and summed it there as a chain of a
// dozen round trips).
__global__ void __launch_bounds__(256) k_l2_c(L2Args a) {
    if (a.ctl->done) return;
    l2_cols(a);
    const int pos = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 4), c = threadIdx.x & 15;
    const bool live = pos < a.nB2;
    double v = 0.0, u = 0.0;
    if (live) {
        const double *ph = a.Phi2 + a.ph_off[pos];
        const int32_t *c3 = a.c3 + a.c3o[pos];
        const int n3j = a.n3p[pos];
        u = a.u2[pos];
#pragma unroll 4
        for (int q = c; q < n3j; q += 16) v += ph[q] * a.u3[c3[q]];
    }
    v = dev::row16_sum(v);
    if (live && c == 0) a.u2[pos] = u + v;
}

// Level 2, phase D (one block per subregion): level-2 interface solution
// x_G = sum_j R_j^T (u_j + (D Phi_j) u3) on the subregion's interface (from
// phase C) and the interior post-correction x_I = v_I - T^T x_G give the
// level-1 coarse solution u_C on the coarse DOFs of the subregion (every
// subregion sharing an interface DOF computes the same value in the same
// order; its owner writes it) for the prolongation, k_prolong.
// Phases A to D of one application, against 4 waves a block everywhere and
// phase C inside D: 125 subregions (90^3) 9 + 11 + 22 -> 8 + 9 + 5 + 7 us, 1,728
// (192^3) 14 + 19 + 43 -> 12 + 19 + 8 + 14 us.
template <int NW>
__global__ void __launch_bounds__(NW * 64) k_l2_d(L2Args a) {
    extern __shared__ double sm[];
    __shared__ double part[NW][64];
    if (a.ctl->done) return;
    l2_cols(a);
    double *uCL = sm;                 // nL: x_I then x_G
    const int j = blockIdx.x;
    const int nL = a.nL[j], nI = a.nI2[j], nB = nL - nI;
    const int b2 = a.B2_off[j];
    for (int k = threadIdx.x; k < nB; k += blockDim.x) {
        const int gi = a.g2[b2 + k];
        const double s = gather_range<4>(a.asm2_idx, a.u2, a.asm2_ptr[gi], a.asm2_ptr[gi + 1], 0.0);
        uCL[nI + k] = s;
    }
    __syncthreads();
    const double *vI2 = a.vI2 + a.I2_off[j];
    cm_matvec<NW>(a.K2 + a.K2_off[j] + (int64_t)nI * nL, nL, 0, nI, nB, uCL + nI, part,
                 [&](int q, double y) { uCL[q] = vI2[q] - y; });
    // cm_matvec ends with a barrier: uCL is complete
    for (int q = threadIdx.x; q < nL; q += blockDim.x)
        if (q < nI || a.own2[b2 + q - nI]) a.uC[a.L[a.L_off[j] + q]] = uCL[q];
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
size_t symv_smem(int prec, int nw, int max_nt) {
    const size_t acc = prec == 64 ? 8 : 4;
    return acc * (size_t)max_nt * TILE * (1 + nw);
}

template <typename T, typename OP>
static int set_limit_t(size_t bytes) {
    const void *f[4] = {(const void *)k_symv<T, 4, 2, OP>, (const void *)k_symv<T, 4, 4, OP>,
                        (const void *)k_symv<T, 8, 2, OP>, (const void *)k_symv<T, 8, 4, OP>};
    for (const void *p : f)
        if (hipFuncSetAttribute(p, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) return -1;
    return 0;
}

int set_symv_smem_limit(size_t bytes) {
    if (set_limit_t<double, OpSchur>(bytes) || set_limit_t<double, OpInterior>(bytes) ||
        set_limit_t<double, OpNeumann>(bytes) || set_limit_t<float, OpNeumann>(bytes) ||
        set_limit_t<uint16_t, OpNeumann>(bytes))
        return -1;
    return 0;
}

template <typename T, typename OP>
static void launch_symv_t(const SymvArgs &a, SymvCfg cfg, size_t smem, hipStream_t s) {
    const dim3 grid(a.op.n_blocks);
    if (cfg.nw == 8) {
        if (cfg.unroll == 4) hipLaunchKernelGGL((k_symv<T, 8, 4, OP>), grid, dim3(512), smem, s, a);
        else hipLaunchKernelGGL((k_symv<T, 8, 2, OP>), grid, dim3(512), smem, s, a);
    } else {
        if (cfg.unroll == 4) hipLaunchKernelGGL((k_symv<T, 4, 4, OP>), grid, dim3(256), smem, s, a);
        else hipLaunchKernelGGL((k_symv<T, 4, 2, OP>), grid, dim3(256), smem, s, a);
    }
}

// The Schur and interior operators are float64 only; the Neumann operators
// come in the three storage precisions.
void launch_symv(const SymvArgs &a, SymvOp op, int prec, SymvCfg cfg, size_t smem, hipStream_t s) {
    if (a.op.n_blocks <= 0) return;
    if (op == SYMV_SCHUR) launch_symv_t<double, OpSchur>(a, cfg, smem, s);
    else if (op == SYMV_INTERIOR) launch_symv_t<double, OpInterior>(a, cfg, smem, s);
    else if (prec == 64) launch_symv_t<double, OpNeumann>(a, cfg, smem, s);
    else if (prec == 32) launch_symv_t<float, OpNeumann>(a, cfg, smem, s);
    else launch_symv_t<uint16_t, OpNeumann>(a, cfg, smem, s);
}

void launch_update(const UpdArgs &a, int grid, hipStream_t s) {
    if (a.n > (int64_t)grid * 256 * 2) hipLaunchKernelGGL(k_update<4>, dim3(grid), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(k_update<1>, dim3(grid), dim3(256), 0, s, a);
}

void launch_prolong(const ProlArgs &a, int prec, int nblocks, int max_nc, hipStream_t s) {
    const size_t smem = (size_t)std::max(1, max_nc) * 8;
    const dim3 grid(nblocks);
    const int uc = a.fused ? UC_SOLVE : a.upC ? UC_PARTS : UC_VEC;
    auto go = [&](auto v64, auto v32, auto v16) {
        hipLaunchKernelGGL(prec == 64 ? v64 : prec == 32 ? v32 : v16, grid, dim3(256), smem, s, a);
    };
    if (uc == UC_SOLVE) go(k_prolong<double, UC_SOLVE>, k_prolong<float, UC_SOLVE>, k_prolong<uint16_t, UC_SOLVE>);
    else if (uc == UC_PARTS) go(k_prolong<double, UC_PARTS>, k_prolong<float, UC_PARTS>, k_prolong<uint16_t, UC_PARTS>);
    else go(k_prolong<double, UC_VEC>, k_prolong<float, UC_VEC>, k_prolong<uint16_t, UC_VEC>);
}

void launch_prolong_cols(const ProlArgs &a, int nblocks, int ncols, hipStream_t s) {
    const dim3 grid(nblocks * ((ncols + PCOLS - 1) / PCOLS));
    if (a.upC) hipLaunchKernelGGL(k_prolong_cols<UC_PARTS>, grid, dim3(256), 0, s, a, ncols);
    else hipLaunchKernelGGL(k_prolong_cols<UC_VEC>, grid, dim3(256), 0, s, a, ncols);
}

// Registers and loads are laid out for KM columns: buckets of 8 up to 48 (a
// basis of 20 in a bucket of 32 issues 12 loads a node for nothing, one of 40
// in a bucket of 48 8).  192^3, both builds in turn on one card, with the sums
// over lanes and the joint loads above: direction update 132 -> 122 us, assembly
// 136 -> 129.
int kmax_bucket(int k) { return k <= 48 ? (k + 7) / 8 * 8 : 64; }

#define KM_SWITCH(kmax, CALL)            \
    switch (kmax) {                      \
        case 0: CALL(0); break;          \
        case 8: CALL(8); break;          \
        case 16: CALL(16); break;        \
        case 24: CALL(24); break;        \
        case 32: CALL(32); break;        \
        case 40: CALL(40); break;        \
        case 48: CALL(48); break;        \
        default: CALL(64); break;        \
    }
void launch_zasm(const ZasmArgs &a, int kmax, int grid, hipStream_t s, int ncols) {
#define ZASM(KM) hipLaunchKernelGGL(k_zasm<KM>, dim3(grid, ncols), dim3(256), 0, s, a)
    KM_SWITCH(kmax, ZASM)
#undef ZASM
}

// nodes per pass of the direction update: two where a thread has more than
// one, up to 24 columns (227 registers; two blocks a compute unit)
template <int KM>
constexpr int pupd_nodes() { return KM <= 24 ? 2 : 1; }

void launch_pupd(const PupdArgs &a, int kmax, int grid, hipStream_t s) {
    const bool two = a.n > (int64_t)grid * 256;
#define PUPD(KM)                                                                                      \
    if (two) hipLaunchKernelGGL((k_pupd<KM, pupd_nodes<KM>()>), dim3(grid), dim3(256), 0, s, a);       \
    else hipLaunchKernelGGL((k_pupd<KM, 1>), dim3(grid), dim3(256), 0, s, a)
    KM_SWITCH(kmax, PUPD)
#undef PUPD
}

void launch_resid(const ResidArgs &a, int kmax, int grid, hipStream_t s) {
#define RESID(KM) hipLaunchKernelGGL(k_resid<KM>, dim3(grid), dim3(256), 0, s, a)
    KM_SWITCH(kmax, RESID)
#undef RESID
}

void launch_defl_init(const DeflArgs &a, int kmax, int grid, hipStream_t s) {
#define DEFL(KM) hipLaunchKernelGGL(k_defl_init<KM>, dim3(grid), dim3(256), 0, s, a)
    KM_SWITCH(kmax, DEFL)
#undef DEFL
}

void launch_reorth(const ReorthArgs &a, int kmax, int grid, hipStream_t s) {
    if (kmax == 0) return;
#define REORTH(KM)                                                                              \
    hipLaunchKernelGGL(k_wtr<(KM > 0 ? KM : 8)>, dim3(grid), dim3(256), 0, s, a);                \
    hipLaunchKernelGGL(k_reorth<(KM > 0 ? KM : 8)>, dim3(grid), dim3(256), 0, s, a)
    KM_SWITCH(kmax, REORTH)
#undef REORTH
}

void launch_reduce(const ReduceArgs &a, hipStream_t s) {
    if (a.ncol > 0) hipLaunchKernelGGL(k_reduce, dim3(a.ncol), dim3(256), 0, s, a);
}

void launch_coarse_dense(const CoarseDenseArgs &a, hipStream_t s, int ncols) {
    if (a.n > 0) hipLaunchKernelGGL(k_coarse_dense, dim3((a.n + CD_ROWS - 1) / CD_ROWS, ncols), dim3(CD_ROWS * 64), 0, s, a);
}

void launch_symblk(const SymBlkArgs &a, hipStream_t s) {
    if (a.n > 0) hipLaunchKernelGGL(k_symblk, dim3(a.nb * (a.nb + 1) / 2 * a.ncols), dim3(256), 0, s, a);
}

void launch_symblk_sum(const SymBlkArgs &a, hipStream_t s) {
    if (a.n > 0) hipLaunchKernelGGL(k_symblk_sum, dim3((a.n + 7) / 8, a.ncols), dim3(256), 0, s, a);
}

#define L2_LAUNCH(K, SMEM)                                                                              \
    do {                                                                                               \
        if (nsr * ncols <= L2_ONE_ROUND) hipLaunchKernelGGL(K<16>, dim3(nsr, ncols), dim3(1024), SMEM, s, a); \
        else hipLaunchKernelGGL(K<4>, dim3(nsr, ncols), dim3(256), SMEM, s, a);                            \
    } while (0)
void launch_l2_a(const L2Args &a, int nsr, int max_nL, hipStream_t s, int ncols) {
    L2_LAUNCH(k_l2_a, (size_t)max_nL * 8);
}
void launch_l2_b(const L2Args &a, int nsr, int max_nL, hipStream_t s, int ncols) {
    L2_LAUNCH(k_l2_b, (size_t)max_nL * 8);
}
size_t l2_d_smem(int max_nL) { return (size_t)std::max(1, max_nL) * 8; }

// (dynamic LDS of the level-2 kernels, beside up to 8 KB of partial sums)
int set_l2_smem_limit(size_t bytes) {
    if (bytes + 8192 <= 65536) return 0;
    for (const void *p : {(const void *)k_l2_a<4>, (const void *)k_l2_b<4>, (const void *)k_l2_d<4>,
                          (const void *)k_l2_a<16>, (const void *)k_l2_b<16>, (const void *)k_l2_d<16>})
        if (hipFuncSetAttribute(p, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) return -1;
    return 0;
}

void launch_l2_d(const L2Args &a, int nsr, size_t smem, hipStream_t s, int ncols) {
    if (a.nB2 > 0) hipLaunchKernelGGL(k_l2_c, dim3((a.nB2 + 15) / 16, ncols), dim3(256), 0, s, a);
    L2_LAUNCH(k_l2_d, smem);
}

}  // namespace bddc
