// Batched symmetric sweeps of the setup (local interior eliminations and
// Schur complements, Section 3.1; constrained-Neumann saddle inverses,
// eq. localCorr; face Schur complements of the adaptive step, Section 3.3;
// dense coarse inverses, Section 3.2), in panels of 64 pivots on the matrix
// cores.
//
// Sweeping a set P of pivots of a symmetric matrix A = [A_PP A_PQ; A_QP A_QQ]
// replaces it by
//     [ -A_PP^{-1}        A_PP^{-1} A_PQ                 ]
//     [ A_QP A_PP^{-1}    A_QQ - A_QP A_PP^{-1} A_PQ     ]
// and sweeping P1 then P2 equals sweeping P1 u P2 (the one-pivot sweep is the
// case |P| = 1).  So after sweeping the interior pivots, the interior block
// holds -K_II^{-1} and the interface block the Schur complement; after
// sweeping all pivots the matrix holds -A^{-1}.
//
// What bounds it: every panel reads and writes the whole trailing matrix (the
// swept rows too), so the bytes are n^2 x panels.  64 pivots a panel instead
// of 16 and the upper triangle of 64 x 64 tiles only (the lower one is
// mirrored once at the end) move an eighth of the bytes.  A 64-pivot update does
// 524,288 flop on a tile of 64 KB read and written, 8 flop/byte: HBM bounds it,
// the matrix cores and a copy meet at about 14 (70 TFLOP/s, 4.9 TB/s copied).  Per panel s (pivots 64 s .. 64 s + b - 1, every pivot checked
// for its expected sign):
//   k_sweep_diag   (one block per matrix) sweeps the b x b block in registers;
//   k_sweep_cols   (one block per 64 columns) U = A(P, :), X = A_PP^{-1} U
//                  (zero on P's own columns) into a panel buffer, and the
//                  panel's rows or columns of the result;
//   k_sweep_update (one block per upper tile) A <- A - U^T X; U and X vanish
//                  on P's columns, so the panel's rows are left as written.
// Matrices are taken with the most pivots first, so the ones still active at
// panel s are a prefix of the block lists: no block starts without work
// however much the sizes differ.
// All sweeps of a setup (local matrices of 729 rows and 343 pivots, saddle
// matrices of about 412, coarse levels), against 16-pivot panels over both
// triangles: 64^3 40.6 -> 10.7 ms, 192^3 1,225 -> 296 ms (update tiles 192 ms,
// 12.4 M of them, 64 KB each through HBM: 4.1 TB/s), holed 64^3 (up to 4,700 rows)
// 257 -> 36 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <numeric>
#include <vector>

#include "internal.h"
#include "kernels.h"

namespace bddc {

namespace {

constexpr int TS = 64;              // pivots per panel, edge of a tile
constexpr int TT = TS * TS;
constexpr int LDX = 80;             // LDS row stride (doubles) of the staged X tile: the four k rows of
                                    // an MFMA operand fall on both halves of the banks in turn
constexpr int LDT = 65;             // LDS row stride of transposed tiles
constexpr size_t PANEL_CAP = size_t(1) << 30;   // panel buffer of one batch of matrices
typedef double dvec4 __attribute__((ext_vector_type(4)));

struct Mat {                        // one matrix: U, X (tiles [J][k][j]) and -A_PP^{-1} in `buf`
    double *A;
    int64_t ld;
    double *buf;
    int32_t n, p1, pos_end, T;      // T = tiles per row
    __device__ double *U(int J) const { return buf + (int64_t)J * TT; }
    __device__ double *X(int J) const { return buf + ((int64_t)T + J) * TT; }
    __device__ double *P() const { return buf + 2 * (int64_t)T * TT; }
};
struct Item { int32_t mat, I, J; };  // one tile (I <= J), or one column tile J

// -A_PP^{-1} of the panel's pivot block: thread t holds 16 columns of row
// t / 4; the sweep keeps the block symmetric, so row k, broadcast through
// LDS, serves as column k too: one barrier and 16 multiply-adds a pivot (the
// pivot's place in its thread's registers is static: 16 pivots unrolled).
// Row k itself is v = 0 - (-1/piv) row, column k the factor r_k / piv.
__global__ void __launch_bounds__(256) k_sweep_diag(const Mat *mats, int s, int *status) {
    __shared__ double rb[2][TS];
    const Mat d = mats[blockIdx.x];
    const int p0 = TS * s, b = min(TS, d.p1 - p0);
    const int t = threadIdx.x, r = t >> 2, cq = t & 3, c0 = cq * 16;
    double v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i)
        v[i] = (r < b && c0 + i < b) ? d.A[(p0 + r) * d.ld + p0 + c0 + i] : 0.0;
    bool ok = true;
    for (int kb = 0; kb < (b + 15) / 16; ++kb) {
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
            const int k = 16 * kb + kk;
            if (k < b) {                    // (block-uniform)
                double *row = rb[kk & 1];
                if (r == k) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) row[c0 + i] = v[i];
                }
                __syncthreads();
                const double piv = row[k], rk = row[r];
                ok = ok && (p0 + k < d.pos_end ? piv > 0.0 : piv < 0.0) && isfinite(piv);
                const double inv = 1.0 / piv, f = r == k ? -inv : rk * inv;
                if (r == k) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) v[i] = 0.0;
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) v[i] -= f * row[c0 + i];
                if (cq == kb) v[kk] = f;
            }
        }
    }
    if (!ok && t == 0) atomicMax(status, 1);
    double *P = d.P() + r * TS + c0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        P[i] = v[i];
        if (r < b && c0 + i < b) d.A[(p0 + r) * d.ld + p0 + c0 + i] = v[i];
    }
}

// U = A(P, J) (read from the rows of the upper triangle: transposed for the
// column tiles left of the panel), X = A_PP^{-1} U = -P U.  Operand layout of
// v_mfma_f64_16x16x4f64: A[i][k] and B[k][j] in lane i (j) + 16 k, result
// (i, j) in lane j + 16 (i % 4), register i / 4.
__global__ void __launch_bounds__(256) k_sweep_cols(const Mat *mats, const Item *items, int s) {
    __shared__ double us[TS][LDT];
    const Item it = items[blockIdx.x];
    const Mat d = mats[it.mat];
    const int p0 = TS * s, b = min(TS, d.p1 - p0), J0 = it.J * TS, n = d.n;
    const int t = threadIdx.x, w = t >> 6, L = t & 63, li = L & 15, lk = L >> 4;
    const bool left = it.J < s;
    const int own1 = p0 + b;        // own columns: [p0, own1)
#pragma unroll 4
    for (int q = 0; q < TS / 4; ++q) {      // line w + 4 q of the tile, entry L
        const int a = w + 4 * q;
        const int k = left ? L : a, j = J0 + (left ? a : L);
        const bool live = k < b && j < n && !(j >= p0 && j < own1);
        us[k][j - J0] = live ? (left ? d.A[j * d.ld + p0 + k] : d.A[(p0 + k) * d.ld + j]) : 0.0;
    }
    __syncthreads();
    double *U = d.U(it.J), *X = d.X(it.J);
    const double *P = d.P();
    for (int e = t; e < TT; e += 256) U[e] = us[e >> 6][e & 63];
    dvec4 acc[4];
#pragma unroll
    for (int tc = 0; tc < 4; ++tc) acc[tc] = dvec4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int q = 0; q < TS / 4; ++q) {
        const int k = 4 * q + lk;
        const double a = -P[k * TS + 16 * w + li];     // (P is symmetric)
#pragma unroll
        for (int tc = 0; tc < 4; ++tc)
            acc[tc] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, us[k][16 * tc + li], acc[tc], 0, 0, 0);
    }
    __syncthreads();
#pragma unroll
    for (int tc = 0; tc < 4; ++tc)
#pragma unroll
        for (int q = 0; q < 4; ++q) us[16 * w + lk + 4 * q][16 * tc + li] = acc[tc][q];
    __syncthreads();
    for (int e = t; e < TT; e += 256) X[e] = us[e >> 6][e & 63];
#pragma unroll 4
    for (int q = 0; q < TS / 4; ++q) {
        const int a = w + 4 * q;
        const int k = left ? L : a, j = J0 + (left ? a : L);
        if (k < b && j < n && !(j >= p0 && j < own1)) {
            // (a last panel of b < 64 pivots: both halves of its diagonal tile)
            if (it.J <= s) d.A[j * d.ld + p0 + k] = us[k][j - J0];
            if (it.J >= s) d.A[(p0 + k) * d.ld + j] = us[k][j - J0];
        }
    }
}

// Blocks go to the 8 XCDs in turn; each XCD takes a consecutive eighth of the
// list, so that a matrix's U and X are read into one L2 instead of eight (update
// tiles of one setup: 64^3 7.7 -> 6.9 ms, 192^3 206 -> 192, holed 64^3 31 -> 28).
constexpr int XCDS = 8;
__device__ __forceinline__ int xcd_item(int n) {
    const int per = (n + XCDS - 1) / XCDS, i = (int)(blockIdx.x / XCDS), x = blockIdx.x % XCDS;
    return x * per + i < n ? x * per + i : -1;
}

// A <- A - U^T X over one 64 x 64 tile: wave w takes rows 16 w .. + 15 and the
// four 16-column tiles; X staged in LDS, U's 16 columns in registers.
__global__ void __launch_bounds__(256) k_sweep_update(const Mat *mats, const Item *items, int nitems) {
    __shared__ double xs[TS][LDX];
    const int id = xcd_item(nitems);
    if (id < 0) return;
    const Item it = items[id];
    const Mat d = mats[it.mat];
    const int n = d.n, I0 = it.I * TS, J0 = it.J * TS;
    const int t = threadIdx.x, w = t >> 6, L = t & 63, li = L & 15, lk = L >> 4;
    const double2 *X = reinterpret_cast<const double2 *>(d.X(it.J));
    const double *U = d.U(it.I) + 16 * w + li;
    double2 xv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) xv[u] = X[t + 256 * u];
    double uv[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) uv[q] = U[(4 * q + lk) * TS];
    dvec4 acc[4];
    const bool full = I0 + TS <= n && J0 + TS <= n;
    double *A = d.A + (I0 + 16 * w + lk) * d.ld + J0 + li;     // this lane's entries: + 4 q rows, + 16 tc columns
    if (full) {
#pragma unroll
        for (int tc = 0; tc < 4; ++tc)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[tc][q] = A[4 * q * d.ld + 16 * tc];
    } else {
#pragma unroll
        for (int tc = 0; tc < 4; ++tc)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc[tc][q] = (I0 + 16 * w + lk + 4 * q < n && J0 + 16 * tc + li < n) ? A[4 * q * d.ld + 16 * tc] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int e = 2 * (t + 256 * u);
        *reinterpret_cast<double2 *>(&xs[e >> 6][e & 63]) = xv[u];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
#pragma unroll
        for (int tc = 0; tc < 4; ++tc)
            acc[tc] = __builtin_amdgcn_mfma_f64_16x16x4f64(-uv[q], xs[4 * q + lk][16 * tc + li], acc[tc], 0, 0, 0);
    }
    if (full) {
#pragma unroll
        for (int tc = 0; tc < 4; ++tc)
#pragma unroll
            for (int q = 0; q < 4; ++q) A[4 * q * d.ld + 16 * tc] = acc[tc][q];
    } else {
#pragma unroll
        for (int tc = 0; tc < 4; ++tc)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (I0 + 16 * w + lk + 4 * q < n && J0 + 16 * tc + li < n) A[4 * q * d.ld + 16 * tc] = acc[tc][q];
    }
}

// the lower triangle of tiles from the upper one
__global__ void __launch_bounds__(256) k_sweep_mirror(const Mat *mats, const Item *items) {
    __shared__ double x[TS][LDT];
    const Item it = items[blockIdx.x];
    if (it.I == it.J) return;
    const Mat d = mats[it.mat];
    const int n = d.n, I0 = it.I * TS, J0 = it.J * TS, w = threadIdx.x >> 6, L = threadIdx.x & 63;
#pragma unroll 4
    for (int q = 0; q < TS / 4; ++q) {
        const int i = w + 4 * q;
        x[i][L] = (I0 + i < n && J0 + L < n) ? d.A[(I0 + i) * d.ld + J0 + L] : 0.0;
    }
    __syncthreads();
#pragma unroll 4
    for (int q = 0; q < TS / 4; ++q) {
        const int j = w + 4 * q;
        if (J0 + j < n && I0 + L < n) d.A[(J0 + j) * d.ld + I0 + L] = x[L][j];
    }
}

// Host plan: matrices with pivots, the most pivots first, in batches whose
// panel buffers fit PANEL_CAP (every batch reuses the buffer).
struct Plan {
    std::vector<int> order;                 // matrices in processing order
    std::vector<size_t> batch;              // first position of every batch, then the end
    size_t panel = 0;                       // bytes of the largest batch's buffers
    size_t tiles = 0, cols = 0;             // list entries
};
int tiles_of(const SweepDesc &h) { return (h.n + TS - 1) / TS; }
size_t panel_bytes(const SweepDesc &h) { return (2 * (size_t)tiles_of(h) + 1) * TT * sizeof(double); }

Plan make_plan(const std::vector<SweepDesc> &h) {
    Plan p;
    for (size_t i = 0; i < h.size(); ++i)
        if (h[i].p1 > 0 && h[i].n > 0) p.order.push_back((int)i);
    std::stable_sort(p.order.begin(), p.order.end(), [&](int a, int b) { return h[a].p1 > h[b].p1; });
    size_t bytes = 0;
    for (size_t q = 0; q < p.order.size(); ++q) {
        const SweepDesc &x = h[p.order[q]];
        if (p.batch.empty() || bytes + panel_bytes(x) > PANEL_CAP) {
            p.batch.push_back(q);
            bytes = 0;
        }
        bytes += panel_bytes(x);
        p.panel = std::max(p.panel, bytes);
        const size_t T = tiles_of(x);
        p.tiles += T * (T + 1) / 2;
        p.cols += T;
    }
    p.batch.push_back(p.order.size());
    return p;
}

size_t up256(size_t x) { return (x + 255) & ~size_t(255); }
size_t lists_bytes(const Plan &p) {
    return up256(p.order.size() * sizeof(Mat)) + up256(p.tiles * sizeof(Item)) + up256(p.cols * sizeof(Item));
}

}  // namespace

size_t sweep_workspace_bound(size_t count, int n) {
    const SweepDesc x{nullptr, n, n, n, n};
    const size_t T = tiles_of(x), pb = panel_bytes(x);
    return up256(count * sizeof(Mat)) + up256(count * T * (T + 1) / 2 * sizeof(Item)) + up256(count * T * sizeof(Item)) +
           std::max<size_t>(256, count * pb <= PANEL_CAP ? count * pb : std::max(PANEL_CAP, pb));
}

size_t sweep_workspace(const std::vector<SweepDesc> &h) {
    const Plan p = make_plan(h);
    return std::max<size_t>(256, lists_bytes(p) + p.panel);
}

int launch_sweeps(const std::vector<SweepDesc> &h, void *ws, int *status, hipStream_t s) {
    const Plan p = make_plan(h);
    if (p.order.empty()) return 0;
    const size_t nm = p.order.size(), o1 = up256(nm * sizeof(Mat)), o2 = o1 + up256(p.tiles * sizeof(Item)),
                 o3 = lists_bytes(p);
    std::vector<char> host(o3, 0);
    Mat *mats = reinterpret_cast<Mat *>(host.data());
    Item *tiles = reinterpret_cast<Item *>(host.data() + o1), *cols = reinterpret_cast<Item *>(host.data() + o2);
    char *dev = static_cast<char *>(ws);
    std::vector<size_t> te(nm + 1, 0), ce(nm + 1, 0);      // list entries before matrix q
    for (size_t b = 0; b + 1 < p.batch.size(); ++b) {
        size_t off = 0;
        for (size_t q = p.batch[b]; q < p.batch[b + 1]; ++q) {
            const SweepDesc &x = h[p.order[q]];
            const int T = tiles_of(x);
            mats[q] = Mat{x.A, x.ld, reinterpret_cast<double *>(dev + o3 + off), x.n, x.p1, x.pos_end, T};
            off += panel_bytes(x);
            size_t t = te[q], c = ce[q];
            for (int I = 0; I < T; ++I) {
                cols[c++] = Item{(int32_t)q, 0, I};
                for (int J = I; J < T; ++J) tiles[t++] = Item{(int32_t)q, I, J};
            }
            te[q + 1] = t;
            ce[q + 1] = c;
        }
    }
    // (synchronous: the host lists end with this call)
    if (hipMemcpy(dev, host.data(), o3, hipMemcpyHostToDevice) != hipSuccess) return -1;
    const Mat *dm = reinterpret_cast<const Mat *>(dev);
    const Item *dt = reinterpret_cast<const Item *>(dev + o1), *dc = reinterpret_cast<const Item *>(dev + o2);
    for (size_t b = 0; b + 1 < p.batch.size(); ++b) {
        const size_t q0 = p.batch[b];
        size_t q1 = p.batch[b + 1];
        for (int st = 0; TS * st < h[p.order[q0]].p1; ++st) {
            while (h[p.order[q1 - 1]].p1 <= TS * st) --q1;
            hipLaunchKernelGGL(k_sweep_diag, dim3((unsigned)(q1 - q0)), dim3(256), 0, s, dm + q0, st, status);
            hipLaunchKernelGGL(k_sweep_cols, dim3((unsigned)(ce[q1] - ce[q0])), dim3(256), 0, s, dm, dc + ce[q0], st);
            hipLaunchKernelGGL(k_sweep_update, dim3((unsigned)((te[q1] - te[q0] + XCDS - 1) / XCDS * XCDS)), dim3(256), 0, s, dm,
                               dt + te[q0], (int)(te[q1] - te[q0]));
        }
        q1 = p.batch[b + 1];
        hipLaunchKernelGGL(k_sweep_mirror, dim3((unsigned)(te[q1] - te[q0])), dim3(256), 0, s, dm, dt + te[q0]);
    }
    return 0;
}

}  // namespace bddc
