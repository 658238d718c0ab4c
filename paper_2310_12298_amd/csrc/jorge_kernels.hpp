// Bandwidth-bound and scalar kernels of the Jorge step for gfx950.
#pragma once

#include <hip/hip_runtime.h>

#include "jorge_gemm.hpp"
#include "jorge_types.hpp"

namespace jorge {

constexpr int kEwThreads = 256;

// Fixed-order sum of n doubles by one wave (every lane gets the total).
__device__ __forceinline__ double wave_sum_array(const double* __restrict__ x, int n) {
    double v = 0.0;
    for (int i = threadIdx.x & 63; i < n; i += 64) v += x[i];
    return wave_sum(v);
}

// Zeroes n 16-byte words (a fill kernel rather than a memset, so that the
// clearing is an ordinary kernel node if the caller captures it).
__global__ __launch_bounds__(kEwThreads) void zero_kernel(f32x4* __restrict__ p, size_t n) {
    const f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
    for (size_t i = (size_t)blockIdx.x * kEwThreads + threadIdx.x; i < n; i += (size_t)gridDim.x * kEwThreads) p[i] = z;
}

// One layer's state copied between the caller's dense tensors and the library's
// scratch: in (out = 0), each tensor with its padding set to zero, or out. One row
// of workgroups (blockIdx.y) per tensor.
struct LentState {
    struct {
        float* user;  // dense rows x cols
        float* held;  // prows x ld, rows x cols of it valid
        int rows, cols, prows, ld;
    } t[4];
};
__global__ __launch_bounds__(kEwThreads) void lent_state_kernel(LentState s, int out) {
    const auto& t = s.t[blockIdx.y];
    const unsigned width = out ? t.cols : t.ld, n = width * (unsigned)(out ? t.rows : t.prows);
    for (unsigned i = blockIdx.x * kEwThreads + threadIdx.x; i < n; i += gridDim.x * kEwThreads) {
        const unsigned r = i / width, c = i - r * width;
        if (out) t.user[i] = t.held[r * (unsigned)t.ld + c];
        else t.held[i] = r < (unsigned)t.rows && c < (unsigned)t.cols ? t.user[r * (unsigned)t.cols + c] : 0.0f;
    }
}

// A_hat = eps^(-1/4) I on the valid diagonal of every factor (the arena is zeroed before).
__global__ void init_factors_kernel(const FactorDev* __restrict__ f, float l0) {
    const FactorDev F = f[blockIdx.x];
    for (int i = threadIdx.x; i < F.d; i += blockDim.x) F.A[(size_t)i * F.dp + i] = l0;
}

// Gradient stage-in over 64 x 64 blocks: copies G (dense m x n, caller's
// buffer) into the padded operand Gp and its transpose Gpt, updates
// m_SGD = beta1 m_SGD + G (Algorithm 3) and writes the block's sum of m_SGD^2.
// Each thread moves groups of four consecutive elements: 16-byte accesses
// where the layer's rows allow them (n a multiple of 4, G 16-byte aligned),
// element by element otherwise. Rows are read and the transpose is written
// in 256-byte runs per 16 threads; the transpose goes through LDS.
__global__ __launch_bounds__(kEwThreads) void stagein_kernel(const LayerDev* __restrict__ layers,
                                                             const StageTile* __restrict__ tiles,
                                                             int layer_base, PtrBatch grads,
                                                             float beta1) {
    __shared__ float blk[64][65];
    __shared__ double red[4];
    const StageTile st = tiles[blockIdx.x];
    const LayerDev& L = layers[st.layer];
    const float* __restrict__ G = grads.p[st.layer - layer_base];
    const int m = L.m, n = L.n;
    const bool vec = (n & 3) == 0 && (reinterpret_cast<uintptr_t>(G) & 15) == 0;
    double part = 0.0;
    // Row r, columns c .. c+3 of the block, for q = 16 r + c / 4.
    if (vec) {
        // Every load of the thread is issued before its first store, so
        // eight 16-byte loads are in flight at once (no store overwrites what
        // a later load of the thread reads, which the compiler cannot prove
        // by itself). The loads are unconditional: a position outside the
        // layer reads the nearest one inside it (n >= 4) and its values are
        // dropped.
        constexpr int kIt = 64 * 16 / kEwThreads;
        float* __restrict__ msgd = L.msgd;
        float* __restrict__ Gp = L.Gp;
        const size_t np = (size_t)L.np;
        f32x4 g[kIt], ms[kIt];
#pragma unroll
        for (int i = 0; i < kIt; ++i) {
            const int q = threadIdx.x + i * kEwThreads;
            const int gr = min(st.r0 + (q >> 4), m - 1), gc = min(st.c0 + (q & 15) * 4, n - 4);
            const size_t gi = (size_t)gr * n + gc;
            g[i] = gload4(G + gi);
            ms[i] = gload4(msgd + gi);
        }
#pragma unroll
        for (int i = 0; i < kIt; ++i) {
            const int q = threadIdx.x + i * kEwThreads, r = q >> 4, c = (q & 15) * 4;
            const int gr = st.r0 + r, gc = st.c0 + c;
#pragma unroll
            for (int j = 0; j < 4; ++j) blk[r][c + j] = g[i][j];
            if (gr >= m || gc >= n) continue;  // gc + 3 < n: n and gc are multiples of 4
            const size_t gi = (size_t)gr * n + gc;
            f32x4 v;
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = beta1 * ms[i][j] + g[i][j];
            *(gfloat4*)(Gp + (size_t)gr * np + gc) = g[i];
            *(gfloat4*)(msgd + gi) = v;
#pragma unroll
            for (int j = 0; j < 4; ++j) part += (double)v[j] * (double)v[j];
        }
    } else {
        for (int q = threadIdx.x; q < 64 * 16; q += kEwThreads) {
            const int r = q >> 4, c = (q & 15) * 4, gr = st.r0 + r, gc = st.c0 + c;
            if (gr >= m || gc >= n) continue;
            const size_t gi = (size_t)gr * n + gc;
            f32x4 g;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                g[j] = 0.0f;
                if (gc + j < n) {
                    g[j] = G[gi + j];
                    L.Gp[(size_t)gr * L.np + gc + j] = g[j];
                    const float w = beta1 * L.msgd[gi + j] + g[j];
                    L.msgd[gi + j] = w;
                    part += (double)w * (double)w;
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) blk[r][c + j] = g[j];
        }
    }
    __syncthreads();
    // Column c, rows r .. r+3 of the block: Gpt[c][r..r+3] (mp is a multiple of 32).
    for (int q = threadIdx.x; q < 64 * 16; q += kEwThreads) {
        const int c = q >> 4, r = (q & 15) * 4, gr = st.r0 + r, gc = st.c0 + c;
        if (gc >= n || gr >= m) continue;
        float* dst = L.Gpt + (size_t)gc * L.mp + gr;
        if (gr + 3 < m) {
            f32x4 t;
#pragma unroll
            for (int j = 0; j < 4; ++j) t[j] = blk[r + j][c];
            *reinterpret_cast<f32x4*>(dst) = t;
        } else {
            for (int j = 0; gr + j < m; ++j) dst[j] = blk[r + j][c];
        }
    }
    const double total = block_sum_256(part, red);
    if (threadIdx.x == 0) L.part_sgd[st.slot] = total;
}

// (beta, c, s) of one factor update from nu = ||X||_F (Algorithm 2; Appendix
// A.1, Eq. 8-9). The dynamic branch forms c = 1/nu and s = (1 + 1/nu)^(1/4)
// directly, never 1 - beta.
__device__ __forceinline__ FactorScalars factor_scalars(double nu, double beta2, int mode) {
    bool dyn = false;
    if (mode == 1) dyn = nu > 0.0;                           // DYNAMIC
    else if (mode == 2) dyn = nu > beta2 / (1.0 - beta2);    // CLAMPED: nu/(nu+1) > beta2
    FactorScalars out;
    if (dyn) {
        out.beta = nu / (nu + 1.0);
        out.c = 1.0 / nu;
        out.s = sqrt(sqrt(1.0 + 1.0 / nu));  // (1 + 1/nu)^(1/4)
    } else {
        out.beta = beta2;
        out.c = (1.0 - beta2) / beta2;
        out.s = 1.0 / sqrt(sqrt(beta2));     // beta2^(-1/4)
    }
    out.nu = nu;
    out.a = (float)(0.25 * out.c);
    out.b = (float)(0.15625 * out.c * out.c);
    out.sf = (float)out.s;
    out.e = (float)(0.1171875 * out.c * out.c * out.c);
    return out;
}

// nu = ||X||_F from the per-tile partial sums, then the factor's scalars.
// One wave per factor of the list (the factors of the grouped levels). The factored form's partials are terms of an inner
// product of two positive semidefinite matrices whose exact sum is ||X||_F^2;
// a sum that rounding left below zero is read as zero.
__global__ void factor_finalize_kernel(const FactorDev* __restrict__ f, const int* __restrict__ list,
                                       double beta2, int mode) {
    const FactorDev F = f[list[blockIdx.x]];
    const double nu = sqrt(fmax(0.0, wave_sum_array(F.partials, F.nparts)));
    if (threadIdx.x == 0) *F.sc = factor_scalars(nu, beta2, mode);
}

// A_hat <- (Z + Z^T)/2 (or Z when not symmetrizing) for the pair of 64 x 64
// tiles (ti, tj), (tj, ti) of a factor in the explicit form; a diagonal tile
// (ti = tj) is its own partner and is read once. fp32 addition commutes, so
// the result is bitwise symmetric. za, zb: 64 x 65 floats of LDS each. All
// threads of the workgroup call it; it ends with a barrier so the LDS can be
// reused. Global memory is addressed as such (not through generic pointers).
__device__ __forceinline__ void symmetrize_pair(const FactorDev& F, int ti, int tj, int symmetrize,
                                                float (*za)[65], float (*zb)[65]) {
    const int dp = F.dp, i0 = ti * 64, j0 = tj * 64;
    const int tid = threadIdx.x;
    const bool diag = ti == tj;
    float (*const pb)[65] = diag ? za : zb;  // the partner tile's LDS copy
    // 64 rows x 16 float4 per tile, 4 per thread; every load before the first LDS store.
    f32x4 va[4], vb[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int u = tid + q * kEwThreads, r = u >> 4, c = (u & 15) * 4;
        if (i0 + r < dp && j0 + c < dp) va[q] = gload4(F.Z + (size_t)(i0 + r) * dp + j0 + c);
        if (!diag && j0 + r < dp && i0 + c < dp) vb[q] = gload4(F.Z + (size_t)(j0 + r) * dp + i0 + c);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int u = tid + q * kEwThreads, r = u >> 4, c = (u & 15) * 4;
        if (i0 + r < dp && j0 + c < dp) {
            za[r][c] = va[q][0]; za[r][c + 1] = va[q][1]; za[r][c + 2] = va[q][2]; za[r][c + 3] = va[q][3];
        }
        if (!diag && j0 + r < dp && i0 + c < dp) {
            zb[r][c] = vb[q][0]; zb[r][c + 1] = vb[q][1]; zb[r][c + 2] = vb[q][2]; zb[r][c + 3] = vb[q][3];
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int u = tid + q * kEwThreads, r = u >> 4, c = (u & 15) * 4;
        if (i0 + r < dp && j0 + c < dp) {
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[e] = symmetrize ? 0.5f * (za[r][c + e] + pb[c + e][r]) : za[r][c + e];
            *(gfloat4*)(F.A + (size_t)(i0 + r) * dp + j0 + c) = v;
        }
        if (!diag && j0 + r < dp && i0 + c < dp) {
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[e] = symmetrize ? 0.5f * (zb[r][c + e] + za[c + e][r]) : zb[r][c + e];
            *(gfloat4*)(F.A + (size_t)(j0 + r) * dp + i0 + c) = v;
        }
    }
    __syncthreads();
}

__global__ __launch_bounds__(kEwThreads) void symmetrize_kernel(const FactorDev* __restrict__ f,
                                                                const SymTile* __restrict__ tiles,
                                                                int symmetrize) {
    __shared__ float za[64][65];
    __shared__ float zb[64][65];
    const SymTile st = tiles[blockIdx.x];
    symmetrize_pair(f[st.factor], st.ti, st.tj, symmetrize, za, zb);
}

// ---------------------------------------------------------------- small contexts
// Contexts whose factors all have padded size <= 128. A factor's whole update
// runs in one team of waves, in the explicit order of Algorithm 2 with its
// matrices in LDS: A^2, A^4, M = H H^T, X = A^4 M with ||X||_F, (beta, c, s)
// (Appendix A.1, Eq. 8-9), P - I = -(c/4) X + (5c^2/32) X X (Eq. 6; with series
// order 3, -a X + X V, V = b X - e X X), Z = s A + s A (P - I) and A <- (Z + Z^T)/2 (or
// Z). The rest of the step (m_SGD, L G R, momentum, norms, grafted weight update)
// runs in one workgroup per layer, which holds the gradient in LDS and sums the
// norms itself, so nothing of the step but its state passes through memory.
//
// Every product is C = A B with both operands held in LDS as fp32 rows that
// are contiguous in k: A's rows and B's columns (the rows of B^T). They are
// split into bf16 terms as they are read (split_pair): a piece of 16 BI x
// 16 BJ costs BI + BJ splits per 6 BI BJ MFMAs. What bounds a team is the chain
// of six dependent products with barriers between them.

// A team of WAVES waves works on matrices of at most D x D; its product is cut
// into pieces of 16 BI x 16 BJ, one per wave, GRID_X to a row.
template <int D_, int WAVES_, int BI_, int BJ_>
struct Team {
    static constexpr int D = D_, WAVES = WAVES_, BI = BI_, BJ = BJ_, THREADS = 64 * WAVES_;
    static constexpr int GRID_X = D_ / (16 * BJ_);
    static constexpr int LD = D_ + 4;              // LDS row stride: 16-byte reads of 16 rows fall in distinct bank quads
    static constexpr int MAT = D_ * LD;            // floats per LDS matrix
    static constexpr int AV = D_ * D_ / 4 / THREADS;  // 16-byte pieces of a factor per thread
    static constexpr int GV = D_ * D_ / THREADS;      // gradient elements per thread
    static_assert(WAVES_ / GRID_X * 16 * BI_ == D_, "the pieces cover the product");
};
typedef Team<64, 4, 2, 2> Team64;     // a factor up to 64
typedef Team<128, 8, 4, 2> Team128;   // a factor up to 128; the rest of a layer's step
typedef Team<64, 8, 2, 1> Apply64;    // the rest of the step of a layer with m, n <= 64
constexpr int kSmallThreads = 512;

// A wave's piece of an M x N product (M, N multiples of 32): first row and
// column, and how many of its 16-row blocks lie inside (0: none of the piece).
struct Piece {
    int row, col, nbi;
};
template <class T>
__device__ __forceinline__ Piece piece_of(int wave, int M, int N) {
    Piece p;
    p.row = wave / T::GRID_X * (16 * T::BI);
    p.col = wave % T::GRID_X * (16 * T::BJ);
    p.nbi = p.col < N ? max(0, min(T::BI, (M - p.row) / 16)) : 0;
    return p;
}

// acc += a (rows) x b^T (rows) over k in [0, K), K a multiple of 32, for NBI of
// the piece's block rows. Lane l takes k = k0 + 4 (l / 16) .. + 3 and k0 + 16 + 4
// (l / 16) .. + 3 of row l % 16 of a block, for a and b alike, so every product
// is formed once. The next 32 k are read while the current ones are multiplied.
template <class T, int NBI>
__device__ __forceinline__ void piece_mma_n(const float* a, const float* b, int K, f32x4 (&acc)[T::BI * T::BJ]) {
    constexpr int LD = T::LD, BJ = T::BJ;
    constexpr int kA[6] = {2, 1, 0, 1, 0, 0}, kB[6] = {0, 1, 2, 0, 1, 0};
    const int lane = threadIdx.x & 63;
    const float* pa = a + (lane & 15) * LD + 4 * (lane >> 4);
    const float* pb = b + (lane & 15) * LD + 4 * (lane >> 4);
    f32x4 fa[NBI][2], fb[BJ][2];
    auto read = [&](int k0) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int j = 0; j < BJ; ++j) fb[j][h] = *reinterpret_cast<const f32x4*>(pb + 16 * j * LD + k0 + 16 * h);
#pragma unroll
            for (int i = 0; i < NBI; ++i) fa[i][h] = *reinterpret_cast<const f32x4*>(pa + 16 * i * LD + k0 + 16 * h);
        }
    };
    unsigned lost = 0;
    read(0);
    for (int k0 = 0; k0 < K; k0 += 32) {
        SplitOct sb[BJ], sa[NBI];
#pragma unroll
        for (int j = 0; j < BJ; ++j) sb[j] = split_oct(fb[j][0], fb[j][1], lost);
#pragma unroll
        for (int i = 0; i < NBI; ++i) sa[i] = split_oct(fa[i][0], fa[i][1], lost);
        read(k0 + 32 < K ? k0 + 32 : 0);  // past the end: group 0 again, never multiplied
#pragma unroll
        for (int i = 0; i < NBI; ++i)
#pragma unroll
            for (int u = 0; u < 6; ++u)
#pragma unroll
                for (int j = 0; j < BJ; ++j)
                    acc[i * BJ + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sa[i].t[kA[u]], sb[j].t[kB[u]],
                                                                             acc[i * BJ + j], 0, 0, 0);
    }
    if (__builtin_expect(__any(split_lost(lost) || any_non_finite(acc)), 0)) {  // see fp32_blocks
#pragma unroll
        for (int q = 0; q < NBI * BJ; ++q) acc[q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
        for (int k0 = 0; k0 < K; k0 += 16) {
            f32x4 ga[NBI], gb[BJ];
#pragma unroll
            for (int j = 0; j < BJ; ++j) gb[j] = *reinterpret_cast<const f32x4*>(pb + 16 * j * LD + k0);
#pragma unroll
            for (int i = 0; i < NBI; ++i) ga[i] = *reinterpret_cast<const f32x4*>(pa + 16 * i * LD + k0);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < NBI; ++i)
#pragma unroll
                    for (int j = 0; j < BJ; ++j)
                        acc[i * BJ + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ga[i][e], gb[j][e], acc[i * BJ + j], 0, 0, 0);
        }
    }
}

// The wave's piece of a product (acc from zero); a piece outside it does nothing.
template <class T>
__device__ __forceinline__ void piece_mma(const Piece& p, const float* a, const float* b, int K,
                                          f32x4 (&acc)[T::BI * T::BJ]) {
#pragma unroll
    for (int i = 0; i < T::BI * T::BJ; ++i) acc[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const float* pa = a + p.row * T::LD;
    const float* pb = b + p.col * T::LD;
    if (p.nbi == T::BI) piece_mma_n<T, T::BI>(pa, pb, K, acc);
    else if (T::BI > 2 && p.nbi == 2) piece_mma_n<T, 2>(pa, pb, K, acc);
}

// Every element of the wave's piece: f(row, col, block, e), e-th of four
// consecutive rows of a column.
template <class T, typename Fn>
__device__ __forceinline__ void piece_each(const Piece& p, Fn f) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < T::BI; ++i) {
        if (i >= p.nbi) continue;
#pragma unroll
        for (int j = 0; j < T::BJ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                f(p.row + 16 * i + 4 * (lane >> 4) + e, p.col + 16 * j + (lane & 15), i * T::BJ + j, e);
    }
}

// The wave's blocks to LDS: m[row][col], or with TR m[col][row] (four
// consecutive rows of a column are one 16-byte store).
template <class T, bool TR>
__device__ __forceinline__ void piece_store(const Piece& p, float* m, const f32x4 (&v)[T::BI * T::BJ]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < T::BI; ++i) {
        if (i >= p.nbi) continue;
#pragma unroll
        for (int j = 0; j < T::BJ; ++j) {
            const int row = p.row + 16 * i + 4 * (lane >> 4), col = p.col + 16 * j + (lane & 15);
            if constexpr (TR) {
                *reinterpret_cast<f32x4*>(m + col * T::LD + row) = v[i * T::BJ + j];
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) m[(row + e) * T::LD + col] = v[i * T::BJ + j][e];
            }
        }
    }
}

// A factor (dp x dp, global) through registers to LDS rows, or with tr its
// transpose: thread t holds columns 4 (t % (D / 4)) .. + 3 of rows t / (D / 4) + i (4
// THREADS / D). Positions outside are read from the nearest one inside, and land
// in rows and columns of the LDS matrix that no product reads.
template <class T>
__device__ __forceinline__ void factor_load(int t, const float* __restrict__ A, int dp, f32x4 (&r)[T::AV]) {
    const int c = min(4 * (t % (T::D / 4)), dp - 4);
#pragma unroll
    for (int i = 0; i < T::AV; ++i) {
        const int row = min(t / (T::D / 4) + i * (4 * T::THREADS / T::D), dp - 1);
        r[i] = *(global_f32x4*)((const gcchar*)A + 4u * (unsigned)(row * dp + c));
    }
}
template <class T>
__device__ __forceinline__ void factor_store(int t, const f32x4 (&r)[T::AV], float* m, bool tr) {
    const int c = 4 * (t % (T::D / 4));
#pragma unroll
    for (int i = 0; i < T::AV; ++i) {
        const int row = t / (T::D / 4) + i * (4 * T::THREADS / T::D);
        if (tr) {
#pragma unroll
            for (int q = 0; q < 4; ++q) m[(c + q) * T::LD + row] = r[i][q];
        } else {
            *reinterpret_cast<f32x4*>(m + row * T::LD + c) = r[i];
        }
    }
}

// The gradient (m x n, row stride ld, any alignment) through registers: thread t holds
// column t % D of rows t / D + i (THREADS / D), zero outside the layer. The loads are
// unconditional (positions outside read the nearest one inside), so all are in
// flight at once.
template <class T>
__device__ __forceinline__ void grad_load(int t, const float* __restrict__ G, int m, int n, int ld, float (&r)[T::GV]) {
    const int c = t % T::D, cc = min(c, n - 1);
#pragma unroll
    for (int i = 0; i < T::GV; ++i) {
        const int row = t / T::D + i * (T::THREADS / T::D);
        r[i] = ld_at(G, 4u * (unsigned)(min(row, m - 1) * ld + cc));
    }
#pragma unroll
    for (int i = 0; i < T::GV; ++i) {
        const int row = t / T::D + i * (T::THREADS / T::D);
        r[i] = (row < m && c < n) ? r[i] : 0.0f;
    }
}
// To LDS rows, or with tr its transpose (the whole D x D matrix, zero outside the layer).
template <class T>
__device__ __forceinline__ void grad_store(int t, const float (&r)[T::GV], float* l, bool tr) {
    const int c = t % T::D;
#pragma unroll
    for (int i = 0; i < T::GV; ++i) {
        const int row = t / T::D + i * (T::THREADS / T::D);
        l[tr ? c * T::LD + row : row * T::LD + c] = r[i];
    }
}

// Sum of one double per thread over the first N waves of red, in index order (after a barrier).
template <int N>
__device__ __forceinline__ double sum_waves(const double* red) {
    double v = red[0];
#pragma unroll
    for (int w = 1; w < N; ++w) v += red[w];
    return v;
}

// One factor's update by a team (threads t = 0 .. T::THREADS - 1, wave = t / 64).
// m0, m1: two LDS matrices of T::MAT floats; red: T::WAVES doubles. g: the layer's
// gradient in the team's registers, with WIDE its first D columns (rows for R_hat):
// the others, if kp > D, are loaded under the product of the first (deep: some team of
// the workgroup has such a factor). live: the team stores its results. Every thread of the
// workgroup calls it (all its teams meet the same barriers). On return the new
// factor is in global memory and, for side R of a non-symmetric factor
// transposed, in m1 (behind a barrier).
template <class T, bool WIDE = false>
__device__ __forceinline__ void chain_update(const FactorDev& F, int side, int t, int wave, float (&g)[T::GV],
                                             const LayerDev& L, const float* __restrict__ G, bool deep, bool live,
                                             double beta2, int mode, int symmetrize, int order, float* m0, float* m1,
                                             double* red) {
    constexpr int NB = T::BI * T::BJ;
    const int dp = F.dp, kp = F.kp;
    const Piece p = piece_of<T>(wave, dp, dp);
    f32x4 av[T::AV], acc[NB];
    factor_load<T>(t, F.A, dp, av);
    factor_store<T>(t, av, m0, false);
    if (!symmetrize) factor_store<T>(t, av, m1, true);
    __syncthreads();
    // A^2 and A^4, each over the last in m0 (its transpose in m1 when not symmetric)
    piece_mma<T>(p, m0, symmetrize ? m0 : m1, dp, acc);
    __syncthreads();
    piece_store<T, false>(p, m0, acc);
    if (!symmetrize) piece_store<T, true>(p, m1, acc);
    __syncthreads();
    piece_mma<T>(p, m0, symmetrize ? m0 : m1, dp, acc);
    __syncthreads();
    piece_store<T, false>(p, m0, acc);
    // H: G for L_hat, G^T for R_hat
    grad_store<T>(t, g, m1, side != 0);
    __syncthreads();
    // M = H H^T
    const bool more = WIDE && kp > T::D;
    if (more) {
        if (side == 0) grad_load<T>(t, G + T::D, L.m, L.n - T::D, L.n, g);
        else grad_load<T>(t, G + T::D * L.n, L.m - T::D, L.n, L.n, g);
    }
    piece_mma<T>(p, m1, m1, more ? T::D : kp, acc);
    __syncthreads();
    if (WIDE && deep) {
        if (more) grad_store<T>(t, g, m1, side != 0);
        __syncthreads();
        f32x4 rest[NB];
        piece_mma<T>(p, m1, m1, more ? kp - T::D : 0, rest);
#pragma unroll
        for (int q = 0; q < NB; ++q) acc[q] += rest[q];
        __syncthreads();
    }
    piece_store<T, false>(p, m1, acc);
    __syncthreads();
    // X = A^4 M (M symmetric: its rows are its columns) with ||X||_F^2; the wave
    // keeps its piece of X in x.
    f32x4 x[NB];
    piece_mma<T>(p, m0, m1, dp, x);
    double part = 0.0;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) part += (double)x[b][e] * (double)x[b][e];
    part = wave_sum(part);
    if ((t & 63) == 0) red[wave] = part;
    __syncthreads();
    piece_store<T, false>(p, m0, x);
    piece_store<T, true>(p, m1, x);
    // A again, for Z: its loads run under the next product.
    f32x4 av2[T::AV];
    factor_load<T>(t, F.A, dp, av2);
    const FactorScalars fs = factor_scalars(sqrt(sum_waves<T::WAVES>(red)), beta2, mode);
    if (t == 0 && live) *F.sc = fs;
    const float a = fs.a, b = fs.b, sf = fs.sf, ce = fs.e;
    __syncthreads();
    // X X (B = X: its rows in k are the rows of X^T in m1)
    piece_mma<T>(p, m0, m1, dp, acc);
    float bb = b;
    if (order == 3) {
        // V = b X - e X X, stored transposed over X^T; then X V
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NB; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[q][e] = b * x[q][e] - ce * acc[q][e];
        piece_store<T, true>(p, m1, acc);
        __syncthreads();
        piece_mma<T>(p, m0, m1, dp, acc);
        bb = 1.0f;
    }
    __syncthreads();
    // P - I = -a X + b X X (or -a X + X V), stored transposed; A takes X's place
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[q][e] = bb * acc[q][e] - a * x[q][e];
    piece_store<T, true>(p, m1, acc);
    factor_store<T>(t, av2, m0, false);
    __syncthreads();
    // Z = s A + s A (P - I) (B = P - I: its rows in k are the rows of its transpose in m1;
    // the identity stays out of the product as in the levels, see add_explicit)
    piece_mma<T>(p, m0, m1, dp, acc);
    piece_each<T>(p, [&](int row, int col, int q, int e) { acc[q][e] = sf * m0[row * T::LD + col] + sf * acc[q][e]; });
    __syncthreads();
    piece_store<T, false>(p, m0, acc);
    __syncthreads();
    // A <- (Z + Z^T)/2 or Z, in the accumulators' layout: four consecutive rows of a
    // column of Z^T are one 16-byte read of m0, and of the symmetric result one
    // 16-byte store. fp32 addition commutes, so the result is bitwise symmetric.
    const int lane = t & 63;
#pragma unroll
    for (int i = 0; i < T::BI; ++i) {
        if (i >= p.nbi) continue;
#pragma unroll
        for (int j = 0; j < T::BJ; ++j) {
            const int row = p.row + 16 * i + 4 * (lane >> 4), col = p.col + 16 * j + (lane & 15);
            f32x4& z = acc[i * T::BJ + j];
            if (symmetrize) {
                const f32x4 zt = *reinterpret_cast<const f32x4*>(m0 + col * T::LD + row);
#pragma unroll
                for (int e = 0; e < 4; ++e) z[e] = 0.5f * (z[e] + zt[e]);
                if (live) st4_at(F.A, 4u * (unsigned)(col * dp + row), z);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) st_at(F.A, 4u * (unsigned)((row + e) * dp + col), z[e]);
            }
        }
    }
    if (symmetrize || side != 0) piece_store<T, true>(p, m1, acc);
    else piece_store<T, false>(p, m1, acc);
    __syncthreads();
}

// Scalars of a step that the layer kernels take by value.
struct StepScalars {
    double lr, wd;
    float beta1;
    int graft;
};

// (norm_m, norm_sgd) to the grafted step g (Algorithm 3) and the decoupled decay
// rate lr * wd (Section 4).
__device__ __forceinline__ LayerScalars layer_scalars(double nm, double ns, double lr, double wd, int graft) {
    double g = lr;
    if (graft) g = nm > 0.0 ? lr * ns / nm : 0.0;
    LayerScalars out;
    out.norm_m = nm;
    out.norm_sgd = ns;
    out.g = g;
    out.gf = (float)g;
    out.lw = (float)(lr * wd);
    return out;
}

// A NaN or infinity anywhere in this step's G reaches m_SGD = beta1 m_SGD + G, and
// with it this norm: the layer's flag records it for the host.
__device__ __forceinline__ void flag_nonfinite(const LayerDev& L, const LayerScalars& s) {
    if (!isfinite(s.norm_sgd)) *L.nonfinite = 1;
}

// m_SGD <- beta1 m_SGD + G by a workgroup holding the gradient as grad_load
// leaves it. Returns the thread's share of ||m_SGD||^2.
template <class T>
__device__ __forceinline__ double msgd_update(const LayerDev& L, const float (&g)[T::GV], float beta1) {
    const int t = threadIdx.x, c = t % T::D;
    float ms[T::GV];
#pragma unroll
    for (int i = 0; i < T::GV; ++i) {
        const int row = t / T::D + i * (T::THREADS / T::D);
        ms[i] = ld_at(L.msgd, 4u * (unsigned)(min(row, L.m - 1) * L.n + min(c, L.n - 1)));
    }
    double part = 0.0;
#pragma unroll
    for (int i = 0; i < T::GV; ++i) {
        const int row = t / T::D + i * (T::THREADS / T::D);
        if (row < L.m && c < L.n) {
            const float v = beta1 * ms[i] + g[i];
            st_at(L.msgd, 4u * (unsigned)(row * L.n + c), v);
            part += (double)v * (double)v;
        }
    }
    return part;
}

// The rest of a layer's step by a workgroup of eight waves, given L_hat (rows)
// in lm, G^T (np x mp rows) in gm, and tm free for T = L_hat G (tm may be lm).
// R_hat's transpose (rows) is in rm or, with R_LATE, R_hat (symmetric) is read
// from global memory into rm = gm once G^T has been used. ps: the thread's share
// of ||m_SGD||^2. red: 16 doubles.
//   m <- beta1 m + (1 - beta1) L_hat G R_hat; theta <- theta - (lr wd theta + g m)
// (see weight_kernel).
template <class T, bool R_LATE>
__device__ __forceinline__ void layer_apply(const LayerDev& L, const FactorDev& FR, float* __restrict__ theta,
                                            double ps, const StepScalars& sc, const float* lm, float* gm, float* tm,
                                            float* rm, double* red, float* coef) {
    constexpr int NB = T::BI * T::BJ;
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int m = L.m, n = L.n;
    const Piece p = piece_of<T>(wave, L.mp, L.np);
    // The state this thread updates, in the accumulators' layout.
    f32x4 mo[NB], th[NB];
    piece_each<T>(p, [&](int row, int col, int q, int e) {
        const unsigned at = 4u * (unsigned)(min(row, m - 1) * n + min(col, n - 1));  // outside: read, not used
        mo[q][e] = ld_at(L.mom, at);
        th[q][e] = ld_at(theta, at);
    });
    f32x4 acc[NB];
    piece_mma<T>(p, lm, gm, L.mp, acc);  // T = L_hat G
    f32x4 rv[T::AV];
    if constexpr (R_LATE) factor_load<T>(t, FR.A, FR.dp, rv);
    __syncthreads();
    piece_store<T, false>(p, tm, acc);
    if constexpr (R_LATE) factor_store<T>(t, rv, rm, false);
    __syncthreads();
    piece_mma<T>(p, tm, rm, L.np, acc);  // G~ = T R_hat
    double pm = 0.0;
    piece_each<T>(p, [&](int row, int col, int q, int e) {
        if (row < m && col < n) {
            const float v = sc.beta1 * mo[q][e] + (1.0f - sc.beta1) * acc[q][e];
            mo[q][e] = v;
            st_at(L.mom, 4u * (unsigned)(row * n + col), v);
            pm += (double)v * (double)v;
        }
    });
    pm = wave_sum(pm);
    ps = wave_sum(ps);
    if ((t & 63) == 0) {
        red[wave] = pm;
        red[T::WAVES + wave] = ps;
    }
    __syncthreads();
    if (t == 0) {
        const LayerScalars s = layer_scalars(sqrt(sum_waves<T::WAVES>(red)), sqrt(sum_waves<T::WAVES>(red + T::WAVES)),
                                             sc.lr, sc.wd, sc.graft);
        flag_nonfinite(L, s);
        *L.ls = s;
        coef[0] = s.gf;
        coef[1] = s.lw;
    }
    __syncthreads();
    const float gf = coef[0], lw = coef[1];
    piece_each<T>(p, [&](int row, int col, int q, int e) {
        if (row < m && col < n)
            st_at(theta, 4u * (unsigned)(row * n + col), th[q][e] - (lw * th[q][e] + gf * mo[q][e]));
    });
}

// Layers with m, n <= 64: the whole step in one workgroup, L_hat's update in its
// first four waves and R_hat's in the other four.
__global__ __launch_bounds__(kSmallThreads) void small_step64_kernel(const LayerDev* __restrict__ layers,
                                                                     const FactorDev* __restrict__ f, int layer_base,
                                                                     PtrPack ptrs, StepScalars sc, int update,
                                                                     double beta2, int mode, int symmetrize,
                                                                     int order) {
    __shared__ __attribute__((aligned(16))) float mat[4][Team64::MAT];
    __shared__ double red[16];
    __shared__ float coef[2];
    const int li = layer_base + blockIdx.x;
    const LayerDev L = layers[li];
    const float* G = ptrs.grad(blockIdx.x);
    const int tid = threadIdx.x, team = __builtin_amdgcn_readfirstlane(tid >> 8), t = tid & 255;
    const FactorDev F = f[2 * li + team];
    float ga[Apply64::GV];
    grad_load<Apply64>(tid, G, L.m, L.n, L.n, ga);
    const double ps = msgd_update<Apply64>(L, ga, sc.beta1);
    if (update) {
        float gt[Team64::GV];
        grad_load<Team64>(t, G, L.m, L.n, L.n, gt);
        chain_update<Team64>(F, team, t, __builtin_amdgcn_readfirstlane(t >> 6), gt, L, G, false, true, beta2, mode,
                             symmetrize, order, mat[2 * team], mat[2 * team + 1], red + 4 * team);
    } else {
        f32x4 av[Team64::AV];
        factor_load<Team64>(t, F.A, F.dp, av);
        factor_store<Team64>(t, av, mat[2 * team + 1], team != 0 && !symmetrize);
    }
    grad_store<Apply64>(tid, ga, mat[0], true);
    __syncthreads();
    layer_apply<Apply64, false>(L, F, ptrs.param(blockIdx.x), ps, sc, mat[1], mat[0], mat[2], mat[3], red, coef);
}

// Layers up to 128 (symmetric factors): the factors' updates, first those above
// 64 in a workgroup each (the list's first `large`), then the others two to a workgroup,
// one per team of four waves. LDS and registers let one workgroup run per CU whatever
// its factors' sizes; alone in one, a factor up to 64 would use two of its eight waves.
// 512 layers of 32-64 with one of 96 x 96 take 131 us per step, with one factor to each
// workgroup 171; 256 of them 91 against 111; 512 of 48 x 96 the same 150 ...
__global__ __launch_bounds__(kSmallThreads) void small_chain128_kernel(const FactorDev* __restrict__ f,
                                                                       const int* __restrict__ list, int count,
                                                                       int large,
                                                                       const LayerDev* __restrict__ layers,
                                                                       int layer_base, PtrBatch grads, double beta2,
                                                                       int mode, int order) {
    __shared__ __attribute__((aligned(16))) float mat[2][Team128::MAT];
    __shared__ double red[Team128::WAVES];
    static_assert(4 * Team64::MAT <= 2 * Team128::MAT && 2 * Team64::WAVES == Team128::WAVES, "two teams fit");
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < large) {
        const int fi = list[blockIdx.x];
        const FactorDev F = f[fi];
        const LayerDev& L = layers[fi >> 1];
        const float* G = grads.p[(fi >> 1) - layer_base];
        float g[Team128::GV];
        grad_load<Team128>(tid, G, L.m, L.n, L.n, g);
        chain_update<Team128, false>(F, fi & 1, tid, __builtin_amdgcn_readfirstlane(tid >> 6), g, L, G, false, true,
                                     beta2, mode, 1, order, mat[0], mat[1], red);
        return;
    }
    const int team = __builtin_amdgcn_readfirstlane(tid >> 8), t = tid & 255;
    const int first = large + 2 * ((int)blockIdx.x - large), mine = first + team;
    // The last workgroup's second team may be one too many: it follows the first and stores nothing.
    const bool live = mine < count;
    const int fi = list[live ? mine : first], other = list[live && first + 1 < count ? first + 1 - team : first];
    const FactorDev F = f[fi];
    const LayerDev& L = layers[fi >> 1];
    const float* G = grads.p[(fi >> 1) - layer_base];
    const bool deep = max(F.kp, f[other].kp) > Team64::D;  // for both teams alike: they share their barriers
    float g[Team64::GV];
    grad_load<Team64>(t, G, L.m, L.n, L.n, g);
    float* const m0 = mat[0] + 2 * team * Team64::MAT;
    chain_update<Team64, true>(F, fi & 1, t, __builtin_amdgcn_readfirstlane(t >> 6), g, L, G, deep, live, beta2, mode, 1,
                               order, m0, m0 + Team64::MAT, red + team * Team64::WAVES);
}

// ... and the rest of each layer's step in one.
__global__ __launch_bounds__(kSmallThreads) void small_apply128_kernel(const LayerDev* __restrict__ layers,
                                                                       const FactorDev* __restrict__ f, int layer_base,
                                                                       PtrPack ptrs, StepScalars sc) {
    __shared__ __attribute__((aligned(16))) float mat[2][Team128::MAT];
    __shared__ double red[16];
    __shared__ float coef[2];
    const int li = layer_base + blockIdx.x, t = threadIdx.x;
    const LayerDev L = layers[li];
    const FactorDev FL = f[2 * li], FR = f[2 * li + 1];
    float g[Team128::GV];
    grad_load<Team128>(t, ptrs.grad(blockIdx.x), L.m, L.n, L.n, g);
    f32x4 av[Team128::AV];
    factor_load<Team128>(t, FL.A, FL.dp, av);
    const double ps = msgd_update<Team128>(L, g, sc.beta1);
    factor_store<Team128>(t, av, mat[0], false);
    grad_store<Team128>(t, g, mat[1], true);
    __syncthreads();
    layer_apply<Team128, true>(L, FR, ptrs.param(blockIdx.x), ps, sc, mat[0], mat[1], mat[0], mat[1], red, coef);
}

// Per-layer norms of m and m_SGD from their partial sums, and the grafted
// step g (Algorithm 3) with the decoupled decay rate lr * wd (Section 4). One
// wave per layer.
__global__ void layer_finalize_kernel(const LayerDev* __restrict__ layers, double lr, double wd,
                                      int graft) {
    const LayerDev L = layers[blockIdx.x];
    const double nm = sqrt(wave_sum_array(L.part_m, L.n_part_m));
    const double ns = sqrt(wave_sum_array(L.part_sgd, L.n_part_sgd));
    if (threadIdx.x != 0) return;
    const LayerScalars s = layer_scalars(nm, ns, lr, wd, graft);
    flag_nonfinite(L, s);
    *L.ls = s;
}

// Partial sums of either norm that a workgroup of the weight update sums itself
// (two per lane); with more, one wave per layer sums them in a launch of its own.
// Without that launch: 64 x 576 74.7 -> 72.8 us per step, 512 layers of 32-256
// between updates 141 -> 139; nothing on ResNet-50 (968 against 969, 576 sums).
constexpr int kFusedNormParts = 128;

// theta <- theta (1 - lr wd) - g m over a flat chunk of one layer, evaluated as
// theta - (lr wd theta + g m): the small correction is formed first, so the
// stored parameter is rounded once (1 - lr wd in fp32 would itself be off by up
// to 2^-25, a systematic error of that size on every parameter).
// With SUM the workgroup also does layer_finalize_kernel's work for its layer,
// whose norms have at most kFusedNormParts partial sums each way (the same sums in
// the same order by one wave each), and the layer's first workgroup stores the
// scalars: one launch fewer.
template <bool SUM>
__global__ __launch_bounds__(kEwThreads) void weight_kernel(const LayerDev* __restrict__ layers,
                                                            const FlatChunk* __restrict__ chunks,
                                                            int layer_base, MutPtrBatch params, StepScalars sc) {
    const FlatChunk ck = chunks[blockIdx.x];
    const LayerDev& L = layers[ck.layer];
    float* __restrict__ th = params.p[ck.layer - layer_base];
    float g, lw;
    if constexpr (SUM) {
        __shared__ double norm[2];
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        if (wave < 2) {
            const double v = sqrt(wave ? wave_sum_array(L.part_sgd, L.n_part_sgd) : wave_sum_array(L.part_m, L.n_part_m));
            if ((threadIdx.x & 63) == 0) norm[wave] = v;
        }
        __syncthreads();
        const LayerScalars s = layer_scalars(norm[0], norm[1], sc.lr, sc.wd, sc.graft);
        if (ck.start == 0 && threadIdx.x == 0) {
            flag_nonfinite(L, s);
            *L.ls = s;
        }
        g = s.gf;
        lw = s.lw;
    } else {
        g = L.ls->gf;
        lw = L.ls->lw;
    }
    const float* __restrict__ m = L.mom;
    if ((ck.count & 3) == 0 && (reinterpret_cast<uintptr_t>(th) & 15) == 0) {
        const int n4 = ck.count >> 2;
        // Global (not generic) accesses, four per array per thread in flight:
        // each group of four iterations issues its loads before its stores,
        // then the remainder goes one by one.
        gfloat4* t4 = (gfloat4*)(th + ck.start);
        const global_f32x4* m4 = (const global_f32x4*)(m + ck.start);
        int e = threadIdx.x;
        for (; e + 3 * kEwThreads < n4; e += 4 * kEwThreads) {
            f32x4 t[4], mv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                t[i] = t4[e + i * kEwThreads];
                mv[i] = m4[e + i * kEwThreads];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
#pragma unroll
                for (int q = 0; q < 4; ++q) t[i][q] = t[i][q] - (lw * t[i][q] + g * mv[i][q]);
                t4[e + i * kEwThreads] = t[i];
            }
        }
        for (; e < n4; e += kEwThreads) {
            f32x4 t = t4[e];
            const f32x4 mv = m4[e];
#pragma unroll
            for (int q = 0; q < 4; ++q) t[q] = t[q] - (lw * t[q] + g * mv[q]);
            t4[e] = t;
        }
    } else {
        for (int e = threadIdx.x; e < ck.count; e += kEwThreads) {
            const int i = ck.start + e;
            th[i] = th[i] - (lw * th[i] + g * m[i]);
        }
    }
}

}  // namespace jorge
