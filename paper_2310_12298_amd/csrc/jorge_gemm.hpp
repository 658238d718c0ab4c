// Grouped fp32 GEMM for gfx950 with fused epilogues.
//
// One launch covers every tile of a list of independent products (all
// factors' products of one dependency level of the step). Each product
// carries its own epilogue (flags and coefficient set, decided at run time
// per problem), so products with different epilogues share a launch. A
// workgroup of 256 threads computes one 128 x 128 tile of C = A * B; its
// four waves each own a 64 x 64 sub-tile held as 4 x 4 blocks of 16 x 16
// accumulators. Operands and results are fp32.
//
// Products run on the bf16 matrix pipe without giving up fp32: each operand
// element is split into three bf16 terms that sum to it exactly (24 bits), and
// the six term products down to 2^-16 of the whole are accumulated in fp32 (see
// split_pair below). A is K-contiguous; B is K-contiguous (NT: every product of
// the symmetric mode) or MN-contiguous (NN: the literal mode's powers).
#pragma once

#include <hip/hip_runtime.h>

#include "jorge_types.hpp"

namespace jorge {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Accumulator layout. A wave's 64 x 64 quadrant (wy, wx) of its tile is a
// 4 x 4 grid of 16 x 16 blocks; block b = 4 i + j (rows 16 i, columns 16 j of
// the quadrant) is one v_mfma_f32_16x16x32_bf16 accumulator, in which lane l
// holds column l % 16, rows 4 (l / 16) .. 4 (l / 16) + 3. Each lane thus
// holds, for each of its 16 blocks, four consecutive rows of one column.
// Where a lane's accumulators lie in the result: the first of block b's four
// values is at row + 16 (b / 4), col + 16 (b % 4).
struct Place {
    int row, col;
    bool diag;  // on a diagonal tile or block of the result (row = col may occur in it)
};
// Of quadrant `wave` of the 128 x 128 tile (tm, tn).
__device__ __forceinline__ Place place_of(int tm, int tn, int lane, int wave) {
    return {tm * 128 + (wave >> 1) * 64 + (lane >> 4) * 4, tn * 128 + (wave & 1) * 64 + (lane & 15), tm == tn};
}

constexpr int kTile = 128;                    // tile rows = tile columns
constexpr int kSlab = 32;                     // K per LDS stage
constexpr int kGemmThreads = 256;
// A slab sits in LDS as three planes (one per term of the split), each of 16
// blocks of 16 rows: rows of A in blocks 0-7, columns of B in blocks 8-15. A
// block is 1 KB: 64 slots of 16 bytes, slot 16 c + (r ^ swizzle(c, block))
// holding k = 8 c .. 8 c + 7 of row r. A fragment read (lane l: row l % 16, c = l /
// 16) takes the whole block in one 16-byte read per lane; the swizzle spreads
// it, and the 8-byte writes of both operand layouts, over the banks.
constexpr int kBlockBytes = 1024;
constexpr int kPlaneBytes = 2 * (kTile / 16) * kBlockBytes;
constexpr int kSlabBytes = 3 * kPlaneBytes;

// Pointers into global memory (address space 1): loads through them compile
// to global_load rather than flat_load, which would also count against the
// LDS wait counter and make every LDS wait drain the in-flight prefetch.
typedef __attribute__((address_space(1))) const f32x4 global_f32x4;

__device__ __forceinline__ f32x4 gload4(const float* p) {
    return *(global_f32x4*)p;
}

// ---------------------------------------------------------------- three-term split
// x = x0 + x1 + x2: x0 is x rounded to its upper half, x1 the upper half of x - x0,
// x2 what is left. Both differences are exact in fp32 and 3 x 8 significant bits
// hold all 24 of x from 2^-110 to 3.39e38 (split_lost tells of the rest). The
// scheme is that of Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations" (arXiv 1904.06376).
// x0 is rounded, not cut off: x1 and x2 then have either sign, and the terms
// left out of a sum cancel where cut-off ones would all have the product's sign
// (a bias of 2^-24 per product, which ResNet-50's and the 4096-wide layers' powers
// added up to 2.1e-6 and 1.4e-6 of a factor).
// A product a b is summed as a2 b0 + a1 b1 + a0 b2 + a1 b0 + a0 b1 + a0 b0, every term exact and accumulated in fp32; the three left out are below
// 2^-23 |a b| together, and a K-long sum takes 6 K / 32 roundings of the
// accumulator where the fp32 MFMA takes K / 4. Measured against fp64 on Gaussian
// operands (relative 2-norm): 3.4e-7 at K = 512 and 1.04e-6 at K = 4096, where the
// fp32 MFMA has 4.0e-7 and 1.1e-6; over the steps of 38 shapes 0.66 of its error in the
// geometric mean (0.82 by the products alone). A sum with one live term has only its own roundings and is behind:
// 5.7e-8 against 4.4e-8 for L G R with diagonal L and R (from the largest term product to
// the smallest 8.1e-8, with the second-order terms before the leading one 7.1e-8).
// The bf16 MFMA does 16 times the fp32 one's flops per cycle, so six of them are
// 2.7 times as fast at the same clock; but the clock gives way under their power:
// 4096^3 of random operands runs at 212-215 TFLOP/s and 1.84 GHz (of zeros at 291
// and 2.40 GHz) against 135 with the fp32 MFMA, K = 512 at 190 against 128.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
constexpr int kTerms = 3;
struct SplitPair {
    bf16x2 t[kTerms];
};
// Elements the three terms do not hold: magnitudes below 2^-110 (x2 runs out of bf16's
// exponents and drops bits), infinities and magnitudes that round to 2^128. A product
// with one among its operands is formed by the fp32 MFMA instead (fp32_blocks): the
// split collects the bits it drops (lost, in its lower half), and the other two kinds
// leave no finite sum, as does a term product that overflows where the fp32 one does not.
__device__ __forceinline__ bool split_lost(unsigned lost) { return (lost & 0xffffu) != 0; }

template <int N>
__device__ __forceinline__ bool any_non_finite(const f32x4 (&acc)[N]) {
    float z = 0.0f;
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) z += 0.0f * acc[b][e];
    return !(z == 0.0f);
}

// Fourteen instructions of the plain VALU for two elements, one of them for lost. Rounding conversions
// and dot products (v_cvt_pk_bf16_f32, v_dot2c_f32_bf16) make it in seven, but
// those run at half rate and hold up the MFMAs, while these take two waves'
// instructions at once and run beside the MFMAs: cycles for 24 pairs and 48 MFMAs
// of each of two waves per SIMD, 2528 this way (without the rounding) and 4012 that
// way (MFMAs alone 1564).
__device__ __forceinline__ SplitPair split_pair(float a, float b, unsigned& lost) {
    SplitPair o;
    unsigned ua, ub;
#pragma unroll
    for (int t = 0; t < kTerms; ++t) {
        ua = __builtin_bit_cast(unsigned, a) + (t == 0 ? 0x8000u : 0u);
        ub = __builtin_bit_cast(unsigned, b) + (t == 0 ? 0x8000u : 0u);
        o.t[t] = __builtin_bit_cast(bf16x2, __builtin_amdgcn_perm(ub, ua, 0x07060302));
        a -= __builtin_bit_cast(float, ua & 0xffff0000u);
        b -= __builtin_bit_cast(float, ub & 0xffff0000u);
    }
    lost |= ua | ub;
    asm("" : "+v"(lost));  // in this order: gathered at the end of a slab, 32 residuals would stay in registers (32 spilled)
    return o;
}

struct SplitOct {
    bf16x8 t[kTerms];
};
__device__ __forceinline__ SplitOct split_oct(f32x4 u, f32x4 v, unsigned& lost) {
    const SplitPair a = split_pair(u[0], u[1], lost), b = split_pair(u[2], u[3], lost);
    const SplitPair c = split_pair(v[0], v[1], lost), d = split_pair(v[2], v[3], lost);
    asm volatile("" : "+v"(lost));  // (106 registers in gemm_wave_split, 130 without: one workgroup per CU fewer)
    SplitOct o;
#pragma unroll
    for (int t = 0; t < kTerms; ++t)
        o.t[t] = bf16x8{a.t[t][0], a.t[t][1], b.t[t][0], b.t[t][1], c.t[t][0], c.t[t][1], d.t[t][0], d.t[t][1]};
    return o;
}

// Which of a wave's 16 blocks it multiplies: every block; on a diagonal
// tile of a symmetric result, only blocks on or above the diagonal (i <= j)
// of a diagonal quadrant; or none, for the quadrant below the diagonal. The
// epilogue of a symmetric result never reads the blocks left out.
enum BlockSet : int { BS_ALL = 0, BS_UPPER = 1, BS_NONE = 2 };

// Sum of one double per lane over a 64-lane wave, in a fixed order.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// Sum of one double per thread over the workgroup, in a fixed order.
__device__ __forceinline__ double block_sum_256(double v, double* red) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

typedef __attribute__((address_space(1))) const char gcchar;

// One thread's share of a slab in registers, 16 floats of each operand. A (and
// a K-contiguous B): rows tid / 8 + 32 v, k = 4 (tid % 8) .. + 3 in v[v], so
// eight lanes read one 128-byte row. An MN-contiguous B: columns 4 (tid % 32) ..
// + 3 at k = 4 (tid / 32) + v.
struct SlabRegs {
    f32x4 a[4], b[4];
};

// Byte offsets of those loads from the operand's base at the slab's first k.
// Rows (columns) past the extent are clamped to the last valid one: they only
// feed outputs that the epilogue discards. The same for every slab of a tile and
// for both K segments (lda2 = lda, ldb2 = ldb).
struct SlabOffsets {
    unsigned a[4], b[4];
};

template <bool BK>
__device__ __forceinline__ void slab_offsets(const GemmProblem& p, int row0, int col0, SlabOffsets& o) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = (tid >> 3) + 32 * v;
        o.a[v] = (unsigned)min(row0 + r, p.M - 1) * (unsigned)p.lda * 4u + (tid & 7) * 16u;
        if constexpr (BK)
            o.b[v] = (unsigned)min(col0 + r, p.N - 1) * (unsigned)p.ldb * 4u + (tid & 7) * 16u;
        else
            o.b[v] = (unsigned)(4 * (tid >> 5) + v) * (unsigned)p.ldb * 4u + (unsigned)min(col0 + 4 * (tid & 31), p.N - 4) * 4u;
    }
}

// Starts the loads of the slab at absolute k.
template <bool BK>
__device__ __forceinline__ void load_slab(const GemmProblem& p, const SlabOffsets& o, int k, SlabRegs& r) {
    // Segment selection by selects, not branches, so the loads stay in the
    // scheduling region of the MFMAs.
    const bool two = k >= p.K1;
    const int kl = two ? k - p.K1 : k;
    const gcchar* a = (const gcchar*)((two ? p.A2 : p.A) + kl);
    const gcchar* b = (const gcchar*)((two ? p.B2 : p.B) + (BK ? (size_t)kl : (size_t)kl * p.ldb));
#pragma unroll
    for (int v = 0; v < 4; ++v) r.a[v] = *(global_f32x4*)(a + o.a[v]);
#pragma unroll
    for (int v = 0; v < 4; ++v) r.b[v] = *(global_f32x4*)(b + o.b[v]);
}

// The same share split into its terms: v-th row of A and of B, four k each.
struct SlabTerms {
    bf16x4 a[4][kTerms], b[4][kTerms];
};

template <bool BK>
__device__ __forceinline__ void split_slab(const SlabRegs& r, SlabTerms& s, unsigned& lost) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const SplitPair x = split_pair(r.a[v][0], r.a[v][1], lost), y = split_pair(r.a[v][2], r.a[v][3], lost);
        const SplitPair z = BK ? split_pair(r.b[v][0], r.b[v][1], lost) : split_pair(r.b[0][v], r.b[1][v], lost);
        const SplitPair w = BK ? split_pair(r.b[v][2], r.b[v][3], lost) : split_pair(r.b[2][v], r.b[3][v], lost);
#pragma unroll
        for (int t = 0; t < kTerms; ++t) {
            s.a[v][t] = bf16x4{x.t[t][0], x.t[t][1], y.t[t][0], y.t[t][1]};
            s.b[v][t] = bf16x4{z.t[t][0], z.t[t][1], w.t[t][0], w.t[t][1]};
        }
    }
}

// Slot of row r (0-15), chunk c of a block: see the LDS layout above.
__device__ __forceinline__ int slab_slot(int r, int c, int block) {
    return 16 * c + (r ^ ((0xEA40 >> (4 * c)) & 15) ^ (block & 3));
}

// LDS byte offsets (within a plane) of a thread's writes, v = 0, and of a lane's fragments.
struct SlabLds {
    int wa, wb, frag;
};

template <bool BK>
__device__ __forceinline__ SlabLds slab_lds() {
    const int tid = threadIdx.x, lane = tid & 63;
    SlabLds o;
    const int r = tid >> 3, c = (tid & 7) >> 1;
    o.wa = (r >> 4) * kBlockBytes + slab_slot(r & 15, c, r >> 4) * 16 + (tid & 1) * 8;
    if constexpr (BK) {
        o.wb = o.wa + (kTile / 16) * kBlockBytes;
    } else {
        const int n = 4 * (tid & 31), kg = tid >> 5;
        o.wb = (kTile / 16 + (n >> 4)) * kBlockBytes + slab_slot(n & 15, kg >> 1, n >> 4) * 16 + (kg & 1) * 8;
    }
    o.frag = slab_slot(lane & 15, lane >> 4, 0) * 16;
    return o;
}

template <bool BK>
__device__ __forceinline__ void store_slab(char* lds, const SlabLds& o, const SlabTerms& s) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        // 32 rows on are two blocks on, whose swizzle differs in bit 1; the next row of a block, in the row.
        const int step = (v & 1) * 32, wa = (o.wa ^ step) + v * 2 * kBlockBytes;
        const int wb = BK ? (o.wb ^ step) + v * 2 * kBlockBytes : o.wb ^ (v * 16);
#pragma unroll
        for (int t = 0; t < kTerms; ++t) {
            *reinterpret_cast<bf16x4*>(lds + t * kPlaneBytes + wa) = s.a[v][t];
            *reinterpret_cast<bf16x4*>(lds + t * kPlaneBytes + wb) = s.b[v][t];
        }
    }
}

// The MFMAs of one slab for the calling wave's block set. The term products go
// from the smallest to the largest; four independent blocks between two that
// share an accumulator.
template <int BS>
__device__ __forceinline__ void mma_slab(const char* lds, const SlabLds& o, int wy, int wx, f32x4 (&acc)[16]) {
    if constexpr (BS == BS_NONE) return;
    constexpr int kA[6] = {2, 1, 0, 1, 0, 0}, kB[6] = {0, 1, 2, 0, 1, 0};
    bf16x8 b[4][kTerms];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int t = 0; t < kTerms; ++t)
            b[j][t] = *reinterpret_cast<const bf16x8*>(lds + t * kPlaneBytes + (kTile / 16 + wx * 4 + j) * kBlockBytes +
                                                       (o.frag ^ (j * 16)));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        bf16x8 a[kTerms];
#pragma unroll
        for (int t = 0; t < kTerms; ++t)
            a[t] = *reinterpret_cast<const bf16x8*>(lds + t * kPlaneBytes + (wy * 4 + i) * kBlockBytes + (o.frag ^ (i * 16)));
#pragma unroll
        for (int u = 0; u < 6; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (BS == BS_ALL || i <= j)
                    acc[i * 4 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kA[u]], b[j][kB[u]], acc[i * 4 + j], 0, 0, 0);
    }
}

// Spreads the split's VALU instructions evenly among a slab's MFMAs, the LDS
// reads of a block row ahead of its MFMAs and the next loads last. Left to itself
// the compiler puts the whole split before the first MFMA (and spills): ResNet-50's
// step 7.2 ms, against 5.2 with the seven-instruction split, which it interleaved,
// and 4.9 with this order.
template <int N, int VALU>
__device__ __forceinline__ void interleave_row() {
#pragma unroll
    for (int q = 0; q < N; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);     // MFMA
        __builtin_amdgcn_sched_group_barrier(0x2, VALU, 0);  // VALU
        if (q == N / 3) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);  // LDS reads of the next row
    }
}
template <int BS, bool LOADS>
__device__ __forceinline__ void interleave_slab() {
    if constexpr (BS == BS_NONE) return;
    __builtin_amdgcn_sched_group_barrier(0x100, 15, 0);  // LDS reads
    // 224 of the split and the addresses' few over 96 (60) MFMAs.
    constexpr int V = BS == BS_ALL ? 2 : 4;
    interleave_row<24, V>();
    interleave_row<BS == BS_ALL ? 24 : 18, V>();
    interleave_row<BS == BS_ALL ? 24 : 12, BS == BS_ALL ? 3 : 4>();
    interleave_row<BS == BS_ALL ? 24 : 6, BS == BS_ALL ? 3 : 4>();
    if constexpr (LOADS) __builtin_amdgcn_sched_group_barrier(0x20, 8, 0);  // global loads
}

// Workgroup barrier that waits for this wave's LDS accesses but leaves its
// global loads in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The slab loop of gemm_mainloop for the calling wave's block set BS (one
// copy per set, so the loop itself has no branches on it). Slab 0 is in LDS and
// slab 1's loads are in flight.
template <bool BK, int BS>
__device__ __forceinline__ void slab_loop(const GemmProblem& p, const SlabOffsets& o, const SlabLds& l, int k0, int nk,
                                          char* lds, SlabRegs& r, int wy, int wx, f32x4 (&acc)[16], unsigned& lost) {
    // One LDS buffer: the next slab is split under this slab's MFMAs (its raw
    // values, loaded a slab earlier, make room for the loads of the slab after
    // it) and written between two barriers; the other workgroup of the CU
    // fills that gap. Raised issue priority while the wave runs its MFMAs.
    SlabTerms s;
    int kt = 0;
    __builtin_amdgcn_s_setprio(1);
    for (; kt + 2 < nk; ++kt) {
        split_slab<BK>(r, s, lost);
        load_slab<BK>(p, o, k0 + (kt + 2) * kSlab, r);
        mma_slab<BS>(lds, l, wy, wx, acc);
        interleave_slab<BS, true>();
        __builtin_amdgcn_s_setprio(0);
        lds_barrier();
        store_slab<BK>(lds, l, s);
        lds_barrier();
        __builtin_amdgcn_s_setprio(1);
    }
    if (kt + 1 < nk) {
        split_slab<BK>(r, s, lost);
        mma_slab<BS>(lds, l, wy, wx, acc);
        interleave_slab<BS, false>();
        __builtin_amdgcn_s_setprio(0);
        lds_barrier();
        store_slab<BK>(lds, l, s);
        lds_barrier();
        __builtin_amdgcn_s_setprio(1);
    }
    mma_slab<BS>(lds, l, wy, wx, acc);
    __builtin_amdgcn_s_setprio(0);
}

// The product of BI x BJ blocks of 16 x 16 at (row0, col0) over [kb, ke), by the
// calling wave alone and with the fp32 MFMA, straight from global memory: for operands
// that the split does not hold, so it is short rather than fast. Lane l loads k = 4 (l /
// 16) .. + 3 of each 16; rows and columns past the extent are clamped as in a slab.
// A sum that is NaN stays NaN, so the wave stops once all of its sums are: a step of
// four 2048 x 2048 layers on a state that is NaN throughout takes 3.6 ms, 9.3 with
// every sum taken to its end.
template <bool BK, int BI, int BJ, int LDB, int NB>
__device__ __forceinline__ void fp32_blocks(const GemmProblem& p, int row0, int col0, int kb, int ke, int lane,
                                            f32x4 (&acc)[NB]) {
    const int r = lane & 15, c = 4 * (lane >> 4);
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
    for (int k = kb; k < ke; k += 16) {
        const bool two = k >= p.K1;
        const int kl = (two ? k - p.K1 : k) + c;
        const float* A = (two ? p.A2 : p.A) + kl;
        const float* B = two ? p.B2 : p.B;
        f32x4 a[BI], b[BJ];
#pragma unroll
        for (int i = 0; i < BI; ++i) a[i] = gload4(A + (size_t)min(row0 + 16 * i + r, p.M - 1) * p.lda);
#pragma unroll
        for (int j = 0; j < BJ; ++j) {
            const int col = min(col0 + 16 * j + r, p.N - 1);
            if constexpr (BK) {
                b[j] = gload4(B + (size_t)col * p.ldb + kl);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) b[j][e] = B[(size_t)(kl + e) * p.ldb + col];
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < BI; ++i)
#pragma unroll
                for (int j = 0; j < BJ; ++j)
                    acc[i * LDB + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], b[j][e], acc[i * LDB + j], 0, 0, 0);
        if ((k - kb) % 256 == 0) {
            bool live = false;
#pragma unroll
            for (int i = 0; i < BI; ++i)
#pragma unroll
                for (int j = 0; j < BJ; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) live |= acc[i * LDB + j][e] == acc[i * LDB + j][e];
            if (!__any(live)) return;
        }
    }
}

// The product of one 128 x 128 tile (tm, tn) of problem p over K range
// [k0, k1), accumulated by the whole workgroup into acc. Every thread of the
// workgroup must call it. inexact: an int of LDS, for the workgroup's verdict on
// the split.
template <bool BK>
__device__ __forceinline__ void gemm_mainloop(const GemmProblem& p, int tm, int tn, int k0, int k1, char* lds,
                                              int* inexact, f32x4 (&acc)[16]) {
    const int row0 = tm * kTile, col0 = tn * kTile;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wy = wave >> 1, wx = wave & 1;
    const int nk = (k1 - k0) / kSlab;
    SlabOffsets o;
    slab_offsets<BK>(p, row0, col0, o);
    SlabRegs r;
    load_slab<BK>(p, o, k0, r);
#pragma unroll
    for (int b = 0; b < 16; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[b][e] = 0.0f;
    const SlabLds l = slab_lds<BK>();
    unsigned lost = 0;
    if (threadIdx.x == 0) *inexact = 0;
    {
        SlabTerms s;
        split_slab<BK>(r, s, lost);
        if (nk > 1) load_slab<BK>(p, o, k0 + kSlab, r);
        store_slab<BK>(lds, l, s);
    }
    lds_barrier();
    // A quadrant that lies wholly past the product's padded extent (a product
    // 32 or 64 rows or columns wide, or an edge tile) multiplies nothing: its
    // outputs are discarded. On a diagonal tile of a symmetric result the
    // quadrant below the diagonal is not needed and the diagonal quadrants
    // only on and above it.
    const bool outside = row0 + wy * 64 >= p.M || col0 + wx * 64 >= p.N;
    if (outside) {
        slab_loop<BK, BS_NONE>(p, o, l, k0, nk, lds, r, wy, wx, acc, lost);
    } else if (p.upper && tm == tn) {
        if (wy > wx) slab_loop<BK, BS_NONE>(p, o, l, k0, nk, lds, r, wy, wx, acc, lost);
        else if (wy == wx) slab_loop<BK, BS_UPPER>(p, o, l, k0, nk, lds, r, wy, wx, acc, lost);
        else slab_loop<BK, BS_ALL>(p, o, l, k0, nk, lds, r, wy, wx, acc, lost);
    } else {
        slab_loop<BK, BS_ALL>(p, o, l, k0, nk, lds, r, wy, wx, acc, lost);
    }
    // Each thread split its share of the whole tile's operands, so one verdict for all waves.
    if (split_lost(lost) || any_non_finite(acc)) *inexact = 1;
    lds_barrier();
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(*inexact), 0) && !outside)
        fp32_blocks<BK, 4, 4, 4>(p, row0 + wy * 64, col0 + wx * 64, k0, k1, threadIdx.x & 63, acc);
}

// Partial products of split tiles: thread t (= 64 wave + lane) keeps its 64
// accumulators as 16 float4 (one per block), float4 b of a partial at
// b * 1024 + 4 t (coalesced across threads).
__device__ __forceinline__ void store_partial(float* __restrict__ blk, const f32x4 (&acc)[16]) {
#pragma unroll
    for (int b = 0; b < 16; ++b) *reinterpret_cast<f32x4*>(blk + b * 1024 + 4 * threadIdx.x) = acc[b];
}

typedef __attribute__((address_space(1))) float gfloat;
typedef __attribute__((address_space(1))) f32x4 gfloat4;
typedef __attribute__((address_space(1))) char gchar;

// Global accesses at a 32-bit byte offset from a uniform base: they compile to
// the base-in-SGPR, offset-in-VGPR form with no 64-bit address arithmetic.
// Every matrix here spans at most 32768^2 floats, so byte offsets fit in 32 bits.
__device__ __forceinline__ float ld_at(const float* base, unsigned byte_off) {
    return *(const gfloat*)((const gchar*)base + byte_off);
}
__device__ __forceinline__ void st_at(float* base, unsigned byte_off, float v) {
    *(gfloat*)((gchar*)base + byte_off) = v;
}
__device__ __forceinline__ void st4_at(float* base, unsigned byte_off, f32x4 v) {
    *(gfloat4*)((gchar*)base + byte_off) = v;
}

// The epilogue body for one combination of flags F and symmetry UP, known
// at compile time. value = cx X + cc acc.
// Offsets are 32-bit (every matrix has fewer than 2^32 elements) from
// uniform base pointers; per-element masks are only evaluated on edge tiles
// and on diagonal tiles of symmetric results.
template <int F, bool UP, bool MASKED, int NB>
__device__ __forceinline__ double epilogue_body(const GemmProblem& p, const Place& at, const f32x4 (&acc)[NB],
                                                float cx, float cc) {
    constexpr bool kReadX = (F & EF_READX) != 0;
    constexpr bool kRead = (F & (EF_READX | EF_DOT)) != 0;
    const bool diag = MASKED && UP && at.diag;
    constexpr double w_off = UP ? 2.0 : 1.0;   // off-diagonal tiles of a symmetric result
    float* C = p.C;
    float* C2 = p.C2;
    const float* X = p.X;
    // Row strides in bytes.
    const unsigned sc = 4u * p.ldc, sc2 = 4u * p.ldc2, sx = 4u * p.ldx;

    // Every X value the thread will use is loaded before anything is stored,
    // so one memory round trip serves the whole tile (X may be C itself, and
    // the compiler keeps loads after earlier stores it cannot tell apart).
    // Masked tiles clamp positions outside M x N to the last row and column
    // and drop those values; every position the thread uses is also one it
    // writes, and no other thread writes it.
    f32x4 xv[NB];
    if constexpr (kRead) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int col = at.col + (b & 3) * 16;
            const int colc = MASKED ? min(col, p.N - 1) : col;
            // rowb .. rowb+3 are all inside M when rowb is (M is a multiple of 4).
            const int rowb = at.row + (b >> 2) * 16;
            const int rowc = MASKED ? min(rowb, p.M - 4) : rowb;
            const unsigned ox = (unsigned)rowc * sx + 4u * (unsigned)colc;
#pragma unroll
            for (int e = 0; e < 4; ++e) xv[b][e] = ld_at(X, ox + e * sx);
        }
    }

    double part = 0.0;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int col = at.col + (b & 3) * 16;
        const int rowb = at.row + (b >> 2) * 16;
        // rowb .. rowb+3 are all inside M when rowb is (M is a multiple of 4).
        if (MASKED && (rowb >= p.M || col >= p.N)) continue;
        // X at positions this thread writes (read and written by the same thread).
        f32x4 x;
        f32x4 out;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float v = acc[b][e];
            float o = cc * v;
            if constexpr (kRead) x[e] = xv[b][e];
            if constexpr (kReadX) o = cx * x[e] + o;
            out[e] = o;
        }
        if (!diag) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr ((F & EF_NORM) != 0) part += w_off * (double)out[e] * (double)out[e];
                if constexpr ((F & EF_DOT) != 0) part += w_off * (double)acc[b][e] * (double)x[e];
            }
            if constexpr ((F & EF_STORE) != 0) {
                const unsigned oc = (unsigned)rowb * sc + 4u * (unsigned)col;
#pragma unroll
                for (int e = 0; e < 4; ++e) st_at(C, oc + e * sc, out[e]);
                if constexpr (UP) st4_at(C, (unsigned)col * sc + 4u * (unsigned)rowb, out);
            }
            if constexpr ((F & EF_STORE_T) != 0) st4_at(C2, (unsigned)col * sc2 + 4u * (unsigned)rowb, out);
        } else {
            // Diagonal tile of a symmetric result: element (row, col) with
            // row <= col is written at both positions.
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = rowb + e;
                if (row > col) continue;
                const double w = row != col ? 2.0 : 1.0;
                if constexpr ((F & EF_NORM) != 0) part += w * (double)out[e] * (double)out[e];
                if constexpr ((F & EF_DOT) != 0) part += w * (double)acc[b][e] * (double)x[e];
                if constexpr ((F & EF_STORE) != 0) {
                    st_at(C, (unsigned)row * sc + 4u * (unsigned)col, out[e]);
                    if (row != col) st_at(C, (unsigned)col * sc + 4u * (unsigned)row, out[e]);
                }
            }
        }
    }
    return part;
}

// The epilogue for a flag combination without a compiled body (not used by
// the launch tables the library builds; kept so every combination works).
template <int NB>
__device__ __forceinline__ double epilogue_generic(const GemmProblem& p, const Place& at, const f32x4 (&acc)[NB],
                                                   float cx, float cc) {
    double part = 0.0;
    const int F = p.flags;
    const bool up = p.upper != 0;
    float* C = p.C;
    float* C2 = p.C2;
    const float* X = p.X;
    const unsigned sc = 4u * p.ldc, sc2 = 4u * p.ldc2, sx = 4u * p.ldx;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int col = at.col + (b & 3) * 16;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = at.row + (b >> 2) * 16 + e;
            if (row >= p.M || col >= p.N || (up && row > col)) continue;
            const float v = acc[b][e];
            const float xe = (F & (EF_READX | EF_DOT)) ? ld_at(X, (unsigned)row * sx + 4u * (unsigned)col) : 0.f;
            float o = cc * v;
            if (F & EF_READX) o = cx * xe + o;
            const double w = (up && row != col) ? 2.0 : 1.0;
            if (F & EF_NORM) part += w * (double)o * (double)o;
            if (F & EF_DOT) part += w * (double)v * (double)xe;
            if (F & EF_STORE) {
                st_at(C, (unsigned)row * sc + 4u * (unsigned)col, o);
                if (up && row != col) st_at(C, (unsigned)col * sc + 4u * (unsigned)row, o);
            }
            if (F & EF_STORE_T) st_at(C2, (unsigned)col * sc2 + 4u * (unsigned)row, o);
        }
    }
    return part;
}

// m = beta1 m + (1 - beta1) acc on the dense valid_m x valid_n momentum.
template <bool MASKED, int NB>
__device__ __forceinline__ double epilogue_momentum(const GemmProblem& p, const Place& at, const f32x4 (&acc)[NB],
                                                    float beta1) {
    float* mom = p.mom;
    const unsigned sm = 4u * p.ldmom;
    // All of this thread's momentum values are loaded before any is stored
    // (one memory round trip per tile); masked tiles clamp positions outside
    // the dense valid_m x valid_n momentum to its last row and column and
    // drop those values.
    f32x4 mv[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int col = at.col + (b & 3) * 16;
        const int colc = MASKED ? min(col, p.valid_n - 1) : col;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = at.row + (b >> 2) * 16 + e;
            const int rowc = MASKED ? min(row, p.valid_m - 1) : row;
            mv[b][e] = ld_at(mom, (unsigned)rowc * sm + 4u * (unsigned)colc);
        }
    }
    double part = 0.0;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int col = at.col + (b & 3) * 16;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = at.row + (b >> 2) * 16 + e;
            if (MASKED && !(row < p.valid_m && col < p.valid_n)) continue;
            const unsigned o = (unsigned)row * sm + 4u * (unsigned)col;
            const float mn = beta1 * mv[b][e] + (1.0f - beta1) * acc[b][e];
            st_at(mom, o, mn);
            part += (double)mn * (double)mn;
        }
    }
    return part;
}

// The epilogue of problem p for the product in acc at `at` (this lane's NB
// blocks); beta1 is the momentum of EF_MOMENTUM, [row_end, col_end) bounds the tile.
// One uniform switch picks the compiled body for the problem's flags. Returns
// the lane's share of the partial sum (norm, dot product).
//
// Symmetric results (p.upper): only tiles with tm <= tn are computed. An
// element (row, col) with row <= col is written at (row, col) and at
// (col, row), elements below the diagonal of a diagonal tile are skipped,
// so the stored matrix is bitwise symmetric whatever the product's rounding.
// The epilogue reads X only at the positions it is about to write, by the
// same thread, so X may alias C (an in-place update).
template <int NB>
__device__ __forceinline__ double gemm_epilogue_part(const GemmProblem& p, const Place& at, int row_end, int col_end,
                                                     float beta1, const f32x4 (&acc)[NB]) {
    const int flags = p.flags;
    double part = 0.0;
    if (flags & EF_MOMENTUM) {
        // Interior tiles of the dense valid_m x valid_n momentum need no masks.
        if (row_end <= p.valid_m && col_end <= p.valid_n)
            part = epilogue_momentum<false>(p, at, acc, beta1);
        else
            part = epilogue_momentum<true>(p, at, acc, beta1);
    } else {
        float cx = 0.f, cc = 1.f;
        if (p.coef != CO_ONE) {
            const FactorScalars* sc = p.sc;
            switch (p.coef) {
                case CO_POLY: cx = -sc->a; cc = sc->b; break;
                case CO_SCALE: cx = sc->sf; cc = sc->sf; break;
                case CO_WMIX: cx = sc->a; cc = -sc->b; break;
                case CO_SYR2K: cx = sc->sf; cc = -0.5f * sc->sf; break;
                case CO_LITUPD: cx = sc->sf; cc = -sc->sf; break;
                case CO_VSER: cx = sc->b; cc = -sc->e; break;
                case CO_POLY3: cx = -sc->a; break;
                case CO_WMIX3: cx = sc->a; cc = -1.f; break;
                default: break;
            }
        }
        const int key = flags | (p.upper ? 256 : 0);
        const bool masked = row_end > p.M || col_end > p.N || (p.upper && at.diag);
        switch (key) {
            case EF_STORE: part = masked ? epilogue_body<EF_STORE, false, true>(p, at, acc, cx, cc)
                            : epilogue_body<EF_STORE, false, false>(p, at, acc, cx, cc); break;
            case EF_STORE | 256: part = masked ? epilogue_body<EF_STORE, true, true>(p, at, acc, cx, cc)
                            : epilogue_body<EF_STORE, true, false>(p, at, acc, cx, cc); break;
            case EF_STORE_T: part = masked ? epilogue_body<EF_STORE_T, false, true>(p, at, acc, cx, cc)
                            : epilogue_body<EF_STORE_T, false, false>(p, at, acc, cx, cc); break;
            case EF_DOT | 256: part = masked ? epilogue_body<EF_DOT, true, true>(p, at, acc, cx, cc)
                            : epilogue_body<EF_DOT, true, false>(p, at, acc, cx, cc); break;
            case EF_STORE | EF_STORE_T | EF_NORM:
                part = masked ? epilogue_body<EF_STORE | EF_STORE_T | EF_NORM, false, true>(p, at, acc, cx, cc)
                            : epilogue_body<EF_STORE | EF_STORE_T | EF_NORM, false, false>(p, at, acc, cx, cc);
                break;
            case EF_STORE_T | EF_READX:
                part = masked ? epilogue_body<EF_STORE_T | EF_READX, false, true>(p, at, acc, cx, cc)
                            : epilogue_body<EF_STORE_T | EF_READX, false, false>(p, at, acc, cx, cc);
                break;
            case EF_STORE | EF_READX:
                part = masked ? epilogue_body<EF_STORE | EF_READX, false, true>(p, at, acc, cx, cc)
                            : epilogue_body<EF_STORE | EF_READX, false, false>(p, at, acc, cx, cc);
                break;
            case EF_STORE | EF_STORE_T:
                part = masked ? epilogue_body<EF_STORE | EF_STORE_T, false, true>(p, at, acc, cx, cc)
                              : epilogue_body<EF_STORE | EF_STORE_T, false, false>(p, at, acc, cx, cc);
                break;
            case EF_STORE | EF_STORE_T | EF_READX:
                part = masked ? epilogue_body<EF_STORE | EF_STORE_T | EF_READX, false, true>(p, at, acc, cx, cc)
                              : epilogue_body<EF_STORE | EF_STORE_T | EF_READX, false, false>(p, at, acc, cx, cc);
                break;
            case EF_STORE | EF_READX | 256:
                part = masked ? epilogue_body<EF_STORE | EF_READX, true, true>(p, at, acc, cx, cc)
                            : epilogue_body<EF_STORE | EF_READX, true, false>(p, at, acc, cx, cc);
                break;
            default:  // any other combination: every flag tested at run time
                part = epilogue_generic(p, at, acc, cx, cc);
                break;
        }
    }
    return part;
}

// The same for quadrant `wave` of tile (tm, tn), whose partial sum goes to
// sub-slot `wave` of the tile's slot.
__device__ __forceinline__ void gemm_epilogue(const GemmProblem& p, int tm, int tn, int slot, float beta1,
                                              const f32x4 (&acc)[16], int lane, int wave) {
    const double part = gemm_epilogue_part(p, place_of(tm, tn, lane, wave), (tm + 1) * kTile, (tn + 1) * kTile, beta1, acc);
    if (p.flags & (EF_NORM | EF_DOT | EF_MOMENTUM)) {
        const double total = wave_sum(part);
        if (lane == 0) p.partials[(size_t)slot * kWaveSlots + wave] = total;
    }
}

// The product of the BI x BJ blocks of 16 x 16 at (row0, col0) of problem p over
// [kb, ke), by the calling wave alone, with no LDS and no barrier: lane l loads k =
// 8 (l / 16) .. + 7 of rows l % 16 of each block row, 32 bytes that are its MFMA
// operand once split. The next slab's loads run under the current one's MFMAs.
// UPPER: on the diagonal of a symmetric result, whose blocks below the diagonal
// are left out. One copy per block shape, so the loop has no branches on it.
// Short products are bound by the latency of the first loads and the epilogue;
// this saves the LDS round trip and the fp32 MFMA's time: 512 layers of 32-256
// 521 -> 505 us per step, between updates 150 -> 139. (Also for products up to 128
// wide, whose tiles' four waves would share their operands through LDS, it is
// slower: 505 -> 536.)
template <bool UPPER, int BI, int BJ, int LDB = 4>
__device__ __forceinline__ void direct_loop(const GemmProblem& p, int row0, int col0, int kb, int ke, int lane,
                                            f32x4 (&acc)[4 * LDB]) {
    unsigned lost = 0;
    constexpr int kA[6] = {2, 1, 0, 1, 0, 0}, kB[6] = {0, 1, 2, 0, 1, 0};
    const int r = lane & 15, c = lane >> 4;
    unsigned oa[BI], ob[BJ];
#pragma unroll
    for (int i = 0; i < BI; ++i) oa[i] = (unsigned)min(row0 + 16 * i + r, p.M - 1) * (unsigned)p.lda * 4u + c * 32u;
#pragma unroll
    for (int j = 0; j < BJ; ++j) ob[j] = (unsigned)min(col0 + 16 * j + r, p.N - 1) * (unsigned)p.ldb * 4u + c * 32u;
    f32x4 ra[BI][2], rb[BJ][2];
    auto load = [&](int k) {
        const bool two = k >= p.K1;
        const int kl = two ? k - p.K1 : k;
        const gcchar* a = (const gcchar*)((two ? p.A2 : p.A) + kl);
        const gcchar* b = (const gcchar*)((two ? p.B2 : p.B) + kl);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int i = 0; i < BI; ++i) ra[i][h] = *(global_f32x4*)(a + oa[i] + 16 * h);
#pragma unroll
            for (int j = 0; j < BJ; ++j) rb[j][h] = *(global_f32x4*)(b + ob[j] + 16 * h);
        }
    };
    // One slab: split, then `refill` (the next slab's loads), then the MFMAs.
    auto slab = [&](auto refill) {
        SplitOct a[BI], b[BJ];
#pragma unroll
        for (int i = 0; i < BI; ++i) a[i] = split_oct(ra[i][0], ra[i][1], lost);
#pragma unroll
        for (int j = 0; j < BJ; ++j) b[j] = split_oct(rb[j][0], rb[j][1], lost);
        refill();
#pragma unroll
        for (int i = 0; i < BI; ++i)
#pragma unroll
            for (int u = 0; u < 6; ++u)
#pragma unroll
                for (int j = 0; j < BJ; ++j)
                    if (!UPPER || i <= j)
                        acc[i * LDB + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i].t[kA[u]], b[j].t[kB[u]],
                                                                                   acc[i * LDB + j], 0, 0, 0);
    };
    load(kb);
    int k = kb;
    for (; k + kSlab < ke; k += kSlab) slab([&] { load(k + kSlab); });
    slab([] {});
    if (__builtin_expect(__any(split_lost(lost) || any_non_finite(acc)), 0))
        fp32_blocks<true, BI, BJ, LDB>(p, row0, col0, kb, ke, lane, acc);
}

// One small-mode block: its K loop, then the epilogue of the block's
// quadrant, and the zeroing of the partial sums of its tile's quadrants that
// no block computes. The block's shape (on the diagonal of a symmetric
// result or not; 2 or 4 of its 16-row and 16-column strips inside the
// product) is uniform over the wave and picks the loop once.
__device__ __forceinline__ void small_unit(const GemmProblem& p, const SmallUnit& su, float beta1, int lane) {
    f32x4 acc[16];
#pragma unroll
    for (int b = 0; b < 16; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[b][e] = 0.0f;
    const int row0 = su.bm * kSmallDim, col0 = su.bn * kSmallDim, K = p.K;
    const bool diag = p.upper && su.bm == su.bn;   // uniform: the block is read with scalar loads
    // Strips inside the product: M and N are multiples of 32.
    const int bi = min(4, (p.M - row0) / 16), bj = min(4, (p.N - col0) / 16);
    if (diag) {  // a diagonal block is square: symmetric results have M = N
        if (bi == 4) direct_loop<true, 4, 4>(p, row0, col0, 0, K, lane, acc);
        else direct_loop<true, 2, 2>(p, row0, col0, 0, K, lane, acc);
    } else {
        if (bi == 4 && bj == 4) direct_loop<false, 4, 4>(p, row0, col0, 0, K, lane, acc);
        else if (bi == 4) direct_loop<false, 4, 2>(p, row0, col0, 0, K, lane, acc);
        else if (bj == 4) direct_loop<false, 2, 4>(p, row0, col0, 0, K, lane, acc);
        else direct_loop<false, 2, 2>(p, row0, col0, 0, K, lane, acc);
    }
    const int quadrant = ((su.bm & 1) << 1) | (su.bn & 1);
    gemm_epilogue(p, su.bm >> 1, su.bn >> 1, su.slot, beta1, acc, lane, quadrant);
    if (su.zero_mask && lane == 0) {
#pragma unroll
        for (int q = 0; q < kWaveSlots; ++q)
            if ((su.zero_mask >> q) & 1) p.partials[(size_t)su.slot * kWaveSlots + q] = 0.0;
    }
}

// Grouped launch: one workgroup per work unit of the list. The list is in
// dispatch order: consecutive workgroups go round-robin to the 8 XCDs, and
// the host arranged it so each XCD's share is balanced and reuses operand
// panels in its own L2. Units of split tiles leave their partial product in
// ws for gemm_fixup. A small-mode unit is a group of up to four 64 x 64
// blocks (small), one per wave.
template <bool BK>
__global__ __launch_bounds__(kGemmThreads, 2) void gemm_grouped(const GemmProblem* __restrict__ probs,
                                                                const TileDesc* __restrict__ tiles,
                                                                const SmallUnit* __restrict__ small,
                                                                float beta1, float* __restrict__ ws) {
    __shared__ __attribute__((aligned(16))) char lds[kSlabBytes];
    __shared__ int inexact;
    const TileDesc td = tiles[blockIdx.x];
    if (td.part == kSmallGroup) {
        if constexpr (BK) {
            const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform: its block is read with scalar loads
            if (w < td.tn) {
                const SmallUnit su = small[td.tm + w];
                small_unit(probs[su.prob], su, beta1, threadIdx.x & 63);
            }
        }
        return;
    }
    const GemmProblem p = probs[td.prob];
    f32x4 acc[16];
    gemm_mainloop<BK>(p, td.tm, td.tn, td.k0, td.k1, lds, &inexact, acc);
    if (td.part >= 0)
        store_partial(ws + (size_t)td.part * kSplitBlock, acc);
    else
        gemm_epilogue(p, td.tm, td.tn, td.slot, beta1, acc, threadIdx.x & 63, threadIdx.x >> 6);
}

// Wave-split launch, for a level with too few tiles to fill the GPU: one
// workgroup of eight waves per 32 x 32 block (blocks bm, bn of SmallUnit in units
// of 32; slot: the block's place in the problem's partial sums). Each wave takes an
// eighth of K straight from global memory (direct_loop); the eight partial
// products meet in LDS, where four waves sum one 16 x 16 piece each, in K order,
// and run the epilogue. No partial product leaves the CU and no second launch
// gathers them. Bound by latency: first loads, a few slabs per wave, epilogue.
constexpr int kWaveSplit = 8;
constexpr int kWaveSplitThreads = 64 * kWaveSplit;
__global__ __launch_bounds__(kWaveSplitThreads) void gemm_wave_split(const GemmProblem* __restrict__ probs,
                                                                     const SmallUnit* __restrict__ blocks,
                                                                     float beta1) {
    __shared__ f32x4 sum[kWaveSplit][4][64];
    __shared__ double red[4];
    const SmallUnit u = blocks[blockIdx.x];
    const GemmProblem p = probs[u.prob];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row0 = u.bm * 32, col0 = u.bn * 32, ns = p.K / kSlab;
    f32x4 acc[8];  // 2 x 2 blocks, row stride 2 (the last four unused)
#pragma unroll
    for (int b = 0; b < 8; ++b) acc[b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int kb = wave * ns / kWaveSplit * kSlab, ke = (wave + 1) * ns / kWaveSplit * kSlab;
    if (kb < ke) direct_loop<false, 2, 2, 2>(p, row0, col0, kb, ke, lane, acc);
#pragma unroll
    for (int b = 0; b < 4; ++b) sum[wave][b][lane] = acc[b];
    __syncthreads();
    double part = 0.0;
    if (wave < 4) {
        f32x4 v[1] = {sum[0][wave][lane]};
#pragma unroll
        for (int w = 1; w < kWaveSplit; ++w)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[0][e] += sum[w][wave][lane][e];
        const Place at = {row0 + (wave >> 1) * 16 + (lane >> 4) * 4, col0 + (wave & 1) * 16 + (lane & 15), u.bm == u.bn};
        part = gemm_epilogue_part(p, at, row0 + 32, col0 + 32, beta1, v);
    }
    if (p.flags & (EF_NORM | EF_DOT | EF_MOMENTUM)) {
        part = wave_sum(part);
        if (wave < 4 && lane == 0) red[wave] = part;
        __syncthreads();
        if (threadIdx.x == 0) p.partials[u.slot] = (red[0] + red[1]) + (red[2] + red[3]);
    }
}

// Split tiles of a grouped launch: sums the partial products in K order
// (a fixed order, so results are deterministic) and runs the epilogue. One
// workgroup per 64 x 64 quadrant of each split tile (workgroup b: tile b / 4,
// quadrant b % 4), whose wave w takes the w-th row of four 16 x 16 blocks of the
// quadrant, as wave b % 4 of the computing workgroups kept them. Bound by the
// latency of the pieces and of what the epilogue reads: four waves with four blocks
// each in place of one with sixteen, 512 x 4608's step (seven fixups) 910 -> 901 us.
constexpr int kFixupThreads = 256;
__global__ __launch_bounds__(kFixupThreads) void gemm_fixup(const GemmProblem* __restrict__ probs,
                                                            const FixupDesc* __restrict__ fix, float beta1,
                                                            const float* __restrict__ ws) {
    __shared__ double red[4];
    const FixupDesc fd = fix[blockIdx.x / kWaveSlots];
    const int quadrant = blockIdx.x % kWaveSlots, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const GemmProblem p = probs[fd.prob];
    // The pieces' first block of this wave, at thread 64 quadrant + lane of the computing workgroup.
    const float* src = ws + (size_t)fd.part0 * kSplitBlock + wave * 4 * 1024 + 4 * (quadrant * 64 + lane);
    auto load = [&](int s, f32x4 (&v)[4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = gload4(src + (size_t)s * kSplitBlock + j * 1024);
    };
    f32x4 acc[4], v0[4], v1[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto add = [&](const f32x4 (&v)[4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[j][e] += v[j][e];
    };
    // The loads of the next piece are in flight while the current one is added (nsplit >= 2).
    load(0, v0);
    int s = 0;
    for (; s + 2 <= fd.nsplit; s += 2) {
        load(s + 1, v1);
        add(v0);
        if (s + 2 < fd.nsplit) load(s + 2, v0);
        add(v1);
    }
    if (s < fd.nsplit) add(v0);
    Place at = place_of(fd.tm, fd.tn, lane, quadrant);
    at.row += 16 * wave;
    double part = gemm_epilogue_part(p, at, (fd.tm + 1) * kTile, (fd.tn + 1) * kTile, beta1, acc);
    if (p.flags & (EF_NORM | EF_DOT | EF_MOMENTUM)) {
        part = wave_sum(part);
        if (lane == 0) red[wave] = part;
        __syncthreads();
        if (threadIdx.x == 0)
            p.partials[(size_t)fd.slot * kWaveSlots + quadrant] = (red[0] + red[1]) + (red[2] + red[3]);
    }
}

}  // namespace jorge
