// Register-operand tile (F32 and split-bf16x3): MFMA operands go from global
// memory straight into the registers of the lane that owns them; LDS only
// sums the waves that share a tile's K.
//
// Why: the LDS pipelines of tile_packed.h and tile_inplace.h give a 64 x 64
// tile to a workgroup and walk its K in 16-deep panels with a barrier each.  A
// problem of a few dozen tiles then runs one wave per SIMD on a part of the
// chip and waits out the memory latency at every panel.  Here a workgroup's
// tile can be as small as one 32 x 32 block, its four waves take its K in turns
// of 16 (a chunk), and no wave waits for another until the final sum.  An F32
// MFMA takes 64 cycles for 8 bytes per lane, so the operand loads of a 32 x 32
// block (16 bytes a cycle per CU with four waves, half of the L1's rate) need no
// LDS to be shared.
//
// Both operands may be stored either way: K contiguous (A row-major, B^T
// row-major) or row contiguous (A^T row-major, B row-major), so products of
// transposed matrices need no transposing pass.  In a chunk, lane half h takes
// k = 8h + q (q = 0..7) of its row for both operands: two 16-byte loads, which
// between the halves use 64 contiguous bytes of a K-contiguous row, or eight
// 4-byte loads of which each covers two 128-byte runs of 32 consecutive rows.
// MFMA q pairs equal k.
//
// Edges.  Rows past the end are clamped to the last row (their sums are never
// stored).  The chunk that holds K's end loads element by element at clamped
// k and replaces what lies past K by zero on both sides, so every load stays
// inside the matrix and nothing beyond it (a NaN, say) reaches a sum.
#pragma once
#include <hip/hip_runtime.h>

#include "tile_f32x3.h"

namespace tg {

struct RegArgs {
    const float* A;
    const float* B;
    float* C;
    int64_t lda, ldb, ldc;  // elements between rows (K contiguous) or between k (row contiguous)
    int64_t sA, sB, sC;     // elements between the problems of a batch
    int M, N, K, batch;
    float alpha, beta;
    int tiles_m, tiles_n, group_m, xcd_remap;
};

// A tile of TM x TN blocks of 32 x 32; AK / BK: A / B has K contiguous.  OCC:
// waves per SIMD to compile for.
template <int MODE_, bool AK_, bool BK_, int TM_, int TN_, int OCC_>
struct RCfg {
    static constexpr int MODE = MODE_, TM = TM_, TN = TN_, OCC = OCC_;
    static constexpr int WK = 4;        // waves, over K
    static constexpr int CH = 16;       // k per chunk
    static constexpr int KL = CH / 2;   // k per lane and chunk
    static constexpr bool AK = AK_, BK = BK_;
    static constexpr int BM = 32 * TM, BN = 32 * TN;
    static constexpr int NT = 64 * WK;
    static constexpr int AR = 16 / WK;  // sums per lane and block that a wave stores
    static constexpr int LDS_BYTES = WK * TM * TN * 4096;  // every wave's sums
    static_assert(MODE == MODE_F32 || MODE == MODE_X3, "float32 operands");
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t reg_rsrc(const char* base)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, 0x7fffffff, 0x00020000);
}

// One operand's chunk loads for T blocks: rows r0 + 32 i of a matrix of R rows.
template <bool KC, int T, int CH>
struct RegOperand {
    static constexpr int KL = CH / 2;
    const char* base;
    int64_t ld4;
    int ld, h;
    int voff[T];  // this lane's row of block i, and its first k of a chunk

    __device__ __forceinline__ void init(const float* X, int64_t ldx, int r0, int R, int lane)
    {
        h = lane >> 5;
        ld4 = ldx * 4;
        ld = (int)ld4;
        base = reinterpret_cast<const char*>(KC ? X + (int64_t)r0 * ldx : X + r0);
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int row = min(r0 + 32 * i + (lane & 31), R - 1) - r0;
            voff[i] = KC ? row * ld + 4 * KL * h : row * 4 + KL * h * ld;
        }
    }

    // Chunk c, which lies inside K.
    __device__ __forceinline__ void load(int c, float (&v)[T][KL]) const
    {
        const int k0 = c * CH;
        const __amdgpu_buffer_rsrc_t r = reg_rsrc(base + (KC ? (int64_t)k0 * 4 : k0 * ld4));
#pragma unroll
        for (int i = 0; i < T; ++i) {
            if constexpr (KC) {
#pragma unroll
                for (int q = 0; q < KL / 4; ++q) {
                    const f32x4 x = __builtin_bit_cast(
                        f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, voff[i] + 16 * q, 0, 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[i][4 * q + e] = x[e];
                }
            } else {
#pragma unroll
                for (int q = 0; q < KL; ++q)
                    v[i][q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff[i], q * ld, 0));
            }
        }
    }

    // The chunk that holds K's end (left of its k exist, 1 .. CH - 1).
    __device__ __forceinline__ void load_tail(int c, int left, float (&v)[T][KL]) const
    {
        const int k0 = c * CH;
        const __amdgpu_buffer_rsrc_t r = reg_rsrc(base + (KC ? (int64_t)k0 * 4 : k0 * ld4));
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int q = 0; q < KL; ++q) {
                const int k = KL * h + q, kk = min(k, left - 1);
                const float x = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                    r, (KC ? voff[i] - 4 * KL * h + kk * 4 : voff[i] + (kk - KL * h) * ld), 0, 0));
                v[i][q] = k < left ? x : 0.f;
            }
    }
};

template <class CF>
struct RegOps {
    float a[CF::TM][CF::KL], b[CF::TN][CF::KL];
};

template <class CF>
__device__ __forceinline__ void reg_mma(const RegOps<CF>& o, f32x16 (&acc)[CF::TM][CF::TN])
{
    if constexpr (CF::MODE == MODE_F32) {
#pragma unroll
        for (int q = 0; q < CF::KL; ++q)
#pragma unroll
            for (int i = 0; i < CF::TM; ++i)
#pragma unroll
                for (int j = 0; j < CF::TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(o.a[i][q], o.b[j][q], acc[i][j], 0, 0, 0);
    } else {
        // two 16-deep MFMA groups: each lane half gives eight of its k
#pragma unroll
        for (int g = 0; g < CF::KL / 8; ++g) {
            bf16x8 ah[CF::TM], al[CF::TM], bh[CF::TN], bl[CF::TN];
#pragma unroll
            for (int i = 0; i < CF::TM; ++i) split_bf16x8(o.a[i] + 8 * g, ah[i], al[i]);
#pragma unroll
            for (int j = 0; j < CF::TN; ++j) split_bf16x8(o.b[j] + 8 * g, bh[j], bl[j]);
            // small terms first: lo*hi, hi*lo, then hi*hi
#pragma unroll
            for (int i = 0; i < CF::TM; ++i)
#pragma unroll
                for (int j = 0; j < CF::TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[i], bh[j], acc[i][j], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < CF::TM; ++i)
#pragma unroll
                for (int j = 0; j < CF::TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bl[j], acc[i][j], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < CF::TM; ++i)
#pragma unroll
                for (int j = 0; j < CF::TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bh[j], acc[i][j], 0, 0, 0);
        }
    }
}

// What a wave holds of its blocks after the sum over the K waves: sums r = 0 ..
// AR - 1 of block (i, j), at row m0 + 32 i + row(r) + 4 (lane / 32), column
// n0 + 32 j + lane % 32.
template <class CF>
struct RegSums {
    float v[CF::TM][CF::TN][CF::AR];
    int m0, n0, first;  // first: number of this wave's first sum among the block's 16

    __device__ __forceinline__ int row(int r) const { return 8 * ((first + r) >> 2) + ((first + r) & 3); }
};

// Column sums of B over the tile's K (COLSUM): cs[j] of lane l < 32 in K wave 0
// is the sum over all k of B's column 32 j + l.
template <class CF, bool COLSUM = false, class EPI>
__device__ __forceinline__ void reg_tile(const RegArgs& a, int m0, int n0, char* lds, const EPI& epi)
{
    const int t = threadIdx.x, lane = t & 63;
    const int wk = __builtin_amdgcn_readfirstlane(t >> 6);

    RegOperand<CF::AK, CF::TM, CF::CH> la;
    RegOperand<CF::BK, CF::TN, CF::CH> lb;
    la.init(a.A, a.lda, m0, a.M, lane);
    lb.init(a.B, a.ldb, n0, a.N, lane);

    f32x16 acc[CF::TM][CF::TN];
#pragma unroll
    for (int i = 0; i < CF::TM; ++i)
#pragma unroll
        for (int j = 0; j < CF::TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    float cs[CF::TN] = {};

    RegOps<CF> x, y;
    auto load = [&](int c, RegOps<CF>& o) {
        la.load(c, o.a);
        lb.load(c, o.b);
    };
    auto use = [&](const RegOps<CF>& o) {
        if constexpr (COLSUM) {
#pragma unroll
            for (int j = 0; j < CF::TN; ++j)
#pragma unroll
                for (int q = 0; q < CF::KL; ++q) cs[j] += o.b[j][q];
        }
        reg_mma<CF>(o, acc);
    };
    // Wave wk takes the whole chunks wk, wk + WK, ...; the one whose turn would
    // be next takes K's last, partial chunk, and takes it first.  The next
    // chunk's loads are in flight during the MFMAs of this one.
    const int nc = a.K / CF::CH, left = a.K % CF::CH;
    const bool tail = left != 0 && nc % CF::WK == wk;
    int c = wk;
    if (tail) {
        la.load_tail(nc, left, x.a);
        lb.load_tail(nc, left, x.b);
    } else if (c < nc) {
        load(c, x);
        c += CF::WK;
    }
    if (tail || c - CF::WK >= 0) {
        while (true) {  // x holds a chunk; c is the next one
            if (c >= nc) {
                use(x);
                break;
            }
            load(c, y);
            use(x);
            if (c + CF::WK >= nc) {
                use(y);
                break;
            }
            load(c + CF::WK, x);
            use(y);
            c += 2 * CF::WK;
        }
    }

    RegSums<CF> s;
    s.m0 = m0;
    s.n0 = n0;
    s.first = wk * CF::AR;
    float* red = reinterpret_cast<float*>(lds);
    // the four sums of a lane's group g of block b, of K wave k (one 16-byte LDS access)
    static_assert(CF::AR == 4, "a wave stores one group of every block");
    auto at = [&](int k, int b, int g) { return red + ((k * CF::TM * CF::TN + b) * 4 + g) * 256 + lane * 4; };
#pragma unroll
    for (int b = 0; b < CF::TM * CF::TN; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) at(wk, b, g)[e] = acc[b / CF::TN][b % CF::TN][g * 4 + e];
    __syncthreads();
#pragma unroll
    for (int b = 0; b < CF::TM * CF::TN; ++b)
#pragma unroll
        for (int r = 0; r < CF::AR; ++r) s.v[b / CF::TN][b % CF::TN][r] = 0.f;
#pragma unroll
    for (int k = 0; k < CF::WK; ++k)
#pragma unroll
        for (int b = 0; b < CF::TM * CF::TN; ++b)
#pragma unroll
            for (int r = 0; r < CF::AR; ++r) s.v[b / CF::TN][b % CF::TN][r] += at(k, b, wk)[r];
    if constexpr (COLSUM) {
#pragma unroll
        for (int j = 0; j < CF::TN; ++j) cs[j] += __shfl_xor(cs[j], 32);
        __syncthreads();
        if (lane < 32)
#pragma unroll
            for (int j = 0; j < CF::TN; ++j) red[(wk * CF::TN + j) * 32 + lane] = cs[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < CF::TN; ++j) {
            cs[j] = 0.f;
#pragma unroll
            for (int k = 0; k < CF::WK; ++k) cs[j] += red[(k * CF::TN + j) * 32 + (lane & 31)];
        }
        if (wk == 0 && lane < 32) epi.columns(cs, s, lane);
    }
    epi(s, lane);
}

// C = alpha * sums + beta * C.
template <class CF>
struct RegStoreC {
    const RegArgs& a;
    float* C;
    __device__ __forceinline__ void operator()(const RegSums<CF>& s, int lane) const
    {
        write_c<CF::TM, CF::TN, CF::AR>(
            C, a.ldc, a.M, a.N, a.beta, 4 * (lane >> 5), lane & 31,
            [&](int i, int j, float (&v)[CF::AR]) {
#pragma unroll
                for (int r = 0; r < CF::AR; ++r) v[r] = a.alpha * s.v[i][j][r];
            },
            [&](int i, int j, int& r0, int& c0) {
                r0 = s.m0 + 32 * i;
                c0 = s.n0 + 32 * j;
            },
            [&](int r) { return s.row(r); });
    }
};

// Tile `wg` of a (batched) problem.  The XCD remap runs over all tiles of the
// batch, so the tiles of one problem share an L2.
template <class CF>
__device__ __forceinline__ void reg_gemm_tile(RegArgs a, int wg, char* lds)
{
    const int per = a.tiles_m * a.tiles_n;
    int b = 0;
    TileCoord tc;
    if (a.batch > 1) {
        const int T = per * a.batch;
        const int x = wg % kNumXcd, base = T / kNumXcd, rem = T % kNumXcd;
        const int s = x * base + min(x, rem) + wg / kNumXcd;
        b = s / per;
        tc = map_tile(s - b * per, a.tiles_m, a.tiles_n, a.group_m, 0);
    } else {
        tc = map_tile(wg, a.tiles_m, a.tiles_n, a.group_m, a.xcd_remap);
    }
    a.A += b * a.sA;
    a.B += b * a.sB;
    reg_tile<CF>(a, tc.tm * CF::BM, tc.tn * CF::BN, lds, RegStoreC<CF>{a, a.C + b * a.sC});
}

}  // namespace tg
