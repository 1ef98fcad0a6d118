// Gemm on register-operand tiles (tile_reg.h), F32 and split-bf16x3: one
// problem or a batch at fixed strides, each operand stored either way.  Serves
// problems of few tiles, which leave the LDS pipelines' 64 x 64 and larger
// tiles waiting (see reg_choice for the line and both sides' times).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "../../include/tgemm.h"
#include "gemm_reg.h"
#include "kargs.h"
#include "registry.h"
#include "tile_reg.h"

namespace tg {

template <class CF>
__global__ void __launch_bounds__(CF::NT, CF::OCC) reg_gemm_kernel(RegArgs a)
{
    __shared__ __attribute__((aligned(16))) char lds[CF::LDS_BYTES];
    reg_gemm_tile<CF>(a, blockIdx.x, lds);
}

namespace {

// Tile shapes: 32 x 32, 64 x 32 and (x3 only) 64 x 64 blocks per wave, four
// waves over K in chunks of 16.  Occupancy is what the registers allow: 7, 4
// and 2 workgroups per CU for f32's 70 and 120 and x3's 216 VGPRs.  Chunks of
// 32 cost f32 32 x 32 tiles a third of their occupancy (105 VGPRs; 1060^3
// 34.6 us against 29.7), and compiling for 8 spills (40.5 us).  Eight or
// sixteen waves over K gain nothing: four already use every SIMD of a CU.
template <int MODE, bool AK, bool BK>
struct RegTiles {
    using T0 = RCfg<MODE, AK, BK, 1, 1, 6>;
    using T1 = RCfg<MODE, AK, BK, 2, 1, 4>;
    using T2 = RCfg<MODE, AK, BK, 2, 2, 2>;
};

template <class CF>
int launch(RegArgs a, hipStream_t s)
{
    a.tiles_m = (int)(((int64_t)a.M + CF::BM - 1) / CF::BM);
    a.tiles_n = (int)(((int64_t)a.N + CF::BN - 1) / CF::BN);
    const int64_t per = (int64_t)a.tiles_m * a.tiles_n;
    if (per > INT32_MAX || !grid_fits(per * a.batch, CF::NT)) return TGEMM_NOT_SUPPORTED;
    const int64_t tiles = per * a.batch;
    hipLaunchKernelGGL(reg_gemm_kernel<CF>, dim3((unsigned)tiles), dim3(CF::NT), 0, s, a);
    return hipGetLastError() == hipSuccess ? TGEMM_SUCCESS : TGEMM_LAUNCH_FAILED;
}

template <int MODE, bool AK, bool BK>
int launch_tile(int tile, const RegArgs& a, hipStream_t s)
{
    using T = RegTiles<MODE, AK, BK>;
    if (tile == 0) return launch<typename T::T0>(a, s);
    if constexpr (MODE == MODE_X3)
        if (tile == 2) return launch<typename T::T2>(a, s);
    return launch<typename T::T1>(a, s);
}

template <int MODE>
int launch_mode(int tile, bool ak, bool bk, const RegArgs& a, hipStream_t s)
{
    if (ak) return bk ? launch_tile<MODE, true, true>(tile, a, s) : launch_tile<MODE, true, false>(tile, a, s);
    return bk ? launch_tile<MODE, false, true>(tile, a, s) : launch_tile<MODE, false, false>(tile, a, s);
}

}  // namespace

// The fastest tile by the time its busiest CU needs: rounds of 256 tiles times
// (fixed part + part per k), in microseconds, fitted to MI355X times of M, N in
// 32 .. 2048, K in 64 .. 4096 (one 32 x 32 tile per CU: f32 and x3 4.2 us at
// K = 256; 64 x 32: 5.8 and 5.4; 64 x 64, x3: 6.5).
int reg_best_tile(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype)
{
    auto cost = [&](int bm, int bn, double fixed, double per_k) {
        const int64_t t = ((M + bm - 1) / bm) * ((N + bn - 1) / bn) * batch;
        return (double)((t + 255) / 256) * (fixed + per_k * (double)K);
    };
    const bool x3 = dtype == TGEMM_F32_BF16X3;
    double best = cost(32, 32, 0.3, x3 ? 0.0054 : 0.0061);
    int tile = 0;
    const double c1 = cost(64, 32, 0.9, x3 ? 0.0090 : 0.0100);
    if (c1 < best) {
        best = c1;
        tile = 1;
    }
    if (x3 && cost(64, 64, 1.8, 0.0110) < best) tile = 2;
    return tile;
}

// Register tiles pay on few tiles.  MI355X, microseconds, against the best
// LDS-pipeline schedule:
//  - f32, up to 640 tiles of 64 x 64 (256 with K below 64): 256^3 4.2 against
//    10.2, 700^3 10.2 / 22.8, 1060^3 30 / 49, 1600^2 x 1500 77 / 89, 1600^2 x 64
//    9.7 / 10.0; past the line 2048^2 x 256 26.7 / 25.7, 3000^2 x 700 121 / 116;
//    below it with shallow K 1600^2 x 30 9.2 / 8.1;
//  - x3, up to 1280, or where the packed schedules start (768 tiles, K from
//    1024): 512^2 x 256 4.2 / 10.0, 1000^2 x 1024 14.9 / 31, 2048^2 x 256 17.1 /
//    18.0; past it 3000^2 x 256 32.7 / 30.4;
//  - both, up to 512 with K from 4096, where stream-K is the other side: f32
//    256^2 x 8192 46 / 427, 1000^2 x 8192 161 / 219, 64 x 4096^2 26 / 118 (x3 41 /
//    389, 87 / 136, 23 / 93); past it 1500^2 x 6000 284 / 279 (x3 174 / 174).
int reg_choice(int64_t M, int64_t N, int64_t K, int dtype)
{
    if (dtype != TGEMM_F32 && dtype != TGEMM_F32_BF16X3) return -1;
    const int64_t t64 = ((M + 63) / 64) * ((N + 63) / 64);
    const int64_t most = K < 64 ? 256 : K >= 4096 ? 512 : dtype == TGEMM_F32 ? 640 : K < 1024 ? 1280 : 767;
    return t64 <= most ? reg_best_tile(M, N, K, 1, dtype) : -1;
}

// Batches.  Nothing copied: up to 1100 tiles of 64 x 64 with K from 128, or 256
// of any K (MI355X, microseconds, against the grouped launch: f32 16 x 256^3
// 11.7 / 25.4, 64 x 256^3 27.4 / 29.2, 4 x 1024^3 74 / 82, x3 19 / 22 and 44 / 58
// for the last two; past the line f32 256 x 256^3 93 / 81 and 1000 x 64^3 15.2 /
// 13.8).  Otherwise the copies cost 1.33 us a megabyte and the larger tiles
// save 1.0 us (f32) or 1.43 us (x3) a gigaflop: f32 64 x 256^3 26 / 75, 2 x 4096^2
// x 2048 1052 / 1157, x3 4 x 2048^2 x 1024 158 / 208; past it x3 2 x 4096^2 x 2048
// 659 / 614.  Products of at most 32 x 32 have a kernel of their own.
bool reg_strided_pays(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, int64_t copied)
{
    if (std::max(M, N) <= 32) return false;
    if (copied > 0)
        return 2e-9 * (double)M * N * K * batch * (dtype == TGEMM_F32 ? 1.0 : 1.43) < 4e-6 * (double)copied * 1.33;
    const int64_t t64 = ((M + 63) / 64) * ((N + 63) / 64) * batch;
    return t64 <= (K < 128 ? 256 : 1100);
}

// Every offset inside a tile's chunk fits in 31 bits and floats are 4-byte
// aligned: K contiguous, 64 rows; row contiguous, 16 k (and 64 floats).
bool reg_serves(const void* A, bool ak, int64_t lda, const void* B, bool bk, int64_t ldb)
{
    if (((reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(B)) & 3) != 0) return false;
    auto reach = [](bool kc, int64_t ld) { return ld <= (int64_t)INT32_MAX / 4 / (kc ? 65 : 17); };
    return reach(ak, lda) && reach(bk, ldb);
}

int run_reg(int tile, int dtype, int64_t M, int64_t N, int64_t K, int64_t batch, float alpha, const float* A,
            bool ak, int64_t lda, int64_t sA, const float* B, bool bk, int64_t ldb, int64_t sB, float beta, float* C,
            int64_t ldc, int64_t sC, int group_m, int xcd_remap, hipStream_t s)
{
    if (batch < 1 || batch > INT32_MAX || !reg_serves(A, ak, lda, B, bk, ldb)) return TGEMM_NOT_SUPPORTED;
    RegArgs a{};
    a.A = A;
    a.B = B;
    a.C = C;
    a.lda = lda;
    a.ldb = ldb;
    a.ldc = ldc;
    a.sA = sA;
    a.sB = sB;
    a.sC = sC;
    a.M = (int)M;
    a.N = (int)N;
    a.K = (int)K;
    a.batch = (int)batch;
    a.alpha = alpha;
    a.beta = beta;
    a.group_m = std::max(group_m, 1);
    a.xcd_remap = xcd_remap ? 1 : 0;
    return dtype == TGEMM_F32 ? launch_mode<MODE_F32>(tile, ak, bk, a, s) : launch_mode<MODE_X3>(tile, ak, bk, a, s);
}

}  // namespace tg
