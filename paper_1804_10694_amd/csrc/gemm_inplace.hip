// One-problem gemm on in-place tiles (F32 and split-bf16x3): one workgroup per
// macro-tile of the tiling map (Section III-C; tile order as in kargs.h), K
// panels loaded from the caller's A and B straight into LDS by direct-to-LDS
// buffer loads (tile_inplace.h), so no packing pass runs.  Tile edges need no
// separate code path: loads past M, N or K return zero from the buffer range
// and the epilogue drops stores outside C (the full/partial tile split of
// Section V-A is done by the hardware's range check).  The small tiles' low
// LDS and register footprint lets several workgroups share a CU, which hides
// the panel latency on problems too small to keep the large packed tiles busy.
#include <hip/hip_runtime.h>

#include "kargs.h"
#include "registry.h"
#include "tile_inplace.h"
#include "../../include/tgemm.h"

namespace tg {

__device__ __forceinline__ PackedArgs inplace_args(const GemmArgs& g)
{
    PackedArgs a;
    a.A = static_cast<const char*>(g.A);
    a.Alo = nullptr;
    a.B = static_cast<const char*>(g.B);
    a.Blo = nullptr;
    a.C = g.C;
    a.sA = nullptr;
    a.sB = nullptr;
    a.ldc = g.ldc;
    a.lds_a = 0;
    a.lds_b = 0;
    a.lda = g.lda;
    a.ldb = g.ldb;
    a.M = g.M;
    a.N = g.N;
    a.K = g.K;
    a.Kp = 0;
    a.alpha = g.alpha;
    a.beta = g.beta;
    a.tiles_m = g.tiles_m;
    a.tiles_n = g.tiles_n;
    a.group_m = g.group_m;
    a.xcd_remap = g.xcd_remap;
    return a;
}

template <class CF>
__device__ __forceinline__ void inplace_any(const GemmArgs& g, int m0, int n0, char* lds)
{
    const PackedArgs a = inplace_args(g);
    // 16-byte loads at any 4-byte aligned address (float32 data always is)
    const bool vec = ((reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.B)) & 3) == 0;
    if (vec) inplace_tile<CF, true>(a, m0, n0, lds);
    else inplace_tile<CF, false>(a, m0, n0, lds);
}

template <class CF, int OCC>
__global__ void __launch_bounds__(CF::NT, OCC) inplace_gemm_kernel(GemmArgs g)
{
    __shared__ __attribute__((aligned(1024))) char lds[CF::LDS_BYTES];
    const TileCoord tc = map_tile(blockIdx.x, g.tiles_m, g.tiles_n, g.group_m, g.xcd_remap);
    inplace_any<CF>(g, tc.tm * CF::BM, tc.tn * CF::BN, lds);
}

// f32 128 x 128 tiles, the last `rest` of the tile order as quarters of 64 x 64 that
// follow the whole ones.  The matrix cores bind it, and tiles / 256 is a few, so one
// CU's extra tile is the time of the launch: with the tiles past whole multiples of
// 256 in quarters no CU has more than a quarter or three over (the sums are the same
// bit for bit).  MI355X, 128 x 128 / 64 x 64 only / so: 4097 x 3001 x 2053 (792 tiles)
// 485 / 419 / 402 us, 3706 x 4759 x 2398 (1102) 740 / 759 / 677, 1108 x 7966 x 1210
// (567) 224 / 188 / 169, 7258 x 4740 x 3343 (2166) 1784 / 1862 / 1671.  Quarters first
// took the workgroup slots that whole tiles then waited for: 864 tiles 902 us
// against 724.
__global__ void __launch_bounds__(256, kInplace128Occ<MODE_F32>) inplace_rest_kernel(GemmArgs g, int rest)
{
    using CF = InplaceCfg128<MODE_F32>;
    using Q = InplaceCfg64<MODE_F32>;
    static_assert(CF::NT == 256 && Q::NT == 256 && Q::BM * 2 == CF::BM && Q::BN * 2 == CF::BN, "quarters of a tile");
    __shared__ __attribute__((aligned(1024))) char lds[CF::LDS_BYTES];
    const int whole = g.tiles_m * g.tiles_n - rest, wg = blockIdx.x;
    if (wg < whole) {
        const TileCoord tc = map_tile(g.xcd_remap ? xcd_order(wg, whole) : wg, g.tiles_m, g.tiles_n, g.group_m, 0);
        inplace_any<CF>(g, tc.tm * CF::BM, tc.tn * CF::BN, lds);
    } else {
        const int q = wg - whole;
        const TileCoord tc = map_tile(whole + q / 4, g.tiles_m, g.tiles_n, g.group_m, 0);
        const int m0 = tc.tm * CF::BM + (q / 2 % 2) * Q::BM, n0 = tc.tn * CF::BN + (q % 2) * Q::BN;
        if (m0 < g.M && n0 < g.N) inplace_any<Q>(g, m0, n0, lds);
    }
}

// Past three quarters of a round every CU would have three quarters or a fourth, at
// the 64 x 64 tile's lower rate: 697 tiles (185 over) 248 us against 253, 708 (196)
// 410 against 398, 741 (229) 354 against 336.
constexpr int kRestTiles = 192;

// Whether 128 x 128 tiles serve these sizes better than 64 x 64: at any number past one
// per CU where the ones left over go out as quarters, unless they pad M x N by more than
// 4% above what 64 x 64 tiles do.  Time against 64 x 64 tiles, 31 shapes of M, N in [1000,
// 8192] and K in [300, 4096]: 0.87 to 0.97; padding 5.8% more 1.05 (2200^2 x 200), 20%
// more 1.08 (300 x 15000 x 512).
bool inplace_joined(int64_t M, int64_t N)
{
    auto tiles = [&](int64_t b) { return ((M + b - 1) / b) * ((N + b - 1) / b); };
    const int64_t t = tiles(128);
    return M >= 256 && N >= 256 && t > 256 && t % 256 <= kRestTiles && 100 * t <= 26 * tiles(64);
}

hipError_t launch_inplace(const SchedDesc& d, const GemmArgs& a, hipStream_t s)
{
    const int tiles = a.tiles_m * a.tiles_n;
    const int rest = d.dtype == TGEMM_F32 && d.BM == 128 && tiles > 256 ? tiles % 256 : 0;
    if (rest == 0 || rest > kRestTiles || !grid_fits(tiles + 3 * rest, d.threads)) {
        hipLaunchKernelGGL(d.kernel, dim3((unsigned)tiles), dim3(d.threads), 0, s, a);
    } else {
        const dim3 grid((unsigned)(tiles + 3 * rest));
        hipLaunchKernelGGL(inplace_rest_kernel, grid, dim3(256), 0, s, a, rest);
    }
    return hipGetLastError();
}

#define TG_ISCHED(DT, CF, OCC) \
    {DT, CF::BM, CF::BN, CF::BK, CF::WGM, CF::WGN, 1, CF::LDS_BYTES, CF::NT, &inplace_gemm_kernel<CF, OCC>, 0, 32, 1}

static const SchedDesc kInplaceSchedules[] = {
    TG_ISCHED(TGEMM_F32, InplaceCfg64<MODE_F32>, kInplace64Occ<MODE_F32>),
    TG_ISCHED(TGEMM_F32, InplaceCfg128<MODE_F32>, kInplace128Occ<MODE_F32>),
    TG_ISCHED(TGEMM_F32_BF16X3, InplaceCfg64<MODE_X3>, kInplace64Occ<MODE_X3>),
    TG_ISCHED(TGEMM_F32_BF16X3, InplaceCfg128<MODE_X3>, kInplace128Occ<MODE_X3>),
};

const SchedDesc* inplace_schedules(int* n)
{
    *n = (int)(sizeof(kInplaceSchedules) / sizeof(kInplaceSchedules[0]));
    return kInplaceSchedules;
}

// A tile's rows of A and a panel's rows of B must lie within the 2^31-byte
// reach of a buffer offset.
bool inplace_reach_ok(const SchedDesc& d, int64_t lda, int64_t ldb)
{
    return (int64_t)d.BM * lda * 4 <= INT32_MAX && (int64_t)d.BK * ldb * 4 <= INT32_MAX;
}

}  // namespace tg
