// Back-to-back gemm with the intermediate kept on chip (project addition; the
// paper's VGG block fuses its two layers so that the intermediate stays close
// to the arithmetic, Section VI-A):
//
//   T = act(A B)                 A: M x K, B: K x N1 (N1 <= 256)
//   E = alpha * T D + beta * E   D: N1 x N2, E: M x N2
//
// One workgroup of four waves owns 64 rows of the output (or 32, below).  Phase 1
// computes its 64 x N1 block of T, a quarter of the columns per wave: 32-deep
// panels of A go from memory into a ring in LDS, three ahead of the one being
// read; B goes from L2 straight into each wave's registers, one panel ahead
// (no other wave of the workgroup needs those columns).  act is applied in
// registers and T stored into LDS as N1/32 panels in the layout of A's, over the
// ring; T never goes to memory.  Phase 2 walks E's columns in chunks of 256 (or
// 128), each wave with A operands from the resident T panels and its columns of D
// in registers, without a barrier, then writes alpha * acc + beta * E.  A workgroup
// holds T only: two per CU for N1 up to 256, three up to 128.  Columns of T at or
// past N1 are stored as zero, so that nothing read past N1 (whatever B holds
// there) can reach E.  T is kept in FP32; the x3 form splits it, like every
// operand, into bf16 high and low parts when it reads it from LDS.
//
// What bounds it: the matrix cores (f32 at 98304 x 256 x 256 x 256: 167 us of MFMAs
// in 198), and the waves of a CU reaching their epilogues together.  With B and D
// through LDS in 16-deep panels, a barrier each, and E in chunks of 128 columns, f32
// took 212 there and x3 114, now 93.  A workgroup alone on its CU takes 1.7 times
// as long as its MFMAs, so the rows past the last whole round of workgroups go out in
// 32s, and first, beside others: 100352 rows f32 236 -> 217 us, x3 130 -> 100;
// 8192 x 1024 x 256 x 1024 f32 158 -> 83; 1000 rows 42 -> 24.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "../../include/tgemm.h"
#include "kargs.h"
#include "registry.h"
#include "tile_inplace.h"

namespace tg {

int ensure_device(hipStream_t stream);

struct G2Args {
    const char* A;
    const char* B;
    const char* D;
    float* E;
    int64_t lda, ldb, ldd, lde;
    int M, N1, N2, K;
    float alpha, beta;
    int relu;
    int tall;  // workgroups of 64 rows; those before them take 32 each of the rows left
};

template <int MODE, int N1P, int RB>
struct G2Cfg {
    static constexpr int BK = 32, AHEAD = 3;
    using P1 = ICfg<MODE, RB, N1P, BK, 1, 4, 2>;  // phase 1: an RB x N1P block of T, 4 waves side by side
    template <int TN>
    using P2 = ICfg<MODE, RB, 128 * TN, BK, 1, 4, 2>;  // phase 2: an RB x 128 TN chunk of E
    static constexpr int PANEL = RB * BK * 4;  // one 32-column panel of A or T (8 units a row)
    static constexpr int NPAN = N1P / BK;
    static constexpr int LDS_BYTES = NPAN * PANEL;
    static_assert(AHEAD < NPAN, "A panels in flight and the one being read fit where T goes");
};

// Rows of B or D from one on: what follows in bytes (0 past the last row or column).
// A panel's range and the lanes' offsets into it are unsigned 32-bit numbers up to 2^32.
struct G2Src {
    __amdgpu_buffer_rsrc_t r;
    uint32_t row_bytes;
};
constexpr int64_t kG2RowFloats = INT32_MAX / 64;  // longest rows of B and D
template <class G>
constexpr bool kG2Reach = G::BK * 4 * kG2RowFloats <= (int64_t)UINT32_MAX &&
                          (G::BK - 1) * 4 * kG2RowFloats + 128 * (G::template P2<2>::TN + 1) <= (int64_t)UINT32_MAX;
static_assert(kG2Reach<G2Cfg<MODE_F32, 256, 64>> && kG2Reach<G2Cfg<MODE_X3, 256, 64>>,
              "a panel of the longest rows, and its last row's last lane");

// Rows k0 .. k0 + BK of the columns from n0 on of a K x N matrix.
template <int BK>
__device__ __forceinline__ G2Src g2_rows(const char* base, int64_t ld, int K, int N, int k0, int n0)
{
    const int rows = min(BK, K - k0), cols = N - n0;
    const bool any = rows > 0 && cols > 0;
    const uint32_t row_bytes = (uint32_t)ld * 4u;
    return {make_rsrc(base + (any ? k0 * ld + n0 : 0) * 4,
                      any ? (int)((uint32_t)(rows - 1) * row_bytes + (uint32_t)cols * 4u) : 0), row_bytes};
}

// One panel (BK rows) of B or D in registers, one 4-byte load per value: lane half h
// holds rows MK g + HS h + e of group g, column 32 j + lane % 32 of the wave's columns.
// The row goes into the buffer resource (scalar registers), not into lane offsets,
// which the compiler would keep in 16 vector registers.
template <class CF>
struct G2Rows {
    float v[CF::NG][CF::TN][CF::HS];

    __device__ __forceinline__ void load_group(const G2Src& src, uint32_t at, int g)
    {
#pragma unroll
        for (int e = 0; e < CF::HS; ++e) {
            const uint32_t off = at + (uint32_t)(CF::MK * g + e) * src.row_bytes;
#pragma unroll
            for (int j = 0; j < CF::TN; ++j)
                v[g][j][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(src.r, (int)(off + 128 * j), 0, 0));
        }
    }
};

// The MFMAs of group g: A operands as read from LDS, B operands from registers.
template <class CF>
__device__ __forceinline__ void g2_mma(const typename InplaceOps<CF>::Ops& oa, const G2Rows<CF>& b, int g,
                                       f32x16 (&acc)[CF::TM][CF::TN])
{
    typename InplaceOps<CF>::Ops o = oa;
#pragma unroll
    for (int j = 0; j < CF::TN; ++j) {
        if constexpr (CF::MODE == MODE_F32) {
#pragma unroll
            for (int e = 0; e < 4; ++e) o.b[j][e] = b.v[g][j][e];
        } else {
            split_bf16x8(b.v[g][j], o.bh[j], o.bl[j]);
        }
    }
    InplaceOps<CF>::compute(o, acc);
}

// One panel: A from LDS at `la`, B from registers, each group's registers refilled
// from the next panel (through `next`) once its MFMAs have been issued.
template <class CF>
__device__ __forceinline__ void g2_panel(const char* la, G2Rows<CF>& b, const G2Src& next, uint32_t at,
                                         f32x16 (&acc)[CF::TM][CF::TN], int lane)
{
    using OP = InplaceOps<CF>;
    typename OP::Ops oa[2];
    OP::load_a(la, oa[0], 0, 0, lane);
#pragma unroll
    for (int g = 0; g < CF::NG; ++g) {
        if (g + 1 < CF::NG) OP::load_a(la, oa[(g + 1) & 1], g + 1, 0, lane);
        g2_mma<CF>(oa[g & 1], b, g, acc);
        b.load_group(next, at, g);
    }
}

template <class CF>
__device__ __forceinline__ void zero_acc(f32x16 (&acc)[CF::TM][CF::TN])
{
#pragma unroll
    for (int i = 0; i < CF::TM; ++i)
#pragma unroll
        for (int j = 0; j < CF::TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
}

// Phase 2: E[m0:m0+RB, :] = alpha * T D + beta * E in chunks of 128 TN columns, a
// quarter per wave.  No barriers: T only is shared, and it stays.
template <class G, int TN>
__device__ __forceinline__ void g2_second(const G2Args& g, const char* tbuf, int m0, int wave, int lane)
{
    using P2 = typename G::template P2<TN>;
    const int h = lane >> 5, l32 = lane & 31;
    const int wn0 = wave * P2::WTN;
    const int npanel = (g.N1 + G::BK - 1) / G::BK;
    const uint32_t at = (uint32_t)(P2::HS * h) * (uint32_t)g.ldd * 4u + (uint32_t)l32 * 4u;
    G2Rows<P2> b;
    const G2Src first = g2_rows<G::BK>(g.D, g.ldd, g.N1, g.N2, 0, wn0);
#pragma unroll
    for (int q = 0; q < P2::NG; ++q) b.load_group(first, at, q);
    for (int n0 = wn0; n0 < g.N2; n0 += P2::BN) {
        f32x16 acc[P2::TM][P2::TN];
        zero_acc<P2>(acc);
        for (int s = 0; s < npanel; ++s) {
            const bool last = s + 1 == npanel;  // the next chunk's first panel follows
            g2_panel<P2>(tbuf + s * G::PANEL, b,
                         g2_rows<G::BK>(g.D, g.ldd, g.N1, g.N2, last ? 0 : (s + 1) * G::BK, last ? n0 + P2::BN : n0),
                         at, acc, lane);
        }
        write_c<P2::TM, P2::TN, 16>(
            g.E, g.lde, g.M, g.N2, g.beta, 4 * h, l32,
            [&](int i, int j, float (&v)[16]) {
#pragma unroll
                for (int r = 0; r < 16; ++r) v[r] = g.alpha * acc[i][j][r];
            },
            [&](int i, int j, int& r0, int& c0) {
                r0 = m0 + 32 * i;
                c0 = n0 + 32 * j;
            },
            [](int r) { return 8 * (r >> 2) + (r & 3); });
    }
}

template <int MODE, int N1P, int RB, bool VEC>
__device__ __forceinline__ void g2_block(const G2Args& g, int m0, char* lds)
{
    using G = G2Cfg<MODE, N1P, RB>;
    using P1 = typename G::P1;
    const int t = threadIdx.x, lane = t & 63, h = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);

    // ---- phase 1: T block = act(A[m0:m0+RB, :] B)
    {
        PackedArgs a{};
        a.A = g.A;
        a.lda = g.lda;
        a.M = g.M;
        a.K = g.K;
        InplaceA<P1, VEC> al;
        al.init(a, m0, lane, wave, typename InplaceA<P1, VEC>::Geom());
        const int wn0 = wave * P1::WTN;
        const int npanel = (g.K + G::BK - 1) / G::BK;
        const uint32_t at = (uint32_t)(P1::HS * h) * (uint32_t)g.ldb * 4u + (uint32_t)l32 * 4u;
        for (int s = 0; s < G::AHEAD && s < npanel; ++s) al.issue(s, lds + s * G::PANEL);
        G2Rows<P1> b;
        const G2Src first = g2_rows<G::BK>(g.B, g.ldb, g.K, g.N1, 0, wn0);
#pragma unroll
        for (int q = 0; q < P1::NG; ++q) b.load_group(first, at, q);
        f32x16 acc[P1::TM][P1::TN];
        zero_acc<P1>(acc);
        wait_vmcnt<0>();
        for (int s = 0; s < npanel; ++s) {
            // A panel s was issued at panel s - 3 (or before the wait above), and the
            // panels since issued more loads of B than may be in flight here
            constexpr int FLIGHT = P1::NG * P1::HS * P1::TN;
            wait_vmcnt<FLIGHT>();
            wait_lds_reads();  // of panel s - 1, whose stage may be refilled from here on
            lds_barrier();
            if (s + G::AHEAD < npanel) al.issue(s + G::AHEAD, lds + (s + G::AHEAD) % G::NPAN * G::PANEL);
            g2_panel<P1>(lds + s % G::NPAN * G::PANEL, b,
                         g2_rows<G::BK>(g.B, g.ldb, g.K, g.N1, (s + 1) * G::BK, wn0), at, acc, lane);
        }
        // act(acc) -> T panels, over the A panels once every wave is done with
        // them; columns at or past N1 become zero
        wait_lds_reads();
        lds_barrier();
        const bool pad = wn0 + P1::WTN > g.N1;
#pragma unroll
        for (int j = 0; j < P1::TN; ++j) {
            // block j's columns are one T panel; row 32 i + 8 (r / 4) + 4 h + r % 4 of column
            // l32 is unit l32 / 4, XORed as pk_slot<8> has it with row / 2 =
            // 4 (r / 4) + 2 h + (r % 4) / 2, mod 8
            const int col = (wn0 / 32 + j) * G::PANEL + 4 * h * 128 + ((l32 / 4) ^ (2 * h)) * 16 + (l32 % 4) * 4;
            const bool out = wn0 + 32 * j + l32 >= g.N1;
#pragma unroll
            for (int i = 0; i < P1::TM; ++i) {
                f32x16 v = acc[i][j];
                if (g.relu)
#pragma unroll
                    for (int r = 0; r < 16; ++r) v[r] = v[r] < 0.f ? 0.f : v[r];  // max(v, 0); NaN stays NaN
                if (pad)
#pragma unroll
                    for (int r = 0; r < 16; ++r) v[r] = out ? 0.f : v[r];
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int flip = (4 * (r >> 2) + ((r & 3) >> 1)) & 7;
                    *reinterpret_cast<float*>(lds + (col ^ (flip * 16)) + (32 * i + 8 * (r >> 2) + (r & 3)) * 128) = v[r];
                }
            }
        }
        __syncthreads();  // T complete and visible to every wave
    }

    if (N1P == 128 || ((g.N2 + 127) / 128 & 1)) g2_second<G, 1>(g, lds, m0, wave, lane);
    else g2_second<G, 2>(g, lds, m0, wave, lane);
}

template <int MODE, int N1P, bool VEC>
__global__ void __launch_bounds__(256, (N1P == 128 ? 3 : 2)) gemm2_kernel(G2Args g)
{
    __shared__ __attribute__((aligned(1024))) char lds[G2Cfg<MODE, N1P, 64>::LDS_BYTES];  // A panels in turn, then T
    const int low = gridDim.x - g.tall, wg = blockIdx.x;
    if (wg < low) g2_block<MODE, N1P, 32, VEC>(g, 64 * g.tall + 32 * wg, lds);
    else g2_block<MODE, N1P, 64, VEC>(g, 64 * (wg - low), lds);
}

namespace {

typedef void (*G2Kernel)(G2Args);

template <int MODE, int N1P>
G2Kernel pick(bool vec)
{
    return vec ? &gemm2_kernel<MODE, N1P, true> : &gemm2_kernel<MODE, N1P, false>;
}

}  // namespace
}  // namespace tg

extern "C" int tgemm_gemm2(int64_t M, int64_t N1, int64_t N2, int64_t K, float alpha, const float* A,
                           int64_t lda, const float* B, int64_t ldb, int act, const float* D, int64_t ldd,
                           float beta, float* E, int64_t lde, int dtype, void* stream)
{
    using namespace tg;
    if (M < 0 || N1 < 0 || N2 < 0 || K < 0) return TGEMM_INVALID_VALUE;
    if (act != TGEMM_ACT_NONE && act != TGEMM_ACT_RELU) return TGEMM_INVALID_VALUE;
    if (dtype != TGEMM_F32 && dtype != TGEMM_F32_BF16X3) return TGEMM_NOT_SUPPORTED;
    if (!(alpha == alpha) || !(beta == beta)) return TGEMM_INVALID_VALUE;
    if (lde < (N2 > 1 ? N2 : 1)) return TGEMM_INVALID_VALUE;
    if (N1 > 256) return TGEMM_NOT_SUPPORTED;
    if (M > INT32_MAX || N2 > INT32_MAX || K > INT32_MAX) return TGEMM_NOT_SUPPORTED;
    if (M == 0 || N2 == 0) return TGEMM_SUCCESS;
    if (!E) return TGEMM_INVALID_VALUE;
    const bool reads = K > 0 && N1 > 0 && alpha != 0.f;
    if (reads) {
        if (!A || !B || !D) return TGEMM_INVALID_VALUE;
        if (lda < K || ldb < N1 || ldd < N2) return TGEMM_INVALID_VALUE;
        // a 64-row block of A within a buffer's 31-bit offsets, a panel of B or D within 32 bits
        if (64 * lda * 4 > INT32_MAX || ldb > kG2RowFloats || ldd > kG2RowFloats) return TGEMM_NOT_SUPPORTED;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    int rc = ensure_device(s);
    if (rc != TGEMM_SUCCESS) return rc;
    if (!reads)  // T = act(0) = 0: E = beta * E
        return launch_scale_c((int)M, (int)N2, beta, E, lde, s) == hipSuccess ? TGEMM_SUCCESS
                                                                              : TGEMM_LAUNCH_FAILED;
    auto al16 = [](const void* p, int64_t ld) { return reinterpret_cast<uintptr_t>(p) % 16 == 0 && ld % 4 == 0; };
    const bool vec = al16(A, lda) && al16(B, ldb) && al16(D, ldd) && K % 4 == 0 && N1 % 4 == 0 && N2 % 4 == 0;
    G2Args g;
    g.B = reinterpret_cast<const char*>(B);
    g.D = reinterpret_cast<const char*>(D);
    g.lda = lda;
    g.ldb = ldb;
    g.ldd = ldd;
    g.lde = lde;
    g.N1 = (int)N1;
    g.N2 = (int)N2;
    g.K = (int)K;
    g.alpha = alpha;
    g.beta = beta;
    g.relu = act == TGEMM_ACT_RELU ? 1 : 0;
    const bool x3 = dtype == TGEMM_F32_BF16X3;
    const bool wide = N1 > 128;
    G2Kernel k = x3 ? (wide ? pick<MODE_X3, 256>(vec) : pick<MODE_X3, 128>(vec))
                    : (wide ? pick<MODE_F32, 256>(vec) : pick<MODE_F32, 128>(vec));
    // whole rounds of 64-row workgroups; what is left as 32-row ones, where these fit
    // one round.  A launch takes at most 2^29 rows: a grid counts threads in 32 bits.
    constexpr int64_t kRows = int64_t(1) << 29;
    static_assert(grid_fits(kRows / 64 + 768, 256), "the workgroups of a launch, 32-row ones among them");
    const int64_t slots = wide ? 512 : 768;
    for (int64_t m = 0; m < M; m += kRows) {
        const int64_t rows = std::min(M - m, kRows), of64 = (rows + 63) / 64, rounds = rows / 64 / slots * slots;
        g.A = reinterpret_cast<const char*>(A + m * lda);
        g.E = E + m * lde;
        g.M = (int)rows;
        g.tall = (int)(of64 - rounds <= slots / 2 ? rounds : of64);
        const int64_t low = rows - 64 * (int64_t)g.tall, blocks = g.tall + (low > 0 ? (low + 31) / 32 : 0);
        hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(256), 0, s, g);
    }
    return hipGetLastError() == hipSuccess ? TGEMM_SUCCESS : TGEMM_LAUNCH_FAILED;
}
