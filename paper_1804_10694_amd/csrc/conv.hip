// Convolution layer as an implicit gemm (the paper's Conv benchmark layer,
// Section VI-A, and the observation there that sgemm is the building block of
// convolutions), for R x R filters (R odd).  The 3 x 3 case is written below;
// for R x R read R*R taps and padding R / 2.  Every kernel exists twice: with
// R = 3 fixed at compile time (the paper credits its Conv result to such
// filter-size specialisation) and with R taken at run time.
//
// Y[n, y, x, co] = alpha * sum_{dy, dx, ci} Xpad[n, y + dy, x + dx, ci] * Wt[dy, dx, ci, co]
//                  + beta * Y[n, y, x, co]
// with X, Y in NHWC, Wt as 3 x 3 x Cin x Cout, stride 1 and zero padding 1.
// As a gemm: M = batch * H * W output pixels, N = Cout, K = 9 * Cin; B = Wt
// read as a K x Cout row-major matrix, C = Y as an M x Cout row-major matrix,
// and A the im2col matrix, which is never materialised: while packing a K
// panel into LDS, each 16-byte unit of A (KU consecutive k of one output
// pixel) is read straight from the input pixel its tap points at, or set to
// zero where the tap falls into the padding.  Cin is a multiple of KU, so a
// unit never straddles two taps and is one vector load of KU channels.
//
// Two kernels share this scheme.  The direct one runs the gemm tile body of
// tile_f32x3.h (register-staged loads, full/partial tiles, fused epilogue).
// The packed one runs the LDS pipeline of tile_packed.h: the filter is packed
// once into K-contiguous rows of B^T (array packing, Section I), and each A
// panel is brought into LDS by 16-byte buffer loads whose per-lane offsets
// point at the input pixels of the lane's unit; units in the padding get an
// offset past the end of the buffer, which reads as zero.  The x3 form first
// splits X into its high and low bf16 parts (same NHWC layout), so both
// operands of every product come from memory as bf16.
#include <hip/hip_runtime.h>

#include <cstring>

#include "../../include/tgemm.h"
#include "kargs.h"
#include "registry.h"
#include "tile_f32x3.h"
#include "tile_packed.h"

namespace tg {

int ensure_device(hipStream_t stream);

// NHWC input geometry and the filter size R (odd; padding R / 2, stride 1).
struct ConvGeom {
    int H, W, C, R;
    int inner = 0;  // x3 in steps of 16 channels: steps per tap and group of channels (0: a tap's all)
};

// Tap t of an R x R filter (row-major over dy, dx) as an offset from the output
// pixel.  FR > 0 fixes R at compile time (divisions by a constant); FR == 0
// takes R from the geometry.
template <int FR>
__device__ __forceinline__ void tap_offset(int tap, const ConvGeom& g, int& dy, int& dx)
{
    const int R = FR > 0 ? FR : g.R;
    const int q = tap / R;
    dy = q - R / 2;
    dx = tap - q * R - R / 2;
}

template <class CF, int FR>
struct ConvPanel : Panel<CF> {
    using Geom = ConvGeom;
    static constexpr int KU = CF::KU, UK = CF::UK, NT = CF::NT;

    // Output pixel of each A unit this thread loads (its row r is fixed across
    // panels): flat index n*H*W + y*W + x (-1 past the last pixel), and y, x.
    int pix[CF::A_PER_T], py[CF::A_PER_T], px[CF::A_PER_T];

    __device__ __forceinline__ void init(const GemmArgs& a, int m0, int t, const Geom& g)
    {
#pragma unroll
        for (int p = 0; p < CF::A_PER_T; ++p) {
            const int m = m0 + (t + p * NT) / UK;
            const bool in = m < a.M;
            const int row = m / g.W;
            pix[p] = in ? m : -1;
            px[p] = m - row * g.W;
            py[p] = row % g.H;
        }
    }

    template <bool PRED>
    __device__ __forceinline__ void load(const GemmArgs& a, int m0, int n0, int k0, int t, const Geom& g)
    {
        const float* X = static_cast<const float*>(a.A);
#pragma unroll
        for (int p = 0; p < CF::A_PER_T; ++p) {
            const int kb = k0 + ((t + p * NT) % UK) * KU;
            typename Panel<CF>::fu v;
#pragma unroll
            for (int e = 0; e < KU; ++e) v[e] = 0.f;
            if (pix[p] >= 0 && kb < a.K) {
                const int tap = kb / g.C, ci = kb - tap * g.C;
                int dy, dx;
                tap_offset<FR>(tap, g, dy, dx);
                const int iy = py[p] + dy, ix = px[p] + dx;
                if (iy >= 0 && iy < g.H && ix >= 0 && ix < g.W) {
                    const float* src = X + (int64_t)(pix[p] + dy * g.W + dx) * g.C + ci;
#pragma unroll
                    for (int c = 0; c < KU / 4; ++c) {
                        const f32x4 q = *reinterpret_cast<const f32x4*>(src + 4 * c);
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[4 * c + e] = q[e];
                    }
                }
            }
            this->ra[p] = v;
        }
        this->template load_b<PRED>(a, n0, k0, t);
    }
};

template <class CF, int FR>
__global__ void __launch_bounds__(CF::NT) conv_kernel(GemmArgs a, ConvGeom g)
{
    __shared__ __attribute__((aligned(16))) char lds[CF::LDS_BYTES];
    const TileCoord tc = map_tile(blockIdx.x, a.tiles_m, a.tiles_n, a.group_m, a.xcd_remap);
    const int m0 = tc.tm * CF::BM, n0 = tc.tn * CF::BN;
    if (m0 + CF::BM <= a.M && n0 + CF::BN <= a.N) tile_body<CF, false, ConvPanel<CF, FR>>(a, m0, n0, lds, g);
    else tile_body<CF, true, ConvPanel<CF, FR>>(a, m0, n0, lds, g);
}

// A panels of the packed kernel, read from the NHWC input (X, or its bf16 hi
// and lo parts for x3) instead of packed rows.  Each lane of load instruction
// i fills the LDS slot that the packed layout assigns to it: row
// ig * (64 / UK) + lane / UK of the tile (ig = wave * A_INSTR + i) and the
// unit u of that row given by the swizzle of tile_packed.h (pk_slot), i.e.
// channels [ci, ci + KU) of tap `tap` for k = panel * BK + u * KU.
template <class CF, int FR>
struct ConvRowsA {
    using Geom = ConvGeom;
    static constexpr int NI = CF::A_INSTR, UK = CF::UK, KU = CF::KU;
    static constexpr int LOADS = CF::NARR * NI;  // loads per wave per panel
    static constexpr int OOB = INT32_MIN;  // offset 2^31: beyond any resource here, reads zero

    // Instructions DS apart load the same unit of their rows (the swizzle of pk_slot
    // repeats), so there are DS positions in k.  Panels are issued in order, so a tap
    // and channel advance by addition: beside waves that keep the matrix core busy each
    // instruction of a division takes about an MFMA's time.  With two divisions per load
    // and panel, 3 x 3 layers f32 32 x 56 x 56 x 256 -> 256 1045 us, now 1000; 32 x 28 x 28
    // x 128 -> 128 109 -> 98; x3 there 58.7 -> 50.9, 8 x 14 x 14 x 512 -> 512 148 -> 127.
    static constexpr int DS = UK <= 4 ? 1 : UK / 4 < NI ? UK / 4 : NI;

    __amdgpu_buffer_rsrc_t r, rl;
    int wave, K, H, W, C, R;
    int k[DS], ci[DS], dy[DS], dx[DS];  // next panel's k, its channel and tap
    uint32_t at[NI];                    // byte of this lane's output pixel
    int py[NI], px[NI];                 // its y (far outside past M) and x

    __device__ __forceinline__ void place(int d)
    {
        const int tap = k[d] / C;
        ci[d] = k[d] - tap * C;
        const int q = tap / R;
        dy[d] = q - R / 2;
        dx[d] = tap - q * R - R / 2;
    }

    __device__ __forceinline__ void init(const PackedArgs& a, int m0, int lane, int wave_, const Geom& g)
    {
        wave = wave_;
        K = a.K;
        H = g.H;
        W = g.W;
        C = g.C;
        R = FR > 0 ? FR : g.R;
        const int bytes = a.M * C * CF::ES;  // below 2^31 (checked on the host)
        r = make_rsrc(a.A, bytes);
        rl = CF::MODE == MODE_X3 ? make_rsrc(a.Alo, bytes) : r;
#pragma unroll
        for (int d = 0; d < DS; ++d) {
            k[d] = (((lane % UK) ^ (4 * (wave * NI + d) + lane / 16)) & (UK - 1)) * KU;
            place(d);
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int m = m0 + (wave * NI + i) * (64 / UK) + lane / UK;
            const int row = m / W;
            px[i] = m - row * W;
            py[i] = m < a.M ? row % H : INT32_MIN / 2;
            at[i] = (uint32_t)m * (uint32_t)(C * CF::ES);
        }
    }

    __device__ __forceinline__ void issue(int, char* stage)
    {
        uint32_t off[DS];
#pragma unroll
        for (int d = 0; d < DS; ++d) off[d] = ((uint32_t)(dy[d] * W + dx[d]) * (uint32_t)C + ci[d]) * CF::ES;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int ig = wave * NI + i, d = i % DS;
            const bool in = k[d] < K && (unsigned)(py[i] + dy[d]) < (unsigned)H &&
                            (unsigned)(px[i] + dx[d]) < (unsigned)W;
            const int voff = in ? (int)(at[i] + off[d]) : OOB;
            auto* dst = (__attribute__((address_space(3))) void*)(stage + ig * 64 * 16);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, voff, 0, 0, 0);
            if (CF::MODE == MODE_X3) {
                auto* dlo = (__attribute__((address_space(3))) void*)(stage + CF::LDS_A + ig * 64 * 16);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rl, dlo, 16, voff, 0, 0, 0);
            }
        }
#pragma unroll
        for (int d = 0; d < DS; ++d) {
            k[d] += CF::BK;
            if (C < CF::BK) {  // a panel is more than one tap further
                place(d);
                continue;
            }
            ci[d] += CF::BK;
            const bool wrap = ci[d] >= C;
            ci[d] -= wrap ? C : 0;
            dx[d] += wrap;
            const bool line = dx[d] > R / 2;
            dy[d] += line;
            dx[d] -= line ? R : 0;
        }
    }
};

// A steps of the kernel that takes turns (TCfg, x3): X split beforehand into
// units of eight channels' high parts, then their low parts, so the four units
// of a pixel's step are one run of 64 bytes (within a tap).  Unit u of a row
// is channels 8 (u % 2) .. of the step, high (u < 2) or low.  Steps are issued
// in order, so the tap and channel advance by addition; a division per unit and
// step would take longer than the slot its issue has.
template <class CF, int FR>
struct ConvStepsA {
    using Geom = ConvGeom;
    using SP = StepPack<CF::MODE>;
    static constexpr int NI = CF::BM * SP::UK / 64 / CF::NW;
    static constexpr int LOADS = NI;
    static constexpr uint32_t OOB = 0xfffffff0u;  // at or past the end of any X here (below 2^32 - 31 bytes)

    __amdgpu_buffer_rsrc_t r;
    int wave, H, W, C, half, inner, part;
    int taps;                        // taps left from the current one on (0: past K); inner: steps
    int ci, dy, dx;                  // channel and tap of k
    uint32_t at[NI];                 // byte offset of (output pixel, channel 0), the unit's array added
    int py[NI], px[NI];              // output pixel's y (far outside past M) and x

    __device__ __forceinline__ void init(const PackedArgs& a, int m0, int lane, int wave_, const Geom& g)
    {
        static_assert(CF::MODE == MODE_X3 && CF::BK == 16, "steps of two units of eight channels");
        wave = wave_;
        H = g.H;
        W = g.W;
        C = g.C;
        const int R = FR > 0 ? FR : g.R;
        half = R / 2;
        r = make_rsrc(a.A, (int)((uint32_t)a.M * (uint32_t)C * 4u));
        // the lane's unit is the same in every instruction: 16 rows further the
        // swizzle of pk_slot repeats
        const int u = ((lane % SP::UK) ^ (lane / 16)) & (SP::UK - 1);
        const int first = 8 * (u & 1);
        const int tap = first / C;  // C is 8 or more
        ci = first - tap * C;
        dy = -half + tap / R;
        dx = -half + tap % R;
        inner = g.inner;
        part = 0;
        taps = inner ? R * R * (C / 16) : R * R - tap;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int m = m0 + (wave * NI + i) * (64 / SP::UK) + lane / SP::UK;
            const int row = m / W;
            px[i] = m - row * W;
            py[i] = m < a.M ? row % H : INT32_MIN / 2;
            at[i] = (uint32_t)m * (uint32_t)C * 4u + (u >> 1) * 16;
        }
    }

    __device__ __forceinline__ void issue(int, char* stage)
    {
        const uint32_t off = (uint32_t)((dy * W + dx) * C + ci) * 4u;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int iy = py[i] + dy, ix = px[i] + dx;
            const bool in = taps > 0 && iy >= 0 && iy < H && ix >= 0 && ix < W;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                r, (__attribute__((address_space(3))) void*)(stage + (wave * NI + i) * 1024), 16,
                (int)(in ? at[i] + off : OOB), 0, 0, 0);
        }
        if (inner) {
            --taps;
            ci += 16;
            if (++part < inner) return;
            part = 0;
            const bool line = ++dx > half;
            dx = line ? -half : dx;
            dy += line;
            const bool all = dy > half;
            dy = all ? -half : dy;
            ci -= all ? 0 : 16 * inner;
            return;
        }
        ci += 16;
#pragma unroll
        for (int w = 0; w < 2; ++w) {  // 16 channels on are two taps at most
            const bool wrap = ci >= C;
            ci -= wrap ? C : 0;
            dx += wrap;
            taps -= wrap;
            const bool line = dx > half;
            dy += line;
            dx = line ? -half : dx;
        }
    }
};

// Eight channels at a time: 32 bytes of X into 16 bytes of high and 16 of low
// parts.
__global__ void __launch_bounds__(256) conv_split_kernel(const float* X, char* out, int64_t groups)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < groups; i += (int64_t)gridDim.x * blockDim.x) {
        const f32x4 v0 = *reinterpret_cast<const f32x4*>(X + 8 * i), v1 = *reinterpret_cast<const f32x4*>(X + 8 * i + 4);
        const float x[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
        bf16x8 h, l;
        split_bf16x8(x, h, l);
        *reinterpret_cast<bf16x8*>(out + 32 * i) = h;
        *reinterpret_cast<bf16x8*>(out + 32 * i + 16) = l;
    }
}

// The filter in steps of 16 channels of one tap, taps inside (ConvGeom::inner): step
// s of column n is part s % inner of (channel group) * taps + tap = s / inner, in units as
// StepPack has them.  A block has 256 columns of one step.
__global__ void __launch_bounds__(256) conv_filter_kernel(const float* Wt, int C, int N, int taps, int inner, char* P,
                                                         int Kp, int Np)
{
    using SP = StepPack<MODE_X3>;
    const int blocks = Np / 256, s = blockIdx.x / blocks, n = (blockIdx.x - s * blocks) * 256 + threadIdx.x;
    const int group = s / (taps * inner), rest = s - group * taps * inner;
    const int tap = rest / inner, c0 = group * inner + rest - tap * inner;
    char* dst = P + ((int64_t)(n / SP::ROWS) * (Kp / SP::HK) + s) * SP::CHUNK;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            x[e] = n < N ? Wt[((int64_t)tap * C + 16 * c0 + 8 * g + e) * N + n] : 0.f;
        bf16x8 h, l;
        split_bf16x8(x, h, l);
        *reinterpret_cast<bf16x8*>(dst + pk_slot<SP::UK>(n % SP::ROWS, g) * 16) = h;
        *reinterpret_cast<bf16x8*>(dst + pk_slot<SP::UK>(n % SP::ROWS, 2 + g) * 16) = l;
    }
}

template <class CF, int FR>
__global__ void __launch_bounds__(CF::NT, CF::WAVES_PER_EU) conv_turns_kernel(PackedArgs a, ConvGeom g)
{
    static_assert(kPackK % CF::BK == 0 && kPackRows % CF::BN == 0, "panels and tiles divide the packing padding");
    __shared__ __attribute__((aligned(1024))) char lds[CF::LDS_BYTES];
    const TileCoord tc = map_tile(blockIdx.x, a.tiles_m, a.tiles_n, a.group_m, a.xcd_remap);
    packed_tile<CF, ConvStepsA<CF, FR>>(a, tc.tm * CF::BM, tc.tn * CF::BN, lds, g);
}

template <class CF, int FR>
__global__ void __launch_bounds__(CF::NT, CF::WAVES_PER_EU) conv_packed_kernel(PackedArgs a, ConvGeom g)
{
    static_assert(kPackK % CF::BK == 0 && kPackRows % CF::BN == 0, "panels and tiles divide the packing padding");
    __shared__ __attribute__((aligned(1024))) char lds[CF::LDS_BYTES];
    const TileCoord tc = map_tile(blockIdx.x, a.tiles_m, a.tiles_n, a.group_m, a.xcd_remap);
    packed_tile<CF, ConvRowsA<CF, FR>>(a, tc.tm * CF::BM, tc.tn * CF::BN, lds, g);
}

namespace {

// Every kernel exists twice: specialised for 3 x 3 filters (FR = 3) and for a
// filter size given at run time (FR = 0).
struct ConvPacked {
    int dtype, mode, BM, BN, BK, NS, threads;
    void (*kernel[2])(PackedArgs, ConvGeom);  // [0]: 3 x 3, [1]: any R
    bool turns = false;                       // TCfg: step-packed filter, X split unit by unit
};

#define TG_CONVP(DT, MODE, BM, BN, BK, WGM, WGN, NS)                         \
    {DT, MODE, BM, BN, BK, NS, PCfg<MODE, BM, BN, BK, WGM, WGN, NS>::NT,    \
     {&conv_packed_kernel<PCfg<MODE, BM, BN, BK, WGM, WGN, NS>, 3>,         \
      &conv_packed_kernel<PCfg<MODE, BM, BN, BK, WGM, WGN, NS>, 0>}}

// Tile shapes of the packed kernel.  Default (measured over 3x3 layers of
// 64 to 512 channels and 14 x 14 to 112 x 112 pixels): f32 takes shape 0
// (four workgroups per CU) everywhere; x3 takes shape 1 (256 x 256, eight
// waves) when Cout >= 256 and the layer has at least one 256 x 256 tile per
// CU, shape 0 otherwise.
const ConvPacked kConvPacked[] = {
    TG_CONVP(TGEMM_F32, MODE_F32, 128, 128, 16, 2, 2, 2),
    TG_CONVP(TGEMM_F32, MODE_F32, 128, 128, 16, 2, 2, 4),
    TG_CONVP(TGEMM_F32, MODE_F32, 256, 256, 32, 2, 4, 2),
    TG_CONVP(TGEMM_F32, MODE_F32, 256, 128, 32, 2, 4, 3),
    TG_CONVP(TGEMM_F32_BF16X3, MODE_X3, 128, 128, 32, 2, 2, 2),
    {TGEMM_F32_BF16X3, MODE_X3, 256, 256, 32, 2, TCfg<MODE_X3, 256, 256, 2, 4, 4>::NT,
     {&conv_turns_kernel<TCfg<MODE_X3, 256, 256, 2, 4, 4>, 3>, &conv_turns_kernel<TCfg<MODE_X3, 256, 256, 2, 4, 4>, 0>},
     true},
    TG_CONVP(TGEMM_F32_BF16X3, MODE_X3, 256, 128, 32, 2, 4, 3),
    TG_CONVP(TGEMM_F32_BF16X3, MODE_X3, 128, 128, 16, 2, 2, 2),
};

// f32 layers of fewer than 128 tiles of 128 x 128 leave half of the CUs idle in the
// packed kernel.  Time of the direct one on 64 x 64 tiles against it, 18 layers of 2 to
// 124 tiles: 1 x 1 filters 0.47 to 0.78, 3 x 3 0.49 to 0.79, 5 x 5 0.55 to 0.83, 7 x 7
// 0.56 to 0.83 (52 tiles, 8 x 14 x 14 x 512 -> 512, 3 x 3 192 us / 351; 124, 10 x 28 x 28 x
// 256 -> 256, 136 / 180), and the same with filters off 16-byte alignment.  Past the line,
// 148 tiles: 0.81, 0.97, 1.06, 1.08; 196: 0.86, 1.19, 1.36, 1.39.  x3 gains less than the
// 8% it loses elsewhere (126 / 136, 71 / 67).
bool conv_few_tiles(int dtype, int64_t M, int64_t Cout)
{
    return dtype == TGEMM_F32 && Cout % 4 == 0 && ((M + 127) / 128) * ((Cout + 127) / 128) < 128;
}

int conv_default_shape(int dtype, int64_t M, int64_t Cout)
{
    if (dtype != TGEMM_F32_BF16X3) return 0;
    return Cout >= 256 && ((M + 255) / 256) * ((Cout + 255) / 256) >= 256 ? 1 : 0;
}

const ConvPacked* conv_packed(int dtype, int i)
{
    for (const ConvPacked& c : kConvPacked)
        if (c.dtype == dtype && i-- == 0) return &c;
    return nullptr;
}

struct ConvSched {
    int dtype, BM, BN, vec, threads;
    void (*kernel[2])(GemmArgs, ConvGeom);  // [0]: 3 x 3, [1]: any R
};

#define TG_CONV(DT, MODE, BM, BN, BK, VEC)                                      \
    {DT, BM, BN, VEC, Cfg<MODE, BM, BN, BK, 2, 2, VEC>::NT,                    \
     {&conv_kernel<Cfg<MODE, BM, BN, BK, 2, 2, VEC>, 3>, &conv_kernel<Cfg<MODE, BM, BN, BK, 2, 2, VEC>, 0>}}

// 128 x 128 tiles for layers with enough output pixels, 64 x 64 otherwise;
// 16-byte filter loads when Cout and the filter's address allow them.
const ConvSched kConv[] = {
    TG_CONV(TGEMM_F32, MODE_F32, 128, 128, 32, 4),        TG_CONV(TGEMM_F32, MODE_F32, 128, 128, 32, 1),
    TG_CONV(TGEMM_F32, MODE_F32, 64, 64, 16, 4),          TG_CONV(TGEMM_F32, MODE_F32, 64, 64, 16, 1),
    TG_CONV(TGEMM_F32_BF16X3, MODE_X3, 128, 128, 32, 4),  TG_CONV(TGEMM_F32_BF16X3, MODE_X3, 128, 128, 32, 1),
    TG_CONV(TGEMM_F32_BF16X3, MODE_X3, 64, 64, 32, 4),    TG_CONV(TGEMM_F32_BF16X3, MODE_X3, 64, 64, 32, 1),
};

}  // namespace

}  // namespace tg

namespace tg {
namespace {

// Kernel variant: 0 = specialised for 3 x 3, 1 = filter size at run time.
int variant(const ConvGeom& g, bool runtime_r) { return (g.R == 3 && !runtime_r) ? 0 : 1; }

int conv_direct(int64_t M, int64_t Cout, int64_t K, float alpha, const float* X, const float* Wt, float beta,
                float* Y, int dtype, const ConvGeom& g, bool runtime_r, hipStream_t s)
{
    const bool vec = (Cout % 4 == 0) && reinterpret_cast<uintptr_t>(Wt) % 16 == 0;
    const int tile = ((M + 127) / 128) * ((Cout + 127) / 128) >= 192 ? 128 : 64;
    const ConvSched* pick = nullptr;
    for (const ConvSched& c : kConv)
        if (c.dtype == dtype && c.BM == tile && c.vec == (vec ? 4 : 1)) pick = &c;
    if (!pick) return TGEMM_INTERNAL;

    GemmArgs a;
    std::memset(&a, 0, sizeof(a));
    a.A = X;
    a.B = Wt;
    a.C = Y;
    a.lda = K;
    a.ldb = Cout;
    a.ldc = Cout;
    a.M = (int)M;
    a.N = (int)Cout;
    a.K = (int)K;
    a.alpha = alpha;
    a.beta = beta;
    a.tiles_m = (int)((M + pick->BM - 1) / pick->BM);
    a.tiles_n = (int)((Cout + pick->BN - 1) / pick->BN);
    a.group_m = 8;
    a.xcd_remap = 1;
    if (!grid_fits((int64_t)a.tiles_m * a.tiles_n, pick->threads)) return TGEMM_NOT_SUPPORTED;
    hipLaunchKernelGGL(pick->kernel[variant(g, runtime_r)], dim3((unsigned)(a.tiles_m * a.tiles_n)),
                       dim3(pick->threads), 0, s, a, g);
    return hipGetLastError() == hipSuccess ? TGEMM_SUCCESS : TGEMM_LAUNCH_FAILED;
}

// Whether the packed kernel can address the problem: X (or each bf16 part)
// and a 256-row block of packed filter rows must span fewer than 2^31 bytes.
bool conv_packed_ok(int64_t M, int64_t Cin, int64_t K, int dtype)
{
    const int64_t es = dtype == TGEMM_F32 ? 4 : 2;
    return M * Cin * es <= INT32_MAX && packed_k_ok(K, dtype);
}

int conv_packed_run(const ConvPacked& p, int64_t M, int64_t Cin, int64_t Cout, int64_t K, float alpha,
                    const float* X, const float* Wt, float beta, float* Y, const ConvGeom& g, bool runtime_r,
                    hipStream_t s)
{
    const int64_t Np = (Cout + kPackRows - 1) / kPackRows * kPackRows;
    const int64_t Kp = (K + kPackK - 1) / kPackK * kPackK;
    const bool x3 = p.mode == MODE_X3;
    const int64_t es = x3 ? 2 : 4, arrays = x3 ? 2 : 1;
    const int64_t wbytes = Np * Kp * es * arrays, xbytes = x3 ? 2 * M * Cin * es : 0;
    void* ws = nullptr;
    int rc = packed_workspace(s, (size_t)(wbytes + xbytes), &ws);
    if (rc != TGEMM_SUCCESS) return rc;
    char* Bp = static_cast<char*>(ws);
    char* Blo = x3 ? Bp + Np * Kp * es : nullptr;
    char* Ah = x3 ? Bp + wbytes : nullptr;
    char* Al = x3 ? Ah + M * Cin * es : nullptr;
    ConvGeom geom = g;
    if (p.turns) {
        // k in the order (64, 32 or 16 channels, tap, channel): a tile's nine reads of a pixel
        // come within a few steps, while its line is in the XCD's L2; tap by tap over all
        // channels they are C / 16 steps apart (8 MB of X per XCD at 256) and come from the
        // Infinity Cache, whose 28 bytes/ns per CU are about what the matrix cores ask of X.
        // 3 x 3, 32 x 56 x 56 x 256 -> 256 377 us -> 359, 16 x 112 x 112 x 128 -> 256 385 -> 367,
        // 32 x 28 x 28 x 512 -> 1024 612 -> 583; 16 channels at a time 366, 372, 591.
        geom.inner = Cin % 64 == 0 ? 4 : Cin % 32 == 0 ? 2 : Cin % 16 == 0 ? 1 : 0;
        if (geom.inner) {
            hipLaunchKernelGGL(conv_filter_kernel, dim3((unsigned)(Np / 256 * (K / 16))), dim3(256), 0, s, Wt,
                               (int)Cin, (int)Cout, g.R * g.R, geom.inner, Bp, (int)Kp, (int)Np);
        } else {
            rc = launch_step_cols(p.mode, Wt, Cout, K, Cout, Bp, Np, Kp, s);
            if (rc != TGEMM_SUCCESS) return rc;
        }
        const int64_t groups = M * Cin / 8;
        hipLaunchKernelGGL(conv_split_kernel, dim3((unsigned)std::min<int64_t>((groups + 255) / 256, 65536)), dim3(256),
                           0, s, X, Ah, groups);
    } else {
        rc = launch_pack_cols(p.mode, Wt, Cout, K, Cout, Bp, Blo, Np, Kp, s);
        if (rc == TGEMM_SUCCESS && x3) rc = launch_pack_rows(MODE_X3, X, Cin, M, Cin, Ah, Al, M, Cin, s);
        if (rc != TGEMM_SUCCESS) return rc;
    }

    PackedArgs a;
    std::memset(&a, 0, sizeof(a));
    a.A = x3 ? Ah : reinterpret_cast<const char*>(X);
    a.Alo = Al;
    a.B = Bp;
    a.Blo = Blo;
    a.C = Y;
    a.ldc = Cout;
    a.M = (int)M;
    a.N = (int)Cout;
    a.K = (int)K;
    a.Kp = (int)Kp;
    a.alpha = alpha;
    a.beta = beta;
    a.tiles_m = (int)((M + p.BM - 1) / p.BM);
    a.tiles_n = (int)((Cout + p.BN - 1) / p.BN);
    a.group_m = 8;
    a.xcd_remap = 1;
    if (!grid_fits((int64_t)a.tiles_m * a.tiles_n, p.threads)) return TGEMM_NOT_SUPPORTED;
    hipLaunchKernelGGL(p.kernel[variant(g, runtime_r)], dim3((unsigned)(a.tiles_m * a.tiles_n)),
                       dim3(p.threads), 0, s, a, geom);
    return hipGetLastError() == hipSuccess ? TGEMM_SUCCESS : TGEMM_LAUNCH_FAILED;
}

int conv_run(int64_t batch, int64_t H, int64_t W, int64_t Cin, int64_t Cout, int64_t R, float alpha,
             const float* X, const float* Wt, float beta, float* Y, int dtype, int path, void* stream)
{
    if (batch < 0 || H < 0 || W < 0 || Cin < 0 || Cout < 0) return TGEMM_INVALID_VALUE;
    if (R < 1 || R % 2 == 0 || R > 31) return TGEMM_INVALID_VALUE;
    if (dtype != TGEMM_F32 && dtype != TGEMM_F32_BF16X3) return TGEMM_NOT_SUPPORTED;
    const bool runtime_r = (path & TGEMM_CONV_RUNTIME_R) != 0;
    path &= ~TGEMM_CONV_RUNTIME_R;
    const ConvPacked* packed = nullptr;
    if (path >= TGEMM_CONV_PACKED) {
        packed = conv_packed(dtype, path - TGEMM_CONV_PACKED);
        if (!packed) return TGEMM_INVALID_VALUE;
    } else if (path != TGEMM_CONV_AUTO && path != TGEMM_CONV_DIRECT) {
        return TGEMM_INVALID_VALUE;
    }
    // the kernels index pixels, k and columns with 32-bit integers
    if (batch > INT32_MAX || H > INT32_MAX || W > INT32_MAX || Cin > INT32_MAX / (R * R) || Cout > INT32_MAX)
        return TGEMM_NOT_SUPPORTED;
    const int64_t HW = H * W;
    if (HW > INT32_MAX || (HW > 0 && batch > INT32_MAX / HW)) return TGEMM_NOT_SUPPORTED;
    const int64_t M = batch * HW, K = R * R * Cin;
    if (M == 0 || Cout == 0) return TGEMM_SUCCESS;
    if (!Y) return TGEMM_INVALID_VALUE;
    const bool reads_xw = K > 0 && alpha != 0.f;
    if (reads_xw && (!X || !Wt)) return TGEMM_INVALID_VALUE;
    // a 16-byte unit of A is KU channels of one input pixel
    const int ku = dtype == TGEMM_F32 ? 4 : 8;
    if (reads_xw && (Cin % ku != 0 || reinterpret_cast<uintptr_t>(X) % 16 != 0)) return TGEMM_NOT_SUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    int rc = ensure_device(s);
    if (rc != TGEMM_SUCCESS) return rc;
    if (!reads_xw)
        return launch_scale_c((int)M, (int)Cout, beta, Y, Cout, s) == hipSuccess ? TGEMM_SUCCESS
                                                                                 : TGEMM_LAUNCH_FAILED;
    const ConvGeom g{(int)H, (int)W, (int)Cin, (int)R};
    const bool packed_ok = conv_packed_ok(M, Cin, K, dtype);
    if (packed && !packed_ok) return TGEMM_NOT_SUPPORTED;
    if (path == TGEMM_CONV_AUTO && packed_ok && !conv_few_tiles(dtype, M, Cout))
        packed = conv_packed(dtype, conv_default_shape(dtype, M, Cout));
    if (packed) {
        rc = conv_packed_run(*packed, M, Cin, Cout, K, alpha, X, Wt, beta, Y, g, runtime_r, s);
        // under capture with no workspace yet: the direct kernel needs none
        if (!(rc == TGEMM_CAPTURE_UNPLANNED && path == TGEMM_CONV_AUTO)) return rc;
    }
    return conv_direct(M, Cout, K, alpha, X, Wt, beta, Y, dtype, g, runtime_r, s);
}

}  // namespace
}  // namespace tg

extern "C" int tgemm_conv3x3(int64_t batch, int64_t H, int64_t W, int64_t Cin, int64_t Cout, float alpha,
                             const float* X, const float* Wt, float beta, float* Y, int dtype, void* stream)
{
    return tg::conv_run(batch, H, W, Cin, Cout, 3, alpha, X, Wt, beta, Y, dtype, TGEMM_CONV_AUTO, stream);
}

extern "C" int tgemm_conv3x3_path(int64_t batch, int64_t H, int64_t W, int64_t Cin, int64_t Cout, float alpha,
                                  const float* X, const float* Wt, float beta, float* Y, int dtype, int path,
                                  void* stream)
{
    return tg::conv_run(batch, H, W, Cin, Cout, 3, alpha, X, Wt, beta, Y, dtype, path, stream);
}

extern "C" int tgemm_conv2d(int64_t batch, int64_t H, int64_t W, int64_t Cin, int64_t Cout, int64_t R, float alpha,
                            const float* X, const float* Wt, float beta, float* Y, int dtype, int path,
                            void* stream)
{
    return tg::conv_run(batch, H, W, Cin, Cout, R, alpha, X, Wt, beta, Y, dtype, path, stream);
}

extern "C" int tgemm_conv3x3_packed_shape(int dtype, int i, int* bm, int* bn, int* bk, int* stages)
{
    const tg::ConvPacked* p = i >= 0 ? tg::conv_packed(dtype, i) : nullptr;
    if (!p) return TGEMM_INVALID_VALUE;
    if (bm) *bm = p->BM;
    if (bn) *bn = p->BN;
    if (bk) *bk = p->BK;
    if (stages) *stages = p->NS;
    return TGEMM_SUCCESS;
}
