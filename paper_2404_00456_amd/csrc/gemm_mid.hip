// Integer GEMMs on middling grids (about a hundred to a few thousand X rows),
// for gfx950: the same y and acc as the kernels of gemm_w4a4.hip, bit for bit.
//
// Those kernels put 128 x 256 or 256 x 256 tiles on the CUs, which leaves
// half of them idle on outputs of a few million elements, and run one wave
// per SIMD on 128-row int4 and int8 tiles.  Here a block of eight waves
// (2 (m) x 4 (n)) computes a 32 MI x 64 NI tile, from 64 x 64 to 256 x 192,
// picked so that the grid comes out in few, full rounds.  Operands come by
// global -> LDS DMA into a ring as deep as 160 KB of LDS allow (3 to 8
// stages), because the bound is what a CU can bring in: 60 to 80 GB/s per CU
// were measured at every tile and load (about 32 bytes per clock), 16 TB/s
// with all of them busy, and a k-step's reads and MFMAs fit under that.
// Double-buffering the operands in registers across the barrier changed
// nothing (e3m2) or lost 5 to 15% (int4), and W read straight to registers
// with X through LDS lost 5% (e3m2) to 70% (int8, whose 64-byte row pieces
// gather badly).
//
// Measured against the tiled kernels: e3m2 333 x 11008 (K = 4096)
// 28.4 -> 18.7 us, 1024 x 4096 (K = 4096) 24.2 -> 15.6, 517 x 5120
// (K = 13824) 64 -> 37; int4 1777 x 4096 (K = 4096) 51 -> 32.6; int8
// 517 x 5120 (K = 13824) 137 -> 58 us.
#include "gemm_common.hpp"

namespace quarot {
namespace {

using namespace gemm;

constexpr int MID_WAVES = 8;  // 2 (m) x 4 (n)
constexpr int MID_LDS = 160 * 1024;

template <int BITS, int MI, int NI>
struct Mid {
    static constexpr int TM = 32 * MI, TN = 64 * NI, ROWS = TM + TN;
    static constexpr int KB = BITS == 6 ? 96 : 64;  // bytes per row per k-step
    static constexpr int STAGE = ROWS * KB;
    static constexpr int R = MID_LDS / STAGE < 8 ? MID_LDS / STAGE : 8;  // ring stages
    static constexpr int HC = ROWS / 16;                                 // head chunks (1 KB)
    static constexpr int CHUNKS = STAGE / 1024;
    static constexpr int DPW = (CHUNKS + MID_WAVES - 1) / MID_WAVES;  // DMAs per wave and k-step
    static constexpr int LDS = R * STAGE;
};

template <int BITS, int MI, int NI>
__global__ __launch_bounds__(64 * MID_WAVES, 1) void k_gemm_mid(GemmArgs a)
{
    typedef Mid<BITS, MI, NI> C;
    typedef typename std::conditional<BITS == 6, v4f, v4i>::type Acc;
    constexpr int R = C::R, DPW = C::DPW;
    extern __shared__ __align__(16) uint8_t lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int M = a.M, N = a.N, K = a.K;
    const int64_t ldk = BITS == 4 ? K / 2 : K;
    const int KT = BITS == 8 ? K / 64 : K / 128;
    // consecutive tiles, m fastest, on one XCD (block b runs on XCD b % 8)
    const int TMs = (M + C::TM - 1) / C::TM;
    const int nblk = gridDim.x, b = blockIdx.x;
    const int xc = b & 7;
    const int t = xc * (nblk >> 3) + min(xc, nblk & 7) + (b >> 3);
    const int m0 = (t % TMs) * C::TM, n0 = (t / TMs) * C::TN;

    // the scales of this lane's outputs
    const int r16 = lane & 15, g = lane >> 4;
    uint16_t sxh[MI];
    uint16_t swh[NI][4];
#pragma unroll
    for (int j = 0; j < MI; ++j)
        sxh[j] = a.sx[min(m0 + wm * 16 * MI + 16 * j + r16, M - 1)];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            swh[i][r] = a.sw[min(n0 + wn * 16 * NI + 16 * i + 4 * g + r, N - 1)];

    // DMA i of this wave moves chunk wave + 8 i of a stage (a wave past the
    // last chunk moves it again): heads of the X rows, of the W rows, then
    // the tails.
    uint32_t vo[DPW];
    const uint8_t *base[DPW];
    int64_t step[DPW];
    uint32_t dst[DPW];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void *)lds;
#pragma unroll
    for (int i = 0; i < DPW; ++i) {
        const int c = min(wave + MID_WAVES * i, C::CHUNKS - 1);
        const bool head = c < C::HC;
        const int row = head ? 16 * c : 32 * (c - C::HC);
        const bool xop = row < C::TM;
        const int r0 = xop ? row : row - C::TM;
        const int64_t rows = xop ? M : N;
        const int org = xop ? m0 : n0;
        const int lim = (int)rows - org - 1;
        const uint8_t *p = xop ? a.xq : a.wq;
        dst[i] = lds0 + 1024u * (uint32_t)c;
        if constexpr (BITS == 6) {
            step[i] = rows * 96;
            base[i] = head ? p + (int64_t)org * 64 : p + rows * 64 + (int64_t)org * 32;
            vo[i] = head ? (uint32_t)(min(r0 + (lane >> 2), lim) * 64 + (lane & 3) * 16)
                         : (uint32_t)(min(r0 + (lane >> 1), lim) * 32 + (lane & 1) * 16);
        } else {
            step[i] = 64;
            base[i] = p + (int64_t)org * ldk;
            vo[i] = (uint32_t)(min(r0 + (lane >> 2), lim) * (int)ldk +
                               (((lane & 3) ^ ((lane >> 3) & 3)) << 4));
        }
    }
    auto issue = [&](int stage) {
#pragma unroll
        for (int i = 0; i < DPW; ++i) {
            dma16s(vo[i], base[i], dst[i] + stage * C::STAGE);
            base[i] += step[i];
        }
    };

    const int ounit = (g ^ ((r16 >> 1) & 3)) << 4;
    const int brow = (wm * 16 * MI + r16) * 64 + ounit;
    const int arow = (C::TM + wn * 16 * NI + r16) * 64 + ounit;
    constexpr int HEADS = C::ROWS * 64;
    const int toff = 8 * (g ^ ((r16 >> 2) & 3));
    const int btail = HEADS + (wm * 16 * MI + r16) * 32 + toff;
    const int atail = HEADS + (C::TM + wn * 16 * NI + r16) * 32 + toff;

    Acc acc[NI][MI];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j)
            acc[i][j] = Acc{0, 0, 0, 0};

    auto compute = [&](int stage) {
        const uint8_t *sb = lds + stage * C::STAGE;
        if constexpr (BITS == 6) {
            Op6 A[NI], B[MI];
            auto rd = [&](Op6 &o, int head, int tail) {
                o.h = *reinterpret_cast<const uint4 *>(sb + head);
                // volatile: not paired with another slice's tail (see gemm_main)
                const uint64_t tt = *(const volatile lds_u64 *)(lds_void *)(sb + tail);
                o.t = make_uint2((uint32_t)tt, (uint32_t)(tt >> 32));
            };
#pragma unroll
            for (int i = 0; i < NI; ++i)
                rd(A[i], arow + i * 1024, atail + i * 512);
#pragma unroll
            for (int j = 0; j < MI; ++j)
                rd(B[j], brow + j * 1024, btail + j * 512);
#pragma unroll
            for (int j = 0; j < MI; ++j)
#pragma unroll
                for (int i = 0; i < NI; ++i)
                    acc[i][j] = mfma6(A[i], B[j], acc[i][j]);
        } else {
            uint4 A[NI], B[MI];
#pragma unroll
            for (int i = 0; i < NI; ++i)
                A[i] = *reinterpret_cast<const uint4 *>(sb + arow + i * 1024);
#pragma unroll
            for (int j = 0; j < MI; ++j)
                B[j] = *reinterpret_cast<const uint4 *>(sb + brow + j * 1024);
            if constexpr (BITS == 8) {
#pragma unroll
                for (int j = 0; j < MI; ++j)
#pragma unroll
                    for (int i = 0; i < NI; ++i)
                        acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                            __builtin_bit_cast(v4i, A[i]), __builtin_bit_cast(v4i, B[j]),
                            acc[i][j], 0, 0, 0);
            } else {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    v4i aw[NI];
#pragma unroll
                    for (int i = 0; i < NI; ++i)
                        aw[i] = widen(s ? make_uint2(A[i].z, A[i].w) : make_uint2(A[i].x, A[i].y));
#pragma unroll
                    for (int j = 0; j < MI; ++j) {
                        const v4i bw =
                            widen(s ? make_uint2(B[j].z, B[j].w) : make_uint2(B[j].x, B[j].y));
#pragma unroll
                        for (int i = 0; i < NI; ++i)
                            acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(aw[i], bw, acc[i][j],
                                                                              0, 0, 0);
                    }
                }
            }
        }
    };

    // Ring: step k in stage k % R, R - 1 steps in flight.  The barrier of
    // step k comes after every wave's wait for its own DMAs of step k, and
    // after every wave's reads of step k - 1, whose stage the DMAs issued
    // next overwrite.
    for (int s = 0; s < R - 1 && s < KT; ++s)
        issue(s);
    int stage = 0, kt = 0;
    for (; kt + R - 1 < KT; ++kt) {
        __asm__ volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(waitcnt_imm((R - 2) * DPW, 0));
        __builtin_amdgcn_s_barrier();
        __asm__ volatile("" ::: "memory");
        issue(stage == 0 ? R - 1 : stage - 1);
        compute(stage);
        stage = stage == R - 1 ? 0 : stage + 1;
    }
    // the last steps: everything lands, nothing is overwritten any more
    __asm__ volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
    __builtin_amdgcn_s_barrier();
    __asm__ volatile("" ::: "memory");
    for (; kt < KT; ++kt) {
        compute(stage);
        stage = stage == R - 1 ? 0 : stage + 1;
    }

    // lane holds n = 4 g + r (r = 0..3) of m = r16 of each 16 x 16 slice pair
    const bool vec = (N & 3) == 0;
#pragma unroll
    for (int j = 0; j < MI; ++j) {
        const int m = m0 + wm * 16 * MI + 16 * j + r16;
        if (m >= M)
            continue;
        const float sxf = h2f(sxh[j]);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int nb = n0 + wn * 16 * NI + 16 * i + 4 * g;
            int iv[4];
            uint16_t hv[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                iv[r] = BITS == 4 ? (int)acc[i][j][r] >> 8 : (int)acc[i][j][r];
                const float tt = (float)iv[r] * sxf;
                hv[r] = f2h(tt * h2f(swh[i][r]));
            }
            uint16_t *yrow = a.y + (int64_t)m * N;
            int32_t *arw = a.acc ? a.acc + (int64_t)m * N : nullptr;
            if (vec && nb + 3 < N) {
                *reinterpret_cast<uint2 *>(yrow + nb) =
                    make_uint2((uint32_t)hv[0] | ((uint32_t)hv[1] << 16),
                               (uint32_t)hv[2] | ((uint32_t)hv[3] << 16));
                if (arw)
                    *reinterpret_cast<int4 *>(arw + nb) = make_int4(iv[0], iv[1], iv[2], iv[3]);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (nb + r < N) {
                        yrow[nb + r] = hv[r];
                        if (arw)
                            arw[nb + r] = iv[r];
                    }
            }
        }
    }
}

template <int BITS, int MI, int NI>
hipError_t go(const GemmArgs &a, int grid, hipStream_t s)
{
    typedef Mid<BITS, MI, NI> C;
    static_assert(C::R >= 3, "ring depth");
    static_assert(C::TM % 32 == 0 && C::TN % 32 == 0, "DMA chunks of one operand each");
    const void *fn = (const void *)k_gemm_mid<BITS, MI, NI>;
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
    if (e != hipSuccess)
        return e;
    GemmArgs args = a;
    void *params[] = {&args};
    return hipLaunchKernel(fn, dim3((unsigned)grid), dim3(64 * MID_WAVES), params, (size_t)C::LDS,
                           s);
}

template <int BITS>
hipError_t pick(const GemmArgs &a, const PathPlan &p, hipStream_t s)
{
    switch (10 * p.a + p.b) {
    case 21: return go<BITS, 2, 1>(a, p.grid, s);
    case 22: return go<BITS, 2, 2>(a, p.grid, s);
    case 42: return go<BITS, 4, 2>(a, p.grid, s);
    case 43: return go<BITS, 4, 3>(a, p.grid, s);
    case 44: return go<BITS, 4, 4>(a, p.grid, s);
    case 83: return go<BITS, 8, 3>(a, p.grid, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_gemm_mid(const GemmArgs &a, const PathPlan &p, int bits, hipStream_t s)
{
    hipError_t e = bits == 6 ? pick<6>(a, p, s) : bits == 8 ? pick<8>(a, p, s) : pick<4>(a, p, s);
    return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace quarot
