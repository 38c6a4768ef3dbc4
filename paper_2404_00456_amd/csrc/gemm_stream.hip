// Integer GEMMs with few X rows (decoding steps, short prompts), for gfx950:
// the same y and acc as the tiled kernels of gemm_w4a4.hip, bit for bit.
//
// With M rows of X the product reads N * K weight codes for 2 M N K
// operations: up to a few hundred rows that is less matrix time than the
// weights take from HBM, so W goes straight from memory to registers, each
// code read once per 16 MT rows, and no LDS ring stands in between.  The
// tiled kernels put one block on a 256 x 256 tile, which for N = 4096 is 16
// of 256 CUs, and spend a whole tile's MFMAs on rows that are not there.
//
// A block computes 16 MT rows by 16 NT columns over the whole of K: its WV
// waves take runs of U consecutive k-steps in turn, hold the block's tile as
// NT x MT accumulators each and meet in LDS at the end.  The partial sums
// are integers (below 2^24 where they are binary32), so their order does not
// matter.  Splitting K inside the block instead of across blocks needs no
// workspace and gives N / (16 NT) blocks of WV waves, which is what fills
// the chip when M is one tile.
//
// Measured against the tiled kernels (e3m2 codes, graph replays over three
// sets of operands, same process):
//   1 x 4096, K = 4096        27.9 ->  3.7 us
//   16 x 28672, K = 8192      51.6 -> 31.8 us (176 MB of W: 5.5 TB/s)
//   16 x 8192, K = 28672     161.6 -> 29.9 us (5.9 TB/s)
//   61 x 8192, K = 28672     163.3 -> 41.6 us
// and 256 x 4096, K = 11008: e3m2 46.4 -> 15.7, int4 117 -> 23, int8
// 112 -> 41.5 us.  Up to 16 rows the bound is the read of W; beyond, each
// block's re-read of its X rows (N / (16 NT) times X in all, from the L2).
#include "gemm_common.hpp"
#include "gemm_plan.hpp"

namespace quarot {
namespace {

using namespace gemm;

// One operand slice (16 rows x one k-step) of a lane.
template <int BITS>
struct Slice {
    uint4 h;
};
template <>
struct Slice<6> {
    uint4 h;
    uint2 t;
};

template <int BITS>
struct StreamAcc {
    typedef v4i type;
};
template <>
struct StreamAcc<6> {
    typedef v4f type;
};

// Reads as buffer loads, a wave-uniform base (in the descriptor) and a 32-bit
// lane offset: with plain pointers the compiler carries 64-bit lane
// addresses per slice through the loop and spills them.  Offsets at or past
// `size` read nothing and return 0.
typedef __amdgpu_buffer_rsrc_t Rsrc;
typedef uint32_t u4v __attribute__((ext_vector_type(4)));
typedef uint32_t u2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ Rsrc rsrc(const uint8_t *p, int size)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p), 0, size, 0x00027000);
}
__device__ __forceinline__ uint4 ld16(Rsrc r, uint32_t off)
{
    const u4v v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
    return make_uint4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ uint2 ld8(Rsrc r, uint32_t off)
{
    const u2v v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
    return make_uint2(v[0], v[1]);
}

// LDS pitch of a tile row (one m, 16 n): 16-byte writes of 8 consecutive
// rows at 80 bytes hit distinct banks.
constexpr int RED_PITCH = 20;
constexpr int RED_TILE = 16 * RED_PITCH;  // dwords per 16 x 16 tile

template <int BITS, int MT, int NT, int WV, int U>
__global__ __launch_bounds__(64 * WV) void k_gemm_stream(GemmArgs a)
{
    typedef typename StreamAcc<BITS>::type Acc;
    typedef Slice<BITS> Sl;
    extern __shared__ __align__(16) uint32_t red[];  // [WV][NT * MT][RED_TILE]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.M, N = a.N, K = a.K;
    const int TM = (M + 16 * MT - 1) / (16 * MT);
    // consecutive tiles, m fastest, on one XCD (block b runs on XCD b % 8),
    // so that the m-tiles of a column share its W in one L2
    const int nblk = gridDim.x, b = blockIdx.x;
    const int x = b & 7, per = nblk >> 3, extra = nblk & 7;
    const int t = x * per + min(x, extra) + (b >> 3);
    const int m0 = (t % TM) * 16 * MT, n0 = (t / TM) * 16 * NT;

    constexpr int KSTEP = BITS == 8 ? 64 : 128;
    const int KT = K / KSTEP;
    const int r16 = lane & 15, g = lane >> 4;

    // Lane offsets of a slice within a k-step.  e3m2 (tiled layout): unit g
    // of its row; 4- and 8-bit codes (row-major): the 16-byte unit g of the
    // row's 64 bytes.  Rows past the edge read the last row instead.
    uint32_t xo[MT], wo[NT];
    auto row_off = [&](int row) -> uint32_t {
        if constexpr (BITS == 6)
            return (uint32_t)row * 64u + 16u * (uint32_t)(g ^ ((row >> 1) & 3));
        else
            return (uint32_t)row * (uint32_t)(BITS == 4 ? K / 2 : K) + 16u * (uint32_t)g;
    };
    auto tail_off = [&](int row) -> uint32_t {
        return (uint32_t)row * 32u + 8u * (uint32_t)(g ^ ((row >> 2) & 3));
    };
    // (tiles start at multiples of 16 rows, so the swizzles see the row's
    // place in the tile)
    uint32_t xt[MT], wt[NT];
#pragma unroll
    for (int j = 0; j < MT; ++j) {
        const int r = min(m0 + 16 * j + r16, M - 1) - m0;
        xo[j] = row_off(r);
        xt[j] = tail_off(r);
    }
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        const int r = min(n0 + 16 * i + r16, N - 1) - n0;
        wo[i] = row_off(r);
        wt[i] = tail_off(r);
    }
    // bytes from one k-step to the next, and the tile's first byte
    const int64_t xstep = BITS == 6 ? (int64_t)M * 96 : 64;
    const int64_t wstep = BITS == 6 ? (int64_t)N * 96 : 64;
    const int64_t pitch = BITS == 4 ? K / 2 : K;
    const uint8_t *xb = a.xq + (BITS == 6 ? (int64_t)m0 * 64 : m0 * pitch);
    const uint8_t *wb = a.wq + (BITS == 6 ? (int64_t)n0 * 64 : n0 * pitch);
    const int64_t xtail = (int64_t)M * 64 - (int64_t)m0 * 32;  // from a step's heads to its tails
    const int64_t wtail = (int64_t)N * 64 - (int64_t)n0 * 32;

    auto load = [&](Sl (&xs)[MT], Sl (&ws)[NT], int kt) {
        // k-steps past the last read nothing and come back as zeros
        const int size = kt < KT ? 0x7FFFFFFF : 0;
        const uint8_t *wp = wb + kt * wstep, *xp = xb + kt * xstep;
        const Rsrc wh = rsrc(wp, size), xh = rsrc(xp, size);
        const Rsrc wq = rsrc(wp + wtail, size), xq = rsrc(xp + xtail, size);
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            ws[i].h = ld16(wh, wo[i]);
            if constexpr (BITS == 6)
                ws[i].t = ld8(wq, wt[i]);
        }
#pragma unroll
        for (int j = 0; j < MT; ++j) {
            xs[j].h = ld16(xh, xo[j]);
            if constexpr (BITS == 6)
                xs[j].t = ld8(xq, xt[j]);
        }
    };

    Acc acc[NT][MT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
            acc[i][j] = Acc{0, 0, 0, 0};

    auto mac = [&](const Sl (&xs)[MT], const Sl (&ws)[NT]) {
        if constexpr (BITS == 6) {
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = 0; j < MT; ++j)
                    acc[i][j] = mfma6(Op6{ws[i].h, ws[i].t}, Op6{xs[j].h, xs[j].t}, acc[i][j]);
        } else if constexpr (BITS == 8) {
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = 0; j < MT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                        __builtin_bit_cast(v4i, ws[i].h), __builtin_bit_cast(v4i, xs[j].h),
                        acc[i][j], 0, 0, 0);
        } else {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                v4i xw[MT];
#pragma unroll
                for (int j = 0; j < MT; ++j)
                    xw[j] = widen(s ? make_uint2(xs[j].h.z, xs[j].h.w)
                                    : make_uint2(xs[j].h.x, xs[j].h.y));
#pragma unroll
                for (int i = 0; i < NT; ++i) {
                    const v4i ww = widen(s ? make_uint2(ws[i].h.z, ws[i].h.w)
                                           : make_uint2(ws[i].h.x, ws[i].h.y));
#pragma unroll
                    for (int j = 0; j < MT; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ww, xw[j], acc[i][j], 0,
                                                                          0, 0);
                }
            }
        }
    };

    // this thread's outputs: one column n, every 64 WV / (16 NT)-th row
    constexpr int COLS = 16 * NT, ROWS = 16 * MT;
    constexpr int RSTEP = 64 * WV / COLS;
    constexpr int PER = (ROWS + RSTEP - 1) / RSTEP;
    const int on = n0 + tid % COLS, om = tid / COLS;
    uint16_t swh = a.sw[min(on, N - 1)], sxh[PER];
#pragma unroll
    for (int p = 0; p < PER; ++p)
        sxh[p] = a.sx[min(m0 + om + p * RSTEP, M - 1)];

    // Runs of U k-steps, double buffered in registers: the next run's loads
    // are issued before this run's MFMAs (the fences keep them there), in
    // straight-line code so that the waits can count them.  Every wave makes the same number of runs; k-steps
    // past the last are zeros.
    Sl xs[2][U][MT], ws[2][U][NT];
    auto load_run = [&](int buf, int k0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            load(xs[buf][u], ws[buf][u], k0 + u);
    };
    auto mac_run = [&](int buf) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            mac(xs[buf][u], ws[buf][u]);
    };
    constexpr int NEXT = WV * U;
    auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
    int k0 = wave * U, runs = (KT + NEXT - 1) / NEXT;
    load_run(0, k0);
    for (; runs > 2; runs -= 2) {
        load_run(1, k0 += NEXT);
        fence();
        mac_run(0);
        fence();
        load_run(0, k0 += NEXT);
        fence();
        mac_run(1);
        fence();
    }
    if (runs == 2) {
        load_run(1, k0 + NEXT);
        fence();
        mac_run(0);
        mac_run(1);
    } else {
        mac_run(0);
    }

    // lane holds n = 4 g + r (r = 0..3) of m = r16 of each 16 x 16 tile
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
            *reinterpret_cast<uint4 *>(red + (wave * (NT * MT) + i * MT + j) * RED_TILE +
                                       r16 * RED_PITCH + 4 * g) =
                __builtin_bit_cast(uint4, acc[i][j]);
    __syncthreads();

    const float swf = h2f(swh);
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int lm = om + p * RSTEP, m = m0 + lm;
        if (lm >= ROWS || m >= M || on >= N)
            continue;
        const int cell = ((tid % COLS) / 16 * MT + lm / 16) * RED_TILE + (lm & 15) * RED_PITCH +
                         (tid & 15);
        int iv;
        if constexpr (BITS == 6) {
            float s = 0.0f;
#pragma unroll
            for (int w = 0; w < WV; ++w)
                s += __uint_as_float(red[w * (NT * MT) * RED_TILE + cell]);
            iv = (int)s;
        } else {
            uint32_t s = 0;
#pragma unroll
            for (int w = 0; w < WV; ++w)
                s += red[w * (NT * MT) * RED_TILE + cell];
            iv = BITS == 4 ? (int)s >> 8 : (int)s;
        }
        const float tt = (float)iv * h2f(sxh[p]);
        a.y[(int64_t)m * N + on] = f2h(tt * swf);
        if (a.acc)
            a.acc[(int64_t)m * N + on] = iv;
    }
}

template <int BITS, int MT, int NT, int WV, int U>
hipError_t go(const GemmArgs &a, int grid, hipStream_t s)
{
    constexpr int lds = WV * NT * MT * RED_TILE * 4;
    const void *fn = (const void *)k_gemm_stream<BITS, MT, NT, WV, U>;
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess)
            return e;
    }
    GemmArgs args = a;
    void *params[] = {&args};
    return hipLaunchKernel(fn, dim3((unsigned)grid), dim3(64 * WV), params, (size_t)lds, s);
}

// Eight waves per block; U, the k-steps per run, keeps two runs of slices in
// the registers of two blocks per CU where the tile is small, of one where
// it is not.
template <int BITS>
hipError_t pick(const GemmArgs &a, const PathPlan &p, hipStream_t s)
{
    switch (10 * p.a + p.b) {
    case 11: return go<BITS, 1, 1, 8, 4>(a, p.grid, s);
    case 12: return go<BITS, 1, 2, 8, 4>(a, p.grid, s);
    case 14: return go<BITS, 1, 4, 8, 2>(a, p.grid, s);
    case 21: return go<BITS, 2, 1, 8, 4>(a, p.grid, s);
    case 22: return go<BITS, 2, 2, 8, 2>(a, p.grid, s);
    case 24: return go<BITS, 2, 4, 8, 2>(a, p.grid, s);
    case 41: return go<BITS, 4, 1, 8, 2>(a, p.grid, s);
    case 42: return go<BITS, 4, 2, 8, 1>(a, p.grid, s);
    case 44: return go<BITS, 4, 4, 8, 1>(a, p.grid, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_gemm_stream(const GemmArgs &a, const PathPlan &p, int bits, hipStream_t s)
{
    hipError_t e = bits == 6 ? pick<6>(a, p, s) : bits == 8 ? pick<8>(a, p, s) : pick<4>(a, p, s);
    return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace quarot
