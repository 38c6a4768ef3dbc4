// Host-side choice of the integer GEMM kernel and its grid from the
// problem's shape and the device's CU count.  Plain C++ with no HIP, so the
// rule builds and is checked on any host.
#pragma once

#include <cstdint>

namespace quarot {
namespace gemm {

enum class GemmKernel {
    K64,      // int4 codes with K not a multiple of 128: one 256 x 256 tile per block
    Tile256,  // persistent, 256 x 256 block tiles
    Tile128,  // e3m2 only: persistent, 128 x 256 block tiles, one wave per SIMD
    Ksplit,   // e3m2 only: 128 x 256 tiles, k-steps split between two wave groups
};

struct GemmPlan {
    GemmKernel kernel;
    int grid;  // blocks
};

// bits: 4 (int4 codes widened to int8), 6 (int4 codes as e3m2 numbers) or
// 8 (int8 codes); cus: the device's compute units; stages: the depth of the
// persistent kernels' LDS ring.  M, N > 0; the caller returns before
// planning an empty output.
inline GemmPlan plan_gemm(int64_t M, int64_t N, int64_t K, int bits, int cus, int stages)
{
    constexpr int64_t TILE = 256;
    if (bits == 4 && K % 128 != 0)
        return {GemmKernel::K64, (int)(((M + TILE - 1) / TILE) * ((N + TILE - 1) / TILE))};
    const int64_t ksteps = bits == 8 ? K / 64 : K / 128;
    // 128-row block tiles when that takes less time over the CUs: with one
    // wave per SIMD a 128 x 256 tile takes about 0.9 of a 256 x 256 tile's
    // time (measured on the 7B down-projection shape: 74.6 against 81.8 us
    // for one round each), so only grids that leave CUs idle gain (2048 x
    // 4096 outputs: 128 large tiles for 256 CUs), not the 16384-token ones.
    const int64_t TN = (N + TILE - 1) / TILE;
    const int64_t t256 = ((M + 255) / 256) * TN, t128 = ((M + 127) / 128) * TN;
    const int64_t r256 = (t256 + cus - 1) / cus, r128 = (t128 + cus - 1) / cus;
    // e3m2 codes with K a multiple of 256: the 128-row tiles with the
    // k-steps split between two wave groups, which take about KSPLIT_COST %
    // of a 256 x 256 tile's time
    constexpr int64_t KSPLIT_COST = 70;
    const bool ksplit =
        bits == 6 && K % 256 == 0 && K >= 512 && M > 128 && r128 * KSPLIT_COST < r256 * 100;
    const bool m128 =
        ksplit || (bits == 6 && ksteps >= stages && M > 128 && r128 * 90 < r256 * 100);
    const int64_t tiles = m128 ? t128 : t256;
    // persistent: one block per CU, or fewer for small problems (the LDS
    // ring allows one resident block per CU); with fewer than `stages`
    // k-steps, one tile per block.  A grid of whole groups of eight when the
    // tiles come in such groups, so that each XCD takes the same share.
    int64_t grid = (tiles < cus || ksteps < stages) ? tiles : cus;
    if (grid >= 8 && tiles % 8 == 0)
        grid -= grid % 8;
    return {ksplit ? GemmKernel::Ksplit : m128 ? GemmKernel::Tile128 : GemmKernel::Tile256,
            (int)grid};
}

// Blocks of 512 threads that one launch can hold: fewer than 2^32 threads.
constexpr int64_t MOST_BLOCKS = (int64_t(1) << 23) - 1;

// The path of a product: the tiled plan above, or the kernels for fewer rows
// or outputs than fill it.
enum class GemmPath {
    Tiled,   // plan_gemm
    Stream,  // gemm_stream.hip, tile 16 a x 16 b
    Mid,     // gemm_mid.hip, tile 32 a x 64 b
};

struct PathPlan {
    GemmPath path;
    int a, b, grid;
};

// Times are estimated in ns and the smallest wins.  The constants were fitted
// to measured shapes of e3m2, int4 and int8 codes on 256 CUs: 327 of serving
// programs (K = 4096 .. 28672), then, for what a round of blocks costs beside
// its k-steps, 4653 random ones (M = 1 .. 30000, N = 16 .. 32768, K = 64 ..
// 30720).  Over the latter the choice takes 2.9% more time than the fastest of
// all tiles on average, 6 shapes lose more than 4% against the tiled kernels
// and the worst 14%; without the costs per round 65 lost more than 4% and the
// worst took 2.8 times the time (11964 x 1612, K = 128 on int4: stream 68 us,
// tiled 24, mid 18).  A kernel's time is a start-up plus rounds of its blocks
// over the CUs times k-steps times what one step of a tile takes:
//  * Stream: a block's time per k-step goes with its 16 b columns plus its
//    rows, at a rate set by the CU (LO) or, with every CU busy, by the L2s
//    (HI).  Of its widths b, rounds * (16 b + rows) picks the fastest (within
//    9% in 120 shapes): wide where N gives every CU a block all the same
//    (61 x 28672, K = 8192: 1, 2, 4 take 68, 52, 40 us), narrow where it does not
//    (61 x 4096, K = 4096: 5.3, 6.2, 7.9 us).  With few k-steps a block's
//    start and end are what takes time, 1.1 us and 0.9 per 1000 outputs.
//  * Mid: STEP, a fifth more for the small tiles when they come in several
//    rounds (their operand traffic then meets the L2s' limit), 1 us per round
//    and 0.06 per 1000 outputs of a tile for each round but the last.
//  * Tiled: the 128-row tiles take 530 to 1250 ns per k-step, the 256-row
//    tiles 850 to 1500 (600 when half of them is padding); the split-k kernel
//    starts up in 11 us and waits for HBM when W exceeds the last-level cache.
//    2 and 4 us for the stores of each round but the last.
// For instance 333 x 11008, K = 4096 on e3m2: stream 33 us, mid 128 x 192
// 18.7, tiled 28.4; 2048 x 4096, K = 11008: mid 58.4, tiled 55.5.
inline PathPlan plan_path(int64_t M, int64_t N, int64_t K, int bits, int cus, int stages)
{
    if (bits == 4 && K % 128 != 0)
        return {GemmPath::Tiled, 0, 0, 0};
    auto up = [](int64_t x, int64_t d) { return (x + d - 1) / d; };
    const int64_t ks = bits == 8 ? K / 64 : K / 128;
    const int f = bits == 6 ? 0 : bits == 4 ? 1 : 2;

    const GemmPlan g = plan_gemm(M, N, K, bits, cus, stages);
    const bool big = g.kernel == GemmKernel::Tile256;
    const int64_t rounds = up(up(M, big ? 256 : 128) * up(N, 256), g.grid < cus ? g.grid : cus);
    int64_t step;
    if (big)
        step = M > 128 ? (bits == 6 ? 980 : bits == 4 ? 1500 : 850)
                       : (bits == 6 ? 600 : bits == 4 ? 1250 : 610);
    else
        step = bits == 6 ? (N * K > 100000000 ? 660 : 530) : bits == 4 ? 1250 : 610;
    int64_t best = (g.kernel == GemmKernel::Ksplit ? 11000 : 8000) + rounds * ks * step +
                   (rounds - 1) * (big ? 4000 : 2000);
    PathPlan plan = {GemmPath::Tiled, 0, 0, 0};

    const int mt = M <= 16 ? 1 : M <= 32 ? 2 : 4;
    const int64_t rows = M < 16 * mt ? M : 16 * mt, tm = up(M, 16 * mt);
    int nt = 0;
    int64_t units = 0, blocks = 0;
    for (int b = 1; b <= 4; b *= 2) {
        const int64_t n = tm * up(N, 16 * b), u = up(n, cus) * (16 * b + rows);
        if (nt == 0 || u < units) {
            nt = b;
            units = u;
            blocks = n;
        }
    }
    const int64_t lo = bits == 6 ? 145 : 190, hi = bits == 6 ? 175 : 210;  // 1/100 ns
    const int64_t cu = lo * units, l2 = hi * blocks * (16 * nt + rows) / cus;
    const int64_t steps = ks * (cu > l2 ? cu : l2) / 100;
    const int64_t ends = blocks > cus ? blocks * (1100 + 14 * nt * rows) / cus : 0;
    const int64_t stream = 2000 + (steps > ends ? steps : ends);
    if (stream < best && blocks <= MOST_BLOCKS) {
        best = stream;
        plan = {GemmPath::Stream, mt, nt, (int)blocks};
    }

    static constexpr struct {
        int a, b, step[3], more;  // ns per k-step (e3m2, int4, int8); percent in several rounds
    } mids[] = {
        {2, 1, {190, 225, 120}, 120}, {2, 2, {250, 350, 195}, 120}, {4, 2, {365, 540, 270}, 120},
        {4, 3, {520, 750, 400}, 105}, {4, 4, {690, 920, 560}, 100}, {8, 3, {890, 1250, 740}, 100},
    };
    for (const auto &m : mids) {
        const int64_t n = up(M, 32 * m.a) * up(N, 64 * m.b), r = up(n, cus);
        // 3% on the safe side
        const int64_t t = (2500 + r * (ks * m.step[f] * (r > 1 ? m.more : 100) / 100 + 1000) +
                           (r - 1) * (50 + 120 * m.a * m.b)) *
                          103 / 100;
        if (t < best && n <= MOST_BLOCKS) {
            best = t;
            plan = {GemmPath::Mid, m.a, m.b, (int)n};
        }
    }
    return plan;
}

// Group-wise products: row tiles (16 rows each) per block of the kernel for few
// rows, or 0 where the 256 x 128 tiles are the better.  Both times are straight
// lines in K: the tiles take 6 us and a rate per channel for each round of the
// CUs, whatever part of a tile is there (one rate with the ring, M and N
// multiples of 8, and one without); the few-row kernel a start, and then for
// each block a CU gets a fixed part and a rate per channel.  Fitted to 1981
// measured products (M = 1 .. 512, N = 16 .. 40000, K = 128 .. 13824, groups of
// 64, 128, 256, 256 CUs) with an error of 8% for the tiles and 17% for the few
// rows, and 6% on the safe side: the choice takes 0.3% more time than the
// faster of the two, 13 products lose more than 4% against the tiles.  Lines on
// blocks per CU alone, without K, lost 2.6% and 101 (groups of 256, 32 x 31264,
// K = 256: few 33 us, tiles 9.5; groups of 128, 256 x 4096, K = 4096: 39 against
// 57).  Rows past 512 were not measured.
inline int few_tiles(int64_t M, int64_t N, int64_t K, int group, int cus)
{
    if (M > 512)
        return 0;
    const int i = M <= 16 ? 0 : M <= 32 ? 1 : 2, g = group / 128, rows = 16 << i;
    // ns per round and 1/10 ns per channel; ns per block and 1/100 ns per channel
    static constexpr int tile[3][2] = {{253, 197}, {178, 125}, {224, 133}};
    static constexpr int start[3] = {5000, 3400, 3000};
    static constexpr int block[3][3] = {{200, 1700, 1650}, {900, 2900, 2500}, {1000, 2650, 1600}};
    static constexpr int chan[3][3] = {{107, 303, 517}, {59, 122, 206}, {45, 95, 119}};
    const int64_t tiles = (M + 255) / 256 * ((N + 127) / 128);
    const int64_t rounds = (tiles + cus - 1) / cus;
    const int64_t tiled = rounds * (6000 + K * tile[g][M % 8 == 0 && N % 8 == 0] / 10);
    const int64_t blocks = (M + rows - 1) / rows * ((N + 15) / 16);
    const int64_t per = 100 * block[g][i] + K * chan[g][i];
    const int64_t few = start[i] + (blocks > cus ? blocks : cus) * per / (100 * cus);
    return blocks <= MOST_BLOCKS && few * 106 <= tiled * 100 ? 1 << i : 0;
}

}  // namespace gemm
}  // namespace quarot
