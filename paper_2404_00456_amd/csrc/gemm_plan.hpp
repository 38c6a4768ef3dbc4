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
    Tile128,  // persistent, 128 x 256 block tiles, one wave per SIMD
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
    const bool m128 = ksplit || (ksteps >= stages && M > 128 && r128 * 90 < r256 * 100);
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

// The streaming kernels' plan (gemm_stream.hip): tile 16 mt x 16 nt, blocks;
// mt = 0: the problem takes the tiled plan above.
struct StreamPlan {
    int mt, nt, grid;
};

// A block of the streaming kernels reads its nt W slices and its X rows once
// per k-step, at a rate that hardly depends on the tile, so the time goes
// with rounds of blocks over the CUs times (16 nt + rows).  That product
// picked the fastest of nt = 1, 2, 4 in 117 of 120 measured shapes (e3m2,
// int4 and int8 codes, M = 1 .. 256, N = 1024 .. 28672, K = 4096 .. 28672),
// within 9% in the others: wide tiles where N gives every CU a block all the same
// (N = 28672, M = 61: nt = 1, 2, 4 take 68, 52, 40 us), narrow ones where it
// does not (N = 4096, K = 4096: 5.3, 6.2, 7.9 us).
//
// Against the tiled kernels the estimate is 2 us and STREAM ns per row of
// the sum above and k-step, against 8 us and TILED ns per round of tiles
// and k-step (twice that for 256-row tiles with more than 128 rows in use).
// Both were fitted to the same shapes: 256 x 28672, K = 8192 takes 104 us
// streamed and 60 us tiled, 256 x 8192, K = 28672 88 and 168 us.
inline StreamPlan plan_stream(int64_t M, int64_t N, int64_t K, int bits, int cus, int stages)
{
    if (bits == 4 && K % 128 != 0)
        return {0, 0, 0};
    const int mt = M <= 16 ? 1 : M <= 32 ? 2 : 4;
    const int64_t rows = M < 16 * mt ? M : 16 * mt;
    const int64_t TM = (M + 16 * mt - 1) / (16 * mt);
    int best = 0;
    int64_t units = 0, grid = 0;
    for (int nt = 1; nt <= 4; nt *= 2) {
        const int64_t blocks = TM * ((N + 16 * nt - 1) / (16 * nt));
        const int64_t u = (blocks + cus - 1) / cus * (16 * nt + rows);
        if (!best || u < units) {
            best = nt;
            units = u;
            grid = blocks;
        }
    }
    const GemmPlan g = plan_gemm(M, N, K, bits, cus, stages);
    const int64_t ksteps = bits == 8 ? K / 64 : K / 128;
    const int64_t half = g.kernel == GemmKernel::Tile256 ? 256 : 128;
    const int64_t tiles = (M + half - 1) / half * ((N + 255) / 256);
    const int64_t rounds = (tiles + g.grid - 1) / g.grid;
    const int64_t full = half == 256 && M > 128 ? 2 : 1;
    const int64_t stream = bits == 6 ? 180 : 210, tiled = bits == 4 ? 1200 : 600;  // 1/100, 1 ns
    if (2000 + units * ksteps * stream / 100 >= 8000 + rounds * full * ksteps * tiled)
        return {0, 0, 0};
    return {mt, best, (int)grid};
}

}  // namespace gemm
}  // namespace quarot
