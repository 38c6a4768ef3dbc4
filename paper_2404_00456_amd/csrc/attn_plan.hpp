// Host-side choice of the decode attention's matrix-core kernel, its waves per
// block and its split of a sequence (head_dim 128, one group per cached row).
// Plain C++ with no HIP, so the rule builds and is checked on any host.
#pragma once

#include <algorithm>
#include <cstdint>

namespace quarot {
namespace attn {

constexpr int SHARED_ROWS = 8;  // query rows of a block that shares a cache row

struct Plan {
    bool shared;  // k_kv_attn_gqa: up to 8 query rows of a cache row per block;
                  // otherwise k_kv_attn_mfma: a query row per block
    int waves;    // per block, 4 or 8
    int splits;   // blocks that share a sequence, 1 .. most
};

// Blocks of a split along the query and cache rows.
inline int64_t plan_blocks(bool shared, int64_t nkv, int rep)
{
    return shared ? nkv * ((rep + SHARED_ROWS - 1) / SHARED_ROWS) : nkv * rep;
}

// nkv cache rows with rep query rows each, seq tokens, at most `most` splits (the
// workspace's), cus compute units.
//
// The time of a choice is estimated in ns and the smallest wins:
//  * a start and an end, the end of the shared kernel also per query row;
//  * the chain of a block's steps (a wave's 64 tokens, 32 in the shared kernel),
//    each 11% longer with every CU busy; or what the blocks of a CU take of it:
//    one of four waves 0.6 to 0.9 of the steps that its tokens fill, one of eight
//    1.3 to 1.5, and the filling, the last block's beside the others;
//  * a part per further block that a CU gets;
//  * the combining pass of a split: its launch, its splits and what it reads.
// The constants were fitted to the choice itself over 3116 measured calls (1 ..
// 1100 cache rows of 1 .. 16 queries, 20 .. 16000 tokens, up to 32 choices each,
// 256 CUs): it takes 0.4% more time than the fastest of them on average.  Against
// one block of four waves per query row, cut as far as the workspace allows, 31
// calls lose more than 5% (the worst 20%) and the average gains 21%.  Whole rows of
// eight waves wherever they fill half of the card, and the shared kernel wherever
// queries share a row, took 12% more: 8 rows of 8 queries, 1000 tokens: shared
// 10.6 us, a block per query 8.3; 300 rows, 8000 tokens: whole 82.7 us, in seven
// 65.0; 129 rows, 8000 tokens: whole 49.2, in sixteen 39.3.  On the other side 40
// rows of 8 queries, 4099 tokens: shared 14.8 us, a block per query 37; 512 rows,
// 2047 tokens: whole 30.2 us, in four 36.6.
inline Plan plan(int64_t nkv, int rep, int64_t seq, int64_t most, int cus)
{
    // by kernel (query, shared) and waves (4, 8)
    static constexpr double start[4] = {2106, 2425, 3860, 2711}, step[4] = {2209, 2405, 1614, 1300},
                            share[4] = {0.934, 1.342, 0.637, 1.457},
                            fill[4] = {0.36, 0.51, -0.68, 1.13}, block[2] = {149, 246};
    Plan best = {rep > 1, 4, 1};
    double least = -1;
    for (int k = 0; k < (rep > 1 ? 2 : 1); ++k) {
        const int64_t rows = plan_blocks(k, nkv, rep), R = k ? std::min(rep, SHARED_ROWS) : 1;
        // a few blocks per row, or as many as give every CU one to four
        for (int64_t want : {int64_t(1), int64_t(2), int64_t(3), int64_t(4), cus / rows,
                             2 * cus / rows, 3 * cus / rows, 4 * cus / rows}) {
            const int64_t splits = std::min(most, std::max<int64_t>(1, want));
            const int64_t blocks = rows * splits;
            const int64_t chunk = ((seq + splits - 1) / splits + 63) / 64 * 64;
            for (int w = 0; w < 2; ++w) {
                const int waves = w ? 8 : 4, c = 2 * k + w;
                // a launch holds fewer than 2^32 threads
                if (blocks * 64 * waves > 0xFFFFFFFFll)
                    continue;
                const int64_t tokens = waves * (k ? 32 : 64);
                const double steps = (double)((std::min(chunk, seq) + tokens - 1) / tokens);
                const double filled = (double)std::min(chunk, seq) / (double)tokens;
                const double u = (double)blocks / cus;
                const double per = u > 6 ? u : (double)((blocks + cus - 1) / cus);
                double t = start[c] + step[c] * std::max(steps * (1 + 0.109 * std::min(u, 1.0)),
                                                         per * share[c] * (filled + fill[c]) - fill[c]);
                t += std::max(0.0, u - 1) * block[k] * (double)R;
                if (k)
                    t += 238.0 * (double)R;
                if (splits > 1)
                    t += 3181 + 41.0 * (double)splits + 0.34 * (double)(nkv * rep * splits);
                if (least < 0 || t < least) {
                    least = t;
                    best = {k == 1, waves, (int)splits};
                }
            }
        }
    }
    return best;
}

}  // namespace attn
}  // namespace quarot
