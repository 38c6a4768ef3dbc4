// The decode attention's choice of kernel, waves and splits (csrc/attn_plan.hpp
// and kv_attn_splits of csrc/host_rules.cpp), built for the host: over a sweep
// of rows, queries per row, tokens and CU counts every plan is a compiled
// kernel, takes no more splits than the workspace holds, covers every token and
// launches fewer than 2^32 threads where that is possible, and calls the rule
// was fitted to fall on the side that was measured faster.
#include <algorithm>
#include <cstdio>
#include <initializer_list>

#include "attn_plan.hpp"

using quarot::attn::plan;
using quarot::attn::plan_blocks;

// kv_attn_splits of host_rules.cpp, which the workspace is sized by
static long long most_splits(long long nq, long long seq)
{
    return std::max<long long>(1, std::min((2048 + nq - 1) / nq, (seq + 255) / 256));
}

int main()
{
    int failures = 0, taken[2][2] = {}, cut = 0;
    for (long long nkv : {1, 2, 7, 8, 31, 40, 64, 100, 128, 129, 160, 255, 256, 257, 300, 512, 1024,
                          5000, 1 << 20, (1 << 23) - 1, 1 << 23, (1 << 23) + 3, 1 << 24})
        for (int rep : {1, 2, 3, 7, 8, 9, 16, 17, 33, 64})
            for (long long seq : {1, 2, 31, 64, 65, 100, 255, 256, 257, 600, 1000, 4099, 16000,
                                  1 << 20, 0x7FFFFFFF})
                for (int cus : {1, 64, 256, 304}) {
                    const long long nq = nkv * rep, most = most_splits(nq, seq);
                    if (nq > 0x7FFFFFFF)
                        continue;
                    const auto p = plan(nkv, rep, seq, most, cus);
                    const long long blocks = plan_blocks(p.shared, nkv, rep);
                    const long long chunk = ((seq + p.splits - 1) / p.splits + 63) / 64 * 64;
                    const bool fits = plan_blocks(rep > 1, nkv, rep) < 1 << 24;
                    if ((p.waves != 4 && p.waves != 8) || p.splits < 1 || p.splits > most ||
                        (p.shared && rep == 1) || chunk * p.splits < seq ||
                        (fits && blocks * p.splits * 64 * p.waves > 0xFFFFFFFFll)) {
                        std::printf("FAIL nkv=%lld rep=%d seq=%lld cus=%d: shared %d waves %d splits %d\n",
                                    nkv, rep, seq, cus, p.shared, p.waves, p.splits);
                        ++failures;
                    }
                    ++taken[p.shared][p.waves == 8];
                    cut += p.splits > 1;
                }
    if (!taken[0][0] || !taken[0][1] || !taken[1][0] || !taken[1][1] || !cut) {
        std::printf("FAIL a kernel is never taken\n");
        ++failures;
    }
    // (fewest and most splits that measured alike)
    const struct {
        long long nkv;
        int rep;
        long long seq;
        bool shared;
        int lo, hi;
    } fitted[] = {
        // short or few rows of several queries: a block per query is the faster
        {1, 8, 100, false, 1, 1},    {8, 8, 100, false, 1, 1},    {8, 8, 1000, false, 2, 4},
        {8, 4, 1000, false, 2, 4},   {32, 2, 1000, false, 1, 4},  {264, 2, 48, false, 1, 1},
        // and their shared kernel where the rows are long or many
        {40, 8, 4099, true, 6, 12},  {192, 8, 3000, true, 1, 1},  {64, 4, 4000, true, 3, 6},
        // rows that leave a wave of blocks half empty are cut, others not
        {129, 1, 8000, false, 3, 16}, {136, 1, 8000, false, 3, 16}, {300, 1, 8000, false, 2, 7},
        {512, 1, 2047, false, 1, 1}, {256, 1, 4000, false, 1, 1}, {32, 1, 500, false, 1, 1},
    };
    for (const auto &c : fitted) {
        const auto p = plan(c.nkv, c.rep, c.seq, most_splits(c.nkv * c.rep, c.seq), 256);
        if (p.shared != c.shared || p.splits < c.lo || p.splits > c.hi) {
            std::printf("FAIL nkv=%lld rep=%d seq=%lld: shared %d waves %d splits %d, want shared %d splits %d .. %d\n",
                        c.nkv, c.rep, c.seq, p.shared, p.waves, p.splits, c.shared, c.lo, c.hi);
            ++failures;
        }
    }
    // the calls by which tests/test_gpu_kv_gqa.py reaches the shared kernel
    const long long shared[][3] = {
        {130, 2, 129}, {130, 2, 257}, {130, 2, 2049}, {130, 3, 255}, {130, 5, 65}, {130, 7, 257},
        {130, 8, 17},  {130, 8, 33},  {130, 9, 129},  {130, 9, 255}, {130, 16, 33}, {130, 17, 2049},
        {130, 33, 1},  {130, 33, 257}, {520, 2, 33},  {520, 2, 513}, {520, 3, 17}, {520, 5, 1},
        {520, 7, 1025}, {60, 8, 513}, {60, 8, 1025},  {60, 5, 2049}, {300, 2, 1025}, {300, 3, 2049},
        {60, 8, 1500}, {130, 8, 600}, {130, 8, 40},
    };
    int waves[2] = {}, split[2] = {};
    for (const auto &c : shared) {
        const auto p = plan(c[0], (int)c[1], c[2], most_splits(c[0] * c[1], c[2]), 256);
        if (!p.shared) {
            std::printf("FAIL nkv=%lld rep=%lld seq=%lld: a block per query row\n", c[0], c[1], c[2]);
            ++failures;
        }
        ++waves[p.waves == 8];
        ++split[p.splits > 1];
    }
    if (waves[0] < 5 || waves[1] < 5 || split[0] < 5 || split[1] < 5) {
        std::printf("FAIL shared calls: %d of four waves, %d of eight, %d whole, %d split\n", waves[0],
                    waves[1], split[0], split[1]);
        ++failures;
    }
    if (failures)
        return 1;
    std::printf("ok\n");
    return 0;
}
