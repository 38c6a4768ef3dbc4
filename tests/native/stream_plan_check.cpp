// The streaming GEMMs' plan (csrc/gemm_plan.hpp), built for the host: over a
// sweep of shapes, code widths and CU counts every plan is a compiled tile
// whose grid covers the output exactly once, int4 codes with K not a multiple
// of 128 never stream, and the shapes the rule was fitted to fall on the side
// that was measured faster.
#include <cstdio>
#include <initializer_list>

#include "gemm_plan.hpp"

using quarot::gemm::plan_stream;

int main()
{
    const long long Ms[] = {1, 15, 16, 17, 32, 33, 64, 65, 128, 333, 1024, 16384, 1 << 20};
    const long long Ns[] = {1, 16, 17, 250, 4096, 8190, 11008, 28672, 1 << 20};
    const long long Ks[] = {64, 128, 192, 256, 4096, 11008, 28672, 65536};
    int failures = 0;
    for (long long M : Ms)
        for (long long N : Ns)
            for (long long K : Ks)
                for (int bits : {4, 6, 8})
                    for (int cus : {64, 256, 304}) {
                        if (bits == 6 && K % 128)
                            continue;
                        const auto p = plan_stream(M, N, K, bits, cus, 3);
                        if (p.mt == 0)
                            continue;
                        const bool tile = (p.mt == 1 || p.mt == 2 || p.mt == 4) &&
                                          (p.nt == 1 || p.nt == 2 || p.nt == 4);
                        const long long want = (M + 16 * p.mt - 1) / (16 * p.mt) *
                                               ((N + 16 * p.nt - 1) / (16 * p.nt));
                        if (!tile || p.grid != want || (bits == 4 && K % 128)) {
                            std::printf("FAIL M=%lld N=%lld K=%lld bits=%d: %d %d grid %d\n", M, N,
                                        K, bits, p.mt, p.nt, p.grid);
                            ++failures;
                        }
                    }
    struct {
        long long M, N, K;
        int bits, mt, nt;
    } fitted[] = {
        {1, 4096, 4096, 6, 1, 1},     {16, 8192, 28672, 6, 1, 2},   {16, 28672, 8192, 6, 1, 4},
        {61, 28672, 8192, 6, 4, 4},   {61, 8192, 28672, 6, 4, 2},   {128, 28672, 8192, 6, 0, 0},
        {256, 28672, 8192, 6, 0, 0},  {256, 8192, 28672, 6, 4, 4},  {2048, 11008, 4096, 6, 0, 0},
        {16384, 28672, 8192, 6, 0, 0}, {256, 28672, 8192, 4, 0, 0}, {256, 28672, 8192, 8, 0, 0},
        {32, 4096, 11008, 8, 2, 1},
    };
    for (const auto &c : fitted) {
        const auto p = plan_stream(c.M, c.N, c.K, c.bits, 256, 3);
        if (p.mt != c.mt || p.nt != c.nt) {
            std::printf("FAIL M=%lld N=%lld K=%lld bits=%d: tile %d x %d, want %d x %d\n", c.M,
                        c.N, c.K, c.bits, p.mt, p.nt, c.mt, c.nt);
            ++failures;
        }
    }
    if (failures)
        return 1;
    std::printf("ok\n");
    return 0;
}
