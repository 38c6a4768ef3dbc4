// The choice between the GEMM kernels (csrc/gemm_plan.hpp), built for the
// host: over a sweep of shapes, code widths and CU counts every plan is a
// compiled tile whose grid covers the output exactly once, int4 codes with K
// not a multiple of 128 stay on the tiled path, and shapes the rule was
// fitted to fall on the side that was measured faster.
#include <cstdio>
#include <initializer_list>

#include "gemm_plan.hpp"

using quarot::gemm::few_tiles;
using quarot::gemm::GemmPath;
using quarot::gemm::plan_path;

int main()
{
    const long long Ms[] = {1,  15,  16,  17,  32,   33,    64,      65,
                            90, 128, 333, 517, 1024, 16384, 1 << 20, 1 << 30};
    const long long Ns[] = {1,    16,    17,    250,     1376,    4096,   8190,
                            11008, 28672, 1 << 20, 1 << 27, 1 << 29, 1 << 30};
    const long long Ks[] = {64, 128, 192, 256, 4096, 11008, 28672, 65536};
    int failures = 0, taken[3] = {0, 0, 0};
    for (long long M : Ms)
        for (long long N : Ns)
            for (long long K : Ks)
                for (int bits : {4, 6, 8})
                    for (int cus : {64, 256, 304}) {
                        if (bits == 6 && K % 128)
                            continue;
                        if ((M + 255) / 256 * ((N + 255) / 256) > 0x7FFFFFFF)
                            continue;  // refused before planning
                        const auto p = plan_path(M, N, K, bits, cus, 3);
                        ++taken[(int)p.path];
                        if (p.path == GemmPath::Tiled)
                            continue;
                        const int t = 10 * p.a + p.b;
                        bool ok;
                        long long um, un;
                        if (p.path == GemmPath::Stream) {
                            ok = t == 11 || t == 12 || t == 14 || t == 21 || t == 22 || t == 24 ||
                                 t == 41 || t == 42 || t == 44;
                            um = 16 * p.a;
                            un = 16 * p.b;
                        } else {
                            ok = t == 21 || t == 22 || t == 42 || t == 43 || t == 44 || t == 83;
                            um = 32 * p.a;
                            un = 64 * p.b;
                        }
                        const long long want = (M + um - 1) / um * ((N + un - 1) / un);
                        // blocks of 512 threads, fewer than 2^32 threads in a launch
                        if (!ok || p.grid != want || want >= 1 << 23 ||
                            (bits == 4 && K % 128)) {
                            std::printf("FAIL M=%lld N=%lld K=%lld bits=%d: path %d %d %d grid %d\n",
                                        M, N, K, bits, (int)p.path, p.a, p.b, p.grid);
                            ++failures;
                        }
                    }
    // group-wise products: the same bound
    for (long long M : Ms)
        for (long long N : Ns)
            for (long long K : Ks)
                for (int group : {64, 128, 256})
                    for (int cus : {64, 256, 304}) {
                        const int tiles = few_tiles(M, N, K, group, cus);
                        const long long rows = 16 * tiles;
                        if (tiles != 0 &&
                            ((tiles != 1 && tiles != 2 && tiles != 4) || M > 512 ||
                             (M + rows - 1) / rows * ((N + 15) / 16) >= 1 << 23)) {
                            std::printf("FAIL group-wise M=%lld N=%lld K=%lld group=%d: %d\n", M, N,
                                        K, group, tiles);
                            ++failures;
                        }
                    }
    const struct {
        long long M, N, K;
        int group, tiles;
    } grouped[] = {
        {1, 4096, 4096, 128, 1},    {16, 11008, 4096, 128, 1},  {64, 5120, 13824, 128, 4},
        {256, 4096, 4096, 128, 4},  {384, 4096, 4096, 128, 0},  {512, 4096, 11008, 256, 4},
        {2048, 11008, 4096, 128, 0}, {30, 4096, 4096, 64, 2},
        // few groups: the few-row kernel's fixed part per block is what takes time
        {32, 31264, 256, 256, 0},   {16, 28672, 256, 128, 0},   {464, 4096, 256, 256, 0},
        {80, 8192, 128, 128, 0},    {32, 11008, 256, 128, 0},
    };
    for (const auto &c : grouped) {
        const int tiles = few_tiles(c.M, c.N, c.K, c.group, 256);
        if (tiles != c.tiles) {
            std::printf("FAIL group-wise M=%lld N=%lld K=%lld group=%d: %d, want %d\n", c.M, c.N,
                        c.K, c.group, tiles, c.tiles);
            ++failures;
        }
    }
    for (int n : taken)
        if (!n) {
            std::printf("FAIL a path is never taken\n");
            ++failures;
        }
    const GemmPath T = GemmPath::Tiled, S = GemmPath::Stream, D = GemmPath::Mid;
    const struct {
        long long M, N, K;
        int bits;
        GemmPath path;
        int a, b;
    } fitted[] = {
        {1, 4096, 4096, 6, S, 1, 1},     {16, 8192, 28672, 6, S, 1, 2},
        {16, 28672, 8192, 6, S, 1, 4},   {33, 28672, 8192, 4, S, 4, 4},
        {61, 8192, 28672, 6, S, 4, 2},   {128, 28672, 8192, 6, D, 4, 2},
        {333, 11008, 4096, 6, D, 4, 3},  {1024, 4096, 4096, 6, D, 4, 2},
        {2048, 4096, 11008, 6, T, 0, 0}, {16384, 28672, 8192, 6, T, 0, 0},
        {16384, 8192, 28672, 6, T, 0, 0}, {1777, 4096, 4096, 4, D, 4, 4},
        {16384, 28672, 8192, 4, T, 0, 0}, {517, 5120, 13824, 8, D, 4, 2},
        {32, 4096, 11008, 8, S, 2, 1},   {3000, 8192, 8192, 8, T, 0, 0},
        // few k-steps over many rounds of blocks: not the streaming kernel
        {11964, 1612, 128, 4, D, 8, 3},  {3318, 2788, 128, 6, D, 8, 3},
        {6515, 1660, 128, 4, D, 8, 3},   {86, 27196, 128, 8, D, 4, 2},
        {6610, 724, 256, 6, D, 4, 3},    {1, 26690, 128, 6, D, 2, 2},
    };
    for (const auto &c : fitted) {
        const auto p = plan_path(c.M, c.N, c.K, c.bits, 256, 3);
        if (p.path != c.path || p.a != c.a || p.b != c.b) {
            std::printf("FAIL M=%lld N=%lld K=%lld bits=%d: path %d tile %d x %d, want %d %d x %d\n",
                        c.M, c.N, c.K, c.bits, (int)p.path, p.a, p.b, (int)c.path, c.a, c.b);
            ++failures;
        }
    }
    // the shapes by which tests/test_gpu_gemm_tiled.py reaches the tiled kernels
    typedef quarot::gemm::GemmKernel Kn;
    const Kn L = Kn::Tile256, W = Kn::Tile128, X = Kn::Ksplit;
    const struct {
        long long M, N, K;
        Kn kernel;
    } tiled[] = {
        {646, 33753, 128, L},   {646, 33753, 256, L},  {646, 33753, 384, L},   {646, 33753, 512, L},
        {646, 33753, 640, L},   {650, 33764, 256, L},  {650, 33764, 768, L},   {388, 25203, 640, L},
        {646, 33753, 64, L},    {646, 33753, 192, L},  {646, 33753, 320, L},   {650, 33764, 192, L},
        {388, 25203, 320, L},   {260, 33753, 2176, W}, {270, 33764, 2176, W},
        {519, 49162, 768, X},   {800, 33753, 1536, X}, {8317, 607, 8192, X},   {1409, 4100, 11008, X},
        {1282, 11008, 4096, X}, {2047, 4095, 11008, X},
    };
    for (const auto &c : tiled)
        for (int bits : {4, 6, 8}) {
            // int8 codes: K to 320; int4 and e3m2 codes: K in 128s
            if (bits == 8 ? c.K > 320 : c.K % 128 || (bits == 4 && c.kernel != L))
                continue;
            const auto p = plan_path(c.M, c.N, c.K, bits, 256, 3);
            const auto g = quarot::gemm::plan_gemm(c.M, c.N, c.K, bits, 256, 3);
            if (p.path != T || g.kernel != c.kernel) {
                std::printf("FAIL M=%lld N=%lld K=%lld bits=%d: path %d kernel %d, want tiled %d\n", c.M,
                            c.N, c.K, bits, (int)p.path, (int)g.kernel, (int)c.kernel);
                ++failures;
            }
        }
    // and test_gpu_gemm_stream.py and test_gpu_gemm_mid.py theirs, on every width
    const struct {
        long long M, N, K;
        GemmPath path;
        int a, b;
    } reached[] = {
        {1, 1, 128, S, 1, 1},       {5, 8190, 512, S, 1, 2},    {9, 8913, 256, S, 1, 4},
        {14, 8915, 1152, S, 1, 4},  {17, 33, 512, S, 2, 1},     {17, 4442, 256, S, 2, 2},
        {30, 4445, 1152, S, 2, 2},  {31, 8200, 512, S, 2, 4},   {17, 8913, 256, S, 2, 4},
        {33, 64, 1024, S, 4, 1},    {40, 8190, 384, S, 4, 2},   {65, 2199, 256, S, 4, 2},
        {100, 2201, 1152, S, 4, 2}, {65, 4442, 256, S, 4, 4},   {120, 4444, 640, S, 4, 4},
        {75, 8190, 28672, D, 2, 1}, {70, 9003, 2048, D, 2, 2},  {250, 9002, 1152, D, 4, 2},
        {500, 9001, 1152, D, 4, 3}, {700, 9004, 640, D, 4, 4},  {1000, 9001, 512, D, 8, 3},
        {1500, 16001, 128, D, 8, 3}, {61, 16390, 256, D, 2, 2}, {500, 9001, 320, D, 4, 3},
    };
    for (const auto &c : reached)
        for (int bits : {4, 6, 8}) {
            if (bits != 8 && c.K % 128)
                continue;
            const auto p = plan_path(c.M, c.N, c.K, bits, 256, 3);
            if (p.path != c.path || p.a != c.a || p.b != c.b) {
                std::printf("FAIL M=%lld N=%lld K=%lld bits=%d: path %d tile %d x %d, want %d %d x %d\n",
                            c.M, c.N, c.K, bits, (int)p.path, p.a, p.b, (int)c.path, c.a, c.b);
                ++failures;
            }
        }
    if (failures)
        return 1;
    std::printf("ok\n");
    return 0;
}
