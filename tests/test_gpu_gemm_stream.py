"""The streaming GEMM kernels (few X rows, csrc/gemm_stream.hip) against the
CPU oracle on e3m2, int4 and int8 codes: int32 accumulators and fp16 outputs
bit for bit, at the edges of their tiles (16, 32 and 64 rows; 16, 32 and 64
columns), of their runs of k-steps (1, 2 and more per wave, whole and short)
and of the rule that picks the tile (csrc/gemm_plan.hpp)."""
import numpy as np
import pytest

from test_gpu_parity import H, T, assert_same, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2404_00456_amd as q
    q.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("fmt", ["e3m2", "int4", "int8"])
@pytest.mark.parametrize("M,N,K", [
    # one row and column, one k-step; edges of the 16-, 32- and 64-row tiles
    (1, 1, 128), (15, 17, 256), (16, 16, 384), (17, 33, 512), (32, 250, 640), (33, 64, 1024),
    (63, 100, 1152), (64, 65, 4096), (65, 48, 4224), (130, 31, 4352),
    # more than one run of k-steps per wave, an odd and an even number
    (3, 40, 8192), (20, 40, 12416), (50, 24, 28672), (2, 3, 65536),
    # 32 and 64 columns per block (a block per CU at 256 CUs), ragged last, on
    # 16, 32 and 64 rows
    (5, 8190, 512), (31, 8200, 512), (40, 8190, 384), (9, 8913, 256), (14, 8915, 1152),
    (17, 4442, 256), (30, 4445, 1152), (17, 8913, 256), (65, 2199, 256), (100, 2201, 1152),
    (65, 4442, 256), (120, 4444, 640),
    # more blocks than CUs and few k-steps: the middling kernels
    (9, 20001, 256), (29, 16390, 256), (61, 16390, 256), (200, 4100, 512)])
def test_gemm_stream_exact(dev, orc, fmt, M, N, K):
    import paper_2404_00456_amd as q
    say(f"stream gemm {fmt} M={M} N={N} K={K}")
    rng = np.random.default_rng(M * 5 + N * 3 + K)
    sx = rng.uniform(0.001, 0.05, M).astype(np.float16)
    sw = rng.uniform(0.0005, 0.01, N).astype(np.float16)
    if fmt == "int8":
        xq = rng.integers(-128, 128, size=(M, K), dtype=np.int8)
        wq = rng.integers(-128, 128, size=(N, K), dtype=np.int8)
        call, racc = q.quarot_w8a8_gemm, orc.gemm_i8(xq, wq)
        args = (T(xq, dev), T(sx, dev), T(wq, dev), T(sw, dev))
    else:
        xq = rng.integers(0, 256, size=(M, K // 2), dtype=np.uint8)
        wq = rng.integers(0, 256, size=(N, K // 2), dtype=np.uint8)
        xq[0] = wq[0] = 0x88  # -8 . -8 over all of K: the largest accumulator
        racc = orc.gemm_i32(xq, wq)
        xd, wd = T(xq, dev), T(wq, dev)
        if fmt == "e3m2":
            call, xd, wd = q.quarot_w4a4_gemm_e3m2, q.quarot_pack_e3m2(xd), q.quarot_pack_e3m2(wd)
        else:
            call = q.quarot_w4a4_gemm
        args = (xd, T(sx, dev), wd, T(sw, dev))
    y, acc = call(*args, want_acc=True)
    assert_same(H(acc), racc, f"stream acc {fmt} M={M} N={N} K={K}")
    ry = orc.dequant(racc, sx, sw).view(np.uint16)
    assert_same(H(y).view(np.uint16), ry, f"stream y {fmt} M={M} N={N} K={K}")
    assert_same(H(call(*args)).view(np.uint16), ry, f"stream y alone {fmt} M={M} N={N} K={K}")
