"""The GEMM kernels for middling grids (csrc/gemm_mid.hip) against the CPU
oracle on e3m2, int4 and int8 codes: int32 accumulators and fp16 outputs bit
for bit, with and without the int32 output, over every tile the rule of
csrc/gemm_plan.hpp picks (named beside each shape for 256 CUs), ragged in both
directions, with fewer, as many and more k-steps than the ring has stages."""
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
    (75, 8190, 28672),   # 64 x 64 on e3m2
    (100, 5001, 1152),   # 64 x 64 on int8
    (70, 9003, 2048),    # 64 x 128
    (250, 9002, 1152),   # 128 x 128
    (700, 5004, 640),    # 128 x 128 on e3m2 and int4
    (500, 9001, 1152),   # 128 x 192
    (300, 16001, 384),   # 128 x 192, three 128-k steps
    (700, 9004, 640),    # 128 x 256
    (500, 16002, 256),   # 128 x 256, two steps
    (1000, 9001, 512),   # 256 x 192
    (1500, 16001, 128),  # 256 x 192, one step, more tiles than CUs
])
def test_gemm_mid_exact(dev, orc, fmt, M, N, K):
    import paper_2404_00456_amd as q
    say(f"mid gemm {fmt} M={M} N={N} K={K}")
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
    ry = orc.dequant(racc, sx, sw).view(np.uint16)
    assert_same(H(call(*args)).view(np.uint16), ry, f"mid y {fmt} M={M} N={N} K={K}")
    y, acc = call(*args, want_acc=True)
    assert_same(H(acc), racc, f"mid acc {fmt} M={M} N={N} K={K}")
    assert_same(H(y).view(np.uint16), ry, f"mid y with acc {fmt} M={M} N={N} K={K}")


def test_gemm_mid_int8_odd_steps(dev, orc):
    """int8 codes with K a multiple of 64 only (five k-steps)."""
    import paper_2404_00456_amd as q
    M, N, K = 500, 9001, 320
    say(f"mid gemm int8 M={M} N={N} K={K}")
    rng = np.random.default_rng(5)
    xq = rng.integers(-128, 128, size=(M, K), dtype=np.int8)
    wq = rng.integers(-128, 128, size=(N, K), dtype=np.int8)
    sx = rng.uniform(0.001, 0.05, M).astype(np.float16)
    sw = rng.uniform(0.0005, 0.01, N).astype(np.float16)
    racc = orc.gemm_i8(xq, wq)
    y, acc = q.quarot_w8a8_gemm(T(xq, dev), T(sx, dev), T(wq, dev), T(sw, dev), want_acc=True)
    assert_same(H(acc), racc, "mid int8 odd steps acc")
    assert_same(H(y).view(np.uint16), orc.dequant(racc, sx, sw).view(np.uint16),
                "mid int8 odd steps y")
