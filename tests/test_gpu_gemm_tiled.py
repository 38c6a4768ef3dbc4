"""The tiled GEMM kernels (csrc/gemm_w4a4.hip) at shapes that the plan of csrc/gemm_plan.hpp leaves to them: 256 x 256
tiles on e3m2, int4 and int8 codes, 128 x 256 e3m2 tiles with one wave per SIMD and with split k-steps.  Ragged in both
directions, with N a multiple of 4 and not, blocks that walk one tile and several, k-steps below, at and above the depth
of the LDS ring, with and without the int32 output.  Every accumulator against a binary64 product of the codes on the
GPU (exact: integers below 2^53), every output against that through the definition's roundings, and sampled rows against
the CPU oracle.  The host check of the plan (tests/native/gemm_path_check.cpp) holds these shapes to their kernels."""
import numpy as np
import pytest

from test_gpu_parity import H, assert_same, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2404_00456_amd as q
    q.lib()
    return torch.device("cuda:0")


# 396 tiles of 256 x 256 on 256 CUs, and fewer tiles than CUs
LARGE = [(646, 33753, 128), (646, 33753, 256), (646, 33753, 384), (646, 33753, 512), (646, 33753, 640),
         (650, 33764, 256), (650, 33764, 768), (388, 25203, 640)]
LARGE_INT8 = [(646, 33753, 64), (646, 33753, 128), (646, 33753, 192), (646, 33753, 256), (646, 33753, 320),
              (650, 33764, 192), (388, 25203, 320)]
# 128 x 256: an odd number of k-steps
SMALL = [(260, 33753, 2176), (270, 33764, 2176)]
# 128 x 256 with split k-steps
SPLIT = [(519, 49162, 768), (800, 33753, 1536), (8317, 607, 8192), (1409, 4100, 11008), (1282, 11008, 4096),
         (2047, 4095, 11008)]


@pytest.mark.parametrize("fmt,M,N,K", [("e3m2",) + s for s in LARGE + SMALL + SPLIT] +
                         [("int4",) + s for s in LARGE] + [("int8",) + s for s in LARGE_INT8])
def test_gemm_tiled_exact(dev, orc, fmt, M, N, K):
    import torch
    import paper_2404_00456_amd as q
    say(f"tiled gemm {fmt} M={M} N={N} K={K}")
    g = torch.Generator(device=dev).manual_seed(M * 3 + N + K)
    sx = (torch.rand(M, generator=g, device=dev) * 0.05 + 0.01).half()
    sw = (torch.rand(N, generator=g, device=dev) * 0.002 + 0.0005).half()
    if fmt == "int8":
        xq = torch.randint(-128, 128, (M, K), generator=g, device=dev, dtype=torch.int8)
        wq = torch.randint(-128, 128, (N, K), generator=g, device=dev, dtype=torch.int8)
        call, args, codes = q.quarot_w8a8_gemm, (xq, sx, wq, sw), lambda t: t.double()
    else:
        xq = torch.randint(0, 256, (M, K // 2), generator=g, device=dev, dtype=torch.uint8)
        wq = torch.randint(0, 256, (N, K // 2), generator=g, device=dev, dtype=torch.uint8)
        xq[0] = wq[0] = 0x88  # -8 . -8 over all of K: the largest accumulator

        def codes(t):
            b = t.to(torch.int16)
            return torch.stack(((b & 15) ^ 8, (b >> 4) ^ 8), 2).reshape(t.shape[0], K).double() - 8
        if fmt == "e3m2":
            call, args = q.quarot_w4a4_gemm_e3m2, (q.quarot_pack_e3m2(xq), sx, q.quarot_pack_e3m2(wq), sw)
        else:
            call, args = q.quarot_w4a4_gemm, (xq, sx, wq, sw)
    ref = torch.mm(codes(xq), codes(wq).T.contiguous())
    ry = ((ref.float() * sx.float()[:, None]) * sw.float()[None, :]).half()
    y, acc = call(*args, want_acc=True)
    assert torch.equal(acc, ref.int()), f"acc: {int((acc != ref.int()).sum())} of {M * N} differ"
    assert torch.equal(y.view(torch.int16), ry.view(torch.int16)), "y with acc"
    y = call(*args)
    assert torch.equal(y.view(torch.int16), ry.view(torch.int16)), "y alone"
    rows = torch.tensor([0, M // 2, M - 1], device=dev)
    xs, ws = H(xq[rows]), H(wq)
    racc = orc.gemm_i8(xs, ws) if fmt == "int8" else orc.gemm_i32(xs, ws)
    assert_same(H(acc[rows]), racc, "sampled rows")
    assert_same(H(y[rows]).view(np.uint16), orc.dequant(racc, H(sx[rows]), H(sw)).view(np.uint16),
                "sampled rows of y")
