"""The m = 108 and 172 rotations (csrc/rotate_quant.hip, k_rot_largem_f16)
against the CPU oracle on rows that reach its edges: every number of 16-group
tiles, values just below and at 512 (where the operand split changes), the
largest fp16, the smallest subnormals beside large values, zero rows, more rows
than resident blocks, every epilogue and the SwiGLU prologue, bit for bit."""
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


def edge_rows(n, rows, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((rows, n)).astype(np.float16)
    x[0] = 0
    x[1, :] = rng.choice(np.array([511.5, -511.75, 2.0 ** -24, 0.0], np.float16), n)
    x[2, n - 1] = 512.0  # the first value of the wide path, in the last slot
    x[3] = (rng.standard_normal(n) * 20000).clip(-65504, 65504).astype(np.float16)
    x[4] = np.float16(65504) * rng.choice([-1, 1], n)
    x[5] = (rng.integers(0, 1024, n).astype(np.uint16) | (rng.integers(0, 2, n).astype(
        np.uint16) << 15)).view(np.float16)  # subnormals
    x[6] = np.ldexp(1.0, rng.integers(-24, 16, n)).astype(np.float16)
    x[7, ::97] = 300.0
    return x


@pytest.mark.parametrize("n,rows", [(1728, 9), (3456, 11), (6912, 530), (13824, 1030), (2752, 9),
                                    (5504, 11), (11008, 600)])
def test_largem_edge_rows(dev, orc, n, rows):
    import paper_2404_00456_amd as q
    say(f"largem edge rows n={n} rows={rows}")
    x = edge_rows(n, rows, n)
    xd = T(x, dev)
    rq, rs = orc.quant_int4(x, rotate=True, clip=0.9)
    codes, scale = q.quarot_quant_int4(xd, clip_ratio=0.9)
    assert_same(H(codes), rq, f"int4 codes n={n}")
    assert_same(H(scale).view(np.uint16), rs.view(np.uint16), f"int4 scales n={n}")
    if n % 128 == 0 and n not in (1728, 2752):
        q6, s6 = q.quarot_quant_int4_e3m2(xd, clip_ratio=0.9)
        assert_same(H(q6), H(q.quarot_pack_e3m2(codes)), f"e3m2 codes n={n}")
        assert_same(H(s6).view(np.uint16), rs.view(np.uint16), f"e3m2 scales n={n}")
    few = x[:40]
    fd = T(few, dev)
    c8, s8 = q.quarot_quant_int8(fd, clip_ratio=0.9, bits=8)
    r8, t8 = orc.quant_int8(few, rotate=True, clip=0.9, bits=8)
    assert_same(H(c8), r8, f"int8 codes n={n}")
    assert_same(H(s8).view(np.uint16), t8.view(np.uint16), f"int8 scales n={n}")
    fin = few[[0, 1, 2, 5, 6, 7, 8]]  # rows whose rotation stays within fp16
    y = orc.hadamard(fin)
    fy = T(fin, dev)
    assert_same(H(q.quarot_hadamard(fy)).view(np.uint16), y.view(np.uint16), f"fp16 n={n}")
    q.quarot_hadamard(fy, y=fy)
    assert_same(H(fy).view(np.uint16), y.view(np.uint16), f"fp16 in place n={n}")
    g, gs = q.quarot_quant_int4_grouped(fd, group=32)
    rg, rgs = orc.quant_int4_grouped(few, group=32, rotate=True)
    assert_same(H(g), rg, f"grouped codes n={n}")
    assert_same(H(gs).view(np.uint16), rgs.view(np.uint16), f"grouped scales n={n}")


@pytest.mark.parametrize("n", [13824, 11008])
def test_largem_swiglu_edge_rows(dev, orc, n):
    import paper_2404_00456_amd as q
    say(f"largem swiglu edge rows n={n}")
    rng = np.random.default_rng(n)
    gate = (rng.standard_normal((520, n)) * 1.5).astype(np.float16)
    up = rng.standard_normal((520, n)).astype(np.float16)
    up[3] *= np.float16(300)   # products past 512
    up[4, n - 1], gate[4, n - 1] = 60.0, 10.0
    gate[5] = 0
    rq, rs = orc.swiglu_quant_int4(gate, up, rotate=True, clip=0.9)
    codes, scale = q.quarot_swiglu_quant_int4(T(gate, dev), T(up, dev), clip_ratio=0.9)
    assert_same(H(codes), rq, f"swiglu int4 codes n={n}")
    assert_same(H(scale).view(np.uint16), rs.view(np.uint16), f"swiglu int4 scales n={n}")
    q6, s6 = q.quarot_swiglu_quant_e3m2(T(gate, dev), T(up, dev), clip_ratio=0.9)
    assert_same(H(q6), H(q.quarot_pack_e3m2(codes)), f"swiglu e3m2 codes n={n}")
    assert_same(H(s6).view(np.uint16), rs.view(np.uint16), f"swiglu e3m2 scales n={n}")


@pytest.mark.parametrize("n,rows", [(1728, 1024), (1728, 1025), (2752, 2049)])
def test_largem_swiglu_row_counts(dev, orc, n, rows):
    """512 blocks up to 1024 rows, 1024 blocks past them: every row is written
    once, also the wide ones of a block's second and third turn."""
    import paper_2404_00456_amd as q
    say(f"largem swiglu row counts n={n} rows={rows}")
    rng = np.random.default_rng(rows)
    gate = (rng.standard_normal((rows, n)) * 1.5).astype(np.float16)
    up = rng.standard_normal((rows, n)).astype(np.float16)
    up[::7] *= np.float16(300)
    up[rows - 1, 0], gate[rows - 1, 0] = 60.0, 10.0
    rq, rs = orc.swiglu_quant_int4(gate, up, rotate=True, clip=0.9)
    codes, scale = q.quarot_swiglu_quant_int4(T(gate, dev), T(up, dev), clip_ratio=0.9)
    assert_same(H(codes), rq, f"swiglu int4 codes n={n} rows={rows}")
    assert_same(H(scale).view(np.uint16), rs.view(np.uint16), f"swiglu int4 scales n={n} rows={rows}")


def test_swiglu_infinite_gate(dev):
    """silu(+inf) = inf and silu(-inf) = -inf / (1 + e^88) = -inf in the
    binary32 recipe; NaN stays NaN."""
    import paper_2404_00456_amd as q
    g = np.array([np.inf, -np.inf, np.nan, np.inf, -np.inf, 3.0, 0.0, -0.0], np.float16)
    u = np.array([2.0, 2.0, 2.0, -2.0, -2.0, np.inf, 1.0, 1.0], np.float16)
    got = H(q.quarot_swiglu(T(g, dev), T(u, dev)))
    ref = np.array([np.inf, -np.inf, np.nan, -np.inf, np.inf, np.inf, 0.0, -0.0], np.float16)
    assert np.isnan(got[2])
    assert_same(got[[0, 1, 3, 4, 5, 6, 7]].view(np.uint16),
                ref[[0, 1, 3, 4, 5, 6, 7]].view(np.uint16), "infinite gates")


@pytest.mark.parametrize("n", [1728, 3456, 6912, 13824, 2752, 5504, 11008])
def test_largem_past_the_largest_fp16(dev, orc, n):
    """A product silu(g) u past the largest fp16 is an infinity in h.  The
    rotation reads an exponent of all ones as the next binade (infinity as
    65536), so that such a row keeps its codes: those of half the row, with
    twice its scale."""
    import paper_2404_00456_amd as q
    say(f"largem past fp16 n={n}")
    rng = np.random.default_rng(n)
    half = (rng.standard_normal((6, n)) * 40).astype(np.float16)
    half[np.abs(half) < 1] = 1  # exact when halved or doubled
    half[0, 5] = half[1, n - 1] = 32768
    signs = rng.choice(np.array([-1, 1], np.float16), n)
    half[1, ::301] = 32768 * signs[::301]
    half[2] = 32768 * signs
    half[3, ::7] = (32768 + 32 * 777) * signs[::7]  # a NaN's significand, doubled
    half[4, ::11] = 32752 * signs[::11]  # the largest fp16, doubled
    with np.errstate(over="ignore"):
        x = half * np.float16(2)
    top = np.abs(half) >= 32768  # the exponent's last step, same significand
    x[top] = (half[top].view(np.uint16) + 0x0400).view(np.float16)
    rq, rs = orc.quant_int4(half, rotate=True, clip=0.9)
    twice = (rs.astype(np.float32) * 2).astype(np.float16).view(np.uint16)
    codes, scale = q.quarot_quant_int4(T(x, dev), clip_ratio=0.9)
    assert_same(H(codes), rq, f"codes n={n}")
    assert_same(H(scale).view(np.uint16), twice, f"scales n={n}")
    # silu(64) = 64 in binary32, so h = 64 u, infinite from |u| = 1024 on
    up = half[[0, 1, 2, 4, 5]] / np.float16(32)
    rq, rs = orc.swiglu_quant_int4(np.full_like(up, 32), up, rotate=True, clip=0.9)
    twice = (rs.astype(np.float32) * 2).astype(np.float16).view(np.uint16)
    codes, scale = q.quarot_swiglu_quant_int4(T(np.full_like(up, 64), dev), T(up, dev),
                                              clip_ratio=0.9)
    assert_same(H(codes), rq, f"swiglu codes n={n}")
    assert_same(H(scale).view(np.uint16), twice, f"swiglu scales n={n}")
