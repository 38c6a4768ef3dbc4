"""GPU parity of decode attention at head_dim 128 with one scale per cached
row, where several query rows share a cache row and where a row's tokens are
split over blocks, against the CPU oracle.

The bound: the kernel keeps 22 bits of the weights times the value scales,
accumulates in binary32 and rounds the result to fp16 (2^-11 of it), so with
weights summing to 1 the error is at most 2^-11 |out| plus binary32 terms of
the size of scale * code, at most 0.6 * 15 = 9 here: exp and the scores'
rounding give each weight some 2^-18, the sums less.  2^-16 * 9 covers them.
The oracle's own output is fp16 too (another 2^-11 |out|)."""
import numpy as np
import pytest

from test_gpu_kv_decode import rand_cache
from test_gpu_parity import H, T, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2404_00456_amd as q
    q.lib()
    return torch.device("cuda:0")


def run(dev, orc, nkv, rep, s_max, seq, k=None, v=None, q=None):
    import paper_2404_00456_amd as qq
    rng = np.random.default_rng(nkv * 131 + rep * 17 + seq)
    k = k or rand_cache(rng, nkv, s_max, 128, 128)
    v = v or rand_cache(rng, nkv, s_max, 128, 128)
    q = (rng.standard_normal((nkv * rep, 128)) * 0.5).astype(np.float16) if q is None else q
    got = H(qq.quarot_kv_decode_attention(T(q, dev), tuple(T(x, dev) for x in k),
                                          tuple(T(x, dev) for x in v), seq)).astype(np.float64)
    ref = orc.kv_attention(q, k, v, seq, group=128).astype(np.float64)
    err = np.abs(got - ref)
    say(f"nkv={nkv} rep={rep} seq={seq}: max err {err.max():.3g}, norm "
        f"{np.linalg.norm(err) / np.linalg.norm(ref):.3g}")
    assert np.all(err <= 2.0 ** -10 * np.abs(ref) + 2.0 ** -16 * 9.0), err.max()


# one query to five blocks of 8 per cache row
@pytest.mark.parametrize("rep", [1, 2, 3, 5, 7, 8, 9, 16, 17, 33])
# a token, part of a wave's 32, its edges, a block's 256 and its edges
@pytest.mark.parametrize("seq", [1, 17, 32, 33, 255, 257])
def test_queries_per_cache_row(dev, orc, rep, seq):
    run(dev, orc, 2, rep, seq + 6, seq)


# both sides of the split of a row: whole, two blocks, many, a last short chunk
@pytest.mark.parametrize("nkv,rep,seq", [
    (3, 1, 600), (3, 1, 610), (3, 1, 4099), (100, 1, 1201), (128, 1, 1199), (128, 1, 1217),
    (129, 1, 1500), (256, 1, 513), (2, 4, 606), (2, 8, 1025), (5, 20, 2049), (40, 8, 4099)])
def test_splits_of_a_row(dev, orc, nkv, rep, seq):
    run(dev, orc, nkv, rep, seq + seq % 3, seq)


@pytest.mark.parametrize("rep", [1, 8])
def test_growing_scores_rescale(dev, orc, rep):
    """Scores that rise with the token: every step raises the running maximum."""
    rng = np.random.default_rng(rep)
    k, v = rand_cache(rng, 2, 1500, 128, 128), rand_cache(rng, 2, 1500, 128, 128)
    k[2][:] = np.linspace(-3, 3, 1500).astype(np.float16)[None, :, None]
    q = (0.25 + 0.5 * np.abs(rng.standard_normal((2 * rep, 128)))).astype(np.float16)
    run(dev, orc, 2, rep, 1500, 1500, k, v, q)


@pytest.mark.parametrize("rep", [1, 8])
def test_tokens_of_infinite_negative_score(dev, rep):
    """Zero points of -inf give scores of -inf: such tokens weigh nothing, also
    where they fill whole steps of a wave."""
    import paper_2404_00456_amd as qq
    rng = np.random.default_rng(50 + rep)
    k, v = rand_cache(rng, 2, 2000, 128, 128), rand_cache(rng, 2, 2000, 128, 128)
    q = np.abs(rng.standard_normal((2 * rep, 128))).astype(np.float16)
    cut = tuple(x[:, 1111:].copy() for x in k), tuple(x[:, 1111:].copy() for x in v)
    k[2][:, :1111] = -np.inf
    full = H(qq.quarot_kv_decode_attention(T(q, dev), tuple(T(x, dev) for x in k),
                                           tuple(T(x, dev) for x in v), 2000))
    part = H(qq.quarot_kv_decode_attention(T(q, dev), tuple(T(x, dev) for x in cut[0]),
                                           tuple(T(x, dev) for x in cut[1]), 889))
    d = np.abs(full.astype(np.float64) - part.astype(np.float64))
    assert np.all(d <= 2.0 ** -10 * np.abs(part.astype(np.float64)) + 2.0 ** -16 * 9.0)


@pytest.mark.parametrize("rep", [1, 8])
@pytest.mark.parametrize("inf", [np.inf, -np.inf])
def test_infinite_value_scale(dev, rep, inf):
    """An infinite scale of a value row whose codes are all positive: the
    output is that infinity, not the NaN of its parts' difference."""
    import paper_2404_00456_amd as qq
    rng = np.random.default_rng(70 + rep)
    k, v = rand_cache(rng, 2, 40, 128, 128), rand_cache(rng, 2, 40, 128, 128)
    v[0][:, 0], v[1][:, 0] = 0x31, inf
    q = (rng.standard_normal((2 * rep, 128)) * 0.1).astype(np.float16)
    out = H(qq.quarot_kv_decode_attention(T(q, dev), tuple(T(x, dev) for x in k),
                                          tuple(T(x, dev) for x in v), 40))
    assert np.all(out == inf)


def test_more_rows_than_a_wide_launch_holds(dev, orc):
    """2^23 rows of one token: out is the dequantized value row."""
    import torch
    import paper_2404_00456_amd as qq
    n = (1 << 23) + 3
    g = torch.Generator(device=dev).manual_seed(3)
    q = torch.ones((n, 128), dtype=torch.float16, device=dev)
    codes = torch.randint(0, 256, (n, 1, 64), dtype=torch.uint8, device=dev, generator=g)
    scale = torch.rand((n, 1, 1), device=dev, generator=g).half()
    zero = -scale
    out = qq.quarot_kv_decode_attention(q, (codes, scale, zero), (codes, scale, zero), 1)
    for rows in (slice(0, 64), slice(n - 64, n)):
        c = codes[rows, 0].int()
        x = torch.stack((c & 15, c >> 4), dim=2).reshape(-1, 128).double()
        ref = x * scale[rows, 0].double() + zero[rows, 0].double()
        assert ((out[rows].double() - ref).abs() <= 2.0 ** -11 * ref.abs() + 2.0 ** -16 * 15.0).all()
