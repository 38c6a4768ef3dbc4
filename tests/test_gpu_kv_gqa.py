"""GPU parity of decode attention at head_dim 128 with one scale per cached
row, where several query rows share a cache row and where a row's tokens are
split over blocks, against the CPU oracle.

The bound: the kernel keeps 22 bits of the weights times the value scales (of
those below 2^-3 what is above 2^-25, errors that cancel over the tokens),
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


# one query to 33 per cache row; few rows, so a block per query row takes them
# (tests/native/attn_plan_check.cpp)
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


# blocks of 8 query rows (csrc/kv_attention.hip, k_kv_attn_gqa): one block to
# five per cache row, whole and short ones, four and eight waves, a token, a
# wave's 32, a block's 128 and 256 and their edges, whole rows and split ones.
# The host check of the plan holds these calls to that kernel.
SHARED = [(130, 2, 129), (130, 2, 257), (130, 2, 2049), (130, 3, 255), (130, 5, 65),
          (130, 7, 257), (130, 8, 17), (130, 8, 33), (130, 9, 129), (130, 9, 255),
          (130, 16, 33), (130, 17, 2049), (130, 33, 1), (130, 33, 257), (520, 2, 33),
          (520, 2, 513), (520, 3, 17), (520, 5, 1), (520, 7, 1025), (60, 8, 513),
          (60, 8, 1025), (60, 5, 2049), (300, 2, 1025), (300, 3, 2049)]


@pytest.mark.parametrize("nkv,rep,seq", SHARED)
def test_shared_cache_rows(dev, orc, nkv, rep, seq):
    run(dev, orc, nkv, rep, seq + 5, seq)


def test_shared_rows_growing_scores(dev, orc):
    rng = np.random.default_rng(9)
    k, v = rand_cache(rng, 60, 1500, 128, 128), rand_cache(rng, 60, 1500, 128, 128)
    k[2][:] = np.linspace(-3, 3, 1500).astype(np.float16)[None, :, None]
    q = (0.25 + 0.5 * np.abs(rng.standard_normal((480, 128)))).astype(np.float16)
    run(dev, orc, 60, 8, 1500, 1500, k, v, q)


def test_shared_rows_infinite_scores_and_scales(dev, orc):
    """Tokens whose zero point is -inf weigh nothing, also where they fill whole
    steps of a wave; an infinite value scale gives its infinity."""
    import paper_2404_00456_amd as qq
    rng = np.random.default_rng(10)
    n, seq, cut = 130, 600, 333
    k, v = rand_cache(rng, n, seq, 128, 128), rand_cache(rng, n, seq, 128, 128)
    q = np.abs(rng.standard_normal((8 * n, 128))).astype(np.float16)
    k[2][:, :cut] = -np.inf
    full = H(qq.quarot_kv_decode_attention(T(q, dev), tuple(T(x, dev) for x in k),
                                           tuple(T(x, dev) for x in v), seq))
    part = orc.kv_attention(q, tuple(np.ascontiguousarray(x[:, cut:]) for x in k),
                            tuple(np.ascontiguousarray(x[:, cut:]) for x in v), seq - cut, group=128)
    d = np.abs(full.astype(np.float64) - part.astype(np.float64))
    assert np.all(d <= 2.0 ** -10 * np.abs(part.astype(np.float64)) + 2.0 ** -16 * 9.0)
    for inf in (np.inf, -np.inf):
        k, v = rand_cache(rng, n, 40, 128, 128), rand_cache(rng, n, 40, 128, 128)
        v[0][:, 0], v[1][:, 0] = 0x31, inf
        q = (rng.standard_normal((8 * n, 128)) * 0.1).astype(np.float16)
        out = H(qq.quarot_kv_decode_attention(T(q, dev), tuple(T(x, dev) for x in k),
                                              tuple(T(x, dev) for x in v), 40))
        assert np.all(out == inf)


@pytest.mark.parametrize("nkv,rep,seq", [(16, 1, 3000), (300, 1, 2000), (60, 8, 1500),
                                         (130, 2, 2049), (8, 8, 1000)])
def test_same_bits_again(dev, nkv, rep, seq):
    """The same call gives the same bits, whatever its workspace held."""
    import torch
    import paper_2404_00456_amd as qq
    rng = np.random.default_rng(nkv + seq)
    k, v = rand_cache(rng, nkv, seq, 128, 128), rand_cache(rng, nkv, seq, 128, 128)
    k, v = tuple(T(x, dev) for x in k), tuple(T(x, dev) for x in v)
    q = T((rng.standard_normal((nkv * rep, 128)) * 0.5).astype(np.float16), dev)
    first = qq.quarot_kv_decode_attention(q, k, v, seq)
    need = int(qq.lib().quarot_kv_attention_workspace_size(nkv * rep, seq, 128))
    for fill in (0xFF, 0x7F, 0x00):
        ws = torch.full((max(need, 16),), fill, dtype=torch.uint8, device=dev)
        again = qq.quarot_kv_decode_attention(q, k, v, seq, workspace=ws)
        assert torch.equal(first.view(torch.int16), again.view(torch.int16)), fill


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
