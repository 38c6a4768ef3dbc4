"""The calls that a program serving a QuaRot model makes of this library, as
measured cases: the 4-bit linear layers from one token to a full prefill, the
two places where the rotation is online (before down_proj and before out_proj),
the 8-bit and group-wise variants, and the 4-bit KV cache filled and read.

A case is a dict of plain values; ``prepare`` makes its inputs and weights on
the GPU from a seed, ``run`` is one pass through the public entry points and
``exact`` the same result in binary64 from plain torch.
"""
import math

import torch

import paper_2404_00456_amd as quarot

DEV = "cuda"
CLIP_ACT = 0.9   # clipping ratio of the activations (paper, section 5, Setup)
CLIP_KV = 0.95   # and of the KV cache

# Layer widths of the paper's Llama-2 7B, 13B and 70B timings (in -> out).
UP = [(4096, 11008), (8192, 28672)]
DOWN = [(11008, 4096), (13824, 5120), (28672, 8192)]
ATTN_OUT = [(32, 4096), (64, 8192)]  # heads of 128, width


def _linear(name, fmt, M, K, N, **more):
    return dict(name=name, kind="linear", fmt=fmt, M=M, K=K, N=N, **more)


def listed():
    return [
        # one new token through an attention projection of the 7B model: the
        # smallest call, latency and the read of 12.6 MB of weights
        _linear("linear_1tok_7b", "e3m2", 1, 4096, 4096),
        # 16 sequences decoding together, up projection of the 70B model:
        # 176 MB of weights read for little arithmetic
        _linear("linear_16tok_70b_up", "e3m2", 16, 8192, 28672),
        # 61 sequences decoding, down projection with its SwiGLU and online
        # Hadamard (H_1024 x H_28)
        dict(name="ffn_down_61tok_70b", kind="ffn_down", M=61, K=28672, N=8192),
        # one short prompt of odd length, up projection of the 7B model
        _linear("linear_333tok_7b_up", "e3m2", 333, 4096, 11008),
        # one full prompt of the 7B model, down projection (H_64 x H_172)
        dict(name="ffn_down_2048tok_7b", kind="ffn_down", M=2048, K=11008, N=4096),
        # prefill of 8 x 2048 tokens, up projection of the 70B model: the
        # largest call
        _linear("linear_16384tok_70b_up", "e3m2", 16384, 8192, 28672),
        # out projection of the 7B model: Hadamard across heads, then the
        # packed int4 operands (the smaller weight format)
        dict(name="out_proj_1777tok_7b", kind="out_proj", M=1777, heads=32, N=4096),
        # 8-bit codes, down projection of the 13B model (H_128 x H_108),
        # a batch of short prompts
        _linear("w8a8_517tok_13b_down", "int8", 517, 13824, 5120),
        # a scale per 128 input channels, one full prompt of the 7B model
        _linear("grouped_2048tok_7b_up", "grouped", 2048, 4096, 11008, group=128),
        # a prompt's keys (rotated) and values (already rotated by the fused
        # weights) go into the cache: 4 sequences of 2048, 64 heads
        dict(name="kv_prefill_4x2048", kind="kv_fill", rows=4 * 64 * 2048, D=128, group=128),
        # one decode step: append, query rotation, attention over the cache;
        # 16 sequences of 32 heads near 2047 tokens
        dict(name="decode_16seq_32heads", kind="decode", B=16, heads=32, kv_heads=32, seq=2047,
             D=128, group=128),
        # and 5 sequences whose 64 query heads share 8 KV heads
        dict(name="decode_5seq_64on8heads", kind="decode", B=5, heads=64, kv_heads=8, seq=4099,
             D=128, group=128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "ffn_down", "ffn_down", "out_proj",
                       "variant", "kv_fill", "decode", "decode"])
    if kind == "linear":
        K, N = rng.choice(UP + [(4096, 4096), (8192, 8192)])
        # up to the largest listed prefill; output channels whole or one
        # GPU's slice of them
        return dict(kind="linear", fmt=rng.choice(["e3m2", "e3m2", "int4"]),
                    M=_log_int(rng, 1, 12000), K=K, N=N // rng.choice([1, 1, 2, 4]))
    if kind == "ffn_down":
        K, N = rng.choice(DOWN)
        return dict(kind="ffn_down", M=_log_int(rng, 1, 8192), K=K, N=N)
    if kind == "out_proj":
        heads, N = rng.choice(ATTN_OUT)
        return dict(kind="out_proj", M=_log_int(rng, 1, 8192), heads=heads, N=N)
    if kind == "variant":
        fmt = rng.choice(["int8", "grouped"])
        K, N = rng.choice([(4096, 11008), (4096, 4096), (13824, 5120)])
        case = dict(kind="linear", fmt=fmt, M=_log_int(rng, 1, 4096), K=K, N=N)
        if fmt == "grouped":
            case["group"] = rng.choice([64, 128, 128, 256])
        return case
    if kind == "kv_fill":
        D = rng.choice([64, 128, 128])
        return dict(kind="kv_fill", rows=_log_int(rng, 500, 1 << 20), D=D,
                    group=rng.choice([D, D, 64]))
    heads, kv_heads = rng.choice([(32, 32), (40, 40), (64, 64), (64, 8), (32, 8)])
    D = rng.choice([64, 128, 128, 128])
    return dict(kind="decode", B=_log_int(rng, 1, 24), heads=heads, kv_heads=kv_heads,
                seq=_log_int(rng, 60, 8000), D=D, group=rng.choice([D, D, 64]))


# ---- inputs ----------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _activations(g, rows, n):
    """Normal rows with 1% outlier channels (x 50), the same for every token."""
    x = torch.randn((rows, n), generator=g, device=DEV, dtype=torch.float32)
    idx = torch.randperm(n, generator=g, device=DEV)[:max(1, round(0.01 * n))]
    x[:, idx] *= 50.0
    return x.half()


def _weight(g, N, K):
    return torch.empty((N, K), device=DEV, dtype=torch.float16).normal_(0.0, 0.02, generator=g)


def _gate_up(g, M, K):
    gate = torch.randn((M, K), generator=g, device=DEV).mul_(1.5).half()
    up = _activations(g, M, K)
    return gate, up


def _inputs(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "linear":
        return _activations(g, case["M"], case["K"]), _weight(g, case["N"], case["K"])
    if kind == "ffn_down":
        gate, up = _gate_up(g, case["M"], case["K"])
        return gate, up, _weight(g, case["N"], case["K"])
    if kind == "out_proj":
        K = case["heads"] * 128
        z = torch.randn((case["M"], K), generator=g, device=DEV).half()
        return z, _weight(g, case["N"], K)

    def heads(rows, tokens, D):  # two outlier dims per head row (x 20)
        t = torch.randn((rows, tokens, D), generator=g, device=DEV, dtype=torch.float32)
        at = torch.randint(0, D, (rows, 1, 2), generator=g, device=DEV).expand(rows, tokens, 2)
        return t.scatter_(2, at, t.gather(2, at) * 20.0).half()

    D = case["D"]
    if kind == "kv_fill":
        r = case["rows"]
        return heads(1, r, D).reshape(r, D), heads(1, r, D).reshape(r, D)
    nkv, s_max = case["B"] * case["kv_heads"], _s_max(case)
    q = torch.randn((case["B"] * case["heads"], D), generator=g, device=DEV).half()
    new = [torch.randn((nkv, D), generator=g, device=DEV).half() for _ in range(2)]
    return q, new[0], new[1], heads(nkv, s_max, D), heads(nkv, s_max, D)


def _s_max(case):
    return -(-(case["seq"] + 1) // 256) * 256  # cache capacity, whole pages of 256


def prepare(case, seed):
    kind = case["kind"]
    t = _inputs(case, seed)
    s = dict(case=case)
    if kind == "linear":
        x, w = t
        s["x"] = x
        if case["fmt"] == "e3m2":
            s["w"], s["sw"] = quarot.prepare_weight_e3m2(w)
        elif case["fmt"] == "int4":
            s["w"], s["sw"] = quarot.prepare_weight(w)
        elif case["fmt"] == "int8":
            s["w"], s["sw"] = quarot.quarot_quant_int8(w, bits=8)
        else:
            s["w"], s["sw"] = quarot.quarot_quant_int4_grouped(w, group=case["group"])
    elif kind == "ffn_down":
        s["gate"], s["up"] = t[:2]
        s["w"], s["sw"] = quarot.prepare_weight_e3m2(t[2])
    elif kind == "out_proj":
        # W_out's columns take the head-wise rotation offline
        s["z"] = t[0]
        s["w"], s["sw"] = quarot.quarot_hadamard_heads_quant_int4(t[1], case["heads"])
    elif kind == "kv_fill":
        s["k"], s["v"] = t
    else:
        s["q"], s["kn"], s["vn"] = t[:3]
        s["k"] = quarot.quarot_kv_quant(t[3], group=case["group"], clip_ratio=CLIP_KV)
        s["v"] = quarot.quarot_kv_quant(t[4], group=case["group"], rotate=False,
                                        clip_ratio=CLIP_KV)
    return s


# ---- one pass --------------------------------------------------------------

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "linear":
        if case["fmt"] == "e3m2":
            return quarot.quarot_linear_e3m2(s["x"], s["w"], s["sw"], clip_ratio=CLIP_ACT)
        if case["fmt"] == "int4":
            return quarot.quarot_linear(s["x"], s["w"], s["sw"], clip_ratio=CLIP_ACT)
        if case["fmt"] == "int8":
            return quarot.quarot_linear_w8a8(s["x"], s["w"], s["sw"], clip_ratio=CLIP_ACT, bits=8)
        return quarot.quarot_linear_w4a4_grouped(s["x"], s["w"], s["sw"], group=case["group"],
                                                 clip_ratio=CLIP_ACT)
    if kind == "ffn_down":
        x6, sx = quarot.quarot_swiglu_quant_e3m2(s["gate"], s["up"], clip_ratio=CLIP_ACT)
        return quarot.quarot_w4a4_gemm_e3m2(x6, sx, s["w"], s["sw"])
    if kind == "out_proj":
        xq, sx = quarot.quarot_hadamard_heads_quant_int4(s["z"], case["heads"],
                                                         clip_ratio=CLIP_ACT)
        return quarot.quarot_w4a4_gemm(xq, sx, s["w"], s["sw"])
    G = case["group"]
    if kind == "kv_fill":
        k = quarot.quarot_kv_quant(s["k"], group=G, clip_ratio=CLIP_KV)
        v = quarot.quarot_kv_quant(s["v"], group=G, rotate=False, clip_ratio=CLIP_KV)
        return k, v
    pos = case["seq"] - 1
    quarot.quarot_kv_append(s["kn"], *s["k"], pos, group=G, clip_ratio=CLIP_KV)
    quarot.quarot_kv_append(s["vn"], *s["v"], pos, group=G, rotate=False, clip_ratio=CLIP_KV)
    q = quarot.quarot_hadamard(s["q"])
    out = quarot.quarot_kv_decode_attention(q, s["k"], s["v"], case["seq"], group=G)
    return out, s["k"], s["v"]


# ---- what a pass cannot do without -----------------------------------------

def work(case):
    kind = case["kind"]
    if kind in ("linear", "ffn_down", "out_proj"):
        M, N = case["M"], case["N"]
        K = case["heads"] * 128 if kind == "out_proj" else case["K"]
        fmt = {"ffn_down": "e3m2", "out_proj": "int4"}.get(kind) or case["fmt"]
        per = {"e3m2": 0.75, "int4": 0.5, "int8": 1.0, "grouped": 0.5}[fmt]
        scales = 2 * N * (K // case["group"] if fmt == "grouped" else 1)
        inputs = 2 * M * K * (2 if kind == "ffn_down" else 1)
        return {"bytes": inputs + per * N * K + scales + 2 * M * N, "flops": 2.0 * M * N * K}
    D, G = case["D"], case["group"]
    code_row = D // 2 + 4 * (D // G)  # codes, scale and zero of one head row
    if kind == "kv_fill":
        r = case["rows"]
        return {"bytes": 2 * r * (2 * D + code_row), "flops": r * D * math.log2(D)}
    nq, nkv = case["B"] * case["heads"], case["B"] * case["kv_heads"]
    return {"bytes": 2 * nkv * case["seq"] * code_row + 2 * nkv * 2 * D + 2 * nq * 2 * D,
            "flops": 4.0 * nq * case["seq"] * D}


def tolerance(case):
    # The library's header fixes the codes, scales and outputs of every call
    # but the attention to the bit.
    if case["kind"] != "decode":
        return "exact"
    return {"rel": 2e-3, "max": 2e-2, "differ": 0.0}


# ---- the same in binary64 --------------------------------------------------

def _hadamard_factor(m):
    """H_m, m in {1, 12, 20, 28, 108, 172}, from the published constructions."""
    if m == 1:
        return torch.ones((1, 1), dtype=torch.float64)

    def chi(a, p):
        a %= p
        return 0 if a == 0 else (1 if pow(a, (p - 1) // 2, p) == 1 else -1)

    if m in (12, 20, 108):  # Paley I
        p = m - 1
        h = [[(1 if r == s else 0) + (0 if r == s == 0 else 1 if r == 0 else -1 if s == 0
                                      else chi(s - r, p)) for s in range(m)] for r in range(m)]
        return torch.tensor(h, dtype=torch.float64)
    if m == 28:  # Paley II
        c = torch.tensor([[0 if r == s else 1 if 0 in (r, s) else chi(s - r, 13)
                           for s in range(14)] for r in range(14)], dtype=torch.float64)
        a = torch.tensor([[1.0, 1.0], [1.0, -1.0]], dtype=torch.float64)
        b = torch.tensor([[1.0, -1.0], [-1.0, -1.0]], dtype=torch.float64)
        return torch.kron(c, a) + torch.kron(torch.eye(14, dtype=torch.float64), b)
    # 172: Goethals-Seidel array of four circulants of order 43, whose rows
    # are unions of order-6 cyclotomic classes
    p, cls, v = 43, {}, 1
    for t in range(p - 1):
        cls[v], v = t % 6, v * 3 % p
    mats = []
    for first, minus in ((-1, (0, 1)), (1, (0, 1, 3)), (1, (0, 1, 3)), (1, (0, 2, 3))):
        x = [first] + [-1 if cls[j] in minus else 1 for j in range(1, p)]
        mats.append(torch.tensor([[x[(c - i) % p] for c in range(p)] for i in range(p)],
                                 dtype=torch.float64))
    A, B, C, D = mats
    R = torch.eye(p, dtype=torch.float64).flip(0)
    rows = [[A, B @ R, C @ R, D @ R], [-B @ R, A, D.T @ R, -C.T @ R],
            [-C @ R, -D.T @ R, A, B.T @ R], [-D @ R, C.T @ R, -B.T @ R, A]]
    return torch.cat([torch.cat(r, 1) for r in rows], 0)


def _wht(t):
    """Walsh-Hadamard transform (Sylvester order) of dimension 1 of [r, a, b]."""
    r, a, b = t.shape
    h = 1
    while h < a:
        v = t.view(r, a // (2 * h), 2, h, b)
        t = torch.stack((v[:, :, 0] + v[:, :, 1], v[:, :, 0] - v[:, :, 1]), 2).view(r, a, b)
        h *= 2
    return t


def _rotate(x):
    rows, n = x.shape
    m = next(m for m in (1, 12, 20, 28, 108, 172) if n % m == 0 and (n // m) & (n // m - 1) == 0)
    t = x.double()
    if m > 1:
        t = t.reshape(-1, m) @ _hadamard_factor(m).to(x.device)
    return _wht(t.reshape(rows, n // m, m)).reshape(rows, n) / math.sqrt(n)


def _sym(y, clip, qmax=7):
    """(codes, scales) of binary64 rows: symmetric, a scale per row, stored
    in binary16."""
    s = (y.abs().amax(-1, keepdim=True) * clip / qmax).half().double()
    q = torch.where(s > 0, (y / torch.where(s > 0, s, torch.ones_like(s))).round(),
                    torch.zeros_like(y))
    return q.clamp_(-qmax - 1, qmax), s


def _chunks(x, f, rows=1024):
    parts = [f(x[i:i + rows]) for i in range(0, x.shape[0], rows)]
    return [torch.cat(p, 0) for p in zip(*parts)]


def _kv(x, group, rotate):
    """(codes, scale, zero), codes as values, scale and zero in binary16."""
    lead, D = x.shape[:-1], x.shape[-1]

    def f(r):
        y = _rotate(r) if rotate else r.double()
        y = y.view(-1, D // group, group)
        mx, mn = y.amax(-1, keepdim=True) * CLIP_KV, y.amin(-1, keepdim=True) * CLIP_KV
        s, z = ((mx - mn) / 15).half().double(), mn.half().double()
        q = torch.where(s > 0, ((y - z) / torch.where(s > 0, s, torch.ones_like(s))).round(),
                        torch.zeros_like(y)).clamp_(0, 15)
        return q.to(torch.int8), s.squeeze(-1), z.squeeze(-1)

    q, s, z = _chunks(x.reshape(-1, D), f, 1 << 16)
    return (q.view(lead + (D // group, group)), s.view(lead + (D // group,)),
            z.view(lead + (D // group,)))


def exact(case, seed):
    kind = case["kind"]
    t = _inputs(case, seed)
    if kind == "linear":
        x, w = t
        if case["fmt"] == "grouped":
            G = case["group"]

            def grouped(clip):
                def f(r):
                    y = _rotate(r)
                    q, s = _sym(y.view(y.shape[0], -1, G), clip)
                    return ((q * s).view(y.shape),)
                return f
            xd, = _chunks(x, grouped(CLIP_ACT))
            wd, = _chunks(w, grouped(1.0))
            return xd @ wd.T
        qmax = 127 if case["fmt"] == "int8" else 7
        xq, sx = _chunks(x, lambda r: _sym(_rotate(r), CLIP_ACT, qmax))
        wq, sw = _chunks(w, lambda r: _sym(_rotate(r), 1.0, qmax))
        return (xq @ wq.T) * sx * sw.view(1, -1)
    if kind == "ffn_down":
        def h(r):
            g, u = r[:, 0].double(), r[:, 1].double()
            return (g / (1.0 + torch.exp(-g)) * u).half()
        xq, sx = _chunks(torch.stack(t[:2], 1), lambda r: _sym(_rotate(h(r)), CLIP_ACT))
        wq, sw = _chunks(t[2], lambda r: _sym(_rotate(r), 1.0))
        return (xq @ wq.T) * sx * sw.view(1, -1)
    if kind == "out_proj":
        nh = case["heads"]

        def across(r):
            return _wht(r.double().view(r.shape[0], nh, 128)).view(r.shape) / math.sqrt(nh)
        xq, sx = _chunks(t[0], lambda r: _sym(across(r), CLIP_ACT))
        wq, sw = _chunks(t[1], lambda r: _sym(across(r), 1.0))
        return (xq @ wq.T) * sx * sw.view(1, -1)
    G = case["group"]
    if kind == "kv_fill":
        _, ks, kz = _kv(t[0], G, True)
        _, vs, vz = _kv(t[1], G, False)
        return (None, ks, kz), (None, vs, vz)
    q, kn, vn, k, v = t
    seq, D = case["seq"], case["D"]
    k[:, seq - 1], v[:, seq - 1] = kn, vn
    qk, ks, kz = _kv(k, G, True)
    qv, vs, vz = _kv(v, G, False)
    qr = _rotate(q).half().double()  # the query row is binary16 between the calls
    rep = case["heads"] // case["kv_heads"]
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    for r in range(k.shape[0]):  # one cache row: its rep query rows
        kh = (qk[r, :seq].double() * ks[r, :seq, :, None] + kz[r, :seq, :, None]).view(seq, D)
        vh = (qv[r, :seq].double() * vs[r, :seq, :, None] + vz[r, :seq, :, None]).view(seq, D)
        p = torch.softmax(qr[r * rep:(r + 1) * rep] @ kh.T / math.sqrt(D), -1)
        out[r * rep:(r + 1) * rep] = p @ vh
    return out, (None, ks, kz), (None, vs, vz)
