"""The calls whose time on one MI355X is followed over the life of this library, and what they compute.

A case is a call that a serving or finetuning program makes through the package's entry points (`binding`, `host`),
at the layer shapes of the 8B, 14B and 32B models the library is built for, or at the small fp32 shape.  `listed()` are
the cases that are followed; `draw()` gives others of the same ranges.  `exact()` is the same computation in 64-bit
torch, with nothing of this package in it.

Weights N(0, 0.02), norm gains 1 + N(0, 0.02), biases N(0, 0.02), LoRA A N(0, 0.02), LoRA B N(0, 0.01), layer inputs and
cached keys / values N(0, 1): rounded to the configuration's storage type.  Context lengths are a function of the case
alone (quantiles of its length law); which physical pages hold them, and every value, comes from the seed.
"""
import math
from types import SimpleNamespace

import torch

from paper_2402_18789_amd import binding as B
from paper_2402_18789_amd import host as HH

ALL = ("q", "k", "v", "o", "gate", "up", "down")
DECODE, PREFILL, FINETUNE = 0, 1, 2


class _Cfg(SimpleNamespace):
    """layer shape: what `host` reads of a layer configuration"""

    q_dim = property(lambda c: c.n_q_heads * c.head_dim)
    kv_dim = property(lambda c: c.n_kv_heads * c.head_dim)


_MODELS = {
    # hidden, query heads, kv heads, head_dim, ffn, dtype, eps, rope base, LoRA rank and targets, QKV bias, vocabulary
    "tiny": (256, 4, 4, 64, 688, "f32", 1e-5, 1e4, 8, ("q", "v", "down"), False, 1000),
    "8b": (4096, 32, 8, 128, 14336, "bf16", 1e-5, 5e5, 16, ("q", "k", "v", "o", "down"), False, 128256),
    "14b": (5120, 40, 8, 128, 13824, "bf16", 1e-6, 1e6, 16, ALL, True, 152064),
    "32b": (5120, 40, 8, 128, 27648, "bf16", 1e-6, 1e6, 32, ALL, True, 152064),
}


def _cfg(case):
    h, nq, nkv, d, f, dt, eps, theta, r, targets, bias, vocab = _MODELS[case["model"]]
    if case["op"] == "ia3":
        targets = ()
    return _Cfg(hidden=h, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=f, dtype=dt, rms_eps=eps, rope_theta=theta,
                page_size=16, lora_rank=r, lora_targets=targets, lora_scale=2.0, qkv_bias=bias, vocab=vocab)


# ---- the cases ------------------------------------------------------------------------------------------------------

def _batch(decode=0, lo=0, hi=0, median=0, sigma=0.0, prefill="", window=0, seq=0, adapters=1):
    """decode requests with contexts uniform in lo..hi (median 0) or log-normal, clipped to lo..hi; prefill chunks
    "tokens@start" separated by blanks; the last `window` tokens of a finetune sequence of `seq` tokens; adapters > 1:
    the inference requests take ids -1, 0, 1, ... in turn, else they run the base model."""
    return {"decode": decode, "lo": lo, "hi": hi, "median": median, "sigma": sigma, "prefill": prefill, "window": window,
            "seq": seq, "adapters": adapters}


def listed():
    return [
        # an interactive server with a handful of users: one layer of a decode step, where weights are the bytes
        dict(name="decode_8b_8", op="forward", model="8b", **_batch(decode=8, lo=256, hi=1024)),
        # a decode step of a server of several adapters on one backbone
        dict(name="decode_14b_48_adapters", op="forward", model="14b", **_batch(decode=48, lo=200, hi=2048, adapters=4)),
        # the benchmark's batch: 256 decode tokens, two prefill chunks, a finetune window, 1024 tokens in all
        dict(name="mixed_8b_1024", op="forward", model="8b", **_batch(decode=256, lo=512, hi=4096, prefill="256@0 256@768", window=256, seq=2048)),
        # a 2048-token budget, half of it inference, beside a window of 1024 tokens (LoRA on all seven projections)
        dict(name="mixed_14b_2048", op="forward", model="14b", **_batch(decode=512, lo=16, hi=8192, median=1024, sigma=0.8, prefill="128@0 384@0", window=1024, seq=4096)),
        # no request is decoding: ragged prefill chunks and the window that finetuning gets beside them
        dict(name="chunks_32b_1405", op="forward", model="32b", **_batch(prefill="713@0 487@500", window=205, seq=4096)),
        # the window's way back through one layer
        dict(name="backward_8b_256", op="backward", model="8b", **_batch(window=256, seq=2048)),
        dict(name="backward_14b_1024", op="backward", model="14b", **_batch(window=1024, seq=4096)),
        # the other bypass network: a co-served iteration, forward and the window's backward, of one layer
        dict(name="ia3_8b_205", op="ia3", model="8b", **_batch(decode=96, lo=128, hi=2048, prefill="211@0", window=205, seq=2000)),
        # loss head of a finetune window and the gradient its backward starts from
        dict(name="head_8b_512", op="head", model="8b", window=512, seq=2048),
        # the optimizer, once per finetune sequence: every bypass matrix of the 32-layer model in one call
        dict(name="adam_8b", op="adam", model="8b", layers=32),
        # a whole iteration through a model: all layers (here two), loss head, backward through all layers
        dict(name="step_8b_2048", op="step", model="8b", layers=2, **_batch(decode=512, lo=16, hi=8192, median=1024, sigma=0.8, prefill="611@0 413@0", window=512, seq=2048)),
        # the fp32 configuration, a co-served iteration: forward and the window's backward of one layer
        dict(name="tiny_f32", op="step", model="tiny", layers=1, **_batch(decode=4, lo=16, hi=64, prefill="32@0", window=32, seq=64)),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(("decode", "decode", "mixed", "mixed", "chunks", "backward", "backward", "ia3", "head", "adam", "step", "tiny"))
    model = rng.choice(("8b", "14b", "32b"))
    chunk = lambda most: "%d@%d" % (_log(rng, 17, most), rng.choice((0, rng.randint(1, 1500))))  # noqa: E731
    chunks = lambda n, most: " ".join(chunk(most) for _ in range(n))  # noqa: E731
    seq = rng.randint(1200, 4096)
    if op == "decode":
        lo = rng.randint(16, 400)
        return dict(op="forward", model=model, **_batch(decode=_log(rng, 1, 256), lo=lo, hi=rng.randint(lo + 50, 3000), adapters=rng.choice((1, 1, 2, 4))))
    if op == "mixed":
        n = _log(rng, 24, 384)
        laws = ({"lo": 100, "hi": rng.randint(1000, 4096)}, {"lo": 16, "hi": 8192, "median": rng.randint(300, 1024), "sigma": 0.8})
        window = _log(rng, 32, 512)
        return dict(op="forward", model=model, **_batch(decode=n, prefill=chunks(rng.randint(1, 2), 400), window=window, seq=seq, adapters=rng.choice((1, 1, 3)), **rng.choice(laws)))
    if op == "chunks":
        return dict(op="forward", model=model, **_batch(prefill=chunks(rng.randint(1, 3), 450), window=rng.choice((0, _log(rng, 32, 400))), seq=seq))
    if op == "backward":
        return dict(op="backward", model=model, **_batch(window=_log(rng, 64, 768), seq=seq))
    if op == "ia3":
        return dict(op="ia3", model=model, **_batch(decode=_log(rng, 8, 128), lo=100, hi=rng.randint(300, 2048), prefill=chunks(1, 256), window=_log(rng, 32, 320), seq=seq))
    if op == "head":
        return dict(op="head", model=model, window=_log(rng, 64, 640), seq=seq)
    if op == "adam":
        return dict(op="adam", model=model, layers=rng.randint(4, 32))
    if op == "step":
        return dict(op="step", model="8b", layers=rng.randint(1, 2), **_batch(decode=_log(rng, 16, 384), lo=16, hi=4096, median=rng.randint(300, 1024), sigma=0.8, prefill=chunks(1, 500), window=_log(rng, 64, 384), seq=seq))
    window = _log(rng, 8, 128)
    return dict(op="step", model="tiny", layers=rng.randint(1, 2), **_batch(decode=_log(rng, 1, 16), lo=8, hi=rng.randint(32, 200), prefill=chunk(128).split("@")[0] + "@0", window=window, seq=window + rng.randint(1, 128)))


def _lengths(case):
    """context length of each decode request, the new token included"""
    n, out = case["decode"], []
    for i in range(n):
        u = (i + 0.5) / n
        if case["median"]:
            z = math.sqrt(2.0) * float(torch.erfinv(torch.tensor(2 * u - 1, dtype=torch.float64)))
            c = case["median"] * math.exp(case["sigma"] * z)
        else:
            c = case["lo"] + u * (case["hi"] + 1 - case["lo"])
        out.append(max(1, min(case["hi"], max(case["lo"], int(c)))))
    return out


def _requests(case):
    """[(kind, first position, new tokens, adapter id, tokens the sequence's pages hold)]"""
    reqs = [(DECODE, n - 1, 1, n) for n in _lengths(case)]
    for p in case["prefill"].split():
        n, start = (int(v) for v in p.split("@"))
        reqs.append((PREFILL, start, n, start + n))
    a = case["adapters"]
    ids = [-1] if a == 1 else [-1] + list(range(a))
    reqs = [(k, s, n, ids[i % len(ids)], cap) for i, (k, s, n, cap) in enumerate(reqs)]
    if case["window"]:
        w = min(case["window"], case["seq"])
        reqs.append((FINETUNE, case["seq"] - w, w, 0, case["seq"]))
    return reqs


# ---- inputs ---------------------------------------------------------------------------------------------------------

def _dims(c, t):
    return {"q": (c.hidden, c.q_dim), "k": (c.hidden, c.kv_dim), "v": (c.hidden, c.kv_dim), "o": (c.q_dim, c.hidden),
            "gate": (c.hidden, c.ffn), "up": (c.hidden, c.ffn), "down": (c.ffn, c.hidden)}[t]


class _Source:
    """seeded values on the GPU"""

    def __init__(self, c, seed):
        self.dt = HH.TORCH_DTYPE[c.dtype]
        self.g = torch.Generator(device="cuda").manual_seed(1000003 * (seed + 1))
        self.order = torch.Generator().manual_seed(seed + 77)

    def normal(self, *shape, std=1.0, mean=0.0, dtype=None):
        t = torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32)
        return t.mul_(std).add_(mean).to(dtype or self.dt)

    def big_normal(self, *shape):
        return torch.randn(shape, generator=self.g, device="cuda", dtype=self.dt)


def _weights(c, src):
    w = {"wqkv": src.normal(c.q_dim + 2 * c.kv_dim, c.hidden, std=0.02), "wo": src.normal(c.hidden, c.q_dim, std=0.02),
         "wgu": src.normal(2 * c.ffn, c.hidden, std=0.02), "wd": src.normal(c.hidden, c.ffn, std=0.02),
         "g1": src.normal(c.hidden, std=0.02, mean=1.0), "g2": src.normal(c.hidden, std=0.02, mean=1.0), "bqkv": None}
    if c.qkv_bias:
        w["bqkv"] = src.normal(c.q_dim + 2 * c.kv_dim, std=0.02)
    return w


def _adapter(c, src):
    return {t: (src.normal(c.lora_rank, _dims(c, t)[0], std=0.02), src.normal(_dims(c, t)[1], c.lora_rank, std=0.01)) for t in c.lora_targets}


def _inputs(case, seed):
    """what the call reads, as torch tensors"""
    c = _cfg(case)
    src = _Source(c, seed)
    d = SimpleNamespace(c=c, op=case["op"])
    if case["op"] == "adam":
        n = case["layers"] * HH.lora_param_elems(c)
        d.param = src.normal(n, std=0.02)
        d.master = d.param.float() + src.normal(n, std=1e-5, dtype=torch.float32)
        d.grad = src.normal(n, std=1e-3, dtype=torch.float32)
        d.m, d.v = src.normal(n, std=3e-4, dtype=torch.float32), src.normal(n, std=1e-3, dtype=torch.float32).square_()
        d.lr, d.step = 1e-4, 7
        return d
    if case["op"] in ("head", "step"):
        d.gain, d.w_lm = src.normal(c.hidden, std=0.02, mean=1.0), src.normal(c.vocab, c.hidden, std=0.02)
        d.targets = torch.randint(0, c.vocab, (case["window"],), generator=src.g, device="cuda", dtype=torch.int32)
        d.targets[-1] = -1          # the sequence's last token has no next one
        d.scale = 1.0 / case["seq"]
        if case["op"] == "head":
            d.x = src.normal(case["window"], c.hidden, std=3.0)
            return d
    d.reqs = _requests(case)
    pages = [-(-r[4] // c.page_size) for r in d.reqs]
    d.num_pages = sum(pages) + 3
    ids = torch.randperm(d.num_pages, generator=src.order).to(torch.int32)
    d.pages, at = [], 0
    for n in pages:
        d.pages.append(ids[at:at + n])
        at += n
    d.T = sum(r[2] for r in d.reqs)
    ft = [i for i, r in enumerate(d.reqs) if r[0] == FINETUNE]
    d.ft = ft[0] if ft else None
    d.layers = [SimpleNamespace(w=_weights(c, src), lora=[_adapter(c, src) for _ in range(case["adapters"])] if c.lora_targets else [],
                                k=src.big_normal(d.num_pages, c.n_kv_heads, c.page_size, c.head_dim),
                                v=src.big_normal(d.num_pages, c.n_kv_heads, c.head_dim, c.page_size))
                for _ in range(case.get("layers", 1))]
    d.x = src.normal(d.T, c.hidden)
    if case["op"] in ("backward", "ia3"):
        d.dy = src.normal(case["window"], c.hidden, std=1e-3)
    if case["op"] == "ia3":
        d.ia3 = {n: src.normal(w, std=0.25, mean=1.0) for n, w in (("k", c.kv_dim), ("v", c.kv_dim), ("ff", c.ffn))}
    return d


def _empty_state(c, L, dtype, ia3=False, keep_u=True):
    z = lambda w, dt=dtype: torch.zeros((L, w), dtype=dt, device="cuda")  # noqa: E731
    wide = torch.float64 if dtype == torch.float64 else torch.float32
    st = {"q_cache": z(c.q_dim), "attn": z(c.q_dim), "x": z(c.hidden), "x2": z(c.hidden), "gate": z(c.ffn), "up": z(c.ffn), "lse": z(c.n_q_heads, wide)}
    for t in c.lora_targets if keep_u else ():
        st["u_" + t] = z(c.lora_rank, wide)
    if ia3:
        st["k0"], st["v0"] = z(c.kv_dim), z(c.kv_dim)
    return st


# ---- the same in 64 bits --------------------------------------------------------------------------------------------

def _norm64(x, g, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * g


def _norm64_bwd(x, g, eps, dh):
    r = torch.rsqrt(x.square().mean(-1, keepdim=True) + eps)
    gd = g * dh
    return r * gd - x * r ** 3 * (x * gd).mean(-1, keepdim=True)


def _rope64(c, t, pos, back=False):
    half = c.head_dim // 2
    f = c.rope_theta ** (-torch.arange(half, dtype=torch.float64, device=t.device) * 2 / c.head_dim)
    a = pos.double()[:, None] * f
    cos, sin = a.cos()[:, None], (-a if back else a).sin()[:, None]
    t = t.view(t.shape[0], -1, c.head_dim)
    p, q = t[..., :half], t[..., half:]
    return torch.cat((p * cos - q * sin, q * cos + p * sin), -1).reshape(t.shape[0], -1)


def _cached(c, d, layer, i, n):
    """the first n key / value rows of request i's sequence, [kv heads, n, head_dim] in 64 bits"""
    p = d.pages[i].to("cuda").long()[: -(-n // c.page_size)]
    k = layer.k[p].double().permute(1, 0, 2, 3).reshape(c.n_kv_heads, -1, c.head_dim)
    v = layer.v[p].double().permute(1, 0, 3, 2).reshape(c.n_kv_heads, -1, c.head_dim)
    return k[:, :n], v[:, :n]


def _scores64(c, q, k, start):
    """scaled logits [kv heads, group, rows, keys], later keys masked"""
    n, g = q.shape[0], c.n_q_heads // c.n_kv_heads
    s = torch.matmul(q.view(n, c.n_kv_heads, g, c.head_dim).permute(1, 2, 0, 3).reshape(c.n_kv_heads, g * n, c.head_dim), k.transpose(1, 2).contiguous())
    s = s.view(c.n_kv_heads, g, n, -1) / math.sqrt(c.head_dim)
    later = torch.arange(k.shape[1], device="cuda")[None] > start + torch.arange(n, device="cuda")[:, None]
    return s.masked_fill_(later, -math.inf)


def _attend64(c, q, k, v, start):
    n, g = q.shape[0], c.n_q_heads // c.n_kv_heads
    s = _scores64(c, q, k, start)
    lse = torch.logsumexp(s, -1)
    o = torch.matmul((s - lse[..., None]).exp_().view(c.n_kv_heads, g * n, -1), v)
    return o.view(c.n_kv_heads, g, n, -1).permute(2, 0, 1, 3).reshape(n, -1), lse.permute(2, 0, 1).reshape(n, -1)


def _forward64(d, layer, x, store=lambda t: t, ia3=None):
    """one layer over the batch; store: what writing a tensor to memory does to it.  Returns the output, the window's
    state and the new key / value rows of each request."""
    c, w = d.c, {n: (None if t is None else t.double()) for n, t in layer.w.items()}
    rows, at = [], 0
    for r in d.reqs:
        rows.append(slice(at, at + r[2]))
        at += r[2]
    pos = torch.cat([torch.arange(r[1], r[1] + r[2], device="cuda") for r in d.reqs])
    win = rows[d.ft] if d.ft is not None else None
    st = {}

    def lora(t, xs, y):
        if t not in c.lora_targets:
            return
        for (_, _, _, a, _), sl in zip(d.reqs, rows):
            if a >= 0:
                A, Bm = (m.double() for m in layer.lora[a][t])
                u = xs[sl] @ A.T
                y[sl] += c.lora_scale * u @ Bm.T
                if sl is win:
                    st["u_" + t] = u

    def scale(y, name):
        if ia3 is not None:
            for (_, _, _, a, _), sl in zip(d.reqs, rows):
                if a >= 0:
                    y[sl] *= ia3[name].double()

    h = store(_norm64(x, w["g1"], c.rms_eps))
    qkv = h @ w["wqkv"].T
    if w["bqkv"] is not None:
        qkv += w["bqkv"]
    q, k, v = qkv[:, :c.q_dim], qkv[:, c.q_dim:c.q_dim + c.kv_dim], qkv[:, c.q_dim + c.kv_dim:]
    for t, y in (("q", q), ("k", k), ("v", v)):
        lora(t, h, y)
    if win is not None and ia3 is not None:
        st["k0"], st["v0"] = k[win].clone(), v[win].clone()
    scale(k, "k")
    scale(v, "v")
    q, k, v = store(_rope64(c, q, pos)), store(_rope64(c, k, pos)), store(v)
    o, lse = torch.empty_like(q), torch.empty((d.T, c.n_q_heads), dtype=torch.float64, device="cuda")
    new = []
    for i, (r, sl) in enumerate(zip(d.reqs, rows)):
        kn, vn = (t[sl].view(-1, c.n_kv_heads, c.head_dim).permute(1, 0, 2) for t in (k, v))
        if r[1]:
            kc, vc = _cached(c, d, layer, i, r[1])
            o[sl], lse[sl] = _attend64(c, q[sl], torch.cat((kc, kn), 1), torch.cat((vc, vn), 1), r[1])
        else:
            o[sl], lse[sl] = _attend64(c, q[sl], kn, vn, 0)
        new.append((kn, vn))
    o = store(o)
    x2 = x + o @ w["wo"].T
    lora("o", o, x2)
    x2 = store(x2)
    h2 = store(_norm64(x2, w["g2"], c.rms_eps))
    gu = h2 @ w["wgu"].T
    lora("gate", h2, gu[:, :c.ffn])
    lora("up", h2, gu[:, c.ffn:])
    gate, up = store(gu[:, :c.ffn]), store(gu[:, c.ffn:])
    act = torch.nn.functional.silu(gate) * up
    scale(act, "ff")
    act = store(act)
    y = x2 + act @ w["wd"].T
    lora("down", act, y)
    if win is not None:
        st.update(q_cache=q[win], attn=o[win], x=x[win], x2=x2[win], gate=gate[win], up=up[win], lse=lse[win])
    return y, st, new


def _pool64(d, layer, new):
    """the pool after the new rows were appended"""
    k, v = layer.k.double(), layer.v.double()
    for r, pages, (kn, vn) in zip(d.reqs, d.pages, new):
        p = torch.arange(r[1], r[1] + r[2])
        pg, off = pages.long()[p // d.c.page_size].to("cuda"), (p % d.c.page_size).to("cuda")
        k[pg, :, off, :] = kn.permute(1, 0, 2)
        v[pg, :, :, off] = vn.permute(1, 0, 2)
    return k, v


def _backward64(d, layer, st, k, v, dy, ia3=None):
    """the last window's way back through one layer from the state st, k, v the sequence's rows [kv heads, L, head_dim]"""
    c, w, lora = d.c, {n: (None if t is None else t.double()) for n, t in layer.w.items()}, layer.lora[0] if layer.lora else {}
    st = {n: t.double() for n, t in st.items()}
    _, start, n, _, _ = d.reqs[d.ft]
    g = c.n_q_heads // c.n_kv_heads
    grads = {}

    def back(t, xs, dyt, dx):
        if t in c.lora_targets:
            A, Bm = (m.double() for m in lora[t])
            grads["dB_" + t] = c.lora_scale * dyt.T @ (xs @ A.T)
            tt = c.lora_scale * dyt @ Bm
            grads["dA_" + t] = tt.T @ xs
            dx += tt @ A

    sig = torch.sigmoid(st["gate"])
    act = st["gate"] * sig * st["up"]
    dact = dy @ w["wd"]
    if ia3 is not None:
        grads["dl_ff"] = (dact * act).sum(0)
        dact = dact * ia3["ff"].double()
    back("down", act, dy, dact)
    dgu = torch.cat((dact * st["up"] * sig * (1 + st["gate"] * (1 - sig)), dact * st["gate"] * sig), 1)
    h2 = _norm64(st["x2"], w["g2"], c.rms_eps)
    dh2 = dgu @ w["wgu"]
    back("gate", h2, dgu[:, :c.ffn], dh2)
    back("up", h2, dgu[:, c.ffn:], dh2)
    dx2 = dy + _norm64_bwd(st["x2"], w["g2"], c.rms_eps, dh2)
    do = dx2 @ w["wo"]
    back("o", st["attn"], dx2, do)
    # attention
    q = st["q_cache"]
    p = (_scores64(c, q, k, start) - st["lse"].view(n, c.n_kv_heads, g).permute(1, 2, 0)[..., None]).exp_().view(c.n_kv_heads, g * n, -1)
    split = lambda t: t.view(n, c.n_kv_heads, g, c.head_dim).permute(1, 2, 0, 3).reshape(c.n_kv_heads, g * n, c.head_dim)  # noqa: E731
    dos, qs = split(do), split(q)
    dv = torch.matmul(p.transpose(1, 2).contiguous(), dos)
    ds = torch.matmul(dos, v.transpose(1, 2).contiguous())
    ds -= (dos * split(st["attn"])).sum(-1, keepdim=True)
    ds.mul_(p).mul_(1 / math.sqrt(c.head_dim))
    dq = torch.matmul(ds, k.contiguous()).view(c.n_kv_heads, g, n, -1).permute(2, 0, 1, 3).reshape(n, -1)
    dk = torch.matmul(ds.transpose(1, 2).contiguous(), qs).permute(1, 0, 2).reshape(start + n, -1)
    dv = dv.permute(1, 0, 2).reshape(start + n, -1)
    pos = torch.arange(start, start + n, device="cuda")
    dqr, dkr, dvr = _rope64(c, dq, pos, True), _rope64(c, dk[start:], pos, True), dv[start:]
    if ia3 is not None:
        grads["dl_k"], grads["dl_v"] = (dkr * st["k0"]).sum(0), (dvr * st["v0"]).sum(0)
        dkr, dvr = dkr * ia3["k"].double(), dvr * ia3["v"].double()
    h = _norm64(st["x"], w["g1"], c.rms_eps)
    dh = torch.cat((dqr, dkr, dvr), 1) @ w["wqkv"]
    for t, y in (("q", dqr), ("k", dkr), ("v", dvr)):
        back(t, h, y, dh)
    return dx2 + _norm64_bwd(st["x"], w["g1"], c.rms_eps, dh), grads, dk, dv


def _sequence64(d, layer, new=None):
    """all key / value rows of the finetune sequence: the cached ones, and the window's where they are given"""
    _, start, n, _, L = d.reqs[d.ft]
    if new is None:
        return _cached(d.c, d, layer, d.ft, L)
    k, v = _cached(d.c, d, layer, d.ft, start) if start else (new[d.ft][0][:, :0], new[d.ft][1][:, :0])
    return torch.cat((k, new[d.ft][0]), 1), torch.cat((v, new[d.ft][1]), 1)


def _head64(d, x):
    c = d.c
    h = _norm64(x, d.gain.double(), c.rms_eps)
    z = h @ d.w_lm.double().T
    lse = torch.logsumexp(z, 1)
    ok = (d.targets >= 0).nonzero()[:, 0]
    t = d.targets.long()[ok]
    loss = d.scale * (lse[ok] - z[ok, t]).sum()
    dz = z.sub_(lse[:, None]).exp_()
    dz[ok, t] -= 1
    dz[d.targets < 0] = 0
    return loss.view(1), _norm64_bwd(x, d.gain.double(), c.rms_eps, d.scale * (dz @ d.w_lm.double()))


def _placed(c, d, st, dtype, ia3=False):
    """the whole-sequence buffers with the window's rows in place"""
    _, start, n, _, L = d.reqs[d.ft]
    full = _empty_state(c, L, dtype, ia3)
    for name, t in full.items():
        t[start:start + n] = st[name].to(t.dtype)
    return full


def exact(case, seed):
    with torch.no_grad():
        d = _inputs(case, seed)
        c = d.c
        if d.op == "adam":
            b1, b2, eps = 0.9, 0.999, 1e-8
            g = d.grad.double()
            m, v = b1 * d.m.double() + (1 - b1) * g, b2 * d.v.double() + (1 - b2) * g * g
            p = d.master.double() - d.lr * (m / (1 - b1 ** d.step)) / ((v / (1 - b2 ** d.step)).sqrt() + eps)
            return {"param": p, "master": p, "m": m, "v": v}
        if d.op == "head":
            loss, dx = _head64(d, d.x.double())
            return {"loss": loss, "dx": dx}
        if d.op == "backward":
            st = _window_state(d)
            k, v = _sequence64(d, d.layers[0])
            dx, grads, dk, dv = _backward64(d, d.layers[0], st, k, v, d.dy.double())
            return {"dx": dx, "grads": grads, "dk": dk, "dv": dv}
        if d.op == "step":
            x, kept = d.x.double(), []
            for layer in d.layers:
                x, st, new = _forward64(d, layer, x)
                kept.append((st, new))
            n = d.reqs[d.ft][2]
            loss, dy = _head64(d, x[-n:])
            out = {"y": x, "loss": loss, "layers": []}
            for layer, (st, new) in list(zip(d.layers, kept))[::-1]:
                k, v = _sequence64(d, layer, new)
                dy, grads, dk, dv = _backward64(d, layer, {s: t for s, t in st.items() if s[:2] != "u_"}, k, v, dy)
                out["layers"].insert(0, {"grads": grads, "dk": dk, "dv": dv})
            return out
        y, st, new = _forward64(d, d.layers[0], d.x.double(), ia3=getattr(d, "ia3", None))
        k, v = _pool64(d, d.layers[0], new)
        out = {"y": y, "k": k, "v": v}
        if d.ft is not None:
            out["state"] = _placed(c, d, st, torch.float64, d.op == "ia3")
        if d.op == "ia3":
            ks, vs = _sequence64(d, d.layers[0], new)
            dx, grads, dk, dv = _backward64(d, d.layers[0], st, ks, vs, d.dy.double(), d.ia3)
            out.update(dx=dx, grads=grads, dk=dk, dv=dv)
        return out


def _window_state(d):
    """the state an earlier forward pass over the window left (rows of the window), its key / value rows in the pool"""
    dt = HH.TORCH_DTYPE[d.c.dtype]
    layer = d.layers[0]
    _, st, new = _forward64(d, layer, d.x.double(), store=lambda t: t.to(dt).double())
    _, start, n, _, _ = d.reqs[d.ft]
    p = torch.arange(start, start + n)
    pg, off = d.pages[d.ft].long()[p // d.c.page_size].to("cuda"), (p % d.c.page_size).to("cuda")
    layer.k[pg, :, off, :] = new[d.ft][0].permute(1, 0, 2).to(dt)
    layer.v[pg, :, :, off] = new[d.ft][1].permute(1, 0, 2).to(dt)
    return {name: t.to(torch.float32 if name == "lse" or name[:2] == "u_" else dt) for name, t in st.items()}


# ---- the calls ------------------------------------------------------------------------------------------------------

def _addr(t):
    return None if t is None else t.data_ptr()


def _device_layer(c, d, layer, arena):
    """the layer's device objects as a program keeps them: weights, adapters with their gradients, pool, finetune state"""
    o = SimpleNamespace(src=layer, grads={})
    w = layer.w
    o.w = B.BaseWeights(*[_addr(w[n]) for n in ("wqkv", "bqkv", "wo", "wgu", "wd", "g1", "g2")])
    o.adapters = []
    for a, mats in enumerate(layer.lora):
        l = B.Lora()
        for t, (A, Bm) in mats.items():
            i = B.TARGET_NAMES.index(t)
            l.A[i], l.B[i] = A.data_ptr(), Bm.data_ptr()
            if a == 0 and arena is not None:      # the finetune sequence trains the first adapter
                o.grads["dA_" + t], o.grads["dB_" + t] = arena.take(A.shape)[1], arena.take(Bm.shape)[1]
                l.dA[i], l.dB[i] = o.grads["dA_" + t].data_ptr(), o.grads["dB_" + t].data_ptr()
        o.adapters.append(l)
    o.pool = B.KVPool(layer.k.data_ptr(), layer.v.data_ptr(), d.num_pages, c.page_size)
    o.ft = None
    if d.ft is not None:
        o.state = HH.DeviceFtState(c, d.reqs[d.ft][4], ia3=d.op == "ia3")
        o.ft = o.state.c
    return o


def _kept(state):
    """the buffers of a finetune state by the names exact() gives them"""
    out = {"q_cache": state.q_cache, "attn": state.attn, "x": state.x, "x2": state.x2, "gate": state.gate, "up": state.up, "lse": state.lse}
    out.update({"u_" + t: u for t, u in state.u.items()})
    if hasattr(state, "k0"):
        out.update(k0=state.k0, v0=state.v0)
    return out


def prepare(case, seed):
    with torch.no_grad():
        d = _inputs(case, seed)
        c, s = d.c, SimpleNamespace(d=d, op=d.op)
        dt = HH.TORCH_DTYPE[c.dtype]
        new = lambda *shape: torch.empty(shape, dtype=dt, device="cuda")  # noqa: E731
        if d.op == "adam":
            return s
        if d.op in ("head", "step"):
            s.head = B.LmHead(c.hidden, c.vocab, HH.DTYPE_CODE[c.dtype], c.rms_eps, d.gain.data_ptr(), d.w_lm.data_ptr())
            s.n = case["window"]
            s.head_bytes = B.flexco_lm_loss_workspace_bytes(s.head, s.n)
            s.head_ws = torch.empty(s.head_bytes, dtype=torch.uint8, device="cuda")
            s.loss = torch.zeros(1, dtype=torch.float32, device="cuda")
            s.dx, s.dtmp = new(s.n, c.hidden), new(s.n, c.hidden)
            if d.op == "head":
                return s
        s.cfg = HH.c_cfg(c)
        s.arena = None
        if c.lora_targets and d.op in ("backward", "step"):
            s.arena = HH.ParamArena(len(d.layers) * HH.lora_param_elems(c), dt)
        s.layers = [_device_layer(c, d, layer, s.arena) for layer in d.layers]
        n, L = (d.reqs[d.ft][2], d.reqs[d.ft][4]) if d.ft is not None else (0, 0)
        if d.ft is not None:
            s.pages, s.start, s.n = d.pages[d.ft].to("cuda"), d.reqs[d.ft][1], n
        if d.op == "backward":
            for name, t in _window_state(d).items():
                _kept(s.layers[0].state)[name][s.start:s.start + n] = t
            s.ws = HH.Workspace(s.cfg, 1, 1, n, L)
            s.dx = new(n, c.hidden)
            return s
        reqs = [SimpleNamespace(kind=k, seq_id=i, start_pos=p, n_new=m, adapter=a) for i, (k, p, m, a, _) in enumerate(d.reqs)]
        s.batch = HH.DeviceBatch(c, reqs, [p.numpy() for p in d.pages], d.num_pages)
        s.ws = HH.Workspace(s.cfg, d.T, s.batch.host_maps.n_parts, n, L)
        s.y = new(d.T, c.hidden)
        if d.op == "ia3":
            s.dx = new(n, c.hidden)
            s.dl = {"dl_" + name: torch.zeros(t.shape, dtype=torch.float32, device="cuda") for name, t in d.ia3.items()}
            s.ia3 = B.Ia3(*[d.ia3[m].data_ptr() for m in ("k", "v", "ff")], *[s.dl["dl_" + m].data_ptr() for m in ("k", "v", "ff")])
        if d.op == "step":
            s.tmp = new(d.T, c.hidden)
            s.arr, s.keep = B.make_model_layers([(l.w, l.adapters[0], l.pool, l.ft) for l in s.layers])
        return s


def run(s):
    d = s.d
    if s.op == "adam":
        B.flexco_adam_step(d.param, d.master, d.grad, d.m, d.v, d.param.numel(), B.FLEXCO_BF16, d.lr, 0.9, 0.999, 1e-8, d.step)
        return {"param": d.param, "master": d.master, "m": d.m, "v": d.v}
    if s.op == "head":
        s.loss.zero_()
        B.flexco_lm_loss(s.head, d.x, d.targets, s.n, d.scale, s.loss, s.dx, s.head_ws, s.head_bytes)
        return {"loss": s.loss, "dx": s.dx}
    l = s.layers[0]
    if s.op == "backward":
        # a sequence's first backward window: gradients and the KV-gradient accumulator start from zero
        s.arena.grad.zero_()
        l.state.zero_accum()
        B.flexco_lora_bwd(s.cfg, l.w, l.adapters[0], l.pool, s.pages, len(s.pages), l.ft, s.start, s.n, d.dy, s.dx, s.ws.ptr, s.ws.bytes)
        return {"dx": s.dx, "grads": l.grads, "dk": l.state.dk_accum, "dv": l.state.dv_accum}
    if s.op == "step":
        s.arena.grad.zero_()
        s.loss.zero_()
        for m in s.layers:
            m.state.zero_accum()
        B.flexco_model_forward(s.cfg, s.arr, len(s.layers), s.batch.maps, d.x, s.y, s.tmp, s.ws.ptr, s.ws.bytes)
        B.flexco_lm_loss(s.head, s.y[d.T - s.n:], d.targets, s.n, d.scale, s.loss, s.dx, s.head_ws, s.head_bytes)
        B.flexco_model_backward(s.cfg, s.arr, len(s.layers), s.pages, len(s.pages), s.start, s.n, s.dx, s.dtmp, False, s.ws.ptr, s.ws.bytes)
        return {"y": s.y, "loss": s.loss, "layers": [{"grads": m.grads, "dk": m.state.dk_accum, "dv": m.state.dv_accum} for m in s.layers]}
    out = {"y": s.y, "k": l.src.k, "v": l.src.v}
    if d.ft is not None:
        out["state"] = _kept(l.state)
    if s.op == "ia3":
        for t in s.dl.values():
            t.zero_()
        l.state.zero_accum()
        B.flexco_layer_forward_ia3(s.cfg, l.w, s.ia3, s.batch.maps, d.x, s.y, l.pool, l.ft, s.ws.ptr, s.ws.bytes)
        B.flexco_ia3_bwd(s.cfg, l.w, s.ia3, l.pool, s.pages, len(s.pages), l.ft, s.start, s.n, d.dy, s.dx, s.ws.ptr, s.ws.bytes)
        out.update(dx=s.dx, grads=s.dl, dk=l.state.dk_accum, dv=l.state.dv_accum)
    elif len(l.adapters) > 1:
        B.flexco_layer_forward_multi(s.cfg, l.w, l.adapters, s.batch.maps, d.x, s.y, l.pool, l.ft, s.ws.ptr, s.ws.bytes)
    else:
        B.flexco_layer_forward(s.cfg, l.w, l.adapters[0], s.batch.maps, d.x, s.y, l.pool, l.ft, s.ws.ptr, s.ws.bytes)
    return out


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def work(case):
    c = _cfg(case)
    e = 4 if c.dtype == "f32" else 2
    if case["op"] == "adam":
        n = case["layers"] * HH.lora_param_elems(c)
        return {"bytes": n * (2 * e + 8 + 4 + 16), "flops": 12 * n}
    head_b = head_f = 0
    if case["op"] in ("head", "step"):
        n = case["window"]
        head_b, head_f = e * (c.vocab * c.hidden + 2 * n * c.hidden), 4 * n * c.vocab * c.hidden
        if case["op"] == "head":
            return {"bytes": head_b, "flops": head_f}
    reqs, layers = _requests(case), case.get("layers", 1)
    T = sum(r[2] for r in reqs)
    p = (c.q_dim + 2 * c.kv_dim) * c.hidden + c.q_dim * c.hidden + 3 * c.hidden * c.ffn
    lora = sum(c.lora_rank * sum(_dims(c, t)) for t in c.lora_targets)
    kept = 2 * c.q_dim + 2 * c.hidden + 2 * c.ffn          # of a window's token
    visible = sum(n * s + n * (n + 1) // 2 for _, s, n, _, _ in reqs)
    on = sum(r[2] for r in reqs if r[3] >= 0)
    b = f = 0
    if case["op"] != "backward":
        b += e * (p + 2 * T * c.hidden + 2 * c.kv_dim * sum(r[1] + r[2] for r in reqs))
        f += 2 * T * p + 4 * c.q_dim * visible + 2 * on * lora
        b += e * (lora * min(case["adapters"], on) + (case["window"] * kept))
    if case["op"] != "forward":
        n, s = reqs[-1][2], reqs[-1][1]
        vis = n * s + n * (n + 1) // 2
        b += e * (p + n * (kept + 2 * c.hidden) + 2 * c.kv_dim * (s + n)) + (e + 8) * lora + 16 * c.kv_dim * (s + n)
        f += 2 * n * p + 10 * c.q_dim * vis + 6 * n * lora
    return {"bytes": layers * b + head_b, "flops": layers * f + head_f}


def tolerance(case):
    # about four times the distance to exact() measured per operation (bf16 storage: 4e-3 to 8e-3 through a layer one way,
    # 1.2e-2 through the layers, the head and back; fp32: 8e-7); adam: a rounded parameter may take the neighbouring bf16 value
    if case["model"] == "tiny":
        return {"rel": 5e-6, "max": 1e-3}
    if case["op"] == "adam":
        return {"rel": 1e-4, "max": 1e-2}
    return {"rel": {"head": 1e-2, "ia3": 3e-2, "step": 3e-2}.get(case["op"], 2e-2), "max": 0.3}
