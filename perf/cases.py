"""Performance cases: the calls a user of this library makes, through the
binding and `DenseDecoder`, with the values they meet in earnest (weights
N(0, 0.02^2) quantised by the library, activations and cached keys and values
N(0, 1), router logits N(0, 1)).

Kinds of case (`kind`):

  gemv          one decode projection, launched eagerly
  gemm          the projections that share one input (one grouped call; a
                single matrix is one plain call), over `layers` layers
  moe           routing, bucketing and the expert layer of `layers` layers
  attn_decode   decode attention of one token over the caches of `layers` layers
  attn_prefill  causal attention of one layer's prompt chunk, fp16 rows out
  decode        a whole decode step of a dense decoder at position `pos`
  prefill       a whole prompt chunk of `m` tokens from position `p0`

`graph`: the calls are captured in a HIP graph and a pass replays it, as the
decode loop and the prompt path of `DenseDecoder` are meant to be used;
otherwise they are launched one by one.  Buffers and workspaces are the
caller's and are kept between passes, as the library asks of its users.
"""

import math

import torch

from paper_2607_00501_amd import binding as B
from paper_2607_00501_amd import decoder as D
from paper_2607_00501_amd import workloads

FORMATS = {"q4": B.Q4_G32, "q8": B.Q8_G32, "q2": B.Q2_G32, "q3": B.Q3_G32, "q5": B.Q5_G32, "q6": B.Q6_G32,
           "f16": B.F16, "bf16": B.BF16}
MODELS = {"qwen3-0.6b": workloads.QWEN3_06B_DECODER, "llama-3.2-1b": workloads.LLAMA32_1B_DECODER}
SIGMA = 0.02
EPS = 1e-6
DEV = "cuda"


def listed():
    return [
        # The smallest call: one 1024 x 1024 Q4 projection of a small model at batch 1.
        dict(name="gemv_q4_1024", kind="gemv", fmt="q4", n=1024, k=1024),
        # The largest projection of a decode step: the LM head of a 3B model.
        dict(name="gemv_q4_lm_head", kind="gemv", fmt="q4", n=128256, k=3072),
        # One token of greedy decoding at an ordinary position, the whole model.
        dict(name="decode_qwen3_0.6b", kind="decode", model="qwen3-0.6b", fmt="q4", pos=700),
        # Eight sequences decoded together (or a very short prompt): gate and
        # up projections of four layers of a 3B model.
        dict(name="gemm_q4_m8", kind="gemm", fmt="q4", m=8, k=3072, ns="8192,8192", layers=4, graph=True),
        # A short prompt of odd length in another format: q, k and v of four layers of a 1B model.
        dict(name="gemm_q6_m77", kind="gemm", fmt="q6", m=77, k=2048, ns="2048,512,512", layers=4, graph=True),
        # An ordinary prompt chunk: gate and up projections of a 1B model.
        dict(name="gemm_q4_m512", kind="gemm", fmt="q4", m=512, k=2048, ns="8192,8192", layers=1, graph=False),
        # A long prompt in the 8-bit format: the down projection of a 1B model.
        dict(name="gemm_q8_m2048", kind="gemm", fmt="q8", m=2048, k=8192, ns="2048", layers=1, graph=False),
        # Mixture-of-experts decoding, one token: four layers.
        dict(name="moe_q4_m1", kind="moe", fmt="q4", m=1, experts=128, top_k=8, hidden=2048, inter=768, layers=4,
             graph=True),
        # Mixture-of-experts prefill of an ordinary chunk: one layer.
        dict(name="moe_q4_m512", kind="moe", fmt="q4", m=512, experts=128, top_k=8, hidden=2048, inter=768, layers=1,
             graph=False),
        # Decode attention at a long context of odd length: four layers' caches.
        dict(name="attn_decode_6007", kind="attn_decode", hq=16, hkv=8, d=128, len=6007, layers=4, graph=True),
        # Causal attention of a long prompt.
        dict(name="attn_prefill_2048", kind="attn_prefill", hq=32, hkv=8, d=64, m=2048, p0=0),
        # A whole 512-token prompt chunk of a 1B model, with the last token's logits.
        dict(name="prefill_llama_1b_512", kind="prefill", model="llama-3.2-1b", fmt="q4", m=512, p0=0),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["gemv", "gemm", "gemm", "gemm", "moe", "moe", "attn_decode", "attn_prefill", "decode",
                       "prefill"])
    fmt = rng.choice(["q4", "q4", "q4", "q8", "q8", "q2", "q3", "q5", "q6", "f16", "bf16"])
    if kind == "gemv":
        return dict(kind=kind, fmt=fmt, n=_log_int(rng, 200, 130000), k=32 * _log_int(rng, 16, 256))
    if kind == "gemm":
        m, k = _log_int(rng, 2, 2048), 32 * _log_int(rng, 16, 256)
        count = rng.randint(1, 3)
        ns = ",".join(str(_log_int(rng, 200, 8192)) for _ in range(count))
        small = m <= 64
        return dict(kind=kind, fmt=fmt, m=m, k=k, ns=ns, layers=4 if small else 1, graph=small)
    if kind == "moe":
        m = _log_int(rng, 1, 1024)
        fmt = fmt if fmt not in ("f16", "bf16") else "q4"
        experts, top_k = rng.choice([(128, 8), (64, 6), (32, 4)])
        return dict(kind=kind, fmt=fmt, m=m, experts=experts, top_k=top_k, hidden=32 * rng.randint(32, 64),
                    inter=32 * rng.randint(16, 40), layers=2 if m <= 64 else 1, graph=m <= 64)
    if kind == "attn_decode":
        hkv = rng.choice([4, 8])
        return dict(kind=kind, hq=hkv * rng.choice([1, 2, 3, 4, 7, 8]), hkv=hkv, d=rng.choice([64, 128]),
                    len=_log_int(rng, 40, 40000), layers=4, graph=True)
    if kind == "attn_prefill":
        hq, d = rng.choice([(32, 64), (16, 128), (24, 128)])
        m = _log_int(rng, 16, 2048)
        return dict(kind=kind, hq=hq, hkv=8, d=d, m=m, p0=rng.choice([0, 0, _log_int(rng, 100, 16000)]))
    model = rng.choice(sorted(MODELS))
    fmt = rng.choice(["q4", "q4", "q8", "q6"])
    if kind == "decode":
        return dict(kind=kind, model=model, fmt=fmt, pos=_log_int(rng, 1, 2000))
    return dict(kind=kind, model=model, fmt=fmt, m=_log_int(rng, 8, 448), p0=rng.choice([0, rng.randint(1, 600)]))


# --------------------------------------------------------------- inputs


def _normal(seed, tag, shape, sigma=1.0, mean=0.0):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + tag * 7919 + 17) % (1 << 62))
    t = torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)
    return t.mul_(sigma).add_(mean) if mean else t.mul_(sigma)


def _half(seed, tag, shape, sigma=1.0, mean=0.0):
    return _normal(seed, tag, shape, sigma, mean).to(torch.float16)


def _weight(seed, tag, shape, fmt, rope=None):
    """A quantised weight in the device layout; rope: (heads, head_dim) of
    projections whose rows the fused q/k/v call expects interleaved."""
    w = _normal(seed, tag, shape, SIGMA)
    if rope is not None:
        w = B.rope_interleave_rows(w, *rope)
    return B.qm_repack(B.qm_quantise(w, FORMATS[fmt]), B.LAYOUT_DEVICE)


def _ns(case):
    return [int(v) for v in case["ns"].split(",")]


def _captured(fn):
    """fn's calls in a HIP graph (run once eagerly first)."""
    fn()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        fn()
    return g


def _config(model):
    c = MODELS[model]
    return D.DecoderConfig(hidden=c["hidden"], n_q_heads=c["n_q_heads"], n_kv_heads=c["n_kv_heads"],
                           head_dim=c["head_dim"], inter=c["inter"], vocab=c["vocab"], layers=c["layers"], eps=EPS,
                           theta=c["theta"], rope_scaling=c.get("rope_scaling"))


def _projections(c):
    """(name, rows, columns) of a layer's matrices, in the order of their tags."""
    qd, kvd = c.n_q_heads * c.head_dim, c.n_kv_heads * c.head_dim
    return [("wq", qd, c.hidden), ("wk", kvd, c.hidden), ("wv", kvd, c.hidden), ("wo", c.hidden, qd),
            ("wg", c.inter, c.hidden), ("wu", c.inter, c.hidden), ("wd", c.hidden, c.inter)]


def _decoder(case, seed, max_len, max_chunk):
    c = _config(case["model"])
    layers = []
    for li in range(c.layers):
        w = {}
        for ti, (name, n, k) in enumerate(_projections(c)):
            heads = {"wq": c.n_q_heads, "wk": c.n_kv_heads}.get(name)
            w[name] = _weight(seed, 100 * (li + 1) + ti, (n, k), case["fmt"],
                              rope=(heads, c.head_dim) if heads else None)
        layers.append(D.LayerWeights(**w, attn_norm=_half(seed, 100 * (li + 1) + 10, (c.hidden,), 0.1, 1.0),
                                     ffn_norm=_half(seed, 100 * (li + 1) + 11, (c.hidden,), 0.1, 1.0)))
    return D.DenseDecoder(c, _half(seed, 1, (c.vocab, c.hidden)), layers, _half(seed, 2, (c.hidden,), 0.1, 1.0),
                          _weight(seed, 3, (c.vocab, c.hidden), case["fmt"]), max_len=max_len,
                          rope_rows_interleaved=True, max_chunk=max_chunk)


def _past(case, seed, li, c, rows):
    """Cached keys and values of a layer's earlier positions."""
    shape = (c.n_kv_heads, rows, c.head_dim)
    return _half(seed, 100 * (li + 1) + 20, shape), _half(seed, 100 * (li + 1) + 21, shape)


def _tokens(case, seed, m):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 31 + 5)
    return torch.randint(0, MODELS[case["model"]]["vocab"], (m,), generator=g, device=DEV, dtype=torch.int32)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "gemv":
        w = _weight(seed, 1, (case["n"], case["k"]), case["fmt"])
        return dict(kind=kind, w=w, x=_half(seed, 2, (case["k"],)), out=torch.empty(case["n"], device=DEV))
    if kind == "gemm":
        sets = []
        for li in range(case["layers"]):
            ws = [_weight(seed, 10 * (li + 1) + i, (n, case["k"]), case["fmt"]) for i, n in enumerate(_ns(case))]
            x = _half(seed, 10 * (li + 1) + 9, (case["m"], case["k"]))
            sets.append((ws, x, [torch.empty((case["m"], n), device=DEV) for n in _ns(case)]))

        def calls():
            for ws, x, outs in sets:
                if len(ws) == 1:
                    B.qmatmul_gemm(ws[0], x, out=outs[0])
                else:
                    B.qmatmul_gemm_grouped(ws, x, outs=outs)
        outs = [o for s in sets for o in s[2]]
    elif kind == "moe":
        m, e, h, f = case["m"], case["experts"], case["hidden"], case["inter"]
        ws = torch.empty(max(16, B.qmoe_workspace_bytes(m, e, case["top_k"], h, f)), dtype=torch.uint8, device=DEV)
        sets = []
        for li in range(case["layers"]):
            w = [_weight(seed, 10 * (li + 1) + i, s, case["fmt"]) for i, s in
                 enumerate([(e, f, h), (e, f, h), (e, h, f)])]
            logits = _normal(seed, 10 * (li + 1) + 8, (m, e))
            r = B.qmoe_route(logits, case["top_k"])
            sets.append((w, _half(seed, 10 * (li + 1) + 9, (m, h)), logits, r, torch.empty((m, h), device=DEV)))

        def calls():
            for w, x, logits, r, out in sets:
                B.qmoe_route(logits, case["top_k"], out=r)
                B.qmoe_grouped_gemm(*w, x, r, out=out, workspace=ws)
        outs = [s[4] for s in sets]
    elif kind == "attn_decode":
        hq, hkv, d, n = case["hq"], case["hkv"], case["d"], case["len"]
        ws = torch.empty(B.qattn_decode_workspace_bytes(hq, d), dtype=torch.uint8, device=DEV)
        max_len = (n + 511) // 512 * 512
        sets = [(_half(seed, 10 * li + 1, (hq, d)), _half(seed, 10 * li + 2, (hkv, max_len, d)),
                 _half(seed, 10 * li + 3, (hkv, max_len, d)), torch.empty((hq, d), dtype=torch.float16, device=DEV))
                for li in range(case["layers"])]

        def calls():
            for q, k, v, out in sets:
                B.qattn_decode(q, k, v, n, 1.0 / math.sqrt(d), out=out, workspace=ws)
        outs = [s[3] for s in sets]
    elif kind == "attn_prefill":
        hq, hkv, d, m, p0 = case["hq"], case["hkv"], case["d"], case["m"], case["p0"]
        max_len = (p0 + m + 511) // 512 * 512
        q, k, v = _half(seed, 1, (hq, m, d)), _half(seed, 2, (hkv, max_len, d)), _half(seed, 3, (hkv, max_len, d))
        ws = torch.empty(max(16, B.qattn_prefill_workspace_bytes(hq, d, m, p0)), dtype=torch.uint8, device=DEV)
        out = torch.empty((m, hq * d), dtype=torch.float16, device=DEV)

        def calls():
            B.qattn_prefill_rows_f16(q, k, v, p0, 1.0 / math.sqrt(d), out=out, workspace=ws)
        outs = [out]
    elif kind == "decode":
        pos = case["pos"]
        dec = _decoder(case, seed, (pos + 512) // 512 * 512, 512)
        for li in range(dec.cfg.layers):
            dec.k_cache[li, :, :pos], dec.v_cache[li, :, :pos] = _past(case, seed, li, dec.cfg, pos)
        token = _tokens(case, seed, 1)
        dec.token.copy_(token)
        g = _captured(lambda: dec.step(pos))
        return dict(kind=kind, dec=dec, token=token, graph=g,
                    outs=[dec.logits, dec.k_cache[:, :, pos], dec.v_cache[:, :, pos]])
    else:
        m, p0 = case["m"], case["p0"]
        dec = _decoder(case, seed, (p0 + m + 511) // 512 * 512, max(m, 512))
        for li in range(dec.cfg.layers):
            dec.k_cache[li, :, :p0], dec.v_cache[li, :, :p0] = _past(case, seed, li, dec.cfg, p0)
        tokens = _tokens(case, seed, m)
        return dict(kind=kind, dec=dec, tokens=tokens, graph=_captured(lambda: dec.prefill(tokens, p0)),
                    outs=[dec.logits, dec.k_cache[:, :, p0:p0 + m], dec.v_cache[:, :, p0:p0 + m]])
    return dict(kind=kind, calls=calls, graph=_captured(calls) if case.get("graph") else None, outs=outs)


def run(state):
    if state["kind"] == "gemv":
        return B.qmatmul_gemv(state["w"], state["x"], out=state["out"])
    if state["kind"] == "decode":
        state["dec"].token.copy_(state["token"])    # the step leaves its greedy choice there
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        state["calls"]()
    return state["outs"]


# ------------------------------------------------------ work, tolerance


def _attn_prefill_flops(hq, d, m, p0):
    return 4 * d * hq * (m * p0 + m * (m + 1) // 2)


def work(case):
    kind = case["kind"]
    wb = lambda k, n: workloads.weight_bytes(FORMATS[case["fmt"]], k, n)
    if kind == "gemv":
        n, k = case["n"], case["k"]
        return dict(bytes=wb(k, n) + 2 * k + 4 * n, flops=2 * n * k)
    if kind == "gemm":
        m, k, ns = case["m"], case["k"], _ns(case)
        return dict(bytes=case["layers"] * (sum(wb(k, n) + 4 * m * n for n in ns) + 2 * m * k),
                    flops=case["layers"] * 2 * m * k * sum(ns))
    if kind == "moe":
        m, e, t, h, f = case["m"], case["experts"], case["top_k"], case["hidden"], case["inter"]
        used = e * (1 - (1 - t / e) ** m)            # experts that some token takes, in the mean
        return dict(bytes=case["layers"] * (used * (2 * wb(h, f) + wb(f, h)) + m * (2 * h + 4 * e + 4 * h)),
                    flops=case["layers"] * 6 * m * t * h * f)
    if kind == "attn_decode":
        hq, hkv, d, n = case["hq"], case["hkv"], case["d"], case["len"]
        return dict(bytes=case["layers"] * (4 * hkv * n * d + 4 * hq * d), flops=case["layers"] * 4 * hq * n * d)
    if kind == "attn_prefill":
        hq, hkv, d, m, p0 = case["hq"], case["hkv"], case["d"], case["m"], case["p0"]
        return dict(bytes=4 * hkv * (p0 + m) * d + 4 * hq * m * d, flops=_attn_prefill_flops(hq, d, m, p0))
    c = _config(case["model"])
    m, p0 = (1, case["pos"]) if kind == "decode" else (case["m"], case["p0"])
    weights = sum(n * k for _, n, k in _projections(c))
    cache = 4 * c.n_kv_heads * c.head_dim
    return dict(bytes=c.layers * (sum(wb(k, n) for _, n, k in _projections(c)) + cache * (p0 + m)) +
                wb(c.hidden, c.vocab) + 4 * c.vocab + 2 * m * c.hidden,
                flops=c.layers * (2 * m * weights + _attn_prefill_flops(c.n_q_heads, c.head_dim, m, p0)) +
                2 * c.vocab * c.hidden)


def tolerance(case):
    # About four times the error measured against exact(): weights rounded to
    # fp16 for the matrix cores (GEMM 2.1e-4), fp16 between the kernels of a
    # layer (MoE 4.6e-4), fp16 results (decode attention 2.1e-4; prefill
    # attention, with fp16 probabilities, 3.9e-4), both through a whole model
    # (decode 8.8e-4, prefill 1.3e-3).  GEMV: fp32 sums of exact products,
    # whose order alone moves the last bits (measured up to 2e-7).
    return {"gemv": {"rel": 1e-6}, "gemm": {"rel": 8e-4}, "moe": {"rel": 1.8e-3}, "attn_decode": {"rel": 8e-4},
            "attn_prefill": {"rel": 1.6e-3}, "decode": {"rel": 4e-3}, "prefill": {"rel": 5e-3}}[case["kind"]]


# ---------------------------------------------------- 64-bit references


def _exact_weight(seed, tag, shape, fmt):
    """The weights that the codes and scales of _weight() stand for, in 64 bits."""
    w = _normal(seed, tag, shape, SIGMA)
    if fmt == "f16":
        return w.to(torch.float16).double()
    if fmt == "bf16":
        return w.to(torch.bfloat16).double()
    bits = int(fmt[1:])
    top = 2 ** (bits - 1) - 1
    low = -top if bits == 8 else -top - 1
    g = w.view(*shape[:-1], shape[-1] // 32, 32)
    # single-precision quotients, by way of 64 bits (the second rounding is harmless)
    s = (g.abs().amax(-1, keepdim=True).double() / top).float().half()
    q = torch.where(s == 0, torch.zeros((), device=DEV), torch.round((g.double() / s.double()).float()))
    return (q.clamp(low, top).double() * s.double()).view(shape)


def _silu(x):
    return x / (1 + torch.exp(-x))


def _rmsnorm(x, gain):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * gain


def _causal(q, k, v, p0, scale):
    """q [Hq][m][D] at positions p0.., k, v [Hkv][p0 + m][D] -> [m][Hq * D]."""
    hq, m, d = q.shape
    g = hq // k.shape[0]
    seen = torch.arange(p0 + m, device=DEV)[None, :] <= p0 + torch.arange(m, device=DEV)[:, None]
    out = torch.empty((m, hq, d), dtype=torch.float64, device=DEV)
    for h in range(hq):
        s = (q[h] @ k[h // g].t().contiguous()) * scale
        out[:, h] = torch.softmax(s.masked_fill(~seen, -math.inf), -1) @ v[h // g]
    return out.view(m, hq * d)


def _angles(c, positions):
    i = torch.arange(c.head_dim // 2, device=DEV, dtype=torch.float64)
    f = c.theta ** (-2 * i / c.head_dim)
    if c.rope_scaling is not None:
        factor, low, high, orig = c.rope_scaling
        wave = 2 * math.pi / f
        t = ((orig / wave - low) / (high - low)).clamp(0, 1)
        f = (1 - t) * f / factor + t * f
    return positions.double()[:, None] * f


def _rope(x, ang):
    """x [m][heads][D], rotate-half."""
    a, b = x.chunk(2, -1)
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]
    return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)


def _exact_model(case, seed, tokens, p0):
    c, m = _config(case["model"]), tokens.numel()
    scale = 1.0 / math.sqrt(c.head_dim)
    x = _half(seed, 1, (c.vocab, c.hidden))[tokens.long()].double()
    ang = _angles(c, p0 + torch.arange(m, device=DEV))
    new_k, new_v = [], []
    for li in range(c.layers):
        w = lambda i: _exact_weight(seed, 100 * (li + 1) + i, _projections(c)[i][1:], case["fmt"]).t().contiguous()
        h = _rmsnorm(x, _half(seed, 100 * (li + 1) + 10, (c.hidden,), 0.1, 1.0).double())
        q = _rope((h @ w(0)).view(m, c.n_q_heads, c.head_dim), ang)
        k = _rope((h @ w(1)).view(m, c.n_kv_heads, c.head_dim), ang)
        v = (h @ w(2)).view(m, c.n_kv_heads, c.head_dim)
        k, v = k.transpose(0, 1).contiguous(), v.transpose(0, 1).contiguous()
        new_k.append(k)
        new_v.append(v)
        pk, pv = _past(case, seed, li, c, p0)
        a = _causal(q.transpose(0, 1).contiguous(), torch.cat([pk.double(), k], 1), torch.cat([pv.double(), v], 1),
                    p0, scale)
        x = x + a @ w(3)
        h = _rmsnorm(x, _half(seed, 100 * (li + 1) + 11, (c.hidden,), 0.1, 1.0).double())
        x = x + (_silu(h @ w(4)) * (h @ w(5))) @ w(6)
    h = _rmsnorm(x[-1], _half(seed, 2, (c.hidden,), 0.1, 1.0).double())
    logits = _exact_weight(seed, 3, (c.vocab, c.hidden), case["fmt"]) @ h
    k, v = torch.stack(new_k), torch.stack(new_v)
    return [logits, k[:, :, 0], v[:, :, 0]] if case["kind"] == "decode" else [logits, k, v]


def exact(case, seed):
    kind = case["kind"]
    if kind == "gemv":
        return _exact_weight(seed, 1, (case["n"], case["k"]), case["fmt"]) @ _half(seed, 2, (case["k"],)).double()
    if kind == "gemm":
        outs = []
        for li in range(case["layers"]):
            x = _half(seed, 10 * (li + 1) + 9, (case["m"], case["k"])).double()
            outs += [x @ _exact_weight(seed, 10 * (li + 1) + i, (n, case["k"]), case["fmt"]).t().contiguous()
                     for i, n in enumerate(_ns(case))]
        return outs
    if kind == "moe":
        m, e, h, f = case["m"], case["experts"], case["hidden"], case["inter"]
        outs = []
        for li in range(case["layers"]):
            tag = 10 * (li + 1)
            x = _half(seed, tag + 9, (m, h)).double()
            top, ids = torch.sort(_normal(seed, tag + 8, (m, e)).double(), dim=-1, descending=True, stable=True)
            gates, ids = torch.softmax(top[:, :case["top_k"]], -1), ids[:, :case["top_k"]]
            wg, wu, wd = (_exact_weight(seed, tag + i, s, case["fmt"]) for i, s in
                          enumerate([(e, f, h), (e, f, h), (e, h, f)]))
            y = torch.zeros((m, h), dtype=torch.float64, device=DEV)
            for j in range(e):
                t, slot = (ids == j).nonzero(as_tuple=True)
                if t.numel():
                    a = _silu(x[t] @ wg[j].t().contiguous()) * (x[t] @ wu[j].t().contiguous())
                    y[t] += gates[t, slot][:, None] * (a @ wd[j].t().contiguous())
            outs.append(y)
        return outs
    if kind == "attn_decode":
        hq, hkv, d, n = case["hq"], case["hkv"], case["d"], case["len"]
        max_len = (n + 511) // 512 * 512
        outs = []
        for li in range(case["layers"]):
            q = _half(seed, 10 * li + 1, (hq, d)).double()
            k, v = (_half(seed, 10 * li + i, (hkv, max_len, d))[:, :n].double() for i in (2, 3))
            outs.append(_causal(q[:, None], k, v, n - 1, 1.0 / math.sqrt(d)).view(hq, d))
        return outs
    if kind == "attn_prefill":
        hq, hkv, d, m, p0 = case["hq"], case["hkv"], case["d"], case["m"], case["p0"]
        max_len = (p0 + m + 511) // 512 * 512
        q = _half(seed, 1, (hq, m, d)).double()
        k, v = (_half(seed, i, (hkv, max_len, d))[:, :p0 + m].double() for i in (2, 3))
        return [_causal(q, k, v, p0, 1.0 / math.sqrt(d))]
    if kind == "decode":
        return _exact_model(case, seed, _tokens(case, seed, 1), case["pos"])
    return _exact_model(case, seed, _tokens(case, seed, case["m"]), case["p0"])
