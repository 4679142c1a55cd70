"""Performance cases of the verification hot path, run through the Python binding.

Each case is one pass of a user's program: a verify call (one sequence, a batch of sequences, a decode step), a
prompt's prefill with its first verify call, a full-recompute verify, an acceptance test, or a skip decision.
The model cases hold a few layers of the named shapes (the whole depth repeats the same layer), with the LM
head and the whole vocabulary.  Weights, prompts, drafts and logits are synthetic and made from the seed on the
GPU.  A model case returns its logits: the argmax tokens of random-weight BF16 logits flip on near ties between
any two correct BF16 forwards, so they are computed but not returned (the fp32 case returns them).

exact() recomputes the outputs with plain torch in float64 from the same weights and inputs.
"""
import math

import torch

import workloads as W
from paper_2608_14787_amd import sdd

SHAPES = {"tiny": W.TINY, "qwen7b": W.QWEN7B, "qwen32b": W.QWEN32B}
MODES = {"greedy": sdd.GREEDY, "topk": sdd.TOPK, "lenient": sdd.LENIENT, "ratio": sdd.RATIO}
DEV = "cuda"


def listed():
    return [
        # the smallest model in use (fp32, 2 layers): a whole round, bound by its launches
        dict(name="tiny_round", path="verify", shape="tiny", layers=2, gamma=8, ctx="64", ws_rows=64),
        # a plain decode step after a code-length prompt
        dict(name="decode_7b", path="verify", shape="qwen7b", layers=4, gamma=0, ctx="512", ws_rows=64),
        # one sequence's block verification, the call the whole method is built around, at both named shapes
        dict(name="verify_7b", path="verify", shape="qwen7b", layers=4, gamma=32, ctx="512", ws_rows=256),
        dict(name="verify_32b", path="verify", shape="qwen32b", layers=4, gamma=32, ctx="1024", ws_rows=256),
        # the blocks of several sequences of ragged length in one call: the few that a round's skip decisions
        # leave, and all eight
        dict(name="batch3_32b", path="verify", shape="qwen32b", layers=2, gamma=32, ctx="2837,513,1900", ws_rows=99),
        dict(name="batch8_32b", path="verify", shape="qwen32b", layers=2, gamma=32,
             ctx="2837,513,3391,1900,1088,3761,284,2250", ws_rows=264),
        # the verifier without a cache: every position of context and drafts again on each call
        dict(name="full_32b", path="full", shape="qwen32b", layers=2, gamma=32, ctx="1024", ws_rows=256),
        # a new sequence: its prompt into the cache, then its first block
        dict(name="prefill_32b", path="prefill", shape="qwen32b", layers=2, gamma=32, ctx="3391", ws_rows=264),
        # the acceptance test of a batch, by argmax and by the ratio of the two models' probabilities
        dict(name="accept_greedy", path="accept", B=16, gamma=32, V=151936, dtype="bf16", mode="greedy", k=1, lenience=1.0),
        dict(name="accept_ratio", path="accept", B=16, gamma=32, V=151936, dtype="bf16", mode="ratio", k=1, lenience=1.0),
        # the skip decision of a batch from the drafter's logits, and of one block from the survival predictor
        dict(name="gate_confidence", path="gate", B=16, gamma=32, V=151936, dtype="bf16"),
        dict(name="gate_survival", path="survival", B=1, gamma=32, d_hid=3584, n_sc=19, H=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["verify", "verify", "verify", "prefill", "full", "accept", "accept", "gate", "survival"])
    if path in ("verify", "prefill", "full"):
        shape = rng.choice(["tiny", "qwen7b", "qwen7b", "qwen32b", "qwen32b"])
        layers = 2 if shape == "tiny" else rng.randint(1, 2)
        n_seq = rng.choice([1, 1, 2, 3, 4, 5, 6, 7, 8]) if path == "verify" else 1
        gamma = rng.choice([0, 1, 3, 7, 8, 15, 16, 31, 32, 32, 32, 33, 47, 63, 64])
        hi = {"verify": 4000, "prefill": 3300, "full": 3300}[path]
        ctx = ",".join(str(_log_int(rng, 16, 300 if shape == "tiny" else hi)) for _ in range(n_seq))
        # the workspace a program allocates: for its verify call, or the 256 rows of the benchmark, or larger
        rows = max(n_seq * (gamma + 1), rng.choice([16, 64, 256, 256, 512, 1024]))
        return dict(path=path, shape=shape, layers=layers, gamma=gamma, ctx=ctx, ws_rows=rows)
    if path == "survival":
        return dict(path=path, B=_log_int(rng, 1, 48), gamma=rng.choice([4, 8, 16, 31, 32, 33]), d_hid=rng.choice([1024, 2048, 3584]),
                    n_sc=19, H=256)
    B, gamma = _log_int(rng, 1, 16), rng.choice([1, 3, 7, 8, 15, 16, 31, 32])
    V = rng.choice([4096, 32000, 50257, 65537, 128256, 151936, 152064])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    if path == "gate":
        return dict(path=path, B=B, gamma=gamma, V=V, dtype=dtype)
    mode = rng.choice(["greedy", "greedy", "topk", "lenient", "ratio"])
    return dict(path=path, B=B, gamma=gamma, V=V, dtype=dtype, mode=mode, k=rng.choice([2, 4, 16]) if mode == "topk" else 1,
                lenience=rng.choice([0.1, 0.3, 0.7]) if mode == "lenient" else 1.0)


def _gen(seed, *ids):
    s = int(seed)
    for i in ids:
        s = (s * 1000003 + int(i) + 17) % (1 << 61)
    return torch.Generator(device=DEV).manual_seed(s)


# ---- decoder -------------------------------------------------------------------------------


def _shape(case):
    return SHAPES[case["shape"]].with_layers(case["layers"])


def _lens(case):
    return [int(x) for x in case["ctx"].split(",")]


def _tensor_shapes(s):
    d, hq, hk = s.d_model, s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim
    top = {sdd.T_EMBED: (s.vocab, d), sdd.T_LM_HEAD: (s.vocab, d), sdd.T_FINAL_NORM: (d,)}
    layer = {sdd.T_WQ: (hq, d), sdd.T_WK: (hk, d), sdd.T_WV: (hk, d), sdd.T_WO: (d, hq), sdd.T_WGATE: (s.d_ff, d),
             sdd.T_WUP: (s.d_ff, d), sdd.T_WDOWN: (d, s.d_ff), sdd.T_ATTN_NORM: (d,), sdd.T_FFN_NORM: (d,)}
    if s.qk_norm:
        layer[sdd.T_Q_NORM] = layer[sdd.T_K_NORM] = (s.head_dim,)
    return top, layer


def _weight(seed, s, kind, layer, shape):
    """Matrices N(0, 0.02) in the model's type, norm gains 1 + 0.1 N(0, 1) in fp32."""
    g = _gen(seed, 1, kind, layer)
    if len(shape) == 1:
        return 1.0 + 0.1 * torch.randn(shape, generator=g, device=DEV)
    dt = torch.bfloat16 if s.dtype == "bf16" else torch.float32
    return torch.empty(shape, dtype=dt, device=DEV).normal_(0.0, W.WEIGHT_SIGMA, generator=g)


def _tokens(case, seed):
    """Per sequence its prompt (ctx + 1 tokens, the last one pending) and the drafted block."""
    s = _shape(case)
    prompts = [torch.randint(0, s.vocab, (n + 1,), generator=_gen(seed, 2, i), device=DEV, dtype=torch.int32)
               for i, n in enumerate(_lens(case))]
    drafts = torch.randint(0, s.vocab, (len(prompts), case["gamma"]), generator=_gen(seed, 3), device=DEV, dtype=torch.int32)
    return prompts, drafts


def _prepare_model(case, seed):
    s = _shape(case)
    model = sdd.Model(s)
    top, layer = _tensor_shapes(s)
    for kind, shp in top.items():
        model.load_tensor(kind, 0, _weight(seed, s, kind, 0, shp))
    for l in range(s.n_layers):
        for kind, shp in layer.items():
            model.load_tensor(kind, l, _weight(seed, s, kind, l, shp))
    prompts, drafts = _tokens(case, seed)
    n, gamma = len(prompts), case["gamma"]
    kv = sdd.KVCache(model, n, max(_lens(case)) + 2 * (gamma + 1) + 8)
    ws = model.workspace(max(case["ws_rows"], n * (gamma + 1)))
    st = dict(case=case, model=model, kv=kv, ws=ws, drafts=drafts, prompts=prompts,
              seqs=torch.arange(n, dtype=torch.int32, device=DEV),
              logits=torch.zeros((n, gamma + 1, s.vocab), dtype=torch.float32, device=DEV),
              argmax=torch.zeros((n, gamma + 1), dtype=torch.int32, device=DEV))
    if case["path"] == "verify":
        for i, p in enumerate(prompts):
            kv.prefill(i, p, ws)
    if case["path"] == "full":
        st["tokens"] = torch.cat([prompts[0], drafts[0]]).contiguous()
    if s.dtype == "f32":
        st["acc_ws"] = sdd.rowstats_workspace(n, gamma, s.vocab)
        st["outs"] = tuple(torch.zeros(n, dtype=torch.int32, device=DEV) for _ in range(3))
    return st


def _run_model(st):
    case, kv, ws = st["case"], st["kv"], st["ws"]
    if case["path"] == "full":
        kv.verify_full(st["tokens"], case["gamma"], st["logits"], st["argmax"], ws)
    else:
        if case["path"] == "prefill":
            kv.prefill(0, st["prompts"][0], ws)
        kv.verify(st["seqs"], st["drafts"], st["logits"], st["argmax"], ws)
    if "outs" not in st:
        return [st["logits"]]
    sdd.accept(st["drafts"], st["logits"], sdd.GREEDY, ws=st["acc_ws"], out=st["outs"])
    return [st["logits"], st["argmax"], st["outs"][0], st["outs"][1]]


def _exact_model(case, seed):
    s = _shape(case)
    top, layer = _tensor_shapes(s)
    prompts, drafts = _tokens(case, seed)
    seqs = [torch.cat([p, d]).long() for p, d in zip(prompts, drafts)]
    lens = [t.numel() for t in seqs]
    hd, hq, hk, eps = s.head_dim, s.n_q_heads, s.n_kv_heads, s.rms_eps
    f64 = torch.float64
    inv = float(s.rope_theta) ** (-torch.arange(0, hd, 2, device=DEV, dtype=f64) / hd)
    ang = torch.arange(max(lens), device=DEV, dtype=f64)[:, None] * inv
    cos, sin = torch.cat([ang.cos()] * 2, -1), torch.cat([ang.sin()] * 2, -1)
    w = lambda kind, l, shp: _weight(seed, s, kind, l, shp).to(f64)  # noqa: E731
    norm = lambda x, g: x * (x.pow(2).mean(-1, keepdim=True) + eps).rsqrt() * g  # noqa: E731
    lin = lambda x, m: torch.cat([c @ m.t() for c in x.split(4096)])  # noqa: E731

    def rope(x, n):  # [n, h, hd]
        rot = torch.cat([-x[..., hd // 2:], x[..., : hd // 2]], -1)
        return x * cos[:n, None] + rot * sin[:n, None]

    x = _weight(seed, s, sdd.T_EMBED, 0, top[sdd.T_EMBED])[torch.cat(seqs)].to(f64)
    for l in range(s.n_layers):
        t = {k: w(k, l, shp) for k, shp in layer.items()}
        h = norm(x, t[sdd.T_ATTN_NORM])
        q, k, v = (lin(h, t[kk]).view(-1, nh, hd) for kk, nh in ((sdd.T_WQ, hq), (sdd.T_WK, hk), (sdd.T_WV, hk)))
        if s.qk_norm:
            q, k = norm(q, t[sdd.T_Q_NORM]), norm(k, t[sdd.T_K_NORM])
        o = torch.empty_like(q)
        at = 0
        for n in lens:
            qs, ks, vs = rope(q[at:at + n], n), rope(k[at:at + n], n), v[at:at + n]
            for j in range(hk):
                qh = qs[:, j * (hq // hk):(j + 1) * (hq // hk)]
                for r in range(0, n, 1024):
                    e = min(n, r + 1024)
                    sc = torch.einsum("rhd,pd->hrp", qh[r:e], ks[:e, j]) / math.sqrt(hd)
                    sc.masked_fill_(torch.arange(e, device=DEV) > torch.arange(r, e, device=DEV)[:, None], -math.inf)
                    o[at + r:at + e, j * (hq // hk):(j + 1) * (hq // hk)] = torch.einsum("hrp,pd->rhd", sc.softmax(-1), vs[:e, j])
            at += n
        x = x + lin(o.reshape(-1, hq * hd), t[sdd.T_WO])
        h = norm(x, t[sdd.T_FFN_NORM])
        y = torch.empty_like(x)
        for r in range(0, x.shape[0], 4096):
            c = h[r:r + 4096]
            y[r:r + 4096] = (torch.nn.functional.silu(c @ t[sdd.T_WGATE].t()) * (c @ t[sdd.T_WUP].t())) @ t[sdd.T_WDOWN].t()
        x = x + y
    R = case["gamma"] + 1
    ends = torch.tensor(lens).cumsum(0).tolist()
    rows = torch.cat([x[e - R:e] for e in ends])
    logits = norm(rows, w(sdd.T_FINAL_NORM, 0, (s.d_model,))) @ w(sdd.T_LM_HEAD, 0, top[sdd.T_LM_HEAD]).t()
    return [logits.view(len(lens), R, s.vocab)] + ([None, None, None] if s.dtype == "f32" else [])


def _work_model(case):
    s = _shape(case)
    es = 2 if s.dtype == "bf16" else 4
    d, hd, L, lens, R = s.d_model, s.head_dim, s.n_layers, _lens(case), case["gamma"] + 1
    per_layer = d * (s.n_q_heads + 2 * s.n_kv_heads) * hd + s.n_q_heads * hd * d + 3 * d * s.d_ff
    out_rows = R * len(lens)
    rows = out_rows if case["path"] == "verify" else lens[0] + R
    # (query, position) pairs of the causal attention
    pairs = sum(R * n + R * (R + 1) // 2 for n in lens) if case["path"] == "verify" else rows * (rows + 1) // 2
    kv_row = 2 * s.n_kv_heads * hd * es
    read = sum(lens) if case["path"] == "verify" else 0
    return {"bytes": (L * per_layer + s.vocab * d) * es + rows * d * es + L * (read + rows) * kv_row + out_rows * s.vocab * 4,
            "flops": 2.0 * rows * L * per_layer + 2.0 * out_rows * s.vocab * d + 4.0 * L * pairs * s.n_q_heads * hd}


# ---- acceptance and skip decisions ----------------------------------------------------------


def _dt(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _prepare_accept(case, seed):
    """Target rows 4 N(0, 1); the draft token is the row's largest by a wide margin with probability 0.85 (prefixes
    of geometric length); the drafter's rows are the target's plus 0.7 N(0, 1)."""
    B, gamma, V, dt = case["B"], case["gamma"], case["V"], _dt(case)
    g = _gen(seed, 4)
    draft = torch.randint(0, V, (B, gamma), generator=g, device=DEV, dtype=torch.int32)
    p = torch.randn((B, gamma + 1, V), generator=g, device=DEV).mul_(4.0)
    top = p[:, :gamma].amax(-1) + 8.0
    hit = torch.rand((B, gamma), generator=g, device=DEV) < 0.85
    idx = draft.long().unsqueeze(-1)
    p[:, :gamma].scatter_(2, idx, torch.where(hit, top, p[:, :gamma].gather(2, idx).squeeze(-1)).unsqueeze(-1))
    q = u = None
    if case["mode"] == "ratio":
        q = torch.randn((B, gamma, V), generator=g, device=DEV).mul_(0.7).add_(p[:, :gamma]).to(dt)
        u = torch.rand((B, gamma), generator=g, device=DEV)
    return dict(case=case, draft=draft, p=p.to(dt), q=q, u=u, ws=sdd.rowstats_workspace(B, gamma, V),
                out=tuple(torch.zeros(B, dtype=torch.int32, device=DEV) for _ in range(3)))


def _run_accept(st):
    c = st["case"]
    return list(sdd.accept(st["draft"], st["p"], MODES[c["mode"]], q=st["q"], uniforms=st["u"], k=c["k"],
                           lenience=c["lenience"], ws=st["ws"], out=st["out"]))


def _prepare_gate(case, seed):
    """Drafter rows 3 N(0, 1) with the draft token raised above the row's maximum by U[0, 30] (confidences from near
    0 to near 1)."""
    B, gamma, V = case["B"], case["gamma"], case["V"]
    g = _gen(seed, 5)
    draft = torch.randint(0, V, (B, gamma), generator=g, device=DEV, dtype=torch.int32)
    z = torch.randn((B, gamma, V), generator=g, device=DEV).mul_(3.0)
    top = z.amax(-1) + torch.rand((B, gamma), generator=g, device=DEV) * 30.0
    z.scatter_(2, draft.long().unsqueeze(-1), top.unsqueeze(-1))
    i32 = lambda: torch.zeros(B, dtype=torch.int32, device=DEV)  # noqa: E731
    return dict(case=case, draft=draft, z=z.to(_dt(case)), ws=sdd.rowstats_workspace(B, gamma, V), skip=i32(),
                log_conf=torch.zeros((B, gamma), dtype=torch.float32, device=DEV), D=i32(), out=(i32(), i32(), i32()))


def _run_gate(st):
    gamma = st["case"]["gamma"]
    skip, lc, lp = sdd.confidence_prefix(st["z"], gamma, 0.7, draft=st["draft"], log_conf=st["log_conf"], ws=st["ws"],
                                         out=st["skip"])
    K, Kh, why = sdd.schedule(lc, st["D"], sdd.SIG_RAW, 0.7, 0.8, k_min=2, s_max=64, draft=st["draft"], rep_max=4, out=st["out"])
    return [lc, lp, skip, K, Kh, why, st["D"]]


def _exact_gate(case, seed):
    st = _prepare_gate(case, seed)
    ls = torch.cat([c.double().log_softmax(-1).unsqueeze(0) for c in st["z"]])
    return [ls.amax(-1), ls.gather(2, st["draft"].long().unsqueeze(-1)).squeeze(-1)] + [None] * 5


def _survival_inputs(case, seed):
    g = _gen(seed, 6)
    n, d_hid, n_sc, H = case["B"] * case["gamma"], case["d_hid"], case["n_sc"], case["H"]
    hidden = (torch.randn((n, d_hid), generator=g, device=DEV) * 1.5).to(torch.bfloat16)
    scalars = torch.rand((n, n_sc), generator=g, device=DEV) * torch.logspace(0, 2, n_sc, device=DEV)
    d_in = d_hid + n_sc
    mu, sigma = torch.zeros(d_in, device=DEV), torch.full((d_in,), 1.5, device=DEV)
    mu[d_hid:], sigma[d_hid:] = scalars.mean(0), torch.logspace(0, 2, n_sc, device=DEV) * 0.29

    def lin(o, i):  # a fresh Linear
        b = 1.0 / math.sqrt(i)
        return ((torch.rand((o, i), generator=g, device=DEV) * 2 - 1) * b, (torch.rand((o,), generator=g, device=DEV) * 2 - 1) * b)

    w = [t for o, i in ((H, d_in), (H, H), (H, H), (1, H)) for t in lin(o, i)]
    return hidden, scalars, mu, sigma, w


def _prepare_survival(case, seed):
    hidden, scalars, mu, sigma, w = _survival_inputs(case, seed)
    B, gamma = case["B"], case["gamma"]
    mlp = sdd.SurvivalMLP(mu, sigma, *w[:7], b4=float(w[7][0]), d_hid=case["d_hid"])
    i32 = lambda: torch.zeros(B, dtype=torch.int32, device=DEV)  # noqa: E731
    return dict(case=case, mlp=mlp, hidden=hidden, scalars=scalars, ws=mlp.workspace(B * gamma),
                score=torch.zeros((B, gamma), dtype=torch.float32, device=DEV),
                logit=torch.zeros((B, gamma), dtype=torch.float32, device=DEV), D=i32(), out=(i32(), i32(), i32()))


def _run_survival(st):
    st["mlp"](st["hidden"], st["scalars"], ws=st["ws"], out=st["score"], logit=st["logit"])
    K, Kh, why = sdd.schedule(st["score"], st["D"], sdd.SIG_CONDITIONAL, 0.3, 0.05, s_max=64, out=st["out"])
    return [st["score"], st["logit"], K, Kh, why, st["D"]]


def _exact_survival(case, seed):
    hidden, scalars, mu, sigma, w = _survival_inputs(case, seed)
    gelu, w = torch.nn.functional.gelu, [t.double() for t in w]
    h = (torch.cat([hidden.double(), scalars.double()], -1) - mu.double()) / sigma.double()
    for i in (0, 2, 4):
        h = gelu(h @ w[i].t() + w[i + 1])
    z = (h @ w[6].t() + w[7]).view(case["B"], case["gamma"])
    return [torch.nn.functional.logsigmoid(z), z] + [None] * 4


# ---- the file's interface ----------------------------------------------------------------------

_PREPARE = {"accept": _prepare_accept, "gate": _prepare_gate, "survival": _prepare_survival}
_RUN = {"accept": _run_accept, "gate": _run_gate, "survival": _run_survival}
_EXACT = {"accept": lambda case, seed: None, "gate": _exact_gate, "survival": _exact_survival}


def prepare(case, seed):
    return _PREPARE.get(case["path"], _prepare_model)(case, seed)


def run(state):
    return _RUN.get(state["case"]["path"], _run_model)(state)


def exact(case, seed):
    return _EXACT.get(case["path"], _exact_model)(case, seed)


def work(case):
    path = case["path"]
    if path in ("verify", "prefill", "full"):
        return _work_model(case)
    if path == "survival":
        n, d_in, H = case["B"] * case["gamma"], case["d_hid"] + case["n_sc"], case["H"]
        return {"bytes": 4 * (H * d_in + 2 * H * H + 4 * H + 2 * d_in) + n * (case["d_hid"] * 2 + case["n_sc"] * 4 + 8),
                "flops": 2.0 * n * (H * d_in + 2 * H * H + H)}
    es = 2 if case["dtype"] == "bf16" else 4
    rows = case["gamma"] + (1 if path == "accept" else 0) + (case["gamma"] if case.get("mode") == "ratio" else 0)
    return {"bytes": case["B"] * rows * case["V"] * es, "flops": 4.0 * case["B"] * rows * case["V"]}


def tolerance(case):
    path = case["path"]
    if path == "accept":
        return "exact"
    if path in ("gate", "survival"):
        return {"rel": 1e-5, "max": 1e-4}
    # BF16: GEMM inputs, q/k/v, the attention output and the hidden layer are rounded to 8 bits in each layer
    return {"rel": 1e-5, "max": 1e-4} if case["shape"] == "tiny" else {"rel": 2.5e-2, "max": 0.3}
