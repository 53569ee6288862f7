"""The calls whose speed this framework is held to, with their inputs, their
unavoidable work and the accuracy they owe.

A student of visual on-policy distillation is rolled out (speculative-Jacobi
windows or cached autoregression), its finished sequences are scored against a
teacher, and the sampling side is also called on its own. The cases are those
calls, through the package's public entry points, on the LlamaGen shapes the
workloads of this repository use (B 768, L 1024, XL 1280 wide, vocabulary
16384, 16x16 and 24x24 grids) and the tiny fp32 one. The wider models run with
fewer layers than they have: their layers are alike, and a pass then costs a
few hundred milliseconds.

Weights depend only on the model (random-init, N(0, 0.02), a fixed seed) and
are loaded once per process, as a training program does; prefixes, labels and
sampling seeds come from the case's seed.
"""
import math

import numpy as np
import torch

import paper_2608_18183_amd as hb

# layers, d, heads, f, vocab, classes, dtype
MODELS = {
    "tiny": (2, 64, 4, 176, 256, 10, "f32"),
    "b": (12, 768, 12, 2048, 16384, 1000, "bf16"),
    "l": (24, 1024, 16, 2816, 16384, 1000, "bf16"),
    "xl": (36, 1280, 20, 3456, 16384, 1000, "bf16"),
}
HISTORY = 24
EPS = 1e-5
ROPE_BASE = 10000.0


def listed():
    return [
        # the exact-parity mode on its test model, the smallest call there is
        # (latency and launches), with the student's logits on the finished
        # sequences, which the distillation loss takes
        dict(name="rollout_tiny_f32", kind="rollout", model="tiny", layers=2, grid=8, batch=4,
             window=4, top_k=0, cfg=0.0, lo=0, hi=16, mode="sjd", commit=2.0, logits=True),
        # the B student's rollout step: short ragged prefixes, rounds of 544
        # rows that are bound by latency and weights
        dict(name="rollout_b", kind="rollout", model="b", layers=12, grid=16, batch=32,
             window=16, top_k=2000, cfg=0.0, lo=0, hi=128, mode="sjd", commit=3.3, logits=False),
        # the cached autoregressive baseline on the same batch: one row per
        # image and round, about 250 rounds
        dict(name="rollout_b_ar", kind="rollout", model="b", layers=12, grid=16, batch=32,
             window=16, top_k=2000, cfg=0.0, lo=0, hi=128, mode="ar", commit=1.0, logits=False),
        # the L student on the 24x24 grid: 1088-row rounds, caches up to 593
        # positions
        dict(name="rollout_l", kind="rollout", model="l", layers=6, grid=24, batch=64,
             window=16, top_k=2000, cfg=0.0, lo=0, hi=288, mode="sjd", commit=3.3, logits=False),
        # the XL student under guidance, the largest rollout: 8448-row rounds
        # at first, a long tail of few active images at last
        dict(name="rollout_xl_cfg", kind="rollout", model="xl", layers=9, grid=16, batch=128,
             window=32, top_k=1000, cfg=2.0, lo=0, hi=128, mode="sjd", commit=2.1, logits=False),
        # one short teacher-forced sequence through the whole B model: the
        # smallest forward, launches and latency
        dict(name="forward_b_one", kind="forward", model="b", layers=12, grid=16, seqs=1, lo=17,
             hi=17),
        # ragged teacher-forced sequences of every length through L layers
        dict(name="forward_l_ragged", kind="forward", model="l", layers=4, grid=24, seqs=24,
             lo=0, hi=576),
        # the XL block at its full width of rows (the prefill of 256 guided
        # sequences has as many): matrix products near the MFMA bound
        dict(name="forward_xl_block", kind="forward", model="xl", layers=2, grid=16, seqs=64,
             lo=131, hi=131),
        # the distillation loss of a finished B batch against an L-wide teacher
        dict(name="score_b", kind="score", model="b", layers=12, teacher="l", teacher_layers=6,
             grid=16, batch=32, lo=0, hi=128),
        # the sampler on one B round's rows: flat logits, top-k 2000
        dict(name="transform_b", kind="transform", rows=544, vocab=16384, cfg=0.0, top_k=2000,
             bias=0.0),
        # the sampler on one XL round's guided rows, peaked and flat
        # temperatures alternating
        dict(name="transform_xl_cfg", kind="transform", rows=4224, vocab=16384, cfg=2.0,
             top_k=1000, bias=4.0),
        # explicit verification of 128 windows of 32 drafts
        dict(name="verify_xl", kind="verify", batch=128, window=32, vocab=16384),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["rollout", "rollout", "forward", "forward", "score", "transform",
                       "transform", "verify"])
    grid = rng.choice([16, 24])
    T = grid * grid
    if kind == "rollout":
        model = rng.choice(["b", "b", "l", "xl"])
        layers = rng.randint(2, {"b": 12, "l": 6, "xl": 4}[model])
        batch = _log(rng, 1, {"b": 64, "l": 48, "xl": 64}[model])
        hi = rng.randint(T // 4, T - 16)
        return dict(kind=kind, model=model, layers=layers, grid=grid, batch=batch,
                    window=_log(rng, 2, 32), top_k=rng.choice([0, 1000, 2000, rng.randint(1, 4000)]),
                    cfg=rng.choice([0.0, 2.0]), lo=hi // 2, hi=hi,
                    mode=rng.choice(["sjd", "sjd", "sjd", "greedy", "ar"]), commit=2.5,
                    logits=False)
    if kind == "forward":
        model = rng.choice(["b", "l", "xl"])
        seqs = _log(rng, 1, 64)
        hi = rng.randint(8, min(T, 9000 // seqs))
        return dict(kind=kind, model=model, layers=rng.randint(1, {"b": 12, "l": 4, "xl": 2}[model]),
                    grid=grid, seqs=seqs, lo=rng.randint(0, hi), hi=hi)
    if kind == "score":
        return dict(kind=kind, model="b", layers=rng.randint(2, 12), teacher="l",
                    teacher_layers=rng.randint(2, 6), grid=16, batch=_log(rng, 1, 32), lo=0,
                    hi=rng.randint(16, 256))
    if kind == "transform":
        vocab = 4 * _log(rng, 256, 4096)
        return dict(kind=kind, rows=_log(rng, 1, 4224), vocab=vocab, cfg=rng.choice([0.0, 2.0]),
                    top_k=rng.choice([0, rng.randint(1, vocab), vocab // 8]),
                    bias=rng.choice([0.0, 4.0]))
    return dict(kind="verify", batch=_log(rng, 1, 128), window=_log(rng, 1, 32),
                vocab=4 * _log(rng, 256, 4096))


# ------------------------------------------------------------------ models

def _layout(model, layers):
    """(rows, columns or None, kind) of each array of the weight blob, in order."""
    _, d, _, f, V, C, _ = MODELS[model]
    out = [((V, d), "w"), ((C + 1, d), "w")]
    for _ in range(layers):
        out += [((d,), "g"), ((3 * d, d), "w"), ((d, d), "w"), ((d,), "g"), ((f, d), "w"),
                ((f, d), "w"), ((d, f), "w")]
    return out + [((d,), "g"), ((V, d), "w")]


def _blob(model, layers):
    """The fp32 weight blob on the GPU and views of its arrays."""
    lay = _layout(model, layers)
    sizes = [int(np.prod(s)) for s, _ in lay]
    gen = torch.Generator("cuda").manual_seed(1234 + layers)
    blob = torch.randn(sum(sizes), generator=gen, device="cuda") * 0.02
    views, off = [], 0
    for (shape, kind), n in zip(lay, sizes):
        v = blob[off:off + n].view(shape)
        if kind == "g":
            v.fill_(1.0)
        views.append(v)
        off += n
    return blob, views


_contexts = {}


def _context(model, layers, grid):
    """The loaded model, kept for the life of the process (the last few)."""
    key = (model, layers, grid)
    if key not in _contexts:
        while len(_contexts) >= 4:
            _contexts.pop(next(iter(_contexts))).close()
        _, d, heads, f, V, C, dt = MODELS[model]
        ctx = hb.Context(hb.ModelDesc(layers, d, heads, f, V, C, grid,
                                      hb.DTYPE_F32 if dt == "f32" else hb.DTYPE_BF16))
        ctx.hbsjd_load_weights(_blob(model, layers)[0].cpu().numpy())
        _contexts[key] = ctx
    else:
        _contexts[key] = _contexts.pop(key)   # last used goes last
    return _contexts[key]


def _tokens(case, n, vocab, gen):
    T = case["grid"] ** 2
    return torch.randint(0, vocab, (n, T), generator=gen, device="cuda", dtype=torch.int32)


def _lens(case, n, rng):
    return rng.integers(case["lo"], case["hi"], size=n, endpoint=True).astype(np.int32)


# ------------------------------------------------------------------ inputs

def _rows(n, vocab, bias, gen):
    x = 0.7 * torch.randn(n, vocab, generator=gen, device="cuda")
    if bias:
        x += bias * torch.randn(vocab, generator=gen, device="cuda")
    return x


def prepare(case, seed):
    gen = torch.Generator("cuda").manual_seed(seed)
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    st = dict(case=case)
    if kind == "rollout":
        _, _, _, _, V, C, _ = MODELS[case["model"]]
        B, T = case["batch"], case["grid"] ** 2
        st.update(ctx=_context(case["model"], case["layers"], case["grid"]),
                  prefix=_tokens(case, B, V, gen), plen=_lens(case, B, rng),
                  labels=rng.integers(0, C, B).astype(np.int32),
                  tau=np.ones(B, np.float32), seed=int(rng.integers(1, 1 << 30)),
                  tokens=torch.empty((B, T), dtype=torch.int32, device="cuda"),
                  counts=torch.empty((T, B), dtype=torch.int32, device="cuda"))
    elif kind == "forward":
        _, _, _, _, V, C, _ = MODELS[case["model"]]
        n = case["seqs"]
        st.update(ctx=_context(case["model"], case["layers"], case["grid"]),
                  tokens=_tokens(case, n, V, gen),
                  # evenly spread lengths in a random order: every seed has as many rows
                  lens=rng.permutation(np.linspace(case["lo"], case["hi"], n).astype(np.int32)),
                  labels=rng.integers(0, C + 1, n).astype(np.int32))
    elif kind == "score":
        _, _, _, _, V, C, _ = MODELS[case["model"]]
        B = case["batch"]
        st.update(ctx=_context(case["model"], case["layers"], case["grid"]),
                  teacher=_context(case["teacher"], case["teacher_layers"], case["grid"]),
                  tokens=_tokens(case, B, V, gen), plen=_lens(case, B, rng),
                  labels=rng.integers(0, C, B).astype(np.int32))
    elif kind == "transform":
        n, V = case["rows"], case["vocab"]
        x = _rows(n, V, case["bias"], gen)
        if case["cfg"]:   # the unconditional row is close to the conditional one
            x = torch.stack([x, 0.9 * x + 0.3 * torch.randn(n, V, generator=gen, device="cuda")], 1)
        tau = torch.ones(n, device="cuda")
        if case["bias"]:
            tau[0::2], tau[1::2] = 0.3, 1.5
        st.update(logits=x.contiguous(), tau=tau, seed=int(rng.integers(1, 1 << 30)),
                  pos=torch.randint(1, 577, (n,), generator=gen, device="cuda", dtype=torch.int32))
    else:
        B, W, V = case["batch"], case["window"], case["vocab"]
        x = _rows(B * W, V, 4.0, gen)
        p = torch.softmax(x, 1).view(B, W, V)
        q = torch.softmax(x + 0.5 * torch.randn(B * W, V, generator=gen, device="cuda"), 1)
        st.update(p=p.contiguous(), q=q.view(B, W, V).contiguous(),
                  drafts=torch.multinomial(q, 1, generator=gen).view(B, W).int().contiguous(),
                  ua=torch.rand(B, W, generator=gen, device="cuda"),
                  ur=torch.rand(B, generator=gen, device="cuda"))
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "rollout":
        mode = {"sjd": hb.VERIFY_PROB, "greedy": hb.VERIFY_GREEDY, "ar": hb.VERIFY_AR}[case["mode"]]
        # gamma = batch is what the calibration of this hardware returns
        st["ctx"].hbsjd_rollout(st["prefix"], st["plen"], st["labels"], st["tau"], case["window"],
                                history=HISTORY, top_k=case["top_k"], cfg_scale=case["cfg"],
                                seed=st["seed"], verify_mode=mode, gamma=case["batch"],
                                max_rounds=case["grid"] ** 2, out_tokens=st["tokens"],
                                out_counts=st["counts"])
        out = dict(tokens=st["tokens"], counts=st["counts"])
        if case["logits"]:
            T = case["grid"] ** 2
            out["logits"] = st["ctx"].hbsjd_forward(
                st["tokens"], np.full(case["batch"], T, np.int32), st["labels"])
        return out
    if kind == "forward":
        return st["ctx"].hbsjd_forward(st["tokens"], st["lens"], st["labels"])
    if kind == "score":
        per, loss = st["ctx"].hbsjd_score_bikl(st["teacher"], st["tokens"], st["plen"],
                                               st["labels"])
        return dict(per_position=per, loss=loss)
    if kind == "transform":
        p, amax, z = hb.hbsjd_transform_rows(st["logits"], st["tau"], st["pos"],
                                             top_k=case["top_k"], cfg_scale=case["cfg"],
                                             seed=st["seed"])
        return dict(p=p, argmax=amax, draw=z)
    counts, tokens = hb.hbsjd_verify_probs(st["p"], st["q"], st["drafts"], st["ua"], st["ur"])
    return dict(counts=counts, tokens=tokens)


# ------------------------------------------------------------------ work

def _layer_weights(model):
    _, d, _, f, _, _, _ = MODELS[model]
    return 4 * d * d + 3 * d * f


def _esz(model):
    return 4 if MODELS[model][6] == "f32" else 2


def _forward_work(model, layers, lens, out_rows, logits_bytes):
    """A teacher-forced forward over sequences of lens + 1 rows, logits of out_rows of them."""
    _, d, _, _, V, _, _ = MODELS[model]
    rows = float(np.sum(np.asarray(lens) + 1))
    pairs = float(np.sum((np.asarray(lens) + 1.0) * (np.asarray(lens) + 2.0) / 2))
    wl = layers * _layer_weights(model)
    flops = 2 * rows * wl + 4.0 * d * layers * pairs + 2.0 * out_rows * V * d
    return (wl + V * d) * _esz(model) + logits_bytes, flops


def work(case):
    kind = case["kind"]
    if kind == "rollout":
        # whole rounds of the algorithm at the mean committed count the
        # random-init students show: every round reads the weights once and the
        # committed keys and values of its active images, and computes W + 1 rows of each
        model, L = case["model"], case["layers"]
        _, d, _, _, V, _, _ = MODELS[model]
        T = case["grid"] ** 2
        B, ncfg = case["batch"], 2 if case["cfg"] else 1
        W = 0 if case["mode"] == "ar" else case["window"]
        commit = min(case["commit"], max(W, 1))
        k = (case["lo"] + case["hi"]) / 2
        rounds = (T - case["lo"]) / commit
        image_rounds = B * (T - k) / commit
        rows = image_rounds * ncfg * (W + 1)
        wl = L * _layer_weights(model)
        ctxlen = (T + k) / 2
        kv = image_rounds * ncfg * ctxlen * 2 * d * L * _esz(model)
        logits = image_rounds * (W + 1) * V * 4 * (ncfg + 1)
        pre = _forward_work(model, L, [k] * (B * ncfg), B * ncfg, 0)
        flops = rows * (2.0 * wl + 2.0 * V * d + 4.0 * d * L * ctxlen) + pre[1]
        out = dict(bytes=rounds * (wl + V * d) * _esz(model) + kv + logits + pre[0], flops=flops)
        if case["logits"]:
            b, fl = _forward_work(model, L, [T] * B, B * (T + 1), B * (T + 1) * V * 4)
            out = dict(bytes=out["bytes"] + b, flops=out["flops"] + fl)
        return out
    if kind == "forward":
        lens = [(case["lo"] + case["hi"]) / 2] * case["seqs"]
        rows = sum(x + 1 for x in lens)
        b, fl = _forward_work(case["model"], case["layers"], lens, rows,
                              rows * MODELS[case["model"]][4] * 4)
        return dict(bytes=b, flops=fl)
    if kind == "score":
        T, B = case["grid"] ** 2, case["batch"]
        out_rows = B * (T - (case["lo"] + case["hi"]) / 2)
        b = fl = 0.0
        for m, layers in ((case["model"], case["layers"]), (case["teacher"], case["teacher_layers"])):
            # the scored logits are written once and read once
            x, y = _forward_work(m, layers, [T - 1] * B, out_rows, out_rows * MODELS[m][4] * 8)
            b, fl = b + x, fl + y
        return dict(bytes=b, flops=fl)
    if kind == "transform":
        n, V = case["rows"], case["vocab"]
        return dict(bytes=n * V * 4.0 * (3 if case["cfg"] else 2) + n * 20, flops=n * V * 8.0)
    # a few probabilities of every draft, and at most one pair of rows per image
    B, W, V = case["batch"], case["window"], case["vocab"]
    return dict(bytes=B * W * 20.0 + B * 2 * V * 4.0, flops=B * V * 4.0)


def tolerance(case):
    kind = case["kind"]
    if kind == "rollout":
        # A rollout's tokens are draws: one flipped draw changes the rest of
        # its image. The same weights, seed and arithmetic give the same tokens.
        return dict(rel=1e-5, max=1e-3, differ=0.01) if case["logits"] else "exact"
    if kind == "forward":
        # attention summed in another order moves the logits by 6.3e-4 of their
        # norm, 3.6e-3 of their rms at most
        return dict(rel=2.5e-3, max=0.015)
    if kind == "score":
        # the same change of order: 2.5e-5 and 1.1e-4
        return dict(rel=1e-4, max=4e-4)
    if kind == "transform":
        return dict(rel=1e-5, max=1e-3, differ=0.005)
    return "exact"


# ------------------------------------------------------------------ 64-bit values

def _exact_forward(model, layers, grid, tokens, lens, labels):
    """fp64 residual rows (before the final norm) of [class, x_1..x_len] of each
    sequence, concatenated, and the fp64 lm_head."""
    _, d, H, f, V, C, dt = MODELS[model]
    _, w = _blob(model, layers)
    mats = [(v if v.dim() == 1 or dt == "f32" else v.bfloat16()) for v in w]
    del w
    T = grid * grid
    s = torch.arange(T + 1, device="cuda")
    row = torch.where(s > 0, (s - 1) // grid, 0).double()
    col = torch.where(s > 0, (s - 1) % grid, 0).double()
    dh = d // H
    th = ROPE_BASE ** (-4.0 * torch.arange(dh // 4, device="cuda", dtype=torch.float64) / dh)
    ang = torch.cat([row[:, None] * th, col[:, None] * th], 1)
    ang[0] = 0
    cs, sn = ang.cos(), ang.sin()
    rows = [int(n) + 1 for n in lens]
    tok_emb, cls_emb = mats[0].double(), mats[1].double()
    h = torch.cat([torch.cat([cls_emb[int(labels[q])][None], tok_emb[tokens[q, :rows[q] - 1].long()]])
                   for q in range(len(rows))])
    pos = torch.cat([torch.arange(n, device="cuda") for n in rows])
    c, sn = cs[pos][:, None], sn[pos][:, None]

    def norm(x, g):
        return x * torch.rsqrt(x.square().mean(1, keepdim=True) + EPS) * g.double()

    def rope(x):
        x = x.view(-1, H, dh // 2, 2)
        a, b = x[..., 0], x[..., 1]
        return torch.stack([a * c - b * sn, a * sn + b * c], -1).view(-1, H, dh)

    for layer in range(layers):
        ga, wqkv, wo, gf, w1, w3, w2 = mats[2 + 7 * layer:9 + 7 * layer]
        x = norm(h, ga) @ wqkv.double().t().contiguous()
        q, k, v = rope(x[:, :d]), rope(x[:, d:2 * d]), x[:, 2 * d:].view(-1, H, dh)
        o, r0 = torch.empty_like(v), 0
        for n in rows:
            qq, kk, vv = (t[r0:r0 + n].transpose(0, 1).contiguous() for t in (q, k, v))
            a = qq @ kk.transpose(1, 2).contiguous() / math.sqrt(dh)
            a = a.masked_fill(torch.ones(n, n, dtype=torch.bool, device="cuda").triu(1), -math.inf)
            o[r0:r0 + n] = (torch.softmax(a, -1) @ vv).transpose(0, 1)
            r0 += n
        h = h + o.reshape(-1, d) @ wo.double().t().contiguous()
        x = norm(h, gf)
        x = torch.nn.functional.silu(x @ w1.double().t().contiguous()) * (x @ w3.double().t().contiguous())
        h = h + x @ w2.double().t().contiguous()
    return norm(h, mats[-2]), mats[-1].double().t().contiguous()


def exact(case, seed):
    kind = case["kind"]
    if kind in ("rollout", "verify"):
        return None
    st = prepare(case, seed)
    if kind == "forward":
        h, w = _exact_forward(case["model"], case["layers"], case["grid"], st["tokens"],
                              st["lens"], st["labels"])
        return h @ w
    if kind == "score":
        T, B = case["grid"] ** 2, case["batch"]
        per = torch.zeros(B, T, dtype=torch.float64, device="cuda")
        rows = [_exact_forward(m, n, case["grid"], st["tokens"], [T - 1] * B, st["labels"])
                for m, n in ((case["model"], case["layers"]),
                             (case["teacher"], case["teacher_layers"]))]
        for b in range(B):
            k = int(st["plen"][b])
            if k >= T:
                continue
            ls, lt = (torch.log_softmax(h[b * T + k:(b + 1) * T] @ w, 1) for h, w in rows)
            per[b, k:] = ((ls.exp() - lt.exp()) * (ls - lt)).sum(1) / 2
        n = torch.tensor(T - st["plen"], device="cuda").clamp(min=1).double()
        return dict(per_position=per, loss=per.sum(1) / n)
    x = st["logits"].double()
    V = case["vocab"]
    l = x[:, 1] + case["cfg"] * (x[:, 0] - x[:, 1]) if case["cfg"] else x
    y = l / st["tau"].double()[:, None]
    if 0 < case["top_k"] < V:
        y = y.masked_fill(y < y.topk(case["top_k"], 1).values[:, -1:], -math.inf)
    return dict(p=torch.softmax(y, 1), argmax=None, draw=None)
