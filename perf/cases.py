"""The work that performance is measured on: calls of the framework's public entry points as a training program makes
them, over the range of shapes it supports.

Kinds of case:
  stage      forward and backward of a pipeline stage (mls.Stage): `layers` decoder layers over `microbatches`
             micro-batches.  `order`: "batched" = all forwards, then one backward call that writes the gradients;
             "1f1b" = one forward, one backward, the first call writing the gradients and the others adding to them;
             "forward" = forward only (evaluation), the stash dropped afterwards.
  head       last stage: final RMSNorm, LM head, loss, and their backward over `microbatches` (mls.Ends)
  embedding  first stage: token embedding and its gradient over `microbatches` (mls.Ends)
  update     between two steps: AdamW on a layer's parameters and their write-back into the stage

Every pass of a head or embedding case adds to the same gradient vector, as the calls of one step do.  All inputs are
drawn from the seed on the GPU: activations and upstream gradients N(0, 1), projections 0.02 N(0, 1), gains
1 + 0.02 N(0, 1), token ids uniform over the vocabulary.
"""
import math

import torch

import paper_2410_13333_amd as mls

EPS, ROPE_BASE = 1e-5, 10000.0


def _stage(name, hidden, n_q, n_kv, head_dim, ffn, seq, micro_batch, layers, microbatches, order="batched", dtype="bf16",
           recompute=False):
    return {"name": name, "kind": "stage", "hidden": hidden, "n_q": n_q, "n_kv": n_kv, "head_dim": head_dim, "ffn": ffn,
            "seq": seq, "micro_batch": micro_batch, "layers": layers, "microbatches": microbatches, "order": order,
            "dtype": dtype, "recompute": recompute}


def listed():
    return [
        # the smallest model a test or a smoke run trains: launches and latency
        _stage("tiny_step", 256, 4, 4, 64, 688, 128, 2, 2, 1),
        # a small model with grouped KV heads, an odd sequence length and an ffn that is no multiple of 32, in the
        # one-forward-one-backward order of a pipeline
        _stage("ragged_gqa_1f1b", 1024, 16, 4, 64, 2728, 1000, 2, 1, 3, order="1f1b"),
        # an ordinary mid-size layer
        _stage("mid_layer", 2048, 16, 16, 128, 5504, 2048, 1, 1, 2),
        # the stage step of the headline benchmark: 7B layer shape, 4 layers x 4 micro-batches
        _stage("stage_7b_4x4", 4096, 32, 32, 128, 11008, 4096, 1, 4, 4),
        # evaluation: one 7B layer forward
        _stage("forward_7b_layer", 4096, 32, 32, 128, 11008, 4096, 1, 1, 1, order="forward"),
        # the other two large layer shapes of the benchmark
        _stage("layer_13b", 5120, 40, 40, 128, 13824, 4096, 1, 1, 2),
        _stage("layer_70b_tp4", 8192, 16, 2, 128, 7168, 4096, 1, 1, 2),
        # the shorter context of the plan sweep, memory-bound plan: activation recomputation, pipeline order
        _stage("sweep_recompute_1f1b", 4096, 32, 32, 128, 11008, 2048, 1, 2, 2, order="1f1b", recompute=True),
        # the fp32 storage mode that gradients are validated with
        _stage("fp32_step", 512, 8, 4, 64, 1376, 256, 2, 1, 2, dtype="fp32"),
        # last and first stage of a 7B-shaped model (vocabulary 32000), and the update of one of its layers
        {"name": "head_7b", "kind": "head", "hidden": 4096, "vocab": 32000, "seq": 4096, "micro_batch": 1,
         "microbatches": 2, "dtype": "bf16"},
        {"name": "embedding_7b", "kind": "embedding", "hidden": 4096, "vocab": 32000, "seq": 4096, "micro_batch": 1,
         "microbatches": 4, "dtype": "bf16"},
        {"name": "update_7b_layer", "kind": "update", "hidden": 4096, "n_q": 32, "n_kv": 32, "head_dim": 128, "ffn": 11008,
         "layers": 1, "dtype": "bf16"},
    ]


def draw(rng):
    def log_int(lo, hi, mult=1):
        v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        return max(lo, min(hi, int(round(v / mult)) * mult))

    kind = rng.choice(["stage"] * 7 + ["head", "embedding", "update"])
    if kind == "stage":
        fp32 = rng.random() < 0.1
        for _ in range(100):
            c = _stage("", log_int(192, 768 if fp32 else 8192, 8), 0, rng.choice([1, 2, 3, 4, 8, 16, 32]),
                       rng.choice([64, 128]), 0, log_int(48, 384 if fp32 else 4096), rng.choice([1, 1, 2, 3]),
                       rng.choice([1, 1, 2]), rng.choice([1, 2, 3]), order=rng.choice(["batched", "batched", "1f1b", "forward"]),
                       dtype="fp32" if fp32 else "bf16", recompute=rng.random() < 0.15)
            del c["name"]
            if rng.random() < 0.5:  # common widths are multiples of 256
                c["hidden"] = max(256, c["hidden"] // 256 * 256)
            c["n_q"] = c["n_kv"] * rng.choice([1, 1, 2, 4, 8])
            c["ffn"] = max(64, int(c["hidden"] * rng.uniform(0.8, 3.6)) // 8 * 8)
            qd = c["n_q"] * c["head_dim"]
            # query width in proportion to the hidden width, and no more work than the largest listed case
            if c["hidden"] / 4 <= qd <= 2 * c["hidden"] and _stage_flops(c) < 4e13:
                return c
        return _stage("", 512, 8, 4, 64, 1376, 513, 1, 1, 2) | {"seq": rng.randrange(65, 2048)}
    dt = "fp32" if rng.random() < 0.1 else "bf16"
    if kind == "head":
        return {"kind": kind, "hidden": log_int(256, 1024 if dt == "fp32" else 8192, 8), "vocab": log_int(512, 4096 if dt == "fp32" else 50304, 8),
                "seq": log_int(64, 512 if dt == "fp32" else 4096), "micro_batch": rng.choice([1, 2]), "microbatches": rng.choice([1, 2, 3]), "dtype": dt}
    if kind == "embedding":
        return {"kind": kind, "hidden": log_int(256, 8192, 8), "vocab": log_int(512, 50304, 8), "seq": log_int(64, 4096),
                "micro_batch": rng.choice([1, 2]), "microbatches": rng.choice([1, 2, 4]), "dtype": dt}
    h = log_int(256, 4096, 8)
    hd = rng.choice([64, 128])
    nkv = max(1, h // hd // rng.choice([1, 2, 4]))
    return {"kind": kind, "hidden": h, "n_q": nkv * rng.choice([1, 2]), "n_kv": nkv, "head_dim": hd,
            "ffn": int(h * rng.uniform(1, 3)) // 8 * 8, "layers": rng.choice([1, 2]), "dtype": dt}


# ---------------------------------------------------------------- layouts and inputs
def _widths(c):
    qd, kvd = c["n_q"] * c["head_dim"], c["n_kv"] * c["head_dim"]
    return qd, kvd


def _layer_shapes(c):
    """(name, rows, cols) of one layer's parameters in the public order."""
    h, f = c["hidden"], c["ffn"]
    qd, kvd = _widths(c)
    return [("gamma1", 1, h), ("w_qkv", h, qd + 2 * kvd), ("w_o", qd, h), ("gamma2", 1, h), ("w_gu", h, 2 * f), ("w_d", f, h)]


def _ends_shapes(c):
    return [("embed", c["vocab"], c["hidden"]), ("gamma_f", 1, c["hidden"]), ("w_lm", c["hidden"], c["vocab"])]


def _views(flat, shapes, layers=1):
    out, at = [], 0
    for _ in range(layers):
        d = {}
        for name, r, k in shapes:
            d[name] = flat[at:at + r * k].view(r, k)
            at += r * k
        out.append(d)
    return out


def _dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)


def _params(shapes, layers, dtype, g):
    n = layers * sum(r * k for _, r, k in shapes)
    flat = torch.empty(n, dtype=dtype, device="cuda")
    for d in _views(flat, shapes, layers):
        for name, t in d.items():
            z = torch.randn(t.shape, device="cuda", generator=g) * 0.02
            t.copy_(z + 1.0 if name.startswith("gamma") else z)
    return flat


def _normal(shape, dtype, g):
    return torch.randn(shape, device="cuda", generator=g).to(dtype)


def _inputs(c, seed):
    """Everything that is drawn from the seed, on the GPU."""
    g, dt = _gen(seed), _dtype(c)
    if c["kind"] == "stage":
        m, act = c["microbatches"], (c["micro_batch"], c["seq"], c["hidden"])
        return {"params": _params(_layer_shapes(c), c["layers"], dt, g), "x": [_normal(act, dt, g) for _ in range(m)],
                "dy": _normal((m,) + act, dt, g)}
    if c["kind"] == "update":
        p = _params(_layer_shapes(c), c["layers"], dt, g)
        return {"params": p, "grads": torch.randn(p.numel(), device="cuda", generator=g) * 0.01}
    m, T, act = c["microbatches"], c["micro_batch"] * c["seq"], (c["micro_batch"], c["seq"], c["hidden"])
    ids = lambda: torch.randint(0, c["vocab"], (T,), device="cuda", generator=g, dtype=torch.int32)  # noqa: E731
    p = _params(_ends_shapes(c), 1, dt, g)
    if c["kind"] == "head":
        return {"params": p, "y": [_normal(act, dt, g) for _ in range(m)], "targets": [ids() for _ in range(m)]}
    return {"params": p, "tokens": [ids() for _ in range(m)], "dx": _normal((m,) + act, dt, g)}


# ---------------------------------------------------------------- what a program has in hand, and one pass
def prepare(case, seed):
    c, s = case, _inputs(case, seed)
    s["case"] = c
    if c["kind"] in ("stage", "update"):
        up = c["kind"] == "update"
        st = mls.Stage(c["hidden"], c["n_q"], c["n_kv"], c["head_dim"], c["ffn"], 128 if up else c["seq"],
                       1 if up else c["micro_batch"], c["layers"], 1 if up or c["order"] != "batched" else c["microbatches"],
                       EPS, ROPE_BASE, c["dtype"], seed=seed, recompute=not up and c["recompute"])
        s["stage"] = st
        if up:
            s["optim"] = mls.Optim(s["params"])
        else:
            st.set_params(s.pop("params"))
            s["y"] = [torch.empty_like(x) for x in s["x"]]
            if c["order"] != "forward":
                s["dx"] = torch.empty_like(s["dy"])
                s["grads"] = torch.zeros(st.grad_elems, dtype=torch.float32, device="cuda")
    else:
        en = mls.Ends(c["hidden"], c["vocab"], c["seq"], c["micro_batch"], c["microbatches"], EPS, c["dtype"], seed=seed)
        en.set_params(s.pop("params"))
        s["ends"] = en
        s["grads"] = torch.zeros(en.grad_elems, dtype=torch.float32, device="cuda")
        if c["kind"] == "head":
            s["dy"] = torch.empty((c["microbatches"],) + tuple(s["y"][0].shape), dtype=s["y"][0].dtype, device="cuda")
            s["loss"] = torch.zeros(c["microbatches"], dtype=torch.float32, device="cuda")
        else:
            s["x"] = [torch.empty_like(s["dx"][0]) for _ in range(c["microbatches"])]
    return s


def run(state):
    s, c = state, state["case"]
    m = c.get("microbatches", 1)
    if c["kind"] == "stage":
        st, k = s["stage"], c["layers"]
        if c["order"] == "forward":
            for i in range(m):
                st.forward(s["x"][i], k, s["y"][i])
                st.reset()
            return {"y": s["y"]}
        if c["order"] == "batched":
            for i in range(m):
                st.forward(s["x"][i], k, s["y"][i])
            st.backward(s["dy"], s["grads"], m, s["dx"], overwrite=True)
        else:
            for i in range(m):
                st.forward(s["x"][i], k, s["y"][i])
                st.backward(s["dy"][i:i + 1], s["grads"], 1, s["dx"][i:i + 1], overwrite=i == 0)
        return {"y": s["y"], "dx": s["dx"], "grads": _views(s["grads"], _layer_shapes(c), k)}
    if c["kind"] == "head":
        en = s["ends"]
        for i in range(m):
            en.head_forward(s["y"][i], s["targets"][i], 1.0 / m, s["loss"][i:i + 1])
        en.head_backward(s["grads"], m, s["dy"])
        d = _views(s["grads"], _ends_shapes(c))[0]
        return {"loss": s["loss"], "dy": s["dy"], "gamma_f": d["gamma_f"], "w_lm": d["w_lm"]}
    if c["kind"] == "embedding":
        en = s["ends"]
        for i in range(m):
            en.embed_forward(s["tokens"][i], s["x"][i])
        en.embed_backward(s["dx"], s["grads"], m)
        return {"x": s["x"], "embed": _views(s["grads"], _ends_shapes(c))[0]["embed"]}
    s["optim"].step(s["grads"], s["params"], lr=3e-4, grad_scale=0.25)
    s["stage"].set_params(s["params"])
    return s["params"]


# ---------------------------------------------------------------- work, tolerance
def _layer_elems(c):
    return sum(r * k for _, r, k in _layer_shapes(c))


def _stage_flops(c):
    T, (qd, kvd) = c["seq"] * c["micro_batch"], _widths(c)
    mats = c["hidden"] * (qd + 2 * kvd) + qd * c["hidden"] + 3 * c["hidden"] * c["ffn"]
    one = 2 * T * mats + 4 * c["micro_batch"] * qd * c["seq"] * (c["seq"] + 1) // 2
    return (1 if c["order"] == "forward" else 3) * one * c["layers"] * c["microbatches"]


def work(case):
    c, es = case, 2 if case["dtype"] == "bf16" else 4
    if c["kind"] == "update":  # master, two moments, gradient in; master, moments, parameters out; parameters to the stage
        n = c["layers"] * _layer_elems(c)
        return {"bytes": n * (28 + 2 * es), "flops": 12 * n}
    m, act = c["microbatches"], c["micro_batch"] * c["seq"] * c["hidden"] * es
    if c["kind"] == "stage":
        n = c["layers"] * _layer_elems(c)
        if c["order"] == "forward":
            return {"bytes": n * es + 2 * m * act, "flops": _stage_flops(c)}
        return {"bytes": n * (es + 4) + 4 * m * act, "flops": _stage_flops(c)}
    T, h, V = c["micro_batch"] * c["seq"], c["hidden"], c["vocab"]
    if c["kind"] == "head":  # w_lm once, its fp32 gradient read and written, y and dY
        return {"bytes": h * V * (es + 8) + 2 * m * act, "flops": 6 * m * T * h * V}
    rows = V * (1 - (1 - 1 / V) ** (m * T))  # table rows that some token names: gathered, their gradient read and written
    return {"bytes": int(rows * h * (es + 8)) + 2 * m * act, "flops": m * T * h}


def tolerance(case):
    """bf16 storage: relative error of a correct bf16 path grows with depth (one 7B layer measures 4e-3 in y and 8e-3 in
    its worst parameter gradient against 64 bits, four layers 2.3e-2); fp32 storage and sums: 1e-5."""
    c = case
    if c["kind"] == "embedding":
        return {"rel": 1e-5, "max": 1e-4}
    if c["kind"] == "update":  # a parameter on the edge between two bf16 values may round either way
        return {"rel": 2e-4, "max": 0.02} if c["dtype"] == "bf16" else {"rel": 1e-6, "max": 1e-5}
    if c["dtype"] == "fp32":
        return {"rel": 2e-5, "max": 1e-3}
    if c["kind"] == "head":
        return {"rel": 1e-2, "max": 0.3}
    return {"rel": min(0.025, 0.006 * (1 + c["layers"])), "max": 0.5}


# ---------------------------------------------------------------- the same in 64 bits
def _rms_fwd(x, gamma):
    r = (x.square().mean(-1, keepdim=True) + EPS).rsqrt()
    return x * r * gamma, r


def _rms_bwd(da, x, gamma, r):
    n, dn = x * r, da * gamma
    return r * (dn - n * (dn * n).mean(-1, keepdim=True)), (da * n).sum(0, keepdim=True)


def _rotate(u, cs, sn):
    """u [b, S, heads, d], angles [S, d/2]"""
    a, b = u.chunk(2, dim=-1)
    cs, sn = cs[None, :, None], sn[None, :, None]
    return torch.cat([a * cs - b * sn, a * sn + b * cs], dim=-1)


def _layer_fwd(x, w, c, cs, sn):
    b, S, h = c["micro_batch"], c["seq"], c["hidden"]
    nq, nkv, d, f = c["n_q"], c["n_kv"], c["head_dim"], c["ffn"]
    qd, kvd = _widths(c)
    a, r1 = _rms_fwd(x, w["gamma1"])
    qkv = a @ w["w_qkv"]
    qk = _rotate(qkv[:, :qd + kvd].reshape(b, S, nq + nkv, d), cs, sn)
    v = qkv[:, qd + kvd:].reshape(b, S, nkv, d)
    mask = torch.ones(S, S, dtype=torch.bool, device=x.device).triu(1)
    o = torch.empty(b, S, nq, d, dtype=x.dtype, device=x.device)
    for i in range(b):
        for q in range(nq):
            k = q // (nq // nkv)
            p = (qk[i, :, q] @ qk[i, :, nq + k].t() / math.sqrt(d)).masked_fill_(mask, -math.inf).softmax(-1)
            o[i, :, q] = p @ v[i, :, k]
    o = o.reshape(b * S, qd)
    hh = x + o @ w["w_o"]
    bb, r2 = _rms_fwd(hh, w["gamma2"])
    gu = bb @ w["w_gu"]
    g, u = gu[:, :f], gu[:, f:]
    z = g * torch.sigmoid(g) * u
    return hh + z @ w["w_d"], (x, a, r1, qk, v, o, hh, bb, r2, g, u, z, mask)


def _layer_bwd(dy, w, cache, c, cs, sn):
    x, a, r1, qk, v, o, hh, bb, r2, g, u, z, mask = cache
    b, S = c["micro_batch"], c["seq"]
    nq, nkv, d = c["n_q"], c["n_kv"], c["head_dim"]
    G = {"w_d": z.t() @ dy}
    dz = dy @ w["w_d"].t()
    s = torch.sigmoid(g)
    dgu = torch.cat([dz * u * s * (1 + g * (1 - s)), dz * g * s], dim=1)
    G["w_gu"] = bb.t() @ dgu
    dn, G["gamma2"] = _rms_bwd(dgu @ w["w_gu"].t(), hh, w["gamma2"], r2)
    dh = dy + dn
    G["w_o"] = o.t() @ dh
    do = (dh @ w["w_o"].t()).reshape(b, S, nq, d)
    dqk, dv = torch.zeros_like(qk), torch.zeros_like(v)
    for i in range(b):
        for q in range(nq):
            k = q // (nq // nkv)
            Q, K, V, dO = qk[i, :, q], qk[i, :, nq + k], v[i, :, k], do[i, :, q]
            p = (Q @ K.t() / math.sqrt(d)).masked_fill_(mask, -math.inf).softmax(-1)
            dv[i, :, k] += p.t() @ dO
            dp = dO @ V.t()
            ds = p * (dp - (p * dp).sum(-1, keepdim=True)) / math.sqrt(d)
            dqk[i, :, q] = ds @ K
            dqk[i, :, nq + k] += ds.t() @ Q
    dqkv = torch.cat([_rotate(dqk, cs, -sn).reshape(b * S, -1), dv.reshape(b * S, -1)], dim=1)
    G["w_qkv"] = a.t() @ dqkv
    dn, G["gamma1"] = _rms_bwd(dqkv @ w["w_qkv"].t(), x, w["gamma1"], r1)
    return dh + dn, G


def _exact_stage(c, s):
    shapes = _layer_shapes(c)
    W = [{n: t.double() for n, t in d.items()} for d in _views(s["params"], shapes, c["layers"])]
    theta = ROPE_BASE ** (-2.0 * torch.arange(c["head_dim"] // 2, dtype=torch.float64, device="cuda") / c["head_dim"])
    ang = torch.arange(c["seq"], dtype=torch.float64, device="cuda")[:, None] * theta[None, :]
    cs, sn = ang.cos(), ang.sin()
    T, h, ys, dxs, grads = c["seq"] * c["micro_batch"], c["hidden"], [], [], None
    for i, x in enumerate(s["x"]):
        t, caches = x.double().reshape(T, h), []
        for w in W:
            t, cache = _layer_fwd(t, w, c, cs, sn)
            caches.append(cache)
        ys.append(t.reshape(x.shape))
        if c["order"] == "forward":
            continue
        d, own = s["dy"][i].double().reshape(T, h), []
        for w, cache in zip(reversed(W), reversed(caches)):
            d, G = _layer_bwd(d, w, cache, c, cs, sn)
            own.insert(0, G)
        dxs.append(d.reshape(x.shape))
        if grads is None:
            grads = own
        else:
            for a, b in zip(grads, own):
                for n in a:
                    a[n] += b[n]
    return {"y": ys} if c["order"] == "forward" else {"y": ys, "dx": torch.stack(dxs), "grads": grads}


def _exact_head(c, s):
    p = {n: t.double() for n, t in _views(s["params"], _ends_shapes(c))[0].items()}
    T, h, m = c["seq"] * c["micro_batch"], c["hidden"], c["microbatches"]
    loss, dys, gw, gg = [], [], torch.zeros_like(p["w_lm"]), torch.zeros_like(p["gamma_f"])
    for y, tgt in zip(s["y"], s["targets"]):
        t = y.double().reshape(T, h)
        n, r = _rms_fwd(t, p["gamma_f"])
        z = n @ p["w_lm"]
        lse = z.logsumexp(-1)
        at = tgt.long()[:, None]
        loss.append((lse - z.gather(1, at)[:, 0]).mean())
        dz = (z - lse[:, None]).exp_()
        dz.scatter_add_(1, at, torch.full_like(at, -1, dtype=dz.dtype))
        dz /= T * m
        gw += n.t() @ dz
        d, dg = _rms_bwd(dz @ p["w_lm"].t(), t, p["gamma_f"], r)
        gg += dg
        dys.append(d.reshape(y.shape))
    return {"loss": torch.stack(loss), "dy": torch.stack(dys), "gamma_f": gg, "w_lm": gw}


def exact(case, seed):
    c, s = case, _inputs(case, seed)
    if c["kind"] == "stage":
        return _exact_stage(c, s)
    if c["kind"] == "head":
        return _exact_head(c, s)
    if c["kind"] == "embedding":
        E = _views(s["params"], _ends_shapes(c))[0]["embed"]
        x = [E.double()[t.long()].reshape(s["dx"][0].shape) for t in s["tokens"]]
        g = torch.zeros(E.shape, dtype=torch.float64, device="cuda")
        for t, d in zip(s["tokens"], s["dx"]):
            g.index_add_(0, t.long(), d.double().reshape(t.numel(), -1))
        return {"x": x, "embed": g}
    w, g = s["params"].double(), s["grads"].double() * 0.25  # first step: both moments start at zero
    return w - 3e-4 * (g / (g.abs() + 1e-8) + 0.1 * w)
