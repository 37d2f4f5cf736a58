"""The calls this package is used for, as measurable cases.

A case is a dict of plain values.  "op" names the layer of an AF3 pair stack:

  attn  triangle attention over a whole pair map, or over a batch of them
        (binding.fwd, binding.bwd, binding.triangle_attention)
  rows  one GPU's share of a row-sharded triangle attention
        (binding.rows_fwd, binding.rows_bwd)
  lnl   the fused layer-norm + linear projection that makes the attention's
        inputs from the pair representation (binding.ln_linear_fwd / _bwd)
  trn   the fused transition layer (binding.transition_fwd / _bwd)

and "mode" is what the caller does with it: "infer" (a forward), "train" (a
forward and its backward, called one after the other) or "autograd" (the same
through torch.autograd).  The pair representation of a map of n tokens has
m = n * n rows for lnl and trn.
"""
import math

import torch

from paper_2506_20686_amd import binding as B

EPS = 1e-5


def _attn(name, n, mode, node="start", dtype="bf16", h=4, d=32, batch=0, pad=0, bias_std=1.0):
    return {"name": name, "op": "attn", "mode": mode, "node": node, "dtype": dtype, "batch": batch,
            "n": n, "h": h, "d": d, "pad": pad, "bias_std": bias_std}


def listed():
    return [
        # the smallest training call: a short peptide in fp32, bound by launches
        _attn("attn_f32_n32_train", 32, "train", dtype="f32"),
        # inference on a small, padded complex (the last tenth of the keys masked)
        _attn("attn_n256_pad_infer", 256, "infer", pad=25),
        # training at a crop of 384 tokens, ending node, random padding length
        _attn("attn_n384_end_autograd", 384, "autograd", node="end", pad=41),
        # training at a crop of 768 tokens: the benchmark's map, starting node
        _attn("attn_n768_train", 768, "train", bias_std=math.sqrt(2.0)),
        # inference on a long complex (the last keys padded): the largest call
        _attn("attn_n1536_pad_infer", 1536, "infer", pad=76),
        # a batch of small ragged maps with narrow heads, ending node, training
        _attn("attn_b4_n201_d16_end_train", 201, "train", node="end", d=16, batch=4, pad=12,
              bias_std=math.sqrt(2.0)),
        # a ragged map with wide heads, starting node, training
        _attn("attn_n333_d64_train", 333, "train", d=64),
        # fp32 inference on a ragged map: reference runs and debugging
        _attn("attn_f32_n193_infer", 193, "infer", dtype="f32", pad=9),
        # one of eight GPUs' rows of the 768-token map, training
        {"name": "rows_n768_r96_train", "op": "rows", "mode": "train", "dtype": "bf16", "n": 768,
         "rows": 96, "h": 4, "d": 32, "pad": 0, "bias_std": math.sqrt(2.0)},
        # the attention's input projection (Q, K, V, G, bias) at 768 tokens, training
        {"name": "lnl_n768_train", "op": "lnl", "mode": "train", "m": 768 * 768,
         "widths": "128,128,128,128,4"},
        # the pair transition (hidden width 4 * 128) at 768 tokens, training
        {"name": "trn_n768_train", "op": "trn", "mode": "train", "m": 768 * 768, "f": 512},
        # the pair transition on a ragged mid-sized map, inference
        {"name": "trn_n345_infer", "op": "trn", "mode": "infer", "m": 345 * 345, "f": 512},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# the largest listed call's multiply-adds bound a drawn one's
MAX_FLOPS = 1.5e12


def draw(rng):
    op = rng.choice(["attn"] * 5 + ["rows"] + ["lnl"] * 2 + ["trn"] * 2)
    if op == "attn":
        dtype = rng.choice(["bf16"] * 4 + ["f32"])
        mode = rng.choice(["infer", "train", "autograd"])
        d = rng.choice([32, 32, 32, 16, 64])
        h = rng.choice([4, 4, 4, 8, 2])
        batch = rng.choice([0, 0, 0, 2, 3])
        n = _log_int(rng, 24, 900 if dtype == "bf16" else 224)
        while 14.0 * max(batch, 1) * n ** 3 * h * d > MAX_FLOPS:
            n = n * 7 // 8
        pad = rng.choice([0, rng.randint(0, n * 15 // 100)])
        return {"op": op, "mode": mode, "node": rng.choice(["start", "end"]), "dtype": dtype,
                "batch": batch, "n": n, "h": h, "d": d, "pad": pad,
                "bias_std": rng.choice([1.0, math.sqrt(2.0)])}
    if op == "rows":
        n = _log_int(rng, 96, 1024)
        rows = max(1, n // rng.choice([2, 4, 8, 16]) + rng.randint(0, 3))
        return {"op": op, "mode": rng.choice(["infer", "train"]), "dtype": "bf16", "n": n,
                "rows": rows, "h": 4, "d": 32, "pad": rng.choice([0, n * 5 // 100]),
                "bias_std": math.sqrt(2.0)}
    mode = rng.choice(["infer", "train", "train"])
    n = _log_int(rng, 24, 768)
    m = n * max(1, n // rng.choice([1, 1, 1, 4]))  # whole maps, and row shards of them
    if op == "lnl":
        widths = rng.choice(["128,128,128,128,4", "128,128,128,128,4", "128,128,128,128,8",
                             "64,64,64,64,4", "128,128,128"])
        return {"op": op, "mode": mode, "m": m, "widths": widths}
    return {"op": op, "mode": mode, "m": m, "f": rng.choice([512, 512, 256, 128])}


# ---- inputs ------------------------------------------------------------------------

def _normal(gen, shape, std=1.0, mean=0.0, dtype=torch.bfloat16):
    t = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
    return t.mul_(std).add_(mean).to(dtype)


def _widths(case):
    return [int(c) for c in case["widths"].split(",")]


def _node(case):
    return B.ENDING if case.get("node") == "end" else B.STARTING


def _inputs(case, seed):
    gen = torch.Generator("cuda").manual_seed(int(seed))
    op = case["op"]
    if op in ("attn", "rows"):
        dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        n, h, d = case["n"], case["h"], case["d"]
        lead = (case["batch"],) if case.get("batch") else ()
        r = case["rows"] if op == "rows" else n
        s = {k: _normal(gen, lead + (r, n, h, d), dtype=dtype) for k in ("q", "k", "v", "g")}
        s["bias"] = _normal(gen, lead + (n, n, h), case["bias_std"], dtype=dtype)
        s["dout"] = _normal(gen, lead + (r, n, h, d), dtype=dtype)
        s["mask"] = None
        if case["pad"]:
            # padded tokens are never keys: the key is the second pair axis of
            # the starting node and the first one of the ending node
            ok = (torch.arange(n, device="cuda") < n - case["pad"]).to(torch.uint8)
            line = ok[:, None] if case.get("node") == "end" else ok[None, :]
            s["mask"] = line.expand(lead + (r, n)).contiguous()
        return s
    m, c = case["m"], 128
    s = {"x": _normal(gen, (m, c), 1.5, 0.3), "gamma": _normal(gen, (c,), 0.2, 1.0),
         "beta": _normal(gen, (c,), 0.2)}
    if op == "lnl":
        widths = _widths(case)
        s["w"] = _normal(gen, (c, sum(widths)), 1.0 / math.sqrt(c))
        s["douts"] = [_normal(gen, (m, n)) for n in widths] if case["mode"] == "train" else None
    else:
        f = case["f"]
        s["w1"] = _normal(gen, (c, 2 * f), 1.0 / math.sqrt(c))
        s["w2"] = _normal(gen, (f, c), 1.0 / math.sqrt(f))
        s["dout"] = _normal(gen, (m, c)) if case["mode"] == "train" else None
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    if case["mode"] == "autograd":
        for k in ("q", "k", "v", "g", "bias"):
            s[k].requires_grad_(True)
    s["case"] = dict(case)
    return s


# ---- one pass ----------------------------------------------------------------------

def run(state):
    s, case = state, state["case"]
    op, mode = case["op"], case["mode"]
    if op == "attn":
        args = (s["q"], s["k"], s["v"], s["g"], s["bias"])
        node = _node(case)
        if mode == "autograd":
            out = B.triangle_attention(*args, s["mask"], node)
            return (out.detach(), *torch.autograd.grad(out, args, s["dout"]))
        out, lse = B.fwd(*args, s["mask"], node)
        if mode == "infer":
            return out, lse
        return (out, lse, *B.bwd(*args, out, lse, s["dout"], s["mask"], node))
    if op == "rows":
        args = (s["q"], s["k"], s["v"], s["g"], s["bias"])
        out, lse = B.rows_fwd(*args, s["mask"])
        if mode == "infer":
            return out, lse
        return (out, lse, *B.rows_bwd(*args, out, lse, s["dout"], s["mask"]))
    if op == "lnl":
        args = (s["x"], s["gamma"], s["beta"], s["w"])
        outs, mean, rstd = B.ln_linear_fwd(*args, _widths(case), EPS)
        if mode == "infer":
            return (*outs, mean, rstd)
        return (*outs, mean, rstd, *B.ln_linear_bwd(*args, mean, rstd, s["douts"]))
    args = (s["x"], s["gamma"], s["beta"], s["w1"], s["w2"])
    out, mean, rstd = B.transition_fwd(*args, EPS)
    if mode == "infer":
        return out, mean, rstd
    return (out, mean, rstd, *B.transition_bwd(*args, mean, rstd, s["dout"]))


# ---- what a pass cannot do without ---------------------------------------------------

def work(case):
    """Bytes: every input read once, every output written once.  Flops: the
    matrix products of the method (two of them in the attention's forward and
    five in its backward, over the keys that are not masked)."""
    op, train = case["op"], case["mode"] != "infer"
    if op in ("attn", "rows"):
        n, h, d = case["n"], case["h"], case["d"]
        b = case.get("batch") or 1
        r = case["rows"] if op == "rows" else n
        e = 4 if case["dtype"] == "f32" else 2
        wide, narrow = b * r * n * h * d * e, b * n * n * h
        nbytes = 5 * wide + narrow * e + b * r * n * h * 4 + (b * r * n if case["pad"] else 0)
        if train:
            nbytes += 5 * wide + narrow * (4 if op == "rows" else e)
        return {"bytes": nbytes,
                "flops": (14 if train else 4) * b * r * n * (n - case["pad"]) * h * d}
    m, c = case["m"], 128
    if op == "lnl":
        n = sum(_widths(case))
        nbytes = m * c * 2 + m * n * 2 + m * 8 + c * n * 2
        if train:
            nbytes += m * n * 2 + m * c * 2 + c * n * 4
        return {"bytes": nbytes, "flops": (6 if train else 2) * m * c * n}
    f = case["f"]
    nbytes = 2 * m * c * 2 + m * 8 + 3 * c * f * 2
    if train:
        nbytes += 2 * m * c * 2 + 3 * c * f * 4
    return {"bytes": nbytes, "flops": (18 if train else 6) * m * c * f}


# ---- tolerance -----------------------------------------------------------------------

def tolerance(case):
    """About four times the largest error against exact() that was measured
    over the listed and a dozen drawn cases (MI355X): fp32 4.9e-7 and 7.7e-6
    of an output's norm and largest value; bf16 0.0029 and 0.069 in the
    attention, 0.0024 and 0.013 in the projection, 0.0034 and 0.026 in the
    transition, where the rounding of the outputs alone gives 0.0017."""
    if case.get("dtype") == "f32":
        return {"rel": 2e-6, "max": 3e-5}
    return {"attn": {"rel": 0.012, "max": 0.28}, "rows": {"rel": 0.012, "max": 0.28},
            "lnl": {"rel": 0.01, "max": 0.052}, "trn": {"rel": 0.014, "max": 0.11}}[case["op"]]


# ---- the same in 64 bits ---------------------------------------------------------------

def _exact_attn_map(q, k, v, g, bias, dout, valid, scale, train):
    """Starting node over rows: q .. dout [r, n, h, d], bias [n, n, h], valid
    [r, n] or None.  A few rows at a time, fp64."""
    r, n, h, d = q.shape
    f8 = torch.float64

    def head_major(t):
        return t.to(f8).permute(0, 2, 1, 3).contiguous()

    bh = bias.to(f8).permute(2, 0, 1).contiguous()
    out, lse = torch.empty((r, n, h, d), dtype=f8, device=q.device), \
        torch.empty((r, n, h), dtype=f8, device=q.device)
    grads = [torch.empty_like(out) for _ in range(4)] if train else []
    dbias = torch.zeros_like(bh)
    step = max(1, int(2e8 // (n * n * h)))
    for a in range(0, r, step):
        sl = slice(a, min(r, a + step))
        qh, kh, vh, gh = (head_major(t[sl]) for t in (q, k, v, g))
        s = torch.matmul(qh, kh.transpose(2, 3).contiguous()).mul_(scale).add_(bh)
        if valid is not None:
            s.masked_fill_(~valid[sl][:, None, None, :], -math.inf)
        ls = torch.logsumexp(s, dim=3)
        p = s.sub_(ls[..., None]).exp_()
        att, sg = torch.matmul(p, vh), torch.sigmoid(gh)
        out[sl] = (att * sg).permute(0, 2, 1, 3)
        lse[sl] = ls.permute(0, 2, 1)
        if not train:
            continue
        doh = head_major(dout[sl])
        da = doh * sg
        dg = doh * att * sg * (1.0 - sg)
        dv = torch.matmul(p.transpose(2, 3).contiguous(), da)
        ds = torch.matmul(da, vh.transpose(2, 3).contiguous())
        ds.sub_((da * att).sum(dim=3, keepdim=True)).mul_(p)
        dbias += ds.sum(dim=0)
        dq = torch.matmul(ds, kh) * scale
        dk = torch.matmul(ds.transpose(2, 3).contiguous(), qh) * scale
        for dst, src in zip(grads, (dq, dk, dv, dg)):
            dst[sl] = src.permute(0, 2, 1, 3)
    return [out, lse, *grads] + ([dbias.permute(1, 2, 0).contiguous()] if train else [])


def _exact_attn(case, s):
    train, scale = case["mode"] != "infer", 1.0 / math.sqrt(case["d"])
    end, batch = case.get("node") == "end", case.get("batch") or 0

    def swap(t):
        return t.transpose(0, 1).contiguous() if end and t is not None else t

    maps = []
    for b in range(max(batch, 1)):
        t = {k: s[k] if s[k] is None or not batch else s[k][b]
             for k in ("q", "k", "v", "g", "bias", "dout", "mask")}
        valid = None if t["mask"] is None else swap(t["mask"]).bool()
        got = _exact_attn_map(*(swap(t[k]) for k in ("q", "k", "v", "g", "bias", "dout")),
                              valid, scale, train)
        maps.append([swap(x) for x in got])
    res = [torch.stack(x) for x in zip(*maps)] if batch else maps[0]
    if case["mode"] == "autograd":
        del res[1]  # the autograd call gives no log-sum-exp
    return tuple(res)


def _norm_rows(x):
    mean = x.mean(dim=1)
    rstd = 1.0 / torch.sqrt(((x - mean[:, None]) ** 2).mean(dim=1) + EPS)
    return mean, rstd, (x - mean[:, None]) * rstd[:, None]


def _norm_grad(do1, gamma, xhat, rstd):
    wdy = do1 * gamma
    c1, c2 = (wdy * xhat).mean(dim=1, keepdim=True), wdy.mean(dim=1, keepdim=True)
    return (wdy - c1 * xhat - c2) * rstd[:, None]


def _blocks(m, step=65536):
    return [slice(a, min(m, a + step)) for a in range(0, m, step)]


def _exact_lnl(case, s):
    f8, train, widths = torch.float64, case["mode"] == "train", _widths(case)
    gamma, beta, w = (s[k].to(f8) for k in ("gamma", "beta", "w"))
    wt = w.t().contiguous()
    rows, dw = [], torch.zeros_like(w)
    dgamma, dbeta = torch.zeros_like(gamma), torch.zeros_like(beta)
    for sl in _blocks(case["m"]):
        mean, rstd, xhat = _norm_rows(s["x"][sl].to(f8))
        o1 = xhat * gamma + beta
        got = [*torch.split(torch.matmul(o1, w), widths, dim=1), mean, rstd]
        if train:
            do2 = torch.cat([t[sl].to(f8) for t in s["douts"]], dim=1)
            do1 = torch.matmul(do2, wt)
            dw += torch.matmul(o1.t().contiguous(), do2)
            dgamma += (do1 * xhat).sum(dim=0)
            dbeta += do1.sum(dim=0)
            got.append(_norm_grad(do1, gamma, xhat, rstd))
        rows.append(got)
    res = [torch.cat(t) for t in zip(*rows)]
    return tuple(res + [dw, dgamma, dbeta]) if train else tuple(res)


def _exact_trn(case, s):
    f8, train, f = torch.float64, case["mode"] == "train", case["f"]
    gamma, beta, w1, w2 = (s[k].to(f8) for k in ("gamma", "beta", "w1", "w2"))
    w1t, w2t = w1.t().contiguous(), w2.t().contiguous()
    rows, dw1, dw2 = [], torch.zeros_like(w1), torch.zeros_like(w2)
    dgamma, dbeta = torch.zeros_like(gamma), torch.zeros_like(beta)
    for sl in _blocks(case["m"]):
        mean, rstd, xhat = _norm_rows(s["x"][sl].to(f8))
        o1 = xhat * gamma + beta
        hidden = torch.matmul(o1, w1)
        a, b = hidden[:, :f], hidden[:, f:]
        sg = torch.sigmoid(a)
        u = a * sg * b
        got = [torch.matmul(u, w2), mean, rstd]
        if train:
            dout = s["dout"][sl].to(f8)
            du = torch.matmul(dout, w2t)
            dh = torch.cat([du * b * sg * (1.0 + a * (1.0 - sg)), du * a * sg], dim=1)
            dw2 += torch.matmul(u.t().contiguous(), dout)
            dw1 += torch.matmul(o1.t().contiguous(), dh)
            do1 = torch.matmul(dh, w1t)
            dgamma += (do1 * xhat).sum(dim=0)
            dbeta += do1.sum(dim=0)
            got.append(_norm_grad(do1, gamma, xhat, rstd))
        rows.append(got)
    res = [torch.cat(t) for t in zip(*rows)]
    return tuple(res + [dw1, dw2, dgamma, dbeta]) if train else tuple(res)


def exact(case, seed):
    s = _inputs(case, seed)
    if case["op"] in ("attn", "rows"):
        return _exact_attn(case, s)
    return _exact_lnl(case, s) if case["op"] == "lnl" else _exact_trn(case, s)
