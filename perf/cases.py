"""The work an AlphaFold training or inference program has this library do, as
cases to be timed: whole passes through the Python entry points, on buffers
the program allocates once, the way bench.py and graph.MSARowAttentionStep
call them.

A case's "kind" names the pass:
  attn       evo_attn_fwd and, unless "train" is False, evo_attn_bwd
  ln         layernorm_fwd + layernorm_bwd
  proj       ln_proj_fwd (saving what its backward reads) + ln_proj_bwd: the
             four q/k/v/gate projections of an attention's input
  linear     linear_fwd + linear_bwd: an attention's output projection
  pair_bias  ln_pair_bias_fwd + ln_pair_bias_bwd
  optim      gradient clipping + Adam + SWA over a model's tensors
  module     one whole MSA-row attention module step, replayed from the graph cache
"""
from __future__ import annotations

import math

import torch

from paper_2404_11068_amd import evo_attn as ea
from paper_2404_11068_amd import graph as gr
from paper_2404_11068_amd import layernorm as ln
from paper_2404_11068_amd import optim as op
from paper_2404_11068_amd import proj as pj
from paper_2404_11068_amd import workloads as W

_DT = {"bf16": torch.bfloat16, "f32": torch.float32}
_EPS = 1e-5


def _attn(rows, keys, heads, dim, dtype="bf16", bias=True, mask="length", planes=1, train=True, ending=False):
    return {"kind": "attn", "rows": rows, "keys": keys, "heads": heads, "dim": dim, "dtype": dtype, "bias": bias,
            "mask": mask, "planes": planes, "train": train, "ending": ending}


def listed():
    return [
        # triangle attention around the starting node, one training step at the 256-residue crop
        dict(_attn(256, 256, 4, 32), name="attn_tri_train"),
        # triangle attention around the ending node (strided views) at the 384-residue fine-tuning crop
        dict(_attn(384, 384, 4, 32, ending=True), name="attn_tri_end_384_train"),
        # MSA row attention with pair bias, one GPU's share when the rows are split over 8
        dict(_attn(16, 256, 8, 32), name="attn_msa_row_share8_train"),
        # MSA column attention: no pair bias, short rows, a padded tail
        dict(_attn(256, 128, 8, 32, bias=False, mask="pad"), name="attn_msa_col_train"),
        # the extra-MSA stack's row attention: the largest attention of a training step
        dict(_attn(1024, 256, 8, 8, mask="drop"), name="attn_extra_msa_train"),
        # inference on one protein of an odd number of residues: forward only, nothing padded
        dict(_attn(317, 317, 4, 32, mask="none", train=False), name="attn_tri_infer_317"),
        # a small fp32 step, as in a debugging or validation run: launches and host time count
        dict(_attn(32, 32, 4, 32, dtype="f32", mask="drop"), name="attn_tri_f32_small"),
        # the pair representation's LayerNorm, one of many per block
        {"kind": "ln", "rows": 65536, "cols": 128, "dtype": "bf16", "name": "ln_pair_train"},
        # MSA attention input: LayerNorm + q/k/v/gate
        {"kind": "proj", "rows": 32768, "c_in": 256, "proj_dim": 256, "name": "proj_msa_train"},
        # pair bias of the triangle attention around the ending node (transposed layout)
        {"kind": "pair_bias", "len": 256, "c_in": 128, "heads": 4, "transpose": True, "name": "pair_bias_tri_end_train"},
        # the optimizer step of the whole model: about 5000 tensors, 94M parameters
        {"kind": "optim", "every": 1, "name": "adam_swa_alphafold"},
        # one MSA-row attention module, forward and backward, at one GPU's share of 8, replayed as a graph
        {"kind": "module", "rows": 16, "len": 256, "name": "module_msa_row_share8"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attn", "attn", "attn", "attn", "attn", "ln", "proj", "proj", "linear", "pair_bias", "optim",
                       "module"])
    if kind == "attn":
        dtype = "f32" if rng.random() < 0.15 else "bf16"
        dim = rng.choice([8, 16, 32, 32])
        heads = rng.choice([4, 8])
        keys = _log(rng, 17, 256 if dtype == "f32" else 512)
        if rng.random() < 0.5:
            keys = max(16, keys // 8 * 8)
        rows = _log(rng, 4, 1024)
        most = (1 << 25) if dtype == "f32" else (1 << 28) if dim == 8 else (1 << 27)  # logits in all
        rows = max(1, min(rows, most // (heads * keys * keys)))
        planes = 2 if rng.random() < 0.2 else 1
        rows = max(rows // planes, 1) * planes
        return _attn(rows, keys, heads, dim, dtype, bias=rng.random() < 0.75,
                     mask=rng.choice(["none", "length", "drop", "pad"]), planes=planes, train=rng.random() < 0.75,
                     ending=rng.random() < 0.25)
    if kind == "ln":
        cols = rng.choice([64, 128, 256, 512, 1024])
        return {"kind": "ln", "rows": _log(rng, 64, (1 << 24) // cols), "cols": cols,
                "dtype": rng.choice(["bf16", "bf16", "f32"])}
    if kind in ("proj", "linear"):
        c_in = rng.choice([64, 128, 256])
        return {"kind": kind, "rows": _log(rng, 256, (1 << 24) // c_in), "c_in": c_in, "proj_dim": c_in}
    if kind == "pair_bias":
        return {"kind": "pair_bias", "len": 8 * rng.randint(8, 48), "c_in": rng.choice([64, 128]),
                "heads": rng.choice([4, 8]), "transpose": rng.random() < 0.5}
    if kind == "optim":
        return {"kind": "optim", "every": _log(rng, 2, 40)}
    return {"kind": "module", "rows": _log(rng, 4, 128), "len": 8 * rng.randint(8, 32)}


# ---------------------------------------------------------------------------
# inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, *shape, dtype=torch.float32, scale=1.0, shift=0.0):
    return (torch.randn(*shape, generator=g, device="cuda") * scale + shift).to(dtype)


def _residual(g, rows, cols, dtype):
    """Rows of a residual stream: each with an offset and a spread of its own."""
    off = torch.randn(rows, 1, generator=g, device="cuda") * 2
    spread = torch.rand(rows, 1, generator=g, device="cuda") * 3.75 + 0.25
    return (torch.randn(rows, cols, generator=g, device="cuda") * spread + off).to(dtype)


def _keep(case, g):
    N, L, mask = case["rows"], case["keys"], case["mask"]
    if mask == "none":
        return None
    u = torch.rand(N, L, generator=g, device="cuda")
    j = torch.arange(L, device="cuda")
    if mask == "drop":  # single residues missing; one key of each row is always there
        keep = (u >= 0.05) | (j == 0)
    else:  # a padded tail, at most an eighth of the row ("length") or a sixteenth ("pad")
        cut = L // 8 if mask == "length" else L // 16
        n = L - int(torch.randint(0, cut + 1, (1,), generator=g, device="cuda").item())
        keep = (j < n).expand(N, L)
    return keep.to(torch.uint8).contiguous()


def _prepare_attn(case, seed):
    g, dt = _gen(seed), _DT[case["dtype"]]
    N, L, H, d = case["rows"], case["keys"], case["heads"], case["dim"]

    def tok(scale=1.0, empty=False):
        shape = (L, N, H, d) if case["ending"] else (N, L, H, d)
        t = torch.empty(shape, dtype=dt, device="cuda") if empty else _normal(g, *shape, dtype=dt, scale=scale)
        return t.transpose(0, 1) if case["ending"] else t

    scale = 1.0 if case["bias"] else d ** -0.5
    s = {"q": tok(scale), "k": tok(scale), "v": tok(scale), "gate": tok(), "out": tok(empty=True),
         "lse": torch.empty(N, H, L, device="cuda"), "rpb": N // case["planes"], "train": case["train"]}
    s["bias"] = _normal(g, case["planes"], H, L, L, dtype=dt) if case["bias"] else None
    s["mask"] = _keep(case, g)
    if case["train"]:
        s["dout"] = tok()
        s["grads"] = {n: tok(empty=True) for n in ("dq", "dk", "dv", "dgate")}
        if case["bias"]:
            s["grads"]["dbias"] = torch.empty(case["planes"], H, L, L, device="cuda")
        n = ea.evo_attn_bwd_workspace_size(s["q"], s["rpb"])
        s["grads"]["workspace"] = torch.empty(max(n, 1), dtype=torch.uint8, device="cuda")
    return s


def _run_attn(s):
    args = (s["q"], s["k"], s["v"], s["gate"], s["bias"], s["mask"])
    out, lse = ea.evo_attn_fwd(*args, rows_per_bias=s["rpb"], out=s["out"], lse=s["lse"])
    if not s["train"]:
        return out, lse
    return (out, lse) + tuple(ea.evo_attn_bwd(*args, out, lse, s["dout"], rows_per_bias=s["rpb"], **s["grads"]))


def _prepare_ln(case, seed):
    g, dt = _gen(seed), _DT[case["dtype"]]
    R, C = case["rows"], case["cols"]
    x = _residual(g, R, C, dt)
    s = {"x": x, "w": _normal(g, C, scale=0.2, shift=1.0), "b": _normal(g, C, scale=0.2),
         "dy": _normal(g, R, C, dtype=dt)}
    s["fwd"] = {"y": torch.empty_like(x), "mean": torch.empty(R, device="cuda"), "rstd": torch.empty(R, device="cuda")}
    s["bwd"] = {"dx": torch.empty_like(x), "dweight": torch.empty(C, device="cuda"),
                "dbias": torch.empty(C, device="cuda"),
                "workspace": torch.empty(max(ln.workspace_size(x, _EPS), 1), dtype=torch.uint8, device="cuda")}
    return s


def _run_ln(s):
    y, mean, rstd = ln.layernorm_fwd(s["x"], s["w"], s["b"], _EPS, **s["fwd"])
    return (y, mean, rstd) + tuple(ln.layernorm_bwd(s["x"], s["w"], mean, rstd, s["dy"], eps=_EPS, **s["bwd"]))


def _prepare_proj(case, seed):
    g, bf = _gen(seed), torch.bfloat16
    R, C, HD, P = case["rows"], case["c_in"], case["proj_dim"], 4 if case["kind"] == "proj" else 1
    s = {"norm": P == 4, "x": _residual(g, R, C, bf) if P == 4 else _normal(g, R, C, dtype=bf, scale=0.5),
         "w": _normal(g, P * HD, C, dtype=bf, scale=C ** -0.5), "b": _normal(g, P * HD, scale=0.1), "P": P,
         "lnw": _normal(g, C, scale=0.2, shift=1.0), "lnb": _normal(g, C, scale=0.2),
         "douts": [_normal(g, R, HD, dtype=bf) for _ in range(P)],
         "outs": [torch.empty(R, HD, dtype=bf, device="cuda") for _ in range(P)],
         "mean": torch.empty(R, device="cuda"), "rstd": torch.empty(R, device="cuda"),
         "y": torch.empty(R, C, dtype=bf, device="cuda")}
    f32 = lambda *n: torch.empty(*n, device="cuda")
    s["bwd"] = {"dx": torch.empty(R, C, dtype=bf, device="cuda"), "dweight": f32(P * HD, C), "dbias": f32(P * HD)}
    dims = pj.evo_proj_dims(ea.EVO_DTYPE_BF16, C, P, HD, R, _EPS if P == 4 else 0.0, 0)
    size = pj._lib().evo_ln_proj_bwd_workspace_size if P == 4 else pj._lib().evo_linear_bwd_workspace_size
    s["bwd"]["workspace"] = torch.empty(max(int(size(dims)), 1), dtype=torch.uint8, device="cuda")
    if P == 4:
        s["bwd"].update(dln_weight=f32(C), dln_bias=f32(C))
    return s


def _run_proj(s):
    if not s["norm"]:
        outs = pj.linear_fwd(s["x"], s["w"], s["b"], n_proj=1, outs=s["outs"])
        return list(outs) + list(pj.linear_bwd(s["x"], s["w"], s["douts"], **s["bwd"]))
    outs, mean, rstd = pj.ln_proj_fwd(s["x"], s["lnw"], s["lnb"], s["w"], s["b"], n_proj=4, eps=_EPS, outs=s["outs"],
                                      mean=s["mean"], rstd=s["rstd"], y_norm=s["y"])
    return list(outs) + [mean, rstd, s["y"]] + list(
        pj.ln_proj_bwd(s["x"], s["lnw"], mean, rstd, s["y"], s["w"], s["douts"], eps=_EPS, **s["bwd"]))


def _prepare_pair_bias(case, seed):
    g, bf = _gen(seed), torch.bfloat16
    L, C, H, tr = case["len"], case["c_in"], case["heads"], case["transpose"]
    z = _residual(g, L * L, C, bf).view(1, L, L, C)
    s = {"z": z, "lnw": _normal(g, C, scale=0.2, shift=1.0), "lnb": _normal(g, C, scale=0.2), "tr": tr,
         "w": _normal(g, H, C, dtype=bf, scale=C ** -0.5), "dbias": _normal(g, 1, H, L, L),
         "out": torch.empty(1, H, L, L, dtype=bf, device="cuda")}
    n = pj.pair_bias_bwd_workspace_size(1, L, L, C, H, tr, _EPS)
    s["bwd"] = {"dz": torch.empty_like(z), "dweight": torch.empty(H, C, device="cuda"),
                "dln_weight": torch.empty(C, device="cuda"), "dln_bias": torch.empty(C, device="cuda"),
                "workspace": torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")}
    return s


def _run_pair_bias(s):
    out = pj.ln_pair_bias_fwd(s["z"], s["lnw"], s["lnb"], s["w"], _EPS, s["tr"], out=s["out"])
    return (out,) + tuple(pj.ln_pair_bias_bwd(s["z"], s["lnw"], s["lnb"], s["w"], s["dbias"], _EPS, s["tr"], **s["bwd"]))


def _optim_shapes(case):
    return W.alphafold_param_shapes()[::case["every"]]


def _prepare_optim(case, seed):
    """Every tensor a view of one flat buffer of its kind, its start 512-byte aligned as a program's own tensors are."""
    g = _gen(seed)
    sizes = [math.prod(s) for s in _optim_shapes(case)]
    starts, n = [], 0
    for k in sizes:
        starts.append(n)
        n += -(-k // 128) * 128
    used = torch.zeros(n, device="cuda")
    for a, k in zip(starts, sizes):
        used[a:a + k] = 1.0
    flat = {"params": _normal(g, n, scale=0.02) * used, "grads": _normal(g, n, scale=1e-3) * used,
            "exp_avg": _normal(g, n, scale=1e-4) * used, "exp_avg_sq": _normal(g, n, scale=1e-6).abs_() * used}
    flat["swa"] = flat["params"] + _normal(g, n, scale=1e-4) * used
    lists = {k: [v[a:a + m] for a, m in zip(starts, sizes)] for k, v in flat.items()}
    o = op.FusedAdamSWA(lists["params"], lists["grads"], lists["exp_avg"], lists["exp_avg_sq"], lists["swa"])
    o.step_count = 9
    return {"opt": o, "flat": flat}


def _run_optim(s):
    s["opt"].step(max_norm=0.1)
    f = s["flat"]
    return {"params": f["params"], "exp_avg": f["exp_avg"], "exp_avg_sq": f["exp_avg_sq"], "swa": f["swa"],
            "norm": s["opt"].norm}


# the module's results: its output and every gradient but the pair LayerNorm's bias gradient,
# which is zero in exact arithmetic (every row of the logits' gradient sums to zero)
_MODULE_OUTS = ("m_out", "dm", "dw_qkvg", "db_qkvg", "dln_m_w", "dln_m_b", "dz", "dw_bias", "dln_z_w", "dw_out", "db_out")


def _prepare_module(case, seed):
    step = gr.MSARowAttentionStep(case["rows"], case["len"], seed=int(seed))
    return {"step": step, "cache": gr.GraphCache(4), "stream": torch.cuda.Stream()}


def _run_module(s):
    step, stream = s["step"], s["stream"]
    stream.wait_stream(torch.cuda.current_stream())
    s["cache"].run(step.key(), step.record, stream)
    torch.cuda.current_stream().wait_stream(stream)
    return {n: getattr(step, n) for n in _MODULE_OUTS}


_PREPARE = {"attn": _prepare_attn, "ln": _prepare_ln, "proj": _prepare_proj, "linear": _prepare_proj,
            "pair_bias": _prepare_pair_bias, "optim": _prepare_optim, "module": _prepare_module}
_RUN = {"attn": _run_attn, "ln": _run_ln, "proj": _run_proj, "linear": _run_proj, "pair_bias": _run_pair_bias,
        "optim": _run_optim, "module": _run_module}


def prepare(case, seed):
    s = _PREPARE[case["kind"]](case, seed)
    s["run"] = _RUN[case["kind"]]
    return s


def run(state):
    return state["run"](state)


# ---------------------------------------------------------------------------
# what a pass cannot do without

def work(case):
    k = case["kind"]
    if k == "attn":
        N, L, H, d, B = case["rows"], case["keys"], case["heads"], case["dim"], case["planes"]
        es = 2 if case["dtype"] == "bf16" else 4
        tok, plane = N * L * H * d, B * H * L * L if case["bias"] else 0
        mask = N * L if case["mask"] != "none" else 0
        # q, k, v, gate, bias and mask in, out and lse out; then dout in, dq, dk, dv, dgate and dbias out
        by = 5 * tok * es + plane * es + mask + 4 * N * H * L
        if case["train"]:
            by += 5 * tok * es + 4 * plane
        return {"bytes": by, "flops": (14 if case["train"] else 4) * N * H * L * L * d}
    if k == "ln":
        n, es = case["rows"] * case["cols"], 2 if case["dtype"] == "bf16" else 4
        return {"bytes": 4 * n * es + 8 * case["rows"] + 16 * case["cols"], "flops": 16 * n}
    if k in ("proj", "linear"):
        R, C, HD, P = case["rows"], case["c_in"], case["proj_dim"], 4 if k == "proj" else 1
        F = P * HD
        # x, weight, douts in, outs, dx, dweight, dbias out; the normalised input and the statistics out
        by = 4 * R * C + 4 * R * F + 2 * F * C + 4 * F * C + 8 * F + ((2 * R * C + 8 * R + 16 * C) if P == 4 else 0)
        return {"bytes": by, "flops": 6 * R * C * F}
    if k == "pair_bias":
        L, C, H = case["len"], case["c_in"], case["heads"]
        return {"bytes": 4 * L * L * C + 6 * H * L * L + 6 * H * C + 16 * C, "flops": 6 * L * L * C * H}
    if k == "optim":
        n = sum(math.prod(s) for s in _optim_shapes(case))
        return {"bytes": 36 * n, "flops": 20 * n}
    N, L, c_m, c_z, H, d = case["rows"], case["len"], 256, 128, 8, 32
    # m, z and the upstream gradient in, the output, dm and dz out; the weights in, their gradients out
    weights = 4 * H * d * c_m + c_m * H * d + H * c_z
    by = 2 * (N * L * c_m * 4 + L * L * c_z * 2) + 6 * weights
    fl = 14 * N * H * L * L * d + 6 * N * L * c_m * 5 * H * d + 6 * L * L * c_z * H
    return {"bytes": by, "flops": fl}


def tolerance(case):
    k = case["kind"]
    if k == "attn":
        return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-5}
    if k == "ln":
        return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-5}
    if k in ("proj", "linear", "pair_bias"):
        return {"rel": 1e-2}
    if k == "optim":
        return {"rel": 1e-5}
    return {"rel": 2.5e-2}


# ---------------------------------------------------------------------------
# the same results in 64 bits

def _ln64(x, w, b, eps=_EPS):
    mean = x.mean(-1, keepdim=True)
    xc = x - mean
    rstd = (xc.square().mean(-1, keepdim=True) + eps).rsqrt()
    xhat = xc * rstd
    return xhat * w + b, mean.squeeze(-1), rstd.squeeze(-1), xhat


def _ln64_bwd(dy, w, xhat, rstd):
    """dx, dweight, dbias; rstd without its last axis."""
    gx = dy * w
    dx = rstd.unsqueeze(-1) * (gx - gx.mean(-1, keepdim=True) - xhat * (gx * xhat).mean(-1, keepdim=True))
    return dx, (dy * xhat).flatten(0, -2).sum(0), dy.flatten(0, -2).sum(0)


def _attn64(q, k, v, gate, bias, mask, dout, rpb):
    """(out, lse) and, with dout, (dq, dk, dv, dgate, dbias): rows in chunks, so that a chunk's logits stay small."""
    N, L, H, d = q.shape
    sc = d ** -0.5
    o = torch.empty(N, L, H, d, dtype=torch.float64, device=q.device)
    ls = torch.empty(N, H, L, dtype=torch.float64, device=q.device)
    gr_ = [torch.empty_like(o) for _ in range(4)] if dout is not None else None
    db = torch.zeros(bias.shape, dtype=torch.float64, device=q.device) if bias is not None else None
    step = max(1, (1 << 26) // (H * L * L))
    for plane in range(N // rpb):
        for a in range(plane * rpb, (plane + 1) * rpb, step):
            r = slice(a, min(a + step, (plane + 1) * rpb))
            Q, K, V, G = (t[r].double().transpose(1, 2).contiguous() for t in (q, k, v, gate))
            S = torch.matmul(Q, K.transpose(2, 3).contiguous()) * sc
            if bias is not None:
                S += bias[plane].double()
            if mask is not None:
                S.masked_fill_(mask[r, None, None, :] == 0, -math.inf)
            lse = torch.logsumexp(S, -1)
            P = torch.exp(S - lse.unsqueeze(-1))
            A, sg = torch.matmul(P, V), torch.sigmoid(G)
            o[r], ls[r] = (A * sg).transpose(1, 2), lse
            if dout is None:
                continue
            D = dout[r].double().transpose(1, 2).contiguous()
            dA = D * sg
            dP = torch.matmul(dA, V.transpose(2, 3).contiguous())
            dS = P * (dP - (P * dP).sum(-1, keepdim=True))
            gr_[0][r] = torch.matmul(dS, K).transpose(1, 2) * sc
            gr_[1][r] = torch.matmul(dS.transpose(2, 3).contiguous(), Q).transpose(1, 2) * sc
            gr_[2][r] = torch.matmul(P.transpose(2, 3).contiguous(), dA).transpose(1, 2)
            gr_[3][r] = (D * A * sg * (1 - sg)).transpose(1, 2)
            if db is not None:
                db[plane] += dS.sum(0)
    return (o, ls) if dout is None else (o, ls, *gr_, db)


def exact(case, seed):
    k = case["kind"]
    s = prepare(case, seed)
    if k == "attn":
        return _attn64(s["q"], s["k"], s["v"], s["gate"], s["bias"], s["mask"], s.get("dout"), s["rpb"])
    if k == "ln":
        y, mean, rstd, xhat = _ln64(s["x"].double(), s["w"].double(), s["b"].double())
        return (y, mean, rstd) + _ln64_bwd(s["dy"].double(), s["w"].double(), xhat, rstd)
    if k in ("proj", "linear"):
        x, w, b, P = s["x"].double(), s["w"].double(), s["b"].double(), s["P"]
        y, mean, rstd, xhat = _ln64(x, s["lnw"].double(), s["lnb"].double()) if P == 4 else (x, None, None, None)
        outs = list((y @ w.t() + b).chunk(P, -1))
        d = torch.cat([t.double() for t in s["douts"]], -1)
        dy, dw, db = d @ w, d.t() @ y, d.sum(0)
        if P == 1:
            return outs + [dy, dw, db]
        dx, dlw, dlb = _ln64_bwd(dy, s["lnw"].double(), xhat, rstd)
        return outs + [mean, rstd, y, dx, dw, db, dlw, dlb]
    if k == "pair_bias":
        y, _, rstd, xhat = _ln64(s["z"].double(), s["lnw"].double(), s["lnb"].double())
        w, g = s["w"].double(), s["dbias"].double()
        out = (y @ w.t()).permute(0, 3, 2, 1) if s["tr"] else (y @ w.t()).permute(0, 3, 1, 2)
        ge = (g.permute(0, 3, 2, 1) if s["tr"] else g.permute(0, 2, 3, 1)).contiguous()
        dx, dlw, dlb = _ln64_bwd(ge @ w, s["lnw"].double(), xhat, rstd)
        return out, dx, ge.flatten(0, 2).t() @ y.flatten(0, 2), dlw, dlb
    if k == "optim":
        f = {n: t.double() for n, t in s["flat"].items()}
        o, t = s["opt"], s["opt"].step_count + 1
        norm = f["grads"].square().sum().sqrt()
        g = f["grads"] * torch.clamp(0.1 / (norm + 1e-6), max=1.0)
        b1, b2 = o.betas
        m = b1 * f["exp_avg"] + (1 - b1) * g
        v = b2 * f["exp_avg_sq"] + (1 - b2) * g.square()
        p = f["params"] - o.lr / (1 - b1 ** t) * m / ((v / (1 - b2 ** t)).sqrt() + o.eps)
        return {"params": p, "exp_avg": m, "exp_avg_sq": v,
                "swa": o.swa_decay * f["swa"] + (1 - o.swa_decay) * p, "norm": norm.reshape(1)}
    st = s["step"]
    N, L, H, d = st.N, st.L, st.H, st.d
    y, _, rstd, xhat = _ln64(st.m.double(), st.ln_m_w.double(), st.ln_m_b.double())
    wq, wo, wb = st.w_qkvg.double(), st.w_out.double(), st.w_bias.double()
    q, kk, v, gt = (t.reshape(N, L, H, d) for t in (y @ wq.t() + st.b_qkvg.double()).chunk(4, -1))
    yz, _, rz, zhat = _ln64(st.z.double(), st.ln_z_w.double(), st.ln_z_b.double())
    bias = (yz @ wb.t()).permute(0, 3, 1, 2).contiguous()
    dm_out = st.d_m_out.double()
    dout = (dm_out @ wo).reshape(N, L, H, d)
    o, _, dq, dk, dv, dg, db = _attn64(q, kk, v, gt, bias, st.mask, dout, N)
    of = o.reshape(N * L, H * d)
    df = torch.cat([t.reshape(N, L, H * d) for t in (dq, dk, dv, dg)], -1)
    dm, dlw, dlb = _ln64_bwd(df @ wq, st.ln_m_w.double(), xhat, rstd)
    ge = db.permute(0, 2, 3, 1).contiguous()
    dz, dlzw, _ = _ln64_bwd(ge @ wb, st.ln_z_w.double(), zhat, rz)
    return {"m_out": (of @ wo.t() + st.b_out.double()).reshape(N, L, -1), "dm": dm,
            "dw_qkvg": df.flatten(0, 1).t() @ y.flatten(0, 1), "db_qkvg": df.flatten(0, 1).sum(0),
            "dln_m_w": dlw, "dln_m_b": dlb, "dz": dz, "dw_bias": ge.flatten(0, 2).t() @ yz.flatten(0, 2),
            "dln_z_w": dlzw, "dw_out": dm_out.flatten(0, 1).t() @ of, "db_out": dm_out.flatten(0, 1).sum(0)}
