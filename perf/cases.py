"""The workloads this library's performance is measured on.

Each case is one call sequence that a training or serving program makes through the public
binding, with the buffers such a program keeps (outputs and workspaces are allocated once,
as the library never allocates):

  step       laga_reconstruct_kv + laga_attn_fwd + laga_attn_bwd (with K/V rebuilt on chip:
             laga_attn_fwd + laga_attn_bwd alone), one training step of the attention block
  forward    laga_reconstruct_kv + laga_attn_fwd (prefill / evaluation)
  producers  laga_prologue_fwd + laga_prologue_bwd, the per-token steps around the gather
  out_proj   laga_out_proj_fwd + laga_out_proj_bwd, the output projection

over the head widths, element types and modes that the library has. ``listed`` names the
cases, ``draw`` gives others of the same ranges; ``exact`` is the same mathematics in plain
float64 torch.
"""
from __future__ import annotations

import math

import torch

import paper_2607_17644_amd as laga

# (d_nope, d_rope, d_v) by name
WIDTHS = {"v3": (128, 64, 128), "half": (64, 32, 64), "small": (32, 16, 32)}

_STEP = dict(kind="step", batch=1, heads=16, d_c=512, widths="v3", dtype="bf16", causal=True, fused=False,
             recompute=False, noalloc=False)


def listed():
    return [
        # the training step at the rank's share (16 of 128 heads), longest and shortest of the sweep
        dict(_STEP, name="train_s16384", seq=16384),
        dict(_STEP, name="train_s2048", seq=2048),
        # a batch of ragged sequences
        dict(_STEP, name="train_b2_s5001", batch=2, seq=5001),
        # the backward without an S x S buffer
        dict(_STEP, name="recompute_s8192", seq=8192, recompute=True),
        # K/V rebuilt on chip from the latent
        dict(_STEP, name="fused_s4096", seq=4096, fused=True),
        # a short step for callers that cannot allocate
        dict(_STEP, name="noalloc_s1000", seq=1000, noalloc=True),
        # half-width heads, a batch of short sequences
        dict(_STEP, name="half_b4_s2000", batch=4, seq=2000, d_c=256, widths="half"),
        # the fp32 mode: the small widths (smallest call) and the full ones
        dict(_STEP, name="fp32_small_s256", seq=256, heads=4, d_c=64, widths="small", dtype="fp32"),
        dict(_STEP, name="fp32_s2048", seq=2048, dtype="fp32"),
        # every head on one device, forward only
        dict(kind="forward", name="forward_h128_s4096", batch=1, seq=4096, heads=128, d_c=512, widths="v3",
             dtype="bf16", causal=True, fused=False),
        dict(kind="producers", name="producers_s16384", batch=1, seq=16384, heads=16, d_c=512, widths="v3",
             dtype="bf16", gamma=True, offset=0),
        # W_o on one rank's tokens with every head
        dict(kind="out_proj", name="out_proj_t2048", tokens=2048, heads=128, d_v=128, d_model=7168, dtype="bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _pairs(case):
    s = case["seq"]
    return case["batch"] * case["heads"] * (s * (s + 1) // 2 if case["causal"] else s * s)


def draw(rng):
    kind = rng.choice(["train", "train", "train", "recompute", "fused", "noalloc", "half", "fp32", "forward",
                       "producers", "out_proj"])
    if kind == "producers":
        return dict(kind=kind, batch=rng.choice([1, 1, 2]), seq=_log_int(rng, 64, 16384), heads=rng.choice([8, 16, 16]),
                    d_c=rng.choice([256, 512, 512]), widths=rng.choice(["v3", "v3", "half"]),
                    dtype=rng.choice(["bf16", "bf16", "fp32"]), gamma=rng.random() < 0.75,
                    offset=rng.choice([0, 2048, 14336]))
    if kind == "out_proj":
        c = dict(kind=kind, tokens=_log_int(rng, 64, 2048), heads=rng.choice([16, 32, 64, 128]), d_v=128,
                 d_model=16 * _log_int(rng, 64, 448), dtype=rng.choice(["bf16", "bf16", "bf16", "fp32"]))
        if c["dtype"] == "fp32":
            c["heads"] = 16
        return c
    if kind == "forward":
        c = dict(kind=kind, batch=rng.choice([1, 2]), seq=_log_int(rng, 64, 8192), heads=rng.choice([16, 32, 64, 128]),
                 d_c=512, widths=rng.choice(["v3", "v3", "half"]), dtype="bf16", causal=rng.random() < 0.8,
                 fused=rng.random() < 0.3)
    else:
        c = dict(_STEP, batch=rng.choice([1, 1, 2]), heads=rng.choice([8, 16, 16, 32]), causal=rng.random() < 0.85)
        if kind == "train":
            c.update(seq=_log_int(rng, 64, 16384))
        elif kind == "recompute":
            c.update(seq=_log_int(rng, 512, 16384), recompute=True)
        elif kind == "fused":
            c.update(seq=_log_int(rng, 128, 8192), fused=True, d_c=rng.choice([256, 512, 512]))
        elif kind == "noalloc":
            c.update(seq=_log_int(rng, 32, 1024), batch=1, heads=rng.choice([8, 16]), causal=True, noalloc=True)
        elif kind == "half":
            c.update(seq=_log_int(rng, 64, 4096), batch=rng.choice([1, 2, 4]), widths="half", d_c=rng.choice([128, 256]))
        else:
            c.update(seq=_log_int(rng, 32, 2048), widths=rng.choice(["v3", "half", "small"]), dtype="fp32",
                     d_c=rng.choice([64, 256, 512]))
    # no more work than the longest listed step (fused and fp32 run slower per pair)
    slow = 3 if c["fused"] else 24 if c["dtype"] == "fp32" else 1
    most = 16 * 16384 * 16385 // 2
    while slow * _pairs(c) > most:
        c["seq"] = c["seq"] * 2 // 3
    return c


def _torch_dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _problem(case):
    dn, dr, dv = WIDTHS[case["widths"]]
    return laga.Problem(batch=case["batch"], seq_len=case["seq"], n_heads=case["heads"], d_c=case["d_c"], d_nope=dn,
                        d_rope=dr, d_v=dv, softmax_scale=1.0 / math.sqrt(dn + dr), causal=int(case.get("causal", True)),
                        dtype=laga.DTYPE_BF16 if case["dtype"] == "bf16" else laga.DTYPE_FP32,
                        kv_mode=laga.KV_FUSED if case.get("fused") else laga.KV_MATERIALIZED,
                        dq_mode=laga.DQ_RECOMPUTE if case.get("recompute") else laga.DQ_FROM_STORE)


def _out_problem(case):
    return laga.OutProj(tokens=case["tokens"], n_heads=case["heads"], d_v=case["d_v"], d_model=case["d_model"],
                        dtype=laga.DTYPE_BF16 if case["dtype"] == "bf16" else laga.DTYPE_FP32)


def _inputs(case, seed):
    """The call's inputs on the GPU, from the seed alone: an RMS-normalised latent, N(0, 1)
    queries, rope keys and upstream gradients, weights ~ N(0, 1 / fan-in); raw producer
    latents at a log-uniform scale per token; attention outputs below unit scale."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = _torch_dtype(case)

    def normal(shape, scale=1.0, to=dt):
        return torch.randn(shape, generator=gen, device="cuda").mul_(scale).to(to)

    if case["kind"] == "out_proj":
        T, D, F = case["tokens"], case["d_model"], case["heads"] * case["d_v"]
        return {"out": normal((T, case["heads"], case["d_v"]), 0.25), "w_o": normal((F, D), F ** -0.5),
                "dy": normal((T, D))}
    sh = _problem(case).shapes()
    if case["kind"] == "producers":
        scale = torch.empty(sh["c_kv"][:2] + (1,), device="cuda").uniform_(math.log(0.1), math.log(10.0),
                                                                          generator=gen).exp_()
        x = {"latent_raw": (torch.randn(sh["c_kv"], generator=gen, device="cuda") * scale).to(dt),
             "kpe_raw": normal(sh["k_pe"]), "q_raw": normal(sh["q"]), "dc_kv": normal(sh["c_kv"], to=torch.float32),
             "dk_pe": normal(sh["k_pe"], to=torch.float32), "dq_raw": normal(sh["q"]), "gamma": None}
        if case["gamma"]:
            x["gamma"] = torch.empty((case["d_c"],), device="cuda").uniform_(0.5, 1.5, generator=gen).to(dt)
        return x
    c = torch.randn(sh["c_kv"], generator=gen, device="cuda")
    c *= torch.rsqrt(c.square().mean(-1, keepdim=True) + 1e-6)
    x = {"c_kv": c.to(dt), "k_pe": normal(sh["k_pe"]), "q": normal(sh["q"]),
         "w_kv_b": normal(sh["w_kv_b"], case["d_c"] ** -0.5)}
    if case["kind"] == "step":
        x["dout"] = normal(sh["dout"])
    return x


def prepare(case, seed):
    s = {"case": case, "x": _inputs(case, seed)}
    dt, f32 = _torch_dtype(case), torch.float32

    def new(shape, dtype):
        return torch.empty(shape, dtype=dtype, device="cuda")

    def workspace(nbytes):
        return new((max(1, nbytes),), torch.uint8)

    if case["kind"] == "out_proj":
        p = s["p"] = _out_problem(case)
        sh = p.shapes()
        s["buf"] = {"y": new(sh["y"], dt), "d_out": new(sh["d_out"], dt), "dw_o": new(sh["dw_o"], f32)}
        s["ws"] = workspace(laga.laga_out_proj_workspace_bytes(p))
        return s
    p = s["p"] = _problem(case)
    sh = p.shapes()
    if case["kind"] == "producers":
        s["buf"] = {"c_kv": new(sh["c_kv"], dt), "k_pe": new(sh["k_pe"], dt), "rstd": new(sh["c_kv"][:2], f32),
                    "q": s["x"]["q_raw"].clone(), "dq": s["x"]["dq_raw"].clone(),
                    "d_latent_raw": new(sh["c_kv"], f32), "d_kpe_raw": new(sh["k_pe"], f32),
                    "d_gamma": new((case["d_c"],), f32) if case["gamma"] else None}
        s["ws"] = workspace(laga.laga_workspace_bytes(p, laga.OP_PROLOGUE_BWD))
        return s
    s["buf"] = {"out": new(sh["out"], dt), "lse": new(sh["lse"], f32)}
    s["kv"] = None if case["fused"] else new(sh["kv"], dt)
    s["ws_fwd"] = workspace(laga.laga_workspace_bytes(p, laga.OP_FWD))
    if case["kind"] == "step":
        s["buf"].update(dq=new(sh["dq"], dt), dc_kv=new(sh["dc_kv"], f32), dk_pe=new(sh["dk_pe"], f32),
                        dw_kv_b=new(sh["dw_kv_b"], f32))
        s["ws_bwd"] = None if case["noalloc"] else workspace(laga.laga_workspace_bytes(p, laga.OP_BWD))
    return s


def run(s):
    case, p, x, buf = s["case"], s["p"], s["x"], s["buf"]
    if case["kind"] == "out_proj":
        laga.laga_out_proj_fwd(p, x["out"], x["w_o"], y=buf["y"])
        laga.laga_out_proj_bwd(p, x["out"], x["w_o"], x["dy"], d_out=buf["d_out"], dw_o=buf["dw_o"],
                               workspace=s["ws"])
        return buf
    if case["kind"] == "producers":
        # the bands are rotated in place: each pass starts from new q and dq there
        dn = p.d_nope
        buf["q"][..., dn:].copy_(x["q_raw"][..., dn:])
        laga.laga_prologue_fwd(p, x["latent_raw"], x["kpe_raw"], q=buf["q"], gamma=x["gamma"],
                               position_offset=case["offset"], c_kv=buf["c_kv"], k_pe=buf["k_pe"], rstd=buf["rstd"])
        buf["dq"][..., dn:].copy_(x["dq_raw"][..., dn:])
        laga.laga_prologue_bwd(p, x["latent_raw"], buf["rstd"], x["dc_kv"], x["dk_pe"], dq=buf["dq"],
                               gamma=x["gamma"], position_offset=case["offset"], d_latent_raw=buf["d_latent_raw"],
                               d_kpe_raw=buf["d_kpe_raw"], d_gamma=buf["d_gamma"], workspace=s["ws"])
        return buf
    kv = s["kv"]
    if kv is not None:
        laga.laga_reconstruct_kv(p, x["c_kv"], x["w_kv_b"], kv=kv)
    laga.laga_attn_fwd(p, x["q"], x["c_kv"], x["k_pe"], x["w_kv_b"], kv, out=buf["out"], lse=buf["lse"],
                       workspace=s["ws_fwd"])
    if case["kind"] == "forward":
        return dict(buf, kv=kv)
    args = (p, x["q"], x["c_kv"], x["k_pe"], x["w_kv_b"], kv, buf["out"], buf["lse"], x["dout"])
    grads = {k: buf[k] for k in ("dq", "dc_kv", "dk_pe", "dw_kv_b")}
    if case["noalloc"]:
        laga.laga_attn_bwd_noalloc(*args, **grads)
    else:
        laga.laga_attn_bwd(*args, **grads, workspace=s["ws_bwd"])
    return buf


def work(case):
    e = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "out_proj":
        T, F, D = case["tokens"], case["heads"] * case["d_v"], case["d_model"]
        return {"bytes": e * (2 * T * F + 2 * T * D + F * D) + 4 * F * D, "flops": 6 * T * F * D}
    dn, dr, dv = WIDTHS[case["widths"]]
    tok, H, dc = case["batch"] * case["seq"], case["heads"], case["d_c"]
    if case["kind"] == "producers":
        fwd = e * (2 * dc + 2 * dr + 2 * H * dr) + 4
        bwd = e * (dc + 2 * H * dr) + 4 + 4 * (2 * dc + 2 * dr)
        return {"bytes": tok * (fwd + bwd), "flops": tok * (10 * dc + 6 * (2 * dr + 2 * H * dr))}
    # q, c_kv, k_pe and W read, out and lse written (and kv, where it is a result)
    bytes_ = e * (tok * (H * (dn + dr) + dc + dr + H * dv) + dc * H * (dn + dv)) + 4 * tok * H
    up, att = 2 * tok * dc * H * (dn + dv), 2 * _pairs(case) * (dn + dr + dv)
    if not case["fused"] and case["kind"] == "forward":
        bytes_ += e * tok * H * (dn + dv)
    if case["kind"] == "forward":
        return {"bytes": bytes_, "flops": up + att}
    # dout read; dq, dc_kv, dk_pe, dW written
    bytes_ += e * tok * H * (dv + dn + dr) + 4 * (tok * (dc + dr) + dc * H * (dn + dv))
    return {"bytes": bytes_, "flops": 3 * up + 3 * att}


def tolerance(case):
    # about four times the largest error against float64 that each kind of call shows
    if case["dtype"] == "fp32":
        return {"rel": 1e-5}
    if case["kind"] in ("producers", "out_proj"):
        return {"rel": 7e-3}
    return {"rel": 1.4e-2}


def _rope(x, pos, base, sign):
    d = x.shape[-1]
    ang = pos[:, None] * base ** (-torch.arange(0, d, 2, dtype=torch.float64, device=x.device) / d)
    c, s = torch.cos(ang), sign * torch.sin(ang)
    if x.dim() == 4:
        c, s = c[:, None], s[:, None]
    x0, x1 = x[..., 0::2], x[..., 1::2]
    return torch.stack((x0 * c - x1 * s, x0 * s + x1 * c), -1).flatten(-2)


def exact(case, seed):
    x = {k: v.double() if v is not None else None for k, v in _inputs(case, seed).items()}
    if case["kind"] == "out_proj":
        F = case["heads"] * case["d_v"]
        o = x["out"].reshape(-1, F)
        return {"y": o @ x["w_o"], "d_out": (x["dy"] @ x["w_o"].t()).reshape(x["out"].shape), "dw_o": o.t() @ x["dy"]}
    dn, dr, dv = WIDTHS[case["widths"]]
    B, S, H = case["batch"], case["seq"], case["heads"]
    if case["kind"] == "producers":
        pos = case["offset"] + torch.arange(S, dtype=torch.float64, device="cuda")
        lat, g, dc = x["latent_raw"], x["gamma"], x["dc_kv"]
        rstd = torch.rsqrt(lat.square().mean(-1) + 1e-6)
        y = lat * rstd[..., None]
        gd = dc if g is None else dc * g
        q, dq = x["q_raw"], x["dq_raw"]
        q[..., dn:] = _rope(q[..., dn:], pos, 10000.0, 1.0)
        dq[..., dn:] = _rope(dq[..., dn:], pos, 10000.0, -1.0)
        return {"c_kv": y if g is None else y * g, "k_pe": _rope(x["kpe_raw"], pos, 10000.0, 1.0), "rstd": rstd,
                "q": q, "dq": dq,
                "d_latent_raw": rstd[..., None] * (gd - y * (gd * y).mean(-1, keepdim=True)),
                "d_kpe_raw": _rope(x["dk_pe"], pos, 10000.0, -1.0),
                "d_gamma": None if g is None else (dc * y).sum((0, 1))}
    step = case["kind"] == "step"
    scale = 1.0 / math.sqrt(dn + dr)
    kv = (x["c_kv"].reshape(B * S, -1) @ x["w_kv_b"]).reshape(B, S, H, dn + dv)
    out = torch.empty((B, S, H, dv), dtype=torch.float64, device="cuda")
    lse = torch.empty((B, H, S), dtype=torch.float64, device="cuda")
    if step:
        dq, dkv = torch.empty_like(x["q"]), torch.zeros_like(kv)
        dk_pe = torch.zeros_like(x["k_pe"])
    rows = 2048
    for b in range(B):
        for h in range(H):
            k = torch.cat((kv[b, :, h, :dn], x["k_pe"][b]), -1)
            v, qh = kv[b, :, h, dn:].contiguous(), x["q"][b, :, h].contiguous()
            for i in range(0, S, rows):
                j = min(S, i + rows)
                n = j if case["causal"] else S
                z = (qh[i:j] @ k[:n].t()).mul_(scale)
                if case["causal"]:
                    z[:, i:].masked_fill_(torch.ones((j - i, n - i), dtype=torch.bool, device="cuda").triu(1), -math.inf)
                lse[b, h, i:j] = torch.logsumexp(z, -1)
                z = z.sub_(lse[b, h, i:j, None]).exp_()
                o = z @ v[:n]
                out[b, i:j, h] = o
                if not step:
                    continue
                do = x["dout"][b, i:j, h]
                dkv[b, :n, h, dn:] += z.t() @ do
                dz = (do @ v[:n].t()).sub_((do * o).sum(-1, keepdim=True)).mul_(z).mul_(scale)
                dq[b, i:j, h] = dz @ k[:n]
                dk = dz.t() @ qh[i:j]
                dkv[b, :n, h, :dn] += dk[:, :dn]
                dk_pe[b, :n] += dk[:, dn:]
    if not step:
        return {"out": out, "lse": lse, "kv": None if case["fused"] else kv}
    dkv = dkv.reshape(B * S, -1)
    return {"out": out, "lse": lse, "dq": dq, "dc_kv": (dkv @ x["w_kv_b"].t()).reshape(B, S, -1), "dk_pe": dk_pe,
            "dw_kv_b": x["c_kv"].reshape(B * S, -1).t() @ dkv}
