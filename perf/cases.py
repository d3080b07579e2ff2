"""The work that a program using this library has it do, as cases that can be timed and checked.

A draft step of a speculative decoder calls `retrieve_fuse` once per tree depth on bf16
states, then `lm_topk` for the next depth's tokens; every new image costs one
`build_memory`.  A trainer runs the fp32 step, its backward and the memory build's
backward.  The cases span one request to a full batch, LLaVA- and Qwen-VL-class widths,
a single image to a video, and every option that such programs set (a padding mask,
fixed and mass-driven cardinality, the optional outputs).

Inputs are synthetic and drawn on the GPU from the seed: weights N(0, 1/fan_in), states
N(0, 1), keys in 16 spatial clusters whose scale sets the spread of the scores (the
softmax temperature that a trained module ends at differs per request).
"""

import math

import torch

from paper_2608_22883_amd import fovea as lib

DEV = "cuda"
D_C = 512      # hidden width of the correction and gate nets
N_DEPTH = 7    # tree depths 0..6


def _step(**kw):
    base = dict(kind="step", dtype="bf16", B=1, T=60, M=576, M_lo=0, d=4096, d_m=1024, k_min=1,
                k_max=64, tau=0.8, tau_hi=0.8, s_lo=2.0, s_hi=2.0, valid=1.0, diag=False)
    base.update(kw)
    return base


def listed():
    return [
        # one user, one image, one draft depth: the smallest call, latency bound
        _step(name="step_one_request"),
        # the same with the key width equal to the hidden size and 32 to 256 entries a node
        _step(name="step_one_request_wide", d_m=4096, k_min=32, k_max=256, s_lo=1.4, s_hi=1.4),
        # a serving batch: 32 requests of 60 nodes, one 24 x 24 patch image each
        _step(name="step_batch", B=32, tau=0.6, tau_hi=0.95, s_lo=1.2, s_hi=8.0),
        # dynamic-resolution images: ragged, padded memories; every optional output is read
        _step(name="step_ragged", B=16, T=48, M=4096, M_lo=256, d=3584, d_m=896, k_max=128,
              tau=0.85, tau_hi=0.85, s_lo=2.0, s_hi=3.0, valid=0.9, diag=True),
        # long video memories, the largest a request may have
        _step(name="step_video", B=8, T=64, M=16384, d=5120, d_m=1280, k_max=256, tau=0.9,
              tau_hi=0.9, s_lo=0.3, s_hi=60.0),
        # the trainer's forward: fp32, cardinality held at 16
        _step(name="step_train", dtype="f32", B=32, k_min=16, k_max=16, s_lo=1.2, s_hi=8.0),
        # the trainer's backward of that step
        dict(name="step_backward", kind="step_backward", B=32, T=60, M=576, d=4096, d_m=1024,
             k=16, s_lo=1.2, s_hi=8.0),
        # a new image arrives: 576 visual tokens
        dict(name="build_image", kind="build", dtype="bf16", rows=576, d=4096, d_m=1024),
        # the images of a whole batch at once
        dict(name="build_batch", kind="build", dtype="bf16", rows=18432, d=4096, d_m=1024),
        # the trainer's backward of the memory build, 8 images
        dict(name="build_backward", kind="build_backward", rows=4608, d=4096, d_m=1024),
        # draft tokens of one request's nodes: bound by reading the head
        dict(name="lm_one_request", kind="lm", dtype="bf16", rows=60, vocab=32000, d=4096, k=6),
        # draft tokens of a batch over a large vocabulary
        dict(name="lm_batch", kind="lm", dtype="bf16", rows=768, vocab=152064, d=3584, k=6),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges; costs are capped by the largest listed cases."""
    kind = rng.choice(["step"] * 6 + ["train", "step_backward", "build", "build_backward", "lm", "lm"])
    d, d_m = rng.choice([(4096, 1024), (3584, 896), (5120, 1280), (4096, 4096), (2048, 512)])
    if kind in ("step", "train"):
        B, T = _log_int(rng, 1, 32), rng.randint(4, 64)
        M = _log_int(rng, 100, 4096 if rng.random() < 0.7 else 16384)
        if kind == "train":
            B, M = min(B, 16), min(M, 1024)
        while B > 1 and B * M * d_m > 8 * 16384 * 1280:
            B //= 2
        lo = rng.uniform(0.8, 2.0)
        tau = round(rng.uniform(0.6, 0.9), 2)
        c = _step(B=B, T=T, M=M, M_lo=max(1, M // 8) if rng.random() < 0.4 else 0, d=d, d_m=d_m,
                  tau=tau, tau_hi=round(min(0.95, tau + rng.uniform(0, 0.2)), 2), s_lo=lo,
                  s_hi=lo * rng.uniform(1.0, 6.0), valid=rng.choice([1.0, 1.0, 0.9]))
        c["k_min"], c["k_max"] = rng.choice([(1, 64), (1, 128), (32, 256), (16, 16)])
        if kind == "train":
            c.update(dtype="f32", k_min=16, k_max=16)
        # one node more or less in K is over the comparison's bound on a handful of nodes
        c["diag"] = kind == "step" and (c["k_min"] == c["k_max"] or B * T >= 400) and rng.random() < 0.5
        return c
    if kind == "step_backward":
        return dict(kind=kind, B=_log_int(rng, 1, 32), T=rng.randint(8, 60), M=_log_int(rng, 100, 1024),
                    d=d, d_m=min(d_m, 1280), k=16, s_lo=1.2, s_hi=rng.uniform(2.0, 8.0))
    if kind == "build":
        rows = _log_int(rng, 144, 18432)
        return dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "f32"]) if rows < 4608 else "bf16",
                    rows=rows, d=d, d_m=min(d_m, 1280))
    if kind == "build_backward":
        return dict(kind=kind, rows=_log_int(rng, 144, 4608), d=d, d_m=min(d_m, 1280))
    vocab, d = rng.choice([(32000, 4096), (152064, 3584), (32064, 2048), (50257, 5120)])
    rows = _log_int(rng, 1, 1920)
    while rows > 1 and rows * vocab * d > 768 * 152064 * 3584:
        rows = rows * 2 // 3
    return dict(kind=kind, dtype="bf16", rows=rows, vocab=vocab, d=d, k=rng.choice([1, 4, 6, 6, 10, 16]))


# ---- inputs ---------------------------------------------------------------------------


class _Gen:
    """Normal and uniform draws on the GPU from one seed, rounded once to the storage type."""

    def __init__(self, seed, dtype):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed) % (1 << 62))
        self.dtype = torch.bfloat16 if dtype == "bf16" else torch.float32

    def raw(self, *shape):
        return torch.randn(*shape, generator=self.g, device=DEV)

    def normal(self, shape, std):
        return (self.raw(*shape) * std).to(self.dtype)


def _weights(g, d, d_m, affine):
    """`affine`: LayerNorm gains, biases and the nets' biases away from their initial 1 and 0."""
    one = lambda n: (1.0 + affine * g.raw(n)).to(g.dtype)  # noqa: E731
    zero = lambda n: g.normal((n,), affine)  # noqa: E731
    s = 1.0 / math.sqrt(d)
    s1 = 1.0 / math.sqrt(d + d_m)
    return dict(
        q_ln_g=one(d), q_ln_b=zero(d), E_dep=g.normal((N_DEPTH, d), 0.5), W_Q=g.normal((d_m, d), s),
        W_c1=g.normal((D_C, d + d_m), s1), b_c1=zero(D_C),
        W_c2=g.normal((d, D_C), 1.0 / math.sqrt(D_C)), b_c2=zero(d),
        W_g1=g.normal((D_C, d + d_m), s1), b_g1=zero(D_C), w_g2=g.normal((D_C,), 1.0 / math.sqrt(D_C)),
        b_g2=-2.0, rms_w=one(d), mem_ln_g=one(d), mem_ln_b=zero(d), W_K=g.normal((d_m, d), s),
        W_U=g.normal((d_m, d), s))


def _draft_step(case, seed, g):
    """Offsets, memory and states of B requests; fp64 lists stay on the host."""
    B, T, M, d, d_m = (case[k] for k in ("B", "T", "M", "d", "d_m"))
    lo = case.get("M_lo") or M
    host = torch.Generator()
    host.manual_seed(int(seed) % (1 << 62))
    Ms = torch.randint(lo, M + 1, (B,), generator=host).tolist()
    off = [0]
    for m in Ms:
        off.append(off[-1] + m)
    n_mem = off[-1]
    keys = torch.empty(n_mem, d_m, dtype=g.dtype, device=DEV)
    values = torch.empty(n_mem, d_m, dtype=g.dtype, device=DEV)
    half = math.sqrt(0.5 / d_m)  # half of an entry's variance lies in its cluster's centre
    for b, m in enumerate(Ms):
        t = (b + 0.5) / B
        spread = math.exp((1 - t) * math.log(case["s_lo"]) + t * math.log(case["s_hi"]))
        scale = spread * math.sqrt(d_m) / 1.12  # |q_i| is about 1.12 (states plus depth embedding)
        c = torch.arange(m, device=DEV) * 16 // m
        boost = 1.0 + (torch.rand(m, 1, generator=g.g, device=DEV) < 0.1).float()
        keys[off[b]:off[b + 1]] = ((g.raw(16, d_m)[c] + g.raw(m, d_m)) * half * scale * boost).to(g.dtype)
        values[off[b]:off[b + 1]] = ((g.raw(16, d_m)[c] + g.raw(m, d_m)) * half).to(g.dtype)
    j = torch.arange(T)
    depth = torch.where(j == 0, 0, torch.where(j < 7, 1, 2 + (j - 7) * 5 // max(T - 7, 1))).to(torch.int32)
    valid = None
    if case.get("valid", 1.0) < 1.0:
        valid = (torch.rand(n_mem, generator=g.g, device=DEV) < case["valid"]).to(torch.uint8)
    tau_lo, tau_hi = case.get("tau", 0.8), case.get("tau_hi", 0.8)
    return dict(
        mem_off=torch.tensor(off, dtype=torch.int64, device=DEV), keys=keys, values=values, valid=valid,
        node_off=(torch.arange(B + 1) * T).to(device=DEV, dtype=torch.int32),
        h=g.normal((B * T, d), 1.0), depth=depth.repeat(B).to(DEV),
        tau=tau_lo + (tau_hi - tau_lo) * torch.rand(B, generator=g.g, device=DEV),
        m_max=max(Ms), t_max=T, off=off)


def _query64(W, x):
    h = x["h"].double()
    mu = h.mean(1, keepdim=True)
    rstd = ((h - mu).square().mean(1, keepdim=True) + 1e-5).rsqrt()
    xe = (h - mu) * rstd * W["q_ln_g"].double() + W["q_ln_b"].double() + W["E_dep"].double()[x["depth"].long()]
    return xe @ W["W_Q"].double().t()


def _inputs(case, seed):
    g = _Gen(seed, case.get("dtype", "f32"))
    kind, d = case["kind"], case["d"]
    # bf16 modules keep the affine parameters' initial values, so that folding a gain into
    # a weight rounds nothing; fp32 ones have trained-looking gains and biases
    W = _weights(g, d, case.get("d_m", 1024), 0.0 if case.get("dtype") == "bf16" else 0.1)
    if kind == "step":
        return W, _draft_step(case, seed, g)
    if kind == "step_backward":
        x = _draft_step(case, seed, g)
        q, k = _query64(W, x), min(case["k"], x["m_max"])
        T, idx = case["T"], []
        for b in range(case["B"]):
            s = q[b * T:(b + 1) * T] @ x["keys"][x["off"][b]:x["off"][b + 1]].double().t()
            idx.append(s.topk(k, dim=1).indices)
        x["idx"] = torch.cat(idx).to(torch.int32)
        x["K"] = torch.full((x["h"].shape[0],), k, dtype=torch.int32, device=DEV)
        x["dh_hat"] = g.raw(*x["h"].shape)
        return W, x
    if kind == "lm":
        return W, dict(h=g.normal((case["rows"], d), 1.0), W_LM=g.normal((case["vocab"], d), 1.0 / math.sqrt(d)))
    x = dict(V=g.normal((case["rows"], d), 1.0))
    if kind == "build_backward":  # about half of the entries were selected by some node
        for name in ("dkeys", "dvalues"):
            hit = (torch.rand(case["rows"], 1, generator=g.g, device=DEV) < 0.5).float()
            x[name] = g.raw(case["rows"], case["d_m"]) * 0.1 * hit
    return W, x


# ---- the calls ------------------------------------------------------------------------


def prepare(case, seed):
    W, x = _inputs(case, seed)
    bf16 = case.get("dtype") == "bf16"
    fv = lib.Fovea(dict(d=case["d"], d_v=case["d"], d_m=case.get("d_m", 1024), d_c=D_C, n_depth=N_DEPTH,
                        dtype=lib.FOVEA_BF16 if bf16 else lib.FOVEA_F32, ln_eps=1e-5, rms_eps=1e-6),
                   W, device=DEV)
    st = dict(case=case, fv=fv, x=x)
    n = x["h"].shape[0] if "h" in x else 0
    if case["kind"] == "step":
        x["k_min"], x["k_max"] = case["k_min"], case["k_max"]
        st["out"] = fv.alloc_outputs(n, case["k_max"], case["d"], case["d_m"])
        fv.ensure_workspace(case["B"], n, x["keys"].shape[0], x["m_max"], case["k_max"])
    elif case["kind"] == "build":
        dt = x["V"].dtype
        st["keys"], st["values"] = (torch.empty(case["rows"], case["d_m"], dtype=dt, device=DEV) for _ in "ku")
        need = lib.fovea_build_memory_workspace(fv.ctx, case["rows"])
        st["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV)
    elif case["kind"] == "lm":
        st["idx"] = torch.empty(n, case["k"], dtype=torch.int32, device=DEV)
        st["logit"] = torch.empty(n, case["k"], dtype=torch.float32, device=DEV)
    return st


def run(st):
    case, fv, x, kind = st["case"], st["fv"], st["x"], st["case"]["kind"]
    if kind == "step":
        out = st["out"]
        if case["diag"]:
            fv.retrieve_fuse(x, out)
            return dict(h=out.h_out, k=out.k, idx=out.idx, gate=out.gate, mass=out.mass, r=out.r)
        if case["dtype"] == "bf16":
            fv.retrieve_fuse(x, out, debug=False)
            return dict(h=out.h_out)
        # a trainer keeps the selection for the backward, and no other optional output
        lib.fovea_retrieve_fuse(
            fv.ctx, case["B"], x["mem_off"], x["keys"].shape[0], x["m_max"], x["keys"], x["values"],
            x["valid"], x["node_off"], x["h"].shape[0], x["t_max"], x["h"], x["depth"], x["tau"],
            x["k_min"], x["k_max"], out.h_out, k_out=out.k, idx_out=out.idx, workspace=fv.workspace)
        return dict(h=out.h_out, k=out.k, idx=out.idx)
    if kind == "step_backward":
        return fv.retrieve_fuse_backward(x, x["K"], x["idx"], x["dh_hat"])
    if kind == "build":
        keys, values = fv.build_memory(x["V"], st["keys"], st["values"], st["ws"])
        return dict(keys=keys, values=values)
    if kind == "build_backward":
        return fv.build_memory_backward(x["V"], x["dkeys"], x["dvalues"])
    idx, logit = fv.lm_topk(x["h"], x["W_LM"], case["k"], st["idx"], st["logit"])
    return dict(idx=idx, logit=logit)


# ---- what a pass cannot do without ------------------------------------------------------


def work(case):
    d, d_m, kind = case["d"], case.get("d_m", 1024), case["kind"]
    es = 2 if case.get("dtype") == "bf16" else 4
    w_step = d * (d_m + 2 * D_C) + 2 * D_C * d_m + d * D_C
    if kind in ("step", "step_backward"):
        B, T, n = case["B"], case["T"], case["B"] * case["T"]
        M = (case["M"] + (case.get("M_lo") or case["M"])) / 2
    if kind == "step":
        rows = B * min(M, T * max(4, case["k_min"]))  # distinct value rows read, at least about this
        byts = es * (B * M * d_m + rows * d_m + 2 * n * d + w_step)
        if case["diag"]:
            byts += 4 * n * (d_m + case["k_max"] + 3)
        return dict(bytes=byts, flops=2 * n * w_step + 2 * n * M * d_m)
    if kind == "step_backward":
        k = case["k"]
        rows = B * min(M, T * k / 2)
        byts = 4 * (3 * n * d + 2 * w_step + 2 * rows * d_m + 2 * B * M * d_m)
        return dict(bytes=byts, flops=3 * 2 * n * w_step + 8 * n * k * d_m)
    if kind == "build":
        r = case["rows"]
        return dict(bytes=es * (r * d + 2 * r * d_m + 2 * d_m * d), flops=4 * r * d * d_m)
    if kind == "build_backward":
        r = case["rows"]
        return dict(bytes=4 * (2 * r * d + 2 * r * d_m + 4 * d_m * d), flops=8 * r * d * d_m)
    r, v, k = case["rows"], case["vocab"], case["k"]
    return dict(bytes=2 * (r * d + v * d) + 8 * r * k, flops=2 * r * v * d)


def tolerance(case):
    """About four times what the outputs are off `exact` by (largest output of a case)."""
    kind, bf16 = case["kind"], case.get("dtype") == "bf16"
    if kind == "step":
        # bf16 states 2.4e-3 (rounded once), fp32 ones 2.2e-7.  Two entries whose scores tie, or
        # a prefix mass that meets tau, may fall either way: that moves r of one node by up to
        # its own size ("max") and an entry or two of the selections ("differ")
        return dict(rel=8e-3, max=0.9, differ=5e-3) if bf16 else dict(rel=1e-6, max=1e-3, differ=1e-3)
    if kind == "build":  # 1.7e-3 and 3e-7
        return dict(rel=7e-3, max=0.05) if bf16 else dict(rel=1.5e-6, max=1e-4)
    if kind == "lm":  # 3.5e-7; near ties change places
        return dict(rel=1.5e-6, max=1e-4, differ=2e-3)
    if kind == "step_backward":  # 3.2e-5 (the gradients through the scores)
        return dict(rel=1.3e-4, max=2e-2)
    return dict(rel=2e-5, max=2e-3)  # build_backward 4.9e-6


# ---- the same in 64 bits ----------------------------------------------------------------


def _exact_step(case, W, x):
    D = {k: v.double() if torch.is_tensor(v) else v for k, v in W.items()}
    q = _query64(W, x)
    n, d, d_m, T = x["h"].shape[0], case["d"], case["d_m"], case["T"]
    r = torch.zeros(n, d_m, dtype=torch.float64, device=DEV)
    mass = torch.zeros(n, dtype=torch.float64, device=DEV)
    clear = True  # no node's selection hangs on the last bits of a score
    for b in range(case["B"]):
        m0, m1 = x["off"][b], x["off"][b + 1]
        s = q[b * T:(b + 1) * T] @ x["keys"][m0:m1].double().t() / math.sqrt(d_m)
        live = m1 - m0
        if x["valid"] is not None:
            s = s.masked_fill(x["valid"][m0:m1] == 0, -math.inf)
            live = int(x["valid"][m0:m1].sum())
        if live == 0:
            continue
        top, at = torch.sort(s, dim=1, descending=True, stable=True)
        cum = torch.softmax(top, dim=1).cumsum(1)
        tau = x["tau"][b].double()
        C = min(live, case["k_max"])
        reach = cum[:, :C] >= tau
        raw = torch.where(reach.any(1), reach.int().argmax(1) + 1, live if C == live else case["k_max"] + 1)
        K = raw.clamp(min=case["k_min"]).clamp(max=C)
        if case["k_min"] < case["k_max"] and bool(((cum[:, :C] - tau).abs() < 2e-5).any()):
            clear = False
        if live > C or case["k_min"] < case["k_max"]:
            nxt = top.gather(1, K.clamp(max=top.shape[1] - 1)[:, None])[:, 0]
            gap = top.gather(1, (K - 1)[:, None])[:, 0] - nxt
            if bool((gap < 1e-4).any()):
                clear = False
        sel = torch.arange(C, device=DEV)[None, :] < K[:, None]
        p = torch.softmax(top[:, :C].masked_fill(~sel, -math.inf), dim=1)
        w = torch.zeros_like(s).scatter_(1, at[:, :C], p)
        r[b * T:(b + 1) * T] = w @ x["values"][m0:m1].double()
        mass[b * T:(b + 1) * T] = cum.gather(1, (K - 1)[:, None])[:, 0]
    h = x["h"].double()
    y = torch.cat([h, r], 1)
    silu = torch.nn.functional.silu
    c = silu(y @ D["W_c1"].t() + D["b_c1"]) @ D["W_c2"].t() + D["b_c2"]
    gate = torch.sigmoid(silu(y @ D["W_g1"].t() + D["b_g1"]) @ D["w_g2"] + D["b_g2"])
    hp = h + gate[:, None] * c
    out = dict(h=hp * (hp.square().mean(1, keepdim=True) + 1e-6).rsqrt() * D["rms_w"], k=None, idx=None)
    if case["diag"]:
        out.update(gate=gate, mass=mass if clear else None, r=r if clear else None)
    return out


def _exact_backward(case, W, x):
    leaf = lambda t: t.double().detach().requires_grad_()  # noqa: E731
    P = {k: leaf(v) for k, v in W.items() if torch.is_tensor(v)}
    b_g2 = torch.tensor([W["b_g2"]], dtype=torch.float64, device=DEV, requires_grad=True)
    h, keys, values = leaf(x["h"]), leaf(x["keys"]), leaf(x["values"])
    T, B = case["T"], case["B"]
    mu = h.mean(1, keepdim=True)
    xc = h - mu
    xe = xc * (xc.square().mean(1, keepdim=True) + 1e-5).rsqrt() * P["q_ln_g"] + P["q_ln_b"] + P["E_dep"][x["depth"].long()]
    q = xe @ P["W_Q"].t()
    row = x["idx"].long() + torch.tensor(x["off"][:B], device=DEV).repeat_interleave(T)[:, None]
    r = []
    for b in range(B):  # request by request: the gathered rows stay small
        i = row[b * T:(b + 1) * T]
        s = (q[b * T:(b + 1) * T, None, :] * keys[i]).sum(-1) / math.sqrt(case["d_m"])
        r.append((torch.softmax(s, 1)[:, :, None] * values[i]).sum(1))
    y = torch.cat([h, torch.cat(r)], 1)
    silu = torch.nn.functional.silu
    c = silu(y @ P["W_c1"].t() + P["b_c1"]) @ P["W_c2"].t() + P["b_c2"]
    gate = torch.sigmoid(silu(y @ P["W_g1"].t() + P["b_g1"]) @ P["w_g2"] + b_g2)
    hp = h + gate[:, None] * c
    hat = hp * (hp.square().mean(1, keepdim=True) + 1e-6).rsqrt() * P["rms_w"]
    hat.backward(x["dh_hat"].double())
    out = {"d" + k: P[k].grad for k in ("W_Q", "q_ln_g", "q_ln_b", "E_dep", "W_c1", "b_c1", "W_c2", "b_c2",
                                        "W_g1", "b_g1", "w_g2", "rms_w")}
    out.update(db_g2=b_g2.grad, dh=h.grad, dkeys=keys.grad, dvalues=values.grad)
    return out


def exact(case, seed):
    W, x = _inputs(case, seed)
    kind = case["kind"]
    if kind == "step":
        return _exact_step(case, W, x)
    if kind == "step_backward":
        return _exact_backward(case, W, x)
    if kind == "lm":
        best = None
        for v0 in range(0, case["vocab"], 16384):
            z = x["h"].double() @ x["W_LM"][v0:v0 + 16384].double().t()
            z = z if best is None else torch.cat([best, z], 1)
            best = z.topk(min(case["k"], z.shape[1]), dim=1).values
        return dict(idx=None, logit=best)
    V = x["V"].double()
    mu = V.mean(1, keepdim=True)
    rstd = ((V - mu).square().mean(1, keepdim=True) + 1e-5).rsqrt()
    hat = (V - mu) * rstd
    g, b, W_K, W_U = (W[k].double() for k in ("mem_ln_g", "mem_ln_b", "W_K", "W_U"))
    ln = hat * g + b
    if kind == "build":
        return dict(keys=ln @ W_K.t(), values=ln @ W_U.t())
    dk, du = x["dkeys"].double(), x["dvalues"].double()
    dln = dk @ W_K + du @ W_U
    t = dln * g
    dV = rstd * (t - t.mean(1, keepdim=True) - hat * (t * hat).mean(1, keepdim=True))
    return dict(dW_K=dk.t() @ ln, dW_U=du.t() @ ln, dmem_ln_g=(dln * hat).sum(0), dmem_ln_b=dln.sum(0), dV=dV)
