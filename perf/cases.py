"""The workloads that the framework's speed is measured on.

Each case is a dict of plain values; `prepare` makes what a user's program has in hand
before the call, `run` makes one pass through the public entry points, and `exact` gives
the same outputs in 64 bits from plain torch.  Six kinds of case:

  train    one training step of the sequence operators of a layer: causal_conv1d_fwd,
           selective_scan_fwd (saving states, unless `recompute`), selective_scan_bwd,
           causal_conv1d_bwd; the conv's output is the scan's input and the scan's du is
           the conv's upstream gradient.  `states`: every row continues a sequence cut at
           the end of another row, with initial and final states and their gradients.
  prefill  conv and scan forward without anything kept for a backward, each row
           continuing a sequence, final states returned for what follows.
  decode   the same two calls on the few tokens of one generation step, from the states
           that the step before left.
  norm     rmsnorm forward and backward, the residual's gradient added.
  block    one packed Mamba block forward and backward.
  conv     the packed conv alone, forward and backward.
"""
import math
import random

import numpy as np
import torch
import torch.nn.functional as F

import paper_2408_03865_amd as P
from paper_2408_03865_amd import block as BK

N = 16                      # d_state
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def listed():
    logn = dict(law="lognormal", lo=16, hi=4096, mu=6.0, sigma=1.0)
    return [
        # serving: 64 sequences of a 1.4B-wide model, one new token each
        dict(name="decode-1.4b", kind="decode", batch=64, seqlen=1, dim=4096, width=4, dtype="bf16"),
        # the framework's smallest configuration: a unit test's or a toy model's training
        # step, where launches and host work count
        dict(name="train-tiny", kind="train", batch=1, seqlen=256, dim=64, width=4, dtype="f32",
             law="short", lo=16, hi=96),
        # serving: prompts of an odd total length, cut rows with states passed on
        dict(name="prefill-130m", kind="prefill", batch=2, seqlen=3001, dim=1536, width=4, dtype="bf16",
             law="lognormal", lo=8, hi=2048, mu=5.5, sigma=1.0),
        # training at the Mamba-130M layer shape
        dict(name="train-130m", kind="train", batch=4, seqlen=2048, dim=1536, width=4, dtype="bf16",
             law="lognormal", lo=8, hi=2048, mu=5.5, sigma=1.0),
        # a length that is no multiple of anything, with states recomputed in the backward
        # (no activations kept) at the 2.8B width
        dict(name="train-ragged", kind="train", batch=3, seqlen=2049, dim=5120, width=4, dtype="bf16",
             recompute=True, **logn),
        # many short sequences (chat turns) in two rows
        dict(name="train-short-seqs", kind="train", batch=2, seqlen=8192, dim=2048, width=4, dtype="bf16",
             law="short", lo=1, hi=64),
        # long documents: one row of three sequences
        dict(name="train-long-row", kind="train", batch=1, seqlen=65536, dim=2048, width=4, dtype="bf16",
             law="long", lo=10000, hi=30000),
        # the headline workload: the Mamba-1.4B layer shape
        dict(name="train-1.4b", kind="train", batch=8, seqlen=4096, dim=4096, width=4, dtype="bf16", **logn),
        # the same with 32-bit activations
        dict(name="train-1.4b-f32", kind="train", batch=8, seqlen=4096, dim=4096, width=4, dtype="f32", **logn),
        # the block's norm at its 1.4B shape
        dict(name="norm-1.4b", kind="norm", batch=8, seqlen=4096, dim=2048, dtype="bf16"),
        # whole blocks: Mamba-130M and Mamba-1.4B
        dict(name="block-130m", kind="block", batch=4, seqlen=2048, d_model=768, dim=1536, rank=48, width=4,
             dtype="bf16", law="lognormal", lo=8, hi=2048, mu=5.5, sigma=1.0),
        dict(name="block-1.4b", kind="block", batch=8, seqlen=4096, d_model=2048, dim=4096, rank=128, width=4,
             dtype="bf16", **logn),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["train"] * 5 + ["prefill", "prefill", "decode", "norm", "block", "conv"])
    # channel counts: mostly the multiples of 64 that models have, sometimes any
    dim = _log_uniform(rng, 64, 5120)
    if rng.random() < 0.75:
        dim = max(64, dim // 64 * 64)
    dtype = "bf16" if rng.random() < 0.75 else "f32"
    law = rng.choice(["lognormal", "lognormal", "short", "long", "one"])
    lens = {"lognormal": dict(lo=8, hi=4096, mu=round(rng.uniform(4.5, 6.5), 2), sigma=1.0),
            "short": dict(lo=1, hi=rng.choice([16, 64, 96])),
            "long": dict(lo=2000, hi=30000), "one": {}}[law]
    width = 4 if rng.random() < 0.8 else rng.choice([2, 3])
    if kind == "decode":
        return dict(kind=kind, batch=_log_uniform(rng, 1, 128), seqlen=rng.choice([1, 1, 1, 2, 3, 5, 8]), dim=dim,
                    width=width, dtype=dtype)
    seqlen = _log_uniform(rng, 64, 16384)
    if rng.random() < 0.5:
        seqlen = max(64, seqlen // 64 * 64)
    if kind == "block":
        d_model = rng.choice([256, 512, 768, 1024, 2048])
        seqlen = max(64, min(seqlen, 8192) // 64 * 64)
        batch = max(1, min(rng.choice([1, 2, 4, 8]), 32768 // seqlen))
        return dict(kind=kind, batch=batch, seqlen=seqlen, d_model=d_model, dim=2 * d_model, rank=d_model // 16,
                    width=4, dtype="bf16", law=law, **lens)
    most = (1 << 26) if dtype == "f32" else (1 << 27)       # elements of one activation
    batch = max(1, min(_log_uniform(rng, 1, 16), most // (seqlen * dim)))
    if kind == "norm":
        return dict(kind=kind, batch=batch, seqlen=seqlen, dim=max(64, dim // 2), dtype=dtype)
    case = dict(kind=kind, batch=batch, seqlen=seqlen, dim=dim, width=width, dtype=dtype, law=law, **lens)
    if kind == "train":
        case["recompute"] = rng.random() < 0.2
        case["states"] = rng.random() < 0.2
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _positions(case, rng, first=None):
    """Position indices (batch, seqlen): rows filled with sequences of the case's length
    law, the last cut at the row end.  `first` (batch ints): each row continues a sequence
    of which that many tokens lie in another row."""
    L = case["seqlen"]
    pos = np.empty((case["batch"], L), dtype=np.int32)
    law = case.get("law", "one")
    for b in range(case["batch"]):
        off = 0
        while off < L:
            if law == "lognormal":
                n = min(max(int(round(math.exp(rng.gauss(case["mu"], case["sigma"])))), case["lo"]), case["hi"])
            elif law in ("short", "long"):
                n = rng.randint(case["lo"], case["hi"])
            else:
                n = L
            n = min(n, L - off)
            start = first[b] if first is not None and off == 0 else 0
            pos[b, off:off + n] = np.arange(start, start + n, dtype=np.int32)
            off += n
    return torch.from_numpy(pos).cuda()


def prepare(case, seed):
    rng = random.Random(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = DTYPES[case["dtype"]]
    kind = case["kind"]
    Nb, L, Dn = case["batch"], case["seqlen"], case["dim"]

    def normal(*shape, dtype=torch.float32):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(dtype)

    def uniform(lo, hi, *shape):
        return torch.rand(shape, generator=gen, device="cuda", dtype=torch.float32) * (hi - lo) + lo

    s = {"case": dict(case)}
    if kind == "norm":
        s.update(x=normal(Nb, Dn, L, dtype=dt), w=uniform(0.5, 1.5, Dn), dout=normal(Nb, Dn, L, dtype=dt),
                 dres=normal(Nb, Dn, L, dtype=dt))
        return s
    continued = kind in ("prefill", "decode") or case.get("states", False)
    s["pos"] = _positions(case, rng, [rng.randint(1, 2000) for _ in range(Nb)] if continued else None)
    W = case["width"]
    if kind == "block":
        M, R = case["d_model"], case["rank"]

        def weight(rows, cols):
            return (normal(rows, cols) / math.sqrt(cols)).to(dt)

        s["p"] = dict(norm_w=uniform(0.5, 1.5, M), W_in=weight(2 * Dn, M), conv_w=uniform(-0.5, 0.5, Dn, W),
                      conv_b=uniform(-0.5, 0.5, Dn), W_x=weight(R + 2 * N, Dn), W_dt=weight(Dn, R),
                      dt_bias=torch.log(torch.expm1(uniform(1e-3, 1e-1, Dn))),
                      A=-torch.exp(normal(Dn, N) * 0.5), D=normal(Dn), W_out=weight(M, Dn))
        s["x"] = normal(Nb, M, L, dtype=dt)
        s["dout"] = normal(Nb, M, L, dtype=dt)
        return s
    s.update(x=normal(Nb, Dn, L, dtype=dt), w=uniform(-0.5, 0.5, Dn, W), bias=uniform(-0.5, 0.5, Dn))
    if kind in ("train", "conv"):
        s["dout"] = normal(Nb, Dn, L, dtype=dt)
    if kind == "conv":
        return s
    s.update(z=normal(Nb, Dn, L, dtype=dt), delta=normal(Nb, Dn, L, dtype=dt), B=normal(Nb, N, L, dtype=dt),
             C=normal(Nb, N, L, dtype=dt), A=-torch.exp(normal(Dn, N) * 0.5), D=normal(Dn),
             dbias=torch.log(torch.expm1(uniform(1e-3, 1e-1, Dn))))
    if continued:
        s.update(x0=normal(Nb, Dn, W - 1, dtype=dt), h0=normal(Nb, Dn, N))
        if kind == "train":
            s.update(dxf=normal(Nb, Dn, W - 1, dtype=dt), dhf=normal(Nb, Dn, N))
    return s


# ---------------------------------------------------------------------------
# one pass through the public entry points
# ---------------------------------------------------------------------------

def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "norm":
        out, rstd = P.rmsnorm_fwd(s["x"], s["w"])
        dx, dw = P.rmsnorm_bwd(s["x"], s["w"], rstd, s["dout"], dresidual=s["dres"])
        return dict(out=out, rstd=rstd, dx=dx, dw=dw)
    if kind == "block":
        out, ctx = BK.block_forward(s["x"], s["pos"], s["p"])
        g = BK.block_backward(s["dout"], ctx, s["p"])
        return dict(out=out, **{"d" + k: v for k, v in g.items()})
    if kind == "conv":
        u = P.causal_conv1d_fwd(s["x"], s["w"], s["bias"], s["pos"], silu=True)
        dx, dw, db = P.causal_conv1d_bwd(s["x"], s["w"], s["bias"], s["pos"], s["dout"], silu=True)
        return dict(u=u, dx=dx, dw=dw, db=db)
    scan = lambda u: (u, s["delta"], s["A"], s["B"], s["C"], s["D"], s["z"], s["dbias"], True, s["pos"])  # noqa: E731
    if kind in ("prefill", "decode"):
        u, xf = P.causal_conv1d_fwd(s["x"], s["w"], s["bias"], s["pos"], silu=True, initial_x=s["x0"],
                                    return_final=True)
        y, hf = P.selective_scan_fwd(*scan(u), initial_state=s["h0"], return_final=True)
        return dict(u=u, xf=xf, y=y, hf=hf)
    r = {}
    if c.get("states"):
        u, r["xf"] = P.causal_conv1d_fwd(s["x"], s["w"], s["bias"], s["pos"], silu=True, initial_x=s["x0"],
                                         return_final=True)
        if c.get("recompute"):
            y, r["hf"] = P.selective_scan_fwd(*scan(u), initial_state=s["h0"], return_final=True)
            st = None
        else:
            y, st, r["hf"] = P.selective_scan_fwd(*scan(u), return_states=True, initial_state=s["h0"],
                                                  return_final=True)
        g = P.selective_scan_bwd(*scan(u), s["dout"], saved_states=st, initial_state=s["h0"], dfinal_state=s["dhf"])
        r["dx"], r["dw"], r["db"], r["dx0"] = P.causal_conv1d_bwd(s["x"], s["w"], s["bias"], s["pos"], g["du"],
                                                                  silu=True, initial_x=s["x0"], dfinal_x=s["dxf"])
    else:
        u = P.causal_conv1d_fwd(s["x"], s["w"], s["bias"], s["pos"], silu=True)
        if c.get("recompute"):
            y, st = P.selective_scan_fwd(*scan(u)), None
        else:
            y, st = P.selective_scan_fwd(*scan(u), return_states=True)
        g = P.selective_scan_bwd(*scan(u), s["dout"], saved_states=st)
        r["dx"], r["dw"], r["db"] = P.causal_conv1d_bwd(s["x"], s["w"], s["bias"], s["pos"], g["du"], silu=True)
    r.update(u=u, y=y, **{k: v for k, v in g.items() if v is not None})
    return r


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    """Bytes: every input of each call read once and every output written once.  Flops: a
    multiply-add counts two, an exponential one."""
    kind = case["kind"]
    Nb, L, Dn = case["batch"], case["seqlen"], case["dim"]
    s = 4 if case["dtype"] == "f32" else 2
    E, T = Nb * L * Dn, Nb * L
    if kind == "norm":
        return {"bytes": 6 * s * E + 8 * T + 12 * Dn, "flops": 14 * E}
    W = case["width"]
    par = 4 * (Dn * N + 2 * Dn)
    # recurrence: dt A, exp, dt B u, h, y per state; the backward replays it and adds dh,
    # the two sums over states and the terms of dA, dB and dC
    conv_f = (2 * s * E + 4 * T + 4 * Dn * (W + 1), (2 * W + 5) * E)
    conv_b = (3 * s * E + 4 * T + 8 * Dn * (W + 1), (6 * W + 12) * E)
    scan_f = (4 * s * E + T * (2 * N * s + 4) + par, (7 * N + 20) * E)
    scan_b = (7 * s * E + T * (2 * N * s + 4 + 8 * N) + 2 * par, (22 * N + 30) * E)
    if kind == "conv":
        parts = [conv_f, conv_b]
    elif kind in ("prefill", "decode"):
        parts = [conv_f, scan_f, (2 * Nb * Dn * ((W - 1) * s + 4 * N), 0)]
    else:
        parts = [conv_f, scan_f, scan_b, conv_b]
        if case.get("states"):
            parts.append((4 * Nb * Dn * ((W - 1) * s + 4 * N), 0))
    if kind == "block":
        M, R = case["d_model"], case["rank"]
        weights = 2 * Dn * M + (R + 2 * N) * Dn + Dn * R + M * Dn
        X = T * M
        # the projections: each weight and activation once per product (forward, input
        # gradient, weight gradient)
        act = (X + 2 * E) + (E + T * (R + 2 * N)) + (T * R + E) + (E + 2 * X)
        parts.append((3 * s * (weights + act), 6 * T * weights))
        parts.append((6 * s * X + 8 * T + 12 * M, 14 * X))
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def tolerance(case):
    # The distance of the results from `exact` over the listed and drawn cases, times about
    # four.  32-bit results are up to 4.4e-7 off (sums over up to 2^17 tokens in some order).
    # bf16 results carry one rounding (1.7e-3 in the 2-norm, one ulp at most 2^-7 of a
    # value); in a block a rounding that falls the other way travels on (up to 2.3e-3).
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 1e-4}
    if case["kind"] == "block":
        return {"rel": 1e-2, "max": 0.2}
    return {"rel": 7e-3, "max": 0.03}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _conv64(x, w, bias, pos, x0=None):
    """(pre-activation, SiLU of it); x0: inputs before each row."""
    Wd, L = w.shape[1], x.shape[2]
    pad = x.new_zeros(*x.shape[:2], Wd - 1) if x0 is None else x0
    xp = torch.cat([pad, x], 2)
    pre = bias[None, :, None] + torch.zeros_like(x)
    for k in range(Wd):
        pre += (pos >= k).to(x.dtype)[:, None, :] * w[:, Wd - 1 - k][None, :, None] * xp[:, :, Wd - 1 - k:Wd - 1 - k + L]
    return pre, pre * torch.sigmoid(pre)


def _conv64_bwd(x, w, bias, pos, dout, x0=None, dxf=None):
    Wd, L = w.shape[1], x.shape[2]
    pre, _ = _conv64(x, w, bias, pos, x0)
    sg = torch.sigmoid(pre)
    g = dout * sg * (1 + pre * (1 - sg))
    pad = x.new_zeros(*x.shape[:2], Wd - 1) if x0 is None else x0
    xp = torch.cat([pad, x], 2)
    dxp = torch.zeros_like(xp)
    if dxf is not None:
        dxp[:, :, L:] += dxf
    dw = torch.zeros_like(w)
    for k in range(Wd):
        gk = (pos >= k).to(x.dtype)[:, None, :] * g
        at = slice(Wd - 1 - k, Wd - 1 - k + L)
        dxp[:, :, at] += gk * w[:, Wd - 1 - k][None, :, None]
        dw[:, Wd - 1 - k] = (gk * xp[:, :, at]).sum((0, 2))
    return dxp[:, :, Wd - 1:], dw, g.sum((0, 2)), dxp[:, :, :Wd - 1]


def _scan64(u, delta, A, B, C, D, z, dbias, pos, h0=None, dout=None, dhf=None):
    """(out, final state, gradients or None), one batch row at a time."""
    rows = []
    for b in range(u.shape[0]):
        rows.append(_scan64_row(u[b], delta[b], A, B[b], C[b], D, z[b], dbias, pos[b],
                                None if h0 is None else h0[b], None if dout is None else dout[b],
                                None if dhf is None else dhf[b]))
    out, hf = torch.stack([r[0] for r in rows]), torch.stack([r[1] for r in rows])
    if dout is None:
        return out, hf, None
    g = {}
    for k in rows[0][2]:
        v = torch.stack([r[2][k] for r in rows])
        g[k] = v.sum(0) if k in ("dA", "dD", "ddelta_bias") else v
    return out, hf, g


def _scan64_row(u, delta, A, B, C, D, z, dbias, pos, h0, dout, dhf):
    T = 256                                             # tokens per chunk of the loops
    u, z = u.t().contiguous(), z.t().contiguous()       # (L, dim): time first
    raw = delta.t().contiguous() + dbias
    L, Dn = u.shape
    dt = F.softplus(raw, threshold=60.0)
    B, C = B.t().contiguous()[:, None, :], C.t().contiguous()[:, None, :]       # (L, 1, N)
    alive = (pos != 0).to(u.dtype)[:, None, None]
    H = torch.empty(L, Dn, N, dtype=u.dtype, device=u.device)
    first = torch.zeros(Dn, N, dtype=u.dtype, device=u.device) if h0 is None else h0
    h = first
    y = torch.empty_like(u)
    for c in range(0, L, T):
        e = torch.exp(dt[c:c + T, :, None] * A) * alive[c:c + T]
        bx = (dt[c:c + T] * u[c:c + T])[:, :, None] * B[c:c + T]
        for t in range(e.shape[0]):
            h = torch.addcmul(bx[t], e[t], h, out=H[c + t])
        y[c:c + T] = (H[c:c + T] * C[c:c + T]).sum(-1)
    y += D * u
    sz = torch.sigmoid(z)
    out = (y * z * sz).t()
    if dout is None:
        return out, H[-1].clone(), None
    dout = dout.t().contiguous()
    g = dict(dz=(dout * y * sz * (1 + z * (1 - sz))).t())
    dy = dout * z * sz
    x = torch.zeros(Dn, N, dtype=u.dtype, device=u.device) if dhf is None else dhf.clone()
    dA = torch.zeros_like(A)
    du, dd = torch.empty_like(u), torch.empty_like(u)
    dB, dC = torch.empty(L, N, dtype=u.dtype, device=u.device), torch.empty(L, N, dtype=u.dtype, device=u.device)
    for c in reversed(range(0, L, T)):
        n = slice(c, min(c + T, L))
        e = torch.exp(dt[n, :, None] * A) * alive[n]
        G = dy[n, :, None] * C[n]
        for t in reversed(range(e.shape[0])):
            G[t].add_(x)
            torch.mul(e[t], G[t], out=x)
        before = first if c == 0 else H[c - 1]
        q = G * e * torch.cat([before[None], H[c:n.stop - 1]], 0)
        dA += (q * dt[n, :, None]).sum(0)
        gb = (G * B[n]).sum(-1)
        du[n] = dt[n] * gb + dy[n] * D
        dd[n] = (q * A).sum(-1) + u[n] * gb
        dB[n] = (G * (dt[n] * u[n])[:, :, None]).sum(1)
        dC[n] = (H[n] * dy[n, :, None]).sum(1)
    dd *= torch.sigmoid(raw)
    g.update(du=du.t(), ddelta=dd.t(), dA=dA, dB=dB.t(), dC=dC.t(), dD=(dy * u).sum(0), ddelta_bias=dd.sum(0))
    if h0 is not None:
        g["dinitial_state"] = x
    return out, H[-1].clone(), g


def exact(case, seed):
    """Intermediates that are stored between two calls are rounded to their type there, as
    in `run`; everything else stays in 64 bits."""
    s = prepare(case, seed)
    kind, dt = case["kind"], DTYPES[case["dtype"]]
    d = {k: v.double() for k, v in s.items() if torch.is_tensor(v) and v.is_floating_point()}
    pos = s.get("pos")
    stored = lambda v: v.to(dt).double()  # noqa: E731
    if kind == "norm":
        x, w, g = d["x"], d["w"][None, :, None], d["dout"]
        r = torch.rsqrt((x * x).mean(1, keepdim=True) + 1e-5)
        dot = (g * w * x).sum(1, keepdim=True)
        dx = r * (g * w - x * r * r * dot / x.shape[1]) + d["dres"]
        return dict(out=x * r * w, rstd=r[:, 0], dx=dx, dw=(g * x * r).sum((0, 2)))
    if kind == "block":
        return _block64(d["x"], pos, {k: v.double() for k, v in s["p"].items()}, d["dout"], stored)
    if kind == "conv":
        u = _conv64(d["x"], d["w"], d["bias"], pos)[1]
        dx, dw, db, _ = _conv64_bwd(d["x"], d["w"], d["bias"], pos, d["dout"])
        return dict(u=u, dx=dx, dw=dw, db=db)
    u = _conv64(d["x"], d["w"], d["bias"], pos, d.get("x0"))[1]
    r = dict(u=u)
    if "x0" in d:
        W1 = case["width"] - 1
        r["xf"] = torch.cat([d["x0"], d["x"]], 2)[:, :, -W1:]
    us = stored(u)
    out, hf, g = _scan64(us, d["delta"], d["A"], d["B"], d["C"], d["D"], d["z"], d["dbias"], pos, d.get("h0"),
                         d.get("dout"), d.get("dhf"))
    r["y"] = out
    if "h0" in d:
        r["hf"] = hf
    if kind == "train":
        r.update(g)
        dx, dw, db, dx0 = _conv64_bwd(d["x"], d["w"], d["bias"], pos, stored(g["du"]), d.get("x0"), d.get("dxf"))
        r.update(dx=dx, dw=dw, db=db)
        if "x0" in d:
            r["dx0"] = dx0
    return r


def _block64(x, pos, p, dout, stored):
    Dn, R = p["D"].shape[0], p["W_dt"].shape[1]
    w = p["norm_w"][None, :, None]
    r = torch.rsqrt((x * x).mean(1, keepdim=True) + BK.EPS)
    h = stored(x * r * w)
    xz = stored(torch.matmul(p["W_in"], h))
    xi, z = xz[:, :Dn], xz[:, Dn:]
    u = stored(_conv64(xi, p["conv_w"], p["conv_b"], pos)[1])
    xdbl = stored(torch.matmul(p["W_x"], u))
    dtl, B, C = xdbl[:, :R], xdbl[:, R:R + N], xdbl[:, R + N:]
    delta = stored(torch.matmul(p["W_dt"], dtl))
    dy = stored(torch.matmul(p["W_out"].t(), dout))
    y, _, s = _scan64(u, delta, p["A"], B, C, p["D"], z, p["dt_bias"], pos, dout=dy)
    y = stored(y)
    out = x + torch.matmul(p["W_out"], y)

    def dw(d_out, a):
        return torch.stack([d_out[b] @ a[b].t() for b in range(a.shape[0])]).sum(0)

    dd, dz = stored(s["ddelta"]), stored(s["dz"])
    dxdbl = torch.cat([stored(torch.matmul(p["W_dt"].t(), dd)), stored(s["dB"]), stored(s["dC"])], 1)
    du = stored(stored(s["du"]) + torch.matmul(p["W_x"].t(), dxdbl))
    dxi, dcw, dcb, _ = _conv64_bwd(xi, p["conv_w"], p["conv_b"], pos, du)
    dxz = torch.cat([stored(dxi), dz], 1)
    dh = stored(torch.matmul(p["W_in"].t(), dxz))
    dot = (dh * w * x).sum(1, keepdim=True)
    return dict(out=out, dx=r * (dh * w - x * r * r * dot / x.shape[1]) + dout, dnorm_w=(dh * x * r).sum((0, 2)),
                dW_in=dw(dxz, h), dconv_w=dcw, dconv_b=dcb, dW_x=dw(dxdbl, u), dW_dt=dw(dd, dtl),
                ddt_bias=s["ddelta_bias"], dA=s["dA"], dD=s["dD"], dW_out=dw(dout, y))
