"""GPU: an infinity or a NaN stays where it belongs.  In the conv a tap of another sequence is
left out, not multiplied by 0; in the scan nothing passes to other channels, batch rows or, in
the forward, earlier tokens, and, in the backward, later ones.  Everything outside its reach has
the bits that it has without it, in each launch shape of the kernels."""
import numpy as np
import pytest

import workloads as W
from gpu_common import act, f32, i32, note

pytestmark = pytest.mark.gpu

BAD = [np.inf, -np.inf, np.nan]


def _same(a, b):
    import torch
    return torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8))


# rows within a wave's span, tiles of one and several channels a wave, a block per row (bf16)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(2, 70, 3), (3, 40, 200), (2, 9, 1300), (64, 520, 640), (1, 1024, 2056)],
                         ids=lambda s: "x".join(map(str, s)))
def test_conv_forward_masks_select(shape, dtype):
    import torch
    import paper_2408_03865_amd as P
    batch, dim, L = shape
    rng = np.random.default_rng(batch + dim + L)
    pos = W.positions_from_lengths(W.draw_row_lengths(("lognormal", 3.0, 1.0, 1, L), rng, batch, L), L)
    seq = np.cumsum(pos == 0, 1)
    x = act(rng.standard_normal(shape).astype(np.float32), dtype)
    w, bias = f32(rng.uniform(0.1, 0.5, (dim, 4)).astype(np.float32)), f32(np.zeros(dim, np.float32))
    p = i32(pos)
    note(f"conv nonfinite {shape} {dtype}")
    for silu in (True, False):
        clean = P.causal_conv1d_fwd(x, w, bias, p, silu=silu)
        for i, bad in enumerate(BAD):
            odd = torch.from_numpy((seq % 2 == i % 2)[:, None, :]).cuda()        # every other sequence is bad
            got = P.causal_conv1d_fwd(torch.where(odd, torch.full_like(x, bad), x), w, bias, p, silu=silu)
            keep = (~odd).expand(shape)
            assert _same(got[keep], clean[keep])
            assert not bool(torch.isfinite(got[odd.expand(shape)]).any())        # (SiLU of -inf: -inf times 0)


# short rows, 64, 32 and 16 lanes a channel, split rows, 16 lanes unsplit
SCAN = [(2, 40, 7), (1, 5, 300), (2, 300, 1300), (16, 250, 300), (1, 1600, 2049), (28, 256, 270)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SCAN, ids=lambda s: "x".join(map(str, s)))
def test_scan_reach(shape, dtype):
    import torch
    import paper_2408_03865_amd as P
    batch, dim, L = shape
    cfg = W.Config("bad", "bad", batch, L, dim, 16, 4, dtype, ("lognormal", 4.0, 1.0, 1, L), 900 + batch + dim + L)
    d = W.make_inputs(cfg, variant="general")
    g = {k: act(d[k], dtype) for k in ("u", "delta", "B", "C", "z", "dout")}
    par = [f32(d[k]) for k in ("A", "D", "delta_bias")]
    p = i32(d["pos"])
    note(f"scan nonfinite {shape} {dtype}")

    def fwd(u):
        return P.selective_scan_fwd(u, g["delta"], par[0], g["B"], g["C"], par[1], g["z"], par[2], True, p, return_final=True)

    def bwd(dout):
        _, st = P.selective_scan_fwd(g["u"], g["delta"], par[0], g["B"], g["C"], par[1], g["z"], par[2], True, p, return_states=True)
        return P.selective_scan_bwd(g["u"], g["delta"], par[0], g["B"], g["C"], par[1], g["z"], par[2], True, p, dout, saved_states=st)

    b, c, t = batch - 1, dim // 2, (2 * L) // 3                                # the bad token
    others = torch.ones(shape, dtype=torch.bool, device="cuda")
    others[b, c] = False
    before, after = others.clone(), others.clone()
    before[b, c, :t] = True
    after[b, c, t + 1:] = True
    out, fin = fwd(g["u"])
    ref = bwd(g["dout"])
    tok = torch.ones((batch, 16, L), dtype=torch.bool, device="cuda")
    tok[b, :, :t + 1] = False
    for bad in BAD:
        u = g["u"].clone()
        u[b, c, t] = bad
        out2, fin2 = fwd(u)
        assert _same(out2[before], out[before]) and not bool(torch.isfinite(out2[b, c, t]))
        assert _same(fin2[others[:, :, 0]], fin[others[:, :, 0]])
        dout = g["dout"].clone()
        dout[b, c, t] = bad
        r = bwd(dout)
        for k in ("du", "ddelta", "dz"):
            assert _same(r[k][after], ref[k][after]), k
        assert not bool(torch.isfinite(r["du"][b, c, t]))
        for k in ("dB", "dC"):
            assert _same(r[k][tok], ref[k][tok]), k
        rest = torch.arange(dim, device="cuda") != c
        for k in ("dA", "dD", "ddelta_bias"):
            assert _same(r[k][rest], ref[k][rest]), k
