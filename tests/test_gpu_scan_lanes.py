"""GPU parity of the scan forward in each of its launch shapes (16, 32 or 64 lanes per channel,
the fp32 forward 16 instead of 32 above 256 blocks or segments of 16 channels; rows split or
not) at ragged lengths around the 256-token chunk: outputs, final states, the chunk states,
and, through the backward, the dz factor, whose order in memory is the same for every number
of lanes."""
import numpy as np
import pytest

import workloads as W
from gpu_common import TOL, act, assert_close, f32, host, i32, note

pytestmark = pytest.mark.gpu

# (batch, dim, seqlen): segments
SHAPES = {
    "64 lanes": [(1, 5, 130), (1, 3, 255), (2, 33, 256), (1, 4, 257), (1, 64, 700)],
    "32 lanes split": [(2, 300, 1300), (1, 500, 1537), (4, 256, 1000)],
    "32 lanes unsplit": [(16, 250, 300), (20, 247, 511), (24, 256, 77), (13, 250, 1536), (24, 256, 1600)],
    "bf16: 32 lanes split, fp32: 16": [(3, 512, 1000), (5, 96, 2300)],
    "16 lanes split": [(5, 170, 1700), (1, 1600, 2049), (13, 250, 1537), (16, 256, 1700)],
    "16 lanes unsplit": [(28, 256, 270), (30, 241, 513), (25, 254, 1025)],
    "bf16: 32 lanes unsplit, fp32: 16 lanes split": [(17, 250, 2048), (18, 249, 1601)],
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [s for v in SHAPES.values() for s in v], ids=lambda s: "x".join(map(str, s)))
def test_scan_forward_lanes(shape, dtype):
    import oracle as O
    import paper_2408_03865_amd as P
    batch, dim, L = shape
    cfg = W.Config("lanes", "lanes", batch, L, dim, 16, 4, dtype, ("lognormal", 4.5, 1.0, 1, L), 6600 + batch + dim + L)
    d = W.make_inputs(cfg, variant="general")
    h0 = np.random.default_rng(L).standard_normal((batch, dim, 16)).astype(np.float32)
    pos = d["pos"].copy()
    first = np.argmax(np.concatenate([pos[:, 1:] == 0, np.ones((batch, 1), bool)], 1), 1) + 1
    for b in range(batch):
        pos[b, :first[b]] += 9                      # every row continues a sequence
    note(f"lanes {shape} {dtype} segments fwd={P.segments(*shape, 'fwd')}")
    g = {k: act(d[k], dtype) for k in ("u", "delta", "B", "C", "z", "dout")}
    a = (g["u"], g["delta"], f32(d["A"]), g["B"], g["C"], f32(d["D"]), g["z"], f32(d["delta_bias"]), True, i32(pos))
    kw = dict(out_f32=dtype == "bf16", initial_state=f32(h0))
    out, st, fin = P.selective_scan_fwd(*a, return_states=True, return_final=True, **kw)
    out2, fin2 = P.selective_scan_fwd(*a, return_final=True, **kw)
    gr = P.selective_scan_bwd(*a, g["dout"], saved_states=st, **kw)
    args = dict(u=d["u"], delta=d["delta"], A=d["A"], B=d["B"], C=d["C"], D=d["D"], z=d["z"],
                delta_bias=d["delta_bias"], delta_softplus=True, pos=pos)
    ref, rfin = O.scan_fwd(**args, h0=h0, return_final=True)
    rg = O.scan_bwd(**args, dout=d["dout"], h0=h0)
    tol = TOL["f32"]                                # same inputs and fp32 arithmetic for both types
    assert_close("out", host(out), ref, tol)
    assert_close("final", host(fin), rfin, tol)
    assert np.array_equal(host(out), host(out2)) and np.array_equal(host(fin), host(fin2))
    last = host(P.chunk_states(st, batch, dim, L))[:, :, -1]
    assert np.array_equal(last, host(fin))          # the last chunk's state is the final state
    for k in ("dz", "du", "ddelta", "dB", "dC"):
        assert_close(k, host(gr[k]), rg[k], tol)
