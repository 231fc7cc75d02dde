"""GPU parity of rows cut into many segments, whose maps every block chains by itself in runs of
eight: segment counts around those runs, in both directions, with initial and final states, in
both types, without a reset and with sequence starts inside some of the segments."""
import numpy as np
import pytest

import workloads as W
from gpu_common import TOL, act, assert_close, f32, host, i32, note

pytestmark = pytest.mark.gpu


# one sequence per row, slow decay: every map matters.  dim 16 gives as many segments as
# the row has 256-token units: 7, 8, 9, 17 (the last one token long).  `starts`: sequences begin
# at a segment's first and last token and inside one, so that some maps pass nothing on
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("starts", [False, True], ids=["whole", "starts"])
@pytest.mark.parametrize("L", [1790, 2048, 2100, 4097])
def test_segment_chains(L, starts, dtype):
    import oracle as O
    import paper_2408_03865_amd as P
    batch, dim = 2, 16
    assert P.segments(batch, dim, L, "fwd") == P.segments(batch, dim, L, "bwd") == (L + 255) // 256
    cfg = W.Config("chain", "chain", batch, L, dim, 16, 4, dtype, ("arange",), 7700 + L)
    d = W.make_inputs(cfg, variant="general")
    A = d["A"] * np.float32(0.02)
    rng = np.random.default_rng(L)
    h0, dhf = (rng.standard_normal((batch, dim, 16)).astype(np.float32) for _ in range(2))
    pos = d["pos"] + 3                                  # the rows continue sequences: no reset at all
    if starts:
        for b, at in enumerate([(256, 1023, 1400), (511,)]):
            for t in at:
                pos[b, t:] = np.arange(L - t)
    note(f"chain L={L} {dtype} starts={starts}")
    g = {k: act(d[k], dtype) for k in ("u", "delta", "B", "C", "z", "dout")}
    a = (g["u"], g["delta"], f32(A), g["B"], g["C"], f32(d["D"]), g["z"], f32(d["delta_bias"]), True, i32(pos))
    kw = dict(out_f32=dtype == "bf16", initial_state=f32(h0))         # same inputs and fp32 arithmetic for both types
    y, st, fin = P.selective_scan_fwd(*a, return_states=True, return_final=True, **kw)
    gr = P.selective_scan_bwd(*a, g["dout"], saved_states=st, dfinal_state=f32(dhf), **kw)
    args = dict(u=d["u"], delta=d["delta"], A=A, B=d["B"], C=d["C"], D=d["D"], z=d["z"], delta_bias=d["delta_bias"],
                delta_softplus=True, pos=pos)
    ry, rfin = O.scan_fwd(**args, h0=h0, return_final=True)
    ref = O.scan_bwd(**args, dout=d["dout"], h0=h0, dhfinal=dhf)
    # sums of up to L terms of either sign: an ulp of the largest value stands beside the bound
    for k, got, want in [("out", y, ry), ("final", fin, rfin), ("du", gr["du"], ref["du"]), ("ddelta", gr["ddelta"], ref["ddelta"]),
                         ("dA", gr["dA"], ref["dA"]), ("dB", gr["dB"], ref["dB"]), ("dC", gr["dC"], ref["dC"]),
                         ("dh0", gr["dinitial_state"], ref["dh0"])]:
        want = np.asarray(want, dtype=np.float64)
        floor = 16 * 2.0 ** -24 * np.max(np.abs(want))
        err = np.abs(host(got) - want)
        assert np.all(err <= TOL["f32"] * (1 + np.abs(want)) + floor), f"{k}: {err.max():.3e}"
