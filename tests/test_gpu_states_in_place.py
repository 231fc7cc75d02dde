"""GPU: states updated in place, as a serving loop does: the final states written into the
initial states' buffer, and the initial states' gradient into the final states', give the bits
that separate buffers give.  Rows of one segment and of several (whose blocks all start from the
row's state), and short rows."""
import numpy as np
import pytest

import workloads as W
from gpu_common import act, f32, i32, note

pytestmark = pytest.mark.gpu

# (batch, dim, seqlen): tokens of the short-row kernel, one chunk, unsplit, 4 and 9 segments
SHAPES = [(3, 70, 2), (2, 40, 200), (30, 241, 513), (2, 48, 1000), (1, 16, 2100)]


def _same(a, b):
    import torch
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_states_in_place(shape, dtype):
    import torch
    from paper_2408_03865_amd import _lib
    batch, dim, L = shape
    lib, code = _lib.load(), {"f32": 0, "bf16": 1}[dtype]
    cfg = W.Config("inplace", "inplace", batch, L, dim, 16, 4, dtype, ("lognormal", 4.0, 1.0, 1, L), 5100 + batch + dim + L)
    d = W.make_inputs(cfg, variant="general")
    pos = d["pos"].copy()
    for b in range(batch):                                 # every other row is one sequence, continued throughout
        if b % 2 == 0:
            pos[b] = np.arange(L) + 7
    rng = np.random.default_rng(L)
    h0, dhf = (f32(rng.standard_normal((batch, dim, 16)).astype(np.float32)) for _ in range(2))
    note(f"in place {shape} {dtype}")
    g = {k: act(d[k], dtype) for k in ("u", "delta", "B", "C", "z", "dout")}
    g.update({k: f32(d[k]) for k in ("A", "D", "delta_bias")})
    p = i32(pos)
    sizes = (batch, dim, L, 16)

    def ws(n):
        return torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")

    def fwd(hi, hf, states):
        out = torch.empty_like(g["u"])
        w = ws(lib.packmamba_selective_scan_fwd_workspace_size(*sizes))
        st = ws(lib.packmamba_selective_scan_fwd_saved_states_size(*sizes)) if states else None
        e = lib.packmamba_selective_scan_fwd(
            *(g[k].data_ptr() for k in ("u", "delta", "A", "B", "C", "D", "z", "delta_bias")), 1, p.data_ptr(),
            hi.data_ptr(), out.data_ptr(), hf.data_ptr(), st.data_ptr() if states else None, w.data_ptr(), w.numel(),
            *sizes, code, torch.cuda.current_stream().cuda_stream)
        assert e == 0
        return out, st

    def bwd(hi, dhfin, dh0, st):
        r = {k: torch.empty_like(g[k[1:]]) for k in ("du", "ddelta", "dA", "dD", "dz", "ddelta_bias")}
        r.update({k: torch.empty((batch, 16, L), device="cuda") for k in ("dB", "dC")})
        w = ws(lib.packmamba_selective_scan_bwd_workspace_size(*sizes))
        e = lib.packmamba_selective_scan_bwd(
            *(g[k].data_ptr() for k in ("u", "delta", "A", "B", "C", "D", "z", "delta_bias")), 1, p.data_ptr(),
            hi.data_ptr(), g["dout"].data_ptr(), dhfin.data_ptr(), st.data_ptr() if st is not None else None,
            *(r[k].data_ptr() for k in ("du", "ddelta", "dA", "dB", "dC", "dD", "dz", "ddelta_bias")), dh0.data_ptr(),
            w.data_ptr(), w.numel(), *sizes, code, torch.cuda.current_stream().cuda_stream)
        assert e == 0
        return r

    st = None
    for states in (False, True):
        hf, io = torch.empty_like(h0), h0.clone()
        out, st = fwd(h0, hf, states)
        out2, _ = fwd(io, io, states)
        assert torch.equal(out, out2) and _same(hf, io)
        # a recomputing backward (no saved states) passes through both aggregate passes
        dh0, dio = torch.empty_like(h0), dhf.clone()
        r, r2 = bwd(h0, dhf, dh0, st), bwd(h0, dio, dio, st)
        for k in r:
            assert torch.equal(r[k], r2[k]), k
        assert _same(dh0, dio)
