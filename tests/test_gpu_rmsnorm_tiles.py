"""GPU parity of RMSNorm around its launch rules: narrow and wide tiles (below and from 512 tiles
of 8 vectors), features kept in registers and beyond them, tiles that cross the row end, and
partial rows around the finalize's 32 row groups."""
import numpy as np
import pytest

from gpu_common import TOL, act, assert_close, f32, host, note

pytestmark = pytest.mark.gpu

# narrow: 4 vectors a row, 256 slices, 8 kept: 2048 features; wide: 8 vectors, 128 or 64
# slices: 1024 and 512 kept features
SHAPES = [(1, 2047, 33), (1, 2049, 31), (2, 300, 1023), (3, 7, 16 * 33 + 1),
          (8, 511, 4096), (8, 513, 4089), (16, 1025, 2041), (512, 17, 9)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_rmsnorm_tiles(shape, dtype):
    import paper_2408_03865_amd as P
    import torch
    b, d, L = shape
    rng = np.random.default_rng(b + d + L)
    x, g, res = (act(rng.standard_normal(shape, dtype=np.float32), dtype) for _ in range(3))
    w = f32(rng.uniform(0.5, 1.5, d))
    note(f"rmsnorm tiles {shape} {dtype}")
    out32 = dtype == "bf16"
    o, rs = P.rmsnorm_fwd(x, w, out_f32=out32)
    dx, dw = P.rmsnorm_bwd(x, w, rs, g, dresidual=res, out_f32=out32)
    x, g, res, w = x.double(), g.double(), res.double(), w.double()[None, :, None]
    r = torch.rsqrt((x * x).mean(1, keepdim=True) + 1e-5)
    dot = (g * w * x).sum(1, keepdim=True)
    assert_close("rstd", host(rs), host(r[:, 0]), TOL["f32"])
    assert_close("out", host(o), host(x * r * w), TOL["f32"])
    assert_close("dx", host(dx), host(r * (g * w - x * r * r * dot / d) + res), TOL["f32"])
    assert_close("dw", host(dw), host((g * x * r).sum((0, 2))), TOL["f32"])
