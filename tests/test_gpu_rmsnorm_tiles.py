"""GPU parity of RMSNorm around its launch rules: the forward's narrow and wide tiles (below and
from 256 tiles of 8 vectors) and its few-features form, the backward's one to eight blocks a tile,
features kept in registers and beyond them, tiles that cross the row end, partial rows around the
finalize's 32 row groups, and a workspace of exactly the reported size."""
import numpy as np
import pytest

from gpu_common import TOL, act, assert_close, f32, host, note

pytestmark = pytest.mark.gpu

# forward: 2048 features kept in narrow tiles, 1024 in wide ones (256 threads, up to 256
# features: 256, 128).  Backward: 512 kept by one block, 1024 by two, ... 4096 by eight
SHAPES = [(1, 2047, 33), (1, 2049, 31), (1, 2049, 65), (2, 300, 1023), (3, 7, 16 * 33 + 1),
          (8, 511, 4096), (8, 513, 4089), (16, 1025, 2041), (512, 17, 9),
          (4, 256, 4096), (4, 257, 4101), (300, 130, 65), (2, 255, 70), (1, 129, 64),
          (1, 4097, 128), (2, 4095, 190), (1, 2049, 64 * 40), (1, 1025, 64 * 70 - 1), (2, 1024, 64 * 64),
          (1, 800, 64 * 129), (8, 300, 1000), (2, 520, 72)]


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
    need = P.load().packmamba_rmsnorm_bwd_workspace_size(*shape)
    buf = torch.full((need + 4096,), 0x5a, dtype=torch.uint8, device="cuda")
    dx, dw = P.rmsnorm_bwd(x, w, rs, g, dresidual=res, out_f32=out32, workspace=buf[:need])
    assert bool((buf[need:] == 0x5a).all())
    x, g, res, w = x.double(), g.double(), res.double(), w.double()[None, :, None]
    r = torch.rsqrt((x * x).mean(1, keepdim=True) + 1e-5)
    dot = (g * w * x).sum(1, keepdim=True)
    assert_close("rstd", host(rs), host(r[:, 0]), TOL["f32"])
    assert_close("out", host(o), host(x * r * w), TOL["f32"])
    assert_close("dx", host(dx), host(r * (g * w - x * r * r * dot / d) + res), TOL["f32"])
    assert_close("dw", host(dw), host((g * x * r).sum((0, 2))), TOL["f32"])
