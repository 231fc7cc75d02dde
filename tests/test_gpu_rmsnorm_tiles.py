"""GPU parity of RMSNorm around its launch rules: the forward's narrow and wide tiles (below and
from 256 tiles of 8 vectors) and its few-features form, the backward's one to eight blocks a tile,
features kept in registers and beyond them, tiles that cross the row end, partial rows around the
finalize's 32 row groups, and a workspace of exactly the reported size."""
import numpy as np
import pytest

from gpu_common import TOL, act, assert_close, f32, host, note

pytestmark = pytest.mark.gpu

# forward: 2048 features kept in narrow tiles, 1024 in wide ones (256 threads, up to 128 features
# or in narrow tiles: 256, 128; 512 threads, up to 512 features: all; 4 kept of each thread's,
# bf16 just over 256 tiles: 512).  Backward: 512 kept by one block, 1024 by two, ... 4096 by eight
SHAPES = [(1, 2047, 33), (1, 2049, 31), (1, 2049, 65), (2, 300, 1023), (3, 7, 16 * 33 + 1),
          (8, 511, 4096), (8, 513, 4089), (16, 1025, 2041), (512, 17, 9),
          (4, 256, 4096), (4, 257, 4101), (300, 130, 65), (2, 255, 70), (1, 129, 64),
          (1, 4097, 128), (2, 4095, 190), (1, 2049, 64 * 40), (1, 1025, 64 * 70 - 1), (2, 1024, 64 * 64),
          (1, 800, 64 * 129), (8, 300, 1000), (2, 520, 72), (20, 200, 830), (20, 128, 1000), (40, 256, 1024),
          (40, 129, 1024), (5, 512, 3392), (3, 512, 640), (9, 400, 2050), (17, 512, 1024), (17, 513, 1020), (5, 700, 4096),
          (3, 1025, 990), (10, 1025, 1024), (2, 2049, 4090), (6, 600, 1000), (4, 600, 1000), (4, 1024, 96)]


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


# one block a tile, and eight, four and two that share one; ragged rows.  dx in the place of x,
# dout or the residual's gradient, and the forward's output in the place of x
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(3, 130, 70), (1, 4097, 128), (2, 2049, 190), (1, 1025, 64 * 70 - 1), (1, 1024, 64 * 129),
                                   (64, 640, 4096 // 16)], ids=lambda s: "x".join(map(str, s)))
def test_rmsnorm_in_place(shape, dtype):
    import torch
    from paper_2408_03865_amd import _lib
    b, d, L = shape
    lib, code = _lib.load(), {"f32": 0, "bf16": 1}[dtype]
    rng = np.random.default_rng(b + d + L)
    x, g, res = (act(rng.standard_normal(shape, dtype=np.float32), dtype) for _ in range(3))
    w = f32(rng.uniform(0.5, 1.5, d))
    rs = torch.empty((b, L), device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    ws = torch.empty(lib.packmamba_rmsnorm_bwd_workspace_size(*shape), dtype=torch.uint8, device="cuda")
    note(f"rmsnorm in place {shape} {dtype}")

    def fwd(xi, out):
        assert lib.packmamba_rmsnorm_fwd(xi.data_ptr(), w.data_ptr(), 1e-5, out.data_ptr(), rs.data_ptr(), *shape, code, stream) == 0
        return out

    def bwd(xi, gi, ri, dx):
        dw = torch.empty_like(w)
        assert lib.packmamba_rmsnorm_bwd(xi.data_ptr(), w.data_ptr(), rs.data_ptr(), gi.data_ptr(), ri.data_ptr(), dx.data_ptr(),
                                         dw.data_ptr(), ws.data_ptr(), ws.numel(), *shape, code, stream) == 0
        return dx, dw

    def same(got, want):
        # several blocks of a tile take its features in another order than one: fp32 sums within their
        # rounding, so that a bf16 result is at most one rounding (2^-7 of it) off
        assert_close("in place", host(got), host(want), TOL["f32"] if dtype == "f32" else 2.0 ** -7)

    out = fwd(x, torch.empty_like(x))
    xi = x.clone()
    assert torch.equal(fwd(xi, xi), out)
    dx, dw = bwd(x, g, res, torch.empty_like(x))
    for i in range(3):
        t = [x, g, res]
        t[i] = t[i].clone()
        dx2, dw2 = bwd(*t, t[i])
        same(dx2, dx)
        same(dw2, dw)
