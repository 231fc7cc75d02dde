"""GPU parity of the paths whose launch depends on the row length: the scan forward's short-row
kernel (no saved states, up to 20 to 32 tokens by the number of channels) on both sides of its
limits, and the conv forward's
lanes per row, tiles per row and rows per lane, against the oracle."""
import numpy as np
import pytest

import workloads as W
from gpu_common import TOL, act, assert_close, bf16_bits_of, f32, host, i32, note, rne_bf16

pytestmark = pytest.mark.gpu


def _cfg(batch, dim, seqlen, width, dtype):
    return W.Config("short", "short", batch, seqlen, dim, 16, width, dtype, ("lognormal", 1.5, 1.0, 1, max(seqlen, 1)),
                    8800 + batch * 13 + dim * 3 + seqlen)


# tokens: one vector and less, and around the most that the short kernel ever takes; channels:
# one, a block of 64 and one on either side
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("states", [False, True], ids=["fresh", "continued"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 65, 1), (2, 64, 2), (2, 63, 7), (1, 130, 31), (2, 40, 32), (2, 40, 33)],
                         ids=lambda s: "x".join(map(str, s)))
def test_scan_forward_short_rows(shape, states, dtype):
    import oracle as O
    import paper_2408_03865_amd as P
    batch, dim, L = shape
    d = W.make_inputs(_cfg(batch, dim, L, 4, dtype), variant="general")
    pos, h0 = d["pos"].copy(), None
    if states:
        first = np.argmax(np.concatenate([pos[:, 1:] == 0, np.ones((batch, 1), bool)], 1), 1) + 1
        for b in range(batch):
            pos[b, :first[b]] += 5
        h0 = np.random.default_rng(L).standard_normal((batch, dim, 16)).astype(np.float32)
    note(f"short scan {shape} {dtype} states={states}")
    g = {k: act(d[k], dtype) for k in ("u", "delta", "B", "C", "z")}
    par = {k: f32(d[k]) for k in ("A", "D", "delta_bias")}
    for opts in (dict(D=True, z=True, bias=True, softplus=True), dict(D=False, z=False, bias=False, softplus=False)):
        got, fin = P.selective_scan_fwd(g["u"], g["delta"], par["A"], g["B"], g["C"], par["D"] if opts["D"] else None,
                                        g["z"] if opts["z"] else None, par["delta_bias"] if opts["bias"] else None,
                                        opts["softplus"], i32(pos), out_f32=dtype == "bf16", initial_state=f32(h0),
                                        return_final=True)
        ref, rfin = O.scan_fwd(u=d["u"], delta=d["delta"], A=d["A"], B=d["B"], C=d["C"],
                               D=d["D"] if opts["D"] else None, z=d["z"] if opts["z"] else None,
                               delta_bias=d["delta_bias"] if opts["bias"] else None, delta_softplus=opts["softplus"],
                               pos=pos, h0=h0, return_final=True)
        assert_close("out", host(got), ref, TOL["f32"])        # same inputs and fp32 arithmetic for both types
        assert_close("final", host(fin), rfin, TOL["f32"])


# the short kernel's limits and one token beyond: 20 tokens below 128 blocks of 16 channels, 24
# below 384, 32 from there, in fp32 28 from 8192 blocks.  The bf16 output is the fp32 one, rounded
# once.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(2, 40, 3), (2, 40, 20), (2, 40, 21), (16, 127, 24), (16, 127, 25), (48, 120, 32),
                                   (48, 120, 33), (127, 1030, 28), (127, 1030, 29)], ids=lambda s: "x".join(map(str, s)))
def test_scan_forward_short_row_limits(shape, dtype):
    import oracle as O
    import paper_2408_03865_amd as P
    batch, dim, L = shape
    d = W.make_inputs(_cfg(batch, dim, L, 4, dtype), variant="general")
    h0 = np.random.default_rng(L).standard_normal((batch, dim, 16)).astype(np.float32)
    pos = d["pos"].copy()
    pos[::2] = np.arange(L) + 5                              # every other row continues a sequence throughout
    note(f"short scan limits {shape} {dtype}")
    for softplus in (True, False):
        delta = d["delta"] if softplus else np.abs(d["delta"])
        g = {k: act(d[k], dtype) for k in ("u", "B", "C", "z")}
        a = (g["u"], act(delta, dtype), f32(d["A"]), g["B"], g["C"], f32(d["D"]), g["z"], f32(d["delta_bias"]) if softplus else None,
             softplus, i32(pos))
        got, fin = P.selective_scan_fwd(*a, out_f32=dtype == "bf16", initial_state=f32(h0), return_final=True)
        ref, rfin = O.scan_fwd(u=d["u"], delta=delta, A=d["A"], B=d["B"], C=d["C"], D=d["D"], z=d["z"],
                               delta_bias=d["delta_bias"] if softplus else None, delta_softplus=softplus, pos=pos, h0=h0,
                               return_final=True)
        assert_close("out", host(got), ref, TOL["f32"])        # same inputs and fp32 arithmetic for both types
        assert_close("final", host(fin), rfin, TOL["f32"])
        if dtype == "bf16":
            b16, fin16 = P.selective_scan_fwd(*a, initial_state=f32(h0), return_final=True)
            assert np.array_equal(bf16_bits_of(b16), rne_bf16(got)) and np.array_equal(host(fin16), host(fin))


# tokens around one lane's vector (4 and 8), around the powers of two of lanes per row, a wave's
# span (256 and 512) and more tiles; channels that leave a wave's rows ragged.  The last shapes
# have enough rows for several per lane: 64 rows a wave, and one row in two tiles.
CONV_SHAPES = [(1, 1, 1), (2, 70, 2), (3, 33, 5), (2, 5, 8), (2, 17, 9), (1, 9, 31), (2, 3, 255), (1, 6, 257),
               (2, 3, 512), (1, 5, 513), (1, 2, 1541), (64, 33000, 1), (130, 131, 513)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("width", [2, 3, 4])
@pytest.mark.parametrize("shape", CONV_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_conv_forward_lanes_and_tiles(shape, width, dtype):
    if shape[0] * shape[1] * shape[2] > 1 << 20 and width != 4:
        pytest.skip("the large shapes run at one width")
    _conv_forward(shape, width, dtype)


# bf16 rows that a block each walks (aligned, 2049 to 32767 tokens, 768 rows), and each limit
# missed: one row fewer, 2048 tokens, unaligned
@pytest.mark.parametrize("shape", [(1, 768, 2056), (4, 257, 4104), (1, 767, 2056), (2, 520, 2048), (1, 1024, 2060)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("width", [2, 3, 4])
def test_conv_forward_by_row(shape, width):
    _conv_forward(shape, width, "bf16")


def _conv_forward(shape, width, dtype):
    import oracle as O
    import paper_2408_03865_amd as P
    batch, dim, L = shape
    rng = np.random.default_rng(batch + dim + L + width)
    rnd = W.bf16_round if dtype == "bf16" else (lambda a: a)
    x = rnd(rng.standard_normal((batch, dim, L)).astype(np.float32))
    xi = rnd(rng.standard_normal((batch, dim, width - 1)).astype(np.float32))
    w = rng.uniform(-0.5, 0.5, (dim, width)).astype(np.float32)
    bias = rng.uniform(-0.5, 0.5, dim).astype(np.float32)
    pos = W.positions_from_lengths(W.draw_row_lengths(("lognormal", 4.0, 2.0, 1, L), rng, batch, L), L)
    first = np.argmax(np.concatenate([pos[:, 1:] == 0, np.ones((batch, 1), bool)], 1), 1) + 1
    for b in range(0, batch, 2):                       # every other row continues a sequence
        pos[b, :first[b]] += 1 + b % 4
    note(f"conv {shape} W={width} {dtype}")
    got, fin = P.causal_conv1d_fwd(act(x, dtype), f32(w), f32(bias), i32(pos), out_f32=dtype == "bf16",
                                   initial_x=act(xi, dtype), return_final=True)
    ref, rfin = O.conv1d_fwd(x, w, bias, pos, xinit=xi, return_final=True)
    assert_close("out", host(got), ref, TOL["f32"])
    assert np.array_equal(host(fin), np.asarray(rfin, dtype=np.float64))
    plain = P.causal_conv1d_fwd(act(x, dtype), f32(w), None, i32(pos), silu=False, out_f32=dtype == "bf16")
    assert_close("plain", host(plain), O.conv1d_fwd(x, w, None, pos, silu=False), TOL["f32"])


# (batch, channels, tokens): waves per channel.  One block gathers up to 4, 8 or 16 within 8192
# waves in all, 5 to 7 within 6144 and others up to 16 within 4096, both with 2^22 elements at most:
# both sides of each limit
GATHERED = {(1, 3, 70): 1, (3, 5, 1030): 9, (4, 6, 2048): 16, (4, 6, 2049): 20, (17, 4, 30): 17, (4, 1100, 70): 4,
            (6, 1024, 100): 6, (6, 1025, 100): 6, (6, 700, 990): 6, (6, 700, 1000): 6, (8, 1024, 70): 8, (8, 1025, 70): 8,
            (12, 512, 64): 12, (12, 341, 64): 12, (13, 315, 64): 13, (13, 316, 64): 13, (16, 512, 30): 16, (16, 513, 30): 16,
            (1, 600, 3500): 7, (4, 4100, 2050): 4}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("states", [False, True], ids=["fresh", "continued"])
@pytest.mark.parametrize("shape", GATHERED, ids=lambda s: "x".join(map(str, s)))
def test_conv_backward_gathered_waves(shape, states, dtype):
    import oracle as O
    import paper_2408_03865_amd as P
    batch, dim, L = shape
    if states and batch * dim * L > 1 << 22:
        pytest.skip("the large shapes run without states")
    need = P.load().packmamba_causal_conv1d_bwd_workspace_size(batch, dim, L, 4)
    assert need == -(-GATHERED[shape] * dim * 5 * 4 // 256) * 256      # a partial per wave, channel and sum
    rng = np.random.default_rng(batch * 7 + dim + L)
    rnd = W.bf16_round if dtype == "bf16" else (lambda a: a)
    x, g = (rnd(rng.standard_normal((batch, dim, L)).astype(np.float32)) for _ in range(2))
    xi, dxf = (rnd(rng.standard_normal((batch, dim, 3)).astype(np.float32)) for _ in range(2))
    w = rng.uniform(-0.5, 0.5, (dim, 4)).astype(np.float32)
    bias = rng.uniform(-0.5, 0.5, dim).astype(np.float32)
    pos = W.positions_from_lengths(W.draw_row_lengths(("lognormal", 4.0, 1.0, 1, L), rng, batch, L), L)
    if states:                                             # every row continues a sequence
        first = np.argmax(np.concatenate([pos[:, 1:] == 0, np.ones((batch, 1), bool)], 1), 1) + 1
        for b in range(batch):
            pos[b, :first[b]] += 1 + b % 4
    note(f"conv bwd {shape} {dtype} states={states}")
    kw = dict(initial_x=act(xi, dtype), dfinal_x=act(dxf, dtype)) if states else {}
    got = P.causal_conv1d_bwd(act(x, dtype), f32(w), f32(bias), i32(pos), act(g, dtype), out_f32=dtype == "bf16", **kw)
    ref = O.conv1d_bwd(x, w, bias, pos, g, **(dict(xinit=xi, dxfinal=dxf) if states else {}))
    for k, v in zip(("dx", "dw", "dbias", "dxinit"), got):
        assert_close(k, host(v), ref[k], TOL["f32"])
