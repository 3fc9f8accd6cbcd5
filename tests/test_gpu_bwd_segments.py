"""The backward's 64-row workgroups and its segments: every gradient against the
oracle where rows, tiles and segments end raggedly (D below, at and past a
wavefront's 16 rows and a workgroup's 64; one segment to many; odd L, whose
steps are read one by one, beside even L), gradients in bf16 against the fp32
ones rounded once, and a call repeated bit for bit."""
import numpy as np
import pytest

import oracle
from gate import assert_gate, fp_gate
from test_gpu_bwd import _bf16_dev, _check_all, _dev, _inputs, _ref, _run, sw  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

_ALL = ("z", "bias", "softplus", "h0", "dhl")
# (B, D, N, L): D at the edges of 16 and 64; L at the edges of a tile; long L
# on few rows takes many segments (a last one shorter than the others)
_SHAPES = [(1, 1, 16, 1), (2, 15, 16, 8), (1, 17, 16, 9), (1, 63, 16, 40), (2, 65, 16, 33),
           (1, 130, 16, 1000), (1, 64, 16, 2501), (2, 16, 13, 1026), (1, 20, 33, 515)]


@pytest.mark.parametrize("shape", _SHAPES)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("opts", [(), _ALL, ("dybf16", "h0", "dhl")])
def test_bwd_rows_and_segments(sw, shape, dtype, opts):  # noqa: F811
    B, D, N, L = shape
    print("case bwd segments", dtype, shape, opts, flush=True)
    inp, ex = _inputs(B, D, N, L, 2200 + B + D + N + L, dtype, opts)
    g = _run(sw, inp, ex, dtype, opts)
    if L > 1000 and N <= 16:
        assert "segments)" in sw.last_launch(), sw.last_launch()
    keys = ["dx", "ddelta", "dA", "dB", "dC", "dDskip", "dh0"]
    keys += ["dz"] if "z" in opts else []
    keys += ["ddelta_bias"] if "bias" in opts else []
    _check_all(g, _ref(inp, ex, opts), f"{dtype} {shape} {opts}", keys)
    g2 = _run(sw, inp, ex, dtype, opts)
    for k in g:
        assert torch.equal(g[k], g2[k]), k


# D at the edges of 16 rows beside those above, L at the edges of the four tiles
# that loads run ahead, a last state group that is not full
@pytest.mark.parametrize("shape", _SHAPES + [(1, 16, 16, 24), (3, 33, 16, 31), (1, 48, 16, 32),
                                             (2, 18, 47, 25)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("opts", [(), _ALL, ("dybf16", "h0", "dhl")])
@pytest.mark.parametrize("rows", ["16", "64"])
def test_bwd_kernels_of_16_and_64_rows(sw, monkeypatch, shape, dtype, opts, rows):  # noqa: F811
    """Both kernels of the backward on every shape, whichever the rule takes."""
    monkeypatch.setenv("SW_SS_BWD_ROWS", rows)
    B, D, N, L = shape
    print("case bwd rows", rows, dtype, shape, opts, flush=True)
    inp, ex = _inputs(B, D, N, L, 2800 + B + D + N + L, dtype, opts)
    g = _run(sw, inp, ex, dtype, opts)
    assert ("rows16" in sw.last_launch()) == (rows == "16"), sw.last_launch()
    keys = ["dx", "ddelta", "dA", "dB", "dC", "dDskip", "dh0"]
    keys += ["dz"] if "z" in opts else []
    keys += ["ddelta_bias"] if "bias" in opts else []
    _check_all(g, _ref(inp, ex, opts), f"rows {rows} {dtype} {shape} {opts}", keys)


@pytest.mark.parametrize("rows", ["16", "64"])
@pytest.mark.parametrize("shape", [(2, 37, 16, 200), (1, 70, 16, 203), (2, 9, 5, 64)])
def test_bf16_gradients_of_both_kernels(sw, monkeypatch, shape, rows):  # noqa: F811
    monkeypatch.setenv("SW_SS_BWD_ROWS", rows)
    test_autograd_bf16_gradients_are_the_fp32_ones_rounded(sw, shape)
    assert ("rows16" in sw.last_launch()) == (rows == "16"), sw.last_launch()


@pytest.mark.parametrize("shape,rows16", [((8, 1536, 16, 1024), True), ((4, 1536, 16, 128), True),
                                          ((4, 1024, 16, 1024), False), ((8, 2048, 16, 256), False)])
def test_bwd_takes_the_kernel_that_fills_the_gpu(sw, shape, rows16):  # noqa: F811
    """The rule between the kernels on a 256-CU part: 16 rows a workgroup where
    those are two or three per compute unit and 64-row ones leave units idle."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("priced for 256 compute units")
    B, D, N, L = shape
    x = torch.randn((B, D, L), device="cuda").bfloat16()
    Bm = torch.randn((B, L, N), device="cuda").bfloat16()
    A = -torch.rand((D, N), device="cuda")
    sw.selective_scan_bwd(x, x.abs() * 0.01, A, Bm, Bm, None, x)
    assert ("rows16" in sw.last_launch()) == rows16, sw.last_launch()


@pytest.mark.parametrize("A", ["zero", "growth"])
def test_bwd_segments_without_decay(sw, A):  # noqa: F811
    """The adjoint carried across segments where it does not fade."""
    B, D, N, L = 1, 18, 16, 1200
    inp, ex = _inputs(B, D, N, L, 2400, "f32", ("dhl",))
    inp["A"] = np.zeros_like(inp["A"]) if A == "zero" else np.abs(inp["A"]) * np.float32(1e-3)
    g = _run(sw, inp, ex, "f32", ("dhl",))
    o = _ref(inp, ex, ("dhl",))
    _check_all(g, o, A, ["dx", "ddelta", "dA", "dB", "dC", "dDskip", "dh0"])


@pytest.mark.parametrize("shape", [(2, 37, 16, 200), (1, 70, 16, 203), (2, 9, 5, 64)])
def test_autograd_bf16_gradients_are_the_fp32_ones_rounded(sw, shape):  # noqa: F811
    B, D, N, L = shape
    inp, ex = _inputs(B, D, N, L, 2500 + L, "bf16", ("z", "bias", "softplus"))
    t = {"x": _bf16_dev(inp["x_bf16"]), "delta": _bf16_dev(inp["delta_bf16"]), "A": _dev(inp["A"]),
         "Bm": _bf16_dev(inp["Bm_bf16"]), "Cm": _bf16_dev(inp["Cm_bf16"]), "Dskip": _dev(inp["Dskip"]),
         "z": _bf16_dev(ex["z_bits"]), "delta_bias": _dev(ex["delta_bias"])}
    leaves = {k: v.requires_grad_() for k, v in t.items()}
    y = sw.selective_scan_fn(*(leaves[k] for k in ("x", "delta", "A", "Bm", "Cm", "Dskip")),
                             z=leaves["z"], delta_bias=leaves["delta_bias"], delta_softplus=True)
    dy = _dev(ex["dy"])
    got = torch.autograd.grad(y, list(leaves.values()), dy)
    d = {k: v.detach() for k, v in leaves.items()}
    ck = sw.new_ckpt(d["x"], N)
    sp = torch.empty((B, D, L), device="cuda")
    kw = dict(z=d["z"], delta_bias=d["delta_bias"], delta_softplus=True)
    args = [d[k] for k in ("x", "delta", "A", "Bm", "Cm", "Dskip")]
    sw.selective_scan_fwd(*args, ckpt=ck, s_pre=sp, **kw)
    g = sw.selective_scan_bwd(*args, dy, ckpt=ck, s_pre=sp, **kw)
    names = dict(zip(leaves, ("dx", "ddelta", "dA", "dB", "dC", "dDskip", "dz", "ddelta_bias")))
    for (k, leaf), v in zip(leaves.items(), got):
        assert v.dtype == leaf.dtype and torch.equal(v, g[names[k]].to(leaf.dtype)), k


# N = 16, and the states below 16 that the 16-lane kernels take as one group
# (N = 4: long calls on few rows)
@pytest.mark.parametrize("N,L,segs", [(16, 1024, "4"), (16, 1003, "3"), (12, 1024, "4"),
                                      (10, 1003, "3"), (4, 1601, "3")])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_segmented_training_forward(sw, monkeypatch, N, L, segs, dtype):  # noqa: F811
    """Under autograd the forward may cut its rows: its checkpoints, pre-gate
    output and y are those of the whole-row walk within fp32 rounding (the
    composed state is one more rounding per segment of terms that the walk
    rounds at every step: 2^-18 of the largest, against 2^-24 a step), and the
    gradients are the oracle's."""
    B, D = 1, 21
    opts = ("z", "bias", "softplus", "h0")
    inp, ex = _inputs(B, D, N, L, 2600 + L, dtype, opts)
    conv = (lambda k: _bf16_dev(inp[k + "_bf16"])) if dtype == "bf16" else (lambda k: _dev(inp[k]))
    x, dl, Bm, Cm = (conv(k) for k in ("x", "delta", "Bm", "Cm"))
    z = _bf16_dev(ex["z_bits"]) if dtype == "bf16" else _dev(ex["z"])
    A, Dk = _dev(inp["A"]), _dev(inp["Dskip"])
    rest = (z, _dev(ex["delta_bias"]), _dev(ex["h0"]), True, torch.float32)
    got = []
    for count, seg in (("1", False), (segs, True)):
        monkeypatch.setenv("SW_SS_SEGMENTS", count)
        ck = sw.new_ckpt(x, N).fill_(float("nan"))
        sp = torch.full((B, D, L), float("nan"), device="cuda")
        y, hl = sw._fwd(x, dl, A, Bm, Cm, Dk, None, None, True, *rest, ck, sp, seg)
        assert (f"{segs} segments" in sw.last_launch()) == seg, sw.last_launch()
        got.append((y, hl, ck[..., :N], sp))  # (slots past N hold no state)
    for a, b in zip(*got):
        assert bool(torch.isfinite(b).all())
        assert (a - b).abs().max() <= 2 ** -18 * a.abs().max()
    leaves = [t.requires_grad_() for t in (x, dl, A, Bm, Cm, Dk, z)]
    y = sw.selective_scan_fn(*leaves, delta_bias=rest[1], h0=rest[2], delta_softplus=True)
    g = torch.autograd.grad(y, leaves, _dev(ex["dy"]))
    o = _ref(inp, ex, opts)
    for v, k in zip(g, ("dx", "ddelta", "dA", "dB", "dC", "dDskip", "dz")):
        if v.dtype == torch.float32:
            assert_gate(fp_gate(v.cpu().numpy(), o[k], o["m_" + k]), f"segmented {k}")
        else:  # rounded once more, half a unit of 8 bits
            err = np.abs(v.float().cpu().numpy() - o[k])
            assert (err <= 2.0 ** -8 * np.abs(o[k]) + 1.01e-4 * o["m_" + k]).all(), k


@pytest.mark.parametrize("lo,hi", [(-60.0, -15.0), (-20.0, 20.0), (15.0, 90.0)])
def test_bwd_softplus_over_its_range(sw, lo, hi):  # noqa: F811
    """softplus and its derivative where 1 + e^-|v| rounds to 1, around 0 and
    where softplus(v) is v, zero of either sign included."""
    B, D, N, L = 2, 19, 16, 70
    opts = ("softplus", "z", "h0")
    inp, ex = _inputs(B, D, N, L, 2700 + int(hi), "f32", opts)
    v = np.random.Generator(np.random.PCG64(27)).uniform(lo, hi, (B, D, L))
    inp["delta"] = v.astype(np.float32)
    inp["delta"][:, :2, ::7] = np.float32([0.0, -0.0])[:, None]
    inp["A"] = inp["A"] * np.float32(1.0 / 64)
    g = _run(sw, inp, ex, "f32", opts)
    _check_all(g, _ref(inp, ex, opts), f"softplus {lo} {hi}",
               ["dx", "ddelta", "dA", "dB", "dC", "dDskip", "dz", "dh0"])


@pytest.mark.parametrize("N,L,k", [(5, 3, 0), (5, 3, 1), (4, 2, 1)])
def test_bwd_of_no_rows_clears_odd_bf16_gradients(sw, N, L, k):  # noqa: F811
    """No rows (D = 0): dB and dC are sums of nothing, cleared whole, in bf16
    also where their number is odd or they start off a 4-byte boundary, and
    nothing beside them is."""
    n = L * N
    bufs = [torch.full((n + 8,), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    B16, F32 = 1, 0
    ptr = [b.data_ptr() + 2 * k for b in bufs]
    args = [None] * 16 + [ptr[0], ptr[1]] + [None] * 4
    with sw._on(bufs[0].device):
        st = sw.lib().sw_selective_scan_bwd_ex(*args, 1, 0, N, L, B16, F32, B16, 0, None, 0)
    assert st == 0, sw.lib().sw_last_error()
    for b in bufs:
        assert torch.count_nonzero(b[k:k + n]) == 0 and bool(torch.isnan(b[:k]).all())
        assert bool(torch.isnan(b[k + n:]).all())
