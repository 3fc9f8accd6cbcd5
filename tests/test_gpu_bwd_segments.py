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
