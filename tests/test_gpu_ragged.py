"""The 16-lane forward (N = 16) on rows of any length and alignment: the oracle
at lengths around a lane's vector, a tile and a super-tile, whole rows and
segments of either form; and, where the rows are whole vectors, the same bits
whether the arrays are 16-byte aligned or one element off."""
import numpy as np
import pytest

from gate import assert_gate, fp_gate
from test_gpu_parity import _ex_inputs, _ex_oracle, _run_ex, _y_gate, sw  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (B, D, L), forced segments ("" : the library's choice), form
_CASES = [((1, 5, 17), "", ""), ((2, 37, 31), "", ""), ((1, 18, 33), "1", ""),
          ((1, 16, 127), "1", ""), ((2, 17, 129), "1", ""), ((1, 7, 1999), "", ""),
          ((1, 21, 1003), "3", "1"), ((2, 33, 1001), "4", "2"), ((1, 16, 387), "2", "1"),
          ((1, 3, 4093), "16", "2"), ((1, 3, 4094), "16", "1")]


@pytest.mark.parametrize("case", _CASES)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("opts", [(), ("h0", "bias", "softplus", "z"),
                                  ("h0", "bias", "softplus", "z", "ybf16")])
def test_ragged_rows_match_oracle(sw, monkeypatch, case, dtype, opts):  # noqa: F811
    (B, D, L), segs, form = case
    if segs:
        monkeypatch.setenv("SW_SS_SEGMENTS", segs)
    if form:
        monkeypatch.setenv("SW_SS_SEGFORM", form)
    print("case ragged", dtype, case, opts, flush=True)
    inp, ex = _ex_inputs(B, D, 16, L, 5100 + B + D + L, dtype, opts)
    y, hl = _run_ex(sw, inp, ex, dtype, "softplus" in opts, "ybf16" in opts)
    assert sw.last_launch().startswith("selective_row16_kernel"), sw.last_launch()
    if segs not in ("", "1") and not ("ybf16" in opts and form == "2"):
        assert "segments" in sw.last_launch(), sw.last_launch()
    o = _ex_oracle(inp, ex, "softplus" in opts)
    _y_gate(y, o, "ybf16" in opts, f"ragged y {dtype} {case} {opts}")
    assert_gate(fp_gate(hl.cpu().numpy(), o["h_last"], o["h_mag"], o["h_sens"]),
                f"ragged h_last {dtype} {case} {opts}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("segs,form", [("1", ""), ("3", "1"), ("3", "2")])
@pytest.mark.parametrize("opts", [(), ("h0", "bias", "softplus", "z")])
def test_unaligned_rows_give_the_aligned_bits(sw, monkeypatch, dtype, segs, form, opts):  # noqa: F811
    B, D, L = 2, 19, 648
    monkeypatch.setenv("SW_SS_SEGMENTS", segs)
    monkeypatch.setenv("SW_SS_QUAD", "0")
    if form:
        monkeypatch.setenv("SW_SS_SEGFORM", form)
    print("case unaligned", dtype, segs, form, opts, flush=True)
    inp, ex = _ex_inputs(B, D, 16, L, 5300, dtype, opts)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")  # noqa: E731

    def arr(a, k):  # the array k elements past a 16-byte boundary
        buf = torch.empty(a.size + 16, dtype=tdt, device="cuda")
        return buf[k:k + a.size].view(*a.shape).copy_(dev(a).to(tdt))

    def run(ks):
        kw = {}
        if opts:
            kw = dict(z=arr(ex["z"], ks[2]), delta_bias=dev(ex["delta_bias"]), h0=dev(ex["h0"]),
                      delta_softplus=True)
        y = torch.empty(B * D * L + 16, device="cuda")[ks[3]:ks[3] + B * D * L].view(B, D, L)
        return sw.selective_scan_fwd(arr(inp["x"], ks[0]), arr(inp["delta"], ks[1]), dev(inp["A"]),
                                     arr(inp["Bm"], 0), arr(inp["Cm"], 0), dev(inp["Dskip"]), y=y, **kw)

    y0, h0 = run((0, 0, 0, 0))
    for ks in ((1, 0, 0, 0), (0, 3, 1, 2), (1, 1, 2, 1)):
        y1, h1 = run(ks)
        torch.cuda.synchronize()
        assert torch.equal(y0, y1) and torch.equal(h0, h1), ks


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L", [77, 203])
def test_ragged_checkpoints(sw, dtype, L):  # noqa: F811
    """Checkpoints and pre-gate output of a ragged training forward: the
    backward fed with them gives the bits of the backward that rebuilds them,
    and the pre-gate output stays inside its array."""
    B, D, N = 2, 19, 16
    opts = ("h0", "bias", "softplus", "z")
    inp, ex = _ex_inputs(B, D, N, L, 5500 + L, dtype, opts)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    dev = lambda a, dt=torch.float32: torch.from_numpy(np.ascontiguousarray(a)).to("cuda").to(dt)  # noqa: E731
    x, dl, z = dev(inp["x"], tdt), dev(inp["delta"], tdt), dev(ex["z"], tdt)
    A, Bm, Cm, Dk = dev(inp["A"]), dev(inp["Bm"], tdt), dev(inp["Cm"], tdt), dev(inp["Dskip"])
    kw = dict(delta_bias=dev(ex["delta_bias"]), h0=dev(ex["h0"]), delta_softplus=True)
    ck = sw.new_ckpt(x, N)
    guard = torch.full((B * D * L + 8,), 7.0, device="cuda")
    sp = guard[4:-4].view(B, D, L)
    sw.selective_scan_fwd(x, dl, A, Bm, Cm, Dk, z=z, ckpt=ck, s_pre=sp, **kw)
    torch.cuda.synchronize()
    assert bool((guard[:4] == 7.0).all()) and bool((guard[-4:] == 7.0).all())
    dy = torch.randn((B, D, L), device="cuda")
    args = (x, dl, A, Bm, Cm, Dk, dy)
    g1 = sw.selective_scan_bwd(*args, z=z, ckpt=ck, s_pre=sp, **kw)
    g0 = sw.selective_scan_bwd(*args, z=z, **kw)
    n1 = sw.selective_scan_bwd(*args, ckpt=ck, **kw)
    n0 = sw.selective_scan_bwd(*args, **kw)  # the backward kernel's own sweep
    torch.cuda.synchronize()
    for k in g0:
        assert torch.equal(g0[k], g1[k]), k
    for k in n0:
        assert torch.equal(n0[k], n1[k]), k


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(2, 70, 64), (1, 33, 1056)])
def test_quad_whole_rows_in_bf16(sw, monkeypatch, dtype, shape):  # noqa: F811
    """bf16 y of the quad layout on whole rows: the fp32 y rounded once."""
    B, D, L = shape
    monkeypatch.setenv("SW_SS_QUAD", "1")
    monkeypatch.setenv("SW_SS_SEGMENTS", "1")
    inp, ex = _ex_inputs(B, D, 16, L, 5700 + L, dtype, ("h0", "bias", "softplus", "z"))
    y32, h32 = _run_ex(sw, inp, ex, dtype, True, False)
    assert sw.last_launch() == "selective_quad_kernel: whole rows", sw.last_launch()
    y16, h16 = _run_ex(sw, inp, ex, dtype, True, True)
    assert sw.last_launch() == "selective_quad_kernel: whole rows", sw.last_launch()
    assert torch.equal(y16, y32.to(torch.bfloat16)) and torch.equal(h16, h32)
