"""The forward on an even N other than 16: states in groups of 16 lanes,
one group (N = 10, 14; N = 4, 8 on long
calls of few rows) writing y itself and several adding up planes of y (the
last group full or not), whole rows and segments of either form, at aligned
and ragged lengths, against the oracle."""
import numpy as np
import pytest

from gate import assert_gate, fp_gate
from test_gpu_parity import _ex_inputs, _ex_oracle, _run_ex, _y_gate, sw  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (B, D, N, L), forced segments, form
_CASES = [((2, 19, 10, 100), "", ""), ((1, 33, 14, 517), "3", "1"), ((1, 17, 24, 1000), "1", ""),
          ((2, 16, 32, 515), "", ""), ((1, 21, 48, 777), "3", "2"), ((1, 16, 64, 640), "4", "1"),
          ((1, 5, 34, 367), "", ""), ((1, 20, 4, 1500), "", ""), ((2, 9, 8, 1601), "", ""), ((1, 18, 62, 2049), "5", "2")]


@pytest.mark.parametrize("case", _CASES)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("opts", [(), ("h0", "bias", "softplus", "z"),
                                  ("h0", "bias", "softplus", "z", "ybf16")])
def test_state_groups(sw, monkeypatch, case, dtype, opts):  # noqa: F811
    (B, D, N, L), segs, form = case
    if segs:
        monkeypatch.setenv("SW_SS_SEGMENTS", segs)
    if form:
        monkeypatch.setenv("SW_SS_SEGFORM", form)
    print("case groups", dtype, case, opts, flush=True)
    inp, ex = _ex_inputs(B, D, N, L, 6100 + B + D + N + L, dtype, opts)
    y, hl = _run_ex(sw, inp, ex, dtype, "softplus" in opts, "ybf16" in opts)
    assert sw.last_launch().startswith("selective_row16_kernel"), sw.last_launch()
    o = _ex_oracle(inp, ex, "softplus" in opts)
    _y_gate(y, o, "ybf16" in opts, f"groups y {dtype} {case} {opts}")
    assert_gate(fp_gate(hl.cpu().numpy(), o["h_last"], o["h_mag"], o["h_sens"]),
                f"groups h_last {dtype} {case} {opts}")
    y2, hl2 = _run_ex(sw, inp, ex, dtype, "softplus" in opts, "ybf16" in opts)
    assert torch.equal(y, y2) and torch.equal(hl, hl2)


def test_group_checkpoints(sw):  # noqa: F811
    """N = 12 (one group): the training forward's checkpoints give the bits of
    the backward that rebuilds them."""
    B, D, N, L = 2, 19, 12, 203
    inp, ex = _ex_inputs(B, D, N, L, 6500, "f32", ("h0",))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")  # noqa: E731
    args = [dev(inp[k]) for k in ("x", "delta", "A", "Bm", "Cm", "Dskip")]
    ck = sw.new_ckpt(args[0], N)
    sw.selective_scan_fwd(*args, h0=dev(ex["h0"]), ckpt=ck)
    dy = torch.randn((B, D, L), device="cuda")
    g1 = sw.selective_scan_bwd(*args, dy, h0=dev(ex["h0"]), ckpt=ck)
    g0 = sw.selective_scan_bwd(*args, dy, h0=dev(ex["h0"]))
    for k in g0:
        assert torch.equal(g0[k], g1[k]), k
