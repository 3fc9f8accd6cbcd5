"""The few-step kernel of the fused forward (calls of at most 16 steps):
against the fp64 oracle at the edges of its range -- N below, at and between
the 16-state groups, D off the 64-row blocks, one step and the last length it
takes, unaligned states -- and one token at a time against one call."""
import numpy as np
import pytest

from gate import assert_gate, fp_gate
from test_gpu_parity import _ex_inputs, _ex_oracle, _run_ex, _y_gate, sw  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

_SHAPES = [(1, 1, 1, 1), (2, 65, 16, 1), (3, 64, 16, 16), (2, 37, 20, 3), (1, 130, 64, 2),
           (2, 5, 3, 7), (1, 70, 48, 5)]


@pytest.mark.parametrize("shape", _SHAPES)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("opts", [(), ("h0", "bias", "softplus", "z", "ybf16")])
def test_step_matches_oracle(sw, shape, dtype, opts):  # noqa: F811
    B, D, N, L = shape
    print("case step", dtype, shape, opts, flush=True)
    inp, ex = _ex_inputs(B, D, N, L, 3100 + B + D + N + L, dtype, opts)
    y, hl = _run_ex(sw, inp, ex, dtype, "softplus" in opts, "ybf16" in opts)
    assert sw.last_launch().startswith("selective_step_kernel"), sw.last_launch()
    o = _ex_oracle(inp, ex, "softplus" in opts)
    _y_gate(y, o, "ybf16" in opts, f"step y {dtype} {shape} {opts}")
    assert_gate(fp_gate(hl.cpu().numpy(), o["h_last"], o["h_mag"], o["h_sens"]),
                f"step h_last {dtype} {shape} {opts}")


def test_step_unaligned_states_and_token_by_token(sw):  # noqa: F811
    """Twenty tokens one call each, h_last handed on as h0, the states 4 bytes
    off a 16-byte boundary (element loads): the same as one call over the
    sequence (the 16-lane kernel) within the rounding of the 16-term sums."""
    B, D, N, L = 2, 33, 16, 20
    inp, ex = _ex_inputs(B, D, N, L, 3300, "f32", ("h0",))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")  # noqa: E731
    off = lambda *s: torch.empty(int(np.prod(s)) + 1, device="cuda")[1:].view(*s)  # noqa: E731
    A, Dk, h0 = dev(inp["A"]), dev(inp["Dskip"]), dev(ex["h0"])
    y_one, h_one = sw.selective_scan_fwd(dev(inp["x"]), dev(inp["delta"]), A, dev(inp["Bm"]),
                                         dev(inp["Cm"]), Dk, h0=h0)
    h, ys = off(B, D, N).copy_(h0), []
    for t in range(L):
        nxt = off(B, D, N)
        yt, _ = sw.selective_scan_fwd(dev(inp["x"][:, :, t:t + 1]), dev(inp["delta"][:, :, t:t + 1]),
                                      A, dev(inp["Bm"][:, t:t + 1]), dev(inp["Cm"][:, t:t + 1]), Dk,
                                      h0=h, h_last=nxt)
        ys.append(yt)
        h = nxt
    torch.cuda.synchronize()
    # 20 steps of the same fp32 arithmetic, sums of 17 terms in another order:
    # at most 17 roundings of 2^-24 of the terms' magnitude
    assert (h - h_one).abs().max() <= 2 ** -20 * h_one.abs().max()
    y = torch.cat(ys, dim=2)
    assert (y - y_one).abs().max() <= 2 ** -19 * y_one.abs().max()
