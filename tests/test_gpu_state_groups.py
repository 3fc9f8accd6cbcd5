"""The forward on an even N other than 16: states in groups of 16 lanes,
one group (N = 10, 14; N = 4, 8 on long
calls of few rows) writing y itself and several adding up planes of y (the
last group full or not), whole rows and segments of either form, at aligned
and ragged lengths, against the oracle."""
import ctypes

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


def _pool_high(dev, reset):
    """The most bytes in use of the device's default stream-ordered pool since
    the last reset (hipMemPoolAttrUsedMemHigh)."""
    path = next(ln.split()[-1] for ln in open("/proc/self/maps") if "libamdhip64.so" in ln)
    hip, pool, v = ctypes.CDLL(path), ctypes.c_void_p(), ctypes.c_uint64(0)
    assert hip.hipDeviceGetDefaultMemPool(ctypes.byref(pool), dev) == 0
    if reset:
        assert hip.hipMemPoolSetAttribute(pool, 8, ctypes.byref(v)) == 0
    assert hip.hipMemPoolGetAttribute(pool, 8, ctypes.byref(v)) == 0
    return v.value


@pytest.mark.parametrize("N", [24, 64])
@pytest.mark.parametrize("train", [False, True])
def test_planes_come_from_the_callers_allocator(sw, N, train):  # noqa: F811
    """A forward of several state groups, and the gated backward that runs one
    without the gate, leave no planes in the library's own pool, which never
    gives memory back."""
    B, D, L = 2, 200, 1500
    planes = (N + 15) // 16 * B * D * L * 4
    x, z = (torch.randn((B, D, L), device="cuda") for _ in range(2))
    Bm = torch.randn((B, L, N), device="cuda")
    A = -torch.rand((D, N), device="cuda")
    assert sw.lib().sw_selective_scan_fwd_workspace(B, D, N, L, 0, 1, 1) == planes
    torch.cuda.synchronize()
    before = _pool_high(0, True)
    if train:
        sw.selective_scan_bwd(x, x.abs() * 0.01, A, Bm, Bm, None, x, z=z)
    else:
        sw.selective_scan_fwd(x, x.abs() * 0.01, A, Bm, Bm, z=z)
        assert sw.last_launch().startswith("selective_row16_kernel"), sw.last_launch()
    torch.cuda.synchronize()
    assert _pool_high(0, False) - before < planes


def test_workspace_of_the_forward(sw):  # noqa: F811
    """Planes in the caller's workspace give the bits of planes from the pool;
    one that is too small is refused before anything is enqueued."""
    B, D, N, L = 1, 37, 40, 900
    x = torch.randn((B, D, L), device="cuda")
    dl, Bm = x.abs() * 0.01, torch.randn((B, L, N), device="cuda")
    A = -torch.rand((D, N), device="cuda")
    y = [torch.full_like(x, float("nan")) for _ in range(3)]
    n = sw.lib().sw_selective_scan_fwd_workspace(B, D, N, L, 0, 0, 1)
    ws = torch.empty((n + 64,), dtype=torch.uint8, device="cuda")

    def call(out, wsp, nbytes):
        ptrs = [t.data_ptr() for t in (x, dl, A, Bm, Bm)] + [None] * 4 + [out.data_ptr(), None]
        with sw._on(x.device):
            return sw.lib().sw_selective_scan_fwd_ws(*ptrs, B, D, N, L, 0, 0, 0, wsp, nbytes)

    assert n == 3 * B * D * L * 4
    assert call(y[0], ws.data_ptr(), n) == 0 and call(y[1], None, 0) == 0
    assert torch.equal(y[0], y[1]) and bool(torch.isfinite(y[0]).all())
    assert call(y[2], ws.data_ptr(), n - 16) == 1  # SW_ERR_INVALID_ARG
    assert call(y[2], ws.data_ptr() + 4, n) == 1  # not 16-byte aligned
    assert call(y[2], y[2].data_ptr(), n) == 1  # overlaps y
    assert bool(torch.isnan(y[2]).all())
