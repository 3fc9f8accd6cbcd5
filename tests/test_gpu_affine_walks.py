"""The bare scan's walks at the edges of their rules: one wavefront per row (up
to 512 steps, 1 to 8 steps a lane), one workgroup per row, and segments (few
rows of many chunks), each at ragged lengths, with the arrays off any 16-byte
boundary; int32 against the exact ring, the elementwise form against its
oracle, and the segmented fp32 walk against itself, bit for bit."""
import numpy as np
import pytest

import oracle
import workloads as wl
from gate import assert_gate, fp_gate
from test_gpu_parity import sw  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _off(a, k=1):
    """The array on the GPU, k elements past a 16-byte boundary."""
    a = np.ascontiguousarray(a)
    t = torch.from_numpy(a)
    buf = torch.empty(a.size + 8, dtype=t.dtype, device="cuda")
    return buf[k:k + a.size].view(*a.shape).copy_(t)


_ROWS = [(1, 5), (2, 3), (3, 4), (5, 63), (5, 65), (7, 127), (6, 129), (5, 255), (3, 257), (9, 511),
         (3, 513), (2, 1023), (4, 1025), (3, 2049), (2, 22527), (65, 22531), (64, 24577), (3, 70001)]


@pytest.mark.parametrize("R,L", _ROWS)
@pytest.mark.parametrize("k", [0, 1, 3])
def test_i32_walks(sw, R, L, k):  # noqa: F811
    print("case affine walk i32", R, L, k, flush=True)
    inp = wl.affine_inputs_i32(1, R, L, 100 + R + L, "odd")
    h0 = wl.affine_inputs_i32(1, R, 1, 200 + L, "h0")["h0"]
    out = _off(np.zeros((1, R, L), np.int32), (k + 1) % 4)
    sw.affine_scan_i32(_off(inp["a"], k), _off(inp["bx"], (2 * k) % 4), _off(h0), out=out)
    assert np.array_equal(out.cpu().numpy(), oracle.affine_scan_i32(inp["a"], inp["bx"], h0))


@pytest.mark.parametrize("R,L", [(5, 3), (4, 62), (3, 510), (5, 1021), (3, 4099), (7, 30003)])
@pytest.mark.parametrize("with_x,with_c", [(True, True), (False, True), (True, False)])
def test_proj_walks(sw, R, L, with_x, with_c):  # noqa: F811
    print("case proj walk", R, L, with_x, with_c, flush=True)
    rng = np.random.default_rng(R + L)
    draw = lambda: rng.integers(-2**31, 2**31, (1, R, L), dtype=np.int64).astype(np.int32)  # noqa: E731
    a, b = draw(), draw()
    x = draw() if with_x else None
    c = draw() if with_c else None
    h0 = draw()[:, :, 0].copy()
    y, hl = sw.affine_scan_proj_i32(*(None if v is None else _off(v) for v in (a, b, x, c, h0)))
    ry, rh = oracle.affine_proj_i32(a, b, x, c, h0)
    assert np.array_equal(y.cpu().numpy(), ry) and np.array_equal(hl.cpu().numpy(), rh)


def test_f32_segments_are_reproducible(sw):  # noqa: F811
    R, L = 6, 100003
    inp = wl.affine_inputs(1, R, L, 31, with_h0=True)
    a, bx, h0 = (torch.from_numpy(inp[k]).cuda() for k in ("a", "bx", "h0"))
    h = sw.affine_scan(a, bx, h0)
    want, mag, sens = oracle.affine_scan(inp["a"], inp["bx"], inp["h0"], bounds=True)
    assert_gate(fp_gate(h.cpu().numpy(), want, mag, sens), "segments f32")
    for _ in range(5):
        assert torch.equal(sw.affine_scan(a, bx, h0), h)
    assert torch.equal(sw.affine_scan_noalloc(a, bx, h0), h)


def test_more_rows_than_a_grid_holds(sw):  # noqa: F811
    """2^26 rows of one step, one more than a launch of a workgroup per four
    rows may have (2^32 threads): the workgroups take several each."""
    R = 2 ** 26 + 5
    bx = torch.arange(R, dtype=torch.int32, device="cuda").view(1, R, 1)
    a = torch.full_like(bx, 3)
    assert torch.equal(sw.affine_scan_i32(a, bx), bx)
    h0 = bx.view(1, R)
    y, hl = sw.affine_scan_proj_i32(a, bx, None, a, h0)
    assert torch.equal(hl, 4 * h0) and torch.equal(y, 12 * bx)


def test_more_rows_than_a_grid_holds_blelloch(sw):  # noqa: F811
    """The paper's schedule, a workgroup per row, on more than 2^24 rows."""
    R = 2 ** 24 + 5
    bx = torch.arange(R, dtype=torch.int32, device="cuda").view(1, R, 1)
    h = sw.affine_scan_schedule_i32(torch.full_like(bx, 3), bx, bx.view(1, R), schedule="blelloch")
    assert torch.equal(h, 4 * bx)
    x = bx.float()
    one = torch.ones((1, 1, 1), device="cuda")
    y, hl = sw.selective_scan_fwd_schedule(x, torch.ones_like(x), -torch.ones((R, 1), device="cuda"),
                                           one, one, schedule="blelloch")
    assert torch.equal(y, x) and torch.equal(hl, x)
