"""The fused forward captured into a HIP graph (through torch's graph capture)
and replayed: every replay, with eager calls and synchronizations between the
replays, gives the eager result bit for bit.

The N = 16 forward takes no scratch memory and allocates nothing, so it can be
captured; the calls that use the per-stream scratch (the bare scan's
segments, the persistent kernel of N != 16) or allocate (the backward) are
not graph-replay safe, and the library refuses them while the stream is
capturing (checked here).  The bare scan's entry point that allocates
nothing keeps its tickets and records in a static array that every call clears
with a fill kernel, so its segments can be captured too (checked here).
"""
import sys

import numpy as np
import pytest

import oracle
import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def sw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_00601_amd as pkg
    pkg.lib()
    return pkg


def _bf(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).to("cuda").view(
        torch.bfloat16)


@pytest.mark.parametrize("options", [False, True])
def test_forward_graph_replays_match_eager(sw, options):
    B, D, N, L = 2, 48, 16, 512
    _say("case graph replay", B, D, N, L, "options" if options else "plain")
    inp = wl.selective_inputs(B, D, N, L, 777, "bf16")
    x, dl = _bf(inp["x_bf16"]), _bf(inp["delta_bf16"])
    Bm, Cm = _bf(inp["Bm_bf16"]), _bf(inp["Cm_bf16"])
    A = torch.from_numpy(inp["A"]).to("cuda")
    Dk = torch.from_numpy(inp["Dskip"]).to("cuda")
    kw = {}
    if options:
        rng = np.random.Generator(np.random.PCG64(778))
        kw = dict(z=_bf(wl.bf16_round(rng.standard_normal((B, D, L)).astype(np.float32))),
                  delta_bias=torch.from_numpy(rng.uniform(-2, 0, D).astype(np.float32)).to("cuda"),
                  h0=torch.from_numpy(rng.standard_normal((B, D, N)).astype(np.float32)).to("cuda"),
                  delta_softplus=True)
    y_ref, h_ref = sw.selective_scan_fwd(x, dl, A, Bm, Cm, Dk, **kw)
    torch.cuda.synchronize()
    y = torch.empty_like(y_ref)
    hl = torch.empty_like(h_ref)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):  # warm-up on the capture stream
        sw.selective_scan_fwd(x, dl, A, Bm, Cm, Dk, y=y, h_last=hl, **kw)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        sw.selective_scan_fwd(x, dl, A, Bm, Cm, Dk, y=y, h_last=hl, **kw)
    for i in range(4):
        y.fill_(float("nan"))
        hl.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, y_ref), f"replay {i}: y differs"
        assert torch.equal(hl, h_ref), f"replay {i}: h_last differs"
        # eager work of the program between replays
        y2, h2 = sw.selective_scan_fwd(x, dl, A, Bm, Cm, Dk, **kw)
        torch.cuda.synchronize()
        assert torch.equal(y2, y_ref) and torch.equal(h2, h_ref)


def test_capture_refuses_calls_that_need_scratch_or_workspace(sw):
    """While the stream is capturing, the calls that use the per-stream scratch
    (the bare scan's segments of a few long rows, the persistent
    kernel of N != 16) or allocate a workspace (the backward) raise instead of
    recording a graph whose replay would write nothing; a legal call captured
    beside them replays correctly, and the refused calls still work eagerly."""
    _say("case capture refusals")
    rng = np.random.Generator(np.random.PCG64(779))
    dev = "cuda"
    # bare scan (int32 ring: exact, so any carry order gives the same bits),
    # 4 rows of 16384 steps: 8 chunks per row, a segment each
    ai = torch.from_numpy(rng.integers(-2**31, 2**31, (1, 4, 16384), dtype=np.int64)
                          .astype(np.int32)).to(dev)
    bi = torch.from_numpy(rng.integers(-2**31, 2**31, (1, 4, 16384), dtype=np.int64)
                          .astype(np.int32)).to(dev)
    # fused forward with N = 8 (persistent kernel with a ticket counter)
    B, D, L = 1, 16, 64
    f32 = lambda *s: torch.from_numpy(rng.standard_normal(s).astype(np.float32)).to(dev)
    x, dl = f32(B, D, L), torch.from_numpy(
        rng.uniform(0.01, 0.1, (B, D, L)).astype(np.float32)).to(dev)
    A8 = -torch.from_numpy(rng.uniform(0.5, 2.0, (D, 8)).astype(np.float32)).to(dev)
    B8, C8 = f32(B, L, 8), f32(B, L, 8)
    # legal: N = 16 forward; the backward of the same (refused: workspace)
    A16 = -torch.from_numpy(rng.uniform(0.5, 2.0, (D, 16)).astype(np.float32)).to(dev)
    B16, C16, Dk, dy = f32(B, L, 16), f32(B, L, 16), f32(D), f32(B, D, L)

    refused = {
        "bare scan in segments": lambda: sw.affine_scan_i32(ai, bi),
        "forward N=8": lambda: sw.selective_scan_fwd(x, dl, A8, B8, C8, Dk),
        "backward": lambda: sw.selective_scan_bwd(x, dl, A16, B16, C16, Dk, dy),
    }
    y_ref, h_ref = sw.selective_scan_fwd(x, dl, A16, B16, C16, Dk)
    eager = {k: f() for k, f in refused.items()}
    torch.cuda.synchronize()
    y = torch.empty_like(y_ref)
    hl = torch.empty_like(h_ref)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        sw.selective_scan_fwd(x, dl, A16, B16, C16, Dk, y=y, h_last=hl)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        sw.selective_scan_fwd(x, dl, A16, B16, C16, Dk, y=y, h_last=hl)
        for name, fn in refused.items():
            with pytest.raises(sw.ScanWeaverError, match="captured") as ei:
                fn()
            assert ei.value.status == 2, name  # SW_ERR_UNSUPPORTED
    for i in range(3):
        y.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, y_ref) and torch.equal(hl, h_ref), f"replay {i}"
    # the refused calls, eagerly again, give what they gave before the capture
    def parts(v):
        if isinstance(v, dict):
            return [v[k] for k in sorted(v)]
        return [t for t in (v if isinstance(v, (tuple, list)) else (v,)) if t is not None]

    for name, fn in refused.items():
        got = parts(fn())
        torch.cuda.synchronize()
        ref = parts(eager[name])
        assert len(got) == len(ref) and len(got) > 0, name
        for gi, ri in zip(got, ref):
            assert torch.equal(gi, ri), name


def test_noalloc_scan_graph_replays_match_eager(sw):
    """The bare scan through the entry point that allocates nothing, on its
    segments (three rows of 40 chunks: records and tickets in the
    library's static array, cleared by a fill kernel at every call), captured
    into a HIP graph: every replay, with eager calls of both bare-scan entry
    points between the replays, gives the eager result bit for bit.  The
    inputs keep every partial composition an integer below 2^24 (a in {0, 1},
    small integer bx), exact in fp32 in any association order, so the
    cuts cannot change a bit."""
    B, D, L = 1, 3, 40 * 2048 - 5
    _say("case graph replay noalloc", B, D, L)
    g_ = np.random.default_rng(780)
    a_np = (g_.random((B, D, L)) < 0.9995).astype(np.float32)
    bx_np = g_.integers(-8, 9, (B, D, L)).astype(np.float32)
    a = torch.from_numpy(a_np).to("cuda")
    bx = torch.from_numpy(bx_np).to("cuda")
    h_ref = sw.affine_scan_noalloc(a, bx)  # also looks up the static array's address
    torch.cuda.synchronize()
    assert torch.equal(h_ref, sw.affine_scan(a, bx))
    h = torch.empty_like(h_ref)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):  # warm-up on the capture stream
        sw.affine_scan_noalloc(a, bx, out=h)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        sw.affine_scan_noalloc(a, bx, out=h)
    for i in range(4):
        h.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(h, h_ref), f"replay {i}: h differs"
        # eager work of the program between replays, on the same static array
        h2 = sw.affine_scan_noalloc(a, bx)
        h3 = sw.affine_scan(a, bx)
        torch.cuda.synchronize()
        assert torch.equal(h2, h_ref) and torch.equal(h3, h_ref)
    assert np.array_equal(h_ref.cpu().numpy()[:, :1, :4096],
                          oracle.affine_scan(a_np[:, :1, :4096], bx_np[:, :1, :4096]))
