"""The work that users of this framework have it do, as measured cases.

Every case goes through the package's public functions:

* ``scan``: ``affine_scan`` / ``affine_scan_i32``, the bare recurrence of
  linear attention and gated RNN layers (and, in int32, of exact rolling
  hashes and counters) over (B, D, L);
* ``proj``: ``affine_scan_proj``, the elementwise form with input and output
  projections and an initial state;
* ``fwd``: ``selective_scan_fwd``, a Mamba layer's scan over a prompt; plain,
  or (``block``) with everything a Mamba block fuses into it: output gate,
  delta bias, softplus, and y in the inputs' type;
* ``decode``: ``selective_scan_fwd`` one token at a time, the state carried
  through ``h0`` and ``h_last``;
* ``train``: ``selective_scan_fn`` forward and its gradients through autograd.

Sizes are those of the repository's workloads, tests and ablations (D = 768 to
5120, N = 16, L = 512 to 65536) and ragged ones beside them: prompts have any
length.  Values follow the generators in ``workloads``: decay in [0.9, 1) for
the bare scan, delta around 0.02 and A in [-16, -1] for the selective scan.
"""
import math

import torch
import torch.nn.functional as F

import paper_2606_00601_amd as sw

_MOST = 1.0e9  # (b,d,t,n) elements of a drawn selective case


def listed():
    return [
        # the smallest call: a short sequence of one head, launch-sized
        {"name": "scan_small", "kind": "scan", "dtype": "f32", "B": 1, "D": 64, "L": 1024},
        # a layer's bare recurrence over a batch: many rows of a common length
        {"name": "scan_rows", "kind": "scan", "dtype": "f32", "B": 8, "D": 1536, "L": 2048},
        # few rows of a long sequence, exact ring arithmetic
        {"name": "scan_few_long", "kind": "scan", "dtype": "i32", "B": 1, "D": 64, "L": 65536},
        # projections and an initial state, at a ragged length
        {"name": "proj_ragged", "kind": "proj", "dtype": "f32", "B": 2, "D": 1000, "L": 3001},
        # a small model's layer over a short prompt
        {"name": "fwd_small", "kind": "fwd", "dtype": "f32", "B": 2, "D": 256, "N": 16, "L": 512,
         "block": False},
        # the usual batch of a 130M-sized model in bf16
        {"name": "fwd_bf16", "kind": "fwd", "dtype": "bf16", "B": 8, "D": 1536, "N": 16,
         "L": 2048, "block": False},
        # the largest: one long document through a wide layer in fp32
        {"name": "fwd_long", "kind": "fwd", "dtype": "f32", "B": 1, "D": 5120, "N": 16,
         "L": 65536, "block": False},
        # a Mamba block's scan over prompts of a length that nothing divides
        {"name": "fwd_block_ragged", "kind": "fwd", "dtype": "bf16", "B": 4, "D": 2048, "N": 16,
         "L": 1999, "block": True},
        # the largest state the operation takes
        {"name": "fwd_n64", "kind": "fwd", "dtype": "f32", "B": 2, "D": 1024, "N": 64, "L": 1024,
         "block": False},
        # serving: one token for every sequence of a batch, through a wide block
        {"name": "decode", "kind": "decode", "dtype": "bf16", "B": 64, "D": 5120, "N": 16, "L": 1,
         "block": True},
        # a training step of the usual batch: forward, every gradient
        {"name": "train_bf16", "kind": "train", "dtype": "bf16", "B": 8, "D": 1536, "N": 16,
         "L": 2048, "block": True},
        # fine-tuning on one ragged sequence in fp32
        {"name": "train_ragged", "kind": "train", "dtype": "f32", "B": 1, "D": 1000, "N": 16,
         "L": 1501, "block": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _length(rng, lo, hi):
    """Any length, or one a program pads to."""
    n = _log(rng, lo, hi)
    return n if rng.random() < 0.5 else max(lo, n // 64 * 64)


def _width(rng, lo, hi):
    """Any width, or a model's."""
    if rng.random() < 0.3:
        return _log(rng, lo, hi)
    return rng.choice([d for d in (256, 512, 768, 1024, 1536, 2048, 2560, 5120) if lo <= d <= hi])


def draw(rng):
    kind = rng.choice(["scan", "proj", "fwd", "fwd", "fwd", "decode", "train", "train"])
    if kind in ("scan", "proj"):
        L = _length(rng, 64, 65536)
        rows = _log(rng, 16, max(17, min(16384, 60_000_000 // L)))
        B = min(rng.choice([1, 1, 2, 4, 8]), rows)
        return {"kind": kind, "dtype": rng.choice(["f32", "f32", "i32"]), "B": B,
                "D": rows // B, "L": L}
    dtype = rng.choice(["f32", "bf16", "bf16"])
    if kind == "decode":
        return {"kind": kind, "dtype": dtype, "B": _log(rng, 1, 256), "D": _width(rng, 256, 5120),
                "N": 16, "L": 1, "block": True}
    N = 16 if rng.random() < 0.75 else rng.choice([4, 8, 24, 32, 48, 64])
    D = _width(rng, 200, 5120)
    B = rng.choice([1, 1, 2, 4, 8, 16])
    most = _MOST if kind == "fwd" else 0.4 * _MOST
    L = _length(rng, 64, int(max(128, min(32768, most / (B * D * N)))))
    return {"kind": kind, "dtype": dtype, "B": B, "D": D, "N": N, "L": L,
            "block": rng.random() < 0.5}


def _affine_inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, D, L = case["B"], case["D"], case["L"]
    proj = case["kind"] == "proj"
    s = {}
    if case["dtype"] == "i32":
        def ints(*shape):
            return torch.randint(-2 ** 31, 2 ** 31, shape, generator=g, device="cuda",
                                 dtype=torch.int64).to(torch.int32)
        s["a"], s["bx"] = ints(B, D, L), ints(B, D, L)
        if proj:
            s["x"], s["c"], s["h0"] = ints(B, D, L), ints(B, D, L), ints(B, D)
        return s
    f32 = dict(generator=g, device="cuda", dtype=torch.float32)
    s["a"] = (0.9 + 0.1 * torch.rand(B, D, L, **f32)).clamp_(max=1.0 - 2.0 ** -24)
    s["bx"] = torch.randn(B, D, L, **f32)
    if proj:
        s["x"], s["c"] = torch.randn(B, D, L, **f32), torch.randn(B, D, L, **f32)
        s["h0"] = torch.randn(B, D, **f32)
    return s


def _selective_inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, D, N, L = case["B"], case["D"], case["N"], case["L"]
    f32 = dict(generator=g, device="cuda", dtype=torch.float32)
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    s = {"x": torch.randn(B, D, L, **f32).to(dt)}
    raw = torch.randn(B, D, L, **f32).mul_(0.5)
    if case["block"]:
        # delta before bias and softplus; the bias holds the mean of -4
        s["delta"] = raw.to(dt)
    else:
        s["delta"] = F.softplus(raw.sub_(4.0)).to(dt)
    del raw
    s["A"] = -torch.exp(torch.rand(D, N, **f32) * math.log(16.0))
    s["Bm"] = torch.randn(B, L, N, **f32).to(dt)
    s["Cm"] = torch.randn(B, L, N, **f32).to(dt)
    s["Dskip"] = torch.randn(D, **f32)
    s["z"] = s["delta_bias"] = s["h0"] = None
    if case["block"]:
        s["z"] = torch.randn(B, D, L, **f32).to(dt)
        s["delta_bias"] = torch.randn(D, **f32).mul_(0.1).sub_(4.0)
    if case["kind"] == "decode":
        s["h0"] = torch.randn(B, D, N, **f32)
    if case["kind"] == "train":
        s["dy"] = torch.randn(B, D, L, **f32)
    return s


_GRADS = ("x", "delta", "A", "Bm", "Cm", "Dskip", "z", "delta_bias")


def prepare(case, seed):
    if case["kind"] in ("scan", "proj"):
        s = _affine_inputs(case, seed)
    else:
        s = _selective_inputs(case, seed)
    if case["kind"] == "train":
        s["wrt"] = [s[k].requires_grad_(True) for k in _GRADS if s[k] is not None]
    s["case"] = case
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "scan":
        fn = sw.affine_scan if case["dtype"] == "f32" else sw.affine_scan_i32
        return fn(s["a"], s["bx"])
    if kind == "proj":
        fn = sw.affine_scan_proj if case["dtype"] == "f32" else sw.affine_scan_proj_i32
        return fn(s["a"], s["bx"], s["x"], s["c"], s["h0"])
    if kind == "train":
        y = sw.selective_scan_fn(s["x"], s["delta"], s["A"], s["Bm"], s["Cm"], s["Dskip"],
                                 z=s["z"], delta_bias=s["delta_bias"],
                                 delta_softplus=case["block"])
        return (y.detach(), *torch.autograd.grad(y, s["wrt"], s["dy"]))
    if case["block"]:
        return sw.selective_scan_fwd(s["x"], s["delta"], s["A"], s["Bm"], s["Cm"], s["Dskip"],
                                     z=s["z"], delta_bias=s["delta_bias"], h0=s["h0"],
                                     delta_softplus=True, y_dtype=s["x"].dtype)
    return sw.selective_scan_fwd(s["x"], s["delta"], s["A"], s["Bm"], s["Cm"], s["Dskip"])


def work(case):
    B, D, L = case["B"], case["D"], case["L"]
    R = B * D
    if case["kind"] == "scan":
        return {"bytes": 12 * R * L, "flops": 2 * R * L}
    if case["kind"] == "proj":
        return {"bytes": 20 * R * L + 8 * R, "flops": 4 * R * L}
    N = case["N"]
    es = 4 if case["dtype"] == "f32" else 2
    block = case["block"]
    shared = 2 * B * L * N * es + D * N * 4 + 4 * D + (4 * D if block else 0)
    rows = R * L * es * (3 if block else 2)  # x, delta (and z)
    elems = R * L * N
    if case["kind"] == "train":
        # the inputs, dy and y once, every gradient in its input's type
        return {"bytes": 2 * (shared + rows) + 8 * R * L, "flops": 20 * elems}
    ys = es if block else 4
    state = 4 * R * N * (2 if case["kind"] == "decode" else 1)
    return {"bytes": shared + rows + ys * R * L + state, "flops": 6 * elems}


def tolerance(case):
    if case["dtype"] == "i32":
        return "exact"
    if case["kind"] in ("scan", "proj"):
        return {"rel": 1e-6, "max": 1e-5}
    if case["dtype"] == "bf16" and (case["block"] or case["kind"] == "train"):
        # outputs in bf16: one rounding, at half a unit of the last of 8 bits
        return {"rel": 4e-3, "max": 1.6e-2}
    if case["kind"] == "train":
        # fp32 sums over a batch and a sequence: 1.2e-6 from 64 bits at most as measured (dA)
        return {"rel": 5e-6, "max": 1e-4}
    return {"rel": 1e-6, "max": 2e-5}  # 1.2e-7 from 64 bits as measured


# ---- the same in 64 bits, plain torch


def _steps_first(t):
    return t.double().permute(2, 0, 1).contiguous()


def _exact_affine(case, s):
    a, u = _steps_first(s["a"]), _steps_first(s["bx"])
    if "x" in s:
        u *= _steps_first(s["x"])
    h = s["h0"].double() if "h0" in s else torch.zeros_like(u[0])
    for t in range(a.shape[0]):
        h = torch.addcmul(u[t], a[t], h, out=u[t])
    last = h.clone()
    if "c" in s:
        u *= _steps_first(s["c"])
    y = u.permute(1, 2, 0).contiguous()
    return (y, last) if case["kind"] == "proj" else y


def _exact_selective(case, s):
    B, D, N, L = case["B"], case["D"], case["N"], case["L"]
    train = case["kind"] == "train"
    raw = s["delta"].detach().permute(2, 0, 1).contiguous()
    x = s["x"].detach().permute(2, 0, 1).contiguous()
    z = s["z"].detach().permute(2, 0, 1).contiguous() if s["z"] is not None else None
    Bm, Cm = (s[k].detach().transpose(0, 1).contiguous() for k in ("Bm", "Cm"))  # (L, B, N)
    A, Dskip = s["A"].detach().double(), s["Dskip"].detach().double()
    bias = s["delta_bias"].detach().double() if s["delta_bias"] is not None else 0.0

    def delta_of(i, j):
        v = raw[i:j].double() + bias
        return F.softplus(v, threshold=700.0) if case["block"] else v

    chunk = max(1, min(L, 60_000_000 // (B * D * N)))
    parts = [(i, min(L, i + chunk)) for i in range(0, L, chunk)]
    h = (s["h0"].double() if s["h0"] is not None
         else torch.zeros(B, D, N, dtype=torch.float64, device="cuda"))
    y = torch.empty(B, D, L, dtype=torch.float64, device="cuda")
    starts = []
    for i, j in parts:
        starts.append(h)
        dl = delta_of(i, j)
        a = torch.exp(dl.unsqueeze(-1) * A)
        H = (dl * x[i:j].double()).unsqueeze(-1) * Bm[i:j].double().unsqueeze(2)
        for t in range(j - i):
            h = torch.addcmul(H[t], a[t], h, out=H[t])
        h = h.clone()
        del a
        o = H.mul_(Cm[i:j].double().unsqueeze(2)).sum(-1) + Dskip * x[i:j].double()
        if z is not None:
            o = o * F.silu(z[i:j].double())
        y[:, :, i:j] = o.permute(1, 2, 0)
        del H
    if not train:
        return y, h
    # gradients, the chunks in reverse with the states of each rebuilt
    dy = s["dy"].permute(2, 0, 1).contiguous()
    new = lambda *shape: torch.zeros(*shape, dtype=torch.float64, device="cuda")  # noqa: E731
    dx, dd = new(L, B, D), new(L, B, D)
    dz = new(L, B, D) if z is not None else None
    dA, dB, dC, dDs = new(D, N), new(L, B, N), new(L, B, N), new(D)
    carry = new(B, D, N)  # a_{t+1} lam_{t+1}
    for (i, j), h in reversed(list(zip(parts, starts))):
        dl, xv = delta_of(i, j), x[i:j].double()
        bm, cm = Bm[i:j].double().unsqueeze(2), Cm[i:j].double().unsqueeze(2)
        a = torch.exp(dl.unsqueeze(-1) * A)
        H = (dl * xv).unsqueeze(-1) * bm
        prev = torch.empty_like(H)
        for t in range(j - i):
            prev[t] = h
            h = torch.addcmul(H[t], a[t], h, out=H[t])
        ds = dy[i:j].double()
        if z is not None:
            zv = z[i:j].double()
            sg = torch.sigmoid(zv)
            pre = (H * cm).sum(-1) + Dskip * xv
            dz[i:j] = ds * pre * sg * (1.0 + zv * (1.0 - sg))
            ds = ds * zv * sg
        dC[i:j] = (ds.unsqueeze(-1) * H).sum(2)
        dDs += (ds * xv).sum((0, 1))
        lam = H.copy_(ds.unsqueeze(-1) * cm)
        for t in range(j - i - 1, -1, -1):
            lam[t] += carry
            torch.mul(a[t], lam[t], out=carry)
        dB[i:j] = (lam * (dl * xv).unsqueeze(-1)).sum(2)
        lb = (lam * bm).sum(-1)
        dx[i:j] = dl * lb + ds * Dskip
        q = prev.mul_(a).mul_(lam)  # lam a h_{t-1}
        dA += (q * dl.unsqueeze(-1)).sum((0, 1))
        dd[i:j] = (q * A).sum(-1) + xv * lb
        del a, H, prev, lam, q
    if case["block"]:
        dd *= torch.sigmoid(raw.double() + bias)
    back = lambda t: t.permute(1, 2, 0).contiguous()  # noqa: E731
    out = [y, back(dx), back(dd), dA, dB.transpose(0, 1).contiguous(),
           dC.transpose(0, 1).contiguous(), dDs]
    if z is not None:
        out.append(back(dz))
    if s["delta_bias"] is not None:
        out.append(dd.sum((0, 1)))
    return tuple(out)


def exact(case, seed):
    if case["dtype"] == "i32":
        return None
    with torch.no_grad():
        if case["kind"] in ("scan", "proj"):
            return _exact_affine(case, _affine_inputs(case, seed))
        return _exact_selective(case, _selective_inputs(case, seed))
