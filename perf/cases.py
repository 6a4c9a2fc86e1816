"""Workloads of the structure-tensor library, sized and filled as its users meet them.

A case is a dict of plain values; ``kind`` selects the entry point:

  tensor     ``st_compute`` with the outputs and workspace kept by the caller
  noalloc    ``st_compute_noalloc`` (serving loops over small crops)
  angles     ``st_angles`` (a fibre field re-angled about another axis)
  batch      ``Batch.launch`` of uneven halo-padded chunks
  surrogate  ``st_surrogate_infer`` with the shipped weights, alone or with fallback
  train      ``st_surrogate_grad`` on a stack of patches

``listed`` and ``draw`` give the cases, ``prepare`` what a program holds before
the call, ``run`` one pass through the entry point, ``work`` the bytes and
operations one pass cannot do without, and ``exact`` the same outputs from
plain torch in float64.
"""

from __future__ import annotations

import math
import os

import numpy as np
import torch

import paper_2508_07476_amd as st

TRUNCATE = 4.0
PERIOD = 4.0                     # rod spacing of the synthetic tissue (voxels)
DIRECTION = (1.0, 0.04, -0.03)   # long axis, slightly tilted (z, y, x)
OUTPUTS = {
    "maps": ("e3", "fa", "ha", "ia"),
    "default": ("e3", "fa", "ha", "ia", "flags"),
    "all": ("e3", "evals", "fa", "ha", "ia", "flags"),
}
TAPS = [(t // 9 - 1, (t // 3) % 3 - 1, t % 3 - 1) for t in range(27)]


# ---- cases -------------------------------------------------------------------

def listed():
    return [
        # the smallest whole call: 64^3 float32, the parity configuration
        _tensor("tensor_64_f32", 64, 64, 64, "f32", 1.0, 3.0, False, "default"),
        # one crop of a serving loop that must not allocate, odd sides, mask
        {"name": "noalloc_93x101x77_u16", "kind": "noalloc", "nz": 93, "ny": 101, "nx": 77, "dtype": "u16",
         "sigma": 1.0, "rho": 2.0, "mask": True, "outputs": "default"},
        # an ordinary chunk of a scan with ragged sides and every output
        _tensor("tensor_ragged_u16", 151, 210, 333, "u16", 1.5, 4.0, True, "all"),
        # 512^3 uint16 with its tissue mask, the usual scales
        _tensor("tensor_512_u16", 512, 512, 512, "u16", 1.5, 4.0, True, "maps"),
        # the largest: half a gigavoxel without a mask at the coarse scales
        _tensor("tensor_512x1024x1024_u16", 512, 1024, 1024, "u16", 2.0, 6.0, False, "maps"),
        # scales beyond the fused gradient's radius, on a float32 reconstruction
        _tensor("tensor_coarse_f32", 190, 226, 250, "f32", 3.0, 8.0, False, "default"),
        # a stored fibre field re-angled about a corrected axis
        {"name": "angles_250x510x509", "kind": "angles", "nz": 250, "ny": 510, "nx": 509, "mask": True},
        # chunk processing with halos: uneven chunks, three integration scales
        {"name": "batch_12_chunks", "kind": "batch", "chunks": 12, "lo": 64, "hi": 384, "pick": 4, "sigma": 1.0},
        # learned surrogate on one small crop (launches and latency)
        _surrogate("surrogate_48", 48, 48, 48, "u16", False, 0.0),
        # learned surrogate alone on a block of a scan
        _surrogate("surrogate_256x320x384", 256, 320, 384, "u16", True, 0.0),
        # learned surrogate with the tensor path wherever it is unsure
        _surrogate("surrogate_fallback_192x256x250", 192, 256, 250, "u16", True, 0.9),
        # one training step's gradient: the trainer's 32 patches of 32^3
        {"name": "train_32x32", "kind": "train", "patches": 32, "edge": 32, "dtype": "u16"},
    ]


def draw(rng):
    kind = rng.choice(["tensor", "tensor", "tensor", "noalloc", "angles", "batch", "surrogate", "surrogate", "train"])

    def side(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def shape(lo, hi, most):
        while True:
            s = [side(lo, hi) for _ in range(3)]
            if s[0] * s[1] * s[2] <= most:
                return s

    if kind == "tensor":
        nz, ny, nx = shape(24, 900, 1 << 28)
        return _tensor(None, nz, ny, nx, rng.choice(["u16", "u16", "f32"]), rng.choice([0.8, 1.0, 1.5, 2.0, 2.6, 3.0]),
                       rng.choice([2.0, 3.0, 4.0, 6.0, 8.0]), rng.random() < 0.5, rng.choice(sorted(OUTPUTS)))
    if kind == "noalloc":
        nz, ny, nx = shape(32, 120, 1 << 20)
        return {"kind": "noalloc", "nz": nz, "ny": ny, "nx": nx, "dtype": rng.choice(["u16", "f32"]),
                "sigma": rng.choice([1.0, 1.5, 2.0]), "rho": rng.choice([2.0, 3.0, 4.0]), "mask": rng.random() < 0.5,
                "outputs": "default"}
    if kind == "angles":
        nz, ny, nx = shape(40, 700, 1 << 27)
        return {"kind": "angles", "nz": nz, "ny": ny, "nx": nx, "mask": rng.random() < 0.5}
    if kind == "batch":
        return {"kind": "batch", "chunks": rng.randint(3, 12), "lo": rng.randint(40, 80), "hi": rng.randint(120, 384),
                "pick": rng.randint(5, 1 << 20), "sigma": rng.choice([1.0, 1.5])}
    if kind == "surrogate":
        nz, ny, nx = shape(40, 400, 1 << 25)
        return _surrogate(None, nz, ny, nx, rng.choice(["u16", "u16", "f32"]), rng.random() < 0.7,
                          rng.choice([0.0, 0.0, 0.9, 0.5]))
    return {"kind": "train", "patches": rng.randint(4, 48), "edge": rng.randint(16, 32), "dtype": rng.choice(["u16", "f32"])}


def _tensor(name, nz, ny, nx, dtype, sigma, rho, mask, outputs):
    c = {"kind": "tensor", "nz": nz, "ny": ny, "nx": nx, "dtype": dtype, "sigma": sigma, "rho": rho, "mask": mask,
         "outputs": outputs}
    return c if name is None else dict(c, name=name)


def _surrogate(name, nz, ny, nx, dtype, mask, min_confidence):
    c = {"kind": "surrogate", "nz": nz, "ny": ny, "nx": nx, "dtype": dtype, "mask": mask,
         "min_confidence": min_confidence, "sigma": 1.0, "rho": 2.0}
    return c if name is None else dict(c, name=name)


# ---- inputs ------------------------------------------------------------------

def _tissue(shape, dtype, seed, annulus, period=PERIOD, noise=0.05, fibre=False):
    """A helical rod lattice about the z axis of the volume (helix angle +60 to
    -60 degrees across the wall) with noise.  ``annulus``: tissue only at 0.19 to
    0.44 of the in-plane size, zeros elsewhere, with its mask; else tissue
    everywhere.  Returns volume, mask (or None), centre and, with ``fibre``, the
    true fibre field."""
    dev = torch.device("cuda")
    nz, ny, nx = shape
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    cz, cy, cx = ((n - 1) / 2.0 for n in shape)
    size = float(min(ny, nx))
    r_in, r_out = (0.1875 * size, 0.4375 * size) if annulus else (0.0, 0.5 * math.hypot(ny, nx) + period)
    y = (torch.arange(ny, device=dev, dtype=torch.float32) - cy).view(1, ny, 1)
    x = (torch.arange(nx, device=dev, dtype=torch.float32) - cx).view(1, 1, nx)
    r = torch.sqrt(y * y + x * x)
    theta = torch.atan2(y, x)
    rm = r_in + (torch.floor((r - r_in) / period).clamp_min(0.0) + 0.5) * period
    alpha = math.radians(60.0) * (1.0 - 2.0 * ((rm - r_in) / (r_out - r_in)).clamp(0.0, 1.0))
    inside = (r >= r_in) & (r <= r_out)
    vol = torch.empty(shape, device=dev, dtype=torch.float32 if dtype == "f32" else torch.uint16)
    slab = max(1, (1 << 25) // (ny * nx))
    for a in range(0, nz, slab):
        b = min(nz, a + slab)
        z = (torch.arange(a, b, device=dev, dtype=torch.float32) - cz).view(-1, 1, 1)
        u = z * torch.cos(alpha) - rm * theta * torch.sin(alpha)
        u = torch.remainder(u + 0.5 * period, period) - 0.5 * period
        v = 0.5 + 0.4 * torch.sin((2.0 * math.pi / period) * torch.sqrt(u * u + (r - rm) ** 2))
        v += noise * torch.randn(v.shape, generator=gen, device=dev)
        if annulus:
            v *= inside
        vol[a:b] = v if dtype == "f32" else (v.clamp_(0.0, 1.0) * 65535.0).round_().to(torch.int32).to(torch.uint16)
    mask = inside.expand(nz, ny, nx).to(torch.uint8).contiguous() if annulus else None
    out = [vol, mask, (cz, cy, cx)]
    if fibre:
        rr = r.clamp_min(1.0)
        f = torch.stack([torch.sin(alpha), torch.cos(alpha) * x / rr, -torch.cos(alpha) * y / rr])
        f = f / f.norm(dim=0, keepdim=True).clamp_min(1e-6)
        out.append(f.expand(3, nz, ny, nx).contiguous())
    return out


def _like(names, shape):
    out = {}
    for k in names:
        s = (3,) + tuple(shape) if k in ("e3", "evals") else tuple(shape)
        out[k] = torch.empty(s, device="cuda", dtype=torch.uint8 if k == "flags" else torch.float32)
    return out


def _weights():
    path = os.path.join(os.path.dirname(st.__file__), "surrogate_weights.npy")
    return torch.from_numpy(np.load(path)).cuda()


def _chunks(case):
    """(shape, rho) of every chunk: interior sides uniform in [lo, hi], a halo of
    3 rho on every side."""
    rng = np.random.default_rng(case["pick"])
    got = []
    for _ in range(case["chunks"]):
        rho = float(rng.choice((2.0, 3.0, 4.0)))
        got.append((tuple(int(s) + 2 * int(round(3 * rho)) for s in rng.integers(case["lo"], case["hi"] + 1, size=3)), rho))
    return got


def _shape(case):
    return case["nz"], case["ny"], case["nx"]


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("tensor", "noalloc"):
        shape = _shape(case)
        vol, mask, centre = _tissue(shape, case["dtype"], seed, case["mask"])
        names = OUTPUTS[case["outputs"]]
        s = {"case": case, "volume": vol, "mask": mask, "centre": centre, "names": names, "out": _like(names, shape)}
        if kind == "tensor":
            s["workspace"] = torch.empty(st.st_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
        return s
    if kind == "angles":
        shape = _shape(case)
        _, mask, centre, fibre = _tissue(shape, "u16", seed, case["mask"], fibre=True)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(int(seed))
        fibre += 0.1 * torch.randn(fibre.shape, generator=gen, device="cuda")
        return {"case": case, "e3": fibre, "mask": mask, "centre": tuple(c + 1.5 for c in centre),
                "out": _like(("ha", "ia"), shape)}
    if kind == "batch":
        chunks = []
        for i, (shape, rho) in enumerate(_chunks(case)):
            vol, mask, _ = _tissue(shape, "u16", seed * 1000 + i, i % 2 == 0)
            chunks.append({"volume": vol, "mask": mask, "rho": rho, "origin": (13.0 * i, 7.0 * i, -5.0 * i)})
        batch = st.Batch(chunks, sigma=case["sigma"], truncate=TRUNCATE, axis_center=(120.0, 130.5, 140.0),
                         axis_direction=DIRECTION, outputs=OUTPUTS["default"])
        return {"case": case, "batch": batch, "chunks": chunks}
    if kind == "surrogate":
        shape = _shape(case)
        vol, mask, centre = _tissue(shape, case["dtype"], seed, case["mask"], period=5.0)
        if case["dtype"] == "f32":
            vol *= 65535.0  # the intensity range of the weights
        return {"case": case, "volume": vol, "mask": mask, "centre": centre, "weights": _weights(),
                "out": _like(st.SURROGATE_OUTPUTS, shape)}
    P, n = case["edge"], case["patches"]
    shape = (n * P, P, P)
    vol, _, _, fibre = _tissue(shape, case["dtype"], seed, False, fibre=True)
    if case["dtype"] == "f32":
        vol *= 65535.0
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    core = torch.zeros((n, P, P, P), dtype=torch.uint8, device="cuda")
    core[:, 5:P - 5, 5:P - 5, 5:P - 5] = 1
    core *= torch.rand(core.shape, generator=gen, device="cuda") < 0.9  # degenerate voxels carry no loss
    return {"case": case, "patches": vol, "target": fibre, "weight": core.view(shape),
            "fa": 0.6 + 0.3 * torch.rand(shape, generator=gen, device="cuda"), "params": _weights(),
            "grad": torch.empty(st.ST_SURROGATE_WEIGHTS, device="cuda"), "stats": torch.empty(8, device="cuda"),
            "workspace": torch.empty(st.st_surrogate_grad_workspace_bytes(n, P), dtype=torch.uint8, device="cuda")}


# ---- one pass ----------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "tensor":
        return st.st_compute(state["volume"], case["sigma"], case["rho"], TRUNCATE, mask=state["mask"],
                             axis_center=state["centre"], axis_direction=DIRECTION, outputs=state["names"],
                             out=state["out"], workspace=state["workspace"])
    if kind == "noalloc":
        return st.st_compute_noalloc(state["volume"], case["sigma"], case["rho"], TRUNCATE, mask=state["mask"],
                                     axis_center=state["centre"], axis_direction=DIRECTION, outputs=state["names"],
                                     out=state["out"])
    if kind == "angles":
        return st.st_angles(state["e3"], state["centre"], DIRECTION, mask=state["mask"], out=state["out"])
    if kind == "batch":
        state["batch"].launch()
        return state["batch"].results
    if kind == "surrogate":
        return st.st_surrogate_infer(state["volume"], state["weights"], min_confidence=case["min_confidence"],
                                     sigma=case["sigma"], rho=case["rho"], truncate=TRUNCATE, mask=state["mask"],
                                     axis_center=state["centre"], axis_direction=DIRECTION,
                                     outputs=st.SURROGATE_OUTPUTS, out=state["out"])
    grad, stats = st.st_surrogate_grad(state["patches"], state["target"], state["fa"], state["weight"],
                                       state["params"], grad=state["grad"], stats=state["stats"],
                                       workspace=state["workspace"])
    return {"grad": grad, "stats": stats}


# ---- what a pass cannot do without -------------------------------------------

def _radius(scale):
    return int(math.floor(TRUNCATE * scale + 0.5))


def _tensor_work(n, dtype, mask, names, sigma, rho):
    size = {"e3": 12, "evals": 12, "fa": 4, "ha": 4, "ia": 4, "flags": 1}
    # eight 1-D gradient filters, six products, eighteen 1-D integrations, the eigen-solve and angles
    ops = 8 * (2 * _radius(sigma) + 1) + 6 + 18 * (2 * _radius(rho) + 1) + 220
    return n * ((2 if dtype == "u16" else 4) + (1 if mask else 0) + sum(size[k] for k in names)), 2.0 * n * ops


def work(case):
    kind = case["kind"]
    if kind == "batch":
        b = f = 0.0
        for i, (s, rho) in enumerate(_chunks(case)):
            w = _tensor_work(s[0] * s[1] * s[2], "u16", i % 2 == 0, OUTPUTS["default"], case["sigma"], rho)
            b, f = b + w[0], f + w[1]
        return {"bytes": b, "flops": f}
    if kind == "train":
        n = case["patches"] * case["edge"] ** 3
        # forward and weight gradient of five layers, data gradient of four, the head both ways
        macs = 2 * 27 * 32 + 3 * 4 * 27 * 1024 + 3 * 160
        return {"bytes": n * ((2 if case["dtype"] == "u16" else 4) + 17) + 8.0 * st.ST_SURROGATE_WEIGHTS,
                "flops": 2.0 * n * macs}
    n = case["nz"] * case["ny"] * case["nx"]
    if kind == "angles":
        return {"bytes": n * (12 + 8 + (1 if case["mask"] else 0)), "flops": 130.0 * n}
    if kind == "surrogate":
        b = n * ((2 if case["dtype"] == "u16" else 4) + (1 if case["mask"] else 0) + 28) + 4.0 * st.ST_SURROGATE_WEIGHTS
        return {"bytes": b, "flops": 2.0 * n * (27 * 32 + 4 * 27 * 1024 + 160)}
    b, f = _tensor_work(n, case["dtype"], case["mask"], OUTPUTS[case["outputs"]], case["sigma"], case["rho"])
    return {"bytes": b, "flops": f}


# ---- the same outputs in float64, from torch alone ----------------------------

def _filter(x, w, axis):
    """Correlation of x with taps w along an axis, half-sample symmetric faces."""
    R, n = len(w) // 2, x.shape[axis]
    i = torch.arange(-R, n + R, device=x.device).remainder(2 * n)
    xp = x.index_select(axis, torch.where(i < n, i, 2 * n - 1 - i))
    y = w[0] * xp.narrow(axis, 0, n)
    for k in range(1, len(w)):
        y.add_(xp.narrow(axis, k, n), alpha=w[k])
    return y


def _gauss(s):
    R = _radius(s)
    k = np.arange(-R, R + 1, dtype=np.float64)
    g = np.exp(-k * k / (2.0 * s * s))
    g /= g.sum()
    return [float(v) for v in g], [float(v) for v in k / (s * s) * g]


def _jacobi(a):
    """Eigenvalues and vectors of symmetric 3x3 fields: a maps (i, j), i <= j, to
    a flat float64 tensor.  Returns three values and a 3 x 3 list (columns)."""
    m = dict(a)
    one, zero = torch.ones_like(a[0, 0]), torch.zeros_like(a[0, 0])
    v = [[one.clone() if i == j else zero.clone() for j in range(3)] for i in range(3)]
    for _ in range(6):
        for p, q in ((0, 1), (0, 2), (1, 2)):
            apq = m[p, q]
            th = (m[q, q] - m[p, p]) / (2.0 * apq)
            t = torch.where(th < 0, -1.0, 1.0) / (th.abs() + torch.sqrt(th * th + 1.0))
            t = torch.where((apq != 0) & torch.isfinite(th), t, zero)
            c = 1.0 / torch.sqrt(t * t + 1.0)
            s = t * c
            r = 3 - p - q
            pr, qr = (min(p, r), max(p, r)), (min(q, r), max(q, r))
            m[p, p], m[q, q], m[p, q] = m[p, p] - t * apq, m[q, q] + t * apq, zero
            m[pr], m[qr] = c * m[pr] - s * m[qr], s * m[pr] + c * m[qr]
            for i in range(3):
                v[i][p], v[i][q] = c * v[i][p] - s * v[i][q], s * v[i][p] + c * v[i][q]
    return [m[i, i] for i in range(3)], v


def _canonical(e):
    a = [c.abs() for c in e]
    lead = torch.where((a[0] >= a[1]) & (a[0] >= a[2]), e[0], torch.where(a[1] >= a[2], e[1], e[2]))
    sign = torch.where(lead < 0, -1.0, 1.0)
    return [c * sign for c in e]


def _frame_angles(e, centre, direction, z0, shape):
    """HA and IA of the field e (z, y, x components of the planes from z0 on)."""
    dev = e[0].device
    d = np.asarray(direction, dtype=np.float64)
    a = [float(v) for v in d / np.linalg.norm(d)]
    q = [(torch.arange(n, device=dev, dtype=torch.float64) + (z0 if i == 0 else 0) - centre[i]).view(
        [-1 if i == j else 1 for j in range(3)]) for i, n in enumerate(shape)]
    qa = q[0] * a[0] + q[1] * a[1] + q[2] * a[2]
    f = [q[i] - qa * a[i] for i in range(3)]
    r = torch.sqrt(f[0] ** 2 + f[1] ** 2 + f[2] ** 2)
    tz, ty, tx = a[2] * f[1] - a[1] * f[2], a[0] * f[2] - a[2] * f[0], a[1] * f[0] - a[0] * f[1]
    on = r < 1e-9
    rs = torch.where(on, 1.0, r)
    fr = (e[0] * f[0] + e[1] * f[1] + e[2] * f[2]) / rs
    ft = (e[0] * tz + e[1] * ty + e[2] * tx) / rs
    fa = e[0] * a[0] + e[1] * a[1] + e[2] * a[2]
    sg = torch.where(ft >= 0, 1.0, -1.0)
    ha, ia = torch.atan2(fa * sg, ft.abs()), torch.atan2(fr * sg, ft.abs())
    return ha.masked_fill(on, 0.0), ia.masked_fill(on, 0.0)


def _tensor64(vol, mask, sigma, rho, centre, direction, names):
    """The whole path in float64, in z slabs with their exact reach of context."""
    nz, ny, nx = vol.shape
    g0, g1 = _gauss(sigma)
    w0, _ = _gauss(rho)
    rr = _radius(rho)
    halo = _radius(sigma) + rr
    out = {k: torch.empty(((3,) if k in ("e3", "evals") else ()) + (nz, ny, nx), dtype=torch.float64, device=vol.device)
           for k in names if k != "flags"}
    step = max(16, (1 << 26) // (ny * nx))
    for a in range(0, nz, step):
        b = min(nz, a + step)
        lo, hi = max(0, a - halo), min(nz, b + halo)
        v = vol[lo:hi].to(torch.float64) if vol.dtype == torch.float32 else vol[lo:hi].to(torch.int32).to(torch.float64)
        y0, y1 = _filter(v, g0, 1), _filter(v, g1, 1)
        yx = _filter(y0, g0, 2)
        g = [_filter(yx, g1, 0), _filter(_filter(y1, g0, 2), g0, 0), _filter(_filter(y0, g1, 2), g0, 0)]
        del v, y0, y1, yx
        s = {}
        for i in range(3):
            for j in range(i, 3):
                t = _filter(g[i] * g[j], w0, 0)[a - lo:b - lo]
                s[i, j] = _filter(_filter(t, w0, 1), w0, 2)
        del g
        lam, vec = _jacobi(s)
        small = torch.where((lam[0] <= lam[1]) & (lam[0] <= lam[2]), 0, torch.where(lam[1] <= lam[2], 1, 2))
        e = [torch.where(small == 0, vec[i][0], torch.where(small == 1, vec[i][1], vec[i][2])) for i in range(3)]
        none = (s[0, 0] + s[1, 1] + s[2, 2]) <= 0
        e = _canonical([e[0].masked_fill(none, 1.0), e[1].masked_fill(none, 0.0), e[2].masked_fill(none, 0.0)])
        del vec
        got = {"e3": torch.stack(e)}
        if "evals" in names:
            got["evals"] = torch.sort(torch.stack(lam), dim=0, descending=True).values
        if "fa" in names:
            m = (lam[0] + lam[1] + lam[2]) / 3.0
            dev2 = sum((x - m) ** 2 for x in lam)
            all2 = sum(x * x for x in lam)
            got["fa"] = torch.where(all2 > 0, torch.sqrt(1.5 * dev2 / all2.clamp_min(1e-300)), 0.0).clamp_max(1.0)
        del lam
        if "ha" in names:
            got["ha"], got["ia"] = _frame_angles(e, centre, direction, a, (b - a, ny, nx))
        for k in out:
            t = got[k]
            out[k][..., a:b, :, :] = t if mask is None else t.masked_fill(mask[a:b] == 0, 0.0)
    if "flags" in names:
        out["flags"] = None
    return out


def _bf16(x):
    return x.to(torch.float32).to(torch.bfloat16).to(torch.float64)


def _unpack(blob):
    b = blob.to(torch.float64)
    w, i = {"scale": float(b[0]), "offset": float(b[1])}, 2
    for l in range(1, 6):
        c = 1 if l == 1 else 32
        w[l] = (b[i:i + 32 * c * 27].view(32, c, 27), b[i + 32 * c * 27:i + 32 * c * 27 + 32])
        i += 32 * c * 27 + 32
    w["head"] = (b[i:i + 160].view(5, 32), b[i + 160:i + 165])
    return w


def _shifted(x, tap):
    """x (Z, Y, X, C) read at the tap's offset, indices clamped at every face."""
    for axis, d in enumerate(tap):
        if d:
            n = x.shape[axis]
            x = x.index_select(axis, (torch.arange(n, device=x.device) + d).clamp_(0, n - 1))
    return x


def _conv(x, w, bias):
    Z, Y, X, C = x.shape
    y = bias.expand(Z * Y * X, w.shape[0]).contiguous()
    for t, tap in enumerate(TAPS):
        y.addmm_(_shifted(x, tap).reshape(-1, C), w[:, :, t].t().contiguous())
    return y.view(Z, Y, X, -1)


def _input(vol, w):
    v = vol if vol.dtype == torch.float32 else vol.to(torch.int32)
    return _bf16(v.to(torch.float64) * w["scale"] + w["offset"]).unsqueeze(-1)


def _network64(vol, mask, blob, centre, direction):
    """The surrogate's outputs, activations of layers 1 to 4 rounded to bfloat16 as documented."""
    w = _unpack(blob)
    nz, ny, nx = vol.shape
    out = {k: torch.empty(((3,) if k == "e3" else ()) + (nz, ny, nx), dtype=torch.float64, device=vol.device)
           for k in st.SURROGATE_OUTPUTS}
    step = max(8, (1 << 24) // (ny * nx))
    for a in range(0, nz, step):
        b = min(nz, a + step)
        lo, hi = max(0, a - 5), min(nz, b + 5)
        x = _input(vol[lo:hi], w)
        for l in range(1, 6):
            x = _conv(x, _bf16(w[l][0]), w[l][1]).clamp_min_(0.0)
            x = _bf16(x) if l < 5 else x
        h = (x[a - lo:b - lo].reshape(-1, 32) @ w["head"][0].t() + w["head"][1]).view(b - a, ny, nx, 5)
        n = torch.sqrt((h[..., :3] ** 2).sum(-1))
        e = [torch.where(n > 0, h[..., i] / n.clamp_min(1e-300), 1.0 if i == 0 else 0.0) for i in range(3)]
        e = _canonical(e)
        got = {"e3": torch.stack(e), "fa": torch.sigmoid(h[..., 3]), "confidence": torch.sigmoid(h[..., 4])}
        got["ha"], got["ia"] = _frame_angles(e, centre, direction, a, (b - a, ny, nx))
        for k in out:
            t = got[k]
            out[k][..., a:b, :, :] = t if mask is None else t.masked_fill(mask[a:b] == 0, 0.0)
    return out


def _train64(state):
    """The objective's gradient and sums, activations and their gradients rounded to bfloat16 as documented."""
    w = _unpack(state["params"])
    wt = state["weight"].to(torch.float64)
    xs = [_input(state["patches"], w)]
    for l in range(1, 6):
        xs.append(_bf16(_conv(xs[-1], _bf16(w[l][0]), w[l][1]).clamp_min_(0.0)))
    wh, bh = w["head"]
    x5 = xs[5].reshape(-1, 32)
    h = x5 @ wh.t() + bh
    t, f, m = state["target"].to(torch.float64).view(3, -1).t(), state["fa"].to(torch.float64).view(-1), wt.view(-1)
    n = torch.sqrt((h[:, :3] ** 2).sum(1, keepdim=True))
    u = h[:, :3] / torch.where(n > 0, n, 1.0)
    dot = (u * t).sum(1, keepdim=True)
    ang = torch.rad2deg(torch.atan2(torch.linalg.cross(u, t).norm(dim=1), dot[:, 0].abs()))
    c = (ang < 2.0).to(torch.float64)
    s3, s4 = torch.sigmoid(h[:, 3]), torch.sigmoid(h[:, 4])
    conf_weight = 0.1
    dh = torch.cat([-2.0 * dot * (t - dot * u) / torch.where(n > 0, n, 1.0),
                    (2.0 * (s3 - f) * s3 * (1.0 - s3)).unsqueeze(1), (conf_weight * (s4 - c)).unsqueeze(1)], 1) * m.unsqueeze(1)
    losses = [1.0 - dot[:, 0] ** 2, (s3 - f) ** 2, torch.nn.functional.softplus(h[:, 4]) - c * h[:, 4]]
    total = float(m.sum())
    ld, lf, lc = (float((m * x).sum()) / total for x in losses)
    stats = torch.tensor([ld, lf, lc, ld + lf + conf_weight * lc, total, float((m * c).sum()),
                          float((m * ang).sum()) / total, total], dtype=torch.float64)
    parts = [torch.cat([(dh.t() @ x5).reshape(-1), dh.sum(0)])]
    g = _bf16((dh @ wh) * (x5 > 0)).view_as(xs[5])
    for l in range(5, 0, -1):
        x, gf = xs[l - 1], g.reshape(-1, 32)
        dw = torch.stack([gf.t() @ _shifted(x, tap).reshape(-1, x.shape[-1]) for tap in TAPS], -1)
        parts.insert(0, torch.cat([dw.reshape(-1), gf.sum(0)]))
        if l > 1:
            back = _bf16(w[l][0]).flip(2).transpose(0, 1).contiguous()
            g = _bf16(_conv(g, back, torch.zeros(32, dtype=torch.float64, device=g.device)) * (x > 0))
    grad = torch.cat([torch.zeros(2, dtype=torch.float64, device=m.device)] + parts)
    grad[2:] /= total
    return {"grad": grad, "stats": stats}


def exact(case, seed):
    kind = case["kind"]
    s = prepare(case, seed)
    if kind in ("tensor", "noalloc"):
        s.pop("workspace", None), s.pop("out")
        return _tensor64(s["volume"], s["mask"], case["sigma"], case["rho"], s["centre"], DIRECTION, s["names"])
    if kind == "angles":
        e = [c.to(torch.float64) for c in s["e3"]]
        ha, ia = _frame_angles(e, s["centre"], DIRECTION, 0, _shape(case))
        if s["mask"] is not None:
            ha, ia = ha.masked_fill(s["mask"] == 0, 0.0), ia.masked_fill(s["mask"] == 0, 0.0)
        return {"ha": ha, "ia": ia}
    if kind == "batch":
        got = []
        for c in s["chunks"]:
            centre = [v - o for v, o in zip((120.0, 130.5, 140.0), c["origin"])]
            got.append(_tensor64(c["volume"], c["mask"], case["sigma"], c["rho"], centre, DIRECTION, OUTPUTS["default"]))
        return got
    if kind == "surrogate":
        net = _network64(s["volume"], s["mask"], s["weights"], s["centre"], DIRECTION)
        if case["min_confidence"] > 0:
            low = net["confidence"] < case["min_confidence"]
            path = _tensor64(s["volume"], s["mask"], case["sigma"], case["rho"], s["centre"], DIRECTION, OUTPUTS["maps"])
            for k in path:
                net[k] = torch.where(low, path[k], net[k])
        return net
    return _train64(s)
