"""Timed cases of the spline x-ray transform, through its public entry points.

A case names a volume size, an acquisition, a B-spline degree, a footprint
form and a call:

  forward   sinogram of a coefficient volume (``Projector.forward``)
  adjoint   back-projection of a sinogram (``Projector.adjoint``)
  both      one of each, as a step of a reconstruction loop over view subsets
  grad      ``project`` under autograd and the gradient of its input
  cgls      a few iterations of the least-squares loop (``cgls``)

The sizes are those of the framework's workloads (``configs``), of its
reconstruction analog (``recon``) and of its smoke test, and odd ones between
them.  Volumes and sinograms are made on the GPU from the seed alone.
"""
from __future__ import annotations

import math
import os
import struct

import numpy as np
import torch

from paper_2511_11078_amd import synth
from paper_2511_11078_amd.ops import Projector, cgls, default_weights, project


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------
def _case(name, call, dims, degree, views, rows, cols, geom, form="quad", field="ellipsoids", iters=0):
    return {"name": name, "call": call, "n1": dims[0], "n2": dims[1], "n3": dims[2], "degree": degree,
            "form": form, "views": views, "rows": rows, "cols": cols, "geom": geom, "field": field,
            "iters": iters}


def listed():
    return [
        # one differentiable projection of a patch: a few views, launches and latency count
        _case("tiny_cone_grad", "grad", (20, 18, 16), 3, 8, 24, 28, "cone"),
        # the smallest named workload, every view, inside a training step
        _case("small_parallel_32_grad", "grad", (32, 32, 32), 3, 32, 48, 48, "fibonacci"),
        # a mid-size parallel acquisition with tilted views, each direction by itself
        _case("parallel_128_forward", "forward", (128, 128, 128), 3, 240, 192, 192, "circle_tilts", field="noisy"),
        _case("parallel_128_adjoint", "adjoint", (128, 128, 128), 3, 240, 192, 192, "circle_tilts", field="noisy"),
        # the benchmark's workload, each direction by itself
        _case("cone_256_forward", "forward", (256, 256, 256), 3, 360, 384, 384, "cone"),
        _case("cone_256_adjoint", "adjoint", (256, 256, 256), 3, 360, 384, 384, "cone"),
        # the largest volume, processed in batches of 32 views: one batch (a 16-degree arc)
        _case("cone_512_batch", "both", (512, 512, 512), 3, 32, 768, 768, "cone_arc", field="smooth"),
        # the reconstruction analog of the paper's experiment: quadratic splines, and voxels
        _case("recon_quadratic_cgls", "cgls", (180, 180, 50), 2, 200, 50, 180, "cone_wide", iters=4),
        _case("recon_voxel_cgls", "cgls", (180, 180, 50), 0, 200, 50, 180, "cone_wide", iters=4),
        # the linear basis on an odd-sized volume and detector, inside a training step
        _case("linear_97_grad", "grad", (97, 75, 61), 1, 90, 111, 147, "cone"),
        # the learned footprint: the smallest workload under autograd, and a batch of views at 128^3
        _case("network_small_32_grad", "grad", (32, 32, 32), 3, 32, 48, 48, "fibonacci", form="mlp"),
        _case("network_128_batch", "both", (128, 128, 128), 3, 32, 192, 192, "circle", form="mlp", field="noisy"),
    ]


def draw(rng):
    form = rng.choices(["quad", "mlp", "pair"], weights=[8, 2, 1])[0]
    degree = rng.choices([3, 2, 1, 0], weights=[4, 2, 1, 1])[0]
    if form != "quad":
        degree = max(degree, 1)
    top = 288 if form == "quad" else 64
    base = math.exp(rng.uniform(math.log(12), math.log(top)))
    dims = [max(4, int(round(base * math.exp(rng.uniform(-0.6, 0.2))))) for _ in range(3)]
    rows = max(5, int(round(dims[2] * math.exp(rng.uniform(-0.2, 0.45)))))
    cols = max(5, int(round(max(dims[:2]) * math.exp(rng.uniform(-0.2, 0.45)))))
    views = int(round(math.exp(rng.uniform(math.log(1), math.log(360 if form == "quad" else 48)))))
    call = rng.choices(["forward", "adjoint", "both", "grad", "cgls"], weights=[3, 3, 2, 2, 1])[0]
    if form != "quad" and call == "cgls":
        call = "both"
    geom = rng.choice(["cone", "cone_wide", "cone_arc", "fibonacci", "circle", "circle_tilts"])
    case = _case("", call, dims, degree, views, rows, cols, geom, form,
                 rng.choice(["ellipsoids", "noisy", "smooth"]), rng.randint(1, 4) if call == "cgls" else 0)
    del case["name"]
    # no dearer than the largest listed case of the form
    limit = 1.0e13 if form == "quad" else 3.0e12 if form == "mlp" else 2.0e11
    while work(case)["flops"] > limit and case["views"] > 1:
        case["views"] = max(1, case["views"] // 2)
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _dims(case):
    return case["n1"], case["n2"], case["n3"]


def _geometry(case):
    V, R, C = case["views"], case["rows"], case["cols"]
    extent = float(max(_dims(case)))
    kind = case["geom"]
    if kind == "cone":            # circular cone beam, source at 2.5 times the extent, detector at 3 times
        return synth.cone_circular_geometry(V, R, C, src_radius=2.5 * extent, src_det=3.0 * extent, angle0=0.01)
    if kind == "cone_arc":        # consecutive views of a circle of 720 (one batch of a larger scan)
        full = synth.cone_circular_geometry(720, R, C, src_radius=2.5 * extent, src_det=3.0 * extent)
        first = 64 % (720 - min(V, 719))
        return full.subset_views(first, first + V)
    if kind == "cone_wide":       # the detector through the rotation axis
        return synth.cone_circular_geometry(V, R, C, src_radius=2.5 * extent, src_det=2.5 * extent)
    if kind == "fibonacci":
        return synth.parallel_geometry(synth.fibonacci_directions(V), R, C)
    if kind == "circle":
        return synth.parallel_geometry(synth.great_circle_plus_tilts(V, 0), R, C)
    tilts = V // 4                # a half circle and a quarter of tilted views
    return synth.parallel_geometry(synth.great_circle_plus_tilts(V - tilts, tilts, seed=2), R, C)


def _volume(case, gen, device):
    """Coefficients [N3, N2, N1]: random ellipsoids (plain, or with noise of
    variance 0.01), or a standardised Gaussian-smoothed random field."""
    n1, n2, n3 = _dims(case)
    if case["field"] == "smooth":
        g = torch.randn(n3, n2, n1, generator=gen, device=device)
        f = [torch.fft.fftfreq(n, device=device) for n in (n3, n2)] + [torch.fft.rfftfreq(n1, device=device)]
        k2 = f[0][:, None, None] ** 2 + f[1][None, :, None] ** 2 + f[2][None, None, :] ** 2
        g = torch.fft.irfftn(torch.fft.rfftn(g) * torch.exp(-0.5 * 16.0 * (2 * math.pi) ** 2 * k2), s=(n3, n2, n1))
        g = g - g.mean()
        return (g / g.std().clamp_min(1e-6)).contiguous()
    ax = [(torch.arange(n, device=device) - 0.5 * (n - 1)) / max(0.5 * (n - 1), 0.5) for n in (n1, n2, n3)]
    c = torch.zeros(n3, n2, n1, device=device)
    u = torch.rand(6, 10, generator=gen, device=device).cpu().numpy()
    for e in u:
        cen = 0.6 * (e[0:3] - 0.5)
        semi = 0.1 + 0.4 * e[3:6]
        q = e[6:10] - 0.5
        q = q / np.linalg.norm(q)
        w, x, y, z = q
        rot = np.array([[1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w)],
                        [2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w)],
                        [2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)]])
        d = [ax[k] - float(cen[k]) for k in range(3)]
        r2 = torch.zeros_like(c)
        for m in range(3):
            p = (d[0][None, None, :] * float(rot[0, m]) + d[1][None, :, None] * float(rot[1, m])
                 + d[2][:, None, None] * float(rot[2, m])) / float(semi[m])
            r2 += p * p
        c += (r2 <= 1.0) * float(0.2 + 0.8 * e[9])
    if case["field"] == "noisy":
        c += 0.1 * torch.randn(n3, n2, n1, generator=gen, device=device)
    return c


def _sinogram(case, gen, device):
    """A measured sinogram [V, R, C]: the shadow of a blob per view, modulated
    from view to view, with noise."""
    V, R, C = case["views"], case["rows"], case["cols"]
    jj = (torch.arange(R, device=device) - 0.5 * (R - 1)) / (0.3 * R)
    ii = (torch.arange(C, device=device) - 0.5 * (C - 1)) / (0.3 * C)
    shift = 0.8 * torch.rand(V, 2, generator=gen, device=device) - 0.4
    amp = 0.1 * max(_dims(case)) * (0.5 + torch.rand(V, generator=gen, device=device))
    pj = torch.exp(-0.5 * (jj[None, :] - shift[:, :1]) ** 2)
    pi = torch.exp(-0.5 * (ii[None, :] - shift[:, 1:]) ** 2)
    y = amp[:, None, None] * pj[:, :, None] * pi[:, None, :]
    y += 0.5 * torch.randn(V, R, C, generator=gen, device=device)
    return y


def _inputs(case, seed, device):
    gen = torch.Generator(device=device)
    gen.manual_seed(int(seed))
    call = case["call"]
    c = _volume(case, gen, device) if call in ("forward", "both", "grad") else None
    y = _sinogram(case, gen, device) if call in ("adjoint", "both", "grad", "cgls") else None
    return c, y


def prepare(case, seed):
    geom = _geometry(case)
    c, y = _inputs(case, seed, torch.device("cuda", 0))
    if case["call"] == "grad":
        c.requires_grad_(True)
    return {"call": case["call"], "iters": case["iters"], "c": c, "y": y,
            "projector": Projector(_dims(case), geom, degree=case["degree"], form=case["form"])}


def run(state):
    P, call = state["projector"], state["call"]
    if call == "forward":
        return P.forward(state["c"])
    if call == "adjoint":
        return P.adjoint(state["y"])
    if call == "both":
        return P.forward(state["c"]), P.adjoint(state["y"])
    if call == "cgls":
        x, hist = cgls(P, state["y"], iters=state["iters"])
        return {"x": x, "hist": hist}
    # the misfit's gradient with respect to the coefficients
    out = project(state["c"], P)
    (grad,) = torch.autograd.grad(out, state["c"], grad_outputs=state["y"])
    return {"sinogram": out.detach(), "grad": grad}


# ---------------------------------------------------------------------------
# the work of a pass
# ---------------------------------------------------------------------------
def _line_units(case, views=16, side=12):
    """Mean knot cells per line, and mean bases whose support a line meets:
    a line of length l through a box crosses about l (|w1| + |w2| + |w3|) unit
    cells, and meets (n + 1)^2 times as many supports of width n + 1."""
    geom = _geometry(case)
    n = case["degree"]
    half = np.array([0.5 * (d + n) for d in _dims(case)])
    vecs = np.asarray(geom.vecs, dtype=np.float64)
    sel = np.unique(np.linspace(0, geom.n_views - 1, min(views, geom.n_views)).astype(int))
    jj = np.linspace(0, geom.det_rows - 1, min(side, geom.det_rows)) - 0.5 * (geom.det_rows - 1)
    ii = np.linspace(0, geom.det_cols - 1, min(side, geom.det_cols)) - 0.5 * (geom.det_cols - 1)
    total = 0.0
    for v in sel:
        e = vecs[v]
        p = e[3:6] + ii[None, :, None] * e[6:9] + jj[:, None, None] * e[9:12]
        w = np.broadcast_to(e[0:3], p.shape) if geom.kind == "parallel" else p - e[0:3]
        w = w / np.linalg.norm(w, axis=-1, keepdims=True)
        w = np.where(np.abs(w) < 1e-12, 1e-12, w)
        ta, tb = (-half - p) / w, (half - p) / w
        t0, t1 = np.minimum(ta, tb).max(-1), np.maximum(ta, tb).min(-1)
        total += float((np.maximum(t1 - t0, 0.0) * np.abs(w).sum(-1)).mean())
    cells = total / len(sel)
    return cells, cells * (n + 1) ** 2


def work(case):
    n = case["degree"]
    vol = case["n1"] * case["n2"] * case["n3"]
    rays = case["views"] * case["rows"] * case["cols"]
    cells, pairs = _line_units(case)
    nb, nodes = n + 1, (3 * n + 2) // 2
    if case["form"] == "mlp":  # per pair, the network's matrix products
        one = rays * pairs * (2.0 * (3 * 64 * 64 + 5 * 64 + 64))
    elif n == 0:
        one = rays * cells * 2.0
    else:  # the exact rule's nodes, each a contraction of the cell's (n + 1)^3 block
        one = rays * cells * nodes * 2.0 * (nb ** 3 + nb ** 2 + nb)
    times = {"forward": 1, "adjoint": 1, "both": 2, "grad": 2, "cgls": 2 * case["iters"] + 1}[case["call"]]
    return {"bytes": 4.0 * (vol + rays) * times, "flops": one * times}


# ---------------------------------------------------------------------------
# the same outputs in 64 bits
# ---------------------------------------------------------------------------
def _lines64(geom, device):
    """Anchor and unit direction of every line, [V R C, 3] each."""
    e = torch.as_tensor(np.asarray(geom.vecs), device=device).double()
    jj = torch.arange(geom.det_rows, device=device).double() - 0.5 * (geom.det_rows - 1)
    ii = torch.arange(geom.det_cols, device=device).double() - 0.5 * (geom.det_cols - 1)
    p = (e[:, None, None, 3:6] + ii[None, None, :, None] * e[:, None, None, 6:9]
         + jj[None, :, None, None] * e[:, None, None, 9:12])
    if geom.kind == "parallel":
        w = e[:, None, None, 0:3].expand_as(p)
    else:
        w = p - e[:, None, None, 0:3]
    w = w / w.norm(dim=-1, keepdim=True)
    p, w = p.reshape(-1, 3), w.reshape(-1, 3)
    return p - (p * w).sum(-1, keepdim=True) * w, w


def _blend64(n, t):
    """Values at local coordinate t of the n + 1 uniform B-splines of degree n
    that are non-zero on a knot cell, stacked last."""
    s = 1.0 - t
    if n == 1:
        b = (s, t)
    elif n == 2:
        b = (0.5 * s * s, 0.5 + t * s, 0.5 * t * t)
    else:
        b = (s ** 3 / 6, 2 / 3 - t * t + 0.5 * t ** 3, 2 / 3 - s * s + 0.5 * s ** 3, t ** 3 / 6)
    return torch.stack(b, dim=-1)


def _segments64(case, a, w):
    """Pieces of the lines between knot planes: mid-point and half-length in
    the line's parameter, [K, S] each (empty pieces have no length)."""
    n = case["degree"]
    h, kap = 0.5 * (n + 1), 0.0 if n % 2 else 0.5
    t0 = torch.full_like(a[:, 0], -1e30)
    t1 = -t0
    cross = []
    for k, N in enumerate(_dims(case)):
        z = a[:, k] + 0.5 * (N - 1)
        wk = torch.where(w[:, k].abs() < 1e-14, torch.full_like(z, 1e-14), w[:, k])
        ta, tb = (-h - z) / wk, (N - 1 + h - z) / wk
        t0, t1 = torch.maximum(t0, torch.minimum(ta, tb)), torch.minimum(t1, torch.maximum(ta, tb))
        planes = kap + torch.arange(-3, N + 3, device=a.device).double()
        cross.append((planes[None, :] - z[:, None]) / wk[:, None])
    t1 = torch.maximum(t0, t1)
    t = torch.cat(cross + [t0[:, None], t1[:, None]], dim=1)
    t = torch.minimum(torch.maximum(t, t0[:, None]), t1[:, None]).sort(dim=1).values
    return 0.5 * (t[:, 1:] + t[:, :-1]), 0.5 * (t[:, 1:] - t[:, :-1])


def _exact_quad(case, geom, c, y, device):
    """Forward of c and transpose of y by the exact rule on every piece."""
    n = case["degree"]
    nb, N = n + 1, _dims(case)
    kap = 0.0 if n % 2 else 0.5
    qoff = {1: 0, 2: 0, 3: -1}[n]
    xs, ws = np.polynomial.legendre.leggauss((3 * n + 2) // 2)
    A, Wd = _lines64(geom, device)
    out = torch.zeros(A.shape[0], dtype=torch.float64, device=device) if c is not None else None
    back = torch.zeros(N[0] * N[1] * N[2], dtype=torch.float64, device=device) if y is not None else None
    cf = c.double().reshape(-1) if c is not None else None
    yf = y.double().reshape(-1) if y is not None else None
    step = max(1, int(6e7) // (nb ** 3 * (sum(N) + 20)))
    for lo in range(0, A.shape[0], step):
        a, w = A[lo:lo + step], Wd[lo:lo + step]
        mid, half = _segments64(case, a, w)
        keep = half > 1e-14
        ray = torch.arange(a.shape[0], device=device)[:, None].expand_as(mid)[keep]
        mid, half = mid[keep], half[keep]
        cell, frac, slope, qs, ok = [], [], [], [], []
        for k in range(3):
            z = a[ray, k] + 0.5 * (N[k] - 1) + mid * w[ray, k] - kap
            m = torch.floor(z)
            frac.append(z - m)
            slope.append(half * w[ray, k])
            q = m.long()[:, None] + qoff + torch.arange(nb, device=device)
            ok.append((q >= 0) & (q < N[k]))
            qs.append(q.clamp(0, N[k] - 1))
        idx = (qs[2][:, :, None, None] * N[1] + qs[1][:, None, :, None]) * N[0] + qs[0][:, None, None, :]
        inside = ok[2][:, :, None, None] & ok[1][:, None, :, None] & ok[0][:, None, None, :]
        wt = torch.zeros(idx.shape, dtype=torch.float64, device=device)
        for x, g in zip(xs, ws):
            b = [_blend64(n, frac[k] + float(x) * slope[k]) for k in range(3)]
            wt += float(g) * b[2][:, :, None, None] * b[1][:, None, :, None] * b[0][:, None, None, :]
        wt = wt * half[:, None, None, None] * inside
        if out is not None:
            out.index_add_(0, ray + lo, (wt * cf[idx]).sum((1, 2, 3)))
        if back is not None:
            back.index_add_(0, idx.reshape(-1), (wt * yf[ray + lo][:, None, None, None]).reshape(-1))
    return out, back


def _network64(degree, device):
    """The learned footprint's weights as shipped (BF16 hidden layers)."""
    with open(default_weights(degree), "rb") as fh:
        blob = fh.read()
    at = struct.calcsize("<8s8I2f")

    def take(count, kind):
        nonlocal at
        a = np.frombuffer(blob, dtype=kind, count=count, offset=at)
        at += a.nbytes
        if kind == "<u2":
            a = (a.astype(np.uint32) << 16).view(np.float32)
        return torch.as_tensor(a.astype(np.float64), device=device)

    layers = [(take(320, "<f4").reshape(64, 5), take(64, "<f4"))]
    for _ in range(3):
        layers.append((take(4096, "<u2").reshape(64, 64), take(64, "<f4")))
    layers.append((take(64, "<f4").reshape(1, 64), take(1, "<f4")))
    return layers


def _exact_network(case, geom, c, y, device):
    """Forward of c and transpose of y with the network's value for every
    (line, basis) pair whose support the line meets."""
    n, N = case["degree"], _dims(case)
    h = 0.5 * (n + 1)
    layers = _network64(n, device)
    A, Wd = _lines64(geom, device)
    out = torch.zeros(A.shape[0], dtype=torch.float64, device=device) if c is not None else None
    back = torch.zeros(N[0] * N[1] * N[2], dtype=torch.float64, device=device) if y is not None else None
    cf = c.double().reshape(-1) if c is not None else None
    yf = y.double().reshape(-1) if y is not None else None
    Nt = torch.tensor(N, device=device)
    # fold: axes sorted by |w| ascending (lower axis first on ties), signs taken out
    aw = Wd.abs()
    wf, perm = aw.sort(dim=1, stable=True)
    sgn = torch.where(Wd.gather(1, perm) < 0, -1.0, 1.0).double()
    u = -wf[:, :1] * wf
    u[:, 0] += 1.0
    u = u / u.norm(dim=1, keepdim=True)
    v = torch.linalg.cross(u, wf)
    span = torch.arange(-int(2 * h) - 1, int(2 * h) + 2, device=device)
    step = max(1, int(2e7) // (span.numel() ** 2 * max(N)))
    for lo in range(0, A.shape[0], step):
        a, w = A[lo:lo + step], Wd[lo:lo + step]
        K = a.shape[0]
        d = aw[lo:lo + step].argmax(dim=1)
        i1 = torch.where(d == 0, 1, 0)
        i2 = torch.where(d == 2, 1, 2)
        off = 0.5 * (Nt - 1).double()
        z = a + off
        pick = lambda t, k: t.gather(1, k[:, None])[:, 0]  # noqa: E731
        r1, r2 = pick(w, i1) / pick(w, d), pick(w, i2) / pick(w, d)
        j = torch.arange(max(N), device=device)
        s = j[None, :].double() - pick(z, d)[:, None]
        P1, P2 = pick(z, i1)[:, None] + s * r1[:, None], pick(z, i2)[:, None] + s * r2[:, None]
        q1 = torch.floor(P1).long()[:, :, None, None] + span[None, None, :, None]
        q2 = torch.floor(P2).long()[:, :, None, None] + span[None, None, None, :]
        ok = ((j[None, :, None, None] < Nt[d][:, None, None, None]) & (q1 >= 0) & (q1 < Nt[i1][:, None, None, None])
              & (q2 >= 0) & (q2 < Nt[i2][:, None, None, None]))
        ray, jj, k1, k2 = ok.nonzero(as_tuple=True)
        q1, q2 = q1[ray, jj, k1, 0], q2[ray, jj, 0, k2]
        u1, u2 = P1[ray, jj] - q1, P2[ray, jj] - q2
        s0, s1 = torch.full_like(u1, -h), torch.full_like(u1, h)
        for uu, rr in ((u1, r1[ray]), (u2, r2[ray])):
            rr = torch.where(rr.abs() < 1e-13, torch.full_like(rr, 1e-13), rr)
            ta, tb = (-h - uu) / rr, (h - uu) / rr
            s0, s1 = torch.maximum(s0, torch.minimum(ta, tb)), torch.minimum(s1, torch.maximum(ta, tb))
        meet = s0 < s1
        ray, jj, q1, q2 = ray[meet], jj[meet], q1[meet], q2[meet]
        q = torch.zeros(ray.numel(), 3, dtype=torch.long, device=device)
        q.scatter_(1, d[ray][:, None], jj[:, None])
        q.scatter_(1, i1[ray][:, None], q1[:, None])
        q.scatter_(1, i2[ray][:, None], q2[:, None])
        x = (z[ray] - q).gather(1, perm[lo + ray]) * sgn[lo + ray]
        f = torch.cat([wf[lo + ray], (u[lo + ray] * x).sum(1, keepdim=True), (v[lo + ray] * x).sum(1, keepdim=True)], 1)
        for k, (wl, bl) in enumerate(layers):
            f = f @ wl.T + bl
            if k < 4:
                f = torch.nn.functional.silu(f)
        f = f[:, 0]
        idx = (q[:, 2] * N[1] + q[:, 1]) * N[0] + q[:, 0]
        if out is not None:
            out.index_add_(0, lo + ray, f * cf[idx])
        if back is not None:
            back.index_add_(0, idx, f * yf[lo + ray])
    return out, back


def exact(case, seed):
    # the loop's iterates and the larger workloads take minutes in 64 bits,
    # the voxel basis' outputs jump where a line lies in a voxel face
    _, pairs = _line_units(case)
    total = case["views"] * case["rows"] * case["cols"] * pairs
    if case["call"] == "cgls" or case["degree"] == 0 or not torch.cuda.is_available():
        return None
    if total > (2.0e9 if case["form"] != "mlp" else 2.0e8):
        return None
    device = torch.device("cuda", 0)
    geom = _geometry(case)
    c, y = _inputs(case, seed, device)
    shape = (case["views"], case["rows"], case["cols"])
    vol = (case["n3"], case["n2"], case["n1"])
    fwd, back = (_exact_network if case["form"] == "mlp" else _exact_quad)(case, geom, c, y, device)
    fwd = fwd.reshape(shape) if fwd is not None else None
    back = back.reshape(vol) if back is not None else None
    return {"forward": fwd, "adjoint": back, "both": (fwd, back),
            "grad": {"sinogram": fwd, "grad": back}}[case["call"]]
