"""Performance cases of the local-potential framework.

Each case is one pass of the work that a plane-wave electronic-structure program
hands to this package again and again: the local potential applied to a block of
bands (complex bands, real bands at Gamma, several k-points at once), the density
of weighted bands, and the local-potential energy with all of its gradients.

A case is a dict of plain values:
  kind       "apply", "gamma", "batch", "density" or "energy"
  n1 n2 n3   FFT grid (lengths with no prime factor other than 2, 3 and 5)
  shape      cell: "ortho" (edges in proportion to the grid, so that the sphere
             takes the same share of every axis), "cubic" (equal edges on any
             grid) or "hex" (a1 and a2 at 120 degrees, edges as "ortho")
  radius     cutoff radius in units of the reciprocal vector of the shortest axis;
             a quarter of that axis' length is the grid that holds V psi exactly
  precision  "f64" or "f32"
  bands      bands of the call ("batch": one count per k-point, "2/4/6")
  kpt        index into KPTS ("batch" takes the k-points 0, 1, 2, ...)
  graph      "batch" only: the call's launches are replayed as a captured graph
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1601_07378_amd import autograd, vloc

# Reduced coordinates: Gamma, a Monkhorst-Pack-like list, the K point of a
# hexagonal cell.
KPTS = ((0.0, 0.0, 0.0), (0.25, 0.0, 0.0), (0.25, 0.25, 0.0), (0.25, 0.25, 0.25),
        (0.5, 0.0, 0.0), (0.5, 0.5, 0.0), (0.5, 0.5, 0.5), (0.25, 0.5, 0.0),
        (1.0 / 3.0, 1.0 / 3.0, 0.0))

LENGTHS = sorted(2 ** i * 3 ** j * 5 ** k for i in range(8) for j in range(5) for k in range(4)
                 if 16 <= 2 ** i * 3 ** j * 5 ** k <= 160)


def _case(name, kind, grid, radius, precision, bands, shape="ortho", kpt=0, graph=False):
    c = dict(kind=kind, n1=grid[0], n2=grid[1], n3=grid[2], shape=shape, radius=radius,
             precision=precision, bands=bands, kpt=kpt, graph=graph)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # a small molecule or primitive cell: the whole call is launches
        _case("small_24_f64", "apply", (24, 24, 24), 6.0, "f64", 8),
        # the few new directions of one iteration of a block eigensolver
        _case("block_64_f64", "apply", (64, 64, 64), 16.0, "f64", 4),
        # a 500-atom metal supercell, every band of an SCF step
        _case("supercell_80_f64", "apply", (80, 80, 80), math.sqrt(413.0), "f64", 1001),
        # an ordinary supercell in both precisions (mixed-precision solvers run
        # their first iterations in FP32)
        _case("bands_96_f64", "apply", (96, 96, 96), 24.0, "f64", 256),
        _case("bands_96_f32", "apply", (96, 96, 96), 24.0, "f32", 256),
        # a large cell at a high cutoff
        _case("bands_128_f64", "apply", (128, 128, 128), 32.0, "f64", 96),
        # a hexagonal slab at its K point
        _case("hex_60_f64", "apply", (60, 60, 100), 15.2, "f64", 37, shape="hex", kpt=8),
        # a low-symmetry cell: three unequal, partly odd lengths, a general k
        _case("ragged_90_f32", "apply", (90, 108, 125), 23.3, "f32", 61, kpt=3),
        # Gamma-only calculation with real bands, an odd number of them
        _case("gamma_96_f64", "gamma", (96, 96, 96), 24.0, "f64", 255),
        # many k-points with few bands each, replayed every solver iteration
        _case("kpts_small_f64", "batch", (72, 96, 128), 18.0, "f64", "2/4/6/8/2/4/6/8",
              shape="cubic", graph=True),
        # few k-points with many bands each
        _case("kpts_large_f32", "batch", (72, 96, 128), 18.0, "f32", "64/128/256/512",
              shape="cubic"),
        # energy and all gradients (differentiable potential), the largest
        _case("energy_128_f32", "energy", (128, 128, 128), 32.0, "f32", 512),
    ]


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50.0)


def draw(rng):
    """One more case: any grid, cell, k-point, precision, kind and band count of
    the same ranges."""
    top = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(("apply", "apply", "apply", "gamma", "batch", "density", "energy"))
        precision = rng.choice(("f64", "f32"))
        es = 16 if precision == "f64" else 8
        top_len = 128 if precision == "f64" else 160
        # the shortest axis over its logarithm, the others up to twice as long
        n = math.exp(rng.uniform(math.log(20.0), math.log(top_len)))
        if rng.random() < 0.5:
            grid = [min(LENGTHS, key=lambda x: abs(x - n))] * 3
        else:
            grid = [min(LENGTHS, key=lambda x, s=n * rng.uniform(1.0, 2.0): abs(x - s))
                    for _ in range(3)]
        if max(grid[:2]) > top_len:
            continue
        small = min(grid)
        radius = round(small * rng.uniform(0.2, 0.3), 3)
        # the occupied part of a z-plane has to fit in a CU's LDS
        if (2 * radius * grid[0] / small + 3) * (grid[1] + 1) * es + 8 * grid[0] * es > 150 * 1024:
            continue
        shape = "hex" if rng.random() < 0.25 and kind != "gamma" else "ortho"
        top_bands = math.exp(rng.uniform(0.0, math.log(1024.0)))
        if kind == "batch":
            nk = rng.randint(2, 8)
            bands = "/".join(str(max(1, int(top_bands / nk * rng.uniform(0.3, 1.7))))
                             for _ in range(nk))
        else:
            bands = max(1, int(top_bands))
        kpt = 0 if kind in ("gamma", "batch") else rng.randrange(len(KPTS))
        case = _case(None, kind, grid, radius, precision, bands, shape, kpt,
                     kind == "batch" and rng.random() < 0.5)
        if _cost(case) <= top:
            return case


# ------------------------------------------------------------- geometry


def _grid(case):
    return case["n1"], case["n2"], case["n3"]


def _cell(case):
    grid = _grid(case)
    small = min(grid)
    edge = [2 * math.pi * (n / small if case["shape"] != "cubic" else 1.0) for n in grid]
    rows = np.diag(edge)
    if case["shape"] == "hex":
        rows[1] = edge[1] * np.array([-0.5, math.sqrt(3.0) / 2.0, 0.0])
    return rows


def _ecut(case):
    return 0.5 * case["radius"] ** 2


def _kpts(case):
    if case["kind"] == "batch":
        return KPTS[: len(str(case["bands"]).split("/"))]
    return (KPTS[case["kpt"]],)


def _nbands(case):
    return [int(b) for b in str(case["bands"]).split("/")]


def _sphere(case, kpt):
    """(h, k, l) of |k + G|^2 <= 2 E_cut, lexicographic, and |k + G|^2."""
    A = _cell(case)
    B = 2 * math.pi * np.linalg.inv(A).T
    ext = case["radius"] * np.linalg.norm(A, axis=1) / (2 * math.pi)
    axes = [np.arange(math.floor(-e - q) - 1, math.ceil(e - q) + 2) for e, q in zip(ext, kpt)]
    hkl = np.stack(np.meshgrid(*axes, indexing="ij"), axis=-1).reshape(-1, 3)
    g2 = (((hkl + np.asarray(kpt)) @ B) ** 2).sum(axis=1)
    keep = g2 <= 2 * _ecut(case) * (1 + 1e-12)
    hkl, g2 = hkl[keep], g2[keep]
    if case["kind"] == "gamma":  # real bands: the half sphere
        h, k, l = hkl.T
        half = (h > 0) | ((h == 0) & (k > 0)) | ((h == 0) & (k == 0) & (l >= 0))
        hkl, g2 = hkl[half], g2[half]
    return hkl, g2


def _types(case):
    return (torch.complex128, torch.float64) if case["precision"] == "f64" else \
        (torch.complex64, torch.float32)


# --------------------------------------------------------------- inputs


def _inputs(case, seed):
    """Bands of every k-point, the potential and the band weights, on the GPU.
    Coefficients fall off as 1 / (1 + |k+G|^2); the potential is a sum of
    Gaussians at random atoms."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    ct, rt = _types(case)
    cs = []
    for kpt, nb in zip(_kpts(case), _nbands(case)):
        hkl, g2 = _sphere(case, kpt)
        x = torch.randn((nb, len(hkl), 2), generator=gen, dtype=rt, device="cuda")
        x *= torch.from_numpy(1.0 / (1.0 + g2)).to("cuda", rt)[None, :, None]
        c = torch.view_as_complex(x)
        if case["kind"] == "gamma":  # real bands have a real average
            zero = int(np.flatnonzero((hkl == 0).all(axis=1))[0])
            c[:, zero] = c[:, zero].real.to(ct)
        cs.append(c)
    n1, n2, n3 = _grid(case)
    atoms = torch.rand((16, 4), generator=gen, dtype=torch.float64, device="cuda")
    V = torch.full((n3, n2, n1), 0.5, dtype=torch.float64, device="cuda")
    for a in atoms:
        e = []
        for n, centre in zip((n3, n2, n1), a[:3]):
            d = torch.remainder(torch.arange(n, dtype=torch.float64, device="cuda") - centre * n
                                + n / 2, n) - n / 2
            e.append(torch.exp(-d * d / 8.0))
        V += (0.5 + a[3]) * e[0][:, None, None] * e[1][None, :, None] * e[2][None, None, :]
    w = 2.0 * torch.rand(_nbands(case)[0], generator=gen, dtype=torch.float64, device="cuda")
    return cs, V.to(rt), w


def prepare(case, seed):
    cs, V, w = _inputs(case, seed)
    grid, cell, ecut, prec = _grid(case), _cell(case), _ecut(case), case["precision"]
    kind = case["kind"]
    if kind == "batch":
        plan = vloc.Batch(grid, cell, ecut, _kpts(case), precision=prec)
        plan.use_graph(bool(case["graph"]))
        return dict(kind=kind, plan=plan, cs=cs, V=V, outs=[torch.empty_like(c) for c in cs])
    plan = vloc.Plan(grid, cell, ecut, _kpts(case)[0], precision=prec, gamma=kind == "gamma")
    if kind == "energy":
        for t in (cs[0], V, w):
            t.requires_grad_(True)
        return dict(kind=kind, plan=plan, c=cs[0], V=V, w=w)
    if kind == "density":
        return dict(kind=kind, plan=plan, c=cs[0], w=w)
    return dict(kind=kind, plan=plan, c=cs[0], V=V, out=torch.empty_like(cs[0]))


def run(state):
    kind, plan = state["kind"], state["plan"]
    if kind == "batch":
        return plan.apply(state["cs"], state["V"], outs=state["outs"])
    if kind == "density":
        return plan.density(state["c"], state["w"])
    if kind == "energy":
        c, V, w = state["c"], state["V"], state["w"]
        c.grad = V.grad = w.grad = None
        E = autograd.local_energy(plan, c, V, w)
        E.backward()
        return dict(E=E.detach(), c=c.grad, V=V.grad, w=w.grad)
    return plan.apply(state["c"], state["V"], out=state["out"])


# ---------------------------------------------------------- what it costs


def work(case):
    """Bytes: bands in, results out, the potential once.  Operations: the compact
    transforms (z on the sticks, y on the occupied x-planes, x everywhere), an
    L-point complex transform counted as 5 L log2 L; two real bands share one
    transform."""
    n1, n2, n3 = _grid(case)
    kind = case["kind"]
    s = 16 if case["precision"] == "f64" else 8
    N = n1 * n2 * n3
    nbytes = flops = 0.0
    for kpt, nb in zip(_kpts(case), _nbands(case)):
        hkl, _ = _sphere(case, kpt)
        npw = len(hkl)
        full = np.concatenate([hkl, -hkl]) if kind == "gamma" else hkl
        nst = len(np.unique(full[:, 0] * 4096 + full[:, 1]))
        nxo = int(full[:, 0].max() - full[:, 0].min() + 1)
        one = 5.0 * (nst * n3 * math.log2(n3) + nxo * n3 * n2 * math.log2(n2)
                     + n2 * n3 * n1 * math.log2(n1))
        passes = nb / 2.0 if kind == "gamma" else float(nb)
        if kind == "density":
            nbytes += nb * npw * s + nb * 8
            flops += nb * (one + 4.0 * N)
        elif kind == "energy":
            nbytes += 2.0 * nb * npw * s + N * s / 2 + nb * 16
            flops += nb * (2.0 * one + 6.0 * N + 10.0 * npw)
        else:
            nbytes += 2.0 * nb * npw * s
            flops += passes * (2.0 * one + 2.0 * N)
    nbytes += N * 8 if kind == "density" else N * s / 2
    return dict(bytes=float(nbytes), flops=float(flops))


# ------------------------------------------------------------- reference


def exact(case, seed):
    """The definition on the whole grid with torch's FFT, in 64 bits:
    psi(r) = sum_G c(G) exp(-i G r), out(G) = (1/N) sum_r exp(+i G r) V(r) psi(r),
    rho(r) = (1/N) sum_n w_n |psi_n(r)|^2, E = sum_n w_n Re <c_n | out_n>."""
    cs, V, w = _inputs(case, seed)
    kind = case["kind"]
    n1, n2, n3 = _grid(case)
    N = n1 * n2 * n3
    V64 = V.to(torch.float64)
    chunk = max(1, (1 << 30) // (16 * N))
    rho = torch.zeros((n3, n2, n1), dtype=torch.float64, device="cuda")
    outs = []
    for kpt, c in zip(_kpts(case), cs):
        hkl, _ = _sphere(case, kpt)
        at = torch.from_numpy((hkl[:, 2] % n3 * n2 + hkl[:, 1] % n2) * n1
                              + hkl[:, 0] % n1).cuda()
        neg = torch.from_numpy((-hkl[:, 2] % n3 * n2 + -hkl[:, 1] % n2) * n1
                               + -hkl[:, 0] % n1).cuda()
        out = torch.empty(c.shape, dtype=torch.complex128, device="cuda")
        for b in range(0, c.shape[0], chunk):
            cb = c[b:b + chunk].to(torch.complex128)
            box = torch.zeros((cb.shape[0], N), dtype=torch.complex128, device="cuda")
            box[:, at] = cb
            if kind == "gamma":
                box[:, neg] = cb.conj()
            psi = torch.fft.fftn(box.view(-1, n3, n2, n1), dim=(1, 2, 3))
            if kind in ("density", "energy"):
                wb = w[b:b + chunk, None, None, None]
                rho += (wb * (psi.real.square() + psi.imag.square())).sum(0) / N
            if kind != "density":
                out[b:b + chunk] = torch.fft.ifftn(psi * V64, dim=(1, 2, 3)).reshape(-1, N)[:, at]
            del box, psi
        outs.append(out)
    if kind == "batch":
        return outs
    if kind == "density":
        return rho
    if kind == "energy":
        c64 = cs[0].to(torch.complex128)
        e = (c64.conj() * outs[0]).real.sum(1)
        return dict(E=(w * e).sum(), c=2.0 * w[:, None] * outs[0], V=rho, w=e)
    return outs[0]
