"""FP64 batches on the lane-quad plane kernel equal their members' plans bit for bit,
whichever of them share the batch: spheres whose k-points leave different rows or
columns empty, so that the kernel compiled for an empty range fits one member and not
another, k-points outside |k| <= 1, and k-points whose occupied x-planes do not straddle
x = 0 (no lane-quad kernel).  Each case against stand-alone plans, the batch's member
plans and the CPU oracle, with the bands in shared launches and cut into chunks."""
import numpy as np
import pytest

import oracle
import synth
from helpers import relerr_per_band

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
vloc = pytest.importorskip("paper_1601_07378_amd.vloc")

# grid, sphere radius on the x axis and on the others (unit reciprocal vectors), k-points
CASES = [
    # reach on y just above a quarter: rows 59 (80) or 71 (96) are occupied for some k only
    ((80, 80, 24), 20.5, 20.5, [(0, 0, 0), (0, 0.9, 0), (0.5, 0, 0)]),
    ((96, 96, 16), 24.0, 24.5, [(0, 0.9, 0), (0, 0, 0), (0, -0.9, 0)]),
    ((72, 96, 16), 18.0, 24.4, [(0, 0, 0), (0.25, 0.9, 0)]),
    ((128, 128, 12), 32.0, 32.5, [(0, 0, 0), (0, 0.9, 0)]),
    # k-points outside |k| <= 1 on x and on y
    ((96, 96, 16), 24.0, 24.0, [(0, 0, 0), (1.5, 0, 0), (0, -2.25, 0), (-5.0, 0, 0)]),
    ((64, 60, 16), 16.0, 16.0, [(3.25, 0, 0), (0, 0, 0)]),
    ((128, 128, 12), 32.0, 32.0, [(0, 0, 0), (1.75, 0, 0)]),
    # x-planes all at h > 0, or all at h < 0
    ((64, 64, 16), 12.0, 12.0, [(0, 0, 0), (-14.0, 0, 0), (0.5, 0.25, 0), (14.5, 0, 0)]),
    ((128, 128, 12), 20.0, 20.0, [(-24.0, 0, 0), (0, 0, 0)]),
]


@pytest.fixture(scope="module", autouse=True)
def _gpu(require_gpu):
    yield


@pytest.mark.parametrize("grid,Rx,Ry,kpts", CASES)
def test_batch_equals_plans(grid, Rx, Ry, kpts):
    print("CASE", dict(test="batch_routes", grid=grid, Rx=Rx, Ry=Ry, kpts=kpts), flush=True)
    # the z axis takes a fifth of its grid
    cell = 2.0 * np.pi * np.diag([1.0, Ry / Rx, 0.2 * grid[2] / Rx])
    ecut = 0.5 * Rx * Rx
    nbs = [3, 2, 4, 1][:len(kpts)]
    V = synth.potential(grid, 4)
    dV = torch.from_numpy(V).cuda()
    own = [vloc.Plan(grid, cell, ecut, k) for k in kpts]
    cs = [synth.coefficients(p.gvectors(), nb, k, ik=i)
          for i, (p, nb, k) in enumerate(zip(own, nbs, kpts))]
    dc = [torch.from_numpy(np.ascontiguousarray(c)).cuda() for c in cs]
    want = [p.apply(c, dV) for p, c in zip(own, dc)]
    # (a parted or whole-plane batch laid out on the union of the ranges may take another
    # y split than a plan by itself)
    for chunk in (0, 2):
        b = vloc.Batch(grid, cell, ecut, kpts, band_chunk=chunk)
        outs = b.apply(dc, dV)
        members = [p.apply(c, dV) for p, c in zip(b.plans, dc)]
        torch.cuda.synchronize()
        for i, (o, w, m, c, k) in enumerate(zip(outs, want, members, cs, kpts)):
            err = relerr_per_band(o.cpu().numpy(),
                                  oracle.apply(grid, cell, ecut, k, c, V)).max()
            print("chunk", chunk, "member", i, "err", err, "equal to plan", torch.equal(o, w),
                  "to member", torch.equal(o, m), flush=True)
            assert err <= 1e-12
            assert torch.equal(o, m), (chunk, i)
            if b.plans[i].layout()["L1y"] == own[i].layout()["L1y"]:
                assert torch.equal(o, w), (chunk, i)
