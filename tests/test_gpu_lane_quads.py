"""GPU parity of the lane-quad plane kernel (FP64, automatic schedule, x axis of
4 Q points with Q a register codelet >= 8): application, density and both in one
pass, against the CPU oracle and against the whole-plane kernel of the same plan
with the layout asked for (plane_xmode 3).

Sizes: Q that four divides and not (a last group of fewer than four values), one
row block and several with a remainder, several planes per workgroup with an odd
band count, the compiled y splits and runtime ones (codelets of at most 12
points and of 15 or 16), spheres from a fifth of the axis to nearly all of it,
k-shifts, batches of uneven k-points.

Tolerance: a transform of N points carries about eps log2 N relative error per
direction, so two FP64 paths agree to 2 * 2.2e-16 * log2(N1 N2 N3) < 1.1e-14; the
oracle gate is the 1e-12 of the other FP64 tests."""
import numpy as np
import pytest

import oracle
import synth
from helpers import relerr, relerr_per_band

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
vloc = pytest.importorskip("paper_1601_07378_amd.vloc")

TOL = 1e-12
PAIR = 1.1e-14

# grid, radius (unit reciprocal vectors), k, bands
CASES = [
    ((32, 16, 12), 5.0, (0, 0, 0), 1),           # Q = 8, one row block
    ((36, 20, 18), 4.2, (0.25, 1 / 3, 0.1), 5),  # Q = 9, rows 16 + 4
    ((40, 45, 16), 7.5, (0.5, 0.5, 0.5), 3),     # Q = 10, near-maximal z, odd rows
    ((48, 75, 20), 9.4, (0, 0.25, 0), 7),        # Q = 12, y 5 x 15
    ((60, 64, 25), 12.2, (1 / 3, 1 / 3, 0), 4),  # Q = 15, y 8 x 8
    ((64, 48, 16), 7.9, (0, 0, 0), 2),           # Q = 16
    ((72, 96, 20), 9.7, (0.25, 0.25, 0), 9),     # Q = 18, two planes per workgroup
    ((80, 80, 30), 14.9, (0, 0, 0), 5),          # Q = 20, compiled y split, narrow sphere
    ((96, 96, 54), 24.0, (0, 0, 0), 11),         # Q = 24, quarter sphere, odd bands
    ((96, 27, 20), 9.0, (-0.25, 0, 0.5), 3),     # Q = 24, y 3 x 9
    ((100, 36, 20), 9.0, (0.1, 0.2, 0.3), 3),    # Q = 25
    ((108, 50, 20), 9.0, (0.5, 0, 0), 3),        # Q = 27
    ((120, 80, 16), 7.0, (0, 0, 0), 2),          # Q = 30
    ((128, 128, 72), 32.0, (0, 0, 0), 3),        # Q = 32, compiled y split
    ((128, 150, 12), 5.5, (0, 0.5, 0), 3),       # Q = 32, ten row blocks on eight waves
]


@pytest.fixture(scope="module", autouse=True)
def _gpu(require_gpu):
    yield


def inputs(grid, R, k, nb):
    cell, ecut = synth.cubic_cell(), synth.ecut_for_radius(R)
    hkl = oracle.sphere_py(cell, ecut, k)
    return cell, ecut, synth.coefficients(hkl, nb, k), synth.potential(grid, 4)


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("grid,R,k,nb", CASES)
def test_lane_quads_vs_oracle_and_whole_plane(grid, R, k, nb):
    print("CASE", dict(test="lane_quads", grid=grid, R=R, k=k, nb=nb), flush=True)
    cell, ecut, c, V = inputs(grid, R, k, nb)
    p = vloc.Plan(grid, cell, ecut, k)
    w = synth.band_weights(nb)
    tc, tV, tw = dev(c), dev(V), dev(w)
    out = p.apply(tc, tV)
    rho = p.density(tc, tw)
    out2, rho2 = p.apply_density(tc, tV, tw)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert relerr_per_band(got, oracle.apply(grid, cell, ecut, k, c, V)).max() <= TOL
    assert torch.equal(out, out2)
    psi = oracle.g2r(grid, cell, ecut, k, c).reshape(nb, -1)
    ref = (w[:, None] * np.abs(psi) ** 2).sum(0) / np.prod(grid)
    assert relerr(rho.cpu().numpy().ravel(), ref) <= TOL
    assert relerr(rho2.cpu().numpy(), rho.cpu().numpy()) <= 1e-15
    # the layout's own kernel (rows in LDS): another order of the same sums
    old = vloc.Plan(grid, cell, ecut, k, plane_xmode=p.layout()["plane_xmode"])
    got_old = old.apply(tc, tV)
    rho_old = old.density(tc, tw)
    torch.cuda.synchronize()
    assert relerr_per_band(got, got_old.cpu().numpy()).max() <= PAIR
    assert relerr(rho.cpu().numpy(), rho_old.cpu().numpy()) <= PAIR


@pytest.mark.parametrize("grid,R", [
    ((60, 64, 25), 10.0),
    ((80, 80, 30), 14.9),    # narrow sphere
    ((80, 80, 50), 24.9),    # some members within 0.315 of the axis, some not
    ((100, 40, 40), 9.8),    # narrower than the compiled classes
    ((64, 64, 60), 16.0),    # the quarter sphere: hmin and hmax differ between members
    ((64, 64, 60), 19.9),    # near the limits of the wider class
    ((72, 96, 20), 9.0),
    ((96, 96, 50), 24.0),    # the quarter sphere, and shifted ones
])
def test_lane_quads_batch_equals_plans(grid, R):
    """Uneven k-points (their own occupied x-planes, odd counts, none) in shared
    launches, band chunks that cut through them, and the plans' own results."""
    print("CASE", dict(test="lane_quads_batch", grid=grid), flush=True)
    cell, ecut = synth.cubic_cell(), synth.ecut_for_radius(R)
    kpts = [(0, 0, 0), (0.9, -0.7, 0.25), (0.5, 0, 0), (-0.6, 0.5, 0.25)]
    nbs = [3, 0, 5, 2]
    V = synth.potential(grid, 4)
    for chunk in (0, 4):
        b = vloc.Batch(grid, cell, ecut, kpts, band_chunk=chunk)
        cs = [synth.coefficients(p.gvectors(), nb, k, ik=i)
              for i, (p, nb, k) in enumerate(zip(b.plans, nbs, kpts))]
        outs = b.apply([dev(c) for c in cs], dev(V))
        torch.cuda.synchronize()
        for o, c, k, nb in zip(outs, cs, kpts, nbs):
            if not nb:
                continue
            assert relerr_per_band(o.cpu().numpy(),
                                   oracle.apply(grid, cell, ecut, k, c, V)).max() <= TOL
            assert torch.equal(o, vloc.Plan(grid, cell, ecut, k).apply(dev(c), dev(V)))
