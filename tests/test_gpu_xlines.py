"""GPU parity of the whole-plane kernels with the x split compiled and the y split at
run time, and of launches narrower than the schedule's workgroup: x lengths with no
lane-quad kernel (FP64) or any (FP32), y lengths of another split, planes of a few
tasks (256 threads), of two workgroups per CU and of one (FP32, 1024 threads), and a
narrow sphere that leaves these kernels for the runtime-sized one; application,
density and both in one pass against the CPU oracle (FP64 1e-12; FP32 2e-6 on
FP32-rounded inputs, 3e-6 for the density), a batch against its members' plans bit
for bit."""
import numpy as np
import pytest

import oracle
import synth
from helpers import relerr, relerr_per_band

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
vloc = pytest.importorskip("paper_1601_07378_amd.vloc")

CASES = [
    ((18, 20, 16), 4.2), ((20, 18, 24), 4.5), ((25, 30, 20), 4.9), ((27, 24, 20), 5.5),
    ((30, 45, 25), 6.3), ((45, 36, 20), 9.3), ((50, 27, 20), 9.6), ((54, 60, 20), 9.9),
    ((81, 48, 30), 14.6), ((90, 108, 36), 17.5), ((100, 120, 40), 19.0), ((36, 40, 36), 8.0),
    ((54, 60, 20), 5.0),
]


@pytest.fixture(scope="module", autouse=True)
def _gpu(require_gpu):
    yield


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("grid,R", CASES)
def test_xlines_vs_oracle(grid, R, precision):
    print("CASE", dict(test="xlines", grid=grid, R=R, precision=precision), flush=True)
    ct, rt = (torch.complex128, torch.float64) if precision == "f64" else \
        (torch.complex64, torch.float32)
    cell, ecut, k, nb = synth.cubic_cell(), synth.ecut_for_radius(R), (0.25, 0.1, 0.3), 3
    hkl = oracle.sphere_py(cell, ecut, k)
    c, V, w = synth.coefficients(hkl, nb, k), synth.potential(grid, 4), synth.band_weights(nb)
    if precision == "f32":
        c = c.astype(np.complex64).astype(np.complex128)
        V = V.astype(np.float32).astype(np.float64)
    tc, tV = torch.from_numpy(c).to("cuda", ct), torch.from_numpy(V).to("cuda", rt)
    tw = torch.from_numpy(w).cuda()
    p = vloc.Plan(grid, cell, ecut, k, precision=precision)
    out, rho = p.apply(tc, tV), p.density(tc, tw)
    out2, rho2 = p.apply_density(tc, tV, tw)
    torch.cuda.synchronize()
    f32 = precision == "f32"
    err = relerr_per_band(out.cpu().numpy().astype(np.complex128),
                          oracle.apply(grid, cell, ecut, k, c, V)).max()
    assert err <= (2e-6 if f32 else 1e-12)
    assert torch.equal(out, out2)
    psi = oracle.g2r(grid, cell, ecut, k, c).reshape(nb, -1)
    ref = (w[:, None] * np.abs(psi) ** 2).sum(0) / np.prod(grid)
    assert relerr(rho.cpu().numpy().ravel(), ref) <= (3e-6 if f32 else 1e-12)
    assert relerr(rho2.cpu().numpy(), rho.cpu().numpy()) <= 1e-15


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("grid,R", [((45, 50, 40), 9.0), ((27, 30, 27), 5.2)])
def test_xlines_batch_equals_plans(grid, R, precision):
    """Members on either side of the compiled kernels' full mask."""
    print("CASE", dict(test="xlines_batch", grid=grid, precision=precision), flush=True)
    ct, rt = (torch.complex128, torch.float64) if precision == "f64" else \
        (torch.complex64, torch.float32)
    cell, ecut = synth.cubic_cell(), synth.ecut_for_radius(R)
    kpts = [(0, 0, 0), (0.9, -0.7, 0.25), (0.5, 0, 0)]
    b = vloc.Batch(grid, cell, ecut, kpts, precision=precision)
    cs = [torch.from_numpy(synth.coefficients(p.gvectors(), nb, k, ik=i)).to("cuda", ct)
          for i, (p, nb, k) in enumerate(zip(b.plans, (3, 2, 4), kpts))]
    V = torch.from_numpy(synth.potential(grid, 4)).to("cuda", rt)
    outs = b.apply(cs, V)
    for o, c, k in zip(outs, cs, kpts):
        own = vloc.Plan(grid, cell, ecut, k, precision=precision).apply(c, V)
        torch.cuda.synchronize()
        assert torch.equal(o, own)
