"""GPU parity of the stick kernels over the compiled z lengths (every 2-3-5-smooth
length from 16 to 160): narrow spheres and ones that reach over 0.4 of the axis,
complex bands at a general k and real bands at Gamma, whose pairs also run the
splitting step.  Against the CPU oracle, at the per-band gates of the other parity
tests (FP64 1e-12; FP32 2e-6 on FP32-rounded inputs)."""
import numpy as np
import pytest

import oracle
import synth
from helpers import relerr_per_band

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
vloc = pytest.importorskip("paper_1601_07378_amd.vloc")

LENGTHS = sorted(2 ** i * 3 ** j * 5 ** k for i in range(8) for j in range(5) for k in range(4)
                 if 16 <= 2 ** i * 3 ** j * 5 ** k <= 160)


@pytest.fixture(scope="module", autouse=True)
def _gpu(require_gpu):
    yield


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("share", [0.25, 0.42])
def test_compiled_z_lengths_vs_oracle(share, precision):
    n1, n2, R = 10, 12, 4.0
    ct, rt = (torch.complex128, torch.float64) if precision == "f64" else \
        (torch.complex64, torch.float32)
    for n3 in LENGTHS:
        print("CASE", dict(test="z_lines", n3=n3, share=share, precision=precision), flush=True)
        # the sphere reaches 4 on the first two axes, share * n3 on the third
        cell = np.diag([2 * np.pi, 2 * np.pi, 2 * np.pi * share * n3 / R])
        ecut = synth.ecut_for_radius(R)
        for gamma in (False, True):
            k = (0, 0, 0) if gamma else (0.25, 0.1, 1 / 3)
            p = vloc.Plan((n1, n2, n3), cell, ecut, k, precision=precision, gamma=gamma)
            hkl = p.gvectors()
            c = synth.coefficients(hkl, 3, k)
            if gamma:
                zero = int(np.flatnonzero((hkl == 0).all(axis=1))[0])
                c[:, zero] = c[:, zero].real
            V = synth.potential((n1, n2, n3), 4)
            if precision == "f32":
                c = c.astype(np.complex64).astype(np.complex128)
                V = V.astype(np.float32).astype(np.float64)
            got = p.apply(torch.from_numpy(c).to("cuda", ct), torch.from_numpy(V).to("cuda", rt))
            torch.cuda.synchronize()
            ref = (oracle.apply_gamma if gamma else oracle.apply)(
                (n1, n2, n3), cell, ecut, *(() if gamma else (k,)), c, V)
            err = relerr_per_band(got.cpu().numpy().astype(np.complex128), ref).max()
            assert err <= (1e-12 if precision == "f64" else 2e-6), (n3, gamma, err)
