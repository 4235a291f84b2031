"""The LDS-resident step on every grid it takes, against the oracle: grids of
12^3 to 24^3 differ in the tile of points a thread owns (one to four planes)
and in the workgroup's size, and a box with three different spacings, two
k-points, spheres that overlap (several colours) and reach across the faces
tells the axes, the wraps and the box's ends apart."""
import numpy as np
import pytest

from synth.systems import build_system, rng_for
from tests.gpu_helpers import gpu_run, oracle_run, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("boundary", ["periodic", "isolated"])
@pytest.mark.parametrize("prec", ["c128", "mixed"])
@pytest.mark.parametrize("n", [12, 16, 20, 24])
def test_fused_grid_matches_oracle(n, prec, boundary):
    rng = rng_for(41, n)
    cell = (0.50 * n, 0.55 * n, 0.61 * n)
    nsteps = 8
    iso = boundary == "isolated"
    centre = 0.0 if iso else 0.5
    # two overlapping atoms inside, one by a corner
    atoms = np.array([[0.05, 0.02, -0.03], [0.05, 0.14, 0.02], [-0.42, 0.40, -0.41]]) * cell + centre * np.array(cell)
    A = np.cumsum(rng.normal(size=(nsteps + 1, 3)), axis=0)
    kpts = np.zeros((1, 3)) if iso else np.array([[0.11, -0.07, 0.05], [-0.02, 0.13, 0.17]])
    s = build_system(name=f"fused-{n}", n=(n, n, n), cell=cell, boundary=boundary, n_orb=3, kpts=kpts,
                     kw=np.ones(1) if iso else np.array([0.4, 0.6]), atoms=atoms, rng=rng, n_proj=4, dt=0.02,
                     nsteps=nsteps, A=A, gauge="length" if iso else "velocity", precision=prec)
    g, o = gpu_run(s), oracle_run(s)
    # FP64 rounding with margin; complex FP32 rounds every component once a step
    tol = 1e-10 if prec == "c128" else 2e-6 * np.sqrt(nsteps)
    assert rel_l2(g["psi"], o["psi"]) < tol
    assert rel_l2(g["rho"], o["rho"]) < tol
    assert np.max(np.abs(g["J"] - o["J"])) < (1e-8 if prec == "c128" else 1e-5) * np.max(np.abs(o["J"]))
