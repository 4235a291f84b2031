"""The Poisson solve of the step over the forms its box can take, against the
oracle: radices 8, 4, 2, 3 and 5 in one and several stages, odd lengths (where
the conjugate half has no Nyquist frequency), equal and different x and y,
planes that fit a workgroup and planes that do not, and the doubled box of an
isolated grid. The orbitals of a strong density over a few steps carry the
potential's error; the sum over atoms behind the nonlocal current is taken
with fewer and with more than sixteen atoms."""
import numpy as np
import pytest

from synth.systems import build_system, rng_for
from tests.gpu_helpers import gpu_run, oracle_run, rel_l2

pytestmark = pytest.mark.gpu

PLANES = [(9, 15, 25), (32, 30, 10), (27, 50, 16), (64, 32, 9), (45, 12, 18), (24, 24, 20)]
LINES = [(50, 45, 9), (81, 27, 10), (16, 160, 9)]
ISOLATED = [(9, 10, 12), (25, 12, 15), (16, 24, 32)]


@pytest.mark.parametrize("n, boundary", [(n, "periodic") for n in PLANES + LINES] +
                         [(n, "isolated") for n in ISOLATED])
def test_poisson_box_matches_oracle(n, boundary):
    rng = rng_for(57, *n)
    h = np.array([0.50, 0.55, 0.61])
    cell = tuple(h * n)
    nsteps = 3
    iso = boundary == "isolated"
    n_atoms = 19 if n[0] % 2 else 3
    atoms = rng.uniform(-0.3, 0.3, size=(n_atoms, 3)) * cell + (0.0 if iso else 0.5) * np.array(cell)
    A = np.cumsum(rng.normal(size=(nsteps + 1, 3)), axis=0)
    s = build_system(name="poisson", n=n, cell=cell, boundary=boundary, n_orb=4, kpts=np.zeros((1, 3)), kw=np.ones(1),
                     atoms=atoms, rng=rng, n_proj=4, dt=0.01, nsteps=nsteps, A=A,
                     gauge="length" if iso else "velocity", precision="c128")
    g, o = gpu_run(s), oracle_run(s)
    assert rel_l2(g["psi"], o["psi"]) < 1e-10
    assert rel_l2(g["rho"], o["rho"]) < 1e-10
    assert np.max(np.abs(g["J"] - o["J"])) < 1e-8 * np.max(np.abs(o["J"]))
