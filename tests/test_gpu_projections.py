"""The nonlocal term of the per-stage path against the oracle where its work
split can go wrong: one to nine orbitals (wavefronts take four at a time, two
with the moments) of one to several k-points, spheres of a few points, of
about one and of several times 64, disjoint (the term rides on the next
projection) and overlapping (one add-back per colour), few items (one per
workgroup) and more than 4096 (one per wavefront)."""
import numpy as np
import pytest

from synth.systems import build_system, rng_for
from tests.gpu_helpers import gpu_run, oracle_run, rel_l2

pytestmark = pytest.mark.gpu
STREAMING = 8

N = (10, 12, 15)
CELL = (5.0, 6.0, 7.5)


def lattice(shape):
    axes = [(np.arange(m) + 0.35) / m for m in shape]
    return np.stack(np.meshgrid(*axes, indexing="ij"), axis=-1).reshape(-1, 3) * CELL


# orbitals, k-points, atoms, sphere radius
CASES = {
    "one-point-spheres": (1, 1, lattice((1, 1, 2)), 0.35),
    "disjoint": (5, 2, lattice((2, 2, 2)), 1.2),
    "disjoint-large": (4, 1, lattice((1, 1, 2)), 1.6),
    "overlapping": (3, 3, lattice((2, 2, 1)), 2.4),
    "many-items": (5, 64, lattice((3, 3, 4)), 0.8),
    "many-items-overlapping": (9, 40, lattice((3, 3, 4)), 1.1),
}


@pytest.mark.parametrize("prec", ["c128", "mixed"])
@pytest.mark.parametrize("name", CASES)
def test_nonlocal_term_matches_oracle(name, prec):
    n_orb, n_k, atoms, r_c = CASES[name]
    rng = rng_for(73, n_orb, n_k)
    nsteps = 4
    A = np.cumsum(rng.normal(size=(nsteps + 1, 3)), axis=0)
    s = build_system(name=name, n=N, cell=CELL, boundary="periodic", n_orb=n_orb,
                     kpts=rng.uniform(-0.2, 0.2, size=(n_k, 3)), kw=np.full(n_k, 1.0 / n_k), atoms=atoms, rng=rng,
                     n_proj=4, dt=0.01, nsteps=nsteps, A=A, precision=prec, r_c=r_c, sigma=0.6)
    g, o = gpu_run(s, flags=STREAMING), oracle_run(s)
    tol = 1e-10 if prec == "c128" else 2e-6 * np.sqrt(nsteps)
    assert rel_l2(g["psi"], o["psi"]) < tol
    assert rel_l2(g["rho"], o["rho"]) < tol
    assert np.max(np.abs(g["J"] - o["J"])) < (1e-8 if prec == "c128" else 1e-5) * np.max(np.abs(o["J"]))
    assert abs(g["E"] - o["E"]) < (1e-9 if prec == "c128" else 1e-5) * abs(o["E"])
