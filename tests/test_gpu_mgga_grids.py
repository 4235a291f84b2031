"""TB09 and BJ on grids that tell the parts of the density, tau and exchange
passes apart: slabs of the plane sweep that do not divide the column, planes
beyond one workgroup (24 loads per point), more points than one workgroup adds
up for c (65536), one and several chunks of orbitals, an isolated box."""
import numpy as np
import pytest

from oracle import tdks
from synth.systems import build_system, rng_for
from tests.gpu_helpers import announce, rel_l2

pytestmark = pytest.mark.gpu

CASES = {
    "slabs-5-4": ((12, 10, 9), "periodic", 5, 1, "tb09"),
    "slab-of-one": ((10, 12, 16), "periodic", 5, 4, "tb09"),
    "plane-1024": ((32, 32, 10), "periodic", 2, 1, "bj"),
    "plane-beyond": ((45, 25, 9), "periodic", 9, 8, "tb09"),
    "many-points": ((48, 40, 36), "periodic", 2, 1, "tb09"),
    "isolated": ((16, 15, 18), "isolated", 3, 1, "tb09"),
}


@pytest.mark.parametrize("name", CASES)
def test_mgga_grid_matches_oracle(name):
    n, boundary, n_orb, n_k, xc = CASES[name]
    rng = rng_for(67, *n)
    iso = boundary == "isolated"
    cell = tuple(np.array([0.50, 0.55, 0.61]) * n)
    nsteps = 2
    A = np.cumsum(rng.normal(size=(nsteps + 1, 3)), axis=0)
    atoms = rng.uniform(-0.3, 0.3, size=(2, 3)) * cell + (0.0 if iso else 0.5) * np.array(cell)
    s = build_system(name=name, n=n, cell=cell, boundary=boundary, n_orb=n_orb,
                     kpts=np.zeros((1, 3)) if iso else rng.uniform(-0.2, 0.2, size=(n_k, 3)),
                     kw=np.full(n_k, 1.0 / n_k), atoms=atoms, rng=rng, n_proj=4, dt=0.01, nsteps=nsteps, A=A,
                     gauge="length" if iso else "velocity", precision="c128")
    s.xc = xc
    o = tdks.TDKS.from_system(s)
    Jo = o.propagate(A)
    announce(f"mgga {name} n={n} n_orb={n_orb} n_k={n_k} xc={xc}")
    from paper_1804_01404_amd.binding import TDDFT
    with TDDFT(s, precision="c128") as t:
        t.set_potential()
        J = t.propagate(A)
        rho, _ = t.density_current()
        psi, c = t.orbitals(), t.xc_parameter()
    assert rel_l2(psi, o.psi) < 1e-10
    assert rel_l2(rho, o.rho) < 1e-10
    assert np.max(np.abs(J - Jo)) < 1e-8 * np.max(np.abs(Jo))
    assert abs(np.ravel(c)[0] - o.mgga_c) < 1e-12 * abs(o.mgga_c)
