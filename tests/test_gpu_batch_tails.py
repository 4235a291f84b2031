"""The ends of a batch step that a group runs with one launch per kernel for
all of its cells, on the boxes that do not take the Poisson solve by planes:
isolated ones (the solve pass by pass on the doubled box's half spectrum) and
periodic ones without Hartree potential, each with cells of one and of several
chunks of orbitals in the density. Every cell equals its solo run bit for bit."""
import numpy as np
import pytest

from gpu_helpers import announce, gpu_run
from oracle_helpers import tiny_isolated, tiny_periodic
from paper_1804_01404_amd.binding import TDDFTBatch

pytestmark = pytest.mark.gpu
ORBITALS = [3, 16, 17, 40]  # chunks of 16: one, one, two, three
NSTEPS = 6


def _field(seed):
    return np.cumsum(np.random.default_rng(seed).normal(size=(NSTEPS + 1, 3)), axis=0)


@pytest.mark.parametrize("prec", ["c128", "mixed"])
@pytest.mark.parametrize("kind", ["isolated12", "isolated16", "isolated12-free", "periodic12-free"])
def test_grouped_tail_equals_solo_runs(kind, prec):
    n, free = int("".join(ch for ch in kind if ch.isdigit())), kind.endswith("free")
    make = tiny_isolated if kind.startswith("isolated") else tiny_periodic
    cells = [make(n=n, n_orb=m, dt=0.01, nsteps=NSTEPS, A=_field(601 + m), hartree=not free, seed=600 + m)
             for m in ORBITALS]
    announce(f"grouped tail, {kind}, {prec}, orbitals {ORBITALS}")
    with TDDFTBatch(cells, precision=prec) as b:
        J = b.propagate([c.A for c in cells])
        psi = [b.orbitals(i) for i in range(len(cells))]
        rho = [b.density(i) for i in range(len(cells))]
        rep = b.report()
    assert len(rep["groups"]) == 1 and rep["groups"][0]["cells"] == len(cells) and rep["groups"][0]["grouped_tail"]
    for i, c in enumerate(cells):
        solo = gpu_run(c, precision=prec)
        assert np.array_equal(J[i], solo["J"]), i
        assert np.array_equal(psi[i], solo["psi"]), i
        assert np.array_equal(rho[i], solo["rho"]), i
