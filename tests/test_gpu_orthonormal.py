"""One imaginary-time iteration (the step, then Cholesky-QR on the matrix cores)
against the oracle where the 16-wide orbital tiles and the 16-point tiles have
remainders: one orbital, one tile, several tiles with and without remainders,
more orbitals than the single-wavefront factorisation takes, and a grid whose
points do not fill a workgroup's share."""
import numpy as np
import pytest

from oracle import tdks
from paper_1804_01404_amd.binding import FLAG_STREAMING, TDDFT
from synth.systems import build_system, rng_for
from tests.gpu_helpers import rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["c128", "mixed"])
@pytest.mark.parametrize("n_orb,n,flags", [(1, (12, 12, 12), 0), (15, (12, 12, 12), 0), (16, (9, 10, 8), 0),
                                           (17, (12, 12, 12), FLAG_STREAMING), (32, (12, 12, 12), 0),
                                           (33, (9, 8, 10), 0), (49, (10, 9, 8), 0)])
def test_iteration_matches_oracle(n_orb, n, flags, prec):
    rng = rng_for(71, n_orb)
    cell = (6.1, 6.6, 5.8)
    s = build_system(name=f"ortho-{n_orb}", n=n, cell=cell, boundary="periodic", n_orb=n_orb,
                     kpts=np.array([[0.0, 0.0, 0.0], [0.2, -0.1, 0.15]]), kw=np.array([0.5, 0.5]),
                     atoms=np.array([[1.0, 1.2, 0.7], [4.0, 3.9, 3.2]]), rng=rng, n_proj=4, dt=0.02, nsteps=1,
                     A=np.zeros((2, 3)), precision=prec)
    with TDDFT(s, flags=flags) as t:
        t.set_potential()
        E = t.ground_state(2, 0.01)
        psi = t.orbitals()
    o = tdks.TDKS.from_system(s)
    Eo = o.ground_state(2, 0.01)
    # FP64 rounding with margin for the overlap matrix's condition; complex
    # FP32 rounds the orbitals twice an iteration
    assert rel_l2(psi, o.psi) < (1e-10 if prec == "c128" else 5e-6)
    assert np.max(np.abs(E - Eo)) < (1e-11 if prec == "c128" else 1e-5) * np.max(np.abs(Eo))
    dV = np.prod([cell[i] / n[i] for i in range(3)])
    for k in range(2):
        W = psi[k].reshape(n_orb, -1)
        assert np.max(np.abs(dV * (W @ W.conj().T) - np.eye(n_orb))) < (1e-12 if prec == "c128" else 2e-6)
