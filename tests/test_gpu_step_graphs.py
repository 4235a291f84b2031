"""Steps replayed from graphs of one and of several steps against the same steps
enqueued one by one: calls of every length class in one context (shorter than,
equal to and beyond the larger graph, with and without single steps left over),
with observations and a change of the tables' size between them. Same bits."""
import numpy as np
import pytest

from oracle_helpers import tiny_periodic
from tests.gpu_helpers import announce

pytestmark = pytest.mark.gpu
NO_GRAPH, STREAMING, PC = 4, 8, 32
CALLS = [1, 2, 3, 10, 4, 1, 11, 5, 23, 8]


def _system(seed):
    rng = np.random.default_rng(seed)
    total = sum(CALLS)
    A = np.cumsum(rng.normal(size=(total + 1, 3)), axis=0)
    k = np.array([[0.1, 0.0, 0.2], [-0.2, 0.1, 0.0]])
    return tiny_periodic(n=12, L=6.0, n_orb=3, kpts=k, nsteps=total, A=A, dt=0.01, real=False, seed=seed)


def _slices(A):
    n = 0
    for c in CALLS:
        yield A[n:n + c + 1]
        n += c


@pytest.mark.parametrize("flags", [0, STREAMING, PC], ids=["fused", "streaming", "corrector"])
def test_context(flags):
    from paper_1804_01404_amd.binding import TDDFT
    s = _system(5101)
    announce(f"step graphs flags={flags}")
    got = []
    for extra in (0, NO_GRAPH):
        with TDDFT(s, precision="mixed", flags=flags | extra) as t:
            t.set_potential()
            J = []
            for A in _slices(s.A):
                J.append(t.propagate(A))
                t.density_current()
            got.append((np.concatenate(J), t.orbitals(), t.energy()))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1]) and got[0][2] == got[1][2]


def test_batch():
    from paper_1804_01404_amd.binding import TDDFT, TDDFTBatch
    systems = [_system(5102), _system(5103)]
    announce("step graphs, batch")
    with TDDFTBatch(systems, precision="mixed") as b:
        parts = [list(_slices(s.A)) for s in systems]
        J = [b.propagate([p[i] for p in parts]) for i in range(len(CALLS))]
        psi = [b.orbitals(c) for c in range(2)]
    for c, s in enumerate(systems):
        with TDDFT(s, precision="mixed", flags=NO_GRAPH) as t:
            t.set_potential()
            ref = np.concatenate([t.propagate(A) for A in _slices(s.A)])
            assert np.array_equal(np.concatenate([j[c] for j in J]), ref)
            assert np.array_equal(psi[c], t.orbitals())
