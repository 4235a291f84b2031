"""Calls on a live context that run out of device memory: they return ENOMEM
without poisoning the context, and the context is as it was, so that the call
can be repeated and the results are a run's that never failed, bit for bit."""
import numpy as np
import pytest

from gpu_helpers import announce
from oracle_helpers import tiny_periodic
from paper_1804_01404_amd import binding

pytestmark = pytest.mark.gpu


class Refuser:
    """Device allocations by torch, of which number `at` (from the last arm()
    on) is refused once."""

    def __init__(self, monkeypatch):
        self.at, self.count = None, 0
        real = binding._TorchMemory._alloc

        def alloc(mem, nbytes, user):
            self.count += 1
            if self.at is not None and self.count - 1 == self.at:
                self.at = None
                return None
            return real(mem, nbytes, user)
        monkeypatch.setattr(binding._TorchMemory, "_alloc", alloc)

    def arm(self, at):
        self.at, self.count = at, 0

    def refused(self):
        return self.at is None


def _enomem(call):
    with pytest.raises(binding.TDDFTError) as e:
        call()
    assert e.value.status == binding.ENOMEM


@pytest.mark.parametrize("fail_at", [0, 1, 2])
def test_ground_state(fail_at, monkeypatch):
    s = tiny_periodic(n=12, nsteps=1)
    announce(f"ground state, allocation {fail_at} refused")
    with binding.TDDFT(s) as t:
        t.set_potential()
        E0, psi0 = t.ground_state(2, 0.01), t.orbitals()
    mem = Refuser(monkeypatch)
    with binding.TDDFT(s) as t:
        t.set_potential()
        mem.arm(fail_at)
        _enomem(lambda: t.ground_state(2, 0.01))
        assert mem.refused()
        assert np.array_equal(t.ground_state(2, 0.01), E0)
        assert np.array_equal(t.orbitals(), psi0)


@pytest.mark.parametrize("fail_at", [0, 1])
def test_longer_propagate(fail_at, monkeypatch):
    """The A and J tables of a call longer than any before it; shorter calls go
    on with the old ones."""
    s = tiny_periodic(n=12, nsteps=16, A=np.cumsum(np.full((17, 3), 0.1), axis=0))
    calls = [s.A[:3], s.A[2:5], s.A[4:16]]
    announce(f"longer propagate, allocation {fail_at} refused")
    with binding.TDDFT(s) as t:
        t.set_potential()
        J0, psi0 = [t.propagate(A) for A in calls], t.orbitals()
    mem = Refuser(monkeypatch)
    with binding.TDDFT(s) as t:
        t.set_potential()
        J = [t.propagate(calls[0])]
        mem.arm(fail_at)
        _enomem(lambda: t.propagate(calls[2]))
        assert mem.refused()
        J += [t.propagate(A) for A in calls[1:]]
        assert all(np.array_equal(a, b) for a, b in zip(J, J0))
        assert np.array_equal(t.orbitals(), psi0)


@pytest.mark.parametrize("flags,fail_at", [(0, 0), (0, 5), (0, 7), (0, 12), (0, 14), (8, 6), (8, 7), (8, 13)])
def test_replaced_potential(flags, fail_at, monkeypatch):
    """A second potential that is refused (no memory, or unstable at this dt)
    leaves the first one in place: on the LDS-resident step and on the
    per-stage kernels (flags 8), with more atoms than before and less."""
    nsteps = 6
    A = np.cumsum(np.full((nsteps + 1, 3), 0.2), axis=0)
    s = tiny_periodic(n=12, nsteps=nsteps, A=A)
    other = tiny_periodic(n=12, n_atoms=1 if fail_at % 2 else 5, seed=103)
    announce(f"second potential, flags {flags}, allocation {fail_at} refused")

    def second(t):
        t.set_potential(other.v_loc, other.projectors)
    with binding.TDDFT(s, flags=flags) as t:
        t.set_potential()
        J0 = [t.propagate(A[:3]), t.propagate(A[2:5])]
        second(t)
        J0.append(t.propagate(A[4:]))
        psi0 = t.orbitals()
    mem = Refuser(monkeypatch)
    with binding.TDDFT(s, flags=flags) as t:
        mem.arm(fail_at)
        _enomem(lambda: second(t))
        with pytest.raises(binding.TDDFTError) as e:  # still without a potential
            t.propagate(A[:3])
        assert e.value.status == binding.ESTATE
        t.set_potential()
        J = [t.propagate(A[:3])]
        mem.arm(fail_at)
        _enomem(lambda: second(t))
        assert mem.refused()
        with pytest.raises(binding.TDDFTError) as e:
            t.set_potential(other.v_loc - 1e4, other.projectors)
        assert e.value.status == binding.EUNSTABLE
        J.append(t.propagate(A[2:5]))
        second(t)
        J.append(t.propagate(A[4:]))
        assert all(np.array_equal(a, b) for a, b in zip(J, J0))
        assert np.array_equal(t.orbitals(), psi0)


def test_refused_network_workspace():
    """A batch whose workspace exceeds the device (35 TB) is ENOMEM, and the
    refusal is not reported by what the thread launches next."""
    W, H = 4096, 2
    rng = np.random.default_rng(5)
    x = rng.normal(size=(3, W)).astype(np.float32)
    s = tiny_periodic(n=8, nsteps=1)
    announce("network workspace beyond the device")
    with binding.Surrogate(W, H, 0.01 * rng.normal(size=binding.nn_num_params(W, H))) as nn, binding.TDDFT(s) as t:
        t.set_potential()
        y0 = nn.forward(x)
        out = np.empty(3, dtype=np.float32)

        def huge():
            nn._check(nn.lib.tddft_nn_forward(nn.h, 2**31 - 1, binding._fptr(x), binding._fptr(out)))
        _enomem(huge)
        assert np.all(np.isfinite(t.propagate(s.A)))
        _enomem(huge)
        assert np.array_equal(nn.forward(x), y0)
