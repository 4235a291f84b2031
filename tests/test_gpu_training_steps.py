"""The two-launch training step and the linear fit's Cholesky by panels at the
edges of their tiles, against the FP64 oracle."""
import numpy as np
import pytest

from oracle import surrogate
from paper_1804_01404_amd.binding import Surrogate
from synth.configs import surrogate_init
from synth.systems import rng_for

pytestmark = pytest.mark.gpu


# (window, hidden, trajectories, samples each): one and several 16-wide tiles of
# window, hidden layer and batch with and without remainders, the largest shapes
# that take two launches and one past each of them
@pytest.mark.parametrize("W,H,n_traj,T", [(1, 1, 1, 1), (16, 16, 2, 16), (17, 15, 3, 11), (33, 17, 5, 7), (64, 48, 2, 40),
                                          (50, 64, 3, 33), (20, 65, 3, 9), (1024, 8, 2, 21), (1025, 8, 2, 21),
                                          (12, 6, 4, 1024), (12, 6, 17, 241)])
@pytest.mark.parametrize("freeze", [False, True])
def test_training_steps_match_oracle(W, H, n_traj, T, freeze):
    rng = rng_for(61, W, H, T)
    A, J = rng.normal(size=(n_traj, T)), rng.normal(size=(n_traj, T))
    th0 = surrogate_init(W, H, 5)
    th0[-(W + 1):] = 0.1 * rng.normal(size=W + 1)
    lr, eps, steps = 1e-2, 1e-2, 3
    # one batch an epoch: the samples' order does not matter
    with Surrogate(W, H, th0, lr=lr, eps=eps) as nn:
        losses = nn.train(A, J, epochs=steps, batch=n_traj * T, freeze_linear=freeze)
        got = nn.params()
    X, Y = surrogate.windows(A, J, W)
    th = th0.astype(np.float64)
    m, v = np.zeros_like(th), np.zeros_like(th)
    ref = []
    for t in range(1, steps + 1):
        loss, g = surrogate.loss_and_grad(th, X, Y, W, H)
        if freeze:
            g[-(W + 1):] = 0.0
        th, m, v = surrogate.adam_step(th, g, m, v, t, lr=lr, eps=eps)
        ref.append(loss)
    # a gradient of order one carries 1e-6 in FP32; lr / eps = 1 passes that on
    # to the parameters at each of the three steps
    assert np.max(np.abs(got - th)) < 1e-5
    assert np.max(np.abs(losses - ref)) < 1e-5 * max(ref)


# the matrix has W + 1 columns in panels of 32: one panel, exact multiples, one
# more or less, windows longer than the series, lags beyond one scan block
@pytest.mark.parametrize("W,n_traj,T", [(1, 2, 5), (30, 4, 60), (31, 4, 60), (32, 4, 60), (63, 3, 300), (64, 3, 257),
                                        (100, 9, 40), (95, 2, 600)])
def test_linear_fit_panels_match_oracle(W, n_traj, T):
    rng = rng_for(62, W, T)
    A, J = rng.normal(size=(n_traj, T)), rng.normal(size=(n_traj, T))
    lam = 1e-3 if n_traj * T < 10 * W else 1e-10
    with Surrogate(W, 3, surrogate_init(W, 3, 1), a_scale=2.0, j_scale=0.5) as nn:
        nn.fit_linear(A, J, a_fit=100.0, lambda_rel=lam)
        p = nn.params()
    ws, b3 = surrogate.fit_linear(A, J, W, 2.0, 0.5, 100.0, lambda_rel=lam)
    # white-noise windows: a well-conditioned matrix, FP32 weights
    scale = max(np.max(np.abs(ws)), abs(b3))
    assert np.max(np.abs(p[-W:] - ws)) < 1e-6 * scale
    assert abs(p[-W - 1] - b3) < 1e-6 * scale
