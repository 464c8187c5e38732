"""Infinite, NaN and very large values in Eq. 1 and its adjoint: what the sum of
w times the value gives, in the value's own component and env alone; every
other sum is what it is without it.

Bound of the finite sums: 2^-17 of the sum of |terms|, as in the range tests."""
import numpy as np
import pytest

from tests.gpu_util import log
from tests.test_gpu_product_range import BOUND, Pad

pytestmark = pytest.mark.gpu

HUGE = np.float32(3.395e38)      # rounds to infinity in eight bits


def _poke(a, node, other):
    """Values in envs 1 to 4: an infinity, both of them, a NaN, a huge one."""
    a[0, 1, node] = np.inf
    a[1, 2, node], a[1, 2, other] = np.inf, -np.inf
    a[2, 3, node] = np.nan
    a[0, 4, node] = HUGE


def _compare(got, v, w):
    """got [n], v [m] values, w [m][n] weights."""
    with np.errstate(invalid="ignore"):
        ref, size = (v[:, None] * w).sum(0), (np.abs(v)[:, None] * w).sum(0)
    odd = ~np.isfinite(ref)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[odd & ~np.isnan(ref)], ref[odd & ~np.isnan(ref)])
    return float((np.abs(got - ref)[~odd] / size[~odd]).max()) if (~odd).any() else 0.0


@pytest.mark.parametrize("envs", [20, 130, 1030])
def test_forward(envs):
    pad = Pad(alpha=0.5)
    active = pad.pos[0] < 4
    a, p = np.flatnonzero(active[:pad.n]), np.flatnonzero(~active[:pad.n])
    uhat = np.where(active, np.random.default_rng(8).uniform(-1, 1, (3, envs, pad.N)), 0).astype(np.float32)
    _poke(uhat, a[10], a[50])
    u = pad.forward(active, uhat)
    worst = 0.0
    for e in list(range(6)) + [envs - 1]:
        for c in range(3):
            worst = max(worst, _compare(u[c, e, p], uhat[c, e, a].astype(np.float64), pad.w[a][:, p]))
    log(f"[gpu] {envs} envs: error / sum|terms| of the finite sums {worst:.2e}")
    assert worst <= BOUND


@pytest.mark.parametrize("envs", [20, 130, 1030])
def test_adjoint(envs):
    pad = Pad(alpha=0.5)
    active = pad.pos[0] < 4
    a, p = np.flatnonzero(active[:pad.n]), np.flatnonzero(~active[:pad.n])
    rng = np.random.default_rng(9)
    uhat = np.where(active, rng.uniform(-1, 1, (3, envs, pad.N)), 0).astype(np.float32)
    grad = np.where(active, 0, rng.uniform(-1, 1, (3, envs, pad.N))).astype(np.float32)
    _poke(grad, p[10], p[500])
    gh, _ = pad.backward(active, uhat, grad)
    worst = 0.0
    for e in list(range(6)) + [envs - 1]:
        for c in range(3):
            worst = max(worst, _compare(gh[c, e, a], grad[c, e, p].astype(np.float64), pad.w[p][:, a]))
    log(f"[gpu] {envs} envs: error / sum|terms| of the finite sums {worst:.2e}")
    assert worst <= BOUND
