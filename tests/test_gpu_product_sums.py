"""Sums of Eq. 1 and its adjoint over many nodes keep FP64 between blocks of 32
terms: their error does not grow with the number of blocks.

With alpha = 0 every weight is exactly 1 and a value is the sum of its three
parts exactly, so what is left are the roundings of the sums.  A block's sum is
rounded by one matrix instruction (its own partial roundings stay within two
units of the last place, 2 x 2^-23), the result once more (2^-24): 2^-22 + 2^-24
of the sum of |terms|.  dL/dalpha also has the distances' roundings (the
square, its root and the product with the weight, 2^-24 to 2^-23 each) and
sums over the nodes in FP64: 2^-21."""
import numpy as np
import pytest

from tests.gpu_util import log
from tests.test_gpu_product_range import Pad

pytestmark = pytest.mark.gpu

BOUND, BOUND_ALPHA = 2.0 ** -22 + 2.0 ** -24, 2.0 ** -21


@pytest.mark.parametrize("envs", [24, 128, 1024])
def test_forward(envs):
    pad = Pad(89, 23, alpha=0.0)
    active = np.arange(pad.N) < 2000
    uhat = np.where(active, np.random.default_rng(5).uniform(0.5, 1.5, (3, envs, pad.N)), 0).astype(np.float32)
    u = pad.forward(active, uhat)
    ref = uhat.astype(np.float64).sum(-1)
    err = np.abs(u[:, :, 2000:pad.n] - ref[..., None]) / ref[..., None]
    log(f"[gpu] {envs} envs: error / sum {err.max():.2e} (rms {np.sqrt((err ** 2).mean()):.2e}), bound {BOUND:.2e}")
    assert err.max() <= BOUND


@pytest.mark.parametrize("envs", [24, 128, 1024])
def test_adjoint(envs):
    pad = Pad(89, 23, alpha=0.0)
    active = np.arange(pad.N) < 40
    rng = np.random.default_rng(6)
    uhat = np.where(active, rng.uniform(0.5, 1.5, (3, envs, pad.N)), 0).astype(np.float32)
    grad = np.where(active, 0, rng.uniform(0.5, 1.5, (3, envs, pad.N))).astype(np.float32)
    grad[:, :, pad.n:] = 0
    gh, ga = pad.backward(active, uhat, grad)
    ref = grad.astype(np.float64).sum(-1)
    err = np.abs(gh[:, :, :40] - ref[..., None]) / ref[..., None]
    u64, g64 = uhat[:, :, :40].astype(np.float64), grad[:, :, 40:pad.n].astype(np.float64)
    alpha = -(u64 * (g64 @ pad.dist[40:, :40])).sum()
    ea = abs(ga[0] - alpha) / abs(alpha)
    log(f"[gpu] {envs} envs: error / sum {err.max():.2e} (rms {np.sqrt((err ** 2).mean()):.2e}), alpha {ea:.2e}")
    assert err.max() <= BOUND
    assert ea <= BOUND_ALPHA
