"""Eq. 1 and its adjoint where an item's weights and values span many orders of
magnitude: every sum is good to a part of the sum of its own |terms|, however
small that is next to the item's largest weight or value.

Bound: 2^-17 of the sum of |terms|.  A weight and a value are good to 2^-22
(the exponential's and the operands' roundings), and a sum of 32-term blocks
rounds each of its at most 32 x 6 additions to 2^-23 of itself: 2^-15.5 if all
of them fell the same way, a tenth of that as they fall."""
import numpy as np
import pytest

from tests.gpu_util import log, to_dev, torch_dev

pytestmark = pytest.mark.gpu

NX, NY = 40, 25
BOUND = 2.0 ** -17


class Pad:
    """A flat patch of NX x NY nodes 1 mm apart and a small one beside it."""

    def __init__(self, nx=NX, ny=NY, alpha=1.0):
        x, y = (a.ravel() for a in np.meshgrid(np.arange(nx), np.arange(ny)))
        self.n = nx * ny
        self.N = self.n + 7
        self.pos = np.zeros((3, self.N), np.float32)
        self.pos[0, :self.n], self.pos[1, :self.n] = x, y
        self.pos[0, self.n:] = 200.0 + np.arange(7)
        self.nrm = np.zeros((3, self.N), np.float32)
        self.nrm[2] = 1.0
        self.alpha = np.full(2, alpha, np.float32)
        p = self.pos[:, :self.n].astype(np.float64)
        self.dist = np.sqrt(((p[:, :, None] - p[:, None, :]) ** 2).sum(0))
        self.w = np.exp(-float(self.alpha[0]) * self.dist)

    def plan(self, envs, backward=False):
        from paper_2604_20295_amd import _native
        off = np.array([0, self.n, self.N], np.int32)
        origin = np.array([[NX / 2, NY / 2, 0], [203, 0, 0]], np.float32)
        return _native.Plan(off, self.pos, self.nrm, origin, envs, 1, backward)

    def forward(self, active, uhat):
        """U of given contact results, decay only: active [N], uhat [3][E][N]."""
        from paper_2604_20295_amd import _native
        torch, dev = torch_dev()
        E = uhat.shape[1]
        plan = self.plan(E)
        cobj = to_dev(np.tile(np.where(active, 0, -1).astype(np.int8), (E, 1)))
        u = torch.full((3, E, self.N), float("nan"), device=dev)
        _native.etac_propagate(plan, plan.model_struct(1, to_dev(self.alpha), None), E, cobj, to_dev(uhat), u)
        torch.cuda.synchronize()
        return u.cpu().numpy().astype(np.float64)

    def backward(self, active, uhat, grad_u):
        """(dL/du_hat, dL/dalpha) of the same."""
        from paper_2604_20295_amd import _native
        torch, dev = torch_dev()
        E = uhat.shape[1]
        plan = self.plan(E, backward=True)
        cobj = to_dev(np.tile(np.where(active, 0, -1).astype(np.int8), (E, 1)))
        gh = torch.full((3, E, self.N), float("nan"), device=dev)
        ga = torch.full((2,), float("nan"), device=dev)
        _native.etac_propagate_backward(plan, plan.model_struct(1, to_dev(self.alpha), None), E, cobj, to_dev(uhat),
                                        to_dev(grad_u), gh, ga, None)
        torch.cuda.synchronize()
        return gh.cpu().numpy().astype(np.float64), ga.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("envs", [20, 130, 1030])
def test_weights_far_below_the_largest(envs):
    pad = Pad()
    active = pad.pos[0] < 4
    rng = np.random.default_rng(3)
    uhat = np.where(active, rng.uniform(-1, 1, (3, envs, pad.N)), 0).astype(np.float32)
    u = pad.forward(active, uhat)
    a, p = np.flatnonzero(active[:pad.n]), np.flatnonzero(~active[:pad.n])
    worst = 0.0
    for e in (0, 1, envs // 2, envs - 1):
        v = uhat[:, e][:, a].astype(np.float64)
        ref, size = v @ pad.w[a][:, p], np.abs(v) @ pad.w[a][:, p]
        worst = max(worst, float((np.abs(u[:, e][:, p] - ref) / size).max()))
    log(f"[gpu] {envs} envs, weights to 2^{np.log2(pad.w[a][:, p].min()):.0f}: error / sum|terms| {worst:.2e}")
    assert worst <= BOUND


@pytest.mark.parametrize("envs", [20, 130, 1030])
def test_gradients_far_below_the_largest(envs):
    pad = Pad(alpha=2.0)
    active = pad.pos[0] < 4
    rng = np.random.default_rng(4)
    uhat = np.where(active, rng.uniform(-1, 1, (3, envs, pad.N)), 0).astype(np.float32)
    # a billion times larger where no weight is left of it
    grad = np.where(active, 0, rng.uniform(-1, 1, (3, envs, pad.N)) * np.where(pad.pos[0] > 30, 1e9, 1.0)).astype(np.float32)
    gh, _ = pad.backward(active, uhat, grad)
    a, p = np.flatnonzero(active[:pad.n]), np.flatnonzero(~active[:pad.n])
    worst = 0.0
    for e in (0, 1, envs // 2, envs - 1):
        v = grad[:, e][:, p].astype(np.float64)
        ref, size = v @ pad.w[p][:, a], np.abs(v) @ pad.w[p][:, a]
        worst = max(worst, float((np.abs(gh[:, e][:, a] - ref) / size).max()))
    log(f"[gpu] {envs} envs: error / sum|terms| {worst:.2e}")
    assert worst <= BOUND
