"""A plan's regressor rows stay within 256 MB, or one row per item, whatever the
patches' sizes; the longer units of such plans give the same taxels (the
online softmax over twice, four, eight times the nodes: 1e-5 of the largest
output, FP32 sums of a few hundred terms in another order)."""
import numpy as np
import pytest

import scenes
from tests.gpu_util import log, make_plan, to_dev, torch_dev
from tests.test_gpu_forward_shapes import _patches

pytestmark = pytest.mark.gpu


def _pads(side, count):
    return _patches((side * side,) * count, pitch=0.125, gap=60.0)


@pytest.mark.parametrize("side,count,envs,most", [(128, 4, 4096, 1.75e9), (32, 16, 4096, 0.62e9), (16, 8, 64, 0.05e9)])
def test_scratch_of_forward_plans(side, count, envs, most):
    plan = make_plan(_pads(side, count), envs, 4)
    got = plan.info()["scratch_bytes"]
    log(f"[gpu] {envs} envs of {count} {side} x {side} patches: {got / 1e9:.2f} GB")
    assert got <= most
    plan.close()


@pytest.mark.parametrize("side,envs", [(128, 1100), (64, 20000), (33, 40000)])
def test_longer_units(side, envs):
    # the same five envs through a small plan and through one with longer units
    from paper_2604_20295_amd import _native
    torch, dev = torch_dev()
    mesh = _pads(side, 4)
    rng = np.random.default_rng(2)
    reg = to_dev((rng.standard_normal(_native.ETAC_REG_SIZE) * 0.06).astype(np.float32))
    u = to_dev((0.3 * rng.standard_normal((3, 5, mesh.n_nodes))).astype(np.float32))
    na = to_dev(np.array([[1, 5, 0, 2], [0, 0, 0, 1], [3, 3, 3, 3], [1, 0, 0, 0], [9, 9, 0, 9]], np.int32))
    out = []
    for n in (5, envs):
        plan = make_plan(mesh, n, 1)
        y = torch.full((5, 4, 8), float("nan"), device=dev)
        _native.etac_regress(plan, reg, u, na, y)
        torch.cuda.synchronize()
        out.append(y.cpu().numpy().astype(np.float64))
        plan.close()
    err = np.abs(out[1] - out[0]).max() / np.abs(out[0]).max()
    log(f"[gpu] units of {envs} envs of four {side} x {side} pads: {err:.1e} of the largest output")
    assert err <= 1e-5
