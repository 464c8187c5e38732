"""Eq. 1 on patches without a decay matrix (more than 2048 nodes): every number
of runs of 32 nodes within the cutoff, from one to all (alpha 0 has no cutoff),
odd counts and partial last runs, and more items than workgroups meet at once,
against the FP64 oracle with the bounds of the other forward and adjoint tests."""
import numpy as np
import pytest

import scenes
from scenes import MODE_DECAY_ONLY
from tests.gpu_util import TOL_U, gpu_step, log, make_plan
from tests.test_gpu_backward import _close, gpu_step_backward
from tests.test_gpu_forward_shapes import _patches, _spheres

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("alpha", [0.0, 0.4, 1.5, 8.0])
@pytest.mark.parametrize("sizes,envs", [((2049,), 3), ((2113, 70), 5), ((4095, 2600), 40)])
def test_runs(oracle_lib, sizes, envs, alpha):
    mesh = _patches(sizes, pitch=0.6)
    scene = _spheres(mesh, envs, 2, 11)
    model = scenes.draw_model(np.random.default_rng(7), mesh.pitch, MODE_DECAY_ONLY)
    model.alpha[:] = alpha
    some = np.arange(0, envs, max(1, envs // 5))
    u, cobj, _ = gpu_step(make_plan(mesh, envs, 2), scene, model)
    ref = oracle_lib.forward(mesh, scene.select(some), model)
    assert np.array_equal(cobj[some], ref["contact_obj"])
    top = np.abs(ref["u"]).max()
    err = np.abs(u[:, some] - ref["u"]).max()
    log(f"[gpu] far patches {sizes}, {envs} envs, alpha {alpha}: max|dU| {err:.2e} of {top:.2e}")
    assert err <= TOL_U * max(1.0, top)
    w = np.zeros((3, envs, mesh.n_nodes), np.float32)
    w[:, some] = np.random.default_rng(1).standard_normal((3, len(some), mesh.n_nodes))
    g = gpu_step_backward(make_plan(mesh, envs, 2, backward=True), scene, model, w)
    rg = oracle_lib.backward(mesh, scene.select(some), model, w[:, some])
    for name in ("grad_rot", "grad_trans"):
        _close(g[name][some], rg[name], name)
    _close(g["grad_alpha"], rg["grad_alpha"], "grad_alpha")
