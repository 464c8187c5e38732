"""The wide products' units on surfaces of few row blocks or few envs in
contact and on either side of the change of tile height: forward and adjoint
against the FP64 oracle on sampled envs, and no node of any env left out."""
import numpy as np
import pytest

import scenes
from scenes import MODE_DECAY_ONLY
from tests.gpu_util import TOL_U, gpu_step, log, make_plan
from tests.test_gpu_backward import _close, gpu_step_backward
from tests.test_gpu_forward_shapes import _patches, _spheres

pytestmark = pytest.mark.gpu


# one to four row blocks of 64 or 128 nodes, one group of 32 envs to several
@pytest.mark.parametrize("sizes", [(64,), (250,), (256, 130), (300, 64, 513), (64,) * 9])
@pytest.mark.parametrize("envs", [128, 200, 1500, 5000])
def test_every_unit(oracle_lib, sizes, envs):
    mesh = _patches(sizes)
    scene = _spheres(mesh, envs, 2, 3)
    model = scenes.draw_model(np.random.default_rng(6), mesh.pitch, MODE_DECAY_ONLY)
    plan = make_plan(mesh, envs, 2, backward=True)
    u, cobj, na = gpu_step(plan, scene, model)
    assert np.isfinite(u).all()
    some = np.unique(np.linspace(0, envs - 1, 60).astype(int))
    ref = oracle_lib.forward(mesh, scene.select(some), model)
    assert np.array_equal(cobj[some], ref["contact_obj"])
    err = float(np.abs(u[:, some] - ref["u"]).max())
    # weights are positive: a passive node of a touched patch that no unit took would be exactly zero
    for k in range(mesh.n_patches):
        sl = slice(int(mesh.patch_offset[k]), int(mesh.patch_offset[k + 1]))
        hit = na[:, k] > 0
        assert (np.abs(u[:, hit, sl]).max(axis=0) > 0).all()
    w = np.random.default_rng(1).standard_normal((3, envs, mesh.n_nodes)).astype(np.float32)
    g = gpu_step_backward(plan, scene, model, w)
    back = oracle_lib.backward(mesh, scene.select(some), model, w[:, some])
    log(f"[gpu] patches {sizes}, {envs} envs: max|dU| {err:.2e}")
    assert err <= TOL_U
    for name in ("grad_rot", "grad_trans"):
        _close(g[name][some], back[name], name)
    full = oracle_lib.backward(mesh, scene, model, w) if envs <= 200 else None
    if full is not None:
        _close(g["grad_alpha"], full["grad_alpha"], "grad_alpha")
