"""The contact pass at the surface sizes where its kernels change: 32 words of
64 nodes with several workgroups an env, 64 with one (from 1024 envs on), and
16 words, up to which a step's tables and contact share a launch.  Bit for bit
the step's contact, and the oracle's."""
import numpy as np
import pytest

import scenes
from tests.gpu_util import gpu_contact, gpu_step, log, make_plan, max_err
from tests.test_gpu_forward_shapes import _patches, _spheres

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("words,envs", [(1, 1), (1, 1100), (16, 3), (17, 3), (32, 3), (33, 3), (32, 1023), (33, 1023),
                                        (64, 1024), (65, 1024)])
def test_contact(oracle_lib, words, envs):
    sizes = (64 * words - 7,) if words < 16 else (64 * 10 - 3, 64 * (words - 11) - 1, 50)
    mesh = _patches(sizes)
    scene = _spheres(mesh, envs, 2, 3)
    plan = make_plan(mesh, envs, 2)
    cobj, uhat, na = gpu_contact(plan, scene)
    model = scenes.draw_model(np.random.default_rng(6), mesh.pitch, scenes.MODE_DECAY_ONLY)
    _, c2, n2 = gpu_step(plan, scene, model)
    some = np.unique(np.linspace(0, envs - 1, 40).astype(int))
    ref, u_ref, n_ref = oracle_lib.contact(mesh, scene.select(some))
    assert np.array_equal(cobj[some], ref) and np.array_equal(na[some], n_ref)
    assert np.array_equal(cobj, c2) and np.array_equal(na, n2)
    err = max_err(uhat[:, some], u_ref)
    log(f"[gpu] {words} words, {envs} envs: active {int(na.sum())}, max|du_hat| {err:.1e}")
    assert err <= 1e-6
