"""The adjoint's kernels at the edges of their tiles and of their dispatch,
against the FP64 oracle's adjoint: patches around one node, one 16-node tile,
one 64-node word and block and the last patch with a decay matrix (2048
nodes), batches on either side of every change of launch (the small batch
that lists every item, wide tiles from 128 envs, longer env chunks from 256),
with the forward's pooling record and without, and weights that grow with
distance.

Bounds as for the other adjoint tests: 1e-4 of the block's largest gradient
plus 1e-6, on envs whose ReLU and arg-max decisions clear MARGIN (decay-only:
every env).  Growing weights: 1e-4 of the largest gradient (the exponent, up
to 128, is rounded at 2^-24 of itself, so a weight is good to 5e-6)."""
import numpy as np
import pytest

import scenes
from scenes import MODE_DECAY_ONLY, MODE_FULL, MODE_RESIDUAL_ONLY
from tests.gpu_util import log, make_plan
from tests.test_gpu_backward import _close, _compare_all, clean_scene, gpu_step_backward
from tests.test_gpu_forward_shapes import _patches, _spheres

pytestmark = pytest.mark.gpu


def _run(oracle_lib, mesh, scene, model, seed, least=1):
    sc, n_clean = clean_scene(oracle_lib, mesh, scene, model)
    log(f"[gpu]   envs compared {n_clean}/{scene.n_envs}")
    assert n_clean >= least
    w = np.random.default_rng(seed).standard_normal((3, scene.n_envs, mesh.n_nodes))
    plan = make_plan(mesh, scene.n_envs, scene.max_obj, backward=True)
    g = gpu_step_backward(plan, sc, model, w)
    _compare_all(g, oracle_lib.backward(mesh, sc, model, w), model.mode)
    if model.mode != MODE_DECAY_ONLY:
        g2 = gpu_step_backward(plan, sc, model, w, saved=True)
        for k in g:
            assert np.array_equal(g[k], g2[k]), k


@pytest.mark.parametrize("mode", [MODE_FULL, MODE_DECAY_ONLY, MODE_RESIDUAL_ONLY])
@pytest.mark.parametrize("sizes", [(1, 2, 15, 16, 17, 63, 64, 65), (127, 128, 129, 31, 33)])
def test_patch_sizes(oracle_lib, sizes, mode):
    mesh = _patches(sizes)
    model = scenes.draw_model(np.random.default_rng(5), mesh.pitch, mode)
    log(f"[gpu] adjoint, patches {sizes} mode {mode}")
    _run(oracle_lib, mesh, _spheres(mesh, 24, 2, 3), model, 1)


@pytest.mark.parametrize("sizes", [(2048, 64), (2049, 64)])
def test_largest_matrix_patch(oracle_lib, sizes):
    mesh = _patches(sizes)
    model = scenes.draw_model(np.random.default_rng(5), mesh.pitch, MODE_DECAY_ONLY)
    log(f"[gpu] adjoint, patches {sizes}")
    _run(oracle_lib, mesh, _spheres(mesh, 6, 1, 3), model, 2)
    # full model: both patch kinds agree with the oracle where the decisions are clear
    _run(oracle_lib, mesh, _spheres(mesh, 60, 1, 9), model.with_mode(MODE_FULL), 2)


@pytest.mark.parametrize("envs", [1, 17, 65, 127, 128, 255, 256, 289])
def test_batch_sizes(oracle_lib, envs):
    mesh = _patches((64, 65, 17, 33))
    log(f"[gpu] adjoint, {envs} envs")
    for mode in (MODE_DECAY_ONLY, MODE_FULL):
        model = scenes.draw_model(np.random.default_rng(6), mesh.pitch, mode)
        _run(oracle_lib, mesh, _spheres(mesh, envs, 2, 4), model, 3, least=0 if envs == 1 else 1)


@pytest.mark.parametrize("alpha", [-0.05, -3.0])
@pytest.mark.parametrize("envs", [3, 130])
def test_growing_weights(oracle_lib, envs, alpha):
    mesh = _patches((1000, 300), pitch=1.0)
    scene = _spheres(mesh, envs, 1, 8)
    scene.n_obj[12:] = 0
    model = scenes.draw_model(np.random.default_rng(7), mesh.pitch, MODE_DECAY_ONLY)
    model.alpha[:] = alpha
    w = np.random.default_rng(1).standard_normal((3, envs, mesh.n_nodes))
    plan = make_plan(mesh, envs, 1, backward=True)
    g, ref = gpu_step_backward(plan, scene, model, w), oracle_lib.backward(mesh, scene, model, w)
    log(f"[gpu] adjoint, alpha {alpha}, {envs} envs")
    for name in ("grad_rot", "grad_trans", "grad_alpha"):
        _close(g[name], ref[name], name)
