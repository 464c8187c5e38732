"""The forward's kernels at the edges of their tiles and of their dispatch,
against the FP64 oracle: patches around one node, one 16-node tile, one
64-node word, one 64- and 128-row block and the largest patch that has a decay
matrix (2048 nodes; the next one is summed pair by pair), batches on either
side of every change of launch, and decay rates whose weights grow with
distance until a matrix would overflow.

Bounds: masks and counts exact; U to TOL_U = 1e-5 mm, the bound of the other
forward tests; growing weights, whose sums are large, to 1e-4 of the patch's
largest displacement (the exponent, up to 128, is rounded at 2^-24 of itself,
so a weight is good to 128 ln 2 / 2^24 = 5e-6)."""
import numpy as np
import pytest

import scenes
from scenes import MODE_DECAY_ONLY, MODE_FULL, MODE_RESIDUAL_ONLY, SPHERE
from tests.gpu_util import TOL_U, gpu_contact, gpu_propagate, gpu_step, log, make_plan, max_err

pytestmark = pytest.mark.gpu


def _patches(sizes, pitch=0.7, gap=60.0):
    pos, nrm, offs, cen = [], [], [0], []
    for k, n in enumerate(sizes):
        nx = int(np.ceil(np.sqrt(n)))
        i = np.arange(n)
        pos.append(np.stack([(i % nx - (nx - 1) / 2.0) * pitch + gap * k, (i // nx - (nx - 1) / 2.0) * pitch,
                             0.02 * (i % 7)]))
        nrm.append(np.stack([np.zeros(n), np.zeros(n), np.ones(n)]))
        offs.append(offs[-1] + n)
        cen.append((gap * k, 0.0, 0.0))
    return scenes.Mesh(np.array(offs, np.int32), np.concatenate(pos, 1).astype(np.float32),
                       np.concatenate(nrm, 1).astype(np.float32), np.array(cen, np.float32),
                       np.full(len(sizes), pitch), [])


def _spheres(mesh, E, O, seed):
    """O spheres per env on patches in turn, every third env without any."""
    scene = scenes._empty_scene(E, O)
    rng = np.random.default_rng(seed)
    for e in range(E):
        scene.n_obj[e] = 0 if e % 3 == 2 else O
        for o in range(O):
            c = mesh.origin[(e + o) % mesh.n_patches].astype(np.float64)
            r = rng.uniform(3.0, 8.0)
            scene.type[e, o] = SPHERE
            scene.shape[e, o, 0] = r
            scene.trans[e, o] = c + np.array([rng.uniform(-3, 3), rng.uniform(-3, 3), r - rng.uniform(0.3, 2.0)])
    return scene


def _check(oracle_lib, mesh, scene, model, envs=None):
    plan = make_plan(mesh, scene.n_envs, scene.max_obj)
    u, cobj, na = gpu_step(plan, scene, model)
    c2, uh, n2 = gpu_contact(plan, scene)
    assert np.array_equal(cobj, c2) and np.array_equal(na, n2)
    assert np.array_equal(u, gpu_propagate(plan, model, c2, uh))       # the two-call form, bit for bit
    envs = np.arange(scene.n_envs) if envs is None else envs
    ref = oracle_lib.forward(mesh, scene.select(envs), model)
    assert np.array_equal(cobj[envs], ref["contact_obj"])
    assert np.array_equal(na[envs], ref["n_active"])
    err = max_err(u[:, envs], ref["u"])
    log(f"[gpu]   E={scene.n_envs} active {int(na.sum())} max|dU| {err:.2e}")
    assert err <= TOL_U


@pytest.mark.parametrize("mode", [MODE_FULL, MODE_DECAY_ONLY, MODE_RESIDUAL_ONLY])
@pytest.mark.parametrize("sizes", [(1, 2, 15, 16, 17, 63, 64, 65), (127, 128, 129, 31, 33), (2048, 2049, 64)])
def test_patch_sizes(oracle_lib, sizes, mode):
    mesh = _patches(sizes)
    model = scenes.draw_model(np.random.default_rng(5), mesh.pitch, mode)
    log(f"[gpu] forward, patches {sizes} mode {mode}")
    _check(oracle_lib, mesh, _spheres(mesh, 9, 2, 3), model)


@pytest.mark.parametrize("envs", [1, 16, 17, 127, 128, 1023, 1024])
def test_batch_sizes(oracle_lib, envs):
    mesh = _patches((64, 200, 65, 17))
    model = scenes.draw_model(np.random.default_rng(6), mesh.pitch, MODE_FULL)
    log(f"[gpu] forward, {envs} envs")
    scene = _spheres(mesh, envs, 2, 4)
    _check(oracle_lib, mesh, scene, model, np.unique(np.linspace(0, envs - 1, 40).astype(int)))


@pytest.mark.parametrize("alpha", [-0.05, -3.0])
@pytest.mark.parametrize("envs", [3, 130])
def test_growing_weights(oracle_lib, envs, alpha):
    mesh = _patches((1000, 300), pitch=1.0)
    scene = _spheres(mesh, envs, 1, 8)
    model = scenes.draw_model(np.random.default_rng(7), mesh.pitch, MODE_DECAY_ONLY)
    model.alpha[:] = alpha
    plan = make_plan(mesh, envs, 1)
    u, cobj, na = gpu_step(plan, scene, model)
    envs = np.arange(min(envs, 12))
    ref = oracle_lib.forward(mesh, scene.select(envs), model)
    log(f"[gpu] alpha {alpha}: max|U| {np.abs(ref['u']).max():.3e}")
    assert np.array_equal(cobj[envs], ref["contact_obj"])
    assert np.all(np.isfinite(u[:, envs]))
    for k in range(mesh.n_patches):
        sl = slice(int(mesh.patch_offset[k]), int(mesh.patch_offset[k + 1]))
        for e in envs:
            top = np.abs(ref["u"][:, e, sl]).max()
            assert np.abs(u[:, e, sl] - ref["u"][:, e, sl]).max() <= 1e-4 * top + 1e-6
