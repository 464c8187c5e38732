"""Eq. 1 and its adjoint in wide tiles, on either side of every change of tile
height and in every format of the weights (two FP16 parts; three BF16 parts
where weights grow with distance; pair by pair where they would overflow),
against the FP64 oracle, and with values of any scale.

Bounds: U to TOL_U = 1e-5 mm; with growing weights to 1e-4 of the patch's
largest displacement (the weights themselves: the exponent, up to 128, is
rounded at 2^-24 of itself); gradients as in the other adjoint tests.  A power
of two in dL/dU is a power of two in every gradient, bit for bit."""
import numpy as np
import pytest

import scenes
from scenes import MODE_DECAY_ONLY, MODE_FULL
from tests.gpu_util import TOL_U, gpu_step, log, make_plan
from tests.test_gpu_backward import _close, gpu_step_backward
from tests.test_gpu_forward_shapes import _patches, _spheres

pytestmark = pytest.mark.gpu

SIZES = (1000, 257, 64, 300, 33, 7)


def _sparse(envs, live):
    """The scene of `envs` envs of which about `live` have objects, and those envs."""
    mesh = _patches(SIZES, pitch=1.0)
    scene = _spheres(mesh, envs, 2, 8)
    keep = np.unique(np.linspace(0, envs - 1, live).astype(int))
    off = np.setdiff1d(np.arange(envs), keep)
    scene.n_obj[off] = 0
    return mesh, scene, keep


@pytest.mark.parametrize("alpha", [None, -0.05, -1.0, -3.0])
@pytest.mark.parametrize("envs", [128, 1024, 4096, 4099])
def test_forward(oracle_lib, envs, alpha):
    mesh, scene, keep = _sparse(envs, 70)
    model = scenes.draw_model(np.random.default_rng(7), mesh.pitch, MODE_FULL if alpha is None else MODE_DECAY_ONLY)
    if alpha is not None:
        model.alpha[:] = alpha
    u, cobj, _ = gpu_step(make_plan(mesh, envs, 2), scene, model)
    ref = oracle_lib.forward(mesh, scene.select(keep), model)
    assert np.array_equal(cobj[keep], ref["contact_obj"])
    worst = 0.0
    for k in range(mesh.n_patches):
        sl = slice(int(mesh.patch_offset[k]), int(mesh.patch_offset[k + 1]))
        err = np.abs(u[:, keep, sl] - ref["u"][:, :, sl]).max(axis=(0, 2))
        bound = TOL_U if alpha is None else 1e-4 * np.abs(ref["u"][:, :, sl]).max(axis=(0, 2)) + 1e-6
        worst = max(worst, float((err / bound).max()))
    log(f"[gpu] wide forward, {envs} envs, alpha {alpha}: worst error / bound {worst:.2e}")
    assert worst <= 1.0
    assert not u[:, np.setdiff1d(np.arange(envs), keep)].any()


@pytest.mark.parametrize("alpha", [None, -0.05, -1.0, -3.0])
@pytest.mark.parametrize("envs", [128, 1023, 1024])
def test_adjoint(oracle_lib, envs, alpha):
    mesh, scene, keep = _sparse(envs, 20)
    model = scenes.draw_model(np.random.default_rng(7), mesh.pitch, MODE_DECAY_ONLY)
    if alpha is not None:
        model.alpha[:] = alpha
    w = np.random.default_rng(1).standard_normal((3, envs, mesh.n_nodes)).astype(np.float32)
    moderate = alpha is None or alpha == -0.05      # the others' gradients reach 1e30 by themselves
    if moderate:
        w[:, keep[1]] *= 1e-12
        w[:, keep[2]] *= 1e12
    plan = make_plan(mesh, envs, 2, backward=True)
    g = gpu_step_backward(plan, scene, model, w)
    log(f"[gpu] wide adjoint, {envs} envs, alpha {alpha}")
    for i, e in enumerate(keep):      # env by env: their scales differ
        ref = oracle_lib.backward(mesh, scene.select(keep[i:i + 1]), model, w[:, keep[i:i + 1]])
        for name in ("grad_rot", "grad_trans"):
            top = max(float(np.abs(ref[name]).max()), 1e-30)
            _close(g[name][e:e + 1] / top, ref[name] / top, name)
    if moderate:
        for s in (2.0 ** 60, 2.0 ** -60):
            h = gpu_step_backward(plan, scene, model, w * np.float32(s))
            for name in ("grad_rot", "grad_trans", "grad_alpha"):
                assert np.array_equal(h[name], g[name] * np.float32(s)), (name, s)
