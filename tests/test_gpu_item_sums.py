"""Parameter gradients are summed over the items in FP64: items a million times
larger that cancel each other leave the sum of the others untouched.

The large items come in pairs, the same scene with dL/dU negated, in the two
halves of the batch.  What an item adds to the sums are each other's negatives
bit for bit (its FP32 operations are odd in dL/dU), so what is left is the
gradient of the small envs: the usual bounds of the adjoint tests, against the
FP64 oracle on those alone.  Residual network alone: Eq. 1's matrix products
round an item's own sums, and not alike for both signs."""
import numpy as np
import pytest

import scenes
from scenes import MODE_RESIDUAL_ONLY
from tests.gpu_util import log, make_plan
from tests.test_gpu_backward import _close, clean_scene, gpu_step_backward
from tests.test_gpu_forward_shapes import _patches, _spheres

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pairs", [40, 400, 3000])
def test_large_items_that_cancel(oracle_lib, pairs):
    mesh = _patches((64, 65, 17, 33))
    model = scenes.draw_model(np.random.default_rng(6), mesh.pitch, MODE_RESIDUAL_ONLY)
    base = _spheres(mesh, 90, 2, 4)
    clean, n = clean_scene(oracle_lib, mesh, base, model)
    assert n >= 8
    small = np.flatnonzero(clean.n_obj > 0)[:8]
    large = np.resize(np.setdiff1d(np.flatnonzero(base.n_obj > 0), small), pairs)
    # the large envs, each small one among them, the large ones again
    slots = np.linspace(0, 2 * pairs, 8).astype(int)
    order = np.insert(np.concatenate([large, large]), slots, small)
    sign = np.insert(np.concatenate([np.ones(pairs), -np.ones(pairs)]), slots, np.zeros(8))
    scene = base.select(order)
    g = np.random.default_rng(1).standard_normal((3, 90, mesh.n_nodes)).astype(np.float32)
    w = g[:, order] * np.where(sign == 0, 1.0, sign * 2.0 ** 20).astype(np.float32)[None, :, None]
    got = gpu_step_backward(make_plan(mesh, scene.n_envs, 2, backward=True), scene, model, w)
    ref = oracle_lib.backward(mesh, base.select(small), model, g[:, small])
    log(f"[gpu] {pairs} pairs of large items")
    at = np.flatnonzero(sign == 0)
    for name in ("grad_rot", "grad_trans"):
        _close(got[name][at], ref[name], name)
    # block by block: their largest gradients differ
    for name, a, b in (("W1 b1", 0, 640), ("W2 b2", 640, 4800), ("W3 b3", 4800, 8960), ("W4 b4", 8960, 17216),
                       ("W5 b5", 17216, 17411)):
        _close(got["grad_phi"][a:b], ref["grad_phi"][a:b], name)
