"""Articulated hands whose patches have more candidates than the contact pass
holds in LDS (64 rows per env) and more than one round of the pose adjoint's
64 slots: every object's bounding ball reaches every patch.  Against the FP64
oracle, with the other hand tests' bounds."""
import numpy as np
import pytest

import oracle
import scenes
from scenes import articulated as art
from tests.gpu_util import TOL_U, log, max_err
from tests.test_gpu_backward import _close
from tests.test_gpu_hand import OMEGA, DevHand, _check_contact, _item_mask

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("objects", [1, 3, 8])
def test_many_candidates(oracle_lib, objects):
    h, mesh, scene2, links, model = art.config_hand(n_envs=6, seed=5, mode=scenes.MODE_DECAY_ONLY)
    E = scene2.n_envs
    scene = scenes._empty_scene(E, objects)
    rng = np.random.default_rng(objects)
    for e in range(E):
        scene.n_obj[e] = objects
        for o in range(objects):
            # a box as wide as the hand whose face is a little above the palm's plane
            scene.type[e, o] = scenes.BOX
            scene.shape[e, o] = (300.0, 300.0, 20.0, 0.0)
            R, t = links.rot[e, 0].reshape(3, 3), links.trans[e, 0]
            scene.rot[e, o] = np.asarray(R, np.float64).ravel()
            scene.trans[e, o] = t + R @ np.array([0.0, 0.0, rng.uniform(25.0, 33.0)])
    d = DevHand(h, mesh, scene, links, model, backward=True)
    got = d.step()
    ref = oracle.hand_forward(mesh, h, scene, links, model, omega_a=OMEGA, with_margin=True)
    _, n_obj = _check_contact(got, ref, objects)
    assert n_obj > 0
    err = max_err(got["u"], ref["u"])
    live = int((ref["n_active"] > 0).sum(axis=1).max())
    log(f"[gpu] {objects} objects on every patch, up to {live} patches in contact: max|dU| {err:.3e}")
    assert err <= TOL_U * max(1.0, float(np.abs(ref["u"]).max()))
    keep, node_keep = _item_mask(ref, mesh, scenes.MODE_DECAY_ONLY)
    assert (keep & (ref["n_active"] > 0)).any()
    w = (rng.standard_normal(ref["u"].shape) * node_keep[None]).astype(np.float32).astype(np.float64)
    g = d.backward(w)
    rg = oracle.hand_backward(mesh, h, scene, links, model, w)
    for name in ("grad_rot", "grad_trans", "grad_link_rot", "grad_link_trans", "grad_alpha"):
        _close(g[name], rg[name], name)
