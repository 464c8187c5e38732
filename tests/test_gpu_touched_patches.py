"""Calls that touch few of a surface's patches: what the tables of the others
hold is never read.  Each call follows one that filled every table under
another model, and the contact counts of several workgroups an env come out
right call after call."""
import numpy as np
import pytest

import scenes
from scenes import MODE_DECAY_ONLY, MODE_FULL
from tests.gpu_util import TOL_U, DevModel, DevScene, log, make_plan, to_dev, torch_dev
from tests.test_gpu_backward import _compare_all, clean_scene, gpu_step_backward
from tests.test_gpu_forward_shapes import _patches, _spheres

pytestmark = pytest.mark.gpu


def _step(plan, scene, model):
    from paper_2604_20295_amd import _native
    torch, dev = torch_dev()
    ds, dm = DevScene(scene), DevModel(model)
    u = torch.full((3, ds.E, plan.N), float("nan"), device=dev)
    cobj = torch.full((ds.E, plan.N), 99, dtype=torch.int8, device=dev)
    na = torch.full((ds.E, plan.K), -7, dtype=torch.int32, device=dev)
    _native.etac_step(plan, ds.struct(plan), dm.struct(plan), u, cobj, na)
    torch.cuda.synchronize()
    return u.cpu().numpy(), cobj.cpu().numpy(), na.cpu().numpy()


# one workgroup an env and several; items listed and not; every pooling launch
@pytest.mark.parametrize("patches,envs", [(6, 3), (40, 1), (40, 7), (40, 30), (300, 1), (300, 5)])
def test_few_of_many_patches(oracle_lib, patches, envs):
    sizes = tuple((130, 64, 257, 33)[k % 4] for k in range(patches))
    mesh = _patches(sizes)
    model = scenes.draw_model(np.random.default_rng(6), mesh.pitch, MODE_FULL)
    other = scenes.draw_model(np.random.default_rng(7), mesh.pitch, MODE_FULL)
    scene = _spheres(mesh, envs, 2, 3)
    plan = make_plan(mesh, max(envs, 8), 8, backward=True)
    # another model's tables of as many patches as eight objects reach
    wide = scenes._empty_scene(envs, 8)
    wide.n_obj[:] = 8
    for e in range(envs):
        for o in range(8):
            wide.shape[e, o, 0] = 6.0
            wide.trans[e, o] = mesh.origin[(8 * e + o) % patches] + np.array([0, 0, 5.0])
    for mode in (MODE_FULL, MODE_DECAY_ONLY):
        _step(plan, wide, other)
        u, cobj, na = _step(plan, scene, model.with_mode(mode))
        ref = oracle_lib.forward(mesh, scene, model.with_mode(mode))
        assert np.array_equal(cobj, ref["contact_obj"]) and np.array_equal(na, ref["n_active"])
        err = float(np.abs(u - ref["u"]).max())
        log(f"[gpu] {patches} patches, {envs} envs, mode {mode}: max|dU| {err:.2e}")
        assert err <= TOL_U
    clean, n = clean_scene(oracle_lib, mesh, scene, model)
    w = np.random.default_rng(1).standard_normal((3, envs, mesh.n_nodes))
    gpu_step_backward(plan, wide, other, w)
    _compare_all(gpu_step_backward(plan, clean, model, w), oracle_lib.backward(mesh, clean, model, w), MODE_FULL)


@pytest.mark.parametrize("envs", [1, 3, 200])
def test_counts_of_split_envs_repeat(oracle_lib, envs):
    # counts are left at zero by every call: contact alone, steps and adjoints in turn
    from paper_2604_20295_amd import _native
    torch, dev = torch_dev()
    mesh = _patches((900, 257, 64, 300, 33, 1000, 7))
    scene = _spheres(mesh, envs, 2, 5)
    model = scenes.draw_model(np.random.default_rng(6), mesh.pitch, MODE_FULL)
    plan = make_plan(mesh, 200, 2, backward=True)
    ref, _, n_ref = oracle_lib.contact(mesh, scene)[:3]
    ds = DevScene(scene)
    cobj = torch.empty((envs, plan.N), dtype=torch.int8, device=dev)
    uhat = torch.empty((3, envs, plan.N), device=dev)
    na = torch.empty((envs, plan.K), dtype=torch.int32, device=dev)
    w = to_dev(np.random.default_rng(1).standard_normal((3, envs, mesh.n_nodes)).astype(np.float32))
    rot, tr = torch.empty((envs, 2, 9), device=dev), torch.empty((envs, 2, 3), device=dev)
    for rep in range(4):
        na.fill_(-7)
        _native.etac_contact(plan, ds.struct(plan), cobj, uhat, na)
        assert np.array_equal(na.cpu().numpy(), n_ref) and np.array_equal(cobj.cpu().numpy(), ref)
        _native.etac_contact_backward(plan, ds.struct(plan), w, rot, tr)
        _, c, n = _step(plan, scene, model)
        assert np.array_equal(n, n_ref) and np.array_equal(c, ref)
    log(f"[gpu] {envs} envs: counts of four rounds")
