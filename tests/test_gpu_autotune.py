"""etac_plan_autotune: the launch knobs change no launch, so the call keeps the
shape it finds, makes one step (and its adjoint) and reports argument errors."""
import numpy as np
import pytest

import scenes
from tests.gpu_util import DevModel, DevScene, log, make_plan, to_dev, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("backward", [False, True])
def test_autotune_keeps_the_shape_and_fills_the_outputs(backward):
    from paper_2604_20295_amd import _native
    torch, dev = torch_dev()
    mesh, scene, model = scenes.config2(n_envs=16)
    E, O, N, K = 16, 3, mesh.n_nodes, mesh.n_patches
    plan = make_plan(mesh, E, O, backward=backward)
    ds, dm = DevScene(scene), DevModel(model)
    sc, md = ds.struct(plan), dm.struct(plan)
    gu = to_dev(np.random.default_rng(4).standard_normal((3, E, N)).astype(np.float32))

    def outs():
        return dict(u=torch.full((3, E, N), 7.0, device=dev),
                    cobj=torch.full((E, N), 7, dtype=torch.int8, device=dev),
                    na=torch.full((E, K), -7, dtype=torch.int32, device=dev),
                    grot=torch.full((E, O, 9), 7.0, device=dev), gt=torch.full((E, O, 3), 7.0, device=dev),
                    ga=torch.full((K,), 7.0, device=dev), gp=torch.full((17411,), 7.0, device=dev))

    ref, got = outs(), outs()
    _native.etac_step(plan, sc, md, ref["u"], ref["cobj"], ref["na"])
    if backward:
        _native.etac_step_backward(plan, sc, md, gu, ref["grot"], ref["gt"], ref["ga"], ref["gp"])
    torch.cuda.synchronize()
    shape = (3, 32, 32, 5, 8)          # none of the built-in values
    plan.set_launch(*shape)
    log(f"[gpu] autotune keeps {shape}, adjoint {backward}")
    grads = (gu, got["grot"], got["gt"], got["ga"], got["gp"]) if backward else ()
    assert _native.etac_plan_autotune(plan, sc, md, got["u"], got["cobj"], got["na"], *grads, reps=3) == shape
    assert plan.launch() == shape
    for k in ref:
        assert torch.equal(got[k], ref[k]), k
    for reps in (0, 1001):
        with pytest.raises(_native.EtacError):
            _native.etac_plan_autotune(plan, sc, md, got["u"], got["cobj"], got["na"], *grads, reps=reps)
    if not backward:
        with pytest.raises(_native.EtacError):           # the plan holds no adjoint workspace
            _native.etac_plan_autotune(plan, sc, md, got["u"], got["cobj"], got["na"], gu, got["grot"], got["gt"],
                                       got["ga"], got["gp"])
    assert plan.launch() == shape
