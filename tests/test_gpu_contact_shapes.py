"""The contact passes at the edges of their chunks: surfaces of one node, a
node more or less than a chunk of 512, patches that end inside a 64-node word
and a chunk, and batches on either side of the change from several workgroups
per env to one, against the FP64 oracle.

Masks and counts are exact; u_hat to TOL_U, the bound of the other contact
tests (the arithmetic is FP64, rounded once)."""
import numpy as np
import pytest

import scenes
from scenes import trimeshes as tm
from tests.gpu_util import TOL_U, gpu_contact, log, make_plan, max_err
from tests.test_gpu_forward_shapes import _patches, _spheres
from tests.test_gpu_mesh import gpu_contact_mesh

pytestmark = pytest.mark.gpu


def _compare(label, got, ref):
    err = max_err(got[1].astype(np.float64), ref[1])
    log(f"[gpu] {label}: active {int((ref[0] >= 0).sum())} nodes, max|du_hat| {err:.2e}")
    assert np.array_equal(got[0], ref[0]) and np.array_equal(got[2], ref[2])
    assert err <= TOL_U
    assert not got[1][:, ref[0] < 0].any()


@pytest.mark.parametrize("sizes", [(1,), (3, 60), (511,), (512,), (513,), (500, 12, 1, 700), (64, 448, 512, 1025)])
@pytest.mark.parametrize("E", [1, 5])
def test_mesh_chunks(oracle_lib, sizes, E):
    from paper_2604_20295_amd import _native
    mesh = _patches(sizes)
    ms = tm.object_set(scale=0.2)
    rng = np.random.default_rng(len(sizes) + sizes[0])
    scene = _spheres(mesh, E, 3, sizes[0])
    for e in range(E):
        for o in range(3):
            if (e + o) % 3 == 1:
                continue
            m = int(rng.integers(0, 4))
            R = scenes.random_rotation(rng)
            c = mesh.origin[(e + o) % mesh.n_patches].astype(np.float64)
            scene.type[e, o] = tm.MESH
            scene.shape[e, o] = (float(m), 0, 0, 0)
            scene.rot[e, o] = R.ravel()
            h = ms.support_extent(m, R, np.array([0.0, 0.0, -1.0]))
            scene.trans[e, o] = c + np.array([rng.uniform(-1, 1), rng.uniform(-1, 1), h - rng.uniform(0.5, 2.0)])
    plan = make_plan(mesh, E, 3)
    got = gpu_contact_mesh(plan, _native.MeshSet.from_set(ms), scene)
    _compare(f"mesh contact, patches {sizes}, {E} envs", got, oracle_lib.contact_mesh(mesh, scene, ms))


@pytest.mark.parametrize("sizes", [(1,), (2, 1, 3), (63, 65, 127, 5), (700, 321, 64)])
@pytest.mark.parametrize("E", [1, 7, 300, 1100])
def test_primitive_chunks(oracle_lib, sizes, E):
    mesh = _patches(sizes)
    scene = _spheres(mesh, E, 3, E)
    plan = make_plan(mesh, E, 3)
    got = gpu_contact(plan, scene)
    ref = oracle_lib.forward(mesh, scene, scenes.draw_model(np.random.default_rng(5), mesh.pitch, scenes.MODE_DECAY_ONLY))
    _compare(f"contact, patches {sizes}, {E} envs", got, (ref["contact_obj"], ref["uhat"], ref["n_active"]))
