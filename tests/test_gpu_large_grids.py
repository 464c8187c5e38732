"""Batches whose launches would not fit one grid (2^32 threads)."""
import numpy as np
import pytest

from scenes import trimeshes as tm
from tests.gpu_util import log, torch_dev

pytestmark = pytest.mark.gpu


def test_mesh_contact_of_two_to_the_thirty_nodes():
    # 2^23 envs of 128 nodes; objects in a few of them, the last one included
    from paper_2604_20295_amd import _native
    torch, dev = torch_dev()
    E, n = 1 << 23, 128
    x, y = (a.ravel() for a in np.meshgrid(np.arange(16.0), np.arange(8.0)))
    pos = np.stack([x, y, 0 * x]).astype(np.float32)
    nrm = np.stack([0 * x, 0 * x, 0 * x + 1]).astype(np.float32)
    args = (np.array([0, n], np.int32), pos, nrm, np.zeros((1, 3), np.float32))
    ms = _native.MeshSet.from_set(tm.object_set(scale=0.2))
    at = [0, 5, E // 2 - 1, E // 2, E - 1]

    def scene(plan, envs):
        m = len(envs)
        n_obj = torch.zeros(E if m > 5 else m, dtype=torch.int32, device=dev)
        k = n_obj.shape[0]
        ty = torch.full((k, 1), 3, dtype=torch.int32, device=dev)
        sh = torch.zeros((k, 1, 4), device=dev)
        rot = torch.eye(3, device=dev).reshape(1, 1, 9).repeat(k, 1, 1)
        tr = torch.zeros((k, 1, 3), device=dev)
        for i, e in enumerate(at):
            j = e if m > 5 else i
            n_obj[j] = 1
            sh[j, 0, 0] = i % 4
            tr[j, 0] = torch.tensor([3.0 + 2 * i, 3.0, 2.0])
        return plan.scene_struct(n_obj, ty, sh, rot, tr)

    log(f"[gpu] mesh contact, {E} envs of {n} nodes")
    few = _native.Plan(*args, 5, 1)
    cobj = torch.full((5, n), 9, dtype=torch.int8, device=dev)
    na = torch.full((5, 1), -7, dtype=torch.int32, device=dev)
    _native.etac_contact_mesh(few, ms, scene(few, at), cobj, None, na)
    plan = _native.Plan(*args, E, 1)
    big = torch.full((E, n), 9, dtype=torch.int8, device=dev)
    nb = torch.full((E, 1), -7, dtype=torch.int32, device=dev)
    _native.etac_contact_mesh(plan, ms, scene(plan, range(E)), big, None, nb)
    torch.cuda.synchronize()
    assert (na > 0).all()
    assert torch.equal(big[at], cobj) and torch.equal(nb[at], na)
    assert int((big >= 0).sum()) == int(na.sum()) == int(nb.sum())
    assert int((big == 9).sum()) == 0
