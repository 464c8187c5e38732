"""The taxel regressor's units of 256 nodes: patches of a unit, a node more or
less and several units, more units than waves, and scores that differ between
the units of an item, against the FP64 oracle within the other regressor
tests' bound."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import make_plan
from tests.test_gpu_regress import _check, _gpu_regress, _ragged_mesh, _reg, _synthetic_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,E", [((255, 256, 257), 3), ((512, 1, 513), 1), ((2049, 15), 2), ((300, 31, 257, 16), 900)])
@pytest.mark.parametrize("frac", [0.0, 0.5, 1.0])
def test_units(sizes, E, frac):
    mesh = _ragged_mesh(list(sizes), seed=6)
    # positions far apart between the ends of a patch: its units' largest scores differ
    for k in range(mesh.n_patches):
        sl = slice(int(mesh.patch_offset[k]), int(mesh.patch_offset[k + 1]))
        mesh.pos[0, sl] += np.linspace(0.0, 12.0, sl.stop - sl.start, dtype=np.float32)
    u, na = _synthetic_field(mesh, E, frac, seed=7)
    reg = _reg(8)
    y = _gpu_regress(make_plan(mesh, E, 1), reg, u, na)
    envs = np.unique(np.linspace(0, E - 1, 12).astype(int))
    ref = oracle.regress(mesh, reg.astype(np.float64), np.ascontiguousarray(u[:, envs]).astype(np.float64))
    _check(y[envs], ref, f"units, patches {sizes}, {E} envs, {frac:.0%} in contact")
