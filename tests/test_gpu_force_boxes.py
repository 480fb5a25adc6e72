"""Nonlocal forces with cut-offs around the grid spacing: truncation spheres
that hold no point (boxes without a plane along an axis, whose walk has to
end), one point, or a few, next to each other in one call.  Bar as in the other
force parity tests: 1e-11 of the largest component."""
from dataclasses import replace

import numpy as np
import pytest

from oracle import forces

from gpu_helpers import log, ragged_system, require_gpu
from test_gpu_forces import _gpu_forces, _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rcut", [0.03, 0.12, 0.2, 0.4])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_force_boxes_below_the_spacing(rcut, dtype):
    torch = require_gpu()
    s = ragged_system(n_states=17)
    # on a grid point, between points along one axis, between points along all
    pos = np.array(s.pos)
    h = np.array(s.h)
    pos[0] = 5 * h
    pos[1] = (np.array([7, 8, 3]) + [0.0, 0.5, 0.0]) * h
    pos[2] = (np.array([20, 30, 6]) + 0.5) * h
    s = replace(s, pos=pos, rcut_nl=rcut)
    phi, blocks, w = _inputs(s, 17, 5)
    blocks = [b.astype(dtype).astype(np.float64) for b in blocks]
    log(f"force boxes: rcut {rcut}, spacing {s.h}, {dtype}")
    got = _gpu_forces(torch, s, phi, blocks, w, dtype=getattr(torch, dtype))
    ref = forces.forces(s, phi, blocks, w)
    assert np.max(np.abs(got - ref)) <= 1e-11 * np.max(np.abs(ref))


@pytest.mark.parametrize("ncol", [33, 49, 65, 97])
def test_force_tiles_and_parts(ncol):
    """Three, four and five 16-column tiles in a workgroup and two chunks of
    four, on spheres that few atoms leave to many workgroups."""
    torch = require_gpu()
    s = ragged_system(n_states=97)
    phi, blocks, w = _inputs(s, ncol, 6)
    log(f"force tiles: {ncol} columns")
    got = _gpu_forces(torch, s, phi, blocks, w)
    ref = forces.forces(s, phi, blocks, w)
    assert np.max(np.abs(got - ref)) <= 1e-11 * np.max(np.abs(ref))
