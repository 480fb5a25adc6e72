"""Nonlocal forces where the tiles of columns end: 16-column tiles, up to five of
them in a workgroup, on boxes that wrap around the cell's faces, in FP64 and
FP32.  Bar as in the other force parity tests: 1e-11 of the largest component
(the same terms in different orders)."""
import numpy as np
import pytest

from oracle import forces

from gpu_helpers import log, ragged_system, require_gpu, small_images_system
from test_gpu_forces import _gpu_forces, _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncol", [1, 16, 17, 80, 81])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_force_column_tiles(ncol, dtype):
    torch = require_gpu()
    s = ragged_system(n_states=81) if ncol % 2 else small_images_system(n_states=81)
    phi, blocks, w = _inputs(s, ncol, 21)
    blocks = [b.astype(dtype).astype(np.float64) for b in blocks]
    log(f"force column tiles: grid {s.n}, {s.n_atoms} atoms, {ncol} columns {dtype}")
    got = _gpu_forces(torch, s, phi, blocks, w, dtype=getattr(torch, dtype))
    ref = forces.forces(s, phi, blocks, w)
    assert np.max(np.abs(got - ref)) <= 1e-11 * np.max(np.abs(ref))
