"""Rayleigh-Ritz at the block widths where the dense products change tiles:
strips of 16 columns (16, 17), narrow tiles (32, 33), one or two 64-column tiles
(64, 65), 128- and 160-column tiles (128, 130, 161, 257), on grids whose point
count is no multiple of a step's or a tile's rows.

Tolerances: those of the Rayleigh-Ritz parity tests (Ritz values 1e-10 and 2e-4
of the largest, dV X^T X = I within 1e-11 and 1e-5, FP64 and FP32)."""
import numpy as np
import pytest

import workloads as W
from oracle import chefsi

from gpu_helpers import log, require_gpu, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncol", [2, 16, 17, 32, 33, 64, 65, 128, 130, 161, 257])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_rayleigh_ritz_sizes(ncol, dtype):
    torch = require_gpu()
    from paper_2005_10431_amd import Context
    n = (17, 13, 15) if ncol % 2 else (14, 16, 19)
    L = tuple(0.35 * v for v in n)
    s = W.tiny_system(n=n, L=L, n_atoms=1, with_nonlocal=False, seed=2, n_states=ncol)
    v = np.random.default_rng(5).uniform(-1.0, 0.5, s.nd)
    X = W.initial_orbitals(s.nd, ncol, 4).astype(dtype)
    _, lam = chefsi.rayleigh_ritz(s, v, [], X.astype(np.float64))
    ctx = Context(s)
    ctx.set_veff(to_dev(torch, v))
    # padded columns: the pad stays as it is
    Xp = np.full((ncol, s.nd + 5), 7.0, dtype=dtype)
    Xp[:, :s.nd] = X
    Xd = to_dev(torch, Xp)
    eig = torch.zeros(ncol, dtype=torch.float64, device="cuda")
    ctx.rayleigh_ritz(Xd, eig)
    Xg = to_np(Xd).astype(np.float64)
    err = float(np.max(np.abs(to_np(eig) - lam)) / max(1.0, np.max(np.abs(lam))))
    O = s.dV * Xg[:, :s.nd] @ Xg[:, :s.nd].T
    ortho = float(np.max(np.abs(O - np.eye(ncol))))
    log(f"{ncol} {dtype}: eigenvalues {err:.2e} orthonormality {ortho:.2e}")
    assert err <= (1e-10 if dtype == "float64" else 2e-4)
    assert ortho <= (1e-11 if dtype == "float64" else 1e-5)
    assert np.all(Xg[:, s.nd:] == 7.0)
