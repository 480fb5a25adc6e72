"""The nonlocal pass of the Gamma-point Hamiltonian (projections and their
application as matrix products over 16-point blocks of a plane) against the
oracle, where its tables can go wrong: planes that are no multiple of 16
points (a last block that starts early, odd leftovers), pencils with fewer
blocks than places, one plane range and several, blocks of columns around the
16-column tiles and the 64-column workgroups, supports that meet their own
images, and atoms so dense that the pairs of a pencil need more than 16 slots
or a second layer of slots.

Tolerances as for the other parity tests of H X and the filter: 1e-12 and
1e-11 relative in FP64 (rounding of about 1e-16 per operation over the 37
stencil terms and the support sums, the filter amplifying it by its degree),
2e-6 for H X in FP32 (float rounding 6e-8 times the same factor)."""
from dataclasses import replace

import numpy as np
import pytest

import workloads as W
from oracle import atoms, chefsi, hamiltonian

from gpu_helpers import log, rel_err, require_gpu, to_dev, to_np

pytestmark = pytest.mark.gpu


def _lattice(n, L, cells, rc, rcut, seed, n_states):
    """A jittered simple cubic lattice of cells[0] x cells[1] x cells[2] atoms."""
    rng = np.random.default_rng(seed)
    base = W.tiny_system(n=n, L=L, n_atoms=1, seed=seed, n_states=n_states)
    at = np.array([[i, j, k] for k in range(cells[2]) for j in range(cells[1]) for i in range(cells[0])])
    pos = np.mod((at + 0.5) * (np.array(L) / cells) + rng.normal(0.0, 0.03, at.shape), L)
    na = len(pos)
    return replace(base, pos=pos, Z=np.full(na, 2.0), rc_loc=np.full(na, 0.8),
                   gamma=rng.uniform(-1.0, 1.0, (na, 2)), n_electrons=float(n_states), rc_nl=rc, rcut_nl=rcut)


SYSTEMS = {
    # 221 points per plane: 13 complete blocks and 13 points; supports meet their images
    "odd_plane": lambda ns: W.tiny_system(n=(13, 17, 19), L=(4.1, 5.0, 5.6), n_atoms=2, seed=4, n_states=ns),
    # 272 = 17 x 16 points: every block whole, the last pencils short
    "whole_blocks": lambda ns: W.tiny_system(n=(16, 17, 14), L=(5.0, 5.2, 4.4), n_atoms=3, seed=6, n_states=ns),
    # 1020 points (tail of 12), several pencils along x
    "wide": lambda ns: W.tiny_system(n=(51, 20, 15), L=(14.3, 5.6, 4.2), n_atoms=5, seed=7, n_states=ns),
    # a single atom in a large cell: most blocks meet no pair
    "sparse": lambda ns: W.tiny_system(n=(40, 24, 33), L=(11.2, 6.7, 9.2), n_atoms=1, seed=8, n_states=ns),
    # more than 16 pairs at a time in a pencil, and more than 24
    "dense": lambda ns: _lattice((30, 16, 15), (12.0, 6.4, 6.0), (8, 4, 4), 0.6, 1.35, 9, ns),
    "layers": lambda ns: _lattice((40, 13, 14), (20.0, 6.5, 7.0), (14, 5, 5), 0.6, 1.2, 10, ns),
}


def _veff(s, seed):
    return np.random.default_rng(seed).uniform(-1.0, 0.5, s.nd)


@pytest.mark.parametrize("system", sorted(SYSTEMS))
@pytest.mark.parametrize("ncol", [1, 17, 70])
def test_nonlocal_pass_matches_oracle(system, ncol):
    torch = require_gpu()
    from paper_2005_10431_amd import Context
    s = SYSTEMS[system](max(ncol, 8))
    v = _veff(s, 3)
    projs = atoms.projectors(s)
    ctx = Context(s)
    ctx.set_veff(to_dev(torch, v))
    ld = s.nd + (5 if ncol == 17 else 0)     # an odd leading dimension too
    X = np.full((ncol, ld), np.nan)
    X[:, :s.nd] = W.initial_orbitals(s.nd, ncol, 2)
    ref = hamiltonian.apply_H(s, v, projs, X[:, :s.nd])
    Xd, Yd = to_dev(torch, X), to_dev(torch, np.full_like(X, 7.0))
    ctx.apply_H(Xd, Yd)
    Y = to_np(Yd)
    err = rel_err(Y[:, :s.nd], ref)
    log(f"{system} ncol {ncol}: H X fp64 {err:.2e}")
    assert err <= 1e-12
    assert np.all(Y[:, s.nd:] == 7.0)
    X32 = X.astype(np.float32)
    Yd = to_dev(torch, np.full_like(X32, 7.0))
    ctx.apply_H(to_dev(torch, X32), Yd)
    Y = to_np(Yd)
    err = rel_err(Y[:, :s.nd].astype(np.float64),
                  hamiltonian.apply_H(s, v, projs, X32[:, :s.nd].astype(np.float64)))
    log(f"{system} ncol {ncol}: H X fp32 {err:.2e}")
    assert err <= 2e-6
    assert np.all(Y[:, s.nd:] == 7.0)
    lo, hi = hamiltonian.spectrum_bounds(s, v, projs)
    a, b, a0 = lo + 0.3 * (hi - lo), hi, lo
    ref = chefsi.chebyshev_filter(s, v, projs, X[:, :s.nd], 5, a, b, a0)
    Wd = torch.empty_like(Xd)
    X2 = Xd.clone()
    W2 = torch.empty_like(X2)
    ctx.chebyshev_filter(Xd, Wd, 5, a, b, a0)
    ctx.chebyshev_filter_noalloc(X2, W2, 5, a, b, a0)
    err = rel_err(to_np(Xd)[:, :s.nd], ref)
    log(f"{system} ncol {ncol}: filter fp64 {err:.2e}")
    assert err <= 1e-11
    assert torch.equal(Xd[:, :s.nd], X2[:, :s.nd])
