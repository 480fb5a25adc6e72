"""The local sweep against the oracle where its vectors, slabs and z ranges can
go wrong: rows of 1, 2 and 4 points a thread, the shortest axes, slabs of fewer
than 12 rows (rows of more than 128 points, which need two or three halo vectors
per thread) and, with Bloch columns, of fewer than 4 (wide odd rows), blocks so narrow that z is
cut into ranges and blocks wide enough for whole rounds with a cut remainder.

Tolerances: 1e-12 (H X) and 1e-11 (filter) relative in FP64 as in the other
parity tests; 2e-6 and 1e-5 in FP32 (float rounding 6e-8 per operation over 37
terms, amplified by the filter's degree)."""
import numpy as np
import pytest

import workloads as W
from oracle import chefsi, hamiltonian

from gpu_helpers import log, rel_err, require_gpu, to_dev, to_np

pytestmark = pytest.mark.gpu

GRIDS = [(13, 13, 13), (14, 15, 16), (15, 13, 24), (16, 29, 13), (17, 40, 19), (24, 24, 24), (130, 14, 13),
         (131, 13, 14), (256, 17, 13), (250, 13, 15)]


@pytest.mark.parametrize("n", GRIDS)
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_sweep_matches_oracle(n, dtype):
    torch = require_gpu()
    from paper_2005_10431_amd import Context
    L = tuple(0.3 * v * (1 + 0.02 * d) for d, v in enumerate(n))
    # more than one round of workgroups on the small grids, fewer than one on the wide ones
    ncol = 3 if n[0] > 100 else 70
    s = W.tiny_system(n=n, L=L, n_atoms=1, with_nonlocal=False, seed=2, n_states=ncol)
    v = np.random.default_rng(5).uniform(-1.0, 0.5, s.nd)
    X = W.initial_orbitals(s.nd, ncol, 4).astype(dtype)
    ctx = Context(s)
    ctx.set_veff(to_dev(torch, v))
    ref = hamiltonian.apply_H(s, v, [], X.astype(np.float64))
    tol_h, tol_f = (1e-12, 1e-11) if dtype == "float64" else (2e-6, 1e-5)
    lo, hi = hamiltonian.spectrum_bounds(s, v, [])
    a, b, a0 = lo + 0.3 * (hi - lo), hi, lo
    for nc in (ncol, 1):
        Xd = to_dev(torch, X[:nc])
        Yd = torch.full_like(Xd, 7.0)
        ctx.apply_H(Xd, Yd)
        err = rel_err(to_np(Yd).astype(np.float64), ref[:nc])
        Wd = torch.empty_like(Xd)
        ctx.chebyshev_filter(Xd, Wd, 4, a, b, a0)
        reff = chefsi.chebyshev_filter(s, v, [], X[:nc].astype(np.float64), 4, a, b, a0)
        errf = rel_err(to_np(Xd).astype(np.float64), reff)
        log(f"{n} {dtype} {nc} columns: H X {err:.2e} filter {errf:.2e}")
        assert err <= tol_h and errf <= tol_f


def test_sweep_rounds_do_not_change_results(monkeypatch):
    """Every point's sum is the same whatever the slab height and the z ranges."""
    torch = require_gpu()
    from paper_2005_10431_amd import Context
    s = W.tiny_system(n=(40, 37, 29), L=(12.0, 11.1, 8.7), n_atoms=1, with_nonlocal=False, seed=5, n_states=300)
    v = np.random.default_rng(6).uniform(-1.0, 0.5, s.nd)
    g = torch.Generator(device="cuda").manual_seed(3)
    X = torch.rand((300, s.nd), generator=g, device="cuda", dtype=torch.float64) - 0.5
    ctx = Context(s)
    ctx.set_veff(to_dev(torch, v))
    outs = []
    for ty, nc in (("", 300), ("5", 300), ("13", 300), ("24", 300), ("", 7)):
        monkeypatch.setenv("SPARC_GPU_SWEEP_TY", ty)
        Xd = X[:nc].clone()
        Wd = torch.empty_like(Xd)
        ctx.chebyshev_filter(Xd, Wd, 5, 20.0, 120.0, -2.0)
        outs.append(to_np(Xd[:7]))
    for o in outs[1:]:
        assert np.array_equal(o, outs[0])


@pytest.mark.parametrize("n", [(13, 13, 13), (17, 15, 24), (24, 24, 24), (130, 14, 13), (253, 13, 14), (255, 14, 13), (149, 13, 13)])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_bloch_sweep_matches_oracle(n, dtype):
    """The Bloch form of the sweep (wrapped values times exp(+-i k L)) and of the
    nonlocal pass at a general k, contiguous and padded columns."""
    torch = require_gpu()
    from oracle import kpoints
    from paper_2005_10431_amd import Context
    L = tuple(0.3 * v * (1 + 0.02 * d) for d, v in enumerate(n))
    ncol = 2 if n[0] > 100 else 9
    s = W.tiny_system(n=n, L=L, n_atoms=2, seed=2, n_states=ncol)
    s.rcut_nl, s.rc_nl = 1.4, 0.6
    k = (0.31, -0.17, 0.23)
    v = np.random.default_rng(5).uniform(-1.0, 0.5, s.nd)
    Z = W.initial_orbitals_k(s.nd, ncol, 4)
    projs = kpoints.projectors_k(s, k)
    ctx = Context(s)
    ctx.set_veff(to_dev(torch, v))
    for pad in (0, 3):
        X = np.zeros((ncol, 2 * s.nd + pad), dtype=dtype)
        X[:, :s.nd], X[:, s.nd:2 * s.nd] = Z.real, Z.imag
        Zx = X[:, :s.nd].astype(np.float64) + 1j * X[:, s.nd:2 * s.nd].astype(np.float64)
        ref = kpoints.apply_H_k(s, v, projs, Zx, k)
        Xd = to_dev(torch, X)
        Yd = torch.full_like(Xd, 7.0)
        ctx.apply_H_k(k, Xd, Yd)
        Y = to_np(Yd).astype(np.float64)
        err = rel_err(Y[:, :s.nd] + 1j * Y[:, s.nd:2 * s.nd], ref)
        log(f"{n} {dtype} pad {pad}: H_k X {err:.2e}")
        assert err <= (1e-12 if dtype == "float64" else 2e-6)
        assert np.all(Y[:, 2 * s.nd:] == 7.0)
