"""Infinities and NaN in a block: H X and the filter pass them on to the points
that the stencil and the projectors connect and to no others, although the
nonlocal pass multiplies whole 16-point blocks with whole groups of pairs.

A value that is not finite is put next to a support, in a block that holds
points of it, and inside one.  The points at which the result is not finite
must be those of the oracle, and the finite values must agree to the bars of
the other parity tests of H X (1e-12 in FP64, 2e-6 in FP32)."""
from dataclasses import replace

import numpy as np
import pytest

import workloads as W
from oracle import atoms, hamiltonian, kpoints

from gpu_helpers import log, require_gpu, to_dev, to_np
from test_gpu_nonlocal import SYSTEMS

pytestmark = pytest.mark.gpu


def _system(name):
    return replace(SYSTEMS[name](8), rc_nl=0.6, rcut_nl=1.4)


def _places(s):
    """A point outside every support whose 16-point block meets one, and a point inside one."""
    covered = np.zeros(s.nd, bool)
    for P in atoms.projectors(s):
        covered[P.idx] = True
    plane = s.n[0] * s.n[1]
    block = np.arange(s.nd) // plane * plane + np.arange(s.nd) % plane // 16 * 16
    met = np.zeros(s.nd, bool)
    met[block[covered]] = True
    near = np.flatnonzero(~covered & met[block])
    return int(near[len(near) // 2]), int(np.flatnonzero(covered)[covered.sum() // 2])


def _compare(Y, ref, bar, what):
    got, want = np.isfinite(Y), np.isfinite(ref)
    log(f"  {what}: {np.sum(~want)} points not finite, {np.sum(got != want)} differ")
    assert np.array_equal(got, want)
    err = np.max(np.abs(Y[want] - ref[want])) / np.max(np.abs(ref[want]))
    assert err <= bar, err


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("system", ["sparse", "wide"])
def test_values_that_are_not_finite_stay_in_their_supports(system, dtype, value):
    torch = require_gpu()
    from paper_2005_10431_amd import Context
    s = _system(system)
    v = np.random.default_rng(3).uniform(-1.0, 0.5, s.nd)
    projs = atoms.projectors(s)
    ctx = Context(s)
    ctx.set_veff(to_dev(torch, v))
    bar = 1e-12 if dtype == "float64" else 2e-6
    near, inside = _places(s)
    for place, what in ((near, "next to a support"), (inside, "inside one")):
        X = W.initial_orbitals(s.nd, 5, 2).astype(dtype)
        X[1, place] = value
        with np.errstate(invalid="ignore"):
            ref = hamiltonian.apply_H(s, v, projs, X.astype(np.float64))
        Xd = to_dev(torch, X)
        Yd = torch.full_like(Xd, 7.0)
        ctx.apply_H(Xd, Yd)
        _compare(to_np(Yd).astype(np.float64), ref, bar, f"{system} {dtype} {value} {what}")
        # two steps of the recurrence: the second one's projections are formed
        # from values that the pass itself has completed
        a, b, a0 = 20.0, 120.0, -2.0
        e, c = 0.5 * (b - a), 0.5 * (b + a)
        s1 = e / (a0 - c)
        s2 = 1.0 / (2.0 / s1 - s1)
        with np.errstate(invalid="ignore"):
            Y1 = s1 / e * (ref - c * X)
            Y2 = 2 * s2 / e * (hamiltonian.apply_H(s, v, projs, Y1) - c * Y1) - s1 * s2 * X
        Wd = torch.empty_like(Xd)
        X2, W2 = Xd.clone(), torch.empty_like(Xd)
        ctx.chebyshev_filter(Xd, Wd, 2, a, b, a0)
        ctx.chebyshev_filter_noalloc(X2, W2, 2, a, b, a0)
        assert torch.equal(torch.nan_to_num(Xd), torch.nan_to_num(X2))
        _compare(to_np(Xd).astype(np.float64), Y2, 10 * bar, f"{system} {dtype} {value} {what}, filter")


@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_bloch_values_that_are_not_finite_stay_in_their_supports(dtype):
    torch = require_gpu()
    from paper_2005_10431_amd import Context
    s = _system("wide")
    k = (0.31, -0.17, 0.23)
    v = np.random.default_rng(3).uniform(-1.0, 0.5, s.nd)
    projs = kpoints.projectors_k(s, k)
    ctx = Context(s)
    ctx.set_veff(to_dev(torch, v))
    for place in _places(s):
        Z = W.initial_orbitals_k(s.nd, 3, 4).astype(np.complex128 if dtype == "float64" else np.complex64)
        Z[1, place] = np.nan + 1j * np.nan
        with np.errstate(invalid="ignore"):
            ref = kpoints.apply_H_k(s, v, projs, Z.astype(np.complex128), k)
        Xd = to_dev(torch, np.concatenate([Z.real, Z.imag], axis=1).astype(dtype))
        Yd = torch.full_like(Xd, 7.0)
        ctx.apply_H_k(k, Xd, Yd)
        Y = to_np(Yd).astype(np.float64)
        _compare(Y[:, :s.nd] + 1j * Y[:, s.nd:], ref, 1e-12 if dtype == "float64" else 2e-6, f"Bloch {dtype}")
