"""Blocks narrower than the context's: the nonlocal pass cuts z into other
ranges for them, and up to 16 columns are shared by the waves of a workgroup.
H X and the filter of 1 to all columns of contexts of 200 states against the
oracle, the allocation-free filter bitwise equal to the filter, and Bloch
columns (real and imaginary halves in tiles of 16) at a general k.  One system
needs a second layer of slots.

Tolerances as for the other parity tests: 1e-12 for H X and 1e-11 for the filter
in FP64, 2e-6 for H X in FP32."""
import re

import numpy as np
import pytest

import workloads as W
from oracle import atoms, chefsi, hamiltonian, kpoints

from gpu_helpers import log, rel_err, require_gpu, to_dev, to_np
from test_gpu_nonlocal import SYSTEMS

pytestmark = pytest.mark.gpu


def _system(name):
    if name == "deep":   # several cuts of z, a tail block
        return W.tiny_system(n=(21, 17, 62), L=(5.9, 4.8, 17.4), n_atoms=6, seed=11, n_states=200)
    return SYSTEMS[name](200)


@pytest.mark.parametrize("system", ["deep", "odd_plane", "layers", "dense"])
def test_narrow_blocks_match_oracle(system):
    torch = require_gpu()
    from paper_2005_10431_amd import Context
    s = _system(system)
    v = np.random.default_rng(3).uniform(-1.0, 0.5, s.nd)
    projs = atoms.projectors(s)
    ctx = Context(s)
    ctx.set_veff(to_dev(torch, v))
    X = W.initial_orbitals(s.nd, 200, 2)
    lo, hi = hamiltonian.spectrum_bounds(s, v, projs)
    a, b, a0 = lo + 0.3 * (hi - lo), hi, lo
    href = hamiltonian.apply_H(s, v, projs, X[:40])
    fref = chefsi.chebyshev_filter(s, v, projs, X[:17], 4, a, b, a0)
    for nc in (1, 7, 16, 17, 40, 200):
        Xd = to_dev(torch, X[:nc])
        Yd = torch.full_like(Xd, 7.0)
        ctx.apply_H(Xd, Yd)
        m = min(nc, 40)
        err = rel_err(to_np(Yd)[:m], href[:m])
        X32 = Xd.float()
        Y32 = torch.full_like(X32, 7.0)
        ctx.apply_H(X32, Y32)
        ref32 = hamiltonian.apply_H(s, v, projs, to_np(X32)[:m].astype(np.float64))
        err32 = rel_err(to_np(Y32)[:m].astype(np.float64), ref32)
        X2, Wd = Xd.clone(), torch.empty_like(Xd)
        ctx.chebyshev_filter(Xd, Wd, 4, a, b, a0)
        ctx.chebyshev_filter_noalloc(X2, Wd, 4, a, b, a0)
        m = min(nc, 17)
        errf = rel_err(to_np(Xd)[:m], fref[:m])
        log(f"{system} {nc} of 200 columns: H X {err:.2e} fp32 {err32:.2e} filter {errf:.2e}")
        assert err <= 1e-12 and err32 <= 2e-6 and errf <= 1e-11
        assert torch.equal(Xd, X2)


@pytest.mark.parametrize("system", ["odd_plane", "layers"])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_narrow_bloch_blocks_match_oracle(system, dtype):
    torch = require_gpu()
    from paper_2005_10431_amd import Context
    s = _system(system)
    k = (0.31, -0.17, 0.23)
    v = np.random.default_rng(3).uniform(-1.0, 0.5, s.nd)
    projs = kpoints.projectors_k(s, k)
    ctx = Context(s)
    ctx.set_veff(to_dev(torch, v))
    Z = W.initial_orbitals_k(s.nd, 40, 4)
    X = np.concatenate([Z.real, Z.imag], axis=1).astype(dtype)
    Z = X[:, :s.nd].astype(np.float64) + 1j * X[:, s.nd:].astype(np.float64)
    ref = kpoints.apply_H_k(s, v, projs, Z, k)
    for nc in (1, 8, 9, 40):
        Xd = to_dev(torch, X[:nc])
        Yd = torch.full_like(Xd, 7.0)
        ctx.apply_H_k(k, Xd, Yd)
        Y = to_np(Yd).astype(np.float64)
        err = rel_err(Y[:, :s.nd] + 1j * Y[:, s.nd:], ref[:nc])
        log(f"{system} {dtype} {nc} Bloch columns: {err:.2e}")
        assert err <= (1e-12 if dtype == "float64" else 2e-6)


def test_dense_systems_reach_all_slots_and_a_second_layer(capfd, monkeypatch):
    """The systems of these tests are as dense as they are meant to be."""
    require_gpu()
    from paper_2005_10431_amd import Context
    monkeypatch.setenv("SPARC_GPU_DEBUG", "1")
    seen = {}
    for name in ("dense", "layers", "odd_plane"):
        for ns in (8, 200):
            capfd.readouterr()
            Context(SYSTEMS[name](ns)).close()
            lines = [l.split() for l in capfd.readouterr().err.splitlines() if "nonlocal pass:" in l]
            assert lines
            seen[name, ns] = [(int(l[l.index("slots") - 1]), int(l[l.index("layers,") - 1])) for l in lines]
    log(seen)
    for ns in (8, 200):
        assert all(s == 24 for s, _ in seen["dense", ns])
        assert any(n > 1 for _, n in seen["layers", ns])
        assert all(s <= 16 and n == 1 for s, n in seen["odd_plane", ns])


@pytest.mark.parametrize("system", ["deep", "whole_blocks", "wide", "sparse", "layers"])
@pytest.mark.parametrize("ncol", [48, 64])
def test_h_written_by_the_pass(system, ncol):
    """Blocks that fill the pass's workgroups: the projector term is written
    before the local part is added, where the units hold every point (not in
    the sparse system and not with a second layer).  What Y held before must
    not matter, padding stays, and a NaN reaches what it reaches in a narrow
    block."""
    torch = require_gpu()
    from paper_2005_10431_amd import Context
    s = _system(system)
    v = np.random.default_rng(3).uniform(-1.0, 0.5, s.nd)
    projs = atoms.projectors(s)
    ctx = Context(s)
    ctx.set_veff(to_dev(torch, v))
    for dtype, bar in (("float64", 1e-12), ("float32", 2e-6)):
        X = np.full((ncol, s.nd + 3), 5.0, dtype=dtype)
        X[:, :s.nd] = W.initial_orbitals(s.nd, ncol, 2)
        Xd = to_dev(torch, X)
        Y = torch.full_like(Xd, float("nan"))
        ctx.apply_H(Xd, Y)
        got = to_np(Y)
        err = rel_err(got[:, :s.nd].astype(np.float64),
                      hamiltonian.apply_H(s, v, projs, X[:, :s.nd].astype(np.float64)))
        log(f"{system} {ncol} {dtype}: {err:.2e}")
        assert err <= bar and np.all(np.isnan(got[:, s.nd:]))
        Xd[3, s.nd // 2] = float("nan")
        Y1 = torch.zeros_like(Xd[:5])
        ctx.apply_H(Xd, Y)
        ctx.apply_H(Xd[:5], Y1)
        assert torch.equal(torch.isnan(Y[:5, :s.nd]), torch.isnan(Y1[:, :s.nd]))
        assert int(torch.isnan(Y[:, :s.nd]).any(dim=1).sum()) == 1


@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_bloch_h_written_by_the_pass(dtype):
    """The same for Bloch columns (FP64 at 32 columns; FP32 takes this way only in
    blocks of more than 128 MB: 62 x 62 x 62 x 96)."""
    torch = require_gpu()
    from paper_2005_10431_amd import Context
    if dtype == "float64":
        s, nc = _system("deep"), 32
    else:
        s, nc = W.tiny_system(n=(62, 62, 62), L=(18.6, 18.6, 18.6), n_atoms=60, seed=3, n_states=72), 96
    k = (0.31, -0.17, 0.23)
    v = np.random.default_rng(3).uniform(-1.0, 0.5, s.nd)
    ctx = Context(s)
    ctx.set_veff(to_dev(torch, v))
    g = torch.Generator(device="cuda").manual_seed(3)
    Xd = (torch.rand((nc, 2 * s.nd), generator=g, device="cuda") - 0.5).to(getattr(torch, dtype))
    Y = torch.full_like(Xd, float("nan"))
    ctx.apply_H_k(k, Xd, Y)
    X = to_np(Xd[:2]).astype(np.float64)
    ref = kpoints.apply_H_k(s, v, kpoints.projectors_k(s, k), X[:, :s.nd] + 1j * X[:, s.nd:], k)
    got = to_np(Y[:2]).astype(np.float64)
    err = rel_err(got[:, :s.nd] + 1j * got[:, s.nd:], ref)
    log(f"Bloch {dtype} {nc}: {err:.2e}")
    assert err <= (1e-12 if dtype == "float64" else 2e-6)
    assert bool(torch.isfinite(Y).all())


@pytest.mark.parametrize("system, slots, layers", [("dense", 24, 1), ("layers", 24, 2)])
def test_dense_systems_reach_the_slots_and_layers_they_stand_for(system, slots, layers, capfd, monkeypatch):
    """The widest slot count, and a further layer, in the pass that the tests of
    these systems run (the diagnostics line of context creation)."""
    require_gpu()
    from paper_2005_10431_amd import Context
    monkeypatch.setenv("SPARC_GPU_DEBUG", "1")
    for n_states in (8, 70, 200):
        capfd.readouterr()
        ctx = Context(SYSTEMS[system](n_states))
        found = re.findall(r"nonlocal pass: .* (\d+) slots \(\d+ used\), (\d+) layers", capfd.readouterr().err)
        del ctx
        assert found
        for s, n in found:
            assert int(s) == slots and int(n) >= layers
