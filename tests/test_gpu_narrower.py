"""A block after a wider one takes no further device memory: a program may capture
calls into a graph, or free what a graph holds, after a first call of the widest
block.  The free memory of the device is compared before and after each narrower
call (H X and the filter in both precisions, Bloch columns, forces) of contexts
whose narrow blocks take more partial sums per column; a growth of less than the
2 MiB that device memory is handed out in would not show, so the wide blocks are
chosen to take several of these."""
import numpy as np
import pytest

import workloads as W

from gpu_helpers import log, require_gpu, to_dev

pytestmark = pytest.mark.gpu


def _lattice(n, h, cells, n_states, seed):
    from dataclasses import replace
    rng = np.random.default_rng(seed)
    L = tuple(h * v for v in n)
    base = W.tiny_system(n=n, L=L, n_atoms=1, seed=seed, n_states=n_states)
    at = np.array([[i, j, k] for k in range(cells[2]) for j in range(cells[1]) for i in range(cells[0])])
    pos = np.mod((at + 0.5) * (np.array(L) / cells) + rng.normal(0.0, 0.1, at.shape), L)
    na = len(pos)
    return replace(base, pos=pos, Z=np.full(na, 4.0), rc_loc=np.full(na, 1.0), gamma=rng.uniform(-1.0, 1.0, (na, 2)),
                   n_electrons=float(n_states), rc_nl=1.2, rcut_nl=3.6)


@pytest.mark.parametrize("n, cells, n_states", [((72, 72, 72), (4, 4, 4), 130), ((48, 40, 96), (3, 2, 6), 260)])
def test_narrower_blocks_take_no_memory(n, cells, n_states):
    torch = require_gpu()
    from paper_2005_10431_amd import Context
    s = _lattice(n, 0.28, cells, n_states, 3)
    ctx = Context(s)
    ctx.set_veff(to_dev(torch, np.random.default_rng(1).uniform(-1.0, 0.5, s.nd)))
    lo, hi = ctx.spectrum_bounds()
    nk = n_states // 2
    X = torch.rand((n_states, 2 * s.nd), device="cuda", dtype=torch.float64) - 0.5
    Y, Wk = torch.empty_like(X), torch.empty_like(X)
    X32, Y32, W32 = X.float(), Y.float(), Wk.float()
    occ = torch.ones(n_states, device="cuda", dtype=torch.float64)
    phi = torch.zeros(s.nd, device="cuda", dtype=torch.float64)
    F = torch.empty((s.n_atoms, 3), device="cuda", dtype=torch.float64)

    def calls(nc):
        yield "H X", lambda: ctx.apply_H(X[:nc], Y[:nc])
        yield "H X fp32", lambda: ctx.apply_H(X32[:nc], Y32[:nc])
        yield "filter", lambda: ctx.chebyshev_filter(Y[:nc], Wk[:nc], 2, 0.5 * (lo + hi), hi, lo)
        yield "filter fp32", lambda: ctx.chebyshev_filter(Y32[:nc], W32[:nc], 2, 0.5 * (lo + hi), hi, lo)
        yield "forces", lambda: ctx.forces(phi, [X[:nc]], occ[:nc], F)
        ck = max(1, nc * nk // n_states)
        yield "H_k X", lambda: ctx.apply_H_k((0.1, 0.2, -0.3), X[:ck], Y[:ck])

    for name, f in calls(n_states):
        f()
    torch.cuda.synchronize()
    widths = sorted({1, 2, 4, 7, 8, 15, 16, 17, *range(32, n_states, 16)})
    for nc in widths:
        for name, f in calls(nc):
            before = torch.cuda.mem_get_info()[0]
            f()
            torch.cuda.synchronize()
            taken = before - torch.cuda.mem_get_info()[0]
            if taken:
                log(f"{n} {name} of {nc} columns after {n_states}: {taken} bytes")
            assert taken == 0, (name, nc)
