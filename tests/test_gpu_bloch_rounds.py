"""The Bloch sweep's sums are the same whatever the slab height, the z ranges
and the block a column comes in: bitwise, as for the real sweep."""
import numpy as np
import pytest

import workloads as W

from gpu_helpers import require_gpu, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(40, 37, 29), (41, 30, 23)])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_bloch_sweep_rounds_do_not_change_results(n, dtype, monkeypatch):
    torch = require_gpu()
    from paper_2005_10431_amd import Context
    s = W.tiny_system(n=n, L=tuple(0.3 * v for v in n), n_atoms=1, with_nonlocal=False, seed=5, n_states=120)
    v = np.random.default_rng(6).uniform(-1.0, 0.5, s.nd)
    k = (0.31, -0.17, 0.23)
    g = torch.Generator(device="cuda").manual_seed(3)
    X = (torch.rand((120, 2 * s.nd), generator=g, device="cuda", dtype=torch.float64) - 0.5).to(getattr(torch, dtype))
    ctx = Context(s)
    ctx.set_veff(to_dev(torch, v))
    outs = []
    for ty, nc in (("", 120), ("3", 120), ("7", 120), ("9", 120), ("", 3)):
        monkeypatch.setenv("SPARC_GPU_SWEEP_TY", ty)
        Xd = X[:nc].clone()
        ctx.chebyshev_filter_k(k, Xd, torch.empty_like(Xd), 5, 20.0, 120.0, -2.0)
        outs.append(to_np(Xd[:3]))
    for o in outs[1:]:
        assert np.array_equal(o, outs[0])
