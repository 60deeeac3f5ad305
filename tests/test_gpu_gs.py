"""FGMRES's two-pass Gram-Schmidt against the oracle's modified Gram-Schmidt: fixed numbers of
cycles with a weak smoother, so that the residual stays far above rounding and every basis
vector counts, at restart lengths below, at and above the vectors of one pass (10) and at
vector lengths on both sides of the block-size rule (256 * 1024 entries).

Tolerance: 1e-10 relative, that of every fixed-count comparison with the oracle
(test_gpu_parity): the iterate is the minimal-residual one of the same Krylov space."""
import numpy as np
import pytest

import workloads as W
from oracle import hierarchy as Hh, multigrid as MG

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _fixed(wl, m, cycles, **weak):
    from paper_2405_05047_amd import gen, mg
    o = Hh.build(wl)
    p = gen.build(wl)
    b = W.rand_vec(4100 + m, o.finest.ndof)
    b[np.asarray(o.finest.mask).ravel() != 0] = 0.0
    h = mg.Hierarchy(p.levels, mg.config_from(wl, gmres_m=m, **weak))
    x = torch.zeros(len(b), dtype=torch.float64, device="cuda")
    st = h.solve(torch.from_numpy(b).cuda(), x, fixed=cycles)
    mgo = MG.Multigrid(o, **weak)
    xr, st_ref = mgo.fgmres(b, m=m, fixed_iters=cycles)
    assert st["iters"] == cycles
    res = np.linalg.norm(b - o.finest.A @ xr)
    assert res > 1e-6 * np.linalg.norm(b), "the comparison wants an unconverged iterate"
    x = x.cpu().numpy()
    assert np.linalg.norm(x - xr) <= 1e-10 * np.linalg.norm(xr)


@pytest.mark.parametrize("m,cycles", [(1, 3), (9, 9), (10, 21), (11, 11), (20, 20), (21, 23), (64, 64)])
def test_restart_lengths(m, cycles):
    _fixed(W.c2_td(band_rounds=2, uniform_rounds=1), m, cycles, omega=0.02, nu1=1, nu2=0)


@pytest.mark.parametrize("n", [8, 9])
def test_vector_lengths(n):
    _fixed(W.td_time(n, coarse_level=4), 10, 10, omega=0.05, nu1=1, nu2=0)
