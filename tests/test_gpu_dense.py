"""The small levels' V-cycle as one dense product against the same cycle step by step
(MGQ1_NO_DENSE=1) and against the oracle: levels up to and just above the 2,048-row limit,
matrices of one and several passes of 512 columns, sweep counts with either order of the
work buffers, the smoothing coarse variant, 1 to 4 components, the finest level inside and
outside the product.

Tolerance: 1e-12 normwise, that of every V-cycle against the oracle (test_gpu_parity)."""
import numpy as np
import pytest

import workloads as W
from oracle import hierarchy as Hh, multigrid as MG

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# unknowns per level: 9 .. 1,089; 81 .. 1,761; 81 .. 5,573 (1,509 inside); 25 .. 2,025 (all but the
# limit's 23 rows); 25 .. 2,209 (the finest above the limit); 81 and 729; 108 and 500
CASES = {
    "poisson33": W.c1_poisson(4), "td": W.c2_td(band_rounds=2, uniform_rounds=1),
    "td_band": W.c2_td(band_rounds=3, uniform_rounds=1),
    "limit": W.c1_poisson(2).with_(coarse=(11, 11), h0=1.0 / 11), "above": W.c1_poisson(1).with_(coarse=(23, 23), h0=1.0 / 23),
    "elast": W.c3_elasticity(2), "oseen": W.c4_oseen(1),
}


@pytest.mark.parametrize("nu", [(2, 2), (1, 2), (0, 1), (3, 0)])
@pytest.mark.parametrize("name", list(CASES))
def test_dense_cycle(name, nu, monkeypatch):
    _check(CASES[name], monkeypatch, nu1=nu[0], nu2=nu[1])


def test_dense_cycle_smoothing_coarse_variant(monkeypatch):
    _check(CASES["td"].with_(coarse_mode=W.COARSE_SMOOTH, coarse_sweeps=5), monkeypatch, nu1=2, nu2=2)


def _check(wl, monkeypatch, **nu):
    from paper_2405_05047_amd import gen, mg
    o = Hh.build(wl)
    p = gen.build(wl)
    rng = np.random.default_rng(17)
    free = np.asarray(o.finest.mask).ravel() == 0
    b, x0 = rng.standard_normal(len(free)) * free, rng.standard_normal(len(free)) * free
    mgo = MG.Multigrid(o, **nu)
    ref, ref_x = mgo.vcycle(b), mgo.gmg(o.L, x0.copy(), b)
    for off in ("1", "0"):
        monkeypatch.setenv("MGQ1_NO_DENSE", off)
        h = mg.Hierarchy(p.levels, mg.config_from(wl, **nu))
        x = torch.full((len(b),), np.nan, dtype=torch.float64, device="cuda")
        h.vcycle(torch.from_numpy(b).cuda(), x)
        assert np.abs(x.cpu().numpy() - ref).max() <= 1e-12 * np.abs(ref).max(), off
        x = torch.from_numpy(x0).cuda()
        h.vcycle(torch.from_numpy(b).cuda(), x, x_is_zero=False)
        assert np.abs(x.cpu().numpy() - ref_x).max() <= 1e-12 * np.abs(ref_x).max(), off
