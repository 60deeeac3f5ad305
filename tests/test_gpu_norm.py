"""The norms that a solve reports, on both sides of the vectors that one workgroup takes (4,096
entries), against the host's sums in FP64 to the rounding of their order (64 ulp)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("coarse,rounds", [((1, 1), 0), ((4, 4), 0), ((32, 31), 1), ((32, 32), 1)],
                         ids=["4", "25", "4095", "4225"])
@pytest.mark.parametrize("outer", [W.OUTER_IR, W.OUTER_FGMRES])
def test_reported_norms(coarse, rounds, outer):
    from paper_2405_05047_amd import gen, mg
    wl = W.c1_poisson(rounds).with_(coarse=coarse, h0=1.0 / coarse[0])
    levels = gen.build(wl).levels
    top = levels[-1]
    h = mg.Hierarchy(levels, mg.config_from(wl, outer=outer))
    b = W.rand_vec(61, top.n) * (top.mask.reshape(-1) == 0)
    x = torch.zeros(top.n, dtype=torch.float64, device="cuda")
    st = h.solve(torch.from_numpy(b).cuda(), x, fixed=1)
    if np.linalg.norm(b) > 0.0:
        assert abs(st["res0"] - np.linalg.norm(b)) <= 64 * np.finfo(float).eps * np.linalg.norm(b)
    rd, norm = torch.empty_like(x), torch.empty(1, dtype=torch.float64, device="cuda")
    h.outer_defect(torch.from_numpy(b).cuda(), x, rd, norm)
    r = rd.cpu().numpy()
    assert abs(st["res_final"] - np.linalg.norm(r)) <= 64 * np.finfo(float).eps * np.linalg.norm(r)
