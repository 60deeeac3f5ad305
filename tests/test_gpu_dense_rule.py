"""Where the V-cycle of the small levels is one dense product: with and without it (MGQ1_NO_DENSE=1)
the last bits differ where it is in use and are the same where it is not; and a batch whose
matrices would exceed their common size takes smaller levels."""
import numpy as np
import pytest

import workloads as W
from test_gpu_dense import CASES

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# precision, smoother, in use; "above" has its second level above the limit
RULE = [(name, "fp64", W.SMOOTH_JACOBI, name != "above") for name in CASES] + \
       [("td", "fp64dict", W.SMOOTH_JACOBI, True), ("td", "fp32", W.SMOOTH_JACOBI, False),
        ("elast", "fp64", W.SMOOTH_CHEBYSHEV, False)]


@pytest.mark.parametrize("name,prec,smoother,used", RULE)
def test_product_is_in_use(name, prec, smoother, used, monkeypatch):
    from paper_2405_05047_amd import gen, mg
    wl = CASES[name]
    levels = gen.build(wl).levels
    b = W.rand_vec(41, levels[-1].n * levels[-1].block) * (levels[-1].mask.reshape(-1) == 0)
    got = []
    for off in ("1", "0"):
        monkeypatch.setenv("MGQ1_NO_DENSE", off)
        h = mg.Hierarchy(levels, mg.config_from(wl, precision=prec, smoother=smoother))
        x = torch.empty(len(b), dtype=torch.float64, device="cuda")
        h.vcycle(torch.from_numpy(b).cuda(), x)
        got.append(x.cpu().numpy())
    assert np.array_equal(*got) != used


def test_batch_matrices_above_their_common_size(monkeypatch):
    """24 problems of 64, 225 and 841 unknowns: matrices of 841 rows would take 136 MB together,
    so those of 225 rows are taken.  Three cycles agree with the level by level batch to 1e-10."""
    from paper_2405_05047_amd import gen, mg
    wls = [W.c1_poisson(2).with_(coarse=(7, 7), h0=1 / 7, seed=k) for k in range(24)]
    probs = [gen.build(wl) for wl in wls]
    b = torch.from_numpy(np.concatenate([W.rand_vec(50 + k, p.finest.n) * (p.finest.mask.reshape(-1) == 0)
                                         for k, p in enumerate(probs)])).cuda()
    got = []
    for off in ("1", "0"):
        monkeypatch.setenv("MGQ1_NO_DENSE", off)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        h = mg.Batch([p.levels for p in probs], mg.config_from(wls[0], outer=W.OUTER_FGMRES, maxit=3, rtol=1e-14))
        torch.cuda.synchronize()
        assert free - torch.cuda.mem_get_info()[0] < 136e6
        x = torch.zeros_like(b)
        _, st = h.solve(b, x)
        assert all(s["iters"] == 3 for s in st)
        got.append(x.cpu().numpy())
    assert not np.array_equal(*got)
    assert np.linalg.norm(got[0] - got[1]) <= 1e-10 * np.linalg.norm(got[0])
