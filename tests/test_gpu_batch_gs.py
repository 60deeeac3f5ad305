"""Gram-Schmidt of the batched FGMRES: restart lengths up to, at and beyond one group of basis
vectors against the single solves of the same problems."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m", [1, 2, 10, 11, 24])
@pytest.mark.parametrize("nrhs", [1, 8])
def test_restart_lengths(m, nrhs):
    """A weak smoother makes the solves long enough to fill the bases.  Both solves reach the
    same relative residual (rtol 1e-10 here), so the solutions agree to that times the
    operator's condition number, below 1e4 at these sizes."""
    from paper_2405_05047_amd import gen, mg
    wls = [w.with_(rtol=1e-10) for w in W.batch_problems(n_problems=2, base_seed=2300, max_levels=4, min_levels=3)]
    probs = [gen.build(wl, nrhs) for wl in wls]
    cfg = dict(precision="fp64", gmres_m=m, omega=0.3, maxit=400)
    h = mg.Batch([p.levels for p in probs], mg.config_from(wls[0], **cfg), nrhs=nrhs)
    b = np.concatenate([np.asarray(p.b, np.float64).reshape(-1) for p in probs])
    x = torch.zeros(b.size, dtype=torch.float64, device="cuda")
    rc, st = h.solve(torch.from_numpy(b).cuda(), x)
    got = x.cpu().numpy()
    for k, p in enumerate(probs):
        s = mg.Hierarchy(p.levels, mg.config_from(wls[k], **cfg))
        seg = got[h.offsets[k]:h.offsets[k + 1]].reshape(-1, nrhs)
        for q in range(nrhs):
            rhs = np.ascontiguousarray(np.asarray(p.b, np.float64).reshape(-1, nrhs)[:, q])
            one = torch.zeros(rhs.size, dtype=torch.float64, device="cuda")
            ref = s.solve(torch.from_numpy(rhs).cuda(), one)
            i = st[k * nrhs + q]
            assert i["converged"] == ref["converged"] and abs(i["iters"] - ref["iters"]) <= 1
            if i["converged"]:
                e = one.cpu().numpy()
                assert np.linalg.norm(seg[:, q] - e) <= 1e-6 * np.linalg.norm(e)
