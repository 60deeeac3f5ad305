"""The batch's two-pass Gram-Schmidt at a fixed number of cycles, far from convergence, where every
basis vector counts: iterates against the single solves.

Tolerance: 1e-10 relative, that of every fixed-count comparison (test_gpu_gs)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m,cycles", [(1, 3), (2, 4), (10, 10), (11, 13), (24, 24)])
@pytest.mark.parametrize("nrhs", [1, 8])
def test_iterates(m, cycles, nrhs):
    from paper_2405_05047_amd import gen, mg
    wls = W.batch_problems(n_problems=2, base_seed=2300, max_levels=4, min_levels=3)
    probs = [gen.build(wl, nrhs) for wl in wls]
    weak = dict(gmres_m=m, omega=0.05, nu1=1, nu2=0, rtol=1e-14)
    h = mg.Batch([p.levels for p in probs], mg.config_from(wls[0], maxit=cycles, **weak), nrhs=nrhs)
    b = np.concatenate([np.asarray(p.b, np.float64).reshape(-1) for p in probs])
    x = torch.zeros(b.size, dtype=torch.float64, device="cuda")
    _, st = h.solve(torch.from_numpy(b).cuda(), x)
    got = x.cpu().numpy()
    for k, p in enumerate(probs):
        s = mg.Hierarchy(p.levels, mg.config_from(wls[k], **weak))
        seg = got[h.offsets[k]:h.offsets[k + 1]].reshape(-1, nrhs)
        for q in range(nrhs):
            rhs = np.ascontiguousarray(np.asarray(p.b, np.float64).reshape(-1, nrhs)[:, q])
            one = torch.zeros(rhs.size, dtype=torch.float64, device="cuda")
            ref = s.solve(torch.from_numpy(rhs).cuda(), one, fixed=cycles)
            assert st[k * nrhs + q]["iters"] == ref["iters"] == cycles
            assert ref["res_final"] > 1e-6 * np.linalg.norm(rhs), "the comparison wants an unconverged iterate"
            e = one.cpu().numpy()
            assert np.linalg.norm(seg[:, q] - e) <= 1e-10 * np.linalg.norm(e)
