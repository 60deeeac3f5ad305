"""The batch's small levels as one dense product (FP64) against the level by level cycle
(MGQ1_NO_DENSE=1): iteration counts and solutions, one and eight right-hand sides, 1, 3 and 4
components, problems that are small as a whole, and a batch that is too large for it."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GROUPS = {
    "nrhs8": (lambda: W.batch_problems(n_problems=5, base_seed=2100, max_levels=5, min_levels=2), 8),
    "nrhs1": (lambda: W.batch_problems(n_problems=5, base_seed=2100, max_levels=6, min_levels=2), 1),
    "elast": (lambda: [W.c3_elasticity(2), W.c3_elasticity(3).with_(coarse_level=1), W.c3_adaptive("edge", 3)], 1),
    "oseen": (lambda: [W.c4_oseen(2), W.c4_oseen(3), W.c4_oseen(2, seed=5)], 1),
}


@pytest.mark.parametrize("use_graph", [0, 1])
@pytest.mark.parametrize("name", list(GROUPS))
def test_dense_levels(name, use_graph, monkeypatch):
    """The cycle is the same linear map; the two orders of summation differ by a few ulp per
    unknown, far below the solve's tolerance."""
    from paper_2405_05047_amd import gen, mg
    make, nrhs = GROUPS[name]
    wls = make()
    probs = [gen.build(wl, nrhs) for wl in wls]
    b = torch.from_numpy(np.concatenate([np.asarray(p.b, np.float64).reshape(-1) for p in probs])).cuda()
    got = []
    for off in ("1", "0"):
        monkeypatch.setenv("MGQ1_NO_DENSE", off)
        h = mg.Batch([p.levels for p in probs], mg.config_from(wls[0], use_graph=use_graph), nrhs=nrhs)
        xs = []
        for _ in range(3):
            x = torch.zeros_like(b)
            rc, st = h.solve(b, x)
            assert rc == 0
            xs.append(x.cpu().numpy())
        assert all(np.array_equal(x, xs[0]) for x in xs)
        got.append((xs[0], [s["iters"] for s in st], h.offsets))
    (a, ia, off), (c, ic, _) = got
    assert ia == ic
    assert not np.array_equal(a, c)                  # the product is in use
    for p in range(len(probs)):
        u, v = a[off[p]:off[p + 1]], c[off[p]:off[p + 1]]
        assert np.linalg.norm(u - v) <= 1e-10 * np.linalg.norm(u)
