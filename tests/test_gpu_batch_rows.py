"""The batch with its launches' blocks shared by a few workgroups (MGQ1_BATCH_GRID) against one
workgroup per block: the same bits while problems converge one after the other; and with
vectors that are only 8-byte aligned."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GROUPS = {
    "nrhs8": (lambda: W.batch_problems(n_problems=5, base_seed=2100, max_levels=5, min_levels=3), 8),
    "nrhs1": (lambda: W.batch_problems(n_problems=5, base_seed=2100, max_levels=5, min_levels=3), 1),
    "elast": (lambda: [W.c3_elasticity(2), W.c3_elasticity(3).with_(coarse_level=1), W.c3_adaptive("edge", 3)], 1),
}


def _solve(name, prec, monkeypatch, grid=None, shift=0, use_graph=0):
    from paper_2405_05047_amd import gen, mg
    make, nrhs = GROUPS[name]
    wls = make()
    probs = [gen.build(wl, nrhs) for wl in wls]
    if grid is None:
        monkeypatch.delenv("MGQ1_BATCH_GRID", raising=False)
    else:
        monkeypatch.setenv("MGQ1_BATCH_GRID", str(grid))
    h = mg.Batch([p.levels for p in probs], mg.config_from(wls[0], precision=prec, use_graph=use_graph), nrhs=nrhs)
    b = np.concatenate([np.asarray(p.b, np.float64).reshape(-1) for p in probs])
    b[: b.size // 3] *= np.random.default_rng(3).uniform(0.5, 1.5, b.size // 3)   # uneven convergence
    bd = torch.zeros(b.size + shift, dtype=torch.float64, device="cuda")[shift:]
    bd.copy_(torch.from_numpy(b))
    x = torch.zeros(b.size + shift, dtype=torch.float64, device="cuda")[shift:]
    _, st = h.solve(bd, x)
    torch.cuda.synchronize()
    return x.cpu().numpy(), [s["iters"] for s in st]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("name", list(GROUPS))
def test_shared_blocks_bitwise_equal(name, prec, monkeypatch):
    ref, iters = _solve(name, prec, monkeypatch)
    assert name == "elast" or len(set(iters)) > 1    # some finish before others
    for grid in (1, 8, 24):
        got, it = _solve(name, prec, monkeypatch, grid=grid)
        assert it == iters and np.array_equal(got, ref), grid


def test_shared_blocks_in_graphs(monkeypatch):
    ref, iters = _solve("nrhs8", "fp64", monkeypatch)
    got, it = _solve("nrhs8", "fp64", monkeypatch, grid=8, use_graph=1)
    assert it == iters and np.array_equal(got, ref)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_vectors_at_any_element(prec, monkeypatch):
    ref, iters = _solve("nrhs8", prec, monkeypatch)
    got, it = _solve("nrhs8", prec, monkeypatch, shift=1)
    assert it == iters and np.array_equal(got, ref)
