"""A batch whose levels bring the caller's smoother blocks: the dense product of the small levels
(FP64) is that of the cycle with these blocks, with one and eight right-hand sides, also
where a diagonal block is singular and could not have given a smoother block."""
import dataclasses

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GROUPS = {
    "nrhs8": (lambda: W.batch_problems(n_problems=3, base_seed=2100, max_levels=5, min_levels=3), 8),
    "nrhs1": (lambda: W.batch_problems(n_problems=3, base_seed=2100, max_levels=5, min_levels=3), 1),
    "elast": (lambda: [W.c3_elasticity(2), W.c3_elasticity(3).with_(coarse_level=1)], 1),
}


def _blocks(rng, lv):
    """Random multiples of the inverse diagonal blocks (the identity where the block is singular)."""
    row = np.repeat(np.arange(lv.n), np.diff(lv.rowptr))
    d = lv.val.reshape(-1, lv.block, lv.block)[row == lv.col].copy()
    d[np.abs(np.linalg.det(d)) == 0.0] = np.eye(lv.block)
    return np.linalg.inv(d) * rng.uniform(0.4, 1.0, (lv.n, 1, 1))


def _zero_diagonal(lv):
    """The level with the diagonal of one unconstrained node zero."""
    i = int(np.flatnonzero(lv.mask.reshape(lv.n, -1).sum(axis=1) == 0)[0])
    val = lv.val.copy()
    val[lv.rowptr[i] + int(np.flatnonzero(lv.col[lv.rowptr[i]:lv.rowptr[i + 1]] == i)[0])] = 0.0
    return dataclasses.replace(lv, val=val)


@pytest.mark.parametrize("singular", [False, True])
@pytest.mark.parametrize("name", list(GROUPS))
def test_caller_smoother_on_dense_levels(name, singular, monkeypatch):
    """Three cycles, unconverged: the batch with the dense product, level by level
    (MGQ1_NO_DENSE=1) and the single solves agree to 1e-10, the bound of every comparison at a
    fixed number of cycles; without the caller's blocks the iterates are others."""
    from paper_2405_05047_amd import gen, mg
    make, nrhs = GROUPS[name]
    wls = make()
    probs = [gen.build(wl, nrhs) for wl in wls]
    levels = [list(p.levels) for p in probs]
    if singular:
        levels[0][1] = _zero_diagonal(levels[0][1])
    rng = np.random.default_rng(31)
    blocks = [[_blocks(rng, lv) for lv in ls] for ls in levels]
    cfg = dict(maxit=3, rtol=1e-14)
    b = np.concatenate([np.asarray(p.b, np.float64).reshape(-1) for p in probs])

    structs = mg.level_structs

    def batch(bl):
        given = iter(bl)
        monkeypatch.setattr(mg, "level_structs", lambda ls, _=None: structs(ls, next(given)))
        h = mg.Batch(levels, mg.config_from(wls[0], **cfg), nrhs=nrhs)
        monkeypatch.setattr(mg, "level_structs", structs)
        x = torch.zeros(b.size, dtype=torch.float64, device="cuda")
        _, st = h.solve(torch.from_numpy(b).cuda(), x)
        assert all(s["iters"] == 3 for s in st)
        return x.cpu().numpy(), h.offsets

    monkeypatch.setenv("MGQ1_NO_DENSE", "0")
    got, off = batch(blocks)
    if not singular:
        assert not np.allclose(got, batch([None] * len(levels))[0], rtol=1e-6, atol=0.0)
    monkeypatch.setenv("MGQ1_NO_DENSE", "1")
    ref, _ = batch(blocks)
    assert not np.array_equal(got, ref)              # the product is in use
    for p, ls in enumerate(levels):
        u, v = got[off[p]:off[p + 1]].reshape(-1, nrhs), ref[off[p]:off[p + 1]].reshape(-1, nrhs)
        h = mg.Hierarchy(ls, mg.config_from(wls[p], **cfg), smoother_blocks=blocks[p])
        rhs = np.asarray(probs[p].b, np.float64).reshape(-1, nrhs)
        for q in range(nrhs):
            one = torch.zeros(len(u), dtype=torch.float64, device="cuda")
            h.solve(torch.from_numpy(np.ascontiguousarray(rhs[:, q])).cuda(), one, fixed=3)
            w = one.cpu().numpy()
            for t in (u[:, q], v[:, q]):
                assert np.linalg.norm(t - w) <= 1e-10 * np.linalg.norm(w), (p, q)
