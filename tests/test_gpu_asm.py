"""GPU-side assembly of the constrained Q1 operators on adaptive meshes against the
oracle, through the C ABI.

A = Z (H^T A_full H) Z + I_C (Sec. 2.2) assembled on the GPU from the generator's mesh
(leaves, hanging nodes, masks, block pattern) must equal the oracle's operator of every
level: sums of at most 64 (3D, more next to hanging nodes) FP64 products of exact 1D
matrix entries, so 1e-13 of the largest entry is a loose bound; repeated assemblies are
bitwise identical (fixed summation order, no atomics); a hierarchy built from the
GPU-assembled values solves to the oracle's solution (1e-10, equal cycle counts)."""
import dataclasses
import sys

import numpy as np
import pytest

import workloads as W
from oracle import hierarchy as Hh, multigrid as MG

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _log(*a):
    print("[gpu-asm]", *a, flush=True)
    sys.stdout.flush()


CASES = {
    "poisson33": W.c1_poisson(4),
    "td_band": W.c2_td(band_rounds=3, uniform_rounds=1),
    "elast17": W.c3_elasticity(3),
    "edge4": W.c3_adaptive("edge", 4),
    "face3": W.c3_adaptive("face", 3),
    "td_time33": W.td_time(5),
}


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def _assemble(p, wl):
    from paper_2405_05047_amd import mg
    out = []
    for lv in p.levels:
        a = mg.Assembly(lv, wl.dim)
        val = torch.empty(lv.nnzb * lv.block * lv.block, dtype=torch.float64, device="cuda")
        a.values(mg.asm_coef(wl), val)
        out.append((a, val))
    return out


@pytest.mark.parametrize("name", list(CASES))
def test_assembled_operators_match_oracle(name):
    from paper_2405_05047_amd import gen, mg
    wl = CASES[name]
    o = Hh.build(wl)
    p = gen.build(wl)
    worst = 0.0
    for l, ((a, val), lo, lg) in enumerate(zip(_assemble(p, wl), o.levels, p.levels)):
        assert np.array_equal(lg.col, lo.col)
        got = host(val).reshape(lo.val.shape)
        err = np.abs(got - lo.val).max() / np.abs(lo.val).max()
        worst = max(worst, err)
        assert err <= 1e-13, (name, l, err)
        again = torch.empty_like(val)
        a.values(mg.asm_coef(wl), again)
        assert np.array_equal(host(again), host(val))
    _log(name, f"{len(o.levels)} levels, worst relative difference {worst:.2e}")


def test_coefficient_change_reassembles():
    """The same mesh, new coefficients: only the numeric phase runs again."""
    from paper_2405_05047_amd import gen, mg
    wl = W.c3_adaptive("edge", 3)
    p = gen.build(wl)
    top = p.finest
    a = mg.Assembly(top, wl.dim)
    val = torch.empty(top.nnzb * 9, dtype=torch.float64, device="cuda")
    for lam, mu in ((1.0, 0.5), (8e4, 2e4), (0.3, 1.7)):
        w2 = wl.with_(lam=lam, mu=mu)
        a.values(mg.asm_coef(w2), val)
        ref = Hh.build(w2).finest.val
        assert np.abs(host(val).reshape(ref.shape) - ref).max() <= 1e-13 * np.abs(ref).max(), (lam, mu)


@pytest.mark.parametrize("name", ["td_band", "edge4"])
def test_solve_with_gpu_assembled_hierarchy(name):
    from paper_2405_05047_amd import gen, mg
    wl = CASES[name]
    o = Hh.build(wl)
    p = gen.build(wl)
    levels = [dataclasses.replace(lv, val=host(val).reshape(lv.val.shape))
              for lv, (a, val) in zip(p.levels, _assemble(p, wl))]
    h = mg.Hierarchy(levels, mg.config_from(wl))
    b = torch.from_numpy(o.b).cuda()
    x = torch.zeros_like(b)
    st = h.solve(b, x)
    xr, sr = MG.Multigrid(o).solve(o.b)
    assert st["converged"] == 1 and st["iters"] == sr.iters
    assert np.linalg.norm(host(x) - xr) <= 1e-10 * np.linalg.norm(xr)


def test_invalid_assembly_input_refused():
    from paper_2405_05047_amd import gen, mg
    wl = W.c2_td(band_rounds=2, uniform_rounds=1)
    top = gen.build(wl).finest
    bad = dataclasses.replace(top, cells=np.where(np.arange(top.cells.size).reshape(top.cells.shape) == 5,
                                                  top.n, top.cells))
    with pytest.raises(mg.MGError):
        mg.Assembly(bad, wl.dim)
    a = mg.Assembly(top, wl.dim)
    val = torch.empty(top.nnzb, dtype=torch.float64, device="cuda")
    with pytest.raises(mg.MGError):
        a.values(mg.asm_coef(W.c3_elasticity(1)), val)     # elasticity on a scalar pattern


@pytest.mark.parametrize("name", ["poisson33", "td_band", "elast17", "edge4", "face3", "td_time33"])
def test_distinct_lists_bitwise_equal(name, monkeypatch):
    """Summing each distinct contribution list once and spreading it over its blocks gives the
    bits of the block-by-block sums, on every level (workgroups of 256 blocks with every kind
    of remainder), also next to hanging nodes and constrained unknowns."""
    from paper_2405_05047_amd import gen
    wl = CASES[name]
    p = gen.build(wl)
    got = []
    for lists in ("0", "1"):
        monkeypatch.setenv("MGQ1_ASM_LISTS", lists)
        got.append([host(val) for _, val in _assemble(p, wl)])
    assert all(np.array_equal(a, b) for a, b in zip(*got))
