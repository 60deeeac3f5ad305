"""Operators in the node form against the same operators in the sliced-ELL form
(MGQ1_NODE_FORM=0 keeps that everywhere, =1 takes the node form on every level that can):
every step of the cycle, the V-cycle, the solve and the exported values are the same bits, in
every precision, on meshes with and without hanging nodes, 1 to 4 components."""
import dataclasses

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = {
    "poisson33": W.c1_poisson(4), "td_band": W.c2_td(band_rounds=3, uniform_rounds=1),
    "td_band_odd": W.c2_td(band_rounds=4, uniform_rounds=2, delta=0.031),
    "time5": W.td_time(6), "elast17": W.c3_elasticity(3), "oseen9": W.c4_oseen(2), "edge4": W.c3_adaptive("edge", 4),
    "face4": W.c3_adaptive("face", 4).with_(coarse=(4, 4, 4), h0=0.25),
}


def _vec(seed, n, real):
    return torch.from_numpy(W.rand_vec(seed, n)).cuda().to(real)


def _everything(levels, wl, prec, smoother, blocks=None):
    from paper_2405_05047_amd import mg
    h = mg.Hierarchy(levels, mg.config_from(wl, precision=prec, smoother=smoother), smoother_blocks=blocks)
    real = torch.float64 if h.cycle_fp64 else torch.float32
    out = []
    for l in range(h.n_levels):
        n = h.ndof(l)
        x, b, prev = _vec(10 + l, n, real), _vec(50 + l, n, real), torch.empty(n, dtype=real, device="cuda")
        for masked in (False, True):
            r = torch.empty_like(x)
            h.defect(l, b, x, r, masked=masked)
            out.append(r)
        y, sw, s0 = torch.empty_like(x), torch.empty_like(x), torch.empty_like(x)
        h.spmv(l, x, y)
        h.sweep(l, b, x, sw)
        h.sweep0(l, b, s0)
        out += [y, sw, s0]
        if l > 0:
            for start in (x, None):
                p = torch.empty_like(prev)
                h.smooth(l, b, start, p, 2)
                out.append(p)
        if prec != "fp64dict":
            out += [torch.from_numpy(np.asarray(a).astype(np.float64)) for a in h.export(l) if a is not None]
    N = h.ndof()
    b = _vec(90, N, torch.float64)
    b[torch.from_numpy(np.ascontiguousarray(levels[-1].mask)).reshape(-1).cuda() != 0] = 0.0
    z = torch.empty_like(b)
    h.vcycle(b, z)
    x = _vec(91, N, torch.float64)
    h.vcycle(b, x, x_is_zero=False)
    r, nrm = torch.empty_like(b), torch.empty(1, dtype=torch.float64, device="cuda")
    h.outer_defect(b, x, r, nrm)
    s = torch.zeros_like(b)
    st = h.solve(b, s, fixed=4)
    torch.cuda.synchronize()
    return out + [z, x, r, s], float(nrm), st["iters"], [h.dictionary_blocks(l) for l in range(h.n_levels)]


def _compare(levels, wl, prec, smoother, monkeypatch, blocks=None):
    got = []
    for form in ("0", "1"):
        monkeypatch.setenv("MGQ1_NODE_FORM", form)
        got.append(_everything(levels, wl, prec, smoother, blocks))
    (a, na, ia, da), (b, nb, ib, db) = got
    assert not any(da) and any(db), (da, db)
    assert ia == ib and len(a) == len(b)
    for k, (u, v) in enumerate(zip(a, b)):
        assert torch.equal(u, v), (k, float((u - v).abs().max()))
    # the reported norm sums its squares in the order of the form's workgroups
    assert abs(na - nb) <= 1e-13 * na


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("name", list(CASES))
def test_node_form_bitwise_equal(name, prec, monkeypatch):
    from paper_2405_05047_amd import gen
    wl = CASES[name]
    _compare(gen.build(wl).levels, wl, prec, W.SMOOTH_JACOBI, monkeypatch)


@pytest.mark.parametrize("name", ["td_band", "elast17", "face4"])
def test_node_form_chebyshev(name, monkeypatch):
    from paper_2405_05047_amd import gen
    wl = CASES[name]
    _compare(gen.build(wl).levels, wl, "fp64", W.SMOOTH_CHEBYSHEV, monkeypatch)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_node_form_caller_smoother(prec, monkeypatch):
    """Smoother blocks given by the caller, different at every node."""
    from paper_2405_05047_amd import gen
    wl = CASES["face4"]
    levels = gen.build(wl).levels
    rng = np.random.default_rng(8)
    blocks = [np.eye(3) * rng.uniform(0.1, 0.4, (lv.n, 1, 1)) for lv in levels]
    _compare(levels, wl, prec, W.SMOOTH_JACOBI, monkeypatch, blocks)


def test_node_form_two_components(monkeypatch):
    """Two components per node: the Kronecker product of the transport operator with a full
    2 x 2 matrix on the unconstrained nodes."""
    from paper_2405_05047_amd import gen
    wl = CASES["td_band"]
    K = np.array([[1.0, 0.25], [-0.125, 1.5]])
    levels = []
    for lv in gen.build(wl).levels:
        val = lv.val * K
        rows = np.repeat(np.arange(lv.n), np.diff(lv.rowptr))
        fixed = lv.mask.reshape(-1)[rows].astype(bool)
        val[fixed] = np.where((rows == lv.col)[fixed][:, None, None], np.eye(2), 0.0)
        levels.append(dataclasses.replace(lv, block=2, val=val, mask=np.repeat(lv.mask.reshape(-1, 1), 2, axis=1)))
    _compare(levels, wl.with_(block=2), "fp64", W.SMOOTH_JACOBI, monkeypatch)


def test_node_form_rule():
    """By itself the node form is taken where the FP64 blocks fill 16 MiB and rows repeat: the
    65^3 elasticity levels above 17^3, not the small ones, and no level of the flow step with
    its varying convection."""
    from paper_2405_05047_amd import gen, mg
    for wl, want in ((W.c3_elasticity(4).with_(coarse_level=2), [False, False, True]),
                     (W.c4_oseen(4).with_(coarse_level=2), [False, False, False])):
        h = mg.Hierarchy(gen.build(wl).levels, mg.config_from(wl))
        assert [h.dictionary_blocks(l) > 0 for l in range(h.n_levels)] == want


@pytest.mark.parametrize("wl", [W.c2_td().with_(coarse_level=3), W.c3_adaptive("face", 6)], ids=["td1m", "face6"])
def test_wide_transfers_bitwise_equal(wl, monkeypatch):
    """Transfers whose slots' columns span 2^16 and more (adaptive meshes of 1.0M and 0.7M
    nodes): the node form with 32-bit columns gives the bits of the per-DoF form, in FP64 and
    FP32."""
    from paper_2405_05047_amd import gen, mg
    levels = gen.build(wl).levels
    for prec, real in (("fp64", torch.float64), ("fp32", torch.float32)):
        got, wide = [], False
        for plain in ("1", "0"):
            monkeypatch.setenv("MGQ1_PLAIN_TRANSFERS", plain)
            h = mg.Hierarchy(levels, mg.config_from(wl, precision=prec))
            if plain == "0":
                wide = any(h.transfer_format(l)[1:] == (4, 1) for l in range(1, h.n_levels))
            out = []
            for l in range(1, h.n_levels):
                d = torch.zeros(h.ndof(l - 1), dtype=real, device="cuda")
                h.restrict(l, _vec(700 + l, h.ndof(l), real), d)
                x = _vec(740 + l, h.ndof(l), real)
                h.prolong(l, _vec(780 + l, h.ndof(l - 1), real), x)
                out += [d, x]
            got.append(out)
        assert wide and all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("name,rounds", [("elast", 1), ("elast", 3), ("oseen", 1), ("oseen", 3), ("poisson3", 3)])
@pytest.mark.parametrize("prec", ["fp64", "fp16"])
def test_relay_bitwise_equal(name, rounds, prec, monkeypatch):
    """The relay kernels of small levels (one slice per workgroup, MGQ1_NODE_FORM=0) against the
    node form's one wave per slice: rows of 8 to 27 blocks, fewer rows than a slice, and the
    one-component form."""
    from paper_2405_05047_amd import gen
    wl = {"elast": W.c3_elasticity(rounds).with_(coarse=(3, 2, 2)), "oseen": W.c4_oseen(rounds).with_(coarse=(2, 3, 2)),
          "poisson3": W.c3_elasticity(rounds).with_(pde=W.PDE_POISSON, block=1, dir_comps=1, rhs=W.RHS_NONE,
                                                    omega=0.8)}[name]
    _compare(gen.build(wl).levels, wl, prec, W.SMOOTH_JACOBI, monkeypatch)
