"""Operators in the flow form against the same operators in the sliced-ELL form: every step of
the cycle, the V-cycle, the solve and the exported values are the same bits, on levels that
do not fill the last slice, with every smoother source, and only where every block has the shape."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from test_gpu_node_form import _everything

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = {"oseen9": W.c4_oseen(2), "oseen17": W.c4_oseen(3), "odd": W.c4_oseen(2).with_(coarse=(3, 5, 2), h0=0.25)}


def _two(levels, wl, prec, smoother, monkeypatch, blocks=None):
    got = []
    for node, flow in (("0", "0"), ("0", "1")):
        monkeypatch.setenv("MGQ1_NODE_FORM", node)
        monkeypatch.setenv("MGQ1_FLOW_FORM", flow)
        got.append(_everything(levels, wl, prec, smoother, blocks))
    (a, na, ia, _), (b, nb, ib, db) = got
    assert not any(db) and ia == ib and len(a) == len(b)
    for k, (u, v) in enumerate(zip(a, b)):
        assert torch.equal(u, v), (k, float((u - v).abs().max()))
    # the reported norm sums its squares in the order of the form's workgroups
    assert abs(na - nb) <= 1e-13 * na


@pytest.mark.parametrize("smoother", [W.SMOOTH_JACOBI, W.SMOOTH_CHEBYSHEV])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("name", list(CASES))
def test_flow_form_bitwise_equal(name, prec, smoother, monkeypatch):
    from paper_2405_05047_amd import gen
    wl = CASES[name]
    _two(gen.build(wl).levels, wl, prec, smoother, monkeypatch)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_flow_form_caller_smoother(prec, monkeypatch):
    from paper_2405_05047_amd import gen
    wl = CASES["odd"]
    levels = gen.build(wl).levels
    rng = np.random.default_rng(5)
    blocks = [np.eye(4) * rng.uniform(0.1, 0.4, (lv.n, 1, 1)) + rng.uniform(-0.05, 0.05, (lv.n, 4, 4))
              for lv in levels]
    _two(levels, wl, prec, W.SMOOTH_JACOBI, monkeypatch, blocks)


@pytest.mark.parametrize("entry,value", [(6, 1e-300), (5, None), (14, -0.0)])
def test_flow_form_one_other_block(entry, value, monkeypatch):
    """One block off the shape (a value in a zero place, another diagonal, a negative zero): the
    level keeps the sliced-ELL form, with the same bits as ever."""
    from paper_2405_05047_amd import gen
    wl = CASES["oseen9"]
    levels = gen.build(wl).levels
    lv = levels[-1]
    val = lv.val.copy()
    k = int(lv.rowptr[lv.n // 2])
    val[k].reshape(-1)[entry] = 1.5 * val[k].reshape(-1)[entry] + 1e-9 if value is None else value
    _two(levels[:-1] + [dataclasses.replace(lv, val=val)], wl, "fp64", W.SMOOTH_JACOBI, monkeypatch)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp64dict"])
def test_flow_form_by_size(prec, monkeypatch):
    """35,937 nodes take the form by themselves (their blocks are too many for a dictionary)."""
    from paper_2405_05047_amd import gen
    wl = W.c4_oseen(4)
    levels = gen.build(wl).levels
    got = []
    for flow in ("0", None):
        monkeypatch.setenv("MGQ1_FLOW_FORM", flow) if flow else monkeypatch.delenv("MGQ1_FLOW_FORM")
        got.append(_everything(levels, wl, prec, W.SMOOTH_JACOBI))
    (a, na, ia, _), (b, nb, ib, _) = got
    assert ia == ib
    for k, (u, v) in enumerate(zip(a, b)):
        assert torch.equal(u, v), k
    assert abs(na - nb) <= 1e-13 * na
