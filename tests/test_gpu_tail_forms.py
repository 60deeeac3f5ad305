"""The single-workgroup tail (MGQ1_TAIL_DOFS) over a hierarchy whose middle level is larger than
the limit: every level in the tail keeps the sliced layout, whatever MGQ1_NODE_FORM asks."""
import dataclasses

import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _levels():
    """5 x 5, 33 x 33 and 17 x 17 nodes of the Poisson problem: prolongation from the first to
    the second over the meshes between them, injection from the second to the third."""
    from paper_2405_05047_amd import gen
    ls = gen.build(W.c1_poisson(4)).levels                     # 3^2, 5^2, 9^2, 17^2, 33^2 nodes
    P = sp.identity(ls[1].n, format="csr")
    for l in (2, 3, 4):
        lv = ls[l]
        P = sp.csr_matrix((lv.p_val, lv.p_col, lv.p_rowptr), shape=(lv.n, ls[l - 1].n)) @ P
    P.sort_indices()
    at = {tuple(c): i for i, c in enumerate(ls[4].lattice.tolist())}
    same = np.array([at[tuple(c)] for c in ls[3].lattice.tolist()], np.int32)
    with_p = lambda lv, rp, col, val, n: dataclasses.replace(  # noqa: E731
        lv, p_rowptr=rp.astype(np.int32), p_col=col.astype(np.int32), p_val=val.astype(np.float64), p_cols=n)
    return [dataclasses.replace(ls[1], p_rowptr=None, p_col=None, p_val=None, p_cols=0),
            with_p(ls[4], P.indptr, P.indices, P.data, ls[1].n),
            with_p(ls[3], np.arange(ls[3].n + 1), same, np.ones(ls[3].n), ls[4].n)]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
def test_level_above_the_limit_inside_the_tail(prec, monkeypatch):
    from paper_2405_05047_amd import mg
    levels = _levels()
    b = torch.from_numpy(W.rand_vec(12, levels[-1].n) * (levels[-1].mask.reshape(-1) == 0)).cuda()
    monkeypatch.setenv("MGQ1_NO_DENSE", "1")
    got = []
    for tail, node in (("0", "0"), ("300", "0"), ("300", "1")):
        monkeypatch.setenv("MGQ1_TAIL_DOFS", tail)
        monkeypatch.setenv("MGQ1_NODE_FORM", node)
        h = mg.Hierarchy(levels, mg.config_from(W.c1_poisson(4), precision=prec))
        if tail != "0":
            assert not any(h.dictionary_blocks(l) for l in range(h.n_levels))
        x = torch.empty_like(b)
        h.vcycle(b, x)
        got.append(x.cpu().numpy())
    assert np.isfinite(got[0]).all() and np.abs(got[0]).max() > 0.0
    # the tail runs the same steps in the same order
    assert np.abs(got[1] - got[0]).max() <= (1e-12 if prec == "fp64" else 1e-5) * np.abs(got[0]).max()
    assert np.array_equal(got[1], got[2])
