"""The host side of the node form on the CPU: for operators of every kind that it accepts (box
meshes with and without hanging nodes, 1 to 4 components, perturbed and random blocks, rows
of one block, fewer rows than a slice, columns too wide for 16 bits) the walk over its arrays
stays in bounds, visits every row once, and gives the sums of a plain block CSR product in
slot order bit for bit."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("node") / "node_form_check.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", os.path.join(HERE, "node_form_check.cpp"), "-o", so], check=True)
    f = C.CDLL(so).node_form_check
    f.restype = C.c_int

    def run(rowptr, col, val, must=True, exps=None, x=None):
        n, B = len(rowptr) - 1, val.shape[1]
        rowptr, col = np.ascontiguousarray(rowptr, np.int32), np.ascontiguousarray(col, np.int32)
        val = np.ascontiguousarray(val, np.float64)
        x = W.rand_vec(77, n * B) if x is None else x
        y, st = np.zeros(n * B), np.zeros(9, np.int64)
        p = lambda a: None if a is None else a.ctypes.data_as(C.c_void_p)  # noqa: E731
        rc = f(C.c_int32(n), C.c_int32(B), p(rowptr), p(col), p(val), p(exps), C.c_int32(int(must)), p(x), p(y),
               p(st))
        assert rc >= 0, rc
        if rc:
            assert np.array_equal(y, _product(rowptr, col, val, x))
        return rc, dict(zip(("slices", "slots", "general", "vu", "cu", "c32", "blocks", "regrouped", "runs"), st.tolist()))

    return run


def _product(rowptr, col, val, x):
    """Row sums in slot order with one fused multiply-add per product."""
    n, B = len(rowptr) - 1, val.shape[1]
    X = x.reshape(n, B)
    acc = np.zeros((n, B))
    ln = np.diff(rowptr)
    for k in range(int(ln.max())):
        rows = np.flatnonzero(ln > k)
        q = rowptr[rows] + k
        for cc in range(B):
            for c in range(B):
                acc[rows, c] = _fma(val[q, c, cc], X[col[q], cc], acc[rows, c])
    return acc.reshape(-1)


_libm = C.CDLL("libm.so.6")
_libm.fma.restype, _libm.fma.argtypes = C.c_double, [C.c_double] * 3


def _fma(a, b, c):
    return np.array([_libm.fma(*t) for t in zip(a.tolist(), b.tolist(), c.tolist())])


CASES = {
    "poisson": W.c1_poisson(4), "td_band": W.c2_td(band_rounds=2, uniform_rounds=1), "elast9": W.c3_elasticity(2), "elast17": W.c3_elasticity(3),
    "oseen9": W.c4_oseen(2), "face3": W.c3_adaptive("face", 3).with_(coarse=(2, 2, 2), h0=0.5),
    "time": W.td_time(5),
}


def _levels(name):
    from paper_2405_05047_amd import gen
    return gen.build(CASES[name]).levels


@pytest.mark.parametrize("name", ["poisson", "td_band", "elast9", "oseen9", "face3", "time"])
def test_walk_equals_product(check, name):
    for lv in _levels(name):
        rc, st = check(lv.rowptr, lv.col, lv.val)
        assert rc == 1 and st["slots"] * 64 >= len(lv.col)
        exps = np.clip(np.round(3 * W.rand_vec(5, lv.n * lv.block)), -2, 2).astype(np.int8)
        assert check(lv.rowptr, lv.col, lv.val, exps=exps)[0] == 1


def test_uniform_elasticity_stages_runs(check):
    lv = _levels("elast17")[-1]                    # 17^3 nodes, 3 components
    rc, st = check(lv.rowptr, lv.col, lv.val, must=False)
    assert rc == 1 and st["cu"] >= 0.9 * st["slices"] and st["runs"] >= 20


def test_uniform_mesh_is_mostly_uniform_slices(check):
    lv = _levels("time")[-1]                       # 33 x 33 nodes
    rc, st = check(lv.rowptr, lv.col, lv.val, must=False)
    assert rc == 1 and st["regrouped"] == 1 and st["cu"] >= 0.7 * st["slices"]


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 4095, 4096, 4097])
@pytest.mark.parametrize("B", [1, 2, 3, 4])
def test_row_counts(check, n, B):
    """Bands of equal rows cut by the slice and window sizes; every 37th row of one block."""
    rng = np.random.default_rng(n * 10 + B)
    kinds = rng.standard_normal((3, B, B))
    rows, cols, vals = [], [], []
    for i in range(n):
        js = [i] if i % 37 == 5 else [j for j in (i - 1, i, i + 1) if 0 <= j < n]
        rows.append(len(js))
        cols += js
        vals += [kinds[j - i + 1] for j in js]
    rc, st = check(np.concatenate([[0], np.cumsum(rows)]), np.array(cols), np.array(vals))
    assert rc == 1 and st["blocks"] <= 4


def test_wide_columns(check):
    """Columns 70,000 rows apart take the 32-bit form in the slices that need it."""
    n = 70200
    i = np.arange(n)
    far = (i * 7919 + 70000 * (i % 2)) % n
    cols = np.stack([np.minimum(i, far), np.maximum(i, far)], 1)
    keep = np.stack([np.ones(n, bool), i != far], 1)
    rp = np.concatenate([[0], np.cumsum(keep.sum(1))])
    val = np.where(cols[keep][:, None, None] == np.repeat(i, keep.sum(1))[:, None, None], 2.0, -0.5)
    rc, st = check(rp, cols[keep], val)
    assert rc == 1 and st["c32"] > 0


def test_refusals(check):
    """Random values: refused when asked to pay off; above 65,535 distinct blocks always."""
    rng = np.random.default_rng(3)
    n = 3000
    i = np.arange(n)
    cols = np.stack([np.maximum(i - 1, 0), i, np.minimum(i + 1, n - 1)], 1)
    keep = np.stack([i > 0, i >= 0, i < n - 1], 1)
    rp = np.concatenate([[0], np.cumsum(keep.sum(1))])
    val = rng.standard_normal((rp[-1], 1, 1))
    assert check(rp, cols[keep], val, must=False)[0] == 0
    assert check(rp, cols[keep], val, must=True)[0] == 1
    n = 33000
    rp = np.arange(n + 1) * 2
    j = np.arange(n)
    cols = np.sort(np.stack([j, (j + 1) % n], 1), axis=1).reshape(-1)
    assert check(rp, cols, rng.standard_normal((2 * n, 1, 1)), must=True)[0] == 0
