"""Host memory that a handle keeps for its levels in the node form: what maps stored values back
(row pointers, positions, block numbers of general slices), not the arrays of the kernels."""
import ctypes
import gc

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


class _Mallinfo(ctypes.Structure):
    _fields_ = [(k, ctypes.c_size_t) for k in ("arena", "ordblks", "smblks", "hblks", "hblkhd", "usmblks", "fsmblks",
                                               "uordblks", "fordblks", "keepcost")]


def _in_use():
    f = ctypes.CDLL(None).mallinfo2
    f.restype = _Mallinfo
    gc.collect()
    m = f()
    return m.uordblks + m.hblkhd


def test_host_memory_of_node_levels():
    """172,505 and 24,367 nodes refined towards a face: two thirds of the slices have columns of
    their own, 2 bytes per slot row and lane.  Kept are 8 bytes per node, at most 2 per stored
    block in general slices (1.7% of the slots), 1 MiB for everything else."""
    from paper_2405_05047_amd import gen, mg
    wl = W.c3_adaptive("face", 5)
    levels = gen.build(wl).levels
    cfg = mg.config_from(wl)
    first = mg.Hierarchy(levels, cfg)                # the runtime's own allocations
    n, nnzb = (sum(first.sizes[l][k] for l in range(first.n_levels)) for k in (0, 2))
    assert first.dictionary_blocks(first.n_levels - 1) > 0
    torch.cuda.synchronize()
    before = _in_use()
    second = mg.Hierarchy(levels, cfg)
    torch.cuda.synchronize()
    kept = _in_use() - before
    assert kept <= 8 * n + 0.05 * 2 * nnzb + (1 << 20), (kept, n, nnzb)
    # and the values can still be mapped back
    val = second.export(second.n_levels - 1)[0]
    assert np.array_equal(np.asarray(val).reshape(-1), np.asarray(levels[-1].val).reshape(-1))
