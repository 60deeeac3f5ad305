"""Which levels take the node form by themselves: by the bytes of the cycle's values, by the share
of uniform slices (one component) and of general ones (several)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# finest level in the node form, per precision
CASES = {
    # 25^3 nodes, 25.7 MiB of FP64 blocks: the relay of the sliced form is faster
    "elast25": (W.c3_elasticity(3).with_(coarse=(3, 3, 3), h0=1 / 3), {"fp64": False, "fp32": False, "fp16": False}),
    # 29^3 nodes: 41, 20 and 10 MiB of values; 33^3 nodes: 61, 30 and 15.2
    "elast29": (W.c3_elasticity(2).with_(coarse=(7, 7, 7), h0=1 / 7), {"fp64": True, "fp32": False, "fp16": False}),
    "elast33": (W.c3_elasticity(4), {"fp64": True, "fp32": True, "fp16": True, "bf16": True}),
    # 45 MiB of FP64 blocks, a fifth of the slots in general slices
    "edge6": (W.c3_adaptive("edge", 6), {"fp64": False, "fp32": False, "fp16": False}),
    # 449^2 and 513^2 nodes: 17, 10 MiB and 22, 13.4, 9 MiB of values and columns
    "poisson449": (W.c1_poisson(6).with_(coarse=(7, 7), h0=1 / 7), {"fp64": True, "fp32": False, "fp16": False}),
    "time9": (W.td_time(9), {"fp64": True, "fp32": True, "fp16": False}),
    # 259,665 nodes, 22 and 13 MiB, 15% of the slices with columns of their own
    "td2d": (W.c2_td(band_rounds=5), {"fp64": False, "fp32": False}),
}


@pytest.mark.parametrize("name", list(CASES))
def test_rule(name):
    from paper_2405_05047_amd import gen, mg
    wl, want = CASES[name]
    levels = gen.build(wl).levels
    for prec, node in want.items():
        h = mg.Hierarchy(levels, mg.config_from(wl, precision=prec))
        assert (h.dictionary_blocks(h.n_levels - 1) > 0) == node, prec
        assert not any(h.dictionary_blocks(l) for l in range(h.n_levels - 1) if h.sizes[l][2] < 200_000)
        b = torch.from_numpy(W.rand_vec(3, h.ndof())).cuda()
        b[torch.from_numpy(np.ascontiguousarray(levels[-1].mask)).reshape(-1).cuda() != 0] = 0.0
        x = torch.empty_like(b)
        h.vcycle(b, x)
        assert bool(torch.isfinite(x).all())
