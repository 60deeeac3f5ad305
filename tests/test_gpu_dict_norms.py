"""MG_PREC_FP64_DICT handles against plain FP64 ones: the reported norms too have the same bits
(both lay a level out in the same slices, so the partial sums are the same), on levels below
and above the size of the node form."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = {
    "poisson33": W.c1_poisson(4), "td_band": W.c2_td(band_rounds=3, uniform_rounds=1), "elast17": W.c3_elasticity(3),
    "oseen9": W.c4_oseen(2), "face4": W.c3_adaptive("face", 4), "elast33": W.c3_elasticity(4).with_(coarse_level=2),
}


@pytest.mark.parametrize("outer", [W.OUTER_IR, W.OUTER_FGMRES])
@pytest.mark.parametrize("name", list(CASES))
def test_norms_bitwise_equal(name, outer):
    from paper_2405_05047_amd import gen, mg
    wl = CASES[name]
    levels = gen.build(wl).levels
    got = []
    for prec in ("fp64", "fp64dict"):
        h = mg.Hierarchy(levels, mg.config_from(wl, precision=prec, outer=outer))
        b, x = (torch.from_numpy(W.rand_vec(s, h.ndof())).cuda() for s in (31, 32))
        b[torch.from_numpy(np.ascontiguousarray(levels[-1].mask)).reshape(-1).cuda() != 0] = 0.0
        out = []
        for defect in (h.outer_defect, h.outer_defect_noalloc):
            r, norm = torch.empty_like(b), torch.empty(1, dtype=torch.float64, device="cuda")
            defect(b, x, r, norm)
            out += [r.cpu().numpy(), norm.cpu().numpy()]
        z = torch.zeros_like(b)
        st = h.solve(b, z, fixed=3)
        out += [z.cpu().numpy(), np.array([st["res0"], st["res_final"]])]
        got.append(out)
        assert prec == "fp64" or all(h.dictionary_blocks(l) > 0 for l in range(1, h.n_levels))
    for a, c in zip(*got):
        assert np.array_equal(a, c)
