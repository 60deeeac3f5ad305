"""Which assemblies sum each distinct contribution list once: shown by the device memory of the
handle (2 bytes per block by lists; 12 bytes per block and 2 per contribution block by block)."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _square(n):
    return W.c1_poisson(7).with_(coarse=(n, n), h0=1.0 / n)


# by lists: 385^2 nodes write 10.5 MB (10.05 MiB), 257^2 4.7 MB; 11,281 nodes refined towards a
# face write 16.5 MB; 8,569 towards an edge 11.4 MB with lists of up to 116; 17^3 nodes 8 MB
CASES = {"square257": (_square(2), False), "square385": (_square(3), True),
         "edge4": (W.c3_adaptive("edge", 4), True), "elast17": (W.c3_elasticity(3), False)}


def _bytes(level, dim, keep):
    """Device memory of eight more handles."""
    from paper_2405_05047_amd import mg
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    keep += [mg.Assembly(level, dim) for _ in range(8)]
    torch.cuda.synchronize()
    return free - torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("name", list(CASES))
def test_route(name, monkeypatch):
    from paper_2405_05047_amd import gen
    wl, lists = CASES[name]
    p = gen.build(wl)
    used, keep = {}, []                              # all stay alive: nothing is reused
    for force in ("0", "1", "0", "1", None):         # the first of each kind also loads kernels
        monkeypatch.delenv("MGQ1_ASM_LISTS", raising=False)
        if force is not None:
            monkeypatch.setenv("MGQ1_ASM_LISTS", force)
        used[force] = _bytes(p.finest, wl.dim, keep)
    assert used["1"] < used["0"]
    assert (2 * used[None] < used["0"] + used["1"]) == lists, used
