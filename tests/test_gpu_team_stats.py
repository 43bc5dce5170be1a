"""GPU: a team's count of rounds stays within the bound that the shifts give, also where its last step of several
rounds reaches past it; and its members by default."""
import numpy as np
import pytest

import inputs
import oracle
from graphs import S, path

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ldd():
    import torch
    assert torch.cuda.is_available()
    import paper_1307_3692_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("kind", ["path", "rgg"])
@pytest.mark.parametrize("blocks", [0, 8, 40])
def test_rounds_within_their_bound(ldd, kind, blocks):
    import torch
    if kind == "path":  # the search from one end takes every round there is
        rp, ci = path(4001)
        s = np.zeros(4001, np.int64)
        s[0] = 4000 * S
    else:
        rp, ci = inputs.rgg(50_000, 6.0, 3)
        s = inputs.make_shifts(50_000, 0.05, 7)
    d = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (rp, ci, s)]
    print(f"{kind} blocks {blocks}", flush=True)
    _, _, st = ldd.decompose(*d, 0.1, stats=True, engine=4, blocks=blocks, tail_vertices=-1)
    assert st["steps"] == 1 and st["blocks"] > 1
    assert st["rounds_bound"] == s.max() // S + 1
    assert st["rounds"] <= st["rounds_bound"]
    if kind == "path":
        assert st["rounds"] == 4001


@pytest.mark.parametrize("n,degree", [(5000, 6.0), (40_000, 6.0), (40_000, 20.0), (40_000, 150.0)])
def test_default_members(ldd, n, degree):
    """They grow with the vertices, and more slowly with the arcs per vertex beyond 7."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rp, ci = inputs.er(n, degree, 5)
    s = inputs.make_shifts(n, 0.2, 5)
    want, _, want_cut = oracle.decompose(rp, ci, s)
    d = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (rp, ci, s)]
    print(f"n {n} degree {degree}", flush=True)
    centre, cut, st = ldd.decompose(*d, 0.2, stats=True, engine=4)
    assert np.array_equal(centre.cpu().numpy(), want) and cut == want_cut
    k = 0.35 * n ** 0.5 * max(1.0, ci.size / (7 * n)) ** 0.25
    assert st["steps"] == 1 and abs(st["blocks"] - min(cus, max(32, k))) < 1.5
