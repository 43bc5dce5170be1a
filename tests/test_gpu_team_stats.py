"""GPU: a team's count of rounds stays within the bound that the shifts give, also where its last step of several
rounds reaches past it."""
import numpy as np
import pytest

import inputs
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
