"""GPU: the launch engine's grid by the size of the graph.  Every size of grid has launch graphs of its own, built
by the first call that needs it and kept: there are few of them, whatever sizes a program passes."""
import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ldd():
    import torch
    assert torch.cuda.is_available()
    import paper_1307_3692_amd as m
    m.lib()
    return m


def test_few_grid_sizes(ldd):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    seen = []
    for n in (500, 17_000, 33_000, 40_001, 46_700, 60_000, 65_536, 80_000, 95_000, 110_000, 131_072, 150_000):
        rp, ci = inputs.er(n, 9.0, n)
        s = inputs.make_shifts(n, 0.2, 3)
        want, _, want_cut = oracle.decompose(rp, ci, s)
        d = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (rp, ci, s)]
        centre, cut, st = ldd.decompose(*d, 0.2, stats=True, engine=2)
        print(f"n {n} blocks {st['blocks']}", flush=True)
        assert np.array_equal(centre.cpu().numpy(), want) and cut == want_cut
        seen.append(st["blocks"])
    assert seen == sorted(seen) and seen[0] >= 128 and seen[-1] == 2 * cus
    assert len(set(seen)) <= 3
