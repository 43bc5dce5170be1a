"""GPU: a team's members wait for the one that has a row of millions of arcs, in the rounds and in the output."""
import numpy as np
import pytest

import inputs

pytestmark = pytest.mark.gpu

S = 1 << 20


@pytest.fixture(scope="module")
def ldd():
    import torch
    assert torch.cuda.is_available()
    import paper_1307_3692_amd as m
    m.lib()
    return m


def star(n, hub):
    """(row_ptr, col_idx) of a star of n vertices whose centre is the given vertex, on the GPU."""
    import torch
    deg = torch.ones(n + 1, dtype=torch.int64, device="cuda")
    deg[0] = 0
    deg[hub + 1] = n - 1
    ids = torch.arange(n, dtype=torch.int32, device="cuda")
    leaves = ids[ids != hub]
    up = torch.full((n - 1,), hub, dtype=torch.int32, device="cuda")
    return torch.cumsum(deg, 0).to(torch.int32), torch.cat((up[:hub], leaves, up[hub:]))


@pytest.mark.parametrize("n", [5000, 6_000_000])
def test_star(ldd, n):
    """The hub takes all leaves but those whose own label is better by more than one unit: a quarter of them."""
    import torch
    hub = n // 3
    rp, ci = star(n, hub)
    s = torch.zeros(n, dtype=torch.int64, device="cuda")
    s[hub] = 2 * S
    s[::4] = 2 * S + 1  # (dist 0 - (2 S + 1)) against dist 1 - 2 S of the hub's label
    s[hub] = 2 * S + 7
    want = torch.full((n,), hub, dtype=torch.int32, device="cuda")
    own = torch.arange(n, dtype=torch.int32, device="cuda")
    want[::4] = own[::4]
    want[hub] = hub
    leaves_cut = int((want != hub).sum())
    grp, gci = inputs.grid2d(60, 50)
    gs = torch.from_numpy(inputs.make_shifts(3000, 0.1, 1)).cuda()
    alone, alone_cut = ldd.decompose(torch.from_numpy(grp).cuda(), torch.from_numpy(gci).cuda(), gs, 0.1, engine=2)
    print(f"star {n}", flush=True)
    centre, cut = ldd.decompose(rp, ci, s, 0.1, engine=4, blocks=16)
    assert torch.equal(centre, want) and cut == leaves_cut
    vo, ao = [0, n, n + 3000], [0, ci.numel(), ci.numel() + gci.size]
    centre, cuts = ldd.decompose_batch(vo, ao, torch.cat((rp, torch.from_numpy(grp).cuda())),
                                       torch.cat((ci, torch.from_numpy(gci).cuda())), torch.cat((s, gs)), team_arcs=1024)
    assert torch.equal(centre[:n], want) and torch.equal(centre[n:], alone)
    assert cuts == [leaves_cut, alone_cut]


def test_star_whose_hub_is_left_to_the_tail(ldd):
    """With tail_vertices = 1 the label-correcting tail may start after the first round, with the hub unreached: its
    seed is one thread's."""
    import torch
    n, hub = 6_000_000, 2_000_000
    rp, ci = star(n, hub)
    s = torch.zeros(n, dtype=torch.int64, device="cuda")
    s[5] = 40 * S  # a leaf: the hub is one round from it, the other leaves two
    print(f"star {n}", flush=True)
    centre, cut = ldd.decompose(rp, ci, s, 0.1, engine=4, blocks=16, tail_vertices=1)
    assert bool((centre == 5).all()) and cut == 0
