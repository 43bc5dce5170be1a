"""GPU: the widest entries of a team member's table of offers already made: with 2^26 vertices an offer's distance from
the step's first label and its vertex fill 64 bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

S = 1 << 20


@pytest.fixture(scope="module")
def ldd():
    import torch
    assert torch.cuda.is_available()
    import paper_1307_3692_amd as m
    m.lib()
    return m


def test_offers_whose_bits_are_all_ones(ldd):
    """The last vertex is the centre of everything: 200 paths leave it, each with two branches from distance 25 on.
    A team of four takes distances 18 to 33 in one step, on more rows than it sends offers for unasked; those of its
    last round have every bit set in centre, fraction and round, and go to vertices of the highest ids.  All other
    vertices have no arcs, so the answer is known without an oracle."""
    import torch
    n, strands, split, length, last_step = 1 << 26, 200, 25, 36, 33
    rng = np.random.default_rng(1)
    layers = [np.array([n - 1])]
    top, low = n - 1, 1000
    for d in range(1, length + 1):
        width = strands if d < split else 2 * strands
        if d == last_step:
            layers.append(top - 1 - rng.permutation(width))  # among the last 4096 ids
        else:
            layers.append(low + np.arange(width))
            low += 2 * width
    src, dst = [], []
    for a, b in zip(layers[:-1], layers[1:]):
        src.append(np.repeat(a, b.size // a.size) if a.size < b.size else a)
        dst.append(b)
    src, dst = np.concatenate(src), np.concatenate(dst)
    key = np.sort(np.concatenate([src * n + dst, dst * n + src]))
    rows, cols = key // n, (key % n).astype(np.int32)
    deg = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    deg.index_add_(0, torch.from_numpy(rows + 1).cuda(), torch.ones(rows.size, dtype=torch.int32, device="cuda"))
    rp = torch.cumsum(deg, 0, dtype=torch.int32)
    rounds = 200
    s = torch.zeros(n, dtype=torch.int64, device="cuda")
    s[0] = rounds * S                 # Delta (a vertex without arcs)
    s[n - 1] = rounds * S - (S - 1)   # round 0, fraction all ones
    print(f"n {n} arcs {cols.size}", flush=True)
    centre, cut, st = ldd.decompose(rp, torch.from_numpy(cols).cuda(), s, 0.1, engine=4, blocks=4, tail_vertices=-1,
                                    stats=True)
    assert st["steps"] == 1 and st["blocks"] == 4
    want = torch.arange(n, dtype=torch.int32, device="cuda")
    for layer in layers:
        want[torch.from_numpy(layer).cuda()] = n - 1
    assert torch.equal(centre, want), int((centre != want).sum())
    assert cut == 0
