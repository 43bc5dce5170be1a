"""GPU: which engine ends a team's call.  A team whose members' LDS or shares overflow inside a step goes on as a
team; one whose shared queue would get more entries than there are vertices (many members lower the same vertices in the
last round of a step) leaves the graph to the launch engine.  Statistics tell them apart: a team's call is one
step and has no frontier statistics."""
import numpy as np
import pytest

import inputs
import oracle
from graphs import S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ldd():
    import torch
    assert torch.cuda.is_available()
    import paper_1307_3692_amd as m
    m.lib()
    return m


def to_dev(*arrays):
    import torch
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


def hubs_behind_paths(strands, length, leaves, seed):
    """Paths of equal length into hubs that share all their leaves: every hub is reached in the same round, and offers
    the leaves another fraction."""
    rng = np.random.default_rng(seed)
    ids = leaves + np.arange(strands * length).reshape(strands, length)
    src = np.concatenate([ids[:, :-1].ravel(), np.repeat(ids[:, -1], leaves)])
    dst = np.concatenate([ids[:, 1:].ravel(), np.tile(np.arange(leaves), strands)])
    n = leaves + strands * length
    rp, ci = inputs.from_edges(n, src, dst)
    s = rng.integers(0, S, n).astype(np.int64)
    s[ids[:, 0]] = 400 * S - 1 - rng.permutation(S - 1)[:strands]
    return rp, ci, s


def tree_behind_a_path(arity, depth, length, chain):
    """A path into the root of a tree, and a path from its last leaf."""
    n = (arity ** (depth + 1) - 1) // (arity - 1)
    v = np.arange(1, n)
    a, b = n + np.arange(length), n + length + np.arange(chain)
    src = np.concatenate([(v - 1) // arity, [0], a[:-1], [n - 1], b[:-1]])
    dst = np.concatenate([v, a[:1], a[1:], b[:1], b[1:]])
    rp, ci = inputs.from_edges(n + length + chain, src, dst)
    s = np.random.default_rng(depth).integers(0, 5 * S, n + length + chain).astype(np.int64)
    s[n + length - 1] = 300 * S
    return rp, ci, s


@pytest.mark.parametrize("blocks", [5, 40])
@pytest.mark.parametrize("graph", ["tree", "er"])
def test_team_keeps_the_graph(ldd, graph, blocks):
    if graph == "tree":  # 59049 leaves in one round, reached by few members inside a step
        rp, ci, s = tree_behind_a_path(9, 5, 120, 100)
    else:
        rp, ci = inputs.er(60_000, 6.0, 3)
        s = inputs.make_shifts(60_000, 0.1, 4)
    want, _, want_cut = oracle.decompose(rp, ci, s)
    print(f"{graph} blocks {blocks}", flush=True)
    centre, cut, st = ldd.decompose(*to_dev(rp, ci, s), 0.1, stats=True, engine=4, blocks=blocks)
    assert st["steps"] == 1 and st["blocks"] == blocks and st["max_frontier"] == 0
    assert np.array_equal(centre.cpu().numpy(), want) and cut == want_cut


@pytest.mark.parametrize("n,degree", [(1024, 30.0), (1500, 50.0), (1500, 100.0), (4096, 50.0)])
@pytest.mark.parametrize("beta", [0.1, 0.4, 1.0])
def test_team_keeps_dense_graphs(ldd, n, degree, beta):
    """The first waves of a dense graph reach most of it within two rounds: in steps of several rounds each member
    would queue the same vertices."""
    rp, ci = inputs.er(n, degree, n)
    s = inputs.make_shifts(n, beta, 4)
    want, _, want_cut = oracle.decompose(rp, ci, s)
    d = to_dev(rp, ci, s)
    for blocks in (2, 4, 16):
        print(f"n {n} degree {degree} beta {beta} blocks {blocks}", flush=True)
        centre, cut, st = ldd.decompose(*d, beta, stats=True, engine=4, blocks=blocks)
        assert st["steps"] == 1 and st["blocks"] == blocks
        assert np.array_equal(centre.cpu().numpy(), want) and cut == want_cut


@pytest.mark.parametrize("leaves", [1023, 1024, 1025, 5000])
@pytest.mark.parametrize("blocks", [3, 40])
def test_one_round_per_step_beside_a_long_row(ldd, leaves, blocks):
    """Paths, and a star of the given number of arcs: above 1024 a team takes one round per step, so that it counts the
    rounds that one workgroup counts; up to there it counts whole steps."""
    n, strands, length = 60_000 + leaves + 1, 200, 300
    ids = np.arange(strands * length).reshape(strands, length)
    hub = strands * length
    src = np.concatenate([ids[:, :-1].ravel(), np.full(leaves, hub)])
    dst = np.concatenate([ids[:, 1:].ravel(), hub + 1 + np.arange(leaves)])
    rp, ci = inputs.from_edges(n, src, dst)
    s = np.random.default_rng(1).integers(0, S, n).astype(np.int64)
    s[ids[:, 0]] += 320 * S
    want, _, want_cut = oracle.decompose(rp, ci, s)
    d = to_dev(rp, ci, s)
    print(f"leaves {leaves} blocks {blocks}", flush=True)
    _, _, alone = ldd.decompose(*d, 0.1, stats=True, engine=3, tail_vertices=-1)
    centre, cut, st = ldd.decompose(*d, 0.1, stats=True, engine=4, blocks=blocks, tail_vertices=-1)
    assert st["steps"] == 1 and st["blocks"] == blocks
    assert np.array_equal(centre.cpu().numpy(), want) and cut == want_cut
    assert (st["rounds"] == alone["rounds"]) == (leaves > 1024)


@pytest.mark.parametrize("strands", [16, 64])
@pytest.mark.parametrize("tail", [0, -1])
def test_queue_overflow_goes_to_the_launch_engine(ldd, strands, tail):
    """Lengths on both sides of the end of a step.  How often a leaf is lowered depends on timing, so that not every
    length has to overflow; every result is exact."""
    left = 0
    for length in (14, 15, 16, 17, 31):
        rp, ci, s = hubs_behind_paths(strands, length, 1000, length)
        want, _, want_cut = oracle.decompose(rp, ci, s)
        d = to_dev(rp, ci, s)
        centre, cut, st = ldd.decompose(*d, 0.1, stats=True, engine=4, blocks=8, tail_vertices=tail)
        print(f"strands {strands} length {length} tail {tail}: steps {st['steps']}", flush=True)
        assert np.array_equal(centre.cpu().numpy(), want) and cut == want_cut
        assert (st["steps"] > 1) == (st["max_frontier"] > 0)
        left += st["steps"] > 1
        centre, cut = ldd.decompose(*d, 0.1, engine=4, blocks=8, tail_vertices=tail)
        assert np.array_equal(centre.cpu().numpy(), want) and cut == want_cut
    assert left


def test_queue_overflow_in_a_batch(ldd):
    gs = [hubs_behind_paths(16, 16, 1000, 1), (*inputs.er(9000, 6.0, 2), inputs.make_shifts(9000, 0.1, 2)),
          hubs_behind_paths(16, 15, 900, 3), (*inputs.grid2d(70, 60), inputs.make_shifts(4200, 0.05, 4))]
    want = [oracle.decompose(*g) for g in gs]
    vo = np.cumsum([0] + [g[0].size - 1 for g in gs])
    ao = np.cumsum([0] + [g[1].size for g in gs])
    d = to_dev(*(np.concatenate([g[i] for g in gs]) for i in range(3)))
    for team_arcs in (4000, 0, -1):
        print(f"team_arcs {team_arcs}", flush=True)
        centre, cuts = ldd.decompose_batch(vo, ao, *d, batch_mode=3, team_arcs=team_arcs)
        got = centre.cpu().numpy()
        for i, (c, _, cut) in enumerate(want):
            assert np.array_equal(got[vo[i]:vo[i + 1]], c) and cuts[i] == cut, (team_arcs, i)
