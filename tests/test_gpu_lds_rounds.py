"""GPU: the workgroup engine's rounds on frontiers in LDS, at the sizes where they change form, bit for bit
against the CPU oracle: the claims' table and bits by vertex count, rows by degree, pulled rounds, frontiers
past the LDS, and a team's steps of several rounds (with members whose LDS overflows inside a step)."""
import numpy as np
import pytest

import inputs
import oracle
from graphs import S, disjoint_union, path, star

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ldd():
    import torch
    assert torch.cuda.is_available()
    import paper_1307_3692_amd as m
    m.lib()
    return m


def check(ldd, rp, ci, s, *modes):
    import torch
    want_c, _, want_cut = oracle.decompose(rp, ci, s)
    d = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (rp, ci, s)]
    for mode in modes:
        print(f"n {rp.size - 1} arcs {ci.size} {mode}", flush=True)
        centre, cut = ldd.decompose(*d, 0.1, **mode)
        got = centre.cpu().numpy()
        assert np.array_equal(got, want_c), (mode, np.count_nonzero(got != want_c))
        assert cut == want_cut, mode


# centres of 16 bits in LDS up to 2^16 vertices, twice the table up to 2^17, claims in LDS up to 2^18
@pytest.mark.parametrize("n", [1 << 16, (1 << 16) + 1, 1 << 17, (1 << 17) + 1, (1 << 18) - 1, 1 << 18, (1 << 18) + 1])
def test_vertex_counts(ldd, n):
    """Erdos-Renyi: the frontier outgrows the LDS within a few rounds and the last ones are pulled."""
    rp, ci = inputs.er(n, 6.0, n)
    check(ldd, rp, ci, inputs.make_shifts(n, 0.1, 3), dict(engine=3), dict(engine=3, tail_vertices=1))


@pytest.mark.parametrize("beta", [0.03, 0.3])
def test_many_rounds_alone(ldd, beta):
    rp, ci = inputs.rgg(90_000, 7.0, 11)
    check(ldd, rp, ci, inputs.make_shifts(90_000, beta, 4), dict(engine=3), dict(engine=3, tail_vertices=-1))


# a row is walked with others up to 32 arcs, by its wave up to 4096, by the workgroup above, of which
# 32 are listed per round and the rest walked by their waves
@pytest.mark.parametrize("leaves,hubs", [(31, 50), (32, 50), (33, 50), (4096, 3), (4097, 3), (4200, 40)])
def test_row_lengths(ldd, leaves, hubs):
    g = disjoint_union(*[star(leaves + 1) for _ in range(hubs)], path(500))
    rp, ci = g
    n = rp.size - 1
    rng = np.random.default_rng(leaves)
    s = rng.integers(0, 3 * S, n).astype(np.int64)
    s[::leaves + 1] += 2 * S  # most hubs wake together
    check(ldd, rp, ci, s, dict(engine=3), dict(engine=4), dict(engine=4, blocks=3))


def tree(arity, depth):
    n = (arity ** (depth + 1) - 1) // (arity - 1)
    v = np.arange(1, n)
    return n, (v - 1) // arity, v


@pytest.mark.parametrize("tail", [0, -1])
def test_frontier_explodes_inside_a_step(ldd, tail):
    """A path (small steady frontiers: several rounds per step of a team) into the root of a tree of arity 9:
    one member reaches more vertices within a step than its LDS holds.  Paths hang from the tree's
    first leaves, so that rounds go on after it, and every tenth vertex may wake on its own."""
    n, src, dst = tree(9, 5)
    length, tails = 120, 60
    es, ed = [src], [dst]
    base = n
    es.append(np.concatenate([[0], np.arange(base, base + length - 1)]))
    ed.append(np.arange(base, base + length))
    base += length
    first_leaf = n - 9 ** 5
    for k in range(40):
        es.append(np.concatenate([[first_leaf + 7 * k], np.arange(base, base + tails - 1)]))
        ed.append(np.arange(base, base + tails))
        base += tails
    rp, ci = inputs.from_edges(base, np.concatenate(es), np.concatenate(ed))
    rng = np.random.default_rng(5)
    s = rng.integers(0, 5 * S, base).astype(np.int64)
    s[::10] += rng.integers(0, 60 * S, s[::10].size)
    s[n + length - 1] = 260 * S  # the path's far end starts the search
    check(ldd, rp, ci, s, dict(engine=4, tail_vertices=tail), dict(engine=4, blocks=5, tail_vertices=tail),
          dict(engine=4, blocks=40, tail_vertices=tail), dict(engine=3, tail_vertices=tail))


# one graph held whole in LDS: four arcs of a vertex are in registers, eight, or eight and the rest read
# from LDS, and above 64 a wave has the row; six vertices of a thread are, further ones are not; and one size past the LDS
@pytest.mark.parametrize("degree", [4, 5, 8, 9, 64, 65, 300])
@pytest.mark.parametrize("n", [301, 1023, 1025, 6144, 6145, 7300])
def test_graph_in_lds(ldd, n, degree):
    """A ring with one vertex of the given degree and a few of four."""
    src = np.arange(n)
    es, ed = [src, np.arange(0, n - n % 7, 7)], [(src + 1) % n, (np.arange(0, n - n % 7, 7) + n // 2) % n]
    es.append(np.full(degree - 2, 5))
    ed.append(5 + 2 * np.arange(1, degree - 1) % n)
    rp, ci = inputs.from_edges(n, np.concatenate(es), np.concatenate(ed) % n)
    check(ldd, rp, ci, inputs.make_shifts(n, 0.02, n + degree), dict(engine=3), dict(engine=3, tail_vertices=-1))


@pytest.mark.parametrize("n,degree,beta", [(20_000, 5.0, 0.2), (90_000, 6.5, 0.08), (150_000, 3.2, 0.2)])
def test_team_tail_from_a_large_frontier(ldd, n, degree, beta):
    """The last rounds' frontier outweighs the vertices left: the tail takes over from it."""
    rp, ci = inputs.er(n, degree, n)
    check(ldd, rp, ci, inputs.make_shifts(n, beta, 6), dict(engine=4), dict(engine=4, blocks=7), dict(engine=4, blocks=256),
          dict(engine=4, tail_vertices=4), dict(engine=4, tail_vertices=-1))


@pytest.mark.parametrize("scale,edges", [(8, 16), (10, 16), (11, 8), (11, 16), (11, 18), (12, 6), (12, 8)])
def test_small_dense_graphs(ldd, scale, edges):
    """Skewed graphs on both sides of the automatic choice's line, and of the size that is held whole in LDS."""
    rp, ci = inputs.rmat(scale, edges, seed=scale + edges)
    check(ldd, rp, ci, inputs.make_shifts(rp.size - 1, 0.1, 8), dict(), dict(engine=3), dict(direction=2))
