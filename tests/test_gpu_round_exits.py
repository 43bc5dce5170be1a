"""GPU: how the workgroup engine's rounds end on bad column ids.  The call is refused, whichever phase reads the
column, and the graphs that the same workgroup decomposes after the bad one have the oracle's centres."""
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


def spoil(rp, ci, s, where):
    """One column out of range, in a row that the rounds walk first (the vertex of the largest shift), in every
    hundredth row (rounds, pulls and tail), or in the rows reached last (read by the output alone when their
    round has ended the search)."""
    ci = ci.copy()
    deg = np.diff(rp)
    if where == "first":
        rows = np.array([int(np.argmax(np.where(deg > 0, s, -1)))])
    elif where == "many":
        rows = np.flatnonzero(deg > 0)[::100]
    else:
        _, dist, _ = oracle.decompose(rp, ci, s)
        rows = np.array([int(np.argmax(np.where(deg > 0, dist, -1)))])
    ci[rp[rows]] = np.resize(np.array([rp.size - 1, -1, 2**31 - 1], np.int64), rows.size).astype(np.int32)
    return ci


# claims and pulls with centres in LDS or not, more vertices than the claims take, and a sparse graph of many rounds
@pytest.mark.parametrize("kind,n", [("er", 20_000), ("er", 90_000), ("er", 300_000), ("rgg", 30_000)])
@pytest.mark.parametrize("where", ["first", "many", "last"])
@pytest.mark.parametrize("tail", [0, 1, -1])
def test_one_bad_graph_of_a_batch(ldd, kind, n, where, tail):
    import torch
    gs = [inputs.er(n, 6.0, 1) if kind == "er" else inputs.rgg(n, 6.0, 1)]
    gs += [inputs.er(6000, 6.0, 2), inputs.grid2d(90, 50), inputs.rgg(2500, 6.0, 3)]
    ss = [inputs.make_shifts(rp.size - 1, 0.1, 10 + i) for i, (rp, _) in enumerate(gs)]
    want = [oracle.decompose(rp, ci, s)[0] for (rp, ci), s in zip(gs, ss)]
    cols = [ci for _, ci in gs]
    cols[0] = spoil(*gs[0], ss[0], where)
    vo = np.cumsum([0] + [rp.size - 1 for rp, _ in gs])
    ao = np.cumsum([0] + [ci.size for ci in cols])
    d = [torch.from_numpy(np.ascontiguousarray(a)).cuda()
         for a in (np.concatenate([rp for rp, _ in gs]), np.concatenate(cols), np.concatenate(ss))]
    centre = torch.full((int(vo[-1]),), -7, dtype=torch.int32, device="cuda")
    print(f"{kind} {n} {where} tail {tail}", flush=True)
    with pytest.raises(ldd.LddError) as e:  # one workgroup takes the four graphs, the bad one (the largest) first
        ldd.decompose_batch(vo, ao, *d, centre=centre, blocks=1, tail_vertices=tail)
    assert e.value.status == ldd.ERR_INVALID_ARG
    got = centre.cpu().numpy()
    for i in range(1, 4):
        assert np.array_equal(got[vo[i]:vo[i + 1]], want[i]), i


@pytest.mark.parametrize("where", ["first", "many", "last"])
@pytest.mark.parametrize("tail", [0, 1, -1])
@pytest.mark.parametrize("mode", [dict(engine=3), dict(engine=4, blocks=3), dict(engine=4, blocks=40)])
def test_bad_column_of_one_graph(ldd, where, tail, mode):
    import torch
    for rp, ci in (inputs.rgg(40_000, 6.0, 4), inputs.er(40_000, 6.0, 5)):
        s = inputs.make_shifts(rp.size - 1, 0.05, 6)
        want, _, want_cut = oracle.decompose(rp, ci, s)
        r, c, b, f = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (rp, ci, spoil(rp, ci, s, where), s))
        print(f"{where} tail {tail} {mode}", flush=True)
        with pytest.raises(ldd.LddError) as e:
            ldd.decompose(r, b, f, 0.05, tail_vertices=tail, **mode)
        assert e.value.status == ldd.ERR_INVALID_ARG
        centre, cut = ldd.decompose(r, c, f, 0.05, tail_vertices=tail, **mode)  # the next call is not disturbed
        assert np.array_equal(centre.cpu().numpy(), want) and cut == want_cut
