"""GPU parity where graphs are renumbered by degree inside the library (32,768
vertices and more): rows of every kind the renumbering treats apart (below, at
and above 64 slots, one long row, isolated vertices at both ends of the id
range), just below and above the size where it starts.  Integer results, so the
tolerance against the oracle is zero."""
import numpy as np
import pytest

import oracle
from graphgen import concat
from graphgen.csr import from_edges

pytestmark = pytest.mark.gpu


def _graph(n, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    ids = rng.permutation(n)[: n - 50]  # some vertices stay isolated
    at = 0
    us, vs = [], []
    hubs = ids[:5]
    for hub, deg in zip(hubs, (63, 64, 65, 130, 700)):
        leaves = ids[10 + at: 10 + at + deg]
        at += deg // 2  # stars overlap
        us.append(np.full(deg, hub))
        vs.append(leaves)
    c = ids[5:17]
    a, b = np.triu_indices(c.size, 1)
    us.append(c[a])
    vs.append(c[b])
    us.append(hubs[:-1])
    vs.append(hubs[1:])
    k = 900
    us.append(ids[rng.integers(0, 1500, k)])
    vs.append(ids[rng.integers(0, 1500, k)])
    return from_edges(n, np.concatenate(us), np.concatenate(vs), name=f"stars({n},{seed})")


@pytest.mark.parametrize("n", [32767, 32768, 33001])
@pytest.mark.parametrize("h", [1, 2, 3])
def test_renumbered_graph_equals_oracle(n, h):
    import paper_2411_06405_amd as ht
    g = _graph(n, n + h)
    print(f"[gpu] renumber n={n} m={g.m} h={h}", flush=True)
    to, ro, _ = oracle.decompose(g, h)
    t, r = ht.decompose_graph(g, h)
    assert np.array_equal(t, to) and np.array_equal(r, ro)
    t, _ = ht.decompose_graph(g, h, with_rounds=False)
    assert np.array_equal(t, to)
    assert np.array_equal(ht.h_support_graph(g, h), oracle.h_support(g, h))
    # lists too short for the larger rounds, and rows compacted every round
    for tune in ({"event_capacity": 64, "item_capacity": 64}, {"flags": 0x10}, {"flags": 0x1}):
        t, r = ht.decompose_graph(g, h, tune=tune)
        assert np.array_equal(t, to) and np.array_equal(r, ro), tune


def test_renumbered_graphs_in_a_batch():
    import paper_2411_06405_amd as ht
    gs = [_graph(32768, 1), _graph(2000, 2), _graph(33001, 3)]
    hs = [2, 3, 3]
    ts, rs = ht.decompose_batch(concat(gs, hs))
    for g, h, t, r in zip(gs, hs, ts, rs):
        to, ro, _ = oracle.decompose(g, h)
        assert np.array_equal(t, to) and np.array_equal(r, ro), g.name
