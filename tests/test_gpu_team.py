"""GPU parity where rounds pass between the team kernel and the whole-chip round
kernels: steps below and above the team's limits, runs of whole-chip rounds,
and batches of fewer, as many and more graphs than there are XCDs and teams.
Integer results, so the tolerance against the oracle, or against rounds that
the host drives one by one, is zero."""
import numpy as np
import pytest

import oracle
from graphgen import concat
from graphgen.csr import from_edges
from graphgen.gen import chung_lu, erdos_renyi, rmat

pytestmark = pytest.mark.gpu

HOST_LOOP, COMPACT_EACH = 0x1, 0x10


@pytest.mark.parametrize("family,size,h", [
    ("er", 90, 3), ("er", 600, 1), ("er", 6000, 2),       # few rounds, large steps
    ("er", 12000, 2),                                     # changes to whole-chip rounds
    ("chung_lu", 9001, 2), ("chung_lu", 900, 3),          # many small rounds
    ("chung_lu", 20011, 1), ("rmat", 11, 2), ("rmat", 9, 3),
])
def test_decompose_equals_host_driven_rounds(family, size, h):
    import paper_2411_06405_amd as ht
    if family == "er":
        g = erdos_renyi(size, 14.0 / size, seed=size + h)
    elif family == "chung_lu":
        g = chung_lu(size, 10.0, 2.4, seed=size + h)
    else:
        g = rmat(size, 16, seed=size + h)
    print(f"[gpu] team {family} n={g.n} m={g.m} h={h}", flush=True)
    to, ro = ht.decompose_graph(g, h, tune={"flags": HOST_LOOP})
    for tune in (None, {"flags": COMPACT_EACH}, {"event_capacity": 96, "item_capacity": 96}):
        t, r = ht.decompose_graph(g, h, tune=tune)
        assert np.array_equal(t, to) and np.array_equal(r, ro), tune


@pytest.mark.parametrize("peeled", [2048, 4096, 4097])
def test_first_round_at_the_limit_of_a_team(peeled):
    # a matching of `peeled` edges peels in one round (4,096: a team's most),
    # then a few cliques in theirs
    import paper_2411_06405_amd as ht
    u = np.arange(peeled) * 2
    us, vs = [u], [u + 1]
    at = 2 * peeled
    for size in (3, 5, 9):
        a, b = np.triu_indices(size, 1)
        us.append(at + a)
        vs.append(at + b)
        at += size
    g = from_edges(at, np.concatenate(us), np.concatenate(vs), name=f"matching({peeled})")
    to, ro, _ = oracle.decompose(g, 2)
    t, r = ht.decompose_graph(g, 2)
    assert np.array_equal(t, to) and np.array_equal(r, ro)


@pytest.mark.parametrize("count", [2, 7, 8, 9, 33, 300])
def test_batch_of_teams_equals_oracle(count):
    import paper_2411_06405_amd as ht
    # every fifth graph is larger than the others
    gs = [erdos_renyi(40 if i % 5 else 260, 0.12 if i % 5 else 0.04, seed=i) for i in range(count)]
    hs = [1 + i % 3 for i in range(count)]
    print(f"[gpu] team batch count={count}", flush=True)
    ts, rs = ht.decompose_batch(concat(gs, hs))
    for g, h, t, r in zip(gs, hs, ts, rs):
        to, ro, _ = oracle.decompose(g, h)
        assert np.array_equal(t, to) and np.array_equal(r, ro), g.name


def test_batch_with_large_steps_equals_single_calls():
    import paper_2411_06405_amd as ht
    gs = [erdos_renyi(n, 14.0 / n, seed=n) for n in (2000, 7000, 14000)] + \
         [chung_lu(n, 10.0, 2.4, seed=n) for n in (300, 3000, 12001)]
    hs = [2, 2, 2, 3, 2, 2]
    ts, rs = ht.decompose_batch(concat(gs, hs))
    for g, h, t, r in zip(gs, hs, ts, rs):
        to, ro = ht.decompose_graph(g, h, tune={"flags": HOST_LOOP})
        assert np.array_equal(t, to) and np.array_equal(r, ro), g.name
