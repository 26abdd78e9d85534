"""GPU parity at h >= 3 on either side of the rule that cuts ball rows into work
items (8 words each, or 64 in rounds with many), where rounds, rows and lists
are just below and above its limits.  Integer results: the tolerance against
the oracle is zero."""
import numpy as np
import pytest

import oracle
from graphgen.csr import from_edges

pytestmark = pytest.mark.gpu


def _uniform(n, deg, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    k = int(n * deg / 2)
    return from_edges(n, rng.integers(0, n, k), rng.integers(0, n, k), name=f"uniform({n},{deg})")


@pytest.mark.parametrize("n,deg,h", [
    (500, 3.0, 4),      # one item a row either way
    (4100, 3.0, 3),     # 72 words: a last item of 8
    (12_000, 5.0, 3),   # rounds of up to 1,700 edges
    (32_768, 2.2, 3),   # 512 words, the longest rows cut by 8
    (32_769, 2.2, 3),   # the shortest never cut so
])
def test_either_cut_equals_oracle(n, deg, h):
    import paper_2411_06405_amd as ht
    g = _uniform(n, deg, seed=n + h)
    print(f"[gpu] word items n={g.n} m={g.m} h={h}", flush=True)
    to, ro, _ = oracle.decompose(g, h)
    # a list that level jumps by 8 words could overflow; host-driven rounds;
    # steps re-run in windows
    for tune in (None, {"item_capacity": 4 * g.m}, {"flags": 0x1}, {"item_capacity": 2048, "event_capacity": 2048}):
        t, r = ht.decompose_graph(g, h, tune=tune)
        assert np.array_equal(t, to) and np.array_equal(r, ro), tune


def test_large_rounds_are_cut_into_fewer_items():
    import paper_2411_06405_amd as ht
    g = _uniform(12_000, 5.0, seed=2)
    ht.decompose_graph(g, 3, tune={"flags": 0x2})
    st = ht.last_stats()["work"]
    words = (g.n + 511) // 512 * 8
    # by 8 words alone every edge but the last round's has two rows of
    # words / 8 items, and its items of level 2 besides
    print(f"[gpu] word items {st['level_items']} of {2 * g.m * words // 8}", flush=True)
    assert st["level_items"] < 2 * g.m * words // 8
