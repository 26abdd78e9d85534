"""GPU parity of support queries on renumbered graphs: supports added up by
slices of the words with either load width, or edge by edge, and brought to the
caller's order.  Small graphs are renumbered by a flag, one by its own size.
Integer results, so the tolerance against the oracle is zero."""
import numpy as np
import pytest

import oracle
from graphgen.csr import from_edges

pytestmark = pytest.mark.gpu

LAYOUT = 0x20


def _graph(n, m, hubs, seed):
    # uniform edges, `hubs` vertices of a few hundred to 2,000 neighbours, and
    # isolated vertices
    rng = np.random.Generator(np.random.PCG64(seed))
    ids = rng.permutation(n)[: n - 40]
    us, vs = [ids[rng.integers(0, ids.size, m)]], [ids[rng.integers(0, ids.size, m)]]
    for i in range(hubs):
        us.append(np.full(2000 // (i + 1), ids[i]))
        vs.append(ids[rng.integers(0, ids.size, 2000 // (i + 1))])
    return from_edges(n, np.concatenate(us), np.concatenate(vs), name=f"graph({n},{m},{hubs})")


def _drop_edges(g, keep):
    src = np.repeat(np.arange(g.n), np.diff(g.row_ptr.astype(np.int64)))
    up = g.col_idx > src
    return from_edges(g.n, src[up][:keep], g.col_idx[up][:keep], name=f"{g.name}[:{keep}]")


@pytest.mark.parametrize("rest", [0, 1, 2, 3])  # edges beyond the last four that 16 lanes take
@pytest.mark.parametrize("n,m,hubs,h", [(32_768, 9000, 6, 2), (33_003, 40_000, 0, 2), (33_003, 6000, 4, 3)])
def test_renumbered_query_equals_oracle(n, m, hubs, h, rest):
    import paper_2411_06405_amd as ht
    g = _graph(n, m, hubs, seed=n + h)
    g = _drop_edges(g, g.m - (g.m - rest) % 4)
    assert g.m % 4 == rest
    print(f"[gpu] support layout n={g.n} m={g.m} h={h}", flush=True)
    want = oracle.h_support(g, h)
    for tune in ({}, {"word_bits": 64}, {"word_bits": 128}, {"edges_per_wave": 4}, {"edges_per_wave": 2, "word_bits": 128},
                 {"edges_per_wave": 8}, {"edges_per_wave": 16, "word_bits": 128}, {"edges_per_wave": 16},
                 {"dense_threshold": 1}, {"dense_threshold": 1 << 30}):
        got = ht.h_support_graph(g, h, tune=dict(tune, flags=LAYOUT))
        assert np.array_equal(got, want), tune
    assert np.array_equal(ht.h_support_graph(g, h), want)


@pytest.mark.parametrize("edges", [1, 3, 5])
def test_few_edges(edges):
    # fewer edges than one group takes; one word of the rows in use
    import paper_2411_06405_amd as ht
    g = from_edges(40_000, np.arange(edges) * 7 + 39_000, np.arange(edges) * 7 + 39_003, name=f"edges({edges})")
    g2 = from_edges(40_000, [5, 5, 39_999, 17], [39_999, 17, 17, 20_000], name="triangle and tail")
    for x in (g, g2):
        for bits in (64, 128):
            got = ht.h_support_graph(x, 2, tune={"word_bits": bits, "flags": LAYOUT})
            assert np.array_equal(got, oracle.h_support(x, 2)), (x.name, bits)


@pytest.mark.parametrize("bits", [0, 64, 128])
def test_query_renumbered_by_its_size_equals_oracle(bits):
    import paper_2411_06405_amd as ht
    g = _graph(100_000, 426_000, 5, seed=9)
    words = (g.n + 511) // 512 * 8
    assert g.m * words >= 600 << 20  # where queries renumber by themselves
    print(f"[gpu] support layout n={g.n} m={g.m} word_bits={bits}", flush=True)
    got = ht.h_support_graph(g, 2, tune={"word_bits": bits} if bits else None)
    assert np.array_equal(got, oracle.h_support(g, 2))
