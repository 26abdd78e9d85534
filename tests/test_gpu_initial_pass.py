"""GPU parity of the initial supports and balls where a frontier holds rows of
every kind (16 lanes, a wavefront, an ORed row; more of them than one pass
takes), and where the supports are added up by slices of the words.  Integer
results, so the tolerance against the oracle is zero."""
import numpy as np
import pytest

import oracle
from graphgen.csr import from_edges

pytestmark = pytest.mark.gpu


def _hubs(n, seed):
    # hubs of 127 to 2,500 neighbours, two of them adjacent to all the others
    rng = np.random.Generator(np.random.PCG64(seed))
    ids = rng.permutation(n)[: n - 20]
    us, vs = [], []
    for i, deg in enumerate((2500, 1100, 130, 129, 128, 127)):
        us.append(np.full(deg, ids[i]))
        vs.append(rng.choice(ids[6:3500], deg, replace=False))
    for hub in ids[:2]:
        us.append(np.full(6, hub))
        vs.append(ids[:6])
    us.append(ids[rng.integers(0, 3500, 4000)])
    vs.append(ids[rng.integers(0, 3500, 4000)])
    return from_edges(n, np.concatenate(us), np.concatenate(vs), name=f"hubs({n},{seed})")


@pytest.mark.parametrize("n", [3600, 32768, 33003])
@pytest.mark.parametrize("h", [2, 3])
def test_supports_equal_oracle(n, h):
    import paper_2411_06405_amd as ht
    g = _hubs(n, n + h)
    want = oracle.h_support(g, h)
    print(f"[gpu] initial pass n={n} m={g.m} h={h}", flush=True)
    for tune in (None, {"word_bits": 64}, {"word_bits": 128, "edges_per_wave": 4}, {"dense_threshold": 1},
                 {"dense_threshold": 1 << 30}):
        assert np.array_equal(ht.h_support_graph(g, h, **({"tune": tune} if tune else {})), want), tune
