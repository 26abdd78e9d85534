"""Sessions driven launch by launch: what one counted launch may do, and that
requests end the same whatever the steps."""
import numpy as np
import pytest

import oracle
from graphgen.gen import chung_lu, erdos_renyi

pytestmark = pytest.mark.gpu

ROUNDS = 128  # most of a slot in one counted launch


@pytest.mark.parametrize("slots,max_h", [(1, 1), (1, 2), (3, 2), (12, 3)])
def test_a_counted_launch_is_a_bounded_number_of_rounds(slots, max_h):
    import paper_2411_06405_amd as ht
    h = max_h
    # long decompositions and a short one, together or one after the other
    gs = [chung_lu(n, 10.0, 2.3, seed=n) for n in {1: (60_011, 40_000), 2: (1501, 2400), 3: (700, 900)}[h]]
    gs.append(erdos_renyi(300, 0.03, seed=1))
    s = ht.Session(4 << 30, max_slots=slots, max_h=max_h)
    tickets = [s.submit(g.row_ptr, g.col_idx, g.n, h) for g in gs]
    done_at, calls = {}, 0
    while len(done_at) < len(gs):
        s.progress(max_graph_launches=1)
        calls += 1
        for k in tickets:
            if k not in done_at and s.poll(k):
                done_at[k] = calls
        assert calls < 4000
    before = 0
    for g, k in zip(gs, tickets):
        t, r = s.result(k)
        to, ro = ht.decompose_graph(g, h)
        assert np.array_equal(t, to) and np.array_equal(r, ro)
        rounds = int(r.max()) + 1
        launches = done_at[k] - (before if slots == 1 else 0)
        print(f"[gpu] {g.name} rounds={rounds} launches={launches}", flush=True)
        assert launches * (ROUNDS + 1) >= rounds
        before = done_at[k]
    to, ro, _ = oracle.decompose(gs[-1], h)
    assert np.array_equal(t, to) and np.array_equal(r, ro)
    s.close()


def test_short_requests_do_not_pay_for_long_graphs():
    # one slot, h = 1, requests of a few rounds each: about what the same
    # decompositions take one by one (launches sized by the session's age
    # instead of the request's took more than three times that)
    import time

    import torch
    import paper_2411_06405_amd as ht
    gs = [erdos_renyi(300 + 10 * i, 10.0 / (300 + 10 * i), seed=i) for i in range(30)]
    dev = [(torch.from_numpy(g.row_ptr.view(np.int32)).cuda(), torch.from_numpy(g.col_idx.view(np.int32)).cuda(), g.n)
           for g in gs]
    ws = ht.alloc_workspace(gs[-1].n, max(g.m for g in gs), 1)
    s = ht.Session(1 << 30, max_slots=1, max_h=1)

    def served():
        ks = [s.submit(*d, 1) for d in dev]
        t0 = time.perf_counter()
        s.progress()
        took = time.perf_counter() - t0
        return took, [s.result(k) for k in ks]

    def alone():
        t0 = time.perf_counter()
        out = [ht.decompose(*d, 1, workspace=ws) for d in dev]
        torch.cuda.synchronize()
        return time.perf_counter() - t0, [(ht.to_numpy_u32(t), ht.to_numpy_u32(r)) for t, r in out]
    a, b = [served() for _ in range(6)], [alone() for _ in range(6)]
    for (t, r), (to, ro) in zip(a[-1][1], b[-1][1]):
        assert np.array_equal(t, to) and np.array_equal(r, ro)
    fast, ref = min(x[0] for x in a), min(x[0] for x in b)
    print(f"[gpu] served {fast * 1e3:.2f} ms, one by one {ref * 1e3:.2f} ms", flush=True)
    assert fast < 2 * ref
    s.close()
