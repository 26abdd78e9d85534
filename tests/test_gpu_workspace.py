"""GPU parity in the smallest workspace each entry point accepts, where a graph
that is renumbered with more room keeps the caller's order.  Integer results,
so the tolerance against the oracle is zero."""
import numpy as np
import pytest

import oracle
from graphgen import concat
from graphgen.csr import from_edges

pytestmark = pytest.mark.gpu

WORKSPACE = -3


def _graph(n, m, seed):
    # uniform, with a few hubs
    rng = np.random.Generator(np.random.PCG64(seed))
    u, v = rng.integers(0, n, m), rng.integers(0, n, m)
    u[: m // 200] = rng.integers(0, 3, m // 200)
    return from_edges(n, u, v, name=f"graph({n},{m})")


def _smallest(call, top):
    """Fewest bytes `call` accepts, no more than `top` (a refused call does no work)."""
    lo, hi = 0, top
    assert call(hi) == 0
    while hi - lo > 4096:
        mid = (lo + hi) // 2
        rc = call(mid)
        assert rc in (0, WORKSPACE)
        lo, hi = (lo, mid) if rc == 0 else (mid, hi)
    return hi


def _on(a):
    import torch
    return torch.from_numpy(a.view(np.int32)).cuda()


def test_support_query_in_its_smallest_workspace():
    import torch
    import paper_2411_06405_amd as ht
    g, h = _graph(100_000, 430_000, 3), 2
    rp, ci = _on(g.row_ptr), _on(g.col_idx)
    ws = torch.empty(ht.workspace_bytes(g.n, g.m, h), dtype=torch.uint8, device="cuda")
    out = torch.empty(g.m, dtype=torch.int32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream

    def call(b):
        return ht.lib.hoTrussHSupport(rp.data_ptr(), ci.data_ptr(), g.n, g.m, h, out.data_ptr(), ws.data_ptr(), b,
                                      None, stream)
    b = _smallest(call, ws.numel())
    want = oracle.h_support(g, h)
    print(f"[gpu] workspace support {b} of {ws.numel()}", flush=True)
    for size in (b, b + 8 * g.m, ws.numel()):
        out.zero_()
        assert call(size) == 0 and np.array_equal(ht.to_numpy_u32(out), want), size


def test_decomposition_and_batch_in_their_smallest_workspace():
    import torch
    import paper_2411_06405_amd as ht
    g, h = _graph(33_001, 30_000, 4), 2
    rp, ci = _on(g.row_ptr), _on(g.col_idx)
    ws = torch.empty(ht.workspace_bytes(g.n, g.m, h), dtype=torch.uint8, device="cuda")
    t, r = torch.empty((2, g.m), dtype=torch.int32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    to, ro, _ = oracle.decompose(g, h)

    def call(b):
        return ht.lib.hoTrussDecompose(rp.data_ptr(), ci.data_ptr(), g.n, g.m, h, t.data_ptr(), r.data_ptr(),
                                       ws.data_ptr(), b, None, stream)
    small = _smallest(call, ws.numel())
    print(f"[gpu] workspace decompose {small} of {ws.numel()}", flush=True)
    assert small < ws.numel() - 4 * g.n  # the renumbering's maps alone are 12 n + 12 m
    for size in (small, ws.numel()):
        t.zero_()
        assert call(size) == 0
        assert np.array_equal(ht.to_numpy_u32(t), to) and np.array_equal(ht.to_numpy_u32(r), ro), size

    gs, hs = [g, _graph(32_768, 9000, 5), _graph(700, 3000, 6)], [2, 2, 3]
    b = concat(gs, hs)
    one = max(ht.batched_workspace_bytes(np.array([0, x.n], np.uint64), np.array([0, x.m], np.uint64),
                                         np.array([y], np.uint32)) for x, y in zip(gs, hs))
    ws = torch.empty(one - 12 * g.n, dtype=torch.uint8, device="cuda")  # not the largest graph renumbered
    ts, rs = ht.decompose_batch(b, workspace=ws)
    for x, y, tt, rr in zip(gs, hs, ts, rs):
        to, ro, _ = oracle.decompose(x, y)
        assert np.array_equal(tt, to) and np.array_equal(rr, ro), x.name
