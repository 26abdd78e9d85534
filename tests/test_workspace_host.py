"""Workspaces that programs sized for earlier versions of the library are still
enough, whatever layout the graph would get with more room.  No GPU: a call
that accepts its workspace goes on to the HIP runtime and fails there."""
import ctypes as C

import numpy as np
import pytest

WORKSPACE, HIP = -3, -4


@pytest.fixture(scope="module")
def ht():
    import torch
    if torch.cuda.is_available():
        pytest.skip("would run on made-up addresses")
    import paper_2411_06405_amd as ht
    return ht


FAKE = C.c_void_p(0x1000)


@pytest.mark.parametrize("n,m,h,bytes_", [
    (200, 1000, 2, 69_888), (33_000, 300_000, 2, 285_630_720), (524_288, 1000, 2, 68_723_715_840),
    # renumbered where there is room
    (100_000, 1_000_000, 2, 2_545_607_680), (100_000, 1_000_000, 3, 3_800_007_680),
])
def test_support_query(ht, n, m, h, bytes_):
    call = lambda b: ht.lib.hoTrussHSupport(FAKE, FAKE, n, m, h, FAKE, FAKE, b, None, None)  # noqa: E731
    assert call(bytes_) == HIP
    assert call(bytes_ // 2) == WORKSPACE
    assert call(ht.workspace_bytes(n, m, h)) == HIP


@pytest.mark.parametrize("n,m,h,tune,bytes_", [
    (2, 1, 1, {}, 1_324_032), (1000, 300, 1, {}, 1_648_384), (5000, 20_000, 3, {}, 223_653_632),
    (30, 90, 2, {"event_capacity": 64, "item_capacity": 64}, 293_120), (30, 90, 2, {"flags": 2}, 3_435_776),
    # renumbered where there is room
    (32_768, 20_000, 2, {}, 529_386_752), (100_000, 250_000, 2, {}, 5_333_073_664),
    (300_000, 100_000, 3, {}, 57_303_074_560),
    (524_288, 1000, 2, {"event_capacity": 64, "item_capacity": 64}, 103_099_010_304),
])
def test_decomposition(ht, n, m, h, tune, bytes_):
    t = ht._lib._tuning(tune)
    call = lambda b: ht.lib.hoTrussDecompose(FAKE, FAKE, n, m, h, FAKE, FAKE, FAKE, b, t, None)  # noqa: E731
    assert call(bytes_) == HIP
    assert call(bytes_ // 2) == WORKSPACE
    assert call(ht.workspace_bytes(n, m, h, tune)) == HIP


@pytest.mark.parametrize("count,n,m,h,bytes_", [
    (1, 200, 1000, 2, 3_584_000), (64, 500, 2000, 3, 5_933_824), (256, 100, 300, 2, 3_476_480),
    (3, 40_000, 60_000, 2, 661_713_920),  # renumbered where there is room
])
def test_batch_of_equal_graphs(ht, count, n, m, h, bytes_):
    vo = np.arange(count + 1, dtype=np.uint64) * np.uint64(n)
    eo = np.arange(count + 1, dtype=np.uint64) * np.uint64(m)
    ao, hs = eo * np.uint64(2), np.full(count, h, np.uint32)
    p = lambda a: a.ctypes.data  # noqa: E731
    call = lambda b: ht.lib.hoTrussDecomposeBatched(FAKE, FAKE, p(vo), p(ao), p(eo), p(hs), count, FAKE,  # noqa: E731
                                                    FAKE, FAKE, b, None, None)
    assert call(bytes_) == HIP
    assert call(bytes_ // 2) == WORKSPACE
    assert call(ht.batched_workspace_bytes(vo, eo, hs)) == HIP


def test_other_queries_did_not_grow(ht):
    # the H-index method and the extraction keep no round state
    assert ht.lib.hoTrussHIndexWorkspaceBytes(1000, 5000, 2) <= 585_984
    assert ht.lib.hoTrussComponentsWorkspaceBytes(1000, 5000) <= 203_264
