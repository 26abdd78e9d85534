"""The autotuner measures the pass it tunes: the library's own setting is among
the candidates, choices measured on another pass are not reused, and the timed
query is laid out as the decomposition will be."""
import numpy as np
import pytest

from paper_2411_06405_amd import autotune as A


def test_the_librarys_own_rule_is_a_candidate():
    assert 0 in A.DENSE_THRESHOLDS
    best = A.search(lambda t: 1.0 if t["dense_threshold"] else 0.5, repeats=1)
    assert best["dense_threshold"] == 0


def test_choices_of_an_earlier_pass_are_not_reused(tmp_path):
    c = A.Cache(tmp_path / "tune.json")
    c.put("MI355X|n2^16|d2^3|s2^9|h2", {"word_bits": 64, "edges_per_wave": 1, "dense_threshold": 32})
    key = A.shape_key("MI355X", 100_000, 500_000, 2, 6000)
    assert key.startswith("MI355X|n2^16|d2^3|s2^9|h2") and A.Cache(c.path).get(key) is None


@pytest.mark.gpu
def test_timed_queries_have_the_layout_of_a_decomposition(tmp_path, monkeypatch):
    import paper_2411_06405_amd as ht
    from graphgen.gen import chung_lu
    g = chung_lu(33_000, 6.0, 2.5, seed=3)  # renumbered by a decomposition only
    seen, made = [], ht._lib._tuning

    def spy(tune):
        seen.append(dict(tune or {}))
        return made(tune)
    monkeypatch.setattr(ht._lib, "_tuning", spy)
    tune = A.autotune(g.row_ptr, g.col_idx, g.n, 2, device="cuda:0", cache=tmp_path / "t.json", repeats=1)
    timed = [t for t in seen if "word_bits" in t]
    assert len(timed) == len(A.DENSE_THRESHOLDS) + len(A.WIDTHS) * len(A.EDGES_PER_WAVE)
    assert all(t["flags"] & ht._lib.HO_FLAG_DECOMPOSE_LAYOUT for t in timed)
    assert set(tune) == {"word_bits", "edges_per_wave", "dense_threshold"}
    a = ht.decompose_graph(g, 2, tune=tune)
    b = ht.decompose_graph(g, 2)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
