"""The autotuner times only what a knob changes: the sort shapes on evaluations
that sort, compared by the sorted lists; the resident block, which changes
nothing, not at all."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_a_wrong_sort_is_noticed(monkeypatch):
    import torch
    from paper_2502_10685_amd import _lib as L
    from paper_2502_10685_amd import api, autotune
    assert torch.cuda.is_available(), "GPU tests need a visible HIP device"
    monkeypatch.setattr(autotune, "SORT_CLASSES", {0: autotune.SORT_CLASSES[0]})
    old = L.tune_get(L.PP_TUNE_SORT_SHAPE, 0)
    real = api.Circuit.terms

    def swapped(self, *a, **kw):
        out = [np.array(v) for v in real(self, *a, **kw)]
        if L.tune_get(L.PP_TUNE_SORT_SHAPE, 0) == 3:
            for v in out:
                v[[0, 1]] = v[[1, 0]]
        return tuple(out)

    try:
        res = autotune.tune_sort(reps=1)
        assert set(res["timings"]["0"]) == {"terms"} | {f"{b}b{i}i" for b, i in autotune.SORT_SHAPES.values()}
        assert res["timings"]["0"]["terms"] == 1 << 16
        L.tune_set(L.PP_TUNE_SORT_SHAPE, 0, old)
        monkeypatch.setattr(api.Circuit, "terms", swapped)
        with pytest.raises(RuntimeError):
            autotune.tune_sort(reps=1)
        assert L.tune_get(L.PP_TUNE_SORT_SHAPE, 0) == old
    finally:
        L.tune_set(L.PP_TUNE_SORT_SHAPE, 0, old)


def test_resident_block_is_left_alone(monkeypatch):
    from paper_2502_10685_amd import _lib as L
    from paper_2502_10685_amd import autotune
    calls = []
    real = L.tune_set
    monkeypatch.setattr(L, "tune_set", lambda key, i, v: (calls.append((key, i, v)), real(key, i, v)))
    monkeypatch.setattr(autotune, "_time_batch", lambda *a, **kw: 1.0)
    saved = {k: L.tune_get(L.PP_TUNE_TILE_KERNEL, k) for k in (4, 5, 6, 7)}
    try:
        table = autotune.tune(sizes=(), m=60, save=False, resident=(5, 6, 7), sort=False)
    finally:
        for k, v in saved.items():
            real(L.PP_TUNE_TILE_KERNEL, k, v)
    assert not [c for c in calls if c[0] == L.PP_TUNE_RESIDENT_BLOCK]
    assert table["resident_block"] == {str(n): L.tune_get(L.PP_TUNE_RESIDENT_BLOCK, n) for n in (5, 6, 7)}
    assert table["timings"]["resident_block"] == {}
