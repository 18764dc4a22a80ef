"""Picks cached for kernels that are gone are timed again (CPU, a fake run)."""
import json

from paper_1804_03901_amd import avl, inputs, tune


def test_picks_of_the_block_sort_passes_are_not_used(tmp_path, monkeypatch):
    class Fake:
        stream = None

        def __init__(self, *a, **kw):
            pass

        def close(self):
            pass

    monkeypatch.setattr(avl, "Simulation", Fake)
    monkeypatch.setattr(tune, "_graph_ms", lambda *a, **kw: 1.0)
    w = inputs.bump_on_tail(nx=16, nv=8, ppc=1)
    path = str(tmp_path / "t.json")
    timed, _ = tune.tune_single(w, markers=inputs.markers(w), cache_path=path)
    cache = json.load(open(path))
    (key, entry), = cache.items()
    stale = tune._to_cache({**timed, avl.TUNE_SORT_BLOCKS: 3}, {k: {0: 1.0} for k in timed})
    assert key.startswith(tune.CACHE_VERSION + "|")
    json.dump({"v2|" + key.split("|", 1)[1]: stale}, open(path, "w"))
    assert tune.tune_single(w, markers=inputs.markers(w), cache_path=path)[0] == timed
