"""A tuning result belongs to the sources it was timed on: the entry says which, and one that was filed under
another hash since is not used (no GPU)."""
import json

from paper_2510_20929_amd import autotune


def test_frozen_entries_were_timed_on_the_sources_of_their_key():
    with open(autotune.DEFAULT_CACHE) as fh:
        cache = json.load(fh)
    assert cache
    for key, e in cache.items():
        assert f"|src{e.get('src')}|" in key, key
        assert autotune.cached_choice(cache, key) == e["tune"]


def test_refiled_entry_is_not_used():
    h = autotune.source_hash()
    e = {"tune": {"variant": 1}, "ms": 1.0, "src": "0" * 12}
    assert autotune.cached_choice({f"gfx950|src{h}|x": e}, f"gfx950|src{h}|x") is None
    del e["src"]
    assert autotune.cached_choice({f"gfx950|src{h}|x": e}, f"gfx950|src{h}|x") is None
    assert autotune.cached_choice({}, f"gfx950|src{h}|x") is None
    e["src"] = h
    assert autotune.cached_choice({f"gfx950|src{h}|x": e}, f"gfx950|src{h}|x") == {"variant": 1}
