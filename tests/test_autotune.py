"""The launch search: groups and one query per wavefront are asked for by
name, launches counted by tiles (which use none of the searched fields) are
timed once with the library's default shape, and the cache keeps no entry of
other sources."""
import json

from paper_cs_0608108_amd import autotune, sphidx


def _tune(monkeypatch, tmp_path, kernel_of):
    cache = tmp_path / "tuned.json"
    cache.write_text(json.dumps({"gfx950|000000000000|workload=old": {"config": {}, "ms": 1.0},
                                 f"gfx950|{autotune.kernel_version()}|workload=kept": {"config": {}, "ms": 1.0}}))
    monkeypatch.setattr(autotune, "CACHE", str(cache))
    timed = []

    def runner(ln):
        timed.append(ln)
        return lambda: None

    # later candidates look a little faster: noise that must not choose
    monkeypatch.setattr(autotune, "time_config", lambda run, reps=3: 1.0 - 1e-4 * len(timed))
    sub = []
    cfg = autotune.tune(dict(workload="w"), runner, kernel_of=kernel_of,
                        subcell_runner=lambda ln, s: sub.append(s) or (lambda: None))
    return cfg, timed, sub, json.loads(cache.read_text())


def test_candidates_ask_for_groups_or_one_query_per_wavefront():
    got = {c["grouped"] for c in autotune.candidates(sphidx.SCHED_PERSISTENT)}
    assert got == {1, 2}


def test_tiles_are_timed_once(monkeypatch, tmp_path):
    cfg, timed, sub, cache = _tune(monkeypatch, tmp_path,
                                   lambda ln: autotune.TILES if ln.grouped == 1 else "count_kernel")
    assert sum(ln.grouped == 1 for ln in timed) == 1
    first = next(ln for ln in timed if ln.grouped == 1)
    assert (first.waves_per_block, first.tile, first.blocks_per_cu, first.sort_cap) == (4, 64, 8, 256)
    assert not any("000000000000" in k for k in cache) and any("workload=kept" in k for k in cache)


def test_tiles_keep_the_default_shape(monkeypatch, tmp_path):
    cfg, timed, sub, cache = _tune(monkeypatch, tmp_path, lambda ln: autotune.TILES)
    assert len(timed) == 1 and not sub
    assert cfg == dict(waves_per_block=4, tile=64, blocks_per_cu=8, sort_cap=256, table_in_lds=0, interior=1, grouped=1)


def test_other_kernels_are_searched(monkeypatch, tmp_path):
    cfg, timed, sub, cache = _tune(monkeypatch, tmp_path, lambda ln: "count_kernel")
    assert len(timed) > 400 and sub == [0, 1, 2, 3] and "long_row_waves" in cfg
