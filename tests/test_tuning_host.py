"""The tuning cache and the autotuner's choices on a stand-in for the HIP
runtime (CPU): every trial takes the same time there, so the first candidate
of each kind is the one kept."""
from tests.hip_stub import run


def test_a_tuned_batch_is_saved_and_loaded(tmp_path):
    """An array that stays in the batch launch has no time split of its own (0)."""
    path = str(tmp_path / "cache.txt")
    out, _ = run(f"""
        shapes = [(32, 64, 2048), (96, 128, 1024), (37, 77, 900)]
        h = X.xeng_plan(shapes)
        X.xeng_autotune(h, [1 << 32] * 3, [s[2] for s in shapes], 1)
        X.xeng_tune_cache_save({path!r})
        X.xeng_tune_cache_clear()
        X.xeng_tune_cache_load({path!r})
        X.xeng_tune_cache_save({path + "2"!r})
        h = X.xeng_plan(shapes)
        call(h, [s[2] for s in shapes])
        print("ok")
    """)
    assert out == ["ok"]
    saved = open(path).read()
    assert saved == open(path + "2").read() and saved.count("gfx950 1 ") == 4
