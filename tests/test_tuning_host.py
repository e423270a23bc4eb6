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


def test_a_choice_for_whole_rows_is_not_one_for_rows_in_phases(tmp_path):
    """F = 1024 and F = 999 share a bucket; N = 99 takes the rows of the first
    whole, those of the second in 16 phases."""
    path = tmp_path / "cache.txt"
    path.write_text("gfx950 0 99 10 8 0 1 0\n")
    _, trace = run(f"""
        X.xeng_tune_cache_load({str(path)!r})
        for f in (1024, 999): call(X.xeng_plan([(99, f, 256)]), [256])
    """)
    assert ["kernel=ring16" in l for l in trace] == [True, False], trace
    # a staging choice is one for any rows; a choice for phases is kept as one
    path.write_text("gfx950 0 99 10 8 2 1 0\ngfx950 0 51 7 9 0 1 0 16\n")
    out, trace = run(f"""
        X.xeng_tune_cache_load({str(path)!r})
        for f in (1024, 999): call(X.xeng_plan([(99, f, 256)]), [256])
        for f in (77, 112): call(X.xeng_plan([(51, f, 500)]), [500])
        X.xeng_tune_cache_save({str(path)!r})
    """)
    assert ["kernel=ring16" in l for l in trace] == [False, False, True, True], trace
    assert "grid=20x16" in trace[2] and "gfx950 0 51 7 9 0 1 0 16\n" in path.read_text()


def test_every_candidate_is_timed_with_the_room_it_would_have():
    """A new plan of a split choice keeps room for the chunks' sums, so no
    trial of a kernel that can store them adds atomically, whatever the plan
    under the tuner was made with; the tuned plan frees all it holds."""
    out, trace = run("""
        d = (96, 1024, 4096)
        h = X.xeng_plan([d]); before = stub.stub_used()
        X.xeng_autotune(h, [1 << 32], [d[2]], 1)
        print(before == X.xeng_accumulator_bytes(*d[:2]), stub.stub_used() == before)
        X.xeng_destroy(h); print(stub.stub_used())
    """)
    assert out == ["True True", "0"]
    split = [l for l in trace if "kernel=ring32" not in l and "x1 threads" not in l]
    assert split and not [l for l in split if "mode=2" in l], split


def test_a_choice_that_needs_more_room_keeps_it():
    """The third candidate (ring kernel, two workgroups per CU) is the fastest."""
    out, trace = run("""
        d = (96, 1024, 4096)
        h = X.xeng_plan([d]); before = stub.stub_used()
        stub.stub_fast(2)
        X.xeng_autotune(h, [1 << 32], [d[2]], 1)
        print(stub.stub_used() // before)
        stub.stub_fast(-1)
        call(h, [d[2]])
        new = X.xeng_plan([d]); call(new, [d[2]])
        X.xeng_destroy(h), X.xeng_destroy(new); print(stub.stub_used())
    """)
    assert int(out[0]) > 1 and out[1] == "0"
    # the tuned plan's next call and a new plan's first
    assert all("kernel=ring16 grid=256x2 threads=256 mode=0 chunks=2" in l for l in trace[-2:]), trace[-2:]


def test_the_batch_tuner_tries_the_modelled_items(tmp_path):
    """Its first candidate is what an untuned plan does (0 items per CU asked for)."""
    path = tmp_path / "cache.txt"
    run(f"""
        X.xeng_autotune(X.xeng_plan([(32, 64, 2048), (96, 128, 1024)]), [1 << 32] * 2, [2048, 1024], 1)
        X.xeng_tune_cache_save({str(path)!r})
    """)
    assert "gfx950 1 0 0 1 0 0 0\n" in path.read_text()
