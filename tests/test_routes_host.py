"""Which kernel and which way of adding up a call takes, read from the trace of
the library's host code on a stand-in for the HIP runtime (CPU)."""
import re

import pytest

from tests.hip_stub import run

LAUNCH = re.compile(r"N=(\d+) F=(\d+) T=(\d+) (?:kernel=(\w+) )?grid=(\d+)x(\d+) threads=\d+ mode=(\d) chunks=(\d+)")
ATOMIC = 2


def launches(trace):
    """(n, f, t), kernel, mode of each plain launch."""
    found = [LAUNCH.search(l) for l in trace]
    return [((int(m[1]), int(m[2]), int(m[3])), m[4], int(m[7])) for m in found if m]


# rows whose stride shares few factors with the load unit: up to 16 phases
LARGE = [(99, 587, 1024), (201, 1001, 1024), (250, 1001, 512), (99, 999, 256), (199, 999, 256), (251, 1001, 256)]
BATCHED = [(37, 1001, 512), (51, 999, 512), (113, 933, 903), (61, 513, 300)]


@pytest.mark.parametrize("batch,shapes", [(0, LARGE), (1, BATCHED)])
def test_phases_without_room_for_their_sums_do_not_add_atomically(batch, shapes):
    _, trace = run(f"""
        for d in {shapes}:
            h = X.xeng_plan([d], {batch})
            call(h, [d[2]]), call(h, [d[2]], True)
            X.xeng_destroy(h)
    """)
    got = launches(trace)
    assert len(got) == 2 * len(shapes)
    # (the staging kernel has one phase; its time chunks still add atomically in a batched plan)
    assert not [g for g in got if g[1] != "staging" and g[2] == ATOMIC], got


def test_the_call_decides_not_the_longest_one_planned():
    """Few rows per phase go to the staging kernel, many to the ring kernel,
    in calls of one plan and in plans for each length alike."""
    d, lengths = (37, 1001), (100, 512, 8192, 100)
    _, trace = run(f"""
        h = X.xeng_plan([({d[0]}, {d[1]}, 8192)])
        for t in {lengths}: call(h, [t])
        for t in {lengths}: call(X.xeng_plan([({d[0]}, {d[1]}, t)]), [t])
    """)
    kernels = [k for _, k, _ in launches(trace)]
    assert kernels == ["staging", "staging", "ring16", "staging"] * 2


def test_rows_of_whole_load_units_stay_on_the_ring_kernel():
    shapes = [(n, f, t) for n in (1, 7, 20, 40, 100, 132, 200, 250) for f in (16, 64, 1024) for t in (1, 100, 4096)]
    _, trace = run(f"""
        for d in {shapes}:
            for batch in (0, 1):
                h = X.xeng_plan([d], batch); call(h, [d[2]]); X.xeng_destroy(h)
    """)
    got = launches(trace)
    assert len(got) == 2 * len(shapes) and {k for _, k, _ in got} == {"ring16"}


def test_shapes_of_the_gpu_tests_take_the_paths_they_name():
    """(tests/test_phases_gpu.py)"""
    _, trace = run("""
        h = X.xeng_plan([(37, 301, 4096)])
        for t in (100, 4096): call(h, [t])
        h = X.xeng_plan([(251, 5, 3000), (53, 3, 3000)])
        call(h, [3000, 3000])
    """)
    assert launches(trace) == [((37, 301, 100), "staging", 0), ((37, 301, 4096), "ring16", 0),
                               ((251, 5, 3000), "ring16", ATOMIC), ((53, 3, 3000), "ring16", ATOMIC)]


def test_a_plan_is_made_where_the_accumulator_alone_fits():
    """The room for time chunks' sums is left out when there is no memory for
    it (the call adds atomically then); nothing stays allocated."""
    out, trace = run("""
        d = (100, 64, 4096)
        acc = X.xeng_accumulator_bytes(100, 64)
        for limit in (1 << 40, 2 * acc, acc, acc - 1):
            stub.stub_limit(limit)
            try:
                h = X.xeng_plan([d])
            except X.XengError as e:
                print(limit < acc, e.status == X.XENG_ENOMEM)
            else:
                call(h, [4096]); print(stub.stub_used() // acc); X.xeng_destroy(h)
        print(stub.stub_used())
    """)
    assert out[1:] == ["1", "1", "True True", "0"] and int(out[0]) > 2
    assert [m for _, _, m in launches(trace)] == [0, ATOMIC, ATOMIC]


def test_a_batch_of_more_items_than_a_grid_holds():
    """A grid holds fewer than 2^32 threads: 17 arrays of 2^20 channel groups
    go in two launches."""
    _, trace = run("""
        h = X.xeng_plan([(16, (1 << 22) - 1, 1)] * 17)
        call(h, [1] * 17)
    """)
    got = [tuple(int(x) for x in re.search(r"batch launch arrays=(\d+) items=(\d+)", l).groups()) for l in trace]
    assert got == [(15, 15 << 20), (2, 2 << 20)]
