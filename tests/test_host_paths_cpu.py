"""What the library's host code enqueues, without a GPU: each scenario below
runs in a process of its own over a runtime that only records launches
(tests/fake_hip.py)."""
import sys

import pytest

from tests import fake_hip


@pytest.fixture(scope="module")
def fake_so(tmp_path_factory):
    return fake_hip.build(str(tmp_path_factory.mktemp("fake")))


def refused_chunk(f, refuse, stop, done):
    """A run until extinction (chunks of 64, 128, ... MCS) of which the
    cooperative launch number `refuse` is refused; stop >= 0: the species die
    out that many MCS into every chunk that is long enough.  The `done` MCS
    before the refused launch are not run again, the others go out one tiled
    launch each."""
    n = 1000
    f.reset(refuse=refuse, words=4, stop=0xFFFFFFFF if stop < 0 else stop)
    assert f.until(f.params(512), n) == 0
    assert len(f.names("patch_kernel")) == refuse
    got = len(f.names("tiled_step_kernel"))
    assert got == n - done, (got, done)
    assert f.lib.escg_last_route() == f.escg.ROUTE_TILED


@pytest.mark.parametrize("refuse,stop,done", [
    (0, -1, 0), (1, -1, 64), (2, -1, 192),
    (1, 10, 0), (2, 100, 64)])  # the re-run of a chunk
def test_refused_chunk_is_not_started_over(fake_so, refuse, stop, done):
    fake_hip.run(fake_so, __file__, "refused_chunk", refuse, stop, done)


WAITING = ("patch_kernel", "tiled_persistent_kernel",
           "tiled_persistent_multi_kernel")


def waiting_launches(f):
    """Launches whose workgroups wait for each other fit the device and never
    run side by side: single jobs' are cooperative (ordered by the runtime),
    and so is a multi-job launch after them; one after another multi-job launch
    is ordinary.  All wait for the event that a multi-job launch records.
    Other launches are ordinary."""
    def check(*kinds):
        log = f.launches()
        for x in log:
            waits = any(k in x.name for k in WAITING)
            assert not waits or x.grid <= 256, x
            if "multi" not in x.name:
                assert x.cooperative == waits, x
        for k in kinds:
            assert f.names(k), (k, log)
        return [x for x in log
                if "event" in x.name or any(k in x.name for k in WAITING)]

    def singles():
        f.reset()
        for p in (f.params(300), f.params(512), f.params(3200, S=9),
                  f.params(3600), f.params(512, tile=(32, 32))):
            assert f.step(p, 50) == 0
        return check("patch_kernel", "tiled_persistent_kernel")

    def batch(wgs):
        f.reset()
        ps = [f.params(400 << (j % 3), S=(3, 9)[j % 2]) for j in range(24)]
        ps[0] = ps[0].with_launch(max_wgs=wgs)
        assert f.step_batch(ps, [500] * 24) == 0
        assert f.lib.escg_last_route() == f.escg.ROUTE_PERSISTENT
        assert not wgs or all(x.grid <= wgs for x in f.names("multi_kernel"))
        return check("tiled_persistent_multi_kernel")

    def kinds(log):
        """w: wait, r: record, C / S: cooperative multi-job / single launch,
        M: ordinary multi-job launch."""
        assert all(x.grid == 1 for x in log if "event" in x.name)
        return "".join(
            "w" if x.name == "event wait" else "r" if "event" in x.name else
            "S" if "multi" not in x.name else "C" if x.cooperative else "M"
            for x in log)

    n = kinds(singles())
    assert set(n) == {"S"}
    first = kinds(batch(0))  # two launches or more: S <= 7 and S > 7
    assert first == "Cr" + "wMr" * (len(first) // 3) and len(first) > 2
    assert kinds(batch(40)).replace("wMr", "") == ""
    assert kinds(singles()) == "wS" * len(n)
    assert kinds(batch(0)) == "wCr" + "wMr" * (len(first) // 3)
    # under capture: no events, cooperative
    f.reset(capture=True)
    assert f.step(f.params(512), 50) == 0
    assert f.step_batch([f.params(400)] * 2, [5, 5]) == 0
    log = check()
    assert len(log) == 2 and all(x.cooperative for x in log)


def refused_multi(f, refuse):
    """Jobs of a refused multi-job launch go out per MCS, all of their MCS;
    the launches before it stay."""
    # S <= 7 and S > 7: two launches
    f.reset(refuse=refuse, capture=True)  # all of them cooperative
    ps = [f.params(400), f.params(136, S=9), f.params(800)]
    assert f.step_batch(ps, [6, 5, 4]) == 0
    assert len(f.names("multi_kernel")) == refuse
    steps = f.names("tiled_step_batch_kernel")
    assert len(steps) == {0: 11, 1: 6, 2: 0}[refuse], steps
    assert f.lib.escg_last_route() == (f.escg.ROUTE_PERSISTENT if refuse
                                       else f.escg.ROUTE_TILED)


def test_launches_that_wait_never_run_side_by_side(fake_so):
    fake_hip.run(fake_so, __file__, "waiting_launches")


@pytest.mark.parametrize("refuse", [0, 1, 2])
def test_refused_multi_job_launch_runs_per_mcs(fake_so, refuse):
    fake_hip.run(fake_so, __file__, "refused_multi", refuse)


def no_tile_plan(f):
    """Sides whose only divisors that are multiples of 8 are 8 and L have
    patches but no equal resident tiles: the persistent path is refused when
    asked for and no cooperative launch is captured; sides with tiles, and
    calls that leave the choice to the library, are as ever."""
    for L, tiles in ((8, False), (2056, False), (3208, False), (16, True),
                     (512, True), (3200, True)):
        for S in (3, 9):
            want = 0 if tiles else f.escg.EUNSUPPORTED
            q = f.params(L, S=S, route="persistent")
            f.reset(words=S + 1)
            assert f.step(q, 6) == want and f.until(q, 6) == want, (L, S)
            assert tiles or not f.launches()
            for capture in (False, True):
                f.reset(capture=capture)
                assert f.step(f.params(L, S=S), 6) == 0
                waits = [x for x in f.launches() if x.cooperative]
                assert bool(waits) == (L >= 72 and (tiles or not capture)), L


def test_sides_without_a_tile_plan(fake_so):
    fake_hip.run(fake_so, __file__, "no_tile_plan")


def short_patch_runs(f):
    """A run on patches that ends before its first halo exchange: patches wait
    for nothing and may start when a neighbour has ended, so they read a copy
    of the lattice, in an ordinary launch; the copy is all the scratch."""
    for L in (96, 250, 402, 512, 700, 1500, 3302):
        for static in (False, True):
            for counts in (False, True):
                f.reset()
                assert f.step(f.params(L), 1, counts, static) == 0
                prep, run = f.launches()
                assert "patch_prep_kernel" in prep.name
                assert prep.grid == min(512, (L * L // 4 + 255) // 256)
                assert "patch_kernel" in run.name and not run.cooperative
                assert f.dll.fake_allocated() == (0 if static else L * L), L
        f.reset()
        assert f.step(f.params(L), 8) == 0
        assert [x.cooperative for x in f.names("patch_kernel")] == [True]
        # with a copy of the lattice at hand
        f.reset(words=4)
        assert f.until(f.params(512), 1) == 0
        prep, run = f.names("patch")
        assert not run.cooperative and prep.grid == 1 # the count rows


def test_runs_without_an_exchange_read_a_copy(fake_so):
    fake_hip.run(fake_so, __file__, "short_patch_runs")


def single_patches(f):
    """A few MCS of a small lattice with L % 8 != 0: one ordinary launch of one
    workgroup, no scratch, and one launch more for count rows."""
    for L, S, most in ((90, 3, 4), (122, 9, 4), (138, 3, 4), (154, 3, 2),
                       (162, 31, 1), (170, 3, 0), (96, 3, 0), (398, 3, 0)):
        for n in range(1, 7):
            for static in (False, True):
                f.reset()
                assert f.step(f.params(L, S=S), n, True, static) == 0
                prep, run = f.names("patch")
                one = n <= most
                assert (run.grid == 1) == one, (L, n, run)
                assert not one or not run.cooperative
                assert not one or f.dll.fake_allocated() == 0
                assert f.escg.last_route() == "persistent"
            f.reset()
            assert f.step(f.params(L, S=S), n, False) == 0
            assert not one or len(f.launches()) == 1


def test_a_few_mcs_on_a_single_patch(fake_so):
    fake_hip.run(fake_so, __file__, "single_patches")


def pair_limits(f, lds):
    """The kernel with two copies of a lattice is taken only up to the quads
    that it gives its threads, and the LDS."""
    f.dll.fake_lds(lds)
    for L, S, pair in ((90, 3, True), (276, 3, True), (278, 3, True),
                       (280, 3, True), (282, 3, lds > 160 * 1024),
                       (284, 3, lds > 160 * 1024), (288, 3, False),
                       (300, 3, False), (90, 9, True), (264, 9, True),
                       (266, 9, lds > 160 * 1024), (300, 9, False)):
        p = f.params(L, S=S, route="lds")
        f.reset(words=S + 1)
        assert f.until(p, 9) == 0
        assert bool(f.names("pair_single_kernel")) == pair, (L, S)
        f.reset()
        assert f.batch([p], [9]) == 0
        assert bool(f.names("pair_batch_kernel")) == pair, (L, S)


@pytest.mark.parametrize("lds", [160 * 1024, 400 * 1024])
def test_limits_of_the_two_copy_kernel(fake_so, lds):
    fake_hip.run(fake_so, __file__, "pair_limits", lds)


if __name__ == "__main__":
    globals()[sys.argv[2]](fake_hip.Fake(sys.argv[1]),
                           *map(int, sys.argv[3:]))
