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


if __name__ == "__main__":
    globals()[sys.argv[2]](fake_hip.Fake(sys.argv[1]),
                           *map(int, sys.argv[3:]))
