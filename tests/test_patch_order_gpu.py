"""Steps that end before the patches' first halo exchange, while another
stream's kernel holds most CUs, so that patches start late: the oracle's bytes
whatever the order the patches run in."""
import numpy as np
import pytest

import oracle as O
from paper_2508_16639_amd import escg
from paper_2508_16639_amd.workloads import random_lattice
from tests.gpu_util import dev, host, pair, probabilities

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("L,n", [(90, 1), (300, 2), (512, 1), (1002, 1),
                                 (3200, 1)])
def test_short_steps_beside_a_batch(L, n):
    p, j = pair(L, 3, [1], 0.5, seed=L)
    g = random_lattice(L, 3, seed=L, domain=2)
    # alternate calls with and without counts, fixed and allocated scratch
    lats = [dev(g) for _ in range(2)]
    cnt = torch.zeros((n + 1) * 4, dtype=torch.int32, device="cuda:0")
    jobs = [pair(256, 3, [1], 0.5, seed=1, replica=i)[0] for i in range(250)]
    buf = torch.empty(250 * 65536, dtype=torch.uint8, device="cuda:0")
    res = torch.empty(250 * escg.BATCH_RESULT_WORDS, dtype=torch.int32,
                      device="cuda:0")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        escg.batch_run(jobs, [i * 65536 for i in range(250)], buf,
                       [1500] * 250, escg.STOP_NONE, True, res)
    rounds = 6
    for k in range(rounds):
        escg.step_mcs(p, lats[0], n * k, n, cnt if k % 2 else None)
        escg.step_mcs_static(p, lats[1], n * k, n, None if k % 2 else cnt)
        assert escg.last_route() == "persistent"
    torch.cuda.synchronize()
    O.o2_run(j, g, 0, rounds * n, want_counts=False)
    for lat in lats:
        assert np.array_equal(host(lat), g)


@pytest.mark.parametrize("L,S,n,moore,prob", [
    (90, 3, 1, False, False), (90, 5, 4, True, False), (94, 13, 2, False, True),
    (100, 3, 3, False, False), (122, 31, 4, True, False),
    (130, 7, 4, False, True), (138, 3, 4, False, False),
    (154, 3, 2, True, False), (162, 8, 1, False, True)])
def test_single_patch_bit_exact(L, S, n, moore, prob):
    """A few MCS of a small lattice with L % 8 != 0: one patch, one and two
    quads a thread, in place."""
    D = O.circulant_matrix(S, [1, 3] if S > 4 else [1])
    P = probabilities(D, seed=L) if prob else None
    p, j = pair(L, S, None, 2.0, seed=L + 5, replica=2, D=D, moore=moore, P=P)
    g0 = random_lattice(L, S, seed=L, domain=3)
    ref = g0.copy()
    rc = O.o2_run(j, ref, 1 << 20, n)
    for fn in (escg.step_mcs, escg.step_mcs_static):
        for counts in (True, False):
            lat = dev(g0)
            cnt = torch.full(((n + 1) * (S + 1),), -1, dtype=torch.int32,
                             device="cuda:0") if counts else None
            fn(p, lat, 1 << 20, n, cnt)
            assert escg.last_route() == "persistent"
            assert np.array_equal(host(lat), ref), counts
            if counts:
                assert np.array_equal(host(cnt).reshape(rc.shape), rc)


def test_run_until_of_a_few_mcs():
    """Chunks and re-runs no longer than the MCS between two exchanges."""
    D = np.array([[0, 1, 1], [0, 0, 0], [0, 0, 0]], np.uint8)
    for L, sel in ((80, 8.0), (406, 30.0)):
        p, j = pair(L, 3, None, 0.1, sel, 0.1, seed=3, D=D)
        g0 = j.init()
        t = int(O.o2_run_until(j, g0.copy(), 0, 400, O.FIRST_EXTINCTION)[1])
        for cap in (1, 2, 3, t, 400):
            g, lat = g0.copy(), dev(g0)
            res = torch.full((6,), -1, dtype=torch.int32, device="cuda:0")
            escg.run_until_extinction(p, lat, 0, cap,
                                      escg.STOP_FIRST_EXTINCTION, res)
            assert escg.last_route() == "persistent"
            ref = O.o2_run_until(j, g, 0, cap, O.FIRST_EXTINCTION)
            assert np.array_equal(host(res), ref), (L, cap)
            assert np.array_equal(host(lat), g), (L, cap)
