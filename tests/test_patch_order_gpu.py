"""Steps that end before the patches' first halo exchange, while another
stream's kernel holds most CUs, so that patches start late: the oracle's bytes
whatever the order the patches run in."""
import numpy as np
import pytest

import oracle as O
from paper_2508_16639_amd import escg
from paper_2508_16639_amd.workloads import random_lattice
from tests.gpu_util import dev, host, pair

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
