"""Calls whose launches hold most of the device and wait among their own
workgroups, on two streams at once: the runtime runs them one after the other
and every lattice is the oracle's."""
import numpy as np
import pytest

import oracle as O
from paper_2508_16639_amd import escg
from paper_2508_16639_amd.workloads import random_lattice
from tests.gpu_util import dev, host, pair

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_step_batch_beside_single_steps():
    streams = [torch.cuda.Stream() for _ in range(2)]
    batch = [pair(L, 3, [1], 0.5, seed=i, replica=i)
             for i, L in enumerate((400, 800, 400, 800, 1600))]
    single = [pair(L, 3, [1], 0.5, seed=L) for L in (300, 512)]
    g = [random_lattice(p.L, 3, seed=p.L + i, domain=2)
         for i, (p, _) in enumerate(batch + single)]
    lats = [dev(x) for x in g]
    nb, n, rounds = 10, 40, 3
    torch.cuda.synchronize()
    for k in range(rounds):
        with torch.cuda.stream(streams[0]):
            escg.step_batch([p for p, _ in batch], lats[:5], [nb * k] * 5,
                            [nb] * 5)
            assert escg.last_route() == "persistent"
        with torch.cuda.stream(streams[1]):
            for (p, _), lat in zip(single, lats[5:]):
                escg.step_mcs(p, lat, n * k, n, None)
                assert escg.last_route() == "persistent"
    torch.cuda.synchronize()
    escg.async_status()
    for i, ((_, j), x, lat) in enumerate(zip(batch + single, g, lats)):
        O.o2_run(j, x, 0, rounds * (nb if i < 5 else n), want_counts=False)
        assert np.array_equal(host(lat), x), (i, j.L)
