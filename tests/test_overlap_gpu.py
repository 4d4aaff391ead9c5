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


def test_two_step_batches_and_threads():
    """Two host threads, each with a stream and its own batch of large jobs,
    and a third with single steps."""
    import threading
    n, rounds, errors, out = 6, 6, [], {}

    def jobs(k):
        sides = ((1600, 800, 400, 1600), (800, 1600, 1600), (200, 512))[k]
        return [pair(L, 3, [1], 0.5, seed=10 * k + i)
                for i, L in enumerate(sides)]

    def drive(k):
        try:
            js = jobs(k)
            g = [random_lattice(p.L, 3, seed=i, domain=2)
                 for i, (p, _) in enumerate(js)]
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                lats = [dev(x) for x in g]
                for r in range(rounds):
                    if k < 2:
                        escg.step_batch([p for p, _ in js], lats,
                                        [n * r] * len(js), [n] * len(js))
                    else:
                        for (p, _), lat in zip(js, lats):
                            escg.step_mcs(p, lat, n * r, n, None)
                    assert escg.last_route() == "persistent"
                s.synchronize()
                out[k] = (js, g, [x.cpu().numpy() for x in lats])
        except Exception as e:  # reported by the main thread
            errors.append(repr(e))

    ts = [threading.Thread(target=drive, args=(k,)) for k in range(3)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors
    escg.async_status()
    for k, (js, g, lats) in out.items():
        for (_, j), x, lat in zip(js, g, lats):
            O.o2_run(j, x, 0, rounds * n, want_counts=False)
            assert np.array_equal(lat, x), (k, j.L)
