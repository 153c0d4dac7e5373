"""hsp_draws gathers a few draws into pinned memory and copies more (or all,
where pinned memory is not to be had): both return the same draws, also where
the ring wraps and at the largest request that is gathered (8188 doubles)."""
import threading

import numpy as np
import pytest

from gpu_util import dataset, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,lam", [(3, False), (31, True), (89, False), (89, True)])
def test_copied_draws_equal_gathered_draws(p, lam):
    torch, hsp = need_gpu()
    d = dataset(500, p, p)
    s = hsp.Sampler(torch.from_numpy(d.X).cuda(), torch.from_numpy(d.y).cuda(), seed=5, max_draws=100, record_lambda=lam)
    s.sweep(230)
    most = 8188 // (p + 1 + (p if lam else 0))
    asked = [(130, 1), (229, 1), (180, 30), (195, 10), (130, min(most, 100)), (130, min(most + 1, 100)), (200, 0)]
    got = {}
    for on in (True, False):
        hsp.hsp_set_gather(s.h, on)
        got[on] = [s.draws(first, count) for first, count in asked]
        with pytest.raises(hsp.HspError):
            s.draws(129, 1)
        with pytest.raises(hsp.HspError):
            s.draws(229, 2)
    for (first, count), a, b in zip(asked, got[True], got[False]):
        for x, y in zip(a, b):
            assert np.array_equal(x, y), (first, count)
        assert a[-1] == 230 and len(a[0]) == count and np.all(a[0] != 0.0)
    s.close()


def test_threads_fetch_different_chains_of_a_batch():
    """The chains of a batch gather through one buffer: threads that fetch different
    chains at the same time each get their own chain's draws."""
    torch, hsp = need_gpu()
    ds = [dataset(400 + 50 * i, 5 + 9 * i, i) for i in range(4)]
    b = hsp.Batch([(torch.from_numpy(d.X).cuda(), torch.from_numpy(d.y).cuda()) for d in ds], 1, seed=5, max_draws=64)
    b.sweep(40)
    want = [c.draws(0, 40) for c in b.chains]
    got = [[] for _ in ds]

    def fetch(i):
        for _ in range(50):
            got[i].append(b.chains[i].draws(0, 40))

    threads = [threading.Thread(target=fetch, args=(i,)) for i in range(len(ds))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for w, g in zip(want, got):
        assert len(g) == 50
        for r in g:
            assert all(np.array_equal(x, y) for x, y in zip(w, r))
    b.close()
