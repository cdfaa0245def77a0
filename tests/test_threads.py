"""Several threads calling on one stream: calls of more than one launch share a queue per
stream, and each must give the results of the call alone, bit for bit."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def apm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2104_07638_amd as m
    return m


def test_minors_on_one_stream(apm):
    """Uniform minors with pivot shifts at every level (zero diagonal) of different orders: the
    corrections of the top levels follow in a second launch (orders above 17 or so leave only
    the levels above their work items to it)."""
    import torch
    rng = np.random.default_rng(4000)
    jobs = []
    for n, B in ((12, 60), (16, 20), (14, 5), (18, 2)):
        A = rng.standard_normal((B, n, n))
        A[::2, np.arange(n), np.arange(n)] = 0.0
        jobs.append(torch.from_numpy(A).cuda())
    want = [apm.all_minors(A, "r64") for A in jobs]
    torch.cuda.synchronize()
    assert all(int(w[2][0]) > 0 for w in want)
    got = [[] for _ in jobs]
    start = threading.Barrier(len(jobs))

    def work(t):
        start.wait()
        for _ in range(30):
            m, _, i = apm.all_minors(jobs[t], "r64")
            got[t].append((m, i))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for (m, _, i), res in zip(want, got):
        assert len(res) == 30
        for m1, i1 in res:
            assert torch.equal(m, m1) and torch.equal(i, i1)
