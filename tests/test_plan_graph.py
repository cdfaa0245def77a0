"""The widest plans, whose launches replay a HIP graph: mixed-order CDet plans of two matrix sets
with orders up to 14 and more are ten kernels (three for the minors of each set, four for the
sums); plans of up to eight are enqueued kernel by kernel (see the other plan tests)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def apm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2104_07638_amd as m
    return m


def _same(a, b):
    import torch
    return torch.equal(a.view(torch.int64), b.view(torch.int64))


@pytest.mark.parametrize("lo,hi,B", [(10, 16, 120), (1, 14, 300), (12, 18, 20)])
def test_two_set_mixed_plan(apm, lo, hi, B):
    """Several replays on new values in the same buffers, on two streams and with eager work
    between, against the direct calls, bit for bit; a zero-diagonal set among the values
    (shifted pivots)."""
    import torch
    lat = W.Lattice(32, 1.0, -0.5, 5.0)
    mats, ns = W.lattice_ragged(B, lo, hi, lat, seed=700 + hi)
    ns[0] = hi
    mats[0] = W.lattice_batch(1, hi, lat, seed=701 + hi)[0]
    up = np.concatenate([m.ravel() for m in mats])
    dn = np.concatenate([W.lattice_batch(1, int(n), lat, seed=800 + b)[0].ravel() for b, n in enumerate(ns)])
    zd = np.concatenate([(m - np.diag(np.diag(m))).ravel() for m in mats])
    vals = [torch.from_numpy(x).cuda() for x in (up, dn, zd)]
    n_t = torch.from_numpy(ns).cuda()
    tot = int(np.sum(np.left_shift(1, ns.astype(np.int64))))
    A, Ad = torch.empty_like(vals[0]), torch.empty_like(vals[0])
    m, md, c, mr, mdr, cr = (torch.empty(tot, dtype=torch.float64, device="cuda") for _ in range(6))
    bd = apm.make_batch(B, 0, n_t, hi)
    plan = apm.plan_cdet(A, m, c, A_dn=Ad, minors_dn=md, n=n_t, n_max=hi)
    assert plan.graphed
    side = torch.cuda.Stream()
    for r in range(5):
        A.copy_(vals[r % 3])
        Ad.copy_(vals[(r + 1) % 3])
        for t in (m, md, c):
            t.fill_(7.0)
        if r % 2:
            side.wait_stream(torch.cuda.current_stream())
            plan.launch(side)
            torch.cuda.current_stream().wait_stream(side)
        else:
            plan.launch()
        apm.all_minors_ragged(vals[r % 3], n_t, hi, "r64", out=mr)
        apm.all_minors_ragged(vals[(r + 1) % 3], n_t, hi, "r64", out=mdr)
        assert apm.apm_connected_sums(apm._ptr(mr), apm._ptr(mdr), bd, apm._ptr(cr), apm.APM_CS_ROOTED,
                                      apm._stream(None)) == apm.APM_OK
        torch.cuda.synchronize()
        assert _same(m, mr) and _same(md, mdr) and _same(c, cr), r
    plan.close()
