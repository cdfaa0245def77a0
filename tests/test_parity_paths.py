"""GPU parity at the edges of the kernels' partitions: batches that leave units of several
matrices partly filled or fill the chip with items of one matrix, the smallest and largest
sizes of a path, and matrices with errors or pivot shifts beside plain ones.  The gates are
those of the other parity tests: 1e-10 of the Hadamard bound (minors) and of the
recursion's own rounding scale (connected sums); minors of split matrices equal the unsplit
ones bit for bit, since every item performs the same operations."""
import numpy as np
import pytest

from oracle import metrics

pytestmark = pytest.mark.gpu
GATE = 1e-10


@pytest.fixture(scope="module")
def apm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2104_07638_amd as m
    return m


def _gauss(rng, shape, cplx, diag):
    A = rng.standard_normal(shape) + diag * np.eye(shape[-1])
    return A + 1j * rng.standard_normal(shape) if cplx else A


def _row_bound(A, mode):
    """Hadamard bound of every entry from the full rows' norms, in output order."""
    n = A.shape[0] // 2
    ln = np.log(np.maximum(np.linalg.norm(A, axis=1), 1e-300))
    if mode == "xor":
        out = []
        for k in range(1, n + 1):
            bits = (np.arange(1 << k)[:, None] >> np.arange(k)[None, :]) & 1
            out.append(np.exp(ln[2 * (n - k + np.arange(k))[None, :] + bits].sum(axis=1)))
        return np.concatenate(out)
    if mode == "xnor":
        bits = (np.arange(1 << n)[:, None] >> np.arange(n)[None, :]) & 1
        return np.exp(bits @ (ln[0::2] + ln[1::2]))
    digits = (np.arange(3 ** n)[:, None] // 3 ** np.arange(n)[None, :]) % 3
    lt = np.stack([np.zeros(n), ln[0::2], ln[1::2]], axis=1)
    return np.exp(lt[np.arange(n)[None, :], digits].sum(axis=1))


@pytest.mark.parametrize("mode,n,B", [("xor", 4, 1), ("xor", 4, 70), ("xor", 7, 5), ("xor", 8, 3), ("xor", 9, 33),
                                      ("xor", 11, 2), ("xnor", 4, 67), ("xnor", 7, 3), ("xnor", 8, 5), ("xnor", 9, 33),
                                      ("xnor", 11, 3), ("nand", 7, 5), ("nand", 8, 3), ("nand", 9, 6)])
def test_block_minors(apm, oracle_mod, mode, n, B):
    """Real and complex; from three matrices on one has a NaN, one a zero pivot (XOR: in every
    path; NAND: shifted), between plain ones."""
    import torch
    rng = np.random.default_rng(2000 + 100 * n + B)
    call = getattr(apm, mode + "_minors")
    for cplx in (False, True):
        A = _gauss(rng, (B, 2 * n, 2 * n), cplx, 3.0)
        if B >= 3:
            A[1, 2, 1] = np.nan
            if mode == "xor":
                A[2, 2 * n - 1, 2 * n - 1] = 0.0
            if mode == "nand":
                A[2, np.arange(2 * n), np.arange(2 * n)] = 0.0
        out, info = call(torch.from_numpy(A).cuda())
        torch.cuda.synchronize()
        got, info = out.cpu().numpy(), info.cpu().numpy()
        if B >= 3:
            assert info[1] == -2 and np.all(np.isnan(got[1].real))
            assert mode != "xor" or info[2] == -3
            assert mode != "nand" or info[2] > 0
        for b in sorted({0, 2, B // 2, B - 2, B - 1} & set(range(B))):
            if info[b] < 0:
                continue
            assert b == 2 or mode == "nand" or info[b] == 0
            ref = getattr(oracle_mod, mode + "_minors")(A[b])
            e = metrics.mixed_err(got[b], ref, _row_bound(A[b], mode))
            assert e.max() <= GATE, (mode, n, cplx, b, float(e.max()), int(np.argmax(e)))


@pytest.mark.parametrize("n,B", [(4, 1), (5, 3), (15, 6), (16, 5), (17, 2), (31, 3), (32, 7)])
def test_leading_batches(apm, oracle_mod, n, B):
    """Batches that leave a wavefront's four matrices partly filled."""
    import torch
    rng = np.random.default_rng(2100 + n)
    for cplx in (False, True):
        A = _gauss(rng, (B, n, n), cplx, 2.0)
        if B >= 3:
            A[1, n - 1, 0] = np.nan
            A[2, 0, 0] = 0.0
        out, info = apm.leading_minors(torch.from_numpy(A).cuda())
        torch.cuda.synchronize()
        got, info = out.cpu().numpy(), info.cpu().numpy()
        for b in range(B):
            if B >= 3 and b in (1, 2):
                assert info[b] < 0
                continue
            assert info[b] == 0
            had = np.array([np.prod(np.linalg.norm(A[b, :k, :k], axis=1)) for k in range(1, n + 1)])
            e = metrics.mixed_err(got[b], oracle_mod.leading_minors(A[b]), had)
            assert e.max() <= GATE, (n, cplx, b, float(e.max()))


@pytest.mark.parametrize("n,B,kind", [(7, 3, "pair"), (10, 5, "square"), (11, 2, "pair"), (12, 3, "given"),
                                      (12, 3, "square"), (13, 2, "pair"), (14, 1, "square"), (15, 1, "pair")])
def test_sums(apm, oracle_mod, n, B, kind):
    """The three kinds of weights, rooted and with all roots, on one wavefront (up to 11
    vertices), one block (12) and several."""
    import torch
    rng = np.random.default_rng(2200 + n)
    up, dn = rng.standard_normal((2, B, 1 << n))
    a = {"given": up, "square": up * up, "pair": up * dn}[kind]
    tu, td = torch.from_numpy(up).cuda(), torch.from_numpy(dn).cuda()
    for mode in (apm.APM_CS_ROOTED, apm.APM_CS_ALL) if n <= 14 else (apm.APM_CS_ROOTED,):
        c = apm.connected_sums(tu, td if kind == "pair" else None, mode=mode, weights=kind == "given")
        torch.cuda.synchronize()
        ref = oracle_mod.connected_sums(a, mode)
        d = oracle_mod.cs_scale(a, ref, mode)
        err = np.abs(c.cpu().numpy() - ref)
        assert np.all(err <= GATE * d + 1e-300), (n, kind, mode, float(np.max(err / np.maximum(d, 1e-300))))


def test_sums_mixed_all_roots(apm, oracle_mod):
    """Orders 1 to 13 in one batch with all roots, at odd offsets."""
    import torch
    rng = np.random.default_rng(2300)
    ns = np.array([5, 13, 1, 9, 12, 2, 10, 8, 11], dtype=np.int32)
    size = 1 << ns.astype(np.int64)
    offs = np.concatenate([[0], np.cumsum(size + 1)[:-1]]) + 3
    a = rng.standard_normal(int(offs[-1] + size[-1]))
    up, ot = torch.from_numpy(a).cuda(), torch.from_numpy(offs).cuda()
    for mode in (apm.APM_CS_ROOTED, apm.APM_CS_ALL):
        c = torch.full_like(up, 7.0)
        bd = apm.make_batch(len(ns), 0, torch.from_numpy(ns).cuda(), 13, ot, ot)
        rc = apm.apm_connected_sums(apm._ptr(up), None, bd, apm._ptr(c), mode | apm.APM_CS_WEIGHTS, apm._stream(None))
        assert rc == 0
        torch.cuda.synchronize()
        got = c.cpu().numpy()
        for n, o in zip(ns, offs):
            s = slice(int(o), int(o) + (1 << int(n)))
            ref = oracle_mod.connected_sums(a[s], mode)
            d = oracle_mod.cs_scale(a[s], ref, mode)
            assert np.all(np.abs(got[s] - ref) <= GATE * d + 1e-300), (mode, int(n))
            assert got[int(o) - 1] == 7.0


@pytest.mark.parametrize("dtype,n,B", [("r64", 12, 1), ("r64", 13, 70), ("r64", 16, 3), ("r64", 17, 2), ("r64", 18, 1),
                                       ("r32s", 16, 2), ("r32s", 17, 2), ("c128", 12, 5), ("c128", 14, 3),
                                       ("c128", 14, 450), ("c128", 15, 2), ("c128", 17, 1), ("c64s", 15, 3),
                                       ("c64s", 17, 1)])
def test_split_minors_match_unsplit(apm, dtype, n, B):
    """Small batches (up to 32 items a matrix) and orders with more than five top levels (items
    that correct their own levels): plain, zero-diagonal (shifted at every level) and
    non-finite matrices against the call that takes one item per matrix."""
    import torch
    dt = apm.DTYPES[dtype]
    cplx, scaled = dtype[0] == "c", dtype[-1] == "s"
    rng = np.random.default_rng(2400 + n)
    A = _gauss(rng, (B, n, n), cplx, 0.0)
    if B > 1:
        A[1, np.arange(n), np.arange(n)] = 0.0
    if B > 2:
        A[2, n - 1, 1] = np.inf
    tA = torch.from_numpy(A).cuda()
    vt = {(False, False): torch.float64, (True, False): torch.complex128, (False, True): torch.float32,
          (True, True): torch.complex64}[(cplx, scaled)]
    got = []
    for call in (apm.apm_all_minors, apm.apm_all_minors_noalloc):
        m = torch.zeros((B, 1 << n), dtype=vt, device="cuda")
        ex = torch.zeros((B, 1 << n), dtype=torch.int16, device="cuda") if scaled else None
        info = torch.zeros(B, dtype=torch.int32, device="cuda")
        assert call(dt, apm._ptr(tA), apm.make_batch(B, n), apm._ptr(m), apm._ptr(ex), apm._ptr(info),
                    apm.apm_opts(0.0, 0), apm._stream(None)) == apm.APM_OK
        torch.cuda.synchronize()
        got.append((m, ex, info))
    (m0, e0, i0), (m1, e1, i1) = got
    assert torch.equal(i0, i1), (i0[:8], i1[:8])
    assert B < 2 or int(i0[1]) > 0
    assert B < 3 or int(i0[2]) == -2
    v0, v1 = (torch.view_as_real(m) if cplx else m for m in (m0, m1))
    assert torch.equal(torch.nan_to_num(v0, nan=3.25), torch.nan_to_num(v1, nan=3.25))
    assert e0 is None or torch.equal(e0[[b for b in range(B) if b != 2]], e1[[b for b in range(B) if b != 2]])


def test_plan_direct_and_captured(apm):
    """A plan of few kernels is launched directly; recorded in a caller's graph and replayed, with
    eager work between the replays, it gives the same results."""
    import torch
    rng = np.random.default_rng(2500)
    A = torch.from_numpy(rng.standard_normal((9, 6, 6))).cuda()
    m = torch.empty((9, 64), dtype=torch.float64, device="cuda")
    c = torch.empty_like(m)
    plan = apm.plan_cdet(A, m, c)
    assert plan.graphed
    plan.launch()
    torch.cuda.synchronize()
    want = c.clone()
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        plan.launch()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        plan.launch()
    for _ in range(3):
        c.zero_()
        plan.launch()
        torch.cuda.synchronize()
        assert torch.equal(c, want)
        c.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(c, want)


@pytest.mark.parametrize("d_in,d_out,B", [(1, 1, 32), (16, 17, 544), (17, 300, 32), (64, 33, 1056)])
def test_mlp_gradients(apm, d_in, d_out, B):
    """Batches that leave the weight gradients' blocks of 512 rows partly filled, inputs of one
    to four tiles, outputs that leave a tile or a pair of tiles partly filled.  Operands enter
    as BF16 (relative 2^-9 each): 2e-2 of the gradient's norm, as in the other network tests."""
    import torch
    from oracle import mlp as omlp
    rng = np.random.default_rng(2600 + d_in)
    dp, op = omlp.dims(d_in, d_out)
    net = apm.Mlp(d_in, d_out)
    shapes = [(128, dp), (128, 128), (op, 128), (128,), (128,), (op,)]
    parts = [np.zeros(s) for s in shapes]
    parts[0][:, :d_in] = 0.5 * rng.standard_normal((128, d_in)) / np.sqrt(d_in)
    parts[1][:] = rng.standard_normal((128, 128)) / np.sqrt(128)
    parts[2][:d_out] = rng.standard_normal((d_out, 128)) / np.sqrt(128)
    p = np.concatenate([v.ravel() for v in parts]).astype(np.float32)
    net.param.copy_(torch.from_numpy(p))
    net.sync()
    x = np.zeros((B, dp), dtype=np.float32)
    x[:, :d_in] = rng.uniform(0, 1, (B, d_in))
    xb = torch.from_numpy(x).to(torch.bfloat16)
    dout = np.zeros((B, op), dtype=np.float32)
    dout[:, :d_out] = rng.standard_normal((B, d_out))
    work = net.work(B)
    net.forward(xb.cuda(), work=work)
    net.backward(torch.from_numpy(dout).cuda(), work)
    got = omlp.unpack(net.grad.cpu().numpy().astype(np.float64), d_in, d_out)
    _, cache = omlp.forward(p.astype(np.float64), xb.to(torch.float64).numpy(), d_in, d_out)
    ref = omlp.unpack(omlp.backward(cache, dout.astype(np.float64)), d_in, d_out)
    for name, a, b in zip(("W1", "W2", "W3", "b1", "b2", "b3"), got, ref):
        err = np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30)
        assert err <= 2e-2, (name, err)
