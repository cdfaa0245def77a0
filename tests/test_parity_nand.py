"""NAND minors of matrices that the register kernel does not finish by itself: non-finite
input beside pivots below the shift threshold, and pivot shifts at single places of the
tree.  Gate: 1e-10 of the Hadamard bound, as in the other parity tests; outputs are filled
beforehand, so that an entry left unwritten shows."""
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


def _matrices(rng, B, n, cplx, diag):
    A = rng.standard_normal((B, 2 * n, 2 * n)) + diag * np.eye(2 * n)
    return A + 1j * rng.standard_normal(A.shape) if cplx else A


def _nand(apm, A):
    """Outputs (filled with 7 beforehand) and info codes (with 99)."""
    import torch
    B, n = A.shape[0], A.shape[1] // 2
    dA = torch.from_numpy(A).cuda()
    out = torch.full((B, 3 ** n), 7.0, dtype=dA.dtype, device="cuda")
    info = torch.full((B,), 99, dtype=torch.int32, device="cuda")
    rc = apm.apm_nand_minors(apm.APM_C128 if A.dtype.kind == "c" else apm.APM_R64, apm._ptr(dA), apm.make_batch(B, n),
                             apm._ptr(out), apm._ptr(info), apm._stream(None))
    assert rc == apm.APM_OK
    torch.cuda.synchronize()
    return out.cpu().numpy(), info.cpu().numpy()


def _bound(A):
    n = A.shape[0] // 2
    ln = np.log(np.maximum(np.linalg.norm(A, axis=1), 1e-300))
    lt = np.stack([np.zeros(n), ln[0::2], ln[1::2]], axis=1)
    digits = (np.arange(3 ** n)[:, None] // 3 ** np.arange(n)[None, :]) % 3
    return np.exp(lt[np.arange(n)[None, :], digits].sum(axis=1))


def _check(oracle_mod, got, A, what):
    e = metrics.mixed_err(got, oracle_mod.nand_minors(A), _bound(A))
    assert e.max() <= GATE, (what, float(e.max()), int(np.argmax(e)))


def _zero_diagonal(A, b):
    i = np.arange(A.shape[-1])
    A[b, i, i] = 0.0


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("n", [7, 8, 9, 11])
def test_lone_non_finite_matrix(apm, n, cplx):
    """A matrix alone in its call, with an Inf in the last block's rows (its pivots are then
    below the threshold) or with a zero diagonal and a NaN: every minor NaN, info -2."""
    rng = np.random.default_rng(3000 + n)
    for kind in ("inf", "nan"):
        A = _matrices(rng, 1, n, cplx, 3.0)
        if kind == "inf":
            A[0, 2 * n - 1, 1] = A[0, 2 * n - 2, 3] = np.inf
        else:
            _zero_diagonal(A, 0)
            A[0, 2, 1] = np.nan
        got, info = _nand(apm, A)
        assert info[0] == -2, (n, cplx, kind, info)
        assert np.all(np.isnan(got)), (n, cplx, kind, int(np.sum(~np.isnan(got))))


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("n,B", [(7, 4), (7, 9), (8, 4), (8, 6)])
def test_non_finite_among_shifted(apm, oracle_mod, n, B, cplx):
    """One non-finite matrix in a batch whose other matrices are shifted throughout."""
    rng = np.random.default_rng(3100 + n)
    A = _matrices(rng, B, n, cplx, 0.0)
    _zero_diagonal(A, np.arange(B)[:, None])
    bad = B // 2
    A[bad, 2, 1] = np.nan
    got, info = _nand(apm, A)
    assert info[bad] == -2 and np.all(np.isnan(got[bad])), (info, int(np.sum(~np.isnan(got[bad]))))
    for b in (0, B - 1):
        assert info[b] > 0
        _check(oracle_mod, got[b], A[b], (n, cplx, b))


@pytest.mark.parametrize("n", [7, 8, 9, 10, 11])
def test_shifts_at_single_places(apm, oracle_mod, n):
    """Matrix b < 2 n has one zero on its diagonal, in row b: that pivot is shifted in the nodes
    that leave every later block out (a level above the parts, inside a part's rows or in its
    lanes, by the block), and most of the tree has no shift.  Then matrices with two such rows,
    of neighbouring and of distant blocks, and a plain one: every entry, and which matrices
    count shifts."""
    rng = np.random.default_rng(3200 + n)
    pairs = [(2 * n - 1, 2 * n - 3), (2 * n - 2, 2 * n - 1), (2 * n - 4, 1), (3, 0), (2 * n - 1, 6)]
    for cplx in (False, True):
        A = _matrices(rng, 2 * n + len(pairs) + 1, n, cplx, 12.0)
        for b in range(2 * n):
            A[b, b, b] = 0.0
        for k, (r, s) in enumerate(pairs):
            A[2 * n + k, r, r] = A[2 * n + k, s, s] = 0.0
        got, info = _nand(apm, A)
        # the rows of the first block are the tree's leaves: a leaf's pivot is not shifted
        first = np.arange(len(A)) < 2
        assert np.all(info >= 0) and np.all(info[:-1][~first[:-1]] > 0), info
        for b in range(len(A)) if n < 10 else (1, 2, 5, 10, 2 * n - 1, 2 * n, 2 * n + 2, 2 * n + 4):
            _check(oracle_mod, got[b], A[b], (n, cplx, b))


def test_every_batch_size_same_bits(apm):
    """A batch with more parts than one pass of the second launch looks at (64 times its grid),
    made of eight matrices over and over (plain, shifted throughout, at one place, non-finite),
    gives the bits of the eight alone, info included; so does the call without info."""
    import torch
    n, rep = 8, 3660
    rng = np.random.default_rng(3300)
    A = _matrices(rng, 8, n, False, 12.0)
    _zero_diagonal(A, 1)
    _zero_diagonal(A, 6)
    for b, r in ((2, 15), (3, 9), (4, 4)):
        A[b, r, r] = 0.0
    A[5, 3, 2] = np.nan
    dA = torch.from_numpy(A).cuda()
    want, info = apm.nand_minors(dA)
    out = torch.full((8 * rep, 3 ** n), 7.0, dtype=torch.float64, device="cuda")
    big, binfo = apm.nand_minors(dA.repeat(rep, 1, 1), out=out)
    torch.cuda.synchronize()
    assert info.tolist()[5] == -2 and all(info[b] > 0 for b in (1, 2, 3, 4, 6)) and info[0] == info[7] == 0
    assert torch.equal(binfo.view(rep, 8), info.expand(rep, 8))
    assert torch.equal(big.view(torch.int64).view(rep, 8, -1), want.view(torch.int64).expand(rep, 8, 3 ** n))
    out2 = torch.full_like(want, 7.0)
    assert apm.apm_nand_minors(apm.APM_R64, apm._ptr(dA), apm.make_batch(8, n), apm._ptr(out2), None,
                               apm._stream(None)) == apm.APM_OK
    assert torch.equal(out2.view(torch.int64), want.view(torch.int64))


@pytest.mark.parametrize("n", [7, 10])
def test_captured_with_shifts(apm, n):
    """A captured call (its workspace sized by an eager one) replayed on new inputs, plain and
    shifted in turn, with eager work between, equals the eager call."""
    import torch
    rng = np.random.default_rng(3400 + n)
    plain = _matrices(rng, 5, n, True, 12.0)
    mixed = plain.copy()
    _zero_diagonal(mixed, 1)
    mixed[3, 2 * n - 1, 2 * n - 1] = 0.0
    src = [torch.from_numpy(x).cuda() for x in (plain, mixed)]
    want = [apm.nand_minors(s) for s in src]
    dA, out, info = src[0].clone(), torch.zeros_like(want[0][0]), torch.zeros_like(want[0][1])
    bd = apm.make_batch(5, n)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    args = (apm.APM_C128, apm._ptr(dA), bd, apm._ptr(out), apm._ptr(info))
    with torch.cuda.stream(side):
        assert apm.apm_nand_minors(*args, apm._stream(None)) == apm.APM_OK
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        assert apm.apm_nand_minors(*args, apm._stream(None)) == apm.APM_OK
    for k in (1, 0, 1, 1, 0):
        dA.copy_(src[k])
        out.fill_(7.0)
        g.replay()
        eager, _ = apm.nand_minors(src[1 - k])
        torch.cuda.synchronize()
        assert torch.equal(torch.view_as_real(out), torch.view_as_real(want[k][0])) and torch.equal(info, want[k][1])
        assert torch.equal(torch.view_as_real(eager), torch.view_as_real(want[1 - k][0]))


def test_threads_on_one_stream(apm):
    """Four threads call on the same stream (a call is three launches over one workspace), each
    with its own plain and shifted matrices of another size: the results of the calls alone."""
    import threading
    import torch
    rng = np.random.default_rng(3500)
    jobs = []
    for t, (n, B) in enumerate([(7, 40), (8, 9), (7, 3), (9, 5)]):
        A = _matrices(rng, B, n, bool(t & 1), 12.0)
        _zero_diagonal(A, t % B)
        A[-1, 2 * n - 1, 2 * n - 1] = 0.0
        jobs.append(torch.from_numpy(A).cuda())
    want = [apm.nand_minors(A) for A in jobs]
    got = [[] for _ in jobs]
    torch.cuda.synchronize()
    start = threading.Barrier(len(jobs))

    def work(t):
        start.wait()
        for _ in range(30):
            got[t].append(apm.nand_minors(jobs[t]))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for (m, i), res in zip(want, got):
        assert len(res) == 30
        for m1, i1 in res:
            assert torch.equal(i, i1)
            assert torch.equal(m.view(torch.float64) if not m.is_complex() else torch.view_as_real(m),
                               m1 if not m.is_complex() else torch.view_as_real(m1))


@pytest.mark.parametrize("n,cplx", [(10, False), (10, True), (11, False)])
def test_left_out_columns_do_not_enter(apm, oracle_mod, n, cplx):
    """Finite minors next to an overflow in a column that they do not have: row 2n - 2 has a pivot
    of 1e160 and 1e250 in block n - 2's first column, row 0 has 1e250 in the pivot's column, so the
    update of (row 0, that column) overflows.  The rest of row 2n - 2 is 1e-90, so that the
    updates of the other columns are of order 1 and no pivot is shifted there.  (The pivot's
    own square and its row and column scale both overflow in the shift test, which then shifts
    nothing.)  With block n - 2 left out, every minor is 1e160 times an ordinary one."""
    rng = np.random.default_rng(3600 + n)
    A = _matrices(rng, 1, n, cplx, 12.0)
    p, k = 2 * n - 2, 2 * n - 4
    A[0, p] *= 1e-90
    A[0, p, p] = 1e160
    A[0, p, k] = A[0, 0, p] = 1e250
    got, _ = _nand(apm, A)
    ref = oracle_mod.nand_minors(A)[0]
    digits = (np.arange(3 ** n)[:, None] // 3 ** np.arange(n)[None, :]) % 3
    sel = (digits[:, n - 1] == 1) & (digits[:, n - 2] == 0)
    # the Schur complement over the pivot, whose rows bound the minors
    S = A[0].copy()
    S[:, k] = 0.0
    S = S - np.outer(S[:, p] / 1e160, S[p])
    ln = np.log(np.linalg.norm(np.delete(S, p, axis=1), axis=1) + 1e-300)
    lt = np.stack([np.zeros(n), ln[0::2], ln[1::2]], axis=1)
    lt[n - 1, 1] = 0.0
    H = np.exp(lt[np.arange(n)[None, :], digits].sum(axis=1)[sel])
    assert np.all(np.isfinite(ref[sel])) and np.all(np.isfinite(got[0][sel])), int(np.sum(~np.isfinite(got[0][sel])))
    e = metrics.mixed_err(got[0][sel] / 1e160, ref[sel] / 1e160, H)
    assert e.max() <= GATE, float(e.max())


@pytest.mark.parametrize("n,B,cplx", [(7, 8192, False), (7, 2816, True), (8, 4096, False), (8, 2816, True),
                                      (9, 1365, False), (9, 2048, False)])
def test_mostly_shifted_batches_same_bits(apm, n, B, cplx):
    """Batches that fill the chip and are shifted nearly throughout, whose parts go to the
    wavefronts in groups of 3 or 9 (the corrections inside a group are its wavefront's): the bits
    of the same eight matrices alone, whose parts go one by one."""
    import torch
    rng = np.random.default_rng(3700 + n)
    A = _matrices(rng, 8, n, cplx, 12.0)
    for b in (0, 1, 2, 4, 5, 7):
        _zero_diagonal(A, b)
    A[5] *= np.outer(np.exp2(rng.integers(-9, 9, 2 * n)), np.exp2(rng.integers(-9, 9, 2 * n)))
    A[3, 3, 2] = np.nan
    A[6, 2 * n - 1, 2 * n - 1] = 0.0
    dA = torch.from_numpy(A).cuda()
    want, info = apm.nand_minors(dA)
    idx = torch.arange(B, device="cuda") % 8
    out = torch.full((B, 3 ** n), 7.0, dtype=dA.dtype, device="cuda")
    big, binfo = apm.nand_minors(dA[idx].contiguous(), out=out)
    torch.cuda.synchronize()
    assert info.tolist()[3] == -2 and all(info[b] > 0 for b in (0, 1, 2, 4, 5, 6, 7))
    assert torch.equal(binfo, info[idx])
    bits = (lambda t: torch.view_as_real(t).contiguous().view(torch.int64)) if cplx else (lambda t: t.view(torch.int64))
    big, want = bits(big), bits(want)
    for b in range(8):
        assert torch.equal(big[b::8], want[b].expand_as(big[b::8])), (n, cplx, b)
