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
