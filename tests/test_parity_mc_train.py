"""The training step's gradient, which is formed inside the backward kernel from the two picked
outputs of every walker: batches of one workgroup, of partly filled blocks of 512 rows, of blocks
that come round in the weight gradients' two buffers (more than 1024 rows) and of the
benchmark's 8192, and orders above 12 (the largest log|c'| from a launch of its own).

The reference takes the step's own log|c'|, with walkers whose weight is unresolved (-inf) among
them, and the logits of the forward kernel, so that the output gradient is known to the bit: g =
bf16(2 (pred - y) / W) at the proposed site's and bin's outputs of each row.
  * b3: sums of at most cnt values g in fp32: cnt 2^-23 of the sum of |g|.
  * W3: the same sums times activations (at most 1, BF16 and from BF16 products: 2e-2, as in the
    other network tests); outputs that no walker picks: exactly zero.
  * W2, W1, b2, b1: 2e-2 of the norm, as in the other network tests; the loss: 1e-6."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import mlp as omlp
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def apm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2104_07638_amd as m
    return m


@pytest.mark.parametrize("n,W", [(10, 32), (10, 512), (10, 544), (10, 1056), (10, 2080), (10, 8192), (12, 96), (13, 288)])
def test_picked_gradient(apm, n, W):
    model = wl.McModel(n=n, L=16, mu=0.0, beta=4.0, n_tau=128, n_bin=16, eps=1.0, resolve=1e-10)
    g0 = torch.from_numpy(wl.mc_g0_table(model)).cuda()
    m = apm.mc_model(model.n, model.L, model.n_tau, model.n_bin, model.eps, g0, model.resolve)
    # a quarter of the walkers spread over the lattice: their weights are below the resolution
    states = wl.mc_cluster_states(W, model, seed=50 + n)
    states[::4] = wl.mc_initial_states(W, model, seed=51 + n)[::4]
    chain = apm.McChain(states)
    p = wl.mlp_init(model.d_in, model.d_out, seed=52)
    net = apm.Mlp(model.d_in, model.d_out, p)
    work = apm.mc_work(m, W, True)
    apm.mc_evaluate(m, chain, work)
    dp, op = omlp.dims(model.d_in, model.d_out)
    moved = torch.empty(W, dtype=torch.int32, device="cuda")
    feat = torch.zeros((W, dp), dtype=torch.bfloat16, device="cuda")
    assert apm.apm_mc_context(m, chain.c, 9, 0, moved.data_ptr(), feat.data_ptr(), None) == apm.APM_OK
    logits = net.forward(feat).cpu().numpy().astype(np.float64).reshape(W, op)
    rec = apm.McRecord(W)
    apm.mc_step(m, chain, work, seed=9, step=0, net=net, train=dict(lr=1e-3, t=1), record=rec)
    torch.cuda.synchronize()

    y = rec.logc_prop.cpu().numpy().copy()
    fin = np.isfinite(y)
    assert fin.any() and (W < 512 or not fin.all())
    floor = y[fin].max() - 30.0
    y = np.where(fin, np.maximum(y, floor), floor)
    v = rec.proposed.cpu().numpy().view(np.uint32)
    f1 = (v & 0xFFFF).astype(np.int64)
    f2 = model.L ** 2 + (v >> 16).astype(np.int64) // (model.n_tau // model.n_bin)
    r = np.arange(W)
    diff = logits[r, f1] + logits[r, f2] - y
    g = torch.from_numpy((2.0 * diff / W).astype(np.float32)).to(torch.bfloat16).double().numpy()
    assert abs(rec.loss.cpu().item() - np.mean(diff ** 2)) <= 1e-6 * np.mean(diff ** 2)
    dout = np.zeros((W, op))
    dout[r, f1] += g
    dout[r, f2] += g
    total = np.abs(dout).sum(axis=0)                      # of |g| by output
    cnt = (dout != 0.0).sum(axis=0)

    x = feat.double().cpu().numpy()
    _, cache = omlp.forward(p.astype(np.float64), x, model.d_in, model.d_out)
    ref = omlp.unpack(omlp.backward(cache, dout), model.d_in, model.d_out)
    got = omlp.unpack(net.grad.cpu().numpy().astype(np.float64), model.d_in, model.d_out)
    for name, a, b in zip(("W1", "W2", "W3", "b1", "b2", "b3"), got, ref):
        if name == "b3":
            err, tol = np.abs(a - b), cnt[:len(b)] * 2.0 ** -23 * total[:len(b)]
            assert np.all(err <= tol), (name, int(np.argmax(err - tol)), float((err - tol).max()))
        elif name == "W3":
            err, tol = np.abs(a - b).max(axis=1), 2e-2 * total[:len(b)]
            assert np.all(err <= tol), (name, int(np.argmax(err - tol)), float((err - tol).max()))
        else:
            e = np.linalg.norm(a - b) / np.linalg.norm(b)
            assert e <= 2e-2, (name, e)
