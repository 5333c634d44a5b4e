"""Autograd calls on small batches wait for nothing on the host: no copy from
ordinary memory after the first launch and no stream synchronisation, and the
tables of a plan that is gone before its launches run have been taken."""
import contextlib

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def sk():
    import paper_2502_20392_amd as P
    return P


@contextlib.contextmanager
def no_host_waits(monkeypatch):
    """Host waits fail: torch's synchronising copies, and stream.synchronize()."""
    def refuse(self):
        raise AssertionError("the host waits for a stream")
    with monkeypatch.context() as m:
        m.setattr(torch.cuda.Stream, "synchronize", refuse)
        torch.cuda.set_sync_debug_mode("error")
        try:
            yield
        finally:
            torch.cuda.set_sync_debug_mode("default")


def sets(dev, n, length, d):
    X = synth.brownian(2 * n, length, d, 0.5 / np.sqrt(d), seed=n + length)
    return (torch.from_numpy(X[:n]).to(dev), torch.from_numpy(X[n:]).to(dev))


@pytest.mark.parametrize("which", ["gram", "cross", "mmd2", "mmd2_both"])
def test_no_host_waits(dev, which, monkeypatch):
    X, Y = sets(dev, 6, 50, 3)
    X.requires_grad_(True)
    if which == "mmd2_both":
        Y.requires_grad_(True)
    with no_host_waits(monkeypatch):
        for _ in range(2):
            X.grad = None
            if which == "gram":
                sk().sigkernel_gram(X, order=8).sum().backward()
            elif which == "cross":
                sk().sigkernel_gram(X, Y, order=8).sum().backward()
            else:
                sk().mmd2(X, Y, order=8).backward()
    assert X.grad is not None


def test_mmd2_weights_and_gradient(dev):
    """The estimator's weights, against its definition from Gram matrices."""
    for nx, ny in ((3, 5), (4, 4), (1, 2)):
        A = synth.brownian(nx + ny, 40, 2, 0.5, seed=nx)
        X = torch.from_numpy(A[:nx]).to(dev).requires_grad_(True)
        Y = torch.from_numpy(A[nx:]).to(dev).requires_grad_(True)
        v = sk().mmd2(X, Y, order=10)
        v.backward()
        got = v.item(), X.grad.clone(), Y.grad.clone()
        X.grad = Y.grad = None
        w = (sk().sigkernel_gram(X, order=10).mean() + sk().sigkernel_gram(Y, order=10).mean()
             - 2 * sk().sigkernel_gram(X, Y, order=10).mean())
        w.backward()
        assert abs(got[0] - w.item()) < 1e-13 * 4
        for a, b in zip(got[1:], (X.grad, Y.grad)):
            assert (a - b).abs().max().item() <= 1e-12 * max(b.abs().max().item(), 1e-3)


@pytest.mark.parametrize("n", [20, 40])
def test_plan_gone_before_its_launches(dev, n):
    """Forward and backward on a side stream that is still busy: the plan (tables of
    20 KB, sent as kernel arguments, and of 79 KB, copied) and its Python object
    are gone before the stream reaches the launches."""
    X, _ = sets(dev, n, 70, 3)
    Xg = X.clone().requires_grad_(True)
    want = sk().sigkernel_gram(Xg, order=8)
    want.sum().backward()
    want, want_g = want.detach(), Xg.grad
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    busy = torch.zeros(1 << 26, device=dev)
    for _ in range(3):
        with torch.cuda.stream(s):
            for _ in range(20):
                busy.add_(1.0)
            Z = X.clone().requires_grad_(True)
            G = sk().sigkernel_gram(Z, order=8)
            G.sum().backward()
            value, grad = G.detach().clone(), Z.grad.clone()
            del G, Z
            # other plans, whose host tables may reuse the memory
            for k in range(3):
                sk().RaggedPlan(np.arange(n + 1) * 3, np.zeros((n * n // 2 + k, 2), np.int32), 3,
                                device=dev)
        torch.cuda.synchronize()
        assert torch.equal(value, want)
        assert (grad - want_g).abs().max().item() <= 1e-12 * want_g.abs().max().item()
