"""The gradient of a long pair in whatever workspace it is given: the caller's
own, from the least-memory blocks' size up, and a smaller one where the
recommended cannot be allocated."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def sk():
    import paper_2502_20392_amd as P
    return P


def setup(dev, n, d, order):
    X = synth.brownian(2, n, d, 0.5 / np.sqrt(d), seed=order + n)
    x, y = (torch.from_numpy(a).to(dev) for a in X)
    rows = max(64, round((14.2 * (n - 1)) ** 0.5 / 64) * 64)
    least, _ = sk().pair_backward_workspace_size(n, n, d, order=order, block_rows=rows)
    roomy, _ = sk().pair_backward_workspace_size(n, n, d, order=order)
    assert least < roomy
    return x, y, least, roomy


def same(a, b):
    # the same cell maps; atomics and Neumann depths in another order
    for u, v in zip(a, b):
        assert (u - v).abs().max().item() <= 1e-12 * max(v.abs().max().item(), 1.0)


@pytest.mark.parametrize("order,d,n", [(5, 8, 1500), (10, 3, 1200), (10, 16, 700)])
def test_callers_workspace_is_used(dev, order, d, n):
    x, y, least, roomy = setup(dev, n, d, order)
    want = sk().pair_backward(x, y, order=order)
    for size in (least, (least + roomy) // 2, roomy):
        ws = torch.full((size,), 255, dtype=torch.uint8, device=dev)
        same(sk().pair_backward(x, y, order=order, ws=ws), want)
        assert sk().last_workspace() is ws
        c = sk().counters(ws)
        assert c["status"] == 0 and c["bwd_cells"] == (n - 1) ** 2, c
    small = torch.zeros(least - 1, dtype=torch.uint8, device=dev)
    same(sk().pair_backward(x, y, order=order, ws=small), want)
    assert sk().last_workspace() is not small


def test_smaller_workspace_where_memory_is_short(dev, monkeypatch):
    x, y, least, roomy = setup(dev, 1500, 8, 5)
    want = sk().pair_backward(x, y, order=5)
    real = sk().api.workspace
    for limit, fits in ((roomy - 1, True), (2 * least, True), (least // 2, False)):
        def short(nbytes, device, limit=limit):
            if nbytes > limit:
                raise torch.cuda.OutOfMemoryError("out of memory")
            return real(nbytes, device)
        monkeypatch.setattr(sk().api, "workspace", short)
        if fits:
            same(sk().pair_backward(x, y, order=5), want)
            assert sk().last_workspace().numel() <= limit
        else:
            with pytest.raises(torch.cuda.OutOfMemoryError):
                sk().pair_backward(x, y, order=5)
