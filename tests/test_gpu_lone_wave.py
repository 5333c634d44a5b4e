"""The 64-column tile in its form of one wave per SIMD: the bits of the form of
two and of the narrow tile, around the edges of chunks, rings and strips, and the
oracle's values at the orders' accuracy (1e-10, the parity bound)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = ((2, 2), (33, 64), (64, 65), (65, 66), (97, 130), (129, 66), (130, 200), (66, 330))


def sk():
    import paper_2502_20392_amd as P
    return P


@pytest.mark.parametrize("order,d", [(8, 16), (10, 3), (10, 16), (12, 8)])
def test_same_values_in_every_form(dev, order, d):
    import oracle
    rows = [n for s in SHAPES for n in s]
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
    paths = [synth.brownian(1, n, d, 0.4 / np.sqrt(d), seed=order + 5 * n + k)[0]
             for k, n in enumerate(rows)]
    pool = torch.from_numpy(np.concatenate(paths)).to(dev)
    pairs = np.arange(len(rows), dtype=np.int32).reshape(-1, 2)
    cells = sum((a - 1) * (b - 1) for a, b in SHAPES)

    def run(copies=1, **kw):
        plan = sk().RaggedPlan(off, np.tile(pairs, (copies, 1)), d, order=order, device=dev, **kw)
        out = plan.run(pool)
        c = sk().counters(plan.ws)
        assert c["status"] == 0 and c["cells"] == copies * cells, (kw, c)
        return out

    lone = run(tile=64, grid=3)
    assert torch.equal(run(tile=64), lone)
    # many pairs: two waves per SIMD
    assert torch.equal(run(copies=1000, tile=64), lone.repeat(1000))
    if order > 8:  # order 8's narrow tile sets its depths over other columns
        for kw in (dict(), dict(tile=32), dict(tile=32, grid=3)):
            assert torch.equal(run(**kw), lone), kw
    ref = np.array([oracle.pair(paths[2 * k], paths[2 * k + 1]) for k in range(len(SHAPES))])
    assert np.max(np.abs(lone.cpu().numpy() - ref) / np.maximum(np.abs(ref), 1.0)) < 1e-10
