"""The forward sweeps around the edges of their chunks, rings and strips: rows
and columns one below, at and one above 32, 64 and 128, for the variants whose
increments and frontier move in pieces of different widths.  Against the CPU
oracle at the orders' accuracy on smooth short pairs (1e-10, the parity bound),
with every cell counted once."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = ((2, 2), (33, 64), (64, 65), (65, 66), (97, 64), (98, 130), (129, 66), (130, 200),
          (66, 330))


def sk():
    import paper_2502_20392_amd as P
    return P


def T(a, dev):
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


def check(dev, order, d, shape, **kw):
    import oracle
    x = synth.brownian(1, shape[0], d, 0.4 / np.sqrt(d), seed=order + shape[0])[0]
    y = synth.brownian(1, shape[1], d, 0.4 / np.sqrt(d), seed=order + 7 * shape[1])[0]
    ref = oracle.pair(x, y)
    k = sk().pair(T(x, dev), T(y, dev), order=order, **kw).item()
    c = sk().counters()
    assert c["status"] == 0 and c["cells"] == (shape[0] - 1) * (shape[1] - 1), (shape, c)
    assert abs(k - ref) / max(abs(ref), 1.0) < 1e-10, (shape, k, ref)


@pytest.mark.parametrize("order,d", [(8, 3), (8, 16), (10, 3), (10, 16), (12, 3), (12, 16),
                                     (16, 3)])
def test_one_wave_edges(dev, order, d):
    """One wave per workgroup (an explicit grid), both work tiles."""
    for shape in SHAPES:
        for tile in sk().api.tile_options(order, d):
            check(dev, order, d, shape, grid=3, tile=tile)
