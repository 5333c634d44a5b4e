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


@pytest.mark.parametrize("order,d", [(4, 2), (5, 8), (6, 3), (8, 16), (10, 3), (10, 16), (12, 3),
                                     (12, 32), (16, 16), (20, 3), (24, 8), (6, 40), (12, 40),
                                     (20, 33)])
def test_team_edges(dev, order, d):
    """Teams of waves (the default for a pair of two strips or more): strips that
    are not a whole team, a last strip of one row, paths shorter than a block of
    steps, several teams in a chain, several pairs.  The same cell maps as the
    one-wave kernel, at Neumann depths chosen over other chunks: equal to a few
    roundings, and both within the parity bound of the oracle."""
    import oracle
    n = 3
    for lx, ly in ((2, 66), (9, 130), (33, 129), (64, 194), (65, 258), (100, 322), (200, 385),
                   (17, 705)):
        X = synth.brownian(n, lx, d, 0.05 if order == 4 else 0.4 / np.sqrt(d), seed=order + lx)
        Y = synth.brownian(2, ly, d, 0.05 if order == 4 else 0.4 / np.sqrt(d), seed=order + ly)
        G = sk().gram(T(X, dev), T(Y, dev), order=order).cpu().numpy()
        c = sk().counters()
        assert not c["status"] & ~1 and c["cells"] == 2 * n * (lx - 1) * (ly - 1), (lx, ly, c)
        G1 = sk().gram(T(X, dev), T(Y, dev), order=order, grid=5).cpu().numpy()
        assert sk().counters()["status"] == c["status"], (lx, ly)
        assert np.max(np.abs(G - G1) / np.maximum(np.abs(G1), 1.0)) < 1e-12, (lx, ly)
        if c["status"] & 1:  # the order is too small for this pair: no parity promised
            continue
        ref = np.array([[oracle.pair(x, y) for y in Y] for x in X])
        assert np.max(np.abs(G - ref) / np.maximum(np.abs(ref), 1.0)) < 1e-10, (lx, ly)


def test_team_nonfinite(dev):
    """A non-finite point anywhere in a pair of several strips still raises the status."""
    X = synth.brownian(1, 150, 3, 0.5, seed=1)[0]
    Y = synth.brownian(1, 300, 3, 0.5, seed=2)[0]
    for which, row in (("x", 0), ("x", 149), ("y", 5), ("y", 299)):
        x, y = X.copy(), Y.copy()
        (x if which == "x" else y)[row, 1] = np.nan
        k = sk().pair(T(x, dev), T(y, dev), order=8).item()
        assert not np.isfinite(k) and sk().counters()["status"] & 2, (which, row)


@pytest.mark.parametrize("scale", [0.02, 1.0])
@pytest.mark.parametrize("npairs", [1, 63, 513, 4096, 4100])
def test_truncation_check_batch_sizes(dev, npairs, scale):
    """The end-of-launch check over one pair (whose wave sets the header itself),
    several loads of estimates and more pairs than the launch checks itself: one
    rough pair among smooth ones counts wherever it stands, and a workspace full
    of another call's bytes changes nothing.  Expected from the per-pair
    estimates of a plan."""
    x = scale * synth.brownian(1, 9, 2, 1.0, seed=5)
    smooth = synth.brownian(npairs, 9, 2, 0.02, seed=6)
    off = np.arange(npairs + 2, dtype=np.int64) * 9
    pairs = np.stack([np.zeros(npairs), 1 + np.arange(npairs)], 1).astype(np.int32)
    plan = sk().RaggedPlan(off, pairs, 2, order=6, device=dev)
    for at in sorted({0, npairs // 2, npairs - 1}):
        Y = smooth.copy()
        rough = Y.copy()
        rough[at] *= 200.0
        ws = torch.full((1 << 22,), 255, dtype=torch.uint8, device=dev)
        for B in (Y, rough, Y):
            plan.run(T(np.concatenate([x, B]).reshape(-1, 2), dev))
            est = plan.estimates().max().item()
            sk().gram(T(x, dev), T(B, dev), order=6, ws=ws)
            c = sk().counters(ws)
            assert c["status"] == int(est > 2.0 ** -36), (at, est, c)
            assert c["cells"] == 64 * npairs and c["order"] == 6, c
            assert abs(c["trunc_est"] - est) <= 1e-12 * est, (est, c)


@pytest.mark.parametrize("order,d", [(5, 3), (8, 8), (10, 3), (10, 16), (12, 3), (16, 3), (24, 3)])
@pytest.mark.parametrize("scale", [0.4, 3.0])
def test_adjoint_two_waves(dev, order, d, scale):
    """The adjoint with a second wave for the recompute (few strips) against the
    one-wave kernel (an explicit grid): rows of one column, one segment, segment
    and chunk edges, several strips, smooth and rough segments.  The same sums,
    and atomics in another order: equal to 1e-12 of the largest component."""
    lens = [(2, 3), (16, 70), (17, 65), (18, 64), (49, 130), (64, 66), (65, 100), (97, 129),
            (130, 200)]
    rows = [l for p in lens for l in p]
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
    pool = np.concatenate([synth.brownian(1, l, d, scale / np.sqrt(d), seed=order + 3 * l + k)[0]
                           for k, l in enumerate(rows)])
    pairs = np.arange(len(rows), dtype=np.int32).reshape(-1, 2)
    go = torch.linspace(-1.0, 1.0, len(pairs), dtype=torch.float64, device=dev)
    got = []
    for grid in (0, 7):
        plan = sk().RaggedPlan(off, pairs, d, order=order, grid=grid, device=dev)
        got.append(plan.backward(T(pool, dev), go).cpu().numpy())
        c = sk().counters(plan.ws)
        assert not c["status"] & ~1, c
        assert c["bwd_cells"] == sum((a - 1) * (b - 1) for a, b in lens), c
    assert np.max(np.abs(got[0] - got[1])) <= 1e-12 * np.max(np.abs(got[1]))


@pytest.mark.parametrize("order,d", [(5, 3), (10, 3), (10, 16), (12, 3), (12, 16), (16, 3),
                                     (20, 16)])
def test_narrow_tile_same_values(dev, order, d):
    """Where the default tile is 64 columns wide, a plan whose launch is bound by
    its chains takes the 32-column one by itself: the same Neumann depths and
    cell maps, so the same bits as either explicit tile."""
    lens = [(17, 70), (40, 65), (64, 200), (65, 129), (97, 64), (130, 300), (333, 66)]
    rows = [l for p in lens for l in p]
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
    pool = np.concatenate([synth.brownian(1, l, d, 0.5 / np.sqrt(d), seed=order + 5 * l + k)[0]
                           for k, l in enumerate(rows)])
    pairs = np.arange(len(rows), dtype=np.int32).reshape(-1, 2)
    assert sk().api.tile_options(order, d) == [64, 32]
    got = [sk().RaggedPlan(off, pairs, d, order=order, tile=tile, device=dev).run(T(pool, dev))
           for tile in (0, 32, 64)]
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])


@pytest.mark.parametrize("order,d,nx,ny,lx,ly", [(10, 3, 24, 0, 257, 257), (10, 16, 40, 9, 131, 300),
                                                 (12, 8, 25, 13, 193, 322), (12, 3, 24, 0, 190, 190)])
def test_gram_tile_rule_same_values(dev, order, d, nx, ny, lx, ly):
    """A Gram call with more strips than SIMDs whose chains still bound it takes the
    narrow tile by itself (variants of two waves per SIMD): the bits of the wide one."""
    X = T(synth.brownian(nx, lx, d, 0.5 / np.sqrt(d), seed=order + lx), dev)
    Y = T(synth.brownian(ny, ly, d, 0.5 / np.sqrt(d), seed=order + ly), dev) if ny else None
    got = sk().gram(X, Y, order=order)
    for tile in (32, 64):
        assert torch.equal(got, sk().gram(X, Y, order=order, tile=tile)), tile
