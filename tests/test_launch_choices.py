"""What the host side launches, recorded without a GPU (launch_recorder.py)."""
import os
import re

import numpy as np
import pytest

from launch_recorder import kernels, record

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_one_lds_limit_per_team_kernel():
    """The dynamic LDS limit of a team kernel is the same whatever team sizes are
    launched (it is shared by every host thread), covers each of them, and is not
    set again by later calls."""
    lens = [65 + 64 * k + 1 for k in range(1, 12)]
    jobs = [dict(call="gram", nx=1, lx=n, d=d, order=p)
            for p, d in ((6, 8), (10, 16), (12, 32), (24, 8), (8, 40)) for n in lens]
    res = record(jobs + jobs)
    first, again = res[:len(jobs)], res[len(jobs):]
    limits, used = {}, {}
    for r in first:
        assert r["rc"] == 0
        for what, name, _, block, lds in r["events"]:
            if what == "attribute":
                limits.setdefault(name, set()).add(lds)
            elif name.startswith("team_kernel"):
                used.setdefault(name, set()).add((block, lds))
    assert len(limits) == 5 and all(len(v) == 1 for v in limits.values()), limits
    for name, sizes in used.items():
        assert len(sizes) > 1, (name, sizes)  # several team sizes were launched
        assert max(lds for _, lds in sizes) <= min(limits[name]), name
    assert not any(e[0] == "attribute" for r in again for e in r["events"])


@pytest.mark.parametrize("cus", [32, 64, 128])
def test_first_call_knows_the_device(cus):
    """On a device of fewer CUs the first call of a process launches what every
    later one does (the CU count enters the choice of kernel and grid)."""
    for job in (dict(call="gram", nx=12, lx=300, d=16, order=10),
                dict(call="gram", nx=9, lx=700, d=3, order=12),
                dict(call="gram", nx=5, lx=2000, d=3, order=6)):
        _, first, again, last = record([dict(call="cus", n=cus), job, job, job])
        for r in (first, again, last):
            r["events"] = [e for e in r["events"] if e[0] == "launch"]
        assert first == again == last, (cus, job)


def least_rows(side):
    """Side of the least-memory blocks: sqrt(14.2 side), in whole strips."""
    return max(64, round((14.2 * side) ** 0.5 / 64) * 64)


@pytest.mark.parametrize("order,d,longer,shorter", [(5, 8, 28001, 27001), (8, 8, 22001, 21001),
                                                    (12, 8, 18001, 17001), (10, 16, 20001, 3000)])
def test_pair_backward_takes_the_workspace_it_is_given(order, d, longer, shorter):
    """A workspace sized for a longer pair serves a shorter one, the least-memory
    blocks' bytes serve a call without block sizes (by blocks no smaller than
    those), and far less is refused before anything is launched."""
    q = dict(call="pair_backward", order=order, d=d)
    sized, = record([dict(q, lx=longer, ly=longer, ws=0)])
    rows = least_rows(shorter - 1)
    least, = record([dict(q, lx=shorter, ly=shorter, rows=rows, ws=0)])
    assert least["rc"] == sized["rc"] == 0 and least["bytes"] < sized["bytes"]
    s = dict(q, lx=shorter, ly=shorter)
    fits, tight, explicit, none = record([dict(s, ws=sized["bytes"]), dict(s, ws=least["bytes"]),
                                          dict(s, ws=least["bytes"], rows=rows),
                                          dict(s, ws=least["bytes"] // 2)])
    assert fits["rc"] == tight["rc"] == explicit["rc"] == 0
    # larger blocks are fewer launches
    assert len(fits["events"]) < len(tight["events"]) <= len(explicit["events"])
    assert none["rc"] == -2 and none["events"] == []


def test_truncation_check_is_fused_in_small_launches_only():
    """The last workgroup checks the estimates where few count themselves; larger
    launches, and few workgroups over many pairs, leave it to a kernel of its own."""
    small = [dict(call="gram", nx=n, lx=20, d=3, order=8) for n in (2, 8, 15)]
    small += [dict(call="plan", lens=[300] * 21, pairs=[[i, i + 1] for i in range(20)], d=3,
                   order=10, steps=["run"])]
    large = [dict(call="gram", nx=n, lx=20, d=d, order=p)
             for n, d, p in ((24, 32, 4), (64, 3, 8), (64, 16, 10), (90, 8, 6))]
    large += [dict(call="gram", nx=64, lx=20, d=3, order=8, grid=16),
              dict(call="gram", nx=24, lx=256, d=3, order=6),
              dict(call="plan", lens=[60] * 301, pairs=[[i, i + 1] for i in range(300)], d=3,
                   order=10, steps=["run"])]
    res = record(small + large)
    assert all("finalize_kernel" not in kernels(r) for r in res[:len(small)])
    assert all("finalize_kernel" in kernels(r) for r in res[len(small):])


def forward(result):
    """(kernel, workgroups) of the forward sweep."""
    (e,) = [e for e in result["events"] if e[0] == "launch" and
            e[1].startswith(("fwd_kernel", "team_kernel"))]
    return e[1], e[2]


def pairs_of(n, length, **kw):
    return dict(call="plan", lens=[length] * (n + 1), pairs=[[i, i + 1] for i in range(n)],
                steps=["run"], **kw)


@pytest.mark.parametrize("order,d", [(10, 3), (10, 16), (12, 8)])
def test_one_wave_per_simd_until_the_work_exceeds_the_chain(order, d):
    """Variants whose 64-column tile runs two waves per SIMD: launches far from
    filling the chip take the narrow tile, those whose work is about their chain
    the form of one wave per SIMD, also where the tile or a grid was asked for, as do
    grids of no more waves; large ones run two waves per SIMD."""
    D = 8 if d <= 8 else 16
    narrow, lone, two = (f"fwd_kernel<{order},{D},0,{t}>" for t in ("32,0", "64,1", "64,0"))
    q = dict(order=order, d=d)
    res = record([pairs_of(60, 1024, **q), pairs_of(136, 1024, **q), pairs_of(256, 1024, **q),
                  pairs_of(256, 1024, tile=64, **q), pairs_of(60, 1024, tile=64, **q),
                  pairs_of(600, 1024, grid=512, **q), pairs_of(600, 1024, **q),
                  pairs_of(256, 1024, grid=2048, **q), pairs_of(600, 1024, grid=2048, **q),
                  pairs_of(136, 1024, tile=32, **q),
                  dict(call="gram", nx=22, lx=1024, **q), dict(call="gram", nx=64, lx=1024, **q)])
    got = [forward(r) for r in res]
    assert got == [(narrow, 960), (lone, 1024), (lone, 1024), (lone, 1024), (lone, 960),
                   (lone, 512), (two, 2048), (lone, 2048), (two, 2048), (narrow, 1024),
                   (lone, 1024), (two, 2048)], got


def test_order_8_wide_tile_in_its_form_of_one_wave_per_simd():
    """d 9-16 at order 8 has it on the other tile, for those who ask for it."""
    q = dict(order=8, d=16)
    got = [forward(r)[0] for r in record([
        dict(call="gram", nx=16, lx=1024, tile=64, **q), dict(call="gram", nx=64, lx=512, tile=64, **q),
        pairs_of(136, 1024, **q), pairs_of(136, 1024, tile=32, **q)])]
    assert got == ["fwd_kernel<8,16,0,64,1>", "fwd_kernel<8,16,0,64,0>", "fwd_kernel<8,16,0,32,0>",
                   "fwd_kernel<8,16,0,32,0>"], got


def test_teams_only_where_they_are_the_faster_kernel():
    """Gram calls measured with both kernels: a team's waves must find SIMDs of their
    own also on the CU that holds the most teams."""
    one = [(4, 8, 256, 24), (5, 8, 256, 24), (6, 3, 256, 24), (8, 16, 128, 24), (10, 8, 128, 24),
           (12, 16, 256, 16), (12, 16, 512, 16), (16, 3, 512, 16), (10, 3, 1024, 22)]
    team = [(6, 8, 4096, 1), (10, 3, 128, 8), (10, 3, 1000, 1), (5, 8, 1024, 8), (12, 32, 300, 4),
            (16, 8, 1024, 4), (8, 16, 500, 8)]
    res = record([dict(call="gram", order=p, d=d, lx=n, nx=nx) for p, d, n, nx in one + team])
    got = [forward(r)[0].startswith("team_kernel") for r in res]
    assert got == [False] * len(one) + [True] * len(team), list(zip(one + team, got))


def test_small_tables_are_taken_when_the_upload_returns():
    """Up to the header's limit the upload copies nothing from host memory, which is
    what lets the autograd calls skip their wait for it; beyond it does.  The
    limit and the table sizes are the binding's."""
    from paper_2502_20392_amd import _lib, api
    text = open(os.path.join(ROOT, "include", "sigk.h")).read()
    limit = int(re.search(r"SIGK_PLAN_ARG_BYTES = (\d+)", text).group(1))
    assert _lib.PLAN_ARG_BYTES == limit
    one, two, none = [0, 0], [0, 1], [0, 2]  # pairs of one, two and no strips
    lens = [30, 100, 1]
    n = limit // 80
    at = [one] * (n - (limit - 80 * n) // 16) + [two] * ((limit - 80 * n) // 16)
    tables = [at, at + [none], at[:-1] + [none], [one] * (n - 1), [one] * (2 * n)]
    small = [64 * len(t) + 16 * (t.count(one) + 2 * t.count(two)) <= limit for t in tables]
    assert small == [True, False, True, True, False]
    jobs = [dict(call="plan", lens=lens, pairs=t, d=3, order=6, steps=["upload"]) for t in tables]
    for t, ok, r in zip(tables, small, record(jobs)):
        assert r["rc"] == 0 and ok == all(e[0] != "copy" for e in r["events"]), (ok, r["events"])
        plan = api.RaggedPlan(np.cumsum([0] + lens), np.array(t, np.int32), 3, order=6, device="cpu")
        assert plan._small_tables() == ok


@pytest.mark.parametrize("order", [5, 8])
def test_benchmark_warms_every_kernel_of_the_long_gradient(order):
    import bench
    q = dict(call="pair_backward", d=8, order=order)
    timed, *warm = record([dict(q, lx=1_000_000, ly=1_000_000)] + [
        dict(q, lx=nx, ly=ny, rows=kw.get("block_rows", 0), cols=kw.get("block_cols", 0))
        for nx, ny, kw in bench.LONG_GRAD_WARMUP])
    assert all(r["rc"] == 0 for r in [timed] + warm)
    need = set(kernels(timed))
    assert {"lines_kernel<%d,8>" % order, "bwd_kernel<%d,8>" % order} <= need
    assert need <= {k for r in warm for k in kernels(r)}
    assert max(r["bytes"] for r in warm) <= timed["bytes"]


def test_two_waves_per_strip_where_they_are_the_faster_adjoint():
    """Few strips take two waves each, except at the orders whose halves spill."""
    for order, d, want in ((5, 32, "two"), (16, 32, "two"), (20, 16, "two"), (20, 32, "one"),
                           (24, 3, "one"), (24, 16, "one"), (24, 32, "one")):
        r, = record([dict(call="plan", lens=[100] * 9, pairs=[[i, i + 1] for i in range(8)], d=d,
                          order=order, steps=["backward"])])
        names = {k.split("<")[0] for k in kernels(r)}
        assert ("bwd_two_kernel" in names) == (want == "two"), (order, d, names)


def test_teams_on_one_pair_of_thousands_of_strips():
    """More teams than are resident, started one after another along one pair."""
    got = [forward(r)[0].split("<")[0] for r in record([
        dict(call="gram", nx=1, lx=n, d=8, order=5) for n in (20001, 100001, 200001, 1_000_000)])]
    assert got == ["team_kernel", "team_kernel", "team_kernel", "fwd_kernel"], got
