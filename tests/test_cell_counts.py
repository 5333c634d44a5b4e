"""The sweep's count of a run of steps: between the ramps the product steps x rows,
elsewhere the general formula; both against a direct count, for every run."""


def direct(t, te, m, n):
    return sum(1 for s in range(t, te) for j in range(n) if 0 <= s - j < m)


def before(t, m, n):
    tri = lambda x: x * (x + 1) // 2 if x > 0 else 0  # noqa: E731
    return tri(t) - tri(t - m) - tri(t - n) + tri(t - m - n)


def test_counts_of_step_runs():
    for m in (1, 2, 5, 9, 17):
        for n in (1, 3, 8, 16):
            T = m + n - 1
            for t in range(T):
                for te in range(t + 1, T + 1):
                    want = direct(t, te, m, n)
                    assert before(te, m, n) - before(t, m, n) == want
                    if t >= n - 1 and te <= m:  # the sweep's test for the product
                        assert (te - t) * n == want, (m, n, t, te)
