"""FLOP counts of the benchmark's rates."""
import itertools

import pytest

from paper_2307_03452_amd import metrics


def comps(l):
    return [(x, y, l - x - y) for x in range(l, -1, -1) for y in range(l - x, -1, -1)]


@pytest.mark.parametrize("ls", [(0, 0, 0, 0), (1, 0, 2, 1), (2, 2, 2, 2), (4, 3, 5, 4)])
def test_grouped_flops_count_the_uv_of_every_row(ls):
    la, lb, lc, ld = ls
    rows = lambda l1, l2: sum((l1 + l2 - a[0] - b[0] + 1) * (l1 + l2 - a[0] - b[0] + 2) // 2  # noqa: E731
                              for a, b in itertools.product(comps(l1), comps(l2)))
    nq, nab = metrics.nherm(lc + ld), metrics.npair(la, lb)
    for kb, kk in ((1, 1), (4, 9)):
        want = 2 * kb * kk * rows(la, lb) * nq + 2 * kk * nab * rows(lc, ld)
        assert metrics.grouped_flops(*ls, kb, kk) == want <= metrics.md4_flops(*ls, kb, kk)


def test_roofline_of_the_benchmark_stays_below_the_peak():
    """512 (ii|ii) in 3.56 ms: the dense count passes the FP64 peak of 78.6 TFLOP/s, the
    products that run do not."""
    t = 3.56e-3
    assert 512 * metrics.md4_flops(6, 6, 6, 6) / t > 78.6e12
    assert 512 * metrics.grouped_flops(6, 6, 6, 6) / t < 0.5 * 78.6e12
