"""Weights and distances at the ends of the range of doubles.

Tolerances: scaling a coefficient by a power of two scales every integral by it
exactly, so that both sides of such a comparison round alike as long as no value is
subnormal; 1e-13 of the largest leaves room for the forms that scale differently.
"""
import numpy as np
import pytest
import torch

from paper_2307_03452_amd import eri4

pytestmark = pytest.mark.gpu
TOL = 1e-13


def up(x, t=torch.float64):
    return torch.tensor(np.ascontiguousarray(x), dtype=t).cuda()


def every_form(ls, c, e, w):
    """The outputs of every kernel that computes this quartet."""
    n = np.ones((1, 4), np.int32)
    s = [up(c), up(e), up(w), up(n, torch.int32)]
    lq = np.array([ls], np.int32)
    g = torch.Generator().manual_seed(sum(ls))
    d = lambda a, b: torch.rand((1, eri4.ncart(a), eri4.ncart(b)), generator=g, dtype=torch.float64).cuda()  # noqa: E731
    pair = lambda x, i: x[:, i:i + 2].contiguous()  # noqa: E731
    args = [pair(x, i) for i in (0, 2) for x in s[:3]]
    jd = d(ls[2], ls[3])
    return {
        "batch": eri4.batch(ls, *s),
        # past every count of quartets at which the call takes another form
        "batch4096": eri4.batch(ls, *[x.repeat([4096] + [1] * (x.dim() - 1)) for x in s])[4095]
        if max(ls) <= 3 else eri4.batch(ls, *s),
        "plan": eri4.Plan(lq, n, 1).execute(*s[:3]),
        "pairs": eri4.PairPlan(lq[:, :2], n[:, :2], lq[:, 2:], n[:, 2:], 1).execute(*args),
        "solid": eri4.batch_solid(ls, *s),
        "solidplan": eri4.SolidPlan(lq, n, 1).execute(*s[:3]),
        "coulomb": eri4.batch_coulomb(ls, *s, jd),
        "jpairs": eri4.CoulombPlan(lq[:, :2], n[:, :2], lq[:, 2:], n[:, 2:], 1).execute(*args, jd.flatten()),
        "exchange": eri4.batch_exchange(ls, *s, d(ls[1], ls[3])),
    }


def quartet(ls, seed):
    r = np.random.default_rng(seed)
    return r.uniform(0.0, 1.5, (1, 4, 3)), r.uniform(0.5, 2.0, (1, 4, 1))


CLASSES = [(0, 0, 0, 0), (1, 0, 0, 0), (2, 2, 2, 2), (3, 3, 3, 3), (3, 2, 1, 0), (0, 0, 4, 0), (4, 1, 1, 0), (4, 4, 4, 4),
           (6, 4, 5, 3), (6, 6, 6, 6), (7, 7, 7, 7)]


@pytest.mark.parametrize("ls", CLASSES)
@pytest.mark.parametrize("tiny", [0, 2])
def test_a_tiny_pair_with_a_large_one(ls, tiny):
    """One side's Gaussian product near 2^-950, the other's coefficients 2^130: the
    product of the two is an ordinary small number."""
    c, e = quartet(ls, 5 + sum(ls))
    a, b = e[0, tiny, 0], e[0, tiny + 1, 0]
    c[0, tiny + 1] = c[0, tiny] + np.array([(950.0 * np.log(2.0) * (a + b) / (a * b)) ** 0.5, 0.0, 0.0])
    w = np.ones((1, 4, 1))
    big = w.copy()
    big[0, 2 - tiny:4 - tiny] = 2.0 ** 65
    one, two = every_form(ls, c, e, w), every_form(ls, c, e, big)
    for k in one:
        x, y = one[k].flatten() * 2.0 ** 130, two[k].flatten()
        assert torch.isfinite(y).all(), k
        # (in "one" values may be subnormal in forms that do not scale)
        m = y.abs().max().item()
        assert m > 0.0 and (x - y).abs().max().item() <= TOL * m, (k, (x - y).abs().max().item() / m)


# (two shells on one centre have a charge only if their l add to an even number)
@pytest.mark.parametrize("ls", [ls for ls in CLASSES if (ls[2] + ls[3]) % 2 == 0])
def test_pairs_far_apart(ls):
    """Two charge distributions a great distance R apart repel as their charges do,
    q q / R: the same times R at every R, up to their extent over R (below 1e-6 from
    1e9 on).  Solid harmonics of different l on one centre have no charge: what is left
    of the Cartesian integrals they are sums of is held against the largest of those."""
    c, e = quartet(ls, 9 + sum(ls))
    w = np.ones((1, 4, 1))
    ref = None
    for R in (1e9, 1e12, 1e16, 1e20, 1e30):
        c[0, 2:] = [R, 0.0, 0.0]
        got = every_form(ls, c, e, w)
        if ref is None:
            ref = {k: x.flatten() * R for k, x in got.items()}
        for k, x in got.items():
            x = x.flatten() * R
            assert torch.isfinite(x).all(), (k, R)
            m = ref["batch" if k.startswith("solid") else k].abs().max().item()
            assert (x - ref[k]).abs().max().item() <= 1e-6 * m, (k, R)


@pytest.mark.parametrize("ls", CLASSES)
@pytest.mark.parametrize("side", [0, 2])
def test_shells_of_a_pair_far_apart(ls, side):
    """A Gaussian product prefactor that is zero gives zeros, wherever the centres are."""
    c, e = quartet(ls, 3 + sum(ls))
    e[0, side + 1] = e[0, side]  # their product sits between them, by the other pair
    for R in (1e3, 1e9, 1e13, 1e16, 1e20):
        c[0, side], c[0, side + 1] = [R, 0.0, 0.0], [-R, 0.0, 0.0]
        for k, x in every_form(ls, c, e, np.ones((1, 4, 1))).items():
            assert (x == 0.0).all(), (k, R)
