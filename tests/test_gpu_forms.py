"""Kernels that reach the same numbers by different code, held against each other
at the edges of their tiles, layouts and rules.

Tolerance: every path sums products of FP64 numbers whose partial sums exceed the
result by up to 1e3 for the shells drawn here (exponents 0.2..5 within 1.5 Bohr),
over fewer than 1e3 terms per step: 1e-16 * 1e3 * 1e2 relative to the largest
integral of the quartet, 1e-11.
"""
import itertools

import numpy as np
import pytest
import torch

from paper_2307_03452_amd import eri4

pytestmark = pytest.mark.gpu
TOL = 1e-11


def shells(ls, nq, kmax, seed, nprim=None):
    rng = np.random.default_rng(seed)
    if nprim is None:
        nprim = rng.integers(1, kmax + 1, size=(nq, 4))
    c = rng.uniform(0.0, 1.5, size=(nq, 4, 3))
    e = np.exp(rng.uniform(np.log(0.2), np.log(5.0), size=(nq, 4, kmax)))
    w = rng.uniform(0.3, 1.0, size=(nq, 4, kmax))
    up = lambda x, t: torch.tensor(np.ascontiguousarray(x), dtype=t).cuda()  # noqa: E731
    return [up(c, torch.float64), up(e, torch.float64), up(w, torch.float64), up(nprim, torch.int32)]


def nc(l):
    return eri4.ncart(l)


def integrals(ls, s):
    nq = s[0].shape[0]
    return eri4.batch(ls, *s).reshape([nq] + [nc(l) for l in ls])


def close(a, b, scale):
    assert torch.isfinite(a).all()
    d = (a - b).abs().max().item()
    assert d <= TOL * scale, (d, scale)


LOW = [ls for ls in itertools.product(range(4), repeat=4) if sum(ls) >= 6]


@pytest.mark.parametrize("part", range(8))
def test_few_quartets_and_many(part):
    """l <= 3: a few quartets take the one-workgroup form, copies of them past any
    count at which the rule allows it (or, where it always does, as a plan) the
    other; one contraction length is out of range."""
    for ls in LOW[part::8]:
        kmax = 1 + sum(ls) % 3
        s = shells(ls, 5, kmax, 7 + part)
        s[3][3, 1] = kmax + 1
        few = integrals(ls, s)
        if ls[0] + ls[1] == 6 and ls[2] + ls[3] >= 4:
            keep = [0, 1, 2, 4]
            t = [x[keep].contiguous() for x in s]
            p = eri4.Plan(np.tile(np.array(ls, np.int32), (4, 1)), t[3].cpu().numpy(), kmax)
            many = torch.empty(few[keep].numel(), dtype=torch.float64, device="cuda")
            p.execute(*t[:3], out=many)
            assert torch.isnan(few[3]).all()
            few, many = few[keep], many.reshape(few[keep].shape)
        else:
            many = integrals(ls, [x.repeat([200] + [1] * (x.dim() - 1)) for x in s])[-5:]
            assert torch.isnan(few[3]).all() and torch.isnan(many[3]).all()
            few, many = few[[0, 1, 2, 4]], many[[0, 1, 2, 4]]
        for a, b in zip(few, many):
            close(a, b, b.abs().max().item())


def test_smallest_classes_as_plan():
    """Total order below 6: the one-wave kernel against the plan's."""
    for ls in itertools.product(range(4), repeat=4):
        if sum(ls) >= 6:
            continue
        s = shells(ls, 3, 2, sum(ls) + 11)
        p = eri4.Plan(np.tile(np.array(ls, np.int32), (3, 1)), s[3].cpu().numpy(), 2)
        a = integrals(ls, s)
        b = p.execute(*s[:3])[: a.numel()].reshape(a.shape)
        for x, y in zip(a, b):
            close(x, y, y.abs().max().item())


# ket orders 0..14 (the shapes of the integral kernels), bra orders at the widths of
# the Coulomb kernels' chunks (8, 16, 32, 64, 128), total orders 15, 16, 17 (a second
# block of the recursion), 19, 20, 24, 25 (layouts) and 28
EDGES = [(4, 0, 0, 0), (0, 4, 1, 0), (4, 4, 1, 1), (5, 4, 2, 1), (4, 0, 4, 0), (4, 2, 4, 1), (4, 4, 4, 2), (4, 4, 4, 3),
         (4, 5, 4, 4), (5, 5, 5, 4), (6, 4, 5, 5), (5, 6, 6, 5), (6, 6, 6, 6), (6, 6, 7, 6), (7, 6, 6, 6), (7, 7, 7, 7),
         (7, 0, 7, 7), (0, 7, 7, 0)]


@pytest.mark.parametrize("ls", EDGES)
def test_contractions_of_the_integrals(ls):
    """J, K and the solid-harmonic integrals against the Cartesian integrals."""
    kmax = 2 if sum(ls) < 20 else 1
    nq = 3
    s = shells(ls, nq, kmax, sum(ls))
    eri = integrals(ls, s)
    g = torch.Generator().manual_seed(sum(ls))
    d = torch.rand((nq, nc(ls[2]), nc(ls[3])), generator=g, dtype=torch.float64).sub_(0.5).cuda()
    j = eri4.batch_coulomb(ls, *s, d).reshape(nq, nc(ls[0]), nc(ls[1]))
    ref = (eri * d[:, None, None]).sum((3, 4))
    scale = (eri.abs() * d.abs()[:, None, None]).sum((3, 4))
    for q in range(nq):
        close(j[q], ref[q], scale[q].max().item())
    d = torch.rand((nq, nc(ls[1]), nc(ls[3])), generator=g, dtype=torch.float64).sub_(0.5).cuda()
    k = eri4.batch_exchange(ls, *s, d).reshape(nq, nc(ls[0]), nc(ls[2]))
    dd = d[:, None, :, None, :]
    ref, scale = (eri * dd).sum((2, 4)), (eri.abs() * dd.abs()).sum((2, 4))
    for q in range(nq):
        close(k[q], ref[q], scale[q].max().item())
    sol = eri4.batch_solid(ls, *s).reshape([nq] + [2 * l + 1 for l in ls])
    ref = eri
    for i, l in enumerate(ls):
        c = torch.as_tensor(np.asarray(eri4.solid_coefficients(l)), dtype=torch.float64).reshape(2 * l + 1, nc(l)).cuda()
        ref = torch.tensordot(ref, c, dims=([i + 1], [1])).movedim(-1, i + 1)
    for q in range(nq):
        close(sol[q], ref[q], eri[q].abs().max().item() * 10.0)


def test_tiny_prefactors():
    """A quartet whose Gaussian products are near the smallest normal number keeps its
    digits in every form, and one that underflows gives zeros."""
    ls = (4, 4, 4, 4)
    s = shells(ls, 3, 1, 3, np.ones((3, 4), np.int64))
    # exp(-a b / (a + b) r^2) of both pairs together: 2^-980 and 2^-1200
    for q, bits in ((0, 980.0), (1, 1200.0)):
        for sh in (0, 2):
            a, b = s[1][q, sh, 0].item(), s[1][q, sh + 1, 0].item()
            r = (0.5 * bits * np.log(2.0) * (a + b) / (a * b)) ** 0.5
            s[0][q, sh + 1] = s[0][q, sh] + torch.tensor([r, 0.0, 0.0], dtype=torch.float64, device="cuda")
    eri = integrals(ls, s)
    assert torch.isfinite(eri).all()
    big = s[2].clone()
    big[0] *= 2.0 ** 100  # 2^400 in all: exact
    ref = integrals(ls, [s[0], s[1], big, s[3]])
    m = ref[0].abs().max().item()
    close(eri[0] * 2.0 ** 400, ref[0], m)
    assert eri[1].abs().max().item() <= 1e-280
