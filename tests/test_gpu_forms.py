"""Kernels that reach the same numbers by different code, held against each other
at the edges of their tiles, layouts and rules.

Tolerance: every path sums products of FP64 numbers whose partial sums exceed the
result by up to 1e3 for the shells drawn here (exponents 0.2..5 within 1.5 Bohr),
over fewer than 1e3 terms per step: 1e-16 * 1e3 * 1e2 relative to the largest
integral of the quartet, 1e-11.
"""
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
