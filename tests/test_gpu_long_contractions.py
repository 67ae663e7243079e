"""Coulomb plans over lists of long, diffuse contractions: a quartet's bra primitive
pairs run one after another in one workgroup, up to 256 of them, each with the ket's
pairs summed.  Held against the contraction per quartet (eri4_batch_coulomb), which
runs one bra primitive pair per workgroup.

Tolerance: both sum the same products in another order; 1e-12 of the largest
sum_j sum_cd |(ab|cd)| |D_cd| (test_gpu_coulomb), the integrals from eri4_batch.
"""
import numpy as np
import pytest
import torch

from paper_2307_03452_amd import eri4

pytestmark = pytest.mark.gpu
TOL = 1e-12


def pair_list(l, k, kmax, n, box, lo, hi, rng):
    return (np.tile(np.array(l, np.int32), (n, 1)), np.full((n, 2), k, np.int32), rng.uniform(0.0, box, (n, 2, 3)),
            np.exp(rng.uniform(np.log(lo), np.log(hi), (n, 2, kmax))), rng.uniform(0.1, 1.0, (n, 2, kmax)))


# (bra, ket, lengths of the bra's and the ket's shells, box, exponents): short rows of
# [r] by long ones of the density, and both sides long
@pytest.mark.parametrize("bra,ket,kb,kk,box,lo,hi", [((0, 0), (7, 7), 6, 6, 8.0, 0.05, 0.5),
                                                     ((0, 0), (7, 7), 8, 8, 8.0, 0.05, 200.0),
                                                     ((0, 0), (7, 7), 16, 3, 8.0, 0.05, 0.5),
                                                     ((0, 0), (5, 4), 8, 8, 8.0, 0.05, 0.5),
                                                     ((4, 4), (5, 4), 10, 6, 4.0, 0.05, 0.5),
                                                     ((1, 0), (3, 2), 16, 16, 8.0, 0.05, 0.5),
                                                     ((7, 7), (0, 0), 6, 6, 8.0, 0.05, 0.5)])
def test_coulomb_plan_of_long_contractions(bra, ket, kb, kk, box, lo, hi):
    rng = np.random.default_rng(100 * sum(bra) + sum(ket) + kb)
    kmax, nb, nk = max(kb, kk), 6, 3
    bl, bn, bc, be, bw = pair_list(bra, kb, kmax, nb, box, lo, hi, rng)
    kl, kn, kc, ke, kw = pair_list(ket, kk, kmax, nk, box, lo, hi, rng)
    nc, nd = eri4.ncart(ket[0]), eri4.ncart(ket[1])
    D = rng.uniform(-1.0, 1.0, (nk, nc, nd))
    up = lambda x, t=torch.float64: torch.tensor(np.ascontiguousarray(x), dtype=t).cuda()  # noqa: E731
    p = eri4.CoulombPlan(bl, bn, kl, kn, kmax)
    got = p.execute(up(bc), up(be), up(bw), up(kc), up(ke), up(kw), up(D.ravel())).reshape(nb, -1)
    i, j = np.repeat(np.arange(nb), nk), np.tile(np.arange(nk), nb)
    s = [up(np.concatenate([b[i], k[j]], axis=1), t)
         for b, k, t in ((bc, kc, torch.float64), (be, ke, torch.float64), (bw, kw, torch.float64), (bn, kn, torch.int32))]
    d = up(D[j])
    ref = eri4.batch_coulomb(bra + ket, *s, d).reshape(nb, nk, -1).sum(1)
    eri = eri4.batch(bra + ket, *s).reshape(nb, nk, -1, nc * nd)
    scale = (eri.abs() * d.abs().reshape(nb, nk, 1, nc * nd)).sum((1, 3))
    assert torch.isfinite(ref).all()
    assert torch.isfinite(got).all()
    for q in range(nb):
        assert (got[q] - ref[q]).abs().max().item() <= TOL * scale[q].max().item(), q
