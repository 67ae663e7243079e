"""Classes of low order and classes with few rows, whose kernels differ from those of
the large ones: J, K, solid-harmonic output and plans against the class's Cartesian
integrals (eri4_batch, held against the oracle elsewhere).

Tolerance, as test_gpu_forms: sums of products of doubles whose partial sums exceed the
result by up to 1e3 over fewer than 1e3 terms, 1e-11 of the largest; plans with FP32
transforms 2e-5 (test_gpu_mixed).
"""
import numpy as np
import pytest
import torch

from paper_2307_03452_amd import eri4

pytestmark = pytest.mark.gpu
TOL = 1e-11


def up(x, t=torch.float64):
    return torch.tensor(np.ascontiguousarray(x), dtype=t).cuda()


def shells(nq, kmax, seed):
    r = np.random.default_rng(seed)
    n = r.integers(1, kmax + 1, (nq, 4)).astype(np.int32)
    n[0] = kmax
    c, e, w = r.uniform(0.0, 1.5, (nq, 4, 3)), np.exp(r.uniform(np.log(0.2), np.log(5.0), (nq, 4, kmax))), \
        r.uniform(0.3, 1.0, (nq, 4, kmax))
    return n, [up(c), up(e), up(w), up(n, torch.int32)]


def nc(l):
    return eri4.ncart(l)


def close(a, b, scale, tol=TOL):
    assert torch.isfinite(a).all()
    assert (a - b).abs().max().item() <= tol * scale, (a - b).abs().max().item() / scale


# total orders 0..10 (8 is the last whose recursion one wave runs), sides of order 6, 7
# and 8, one row and one column, 16, 17, 33 rows and more
CLASSES = [(0, 0, 0, 0), (1, 0, 0, 0), (0, 0, 0, 1), (1, 1, 0, 0), (0, 2, 1, 0), (1, 1, 1, 1), (2, 1, 1, 1), (3, 3, 0, 0),
           (0, 0, 3, 3), (2, 2, 2, 2), (3, 3, 1, 1), (1, 1, 3, 3), (6, 0, 2, 0), (2, 0, 5, 1), (4, 3, 0, 0), (0, 0, 7, 0),
           (4, 4, 0, 0), (0, 0, 4, 4), (3, 2, 2, 2), (3, 3, 3, 0), (5, 1, 0, 0), (5, 0, 1, 1), (4, 2, 4, 0), (7, 1, 1, 0)]


@pytest.mark.parametrize("ls", CLASSES)
@pytest.mark.parametrize("kmax", [1, 2, 3])
def test_contractions_solid_and_plans(ls, kmax):
    nq = 5
    n, s = shells(nq, kmax, 10 * sum(ls) + kmax)
    eri = eri4.batch(ls, *s).reshape([nq] + [nc(l) for l in ls])
    g = torch.Generator().manual_seed(sum(ls))
    bad = s[3].clone()
    bad[2, 3] = kmax + 1
    ok = [0, 1, 3, 4]
    d = torch.rand((nq, nc(ls[2]), nc(ls[3])), generator=g, dtype=torch.float64).sub_(0.5).cuda()
    ref, scale = (eri * d[:, None, None]).sum((3, 4)), (eri.abs() * d.abs()[:, None, None]).sum((3, 4))
    j = eri4.batch_coulomb(ls, *s[:3], bad, d).reshape(ref.shape)
    assert torch.isnan(j[2]).all()
    for q in ok:
        close(j[q], ref[q], scale[q].max().item())
    d = torch.rand((nq, nc(ls[1]), nc(ls[3])), generator=g, dtype=torch.float64).sub_(0.5).cuda()[:, None, :, None, :]
    ref, scale = (eri * d).sum((2, 4)), (eri.abs() * d.abs()).sum((2, 4))
    k = eri4.batch_exchange(ls, *s[:3], bad, d.reshape(nq, nc(ls[1]), nc(ls[3])).contiguous()).reshape(ref.shape)
    assert torch.isnan(k[2]).all()
    for q in ok:
        close(k[q], ref[q], scale[q].max().item())
    ref = eri
    for i, l in enumerate(ls):
        c = torch.as_tensor(np.asarray(eri4.solid_coefficients(l)), dtype=torch.float64).reshape(2 * l + 1, nc(l)).cuda()
        ref = torch.tensordot(ref, c, dims=([i + 1], [1])).movedim(-1, i + 1)
    sol = eri4.batch_solid(ls, *s[:3], bad).reshape(ref.shape)
    assert torch.isnan(sol[2]).all()
    lq = np.tile(np.array(ls, np.int32), (nq, 1))
    solp = eri4.SolidPlan(lq, n, kmax).execute(*s[:3]).reshape(ref.shape)
    for q in range(nq):
        m = eri[q].abs().max().item() * 10.0
        close(solp[q], ref[q], m)
        if q != 2:
            close(sol[q], ref[q], m)
    for precision, tol in (("fp64", TOL), ("fp32", 2e-5)):
        p = eri4.Plan(lq, n, kmax, precision).execute(*s[:3]).reshape(eri.shape)
        for q in range(nq):
            close(p[q], eri[q], eri[q].abs().max().item(), tol)


@pytest.mark.parametrize("ls", [(4, 1, 1, 0), (5, 1, 0, 0), (3, 3, 3, 3), (2, 2, 2, 2), (6, 0, 2, 1), (5, 0, 5, 0)])
def test_many_quartets_and_few(ls):
    """The rule that chooses a form goes by the number of quartets: the first five of
    many against five alone."""
    n, s = shells(5, 2, 7 + sum(ls))
    few = eri4.batch(ls, *s).reshape(5, -1)
    many = eri4.batch(ls, *[x.repeat([600] + [1] * (x.dim() - 1)) for x in s]).reshape(3000, -1)
    p = eri4.Plan(np.tile(np.array(ls, np.int32), (3000, 1)), np.tile(n, (600, 1)), 2)
    plan = p.execute(*[x.repeat([600] + [1] * (x.dim() - 1)) for x in s[:3]]).reshape(3000, -1)
    for q in range(5):
        m = few[q].abs().max().item()
        close(many[q], few[q], m)
        close(many[2995 + q], few[q], m)
        close(plan[q], few[q], m)
        close(plan[2995 + q], few[q], m)


@pytest.mark.parametrize("lv,nb,nk", [((0, 1), 7, 5), ((0, 1, 2, 3), 9, 8), ((0, 1, 4), 40, 35), ((1, 2, 3), 36, 33)])
def test_lists_of_low_and_mixed_classes(lv, nb, nk):
    """Pair lists: integrals and J, of low classes alone and beside others, few and
    many, against calls per quartet."""
    kmax = 3
    r = np.random.default_rng(nb)
    bl, kl = r.choice(lv, (nb, 2)).astype(np.int32), r.choice(lv, (nk, 2)).astype(np.int32)
    bn, kn = r.integers(1, kmax + 1, (nb, 2)).astype(np.int32), r.integers(1, kmax + 1, (nk, 2)).astype(np.int32)
    arr = lambda n: [r.uniform(0.0, 1.5, (n, 2, 3)), np.exp(r.uniform(np.log(0.2), np.log(5.0), (n, 2, kmax))),  # noqa: E731
                     r.uniform(0.3, 1.0, (n, 2, kmax))]
    b, k = arr(nb), arr(nk)
    dens = [r.uniform(-1.0, 1.0, (nc(int(x)), nc(int(y)))) for x, y in kl]
    args = [up(x) for x in b + k]
    pp = eri4.PairPlan(bl, bn, kl, kn, kmax)
    got, off = pp.execute(*args), pp.offsets()
    cj = eri4.CoulombPlan(bl, bn, kl, kn, kmax)
    J, joff = cj.execute(*args, up(np.concatenate([x.ravel() for x in dens]))), cj.offsets()
    for i in range(0, nb, max(1, nb // 6)):
        na = nc(int(bl[i, 0])) * nc(int(bl[i, 1]))
        ref, scale = torch.zeros(na, dtype=torch.float64).cuda(), torch.zeros(na, dtype=torch.float64).cuda()
        for j in range(nk):
            ls = tuple(int(x) for x in (*bl[i], *kl[j]))
            s = [up(np.concatenate([x[i:i + 1], y[j:j + 1]], axis=1)) for x, y in zip(b, k)]
            e = eri4.batch(ls, *s, up(np.concatenate([bn[i], kn[j]])[None], torch.int32)).reshape(na, -1)
            o = int(off[i * nk + j])
            close(got[o:o + e.numel()].reshape(e.shape), e, e.abs().max().item())
            d = up(dens[j].ravel())
            ref += (e * d).sum(1)
            scale += (e.abs() * d.abs()).sum(1)
        close(J[int(joff[i]):int(joff[i]) + na], ref, scale.max().item())


def test_lists_of_two_kernels_replay_in_a_graph():
    """Integrals and J of lists whose quartets take two persistent kernels each (a counter
    of its own per kernel), captured and replayed with other work between: the same bits."""
    kmax, nb, nk = 2, 40, 35
    r = np.random.default_rng(77)
    bl, kl = r.choice((0, 1, 4), (nb, 2)).astype(np.int32), r.choice((0, 1, 4), (nk, 2)).astype(np.int32)
    bn, kn = r.integers(1, kmax + 1, (nb, 2)).astype(np.int32), r.integers(1, kmax + 1, (nk, 2)).astype(np.int32)
    args = [up(x) for n in (nb, nk) for x in (r.uniform(0.0, 1.5, (n, 2, 3)), r.uniform(0.2, 5.0, (n, 2, kmax)),
                                              r.uniform(0.3, 1.0, (n, 2, kmax)))]
    pp, cj = eri4.PairPlan(bl, bn, kl, kn, kmax), eri4.CoulombPlan(bl, bn, kl, kn, kmax)
    d = up(r.uniform(-1.0, 1.0, cj.ket_dens_size))
    work = torch.empty(max(1, cj.work_size), dtype=torch.float64, device="cuda")
    ref, jref = pp.execute(*args).clone(), cj.execute(*args, d, work=work).clone()
    out, j = torch.zeros_like(ref), torch.zeros_like(jref)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        pp.execute(*args, out=out, stream=s)
        cj.execute(*args, d, out=j, work=work, stream=s)
    n, other = shells(8, kmax, 5)
    for rep in range(3):
        out.zero_()
        j.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref) and torch.equal(j, jref), rep
        eri4.batch((1, 0, 4, 0), *other)
        pp.execute(*args)
        torch.cuda.synchronize()
