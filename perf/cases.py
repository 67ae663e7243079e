"""What this library is timed on: calls that a program computing integrals over
Gaussian shells makes, through the Python binding, with the inputs resident on
the GPU and the outputs in a buffer that the program keeps.

A case names the kind of call and its sizes:
  batch      one class (la lb|lc ld) of Cartesian integrals          eri4.batch
  solid      the same over real solid harmonics                      eri4.batch_solid
  coulomb    J_ab = sum_cd (ab|cd) D_cd per quartet                  eri4.batch_coulomb
  exchange   K_ac = sum_bd (ab|cd) D_bd per quartet                  eri4.batch_exchange
  plan       a batch mixing classes and contraction lengths          eri4.Plan
  solidplan  the same over solid harmonics                           eri4.SolidPlan
  pairs      every pair of a bra list with every pair of a ket list  eri4.PairPlan
  solidpairs the same over solid harmonics                           eri4.PairPlan
  jpairs     the Coulomb contraction over two lists                  eri4.CoulombPlan
Single-class kinds give the class as four digits ("ls") and the contraction
length of each shell as four digits ("ks"); the others the angular momenta drawn
from ("lv") and the largest contraction length ("kmax"; "kfix": every shell has
it).  Plans with FP32 transforms are left out: their doubles carry the rounding
of FP32 products, about 1e-7, which moves with any order of summation, so two
of their outputs cannot be held against each other as doubles are.
"""
import math

import numpy as np
import torch

from paper_2307_03452_amd import eri4, inputs

SINGLE = ("batch", "solid", "coulomb", "exchange")
LISTS = ("pairs", "solidpairs", "jpairs")


def listed():
    return [
        # a short call, as a program makes for a few quartets at a time: 64 quartets leave most of the
        # chip waiting on one chain of steps
        {"name": "gggg_k1_64", "kind": "batch", "ls": "4444", "ks": "1111", "nq": 64},
        # the low-l classes of an ordinary basis: one primitive each, and contracted on both sides
        {"name": "dddd_k1_4096", "kind": "batch", "ls": "2222", "ks": "1111", "nq": 4096},
        {"name": "ffff_k25_1024", "kind": "batch", "ls": "3333", "ks": "5151", "nq": 1024},
        # the headline class, uncontracted and contracted
        {"name": "iiii_k1_512", "kind": "batch", "ls": "6666", "ks": "1111", "nq": 512},
        {"name": "iiii_k5_16", "kind": "batch", "ls": "6666", "ks": "5555", "nq": 16},
        # a chunk of a serving stream: all classes of g..k, three primitives per shell
        {"name": "stream_253", "kind": "plan", "lv": "4567", "kmax": 3, "kfix": True, "nq": 253},
        # a batch of uneven work: contraction lengths 1..8
        {"name": "uneven_250", "kind": "plan", "lv": "456", "kmax": 8, "kfix": False, "nq": 250},
        # bra list x ket list, ragged
        {"name": "pairs_41x37", "kind": "pairs", "lv": "456", "kmax": 3, "kfix": False, "nq": 41, "nk": 37},
        # solid-harmonic output
        {"name": "solid_iiii_k1_512", "kind": "solid", "ls": "6666", "ks": "1111", "nq": 512},
        # the Fock-matrix contractions: one class, over lists, and exchange
        {"name": "coulomb_iiii_k1_512", "kind": "coulomb", "ls": "6666", "ks": "1111", "nq": 512},
        {"name": "jpairs_96x80", "kind": "jpairs", "lv": "456", "kmax": 3, "kfix": False, "nq": 96, "nk": 80},
        {"name": "exchange_iiii_k1_256", "kind": "exchange", "ls": "6666", "ks": "1111", "nq": 256},
    ]


def _herm(n):
    return (n + 1) * (n + 2) * (n + 3) // 6


def _cart(l):
    return (l + 1) * (l + 2) // 2


def _dense(ls, kb, kk):
    """Dense matrix FLOPs of the two transforms of one quartet."""
    nab, ncd = _cart(ls[0]) * _cart(ls[1]), _cart(ls[2]) * _cart(ls[3])
    npp, nqq = _herm(ls[0] + ls[1]), _herm(ls[2] + ls[3])
    return 2.0 * nab * nqq * kk * (kb * npp + ncd)


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["batch", "batch", "batch", "plan", "plan", "pairs", "solid", "coulomb", "exchange",
                       "jpairs", "solidplan", "solidpairs"])
    c = {"kind": kind}
    if kind in SINGLE:
        # two batches in five are of low angular momentum; a side's lengths multiply to at most 25
        low = kind == "batch" and rng.random() < 0.4
        ls = [rng.randint(0, 3) if low else rng.randint(4, 7) for _ in range(4)]
        ks = [rng.choice([1, 1, 2, 3, 4, 5]) for _ in range(4)]
        c["ls"], c["ks"] = "".join(map(str, ls)), "".join(map(str, ks))
        # at most 2e12 dense FLOPs, 250 MB of integrals per 1e8 of them, 4e5 primitive quartets in all
        kb, kk = ks[0] * ks[1], ks[2] * ks[3]
        size = _cart(ls[0]) * _cart(ls[1]) * _cart(ls[2]) * _cart(ls[3])
        most = min(2e12 / _dense(ls, kb, kk), 3e8 / size, 4e5 / (kb * kk), 8192)
        if kind == "exchange":  # the F^b workspace of every ket primitive pair
            per = max(ks) ** 2 * _cart(ls[1]) * 16 * ((_cart(ls[2]) + 15) // 16) * (_herm(ls[2] + ls[3]) + 3)
            most = min(most, 5e8 / per)
        c["nq"] = _logint(rng, max(1, min(3, int(most))), max(1, most))
    elif kind in LISTS:
        c["lv"], c["kmax"], c["kfix"] = rng.choice(["45", "456", "56", "4567"]), rng.choice([1, 2, 3]), False
        most = {"45": 44, "456": 38, "56": 32, "4567": 28}[c["lv"]]
        c["nq"], c["nk"] = _logint(rng, 3, most), _logint(rng, 3, most)
    else:
        c["lv"] = rng.choice(["45", "456", "4567", "0123", "3456"])
        c["kmax"], c["kfix"] = rng.choice([1, 2, 3, 4, 6]), rng.random() < 0.3
        c["nq"] = _logint(rng, 5, 240.0 / max(1.0, (c["kmax"] / 3.0) ** 4) if c["kfix"] else 240)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _batch(case, seed):
    """The quartets of a single-class or plan case: seeded centres in an 8-Bohr
    cube, log-uniform exponents, normalised contracted shells."""
    lo, hi = 0.05, 200.0
    if case["kind"] in SINGLE:
        ls = [int(x) for x in case["ls"]]
        ks = [int(x) for x in case["ks"]]
        nq, kmax = case["nq"], max(ks)
        rng = np.random.Generator(np.random.PCG64(seed))
        lq = np.tile(np.array(ls, np.int32), (nq, 1))
        nprim = np.tile(np.array(ks, np.int32), (nq, 1))
        if max(ls) <= 4:
            hi = 50.0
        centers = rng.uniform(0.0, 8.0, size=(nq, 4, 3))
        exps = np.exp(rng.uniform(math.log(lo), math.log(hi), size=(nq, 4, kmax)))
        raw = np.where(nprim[..., None] == 1, 1.0, rng.uniform(0.1, 1.0, size=(nq, 4, kmax)))
        return inputs.Batch(tuple(ls), centers, exps, inputs.normalize_shells(lq, exps, raw, nprim), nprim, lq)
    lv = tuple(int(x) for x in case["lv"])
    b = inputs.uneven_batch(nq=case["nq"], seed=1004, lvals=lv, kmax=case["kmax"],
                            k_fixed=case["kmax"] if case["kfix"] else None)
    b.centers, b.exps, b.coefs = _redraw(b.lq, b.nprim, case["kmax"], seed)
    return b


def _redraw(l, nprim, kmax, seed):
    """Geometry and exponents from the seed for shells whose classes and lengths
    (the basis set of a molecule) the case alone decides."""
    rng = np.random.Generator(np.random.PCG64(seed))
    centers = rng.uniform(0.0, 8.0, size=l.shape + (3,))
    exps = np.exp(rng.uniform(math.log(0.05), math.log(200.0), size=l.shape + (kmax,)))
    raw = np.where(nprim[..., None] == 1, 1.0, rng.uniform(0.1, 1.0, size=l.shape + (kmax,)))
    return centers, exps, inputs.normalize_shells(l, exps, raw, nprim)


def _lists(case, seed):
    lv = tuple(int(x) for x in case["lv"])
    both = []
    for n, fixed in ((case["nq"], 1201), (case["nk"], 1202)):
        p = inputs.pair_list(n, fixed, lvals=lv, kmax=case["kmax"])
        p.centers, p.exps, p.coefs = _redraw(p.l, p.nprim, case["kmax"], 2 * seed + fixed % 2)
        both.append(p)
    return both


def _dens(case, seed):
    """The density of a contraction case: blocks per quartet, or per ket entry."""
    rng = np.random.Generator(np.random.PCG64(seed + 77))
    if case["kind"] == "jpairs":
        ket = _lists(case, seed)[1]
        return rng.uniform(-1.0, 1.0, size=sum(_cart(int(a)) * _cart(int(b)) for a, b in ket.l))
    ls = [int(x) for x in case["ls"]]
    rows = ls[2] if case["kind"] == "coulomb" else ls[1]
    return rng.uniform(-1.0, 1.0, size=(case["nq"], _cart(rows), _cart(ls[3])))


def _up(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind}
    new = lambda n: torch.empty(max(1, n), dtype=torch.float64, device="cuda")  # noqa: E731
    if kind in SINGLE:
        b = _batch(case, seed)
        ls, nq = b.ls, b.nq
        s.update(ls=ls, shells=[_up(b.centers), _up(b.exps), _up(b.coefs), _up(b.nprim)])
        f = inputs.ncart if kind != "solid" else eri4.nsolid
        dims = {"coulomb": ls[:2], "exchange": (ls[0], ls[2])}.get(kind, ls)
        s["out"] = new(nq * math.prod(f(l) for l in dims)).view([nq] + [f(l) for l in dims])
        if kind == "solid":
            s["work"] = new(eri4.solid_work_size(ls, b.kmax, nq))
        elif kind == "coulomb":
            s["work"], s["dens"] = new(eri4.coulomb_work_size(ls, b.kmax, nq)), _up(_dens(case, seed))
        elif kind == "exchange":
            s["work"], s["dens"] = new(eri4.exchange_work_size(ls, b.kmax, nq)), _up(_dens(case, seed))
        return s
    if kind in LISTS:
        bra, ket = _lists(case, seed)
        if kind == "jpairs":
            p = eri4.CoulombPlan(bra.l, bra.nprim, ket.l, ket.nprim, case["kmax"])
            s["dens"] = _up(_dens(case, seed))
        else:
            p = eri4.PairPlan(bra.l, bra.nprim, ket.l, ket.nprim, case["kmax"],
                              functions="solid" if kind == "solidpairs" else "cartesian")
        s["lists"] = [_up(x) for l in (bra, ket) for x in (l.centers, l.exps, l.coefs)]
    else:
        b = _batch(case, seed)
        plan = eri4.SolidPlan if kind == "solidplan" else eri4.Plan
        p = plan(b.lq, b.nprim, b.kmax, tune_file=eri4.TUNE_FILE)
        s["shells"] = [_up(b.centers), _up(b.exps), _up(b.coefs)]
    s["plan"], s["out"] = p, new(p.output_size)
    if kind in ("solidpairs", "solidplan", "jpairs"):
        s["work"] = new(p.work_size)
    return s


def run(s):
    kind = s["kind"]
    if kind == "batch":
        return eri4.batch(s["ls"], *s["shells"], out=s["out"])
    if kind == "solid":
        return eri4.batch_solid(s["ls"], *s["shells"], work=s["work"], out=s["out"])
    if kind == "coulomb":
        return eri4.batch_coulomb(s["ls"], *s["shells"], s["dens"], work=s["work"], out=s["out"])
    if kind == "exchange":
        return eri4.batch_exchange(s["ls"], *s["shells"], s["dens"], work=s["work"], out=s["out"])
    if kind == "plan":
        return s["plan"].execute(*s["shells"], out=s["out"])
    if kind == "solidplan":
        return s["plan"].execute(*s["shells"], out=s["out"], work=s["work"])
    if kind == "pairs":
        return s["plan"].execute(*s["lists"], out=s["out"])
    if kind == "solidpairs":
        return s["plan"].execute(*s["lists"], out=s["out"], work=s["work"])
    return s["plan"].execute(*s["lists"], s["dens"], out=s["out"], work=s["work"])


# ---------------------------------------------------------------------------
# work
# ---------------------------------------------------------------------------

_CHAIN = {}


def _chain(l1, l2):
    """Multiply-adds that take one vector of Hermite functions of a shell pair to
    its Cartesian products one axis at a time (E is a product of one 1-d table
    per axis, and E^t is zero above t = a + b)."""
    if (l1, l2) not in _CHAIN:
        L, n = l1 + l2, 0
        for ax in range(l1 + 1):
            for bx in range(l2 + 1):
                m = L - ax - bx
                n += (ax + bx + 1) * (m + 1) * (m + 2) // 2
                for ay in range(l1 - ax + 1):
                    for by in range(l2 - bx + 1):
                        z = m - ay - by
                        n += (ay + by + 1) * (z + 1) + z + 1
        _CHAIN[l1, l2] = n
    return _CHAIN[l1, l2]


def work(case):
    """Bytes: each input once, each output once.  FLOPs: the two transforms of
    every quartet one axis at a time (dense products over solid functions), the
    recursion for [r] not counted; the contractions as the products of the
    Hermite-space density with [p+q], and of [ab|q] with the density."""
    kind = case["kind"]
    if kind in LISTS:
        bra, ket = _lists(case, 1)
        n = inputs.expand_pairs(bra, ket)
        lq, nprim = n.lq, n.nprim
        rows = 2 * (case["nq"] + case["nk"])
    else:
        b = _batch(case, 1)
        lq, nprim = b.lq, b.nprim
        rows = 4 * b.nq
    kmax = int(case["kmax"]) if "kmax" in case else max(int(x) for x in case["ks"])
    by = {}
    for l, k in zip(lq.tolist(), nprim.tolist()):
        key = tuple(l) + (k[0] * k[1], k[2] * k[3])
        by[key] = by.get(key, 0) + 1
    flops, out = 0.0, 0.0
    for (a, b, c, d, kb, kk), n in by.items():
        npp, nqq, nab, ncd = _herm(a + b), _herm(c + d), _cart(a) * _cart(b), _cart(c) * _cart(d)
        if kind in ("coulomb", "jpairs"):
            flops += n * (2.0 * kb * kk * npp * nqq + 2.0 * kb * _chain(a, b))
            out += n * nab if kind == "coulomb" else 0
        elif kind == "exchange":
            flops += n * 2.0 * kk * (kb * _chain(a, b) * nqq + nab * nqq * _cart(c))
            out += n * _cart(a) * _cart(c)
        elif kind.startswith("solid"):
            sab, scd = (2 * a + 1) * (2 * b + 1), (2 * c + 1) * (2 * d + 1)
            flops += n * 2.0 * sab * kk * nqq * (kb * npp + scd)
            out += n * sab * scd
        else:
            flops += n * 2.0 * kk * (kb * _chain(a, b) * nqq + nab * _chain(c, d))
            out += n * nab * ncd
    if kind == "jpairs":
        out = sum(_cart(int(a)) * _cart(int(b)) for a, b in bra.l)
    dens = _dens(case, 1).size if kind in ("coulomb", "exchange", "jpairs") else 0
    return {"bytes": 8.0 * (out + dens + rows * (3 + 2 * kmax)) + 4.0 * rows, "flops": flops}


# ---------------------------------------------------------------------------
# the same numbers in 64 bits with plain torch
# ---------------------------------------------------------------------------

def _comps(l):
    return [(x, y, l - x - y) for x in range(l, -1, -1) for y in range(l - x, -1, -1)]


def _tuv(L):
    return [(t, u, v) for t in range(L + 1) for u in range(L + 1 - t) for v in range(L + 1 - t - u)]


def _boys(M, T):
    """F_m(T), m = 0..M: a series at M and downward recursion below T = 60, the
    error function and upward recursion above."""
    F = T.new_zeros(T.shape + (M + 1,))
    small = torch.clamp(T, max=60.0)
    term = torch.full_like(T, 1.0 / (2 * M + 1))
    total = term.clone()
    for j in range(1, 260):
        term = term * (2.0 * small / (2 * M + 2 * j + 1))
        total = total + term
    e = torch.exp(-small)
    f = e * total
    G = [None] * (M + 1)
    G[M] = f
    for m in range(M - 1, -1, -1):
        f = (2.0 * small * f + e) / (2 * m + 1)
        G[m] = f
    big = torch.clamp(T, min=60.0)
    e = torch.exp(-big)
    f = 0.5 * torch.sqrt(math.pi / big) * torch.erf(torch.sqrt(big))
    for m in range(M + 1):
        F[:, m] = torch.where(T < 60.0, G[m], f)
        f = ((2 * m + 1) * f - e) / (2.0 * big)
    return F


def _pair(z1, z2, A, B):
    """p = z1 + z2, the product centre and exp(-z1 z2 / p |AB|^2)."""
    p = z1 + z2
    AB = A - B
    return p, (z1[:, None] * A + z2[:, None] * B) / p[:, None], torch.exp(-z1 * z2 / p * (AB * AB).sum(1))


def _etables(l1, l2, z1, z2, A, B):
    """1-d tables [axis][a][b] -> [n, l1 + l2 + 1] by the two recursions."""
    p = z1 + z2
    n, L = p.shape[0], l1 + l2
    h = (0.5 / p)[:, None]
    t1 = torch.arange(1, L + 2, dtype=torch.float64, device=p.device)[None, :]

    def up(e, c):
        z = e.new_zeros(n, 1)
        return h * torch.cat([z, e[:, :-1]], 1) + c * e + t1 * torch.cat([e[:, 1:], z], 1)

    out = []
    for i in range(3):
        pa, pb = (z2 / p * (B[:, i] - A[:, i]))[:, None], (z1 / p * (A[:, i] - B[:, i]))[:, None]
        e = p.new_zeros(n, L + 1)
        e[:, 0] = 1.0
        rows = []
        for a in range(l1 + 1):
            f, row = e, []
            for b in range(l2 + 1):
                row.append(f)
                f = up(f, pb)
            rows.append(torch.stack(row, 1))
            e = up(e, pa)
        out.append(torch.stack(rows, 1))
    return out


def _ematrix(l1, l2, tabs, sign):
    """E[n, (a b), tuv] of one shell pair; sign: times (-1)^(t+u+v)."""
    dev = tabs[0].device
    tuv = torch.tensor(_tuv(l1 + l2), device=dev)
    a = torch.tensor(_comps(l1), device=dev)
    b = torch.tensor(_comps(l2), device=dev)
    E = 1.0
    for i in range(3):
        T = tabs[i][:, a[:, i]][:, :, b[:, i]].reshape(tabs[i].shape[0], -1, tabs[i].shape[3])
        E = E * T[:, :, tuv[:, i]]
    return E * (1.0 - 2.0 * (tuv.sum(1) & 1).double()) if sign else E


def _hermite(L, p, q, P, Q, w):
    """w [t u v] for t, u, v <= L as [n, (L+1)^3], by raising one index at a time."""
    n, D = p.shape[0], P - Q
    rho = p * q / (p + q)
    F = _boys(L, rho * (D * D).sum(1))
    g = w * 2.0 * math.pi ** 2.5 / (p * q * torch.sqrt(p + q))
    g = g[:, None] * F * (-2.0 * rho)[:, None] ** torch.arange(L + 1, device=p.device).double()[None, :]
    i = torch.arange(1, L, dtype=torch.float64, device=p.device)
    x, y, z = (D[:, k].view(n, 1, 1, 1) for k in range(3))
    R = p.new_zeros(n, L + 1, L + 1, L + 1)
    R[:, 0, 0, 0] = g[:, L]
    for m in range(L - 1, -1, -1):
        k = L - m + 1  # orders up to L - m
        old, new = R[:, :k, :k, :k], p.new_zeros(n, k, k, k)
        new[:, 0, 0, 0] = g[:, m]
        new[:, 1:, :1, :1] = x * old[:, :-1, :1, :1]
        new[:, 2:, :1, :1] += i[:k - 2].view(1, -1, 1, 1) * old[:, :-2, :1, :1]
        new[:, :, 1:, :1] = y * old[:, :, :-1, :1]
        new[:, :, 2:, :1] += i[:k - 2].view(1, 1, -1, 1) * old[:, :, :-2, :1]
        new[:, :, :, 1:] = z * old[:, :, :, :-1]
        new[:, :, :, 2:] += i[:k - 2].view(1, 1, 1, -1) * old[:, :, :, :-2]
        R[:, :k, :k, :k] = new
    return R.reshape(n, -1)


def _solid(l):
    """Real solid harmonics m = -l..l in the Cartesian components of shell l
    (Racah normalisation, no Condon-Shortley phase), in closed form."""
    C = torch.zeros(2 * l + 1, _cart(l), dtype=torch.float64)
    where = {c: k for k, c in enumerate(_comps(l))}
    for m in range(-l, l + 1):
        am, v0 = abs(m), 1 if m < 0 else 0
        n = math.sqrt(2.0 * math.factorial(l + am) * math.factorial(l - am) / (2 if m == 0 else 1))
        n /= 2.0 ** am * math.factorial(l)
        for t in range((l - am) // 2 + 1):
            for u in range(t + 1):
                for w in range(v0, am + 1, 2):
                    c = (-1) ** (t + (w - v0) // 2) * 0.25 ** t * math.comb(l, t) * math.comb(l - t, am + t)
                    py = 2 * u + w
                    C[m + l, where[2 * t + am - py, py, l - 2 * t - am]] += n * c * math.comb(t, u) * math.comb(am, w)
    return C


def _class_exact(kind, ls, c, e, w, k, dens):
    """The results for quartets of one class: all primitive quartets as one
    list, in slices, each taken through dense matrices."""
    la, lb, lc, ld = ls
    nq, dev = c.shape[0], c.device
    L, nab, ncd = sum(ls), _cart(la) * _cart(lb), _cart(lc) * _cart(ld)
    n1 = L + 1
    off = lambda l: torch.tensor([(t * n1 + u) * n1 + v for t, u, v in _tuv(l)], device=dev)  # noqa: E731
    idx = (off(la + lb)[:, None] + off(lc + ld)[None, :]).reshape(-1)
    npp, nqq = _herm(la + lb), _herm(lc + ld)
    rows = [(q, i, j, m, n) for q, (ka, kb, kc, kd) in enumerate(k.tolist()) for i in range(ka) for j in range(kb)
            for m in range(kc) for n in range(kd)]
    rows = torch.tensor(rows, device=dev)
    big = kind in ("batch", "plan", "pairs", "solid", "solidplan", "solidpairs", "exchange")
    out = torch.zeros(nq, nab, ncd if big else 1, dtype=torch.float64, device=dev)
    step = max(8, int(1.2e8 / (n1 ** 3 * 3 + npp * nqq + nab * (npp + nqq) + ncd * nqq + (nab * ncd if big else 0))))
    for s in range(0, rows.shape[0], step):
        q, *pr = rows[s:s + step].t()
        z = [e[q, x, pr[x]] for x in range(4)]
        cf = w[q, 0, pr[0]] * w[q, 1, pr[1]] * w[q, 2, pr[2]] * w[q, 3, pr[3]]
        X = [c[q, x] for x in range(4)]
        p, P, wp = _pair(z[0], z[1], X[0], X[1])
        r, Q, wr = _pair(z[2], z[3], X[2], X[3])
        pq = _hermite(L, p, r, P, Q, cf * wp * wr)[:, idx].reshape(-1, npp, nqq)
        Eb = _ematrix(la, lb, _etables(la, lb, z[0], z[1], X[0], X[1]), False)
        Ek = _ematrix(lc, ld, _etables(lc, ld, z[2], z[3], X[2], X[3]), True)
        if big:
            res = torch.bmm(torch.bmm(Eb, pq), Ek.transpose(1, 2).contiguous())
        else:
            d = torch.bmm(Ek.transpose(1, 2).contiguous(), dens[q].reshape(-1, ncd, 1))
            res = torch.bmm(Eb, torch.bmm(pq, d))
        out.index_add_(0, q, res)
    if kind.startswith("solid"):
        C = [_solid(l).to(dev) for l in ls]
        out = torch.matmul(torch.kron(C[0], C[1]), torch.matmul(out, torch.kron(C[2], C[3]).t().contiguous()))
    elif kind == "exchange":
        na, nb, nc, nd = (_cart(l) for l in ls)
        o = out.view(nq, na, nb, nc, nd).permute(0, 1, 3, 2, 4).reshape(nq, na * nc, nb * nd)
        out = torch.bmm(o.contiguous(), dens.reshape(nq, nb * nd, 1))
    return out


def exact(case, seed):
    kind = case["kind"]
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    dens = to(_dens(case, seed)) if kind in ("coulomb", "exchange", "jpairs") else None
    if kind in SINGLE:
        b = _batch(case, seed)
        r = _class_exact(kind, b.ls, to(b.centers), to(b.exps), to(b.coefs), b.nprim, dens)
        f = (lambda l: 2 * l + 1) if kind == "solid" else _cart
        dims = {"coulomb": b.ls[:2], "exchange": (b.ls[0], b.ls[2])}.get(kind, b.ls)
        return r.reshape([b.nq] + [f(l) for l in dims])
    if kind in LISTS:
        bra, ket = _lists(case, seed)
        b = inputs.expand_pairs(bra, ket)
    else:
        b = _batch(case, seed)
    groups = {}
    for q, l in enumerate(b.lq.tolist()):
        groups.setdefault(tuple(l), []).append(q)
    blocks = [None] * b.nq
    if kind == "jpairs":  # each ket entry's block for every bra entry
        ends = np.cumsum([_cart(int(x)) * _cart(int(y)) for x, y in ket.l])
        parts = [dens[n - _cart(int(x)) * _cart(int(y)):n] for n, (x, y) in zip(ends, ket.l)]
    for ls, qs in groups.items():
        d = torch.stack([parts[q % ket.n] for q in qs]) if kind == "jpairs" else None
        r = _class_exact(kind, ls, to(b.centers[qs]), to(b.exps[qs]), to(b.coefs[qs]), b.nprim[qs], d)
        for n, q in enumerate(qs):
            blocks[q] = r[n].reshape(-1)
    if kind == "jpairs":
        blocks = [torch.stack(blocks[i * ket.n:(i + 1) * ket.n]).sum(0) for i in range(bra.n)]
    return torch.cat(blocks)
