// eri4_tables.cpp -- host-side generation of the constant tables liberi4 uploads
// to each device: the Boys-function Taylor grid, the Hermite recursion tables
// and the solid-harmonic coefficients.  Plain host C++, built into liberi4.so.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

#include "eri4_internal.h"

namespace eri4 {

// F_k(T) for k = 0..kmax at one T, in long double (64-bit mantissa).
// The Boys integral of eq. (boys) expands as
//   F_K(T) = exp(-T) sum_{j>=0} (2T)^j / ((2K+1)(2K+3)...(2K+2j+1)),
// a sum of positive terms; lower orders follow from
//   F_k(T) = (2T F_{k+1}(T) + exp(-T)) / (2k+1),
// which is stable in the downward direction.
static void boys_column(int kmax, long double T, long double* F) {
  const long double ex = expl(-T);
  long double term = 1.0L / (2 * kmax + 1);
  long double sum = term;
  for (int j = 1; j < 4000; ++j) {
    term *= 2.0L * T / (2 * kmax + 2 * j + 1);
    sum += term;
    if (term < sum * 1e-22L) break;
  }
  F[kmax] = ex * sum;
  for (int k = kmax - 1; k >= 0; --k) F[k] = (2.0L * T * F[k + 1] + ex) / (2 * k + 1);
}

void make_boys_table(std::vector<double>& tab) {
  tab.assign((size_t)(kBoysRows + 1) * kBoysCols, 0.0);
  {  // Gamma(m+1/2)/2 = (2m-1)!! sqrt(pi) / 2^(m+1)
    long double c = sqrtl(3.14159265358979323846264338327950288L) / 2.0L;
    for (int m = 0; m < kBoysCols; ++m) {
      tab[(size_t)kBoysAsymRow * kBoysCols + m] = (double)c;
      c *= (2.0L * m + 1.0L) / 2.0L;
    }
  }
  std::vector<long double> F(kBoysCols);
  for (int i = 0; i < kBoysRows; ++i) {
    const long double T = (long double)i * (long double)kBoysH;  // exact grid point
    boys_column(kBoysCols - 1, T, F.data());
    for (int k = 0; k < kBoysCols; ++k) tab[(size_t)i * kBoysCols + k] = (double)F[k];
  }
}

// Triples (t,u,v), t+u+v <= L, by total order; within one total order any
// order works because entries of one order only read lower orders.  start[L] is the
// first entry (in uint32 pairs) of a table.
void make_rtabs(std::vector<uint32_t>& tab, std::vector<int>& start) {
  tab.clear();
  start.assign(kMaxL + 1, 0);
  for (int L = 0; L <= kMaxL; ++L) {
    start[L] = (int)(tab.size() / 2);
    for (int n = 0; n <= L; ++n)
      for (int t = n; t >= 0; --t)
        for (int u = n - t; u >= 0; --u) {
          const int v = n - t - u;
          const uint32_t off = (uint32_t)r_offset(false, L, t, u, v);
          uint32_t dir = 0, ri = 0, o1 = 0, o2 = 0;
          if (n > 0) {
            int a[3] = {t, u, v};
            dir = v > 0 ? 2 : (u > 0 ? 1 : 0);
            ri = (uint32_t)a[dir];
            a[dir] -= 1;
            o1 = (uint32_t)r_offset(false, L, a[0], a[1], a[2]);
            if (ri >= 2) {
              a[dir] -= 1;
              o2 = (uint32_t)r_offset(false, L, a[0], a[1], a[2]);
            } else {
              o2 = o1;
            }
          }
          tab.push_back(off | (o1 << 16));
          tab.push_back(o2 | (dir << 16) | (ri << 18));
        }
  }
}

// Real solid harmonics in Cartesian monomials (the coefficient matrices that
// turn E into H, Sec. 2), from the closed-form expansion
//   S_lm = N_lm sum_{t,u,v} (-1)^(t+v-v_m) 4^-t C(l,t) C(l-t,|m|+t) C(t,u) C(|m|,2v)
//                          x^(2t+|m|-2(u+v)) y^(2(u+v)) z^(l-2t-|m|),
//   N_lm = sqrt(2 (l+|m|)! (l-|m|)! / 2^delta(m,0)) / (2^|m| l!),
// t = 0..(l-|m|)/2, u = 0..t, v = v_m, v_m+1, ... <= |m|/2 with v_m = 0 for
// m >= 0 and 1/2 for m < 0 (Helgaker, Jorgensen and Olsen, Sec. 6.4.2).  Rows
// m = -l..l; columns in the integrals' Cartesian order; unit-norm functions
// when the Cartesian components share the coefficient that normalises x^l.
// Every term before the final scaling by N_lm is an exact binary fraction.
void solid_dense(int l, double* C) {
  auto binom = [](int n, int k) {
    if (k < 0 || k > n) return 0.0;
    double r = 1.0;
    for (int i = 1; i <= k; ++i) r = r * (n - k + i) / i;
    return r;
  };
  auto fact = [](int n) {
    double r = 1.0;
    for (int i = 2; i <= n; ++i) r *= i;
    return r;
  };
  const int nc = ncart(l);
  for (int i = 0; i < (2 * l + 1) * nc; ++i) C[i] = 0.0;
  for (int m = -l; m <= l; ++m) {
    const int am = m < 0 ? -m : m;
    double* row = C + (m + l) * nc;
    const int w0 = m < 0 ? 1 : 0;  // 2 v_m
    for (int t = 0; t <= (l - am) / 2; ++t)
      for (int u = 0; u <= t; ++u)
        for (int w = w0; w <= am; w += 2) {  // w = 2v
          const double sign = (((2 * t + w - w0) / 2) & 1) ? -1.0 : 1.0;
          const double c = sign * binom(l, t) * binom(l - t, am + t) * binom(t, u) * binom(am, w) / std::ldexp(1.0, 2 * t);
          const int py = 2 * u + w, px = 2 * t + am - py, pz = l - 2 * t - am;
          if (px < 0) continue;
          row[(l - px) * (l - px + 1) / 2 + pz] += c;
        }
    const double n = std::sqrt(2.0 * fact(l + am) * fact(l - am) / (m == 0 ? 2.0 : 1.0)) /
                     (std::ldexp(1.0, am) * fact(l));
    for (int k = 0; k < nc; ++k) row[k] *= n;
  }
}

// Sparse form for the device: entry (l, m + l) at ((l * kSolidRows) + m + l) *
// kSolidEntry doubles: [0] number of non-zero terms n, [1 + 2j] Cartesian index,
// [2 + 2j] coefficient, j < n.
void make_solid_table(std::vector<double>& tab) {
  tab.assign((kTableLMax + 1) * kSolidRows * kSolidEntry, 0.0);
  std::vector<double> C;
  for (int l = 0; l <= kTableLMax; ++l) {
    const int nc = ncart(l);
    C.assign((2 * l + 1) * nc, 0.0);
    solid_dense(l, C.data());
    for (int m = 0; m < 2 * l + 1; ++m) {
      double* e = tab.data() + (l * kSolidRows + m) * kSolidEntry;
      int n = 0;
      for (int k = 0; k < nc; ++k)
        if (C[m * nc + k] != 0.0) {
          e[1 + 2 * n] = k;
          e[2 + 2 * n] = C[m * nc + k];
          ++n;
        }
      e[0] = n;
    }
  }
}

// Row i of a group (x1, x2) of shell pair (l1, l2), n1 and n2 components of the
// shells with that x (consecutive, z increasing): iy | iz << 7 | component << 14,
// iy and iz the rows of the y and z tables.
static uint32_t side_row(int l1, int l2, int n1, int n2, int i) {
  const int z1 = i / n2, z2 = i % n2, y1 = n1 - 1 - z1, y2 = n2 - 1 - z2;
  const int c1 = (n1 - 1) * n1 / 2 + z1, c2 = (n2 - 1) * n2 / 2 + z2;
  return (uint32_t)((y1 * (l2 + 1) + y2) | ((z1 * (l2 + 1) + z2) << 7) | ((c1 * ncart(l2) + c2) << 14));
}

// The units of the bra rows of shell pair (l1, l2): groups of components with
// one (x1, x2), in blocks of 16, the blocks of a unit with one x1 + x2 (their F
// has one layout), at most 32 rows (two full blocks) and lim.rb blocks.  A unit
// is one or two blocks of one group, or one block of each of up to three.  Every
// unit costs a recursion per primitive quartet and a pass of the second
// transform, so the blocks are packed into few of them: the larger of two
// packings is dropped, that of all blocks and that which keeps two blocks of a
// group together (their operand is read once).
// Unit: 8 words {X | groups << 8 | blocks per group << 16, nuv(L - X), offset of
// the group's row in the x table (4), first block, valid rows per block (4
// bytes)}; block: 16 words (side_row; padding: the all-zero row and component
// 0x3ffff).  Units come in order of decreasing cost.
static TileTableIndex::Side make_bra_side(std::vector<uint32_t>& tab, int l1, int l2, const TileUnitLimits& lim) {
  struct Block {
    int x1, b, rows;  // group, block of the group, valid rows
  };
  struct Unit {
    int X, np, nb;
    std::vector<Block> blocks;
    double cost;
  };
  const int L = l1 + l2, trow = odd_row(L + 2);
  std::vector<Unit> units;
  for (int X = 0; X <= L; ++X) {
    // groups whose F fits beside each other
    const int fsize = tile_f_row(L - X, lim.Lk, L - X + lim.Lk + 1, 0);
    const int most = std::max(1, std::min(lim.rb, lim.fmax / fsize));
    std::vector<Unit> best;
    for (int keep = 0; keep < 2; ++keep) {
      std::vector<Unit> got;
      std::vector<Block> loose;
      for (int x1 = std::max(0, X - l2); x1 <= std::min(l1, X); ++x1) {
        const int m = (l1 - x1 + 1) * (l2 - X + x1 + 1), n = (m + 15) / 16;
        for (int b = 0; b < n; ++b) {
          const Block k{x1, b, std::min(16, m - 16 * b)};
          // two blocks of a group: always where the groups of a unit are one
          if (b + 1 < n && (keep || most == 1)) {
            const Block k2{x1, b + 1, std::min(16, m - 16 * (b + 1))};
            got.push_back(Unit{X, 1, 2, {k, k2}, 0.0});
            ++b;
          } else {
            loose.push_back(k);
          }
        }
      }
      std::stable_sort(loose.begin(), loose.end(), [](const Block& p, const Block& q) { return p.rows > q.rows; });
      std::vector<Unit> bins;
      for (const Block& k : loose) {
        Unit* to = nullptr;
        for (Unit& u : bins) {
          int rows = k.rows;
          for (const Block& o : u.blocks) rows += o.rows;
          if (rows <= 32 && (int)u.blocks.size() < most) {
            to = &u;
            break;
          }
        }
        if (!to) {
          bins.push_back(Unit{X, 0, 1, {}, 0.0});
          to = &bins.back();
        }
        to->blocks.push_back(k);
        ++to->np;
      }
      got.insert(got.end(), bins.begin(), bins.end());
      if (keep == 0 || got.size() <= best.size()) best = got;
    }
    for (Unit& u : best) {
      // per step of 4 k: products, reads, the rest
      u.cost = ((nuv(L - X) + 3) / 4) * (128.0 * u.blocks.size() + 24.0 * u.np + 60.0) + 800.0;
      units.push_back(u);
    }
  }
  std::stable_sort(units.begin(), units.end(), [](const Unit& a, const Unit& b) { return a.cost > b.cost; });
  TileTableIndex::Side side;
  side.nunits = (int)units.size();
  side.units = (int)tab.size();
  int blocks = 0;
  std::vector<uint32_t> rows;
  const uint32_t zero = (uint32_t)((l1 + 1) * (l2 + 1)), none = zero | (zero << 7) | (0x3ffffu << 14);
  for (const Unit& u : units) {
    uint32_t w[8] = {(uint32_t)(u.X | (u.np << 8) | (u.nb << 16)), (uint32_t)nuv(L - u.X), 0, 0, 0, 0, (uint32_t)blocks, 0};
    for (int i = 0; i < (int)u.blocks.size(); ++i, ++blocks) {
      const Block& k = u.blocks[i];
      const int x2 = u.X - k.x1, n1 = l1 - k.x1 + 1, n2 = l2 - x2 + 1;
      w[2 + i / u.nb] = (uint32_t)((k.x1 * (l2 + 1) + x2) * trow);
      w[7] |= (uint32_t)k.rows << (8 * i);
      for (int r = 0; r < 16; ++r) rows.push_back(r < k.rows ? side_row(l1, l2, n1, n2, 16 * k.b + r) : none);
    }
    tab.insert(tab.end(), w, w + 8);
  }
  side.nblocks = blocks;
  side.rows = (int)tab.size();
  tab.insert(tab.end(), rows.begin(), rows.end());
  side.list = 0;
  return side;
}

// The same for the columns of a ket: units of 4 or 2 blocks, each with its own
// group, so that a unit is full as far as one c + d allows.  Word 0: X | blocks
// << 8, words 2..5: one x row per block.
static TileTableIndex::Side make_ket_side(std::vector<uint32_t>& tab, int l1, int l2) {
  struct Unit {
    int X, n;
    std::vector<std::pair<int, int>> blocks;  // x1, block of the group
    double cost;
  };
  const int L = l1 + l2, trow = odd_row(L + 2);
  std::vector<Unit> units;
  for (int X = 0; X <= L; ++X) {
    std::vector<std::pair<int, int>> all;
    for (int x1 = std::max(0, X - l2); x1 <= std::min(l1, X); ++x1) {
      const int m = (l1 - x1 + 1) * (l2 - X + x1 + 1);
      for (int b = 0; 16 * b < m; ++b) all.emplace_back(x1, b);
    }
    for (size_t i = 0; i < all.size();) {
      // two blocks where the operands of more than eight t fill the registers
      Unit u{X, X < 8 && all.size() - i > 2 ? 4 : 2, {}, 0.0};
      u.blocks.assign(all.begin() + i, all.begin() + std::min(all.size(), i + u.n));
      i += u.n;
      // per step of 4 k: products and sums over t
      u.cost = ((nuv(L - X) + 3) / 4) * u.n * (128.0 + 32.0 * (X / 4 + 1)) + 800.0;
      units.push_back(u);
    }
  }
  std::stable_sort(units.begin(), units.end(), [](const Unit& a, const Unit& b) { return a.cost > b.cost; });
  TileTableIndex::Side side;
  side.nunits = (int)units.size();
  side.units = (int)tab.size();
  int blocks = 0;
  std::vector<uint32_t> rows;
  const uint32_t zero = (uint32_t)((l1 + 1) * (l2 + 1)), none = zero | (zero << 7) | (0x3ffffu << 14);
  for (const Unit& u : units) {
    uint32_t w[8] = {(uint32_t)(u.X | (u.n << 8)), (uint32_t)nuv(L - u.X), 0, 0, 0, 0, (uint32_t)blocks, 0};
    for (int b = 0; b < u.n; ++b, ++blocks) {
      const bool real = b < (int)u.blocks.size();
      const int x1 = real ? u.blocks[b].first : u.blocks[0].first, x2 = u.X - x1;
      w[2 + b] = (uint32_t)((x1 * (l2 + 1) + x2) * trow);
      const int n1 = l1 - x1 + 1, n2 = l2 - x2 + 1;
      for (int r = 0; r < 16; ++r) {
        const int i = real ? u.blocks[b].second * 16 + r : n1 * n2;
        rows.push_back(i < n1 * n2 ? side_row(l1, l2, n1, n2, i) : none);
      }
    }
    tab.insert(tab.end(), w, w + 8);
  }
  side.nblocks = blocks;
  side.rows = (int)tab.size();
  tab.insert(tab.end(), rows.begin(), rows.end());
  side.list = (int)tab.size();
  std::vector<std::vector<uint32_t>> of(kWaves);
  std::vector<double> load(kWaves, 0.0);
  for (size_t i = 0; i < units.size(); ++i) {
    const size_t w = std::min_element(load.begin(), load.end()) - load.begin();
    of[w].push_back((uint32_t)i);
    load[w] += units[i].cost;
  }
  uint32_t start = 0;
  for (int w = 0; w <= kWaves; ++w) {
    tab.push_back(start);
    if (w < kWaves) start += (uint32_t)of[w].size();
  }
  for (int w = 0; w < kWaves; ++w) tab.insert(tab.end(), of[w].begin(), of[w].end());
  return side;
}

// Coefficients hcoef of the per-axis tables (eri4_tile.h: build_htables) in operand
// order, and tables of the Cartesian integral kernels, 32-bit words:
//   uv    (u, v) in order of increasing s = u + v, then u: u | v << 8 | u << 16 | s << 24
//   qcol  per order n: t | u << 8 | s << 16 of each Hermite function, in (u, v)
//         order, t fastest, padded with zeros to whole blocks of 16
//   task  per order L: the blocks of W, most steps first: first pair (v, j) | ub << 12
//   chunk per bra order (Coulomb kernels): 4 t x 3 u of its Hermite functions: u | v << 8 | t << 16
//   item  per ket order (Coulomb kernels): 3 u of one v, longest first: v | u << 8 | values of t of the
//         first u << 16, place of its first dket (three to a t)
//   qpos  per ket order: the place of each Hermite function (in the order of W) among them
// and the sides (make_bra_side, make_ket_side).
void make_tile_tables(std::vector<uint32_t>& tab, std::vector<double>& hcoef, TileTableIndex& ix) {
  tab.clear();
  hcoef.clear();
  ix.uv = 0;
  for (int s = 0; s <= kMaxL; ++s)
    for (int u = 0; u <= s; ++u) tab.push_back((uint32_t)(u | ((s - u) << 8) | (u << 16) | (s << 24)));
  for (int st = 0; st < h_steps(kMaxL); ++st)
    for (int lane = 0; lane < 64; ++lane) {
      const int t = lane % 16 + (st < 4 ? 0 : 16), j = 4 * (st < 4 ? st : st - 2) + lane / 16;
      long double c = 0.0L;
      if (j <= t && 2 * j >= t && t <= kMaxL) {
        c = 1.0L;  // t! / (a! (t-2a)! 2^a) for a = t - j, an integer below 2^53
        for (int a = 0; a < t - j; ++a) c = c * (long double)((t - 2 * a) * (t - 2 * a - 1)) / (2.0L * (a + 1));
      }
      hcoef.push_back((double)c);
    }
  for (int n = 0; n <= 2 * kTableLMax; ++n) {
    ix.qcol[n] = (int)tab.size();
    for (int s = 0; s <= n; ++s)
      for (int u = 0; u <= s; ++u)
        for (int t = 0; t <= n - s; ++t) tab.push_back((uint32_t)(t | (u << 8) | (s << 16)));
    while ((tab.size() - ix.qcol[n]) % 16) tab.push_back(0);
  }
  for (int L = 0; L <= kMaxL; ++L) {
    ix.task[L] = (int)tab.size();
    if (L >= 16)
      for (int r = 0; r < nuv(L - 16); r += 16) tab.push_back((uint32_t)(r | (1 << 12)));
    for (int r = 0; r < nuv(L); r += 16) tab.push_back((uint32_t)r);
    ix.ntask[L] = (int)tab.size() - ix.task[L];
  }
  for (int n = 0; n <= 2 * kTableLMax; ++n) {
    ix.chunk[n] = (int)tab.size();
    for (int t = 0; t <= n; t += 4)
      for (int v = 0; v <= n - t; ++v)
        for (int u = 0; u <= n - t - v; u += 3) tab.push_back((uint32_t)(u | (v << 8) | (t << 16)));
    ix.nchunk[n] = (int)tab.size() - ix.chunk[n];
    ix.item[n] = (int)tab.size();
    std::vector<int> place((n + 1) * (n + 1), 0);
    int at = 0;
    for (int len = n + 1; len >= 1; --len)
      for (int u = 0; u <= n + 1 - len; u += 3) {
        const int v = n + 1 - len - u;
        tab.push_back((uint32_t)(v | (u << 8) | (len << 16)));
        tab.push_back((uint32_t)at);
        for (int b = 0; b < 3 && u + b <= n; ++b) place[(u + b) * (n + 1) + v] = at + b;
        at += 3 * len;
      }
    ix.nitem[n] = ((int)tab.size() - ix.item[n]) / 2;
    ix.dsize[n] = at;
    ix.qpos[n] = (int)tab.size();
    for (int s = 0; s <= n; ++s)
      for (int u = 0; u <= s; ++u)
        for (int t = 0; t <= n - s; ++t) tab.push_back((uint32_t)(place[u * (n + 1) + s - u] + 3 * t));
  }
  for (int l1 = 0; l1 <= kTableLMax; ++l1)
    for (int l2 = 0; l2 <= kTableLMax; ++l2) {
      for (int i = 0; i < kTileLimits; ++i) ix.bra[i][l1][l2] = make_bra_side(tab, l1, l2, kTileUnitLimits[i]);
      ix.ket[l1][l2] = make_ket_side(tab, l1, l2);
    }
}

}  // namespace eri4
