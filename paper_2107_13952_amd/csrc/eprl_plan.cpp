// Host planner: admissibility, intertwiner ranges, packed booster layout, global index
// windows of the 6j tables (Sec. 2 eq. (vertex-ampl); Sec. 3.1 framed algorithm, steps 1-4).
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <sstream>

#include "eprl_internal.hpp"

namespace eprl {

namespace {

// The four links of each edge; the intertwiner couples (first, second) and (third, fourth).
const int kEdgeLinks[5][4] = {
    {L12, L13, L14, L15}, {L23, L24, L25, L12}, {L34, L35, L13, L23},
    {L45, L14, L24, L34}, {L15, L25, L35, L45}};
// Virtual links of the booster of edges 2..5, in packing order.
const int kEdgeTriple[4][3] = {{L23, L24, L25}, {L34, L35, L23}, {L45, L24, L34}, {L25, L35, L45}};
// Shell coordinate of each virtual link (-1 for the four gauge-fixed links).
const int kShellSlot[10] = {-1, -1, -1, -1, 0, 1, 2, 3, 4, 5};

Range coupled(int a, int b, int c, int d) {
  Range r;
  if ((a + b + c + d) % 2) return r;
  int lo = std::max(std::abs(a - b), std::abs(c - d));
  int hi = std::min(a + b, c + d);
  if (lo > hi) return r;
  r.lo2 = lo;
  r.n = (hi - lo) / 2 + 1;
  return r;
}

// Number of values v = lo, lo + 2, ... (n of them) with |a - v| <= x <= a + v, i.e. in the
// triad (a, v, x).  All two-units.
int triad_count(int lo, int n, int a, int x) {
  if (n <= 0) return 0;
  const int hi = lo + 2 * (n - 1);
  const int vlo = std::max(lo, std::abs(x - a)), vhi = std::min(hi, x + a);
  if (vlo > vhi) return 0;
  if (((vlo - lo) & 1) != 0) return 0;  // parity mismatch: no value closes the triad
  return (vhi - vlo) / 2 + 1;
}

// Smallest |a - b| and largest a + b over a in range ra and fixed b.
int min_gap(Range ra, int b) {
  int hi = ra.lo2 + 2 * (ra.n - 1);
  if (b < ra.lo2) return ra.lo2 - b;
  if (b > hi) return b - hi;
  return (b - ra.lo2) % 2;  // 0 or 1: parity of the triad fixes the lowest reachable value
}

}  // namespace

int make_plan(const int two_j[10], int dl, Plan &p, std::string &err) {
  std::ostringstream msg;
  if (!two_j) {
    err = "two_j is NULL";
    return EPRL_EINVAL;
  }
  if (dl < 0) {
    err = "the number of shells dl must be >= 0";
    return EPRL_EINVAL;
  }
  for (int n = 0; n < 10; ++n) {
    if (two_j[n] < 0) {
      err = "spins must be non-negative";
      return EPRL_EINVAL;
    }
    p.two_j[n] = two_j[n];
  }
  // Spin limit: the largest virtual spin 2 (j + dl) must keep every factorial argument of
  // the 6j evaluation within the factorial table.
  int maxtwo = 0;
  for (int n = 0; n < 10; ++n) maxtwo = std::max(maxtwo, two_j[n] + 2 * dl);
  if (maxtwo > kSixjMaxTwo) {
    msg << "spin 2j + 2dl = " << maxtwo << " exceeds the supported " << kSixjMaxTwo;
    err = msg.str();
    return EPRL_ERANGE;
  }
  p.dl = dl;
  p.nd = dl + 1;
  for (int e = 0; e < 5; ++e) {
    const int *L = kEdgeLinks[e];
    p.i[e] = coupled(two_j[L[0]], two_j[L[1]], two_j[L[2]], two_j[L[3]]);
    if (p.i[e].n == 0) {
      msg << "node " << (e + 1) << " admits no intertwiner (parity or polygon inequality)";
      err = msg.str();
      return EPRL_EINVAL;
    }
  }
  const int nd = p.nd, nd3 = nd * nd * nd;
  p.nshell = (int64_t)nd3 * nd3;
  p.kr.assign(4 * nd3 * 2, 0);
  p.boff.assign(4 * (size_t)nd3 + 1, 0);
  p.kmax = 0;
  for (int e = 0; e < 4; ++e) {
    int klo = 1 << 30, khi = -1;
    for (int t = 0; t < nd3; ++t) {
      int o[3] = {t / (nd * nd), (t / nd) % nd, t % nd};
      int l[10];
      for (int n = 0; n < 10; ++n) l[n] = two_j[n];
      for (int q = 0; q < 3; ++q) l[kEdgeTriple[e][q]] += 2 * o[q];
      const int *L = kEdgeLinks[e + 1];
      Range k = coupled(l[L[0]], l[L[1]], l[L[2]], l[L[3]]);
      p.kr[(e * nd3 + t) * 2 + 0] = k.lo2;
      p.kr[(e * nd3 + t) * 2 + 1] = k.n;
      size_t slot = (size_t)e * nd3 + t;
      p.boff[slot + 1] = p.boff[slot] + (int64_t)p.i[e + 1].n * k.n;
      if (k.n > 0) {
        klo = std::min(klo, k.lo2);
        khi = std::max(khi, k.lo2 + 2 * (k.n - 1));
        p.kmax = std::max(p.kmax, k.n);
      }
    }
    if (khi < 0) {
      err = "no shell has a non-empty virtual intertwiner range";
      return EPRL_EINVAL;
    }
    p.K[e].lo2 = klo;
    p.K[e].n = (khi - klo) / 2 + 1;
  }
  // Global x window: x closes the triads (i1 l25 x), (k5 j14 x), (l35 k4 x), (l24 k3 x),
  // (j13 k2 x) of eq. (15j).
  auto spin_range = [&](int link) {
    Range r;
    r.lo2 = two_j[link];
    r.n = kShellSlot[link] < 0 ? 1 : nd;
    return r;
  };
  struct Pair {
    Range a;
    Range b;
  } pairs[5] = {{p.i[0], spin_range(L25)}, {p.K[3], spin_range(L14)}, {spin_range(L35), p.K[2]},
                {spin_range(L24), p.K[1]}, {spin_range(L13), p.K[0]}};
  int xlo = 0, xhi = 1 << 30;
  for (auto &pr : pairs) {
    int gap = 1 << 30;
    for (int q = 0; q < pr.b.n; ++q) gap = std::min(gap, min_gap(pr.a, pr.b.lo2 + 2 * q));
    xlo = std::max(xlo, gap);
    xhi = std::min(xhi, pr.a.lo2 + 2 * (pr.a.n - 1) + pr.b.lo2 + 2 * (pr.b.n - 1));
  }
  if (xlo > xhi) {
    err = "empty summation range for x";
    return EPRL_EINVAL;
  }
  p.X.lo2 = xlo;
  p.X.n = (xhi - xlo) / 2 + 1;
  int dmax = p.kmax;
  for (int e = 0; e < 5; ++e) dmax = std::max(dmax, p.i[e].n);
  p.D = dmax <= 8 ? 8 : (dmax <= 16 ? 16 : 0);
  // Largest factorial argument of any 6j in the tables: (a + b + c)/2 + 1 for a triad and the
  // sums of four entries; bounded by the largest two-spin met times 2, plus 1.
  int xmax2 = p.X.lo2 + 2 * (p.X.n - 1);
  int kmax2 = 0;
  for (int e = 0; e < 4; ++e) kmax2 = std::max(kmax2, p.K[e].lo2 + 2 * (p.K[e].n - 1));
  int imax2 = 0;
  for (int e = 0; e < 5; ++e) imax2 = std::max(imax2, p.i[e].lo2 + 2 * (p.i[e].n - 1));
  int big = std::max(std::max(maxtwo, xmax2), std::max(kmax2, imax2));
  if (big > kSixjMaxTwo) {
    msg << "a 6j argument of the tables reaches 2j = " << big << ", above the supported "
        << kSixjMaxTwo;
    err = msg.str();
    return EPRL_ERANGE;
  }
  p.fact_max = 2 * big + 2;
  // 6j table sizes (doubles): T1[nd][n_i1][nK5][NX], T2[nd][nd][nK5][nK4][NX],
  // T3[nd][nd][nd][nK4][nK3][NX], T4[nd][nd][nK3][nK2][NX], T5[nd][nK2][n_i1][NX].
  const int64_t NX = p.X.n, n1 = p.i[0].n;
  const int64_t nK2 = p.K[0].n, nK3 = p.K[1].n, nK4 = p.K[2].n, nK5 = p.K[3].n;
  p.tsize[0] = nd * n1 * nK5 * NX;
  p.tsize[1] = (int64_t)nd * nd * nK5 * nK4 * NX;
  p.tsize[2] = (int64_t)nd * nd * nd * nK4 * nK3 * NX;
  p.tsize[3] = (int64_t)nd * nd * nK3 * nK2 * NX;
  p.tsize[4] = nd * nK2 * n1 * NX;
  p.toff[0] = 0;
  for (int t = 0; t < 5; ++t) p.toff[t + 1] = p.toff[t] + ((p.tsize[t] + 31) / 32) * 32;
  p.toff[5] += 128;  // zeros: operand reads of the x-outer kernel run past a table's end
  p.a_size = 1;
  for (int e = 0; e < 5; ++e) p.a_size *= p.i[e].n;
  // Widest core windows of the factorised path.
  p.ring_w4 = p.ring_w3 = 0;
  for (int a = 0; a < nd; ++a) {
    for (int b = 0; b < nd; ++b) {
      int lo4 = 1 << 30, hi4 = -1, lo3 = 1 << 30, hi3 = -1;
      for (int o = 0; o < nd; ++o) {
        // edge 4 triple (l45, l24, l34) with (o24, o34) = (a, b)
        const int t4 = (o * nd + a) * nd + b;
        const int klo4 = p.kr[(2 * nd3 + t4) * 2], kn4 = p.kr[(2 * nd3 + t4) * 2 + 1];
        if (kn4 > 0) {
          lo4 = std::min(lo4, klo4);
          hi4 = std::max(hi4, klo4 + 2 * (kn4 - 1));
        }
        // edge 3 triple (l34, l35, l23) with (o34, o35) = (a, b)
        const int t3 = (a * nd + b) * nd + o;
        const int klo3 = p.kr[(1 * nd3 + t3) * 2], kn3 = p.kr[(1 * nd3 + t3) * 2 + 1];
        if (kn3 > 0) {
          lo3 = std::min(lo3, klo3);
          hi3 = std::max(hi3, klo3 + 2 * (kn3 - 1));
        }
      }
      if (hi4 >= 0) p.ring_w4 = std::max(p.ring_w4, (hi4 - lo4) / 2 + 1);
      if (hi3 >= 0) p.ring_w3 = std::max(p.ring_w3, (hi3 - lo3) / 2 + 1);
    }
  }
  int imaxn = 0;
  for (int e = 0; e < 5; ++e) imaxn = std::max(imaxn, p.i[e].n);
  const int w = std::max(p.ring_w4, p.ring_w3);
  p.ring_DI = imaxn <= 8 ? 8 : (imaxn <= 16 ? 16 : 0);
  p.ring_DK = p.kmax <= 8 ? 8 : (p.kmax <= 16 ? 16 : 0);
  p.ring_KW = w <= 16 ? 16 : (w <= 32 ? 32 : 0);
  if (p.ring_DI == 0 || p.ring_DK == 0 || p.ring_KW == 0 || nd > kRingMaxNd) p.ring_KW = 0;
  p.ring_cls = p.ring_KW ? ring_class(p.ring_DI, p.ring_DK, p.ring_KW) : -1;
  p.ring_cls8 = p.ring_cls;
  // The x-outer kernel for every class whose tiles fit; it runs the 16-wide classes (4..7, a boundary
  // dimension above 8) as class 8.
  if (p.ring_cls >= 0 && chain_plan(p) && p.ring_cls >= 4) p.ring_cls = kWideClass;
  return EPRL_OK;
}

int ring_schedule(const Plan &p, int target_wg, std::vector<int> &bounds,
                  std::vector<double> *chunk_cost, int core_lo, int core_hi) {
  const int nd = p.nd, nd3 = nd * nd * nd, d1 = p.i[0].n;
  const int ncore = nd * nd3;
  if (core_hi < 0) core_hi = ncore;
  const int nrange = std::max(1, core_hi - core_lo);
  const int nrb = p.ring_cls >= 0 ? ring_row_blocks(p) : 1;
  int nchunk = std::max(1, target_wg / (d1 * nrb));
  nchunk = (int)std::min<int64_t>(nchunk, std::max<int64_t>(1, (int64_t)(kRingMaxPartialBytes / ((size_t)p.a_size * sizeof(double)))));
  nchunk = std::min(nchunk, nrange);
  const int *J = p.two_j;
  const int xlo_g = p.X.lo2, xhi_g = p.X.lo2 + 2 * (p.X.n - 1);
  std::vector<double> cost((size_t)d1 * ncore, 0.0);
  for (int core = core_lo; core < core_hi; ++core) {
    // Core order of the kernels: (l24, l25, l34, l35) with l35 fastest.
    const int o24 = core / nd3, o25 = (core / (nd * nd)) % nd;
    const int o34 = (core / nd) % nd, o35 = core % nd;
    // Windows of k4 over l45 and of k3 over l23 (pairs with an empty range left out), as the
    // kernel forms them.
    int w4lo = 1 << 30, w4hi = -1, w3lo = 1 << 30, w3hi = -1;
    for (int o = 0; o < nd; ++o) {
      const int t5 = (o25 * nd + o35) * nd + o, t4 = (o * nd + o24) * nd + o34;
      const int t2 = (o * nd + o24) * nd + o25, t3 = (o34 * nd + o35) * nd + o;
      const int n5 = p.kr[(3 * nd3 + t5) * 2 + 1], n4 = p.kr[(2 * nd3 + t4) * 2 + 1];
      const int n2 = p.kr[(0 * nd3 + t2) * 2 + 1], n3 = p.kr[(1 * nd3 + t3) * 2 + 1];
      if (n5 > 0 && n4 > 0) {
        const int lo = p.kr[(2 * nd3 + t4) * 2];
        w4lo = std::min(w4lo, lo);
        w4hi = std::max(w4hi, lo + 2 * (n4 - 1));
      }
      if (n2 > 0 && n3 > 0) {
        const int lo = p.kr[(1 * nd3 + t3) * 2];
        w3lo = std::min(w3lo, lo);
        w3hi = std::max(w3hi, lo + 2 * (n3 - 1));
      }
    }
    if (w4hi < 0 || w3hi < 0) {
      for (int n1 = 0; n1 < d1; ++n1) cost[(size_t)n1 * ncore + core] = 0.1;
      continue;
    }
    const int l24 = J[L24] + 2 * o24, l25 = J[L25] + 2 * o25, l35 = J[L35] + 2 * o35;
    // x runs over (i1 l25 x) in steps of 2; both windows are non-empty exactly on
    // max(w4lo - l35, l35 - w4hi) <= x <= l35 + w4hi and the same with (l24, w3).
    const int lo_w = std::max(std::max(w4lo - l35, l35 - w4hi), std::max(w3lo - l24, l24 - w3hi));
    const int hi_w = std::min(l35 + w4hi, l24 + w3hi);
    for (int n1 = 0; n1 < d1; ++n1) {
      const int i1 = p.i[0].lo2 + 2 * n1;
      const int xlo = std::max(std::abs(i1 - l25), xlo_g), xhi = std::min(i1 + l25, xhi_g);
      int lo = std::max(xlo, lo_w);
      if ((lo - xlo) & 1) ++lo;
      const int hi = std::min(xhi, hi_w);
      const int nx = hi >= lo ? (hi - lo) / 2 + 1 : 0;
      cost[(size_t)n1 * ncore + core] = 1.0 + nx;
    }
  }
  bounds.assign((size_t)d1 * (nchunk + 1), 0);
  if (chunk_cost) chunk_cost->assign((size_t)d1 * nchunk, 0.0);
  for (int n1 = 0; n1 < d1; ++n1) {
    const double *cs = cost.data() + (size_t)n1 * ncore;
    double total = 0.0;
    for (int k = core_lo; k < core_hi; ++k) total += cs[k];
    int *bd = bounds.data() + (size_t)n1 * (nchunk + 1);
    double run = 0.0;
    int k = core_lo;
    for (int ch = 1; ch < nchunk; ++ch) {
      const double target = total * ch / nchunk;
      while (k < core_hi && run + 0.5 * cs[k] < target) run += cs[k++];
      bd[ch] = k;
    }
    bd[0] = core_lo;
    bd[nchunk] = core_hi;
    if (chunk_cost)
      for (int ch = 0; ch < nchunk; ++ch)
        for (int q = bd[ch]; q < bd[ch + 1]; ++q)
          (*chunk_cost)[(size_t)n1 * nchunk + ch] += cost[(size_t)n1 * ncore + q];
  }
  return nchunk;
}

int chain_schedule(const Plan &p, int target_wg, std::vector<int> &bounds,
                   std::vector<double> *chunk_cost, int core_lo, int core_hi) {
  const int nd = p.nd, nd2 = nd * nd, d1 = p.i[0].n, nx = p.X.n;
  const int ncore = nd2 * nd2;
  if (core_hi < 0) core_hi = ncore;
  const bool all = core_lo == 0 && core_hi == ncore;
  const int *J = p.two_j;
  const ChainGeom &g = p.ch;
  const int w4lo = p.K[2].lo2, w4hi = w4lo + 2 * (p.K[2].n - 1);
  const int w3lo = p.K[1].lo2, w3hi = w3lo + 2 * (p.K[1].n - 1);
  // Cost of the pairs (unit, l34) with non-empty windows, in matrix-core steps of a wavefront: the
  // update and P, and about as much again as thirty of them for the G / H stage and the barrier.
  auto pair_cost = [&](int o24, int xi, int o35, int o34) {
    const int x = p.X.lo2 + 2 * xi, l24 = J[L24] + 2 * o24, l34 = J[L34] + 2 * o34, l35 = J[L35] + 2 * o35;
    const int a4 = std::max(std::max(std::abs(l24 - l34), std::abs(l35 - x)), w4lo);
    const int a3 = std::max(std::max(std::abs(l34 - l35), std::abs(l24 - x)), w3lo);
    const int n4 = (std::min(std::min(l24 + l34, l35 + x), w4hi) - a4) / 2 + 1;
    const int n3 = (std::min(std::min(l34 + l35, l24 + x), w3hi) - a3) / 2 + 1;
    if (a4 > std::min(std::min(l24 + l34, l35 + x), w4hi) || a3 > std::min(std::min(l34 + l35, l24 + x), w3hi))
      return 0.0;
    const int s4 = (n4 + 3) / 4, s3 = (n3 + 3) / 4, nq = (n3 + 15) / 16;
    return 30.0 + g.ctb * s3 + nq * s4;
  };
  std::vector<double> unit((size_t)nd * nx * nd, 0.0);  // [o24][x][o35], every l34
  for (int o24 = 0; o24 < nd; ++o24)
    for (int xi = 0; xi < nx; ++xi)
      for (int o35 = 0; o35 < nd; ++o35) {
        double c = 0.0;
        for (int o34 = 0; o34 < nd; ++o34) c += pair_cost(o24, xi, o35, o34);
        unit[((size_t)o24 * nx + xi) * nd + o35] = c > 0.0 ? c + 15.0 : 0.05;
      }
  // Units of a core range: those of its (l24, l25) pairs; a partial pair keeps the whole pair's cost.
  const int pair_lo = core_lo / nd2, pair_hi = core_hi > core_lo ? (core_hi + nd2 - 1) / nd2 : pair_lo;
  const int u_lo = pair_lo * nx * nd, u_hi = (all ? nd2 : pair_hi) * nx * nd;
  // Every workgroup writes a slice of A that the reduction reads: about 3.6 ps an entry for both, and 10 ns a
  // chunk for the serial part of the reduction.  A step of one wavefront takes 65 ps of the whole chip (256
  // CUs).  With r rounds of the resident workgroups about half a chunk's time is lost at the end, so
  // r = sqrt(work / (2 slices of a round)) balances the two; whole rounds, as the chunks cost about the same
  // (two_j = 12 .. 14, 1 shell 260 us at 1.1 rounds, 212 at one), and one where r is below two (r = 1.9:
  // two_j = 1, 9 shells 154 us at one, 179 at two; spins 2 .. 11 / 2, 6 shells 131 and 139).  With all of
  // target_wg, or every unit by itself, for whatever work: two_j = 12, 1 shell 343 us at 1300 workgroups, 204
  // at 256 (ring.hip's kernels 246); two_j = 6, 3 shells 158 us at 5800, 100 at 1024; two_j = 8, 3 shells 393
  // at 5100, 302 at 2048; two_j = 6, 8 shells and two_j = 10 .. 14, 6 shells are fastest, and flat, from 4096
  // to 16384.
  double work = 0.0;
  for (int o24 = pair_lo / nd; o24 < nd && o24 * nd < pair_hi; ++o24)
    for (int xi = 0; xi < nx; ++xi) {
      double c = 0.0;
      for (int o35 = 0; o35 < nd; ++o35) c += unit[((size_t)o24 * nx + xi) * nd + o35];
      for (int o25 = 0; o25 < nd; ++o25)
        if (o24 * nd + o25 >= pair_lo && o24 * nd + o25 < pair_hi)
          work += c * triad_count(p.i[0].lo2, d1, J[L25] + 2 * o25, p.X.lo2 + 2 * xi);
    }
  const double slices = g.resident * (3.6e-3 * ((double)p.a_size / (d1 * g.nrb)) + 10.0 / (d1 * g.nrb));
  const double rounds = std::sqrt(65e-3 * work * g.nrb * g.waves / (2.0 * slices));
  if (target_wg >= g.resident)
    target_wg = g.resident * (rounds < 2.0 ? 1 : (int)std::min<double>(rounds + 0.5, target_wg / g.resident));
  int nchunk = std::max(1, target_wg / (d1 * g.nrb));
  nchunk = (int)std::min<int64_t>(nchunk, std::max<int64_t>(1, (int64_t)(kRingMaxPartialBytes / ((size_t)p.a_size * sizeof(double)))));
  nchunk = std::min(nchunk, std::max(1, u_hi - u_lo));
  bounds.assign((size_t)d1 * (nchunk + 1), 0);
  if (chunk_cost) chunk_cost->assign((size_t)d1 * nchunk, 0.0);
  std::vector<double> cs((size_t)std::max(0, u_hi - u_lo));
  for (int n1 = 0; n1 < d1; ++n1) {
    const int i1 = p.i[0].lo2 + 2 * n1;
    double total = 0.0;
    size_t k = 0;
    for (int pr = pair_lo; pr < (all ? nd2 : pair_hi); ++pr) {
      const int o24 = pr / nd, l25 = J[L25] + 2 * (pr % nd);
      for (int xi = 0; xi < nx; ++xi) {
        const int x = p.X.lo2 + 2 * xi;
        const bool live = x >= std::abs(i1 - l25) && x <= i1 + l25;
        const double *uc = unit.data() + ((size_t)o24 * nx + xi) * nd;
        for (int o35 = 0; o35 < nd; ++o35) total += cs[k++] = live ? uc[o35] : 0.01;
      }
    }
    int *bd = bounds.data() + (size_t)n1 * (nchunk + 1);
    double run = 0.0;
    int q = 0;
    const int nu = u_hi - u_lo;
    for (int ch = 1; ch < nchunk; ++ch) {
      const double target = total * ch / nchunk;
      while (q < nu && run + 0.5 * cs[q] < target) run += cs[q++];
      bd[ch] = u_lo + q;
    }
    bd[0] = u_lo;
    bd[nchunk] = u_hi;
    if (chunk_cost)
      for (int ch = 0; ch < nchunk; ++ch)
        for (int u = bd[ch]; u < bd[ch + 1]; ++u) (*chunk_cost)[(size_t)n1 * nchunk + ch] += cs[u - u_lo];
  }
  return nchunk;
}

void count_terms(const Plan &p, int64_t &live, double &terms) {
  const int nd = p.nd, nd3 = nd * nd * nd;
  live = 0;
  terms = 0.0;
  for (int64_t s = 0; s < p.nshell; ++s) {
    int o[6];
    int64_t r = s;
    for (int q = 5; q >= 0; --q) {
      o[q] = (int)(r % nd);
      r /= nd;
    }
    // edge triples in (o23, o24, o25, o34, o35, o45) coordinates
    const int t[4] = {(o[0] * nd + o[1]) * nd + o[2], (o[3] * nd + o[4]) * nd + o[0],
                      (o[5] * nd + o[1]) * nd + o[3], (o[2] * nd + o[4]) * nd + o[5]};
    double prod = p.i[0].n;
    bool ok = true;
    for (int e = 0; e < 4; ++e) {
      int kn = p.kr[(e * nd3 + t[e]) * 2 + 1];
      if (kn == 0) {
        ok = false;
        break;
      }
      prod *= kn;
    }
    if (!ok) continue;
    ++live;
    terms += prod;
  }
}

void count_work(const Plan &p, double out[5]) {
  const int nd = p.nd, nd3 = nd * nd * nd;
  const int *J = p.two_j;
  const int d1 = p.i[0].n, d2 = p.i[1].n, d3 = p.i[2].n, d4 = p.i[3].n, d5 = p.i[4].n;
  const int xlo = p.X.lo2, xhi = p.X.lo2 + 2 * (p.X.n - 1);
  double terms = 0, modes = 0, xterms = 0;
  for (int64_t s = 0; s < p.nshell; ++s) {
    int o[6];
    int64_t r = s;
    for (int q = 5; q >= 0; --q) {
      o[q] = (int)(r % nd);
      r /= nd;
    }
    const int t[4] = {(o[0] * nd + o[1]) * nd + o[2], (o[3] * nd + o[4]) * nd + o[0],
                      (o[5] * nd + o[1]) * nd + o[3], (o[2] * nd + o[4]) * nd + o[5]};
    int klo[4], kn[4];
    bool live = true;
    for (int e = 0; e < 4; ++e) {
      klo[e] = p.kr[(e * nd3 + t[e]) * 2];
      kn[e] = p.kr[(e * nd3 + t[e]) * 2 + 1];
      live = live && kn[e] > 0;
    }
    if (!live) continue;
    const double k2 = kn[0], k3 = kn[1], k4 = kn[2], k5 = kn[3];
    terms += d1 * k2 * k3 * k4 * k5;
    modes += d1 * k2 * k3 * k4 * k5 * d5 + d1 * k2 * k3 * k4 * d5 * d4 + d1 * k2 * k3 * d4 * d5 * d3 +
             d1 * k2 * d3 * d4 * d5 * d2;
    const int l24 = J[L24] + 2 * o[1], l25 = J[L25] + 2 * o[2], l35 = J[L35] + 2 * o[4];
    for (int x = xlo; x <= xhi; x += 2) {
      xterms += (double)triad_count(p.i[0].lo2, d1, l25, x) * triad_count(klo[3], kn[3], J[L14], x) *
                triad_count(klo[2], kn[2], l35, x) * triad_count(klo[1], kn[1], l24, x) *
                triad_count(klo[0], kn[0], J[L13], x);
    }
  }
  out[0] = terms;
  out[1] = 2.0 * modes + 6.0 * xterms;
  // Factorised order: useful flops and MFMA-executed flops (padded tiles), as the ring
  // kernel evaluates them: per (core, i1, x) with non-empty active k4 and k3 windows.
  double useful = 0, executed = 0;
  const int KW = p.ring_KW > 0 ? p.ring_KW : 16;
  const int DI = p.ring_DI > 0 ? p.ring_DI : 8;
  const double rows = (double)DI * DI, cols = (double)DI * DI;  // padded tile rows / columns
  for (int o24 = 0; o24 < nd; ++o24)
    for (int o25 = 0; o25 < nd; ++o25)
      for (int o34 = 0; o34 < nd; ++o34)
        for (int o35 = 0; o35 < nd; ++o35) {
          const int l24 = J[L24] + 2 * o24, l25 = J[L25] + 2 * o25;
          const int l34 = J[L34] + 2 * o34, l35 = J[L35] + 2 * o35;
          (void)l34;
          int lo5[64], n5[64], lo4[64], n4[64], lo2[64], n2[64], lo3[64], n3[64];
          int w4lo = 1 << 30, w4hi = -1, w3lo = 1 << 30, w3hi = -1;
          for (int o = 0; o < nd && o < 64; ++o) {
            const int t5 = (o25 * nd + o35) * nd + o, t4 = (o * nd + o24) * nd + o34;
            const int t2 = (o * nd + o24) * nd + o25, t3 = (o34 * nd + o35) * nd + o;
            lo5[o] = p.kr[(3 * nd3 + t5) * 2];
            n5[o] = p.kr[(3 * nd3 + t5) * 2 + 1];
            lo4[o] = p.kr[(2 * nd3 + t4) * 2];
            n4[o] = p.kr[(2 * nd3 + t4) * 2 + 1];
            lo2[o] = p.kr[(0 * nd3 + t2) * 2];
            n2[o] = p.kr[(0 * nd3 + t2) * 2 + 1];
            lo3[o] = p.kr[(1 * nd3 + t3) * 2];
            n3[o] = p.kr[(1 * nd3 + t3) * 2 + 1];
            if (n5[o] == 0 || n4[o] == 0) n5[o] = n4[o] = 0;
            if (n2[o] == 0 || n3[o] == 0) n2[o] = n3[o] = 0;
            if (n4[o] > 0) {
              w4lo = std::min(w4lo, lo4[o]);
              w4hi = std::max(w4hi, lo4[o] + 2 * (n4[o] - 1));
            }
            if (n3[o] > 0) {
              w3lo = std::min(w3lo, lo3[o]);
              w3hi = std::max(w3hi, lo3[o] + 2 * (n3[o] - 1));
            }
          }
          if (w4hi < 0 || w3hi < 0) continue;
          for (int n1 = 0; n1 < d1; ++n1) {
            const int i1 = p.i[0].lo2 + 2 * n1;
            const int xa = std::max(std::abs(i1 - l25), xlo), xb = std::min(i1 + l25, xhi);
            for (int x = xa; x <= xb; x += 2) {
              const int a4 = std::max(w4lo, std::abs(l35 - x)), b4 = std::min(w4hi, l35 + x);
              const int a3 = std::max(w3lo, std::abs(l24 - x)), b3 = std::min(w3hi, l24 + x);
              if (a4 > b4 || a3 > b3) continue;
              const int na4 = (b4 - a4) / 2 + 1, na3 = (b3 - a3) / 2 + 1;
              for (int o = 0; o < nd && o < 64; ++o) {
                if (n5[o] > 0) {
                  const int c4 = triad_count(lo4[o], n4[o], l35, x);
                  const int c5 = triad_count(lo5[o], n5[o], J[L14], x);
                  useful += (double)d5 * c4 * (3.0 * c5 + 2.0 * d4);
                }
                if (n2[o] > 0) {
                  const int c3 = triad_count(lo3[o], n3[o], l24, x);
                  const int c2 = triad_count(lo2[o], n2[o], J[L13], x);
                  useful += (double)d2 * c3 * (3.0 * c2 + 2.0 * d3);
                }
              }
              useful += 2.0 * d5 * d4 * na4 * na3 + 2.0 * d5 * d4 * na3 * d3 * d2;
              const int s4 = ((b4 - w4lo) / 2) / 4 - ((a4 - w4lo) / 2) / 4 + 1;
              const int s3 = ((b3 - w3lo) / 2) / 4 - ((a3 - w3lo) / 2) / 4 + 1;
              if (p.chain) {
                // 16x16x4 matrix-core steps (2048 flops each) of P and the update; G and H run on
                // 4x4x4 tiles and T5, T2 are made once, neither is counted.
                const int RT = (d5 * d4 + 15) / 16, q4 = (na4 + 3) / 4, q3 = (na3 + 3) / 4;
                executed += 2048.0 * RT * p.ch.nrb * ((q3 + 3) / 4 * q4 + p.ch.ctb * q3);
              } else {
                executed += 2.0 * rows * KW * 4 * s4 + 2.0 * rows * cols * 4 * s3;
              }
            }
          }
        }
  out[2] = useful;
  out[3] = executed;
  out[4] = p.ring_cls;
}

void count_chain_work(const Plan &p, double out[2]) {
  out[0] = out[1] = 0.0;
  if (!p.chain) return;
  const int nd = p.nd, nd3 = nd * nd * nd;
  const int *J = p.two_j;
  const int d1 = p.i[0].n, d2 = p.i[1].n, d3 = p.i[2].n, d4 = p.i[3].n, d5 = p.i[4].n;
  const int xlo = p.X.lo2, xhi = xlo + 2 * (p.X.n - 1);
  auto kr = [&](int e, int t) { return Range{p.kr[(e * nd3 + t) * 2], p.kr[(e * nd3 + t) * 2 + 1]}; };
  // Values of k with the triads (a b k) and (c x k).
  auto both = [](int a, int b, int c, int x) {
    const int lo = std::max(std::abs(a - b), std::abs(c - x)), hi = std::min(a + b, c + x);
    return hi < lo || ((a + b + c + x) & 1) ? 0 : (hi - lo) / 2 + 1;
  };
  auto add = [](Range &w, Range r) {  // hull of the windows of several spins
    const int lo = w.n > 0 ? std::min(w.lo2, r.lo2) : r.lo2;
    const int hi = std::max(w.n > 0 ? w.lo2 + 2 * (w.n - 1) : lo, r.lo2 + 2 * (r.n - 1));
    w = Range{lo, (hi - lo) / 2 + 1};
  };
  for (int o25 = 0; o25 < nd; ++o25)
    for (int x = xlo; x <= xhi; x += 2) {
      const int n1 = triad_count(p.i[0].lo2, d1, J[L25] + 2 * o25, x);
      if (n1 == 0) continue;
      for (int o = 0; o < nd; ++o)
        for (int q = 0; q < nd; ++q) {
          // T5: (l25, x, l35 = q), l45 = o; T2: (l24 = q, l25, x), l23 = o
          const Range k5 = kr(3, (o25 * nd + q) * nd + o), k2 = kr(0, (o * nd + q) * nd + o25);
          out[1] += 3.0 * n1 * d5 * both(J[L45] + 2 * o, J[L14], J[L35] + 2 * q, x) * triad_count(k5.lo2, k5.n, J[L14], x);
          out[1] += 3.0 * n1 * d2 * both(J[L23] + 2 * o, J[L13], J[L24] + 2 * q, x) * triad_count(k2.lo2, k2.n, J[L13], x);
        }
      for (int o24 = 0; o24 < nd; ++o24)
        for (int o34 = 0; o34 < nd; ++o34)
          for (int o35 = 0; o35 < nd; ++o35) {
            const int l24 = J[L24] + 2 * o24, l35 = J[L35] + 2 * o35;
            double g = 0.0, h = 0.0;
            Range w4, w3;
            for (int o = 0; o < nd; ++o) {
              const Range k4 = kr(2, (o * nd + o24) * nd + o34), k3 = kr(1, (o34 * nd + o35) * nd + o);
              if (k4.n > 0 && kr(3, (o25 * nd + o35) * nd + o).n > 0) {
                add(w4, k4);
                g += triad_count(k4.lo2, k4.n, l35, x);
              }
              if (k3.n > 0 && kr(0, (o * nd + o24) * nd + o25).n > 0) {
                add(w3, k3);
                h += triad_count(k3.lo2, k3.n, l24, x);
              }
            }
            const double a4 = triad_count(w4.lo2, w4.n, l35, x), a3 = triad_count(w3.lo2, w3.n, l24, x);
            if (a4 > 0 && a3 > 0)
              out[0] += 2.0 * n1 * (d5 * d4 * g + d2 * d3 * h + d5 * d4 * a4 * a3 + (double)d5 * d4 * a3 * d3 * d2);
          }
    }
}

// Booster blocks of a configuration in packing order (eq. (booster); edges 2..5, offset
// triples of their virtual links): the boundary and virtual spins of the edge's four links,
// the intertwiner ranges and the block's offset in the packed buffer.  Empty blocks are left out.
void booster_blocks(const Plan &p, std::vector<BoosterBlock> &out) {
  out.clear();
  const int nd = p.nd, nd3 = nd * nd * nd;
  for (int e = 0; e < 4; ++e)
    for (int t = 0; t < nd3; ++t) {
      const int kn = p.kr[(e * nd3 + t) * 2 + 1];
      if (kn == 0 || p.i[e + 1].n == 0) continue;
      const int o[3] = {t / (nd * nd), (t / nd) % nd, t % nd};
      int l[10];
      for (int n = 0; n < 10; ++n) l[n] = p.two_j[n];
      for (int q = 0; q < 3; ++q) l[kEdgeTriple[e][q]] += 2 * o[q];
      BoosterBlock b;
      b.edge = e;
      const int *L = kEdgeLinks[e + 1];
      for (int a = 0; a < 4; ++a) {
        b.jb[a] = p.two_j[L[a]];
        b.lb[a] = l[L[a]];
      }
      b.two_ilo = p.i[e + 1].lo2;
      b.idim = p.i[e + 1].n;
      b.two_klo = p.kr[(e * nd3 + t) * 2];
      b.kdim = kn;
      b.off = p.boff[(size_t)e * nd3 + t];
      out.push_back(b);
    }
}

}  // namespace eprl
