// FP64 6j symbols on the device and the five 6j tables of the vertex computation
// (Sec. 3.1 framed algorithm, step 4; the tensors S of eq. (15j)).
//
// Racah's single-sum formula (Racah 1942):
//   {a b c; d e f} = sqrt(P) sum_t (-1)^t (t+1)! / [prod_i (t - alpha_i)! prod_j (beta_j - t)!]
//   alpha = (a+b+c, a+e+f, d+b+f, d+e+c),  beta = (a+b+d+e, a+c+d+f, b+c+e+f),
//   P = prod over the four triads (x y z) of (x+y-z)! (x-y+z)! (-x+y+z)! / (x+y+z+1)!.
//
// Evaluation, designed so that the result is within a few ulp of the exact value:
//  * The common factor sqrt(P) * T0 (T0 = |first term|) is a product of sqrt(n!) and 1 / sqrt(n!),
//    squared for T0, from a table of both in double-double with a separate binary exponent.  The
//    table's error grows by 2^-104 per factor of n!, so 24 factors of n <= 400 stay within 2^-90.
//    (Assembling the factor from prime exponents took a loop over all primes, 23 exponent
//    reads and a power for each: 224 us for the tables at two_j = 6, 8 shells, now 50 us with the slices of ring_table_slice.)
//  * The remaining sum is 1 + r_0 + r_0 r_1 + ... with exact integer ratios
//    r_t = -(t+2) prod_j (beta_j - t) / prod_i (t + 1 - alpha_i); the ratios and the running
//    products and sum are carried in double-double, which removes the effect of the
//    alternating-sign cancellation at the spins handled here.
// Double-double primitives follow Dekker (1971) and Knuth (TAOCP vol. 2, 4.2.2).
#include "dd.hpp"
#include "eprl_internal.hpp"

#pragma clang fp contract(off)  // (dd.hpp)

namespace eprl {

namespace {

// Running product of factors sqrt(n!) and 1 / sqrt(n!): m * 2^e.
struct FactProduct {
  dd m{1.0, 0.0};
  int e = 0;
  __device__ __forceinline__ void times(const FactTables &ft, int n) {
    const double4 f = ft.f[n];
    m = dd_mul(m, {f.x, f.y});
    e += ft.e[n];
  }
  __device__ __forceinline__ void over(const FactTables &ft, int n) {
    const double4 f = ft.f[n];
    m = dd_mul(m, {f.z, f.w});
    e -= ft.e[n];
  }
  __device__ __forceinline__ void triad(const FactTables &ft, int x, int y, int z) {
    times(ft, (x + y - z) / 2);
    times(ft, (x - y + z) / 2);
    times(ft, (-x + y + z) / 2);
    over(ft, (x + y + z) / 2 + 1);
    __builtin_amdgcn_sched_barrier(0);  // (the table reads of all factors at once spill)
  }
};

__device__ __forceinline__ bool triad_ok(int a, int b, int c) {
  return ((a + b + c) & 1) == 0 && c >= (a > b ? a - b : b - a) && c <= a + b;
}

// {a b c; d e f}, all arguments in two-units.
__device__ __forceinline__ double sixj_device(int a, int b, int c, int d, int e, int f, FactTables ft) {
  if (!(triad_ok(a, b, c) && triad_ok(a, e, f) && triad_ok(d, b, f) && triad_ok(d, e, c)))
    return 0.0;
  const int al[4] = {(a + b + c) / 2, (a + e + f) / 2, (d + b + f) / 2, (d + e + c) / 2};
  const int be[3] = {(a + b + d + e) / 2, (a + c + d + f) / 2, (b + c + e + f) / 2};
  int tmin = al[0], tmax = be[0];
  for (int q = 1; q < 4; ++q) tmin = al[q] > tmin ? al[q] : tmin;
  for (int q = 1; q < 3; ++q) tmax = be[q] < tmax ? be[q] : tmax;
  FactProduct pref, first;  // sqrt(P), sqrt(T0)
  pref.triad(ft, a, b, c);
  pref.triad(ft, a, e, f);
  pref.triad(ft, d, b, f);
  pref.triad(ft, d, e, c);
  first.times(ft, tmin + 1);
  for (int q = 0; q < 4; ++q) first.over(ft, tmin - al[q]);
  __builtin_amdgcn_sched_barrier(0);
  for (int q = 0; q < 3; ++q) first.over(ft, be[q] - tmin);
  // Series in double-double.  Terms can grow far beyond the first one before they fall off:
  // the running term and sum are scaled down together by 2^-768 (exact) whenever the term
  // passes 2^768, and the scale is put back at the end.
  dd rho{1.0, 0.0}, sum{1.0, 0.0};
  int sexp = 0;
#pragma unroll 1
  for (int t = tmin; t < tmax; ++t) {
    double nu = -(double)(t + 2) * (double)(be[0] - t) * (double)(be[1] - t) * (double)(be[2] - t);
    double de = (double)(t + 1 - al[0]) * (double)(t + 1 - al[1]) * (double)(t + 1 - al[2]) *
                (double)(t + 1 - al[3]);
    rho = dd_mul(rho, dd_ratio(nu, de));
    sum = dd_add(sum, rho);
    if (__builtin_fabs(rho.hi) > 0x1p768) {
      rho = {__builtin_ldexp(rho.hi, -768), __builtin_ldexp(rho.lo, -768)};
      sum = {__builtin_ldexp(sum.hi, -768), __builtin_ldexp(sum.lo, -768)};
      sexp += 768;
    }
  }
  // value = (-1)^tmin * sqrt(P) * T0 * sum
  dd v = dd_mul(dd_mul(pref.m, dd_mul(first.m, first.m)), sum);
  double r = __builtin_ldexp(v.hi + v.lo, pref.e + 2 * first.e + sexp);
  return (tmin & 1) ? -r : r;
}

// Wigner 3jm symbol (j1 j2 j3; m1 m2 m3), arguments in two-units, by Racah's single sum
//   (-1)^(j1-j2-m3) sqrt(D(j1 j2 j3) prod_a (j_a+m_a)! (j_a-m_a)!)
//     * sum_t (-1)^t / [t! (j3-j2+t+m1)! (j3-j1+t-m2)! (j1+j2-j3-t)! (j1-t-m1)! (j2-t+m2)!],
// D(abc) = (a+b-c)! (a-b+c)! (-a+b+c)! / (a+b+c+1)!, evaluated like the 6j symbol above: the
// common factor sqrt(D prod (j +- m)!) T0 from the factorial table, the
// series 1 + r_0 + r_0 r_1 + ... with exact integer ratios in double-double.
__device__ __forceinline__ double threejm_device(int j1, int j2, int j3, int m1, int m2, int m3, FactTables ft) {
  if (m1 + m2 + m3 != 0 || !triad_ok(j1, j2, j3)) return 0.0;
  const int jj[3] = {j1, j2, j3}, mm[3] = {m1, m2, m3};
  for (int q = 0; q < 3; ++q)
    if (mm[q] > jj[q] || -mm[q] > jj[q] || ((jj[q] - mm[q]) & 1)) return 0.0;
  // Integer (not two-unit) quantities.
  const int a1 = (j1 + j2 - j3) / 2, a2 = (j1 - m1) / 2, a3 = (j2 + m2) / 2;   // (. - t)!
  const int b1 = (j3 - j2 + m1) / 2, b2 = (j3 - j1 - m2) / 2;                   // (. + t)!
  int tmin = 0, tmax = a1;
  if (-b1 > tmin) tmin = -b1;
  if (-b2 > tmin) tmin = -b2;
  if (a2 < tmax) tmax = a2;
  if (a3 < tmax) tmax = a3;
  if (tmin > tmax) return 0.0;
  FactProduct pref, first;  // sqrt(D prod (j +- m)!), sqrt(T0)
  pref.triad(ft, j1, j2, j3);
  for (int q = 0; q < 3; ++q) {
    pref.times(ft, (jj[q] + mm[q]) / 2);
    pref.times(ft, (jj[q] - mm[q]) / 2);
  }
  first.over(ft, tmin);
  first.over(ft, b1 + tmin);
  first.over(ft, b2 + tmin);
  first.over(ft, a1 - tmin);
  first.over(ft, a2 - tmin);
  first.over(ft, a3 - tmin);
  // term(t+1) / term(t) = -(a1 - t)(a2 - t)(a3 - t) / ((t + 1)(b1 + t + 1)(b2 + t + 1))
  dd rho{1.0, 0.0}, sum{1.0, 0.0};
#pragma unroll 1
  for (int t = tmin; t < tmax; ++t) {
    const double nu = -(double)(a1 - t) * (double)(a2 - t) * (double)(a3 - t);
    const double de = (double)(t + 1) * (double)(b1 + t + 1) * (double)(b2 + t + 1);
    rho = dd_mul(rho, dd_ratio(nu, de));
    sum = dd_add(sum, rho);
  }
  dd v = dd_mul(dd_mul(pref.m, dd_mul(first.m, first.m)), sum);
  const double r = __builtin_ldexp(v.hi + v.lo, pref.e + 2 * first.e);
  const int ph = (j1 - j2 - m3) / 2 + tmin;
  return (ph & 1) ? -r : r;
}

// 4jm(j1 j2 j3 j4; m1 m2 m3 m4)^(i): (j1 j2) coupled to i, then i with (j3 j4),
//   (-1)^(i - mi) (j1 j2 i; m1 m2 mi) (i j3 j4; -mi m3 m4),  mi = -(m1 + m2).
__device__ double fourjm_device(const int *j, const int *m, int i, FactTables ft) {
  const int mi = -(m[0] + m[1]);
  if (mi - m[2] - m[3] != 0) return 0.0;
  const double v = threejm_device(j[0], j[1], i, m[0], m[1], mi, ft) *
                   threejm_device(i, j[2], j[3], -mi, m[2], m[3], ft);
  return (((i - mi) / 2) & 1) ? -v : v;
}

// Coefficient tables of the booster contraction: set s (blockIdx.y), entry (m, i) of its
// M x n table = 4jm(j; m-tuple m; two_lo + 2 i).
__global__ void fourjm_table_kernel(const FourjmSet *sets, const int *mtuples, double *out,
                                    FactTables ft) {
  const FourjmSet st = sets[blockIdx.y];
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= st.M * st.n) return;
  const int m = idx / st.n, i = idx % st.n;
  out[st.out + idx] = fourjm_device(st.j, mtuples + st.mt + 4 * m, st.two_lo + 2 * i, ft);
}

__global__ void threejm_batch_kernel(const int *args, int n, double *out, FactTables ft) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n) return;
  const int *a = args + 6 * idx;
  out[idx] = threejm_device(a[0], a[1], a[2], a[3], a[4], a[5], ft);
}

// sqrt(n!) = (x + y) 2^e with x in [0.5, 1), 1 / sqrt(n!) = (z + w) 2^-e for n <= fact_max (one thread:
// each entry is the one before times sqrt(n); once per context and growth).
__global__ void fact_kernel(double4 *f, int *e, int fact_max) {
  if (threadIdx.x || blockIdx.x) return;
  dd s{1.0, 0.0};
  int es = 0;
  for (int n = 0; n <= fact_max; ++n) {
    if (n > 1) s = dd_mul(s, dd_sqrt_int((double)n));
    int k;
    const double h = __builtin_frexp(s.hi, &k);
    s = {h, __builtin_ldexp(s.lo, -k)};
    es += k;
    const double q = 1.0 / s.hi;
    const dd p = dd_mul({q, 0.0}, s);
    const dd r = dd_add({1.0, 0.0}, {-p.hi, -p.lo});
    const dd g = fast_two_sum(q, r.hi / s.hi);
    f[n] = {s.hi, s.lo, g.hi, g.lo};
    e[n] = es;
  }
}

// One thread per table entry.  Table t (0..4), its linear index decomposed row-major.
__global__ void sixj_table_kernel(TableParams tp, int64_t total) {
  int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= total) return;
  int t = 0;
  while (t < 4 && g >= tp.toff[t + 1]) ++t;
  int64_t idx = g - tp.toff[t];
  const int nd = tp.nd;
  const int *J = tp.two_j;
  const int NX = tp.NX;
  int64_t size;
  switch (t) {
    case 0: size = (int64_t)nd * tp.i1_n * tp.K_n[3] * NX; break;
    case 1: size = (int64_t)nd * nd * tp.K_n[3] * tp.K_n[2] * NX; break;
    case 2: size = (int64_t)nd * nd * nd * tp.K_n[2] * tp.K_n[1] * NX; break;
    case 3: size = (int64_t)nd * nd * tp.K_n[1] * tp.K_n[0] * NX; break;
    default: size = (int64_t)nd * tp.K_n[0] * tp.i1_n * NX; break;
  }
  if (idx >= size) return;  // alignment padding between tables
  const int x = tp.X_lo2 + 2 * (int)(idx % NX);
  int64_t r = idx / NX;
  int args[6];
  if (t == 0) {  // T1[o25][i1][k5][x] = {i1 l25 x; k5 j14 j15}
    int k5 = tp.K_lo2[3] + 2 * (int)(r % tp.K_n[3]); r /= tp.K_n[3];
    int i1 = tp.i1_lo2 + 2 * (int)(r % tp.i1_n); r /= tp.i1_n;
    int l25 = J[L25] + 2 * (int)r;
    int a6[6] = {i1, l25, x, k5, J[L14], J[L15]};
    for (int q = 0; q < 6; ++q) args[q] = a6[q];
  } else if (t == 1) {  // T2[o35][o45][k5][k4][x] = {j14 k5 x; l35 k4 l45}
    int k4 = tp.K_lo2[2] + 2 * (int)(r % tp.K_n[2]); r /= tp.K_n[2];
    int k5 = tp.K_lo2[3] + 2 * (int)(r % tp.K_n[3]); r /= tp.K_n[3];
    int l45 = J[L45] + 2 * (int)(r % nd); r /= nd;
    int l35 = J[L35] + 2 * (int)r;
    int a6[6] = {J[L14], k5, x, l35, k4, l45};
    for (int q = 0; q < 6; ++q) args[q] = a6[q];
  } else if (t == 2) {  // T3[o24][o34][o35][k4][k3][x] = {k4 l35 x; k3 l24 l34}
    int k3 = tp.K_lo2[1] + 2 * (int)(r % tp.K_n[1]); r /= tp.K_n[1];
    int k4 = tp.K_lo2[2] + 2 * (int)(r % tp.K_n[2]); r /= tp.K_n[2];
    int l35 = J[L35] + 2 * (int)(r % nd); r /= nd;
    int l34 = J[L34] + 2 * (int)(r % nd); r /= nd;
    int l24 = J[L24] + 2 * (int)r;
    int a6[6] = {k4, l35, x, k3, l24, l34};
    for (int q = 0; q < 6; ++q) args[q] = a6[q];
  } else if (t == 3) {  // T4[o23][o24][k3][k2][x] = {l24 k3 x; j13 k2 l23}
    int k2 = tp.K_lo2[0] + 2 * (int)(r % tp.K_n[0]); r /= tp.K_n[0];
    int k3 = tp.K_lo2[1] + 2 * (int)(r % tp.K_n[1]); r /= tp.K_n[1];
    int l24 = J[L24] + 2 * (int)(r % nd); r /= nd;
    int l23 = J[L23] + 2 * (int)r;
    int a6[6] = {l24, k3, x, J[L13], k2, l23};
    for (int q = 0; q < 6; ++q) args[q] = a6[q];
  } else {  // T5[o25][k2][i1][x] = {k2 j13 x; i1 l25 j12}
    int i1 = tp.i1_lo2 + 2 * (int)(r % tp.i1_n); r /= tp.i1_n;
    int k2 = tp.K_lo2[0] + 2 * (int)(r % tp.K_n[0]); r /= tp.K_n[0];
    int l25 = J[L25] + 2 * (int)r;
    int a6[6] = {k2, J[L13], x, i1, l25, J[L12]};
    for (int q = 0; q < 6; ++q) args[q] = a6[q];
  }
  tp.tables[g] = sixj_device(args[0], args[1], args[2], args[3], args[4], args[5], tp.fact);
}

// Signed, x-major tables for the factorised (ring) assembly.  The phase (-1)^R of eq. (15j)
// splits over the five closed triads (i1 j12 j13), (k2 l23 l24), (k3 l34 l35), (k4 j14 l45),
// (k5 j15 l25), each with an integer half-sum r_n; every factor goes into the one table that
// carries all of its spins, and (2x+1) goes into the first table:
//   U1[o25][x][i1][k5]  = (2x+1) (-1)^{r1 + r5} {i1 l25 x; k5 j14 j15}
//   U2[o35][o45][x][k5][k4] = (-1)^{r4} {j14 k5 x; l35 k4 l45}
//   U3[o24][o34][o35][x][k4][k3] = (-1)^{r3} {k4 l35 x; k3 l24 l34}
//   U4[o23][o24][x][k3][k2] = (-1)^{r2} {l24 k3 x; j13 k2 l23}
//   U5[o25][x][k2][i1]  = {k2 j13 x; i1 l25 j12}
// so that W(i1, k2..k5) = sum_x U1 U2 U3 U4 U5 exactly.
// One slice of a table (all but its last two indices fixed) per wavefront: the two indices' triads do not
// couple them, so the entries that are not zero are a window of rows times a window of columns; the
// lanes take those densely, after writing the zeros of the rest.  (A thread per entry spent its time
// on the 64-bit index divisions of entries that are mostly zero: 224 us for two_j = 6, 8 shells with
// 3.6 M entries, 0.5 M of them not zero; this 134 us, and 50 us with the factorial table.)
__device__ __forceinline__ void ring_table_slice(const TableParams &tp, int slice) {
  const int nd = tp.nd, NX = tp.NX;
  const int *J = tp.two_j;
  const int lane = threadIdx.x & 63;
  const int n1 = nd * NX, n2 = nd * n1, n3 = nd * n2;
  int t, s = slice;
  if (s < n3) t = 2;
  else if ((s -= n3) < n2) t = 1;
  else if ((s -= n2) < n2) t = 3;
  else if ((s -= n2) < n1) t = 0;
  else if ((s -= n1) < n1) t = 4;
  else return;
  const bool last = s == (t == 2 ? n3 : t == 1 || t == 3 ? n2 : n1) - 1;
  const int x = tp.X_lo2 + 2 * (s % NX);
  const int o0 = s / NX % nd, o1 = s / NX / nd % nd, o2 = s / NX / nd / nd;  // innermost spin offset first
  // Row and column ranges (lowest, count) of the table and the two pairs of spins that close a triad
  // with each.
  int rlo, rn, clo, cn, r0, r1, r2, r3, c0, c1, c2, c3;
  auto set = [&](int a, int b, int c, int d, int e, int f, int g, int h) {
    r0 = a; r1 = b; r2 = c; r3 = d; c0 = e; c1 = f; c2 = g; c3 = h;
  };
  int la, lb, lc = 0;
  if (t == 0) {         // {i1 l25 x; k5 j14 j15}
    la = J[L25] + 2 * o0; lb = 0;
    rlo = tp.i1_lo2; rn = tp.i1_n; clo = tp.K_lo2[3]; cn = tp.K_n[3];
    set(la, x, J[L14], J[L15], la, J[L15], J[L14], x);
  } else if (t == 1) {  // {j14 k5 x; l35 k4 l45}
    lb = J[L45] + 2 * o0; la = J[L35] + 2 * o1;
    rlo = tp.K_lo2[3]; rn = tp.K_n[3]; clo = tp.K_lo2[2]; cn = tp.K_n[2];
    set(J[L14], x, la, lb, J[L14], lb, la, x);
  } else if (t == 2) {  // {k4 l35 x; k3 l24 l34}
    lc = J[L35] + 2 * o0; lb = J[L34] + 2 * o1; la = J[L24] + 2 * o2;
    rlo = tp.K_lo2[2]; rn = tp.K_n[2]; clo = tp.K_lo2[1]; cn = tp.K_n[1];
    set(lc, x, la, lb, lc, lb, la, x);
  } else if (t == 3) {  // {l24 k3 x; j13 k2 l23}
    la = J[L24] + 2 * o0; lb = J[L23] + 2 * o1;
    rlo = tp.K_lo2[1]; rn = tp.K_n[1]; clo = tp.K_lo2[0]; cn = tp.K_n[0];
    set(la, x, J[L13], lb, la, lb, J[L13], x);
  } else {              // {k2 j13 x; i1 l25 j12}
    la = J[L25] + 2 * o0; lb = 0;
    rlo = tp.K_lo2[0]; rn = tp.K_n[0]; clo = tp.i1_lo2; cn = tp.i1_n;
    set(J[L13], x, la, J[L12], J[L13], J[L12], la, x);
  }
  // Windows [w, w + n) of positions; empty when a parity or a range does not fit.
  auto window = [](int lo, int n, int a, int b, int c, int d, int &w) {
    const int ab = a > b ? a - b : b - a, cd = c > d ? c - d : d - c;
    int kl = ab > cd ? ab : cd, kh = a + b < c + d ? a + b : c + d;
    if (((a + b + lo) & 1) || ((c + d + lo) & 1)) return 0;
    kl = kl > lo ? kl : lo;
    kh = kh < lo + 2 * (n - 1) ? kh : lo + 2 * (n - 1);
    w = (kl - lo) / 2;
    return kh < kl ? 0 : (kh - kl) / 2 + 1;
  };
  int rw = 0, cw = 0;
  int nr = window(rlo, rn, r0, r1, r2, r3, rw), nc = window(clo, cn, c0, c1, c2, c3, cw);
  if (nr == 0 || nc == 0) nr = nc = 0;
  double *out = tp.tables + tp.toff[t] + (int64_t)s * rn * cn;
  for (int q = lane; q < rn * cn; q += 64) {
    const int r = q / cn, c = q - r * cn;
    if ((unsigned)(r - rw) >= (unsigned)nr || (unsigned)(c - cw) >= (unsigned)nc) out[q] = 0.0;
  }
  // Padding: read (times zero) by operand reads that run past a table's end.
  if (last)
    for (int64_t q = tp.toff[t] + (int64_t)(s + 1) * rn * cn + lane; q < tp.toff[t + 1]; q += 64) tp.tables[q] = 0.0;
  for (int q = lane; q < nr * nc; q += 64) {
    const int r = q / nc, row = rlo + 2 * (rw + r), col = clo + 2 * (cw + q - r * nc);
    int a, b, d, e, f;  // {a b x; d e f}
    int ph;             // exponent of -1
    if (t == 0) {
      a = row; b = la; d = col; e = J[L14]; f = J[L15];
      ph = (row + J[L12] + J[L13]) / 2 + (col + J[L15] + la) / 2;
    } else if (t == 1) {
      a = J[L14]; b = row; d = la; e = col; f = lb;
      ph = (col + J[L14] + lb) / 2;
    } else if (t == 2) {
      a = row; b = lc; d = col; e = la; f = lb;
      ph = (col + lb + lc) / 2;
    } else if (t == 3) {
      a = la; b = row; d = J[L13]; e = col; f = lb;
      ph = (col + lb + la) / 2;
    } else {
      a = row; b = J[L13]; d = col; e = la; f = J[L12];
      ph = 0;
    }
    double v = sixj_device(a, b, x, d, e, f, tp.fact);
    if (t == 0) v *= (double)(x + 1);
    out[(rw + r) * cn + cw + q - r * nc] = (ph & 1) ? -v : v;
  }
}

__global__ __launch_bounds__(256) void ring_table_kernel(TableParams tp) {
  ring_table_slice(tp, __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6)));
}

// The tables of several configurations in one launch.
__global__ __launch_bounds__(256) void ring_table_batch_kernel(const TableParams *__restrict__ tps,
                                                               const BatchJob *__restrict__ jobs, int njobs) {
  int b = blockIdx.x;
  const TableParams &tp = tps[batch_job(jobs, njobs, b)];
  ring_table_slice(tp, __builtin_amdgcn_readfirstlane(b * 4 + (threadIdx.x >> 6)));
}

__global__ void sixj_batch_kernel(const int *args, int n, double *out, FactTables ft, int fact_max) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int *a = args + 6 * i;
  // Arguments beyond the factorial table are rejected by the host; guard anyway.
  int s = 0;
  for (int q = 0; q < 6; ++q) s = a[q] > s ? a[q] : s;
  if (2 * s + 2 > fact_max) {
    out[i] = __builtin_nan("");
    return;
  }
  out[i] = sixj_device(a[0], a[1], a[2], a[3], a[4], a[5], ft);
}

}  // namespace

hipError_t launch_fact_table(double4 *f, int *e, int fact_max, hipStream_t s) {
  fact_kernel<<<1, 64, 0, s>>>(f, e, fact_max);
  return hipGetLastError();
}

hipError_t launch_sixj_tables(const TableParams &tp, int64_t total, hipStream_t s) {
  int64_t blocks = (total + 255) / 256;
  sixj_table_kernel<<<(unsigned)blocks, 256, 0, s>>>(tp, total);
  return hipGetLastError();
}

hipError_t launch_ring_tables(const TableParams &tp, hipStream_t s) {
  ring_table_kernel<<<(unsigned)ring_table_blocks(tp.nd, tp.NX), 256, 0, s>>>(tp);
  return hipGetLastError();
}

// Four slices to a workgroup.
int64_t ring_table_blocks(int64_t nd, int64_t nx) { return (nd * nx * (nd * nd + 2 * nd + 2) + 3) / 4; }

hipError_t launch_ring_tables_batch(const TableParams *tps, const BatchJob *jobs, int njobs, int64_t blocks,
                                    hipStream_t s) {
  if (njobs <= 0) return hipSuccess;
  ring_table_batch_kernel<<<(unsigned)blocks, 256, 0, s>>>(tps, jobs, njobs);
  return hipGetLastError();
}

hipError_t launch_fourjm_tables(const FourjmSet *sets_dev, int nsets, int max_entries,
                                const int *mtuples_dev, double *out, FactTables ft, hipStream_t s) {
  if (nsets <= 0 || max_entries <= 0) return hipSuccess;
  dim3 grid((unsigned)((max_entries + 255) / 256), (unsigned)nsets);
  fourjm_table_kernel<<<grid, 256, 0, s>>>(sets_dev, mtuples_dev, out, ft);
  return hipGetLastError();
}

hipError_t launch_threejm_batch(const int *args, int n, double *out, FactTables ft, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  threejm_batch_kernel<<<(n + 255) / 256, 256, 0, s>>>(args, n, out, ft);
  return hipGetLastError();
}

hipError_t launch_sixj_batch(const int *args, int n, double *out, FactTables ft, int fact_max, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  sixj_batch_kernel<<<(n + 255) / 256, 256, 0, s>>>(args, n, out, ft,
                                                    fact_max);
  return hipGetLastError();
}

}  // namespace eprl
