// Factorised evaluation of the vertex tensor, eq. (vertex-ampl) with eq. (15j), one x of the
// {15j} sum at a time: the default kernel for intertwiner dimensions up to 16.
//
// For a fixed i1 and x the sum over the virtual intertwiners is the chain
//   T5(l45; i5, k4) = sum_k5 U1(i1, k5) M5(i5, k5) U2(k5, k4)      depends on (l25, l35)
//   T2(l23; i2, k3) = sum_k2 U5(k2, i1) M2(i2, k2) U4(k3, k2)      depends on (l24, l25)
//   G(k4; i5, i4)   = sum_l45 T5(l45; i5, k4) M4(l45; i4, k4)      depends on (l24, l25, l34, l35)
//   H(k3; i3, i2)   = sum_l23 M3(l23; i3, k3) T2(l23; i2, k3)
//   P(k3; i5, i4)   = sum_k4 U3(k4, k3) G(k4; i5, i4)
//   A(i1; i5 i4, i3 i2) += sum_k3 P(k3; i5, i4) H(k3; i3, i2)
// (M_e = (2k_e + 1) B_e, U = signed 6j tables).  T5 does not depend on l24 and l34, T2 not on l34
// and l35: with x outside the sums over the virtual spins both are made once, by
// chain_prep_kernel, instead of once per (l24, l25, l34, l35) and x; so are the weighted boosters
// M4 and M3 in the order the main kernel reads them.
//
// chain_kernel: a workgroup owns A(i1; rows, columns) (rows (i5, i4), columns (i3, i2), both packed
// densely) for a range of units (l24, l25, x, l35) and walks l34 inside a unit.  A wavefront keeps
// one or two row tiles and every column tile in matrix-core accumulators.  Per (unit, l34):
//   * G and H on v_mfma_f64_4x4x4 (four independent 4 x 4 blocks, the rate per multiply-add of the
//     16 x 16 instruction): one product of d5 x nd by nd x d4 for every k4, whose blocks lie along
//     the booster columns or, for few columns, along k4; 16 x 16 tiles would be mostly padding.  The
//     booster operand is read from global memory in the operands' order, a chunk of k4 ahead; T5 and
//     T2 of the unit are in LDS.  The chunks of both products are dealt out to the wavefronts.
//   * P transposed as U3^T G^T on v_mfma_f64_16x16x4: its result registers are the A operand of
//     the update as they stand (lane 16 g + c, register r = P(k3 = g + 4 r; row c)), so neither P
//     nor its transpose passes through LDS; U3 is read from global memory a step ahead,
//   * the update, one matrix-core step per (four k3, column tile).
// Operand entries past a window need no masks: k4 (k3) beyond a triad has a zero T row or a zero
// booster entry, so G and H are zero there and meet finite values of U3.
// What bounds it: at two_j = 6, 8 shells (7^5 outputs, 303 k steps over all i1) a call takes 1.33 ms
// here (2.61 ms for the kernel with the half chains inside the core loop), at two_j = 10 .. 14, 6
// shells 5.35 ms (12.3).  The matrix cores are busy 38 % of the cycles; a wavefront spends a third of
// its time in waits (the LDS operands of the 4 x 4 products, U3, two barriers a step) and issues 230
// scalar and 270 vector instructions a step around 52 matrix instructions.  Every variant spills 94 to
// 123 scalar registers (two sides, two steps, the unit's counters, pointers and strides are live at
// once), and each reload of one is a vector instruction.  The accumulators allow two wavefronts per
// SIMD.  Measured and not taken: G and H twice in LDS and one barrier a step (no change, fewer
// workgroups fit), 16 x 16 tiles for G and H of large dimensions (6.3 -> 6.7 ms), row blocks (each
// repeats H: 6.3 -> 11.0 ms for two), one wavefront per workgroup without barriers (1.49 -> 1.69 ms),
// rt = 1 (6.95 -> 8.36 ms: each H operand then serves one row tile).
// Lane layout (lane l = 16 g + c, measured on the device): v_mfma_f64_16x16x4 operand A[c][g],
// operand B[g][c], result register r = D[g + 4 r][c]; v_mfma_f64_4x4x4 block b = c >> 2, operand
// A[c & 3][g], operand B[g][c & 3], result D[g][c & 3].
#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "eprl_internal.hpp"

namespace eprl {

namespace {

typedef double d4v __attribute__((ext_vector_type(4)));
typedef double d2v __attribute__((ext_vector_type(2)));

// Device buffers reached through pointers held in memory are read and written as global memory
// (a generic access would also count as an LDS access in the waits).
__device__ __forceinline__ d2v ldg2(const double *p) {
  return *(const __attribute__((address_space(1))) d2v *)p;
}
// Entry off (in doubles) past a base that is the same for the whole wavefront: the address is a
// scalar base and one 32-bit offset register.
__device__ __forceinline__ double ldg_at(const double *base, uint32_t off) {
  return *(const __attribute__((address_space(1))) double *)((const __attribute__((address_space(1))) char *)base + off * 8u);
}
__device__ __forceinline__ d2v ldg2_at(const double *base, uint32_t off) {
  return *(const __attribute__((address_space(1))) d2v *)((const __attribute__((address_space(1))) char *)base + off * 8u);
}
__device__ __forceinline__ void stg(double *p, double v) { *(__attribute__((address_space(1))) double *)p = v; }

__device__ __forceinline__ int iabs(int v) { return v < 0 ? -v : v; }
__device__ __forceinline__ int imax(int a, int b) { return a > b ? a : b; }
__device__ __forceinline__ int imin(int a, int b) { return a < b ? a : b; }

// Lowest k4 of l45 = o (lowest k3 of l23 = o for the H side) in the T rows: the triad with j14 (j13),
// inside the configuration's range.
__host__ __device__ inline int chain_klo(const int *J, const int *wlo, const int *whi, bool h, int o) {
  const int d = J[h ? L23 : L45] + 2 * o - J[h ? L13 : L14], lo = d < 0 ? -d : d, q = h ? 0 : 1;
  return lo < wlo[q] ? wlo[q] : lo > whi[q] ? whi[q] : lo;
}

__device__ __forceinline__ double mfma4(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ d4v mfma(double a, double b, d4v c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

constexpr int kPrepThreads = 256;

// The pairs (o24, o25) of a core range, first .. first + n - 1, and how many o25 they hold (from that of
// the first on, cyclic).
struct PrepPairs {
  int first, n, n25;
  __host__ __device__ explicit PrepPairs(const RingParams &rp) {
    const int nd2 = rp.nd * rp.nd;
    first = rp.core_lo / nd2;
    n = rp.core_hi > rp.core_lo ? (rp.core_hi + nd2 - 1) / nd2 - first : 0;
    n25 = n < rp.nd ? n : rp.nd;
  }
};

// T5, T2 and the weighted boosters M4, M3 of one configuration.
//   T5[o25][x][o35][i1][o45][kap][S]: entry i5, k4 = max(|l45 - j14|, k4lo) + 2 kap, and zero rows behind
//   the last o45 (ChainGeom::tmid)
//   T2[o24][o25][x][i1][o23][kap][S]: entry i2, k3 = max(|l23 - j13|, k3lo) + 2 kap
//   M4[o24][o34][pos][.], k4 = max(|l24 - l34|, k4lo) + 2 pos, the entries (o45, i4) as chain_mrow says
//   M3[o34][o35][pos][.], k3 = max(|l34 - l35|, k3lo) + 2 pos, the entries (o23, i3)
// (x over the configuration's own range; entries outside a booster block or a triad are zeros; the
// (x, i1) that do not close (i1 l25 x) are not written).  One block per T5 (o25, x, o35), per T2
// (o24, o25, x), then the boosters.  T5 and T2 of the core range's pairs (o24, o25) only: a
// call for one core at two_j = 14, 10 shells takes 1102 us, 3405 with all of them (ring.hip's kernels: 2722).
__device__ __forceinline__ void chain_prep_block(const RingParams &rp, int b) {
  const int nd = rp.nd, nd3 = nd * nd * nd, nx = rp.nx, d1 = rp.i_n[0];
  const PrepPairs pr(rp);
  const int nb5 = pr.n25 * nx * nd, nb2 = pr.n * nx, nbs = (nd * nx * nd + kPrepThreads - 1) / kPrepThreads;
  const int *J = rp.two_j;
  const int NX = rp.NX, nK2 = rp.K_n[0], nK3 = rp.K_n[1], nK4 = rp.K_n[2], nK5 = rp.K_n[3];
  const int S = rp.ts;
  if (b < nb5 + nb2) {
    const bool five = b < nb5;
    if (!five) b -= nb5;
    int o24 = 0, o25, xi, o35 = 0;
    if (five) {
      o35 = b % nd;
      xi = (b / nd) % nx;
      o25 = (pr.first + b / (nd * nx)) % nd;
      b = (o25 * nx + xi) * nd + o35;
    } else {
      b += pr.first * nx;
      xi = b % nx;
      o25 = (b / nx) % nd;
      o24 = b / (nx * nd);
    }
    const int x = rp.xlo2 + 2 * xi, xg = (x - rp.X_lo2) / 2, l25 = J[L25] + 2 * o25;
    const int nt = five ? rp.n4t : rp.n3t, per = five ? rp.t5r : nd * nt;
    const int khi = five ? rp.whi[1] : rp.whi[0], jq = five ? J[L14] : J[L13];
    const int di = five ? rp.i_n[4] : rp.i_n[1];
    double *out = (five ? rp.T5 : rp.T2) + (int64_t)b * d1 * per * S;
    const FastDiv by_per(per), by_nt(nt);
    for (int q = threadIdx.x; q < d1 * per; q += kPrepThreads) {
      const int n1 = by_per(q), r = q - n1 * per, o = by_nt(r), kap = r - o * nt;
      const int i1 = rp.i_lo2[0] + 2 * n1;
      if (x < iabs(i1 - l25) || x > i1 + l25) continue;
      double *row = out + (int64_t)q * S;
      if (o >= nd) {  // the zero rows behind a slice of T5
        for (int i = 0; i < S; ++i) row[i] = 0.0;
        continue;
      }
      const int lo = chain_klo(J, rp.wlo, rp.whi, !five, o), k = lo + 2 * kap;
      const int t = five ? (o25 * nd + o35) * nd + o : (o * nd + o24) * nd + o25;  // block of M5 / M2
      const int e = five ? 3 : 0;
      const int klb = rp.kr[(e * nd3 + t) * 2], kn = rp.kr[(e * nd3 + t) * 2 + 1];
      // summed k (k5 or k2): the block's range and the triad with j14 (j13) and x
      const int ka = imax(klb, iabs(x - jq)), kb = imin(klb + 2 * (kn - 1), x + jq);
      const int c = k <= khi && kn > 0 && kb >= ka ? (kb - ka) / 2 + 1 : 0;
      double a[16];
      if (c > 0) {
        const double *pa, *pb;
        int sa, sb;
        if (five) {
          const int g0 = (ka - rp.K_lo2[3]) / 2, kg = (k - rp.K_lo2[2]) / 2;
          pa = rp.U1 + (((int64_t)o25 * NX + xg) * d1 + n1) * nK5 + g0;
          sa = 1;
          pb = rp.U2 + ((((int64_t)o35 * rp.tnd + o) * NX + xg) * nK5 + g0) * nK4 + kg;
          sb = nK4;
        } else {
          const int g0 = (ka - rp.K_lo2[0]) / 2, kg = (k - rp.K_lo2[1]) / 2;
          pa = rp.U5 + (((int64_t)o25 * NX + xg) * nK2 + g0) * d1 + n1;
          sa = d1;
          pb = rp.U4 + ((((int64_t)o * rp.tnd + o24) * NX + xg) * nK3 + kg) * nK2 + g0;
          sb = 1;
        }
#pragma unroll
        for (int s = 0; s < 16; ++s)
          a[s] = s < c ? pa[s * sa] * pb[(int64_t)s * sb] * (double)(ka + 2 * s + 1) : 0.0;
      }
      const double *m = rp.B + rp.boff[e * nd3 + t] + (c > 0 ? (ka - klb) / 2 : 0);
      for (int i = 0; i < S; ++i) {
        double v = 0.0;
        if (i < di && c > 0) {
#pragma unroll
          for (int s = 0; s < 16; ++s)
            if (s < c) v += a[s] * m[(int64_t)i * kn + s];
        }
        row[i] = v;
      }
    }
    return;
  }
  b -= nb5 + nb2;
  const int rows = rp.wm + 3;  // window positions of M4 and M3
  if (b < nbs) {
    // The steps of a unit (o24, x, o35): its l34 with non-empty windows, then an empty one.
    const int t = b * kPrepThreads + threadIdx.x;
    if (t >= nd * nx * nd) return;
    const int o35 = t % nd, xi = t / nd % nx, o24 = t / (nd * nx);
    const int x = rp.xlo2 + 2 * xi, l24 = J[L24] + 2 * o24, l35 = J[L35] + 2 * o35;
    ChainStep *out = rp.steps + t * nd;
    int n = 0;
    for (int o34 = 0; o34 < nd; ++o34) {
      // The triads (k4 l24 l34), (k4 l35 x) and (k3 l34 l35), (k3 l24 x).
      const int l34 = J[L34] + 2 * o34;
      const int m4 = imax(iabs(l24 - l34), rp.wlo[1]), m3 = imax(iabs(l34 - l35), rp.wlo[0]);
      const int a4 = imax(m4, iabs(l35 - x)), a3 = imax(m3, iabs(l24 - x));
      const int b4 = imin(imin(l24 + l34, l35 + x), rp.whi[1]), b3 = imin(imin(l34 + l35, l24 + x), rp.whi[0]);
      if (a4 > b4 || a3 > b3) continue;
      ChainStep st;
      st.n4 = (b4 - a4) / 2 + 1;
      st.n3 = (b3 - a3) / 2 + 1;
      st.u3 = (((((o24 * rp.tnd + o34) * rp.tnd + o35) * NX + (x - rp.X_lo2) / 2) * nK4) + (a4 - rp.K_lo2[2]) / 2) * nK3 +
              (a3 - rp.K_lo2[1]) / 2;
      st.m4 = ((o24 * nd + o34) * rows + (a4 - m4) / 2) * rp.mr4;
      st.m3 = ((o34 * nd + o35) * rows + (a3 - m3) / 2) * rp.mr3;
      st.t5 = a4 * (S / 2);
      st.t2 = a3 * (S / 2);
      st.o34 = (short)o34;
      st.more = 1;
      out[n++] = st;
    }
    if (n > 0) out[n - 1].more = 0;
    if (n < nd) out[n].n4 = 0;
    return;
  }
  b -= nbs;
  const int64_t n4 = (int64_t)nd * nd * rows * rp.mr4, n3 = (int64_t)nd * nd * rows * rp.mr3;
  int64_t q = (int64_t)b * kPrepThreads + threadIdx.x;
  const bool four = q < n4;
  if (!four) q -= n4;
  if (!four && q >= n3) return;
  const int mr = four ? rp.mr4 : rp.mr3, di = four ? rp.i_n[3] : rp.i_n[2];
  double *out = (four ? rp.M4 : rp.M3) + q;
  int64_t r = q;
  const int e0 = (int)(r % mr);
  r /= mr;
  const int jw = di <= 4 ? 4 : di <= 8 ? 8 : 16, ks = (nd + 3) >> 2;
  int i, o;
  if (e0 < (ks >> 1) * 8 * jw) {  // [pair][g][column][group of the pair], spin value 4 (2 pair + group) + g
    const int e = e0 >> 1;
    i = e % jw;
    o = 8 * (e / (4 * jw)) + 4 * (e0 & 1) + e / jw % 4;
  } else {  // the odd last group, [g][column]
    const int e = e0 - (ks >> 1) * 8 * jw;
    i = e % jw;
    o = 4 * (ks - 1) + e / jw;
  }
  const int pos = (int)(r % rows);
  r /= rows;
  const int c1 = (int)(r % nd), c0 = (int)(r / nd);
  double v = 0.0;
  if (o < nd && i < di) {
    // M4: (c0, c1) = (o24, o34), o = o45; M3: (c0, c1) = (o34, o35), o = o23
    const int t = four ? (o * nd + c0) * nd + c1 : (c0 * nd + c1) * nd + o, e = four ? 2 : 1;
    const int klb = rp.kr[(e * nd3 + t) * 2], kn = rp.kr[(e * nd3 + t) * 2 + 1];
    const int lo = four ? imax(iabs(J[L24] + 2 * c0 - J[L34] - 2 * c1), rp.wlo[1])
                        : imax(iabs(J[L34] + 2 * c0 - J[L35] - 2 * c1), rp.wlo[0]);
    const int k = lo + 2 * pos, kk = (k - klb) >> 1;
    if (k >= klb && kk < kn) v = rp.B[rp.boff[e * nd3 + t] + (int64_t)i * kn + kk] * (double)(k + 1);
  }
  *out = v;
}

__global__ __launch_bounds__(kPrepThreads) void chain_prep_kernel(RingParams rp) { chain_prep_block(rp, blockIdx.x); }

// The derived tables of several configurations in one launch.
__global__ __launch_bounds__(kPrepThreads) void chain_prep_batch_kernel(const RingParams *__restrict__ cfgs,
                                                                        const BatchJob *__restrict__ jobs, int njobs) {
  int b = blockIdx.x;
  const RingParams &rp = cfgs[batch_job(jobs, njobs, b)];
  chain_prep_block(rp, b);
}

typedef int i8v __attribute__((ext_vector_type(8)));
static_assert(sizeof(ChainStep) == sizeof(i8v), "a step is one eight-word scalar load");

// A step through the scalar cache (the table is not written while chain_kernel runs).
__device__ __forceinline__ ChainStep step_at(const ChainStep *p) {
  const i8v v = *(const __attribute__((address_space(4))) i8v *)p;
  ChainStep s;
  __builtin_memcpy(&s, &v, sizeof(s));
  return s;
}

// Doubles of one window position of M4 (M3): pairs of groups of four spin values, [g][column][group of
// the pair], then an odd last group, [g][column].
__host__ __device__ inline int chain_mrow(int nd, int dm) { return 4 * ((nd + 3) / 4) * (dm <= 4 ? 4 : dm <= 8 ? 8 : 16); }

// RT row tiles per wavefront, CT column tiles, KS groups of four spin values; windows of at most 32
// positions.
template <int RT, int CT, int KS>
__device__ __forceinline__ void chain_item(const RingParams &rp, int chunk, int n1, int cb, double *smem) {
  constexpr int SM = 8;                      // steps of four window positions
  // Instructions per T row group in a chunk: more in flight, more registers (two everywhere: 1.36 -> 1.51
  // ms at two_j = 6, 8 shells; four everywhere: spills from 14 accumulator tiles on, 6.78 -> 6.95 ms at
  // two_j = 10 .. 14, 6 shells).
  constexpr int NB = RT * CT >= 14 ? 2 : 4;
  constexpr int HG = RT * CT >= 18 ? 2 : 4;  // columns of H in flight (registers)
  const int tid = threadIdx.x, nthr = blockDim.x, nw = nthr >> 6;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, g = l >> 4, c = l & 15;
  const int nd = rp.nd, nx = rp.nx;
  const int d1 = rp.i_n[0], d2 = rp.i_n[1], d3 = rp.i_n[2], d4 = rp.i_n[3], d5 = rp.i_n[4];
  const int R = d5 * d4, C = d3 * d2;
  const int sig0 = cb * rp.ctb * 16, CW = imin(C - sig0, rp.ctb * 16);  // columns of this block
  const int S = rp.ts, t5n = rp.t5r * S, t2n = nd * rp.n3t * S;
  // LDS: T rows of the unit between zero rows (a k outside a spin's rows reads another spin's or a zero
  // row, times a zero booster entry; never a row of the other table, whose infinities or NaN, from a
  // booster entry of another edge, would then show up in entries that do not depend on it), G, H.
  double *T5s = smem + rp.tpre * S, *T2s = T5s + t5n;
  double *Gs = T2s + t2n + rp.tpost * S, *Hs = Gs + rp.sp * 8 * R;
  const int nK3 = rp.K_n[1];
  const double *U3 = rp.U3;
  const double *T5 = rp.T5 + n1 * t5n, *T2 = rp.T2 + n1 * t2n;
  const int two_i1 = rp.i_lo2[0] + 2 * n1, l25_0 = rp.two_j[L25], xlo2 = rp.xlo2;
  const int core_lo = rp.core_lo, core_hi = rp.core_hi;

  d4v acc[RT][CT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int t = 0; t < CT; ++t) acc[r][t] = d4v{0.0, 0.0, 0.0, 0.0};

  // One side of the G / H stage: T rows (dt) x booster columns (dm), one product per window position.
  // The four blocks of a v_mfma_f64_4x4x4 are 4 / 2^wp groups of four booster columns times 2^wp
  // positions; nq instructions cover the T rows (from LDS), so that no lane reads a booster entry
  // from memory that another lane of the instruction reads.  A chunk is NB instructions per T row
  // group: positions p, p + 4 and, for NB = 4, the same astep further on.
  struct Side {
    const double *M;
    int mr, wp, astep, lgs, nq;  // lgs: log2 of the positions of a chunk
    int wstep;                   // doubles of the buffer from a position to the one astep further on
    int W, rel0, relq;           // columns of the buffer; this lane's for T row group 0, step per group
    int rows;                    // T rows (none: a column of the padding)
    uint32_t mp, ms;
    int to[KS];  // T row of spin value 4 s + g, k = 0 (a spin beyond nd: times a zero booster)
    int wo;
  };
  auto make_side = [&](bool h) {
    Side q;
    const int dt = h ? d2 : d5, dm = h ? d3 : d4, wj = dm <= 4 ? 0 : dm <= 8 ? 1 : 2;
    q.M = h ? rp.M3 : rp.M4;
    q.mr = h ? rp.mr3 : rp.mr4;
    q.wp = 2 - wj;
    q.astep = q.wp == 2 ? 8 : 1 << q.wp;
    q.lgs = (NB == 4 ? 2 : 1) + q.wp;
    q.nq = (dt + 3) >> 2;
    const int b = c >> 2, bp = b >> wj, jm = 4 * (b & ((1 << wj) - 1)) + (c & 3);
    q.W = h ? CW : R;
    q.wstep = imin(q.astep, 4) * 2 * q.W;
    q.rel0 = h ? jm * d2 + g - sig0 : g * d4 + jm;
    q.relq = h ? 4 : 4 * d4;
    q.rows = jm < dm ? dt : 0;
    q.mp = bp * q.mr + ((g * 4 << wj) + jm) * 2;
    q.ms = bp * q.mr + (KS - 1) * (16 << wj) + (g * 4 << wj) + jm;
    const int nt = h ? rp.n3t : rp.n4t;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int o = imin(4 * s + g, nd - 1);
      q.to[s] = (o * nt * 2 - chain_klo(rp.two_j, rp.wlo, rp.whi, h, o)) * (S / 2) + bp * S + (c & 3);
    }
    // Entry (position p, column) of G and H: ((p >> 3) * 4 + (p & 3)) * 2 W + 2 column + (p >> 2 & 1),
    // so that the operands of two consecutive steps of four positions are one 16-byte read.
    q.wo = bp * 2 * q.W;
    return q;
  };
  const Side sg = make_side(false), sh = make_side(true);

  // Booster operands of a chunk: two groups of four spin values to a read, an odd last one by itself.
  struct Mops {
    d2v p[KS / 2 > 0 ? KS / 2 : 1][NB];
    double s[NB];
  };
  auto chunks = [&](const Side &q, int n) {
    return q.lgs >= 3 ? (n + (1 << q.lgs) - 1) >> q.lgs : ((n + 7) >> 3) << (3 - q.lgs);
  };
  auto first_of = [&](const Side &q, int ch) {
    const int sub = 3 - q.lgs;
    return sub <= 0 ? ch << q.lgs : (ch >> sub) * 8 + ((ch & ((1 << sub) - 1)) << (q.lgs - 1));
  };
  auto load_m = [&](const Side &q, int m0, int ch, Mops &m) {
    const int at = m0 + first_of(q, ch) * q.mr;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const uint32_t off = at + (i % (NB / 2) * q.astep + i / (NB / 2) * 4) * q.mr;
#pragma unroll
      for (int s = 0; s < KS / 2; ++s) m.p[s][i] = ldg2_at(q.M, q.mp + off + s * (8 * 16 >> q.wp));
      if (KS & 1) m.s[i] = ldg_at(q.M, q.ms + off);
    }
  };
  // T row groups q0 .. q0 + QN - 1 of a chunk.
  auto multiply_rows = [&](const Side &q, int (&ta)[KS], bool two, double *dst, int q0, const Mops &m, auto qn) {
    constexpr int QN = decltype(qn)::value;
    double d[QN][NB];
#pragma unroll
    for (int k = 0; k < QN; ++k)
#pragma unroll
      for (int i = 0; i < NB; ++i) d[k][i] = 0.0;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      double t[QN][NB];
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int k = 0; k < QN; ++k)
          t[k][i] = T5s[ta[s] + (i % (NB / 2) * q.astep + i / (NB / 2) * 4) * S + 4 * k];
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        if (i == NB / 2 && !two) break;
        const double b = s < (KS & ~1) ? ((s & 1) ? m.p[s / 2][i].y : m.p[s / 2][i].x) : m.s[i];
#pragma unroll
        for (int k = 0; k < QN; ++k) d[k][i] = mfma4(t[k][i], b, d[k][i]);
      }
    }
#pragma unroll
    for (int k = 0; k < QN; ++k) {
      const int rel = q.rel0 + (q0 + k) * q.relq;
      if (4 * (q0 + k) + g < q.rows && (unsigned)rel < (unsigned)q.W) {
#pragma unroll
        for (int i = 0; i < NB / 2; ++i)
          *reinterpret_cast<d2v *>(dst + i * q.wstep + 2 * rel) = d2v{d[k][i], d[k][i + NB / 2]};
      }
    }
  };
  auto multiply = [&](const Side &q, double *buf, int trow, int n, int ch, const Mops &m) {
    const int p0 = first_of(q, ch);
    const bool two = (p0 & ~7) + 4 < n;  // (else the second half is past the window)
    double *dst = buf + ((p0 >> 3) * 4 + (p0 & 3)) * 2 * q.W + q.wo;
    int ta[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) ta[s] = q.to[s] + trow + p0 * S;
    int k = 0;
    for (; k + 2 <= q.nq; k += 2) {
      multiply_rows(q, ta, two, dst, k, m, std::integral_constant<int, 2>());
#pragma unroll
      for (int s = 0; s < KS; ++s) ta[s] += 8;
    }
    if (k < q.nq) multiply_rows(q, ta, two, dst, k, m, std::integral_constant<int, 1>());
  };
  // This wavefront's chunks of a side: ch, ch + nw, ...; m holds the first one's operands.
  auto side_stage = [&](const Side &q, double *buf, int trow, int n, int m0, int ch, Mops &m) {
    const int nc = chunks(q, n);
    if (ch >= nc) return;
    for (;;) {
      const int next = ch + nw;
      if (next >= nc) break;
      Mops mx;
      load_m(q, m0, next, mx);
      multiply(q, buf, trow, n, ch, m);
      m = mx;
      ch = next;
    }
    multiply(q, buf, trow, n, ch, m);
  };
  Mops mg, mh;
  auto prefetch_m = [&](const ChainStep &st) {
    if (w < chunks(sg, st.n4)) load_m(sg, st.m4, w, mg);
    if (nw - 1 - w < chunks(sh, st.n3)) load_m(sh, st.m3, nw - 1 - w, mh);
  };
  // U3 of the first 16 k4 and k3; the rest, rare, is read where it is used (all 32 k4 a step ahead
  // spilled: 5.8 -> 5.35 ms at two_j = 10 .. 14, 6 shells).
  double u3[SM / 2];
  const uint32_t uo = g * nK3 + c;
  auto load_u3 = [&](const ChainStep &st, int k3) {
    const double *base = U3 + st.u3 + k3;
#pragma unroll
    for (int s = 0; s < SM / 2; ++s) {
      if (4 * s >= st.n4) break;
      u3[s] = ldg_at(base, uo + 4 * s * nK3);
    }
  };

  // Zero rows, and finite values wherever an operand read can run past what has been written.
  for (int q = tid; q < rp.lds; q += nthr) smem[q] = 0.0;
  // (read through scalar registers: everything derived from them is then scalar work)
  const int u0 = __builtin_amdgcn_readfirstlane(rp.bounds[n1 * (rp.nchunk + 1) + chunk]);
  const int u1 = __builtin_amdgcn_readfirstlane(rp.bounds[n1 * (rp.nchunk + 1) + chunk + 1]);
  int o35 = u0 % nd, xi = u0 / nd % nx, o25 = u0 / (nd * nx) % nd, o24 = u0 / (nd * nx * nd);
  int have2 = -1;
  for (int u = u0; u < u1;) {
    const int x = xlo2 + 2 * xi, l25 = l25_0 + 2 * o25;
    const bool closes = x >= iabs(two_i1 - l25) && x <= two_i1 + l25;
    const ChainStep *sp = rp.steps + ((o24 * nx + xi) * nd + o35) * nd;
    const int core0 = (o24 * nd + o25) * nd * nd + o35;
    const int k2 = (o24 * nd + o25) * nx + xi, k5 = (o25 * nx + xi) * nd + o35;
    const int skip = closes ? 1 : nd - o35;  // an x that does not close: its remaining l35 with it
    u += skip;
    o35 += skip;
    if (o35 == nd) {
      o35 = 0;
      if (++xi == nx) {
        xi = 0;
        if (++o25 == nd) {
          o25 = 0;
          ++o24;
        }
      }
    }
    if (!closes) continue;
    // The unit's steps (l34 with non-empty windows), those of the core range.
    ChainStep st = step_at(sp);
    while (st.n4 > 0 && st.more && core0 + st.o34 * nd < core_lo) st = step_at(++sp);
    if (st.n4 == 0 || core0 + st.o34 * nd < core_lo || core0 + st.o34 * nd >= core_hi) continue;
    prefetch_m(st);
    load_u3(st, 0);
    __syncthreads();  // every wavefront is past the previous unit's steps
    {
      const double *src = T5 + (int64_t)k5 * d1 * t5n;
#pragma unroll 4
      for (int q = tid; q < t5n / 2; q += nthr) reinterpret_cast<d2v *>(T5s)[q] = ldg2(src + 2 * q);
    }
    if (k2 != have2) {
      const double *src = T2 + (int64_t)k2 * d1 * t2n;
#pragma unroll 4
      for (int q = tid; q < t2n / 2; q += nthr) reinterpret_cast<d2v *>(T2s)[q] = ldg2(src + 2 * q);
      have2 = k2;
    }
    __syncthreads();
    for (;;) {
      // ---- G and H, the wavefronts' chunks of G from the first on, of H from the last
      side_stage(sg, Gs, st.t5, st.n4, st.m4, w, mg);
      side_stage(sh, Hs, t5n + st.t2, st.n3, st.m3, nw - 1 - w, mh);
      ChainStep sn = st;
      bool more = st.more != 0;
      if (more) {
        sn = step_at(++sp);
        more = core0 + sn.o34 * nd < core_hi;
        if (more) prefetch_m(sn);
      }
      __syncthreads();
      const int s4 = (st.n4 + 3) >> 2;
      const d2v *gp = reinterpret_cast<const d2v *>(Gs) + g * R + w * RT * 16 + c;
      const d2v *hp = reinterpret_cast<const d2v *>(Hs) + g * CW + c;
      // Sixteen k3 at a time (more than sixteen are rare, and the rows of U3 are then read in place).
      for (int k3 = 0;; k3 += 16) {
        // ---- P transposed: rows k3, columns (i5, i4)
        d4v pt[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) pt[r] = d4v{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < SM / 2; ++s) {
          if (2 * s >= s4) break;
          double ua, ub;
          if (s < SM / 4) {
            ua = u3[2 * s];
            ub = u3[2 * s + 1];
          } else {
            ua = ldg_at(U3 + st.u3 + k3, uo + 8 * s * nK3);
            ub = ldg_at(U3 + st.u3 + k3, uo + (2 * s + 1 < s4 ? 8 * s + 4 : 8 * s) * nK3);
          }
          d2v gv[RT];
#pragma unroll
          for (int r = 0; r < RT; ++r) gv[r] = gp[s * 4 * R + r * 16];
#pragma unroll
          for (int r = 0; r < RT; ++r) pt[r] = mfma(ua, gv[r].x, pt[r]);
          if (2 * s + 1 >= s4) break;
#pragma unroll
          for (int r = 0; r < RT; ++r) pt[r] = mfma(ub, gv[r].y, pt[r]);
        }
        const bool last = k3 + 16 >= st.n3;
        if (!last) load_u3(st, k3 + 16);
        else if (more) load_u3(sn, 0);
        // ---- A(i1) += P H
        const int s3 = (st.n3 - k3 + 3) >> 2;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          if (2 * s >= s3) break;
          const bool both = 2 * s + 1 < s3;
#pragma unroll
          for (int t0 = 0; t0 < CT; t0 += HG) {
            d2v hv[HG];
#pragma unroll
            for (int t = t0; t < t0 + HG && t < CT; ++t) hv[t - t0] = hp[s * 4 * CW + t * 16];
#pragma unroll
            for (int t = t0; t < t0 + HG && t < CT; ++t)
#pragma unroll
              for (int r = 0; r < RT; ++r) acc[r][t] = mfma(pt[r][2 * s], hv[t - t0].x, acc[r][t]);
            if (both) {
#pragma unroll
              for (int t = t0; t < t0 + HG && t < CT; ++t)
#pragma unroll
                for (int r = 0; r < RT; ++r) acc[r][t] = mfma(pt[r][2 * s + 1], hv[t - t0].y, acc[r][t]);
            }
          }
        }
        if (last) break;
        hp += 8 * CW;
      }
      if (!more) break;  // (the next unit begins with a barrier)
      __syncthreads();
      st = sn;
    }
  }
  // Flush the partial A(i1, ...): row (i5, i4), column (i3, i2).
  double *out = rp.partial + ((int64_t)chunk * d1 + n1) * ((int64_t)R * C);
  const FastDiv by_d2(d2), by_d4(d4);
#pragma unroll
  for (int t = 0; t < CT; ++t) {
    const int sl = t * 16 + c, sig = sig0 + sl, i3 = by_d2(sig), i2 = sig - i3 * d2;
#pragma unroll
    for (int r0 = 0; r0 < RT; ++r0)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int rho = (w * RT + r0) * 16 + g + 4 * r, i5 = by_d4(rho), i4 = rho - i5 * d4;
        if (rho < R && sl < CW) stg(out + ((i2 * d3 + i3) * d4 + i4) * d5 + i5, acc[r0][t][r]);
      }
  }
}

// Wavefronts per SIMD the registers are budgeted for, and the most wavefronts of a workgroup.
constexpr int chain_waves(int RT, int CT, int KS) {
  // Accumulators and P; booster operands; U3, addresses, operands in flight.  With 80 for the last, one
  // wavefront more for the small tiles, these spilled: 244 against 205 us for spins 3 .. 12 / 2, 5 shells.
  // Vector registers spilled as it is, of two row tiles: none up to eight column tiles with one or two spin
  // groups, from nine on 3 to 76; with three groups 2 to 20 from five column tiles on (none at seven), 122
  // and 136 at ten and eleven; with four 5 to 78 from three on, 93 and 188 at ten and eleven.  Of one row
  // tile, four for <1, 2, 2> and <1, 5, 1>, none else with up to two groups.
  const int need = 8 * RT * CT + 8 * RT + (RT * CT >= 14 ? 12 : 24) * KS + 104;
  return need <= 128 ? 4 : need <= 176 ? 3 : 2;
}
constexpr int kChainWg = 8;  // wavefronts of a workgroup

// Block b runs item b of the list (configuration, chunk, i1, column block), or, without a list,
// configuration 0's chunk b / (d1 nrb), i1 and column block from b % (d1 nrb).
template <int RT, int CT, int KS>
__global__ __launch_bounds__(kChainWg * 64, chain_waves(RT, CT, KS))
void chain_kernel(const RingParams *__restrict__ cfgs, const int *__restrict__ items) {
  extern __shared__ double smem[];
  int q0 = 0, q1, q2, q3;
  if (items) {
    const int *it = items + 4 * (int64_t)blockIdx.x;
    q0 = __builtin_amdgcn_readfirstlane(it[0]);
    q1 = __builtin_amdgcn_readfirstlane(it[1]);
    q2 = __builtin_amdgcn_readfirstlane(it[2]);
    q3 = __builtin_amdgcn_readfirstlane(it[3]);
  } else {
    const int per = cfgs[0].i_n[0] * cfgs[0].nrb, b = blockIdx.x, r = b % per;
    q1 = b / per;
    q2 = r / cfgs[0].nrb;
    q3 = r % cfgs[0].nrb;
  }
  chain_item<RT, CT, KS>(cfgs[q0], q1, q2, q3, smem);
}

// Kernel variants: row tiles per wavefront, column tiles, groups of four spin values.
// Most column tiles of a workgroup: a second column block repeats G, more tiles spill more (chain_waves).
// 16 large configurations (two spin groups, up to eleven tiles): 189, 169, 161, 159 ms with at most 8, 9, 10,
// 11.  With at most 8 against 11, ranges of cores: three groups, ten tiles 5.76 against 5.44 ms, eleven 11.38
// against 12.14; four groups, ten tiles 21.0 against 18.0 ms, eleven 36.5 against 32.2.
constexpr int kChainCT = 11;
constexpr int chain_key(int rt, int ct, int ks) { return ((rt - 1) * 16 + ct) * 4 + ks - 1; }
constexpr int kChainKeys = 2 * 64;

template <typename F>
hipError_t chain_dispatch(int key, F &&f) {
#define EPRL_K(r, c, k) \
  case chain_key(r, c, k): return f(chain_kernel<r, c, k>);
#define EPRL_C(c)                                         \
  EPRL_K(1, c, 1) EPRL_K(1, c, 2) EPRL_K(1, c, 3) EPRL_K(1, c, 4) \
  EPRL_K(2, c, 1) EPRL_K(2, c, 2) EPRL_K(2, c, 3) EPRL_K(2, c, 4)
  switch (key) {
    EPRL_C(1) EPRL_C(2) EPRL_C(3) EPRL_C(4) EPRL_C(5) EPRL_C(6) EPRL_C(7) EPRL_C(8) EPRL_C(9) EPRL_C(10) EPRL_C(11)
    default: return hipErrorInvalidValue;
  }
#undef EPRL_K
#undef EPRL_C
}

}  // namespace

bool chain_plan(Plan &p) {
  const int nd = p.nd;
  const int *J = p.two_j;
  const int d2 = p.i[1].n, d3 = p.i[2].n, d4 = p.i[3].n, d5 = p.i[4].n;
  p.chain = false;
  if (p.ring_KW == 0) return false;
  ChainGeom &g = p.ch;
  auto hi2 = [](const Range &r) { return r.lo2 + 2 * (r.n - 1); };
  // Rows of T5 / M4 per l45 and of T2 / M3 per l23; widest windows of k4 (l24, l34) and k3 (l34, l35).
  g.n4t = g.n3t = 1;
  int w = 1;
  for (int o = 0; o < nd; ++o) {
    const int l45 = J[L45] + 2 * o, l23 = J[L23] + 2 * o;
    g.n4t = std::max(g.n4t, (std::min(l45 + J[L14], hi2(p.K[2])) - std::max(std::abs(l45 - J[L14]), p.K[2].lo2)) / 2 + 1);
    g.n3t = std::max(g.n3t, (std::min(l23 + J[L13], hi2(p.K[1])) - std::max(std::abs(l23 - J[L13]), p.K[1].lo2)) / 2 + 1);
    for (int q = 0; q < nd; ++q) {
      const int l24 = J[L24] + 2 * o, l34 = J[L34] + 2 * q, m34 = J[L34] + 2 * o, l35 = J[L35] + 2 * q;
      w = std::max(w, (std::min(l24 + l34, hi2(p.K[2])) - std::max(std::abs(l24 - l34), p.K[2].lo2)) / 2 + 1);
      w = std::max(w, (std::min(m34 + l35, hi2(p.K[1])) - std::max(std::abs(m34 - l35), p.K[1].lo2)) / 2 + 1);
    }
  }
  if (w > 32) return false;
  const int R = d5 * d4, C = d3 * d2, RT = (R + 15) / 16;
  g.wm = w;
  // Rows that row offsets reach before the first T5 row, and past T5, before T2 and past T2 at the positions
  // that are used, up to three past a window's end.  Positions run up to fifteen past it: `over` rows past
  // T2's last, where G and H may lie.
  g.tpre = g.tmid = g.tpost = 0;
  int over = 0;
  const int wlo[2] = {p.K[1].lo2, p.K[2].lo2}, whi[2] = {hi2(p.K[1]), hi2(p.K[2])};
  for (int o = 0; o < nd; ++o) {
    g.tmid = std::max(g.tmid, (whi[1] + 6 - chain_klo(J, wlo, whi, false, o)) / 2 + 1 - (nd - o) * g.n4t);
    g.tmid = std::max(g.tmid, (chain_klo(J, wlo, whi, true, o) - wlo[0]) / 2 - o * g.n3t);
  }
  for (int o = 0; o < nd; ++o) {
    g.tpre = std::max(g.tpre, (chain_klo(J, wlo, whi, false, o) - wlo[1]) / 2 - o * g.n4t);
    g.tpost = std::max(g.tpost, (whi[0] + 6 - chain_klo(J, wlo, whi, true, o)) / 2 + 1 - (nd - o) * g.n3t);
    over = std::max(over, (whi[0] + 30 - chain_klo(J, wlo, whi, true, o)) / 2 + 1 - (nd - o) * g.n3t + 1);
    over = std::max(over, (whi[1] + 30 - chain_klo(J, wlo, whi, false, o)) / 2 + 1 - (nd - o) * g.n4t - g.tmid - nd * g.n3t + 1);
    g.tpre = std::max(g.tpre, (chain_klo(J, wlo, whi, true, o) - wlo[0]) / 2 - o * g.n3t - g.tmid - nd * g.n4t);
  }
  g.ts = (std::max(d5, d2) + 1) & ~1;
  g.mr4 = chain_mrow(nd, d4);
  g.mr3 = chain_mrow(nd, d3);
  g.sp = (w + 7) / 8;
  if (std::min(d3, d4) <= 4) g.sp = (g.sp + 1) & ~1;  // chunks of sixteen positions
  // Two row tiles per wavefront (each H operand serves both), all rows in one workgroup, as many
  // column blocks as keep the tiles of a wavefront and the LDS in bounds.
  const int CT = (C + 15) / 16, rt = RT > 1 ? 2 : 1;
  g.nrb = (CT + kChainCT - 1) / kChainCT;
  const int tpost = g.tpost;
  for (;; ++g.nrb) {
    if (g.nrb > CT) return false;
    g.ctb = (CT + g.nrb - 1) / g.nrb;
    g.tpost = std::max(tpost, over - g.sp * 8 * (R + std::min(C, g.ctb * 16)) / g.ts);
    if (chain_smem_bytes(p) <= kChainMaxLds) break;
  }
  g.waves = (RT + rt - 1) / rt;
  g.key = chain_key(rt, g.ctb, (nd + 3) / 4);
  g.lds = (int)(chain_smem_bytes(p) / sizeof(double));
  const int fit = std::min(4 * chain_waves(rt, g.ctb, (nd + 3) / 4) / g.waves, (int)(kChainMaxLds / chain_smem_bytes(p)));
  g.resident = 256 * std::max(1, fit);
  const int64_t nx = p.X.n, d1 = p.i[0].n;
  auto pad = [](int64_t v) { return (v + 31) / 32 * 32; };
  g.t5 = pad((int64_t)nd * nx * nd * d1 * (nd * g.n4t + g.tmid) * g.ts);
  g.t2 = pad((int64_t)nd * nd * nx * d1 * nd * g.n3t * g.ts);
  // Booster rows per (l24, l34) or (l34, l35); reads run up to 16 positions past the last.
  const int64_t rows = w + 3;
  g.m4 = pad(nd * nd * rows * g.mr4 + 16 * g.mr4);
  g.m3 = pad(nd * nd * rows * g.mr3 + 16 * g.mr3);
  g.steps = pad((int64_t)nd * nx * nd * nd * (int64_t)(sizeof(ChainStep) / sizeof(double)));
  // The steps hold 32-bit offsets into U3, M4 and M3; those into M4 and M3 are used in bytes.
  constexpr int64_t kMax = UINT32_MAX / 8;
  if (p.tsize[2] > INT32_MAX || g.m4 > kMax || g.m3 > kMax) return false;
  p.chain = true;
  return true;
}

size_t chain_smem_bytes(const Plan &p) {
  const ChainGeom &g = p.ch;
  const int R = p.i[4].n * p.i[3].n, C = p.i[2].n * p.i[1].n;
  const int CW = std::min(C, g.ctb * 16);
  // The last row of G or H is read past its end by up to 31 columns (results never used).
  return sizeof(double) * ((size_t)(p.nd * (g.n4t + g.n3t) + g.tpre + g.tmid + g.tpost) * g.ts + (size_t)g.sp * 8 * (R + CW) + 64);
}

hipError_t chain_init_attributes() {
  for (int key = 0; key < kChainKeys; ++key) {
    hipError_t e = chain_dispatch(key, [](auto k) {
      return hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kChainMaxLds);
    });
    if (e != hipSuccess && e != hipErrorInvalidValue) return e;
  }
  return hipSuccess;
}

void chain_params(const Plan &p, double *derived, RingParams &rp) {
  const ChainGeom &g = p.ch;
  rp.T5 = derived;
  rp.T2 = rp.T5 + g.t5;
  rp.M4 = rp.T2 + g.t2;
  rp.M3 = rp.M4 + g.m4;
  rp.steps = reinterpret_cast<ChainStep *>(rp.M3 + g.m3);
  rp.n4t = g.n4t;
  rp.n3t = g.n3t;
  rp.ts = g.ts;
  rp.sp = g.sp;
  rp.wm = g.wm;
  rp.tpre = g.tpre;
  rp.tpost = g.tpost;
  rp.t5r = p.nd * g.n4t + g.tmid;
  rp.lds = g.lds;
  rp.mr4 = g.mr4;
  rp.mr3 = g.mr3;
  rp.ctb = g.ctb;
  rp.nrb = g.nrb;
  rp.nx = p.X.n;
  for (int q = 0; q < 2; ++q) {
    rp.wlo[q] = p.K[1 + q].lo2;
    rp.whi[q] = p.K[1 + q].lo2 + 2 * (p.K[1 + q].n - 1);
  }
  rp.core_lo = 0;
  rp.core_hi = p.nd * p.nd * p.nd * p.nd;
}

int64_t chain_prep_blocks(const RingParams &rp) {
  const int64_t nd = rp.nd, m = nd * nd * (rp.wm + 3) * (rp.mr4 + rp.mr3);
  const PrepPairs pr(rp);
  return pr.n25 * rp.nx * nd + pr.n * rp.nx + (nd * rp.nx * nd + kPrepThreads - 1) / kPrepThreads +
         (m + kPrepThreads - 1) / kPrepThreads;
}

hipError_t launch_chain_prep(const RingParams &rp, hipStream_t s) {
  chain_prep_kernel<<<(unsigned)chain_prep_blocks(rp), kPrepThreads, 0, s>>>(rp);
  return hipGetLastError();
}

hipError_t launch_chain_prep_batch(const RingParams *cfgs, const BatchJob *jobs, int njobs, int64_t blocks,
                                   hipStream_t s) {
  if (njobs <= 0) return hipSuccess;
  chain_prep_batch_kernel<<<(unsigned)blocks, kPrepThreads, 0, s>>>(cfgs, jobs, njobs);
  return hipGetLastError();
}

hipError_t launch_chain(const RingParams *cfgs, const int *items, int nitems, int key, int waves,
                        size_t smem, hipStream_t s) {
  if (nitems <= 0) return hipSuccess;
  return chain_dispatch(key, [&](auto k) {
    k<<<(unsigned)nitems, 64 * waves, smem, s>>>(cfgs, items);
    return hipGetLastError();
  });
}

}  // namespace eprl
