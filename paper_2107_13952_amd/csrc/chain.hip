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
// What bounds it: at two_j = 6, 8 shells (7^5 outputs, 258 k steps) the matrix instructions of a
// step take about a third of its time; the rest are LDS reads of T and of G, H (a 4 x 4 x 4 operand
// serves one instruction), the two barriers and the scalar work per step, which two to three
// workgroups per CU hide only in part.  Doubling G and H in LDS (one barrier per step) was no faster
// (fewer workgroups fit).  Two row tiles per wavefront instead of one: 1800 against 1870 us for that
// tensor, 6950 against 8360 us at two_j = 10, 6 shells (each H operand is read half as often).
// Lane layout (lane l = 16 g + c, measured on the device): v_mfma_f64_16x16x4 operand A[c][g],
// operand B[g][c], result register r = D[g + 4 r][c]; v_mfma_f64_4x4x4 block b = c >> 2, operand
// A[c & 3][g], operand B[g][c & 3], result D[g][c & 3].
#include <algorithm>
#include <cstdint>

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

// Quotient by a divisor that is the same for the whole kernel, dividends below 2^16.
struct FastDiv {
  uint32_t m;
  int d;
  __device__ explicit FastDiv(int d_)
      : m(d_ > 1 ? (uint32_t)((0x100000000ull + (uint64_t)d_ - 1) / (uint64_t)d_) : 0u), d(d_) {}
  __device__ int operator()(int q) const { return d > 1 ? (int)__umulhi((uint32_t)q, m) : q; }
};

constexpr int kPrepThreads = 256;

// T5, T2 and the weighted boosters M4, M3 of one configuration.
//   T5[o25][x][o35][i1][o45][kap][S]: entry i5, k4 = max(|l45 - j14|, k4lo) + 2 kap
//   T2[o24][o25][x][i1][o23][kap][S]: entry i2, k3 = max(|l23 - j13|, k3lo) + 2 kap
//   M4[o24][o34][pos][.], k4 = max(|l24 - l34|, k4lo) + 2 pos, the entries (o45, i4) as chain_mrow says
//   M3[o34][o35][pos][.], k3 = max(|l34 - l35|, k3lo) + 2 pos, the entries (o23, i3)
// (x over the configuration's own range; entries outside a booster block or a triad are zeros; the
// (x, i1) that do not close (i1 l25 x) are not written).  One block per T5 (o25, x, o35), per T2
// (o24, o25, x), then the boosters.
__global__ __launch_bounds__(kPrepThreads) void chain_prep_kernel(RingParams rp, int nb5, int nb2, int nbs) {
  const int nd = rp.nd, nd3 = nd * nd * nd, nx = rp.nx, d1 = rp.i_n[0];
  const int *J = rp.two_j;
  const int NX = rp.NX, nK2 = rp.K_n[0], nK3 = rp.K_n[1], nK4 = rp.K_n[2], nK5 = rp.K_n[3];
  const int S = rp.ts;
  int b = blockIdx.x;
  if (b < nb5 + nb2) {
    const bool five = b < nb5;
    if (!five) b -= nb5;
    int o24 = 0, o25, xi, o35 = 0;
    if (five) {
      o35 = b % nd;
      xi = (b / nd) % nx;
      o25 = b / (nd * nx);
    } else {
      xi = b % nx;
      o25 = (b / nx) % nd;
      o24 = b / (nx * nd);
    }
    const int x = rp.xlo2 + 2 * xi, xg = (x - rp.X_lo2) / 2, l25 = J[L25] + 2 * o25;
    const int nt = five ? rp.n4t : rp.n3t, per = nd * nt;
    const int khi = five ? rp.whi[1] : rp.whi[0], jq = five ? J[L14] : J[L13];
    const int di = five ? rp.i_n[4] : rp.i_n[1];
    double *out = (five ? rp.T5 : rp.T2) + (int64_t)b * d1 * per * S;
    const FastDiv by_per(per), by_nt(nt);
    for (int q = threadIdx.x; q < d1 * per; q += kPrepThreads) {
      const int n1 = by_per(q), r = q - n1 * per, o = by_nt(r), kap = r - o * nt;
      const int i1 = rp.i_lo2[0] + 2 * n1;
      if (x < iabs(i1 - l25) || x > i1 + l25) continue;
      const int lo = chain_klo(J, rp.wlo, rp.whi, !five, o), k = lo + 2 * kap;
      const int t = five ? (o25 * nd + o35) * nd + o : (o * nd + o24) * nd + o25;  // block of M5 / M2
      const int e = five ? 3 : 0;
      const int klb = rp.kr[(e * nd3 + t) * 2], kn = rp.kr[(e * nd3 + t) * 2 + 1];
      // summed k (k5 or k2): the block's range and the triad with j14 (j13) and x
      const int ka = imax(klb, iabs(x - jq)), kb = imin(klb + 2 * (kn - 1), x + jq);
      double *row = out + (int64_t)q * S;
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

typedef int i8v __attribute__((ext_vector_type(8)));
static_assert(sizeof(ChainStep) == sizeof(i8v), "a step is one eight-word scalar load");

// A step through the scalar cache (the table is not written while chain_kernel runs).
__device__ __forceinline__ ChainStep step_at(const ChainStep *p) {
  const i8v v = *(const __attribute__((address_space(4))) i8v *)p;
  ChainStep s;
  __builtin_memcpy(&s, &v, sizeof(s));
  return s;
}

// How the four blocks of a v_mfma_f64_4x4x4 are used for the products of a side (T rows x booster
// columns, dt x dm, one product per window position): 2^wj blocks along the booster columns, 2^wp
// positions; nq instructions cover the T rows (from LDS), so that no lane reads a booster entry
// from memory that another lane of the instruction reads.
struct Blocks {
  int wj, wp, nq;
  __host__ __device__ Blocks(int dt, int dm) {
    wj = dm <= 4 ? 0 : dm <= 8 ? 1 : 2;
    wp = 2 - wj;
    nq = (dt + 3) >> 2;
  }
};

// Doubles of one window position of M4 (M3): pairs of groups of four spin values, [g][column][group of
// the pair], then an odd last group, [g][column].
__host__ __device__ inline int chain_mrow(int nd, int dm) { return 4 * ((nd + 3) / 4) * (dm <= 4 ? 4 : dm <= 8 ? 8 : 16); }

// RT row tiles per wavefront, CT column tiles; windows of at most 16 NQ positions.
template <int RT, int CT, int NQ>
__device__ __forceinline__ void chain_item(const RingParams &rp, int chunk, int n1, int rb, double *smem) {
  constexpr int SM = 4 * NQ;  // steps of four window positions
  constexpr int NB = 4;       // groups of a chunk of the G / H stage
  const int tid = threadIdx.x, nthr = blockDim.x, nw = nthr >> 6;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, g = l >> 4, c = l & 15;
  const int nd = rp.nd, nx = rp.nx;
  const int d1 = rp.i_n[0], d2 = rp.i_n[1], d3 = rp.i_n[2], d4 = rp.i_n[3], d5 = rp.i_n[4];
  const int R = d5 * d4, C = d3 * d2;
  const int rho0 = rb * rp.rtb * 16, GW = imin(R - rho0, rp.rtb * 16);  // rows of this block
  const int S = rp.ts, t5n = nd * rp.n4t * S, t2n = nd * rp.n3t * S, SP = (rp.smax + 1) / 2;
  // LDS: T rows of the unit between zero rows (a k outside a spin's rows reads another spin's or a zero
  // row, times a zero booster entry), G, H.
  double *T5s = smem + rp.tpre * S, *T2s = T5s + t5n;
  double *Gs = T2s + t2n + rp.tpost * S, *Hs = Gs + SP * 8 * GW;
  const int nK3 = rp.K_n[1], ks = (nd + 3) >> 2;
  const Blocks bg(d5, d4), bh(d2, d3);
  const int mr4 = rp.mr4, mr3 = rp.mr3;  // booster entries of one window position
  const double *M4 = rp.M4, *M3 = rp.M3, *U3 = rp.U3;
  const double *T5 = rp.T5 + n1 * t5n, *T2 = rp.T2 + n1 * t2n;
  const int two_i1 = rp.i_lo2[0] + 2 * n1, l25_0 = rp.two_j[L25], xlo2 = rp.xlo2;
  const int core_lo = rp.core_lo, core_hi = rp.core_hi;

  d4v acc[RT][CT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int t = 0; t < CT; ++t) acc[r][t] = d4v{0.0, 0.0, 0.0, 0.0};

  // This lane's block along the booster columns (bj) and the positions (bp), each side; its place in
  // the operands: spin value 4 s + g, T row (booster column) c & 3 of the block.
  const int bj4 = (c >> 2) & ((1 << bg.wj) - 1), bp4 = (c >> 2) >> bg.wj, jm4 = 4 * bj4 + (c & 3);
  const int bj3 = (c >> 2) & ((1 << bh.wj) - 1), bp3 = (c >> 2) >> bh.wj, jm3 = 4 * bj3 + (c & 3);
  const uint32_t mp4 = bp4 * mr4 + ((g * 4 << bg.wj) + jm4) * 2, ms4 = bp4 * mr4 + (g * 4 << bg.wj) + jm4;
  const uint32_t mp3 = bp3 * mr3 + ((g * 4 << bh.wj) + jm3) * 2, ms3 = bp3 * mr3 + (g * 4 << bh.wj) + jm3;
  int to4[4], to3[4];  // T rows of spin value 4 s + g for k = 0 (a spin beyond nd: times a zero booster)
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int o = imin(4 * s + g, nd - 1);
    to4[s] = (o * rp.n4t * 2 - chain_klo(rp.two_j, rp.wlo, rp.whi, false, o)) * (S / 2) + bp4 * S + (c & 3);
    to3[s] = (o * rp.n3t * 2 - chain_klo(rp.two_j, rp.wlo, rp.whi, true, o)) * (S / 2) + bp3 * S + (c & 3);
  }
  // Entry (position p, column) of G and H: ((p >> 3) * 4 + (p & 3)) * 2 W + 2 column + (p >> 2 & 1), so
  // that the operands of two consecutive steps of four positions are one 16-byte read; a lane's
  // results have T row 4 q + g and booster column jm.
  const int wo4 = bp4 * 2 * GW + 2 * (g * d4 + jm4 - rho0), wo3 = bp3 * 2 * C + 2 * (jm3 * d2 + g);

  // Booster operands of a chunk of NB groups: two groups of four spin values to a read, an odd last
  // group by itself.
  struct Mops {
    d2v p[NB];
    double s[NB];
  };
  // Chunk ch of a step: side and first position; false past the last.
  auto chunk_of = [&](const ChainStep &st, int ch, bool &h, int &pos) {
    const int cg = ((((st.n4 + 3) & ~3) >> bg.wp) + NB - 1) / NB;
    const int cht = cg + ((((st.n3 + 3) & ~3) >> bh.wp) + NB - 1) / NB;
    h = ch >= cg;
    pos = h ? ((ch - cg) * NB) << bh.wp : (ch * NB) << bg.wp;
    return ch < cht;
  };
  auto load_m = [&](const ChainStep &st, int ch, Mops &m) {
    bool h;
    int pos;
    if (!chunk_of(st, ch, h, pos)) return;
    const double *base = h ? M3 + st.m3 + pos * mr3 : M4 + st.m4 + pos * mr4;
    const int step = h ? mr3 << bh.wp : mr4 << bg.wp;
    if (ks > 1) {
#pragma unroll
      for (int i = 0; i < NB; ++i) m.p[i] = ldg2_at(base + i * step, h ? mp3 : mp4);
    }
    if (ks & 1) {
      base += (ks - 1) * (4 * 4) << (h ? bh.wj : bg.wj);
#pragma unroll
      for (int i = 0; i < NB; ++i) m.s[i] = ldg_at(base + i * step, h ? ms3 : ms4);
    }
  };
  auto multiply = [&](const ChainStep &st, int ch, const Mops &m) {
    bool h;
    int pos;
    chunk_of(st, ch, h, pos);
    const int wp = h ? bh.wp : bg.wp, nq = h ? bh.nq : bg.nq;
    const int np = ((h ? st.n3 : st.n4) + 3) & ~3, W = h ? C : GW;
    const double *Ts = (h ? T2s + st.t2 : T5s + st.t5) + pos * S;
    double *dst = (h ? Hs + wo3 : Gs + wo4);
    d2v m2[NB];  // spin values 8 .. 15 when there are four groups of them
    if (ks == 4) {
      const double *base = (h ? M3 + st.m3 + pos * mr3 : M4 + st.m4 + pos * mr4) + (4 * 8 << (h ? bh.wj : bg.wj));
#pragma unroll
      for (int i = 0; i < NB; ++i) m2[i] = ldg2_at(base + i * (h ? mr3 << wp : mr4 << wp), h ? mp3 : mp4);
    }
    for (int q = 0; q < nq; ++q) {
      double d[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) d[i] = 0.0;
      auto step = [&](int s, auto operand) {
        double t[NB];
        const double *tq = Ts + (h ? to3[s] : to4[s]) + 4 * q;
#pragma unroll
        for (int i = 0; i < NB; ++i) t[i] = tq[(i << wp) * S];
#pragma unroll
        for (int i = 0; i < NB; ++i) d[i] = mfma4(t[i], operand(i), d[i]);
      };
      if (ks > 1) {
        step(0, [&](int i) { return m.p[i].x; });
        step(1, [&](int i) { return m.p[i].y; });
      }
      if (ks & 1) {
        if (ks == 1) step(0, [&](int i) { return m.s[i]; });
        else step(2, [&](int i) { return m.s[i]; });
      }
      if (ks == 4) {
        step(2, [&](int i) { return m2[i].x; });
        step(3, [&](int i) { return m2[i].y; });
      }
      const int it = 4 * q + g, rho = it * d4 + jm4 - rho0;
      if (h ? it < d2 && jm3 < d3 : it < d5 && jm4 < d4 && (unsigned)rho < (unsigned)GW) {
        double *dq = dst + (h ? 8 * q : 8 * q * d4);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          const int p = pos + (i << wp);  // uniform; a multiple of 2^wp
          if (p < np) dq[((p >> 3) * 4 + (p & 3)) * 2 * W + ((p >> 2) & 1)] = d[i];
        }
      }
    }
  };
  Mops ma, mb;
  double u3[SM][NQ];
  const uint32_t uo = g * nK3 + c;
  auto load_u3 = [&](const ChainStep &st) {
    const double *base = U3 + st.u3;
#pragma unroll
    for (int s = 0; s < SM; ++s)
      if (4 * s < st.n4) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) u3[s][q] = ldg_at(base + 4 * s * nK3 + 16 * q, uo);
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
    load_m(st, w, ma);
    load_u3(st);
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
      // ---- G and H, a chunk's booster entries read during the products of the one before
      bool h;
      int pos;
      if (chunk_of(st, w, h, pos)) {
        for (int ch = w;; ch += 2 * nw) {
          load_m(st, ch + nw, mb);
          multiply(st, ch, ma);
          if (!chunk_of(st, ch + nw, h, pos)) break;
          load_m(st, ch + 2 * nw, ma);
          multiply(st, ch + nw, mb);
          if (!chunk_of(st, ch + 2 * nw, h, pos)) break;
        }
      }
      ChainStep sn = st;
      bool more = st.more != 0;
      if (more) {
        sn = step_at(++sp);
        more = core0 + sn.o34 * nd < core_hi;
        if (more) load_m(sn, w, ma);
      }
      __syncthreads();
      const int s4 = (st.n4 + 3) >> 2, s3 = (st.n3 + 3) >> 2;
      const d2v *gp = reinterpret_cast<const d2v *>(Gs) + g * GW + w * RT * 16 + c;
      const d2v *hp = reinterpret_cast<const d2v *>(Hs) + g * C + c;
#pragma unroll
      for (int r0 = 0; r0 < RT; r0 += 2) {
        // ---- P of two row tiles, transposed: rows k3, columns (i5, i4)
        constexpr int NR = 2;
        d4v pt[NR][NQ];
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
          for (int q = 0; q < NQ; ++q) pt[r][q] = d4v{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < SM / 2; ++s) {
          if (2 * s < s4) {
            d2v gv[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r)
              if (r0 + r < RT) gv[r] = gp[s * 4 * GW + (r0 + r) * 16];
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
              for (int r = 0; r < NR; ++r)
                if (r0 + r < RT) pt[r][q] = mfma(u3[2 * s][q], gv[r].x, pt[r][q]);
            if (2 * s + 1 < s4) {
#pragma unroll
              for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int r = 0; r < NR; ++r)
                  if (r0 + r < RT) pt[r][q] = mfma(u3[2 * s + 1][q], gv[r].y, pt[r][q]);
            }
          }
        }
        if (r0 + 2 >= RT && more) load_u3(sn);
        // ---- A(i1) += P H
#pragma unroll
        for (int s = 0; s < SM / 2; ++s) {
          if (2 * s < s3) {
            const bool both = 2 * s + 1 < s3;
#pragma unroll
            for (int t0 = 0; t0 < CT; t0 += 4) {
              d2v hv[4];
#pragma unroll
              for (int t = t0; t < t0 + 4 && t < CT; ++t) hv[t - t0] = hp[s * 4 * C + t * 16];
#pragma unroll
              for (int t = t0; t < t0 + 4 && t < CT; ++t)
#pragma unroll
                for (int r = 0; r < NR; ++r)
                  if (r0 + r < RT) acc[r0 + r][t] = mfma(pt[r][s >> 1][(2 * s) & 3], hv[t - t0].x, acc[r0 + r][t]);
              if (both) {
#pragma unroll
                for (int t = t0; t < t0 + 4 && t < CT; ++t)
#pragma unroll
                  for (int r = 0; r < NR; ++r)
                    if (r0 + r < RT) acc[r0 + r][t] = mfma(pt[r][s >> 1][(2 * s + 1) & 3], hv[t - t0].y, acc[r0 + r][t]);
              }
            }
          }
        }
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
    const int sig = t * 16 + c, i3 = by_d2(sig), i2 = sig - i3 * d2;
#pragma unroll
    for (int r0 = 0; r0 < RT; ++r0)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int rl = (w * RT + r0) * 16 + g + 4 * r, rho = rho0 + rl, i5 = by_d4(rho), i4 = rho - i5 * d4;
        if (rl < GW && sig < C) stg(out + ((i2 * d3 + i3) * d4 + i4) * d5 + i5, acc[r0][t][r]);
      }
  }
}

// Wavefronts per SIMD the registers are budgeted for, and the most wavefronts of a workgroup.
template <int RT, int CT, int NQ>
constexpr int chain_waves() {
  constexpr int need = 8 * RT * CT + 8 * RT * NQ + (NQ == 2 ? 144 : 128);  // accumulators, P, operands in flight
  return need <= 128 ? 4 : need <= 176 ? 3 : 2;
}
constexpr int kChainWg = 12;  // wavefronts of a workgroup

// Block b runs item b of the list (configuration, chunk, i1, row block), or, without a list,
// configuration 0's chunk b / (d1 nrb), i1 and row block from b % (d1 nrb).
template <int RT, int CT, int NQ>
__global__ __launch_bounds__((chain_waves<RT, CT, NQ>() >= 3 ? kChainWg : 8) * 64, (chain_waves<RT, CT, NQ>()))
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
  chain_item<RT, CT, NQ>(cfgs[q0], q1, q2, q3, smem);
}

// Kernel variants: row tiles per wavefront, column tiles, window class.
constexpr int chain_key(int rt, int ct, int nq) { return (rt - 1) * 64 + ct * 2 + nq - 1; }
constexpr int kChainKeys = 2 * 64;

template <typename F>
hipError_t chain_dispatch(int key, F &&f) {
#define EPRL_RC(r, c)                                        \
  case chain_key(r, c, 1): return f(chain_kernel<r, c, 1>); \
  case chain_key(r, c, 2): return f(chain_kernel<r, c, 2>);
#define EPRL_C(c) EPRL_RC(1, c) EPRL_RC(2, c)
  switch (key) {
    EPRL_C(1) EPRL_C(2) EPRL_C(3) EPRL_C(4) EPRL_C(5) EPRL_C(6) EPRL_C(7) EPRL_C(8) EPRL_C(9) EPRL_C(10)
    EPRL_RC(1, 11) EPRL_RC(1, 12) EPRL_RC(1, 13) EPRL_RC(1, 14) EPRL_RC(1, 16)
    default: return hipErrorInvalidValue;
  }
#undef EPRL_RC
#undef EPRL_C
}

}  // namespace

// Row tiles per wavefront (rt) and row blocks (nrb) of A(i1) for RT x ct tiles.
static void chain_split(int RT, int ct, int nq, ChainGeom &g) {
  g.rt = RT >= 2 && ct <= 10 ? 2 : 1;
  g.nrb = 1;
  const int maxw = 8;
  while ((((RT + g.nrb - 1) / g.nrb) + g.rt - 1) / g.rt > maxw) ++g.nrb;
}

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
  g.ct = (C + 15) / 16;
  g.smax = (w + 3) / 4;
  g.wm = w;
  // Rows that row offsets reach before the first T5 row and past the last T2 row (positions run up to
  // three past a window's end).
  g.tpre = g.tpost = 0;
  const int wlo[2] = {p.K[1].lo2, p.K[2].lo2}, whi[2] = {hi2(p.K[1]), hi2(p.K[2])};
  for (int o = 0; o < nd; ++o) {
    g.tpre = std::max(g.tpre, (chain_klo(J, wlo, whi, false, o) - wlo[1]) / 2 - o * g.n4t);
    g.tpost = std::max(g.tpost, (whi[0] + 6 - chain_klo(J, wlo, whi, true, o)) / 2 + 1 - (nd - o) * g.n3t + 1);
    // T5's offsets past its rows and T2's before them stay inside the T rows.
    g.tpost = std::max(g.tpost, (whi[1] + 6 - chain_klo(J, wlo, whi, false, o)) / 2 + 1 - (nd - o) * g.n4t - nd * g.n3t + 1);
    g.tpre = std::max(g.tpre, (chain_klo(J, wlo, whi, true, o) - wlo[0]) / 2 - o * g.n3t - nd * g.n4t);
  }
  const int nq = g.smax > 4 ? 2 : 1;
  if (g.ct == 15) g.ct = 16;
  g.ts = (std::max(d5, d2) + 1) & ~1;
  g.mr4 = chain_mrow(nd, d4);
  g.mr3 = chain_mrow(nd, d3);
  chain_split(RT, g.ct, nq, g);
  for (;; ++g.nrb) {
    if (g.nrb > RT) return false;
    g.rtb = (RT + g.nrb - 1) / g.nrb;
    if (chain_smem_bytes(p) <= kChainMaxLds) break;
  }
  g.waves = (g.rtb + g.rt - 1) / g.rt;
  g.key = chain_key(g.rt, g.ct, nq);
  g.lds = (int)(chain_smem_bytes(p) / sizeof(double));
  const int64_t nx = p.X.n, d1 = p.i[0].n;
  auto pad = [](int64_t v) { return (v + 31) / 32 * 32; };
  g.t5 = pad((int64_t)nd * nx * nd * d1 * nd * g.n4t * g.ts);
  g.t2 = pad((int64_t)nd * nd * nx * d1 * nd * g.n3t * g.ts);
  // Booster rows per (l24, l34) or (l34, l35); reads run up to 16 positions past the last.
  const int64_t rows = w + 3;
  g.m4 = pad(nd * nd * rows * g.mr4 + 16 * g.mr4);
  g.m3 = pad(nd * nd * rows * g.mr3 + 16 * g.mr3);
  g.steps = pad((int64_t)nd * nx * nd * nd * (int64_t)(sizeof(ChainStep) / sizeof(double)));
  // The steps hold 32-bit offsets into U3, M4 and M3.
  if (p.tsize[2] > INT32_MAX || g.m4 > INT32_MAX || g.m3 > INT32_MAX) return false;
  p.chain = true;
  return true;
}

size_t chain_smem_bytes(const Plan &p) {
  const ChainGeom &g = p.ch;
  const int R = p.i[4].n * p.i[3].n, C = p.i[2].n * p.i[1].n, SP = (g.smax + 1) / 2;
  const int GW = std::min(R, g.rtb * 16);
  // The last row of G or H is read past its end by up to 31 columns (results never used).
  return sizeof(double) * ((size_t)(p.nd * (g.n4t + g.n3t) + g.tpre + g.tpost) * g.ts + (size_t)SP * 8 * (GW + C) + 64);
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
  rp.smax = g.smax;
  rp.wm = g.wm;
  rp.tpre = g.tpre;
  rp.tpost = g.tpost;
  rp.lds = g.lds;
  rp.mr4 = g.mr4;
  rp.mr3 = g.mr3;
  rp.rtb = g.rtb;
  rp.nrb = g.nrb;
  rp.nx = p.X.n;
  for (int q = 0; q < 2; ++q) {
    rp.wlo[q] = p.K[1 + q].lo2;
    rp.whi[q] = p.K[1 + q].lo2 + 2 * (p.K[1 + q].n - 1);
  }
  rp.core_lo = 0;
  rp.core_hi = p.nd * p.nd * p.nd * p.nd;
}

hipError_t launch_chain_prep(const RingParams &rp, hipStream_t s) {
  const int nd = rp.nd, nb5 = nd * rp.nx * nd, nb2 = nd * nd * rp.nx;
  const int64_t m = (int64_t)nd * nd * (rp.wm + 3) * (rp.mr4 + rp.mr3);
  const int nbs = (nd * rp.nx * nd + kPrepThreads - 1) / kPrepThreads;
  const int64_t blocks = nb5 + nb2 + nbs + (m + kPrepThreads - 1) / kPrepThreads;
  chain_prep_kernel<<<(unsigned)blocks, kPrepThreads, 0, s>>>(rp, nb5, nb2, nbs);
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
