// Booster functions of eq. (booster) by quadrature on the device (Sec. 3.1 "Booster
// coefficients"):
//
//   B4(j, l; i, k) = sum_{m1..m4} 4jm(j; m; i) 4jm(l; m; k)
//                    * int_0^inf dr sinh^2(r) / (4 pi) prod_a d^{(rho_a, j_a)}_{j_a l_a m_a}(r),
//   rho_a = gamma (j_a + 1)  (the Y-map of eq. (booster)).
//
// The boost matrix elements d are computed from the principal-series realisation of SL(2,C) on
// functions on SU(2): a boost of rapidity r acts on the polar angle of SU(2) and multiplies by a
// power of the modulus of its lower-triangular factor, which gives
//
//   d_{jlm}(r) = sqrt((2j+1)(2l+1)) / (2 sinh r) int_{-r}^{r} ds e^{i rho s}
//                d^j_{j m}(beta(s)) d^l_{j m}(beta'(s)),
//   cos^2(beta/2) = (e^s - e^{-r}) / (2 sinh r),  sin^2(beta/2) = (e^r - e^s) / (2 sinh r),
//   cos^2(beta'/2) = e^{r-s} cos^2(beta/2),        sin^2(beta'/2) = e^{-r-s} sin^2(beta/2),
//
// times a phase exp(-i phi_{jl}) that fixes the basis convention (purely imaginary generator
// elements between l and l + 1, and d_{j l -m} = (-1)^{l-j} conj(d_{j l m}), under which the
// boosters are real).  The s integral is a Gauss-Legendre sum (the integrand is analytic); the
// SU(2) functions are evaluated in their Jacobi-polynomial form
//   d^J_{m' m}(beta) = xi sqrt(s! (s+mu+nu)! / ((s+mu)! (s+nu)!)) sin^mu(beta/2) cos^nu(beta/2)
//                      P_s^{(mu, nu)}(cos beta),   mu = |m - m'|, nu = |m + m'|,
// with the stable three-term recurrence of P in its degree, cos beta = cos^2 - sin^2 and the
// half-angle functions as square roots of the expressions above (no angle is formed).
//
// The r integral follows the quadrature of Sec. 3.1: u = e^{-r} maps it to (0, 1], cut into n
// subintervals growing linearly from u = 0; each gets a 30- and a 61-point Gauss-Legendre rule
// (the host builds the nodes); the 61-point sum is the value and |61 - 30| the error estimate.
//
// Kernels: (1) d on every (j, l, m) and r node (one wavefront per (j, l) and r, lanes over the s
// nodes, everything that does not depend on m made once); (2) the r integrals of the products of
// four d as matrix products over the r nodes, on the matrix cores (edges of few blocks: block by block); (3) per block the contraction
// with the 4jm coefficient tables (sixj.hip) and the error and magnitude statistics.  All sums run
// in a fixed order.
#include "eprl_internal.hpp"

namespace eprl {

namespace {

__device__ __forceinline__ double ipow(double x, int n) {
  double r = 1.0;
  for (int q = 0; q < n; ++q) r *= x;
  return r;
}

// Jacobi polynomial P_n^{(a, b)}(x) by the recurrence in the degree.
__device__ double jacobi(int n, int a, int b, double x) {
  if (n == 0) return 1.0;
  double p0 = 1.0, p1 = (a + 1) + 0.5 * (a + b + 2) * (x - 1.0);
  for (int k = 2; k <= n; ++k) {
    const double c = 2.0 * k + a + b;
    const double a1 = 2.0 * k * (k + a + b) * (c - 2.0);
    const double a2 = (c - 1.0) * ((double)a * a - (double)b * b);
    const double a3 = (c - 1.0) * c * (c - 2.0);
    const double a4 = 2.0 * (k + a - 1.0) * (k + b - 1.0) * c;
    const double p2 = ((a2 + a3 * x) * p1 - a4 * p0) / a1;
    p0 = p1;
    p1 = p2;
  }
  return p1;
}

// SU(2) d in Jacobi form from sin and cos of the half angle and cos of the angle.
__device__ __forceinline__ double dsu2(double norm, int mu, int nu, int s, double sh, double ch, double cb) {
  return norm * ipow(sh, mu) * ipow(ch, nu) * jacobi(s, mu, nu, cb);
}

__device__ __forceinline__ double wave_sum(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
  return v;
}

// (1) d_{jlm}(r) for the keys of group `grp` (one (j, l), m = -j..j) at r node `ir`: one wavefront,
// lanes over the s nodes.  The exponentials, the half-angle functions and the phase do not depend
// on m: a wavefront per key made them 2 j + 1 times (484 us for two_j = 6, 8 shells, now 216 us).
__global__ __launch_bounds__(256) void booster_dfun_kernel(BoosterParams bp) {
  constexpr int kS = 4;  // s nodes of a lane held at a time
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (wave >= (int64_t)bp.ngroups * bp.nr) return;  // uniform over the wavefront
  const int grp = __builtin_amdgcn_readfirstlane((int)(wave / bp.nr)), ir = (int)(wave % bp.nr);
  const int k0 = bp.groups[grp], k1 = bp.groups[grp + 1];
  const double rho = bp.keys[k0].rho;
  const double r = bp.r[ir];
  const double sh2 = 2.0 * sinh(r), emr = exp(-r);
  for (int q0 = lane; q0 < bp.ns; q0 += 64 * kS) {
    double sh[kS], ch[kS], cb[kS], shp[kS], chp[kS], cbp[kS], wc[kS], wn[kS];
#pragma unroll
    for (int i = 0; i < kS; ++i) {
      const int q = q0 + 64 * i;
      const double x = q < bp.ns ? bp.sx[q] : 0.0, w = q < bp.ns ? bp.sw[q] : 0.0;
      const double s = r * x;
      // e^s - e^-r = e^-r expm1(r (1 + x)) and e^r - e^s = e^s expm1(r (1 - x)): no cancellation
      // at small r.
      const double ep = expm1(r * (1.0 + x)), em = expm1(r * (1.0 - x));
      const double es = exp(s), ems = exp(-s);
      const double c2 = emr * ep / sh2, s2 = es * em / sh2;
      const double c2p = ems * ep / sh2, s2p = emr * em / sh2;
      sh[i] = __builtin_sqrt(s2 > 0.0 ? s2 : 0.0);
      ch[i] = __builtin_sqrt(c2 > 0.0 ? c2 : 0.0);
      shp[i] = __builtin_sqrt(s2p > 0.0 ? s2p : 0.0);
      chp[i] = __builtin_sqrt(c2p > 0.0 ? c2p : 0.0);
      cb[i] = c2 - s2;
      cbp[i] = c2p - s2p;
      double sn, cs;
      sincos(rho * s, &sn, &cs);
      wc[i] = w * cs;
      wn[i] = w * sn;
    }
    for (int key = k0; key < k1; ++key) {
      const DKey &K = bp.keys[key];
      const double nj = K.nj, nl = K.nl;
      const int muj = K.muj, nuj = K.nuj, sj = K.sj, mul = K.mul, nul = K.nul, sl = K.sl;
      double re = 0.0, im = 0.0;
#pragma unroll
      for (int i = 0; i < kS; ++i) {
        const double f = dsu2(nj, muj, nuj, sj, sh[i], ch[i], cb[i]) * dsu2(nl, mul, nul, sl, shp[i], chp[i], cbp[i]);
        re += f * wc[i];
        im += f * wn[i];
      }
      re = wave_sum(re);
      im = wave_sum(im);
      if (lane == 0) {
        const double scale = K.pre * r / sh2;
        const int64_t at = 2 * ((int64_t)key * bp.nr + ir);
        const double vr = scale * (re * K.ph_re - im * K.ph_im), vi = scale * (re * K.ph_im + im * K.ph_re);
        bp.dtab[at] = q0 == 0 ? vr : bp.dtab[at] + vr;
        bp.dtab[at + 1] = q0 == 0 ? vi : bp.dtab[at + 1] + vi;
      }
    }
  }
}

typedef double d4v __attribute__((ext_vector_type(4)));
typedef double d2v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ d2v cmul(d2v a, d2v b) { return d2v{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }

// (2) The two rules' integrals of the products of four d, sum_r w(r) X(r) Y(r) with X = d_1 d_2 of the
// first two links and Y = d_3 d_4 of the others: for one edge and m-tuple a complex matrix product of
// the edge's distinct X (rows) and Y (columns) over the r nodes.  One workgroup per m-tuple and 16 x 16
// tile of (row, column) pairs; its eight wavefronts share the r nodes, three the 30-point rule, five
// the 61-point rule, and their sums are added in order.  Bound by the matrix instructions (four per
// four r nodes) and the reads of d from L2 about evenly; a wavefront per (block, m-tuple) read four
// complex d for every product and took 2490 us for two_j = 6, 8 shells, this 573 us.
constexpr int kIntWaves = 8, kInt30 = 3;
__global__ __launch_bounds__(64 * kIntWaves) void booster_integrals_kernel(BoosterParams bp) {
  __shared__ d2v part[kIntWaves][4][64];
  const int *tl = bp.tiles + 4 * blockIdx.y;
  const int e = tl[0], row0 = tl[1], col0 = tl[2];
  const int mi = blockIdx.x;
  const BoosterGrid &gr = bp.grid[e];
  if (mi >= gr.M) return;
  const int *mt = bp.mtuples + bp.mt_edge[e] + 4 * mi;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  // This lane's row and column (padding: the last one, results unused).
  const int row = row0 + c < gr.nrow ? row0 + c : gr.nrow - 1, col = col0 + c < gr.ncol ? col0 + c : gr.ncol - 1;
  const d2v *d[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const int base = bp.pairs[(a < 2 ? gr.rows + 2 * row : gr.cols + 2 * col) + (a & 1)];
    d[a] = reinterpret_cast<const d2v *>(bp.dtab) + (int64_t)(base + (mt[a] + bp.jb_edge[e][a]) / 2) * bp.nr;
  }
  // Groups of four nodes of this wavefront.
  const bool r61 = w >= kInt30;
  const int q0 = r61 ? bp.nr30 : 0, q1 = r61 ? bp.nr : bp.nr30, ng = (q1 - q0 + 3) / 4;
  const int part_n = r61 ? kIntWaves - kInt30 : kInt30, part_i = r61 ? w - kInt30 : w;
  const int b0 = ng * part_i / part_n, b1 = ng * (part_i + 1) / part_n;
  d4v re = {0.0, 0.0, 0.0, 0.0}, im = re, im2 = re, re2 = re;
#pragma unroll 4
  for (int b = b0; b < b1; ++b) {
    const int q = q0 + 4 * b + g;
    const bool in = q < q1;
    const int qq = in ? q : q1 - 1;
    const d2v x = cmul(d[0][qq], d[1][qq]), y = cmul(d[2][qq], d[3][qq]);
    const double wt = in ? bp.rw[qq] : 0.0;
    const double xr = wt * x.x, xi = wt * x.y;
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(xr, y.x, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(xr, y.y, im, 0, 0, 0);
    re2 = __builtin_amdgcn_mfma_f64_16x16x4f64(xi, y.y, re2, 0, 0, 0);
    im2 = __builtin_amdgcn_mfma_f64_16x16x4f64(xi, y.x, im2, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) part[w][r][lane] = d2v{re[r] - re2[r], im[r] + im2[r]};
  __syncthreads();
  // Thread (w < 4): register w of every lane: entry (row g + 4 w, column c).
  if (w >= 4) return;
  const int rr = row0 + g + 4 * w, cc = col0 + c;
  if (rr >= gr.nrow || cc >= gr.ncol) return;
  const int moff = bp.bmap[gr.map + rr * gr.ncol + cc];
  if (moff < 0) return;
  d2v v[2] = {d2v{0.0, 0.0}, d2v{0.0, 0.0}};
  for (int q = 0; q < kIntWaves; ++q) v[q >= kInt30] += part[q][w][lane];
  double *out = bp.I + 4 * (int64_t)(moff + mi);
  out[0] = v[0].x;
  out[1] = v[0].y;
  out[2] = v[1].x;
  out[3] = v[1].y;
}

// (2) block by block (bp.singles[blockIdx.y]) and m-tuple: one wavefront each, lanes over the r nodes.  For
// calls whose tiles hold few blocks (below 16 of 256): a tile costs the same however many it holds, at spins 7
// 153 us an edge against 10 us a block here (dl = 0, one block to an edge, 610 -> 41 us for all four).
__global__ __launch_bounds__(256) void booster_block_integrals_kernel(BoosterParams bp) {
  const int *bi = bp.binfo + 9 * bp.singles[blockIdx.y];
  const int lane = threadIdx.x & 63;
  const int mi = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const int e = bi[0], M = bi[3], moff = bi[4];
  if (mi >= M) return;
  const int *mt = bp.mtuples + bp.mt_edge[e] + 4 * mi;
  const d2v *d[4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
    d[a] = reinterpret_cast<const d2v *>(bp.dtab) + (int64_t)(bi[5 + a] + (mt[a] + bp.jb_edge[e][a]) / 2) * bp.nr;
  double *out = bp.I + 4 * (int64_t)(moff + mi);
  for (int rule = 0; rule < 2; ++rule) {
    const int q0 = rule ? bp.nr30 : 0, q1 = rule ? bp.nr : bp.nr30;
    double re = 0.0, im = 0.0;
    for (int q = q0 + lane; q < q1; q += 64) {
      const d2v v = cmul(cmul(d[0][q], d[1][q]), cmul(d[2][q], d[3][q]));
      re += bp.rw[q] * v.x;
      im += bp.rw[q] * v.y;
    }
    re = wave_sum(re);
    im = wave_sum(im);
    if (lane == 0) {
      out[2 * rule] = re;
      out[2 * rule + 1] = im;
    }
  }
}

// (3) One workgroup per block: entry (i, k) = sum over the m-tuples of 4jm(j; m; i) 4jm(l; m; k)
// times each rule's integral; the 61-point real part is the booster, |61 - 30| its error.
__global__ __launch_bounds__(256) void booster_assemble_kernel(BoosterParams bp) {
  __shared__ double red[3][256];
  const int b = blockIdx.x;
  const int *bi = bp.binfo + 9 * b;
  const int e = bi[0], idim = bi[1], kdim = bi[2], M = bi[3], moff = bi[4];
  const double *ci = bp.ci + bp.ci_edge[e];
  const double *ck = bp.ck + bp.boffs[2 * b + 1];
  double *out = bp.B + bp.boffs[2 * b];
  double err = 0.0, mag = 0.0, imag = 0.0;
  for (int idx = threadIdx.x; idx < idim * kdim; idx += blockDim.x) {
    const int i = idx / kdim, k = idx % kdim;
    double g30r = 0.0, g30i = 0.0, g61r = 0.0, g61i = 0.0;
    for (int m = 0; m < M; ++m) {
      const double c = ci[(int64_t)m * idim + i] * ck[(int64_t)m * kdim + k];
      const double *I = bp.I + 4 * (int64_t)(moff + m);
      g30r += c * I[0];
      g30i += c * I[1];
      g61r += c * I[2];
      g61i += c * I[3];
    }
    out[idx] = g61r;
    err = fmax(err, hypot(g61r - g30r, g61i - g30i));
    mag = fmax(mag, hypot(g61r, g61i));
    imag = fmax(imag, __builtin_fabs(g61i));
  }
  red[0][threadIdx.x] = err;
  red[1][threadIdx.x] = mag;
  red[2][threadIdx.x] = imag;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int q = 0; q < 3; ++q) red[q][threadIdx.x] = fmax(red[q][threadIdx.x], red[q][threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x < 3) bp.stat[3 * b + threadIdx.x] = red[threadIdx.x][0];
}

// Maxima of the per-block statistics.
__global__ __launch_bounds__(256) void booster_stat_kernel(const double *stat, int nblocks, double *out) {
  __shared__ double red[3][256];
  double v[3] = {0.0, 0.0, 0.0};
  for (int b = threadIdx.x; b < nblocks; b += blockDim.x)
    for (int q = 0; q < 3; ++q) v[q] = fmax(v[q], stat[3 * b + q]);
  for (int q = 0; q < 3; ++q) red[q][threadIdx.x] = v[q];
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int q = 0; q < 3; ++q) red[q][threadIdx.x] = fmax(red[q][threadIdx.x], red[q][threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x < 3) out[threadIdx.x] = red[threadIdx.x][0];
}

}  // namespace

hipError_t launch_booster_dfun(const BoosterParams &bp, hipStream_t s) {
  const int64_t waves = (int64_t)bp.ngroups * bp.nr;
  if (waves == 0) return hipSuccess;
  booster_dfun_kernel<<<(unsigned)((waves + 3) / 4), 256, 0, s>>>(bp);
  return hipGetLastError();
}

hipError_t launch_booster_integrals(const BoosterParams &bp, hipStream_t s) {
  if (bp.Mmax == 0) return hipSuccess;
  if (bp.ntiles > 0) {
    dim3 grid((unsigned)bp.Mmax, (unsigned)bp.ntiles);
    booster_integrals_kernel<<<grid, 64 * kIntWaves, 0, s>>>(bp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (bp.nsingles > 0) {
    dim3 grid((unsigned)((bp.Mmax + 3) / 4), (unsigned)bp.nsingles);
    booster_block_integrals_kernel<<<grid, 256, 0, s>>>(bp);
  }
  return hipGetLastError();
}

hipError_t launch_booster_assemble(const BoosterParams &bp, double *stat3, hipStream_t s) {
  if (bp.nblocks == 0) return hipSuccess;
  booster_assemble_kernel<<<bp.nblocks, 256, 0, s>>>(bp);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  booster_stat_kernel<<<1, 256, 0, s>>>(bp.stat, bp.nblocks, stat3);
  return hipGetLastError();
}

}  // namespace eprl
