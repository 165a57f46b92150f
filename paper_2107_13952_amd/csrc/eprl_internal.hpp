// Internal declarations shared by the host planner, the kernels and the C ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/eprl.h"

// Not part of the interface, for tests: most bytes the derived tables of a batch's pass take on this
// context.
extern "C" int eprl_internal_batch_pass(eprl_ctx *ctx, size_t derived_bytes);

namespace eprl {

// A range of spins in two-units: values lo2, lo2 + 2, ..., lo2 + 2 (n - 1).
struct Range {
  int lo2 = 0;
  int n = 0;
};

// Link indices in the order (12, 13, 14, 15, 23, 24, 25, 34, 35, 45).
enum Link { L12 = 0, L13, L14, L15, L23, L24, L25, L34, L35, L45 };

// Shape of the x-outer factorised kernel (chain.hip) for one configuration.
struct ChainGeom {
  int n4t = 0, n3t = 0;   // k4 (k3) values per l45 (l23) of its derived tables
  int ts = 0;             // entries of a row of those tables (i5 or i2, padded)
  int wm = 0, sp = 0;     // widest k4 or k3 window; eights of positions of G and H
  int tpre = 0, tmid = 0, tpost = 0;  // zero rows before, between and after the T rows in LDS
  int nrb = 1, ctb = 1;   // column blocks, column tiles per block
  int waves = 1;          // wavefronts per workgroup
  int resident = 256;     // workgroups the chip (256 CUs) holds at a time
  int lds = 0;            // LDS of a workgroup, in doubles
  int mr4 = 0, mr3 = 0;   // entries of a row of M4, M3
  int key = 0;            // kernel variant
  int64_t t5 = 0, t2 = 0, m4 = 0, m3 = 0, steps = 0;  // derived tables, in doubles
};

// Everything the kernels need to know about one configuration (two_j, dl); built on the host.
struct Plan {
  int two_j[10];
  int dl = 0;
  int nd = 1;                 // dl + 1
  Range i[5];                 // boundary intertwiners i1..i5
  Range K[4];                 // union over shells of the k2..k5 ranges (global windows)
  Range X;                    // global window of the x summation spin
  int kmax = 0;               // largest k range of any shell
  int D = 0;                  // padded tile dimension of the assembly kernel (8 or 16)
  int64_t nshell = 0;         // (dl + 1)^6
  std::vector<int64_t> boff;  // packed booster offsets, 4 nd^3 + 1
  std::vector<int> kr;        // [4][nd^3][2]: lowest two_k and size of k_e per edge triple
  int fact_max = 0;           // largest factorial argument met by any 6j of the tables
  // 6j tables: sizes in doubles and offsets into one allocation.
  int64_t tsize[5] = {0, 0, 0, 0, 0};
  int64_t toff[6] = {0, 0, 0, 0, 0, 0};
  int64_t a_size = 0;         // entries of the vertex tensor
  // Factorised (ring) path: widest union over l45 of the k4 ranges of a core
  // (l24, l34 fixed) and over l23 of the k3 ranges (l34, l35 fixed); the ring kernel needs
  // them to fit its KW-wide LDS tiles, and all i and k ranges to fit 8.
  int ring_w4 = 0, ring_w3 = 0;
  int ring_KW = 0;            // 16 or 32 when the ring path applies, else 0
  int ring_DI = 0, ring_DK = 0;  // padded boundary / virtual intertwiner tile sizes (8 or 16)
  int ring_cls = -1;          // tile class of the ring kernel, -1 when it does not apply
  int ring_cls8 = -1;         // class among 0..7 (half chains on vector ALUs), -1 when none
  bool chain = false;         // evaluated by the x-outer kernel
  ChainGeom ch;
};

// Largest 6j argument (two-units) the device evaluation is built for: up to it the alternating
// Racah sum cancels by at most ~1e15, which double-double arithmetic absorbs with a few ulp to
// spare; beyond it the cancellation grows past what 106 bits hold.
constexpr int kSixjMaxTwo = 200;

// Build a plan; returns EPRL_OK or an error code with a message in `err`.
int make_plan(const int two_j[10], int dl, Plan &p, std::string &err);
// Live-shell and term counts (host enumeration).
void count_terms(const Plan &p, int64_t &live, double &terms);
// Exact work counts: terms, per-shell-order flops, factorised-order useful and executed flops.
void count_work(const Plan &p, double out[5]);
// Useful flops of the x-outer kernel and of its derived tables.
void count_chain_work(const Plan &p, double out[2]);

// ---- kernel-side parameter blocks (passed by value) ----

// sqrt(n!) and its inverse, n <= fact_max: (f.x + f.y) 2^e and (f.z + f.w) 2^-e.
struct FactTables {
  const double4 *f = nullptr;
  const int *e = nullptr;
};

struct TableParams {
  int two_j[10];
  int nd;
  int i1_lo2, i1_n;
  int K_lo2[4], K_n[4];
  int X_lo2, NX;
  int64_t toff[6];
  double *tables;
  FactTables fact;
};

struct VertexParams {
  int two_j[10];
  int nd;
  int i_lo2[5], i_n[5];
  int K_lo2[4], K_n[4];
  int X_lo2, NX;
  const double *T1, *T2, *T3, *T4, *T5;
  const double *B;
  const int64_t *boff;
  const int *kr;
  double *partial;        // [nchunk][i1][i2][i3][i4][i5]
  int64_t shell_begin, shell_end, chunk;
  int nchunk;
};

// One step of the x-outer kernel, (l24, x, l35; l34): sizes of the k4 and k3 windows, offsets of
// the windows' starts in U3, M4, M3 and in the T rows (of k = 0's row), whether the unit has more.
struct alignas(32) ChainStep {
  int n4, n3, u3, m4, m3, t5, t2;
  short o34, more;
};

struct RingParams {
  int two_j[10];
  int nd;
  int i_lo2[5], i_n[5];
  // Index ranges of the ring tables U1..U5 (virtual spins, x) and the spin count tnd that strides
  // them: the configuration's own, or those of a configuration of the same spins at a larger dl
  // whose tables it shares (every index range of its own lies inside them).
  int K_lo2[4], K_n[4];
  int X_lo2, NX;
  int tnd;
  int xlo2, xhi2;         // the configuration's own x range (the loops' bounds)
  const double *U1, *U2, *U3, *U4, *U5;
  const double *B;
  const int64_t *boff;
  const int *kr;
  double *partial;        // [nchunk][i1][i2][i3][i4][i5]
  const int *bounds;      // [i1][nchunk + 1]: first core of each chunk of that i1
  int nchunk;
  int nrb;                // row (x-outer kernel: column) blocks of A(i1)
  // x-outer kernel: derived tables and their shape (ChainGeom), own x count, own windows of k3
  // (0) and k4 (1), range of cores; bounds then holds units (l24, l25, x, l35).
  double *T5, *T2, *M4, *M3;
  ChainStep *steps;
  int n4t, n3t, ts, wm, sp, tpre, tpost, ctb, nx, lds, mr4, mr3;
  int wlo[2], whi[2];
  int core_lo, core_hi;
  // Rows of a slice of T5.  (Last: with the fields before it at other offsets the scalar loads group
  // differently, which cost chain_kernel<2, 11, 2> eight spilled registers, 17.9 -> 18.5 ms at two_j = 12.)
  int t5r;
};

// One launch over several configurations: job q has the blocks from jobs[q].first to the next job's
// first, and works on entry jobs[q].index of the launch's parameter array.
struct BatchJob {
  int first, index;
};

// Division of 32-bit indices by a divisor that is the same for the whole launch: floor(n m / 2^32) with
// m = floor((2^32 - 1) / d) is the quotient or one less.
struct IndexDiv {
  uint32_t m = 0, d = 1;
  __host__ __device__ IndexDiv() {}
  __host__ __device__ explicit IndexDiv(int d_) : m(0xffffffffu / (uint32_t)d_), d((uint32_t)d_) {}
#ifdef __HIPCC__
  // r becomes r / d; returns the remainder.
  __device__ __forceinline__ int take(uint32_t &r) const {
    uint32_t q = __umulhi(r, m), rest = r - q * d;
    if (rest >= d) {
      ++q;
      rest -= d;
    }
    r = q;
    return (int)rest;
  }
  // (indices past 32 bits)
  __device__ __forceinline__ int take(int64_t &r) const {
    const int rest = (int)(r % d);
    r /= d;
    return rest;
  }
#endif
};

#ifdef __HIPCC__
// Division by a size that is the same for the whole kernel, as a multiply-high by the rounded-up
// reciprocal: exact for dividends and divisors below 2^16, and one instruction where the generic integer
// division takes dozens.
struct FastDiv {
  uint32_t m;
  int d;
  __device__ explicit FastDiv(int d_)
      : m(d_ > 1 ? (uint32_t)((0x100000000ull + (uint64_t)d_ - 1) / (uint64_t)d_) : 0u), d(d_) {}
  __device__ int operator()(int q) const { return d > 1 ? (int)__umulhi((uint32_t)q, m) : q; }
};

// The job of block b (the last whose first block is not past it); b becomes the block within the job.
__device__ __forceinline__ int batch_job(const BatchJob *jobs, int njobs, int &b) {
  int lo = 0, hi = njobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs[mid].first <= b) lo = mid;
    else hi = mid - 1;
  }
  b -= jobs[lo].first;
  return __builtin_amdgcn_readfirstlane(jobs[lo].index);
}
#endif

struct ReduceParams {
  const double *partial;
  int nchunk;
  int64_t a_size;
  int i_lo2[5], i_n[5];
  double *A;
  int accumulate;
};

// Kernel launchers (defined in the .hip files).  They return hipSuccess or the launch error.
hipError_t launch_fact_table(double4 *f, int *e, int fact_max, hipStream_t s);
hipError_t launch_sixj_tables(const TableParams &tp, int64_t total, hipStream_t s);
hipError_t launch_ring_tables(const TableParams &tp, hipStream_t s);
int64_t ring_table_blocks(int64_t nd, int64_t nx);
hipError_t launch_ring_tables_batch(const TableParams *tps_dev, const BatchJob *jobs_dev, int njobs, int64_t blocks,
                                    hipStream_t s);
hipError_t launch_sixj_batch(const int *args, int n, double *out, FactTables fact, int fact_max, hipStream_t s);
hipError_t launch_assemble(const VertexParams &vp, int D, hipStream_t s);
hipError_t launch_reduce(const ReduceParams &rp, hipStream_t s);
int64_t reduce_blocks(int64_t a_size);
hipError_t launch_reduce_batch(const ReduceParams *rps_dev, const BatchJob *jobs_dev, int njobs, int64_t blocks,
                               hipStream_t s);
int ring_class(int DI, int DK, int KW);
// Tile classes: 0..7 by the padded tiles of ring.hip's kernels, kWideClass a boundary dimension
// above 8 in the x-outer kernel of chain.hip (which also runs classes 0..3).
constexpr int kWideClass = 8;
constexpr int kRingClasses = 9;
// x-outer factorised kernel (chain.hip).  chain_plan sets p.chain and p.ch (false when the
// configuration's windows or tiles do not fit); derived tables of p.ch.t5 + t2 + m4 + m3 doubles.
constexpr size_t kChainMaxLds = 160 * 1024 - 256;
bool chain_plan(Plan &p);
size_t chain_smem_bytes(const Plan &p);
hipError_t chain_init_attributes();
void chain_params(const Plan &p, double *derived, RingParams &rp);
hipError_t launch_chain_prep(const RingParams &rp, hipStream_t s);
int64_t chain_prep_blocks(const RingParams &rp);
hipError_t launch_chain_prep_batch(const RingParams *cfgs_dev, const BatchJob *jobs_dev, int njobs, int64_t blocks,
                                   hipStream_t s);
// items: (configuration, chunk, i1, column block) in device memory, or null for every item of
// configuration 0; waves: wavefronts per workgroup.
hipError_t launch_chain(const RingParams *cfgs_dev, const int *items_dev, int nitems, int key, int waves,
                        size_t smem, hipStream_t s);
// Chunks of units (l24, l25, x, l35) of equal estimated cost for each i1, as ring_schedule does
// with cores.
int chain_schedule(const Plan &p, int target_wg, std::vector<int> &bounds,
                   std::vector<double> *chunk_cost = nullptr, int core_lo = 0, int core_hi = -1);
// Splits the cores of the factorised path, for each i1, into chunks of equal estimated cost
// (x iterations plus the per-core set-up), about target_wg workgroups in all and at most
// kRingMaxPartialBytes of partial sums; fills bounds ([i1][nchunk + 1]) and, if asked for, the
// estimated cost of each chunk ([i1][nchunk], in x iterations) and returns nchunk.  Only the
// cores [core_lo, core_hi) are split (core_hi < 0: all); core index
// ((o24 * nd + o25) * nd + o34) * nd + o35 over the offsets of l24, l25, l34, l35.
constexpr size_t kRingMaxPartialBytes = size_t(256) << 20;
int ring_schedule(const Plan &p, int target_wg, std::vector<int> &bounds,
                  std::vector<double> *chunk_cost = nullptr, int core_lo = 0, int core_hi = -1);
int ring_row_blocks(const Plan &p);
// LDS bytes of the tile class at nd with staging level stg (-1: the most that fits).
size_t ring_smem_bytes(int cls, int nd, int stg = -1);
// Booster staging levels of the tile class that fit in LDS at nd, most first; returns their count.
int ring_stage_levels(int cls, int nd, int levels[3]);
// Largest dl + 1 the ring kernels stage booster blocks for.
constexpr int kRingMaxNd = 16;
hipError_t ring_init_attributes();
hipError_t launch_ring(const RingParams &rp, int cls, int stg, hipStream_t s);
hipError_t launch_ring_batch(const RingParams *cfgs_dev, const int *items_dev, int nitems, int cls,
                             int max_nd, int stg, int grid, int *next, hipStream_t s);
hipError_t launch_reset_counters(int *c, int n, hipStream_t s);
hipError_t launch_shell_fifteenj(const VertexParams &vp, int64_t shell, double *W,
                                 hipStream_t s);
// BF vertex of a plan made with dl = 0 (tables of the per-shell layout); total = entries of A.
hipError_t launch_bf_vertex(const VertexParams &vp, double *A, int64_t total, hipStream_t s);

struct ContractParams {
  int n[5];
  const double *A;
  const double *psi[5];
  double *partial;  // complex partial sums
  int nblocks;
  IndexDiv by[5];   // by n (set by the launchers)
};
struct GradPsiOut {
  double *p[5];
};
hipError_t launch_contract(const ContractParams &cp, double *F, hipStream_t s);
// Complex partial-sum slots of the fixed device scratch of the contraction (one per block of
// contract_partial_kernel) and its device address on the current device.
constexpr int kContractScratchSlots = 256;
hipError_t contract_scratch_address(double **ptr);
hipError_t launch_grad_psi(const ContractParams &cp, double gre, double gim, double *const out[5],
                           hipStream_t s);

// Booster builder (boosters.hip; 4jm coefficient tables in sixj.hip).
// One booster block: edge e (0..3 for edges 2..5), boundary and virtual spins of its four links
// (two-units, pairing (first second)(third fourth)), intertwiner ranges, packed offset.
struct BoosterBlock {
  int edge;
  int jb[4], lb[4];
  int two_ilo, idim, two_klo, kdim;
  int64_t off;
};
void booster_blocks(const Plan &p, std::vector<BoosterBlock> &out);
// A table of 4jm coefficients: out[o + m n + i] = 4jm(j; m-tuple m; two_lo + 2 i) for the M
// m-tuples at mtuples[mt + 4 m ..].
struct FourjmSet {
  int j[4];
  int two_lo, n;
  int M, mt;
  int64_t out;
};
hipError_t launch_fourjm_tables(const FourjmSet *sets_dev, int nsets, int max_entries,
                                const int *mtuples_dev, double *out, FactTables fact, hipStream_t s);
hipError_t launch_threejm_batch(const int *args, int n, double *out, FactTables fact, hipStream_t s);
// A boost matrix element d^{(rho, k = j)}_{j l m}(r): spins, the Y-map rho = gamma (j + 1), the
// phase factor of the basis convention, and the Jacobi-form constants of the two SU(2) d
// functions it integrates, d^j_{j m} and d^l_{j m}.
struct DKey {
  double rho, ph_re, ph_im, pre;      // pre = sqrt((2j+1)(2l+1))
  double nj, nl;                      // xi * sqrt(s! (s+mu+nu)! / ((s+mu)! (s+nu)!)) of each d
  int muj, nuj, sj, mul, nul, sl;     // Jacobi parameters of each d
};
// The blocks of one edge as a matrix: rows, the distinct pairs of key bases of the first two links;
// columns, those of the other two.
struct BoosterGrid {
  int M, nrow, ncol;       // m-tuples, rows, columns
  int rows, cols, map;     // offsets in pairs (two key bases each) and bmap
};

struct BoosterParams {
  const DKey *keys;
  int nkeys;
  const double *sx, *sw;   // Gauss-Legendre nodes and weights of the s integral on [-1, 1]
  int ns;
  const double *r, *rw;    // r nodes (30-point rule, then 61-point rule) and their weights,
  int nr, nr30;            //   rw including sinh^2 r / (4 pi) and the Jacobian of u = e^{-r}
  double *dtab;            // complex [key][r]
  // blocks
  const int *binfo;        // per block: edge, idim, kdim, M, moff, kb[4]  (9 ints)
  const int64_t *boffs;    // per block: packed offset, ck offset
  const int *mtuples;      // per edge: its m-tuples (4 ints each), edge e at mt_edge[e]
  int mt_edge[4];
  int jb_edge[4][4];       // boundary spins of each edge's four links
  const double *ci;        // per edge: M x idim 4jm of the boundary spins, edge e at ci_edge[e]
  int64_t ci_edge[4];
  const double *ck;        // per block: M x kdim 4jm of the virtual spins
  double *I;               // per block and m-tuple: the two rules' integrals, complex (4 doubles)
  double *B;               // packed boosters (real parts of the 61-point values)
  double *stat;            // per block: max |G61 - G30|, max |G61|, max |Im G61|
  int nblocks, Mmax;
  // grouped for the kernels: keys of one (j, l) together, group g from groups[g]; the blocks' matrices,
  // bmap[row][column] the block's offset in I (-1: no block), and their 16 x 16 tiles (edge, row,
  // column, 0); or, where the tiles would be sparse, the blocks by themselves
  const int *groups;
  int ngroups;
  BoosterGrid grid[4];
  const int *pairs, *bmap, *tiles, *singles;
  int ntiles, nsingles;
};
hipError_t launch_booster_dfun(const BoosterParams &bp, hipStream_t s);
hipError_t launch_booster_integrals(const BoosterParams &bp, hipStream_t s);
hipError_t launch_booster_assemble(const BoosterParams &bp, double *stat3, hipStream_t s);

// Multi-vertex contractions (network.hip).
struct TrailParams {
  const double *A;        // [lead][S] row-major
  int m;                  // trailing intertwiners contracted
  int n[5];               // their dimensions
  const double *psi[5];   // their vectors (complex)
  int64_t S;              // prod n[0..m-1]
  int nsplit;             // blocks per leading row
  double *T;              // complex [lead]
  double *partial;        // complex [lead][nsplit] when nsplit > 1
  IndexDiv by[5];         // by n (set by the launcher)
};
hipError_t launch_contract_vertices(const double *A, const double *B, int64_t total, int nblocks,
                                    double *partial, double *F, hipStream_t s);
int trailing_splits(int64_t nlead, int64_t S);
hipError_t launch_contract_trailing(const TrailParams &tp, int64_t nlead, hipStream_t s);
hipError_t launch_delta3(int n, int two_klo, int two_x, const double *TA, const double *TB,
                         const double *TC, double *F, hipStream_t s);

struct AdjointParams {
  VertexParams v;
  const double *psi[5];
  double *shell_g;        // [nshell][4][kmaxpad] complex
  int kpad;
};
hipError_t launch_adjoint_shells(const AdjointParams &ap, hipStream_t s);
// Adjoint in the factorised order (one workgroup per core, then a fixed-order sum per booster
// entry of `total`); the per-core G vectors go to gbuf (adjoint_ring_gbuf_bytes).  Applies where
// the factorised vertex kernels do, with dl + 1 <= kAdjRingMaxNd.
constexpr int kAdjRingMaxNd = 11;
constexpr size_t kAdjRingMaxLds = 160 * 1024 - 256;
// LDS sizes of the kernel for a configuration: kl = largest k range of a spin, iw = number of i1
// values, kw = widest core window of k5, k4 (over l45), k3 or k2 (over l23), ng = spins per group
// of the two halves.  kl = 0 when the windows are too wide for the kernel.
void adjoint_ring_dims(const Plan &p, int &kl, int &iw, int &kw, int &ng);
size_t adjoint_ring_smem(int nd, int kl, int iw, int kw, int ng);
size_t adjoint_ring_gbuf_bytes(int nd, int kl);
// Launch order of the adjoint's cores, longest first by an estimate of their work (the x values
// with both core windows non-empty, times the windows' widths), so that the last workgroups to
// start are short ones; every core writes its own G vectors, so the order changes no result.
void adjoint_ring_order(const Plan &p, std::vector<int> &order);
hipError_t adjoint_ring_init_attributes();
hipError_t launch_adjoint_ring(const RingParams &rp, int kl, int iw, int kw, int ng,
                               const int *order, const double *const psi[5], double *gbuf,
                               int64_t total, double gre, double gim, double *grad_b, hipStream_t s);
hipError_t launch_adjoint_reduce(const AdjointParams &ap, int64_t total, double gre, double gim,
                                 double *grad_b, hipStream_t s);

}  // namespace eprl
