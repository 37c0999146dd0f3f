// Device side of the smoothed-aggregation AMG preconditioner for the pressure CG.
//
// One V-cycle, z = M^-1 r, from level 0 (the cell-slot matrix K of the mesh, internal order) down to
// a coarsest level solved with its dense inverse:
//   down, level l:  x_l = S_l(b_l) (smoothing from zero),  res_l = b_l - A_l x_l,
//                   b_{l+1} = R_l res_l                         (b_0 = r)
//   coarsest:       x_L = A_L^-1 b_L
//   up, level l:    t_l = x_l + P_l x_{l+1},  x_l = t_l + S_l(b_l - A_l t_l)   (z = x_0)
// Every smoother is one degree-2 Chebyshev sweep in D_l^-1 A_l over [hi_l / 10, hi_l] (a fixed
// polynomial in D^-1 A times D^-1), the same before and after the coarse correction, and R_l = P_l^T,
// so M^-1 is symmetric; it is positive definite while the spectrum of D^-1 A stays below
// hi + lo = 1.1 hi, where the smoothing polynomial contracts.  hi_0 is a Gershgorin bound of D^-1 K
// (at least 2, which bounds every weakly diagonally dominant K); hi_l = 1.1 times the setup's
// power-iteration estimate of rho(D_l^-1 A_l) on the stored coarse operators, capped by their
// Gershgorin bound.  A sweep takes two passes over the level's operator: from zero, D^-1 b gives d0
// without one; on the way up the first pass uses b_l - A_l t_l = res_l - (A_l P_l) x_{l+1}, with
// A_l P_l stored, so prolongation and that residual are one pass on levels 1 <= l < L-1 (level 0 smooths
// with the operator of the current solve and keeps the prolongation a pass of its own; level L-1 and the
// coarsest together take two or three launches, AmgFused).  Degree-2 Chebyshev on every level takes about half the
// CG iterations of one damped-Jacobi step per level, which more than pays for the extra passes.
// Each stage is one kernel: row kernels on the cell-slot layout for level 0, CSR kernels with SW
// lanes per row (rows summed by a fixed tree of lane exchanges) elsewhere, so every result is deterministic.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "amg_dev.h"
#include "host_rows.h"
#include "krylov_util.h"

namespace difvm {

namespace {

struct DevCsr {
  int n = 0, nnz = 0, sw = 1;  // sw: lanes per row in the CSR kernels
  int32_t *ptr = nullptr, *col = nullptr;
  double *val = nullptr, *diag = nullptr;
  double* val2 = nullptr;  // A P: P's values on its pattern
};
// Transfers laid out for a solve in one block (k_amg_pcg_block).
constexpr int BLOCK_COARSE = 384, BLOCK_NT = 512, BLOCK_R_LANES = 2, BLOCK_R_FOURS = 4;
constexpr int BLOCK_R_ROWS = BLOCK_NT / BLOCK_R_LANES, BLOCK_R_PASSES = (BLOCK_COARSE + BLOCK_R_ROWS - 1) / BLOCK_R_ROWS;
// P: the first four entries of row i as columns pcol[i] and values pval[i], pval[4 TILE + i] (rows past the last:
// zeros).  R: pass r takes the rows r BLOCK_R_ROWS ..., thread t its row t / BLOCK_R_LANES,
// every BLOCK_R_LANES-th four entries from t % BLOCK_R_LANES; fours e of thread t: columns at (first[r] + e) BLOCK_NT + t,
// values there with twice the first index (padded with zeros).  inv: leading dimension ld, padded.
struct AmgBlock {
  int n2 = 0;  // coarsest rows (0: not built)
  int ld = 0;
  ushort4 *pcol = nullptr, *rcol = nullptr;
  double2 *pval = nullptr, *rval = nullptr, *inv = nullptr;
  int nlong = 0;  // rows of P with more than four entries: row, then CSR of the others
  int32_t *lrow = nullptr, *lptr = nullptr, *lcol = nullptr;
  double* lval = nullptr;
  int first[BLOCK_R_PASSES + 1] = {};
  Cheb c{};
};
}  // namespace

struct AmgDev {
  difvm_mesh* mesh = nullptr;
  int L = 0;                     // coarse levels 1..L (level L is the coarsest)
  std::vector<DevCsr> A;         // A[l], l = 1..L (A[0] unused: level 0 is K)
  DevCsr P0;                     // prolongation from level 1 to level 0
  std::vector<DevCsr> R, AP;     // R[l]: rows of level l+1, columns of l; AP[l] (l >= 1): rows of l; neither at
                                 // level L-1 >= 1
  std::vector<double*> b, bd, res, x;  // per level (index 0: res only; bd: D^-1 b, levels 1..L-1)
  std::vector<double*> xs, t, d0;      // levels 1..L-1 (t, d0: L-2): pre-smoothed x, xs + P x_{l+1}, first
                                       // post-smoothing step
  std::vector<double> hi;        // levels 0..L-1: upper end of the Chebyshev interval
  double* cinv = nullptr;        // dense inverse of A_L, row-major
  // level L-1 >= 1 in three passes (AmgFused), or with L = 2 in two (S.n > 0): H = G A_2^-1, dense rows(1) x rows(2)
  DevCsr G, GT, S, RS;
  double* H = nullptr;
  double alpha = 0.0, beta = 0.0;
  AmgBlock block;
  std::vector<int> rows;
  std::vector<void*> allocs;
};

namespace {

template <class T>
T* up(AmgDev* a, const std::vector<T>& v, hipStream_t s) {
  T* p = dalloc<T>(ctx_of(a->mesh), v.size());
  a->allocs.push_back(p);
  upload(p, v, s);
  return p;
}
// Waits for the stream when it goes out of scope: declared after host arrays that uploads read, so that an exception
// (a failed allocation) does not free them under a copy.
struct Drain {
  hipStream_t s;
  ~Drain() { (void)hipStreamSynchronize(s); }
};
double* work(AmgDev* a, size_t n) {
  double* p = dalloc<double>(ctx_of(a->mesh), n);
  a->allocs.push_back(p);
  return p;
}

// Lanes per CSR row: per_lane to 2 per_lane entries per lane on average.  The single-product kernels
// take 4 to 8 (their eight loads in flight hide the gather latency without many short-lived waves;
// they wait on memory latency more than on bandwidth); the two-product pass over A P takes 2 to 4.
// A matrix of few rows gets more lanes (down to 2 entries each) until the launch has 64k threads:
// there the chip is far from full and each lane's chain of loads is the whole kernel's time.
int lanes_for(int n, size_t nnz, int per_lane) {
  double avg = n ? (double)nnz / n : 0.0;
  int sw = 1;
  while (sw < 64 && sw * 2 * per_lane <= avg) sw *= 2;
  while (sw < 64 && (size_t)n * sw < 65536 && sw * 4 <= avg) sw *= 2;
  return sw;
}

DevCsr upload_csr(AmgDev* a, const AmgCsr& M, bool with_diag, hipStream_t s, int per_lane = 4) {
  DevCsr d;
  d.n = M.n;
  d.nnz = (int)M.col.size();
  d.sw = lanes_for(M.n, M.col.size(), per_lane);
  d.ptr = up(a, M.ptr, s);
  d.col = up(a, M.col, s);
  d.val = up(a, M.val, s);
  if (with_diag) d.diag = up(a, M.diag, s);
  return d;
}

// ---- kernels ------------------------------------------------------------------------------------
// Every segment's CG stopped: the V-cycle of an iteration queued past the stop has nothing to do.
// The flags are written by the CG kernels queued before the V-cycle on the same stream and by the test
// blocks of its first kernel (below): every wave reads them itself, one segment per lane, and votes (no
// barrier).  A wave of the first kernel may see them either way; the others see what was written before
// them.  LATE (meshes of few tiles, where a kernel's time is its chain of dependent loads): the vote is
// taken when a value is stored, so that no load waits for the flags; the kernels of an iteration queued past
// the stop then read what they would, which there costs less.  Otherwise it is taken first and the wave returns.
struct StopFlags {
  const PcgCtl* ctl;  // nullptr: never stopped
  int nseg;
};
__device__ __forceinline__ int load_stops(const StopFlags& st) {  // 1 if this lane saw only stopped segments
  if (!st.ctl) return 0;
  if (st.nseg == 1) return st.ctl->done;  // a scalar load
  const int lane = threadIdx.x & 63;
  int all = st.ctl[min(lane, st.nseg - 1)].done;  // (no loop around the first load, which would wait for it)
  for (int g = lane + 64; g < st.nseg; g += 64) all &= st.ctl[g].done;
  return all;
}
__device__ __forceinline__ bool stopped(int flags) { return __all(flags) != 0; }

// The stopping test of CG iterate k (its r.r partials rr), which the product of iteration k + 1 would make:
// the cycle's first kernel makes it in blocks of their own, one segment after another, so that after the
// last iteration the rest of the cycle returns at once.
struct CycleTest {
  PcgCtl* ctl;
  double* rr;
  int k, nseg;
  int blocks;  // the launch's first blocks (a multiple of 8, so that the others keep their XCDs)
};
template <bool FINE>
__device__ __forceinline__ void test_iterate(const CycleTest& t, const Tiles& T) {
  for (int s = blockIdx.x; s < t.nseg; s += t.blocks) {
    PcgCtl* ctl = t.ctl + s;
    const int done = ctl->done, maxit = ctl->maxit;  // uniform over the block: only this block writes them
    const double tol = ctl->tol, bn = ctl->bn;
    double rr[1];
    seg_totals<1, BLOCK, FINE>(t.rr, T.ntile, seg_first(T, s), seg_count(T, s), rr);
    const double rn = sqrt(rr[0]);
    const bool conv = rn <= tol * bn;
    if (threadIdx.x == 0 && !done && (conv || t.k >= maxit)) {
      ctl->done = 1;
      ctl->iters = t.k;
      ctl->res = rn / bn;
      ctl->status = conv ? 0 : DIFVM_WARN_NOT_CONVERGED;
    }
  }
}

// Sum of val[q] x(col[q]) over q = lo, lo + SW, lo + 2 SW, ... < hi (one lane's share of a CSR row),
// in that order, with the loads of UN entries in flight together (rows of a few entries per lane
// would otherwise wait on one load chain per entry; with 4 to 8 entries per lane, one round).  Entries past the row's end load its last entry
// (no branch around a load, which would make each one wait) and are not added.
template <int SW, int UN = 8, class X>
__device__ __forceinline__ double csr_lane_dot(int lo, int hi, const int32_t* __restrict__ col,
                                               const double* __restrict__ val, X&& x) {
  double s = 0.0;
  for (int q = lo; q < hi; q += UN * SW) {
    int c[UN];
    double v[UN], xv[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      int k = min(q + u * SW, hi - 1);
      c[u] = col[k];
      v[u] = val[k];
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) xv[u] = x(c[u]);
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (q + u * SW < hi) s += v[u] * xv[u];
  }
  return s;
}

// The first UN entries of a lane's share, loaded, gathered and summed in three steps, so that a kernel can have two
// matrices' in flight together; the rest after them.
template <int SW, int UN>
struct CsrBatch {
  int c[UN];
  double v[UN], xv[UN];
  __device__ __forceinline__ void load(int lo, int hi, const int32_t* __restrict__ col, const double* __restrict__ val) {
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int k = max(min(lo + u * SW, hi - 1), 0);  // an empty row: the array's first entry, not added
      c[u] = col[k];
      v[u] = val[k];
    }
  }
  __device__ __forceinline__ void gather(const double* __restrict__ x) {
#pragma unroll
    for (int u = 0; u < UN; ++u) xv[u] = x[c[u]];
  }
  __device__ __forceinline__ double sum(int lo, int hi, const int32_t* __restrict__ col, const double* __restrict__ val,
                                        const double* __restrict__ x) const {
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (lo + u * SW < hi) s += v[u] * xv[u];
    return s + csr_lane_dot<SW, UN>(lo + UN * SW, hi, col, val, [&](int j) { return x[j]; });
  }
};

// The same for two value arrays on one pattern: sa = sum va[q] x(col[q]), sb = sum vb[q] x(col[q]).
template <int SW, int UN = 4, class X>
__device__ __forceinline__ void csr_lane_dot2(int lo, int hi, const int32_t* __restrict__ col,
                                              const double* __restrict__ va, const double* __restrict__ vb, X&& x,
                                              double& sa, double& sb) {
  sa = 0.0;
  sb = 0.0;
  for (int q = lo; q < hi; q += UN * SW) {
    int c[UN];
    double a[UN], b[UN], xv[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      int k = min(q + u * SW, hi - 1);
      c[u] = col[k];
      a[u] = va[k];
      b[u] = vb[k];
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) xv[u] = x(c[u]);
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (q + u * SW < hi) {
        sa += a[u] * xv[u];
        sb += b[u] * xv[u];
      }
  }
}

// column of slot `at` in row i (16-bit offsets when the mesh has them)
template <bool OFF16>
__device__ __forceinline__ int slot_col_of(const SellView& K, int i, int at) {
  if constexpr (OFF16) return i + K.off16[at];
  else return K.col[at];
}

// Off-diagonal part of row i of K applied to f: sum over the row's slots of K_ij f(j) (padding and
// boundary slots hold 0 and the row's own index)
// (slots in layout order, the first four with every load issued before any is used)
template <bool OFF16, class F>
__device__ __forceinline__ double sell_offdiag(const SellView& K, int i, SlotRange R, F&& f) {
  double acc = 0.0;
  walk_row<4>(R.width, [&](auto Wc, int k0) {
    constexpr int N = decltype(Wc)::value;
    double a[N], fj[N];
    int j[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
      int at = R.base + (k0 + k) * SLICE;
      a[k] = K.val[at];
      j[k] = slot_col_of<OFF16>(K, i, at);
    }
#pragma unroll
    for (int k = 0; k < N; ++k) fj[k] = f(j[k]);
#pragma unroll
    for (int k = 0; k < N; ++k) acc = __builtin_fma(a[k], fj[k], acc);
  });
  return acc;
}

// The degree-2 Chebyshev sweep in D^-1 A over [lo, hi] (hi bounds the spectrum of D^-1 A), the same
// before and after the coarse correction.  From x with residual rh0 = D^-1 (b - A x):  d0 = rh0 / theta,  rh1 = rh0 - D^-1 K d0,  d1 = c_d d0 + c_r rh1,
// x <- x + d0 + d1 (coefficients: Cheb, amg.h).
// That sweep from zero at a finest-level cell: r its right-hand side, d the diagonal, s the off-diagonal part of K on
// cheb_d0 (one arithmetic, written out, for both kernels that make it: a solve has the same bits with either).
__device__ __forceinline__ double cheb_d0(double r, double d, const Cheb& c) { return r / d * c.inv_theta; }
__device__ __forceinline__ double cheb_from_zero(double r, double d, double s, const Cheb& c) {
#pragma clang fp contract(off)
  const double d0 = cheb_d0(r, d, c), rh1 = r / d - __builtin_fma(d, d0, s) / d;
  return d0 + __builtin_fma(c.c_r, rh1, c.c_d * d0);
}

// Row range of cell I of a finest-level pass, loaded at a clamped index, without a branch around the load, so
// that it is in flight together with the flag reads.  Threads past the last cell take that cell's row and
// store nothing: every lane stays active for the vote.
#define DIFVM_AMG_CELL(I)                                 \
  const int flags = load_stops(ctl);                      \
  const bool in = I < K.nc;                               \
  I = min(I, K.nc - 1);                                   \
  SlotRange R = slots_of(K, I);                           \
  if (!LATE && (stopped(flags) || !in)) return

// the stopping test in the kernel's first blocks (LATE and quarter-tile partials go together: fine_spans)
#define DIFVM_AMG_TEST                 \
  if ((int)blockIdx.x < test.blocks) { \
    test_iterate<LATE>(test, T);       \
    return;                            \
  }

// level 0, down, first pass (x = 0, b = r): xs = d0 + d1, with d0 = D^-1 r / theta
template <bool OFF16, bool LATE>
__global__ __launch_bounds__(BLOCK) void k_amg_cheb_pre1(SellView K, Tiles T, CycleTest test,
                                                         const double* __restrict__ r, double* __restrict__ xs, Cheb c,
                                                         StopFlags ctl) {
  DIFVM_AMG_TEST;
  int i = xcd_tile(blockIdx.x - test.blocks, gridDim.x - test.blocks) * BLOCK + threadIdx.x;
  DIFVM_AMG_CELL(i);
  const double di = K.diag[i], ri = r[i];
  const double s = sell_offdiag<OFF16>(K, i, R, [&](int j) { return cheb_d0(r[j], K.diag[j], c); });
  if (!LATE || (!stopped(flags) && in)) xs[i] = cheb_from_zero(ri, di, s, c);
}

// The same on meshes of few tiles (fine_spans), joined with the update of the CG iteration before it: x and r, the
// partials of r.r, xs.  Each cell makes its neighbours' new residuals again from the old ones (the same
// operations, so the same bits) instead of waiting for a kernel that stores them, which is why r goes to a
// second array.  12 gathers per cell instead of 8, and a launch less: there an iteration's time is its launches
// and each kernel's chain of loads.  A segment that has stopped hands its r on.
// Per CG iteration, separate kernels -> joint: 48,000 cells 41.6 -> 38.9 us, 93,750 47.7 -> 44.4, 384,000 77.0 -> 75.0.
template <bool OFF16>
__global__ __launch_bounds__(QUARTER) void k_amg_step_pre1(SellView K, Tiles T, CgStep st, double* __restrict__ xs,
                                                           double* __restrict__ rr, int k, Cheb c, PcgCtl* ctls) {
  constexpr int W = 4;
  const Span ti = span_of<true>(T);
  PcgCtl* ctl = ctls + ti.s;
  const bool done = ctl->done != 0;
  const double rho = ctl->rho[(k - 1) & 1];
  const int i0 = ti.lo + (int)threadIdx.x, i = min(i0, ti.end - 1);
  const SlotRange R = slots_of(K, i);
  const double xi = st.x[i], pi = st.p[i], r_i = st.r[i], q_i = st.q[i], di = K.diag[i];
  double a[W], rj[W], qj[W], dj[W];
  const int n0 = min(R.width, W);
  if (n0 > 0) {
    int j[W];
#pragma unroll
    for (int s = 0; s < W; ++s) {
      const int at = R.base + (s < n0 ? s : 0) * SLICE;  // past n0 the first slot again, not added
      a[s] = K.val[at];
      j[s] = slot_col_of<OFF16>(K, i, at);
    }
#pragma unroll
    for (int s = 0; s < W; ++s) {
      rj[s] = st.r[j[s]];
      qj[s] = st.q[j[s]];
      dj[s] = K.diag[j[s]];
    }
  }
  double pq[1];
  seg_totals<1, QUARTER, true>(st.pq, T.ntile, seg_first(T, ti.s), seg_count(T, ti.s), pq);
  const double alpha = rho / pq[0];
  auto residual = [&](double ro, double qo) { return done ? ro : __builtin_fma(-alpha, qo, ro); };
  const double ri = residual(r_i, q_i);
  double acc = 0.0;
#pragma unroll
  for (int s = 0; s < W; ++s)
    if (s < n0) acc = __builtin_fma(a[s], cheb_d0(residual(rj[s], qj[s]), dj[s], c), acc);
  for (int s = W; s < R.width; ++s) {
    const int at = R.base + s * SLICE, j = slot_col_of<OFF16>(K, i, at);
    acc = __builtin_fma(K.val[at], cheb_d0(residual(st.r[j], st.q[j]), K.diag[j], c), acc);
  }
  double v[1] = {0.0};
  if (i0 < ti.hi) {
    if (!done) st.x[i] = __builtin_fma(alpha, pi, xi);
    st.r_new[i] = ri;
    xs[i] = cheb_from_zero(ri, di, acc, c);
    v[0] = ri * ri;
  }
  put_partial<1, QUARTER, true>(v, rr, T.ntile, ti);
}

// level 0, down, second pass: res = r - K xs
template <bool OFF16, bool LATE>
__global__ __launch_bounds__(BLOCK) void k_amg_cheb_pre2(SellView K, Tiles T, CycleTest test, const double* __restrict__ r,
                                                         const double* __restrict__ xs, double* __restrict__ res,
                                                         StopFlags ctl) {
  DIFVM_AMG_TEST;
  int i = xcd_tile(blockIdx.x - test.blocks, gridDim.x - test.blocks) * BLOCK + threadIdx.x;
  DIFVM_AMG_CELL(i);
  const double ri = r[i];
  double kx = K.diag[i] * xs[i] + sell_offdiag<OFF16>(K, i, R, [&](int j) { return xs[j]; });
  if (!LATE || (!stopped(flags) && in)) res[i] = ri - kx;
}

// level 0, up, first pass (x = t): d0 = D^-1 (r - K t) / theta
template <bool OFF16, bool LATE>
__global__ __launch_bounds__(BLOCK) void k_amg_cheb_post1(SellView K, const double* __restrict__ r,
                                                          const double* __restrict__ t, double* __restrict__ d0,
                                                          Cheb c, StopFlags ctl) {
  int i = xcd_tile(blockIdx.x, gridDim.x) * BLOCK + threadIdx.x;
  DIFVM_AMG_CELL(i);
  const double di = K.diag[i], ri = r[i];
  double kt = di * t[i] + sell_offdiag<OFF16>(K, i, R, [&](int j) { return t[j]; });
  if (!LATE || (!stopped(flags) && in)) d0[i] = (ri - kt) / di * c.inv_theta;
}

// level 0, up, second pass: z = t + d0 + d1 (in t's place) with rh1 = theta d0 - D^-1 K d0, and per-tile partials
// of r.z (part[k] by tile or by quarter, as the CG reads them).  One cell per thread, like the other
// finest-level passes (four cells per thread left each thread's rows one after another).
template <bool OFF16, bool FINE>
__global__ __launch_bounds__(FINE ? QUARTER : TILE) void k_amg_cheb_post2(SellView K, Tiles T, const double* __restrict__ r,
                                                             const double* __restrict__ d0, double* __restrict__ z,
                                                             double* __restrict__ part, Cheb c, StopFlags ctl) {
  const Span sp = span_of<FINE>(T);
  const int flags = load_stops(ctl);
  if (!FINE && stopped(flags)) return;
  double v[1] = {0.0};
  double zi = 0.0;
  const int i = sp.lo + (int)threadIdx.x;
  if (i < sp.hi) {
    SlotRange R = slots_of(K, i);
    const double di = K.diag[i], d0i = d0[i], ti = z[i], ri = r[i];
    double kd0 = di * d0i + sell_offdiag<OFF16>(K, i, R, [&](int j) { return d0[j]; });
    double rh1 = c.theta * d0i - kd0 / di;
    zi = ti + d0i + (c.c_d * d0i + c.c_r * rh1);
    v[0] = ri * zi;
  }
  if (FINE && stopped(flags)) return;  // every wave of the block alike: written before this launch
  if (i < sp.hi) z[i] = zi;
  if (part) put_partial<1, FINE ? QUARTER : TILE, FINE>(v, part, T.ntile, sp);
}

// Coarse levels smooth with the same degree-2 Chebyshev sweep as level 0 (interval [hi / 10, hi],
// hi from the setup), two CSR passes per sweep.
// Row bounds are loaded at a clamped index before the flag reads (no branch around the loads, so
// both are in flight together); rows past the end get an empty range.  The kernels load their own
// row's values (at the clamped index rr) before the row's entries, so that those loads are in flight
// with the entries' and not issued after the gathers.  Blocks map to rows XCD by XCD
// (each XCD a contiguous run of rows), so the finer-level entries that neighbouring rows gather meet
// in one L2.
#define DIFVM_AMG_ROW(ptr, n)                                  \
  int g = xcd_tile(blockIdx.x, gridDim.x) * BLOCK + threadIdx.x; \
  int row = g / SW, lane = g % SW;                             \
  const int rr = min(row, n - 1);                              \
  int p0 = ptr[rr], p1 = ptr[rr + 1];                          \
  const int flags = load_stops(ctl);                           \
  if (!LATE && stopped(flags)) return;                         \
  int lo = p0 + lane, hi = row < n ? p1 : 0

// out = R x (rows of the coarser level); with diag, also outd = out / diag (what the coarser level's
// pre-smoothing gathers)
template <int SW, bool LATE>
__global__ __launch_bounds__(BLOCK) void k_amg_restrict(int n, const int32_t* __restrict__ ptr,
                                                        const int32_t* __restrict__ col, const double* __restrict__ val,
                                                        const double* __restrict__ xin, const double* __restrict__ diag,
                                                        double* __restrict__ out, double* __restrict__ outd,
                                                        StopFlags ctl) {
  DIFVM_AMG_ROW(ptr, n);
  const double dg = diag ? diag[rr] : 1.0;
  double s = csr_lane_dot<SW>(lo, hi, col, val, [&](int j) { return xin[j]; });
  s = lanes_sum<SW>(s);
  if ((!LATE || !stopped(flags)) && row < n && lane == 0) {
    out[row] = s;
    if (diag) outd[row] = s / dg;
  }
}

// coarse level, down, first pass (x = 0): xs = d0 + d1 with d0 = bd / theta (bd = D^-1 b)
template <int SW, bool LATE>
__global__ __launch_bounds__(BLOCK) void k_amg_cpre1(int n, const int32_t* __restrict__ ptr,
                                                     const int32_t* __restrict__ col, const double* __restrict__ val,
                                                     const double* __restrict__ diag, const double* __restrict__ bd,
                                                     double* __restrict__ xs, Cheb c, StopFlags ctl) {
  DIFVM_AMG_ROW(ptr, n);
  const double di = diag[rr], rh0 = bd[rr];
  double s = csr_lane_dot<SW>(lo, hi, col, val, [&](int j) { return bd[j]; });
  s = lanes_sum<SW>(s);
  if ((!LATE || !stopped(flags)) && row < n && lane == 0) {
    double d0 = rh0 * c.inv_theta;
    double kd0 = di * d0 + s * c.inv_theta;
    double rh1 = rh0 - kd0 / di;
    xs[row] = d0 + (c.c_d * d0 + c.c_r * rh1);
  }
}

// coarse level, down, second pass: res = b - A xs
template <int SW, bool LATE>
__global__ __launch_bounds__(BLOCK) void k_amg_cpre2(int n, const int32_t* __restrict__ ptr,
                                                     const int32_t* __restrict__ col, const double* __restrict__ val,
                                                     const double* __restrict__ diag, const double* __restrict__ b,
                                                     const double* __restrict__ xs, double* __restrict__ res,
                                                     StopFlags ctl) {
  DIFVM_AMG_ROW(ptr, n);
  const double bi = b[rr], di = diag[rr], xi = xs[rr];
  double s = csr_lane_dot<SW>(lo, hi, col, val, [&](int j) { return xs[j]; });
  s = lanes_sum<SW>(s);
  if ((!LATE || !stopped(flags)) && row < n && lane == 0) res[row] = bi - di * xi - s;
}

// coarse level, up, first pass: t = xs + P xc and, since b - A t = res - (A P) xc,
// d0 = D^-1 (res - (A P) xc) / theta; one pass over the pattern of A P
template <int SW, bool LATE>
__global__ __launch_bounds__(BLOCK) void k_amg_cup1(int n, const int32_t* __restrict__ ptr,
                                                    const int32_t* __restrict__ col, const double* __restrict__ ap,
                                                    const double* __restrict__ pv, const double* __restrict__ diag,
                                                    const double* __restrict__ xs, const double* __restrict__ res,
                                                    const double* __restrict__ xc, double* __restrict__ t,
                                                    double* __restrict__ d0, Cheb c, StopFlags ctl) {
  DIFVM_AMG_ROW(ptr, n);
  const double xi = xs[rr], ri = res[rr], di = diag[rr];
  double sp, sq;
  csr_lane_dot2<SW>(lo, hi, col, pv, ap, [&](int j) { return xc[j]; }, sp, sq);
  sp = lanes_sum<SW>(sp);
  sq = lanes_sum<SW>(sq);
  if ((!LATE || !stopped(flags)) && row < n && lane == 0) {
    t[row] = xi + sp;
    d0[row] = (ri - sq) / di * c.inv_theta;
  }
}

// coarse level, up, second pass: x = t + d0 + d1 with rh1 = theta d0 - D^-1 A d0
template <int SW, bool LATE>
__global__ __launch_bounds__(BLOCK) void k_amg_cup2(int n, const int32_t* __restrict__ ptr,
                                                    const int32_t* __restrict__ col, const double* __restrict__ val,
                                                    const double* __restrict__ diag, const double* __restrict__ t,
                                                    const double* __restrict__ d0, double* __restrict__ x, Cheb c,
                                                    StopFlags ctl) {
  DIFVM_AMG_ROW(ptr, n);
  const double di = diag[rr], d0i = d0[rr], ti = t[rr];
  double s = csr_lane_dot<SW>(lo, hi, col, val, [&](int j) { return d0[j]; });
  s = lanes_sum<SW>(s);
  if ((!LATE || !stopped(flags)) && row < n && lane == 0) {
    double rh1 = c.theta * d0i - (di * d0i + s) / di;
    x[row] = ti + d0i + (c.c_d * d0i + c.c_r * rh1);
  }
}

// coarsest: x = A_L^-1 b with the dense inverse (row-major, n <= 2048): one block per row, threads
// over the columns (every load of a thread in flight at once: n / BLOCK <= 8), per-wave shuffle trees
// and the four wave sums added in order; b is read through L2
constexpr int MAX_DENSE = 2048;
template <bool LATE>
__device__ __forceinline__ void dense_row(int i, int n, const double* __restrict__ inv, const double* __restrict__ b,
                                          double* __restrict__ x, int flags) {
  __shared__ double ws[BLOCK / 64];
  const double* row = inv + (size_t)i * n;
  constexpr int U = MAX_DENSE / BLOCK;
  double v[U], w[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {  // columns past the end load column n-1 (no branch around a load)
    int j = min((int)threadIdx.x + u * BLOCK, n - 1);
    v[u] = row[j];
    w[u] = b[j];
  }
  double s = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u)
    if ((int)threadIdx.x + u * BLOCK < n) s += v[u] * w[u];
  s = lanes_sum<64>(s);
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = s;
  __syncthreads();
  const bool go = !LATE || !stopped(flags);
  if (threadIdx.x == 0 && go) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < BLOCK / 64; ++w) t += ws[w];
    x[i] = t;
  }
}
template <bool LATE>
__global__ __launch_bounds__(BLOCK) void k_amg_coarsest(int n, const double* __restrict__ inv,
                                                        const double* __restrict__ b, double* __restrict__ x,
                                                        StopFlags ctl) {
  const int flags = load_stops(ctl);
  if (!LATE && stopped(flags)) return;
  dense_row<LATE>(blockIdx.x, n, inv, b, x, flags);
}

// The level above the coarsest in three passes (AmgFused), each two kernels' work in one launch: rows of that level
// (SW lanes each) in the first blocks, rows of the coarsest in the others.
// A cycle has three launches less than with six passes and the coarsest solve, and gathers as much: what bounds it on
// large meshes are those gathers, a cache line a cycle and compute unit.  Per CG iteration 384,000 cells 74 -> 66 us,
// 1,053,696 140 -> 138.
#define DIFVM_AMG_MID(ptr, n)                                                \
  const int flags = load_stops(ctl);                                         \
  if (!LATE && stopped(flags)) return;                                       \
  const int blocks1 = ((n) * SW + BLOCK - 1) / BLOCK;                        \
  const int g = xcd_tile(blockIdx.x, blocks1) * BLOCK + threadIdx.x;         \
  const int row = g / SW, lane = g % SW, rr = min(row, (n) - 1)

// xs = alpha bd - beta D^-1 A bd (bd = D^-1 b);  b2 = G^T b, a wave per row
template <int SW, bool LATE>
__global__ __launch_bounds__(BLOCK) void k_amg_mid1(int n, const int32_t* __restrict__ ptr,
                                                    const int32_t* __restrict__ col, const double* __restrict__ val,
                                                    const double* __restrict__ diag, const double* __restrict__ bd,
                                                    double* __restrict__ xs, double alpha, double beta, int n2,
                                                    const int32_t* __restrict__ tptr, const int32_t* __restrict__ tcol,
                                                    const double* __restrict__ tval, const double* __restrict__ b,
                                                    double* __restrict__ b2, StopFlags ctl) {
  DIFVM_AMG_MID(ptr, n);
  if ((int)blockIdx.x < blocks1) {
    const int p0 = ptr[rr], p1 = ptr[rr + 1];
    const double di = diag[rr], bi = bd[rr];
    const double a = lanes_sum<SW>(
        csr_lane_dot<SW>(p0 + lane, row < n ? p1 : 0, col, val, [&](int j) { return bd[j]; }));
    if ((!LATE || !stopped(flags)) && row < n && lane == 0) xs[row] = alpha * bi - beta / di * (di * bi + a);
  } else {
    const int row2 = ((int)blockIdx.x - blocks1) * (BLOCK / 64) + (threadIdx.x >> 6), r2 = min(row2, n2 - 1);
    const int p0 = tptr[r2], p1 = tptr[r2 + 1];
    const double s = lanes_sum<64>(csr_lane_dot<64, 12>(p0 + (threadIdx.x & 63), row2 < n2 ? p1 : 0, tcol, tval,
                                                    [&](int j) { return b[j]; }));
    if ((!LATE || !stopped(flags)) && row2 < n2 && (threadIdx.x & 63) == 0) b2[row2] = s;
  }
}

// resd = D^-1 (b - A xs);  x2 = A_2^-1 b2, a block per row
template <int SW, bool LATE>
__global__ __launch_bounds__(BLOCK) void k_amg_mid2(int n, const int32_t* __restrict__ ptr,
                                                    const int32_t* __restrict__ col, const double* __restrict__ val,
                                                    const double* __restrict__ diag, const double* __restrict__ b,
                                                    const double* __restrict__ xs, double* __restrict__ resd, int n2,
                                                    const double* __restrict__ inv, const double* __restrict__ b2,
                                                    double* __restrict__ x2, StopFlags ctl) {
  DIFVM_AMG_MID(ptr, n);
  if ((int)blockIdx.x < blocks1) {
    const int p0 = ptr[rr], p1 = ptr[rr + 1];
    const double bi = b[rr], di = diag[rr], xi = xs[rr];
    const double s = lanes_sum<SW>(
        csr_lane_dot<SW>(p0 + lane, row < n ? p1 : 0, col, val, [&](int j) { return xs[j]; }));
    if ((!LATE || !stopped(flags)) && row < n && lane == 0) resd[row] = (bi - di * xi - s) / di;
  } else {
    dense_row<LATE>((int)blockIdx.x - blocks1, n2, inv, b2, x2, flags);
  }
}

// x = xs + q(res) + G x2
template <int SW, bool LATE>
__global__ __launch_bounds__(BLOCK) void k_amg_up(int n, const int32_t* __restrict__ ptr,
                                                  const int32_t* __restrict__ col, const double* __restrict__ val,
                                                  const double* __restrict__ diag, const int32_t* __restrict__ gptr,
                                                  const int32_t* __restrict__ gcol, const double* __restrict__ gval,
                                                  double alpha, double beta, const double* __restrict__ xs,
                                                  const double* __restrict__ resd, const double* __restrict__ x2,
                                                  double* __restrict__ x, StopFlags ctl) {
  DIFVM_AMG_ROW(ptr, n);
  const int glo = gptr[rr] + lane, ghi = row < n ? gptr[rr + 1] : 0;
  const double di = diag[rr], rd = resd[rr], xi = xs[rr];
  CsrBatch<SW, 4> ba;
  CsrBatch<SW, 6> bg;
  ba.load(lo, hi, col, val);
  bg.load(glo, ghi, gcol, gval);
  ba.gather(resd);
  bg.gather(x2);
  const double a = lanes_sum<SW>(ba.sum(lo, hi, col, val, resd)), s = lanes_sum<SW>(bg.sum(glo, ghi, gcol, gval, x2));
  if ((!LATE || !stopped(flags)) && row < n && lane == 0) x[row] = xi + (alpha * rd - beta / di * (di * rd + a)) + s;
}

// The same of three levels on small meshes (amg_create) in two passes, the whole way down: rows of level 1 (SW lanes each) in the first blocks,
//   xs = alpha bd - beta D^-1 A bd,  resd = D^-1 S bd
// and rows of level 2 (a wave each) in the others, b2 = (R S) bd.  With the pass below it stands for the
// six of the level and the dense solve: on meshes of few tiles a cycle's time is its number of launches
// (each some 3 us on the device and 2.7 for the host), while the 4.5 times as many entries of S stay
// in the caches.  A CG iteration's 14 launches become 10: 48,000 cells 58 to 42 us, 93,750 61 to 47,
// 162,000 67 to 52 (31, 38 and 45 us where the host is fast enough for the device to be the limit).  Eight
// or 32 lanes per row measured the same or slower, 64 slower (38 to 42 us at 93,750 cells).
template <int SW, bool LATE>
__global__ __launch_bounds__(BLOCK) void k_amg_down1(int n, const int32_t* __restrict__ aptr,
                                                     const int32_t* __restrict__ acol, const double* __restrict__ aval,
                                                     const double* __restrict__ diag, const int32_t* __restrict__ sptr,
                                                     const int32_t* __restrict__ scol, const double* __restrict__ sval,
                                                     int n2, const int32_t* __restrict__ rptr,
                                                     const int32_t* __restrict__ rcol, const double* __restrict__ rval,
                                                     double alpha, double beta, const double* __restrict__ bd,
                                                     double* __restrict__ xs, double* __restrict__ resd,
                                                     double* __restrict__ b2, StopFlags ctl) {
  const int flags = load_stops(ctl);
  if (!LATE && stopped(flags)) return;
  const int blocks1 = (n * SW + BLOCK - 1) / BLOCK;
  auto x = [&](int j) { return bd[j]; };
  if ((int)blockIdx.x < blocks1) {
    const int g = blockIdx.x * BLOCK + threadIdx.x, row = g / SW, lane = g % SW, rr = min(row, n - 1);
    const int a0 = aptr[rr], a1 = aptr[rr + 1], s0 = sptr[rr], s1 = sptr[rr + 1];
    const double di = diag[rr], bi = bd[rr];
    double s = csr_lane_dot<SW>(s0 + lane, row < n ? s1 : 0, scol, sval, x);
    double a = csr_lane_dot<SW, 4>(a0 + lane, row < n ? a1 : 0, acol, aval, x);
    s = lanes_sum<SW>(s);
    a = lanes_sum<SW>(a);
    if ((!LATE || !stopped(flags)) && row < n && lane == 0) {
      resd[row] = s / di;
      xs[row] = alpha * bi - beta / di * (di * bi + a);
    }
  } else {
    const int row = ((int)blockIdx.x - blocks1) * (BLOCK / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int rr = min(row, n2 - 1);
    const int p0 = rptr[rr], p1 = rptr[rr + 1];
    double s = lanes_sum<64>(csr_lane_dot<64>(p0 + lane, row < n2 ? p1 : 0, rcol, rval, x));
    if ((!LATE || !stopped(flags)) && row < n2 && lane == 0) b2[row] = s;
  }
}

// and up: x = xs + q(res) + H b2, the dense row of H by SW lanes, four loads in flight
template <int SW, bool LATE>
__global__ __launch_bounds__(BLOCK) void k_amg_up1(int n, const int32_t* __restrict__ ptr,
                                                   const int32_t* __restrict__ col, const double* __restrict__ val,
                                                   const double* __restrict__ diag, int n2,
                                                   const double* __restrict__ H, double alpha, double beta,
                                                   const double* __restrict__ xs, const double* __restrict__ resd,
                                                   const double* __restrict__ b2, double* __restrict__ x,
                                                   StopFlags ctl) {
  DIFVM_AMG_ROW(ptr, n);
  const double di = diag[rr], rd = resd[rr], xi = xs[rr];
  const double* h = H + (size_t)rr * n2;
  double a = csr_lane_dot<SW, 4>(lo, hi, col, val, [&](int j) { return resd[j]; });
  double s = 0.0;
  constexpr int UN = 8;
  for (int q = lane; q < n2; q += UN * SW) {
    double v[UN], w[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int k = min(q + u * SW, n2 - 1);
      v[u] = h[k];
      w[u] = b2[k];
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (q + u * SW < n2) s += v[u] * w[u];
  }
  a = lanes_sum<SW>(a);
  s = lanes_sum<SW>(s);
  if ((!LATE || !stopped(flags)) && row < n && lane == 0) x[row] = xi + (alpha * rd - beta / di * (di * rd + a)) + s;
}

// setup: H = G A_2^-1, one block per row of G
__global__ __launch_bounds__(BLOCK) void k_amg_h(int n2, const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                                 const double* __restrict__ val, const double* __restrict__ inv,
                                                 double* __restrict__ H) {
  const int p0 = ptr[blockIdx.x], p1 = ptr[blockIdx.x + 1];
  for (int c = threadIdx.x; c < n2; c += BLOCK) {
    double s = 0.0;
    for (int q = p0; q < p1; ++q) s += val[q] * inv[(size_t)col[q] * n2 + c];
    H[(size_t)blockIdx.x * n2 + c] = s;
  }
}

// level 0, up: t = xs + P xc in xs's place (one thread per row; almost every row of the finest prolongator has at
// most four entries, so four in flight)
template <bool LATE>
__global__ __launch_bounds__(BLOCK) void k_amg_prolong(int n, const int32_t* __restrict__ ptr,
                                                       const int32_t* __restrict__ col, const double* __restrict__ val,
                                                       const double* __restrict__ xc, double* __restrict__ t,
                                                       StopFlags ctl) {
  int i = xcd_tile(blockIdx.x, gridDim.x) * BLOCK + threadIdx.x;
  const int ii = min(i, n - 1);
  int lo = ptr[ii], hi = ptr[ii + 1];
  const int flags = load_stops(ctl);
  if (!LATE && (stopped(flags) || i >= n)) return;
  const double xi = t[ii];
  double s = csr_lane_dot<1, 4>(lo, hi, col, val, [&](int j) { return xc[j]; });
  if (!LATE || (!stopped(flags) && i < n)) t[i] = xi + s;
}

// ---------------------------------------------------------------------------------------------
// AMG-CG of a small mesh (one segment of at most four tiles, uniform rows of three or four slots, two levels, at
// most BLOCK_COARSE coarse rows), the whole solve in one block and launch, as k_pcg_segment does for Jacobi-CG: K's
// rows, the diagonal, r and p in registers (thread tid holds cells tid + c BLOCK_NT), x in LDS, the vector that a
// product gathers in LDS too, in two arrays by turns so that one barrier parts two passes.  An iteration is
// thirteen barriers (one more where P has rows of more than four entries) and three reductions instead of eight kernels.  What does not fit is read from L2 in every cycle,
// R and the coarse inverse (with more than four cells per thread P too): one compute unit gets 55 bytes a cycle
// by loads of 16 bytes per lane (30 by loads of 8) and 600 ns pass between a load and its use, so all of
// it is laid out again for whole 1 KB loads (AmgBlock) and taken several loads at a time.  The inverse grows with
// the square of its rows and bounds the largest of these meshes (8.9k of 39k cycles at 222 rows, 16.6k at 336).
// Per iteration in us, eight launches -> this: 968 prisms 33 -> 5.4, 2,048 34 -> 7.9, 3,872 (336 coarse rows) 34 -> 17,
// 1,296 tets 33 -> 7.7, 3,072 34 -> 11.8, 3,888 34 -> 16.  Replayed from a graph, ten PISO steps of 968 / 1,922 / 2,178 /
// 4,050 prisms 7.4 / 7.9 / 7.9 / 8.6 -> 3.0 / 3.6 / 4.6 / 6.9 ms.  With rows of any length (hexahedra),
// read from L2 in each of the five products, it took 24 us at 1,728 cells and 47 at 4,096 against 35: they take
// the eight launches, and so do more coarse rows (at 512 their reads alone are 16 us).
// A launch makes at most `chunk` iterations; what a further launch needs is stored when it ends unconverged.
// ---------------------------------------------------------------------------------------------
// acc + the four products of values a, b and entries j of f
__device__ __forceinline__ double four(double2 a, double2 b, ushort4 j, const double* f, double acc) {
  acc = __builtin_fma(a.x, f[j.x], acc);
  acc = __builtin_fma(a.y, f[j.y], acc);
  acc = __builtin_fma(b.x, f[j.z], acc);
  return __builtin_fma(b.y, f[j.w], acc);
}

// barrier that orders LDS alone: loads from memory stay in flight over it (what the waves share between two barriers
// is in LDS)
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int C, int W>
__global__ __launch_bounds__(BLOCK_NT) void k_amg_pcg_block(SellView K, int nt, AmgBlock M, const double* __restrict__ b,
                                                      double* __restrict__ x, double* __restrict__ rbuf,
                                                      double* __restrict__ pbuf, double tol, int maxit, int chunk,
                                                      bool first, PcgCtl* ctl) {
  constexpr int NT = BLOCK_NT, NTILE = NT * C / TILE, WAVES = NT / 64;
  static_assert(NTILE <= 4, "the tiles' sums fill one wave");
  __shared__ double va[C * NT], vb[C * NT], xs[C * NT], bc[BLOCK_COARSE], xc[BLOCK_COARSE], gs[2][64];
  __shared__ double2 xp[NT];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, n = K.nc;
  if (!first && ctl->done) return;
  if (first && tid == 0) ctl_start(ctl, tol, maxit);
  const int k0 = first ? 0 : ctl->next;
  double r[C], p[C], d[C], di[C];  // di: 1 / d
  // totals of NV values per cell (in the order of k_pcg_segment's); gs may be written again after the next barrier
  auto totals = [&](auto&& v, auto& tot) {
    constexpr int NV = sizeof(tot) / sizeof(double);
    wave_sums<NV * C>([&](int e) { return e % C * NT + tid < n ? v(e / C, e % C) : 0.0; },
                      [&](int e, double sum) { gs[e / C][e % C * WAVES + wid] = sum; });
    lds_barrier();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      double t = row_sum(gs[k][lane]);
      if (lane / TILE_WAVES >= nt) t = 0.0;
      t = swap_add16(t, t);
      tot[k] = wave_first(NTILE > 2 ? swap_add32(t, t) : t);
    }
  };
  double av[C][W];
  int jv[C][W];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    // cells past the last: an empty row, so that no branch is needed for them
    const int i = c * NT + tid;
    const bool in = i < n;
    const int ii = in ? i : 0, base = (ii >> 6) * (SLICE * W) + (ii & (SLICE - 1));  // uniform rows
#pragma unroll
    for (int k = 0; k < W; ++k) {
      const double a = K.val[base + k * SLICE];
      const int j = K.off16[base + k * SLICE];
      av[c][k] = in ? a : 0.0;
      jv[c][k] = i + (in ? j : 0);
    }
    xs[i] = in ? x[i] : 0.0;  // only this thread's entries are read
    d[c] = in ? K.diag[i] : 1.0;
    di[c] = 1.0 / d[c];
    r[c] = in && k0 > 0 ? rbuf[i] : 0.0;
    p[c] = in && k0 > 0 ? pbuf[i] : 0.0;
  }
  // out(c, off-diagonal part of row c applied to the vector f in LDS) for this thread's cells
  auto rows = [&](const double* f, auto&& out) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      double acc = 0.0;
#pragma unroll
      for (int k = 0; k < W; ++k) acc = __builtin_fma(av[c][k], f[jv[c][k]], acc);
      out(c, acc);
    }
  };
  const Cheb ch = M.c;
  double z[C], rho, rho_old = 0.0, bn, one[1], two[2];
  // What of the transfers and the inverse is in flight at once.  With four cells per thread there are registers
  // to load the first of each before the pass in front of its own; an offset that is zero, which the
  // compiler does not know, keeps it from holding all of it in scratch memory from before the loop.
  constexpr bool AHEAD = C <= 4;
  constexpr int UR = BLOCK_R_FOURS, UD = 8, CB = C < 4 ? C : C % 4 ? 3 : 4;  // fours of R, columns of the inverse, cells of P
  const int h = M.ld / 2, G = NT / h, g = tid / h;
  ushort4 rj[UR], pj[CB];
  double2 rv[UR][2], dv[UD], pv[CB][2];
  int again = 0;
  auto load_r = [&](int e) {
#pragma unroll
    for (int u = 0; u < UR; ++u) {
      const int f = e + u;
      rj[u] = M.rcol[f * NT + tid + again];
      rv[u][0] = M.rval[2 * f * NT + tid + again];
      rv[u][1] = M.rval[(2 * f + 1) * NT + tid + again];
    }
  };
  // thread t takes the pair of rows t % h of the inverse and every G-th column from t / h, so that a load of the block
  // is one run of the array
  auto load_d = [&](int q) {
#pragma unroll
    for (int u = 0; u < UD; ++u) dv[u] = M.inv[min(min(q + u * G, M.n2 - 1) * h + tid - g * h, M.n2 * h - 1) + again];
  };
  auto load_p = [&](int c0) {
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const int i = (c0 + c) * NT + tid + again;
      pj[c] = M.pcol[i];
      pv[c][0] = M.pval[i];
      pv[c][1] = M.pval[4 * TILE + i];
    }
  };
  if constexpr (AHEAD) load_p(0);  // kept
  // z = M^-1 r and rho = r.z; vb and gs are free at the start (every read is behind a barrier)
  auto cycle = [&]() {
    asm volatile("" : "+s"(again));
#pragma unroll
    for (int c = 0; c < C; ++c) vb[c * NT + tid] = r[c] * di[c] * ch.inv_theta;
    if constexpr (AHEAD) load_r(0);
    lds_barrier();
    rows(vb, [&](int c, double s) {  // rh1 = D^-1 (r - K d0), s without K's diagonal
      const double d0 = vb[c * NT + tid], rh1 = (r[c] - s) * di[c] - d0;
      va[c * NT + tid] = d0 + (ch.c_d * d0 + ch.c_r * rh1);
    });
    if constexpr (AHEAD) load_d(g);
    lds_barrier();
    rows(va, [&](int c, double s) { vb[c * NT + tid] = r[c] - __builtin_fma(d[c], va[c * NT + tid], s); });
    lds_barrier();
    for (int ps = 0; ps * BLOCK_R_ROWS < M.n2; ++ps) {  // b = R res
      const int e1 = M.first[ps + 1];
      double s = 0.0;
      for (int e = M.first[ps]; e < e1; e += UR) {
        if (!AHEAD || e > 0) load_r(e);
#pragma unroll
        for (int u = 0; u < UR; ++u) s = four(rv[u][0], rv[u][1], rj[u], vb, s);
      }
      s = lanes_sum<BLOCK_R_LANES>(s);
      if (const int row = ps * BLOCK_R_ROWS + tid / BLOCK_R_LANES; lane % BLOCK_R_LANES == 0 && row < M.n2) bc[row] = s;
    }
    lds_barrier();
    {  // x_2 = A_2^-1 b; past the last column zeros
      double s0 = 0.0, s1 = 0.0;
      for (int q = g; q < M.n2; q += UD * G) {
        if (!AHEAD || q > g) load_d(q);
        double bq[UD];
#pragma unroll
        for (int u = 0; u < UD; ++u) bq[u] = bc[min(q + u * G, M.n2 - 1)];
#pragma unroll
        for (int u = 0; u < UD; ++u) {
          if (q + u * G >= M.n2) bq[u] = 0.0;
          s0 = __builtin_fma(dv[u].x, bq[u], s0);
          s1 = __builtin_fma(dv[u].y, bq[u], s1);
        }
      }
      xp[tid] = {s0, s1};  // threads from G h on: not read
    }
    lds_barrier();
    for (int row = tid; row < M.n2; row += NT) {
      double s = 0.0;
      for (int k = 0; k < G; ++k) s += reinterpret_cast<const double*>(xp)[k * M.ld + row];
      xc[row] = s;
    }
    lds_barrier();
    // t = xs + P x_2, each thread's own entries of va, which no pass since the last barriers but one reads
#pragma unroll
    for (int c0 = 0; c0 < C; c0 += CB) {
      if (!AHEAD) load_p(c0);
#pragma unroll
      for (int c = 0; c < CB; ++c) va[(c0 + c) * NT + tid] = four(pv[c][0], pv[c][1], pj[c], xc, va[(c0 + c) * NT + tid]);
    }
    if (M.nlong) {
      lds_barrier();
      for (int k = tid; k < M.nlong; k += NT) {
        double s = va[M.lrow[k]];
        for (int q = M.lptr[k]; q < M.lptr[k + 1]; ++q) s = __builtin_fma(M.lval[q], xc[M.lcol[q]], s);
        va[M.lrow[k]] = s;
      }
    }
    lds_barrier();
    rows(va, [&](int c, double s) {
      vb[c * NT + tid] = (r[c] - __builtin_fma(d[c], va[c * NT + tid], s)) * di[c] * ch.inv_theta;
    });
    lds_barrier();
    rows(vb, [&](int c, double s) {
      const double d0 = vb[c * NT + tid], rh1 = ch.theta * d0 - (d0 + s * di[c]);
      z[c] = va[c * NT + tid] + d0 + (ch.c_d * d0 + ch.c_r * rh1);
    });
    totals([&](int, int c) { return r[c] * z[c]; }, one);
    rho = one[0];
  };
  if (k0 == 0) {
#pragma unroll
    for (int c = 0; c < C; ++c) va[c * NT + tid] = xs[c * NT + tid];
    lds_barrier();
    double bv[C];
    rows(va, [&](int c, double s) {
      const int i = c * NT + tid;
      bv[c] = i < n ? b[i] : 0.0;
      r[c] = bv[c] - __builtin_fma(d[c], xs[i], s);
    });
    totals([&](int k, int c) { return k == 0 ? bv[c] * bv[c] : r[c] * r[c]; }, two);
    bn = sqrt(two[0]);
    const double rn = sqrt(two[1]);
    const bool zero_b = bn == 0.0, stop = zero_b || rn <= tol * bn, capped = !stop && maxit <= 0;
    if (tid == 0) {
      ctl->bn = bn;
      ctl->res = zero_b ? 0.0 : rn / bn;
      ctl->done = stop || capped ? 1 : 0;
      if (capped) ctl->status = DIFVM_WARN_NOT_CONVERGED;
    }
    if (zero_b)
#pragma unroll
      for (int c = 0; c < C; ++c)
        if (c * NT + tid < n) x[c * NT + tid] = 0.0;
    if (stop || capped) return;
    lds_barrier();  // gs is read
  } else {
    bn = ctl->bn;
    rho_old = ctl->rho[0];
  }
  int k = k0 + 1;
  bool done = false;
  for (; k - k0 <= chunk; ++k) {
    cycle();
    const double beta = k >= 2 ? rho / rho_old : 0.0;
#pragma unroll
    for (int c = 0; c < C; ++c) {  // the last reads of va are behind the barrier of rho's sum
      p[c] = __builtin_fma(beta, p[c], z[c]);
      va[c * NT + tid] = p[c];
    }
    lds_barrier();
    rows(va, [&](int c, double s) { z[c] = __builtin_fma(d[c], p[c], s); });  // z holds q
    totals([&](int, int c) { return p[c] * z[c]; }, one);
    const double alpha = rho / one[0];
    lds_barrier();  // gs is read
#pragma unroll
    for (int c = 0; c < C; ++c) {
      xs[c * NT + tid] = __builtin_fma(alpha, p[c], xs[c * NT + tid]);
      r[c] = __builtin_fma(-alpha, z[c], r[c]);
    }
    totals([&](int, int c) { return r[c] * r[c]; }, one);
    const double rn = sqrt(one[0]);
    const bool conv = rn <= tol * bn;
    if (conv || k >= maxit) {
      done = true;
      if (tid == 0) {
        ctl->done = 1;
        ctl->iters = k;
        ctl->res = rn / bn;
        ctl->status = conv ? 0 : DIFVM_WARN_NOT_CONVERGED;
      }
      break;
    }
    rho_old = rho;
  }
#pragma unroll
  for (int c = 0; c < C; ++c)
    if (const int i = c * NT + tid; i < n) {
      x[i] = xs[i];
      if (!done) {
        rbuf[i] = r[c];
        pbuf[i] = p[c];
      }
    }
  if (!done && tid == 0) {
    ctl->next = k - 1;
    ctl->rho[0] = rho_old;
  }
}

// setup: row blockIdx.x of the n x n matrix M copied with leading dimension ld, zeros past its end
__global__ __launch_bounds__(BLOCK) void k_amg_pad(int n, int ld, const double* __restrict__ M, double* __restrict__ out) {
  for (int j = threadIdx.x; j < ld; j += BLOCK)
    out[(size_t)blockIdx.x * ld + j] = j < n ? M[(size_t)blockIdx.x * n + j] : 0.0;
}

// Setup: in-place Gauss-Jordan inversion of the dense SPD coarsest matrix M (row-major), one pivot k
// per pair of launches.  Without pivoting: the pivots of an SPD matrix are Schur-complement diagonals,
// all positive; a pivot that is not sets *bad.
//   for i, j != k:  m_ij <- m_ij - m_ik m_kj / p;   m_kj <- m_kj / p;   m_ik <- -m_ik / p;   m_kk <- 1 / p
// with p = m_kk; after the last pivot M holds M^-1.  Row and column k are copied first, so the update
// reads no entry it writes.
__global__ __launch_bounds__(BLOCK) void k_gj_save(int n, int k, const double* __restrict__ M, double* __restrict__ rowk,
                                                   double* __restrict__ colk, int* __restrict__ bad) {
  int i = blockIdx.x * BLOCK + threadIdx.x;
  if (i >= n) return;
  rowk[i] = M[(size_t)k * n + i];
  colk[i] = M[(size_t)i * n + k];
  if (i == k && !(M[(size_t)k * n + k] > 0.0)) *bad = 1;
}
__global__ __launch_bounds__(BLOCK) void k_gj_step(int n, int k, double* __restrict__ M, const double* __restrict__ rowk,
                                                   const double* __restrict__ colk) {
  size_t e = (size_t)blockIdx.x * BLOCK + threadIdx.x;
  if (e >= (size_t)n * n) return;
  int i = (int)(e / n), j = (int)(e % n);
  double p = rowk[k];
  double v;
  if (i == k) v = j == k ? 1.0 / p : rowk[j] / p;
  else if (j == k) v = -colk[i] / p;
  else v = M[e] - colk[i] * rowk[j] / p;
  M[e] = v;
}
// exact symmetry: m_ij and m_ji replaced by their mean
__global__ __launch_bounds__(BLOCK) void k_symmetrise(int n, double* __restrict__ M) {
  size_t e = (size_t)blockIdx.x * BLOCK + threadIdx.x;
  if (e >= (size_t)n * n) return;
  int i = (int)(e / n), j = (int)(e % n);
  if (j <= i) return;
  double m = 0.5 * (M[e] + M[(size_t)j * n + i]);
  M[e] = m;
  M[(size_t)j * n + i] = m;
}
__global__ void k_zero_int(int* p) {
  if (threadIdx.x == 0) *p = 0;
}

// M <- M^-1 for the dense SPD coarsest matrix (device, n x n); throws when a pivot is not positive
void dense_inverse_spd(const Ctx& c, int n, double* M, hipStream_t s) {
  double* rc = dalloc<double>(c, 2 * (size_t)n);
  int* bad = nullptr;
  int hbad = 0;
  try {
    bad = dalloc<int>(c, 1);
    k_zero_int<<<1, 64, 0, s>>>(bad);
    const int ge = (int)(((size_t)n * n + BLOCK - 1) / BLOCK);
    for (int k = 0; k < n; ++k) {
      k_gj_save<<<grid_for(n), BLOCK, 0, s>>>(n, k, M, rc, rc + n, bad);
      k_gj_step<<<ge, BLOCK, 0, s>>>(n, k, M, rc, rc + n);
    }
    k_symmetrise<<<ge, BLOCK, 0, s>>>(n, M);
    DIFVM_HIP(hipGetLastError());
    DIFVM_HIP(hipMemcpyAsync(&hbad, bad, sizeof(int), hipMemcpyDeviceToHost, s));
    DIFVM_HIP(hipStreamSynchronize(s));
  } catch (...) {
    dfree(c, rc);
    dfree(c, bad);
    throw;
  }
  dfree(c, rc);
  dfree(c, bad);
  DIFVM_CHECK(!hbad, DIFVM_ERR_UNSUPPORTED, "AMG setup: coarsest matrix is not positive definite");
}

// largest rows(1) x rows(2) of the fused passes' dense matrix (32 MB: it is read in every cycle; 162,000
// cells have 22 MB, 384,000 would have 110)
constexpr size_t FUSE_MAX_DENSE = size_t(4) << 20;
constexpr int FUSE_LANES = 16;  // per row of level 1: its S row has some 90 entries, H's some hundreds

#define DIFVM_AMG_LAUNCH(KERNEL, SW, N, S, ...)                                                           \
  KERNEL<SW, LATE><<<(int)(((size_t)(N) * (SW) + BLOCK - 1) / BLOCK), BLOCK, 0, S>>>(__VA_ARGS__)

#define DIFVM_AMG_MID_LAUNCH(KERNEL, SW, N, MORE, S, ...) \
  KERNEL<SW, LATE><<<((N) * SW + BLOCK - 1) / BLOCK + (MORE), BLOCK, 0, S>>>(__VA_ARGS__)
#define DIFVM_AMG_MID_DISPATCH(KERNEL, sw, N, MORE, S, ...)                     \
  switch (sw) {                                                                 \
    case 1: DIFVM_AMG_MID_LAUNCH(KERNEL, 1, N, MORE, S, __VA_ARGS__); break;    \
    case 2: DIFVM_AMG_MID_LAUNCH(KERNEL, 2, N, MORE, S, __VA_ARGS__); break;    \
    case 4: DIFVM_AMG_MID_LAUNCH(KERNEL, 4, N, MORE, S, __VA_ARGS__); break;    \
    case 8: DIFVM_AMG_MID_LAUNCH(KERNEL, 8, N, MORE, S, __VA_ARGS__); break;    \
    case 16: DIFVM_AMG_MID_LAUNCH(KERNEL, 16, N, MORE, S, __VA_ARGS__); break;  \
    case 32: DIFVM_AMG_MID_LAUNCH(KERNEL, 32, N, MORE, S, __VA_ARGS__); break;  \
    default: DIFVM_AMG_MID_LAUNCH(KERNEL, 64, N, MORE, S, __VA_ARGS__); break;  \
  }
#define DIFVM_AMG_DISPATCH(KERNEL, sw, N, S, ...)               \
  switch (sw) {                                                 \
    case 1: DIFVM_AMG_LAUNCH(KERNEL, 1, N, S, __VA_ARGS__); break;   \
    case 2: DIFVM_AMG_LAUNCH(KERNEL, 2, N, S, __VA_ARGS__); break;   \
    case 4: DIFVM_AMG_LAUNCH(KERNEL, 4, N, S, __VA_ARGS__); break;   \
    case 8: DIFVM_AMG_LAUNCH(KERNEL, 8, N, S, __VA_ARGS__); break;   \
    case 16: DIFVM_AMG_LAUNCH(KERNEL, 16, N, S, __VA_ARGS__); break; \
    case 32: DIFVM_AMG_LAUNCH(KERNEL, 32, N, S, __VA_ARGS__); break; \
    default: DIFVM_AMG_LAUNCH(KERNEL, 64, N, S, __VA_ARGS__); break; \
  }

}  // namespace

// the transfers of a two-level hierarchy of a small mesh as k_amg_pcg_block reads them
static AmgBlock amg_block(AmgDev* a, const AmgHierarchy& H, hipStream_t s) {
  const difvm_mesh* m = a->mesh;
  const int uw = m->d.uw, n = m->d.nc, n2 = a->rows[1];
  AmgBlock B;
  if (m->d.nseg != 1 || m->d.ntile > SEG_TILES || !m->d.slot_off16 || (uw != 3 && uw != 4) || n2 > BLOCK_COARSE) return B;
  const AmgCsr &P = H.levels[0].P, &R = H.levels[0].R;
  constexpr int ROWS = SEG_TILES * TILE;
  std::vector<ushort4> pcol(ROWS, ushort4{0, 0, 0, 0}), rcol;
  std::vector<double2> pval(2 * ROWS, double2{0.0, 0.0}), rval;
  auto put = [](ushort4& col, double2& v0, double2& v1, int k, int c, double v) {
    (k == 0 ? col.x : k == 1 ? col.y : k == 2 ? col.z : col.w) = (uint16_t)c;
    (k == 0 ? v0.x : k == 1 ? v0.y : k == 2 ? v1.x : v1.y) = v;
  };
  std::vector<int32_t> lrow, lptr = {0}, lcol;
  std::vector<double> lval;
  const Drain drain{s};
  for (int i = 0; i < n; ++i) {
    const int q4 = std::min(P.ptr[i + 1], P.ptr[i] + 4);
    for (int q = P.ptr[i]; q < q4; ++q) put(pcol[i], pval[i], pval[ROWS + i], q - P.ptr[i], P.col[q], P.val[q]);
    if (q4 == P.ptr[i + 1]) continue;
    lrow.push_back(i);
    lcol.insert(lcol.end(), P.col.begin() + q4, P.col.begin() + P.ptr[i + 1]);
    lval.insert(lval.end(), P.val.begin() + q4, P.val.begin() + P.ptr[i + 1]);
    lptr.push_back((int32_t)lcol.size());
  }
  B.nlong = (int)lrow.size();
  if (B.nlong) {
    B.lrow = up(a, lrow, s);
    B.lptr = up(a, lptr, s);
    B.lcol = up(a, lcol, s);
    B.lval = up(a, lval, s);
  }
  constexpr int PER = 4 * BLOCK_R_LANES;
  for (int ps = 0; ps < BLOCK_R_PASSES; ++ps) {
    int most = 0;
    for (int I = ps * BLOCK_R_ROWS; I < std::min((ps + 1) * BLOCK_R_ROWS, n2); ++I)
      most = std::max(most, (R.ptr[I + 1] - R.ptr[I] + PER - 1) / PER);
    B.first[ps + 1] = B.first[ps] + (most + BLOCK_R_FOURS - 1) / BLOCK_R_FOURS * BLOCK_R_FOURS;
  }
  rcol.assign((size_t)B.first[BLOCK_R_PASSES] * BLOCK_NT, ushort4{0, 0, 0, 0});
  rval.assign(2 * rcol.size(), double2{0.0, 0.0});
  for (int I = 0; I < n2; ++I)
    for (int q = R.ptr[I]; q < R.ptr[I + 1]; ++q) {
      const int k = q - R.ptr[I], t = I % BLOCK_R_ROWS * BLOCK_R_LANES + k / 4 % BLOCK_R_LANES;
      const size_t e = B.first[I / BLOCK_R_ROWS] + k / PER;
      put(rcol[e * BLOCK_NT + t], rval[2 * e * BLOCK_NT + t], rval[(2 * e + 1) * BLOCK_NT + t], k % 4, R.col[q], R.val[q]);
    }
  B.pcol = up(a, pcol, s);
  B.pval = up(a, pval, s);
  B.rcol = up(a, rcol, s);
  B.rval = up(a, rval, s);
  B.ld = (n2 + 15) & ~15;
  double* inv = work(a, (size_t)n2 * B.ld);
  k_amg_pad<<<n2, BLOCK, 0, s>>>(n2, B.ld, a->cinv, inv);
  DIFVM_HIP(hipGetLastError());
  B.inv = reinterpret_cast<double2*>(inv);
  B.c = cheb_coefficients(0.1 * a->hi[0], a->hi[0]);
  B.n2 = n2;
  return B;
}

// cells per thread of the copy of K to CSR (a cell takes about 50 ns, starting a thread 20 us)
constexpr int CSR_ROWS = 8192;

AmgDev* amg_create(difvm_mesh* m, SellMatrix K, const AmgOptions& opt) {
  const DMesh& d = m->d;
  const HostLayout& L = m->host;
  hipStream_t s = stream_of(m);
  std::vector<double> diag(d.nc), val(d.nslot);
  DIFVM_HIP(hipMemcpyAsync(diag.data(), K.diag, sizeof(double) * d.nc, hipMemcpyDeviceToHost, s));
  DIFVM_HIP(hipMemcpyAsync(val.data(), K.val, sizeof(double) * d.nslot, hipMemcpyDeviceToHost, s));
  DIFVM_HIP(hipStreamSynchronize(s));
  // cell-slot rows -> CSR (internal faces only; columns ascending)
  AmgCsr A0;
  A0.n = d.nc;
  A0.ptr.assign(d.nc + 1, 0);
  A0.diag = diag;
  auto each_slot = [&](int i, auto&& f) {
    int sl = i >> 6, base = L.slice_start[sl] + (i & (SLICE - 1));
    int width = (L.slice_start[sl + 1] - L.slice_start[sl]) >> 6;
    for (int k = 0; k < width; ++k) {
      int at = base + k * SLICE;
      int sf = L.slot_face[at];
      if (sf != SLOT_PAD && sf < d.nfi) f(at);
    }
  };
  parallel_rows(d.nc, CSR_ROWS, [&](int, int a, int b) {
    for (int i = a; i < b; ++i) each_slot(i, [&](int) { ++A0.ptr[i + 1]; });
  });
  for (int i = 0; i < d.nc; ++i) A0.ptr[i + 1] += A0.ptr[i];
  A0.col.resize(A0.ptr[d.nc]);
  A0.val.resize(A0.ptr[d.nc]);
  parallel_rows(d.nc, CSR_ROWS, [&](int, int a, int b) {
    std::vector<std::pair<int32_t, double>> row;
    for (int i = a; i < b; ++i) {
      row.clear();
      each_slot(i, [&](int at) { row.push_back({L.slot_col[at], val[at]}); });
      std::sort(row.begin(), row.end());
      int q = A0.ptr[i];
      for (auto& e : row) {
        A0.col[q] = e.first;
        A0.val[q++] = e.second;
      }
    }
  });
  for (int i = 0; i < d.nc; ++i)
    DIFVM_CHECK(diag[i] > 0.0, DIFVM_ERR_INVALID_ARG, "AMG needs a matrix with a positive diagonal");
  AmgHierarchy H;
  try {
    amg_build(A0, opt, H);
  } catch (const AmgError& e) {
    throw Error{DIFVM_ERR_UNSUPPORTED, "AMG setup: " + e.msg};
  }
  AmgDev* a = new AmgDev();
  try {
    a->mesh = m;
    a->L = (int)H.levels.size();
    int L_ = a->L;
    a->A.resize(L_ + 1);
    a->R.resize(L_);
    a->AP.resize(L_);
    a->b.assign(L_ + 1, nullptr);
    a->bd.assign(L_ + 1, nullptr);
    a->res.assign(L_ + 1, nullptr);
    a->x.assign(L_ + 1, nullptr);
    a->rows.push_back(d.nc);
    a->P0 = upload_csr(a, H.levels[0].P, false, s);
    for (int l = 0; l < L_; ++l) {
      const bool mid = l > 0 && l == L_ - 1;
      if (l > 0 && !mid) {
        a->AP[l] = upload_csr(a, H.levels[l].AP, false, s, 1);
        a->AP[l].val2 = up(a, H.levels[l].P_on_AP, s);
      }
      if (!mid) a->R[l] = upload_csr(a, H.levels[l].R, false, s);
      a->A[l + 1] = upload_csr(a, H.coarse[l], true, s);
      a->rows.push_back(H.coarse[l].n);
    }
    // Gershgorin: the eigenvalues of D^-1 K lie in the discs around 1 of radius sum_j |k_ij| / k_ii.
    // At least 2, the bound of every weakly diagonally dominant K (the pressure operators), so that it
    // holds for the later operators of the same kind the preconditioner is applied with.
    double g = 2.0;
    for (int i = 0; i < d.nc; ++i) {
      double off = 0.0;
      for (int q = A0.ptr[i]; q < A0.ptr[i + 1]; ++q) off += std::fabs(A0.val[q]);
      g = std::max(g, 1.0 + off / diag[i]);
    }
    a->hi.push_back(g);
    for (int l = 1; l < L_; ++l) a->hi.push_back(H.levels[l].hi);
    for (int l = 0; l <= L_; ++l) {
      size_t n = a->rows[l];
      a->res[l] = work(a, n);
      if (l < L_) {
        a->xs.push_back(l ? work(a, n) : nullptr);
        a->t.push_back(l && l < L_ - 1 ? work(a, n) : nullptr);
        a->d0.push_back(l && l < L_ - 1 ? work(a, n) : nullptr);
      }
      if (l > 0) {
        a->b[l] = work(a, n);
        a->x[l] = work(a, n);
        if (l < L_) a->bd[l] = work(a, n);
      }
    }
    DIFVM_CHECK(H.n_coarsest <= MAX_DENSE, DIFVM_ERR_UNSUPPORTED, "coarsest AMG level too large");
    a->cinv = up(a, H.coarsest_dense, s);
    dense_inverse_spd(ctx_of(m), H.n_coarsest, a->cinv, s);
    if (L_ == 1) a->block = amg_block(a, H, s);
    AmgFused F;
    const Drain drain{s};
    if (L_ >= 2) {
      const bool two = L_ == 2 && fine_spans(m) && (size_t)a->rows[1] * a->rows[2] <= FUSE_MAX_DENSE;
      F = amg_fuse(H, two);
      a->alpha = F.alpha;
      a->beta = F.beta;
      a->G = upload_csr(a, F.G, false, s);
      a->G.sw = lanes_for(F.G.n, F.G.col.size() + H.coarse[L_ - 2].col.size(), 4);
      if (two) {
        a->S = upload_csr(a, F.S, false, s);
        a->RS = upload_csr(a, F.RS, false, s);
        a->H = work(a, (size_t)a->rows[1] * a->rows[2]);
        k_amg_h<<<a->rows[1], BLOCK, 0, s>>>(a->rows[2], a->G.ptr, a->G.col, a->G.val, a->cinv, a->H);
        DIFVM_HIP(hipGetLastError());
      } else {
        a->GT = upload_csr(a, F.GT, false, s);
      }
    }
    DIFVM_HIP(hipStreamSynchronize(s));
  } catch (...) {
    amg_free(a);
    throw;
  }
  return a;
}

void amg_free(AmgDev* a) {
  if (!a) return;
  if (a->mesh) (void)hipStreamSynchronize(stream_of(a->mesh));
  for (void* p : a->allocs) dfree(ctx_of(a->mesh), p);
  delete a;
}

int amg_levels(const AmgDev* a, int* rows, int cap) {
  int n = (int)a->rows.size();
  for (int l = 0; l < n && l < cap; ++l) rows[l] = a->rows[l];
  return n;
}

double amg_vcycle_bytes(const AmgDev* a) {
  const difvm_mesh* m = a->mesh;
  const int L = a->L;
  auto rows = [&](int l) { return (double)a->rows[l]; };
  auto csr = [](const DevCsr& M, bool diag, int val_words) {
    return 4.0 * (M.n + 1) + (4.0 + 8.0 * val_words) * M.nnz + (diag ? 8.0 * M.n : 0.0);
  };
  const double n0 = m->d.nc;
  const double K = 8.0 * n0 + 16.0 * m->d.nfi;  // LDU: diagonal; owner, neighbour, coefficient per face
  double b = 0.0;
  b += K + 16.0 * n0;  // first pre-smoothing pass: r -> xs
  b += K + 24.0 * n0;  // second: r, xs -> res
  for (int l = 0; l < L; ++l) {
    if (l > 0 && a->S.n) {
      b += csr(a->A[1], true, 1) + csr(a->S, false, 1) + csr(a->RS, false, 1) + 24.0 * rows(1) + 8.0 * rows(2);
      b += csr(a->A[1], true, 1) + 8.0 * rows(1) * rows(2) + 24.0 * rows(1) + 8.0 * rows(2);  // xs, resd, b_2 -> x
      break;
    }
    if (l > 0) {
      b += csr(a->A[l], true, 1) + 16.0 * rows(l);  // bd -> xs
      b += csr(a->A[l], true, 1) + 24.0 * rows(l);  // b, xs -> res
    }
    if (l > 0 && l == L - 1) {
      b += csr(a->GT, false, 1) + 8.0 * rows(l) + 8.0 * rows(L);  // b -> b_L
    } else {
      bool coarsest = l + 1 == L;
      b += csr(a->R[l], false, 1) + 8.0 * rows(l) + (coarsest ? 8.0 : 24.0) * rows(l + 1);  // res -> b (, D^-1 b)
    }
  }
  if (!a->S.n) b += 8.0 * rows(L) * rows(L) + 16.0 * rows(L);  // dense solve
  if (L >= 2 && !a->S.n)
    b += csr(a->A[L - 1], true, 1) + csr(a->G, false, 1) + 24.0 * rows(L - 1) + 8.0 * rows(L);  // xs, res, x_L -> x
  for (int l = L - 2; l >= 1; --l) {
    b += csr(a->AP[l], true, 2) + 32.0 * rows(l) + 8.0 * rows(l + 1);  // xs, res, x_c -> t, d0
    b += csr(a->A[l], true, 1) + 24.0 * rows(l);                       // t, d0 -> x
  }
  b += csr(a->P0, false, 1) + 16.0 * n0 + 8.0 * rows(1);  // xs, x_1 -> t
  b += K + 24.0 * n0;                                     // r, t -> d0
  b += K + 32.0 * n0;                                     // r, t, d0 -> z
  return b;
}

template <bool LATE>
static void launch_vcycle(const AmgDev* a, hipStream_t s, SellMatrix Km, const double* r, double* z, double* part,
                          StopFlags ctl, CycleTest test, const CgStep* step, double* res) {
  difvm_mesh* m = a->mesh;
  SellView K = sview(m, Km);
  const int L = a->L, nc = m->d.nc;
  std::vector<Cheb> c(L);
  for (int l = 0; l < L; ++l) c[l] = cheb_coefficients(0.1 * a->hi[l], a->hi[l]);
  const Tiles T = tiles_of(m);
  const int G = grid_for(nc);
  // xs and t of the finest level live in z, d0 in res, and res in a vector that the caller has free (q): at 1,053,696
  // cells an iteration touches the matrix and the hierarchy, 183 MB, and six vectors of 8.4 instead of ten, 233 MB
  // instead of 267, which fits the 256 MB cache (141 to 129 us per iteration; up to 900,000 cells no difference)
  // down
  const CycleTest none{};
  if (step)
    (K.off16 ? k_amg_step_pre1<true> : k_amg_step_pre1<false>)<<<n_spans(m), QUARTER, 0, s>>>(
        K, T, *step, z, test.rr, test.k, c[0], test.ctl);
  else
    (K.off16 ? k_amg_cheb_pre1<true, LATE> : k_amg_cheb_pre1<false, LATE>)<<<G + test.blocks, BLOCK, 0, s>>>(
        K, T, test, r, z, c[0], ctl);
  // after the joint kernel the test is here: it needs every block's partials of r.r
  const CycleTest& t2 = step ? test : none;
  (K.off16 ? k_amg_cheb_pre2<true, LATE> : k_amg_cheb_pre2<false, LATE>)<<<G + t2.blocks, BLOCK, 0, s>>>(
      K, T, t2, r, z, res, ctl);
  for (int l = 0; l < L; ++l) {
    if (l > 0) {
      const DevCsr& A = a->A[l];
      if (a->S.n) {  // and the coarsest
        const DevCsr &S = a->S, &Q = a->RS;
        const int blocks = (S.n * FUSE_LANES + BLOCK - 1) / BLOCK + (Q.n + BLOCK / 64 - 1) / (BLOCK / 64);
        k_amg_down1<FUSE_LANES, LATE><<<blocks, BLOCK, 0, s>>>(A.n, A.ptr, A.col, A.val, A.diag, S.ptr, S.col, S.val, Q.n,
                                                               Q.ptr, Q.col, Q.val, a->alpha, a->beta, a->bd[1],
                                                               a->xs[1], a->res[1], a->b[2], ctl);
        break;
      }
      if (l == L - 1) {  // and the coarsest
        const DevCsr& GT = a->GT;
        const int n2 = GT.n;
        DIFVM_AMG_MID_DISPATCH(k_amg_mid1, A.sw, A.n, (n2 + BLOCK / 64 - 1) / (BLOCK / 64), s, A.n, A.ptr, A.col, A.val,
                               A.diag, a->bd[l], a->xs[l], a->alpha, a->beta, n2, GT.ptr, GT.col, GT.val, a->b[l],
                               a->b[L], ctl);
        DIFVM_AMG_MID_DISPATCH(k_amg_mid2, A.sw, A.n, n2, s, A.n, A.ptr, A.col, A.val, A.diag, a->b[l], a->xs[l],
                               a->res[l], n2, a->cinv, a->b[L], a->x[L], ctl);
        break;
      }
      DIFVM_AMG_DISPATCH(k_amg_cpre1, A.sw, A.n, s, A.n, A.ptr, A.col, A.val, A.diag, a->bd[l], a->xs[l], c[l], ctl);
      DIFVM_AMG_DISPATCH(k_amg_cpre2, A.sw, A.n, s, A.n, A.ptr, A.col, A.val, A.diag, a->b[l], a->xs[l], a->res[l],
                         ctl);
    }
    const DevCsr& R = a->R[l];
    const double* dc = l + 1 < L ? a->A[l + 1].diag : nullptr;  // the coarsest level needs no D^-1 b
    DIFVM_AMG_DISPATCH(k_amg_restrict, R.sw, R.n, s, R.n, R.ptr, R.col, R.val, l ? a->res[l] : res, dc, a->b[l + 1],
                       a->bd[l + 1], ctl);
  }
  // up
  if (L == 1) {
    k_amg_coarsest<LATE><<<a->rows[L], BLOCK, 0, s>>>(a->rows[L], a->cinv, a->b[L], a->x[L], ctl);
  } else if (a->S.n) {
    const DevCsr& A = a->A[1];
    k_amg_up1<FUSE_LANES, LATE><<<(A.n * FUSE_LANES + BLOCK - 1) / BLOCK, BLOCK, 0, s>>>(
        A.n, A.ptr, A.col, A.val, A.diag, a->rows[2], a->H, a->alpha, a->beta, a->xs[1], a->res[1], a->b[2], a->x[1], ctl);
  } else {
    const int l = L - 1;
    const DevCsr &A = a->A[l], &Q = a->G;
    DIFVM_AMG_DISPATCH(k_amg_up, Q.sw, A.n, s, A.n, A.ptr, A.col, A.val, A.diag, Q.ptr, Q.col, Q.val, a->alpha, a->beta,
                       a->xs[l], a->res[l], a->x[L], a->x[l], ctl);
  }
  for (int l = L - 2; l >= 1; --l) {
    const DevCsr& Q = a->AP[l];
    const DevCsr& A = a->A[l];
    DIFVM_AMG_DISPATCH(k_amg_cup1, Q.sw, Q.n, s, Q.n, Q.ptr, Q.col, Q.val, Q.val2, A.diag, a->xs[l], a->res[l],
                       a->x[l + 1], a->t[l], a->d0[l], c[l], ctl);
    DIFVM_AMG_DISPATCH(k_amg_cup2, A.sw, A.n, s, A.n, A.ptr, A.col, A.val, A.diag, a->t[l], a->d0[l], a->x[l], c[l],
                       ctl);
  }
  k_amg_prolong<LATE><<<G, BLOCK, 0, s>>>(nc, a->P0.ptr, a->P0.col, a->P0.val, a->x[1], z, ctl);
  (K.off16 ? k_amg_cheb_post1<true, LATE> : k_amg_cheb_post1<false, LATE>)<<<G, BLOCK, 0, s>>>(K, r, z, res, c[0],
                                                                                               ctl);
  (K.off16 ? k_amg_cheb_post2<true, LATE> : k_amg_cheb_post2<false, LATE>)<<<n_spans(m), LATE ? QUARTER : TILE, 0, s>>>(
      K, T, r, res, z, part, c[0], ctl);
  DIFVM_HIP(hipGetLastError());
}

bool amg_pcg_in_block(const AmgDev* a) { return a->block.n2 > 0; }

template <int W>
static auto block_kernel(int ntile) {
  return ntile == 1 ? k_amg_pcg_block<2, W>
         : ntile == 2 ? k_amg_pcg_block<4, W>
         : ntile == 3 ? k_amg_pcg_block<6, W>
                      : k_amg_pcg_block<8, W>;
}

void amg_pcg_block(const AmgDev* a, SellMatrix Km, const double* b, double* x, double* r, double* p, double tol,
                   int maxit, int chunk, bool first, PcgCtl* ctl) {
  const difvm_mesh* m = a->mesh;
  const SellView K = sview(m, Km);
  auto kernel = K.uw == 4 ? block_kernel<4>(m->d.ntile) : block_kernel<3>(m->d.ntile);
  kernel<<<1, BLOCK_NT, 0, stream_of(m)>>>(K, m->d.ntile, a->block, b, x, r, p, tol, maxit, chunk, first, ctl);
  DIFVM_HIP(hipGetLastError());
}

void amg_vcycle(const AmgDev* a, SellMatrix Km, const double* r, double* z, double* part, PcgCtl* ctls,
                double* rr, int k, const CgStep* step, double* res) {
  difvm_mesh* m = a->mesh;
  const int nseg = m->d.nseg;
  const CycleTest test{ctls, rr, k, nseg, rr ? std::min(64, (nseg + 7) & ~7) : 0};
  // queued kernel by kernel on the solve's stream (inside a captured step they join that graph): the
  // host queues a cycle in well under one iteration's GPU time, and a replayed graph of the cycle
  // cost about 9 us of idle GPU between its end and the next kernel on the stream
  (fine_spans(m) ? launch_vcycle<true> : launch_vcycle<false>)(a, ctx_of(m).stream, Km, r, z, part, StopFlags{ctls, nseg},
                                                               test, step, res ? res : a->res[0]);
}

}  // namespace difvm
