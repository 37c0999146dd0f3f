// Krylov solvers of libdifvm on the cell-slot matrix: Jacobi-preconditioned CG (pressure) and
// right-Jacobi BiCGStab (momentum, up to three systems sharing one matrix).  Paper Sec. "Numerical
// schemes and linear solvers": CG for the symmetric pressure system, BiCGStab for momentum.
//
// Every dot product is reduced deterministically (per-tile partials re-summed in a fixed order by the
// next kernel).  The scalars live in device memory and every kernel checks the solver's "done" flag
// first, so iterations queued after convergence are no-ops and the iterate is exactly the one at
// which the stopping test first held; the host reads the flag only once per block of iterations.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "amg_dev.h"
#include "device.h"
#include "krylov_util.h"
#include "ops.h"

// One arithmetic for every form of a solver (by tile, by quarter, a segment per block): products and sums
// are fused where an fma is written and nowhere else.
#pragma clang fp contract(off)

namespace difvm {

// BiCGStab state of one segment (up to three systems sharing its matrix) during one iteration
struct BiState {
  double tol;
  double bn[3], rho[3], alpha[3], omega[3], res[3], sres[3];  // rho = rhat.r entering the iteration
  int maxit, any;
  int iters[3], active[3], so[3], status[3];
  int next[3], pad;  // iteration that a further launch of k_bi_segment starts with
};
// outcome of the test on s (BiState::so)
enum { BI_SO_GO = 0, BI_SO_DONE = 1, BI_SO_BREAKDOWN = 2 };

struct KrylovWork {
  int nc = 0, ntile = 0;
  double *r = nullptr, *p = nullptr, *q = nullptr, *rh = nullptr, *v = nullptr, *z = nullptr,
         *t = nullptr;
  double* colscaled = nullptr;   // [n_slots] off-diagonals of A D^-1 (BiCGStab)
  double* partials = nullptr;
  struct PcgCtl* pcg = nullptr;  // [nseg]
  BiState* bi = nullptr;         // [2][nseg], by the parity of the iteration
  void* host_state[2] = {nullptr, nullptr};  // pinned mirrors of the solver states (two polls in flight)
  hipEvent_t poll_ev[2] = {nullptr, nullptr};
  const Ctx* ctx = nullptr;  // allocator of the buffers above
};

KrylovWork* krylov_work(difvm_mesh* m) { return m->krylov; }

void krylov_work_free(KrylovWork* w);

static KrylovWork* make_work(difvm_mesh* m) {
  if (m->krylov) return m->krylov;
  KrylovWork* w = new KrylovWork();
  try {
    int nc = m->d.nc;
    w->nc = nc;
    w->ntile = m->d.ntile;  // reduction tiles over all segments (at least ceil(nc / 1024))
    size_t n3 = (size_t)nc * 3;
    const Ctx& c = ctx_of(m);
    w->ctx = &c;
    w->r = dalloc<double>(c, n3); w->p = dalloc<double>(c, n3); w->q = dalloc<double>(c, n3);
    w->rh = dalloc<double>(c, n3); w->v = dalloc<double>(c, n3);
    w->z = dalloc<double>(c, n3); w->t = dalloc<double>(c, n3);
    w->colscaled = dalloc<double>(c, m->d.nslot);
    const int nseg = m->d.nseg;
    // values per span: PCG uses 6, BiCGStab 6 + 3 + 9 and as many totals per segment
    w->partials = dalloc<double>(c, (size_t)18 * (n_spans(m) + nseg));
    w->pcg = static_cast<PcgCtl*>(dmalloc(c, sizeof(BiState) * nseg));  // PcgCtl is smaller (asserted below)
    w->bi = dalloc<BiState>(c, 2 * (size_t)nseg);
    for (int q = 0; q < 2; ++q) {
      DIFVM_HIP(hipHostMalloc((void**)&w->host_state[q], sizeof(BiState) * nseg, hipHostMallocDefault));
      DIFVM_HIP(hipEventCreateWithFlags(&w->poll_ev[q], hipEventDisableTiming));
    }
  } catch (...) {
    krylov_work_free(w);
    throw;
  }
  m->krylov = w;
  return w;
}

void krylov_work_free(KrylovWork* w) {
  if (!w) return;
  if (w->ctx) {
    const Ctx& c = *w->ctx;
    for (double* a : {w->r, w->p, w->q, w->rh, w->v, w->z, w->t, w->colscaled, w->partials}) dfree(c, a);
    dfree(c, w->pcg);
    dfree(c, w->bi);
  }
  for (int q = 0; q < 2; ++q) {
    if (w->host_state[q]) (void)hipHostFree(w->host_state[q]);
    if (w->poll_ev[q]) (void)hipEventDestroy(w->poll_ev[q]);
  }
  delete w;
}

// ---------------------------------------------------------------------------------------------
// matrix helpers (SellView: krylov_util.h)
// ---------------------------------------------------------------------------------------------
// Slot values from face values, the rows that fill the last slice included (their slots are padding: zeros), so
// that no clearing pass is needed; a row's first four slots in flight together (one at a time before).  Clearing pass
// and this kernel -> this: 1,053,696 cells 33.8 -> 15.2 us, 162,000 9.5 -> 4.4.
__global__ __launch_bounds__(BLOCK) void k_sell_from_ldu(int rows, int nfi, const int32_t* __restrict__ slice_start, int uw,
                                                         const int32_t* __restrict__ slot_face, const double* __restrict__ up,
                                                         const double* __restrict__ lo, double* __restrict__ val) {
  int i = xcd_tile(blockIdx.x, gridDim.x) * BLOCK + threadIdx.x;
  if (i >= rows) return;
  SlotRange R = slots_of(slice_start, uw, i);
  walk_row<4>(R.width, [&](auto Wc, int k0) {
    constexpr int N = decltype(Wc)::value;
    int sf[N];
    double a[N];
#pragma unroll
    for (int k = 0; k < N; ++k) sf[k] = slot_face[R.base + (k0 + k) * SLICE];
#pragma unroll
    for (int k = 0; k < N; ++k) a[k] = (sf[k] < 0 ? lo : up)[slot_face_index(sf[k], nfi)];  // others read entry 0
#pragma unroll
    for (int k = 0; k < N; ++k) val[R.base + (k0 + k) * SLICE] = slot_internal(sf[k], nfi) ? a[k] : 0.0;
  });
}

void sell_from_ldu(const difvm_mesh* m, const double* upper, const double* lower, double* val) {
  const DMesh& d = m->d;
  if (!lower) lower = upper;
  if (d.nfi == 0) upper = lower = val;  // the caller may pass NULL; entry 0 is read and not used
  const int rows = d.nslice * SLICE;
  if (d.nslot == 0) return;
  k_sell_from_ldu<<<grid_for(rows), BLOCK, 0, stream_of(m)>>>(rows, d.nfi, d.slice_start, d.uw, d.slot_face, upper, lower,
                                                              val);
  DIFVM_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------------------------
// PCG: two kernels per iteration and no memory fences.
//
// Partials of each kernel are re-summed (per segment, fixed order) at the start of the NEXT kernel
// in every block, so no tile waits for another and no L2 write-back is needed.  The direction update
// p_k = z_{k-1} + beta p_{k-1} is fused into the product q = A p_k: each cell forms its own and its
// neighbours' p_k from z and p_{k-1} (separate arrays, so every store writes whole cache lines);
// p and the published rho_k = r_k.z_k are double-buffered by parity.
//   init1:  r = b - A x                               partials (b.b, r.r)
//   init2:  stopping test at k = 0; z0 = r/d; p0 = 0  partials B = (r.r, r.z)
//   spmv_k: rho_{k-1} and the stopping test of iterate k-1 (from B), beta; p_k; q = A p_k
//                                                     partials A = (p.q); first tile publishes rho
//   upd_k:  alpha = rho_{k-1}/(p.q); x += alpha p; r -= alpha q; z = r/d   partials B
// The segment's first tile records iterations / residual / status; its kernels return at once
// after its stop.  Large meshes: the product runs 512 threads x 2 cells per 1024-cell tile, the update
// 256 x 4 (measured best on gfx950 for these two memory patterns); the first four slots of a row are
// unrolled so their loads are in flight together.
//
// Up to FINE_TILES tiles a block takes a quarter of a tile (see Span), a thread a cell, and every load that
// does not wait for the scalars (row, neighbours' z and p, own values) is issued before the partials are
// summed: there a kernel's time is its chain of dependent loads, while at 1,029 tiles the registers of the
// loads in flight halve the resident blocks (25.6 us and more for the product against 19.8).  Jacobi-CG per
// iteration at 93,750 cells: 12.7 us with blocks of a tile, 9.0 now (product 7.2 to 5.0 us).
//
// Meshes whose segments have at most SEG_TILES tiles do not come here at all: see k_pcg_segment.  The
// arithmetic of an iteration is the same in every form, operation by operation (written with explicit fma,
// reduced in one order), so a member of a batch has its bits whichever form its neighbours bring about.
// ---------------------------------------------------------------------------------------------
static_assert(sizeof(PcgCtl) <= sizeof(BiState), "PCG states share the BiState-sized allocation");

constexpr int PCG_SPMV_NT = 512;  // threads per block of the product kernel (TILE / NT cells each)

__device__ __forceinline__ double cg_dir(double z, double beta, double p) { return __builtin_fma(beta, p, z); }

template <bool FINE>
__global__ __launch_bounds__(FINE ? QUARTER : TILE) void k_pcg_init1(SellView A, Tiles T, const double* __restrict__ b,
                                                                     const double* __restrict__ x,
                                                                     double* __restrict__ r,
                                                                     double* __restrict__ part) {
  const Span ti = span_of<FINE>(T);
  const int i = ti.lo + (int)threadIdx.x;
  double v[2] = {0.0, 0.0};
  if (i < ti.hi) {
    const double bi = b[i];
    double ax = A.diag[i] * x[i];
    SlotRange R = slots_of(A, i);
    const bool off16 = A.off16 != nullptr;  // the same for every thread: a uniform branch
    walk_row<4>(row_len(A, i, R), [&](auto Wc, int k0) {
      constexpr int N = decltype(Wc)::value;
      double a[N], xj[N];
      int j[N];
#pragma unroll
      for (int k = 0; k < N; ++k) {
        int at = R.base + (k0 + k) * SLICE;
        a[k] = A.val[at];
        j[k] = off16 ? i + A.off16[at] : A.col[at];
      }
#pragma unroll
      for (int k = 0; k < N; ++k) xj[k] = x[j[k]];
#pragma unroll
      for (int k = 0; k < N; ++k) ax = __builtin_fma(a[k], xj[k], ax);
    });
    const double ri = bi - ax;
    r[i] = ri;
    v[0] = bi * bi;
    v[1] = ri * ri;
  }
  put_partial<2, FINE ? QUARTER : TILE, FINE>(v, part, T.ntile, ti);
}

// JAC: Jacobi preconditioner (z = r/d here); otherwise z and the r.z partials come from the V-cycle
// that follows, and this kernel stores only the r.r partials
template <bool JAC, bool FINE>
__global__ __launch_bounds__(FINE ? QUARTER : TILE) void k_pcg_init2(
    SellView A, Tiles T, double* __restrict__ x, const double* __restrict__ r, double* __restrict__ z,
    double* __restrict__ p0, const double* __restrict__ part_in, double* __restrict__ partB, PcgCtl* ctls) {
  constexpr int NT = FINE ? QUARTER : TILE;
  const Span ti = span_of<FINE>(T);
  PcgCtl* ctl = ctls + ti.s;
  const int i = ti.lo + (int)threadIdx.x, ii = min(i, ti.end - 1);
  const double ri = r[ii], di = JAC ? A.diag[ii] : 1.0, tol = ctl->tol;
  double s[2];
  seg_totals<2, NT, FINE>(part_in, T.ntile, seg_first(T, ti.s), seg_count(T, ti.s), s);
  double bn = sqrt(s[0]), rn = sqrt(s[1]);
  bool zero_b = bn == 0.0;
  bool stop = zero_b || rn <= tol * bn;
  if (ti.t == seg_first(T, ti.s) && ti.j == 0 && threadIdx.x == 0) {
    ctl->bn = bn;
    ctl->res = zero_b ? 0.0 : rn / bn;
    ctl->iters = 0;
    ctl->status = 0;
    ctl->done = stop ? 1 : 0;
  }
  if (zero_b && i < ti.hi) x[i] = 0.0;
  if (stop) return;
  if (i < ti.hi) p0[i] = 0.0;  // p_1 = z_0 + 0 * p_0
  if constexpr (JAC) {
    const double zi = ri / di;
    if (i < ti.hi) z[i] = zi;
    double v[2] = {i < ti.hi ? ri * ri : 0.0, i < ti.hi ? ri * zi : 0.0};
    put_partial<2, NT, FINE>(v, partB, T.ntile, ti);
  } else {
    double v[1] = {i < ti.hi ? ri * ri : 0.0};
    put_partial<1, NT, FINE>(v, partB, T.ntile, ti);
  }
}

// (A (z + beta p))_i added to acc, with the loads of the row's first m <= W slots issued together
// OFF16: columns read as 16-bit offsets from the row (half the index bytes of the 32-bit columns)
template <int W, bool OFF16>
struct CgRow {
  double a[W], zj[W], pj[W];
  __device__ __forceinline__ void load(const SellView& A, int i, int base, const double* __restrict__ z,
                                       const double* __restrict__ pp, int m = W) {
    int j[W];
#pragma unroll
    for (int sl = 0; sl < W; ++sl) {
      const int at = base + (sl < m ? sl : 0) * SLICE;  // past m the first slot again, not added
      a[sl] = A.val[at];
      if constexpr (OFF16) j[sl] = i + A.off16[at];
      else j[sl] = A.col[at];
    }
#pragma unroll
    for (int sl = 0; sl < W; ++sl) {
      zj[sl] = z[j[sl]];
      pj[sl] = pp[j[sl]];
    }
  }
  __device__ __forceinline__ double add(double acc, double beta, int m = W) const {
#pragma unroll
    for (int sl = 0; sl < W; ++sl)
      if (sl < m) acc = __builtin_fma(a[sl], cg_dir(zj[sl], beta, pj[sl]), acc);
    return acc;
  }
};

// Tiles of this block: one tile per block when the grid has one block per tile (XCD-aware order),
// otherwise (a grid of G < ntile blocks, G a multiple of 8) block b walks tiles lo + b/8, lo + b/8 +
// G/8, ... of the contiguous eighth of the tiles that its XCD (b mod 8) owns.  Which block computes a
// tile does not change the tile's arithmetic or its partial.
struct TileWalk {
  int t, step, end;
};
__device__ __forceinline__ TileWalk tile_walk(int ntile) {
  int b = blockIdx.x, G = gridDim.x;
  if (G >= ntile) {
    int t = xcd_tile(b, G);
    return {t, 1, t + 1};
  }
  int x = b & 7, per = G >> 3;
  int lo = (int)((long long)ntile * x / 8), hi = (int)((long long)ntile * (x + 1) / 8);
  return {lo + (b >> 3), per, hi};
}

// iteration k >= 1: stopping test of iterate k-1, then p_k and q = A p_k.  FINE: a quarter of a tile per
// block, every load issued before the partial sums (at most four slots of a row; the rest after).
template <bool OFF16, bool FINE>
__global__ __launch_bounds__(FINE ? QUARTER : PCG_SPMV_NT) void k_pcg_spmv(
    SellView A, Tiles T, int k, const double* __restrict__ z, const double* __restrict__ p_prev,
    double* __restrict__ p_cur, double* __restrict__ q, const double* __restrict__ partB, double* __restrict__ partA,
    PcgCtl* ctls) {
  constexpr int NT = FINE ? QUARTER : PCG_SPMV_NT, C = FINE ? 1 : TILE / NT;
  const TileWalk tw = FINE ? TileWalk{xcd_tile(blockIdx.x, gridDim.x), 1, 0} : tile_walk(T.ntile);
  int cur = -1;
  bool skip = true;
  double beta = 0.0;
  __shared__ int done_sh;
  for (int b = tw.t; b < (FINE ? tw.t + 1 : tw.end); b += tw.step) {
    const Span ti = span_at<FINE>(T, b);
    const int s = ti.s;
    // FINE: the row's loads, in flight with the segment's
    CgRow<4, OFF16> row;
    SlotRange R0{0, 0};
    int n0 = 0;
    double zi = 0.0, pi0 = 0.0, di = 0.0;
    if constexpr (FINE) {
      const int i = min(ti.lo + (int)threadIdx.x, ti.end - 1);
      R0 = slots_of(A, i);
      n0 = row_len(A, i, R0);
      zi = z[i];
      pi0 = p_prev[i];
      di = A.diag[i];
      if (n0 > 0) row.load(A, i, R0.base, z, p_prev, n0);
    }
    if (s != cur) {
      // first tile of segment s for this block: the segment's stopping test and beta.  Every load
      // that needs only s (the flag's included) is issued at once, then the partials', so the block
      // waits for two load latencies before its sum instead of five.
      cur = s;
      PcgCtl* ctl = ctls + s;
      const int f = seg_first(T, s), n = seg_count(T, s), maxit = ctl->maxit, done = ctl->done;
      const double tol = ctl->tol, bn = ctl->bn, rho_older = ctl->rho[k & 1];  // rho_{k-2}
      double s2[2];  // (r_{k-1}.r_{k-1}, r_{k-1}.z_{k-1})
      // thread 0's read of the flag decides for the block: the segment's first tile may be setting it
      // during this launch (the totals' barriers order it; the one before them frees the previous value)
      __syncthreads();
      if (threadIdx.x == 0) done_sh = done;
      seg_totals<2, NT, FINE>(partB, T.ntile, f, n, s2);
      skip = done_sh != 0;
      if (!skip) {
        bool lead = ti.t == f && ti.j == 0 && threadIdx.x == 0;  // the segment's first block
        double rho = s2[1];
        if (lead) ctl->rho[(k - 1) & 1] = rho;
        beta = 0.0;
        if (k >= 2) {
          double rn = sqrt(s2[0]);
          bool conv = rn <= tol * bn;
          if (conv || k - 1 >= maxit) {
            if (lead) {
              ctl->done = 1;
              ctl->iters = k - 1;
              ctl->res = rn / bn;
              ctl->status = conv ? 0 : DIFVM_WARN_NOT_CONVERGED;
            }
            skip = true;
          } else {
            beta = rho / rho_older;  // rho_{k-1} / rho_{k-2}
          }
        } else if (maxit <= 0) {
          if (lead) {
            ctl->done = 1;
            ctl->status = DIFVM_WARN_NOT_CONVERGED;
          }
          skip = true;
        }
      }
    }
    if (skip) continue;
    double v[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int i = ti.lo + c * NT + (int)threadIdx.x;
      v[c] = 0.0;
      if (i < ti.hi) {
        double pi, acc;
        if constexpr (FINE) {
          pi = cg_dir(zi, beta, pi0);
          acc = row.add(di * pi, beta, n0);
          for (int k0 = 4; k0 < n0; ++k0) {
            CgRow<1, OFF16> one;
            one.load(A, i, R0.base + k0 * SLICE, z, p_prev);
            acc = one.add(acc, beta);
          }
        } else {
          pi = cg_dir(z[i], beta, p_prev[i]);
          SlotRange R = slots_of(A, i);
          acc = A.diag[i] * pi;
          walk_row<4>(row_len(A, i, R), [&](auto Wc, int k0) {
            CgRow<decltype(Wc)::value, OFF16> chunk;
            chunk.load(A, i, R.base + k0 * SLICE, z, p_prev);
            acc = chunk.add(acc, beta);
          });
        }
        p_cur[i] = pi;
        q[i] = acc;
        v[c] = pi * acc;
      }
    }
    put_partial<1, NT, FINE>(v, partA, T.ntile, ti);
  }
}

// G blocks walking the tiles, or (G = 0) a block per quarter
static void launch_pcg_spmv(int G, hipStream_t s, const SellView& V, const Tiles& T, int k, const double* z,
                            const double* p_prev, double* p_cur, double* q, const double* partB, double* partA,
                            PcgCtl* ctls) {
  if (G == 0) {
    if (V.off16) k_pcg_spmv<true, true><<<4 * T.ntile, QUARTER, 0, s>>>(V, T, k, z, p_prev, p_cur, q, partB, partA, ctls);
    else k_pcg_spmv<false, true><<<4 * T.ntile, QUARTER, 0, s>>>(V, T, k, z, p_prev, p_cur, q, partB, partA, ctls);
  } else {
    if (V.off16) k_pcg_spmv<true, false><<<G, PCG_SPMV_NT, 0, s>>>(V, T, k, z, p_prev, p_cur, q, partB, partA, ctls);
    else k_pcg_spmv<false, false><<<G, PCG_SPMV_NT, 0, s>>>(V, T, k, z, p_prev, p_cur, q, partB, partA, ctls);
  }
}

// iteration k: alpha, x and r updates, z = r/d, partials of r.r and r.z (streaming loads issued
// before the partial sum so they overlap its latency).  FINE: a quarter of a
// tile per block, and the loads do not wait for the stop flag either.
template <bool JAC, bool FINE>
__global__ __launch_bounds__(FINE ? QUARTER : BLOCK) void k_pcg_update(
    SellView A, Tiles T, double* __restrict__ x, double* __restrict__ r, double* __restrict__ z,
    const double* __restrict__ p_cur, const double* __restrict__ q, const double* __restrict__ partA,
    double* __restrict__ partB, int k, PcgCtl* ctls) {
  constexpr int NT = FINE ? QUARTER : BLOCK, C = FINE ? 1 : TILE / NT, NV = JAC ? 2 : 1;
  const Span ti = span_of<FINE>(T);
  PcgCtl* ctl = ctls + ti.s;
  // only earlier launches write the flag, so every wave reads the same value and the block needs
  // no barrier to agree on it
  const int done = ctl->done;
  if (!FINE && done) return;
  const int f = seg_first(T, ti.s), n = seg_count(T, ti.s);
  const double rho = ctl->rho[(k - 1) & 1];
  double xv[C], pv[C], rv[C], qv[C], dv[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    int i = min(ti.lo + c * NT + (int)threadIdx.x, ti.end - 1);  // tiles are never empty
    xv[c] = x[i];
    pv[c] = p_cur[i];
    rv[c] = r[i];
    qv[c] = q[i];
    dv[c] = JAC ? A.diag[i] : 1.0;
  }
  double pq[1];
  seg_totals<1, NT, FINE>(partA, T.ntile, f, n, pq);
  if (FINE && done) return;
  double alpha = rho / pq[0];
  double v[NV * C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    int i = ti.lo + c * NT + (int)threadIdx.x;
#pragma unroll
    for (int e = 0; e < NV; ++e) v[e * C + c] = 0.0;
    if (i < ti.hi) {
      x[i] = __builtin_fma(alpha, pv[c], xv[c]);
      double ri = __builtin_fma(-alpha, qv[c], rv[c]);
      r[i] = ri;
      v[c] = ri * ri;
      if constexpr (JAC) {
        double zi = ri / dv[c];
        z[i] = zi;
        v[C + c] = ri * zi;
      }
    }
  }
  put_partial<NV, NT, FINE>(v, partB, T.ntile, ti);
}

// ---------------------------------------------------------------------------------------------
// Jacobi-PCG of small segments, one block per segment and the whole solve in one launch: the direction
// vector in LDS, x, r, z (q in z's place) and the diagonal in registers (thread tid holds cells
// tid + c NT), uniform rows of three or four slots too.  An iteration is four block barriers and two
// reductions instead of two kernels; its time is their latency, which few waves keep short (every wave
// repeats the scalar work), so with rows in registers a block holds no more cells than the largest segment's tiles.
// Per iteration, two kernels -> this: 968 prisms 6.8 -> 1.35 us, 2,048 6.9 -> 1.8, 3,872 6.9 -> 2.7, 3,072 tets 7.2 -> 2.6.
// Other rows (hexahedra, mixed cells) are read from L2 in every iteration, always by 512 threads, and its time grows
// with the cells: 512 hexes 6.7 -> 3.3, 1,000 7.3 -> 3.9, 1,728 7.5 -> 4.9, 2,744 7.6 -> 6.1, 4,096 7.6 -> 7.4, which is why
// they too stop at four tiles.  In packs: 64 x 4,096 hexes 11.2 -> 7.5, 256 x 1,728 19.5 -> 6.5, 1,024 x 64
// 12.4 -> 10.6.  (Blocks as large as the tiles would take 3.5 us at 1,000 hexes and 5.7 at 2,744, but 5.4 at 1,728.)  Above
// four tiles the rows do not fit one compute unit's registers; read from L2 they took 8 to 9 us at five
// to eight tiles and 16 at eleven against 7.1, so those segments take the two kernels.
// A launch makes at most `chunk` iterations; what a further launch needs is stored when it ends unconverged.
// ---------------------------------------------------------------------------------------------
// most iterations per launch, which so stays under some 16 ms (7.4 us per iteration at 4,096 hexes), and of
// k_amg_pcg_block under 5 (17 us)
constexpr int SEG_CHUNK = 2048, AMG_CHUNK = 256;

// NT threads with C cells each; W: slots of every row, kept in registers (0: rows of any length, read in every
// iteration)
template <int NT, int C, int W>
__global__ __launch_bounds__(NT) void k_pcg_segment(SellView A, Tiles T, const double* __restrict__ b,
                                                    double* __restrict__ x, double* __restrict__ rbuf,
                                                    double* __restrict__ zbuf, double* __restrict__ pbuf, double tol,
                                                    int maxit, int chunk, bool first, PcgCtl* ctls) {
  constexpr int NTILE = NT * C / TILE, WAVES = NT / 64;
  constexpr bool REG = W > 0;
  static_assert(NTILE <= 4, "the tiles' sums fill one wave");
  __shared__ double sp[C * NT];
  __shared__ double gs[2][64];
  const int s = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  PcgCtl* ctl = ctls + s;
  if (!first && ctl->done) return;
  if (first && tid == 0) ctl_start(ctl, tol, maxit);
  const int f = seg_first(T, s), nt = seg_count(T, s);
  const TileIdx t0 = tile_at(T, f), t1 = tile_at(T, f + nt - 1);
  const int lo = t0.lo, n = t1.hi - lo;  // the segment's cells are consecutive
  const int k0 = first ? 0 : ctl->next;
  double xv[C], r[C], z[C], d[C];
  double own[REG ? C : 1];  // this thread's entries of sp
  // the totals of NV values per cell over the segment, in the order of the tiles' partials; v(k, c): value k
  // of this thread's cell c, formed when its group of values is summed
  auto totals = [&](auto&& v, auto& tot) {
#pragma clang fp contract(off)
    constexpr int NV = sizeof(tot) / sizeof(double);
    wave_sums<NV * C>([&](int e) { return e % C * NT + tid < n ? v(e / C, e % C) : 0.0; },
                      [&](int e, double sum) { gs[e / C][e % C * WAVES + wid] = sum; });
    __syncthreads();
    // every wave: the tiles' 16 groups in rows of lanes, then the order of a wave sum over the tiles
    // (distance 1, then 2)
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      double t = row_sum(gs[k][lane]);
      if (lane / TILE_WAVES >= nt) t = 0.0;
      t = swap_add16(t, t);
      tot[k] = wave_first(NTILE > 2 ? swap_add32(t, t) : t);
    }
  };
  constexpr int WR = REG ? W : 1;
  double av[REG ? C : 1][WR];
  int jv[REG ? C : 1][WR];
  if constexpr (REG) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      // cells past the segment: an empty row, so that no branch is needed for them
      const bool in = c * NT + tid < n;
      const int i = in ? lo + c * NT + tid : lo, base = (i >> 6) * (SLICE * W) + (i & (SLICE - 1));  // uniform rows
#pragma unroll
      for (int k = 0; k < W; ++k) {
        const double a = A.val[base + k * SLICE];
        const int j = A.off16[base + k * SLICE];
        av[c][k] = in ? a : 0.0;
        jv[c][k] = c * NT + tid + (in ? j : 0);
      }
    }
  }
  // out(c, (A w)_c) for this thread's cells c, w the vector in sp
  auto rows = [&](auto&& out) {
    if constexpr (REG) {
#pragma unroll
      for (int c = 0; c < C; ++c) {
        double acc = d[c] * own[c];
#pragma unroll
        for (int k = 0; k < W; ++k) acc = __builtin_fma(av[c][k], sp[jv[c][k]], acc);
        out(c, acc);
      }
    } else {
#pragma unroll
      for (int c = 0; c < C; ++c)
        if (const int me = c * NT + tid; me < n) {
          const int i = lo + me;
          SlotRange R = slots_of(A, i);
          double acc = d[c] * sp[me];
          walk_row<4>(row_len(A, i, R), [&](auto Wc, int q0) {
            constexpr int N = decltype(Wc)::value;
            double a[N];
            int j[N];
#pragma unroll
            for (int k = 0; k < N; ++k) {
              a[k] = A.val[R.base + (q0 + k) * SLICE];
              j[k] = me + A.off16[R.base + (q0 + k) * SLICE];
            }
#pragma unroll
            for (int k = 0; k < N; ++k) acc = __builtin_fma(a[k], sp[j[k]], acc);
          });
          out(c, acc);
        }
    }
  };
  double bn, rr, rho, rho_old;
  auto rr_rz = [&](int k, int c) { return k == 0 ? r[c] * r[c] : r[c] * z[c]; };
  double t1v[1], t2v[2];
  auto mine = [&](int c) {
    if constexpr (REG) return own[c];
    else return sp[c * NT + tid];
  };
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const bool in = c * NT + tid < n;
    const int i = lo + c * NT + tid;
    xv[c] = in ? x[i] : 0.0;
    d[c] = in ? A.diag[i] : 1.0;
    const double w0 = k0 == 0 ? xv[c] : in ? pbuf[i] : 0.0;
    sp[c * NT + tid] = w0;
    if constexpr (REG) own[c] = w0;
    if (k0 > 0) {
      r[c] = in ? rbuf[i] : 0.0;
      z[c] = in ? zbuf[i] : 0.0;
    }
  }
  if (k0 == 0) {
    __syncthreads();
#pragma unroll
    for (int c = 0; c < C; ++c) r[c] = z[c] = 0.0;  // z: b
    rows([&](int c, double ax) {
      const int e = c * NT + tid;
      if (e < n) z[c] = b[lo + e];
      r[c] = z[c] - ax;
    });
    totals([&](int k, int c) { return k == 0 ? z[c] * z[c] : r[c] * r[c]; }, t2v);
    bn = sqrt(t2v[0]);
    const double rn = sqrt(t2v[1]);
    const bool zero_b = bn == 0.0, stop = zero_b || rn <= tol * bn;
    if (tid == 0) {
      ctl->bn = bn;
      ctl->res = zero_b ? 0.0 : rn / bn;
      ctl->done = stop ? 1 : 0;
    }
    if (zero_b)
#pragma unroll
      for (int c = 0; c < C; ++c)
        if (c * NT + tid < n) x[lo + c * NT + tid] = 0.0;
    if (stop) return;
    __syncthreads();  // gs is read, sp too
#pragma unroll
    for (int c = 0; c < C; ++c) {
      z[c] = r[c] / d[c];
      sp[c * NT + tid] = 0.0;
      if constexpr (REG) own[c] = 0.0;
    }
    totals(rr_rz, t2v);
    rr = t2v[0];
    rho = t2v[1];
    rho_old = 0.0;
  } else {
    bn = ctl->bn;
    rr = ctl->rr;
    rho = ctl->rho[0];
    rho_old = ctl->rho[1];
  }
  int k = k0 + 1;
  bool done = false;
  for (;; ++k) {
    double beta = 0.0;
    if (k >= 2) {
      const double rn = sqrt(rr);
      const bool conv = rn <= tol * bn;
      if (conv || k - 1 >= maxit) {
        done = true;
        if (tid == 0) {
          ctl->done = 1;
          ctl->iters = k - 1;
          ctl->res = rn / bn;
          ctl->status = conv ? 0 : DIFVM_WARN_NOT_CONVERGED;
        }
        break;
      }
      beta = rho / rho_old;
    } else if (maxit <= 0) {
      done = true;
      if (tid == 0) {
        ctl->done = 1;
        ctl->status = DIFVM_WARN_NOT_CONVERGED;
      }
      break;
    }
    if (k - k0 > chunk) break;
#pragma unroll
    for (int c = 0; c < C; ++c) {  // read by others only after the barrier, and before the sums' own
      const double p = cg_dir(z[c], beta, mine(c));
      sp[c * NT + tid] = p;
      if constexpr (REG) own[c] = p;
    }
    __syncthreads();
    if constexpr (!REG)
#pragma unroll
      for (int c = 0; c < C; ++c) z[c] = 0.0;
    rows([&](int c, double q) { z[c] = q; });  // z holds q until r is updated
    totals([&](int, int c) { return mine(c) * z[c]; }, t1v);
    const double alpha = rho / t1v[0];
    __syncthreads();  // gs is read
#pragma unroll
    for (int c = 0; c < C; ++c) {
      xv[c] = __builtin_fma(alpha, mine(c), xv[c]);
      r[c] = __builtin_fma(-alpha, z[c], r[c]);
      z[c] = r[c] / d[c];
    }
    totals(rr_rz, t2v);
    rr = t2v[0];
    rho_old = rho;
    rho = t2v[1];
    // (the next iteration's barrier after the directions also separates these sums' reads from the
    // next ones' writes)
  }
#pragma unroll
  for (int c = 0; c < C; ++c)
    if (const int e = c * NT + tid; e < n) {
      x[lo + e] = xv[c];
      if (!done) {
        rbuf[lo + e] = r[c];
        zbuf[lo + e] = z[c];
        pbuf[lo + e] = sp[e];
      }
    }
  if (!done && tid == 0) {
    ctl->next = k - 1;
    ctl->rr = rr;
    ctl->rho[0] = rho;
    ctl->rho[1] = rho_old;
  }
}

// most tiles of a segment
static int max_seg_tiles(const difvm_mesh* m) {
  int n = 0;
  for (int32_t c : m->host.seg_tile_n) n = std::max(n, (int)c);
  return n;
}

static void launch_pcg_segment(const difvm_mesh* m, int nt, const SellView& V, const Tiles& T, const double* b,
                               double* x, KrylovWork* w, double tol, int maxit, int chunk, bool first, PcgCtl* ctls) {
  const int G = m->d.nseg;
  hipStream_t s = stream_of(m);
// as many cells as the tiles hold
#define DIFVM_SEG_TILES(W)             \
  switch (nt) {                        \
    case 1: DIFVM_SEG(256, 4, W); break; \
    case 2: DIFVM_SEG(256, 8, W); break; \
    case 3: DIFVM_SEG(512, 6, W); break; \
    default: DIFVM_SEG(512, 8, W);     \
  }
#define DIFVM_SEG(NT, C, W) \
  k_pcg_segment<NT, C, W><<<G, NT, 0, s>>>(V, T, b, x, w->r, w->z, w->p, tol, maxit, chunk, first, ctls)
  if (V.uw == 4) DIFVM_SEG_TILES(4)
  else if (V.uw == 3) DIFVM_SEG_TILES(3)
  else DIFVM_SEG(512, 8, 0);
#undef DIFVM_SEG_TILES
#undef DIFVM_SEG
  DIFVM_HIP(hipGetLastError());
}

// per-segment control state set on the device (no host buffer, so the launch can be captured)
__global__ void k_pcg_ctl_init(PcgCtl* ctls, int nseg, double tol, int maxit) {
  int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g < nseg) ctl_start(ctls + g, tol, maxit);
}

// copies n doubles (solver states are made of doubles and ints, 8-byte multiples)
__global__ void k_copy_words(double* __restrict__ dst, const double* __restrict__ src, int n) {
  int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) dst[q] = src[q];
}
static void copy_state(void* dst, const void* src, size_t bytes, hipStream_t s) {
  int n = (int)(bytes / sizeof(double));
  k_copy_words<<<(n + 255) / 256, 256, 0, s>>>(static_cast<double*>(dst), static_cast<const double*>(src), n);
  DIFVM_HIP(hipGetLastError());
}

size_t pcg_state_bytes(const difvm_mesh* m) { return sizeof(PcgCtl) * m->d.nseg; }

// grid of the product kernel: one block per tile, or the tuned persistent grid (a multiple of 8)
int pcg_spmv_grid(const difvm_mesh* m) {
  int nt = m->d.ntile, g = m->tune[DIFVM_TUNE_PCG_GRID];
  if (g <= 0 || g >= nt) return nt;
  return std::max(8, g & ~7);
}

// the same as launch_pcg_spmv takes it: 0 (a block per quarter of a tile) on meshes of few tiles, which no
// persistent grid suits
static int pcg_spmv_launch_grid(const difvm_mesh* m) { return fine_spans(m) ? 0 : pcg_spmv_grid(m); }

SolveResult pcg_result(const difvm_mesh* m, const void* host_state, bool* complete) {
  const PcgCtl* hs = static_cast<const PcgCtl*>(host_state);
  int nseg = m->d.nseg;
  SolveResult R;
  R.seg.resize(nseg);
  bool all = true;
  for (int g = 0; g < nseg; ++g) {
    const PcgCtl& c = hs[g];
    all = all && c.done;
    int st = c.done ? c.status : (int)DIFVM_WARN_NOT_CONVERGED;
    R.seg[g] = {{c.iters, 0, 0}, {c.res, 0, 0}, st};
    R.iters[0] = std::max(R.iters[0], c.iters);
    R.res[0] = std::max(R.res[0], c.res);
    R.status = std::max(R.status, st);
  }
  if (complete) *complete = all;
  return R;
}

// Polling without draining the queue: the host copies the per-segment states into one of two pinned
// buffers after a block of iterations and records an event, queues the next block, and only then
// waits for the earlier copy; iterations queued past a segment's stop are predicated no-ops, so the
// extra block changes nothing.
static void post_poll(difvm_mesh* m, KrylovWork* w, const void* dstate, size_t bytes, int slot) {
  hipStream_t s = stream_of(m);
  DIFVM_HIP(hipMemcpyAsync(w->host_state[slot], dstate, bytes, hipMemcpyDeviceToHost, s));
  DIFVM_HIP(hipEventRecord(w->poll_ev[slot], s));
}
static const void* wait_poll(KrylovWork* w, int slot) {
  DIFVM_HIP(hipEventSynchronize(w->poll_ev[slot]));
  return w->host_state[slot];
}

SolveResult pcg(difvm_mesh* m, SellMatrix A, const double* b, double* x, double tol, int maxit, const QueueOnly* qo,
                const AmgDev* amg, int* hint) {
  KrylovWork* w = make_work(m);
  hipStream_t s = stream_of(m);
  SellView V = sview(m, A);
  Tiles T = tiles_of(m);
  const int nseg = m->d.nseg;
  const size_t prof_mark = ctx_of(m).prof.pending.size();  // timed launches of this solve start here
  const int seg_tiles = max_seg_tiles(m);
  // launches inside a captured step are never timed, so a step captured meanwhile is the one that replays keep
  const Profiler& prof = ctx_of(m).prof;
  const bool timed = prof.on && !ctx_of(m).capturing;
  if (amg ? amg_pcg_in_block(amg) : seg_tiles <= SEG_TILES && !timed) {
    // one block per segment makes the whole solve (with Jacobi, while the kernels of an iteration are being timed,
    // it is made by them: the same bits)
    const int budget = qo ? std::min(qo->budget, maxit) : maxit;
    const size_t bytes = pcg_state_bytes(m);
    PcgCtl* ctls = qo ? static_cast<PcgCtl*>(qo->state_out) : w->pcg;
    int made = 0;
    do {
      const int chunk = std::min(amg ? AMG_CHUNK : SEG_CHUNK, budget - made);
      if (amg) {
        ProfScope ps(m, "pcg_amg_block");
        amg_pcg_block(amg, A, b, x, w->r, w->p, tol, maxit, chunk, made == 0, ctls);
      } else {
        launch_pcg_segment(m, seg_tiles, V, T, b, x, w, tol, maxit, chunk, made == 0, ctls);
      }
      made += chunk;
      if (qo) continue;
      post_poll(m, w, w->pcg, bytes, 0);
      const PcgCtl* hs = static_cast<const PcgCtl*>(wait_poll(w, 0));
      bool all = true;
      for (int g = 0; g < nseg; ++g) all = all && hs[g].done;
      if (all) break;
    } while (made < budget);
    if (qo) return SolveResult{};
    SolveResult R = pcg_result(m, w->host_state[0], nullptr);
    if (hint) *hint = R.iters[0];
    return R;
  }
  k_pcg_ctl_init<<<(nseg + 63) / 64, 64, 0, s>>>(w->pcg, nseg, tol, maxit);
  const int GS = pcg_spmv_launch_grid(m);
  const bool fine = fine_spans(m);
  const int NP = n_spans(m), NTB = fine ? QUARTER : TILE;  // partials of one value; threads of the init kernels
  double* Rk[2] = {w->r, w->rh};  // r_k at parity k & 1 (joint), else r
  double* r = w->r;
  double* q = w->q;
  double* z = w->z;
  double* Pk[2] = {w->p, w->v};  // p_k at parity k & 1
  double* partA = w->partials;
  double* partB = w->partials + 2 * (size_t)NP;
  double* part0 = w->partials + 4 * (size_t)NP;
  // z = M^-1 r: Jacobi inside the init / update kernels, or one V-cycle after them (which also stores
  // the r.z partials)
  // (the V-cycle's kernels skip their work once every segment has stopped; while some segment runs
  // on they compute for all, which changes nothing a stopped segment reads)
  // the cycle's first kernel makes iterate kk's stopping test, so that the last cycle ends with it; while every
  // launch is being timed the product makes it and every timed cycle is a whole one
  const bool cycle_test = !(timed && prof.stride == 1);
  auto precondition = [&](int kk, const CgStep* step = nullptr) {
    if (!amg) return;
    ProfScope ps(m, "pcg_amg_vcycle", cycle_test ? kk + 1 : kk);  // a whole cycle if iteration kk + 1 runs
    amg_vcycle(amg, A, step ? step->r_new : r, z, partB + NP, w->pcg, cycle_test && kk > 0 ? partB : nullptr, kk, step,
               q);  // q is free until the next product
  };
  (fine ? k_pcg_init1<true> : k_pcg_init1<false>)<<<NP, NTB, 0, s>>>(V, T, b, x, r, part0);
  (amg ? fine ? k_pcg_init2<false, true> : k_pcg_init2<false, false>
       : fine ? k_pcg_init2<true, true> : k_pcg_init2<true, false>)<<<NP, NTB, 0, s>>>(V, T, x, r, z, Pk[0], part0, partB,
                                                                                        w->pcg);
  DIFVM_HIP(hipGetLastError());
  precondition(0);
  // on meshes of few tiles the update is made by the cycle's first kernel (while kernels are being timed by
  // name, by its own: the same bits)
  const bool joint = amg && fine && !timed;
  auto update = [&](int kk) {
    if (joint) {
      const CgStep step{x, Pk[kk & 1], Rk[(kk - 1) & 1], q, partA, Rk[kk & 1]};
      precondition(kk, &step);
      return;
    }
    {
      ProfScope ps(m, "pcg_update_dot", kk);
      auto kernel = fine ? (amg ? k_pcg_update<false, true> : k_pcg_update<true, true>)
                         : (amg ? k_pcg_update<false, false> : k_pcg_update<true, false>);
      kernel<<<NP, fine ? QUARTER : BLOCK, 0, s>>>(V, T, x, r, z, Pk[kk & 1], q, partA, partB, kk, w->pcg);
    }
    precondition(kk);
  };
  if (qo) {
    // queue-only: iterations 1..K and the stopping test of iterate K, no read-back
    int K = std::min(qo->budget, maxit);
    const int last = amg && cycle_test && K > 0 ? K : K + 1;  // the launch that tests iterate K
    for (int kk = 1; kk <= last; ++kk) {
      {
        ProfScope ps(m, "pcg_spmv_dot", kk);
        launch_pcg_spmv(GS, s, V, T, kk, z, Pk[(kk - 1) & 1], Pk[kk & 1], q, partB, partA, w->pcg);
      }
      if (kk <= K) update(kk);
    }
    DIFVM_HIP(hipGetLastError());
    copy_state(qo->state_out, w->pcg, pcg_state_bytes(m), s);
    return SolveResult{};
  }
  // First block sized from the previous solve, then blocks of one iteration, each queued before the
  // host waits for the state copied after the block before it (an iteration's GPU time covers the
  // host's queueing of the next block); iterations queued past the stop are idle launches, one or two
  // per solve.  Iteration k's stopping test runs at the start of iteration k+1, so the host
  // queues up to iteration maxit+1.
  int k = 1;  // next iteration to queue
  auto queue_block = [&](int nb) {
    for (int n = 0; n < nb && k <= maxit + 1; ++n, ++k) {
      {
        ProfScope ps(m, "pcg_spmv_dot", k);
        launch_pcg_spmv(GS, s, V, T, k, z, Pk[(k - 1) & 1], Pk[k & 1], q, partB, partA, w->pcg);
      }
      if (k <= maxit) update(k);
    }
    DIFVM_HIP(hipGetLastError());
  };
  const size_t bytes = pcg_state_bytes(m);
  queue_block(std::max(4, (hint ? *hint : 0) - 2));
  int slot = 0;
  post_poll(m, w, w->pcg, bytes, slot);
  const PcgCtl* hs = nullptr;
  while (true) {
    bool more = k <= maxit + 1;
    if (more) {
      queue_block(1);
      post_poll(m, w, w->pcg, bytes, slot ^ 1);
    }
    hs = static_cast<const PcgCtl*>(wait_poll(w, slot));
    bool all = true;
    for (int g = 0; g < nseg; ++g) all = all && hs[g].done;
    if (all || !more) break;
    slot ^= 1;
  }
  SolveResult R = pcg_result(m, hs, nullptr);
  // iteration k's kernels ran while some segment had not stopped, i.e. for k <= the largest count (and the
  // cycle after the last one ended with its first kernel)
  prof_idle_after(ctx_of(m), prof_mark, R.iters[0]);  // iters[0]: the largest over the segments
  if (hint) *hint = R.iters[0];
  return R;
}

// ---------------------------------------------------------------------------------------------
// BiCGStab kernels (NC systems sharing one matrix per segment, interleaved vectors): five launches per
// iteration and no kernel for the scalars.  As in PCG, each reduction's per-tile partials are summed
// again (per segment, fixed order) by every block of the next kernel that needs them:
//   init:   r = b - A x, rhat = r; off-diagonals of A D^-1          partials X = (b.b, r.r)
//   dir_k:  (from X) stopping test of iterate k-1, beta; p = r + beta (p - omega v)
//   v_k:    v = A D^-1 p                                            partials V = rhat.v
//   s_k:    (from V) alpha; s = r - alpha v, in r's place
//   t_k:    t = A D^-1 s                                            partials T = (t.s, t.t, s.s)
//   x_k:    (from T) test on s, omega; x += D^-1 (alpha p + omega s); r = s - omega t
//                                                                   partials X = (r.r, rhat.r)
// The state of iteration k lives in copy k & 1: dir_k reads copy k-1 and its segment's first tile writes
// copy k whole; that tile's block of s_k adds alpha and of x_k adds omega and the outcome of the test on
// s, fields that no block of the same launch reads.  Columns are scaled by 1/d once per solve, so the
// products gather p and s alone (not d beside them, with a division for each neighbour).
// Blocks have one thread per cell, of a tile or of a quarter of one (see Span): four cells per thread left
// each thread's rows one after another.
// At 167,400 cells (3 components) an iteration's kernels took 73 us as eight launches of 256-thread
// blocks, 36 us now; at 1,053,696 cells 160, 129 now (dir 19.4, v 25.2, s 12.0, t 24.0, x 34.1, totals 14).
// ---------------------------------------------------------------------------------------------

// (B f)_i for NC interleaved components, B the off-diagonals in val plus DIAG f_i; padding and boundary
// slots carry val = 0 and col = i.  The row's slots in layout order, the first four with every load issued
// before any is used.
template <int NC>
__device__ __forceinline__ void scaled_row(const SellView& A, const double* __restrict__ val, int i,
                                           const double* __restrict__ f, double (&acc)[NC]) {
  SlotRange R = slots_of(A, i);
  const bool off16 = A.off16 != nullptr;  // the same for every thread: a uniform branch
  walk_row<4>(R.width, [&](auto Wc, int k0) {
    constexpr int N = decltype(Wc)::value;
    double a[N], fj[N][NC];
    int j[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
      int at = R.base + (k0 + k) * SLICE;
      a[k] = val[at];
      j[k] = off16 ? i + A.off16[at] : A.col[at];
    }
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
      for (int c = 0; c < NC; ++c) fj[k][c] = f[(size_t)j[k] * NC + c];
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[c] = __builtin_fma(a[k], fj[k][c], acc[c]);
  });
}

// The NV totals of the segment for a kernel that needs them: summed here by every block (FINE), or read from
// the array that k_bi_totals filled.  Same sums, same bits.
template <int NV, bool FINE>
__device__ __forceinline__ void bi_totals(const double* __restrict__ part, const Tiles& T, int s, double (&tot)[NV]) {
  if constexpr (FINE) {
    seg_totals<NV, QUARTER, true>(part, T.ntile, seg_first(T, s), seg_count(T, s), tot);
  } else {
#pragma unroll
    for (int k = 0; k < NV; ++k) tot[k] = part[s * NV + k];
  }
}
// Above FINE_TILES tiles the totals get a kernel of their own, three per iteration of 4.7 us: at 1,029 tiles
// every block summing 6 partials per tile by itself made the direction pass 32.2 us against 19.6 + 4.7.
template <int NV>
__global__ __launch_bounds__(TILE) void k_bi_totals(const double* __restrict__ part, Tiles T, double* __restrict__ out) {
  const int s = blockIdx.x;
  double tot[NV];
  seg_totals<NV, TILE, false>(part, T.ntile, seg_first(T, s), seg_count(T, s), tot);
  if (threadIdx.x == 0)
#pragma unroll
    for (int k = 0; k < NV; ++k) out[s * NV + k] = tot[k];
}

// r = b - A x, rhat = r, partials b.b and r.r; val of A D^-1 (p and v start at zero: the first direction
// pass writes p = r without reading them)
template <int NC, bool FINE>
__global__ __launch_bounds__(FINE ? QUARTER : TILE) void k_bi_init(SellView A, Tiles T, const double* __restrict__ b,
                                                  const double* __restrict__ x, double* __restrict__ r,
                                                  double* __restrict__ rh, double* __restrict__ colscaled,
                                                  double* __restrict__ part) {
  constexpr int NT = FINE ? QUARTER : TILE;
  const Span ti = span_of<FINE>(T);
  const int i = ti.lo + (int)threadIdx.x;
  double acc[2 * NC], ri[NC];
#pragma unroll
  for (int k = 0; k < 2 * NC; ++k) acc[k] = 0.0;
  if (i < ti.hi) {
    double ax[NC], bi[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) bi[c] = b[(size_t)i * NC + c];
    SlotRange R = slots_of(A, i);
    const double di = A.diag[i];
#pragma unroll
    for (int c = 0; c < NC; ++c) ax[c] = di * x[(size_t)i * NC + c];
    walk_row<4>(R.width, [&](auto Wc, int k0) {
      constexpr int N = decltype(Wc)::value;
      double a[N], dj[N], xj[N][NC];
      int j[N];
#pragma unroll
      for (int k = 0; k < N; ++k) {
        int at = R.base + (k0 + k) * SLICE;
        a[k] = A.val[at];
        j[k] = A.off16 ? i + A.off16[at] : A.col[at];
      }
#pragma unroll
      for (int k = 0; k < N; ++k) {
        dj[k] = A.diag[j[k]];
#pragma unroll
        for (int c = 0; c < NC; ++c) xj[k][c] = x[(size_t)j[k] * NC + c];
      }
#pragma unroll
      for (int k = 0; k < N; ++k) {
        colscaled[R.base + (k0 + k) * SLICE] = a[k] / dj[k];
#pragma unroll
        for (int c = 0; c < NC; ++c) ax[c] = __builtin_fma(a[k], xj[k][c], ax[c]);
      }
    });
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      ri[c] = bi[c] - ax[c];
      acc[c] = bi[c] * bi[c];
      acc[NC + c] = ri[c] * ri[c];
    }
  }
  if constexpr (NC == 1) {
    if (i < ti.hi) r[i] = rh[i] = ri[0];
  } else {
    __shared__ double lds[NC * NT];
    store_rows<NC>(r, ti.lo, ti.hi, ri, lds);
    store_rows<NC>(rh, ti.lo, ti.hi, ri, lds);
  }
  put_partial<2 * NC, NT, FINE>(acc, part, T.ntile, ti);
}

// component c's value of an array held in registers (no run-time index, which would move it to memory)
template <int NC, class T>
__device__ __forceinline__ T pick(const T (&a)[NC], int c) {
  if constexpr (NC == 1) {
    return a[0];
  } else {
    static_assert(NC == 3, "one or three components");
    const T a0 = a[0], a1 = a[1], a2 = a[2];
    return c == 0 ? a0 : c == 1 ? a1 : a2;
  }
}

// copies the first NC systems' state, field by field (a whole-struct copy of unused ones goes through memory)
template <int NC>
__device__ __forceinline__ void copy_systems(BiState& d, const BiState& s) {
  d.tol = s.tol;
  d.maxit = s.maxit;
  d.any = s.any;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    d.bn[c] = s.bn[c];
    d.rho[c] = s.rho[c];
    d.alpha[c] = s.alpha[c];
    d.omega[c] = s.omega[c];
    d.res[c] = s.res[c];
    d.sres[c] = s.sres[c];
    d.iters[c] = s.iters[c];
    d.active[c] = s.active[c];
    d.so[c] = s.so[c];
    d.status[c] = s.status[c];
  }
}

// iteration it >= 1: stopping test of iterate it - 1 (it = 1: of the initial guess), then the direction.
// One thread per value of the tile's rows (consecutive lanes, consecutive doubles), NC rounds.
template <int NC, bool FINE>
__global__ __launch_bounds__(FINE ? QUARTER : TILE, FINE ? 1 : 8) void k_bi_dir(Tiles T, int it, const double* __restrict__ r, double* __restrict__ p,
                                                 const double* __restrict__ v, double* __restrict__ x,
                                                 const double* __restrict__ part, BiState* sts, int nseg) {
  constexpr int NT = FINE ? QUARTER : TILE;
  const Span ti = span_of<FINE>(T);
  const BiState* prev = sts + (size_t)((it - 1) & 1) * nseg + ti.s;
  BiState S;
  copy_systems<NC>(S, *prev);
  const bool lead = ti.t == seg_first(T, ti.s) && ti.j == 0 && threadIdx.x == 0;
  BiState* cur = sts + (size_t)(it & 1) * nseg + ti.s;
  const int e0 = NC * ti.lo, e1 = NC * ti.hi;
  if (it > 1 && !S.any) {  // stopped before: the state moves on with the parity
    if (lead) copy_systems<NC>(*cur, S);
    return;
  }
  double rv[NC], pv[NC], vv[NC];  // in flight with the partials
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int e = min(e0 + q * NT + (int)threadIdx.x, NC * ti.end - 1);
    rv[q] = r[e];
    pv[q] = vv[q] = 0.0;
    if (it > 1) {
      pv[q] = p[e];
      vv[q] = v[e];
    }
  }
  double tot[2 * NC];
  bi_totals<2 * NC, FINE>(part, T, ti.s, tot);
  double beta[NC], omega[NC];
  bool act[NC], zero[NC];
  S.any = 0;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    beta[c] = omega[c] = 0.0;
    zero[c] = false;
    if (it == 1) {
      const double bn = sqrt(tot[c]), rn = sqrt(tot[NC + c]);
      S.bn[c] = bn;
      S.res[c] = bn == 0.0 ? 0.0 : rn / bn;
      S.rho[c] = tot[NC + c];  // rhat = r, so rhat.r = r.r
      S.active[c] = (bn == 0.0 || rn <= S.tol * bn) ? 0 : 1;
      zero[c] = bn == 0.0;  // b = 0 gives x = 0
      if (S.active[c] && S.maxit <= 0) {
        S.active[c] = 0;
        S.status[c] = DIFVM_WARN_NOT_CONVERGED;
      } else if (S.active[c] && S.rho[c] == 0.0) {
        S.active[c] = 0;
        S.status[c] = DIFVM_WARN_BREAKDOWN;
      }
    } else if (S.active[c]) {
      if (S.so[c] == BI_SO_BREAKDOWN) {
        S.active[c] = 0;
        S.status[c] = DIFVM_WARN_BREAKDOWN;
      } else {
        S.iters[c] = it - 1;
        if (S.so[c] == BI_SO_DONE) {
          S.active[c] = 0;
          S.res[c] = S.sres[c];
        } else {
          const double rn = sqrt(tot[c]), rho = S.rho[c];
          S.res[c] = rn / S.bn[c];
          if (rn <= S.tol * S.bn[c]) {
            S.active[c] = 0;
          } else if (it - 1 >= S.maxit) {
            S.active[c] = 0;
            S.status[c] = DIFVM_WARN_NOT_CONVERGED;
          } else {
            S.rho[c] = tot[NC + c];
            if (S.rho[c] == 0.0) {
              S.active[c] = 0;
              S.status[c] = DIFVM_WARN_BREAKDOWN;
            } else {
              omega[c] = S.omega[c];
              beta[c] = (S.rho[c] / rho) * (S.alpha[c] / omega[c]);
            }
          }
        }
      }
    }
    S.so[c] = BI_SO_GO;
    act[c] = S.active[c] != 0;
    S.any |= S.active[c];
  }
  if (lead) copy_systems<NC>(*cur, S);
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int e = e0 + q * NT + (int)threadIdx.x;
    if (e >= e1) continue;
    const int c = e % NC;
    if (pick(zero, c)) x[e] = 0.0;
    if (!pick(act, c)) continue;
    p[e] = it == 1 ? rv[q]
                   : __builtin_fma(pick(beta, c), __builtin_fma(-pick(omega, c), vv[q], pv[q]), rv[q]);
  }
}

// v = A D^-1 p; partial rhat . v
template <int NC, bool FINE>
__global__ __launch_bounds__(FINE ? QUARTER : TILE) void k_bi_v(SellView A, const double* __restrict__ colscaled, Tiles T, int it,
                                               const double* __restrict__ p, double* __restrict__ v,
                                               const double* __restrict__ rh, double* __restrict__ part,
                                               const BiState* sts, int nseg) {
  constexpr int NT = FINE ? QUARTER : TILE;
  const Span ti = span_of<FINE>(T);
  const BiState* st = sts + (size_t)(it & 1) * nseg + ti.s;
  if (!st->any) return;
  bool act[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) act[c] = st->active[c] != 0;
  const int i = ti.lo + (int)threadIdx.x;
  double ay[NC], acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) ay[c] = acc[c] = 0.0;
  if (i < ti.hi) {
    double rhi[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {  // own values, in flight with the row's loads
      rhi[c] = rh[(size_t)i * NC + c];
      ay[c] = p[(size_t)i * NC + c];
    }
    scaled_row<NC>(A, colscaled, i, p, ay);
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = act[c] ? rhi[c] * ay[c] : 0.0;
  }
  if constexpr (NC == 1) {
    if (i < ti.hi) v[i] = ay[0];
  } else {
    __shared__ double lds[NC * NT];
    store_rows_if<NC>(v, ti.lo, ti.hi, ay, act, lds);
  }
  put_partial<NC, NT, FINE>(acc, part, T.ntile, ti);
}

// alpha, s = r - alpha v, one thread per value of the tile's rows (as k_bi_dir)
template <int NC, bool FINE>
__global__ __launch_bounds__(FINE ? QUARTER : TILE, FINE ? 1 : 8) void k_bi_s(Tiles T, int it, double* __restrict__ r,
                                               const double* __restrict__ v, const double* __restrict__ part, BiState* sts, int nseg) {
  constexpr int NT = FINE ? QUARTER : TILE;
  const Span ti = span_of<FINE>(T);
  BiState* st = sts + (size_t)(it & 1) * nseg + ti.s;
  if (!st->any) return;
  const int e0 = NC * ti.lo, e1 = NC * ti.hi;
  double rv[NC], vv[NC];  // in flight with the partials
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int e = min(e0 + q * NT + (int)threadIdx.x, NC * ti.end - 1);
    rv[q] = r[e];
    vv[q] = v[e];
  }
  double tot[NC], alpha[NC];
  bool act[NC];
  bi_totals<NC, FINE>(part, T, ti.s, tot);
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    act[c] = st->active[c] != 0;
    alpha[c] = st->rho[c] / tot[c];
  }
  if (ti.t == seg_first(T, ti.s) && ti.j == 0 && threadIdx.x == 0)
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (act[c]) st->alpha[c] = alpha[c];
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int e = e0 + q * NT + (int)threadIdx.x;
    if (e >= e1) continue;
    const int c = e % NC;
    if (pick(act, c)) r[e] = __builtin_fma(-pick(alpha, c), vv[q], rv[q]);
  }
}

// t = A D^-1 s (s gathered from the pass above); partials t.s, t.t, s.s
template <int NC, bool FINE>
__global__ __launch_bounds__(FINE ? QUARTER : TILE) void k_bi_t(SellView A, const double* __restrict__ colscaled, Tiles T, int it,
                                               const double* __restrict__ s, double* __restrict__ t,
                                               double* __restrict__ part, const BiState* sts, int nseg) {
  constexpr int NT = FINE ? QUARTER : TILE;
  const Span ti = span_of<FINE>(T);
  const BiState* st = sts + (size_t)(it & 1) * nseg + ti.s;
  if (!st->any) return;
  bool act[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) act[c] = st->active[c] != 0;
  const int i = ti.lo + (int)threadIdx.x;
  double az[NC], acc[3 * NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) az[c] = acc[c] = acc[NC + c] = acc[2 * NC + c] = 0.0;
  if (i < ti.hi) {
    double si[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) az[c] = si[c] = s[(size_t)i * NC + c];
    scaled_row<NC>(A, colscaled, i, s, az);
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (act[c]) {
        acc[c] = az[c] * si[c];
        acc[NC + c] = az[c] * az[c];
        acc[2 * NC + c] = si[c] * si[c];
      }
  }
  if constexpr (NC == 1) {
    if (i < ti.hi) t[i] = az[0];
  } else {
    __shared__ double lds[NC * NT];
    store_rows_if<NC>(t, ti.lo, ti.hi, az, act, lds);
  }
  put_partial<3 * NC, NT, FINE>(acc, part, T.ntile, ti);
}

// the test on s (the iteration ends with x += alpha D^-1 p if it passes) and omega;
// x += alpha D^-1 p (+ omega D^-1 s); r = s - omega t; partials r.r, rhat.r
template <int NC, bool FINE>
__global__ __launch_bounds__(FINE ? QUARTER : TILE, FINE ? 1 : 8) void k_bi_x(SellView A, Tiles T, int it, double* __restrict__ x,
                                               double* __restrict__ r, const double* __restrict__ rh,
                                               const double* __restrict__ p, const double* __restrict__ t,
                                               const double* __restrict__ part_in,
                                               double* __restrict__ part, BiState* sts, int nseg) {
  constexpr int NT = FINE ? QUARTER : TILE;
  const Span ti = span_of<FINE>(T);
  BiState* st = sts + (size_t)(it & 1) * nseg + ti.s;
  if (!st->any) return;
  const int i = ti.lo + (int)threadIdx.x, ii = min(i, ti.end - 1);
  double pv[NC], sv[NC], tv[NC], xv[NC], hv[NC];  // in flight with the partials
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const size_t at = (size_t)ii * NC + c;
    xv[c] = x[at];
    pv[c] = p[at];
    sv[c] = r[at];  // s
    tv[c] = t[at];
    hv[c] = rh[at];
  }
  const double di = A.diag[ii];
  double tot[3 * NC];
  bi_totals<3 * NC, FINE>(part_in, T, ti.s, tot);
  const bool lead = ti.t == seg_first(T, ti.s) && ti.j == 0 && threadIdx.x == 0;
  bool keep_x[NC], keep_r[NC];
  double acc[2 * NC], rv[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const double alpha = st->alpha[c], sn = sqrt(tot[2 * NC + c]), bn = st->bn[c];
    const bool small = sn <= st->tol * bn, bad = !small && tot[NC + c] == 0.0;
    const double omega = tot[c] / tot[NC + c];
    keep_x[c] = st->active[c] != 0 && !bad;
    keep_r[c] = keep_x[c] && !small;
    if (lead && st->active[c]) {
      st->so[c] = small ? BI_SO_DONE : bad ? BI_SO_BREAKDOWN : BI_SO_GO;
      st->sres[c] = sn / bn;
      st->omega[c] = omega;
    }
    const double y = pv[c] / di, z = sv[c] / di;
    xv[c] = __builtin_fma(alpha, y, keep_r[c] ? __builtin_fma(omega, z, xv[c]) : xv[c]);
    rv[c] = __builtin_fma(-omega, tv[c], sv[c]);
    const bool in = keep_r[c] && i < ti.hi;
    acc[c] = in ? rv[c] * rv[c] : 0.0;
    acc[NC + c] = in ? hv[c] * rv[c] : 0.0;
  }
  if constexpr (NC == 1) {
    if (i < ti.hi && keep_x[0]) x[i] = xv[0];
    if (i < ti.hi && keep_r[0]) r[i] = rv[0];
  } else {
    __shared__ double lds[NC * NT];
    store_rows_if<NC>(x, ti.lo, ti.hi, xv, keep_x, lds);
    store_rows_if<NC>(r, ti.lo, ti.hi, rv, keep_r, lds);
  }
  put_partial<2 * NC, NT, FINE>(acc, part, T.ntile, ti);
}

// ---------------------------------------------------------------------------------------------
// BiCGStab of small segments with uniform rows of three or four slots, one block per segment and component and
// the whole solve in one launch (as k_pcg_segment): the gathered vector (p, then s) and x in LDS, the rest and
// the scaled rows in registers.  Same sums in the same order as the kernels above, so the same bits.  Six
// barriers and three reductions an iteration instead of five kernels.  Ten PISO steps replayed from a graph (each with
// one solve of three components, some five iterations, and with the launches that make and copy the solvers' states
// gone): 968 / 1,922 / 2,178 / 4,050 prisms 2.95 / 3.61 / 4.58 / 6.92 -> 2.05 / 2.78 / 3.36 / 6.19 ms.
// Block (s, c) writes its component's fields of the segment's state; the first launch makes them.
// ---------------------------------------------------------------------------------------------
template <int NT, int C, int W>
__global__ __launch_bounds__(NT) void k_bi_segment(SellView A, Tiles T, int nc, const double* __restrict__ b,
                                                   double* __restrict__ x, double* __restrict__ rbuf,
                                                   double* __restrict__ hbuf, double* __restrict__ pbuf, double tol,
                                                   int maxit, int chunk, bool first, BiState* sts) {
  constexpr int NTILE = NT * C / TILE, WAVES = NT / 64;
  static_assert(NTILE <= 4, "the tiles' sums fill one wave");
  __shared__ double sp[C * NT], sx[C * NT];
  __shared__ double gs[3][64];
  const int s = blockIdx.x / nc, comp = blockIdx.x % nc, tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  BiState* st = sts + s;
  if (!first && !st->active[comp]) return;
  const int f = seg_first(T, s), nt = seg_count(T, s);
  const TileIdx t0 = tile_at(T, f), t1 = tile_at(T, f + nt - 1);
  const int lo = t0.lo, n = t1.hi - lo;  // the segment's cells are consecutive
  auto totals = [&](auto&& v, auto& tot) {  // as in k_pcg_segment
#pragma clang fp contract(off)
    constexpr int NV = sizeof(tot) / sizeof(double);
    wave_sums<NV * C>([&](int e) { return e % C * NT + tid < n ? v(e / C, e % C) : 0.0; },
                      [&](int e, double sum) { gs[e / C][e % C * WAVES + wid] = sum; });
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      double t = row_sum(gs[k][lane]);
      if (lane / TILE_WAVES >= nt) t = 0.0;
      t = swap_add16(t, t);
      tot[k] = wave_first(NTILE > 2 ? swap_add32(t, t) : t);
    }
  };
  double av[C][W], r[C], rh[C], p[C], v[C], t[C], d[C];
  int jv[C][W];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    // cells past the segment: an empty row
    const int me = c * NT + tid;
    const bool in = me < n;
    const int i = in ? lo + me : lo, base = (i >> 6) * (SLICE * W) + (i & (SLICE - 1));  // uniform rows
#pragma unroll
    for (int k = 0; k < W; ++k) {
      const double a = A.val[base + k * SLICE];
      const int j = A.off16[base + k * SLICE];
      av[c][k] = in ? a : 0.0;
      jv[c][k] = me + (in ? j : 0);
    }
    const size_t at = (size_t)i * nc + comp;
    d[c] = in ? A.diag[i] : 1.0;
    sx[me] = in ? x[at] : 0.0;
    sp[me] = sx[me];
    r[c] = in ? (first ? b[at] : rbuf[at]) : 0.0;
    rh[c] = in && !first ? hbuf[at] : 0.0;
    p[c] = in && !first ? pbuf[at] : 0.0;
  }
  // out(c, own[c] + off-diagonals of row c on the vector in sp)
  auto rows = [&](auto&& own, auto&& out) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      double acc = own(c);
#pragma unroll
      for (int k = 0; k < W; ++k) acc = __builtin_fma(av[c][k], sp[jv[c][k]], acc);
      out(c, acc);
    }
  };
  double one[1], two[2], three[3], bn, rho, res;
  int it = 1, status = 0;
  bool active = true, bad = false;
  if (first) {
    __syncthreads();
    double bv[C];
    rows([&](int c) { return d[c] * sp[c * NT + tid]; },
         [&](int c, double ax) {
           bv[c] = r[c];
           r[c] = rh[c] = p[c] = c * NT + tid < n ? bv[c] - ax : 0.0;
         });
    totals([&](int k, int c) { return k == 0 ? bv[c] * bv[c] : r[c] * r[c]; }, two);
    bn = sqrt(two[0]);
    const double rn = sqrt(two[1]);
    rho = two[1];
    res = bn == 0.0 ? 0.0 : rn / bn;
    active = !(bn == 0.0 || rn <= tol * bn);
    if (active && maxit <= 0) {
      active = false;
      status = DIFVM_WARN_NOT_CONVERGED;
    } else if (active && rho == 0.0) {
      active = false;
      status = DIFVM_WARN_BREAKDOWN;
    }
    if (tid == 0) {
      if (comp == 0) {
        st->tol = tol;
        st->maxit = maxit;
        st->any = 0;
      }
      st->bn[comp] = bn;
      st->res[comp] = res;
      st->iters[comp] = 0;
      st->next[comp] = 1;
      st->rho[comp] = rho;
      st->status[comp] = status;
      st->active[comp] = active ? 1 : 0;
    }
    if (bn == 0.0)
#pragma unroll
      for (int c = 0; c < C; ++c)
        if (const int me = c * NT + tid; me < n) x[(size_t)(lo + me) * nc + comp] = 0.0;
    if (!active) return;
    // columns scaled by 1/d, through sp (the sums' barrier is behind the last reads)
#pragma unroll
    for (int c = 0; c < C; ++c) sp[c * NT + tid] = d[c];
    __syncthreads();
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int k = 0; k < W; ++k) av[c][k] = av[c][k] / sp[jv[c][k]];
  } else {
#pragma unroll
    for (int c = 0; c < C; ++c) sp[c * NT + tid] = d[c];
    __syncthreads();
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int k = 0; k < W; ++k) av[c][k] = av[c][k] / sp[jv[c][k]];
    bn = st->bn[comp];
    rho = st->rho[comp];
    res = st->res[comp];
    it = st->next[comp];
  }
  __syncthreads();
  for (int made = 0; active && made < chunk; ++made, ++it) {
#pragma unroll
    for (int c = 0; c < C; ++c) sp[c * NT + tid] = p[c];
    __syncthreads();
    rows([&](int c) { return p[c]; }, [&](int c, double y) { v[c] = y; });
    totals([&](int, int c) { return rh[c] * v[c]; }, one);
    const double alpha = rho / one[0];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      r[c] = __builtin_fma(-alpha, v[c], r[c]);
      sp[c * NT + tid] = r[c];
    }
    __syncthreads();
    rows([&](int c) { return r[c]; }, [&](int c, double y) { t[c] = y; });
    totals([&](int k, int c) { return k == 0 ? t[c] * r[c] : k == 1 ? t[c] * t[c] : r[c] * r[c]; }, three);
    const double sn = sqrt(three[2]), omega = three[0] / three[1];
    const bool small = sn <= tol * bn;
    bad = !small && three[1] == 0.0;
    if (bad) {  // x, count and residual stay the previous iterate's
      active = false;
      status = DIFVM_WARN_BREAKDOWN;
      break;
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int me = c * NT + tid;
      const double y = p[c] / d[c], z = r[c] / d[c];
      sx[me] = __builtin_fma(alpha, y, small ? sx[me] : __builtin_fma(omega, z, sx[me]));
    }
    if (small) {
      active = false;
      res = sn / bn;
      break;
    }
#pragma unroll
    for (int c = 0; c < C; ++c) r[c] = __builtin_fma(-omega, t[c], r[c]);
    __syncthreads();  // gs is read
    totals([&](int k, int c) { return k == 0 ? r[c] * r[c] : rh[c] * r[c]; }, two);
    const double rn = sqrt(two[0]), rho_old = rho;
    res = rn / bn;
    if (rn <= tol * bn) {
      active = false;
      break;
    }
    if (it >= maxit) {
      active = false;
      status = DIFVM_WARN_NOT_CONVERGED;
      break;
    }
    rho = two[1];
    if (rho == 0.0) {
      active = false;
      status = DIFVM_WARN_BREAKDOWN;
      break;
    }
    const double beta = (rho / rho_old) * (alpha / omega);
#pragma unroll
    for (int c = 0; c < C; ++c) p[c] = __builtin_fma(beta, __builtin_fma(-omega, v[c], p[c]), r[c]);
  }
  if (tid == 0) {
    st->iters[comp] = active || bad ? it - 1 : it;
    st->res[comp] = res;
    st->status[comp] = status;
    st->active[comp] = active ? 1 : 0;
    st->rho[comp] = rho;
    st->next[comp] = it;
  }
#pragma unroll
  for (int c = 0; c < C; ++c)
    if (const int me = c * NT + tid; me < n) {
      const size_t at = (size_t)(lo + me) * nc + comp;
      x[at] = sx[me];
      if (active) {
        rbuf[at] = r[c];
        hbuf[at] = rh[c];
        pbuf[at] = p[c];
      }
    }
}

__global__ void k_bi_state_init(BiState* sts, int nseg, double tol, int maxit) {
  int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= nseg) return;
  BiState st{};
  st.tol = tol;
  st.maxit = maxit;
  sts[g] = st;
}

size_t bicgstab_state_bytes(const difvm_mesh* m) { return sizeof(BiState) * m->d.nseg; }

SolveResult bicgstab_result(const difvm_mesh* m, int ncomp, const void* host_state, bool* complete) {
  const BiState* hs = static_cast<const BiState*>(host_state);
  int nseg = m->d.nseg;
  SolveResult R;
  R.seg.resize(nseg);
  bool all = true;
  for (int g = 0; g < nseg; ++g) {
    const BiState& st = hs[g];
    for (int c = 0; c < ncomp; ++c) all = all && !st.active[c];
    SegResult& sr = R.seg[g];
    sr.status = 0;
    for (int c = 0; c < ncomp; ++c) {
      sr.iters[c] = st.iters[c];
      sr.res[c] = st.res[c];
      sr.status = std::max(sr.status, st.active[c] ? (int)DIFVM_WARN_NOT_CONVERGED : st.status[c]);
      R.iters[c] = std::max(R.iters[c], st.iters[c]);
      R.res[c] = std::max(R.res[c], st.res[c]);
    }
    R.status = std::max(R.status, sr.status);
  }
  if (complete) *complete = all;
  return R;
}

template <int W>
static auto bi_segment_kernel(int nt) {
  return nt == 1 ? k_bi_segment<256, 4, W>
         : nt == 2 ? k_bi_segment<256, 8, W>
         : nt == 3 ? k_bi_segment<512, 6, W>
                   : k_bi_segment<512, 8, W>;
}

template <int NC, bool FINE>
static SolveResult bicgstab_nc(difvm_mesh* m, SellMatrix A, const double* b, double* x, double tol, int maxit,
                               const QueueOnly* qo, int* hint) {
  KrylovWork* w = make_work(m);
  hipStream_t s = stream_of(m);
  SellView V = sview(m, A);
  Tiles T = tiles_of(m);
  constexpr int NT = FINE ? QUARTER : TILE;
  const int G = n_spans(m), nseg = m->d.nseg;
  const size_t bytes = bicgstab_state_bytes(m);
  if (const int nt = max_seg_tiles(m); nt <= SEG_TILES && V.off16 && (V.uw == 3 || V.uw == 4)) {
    const int budget = qo ? std::min(qo->budget, maxit) : maxit;
    BiState* sts = qo ? static_cast<BiState*>(qo->state_out) : w->bi;
    auto kernel = V.uw == 4 ? bi_segment_kernel<4>(nt) : bi_segment_kernel<3>(nt);
    int made = 0;
    do {
      const int chunk = std::min(SEG_CHUNK, budget - made);
      kernel<<<nseg * NC, nt <= 2 ? 256 : 512, 0, s>>>(V, T, NC, b, x, w->r, w->rh, w->p, tol, maxit, chunk, made == 0, sts);
      DIFVM_HIP(hipGetLastError());
      made += chunk;
      if (qo) continue;
      post_poll(m, w, sts, bytes, 0);
      const BiState* hs = static_cast<const BiState*>(wait_poll(w, 0));
      bool any = false;
      for (int g = 0; g < nseg; ++g)
        for (int c = 0; c < NC; ++c) any = any || hs[g].active[c];
      if (!any) break;
    } while (made < budget);
    if (qo) return SolveResult{};
    SolveResult R = bicgstab_result(m, NC, static_cast<const BiState*>(w->host_state[0]), nullptr);
    if (hint) *hint = std::max(R.iters[0], std::max(R.iters[1], R.iters[2]));
    return R;
  }
  k_bi_state_init<<<(nseg + 63) / 64, 64, 0, s>>>(w->bi, nseg, tol, maxit);
  double* partX = w->partials;
  double* partV = partX + 2 * NC * (size_t)G;
  double* partT = partV + NC * (size_t)G;
  double* tots = partX + 18 * (size_t)G;
  auto dir = [&](int it) {
    if (!FINE) k_bi_totals<2 * NC><<<nseg, TILE, 0, s>>>(partX, T, tots);
    k_bi_dir<NC, FINE><<<G, NT, 0, s>>>(T, it, w->r, w->p, w->v, x, FINE ? partX : tots, w->bi, nseg);
  };
  k_bi_init<NC, FINE><<<G, NT, 0, s>>>(V, T, b, x, w->r, w->rh, w->colscaled, partX);
  dir(1);
  DIFVM_HIP(hipGetLastError());
  int done = 0;  // iterations queued
  auto queue_iters = [&](int nb) {
    for (int n = 0; n < nb; ++n) {
      const int it = ++done;
      k_bi_v<NC, FINE><<<G, NT, 0, s>>>(V, w->colscaled, T, it, w->p, w->v, w->rh, partV, w->bi, nseg);
      if (!FINE) k_bi_totals<NC><<<nseg, TILE, 0, s>>>(partV, T, tots);
      k_bi_s<NC, FINE><<<G, NT, 0, s>>>(T, it, w->r, w->v, FINE ? partV : tots, w->bi, nseg);
      k_bi_t<NC, FINE><<<G, NT, 0, s>>>(V, w->colscaled, T, it, w->r, w->t, partT, w->bi, nseg);
      if (!FINE) k_bi_totals<3 * NC><<<nseg, TILE, 0, s>>>(partT, T, tots);
      k_bi_x<NC, FINE><<<G, NT, 0, s>>>(V, T, it, x, w->r, w->rh, w->p, w->t, FINE ? partT : tots, partX, w->bi, nseg);
      dir(it + 1);
    }
    DIFVM_HIP(hipGetLastError());
  };
  // the state after the iterations queued so far
  auto state = [&]() { return w->bi + (size_t)((done + 1) & 1) * nseg; };
  if (qo) {
    queue_iters(std::min(qo->budget, maxit));
    copy_state(qo->state_out, state(), bytes, s);
    return SolveResult{};
  }
  queue_iters(std::min(maxit, std::max(2, (hint ? *hint : 0) - 1)));
  int slot = 0;
  post_poll(m, w, state(), bytes, slot);
  const BiState* hs = nullptr;
  while (true) {
    bool more = done < maxit;
    if (more) {
      queue_iters(std::min(1, maxit - done));
      post_poll(m, w, state(), bytes, slot ^ 1);
    }
    hs = static_cast<const BiState*>(wait_poll(w, slot));
    bool any = false;
    for (int g = 0; g < nseg; ++g) any = any || hs[g].any;
    if (!any || !more) break;
    slot ^= 1;
  }
  SolveResult R = bicgstab_result(m, NC, hs, nullptr);
  if (hint) *hint = std::max(R.iters[0], std::max(R.iters[1], R.iters[2]));
  return R;
}

SolveResult bicgstab(difvm_mesh* m, int ncomp, SellMatrix A, const double* b, double* x, double tol, int maxit,
                     const QueueOnly* qo, int* hint) {
  const bool fine = fine_spans(m);
  if (ncomp == 1) return (fine ? bicgstab_nc<1, true> : bicgstab_nc<1, false>)(m, A, b, x, tol, maxit, qo, hint);
  return (fine ? bicgstab_nc<3, true> : bicgstab_nc<3, false>)(m, A, b, x, tol, maxit, qo, hint);
}

// ---------------------------------------------------------------------------------------------
// timing of the product kernel for the autotuner: `reps` launches at iteration 2 on scratch data
// (matrix values, vectors and partials set to constants, a control state that never stops), so no
// solve state is involved; returns seconds per launch
// ---------------------------------------------------------------------------------------------
__global__ void k_fill_const(double* __restrict__ a, size_t n, double v) {
  size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) a[q] = v;
}
__global__ void k_tune_ctl(PcgCtl* ctls, int nseg) {
  int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= nseg) return;
  PcgCtl c{};
  c.tol = 0.0;
  c.bn = 1.0;
  c.rho[0] = c.rho[1] = 1.0;
  c.maxit = 1 << 30;
  ctls[g] = c;
}

double time_pcg_spmv(difvm_mesh* m, int grid, int reps, hipEvent_t e0, hipEvent_t e1) {
  KrylovWork* w = make_work(m);
  hipStream_t s = stream_of(m);
  const DMesh& d = m->d;
  const Ctx& cx = ctx_of(m);
  double* val = dalloc<double>(cx, d.nslot);
  double* diag = nullptr;
  PcgCtl* ctl = nullptr;
  double t = 0.0;
  try {
    diag = dalloc<double>(cx, d.nc);
    ctl = static_cast<PcgCtl*>(dmalloc(cx, sizeof(PcgCtl) * d.nseg));
    auto fill = [&](double* a, size_t n, double v) {
      k_fill_const<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(a, n, v);
    };
    fill(val, d.nslot, -0.25);
    fill(diag, d.nc, 4.0);
    fill(w->z, d.nc, 1.0);
    fill(w->p, d.nc, 1.0);
    fill(w->partials, (size_t)8 * n_spans(m), 1.0);
    k_tune_ctl<<<(d.nseg + 63) / 64, 64, 0, s>>>(ctl, d.nseg);
    DIFVM_HIP(hipGetLastError());
    int old = m->tune[DIFVM_TUNE_PCG_GRID];
    m->tune[DIFVM_TUNE_PCG_GRID] = grid;
    int GS = pcg_spmv_launch_grid(m);
    m->tune[DIFVM_TUNE_PCG_GRID] = old;
    SellView V = sview(m, SellMatrix{diag, val});  // the same column form the solves read
    Tiles T = tiles_of(m);
    double* partA = w->partials;
    double* partB = w->partials + 2 * (size_t)n_spans(m);
    launch_pcg_spmv(GS, s, V, T, 2, w->z, w->p, w->v, w->q, partB, partA, ctl);
    DIFVM_HIP(hipEventRecord(e0, s));
    for (int r = 0; r < reps; ++r)
      launch_pcg_spmv(GS, s, V, T, 2, w->z, w->p, w->v, w->q, partB, partA, ctl);
    DIFVM_HIP(hipEventRecord(e1, s));
    DIFVM_HIP(hipGetLastError());
    DIFVM_HIP(hipEventSynchronize(e1));
    float ms = 0.f;
    DIFVM_HIP(hipEventElapsedTime(&ms, e0, e1));
    t = ms * 1e-3 / reps;
  } catch (...) {
    (void)hipStreamSynchronize(s);
    dfree(cx, val);
    dfree(cx, diag);
    dfree(cx, ctl);
    throw;
  }
  dfree(cx, val);
  dfree(cx, diag);
  dfree(cx, ctl);
  return t;
}

}  // namespace difvm
