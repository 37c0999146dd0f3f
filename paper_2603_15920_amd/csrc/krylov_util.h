// Helpers shared by the Krylov solvers and the AMG V-cycle: the cell-slot matrix view, reduction
// tiles with deterministic per-segment sums, and the PCG control state.
#pragma once

#include "device.h"
#include "ops.h"

namespace difvm {

// ---------------------------------------------------------------------------------------------
// matrix helpers
// ---------------------------------------------------------------------------------------------
struct SellView {
  int nc;
  const uint8_t* __restrict__ nslot;
  const int32_t* __restrict__ slice_start;
  const int32_t* __restrict__ col;
  const double* __restrict__ val;
  const double* __restrict__ diag;
  const int16_t* __restrict__ off16;  // col - row in 16 bits (NULL when it does not fit)
  int uw;                             // uniform row width (0: rows of varying width)
};

inline SellView sview(const difvm_mesh* m, SellMatrix A) {
  return {m->d.nc, m->d.cell_nslot, m->d.slice_start, m->d.slot_col, A.val, A.diag, m->d.slot_off16, m->d.uw};
}

// ---------------------------------------------------------------------------------------------
// Reduction tiles: TILE = 1024 cells, listed per segment.  A segment is one
// independent mesh of a block-diagonal batch (a single mesh is one segment); its dot products are
// the fixed-order sums of its own tiles' partials, so a batch member computes exactly what it would
// alone.
// ---------------------------------------------------------------------------------------------
struct Tiles {
  int ntile;
  int one_nc;  // > 0: one segment of that many cells (tile t starts at cell t TILE), else 0
  const int32_t* __restrict__ lo;
  const int32_t* __restrict__ hi;
  const int32_t* __restrict__ seg;
  const int32_t* __restrict__ first;  // per segment
  const int32_t* __restrict__ count;  // per segment
};
inline Tiles tiles_of(const difvm_mesh* m) {
  const DMesh& d = m->d;
  return {d.ntile, d.nseg == 1 ? d.nc : 0, d.tile_lo, d.tile_hi, d.tile_seg, d.seg_tile_first, d.seg_tile_n};
}

struct TileIdx {
  int t, s, lo, hi;
};
// with one segment every index follows from t, so that no load waits for the tile tables
__device__ __forceinline__ TileIdx tile_at(const Tiles& T, int t) {
  if (T.one_nc > 0) return {t, 0, t * TILE, min(t * TILE + TILE, T.one_nc)};
  return {t, T.seg[t], T.lo[t], T.hi[t]};
}
// The cells of a block: a tile, or on meshes of at most FINE_TILES tiles a quarter of one.  A block of a
// whole tile gathers its rows' neighbours through one compute unit, which takes about one cache line a
// cycle: 8,192 of them (two vectors, four slots) are 3.4 us, and a mesh of 100 tiles leaves half the chip
// idle meanwhile.  Quarters cost the kernels that sum the partials four loads per tile instead of one.
constexpr int FINE_TILES = 384;
constexpr int QUARTER = TILE / 4;
struct Span {
  int t, j, s, lo, hi, end;  // tile, quarter (0), segment, cells [lo, hi) (hi <= lo: none), end of the tile
};
template <bool FINE>
__device__ __forceinline__ Span span_at(const Tiles& T, int b) {
  const int t = FINE ? b >> 2 : b, j = FINE ? b & 3 : 0;
  const TileIdx ti = tile_at(T, t);
  if constexpr (FINE) return {t, j, ti.s, ti.lo + j * QUARTER, min(ti.hi, ti.lo + (j + 1) * QUARTER), ti.hi};
  else return {t, 0, ti.s, ti.lo, ti.hi, ti.hi};
}
template <bool FINE>
__device__ __forceinline__ Span span_of(const Tiles& T) {
  return span_at<FINE>(T, xcd_tile(blockIdx.x, gridDim.x));
}
inline bool fine_spans(const difvm_mesh* m) { return m->d.ntile <= FINE_TILES; }
inline int n_spans(const difvm_mesh* m) { return fine_spans(m) ? 4 * m->d.ntile : m->d.ntile; }
__device__ __forceinline__ int seg_first(const Tiles& T, int s) { return T.one_nc > 0 ? 0 : T.first[s]; }
__device__ __forceinline__ int seg_count(const Tiles& T, int s) { return T.one_nc > 0 ? T.ntile : T.count[s]; }

// ---------------------------------------------------------------------------------------------
// Reductions.  Their order is the same whatever the shape of the launch: a tile's sum is the tree (row_sum)
// over its 16 groups of 64 consecutive cells, each the sum of the group's wave; a segment's total adds its
// tiles q in four chains (q / 64) mod 4, lane q mod 64 of each adding its own tiles in order, then a wave
// sum per chain and the four in order.  So a kernel may give a block a tile or a quarter of one, a thread
// one cell or several, or hold a whole segment in one block, with the same bits.
//
// Several values are summed over a wave by halving the set at each of the first steps (a lane keeps the
// half its lane bit names and gives away the other), which leaves one value per group of lanes after
// log2 P steps: 10 exchanges for 8 values instead of 48, each value with wave_sum's pairing and so its bits.
// ---------------------------------------------------------------------------------------------
constexpr int TILE_WAVES = TILE / 64;

// v[0..P) summed over the wave (P = 1, 2, 4, 8): value k ends in v[0] of the lanes k 64/P .. (k+1) 64/P - 1
template <int P>
__device__ __forceinline__ void wave_sum_split(double (&v)[P]) {
#pragma clang fp contract(off)
  static_assert(P <= 8, "at most eight values");
  constexpr int M32 = P > 1 ? P / 2 : 1, M16 = P > 2 ? P / 4 : 1;
#pragma unroll
  for (int k = 0; k < M32; ++k) v[k] = swap_add32(v[k], v[P > 1 ? k + M32 : k]);
#pragma unroll
  for (int k = 0; k < M16; ++k) v[k] = swap_add16(v[k], v[P > 2 ? k + M16 : k]);
  if constexpr (P == 8) {
    const bool up = threadIdx.x & 8;
    const double mine = up ? v[1] : v[0], send = up ? v[0] : v[1];
    v[0] = mine + dpp_mov<DPP_ROR8>(send);
  } else {
    v[0] += dpp_mov<DPP_ROR8>(v[0]);
  }
  v[0] = lanes_sum<8>(v[0]);
}

// wave sums of v(0..M-1) stored as out(k, sum); groups of 8 values, then what is left
template <int M, int K0 = 0, class V, class F>
__device__ __forceinline__ void wave_sums(V&& v, F&& out) {
  constexpr int N = M - K0, P = N > 4 ? 8 : N > 2 ? 4 : N;
  const int lane = threadIdx.x & 63;
  double a[P];
#pragma unroll
  for (int k = 0; k < P; ++k) a[k] = k < N ? v(K0 + (k < N ? k : 0)) : 0.0;
  wave_sum_split<P>(a);
  if (const int k = lane / (64 / P); lane % (64 / P) == 0 && k < N) out(K0 + k, a[0]);
  if constexpr (N > P) wave_sums<M, K0 + P>(v, out);
}

// the sums of NV values per cell over a block's span, by a block of NT threads with C cells each (thread tid
// holds cells tid + c NT of the span, value k of cell c in v[k C + c]): a tile's into part[k ntile + t], a
// quarter's (FINE, C = 1) into part[k 4 ntile + 4 t + j]
template <int NV, int NT, bool FINE>
__device__ __forceinline__ void put_partial(const double (&v)[NV * (FINE ? 1 : TILE / NT)], double* __restrict__ part,
                                            int ntile, const Span& sp) {
  constexpr int C = FINE ? 1 : TILE / NT, GROUPS = NT * C / 64, LANES = (NV * GROUPS + 63) / 64 * 64;
  static_assert(LANES <= NT && (FINE ? GROUPS == 4 : GROUPS == 16), "one lane per group sum");
  __shared__ double lds[LANES];
  const int wid = threadIdx.x >> 6;
  __syncthreads();  // a previous tile's sums are out of lds
  wave_sums<NV * C>([&](int e) { return v[e]; },
                    [&](int e, double sum) { lds[e / C * GROUPS + e % C * (NT / 64) + wid] = sum; });
  __syncthreads();
  if (threadIdx.x < LANES) {  // whole waves; lanes past the values sum what the array holds, unused
    const double s = FINE ? quad_sum(lds[threadIdx.x]) : row_sum(lds[threadIdx.x]);
    const int k = threadIdx.x / GROUPS;
    if (threadIdx.x % GROUPS == 0 && k < NV)
      part[FINE ? (size_t)k * 4 * ntile + 4 * sp.t + sp.j : (size_t)k * ntile + sp.t] = s;
  }
}

// the segment's totals of NV partials (n tiles from tile f, by tile or by quarter) for every thread of a
// block of NT threads; waves 4g .. 4g+3 take the four chains of the values g, g + NT / 256, ...; several
// loads of a lane in flight
template <int NV, int NT, bool FINE>
__device__ __forceinline__ void seg_totals(const double* __restrict__ part, int ntile, int f, int n,
                                           double (&tot)[NV]) {
#pragma clang fp contract(off)
  constexpr int G = NT / 256, K = (NV + G - 1) / G, UN = K > 2 ? 1 : K > 1 ? 2 : 4;
  __shared__ double sh[NV][4];
  const int lane = threadIdx.x & 63, chain = (threadIdx.x >> 6) & 3, g = threadIdx.x >> 8;
  double s[K];
#pragma unroll
  for (int k = 0; k < K; ++k) s[k] = 0.0;
  for (int q = 64 * chain + lane; q < n; q += UN * 256) {
    double w[UN][K];
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int k = 0; k < K; ++k) {  // past the end (tiles or values) the last one, not added
        const size_t at = (size_t)min(g + k * G, NV - 1) * ntile + f + min(q + u * 256, n - 1);
        if constexpr (FINE) {
          const double2 *h = reinterpret_cast<const double2*>(part) + 2 * at, a = h[0], b = h[1];
          w[u][k] = (a.x + a.y) + (b.x + b.y);
        } else {
          w[u][k] = part[at];
        }
      }
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (q + u * 256 < n) s[k] += w[u][k];
  }
  __syncthreads();  // a previous call's totals have been read
#pragma unroll
  for (int k = 0; k < K; ++k) {
    s[k] = wave_sum(s[k]);
    if (lane == 0 && g + k * G < NV) sh[g + k * G][chain] = s[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NV; ++k) tot[k] = ((sh[k][0] + sh[k][1]) + sh[k][2]) + sh[k][3];
}

constexpr int SEG_TILES = 4;  // most tiles of a segment whose whole solve one block makes
// per-segment PCG state (device)
struct PcgCtl {
  double tol, bn, res;
  double rho[2];  // rho_k at index k & 1
  double rr;      // r.r between two launches of a solve in one block
  int maxit, done, iters, status;
  int next, pad;  // iterations made by those launches so far
};
__device__ __forceinline__ void ctl_start(PcgCtl* ctl, double tol, int maxit) {
  PcgCtl c{};
  c.tol = tol;
  c.maxit = maxit;
  *ctl = c;
}

}  // namespace difvm
