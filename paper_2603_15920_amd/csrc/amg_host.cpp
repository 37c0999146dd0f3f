// Smoothed-aggregation algebraic multigrid hierarchy for the pressure matrix (plain C++, host side).
//
// The paper preconditions its pressure CG with ILU; on a GPU an incomplete factorisation runs as long
// chains of dependent triangular sweeps, so the library offers Jacobi (every iteration fully parallel)
// and, as a stronger option, a multigrid V-cycle whose every stage is a parallel sparse product.  The
// hierarchy is built once on the host from one pressure matrix (Vanek-Mandel-Brezina smoothed
// aggregation with the constant vector as near-null space) and then kept fixed: the finest level of
// each V-cycle uses the current matrix, the coarser levels the stored Galerkin operators, so the
// preconditioner stays symmetric positive definite for every solve.
#include "amg.h"
#include "host_rows.h"

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <numeric>
#include <vector>

namespace difvm {

namespace {

// Sparse accumulator for one row at a time: values summed per column, columns listed in ascending
// order when the row is flushed (or as they came).
struct SparseAcc {
  std::vector<double> acc;
  std::vector<int32_t> mark, touched;
  int32_t stamp = 0;
  explicit SparseAcc(int n) : acc(n, 0.0), mark(n, -1) {}
  void add(int I, double v) {
    if (mark[I] != stamp) {
      mark[I] = stamp;
      acc[I] = 0.0;
      touched.push_back(I);
    }
    acc[I] += v;
  }
  template <class F>
  void flush(F&& out, bool sorted = true) {
    if (sorted) std::sort(touched.begin(), touched.end());
    for (int I : touched) out(I, acc[I]);
    touched.clear();
    ++stamp;
  }
};

// CSR rows 0..n-1 (ptr, col, val) over n_cols columns: row(i, acc) adds row i's entries, keep(i, column,
// value) says whether an entry is stored
// a row takes 0.1 us (prolongator) to 2 us (product of a coarse level), starting a thread 20 us: with 256 rows a
// thread the setup of 49,536 cells takes 15.9 ms, with 1,024 18.8
constexpr int ROWS_PER_THREAD = 256;
template <class Row, class Keep>
void build_rows(int n, int n_cols, AmgCsr& C, bool sorted, Row&& row, Keep&& keep) {
  struct Part {
    std::vector<int32_t> col;
    std::vector<double> val;
  };
  std::vector<Part> part(n_chunks(n, ROWS_PER_THREAD));
  C.n = n;
  C.ptr.assign(n + 1, 0);
  parallel_rows(n, ROWS_PER_THREAD, [&](int t, int a, int b) {
    SparseAcc sa(n_cols);
    Part& P = part[t];
    for (int i = a; i < b; ++i) {
      row(i, sa);
      const size_t before = P.col.size();
      sa.flush(
          [&](int I, double v) {
            if (!keep(i, I, v)) return;
            P.col.push_back(I);
            P.val.push_back(v);
          },
          sorted);
      C.ptr[i + 1] = (int32_t)(P.col.size() - before);
    }
  });
  for (int i = 0; i < n; ++i) C.ptr[i + 1] += C.ptr[i];
  C.col.resize(C.ptr[n]);
  C.val.resize(C.ptr[n]);
  size_t at = 0;
  for (const Part& P : part) {
    std::copy(P.col.begin(), P.col.end(), C.col.begin() + at);
    std::copy(P.val.begin(), P.val.end(), C.val.begin() + at);
    at += P.col.size();
  }
}

// strong couplings of row i: |a_ij| >= theta sqrt(d_i d_j)
inline bool strong(double aij, double di, double dj, double theta) {
  return std::fabs(aij) >= theta * std::sqrt(std::fabs(di * dj));
}

// Three-phase greedy aggregation in row order.  Returns the number of aggregates; agg[i] in [0, n_agg).
int aggregate1(const AmgCsr& A, double theta, std::vector<int32_t>& agg) {
  const int n = A.n;
  agg.assign(n, -1);
  std::vector<char> phase1(n, 0);
  int na = 0;
  // phase 1: a root whose strong neighbourhood is entirely free takes it whole
  for (int i = 0; i < n; ++i) {
    if (agg[i] >= 0) continue;
    bool free = true;
    for (int q = A.ptr[i]; q < A.ptr[i + 1] && free; ++q) {
      int j = A.col[q];
      if (strong(A.val[q], A.diag[i], A.diag[j], theta) && agg[j] >= 0) free = false;
    }
    if (!free) continue;
    agg[i] = na;
    for (int q = A.ptr[i]; q < A.ptr[i + 1]; ++q) {
      int j = A.col[q];
      if (strong(A.val[q], A.diag[i], A.diag[j], theta)) agg[j] = na;
    }
    ++na;
  }
  for (int i = 0; i < n; ++i) phase1[i] = agg[i] >= 0;
  // phase 2: a free row joins the phase-1 aggregate it is most strongly coupled to
  std::vector<int32_t> join(n, -1);
  for (int i = 0; i < n; ++i) {
    if (phase1[i]) continue;
    double best = 0.0;
    for (int q = A.ptr[i]; q < A.ptr[i + 1]; ++q) {
      int j = A.col[q];
      if (!phase1[j] || !strong(A.val[q], A.diag[i], A.diag[j], theta)) continue;
      double s = std::fabs(A.val[q]);
      if (s > best) {
        best = s;
        join[i] = agg[j];
      }
    }
  }
  for (int i = 0; i < n; ++i)
    if (join[i] >= 0) agg[i] = join[i];
  // phase 3: what is left forms aggregates with its free strong neighbours (or alone)
  for (int i = 0; i < n; ++i) {
    if (agg[i] >= 0) continue;
    agg[i] = na;
    for (int q = A.ptr[i]; q < A.ptr[i + 1]; ++q) {
      int j = A.col[q];
      if (agg[j] < 0 && strong(A.val[q], A.diag[i], A.diag[j], theta)) agg[j] = na;
    }
    ++na;
  }
  return na;
}

// strong-connection graph squared (distance-2 neighbours), as a CSR pattern with unit values
AmgCsr strong_square(const AmgCsr& A, double theta) {
  const int n = A.n;
  std::vector<int32_t> sp(n + 1, 0), sc;
  for (int i = 0; i < n; ++i) {
    for (int q = A.ptr[i]; q < A.ptr[i + 1]; ++q)
      if (strong(A.val[q], A.diag[i], A.diag[A.col[q]], theta)) sc.push_back(A.col[q]);
    sp[i + 1] = (int32_t)sc.size();
  }
  AmgCsr G;
  G.n = n;
  G.ptr.assign(n + 1, 0);
  G.diag.assign(n, 1.0);
  std::vector<std::vector<int32_t>> part(n_chunks(n, ROWS_PER_THREAD));
  parallel_rows(n, ROWS_PER_THREAD, [&](int t, int a, int b) {
    std::vector<int32_t> mark(n, -1);
    std::vector<int32_t>& out = part[t];
    for (int i = a; i < b; ++i) {
      const size_t before = out.size();
      mark[i] = i;
      for (int q = sp[i]; q < sp[i + 1]; ++q) {
        int j = sc[q];
        if (mark[j] != i) { mark[j] = i; out.push_back(j); }
        for (int r = sp[j]; r < sp[j + 1]; ++r) {
          int k = sc[r];
          if (mark[k] != i) { mark[k] = i; out.push_back(k); }
        }
      }
      G.ptr[i + 1] = (int32_t)(out.size() - before);
    }
  });
  for (int i = 0; i < n; ++i) G.ptr[i + 1] += G.ptr[i];
  G.col.reserve(G.ptr[n]);
  for (const auto& c : part) G.col.insert(G.col.end(), c.begin(), c.end());
  G.val.assign(G.col.size(), 1.0);
  return G;
}

int aggregate(const AmgCsr& A, double theta, std::vector<int32_t>& agg, int radius) {
  if (radius <= 1) return aggregate1(A, theta, agg);
  AmgCsr G = strong_square(A, theta);
  return aggregate1(G, 0.0, agg);
}

// largest eigenvalue of D^-1 A by power iteration from a fixed start vector
double spectral_radius_dinv_a(const AmgCsr& A, int iters) {
  const int n = A.n;
  std::vector<double> v(n), w(n);
  for (int i = 0; i < n; ++i) v[i] = 1.0 + 0.5 * std::sin(0.7 * i + 0.3);  // deterministic, not constant
  double lam = 0.0, nv = 0.0;
  for (int i = 0; i < n; ++i) nv += v[i] * v[i];
  for (int it = 0; it < iters; ++it) {
    nv = std::sqrt(nv);
    if (nv == 0.0) return 1.0;
    for (int i = 0; i < n; ++i) v[i] /= nv;
    parallel_rows(n, 16384, [&](int, int a, int b) {
      for (int i = a; i < b; ++i) {
        double s = A.diag[i] * v[i];
        for (int q = A.ptr[i]; q < A.ptr[i + 1]; ++q) s += A.val[q] * v[A.col[q]];
        w[i] = s / A.diag[i];
      }
    });
    double num = 0.0;
    nv = 0.0;  // of the next iteration
    for (int i = 0; i < n; ++i) {
      num += v[i] * w[i];
      nv += w[i] * w[i];
    }
    lam = num;
    v.swap(w);
  }
  return std::max(lam, 1e-12);
}

// transpose of a CSR matrix with m columns
AmgCsr transpose(const AmgCsr& P, int m) {
  AmgCsr R;
  R.n = m;
  R.ptr.assign(m + 1, 0);
  for (int32_t c : P.col) R.ptr[c + 1]++;
  for (int I = 0; I < m; ++I) R.ptr[I + 1] += R.ptr[I];
  R.col.resize(P.col.size());
  R.val.resize(P.val.size());
  std::vector<int32_t> at(R.ptr.begin(), R.ptr.end() - 1);
  for (int i = 0; i < P.n; ++i)
    for (int q = P.ptr[i]; q < P.ptr[i + 1]; ++q) {
      int I = P.col[q];
      R.col[at[I]] = i;
      R.val[at[I]] = P.val[q];
      ++at[I];
    }
  return R;
}

}  // namespace

// One coarsening step: aggregates, smoothed prolongator P (fine rows), restriction R = P^T (coarse
// rows), Galerkin operator P^T A P (off-diagonals in CSR, diagonal apart, symmetrised exactly), the
// coarse near-null-space vector and, with_ap, A P with P's values on its pattern.
static bool coarsen(const AmgCsr& A, const std::vector<double>& B, double theta, int radius, bool with_ap,
                    AmgLevel& L, AmgCsr& Ac, std::vector<double>& Bc, std::vector<int32_t>& agg) {
  const int n = A.n;
  int na = aggregate(A, theta, agg, radius);
  if (na >= n || na == 0) return false;
  // tentative prolongator: the near-null-space vector restricted to each aggregate, normalised
  Bc.assign(na, 0.0);
  for (int i = 0; i < n; ++i) Bc[agg[i]] += B[i] * B[i];
  for (int I = 0; I < na; ++I) Bc[I] = std::sqrt(Bc[I]);
  std::vector<double> tent(n);
  for (int i = 0; i < n; ++i) tent[i] = Bc[agg[i]] > 0.0 ? B[i] / Bc[agg[i]] : 0.0;
  // smoothed prolongator P = (I - w D^-1 A) P_tent, w = 4 / (3 rho(D^-1 A))
  double w = 4.0 / (3.0 * spectral_radius_dinv_a(A, 20));
  if (with_ap) {
    // upper end of the level's Chebyshev smoothing interval: 1.1 times a longer power iteration's
    // estimate of rho(D^-1 A), at least 1.1 (the eigenvalues of D^-1 A average 1, so rho >= 1), capped
    // by the Gershgorin bound (discs around 1 of radius sum_j |a_ij| / a_ii), which always holds
    double g = 0.0;
    for (int i = 0; i < n; ++i) {
      double off = 0.0;
      for (int q = A.ptr[i]; q < A.ptr[i + 1]; ++q) off += std::fabs(A.val[q]);
      g = std::max(g, 1.0 + off / A.diag[i]);
    }
    L.hi = std::min(g, 1.1 * std::max(1.0, spectral_radius_dinv_a(A, 50)));
  }
  auto all = [](int, int, double) { return true; };
  AmgCsr& P = L.P;
  build_rows(
      n, na, P, true,
      [&](int i, SparseAcc& sa) {
        double s = w / A.diag[i];
        sa.add(agg[i], tent[i] - s * A.diag[i] * tent[i]);
        for (int q = A.ptr[i]; q < A.ptr[i + 1]; ++q) {
          int j = A.col[q];
          sa.add(agg[j], -s * A.val[q] * tent[j]);
        }
      },
      all);
  L.R = transpose(P, na);
  // A P by fine rows (A = diag + off-diagonals)
  AmgCsr AP;
  build_rows(
      n, na, AP, true,
      [&](int i, SparseAcc& sa) {
        for (int q = P.ptr[i]; q < P.ptr[i + 1]; ++q) sa.add(P.col[q], A.diag[i] * P.val[q]);
        for (int q = A.ptr[i]; q < A.ptr[i + 1]; ++q) {
          int j = A.col[q];
          for (int r = P.ptr[j]; r < P.ptr[j + 1]; ++r) sa.add(P.col[r], A.val[q] * P.val[r]);
        }
      },
      all);
  // A_c = R (A P) by coarse rows
  Ac.diag.assign(na, 0.0);
  const AmgCsr& R = L.R;
  build_rows(
      na, na, Ac, true,
      [&](int I, SparseAcc& sa) {
        for (int q = R.ptr[I]; q < R.ptr[I + 1]; ++q) {
          int i = R.col[q];
          double r = R.val[q];
          for (int s2 = AP.ptr[i]; s2 < AP.ptr[i + 1]; ++s2) sa.add(AP.col[s2], r * AP.val[s2]);
        }
      },
      [&](int I, int J, double v) {
        if (J == I) Ac.diag[I] = v;
        return J != I;
      });
  if (with_ap) {
    L.P_on_AP.assign(AP.val.size(), 0.0);
    for (int i = 0; i < n; ++i) {
      int q = P.ptr[i];
      for (int k = AP.ptr[i]; k < AP.ptr[i + 1] && q < P.ptr[i + 1]; ++k)
        if (P.col[q] == AP.col[k]) L.P_on_AP[k] = P.val[q++];
      if (q != P.ptr[i + 1]) throw AmgError{"prolongator pattern not inside that of A P"};
    }
    L.AP = std::move(AP);
  }
  // exact symmetry: a_IJ and a_JI replaced by their mean (rounding made them differ in the last bits)
  AmgCsr T = transpose(Ac, na);
  std::vector<double> sym(Ac.val.size());
  for (int I = 0; I < na; ++I) {
    // rows of Ac and of its transpose hold the same column set (the pattern is symmetric)
    int a = Ac.ptr[I], b = T.ptr[I];
    for (; a < Ac.ptr[I + 1]; ++a) {
      while (b < T.ptr[I + 1] && T.col[b] < Ac.col[a]) ++b;
      double t = (b < T.ptr[I + 1] && T.col[b] == Ac.col[a]) ? T.val[b] : 0.0;
      sym[a] = 0.5 * (Ac.val[a] + t);
    }
  }
  Ac.val.swap(sym);
  return true;
}

void amg_build(const AmgCsr& A0, const AmgOptions& opt, AmgHierarchy& H) {
  H.levels.clear();
  H.coarse.clear();
  H.coarsest_dense.clear();
  std::vector<double> B(A0.n, 1.0);
  AmgCsr A = A0;
  for (int l = 0; l < opt.max_levels; ++l) {
    if (A.n <= (l == 0 ? opt.tiny : opt.coarsest)) break;
    AmgLevel L;
    AmgCsr Ac;
    std::vector<double> Bc;
    std::vector<int32_t> agg;
    if (!coarsen(A, B, l == 0 ? opt.theta_fine : opt.theta, l == 0 ? opt.radius_fine : opt.radius, l > 0, L, Ac, Bc,
                 agg))
      break;
    if (l == 0) H.agg0 = agg;
    if (Ac.n > (int)(0.85 * A.n)) break;  // no real coarsening: stop here
    H.levels.push_back(std::move(L));
    H.coarse.push_back(Ac);
    A = std::move(Ac);
    B = std::move(Bc);
  }
  if (H.levels.empty()) throw AmgError{"the matrix does not coarsen"};
  if (A.n > opt.max_dense) throw AmgError{"coarsest AMG level too large for the dense solve"};
  H.n_coarsest = A.n;
  const size_t n = A.n;
  H.coarsest_dense.assign(n * n, 0.0);
  for (size_t i = 0; i < n; ++i) {
    H.coarsest_dense[i * n + i] = A.diag[i];
    for (int q = A.ptr[i]; q < A.ptr[i + 1]; ++q) H.coarsest_dense[i * n + A.col[q]] = A.val[q];
  }
}

Cheb cheb_coefficients(double lo, double hi) {
  double theta = 0.5 * (hi + lo), delta = 0.5 * (hi - lo);
  double sigma = theta / delta, rho0 = 1.0 / sigma, rho1 = 1.0 / (2.0 * sigma - rho0);
  return {theta, 1.0 / theta, rho1 * rho0, 2.0 * rho1 / delta};
}

// C = X + s Y diag(d)^-1 Z for CSR matrices of whole rows (nothing apart), n_cols columns
static AmgCsr add_product(const AmgCsr& X, double s, const AmgCsr& Y, const std::vector<double>* d, const AmgCsr& Z,
                          int n_cols) {
  AmgCsr C;
  build_rows(
      Y.n, n_cols, C, false,
      [&](int i, SparseAcc& sa) {
        if (X.n)
          for (int q = X.ptr[i]; q < X.ptr[i + 1]; ++q) sa.add(X.col[q], X.val[q]);
        for (int q = Y.ptr[i]; q < Y.ptr[i + 1]; ++q) {
          const int j = Y.col[q];
          const double y = s * Y.val[q] / (d ? (*d)[j] : 1.0);
          for (int r = Z.ptr[j]; r < Z.ptr[j + 1]; ++r) sa.add(Z.col[r], y * Z.val[r]);
        }
      },
      [](int, int, double) { return true; });
  return C;
}

AmgFused amg_fuse(const AmgHierarchy& H, bool two) {
  const size_t l = H.levels.size() - 1;
  const AmgLevel& L = H.levels[l];
  const AmgCsr& A = H.coarse[l - 1];
  const int n = A.n, n2 = H.n_coarsest;
  AmgFused F;
  const Cheb c = cheb_coefficients(0.1 * L.hi, L.hi);
  F.alpha = (1.0 + c.c_d) * c.inv_theta + c.c_r;
  F.beta = c.c_r * c.inv_theta;
  AmgCsr W, X = L.AP;  // A with its diagonal in the rows; D (P - alpha D^-1 A P) on the pattern of A P
  W.n = n;
  W.ptr.assign(1, 0);
  W.col.reserve(A.col.size() + n);
  W.val.reserve(A.val.size() + n);
  for (int i = 0; i < n; ++i) {
    W.col.push_back(i);
    W.val.push_back(A.diag[i]);
    W.col.insert(W.col.end(), A.col.begin() + A.ptr[i], A.col.begin() + A.ptr[i + 1]);
    W.val.insert(W.val.end(), A.val.begin() + A.ptr[i], A.val.begin() + A.ptr[i + 1]);
    W.ptr.push_back((int32_t)W.col.size());
    for (int q = X.ptr[i]; q < X.ptr[i + 1]; ++q) X.val[q] = A.diag[i] * L.P_on_AP[q] - F.alpha * L.AP.val[q];
  }
  F.G = add_product(X, F.beta, W, &A.diag, L.AP, n2);  // D G
  for (int i = 0; i < n; ++i)
    for (int q = F.G.ptr[i]; q < F.G.ptr[i + 1]; ++q) F.G.val[q] /= A.diag[i];
  if (!two) {
    F.GT = transpose(F.G, n2);
    return F;
  }
  X = W;  // D - alpha A
  for (size_t q = 0; q < X.val.size(); ++q) X.val[q] *= -F.alpha;
  for (int i = 0; i < n; ++i) X.val[X.ptr[i]] += A.diag[i];
  F.S = add_product(X, F.beta, W, &A.diag, W, n);
  F.RS = add_product(AmgCsr{}, 1.0, L.R, nullptr, F.S, n);
  return F;
}

}  // namespace difvm
