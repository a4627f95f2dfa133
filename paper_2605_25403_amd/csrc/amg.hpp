// Multigrid preconditioner of the pressure Poisson CG, host side: a smoothed
// aggregation hierarchy (Vanek, Mandel and Brezina 1996) of the pressure
// stiffness matrix Kp (Section 2.2.1, eq. (9), second line), built once per
// mesh and flattened into a few sparse products.
//
// One symmetric V(1,1) cycle with damped Jacobi smoothing is, on level k with
// S = I - w D^{-1} A,
//   B_k r = Lam_k r + Q_k B_{k+1} Q_k^T r,
//   Lam = w (2 I - w D^{-1} A) D^{-1},  Q = S P,
// P = (I - w_p D^{-1} A) T the smoothed prolongator over the aggregates T: the
// cycle's smoothing steps move into Q, which is formed here once (small plane
// meshes: a V(2,2) cycle, Q = S^2 P, Lam = w (I + S + S^2 + S^3) D^{-1}). Written out,
// the levels no longer wait for one another on the way down and up:
//   e_k = Lam_k r_k with r_k = (Q_b ... Q_{k-1})^T r_b,
//   B r_b = Lam_b r_b + sum_k (Q_b ... Q_{k-1}) e_k,
// so the cycle below any base level b is three products whatever the number of
// levels: all restrictions from r_b, all Lam_k (and the dense inverse of the
// last level), and one row [Lam_b | Q_b | Q_b Q_{b+1} | ...] per unknown of
// level b. A kernel boundary costs about 2.5 us on this GPU, a composed
// product of a few hundred thousand entries less, so that form is taken from
// the finest level (b = 0, three products) where its entries are few, and from
// the second one (b = 1, five products) on large meshes, where the composed
// products of the finest level would cost more traffic than two launches.
//
// Part of parts.cpp (the mesh's host data).
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <exception>
#include <memory>
#include <vector>

#ifdef _OPENMP
#include <omp.h>
#endif

#include "mesh.hpp"

namespace ipcs {
namespace amg {

struct Csr {
  int64_t n = 0, m = 0;            // rows, columns
  std::vector<int32_t> rp;         // [n + 1]
  RawVec<int32_t> col;
  RawVec<double> val;
  int64_t nnz() const { return rp.empty() ? 0 : rp.back(); }
};

inline int max_threads() {
#ifdef _OPENMP
  return omp_get_max_threads();
#else
  return 1;
#endif
}

// Runs f(t) for t in [0, nt), one thread each. An exception (memory that runs out
// inside f) may not leave a parallel region: the first one is thrown after it.
template <class F>
void team(int nt, F f) {
  std::exception_ptr first;
#pragma omp parallel for num_threads(nt) schedule(static, 1)
  for (int t = 0; t < nt; ++t) {
    try {
      f(t);
    } catch (...) {
#pragma omp critical(ipcs_amg_team)
      if (!first) first = std::current_exception();
    }
  }
  if (first) std::rethrow_exception(first);
}

// Runs f(t, lo, hi) over contiguous ranges of [0, n), one per thread.
template <class F>
void ranges(int64_t n, F f) {
  const int nt = (int)std::min<int64_t>(max_threads(), std::max<int64_t>(1, n / 512));
  team(nt, [&](int t) { f(t, n * t / nt, n * (t + 1) / nt); });
}

// Row pointers from the row lengths held in C.rp[1..], and room for the
// entries (not filled). False if they exceed the 32-bit index range.
inline bool allocate(Csr& C) {
  int64_t at = 0;
  C.rp[0] = 0;
  for (int64_t i = 0; i < C.n; ++i) {
    at += C.rp[i + 1];
    if (at >= (int64_t(1) << 31)) {
      C = Csr{};
      return false;
    }
    C.rp[i + 1] = (int32_t)at;
  }
  C.col.alloc((size_t)at);
  C.val.alloc((size_t)at);
  return true;
}

// X + diag(d) (A B) (X null: none; d null: ones), columns in first-seen order;
// empty (n = 0) if it has too many entries
inline Csr product(const Csr& A, const Csr& B, const Csr* X = nullptr, const double* d = nullptr) {
  Csr C;
  C.n = A.n;
  C.m = B.m;
  C.rp.assign(C.n + 1, 0);
  ranges(C.n, [&](int, int64_t lo, int64_t hi) {
    std::vector<int32_t> seen(B.m, -1);
    for (int64_t i = lo; i < hi; ++i) {
      int32_t k = 0;
      auto mark = [&](const Csr& Y, int64_t r) {
        for (int32_t q = Y.rp[r]; q < Y.rp[r + 1]; ++q)
          if (seen[Y.col[q]] != (int32_t)i) {
            seen[Y.col[q]] = (int32_t)i;
            ++k;
          }
      };
      if (X) mark(*X, i);
      for (int32_t p = A.rp[i]; p < A.rp[i + 1]; ++p) mark(B, A.col[p]);
      C.rp[i + 1] = k;
    }
  });
  if (!allocate(C)) return C;
  ranges(C.n, [&](int, int64_t lo, int64_t hi) {
    std::vector<int32_t> at(B.m, -1);
    for (int64_t i = lo; i < hi; ++i) {
      const int32_t base = C.rp[i];
      int32_t k = base;
      auto add = [&](int32_t j, double w) {
        if (at[j] < base) {   // not seen in this row (rows come in order)
          at[j] = k;
          C.col[k] = j;
          C.val[k] = w;
          ++k;
        } else {
          C.val[at[j]] += w;
        }
      };
      if (X)
        for (int32_t q = X->rp[i]; q < X->rp[i + 1]; ++q) add(X->col[q], X->val[q]);
      const double s = d ? d[i] : 1.0;
      for (int32_t p = A.rp[i]; p < A.rp[i + 1]; ++p) {
        const double a = s * A.val[p];
        const int32_t r = A.col[p];
        for (int32_t q = B.rp[r]; q < B.rp[r + 1]; ++q) add(B.col[q], a * B.val[q]);
      }
    }
  });
  return C;
}

// A^T; within a row the entries follow A's rows (each thread counts and then
// places the entries of its own range of A's rows)
inline Csr transpose(const Csr& A) {
  Csr T;
  T.n = A.m;
  T.m = A.n;
  T.rp.assign(T.n + 1, 0);
  T.col.alloc(A.nnz());
  T.val.alloc(A.nnz());
  const int nt = (int)std::min<int64_t>(max_threads(), std::max<int64_t>(1, A.n / 4096));
  std::vector<std::vector<int32_t>> pos(nt);
  team(nt, [&](int t) {
    pos[t].assign(T.n, 0);
    for (int32_t q = A.rp[A.n * t / nt]; q < A.rp[A.n * (t + 1) / nt]; ++q) pos[t][A.col[q]] += 1;
  });
  int32_t at = 0;
  for (int64_t i = 0; i < T.n; ++i) {
    T.rp[i] = at;
    for (int t = 0; t < nt; ++t) {
      const int32_t c = pos[t][i];
      pos[t][i] = at;
      at += c;
    }
  }
  T.rp[T.n] = at;
  team(nt, [&](int t) {
    for (int64_t i = A.n * t / nt; i < A.n * (t + 1) / nt; ++i)
      for (int32_t q = A.rp[i]; q < A.rp[i + 1]; ++q) {
        const int32_t k = pos[t][A.col[q]]++;
        T.col[k] = (int32_t)i;
        T.val[k] = A.val[q];
      }
  });
  return T;
}

inline std::vector<double> diagonal(const Csr& A) {
  std::vector<double> d(A.n, 0.0);
  for (int64_t i = 0; i < A.n; ++i)
    for (int32_t q = A.rp[i]; q < A.rp[i + 1]; ++q)
      if (A.col[q] == i) d[i] = A.val[q];
  return d;
}

// Estimate of the largest eigenvalue of D^{-1} A: 16 power iterations from a fixed
// rough start, times 1.06. On squares, strips, cubes and boxes of both spaces it
// lies between 0.97 and 1.03 of the eigenvalue; the weights 1.62 and 4/3 over the
// estimate stay below 2 over the eigenvalue, as the smoothing steps need, down to
// estimates of 0.81 of it. The norms are summed chunk by chunk, so the
// result, and with it every bit of the hierarchy, is the same whatever the
// number of threads.
inline double lambda_max(const Csr& A, const std::vector<double>& dinv) {
  constexpr int64_t kChunk = 2048;
  const int64_t nc = (A.n + kChunk - 1) / kChunk;
  std::vector<double> x(A.n), y(A.n), xs(nc), ys(nc);
  for (int64_t i = 0; i < A.n; ++i) {   // a fixed sequence without structure
    const uint32_t h = (uint32_t)i * 2654435761u;
    x[i] = ((h >> 8) & 0xffff) / 65536.0 - 0.5;
  }
  double l = 1.0, f = 1.0;
  for (int it = 0; it < 16; ++it) {
#pragma omp parallel for schedule(static) if (nc > 1)
    for (int64_t c = 0; c < nc; ++c) {
      double xx = 0.0, yy = 0.0;
      for (int64_t i = c * kChunk; i < std::min(A.n, (c + 1) * kChunk); ++i) {
        double s = 0.0;
        for (int32_t q = A.rp[i]; q < A.rp[i + 1]; ++q) s += A.val[q] * x[A.col[q]];
        y[i] = f * dinv[i] * s;
        xx += f * x[i] * f * x[i];
        yy += y[i] * y[i];
      }
      xs[c] = xx;
      ys[c] = yy;
    }
    double xx = 0.0, yy = 0.0;
    for (int64_t c = 0; c < nc; ++c) {
      xx += xs[c];
      yy += ys[c];
    }
    if (!(yy > 0.0) || !std::isfinite(yy)) return 0.0;
    l = std::sqrt(yy / xx);
    f = 1.0 / std::sqrt(yy);   // scales the next pass's input
    x.swap(y);
  }
  return 1.06 * l;
}

// Aggregates of the graph of strong connections |a_ij| >= theta sqrt(a_ii a_jj):
// a root takes its whole free neighbourhood, what is left joins the aggregate
// it is most strongly tied to. Returns the count; agg[i] in [0, count).
inline int64_t aggregate(const Csr& A, const std::vector<double>& diag, double theta,
                         std::vector<int32_t>& agg) {
  const int64_t n = A.n;
  std::vector<double> rd(n);
  for (int64_t i = 0; i < n; ++i) rd[i] = std::sqrt(std::fabs(diag[i]));
  auto strong = [&](int64_t i, int32_t q) {
    const int32_t j = A.col[q];
    return j != i && std::fabs(A.val[q]) >= theta * rd[i] * rd[j];
  };
  agg.assign(n, -1);
  int32_t na = 0;
  for (int64_t i = 0; i < n; ++i) {
    if (agg[i] >= 0) continue;
    bool open = true;
    for (int32_t q = A.rp[i]; q < A.rp[i + 1] && open; ++q)
      if (strong(i, q)) open = agg[A.col[q]] < 0;
    if (!open) continue;
    agg[i] = na;
    for (int32_t q = A.rp[i]; q < A.rp[i + 1]; ++q)
      if (strong(i, q)) agg[A.col[q]] = na;
    ++na;
  }
  const std::vector<int32_t> first = agg;
  for (int64_t i = 0; i < n; ++i) {
    if (agg[i] >= 0) continue;
    double best = -1.0;
    for (int32_t q = A.rp[i]; q < A.rp[i + 1]; ++q)
      if (strong(i, q) && first[A.col[q]] >= 0) {
        const double w = std::fabs(A.val[q]) / rd[A.col[q]];
        if (w > best) {
          best = w;
          agg[i] = first[A.col[q]];
        }
      }
  }
  for (int64_t i = 0; i < n; ++i) {
    if (agg[i] >= 0) continue;
    agg[i] = na;
    for (int32_t q = A.rp[i]; q < A.rp[i + 1]; ++q)
      if (strong(i, q) && agg[A.col[q]] < 0) agg[A.col[q]] = na;
    ++na;
  }
  return na;
}

// Inverse of the last level's matrix; a singular one is made definite on the
// constants it does not see (Kp 1 = 0, and P keeps constants on every level). False if the
// matrix is not positive.
inline bool coarse_inverse(const Csr& A, bool singular, Csr& B) {
  const int64_t n = A.n;
  std::vector<double> L(n * n, 0.0), inv(n * n, 0.0);
  double dm = 0.0;
  for (int64_t i = 0; i < n; ++i)
    for (int32_t q = A.rp[i]; q < A.rp[i + 1]; ++q) {
      L[i * n + A.col[q]] += A.val[q];
      if (A.col[q] == i) dm += A.val[q] / n;
    }
  if (singular)
    for (double& v : L) v += dm / n;
  for (int64_t j = 0; j < n; ++j) {          // Cholesky, rows of L
    for (int64_t i = j; i < n; ++i) {
      double s = L[i * n + j];
      for (int64_t k = 0; k < j; ++k) s -= L[i * n + k] * L[j * n + k];
      if (i == j) {
        if (!(s > 1e-12 * dm)) return false;
        L[j * n + j] = std::sqrt(s);
      } else {
        L[i * n + j] = s / L[j * n + j];
      }
    }
  }
  // inv row c: column c of the inverse (symmetric)
#pragma omp parallel for schedule(static) if (n > 64)
  for (int64_t c = 0; c < n; ++c) {
    double* x = inv.data() + c * n;
    x[c] = 1.0;
    for (int64_t i = c; i < n; ++i) {
      double s = x[i];
      for (int64_t k = c; k < i; ++k) s -= L[i * n + k] * x[k];
      x[i] = s / L[i * n + i];
    }
    for (int64_t i = n - 1; i >= 0; --i) {
      double s = x[i];
      for (int64_t k = i + 1; k < n; ++k) s -= L[k * n + i] * x[k];
      x[i] = s / L[i * n + i];
    }
  }
  B.n = B.m = n;
  B.rp.resize(n + 1);
  B.col.alloc(n * n);
  B.val.alloc(n * n);
  for (int64_t i = 0; i <= n; ++i) B.rp[i] = (int32_t)(i * n);
  for (int64_t i = 0; i < n; ++i)
    for (int64_t j = 0; j < n; ++j) {
      B.col[i * n + j] = (int32_t)j;
      B.val[i * n + j] = 0.5 * (inv[i * n + j] + inv[j * n + i]);
    }
  return true;
}

struct Level {
  Csr A, Q;                        // matrix; Q = S^m P to the next level (empty on the last)
  std::vector<double> dinv;
  double omega = 0.0;
};

// f(q, p) for every entry p of Sub, q the entry of Big at its place (the pattern
// of Big holds Sub's); rows in parallel.
template <class F>
void each_match(const Csr& Big, const Csr& Sub, F f) {
  ranges(Big.n, [&](int, int64_t lo, int64_t hi) {
    std::vector<int32_t> at(Big.m, 0);
    for (int64_t i = lo; i < hi; ++i) {
      for (int32_t q = Big.rp[i]; q < Big.rp[i + 1]; ++q) at[Big.col[q]] = q;
      for (int32_t p = Sub.rp[i]; p < Sub.rp[i + 1]; ++p) f(at[Sub.col[p]], p);
    }
  });
}

// X = P - w D^{-1} (A P), s = -w D^{-1}: the pattern of A P holds P's
inline Csr smoothed(const Csr& P, const Csr& AP, const std::vector<double>& s) {
  Csr Q;
  Q.n = P.n;
  Q.m = P.m;
  Q.rp = AP.rp;
  Q.col.alloc(AP.nnz());
  Q.val.alloc(AP.nnz());
  ranges(Q.n, [&](int, int64_t lo, int64_t hi) {
    for (int64_t i = lo; i < hi; ++i)
      for (int32_t q = AP.rp[i]; q < AP.rp[i + 1]; ++q) {
        Q.col[q] = AP.col[q];
        Q.val[q] = s[i] * AP.val[q];
      }
  });
  each_match(Q, P, [&](int32_t q, int32_t p) { Q.val[q] += P.val[p]; });
  return Q;
}


// [parts[0]; parts[1]; ..], part p's columns shifted by shift[p]
inline Csr stack_rows(const std::vector<const Csr*>& parts, const std::vector<int32_t>& shift) {
  Csr C;
  for (size_t p = 0; p < parts.size(); ++p) {
    C.n += parts[p]->n;
    C.m = std::max<int64_t>(C.m, parts[p]->m + shift[p]);
  }
  C.rp.reserve(C.n + 1);
  C.rp.push_back(0);
  for (const Csr* X : parts)
    for (int64_t i = 0; i < X->n; ++i) C.rp.push_back(X->rp[i + 1] - X->rp[i]);
  if (!allocate(C)) return C;
  int64_t e0 = 0;
  for (size_t p = 0; p < parts.size(); ++p) {
    const Csr& X = *parts[p];
    ranges(X.nnz(), [&](int, int64_t lo, int64_t hi) {
      for (int64_t q = lo; q < hi; ++q) {
        C.col[e0 + q] = X.col[q] + shift[p];
        C.val[e0 + q] = X.val[q];
      }
    });
    e0 += X.nnz();
  }
  return C;
}

// row i: [parts[0] row i | parts[1] row i | ..], part p's columns shifted by shift[p]
inline Csr concat_cols(const std::vector<const Csr*>& parts, const std::vector<int32_t>& shift) {
  Csr C;
  C.n = parts[0]->n;
  C.rp.assign(C.n + 1, 0);
  for (size_t p = 0; p < parts.size(); ++p) {
    C.m = std::max<int64_t>(C.m, parts[p]->m + shift[p]);
    for (int64_t i = 0; i < C.n; ++i) C.rp[i + 1] += parts[p]->rp[i + 1] - parts[p]->rp[i];
  }
  if (!allocate(C)) return C;
  ranges(C.n, [&](int, int64_t lo, int64_t hi) {
    for (int64_t i = lo; i < hi; ++i) {
      int32_t k = C.rp[i];
      for (size_t p = 0; p < parts.size(); ++p) {
        const Csr& X = *parts[p];
        for (int32_t q = X.rp[i]; q < X.rp[i + 1]; ++q, ++k) {
          C.col[k] = X.col[q] + shift[p];
          C.val[k] = X.val[q];
        }
      }
    }
  });
  return C;
}

// Lam = w (2 I - w D^{-1} A) D^{-1} = w (I + S) D^{-1}; for m = 2
// w (I + S + S^2 + S^3) D^{-1}, which is Lam + S^2 Lam. Empty if it does not fit.
inline Csr smoother(const Level& L, int m) {
  const Csr& A = L.A;
  Csr X;
  X.n = A.n;
  X.m = A.m;
  X.rp = A.rp;
  X.col.alloc(A.nnz());
  X.val.alloc(A.nnz());
  ranges(A.n, [&](int, int64_t lo, int64_t hi) {
    for (int64_t i = lo; i < hi; ++i)
      for (int32_t q = A.rp[i]; q < A.rp[i + 1]; ++q) {
        const int32_t j = A.col[q];
        X.col[q] = j;
        X.val[q] = -L.omega * L.omega * L.dinv[i] * A.val[q] * L.dinv[j];
        if (j == i) X.val[q] += 2.0 * L.omega * L.dinv[i];
      }
  });
  if (m == 1) return X;
  std::vector<double> sc(A.n);
  for (int64_t i = 0; i < A.n; ++i) sc[i] = -L.omega * L.dinv[i];
  const Csr AX = product(A, X);
  if (AX.n == 0) return Csr{};
  const Csr SX = smoothed(X, AX, sc);
  const Csr ASX = product(A, SX);
  if (ASX.n == 0) return Csr{};
  Csr Y = smoothed(SX, ASX, sc);           // its pattern holds X's
  each_match(Y, X, [&](int32_t q, int32_t p) { Y.val[q] += X.val[p]; });
  return Y;
}

// Blocks of a product: rows in runs of about kMgEntries entries, each run with
// one number of lanes per row (a power of two from the rows' mean length).
// Segments (levels) of very different row lengths are cut apart. At most `most`
// blocks (0: any number): the runs grow until they fit.
constexpr int64_t kMgEntries = 1400;
inline void make_jobs(const Csr& X, const std::vector<int64_t>& segs, std::vector<MgJob>& jobs,
                      int64_t most = 0, int64_t entries = kMgEntries) {
  jobs.clear();
  for (size_t s = 0; s + 1 < segs.size(); ++s) {
    const int64_t lo = segs[s], hi = segs[s + 1];
    if (lo == hi) continue;
    const double mean = (double)(X.rp[hi] - X.rp[lo]) / (hi - lo);
    int lg = 2;
    while (lg < 8 && (4 << lg) < mean) ++lg;
    if (lg == 7) lg = 8;                     // one row per wavefront or per block
    const int64_t per = 256 >> lg;           // rows a block takes at once
    const int64_t reps = std::max<int64_t>(1, (int64_t)(entries / std::max(1.0, mean * per)));
    for (int64_t r = lo; r < hi; r += per * reps)
      jobs.push_back(MgJob{(int32_t)r, (int32_t)std::min(hi, r + per * reps), lg, 0});
  }
  if (most > 0 && (int64_t)jobs.size() > most && entries < X.nnz())
    return make_jobs(X, segs, jobs, most, 2 * entries);
  // runs of 8 consecutive blocks per XCD (blocks are dealt to the 8 XCDs in
  // turn): neighbouring rows gather neighbouring entries through one L2
  constexpr int64_t kXcd = 8, kRun = 8, span = kXcd * kRun;
  std::vector<MgJob> out;
  out.reserve(jobs.size());
  const int64_t nj = (int64_t)jobs.size(), full = nj / span;
  for (int64_t p = 0; p < full; ++p)
    for (int64_t k = 0; k < kRun; ++k)
      for (int64_t x = 0; x < kXcd; ++x) out.push_back(jobs[p * span + x * kRun + k]);
  for (int64_t b = full * span; b < nj; ++b) out.push_back(jobs[b]);
  jobs.swap(out);
}

// Row-owner maps of one space of the mesh (P1 or P2 elements).
struct Space {
  int64_t n;
  int nloc;
  const Pattern* pat;
  const Incidence* inc;
  const SlotMap* slots;
};
inline Space pressure_space(const Mesh& m) { return {m.n1, m.nloc1, &m.p11, &m.inc1, &m.s11}; }
inline Space velocity_space(const Mesh& m) { return {m.n2, m.nloc2, &m.p22, &m.inc2, &m.s22}; }

// Sparse matrix of a space's stiffness form on the mesh, P1 or P2, without the
// entries that cancel (right angles). fixed (may be null): nodes whose rows
// and columns keep their diagonal only.
inline Csr stiffness(const Mesh& m, const Space& sp, const uint8_t* fixed) {
  const int d = m.dim, nl = sp.nloc, nvl = d + 1;
  const Pattern& pat = *sp.pat;
  const double mean = 1.0 / (d + 1), off = 1.0 / ((d + 1.0) * (d + 2.0));
  static const int e2[3][2] = {{1, 2}, {2, 0}, {0, 1}};
  static const int e3[6][2] = {{0, 1}, {0, 2}, {0, 3}, {1, 2}, {1, 3}, {2, 3}};
  const int(*ed)[2] = d == 2 ? e2 : e3;
  RawVec<double> full;                    // values on the mesh's pattern
  full.alloc(pat.nnz());
  Csr C;
  C.n = C.m = sp.n;
  C.rp.assign(C.n + 1, 0);
  auto keep = [&](int64_t i, int32_t k, double big) {
    if (pat.col[k] == i) return true;
    return std::fabs(full[k]) > 1e-13 * big && !(fixed && (fixed[i] || fixed[pat.col[k]]));
  };
  auto largest = [&](int64_t i) {
    double big = 0.0;
    for (int32_t k = pat.rowptr[i]; k < pat.rowptr[i + 1]; ++k)
      big = std::max(big, std::fabs(full[k]));
    return big;
  };
  ranges(C.n, [&](int, int64_t lo, int64_t hi) {
    for (int64_t i = lo; i < hi; ++i) {
      double* acc = full.data() + pat.rowptr[i];
      std::fill(acc, full.data() + pat.rowptr[i + 1], 0.0);
      for (int32_t q = sp.inc->ptr[i]; q < sp.inc->ptr[i + 1]; ++q) {
        const int64_t cell = sp.inc->code[q] >> 5;
        const int li = sp.inc->code[q] & 31;
        const int32_t* vt = m.c2dp.data() + cell * m.nloc1;   // its vertices lead
        // barycentric gradients from the edge vectors
        double E[3][3] = {}, g[4][3] = {}, det;
        for (int a = 0; a < d; ++a)
          for (int b = 0; b < d; ++b)
            E[a][b] = m.X[(size_t)vt[a + 1] * d + b] - m.X[(size_t)vt[0] * d + b];
        if (d == 2) {
          det = E[0][0] * E[1][1] - E[0][1] * E[1][0];
          g[1][0] = E[1][1] / det;
          g[1][1] = -E[1][0] / det;
          g[2][0] = -E[0][1] / det;
          g[2][1] = E[0][0] / det;
        } else {
          auto cross = [](const double* x, const double* y, double* z) {
            z[0] = x[1] * y[2] - x[2] * y[1];
            z[1] = x[2] * y[0] - x[0] * y[2];
            z[2] = x[0] * y[1] - x[1] * y[0];
          };
          cross(E[1], E[2], g[1]);
          cross(E[2], E[0], g[2]);
          cross(E[0], E[1], g[3]);
          det = E[0][0] * g[1][0] + E[0][1] * g[1][1] + E[0][2] * g[1][2];
          for (int a = 1; a < 4; ++a)
            for (int b = 0; b < 3; ++b) g[a][b] /= det;
        }
        for (int a = 1; a < nvl; ++a)
          for (int b = 0; b < d; ++b) g[0][b] -= g[a][b];
        const double vol = std::fabs(det) / (d == 2 ? 2.0 : 6.0);
        auto gg = [&](int a, int b) {
          double s = 0.0;
          for (int k = 0; k < d; ++k) s += g[a][k] * g[b][k];
          return s;
        };
        auto I = [&](int a, int b) { return a == b ? 2.0 * off : off; };
        auto ve = [&](int a, const int* e) {   // vertex a against edge e
          return 4.0 * ((4.0 * I(a, e[0]) - mean) * gg(a, e[1]) +
                        (4.0 * I(a, e[1]) - mean) * gg(a, e[0]));
        };
        for (int j = 0; j < nl; ++j) {
          double s;
          if (nl == nvl) s = gg(li, j);
          else if (li < nvl && j < nvl) s = gg(li, j) * (16.0 * I(li, j) - 8.0 * mean + 1.0);
          else if (li < nvl) s = ve(li, ed[j - nvl]);
          else if (j < nvl) s = ve(j, ed[li - nvl]);
          else {
            const int *a = ed[li - nvl], *b = ed[j - nvl];
            s = 16.0 * (I(a[0], b[0]) * gg(a[1], b[1]) + I(a[0], b[1]) * gg(a[1], b[0]) +
                        I(a[1], b[0]) * gg(a[0], b[1]) + I(a[1], b[1]) * gg(a[0], b[0]));
          }
          acc[sp.slots->slot[(size_t)q * sp.slots->stride + j]] += vol * s;
        }
      }
      const double big = largest(i);
      for (int32_t k = pat.rowptr[i]; k < pat.rowptr[i + 1]; ++k)
        C.rp[i + 1] += keep(i, k, big) ? 1 : 0;
    }
  });
  if (!allocate(C)) return C;
  ranges(C.n, [&](int, int64_t lo, int64_t hi) {
    for (int64_t i = lo; i < hi; ++i) {
      const double big = largest(i);
      int32_t at = C.rp[i];
      for (int32_t k = pat.rowptr[i]; k < pat.rowptr[i + 1]; ++k)
        if (keep(i, k, big)) {
          C.col[at] = pat.col[k];
          C.val[at++] = full[k];
        }
    }
  });
  return C;
}

// P1 mass matrix in the SELL-64 layout of the pressure pattern (padding 0).
inline std::vector<double> p1_mass_sell(const Mesh& m) {
  std::vector<double> v(m.e11.nent, 0.0);
  const int d = m.dim;
  const double off = 1.0 / ((d + 1.0) * (d + 2.0));
  ranges(m.n1, [&](int, int64_t lo, int64_t hi) {
    for (int64_t i = lo; i < hi; ++i)
      for (int32_t q = m.inc1.ptr[i]; q < m.inc1.ptr[i + 1]; ++q) {
        const int32_t* vt = m.c2dp.data() + (int64_t)(m.inc1.code[q] >> 5) * m.nloc1;
        const int li = m.inc1.code[q] & 31;
        double E[3][3] = {};
        for (int a = 0; a < d; ++a)
          for (int b = 0; b < d; ++b)
            E[a][b] = m.X[(size_t)vt[a + 1] * d + b] - m.X[(size_t)vt[0] * d + b];
        const double det =
            d == 2 ? E[0][0] * E[1][1] - E[0][1] * E[1][0]
                   : E[0][0] * (E[1][1] * E[2][2] - E[1][2] * E[2][1]) -
                         E[0][1] * (E[1][0] * E[2][2] - E[1][2] * E[2][0]) +
                         E[0][2] * (E[1][0] * E[2][1] - E[1][1] * E[2][0]);
        const double vol = std::fabs(det) / (d == 2 ? 2.0 : 6.0);
        for (int j = 0; j <= d; ++j)
          v[m.e11.index(i, m.s11.slot[(size_t)q * m.s11.stride + j])] +=
              vol * off * (j == li ? 2.0 : 1.0);
      }
  });
  return v;
}

// Two damped Jacobi steps before and after (m = 2) instead of one on matrices of
// at most this many entries whose square has at most three times as many (plane
// meshes). There an iteration is bound by its launches and not by the products'
// entries: 64^2 squares take 12 iterations for 17 and 0.37 ms for 0.48; at 128^2
// it is 13 for 18, 0.46 for 0.50 ms and 6 ms more of setup, at 165^2 0.63 ms
// for 0.61; 21^3 cubes would take 14 for 20 with products three times as dense.
constexpr int64_t kSweepsEntries = 50000;
// Most entries of the last product with w = A z beside z (A times its rows, 20
// bytes an entry). It saves the launch of the product w = A z, 4 to 5 us: the
// Poisson phase on 64^2 squares (264 thousand entries, 12 iterations) takes
// 0.33 ms for 0.37, on 14^3 and 21^3 cubes (727 thousand, 19 iterations) 0.39
// for 0.47 and 0.49 for 0.52; at 145^2 (857 thousand) 0.56 either way.
constexpr int64_t kWithW = 750000;
constexpr int64_t kCoarsest = 200;       // last level: solved by its dense inverse
constexpr int64_t kComposeMax = 1200000; // entries of Q_0 times the levels below, for base 0

// P2 pressure nodes from the vertices: a vertex keeps its value, an edge node
// takes the mean of its two. The Galerkin matrix is then the P1 stiffness
// matrix, which aggregation coarsens well (aggregating the P2 nodes themselves
// took 40 iterations where this takes 18, and its coarse rows are denser).
inline Csr p1_to_p2(const Mesh& m) {
  Csr P;
  P.n = m.n1;
  P.m = m.nv;
  P.rp.resize(P.n + 1);
  P.col.alloc(2 * m.n1 - m.nv);
  P.val.alloc(2 * m.n1 - m.nv);
  for (int64_t i = 0; i <= P.n; ++i) P.rp[i] = (int32_t)(i < m.nv ? i : 2 * i - m.nv);
  for (int64_t i = 0; i < m.nv; ++i) {
    P.col[i] = (int32_t)i;
    P.val[i] = 1.0;
  }
  for (int64_t q = m.nv; q < P.nnz(); ++q) {
    P.col[q] = m.edges[q - m.nv];
    P.val[q] = 0.5;
  }
  return P;
}

// P2 velocity nodes off the boundary from the vertices off the boundary, as
// p1_to_p2; empty rows on the boundary. Empty (m = 0) without such vertices.
inline Csr p1_to_velocity(const Mesh& m) {
  std::vector<int32_t> inner(m.nv, -1), ends(2 * m.n2, -1);
  int32_t ni = 0;
  for (int64_t v = 0; v < m.nv; ++v)
    if (!m.bmask[v]) inner[v] = ni++;
  static const int e2[3][2] = {{1, 2}, {2, 0}, {0, 1}};
  static const int e3[6][2] = {{0, 1}, {0, 2}, {0, 3}, {1, 2}, {1, 3}, {2, 3}};
  const int(*ed)[2] = m.dim == 2 ? e2 : e3;
  for (int64_t c = 0; c < m.nc; ++c)
    for (int j = m.dim + 1; j < m.nloc2; ++j)
      for (int k = 0; k < 2; ++k)
        ends[2 * (size_t)m.c2d[c * m.nloc2 + j] + k] =
            m.c2dp[c * m.nloc1 + ed[j - m.dim - 1][k]];
  Csr P;
  P.n = m.n2;
  P.m = ni;
  P.rp.assign(P.n + 1, 0);
  auto entries = [&](int64_t i, int32_t* c) {
    int k = 0;
    if (m.bmask[i]) return k;
    if (i < m.nv) c[k++] = inner[i];
    else
      for (int e = 0; e < 2; ++e)
        if (inner[ends[2 * i + e]] >= 0) c[k++] = inner[ends[2 * i + e]];
    return k;
  };
  int32_t c[2];
  for (int64_t i = 0; i < P.n; ++i) P.rp[i + 1] = entries(i, c);
  allocate(P);
  for (int64_t i = 0; i < P.n; ++i) {
    const int k = entries(i, c);
    for (int e = 0; e < k; ++e) {
      P.col[P.rp[i] + e] = c[e];
      P.val[P.rp[i] + e] = i < m.nv ? 1.0 : 0.5;
    }
  }
  return P;
}

// The hierarchy's products for the symmetric matrix A (constants in its null
// space if singular), or null where aggregation does not coarsen it or a product
// has too many entries. P0 (may be null):
// the prolongator of the finest level, taken over.
inline std::shared_ptr<MgHierarchy> build(Csr A0, Csr* P0, bool singular) {
  std::vector<Level> lev;
  Csr B;
  double theta = 0.08;
  const int sweeps = !P0 && A0.n > kCoarsest && A0.nnz() <= kSweepsEntries &&
                             product(A0, A0).nnz() <= 3 * A0.nnz()
                         ? 2
                         : 1;
  for (Csr A = std::move(A0);; theta *= lev.size() == 1 && P0 ? 1.0 : 0.5) {
    Level L;
    std::vector<double> dg = diagonal(A);
    L.dinv.resize(A.n);
    for (int64_t i = 0; i < A.n; ++i) {
      if (!(dg[i] > 0.0)) return nullptr;
      L.dinv[i] = 1.0 / dg[i];
    }
    if (A.n <= kCoarsest && !(lev.empty() && P0)) {
      if (A.n == 0 || !coarse_inverse(A, singular, B)) return nullptr;
      L.A = std::move(A);
      lev.push_back(std::move(L));
      break;
    }
    const double lam = lambda_max(A, L.dinv);
    if (!(lam > 0.0) || lev.size() > 12) return nullptr;
    L.omega = 1.62 / lam;
    std::vector<double> s(A.n);
    Csr P;
    if (lev.empty() && P0) {
      P = std::move(*P0);
    } else {
      std::vector<int32_t> agg;
      const int64_t na = aggregate(A, dg, theta, agg);
      if (na >= A.n * 3 / 4) return nullptr;
      Csr T;
      T.n = A.n;
      T.m = na;
      T.rp.resize(A.n + 1);
      for (int64_t i = 0; i <= A.n; ++i) T.rp[i] = (int32_t)i;
      T.col.alloc(A.n);
      T.val.alloc(A.n);
      for (int64_t i = 0; i < A.n; ++i) {
        T.col[i] = agg[i];
        T.val[i] = 1.0;
      }
      for (int64_t i = 0; i < A.n; ++i) s[i] = -4.0 / 3.0 / lam * L.dinv[i];
      P = product(A, T, &T, s.data());
    }
    if (P.n == 0) return nullptr;
    const Csr AP = product(A, P);
    if (AP.n == 0) return nullptr;
    for (int64_t i = 0; i < A.n; ++i) s[i] = -L.omega * L.dinv[i];
    L.Q = smoothed(P, AP, s);
    if (sweeps == 2) {
      const Csr AQ = product(A, L.Q);
      if (AQ.n == 0) return nullptr;
      L.Q = smoothed(L.Q, AQ, s);
    }
    Csr Ac = product(transpose(P), AP);
    if (Ac.n == 0) return nullptr;
    L.A = std::move(A);
    lev.push_back(std::move(L));
    A = std::move(Ac);
  }
  const int nl = (int)lev.size();
  if (nl < 2) return nullptr;
  auto h = std::make_shared<MgHierarchy>();
  h->n = lev[0].A.n;
  h->levels = nl;
  const int base = nl < 3 || lev[0].Q.nnz() * (nl - 1) <= kComposeMax ? 0 : 1;
  h->base = base;
  // C[k] takes level base + 1 + k to base; the products of the levels below
  std::vector<Csr> C(nl - base), Rt(nl), Sm(nl);
  for (int k = base + 1; k < nl; ++k)
    C[k - base] = k == base + 1 ? Csr{} : product(k == base + 2 ? lev[base].Q : C[k - base - 1],
                                                  lev[k - 1].Q);
  auto from = [&](int k) -> const Csr& { return k == base + 1 ? lev[base].Q : C[k - base]; };
  std::vector<int64_t> segs{0};
  std::vector<const Csr*> rows, diags, parts;
  std::vector<int32_t> zero, block, shift{0};
  const Csr lam = smoother(lev[base], sweeps);
  if (lam.n == 0) return nullptr;
  parts.push_back(&lam);
  for (int k = base + 1; k < nl; ++k) {
    if (from(k).n == 0) return nullptr;
    Rt[k] = transpose(from(k));
    if (k + 1 < nl) {
      Sm[k] = smoother(lev[k], sweeps);
      if (Sm[k].n == 0) return nullptr;
    }
    rows.push_back(&Rt[k]);
    diags.push_back(k + 1 < nl ? &Sm[k] : &B);
    parts.push_back(&from(k));
    zero.push_back(0);
    block.push_back((int32_t)segs.back());
    shift.push_back((int32_t)(lev[base].A.n + segs.back()));
    segs.push_back(segs.back() + lev[k].A.n);
  }
  Csr R = stack_rows(rows, zero), Dg = stack_rows(diags, block), up = concat_cols(parts, shift);
  if (R.n == 0 || Dg.n == 0 || up.n == 0) return nullptr;
  h->below = segs.back();
  h->nbase = lev[base].A.n;
  auto put = [&](int slot, Csr& X, const std::vector<int64_t>& s) {
    MgProduct& p = h->st[slot];
    p.n = X.n;
    make_jobs(X, s, p.jobs, slot == MG_SLOTS - 1 ? MG_LAST_JOBS : 0);
    p.rp = std::move(X.rp);
    p.col = std::move(X.col);
    p.val = std::move(X.val);
  };
  if (base == 0) {
    put(0, R, segs);
    put(2, Dg, segs);
    // w = A z beside z, while the denser rows cost less than a launch of its own
    // (an upper bound first: most large meshes are past the line)
    Csr W;
    if (singular && up.nnz() <= kWithW) W = product(lev[0].A, up);
    if (W.n != 0 && W.nnz() <= kWithW) {
      RawVec<double> z;
      z.alloc(W.nnz());
      std::fill(z.data(), z.data() + z.size(), 0.0);
      each_match(W, up, [&](int32_t q, int32_t p) { z[q] = up.val[p]; });
      h->st[4].val2 = std::move(W.val);
      W.val = std::move(z);
      up = std::move(W);
    }
    put(4, up, {0, up.n});
  } else {
    Csr R1 = transpose(lev[0].Q);
    const Csr lam0 = smoother(lev[0], sweeps);
    Csr up0 = concat_cols({&lam0, &lev[0].Q}, {0, (int32_t)h->n});
    if (up0.n == 0) return nullptr;
    put(0, R1, {0, R1.n});
    put(1, R, segs);
    put(2, Dg, segs);
    put(3, up, {0, up.n});
    put(4, up0, {0, up0.n});
  }
  return h;
}

}  // namespace amg
}  // namespace ipcs
