// Checks of the multigrid hierarchy (amg.hpp) on the CPU: every row of every
// product in exactly one block of a bounded number of blocks, a symmetric and
// positive cycle; memory that runs out anywhere in its construction; products of
// too many entries.
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <new>
#include <vector>

#include "amg.hpp"
#include "common.hpp"
#include "device.hpp"
#include "mesh.hpp"

using namespace ipcs;

#define CHECK(c)                                                             \
  do {                                                                       \
    if (!(c)) {                                                              \
      std::fprintf(stderr, "check failed: %s (%s:%d)\n", #c, __FILE__, __LINE__); \
      std::exit(2);                                                          \
    }                                                                        \
  } while (0)

// The allocation that is to fail, counted down from where it is armed (< 0: none).
static std::atomic<long> g_left{-1};
static std::atomic<bool> g_armed{false};
static void* counted(std::size_t n) {
  if (g_armed && g_left.fetch_sub(1) == 0) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void* operator new(std::size_t n) { return counted(n); }
void* operator new[](std::size_t n) { return counted(n); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete[](void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
void operator delete[](void* p, std::size_t) noexcept { std::free(p); }

// Each allocation of a hierarchy fails in turn: the call throws, and the next
// one builds it. (Enough rows for several threads.)
static void out_of_memory() {
  for (int pair : {0, 1})
    for (bool velocity : {false, true}) {
      if (velocity && pair == 1) continue;   // P2-P1 only
      std::unique_ptr<Mesh> m(pair ? build_unit_square(20, 20, 1) : build_unit_square(36, 36));
      long failed = 0;
      for (long k = 0;; ++k) {
        g_left = k;
        g_armed = true;
        bool threw = false;
        std::shared_ptr<const MgHierarchy> h;
        try {
          h = velocity ? m->velocity_multigrid() : m->multigrid();
        } catch (const std::bad_alloc&) {
          threw = true;
        }
        g_armed = false;
        if (!threw) {
          CHECK(h != nullptr && g_left >= 0);
          break;
        }
        ++failed;
      }
      std::printf("pair %d velocity %d: %ld allocations\n", pair, (int)velocity, failed);
      CHECK(failed > 50);
    }
}

// A product past 2^31 entries (4200 rows of 600000) has no hierarchy.
static void too_many_entries() {
  const int32_t n = 4200, m = 600000;
  amg::Csr A, P;
  A.n = A.m = P.n = n;
  P.m = m;
  A.rp.push_back(0);
  P.rp.push_back(0);
  for (int32_t i = 0; i < n; ++i) {
    A.rp.push_back(A.rp.back() + (i + 1 < n ? 2 : 1));
    P.rp.push_back(P.rp.back() + (i + 1 < n ? 1 : m));
  }
  A.col.alloc(A.nnz());
  A.val.alloc(A.nnz());
  P.col.alloc(P.nnz());
  P.val.alloc(P.nnz());
  for (int32_t i = 0; i < n; ++i) {
    A.col[A.rp[i]] = i;
    A.val[A.rp[i]] = 2.0;
    if (i + 1 < n) {
      A.col[A.rp[i] + 1] = n - 1;
      A.val[A.rp[i] + 1] = -1.0 / n;
    }
  }
  for (int32_t q = 0; q < P.nnz(); ++q) {
    P.col[q] = q < n - 1 ? q : q - (n - 1);
    P.val[q] = 1.0;
  }
  CHECK(amg::build(std::move(A), &P, true) == nullptr);
}

static void check_jobs(const MgHierarchy& h) {
  for (int k = 0; k < MG_SLOTS; ++k) {
    const MgProduct& p = h.st[k];
    std::vector<uint8_t> seen(p.n, 0);
    for (const MgJob& j : p.jobs) {
      CHECK(0 <= j.row0 && j.row0 < j.row1 && j.row1 <= p.n);
      CHECK(j.lg >= 2 && j.lg <= 8 && j.lg != 7);
      for (int32_t r = j.row0; r < j.row1; ++r) CHECK(seen[r]++ == 0);
    }
    for (int64_t r = 0; r < p.n; ++r) CHECK(seen[r] == 1);
  }
  uint64_t bits = 1469598103934665603u;
  auto hash = [&](const void* p, size_t n) {
    for (size_t i = 0; i < n; ++i) bits = (bits ^ static_cast<const uint8_t*>(p)[i]) * 1099511628211u;
  };
  for (const MgProduct& p : h.st) {
    hash(p.rp.data(), p.rp.size() * 4);
    hash(p.col.data(), p.col.size() * 4);
    hash(p.val.data(), p.val.size() * 8);
    hash(p.val2.data(), p.val2.size() * 8);
  }
  const size_t last = h.st[MG_SLOTS - 1].jobs.size();
  std::printf("%lld rows: %zu blocks in the last product, %016llx\n", (long long)h.n, last,
              (unsigned long long)bits);
  CHECK(last >= 1 && last <= 8192);
}

static std::vector<double> times(const MgProduct& p, const RawVec<double>& val,
                                 const std::vector<double>& x) {
  std::vector<double> y(p.n, 0.0);
  for (int64_t i = 0; i < p.n; ++i)
    for (int32_t q = p.rp[i]; q < p.rp[i + 1]; ++q) {
      CHECK(p.col[q] >= 0 && p.col[q] < (int64_t)x.size());
      y[i] += val[q] * x[p.col[q]];
    }
  return y;
}

static std::vector<double> joined(std::vector<double> a, const std::vector<double>& b) {
  a.insert(a.end(), b.begin(), b.end());
  return a;
}

// z = B r by the products, as mesh.hpp states their inputs; the last one's input
// is left in `in`.
static std::vector<double> cycle(const MgHierarchy& h, const std::vector<double>& r,
                                 std::vector<double>& in) {
  auto mul = [&](int k, const std::vector<double>& x) { return times(h.st[k], h.st[k].val, x); };
  if (h.base == 0) {
    in = joined(r, mul(2, mul(0, r)));
  } else {
    const std::vector<double> r1 = mul(0, r);
    CHECK((int64_t)r1.size() == h.nbase);
    const std::vector<double> e = mul(2, mul(1, r1));
    CHECK((int64_t)e.size() == h.below);
    in = joined(r, mul(3, joined(r1, e)));
  }
  return mul(MG_SLOTS - 1, in);
}

static double dot(const std::vector<double>& a, const std::vector<double>& b) {
  double s = 0.0;
  for (size_t i = 0; i < a.size(); ++i) s += a[i] * b[i];
  return s;
}

// The cycle is symmetric and positive (off the constants, where singular), and
// second values give w = A z.
static void check_cycle(const MgHierarchy& h, const amg::Csr& A, bool singular) {
  CHECK(h.n == A.n);
  std::vector<double> x(h.n), y(h.n), in;
  uint32_t s = 12345;
  double mx = 0.0, my = 0.0;
  for (int64_t i = 0; i < h.n; ++i) {
    x[i] = (s = s * 1664525u + 1013904223u) / 4294967296.0 - 0.5;
    y[i] = (s = s * 1664525u + 1013904223u) / 4294967296.0 - 0.5;
    mx += x[i] / h.n;
    my += y[i] / h.n;
  }
  if (singular)
    for (int64_t i = 0; i < h.n; ++i) {
      x[i] -= mx;
      y[i] -= my;
    }
  const std::vector<double> by = cycle(h, y, in), bx = cycle(h, x, in);
  const double xx = dot(x, bx), yy = dot(y, by);
  CHECK(xx > 0.0 && yy > 0.0);
  CHECK(std::fabs(dot(x, by) - dot(y, bx)) <= 1e-12 * std::sqrt(xx * yy));
  const MgProduct& last = h.st[MG_SLOTS - 1];
  if (last.val2.size() == 0) return;
  const std::vector<double> w = times(last, last.val2, in);
  double err = 0.0, top = 0.0;
  for (int64_t i = 0; i < A.n; ++i) {
    double v = 0.0, a = 0.0;
    for (int32_t q = A.rp[i]; q < A.rp[i + 1]; ++q) {
      v += A.val[q] * bx[A.col[q]];
      a += std::fabs(A.val[q] * bx[A.col[q]]);
    }
    err = std::max(err, std::fabs(v - w[i]));
    top = std::max(top, a);
  }
  CHECK(err <= 1e-12 * top);
}

// Meshes of both dimensions and pairs, strips, vertices moved and relabelled.
static Mesh* moved(int dim, int n, int pair) {
  std::unique_ptr<Mesh> m(dim == 2 ? build_unit_square(n, n) : build_unit_cube(n, n, n));
  std::vector<double> X(m->nv * dim);
  std::vector<int32_t> at(m->nv), cells(m->nc * (dim + 1));
  uint32_t s = 99;
  for (int64_t v = 0; v < m->nv; ++v) at[v] = (int32_t)v;
  for (int64_t v = m->nv - 1; v > 0; --v)
    std::swap(at[v], at[(s = s * 1664525u + 1013904223u) % (uint32_t)(v + 1)]);
  for (int64_t v = 0; v < m->nv; ++v)
    for (int b = 0; b < dim; ++b)
      X[(size_t)at[v] * dim + b] =
          m->X[(size_t)v * dim + b] +
          (m->bmask[v] ? 0.0 : 0.15 / n * ((s = s * 1664525u + 1013904223u) / 2147483648.0 - 1.0));
  for (int64_t c = 0; c < m->nc; ++c)
    for (int j = 0; j <= dim; ++j) cells[c * (dim + 1) + j] = at[m->c2dp[c * m->nloc1 + j]];
  return build_from_arrays(dim, m->nv, X.data(), m->nc, cells.data(), pair);
}

static void shapes() {
  std::vector<std::unique_ptr<Mesh>> ms;
  for (int n : {1, 2, 3, 15, 40, 53}) ms.emplace_back(build_unit_square(n, n));
  ms.emplace_back(build_unit_square(300, 3));
  ms.emplace_back(build_unit_square(170, 170));      // more than the composed products take
  for (int n : {1, 4, 11}) ms.emplace_back(build_unit_cube(n, n, n));
  ms.emplace_back(build_unit_cube(2, 3, 40));
  for (int n : {1, 9, 24}) ms.emplace_back(build_unit_square(n, n, 1));
  for (int n : {1, 5}) ms.emplace_back(build_unit_cube(n, n, n, 1));
  for (int pair : {0, 1}) {
    ms.emplace_back(moved(2, 22, pair));
    ms.emplace_back(moved(3, 6, pair));
  }
  int made = 0;
  for (const auto& m : ms) {
    if (auto h = m->multigrid()) {
      check_jobs(*h);
      check_cycle(*h, amg::stiffness(*m, amg::pressure_space(*m), nullptr), true);
      ++made;
    }
    if (m->n1 > m->nv) continue;
    if (auto h = m->velocity_multigrid()) {
      check_jobs(*h);
      check_cycle(*h, amg::stiffness(*m, amg::velocity_space(*m), m->bmask.data()), false);
      ++made;
    }
  }
  std::printf("%d hierarchies\n", made);
  CHECK(made > 20);
}

static void large_meshes() {
  std::unique_ptr<Mesh> s(build_unit_square(1024, 1024)), c(build_unit_cube(80, 80, 80));
  for (const Mesh* m : {s.get(), c.get()}) {
    auto h = m->multigrid();
    CHECK(h != nullptr);
    check_jobs(*h);
  }
}

// Launches over more runs than the y dimension takes are cut up.
static void launch_groups() {
  for (int n : {1, 65535, 65536, 65537, 200000}) {
    int at = 0, launches = 0;
    over_groups(n, [&](int first, int count) {
      CHECK(first == at && count >= 1 && count <= 65536);
      at += count;
      ++launches;
    });
    CHECK(at == n && launches == (n + 65535) / 65536);
  }
}

int main(int argc, char** argv) {
  const char* what = argc > 1 ? argv[1] : "";
  if (!std::strcmp(what, "shapes")) shapes();
  else if (!std::strcmp(what, "large")) large_meshes();
  else if (!std::strcmp(what, "groups")) launch_groups();
  else if (!std::strcmp(what, "memory")) out_of_memory();
  else if (!std::strcmp(what, "entries")) too_many_entries();
  else return 1;
  std::printf("ok\n");
}
