// Checks of the multigrid hierarchy (amg.hpp) on the CPU: every row of every
// product in exactly one block of a bounded number of blocks; memory that runs
// out anywhere in its construction; products of too many entries.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <new>
#include <vector>

#include "amg.hpp"
#include "common.hpp"
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
  const size_t last = h.st[MG_SLOTS - 1].jobs.size();
  std::printf("%lld rows: %zu blocks in the last product\n", (long long)h.n, last);
  CHECK(last >= 1 && last <= 8192);
}

static void large_meshes() {
  std::unique_ptr<Mesh> s(build_unit_square(1024, 1024)), c(build_unit_cube(80, 80, 80));
  for (const Mesh* m : {s.get(), c.get()}) {
    auto h = m->multigrid();
    CHECK(h != nullptr);
    check_jobs(*h);
  }
}

int main(int argc, char** argv) {
  const char* what = argc > 1 ? argv[1] : "";
  if (!std::strcmp(what, "large")) large_meshes();
  else if (!std::strcmp(what, "memory")) out_of_memory();
  else if (!std::strcmp(what, "entries")) too_many_entries();
  else return 1;
  std::printf("ok\n");
}
