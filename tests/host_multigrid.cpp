// Checks of the multigrid hierarchy (amg.hpp) on the CPU: every row of every
// product in exactly one block of a bounded number of blocks.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
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
  else return 1;
  std::printf("ok\n");
}
