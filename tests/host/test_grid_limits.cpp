// Grids of launches over very many orbitals: no direction but the first may have more than
// 65535 work-groups, and what does not fit takes another kernel.
#include "host_case.hpp"

int main() {
  sparc_ctx* ctx;
  CHECK(sparc_ctx_create(0, nullptr, &ctx) == SPARC_OK);
  Cell cell({16, 16, 16}, 2);
  const int64_t nd = 4096;
  Block X(16);   // no kernel runs: the blocks are never read
  // orbitals of 65535 groups of the projector update, and one more
  const struct { sparc_dtype dt; int32_t ns; bool update; } cases[] = {
      {SPARC_C128, 2 * 65535, true}, {SPARC_C128, 2 * 65535 + 1, false},
      {SPARC_R64, 4 * 65535, true},  {SPARC_R32, 4 * 65535, true}};
  for (const auto& c : cases) {
    sparc_ham* ham;
    CHECK(sparc_ham_create(ctx, &cell.grid, &cell.atoms, c.dt, &ham) == SPARC_OK);
    fake::clear();
    CHECK(chebyshev_filter(ham, X.p, nd, c.ns, 4, 1.0, 2.0, X.p, (size_t)1 << 60) == SPARC_OK);
    CHECK((fake::count("nl_update_kernel") == 3) == c.update);
    CHECK(fake::count("nl_gather_kernel") == (c.update ? 1 : 4));
    sparc_ham_destroy(ham);
  }
  return 0;
}
