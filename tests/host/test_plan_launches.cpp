// Stencil launches of a plan: one a step and chunk width in the row form, one a step in the tiled form.
#include "host_case.hpp"

struct Plan { std::vector<std::vector<int>> n; std::vector<int32_t> deg; sparc_dtype dt; const char* kernel; int launches; };

int main() {
  sparc_ctx* ctx;
  CHECK(sparc_ctx_create(0, nullptr, &ctx) == SPARC_OK);
  const Plan plans[] = {
      {{{24, 20, 18}, {17, 16, 18}, {40, 36, 32}}, {6, 5, 3}, SPARC_R64, "hrow_batched_kernel", 6 + 5},
      {{{24, 20, 18}, {17, 16, 18}, {17, 20, 16}}, {3, 6, 4}, SPARC_R64, "hrow_batched_kernel", 3 + 6},
      {{{40, 36, 18}, {42, 36, 18}, {43, 36, 16}}, {5, 4, 3}, SPARC_R32, "hrow_batched_kernel", 5 + 4 + 3},
      {{{33, 20, 18}, {45, 16, 18}}, {4, 4}, SPARC_C128, "hrow_batched_kernel", 4},
      {{{32, 20, 18}, {33, 36, 18}}, {4, 2}, SPARC_C64, "hrow_batched_kernel", 4 + 2},
      {{{24, 20, 18}, {17, 16, 15}}, {5, 7}, SPARC_R64, "hstep_batched_kernel", 7},      // 15 nodes
      {{{40, 36, 18}, {43, 16, 16}}, {5, 4}, SPARC_R32, "hstep_batched_kernel", 5}};  // no tile of 43 x 16 rows
  for (const Plan& p : plans) {
    const int n = (int)p.n.size();
    std::vector<sparc_ham*> h(n);
    std::vector<int64_t> ld(n);
    std::vector<int32_t> ns(n, 3);
    std::vector<double> lo(n, 1.0), hi(n, 2.0);
    char x[64];   // no kernel runs: never read
    std::vector<void*> X(n, x);
    for (int i = 0; i < n; ++i) {
      Cell cell(p.n[i], 1);
      CHECK(sparc_ham_create(ctx, &cell.grid, &cell.atoms, p.dt, &h[i]) == SPARC_OK);
      ld[i] = (int64_t)p.n[i][0] * p.n[i][1] * p.n[i][2];
    }
    const size_t bytes = sparc_filter_plan_workspace_bytes(n, h.data(), ns.data(), p.deg.data());
    Block work(bytes / 8 + 1);
    fake::clear();
    CHECK(chebyshev_filter_batched(ctx, n, h.data(), X.data(), ld.data(), ns.data(), p.deg.data(), lo.data(), hi.data(),
                                   work.p, bytes) == SPARC_OK);
    CHECK(fake::count(p.kernel) == p.launches);
  }
  return 0;
}
