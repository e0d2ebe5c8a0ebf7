// Stencil launches of a plan: one a step, in the row form whatever the problems' chunk widths.
#include "host_case.hpp"

struct Plan { std::vector<std::vector<int>> n; std::vector<int32_t> ns, deg; sparc_dtype dt; const char* kernel; };

int main() {
  sparc_ctx* ctx;
  CHECK(sparc_ctx_create(0, nullptr, &ctx) == SPARC_OK);
  const Plan plans[] = {
      {{{24, 20, 18}, {17, 16, 18}, {40, 36, 32}}, {3, 3, 3}, {6, 5, 3}, SPARC_R64, "hrow_mixed_kernel"},
      {{{24, 20, 18}, {32, 16, 18}, {40, 36, 32}}, {3, 9, 3}, {3, 6, 4}, SPARC_R64, "hrow_batched_kernel"},
      {{{17, 20, 18}, {33, 36, 18}}, {3, 9}, {3, 6}, SPARC_R64, "hrow_batched_kernel"},
      {{{40, 36, 18}, {42, 36, 18}, {43, 36, 16}}, {20, 4, 2}, {5, 4, 3}, SPARC_R32, "hrow_mixed_kernel"},
      {{{33, 20, 18}, {45, 16, 18}}, {3, 3}, {4, 4}, SPARC_C128, "hrow_batched_kernel"},
      {{{32, 20, 18}, {33, 36, 18}}, {3, 3}, {4, 2}, SPARC_C64, "hrow_mixed_kernel"},
      // most values in narrow FP32 chunks, enough to fill the chip
      {{{40, 36, 18}, {43, 41, 36}, {38, 40, 40}}, {4, 30, 30}, {5, 4, 3}, SPARC_R32, "hstep_batched_kernel"},
      {{{24, 20, 18}, {17, 16, 15}}, {3, 3}, {5, 7}, SPARC_R64, "hstep_batched_kernel"},       // 15 nodes
      {{{40, 36, 18}, {43, 16, 16}}, {3, 3}, {5, 4}, SPARC_R32, "hstep_batched_kernel"}};      // no tile of 43 x 16 rows
  for (const Plan& p : plans) {
    const int n = (int)p.n.size();
    std::vector<sparc_ham*> h(n);
    std::vector<int64_t> ld(n);
    std::vector<double> lo(n, 1.0), hi(n, 2.0);
    char x[64];   // no kernel runs: never read
    std::vector<void*> X(n, x);
    int32_t steps = 0;
    for (int i = 0; i < n; ++i) {
      Cell cell(p.n[i], 1);
      CHECK(sparc_ham_create(ctx, &cell.grid, &cell.atoms, p.dt, &h[i]) == SPARC_OK);
      ld[i] = (int64_t)p.n[i][0] * p.n[i][1] * p.n[i][2];
      steps = std::max(steps, p.deg[i]);
    }
    const size_t bytes = sparc_filter_plan_workspace_bytes(n, h.data(), p.ns.data(), p.deg.data());
    Block work(bytes / 8 + 1);
    fake::clear();
    CHECK(chebyshev_filter_batched(ctx, n, h.data(), X.data(), ld.data(), p.ns.data(), p.deg.data(), lo.data(), hi.data(),
                                   work.p, bytes) == SPARC_OK);
    int stencil = 0;
    for (const fake::Launch& l : fake::launches) stencil += l.kernel.find("hrow") == 0 || l.kernel.find("hstep") == 0;
    CHECK(fake::count(p.kernel) == steps && stencil == steps);
  }
  return 0;
}
