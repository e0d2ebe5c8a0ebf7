// Every row kernel whose work-groups take more than 64 KB of LDS has its limit raised: the first
// step, recurrence steps and batched steps are kernels of their own.
#include "host_case.hpp"

int main() {
  sparc_ctx* ctx;
  CHECK(sparc_ctx_create(0, nullptr, &ctx) == SPARC_OK);
  Cell cell({96, 96, 32}, 2);
  const int64_t nd = 96 * 96 * 32;
  const int32_t ns[] = {64}, deg[] = {3};
  const double lo[] = {1.0}, hi[] = {2.0};
  char x[64];   // no kernel runs: never read
  void* const X[] = {x};
  for (sparc_dtype dt : {SPARC_R64, SPARC_R32, SPARC_C128, SPARC_C64}) {
    sparc_ham* h;
    CHECK(sparc_ham_create(ctx, &cell.grid, &cell.atoms, dt, &h) == SPARC_OK);
    fake::clear();
    CHECK(chebyshev_filter(h, x, nd, 64, 3, 1.0, 2.0, x, (size_t)1 << 60) == SPARC_OK);
    const size_t bytes = sparc_filter_plan_workspace_bytes(1, &h, ns, deg);
    Block work(bytes / 8 + 1);
    CHECK(chebyshev_filter_batched(ctx, 1, &h, X, &nd, ns, deg, lo, hi, work.p, bytes) == SPARC_OK);
    int large = 0;
    for (const fake::Launch& l : fake::launches) large += l.kernel.find("hrow") == 0 && l.lds > fake::kDefaultLds;
    if (dt == SPARC_R64) CHECK(large == 6);
  }
  return 0;
}
