// Plans of one and two orbitals run row kernels; single calls of that size the point form.
#include "host_case.hpp"

int main() {
  sparc_ctx* ctx;
  CHECK(sparc_ctx_create(0, nullptr, &ctx) == SPARC_OK);
  const std::vector<int> sizes[] = {{20, 16, 40}, {24, 20, 18}, {17, 30, 19}};
  for (sparc_dtype dt : {SPARC_R64, SPARC_R32, SPARC_C128, SPARC_C64})
    for (const auto& n : sizes)
      for (int32_t ns : {1, 2}) {
        Cell cell(n, 1);
        sparc_ham* h;
        CHECK(sparc_ham_create(ctx, &cell.grid, &cell.atoms, dt, &h) == SPARC_OK);
        const int64_t nd = (int64_t)n[0] * n[1] * n[2];
        char x[64], y[64];   // no kernel runs: never read
        void* const X[] = {x};
        const int32_t deg[] = {4};
        const double lo[] = {1.0}, hi[] = {2.0};
        const size_t bytes = sparc_filter_plan_workspace_bytes(1, &h, &ns, deg);
        Block work(bytes / 8 + 1);
        fake::clear();
        CHECK(chebyshev_filter_batched(ctx, 1, &h, X, &nd, &ns, deg, lo, hi, work.p, bytes) == SPARC_OK);
        CHECK(fake::count("hrow_batched_kernel") == 4);
        CHECK(fd_hamiltonian_apply(h, x, nd, y, nd, 1, work.p, bytes) == SPARC_OK);
        CHECK(fake::count("hstep_point_kernel") == 1);
        sparc_ham_destroy(h);
      }
  return 0;
}
