// Blocks whose stencil step was measured in both forms.  Row form: the plan is not the one that took
// 15 to 40 % more than another (and more than the tiled form, or close to it).  Tiled form: the blocks
// that it serves faster.
#include "host_case.hpp"

// slow: work-groups and threads of the plan that is not to be taken (0: the tiled form is; 1: no such plan)
struct Step { std::vector<int> n; int ns; sparc_dtype dt; unsigned slow_wg, slow_nt; };

int main() {
  sparc_ctx* ctx;
  CHECK(sparc_ctx_create(0, nullptr, &ctx) == SPARC_OK);
  const Step steps[] = {
      {{80, 80, 80}, 60, SPARC_R64, 1500, 320},     // 16 rows, 16 planes: 207 us, 166 possible, tiled 180
      {{80, 80, 80}, 60, SPARC_C64, 1500, 320},     // 237, 175, 251
      {{48, 48, 48}, 384, SPARC_R32, 1536, 320},    // 48 rows, 12 planes: 160, 123, 156
      {{64, 64, 64}, 512, SPARC_R32, 512, 512},     // 64 rows, 64 planes: 387, 322, 384
      {{40, 40, 40}, 300, SPARC_C128, 1200, 448},   // 20 rows, 20 planes: 399, 288, 371
      {{26, 22, 23}, 512, SPARC_R32, 512, 128},     // 24 rows, 23 planes: 49, 33, 32
      {{17, 27, 33}, 512, SPARC_R64, 512, 128},     // 28 rows, 33 planes: 75, 52, 88
      {{27, 39, 27}, 404, SPARC_R32, 0, 0},         // tiled 46, rows 60
      {{32, 20, 31}, 512, SPARC_C128, 1, 0},        // row form: tiled 143, rows 121
      {{58, 53, 53}, 178, SPARC_C128, 1, 0},        // 507, 412
      {{51, 60, 56}, 2, SPARC_C128, 1, 0},          // point form 43, rows 17
      {{96, 96, 96}, 24, SPARC_C128, 1, 0},         // tiled 313, rows 249
      {{128, 96, 64}, 8, SPARC_C128, 1, 0},         // 109, 81
      {{112, 112, 48}, 30, SPARC_C128, 0, 0},       // in a plan 232, 249
      {{43, 47, 41}, 82, SPARC_R32, 0, 0}};         // 32, 34
  for (const Step& st : steps) {
    Cell cell(st.n, 1);
    sparc_ham* h;
    CHECK(sparc_ham_create(ctx, &cell.grid, &cell.atoms, st.dt, &h) == SPARC_OK);
    const int64_t nd = (int64_t)st.n[0] * st.n[1] * st.n[2];
    char x[64], y[64];   // no kernel runs: never read
    fake::clear();
    CHECK(fd_hamiltonian_apply(h, x, nd, y, nd, st.ns, x, (size_t)1 << 60) == SPARC_OK);
    for (const fake::Launch& l : fake::launches) {
      if (l.kernel != "hrow_kernel" && l.kernel != "hstep_kernel") continue;
      CHECK((l.kernel == "hrow_kernel") == (st.slow_wg != 0));
      if (st.slow_wg) CHECK(l.grid.x != st.slow_wg || l.block.x != st.slow_nt);
    }
    CHECK(fake::count("hrow_kernel") + fake::count("hstep_kernel") == 1);
    sparc_ham_destroy(h);
  }
  return 0;
}
