// Which conjugate-gradient iteration the Poisson solve of an SCF takes: rows within the one-launch
// form's LDS and up to 2^19 nodes one launch; longer rows and larger grids of the point form two;
// the general loop only past the point form.
#include "host_case.hpp"

struct Route { std::vector<int> n; const char *must, *mustnot; };

int main() {
  hipStream_t stream;
  hipStreamCreateWithFlags(&stream, hipStreamNonBlocking);
  sparc_ctx* ctx;
  CHECK(sparc_ctx_create(0, stream, &ctx) == SPARC_OK);
  const Route routes[] = {{{300, 9, 8}, "cg_step_kernel", "cg_update_kernel"},
                          {{2048, 9, 8}, "cg_step_kernel", "cg_update_kernel"},
                          {{2049, 9, 8}, "cg_update_kernel", "cg_step_kernel"},
                          {{4096, 8, 9}, "cg_update_kernel", "cg_step_kernel"},
                          {{82, 80, 81}, "cg_update_kernel", "cg_step_kernel"}};
  for (const Route& r : routes) {
    Cell cell(r.n, 1, 4);
    const int64_t nd = (int64_t)r.n[0] * r.n[1] * r.n[2];
    Block x0(2 * nd), v0(nd), rho(nd), ritz(2);
    sparc_scf_params P{};
    P.n_s = 2;
    P.degree = P.n_first_passes = P.max_iter = 1;
    P.lanczos_steps = 4;
    P.kT = 0.01;
    P.mix = 0.3;
    P.tol = 1e-3;
    P.n_elec = 2.0;
    P.x0_dev = (const double*)x0.p;
    P.lanczos_v0_dev = (const double*)v0.p;
    sparc_scf_result res{};
    res.rho_dev = (double*)rho.p;
    res.ritz_dev = (double*)ritz.p;
    fake::clear();
    fake::readback = 1.0;   // a residual that never falls: the first solve runs to its limit
    CHECK(sparc_scf_run(ctx, &cell.grid, &cell.atoms, &P, &res) == SPARC_ENOCONV);
    CHECK(fake::count(r.must) == 20000);
    CHECK(fake::count(r.mustnot) == 0);
    CHECK(fake::count("cg_xr_rr_kernel") == 0);
  }
  return 0;
}
