// Device allocations of a Hamiltonian: three atom tables, the force sums, three potentials, and one
// for all projector tables.
#include "host_case.hpp"

int main() {
  sparc_ctx* ctx;
  CHECK(sparc_ctx_create(0, nullptr, &ctx) == SPARC_OK);
  Cell cell({24, 20, 18}, 3), bare({24, 20, 18}, 3);
  bare.atoms.n_chan = 0;
  for (Cell* c : {&cell, &bare})
    for (sparc_dtype dt : {SPARC_R64, SPARC_R32, SPARC_C128, SPARC_C64}) {
      sparc_ham* h;
      fake::clear();
      CHECK(sparc_ham_create(ctx, &c->grid, &c->atoms, dt, &h) == SPARC_OK);
      CHECK(fake::n_malloc == 8 && fake::n_memcpy <= 5);
      sparc_ham_destroy(h);
    }
  return 0;
}
