// Two contexts on two devices, the calling thread's current device being the other one: side
// streams, their events and the raised LDS limits belong to the context's device.
#include "host_case.hpp"

int main() {
  hipStream_t stream[2];
  sparc_ctx* ctx[2];
  sparc_ham* ham[2];
  for (int d = 0; d < 2; ++d) {
    hipSetDevice(d);
    hipStreamCreateWithFlags(&stream[d], hipStreamNonBlocking);
    CHECK(sparc_ctx_create(d, stream[d], &ctx[d]) == SPARC_OK);
  }
  Cell cell({96, 96, 32}, 3);
  for (int d = 0; d < 2; ++d) CHECK(sparc_ham_create(ctx[d], &cell.grid, &cell.atoms, SPARC_R64, &ham[d]) == SPARC_OK);
  fake::readback = 1.0;   // first Gram matrices: Cholesky status 0, condition estimate 1
  const int ns = 64;
  const int64_t nd = 96 * 96 * 32;
  for (int d : {0, 1}) {
    hipSetDevice(1 - d);
    fake::clear();
    Block X(nd * ns), Y(nd * ns), R(4 * ns), W(1 << 27);
    CHECK(fd_hamiltonian_apply(ham[d], X.p, nd, Y.p, nd, ns, W.p, W.bytes()) == SPARC_OK);
    CHECK(fake::count("hrow_kernel") == 1);
    for (const fake::Launch& l : fake::launches) CHECK(l.kernel != "hrow_kernel" || l.lds > fake::kDefaultLds);
    sparc_ham* const hs[] = {ham[d], ham[d]};
    void* const xs[] = {X.p, Y.p};
    const int64_t lds[] = {nd, nd};
    const int32_t nss[] = {ns, ns};
    double* const rs[] = {(double*)R.p, (double*)R.p + 2 * ns};
    CHECK(rayleigh_ritz_batched(ctx[d], 2, hs, xs, lds, nss, SPARC_GEMM_NATIVE, rs, W.p, W.bytes()) == SPARC_OK);
    CHECK(fake::streams_made.size() == 3);
    for (int made : fake::streams_made) CHECK(made == d);
    for (int made : fake::events_made) CHECK(made == d);
    for (const fake::Launch& l : fake::launches) CHECK(l.device == d);
    CHECK(fake::current == 1 - d);   // and the caller's device is left as it was
  }
  return 0;
}
