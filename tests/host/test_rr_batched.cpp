// Batched Rayleigh-Ritz: on a context that autotunes, the first call of a shape times its products
// with nothing on the side streams; later calls use those and time nothing.  The side streams
// stay idle too where the workspace does not hold the problems' dense parts next to the blocks,
// with kernel timing on, for split products, and for two to four problems of a few states.
#include "host_case.hpp"

static sparc_ctx* ctx;
static hipStream_t stream;

struct Seen { int side, timed; };   // launches off the context's stream, waits for timing events

static Seen run(std::vector<sparc_ham*> hams, int ns, sparc_gemm_mode mode = SPARC_GEMM_NATIVE) {
  std::vector<Block*> blocks;
  std::vector<void*> X;
  std::vector<double*> ritz;
  std::vector<int64_t> ld;
  std::vector<int32_t> n;
  for (sparc_ham* h : hams) {
    int64_t nd, ne;
    int32_t np;
    sparc_ham_info(h, &nd, &np, &ne);
    blocks.push_back(new Block(2 * nd * ns));   // complex ones too
    X.push_back(blocks.back()->p);
    blocks.push_back(new Block(ns));
    ritz.push_back((double*)blocks.back()->p);
    ld.push_back(nd);
    n.push_back(ns);
  }
  const size_t bytes = sparc_rr_batched_workspace_bytes((int)hams.size(), hams.data(), n.data());
  Block work(bytes / 8 + 1);
  fake::clear();
  CHECK(rayleigh_ritz_batched(ctx, (int)hams.size(), hams.data(), X.data(), ld.data(), n.data(), mode, ritz.data(),
                              work.p, bytes) == SPARC_OK);
  CHECK(fake::count("inviter_kernel") + fake::count("chol_diag_kernel") > 0);
  Seen s{0, fake::n_event_sync};
  for (const fake::Launch& l : fake::launches) s.side += l.stream != stream;
  for (Block* b : blocks) delete b;
  return s;
}

int main() {
  hipStreamCreateWithFlags(&stream, hipStreamNonBlocking);
  CHECK(sparc_ctx_create(0, stream, &ctx) == SPARC_OK);
  Cell cell({24, 22, 26}, 2), small({12, 10, 8}, 1);
  sparc_ham *h, *g, *f, *tiny;
  CHECK(sparc_ham_create(ctx, &cell.grid, &cell.atoms, SPARC_R64, &h) == SPARC_OK);
  CHECK(sparc_ham_create(ctx, &cell.grid, &cell.atoms, SPARC_C128, &g) == SPARC_OK);
  CHECK(sparc_ham_create(ctx, &cell.grid, &cell.atoms, SPARC_R32, &f) == SPARC_OK);
  CHECK(sparc_ham_create(ctx, &small.grid, &small.atoms, SPARC_R64, &tiny) == SPARC_OK);
  fake::readback = 1.0;   // Cholesky status 0, condition estimate 1: one pass

  Seen s = run({h, g, h}, 30);
  CHECK(s.side > 0 && s.timed == 0);
  CHECK(run({tiny, tiny, tiny, tiny}, 480).side == 0);   // dense parts larger than the blocks
  CHECK(run({f, f}, 32, SPARC_GEMM_BF16X3).side == 0);
  CHECK(run({h, f}, 12).side == 0 && run({g, g}, 4).side == 0 && run({h, f, h, f}, 4).side == 0);
  CHECK(run({h, f}, 13).side > 0 && run({g, g}, 5).side > 0 && run({h, f, h, f}, 5).side > 0);
  CHECK(sparc_ctx_set_timing(ctx, 1) == SPARC_OK);
  CHECK(run({h, g}, 30).side == 0);
  CHECK(sparc_ctx_set_timing(ctx, 0) == SPARC_OK);

  CHECK(sparc_ctx_set_autotune(ctx, 1) == SPARC_OK);
  s = run({h, g, h, f}, 30);
  CHECK(s.side == 0 && s.timed > 0);
  s = run({h, g, h, f}, 30);
  CHECK(s.side > 0 && s.timed == 0);
  s = run({h, g}, 31);
  CHECK(s.side == 0 && s.timed > 0);
  return 0;
}
