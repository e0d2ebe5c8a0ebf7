// A context that autotunes times the stencil shapes of the form a step takes, row plans or tiles,
// for single calls and plans, keeps the fastest (here, whatever was timed last) and times a
// shape once.
#include "host_case.hpp"

static float falling() {
  static float t = 1000.0f;
  return t *= 0.99f;
}

static std::vector<fake::Launch> steps() {
  std::vector<fake::Launch> s;
  for (const fake::Launch& l : fake::launches)
    if (l.kernel.find("hrow") == 0 || l.kernel.find("hstep") == 0) s.push_back(l);
  return s;
}

static bool same(const fake::Launch& a, const fake::Launch& b) {
  return a.grid.x == b.grid.x && a.block.x == b.block.x && a.lds == b.lds;
}

int main() {
  hipStream_t stream;
  CHECK(hipStreamCreateWithFlags(&stream, hipStreamNonBlocking) == hipSuccess);
  sparc_ctx* ctx;
  CHECK(sparc_ctx_create(0, stream, &ctx) == SPARC_OK);
  CHECK(sparc_ctx_set_autotune(ctx, 1) == SPARC_OK);
  fake::elapsed = falling;
  struct { std::vector<int> n; int n_o, ns; sparc_dtype dt; const char* kernel; } cases[] = {
      {{96, 96, 96}, 6, 64, SPARC_R64, "hrow"},  {{45, 38, 50}, 6, 40, SPARC_C64, "hrow"},
      {{40, 40, 40}, 6, 56, SPARC_R32, "hrow"},  {{48, 48, 48}, 6, 128, SPARC_C128, "hrow"},
      {{64, 64, 64}, 4, 32, SPARC_R64, "hstep"}};
  for (const auto& c : cases) {
    Cell cell(c.n, 2, c.n_o);
    const int64_t nd = (int64_t)c.n[0] * c.n[1] * c.n[2];
    sparc_ham* ham;
    CHECK(sparc_ham_create(ctx, &cell.grid, &cell.atoms, c.dt, &ham) == SPARC_OK);
    char x[64], y[64], w[64];   // no kernel runs: never read
    auto apply = [&]() {
      fake::clear();
      CHECK(fd_hamiltonian_apply(ham, x, nd, y, nd, c.ns, w, (size_t)1 << 60) == SPARC_OK);
      for (const auto& l : steps()) CHECK(l.kernel.find(c.kernel) == 0);
      return steps();
    };
    const auto tuned = apply();
    CHECK(tuned.size() >= 2 * 7 + 1 && tuned.size() % 7 == 1);   // two shapes or more, and the step itself
    CHECK(!same(tuned[0], tuned[7]));
    CHECK(same(tuned.back(), tuned[tuned.size() - 2]));
    const auto later = apply();
    CHECK(later.size() == 1 && same(later[0], tuned.back()));

    // a plan of the same cell twice, and one of two chunk widths
    Cell other({c.n[0] + 1, 18, 17}, 1, c.n_o);
    sparc_ham* small;
    CHECK(sparc_ham_create(ctx, &other.grid, &other.atoms, c.dt, &small) == SPARC_OK);
    for (sparc_ham* second : {ham, small}) {
      sparc_ham* const h[] = {ham, second};
      int64_t nd2, ne;
      int32_t np;
      sparc_ham_info(second, &nd2, &np, &ne);
      void* const X[] = {x, y};
      const int64_t ld[] = {nd, nd2};
      const int32_t ns[] = {c.ns, 5}, deg[] = {3, 2};
      const size_t bytes = sparc_filter_plan_workspace_bytes(2, h, ns, deg);
      Block work(bytes / 8 + 1);
      const double lo[] = {1.0, 1.0}, hi[] = {2.0, 2.0};
      std::vector<fake::Launch> run[2];
      for (int k = 0; k < 2; ++k) {
        sparc_filter_plan* plan;
        fake::clear();
        CHECK(sparc_filter_plan_create(ctx, 2, h, X, ld, ns, deg, 0, work.p, bytes, &plan) == SPARC_OK);
        const size_t timed = steps().size();
        CHECK(k == 0 ? timed >= 2 * 7 && timed % 7 == 0 : timed == 0);
        fake::clear();
        CHECK(sparc_filter_plan_run(plan, lo, hi) == SPARC_OK);
        run[k] = steps();
        sparc_filter_plan_destroy(plan);
      }
      CHECK(run[0].size() == run[1].size());
      for (size_t i = 0; i < run[0].size(); ++i) CHECK(same(run[0][i], run[1][i]));
    }
  }
  return 0;
}
