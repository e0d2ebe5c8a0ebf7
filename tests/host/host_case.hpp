// What the host-code tests share: checks, a small cell and blocks of device memory.
#pragma once
#include "fake_hip.hpp"
#include "sparc_hip.h"

#define CHECK(c)                                                                                   \
  do {                                                                                             \
    if (!(c)) {                                                                                    \
      printf("%s:%d: %s (last error: %s)\n", __FILE__, __LINE__, #c, sparc_last_error());           \
      exit(1);                                                                                     \
    }                                                                                              \
  } while (0)

struct Block {
  void* p = nullptr;
  size_t n;
  explicit Block(size_t doubles) : n(doubles * 8) { hipMalloc(&p, n); }
  ~Block() { hipFree(p); }
  size_t bytes() const { return n; }
};

// n_atoms atoms along the diagonal with one s projector each
struct Cell {
  sparc_grid grid{};
  sparc_atoms atoms{};
  std::vector<double> R, one, gamma, rc;
  std::vector<int32_t> chan, l;
  Cell(std::vector<int> n, int n_atoms, int n_o = 6) {
    for (int s = 0; s < 3; ++s) {
      grid.n[s] = n[s];
      grid.L[s] = 0.5 * n[s];
    }
    grid.n_o = n_o;
    for (int a = 0; a < n_atoms; ++a) {
      for (int s = 0; s < 3; ++s) R.push_back(grid.L[s] * (a + 0.5) / n_atoms);
      chan.push_back(a);
    }
    one.assign(n_atoms, 1.0);
    gamma.assign(n_atoms, 0.3);
    rc.assign(n_atoms, 1.6);
    l.assign(n_atoms, 0);
    atoms.n_atoms = atoms.n_chan = n_atoms;
    atoms.R = R.data();
    atoms.vloc_depth = atoms.vloc_width = atoms.Z = one.data();
    atoms.chan_atom = chan.data();
    atoms.chan_l = l.data();
    atoms.chan_gamma = gamma.data();
    atoms.chan_rc = rc.data();
  }
};
