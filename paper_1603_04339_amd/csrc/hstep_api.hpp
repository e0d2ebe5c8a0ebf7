// Stencil step kernels: shared declarations (argument block, tile shapes, launch
// planning) between the launch code and the per-element-type kernel instances.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <vector>

#include "devmath.hpp"

namespace sparc {

template <typename E>
struct StepArgs {
  typedef typename elem<E>::real R;
  int n1, n2, n3;
  int tiles_x, zchunk;
  int tiles, nz;     // tiles per plane, z chunks
  int ns;            // orbitals
  int64_t ldx, ldz, ldo;
  const E* __restrict__ x;
  const E* z;
  E* out;
  const R* __restrict__ veff;
  R centre;        // a * centre coefficient of -1/2 Lap_h
  R tx[8], ty[8], tz[8];
  R va, vb, zc;    // out = lap*a + (a V + b) x + zc z
  double kl[3];    // k_s L_s
  int dmask;       // bit s: zero Dirichlet conditions along direction s
  const E* zplane; // one plane of zeros (read for planes past a Dirichlet z face)
  // Non-local operator applied inside the step (nl_val != nullptr): at every stored
  // node with projector support, out += nla * sum_P gamma_P chi~_P(g) alpha_P(x), from
  // the entry list of each (tile, plane), one entry per (node, atom)
  const int32_t* nl_tpp;    // [tiles * n3 + 1] first entry of (tile, plane)
  const int32_t* nl_ent;    // node | slot << 16
  const E* nl_val;          // [entry * 4 + p] chi~ of the slot's projector p at the node (0 past its own)
  const int32_t* nl_slots;  // [tiles * nl_smax] atoms meeting each column tile (-1: none)
  int nl_smax;              // slots per tile
  const int32_t* atom_pbeg; // first projector of each projector-carrying atom
  const R* gamma;           // [projectors] gamma_P
  const E* alpha;           // projections of x: alpha[P * lda + orbital] (dV included)
  int lda;
  R nla;                    // scale of the projector term (the step's a)
  // row form (hrow_impl.hpp): threads along x and y of a tile, LDS row pitch in chunks
  int txt, tyt, px;
  R pc[3], ps[3];    // e^{i k_s L_s}
};

// dynamic LDS bytes of a fused step launch (after plan_problem): the tile's scaled
// projections of the work-group's orbital, two planes of projector terms (the next
// plane's are accumulated while the current one is computed) and the entry offsets of
// the chunk's planes
template <typename E>
inline size_t nl_lds_bytes(const StepArgs<E>& A, int threads) {
  if (!A.nl_val) return 0;
  const size_t rows = ((size_t)A.nl_smax * 4 * sizeof(E) + 15) / 16 * 16;
  return rows + 2 * (size_t)threads * sizeof(E) + ((size_t)A.zchunk + 1) * 4;
}

// ------------------------------------------------------------ launch planning
// Tile shapes (TX x TY threads).  Without autotuning the choice is the shape with
// the least idle work (tiles that divide n1, n2) weighted by its halo overhead;
// SPARC_HSTEP_TILE (an index into this list) overrides it.
struct TileShape { int tx, ty; };
static const TileShape kTiles[] = {{32, 8}, {32, 16}, {64, 8}, {16, 16}, {48, 8}, {32, 32}, {40, 8}};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);

// z chunks of one orbital's column tile: enough work-groups to fill the chip, at least
// 4 n_o planes per chunk (2 n_o when the step's three blocks, `step_bytes`, stay
// cache-resident, so that the 2 n_o extra planes each chunk reads come from the cache);
// returns the chunk length (the chunk count is ceil(n3 / length))
inline int plan_zchunk(int n3, int64_t tiles, int no, int n_s, int n_cu, double step_bytes = 1e300) {
  const int64_t base = tiles * n_s;
  int nz = 1;
  const int64_t want = 8 * (int64_t)n_cu;
  const int min_len = step_bytes <= 128e6 ? 2 * no : 4 * no;
  while (base * nz < want && n3 / (nz * 2) >= min_len) nz *= 2;
  return (n3 + nz - 1) / nz;
}

// per-problem grid bookkeeping for a tile shape; returns the number of work-groups
template <typename E>
inline int64_t plan_problem(StepArgs<E>& A, int tx, int ty, int no, int n_s, int n_cu) {
  A.tiles_x = (A.n1 + tx - 1) / tx;
  const int tiles_y = (A.n2 + ty - 1) / ty;
  A.tiles = A.tiles_x * tiles_y;
  A.zchunk = plan_zchunk(A.n3, A.tiles, no, n_s, n_cu, 3.0 * A.n1 * A.n2 * A.n3 * n_s * sizeof(E));
  A.nz = (A.n3 + A.zchunk - 1) / A.zchunk;
  A.ns = n_s;
  return (int64_t)A.tiles * A.nz * n_s;
}

// ------------------------------------------------------------ row form
// Step kernel over tiles of whole grid rows (hrow_impl.hpp).  A thread owns a chunk of vx
// reals along x (up to 16 bytes) in each of vy neighbouring rows.
constexpr int kRowNO = 6;          // stencil half-width of the row form's kernels
constexpr int kRowThreads = 768;   // most threads of a row-form work-group (168 registers each)
constexpr size_t kRowLds = 163840; // LDS of a CU
struct RowCfg {
  int vx, vy;   // reals along x and rows per thread (vx = 0: problems of several widths)
  int hm;       // y-halo chunks per thread (1 or 2)
  int full;     // every thread and every row of every tile is inside the grid
  int nt;       // threads per work-group
  size_t lds;   // dynamic LDS bytes
};

// Chunk shape for rows of n1 nodes (cp reals of rb bytes each): the widest chunk up to 16
// bytes that divides a row, in two rows, or a narrower one in four (13 z planes of it live
// in registers either way).
inline void row_chunk(int n1, int cp, int rb, int* vx, int* vy) {
  const int wide = 16 / rb;
  int v = wide;
  while (v > cp && (n1 * cp) % v) v /= 2;
  *vx = v;
  *vy = v == wide ? 2 : 4;
}

// Tile of one problem of n1 x n2 x n3 nodes and n_s orbitals (vx = 0: no tile fits).
struct RowPlan {
  RowCfg cfg{};
  int txt = 0, tyt = 0, px = 0, tiles = 0, zchunk = 0, nz = 0;
  double dur = 0;   // modelled time of a work-group
  double cost = 0;  // and of the launch, us
  int64_t wg(int n_s) const { return (int64_t)tiles * nz * n_s; }
};

// What a launch of several problems imposes on the plan of one of them.
struct RowLaunch {
  int max_nt = kRowThreads;   // most threads of a work-group
  int nt = 0;                 // the launch's threads per work-group (0: the plan's own)
  bool uneven = false;        // grids differ
  bool mixed = false;         // chunk widths differ: one kernel, with the registers of all
};

// Tile height and z chunks for chunk shape (vx, vy).
// The cost of a candidate is its rounds of resident work-groups (k per CU) times its plane steps (and
// the prologue's).  A step takes the root of the squares of its latency, a base and a share per 16
// bytes of the tile, more with fewer than eight waves on the CU, and of the CU's time for the tiles
// of all k, by 16 bytes of tile and of y halo; more than four waves that do not fill the four SIMDs
// evenly cost by how uneven they are.  Chunks narrower than 16 bytes and complex double ones,
// whose x taps read a chunk each, have rates of their own; chunks of one float hold half the
// registers, so four waves fit a SIMD instead of three, and a latency of their own.
// Fitted to 12300 timed (tile, chunk) pairs of 952 blocks from 16^3 x 2 to 96^3 x 512 in all four types.
// Over these the choice costs 1.3 % on average against the fastest timed pair in FP64, 1.6 in FP32 and
// 3.0 in complex single (with the longer of latency and rate in a step's place and fixed prices for
// uneven waves 3.9 to 8.5 %: 80^3 x 60 FP64 207 us then and 179 now, tiled 180; 48^3 x 384 FP32 160
// and 126, tiled 156; 40^3 x 300 complex double 399 and 309, tiled 371).  In complex double the
// choice takes 0.69 of the tiled form's time over 136 blocks, at most 1.03.
// Launches of uneven grids: rounds need not be whole, and what is lost is part of the last
// work-groups' time.  all: every candidate is added to it.
inline RowPlan row_plan(int n1, int n2, int n3, int cp, int rb, int vx, int vy, int64_t n_s, int n_cu,
                        const RowLaunch& launch = RowLaunch(), std::vector<RowPlan>* all = nullptr) {
  RowPlan best;
  const int txt = n1 * cp / vx;
  const int hc = (kRowNO * cp + vx - 1) / vx;
  const int px = txt + 2 * hc;
  const size_t cb = (size_t)vx * rb;
  const bool c128 = cp == 2 && rb == 8, single = cb == 4;
  // step latency, its growth and the CU's rates, us (per 16 bytes of the tile or its halo); the
  // price of few waves and of uneven SIMDs; planes that a chunk's first loads cost
  const double lat = single ? 1.45 : (c128 ? 1.55 : 1.1), lat_chunk = c128 ? 0.22e-3 : 0.26e-3;
  const double rate = c128 ? 1.55e-3 : (cb < 16 ? 2.7e-3 : 1.9e-3), halo_rate = c128 ? 0.94e-3 : 0.43e-3;
  const double few_waves = c128 ? 0.8 : 0.4, uneven_simds = c128 ? 1.0 : 0.5, prologue = c128 ? 2.0 : 1.0;
  double best_cost = 1e300;
  int last = 0;
  for (int tiles = 1; tiles <= n2; ++tiles) {
    const int ty = ((n2 + tiles - 1) / tiles + vy - 1) / vy * vy;
    if (ty == last) continue;
    last = ty;
    const int tyt = ty / vy, tl = (n2 + ty - 1) / ty;
    const int nt = (txt * tyt + 63) / 64 * 64;
    if (nt > launch.max_nt) continue;
    const int hm = (2 * kRowNO * txt + nt - 1) / nt;
    if (hm > 2) break;   // lower tiles need more
    const size_t lds = (size_t)(2 * (ty + 2 * kRowNO) * px + 1) * cb;
    if (lds > kRowLds) continue;
    const int64_t occ = std::max(1, std::min<int>((single && !launch.mixed ? 16 : 12) / (std::max(nt, launch.nt) / 64),
                                                  (int)(kRowLds / lds)));
    const double chunks = (double)nt * vy * (double)cb / 16.0, halo = 2.0 * kRowNO * txt * (double)cb / 16.0;
    const bool full = n2 % ty == 0 && txt * tyt == nt;
    const double simd = (nt + 255) / 256 * 256.0 / nt;   // waves of the fullest SIMD to the average
    const double slow = nt > 256 ? 1.0 + uneven_simds * (simd - 1.0) : 1.0;
    for (int nz = 1; nz == 1 || n3 / nz >= 3; ++nz) {
      const int zc = (n3 + nz - 1) / nz, nzr = (n3 + zc - 1) / zc;
      const int64_t wg = (int64_t)tl * nzr * n_s;
      const int64_t k = std::max<int64_t>(1, std::min<int64_t>(occ, (wg + n_cu - 1) / n_cu));
      const double r = (double)wg / ((double)n_cu * k);
      const double few = 1.0 + few_waves * std::max(0.0, 1.0 - k * nt / 512.0);
      const double step =
          slow * std::hypot(few * (lat + lat_chunk * chunks), k * (rate * chunks + halo_rate * halo));
      const double rounds = launch.uneven ? std::max(1.0, r) + 0.3 : (r < 6 ? std::ceil(r) : r + 0.5);
      const double dur = (zc + prologue) * step, cost = 2.0 + rounds * dur;
      if (all || cost < best_cost * 0.999) {
        RowPlan p;
        p.cfg = RowCfg{vx, vy, hm, full ? 1 : 0, nt, lds};
        p.txt = txt;
        p.tyt = tyt;
        p.px = px;
        p.tiles = tl;
        p.zchunk = zc;
        p.nz = nzr;
        p.dur = dur / k;
        p.cost = cost;
        if (all) all->push_back(p);
        if (cost < best_cost * 0.999) {
          best_cost = cost;
          best = p;
        }
      }
      if (wg > 16 * (int64_t)n_cu) break;
    }
  }
  return best;
}

// the plan's fields of a step's arguments
template <typename E>
inline void row_fill(StepArgs<E>& A, const RowPlan& p, int n_s) {
  A.txt = p.txt;
  A.tyt = p.tyt;
  A.px = p.px;
  A.tiles = p.tiles;
  A.zchunk = p.zchunk;
  A.nz = p.nz;
  A.ns = n_s;
}

// one launch of the row form: a single problem, or a device table of n problems with
// their work-group offsets (hasz: the steps read the recurrence operand)
template <typename E>
int hrow_single(sparc_ctx* ctx, const StepArgs<E>& A, const RowCfg& c, int64_t total);
template <typename E>
int hrow_batched(sparc_ctx* ctx, const void* dprobs, const int* dwg, int n, int64_t total, const RowCfg& c, int hasz);

// one stencil step launch (single problem) with stencil order no and tile shape t
template <typename E>
int hstep_single(sparc_ctx* ctx, StepArgs<E>& A, int32_t n_s, int no, int t);
// one batched stencil step launch over a device table of n problems (dir: some problem
// has a Dirichlet direction; nl_lds: dynamic LDS bytes of the widest fused problem, 0
// when no problem applies its projectors inside the step)
template <typename E>
int hstep_batched(sparc_ctx* ctx, const void* dprobs, const int* dwg, int n, int64_t total, int no, int t, int dir,
                  size_t nl_lds);

}  // namespace sparc
