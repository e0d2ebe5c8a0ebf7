// Row form of the stencil step (fused stencil + local potential + recurrence), for cells
// periodic in all directions and the 12th-order stencil.
//
// One work-group = a tile of whole grid rows (TY of them) of one orbital and a chunk of z
// planes.  A thread owns a chunk of VX reals along x (16 bytes where the row length allows
// it) in each of VY neighbouring rows, and streams along z with the 2 NO + 1 planes of its
// chunks in registers.  The current plane, with NO rows above and below and NO columns on
// both sides, is staged in LDS (double-buffered, one barrier per plane): the columns come
// from the tile's own ends (the row is whole, so its periodic image is inside the tile),
// the rows from global memory.
//
// What bounds it, and why this shape.  A plane step moves 4 reals of HBM traffic per node
// and needs 37 of its values: with one value per thread the taps cost 24 8-byte LDS reads
// per node, 192 bytes, and the halo of a 32 x 16 tile 1.1 extra reads of x per node, which
// arrive from beyond L2 (the tile's neighbours read those lines six planes earlier).  Whole
// rows need no x halo, 16-byte chunks in two rows need 6 16-byte LDS reads per node, and 32
// rows of 96 nodes fetch 0.38 extra values.  Large blocks are then bound by HBM: a bare
// z-march (two reads, one write, no stencil) over the same 96^3 x 512 blocks streams 5.1-5.4
// TB/s (memory is walked in one stream per work-group; a single linear walk reaches 6.4).
// Measured per step of a filter, FP64 (32 x 16-tile kernel or point form -> this one, as planned):
// 96^3 x 512 2.51 -> 2.19 ms, 80^3 x 256 0.78 -> 0.68 ms, 64^3 x 128 0.203 -> 0.151 ms, 48^3 x 64 47
// -> 43 us, 40^3 x 56 34 -> 24 us, 32^3 x 32 42 -> 11.5 us.  A recurrence step of 96^3 x 512 takes
// 2.27 ms as planned, three z chunks (14.8 -> 11.6 GB fetched), and 2.20 in one chunk, which the
// tuner finds (9.4 GB; 5.0 TB/s of 24 B per node).
// Registers are what limits the tile: VX = 2, VY = 2 doubles hold 104 for the queue, so the
// taps are applied in small groups of LDS reads pinned in order (the scheduler would
// otherwise hoist all 24 reads and spill).
#pragma once
#include <atomic>

#include "hstep_api.hpp"

namespace sparc {

template <typename T, int N>
struct vec_of {
  typedef T reg __attribute__((ext_vector_type(N)));
  typedef T mem __attribute__((ext_vector_type(N), aligned(sizeof(T))));   // rows need not be 16-byte aligned
};

// keeps the value where it is in the instruction stream
template <typename T>
__device__ __forceinline__ void pin_reg(T& t) {
  asm volatile("" : "+v"(t));
}
template <int N, typename V>
__device__ __forceinline__ void pin_vec(V& x) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    auto t = x[i];
    pin_reg(t);
    x[i] = t;
  }
}

// (re, im) pairs of a chunk times (c, s) where `on`
template <int VX, typename V, typename R>
__device__ __forceinline__ void rot_chunk(V& x, R c, R s, bool on) {
#pragma unroll
  for (int e = 0; e < VX; e += 2) {
    const R re = x[e], im = x[e + 1];
    x[e] = on ? c * re - s * im : re;
    x[e + 1] = on ? c * im + s * re : im;
  }
}

// Range-checked access: an offset past `bytes` reads zero and is not written.  Lanes past
// the tile and rows past the grid use it with an offset of ~0.
template <int BYTES, typename M>
__device__ __forceinline__ M buf_load(const void* base, unsigned bytes, unsigned off) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00027000);
  if constexpr (BYTES == 16) return __builtin_bit_cast(M, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 2));
  else if constexpr (BYTES == 8) return __builtin_bit_cast(M, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 2));
  else return __builtin_bit_cast(M, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 2));
}
template <int BYTES, typename M>
__device__ __forceinline__ void buf_store(M v, void* base, unsigned bytes, unsigned off) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00027000);
  if constexpr (BYTES == 16) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), r, off, 0, 2);
  else if constexpr (BYTES == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, off, 0, 2);
  else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, off, 0, 2);
}

// L: the work-group's index in the order (tiles, z chunks, orbitals), tiles fastest: the
// work-groups of one orbital sit side by side on one XCD and share their halo planes in L2.
// NTP: the threads that work on this problem (the others only keep the barriers).
template <typename E, int VX, int VY, int HM, bool FULL, bool HASZ>
__device__ __forceinline__ void hrow_body(const StepArgs<E>& A, int64_t L, int NTP, char* smem) {
  typedef typename elem<E>::real R;
  typedef typename vec_of<R, VX>::reg V;
  typedef typename vec_of<R, VX>::mem GV;
  constexpr int NO = kRowNO;
  constexpr int CP = elem<E>::is_cplx ? 2 : 1;
  constexpr int HC = (NO * CP + VX - 1) / VX;   // chunks of the x halo on one side
  constexpr int NV = VX / CP;                   // nodes of a chunk
  typedef typename vec_of<R, NV>::reg VN;
  typedef typename vec_of<R, NV>::mem GVN;
  V* planes = (V*)smem;
  const int TXT = A.txt, TY = A.tyt * VY, ROWS = TY + 2 * NO, PX = A.px;
  const int n2 = A.n2, n3 = A.n3;
  const int yt = (int)(L % A.tiles);
  L /= A.tiles;
  const int zi = (int)(L % A.nz);
  const int n = (int)(L / A.nz);
  const int zb = zi * A.zchunk, ze = min(n3, zb + A.zchunk);
  const int tid = threadIdx.x;
  if (__builtin_amdgcn_readfirstlane(tid) >= NTP) {
    for (int z = zb; z < ze; ++z) __syncthreads();
    return;
  }
  const int rowr = A.n1 * CP;               // reals per row
  const int plane_r = rowr * n2;            // reals per plane
  const int tx = tid % TXT;
  const int ty = min(tid / TXT, A.tyt - 1); // lanes past the tile repeat its last row and store nothing
  const int y0 = yt * TY;
  const R* __restrict__ xc = (const R*)(A.x + (int64_t)n * A.ldx);
  // byte offsets of the own rows inside a plane (FULL: row v is row 0 plus v rows)
  unsigned off[VY];
  unsigned soff[VY];   // the same for the masked accesses (~0: outside)
  const int rowv = FULL ? rowr : 0;
  int yw = 0;          // bit v: own row v is the image of a row across the y face
#pragma unroll
  for (int v = 0; v < VY; ++v) {
    const int gy = y0 + VY * ty + (FULL ? 0 : v);
    const bool wr = !FULL && gy >= n2;
    yw |= wr ? 1 << v : 0;
    off[v] = (unsigned)(((wr ? gy - n2 : gy) * rowr + VX * tx) * (int)sizeof(R));
    soff[v] = (FULL || (!wr && tid < TXT * A.tyt)) ? off[v] : ~0u;
  }
  unsigned h_off[HM];
  int h_lds[HM];
  int h_w[HM];   // y wrap of the halo row
  const int spare = 2 * ROWS * PX;
#pragma unroll
  for (int u = 0; u < HM; ++u) {
    const int c = tid + u * NTP;
    h_lds[u] = -1;
    h_off[u] = 0;
    h_w[u] = 0;
    if (c < 2 * NO * TXT) {
      const int r = c / TXT, cx = c % TXT;
      const int rel = r < NO ? r - NO : TY + r - NO;
      int gy = y0 + rel;
      h_w[u] = gy < 0 ? -1 : (gy >= n2 ? 1 : 0);
      gy -= h_w[u] * n2;
      h_off[u] = (unsigned)((gy * rowr + VX * cx) * (int)sizeof(R));
      h_lds[u] = (rel + NO) * PX + HC + cx;
    }
  }
  const int own = (VY * ty + NO) * PX + HC + tx;
  // the row's ends are also the halo of its other end
  const int edge = tx < HC ? TXT : (tx >= TXT - HC ? -TXT : 0);
  auto ldv = [](const R* p, unsigned o) -> V { return (V)(*(const GV*)((const char*)p + o)); };
  // Bloch rotation of own values from plane image wz
  auto own_rot = [&](V (&x)[VY], int wz) {
    if constexpr (CP == 2) {
      if (wz != 0) {
#pragma unroll
        for (int v = 0; v < VY; ++v) rot_chunk<VX>(x[v], A.pc[2], wz > 0 ? A.ps[2] : -A.ps[2], true);
      }
      if constexpr (!FULL) {
#pragma unroll
        for (int v = 0; v < VY; ++v) rot_chunk<VX>(x[v], A.pc[1], A.ps[1], (yw >> v) & 1);
      }
    }
  };

  // q[d]: own values of plane z - NO + d; the plane of the next load and its image
  V q[2 * NO + 1][VY];
  int sz = zb - NO, wz = 0;
  if (sz < 0) {
    sz += n3;
    wz = -1;
  }
#pragma unroll
  for (int d = 0; d < 2 * NO; ++d) {
    const R* __restrict__ p = xc + (int64_t)plane_r * sz;
#pragma unroll
    for (int v = 0; v < VY; ++v) q[d][v] = ldv(p + v * rowv, off[v]);
    own_rot(q[d], wz);
    if (++sz == n3) {
      sz = 0;
      ++wz;
    }
  }
  V hn[HM];
  {
    const R* __restrict__ p = xc + (int64_t)plane_r * zb;
#pragma unroll
    for (int u = 0; u < HM; ++u) hn[u] = ldv(p, h_off[u]);
  }
  const R* __restrict__ vp = A.veff + (int64_t)(A.n1 * n2) * zb;
  const R* zp = HASZ ? (const R*)(A.z + (int64_t)n * A.ldz) + (int64_t)plane_r * zb : nullptr;
  R* op = (R*)(A.out + (int64_t)n * A.ldo) + (int64_t)plane_r * zb;
  const unsigned plane_b = (unsigned)plane_r * (unsigned)sizeof(R);
  int pb = 0;
  for (int z = zb; z < ze; ++z) {
    V* pl = planes + pb;
    const int pcur = pb;
    pb = ROWS * PX - pb;
#pragma unroll
    for (int v = 0; v < VY; ++v) pl[own + v * PX] = q[NO][v];
    if (edge != 0) {
#pragma unroll
      for (int v = 0; v < VY; ++v) {
        V t = q[NO][v];
        if constexpr (CP == 2) rot_chunk<VX>(t, A.pc[0], edge > 0 ? A.ps[0] : -A.ps[0], true);
        pl[own + edge + v * PX] = t;
      }
    }
#pragma unroll
    for (int u = 0; u < HM; ++u) {
      V t = hn[u];
      if constexpr (CP == 2) rot_chunk<VX>(t, A.pc[1], h_w[u] > 0 ? A.ps[1] : -A.ps[1], h_w[u] != 0);
      planes[h_lds[u] < 0 ? spare : h_lds[u] + pcur] = t;
    }
    // loads of this step, in the order they are waited for: the queue's next plane and the
    // recurrence operand (end of this step), the halo of the next plane (next step)
    const int wq = wz;
    {
      const R* __restrict__ p = xc + (int64_t)plane_r * sz;
#pragma unroll
      for (int v = 0; v < VY; ++v) q[2 * NO][v] = ldv(p + v * rowv, off[v]);
      if (++sz == n3) {
        sz = 0;
        ++wz;
      }
    }
    V zv[VY];
    if constexpr (HASZ) {
#pragma unroll
      for (int v = 0; v < VY; ++v) {
        if constexpr (FULL) zv[v] = (V)__builtin_nontemporal_load((const GV*)((const char*)(zp + v * rowv) + off[v]));
        else zv[v] = buf_load<VX * (int)sizeof(R), V>(zp, plane_b, soff[v]);
      }
    }
    {
      const R* __restrict__ p = xc + (int64_t)plane_r * (z + 1 < ze ? z + 1 : z);
#pragma unroll
      for (int u = 0; u < HM; ++u) hn[u] = ldv(p, h_off[u]);
    }
    __syncthreads();
    // y taps: each LDS row serves the VY own rows within reach
    V acc[VY];
#pragma unroll
    for (int v = 0; v < VY; ++v) {
      acc[v] = (V)(R)0;
#pragma unroll
      for (int w = 0; w < VY; ++w)
        if (w != v) {
          const int d = w > v ? w - v : v - w;
          acc[v] += A.ty[d - 1] * q[NO][w];
        }
    }
#pragma unroll
    for (int j = -NO; j < VY + NO; ++j) {
      if (j >= 0 && j < VY) continue;
      if ((j + NO) % 4 == 0) {
#pragma unroll
        for (int v = 0; v < VY; ++v) pin_vec<VX>(acc[v]);
        __builtin_amdgcn_sched_barrier(0);
      }
      const V c = pl[own + j * PX];
#pragma unroll
      for (int v = 0; v < VY; ++v) {
        const int d = j > v ? j - v : v - j;
        if (d <= NO) acc[v] += A.ty[d - 1] * c;
      }
    }
    // x taps
#pragma unroll
    for (int v = 0; v < VY; ++v) {
#pragma unroll
      for (int w = 0; w < VY; ++w) pin_vec<VX>(acc[w]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = -HC; c <= HC; ++c) {
        const V w = c == 0 ? q[NO][v] : pl[own + v * PX + c];
#pragma unroll
        for (int e = 0; e < VX; ++e)
#pragma unroll
          for (int o = 0; o < VX; ++o) {
            const int P = c * VX + e - o;
            const int d = (P > 0 ? P : -P) / CP;
            if (P % CP == 0 && d >= 1 && d <= NO) acc[v][o] = fma(A.tx[d - 1], w[e], acc[v][o]);
          }
        if (HC > 3 && c != 0 && c % 3 == 0) {
          pin_vec<VX>(acc[v]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
#pragma unroll
    for (int w = 0; w < VY; ++w) pin_vec<VX>(acc[w]);
    __builtin_amdgcn_sched_barrier(0);
    VN vv[VY];
#pragma unroll
    for (int v = 0; v < VY; ++v) vv[v] = (VN)(*(const GVN*)((const char*)(vp + v * (rowv / CP)) + off[v] / CP));
    __builtin_amdgcn_sched_barrier(0);
    own_rot(q[2 * NO], wq);
    // z taps, potential and recurrence
#pragma unroll
    for (int v = 0; v < VY; ++v) {
      V r = A.centre * q[NO][v];
#pragma unroll
      for (int p = 1; p <= NO; ++p) r += A.tz[p - 1] * (q[NO + p][v] + q[NO - p][v]);
      r += acc[v];
#pragma unroll
      for (int e = 0; e < VX; ++e) r[e] = fma(fma(A.va, vv[v][e / CP], A.vb), q[NO][v][e], r[e]);
      if constexpr (HASZ) r += A.zc * zv[v];
      pin_vec<VX>(r);
      if constexpr (FULL) __builtin_nontemporal_store((GV)r, (GV*)((char*)(op + v * rowv) + off[v]));
      else buf_store<VX * (int)sizeof(R)>(r, op, plane_b, soff[v]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < 2 * NO; ++d)
#pragma unroll
      for (int v = 0; v < VY; ++v) q[d][v] = q[d + 1][v];
    vp += A.n1 * n2;
    op += plane_r;
    if constexpr (HASZ) zp += plane_r;
  }
}

// dispatch index -> logical index: every XCD receives one contiguous range
__device__ __forceinline__ int64_t row_order(int64_t L, int64_t G) {
  const int64_t q = G >> 3, r = G & 7, xcd = L & 7, slot = L >> 3;
  return xcd * q + (xcd < r ? xcd : r) + slot;
}

// The arguments are read where they lie, when they are needed: as a plain parameter all of them are
// loaded at the entry and held, more than the scalar registers, and the ones over are kept in lanes of
// vector registers (up to 92 in complex double, whose masked form with two halo chunks a thread then
// spilled to memory).  Over 25 to 32 blocks per type a step takes 0.87 of that time in complex double
// (47 x 40 x 36, 99 orbitals: 147 -> 106 us, tiled 121; 82 x 74 x 48, 54: 312 -> 214) and 0.98 to 1.00
// in the others (96^3 x 256 FP32: 592 -> 579).
template <typename E, int VX, int VY, int HM, bool FULL, bool HASZ>
__global__ __launch_bounds__(kRowThreads) void hrow_kernel(StepArgs<E>) {
  extern __shared__ __align__(16) char row_lds[];
  auto a = (const StepArgs<E> __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr();
  asm("" : "+s"(a));   // not the parameter, for the compiler
  hrow_body<E, VX, VY, HM, FULL, HASZ>(*(const StepArgs<E>*)a, row_order(blockIdx.x, gridDim.x), (int)blockDim.x, row_lds);
}

// Several problems in one launch.  Problem p has the work-groups wg_off[p] <= b <
// wg_off[p+1], padded to a multiple of 8 (the offsets start at wg_off[0]: problems further
// down a table): every XCD takes a contiguous eighth of each problem, so that problems
// whose work-groups take longer than the others' load all of them alike.  Returns the
// work-group's problem and its index there.
template <typename E>
__device__ __forceinline__ const StepArgs<E>& row_problem(const StepArgs<E>* __restrict__ probs,
                                                          const int* __restrict__ wg_off, int n_probs, int64_t* L) {
  const int xcd = blockIdx.x & 7, b = wg_off[0] + (int)(blockIdx.x & ~7u);
  int lo = 0, hi = n_probs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (wg_off[mid] <= b) lo = mid;
    else hi = mid - 1;
  }
  *L = (int64_t)xcd * ((wg_off[lo + 1] - wg_off[lo]) >> 3) + ((b - wg_off[lo]) >> 3);
  return probs[lo];
}

template <typename E, int VX, int VY, int HM, bool FULL, bool HASZ>
__global__ __launch_bounds__(kRowThreads) void hrow_batched_kernel(const StepArgs<E>* __restrict__ probs,
                                                                   const int* __restrict__ wg_off, int n_probs) {
  extern __shared__ __align__(16) char row_lds[];
  int64_t L;
  const StepArgs<E>& A = row_problem(probs, wg_off, n_probs, &L);
  if (L >= (int64_t)A.tiles * A.nz * A.ns) return;
  hrow_body<E, VX, VY, HM, FULL, HASZ>(A, L, (A.txt * A.tyt + 63) / 64 * 64, row_lds);
}

// Problems of several chunk widths in one launch: the width is its problem's for all of a work-group.
template <typename E, bool HASZ>
__global__ __launch_bounds__(kRowThreads) void hrow_mixed_kernel(const StepArgs<E>* __restrict__ probs,
                                                                 const int* __restrict__ wg_off, int n_probs) {
  extern __shared__ __align__(16) char row_lds[];
  constexpr int CP = elem<E>::is_cplx ? 2 : 1, WIDE = 16 / (int)sizeof(typename elem<E>::real);
  int64_t L;
  const StepArgs<E>& A = row_problem(probs, wg_off, n_probs, &L);
  if (L >= (int64_t)A.tiles * A.nz * A.ns) return;
  const int nt = (A.txt * A.tyt + 63) / 64 * 64, vx = A.n1 * CP / A.txt;
  if (vx == WIDE) hrow_body<E, WIDE, 2, 2, false, HASZ>(A, L, nt, row_lds);
  if constexpr (WIDE / 2 >= CP)
    if (vx == WIDE / 2) hrow_body<E, WIDE / 2, 4, 2, false, HASZ>(A, L, nt, row_lds);
  if constexpr (WIDE / 4 >= CP)
    if (vx == WIDE / 4) hrow_body<E, WIDE / 4, 4, 2, false, HASZ>(A, L, nt, row_lds);
}

// a kernel's dynamic LDS limit, raised once per device (the kernel is the template's argument:
// the forms of one element type share a function type)
template <auto Kernel>
static int row_lds_limit(int device) {
  static std::atomic<uint64_t> done{0};
  const uint64_t bit = device < 64 ? 1ull << device : 0;
  if (bit && (done.load() & bit)) return SPARC_OK;
  DeviceScope on(device);
  SPARC_HIP(hipFuncSetAttribute((const void*)Kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kRowLds));
  done.fetch_or(bit);
  return SPARC_OK;
}

template <typename E, int VX, int VY, int HM, bool FULL, bool HASZ>
static int row_launch(sparc_ctx* ctx, const StepArgs<E>* one, const void* probs, const int* wg, int n, int64_t total,
                      const RowCfg& c) {
  if (total > (int64_t)INT32_MAX) return fail(SPARC_ESHAPE, "stencil step: too many work-groups");
  int t;
  if (one) {
    constexpr auto k = hrow_kernel<E, VX, VY, HM, FULL, HASZ>;
    SPARC_TRY(row_lds_limit<k>(ctx->device));
    t = timer_begin(ctx, "hstep");
    k<<<(unsigned)total, c.nt, c.lds, ctx->stream>>>(*one);
  } else {
    constexpr auto k = hrow_batched_kernel<E, VX, VY, HM, FULL, HASZ>;
    SPARC_TRY(row_lds_limit<k>(ctx->device));
    t = timer_begin(ctx, "hstep");
    k<<<(unsigned)total, c.nt, c.lds, ctx->stream>>>((const StepArgs<E>*)probs, wg, n);
  }
  timer_end(ctx, t);
  return check_launch("hrow_kernel");
}

template <typename E, bool HASZ>
static int row_mixed_launch(sparc_ctx* ctx, const void* probs, const int* wg, int n, int64_t total, const RowCfg& c) {
  if (total > (int64_t)INT32_MAX) return fail(SPARC_ESHAPE, "stencil step: too many work-groups");
  constexpr auto k = hrow_mixed_kernel<E, HASZ>;
  SPARC_TRY(row_lds_limit<k>(ctx->device));
  const int t = timer_begin(ctx, "hstep");
  k<<<(unsigned)total, c.nt, c.lds, ctx->stream>>>((const StepArgs<E>*)probs, wg, n);
  timer_end(ctx, t);
  return check_launch("hrow_mixed_kernel");
}

template <typename E, int VX, int VY>
static int row_variant(sparc_ctx* ctx, const StepArgs<E>* one, const void* probs, const int* wg, int n, int64_t total,
                       const RowCfg& c, int hasz) {
#define SPARC_ROW(HM, FULL, HASZ) return row_launch<E, VX, VY, HM, FULL, HASZ>(ctx, one, probs, wg, n, total, c)
  if (c.hm == 1) {
    if (c.full) { if (hasz) SPARC_ROW(1, true, true); SPARC_ROW(1, true, false); }
    if (hasz) SPARC_ROW(1, false, true);
    SPARC_ROW(1, false, false);
  }
  if (c.full) { if (hasz) SPARC_ROW(2, true, true); SPARC_ROW(2, true, false); }
  if (hasz) SPARC_ROW(2, false, true);
  SPARC_ROW(2, false, false);
#undef SPARC_ROW
}

template <typename E>
static int row_any(sparc_ctx* ctx, const StepArgs<E>* one, const void* probs, const int* wg, int n, int64_t total,
                   const RowCfg& c, int hasz) {
  constexpr int cp = elem<E>::is_cplx ? 2 : 1;
  constexpr int wide = 16 / (int)sizeof(typename elem<E>::real);
  if (c.vx == wide && c.vy == 2) return row_variant<E, wide, 2>(ctx, one, probs, wg, n, total, c, hasz);
  if constexpr (wide / 2 >= cp)
    if (c.vx == wide / 2 && c.vy == 4) return row_variant<E, wide / 2, 4>(ctx, one, probs, wg, n, total, c, hasz);
  if constexpr (wide / 4 >= cp)
    if (c.vx == wide / 4 && c.vy == 4) return row_variant<E, wide / 4, 4>(ctx, one, probs, wg, n, total, c, hasz);
  return fail(SPARC_EINVAL, "stencil step: no row kernel for chunk %d x %d", c.vx, c.vy);
}

template <typename E>
int hrow_single(sparc_ctx* ctx, const StepArgs<E>& A, const RowCfg& c, int64_t total) {
  return row_any<E>(ctx, &A, nullptr, nullptr, 1, total, c, A.z != nullptr);
}

template <typename E>
int hrow_batched(sparc_ctx* ctx, const void* dprobs, const int* dwg, int n, int64_t total, const RowCfg& c, int hasz) {
  if (total <= 0) return SPARC_OK;
  if constexpr (!(elem<E>::is_cplx && sizeof(typename elem<E>::real) == 8))   // (one width)
    if (c.vx == 0)
      return hasz ? row_mixed_launch<E, true>(ctx, dprobs, dwg, n, total, c)
                  : row_mixed_launch<E, false>(ctx, dprobs, dwg, n, total, c);
  return row_any<E>(ctx, nullptr, dprobs, dwg, n, total, c, hasz);
}

}  // namespace sparc
