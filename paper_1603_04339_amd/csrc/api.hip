// C-ABI entry points of the CheFSI hot path: H*X, Chebyshev filter,
// Rayleigh-Ritz, Lanczos bounds, density and Fermi level.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "devmath.hpp"

namespace sparc {

// ------------------------------------------------------------ workspace carving
struct Carver {
  char* p;
  size_t left;
  bool ok = true;
  void* take(size_t bytes) {
    size_t b = ((bytes + 255) / 256) * 256;
    if (b > left) { ok = false; return nullptr; }
    void* q = p;
    p += b;
    left -= b;
    return q;
  }
};
static size_t al(size_t b) { return ((b + 255) / 256) * 256; }

int check_ham(const sparc_ham* H, const char* who) {
  if (!H) return fail(SPARC_EINVAL, "%s: ham is NULL", who);
  return SPARC_OK;
}

int check_block(const sparc_ham* H, const void* X, int64_t ldx, int32_t n_s, const char* who) {
  if (!X) return fail(SPARC_EINVAL, "%s: block pointer is NULL", who);
  if (n_s < 1) return fail(SPARC_ESHAPE, "%s: n_s=%d < 1", who, n_s);
  if (ldx < H->n_d) return fail(SPARC_ESHAPE, "%s: ld=%lld < N_d=%lld", who, (long long)ldx, (long long)H->n_d);
  return SPARC_OK;
}

// ------------------------------------------------------------ small element-wise kernels
template <typename E>
__global__ void scale_by_rnorm_kernel(const E* __restrict__ x, E* __restrict__ y, int64_t n, const double* nrm2) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  double s = 1.0 / sqrt(nrm2[0]);
  y[i] = scale((typename elem<E>::real)s, x[i]);
}

template <typename E>
__global__ void sub_kernel(E* __restrict__ w, const E* __restrict__ t, int64_t n) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) w[i] = w[i] + scale((typename elem<E>::real)-1, t[i]);
}

__global__ void herm_sym_kernel(int n, double* A, int cplx) {
  int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= (int64_t)n * n) return;
  int i = (int)(idx % n), j = (int)(idx / n);
  if (i > j) return;
  if (!cplx) {
    double v = 0.5 * (A[i + (int64_t)j * n] + A[j + (int64_t)i * n]);
    A[i + (int64_t)j * n] = v;
    A[j + (int64_t)i * n] = v;
  } else {
    double* a = A + 2 * (i + (int64_t)j * n);
    double* b = A + 2 * (j + (int64_t)i * n);
    double re = 0.5 * (a[0] + b[0]), im = 0.5 * (a[1] - b[1]);
    if (i == j) im = 0;
    a[0] = re; a[1] = im;
    b[0] = re; b[1] = -im;
  }
}

// Lanczos: coefficients -> tridiagonal matrix (dense, n x n) and bookkeeping
__global__ void lanczos_record_kernel(const double* c, int j, int cplx, double* alph) {
  if (threadIdx.x == 0 && blockIdx.x == 0) alph[j] = c[cplx ? 2 * j : j];
}
__global__ void lanczos_beta_kernel(const double* nrm2, int j, double* beta) {
  if (threadIdx.x == 0 && blockIdx.x == 0) beta[j] = sqrt(nrm2[0]);
}
__global__ void tridiag_kernel(int m, const double* alph, const double* beta, double* T) {
  int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= m * m) return;
  int i = idx % m, j = idx / m;
  double v = 0;
  if (i == j) v = alph[i];
  else if (i == j + 1) v = beta[j];
  else if (j == i + 1) v = beta[i];
  T[idx] = v;
}

// ------------------------------------------------------------ density
constexpr int MAXK = 64;
template <typename E>
struct DensArgs {
  const E* x[MAXK];
  int64_t ld[MAXK];
};

template <typename E>
__global__ __launch_bounds__(256) void density_kernel(DensArgs<E> A, int nk, int n_s, int64_t n_d,
                                                      const double* __restrict__ occ, double scale_,
                                                      double* __restrict__ rho) {
  int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (g >= n_d) return;
  double acc = 0;
  for (int b = 0; b < nk; ++b) {
    const E* __restrict__ x = A.x[b];
    const int64_t ld = A.ld[b];
    const double* oc = occ + (int64_t)b * n_s;
    int n = 0;
    for (; n + 4 <= n_s; n += 4) {
      E v0 = x[g + (int64_t)n * ld], v1 = x[g + (int64_t)(n + 1) * ld];
      E v2 = x[g + (int64_t)(n + 2) * ld], v3 = x[g + (int64_t)(n + 3) * ld];
      acc += oc[n] * abs2(v0) + oc[n + 1] * abs2(v1) + oc[n + 2] * abs2(v2) + oc[n + 3] * abs2(v3);
    }
    for (; n < n_s; ++n) acc += oc[n] * abs2(x[g + (int64_t)n * ld]);
  }
  rho[g] = scale_ * acc;
}

// ------------------------------------------------------------ Fermi level
struct FermiArgs {
  double wk[MAXK];
};
__global__ __launch_bounds__(256) void fermi_kernel(int nk, int ns, const double* __restrict__ lam, FermiArgs W,
                                                    double ne, double kT, double* __restrict__ occ_w,
                                                    double* __restrict__ mu_out) {
  __shared__ double red[4];
  __shared__ double s_lo, s_hi;
  const int tid = threadIdx.x;
  const int tot = nk * ns;
  double lmin = 1e300, lmax = -1e300;
  for (int i = tid; i < tot; i += blockDim.x) { lmin = fmin(lmin, lam[i]); lmax = fmax(lmax, lam[i]); }
  // block min / max
  for (int o = 32; o > 0; o >>= 1) {
    lmin = fmin(lmin, __shfl_xor(lmin, o, 64));
    lmax = fmax(lmax, __shfl_xor(lmax, o, 64));
  }
  __shared__ double mn[4], mx[4];
  if ((tid & 63) == 0) { mn[tid >> 6] = lmin; mx[tid >> 6] = lmax; }
  __syncthreads();
  if (tid == 0) {
    double a = mn[0], b = mx[0];
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i) { a = fmin(a, mn[i]); b = fmax(b, mx[i]); }
    s_lo = a - 40.0 * kT - 1.0;
    s_hi = b + 40.0 * kT + 1.0;
  }
  __syncthreads();
  double lo = s_lo, hi = s_hi;
  auto count = [&](double mu) {
    double c = 0;
    for (int i = tid; i < tot; i += blockDim.x) {
      int b = i / ns;
      c += 2.0 * W.wk[b] * 0.5 * (1.0 - tanh((lam[i] - mu) / (2.0 * kT)));
    }
    c = wave_sum(c);
    __syncthreads();
    if ((tid & 63) == 0) red[tid >> 6] = c;
    __syncthreads();
    double s = 0;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s += red[i];
    return s;
  };
  // Brent's method (inverse quadratic interpolation or secant inside a bracket, with
  // bisection whenever the interpolated step is not safely inside it or shrinks too
  // slowly) on f(mu) = count(mu) - ne, which increases with mu; f(lo) < 0 < f(hi).
  // Every thread runs the same scalar iteration on the block-reduced counts.
  double a = lo, b = hi, fa = count(lo) - ne, fb = count(hi) - ne;
  if (fabs(fa) < fabs(fb)) { double t = a; a = b; b = t; t = fa; fa = fb; fb = t; }
  double c = a, fc = fa, d = a;
  bool bisected = true;
  for (int it = 0; it < 200; ++it) {
    if (fabs(fb) < 1e-13 * ne || fabs(b - a) < 1e-15 * fmax(1.0, fabs(b))) break;
    double s;
    if (fa != fc && fb != fc) {  // inverse quadratic interpolation through (a, fa), (b, fb), (c, fc)
      s = a * fb * fc / ((fa - fb) * (fa - fc)) + b * fa * fc / ((fb - fa) * (fb - fc)) +
          c * fa * fb / ((fc - fa) * (fc - fb));
    } else {  // secant through (a, fa), (b, fb)
      s = b - fb * (b - a) / (fb - fa);
    }
    const double q = 0.25 * (3.0 * a + b);
    const double tol = 1e-15 * fmax(1.0, fabs(b));
    const bool outside = !((s > fmin(q, b)) && (s < fmax(q, b)));
    const bool slow = bisected ? (fabs(s - b) >= 0.5 * fabs(b - c) || fabs(b - c) < tol)
                               : (fabs(s - b) >= 0.5 * fabs(c - d) || fabs(c - d) < tol);
    if (outside || slow || !isfinite(s)) {
      s = 0.5 * (a + b);
      bisected = true;
    } else {
      bisected = false;
    }
    const double fs = count(s) - ne;
    d = c;
    c = b;
    fc = fb;
    if ((fa < 0.0) != (fs < 0.0)) { b = s; fb = fs; }
    else { a = s; fa = fs; }
    if (fabs(fa) < fabs(fb)) { double t = a; a = b; b = t; t = fa; fa = fb; fb = t; }
  }
  double mu = b;
  if (tid == 0) *mu_out = mu;
  if (occ_w)
    for (int i = tid; i < tot; i += blockDim.x) {
      int b = i / ns;
      occ_w[i] = W.wk[b] * 0.5 * (1.0 - tanh((lam[i] - mu) / (2.0 * kT)));
    }
}

// ------------------------------------------------------------ Rayleigh-Ritz workspace
struct RRWork {
  void *W1, *W2, *alpha, *M, *T1, *T2, *A1, *tmp, *Z, *Qf, *qp, *gw, *cw, *hw;
  int* info;
  size_t gw_bytes;
};

static size_t rr_layout(const sparc_ham* H, int32_t n_s, void* base, size_t bytes, RRWork* w) {
  const bool cp = dtype_complex(H->dtype);
  const size_t blk = (size_t)H->n_d * n_s * elem_bytes(H->dtype);
  const size_t sm = (size_t)n_s * n_s * (cp ? 16 : 8);
  const size_t gwb = std::max(gram_work_bytes(H->n_d, n_s, n_s, H->dtype),
                              gram_work_bytes(n_s, n_s, n_s, cp ? SPARC_C128 : SPARC_R64));
  size_t need = al(blk) * 2 + al(alpha_bytes(H, n_s)) + al(sm) * 8 + al(gwb) +
                al(chol_orth_work_bytes(n_s, cp)) + al(heev_work_bytes(n_s, cp)) + 256;
  if (w && base) {
    Carver c{(char*)base, bytes};
    w->W1 = c.take(blk);
    w->W2 = c.take(blk);
    w->alpha = c.take(alpha_bytes(H, n_s));
    w->M = c.take(sm);
    w->T1 = c.take(sm);
    w->T2 = c.take(sm);
    w->A1 = c.take(sm);
    w->tmp = c.take(sm);
    w->Z = c.take(sm);
    w->Qf = c.take(sm);
    w->qp = c.take(sm);
    w->gw = c.take(gwb);
    w->gw_bytes = gwb;
    w->cw = c.take(chol_orth_work_bytes(n_s, cp));
    w->hw = c.take(heev_work_bytes(n_s, cp));
    w->info = (int*)c.take(256);
    if (!c.ok) return 0;
  }
  return need;
}

struct LzWork {
  void *V, *w, *t, *alpha, *c, *nrm, *alph, *beta, *T, *S, *theta, *gw, *hw;
  size_t gw_bytes;
};

static size_t lz_layout(const sparc_ham* H, int32_t m, void* base, size_t bytes, LzWork* w) {
  const size_t eb = elem_bytes(H->dtype);
  const size_t vb = (size_t)H->n_d * eb;
  const size_t gwb = gram_work_bytes(H->n_d, m + 1, 1, H->dtype);
  size_t need = al(vb * (m + 1)) + 2 * al(vb) + al(alpha_bytes(H, 1)) + al((m + 1) * 16) + al(64) + 2 * al(m * 8) +
                2 * al((size_t)m * m * 8) + al(m * 8) + al(gwb) + al(heev_work_bytes(m, false)) + 256;
  if (w && base) {
    Carver c{(char*)base, bytes};
    w->V = c.take(vb * (m + 1));
    w->w = c.take(vb);
    w->t = c.take(vb);
    w->alpha = c.take(alpha_bytes(H, 1));
    w->c = c.take((m + 1) * 16);
    w->nrm = c.take(64);
    w->alph = c.take(m * 8);
    w->beta = c.take(m * 8);
    w->T = c.take((size_t)m * m * 8);
    w->S = c.take((size_t)m * m * 8);
    w->theta = c.take(m * 8);
    w->gw = c.take(gwb);
    w->gw_bytes = gwb;
    w->hw = c.take(heev_work_bytes(m, false));
    if (!c.ok) return 0;
  }
  return need;
}

template <typename E>
static int launch_scale(hipStream_t s, const void* x, void* y, int64_t n, const double* nrm2) {
  scale_by_rnorm_kernel<E><<<(unsigned)((n + 255) / 256), 256, 0, s>>>((const E*)x, (E*)y, n, nrm2);
  return check_launch("scale_by_rnorm_kernel");
}
template <typename E>
static int launch_sub(hipStream_t s, void* w, const void* t, int64_t n) {
  sub_kernel<E><<<(unsigned)((n + 255) / 256), 256, 0, s>>>((E*)w, (const E*)t, n);
  return check_launch("sub_kernel");
}
static int scale_rnorm(sparc_dtype dt, hipStream_t s, const void* x, void* y, int64_t n, const double* nrm2) {
  switch (dt) {
    case SPARC_R64: return launch_scale<double>(s, x, y, n, nrm2);
    case SPARC_R32: return launch_scale<float>(s, x, y, n, nrm2);
    case SPARC_C128: return launch_scale<cd>(s, x, y, n, nrm2);
    case SPARC_C64: return launch_scale<cf>(s, x, y, n, nrm2);
  }
  return SPARC_EINVAL;
}
static int sub_vec(sparc_dtype dt, hipStream_t s, void* w, const void* t, int64_t n) {
  switch (dt) {
    case SPARC_R64: return launch_sub<double>(s, w, t, n);
    case SPARC_R32: return launch_sub<float>(s, w, t, n);
    case SPARC_C128: return launch_sub<cd>(s, w, t, n);
    case SPARC_C64: return launch_sub<cf>(s, w, t, n);
  }
  return SPARC_EINVAL;
}

// Chebyshev filter of degree m (three-term recurrence, one stencil step per degree):
// each step projects its input onto the projectors, then the stencil step applies the
// local and (inside the step, or with the scatter kernel after it) non-local terms; in the
// update form the scatter of a step makes the projections for the next one.
int filter_impl(sparc_ham* H, void* X, int64_t ldx, int32_t n_s, int32_t degree, double lcut, double lmax,
                void* Wb, void* alpha) {
  const double c = 0.5 * (lmax + lcut), e = 0.5 * (lmax - lcut);
  const int64_t N = H->n_d;
  const bool upd = nl_update_single(H, n_s);
  SPARC_TRY(nl_project(H, X, ldx, n_s, alpha));
  SPARC_TRY(ham_step(H, X, ldx, nullptr, 0, Wb, N, n_s, 1.0 / e, -c / e, 0.0, alpha,
                     upd && degree > 1 ? STEP_NO_NONLOCAL : 0));
  if (upd && degree > 1) SPARC_TRY(nl_update(H, alpha, n_s, 1.0 / e, Wb, N));
  void* prev = X;
  int64_t ldp = ldx;
  void* cur = Wb;
  int64_t ldc = N;
  for (int j = 1; j < degree; ++j) {
    const bool more = upd && j + 1 < degree;
    if (!upd) SPARC_TRY(nl_project(H, cur, ldc, n_s, alpha));
    SPARC_TRY(ham_step(H, cur, ldc, prev, ldp, prev, ldp, n_s, 2.0 / e, -2.0 * c / e, -1.0, alpha,
                       more ? STEP_NO_NONLOCAL : 0));
    if (more) SPARC_TRY(nl_update(H, alpha, n_s, 2.0 / e, prev, ldp));
    std::swap(prev, cur);
    std::swap(ldp, ldc);
  }
  if (cur != X) {
    size_t eb = elem_bytes(H->dtype);
    SPARC_HIP(hipMemcpy2DAsync(X, ldx * eb, cur, ldc * eb, N * eb, n_s, hipMemcpyDeviceToDevice, H->ctx->stream));
  }
  return SPARC_OK;
}

// Out = A Q for the N_d-long rotations of Rayleigh-Ritz: split-BF16 (x3) products from
// pieces made in W2 (free at every rotation) when the mode asks for them and n is a
// multiple of 16, else the element type's MFMA
// dst(:, c) = src(:, c) for n columns of `bytes` bytes each: one 16-byte element per
// thread, all accesses non-temporal (the block is streamed once); falls back to a 2-D
// runtime copy when the columns or leading dimensions are not 16-byte multiples
typedef double v2d_t __attribute__((ext_vector_type(2)));
__global__ __launch_bounds__(256) void copy_cols_kernel(const v2d_t* __restrict__ src, int64_t lds,
                                                        v2d_t* __restrict__ dst, int64_t ldd, int64_t rows) {
  const int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x;
  const int64_t c = blockIdx.y;
  if (i < rows) __builtin_nontemporal_store(__builtin_nontemporal_load(&src[c * lds + i]), &dst[c * ldd + i]);
}

static int copy_cols(hipStream_t s, void* dst, int64_t ld_dst, const void* src, int64_t ld_src, int64_t bytes,
                     int32_t n) {
  const bool vec = bytes % 16 == 0 && ld_dst % 16 == 0 && ld_src % 16 == 0 && (uintptr_t)dst % 16 == 0 &&
                   (uintptr_t)src % 16 == 0 && n <= 65535 && (bytes / 16 + 255) / 256 <= (int64_t)UINT32_MAX;
  if (!vec) {
    SPARC_HIP(hipMemcpy2DAsync(dst, ld_dst, src, ld_src, bytes, n, hipMemcpyDeviceToDevice, s));
    return SPARC_OK;
  }
  const int64_t rows = bytes / 16;
  copy_cols_kernel<<<dim3((unsigned)((rows + 255) / 256), (unsigned)n), 256, 0, s>>>(
      (const v2d_t*)src, ld_src / 16, (v2d_t*)dst, ld_dst / 16, rows);
  return check_launch("copy_cols_kernel");
}

static int rr_rotate(sparc_ham* H, sparc_gemm_mode mode, int32_t n, const void* A, int64_t lda, const void* Q,
                     void* Out, int64_t ldo, int q_upper, RRWork& w) {
  hipStream_t s = H->ctx->stream;
  if (mode == SPARC_GEMM_BF16X3 && dtype_single(H->dtype) && n % 16 == 0)
    return rotate_split_x3(s, H->dtype, H->n_d, n, n, A, lda, Q, n, Out, ldo, q_upper, w.W2, w.qp);
  return rotate(s, H->dtype, H->n_d, n, n, A, lda, Q, n, Out, ldo, q_upper, H->ctx);
}

// Largest estimated condition number of the column-scaled Gram matrix for which one
// Cholesky-QR pass is taken (orthonormality defect about kappa * eps); above it, two.
constexpr double kSinglePassKappa = 50.0;

// what the first Gram matrix says: Cholesky status and the condition estimate
struct RRFirst {
  int32_t info;
  int32_t pad;
  double kappa;
  bool single_pass() const { return info == 0 && kappa <= kSinglePassKappa; }
};

// T1 from the Gram matrix in w.M, and the condition estimate of the column-scaled matrix, into
// w.info (an RRFirst)
static int rr_first(hipStream_t s, bool cp, int32_t n, RRWork& w) {
  SPARC_TRY(chol_orth(s, cp, n, w.M, w.T1, w.info, w.cw, 0.0));
  return chol_cond_est(s, cp, n, w.M, w.T1, w.info, w.cw, (double*)((char*)w.info + 8));
}

// The dense part of a single-pass problem: Qf = T1 Z and the Ritz values from the projected
// matrix in w.A1
static int rr_dense(hipStream_t s, bool cp, int32_t n, double* ritz, RRWork& w, int ncu) {
  const sparc_dtype sdt = cp ? SPARC_C128 : SPARC_R64;
  SPARC_TRY(rotate(s, sdt, n, n, n, w.A1, n, w.T1, n, w.tmp, n, 1));
  SPARC_TRY(gram(s, sdt, n, n, n, w.T1, n, w.tmp, n, w.A1, n, w.gw, w.gw_bytes, SPARC_GEMM_NATIVE, ncu, true));
  herm_sym_kernel<<<(unsigned)(((int64_t)n * n + 255) / 256), 256, 0, s>>>(n, (double*)w.A1, cp ? 1 : 0);
  SPARC_TRY(check_launch("herm_sym_kernel"));
  SPARC_TRY(heev(s, cp, n, w.A1, ritz, w.Z, w.hw));
  return rotate(s, sdt, n, n, n, w.T1, n, w.Z, n, w.Qf, n, 0);
}

// Rayleigh-Ritz from the first Gram matrix on (w.M, w.T1 as rr_first left them)
static int rr_rest(sparc_ham* H, void* X, int64_t ldx, int32_t n, sparc_gemm_mode mode, double* ritz, RRWork& w,
                   const RRFirst& st, int32_t* info_out) {
  hipStream_t s = H->ctx->stream;
  const sparc_dtype dt = H->dtype;
  const bool cp = dtype_complex(dt);
  const sparc_dtype sdt = cp ? SPARC_C128 : SPARC_R64;
  const int64_t N = H->n_d;
  const int ncu = H->ctx->n_cu;
  int info = st.info;
  bool shifted = false;
  if (st.single_pass()) {
    // a nearly orthogonal block (the steady state of the iteration): one Cholesky-QR pass
    // leaves an orthonormality defect of about kappa * eps, so H X, the projected matrix
    // and the rotation to the Ritz vectors are taken on X itself, T = T1
    SPARC_TRY(nl_project(H, X, ldx, n, w.alpha));
    SPARC_TRY(ham_step(H, X, ldx, nullptr, 0, w.W2, N, n, 1.0, 0.0, 0.0, w.alpha));
    SPARC_TRY(gram(s, dt, N, n, n, X, ldx, w.W2, N, w.A1, n, w.gw, w.gw_bytes, mode, ncu, true, H->ctx));
    SPARC_TRY(rr_dense(s, cp, n, ritz, w, ncu));
    // U = X (T1 Z), formed out of place and copied back
    SPARC_TRY(rr_rotate(H, mode, n, X, ldx, w.Qf, w.W1, N, 0, w));
    SPARC_TRY(copy_cols(s, X, ldx * elem_bytes(dt), w.W1, N * elem_bytes(dt), N * elem_bytes(dt), n));
    if (info_out) *info_out = 0;
    return SPARC_OK;
  }
  if (info != 0) {
    const double shift = 11.0 * ((double)N * n + (double)n * (n + 1)) * 2.2e-16 * n;
    SPARC_TRY(chol_orth(s, cp, n, w.M, w.T1, w.info, w.cw, shift));
    SPARC_HIP(hipMemcpyAsync(&info, w.info, 4, hipMemcpyDeviceToHost, s));
    SPARC_HIP(hipStreamSynchronize(s));
    if (info != 0) {
      if (info_out) *info_out = info;
      return fail(SPARC_ENOTSPD, "rayleigh_ritz: Gram matrix not positive definite at column %d", info);
    }
    shifted = true;
  }
  SPARC_TRY(rr_rotate(H, mode, n, X, ldx, w.T1, w.W1, N, 1, w));
  if (shifted) {  // one more explicit pass after a shifted factorisation
    SPARC_TRY(gram(s, dt, N, n, n, w.W1, N, w.W1, N, w.M, n, w.gw, w.gw_bytes, mode, ncu, false, H->ctx));
    SPARC_TRY(chol_orth(s, cp, n, w.M, w.T1, w.info, w.cw, 0.0));
    SPARC_HIP(hipMemcpyAsync(&info, w.info, 4, hipMemcpyDeviceToHost, s));
    SPARC_HIP(hipStreamSynchronize(s));
    if (info != 0) {
      if (info_out) *info_out = info;
      return fail(SPARC_ENOTSPD, "rayleigh_ritz: Gram matrix not positive definite at column %d", info);
    }
    SPARC_TRY(rr_rotate(H, mode, n, w.W1, N, w.T1, X, ldx, 1, w));
    SPARC_HIP(hipMemcpy2DAsync(w.W1, N * elem_bytes(dt), X, ldx * elem_bytes(dt), N * elem_bytes(dt), n,
                               hipMemcpyDeviceToDevice, s));
  }
  // pass 2 (implicit): T2 from the Gram matrix of X1 = X T1
  SPARC_TRY(gram(s, dt, N, n, n, w.W1, N, w.W1, N, w.M, n, w.gw, w.gw_bytes, mode, ncu, false, H->ctx));
  SPARC_TRY(chol_orth(s, cp, n, w.M, w.T2, w.info, w.cw, 0.0));
  // H X1 and the projected matrix A1 = X1^H H X1 (Hermitian: its upper triangle, mirrored)
  SPARC_TRY(nl_project(H, w.W1, N, n, w.alpha));
  SPARC_TRY(ham_step(H, w.W1, N, nullptr, 0, w.W2, N, n, 1.0, 0.0, 0.0, w.alpha));
  SPARC_TRY(gram(s, dt, N, n, n, w.W1, N, w.W2, N, w.A1, n, w.gw, w.gw_bytes, mode, ncu, true, H->ctx));
  // H~ = T2^H A1 T2 (FP64, Hermitian by the same mirror), symmetrised
  SPARC_TRY(rotate(s, sdt, n, n, n, w.A1, n, w.T2, n, w.tmp, n, 1));
  SPARC_TRY(gram(s, sdt, n, n, n, w.T2, n, w.tmp, n, w.A1, n, w.gw, w.gw_bytes, SPARC_GEMM_NATIVE, ncu, true));
  herm_sym_kernel<<<(unsigned)(((int64_t)n * n + 255) / 256), 256, 0, s>>>(n, (double*)w.A1, cp ? 1 : 0);
  SPARC_TRY(check_launch("herm_sym_kernel"));
  SPARC_HIP(hipMemcpyAsync(&info, w.info, 4, hipMemcpyDeviceToHost, s));
  SPARC_HIP(hipStreamSynchronize(s));
  if (info != 0) {
    if (info_out) *info_out = info;
    return fail(SPARC_ENOTSPD, "rayleigh_ritz: second Gram matrix not positive definite at column %d", info);
  }
  SPARC_TRY(heev(s, cp, n, w.A1, ritz, w.Z, w.hw));
  // U = X1 (T2 Z)
  SPARC_TRY(rotate(s, sdt, n, n, n, w.T2, n, w.Z, n, w.Qf, n, 0));
  SPARC_TRY(rr_rotate(H, mode, n, w.W1, N, w.Qf, X, ldx, 0, w));
  if (info_out) *info_out = 0;
  return SPARC_OK;
}

int rr_impl(sparc_ham* H, void* X, int64_t ldx, int32_t n, sparc_gemm_mode mode, double* ritz, RRWork& w,
            int32_t* info_out) {
  hipStream_t s = H->ctx->stream;
  DeviceScope on(H->ctx->device);
  TimerScope timer_scope(H->ctx);
  // pass 1: T1 from the Gram matrix of X (shifted if it is numerically singular), and the
  // condition estimate of the column-scaled Gram matrix
  SPARC_TRY(gram(s, H->dtype, H->n_d, n, n, X, ldx, X, ldx, w.M, n, w.gw, w.gw_bytes, mode, H->ctx->n_cu, false, H->ctx));
  SPARC_TRY(rr_first(s, dtype_complex(H->dtype), n, w));
  RRFirst st{};
  SPARC_HIP(hipMemcpyAsync(&st, w.info, sizeof(st), hipMemcpyDeviceToHost, s));
  SPARC_HIP(hipStreamSynchronize(s));
  return rr_rest(H, X, ldx, n, mode, ritz, w, st, info_out);
}

// ------------------------------------------------------------ batched Rayleigh-Ritz
// The dense kernels of one problem (Cholesky, condition estimate, eigensolver) are chains of
// small launches, one to a few work-groups each, that leave the chip idle: 1.6 of the 2.9 ms
// of a complex 48^3 problem with 128 states.  The problems' chains run on kSideStreams streams
// next to each other and to the large products, which stay on the context's stream in their
// order; every side stream is joined before the call returns.  Eight such problems: 23 ms one
// by one, 11 ms here (the pass around them 52.5 and 40.2 ms); eight uneven real cells, whose
// 256-state chain is the longest, 12 and 8 ms.
// Their n x n matrices sit at the start of the workspace, where a single call holds its first
// temporary block; the products' output takes the rest (H X, then the rotated block).
constexpr int kSideStreams = 3;   // and the context's: one hardware queue each

static size_t rr_dense_layout(bool cp, int32_t n, char* base, RRWork* w) {
  const size_t sm = (size_t)n * n * (cp ? 16 : 8);
  const size_t gwb = sm * std::max(1, n / 256);   // an n-row product takes no more slabs
  const size_t need = 6 * al(sm) + al(gwb) + al(chol_orth_work_bytes(n, cp)) + al(heev_work_bytes(n, cp));
  if (w) {
    Carver c{base, need};
    w->M = c.take(sm);
    w->T1 = c.take(sm);
    w->A1 = c.take(sm);
    w->tmp = c.take(sm);
    w->Z = c.take(sm);
    w->Qf = c.take(sm);
    w->gw = c.take(gwb);
    w->gw_bytes = gwb;
    w->cw = c.take(chol_orth_work_bytes(n, cp));
    w->hw = c.take(heev_work_bytes(n, cp));
  }
  return need;
}

// side streams and events of the context, held for one call
struct SideStreams {
  sparc_ctx* ctx;
  std::unique_lock<std::mutex> lock;
  explicit SideStreams(sparc_ctx* c) : ctx(c), lock(c->side_lock, std::try_to_lock) {}
  // nothing of this call is left running on a side stream, whichever way it ends
  ~SideStreams() {
    if (lock.owns_lock())
      for (hipStream_t t : ctx->side) hipStreamSynchronize(t);
  }
  bool ready(size_t events) {
    if (!lock.owns_lock()) return false;
    while (ctx->side.size() < (size_t)kSideStreams) {
      hipStream_t t;
      if (hipStreamCreateWithFlags(&t, hipStreamNonBlocking) != hipSuccess) return false;
      ctx->side.push_back(t);
    }
    while (ctx->side_ev.size() < events) {
      hipEvent_t e;
      if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) return false;
      ctx->side_ev.push_back(e);
    }
    return true;
  }
  // the side stream of problem p, after what the context's stream holds now
  int fork(int p, hipStream_t* t) {
    *t = ctx->side[p % kSideStreams];
    SPARC_HIP(hipEventRecord(ctx->side_ev[p], ctx->stream));
    SPARC_HIP(hipStreamWaitEvent(*t, ctx->side_ev[p], 0));
    return SPARC_OK;
  }
  int mark(int p) {
    SPARC_HIP(hipEventRecord(ctx->side_ev[p], ctx->side[p % kSideStreams]));
    return SPARC_OK;
  }
  int join(int p) {
    SPARC_HIP(hipStreamWaitEvent(ctx->stream, ctx->side_ev[p], 0));
    return SPARC_OK;
  }
};

int rr_concurrent(sparc_ctx* ctx, int32_t n_prob, sparc_ham* const* H, void* const* X, const int64_t* ldx,
                  const int32_t* n_s, sparc_gemm_mode mode, double* const* ritz, void* work, size_t work_bytes,
                  std::vector<char>& done) {
  // calls that a single call would refuse, blocks that overlap and split products (their pieces
  // need the second block) are left to it, as is kernel timing, which follows one stream.  So is
  // the first call of a shape on a context that autotunes: its products are timed one after another,
  // not beside the dense chains of other problems
  if (n_prob < 2 || mode != SPARC_GEMM_NATIVE || ctx->timing || !work) return SPARC_OK;
  size_t blk = 0, alpha = 0, gwb = 0, dense = al((size_t)n_prob * sizeof(RRFirst));
  std::vector<std::pair<uintptr_t, uintptr_t>> span;
  for (int p = 0; p < n_prob; ++p) {
    if (!H[p] || H[p]->ctx != ctx || !X[p] || !ritz[p] || n_s[p] < 1 || n_s[p] > 2048 || n_s[p] > H[p]->n_d ||
        ldx[p] < H[p]->n_d || work_bytes < rr_layout(H[p], n_s[p], nullptr, 0, nullptr))
      return SPARC_OK;
    if (ctx->autotune && !rr_products_tuned(H[p]->dtype, H[p]->n_d, n_s[p])) return SPARC_OK;
    const size_t eb = elem_bytes(H[p]->dtype);
    blk = std::max(blk, al((size_t)H[p]->n_d * n_s[p] * eb));
    alpha = std::max(alpha, al(alpha_bytes(H[p], n_s[p])));
    gwb = std::max(gwb, al(gram_work_bytes(H[p]->n_d, n_s[p], n_s[p], H[p]->dtype)));
    dense += rr_dense_layout(dtype_complex(H[p]->dtype), n_s[p], nullptr, nullptr);
    const uintptr_t x = (uintptr_t)X[p], r = (uintptr_t)ritz[p];
    span.push_back({x, x + ((size_t)(n_s[p] - 1) * ldx[p] + H[p]->n_d) * eb});
    span.push_back({r, r + (size_t)n_s[p] * 8});
  }
  std::sort(span.begin(), span.end());
  for (size_t i = 1; i < span.size(); ++i)
    if (span[i].first < span[i - 1].second) return SPARC_OK;
  // Two to four problems of a few states, a complex state counted as three: the chains are short, and the
  // events and stream waits cost more (24^3, 4 + 4 states: one by one 299 us, side by side 342; 9 + 9 363
  // and 394, 12 + 12 389 and 400, 8 + 20 390 and 392, 16 + 16 435 and 399; complex 2 + 2 385 and 421, 4 + 4
  // 422 and 430, 8 + 8 498 and 449; four problems of 2 states 570 and 622, of 4 613 and 630, of 8 706
  // and 640, four complex ones of 2 756 and 692)
  int64_t states = 0;
  for (int p = 0; p < n_prob; ++p) states += n_s[p] * (dtype_complex(H[p]->dtype) ? 3 : 1);
  if (n_prob <= 4 && states <= (n_prob == 2 ? 24 : 16)) return SPARC_OK;
  if (dense + blk + alpha + gwb > work_bytes) return SPARC_OK;
  DeviceScope on(ctx->device);
  SideStreams side(ctx);
  if (!side.ready(n_prob)) return SPARC_OK;

  hipStream_t s = ctx->stream;
  char* at = (char*)work;
  RRFirst* first_dev = (RRFirst*)at;
  at += al((size_t)n_prob * sizeof(RRFirst));
  std::vector<RRWork> w(n_prob);
  for (int p = 0; p < n_prob; ++p) {
    const bool cp = dtype_complex(H[p]->dtype);
    at += rr_dense_layout(cp, n_s[p], at, &w[p]);
    w[p].info = &first_dev[p].info;
  }
  char* W2 = at;
  char* al_dev = W2 + blk;
  char* gw = al_dev + alpha;
  auto gram_first = [&](int p) {
    return gram(s, H[p]->dtype, H[p]->n_d, n_s[p], n_s[p], X[p], ldx[p], X[p], ldx[p], w[p].M, n_s[p], gw, gwb, mode,
                ctx->n_cu, false, ctx);
  };
  std::vector<RRFirst> first(n_prob);
  // The first problem decides: where it needs two passes, which hold both temporary blocks,
  // the others most often do too and all go one by one
  {
    const bool cp = dtype_complex(H[0]->dtype);
    SPARC_TRY(gram_first(0));
    SPARC_TRY(rr_first(s, cp, n_s[0], w[0]));
    SPARC_HIP(hipMemcpyAsync(&first[0], first_dev, sizeof(RRFirst), hipMemcpyDeviceToHost, s));
    SPARC_HIP(hipStreamSynchronize(s));
    if (!first[0].single_pass()) {
      RRWork one;
      if (!rr_layout(H[0], n_s[0], work, work_bytes, &one)) return SPARC_OK;
      const size_t sm = (size_t)n_s[0] * n_s[0] * (cp ? 16 : 8);
      if ((char*)one.M < (char*)w[0].T1 + sm) return SPARC_OK;
      SPARC_HIP(hipMemcpyAsync(one.M, w[0].M, sm, hipMemcpyDeviceToDevice, s));
      SPARC_HIP(hipMemcpyAsync(one.T1, w[0].T1, sm, hipMemcpyDeviceToDevice, s));
      done[0] = 1;
      int32_t info = 0;
      return rr_rest(H[0], X[0], ldx[0], n_s[0], mode, ritz[0], one, first[0], &info);
    }
  }
  for (int p = 1; p < n_prob; ++p) {
    hipStream_t t;
    SPARC_TRY(gram_first(p));
    SPARC_TRY(side.fork(p, &t));
    SPARC_TRY(rr_first(t, dtype_complex(H[p]->dtype), n_s[p], w[p]));
    SPARC_TRY(side.mark(p));
  }
  for (int p = 1; p < n_prob; ++p) SPARC_TRY(side.join(p));
  SPARC_HIP(hipMemcpyAsync(first.data(), first_dev, n_prob * sizeof(RRFirst), hipMemcpyDeviceToHost, s));
  SPARC_HIP(hipStreamSynchronize(s));
  // the longest chains first
  std::vector<int> order;
  for (int p = 0; p < n_prob; ++p)
    if (first[p].single_pass()) order.push_back(p);
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return n_s[a] > n_s[b]; });
  for (size_t i = 0; i < order.size(); ++i) {
    const int p = order[i], n = n_s[p];
    const int64_t N = H[p]->n_d;
    hipStream_t t;
    SPARC_TRY(nl_project(H[p], X[p], ldx[p], n, al_dev));
    SPARC_TRY(ham_step(H[p], X[p], ldx[p], nullptr, 0, W2, N, n, 1.0, 0.0, 0.0, al_dev));
    SPARC_TRY(gram(s, H[p]->dtype, N, n, n, X[p], ldx[p], W2, N, w[p].A1, n, gw, gwb, mode, ctx->n_cu, true, ctx));
    SPARC_TRY(side.fork((int)i, &t));
    SPARC_TRY(rr_dense(t, dtype_complex(H[p]->dtype), n, ritz[p], w[p], ctx->n_cu));
    SPARC_TRY(side.mark((int)i));
  }
  for (size_t i = 0; i < order.size(); ++i) {
    const int p = order[i], n = n_s[p];
    const int64_t N = H[p]->n_d;
    const size_t eb = elem_bytes(H[p]->dtype);
    SPARC_TRY(side.join((int)i));
    SPARC_TRY(rotate(s, H[p]->dtype, N, n, n, X[p], ldx[p], w[p].Qf, n, W2, N, 0, ctx));
    SPARC_TRY(copy_cols(s, X[p], ldx[p] * eb, W2, N * eb, N * eb, n));
    done[p] = 1;
  }
  return SPARC_OK;
}

}  // namespace sparc

using namespace sparc;

extern "C" {

size_t sparc_workspace_bytes(const sparc_ham* H, int32_t n_s, int32_t op) {
  if (!H || n_s < 1) return 0;
  const size_t blk = (size_t)H->n_d * n_s * elem_bytes(H->dtype);
  switch (op) {
    case SPARC_OP_APPLY: return al(alpha_bytes(H, n_s));
    case SPARC_OP_FILTER: return al(blk) + al(alpha_bytes(H, n_s));
    case SPARC_OP_RR: return rr_layout(H, n_s, nullptr, 0, nullptr);
    case SPARC_OP_LANCZOS: return lz_layout(H, n_s, nullptr, 0, nullptr);
    case SPARC_OP_FORCES: return al(alpha_bytes(H, n_s)) + al(force_nl_part_bytes(H, n_s));
  }
  return 0;
}

int fd_hamiltonian_apply(sparc_ham* H, const void* X, int64_t ldx, void* Y, int64_t ldy, int32_t n_s, void* work,
                         size_t work_bytes) {
  SPARC_TRY(check_ham(H, "fd_hamiltonian_apply"));
  SPARC_TRY(check_block(H, X, ldx, n_s, "fd_hamiltonian_apply"));
  SPARC_TRY(check_block(H, Y, ldy, n_s, "fd_hamiltonian_apply"));
  if (X == Y) return fail(SPARC_EINVAL, "fd_hamiltonian_apply: X and Y must not alias");
  size_t need = sparc_workspace_bytes(H, n_s, SPARC_OP_APPLY);
  if (H->n_proj > 0 && (!work || work_bytes < need))
    return fail(SPARC_ENOMEM, "fd_hamiltonian_apply: workspace %zu < %zu bytes", work_bytes, need);
  SPARC_TRY(nl_project(H, X, ldx, n_s, work));
  return ham_step(H, X, ldx, nullptr, 0, Y, ldy, n_s, 1.0, 0.0, 0.0, work);
}

int chebyshev_filter(sparc_ham* H, void* X, int64_t ldx, int32_t n_s, int32_t degree, double lambda_cut,
                     double lambda_max, void* work, size_t work_bytes) {
  SPARC_TRY(check_ham(H, "chebyshev_filter"));
  SPARC_TRY(check_block(H, X, ldx, n_s, "chebyshev_filter"));
  if (degree < 1) return fail(SPARC_EINVAL, "chebyshev_filter: degree=%d < 1", degree);
  if (!(lambda_max > lambda_cut) || !std::isfinite(lambda_max) || !std::isfinite(lambda_cut))
    return fail(SPARC_EINVAL, "chebyshev_filter: need finite lambda_max > lambda_cut");
  size_t need = sparc_workspace_bytes(H, n_s, SPARC_OP_FILTER);
  if (!work || work_bytes < need) return fail(SPARC_ENOMEM, "chebyshev_filter: workspace %zu < %zu bytes", work_bytes, need);
  const size_t blk = (size_t)H->n_d * n_s * elem_bytes(H->dtype);
  return filter_impl(H, X, ldx, n_s, degree, lambda_cut, lambda_max, work, (char*)work + al(blk));
}

int rayleigh_ritz(sparc_ham* H, void* X, int64_t ldx, int32_t n_s, sparc_gemm_mode mode, double* ritz_dev,
                  void* work, size_t work_bytes, int32_t* info) {
  if (info) *info = 0;
  SPARC_TRY(check_ham(H, "rayleigh_ritz"));
  SPARC_TRY(check_block(H, X, ldx, n_s, "rayleigh_ritz"));
  if (!ritz_dev) return fail(SPARC_EINVAL, "rayleigh_ritz: ritz_dev is NULL");
  if (mode != SPARC_GEMM_NATIVE && mode != SPARC_GEMM_BF16X3 && mode != SPARC_GEMM_BF16X6)
    return fail(SPARC_EINVAL, "rayleigh_ritz: unknown GEMM mode %d", (int)mode);
  if (mode != SPARC_GEMM_NATIVE && !dtype_single(H->dtype))
    return fail(SPARC_EINVAL, "rayleigh_ritz: split-BF16 modes take FP32 / complex64 blocks");
  if (n_s > 2048) return fail(SPARC_ESHAPE, "rayleigh_ritz: n_s=%d above 2048", n_s);
  if (n_s > H->n_d) return fail(SPARC_ESHAPE, "rayleigh_ritz: n_s=%d exceeds N_d", n_s);
  RRWork w;
  size_t need = rr_layout(H, n_s, nullptr, 0, nullptr);
  if (!work || work_bytes < need) return fail(SPARC_ENOMEM, "rayleigh_ritz: workspace %zu < %zu bytes", work_bytes, need);
  if (!rr_layout(H, n_s, work, work_bytes, &w)) return fail(SPARC_ENOMEM, "rayleigh_ritz: workspace layout failed");
  return rr_impl(H, X, ldx, n_s, mode, ritz_dev, w, info);
}

int lanczos_bounds(sparc_ham* H, const void* v0, int32_t steps, void* work, size_t work_bytes, double* lmin,
                   double* lmax) {
  SPARC_TRY(check_ham(H, "lanczos_bounds"));
  if (!v0 || !lmin || !lmax) return fail(SPARC_EINVAL, "lanczos_bounds: null argument");
  if (steps < 2 || steps > 512 || steps > H->n_d) return fail(SPARC_EINVAL, "lanczos_bounds: steps=%d outside 2..512", steps);
  LzWork w;
  size_t need = lz_layout(H, steps, nullptr, 0, nullptr);
  if (!work || work_bytes < need) return fail(SPARC_ENOMEM, "lanczos_bounds: workspace %zu < %zu bytes", work_bytes, need);
  if (!lz_layout(H, steps, work, work_bytes, &w)) return fail(SPARC_ENOMEM, "lanczos_bounds: workspace layout failed");
  hipStream_t s = H->ctx->stream;
  const sparc_dtype dt = H->dtype;
  const bool cp = dtype_complex(dt);
  const int64_t N = H->n_d;
  const size_t eb = elem_bytes(dt);
  const int ncu = H->ctx->n_cu;
  char* V = (char*)w.V;
  const int m = steps;
  SPARC_TRY(gram(s, dt, N, 1, 1, v0, N, v0, N, w.nrm, 1, w.gw, w.gw_bytes, SPARC_GEMM_NATIVE, ncu));
  SPARC_TRY(scale_rnorm(dt, s, v0, V, N, (const double*)w.nrm));
  for (int j = 0; j < m; ++j) {
    void* vj = V + (size_t)j * N * eb;
    SPARC_TRY(nl_project(H, vj, N, 1, w.alpha));
    SPARC_TRY(ham_step(H, vj, N, nullptr, 0, w.w, N, 1, 1.0, 0.0, 0.0, w.alpha));
    for (int pass = 0; pass < 2; ++pass) {
      SPARC_TRY(gram(s, dt, N, j + 1, 1, V, N, w.w, N, w.c, j + 1, w.gw, w.gw_bytes, SPARC_GEMM_NATIVE, ncu));
      if (pass == 0) {
        lanczos_record_kernel<<<1, 1, 0, s>>>((const double*)w.c, j, cp ? 1 : 0, (double*)w.alph);
        SPARC_TRY(check_launch("lanczos_record_kernel"));
      }
      SPARC_TRY(rotate(s, dt, N, j + 1, 1, V, N, w.c, j + 1, w.t, N, 0));
      SPARC_TRY(sub_vec(dt, s, w.w, w.t, N));
    }
    SPARC_TRY(gram(s, dt, N, 1, 1, w.w, N, w.w, N, w.nrm, 1, w.gw, w.gw_bytes, SPARC_GEMM_NATIVE, ncu));
    lanczos_beta_kernel<<<1, 1, 0, s>>>((const double*)w.nrm, j, (double*)w.beta);
    SPARC_TRY(check_launch("lanczos_beta_kernel"));
    if (j + 1 < m) SPARC_TRY(scale_rnorm(dt, s, w.w, V + (size_t)(j + 1) * N * eb, N, (const double*)w.nrm));
  }
  tridiag_kernel<<<(m * m + 255) / 256, 256, 0, s>>>(m, (const double*)w.alph, (const double*)w.beta, (double*)w.T);
  SPARC_TRY(check_launch("tridiag_kernel"));
  SPARC_TRY(heev(s, false, m, w.T, (double*)w.theta, w.S, w.hw));
  std::vector<double> theta(m), S(m * m), beta(m);
  SPARC_HIP(hipMemcpyAsync(theta.data(), w.theta, m * 8, hipMemcpyDeviceToHost, s));
  SPARC_HIP(hipMemcpyAsync(S.data(), w.S, m * m * 8, hipMemcpyDeviceToHost, s));
  SPARC_HIP(hipMemcpyAsync(beta.data(), w.beta, m * 8, hipMemcpyDeviceToHost, s));
  SPARC_HIP(hipStreamSynchronize(s));
  double up = theta[m - 1] + std::fabs(beta[m - 1] * S[(m - 1) + (size_t)(m - 1) * m]);
  up += 0.01 * std::fabs(up);
  *lmin = theta[0];
  *lmax = up;
  if (!std::isfinite(*lmin) || !std::isfinite(*lmax)) return fail(SPARC_ENAN, "lanczos_bounds: non-finite bounds");
  return SPARC_OK;
}

int density_from_orbitals(sparc_ctx* ctx, int32_t n_k, const void* const* X, const int64_t* ldx, int32_t n_s,
                          sparc_dtype dtype, const double* occ_w, int64_t n_d, double dV, double* rho_dev) {
  if (!ctx || !X || !ldx || !occ_w || !rho_dev) return fail(SPARC_EINVAL, "density_from_orbitals: null argument");
  if (n_k < 1 || n_k > MAXK) return fail(SPARC_EINVAL, "density_from_orbitals: n_k=%d outside 1..%d", n_k, MAXK);
  if (n_s < 1 || n_d < 1) return fail(SPARC_ESHAPE, "density_from_orbitals: empty block");
  if (!(dV > 0)) return fail(SPARC_EINVAL, "density_from_orbitals: dV must be > 0");
  for (int b = 0; b < n_k; ++b) {
    if (!X[b]) return fail(SPARC_EINVAL, "density_from_orbitals: X[%d] is NULL", b);
    if (ldx[b] < n_d) return fail(SPARC_ESHAPE, "density_from_orbitals: ldx[%d] < n_d", b);
  }
  hipStream_t s = ctx->stream;
  unsigned nb = (unsigned)((n_d + 255) / 256);
  const double sc = 2.0 / dV;
#define DENS(E)                                                                                     \
  {                                                                                                 \
    DensArgs<E> A;                                                                                  \
    for (int b = 0; b < n_k; ++b) { A.x[b] = (const E*)X[b]; A.ld[b] = ldx[b]; }                     \
    density_kernel<E><<<nb, 256, 0, s>>>(A, n_k, n_s, n_d, occ_w, sc, rho_dev);                      \
    return check_launch("density_kernel");                                                          \
  }
  switch (dtype) {
    case SPARC_R64: DENS(double)
    case SPARC_R32: DENS(float)
    case SPARC_C128: DENS(cd)
    case SPARC_C64: DENS(cf)
  }
#undef DENS
  return fail(SPARC_EINVAL, "density_from_orbitals: bad dtype");
}

int sparc_fermi(sparc_ctx* ctx, int32_t n_k, int32_t n_s, const double* lambda_dev, const double* wk, double n_elec,
                double kT, double* occ_w_dev, double* mu) {
  if (!ctx || !lambda_dev || !wk || !mu) return fail(SPARC_EINVAL, "sparc_fermi: null argument");
  if (n_k < 1 || n_k > MAXK || n_s < 1) return fail(SPARC_EINVAL, "sparc_fermi: bad sizes");
  if (!(kT > 0) || !(n_elec > 0)) return fail(SPARC_EINVAL, "sparc_fermi: kT and n_elec must be > 0");
  double wsum = 0;
  for (int b = 0; b < n_k; ++b) wsum += wk[b];
  if (n_elec > 2.0 * n_s * wsum * (1.0 - 1e-12))
    return fail(SPARC_EINVAL, "sparc_fermi: %g electrons do not fit in %d states", n_elec, n_s);
  FermiArgs W;
  for (int b = 0; b < n_k; ++b) W.wk[b] = wk[b];
  double* dmu = ctx->scalars;
  fermi_kernel<<<1, 256, 0, ctx->stream>>>(n_k, n_s, lambda_dev, W, n_elec, kT, occ_w_dev, dmu);
  int rc = check_launch("fermi_kernel");
  double h = 0;
  if (rc == SPARC_OK) {
    hipError_t e = hipMemcpyAsync(&h, dmu, 8, hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) rc = fail(SPARC_EDEVICE, "sparc_fermi: %s", hipGetErrorString(e));
  }
  *mu = h;
  return rc;
}

}  // extern "C"
