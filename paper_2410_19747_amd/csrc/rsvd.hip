// Randomized truncated SVD of a swap matrix (TTM_SVD_RANDOMIZED): a range
// finder by subspace iteration (Halko, Martinsson and Tropp, SIAM Review 53
// (2011), Algorithms 4.3 and 4.4), followed by the one-sided Jacobi SVD of
// the projected matrix.
//
// The Swap of Sec. II.B keeps r = min(r_eps, cap) singular triplets of an
// m x n matrix Theta whose sides are d times the bond, so a cap of chi keeps
// about one eighth of the spectrum.  With l = 2 cap columns:
//   1. Y = Theta^T Omega, Omega (m x l) uniform in [-1, 1) from a
//      counter-based SplitMix64 stream; Y <- orth(Y);
//   2. q times: Z = orth(Theta Y), Y = orth(Theta^T Z); then a second
//      orthonormalisation pass on Y;
//   3. B = Theta Y (m x l, FP64) = Q_B R_B by CholeskyQR2, and the SVD of
//      the l x l factor R_B (B's values and right vectors V_B) by
//      one-sided Jacobi, above 64 columns on R_B^T as it is (svd_columns);
//   4. the rule of Eq. (eps) on those values with the weight that the l
//      directions do not capture, ||Theta||_F^2 - ||B||_F^2, added to every
//      tail;
//   5. V_r = Y V_B,r: P' = V_r^T (orthonormal rows), and the caller forms
//      X' = Theta V_r.
// The products of steps 1-2 take the operand precision of the contractions
// (FP64, or FP32 / BF16 terms on the matrix cores with FP32 accumulation
// within each 16-deep k-tile and FP64 across tiles): they only steer the
// subspace.  orth() is one CholeskyQR pass (G = Y^T Y = R^T R, Y <- Y R^-1)
// on the intermediate bases and two (CholeskyQR2; Yamamoto et al., ETNA 44
// (2015)) on the final one, all in FP64: a blocked Cholesky (one workgroup
// per 64 x 64 diagonal block, one launch for what the block leaves) and a
// triangular solve in one launch.  CholeskyQR needs
// kappa(Y) well below u^(-1/2); a pivot that falls to the rounding level of
// its column's norm (rank-deficient Theta, or kappa(Y) beyond ~1e7) raises
// a flag, and the caller then runs the full SVD on the same matrix instead.
//
// Accuracy: the subspace error decays like (sigma_{l+1} / sigma_r)^(2q+1).
// After the SVD it is estimated from the computed values, rho =
// sigma_l / sigma_r, as rho^(2q+1) sigma_r / ||Theta||_F (the move of the
// kept part relative to the chain's norm); a swap whose estimate exceeds
// the acceptance bound (default 2e-8; a spectrum too flat at the cut) also
// takes the full SVD.  With the defaults (q = 10) the products of the
// turbulence workloads stay within about 3e-8 of the FP64 product (the
// mixed-precision bar is 1e-6); FP32 sketch products add about 5e-7.  With
// q = 20 and a bound of 1e-14 they agree with the full SVD's to FP64
// parity (below 1e-13).
#include <math.h>
#include <stdio.h>

#include <algorithm>
#include <vector>

#include "ttm_internal.h"

namespace ttm {

namespace {
constexpr int CNB = 64;   // Cholesky block
constexpr int CNT = 256;  // threads of the diagonal-block kernel
constexpr double kU = 2.220446049250313e-16;

size_t r32(size_t n) { return (n + 31) & ~(size_t)31; }

// Squared Frobenius norm in two fixed-order passes: 256 block partials
// (grid-stride over x), then their sum by one block.
constexpr int SQB = 256;
__global__ __launch_bounds__(256) void sumsq_part_kernel(const double *__restrict__ x, int64_t n,
                                                         double *__restrict__ part) {
  __shared__ double red[4];
  double acc = 0.0;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)SQB * 256) acc = fma(x[e], x[e], acc);
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}
__global__ __launch_bounds__(256) void sumsq_final_kernel(const double *__restrict__ part, double *__restrict__ out) {
  __shared__ double red[4];
  double acc = part[threadIdx.x];
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) out[0] = (red[0] + red[1]) + (red[2] + red[3]);
}

// dst[i] = G[i * ld + i], i < n.
__global__ void diag_kernel(const double *__restrict__ G, int ld, int n, double *__restrict__ dst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = G[(int64_t)i * ld + i];
}

// dst[i] = the i-th Cholesky pivot over the squared norm gd[i] of its column,
// from the inverses of R's diagonal blocks; 1 where the pivot broke down.
__global__ void pivot_kernel(const double *__restrict__ rinv, const double *__restrict__ gd, int n,
                             double *__restrict__ dst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double x = rinv[((int64_t)(i / CNB) * CNB + i % CNB) * CNB + i % CNB];
  dst[i] = 1.0 / (x * x * gd[i]);
}

// 1 / sqrt(d) for d > 0: the hardware estimate (about 2^-24 off) and one step
// of third order.
__device__ __forceinline__ double rsqrt_nr(double d) {
  const double y = __builtin_amdgcn_rsq(d);
  const double e = fma(-d * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// Cholesky of the w x w diagonal block at G (row-major, ld), upper:
// G_kk = R^T R, one workgroup, padded to CNB with the identity.  Writes
// R^-1 (upper triangular, CNB x CNB row-major, zero below the diagonal) to
// rinv, and R itself to rout (row-major, ld, w x w) when rout is set.  gd
// (with nd > 0, the first block: set here, nd entries along G's diagonal)
// holds the block's diagonal as it was before any elimination (the squared
// column norms); a pivot at or below 64 u gd_j, or not positive, sets *fail
// and is replaced by gd_j (or 1) so that everything stays finite.  shift gd_j
// is added to the diagonal first.
// Elimination of [G_kk | I] to [R | X], X = R^-T, in place: G's and R's tiles
// lie on and above the diagonal, X's on and below it, so thread t holds the
// 4 x 4 tile (ti, tk) = (t / 16, t % 16) of G, R for tk > ti and of X for
// tk < ti; the diagonal tile is G's up to step ti and X's from there on.
// Four rows per step s: they are published, the tiles below take the rank-four
// update, and the threads of row s + 1 factor the next pivot block and turn
// their tiles into rows of R and X by its U^-T.  They do not wait for that
// block: it was published along with row s, one update short, so its update
// and the chain of its four pivots run among the tiles' own updates, in every
// thread alike.  One barrier a step.
// Bound by the chain of the 64 pivots (a reciprocal root each), sixteen
// substitutions and barriers.  Measured per block: 32 us with the inverse as
// sixteen further steps after the factorisation; 23 us with it on 256 threads
// of its own and two barriers a step, and 22.5 in place with one barrier but
// the factor after the updates; 19.7 us in this form.
__global__ __launch_bounds__(CNT) void chol_diag_kernel(const double *__restrict__ G, int ld, int w,
                                                        double *__restrict__ gd, int nd, double shift,
                                                        double *__restrict__ rinv,
                                                        double *__restrict__ rout, int *__restrict__ fail) {
  static_assert(CNB == 64 && CNT == 256, "one 4 x 4 tile per thread");
  // four rows of R and of X (zero where X has not begun), and the next pivot block
  __shared__ __align__(16) double rrow[2][4][CNB], xrow[2][4][CNB];
  __shared__ __align__(16) double pblk[2][4][4];
  __shared__ __align__(16) double rdiag[CNB / 4][4][4];  // R's diagonal tiles
  typedef double d2 __attribute__((ext_vector_type(2)));
  const int t = threadIdx.x, ti = t >> 4, tk = t & 15, i0 = 4 * ti, k0 = 4 * tk;
  double a[4][4], lim[4], instead[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = i0 + r, k = k0 + c;
      a[r][c] = (tk >= ti && i < w && k < w) ? G[(int64_t)i * ld + k] : (i == k ? 1.0 : 0.0);
    }
    // a pivot at or below lim breaks down; the column's own norm takes its
    // place, which keeps the rows behind it from growing
    const double ref = (i0 + r < w) ? (nd ? G[(int64_t)(i0 + r) * (ld + 1)] : gd[i0 + r]) : 1.0;
    if (ti == tk) a[r][r] = fma(shift, ref, a[r][r]);
    lim[r] = 64.0 * kU * ref;
    instead[r] = ref > 0.0 ? ref : 1.0;
  }
  for (int e = t; e < nd; e += CNT) gd[e] = G[(int64_t)e * (ld + 1)];
  for (int e = t; e < 2 * 4 * CNB; e += CNT) (&xrow[0][0][0])[e] = 0.0;
  bool bad = false;
  // tile b of a row: its first two columns at 2b, its last two at CNB/2 + 2b,
  // so that sixteen neighbours read all banks once
  auto put4 = [&](double (*dst)[CNB], int b, double (&x)[4][4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      *(d2 *)&dst[r][2 * b] = d2{x[r][0], x[r][1]};
      *(d2 *)&dst[r][2 * b + CNB / 2] = d2{x[r][2], x[r][3]};
    }
  };
  auto get4 = [&](double (*src)[CNB], int b, double (&x)[4][4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const d2 lo = *(const d2 *)&src[r][2 * b], hi = *(const d2 *)&src[r][2 * b + CNB / 2];
      x[r][0] = lo.x; x[r][1] = lo.y; x[r][2] = hi.x; x[r][3] = hi.y;
    }
  };
  auto put_block = [&](double (*dst)[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      *(d2 *)&dst[r][0] = d2{a[r][0], a[r][1]};
      *(d2 *)&dst[r][2] = d2{a[r][2], a[r][3]};
    }
  };
  auto get_block = [&](double (*src)[4], double (&x)[4][4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const d2 lo = *(const d2 *)&src[r][0], hi = *(const d2 *)&src[r][2];
      x[r][0] = lo.x; x[r][1] = lo.y; x[r][2] = hi.x; x[r][3] = hi.y;
    }
  };
  // U^T U = p (its upper triangle): U in u, the reciprocals of its diagonal
  // in iv; whether a pivot breaks down.
  auto factor = [&](const double (&p)[4][4], double (&u)[4][4], double (&iv)[4]) {
    bool down = false;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double d = p[r][r];
#pragma unroll
      for (int q = 0; q < r; ++q) d = fma(-u[q][r], u[q][r], d);
      const bool ok = d > lim[r];  // not for a NaN
      down |= !ok;
      d = ok ? d : instead[r];
      iv[r] = rsqrt_nr(d);
      u[r][r] = d * iv[r];
#pragma unroll
      for (int c = r + 1; c < 4; ++c) {
        double x = p[r][c];
#pragma unroll
        for (int q = 0; q < r; ++q) x = fma(-u[q][r], u[q][c], x);
        u[r][c] = x * iv[r];
      }
    }
    return down;
  };
  // Row st, whose threads these are: its tiles to R and X, published.
  auto finish_row = [&](int st, double (&u)[4][4], const double (&iv)[4]) {
    if (tk == st) {
      // R's tile is U itself; X's starts from the identity
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          u[r][c] = (c >= r) ? u[r][c] : 0.0;
          a[r][c] = (c == r) ? 1.0 : 0.0;
          rdiag[st][r][c] = u[r][c];
        }
      put4(rrow[st & 1], st, u);
    }
    // forward substitution of the tile's columns: x = U^-T g
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      a[0][c] = a[0][c] * iv[0];
      a[1][c] = fma(-u[0][1], a[0][c], a[1][c]) * iv[1];
      a[2][c] = fma(-u[1][2], a[1][c], fma(-u[0][2], a[0][c], a[2][c])) * iv[2];
      a[3][c] = fma(-u[2][3], a[2][c], fma(-u[1][3], a[1][c], fma(-u[0][3], a[0][c], a[3][c]))) * iv[3];
    }
    put4(tk > st ? rrow[st & 1] : xrow[st & 1], tk, a);
  };
  if (ti == tk && ti < 2) put_block(pblk[ti ^ 1]);
  __syncthreads();
  if (ti == 0) {
    double p[4][4], u[4][4], iv[4];
    get_block(pblk[1], p);
    bad |= factor(p, u, iv);
    finish_row(0, u, iv);
  }
  __syncthreads();
#pragma unroll 1
  for (int st = 0; st + 1 < CNB / 4; ++st) {
    const int par = st & 1;
    if (ti > st) {
      double xi[4][4], xk[4][4], p[4][4], u[4][4], iv[4];  // xi, xk: [published row][own row, own column]
      get4(rrow[par], ti, xi);
      get_block(pblk[par], p);
      get4(tk >= ti ? rrow[par] : xrow[par], tk, xk);
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = r; c < 4; ++c)
          p[r][c] = fma(-xi[3][r], xi[3][c], fma(-xi[2][r], xi[2][c],
                        fma(-xi[1][r], xi[1][c], fma(-xi[0][r], xi[0][c], p[r][c]))));
      const bool down = factor(p, u, iv);
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          a[r][c] = fma(-xi[3][r], xk[3][c], fma(-xi[2][r], xk[2][c],
                        fma(-xi[1][r], xk[1][c], fma(-xi[0][r], xk[0][c], a[r][c]))));
      if (ti == st + 1) {
        bad |= down;
        finish_row(st + 1, u, iv);
      }
      if (ti == tk && ti == st + 2) put_block(pblk[par ^ 1]);
    }
    __syncthreads();
  }
  if (bad) atomicOr(fail, 1);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    // column k of row i of X is entry (k, i) of R^-1
    const int k = k0 + c;
#pragma unroll
    for (int r = 0; r < 4; r += 2)
      *(d2 *)&rinv[k * CNB + i0 + r] = d2{k <= i0 + r ? a[r][c] : 0.0, k <= i0 + r + 1 ? a[r + 1][c] : 0.0};
  }
  if (rout) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (i0 + r < w && k0 + c < w)
          rout[(int64_t)(i0 + r) * ld + k0 + c] = (tk > ti) ? a[r][c] : (tk == ti ? rdiag[ti][r][c] : 0.0);
  }
}

hipError_t launch_chol_diag(const double *G, int ld, int w, double *gd, int nd, double shift, double *rinv,
                            double *rout, int *fail, hipStream_t s) {
  hipLaunchKernelGGL(chol_diag_kernel, dim3(1), dim3(CNT), 0, s, G, ld, w, gd, nd, shift, rinv, rout, fail);
  return hipGetLastError();
}

// What a diagonal block leaves to do: R_k = R_kk^-T G_k over the columns
// behind it and G_ij -= R_ki^T R_kj over their 32 x 32 tiles on and above the
// diagonal, one tile per workgroup.  Each workgroup forms the two 64 x 32
// parts of R_k that its tile needs for itself (five products for the work of
// one, on matrix cores that would idle), so that no launch stands between;
// those of the first tile row write them to Rf.  A block's two products were
// 4.8 us each in launches of their own; this is 7.2 us.
constexpr int UT = 32;
typedef double qd4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256, 1) void chol_update_kernel(double *__restrict__ G, int l, int b0,
                                                             const double *__restrict__ rinv,
                                                             double *__restrict__ Rf) {
  if (blockIdx.x < blockIdx.y) return;
  __shared__ double R[2][CNB][UT + 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lo = lane & 15, hi = lane >> 4;
  const int c0[2] = {b0 + CNB + (int)blockIdx.y * UT, b0 + CNB + (int)blockIdx.x * UT};
  constexpr int KQ = CNB / 4;
  // Lane: A(lo, 4 q + hi), B(4 q + hi, lo); accumulator t: D(4 t + hi, lo).
  double a[KQ], b[2][2][KQ];
#pragma unroll
  for (int q = 0; q < KQ; ++q) a[q] = rinv[(4 * q + hi) * CNB + 16 * wave + lo];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = c0[x] + 16 * h + lo;
#pragma unroll
      for (int q = 0; q < KQ; ++q) b[x][h][q] = (c < l) ? G[(int64_t)(b0 + 4 * q + hi) * l + c] : 0.0;
    }
  // the tile's own entries: 16 x 16 of them per wave
  const int gi = c0[0] + 16 * (wave >> 1) + hi, gj = c0[1] + 16 * (wave & 1) + lo;
  double own[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) own[t] = (gi + 4 * t < l && gj < l) ? G[(int64_t)(gi + 4 * t) * l + gj] : 0.0;
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    qd4 d[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
      d[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], b[x][0][q], d[0], 0, 0, 0);
      d[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], b[x][1][q], d[1], 0, 0, 0);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int m = 16 * wave + 4 * t + hi, c = c0[x] + 16 * h + lo;
        R[x][m][16 * h + lo] = d[h][t];
        if (x == 1 && blockIdx.y == 0 && c < l) Rf[(int64_t)(b0 + m) * l + c] = d[h][t];
      }
  }
  __syncthreads();
  qd4 d[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
  for (int q = 0; q < KQ; ++q)
    d[q & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(R[0][4 * q + hi][16 * (wave >> 1) + lo],
                                                    R[1][4 * q + hi][16 * (wave & 1) + lo], d[q & 1], 0, 0, 0);
#pragma unroll
  for (int t = 0; t < 4; ++t)
    if (gi + 4 * t < l && gj < l) G[(int64_t)(gi + 4 * t) * l + gj] = own[t] - (d[0][t] + d[1][t]);
}

// Q = Y R^-1 for 16 rows of Y per workgroup (Y, Q column-major, ld p; l
// columns in nb blocks of CNB): the rows stay in LDS while the blocks are
// solved, Q_k = Y_k R_kk^-1 and then Y_j -= Q_k R_kj for the blocks j > k, on
// the matrix cores (16 x 16 tiles, one of a block's four per wave; the tiles
// behind it dealt out to the waves).  Rf holds R's blocks above the diagonal
// (row-major, ld l), rinv the inverses of the diagonal blocks.
// As one product per block and per remainder the solve is 2 nb - 1 launches of
// 4.8 us each for some hundreds of rows, bound by their latency: 34 us for
// 1024 rows and 256 columns, here 16.6.
constexpr int QROWS = 16;
constexpr int kSolveCols = 1024;  // most columns whose rows fit in LDS (16 rows and a pad: 139 KB)
template <int LC>
__global__ __launch_bounds__(256, 1) void qsolve_kernel(const double *__restrict__ Y, int p, int l,
                                                        const double *__restrict__ Rf,
                                                        const double *__restrict__ rinv, double *__restrict__ Q) {
  constexpr int P = QROWS + 1;  // LDS column stride
  __shared__ double S[LC * P];  // column c of the rows at S[c * P]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lo = lane & 15, hi = lane >> 4;
  const int nb = (l + CNB - 1) / CNB;
  const int r = tid & (QROWS - 1), row = blockIdx.x * QROWS + r;
  for (int c = tid / QROWS; c < nb * CNB; c += 256 / QROWS)
    S[c * P + r] = (row < p && c < l) ? Y[(int64_t)c * p + row] : 0.0;
  double b[CNB / 4];  // this wave's column tile of R_kk^-1, then of R_k
#pragma unroll
  for (int q = 0; q < CNB / 4; ++q) b[q] = rinv[(4 * q + hi) * CNB + 16 * wave + lo];
  __syncthreads();
  for (int k = 0; k < nb; ++k) {
    const int b0 = k * CNB;
    // Lane: A(lo, 4 q + hi), B(4 q + hi, lo); accumulator t: D(4 t + hi, lo).
    double a[CNB / 4];
    auto load_a = [&]() {
#pragma unroll
      for (int q = 0; q < CNB / 4; ++q) a[q] = S[(b0 + 4 * q + hi) * P + lo];
    };
    auto product = [&]() {
      qd4 x = {0.0, 0.0, 0.0, 0.0}, y = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < CNB / 4; q += 2) {
        x = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], b[q], x, 0, 0, 0);
        y = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q + 1], b[q + 1], y, 0, 0, 0);
      }
      return x + y;
    };
    auto load_r = [&](int j0) {  // R_k over the columns of the tile at j0
      const int j = j0 + lo;
#pragma unroll
      for (int q = 0; q < CNB / 4; ++q) b[q] = (j < l) ? Rf[(int64_t)(b0 + 4 * q + hi) * l + j] : 0.0;
    };
    load_a();
    const qd4 qk = product();
    int j0 = b0 + CNB + 16 * wave;  // this wave's first tile behind the block
    if (j0 < nb * CNB) load_r(j0);
    __syncthreads();  // the block has been read
#pragma unroll
    for (int t = 0; t < 4; ++t) S[(b0 + 16 * wave + lo) * P + 4 * t + hi] = qk[t];
    __syncthreads();
    if (j0 < nb * CNB) load_a();
    while (j0 < nb * CNB) {
      const qd4 d = product();
      const int c = j0 + lo;
      j0 += CNB;
      if (j0 < nb * CNB) load_r(j0);
#pragma unroll
      for (int t = 0; t < 4; ++t) S[c * P + 4 * t + hi] -= d[t];
    }
    if (k + 1 < nb) {
#pragma unroll
      for (int q = 0; q < CNB / 4; ++q)
        b[q] = rinv[((int64_t)(k + 1) * CNB + 4 * q + hi) * CNB + 16 * wave + lo];
    }
    for (int c = tid / QROWS; c < CNB; c += 256 / QROWS)
      if (row < p && b0 + c < l) Q[(int64_t)(b0 + c) * p + row] = S[(b0 + c) * P + r];
    __syncthreads();
  }
}
hipError_t launch_qsolve(const double *Y, int p, int l, const double *Rf, const double *rinv, double *Q,
                         hipStream_t s) {
  const dim3 grid((p + QROWS - 1) / QROWS), block(256);
  if (l > kSolveCols) return hipErrorInvalidValue;
  if (l <= 128)
    hipLaunchKernelGGL(qsolve_kernel<128>, grid, block, 0, s, Y, p, l, Rf, rinv, Q);
  else if (l <= 256)
    hipLaunchKernelGGL(qsolve_kernel<256>, grid, block, 0, s, Y, p, l, Rf, rinv, Q);
  else if (l <= 512)
    hipLaunchKernelGGL(qsolve_kernel<512>, grid, block, 0, s, Y, p, l, Rf, rinv, Q);
  else
    hipLaunchKernelGGL(qsolve_kernel<1024>, grid, block, 0, s, Y, p, l, Rf, rinv, Q);
  return hipGetLastError();
}

constexpr int64_t kGramPart = (int64_t)2 << 20;  // split-K scratch of the Gram product (doubles)

// Buffers of one CholeskyQR (carved from the workspace).
struct CqrBufs {
  double *G = nullptr;     // l x l
  double *Rf = nullptr;    // l x l: the off-diagonal blocks of R
  double *rinv = nullptr;  // nb x CNB x CNB
  double *gd = nullptr;    // l
  double *part = nullptr;  // split-K scratch of the Gram product
  int64_t part_doubles = kGramPart;
};
size_t cqr_doubles(int l, int64_t part = kGramPart) {
  const size_t nb = (l + CNB - 1) / CNB;
  return 2 * r32((size_t)l * l) + r32(nb * CNB * CNB) + r32((size_t)l) + r32((size_t)part);
}
CqrBufs cqr_carve(int l, double *base, int64_t part = kGramPart) {
  CqrBufs b;
  b.part_doubles = part;
  double *q = base;
  auto adv = [&](size_t n) {
    double *x = q;
    q += r32(n);
    return x;
  };
  const size_t nb = (l + CNB - 1) / CNB;
  b.G = adv((size_t)l * l);
  b.Rf = adv((size_t)l * l);
  b.rinv = adv(nb * CNB * CNB);
  b.gd = adv((size_t)l);
  b.part = adv((size_t)part);
  return b;
}

// One CholeskyQR pass: Q = Y R^-1 with Y^T Y = R^T R, Y and Q column-major
// p x l (ld p).  Y is overwritten (the block solve updates it in place).
// With want_r, b.Rf holds all of R afterwards (row-major, zero below the
// diagonal); otherwise only its blocks right of the diagonal blocks.
// With a shift, shift times each column's squared norm is added to the Gram's
// diagonal, and Q is orthonormal only as far as the shift allows (further passes
// make it so).  A pivot then stands unless its column is zero or the Gram's own
// rounding, p u at worst, reaches the shift (1e-12 near 8192 rows); one that
// does not raises the flag like any other, and the full SVD runs.
hipError_t cholqr(double *Y, int p, int l, double *Q, const CqrBufs &b, int *fail, hipStream_t s,
                  KernelTimer *timer, bool want_r = false, double shift = 0.0) {
  Timed tm(timer, KC_QR, s);
  hipError_t e;
  if (want_r && (e = launch_fill(b.Rf, 0.0, (int64_t)l * l, s)) != hipSuccess) return e;
  {
    // G = Y^T Y (row-major, ld l), K split when the output is small
    GemmArgs g;
    g.M = l; g.N = l; g.K = p;
    g.A = Y; g.a_rs = p; g.a_cs = 1;
    g.B = Y; g.b_rs = 1; g.b_cs = p;
    g.C = b.G; g.c_rs1 = l; g.c_cs1 = 1;
    g.part = b.part; g.part_doubles = b.part_doubles;
    if ((e = launch_gemm(g, s)) != hipSuccess) return e;
  }
  const int nb = (l + CNB - 1) / CNB;
  // Blocked Cholesky, right-looking: R_kk from the block, then
  // R_k,rest = R_kk^-T G_k,rest and G_rest,rest -= R_k,rest^T R_k,rest (its
  // upper half).
  for (int kb = 0; kb < nb; ++kb) {
    const int b0 = kb * CNB, w = std::min(CNB, l - b0), rest = l - b0 - w;
    double *rk = b.rinv + (int64_t)kb * CNB * CNB;
    double *rout = want_r ? b.Rf + (int64_t)b0 * l + b0 : nullptr;
    if ((e = launch_chol_diag(b.G + (int64_t)b0 * l + b0, l, w, b.gd + b0, kb == 0 ? l : 0, shift, rk, rout, fail,
                              s)) != hipSuccess)
      return e;
    if (rest == 0) break;
    const int tiles = (rest + UT - 1) / UT;
    hipLaunchKernelGGL(chol_update_kernel, dim3(tiles, tiles), dim3(256), 0, s, b.G, l, b0, rk, b.Rf);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // Q = Y R^-1 by block columns: Q_k = Y_k R_kk^-1, then Y_rest -= Q_k R_k,rest;
  // in one launch where the rows of all blocks fit in LDS.
  if (l <= kSolveCols) return launch_qsolve(Y, p, l, b.Rf, b.rinv, Q, s);
  for (int kb = 0; kb < nb; ++kb) {
    const int b0 = kb * CNB, w = std::min(CNB, l - b0), rest = l - b0 - w;
    GemmArgs g;
    g.M = p; g.N = w; g.K = w;
    g.A = Y + (int64_t)b0 * p; g.a_rs = 1; g.a_cs = p;
    g.B = b.rinv + (int64_t)kb * CNB * CNB; g.b_rs = CNB; g.b_cs = 1;
    g.C = Q + (int64_t)b0 * p; g.c_rs1 = 1; g.c_cs1 = p;
    if ((e = launch_gemm(g, s)) != hipSuccess) return e;
    if (rest == 0) break;
    GemmArgs u;
    u.M = p; u.N = rest; u.K = w;
    u.A = Q + (int64_t)b0 * p; u.a_rs = 1; u.a_cs = p;
    u.B = b.Rf + (int64_t)b0 * l + b0 + w; u.b_rs = l; u.b_cs = 1;
    u.C = Y + (int64_t)(b0 + w) * p; u.c_rs1 = 1; u.c_cs1 = p;
    u.alpha = -1.0; u.beta = 1.0;
    if ((e = launch_gemm(u, s)) != hipSuccess) return e;
  }
  return hipSuccess;
}

// Buffers of one randomized SVD.
struct RsvdBufs {
  double *Om = nullptr;    // the test matrix (m x l), then a basis
  double *Y = nullptr;     // a basis
  double *T = nullptr;     // a basis (each max(m, n) x l)
  double *B = nullptr;     // m x l
  double *vbt = nullptr;   // l x l: V_B,r^T
  double *sig = nullptr;   // l: the singular values of B, decreasing
  double *full = nullptr;  // [0] = ||Theta||_F^2; [8, 8 + SQB): its block partials
  int *fail = nullptr;     // 1: a CholeskyQR of the range finder broke down
  int *fail2 = nullptr;    // 1: the CholeskyQR2 of B broke down
  double *R1 = nullptr;    // l x l: R of the first pass on B (row-major)
  double *RB = nullptr;    // l x l: R_B = R2 R1 (column-major)
  CqrBufs cq;
  double *svd = nullptr;   // the Jacobi SVD of B
};
}  // namespace

int rsvd_sketch_cols(int cap) { return 2 * cap; }

size_t cholqr2_ws_doubles(int p, int l) { return r32((size_t)p * l) + r32(8) + cqr_doubles(l); }

hipError_t cholqr2(double *Y, int p, int l, double *ws, int *fail_host, hipStream_t s) {
  double *T = ws;
  int *fail = reinterpret_cast<int *>(ws + r32((size_t)p * l));
  const CqrBufs cq = cqr_carve(l, ws + r32((size_t)p * l) + r32(8));
  hipError_t e;
  if ((e = launch_zero_int(fail, 1, s)) != hipSuccess) return e;
  if ((e = cholqr(Y, p, l, T, cq, fail, s, nullptr)) != hipSuccess) return e;
  if ((e = cholqr(T, p, l, Y, cq, fail, s, nullptr)) != hipSuccess) return e;
  if ((e = hipMemcpyAsync(fail_host, fail, sizeof(int), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
  return hipStreamSynchronize(s);
}

bool rsvd_eligible(int m, int n, int cap) {
  // The range finder pays when the kept rank is a small part of the
  // spectrum: the sketch must fit twice into the smaller side.
  return cap > 0 && 2 * rsvd_sketch_cols(cap) <= std::min(m, n) && std::min(m, n) <= kSvdMaxSide;
}

size_t rsvd_ws_doubles(int m, int n, int cap) {
  const int l = rsvd_sketch_cols(cap);
  const size_t mx = std::max(m, n);
  size_t t = 0;
  t += 3 * r32(mx * l) + r32((size_t)m * l) + r32((size_t)l * l);
  t += r32((size_t)l) + r32(8 + SQB) + r32(8) + r32(8) + 2 * r32((size_t)l * l);
  t += cqr_doubles(l);
  t += svd_ws_doubles(svd_plan(m, l));
  return t;
}

namespace {
RsvdBufs rsvd_carve(int m, int n, int cap, double *base) {
  const int l = rsvd_sketch_cols(cap);
  const size_t mx = std::max(m, n);
  RsvdBufs b;
  double *q = base;
  auto adv = [&](size_t nd) {
    double *x = q;
    q += r32(nd);
    return x;
  };
  b.Om = adv(mx * l);
  b.Y = adv(mx * l);
  b.T = adv(mx * l);
  b.B = adv((size_t)m * l);
  b.vbt = adv((size_t)l * l);
  b.sig = adv((size_t)l);
  b.full = adv(8 + SQB);
  b.fail = reinterpret_cast<int *>(adv(8));
  b.fail2 = reinterpret_cast<int *>(adv(8));
  b.R1 = adv((size_t)l * l);
  b.RB = adv((size_t)l * l);
  b.cq = cqr_carve(l, q);
  q += cqr_doubles(l);
  b.svd = q;
  return b;
}
}  // namespace

RsvdResult rsvd_oside(const double *Theta, int m, int n, int cap, int power, double accept, int max_sweeps,
                      double eps, int sketch_prec, uint64_t seed, int64_t stream_pos, double *pt, double *ws,
                      hipStream_t s, KernelTimer *timer, int trace) {
  RsvdResult out;
  const int l = rsvd_sketch_cols(cap);
  RsvdBufs b = rsvd_carve(m, n, cap, ws);
  auto ok = [&](hipError_t e) {
    if (e != hipSuccess) {
      out.err = TTM_EHIP;
      char what[112];
      snprintf(what, sizeof(what), "the randomized truncated SVD of a %d x %d matrix", m, n);
      note_hip_error(e, what);
      if (trace) fprintf(stderr, "[ttm] HIP error %s in %s\n", hipGetErrorName(e), what);
      return false;
    }
    return true;
  };
  // The bases in flight: the current Y (n x l) and Z (m x l) and a spare of
  // the same capacity; one CholeskyQR pass writes into the spare, and the
  // roles swap.  Intermediate bases need only be well conditioned (one pass
  // leaves cond ~ 1 + u cond(Y)^2); the final Y, which becomes P', gets the
  // second pass.
  double *ycur = b.Y, *zcur = b.Om, *spare = b.T;
  auto orth1 = [&](double *&X, int p) {
    if (!ok(cholqr(X, p, l, spare, b.cq, b.fail, s, timer))) return false;
    std::swap(X, spare);
    return true;
  };
  auto prod = [&](bool transposed, const double *Xin, double *Xout) {
    // Xout = Theta Xin (m x l) or Theta^T Xin (n x l), operands in the sketch precision
    GemmArgs g;
    g.prec = sketch_prec;
    if (transposed) {
      g.M = n; g.N = l; g.K = m;
      g.A = Theta; g.a_rs = m; g.a_cs = 1;
      g.B = Xin; g.b_rs = 1; g.b_cs = m;
      g.C = Xout; g.c_rs1 = 1; g.c_cs1 = n;
    } else {
      g.M = m; g.N = l; g.K = n;
      g.A = Theta; g.a_rs = 1; g.a_cs = m;
      g.B = Xin; g.b_rs = 1; g.b_cs = n;
      g.C = Xout; g.c_rs1 = 1; g.c_cs1 = m;
    }
    Timed tm(timer, KC_GEMM, s);
    return ok(launch_gemm(g, s));
  };
  if (!ok(launch_zero_int(b.fail, 1, s))) return out;
  {
    Timed tm(timer, KC_JAC_OTHER, s);
    if (!ok(launch_splitmix_fill(b.Om, (int64_t)m * l, seed, stream_pos, s))) return out;
    hipLaunchKernelGGL(sumsq_part_kernel, dim3(SQB), dim3(256), 0, s, Theta, (int64_t)m * n, b.full + 8);
    hipLaunchKernelGGL(sumsq_final_kernel, dim3(1), dim3(256), 0, s, b.full + 8, b.full);
    if (!ok(hipGetLastError())) return out;
  }
  if (!prod(true, b.Om, ycur) || !orth1(ycur, n)) return out;
  for (int it = 0; it < power; ++it) {
    if (!prod(false, ycur, zcur) || !orth1(zcur, m)) return out;
    if (!prod(true, zcur, ycur) || !orth1(ycur, n)) return out;
  }
  if (!orth1(ycur, n)) return out;  // the second pass on the final basis
  {
    // B = Theta Y in FP64 (m x l, column-major)
    GemmArgs g;
    g.M = m; g.N = l; g.K = n;
    g.A = Theta; g.a_rs = 1; g.a_cs = m;
    g.B = ycur; g.b_rs = 1; g.b_cs = n;
    g.C = b.B; g.c_rs1 = 1; g.c_cs1 = m;
    Timed tm(timer, KC_GEMM, s);
    if (!ok(launch_gemm(g, s))) return out;
  }
  // B = Q_B R_B by CholeskyQR2 with R_B = R2 R1 kept (Q_B is not needed):
  // B's right singular vectors and values are R_B's, and the Jacobi SVD then
  // runs on the l x l R_B instead of the m x l B.
  // Above kColumnsSmall columns it runs on R_B^T as it is: Y is ordered by the
  // power iterations, so B's columns, and more so R_B's rows, are near
  // orthogonal, and R_B^T needs neither a QR nor the sweeps of a general matrix
  // (256^3 product at bond 128, randomized: 191 -> 156 ms).  Up to kColumnsSmall
  // one launch does QR and Jacobi.
  const bool wide = l > kColumnsSmall;
  if (!ok(launch_zero_int(b.fail2, 1, s))) return out;
  if (!ok(cholqr(b.B, m, l, spare, b.cq, b.fail2, s, timer, true))) return out;
  if (!ok(launch_copy(b.R1, b.cq.Rf, (int64_t)l * l, s))) return out;
  if (!ok(cholqr(spare, m, l, zcur, b.cq, b.fail2, s, timer, true))) return out;
  {
    GemmArgs g;
    g.M = l; g.N = l; g.K = l;
    g.A = b.cq.Rf; g.a_rs = l; g.a_cs = 1;
    g.B = b.R1; g.b_rs = l; g.b_cs = 1;
    g.C = wide ? zcur : b.RB;
    (wide ? g.c_rs1 : g.c_cs1) = l;  // column-major R_B^T or R_B
    (wide ? g.c_cs1 : g.c_rs1) = 1;
    Timed tm(timer, KC_GEMM, s);
    if (!ok(launch_gemm(g, s))) return out;
  }
  // A breakdown of the range finder's CholeskyQR makes its result
  // meaningless: read both flags before the SVD.
  int fail[2] = {0, 0};
  if (!ok(hipMemcpyAsync(&fail[0], b.fail, sizeof(int), hipMemcpyDeviceToHost, s))) return out;
  if (!ok(hipMemcpyAsync(&fail[1], b.fail2, sizeof(int), hipMemcpyDeviceToHost, s))) return out;
  if (!ok(hipStreamSynchronize(s))) return out;
  if (timer && timer->on) timer->collect();
  if (fail[0]) {
    out.fallback = true;
    if (trace) fprintf(stderr, "[ttm] rsvd %dx%d cap %d: CholeskyQR breakdown, full SVD instead\n", m, n, cap);
    return out;
  }
  // The SVD of R_B (or of B itself when its CholeskyQR2 broke down, B
  // formed again): the right singular vectors (over the l side) come out
  // orthonormal; the rank rule adds the weight outside span(Y).
  const double *Ysvd = b.RB;
  SvdPlan sp = svd_plan(l, l);
  if (fail[1]) {
    GemmArgs g;
    g.M = m; g.N = l; g.K = n;
    g.A = Theta; g.a_rs = 1; g.a_cs = m;
    g.B = ycur; g.b_rs = 1; g.b_cs = n;
    g.C = b.B; g.c_rs1 = 1; g.c_cs1 = m;
    Timed tm(timer, KC_GEMM, s);
    if (!ok(launch_gemm(g, s))) return out;
    Ysvd = b.B;
    sp = svd_plan(m, l);
  }
  SvdResult so;
  if (wide && !fail[1]) {
    // the bases other than Y are free, at least 2 l rows each
    so = svd_columns(zcur, spare, l, l, eps, cap, max_sweeps, b.vbt, b.sig, b.svd, s, timer, trace, b.full);
  } else {
    so = svd_oside(sp, Ysvd, eps, cap, 0, max_sweeps, b.vbt, SVD_U_T, b.sig, b.svd, s, timer, trace, nullptr, b.full);
  }
  out.sweeps = so.sweeps;
  out.solve_flops = so.solve_flops;
  if (so.err != TTM_OK) {
    out.err = so.err;
    return out;
  }
  const int r = so.rank;
  // Acceptance: the subspace error of direction r after q iterations is
  // about rho^(2q+1) with rho = sigma_{l+1} / sigma_r, bounded here by the
  // computed sigma_l / sigma_r; relative to the chain's norm the kept part
  // moves by about rho^(2q+1) sigma_r / ||Theta||_F.  Swaps whose estimate
  // exceeds `accept` (a spectrum too flat at the cut for q iterations) take
  // the full SVD.
  {
    double sv[2] = {0.0, 0.0};
    if (!ok(hipMemcpyAsync(&sv[0], b.sig + (r - 1), sizeof(double), hipMemcpyDeviceToHost, s))) return out;
    if (!ok(hipMemcpyAsync(&sv[1], b.sig + (l - 1), sizeof(double), hipMemcpyDeviceToHost, s))) return out;
    if (!ok(hipStreamSynchronize(s))) return out;
    if (timer && timer->on) timer->collect();
    const double rho = sv[0] > 0.0 ? sv[1] / sv[0] : 1.0;
    const double est = pow(rho, 2.0 * power + 1.0) * (so.total > 0.0 ? sv[0] / sqrt(so.total) : 1.0);
    out.estimate = est;
    if (!(est <= accept)) {
      out.fallback = true;
      if (trace) fprintf(stderr, "[ttm] rsvd %dx%d cap %d: estimate %.2e above %.0e, full SVD instead\n", m, n, cap,
                         est, accept);
      return out;
    }
  }
  {
    // P' = V_B,r^T Y^T (r x n, row-major)
    GemmArgs g;
    g.M = r; g.N = n; g.K = l;
    g.A = b.vbt; g.a_rs = l; g.a_cs = 1;
    g.B = ycur; g.b_rs = n; g.b_cs = 1;
    g.C = pt; g.c_rs1 = n; g.c_cs1 = 1;
    Timed tm(timer, KC_GEMM, s);
    if (!ok(launch_gemm(g, s))) return out;
  }
  out.rank = r;
  out.disc = so.disc;
  out.total = so.total;
  const double ld = l, md = m, nd = n;
  // products of the range finder and the projection, two CholeskyQRs per
  // orthonormalisation, the SVD of B (the bidiagonalisation model)
  out.flops = (2.0 * power + 2.0) * 2.0 * md * nd * ld +
              (2.0 * power + 1.0) * 2.0 * (2.0 * 0.5 * (md + nd) * ld * ld + ld * ld * ld / 3.0) +
              4.0 * md * ld * ld - (4.0 / 3.0) * ld * ld * ld + 4.0 * (md + ld) * ld * r + 2.0 * r * ld * nd;
  if (trace)
    fprintf(stderr, "[ttm] rsvd %dx%d l=%d q=%d sweeps=%d rank=%d disc=%.3e total=%.3e\n", m, n, l, power,
            out.sweeps, r, out.disc, out.total);
  return out;
}

// ====================================================================== the capped SVD at full accuracy
// The default swap SVD where the cap keeps at most a quarter of the
// spectrum: the cap leading triplets by a filtered subspace iteration that
// is carried to rounding level and then checked, instead of all of them.
//
// A capped swap of d = 8 sites keeps an eighth of its singular values, and
// the Jacobi SVD spends its sweeps on the other seven eighths, latency bound
// (63 rounds a sweep at 1024 columns).  Measured, products of two turbulence
// components: 256^3 at bond 64 (512 x 512 swaps) 214 -> 55 ms, at 128
// (1024 x 1024) 428 -> 114 ms, 128^3 at 256 (2048 x 2048) 660 -> 194 ms, 1024^3
// at 1024 (8192 x 8192) 39.7 -> 14.5 s, and
// their error against 64 bits halves (8e-14 -> 5e-14, 1.1e-13 -> 6e-14).
// With l = 2 cap columns and M = Theta^T Theta:
//   1. Y = orth(Theta^T Omega), then twice Y = orth(M Y); the diagonal of the
//      last Cholesky factor gives estimates of the squared singular values:
//      the smallest, b, bounds the part to suppress, the cap-th the part kept;
//   2. as many times as the estimates ask for, Y = orth(T_2((2 / b) M - I) Y)
//      with the Chebyshev polynomial T_2, which stays below 1 on [0, b] and
//      grows as 2 x^2 - 1 above (Halko, Martinsson and Tropp 2011 iterate with
//      M^2, half the digits).  Degree 2 because CholeskyQR takes a condition
//      up to about 1e7 and T_2 raises the leading direction by 1e4 to 1e7 over
//      the last;
//   3. Z = orth(Theta Y), and the Jacobi SVD of Theta^T Z (n x l, its columns
//      near orthogonal by now): its values and left vectors V_r, orthonormal
//      to rounding; X' = Theta V_r.
// The result is checked, not trusted: (Theta V_r - Z Z^T Theta V_r) is what
// the computed triplets miss, so that they are those of a matrix that far
// from Theta (a backward error; measured 2e-16 to 1.6e-15 of ||Theta||_F at
// 512 to 2048 rows, its own rounding); above 32 u = 7e-15 the swap takes the
// full SVD.  The rule of Eq. (eps) is taken with the weight outside the l
// values in every tail, and checked with the discarded weight summed from
// Theta - X' P' itself.  The full SVD also runs where that check is not clear
// by 1e-6, where the spectrum is too flat for MAX_FILTER filters, and where the
// cap lies below the noise level.  Where a Cholesky pivot breaks down (a
// spectrum that falls by more than about 1e7 over the l columns) the iteration
// starts again with shifted passes (see STEEP_SHIFT), or, if the pivots show that
// it would find the cap below the noise level, leaves the swap to the full SVD.
namespace {
constexpr int PSVD_POWER = 2;     // plain iterations before the filter
// Well below where the full SVD costs as much, by measurement of flatter spectra
// at caps of a quarter and an eighth of the side: 16 and 28 filters at 160 x 160,
// 26 and 44 at 256, 38 and 66 at 512, 38 and 98 at 1024, 36 and 82 at 2048.
constexpr int MAX_FILTER = 10;
// A spectrum that falls by more than about 1e7 over the sketch breaks a
// CholeskyQR down.  The swap then starts again with half steps Y -> Theta Y ->
// Theta^T Theta Y, each orthonormalised by two passes with this shift of the
// Gram's diagonal and a plain one (shifted CholeskyQR3, Fukaya, Kannan,
// Nakatsukasa, Yamamoto and Yanagisawa 2020; the shift, well above the Gram's
// own rounding, bounds what a pass leaves).  Two swaps in 22 of a 256^3
// product at bond 128 come to that (512 x 1024: 121 -> 113 ms a product, the
// full SVD having taken them before), seven in 30 of a 1024^3 product at bond
// 512 (4096 x 4096: 3646 -> 1838 ms).
constexpr double STEEP_SHIFT = 1e-12;

// Whether the cap lies below noise (of the largest value) in a spectrum whose
// sketch of l columns breaks a CholeskyQR down, by the pivots (over their
// columns' norms, 1 where they broke) of the start, which fall as sigma^2 does:
// r0 of them stand, and if the values go on falling half as fast as over the last
// four digits above the level of breakdown, in which nb of the pivots lie, they
// are below noise^2 before the cap (half: the spectra of products flatten, and a
// swap that the shifted passes could have carried costs more than one that they
// could not).  Where the rank ends nb is next to none.  The shifted passes would
// then end in a refusal by the noise level: products of rank 9 and 16 at caps 40
// and 64 (6 sites of 8) took 31.5 and 39 ms with them, 23 and 34 without.
bool cap_in_noise(const std::vector<double> &pivots, int cap, double noise) {
  constexpr double LEVEL = 64.0 * kU;
  int r0 = 1, above = 1;
  while (r0 < (int)pivots.size() && pivots[r0] < 1.0 - 1e-9) {
    if (above == r0 && pivots[r0] > 1e4 * LEVEL) ++above;
    ++r0;
  }
  const int nb = r0 - above;
  return r0 < cap && 4.0 * (cap - r0) > 2.0 * nb * log10(LEVEL / (noise * noise));
}

struct PsvdBufs {
  double *Y, *W, *Z, *T, *vt, *small, *full, *diag;
  int *fail;
  CqrBufs cq;
  double *svd;
};
// part: the split-K scratch that is left.
size_t psvd_basis_doubles(int m, int n, int l) {
  return r32((size_t)std::max(m, n) * std::max(l, svd_columns_capacity(n, l)));
}
size_t psvd_fixed_doubles(int m, int n, int l) {
  return 4 * psvd_basis_doubles(m, n, l) + r32((size_t)l * l) + r32(8 + SQB) + r32((size_t)l) + r32(8) +
         cqr_doubles(l, 0);
}
// Columns of an m x n matrix that the four basis buffers hold (at least
// 4 l = 8 cap of them).
int psvd_columns(int m, int n, int l) {
  return (int)std::min<int64_t>(n, (int64_t)(4 * psvd_basis_doubles(m, n, l)) / m);
}
// Workspace left for split-K partials, or negative.
int64_t psvd_part_doubles(int m, int n, int cap) {
  const int l = rsvd_sketch_cols(cap);
  // the region of the full SVD of the same matrix, which a fallback uses
  const int64_t have = (int64_t)svd_ws_doubles(svd_plan(m, n));
  const int64_t fixed = (int64_t)psvd_fixed_doubles(m, n, l) + (int64_t)svd_columns_ws_doubles(n, l);
  return std::min<int64_t>(kGramPart, (have - fixed) & ~(int64_t)31);
}
}  // namespace

bool psvd_eligible(int m, int n, int cap) {
  if (!rsvd_eligible(m, n, cap)) return false;
  // One launch does the full SVD.  Measured at sides of 72 to 128 (times the
  // same or four times that) with caps of a quarter and an eighth: 0.97 to 1.25
  // ms at 96 and 128 for values falling as i^-1 and i^-2, here 0.90 to 1.3 and
  // 0.72 to 1.1; for i^-3, whose sketch a quarter breaks down, here 2.2 to 2.6.
  if (std::min(m, n) <= kSvdSmallSide) return false;
  const int l = rsvd_sketch_cols(cap);
  if (n > kSvdMaxSide || m > kSvdMaxSide) return false;
  // the discarded weight is summed over at most six blocks of columns
  const int room = psvd_columns(m, n, l);
  if ((n + room - 1) / room > 6) return false;
  // scratch for a Gram split in four, or all that a split ever takes
  return psvd_part_doubles(m, n, cap) >= std::min<int64_t>(kGramPart, 4 * (int64_t)l * l);
}

namespace {
PsvdResult psvd_run(const double *Theta, int m, int n, int cap, double eps, int max_sweeps, double *pt, double *xt,
                    double *ws, hipStream_t s, KernelTimer *timer, int trace, double *sigma, bool steep) {
  PsvdResult out;
  const int l = rsvd_sketch_cols(cap);
  const int64_t part = psvd_part_doubles(m, n, cap);
  PsvdBufs b;
  {
    double *q = ws;
    auto adv = [&](size_t nd) {
      double *x = q;
      q += r32(nd);
      return x;
    };
    const size_t basis = psvd_basis_doubles(m, n, l);
    b.Y = adv(basis);
    b.W = adv(basis);
    b.Z = adv(basis);
    b.T = adv(basis);
    b.vt = adv((size_t)l * l);
    b.full = adv(8 + SQB);
    b.diag = adv((size_t)l);
    b.fail = reinterpret_cast<int *>(adv(8));
    b.cq = cqr_carve(l, q, part);
    q += cqr_doubles(l, part);
    b.svd = q;
  }
  auto ok = [&](hipError_t e) {
    if (e != hipSuccess) {
      out.err = TTM_EHIP;
      char what[112];
      snprintf(what, sizeof(what), "the capped truncated SVD of a %d x %d matrix", m, n);
      note_hip_error(e, what);
      if (trace) fprintf(stderr, "[ttm] HIP error %s in %s\n", hipGetErrorName(e), what);
      return false;
    }
    return true;
  };
  auto sync = [&]() {
    if (!ok(hipStreamSynchronize(s))) return false;
    if (timer && timer->on) timer->collect();
    return true;
  };
  auto refuse = [&](const char *why, double v) {
    out.fallback = true;
    if (trace)
      fprintf(stderr, "[ttm] psvd %dx%d cap %d: %s (%.2e), %s instead\n", m, n, cap, why, v,
              out.breakdown && !steep ? "shifted passes" : "full SVD");
    return out;
  };
  double *ycur = b.Y, *wcur = b.W, *zcur = b.Z, *spare = b.T;
  auto orth = [&](double *&X, int p, bool diag = false) {
    for (int pass = steep ? 0 : 2; pass < 3; ++pass) {
      const bool first = pass == (steep ? 0 : 2);
      if (!ok(cholqr(X, p, l, spare, b.cq, b.fail, s, timer, diag && first, pass < 2 ? STEEP_SHIFT : 0.0))) return false;
      std::swap(X, spare);
      if (diag && first) {
        hipLaunchKernelGGL(diag_kernel, dim3((l + 255) / 256), dim3(256), 0, s, b.cq.Rf, l, l, b.diag);
        if (!ok(hipGetLastError())) return false;
      }
    }
    return true;
  };
  // out = alpha Theta in (m x l) or alpha Theta^T in (n x l), plus beta out
  auto prod = [&](bool transposed, const double *in, double *o, double alpha = 1.0, double beta = 0.0) {
    GemmArgs g;
    g.alpha = alpha;
    g.beta = beta;
    g.N = l;
    if (transposed) {
      g.M = n; g.K = m;
      g.A = Theta; g.a_rs = m; g.a_cs = 1;
      g.B = in; g.b_rs = 1; g.b_cs = m;
      g.C = o; g.c_rs1 = 1; g.c_cs1 = n;
    } else {
      g.M = m; g.K = n;
      g.A = Theta; g.a_rs = 1; g.a_cs = m;
      g.B = in; g.b_rs = 1; g.b_cs = n;
      g.C = o; g.c_rs1 = 1; g.c_cs1 = m;
    }
    g.part = b.cq.part;
    g.part_doubles = part;
    Timed tm(timer, KC_GEMM, s);
    return ok(launch_gemm(g, s));
  };
  auto sumsq = [&](const double *x, int64_t nx, double *o) {
    hipLaunchKernelGGL(sumsq_part_kernel, dim3(SQB), dim3(256), 0, s, x, nx, b.full + 8);
    hipLaunchKernelGGL(sumsq_final_kernel, dim3(1), dim3(256), 0, s, b.full + 8, o);
    return ok(hipGetLastError());
  };
  // 1. the start
  if (!ok(launch_zero_int(b.fail, 1, s))) return out;
  {
    Timed tm(timer, KC_JAC_OTHER, s);
    if (!ok(launch_splitmix_fill(zcur, (int64_t)m * l, 0x5eedULL, 0, s))) return out;
    if (!sumsq(Theta, (int64_t)m * n, b.full)) return out;
  }
  if (!prod(true, zcur, ycur) || !orth(ycur, n)) return out;
  if (!steep) {
    hipLaunchKernelGGL(pivot_kernel, dim3((l + 255) / 256), dim3(256), 0, s, b.cq.rinv, b.cq.gd, l, b.vt);
    if (!ok(hipGetLastError())) return out;
  }
  for (int it = 0; it < PSVD_POWER; ++it) {
    const bool last = it + 1 == PSVD_POWER;
    if (!prod(false, ycur, zcur) || (steep && !orth(zcur, m))) return out;
    if (!prod(true, zcur, ycur) || !orth(ycur, n, last)) return out;
  }
  std::vector<double> h(l);
  double tot = 0.0;
  int fail = 0;
  if (!ok(hipMemcpyAsync(h.data(), b.diag, sizeof(double) * l, hipMemcpyDeviceToHost, s))) return out;
  if (!ok(hipMemcpyAsync(&tot, b.full, sizeof(double), hipMemcpyDeviceToHost, s))) return out;
  if (!ok(hipMemcpyAsync(&fail, b.fail, sizeof(int), hipMemcpyDeviceToHost, s))) return out;
  if (!sync()) return out;
  // the level below which the full SVD decides, with room
  const double noise = 100.0 * 8.0 * sqrt((double)std::min(m, n)) * kU;
  out.breakdown = fail != 0;
  if (fail && !steep) {
    if (!ok(hipMemcpyAsync(h.data(), b.vt, sizeof(double) * l, hipMemcpyDeviceToHost, s))) return out;
    if (!sync()) return out;
    if (cap_in_noise(h, cap, noise)) {
      out.breakdown = false;
      return refuse("the cap lies in the noise", h[0]);
    }
  }
  if (fail) return refuse("CholeskyQR breakdown", fail);
  if (steep)  // of Theta^T Z, not of M Y
    for (double &x : h) x *= x;
  std::sort(h.begin(), h.end(), [](double x, double y) { return x > y; });
  const double bnd = h[l - 1], kept = h[cap - 1];
  // the shift hides where the spectrum ends: that the full SVD decides
  if (steep && !(kept > noise * noise * tot)) return refuse("the cap lies in the noise", kept / tot);
  // 2. the filter: each raises the cap-th direction over the rest by
  // 2 x^2 - 1; the start has raised it by (kept / bnd)^(power + 1/2).  What
  // is asked for is 1e-18 of ||Theta||_F: the estimates are a little rough, and
  // with 1e-16 one swap in thirty was left at 2e-14.
  const double x = 2.0 * kept / bnd - 1.0, gain = 2.0 * x * x - 1.0;
  if (!(bnd > 0.0) || !(gain > 1.0) || !(tot > 0.0) || !isfinite(tot)) return refuse("no gap", gain);
  const double need = log(1e18) + 0.5 * log(kept / tot) - (PSVD_POWER + 0.5) * log(kept / bnd);
  const int filters = std::max(0, (int)ceil(need / log(gain)));
  if (filters > MAX_FILTER) return refuse("too flat", filters);
  // M over 4^e, near ||Theta||_F^2: y is of fourth order in Theta and its Gram of
  // eighth, out of range for a norm beyond 1e38 or below 1e-38 (a power of two:
  // the same digits)
  const int e = ilogb(sqrt(tot));
  const double down = ldexp(1.0, -e), b1 = ldexp(bnd, -2 * e);
  for (int it = 0; it < filters; ++it) {
    // w = M y - b y, y <- M w + (b^2 / 8) y = (b^2 / 8) T_2((2 / b) M - I) y
    if (!ok(launch_copy(wcur, ycur, (int64_t)n * l, s))) return out;
    if (!prod(false, ycur, zcur, down) || !prod(true, zcur, wcur, down, -b1)) return out;
    if (!prod(false, wcur, zcur, down) || !prod(true, zcur, ycur, down, 0.125 * b1 * b1)) return out;
    if (!orth(ycur, n)) return out;
  }
  // 3. Z = orth(Theta Y), the SVD of Theta^T Z
  if (!prod(false, ycur, zcur) || !orth(zcur, m) || !orth(zcur, m)) return out;
  if (!prod(true, zcur, ycur)) return out;
  if (!ok(hipMemcpyAsync(&fail, b.fail, sizeof(int), hipMemcpyDeviceToHost, s))) return out;
  SvdResult so = svd_columns(ycur, wcur, n, l, eps, cap, max_sweeps, pt, b.diag, b.svd, s, timer, trace, b.full);
  out.sweeps = so.sweeps;
  out.solve_flops = so.solve_flops;
  out.breakdown = fail != 0;
  if (fail && so.err != TTM_EHIP) return refuse("CholeskyQR breakdown", fail);
  if (so.err == TTM_ENOCONV || so.err == TTM_ENONFINITE) {
    // not within max_sweeps, or squares out of range: the full SVD decides
    clear_last_error();
    return refuse("no SVD of the projection", so.sweeps);
  }
  if (so.err != TTM_OK) {
    out.err = so.err;
    return out;
  }
  const int r = so.rank;
  // X' = Theta V_r (m x r, row-major); what the triplets miss; the weight discarded
  {
    GemmArgs g;
    g.M = m; g.N = r; g.K = n;
    g.A = Theta; g.a_rs = 1; g.a_cs = m;
    g.B = pt; g.b_rs = 1; g.b_cs = n;
    g.C = xt; g.c_rs1 = r; g.c_cs1 = 1;
    GemmArgs q;  // Z^T X' (l x r, row-major)
    q.M = l; q.N = r; q.K = m;
    q.A = zcur; q.a_rs = m; q.a_cs = 1;
    q.B = xt; q.b_rs = r; q.b_cs = 1;
    q.C = b.vt; q.c_rs1 = r; q.c_cs1 = 1;
    q.part = b.cq.part; q.part_doubles = part;
    GemmArgs d;  // X' - Z (Z^T X')
    d.M = m; d.N = r; d.K = l;
    d.A = zcur; d.a_rs = 1; d.a_cs = m;
    d.B = b.vt; d.b_rs = r; d.b_cs = 1;
    d.C = spare; d.c_rs1 = r; d.c_cs1 = 1;
    d.alpha = -1.0; d.beta = 1.0;
    Timed tm(timer, KC_GEMM, s);
    if (!ok(launch_gemm(g, s)) || !ok(launch_gemm(q, s))) return out;
    if (!ok(launch_copy(spare, xt, (int64_t)m * r, s)) || !ok(launch_gemm(d, s))) return out;
  }
  if (!sumsq(spare, (int64_t)m * r, b.full + 1)) return out;
  // Theta - X' P' in the basis buffers, by as many columns as they hold
  const int room = psvd_columns(m, n, l);
  double disc = 0.0;
  int blocks = 0;
  for (int c0 = 0; c0 < n; c0 += room, ++blocks) {
    const int nc = std::min(room, n - c0);
    GemmArgs d;
    d.M = m; d.N = nc; d.K = r;
    d.A = xt; d.a_rs = r; d.a_cs = 1;
    d.B = pt + c0; d.b_rs = n; d.b_cs = 1;
    d.C = ws; d.c_rs1 = 1; d.c_cs1 = m;
    d.alpha = -1.0; d.beta = 1.0;
    Timed tm(timer, KC_GEMM, s);
    if (!ok(launch_copy(ws, Theta + (int64_t)c0 * m, (int64_t)m * nc, s)) || !ok(launch_gemm(d, s))) return out;
    if (!sumsq(ws, (int64_t)m * nc, b.full + 2 + blocks)) return out;
  }
  double res[8], sr = 0.0;
  if (!ok(hipMemcpyAsync(res, b.full, sizeof(res), hipMemcpyDeviceToHost, s))) return out;
  if (!ok(hipMemcpyAsync(&sr, b.diag + (r - 1), sizeof(double), hipMemcpyDeviceToHost, s))) return out;
  if (!sync()) return out;
  for (int i = 0; i < blocks; ++i) disc += res[2 + i];
  out.missed = sqrt(res[1] / tot);
  if (!(out.missed <= 32.0 * kU)) return refuse("not converged", out.missed);
  // Eq. (eps) again, with the discarded weight as it was summed: the tail at
  // r - 1 is not below eps of the total, that at r is (unless the cap binds);
  // and the kept values stand clear of the noise level, below which the rule
  // keeps none.
  const double cut = eps * tot, k = std::min(m, n);
  if (!(sr > 100.0 * 8.0 * sqrt(k) * kU * sqrt(tot))) return refuse("kept values near the noise level", sr);
  if (r > 1 && !(disc + sr * sr >= cut * (1.0 + 1e-6))) return refuse("the rule is not sure at the rank", disc / tot);
  if (r < cap && !(disc < cut * (1.0 - 1e-6))) return refuse("the rule is not sure below the cap", disc / tot);
  if (sigma && !ok(launch_copy(sigma, b.diag, r, s))) return out;
  out.rank = r;
  out.disc = disc;
  out.total = tot;
  out.filters = filters;
  // products, orthonormalisations (Gram, Cholesky and inverse, solve; three
  // passes and half steps besides when steep), the SVD of the projection (the
  // bidiagonalisation model), and the checks
  const double ld = l, md = m, nd = n, starts = 1.0 + PSVD_POWER, passes = steep ? 3.0 : 1.0;
  auto orth_flops = [&](double p) { return passes * (2.0 * p * ld * ld + 2.0 / 3.0 * ld * ld * ld); };
  out.flops = 2.0 * md * nd * ld * (1.0 + 2.0 * PSVD_POWER + 4.0 * filters + 2.0) +
              (starts + filters) * orth_flops(nd) + (2.0 + (steep ? PSVD_POWER : 0)) * orth_flops(md) +
              4.0 * nd * ld * ld - (4.0 / 3.0) * ld * ld * ld + 4.0 * (nd + ld) * ld * r + 4.0 * md * nd * r +
              4.0 * md * ld * r;
  if (trace)
    fprintf(stderr, "[ttm] psvd %dx%d l=%d filters=%d sweeps=%d rank=%d missed=%.2e disc=%.3e total=%.3e\n", m, n, l,
            filters, out.sweeps, r, out.missed, disc, tot);
  return out;
}
}  // namespace

PsvdResult psvd_oside(const double *Theta, int m, int n, int cap, double eps, int max_sweeps, double *pt, double *xt,
                      double *ws, hipStream_t s, KernelTimer *timer, int trace, double *sigma) {
  PsvdResult out = psvd_run(Theta, m, n, cap, eps, max_sweeps, pt, xt, ws, s, timer, trace, sigma, false);
  if (out.breakdown && out.err == TTM_OK) {
    const double before = out.solve_flops;
    out = psvd_run(Theta, m, n, cap, eps, max_sweeps, pt, xt, ws, s, timer, trace, sigma, true);
    out.solve_flops += before;
  }
  return out;
}

}  // namespace ttm
