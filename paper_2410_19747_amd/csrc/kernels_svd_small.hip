// Truncated SVD of a small matrix in one launch: column ordering, Householder
// QR, one-sided Jacobi, the rule of Eq. (eps) and the singular vectors, by one
// workgroup that holds the matrix in registers.
//
// The block method of kernels_svd.hip takes, per sweep, a sort, a Gram, a
// solve and an apply launch per round and one read-back: at k = 64 columns
// about 25 launches and 330 us, of which the matrix's own arithmetic is a few
// per cent.  Here the columns sit in lanes and the rows are spread over the
// registers, the lane groups and the waves, so that a step of the tournament
// is a dot product per column pair, a rotation and its application, without a
// launch or a read-back inside an SVD.
//
// Layout (LN lanes per row group, NW waves): lane l holds columns 4u .. 4u + 3,
// u = l mod LN, as two units of two columns (A: 0, 1; B: 2, 3); the H = 64 / LN
// lane groups and the waves split the rows: group q = w H + l / LN holds the
// rows i Q + q, i < RL, with Q = NW H.  The tile is N = 4 LN columns by as many
// rows, or by 96 for sides of 65 to 96, which need no more (a step's dot
// products and rotations then run over three quarters of the rows: 1223 ->
// 988 us at 96 columns).
//
// What bounds it is the issue and the latency of one wave per SIMD (an
// instruction issues in 4 cycles, an FP64 result returns after about 10, a
// hardware root or reciprocal after 22, a lane swap and add after 43, an LDS
// exchange between four waves after 216), so instructions are what is saved:
//  * up to 32 columns one wave holds the whole tile and a step meets no barrier;
//  * two column pairs per lane share a step: the first lane swap of their dot
//    products merges the two sums into the halves of the wave, and each half
//    computes one rotation;
//  * the tournament moves one unit per lane and only every second step, by
//    one DPP lane permutation (lane u to lane u ^ m) with no lane singled out.
//    The circle method, which moves both units and turns round at the ends,
//    took 1230, 1590 and 2830 cycles per step at 32, 64 and 128 columns,
//    against 780, 1150 and 1910.
// Measured, a k x k matrix with values i^-2, whole SVD with its read-back, by
// the block method and here: k = 8: 446 and 71 us, 16: 522 and 79, 32: 646 and
// 146, 64: 988 and 367, 96: 1476 and 988, 128: 2168 and 1261; 64 x 512: 1065
// and 524, 1024 x 128: 2162 and 1368.  Of it the QR takes 680, 1490, 2150 and
// 3500 cycles a column and a sweep 10.9, 27, 77 and 261 thousand at 16, 32, 64
// and 128 columns (with each sum of a QR step read from LDS behind the store
// of the one before, and the order counted by one thread a column: 860, 1900,
// 3050 and 4150; 12.1, 29, 81 and 275).  Above 128 columns the tile no longer
// fits the registers and LDS of one workgroup.
#include <limits.h>
#include <math.h>

#include "ttm_internal.h"

namespace ttm {
namespace {
typedef double d2 __attribute__((ext_vector_type(2)));

template <int LN, int NW, int ROWS>
struct SmallTile {
  static constexpr int H = 64 / LN;   // lanes of a wave that share a unit pair
  static constexpr int N = 4 * LN;    // columns of the tile
  static constexpr int Q = NW * H;    // row groups
  static constexpr int RL = ROWS / Q;  // rows of a lane
  static constexpr int CL = N / Q;     // columns that a row group counts for the order
  static constexpr int LD = ROWS + 1;    // LDS column stride (odd: lanes of different columns hit different banks)
  static constexpr int NT = 64 * NW;  // threads
};

template <int LN, int NW, int ROWS>
struct SmallSmem {
  typedef SmallTile<LN, NW, ROWS> T;
  double W[T::N * T::LD];       // columns of the matrix, staged
  __align__(16) double part[2][NW][T::N];  // per-wave sums of the columns (or of the pairs), double-buffered
  __align__(16) double row[2][T::N];       // the pivot row of a QR step
  double v[NW][T::H][T::RL];    // the pivot column of a QR step, per wave
  __align__(16) double norm[T::N];         // squared column norms, then the sorted ones
  unsigned count[NW][LN];       // places of four columns, by wave
  int perm[T::N];               // position -> column
  int orow[T::N];               // row of U that each row of W belongs to
  int spos[T::N];               // column -> place among the sorted singular values
  double result[8];
};

__device__ __forceinline__ double swap16_sum(double v) {
  const unsigned lo = __double2loint(v), hi = __double2hiint(v);
  auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  return __hiloint2double(b[0], a[0]) + __hiloint2double(b[1], a[1]);
}
// The sum over the row groups in a half of the wave (lanes l mod LN equal,
// l / 32 equal), bitwise the same in each (every stage adds the same two
// values, in either order).
template <int LN>
__device__ __forceinline__ double half_sum(double v) {
  if (LN <= 4) v += __builtin_amdgcn_mov_dpp(v, 0x124, 0xf, 0xf, false);  // row_ror:4
  if (LN <= 8) v += __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, false);  // row_ror:8
  if (LN <= 16) v = swap16_sum(v);
  return v;
}
// a summed over the halves of the wave in its lower half, b in its upper.
__device__ __forceinline__ double merge_halves(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// The lower half's value to every lane in a, the upper half's in b.
__device__ __forceinline__ void both_halves(double v, double &a, double &b) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
  a = __hiloint2double(hi[0], lo[0]);
  b = __hiloint2double(hi[1], lo[1]);
}
// Sum over all row groups of the wave.
template <int LN>
__device__ __forceinline__ double group_sum(double v) {
  return half_sum<LN>(merge_halves(v, v));
}
// The value of lane l ^ m, m = 1, 2, 7, 15, 16 for K = 1 .. 5: m flips bit
// K - 1 of the lane, and whatever it does to the bits below.
template <int K>
__device__ __forceinline__ double lane_xor(double v) {
  if (K == 1) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, false);   // quad_perm 1 0 3 2
  if (K == 2) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, false);   // quad_perm 2 3 0 1
  if (K == 3) return __builtin_amdgcn_mov_dpp(v, 0x141, 0xf, 0xf, false);  // row_half_mirror
  if (K == 4) return __builtin_amdgcn_mov_dpp(v, 0x140, 0xf, 0xf, false);  // row_mirror
  // rows of 16 exchanged: [0] holds the even rows' values, [1] the odd rows'
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
  const bool odd = (threadIdx.x & 16) != 0;
  return odd ? __hiloint2double(hi[0], lo[0]) : __hiloint2double(hi[1], lo[1]);
}
// 1 / sqrt(x) and 1 / x to rounding, from the hardware estimates and two
// Newton steps (x normal and positive).
__device__ __forceinline__ double rsqrt2(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = y * fma(-0.5 * x * y, y, 1.5);
  return y * fma(-0.5 * x * y, y, 1.5);
}
__device__ __forceinline__ double recip2(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// One workgroup's state: the tile and this lane's place in it.
template <int LN, int NW, int ROWS>
struct Small {
  typedef SmallTile<LN, NW, ROWS> T;
  SmallSmem<LN, NW, ROWS> &sm;
  int lane, w, u, h, q;
  double x[4][T::RL];

  __device__ __forceinline__ explicit Small(SmallSmem<LN, NW, ROWS> &s) : sm(s) {
    lane = threadIdx.x & 63;
    w = threadIdx.x >> 6;
    u = lane % LN;
    h = lane / LN;
    q = w * T::H + h;
  }

  // The lane's columns of the staged matrix, in the order of sm.perm.
  __device__ __forceinline__ void fetch() {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int c = sm.perm[4 * u + e];
#pragma unroll
      for (int i = 0; i < T::RL; ++i) x[e][i] = sm.W[c * T::LD + i * T::Q + q];
    }
  }
  __device__ __forceinline__ void stash() {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < T::RL; ++i) sm.W[(4 * u + e) * T::LD + i * T::Q + q] = x[e][i];
  }
  __device__ __forceinline__ double wave_total(int par, int c) const {
    double t = sm.part[par][0][c];
    if (NW == 4) t = (t + sm.part[par][1][c]) + (sm.part[par][2][c] + sm.part[par][3][c]);
    return t;
  }
  static __device__ __forceinline__ void get4(const double *src, double (&x)[4]) {
    const d2 lo = *(const d2 *)src, hi = *(const d2 *)(src + 2);
    x[0] = lo.x; x[1] = lo.y; x[2] = hi.x; x[3] = hi.y;
  }
  static __device__ __forceinline__ void put4(double *dst, const double (&x)[4]) {
    *(d2 *)dst = d2{x[0], x[1]};
    *(d2 *)(dst + 2) = d2{x[2], x[3]};
  }
  // wave_total of the lane's columns.
  __device__ __forceinline__ void lane_totals(int par, double (&t)[4]) const {
    double p[NW][4];
#pragma unroll
    for (int i = 0; i < NW; ++i) get4(&sm.part[par][i][4 * u], p[i]);
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] = NW == 4 ? (p[0][e] + p[1][e]) + (p[2 % NW][e] + p[3 % NW][e]) : p[0][e];
  }
  // sm.norm = the squared norms of the columns by slot.
  __device__ __forceinline__ void norms() {
    static_assert(NW == 1 || NW == 4, "wave_total");
    __syncthreads();  // part may still be read
    double n[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      double a = 0.0;
#pragma unroll
      for (int i = 0; i < T::RL; ++i) a = fma(x[e][i], x[e][i], a);
      n[e] = group_sum<LN>(a);
    }
    if (h == 0) put4(NW > 1 ? &sm.part[0][w][4 * u] : &sm.norm[4 * u], n);
    __syncthreads();
    if (NW > 1) {
      if (threadIdx.x < T::N) sm.norm[threadIdx.x] = wave_total(0, threadIdx.x);
      __syncthreads();
    }
  }
  // sm.perm = the slots by decreasing norm (ties by slot).  Row group q
  // counts, for the lane's four columns, the norms of slots i Q + q before
  // them; a column's place is the sum over the groups (at most 127, four
  // columns to a word).
  __device__ __forceinline__ void order() {
    double me[4], o[T::CL];
    get4(&sm.norm[4 * u], me);
#pragma unroll
    for (int i = 0; i < T::CL; ++i) o[i] = sm.norm[i * T::Q + q];
    unsigned pos = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      unsigned cnt = 0;
#pragma unroll
      for (int i = 0; i < T::CL; ++i)
        cnt += (unsigned)((o[i] > me[e]) | ((o[i] == me[e]) & (i * T::Q + q < 4 * u + e)));
      pos |= cnt << (8 * e);
    }
    if (LN <= 4) pos += __builtin_amdgcn_update_dpp(pos, pos, 0x124, 0xf, 0xf, false);  // row_ror:4
    if (LN <= 8) pos += __builtin_amdgcn_update_dpp(pos, pos, 0x128, 0xf, 0xf, false);  // row_ror:8
    if (LN <= 16) {
      const auto k = __builtin_amdgcn_permlane16_swap(pos, pos, false, false);
      pos = k[0] + k[1];
    }
    const auto k = __builtin_amdgcn_permlane32_swap(pos, pos, false, false);
    pos = k[0] + k[1];
    if (NW > 1) {
      if (h == 0) sm.count[w][u] = pos;
      if (threadIdx.x < T::N) sm.perm[threadIdx.x] = threadIdx.x;  // every entry a slot, also when a norm is NaN
      __syncthreads();
      pos = 0;
#pragma unroll
      for (int i = 0; i < NW; ++i) pos += sm.count[i][u];
    } else {
      if (threadIdx.x < T::N) sm.perm[threadIdx.x] = threadIdx.x;
      __syncthreads();
    }
    if (w == 0 && h == 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) sm.perm[(pos >> (8 * e)) & 255] = 4 * u + e;
    }
    __syncthreads();
  }

  // The column of largest remaining norm (left: those norms by lane, negative
  // for a column that is no candidate), the same in every lane: the maximum
  // of the norms' high words with the column in their low bits, which leaves
  // at least 13 bits of the mantissa.
  __device__ __forceinline__ int pivot_column(const double (&left)[4]) {
    static_assert(T::N <= 128, "bits of the key");
    int key = INT_MIN;
#pragma unroll
    for (int e = 0; e < 4; ++e) key = max(key, (__double2hiint(left[e]) & ~(T::N - 1)) | (4 * u + e));
    key = max(key, __builtin_amdgcn_update_dpp(key, key, 0xB1, 0xf, 0xf, false));   // quad_perm 1 0 3 2
    key = max(key, __builtin_amdgcn_update_dpp(key, key, 0x4E, 0xf, 0xf, false));   // quad_perm 2 3 0 1
    if (LN >= 8) key = max(key, __builtin_amdgcn_update_dpp(key, key, 0x141, 0xf, 0xf, false));   // row_half_mirror
    if (LN >= 16) key = max(key, __builtin_amdgcn_update_dpp(key, key, 0x140, 0xf, 0xf, false));  // row_mirror
    if (LN >= 32) {
      const auto k2 = __builtin_amdgcn_permlane16_swap(key, key, false, false);
      key = max((int)k2[0], (int)k2[1]);
    }
    return __builtin_amdgcn_readfirstlane(key) & (T::N - 1);
  }
  // left = the squared norms of what remains of the candidates.
  __device__ __forceinline__ void remaining(double (&left)[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      double a = 0.0;
#pragma unroll
      for (int i = 0; i < T::RL; ++i) a = fma(x[e][i], x[e][i], a);
      a = group_sum<LN>(a);
      if (NW > 1) {
        if (h == 0) sm.part[0][w][4 * u + e] = a;
      } else {
        left[e] = left[e] < 0.0 ? left[e] : a;
      }
    }
    if (NW > 1) {
      __syncthreads();
      double a[4];
      lane_totals(0, a);
#pragma unroll
      for (int e = 0; e < 4; ++e) left[e] = left[e] < 0.0 ? left[e] : a[e];
      __syncthreads();
    }
  }

  // Householder QR of the tile with column pivoting (kk reflectors on the
  // first nc columns; the others are zero): leaves (R P^T)^T staged, column j
  // of sm.W = row j of R over the columns in their own slots, columns beyond
  // kk zero.  Finished rows are zeroed in the registers, so a step's dot
  // products run over whole columns: with x the pivot column from row j on,
  // s = x^T x, alpha = x_j, beta = -sign(alpha) sqrt(s) and v = x - beta e_j,
  // every unfinished column c loses v (x^T c - beta c_j) / (s - alpha beta).
  // The remaining norms lose the square of their entry in row j and are
  // formed anew every eight steps; they choose the pivot and nothing else.
  // With the columns only sorted once, Jacobi took 8.4 sweeps on average on
  // the swaps of a product of bond 32 over 18 modes of 2 and 9.6 on those of
  // a 64 x 64 field at bond 32; pivoted, 6.5 and 6.3.
  // qr_rows<I> reduces the rows of slot I, so that every register index is
  // known when it is compiled (one loop body with the slots shifted down
  // between row blocks took 1.2 to 1.4 times as long at 64 and 128 columns).
  template <int I>
  __device__ __forceinline__ void qr_rows(int kk, double (&left)[4]) {
    if constexpr (I < T::RL) {
#pragma unroll 1
      for (int qq = 0; qq < T::Q; ++qq) {
        const int j = I * T::Q + qq;
        if (j >= kk) return;
        if ((j & 7) == 0) remaining(left);
        const int pc = pivot_column(left);
        const int par = qq & 1, je = pc & 3;
        const bool mine = (q == qq);
        if (u == (pc >> 2)) {
#pragma unroll
          for (int i = I; i < T::RL; ++i) {
            const double lo = (je & 1) ? x[1][i] : x[0][i], hi = (je & 1) ? x[3][i] : x[2][i];
            sm.v[w][h][i] = (je & 2) ? hi : lo;
          }
        }
        if (mine) {
          double rc0[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) rc0[e] = x[e][I];
          put4(&sm.row[par][4 * u], rc0);
        }
        wave_sync();
        double vv[T::RL], d[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int i = I; i < T::RL; ++i) {
          vv[i] = sm.v[w][h][i];
#pragma unroll
          for (int e = 0; e < 4; ++e) d[e] = fma(vv[i], x[e][i], d[e]);
        }
        wave_sync();
        // columns 0, 1 (2, 3) merged into the halves, each half the sum of one
        d[0] = half_sum<LN>(merge_halves(d[0], d[1]));
        d[2] = half_sum<LN>(merge_halves(d[2], d[3]));
        if ((lane & 31) < LN) {
          sm.part[par][w][4 * u + (lane >> 5)] = d[0];
          sm.part[par][w][4 * u + 2 + (lane >> 5)] = d[2];
        }
        __syncthreads();
        // all LDS reads of the step at once
        const double s = wave_total(par, pc), alpha = sm.row[par][pc];
        double tot[4], rj[4], f[4], rc[4];
        lane_totals(par, tot);
        get4(&sm.row[par][4 * u], rj);
        // The matrix has norm one, so a column with s below 2^-960 (rounding
        // errors of rounding errors, where the matrix has lost its rank) is
        // zero: no reflection, and 1 / s cannot overflow.
        const bool some = s > 0x1p-960;
        const double sn = some ? s : 1.0, root = sn * rsqrt2(sn);
        const double beta = some ? -copysign(root, alpha) : 0.0;
        const double rec = recip2(fma(fabs(alpha), root, sn)), inv = some ? rec : 0.0;
        const double vj = alpha - beta;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double ff = (tot[e] - beta * rj[e]) * inv;
          const bool piv = 4 * u + e == pc, open = left[e] >= 0.0 && !piv;
          rc[e] = open ? fma(-ff, vj, rj[e]) : (piv ? beta : 0.0);
          f[e] = open ? ff : 0.0;
          left[e] = open ? fmax(fma(-rc[e], rc[e], left[e]), 0.0) : -1.0;
        }
#pragma unroll
        for (int i = I; i < T::RL; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e][i] = fma(-f[e], vv[i], x[e][i]);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e][I] = mine ? 0.0 : x[e][I];
        if (mine && 4 * u < ROWS) {
#pragma unroll
          for (int e = 0; e < 4; ++e) sm.W[j * T::LD + 4 * u + e] = rc[e];
        }
      }
      qr_rows<I + 1>(kk, left);
    }
  }
  __device__ __forceinline__ void qr(int kk, int nc) {
    double left[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) left[e] = (4 * u + e < nc) ? 0.0 : -1.0;
    __syncthreads();  // the staged matrix has been fetched
    qr_rows<0>(kk, left);
    __syncthreads();
#pragma unroll 1
    for (int e = threadIdx.x; e < (T::N - kk) * ROWS; e += T::NT) sm.W[(kk + e / ROWS) * T::LD + e % ROWS] = 0.0;
  }

  // Limits of a sweep: the noise level thr of a squared norm, tol^2, the
  // square of the largest off-diagonal after which no sweep is due, and
  // (F / sqrt(L))^2 (see the header of kernels_svd.hip).
  double thr, tol2, done2, floor2;
  bool big;  // an off-diagonal above done2 was met

  // Two column pairs of the lane, (P0, Q0) and (P1, Q1).  The rotation as in
  // kernels_svd.hip: tan(2 angle) = 2 g / (nq - np) and the smaller angle,
  // t from the hardware root and reciprocal (it need only be close), c with
  // one step of third order on the residual 1 - c^2 - c^2 t^2, so that
  // c^2 + s^2 = 1 to rounding, either way alike: nothing gives the columns their
  // length back afterwards.  (A step on 1 - c^2 (1 + t^2), its product rounded,
  // left 2 u too much wherever 1e-8 < t < 1e-3, and the largest value 490 u too
  // large at 128 columns, 190 u at 64: now 6 and 6, the block method 5 and 5.)
  // The matrix is scaled to norm one, so no square over- or underflows.  The
  // carried norms change by t g; every sweep starts from new ones.
  template <int P0, int Q0, int P1, int Q1>
  __device__ __forceinline__ void step(int par, double (&nn)[4], bool upper) {
    double a0 = 0.0, a1 = 0.0, b0 = 0.0, b1 = 0.0;
#pragma unroll
    for (int i = 0; i < T::RL; i += 2) {
      a0 = fma(x[P0][i], x[Q0][i], a0);
      b0 = fma(x[P1][i], x[Q1][i], b0);
      if (i + 1 < T::RL) {
        a1 = fma(x[P0][i + 1], x[Q0][i + 1], a1);
        b1 = fma(x[P1][i + 1], x[Q1][i + 1], b1);
      }
    }
    if (T::RL > 1) {
      a0 += a1;
      b0 += b1;
    }
    double g = half_sum<LN>(merge_halves(a0, b0));
    if (NW > 1) {
      if ((lane & 31) < LN) sm.part[par][w][2 * u + (lane >> 5)] = g;
      __syncthreads();
      g = wave_total(par, 2 * u + (lane >> 5));
    }
    const double np = upper ? nn[P1] : nn[P0], nq = upper ? nn[Q1] : nn[Q0];
    const double hi2 = np > nq ? np : nq, lo2 = np > nq ? nq : np;
    const double den = hi2 * (lo2 > thr ? lo2 : floor2), gg = g * g;
    const bool live = hi2 > thr, on = live && gg > tol2 * den;
    big |= live && gg > done2 * den;
    const double d = nq - np, v = g + g;
    const double r2 = fma(d, d, v * v);
    const double wv = fma(r2, __builtin_amdgcn_rsq(r2), fabs(d));
    const double t0 = v * __builtin_amdgcn_rcp(copysign(wv, d));
    const double t2 = t0 * t0, y0 = __builtin_amdgcn_rsq(fma(t0, t0, 1.0));
    const double e = fma(-t2, y0 * y0, fma(-y0, y0, 1.0));
    const double y = fma(y0 * e, fma(0.375, e, 0.5), y0);
    const double t = on ? t0 : 0.0;  // 0 / 0 in an idle lane goes no further
    const double cc = on ? y : 1.0, ss = t * cc, tg = t * g;
    double c0, c1, s0, s1, tg0, tg1;
    both_halves(cc, c0, c1);
    both_halves(ss, s0, s1);
    both_halves(tg, tg0, tg1);
    nn[P0] -= tg0;
    nn[Q0] += tg0;
    nn[P1] -= tg1;
    nn[Q1] += tg1;
#pragma unroll
    for (int i = 0; i < T::RL; ++i) {
      const double p0 = c0 * x[P0][i] - s0 * x[Q0][i], p1 = c1 * x[P1][i] - s1 * x[Q1][i];
      x[Q0][i] = s0 * x[P0][i] + c0 * x[Q0][i];
      x[Q1][i] = s1 * x[P1][i] + c1 * x[Q1][i];
      x[P0][i] = p0;
      x[P1][i] = p1;
    }
  }
  // Unit B from lane u ^ m.
  template <int K>
  __device__ __forceinline__ void move(double (&nn)[4]) {
#pragma unroll
    for (int e = 2; e < 4; ++e) {
      nn[e] = lane_xor<K>(nn[e]);
#pragma unroll
      for (int i = 0; i < T::RL; ++i) x[e][i] = lane_xor<K>(x[e][i]);
    }
  }
  // The lower lanes' B (bit K - 1 of u clear) against the upper lanes' A.
  template <int K>
  __device__ __forceinline__ void split(double (&nn)[4]) {
    const bool top = (u >> (K - 1)) & 1;
    auto swap = [&](double &a, double &b) {
      const double r = lane_xor<K>(top ? a : b);
      a = top ? r : a;
      b = top ? b : r;
    };
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      swap(nn[e], nn[2 + e]);
#pragma unroll
      for (int i = 0; i < T::RL; ++i) swap(x[e][i], x[2 + e][i]);
    }
  }
  // One cyclic sweep: the columns of each unit, then a tournament of the
  // 2 LN units, each meeting two steps (four column pairs).  In phase P every
  // A of a group of 2^P lanes meets every B of the group, the Bs moving by
  // lane ^ m with m in Gray-code order; a split then brings the As of the
  // group's two halves together, and the Bs, for phase P - 1.  Columns end
  // in other slots than they began.  nn: the squared norms.  Returns whether
  // another sweep is due.
  __device__ __forceinline__ bool sweep(double (&nn)[4]) {
    constexpr int LOG = LN == 4 ? 2 : LN == 8 ? 3 : LN == 16 ? 4 : 5;
    const bool upper = lane >= 32;
    big = false;
    step<0, 1, 2, 3>(0, nn, upper);
#pragma unroll 1
    for (int p = LOG; p >= 0; --p) {
#pragma unroll 1
      for (int r = 1; r <= (1 << p); ++r) {
        step<0, 2, 1, 3>(1, nn, upper);
        step<0, 3, 1, 2>(0, nn, upper);
        if (r < (1 << p)) {
          const int k = __builtin_ctz(r);
          if (k == 0) move<1>(nn);
          else if (k == 1) move<2>(nn);
          else if (LOG >= 3 && k == 2) move<3>(nn);
          else if (LOG >= 4 && k == 3) move<4>(nn);
          else if (LOG >= 5) move<5>(nn);
        }
      }
      if (p == 1) split<1>(nn);
      else if (p == 2) split<2>(nn);
      else if (LOG >= 3 && p == 3) split<3>(nn);
      else if (LOG >= 4 && p == 4) split<4>(nn);
      else if (LOG >= 5 && p == 5) split<5>(nn);
    }
    return __any(big) != 0;  // every wave has seen every pair
  }
};

template <int LN, int NW, int ROWS, int MODE>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(1, 1))) void svd_small_kernel(SvdSmall a) {
  typedef SmallTile<LN, NW, ROWS> T;
  __shared__ SmallSmem<LN, NW, ROWS> sm;
  Small<LN, NW, ROWS> s(sm);
  const int tid = threadIdx.x;
  // tolerance and noise level of a k-row Jacobi (see kernels_svd.hip)
  const double tol = sqrt((double)a.k) * 2.220446049250313e-16, noise = 8.0 * tol;
  // 1. stage the source, column by column
  if (MODE == SMALL_Y) {
    for (int e = tid; e < T::N * ROWS; e += T::NT) {
      const int c = e / ROWS, r = e % ROWS;
      sm.W[c * T::LD + r] = (r < a.np && c < a.no) ? a.src[(int64_t)c * a.ld + r] : 0.0;
    }
  } else if (MODE == SMALL_R) {
    for (int e = tid; e < T::N * ROWS; e += T::NT) {
      const int j = e / ROWS, c = e % ROWS;
      sm.W[j * T::LD + c] = (j < a.k && c <= j) ? a.src[(int64_t)j * a.ld + c] : 0.0;
    }
  } else {
    // column c of W (or of the matrix that QR takes) is row c of R
    for (int e = tid; e < T::N * ROWS; e += T::NT) {
      const int j = e / T::N, c = e % T::N;  // entry (c, j) of R, c <= j, along a column of S
      sm.W[c * T::LD + j] = (j < a.k && c <= j) ? a.src[(int64_t)j * a.ld + c] : 0.0;
    }
  }
  if (tid < T::N) {
    sm.orow[tid] = (MODE == SMALL_RT && a.rowperm && tid < a.k) ? a.rowperm[tid] : tid;
    sm.perm[tid] = tid;
  }
  __syncthreads();
  // 2. the matrix to norm one (over 2^ex, with ||W||_F / 2^ex in [1/2, 1)),
  // the columns' order and the QR, then sweeps until the largest off-diagonal
  // met in one has off^2 <= tol / 100 (the rule of svd_oside: what remains is
  // of order off^2).  One loop, so that each part's instructions are there
  // once.
  enum { SCALE, QR, SORT, SWEEP };
  int todo = SCALE;
  int sweeps = 0, ex = 0;
  bool conv = false;
#pragma unroll 1
  while (true) {
    s.fetch();
    if ((MODE == SMALL_Y || MODE == SMALL_RTQ) && todo == QR) {
      s.qr(a.k, MODE == SMALL_Y ? a.no : a.k);
      if (tid < T::N) sm.perm[tid] = tid;
      __syncthreads();
      todo = SORT;
      continue;
    }
    if (todo == SWEEP) {
      double nn[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) nn[e] = sm.norm[sm.perm[4 * s.u + e]];
      conv = !s.sweep(nn);
      ++sweeps;
    }
    s.norms();
    s.order();
    if (todo == SCALE) {
      double f = 0.0;  // ||W||_F^2, in a fixed order
      for (int c = s.lane; c < T::N; c += 64) f += sm.norm[c];
      for (int o = 32; o > 0; o >>= 1) f += __shfl_xor(f, o, 64);
      __syncthreads();
      if (f > 0.0 && isfinite(f)) ex = __builtin_amdgcn_frexp_exp(sqrt(f));
      if (tid < T::N) sm.norm[tid] = __builtin_amdgcn_ldexp(sm.norm[tid], -2 * ex);
      f = __builtin_amdgcn_ldexp(f, -2 * ex);
      s.thr = noise * noise * f;
      s.tol2 = tol * tol;
      s.done2 = 0.01 * tol;
      s.floor2 = f / (double)a.k;
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < T::RL; ++i) s.x[e][i] = __builtin_amdgcn_ldexp(s.x[e][i], -ex);
      if (MODE == SMALL_Y && tid < T::N) sm.orow[tid] = sm.perm[tid];
      if (MODE == SMALL_RTQ && tid < T::N) sm.perm[tid] = tid;
      todo = (MODE == SMALL_Y || MODE == SMALL_RTQ) ? QR : SWEEP;
    } else {
      todo = SWEEP;
      if (conv || sweeps >= a.max_sweeps) break;
    }
    s.stash();
    __syncthreads();
  }
  // 3. singular values and the rule of Eq. (eps) (see jacobi_rank_kernel)
  if (tid < T::N) sm.spos[tid] = T::N;
  __syncthreads();
  if (tid < T::N) sm.spos[sm.perm[tid]] = tid;
  double sq = 0.0;
  if (tid < T::N) sq = sm.norm[sm.perm[tid]];
  __syncthreads();
  if (tid < T::N) {
    sm.norm[tid] = sq;
    if (a.sig && tid < a.k) a.sig[tid] = __builtin_amdgcn_ldexp(sqrt(sq), ex);
  }
  __syncthreads();
  if (tid < 64) {
    constexpr int CH = (T::N + 63) / 64;
    double suf[CH], after = 0.0;
    for (int ch = CH - 1; ch >= 0; --ch) {
      const int t = ch * 64 + tid;
      double v = (t < a.k) ? sm.norm[t] : 0.0;
      for (int o = 1; o < 64; o <<= 1) {
        const double y = __shfl_down(v, o, 64);
        v += (tid + o < 64) ? y : 0.0;
      }
      suf[ch] = v + after;  // sum over i >= t
      after = __shfl(suf[ch], 0, 64);
    }
    const double wsum = after;
    const double extra = a.full_total ? fmax(__builtin_amdgcn_ldexp(a.full_total[0], -2 * ex) - wsum, 0.0) : 0.0;
    const double total = wsum + extra;
    const double nz2 = noise * noise * wsum;
    int best = a.k, nsig = 0;
    for (int ch = CH - 1; ch >= 0; --ch) {
      const int t = ch * 64 + tid;
      const double tail = suf[ch] + extra;
      const bool hit = t >= 1 && t < a.k && (tail <= 0.0 || tail < a.eps * total);
      const uint64_t m = __ballot(hit);
      if (m) best = ch * 64 + __ffsll((unsigned long long)m) - 1;
      nsig += __popcll(__ballot(t < a.k && sm.norm[t] > nz2));
    }
    int r = min(best, nsig);
    if (r < 1) r = 1;
    if (a.cap > 0 && r > a.cap) r = a.cap;
    if (a.forced > 0) r = a.forced;
    if (r > a.k) r = a.k;
    double disc = extra;
    for (int ch = 0; ch < CH; ++ch) {
      const double y = __shfl(suf[ch], r & 63, 64);
      if (r < a.k && (r >> 6) == ch) disc = y + extra;
    }
    if (tid == 0) {
      sm.result[0] = (double)r;
      sm.result[1] = __builtin_amdgcn_ldexp(disc, 2 * ex);
      sm.result[2] = __builtin_amdgcn_ldexp(total, 2 * ex);
      sm.result[3] = 0.0;
      sm.result[4] = isfinite(total) ? 0.0 : 1.0;
      sm.result[5] = __builtin_amdgcn_ldexp(wsum, 2 * ex);
      sm.result[6] = (double)nsig;
      sm.result[7] = conv ? (double)sweeps : -(double)sweeps;
      for (int i = 0; i < 8; ++i) a.result[i] = sm.result[i];
    }
  }
  __syncthreads();
  // 4. the vectors: columns of W over their norms (zero where that is zero)
  const int r = (int)sm.result[0], kg = max(r, min(a.k, (int)sm.result[6]));
  const int rows = (MODE == SMALL_Y) ? a.no : a.k;
  const int64_t os = a.u_os ? a.u_os : (int64_t)r;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int t = sm.spos[4 * s.u + e];
    const bool inu = a.u && t < r, inall = a.uall && t < kg;
    if (!inu && !inall) continue;
    const double nrm2 = t < T::N ? sm.norm[t] : 0.0;
    const double inv = nrm2 > 0.0 ? 1.0 / sqrt(nrm2) : 0.0;
#pragma unroll
    for (int i = 0; i < T::RL; ++i) {
      const int row = i * T::Q + s.q;
      if (row < rows) {
        const int o = sm.orow[row];
        const double val = s.x[e][i] * inv;
        if (inu) a.u[(int64_t)o * os + (int64_t)t * a.u_ts] = val;
        if (inall) a.uall[(int64_t)t * a.uall_ld + o] = val;
      }
    }
  }
}

template <int LN, int NW, int ROWS>
void launch_mode(const SvdSmall &a, hipStream_t s) {
  if (a.mode == SMALL_Y)
    hipLaunchKernelGGL((svd_small_kernel<LN, NW, ROWS, SMALL_Y>), dim3(1), dim3(64 * NW), 0, s, a);
  else if (a.mode == SMALL_RT)
    hipLaunchKernelGGL((svd_small_kernel<LN, NW, ROWS, SMALL_RT>), dim3(1), dim3(64 * NW), 0, s, a);
  else if (a.mode == SMALL_RTQ)
    hipLaunchKernelGGL((svd_small_kernel<LN, NW, ROWS, SMALL_RTQ>), dim3(1), dim3(64 * NW), 0, s, a);
  else
    hipLaunchKernelGGL((svd_small_kernel<LN, NW, ROWS, SMALL_R>), dim3(1), dim3(64 * NW), 0, s, a);
}
}  // namespace

hipError_t launch_svd_small(const SvdSmall &a, hipStream_t s) {
  const int side = (a.mode == SMALL_Y) ? (a.np > a.no ? a.np : a.no) : a.k;
  if (a.k < 1 || side > kSvdSmallSide || a.mode < SMALL_Y || a.mode > SMALL_R) return hipErrorInvalidValue;
  if (side <= 16)
    launch_mode<4, 1, 16>(a, s);
  else if (side <= 32)
    launch_mode<8, 1, 32>(a, s);
  else if (side <= 64)
    launch_mode<16, 4, 64>(a, s);
  else if (side <= 96)
    launch_mode<32, 4, 96>(a, s);
  else
    launch_mode<32, 4, 128>(a, s);
  return hipGetLastError();
}

// dst (no x nc, column-major) = src (k x nc, column-major) over zero rows.
__global__ void embed_rows_kernel(double *__restrict__ dst, const double *__restrict__ src, int k, int no, int nc) {
  const int64_t n = (int64_t)no * nc;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    const int t = (int)(e / no), o = (int)(e % no);
    dst[e] = (o < k) ? src[(int64_t)t * k + o] : 0.0;
  }
}

hipError_t launch_embed_rows(double *dst, const double *src, int k, int no, int nc, hipStream_t s) {
  int64_t g = ((int64_t)no * nc + 255) / 256;
  if (g > 4096) g = 4096;
  hipLaunchKernelGGL(embed_rows_kernel, dim3((int)g), dim3(256), 0, s, dst, src, k, no, nc);
  return hipGetLastError();
}

}  // namespace ttm
