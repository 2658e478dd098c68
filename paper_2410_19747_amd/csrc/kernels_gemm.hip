// Batched strided GEMM on the gfx950 matrix cores with a split-stride
// epilogue.  FP64 (v_mfma_f64_16x16x4_f64) throughout, or, for the
// contractions of a mixed-precision product, operands rounded to FP32
// (v_mfma_f32_16x16x4_f32), to BF16 (v_mfma_f32_16x16x16_bf16) or split into
// three BF16 terms (six BF16 products, about FP32 accuracy), all accumulated
// in FP32 within each 16-deep k-tile and in FP64 across k-tiles; inputs and
// outputs stay FP64 in memory.
//
// Used for every contraction of the TTM sweep: the COPY-tensor contraction
// of Eq. (contract) is a batch of d products sharing the physical index; the
// merge of a swap pair is one product whose epilogue stores the leg-exchanged
// unfolding; the R (or S V^T) factor of a gauge move is multiplied into the
// next carriage; the variational baseline's environment contractions.
#include <algorithm>

#include "ttm_internal.h"

namespace ttm {

typedef double dbl4 __attribute__((ext_vector_type(4)));
typedef float flt4 __attribute__((ext_vector_type(4)));

namespace {
constexpr int BM = 64;
constexpr int BN = 64;
constexpr int BK = 16;
constexpr int NT = 256;  // 4 waves of 64 lanes, 2 x 2 over the 64 x 64 tile
constexpr int kDirectK = 256;            // longest K that keeps the tiled kernel's order
constexpr int64_t kSplitTarget = 512;  // workgroups a split product aims for (two per CU)

// A thread's share of an operand tile (64 rows of A or columns of B, 16 k):
// element q is at (row i(q), k(q)).  The fast index over the lanes follows the
// operand's unit stride, so that neighbouring lanes read neighbouring
// addresses: along k 16 k by 4 rows a wave, else 64 rows.  The pointers are
// formed once and advance by a k-tile; rows beyond the operand read its last
// row, whose products no output takes, so that only a last, short k-tile
// checks anything (address arithmetic and checks per element took half as
// long as the matrix cores' work).
struct TileLoad {
  static constexpr int E = BM * BK / NT;  // elements per thread
  static_assert(BM == BN && BM == 64 && NT == 256 && BK == 16, "thread to element mapping below");
  const double *p[E];
  int64_t step;  // one k-tile
  bool kfast;
  __device__ __forceinline__ int row(int q) const {
    return kfast ? (int)(threadIdx.x / BK) + q * (NT / BK) : (int)(threadIdx.x % BM);
  }
  __device__ __forceinline__ int k(int q) const {
    return kfast ? (int)(threadIdx.x % BK) : (int)(threadIdx.x / BM) + q * (NT / BM);
  }
  // rs: stride of the rows (of A; columns of B), ks: of k.
  __device__ __forceinline__ TileLoad(const double *base, int64_t rs, int64_t ks, bool kf, int first, int rows, int kbeg)
      : step(BK * ks), kfast(kf) {
#pragma unroll
    for (int q = 0; q < E; ++q)
      p[q] = base + (int64_t)min(first + row(q), rows - 1) * rs + (int64_t)(kbeg + k(q)) * ks;
  }
  // The next k-tile: whole, or the last `left` < 16 of K (no branch between
  // the two here: a value that comes from either of two loads is waited for
  // at once).
  __device__ __forceinline__ void fetch(double (&v)[E]) {
#pragma unroll
    for (int q = 0; q < E; ++q) v[q] = *p[q];
#pragma unroll
    for (int q = 0; q < E; ++q) p[q] += step;
  }
  __device__ __forceinline__ void fetch_tail(double (&v)[E], int left) const {
#pragma unroll
    for (int q = 0; q < E; ++q) v[q] = (k(q) < left) ? *p[q] : 0.0;
  }
};

// Word of entry (k, i) of a staged 16 x 64 tile.  The matrix cores read four
// consecutive k by 16 consecutive i; writes along k cover 16 k by 4 i, writes
// along i 64 i of one k: with this exclusive or every one of them touches each
// bank pair twice, the least that 64 lanes of 8 bytes can.
__device__ __forceinline__ int tile_word(int k, int i) { return k * BM + (i ^ ((k & 3) << 4) ^ ((k >> 2) << 2)); }

__device__ __forceinline__ int64_t out_index(const GemmArgs &g, int i, int j) {
  int64_t oi = (g.c_rdiv == 1) ? (int64_t)i * g.c_rs1
                               : (int64_t)(i / g.c_rdiv) * g.c_rs1 + (int64_t)(i % g.c_rdiv) * g.c_rs0;
  int64_t oj = (g.c_cdiv == 1) ? (int64_t)j * g.c_cs1
                               : (int64_t)(j / g.c_cdiv) * g.c_cs1 + (int64_t)(j % g.c_cdiv) * g.c_cs0;
  return oi + oj;
}
}  // namespace

// Each workgroup computes one 64 x 64 tile of one batch entry.  Wave w owns
// the 32 x 32 quadrant (w / 2, w % 2) as 2 x 2 MFMA blocks of 16 x 16.
// MFMA operand layout (16x16x4, f64): lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16]; accumulator register t of lane l holds D[4*t + l/16][l % 16]
// (rows interleaved across the four 16-lane groups; measured on gfx950).
__global__ __launch_bounds__(NT, 2) void gemm_f64_kernel(GemmArgs g) {
  __shared__ double As[2][BK * BM];
  __shared__ double Bs[2][BK * BN];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1;
  const int tile_m = blockIdx.y * BM;
  const int tile_n = blockIdx.x * BN;
  const int64_t bz = blockIdx.z / g.ksplit;
  const int kbeg = (g.ksplit > 1) ? (int)(blockIdx.z % g.ksplit) * g.kchunk : 0;
  const int kend = (g.ksplit > 1) ? min(g.K, kbeg + g.kchunk) : g.K;

  dbl4 acc[2][2];
  for (int x = 0; x < 2; ++x)
    for (int y = 0; y < 2; ++y) acc[x][y] = dbl4{0.0, 0.0, 0.0, 0.0};

  // Two k-tiles are in flight: while tile t is multiplied from one half of
  // the LDS, tile t + 1 (loaded during t - 1) goes into the other half and
  // tile t + 2 is loaded, one barrier a tile.  (Four in flight leave one
  // workgroup less per CU: 53 against 60 TFLOP/s at 4096^3.)
  TileLoad la(g.A + bz * g.a_bs, g.a_rs, g.a_cs, g.a_cs == 1, tile_m, g.M, kbeg);
  TileLoad lb(g.B + bz * g.b_bs, g.b_cs, g.b_rs, g.b_cs != 1, tile_n, g.N, kbeg);
  constexpr int E = TileLoad::E;
  double ra[2][E], rb[2][E];
  auto fetch = [&](int r, bool there) {
    if (there) {
      la.fetch(ra[r]);
      lb.fetch(rb[r]);
    }
  };
  auto stash = [&](int h, int r) {
#pragma unroll
    for (int q = 0; q < E; ++q) {
      As[h][tile_word(la.k(q), la.row(q))] = ra[r][q];
      Bs[h][tile_word(lb.k(q), lb.row(q))] = rb[r][q];
    }
  };
  auto multiply = [&](int h) {
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      const int kr = kk + (lane >> 4), c = lane & 15;
      const double a0 = As[h][tile_word(kr, wr * 32 + c)];
      const double a1 = As[h][tile_word(kr, wr * 32 + 16 + c)];
      const double b0 = Bs[h][tile_word(kr, wc * 32 + c)];
      const double b1 = Bs[h][tile_word(kr, wc * 32 + 16 + c)];
      acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
    }
  };
  const int whole = (kend - kbeg) / BK, tail = (kend - kbeg) % BK;
  fetch(0, whole > 0);
  fetch(1, whole > 1);
  stash(0, 0);
  __syncthreads();
  for (int t = 0; t < whole; t += 2) {
    fetch(0, t + 2 < whole);
    multiply(0);
    stash(1, 1);
    __syncthreads();
    if (t + 1 >= whole) break;
    fetch(1, t + 3 < whole);
    multiply(1);
    stash(0, 0);
    __syncthreads();
  }
  if (tail) {
    la.fetch_tail(ra[0], tail);
    lb.fetch_tail(rb[0], tail);
    stash(0, 0);
    __syncthreads();
    multiply(0);
  }

  double *C = g.C + bz * g.c_bs;
#pragma unroll
  for (int x = 0; x < 2; ++x) {
#pragma unroll
    for (int y = 0; y < 2; ++y) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int i = tile_m + wr * 32 + x * 16 + 4 * t + (lane >> 4);
        const int j = tile_n + wc * 32 + y * 16 + (lane & 15);
        if (i < g.M && j < g.N) {
          if (g.ksplit > 1) {
            g.part[((int64_t)blockIdx.z * g.M + i) * g.N + j] = acc[x][y][t];
            continue;
          }
          const int64_t o = out_index(g, i, j);
          double v = g.alpha * acc[x][y][t];
          if (g.beta != 0.0) v += g.beta * C[o];
          C[o] = v;
        }
      }
    }
  }
}

// The same product for outputs too small to fill the device with 64 x 64
// tiles: 32 x 32 tiles, operands straight from memory to the matrix cores'
// registers (lane l loads A[l % 16][k + l / 16] and B[k + l / 16][l % 16];
// what neighbouring waves share comes from the L1), no LDS and no barrier in
// the loop.  KS = 1: each wave one 16 x 16 quadrant over all of K, in the
// order of the tiled kernel (the same bits).  KS = 4: each wave the whole
// tile over every fourth 16 of K, the four sums added at the end in a fixed
// order; a wave then runs four independent chains of products.  Where k is an
// operand's unit stride (AV, BV) the k of a chunk are taken in the order
// 4 (l / 16) + q, so that a lane's four values lie together and are read as
// two 16-byte loads (1024 x 256 x 1024, both so: 30 -> 17 us; with neither the
// order k + l / 16 is kept, 16 against 25 us).
// PREC 1 (operands rounded to FP32) accumulates as gemm_lowp_kernel does: each
// chunk of 16 k in FP32 from zero, the chunks in FP64; the k of a chunk keep
// their order there.
constexpr int DM = 32;  // tile side
template <int PREC, int KS, bool AV, bool BV>
__global__ __launch_bounds__(NT, 2) void gemm_direct_kernel(GemmArgs g) {
  static_assert((KS == 1 || KS == 4) && (PREC == 0 || PREC == 1) && !(PREC == 1 && (AV || BV)), "forms");
  constexpr int R = KS == 1 ? 1 : 2;    // 16-row blocks of a wave, and 16-column blocks
  constexpr int CK = KS * 16;           // k between a wave's chunks of 16
  constexpr int DEPTH = KS == 1 ? 4 : 3;  // chunks in flight
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kq = lane >> 4;
  const int64_t bz = blockIdx.z / g.ksplit;
  const int kbeg = (g.ksplit > 1) ? (int)(blockIdx.z % g.ksplit) * g.kchunk : 0;
  const int kend = (g.ksplit > 1) ? min(g.K, kbeg + g.kchunk) : g.K;
  const int ti = blockIdx.y * DM + (KS == 1 ? (wave >> 1) * 16 : 0);
  const int tj = blockIdx.x * DM + (KS == 1 ? (wave & 1) * 16 : 0);
  const int k0 = kbeg + (KS == 1 ? 0 : 16 * wave);
  typedef double dbl2 __attribute__((ext_vector_type(2)));
  // k of a lane's value q in a chunk
  constexpr int KL = (AV || BV) ? 4 : 1, KQ = (AV || BV) ? 1 : 4;
  // rows and columns beyond the operands read the last one: no output takes them
  const double *pa[R], *pb[R];
#pragma unroll
  for (int x = 0; x < R; ++x) {
    pa[x] = g.A + bz * g.a_bs + (int64_t)min(ti + 16 * x + r16, g.M - 1) * g.a_rs + (int64_t)(k0 + KL * kq) * g.a_cs;
    pb[x] = g.B + bz * g.b_bs + (int64_t)min(tj + 16 * x + r16, g.N - 1) * g.b_cs + (int64_t)(k0 + KL * kq) * g.b_rs;
  }
  const int64_t aq = KQ * g.a_cs, bq = KQ * g.b_rs, ac = CK * g.a_cs, bc = CK * g.b_rs;
  double ra[DEPTH][R][4], rb[DEPTH][R][4];
  dbl4 acc[R][R];
#pragma unroll
  for (int x = 0; x < R; ++x)
#pragma unroll
    for (int y = 0; y < R; ++y) acc[x][y] = dbl4{0.0, 0.0, 0.0, 0.0};
  auto four = [&](const double *p, int64_t st, bool vec, double (&v)[4]) {
    if (vec) {
      const dbl2 lo = *(const dbl2 *)p, hi = *(const dbl2 *)(p + 2);
      v[0] = lo.x; v[1] = lo.y; v[2] = hi.x; v[3] = hi.y;
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = p[q * st];
    }
  };
  auto fetch = [&](int d, bool there) {  // the next whole chunk
    if (there) {
#pragma unroll
      for (int x = 0; x < R; ++x) {
        four(pa[x], aq, AV, ra[d][x]);
        four(pb[x], bq, BV, rb[d][x]);
        pa[x] += ac;
        pb[x] += bc;
      }
    }
  };
  auto multiply = [&](int d) {
    if constexpr (PREC == 0) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int x = 0; x < R; ++x)
#pragma unroll
          for (int y = 0; y < R; ++y)
            acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(ra[d][x][q], rb[d][y][q], acc[x][y], 0, 0, 0);
    } else {
#pragma unroll
      for (int x = 0; x < R; ++x)
#pragma unroll
        for (int y = 0; y < R; ++y) {
          flt4 c = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int q = 0; q < 4; ++q)
            c = __builtin_amdgcn_mfma_f32_16x16x4f32((float)ra[d][x][q], (float)rb[d][y][q], c, 0, 0, 0);
#pragma unroll
          for (int t = 0; t < 4; ++t) acc[x][y][t] += (double)c[t];
        }
    }
  };
  // row of accumulator register t in its 16 x 16 block
  auto arow = [&](int t) { return PREC == 0 ? 4 * t + kq : 4 * kq + t; };
  // this wave's whole chunks, then at most one short one
  const int mine = kend - k0;
  const int whole = mine >= 16 ? (mine - 16) / CK + 1 : 0, tail = mine - whole * CK;
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) fetch(d, d < whole);
  for (int c = 0; c < whole; c += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      if (c + d < whole) {
        multiply(d);
        fetch(d, c + d + DEPTH < whole);
      }
    }
  }
  if (tail > 0) {
#pragma unroll
    for (int x = 0; x < R; ++x)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool in = KQ * q + KL * kq < tail;
        ra[0][x][q] = in ? pa[x][q * aq] : 0.0;
        rb[0][x][q] = in ? pb[x][q * bq] : 0.0;
      }
    multiply(0);
  }
  double *C = g.C + bz * g.c_bs;
  auto put = [&](int i, int j, double v) {
    if (i >= g.M || j >= g.N) return;
    if (g.ksplit > 1) {
      g.part[((int64_t)blockIdx.z * g.M + i) * g.N + j] = v;
      return;
    }
    const int64_t o = out_index(g, i, j);
    v *= g.alpha;
    if (g.beta != 0.0) v += g.beta * C[o];
    C[o] = v;
  };
  if constexpr (KS == 1) {
#pragma unroll
    for (int t = 0; t < 4; ++t) put(ti + arow(t), tj + r16, acc[0][0][t]);
  } else {
    __shared__ double red[4][DM][DM + 1];
#pragma unroll
    for (int x = 0; x < R; ++x)
#pragma unroll
      for (int y = 0; y < R; ++y)
#pragma unroll
        for (int t = 0; t < 4; ++t) red[wave][16 * x + arow(t)][16 * y + r16] = acc[x][y][t];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < DM * DM / NT; ++q) {
      const int e = tid + q * NT, i = e / DM, j = e % DM;
      put(ti + i, tj + j, (red[0][i][j] + red[1][i][j]) + (red[2][i][j] + red[3][i][j]));
    }
  }
}

// Sum of the K slices of a split product, slice 0 first, then the epilogue
// of the unsplit kernel (alpha, beta, split-stride output).
__global__ __launch_bounds__(256) void gemm_splitk_reduce_kernel(GemmArgs g) {
  const int64_t mn = (int64_t)g.M * g.N;
  const int64_t total = mn * g.batch;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t b = e / mn, r = e % mn;
    const double *p = g.part + b * g.ksplit * mn + r;
    double sum = 0.0;
    for (int s = 0; s < g.ksplit; ++s) sum += p[s * mn];
    const int i = (int)(r / g.N), j = (int)(r % g.N);
    double *C = g.C + b * g.c_bs;
    const int64_t o = out_index(g, i, j);
    double v = g.alpha * sum;
    if (g.beta != 0.0) v += g.beta * C[o];
    C[o] = v;
  }
}

// ------------------------------------------------------------------ reduced-precision operands
typedef short shr4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ short bf16_bits(float x) {
  __bf16 h = (__bf16)x;  // round to nearest even
  return __builtin_bit_cast(short, h);
}
__device__ __forceinline__ float bf16_value(short b) { return (float)__builtin_bit_cast(__bf16, b); }

// The same tiling with operands rounded to FP32 or BF16 in LDS.  The matrix
// cores accumulate each 16-deep k-tile in FP32, starting from zero; the
// tile's partial sums are then added to FP64 accumulators, so that FP32
// rounding acts on 16-term partials only, not on running sums over all of K
// (with K up to the bond dimension, FP32 running sums lose about sqrt(K)
// units of 2^-24, which over the N(N-1)/2 swaps of a product at bond 1024
// added up to 3e-6).  PREC: 1 = FP32 (16x16x4 f32 MFMA, 4 k per step), 2 = BF16
// (16x16x16 bf16 MFMA, 16 k per step), 3 = BF16 x 3: x = hi + mid + lo with
// each term BF16, and A B ~ hi hi + hi mid + mid hi + hi lo + mid mid + lo hi
// (the six terms above 2^-24 relative).  Operand layouts: f32 as for f64
// (lane l: A[l%16][l/16], B[l/16][l%16]); bf16 lane l: A[l%16][4(l/16)+j],
// B[4(l/16)+j][l%16], j < 4.  Accumulator register t of lane l holds
// D[4(l/16) + t][l%16] for both (checked on gfx950 by the GEMM tests).
template <int PREC>
__global__ __launch_bounds__(NT, 2) void gemm_lowp_kernel(GemmArgs g) {
  constexpr int NS = (PREC == 3) ? 3 : 1;  // BF16 terms per operand
  __shared__ float As[NS][BK][BM + 1];
  __shared__ float Bs[NS][BK][BN + 1];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1;
  const int tile_m = blockIdx.y * BM;
  const int tile_n = blockIdx.x * BN;
  const int64_t bz = blockIdx.z / g.ksplit;
  const int kbeg = (g.ksplit > 1) ? (int)(blockIdx.z % g.ksplit) * g.kchunk : 0;
  const int kend = (g.ksplit > 1) ? min(g.K, kbeg + g.kchunk) : g.K;
  // Rounded terms of one operand value: FP32, one BF16, or three BF16.
  auto put = [&](float (*dst)[BK][BM + 1], int k, int i, double x) {
    if (PREC == 1) {
      dst[0][k][i] = (float)x;
    } else {
      const float f = (float)x;
      const float hi = bf16_value(bf16_bits(f));
      dst[0][k][i] = hi;
      if (PREC == 3) {
        const float r = (float)(x - (double)hi);
        const float mid = bf16_value(bf16_bits(r));
        dst[1][k][i] = mid;
        dst[2][k][i] = bf16_value(bf16_bits((float)(x - (double)hi - (double)mid)));
      }
    }
  };

  flt4 acc[2][2];
  dbl4 acc64[2][2];
  for (int x = 0; x < 2; ++x)
    for (int y = 0; y < 2; ++y) acc64[x][y] = dbl4{0.0, 0.0, 0.0, 0.0};

  TileLoad la(g.A + bz * g.a_bs, g.a_rs, g.a_cs, g.a_cs == 1, tile_m, g.M, kbeg);
  TileLoad lb(g.B + bz * g.b_bs, g.b_cs, g.b_rs, g.b_cs != 1, tile_n, g.N, kbeg);
  double ra[TileLoad::E], rb[TileLoad::E];
  auto fetch = [&](int left) {
    if (left >= BK) {
      la.fetch(ra);
      lb.fetch(rb);
    } else {
      la.fetch_tail(ra, left);
      lb.fetch_tail(rb, left);
    }
  };
  if (kbeg < kend) fetch(kend - kbeg);
  for (int k0 = kbeg; k0 < kend; k0 += BK) {
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y) acc[x][y] = flt4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int q = 0; q < TileLoad::E; ++q) {
      put(As, la.k(q), la.row(q), ra[q]);
      put(Bs, lb.k(q), lb.row(q), rb[q]);
    }
    __syncthreads();
    if (k0 + BK < kend) fetch(kend - k0 - BK);
    if (PREC == 1) {
#pragma unroll
      for (int kk = 0; kk < BK; kk += 4) {
        const int kr = kk + (lane >> 4);
        const float a0 = As[0][kr][wr * 32 + (lane & 15)], a1 = As[0][kr][wr * 32 + 16 + (lane & 15)];
        const float b0 = Bs[0][kr][wc * 32 + (lane & 15)], b1 = Bs[0][kr][wc * 32 + 16 + (lane & 15)];
        acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b0, acc[0][0], 0, 0, 0);
        acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b1, acc[0][1], 0, 0, 0);
        acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b0, acc[1][0], 0, 0, 0);
        acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b1, acc[1][1], 0, 0, 0);
      }
    } else {
      // one 16-deep step: lane l takes k = 4 (l/16) + j, j < 4
      shr4 a[NS][2], b[NS][2];
#pragma unroll
      for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int kr = 4 * (lane >> 4) + j;
          a[s][0][j] = bf16_bits(As[s][kr][wr * 32 + (lane & 15)]);
          a[s][1][j] = bf16_bits(As[s][kr][wr * 32 + 16 + (lane & 15)]);
          b[s][0][j] = bf16_bits(Bs[s][kr][wc * 32 + (lane & 15)]);
          b[s][1][j] = bf16_bits(Bs[s][kr][wc * 32 + 16 + (lane & 15)]);
        }
      // term pairs (sa, sb) with sa + sb <= 2: hi hi, hi mid, mid hi, hi lo, mid mid, lo hi
#pragma unroll
      for (int sa = 0; sa < NS; ++sa)
#pragma unroll
        for (int sb = 0; sb < NS; ++sb) {
          if (sa + sb > 2) continue;
#pragma unroll
          for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y)
              acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[sa][x], b[sb][y], acc[x][y], 0, 0, 0);
        }
    }
    // this k-tile's FP32 partial sums into the FP64 accumulators
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc64[x][y][t] += (double)acc[x][y][t];
    __syncthreads();
  }

  double *C = g.C + bz * g.c_bs;
#pragma unroll
  for (int x = 0; x < 2; ++x) {
#pragma unroll
    for (int y = 0; y < 2; ++y) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int i = tile_m + wr * 32 + x * 16 + 4 * (lane >> 4) + t;
        const int j = tile_n + wc * 32 + y * 16 + (lane & 15);
        if (i < g.M && j < g.N) {
          if (g.ksplit > 1) {
            g.part[((int64_t)blockIdx.z * g.M + i) * g.N + j] = acc64[x][y][t];
            continue;
          }
          const int64_t o = out_index(g, i, j);
          double v = g.alpha * acc64[x][y][t];
          if (g.beta != 0.0) v += g.beta * C[o];
          C[o] = v;
        }
      }
    }
  }
}

GemmArgs gemm_rowmajor(int M, int N, int K, const double *A, int64_t lda, const double *B,
                       int64_t ldb, double *C, int64_t ldc) {
  GemmArgs g;
  g.M = M; g.N = N; g.K = K; g.batch = 1;
  g.A = A; g.a_rs = lda; g.a_cs = 1;
  g.B = B; g.b_rs = ldb; g.b_cs = 1;
  g.C = C; g.c_rs1 = ldc; g.c_cs1 = 1;
  return g;
}

hipError_t launch_gemm(const GemmArgs &g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return hipSuccess;
  if (g.K <= 0) {
    // Empty inner dimension: C = beta * C.  Never happens on the TTM path
    // (every bond is >= 1); rejected rather than special-cased.
    return hipErrorInvalidValue;
  }
  GemmArgs h = g;
  h.ksplit = 1;
  h.kchunk = 0;
  const int64_t tiles = (int64_t)((g.N + BN - 1) / BN) * ((g.M + BM - 1) / BM) * g.batch;
  const int64_t outs = (int64_t)g.M * g.N * g.batch;
  // FP64 and FP32 outputs of few tiles take the direct kernel: with K split
  // over the waves of a workgroup from kDirectK on, in the tiled kernel's order
  // below (a product that short gains nothing from the split, and its bits
  // stay those of the tiled kernel).  Not where scratch lets the tiled kernel
  // split a large product over workgroups: its tiles read each operand half as
  // often.  Measured, direct and split: 1024 x 256 x 1024 18.7 and 21.6 us,
  // 256 x 256 x 1024 10.7 and 16.2, 4096 x 128 x 1024 36.3 and 32.2, 2048 x 512 x
  // 2048 115 and 83; without scratch 512 x 64 x 4096 52 against 217 unsplit,
  // 1024^3 (256 tiles) 60 and 61.
  const int64_t small = (int64_t)((g.N + DM - 1) / DM) * ((g.M + DM - 1) / DM) * g.batch;
  const bool narrow = (g.prec == GEMM_F64 || g.prec == GEMM_F32) && tiles < 256;
  const bool large = g.part && 2.0 * (double)outs * g.K >= 0x1p30;
  const bool deep = narrow && g.K > kDirectK && !large;
  const bool shallow = narrow && g.K <= kDirectK;
  // Split K over workgroups only when the output tiles leave the device
  // under-filled, and with at least 4 k-steps per slice.
  if (deep ? (g.part && small < 128) : (g.part && tiles < kSplitTarget && g.K >= 8 * BK)) {
    const int64_t slice = deep ? 256 : 4 * BK;
    int64_t ks = std::min<int64_t>((kSplitTarget + (deep ? small : tiles) - 1) / (deep ? small : tiles), g.K / slice);
    ks = std::min<int64_t>(ks, g.part_doubles / outs);
    ks = std::min<int64_t>(ks, 65535 / g.batch);
    if (ks > 1) {
      const int round = deep ? 4 * BK : BK;
      const int kchunk = (int)(((g.K + ks - 1) / ks + round - 1) / round * round);
      h.kchunk = kchunk;
      h.ksplit = (g.K + kchunk - 1) / kchunk;
    }
  }
  if (deep || shallow) {
    dim3 grid((g.N + DM - 1) / DM, (g.M + DM - 1) / DM, g.batch * h.ksplit);
    if (grid.y > 65535u || grid.z > 65535u) return hipErrorInvalidValue;
    // 16-byte loads along k: unit stride there, and every row of every batch
    // entry on a 16-byte boundary (chunks start at multiples of 16)
    auto vec = [](const double *p, int64_t ks, int64_t rs, int64_t bs) {
      return ks == 1 && (reinterpret_cast<uintptr_t>(p) & 15) == 0 && (rs & 1) == 0 && (bs & 1) == 0;
    };
    const bool av = deep && vec(g.A, g.a_cs, g.a_rs, g.batch > 1 ? g.a_bs : 0);
    const bool bv = deep && vec(g.B, g.b_rs, g.b_cs, g.batch > 1 ? g.b_bs : 0);
    if (g.prec == GEMM_F32) {
      if (deep)
        hipLaunchKernelGGL((gemm_direct_kernel<1, 4, false, false>), grid, dim3(NT), 0, s, h);
      else
        hipLaunchKernelGGL((gemm_direct_kernel<1, 1, false, false>), grid, dim3(NT), 0, s, h);
    } else if (!deep) {
      hipLaunchKernelGGL((gemm_direct_kernel<0, 1, false, false>), grid, dim3(NT), 0, s, h);
    } else if (av && bv) {
      hipLaunchKernelGGL((gemm_direct_kernel<0, 4, true, true>), grid, dim3(NT), 0, s, h);
    } else if (av) {
      hipLaunchKernelGGL((gemm_direct_kernel<0, 4, true, false>), grid, dim3(NT), 0, s, h);
    } else if (bv) {
      hipLaunchKernelGGL((gemm_direct_kernel<0, 4, false, true>), grid, dim3(NT), 0, s, h);
    } else {
      hipLaunchKernelGGL((gemm_direct_kernel<0, 4, false, false>), grid, dim3(NT), 0, s, h);
    }
    if (h.ksplit > 1) {
      const int64_t blocks = std::min<int64_t>((outs + 255) / 256, 4096);
      hipLaunchKernelGGL(gemm_splitk_reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, s, h);
    }
    return hipGetLastError();
  }
  dim3 grid((g.N + BN - 1) / BN, (g.M + BM - 1) / BM, g.batch * h.ksplit);
  if (grid.y > 65535u || grid.z > 65535u) return hipErrorInvalidValue;
  if (h.ksplit > 1) {
    switch (g.prec) {
      case GEMM_F64: hipLaunchKernelGGL(gemm_f64_kernel, grid, dim3(NT), 0, s, h); break;
      case GEMM_F32: hipLaunchKernelGGL(gemm_lowp_kernel<1>, grid, dim3(NT), 0, s, h); break;
      case GEMM_BF16: hipLaunchKernelGGL(gemm_lowp_kernel<2>, grid, dim3(NT), 0, s, h); break;
      case GEMM_BF16X3: hipLaunchKernelGGL(gemm_lowp_kernel<3>, grid, dim3(NT), 0, s, h); break;
      default: return hipErrorInvalidValue;
    }
    const int64_t blocks = std::min<int64_t>((outs + 255) / 256, 4096);
    hipLaunchKernelGGL(gemm_splitk_reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, s, h);
    return hipGetLastError();
  }
  switch (g.prec) {
    case GEMM_F64: hipLaunchKernelGGL(gemm_f64_kernel, grid, dim3(NT), 0, s, g); break;
    case GEMM_F32: hipLaunchKernelGGL(gemm_lowp_kernel<1>, grid, dim3(NT), 0, s, g); break;
    case GEMM_BF16: hipLaunchKernelGGL(gemm_lowp_kernel<2>, grid, dim3(NT), 0, s, g); break;
    case GEMM_BF16X3: hipLaunchKernelGGL(gemm_lowp_kernel<3>, grid, dim3(NT), 0, s, g); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace ttm
