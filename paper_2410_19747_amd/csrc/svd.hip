// Truncated SVD driver for the swap and rounding steps: column ordering,
// two Householder QRs as preconditioner, one-sided Jacobi on R2^T, rank rule
// and write-out (the steps are listed with svd_oside in ttm_internal.h).
#include <math.h>
#include <stdio.h>

#include <algorithm>

#include "ttm_internal.h"

namespace ttm {
namespace {
constexpr double kUnitRoundoff = 2.220446049250313e-16;
constexpr int kPanel = 16;  // QR panel width (T factors of 16 x 16 per panel)

size_t r32(size_t n) { return (n + 31) & ~(size_t)31; }

struct SvdBufs {
  double *Xt = nullptr;    // no x np: X = Y^T; later R1^T (np x k), then U_r (no x r)
  double *S = nullptr;     // no x np: ordered copy of X, factored in place (Q1, R1)
  double *qr = nullptr;    // QR scratch (both factorisations)
  double *Tall = nullptr;  // T factors of the first QR
  double *xnorm = nullptr; // np column norms of X
  int *perm1 = nullptr;    // np: ordered position -> column of X
  JacobiBufs jb;
};

size_t qr_ws(const SvdPlan &p) {
  return std::max({qr_inplace_scratch_doubles(p.no, p.np), qr_inplace_scratch_doubles(p.np, p.k),
                   qr_apply_q_scratch_doubles(p.no, p.k)});
}

SvdBufs carve(const SvdPlan &p, double *base) {
  SvdBufs b;
  double *q = base;
  auto adv = [&](size_t nd) {
    double *x = q;
    q += r32(nd);
    return x;
  };
  const JacobiPlan &jp = p.jp;
  b.Xt = adv((size_t)p.np * p.no);
  b.S = adv((size_t)p.np * p.no);
  b.qr = adv(qr_ws(p));
  b.Tall = adv((size_t)((p.k + kPanel - 1) / kPanel) * kPanel * kPanel);
  b.xnorm = adv((size_t)p.np);
  b.perm1 = reinterpret_cast<int *>(adv((size_t)p.np));
  b.jb.W = adv((size_t)jp.L * jp.ncp);
  b.jb.Wt = adv((size_t)jp.L * jp.ncp);
  b.jb.part = adv((size_t)jp.pairs * jp.gsw * 4 * jp.bw * jp.bw);
  b.jb.conv = adv((size_t)jp.rounds * jp.pairs);
  b.jb.qbuf = adv((size_t)jp.pairs * 4 * jp.bw * jp.bw);
  b.jb.flag = reinterpret_cast<int *>(adv((size_t)jp.pairs));
  b.jb.sigma = adv((size_t)jp.ncp);
  b.jb.perm = reinterpret_cast<int *>(adv((size_t)jp.ncp));
  b.jb.result = adv(8);
  return b;
}

__global__ void sorted_sigma_kernel(const double *__restrict__ sigma, const int *__restrict__ perm, int n,
                                    double *__restrict__ out) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) out[t] = sigma[perm[t]];
}
// Jacobi sweeps on b.W until its columns are orthogonal (np, no: the sides
// of the matrix whose SVD this is, for messages).  False with out.err set on
// a failure; out.sweeps counts.
// With near set (columns near orthogonal from the start) NEIGHBOUR_PASSES
// passes over neighbouring blocks go first: what such columns still share
// lies between close singular values, next to each other once sorted.  Six
// rounds then do most of two sweeps' work (nblk - 1 rounds each): 75 to 90
// rounds become 51 on 256 columns of a turbulence product's swaps, 35 become
// 25 on 128, with two passes 54 and 30, with four 53 and 27.  On the
// triangular factor of a whole matrix, whose columns are far from orthogonal,
// they save nothing (341 and 316 to 322 rounds at 512 columns, 150 and 147
// to 156 at 256), so svd_oside does not ask for them.
constexpr int NEIGHBOUR_PASSES = 3;
bool jacobi_sweeps(const JacobiPlan &jp, JacobiBufs &b, int max_sweeps, int np, int no, SvdResult &out, hipStream_t s,
                   KernelTimer *timer, int trace, bool near = false) {
  auto ok = [&](hipError_t e) {
    if (e != hipSuccess) {
      out.err = TTM_EHIP;
      char what[96];
      snprintf(what, sizeof(what), "the Jacobi sweeps of a %d x %d matrix", np, no);
      note_hip_error(e, what);
      if (trace) fprintf(stderr, "[ttm] HIP error %s (%s) in %s\n", hipGetErrorName(e), hipGetErrorString(e), what);
      return false;
    }
    return true;
  };
  auto sync = [&]() {
    if (!ok(hipStreamSynchronize(s))) return false;
    if (timer && timer->on) timer->collect();
    return true;
  };
  // the solve kernel's own arithmetic per pair: the sum of gsw partial Grams,
  // B2 - 1 rotation steps (6 flops per entry of G and Q), and two B2^3 products
  // of the re-orthogonalisation
  const double b2 = 2.0 * jp.bw;
  const double per_pair = jp.gsw * b2 * b2 + 6.0 * b2 * b2 * (b2 - 1.0) + 4.0 * b2 * b2 * b2;
  const double tol = sqrt((double)std::max(jp.L, 1)) * kUnitRoundoff;
  double prev = INFINITY;
  bool conv = false;
  double res[8];
  if (near) {
    {
      Timed tm(timer, KC_JAC_OTHER, s);
      if (!ok(launch_jacobi_sort_columns(jp, b, s))) return false;
    }
    if (!ok(launch_jacobi_neighbours(jp, b, NEIGHBOUR_PASSES, tol, s, timer))) return false;
    out.solve_flops += (double)NEIGHBOUR_PASSES * (2 * jp.pairs - 1) * per_pair;
  }
  for (int sw = 0; sw < max_sweeps; ++sw) {
    {
      Timed tm(timer, KC_JAC_OTHER, s);
      if (!ok(launch_jacobi_sort_columns(jp, b, s))) return false;
    }
    if (!ok(launch_jacobi_sweep(jp, b, tol, s, timer))) return false;
    ++out.sweeps;
    out.solve_flops += (double)jp.rounds * jp.pairs * per_pair;
    if (!ok(hipMemcpyAsync(res, b.result, sizeof(res), hipMemcpyDeviceToHost, s))) return false;
    if (!sync()) return false;
    const double off = res[3];
    if (trace >= 2) fprintf(stderr, "[ttm]   jacobi %dx%d sweep %d off=%.3e tol=%.3e\n", jp.L, jp.nc, sw, off, tol);
    if (!(off == off)) break;  // NaN
    if (off <= tol) {
      conv = true;
      break;
    }
    // Cyclic Jacobi converges quadratically at the end: after a sweep whose
    // largest scaled off-diagonal was off, what remains is of order off^2
    // (measured here: 3.6e-4 -> 7.9e-9 -> at the tolerance).  Once off^2 is
    // a hundredth of the tolerance the next sweep's rotations are below the
    // rounding level, so it is not run.
    if (off * off <= 0.01 * tol) {
      conv = true;
      break;
    }
    // stagnation at the rounding floor
    if (off < 1e3 * tol && off > 0.5 * prev) {
      conv = true;
      break;
    }
    prev = off;
  }
  if (!conv) {
    out.err = TTM_ENOCONV;
    set_last_error("one-sided Jacobi on the %d x %d factor of a %d x %d SVD did not converge in %d sweeps",
                   jp.L, jp.nc, np, no, out.sweeps);
    if (trace) fprintf(stderr, "[ttm] jacobi %dx%d did not converge\n", jp.L, jp.nc);
    return false;
  }
  return true;
}
}  // namespace

SvdPlan svd_plan(int np, int no, int force_bw) {
  SvdPlan p;
  p.np = np;
  p.no = no;
  p.k = std::min(np, no);
  // One workgroup up to 128 columns, the most that its tile holds: faster
  // than the block path below at every size measured (64 x 64: 367 against
  // 988 us, 128 x 128: 1261 against 2168, see kernels_svd_small.hip).
  p.small = force_bw == 0 && p.k <= kSvdSmallSide;
  p.jp = jacobi_plan(p.k, p.k, force_bw);
  return p;
}

size_t svd_ws_doubles(const SvdPlan &p) {
  const JacobiPlan &jp = p.jp;
  size_t n = 0;
  n += 2 * r32((size_t)p.np * p.no);
  n += r32(qr_ws(p));
  n += r32((size_t)((p.k + kPanel - 1) / kPanel) * kPanel * kPanel);
  n += 2 * r32((size_t)p.np);
  n += 2 * r32((size_t)jp.L * jp.ncp);
  n += r32((size_t)jp.pairs * jp.gsw * 4 * jp.bw * jp.bw);
  n += r32((size_t)jp.rounds * jp.pairs);
  n += r32((size_t)jp.pairs * 4 * jp.bw * jp.bw);
  n += r32((size_t)jp.pairs);
  n += 2 * r32((size_t)jp.ncp);
  n += r32(8);
  return n;
}

SvdResult svd_oside(const SvdPlan &p, const double *Y, double eps, int cap, int forced, int max_sweeps,
                    double *u, int u_layout, double *sigma_out, double *ws, hipStream_t s,
                    KernelTimer *timer, int trace, SvdAll *all, const double *full_total) {
  SvdResult out;
  SvdBufs b = carve(p, ws);
  const JacobiPlan &jp = p.jp;
  auto ok = [&](hipError_t e) {
    if (e != hipSuccess) {
      out.err = TTM_EHIP;
      char what[96];
      snprintf(what, sizeof(what), "the truncated SVD of a %d x %d matrix", p.np, p.no);
      note_hip_error(e, what);
      if (trace) fprintf(stderr, "[ttm] HIP error %s (%s) in %s\n", hipGetErrorName(e), hipGetErrorString(e), what);
      return false;
    }
    return true;
  };
  auto sync = [&]() {
    if (!ok(hipStreamSynchronize(s))) return false;
    if (timer && timer->on) timer->collect();
    return true;
  };
  if (p.small) {
    SvdSmall q;
    q.np = p.np; q.no = p.no; q.k = p.k;
    q.eps = eps; q.cap = cap; q.forced = forced; q.max_sweeps = max_sweeps;
    q.full_total = full_total;
    q.result = b.jb.result;
    q.sig = all ? all->sigma : sigma_out;
    q.mode = std::max(p.np, p.no) <= kSvdSmallSide ? SMALL_Y : (p.np > p.no ? SMALL_RT : SMALL_RTQ);
    if (q.mode == SMALL_Y) {
      q.src = Y;
      q.ld = p.np;
    } else {
      // a QR by panels first: of Y (its columns ordered) when the
      // orthonormal side is the short one, else of X = Y^T with its
      // reflectors kept
      const bool tall = q.mode == SMALL_RT;
      const int rows = tall ? p.np : p.no, cols = tall ? p.no : p.np;
      const double *M = tall ? Y : b.Xt;
      {
        Timed tm(timer, KC_JAC_OTHER, s);
        if (!tall && !ok(launch_transpose(b.Xt, Y, p.no, p.np, s))) return out;
        if (!ok(launch_column_norms(M, rows, cols, b.xnorm, s))) return out;
        if (!ok(launch_sort_desc(b.xnorm, cols, b.perm1, s))) return out;
        if (!ok(launch_gather_columns(M, b.perm1, rows, cols, b.S, s))) return out;
      }
      Timed tm(timer, KC_QR, s);
      if (!ok(launch_qr_inplace(b.S, rows, cols, b.qr, nullptr, tall ? nullptr : b.Tall, s))) return out;
      q.src = b.S;
      q.ld = rows;
      if (tall) q.rowperm = b.perm1;
    }
    if (q.mode == SMALL_RTQ) {
      q.uall = b.jb.W;  // U_W, k x kg; Q1 is applied below
      q.uall_ld = p.k;
    } else {
      q.u = u;
      q.u_os = (u_layout == SVD_U_T) ? 1 : 0;
      q.u_ts = (u_layout == SVD_U_T) ? p.no : 1;
      if (all) {
        q.uall = all->u;
        q.uall_ld = p.no;
      }
    }
    {
      Timed tm(timer, KC_JAC_OTHER, s);
      if (!ok(launch_svd_small(q, s))) return out;
    }
    double res[8];
    if (!ok(hipMemcpyAsync(res, b.jb.result, sizeof(res), hipMemcpyDeviceToHost, s))) return out;
    if (!sync()) return out;
    // Not within max_sweeps sweeps of its own: the block method, whose sweeps
    // visit the pairs in another order, may need one less.
    if (res[7] > 0.0) {
      out.sweeps = (int)res[7];
      if (res[4] != 0.0) {
        out.err = TTM_ENONFINITE;
        set_last_error("the singular values of a %d x %d SVD are not finite", p.np, p.no);
        return out;
      }
      out.rank = (int)res[0];
      out.disc = res[1];
      out.total = res[2];
      const int r = out.rank, kg = std::max(r, std::min(p.k, (int)res[6]));
      if (all) all->kg = kg;
      if (q.mode == SMALL_RTQ) {
        double *ucm = (u_layout == SVD_U_T) ? u : b.Xt;
        double *full = all ? all->u : ucm;
        const int nc = all ? kg : r;
        {
          Timed tm(timer, KC_JAC_OTHER, s);
          if (!ok(launch_embed_rows(full, b.jb.W, p.k, p.no, nc, s))) return out;
        }
        {
          Timed tm(timer, KC_QR, s);
          if (!ok(launch_apply_q(b.S, p.no, p.k, b.Tall, full, nc, b.qr, s))) return out;
        }
        Timed tm(timer, KC_JAC_OTHER, s);
        if (all && !ok(launch_copy(ucm, all->u, (int64_t)p.no * r, s))) return out;
        if (u_layout == SVD_U && !ok(launch_transpose(u, ucm, r, p.no, s))) return out;
      }
      if (all && sigma_out && !ok(launch_copy(sigma_out, all->sigma, p.k, s))) return out;
      if (trace)
        fprintf(stderr, "[ttm] svd %dx%d sweeps=%d rank=%d disc=%.3e total=%.3e\n", p.np, p.no, out.sweeps, out.rank,
                out.disc, out.total);
      return out;
    }
  }
  // 1. X = Y^T, its columns in decreasing norm order, ||Y||_F^2
  {
    Timed tm(timer, KC_JAC_OTHER, s);
    if (!ok(launch_transpose(b.Xt, Y, p.no, p.np, s))) return out;
    if (!ok(launch_column_norms(b.Xt, p.no, p.np, b.xnorm, s))) return out;
    if (!ok(launch_sort_desc(b.xnorm, p.np, b.perm1, s))) return out;
    if (!ok(launch_gather_columns(b.Xt, b.perm1, p.no, p.np, b.S, s))) return out;
    if (!ok(launch_frob_from_norms(b.xnorm, p.np, b.jb.result, s))) return out;
  }
  // 2. X P = Q1 R1, then R1^T = Q2 R2
  {
    Timed tm(timer, KC_QR, s);
    // No block column pivoting: it saves a few sweeps (about 2% at every
    // size measured) but its column moves cost more than they save once the
    // columns are presorted by norm.
    if (!ok(launch_qr_inplace(b.S, p.no, p.np, b.qr, nullptr, b.Tall, s))) return out;
  }
  {
    Timed tm(timer, KC_JAC_OTHER, s);
    if (!ok(launch_rt_from_qr(b.S, p.no, p.np, p.k, p.k, b.Xt, s))) return out;
  }
  {
    Timed tm(timer, KC_QR, s);
    if (!ok(launch_qr_inplace(b.Xt, p.np, p.k, b.qr, nullptr, nullptr, s))) return out;
  }
  {
    Timed tm(timer, KC_JAC_OTHER, s);
    if (!ok(launch_rt_from_qr(b.Xt, p.np, p.k, p.k, jp.ncp, b.jb.W, s))) return out;
  }
  // 3. Jacobi sweeps until the columns of W are orthogonal
  if (!jacobi_sweeps(jp, b.jb, max_sweeps, p.np, p.no, out, s, timer, trace)) return out;
  // 4. singular values and the rank rule
  {
    Timed tm(timer, KC_JAC_OTHER, s);
    if (!ok(launch_jacobi_finish(jp, b.jb, eps, cap, forced, s, full_total))) return out;
  }
  double res[8];
  if (!ok(hipMemcpyAsync(res, b.jb.result, sizeof(res), hipMemcpyDeviceToHost, s))) return out;
  if (!sync()) return out;
  if (res[4] != 0.0) {
    out.err = TTM_ENONFINITE;
    set_last_error("the singular values of a %d x %d SVD are not finite", p.np, p.no);
    return out;
  }
  out.rank = (int)res[0];
  out.disc = res[1];
  out.total = res[2];
  // 5. U_r = Q1 [U_W,r; 0] (no x r, column-major), then the caller's layout.
  // U_r^T row-major is that column-major matrix, so SVD_U_T is formed in u.
  const int r = out.rank;
  double *ucm = (u_layout == SVD_U_T) ? u : b.Xt;
  if (all) {
    // every resolved vector; U_r is their leading r columns
    const int kg = std::max(r, std::min(p.k, (int)res[6]));
    all->kg = kg;
    {
      Timed tm(timer, KC_JAC_OTHER, s);
      if (p.k < p.no && !ok(launch_fill(all->u, 0.0, (int64_t)p.no * kg, s))) return out;
      if (!ok(launch_jacobi_write_u(jp, b.jb, nullptr, kg, all->u, 1, p.no, s))) return out;
    }
    {
      Timed tm(timer, KC_QR, s);
      if (!ok(launch_apply_q(b.S, p.no, p.k, b.Tall, all->u, kg, b.qr, s))) return out;
    }
    {
      Timed tm(timer, KC_JAC_OTHER, s);
      if (!ok(launch_copy(ucm, all->u, (int64_t)p.no * r, s))) return out;
      hipLaunchKernelGGL(sorted_sigma_kernel, dim3((p.k + 255) / 256), dim3(256), 0, s, b.jb.sigma, b.jb.perm,
                         p.k, all->sigma);
      if (!ok(hipGetLastError())) return out;
    }
  } else {
    {
      Timed tm(timer, KC_JAC_OTHER, s);
      if (p.k < p.no && !ok(launch_fill(ucm, 0.0, (int64_t)p.no * r, s))) return out;
      if (!ok(launch_jacobi_write_u(jp, b.jb, nullptr, r, ucm, 1, p.no, s))) return out;
    }
    {
      Timed tm(timer, KC_QR, s);
      if (!ok(launch_apply_q(b.S, p.no, p.k, b.Tall, ucm, r, b.qr, s))) return out;
    }
  }
  {
    Timed tm(timer, KC_JAC_OTHER, s);
    if (u_layout == SVD_U && !ok(launch_transpose(u, ucm, r, p.no, s))) return out;
    if (sigma_out) {
      hipLaunchKernelGGL(sorted_sigma_kernel, dim3((p.k + 255) / 256), dim3(256), 0, s, b.jb.sigma, b.jb.perm,
                         p.k, sigma_out);
      if (!ok(hipGetLastError())) return out;
    }
  }
  if (trace)
    fprintf(stderr, "[ttm] svd %dx%d sweeps=%d rank=%d disc=%.3e total=%.3e\n", p.np, p.no, out.sweeps,
            out.rank, out.disc, out.total);
  return out;
}

int svd_columns_capacity(int n, int l) { return l <= kColumnsSmall ? l : jacobi_plan(n, l).ncp; }

size_t svd_columns_ws_doubles(int n, int l) {
  if (l <= kColumnsSmall)
    return r32(std::max(qr_inplace_scratch_doubles(n, l), qr_apply_q_scratch_doubles(n, l))) +
           r32((size_t)((l + kPanel - 1) / kPanel) * kPanel * kPanel) + r32((size_t)l * l) + r32(8);
  const JacobiPlan jp = jacobi_plan(n, l);
  return r32((size_t)jp.pairs * jp.gsw * 4 * jp.bw * jp.bw) + r32((size_t)jp.rounds * jp.pairs) +
         r32((size_t)jp.pairs * 4 * jp.bw * jp.bw) + r32((size_t)jp.pairs) + 2 * r32((size_t)jp.ncp) + r32(8);
}

SvdResult svd_columns(double *C, double *spare, int n, int l, double eps, int cap, int max_sweeps, double *u,
                      double *sigma, double *ws, hipStream_t s, KernelTimer *timer, int trace,
                      const double *full_total) {
  SvdResult out;
  double *q = ws;
  auto adv = [&](size_t nd) {
    double *x = q;
    q += r32(nd);
    return x;
  };
  auto ok = [&](hipError_t e) {
    if (e == hipSuccess) return true;
    out.err = TTM_EHIP;
    char what[96];
    snprintf(what, sizeof(what), "the SVD of %d columns of %d", l, n);
    note_hip_error(e, what);
    if (trace) fprintf(stderr, "[ttm] HIP error %s (%s) in %s\n", hipGetErrorName(e), hipGetErrorString(e), what);
    return false;
  };
  auto read = [&](double *res, const double *result) {
    if (!ok(hipMemcpyAsync(res, result, 8 * sizeof(double), hipMemcpyDeviceToHost, s))) return false;
    if (!ok(hipStreamSynchronize(s))) return false;
    if (timer && timer->on) timer->collect();
    if (res[4] != 0.0) {
      out.err = TTM_ENONFINITE;
      set_last_error("the singular values of %d columns of %d are not finite", l, n);
      return false;
    }
    out.rank = (int)res[0];
    out.disc = res[1];
    out.total = res[2];
    return true;
  };
  double res[8];
  if (l <= kColumnsSmall) {
    // C = Q1 R, Jacobi on R in one launch, U = Q1 U_R
    double *qr = adv(std::max(qr_inplace_scratch_doubles(n, l), qr_apply_q_scratch_doubles(n, l)));
    double *Tall = adv((size_t)((l + kPanel - 1) / kPanel) * kPanel * kPanel);
    double *uw = adv((size_t)l * l);
    SvdSmall a;
    a.result = adv(8);
    a.mode = SMALL_R;
    a.src = C; a.ld = n;
    a.np = l; a.no = n; a.k = l;
    a.eps = eps; a.cap = cap; a.max_sweeps = max_sweeps;
    a.full_total = full_total;
    a.uall = uw; a.uall_ld = l;
    a.sig = sigma;
    {
      Timed tm(timer, KC_QR, s);
      if (!ok(launch_qr_inplace(C, n, l, qr, nullptr, Tall, s))) return out;
    }
    {
      Timed tm(timer, KC_JAC_OTHER, s);
      if (!ok(launch_svd_small(a, s))) return out;
    }
    if (!read(res, a.result)) return out;
    out.sweeps = (int)fabs(res[7]);
    if (!(res[7] > 0.0)) {
      out.err = TTM_ENOCONV;
      set_last_error("one-sided Jacobi on %d columns of %d did not converge in %d sweeps", l, n, out.sweeps);
      return out;
    }
    {
      Timed tm(timer, KC_JAC_OTHER, s);
      if (!ok(launch_embed_rows(u, uw, l, n, out.rank, s))) return out;
    }
    Timed tm(timer, KC_QR, s);
    ok(launch_apply_q(C, n, l, Tall, u, out.rank, qr, s));
    return out;
  }
  const JacobiPlan jp = jacobi_plan(n, l);
  JacobiBufs b;
  b.W = C;
  b.Wt = spare;
  b.part = adv((size_t)jp.pairs * jp.gsw * 4 * jp.bw * jp.bw);
  b.conv = adv((size_t)jp.rounds * jp.pairs);
  b.qbuf = adv((size_t)jp.pairs * 4 * jp.bw * jp.bw);
  b.flag = reinterpret_cast<int *>(adv((size_t)jp.pairs));
  b.sigma = adv((size_t)jp.ncp);
  b.perm = reinterpret_cast<int *>(adv((size_t)jp.ncp));
  b.result = adv(8);
  {
    Timed tm(timer, KC_JAC_OTHER, s);
    if (jp.ncp > l && !ok(launch_fill(C + (int64_t)l * n, 0.0, (int64_t)(jp.ncp - l) * n, s))) return out;
    if (!ok(launch_column_norms(C, n, jp.ncp, b.sigma, s))) return out;
    if (!ok(launch_frob_from_norms(b.sigma, jp.ncp, b.result, s))) return out;
  }
  if (!jacobi_sweeps(jp, b, max_sweeps, n, l, out, s, timer, trace, true)) return out;
  {
    Timed tm(timer, KC_JAC_OTHER, s);
    if (!ok(launch_jacobi_finish(jp, b, eps, cap, 0, s, full_total))) return out;
  }
  if (!read(res, b.result)) return out;
  Timed tm(timer, KC_JAC_OTHER, s);
  if (!ok(launch_jacobi_write_u(jp, b, nullptr, out.rank, u, 1, n, s))) return out;
  hipLaunchKernelGGL(sorted_sigma_kernel, dim3((l + 255) / 256), dim3(256), 0, s, b.sigma, b.perm, l, sigma);
  ok(hipGetLastError());
  return out;
}

}  // namespace ttm
