// The BiCGSTAB recurrence of one system: its scalar steps, shared by the
// kernel that runs them between the operator stages of all systems and the
// kernel that runs whole iterations of a small system in one block.
#pragma once

#include <cmath>

#include "internal.hpp"

namespace cisor {

// STG_TR: FP64 true residual (the stop test); STG_TR0: provisional starting
// residual in the field precision, which never finishes a system with x != 0.
enum : int { STG_ALPHA = 0, STG_OMEGA = 1, STG_TR = 3, STG_TR0 = 4 };

// Residual replacement when the recurrence residual^2 has fallen below this
// fraction of its largest value since the last replacement (a drop by ~31.6x
// in norm).  Measured on the 256^2 x 60 true-phantom solves: the slowest of 60
// systems needed 443-467 iterations instead of 508-933 (the FP32 tail varies
// with rounding; the FP64 solver needs 375), at about 1 % more time per solve
// where the solves are short.
constexpr double REPLACE_DROP2 = 1e-3;

__device__ __forceinline__ cd cd_div(cd a, cd b) {
  const double den = b.x * b.x + b.y * b.y;
  return mk<cd>((a.x * b.x + a.y * b.y) / den, (a.y * b.x - a.x * b.y) / den);
}
__device__ __forceinline__ cd cd_mul(cd a, cd b) { return mk<cd>(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
__device__ __forceinline__ bool cd_ok(cd a) { return isfinite(a.x) && isfinite(a.y); }
__device__ __forceinline__ bool cd_zero(cd a) { return a.x == 0.0 && a.y == 0.0; }

__device__ __forceinline__ TxState initial_state() {
  TxState s{};
  s.status = ST_PAUSED;
  s.flags = FLAG_TR;
  s.restart = 1;
  s.rho = s.rho_prev = s.alpha = s.omega = mk<cd>(1.0, 0.0);
  s.beta = mk<cd>(0.0, 0.0);
  return s;
}

// Advance s by the scalar step `stage` from its inner products acc (at least
// as many as the stage's epilogue forms, see EPI_V, EPI_T and EPI_TR).
__device__ __forceinline__ void advance_state(TxState &s, const double *acc, int stage, double tol, int replace_every,
                                              int maxit) {
  const double tol2 = tol * tol;
  if (stage == STG_ALPHA) {
    const cd rhv = mk<cd>(acc[0], acc[1]);
    s.x_pending = 0;   // stage A has applied the last iteration's x update
    if (cd_zero(rhv) || !cd_ok(rhv)) {
      s.status = ST_PAUSED;
      s.flags = FLAG_TR;
      s.restart = 1;
    } else {
      s.alpha = cd_div(s.rho, rhv);
    }
  } else if (stage == STG_OMEGA) {
    const cd ts = mk<cd>(acc[0], acc[1]);
    const double tt = acc[2], ss = acc[3];
    const cd rs = mk<cd>(acc[4], acc[5]), rt = mk<cd>(acc[6], acc[7]);
    double rr;
    if (tt == 0.0 || !std::isfinite(tt) || !cd_ok(ts)) {
      s.omega = mk<cd>(0.0, 0.0);
      rr = ss;
    } else {
      s.omega = mk<cd>(ts.x / tt, ts.y / tt);
      rr = fmax(ss - (ts.x * ts.x + ts.y * ts.y) / tt, 0.0);   // ||s - omega t||^2
    }
    const cd wrt = cd_mul(s.omega, rt);
    const cd rho_new = mk<cd>(rs.x - wrt.x, rs.y - wrt.y);       // <rhat, s - omega t>
    s.r_fresh = 0;
    s.x_pending = 1;
    s.iters += 1;
    s.rnorm2 = rr;
    s.rmax2 = fmax(s.rmax2, rr);
    const bool conv = rr <= tol2 * s.bnorm2;
    const bool brk = cd_zero(s.omega) || cd_zero(rho_new) || !cd_ok(rho_new) || !std::isfinite(rr);
    if (!brk) {
      s.beta = cd_mul(cd_div(rho_new, s.rho), cd_div(s.alpha, s.omega));
      s.rho_prev = s.rho;
      s.rho = rho_new;
    }
    if (conv) {
      s.status = ST_PAUSED;
      s.flags = FLAG_TR;
      s.restart = brk ? 1 : 0;
    } else if (brk) {
      s.status = ST_PAUSED;
      s.flags = FLAG_TR;
      s.restart = 1;
    } else if (s.iters - s.last_tr >= replace_every || s.iters >= maxit || rr < REPLACE_DROP2 * s.rmax2) {
      s.flags = FLAG_ITER | FLAG_TR;
    }
  } else {  // STG_TR: r = b - A x has just been computed in FP64 (x up to date)
    const double rr = acc[0];
    const cd rhr = mk<cd>(acc[1], acc[2]);
    if (s.restart) s.bnorm2 = acc[3];
    s.last_tr = s.iters;
    s.rmax2 = rr;
    s.rnorm2 = rr;
    s.x_pending = 0;
    s.r_fresh = 1;
    if (s.bnorm2 == 0.0) {
      s.true_rel = 0.0;
      s.status = ST_DONE;
      s.flags = 0;
      s.zero_x = 1;
    } else if (!std::isfinite(rr)) {
      s.true_rel = rr;
      s.status = ST_FAILED;
      s.flags = 0;
    } else {
      s.true_rel = sqrt(rr / s.bnorm2);
      if (rr <= tol2 * s.bnorm2 && stage == STG_TR0) {
        s.status = ST_PAUSED;   // looks converged: confirm with the FP64 residual
        s.flags = FLAG_TR;
      } else if (rr <= tol2 * s.bnorm2) {
        s.status = ST_DONE;
        s.flags = 0;
      } else if (s.restart) {
        s.rho = rhr;
        s.rho_prev = mk<cd>(1.0, 0.0);
        s.alpha = s.omega = mk<cd>(1.0, 0.0);
        s.beta = mk<cd>(0.0, 0.0);
        s.restart = 0;
        s.status = ST_ITER;
        s.flags = FLAG_ITER;
      } else {
        // residual replacement: keep the search directions, rebase rho
        if (cd_zero(rhr) || !cd_ok(rhr)) {
          s.restart = 1;
          s.status = ST_PAUSED;
          s.flags = FLAG_TR;
        } else {
          s.beta = cd_mul(cd_div(rhr, s.rho_prev), cd_div(s.alpha, s.omega));
          s.rho = rhr;
          s.status = ST_ITER;
          s.flags = FLAG_ITER;
        }
      }
    }
  }
}

}  // namespace cisor
