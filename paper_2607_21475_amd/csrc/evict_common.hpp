// evict_common.hpp -- the allocation of eq. (2), shared by the kernels that select a unit's rows: how
// a score is read, pi of a position, and the solve for lambda.
#pragma once

#include "ebd.h"
#include "ebd_device.hpp"

namespace ebd {

// Non-finite and negative scores are read as 0 and flagged.
__device__ __forceinline__ float clean_score(float s, uint32_t &bad) {
  if (!(s >= 0.0f) || isinf(s)) {
    bad = 1u;
    return 0.0f;
  }
  return s == 0.0f ? 0.0f : s;  // -0 becomes +0 (the top-k keys are the score bits)
}

// pi of a position: 1 outside the tail, clip(lambda s, eps, 1) in it.  With lambda = +inf (no
// eviction), lambda s is +inf for s > 0 (pi = 1) and NaN for s = 0, which fmaxf drops (pi = eps).
__device__ __forceinline__ float token_pi(bool tail, float s, float lam, float eps) {
  return tail ? fminf(fmaxf(lam * s, eps), 1.0f) : 1.0f;
}

// Tail statistics of a unit: |T|, positive scores, their sum, the largest score and the smallest
// positive one.
struct TailStats {
  double n_tail, n_pos, s_sum;
  float s_max, s_minp;
};

// lambda of eq. (2) with sum_T clip(lambda s, eps, 1) = m, plus the status bits of the boundary
// cases.  `pass(lf, H, L, S, edges)` gives the unit's totals at lambda = lf: tail positions with
// lf s >= 1 (H), with lf s <= eps (L), and the sum of the scores in between (S).
// g(lambda) = H + eps L + lambda S is piecewise linear and nondecreasing: a Newton step on the
// current piece is exact once the piece is right, and the bracket [lo, hi] with
// g(lo) < m <= g(hi) guards every step (bisection when a step leaves it).
//
// The boundary cases (no tail, the literal lambda = m / sum s, the floor, no eviction): sets
// lambda and the status bits and returns true; false when lambda is interior and needs the
// iteration.
__device__ inline bool lambda_boundary(const TailStats &T, double m, float eps, int pi_mode,
                                       uint32_t &st, double &lam) {
  if (T.n_tail == 0.0) {
    lam = 0.0;
    return true;
  }
  if (pi_mode == 1) {
    if (m <= (double)eps * T.n_tail) st |= EBD_ST_BUDGET_FLOOR;
    lam = (T.s_sum > 0.0 && m > 0.0) ? m / T.s_sum : 0.0;
    return true;
  }
  if (m <= (double)eps * T.n_tail) {
    st |= EBD_ST_BUDGET_FLOOR;
    lam = 0.0;
    return true;
  }
  if (m >= T.n_pos + (double)eps * (T.n_tail - T.n_pos)) {
    st |= EBD_ST_NO_EVICTION;
    lam = INFINITY;
    return true;
  }
  return false;
}

// Where the scores of the evaluated piece lie: the smallest score of H, the largest and smallest
// of the middle, the largest tail score of L.  A lambda whose fp32 products keep every token on
// its side (monotone in s) gives a pass with exactly the same counts and sum.
struct PieceEdges {
  bool valid;  // false: not tracked by this pass
  float h_min, m_max, m_min, l_max;
  __device__ bool keeps(float lf, float eps) const {
    return valid && lf * h_min >= 1.0f && lf * m_max < 1.0f && lf * m_min > eps &&
           lf * l_max <= eps;
  }
};

// Histograms of positive scores: the bins are the fp32 bit patterns shifted right by kHistShift (the
// exponent and five mantissa bits, 32 bins per octave over every positive float).
constexpr int kHistShift = 18;
constexpr int kHistBins = 1 << (31 - kHistShift);

// The iteration for an interior lambda within the bracket [lo, hi] (g(lo) < m <= g(hi)),
// starting at cur.  pass(lf, H, L, S, edges) evaluates the piece at lf.  A Newton step that
// stays on the evaluated piece is final: the next pass would find the same piece and stop there,
// so a pass that reports the piece's edges saves that confirming pass.
template <class Pass>
__device__ double newton_lambda(double m, float eps, double lo, double hi, double cur,
                                Pass &&pass) {
  double pH = -1.0, pL = -1.0, pS = -1.0;
  bool from_newton = false;
  for (int it = 0; it < 96; ++it) {
    const float lf = (float)cur;
    double dH, dL, dS;
    PieceEdges e;
    pass(lf, dH, dL, dS, e);
    if (from_newton && dH == pH && dL == pL && dS == pS) break;  // same piece: cur is exact
    const double g = dH + (double)eps * dL + (double)lf * dS;
    if (g < m) lo = (double)lf;
    else hi = (double)lf;
    if (g == m) break;
    double nxt = dS > 0.0 ? (m - dH - (double)eps * dL) / dS : -1.0;
    from_newton = (nxt > lo && nxt < hi);
    if (!from_newton) nxt = 0.5 * (lo + hi);
    if ((float)nxt == lf || hi - lo <= 1e-9 * hi) {
      cur = from_newton ? nxt : cur;
      break;
    }
    if (from_newton && e.keeps((float)nxt, eps)) {
      cur = nxt;
      break;
    }
    pH = dH;
    pL = dL;
    pS = dS;
    cur = nxt;
  }
  return cur;
}

template <class Pass>
__device__ double solve_lambda(const TailStats &T, double m, float eps, int pi_mode, uint32_t &st,
                               Pass &&pass) {
  double lam;
  if (lambda_boundary(T, m, eps, pi_mode, st, lam)) return lam;
  const double lo = (double)eps / (double)T.s_max;
  const double hi = 1.0 / (double)T.s_minp;
  return newton_lambda(m, eps, lo, hi, fmin(fmax(m / T.s_sum, lo), hi), pass);
}

}  // namespace ebd
