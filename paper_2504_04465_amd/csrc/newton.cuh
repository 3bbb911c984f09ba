// newton.cuh -- numerical (entropy-maximising) equilibrium of the 2-D
// lattices: f_eq = rho exp(-(1 + lambda . m_i)) under the eight moment
// constraints (Eqs. exponential, G0_8mom - G3yaa_8mom); Newton with a
// Cholesky step and backtracking on ||G||_2, FP64 throughout.
//
// One evaluation (expo_sums) is bound by vector issue: it is 13 / 21 / 37
// exponentials and their weighted sums, all in FP64 at four cycles a
// wavefront instruction.  Hence
//  - the velocities are taken by reflection orbits (a, b), a, b >= 0: the
//    exponents of an orbit's (up to four) members are sums of the same four
//    terms, and its contribution to every moment needs only four
//    sign-weighted sums of its exponentials;
//  - the 22 independent moments that the residual and the Newton matrix are
//    made of are accumulated orbit by orbit, so that neither the orbit sums
//    nor a table of all S_pq is held (44 registers instead of 56 plus 26-90);
//  - every orbit is unrolled by template recursion on compile-time
//    constants.  `#pragma unroll` over the same loops was given up by the
//    compiler on D2Q37 (37 velocities x 28 moments), which then evaluated
//    the tables at run time from scratch: 15.3 ms for one step of 262 k
//    cells instead of 0.1 ms on D2Q21;
//  - the exponential is a table of 2^(j/64) and a fifth-degree polynomial.
#pragma once

#include <hip/hip_runtime.h>

#include <utility>

#include "lattice.h"
#include "ops.h"

namespace lbm {

// ---------------------------------------------------------------------------
// exponential, table-driven (Tang 1989, ACM TOMS 15, 144):
// exp(-s) = 2^n 2^(j/64) exp(r), 64 n + j = rint(-64 s / ln 2),
// |r| <= ln 2 / 128.  The Taylor polynomial of degree five leaves
// r^6 / 720 < 4e-17 relative; the argument reduction uses ln 2 / 64 in two
// parts.  The table holds each power and the relative remainder of its
// rounding, which leaves the last operation's rounding alone (without the
// remainder the multipliers' error against 80 bits grew: rms 2.8e-11 with the
// library's exponential, 5.5e-11 without, 2.7e-11 with, 90,000 states; it
// costs the D2Q21 collide 0.8 %).  15 vector instructions and one table read
// where the library's exponential takes about twice as many.
// The integer saturates at +-2^31 and the last operation scales by 2^n, so that
// arguments out of range give 0 and infinity, and the subnormal ones between
// are rounded (n clamped to the exponent range gave 1e-308 and 1e308, and n
// from the bits of the shifted sum, 32 of them, wrapped round beyond 1.5e9: a
// trial step of a diverging solve could find finite exponentials there and be
// taken; both forms take the same time).  Beyond 1e13 r is no longer small; its
// polynomial's magnitude (it may turn negative) still scales to 0 and infinity
// up to 1e77, and above that a positive s gives infinity or NaN instead of 0: a
// trial point with such an exponent is rejected.
// ---------------------------------------------------------------------------
constexpr int EXP_N = 64, EXP_TAB = 2 * EXP_N;

// 2^(j/64), correctly rounded, and what is left of it, relative
static __device__ const double exp_tab_g[EXP_TAB] = {
    0x1.0000000000000p+0, 0x0.0p+0, 0x1.02c9a3e778061p+0, -0x1.160139cd8dc5dp-56,
    0x1.059b0d3158574p+0, 0x1.cd2523567f613p-55, 0x1.0874518759bc8p+0, 0x1.0f74e61e6c861p-57,
    0x1.0b5586cf9890fp+0, 0x1.79aa65d837b6dp-54, 0x1.0e3ec32d3d1a2p+0, 0x1.ebe3d702f9cd1p-60,
    0x1.11301d0125b51p+0, -0x1.556522a2fbd0ep-54, 0x1.1429aaea92de0p+0, -0x1.1c923b9d5f416p-54,
    0x1.172b83c7d517bp+0, -0x1.01b15eaa59348p-55, 0x1.1a35beb6fcb75p+0, 0x1.b898c3f1353bfp-55,
    0x1.1d4873168b9aap+0, 0x1.aecf73e3a2f60p-54, 0x1.2063b88628cd6p+0, 0x1.a6f4144a6c38dp-55,
    0x1.2387a6e756238p+0, 0x1.68efde3a8a894p-54, 0x1.26b4565e27cddp+0, 0x1.0472b981fe7f2p-55,
    0x1.29e9df51fdee1p+0, 0x1.2f7e16d09ab31p-55, 0x1.2d285a6e4030bp+0, 0x1.b3782720c0ab4p-55,
    0x1.306fe0a31b715p+0, 0x1.34d754db0abb6p-55, 0x1.33c08b26416ffp+0, 0x1.fdd395dd3f84ap-55,
    0x1.371a7373aa9cbp+0, -0x1.24aedcc4b5068p-54, 0x1.3a7db34e59ff7p+0, -0x1.1d1e83e9436d2p-56,
    0x1.3dea64c123422p+0, 0x1.59f48a72a4c6dp-55, 0x1.4160a21f72e2ap+0, -0x1.8a78f4817895bp-58,
    0x1.44e086061892dp+0, 0x1.363ed60c2ac11p-59, 0x1.486a2b5c13cd0p+0, 0x1.ecce1daa10379p-57,
    0x1.4bfdad5362a27p+0, 0x1.690cebb7aafb0p-56, 0x1.4f9b2769d2ca7p+0, -0x1.f94340071a38ep-55,
    0x1.5342b569d4f82p+0, -0x1.8dec6bd0f385fp-56, 0x1.56f4736b527dap+0, 0x1.3350518fdd78ep-54,
    0x1.5ab07dd485429p+0, 0x1.063e1e21c5409p-54, 0x1.5e76f15ad2148p+0, 0x1.432e62b64c035p-54,
    0x1.6247eb03a5585p+0, -0x1.c33c53bef4da8p-55, 0x1.6623882552225p+0, -0x1.3cedd78565858p-54,
    0x1.6a09e667f3bcdp+0, -0x1.3b3efbf5e2228p-54, 0x1.6dfb23c651a2fp+0, -0x1.367efb86da9eep-57,
    0x1.71f75e8ec5f74p+0, -0x1.81f647e5a3ecfp-56, 0x1.75feb564267c9p+0, -0x1.619321e55e68ap-55,
    0x1.7a11473eb0187p+0, -0x1.b32dcb94da51dp-56, 0x1.7e2f336cf4e62p+0, 0x1.5ebe1abd66c55p-57,
    0x1.82589994cce13p+0, -0x1.369b6f13b3734p-54, 0x1.868d99b4492edp+0, -0x1.4d450d872576ep-54,
    0x1.8ace5422aa0dbp+0, 0x1.db72fc1f0eab4p-55, 0x1.8f1ae99157736p+0, 0x1.bf68359f35f44p-56,
    0x1.93737b0cdc5e5p+0, -0x1.da9b88b6c1e29p-58, 0x1.97d829fde4e50p+0, -0x1.2434322f4f9aap-54,
    0x1.9c49182a3f090p+0, 0x1.1affc2b91ce27p-56, 0x1.a0c667b5de565p+0, -0x1.7c50422622263p-55,
    0x1.a5503b23e255dp+0, -0x1.1bbd1d3bcbb15p-54, 0x1.a9e6b5579fdbfp+0, 0x1.469846e735ab3p-55,
    0x1.ae89f995ad3adp+0, 0x1.c1a7792cb3387p-55, 0x1.b33a2b84f15fbp+0, -0x1.5c3d956dcaebap-58,
    0x1.b7f76f2fb5e47p+0, -0x1.8d6f438ad9334p-57, 0x1.bcc1e904bc1d2p+0, 0x1.4ffd70a5fddcdp-56,
    0x1.c199bdd85529cp+0, 0x1.36eae30af0cb3p-56, 0x1.c67f12e57d14bp+0, 0x1.4e08fd10959acp-55,
    0x1.cb720dcef9069p+0, 0x1.76b2c6c921968p-57, 0x1.d072d4a07897cp+0, -0x1.fad5d3ffffa6fp-55,
    0x1.d5818dcfba487p+0, 0x1.4a385a63d07a7p-56, 0x1.da9e603db3285p+0, 0x1.e5a50d5c192acp-55,
    0x1.dfc97337b9b5fp+0, -0x1.2d52107b43e1fp-55, 0x1.e502ee78b3ff6p+0, 0x1.4b604603a88d3p-56,
    0x1.ea4afa2a490dap+0, -0x1.ff7128fd391f0p-55, 0x1.efa1bee615a27p+0, 0x1.ec3bc41aa2008p-55,
    0x1.f50765b6e4540p+0, 0x1.a64a931d185eep-55, 0x1.fa7c1819e90d8p+0, 0x1.7893b4d91cd9dp-56
};

// every thread of the block calls it; the caller's next barrier publishes it
__device__ inline void stage_exp_tab(double (&tab)[EXP_TAB]) {
  if (threadIdx.x < EXP_TAB) tab[threadIdx.x] = exp_tab_g[threadIdx.x];
}

// LO: with what the table's rounding left
template <bool LO>
__device__ inline double exp_neg(double s, const double *tab) {
  constexpr double magic = 6755399441055744.0;  // 1.5 2^52: the sum's low bits are the rounded integer
  const double t = __builtin_fma(s, -0x1.71547652b82fep+6, magic);
  const double kf = t - magic;
  int32_t k;
  asm("v_cvt_i32_f64 %0, %1" : "=v"(k) : "v"(kf));  // (saturates; a NaN gives 0)
  double r = __builtin_fma(kf, -0x1.62e42fc000000p-7, -s);
  r = __builtin_fma(kf, -0x1.7d1cf79abc9e4p-34, r);
  double q = __builtin_fma(r, 1.0 / 120.0, 1.0 / 24.0);
  q = __builtin_fma(r, q, 1.0 / 6.0);
  q = __builtin_fma(r, q, 0.5);
  q = __builtin_fma(r, q, 1.0);
  const uint32_t j = 2 * ((uint32_t)k & (EXP_N - 1));
  const double p = __builtin_fma(tab[j], LO ? __builtin_fma(r, q, tab[j + 1]) : r * q, tab[j]);
  return __builtin_amdgcn_ldexp(__builtin_fabs(p), k >> 6);
}

// ---------------------------------------------------------------------------
// reflection orbits of a lattice symmetric under x -> -x and y -> -y
// ---------------------------------------------------------------------------
template <class L>
constexpr int orbit_count() {
  int n = 0;
  for (int i = 0; i < L::Q; ++i) n += (L::S.v[i].x >= 0 && L::S.v[i].y >= 0);
  return n;
}
template <class L>
constexpr Vel orbit_rep(int k) {
  for (int j = 0, n = 0; j < L::Q; ++j)
    if (L::S.v[j].x >= 0 && L::S.v[j].y >= 0 && n++ == k) return L::S.v[j];
  return Vel{0, 0, 0};
}
template <class L>
constexpr int find_velocity(int x, int y) {
  for (int i = 0; i < L::Q; ++i)
    if (L::S.v[i].x == x && L::S.v[i].y == y) return i;
  return -1;
}
// (a variable template: an index expression would be evaluated at run time)
template <class L, int X, int Y>
constexpr int member = find_velocity<L>(X, Y);

// moments sum_i e_i x^p y^q, with n = x^2 + y^2
struct MomSums {
  double s, x, y, xx, xy, yy, xxx, xxy, xyy, yyy;  // the residual's
  double x4, x3y, x2y2, xy3, y4, x3n, x2yn, xy2n, y3n, x2nn, xynn, y2nn;
};

template <int K>
__device__ inline double scaled(double v) {
  return K == 1 ? v : (double)K * v;
}
template <int K>
__device__ inline void acc(double &m, double v) {
  m = K == 1 ? m + v : __builtin_fma((double)K, v, m);
}

template <class L, class C, int K, bool LO>
__device__ inline void orbit_sums(const double *lam, double l01, const double *tab, MomSums &m, C *e) {
  constexpr Vel v = orbit_rep<L>(K);
  constexpr int a = v.x, b = v.y, n = a * a + b * b;
  if constexpr (a == 0 && b == 0) {
    const double e0 = exp_neg<LO>(l01, tab);
    e[member<L, 0, 0>] = (C)e0;
    m.s += e0;
  } else if constexpr (b == 0) {
    const double E = __builtin_fma(lam[3], (double)(a * a), l01);
    const double X = scaled<a>(__builtin_fma(lam[6], (double)n, lam[1]));
    const double ep = exp_neg<LO>(E + X, tab), em = exp_neg<LO>(E - X, tab);
    e[member<L, a, 0>] = (C)ep;
    e[member<L, -a, 0>] = (C)em;
    const double p0 = ep + em, p1 = ep - em;
    m.s += p0;
    acc<a>(m.x, p1);
    acc<a * a>(m.xx, p0);
    acc<a * a * a>(m.xxx, p1);
    acc<a * a * a * a>(m.x4, p0);
    acc<a * a * a * n>(m.x3n, p1);
    acc<a * a * n * n>(m.x2nn, p0);
  } else if constexpr (a == 0) {
    const double E = __builtin_fma(lam[5], (double)(b * b), l01);
    const double Y = scaled<b>(__builtin_fma(lam[7], (double)n, lam[2]));
    const double ep = exp_neg<LO>(E + Y, tab), em = exp_neg<LO>(E - Y, tab);
    e[member<L, 0, b>] = (C)ep;
    e[member<L, 0, -b>] = (C)em;
    const double p0 = ep + em, p2 = ep - em;
    m.s += p0;
    acc<b>(m.y, p2);
    acc<b * b>(m.yy, p0);
    acc<b * b * b>(m.yyy, p2);
    acc<b * b * b * b>(m.y4, p0);
    acc<b * b * b * n>(m.y3n, p2);
    acc<b * b * n * n>(m.y2nn, p0);
  } else {
    const double E = __builtin_fma(lam[5], (double)(b * b), __builtin_fma(lam[3], (double)(a * a), l01));
    const double X = scaled<a>(__builtin_fma(lam[6], (double)n, lam[1]));
    const double Y = scaled<b>(__builtin_fma(lam[7], (double)n, lam[2]));
    const double Ep = __builtin_fma(lam[4], (double)(a * b), E), Em = __builtin_fma(lam[4], -(double)(a * b), E);
    const double S = X + Y, D = X - Y;
    const double epp = exp_neg<LO>(Ep + S, tab), emm = exp_neg<LO>(Ep - S, tab);
    const double epm = exp_neg<LO>(Em + D, tab), emp = exp_neg<LO>(Em - D, tab);
    e[member<L, a, b>] = (C)epp;
    e[member<L, -a, -b>] = (C)emm;
    e[member<L, a, -b>] = (C)epm;
    e[member<L, -a, b>] = (C)emp;
    const double sp = epp + emm, sm = epm + emp, dp = epp - emm, dm = epm - emp;
    const double p0 = sp + sm, p3 = sp - sm, p1 = dp + dm, p2 = dp - dm;
    m.s += p0;
    acc<a>(m.x, p1);
    acc<b>(m.y, p2);
    acc<a * a>(m.xx, p0);
    acc<a * b>(m.xy, p3);
    acc<b * b>(m.yy, p0);
    acc<a * a * a>(m.xxx, p1);
    acc<a * a * b>(m.xxy, p2);
    acc<a * b * b>(m.xyy, p1);
    acc<b * b * b>(m.yyy, p2);
    acc<a * a * a * a>(m.x4, p0);
    acc<a * a * a * b>(m.x3y, p3);
    acc<a * a * b * b>(m.x2y2, p0);
    acc<a * b * b * b>(m.xy3, p3);
    acc<b * b * b * b>(m.y4, p0);
    acc<a * a * a * n>(m.x3n, p1);
    acc<a * a * b * n>(m.x2yn, p2);
    acc<a * b * b * n>(m.xy2n, p1);
    acc<b * b * b * n>(m.y3n, p2);
    acc<a * a * n * n>(m.x2nn, p0);
    acc<a * b * n * n>(m.xynn, p3);
    acc<b * b * n * n>(m.y2nn, p0);
  }
}

template <class L, class C, bool LO, int... K>
__device__ inline void orbits(std::integer_sequence<int, K...>, const double *lam, double l01, const double *tab,
                              MomSums &m, C *e) {
  ((orbit_sums<L, C, K, LO>(lam, l01, tab, m, e), __builtin_amdgcn_sched_barrier(0)), ...);
}

// One pass over the populations at multipliers lam: e_i = exp(-(1 + lam .
// m_i)) and its moments.  e_i is kept only in the collision precision C,
// for the final equilibrium.
template <class L, class C, bool LO = true>
__device__ inline void expo_sums(const double *lam, const double *tab, MomSums &m, C *e) {
  // -0.0 is the neutral element of addition, so the first terms cost nothing
  m = MomSums{-0.0, -0.0, -0.0, -0.0, -0.0, -0.0, -0.0, -0.0, -0.0, -0.0, -0.0,
              -0.0, -0.0, -0.0, -0.0, -0.0, -0.0, -0.0, -0.0, -0.0, -0.0, -0.0};
  orbits<L, C, LO>(std::make_integer_sequence<int, orbit_count<L>()>{}, lam, 1.0 + lam[0], tab, m, e);
}

// G_a = sum_i e_i m_ia - M_a, per unit density
__device__ inline void residual8(const MomSums &m, double ux, double uy, double T, double (&G)[NLAM]) {
  const double uu = ux * ux + uy * uy;
  G[0] = m.s - 1.0;
  G[1] = m.x - ux;
  G[2] = m.y - uy;
  G[3] = m.xx - (ux * ux + T);
  G[4] = m.xy - ux * uy;
  G[5] = m.yy - (uy * uy + T);
  G[6] = (m.xxx + m.xyy) - ux * (uu + 4.0 * T);
  G[7] = (m.xxy + m.yyy) - uy * (uu + 4.0 * T);
}

// H = sum_i e_i m_i m_i^T (packed lower triangle) from the moments
__device__ inline void newton_matrix(const MomSums &m, double (&H)[NLAM * (NLAM + 1) / 2]) {
  const double xn = m.xxx + m.xyy, yn = m.xxy + m.yyy;
  const double xxn = m.x4 + m.x2y2, xyn = m.x3y + m.xy3, yyn = m.x2y2 + m.y4;
  const double v[NLAM * (NLAM + 1) / 2] = {
      m.s,
      m.x, m.xx,
      m.y, m.xy, m.yy,
      m.xx, m.xxx, m.xxy, m.x4,
      m.xy, m.xxy, m.xyy, m.x3y, m.x2y2,
      m.yy, m.xyy, m.yyy, m.x2y2, m.xy3, m.y4,
      xn, xxn, xyn, m.x3n, m.x2yn, m.xy2n, m.x2nn,
      yn, xyn, yyn, m.x2yn, m.xy2n, m.y3n, m.xynn, m.y2nn};
#pragma unroll
  for (int k = 0; k < NLAM * (NLAM + 1) / 2; ++k) H[k] = v[k];
}

__device__ inline double nrm2_8(const double *G) {
  double s = 0.0;
#pragma unroll
  for (int a = 0; a < NLAM; ++a) s += G[a] * G[a];
  return s;
}

// largest |G_a|; a NaN propagates so that it never passes a tolerance test
__device__ inline double nrmmax_8(const double *G) {
  double s = 0.0;
#pragma unroll
  for (int a = 0; a < NLAM; ++a) {
    const double v = fabs(G[a]);
    s = (v > s || v != v) ? v : s;
  }
  return s;
}

// 1 / sqrt(t) of a normal positive t to about an ulp: the hardware's estimate
// and one third-order correction (no special cases: the factorisation tests
// its pivots itself)
__device__ inline double rsqrt_pivot(double t) {
  const double y = __builtin_amdgcn_rsq(t);
  const double e = __builtin_fma(-t * y, y, 1.0);
  return __builtin_fma(y * e, __builtin_fma(e, 0.375, 0.5), y);
}

// d = H^-1 G by an in-place Cholesky factorisation of the packed H (the
// diagonal holds the reciprocals 1 / L_jj, so the solves multiply); false
// when H is not numerically positive definite (d is then of no use; a test
// after the factorisation instead of a return from each column keeps one
// straight line of code, whose registers the compiler can schedule)
__device__ inline bool cholesky_solve(double *H, const double *G, double *d) {
  bool ok = true;
#pragma unroll
  for (int j = 0; j < NLAM; ++j) {
    double t = H[j * (j + 1) / 2 + j];
#pragma unroll
    for (int k = 0; k < j; ++k) t -= H[j * (j + 1) / 2 + k] * H[j * (j + 1) / 2 + k];
    ok = ok && t > 0.0;
    const double inv = rsqrt_pivot(t);
    H[j * (j + 1) / 2 + j] = inv;
#pragma unroll
    for (int i = j + 1; i < NLAM; ++i) {
      double s = H[i * (i + 1) / 2 + j];
#pragma unroll
      for (int k = 0; k < j; ++k) s -= H[i * (i + 1) / 2 + k] * H[j * (j + 1) / 2 + k];
      H[i * (i + 1) / 2 + j] = s * inv;
    }
  }
#pragma unroll
  for (int i = 0; i < NLAM; ++i) {
    double s = G[i];
#pragma unroll
    for (int k = 0; k < i; ++k) s -= H[i * (i + 1) / 2 + k] * d[k];
    d[i] = s * H[i * (i + 1) / 2 + i];
  }
#pragma unroll
  for (int i = NLAM - 1; i >= 0; --i) {
    double s = d[i];
#pragma unroll
    for (int k = i + 1; k < NLAM; ++k) s -= H[k * (k + 1) / 2 + i] * d[k];
    d[i] = s * H[i * (i + 1) / 2 + i];
  }
  return ok;
}

// Newton-Raphson on the eight constraints from the multipliers in lam, with
// backtracking on the 2-norm of the residual (at most 30 halvings).  The
// stopping test max_a |G_a| <= tol is applied before every step; the first
// min_steps steps are always taken, and after exactly min_steps steps the
// looser tolerance tol_first applies (the surrogate's single correction).
// Returns the number of steps, or -1 (not converged within max_it, or H not
// positive definite).  e receives exp(-(1 + lam . m_i)) at the final lam.
// A rejected trial point goes back by the part of the step that is halved
// away, so that the iterate itself is not held beside it.
template <class L, class C>
__device__ inline int newton_lean(double ux, double uy, double T, double *lam, double tol, int max_it,
                                  int min_steps, double tol_first, C *e, const double *tab) {
  double d[NLAM];
  // one evaluation site and one way round: each pass either tests a trial
  // point of the line search or takes a step from an accepted iterate
  int it = 0, h = 0;
  bool trial = false;
  double n0 = 0.0, alpha = 1.0;
  for (;;) {
    MomSums m;
    expo_sums<L, C>(lam, tab, m, e);
    double G[NLAM];
    residual8(m, ux, uy, T, G);
    const double n1 = nrm2_8(G);
    double step;
    if (trial && !(n1 < n0) && h < 30) {
      ++h;
      alpha *= 0.5;
      step = -alpha;
    } else {
      if (trial) ++it;
      if (it >= min_steps && nrmmax_8(G) <= (it == min_steps && min_steps > 0 ? tol_first : tol)) return it;
      if (it == max_it) return -1;
      double H[NLAM * (NLAM + 1) / 2];
      newton_matrix(m, H);
      if (!cholesky_solve(H, G, d)) return -1;
      n0 = n1;
      step = alpha = 1.0;
      h = 0;
      trial = true;
    }
#pragma unroll
    for (int a = 0; a < NLAM; ++a) lam[a] = __builtin_fma(step, d[a], lam[a]);
  }
}

// cold-or-warm Newton solve to tol (the paper's solver); FP64 equilibrium out
template <class L>
__device__ inline int newton_solve(double ux, double uy, double T, double *lam, double tol, int max_it,
                                   double *e) {
  return newton_lean<L, double>(ux, uy, T, lam, tol, max_it, 0, tol, e, exp_tab_g);
}

}  // namespace lbm
