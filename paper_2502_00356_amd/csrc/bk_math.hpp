// bk_math.hpp - per-entry device routines for K_nu(x) by finite-window trapezoid
// quadrature of K_nu(x) = int_0^inf exp(-x cosh t) cosh(nu t) dt (Sec. IV-B).
//
// Notation follows Sec. IV-B: g(t) = log cosh(nu t) - x cosh t is the
// log-integrand, t* its maximiser over t >= 0 ("t_max"), [t0, t1] the window on
// which g(t) >= g(t*) - L, and the trapezoid sum is taken relative to a reference
// point t_ref (Eq. "refined": log K = g(t_ref) + log sum h c_m exp(g(t_m) - g(t_ref))).
//
// The plain FP64 form builds its node terms without cancellation (below); the
// FP32-term forms form the exponent directly (WalkF, further down), which their
// precision allows. With u = t - t_ref, w = u/2:
//   g(t) - g(t_ref) = nu u + log(1+P(t)) - log(1+P(t_ref)) - xterm,
//   P(t) = exp(-2 nu t),   xterm = x (cosh t - cosh t_ref)
//                                = 2 sinh w (x cosh t_ref sinh w + x sinh t_ref cosh w),
// and along the node grid every exponential is an exact geometric progression,
// advanced by one multiply (or fused multiply-add) per node in FP64:
//   V = expm1(|w|), Bw = exp(w), Bb = exp(-w), P = exp(-2 nu t).
// t_ref is the node nearest t*, so w = 0 falls on a node. Left of it |w| shrinks
// and V follows V' = (V - qm1) / q; right of it |w| grows and V' = V q + qm1
// (q = e^(h/2), qm1 = expm1(h/2)). Both directions keep V's relative error at
// a few ulps; 2 sinh w = sign(w) V (1 + e^-|w|) then has no cancellation.
// The log(1+P(t_ref)) term cancels against the prefactor, so
//   K = exp(-x) exp(Delta) h sum_m c_m exp(nu u_m - xterm_m) (1 + P_m),
//   Delta = nu t_ref - ln 2 - 2 x sinh^2(t_ref / 2).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace bk {

constexpr double kLn2 = 0.69314718055994530942;
constexpr double kLog2e = 1.4426950408889634074;
constexpr int kNodeMin = 4;
constexpr int kNodeMax = 512;
constexpr int kRuleCand = 15;

// Tables of the table-driven exponential and log1p (kernels stage them in LDS):
// [0, 64): 2^(j/64); [64, 129): log(1 + j/64); [129, 194): 1 / (1 + j/64).
constexpr int kTabLog1p = 64, kTabInv1p = 129, kTabLen = 194;

// Node-count rule constants, filled on the host: for each strip half-width a_k,
// a_k, 1 - cos a_k and log sec a_k (see node_step); and the tables above.
struct RuleTable {
    double a[kRuleCand];
    double omc[kRuleCand];
    double lsec[kRuleCand];
    double tab[kTabLen];
};

// Taylor coefficients in mu^2 of Temme's Gamma1 and Gamma2 (see temme_k below).
constexpr int kTemmeTerms = 10;

struct TemmeCoef {
    double g1[kTemmeTerms];
    double g2[kTemmeTerms];
};

// kRuleTab and kTemmeTab: the two tables above as device constants (values made
// by gen_tables.py at 60 digits and rounded to double), so no call sets anything
// up on the GPU.
#include "bk_tables.inc"

// The tables as the kernels read them: through a pointer the optimiser cannot see
// through (an empty asm statement), so that their values are fetched by scalar
// loads from the constant segment instead of being folded into the code as
// 64-bit literals, which costs registers (measured: spills in the Matern kernels).
typedef __attribute__((address_space(4))) const RuleTable ConstSegRuleTable;
typedef __attribute__((address_space(4))) const TemmeCoef ConstSegTemmeCoef;

__device__ __forceinline__ const RuleTable& rule_tab()
{
    ConstSegRuleTable* p = (ConstSegRuleTable*)&kRuleTab;
    __asm__ volatile("" : "+s"(p));
    return *(const RuleTable*)p;
}

__device__ __forceinline__ const TemmeCoef& temme_tab()
{
    ConstSegTemmeCoef* p = (ConstSegTemmeCoef*)&kTemmeTab;
    __asm__ volatile("" : "+s"(p));
    return *(const TemmeCoef*)p;
}

// Per-entry quadrature plan.
struct Plan {
    double tref;   // reference point: node mc, the node nearest the peak
    double t0;     // first node
    double h;      // step
    int N;         // intervals; nodes m = 0..N
    int mc;        // index of the reference node (0 <= mc <= N)
};

// Inclusive prefix sum over the 64 lanes of a wave (all active) with DPP lane
// moves instead of LDS: a scan within each 16-lane row by shifts of 1, 2, 4 and 8
// (lanes shifted in from outside the row add 0), then the last lane of row 0 is
// added to row 1 and of row 2 to row 3 (row_bcast:15), and the last lane of row 1
// to rows 2 and 3 (row_bcast:31).
__device__ __forceinline__ unsigned int wave_incl_scan(unsigned int v)
{
    v += __builtin_amdgcn_update_dpp(0u, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0u, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0u, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0u, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0u, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1, 3
    v += __builtin_amdgcn_update_dpp(0u, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2, 3
    return v;
}

// 1/a for a normal nonzero double: hardware reciprocal refined by two Newton
// steps (within about an ulp; no IEEE division sequence).
__device__ __forceinline__ double recip(double a)
{
    double r = __builtin_amdgcn_rcp(a);
    r = fma(r, fma(-a, r, 1.0), r);
    return fma(r, fma(-a, r, 1.0), r);
}

// e^x from T[j] = 2^(j/64), j = 0..63 (Tang's table-driven method): with
// k = floor(64 x log2 e) and f = x - k ln2/64, in [0, ln2/64) up to rounding,
// e^x = 2^(k div 64) T[k mod 64] e^f, and e^f is its Taylor polynomial through f^6
// (truncation below 2e-18). ln2/64 rounded to FP64 is 3.6e-19 short, so the
// reduction adds |k| 3.6e-19 relative: below 1.5e-15 for |x| <= 40, which covers
// every use whose result matters (the walks' node exponents reach below -40 only
// for terms under e^-40 of their sum; the set-up arguments are smaller). Within a
// few ulps overall there. x is clamped at -746, where e^x is already below half the
// smallest subnormal and the final ldexp gives 0 (also for x = -inf); ldexp takes
// large x to infinity. The kernels stage T in LDS.
__device__ __forceinline__ double exp_tab(double x, const double* T)
{
    x = fmax(x, -746.0);
    const double k = floor(x * 92.332482616893656);          // 64 log2 e
    const double f = fma(-k, 0.010830424696249145, x);        // ln2 / 64
    double p = 1.0 / 720.0;
    p = fma(p, f, 1.0 / 120.0);
    p = fma(p, f, 1.0 / 24.0);
    p = fma(p, f, 1.0 / 6.0);
    p = fma(p, f, 0.5);
    p = fma(p, f, 1.0);
    p = fma(p, f, 1.0);
    const int ki = (int)k;
    return ldexp(T[ki & 63] * p, ki >> 6);
}

// e^x as exp_tab for a finite x, as the node walks of the plain form call it: the
// integer is rounded to nearest by adding 1.5 2^52 (its low word is the integer), which
// halves the remainder (|f| <= ln2/128: degree 5, truncation below 4e-17) and leaves 13
// instructions of 18.
__device__ __forceinline__ double exp_node(double x, const double* T)
{
    const double m = fma(x, 92.332482616893656, 6755399441055744.0);
    const int ki = __double2loint(m);
    const double f = fma(-(m - 6755399441055744.0), 0.010830424696249145, x);
    double p = 1.0 / 120.0;
    p = fma(p, f, 1.0 / 24.0);
    p = fma(p, f, 1.0 / 6.0);
    p = fma(p, f, 0.5);
    p = fma(p, f, 1.0);
    const double t = T[ki & 63];
    return ldexp(fma(t * f, p, t), ki >> 6);
}

// e^x for |x| <= 708 from the same table, with ln2/64 in two parts (about an ulp).
__device__ __forceinline__ double exp_wide(double x, const double* T)
{
    const double m = fma(x, 92.332482616893656, 6755399441055744.0);
    const int ki = __double2loint(m);
    const double k = m - 6755399441055744.0;
    const double f = fma(-k, 3.623510646634843e-19, fma(-k, 0.010830424696249145, x));
    double p = 1.0 / 720.0;
    p = fma(p, f, 1.0 / 120.0);
    p = fma(p, f, 1.0 / 24.0);
    p = fma(p, f, 1.0 / 6.0);
    p = fma(p, f, 0.5);
    p = fma(p, f, 1.0);
    const double t = T[ki & 63];
    return ldexp(fma(t * f, p, t), ki >> 6);
}

// log(1 + p) for 0 <= p <= 1 from the same tables: with j = floor(64 p) and
// c = 1 + j/64, log(1 + p) = log c + log(1 + r), r = (p - j/64) / c in [0, 1/64)
// (p - j/64 is exact), the second by its Taylor series through r^9 (truncation
// below 1e-18); a few ulps.
__device__ __forceinline__ double log1p_tab(double p, const double* T)
{
    const int j = min(max((int)(p * 64.0), 0), 64);
    const double r = (p - (double)j * 0.015625) * T[kTabInv1p + j];
    double q = 1.0 / 9.0;
    q = fma(q, -r, 1.0 / 8.0);
    q = fma(q, -r, 1.0 / 7.0);
    q = fma(q, -r, 1.0 / 6.0);
    q = fma(q, -r, 1.0 / 5.0);
    q = fma(q, -r, 1.0 / 4.0);
    q = fma(q, -r, 1.0 / 3.0);
    q = fma(q, -r, 0.5);
    q = fma(q, -r, 1.0);
    return fma(q, r, T[kTabLog1p + j]);
}

// The tables into LDS; every thread of the block must call it (it ends with a
// barrier).
__device__ __forceinline__ void stage_tab(double* s)
{
    for (int j = threadIdx.x; j < kTabLen; j += blockDim.x) s[j] = rule_tab().tab[j];
    __syncthreads();
}

// log y for a positive normal y: y = 2^e m with m in [1/2, 1), log y = (e - 1) ln 2
// + log1p(2m - 1), the second from the tables (a few ulps).
__device__ __forceinline__ double log_tab(double y, const double* T)
{
    int e;
    const double m = frexp(y, &e);
    return fma((double)(e - 1), kLn2, log1p_tab(2.0 * m - 1.0, T));
}

__device__ __forceinline__ void cosh_sinh_tab(double t, double& ch, double& sh, const double* T)
{
    const double e = exp_tab(t, T);
    const double ei = recip(e);
    ch = 0.5 * (e + ei);
    sh = 0.5 * (e - ei);
}

__device__ __forceinline__ void cosh_sinh(double t, double& ch, double& sh)
{
    double e = exp(t);
    double ei = recip(e);
    ch = 0.5 * (e + ei);
    sh = 0.5 * (e - ei);
}

// log cosh(y) for y >= 0 without overflow: y + log1p(exp(-2y)) - ln 2.
__device__ __forceinline__ double logcosh_pos(double y, const double* T)
{
    return y + log1p_tab(exp_tab(-2.0 * y, T), T) - kLn2;
}

// g and its first three derivatives at t >= 0 (g''' for Halley's method on g').
struct GDer {
    double g, g1, g2, g3;
};

__device__ __forceinline__ GDer g_derivs(double nu, double x, double t, const double* T)
{
    GDer d;
    const double p = exp_tab(-2.0 * nu * t, T);
    const double ip = recip(1.0 + p);
    const double th = (1.0 - p) * ip;                 // tanh(nu t)
    const double s2 = 4.0 * p * ip * ip;              // sech^2(nu t)
    double ch, sh;
    cosh_sinh_tab(t, ch, sh, T);
    d.g = nu * t + log1p_tab(p, T) - kLn2 - x * ch;
    d.g1 = nu * th - x * sh;
    d.g2 = nu * nu * s2 - x * ch;
    d.g3 = -2.0 * nu * nu * nu * th * s2 - x * sh;
    return d;
}

// Halley step for a root of f with derivatives f1, f2: 2 f f1 / (2 f1^2 - f f2),
// or the Newton step f / f1 where the Halley denominator is not a positive normal
// number.
__device__ __forceinline__ double halley_step(double f, double f1, double f2)
{
    const double den = 2.0 * f1 * f1 - f * f2;
    return den > 1e-300 ? 2.0 * f * f1 * recip(den) : f / f1;
}

// The three roots below are found by Halley's method (cubic convergence) and
// stop once a step is below 1e-7 (peak) or 1e-5 (window ends) of t: the error
// left after such a step is of order its cube, below 1e-15 relative.

// Starting points of the root searches below. They only seed Halley's method, so
// they come from FP32 hardware operations (a few instructions against the library
// asinh / acosh in FP64), moved outward by 1e-4 relative so that they keep the side
// of the root the searches start from; beyond the FP32 range, log(2y) by the
// table logarithm.
// Upper bound of asinh(y), y > 0.
__device__ __forceinline__ double asinh_start(double y, const double* T)
{
    if (y < 1e18) {
        const float yf = (float)y;
        return (double)(__logf(yf + __fsqrt_rn(fmaf(yf, yf, 1.0f))) * 1.0001f);
    }
    return log_tab(2.0 * y, T) * 1.0001;
}
// Lower bound of acosh(1 + eps), eps > 0: log1p(eps + sqrt(eps (2 + eps))).
__device__ __forceinline__ double acosh1p_start(double eps, const double* T)
{
    if (eps < 1e18) {
        const float e = (float)eps;
        return (double)(log1pf(e + __fsqrt_rn(e * (2.0f + e))) * 0.9999f);
    }
    return log_tab(2.0 * eps, T) * 0.9999;
}

// Maximiser t* of g over t >= 0 when nu^2 > x (Sec. IV-B: otherwise t* = 0), the
// zero of g' = nu tanh(nu t) - x sinh t. Since nu tanh < nu, it lies left of
// asinh(nu/x), where the iteration starts (the bracket search of FINDRANGE is
// replaced by this analytic upper bound); g' is decreasing right of t* and steps
// that would leave t > 0 are halved.
__device__ inline double peak_solve(double nu, double x, const double* T)
{
    double t = asinh_start(fmin(nu / x, 1e300), T);
    for (int it = 0; it < 64; ++it) {
        const GDer d = g_derivs(nu, x, t, T);
        const double dt = halley_step(d.g1, d.g2, d.g3);
        double tn = t - dt;
        if (!(tn > 0.0)) tn = 0.5 * t;
        t = tn;
        if (!(fabs(dt) > 1e-7 * t) || t < 1e-150) break;
    }
    return t;
}

// Root t1 > t* of G(t) = g(t) - gstar + L (g concave and decreasing beyond t*).
// Start at acosh(cosh t* + L/x): there the x-term alone has dropped by L and the
// log cosh term has grown, so G >= 0 (FINDRANGE's lower end). Iterates are kept
// in (t*, t* + 4 (start - t*) + 1].
__device__ inline double window_right(double nu, double x, double tstar, double chstar,
                                      double gstar, double L, const double* T)
{
    double t = acosh1p_start((chstar - 1.0) + L / x, T);
    const double tcap = tstar + 4.0 * (t - tstar) + 1.0;
    for (int it = 0; it < 64; ++it) {
        const GDer d = g_derivs(nu, x, t, T);
        const double dt = halley_step(d.g - gstar + L, d.g1, d.g2);
        double tn = fmin(t - dt, tcap);
        if (!(tn > tstar)) tn = 0.5 * (t + tstar);
        const bool done = !(fabs(tn - t) > 1e-5 * t);
        t = tn;
        if (done) break;
    }
    return t;
}

// Root t0 in (0, t*) of G when G(0) < 0 (only possible if nu t* > L, since g' <= nu).
// Bracket: G(0) < 0 and G(t* - L/nu) >= 0, shrunk at every iterate; a step that
// would leave it is replaced by bisection.
__device__ inline double window_left(double nu, double x, double tstar, double gstar, double L, const double* T)
{
    double lo = 0.0, hi = fmax(tstar - L / nu, 0.0);
    double t = hi;
    for (int it = 0; it < 100; ++it) {
        const GDer d = g_derivs(nu, x, t, T);
        const double G = d.g - gstar + L;
        if (G >= 0.0) hi = t; else lo = t;
        const double dt = halley_step(G, d.g1, d.g2);
        double tn = t - dt;
        if (!(fabs(dt) > 1e-5 * t)) { t = fmin(fmax(tn, lo), hi); break; }
        if (!(tn >= lo && tn <= hi)) tn = 0.5 * (lo + hi);
        t = tn;
        if (hi - lo <= 1e-15 * hi) break;
    }
    return t;
}

// Trapezoid step from the strip bound: the best over the candidate half-widths a
// of 2 pi a / (Lq + ln 2 + x (1 - cos a) + (nu + 1) log sec a).
__device__ inline double node_step(double nu, double x, double Lq, const RuleTable& R)
{
    double base = Lq + kLn2;
    double nu1 = nu + 1.0;
    double bn = R.a[0], bd = base + x * R.omc[0] + nu1 * R.lsec[0];
#pragma unroll
    for (int k = 1; k < kRuleCand; ++k) {
        double den = base + x * R.omc[k] + nu1 * R.lsec[k];
        bool better = R.a[k] * bd > bn * den;
        bn = better ? R.a[k] : bn;
        bd = better ? den : bd;
    }
    return 6.283185307179586477 * bn / bd;
}

__device__ __forceinline__ int node_count(double width, double h)
{
    double r = ceil(width / h);
    if (!(r >= (double)kNodeMin)) r = (double)kNodeMin;   // also maps NaN to the minimum
    if (r > (double)kNodeMax) r = (double)kNodeMax;
    return (int)r;
}

// Plain bracket solver (FP64): peak, window at threshold L, node count for Lq,
// reference node. Also returns, for the prefactor,
// Delta = nu t_ref - ln 2 - 2 x sinh^2(t_ref/2), and the constants
// A = x cosh(t_ref)/2, B = x sinh(t_ref)/2 of the cancellation-free xterm.
struct Solved {
    Plan p;
    double delta, dlo;   // Delta as an unevaluated sum delta + dlo (|dlo| below an ulp of delta)
    double A, B;         // x cosh(t_ref) / 2, x sinh(t_ref) / 2 (single walk, FP32-term walk)
    double E, Ei, Sr;    // e^t_ref, e^-t_ref, expm1(t_ref) (paired walk of the plain sum)
    double gstar;   // g(t*) (used by the window export)
    double t1;
};

// Rounding error of s = a + b (Knuth's two-sum): a + b = s + two_sum_err(a, b, s) exactly.
__device__ __forceinline__ double two_sum_err(double a, double b, double s)
{
    const double bb = s - a;
    return (a - (s - bb)) + (b - bb);
}

// ln 2 - kLn2 (the part of ln 2 below the double kLn2).
constexpr double kLn2Lo = 2.319046813846299558e-17;

// Delta = nu t_ref - ln 2 - q as hi + lo: the product split exactly by a fused
// multiply-add, the two sums' rounding errors carried by two_sum_err. Contraction
// is off here: fusing nu t_ref into the first sum (or q's product into it) would
// round something other than what the error terms describe.
__device__ __forceinline__ void delta_dd(double nu, double tref, double q, double& hi, double& lo)
{
#pragma clang fp contract(off)
    const double pr = nu * tref, pe = fma(nu, tref, -pr);
    const double s1 = pr - q, e1 = two_sum_err(pr, -q, s1);
    const double s2 = s1 - kLn2, e2 = two_sum_err(s1, -kLn2, s2);
    hi = s2;
    lo = ((pe + e1) + e2) - kLn2Lo;
}

// Node grid on [t0, t1] with step at most h0, reference node nearest tpk, and
// the prefactor constants for the node walk. Delta = nu t_ref - ln 2 -
// 2 x sinh^2(t_ref/2) reaches ~120 for large orders at small x, where rounding it
// to one double would cost ~1e-14 of K; it is kept as delta + dlo, with nu t_ref
// split exactly (fused multiply-add) and the sums' rounding errors carried, so
// that what is left is the ~3 ulps of the sinh^2 term.
__device__ inline Solved plan_window(double nu, double x, double t0, double t1, double tpk, double h0)
{
    Solved s;
    int N = node_count(t1 - t0, h0);
    double h = (t1 - t0) / (double)N;
    int mc = 0;
    if (tpk > t0) {
        double r = rint((tpk - t0) / h);
        mc = (int)fmin(fmax(r, 0.0), (double)N);
    }
    double tref = t0 + (double)mc * h;
    double ch, sh;
    cosh_sinh(tref, ch, sh);
    double em = expm1(0.5 * tref);                     // sinh(t/2) = em (em + 2) / (2 (em + 1))
    double sh2 = em * (em + 2.0) / (2.0 * (em + 1.0));
    s.p.tref = tref;
    s.p.t0 = t0;
    s.p.N = N;
    s.p.mc = mc;
    s.p.h = h;
    delta_dd(nu, tref, 2.0 * x * sh2 * sh2, s.delta, s.dlo);
    s.A = 0.5 * x * ch;
    s.B = 0.5 * x * sh;
    s.Sr = em * (em + 2.0);                            // expm1(t_ref), no cancellation
    s.E = s.Sr + 1.0;
    s.Ei = recip(s.E);
    s.gstar = 0.0;
    s.t1 = t1;
    return s;
}

__device__ inline Solved plain_solve(double nu, double x, double L, double Lq, const RuleTable& R,
                                     const double* T)
{
    double tstar = 0.0;
    if (nu * nu > x) tstar = peak_solve(nu, x, T);
    double chs, shs;
    cosh_sinh_tab(tstar, chs, shs, T);
    double gstar = logcosh_pos(nu * tstar, T) - x * chs;
    double t1 = window_right(nu, x, tstar, chs, gstar, L, T);
    double t0 = 0.0;
    if (-x < gstar - L) t0 = window_left(nu, x, tstar, gstar, L, T);
    Solved s = plan_window(nu, x, t0, t1, tstar, node_step(nu, x, Lq, R));
    s.gstar = gstar;
    return s;
}

// Step floor for the learned forms and the plain form: the strip bound of node_step at a single
// half-width, a = min(sqrt(2 (Lq + ln 2) / (x + nu + 1)), 1.3) (the maximiser of
// the bound's small-a expansion, capped), in FP32 with 1 - cos a = 2 sin^2(a/2),
// shrunk by 0.1% so that rounding can only add nodes. Any a in (0, pi/2) gives an
// admissible step; over the grid law this one is within 6% of the best of the 15
// candidates the plain solver tries (median 0.5%), for a fraction of the work.
__device__ __forceinline__ float node_step_learned(float nu, float x, float Lq)
{
    const float c = Lq + 0.693147181f, nu1 = nu + 1.0f;
    const float a = fminf(__builtin_amdgcn_sqrtf(2.0f * c * __builtin_amdgcn_rcpf(x + nu1)), 1.3f);
    const float s = __sinf(0.5f * a);
    // cos a >= cos 1.3 > 0.26: the hardware logarithm needs no range handling
    const float den = c + 2.0f * x * s * s - nu1 * 0.69314718f * __builtin_amdgcn_logf(__cosf(a));
    return 6.28318531f * 0.999f * a * __builtin_amdgcn_rcpf(den);
}

// The plain form's plan without the exact solve: a window that contains {t : g(t) >=
// g(t*) - L}, and a reference near t*, in FP32. A wider window costs nodes, not accuracy:
// here at most ln 2 in L on a side and what one Newton step leaves (about 1% more nodes; a
// second one on either side saves less than a hundredth of a node over nu <= 60), for 130
// instructions in place of the roots' 1,500.
//  - The reference tp = asinh(nu / x) >= t* (0 where nu^2 <= x, as t*); g(tp) <= g(t*), so
//    a threshold below g(tp) lies below g(t*).
//  - Right end: log cosh(nu t) grows by at most nu (t - tp), so G(tp + d) <= -F(d),
//    F(d) = x (cosh(tp + d) - cosh tp) - nu d - L, convex: a Newton step from either side
//    lands at or right of the root. cosh differences as 2 sinh sinh (no cancellation).
//  - Left end: log cosh(nu t) <= nu t and g(tp) >= nu tp - ln 2 - x cosh tp, so G(tp - e)
//    <= F(e) = L + ln 2 - nu e + x (cosh tp - cosh(tp - e)), concave and decreasing: a Newton
//    step lands at or past the root; F(tp) >= 0 leaves the window starting at 0.
// FP32 rounding moves an end by 1e-5 of its distance; L carries 0.01 for it. For 1e-12 <=
// x <= 1e5, nu <= 1e4, 1 <= L <= 500, Lq >= 1 (plan_fast_ok); plain_solve covers the rest: below
// L = 0.09 the right end's start may lie left of F's minimum, where a Newton step goes the other
// way, and below Lq = 0.8 a step may be so long that e^(-2 nu h) is no double.
__device__ __forceinline__ bool plan_fast_ok(double nu, double x, double L, double Lq)
{
    return x >= 1e-12 && x <= 1e5 && nu <= 1e4 && L >= 1.0 && L <= 500.0 && Lq >= 1.0;
}

// Where the window itself still holds, for walks that take both sides by products: x up to 1e8,
// orders up to 1e6 (FP32's roundings of t and of e^t then take up to 0.13 off L).
__host__ __device__ __forceinline__ bool plan_wide_ok(double nu, double x, double L, double Lq)
{
    return x >= 1e-12 && x <= 1e8 && nu <= 1e6 && L >= 1.0 && L <= 500.0 && Lq >= 1.0;
}

__device__ __forceinline__ float exp_fast(float y) { return __builtin_amdgcn_exp2f(y * 1.44269504f); }
__device__ __forceinline__ float asinh_fast(float y)
{
    return 0.69314718f * __builtin_amdgcn_logf(y + __builtin_amdgcn_sqrtf(fmaf(y, y, 1.0f)));
}

// Pairs whose ends' Newton steps start at quadratic bounds of the ends (from the starts below
// they overshoot to several times the window's width: 45 nodes at nu = 1,000, x = 500, where 27
// do). Looked for once a wave (kLarge: any lane's): those of small orders pay for nothing.
__device__ __forceinline__ bool large_pair(float nu, float x) { return nu > 60.0f || x > 1e5f; }

// Upper bound of the d > 0 where x (cosh(t + d) - cosh t) = slope d + L; E, Ei = e^t, e^-t.
template <bool kLarge>
__device__ __forceinline__ float right_end_fast(float t, float E, float Ei, float x, float slope, float L, bool large)
{
    // start: the x term alone drops by L; then it drops by L and the slope's rise up to there
    // (still left of the root), then one Newton step to its right
    const float ix = __builtin_amdgcn_rcpf(x), ec = 0.5f * (E + Ei) - 1.0f;
    auto drop = [&](float l) {
        const float e = fmaf(l, ix, ec);
        return fmaxf(0.69314718f * __builtin_amdgcn_logf(1.0f + e + __builtin_amdgcn_sqrtf(e * (e + 2.0f))) - t, 1e-3f);
    };
    float d = drop(fmaf(slope, drop(L), L));
    if (kLarge && large) {
        // F(d) >= C d^2 / 2 - r d - L, C = x cosh t, r = slope - x sinh t: right of its root
        const float C = 0.5f * x * (E + Ei), r = fmaxf(slope - 0.5f * x * (E - Ei), 0.0f);
        const float s = (r + __builtin_amdgcn_sqrtf(fmaf(r, r, 2.0f * C * L))) * __builtin_amdgcn_rcpf(C);
        if (s <= 1.0f) d = s;
    }
    const float a = exp_fast(0.5f * d), ai = __builtin_amdgcn_rcpf(a);
    const float b = E * a, bi = Ei * ai;                           // e^(t + d/2)
    const float F = 0.5f * x * (a - ai) * (b - bi) - slope * d - L;    // 2 sinh sinh = (a - 1/a)(b - 1/b) / 2
    const float D = 0.5f * x * (b * a - bi * ai) - slope;
    return (d - F * __builtin_amdgcn_rcpf(D)) * 1.0001f;
}

// Left end of the window from tp (e^tp = E): 0, or tp - e with F(e) = 0 (see above).
template <bool kLarge>
__device__ __forceinline__ float left_end_fast(float tp, float E, float Ei, float nu, float x, float L, bool large)
{
    const float L2 = L + 0.69314718f, hx = 0.5f * x;
    const float e0 = L2 + x * (0.5f * (E + Ei) - 1.0f);
    if (!(e0 < nu * tp)) return 0.0f;
    float e = e0 * __builtin_amdgcn_rcpf(nu);
    if (kLarge && large) {
        // F(e) <= L2 - C (e^-e - 1 + e) with C = x cosh tp >= nu, below 0 at sqrt(3 L2 / C) <= 1
        const float b = 3.0f * L2 * __builtin_amdgcn_rcpf(hx * (E + Ei));
        if (b <= 1.0f) e = fminf(e, __builtin_amdgcn_sqrtf(b));
    }
    const float a = exp_fast(0.5f * e), ai = __builtin_amdgcn_rcpf(a);
    const float b = E * ai, bi = Ei * a;                           // e^(tp - e/2)
    const float F = L2 - nu * e + hx * (a - ai) * (b - bi);
    const float D = hx * (b * ai - bi * a) - nu;
    return fmaxf(tp - (e - F * __builtin_amdgcn_rcpf(D)) * 1.0001f, 0.0f);
}

__device__ __forceinline__ void window_fast(float nu, float x, float L, float& t0, float& t1, float& tp)
{
    L += 0.01f;
    tp = nu * nu > x ? asinh_fast(nu * __builtin_amdgcn_rcpf(x)) : 0.0f;
    const float E = exp_fast(tp), Ei = __builtin_amdgcn_rcpf(E);
    const bool large = large_pair(nu, x);
    auto ends = [&](auto any) {
        t1 = tp + right_end_fast<any.value>(tp, E, Ei, x, nu, L, large);
        t0 = left_end_fast<any.value>(tp, E, Ei, nu, x, L, large);
    };
    if (__builtin_expect(__any(large), 0)) ends(std::true_type{});
    else ends(std::false_type{});
}

// expm1(y) for 0 <= y <= 1/8 (Taylor through y^10, truncation below 1e-18 relative).
__device__ __forceinline__ double expm1_small(double y)
{
    double p = 1.0 / 3628800.0;
    p = fma(p, y, 1.0 / 362880.0);
    p = fma(p, y, 1.0 / 40320.0);
    p = fma(p, y, 1.0 / 5040.0);
    p = fma(p, y, 1.0 / 720.0);
    p = fma(p, y, 1.0 / 120.0);
    p = fma(p, y, 1.0 / 24.0);
    p = fma(p, y, 1.0 / 6.0);
    p = fma(p, y, 0.5);
    return fma(p * y, y, y);
}

// The strip bound's step as node_step_learned, with cos a from its series in a^2 (x (1 - cos
// a) without cancellation).
__device__ __forceinline__ float node_step_fast(float nu, float x, float Lq)
{
    const float c = Lq + 0.693147181f, nu1 = nu + 1.0f;
    const float v = fminf(2.0f * c * __builtin_amdgcn_rcpf(x + nu1), 1.69f);       // a^2
    const float u = v * fmaf(fmaf(fmaf(fmaf(v, 1.0f / 3628800.0f, -1.0f / 40320.0f), v, 1.0f / 720.0f), v, -1.0f / 24.0f),
                             v, 0.5f);                                              // 1 - cos a
    const float den = fmaf(x, u, c) - nu1 * 0.69314718f * __builtin_amdgcn_logf(1.0f - u);
    return 6.28318531f * 0.999f * __builtin_amdgcn_sqrtf(v) * __builtin_amdgcn_rcpf(den);
}

// Node count N of [t0, t1] for a step of at most h, and the index mc of the node nearest tp.
__device__ __forceinline__ void node_grid(float t0, float t1, float tp, float h, unsigned int& N, unsigned int& mc)
{
    const float w = t1 - t0;
    const float nf = fminf(fmaxf(ceilf(w * __builtin_amdgcn_rcpf(h)), (float)kNodeMin), (float)kNodeMax);
    N = (unsigned int)nf;
    mc = (unsigned int)fminf(rintf((tp - t0) * nf * __builtin_amdgcn_rcpf(w)), nf);
}

// The fast window with its node count N and the index mc of the reference node.
__device__ __forceinline__ void window_count(double nu, double x, double L, double Lq, float& t0, float& t1,
                                             unsigned int& N, unsigned int& mc)
{
    float tp;
    window_fast((float)nu, (float)x, (float)L, t0, t1, tp);
    node_grid(t0, t1, tp, node_step_fast((float)nu, (float)x, (float)Lq), N, mc);
}

// Set-up of the paired walk on the nodes t0 + m (t1 - t0) / N.
__device__ __forceinline__ Solved plan_setup(double nu, double x, float t0, float t1, unsigned int N, unsigned int mc)
{
    Solved s;
    const double h = ((double)t1 - (double)t0) * recip((double)N);
    const double tref = fma((double)mc, h, (double)t0);
    const double em = expm1(0.5 * tref);
    s.Sr = em * (em + 2.0);                            // expm1(t_ref), no cancellation
    s.E = s.Sr + 1.0;
    s.Ei = recip(s.E);
    const double sh2 = 0.5 * fma(em, recip(em + 1.0), em);   // sinh(t/2) = (em + em / (em + 1)) / 2
    s.p.tref = tref;
    s.p.t0 = (double)t0;
    s.p.N = (int)N;
    s.p.mc = (int)mc;
    s.p.h = h;
    delta_dd(nu, tref, 2.0 * x * sh2 * sh2, s.delta, s.dlo);
    s.A = s.B = 0.0;                                   // not used by the paired walk
    s.gstar = 0.0;
    s.t1 = (double)t1;
    return s;
}

// Plan of the plain sum (both sides by products): the fast window where it applies, else the
// exact solve.
__device__ inline Solved plain_plan(double nu, double x, double L, double Lq, const RuleTable& R, const double* T)
{
    if (!plan_wide_ok(nu, x, L, Lq)) return plain_solve(nu, x, L, Lq, R, T);
    float t0, t1;
    unsigned int N, mc;
    window_count(nu, x, L, Lq, t0, t1, N, mc);
    return plan_setup(nu, x, t0, t1, N, mc);
}

// Geometric-progression state of one entry's node walk.
struct Walk {
    double k, V, Bw, Bb, P;        // at the current node; k = m - mc (exact), u = k h
    double h, q, qm1, qi, rho;     // per-step factors
    int mc;
};

__device__ __forceinline__ Walk walk_begin(double nu, const Plan& p)
{
    Walk w;
    w.mc = p.mc;
    w.k = -(double)p.mc;
    w.V = expm1(0.5 * (double)p.mc * p.h);        // expm1(|w_0|), w_0 = -mc h / 2
    w.Bb = w.V + 1.0;
    w.Bw = recip(w.Bb);
    w.P = exp(-2.0 * nu * p.t0);
    w.h = p.h;
    w.qm1 = expm1(0.5 * p.h);
    w.q = w.qm1 + 1.0;
    w.qi = recip(w.q);
    w.rho = exp(-2.0 * nu * p.h);
    return w;
}

// Exponent nu u - xterm at node m (FP64, cancellation-free).
__device__ __forceinline__ double walk_exponent(const Walk& w, int m, double nu, double A, double B)
{
    double sv = (m < w.mc) ? -w.V : w.V;
    double sg = sv * (1.0 + fmin(w.Bw, w.Bb));   // 2 sinh(u/2)
    double c2 = w.Bw + w.Bb;                      // 2 cosh(u/2)
    double xterm = sg * (A * sg + B * c2);        // x (cosh t - cosh t_ref)
    return nu * (w.k * w.h) - xterm;
}

// Advance from node m to node m + 1.
__device__ __forceinline__ void walk_step(Walk& w, int m)
{
    w.k += 1.0;                                   // u = k h is formed per node: no drift
    w.Bw *= w.q;
    w.Bb *= w.qi;
    w.P *= w.rho;
    double vin = fmax((w.V - w.qm1) * w.qi, 0.0);
    double vout = fma(w.V, w.q, w.qm1);
    w.V = (m + 1 <= w.mc) ? vin : vout;
}

// FP64 trapezoid sum of the plain form, S = sum_m c_m exp(d_m) (1 + P_m),
// c_0 = c_N = 1/2, as a paired walk outward from the reference node: iteration j
// takes node mc + j (right, j <= N - mc) and node mc - j (left, 1 <= j <= mc), with
// d = +- nu j h - X, X = x (cosh t - cosh t_ref), P = e^(-2 nu t). X follows its second
// difference,
//   X_(j+1) = X_j + S_(j+1),  S_(j+1) = S_j + (2 cosh h - 2) (X_j + x cosh t_ref),
// from the exact first step on either side (X_1 = S_1 = +-2 x sinh(h/2) sinh(t_ref +- h/2)):
// it never holds the size of x cosh t itself. On the right all terms are positive and X
// keeps its relative accuracy (about an ulp a step). On the left the recurrence's growing
// solution e^(j h) is not the sum's: a rounding of X (<= nu) there has grown by e^s at a
// distance s, where the term has fallen to about e^(-nu (s - 1)), and s <= ln(2 nu / x). So
// it costs no more than a few ulps of max(nu, 1) where nu >= 1 or x >= 0.1, as in the
// standalone form (Temme's series below); elsewhere (x = 1e-4, nu = 0.3: 1e-14) the left
// side takes the product 2 sinh(j h / 2) 2 sinh(t_ref - j h / 2) from running exponentials,
// kProduct. Three operations a node against seven: 2^24 pairs of the (nu, x) grid 466 ->
// 450 us. T is exp_tab's table; E, Ei, Sr = e^t_ref, e^-t_ref, expm1(t_ref) from the solve.

struct CoshWalk {
    double X, S;
    __device__ __forceinline__ void step(double k2, double c)
    {
        S = fma(k2, X, S + c);
        X += S;
    }
};

template <bool kProduct>
struct CoshPair {
    CoshWalk R, L;
    double k2, c;                        // 2 cosh h - 2, and its product with x cosh t_ref
    double V, Bq, q, qm1, qi, E, Ei, xh; // product form: expm1(w), e^-w, w = j h / 2

    __device__ __forceinline__ CoshPair(double x, double h, double E_, double Ei_, double Sr)
    {
        E = E_;
        Ei = Ei_;
        xh = 0.5 * x;
        qm1 = h <= 0.25 ? expm1_small(0.5 * h) : expm1(0.5 * h);
        q = qm1 + 1.0;
        qi = recip(q);
        V = qm1;
        Bq = qi;
        const double s1 = fma(V, Bq, V), SR = fma(Sr, q, V);         // 2 sinh(h/2), expm1(t_ref + h/2)
        R.X = R.S = xh * s1 * fma(SR, Ei * qi, SR);
        L.X = L.S = -xh * s1 * fma(E, qi, -Ei * q);
        k2 = s1 * s1;
        c = k2 * (xh * (E + Ei));
    }
    __device__ __forceinline__ void step()
    {
        R.step(k2, c);
        if (kProduct) {
            V = fma(V, q, qm1);
            Bq *= qi;
            L.X = -xh * fma(V, Bq, V) * fma(E, Bq, -Ei * (V + 1.0));
        } else {
            L.step(k2, c);
        }
    }
};

// kAny: for windows of any pair. Past x = 1e306 the grid's own roundings reach exponents that
// exp_node does not take.
template <bool kProduct, bool kAny = false>
__device__ inline double sum_f64(double nu, double x, const Plan& p, double E, double Ei, double Sr, const double* T)
{
    const int nr = p.N - p.mc, nl = p.mc, jmax = nr > nl ? nr : nl;
    const double nh = nu * p.h;
    // where e^(-2 nu h) leaves the double range (orders from some 1e4 on, product form) P is 0 on
    // the left as well
    const double rho = exp_tab(-2.0 * nh, T), rhoi = kProduct && rho < 1e-300 ? 0.0 : recip(rho);
    double PR = exp_tab(-2.0 * nu * p.tref, T), PL = PR;   // e^(-2 nu t) at nodes mc + j, mc - j
    double jd = 1.0, S = 0.0, tr = 0.0, tl = 0.0;
    CoshPair<kProduct> W(x, p.h, E, Ei, Sr);
    // node mc: the exponent is 0; it is node 0 if mc = 0 and node N if mc = N
    const double t0 = 1.0 + PR;
    for (int j = 1; j <= jmax; ++j) {
        PR *= rho;
        PL *= rhoi;
        if (j <= nr) {
            const double d = fma(jd, nh, -W.R.X), e = kAny ? exp_tab(d, T) : exp_node(d, T);
            tr = fma(e, PR, e);
            S += tr;
        }
        if (j <= nl) {
            const double d = fma(-jd, nh, -W.L.X), e = kAny ? exp_tab(d, T) : exp_node(d, T);
            tl = fma(e, PL, e);
            S += tl;
        }
        W.step();
        jd += 1.0;
    }
    // trapezoid ends: half of node N and of node 0
    S = fma(-0.5, tr + tl, S);
    return fma(nl == 0 || nr == 0 ? 0.5 : 1.0, t0, S);
}

// Node walk of the FP32-term forms (mixed and learned). Their terms need the
// exponent only to ~1e-9 absolute, so it is formed directly in FP64, in base 2,
//   d_m = log2(e) (nu (t_m - t_ref) - x (cosh t_m - cosh t_ref)),
// with cosh t_m from the three-term recurrence c_{m+1} = 2 cosh(h) c_m - c_{m-1}
// run forward from t_0 (the growing solution: its relative error stays within a
// few m^2 ulps), so the absolute error of d_m is about x cosh(t_m) m^2 2^-53,
// below 1e-10 on the whole (nu, x) range. The factor Q = 1 + e^(-2 nu t) follows
// Q' = rho Q + (1 - rho), rho = e^(-2 nu h) (contracting, so no error growth).
struct WalkF {
    double c, cn, kappa;      // cosh t_m, cosh t_{m+1}, 2 cosh h
    double a2, e, b2;         // d_m = a2 c_m + e_m; e_m = x cosh(t_ref) log2 e + (m - m_ref) b2, advanced by b2
    double Q, rho, omr;       // Q = 1 + e^(-2 nu t_m)
};
// e_m accumulates one rounding per node: m ulps of |e| <= x cosh t_ref + 30, below
// 1e-11 absolute in d_m for the windows here (the FP32 terms need ~1e-8).

// Walk state from the exponentials e = e^{t_0}, ei = e^{-t_0}, q2 = e^h,
// qi2 = e^{-h}, rho = e^{-2 nu h} (given by the caller).
__device__ __forceinline__ WalkF walkf_begin_exp(double nu, double x, double t0, double h, int mref, double xch_ref,
                                                 double e, double ei, double q2, double qi2, double rho)
{
    WalkF w;
    w.kappa = q2 + qi2;
    w.c = 0.5 * (e + ei);
    w.cn = 0.5 * (e * q2 + ei * qi2);
    w.a2 = -x * kLog2e;
    w.b2 = nu * h * kLog2e;
    w.e = fma(-(double)mref, w.b2, xch_ref * kLog2e);
    w.rho = rho;
    w.omr = 1.0 - rho;                // absolute error 2^-53: Q's error stays ~m 2^-53
    // Q only needs FP32 accuracy: e^(-2 nu t_0) in FP32 moves Q by < 6e-8 relative
    w.Q = 1.0 + (double)__expf((float)(-2.0 * nu * t0));
    return w;
}

__device__ __forceinline__ double walkf_exponent2(const WalkF& w) { return fma(w.a2, w.c, w.e); }

__device__ __forceinline__ void walkf_step(WalkF& w)
{
    const double c2n = fma(w.kappa, w.cn, -w.c);
    w.c = w.cn;
    w.cn = c2n;
    w.e += w.b2;
    w.Q = fma(w.Q, w.rho, w.omr);
}

// Mixed form: the walk above with the reference at the node nearest the peak
// (exponents <= about 0), exponential in FP32, Kahan-compensated FP32 sum.
// A = x cosh(t_ref) / 2 from the solve; T is exp_tab's table. Returns
// sum_m c_m e^{d_m} (1 + P_m).
__device__ inline double sum_mixed(double nu, double x, const Plan& p, double A, const double* T)
{
    const double e = exp_tab(p.t0, T), ei = recip(e);
    const double q2 = exp_tab(p.h, T), qi2 = recip(q2);
    WalkF w = walkf_begin_exp(nu, x, p.t0, p.h, p.mc, 2.0 * A, e, ei, q2, qi2, exp_tab(-2.0 * nu * p.h, T));
    float s = 0.0f, c = 0.0f, ends = 0.0f;
#pragma unroll 2
    for (int m = 0; m <= p.N; ++m) {
        const float term = __builtin_amdgcn_exp2f((float)walkf_exponent2(w)) * (float)w.Q;
        const float y = term - c;
        const float t = s + y;
        c = (t - s) - y;
        s = t;
        ends += (m == 0 || m == p.N) ? term : 0.0f;
        walkf_step(w);
    }
    return (double)s - (double)c - 0.5 * (double)ends;
}

// ---------------------------------------------------------------------------
// Derivatives of K_nu(x), FP64 (the paper names them as future work, Sec. VI).
// Differentiating the integral of Sec. IV-B under the integral sign:
//   dK/dx  = -int_0^inf cosh t cosh(nu t) e^(-x cosh t) dt,
//   dK/dnu =  int_0^inf t sinh(nu t) e^(-x cosh t) dt =: D.
// Since cosh t cosh(nu t) = (cosh((nu+1)t) + cosh((nu-1)t)) / 2, the first is
// -(K_{nu+1} + K_{nu-1}) / 2 = -(K_{nu-1} + (nu/x) K_nu) (three-term recurrence);
// a sum of two positive integrals of the K kind, so it costs one more K solve at
// order |nu - 1| and no cancellation.
// D has its own window. Its log-integrand
//   d(t) = log t + log sinh(nu t) - x cosh t
// is strictly concave on t > 0 (each term is), tends to -inf at 0 and has one
// maximiser t_d, the zero of d'(t) = 1/t + nu coth(nu t) - x sinh t. At t_d,
// x sinh t_d = 1/t_d + nu coth(nu t_d), which lies in [max(nu, 2/t_d), 2/t_d + nu]
// (coth y >= 1/y, coth y <= 1 + 1/y), so with sinh t <= 1.1752 t on [0, 1]:
//   t_d >= lo = max(asinh(nu/x), min(1, sqrt(1.70/x))),  t_d <= asinh((2/lo + nu)/x).
// Its window is [t0, t1]: t0 is the left end of K's window (left of it the factor
// t tanh(nu t) is below its value at K's peak, so D's integrand is below e^-L of
// its maximum there; when K's window starts at 0 so does D's, and D's integrand
// is even in t, so the trapezoid keeps its accuracy from t = 0), and t1 > t_d the
// root of d(t) = d(t_d) - L. Node terms reuse the K walk: with P = e^(-2 nu t),
//   t sinh(nu t) e^(-x cosh t) = e^(-x) e^Delta e^(nu u - xterm) t (1 - P),
// and Q = 1 - P follows Q' = Q rho + (1 - rho) (rho = e^(-2 nu h)), a recurrence
// that never amplifies Q's relative error.
// ---------------------------------------------------------------------------
// d and its first three derivatives at t > 0:
//   d'   = 1/t + nu coth(nu t) - x sinh t
//   d''  = -1/t^2 - nu^2 csch^2(nu t) - x cosh t
//   d''' = 2/t^3 + 2 nu^3 coth(nu t) csch^2(nu t) - x sinh t
struct DDer {
    double d, d1, d2, d3;
};

__device__ __forceinline__ DDer dnu_derivs(double nu, double x, double t, const double* T)
{
    DDer r;
    const double omp = -expm1(-2.0 * nu * t);        // 1 - e^(-2 nu t)
    const double p = 1.0 - omp;
    const double it = recip(t), io = recip(omp);
    const double cth = (2.0 - omp) * io;               // coth(nu t)
    const double cs2 = 4.0 * p * io * io;              // csch^2(nu t)
    double ch, sh;
    cosh_sinh_tab(t, ch, sh, T);
    r.d = log_tab(t, T) + nu * t + log_tab(omp, T) - kLn2 - x * ch;
    r.d1 = it + nu * cth - x * sh;
    r.d2 = -it * it - nu * nu * cs2 - x * ch;
    r.d3 = 2.0 * it * it * it + 2.0 * nu * nu * nu * cth * cs2 - x * sh;
    return r;
}

// Maximiser t_d of d: Halley on d' inside the bracket above (bisection when a step
// leaves it), stopped once a step is below 1e-7 of t.
__device__ inline double dnu_peak(double nu, double x, const double* T)
{
    double lo = fmax(asinh(nu / x), fmin(1.0, sqrt(1.70 / x)));
    double hi = asinh((2.0 / lo + nu) / x);
    double t = 0.5 * (lo + hi);
    for (int it = 0; it < 100; ++it) {
        const DDer r = dnu_derivs(nu, x, t, T);
        if (r.d1 > 0.0) lo = t; else hi = t;
        const double dt = halley_step(r.d1, r.d2, r.d3);
        double tn = t - dt;
        if (!(fabs(dt) > 1e-7 * t)) { t = fmin(fmax(tn, lo), hi); break; }
        if (!(tn > lo && tn < hi)) tn = 0.5 * (lo + hi);
        t = tn;
        if (hi - lo <= 1e-15 * hi) break;
    }
    return t;
}

// Root t1 > t_d of d(t) = dstar - L by Halley, from acosh(cosh t_d + L/x): there
// the x term alone has dropped by L while log t + log sinh(nu t) grew, so the start
// is left of the root. Iterates are kept in (t_d, t_d + 4 (start - t_d) + 1].
__device__ inline double dnu_window_right(double nu, double x, double td, double chd, double dstar, double L,
                                          const double* T)
{
    double t = acosh(chd + L / x);
    const double tcap = td + 4.0 * (t - td) + 1.0;
    for (int it = 0; it < 64; ++it) {
        const DDer r = dnu_derivs(nu, x, t, T);
        const double dt = halley_step(r.d - dstar + L, r.d1, r.d2);
        double tn = fmin(t - dt, tcap);
        if (!(tn > td)) tn = 0.5 * (t + td);
        const bool done = !(fabs(tn - t) > 1e-5 * t);
        t = tn;
        if (done) break;
    }
    return t;
}

// Plan for D given K's window start t0 (nu > 0, 0 < x < inf). The node step uses
// the strip bound of K with the extra factor of D's integrand on the strip,
// |t + i a| |sinh(nu (t + i a))| / (t sinh(nu t)) <= (1 + a/t) coth(nu t),
// taken at the maximiser with a = pi/2.
__device__ inline Solved dnu_solve(double nu, double x, double t0, double L, double Lq, const RuleTable& R,
                                   const double* T)
{
    const double td = dnu_peak(nu, x, T);
    const DDer r = dnu_derivs(nu, x, td, T);
    double chd, shd;
    cosh_sinh(td, chd, shd);
    const double t1 = dnu_window_right(nu, x, td, chd, r.d, L, T);
    const double extra = log1p(1.5707963267948966 / td) - log(tanh(nu * td));
    return plan_window(nu, x, t0, t1, td, node_step(nu, x, Lq + extra, R));
}

// FP64 trapezoid sum of D's node terms e^(nu u - xterm) t (1 - P).
__device__ inline double sum_dnu_f64(double nu, const Plan& p, double A, double B, const double* T)
{
    Walk w = walk_begin(nu, p);
    double Q = -expm1(-2.0 * nu * p.t0);
    const double omr = -expm1(-2.0 * nu * p.h);
    double S = 0.0, ends = 0.0;
    for (int m = 0; m <= p.N; ++m) {
        const double t = fma((double)m, p.h, p.t0);
        const double term = exp_tab(walk_exponent(w, m, nu, A, B), T) * t * Q;
        S += term;
        if (m == 0 || m == p.N) ends += term;
        walk_step(w, m);
        Q = fma(Q, w.rho, omr);
    }
    return S - 0.5 * ends;
}

// One window and one walk for K, -dK/dx and dK/dnu together: the three integrands differ by
// the factors cosh t and t tanh(nu t), so they share nodes and exponentials.
//  - Right end: the largest of the three. -dK/dx: cosh t grows by at most e^d past tp, so
//    K's bound with the slope nu + 1 (which also covers K). dK/dnu: from td = max(asinh(nu/x),
//    min(1, sqrt(1.70/x))), a point at or left of its maximiser, sinh(nu t) / sinh(nu td) <=
//    (t / td) e^(nu (t - td)), so t sinh(nu t) grows by at most e^((nu + 2/td) d).
//  - Left end: K's (both factors only fall to its left).
//  - Step: the strip bound at order nu + 1 (cosh t cosh(nu t) <= cosh((nu + 1) t)), its
//    target raised by the growth of t sinh(nu t) on the strip, |t + ia| / t times
//    |sinh(nu (t + ia))| / sinh(nu t) <= (1 + a/t)^2 (|sin b| <= b <= (a/t) sinh(nu t) for b =
//    nu a), at td with a = pi/2.
// For plan_wide_ok and L >= 8 (the Newton starts need the x term to outgrow the slopes).
// Returns whether sum_deriv can walk it: e^(2 nu d) over the left side's length d has to be
// finite, or e^(-2 nu t) below 2^-53 of 1 on all of it.
__device__ __forceinline__ bool deriv_fast_ok(double nu, double x, double L, double Lq)
{
    return plan_wide_ok(nu, x, L, Lq) && L >= 8.0;
}

__device__ __forceinline__ bool deriv_window_count(double nu, double x, double L, double Lq, float& t0, float& t1,
                                                   unsigned int& N, unsigned int& mc)
{
    const float nf = (float)nu, xf = (float)x, Lf = (float)L + 0.01f, ix = __builtin_amdgcn_rcpf(xf);
    const float ta = asinh_fast(nf * ix), tp = nf * nf > xf ? ta : 0.0f;
    const float E = exp_fast(tp), Ei = __builtin_amdgcn_rcpf(E);
    const float td = fmaxf(ta, fminf(1.0f, __builtin_amdgcn_sqrtf(1.70f * ix)));
    const float Ed = exp_fast(td), itd = __builtin_amdgcn_rcpf(td);
    const bool large = large_pair(nf, xf);
    auto ends = [&](auto any) {
        t1 = fmaxf(tp + right_end_fast<any.value>(tp, E, Ei, xf, nf + 1.0f, Lf, large),
                   td + right_end_fast<any.value>(td, Ed, __builtin_amdgcn_rcpf(Ed), xf, fmaf(2.0f, itd, nf), Lf, large));
        t0 = left_end_fast<any.value>(tp, E, Ei, nf, xf, Lf, large);
    };
    const bool any = __any(large);
    if (__builtin_expect(any, 0)) ends(std::true_type{});
    else ends(std::false_type{});
    const float extra = 2.0f * 0.69314718f * __builtin_amdgcn_logf(fmaf(1.5707963f, itd, 1.0f));
    node_grid(t0, t1, tp, node_step_fast(nf + 1.0f, xf, (float)Lq + extra), N, mc);
    if (!any && Lf <= 250.0f) return true;          // d <= (L + ln 2 + nu) / nu
    return 2.0f * nf * (t1 - t0) * (float)mc < 699.0f * (float)N || 2.0f * nf * t0 >= 40.0f;
}

// Trapezoid sums of the paired walk (sum_f64): of the K terms e^d (2 - Q), of those times
// x (cosh t - cosh t_ref), and of e^d t Q, Q = 1 - e^(-2 nu t). Q is formed from its value at
// t_ref by sums that keep its relative accuracy where it is small (small nu or t): right
// Q' = Q rho + (1 - rho), left Q = Q_ref - P_ref expm1(2 nu j h).
struct DerivSums {
    double k, x, d;
};

__device__ inline DerivSums sum_deriv(double nu, double x, const Plan& p, double E, double Ei, double Sr, const double* T)
{
    const int nr = p.N - p.mc, nl = p.mc, jmax = nr > nl ? nr : nl;
    const double h = p.h, nh = nu * h;
    // e^(2 nu h) - 1, e^(-2 nu h) and 1 less that, each to its own relative accuracy
    const double qh = expm1(fmin(2.0 * nh, 700.0)), rho = recip(1.0 + qh), omr = qh * rho;
    // where the powers of e^(2 nu h) leave the double range Q is 1 on the left
    const double qe = 2.0 * nh * nl < 700.0 ? qh : 0.0, re = 1.0 + qe;
    const double Qr = -expm1(-2.0 * nu * p.tref), Pr = exp_tab(-2.0 * nu * p.tref, T);
    double QR = Qr, EL = 0.0, jd = 1.0;
    CoshPair<true> W(x, h, E, Ei, Sr);
    DerivSums S = {0.0, 0.0, 0.0}, r = {0.0, 0.0, 0.0}, l = {0.0, 0.0, 0.0};
    for (int j = 1; j <= jmax; ++j) {
        QR = fma(QR, rho, omr);
        EL = fma(EL, re, qe);
        if (j <= nr) {
            const double e = exp_node(fma(jd, nh, -W.R.X), T);
            r.k = fma(-e, QR, 2.0 * e);
            r.x = r.k * W.R.X;
            r.d = e * QR * fma(jd, h, p.tref);
            S.k += r.k;
            S.x += r.x;
            S.d += r.d;
        }
        if (j <= nl) {
            const double e = exp_node(fma(-jd, nh, -W.L.X), T), Q = fma(-Pr, EL, Qr);
            l.k = fma(-e, Q, 2.0 * e);
            l.x = l.k * W.L.X;
            l.d = e * Q * fma(-jd, h, p.tref);
            S.k += l.k;
            S.x += l.x;
            S.d += l.d;
        }
        W.step();
        jd += 1.0;
    }
    // trapezoid ends: half of node N and of node 0 (the reference's weight if it is one)
    const double w0 = nl == 0 || nr == 0 ? 0.5 : 1.0;
    S.k = fma(w0, 2.0 - Qr, fma(-0.5, r.k + l.k, S.k));
    S.x = fma(-0.5, r.x + l.x, S.x);
    S.d = fma(w0, Qr * p.tref, fma(-0.5, r.d + l.d, S.d));
    return S;
}

// The sums of one entry by kLanes neighbouring lanes (lane sub takes the nodes mc +- j, j =
// sub + 1, sub + 1 + kLanes, ...), for kernels with few entries, whose time is the walk's
// serial chain: k as sum_f64 and, with kDnu, d as sum_deriv. Every lane gets the totals.
template <int kLanes, bool kDnu>
__device__ inline DerivSums sum_split(double nu, double x, const Plan& p, double E, double Ei, double Sr, int sub,
                                      const double* T)
{
    const int nr = p.N - p.mc, nl = p.mc, jmax = nr > nl ? nr : nl;
    const double h = p.h, xh = 0.5 * x, nh = nu * h;
    double qm1 = h <= 0.25 ? expm1_small(0.5 * h) : expm1(0.5 * h), q = qm1 + 1.0, qi = recip(q);
    double rho = exp_tab(-2.0 * nh, T), rhoi = recip(rho);
    const double Pr = exp_tab(-2.0 * nu * p.tref, T), Qr = kDnu ? -expm1(-2.0 * nu * p.tref) : 0.0;
    double omr = kDnu ? -expm1(-2.0 * nh) : 0.0, qe = omr * rhoi;       // 1 - e^(-2 nu h), e^(2 nu h) - 1
    double V = 0.0, Bq = 1.0, SR = Sr, ER = Ei, PR = Pr, PL = Pr, QR = Qr, EL = 0.0;
    auto step = [&]() {
        V = fma(V, q, qm1);
        Bq *= qi;
        SR = fma(SR, q, qm1);
        ER *= qi;
        PR *= rho;
        PL *= rhoi;
        if (kDnu) {
            QR = fma(QR, 1.0 - omr, omr);
            EL = fma(EL, 1.0 + qe, qe);
        }
    };
    for (int k = 0; k <= sub; ++k) step();
#pragma unroll
    for (int k = 1; k < kLanes; k *= 2) {                               // the factors of kLanes nodes
        qm1 = qm1 * (qm1 + 2.0);
        q = qm1 + 1.0;
        qi *= qi;
        rho *= rho;
        rhoi *= rhoi;
        if (kDnu) {
            omr = omr * (2.0 - omr);
            qe = qe * (qe + 2.0);
        }
    }
    DerivSums S = {0.0, 0.0, 0.0};
    const double w0 = nl == 0 || nr == 0 ? 0.5 : 1.0;
    if (sub == 0) {
        S.k = w0 * (1.0 + Pr);
        S.d = w0 * Qr * p.tref;
    }
    for (int j = sub + 1; j <= jmax; j += kLanes) {
        const double jd = (double)j, nuu = jd * nh;
        const double xs = xh * fma(V, Bq, V);
        if (j <= nr) {
            double e = exp_node(fma(-xs, fma(SR, ER, SR), nuu), T);
            if (j == nr) e *= 0.5;
            S.k += fma(e, PR, e);
            if (kDnu) S.d += e * QR * fma(jd, h, p.tref);
        }
        if (j <= nl) {
            double e = exp_node(fma(xs, fma(E, Bq, -Ei * (V + 1.0)), -nuu), T);
            if (j == nl) e *= 0.5;
            S.k += fma(e, PL, e);
            if (kDnu) S.d += e * fma(-Pr, EL, Qr) * fma(-jd, h, p.tref);
        }
        step();
    }
#pragma unroll
    for (int k = 1; k < kLanes; k *= 2) {
        S.k += __shfl_xor(S.k, k, 64);
        if (kDnu) S.d += __shfl_xor(S.d, k, 64);
    }
    return S;
}

// dK/dnu alone: delta and h S of its integral (K's start t0 for the exact solve).
__device__ __forceinline__ void dnu_integral(double nu, double x, double t0, double L, double Lq, const RuleTable& R,
                                             const double* T, double& delta, double& hs)
{
    float a, b;
    unsigned int N, mc;
    if (!deriv_fast_ok(nu, x, L, Lq) || !deriv_window_count(nu, x, L, Lq, a, b, N, mc)) {
        const Solved sd = dnu_solve(nu, x, t0, L, Lq, R, T);
        delta = sd.delta;
        hs = sd.p.h * sum_dnu_f64(nu, sd.p, sd.A, sd.B, T);
        return;
    }
    const Solved s = plan_setup(nu, x, a, b, N, mc);
    delta = s.delta;
    hs = s.p.h * sum_deriv(nu, x, s.p, s.E, s.Ei, s.Sr, T).d;
    hs = fma(hs, s.dlo, hs);
}

// ---------------------------------------------------------------------------
// The paper's refined algorithm, integral branch (Sec. IV-C, Alg. 2): fixed
// window [0, T], b bins, nodes t_m = m h (h = T / b), weights 1/2 at both ends,
// scaled by the largest node value. g is unimodal on t >= 0, so the sum is taken
// relative to the node nearest t* (within one node of the largest) with the
// cancellation-free walk of the plain form: one FP64 exponential and a few
// multiplies per node instead of evaluating g at every node. b may run to the
// thousands, so the walk's multiplicative state is re-seeded from closed forms
// every kReseed nodes (its rounding drift grows with the steps taken) and long
// sums are compensated. The scale factors out of the sum: K = exp(lscale) hs.
// ---------------------------------------------------------------------------
struct FixedOut {
    double lscale;   // log of the factor taken out of the sum
    double hs;       // h * sum_m c_m exp(nu u_m - xterm_m) (1 + P_m), the walk's terms
};

constexpr int kReseed = 32;

// Walk state at node m from closed forms (u = (m - mc) h, V = expm1(|u| / 2)).
__device__ inline void walk_reseed(Walk& w, const Plan& p, double nu, int m)
{
    const int k = m - p.mc;
    w.k = (double)k;
    w.V = expm1(0.5 * p.h * (double)(k < 0 ? -k : k));
    const double big = w.V + 1.0, small = recip(big);
    w.Bw = (k <= 0) ? small : big;                // e^(u/2)
    w.Bb = (k <= 0) ? big : small;                // e^(-u/2)
    w.P = exp(-2.0 * nu * (p.t0 + (double)m * p.h));
}

// Trapezoid sum of the fixed window on the re-seeded walk; Kahan-compensated when
// Comp (b beyond kFixedPlainMax nodes, where plain FP64 accumulation error grows
// past the walk's own).
constexpr int kFixedPlainMax = 256;

template <bool Comp>
__device__ inline double fixed_sum(double nu, const Plan& p, double A, double B, const double* T)
{
    Walk w = walk_begin(nu, p);
    double S = 0.0, c = 0.0, ends = 0.0;
    for (int m = 0; m <= p.N; ++m) {
        if (m > 0 && m % kReseed == 0) walk_reseed(w, p, nu, m);
        const double term = exp_tab(walk_exponent(w, m, nu, A, B), T) * (1.0 + w.P);
        if (Comp) {
            const double y = term - c, t = S + y;
            c = (t - S) - y;
            S = t;
        } else {
            S += term;
        }
        if (m == 0 || m == p.N) ends += term;
        walk_step(w, m);
    }
    return (S - c) - 0.5 * ends;
}

__device__ inline FixedOut paper_fixed(double nu, double x, int bins, double T, const double* E)
{
    const double tstar = (nu * nu > x) ? peak_solve(nu, x, E) : 0.0;
    Plan p;
    p.t0 = 0.0;
    p.h = T / (double)bins;
    p.N = bins;
    p.mc = (int)fmin(fmax(rint(tstar / p.h), 0.0), (double)bins);
    p.tref = (double)p.mc * p.h;
    double ch, sh;
    cosh_sinh(p.tref, ch, sh);
    const double em = expm1(0.5 * p.tref);               // sinh(t/2) = em (em + 2) / (2 (em + 1))
    const double sh2 = em * (em + 2.0) / (2.0 * (em + 1.0));
    const double A = 0.5 * x * ch, B = 0.5 * x * sh;
    FixedOut o;
    o.lscale = nu * p.tref - kLn2 - 2.0 * x * sh2 * sh2 - x;
    o.hs = p.h * (bins > kFixedPlainMax ? fixed_sum<true>(nu, p, A, B, E) : fixed_sum<false>(nu, p, A, B, E));
    return o;
}

// ---------------------------------------------------------------------------
// Temme's series for small x (Sec. IV-A, Eqs. "temme_main", "temme_initpq",
// "temme_initf") with Campbell's forward recurrence (Eq. "recurrence"), the
// paper's branch for x < 0.1 (Alg. 2). With nu = mu + M, M = floor(nu + 1/2),
// mu in [-1/2, 1/2):
//   K_mu = sum_k c_k f_k,  K_{mu+1} = (2/x) sum_k c_k h_k,  c_k = (x^2/4)^k / k!,
//   h_k = p_k - k f_k,  p_k = p_{k-1} / (k - mu),  q_k = q_{k-1} / (k + mu),
//   f_k = (k f_{k-1} + p_{k-1} + q_{k-1}) / (k^2 - mu^2),
//   p_0 = (x/2)^-mu Gamma(1+mu) / 2,  q_0 = (x/2)^mu Gamma(1-mu) / 2,
//   f_0 = (mu pi / sin(mu pi)) (cosh(s) Gamma1 + sinh(s)/s ln(2/x) Gamma2),
//   s = mu ln(2/x), Gamma1 = (1/Gamma(1-mu) - 1/Gamma(1+mu)) / (2 mu),
//   Gamma2 = (1/Gamma(1-mu) + 1/Gamma(1+mu)) / 2,
// then K_{eta+1} = (2 eta / x) K_eta + K_{eta-1} up to nu. Gamma1 and Gamma2 are
// even entire functions of mu, evaluated by their Taylor series in mu^2 (kTemmeTab).
// c_k f_k falls faster than (x^2/4)^k / k!^2: five terms leave below 1e-19 of the sum at
// x = 0.1 (the paper caps the series at 15000 terms).
// ---------------------------------------------------------------------------

// K_nu(x) for 0 < x < 0.1; returns K (not scaled). One reciprocal a term: p and q take their divisors
// k -+ mu from that of k^2 - mu^2, 1/Gamma(1 + mu) and 1/Gamma(1 - mu) give pi mu /
// sin(pi mu) = Gamma(1 + mu) Gamma(1 - mu), and 2/x serves the logarithm, the series and
// the recurrence, whose M factors of its rounding are taken out at the end.
__device__ inline double temme_k(double nu, double x, const TemmeCoef& C, const double* T)
{
    const double M = floor(nu + 0.5);
    const double mu = nu - M, mu2 = mu * mu;
    double G1 = C.g1[kTemmeTerms - 1], G2 = C.g2[kTemmeTerms - 1];
#pragma unroll
    for (int j = kTemmeTerms - 2; j >= 0; --j) {
        G1 = fma(G1, mu2, C.g1[j]);
        G2 = fma(G2, mu2, C.g2[j]);
    }
    const double rgp = G2 - mu * G1;                   // 1 / Gamma(1 + mu)
    const double rgm = G2 + mu * G1;                   // 1 / Gamma(1 - mu)
    const double ix = 2.0 / x;
    const double lx = log(ix);
    const double sg = mu * lx, s2 = sg * sg;
    const double fact = recip(rgp * rgm);              // pi mu / sin(pi mu)
    const double esg = exp_wide(sg, T), esi = recip(esg);
    const double chs = 0.5 * (esg + esi);
    // sinh(s) / s: the series below 0.3 (truncation 1e-17)
    const double ser = fma(fma(fma(fma(fma(s2, 1.0 / 39916800.0, 1.0 / 362880.0), s2, 1.0 / 5040.0), s2, 1.0 / 120.0),
                               s2, 1.0 / 6.0), s2, 1.0);
    const double shs_s = fabs(sg) < 0.3 ? ser : 0.5 * (esg - esi) * recip(sg);
    double f = fact * (G1 * chs + G2 * shs_s * lx);
    double p = 0.5 * esg * (rgm * fact);               // (x/2)^-mu Gamma(1+mu) / 2
    double q = 0.5 * esi * (rgp * fact);               // (x/2)^mu Gamma(1-mu) / 2
    const double d = 0.25 * x * x;
    double c = 1.0, sum = f, sum1 = p;
#pragma unroll
    for (int k = 1; k <= 5; ++k) {
        const double kk = (double)k;
        const double r = recip(fma(kk, kk, -mu2));
        f = (kk * f + p + q) * r;
        c *= d * (1.0 / kk);
        p *= (kk + mu) * r;
        q *= (kk - mu) * r;
        sum = fma(c, f, sum);
        sum1 = fma(c, p - kk * f, sum1);
    }
    double km = sum;                                   // K_mu
    double kp = sum1 * ix;                             // K_{mu+1}
    // forward recurrence K_{eta+1} = (2 eta / x) K_eta + K_{eta-1}, eta = mu + 1, ..., nu - 1
    for (int j = 1; j < (int)M; ++j) {
        const double kn = fma((mu + (double)j) * ix, kp, km);
        km = kp;
        kp = kn;
    }
    if (M < 1.0) return km;
    // kp grows as ix^M (its other term is below x^2 / 4 of it): ix = (2/x)(1 - e). An overflowed
    // kp stays infinite.
    return kp < __builtin_inf() ? fma(kp, M * (0.5 * fma(-x, ix, 2.0)), kp) : kp;
}

}  // namespace bk
