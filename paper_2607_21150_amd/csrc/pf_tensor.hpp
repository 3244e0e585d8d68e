// Pointwise functions of the FP64 applies in tensor form: trial log strain, return
// mapping, tangent and its transpose without a principal frame.
//
// With b_tr = m (I + S), m = tr b_tr / 3 and S traceless, the deviatoric trial log strain
// is an isotropic function of S. As log x is an integral of 1 / (1 + T) - 1 / (x + T) over T > 0,
//     e = p0 S - p1 M,    M = dev K,    K = adj(I + S),
//     p0 = (1/2) int 1 / D,   p1 = (1/2) int T / D,   n_k = (1/2) int T^k / D^2  (k = 2, 3, 4),
//     D(T) = det(I + T (I + S)) = 1 + 3 T + I2 T^2 + I3 T^3,
// moments of one sign that depend on the invariants I2 = 3 - J2 and I3 = 1 - J2 + J3 of I + S only (J2 =
// tr S^2 / 2, J3 = det S). Nothing is divided by a difference of eigenvalues, so repeated eigenvalues
// need no case of their own. With dK = S dS + dS S - dS up to a multiple of I and D's derivatives,
// the strain's derivative (Appendices A-B) is
//     de = (p0 + p1) dS - p1 dev(S dS + dS S) + (n2 a - n3 b) S + (n4 b - n3 a) M,
// a = S:dS, b = M:dS, a self-adjoint map of dS (the transpose uses it again). The products of e come from
// S:S = 2 J2, S:M = 3 J3 - 2 J2 = 3 I3 - I2 and M:M = (2/3) I2^2 - 6 I3, and M S = -M - (I2 / 3) S + ... I.
//
// S resolves the large eigenvalues and M the small ones, and their terms don't cancel; with S and
// dev S^2 = M + S instead, coefficients that grow as 1 / x to 1 / x^3 cancel where two eigenvalues of I + S are of
// the order of x, at the ratio of the eigenvalues squared times the rounding: the Jacobian was off by 4e-11 at
// an isochoric stretch of 9 and by 6e-9 at 20, now by 3e-14 and 3e-13 (2e-14 to 4e-13 with a principal frame,
// by the orientation of the stretch).
//
// The FP64 applies are bound by VALU issue. The principal form (eigenvalues, an orthonormal
// frame with polish rotations, three logarithms, divided differences, the tangent rotated
// there and back) took 1,152 vector instructions per order-3 element in the Jacobian beside its
// 93 matrix-core ones; this form takes 721, and 168 registers (3 waves per SIMD, 1 or 2 spilled) instead of
// 217. Order-3 Jacobian on 48^3 elements 0.465 -> 0.372 ms, with two extra branches on 32^3
// 0.310 -> 0.237, order 4 on 40^3 0.644 -> 0.560, order 2 on 32^3
// 0.097 -> 0.088. The linearisation record and the state commit keep the principal form (their
// data are principal).
#pragma once
#include <hip/hip_runtime.h>

#include "pf_qf.hpp"

namespace pfmf {

// The point's state for the residual, the tangent and its transpose. Symmetric tensors are
// {xx, yy, zz, yz, xz, xy}.
struct TState {
  double Fi[9];               // F^-1
  double S[6], M[6];          // b_tr / m - I and dev adj(b_tr / m)
  double ss, sm, mm;          // S:S, S:M, M:M
  double p0, p1, n2, n3, n4;  // moments of the header comment
  double ee, theta;           // e:e and tr eps
  double g, gp, c, kq, kphi;  // degradation, return factor and its tangent (as in QPState)
  double psi, H, L, dLcoef, ddg_s0, ddg_visc, dg;
  bool tension, hactive, plastic, bad;
};

// Up to this J2 every |s_i| <= 2 sqrt(J2 / 3) is at most 0.1 (principal log strains within 5 %
// of their mean): the coefficients are sums of 13 terms there, 46 multiply-adds in all.
constexpr double LOG_SERIES_J2 = 0.0075;

// The moments for J2 <= LOG_SERIES_J2. With f(s) = log(1 + s) / 2 = sum_n f_n s^n, the Cayley-Hamilton theorem
// (S^n = h_{n-2} S^2 + h_{n-1} S + ..., h_n = J2 h_{n-2} + J3 h_{n-3}) gives e = c1 S + c2 dev S^2 with c1 = sum f_n
// h_{n-1} = p0 + p1 and c2 = sum f_n h_{n-2} = -p1, and the derivatives g3 = dc1/dJ2 = n2 + 2 n3 + n4, g4 = dc1/dJ3 =
// dc2/dJ2 = -(n3 + n4) and g5 = dc2/dJ3 = n4. f' = 1 / (2 (1 + s)) is
// interpolated at 13 Chebyshev nodes of [-0.1, 0.1] and integrated (relative error of f and of
// f' below 4e-17), summed downwards: b_k = sum_n f_n h_{n-k} and q_k = sum_n f_n d_{n-k}, h_n and
// d_n the coefficients of 1 / (1 - J2 t^2 - J3 t^3) and of its square.
template <bool TAN>
__device__ inline void log_series(double J2, double J3, TState& s) {
  constexpr int N = 13;
  constexpr double f[N + 1] = {0.0,
                               0.5,
                               -0.24999999999999917,
                               0.16666666666666613,
                               -0.12500000000114728,
                               0.10000000000091781,
                               -0.08333333272200438,
                               0.07142857090457519,
                               -0.06250015693704912,
                               0.05555569505515478,
                               -0.04997913947686155,
                               0.04543558134260141,
                               -0.04304835441590142,
                               0.03973694253775516};
  double b[N + 4], q[N + 4];
  b[N + 1] = b[N + 2] = b[N + 3] = 0.0;
  q[N + 1] = q[N + 2] = q[N + 3] = 0.0;
#pragma unroll
  for (int k = N; k >= 1; --k) {
    const double fk = k == 1 ? f[k] : kst(f[k]);
    b[k] = k + 2 <= N ? fma(J2, b[k + 2], fk) : fk;
    if (k + 3 <= N) b[k] = fma(J3, b[k + 3], b[k]);
    if (TAN && k >= 3) {
      q[k] = k + 2 <= N ? fma(J2, q[k + 2], b[k]) : b[k];
      if (k + 3 <= N) q[k] = fma(J3, q[k + 3], q[k]);
    }
  }
  s.p0 = b[1] + b[2];
  s.p1 = -b[2];
  if (TAN) {
    s.n2 = q[3] + 2.0 * q[4] + q[5];
    s.n3 = -(q[4] + q[5]);
    s.n4 = q[5];
  }
}

// The same for any positive definite I + S, I2 and I3 given.
// With the eigenvalues in [l, u] and T = t / sqrt(l u) the integrands depend on
// the ratio u / l alone, for which a rule of n nodes is enough up to a limit: Gauss-Legendre nodes
// v mapped by t / (1 + t) = (1 + tanh(c v) / tanh(c)) / 2, c (0.096, 0.355, 0.683, 0.947, 1.207, 1.673) chosen
// per rule for the widest range in which the moments of D^-2 are exact to 1.5e-16 over all triples
// of eigenvalues. The moments of D^-1 (all that the residual takes) converge faster and have wider
// limits, to 2e-17; the tangent takes them from those of D^-2, by the integrals of (T / D)' and
// (T^2 / D)'. A rule is symmetric under t -> 1 / t: half of its nodes {t, weight} are listed.
constexpr int LOG_RULES = 6;
constexpr int LOG_FIRST[LOG_RULES + 1] = {0, 4, 10, 18, 28, 40, 56};  // node pairs of a rule: 8, 12, 16, 20, 24, 32 nodes
constexpr float LOG_RATIO[2][LOG_RULES] = {{1.72f, 5.4f, 21.9f, 74.f, 245.f, 2180.f},
                                           {1.45f, 4.2f, 16.f, 53.f, 155.f, 1250.f}};
// Ratio beyond which K is taken from F^-1 and I + D: adj(I + S) from S holds K's small entries with the rounding
// of its large terms, which p1 multiplies by the ratio.
constexpr float LOG_WIDE = 8.f;
constexpr double LOG_HALF[LOG_FIRST[LOG_RULES]][2] = {
    {0.020138255037087625, 0.026194290990111748},
    {0.11262061675326468, 0.068631810355546441},
    {0.31001587292394411, 0.1346614192413006},
    {0.68921944851820094, 0.25943998725634648},
    {0.0085801794734985393, 0.011094388123626248},
    {0.046724746578257009, 0.02757252205050631},
    {0.12196543372248697, 0.048742857328326138},
    {0.24760474821808001, 0.078873258746406619},
    {0.44823409766569228, 0.12538109951720797},
    {0.76934045848401589, 0.20271518284789292},
    {0.0039837365284311017, 0.0051449781680020573},
    {0.021580838737189138, 0.012653711885053317},
    {0.055761410978053615, 0.021919730069819433},
    {0.11133128832960038, 0.034312758758648754},
    {0.19639815617166972, 0.051818402015395872},
    {0.3240045946317136, 0.077483291115063205},
    {0.51497953928343465, 0.11623031597206854},
    {0.80311204340820996, 0.17647310117814724},
    {0.0020173360113880105, 0.0026032502760562461},
    {0.010889950058838437, 0.0063582924339478063},
    {0.027958590317377068, 0.010880634648877729},
    {0.055300289937880713, 0.016741651505975882},
    {0.096335153581969285, 0.024728649914141598},
    {0.15637114777502886, 0.035967074411776198},
    {0.24345216595420965, 0.052104796077011059},
    {0.36966563675320629, 0.075596627074520695},
    {0.55318213433546937, 0.11017080684629943},
    {0.82154155346127311, 0.16164993502753211},
    {0.0010539063871771242, 0.0013592389093590852},
    {0.0056755085344818799, 0.0033042116564926021},
    {0.014508587549275018, 0.0056082977409746028},
    {0.028521034340004813, 0.0085339071464631093},
    {0.049292778730376657, 0.012437077600069967},
    {0.07924964199509639, 0.017817795215835586},
    {0.12201967756557056, 0.025392550189777496},
    {0.18296259353024077, 0.036196664998377134},
    {0.26994438624939032, 0.051729979807706973},
    {0.39446411585716096, 0.074168108560173113},
    {0.57330003875899016, 0.10667963281595669},
    {0.83095723934735877, 0.15392875119826072},
    {0.00032437570271627521, 0.0004179485900133064},
    {0.0017396178062583591, 0.0010077492945685673},
    {0.0044141370533642829, 0.0016862601896185246},
    {0.0085850190398862984, 0.0025159539434861707},
    {0.014633079476964949, 0.0035793332063693071},
    {0.02313240282327499, 0.0049892846701197766},
    {0.034925461200309961, 0.0069043034428476983},
    {0.051234607367938452, 0.0095500114878653997},
    {0.07382500316861039, 0.013249574111753834},
    {0.10524005999030583, 0.018466441295668542},
    {0.14913824556346861, 0.025863788477475346},
    {0.21076993860200688, 0.036386142154583558},
    {0.29764531999690569, 0.051370086030583802},
    {0.42046005948396731, 0.072693119112912305},
    {0.59436735518174, 0.10297388358530327},
    {0.84071897169437415, 0.14584573103004089},
};
// A pair of nodes t and 1 / t, each with its weight times t^0, ..., t^4.
struct LogPair {
  double t[2], w[2][5];
};
struct LogPairs {
  LogPair p[LOG_FIRST[LOG_RULES]];
};
constexpr LogPairs log_pairs() {
  LogPairs r{};
  for (int k = 0; k < LOG_FIRST[LOG_RULES]; ++k)
    for (int h = 0; h < 2; ++h) {
      const double t = LOG_HALF[k][0];
      r.p[k].t[h] = h ? 1.0 / t : t;
      double w = h ? LOG_HALF[k][1] / (t * t) : LOG_HALF[k][1];
      for (int j = 0; j < 5; ++j, w *= r.p[k].t[h]) r.p[k].w[h][j] = w;
    }
  return r;
}

// Bounds u and 1 / l of the eigenvalues from the invariants by a step of Laguerre's iteration from infinity
// and from 0, which stays outside the roots of a cubic with real roots (l is at least 3/4 of the smallest).
struct LogBounds {
  float u, il;
};
__device__ inline LogBounds log_bounds(double I2, double I3) {
  const float i2 = (float)I2, i3 = (float)I3;
  return LogBounds{1.f + 2.f * __builtin_amdgcn_sqrtf(fmaxf(1.f - i2 * (1.f / 3.f), 0.f)),
                   (i2 + 2.f * __builtin_amdgcn_sqrtf(fmaxf(i2 * i2 - 9.f * i3, 0.f))) * frcp(3.f * i3)};
}

struct LogMoments {
  double p0, p1, n2, n3, n4;
};

// The wave takes one rule, the shortest that serves all its lanes here, so that its nodes are in scalar
// registers: 24 vector instructions per pair of nodes with the tangent, 18 without. Order-3 Jacobian on 24^3
// elements (0.059 ms at strains of 1 %) at isochoric stretches of 1.5, 2, 3 and 5: 0.060, 0.060, 0.061 and
// 0.068 ms; with a principal frame 0.072 to 0.073, and with 12 Gauss nodes in t / (1 + t) on panels that
// halve towards 1 (one per factor 2 of a loose lower bound) 0.083, 0.104, 0.135 and 0.178.
template <bool TAN>
__device__ inline LogMoments log_moments(double I2, double I3, const LogBounds& bd) {
  const float ratio = bd.u * bd.il;
  LogMoments m{0.0, 0.0, 0.0, 0.0, 0.0};
  if (ratio <= LOG_RATIO[TAN][LOG_RULES - 1]) {
    static constexpr LogPairs pairs = log_pairs();
    int rule = 0;
    while (rule < LOG_RULES - 1 && __ballot(ratio > LOG_RATIO[TAN][rule])) ++rule;  // uniform
    const double ia = (double)frsqrt(bd.u * frcp(bd.il)), ia2 = ia * ia;
    const double a1 = 3.0 * ia, a2 = I2 * ia2, a3 = I3 * ia2 * ia;  // D = 1 + a1 t + a2 t^2 + a3 t^3
    double m0 = 0.0, m1 = 0.0, m2 = 0.0, m3 = 0.0;  // moments t^k / D, or t^(k + 1) / D^2 with TAN
#pragma unroll 1
    for (int k = LOG_FIRST[rule]; k < LOG_FIRST[rule + 1]; ++k) {
      const LogPair& p = pairs.p[k];
      const double d0 = fma(p.t[0], fma(p.t[0], fma(p.t[0], a3, a2), a1), 1.0);
      const double d1 = fma(p.t[1], fma(p.t[1], fma(p.t[1], a3, a2), a1), 1.0);
      const double r = frcp(d0 * d1);
      const double i0 = r * d1, i1 = r * d0;
      if (TAN) {
        const double q0 = i0 * i0, q1 = i1 * i1;
        m0 = fma(p.w[1][1], q1, fma(p.w[0][1], q0, m0));
        m1 = fma(p.w[1][2], q1, fma(p.w[0][2], q0, m1));
        m2 = fma(p.w[1][3], q1, fma(p.w[0][3], q0, m2));
        m3 = fma(p.w[1][4], q1, fma(p.w[0][4], q0, m3));
      } else {
        m0 = fma(p.w[1][0], i1, fma(p.w[0][0], i0, m0));
        m1 = fma(p.w[1][1], i1, fma(p.w[0][1], i0, m1));
      }
    }
    if (TAN) {
      const double ia3 = ia2 * ia;
      m.n2 = ia3 * m1;
      m.n3 = ia3 * ia * m2;
      m.n4 = ia3 * ia2 * m3;
      m0 = fma(a1, m0, fma(2.0 * a2, m1, 3.0 * a3 * m2));
      m1 = 0.5 * fma(a1, m1, fma(2.0 * a2, m2, 3.0 * a3 * m3));
    }
    m.p0 = ia * m0;
    m.p1 = ia2 * m1;
  } else {
    // wider still: over t = T / (1 + T) in [0, 1], 12 Gauss nodes on panels that halve towards t = 1, the last
    // one no longer than the distance of the pole beyond it (the error of the rule is then below
    // 1e-17), E(t) = (1 - t)^3 D in powers of t and 1 - t
    constexpr int NG = 12;
    static constexpr double xg[NG / 2] = {0.009219682876640375, 0.04794137181476257, 0.11504866290284765,
                                          0.2063410228566913,   0.3160842505009099,  0.43738329574426554};
    static constexpr double wg[NG / 2] = {0.023587668193255914, 0.05346966299765921, 0.08003916427167311,
                                          0.10158371336153296,  0.1167462682691774,  0.12457352290670139};
    // l with a margin for its rounding, or where FP32 does not reach it, that the other two have at
    // most the mean (3 - l) / 2
    const double lam = fmax(kst(4.0 / 9.0) * I3, (double)(0.999f * frcp(bd.il)));
    double t0 = 0.0, h = 1.0;
    for (int panel = 0; panel < 64; ++panel) {
      const bool last = h * (1.0 - lam) <= lam || panel == 63;
      const double hp = last ? h : 0.5 * h;
#pragma unroll 1
      for (int k = 0; k < NG; ++k) {
        const double x = k < NG / 2 ? xg[k] : 1.0 - xg[NG - 1 - k], wk = wg[k < NG / 2 ? k : NG - 1 - k];
        const double t = fma(hp, x, t0), r = (1.0 - t0) - hp * x;
        const double iE = frcp(fma(t * t, fma(t, I3, r * I2), r * r * fma(2.0, t, 1.0)));
        const double w = 0.5 * hp * wk * iE;
        m.p0 = fma(w, r, m.p0);
        m.p1 = fma(w, t, m.p1);
        if (TAN) {
          const double v = w * iE * t * t;
          m.n2 = fma(v * r, r, m.n2);
          m.n3 = fma(v * r, t, m.n3);
          m.n4 = fma(v * t, t, m.n4);
        }
      }
      if (last) break;
      t0 += hp;
      h = hp;
    }
  }
  return m;
}

// Y = S D + D S of symmetric traceless S and D: with a zero trace S_ii + S_jj = -S_kk.
__device__ inline void sym_anticommutator(const double* S, const double* D, double* Y) {
  Y[0] = 2.0 * (S[0] * D[0] + S[5] * D[5] + S[4] * D[4]);
  Y[1] = 2.0 * (S[5] * D[5] + S[1] * D[1] + S[3] * D[3]);
  Y[2] = 2.0 * (S[4] * D[4] + S[3] * D[3] + S[2] * D[2]);
  Y[3] = S[5] * D[4] + S[4] * D[5] - (S[0] * D[3] + S[3] * D[0]);
  Y[4] = S[5] * D[3] + S[3] * D[5] - (S[1] * D[4] + S[4] * D[1]);
  Y[5] = S[4] * D[3] + S[3] * D[4] - (S[2] * D[5] + S[5] * D[2]);
}

// Frobenius product of two symmetric tensors.
__device__ inline double sym_dot(const double* a, const double* b) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2] + 2.0 * (a[3] * b[3] + a[4] * b[4] + a[5] * b[5]);
}

// A tensor as c1 D + c2 dev(S D + D S) + a S + b M of the point's S and M and a traceless D.
struct LogMap {
  double c1, c2, a, b;
};

// The S coefficient of (p0 + p1) e - p1 dev(S e + e S), p0^2 - p0 p1 - (2/3) I2 p1^2; that of M is -3 p1 (p0 + p1).
__device__ inline double log_eS(const TState& s) {
  return s.p0 * (s.p0 - s.p1) - s.p1 * s.p1 * fma(kst(-1.0 / 3.0), s.ss, 2.0);
}

// L(dS) of the header comment, a = S:dS and b = M:dS given; ede = e:de.
__device__ inline LogMap log_tangent(const TState& s, double a, double b, double& ede) {
  const LogMap m{s.p0 + s.p1, -s.p1, s.n2 * a - s.n3 * b, s.n4 * b - s.n3 * a};
  ede = log_eS(s) * a - 3.0 * s.p1 * m.c1 * b + m.a * (s.p0 * s.ss - s.p1 * s.sm) + m.b * (s.p0 * s.sm - s.p1 * s.mm);
  return m;
}

// out = the tensor of m for D with S:D = SD.
__device__ inline void log_expand(const TState& s, const LogMap& m, const double* D, double SD, double* out) {
  double Y[6];
  sym_anticommutator(s.S, D, Y);
  const double tr = kst(2.0 / 3.0) * m.c2 * SD;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    double v = m.c1 * D[k] + m.c2 * Y[k] + m.a * s.S[k] + m.b * s.M[k];
    if (k < 3) v -= tr;
    out[k] = v;
  }
}

// Row-major 3x3 times symmetric: M = A B.
__device__ inline void mul_sym(const double* A, const double* B, double* M) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const double a0 = A[3 * i], a1 = A[3 * i + 1], a2 = A[3 * i + 2];
    M[3 * i + 0] = a0 * B[0] + a1 * B[5] + a2 * B[4];
    M[3 * i + 1] = a0 * B[5] + a1 * B[1] + a2 * B[3];
    M[3 * i + 2] = a0 * B[4] + a1 * B[3] + a2 * B[2];
  }
}

// M = A B and M = A B^T, row-major 3x3.
__device__ inline void mul33(const double* A, const double* B, double* M) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) M[3 * i + j] = A[3 * i] * B[j] + A[3 * i + 1] * B[3 + j] + A[3 * i + 2] * B[6 + j];
}
__device__ inline void mul33t(const double* A, const double* B, double* M) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      M[3 * i + j] = A[3 * i] * B[3 * j] + A[3 * i + 1] * B[3 * j + 1] + A[3 * i + 2] * B[3 * j + 2];
}

// log(x) / 2 for x > 0 (not a number otherwise): x = 2^n y, y in [sqrt(1/2), sqrt(2)), and
// 2 atanh((y - 1) / (y + 1)) by 12 terms of its series (squared argument up to 0.0295, truncation
// below 1e-18). For the points whose volume changes by more than a quarter.
__device__ inline double half_log(double x) {
  double y = __builtin_amdgcn_frexp_mant(x);
  int n = __builtin_amdgcn_frexp_exp(x);
  if (y < kst(0.70710678118654752440)) {
    y += y;
    --n;
  }
  const double z = (y - 1.0) * frcp(y + 1.0), z2 = z * z;
  double r = kst(1.0 / 23.0);
#pragma unroll
  for (int k = 10; k >= 1; --k) r = fma(r, z2, kst(1.0 / (2 * k + 1)));
  r = fma(z * z2, r, z);
  r = fma((double)n, kst(0.34657359027997265471), r);
  return x > 0.0 ? r : __builtin_nan("");
}

// log(1 + x) / 2 = atanh(x / (2 + x)) for |x| <= 1/4: 6 terms of the series where 1e-3 bounds
// the squared argument (truncation below 1e-19), else 11.
__device__ inline double half_log1p_near(double x) {
  const double z = x * frcp(2.0 + x), z2 = z * z;
  double r;
  if (z2 <= kst(1e-3)) {
    r = kst(1.0 / 11.0);
  } else {
    r = kst(1.0 / 21.0);
#pragma unroll
    for (int k = 9; k >= 5; --k) r = fma(r, z2, kst(1.0 / (2 * k + 1)));
  }
#pragma unroll
  for (int k = 4; k >= 1; --k) r = fma(r, z2, kst(1.0 / (2 * k + 1)));
  return fma(z * z2, r, z);
}

// det(I + D) of D = st[0..5].
__device__ inline double det_plus_one(const double* st) {
  const double a = 1.0 + st[0], b = 1.0 + st[1], c = 1.0 + st[2];
  return a * (b * c - st[3] * st[3]) - st[5] * (st[5] * c - st[3] * st[4]) + st[4] * (st[5] * st[3] - b * st[4]);
}

// M = dev K and I2 = tr K of K = adj(b_tr / m) = (det F / m)^2 F^-T adj(I + D) F^-1, dm = det F / m: the
// products keep the small entries that adj(I + S) = Q - S + I2 / 3 loses.
__device__ inline void dev_adjugate(const double* Fi, const double* st, double dm, double* M, double& I2) {
  const double a = 1.0 + st[0], b = 1.0 + st[1], c = 1.0 + st[2], f = st[3], g = st[4], h = st[5];
  const double A[6] = {b * c - f * f, a * c - g * g, a * b - h * h, h * g - f * a, h * f - g * b, g * f - h * c};
  const double s = dm * dm;
  const int at[3][3] = {{0, 5, 4}, {5, 1, 3}, {4, 3, 2}};
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const double x = s * Fi[j], y = s * Fi[3 + j], z = s * Fi[6 + j];
    const double t[3] = {A[0] * x + A[5] * y + A[4] * z, A[5] * x + A[1] * y + A[3] * z, A[4] * x + A[3] * y + A[2] * z};
#pragma unroll
    for (int i = 0; i <= j; ++i) M[at[i][j]] = Fi[i] * t[0] + Fi[3 + i] * t[1] + Fi[6 + i] * t[2];
  }
  I2 = M[0] + M[1] + M[2];
#pragma unroll
  for (int k = 0; k < 3; ++k) M[k] -= I2 * kst(1.0 / 3.0);
}

// Residual state at one point (Box 1 / Box 2 and Section 3); arguments as for qp_state.
// TAN: also the derivatives of the log coefficients (the tangent and its transpose).
template <bool TAN, bool VOCE, bool MAXW = false>
__device__ inline void ts_state(const MatParams<double>& m, const FracParams<double>& fr, const double* G, double phi,
                                double phin, const double* st, TState& s) {
  double A[6];
  const double det = kinematics<double>(G, st, s.Fi, A);
  const double third = kst(1.0 / 3.0);
  const double t = (A[0] + A[1] + A[2]) * third;
  const double im = frcp(1.0 + t);
#pragma unroll
  for (int k = 0; k < 6; ++k) s.S[k] = (k < 3 ? A[k] - t : A[k]) * im;
  const double* S = s.S;
  double SS[6];  // S^2
  SS[0] = S[0] * S[0] + S[5] * S[5] + S[4] * S[4];
  SS[1] = S[5] * S[5] + S[1] * S[1] + S[3] * S[3];
  SS[2] = S[4] * S[4] + S[3] * S[3] + S[2] * S[2];
  SS[3] = S[5] * S[4] - S[0] * S[3];
  SS[4] = S[5] * S[3] - S[1] * S[4];
  SS[5] = S[4] * S[3] - S[2] * S[5];
  s.ss = SS[0] + SS[1] + SS[2];
  const double J2 = 0.5 * s.ss, J3 = third * sym_dot(S, SS);
  s.sm = 3.0 * J3 - s.ss;
  s.mm = kst(2.0 / 3.0) * J2 * J2 - 2.0 * s.sm - s.ss;
#pragma unroll
  for (int k = 0; k < 6; ++k) s.M[k] = (k < 3 ? fma(-third, s.ss, SS[k]) : SS[k]) - S[k];
  // det F <= 0 or an eigenvalue of b_tr <= 0 (trace, second invariant or determinant <= 0):
  // not physical, the point's values are NaN
  s.bad = !(det > 0.0) || !(t > -1.0);
  const bool far = !(J2 <= kst(LOG_SERIES_J2));
  bool wide = false;
  double db = 0.0;  // det b_tr, where formed
  if (!far) {
    log_series<TAN>(J2, J3, s);
  } else {
    db = det * det * det_plus_one(st);
    double I2 = 3.0 - J2;
    const double I3 = db * (im * im * im);
    s.bad |= !(I2 > 0.0) || !(I3 > 0.0);
    if (!s.bad) {
      const LogBounds bd = log_bounds(I2, I3);
      wide = bd.u * bd.il > LOG_WIDE;
      if (wide) {
        dev_adjugate(s.Fi, st, det * im, s.M, I2);
        s.sm = 3.0 * I3 - I2;
        s.mm = kst(2.0 / 3.0) * I2 * I2 - 6.0 * I3;
      }
      const LogMoments m = log_moments<TAN>(I2, I3, bd);
      s.p0 = m.p0;
      s.p1 = m.p1;
      if (TAN) {
        s.n2 = m.n2;
        s.n3 = m.n3;
        s.n4 = m.n4;
      }
    }
  }
  if (s.bad) s.p0 = s.p1 = __builtin_nan("");
  s.ee = s.p0 * (s.p0 * s.ss - 2.0 * s.p1 * s.sm) + s.p1 * s.p1 * s.mm;
  // tr eps = log(det b_tr) / 2: det b_tr = m^3 (1 - J2 + J3) formed about 1 where it is near 1,
  // else, and where the eigenvalues differ widely (J3 - J2 then holds few digits of I3), det F^2 det(I + D)
  const double v = t * fma(t, kst(3.0) + t, kst(3.0)), w = J3 - J2;
  const double x = wide ? db - 1.0 : v + w + v * w;
  if (fabs(x) <= 0.25) {
    s.theta = half_log1p_near(x);
  } else {
    if (!far) db = det * det * det_plus_one(st);
    s.theta = half_log(db);
  }
  return_map<VOCE, MAXW>(m, fr, phi, phin, st, s.ee, s);
}

// Degraded Kirchhoff stress tau_degr (symmetric).
__device__ inline void ts_stress(const MatParams<double>& m, const TState& s, double* tau) {
  const double a = 2.0 * m.mu * s.c * s.g, kt = m.kappa * s.theta, vol = s.tension ? s.g * kt : kt;
  const double a0 = a * s.p0, a1 = -a * s.p1;
#pragma unroll
  for (int k = 0; k < 6; ++k) tau[k] = fma(a0, s.S[k], k < 3 ? fma(a1, s.M[k], vol) : a1 * s.M[k]);
}

// First Piola stress P = tau_degr F^-T (eq:mechanical-gradient-transformation).
__device__ inline void ts_piola(const MatParams<double>& m, const TState& s, double* P) {
  double t[6];
  ts_stress(m, s, t);
  const double tm[9] = {t[0], t[5], t[4], t[5], t[1], t[3], t[4], t[3], t[2]};
  mul33t(tm, s.Fi, P);
}

// Directional derivative (Appendices B-C): (dG, dphi) -> (dP, dpsi^+). With dl = dG F^-1 and
// U = dl (I + S), the perturbation of b_tr is m (U + U^T) =: m X, so dS = dev X - (tr X / 3) S,
// and dP = (dtau - tau dl^T) F^-T.
__device__ inline void ts_tangent_psi(const MatParams<double>& m, const TState& s, const double* dG, double dphi,
                                      double* dP, double& dpsi) {
  double dl[9], U[9];
  mul33(dG, s.Fi, dl);
  mul_sym(dl, s.S, U);
#pragma unroll
  for (int k = 0; k < 9; ++k) U[k] += dl[k];
  double X[6] = {2.0 * U[0], 2.0 * U[4], 2.0 * U[8], U[5] + U[7], U[2] + U[6], U[1] + U[3]};
  const double t3 = (X[0] + X[1] + X[2]) * kst(1.0 / 3.0);
#pragma unroll
  for (int k = 0; k < 3; ++k) X[k] -= t3;  // dev X: dS = dev X - t3 S
  const double SX = sym_dot(s.S, X);
  const double aS = SX - t3 * s.ss, aM = sym_dot(s.M, X) - t3 * s.sm;  // S:dS, M:dS
  double ede;
  LogMap de = log_tangent(s, aS, aM, ede);
  const double dth = dl[0] + dl[4] + dl[8];
  // linearised return: d(c e) = c de + e (kq e:de + kphi dphi)
  const double kk = s.kq * ede + s.kphi * dphi;
  // degraded stress increment (eq:linear-degraded-stress-linearization) a de + b e + vol I, in
  // terms of dev X: dev(S dS + dS S) = dev(S X + X S) - 2 t3 (M + S)
  const double tm2 = 2.0 * m.mu, kt = m.kappa * s.theta, kdt = m.kappa * dth;
  const double a = s.g * tm2 * s.c, b = tm2 * (s.g * kk + s.gp * dphi * s.c);
  const double vol = s.tension ? s.g * kdt + s.gp * dphi * kt : kdt;
  de.a = a * (de.a - t3 * (s.p0 - s.p1)) + b * s.p0;
  de.b = a * (de.b + 2.0 * t3 * s.p1) - b * s.p1;
  de.c1 *= a;
  de.c2 *= a;
  double dt[6], tau[6];
  log_expand(s, de, X, SX, dt);
#pragma unroll
  for (int k = 0; k < 3; ++k) dt[k] += vol;
  ts_stress(m, s, tau);
  const int ix[9] = {0, 5, 4, 5, 1, 3, 4, 3, 2};
  double Z[9];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      Z[3 * i + j] = dt[ix[3 * i + j]] - (tau[ix[3 * i]] * dl[3 * j] + tau[ix[3 * i + 1]] * dl[3 * j + 1] +
                                          tau[ix[3 * i + 2]] * dl[3 * j + 2]);
  mul33t(Z, s.Fi, dP);
  // psi^+ increment (eq:energy-displacement-linearization)
  dpsi = tm2 * s.c * (s.c * ede + s.ee * kk) + (s.tension ? kt * dth : 0.0);
}

// The tangent of a single block: dL = dLcoef dphi + g' dH, dH = dpsi^+ when the history
// switch is on (eq:history-field-linearization, eq:linearized-local-damage-residual).
__device__ inline void ts_tangent(const MatParams<double>& m, const TState& s, const double* dG, double dphi,
                                  double* dP, double& dL) {
  double dpsi;
  ts_tangent_psi(m, s, dG, dphi, dP, dpsi);
  dL = s.dLcoef * dphi + (s.hactive ? s.gp * dpsi : 0.0);
}

// Transpose of ts_tangent_psi, step by step in reverse: cotangents (Pb of dP, Hb of dpsi^+;
// Hb = 0 when the history switch is off) -> (Gb of dG, phib = phib0 + the branch's terms).
// xe = (Pb F^-1):e, the stress cotangent along e used by the parameter partials.
__device__ inline void ts_tangent_T_psi(const MatParams<double>& m, const TState& s, const double* Pb, double Hb,
                                        double phib0, double* Gb, double& phib, double& xe) {
  const double tm2 = 2.0 * m.mu, kt = m.kappa * s.theta;
  double Zb[9], tau[6];
  mul33(Pb, s.Fi, Zb);
  ts_stress(m, s, tau);
  double E[6] = {Zb[0], Zb[4], Zb[8], 0.5 * (Zb[5] + Zb[7]), 0.5 * (Zb[2] + Zb[6]), 0.5 * (Zb[1] + Zb[3])};
  const double eS0 = sym_dot(s.S, E), eM0 = sym_dot(s.M, E);
  xe = s.p0 * eS0 - s.p1 * eM0;
  const double tz = Zb[0] + Zb[4] + Zb[8];
  // dtau = a de + b e + vol I
  phib = phib0 + tm2 * s.gp * s.c * xe + (s.tension ? s.gp * kt * tz : 0.0);
  double kkb = tm2 * s.g * xe + tm2 * s.c * s.ee * Hb;
  double dthb = (s.tension ? s.g * m.kappa : m.kappa) * tz + (s.tension ? kt * Hb : 0.0);
  phib += s.kphi * kkb;
  const double edeb = s.kq * kkb + tm2 * s.c * s.c * Hb;
  const double a = s.g * tm2 * s.c, tz3 = tz * kst(1.0 / 3.0);
#pragma unroll
  for (int k = 0; k < 3; ++k) E[k] -= tz3;  // the stress cotangent's deviator; de's is a E + edeb e
  // L of it: L(E) by the map, L(e) in S and M alone (log_eS and the rank-2 part)
  const double c1 = s.p0 + s.p1;
  const double eS = a * eS0 + edeb * (s.p0 * s.ss - s.p1 * s.sm), eM = a * eM0 + edeb * (s.p0 * s.sm - s.p1 * s.mm);
  const LogMap lm{a * c1, -a * s.p1, s.n2 * eS - s.n3 * eM + edeb * log_eS(s), s.n4 * eM - s.n3 * eS - 3.0 * edeb * s.p1 * c1};
  double Xb[6];
  log_expand(s, lm, E, eS0, Xb);
  // dS = dev X - (tr X / 3) S
  const double xs3 = sym_dot(s.S, Xb) * kst(1.0 / 3.0);
#pragma unroll
  for (int k = 0; k < 3; ++k) Xb[k] -= xs3;
  // X = U + U^T, U = dl (I + S): dl's cotangent 2 Xb (I + S) - (Zb^T tau), and dth = tr dl
  const int ix[9] = {0, 5, 4, 5, 1, 3, 4, 3, 2};
  double X2[9], lb[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) X2[k] = 2.0 * Xb[ix[k]];
  mul_sym(X2, s.S, lb);
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      lb[3 * i + j] += X2[3 * i + j] - (Zb[i] * tau[ix[j]] + Zb[3 + i] * tau[ix[3 + j]] + Zb[6 + i] * tau[ix[6 + j]]);
  lb[0] += dthb;
  lb[4] += dthb;
  lb[8] += dthb;
  mul33t(lb, s.Fi, Gb);
}

// Transpose of the single block's tangent.
__device__ inline void ts_tangent_T(const MatParams<double>& m, const TState& s, const double* Pb, double Lb,
                                    double* Gb, double& phib, double& xe) {
  ts_tangent_T_psi(m, s, Pb, s.hactive ? s.gp * Lb : 0.0, s.dLcoef * Lb, Gb, phib, xe);
}

}  // namespace pfmf
