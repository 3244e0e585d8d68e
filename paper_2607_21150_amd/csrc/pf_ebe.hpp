// Coarsest multigrid level of order 1 as element matrices (FP32).
//
// The order-1 level operator is the Galerkin product of the fine linearised
// operator: its element matrix K_e[r][c] (r, c = field * 8 + node, 32 x 32) is the
// fine-quadrature sum of the pointwise tangent tested and tried with the order-1
// basis. It is assembled once per linearisation from the FP32 record and then
// summed into a 27-point block stencil (4 x 4 blocks per neighbour), which the
// smoother applies: the same operator as the matrix-free level apply at the fine
// quadrature, at a fraction of its cost.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "pf_brick.hpp"
#include "pf_mg.hpp"
#include "pf_q4.hpp"
#include "pf_qf.hpp"

namespace pfmf {

struct EbeArgs {
  MeshDev m;
  int64_t n_q;
  const float* frame;   // F^-1 N of the block (see MGState)
  RecordSoA rec;
  const uint8_t* phase;
  const MatParams<float>* mats;
  int nph;
  FracParams<float> fr;
  float* K;             // [n_elem][32][32]
  const MatParams<float>* xmats;  // extra branches [nph][n_extra] (record layers 1..n_extra)
  int n_extra;
  const double* qd;     // GEO: mapped elements' geometry record [10][n_q] (J^-1, w det J)
};

// The tangent of one record layer by the displacement gradient's components: with
// E_ab(kL) = N_ka (F^-1 N)_Lb, Lt_ab = sum E_ab(kL) dG_kL (the principal-frame form of
// qp_tangent_psi), Z_aa = sum_b M_ab Lt_bb and Z_ab = p_ab Lt_ab + q_ab Lt_ba, the tangent is
// dP_fJ = sum_ab N_fa (F^-1 N)_Jb Z_ab, dpsi^+ = sum_b h_b Lt_bb + hphi dphi and
// dP/dphi = sum_a N_fa (F^-1 N)_Ja zphi_a.
struct TangentFactors {
  float N[9], R[9];   // frame and F^-1 N, the latter in reference directions (times J^-1 or 2/h)
  float M[9];         // diagonal block
  float p[9], q[9];   // off-diagonal factors (a != b)
  float zphi[3], h[3], hphi;
};

__device__ inline void tangent_factors(const MatParams<float>& m, const QPState<float>& s, TangentFactors& t) {
  const float tm2 = 2.f * m.mu, kt = m.kappa * s.theta, tmc = tm2 * s.c;
  const float kap = s.tension ? s.g * m.kappa : m.kappa;
  const float ee = s.e[0] * s.e[0] + s.e[1] * s.e[1] + s.e[2] * s.e[2];
  float td[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const float taubd = tmc * s.e[i];
    td[i] = s.tension ? s.g * (taubd + kt) : s.g * taubd + kt;
    t.zphi[i] = tm2 * s.g * s.e[i] * s.kphi + s.gp * (s.tension ? taubd + kt : taubd);
    t.h[i] = tmc * (s.c + ee * s.kq) * s.e[i] + (s.tension ? kt : 0.f);
  }
  t.hphi = tmc * ee * s.kphi;
  const float co[9] = {0.f, s.coef[2], s.coef[1], s.coef[2], 0.f, s.coef[0], s.coef[1], s.coef[0], 0.f};
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      t.M[3 * i + j] = s.g * (tmc * ((i == j ? 1.f : 0.f) - 1.f / 3.f) + tm2 * s.kq * s.e[i] * s.e[j]) + kap -
                       (i == j ? td[i] : 0.f);
      t.p[3 * i + j] = co[3 * i + j] * s.bd[j];
      t.q[3 * i + j] = co[3 * i + j] * s.bd[i] - td[i];
    }
#pragma unroll
  for (int k = 0; k < 9; ++k) t.N[k] = s.N[k], t.R[k] = s.R[k];
}

// Adds the columns of trial field K: C[3 (3 f + J) + L] += dP_fJ / dG_KL and
// H[L] += dpsi^+ / dG_KL (reference directions J, L).
template <int K>
__device__ inline void tangent_columns(const TangentFactors& t, float* C, float* H) {
  const float n[3] = {t.N[3 * K], t.N[3 * K + 1], t.N[3 * K + 2]};
  float O[9][3];  // O_ab(L) = sum of (M, p, q) E
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      if (a == b) {
        const float c0 = t.M[3 * a] * n[0], c1 = t.M[3 * a + 1] * n[1], c2 = t.M[3 * a + 2] * n[2];
#pragma unroll
        for (int L = 0; L < 3; ++L) O[4 * a][L] = c0 * t.R[3 * L] + c1 * t.R[3 * L + 1] + c2 * t.R[3 * L + 2];
      } else {
        const float cp = t.p[3 * a + b] * n[a], cq = t.q[3 * a + b] * n[b];
#pragma unroll
        for (int L = 0; L < 3; ++L) O[3 * a + b][L] = cp * t.R[3 * L + b] + cq * t.R[3 * L + a];
      }
    }
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    float X[3][3];
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int L = 0; L < 3; ++L)
        X[b][L] = t.N[3 * f] * O[b][L] + t.N[3 * f + 1] * O[3 + b][L] + t.N[3 * f + 2] * O[6 + b][L];
#pragma unroll
    for (int J = 0; J < 3; ++J)
#pragma unroll
      for (int L = 0; L < 3; ++L)
        C[3 * (3 * f + J) + L] += t.R[3 * J] * X[0][L] + t.R[3 * J + 1] * X[1][L] + t.R[3 * J + 2] * X[2][L];
  }
#pragma unroll
  for (int L = 0; L < 3; ++L)
    H[L] += t.h[0] * n[0] * t.R[3 * L] + t.h[1] * n[1] * t.R[3 * L + 1] + t.h[2] * n[2] * t.R[3 * L + 2];
}

// Shapes of the kernels below for order PF - 1 elements.
template <int PF> struct EbeShape {
  static constexpr int Q = PF, Q2 = Q * Q, Q3 = Q * Q * Q;
  // elements per workgroup: a line per lane in the x pass (NE Q^2 <= 64), a point per thread
  static constexpr int NE = PF == 2 ? 8 : (PF == 3 ? 5 : (PF == 4 ? 4 : 2));
  static constexpr int LQ = Q > 4 ? Q : 4;           // line stride: Q points, then 4 node pairs
  static constexpr int ES = Q * LQ * LQ + 4;         // entry and element stride (padded against bank conflicts)
  static constexpr int NENT = 30;                    // entries of one trial field
  static constexpr int LDS = NENT * NE * ES;
};

// A point of the element matrices' and diagonals' kernels: thread t holds point ql of element
// el (of the workgroup's NE); the block's F^-1 N, the reference-to-physical factors
// A[3 K + J] = d xi_K / d x_J (mapped elements: in FP64, products with them are summed and rounded once) and
// the weight (0 for threads without a point).
template <bool GEO> struct EbePoint {
  int64_t e, gq;
  int el, qx, qy, qz, pidc;
  bool pt;
  float R[9], Fi[9], w;  // Fi: F^-1 in the directions of R's rows (ebe_layer of the block sets it)
  std::conditional_t<GEO, double, float> A[9];
  // grad xi_J . grad xi_L
  __device__ float metric(int J, int L) const {
    return (float)(A[3 * J] * A[3 * L] + A[3 * J + 1] * A[3 * L + 1] + A[3 * J + 2] * A[3 * L + 2]);
  }
};

template <int PF, bool GEO>
__device__ inline void ebe_point(const EbeArgs& a, const DevTablesF* __restrict__ tabs, EbePoint<GEO>& p) {
  using S = EbeShape<PF>;
  constexpr int Q = S::Q, Q2 = S::Q2, Q3 = S::Q3, NE = S::NE;
  const int t = threadIdx.x;
  const int64_t n_elem = (int64_t)a.m.nx * a.m.ny * a.m.nz;
  p.el = t / Q3;
  const int ql = t - p.el * Q3;
  p.qx = ql % Q;
  p.qy = (ql / Q) % Q;
  p.qz = ql / Q2;
  p.e = (int64_t)blockIdx.x * NE + p.el;
  p.pt = p.el < NE && p.e < n_elem;
  p.gq = p.e * Q3 + ql;
#pragma unroll
  for (int k = 0; k < 9; ++k) p.R[k] = p.pt ? a.frame[rec_at<Q3, 9>(p.e, ql) + k * rec_pad(Q3)] : 0.f;
  const float ih[3] = {(float)a.m.ih[0], (float)a.m.ih[1], (float)a.m.ih[2]};
#pragma unroll
  for (int k = 0; k < 9; ++k)
    if constexpr (GEO)
      p.A[k] = p.pt ? a.qd[k * a.n_q + p.gq] : 0.0;
    else
      p.A[k] = k % 4 == 0 ? ih[k / 4] : 0.f;
  p.w = 0.f;
  if (p.pt)
    p.w = GEO ? (float)a.qd[9 * a.n_q + p.gq]
              : tabs->w[Q][p.qx] * tabs->w[Q][p.qy] * tabs->w[Q][p.qz] * (float)a.m.jdet;
  const int pid = p.pt ? a.phase[p.gq] : 0;
  p.pidc = pid < a.nph ? pid : 0;
}

// What the point's phi row takes from its block: the history switch, g' and dL/dphi.
struct EbeBlock {
  bool hact;
  float gp, dLc;
};

// The tangent's factors of record layer j (0: the block, taken first; 1 + j: extra branch j) of
// point p; false where the layer is empty. REF: R in reference directions (mapped elements; the box's
// record holds them).
template <int PF, bool GEO, bool REF = GEO>
__device__ inline bool ebe_layer(const EbeArgs& a, EbePoint<GEO>& p, int j, TangentFactors& tf, EbeBlock& blk) {
  const int64_t o = (int64_t)j * a.n_q + p.gq;
  LinRecord rc;
  rc.flags = p.pt ? a.rec.flags[o] : 0;
  if (j > 0 && (!p.pt || (rc.flags & REC_EMPTY))) return false;
  constexpr int Q3 = PF * PF * PF;
  const int64_t n_elem = (int64_t)a.m.nx * a.m.ny * a.m.nz;
  const float* rr = a.rec.rec + rec_at<Q3, REC_N>(j * n_elem + p.e, (int)(p.gq - p.e * Q3));
#pragma unroll
  for (int k = 0; k < REC_N; ++k) rc.v[k] = p.pt ? rr[k * rec_pad(Q3)] : 0.f;
  const MatParams<float> m = j == 0 ? a.mats[p.pidc] : a.xmats[p.pidc * a.n_extra + j - 1];
  QPState<float> s;
  qp_state_lin<float>(rc, s);
  if (j == 0) {
#pragma unroll
    for (int k = 0; k < 9; ++k) s.R[k] = p.R[k];
    frame_times<float>(p.R, s.N, p.Fi);
  } else {
    frame_product<float>(p.Fi, s.N, nullptr, s.R);
  }
  if (j == 0) blk = EbeBlock{s.hactive, s.gp, s.dLcoef};
  tangent_factors(m, s, tf);
  if (REF && GEO) {
    float R[9];
#pragma unroll
    for (int K = 0; K < 3; ++K)
#pragma unroll
      for (int b = 0; b < 3; ++b)
        R[3 * K + b] = (float)(p.A[3 * K] * tf.R[b] + p.A[3 * K + 1] * tf.R[3 + b] + p.A[3 * K + 2] * tf.R[6 + b]);
#pragma unroll
    for (int k = 0; k < 9; ++k) tf.R[k] = R[k];
  }
  return true;
}

// Element matrices of the order-1 level, K_e[r][c] (r, c = field * 8 + node): the fine-quadrature
// sum of (test basis) x tangent x (trial basis). One thread per point of NE elements; the trial
// fields are taken in turn, and each turn's tangent entries (test field and direction J, trial
// direction L) go through LDS in sum-factorised form: the pair of 1-D order-1 bases of an axis
// contracts that axis' points into the 2 x 2 (test, trial) nodes, x, then y, then z with the sum
// over (J, L). An entry's 1-D pair is B or D on either side by its J and L, so it is uniform over
// a wave and its products come from a table (tabs->pair) through scalar registers.
//
// Bound by vector instructions. Contracting the 10 x 10 tangent of a point with the 32 trial and
// 32 test functions takes 260 k multiply-adds per order-3 element, and forming the tangent by
// ten directional derivatives 130 k more; the factored form takes 60 k and 50 k. Order 3 on 32^3
// elements 1.49 -> 0.31 ms, order 4 on 40^3 9.67 -> 1.38 ms.
// GEO: mapped elements (gradients and weights from the points' geometry record).
template <int PF, bool MB, bool GEO = false>
__global__ __launch_bounds__(NT) void k_ebe_assemble(EbeArgs a, const DevTablesF* __restrict__ tabs) {
  using S = EbeShape<PF>;
  constexpr int Q = S::Q, Q2 = S::Q2, Q3 = S::Q3, NE = S::NE, LQ = S::LQ, ES = S::ES;
  static_assert(NE * Q2 <= 64 && NE * Q3 <= NT, "a line per lane, a point per thread");
  __shared__ float lds[S::LDS];
  const int l = threadIdx.x & 63, wv = wave_id();
  const int64_t n_elem = (int64_t)a.m.nx * a.m.ny * a.m.nz;
  const int64_t e0 = (int64_t)blockIdx.x * NE;
  EbePoint<GEO> p;
  ebe_point<PF, GEO>(a, tabs, p);
  const int el = p.el, qx = p.qx, qy = p.qy, qz = p.qz;
  const float w = p.w;
  const MatParams<float> mp = a.mats[p.pidc];
  EbeBlock blk;
  TangentFactors tf0;
  ebe_layer<PF, GEO>(a, p, 0, tf0, blk);
  const bool hact = blk.hact;
  const float gp = blk.gp, dLc = blk.dLc;
  float* con = lds;
  float* my = con + el * ES + (qz * LQ + qy) * LQ + qx;  // this point's slot of entry 0
  // entry index: trial field g < 3: (3 f + J) 3 + L (f < 3), 27 + L (test phi); g = 3: 3 f + J
  // (trial value), 9 (phi value with phi value), 10 + 3 J + L (grad phi with grad phi)
#pragma unroll 1
  for (int g = 0; g < 4; ++g) {
    const int nent = g < 3 ? 30 : 19;
    if (g < 3) {
      float C[27], H[3] = {0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < 27; ++k) C[k] = 0.f;
      auto columns = [&](const TangentFactors& tf) {
        if (g == 0)
          tangent_columns<0>(tf, C, H);
        else if (g == 1)
          tangent_columns<1>(tf, C, H);
        else
          tangent_columns<2>(tf, C, H);
      };
      columns(tf0);
      if (MB) {
#pragma unroll 1
        for (int j = 0; j < a.n_extra; ++j) {
          TangentFactors tj;
          EbeBlock bj;
          if (ebe_layer<PF, GEO>(a, p, 1 + j, tj, bj)) columns(tj);
        }
      }
      if (el < NE) {
        const float wr = hact ? w * a.fr.s_phi * gp : 0.f;
#pragma unroll
        for (int k = 0; k < 27; ++k) my[k * NE * ES] = w * C[k];
#pragma unroll
        for (int L = 0; L < 3; ++L) my[(27 + L) * NE * ES] = wr * H[L];
      }
    } else {
      float C[9], hphi = tf0.hphi;
      auto phi_column = [&](const TangentFactors& tf) {
#pragma unroll
        for (int f = 0; f < 3; ++f)
#pragma unroll
          for (int J = 0; J < 3; ++J)
            C[3 * f + J] += tf.N[3 * f] * tf.zphi[0] * tf.R[3 * J] + tf.N[3 * f + 1] * tf.zphi[1] * tf.R[3 * J + 1] +
                            tf.N[3 * f + 2] * tf.zphi[2] * tf.R[3 * J + 2];
      };
#pragma unroll
      for (int k = 0; k < 9; ++k) C[k] = 0.f;
      phi_column(tf0);
      if (MB) {
#pragma unroll 1
        for (int j = 0; j < a.n_extra; ++j) {
          TangentFactors tj;
          EbeBlock bj;
          if (ebe_layer<PF, GEO>(a, p, 1 + j, tj, bj)) {
            phi_column(tj);
            hphi += tj.hphi;
          }
        }
      }
      if (el < NE) {
        const float kfg = w * a.fr.kf * mp.Gc;
#pragma unroll
        for (int k = 0; k < 9; ++k) my[k * NE * ES] = w * C[k];
        my[9 * NE * ES] = w * a.fr.s_phi * (dLc + (hact ? gp * hphi : 0.f));
#pragma unroll
        for (int J = 0; J < 3; ++J)
#pragma unroll
          for (int L = 0; L < 3; ++L)
            my[(10 + 3 * J + L) * NE * ES] =
                kfg * p.metric(J, L);
      }
    }
    __syncthreads();
    // test and trial direction of an entry (3: value)
    auto dirs = [&](int ent, int& J, int& L) {
      if (g < 3) {
        L = ent % 3;
        J = ent < 27 ? (ent / 3) % 3 : 3;
      } else if (ent < 10) {
        J = ent < 9 ? ent % 3 : 3;
        L = 3;
      } else {
        J = (ent - 10) / 3;
        L = (ent - 10) % 3;
      }
    };
    // x: a line (element, qz, qy) per lane, entries over the waves
#pragma unroll 1
    for (int ent = wv; ent < nent; ent += NT / 64) {
      int J, L;
      dirs(ent, J, L);
      const float* pr = tabs->pair[Q][(J == 0 ? 1 : 0) + (L == 0 ? 2 : 0)][0];
      if (l < NE * Q2) {
        const int le = l / Q2, r = l - le * Q2;
        float* line = con + (ent * NE + le) * ES + ((r / Q) * LQ + r % Q) * LQ;
        float v[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) v[q] = line[q];
#pragma unroll
        for (int ab = 0; ab < 4; ++ab) {
          float acc = 0.f;
#pragma unroll
          for (int q = 0; q < Q; ++q) acc += pr[ab * 5 + q] * v[q];
          line[ab] = acc;
        }
      }
    }
    __syncthreads();
    // y: a line (element, qz, x pair) per lane
#pragma unroll 1
    for (int ent = wv; ent < nent; ent += NT / 64) {
      int J, L;
      dirs(ent, J, L);
      const float* pr = tabs->pair[Q][(J == 1 ? 1 : 0) + (L == 1 ? 2 : 0)][0];
#pragma unroll
      for (int l0 = 0; l0 < NE * Q * 4; l0 += 64) {
        const int lt = l0 + l;
        if (lt < NE * Q * 4) {
          const int le = lt / (Q * 4), r = lt - le * (Q * 4);
          float* line = con + (ent * NE + le) * ES + (r >> 2) * LQ * LQ + (r & 3);
          float v[Q];
#pragma unroll
          for (int q = 0; q < Q; ++q) v[q] = line[q * LQ];
#pragma unroll
          for (int ab = 0; ab < 4; ++ab) {
            float acc = 0.f;
#pragma unroll
            for (int q = 0; q < Q; ++q) acc += pr[ab * 5 + q] * v[q];
            line[ab * LQ] = acc;
          }
        }
      }
    }
    __syncthreads();
    // z: a test field per wave, (element, xy pair) per lane, the four z pairs summed over (J, L)
#pragma unroll
    for (int r0 = 0; r0 < NE * 16; r0 += 64) {
      const int f = wv, r = r0 + l;
      if (r >= NE * 16) continue;
      const int le = r >> 4, xy = r & 15;
      float acc[4] = {0.f, 0.f, 0.f, 0.f};
      auto add = [&](int ent, int type) {
        const float* col = con + (ent * NE + le) * ES + (xy >> 2) * LQ + (xy & 3);
        const float* pr = tabs->pair[Q][type][0];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const float v = col[q * LQ * LQ];
#pragma unroll
          for (int ab = 0; ab < 4; ++ab) acc[ab] += pr[ab * 5 + q] * v;
        }
      };
      const int nL = g < 3 ? 3 : 1, nJ = f < 3 ? 3 : 1;
#pragma unroll 1
      for (int J = 0; J < nJ; ++J)
#pragma unroll 1
        for (int L = 0; L < nL; ++L) {
          const int ent = g < 3 ? (f < 3 ? 3 * (3 * f + J) + L : 27 + L) : (f < 3 ? 3 * f + J : 9);
          add(ent, (nJ == 3 && J == 2 ? 1 : 0) + (nL == 3 && L == 2 ? 2 : 0));
        }
      if (g == 3 && f == 3) {
#pragma unroll 1
        for (int k = 0; k < 9; ++k) add(10 + k, (k / 3 == 2 ? 1 : 0) + (k % 3 == 2 ? 2 : 0));
      }
      // pair index: test node + 2 trial node per axis
      if (e0 + le < n_elem) {
        const int ax = xy & 1, bx = (xy >> 1) & 1, ay = (xy >> 2) & 1, by = xy >> 3;
        float* Ke = a.K + (e0 + le) * 1024;
#pragma unroll
        for (int ab = 0; ab < 4; ++ab) {
          const int na = ax + 2 * ay + 4 * (ab & 1), nb = bx + 2 * by + 4 * (ab >> 1);
          Ke[(f * 8 + na) * 32 + g * 8 + nb] = acc[ab];
        }
      }
    }
    __syncthreads();
  }
}

// The diagonal block of displacement field K: D[0..5] += dP_KJ / dG_KL for (J, L) = xx, yy, zz,
// xy + yx, xz + zx, yz + zy. GEO: R in physical directions, the block taken to reference directions
// as A C A^T.
template <int K, bool GEO>
__device__ inline void tangent_diagonal(const TangentFactors& t, const EbePoint<GEO>& p, float* D) {
  const float n[3] = {t.N[3 * K], t.N[3 * K + 1], t.N[3 * K + 2]};
  float X[3][3];  // sum_a N_Ka O_ab(L)
#pragma unroll
  for (int b = 0; b < 3; ++b)
#pragma unroll
    for (int L = 0; L < 3; ++L) {
      float v = n[b] * (t.M[3 * b] * n[0] * t.R[3 * L] + t.M[3 * b + 1] * n[1] * t.R[3 * L + 1] +
                        t.M[3 * b + 2] * n[2] * t.R[3 * L + 2]);
#pragma unroll
      for (int c = 0; c < 3; ++c)
        if (c != b) v += n[c] * (t.p[3 * c + b] * n[c] * t.R[3 * L + b] + t.q[3 * c + b] * n[b] * t.R[3 * L + c]);
      X[b][L] = v;
    }
  float C[3][3];
#pragma unroll
  for (int J = 0; J < 3; ++J)
#pragma unroll
    for (int L = 0; L < 3; ++L) C[J][L] = t.R[3 * J] * X[0][L] + t.R[3 * J + 1] * X[1][L] + t.R[3 * J + 2] * X[2][L];
  if constexpr (GEO) {
    double AC[3][3];
#pragma unroll
    for (int J = 0; J < 3; ++J)
#pragma unroll
      for (int L = 0; L < 3; ++L) AC[J][L] = p.A[3 * J] * C[0][L] + p.A[3 * J + 1] * C[1][L] + p.A[3 * J + 2] * C[2][L];
#pragma unroll
    for (int J = 0; J < 3; ++J)
#pragma unroll
      for (int L = 0; L < 3; ++L)
        C[J][L] = (float)(AC[J][0] * p.A[3 * L] + AC[J][1] * p.A[3 * L + 1] + AC[J][2] * p.A[3 * L + 2]);
  }
  D[0] += C[0][0];
  D[1] += C[1][1];
  D[2] += C[2][2];
  D[3] += C[0][1] + C[1][0];
  D[4] += C[0][2] + C[2][0];
  D[5] += C[1][2] + C[2][1];
}

// Point-Jacobi diagonal of a level of PC nodes per direction, evaluated at the fine points: the
// element diagonals, stored to the extended node grid ev [4][nz PC][ny PC][nx PC] and summed per
// node by k_gather_ext<float, PC>. Entries per point: for each displacement field the six
// coefficients of tangent_diagonal, for phi the value's and the gradient's (3 on the box, 6 on
// mapped elements); an axis' squared 1-D bases (B B, B D or D D by the entry's directions, a
// table) contract its points into the PC nodes, x, y, then z with the sum over the entries.
// Order 3 on 32^3 elements, both levels: 0.82 -> 0.24 ms with the node sums (eight colour launches that
// took ten directional derivatives per point and summed all Q^3 points for every node).
template <int PF, int PC, bool MB, bool GEO = false>
__global__ __launch_bounds__(NT) void k_level_diag(EbeArgs a, float* __restrict__ ev, const DevTablesF* __restrict__ tabs) {
  using S = EbeShape<PF>;
  static_assert(PC <= PF, "a level below the fine one");
  constexpr int Q = S::Q, Q2 = S::Q2, Q3 = S::Q3, NE = S::NE, ES = Q3 + 1;
  constexpr int NPHI = GEO ? 7 : 4, NENT = 18 + NPHI;
  constexpr int CON = NENT * NE * ES;
  __shared__ float lds[CON];
  const int l = threadIdx.x & 63, wv = wave_id();
  const int64_t n_elem = (int64_t)a.m.nx * a.m.ny * a.m.nz;
  const int64_t e0 = (int64_t)blockIdx.x * NE;
  EbePoint<GEO> p;
  ebe_point<PF, GEO>(a, tabs, p);
  {
    const MatParams<float> mp = a.mats[p.pidc];
    float D[18];
#pragma unroll
    for (int k = 0; k < 18; ++k) D[k] = 0.f;
    EbeBlock blk;
    float hphi;
    {
      TangentFactors tf;
      ebe_layer<PF, GEO, false>(a, p, 0, tf, blk);
      tangent_diagonal<0>(tf, p, D);
      tangent_diagonal<1>(tf, p, D + 6);
      tangent_diagonal<2>(tf, p, D + 12);
      hphi = tf.hphi;
    }
    if (MB) {
#pragma unroll 1
      for (int j = 0; j < a.n_extra; ++j) {
        TangentFactors tf;
        EbeBlock bj;
        if (ebe_layer<PF, GEO, false>(a, p, 1 + j, tf, bj)) {
          tangent_diagonal<0>(tf, p, D);
          tangent_diagonal<1>(tf, p, D + 6);
          tangent_diagonal<2>(tf, p, D + 12);
          hphi += tf.hphi;
        }
      }
    }
    if (p.el < NE) {
      float* my = lds + p.el * ES + (p.qz * Q + p.qy) * Q + p.qx;
      const float kfg = p.w * a.fr.kf * mp.Gc;
#pragma unroll
      for (int k = 0; k < 18; ++k) my[k * NE * ES] = p.w * D[k];
      my[18 * NE * ES] = p.w * a.fr.s_phi * (blk.dLc + (blk.hact ? blk.gp * hphi : 0.f));
#pragma unroll
      for (int k = 0; k < NPHI - 1; ++k) {
        const int J = k < 3 ? k : (k == 5 ? 1 : 0), L = k < 3 ? k : (k == 3 ? 1 : 2);
        my[(19 + k) * NE * ES] = (k < 3 ? kfg : 2.f * kfg) * p.metric(J, L);
      }
    }
  }
  __syncthreads();
  // type of an entry on an axis: the number of its directions along it (18: the phi value, none)
  auto type = [](int ent, int axis) {
    if (ent == 18) return 0;
    const int k = ent < 18 ? ent % 6 : ent - 19;
    const int J = k < 3 ? k : (k == 5 ? 1 : 0), L = k < 3 ? k : (k == 3 ? 1 : 2);
    return (J == axis ? 1 : 0) + (L == axis ? 1 : 0);
  };
#pragma unroll 1
  for (int ent = wv; ent < NENT; ent += NT / 64) {
    const float* sq = tabs->square[PC][Q][type(ent, 0)][0];
    if (l < NE * Q2) {
      const int le = l / Q2, r = l - le * Q2;
      float* line = lds + (ent * NE + le) * ES + r * Q;
      float v[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) v[q] = line[q];
#pragma unroll
      for (int i = 0; i < PC; ++i) {
        float acc = 0.f;
#pragma unroll
        for (int q = 0; q < Q; ++q) acc += sq[i * 5 + q] * v[q];
        line[i] = acc;
      }
    }
  }
  __syncthreads();
#pragma unroll 1
  for (int ent = wv; ent < NENT; ent += NT / 64) {
    const float* sq = tabs->square[PC][Q][type(ent, 1)][0];
    if (l < NE * Q * PC) {
      const int le = l / (Q * PC), r = l - le * (Q * PC);
      float* line = lds + (ent * NE + le) * ES + (r / PC) * Q2 + r % PC;
      float v[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) v[q] = line[q * Q];
#pragma unroll
      for (int i = 0; i < PC; ++i) {
        float acc = 0.f;
#pragma unroll
        for (int q = 0; q < Q; ++q) acc += sq[i * 5 + q] * v[q];
        line[i * Q] = acc;
      }
    }
  }
  __syncthreads();
  // z: a field per wave, (element, y node, x node) per lane
  static_assert(NE * Q * PC <= 64, "the y lines and z columns fit a wave");
  const int f = wv;
  if (l < NE * PC * PC) {
    const int le = l / (PC * PC), r = l - le * (PC * PC), j = r / PC, i = r % PC;
    float acc[PC];
#pragma unroll
    for (int k = 0; k < PC; ++k) acc[k] = 0.f;
    const int ent0 = 6 * f, ne = f < 3 ? 6 : NPHI;
#pragma unroll 1
    for (int k = 0; k < ne; ++k) {
      const int ent = ent0 + k;
      const float* sq = tabs->square[PC][Q][type(ent, 2)][0];
      const float* col = lds + (ent * NE + le) * ES + j * Q + i;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const float v = col[q * Q2];
#pragma unroll
        for (int n = 0; n < PC; ++n) acc[n] += sq[n * 5 + q] * v;
      }
    }
    const int64_t e = e0 + le;
    if (e < n_elem) {
      const int ex = (int)(e % a.m.nx), ey = (int)((e / a.m.nx) % a.m.ny), ez = (int)(e / ((int64_t)a.m.nx * a.m.ny));
      const int64_t NXe = (int64_t)a.m.nx * PC, NYe = (int64_t)a.m.ny * PC, NZe = (int64_t)a.m.nz * PC;
#pragma unroll
      for (int n = 0; n < PC; ++n)
        ev[((f * NZe + (int64_t)ez * PC + n) * NYe + (int64_t)ey * PC + j) * NXe + (int64_t)ex * PC + i] = acc[n];
    }
  }
}

// The order-1 level as a 27-point block stencil: S[o][f][g][i] couples field f of
// node i with field g of node i + o, o = (dx + 1) + 3 (dy + 1) + 9 (dz + 1). Each
// entry sums the matching element-matrix entries over the (up to 8) elements that
// hold both nodes, in a fixed order, so the result is deterministic. One workgroup per 64 nodes
// and row f: 32 threads read a node's row of an element's matrix (128 contiguous bytes, column
// g * 8 + nb), sums and the transposition to the stencil's blocks in LDS. A thread per (offset,
// node) read one value per cache line: 32^3 elements 164 -> 46 us,
// 40^3 313 -> 86 us.
static __global__ __launch_bounds__(NT) void k_stencil_from_ebe(const float* __restrict__ K, int nx, int ny, int nz,
                                                         int64_t n_nodes, float* __restrict__ S) {
  constexpr int LD = 65;  // padded against bank conflicts
  __shared__ float acc[108 * LD];
  const int nx1 = nx + 1, ny1 = ny + 1;
  const int64_t i0 = (int64_t)blockIdx.x * 64;
  const int f = blockIdx.y, t = threadIdx.x;
  for (int k = t; k < 108 * LD; k += NT) acc[k] = 0.f;
  __syncthreads();
  const int col = t & 31, nb = col & 7, g = col >> 3;
  const int bx = nb & 1, by = (nb >> 1) & 1, bz = nb >> 2;
  for (int n = t >> 5; n < 64; n += NT / 32) {
    const int64_t i = i0 + n;
    if (i >= n_nodes) break;
    const int ix = (int)(i % nx1), iy = (int)((i / nx1) % ny1), iz = (int)(i / ((int64_t)nx1 * ny1));
    float v[8];
#pragma unroll
    for (int na = 0; na < 8; ++na) {
      const int ex = ix - (na & 1), ey = iy - ((na >> 1) & 1), ez = iz - (na >> 2);
      const bool in = ex >= 0 && ex < nx && ey >= 0 && ey < ny && ez >= 0 && ez < nz;
      const int64_t e = in ? (int64_t)ex + (int64_t)nx * (ey + (int64_t)ny * ez) : 0;
      const float k = K[e * 1024 + (f * 8 + na) * 32 + col];
      v[na] = in ? k : 0.f;
    }
#pragma unroll
    for (int na = 0; na < 8; ++na) {
      const int o = (bx - (na & 1) + 1) + 3 * (by - ((na >> 1) & 1) + 1) + 9 * (bz - (na >> 2) + 1);
      // the node's 32 threads hold different (o, g) here, but another na brings one of them to an entry
      // of this one's: the steps stay in order (a node's threads are in one wave)
      acc[(4 * o + g) * LD + n] += v[na];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
  __syncthreads();
  float* So = S + stencil_at(i0, f);
  for (int k = t; k < 108 * 64; k += NT) So[k] = acc[(k >> 6) * LD + (k & 63)];
}

// Diagonal of the stencil.
static __global__ __launch_bounds__(NT) void k_stencil_diag(const float* __restrict__ S, int64_t n, float* __restrict__ out) {
  const int f = blockIdx.y;
  for (int64_t i = blockIdx.x * (int64_t)NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT)
    out[f * n + i] = S[stencil_at(i, f) + (4 * 13 + f) * 64 + (i & 63)];
}

// Apply of the stencil with the epilogue OP; one thread per (node, output field), blockIdx.y =
// field. The epilogue must not write x. Bound by latency up to some 20^3 nodes, by the stencil's
// bytes above: a neighbour outside the lattice is not skipped but reads the node itself with its
// value taken as 0 (its entries of S are 0 and stored), so that no load waits for a branch.
// 17^3 nodes 13.4 -> 5.6 us, 33^3 21.7 -> 14.4 us, 41^3 29.2 -> 23.5 us (119 MB).
template <int OP>
__global__ __launch_bounds__(NT) void k_stencil_apply(const float* __restrict__ S, int nx1, int ny1, int nz1,
                                                      int64_t n, const float* __restrict__ x, Epilogue<float> ep) {
  const int f = blockIdx.y;
  double sq = 0.0;
  for (int64_t i0 = blockIdx.x * (int64_t)NT + 64 * wave_id(); i0 < n; i0 += (int64_t)gridDim.x * NT) {
    const int l = threadIdx.x & 63;
    const bool node = i0 + l < n;
    const int i = (int)(node ? i0 + l : n - 1);
    const int ix = i % nx1, iyz = i / nx1, iy = iyz % ny1, iz = iyz / ny1;
    const EpiIn<float> in = epi_load<OP>(ep, f * n + i);
    const float* So = S + stencil_at(i0, f) + l;
    const int sx[3] = {ix > 0 ? -1 : 0, 0, ix + 1 < nx1 ? 1 : 0};
    const int sy[3] = {iy > 0 ? -nx1 : 0, 0, iy + 1 < ny1 ? nx1 : 0};
    const int sz[3] = {iz > 0 ? -nx1 * ny1 : 0, 0, iz + 1 < nz1 ? nx1 * ny1 : 0};
    float acc = 0.f;
#pragma unroll
    for (int o = 0; o < 27; ++o) {
      const int a = o % 3, b = (o / 3) % 3, c = o / 9;
      const bool inside = (a == 1 || sx[a] != 0) && (b == 1 || sy[b] != 0) && (c == 1 || sz[c] != 0);
      const int j = inside ? i + sx[a] + sy[b] + sz[c] : i;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float v = (x + g * n)[j];
        acc += So[(4 * o + g) * 64] * (inside ? v : 0.f);
      }
    }
    if (!node) continue;
    if (ep.has_dir && ((dir_bits(ep.dir, ix, iy, iz, nx1, ny1, nz1) >> f) & 1u)) acc = 0.f;
    const float y = epi_apply<OP>(ep, in, f * n + i, acc);
    if (OP == E_POWER) sq += (double)y * (double)y;
  }
  if (OP == E_POWER) epi_sum(sq, ep.part, (int)(blockIdx.x + gridDim.x * f));
}

// The coarsest level's solve, all sweeps of the Chebyshev smoother in one workgroup of 8 waves (a
// wave holds 64 nodes of one field, a thread its row's 108 entries, b, r, d and x): a launch per
// apply of a few hundred rows is all latency. 125 nodes, 8 sweeps of degree 3 (23 applies): 37 us,
// 23 launches of 4.3 us and their gaps before. At most COARSE_SOLVE_NODES nodes: beyond them a
// thread's registers do not hold a row, and reading the rows from L2 took 24 us per apply at 216
// nodes against 5.3 us for a launch.
constexpr int COARSE_SOLVE_NODES = 128;
struct ChebCoefs {
  float c0, a[32], c[32];  // start, and steps 1 to degree - 1
};
static __global__ __launch_bounds__(4 * COARSE_SOLVE_NODES) void k_coarse_solve(const float* __restrict__ S, int nx1, int ny1, int nz1,
                                                             int n, const float* __restrict__ b,
                                                             const float* __restrict__ dinv, float* __restrict__ x,
                                                             int degree, int sweeps, ChebCoefs co, DirMask dir,
                                                             int has_dir) {
  constexpr int NV = COARSE_SOLVE_NODES, LD = NV + 1;  // slot NV: the value 0 of a neighbour outside
  __shared__ float vec[2][4 * LD];
  const int w = wave_id(), f = w & 3, blk = w >> 2;
  const int slot = blk * 64 + (threadIdx.x & 63);
  const bool node = slot < n;
  const int i = node ? slot : n - 1;
  const int ix = i % nx1, iyz = i / nx1, iy = iyz % ny1, iz = iyz / ny1;
  // a wave without a block of nodes (n <= 64 blk) reads the last one
  const float* So = S + stencil_at(min(blk * 64, (n - 1) / 64 * 64), f) + (threadIdx.x & 63);
  float row[108];
#pragma unroll
  for (int k = 0; k < 108; ++k) row[k] = So[k * 64];
  const bool fixed = has_dir && ((dir_bits(dir, ix, iy, iz, nx1, ny1, nz1) >> f) & 1u);
  const float bi = b[f * n + i], di = dinv[f * n + i];
  if (threadIdx.x < 8) vec[threadIdx.x >> 2][(threadIdx.x & 3) * LD + NV] = 0.f;
  const int sx[3] = {ix > 0 ? -1 : 0, 0, ix + 1 < nx1 ? 1 : 0};
  const int sy[3] = {iy > 0 ? -nx1 : 0, 0, iy + 1 < ny1 ? nx1 : 0};
  const int sz[3] = {iz > 0 ? -nx1 * ny1 : 0, 0, iz + 1 < nz1 ? nx1 * ny1 : 0};
  int turn = 0;
  // A v of this row, v_i this thread's entry
  auto apply = [&](float vi) {
    float* v = vec[turn];
    turn ^= 1;
    v[f * LD + slot] = vi;
    __syncthreads();
    float acc = 0.f;
#pragma unroll
    for (int o = 0; o < 27; ++o) {
      const int ax = o % 3, ay = (o / 3) % 3, az = o / 9;
      const bool inside = (ax == 1 || sx[ax] != 0) && (ay == 1 || sy[ay] != 0) && (az == 1 || sz[az] != 0);
      const int j = inside ? i + sx[ax] + sy[ay] + sz[az] : NV;
#pragma unroll
      for (int g = 0; g < 4; ++g) acc += row[4 * o + g] * v[g * LD + j];
    }
    return fixed ? 0.f : acc;
  };
  float xi = 0.f;
  for (int s = 0; s < sweeps; ++s) {
    float r = s == 0 ? bi : bi - apply(xi);
    float d = co.c0 * di * r;
    xi += d;
    for (int it = 1; it < degree; ++it) {
      r -= apply(d);
      d = co.a[it - 1] * d + co.c[it - 1] * di * r;
      xi += d;
    }
  }
  if (node) x[f * n + i] = xi;
}

// Galerkin product of a block stencil on a coarser order-1 lattice: Sc = P^T Sf P with P
// the trilinear interpolation from the coarse lattice (every second fine node per
// direction, fine n = 2 nc - 1 nodes) to the fine one; fine node 2I + a (a = -1, 0, 1)
// takes weight 1 (a = 0) or 1/2 (|a| = 1) from coarse node I. Entry (O, f, g) of coarse
// node I: sum over fine i = 2I + a and j = 2(I + O) + b with |j - i| <= 1 per direction
// of w(a) w(b) Sf[j - i][f][g][i] (accumulated in double, fixed order: deterministic).
// One thread per coarse node and row f (4 columns g), blockIdx.y = offset O, so that the bounds of
// a and b are uniform; fine nodes outside the lattice take weight 0 and node 0's entry (-1, -1, -1), and entries
// of Sf towards nodes outside are 0. 33^3 to 17^3 nodes 529 -> 285 us, 41^3 to
// 21^3 1048 -> 601 (a thread per entry, its bounds and index lists formed per lane, before).
static __global__ __launch_bounds__(NT) void k_stencil_rap(const float* __restrict__ Sf, int fx1, int fy1, int fz1,
                                                    float* __restrict__ Sc, int cx1, int cy1, int cz1) {
  const int nc = cx1 * cy1 * cz1;
  const int O = blockIdx.y, f = blockIdx.z;
  const int dO[3] = {O % 3 - 1, (O / 3) % 3 - 1, O / 9 - 1};
  for (int I = blockIdx.x * NT + threadIdx.x; I < nc; I += gridDim.x * NT) {
    const int Ix = I % cx1, Iy = (I / cx1) % cy1, Iz = I / (cx1 * cy1);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int az = -1; az <= 1; ++az)
      for (int ay = -1; ay <= 1; ++ay)
#pragma unroll
        for (int ax = -1; ax <= 1; ++ax) {
          const int x = 2 * Ix + ax, y = 2 * Iy + ay, z = 2 * Iz + az;
          const bool in = x >= 0 && x < fx1 && y >= 0 && y < fy1 && z >= 0 && z < fz1;
          const int64_t i = in ? x + (int64_t)fx1 * (y + (int64_t)fy1 * z) : 0;
          const float wa = in ? (ax ? 0.5f : 1.f) * (ay ? 0.5f : 1.f) * (az ? 0.5f : 1.f) : 0.f;
          // (a NaN or infinity of node 0 does not count: the entry towards a node outside is read, a 0)
          const float* Si = Sf + stencil_at(i, f) + (i & 63);
          const int so = in ? 4 * 64 : 0;
          for (int oz = max(-1, 2 * dO[2] - az - 1); oz <= min(1, 2 * dO[2] - az + 1); ++oz)
            for (int oy = max(-1, 2 * dO[1] - ay - 1); oy <= min(1, 2 * dO[1] - ay + 1); ++oy) {
              const float wy = wa * (oz - 2 * dO[2] + az ? 0.5f : 1.f) * (oy - 2 * dO[1] + ay ? 0.5f : 1.f);
#pragma unroll
              for (int ox = -1; ox <= 1; ++ox) {
                const int bx = ox - 2 * dO[0] + ax;
                if (bx < -1 || bx > 1) continue;  // uniform
                const double w = wy * (bx ? 0.5f : 1.f);
                const float* Se = Si + so * ((ox + 1) + 3 * (oy + 1) + 9 * (oz + 1));
#pragma unroll
                for (int g = 0; g < 4; ++g) acc[g] += w * (double)Se[g * 64];
              }
            }
        }
#pragma unroll
    for (int g = 0; g < 4; ++g) Sc[stencil_at(I, f) + (4 * O + g) * 64 + (I & 63)] = (float)acc[g];
  }
}

}  // namespace pfmf
