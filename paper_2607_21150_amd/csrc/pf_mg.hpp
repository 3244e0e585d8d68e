// FP32 p-multigrid: linearisation record, level operators at the fine
// quadrature, point-Jacobi diagonals, level transfers and Chebyshev vector ops.
//
// Levels are orders p, p-1, ..., coarse_p on the same mesh. Every level is
// evaluated at the fine Gauss points with the fine linearisation record, so a
// coarse operator is the Galerkin product P^T A P of the fine one (the coarse
// space is a subspace of the fine space). Below an order-1 level the hierarchy may
// continue on coarser order-1 lattices (every second node per direction, trilinear
// interpolation), each operator the Galerkin product of the one above, formed once
// per linearisation as a block stencil. Everything an apply needs at a point
// (F^-1 N, frame, log strains, the yield, split and history decisions, the
// return-mapping scalars) comes from the record taken in FP64 by the linearisation.
#pragma once
#include <climits>
#include <hip/hip_runtime.h>

#include "pf_brick.hpp"
#include "pf_ops.hpp"
#include "pf_qf.hpp"
#include "pf_geom.hpp"

namespace pfmf {

template <typename V> struct RecordSoAT {
  V* rec;          // [n_elem][REC_N][rec_pad], slots as in LinRecordT
  uint8_t* flags;  // [n_q]
};
using RecordSoA = RecordSoAT<float>;

// The records lie element by element, a slot's points together and padded to 16 bytes, so that an
// apply reads one run of memory per element with aligned slots. With a slot's points of the whole
// mesh together (24 streams, order-4 slots off the cache lines) the apply on 40^3 order-4 elements
// took 260 us and its order-2 level 221, now 201 and 150; on 32^3 order-3 elements 51.1 and 46.4,
// now 47.5 and 44.4.
constexpr int64_t rec_pad(int q3) { return (q3 + 3) / 4 * 4; }
// Slot k of point ql of element e at k * rec_pad(Q3) from here (e: layer * n_elem + element).
template <int Q3, int SLOTS> __device__ inline int64_t rec_at(int64_t e, int ql) {
  return e * (SLOTS * rec_pad(Q3)) + ql;
}

struct LevelDev {
  int P;           // nodes per direction of this level's elements
  int nx1, ny1;
  int64_t n_nodes;
};

// Block stencil of an order-1 level, [blocks of 64 nodes][4 rows f][27 offsets][4 columns g][64]: a
// wavefront reads the 108 entries of its row as one run of memory. Entry (o, g) of row f of node i is
// at stencil_at(i, f) + (4 o + g) * 64 + i % 64; entries towards nodes outside the lattice are 0, and
// the last block is padded.
__host__ __device__ constexpr int64_t stencil_at(int64_t i, int f) { return (i / 64 * 4 + f) * (108 * 64); }
__host__ __device__ constexpr int64_t stencil_size(int64_t n) { return stencil_at(n + 63, 0); }

constexpr int MG_MAX_LEVELS = 8;

struct MGLevel {
  int p = 0, P = 0;
  // h: coarsening depth of an order-1 level (0: the mesh itself; h > 0: the order-1
  // lattice with 2^h times fewer elements per direction, its operator the Galerkin
  // product of the finer order-1 level's, stored as a block stencil S)
  int h = 0;
  int ne[3] = {0, 0, 0};  // elements per direction of this level's lattice
  int nx1 = 0, ny1 = 0, nz1 = 0;
  int64_t n_nodes = 0;
  float* S = nullptr;  // h > 0: block stencil (stencil_at)
  float *x = nullptr, *r = nullptr, *d = nullptr, *t = nullptr, *b = nullptr;
  float *diag = nullptr, *dinv = nullptr;
  double lmax = 0.0;
  // transfer to the next coarser level: per direction, prolongation rows
  // (fine index -> coarse base + Pc weights) and restriction rows
  // (coarse index -> fine base + (2 pf + 1) weights)
  int* pbase[3] = {nullptr, nullptr, nullptr};
  float* pw[3] = {nullptr, nullptr, nullptr};
  int* rbase[3] = {nullptr, nullptr, nullptr};
  float* rw[3] = {nullptr, nullptr, nullptr};
};

struct MGState {
  int n_levels = 0;
  MGLevel lv[MG_MAX_LEVELS];
  float* frame = nullptr;  // F^-1 N of the block at the linearisation point [n_elem][9][rec_pad] (QPState::R)
  RecordSoA rec{nullptr, nullptr};  // [rec_layers][n_elem][REC_N][rec_pad] and flags [rec_layers][n_q]
  float* tmpA = nullptr;
  float* tmpB = nullptr;
  double* red = nullptr;  // reduction scratch
  float* ebe = nullptr;    // element matrices of the order-1 level on the mesh [n_elem][32][32], and the
                           // levels' element diagonals (both per linearisation)
  float* stencil = nullptr;  // the same level as a block stencil (stencil_at)
  float* ebuf32 = nullptr;   // brick-buffer scatter of the FP32 level applies
  double* rec64 = nullptr;   // stored FP64 linearisation, laid out as rec (flags in rec.flags)
  double* u64 = nullptr;     // u at the linearisation point [3][n_nodes]
  int rec_layers = 0;        // record layers allocated (1 + extra branches)
  int ebe_level = -1;
  bool linearized = false;
  bool lin64_valid = false;  // rec64 / u64 hold the current linearisation
};

inline void mg_free_level(MGLevel& L) {
  float* fs[] = {L.x, L.r, L.d, L.t, L.b, L.diag, L.dinv, L.S};
  for (float* f : fs) (void)hipFree(f);
  for (int k = 0; k < 3; ++k) {
    (void)hipFree(L.pbase[k]);
    (void)hipFree(L.pw[k]);
    (void)hipFree(L.rbase[k]);
    (void)hipFree(L.rw[k]);
  }
  L = MGLevel();
}

inline void mg_free(MGState& mg) {
  for (int l = 0; l < MG_MAX_LEVELS; ++l) mg_free_level(mg.lv[l]);
  (void)hipFree(mg.frame);
  (void)hipFree(mg.rec.rec);
  (void)hipFree(mg.rec.flags);
  (void)hipFree(mg.tmpA);
  (void)hipFree(mg.tmpB);
  (void)hipFree(mg.red);
  (void)hipFree(mg.ebe);
  (void)hipFree(mg.stencil);
  (void)hipFree(mg.ebuf32);
  (void)hipFree(mg.rec64);
  (void)hipFree(mg.u64);
  mg = MGState();
}

// ---------------------------------------------------------------------------
// Linearisation: FP64 decisions -> FP32 record (one launch over all bricks).
// ---------------------------------------------------------------------------

// MODE 0: linearisation record; MODE 1: state commit into state_out.
// Records of a point with extra branches in parallel: layer 0 is the block's record,
// whose flags carry the point's history switch and whose dL slot its dL/dphi (both
// from the total psi^+); layer 1 + j that of extra branch j, or flags REC_EMPTY where
// the point's phase has no branch in slot j. Layer l of the records holds elements
// l * n_elem on (rec_at), its flags sit at flags + l * n_q.
constexpr uint8_t REC_EMPTY = 0x80;

struct LinArgs {
  MeshDev m;
  int nx1, ny1;
  int64_t n_nodes, n_q;
  const double* z;
  const double* phin;
  const double* state;
  const uint8_t* phase;
  const MatParams<double>* mats;
  int nph;
  FracParams<double> fr;
  RecordSoA rec;
  float* frame;          // MODE 0, 2: see MGState
  double* rec64;         // MODE 0: the same record in FP64 (flags shared), or null
  double* state_out;
  int* flag;
  const XBranch* xb;     // extra branches [nph][n_extra] and their states [7*n_extra][n_q]
  const double* xstate;
  int n_extra;
  double* xstate_out;    // MODE 3: the extra branches' committed states
  const double* qd;      // GEO: mapped elements' geometry record [10][n_q] (J^-1, w det J)
};

// MODE 0: record; MODE 2: record with the extra branches' layers; MODE 1: state commit;
// MODE 3: state commit with the extra branches. GEO: mapped elements (gradients through
// each point's J^-1 from a.qd).
template <int P, int Q, int MODE, bool GEO = false>
__global__ __launch_bounds__(NT) void k_linearize(LinArgs a, DevTables* __restrict__ tabs) {
  using S = OpShape<P, Q>;
  constexpr int NB3 = S::NB3, Q3 = S::Q3, ER = S::ER;
  extern __shared__ double lds[];
  double* zb = lds;
  double* tmp = zb + 4 * NB3;
  double* tab = tmp + S::TMP;
  const int brick = xcd_brick_all(a.m, blockIdx.x);  // nothing is shared between bricks: one launch
  if (brick < 0) return;  // padding workgroup (uniform)
  const BrickGeom g = decode_brick_lin(a.m, brick);
  for (int t = threadIdx.x; t < Q * P; t += NT) {
    tab[t] = tabs->B[P][Q][t / P][t % P];
    tab[Q * P + t] = tabs->D[P][Q][t / P][t % P];
  }
  stage_brick<double, double, P, 4>(a.z, a.n_nodes, a.nx1, a.ny1, g, zb);
  __syncthreads();
  const TabRef<double> tb{tab, tab + Q * P};
  const double ih[3] = {a.m.ih[0], a.m.ih[1], a.m.ih[2]};
  double* xb = tmp;
  double* xd = xb + ER * P * P * Q;
  double* ybb = xd + ER * P * P * Q;
  double* ydb = ybb + ER * P * Q * Q;
  double* ybd = ydb + ER * P * Q * Q;
  const int t = threadIdx.x;
  const int el = t / Q3, ql = t % Q3;
  const int qx = ql % Q, qy = (ql / Q) % Q, qz = ql / (Q * Q);
  const int64_t n_elem = (int64_t)a.m.nx * a.m.ny * a.m.nz;
  bool any_bad = false, bad_pid = false;
  for (int r = 0; r < S::ROUNDS; ++r) {
    const int slot0 = r * ER, slot = slot0 + el;
    const int sx = slot & 1, sy = (slot >> 1) & 1, sz = slot >> 2;
    const bool active = (t < ER * Q3) && (slot < 8) && sx < g.nex && sy < g.ney && sz < g.nez;
    double G[9], phi = 0.0;
#pragma unroll 1
    for (int f = 0; f < 4; ++f) {
      fwd_xy<double, P, Q, ER>(zb + f * NB3, slot0, g, tb, f < 3, xb, xd, ybb, ydb, ybd);
      if (t < ER * Q3) {
        double v, d[3];
        fwd_z<double, P, Q>(ybb, ydb, ybd, el, qx, qy, qz, tb, f < 3, v, d);
        if (f < 3) {
#pragma unroll
          for (int J = 0; J < 3; ++J) G[3 * f + J] = GEO ? d[J] : d[J] * ih[J];  // GEO: mapped below
        } else {
          phi = v;
        }
      }
      __syncthreads();
    }
    if (active) {
      const int64_t e = (int64_t)(g.ex0 + sx) + (int64_t)a.m.nx * ((g.ey0 + sy) + (int64_t)a.m.ny * (g.ez0 + sz));
      const int64_t gq = e * Q3 + ql;
      if (GEO) {
        double gA[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) gA[k] = a.qd[k * a.n_q + gq];
#pragma unroll
        for (int f = 0; f < 3; ++f) {
          const double dr[3] = {G[3 * f], G[3 * f + 1], G[3 * f + 2]};
          ref_to_phys<true>(dr, ih, gA, G + 3 * f);
        }
      }
      double st[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) st[k] = a.state[k * a.n_q + gq];
      const int pid = a.phase[gq];
      bad_pid |= pid >= a.nph;  // an id outside the phase table raises the phase flag
      const MatParams<double> mp = a.mats[pid < a.nph ? pid : 0];
      QPState<double> s;
      qp_state<>(mp, a.fr, G, phi, 0.0, st, s);
      any_bad |= s.bad;
      if (MODE == 2) {
        // extra branches: one record layer each; the block's layer takes the point's
        // history switch and dL/dphi from the total psi^+
        double psi = s.psi;
        const int pidc = pid < a.nph ? pid : 0;
#pragma unroll 1
        for (int j = 0; j < a.n_extra; ++j) {
          const int64_t lj = 1 + j;
          const XBranch& b = a.xb[pidc * a.n_extra + j];
          if (b.kind == XB_NONE) {
            a.rec.flags[lj * a.n_q + gq] = REC_EMPTY;
            continue;
          }
          double xs[8];
#pragma unroll
          for (int k = 0; k < 7; ++k) xs[k] = b.kind == XB_HOOKE ? 0.0 : a.xstate[(int64_t)(7 * j + k) * a.n_q + gq];
          xs[7] = 0.0;
          QPState<double> sj;
          qp_state<true, true>(b.m, a.fr, G, phi, 0.0, xs, sj);
          any_bad |= sj.bad;
          psi += sj.psi;
          const int64_t ro = rec_at<Q3, REC_N>(lj * n_elem + e, ql);
          LinRecord rj;
          record_from_state(sj, rj);
#pragma unroll
          for (int k = 0; k < REC_N; ++k) a.rec.rec[ro + k * rec_pad(Q3)] = rj.v[k];
          a.rec.flags[lj * a.n_q + gq] = rj.flags;
          if (a.rec64) {
            LinRecordT<double> r64;
            record_from_state(sj, r64);
#pragma unroll
            for (int k = 0; k < REC_N; ++k) a.rec64[ro + k * rec_pad(Q3)] = r64.v[k];
          }
        }
        s.hactive = psi > st[7];
        const double H = s.hactive ? psi : st[7];
        const double alpha_pp = (a.fr.at == 2) ? 2.0 : 0.0;
        s.dLcoef = 2.0 * H + mp.Gc * a.fr.inv_c0l0 * alpha_pp + a.fr.zeta * a.fr.inv_dt;
      }
      if (MODE == 3) {
        // every branch's state (Box 1 step 4); the block's history takes the total psi^+
        double psi = s.psi;
        const int pidc = pid < a.nph ? pid : 0;
#pragma unroll 1
        for (int j = 0; j < a.n_extra; ++j) {
          const XBranch& b = a.xb[pidc * a.n_extra + j];
          double xs[8];
#pragma unroll
          for (int k = 0; k < 7; ++k) xs[k] = a.xstate[(int64_t)(7 * j + k) * a.n_q + gq];
          xs[7] = 0.0;
          if (b.kind == XB_NONE) {
#pragma unroll
            for (int k = 0; k < 7; ++k) a.xstate_out[(int64_t)(7 * j + k) * a.n_q + gq] = xs[k];
            continue;
          }
          double xk[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) xk[k] = b.kind == XB_HOOKE ? 0.0 : xs[k];
          QPState<double> sj;
          qp_state<true, true>(b.m, a.fr, G, phi, 0.0, xk, sj);
          any_bad |= sj.bad;
          psi += sj.psi;
          double nj[8];
          if (b.kind == XB_HOOKE) {
#pragma unroll
            for (int k = 0; k < 7; ++k) nj[k] = xs[k];
          } else {
            commit_from_state(sj, G, xk, nj);
          }
#pragma unroll
          for (int k = 0; k < 7; ++k) a.xstate_out[(int64_t)(7 * j + k) * a.n_q + gq] = nj[k];
        }
        s.hactive = psi > st[7];
        s.H = s.hactive ? psi : st[7];
      }
      if (MODE == 0 || MODE == 2) {
        const int64_t ro = rec_at<Q3, REC_N>(e, ql);
        LinRecord rc;
        double N[9], R[9];
        record_from_state(s, rc, N);
        frame_product<double>(s.Fi, N, GEO ? nullptr : ih, R);
#pragma unroll
        for (int k = 0; k < 9; ++k) a.frame[rec_at<Q3, 9>(e, ql) + k * rec_pad(Q3)] = (float)R[k];
#pragma unroll
        for (int k = 0; k < REC_N; ++k) a.rec.rec[ro + k * rec_pad(Q3)] = rc.v[k];
        a.rec.flags[gq] = rc.flags;
        if (a.rec64) {
          LinRecordT<double> r64;
          record_from_state(s, r64);
#pragma unroll
          for (int k = 0; k < REC_N; ++k) a.rec64[ro + k * rec_pad(Q3)] = r64.v[k];
        }
      } else {
        double ns[8];
        commit_from_state(s, G, st, ns);
#pragma unroll
        for (int k = 0; k < 8; ++k) a.state_out[k * a.n_q + gq] = ns[k];
      }
    }
  }
  if (any_bad) a.flag[0] = 1;
  if (bad_pid) a.flag[1] = 1;
}

// ---------------------------------------------------------------------------
// Record applies
// ---------------------------------------------------------------------------

// Arguments of the linearised applies from a record: V = float for the FP32 multigrid
// levels, V = double for the FP64 apply from the stored linearisation (fine level).
template <typename V> struct LinApplyArgs {
  MeshDev m;
  LevelDev fine, lev;
  int64_t n_q;
  const V* frame;        // V = float: F^-1 N of the block (see MGState)
  const V* u;            // V = double: fine u at the linearisation point [3][n_fine]
  const V* dz;           // level vector [4][n_lev]
  RecordSoAT<V> rec;
  const uint8_t* phase;
  const MatParams<V>* mats;
  int nph;
  FracParams<V> fr;
  V* out;
  V* ebuf;               // brick-buffer scatter (extended node grid)
  const MatParams<V>* xmats;  // extra branches [nph][n_extra] (record layers 1..n_extra)
  int n_extra;
  const V* qd;           // GEO: mapped elements' geometry record [10][n_q] (J^-1, w det J),
                         // in the working precision
};

// Mapped elements in the record applies: reference derivatives (FP64) to a physical
// gradient in the working precision through the point's J^-1 (FP64).
template <typename V>
__device__ inline void map_grad(double d0, double d1, double d2, const double* A, V* out) {
#pragma unroll
  for (int J = 0; J < 3; ++J) out[J] = (V)(d0 * A[J] + d1 * A[3 + J] + d2 * A[6 + J]);
}

// The level applies' QPState::R. V = float reads it: recomputing F^-1 from u at every apply costs a
// sum factorisation of three fields, an inverse and a product (of 1226 vector instructions per
// wave 250, order 3) against 36 bytes per point.
// V = double (the stored linearisation) recomputes it from u.
template <typename V> constexpr bool FRAME_FROM_U = sizeof(V) == 8;

// Record-based tangent of one point: the block's layer, plus (n_extra > 0) the extra
// branches' layers, their dP and dpsi^+ summed and the switch applied to the total.
// valid = false (a lane without a point) reads no layer.
// MB = false compiles the block's tangent only (kernels launched without branches).
template <typename V, int Q3, bool MB>
__device__ inline void lin_tangent(const RecordSoAT<V>& rec, int64_t n_elem, const MatParams<V>* xmats, int n_extra,
                                   const MatParams<V>& mp, const QPState<V>& s, int pid, int64_t e, int ql, bool valid,
                                   const V* dG, V dphi, V* dP, V& dL) {
  if (!MB || n_extra == 0) {
    qp_tangent<V>(mp, s, dG, dphi, dP, dL);
    return;
  }
  V dpsi;
  qp_tangent_psi<V>(mp, s, dG, dphi, dP, dpsi, true);
  V Fi[9];  // F^-1 in the directions of R's rows
  frame_times<V>(s.R, s.N, Fi);
#pragma unroll 1
  for (int j = 0; j < n_extra; ++j) {
    const int64_t lj = 1 + j;
    const uint8_t fl = valid ? rec.flags[(lj * n_elem + e) * Q3 + ql] : REC_EMPTY;
    if (fl & REC_EMPTY) continue;
    const V* rr = rec.rec + rec_at<Q3, REC_N>(lj * n_elem + e, ql);
    LinRecordT<V> r;
#pragma unroll
    for (int k = 0; k < REC_N; ++k) r.v[k] = rr[k * rec_pad(Q3)];
    r.flags = fl;
    const MatParams<V>& bm = xmats[pid * n_extra + j];
    QPState<V> sj;
    qp_state_lin<V>(r, sj);
    frame_product<V>(Fi, sj.N, nullptr, sj.R);
    V dPj[9], dpj;
    qp_tangent_psi<V>(bm, sj, dG, dphi, dPj, dpj, true);
#pragma unroll
    for (int k = 0; k < 9; ++k) dP[k] += dPj[k];
    dpsi += dpj;
  }
  dL = s.dLcoef * dphi + s.gp * (s.hactive ? dpsi : V(0));
}
using A32Args = LinApplyArgs<float>;

// ---------------------------------------------------------------------------
// What a level apply does with each entry of A d as it is formed: the node gather and the block
// stencil carry the vector operation that follows the apply, so that A d is neither written nor
// read back (a Chebyshev step on n entries moves 28 n bytes beside the apply instead of 40 n, in
// one launch less, and the Dirichlet mask needs no launch of its own). Order 4 on 40^3 elements:
// gather 77 us and step up to 94 us -> 102 us in one launch, the Newton step on the order-3 32^3 mesh
// 70.0 -> 60.7 ms. The last step of a smoother stores x alone: 80 us.
// ---------------------------------------------------------------------------
enum EpiOp {
  E_STORE,  // out = v
  E_RESID,  // r = b - v
  E_FIRST,  // r = b - v, d = c dinv r (the Chebyshev start; x takes d in the first step)
  E_STEP,   // r = r_in - v, d = a d_in + c dinv r, x = x_in + [d_in] + d
  E_LAST,   // the same where r and d are not needed after it
  E_SCALE,  // out = dinv v inv[0]
  E_POWER   // out = dinv v inv[0], and the sum of its squares
};

template <typename T> struct Epilogue {
  T *out, *r, *d, *x;
  const T *b, *r_in, *d_in, *x_in, *dinv;  // x_in null: x starts from zero
  T a, c;
  int x_first;          // E_STEP: the first one, x takes d_in too
  const float* inv;     // E_SCALE, E_POWER: 1 / norm of the vector applied, or null
  double* part;         // E_POWER: one partial sum per workgroup
  DirMask dir;          // constrained entries: v = 0
  int has_dir, nz1;
};

// The epilogue's inputs at entry i, loaded before A d is complete.
template <typename T> struct EpiIn {
  T r, d, x, dinv;
};
template <int OP, typename T>
__device__ inline EpiIn<T> epi_load(const Epilogue<T>& e, int64_t i) {
  EpiIn<T> v{T(0), T(0), T(0), T(0)};
  if (OP == E_RESID || OP == E_FIRST) v.r = e.b[i];
  if (OP == E_STEP || OP == E_LAST) {
    v.r = e.r_in[i];
    v.d = e.d_in[i];
    if (e.x_in) v.x = e.x_in[i];
  }
  if (OP != E_STORE && OP != E_RESID) v.dinv = e.dinv[i];
  return v;
}

// Entry i of A d is v.
template <int OP, typename T>
__device__ inline T epi_apply(const Epilogue<T>& e, const EpiIn<T>& in, int64_t i, T v) {
  if (OP == E_STORE) {
    e.out[i] = v;
  } else if (OP == E_RESID) {
    e.r[i] = in.r - v;
  } else if (OP == E_FIRST) {
    const T r = in.r - v;
    e.r[i] = r;
    e.d[i] = e.c * in.dinv * r;
  } else if (OP == E_STEP || OP == E_LAST) {
    const T r = in.r - v, d = e.a * in.d + e.c * in.dinv * r;
    if (OP == E_STEP) {
      e.r[i] = r;
      e.d[i] = d;
    }
    e.x[i] = (e.x_first ? in.x + in.d : in.x) + d;
  } else {
    const T y = e.inv ? (in.dinv * v) * (T)e.inv[0] : in.dinv * v;
    e.out[i] = y;
    return y;
  }
  return T(0);
}

// E_POWER's partial sum of a workgroup of NT threads (deterministic tree).
__device__ inline void epi_sum(double s, double* part, int block) {
  __shared__ double red[NT];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int st = NT / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[block] = red[0];
}

// The same on a stored A d (the colour launches write it): one thread per node, blockIdx.y = field.
template <int OP>
__global__ __launch_bounds__(NT) void k_epilogue(const float* v, int nx1, int ny1, int64_t n, Epilogue<float> e) {
  const int f = blockIdx.y;
  double s = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT) {
    const EpiIn<float> in = epi_load<OP>(e, f * n + i);
    float w = v[f * n + i];
    if (e.has_dir) {
      const int ix = (int)(i % nx1), iy = (int)((i / nx1) % ny1), iz = (int)(i / ((int64_t)nx1 * ny1));
      if ((dir_bits(e.dir, ix, iy, iz, nx1, ny1, e.nz1) >> f) & 1u) w = 0.f;
    }
    const float y = epi_apply<OP>(e, in, f * n + i, w);
    if (OP == E_POWER) s += (double)y * (double)y;
  }
  if (OP == E_POWER) epi_sum(s, e.part, (int)(blockIdx.x + gridDim.x * f));
}

// ---------------------------------------------------------------------------
// Level transfers (one direction per launch) and vector kernels.
// ---------------------------------------------------------------------------

// out[f][i2][i1][i0] = sum_k w[c*nw + k] in[f][...][base[c] + k][...] along `axis`,
// where c is the output coordinate along axis. in dims: (n0i, n1i, n2i). add: out += the sum;
// has_dir: the sum is 0 on constrained entries of the output lattice.
static __global__ void k_transfer_1d(const float* __restrict__ in, float* __restrict__ out, int n0o, int n1o, int n2o,
                              int n0i, int n1i, int n2i, int axis, const int* __restrict__ base,
                              const float* __restrict__ w, int nw, int add, DirMask dir, int has_dir) {
  const int64_t no = (int64_t)n0o * n1o * n2o;
  const int64_t ni = (int64_t)n0i * n1i * n2i;
  for (int64_t o = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; o < no; o += (int64_t)gridDim.x * blockDim.x) {
    const int i0 = (int)(o % n0o);
    const int i1 = (int)((o / n0o) % n1o);
    const int i2 = (int)(o / ((int64_t)n0o * n1o));
    const int c = axis == 0 ? i0 : (axis == 1 ? i1 : i2);
    const int nin = axis == 0 ? n0i : (axis == 1 ? n1i : n2i);
    const int b0 = base[c];
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < nw; ++k) {
      const int src = b0 + k;
      const float wk = w[(int64_t)c * nw + k];
      if (src < 0 || src >= nin || wk == 0.f) continue;
      int j0 = i0, j1 = i1, j2 = i2;
      if (axis == 0) j0 = src; else if (axis == 1) j1 = src; else j2 = src;
      const int64_t ii = j0 + (int64_t)n0i * (j1 + (int64_t)n1i * j2);
#pragma unroll
      for (int f = 0; f < 4; ++f) acc[f] += wk * in[f * ni + ii];
    }
    const uint32_t bits = has_dir ? dir_bits(dir, i0, i1, i2, n0o, n1o, n2o) : 0u;
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const float v = (bits >> f) & 1u ? 0.f : acc[f];
      out[f * no + o] = add ? out[f * no + o] + v : v;
    }
  }
}

// The three directions in one launch: NW weights per direction (NW^3 inputs per output). One thread
// per (i0, i1) and field (blockIdx.y) for zb outputs along direction 2 (blockIdx.z), which keep the
// NW interpolated planes of the inputs while their base stays the same. add, has_dir: see above.
struct TransferAxes {
  const int* base[3];
  const float* w[3];
};
template <int NW>
static __global__ __launch_bounds__(NT) void k_transfer(const float* __restrict__ in, float* __restrict__ out, int n0o,
                                                        int n1o, int n2o, int n0i, int n1i, int n2i, TransferAxes ax,
                                                        int zb, int add, DirMask dir, int has_dir) {
  const int t = blockIdx.x * NT + threadIdx.x;
  if (t >= n0o * n1o) return;
  const int i1 = t / n0o, i0 = t - i1 * n0o, f = blockIdx.y;
  const float* src = in + (int64_t)f * n0i * n1i * n2i;
  float* dst = out + (int64_t)f * n0o * n1o * n2o;
  int j0[NW], j1[NW];
  float w0[NW], w1[NW];
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    // a weight outside the lattice counts as 0; an input with weight 0 is taken as 0
    const int a = ax.base[0][i0] + k, b = ax.base[1][i1] + k;
    w0[k] = a >= 0 && a < n0i ? ax.w[0][i0 * NW + k] : 0.f;
    w1[k] = b >= 0 && b < n1i ? ax.w[1][i1 * NW + k] : 0.f;
    j0[k] = w0[k] != 0.f ? a : 0;
    j1[k] = w1[k] != 0.f ? b * n0i : 0;
  }
  float plane[NW];
  int have = INT_MIN;  // base of the planes held
  const int z1 = (int)min((int64_t)n2o, (int64_t)(blockIdx.z + 1) * zb);
  for (int i2 = blockIdx.z * zb; i2 < z1; ++i2) {
    const int b2 = ax.base[2][i2];
    if (b2 != have) {  // uniform
      have = b2;
#pragma unroll
      for (int k2 = 0; k2 < NW; ++k2) {
        const int c = b2 + k2;
        plane[k2] = 0.f;
        if (c < 0 || c >= n2i) continue;  // uniform
        const float* s2 = src + (int64_t)c * n0i * n1i;
        float v[NW][NW];
#pragma unroll
        for (int k1 = 0; k1 < NW; ++k1)
#pragma unroll
          for (int k0 = 0; k0 < NW; ++k0) v[k1][k0] = s2[j1[k1] + j0[k0]];
#pragma unroll
        for (int k1 = 0; k1 < NW; ++k1) {
          float r = 0.f;
#pragma unroll
          for (int k0 = 0; k0 < NW; ++k0) r += w0[k0] != 0.f ? w0[k0] * v[k1][k0] : 0.f;
          plane[k2] += w1[k1] != 0.f ? w1[k1] * r : 0.f;
        }
      }
    }
    float acc = 0.f;
#pragma unroll
    for (int k2 = 0; k2 < NW; ++k2) {
      const float wk = ax.w[2][(int64_t)i2 * NW + k2];
      acc += wk != 0.f ? wk * plane[k2] : 0.f;
    }
    if (has_dir && ((dir_bits(dir, i0, i1, i2, n0o, n1o, n2o) >> f) & 1u)) acc = 0.f;
    float* o = dst + ((int64_t)i2 * n1o + i1) * n0o + i0;
    *o = add ? *o + acc : acc;
  }
}

static __global__ void k_vec_copy(const float* __restrict__ a, float* __restrict__ b, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    b[i] = a[i];
}

// y += x
static __global__ void k_vec_add(const float* __restrict__ x, float* __restrict__ y, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] += x[i];
}

// Chebyshev start from x = 0: d = s dinv b (the first step's residual is b, its x is d)
static __global__ void k_cheb_start(const float* __restrict__ b, const float* __restrict__ dinv, float* __restrict__ d,
                             float s, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    d[i] = s * dinv[i] * b[i];
}

// dinv = 1 / diag (0 where the diagonal vanishes)
static __global__ void k_vec_inv(const float* __restrict__ a, float* __restrict__ b, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    b[i] = a[i] != 0.f ? 1.f / a[i] : 0.f;
}

// FP64 -> FP32 copy
static __global__ void k_to_f32(const double* __restrict__ x, float* __restrict__ y, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = (float)x[i];
}

}  // namespace pfmf
