// Host side of the FP32 p-multigrid entry points (included at the end of pfmf.hip).
#pragma once
#include <random>

namespace {

constexpr int VEC_BLOCKS = 2048;
constexpr int EPI_BLOCKS = 512;              // workgroups per field of a launch with partial sums (E_POWER)
constexpr int RED_PARTS = 4 * EPI_BLOCKS;    // their partial sums, one per workgroup and field

inline int vec_grid(int64_t n) {
  const int64_t b = (n + NT - 1) / NT;
  return (int)(b < VEC_BLOCKS ? (b > 0 ? b : 1) : VEC_BLOCKS);
}

// Nodes of the six boundary faces of a lattice, each face counted in full (k_mask's range).
inline int64_t face_nodes(int nx1, int ny1, int nz1) {
  return 2 * ((int64_t)ny1 * nz1 + (int64_t)nx1 * nz1 + (int64_t)nx1 * ny1);
}

// 1-D transfer rows between orders pf (fine) and pc (coarse) on N elements.
void transfer_rows_1d(int pf, int pc, int N, std::vector<int>& pbase, std::vector<float>& pw,
                      std::vector<int>& rbase, std::vector<float>& rw) {
  std::vector<double> xf, xc, B, D;
  gauss_lobatto(pf + 1, xf);
  gauss_lobatto(pc + 1, xc);
  lagrange_tables(xc, xf, B, D);  // B[il][j] = coarse basis j at fine node il
  const int Pc = pc + 1;
  const int nf = pf * N + 1, nc = pc * N + 1;
  pbase.assign(nf, 0);
  pw.assign((size_t)nf * Pc, 0.f);
  for (int i = 0; i < nf; ++i) {
    const int e = std::min(i / pf, N - 1);
    const int il = i - pf * e;
    pbase[i] = pc * e;
    for (int j = 0; j < Pc; ++j) pw[(size_t)i * Pc + j] = (float)B[il * Pc + j];
  }
  const int nw = 2 * pf + 1;
  rbase.assign(nc, 0);
  rw.assign((size_t)nc * nw, 0.f);
  for (int J = 0; J < nc; ++J) {
    int elo, ehi;
    if (J % pc != 0) {
      elo = ehi = J / pc;
    } else {
      elo = J / pc - 1 < 0 ? 0 : J / pc - 1;
      ehi = J / pc < N ? J / pc : N - 1;
    }
    rbase[J] = pf * elo;
    for (int k = 0; k < nw; ++k) {
      const int i = rbase[J] + k;
      if (i > pf * (ehi + 1) || i >= nf) continue;
      const int e = (i <= pf * (elo + 1)) ? elo : ehi;
      const int il = i - pf * e, j = J - pc * e;
      if (j < 0 || j > pc) continue;
      rw[(size_t)J * nw + k] = (float)B[il * Pc + j];
    }
  }
}

// 1-D transfer rows from an order-1 lattice of Nf (even) elements to the one with Nf / 2:
// fine node i takes coarse node i / 2 (even i, weight 1) or the mean of (i - 1) / 2 and
// (i + 1) / 2 (odd i); restriction is the transpose (weights 1/2, 1, 1/2).
void transfer_rows_h(int Nf, std::vector<int>& pbase, std::vector<float>& pw, std::vector<int>& rbase,
                     std::vector<float>& rw) {
  const int nf = Nf + 1, nc = Nf / 2 + 1;
  pbase.assign(nf, 0);
  pw.assign((size_t)nf * 2, 0.f);
  for (int i = 0; i < nf; ++i) {
    pbase[i] = i / 2;
    if (i % 2 == 0) {
      pw[(size_t)i * 2] = 1.f;
    } else {
      pw[(size_t)i * 2] = 0.5f;
      pw[(size_t)i * 2 + 1] = 0.5f;
    }
  }
  rbase.assign(nc, 0);
  rw.assign((size_t)nc * 3, 0.f);
  for (int J = 0; J < nc; ++J) {
    rbase[J] = 2 * J - 1;
    rw[(size_t)J * 3] = 0.5f;
    rw[(size_t)J * 3 + 1] = 1.f;
    rw[(size_t)J * 3 + 2] = 0.5f;
  }
}

template <typename T>
pf_status upload(T** dst, const std::vector<T>& v) {
  if (hipMalloc(dst, v.size() * sizeof(T)) != hipSuccess) return fail(PF_ENOMEM, "multigrid allocation failed");
  HIPCHK(hipMemcpy(*dst, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice));
  return PF_OK;
}

pf_status mg_alloc_levels(pf_ctx* c, const int* orders, int nl);

// Values of one record slot over the mesh (one layer), see rec_at.
size_t rec_points(const pf_ctx* c) {
  const size_t n_elem = (size_t)c->mesh.nx * c->mesh.ny * c->mesh.nz;
  return n_elem * rec_pad((int)(c->n_q / n_elem));
}

pf_status mg_alloc(pf_ctx* c) {
  MGState& mg = c->mg;
  if (mg.n_levels > 0) return PF_OK;
  const int p = c->mesh.p;
  int orders[MG_MAX_LEVELS];
  int nl;
  if (c->n_orders > 0) {
    nl = c->n_orders;
    for (int l = 0; l < c->n_orders; ++l) orders[l] = c->orders[l];
  } else {
    nl = p;
    for (int l = 0; l < p; ++l) orders[l] = p - l;
  }
  // n_levels becomes nl only once every buffer exists; on a failure the partial
  // hierarchy is freed (mg_free) and n_levels stays 0, so a later call starts over
  pf_status st = mg_alloc_levels(c, orders, nl);
  if (st != PF_OK) {
    mg_free(mg);
    return st;
  }
  mg.n_levels = nl;
  return PF_OK;
}

pf_status mg_alloc_levels(pf_ctx* c, const int* orders, int nl) {
  MGState& mg = c->mg;
  const int N[3] = {c->mesh.nx, c->mesh.ny, c->mesh.nz};
  for (int l = 0; l < nl; ++l) {
    MGLevel& L = mg.lv[l];
    L.p = orders[l];
    L.P = L.p + 1;
    // a repeated order 1 coarsens the order-1 lattice by two per direction
    L.h = (l > 0 && L.p == 1 && orders[l - 1] == 1) ? mg.lv[l - 1].h + 1 : 0;
    for (int k = 0; k < 3; ++k) L.ne[k] = L.h > 0 ? mg.lv[l - 1].ne[k] / 2 : N[k];
    L.nx1 = L.p * L.ne[0] + 1;
    L.ny1 = L.p * L.ne[1] + 1;
    L.nz1 = L.p * L.ne[2] + 1;
    L.n_nodes = (int64_t)L.nx1 * L.ny1 * L.nz1;
    const size_t nb = 4 * L.n_nodes * sizeof(float);
    float** bufs[] = {&L.x, &L.r, &L.d, &L.t, &L.b, &L.diag, &L.dinv};
    for (float** b : bufs)
      if (hipMalloc(b, nb) != hipSuccess) return fail(PF_ENOMEM, "multigrid level allocation failed");
    if (L.h > 0 && hipMalloc(&L.S, (size_t)stencil_size(L.n_nodes) * sizeof(float)) != hipSuccess)
      return fail(PF_ENOMEM, "coarse stencil: allocation failed");
    if (l + 1 < nl) {
      const bool hnext = L.p == 1 && orders[l + 1] == 1;
      for (int k = 0; k < 3; ++k) {
        std::vector<int> pb, rb;
        std::vector<float> pw, rw;
        if (hnext)
          transfer_rows_h(L.ne[k], pb, pw, rb, rw);
        else
          transfer_rows_1d(L.p, orders[l + 1], N[k], pb, pw, rb, rw);
        pf_status st;
        if ((st = upload(&L.pbase[k], pb)) || (st = upload(&L.pw[k], pw)) || (st = upload(&L.rbase[k], rb)) ||
            (st = upload(&L.rw[k], rw)))
          return st;
      }
    }
  }
  // the order-1 level on the mesh itself: block stencil, from element matrices; the element diagonals of
  // the levels above it, 4 (order + 1)^3 values, use the same buffer
  size_t ebe = 0;
  for (int l = 0; l < nl && mg.ebe_level < 0; ++l) {
    const MGLevel& L = mg.lv[l];
    ebe = std::max(ebe, L.p == 1 ? (size_t)1024 : (size_t)4 * L.P * L.P * L.P);
    if (L.p == 1) mg.ebe_level = l;
  }
  const int64_t n_elem = (int64_t)N[0] * N[1] * N[2];
  if (hipMalloc(&mg.ebe, n_elem * ebe * sizeof(float)) != hipSuccess ||
      (mg.ebe_level >= 0 &&
       hipMalloc(&mg.stencil, (size_t)stencil_size(mg.lv[mg.ebe_level].n_nodes) * sizeof(float)) != hipSuccess))
    return fail(PF_ENOMEM, "coarse element matrices: allocation failed");
  const size_t nfine = 4 * mg.lv[0].n_nodes * sizeof(float);
  if (hipMalloc(&mg.frame, 9 * rec_points(c) * sizeof(float)) != hipSuccess ||
      hipMalloc(&mg.tmpA, nfine) != hipSuccess || hipMalloc(&mg.tmpB, nfine) != hipSuccess ||
      hipMalloc(&mg.red, (RED_PARTS + 16) * sizeof(double)) != hipSuccess)
    return fail(PF_ENOMEM, "multigrid allocation failed");
  return PF_OK;
}

// Record arrays with one layer per branch (the block and the extra branches),
// reallocated when the number of layers changes.
pf_status ensure_records(pf_ctx* c) {
  MGState& mg = c->mg;
  const int layers = 1 + c->n_extra;
  if (mg.rec.rec && mg.rec_layers == layers) return PF_OK;
  (void)hipFree(mg.rec.rec);
  (void)hipFree(mg.rec.flags);
  (void)hipFree(mg.rec64);
  mg.rec = RecordSoA{nullptr, nullptr};
  mg.rec64 = nullptr;
  mg.rec_layers = 0;
  if (hipMalloc(&mg.rec.rec, layers * REC_N * rec_points(c) * sizeof(float)) != hipSuccess ||
      hipMalloc(&mg.rec.flags, (size_t)layers * c->n_q) != hipSuccess)
    return fail(PF_ENOMEM, "linearisation record: allocation failed");
  mg.rec_layers = layers;
  return PF_OK;
}

// Zero the constrained entries of a level vector (no-op without Dirichlet faces).
pf_status mask_level(pf_ctx* c, int level, float* v, hipStream_t s) {
  if (!c->has_dir) return PF_OK;
  const MGLevel& L = c->mg.lv[level];
  hipLaunchKernelGGL(k_mask<float>, dim3(vec_grid(face_nodes(L.nx1, L.ny1, L.nz1))), dim3(NT), 0, s, v, L.nx1, L.ny1, L.nz1, c->dir);
  HIPCHK(hipGetLastError());
  return PF_OK;
}

pf_status mask_fine64(pf_ctx* c, double* v, hipStream_t s) {
  if (!c->has_dir) return PF_OK;
  hipLaunchKernelGGL(k_mask<double>, dim3(vec_grid(face_nodes(c->nx1, c->ny1, c->nz1))), dim3(NT), 0, s, v, c->nx1, c->ny1, c->nz1, c->dir);
  HIPCHK(hipGetLastError());
  return PF_OK;
}

A32Args a32_args(pf_ctx* c, int level, const float* dz) {
  A32Args a;
  a.m = mesh_dev(c);
  const MGLevel& F = c->mg.lv[0];
  const MGLevel& L = c->mg.lv[level];
  a.fine = LevelDev{F.P, F.nx1, F.ny1, F.n_nodes};
  a.lev = LevelDev{L.P, L.nx1, L.ny1, L.n_nodes};
  a.n_q = c->n_q;
  a.frame = c->mg.frame;
  a.u = nullptr;
  a.dz = dz;
  a.rec = c->mg.rec;
  a.phase = c->qp_phase;
  a.mats = c->d_matsf;
  a.nph = (int)c->phases.size();
  a.fr = frac_params<float>(c->fr);
  a.out = nullptr;
  a.ebuf = nullptr;
  a.xmats = c->d_xmatsf;
  a.n_extra = c->n_extra;
  a.qd = c->d_qd32;
  return a;
}

// Workgroups of a launch with an epilogue: E_POWER leaves one partial sum per workgroup.
template <int OP>
int epi_blocks(int64_t blocks, int most) {
  return (int)std::min<int64_t>(blocks, OP == E_POWER ? EPI_BLOCKS : most);
}

// Node gather of an extended grid of nbx x nby x nbz blocks with the epilogue OP.
template <typename V, int NB, int OP>
pf_status launch_gather(const LinApplyArgs<V>& a, int nbx, int nby, int nbz, const Epilogue<V>& ep, hipStream_t s) {
  const int n_rows = (int)(a.lev.n_nodes / a.lev.nx1);
  hipLaunchKernelGGL((k_gather_ext<V, NB, OP>), dim3(1, epi_blocks<OP>((n_rows + 3) / 4, 65535), 4), dim3(NT), 0, s,
                     (const V*)a.ebuf, nbx, nby, nbz, a.lev.nx1, a.lev.ny1, n_rows, a.lev.n_nodes, ep);
  HIPCHK(hipGetLastError());
  return PF_OK;
}

// Colour launches write A dz whole: where E_STORE and E_POWER put their result, and to the spare
// vector otherwise (the fine level's r, d and x may be the epilogue's inputs); the epilogue follows.
template <int OP>
float* colour_out(pf_ctx* c, const LinApplyArgs<float>& a, const Epilogue<float>& ep) {
  (void)a;
  return OP == E_STORE || OP == E_POWER ? ep.out : c->mg.tmpA;
}
template <int OP>
pf_status colour_epilogue(const LinApplyArgs<float>& a, const Epilogue<float>& ep, hipStream_t s) {
  if (OP == E_STORE && !ep.has_dir) return PF_OK;
  const int nb = epi_blocks<OP>((a.lev.n_nodes + NT - 1) / NT, 65536);
  hipLaunchKernelGGL(k_epilogue<OP>, dim3(nb, 4), dim3(NT), 0, s, (const float*)a.out, a.lev.nx1, a.lev.ny1,
                     a.lev.n_nodes, ep);
  HIPCHK(hipGetLastError());
  return PF_OK;
}

// Linearised apply on the matrix cores: PF = 4 (order-3 mesh, k_a32_q3) or PF = 3
// (order-2 mesh, k_a32_q2); V = float for the FP32 levels, V = double for the apply
// from the stored FP64 linearisation (fine level). The brick buffer of each precision
// is sized for the fine level and shared by the coarser ones.
template <typename V, int PF, int PC, bool MB, bool GEO, int OP>
pf_status launch_lin_mfma_v(pf_ctx* c, LinApplyArgs<V> a, const Epilogue<V>& ep, hipStream_t s) {
  if (use_brick_buffer(c)) {
    V** buf;
    if constexpr (sizeof(V) == 4) buf = &c->mg.ebuf32;
    else buf = &c->d_ebuf;
    constexpr int NBF = 2 * PF - 1;
    if (!*buf && hipMalloc((void**)buf, (size_t)c->n_bricks * 4 * NBF * NBF * NBF * sizeof(V)) != hipSuccess)
      return fail(PF_ENOMEM, "brick buffer: allocation failed");
    a.ebuf = *buf;
    const int ng = xcd_grid_all(c->nbx, c->nby, c->nbz);
    if constexpr (PF == 4) {
      hipLaunchKernelGGL((k_a32_q3<V, PC, true, MB, GEO>), dim3(ng), dim3(NT), 0, s, a, 0, c->d_tab);
    } else if constexpr (!MB && !GEO) {
      // order 2 on box elements without branches: the row-layout kernel (no 3 -> 4 padding)
      if constexpr (sizeof(V) == 4)
        hipLaunchKernelGGL((k_a32_q2r<V, PC>), dim3(ng), dim3(NT), 0, s, a, c->d_tabf);
      else
        hipLaunchKernelGGL((k_a32_q2r<V, PC>), dim3(ng), dim3(NT), 0, s, a, c->d_tab);
    } else {
      hipLaunchKernelGGL((k_a32_q2<V, PC, true, MB, GEO>), dim3(ng), dim3(NT), 0, s, a, 0, c->d_tab);
    }
    HIPCHK(hipGetLastError());
    return launch_gather<V, 2 * PC - 1, OP>(a, a.m.nbx, a.m.nby, a.m.nbz, ep, s);
  }
  if constexpr (sizeof(V) == 4) a.out = colour_out<OP>(c, a, ep);
  else a.out = ep.out;
  for (int col = 0; col < 8; ++col) {
    const int nb = xcd_grid(c->nbx, c->nby, c->nbz, col);
    if (nb == 0) continue;
    if constexpr (PF == 4)
      hipLaunchKernelGGL((k_a32_q3<V, PC, false, MB, GEO>), dim3(nb), dim3(NT), 0, s, a, col, c->d_tab);
    else
      hipLaunchKernelGGL((k_a32_q2<V, PC, false, MB, GEO>), dim3(nb), dim3(NT), 0, s, a, col, c->d_tab);
    HIPCHK(hipGetLastError());
  }
  if constexpr (sizeof(V) == 4) return colour_epilogue<OP>(a, ep, s);
  return PF_OK;
}

template <typename V, int PF, int PC, int OP>
pf_status launch_lin_mfma(pf_ctx* c, const LinApplyArgs<V>& a, const Epilogue<V>& ep, hipStream_t s) {
  if (a.qd)
    return a.n_extra > 0 ? launch_lin_mfma_v<V, PF, PC, true, true, OP>(c, a, ep, s)
                         : launch_lin_mfma_v<V, PF, PC, false, true, OP>(c, a, ep, s);
  return a.n_extra > 0 ? launch_lin_mfma_v<V, PF, PC, true, false, OP>(c, a, ep, s)
                       : launch_lin_mfma_v<V, PF, PC, false, false, OP>(c, a, ep, s);
}

template <typename V, int PC, bool MB, bool GEO, int OP>
pf_status launch_lin_q4_v(pf_ctx* c, const LinApplyArgs<V>& a0, const Epilogue<V>& ep, hipStream_t s) {
  LinApplyArgs<V> a = a0;
  if (use_brick_buffer(c)) {
    // element vectors of the level (buffer sized for the fine level), then the node gather
    V** buf;
    if constexpr (sizeof(V) == 4) buf = &c->mg.ebuf32;
    else buf = &c->d_ebuf;
    const int64_t n_elem = (int64_t)c->mesh.nx * c->mesh.ny * c->mesh.nz;
    if (!*buf && hipMalloc((void**)buf, (size_t)n_elem * 4 * 125 * sizeof(V)) != hipSuccess)
      return fail(PF_ENOMEM, "element-vector buffer: allocation failed");
    a.ebuf = *buf;
    const int ng = xcd_grid_elems(c->mesh.nx, c->mesh.ny, c->mesh.nz);
    if constexpr (sizeof(V) == 4)
      hipLaunchKernelGGL((k_a32_q4<V, PC, MB, GEO, true>), dim3(ng), dim3(NT5), 0, s, a, 0, c->d_tabf);
    else
      hipLaunchKernelGGL((k_a32_q4<V, PC, MB, GEO, true>), dim3(ng), dim3(NT5), 0, s, a, 0, c->d_tab);
    HIPCHK(hipGetLastError());
    return launch_gather<V, PC, OP>(a, a.m.nx, a.m.ny, a.m.nz, ep, s);
  }
  if constexpr (sizeof(V) == 4) a.out = colour_out<OP>(c, a, ep);
  else a.out = ep.out;
  for (int col = 0; col < 8; ++col) {
    const int ng = xcd_grid(c->mesh.nx, c->mesh.ny, c->mesh.nz, col);
    if (ng == 0) continue;
    if constexpr (sizeof(V) == 4)
      hipLaunchKernelGGL((k_a32_q4<V, PC, MB, GEO>), dim3(ng), dim3(NT5), 0, s, a, col, c->d_tabf);
    else
      hipLaunchKernelGGL((k_a32_q4<V, PC, MB, GEO>), dim3(ng), dim3(NT5), 0, s, a, col, c->d_tab);
    HIPCHK(hipGetLastError());
  }
  if constexpr (sizeof(V) == 4) return colour_epilogue<OP>(a, ep, s);
  return PF_OK;
}

template <typename V, int PC, int OP>
pf_status launch_lin_q4(pf_ctx* c, const LinApplyArgs<V>& a, const Epilogue<V>& ep, hipStream_t s) {
  if (a.qd)
    return a.n_extra > 0 ? launch_lin_q4_v<V, PC, true, true, OP>(c, a, ep, s)
                         : launch_lin_q4_v<V, PC, false, true, OP>(c, a, ep, s);
  return a.n_extra > 0 ? launch_lin_q4_v<V, PC, true, false, OP>(c, a, ep, s)
                       : launch_lin_q4_v<V, PC, false, false, OP>(c, a, ep, s);
}

EbeArgs ebe_args(pf_ctx* c) {
  EbeArgs a;
  a.m = mesh_dev(c);
  a.n_q = c->n_q;
  a.frame = c->mg.frame;
  a.rec = c->mg.rec;
  a.phase = c->qp_phase;
  a.mats = c->d_matsf;
  a.nph = (int)c->phases.size();
  a.fr = frac_params<float>(c->fr);
  a.K = c->mg.ebe;
  a.xmats = c->d_xmatsf;
  a.n_extra = c->n_extra;
  a.qd = c->d_qd;
  return a;
}

template <int PF>
pf_status launch_ebe(const EbeArgs& a, const DevTablesF* tabs, hipStream_t s) {
  const int64_t n_elem = (int64_t)a.m.nx * a.m.ny * a.m.nz;
  const dim3 nb((unsigned)((n_elem + EbeShape<PF>::NE - 1) / EbeShape<PF>::NE));
  const bool mb = a.n_extra > 0;
  if constexpr (PF == 2) {  // order 1: no branches, no mapped elements
    hipLaunchKernelGGL((k_ebe_assemble<PF, false>), nb, dim3(NT), 0, s, a, tabs);
  } else {
    if (a.qd && mb)
      hipLaunchKernelGGL((k_ebe_assemble<PF, true, true>), nb, dim3(NT), 0, s, a, tabs);
    else if (a.qd)
      hipLaunchKernelGGL((k_ebe_assemble<PF, false, true>), nb, dim3(NT), 0, s, a, tabs);
    else if (mb)
      hipLaunchKernelGGL((k_ebe_assemble<PF, true>), nb, dim3(NT), 0, s, a, tabs);
    else
      hipLaunchKernelGGL((k_ebe_assemble<PF, false>), nb, dim3(NT), 0, s, a, tabs);
  }
  HIPCHK(hipGetLastError());
  return PF_OK;
}

pf_status ebe_assemble(pf_ctx* c, hipStream_t s) {
  const EbeArgs a = ebe_args(c);
  pf_status st;
  switch (c->mg.lv[0].P) {
    case 2: st = launch_ebe<2>(a, c->d_tabf, s); break;
    case 3: st = launch_ebe<3>(a, c->d_tabf, s); break;
    case 4: st = launch_ebe<4>(a, c->d_tabf, s); break;
    case 5: st = launch_ebe<5>(a, c->d_tabf, s); break;
    default: return fail(PF_EUNSUPPORTED, "order not built");
  }
  if (st) return st;
  const MGLevel& L = c->mg.lv[c->mg.ebe_level];
  hipLaunchKernelGGL(k_stencil_from_ebe, dim3((unsigned)((L.n_nodes + 63) / 64), 4), dim3(NT), 0, s, c->mg.ebe, c->mesh.nx, c->mesh.ny, c->mesh.nz,
                     L.n_nodes, c->mg.stencil);
  HIPCHK(hipGetLastError());
  return PF_OK;
}

// Block stencil of an order-1 level: the mesh's own (mg.stencil) or a coarser lattice's S.
const float* level_stencil(const pf_ctx* c, int level) {
  return c->mg.lv[level].h > 0 ? c->mg.lv[level].S : c->mg.stencil;
}

template <int OP>
pf_status stencil_apply(pf_ctx* c, int level, const float* x, const Epilogue<float>& ep, hipStream_t s) {
  const MGLevel& L = c->mg.lv[level];
  const int nb = epi_blocks<OP>((L.n_nodes + NT - 1) / NT, 65536);
  hipLaunchKernelGGL(k_stencil_apply<OP>, dim3(nb, 4), dim3(NT), 0, s, level_stencil(c, level), L.nx1, L.ny1, L.nz1,
                     L.n_nodes, x, ep);
  HIPCHK(hipGetLastError());
  return PF_OK;
}

// Galerkin stencils of the coarser order-1 lattices, each from the level above it.
pf_status build_h_levels(pf_ctx* c, hipStream_t s) {
  MGState& mg = c->mg;
  for (int l = 1; l < mg.n_levels; ++l) {
    const MGLevel& L = mg.lv[l];
    if (L.h == 0) continue;
    const MGLevel& F = mg.lv[l - 1];
    const float* Sf = F.h > 0 ? F.S : mg.stencil;
    const int nb = (int)std::min<int64_t>((L.n_nodes + NT - 1) / NT, 65536);
    hipLaunchKernelGGL(k_stencil_rap, dim3(nb, 27, 4), dim3(NT), 0, s, Sf, F.nx1, F.ny1, F.nz1, L.S, L.nx1, L.ny1, L.nz1);
    HIPCHK(hipGetLastError());
  }
  return PF_OK;
}

// True where the level's operator is a block stencil: the order-1 level on the mesh and the
// coarser lattices below it.
bool is_stencil(const pf_ctx* c, int level) { return c->mg.lv[level].h > 0 || level == c->mg.ebe_level; }

// Level operator with Dirichlet faces (M A dz: vectors that vanish on constrained entries stay in
// that subspace), each entry passed to the epilogue OP. On a stencil level the epilogue must not
// write dz.
template <int OP>
pf_status level_op(pf_ctx* c, int level, const float* dz, Epilogue<float> ep, hipStream_t s) {
  const MGLevel& L = c->mg.lv[level];
  ep.dir = c->dir;
  ep.has_dir = c->has_dir;
  ep.nz1 = L.nz1;
  if (is_stencil(c, level)) return stencil_apply<OP>(c, level, dz, ep, s);
  const A32Args a = a32_args(c, level, dz);
  switch (c->mg.lv[0].P * 10 + L.P) {
    case 55: return launch_lin_q4<float, 5, OP>(c, a, ep, s);
    case 54: return launch_lin_q4<float, 4, OP>(c, a, ep, s);
    case 53: return launch_lin_q4<float, 3, OP>(c, a, ep, s);
    case 44: return launch_lin_mfma<float, 4, 4, OP>(c, a, ep, s);
    case 43: return launch_lin_mfma<float, 4, 3, OP>(c, a, ep, s);
    case 33: return launch_lin_mfma<float, 3, 3, OP>(c, a, ep, s);
    default: return fail(PF_EUNSUPPORTED, "level order not built");
  }
}

// Partial sums that E_POWER leaves on a level (one per workgroup of the launch that runs it).
pf_status power_parts(const pf_ctx* c, int level, int& parts) {
  const MGLevel& L = c->mg.lv[level];
  const int64_t per_block = is_stencil(c, level) || !use_brick_buffer(c) ? NT : 4 * (int64_t)L.nx1;
  parts = 4 * epi_blocks<E_POWER>((L.n_nodes + per_block - 1) / per_block, 0);
  return parts <= RED_PARTS ? PF_OK : fail(PF_EHIP, "reduction scratch too small");
}

// Point-Jacobi diagonal of one level (unmasked).
template <int PF, int PC>
pf_status launch_diag(pf_ctx* c, const EbeArgs& a, const MGLevel& L, float* out, hipStream_t s) {
  const int64_t n_elem = (int64_t)a.m.nx * a.m.ny * a.m.nz;
  const dim3 nb((unsigned)((n_elem + EbeShape<PF>::NE - 1) / EbeShape<PF>::NE));
  const bool mb = a.n_extra > 0;
  float* ev = c->mg.ebe;
  const DevTablesF* tabs = c->d_tabf;
  if (a.qd && mb)
    hipLaunchKernelGGL((k_level_diag<PF, PC, true, true>), nb, dim3(NT), 0, s, a, ev, tabs);
  else if (a.qd)
    hipLaunchKernelGGL((k_level_diag<PF, PC, false, true>), nb, dim3(NT), 0, s, a, ev, tabs);
  else if (mb)
    hipLaunchKernelGGL((k_level_diag<PF, PC, true>), nb, dim3(NT), 0, s, a, ev, tabs);
  else
    hipLaunchKernelGGL((k_level_diag<PF, PC, false>), nb, dim3(NT), 0, s, a, ev, tabs);
  HIPCHK(hipGetLastError());
  const int n_rows = (int)(L.n_nodes / L.nx1);
  hipLaunchKernelGGL((k_gather_ext<float, PC, E_STORE>), dim3(1, std::min((n_rows + 3) / 4, 65535), 4), dim3(NT), 0, s,
                     (const float*)ev, a.m.nx, a.m.ny, a.m.nz, L.nx1, L.ny1, n_rows, L.n_nodes, store_epilogue(out));
  HIPCHK(hipGetLastError());
  return PF_OK;
}

pf_status level_diagonal(pf_ctx* c, int level, float* out, hipStream_t s) {
  const MGLevel& L = c->mg.lv[level];
  if (is_stencil(c, level)) {
    hipLaunchKernelGGL(k_stencil_diag, dim3(vec_grid(L.n_nodes), 4), dim3(NT), 0, s, level_stencil(c, level), L.n_nodes,
                       out);
    HIPCHK(hipGetLastError());
    return PF_OK;
  }
  const EbeArgs a = ebe_args(c);
  switch (c->mg.lv[0].P * 10 + L.P) {
    case 55: return launch_diag<5, 5>(c, a, L, out, s);
    case 54: return launch_diag<5, 4>(c, a, L, out, s);
    case 53: return launch_diag<5, 3>(c, a, L, out, s);
    case 44: return launch_diag<4, 4>(c, a, L, out, s);
    case 43: return launch_diag<4, 3>(c, a, L, out, s);
    case 33: return launch_diag<3, 3>(c, a, L, out, s);
    default: return fail(PF_EUNSUPPORTED, "level order not built");
  }
}

template <int P, int MODE, bool GEO = false>
pf_status launch_linearize(pf_ctx* c, const LinArgs& a, hipStream_t s) {
  using S = OpShape<P, P>;
  const size_t lds = (4 * S::NB3 + S::TMP + S::TAB) * sizeof(double);
  static bool attr_set = false;
  if (!attr_set) {
    HIPCHK(hipFuncSetAttribute((const void*)k_linearize<P, P, MODE, GEO>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)lds));
    attr_set = true;
  }
  hipLaunchKernelGGL((k_linearize<P, P, MODE, GEO>), dim3(xcd_grid_all(c->nbx, c->nby, c->nbz)), dim3(NT), lds, s, a,
                     c->d_tab);
  HIPCHK(hipGetLastError());
  return PF_OK;
}

// One launch for the three directions up to 4^3 inputs per node: every prolongation, and the
// restriction between order-1 lattices. The small levels pay the launches, the large ones the passes
// over intermediate lattices: 17^3 nodes from 2^3 inputs 12 -> 5 us, 97^3 from 3^3 34 -> 31, 161^3 from
// 3^3 125 -> 92, order 3 to 4 on 32^3 elements 71 -> 66. The 5^3 inputs of the restriction from order 2
// took 25 us on 41^3 nodes against 19 in three passes, so it and the wider ones stay there.
template <int NW>
pf_status transfer_nw(pf_ctx* c, const float* in, const MGLevel& I, float* out, const MGLevel& O, const TransferAxes& ax,
                      bool add, hipStream_t s) {
  const unsigned nb = (unsigned)(((int64_t)O.nx1 * O.ny1 + NT - 1) / NT);
  // outputs per thread: as many as an element's nodes share planes, where the rest fills the chip
  // (256 CUs, 8 workgroups each); at most 65535 groups
  int zb = (int64_t)nb * 4 * O.nz1 >= 4 * 2048 ? 4 : 1;
  zb = std::max(zb, (O.nz1 + 65534) / 65535);
  hipLaunchKernelGGL(k_transfer<NW>, dim3(nb, 4, (O.nz1 + zb - 1) / zb), dim3(NT), 0, s, in, out, O.nx1, O.ny1, O.nz1,
                     I.nx1, I.ny1, I.nz1, ax, zb, add ? 1 : 0, c->dir, c->has_dir ? 1 : 0);
  HIPCHK(hipGetLastError());
  return PF_OK;
}

pf_status transfer(pf_ctx* c, const float* in, const MGLevel& I, float* out, const MGLevel& O, int* const* base,
                   float* const* w, int nw, bool add, hipStream_t s) {
  const TransferAxes ax{{base[0], base[1], base[2]}, {w[0], w[1], w[2]}};
  // vectors that overlap go through the intermediate lattices: one launch would read what it has written
  const bool apart = !overlaps(in, 4 * I.n_nodes * sizeof(float), out, 4 * O.n_nodes * sizeof(float));
  switch (apart ? nw : 0) {
    case 2: return transfer_nw<2>(c, in, I, out, O, ax, add, s);
    case 3: return transfer_nw<3>(c, in, I, out, O, ax, add, s);
    case 4: return transfer_nw<4>(c, in, I, out, O, ax, add, s);
    default: break;
  }
  float* A = c->mg.tmpA;
  float* B = c->mg.tmpB;
  int64_t n = (int64_t)O.nx1 * I.ny1 * I.nz1;
  hipLaunchKernelGGL(k_transfer_1d, dim3(vec_grid(n)), dim3(NT), 0, s, in, A, O.nx1, I.ny1, I.nz1, I.nx1, I.ny1, I.nz1,
                     0, base[0], w[0], nw, 0, c->dir, 0);
  n = (int64_t)O.nx1 * O.ny1 * I.nz1;
  hipLaunchKernelGGL(k_transfer_1d, dim3(vec_grid(n)), dim3(NT), 0, s, A, B, O.nx1, O.ny1, I.nz1, O.nx1, I.ny1, I.nz1,
                     1, base[1], w[1], nw, 0, c->dir, 0);
  n = O.n_nodes;
  hipLaunchKernelGGL(k_transfer_1d, dim3(vec_grid(n)), dim3(NT), 0, s, B, out, O.nx1, O.ny1, O.nz1, O.nx1, O.ny1, I.nz1,
                     2, base[2], w[2], nw, add ? 1 : 0, c->dir, c->has_dir ? 1 : 0);
  HIPCHK(hipGetLastError());
  return PF_OK;
}

// xf (+)= P xc (coarse level l+1 -> level l), masked.
pf_status prolong(pf_ctx* c, int l, const float* xc, float* xf, bool add, hipStream_t s) {
  const MGLevel& F = c->mg.lv[l];
  const MGLevel& C = c->mg.lv[l + 1];
  return transfer(c, xc, C, xf, F, F.pbase, F.pw, C.P, add, s);
}

// rc = P^T rf (level l -> coarse level l+1), masked.
pf_status restrict_(pf_ctx* c, int l, const float* rf, float* rc, hipStream_t s) {
  const MGLevel& F = c->mg.lv[l];
  const MGLevel& C = c->mg.lv[l + 1];
  return transfer(c, rf, F, rc, C, F.rbase, F.rw, 2 * F.p + 1, false, s);
}

// Chebyshev(k) with point Jacobi on level l for A x = b, bounds [0.1, 1.1] * lmax; x_zero: from
// x = 0 (x is written, not read). The correction d alternates between two vectors, since a
// stencil level must not overwrite the vector it applies to.
pf_status chebyshev(pf_ctx* c, int l, const float* b, float* x, int k, bool x_zero, hipStream_t s) {
  MGLevel& L = c->mg.lv[l];
  const int64_t n = 4 * L.n_nodes;
  const int g = vec_grid(n);
  const double lmin = 0.1 * L.lmax, lhi = 1.1 * L.lmax;
  const double theta = 0.5 * (lhi + lmin), delta = 0.5 * (lhi - lmin), sigma = theta / delta;
  double rho = 1.0 / sigma;
  pf_status st;
  Epilogue<float> e{};
  e.dinv = L.dinv;
  e.c = (float)(1.0 / theta);
  if (x_zero) {
    float* d = k > 1 ? L.d : x;
    hipLaunchKernelGGL(k_cheb_start, dim3(g), dim3(NT), 0, s, b, L.dinv, d, e.c, n);
    HIPCHK(hipGetLastError());
    if (k <= 1) return PF_OK;
  } else {
    e.b = b;
    e.r = L.r;
    e.d = L.d;
    if ((st = level_op<E_FIRST>(c, l, x, e, s))) return st;
    if (k <= 1) {
      hipLaunchKernelGGL(k_vec_add, dim3(g), dim3(NT), 0, s, (const float*)L.d, x, n);
      HIPCHK(hipGetLastError());
      return PF_OK;
    }
  }
  float *d = L.d, *dn = L.t;
  for (int it = 1; it < k; ++it) {
    const double rn = 1.0 / (2.0 * sigma - rho);
    e.r_in = it == 1 && x_zero ? b : L.r;
    e.r = L.r;
    e.d_in = d;
    e.d = dn;
    e.x_in = it == 1 && x_zero ? nullptr : x;
    e.x = x;
    e.x_first = it == 1;
    e.a = (float)(rn * rho);
    e.c = (float)(2.0 * rn / delta);
    if ((st = it + 1 < k ? level_op<E_STEP>(c, l, d, e, s) : level_op<E_LAST>(c, l, d, e, s))) return st;
    std::swap(d, dn);
    rho = rn;
  }
  return PF_OK;
}

// The sweeps of the coarsest level in one workgroup (n_nodes <= COARSE_SOLVE_NODES, degree <= 32).
pf_status coarse_solve(pf_ctx* c, int l, const float* b, float* x, int degree, int sweeps, hipStream_t s) {
  const MGLevel& L = c->mg.lv[l];
  const double lmin = 0.1 * L.lmax, lhi = 1.1 * L.lmax;
  const double theta = 0.5 * (lhi + lmin), delta = 0.5 * (lhi - lmin), sigma = theta / delta;
  double rho = 1.0 / sigma;
  ChebCoefs co{};
  co.c0 = (float)(1.0 / theta);
  for (int it = 1; it < degree; ++it) {
    const double rn = 1.0 / (2.0 * sigma - rho);
    co.a[it - 1] = (float)(rn * rho);
    co.c[it - 1] = (float)(2.0 * rn / delta);
    rho = rn;
  }
  const int n = (int)L.n_nodes;
  hipLaunchKernelGGL(k_coarse_solve, dim3(1), dim3(4 * COARSE_SOLVE_NODES), 0, s, level_stencil(c, l), L.nx1, L.ny1,
                     L.nz1, n, b, L.dinv, x, degree, sweeps, co, c->dir, c->has_dir ? 1 : 0);
  HIPCHK(hipGetLastError());
  return PF_OK;
}

pf_status vcycle(pf_ctx* c, int l, const float* b, float* x, const pf_pmg_opts& o, hipStream_t s) {
  MGState& mg = c->mg;
  MGLevel& L = mg.lv[l];
  pf_status st;
  if (l == mg.n_levels - 1) {
    if (is_stencil(c, l) && L.n_nodes <= COARSE_SOLVE_NODES)
      return coarse_solve(c, l, b, x, o.cheb_degree, o.coarse_sweeps, s);
    for (int sw = 0; sw < o.coarse_sweeps; ++sw)
      if ((st = chebyshev(c, l, b, x, o.cheb_degree, sw == 0, s))) return st;
    return PF_OK;
  }
  if ((st = chebyshev(c, l, b, x, o.cheb_degree, true, s))) return st;
  Epilogue<float> e{};
  e.b = b;
  e.r = L.r;
  if ((st = level_op<E_RESID>(c, l, x, e, s))) return st;
  MGLevel& C = mg.lv[l + 1];
  if ((st = restrict_(c, l, L.r, C.b, s))) return st;
  if ((st = vcycle(c, l + 1, C.b, C.x, o, s))) return st;
  if ((st = prolong(c, l, C.x, x, true, s))) return st;
  return chebyshev(c, l, b, x, o.cheb_degree, false, s);
}

pf_status need_lin(pf_ctx* c, int level) {
  pf_status st = check_ctx(c);
  if (st) return st;
  if (!c->mg.linearized) return fail(PF_EINVAL, "call pf_linearize first");
  if (level < 0 || level >= c->mg.n_levels) return fail(PF_EINVAL, "level %d outside 0..%d", level, c->mg.n_levels - 1);
  return PF_OK;
}

}  // namespace

extern "C" {

pf_status pf_linearize(pf_ctx* c, const double* z, void* stream) {
  pf_status st = check_ctx(c);
  if (st) return st;
  if ((st = box_only(c, "pf_linearize"))) return st;
  if (!z) return fail(PF_EINVAL, "null z");
  if (c->n_extra > 0 && c->mesh.p < 2) return fail(PF_EUNSUPPORTED, "extra branches need p >= 2");
  hipStream_t s = (hipStream_t)stream;
  c->last_stream = s;
  if ((st = mg_alloc(c)) || (st = ensure_records(c))) return st;
  MGState& mg = c->mg;
  if (c->store_lin64) {
    if ((!mg.rec64 && hipMalloc(&mg.rec64, mg.rec_layers * REC_N * rec_points(c) * sizeof(double)) != hipSuccess) ||
        (!mg.u64 && hipMalloc(&mg.u64, (size_t)3 * c->n_nodes * sizeof(double)) != hipSuccess))
      return fail(PF_ENOMEM, "stored linearisation: allocation failed");
    HIPCHK(hipMemcpyAsync(mg.u64, z, (size_t)3 * c->n_nodes * sizeof(double), hipMemcpyDeviceToDevice, s));
  }
  LinArgs a;
  a.m = mesh_dev(c);
  a.nx1 = c->nx1;
  a.ny1 = c->ny1;
  a.n_nodes = c->n_nodes;
  a.n_q = c->n_q;
  a.z = z;
  a.phin = c->phi_n;
  a.state = c->qp_state;
  a.phase = c->qp_phase;
  a.mats = c->d_mats;
  a.nph = (int)c->phases.size();
  a.fr = frac_params<double>(c->fr);
  a.rec = mg.rec;
  a.frame = mg.frame;
  a.rec64 = c->store_lin64 ? mg.rec64 : nullptr;
  a.state_out = nullptr;
  a.flag = c->d_flag;
  a.xb = c->d_xb;
  a.xstate = c->xstate;
  a.n_extra = c->n_extra;
  a.xstate_out = nullptr;
  a.qd = c->d_qd;
  const bool mb = c->n_extra > 0;
  if (c->d_qd) {  // mapped elements (orders 2-4: pf_set_geometry checks it)
    switch (c->mesh.p) {
      case 2: st = mb ? launch_linearize<3, 2, true>(c, a, s) : launch_linearize<3, 0, true>(c, a, s); break;
      case 3: st = mb ? launch_linearize<4, 2, true>(c, a, s) : launch_linearize<4, 0, true>(c, a, s); break;
      case 4: st = mb ? launch_linearize<5, 2, true>(c, a, s) : launch_linearize<5, 0, true>(c, a, s); break;
      default: st = fail(PF_EUNSUPPORTED, "order not built");
    }
  } else switch (c->mesh.p) {
    case 1: st = launch_linearize<2, 0>(c, a, s); break;
    case 2: st = mb ? launch_linearize<3, 2>(c, a, s) : launch_linearize<3, 0>(c, a, s); break;
    case 3: st = mb ? launch_linearize<4, 2>(c, a, s) : launch_linearize<4, 0>(c, a, s); break;
    case 4: st = mb ? launch_linearize<5, 2>(c, a, s) : launch_linearize<5, 0>(c, a, s); break;
    default: st = fail(PF_EUNSUPPORTED, "order not built");
  }
  if (st) return st;
  if (mg.ebe_level >= 0 && (st = ebe_assemble(c, s))) return st;
  if ((st = build_h_levels(c, s))) return st;
  mg.linearized = true;
  mg.lin64_valid = c->store_lin64;
  // lambda_max(D^-1 A) per level by 15 power iterations, normalised on the device
  // (no host round trip inside the loop); one synchronisation at the end
  constexpr int POWER_ITS = 15;
  double* nrm = mg.red + RED_PARTS;             // [n_levels] final norms
  float* inv = (float*)(mg.red + RED_PARTS + 8);  // scale of the next vector applied
  for (int l = 0; l < mg.n_levels; ++l) {
    MGLevel& L = mg.lv[l];
    const int64_t n = 4 * L.n_nodes;
    const int g = vec_grid(n);
    if ((st = level_diagonal(c, l, L.diag, s))) return st;
    hipLaunchKernelGGL(k_vec_inv, dim3(g), dim3(NT), 0, s, L.diag, L.dinv, n);
    hipLaunchKernelGGL(k_hash_fill, dim3(g), dim3(NT), 0, s, L.d, n, (uint64_t)(21150 + l));
    if ((st = mask_level(c, l, L.d, s))) return st;
    HIPCHK(hipGetLastError());
    // v <- D^-1 A v / ||v||, the scale applied to A v; the entries start within 1. The norm is taken
    // before the last apply, whose growth is the estimate, and after every fourth: in between v grows by
    // at most lambda^4, far inside the FP32 range, and a norm costs a launch and a gather whose
    // workgroups are limited to its partial sums (linearisation of order 3 on 32^3 elements, three levels:
    // 3.39 -> 3.19 ms without 11 of 16 norms a level)
    Epilogue<float> e{};
    e.dinv = L.dinv;
    e.part = mg.red;
    float *v = L.d, *w = L.t;
    int parts = 0;
    if ((st = power_parts(c, l, parts))) return st;
    for (int it = 0; it < POWER_ITS; ++it) {
      e.out = w;
      if (it % 4 == 3 || it >= POWER_ITS - 2) {
        if ((st = level_op<E_POWER>(c, l, v, e, s))) return st;
        hipLaunchKernelGGL(k_norm_finish, dim3(1), dim3(NT), 0, s, mg.red, parts, nrm + l, inv);
        HIPCHK(hipGetLastError());
        e.inv = inv;
      } else {
        if ((st = level_op<E_SCALE>(c, l, v, e, s))) return st;
        e.inv = nullptr;
      }
      std::swap(v, w);
    }
  }
  double lam[MG_MAX_LEVELS];
  HIPCHK(hipMemcpyAsync(lam, nrm, mg.n_levels * sizeof(double), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  for (int l = 0; l < mg.n_levels; ++l) {
    if (!(lam[l] > 0.0) || !std::isfinite(lam[l])) return fail(PF_ENONPHYSICAL, "eigenvalue estimate failed on level %d", l);
    mg.lv[l].lmax = lam[l];
  }
  return PF_OK;
}

}  // extern "C"

namespace {

// New per-point state after a converged step (see commit_from_state).
pf_status commit_state(pf_ctx* c, const double* z, double* state_out, double* xstate_out, void* stream) {
  pf_status st = check_ctx(c);
  if (st) return st;
  if ((st = box_only(c, "the state commit"))) return st;
  if (!z || !state_out) return fail(PF_EINVAL, "null argument");
  const size_t ns = 8 * c->n_q * sizeof(double);
  const size_t nz = 4 * c->n_nodes * sizeof(double);
  if (overlaps(state_out, ns, c->qp_state, ns)) return fail(PF_EINVAL, "state_out aliases the context's state");
  if (overlaps(state_out, ns, z, nz)) return fail(PF_EINVAL, "state_out aliases z");
  if (xstate_out) {
    const size_t nx = (size_t)7 * c->n_extra * c->n_q * sizeof(double);
    if (overlaps(xstate_out, nx, c->xstate, nx) || overlaps(xstate_out, nx, c->qp_state, ns) ||
        overlaps(xstate_out, nx, state_out, ns) || overlaps(xstate_out, nx, z, nz))
      return fail(PF_EINVAL, "xstate_out aliases an input or state_out");
  }
  hipStream_t s = (hipStream_t)stream;
  c->last_stream = s;
  LinArgs a;
  a.m = mesh_dev(c);
  a.nx1 = c->nx1;
  a.ny1 = c->ny1;
  a.n_nodes = c->n_nodes;
  a.n_q = c->n_q;
  a.z = z;
  a.phin = c->phi_n;
  a.state = c->qp_state;
  a.phase = c->qp_phase;
  a.mats = c->d_mats;
  a.nph = (int)c->phases.size();
  a.fr = frac_params<double>(c->fr);
  a.rec = RecordSoA{nullptr, nullptr};
  a.frame = nullptr;
  a.rec64 = nullptr;
  a.state_out = state_out;
  a.flag = c->d_flag;
  a.xb = c->d_xb;
  a.xstate = c->xstate;
  a.n_extra = c->n_extra;
  a.xstate_out = xstate_out;
  a.qd = c->d_qd;
  const bool mb = c->n_extra > 0;
  if (c->d_qd) {  // mapped elements (orders 2-4: pf_set_geometry checks it)
    switch (c->mesh.p) {
      case 2: return mb ? launch_linearize<3, 3, true>(c, a, s) : launch_linearize<3, 1, true>(c, a, s);
      case 3: return mb ? launch_linearize<4, 3, true>(c, a, s) : launch_linearize<4, 1, true>(c, a, s);
      case 4: return mb ? launch_linearize<5, 3, true>(c, a, s) : launch_linearize<5, 1, true>(c, a, s);
      default: return fail(PF_EUNSUPPORTED, "order not built");
    }
  }
  switch (c->mesh.p) {
    case 1: return launch_linearize<2, 1>(c, a, s);
    case 2: return mb ? launch_linearize<3, 3>(c, a, s) : launch_linearize<3, 1>(c, a, s);
    case 3: return mb ? launch_linearize<4, 3>(c, a, s) : launch_linearize<4, 1>(c, a, s);
    case 4: return mb ? launch_linearize<5, 3>(c, a, s) : launch_linearize<5, 1>(c, a, s);
    default: return fail(PF_EUNSUPPORTED, "order not built");
  }
}

}  // namespace

extern "C" {

pf_status pf_commit_state(pf_ctx* c, const double* z, double* state_out, void* stream) {
  if (c && c->table) return fail(PF_EUNSUPPORTED, "the state commit needs the box lattice");
  if (c && c->n_extra > 0)
    return fail(PF_EUNSUPPORTED, "extra branches attached: use pf_commit_state_branches");
  return commit_state(c, z, state_out, nullptr, stream);
}

pf_status pf_commit_state_branches(pf_ctx* c, const double* z, double* state_out, double* xstate_out,
                                   void* stream) {
  if (c && c->n_extra == 0) return fail(PF_EINVAL, "no extra branch attached: use pf_commit_state");
  if (!xstate_out) return fail(PF_EINVAL, "null xstate_out");
  return commit_state(c, z, state_out, xstate_out, stream);
}

pf_status pf_set_pmg_levels(pf_ctx* c, const int* orders, int n_levels) {
  pf_status st = check_ctx(c);
  if (st) return st;
  if ((st = box_only(c, "pf_set_pmg_levels"))) return st;
  if (n_levels < 0 || n_levels > MG_MAX_LEVELS)
    return fail(PF_EINVAL, "n_levels=%d outside 0..%d", n_levels, MG_MAX_LEVELS);
  if (n_levels > 0 && !orders) return fail(PF_EINVAL, "null orders");
  if (n_levels > 0) {
    if (orders[0] != c->mesh.p) return fail(PF_EINVAL, "the first level must be the mesh order %d", c->mesh.p);
    if (n_levels < 2) return fail(PF_EINVAL, "at least two levels");
    int ne[3] = {c->mesh.nx, c->mesh.ny, c->mesh.nz};
    for (int l = 1; l < n_levels; ++l) {
      if (orders[l] == 1 && orders[l - 1] == 1) {  // a coarser order-1 lattice
        for (int k = 0; k < 3; ++k) {
          if (ne[k] % 2 != 0 || ne[k] < 2)
            return fail(PF_EINVAL, "level %d: an order-1 lattice of %d elements per direction cannot be halved", l,
                        ne[k]);
          ne[k] /= 2;
        }
        continue;
      }
      if (!(orders[l] >= 1 && orders[l] < orders[l - 1]))
        return fail(PF_EINVAL, "orders must decrease to 1, then may repeat 1");
    }
  }
  HIPCHK(hipDeviceSynchronize());
  mg_free(c->mg);
  c->n_orders = n_levels;
  for (int l = 0; l < n_levels; ++l) c->orders[l] = orders[l];
  return PF_OK;
}

pf_status pf_set_dirichlet(pf_ctx* c, const uint32_t* face_fields) {
  pf_status st = check_ctx(c);
  if (st) return st;
  if ((st = box_only(c, "pf_set_dirichlet"))) return st;
  if (!face_fields) return fail(PF_EINVAL, "null face_fields");
  bool any = false;
  for (int k = 0; k < 6; ++k) {
    if (face_fields[k] & ~0xFu) return fail(PF_EINVAL, "face %d: only bits 0..3 (fields) allowed", k);
    c->dir.face[k] = face_fields[k];
    any |= face_fields[k] != 0;
  }
  c->has_dir = any;
  // the diagonals and eigenvalue bounds depend on the mask: linearise again
  c->mg.linearized = false;
  return PF_OK;
}

pf_status pf_level_info(const pf_ctx* c, int level, int* p, int64_t* n_nodes) {
  if (!c) return fail(PF_EINVAL, "null context");
  if (!c->mg.linearized) return fail(PF_EINVAL, "call pf_linearize first");
  if (level < 0 || level >= c->mg.n_levels) return fail(PF_EINVAL, "level %d outside 0..%d", level, c->mg.n_levels - 1);
  if (p) *p = c->mg.lv[level].p;
  if (n_nodes) *n_nodes = c->mg.lv[level].n_nodes;
  return PF_OK;
}

pf_status pf_apply_jacobian_f32(pf_ctx* c, int level, const float* dz, float* y, void* stream) {
  pf_status st = need_lin(c, level);
  if (st) return st;
  if (!dz || !y) return fail(PF_EINVAL, "null vector");
  const size_t nb = 4 * c->mg.lv[level].n_nodes * sizeof(float);
  if (overlaps(dz, nb, y, nb)) return fail(PF_EINVAL, "y aliases dz");
  c->last_stream = (hipStream_t)stream;
  return level_op<E_STORE>(c, level, dz, store_epilogue(y), (hipStream_t)stream);
}

// FP64 Jacobian at the linearisation point from the stored FP64 record: the FP32
// level apply's kernels instantiated in FP64 on the fine level (u from the copy taken
// at pf_linearize).
pf_status pf_apply_jacobian_lin(pf_ctx* c, const double* dz, double* y, void* stream) {
  pf_status st = check_ctx(c);
  if (st) return st;
  if (!c->mg.linearized || !c->mg.lin64_valid)
    return fail(PF_EINVAL, "call pf_linearize with PF_OPT_STORE_LIN64 on first");
  if (!dz || !y) return fail(PF_EINVAL, "null vector");
  const size_t nb = 4 * c->n_nodes * sizeof(double);
  if (overlaps(dz, nb, y, nb)) return fail(PF_EINVAL, "y aliases dz");
  hipStream_t s = (hipStream_t)stream;
  c->last_stream = s;
  LinApplyArgs<double> a;
  a.m = mesh_dev(c);
  const MGLevel& F = c->mg.lv[0];
  a.fine = LevelDev{F.P, F.nx1, F.ny1, F.n_nodes};
  a.lev = a.fine;
  a.n_q = c->n_q;
  a.frame = nullptr;
  a.u = c->mg.u64;
  a.dz = dz;
  a.rec = RecordSoAT<double>{c->mg.rec64, c->mg.rec.flags};
  a.phase = c->qp_phase;
  a.mats = c->d_mats;
  a.nph = (int)c->phases.size();
  a.fr = frac_params<double>(c->fr);
  a.out = y;
  a.ebuf = nullptr;
  a.xmats = c->d_xmats64;
  a.n_extra = c->n_extra;
  a.qd = c->d_qd;
  switch (c->mesh.p) {
    case 2: return launch_lin_mfma<double, 3, 3, E_STORE>(c, a, store_epilogue(y), s);
    case 3: return launch_lin_mfma<double, 4, 4, E_STORE>(c, a, store_epilogue(y), s);
    case 4: return launch_lin_q4<double, 5, E_STORE>(c, a, store_epilogue(y), s);
    default: return fail(PF_EUNSUPPORTED, "the stored-linearisation apply is built for orders 2-4");
  }
}

pf_status pf_prolong(pf_ctx* c, int level, const float* xc, float* xf, void* stream) {
  pf_status st = need_lin(c, level);
  if (st) return st;
  if (level + 1 >= c->mg.n_levels) return fail(PF_EINVAL, "no coarser level below %d", level);
  if (!xc || !xf) return fail(PF_EINVAL, "null vector");
  c->last_stream = (hipStream_t)stream;
  return prolong(c, level, xc, xf, false, (hipStream_t)stream);
}

pf_status pf_restrict(pf_ctx* c, int level, const float* rf, float* rc, void* stream) {
  pf_status st = need_lin(c, level);
  if (st) return st;
  if (level + 1 >= c->mg.n_levels) return fail(PF_EINVAL, "no coarser level below %d", level);
  if (!rf || !rc) return fail(PF_EINVAL, "null vector");
  c->last_stream = (hipStream_t)stream;
  return restrict_(c, level, rf, rc, (hipStream_t)stream);
}

pf_status pf_level_diagonal(pf_ctx* c, int level, float* diag, void* stream) {
  pf_status st = need_lin(c, level);
  if (st) return st;
  if (!diag) return fail(PF_EINVAL, "null vector");
  const int64_t n = 4 * c->mg.lv[level].n_nodes;
  hipLaunchKernelGGL(k_vec_copy, dim3(vec_grid(n)), dim3(NT), 0, (hipStream_t)stream, c->mg.lv[level].diag, diag, n);
  HIPCHK(hipGetLastError());
  return PF_OK;
}

pf_status pf_pmg_vcycle(pf_ctx* c, const float* b, float* x, const pf_pmg_opts* o, void* stream) {
  pf_status st = need_lin(c, 0);
  if (st) return st;
  if (!b || !x) return fail(PF_EINVAL, "null vector");
  const size_t nb = 4 * c->n_nodes * sizeof(float);
  if (overlaps(b, nb, x, nb)) return fail(PF_EINVAL, "x aliases b");
  pf_pmg_opts opt{3, c->mg.lv[c->mg.n_levels - 1].p, 4, 0};
  if (o) {
    if (o->cheb_degree > 0) opt.cheb_degree = o->cheb_degree;
    if (o->coarse_p > 0) opt.coarse_p = o->coarse_p;
    if (o->coarse_sweeps > 0) opt.coarse_sweeps = o->coarse_sweeps;
  }
  if (opt.cheb_degree > 32 || opt.coarse_sweeps > 64) return fail(PF_EINVAL, "smoother degree too large");
  if (opt.coarse_p != c->mg.lv[c->mg.n_levels - 1].p)
    return fail(PF_EINVAL, "coarse_p=%d differs from the coarsest level order %d", opt.coarse_p,
                c->mg.lv[c->mg.n_levels - 1].p);
  c->last_stream = (hipStream_t)stream;
  hipStream_t s = (hipStream_t)stream;
  if (c->has_dir) {
    // work on the masked right-hand side (the V-cycle acts on the unconstrained subspace)
    MGLevel& L = c->mg.lv[0];
    const int64_t n = 4 * L.n_nodes;
    hipLaunchKernelGGL(k_vec_copy, dim3(vec_grid(n)), dim3(NT), 0, s, b, L.b, n);
    if ((st = mask_level(c, 0, L.b, s))) return st;
    return vcycle(c, 0, L.b, x, opt, s);
  }
  return vcycle(c, 0, b, x, opt, s);
}

}  // extern "C"
