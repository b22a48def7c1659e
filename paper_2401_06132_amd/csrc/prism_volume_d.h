// The prism volume group in double precision with flux anti-aliasing (affine
// and curved elements).  Included by kernels_prism.hip; the phases are those
// of prism_volume_mf.h.
//
// FP64 vector and matrix rates are equal and an element needs 24 KB of LDS at
// p = 4, so the vector form keeps the operator tables out of LDS: a
// triangle-plane product runs one (field, plane) per lane with the plane's
// values in registers and reads the operator row by row through the scalar
// cache, one row ahead (SRow), so that a multiply-add takes its operator
// entry from a scalar register and nothing from LDS.  The quadrature columns
// of the workgroup fill one wave; the two waves take half of the zeta levels
// each, re-reading the column from LDS per level (the 20 n values and the
// projection accumulators do not fit the registers together), and add their
// projections through LDS.  Measured (volume group, MI355X) against the form
// with the tables in LDS and two lanes per column (three one-wave workgroups
// per CU at p = 4): 14 858 prisms p = 4 917 -> 424 us, 32^3 cells p = 3
// 1112 -> 764 us, p = 2 488 -> 294 us, 40^3 p = 1 260 -> 187 us; curved, 24^3
// p = 3 506 -> 366 us, 20^3 p = 4 1202 -> 508 us.  Bound by latency: three
// two-wave workgroups per CU at p = 4 (49 KB of LDS each), a vector instruction
// every 15 cycles and SIMD, 57% of the waves' time waiting.
namespace fr {

// one row of K operator entries in scalar registers
template <int K>
struct SRow {
  double a[K];
  __device__ __forceinline__ void load(const double* __restrict__ p) {
#pragma unroll
    for (int k = 0; k < K; ++k) a[k] = p[k];
  }
};

template <int P, bool LIN>
struct PrismD {
  using C = PrismVol<P, LIN>;
  static constexpr int n = P + 1, m = P + 3, NTN = C::NTN, NTQ = C::NTQ, NU = C::NU, NFP = C::NFP, NVF = C::NVF;
  static constexpr int EB = P == 1 ? 8 : (P == 2 ? 5 : (P == 3 ? 3 : 2)), W = 2, NT = 64 * W;
  static_assert(EB * NTQ <= 64, "the quadrature columns fill one wave");
  static constexpr int TQS = NTQ | 1;  // odd row stride
  static constexpr int SZ_T1 = 20 * n * TQS, SZ_Z = 3 * NVF * C::ZVS;
  static constexpr int mx(int a, int b) { return a > b ? a : b; }
  static constexpr int PE = mx(C::SZ_A + C::SZ_JE, mx(SZ_T1, SZ_Z));
  static constexpr int L0 = (m + 1) / 2;  // levels of the first wave
  // the xi (eta) derivative takes no lift from edge 0 (2), whose normal has no
  // such component (p = 4: 455 -> 424 us, the table nearer to the scalar cache's size)
  static constexpr int KG = NTN + 2 * n;
  static constexpr int RP = (NTN + 1) / 2;  // projection rows per wave
};

// device table (doubles): rows of the edge interpolation, of the gradient
// [t][xi, eta][KG], of T_q, and the projection [wave][t_q][d][RP]; each with
// a row of padding behind it (the loops read one row ahead)
template <int P>
struct PrismDTab {
  using M = PrismD<P, true>;
  static constexpr int edge = 0, grad = edge + (3 * M::n + 1) * M::NTN, tq = grad + (2 * M::NTN + 2) * M::KG,
                       proj = tq + (M::NTQ + 1) * M::NTN, PB = (M::NTQ + 1) * 3 * M::RP, size = proj + 2 * PB;
};

template <int P>
static void prism_d_pack(const RefElem& r, double* o) {
  using B = PrismDTab<P>;
  using M = typename B::M;
  constexpr int n = M::n, NTN = M::NTN, NTQ = M::NTQ, KG = M::KG;
  const Tri& T = r.tri;
  for (int i = 0; i < B::size; ++i) o[i] = 0.0;
  for (int i = 0; i < 3 * n * NTN; ++i) o[B::edge + i] = T.Tedge[i];
  const double h = 0.70710678118654752440;
  for (int t = 0; t < NTN; ++t)
    for (int d = 0; d < 2; ++d) {
      double* row = o + B::grad + (2 * t + d) * KG;
      for (int k = 0; k < NTN; ++k) row[k] = d ? T.Deta[t * NTN + k] : T.Dxi[t * NTN + k];
      for (int k = 0; k < 2; ++k) {
        const int e = d ? k : 1 + k;
        const double nrm = e == 1 ? h : -1.0;
        for (int i = 0; i < n; ++i) row[NTN + k * n + i] = nrm * T.LiftEdge[(e * NTN + t) * n + i];
      }
    }
  for (int i = 0; i < NTQ * NTN; ++i) o[B::tq + i] = T.Tq[i];
  for (int g = 0; g < 2; ++g)
    for (int q = 0; q < NTQ; ++q)
      for (int d = 0; d < 3; ++d)
        for (int i = 0; i < M::RP && g * M::RP + i < NTN; ++i)
          o[B::proj + g * B::PB + (q * 3 + d) * M::RP + i] =
              (d == 0 ? T.APxi : (d == 1 ? T.APeta : T.PT))[(g * M::RP + i) * NTQ + q];
}

template <int P, bool BT, bool WARP>
__global__ void __launch_bounds__((PrismD<P, !WARP>::NT)) __attribute__((amdgpu_waves_per_eu(2)))
    prism_volume_d(const Seg one, const BlkRef* __restrict__ bt, const Seg* __restrict__ segs, const bool from_ust,
                   const PrismOps<P, double> op, const PrismTri<P, double>* __restrict__ tri,
                   const double* __restrict__ tab, const Gas<double> g, const double eref, const double rho0) {
  typedef double R;
  constexpr bool LIN = !WARP;
  using M = PrismD<P, LIN>;
  using C = typename M::C;
  using F = PrismCfg<P>;  // face array layout
  using B = PrismDTab<P>;
  constexpr int n = C::n, m = C::m, NTN = C::NTN, NTQ = C::NTQ, NU = C::NU, NFP = C::NFP;
  constexpr int NVF = C::NVF, V0 = C::V0, EB = M::EB, NT_ = M::NT, PE = M::PE, TQS = M::TQS;
  __shared__ R smem[EB * PE];
  __shared__ R sMet[EB][10];
  __shared__ FaceRec sFR[EB * 5];
  __shared__ R sFG[EB * 5][4];
  __shared__ uint8_t sPerm[MAX_PERMS * NFP];
  __shared__ R sV[WARP ? EB : 1][18];  // curved: element vertices
  int e0;
  const Seg sg = seg_of<BT>(one, bt, segs, EB, e0);
  const double* __restrict__ U = from_ust ? sg.ust : sg.U;
  const R* __restrict__ Uf = (const R*)sg.Uf;
  R* __restrict__ Vf = (R*)sg.Vf;
  R* __restrict__ Rp = (R*)sg.Rp;
  const FaceRec* __restrict__ faces = sg.faces;
  const R* __restrict__ fgeo = (const R*)sg.fgeo;
  const uint8_t* __restrict__ perms = sg.perms;
  const R* __restrict__ met = (const R*)sg.met;
  const int E = sg.E, slot_base = sg.slot_base, tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#define XS(le) (smem + (le)*PE)           /* [20][NU]                            */
#define JS(le) (smem + (le)*PE + C::SZ_A) /* [5][5][NFP] neighbour u^f; later EF */
#define TS(le) (smem + (le)*PE)           /* [20][n][TQS]                        */
#define ZS(le) (smem + (le)*PE)           /* [3][NVF][ZVS]                       */

  // phase 0: as in prism_volume_mf
  for (int it = tid; it < EB * 5; it += NT_) {
    const int slot = slot_base + (e0 + it / 5 < E ? e0 * 5 + it : 0);
    sFR[it] = faces[slot];
#pragma unroll
    for (int k = 0; k < 4; ++k) sFG[it][k] = fgeo[4 * slot + k];
  }
  for (int it = tid; it < sg.nperm * NFP; it += NT_) sPerm[it] = perms[it];
  if constexpr (WARP) {
    const R* __restrict__ vx = (const R*)sg.verts;
    for (int it = tid; it < EB * 18; it += NT_) {
      const int le = it / 18;
      sV[le][it - le * 18] = vx[e0 + le < E ? (size_t)e0 * 18 + it : 0];
    }
  }
  for (int it = tid; it < EB * 10; it += NT_) {
    const int le = it / 10, k = it - le * 10, e = e0 + le;
    sMet[le][k] = met[e < E ? (size_t)e * 10 + k : 0];
  }
  const int nv = E - e0 < EB ? E - e0 : EB;  // valid elements of the batch
  constexpr int NR = (5 * NU + NT_ - 1) / NT_;
  double xs[EB][NR];
#pragma unroll
  for (int le = 0; le < EB; ++le)
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const int r = tid + k * NT_;
      xs[le][k] = U[le < nv && r < 5 * NU ? (size_t)(e0 + le) * 5 * NU + r : 0];
    }
  lds_barrier();
  constexpr int NG = (EB * F::PPE + NT_ - 1) / NT_;
  R gv[NG][5];
  auto face_point = [](int q, int& f, int& r) {
    f = q < 2 * NTN ? q / NTN : 2 + (q - 2 * NTN) / NFP;
    r = q - F::foff(f);
  };
#pragma unroll
  for (int k = 0; k < NG; ++k) {
    const int it = tid + k * NT_;
    const int itc = it < EB * F::PPE ? it : 0;
    const int le = itc / F::PPE;
    int f, r;
    face_point(itc - le * F::PPE, f, r);
    const FaceRec fr = sFR[le * 5 + f];
    const R* __restrict__ src = Uf + (size_t)fr.npo * 5 + sPerm[(fr.info >> 1) * NFP + r];
    const int fs = F::fsz(f);
#pragma unroll
    for (int v = 0; v < 5; ++v) gv[k][v] = src[v * fs];
  }
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    const int r = tid + k * NT_;
    if (r < 5 * NU) {
      const double sh = r < NU ? rho0 : (r >= 4 * NU ? eref : 0.0);
#pragma unroll
      for (int le = 0; le < EB; ++le) XS(le)[r] = xs[le][k] - sh;
    }
  }
#pragma unroll
  for (int k = 0; k < NG; ++k) {
    const int it = tid + k * NT_;
    if (it < EB * F::PPE) {
      const int le = it / F::PPE;
      int f, r;
      face_point(it - le * F::PPE, f, r);
      R* dst = JS(le) + f * 5 * NFP + r;
#pragma unroll
      for (int v = 0; v < 5; ++v) dst[v * NFP] = gv[k][v];
    }
  }
  lds_barrier();

  // phase 1: zeta lines: jumps C - u^f at the two triangle faces (eq.
  // FR-conu) and the corrected zeta derivative (eq. FR-qfinal)
  for (int it = tid; it < EB * 5 * NTN; it += NT_) {
    const int le = it / (5 * NTN), r0 = it - le * (5 * NTN), v = r0 / NTN, t = r0 - v * NTN;
    R* X = XS(le);
    R x[n];
    R xm = R(0), xp = R(0);
#pragma unroll
    for (int k = 0; k < n; ++k) {
      x[k] = X[v * NU + t + NTN * k];
      xm += op.lb[k] * x[k];
      xp += op.rb[k] * x[k];
    }
    const R wm = (sFR[le * 5].info & 1) ? R(0.5) + g.beta : R(0.5) - g.beta;
    const R wp = (sFR[le * 5 + 1].info & 1) ? R(0.5) + g.beta : R(0.5) - g.beta;
    const R jm = wm * (JS(le)[(0 * 5 + v) * NFP + t] - xm), jp = wp * (JS(le)[(1 * 5 + v) * NFP + t] - xp);
#pragma unroll
    for (int k = 0; k < n; ++k) {
      R s = op.liftR[k] * jp - op.liftL[k] * jm;
#pragma unroll
      for (int c = 0; c < n; ++c) s += op.D[k][c] * x[c];
      X[(15 + v) * NU + t + NTN * k] = s;
    }
  }
  lds_barrier();

  // phase 2: triangle planes: values at the edge points, jumps in place
  // (each lane its own plane's), the corrected (xi, eta) derivatives (eq.
  // FR-qfinal) and, with one metric per element, q = J^-T q~ (eq. FR-gradcoru)
  {
    constexpr int NI = EB * 5 * n;
    for (int b = wave * 64; b < NI; b += NT_) {
      const int it = b + lane;
      const bool ok = it < NI;
      const int itc = ok ? it : 0, le = itc / (5 * n), r0 = itc - le * (5 * n), v = r0 / n, k = r0 - v * n;
      R* X = XS(le) + NTN * k;
      R* J = JS(le) + (10 + v) * NFP + n * k;
      R x[NTN];
#pragma unroll
      for (int t = 0; t < NTN; ++t) x[t] = X[v * NU + t];
      {
        SRow<NTN> row;
        row.load(tab + B::edge);
#pragma unroll 1
        for (int ed = 0; ed < 3; ++ed) {
          const R w = (sFR[le * 5 + 2 + ed].info & 1) ? R(0.5) + g.beta : R(0.5) - g.beta;
          R* Je = J + ed * 5 * NFP;
#pragma unroll 1
          for (int i = 0; i < n; ++i) {
            SRow<NTN> nxt;
            nxt.load(tab + B::edge + (ed * n + i + 1) * NTN);
            R s = R(0);
#pragma unroll
            for (int t = 0; t < NTN; ++t) s += row.a[t] * x[t];
            const R j = w * (Je[i] - s);
            if (ok) Je[i] = j;
            row = nxt;
          }
        }
      }
      R jq[3 * n];
#pragma unroll
      for (int q = 0; q < 3 * n; ++q) jq[q] = J[(q / n) * 5 * NFP + q % n];
      const R* Mt = sMet[le];  // Mt[3 d + c] = (J^-1)_{dc}
#pragma unroll 1
      for (int t = 0; t < NTN; ++t) {
        const double* __restrict__ gr = tab + B::grad + 2 * t * M::KG;
        R g0 = R(0), g1 = R(0);
#pragma unroll
        for (int c = 0; c < NTN; ++c) g0 += gr[c] * x[c];
#pragma unroll
        for (int q = 0; q < 2 * n; ++q) g0 += gr[NTN + q] * jq[n + q];
#pragma unroll
        for (int c = 0; c < NTN; ++c) g1 += gr[M::KG + c] * x[c];
#pragma unroll
        for (int q = 0; q < 2 * n; ++q) g1 += gr[M::KG + NTN + q] * jq[q];
        if constexpr (WARP) {
          if (ok) {
            X[(5 + v) * NU + t] = g0;
            X[(10 + v) * NU + t] = g1;
          }
        } else {
          const R g2 = X[(15 + v) * NU + t];
          if (ok) {
#pragma unroll
            for (int c = 0; c < 3; ++c) X[(5 + c * 5 + v) * NU + t] = Mt[c] * g0 + Mt[3 + c] * g1 + Mt[6 + c] * g2;
          }
        }
      }
    }
  }
  lds_barrier();
  if constexpr (WARP) {
    for (int it = tid; it < EB * NU; it += NT_) {
      const int le = it / NU;
      wedge_gradient<P, R>(op, tri, &sV[le][0], it - le * NU, XS(le));
    }
    lds_barrier();
  }

  // phase 3: triangle planes of the 20 fields, in registers until phase 5
  // (NIT planes a lane share each operator row); their values at the edge
  // points (gradcoru_fpts) into EF, over the neighbour values
  constexpr int NP = EB * 20 * n, NIT = (NP + NT_ - 1) / NT_;
  R xv[NIT][NTN];
  int pof[NIT];  // plane (le, fld, k): le * PE + the plane's offset in a [20][n] array of stride 1
#pragma unroll
  for (int j = 0; j < NIT; ++j) {
    const int it = tid + j * NT_, itc = it < NP ? it : 0;
    const int le = itc / (20 * n), fk = itc - le * (20 * n), fld = fk / n, k = fk - fld * n;
    const R* x = XS(le) + fld * NU + NTN * k;
    pof[j] = le * PE + C::SZ_A + fld * C::EFS + n * k;
#pragma unroll
    for (int t = 0; t < NTN; ++t) xv[j][t] = x[t];
  }
  {
    SRow<NTN> row;
    row.load(tab + B::edge);
#pragma unroll 1
    for (int ed = 0; ed < 3; ++ed)
#pragma unroll 1
      for (int i = 0; i < n; ++i) {
        SRow<NTN> nxt;
        nxt.load(tab + B::edge + (ed * n + i + 1) * NTN);
#pragma unroll
        for (int j = 0; j < NIT; ++j) {
          R s = R(0);
#pragma unroll
          for (int t = 0; t < NTN; ++t) s += row.a[t] * xv[j][t];
          if (tid + j * NT_ < NP) smem[pof[j] + ed * NFP + i] = s;
        }
        row = nxt;
      }
  }
  lds_barrier();

  // phase 4: normal viscous flux at the own flux points: quadrilateral-face
  // points from EF, triangle nodes (both faces of a line) from the state;
  // the two kinds start from opposite ends, so that the waves share them
  for (int it = tid; it < EB * 3 * NFP; it += NT_) {
    const int le = it / (3 * NFP), r1 = it - le * (3 * NFP), e = e0 + le;
    if (e >= E) continue;
    const int ed = r1 / NFP, r2 = r1 - ed * NFP;
    const int lf = le * 5 + 2 + ed, po = sg.po_base + e * F::PPE + F::foff(2 + ed);
    R nn[3];
    if constexpr (WARP) {
      wedge_quad_normal(op, &sV[le][0], ed, r2, nn);
    } else {
      const R sgn = (sFR[lf].info & 1) ? R(1) : R(-1);
#pragma unroll
      for (int c = 0; c < 3; ++c) nn[c] = sgn * sFG[lf][c];
    }
    const R* EF = JS(le) + r1;
    R u[5], q[3][5], V[4];
#pragma unroll
    for (int fld = 0; fld < 20; ++fld) {
      const R s = EF[fld * C::EFS];
      if (fld < 5)
        u[fld] = s;
      else
        q[(fld - 5) / 5][(fld - 5) % 5] = s;
    }
    normal_viscous(u, q, nn, g, V);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) Vf[(size_t)po * 4 + kk * NFP + r2] = V[kk];
  }
  for (int it = NT_ - 1 - tid; it < EB * 2 * NTN; it += NT_) {
    const int le = it / (2 * NTN), r0 = it - le * (2 * NTN), side = r0 / NTN, t = r0 - side * NTN, e = e0 + le;
    if (e >= E) continue;
    const R* X = XS(le) + t;
    const int lf = le * 5 + side, po = sg.po_base + e * F::PPE + side * NTN;
    R u[5], q[3][5], V[4];
#pragma unroll
    for (int fld = 0; fld < 20; ++fld) {
      R s = R(0);
#pragma unroll
      for (int k = 0; k < n; ++k) s += (side ? op.rb[k] : op.lb[k]) * X[fld * NU + NTN * k];
      if (fld < 5)
        u[fld] = s;
      else
        q[(fld - 5) / 5][(fld - 5) % 5] = s;
      if (fld % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    R nn[3];
    if constexpr (WARP) {
      wedge_tri_normal(tri, &sV[le][0], t, side, nn);
    } else {
      const R sgn = (sFR[lf].info & 1) ? R(1) : R(-1);
#pragma unroll
      for (int c = 0; c < 3; ++c) nn[c] = sgn * sFG[lf][c];
    }
    normal_viscous(u, q, nn, g, V);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) Vf[(size_t)po * 4 + kk * NTN + t] = V[kk];
  }
  lds_barrier();

  // phase 5: triangle-plane interpolation of the 20 fields to the triangle
  // quadrature points (first factor of M7 / M10), over the state
#pragma unroll
  for (int j = 0; j < NIT; ++j) {
    const int it = tid + j * NT_, itc = it < NP ? it : 0, le = itc / (20 * n);
    pof[j] = le * PE + (itc - le * (20 * n)) * TQS;
  }
  {
    SRow<NTN> row;
    row.load(tab + B::tq);
#pragma unroll 1
    for (int q = 0; q < NTQ; ++q) {
      SRow<NTN> nxt;
      nxt.load(tab + B::tq + (q + 1) * NTN);
#pragma unroll
      for (int j = 0; j < NIT; ++j) {
        R s = R(0);
#pragma unroll
        for (int t = 0; t < NTN; ++t) s += row.a[t] * xv[j][t];
        if (tid + j * NT_ < NP) smem[pof[j] + q] = s;
      }
      row = nxt;
    }
  }
  lds_barrier();

  // phase 6: one quadrature column per lane, this wave's zeta levels: zeta
  // interpolation (uqpts, gradcoru_qpts), flux (tdisf) and the zeta part of
  // the projection-divergence
  const bool col = lane < EB * NTQ;
  const int cc = col ? lane : 0, cle = cc / NTQ, ctq = cc - cle * NTQ;
  R acc[3][NVF][n];
#pragma unroll
  for (int d = 0; d < 3; ++d)
#pragma unroll
    for (int v = 0; v < NVF; ++v)
#pragma unroll
      for (int k = 0; k < n; ++k) acc[d][v][k] = R(0);
  {
    const R* T = TS(cle) + ctq;
    R S[3][3];
    const R dj = sMet[cle][9];
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int c = 0; c < 3; ++c) S[d][c] = dj * sMet[cle][3 * d + c];
    R cqx = R(0), cqy = R(0);
    if constexpr (WARP) {
      cqx = tri->qp[ctq][0];
      cqy = tri->qp[ctq][1];
    }
    const int l1 = wave ? m : M::L0;
#pragma unroll 1
    for (int kq = wave ? M::L0 : 0; kq < l1; ++kq) {
      R u[5], q[3][5], f[3][5];
#pragma unroll
      for (int fld = 0; fld < 20; ++fld) {
        R s = R(0);
#pragma unroll
        for (int k = 0; k < n; ++k) s += op.I[kq][k] * T[(fld * n + k) * TQS];
        if (fld < 5)
          u[fld] = s;
        else
          q[(fld - 5) / 5][(fld - 5) % 5] = s;
        // keep the scheduler from hoisting every field's LDS reads
        if (fld % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
      point_flux(u, q, g, f);
      if constexpr (WARP) {
        R det;
        wedge_metric(&sV[cle][0], cqx, cqy, op.xq[kq], S, det);  // det J J^-1 here
      }
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int v = V0; v < 5; ++v) {
          const R ft = S[d][0] * f[0][v] + S[d][1] * f[1][v] + S[d][2] * f[2][v];
#pragma unroll
          for (int k = 0; k < n; ++k) acc[d][v - V0][k] += (d == 2 ? op.AP[k][kq] : op.Pj[k][kq]) * ft;
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  lds_barrier();  // every column has read T1; Z may now overwrite it
  R* Zc = ZS(cle) + ctq * n;
  if (wave == 1 && col) {
#pragma unroll
    for (int i = 0; i < 3 * NVF; ++i)
#pragma unroll
      for (int k = 0; k < n; ++k) Zc[i * C::ZVS + k] = acc[i / NVF][i % NVF][k];
  }
  lds_barrier();
  if (wave == 0 && col) {
#pragma unroll
    for (int i = 0; i < 3 * NVF; ++i)
#pragma unroll
      for (int k = 0; k < n; ++k) Zc[i * C::ZVS + k] += acc[i / NVF][i % NVF][k];
  }
  lds_barrier();

  // phase 7: triangle-plane projection-divergence of one (variable, plane)
  // per lane, half of the rows per wave; LIN: the energy residual takes
  // kap L(rho v) (row 0, from the disu kernel)
  constexpr int NJ = EB * NVF * n, RP = M::RP;
  for (int b = 0; b < NJ; b += 64) {
    const int it = b + lane, itc = it < NJ ? it : 0;
    const int le = itc / (NVF * n), r0 = itc - le * (NVF * n), vv = r0 / n, k = r0 - vv * n, e = e0 + le, v = vv + V0;
    const bool ok = it < NJ && e < E;
    R* out = Rp + (size_t)(ok ? e : e0) * 5 * NU + NTN * k;
    const int t0 = wave * RP;
    R s[RP];
#pragma unroll
    for (int i = 0; i < RP; ++i) s[i] = LIN && v == 4 ? g.kap * out[t0 + i < NTN ? t0 + i : 0] : R(0);
    const R* Z = ZS(le) + vv * C::ZVS + k;
    const double* __restrict__ pt = tab + B::proj + wave * B::PB;
    SRow<3 * RP> row;
    row.load(pt);
#pragma unroll 1
    for (int tq = 0; tq < NTQ; ++tq) {
      SRow<3 * RP> nxt;
      nxt.load(pt + (tq + 1) * 3 * RP);
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const R z = Z[d * NVF * C::ZVS + tq * n];
#pragma unroll
        for (int i = 0; i < RP; ++i) s[i] += row.a[d * RP + i] * z;
      }
      row = nxt;
    }
    if (ok) {
#pragma unroll
      for (int i = 0; i < RP; ++i)
        if (t0 + i < NTN) out[v * NU + t0 + i] = s[i];
    }
  }
#undef XS
#undef JS
#undef TS
#undef ZS
}

}  // namespace fr
