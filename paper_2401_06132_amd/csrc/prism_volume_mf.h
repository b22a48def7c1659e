// The prism volume group in single precision with flux anti-aliasing
// (affine and curved elements): the triangle-plane operators and the zeta
// sweeps on the matrix cores, one column per lane (mf4.h).  Included by
// kernels_prism.hip, which defines the operator structures.
//
// Phases (barriers between them):
//   0  state, metrics and neighbour face states to LDS
//   1  zeta lines: corrected zeta derivative (jumps of the two triangles)
//   2  triangle planes (variable, plane): face values at the edge points,
//      jumps, corrected (xi, eta) derivatives, J^-T        [matrix cores]
//   3  triangle planes (field, plane): the 20 fields at the edge points
//      [matrix cores]; normal viscous flux at the triangle nodes; the edge
//      fields EF to LDS over the state
//   4  normal viscous flux at the quadrilateral-face points
//   5  triangle planes: T_q to the triangle quadrature points, T1 over the
//      state and gradients                                 [matrix cores]
//   6  quadrature columns, two half-wave lanes per column (lane and
//      lane + 32, each a contiguous range of zeta levels): zeta
//      interpolation, flux, zeta projection                [matrix cores]
//   7  triangle planes (variable, plane): projection-divergence [matrix cores]
// The operators come from L2 as packed chunks, a register per 16 chunks, so
// no table sits in LDS, and every LDS array lies over the dead one before it:
// 26 KB per four elements at p = 3 (six two-wave workgroups per CU) and 52 KB
// per five at p = 4 (three four-wave ones), three waves per SIMD at both; at
// p = 4 that costs 8 to 10 spilled registers (curved 17), 42% of what the kernel
// writes to memory, and is faster all the same.  Bound by instruction issue:
// vector and matrix instructions together busy 74% (p = 3) and 66% (p = 4) of
// the time.  Measured (volume group, MI355X): 48^3 cells p = 3 1474 -> 750 us,
// 262 144 prisms p = 4 5586 -> 1795 us, 32 768 curved prisms p = 3 251 -> 141
// us, against the vector kernel with its operator tables in LDS (8 and 7 waves
// per CU); with EF and the face records in LDS of
// their own (five and two workgroups per CU) 817, 2133 and 155 us.
namespace fr {

template <int P, bool LIN>
struct PrismMf {
  using C = PrismVol<P, LIN>;
  static constexpr int n = P + 1, m = P + 3, NTN = C::NTN, NTQ = C::NTQ, NU = C::NU, NFP = C::NFP, NVF = C::NVF;
  // launch shape: 32 quadrature columns (two lanes each) per wave
  static constexpr int EB = P == 1 ? 8 : (P == 2 ? 7 : (P == 3 ? 4 : 5));
  static constexpr int W = P == 1 ? 1 : (P == 4 ? 4 : 2), NT = 64 * W;
  static_assert(EB * NTQ <= 32 * W, "two lanes per quadrature column");
  // LDS per element, every array from offset 0 over the dead one before it:
  // state, gradients and neighbour states with the face records behind them
  // (FRO) | the fields at the edge points EF | T1 | Z.  T1 rows of TQS: on
  // 16-byte boundaries (p <= 3: four outputs of a lane in one store, strides
  // that spread eight lanes' stores over all banks), 8-byte ones at p = 4,
  // where the longer rows would cost a workgroup per CU
  static constexpr int TQS = P == 1 ? 4 : (P == 2 ? 12 : (P == 3 ? 20 : 26));
  static constexpr int SZ_T1 = 20 * n * TQS;
  // Z variables ZVS apart, so that the lanes of a plane sweep (4 variables, n
  // planes) read different banks
  static constexpr int ZVS = P == 4 ? NTQ * n + 8 : C::ZVS, SZ_Z = 3 * NVF * ZVS;
  static constexpr int mx(int a, int b) { return a > b ? a : b; }
  static constexpr int FRO = (mx(C::SZ_A + C::SZ_J, C::SZ_EF) + 3) / 4 * 4;  // records, geometry, permutations
  static constexpr int SZ_F = FRO + 40 + (MAX_PERMS * NFP + 3) / 4;
  static constexpr int PE0 = (mx(SZ_F, mx(SZ_T1, SZ_Z)) + 3) / 4 * 4;
  // p = 3: elements 16 banks apart (a wave's 32 columns lie in two elements)
  static constexpr int PE = P == 3 ? PE0 + 16 : PE0;
  // zeta levels: the lower half wave takes the first L0, the upper the rest
  static constexpr int L0 = (m + 1) / 2;
  static_assert(L0 <= 4 && m - L0 >= 1, "one row tile of levels");
  // row tiles: edge points, gradient, triangle quadrature, projection
  static constexpr int TE = (3 * n + 3) / 4, TG = (2 * NTN + 3) / 4, TT = (NTQ + 3) / 4, TP = (NTN + 3) / 4;
  static constexpr int KG = NTN + 3 * n, KP = 3 * NTQ;
  // projection: IW waves of (element, variable, plane) columns; the waves
  // left over take a share of the row tiles
  static constexpr int IW = (EB * NVF * n + 63) / 64, G = W / IW > 1 ? W / IW : 1, TPG = (TP + G - 1) / G;
};

// device table of the packed operators (floats)
template <int P>
struct PrismMfTab {
  using M = PrismMf<P, true>;
  using MC = PrismMf<P, false>;  // curved: another split of the projection's row tiles
  static constexpr int edge = 0, grad = edge + Mf4Op<M::TE, M::NTN>::FLOATS,
                       tq = grad + Mf4Op<M::TG, M::KG>::FLOATS, zint = tq + Mf4Op<M::TT, M::NTN>::FLOATS,
                       zproj = zint + 64, proj = zproj + 64,
                       projc = proj + M::G * Mf4Op<M::TPG, M::KP>::FLOATS,
                       size = projc + MC::G * Mf4Op<MC::TPG, MC::KP>::FLOATS;
  static_assert(M::n <= 8, "zeta interpolation columns fit a half register");
};

template <int P>
static void prism_mf_pack(const RefElem& r, float* o) {
  using B = PrismMfTab<P>;
  using M = PrismMf<P, true>;
  using MC = PrismMf<P, false>;
  constexpr int n = M::n, m = M::m, NTN = M::NTN, NTQ = M::NTQ, L0 = M::L0;
  const Tri& T = r.tri;
  const Line1D& L = r.line;
  mf4_pack<M::TE, NTN>(o + B::edge, 3 * n, [&](int q, int t) { return T.Tedge[q * NTN + t]; });
  mf4_pack<M::TG, M::KG>(o + B::grad, 2 * NTN, [&](int row, int k) {
    const int d = row / NTN, t = row - d * NTN;
    if (k < NTN) return d ? T.Deta[t * NTN + k] : T.Dxi[t * NTN + k];
    const int e = (k - NTN) / n, i = (k - NTN) - e * n;
    const double h = 0.70710678118654752440, nx = e == 0 ? 0.0 : (e == 1 ? h : -1.0), ny = e == 0 ? -1.0 : (e == 1 ? h : 0.0);
    return (d ? ny : nx) * T.LiftEdge[(e * NTN + t) * n + i];
  });
  mf4_pack<M::TT, NTN>(o + B::tq, NTQ, [&](int q, int t) { return T.Tq[q * NTN + t]; });
  // zeta operators: block 8 h + k of the register, h the half wave; a level
  // past a half's range repeats its last level with zero projection weight
  for (int h = 0; h < 2; ++h)
    for (int b = 0; b < 8; ++b)
      for (int q = 0; q < 4; ++q) {
        float vi = 0.0f, vp = 0.0f;
        const int cnt = h ? m - L0 : L0;
        const int lev = h * L0 + (q < cnt ? q : cnt - 1);
        if (b < n) vi = float(L.I[lev * n + b]);
        // projection: column = level b % 4, row q; P then AP
        const int lb = b % 4;
        if (lb < cnt && q < n) vp = float((b < 4 ? L.P : L.AP)[q * m + h * L0 + lb]);
        o[B::zint + (8 * h + b) * 4 + q] = vi;
        o[B::zproj + (8 * h + b) * 4 + q] = vp;
      }
  auto proj = [&](int t, int k) {
    const int tq = k / 3, d = k - 3 * tq;
    return t >= NTN ? 0.0 : (d == 0 ? T.APxi : (d == 1 ? T.APeta : T.PT))[t * NTQ + tq];
  };
  for (int g = 0; g < M::G; ++g)
    mf4_pack<M::TPG, M::KP>(o + B::proj + g * Mf4Op<M::TPG, M::KP>::FLOATS, 4 * M::TPG,
                            [&](int q, int k) { return proj(g * 4 * M::TPG + q, k); });
  for (int g = 0; g < MC::G; ++g)
    mf4_pack<MC::TPG, MC::KP>(o + B::projc + g * Mf4Op<MC::TPG, MC::KP>::FLOATS, 4 * MC::TPG,
                              [&](int q, int k) { return proj(g * 4 * MC::TPG + q, k); });
}

template <int P, bool BT, bool WARP>
__global__ void __launch_bounds__((PrismMf<P, !WARP>::NT)) __attribute__((amdgpu_waves_per_eu(3)))
    prism_volume_mf(const Seg one, const BlkRef* __restrict__ bt, const Seg* __restrict__ segs, const bool from_ust,
                    const PrismOps<P, float> op, const PrismTri<P, float>* __restrict__ tri,
                    const float* __restrict__ tab, const Gas<float> g, const double eref, const double rho0) {
  typedef float R;
  constexpr bool LIN = !WARP;
  using M = PrismMf<P, LIN>;
  using C = typename M::C;
  using F = PrismCfg<P>;  // face array layout
  using B = PrismMfTab<P>;
  constexpr int n = C::n, m = C::m, NTN = C::NTN, NTQ = C::NTQ, NU = C::NU, NFP = C::NFP;
  constexpr int NVF = C::NVF, V0 = C::V0, EB = M::EB, W = M::W, NT_ = M::NT, PE = M::PE;
  __shared__ __attribute__((aligned(16))) R smem[EB * PE];
  __shared__ R sMet[EB][10];
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
#define JS(le) (smem + (le)*PE + C::SZ_A) /* [5][5][NFP] neighbour u^f           */
#define ES(le) (smem + (le)*PE)           /* [20][EFS] fields at the edge points */
#define TS(le) (smem + (le)*PE)           /* [20][n][TQS]                        */
#define ZS(le) (smem + (le)*PE)           /* [3][NVF][ZVS]                       */
#define FR(le) (reinterpret_cast<FaceRec*>(smem + (le)*PE + M::FRO))       /* [5]    */
#define FG(le) (reinterpret_cast<R(*)[4]>(smem + (le)*PE + M::FRO + 20))   /* [5][4] */
  uint8_t* sPerm = reinterpret_cast<uint8_t*>(smem + M::FRO + 40);         // behind element 0's records

  // phase 0: face records, face geometry and permutations first, so the
  // neighbour gather is one global load per value; out-of-range items load
  // from a valid address and never reach an output
  for (int it = tid; it < EB * 5; it += NT_) {
    const int slot = slot_base + (e0 + it / 5 < E ? e0 * 5 + it : 0);
    FR(it / 5)[it % 5] = faces[slot];
#pragma unroll
    for (int k = 0; k < 4; ++k) FG(it / 5)[it % 5][k] = fgeo[4 * slot + k];
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
  R gv[NG][5], gb[NG][5];
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
    const FaceRec fr = FR(le)[f];
    const R* __restrict__ src = Uf + (size_t)fr.npo * 5 + sPerm[(fr.info >> 1) * NFP + r];
    const int fs = F::fsz(f);
#pragma unroll
    for (int v = 0; v < 5; ++v) gv[k][v] = src[v * fs];
#pragma unroll
    for (int v = 0; v < 5; ++v) gb[k][v] = sg.Ub[(size_t)fr.nbr * 5 + v];  // the face base
  }
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    const int r = tid + k * NT_;
    if (r < 5 * NU) {
      const double sh = r < NU ? rho0 : (r >= 4 * NU ? eref : 0.0);
#pragma unroll
      for (int le = 0; le < EB; ++le) XS(le)[r] = R(xs[le][k] - sh);
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
      for (int v = 0; v < 5; ++v) dst[v * NFP] = gv[k][v] + gb[k][v];
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
    const R wm = (FR(le)[0].info & 1) ? R(0.5) + g.beta : R(0.5) - g.beta;
    const R wp = (FR(le)[1].info & 1) ? R(0.5) + g.beta : R(0.5) - g.beta;
    const R jm = wm * (JS(le)[(0 * 5 + v) * NFP + t] - xm), jp = wp * (JS(le)[(1 * 5 + v) * NFP + t] - xp);
#pragma unroll
    for (int k = 0; k < n; ++k) {
      R s = op.liftR[k] * jp - op.liftL[k] * jm;
#pragma unroll
      for (int c = 0; c < n; ++c) s += op.D[k][c] * x[c];
      X[(15 + v) * NU + t + NTN * k] = s;
    }
  }
  Mf4Op<M::TE, NTN> oe;
  oe.load(tab + B::edge, lane);
  {
    Mf4Op<M::TG, M::KG> og;
    og.load(tab + B::grad, lane);
    lds_barrier();

    // phase 2: triangle planes: values at the edge points, jumps (eq.
    // FR-conu), the corrected (xi, eta) derivatives (eq. FR-qfinal) and, with
    // one metric per element, q = J^-T q~ (eq. FR-gradcoru)
    constexpr int NI = EB * 5 * n;
    for (int b = wave * 64; b < NI; b += NT_) {
      const int it = b + lane, itc = it < NI ? it : 0;
      const int le = itc / (5 * n), r0 = itc - le * (5 * n), v = r0 / n, k = r0 - v * n;
      R* X = XS(le) + NTN * k;
      const R* J = JS(le) + (10 + v) * NFP + n * k;
      R x[NTN], jq[3 * n];
#pragma unroll
      for (int t = 0; t < NTN; ++t) x[t] = X[v * NU + t];
#pragma unroll
      for (int q = 0; q < 3 * n; ++q) jq[q] = J[(q / n) * 5 * NFP + q % n];
      mf4v fe[M::TE];
#pragma unroll
      for (int t = 0; t < M::TE; ++t) fe[t] = mf4v{0, 0, 0, 0};
#pragma unroll
      for (int t = 0; t < NTN; ++t) oe.col(t, x[t], fe);
      mf4v gr[M::TG];
#pragma unroll
      for (int t = 0; t < M::TG; ++t) gr[t] = mf4v{0, 0, 0, 0};
#pragma unroll
      for (int t = 0; t < NTN; ++t) og.col(t, x[t], gr);
#pragma unroll
      for (int q = 0; q < 3 * n; ++q) {
        const R w = (FR(le)[2 + q / n].info & 1) ? R(0.5) + g.beta : R(0.5) - g.beta;
        og.col(NTN + q, w * (jq[q] - fe[q / 4][q % 4]), gr);
      }
      if (it < NI) {
#pragma unroll
        for (int t = 0; t < NTN; ++t) {
          const R g0 = gr[t / 4][t % 4], g1 = gr[(NTN + t) / 4][(NTN + t) % 4];
          if constexpr (WARP) {
            X[(5 + v) * NU + t] = g0;
            X[(10 + v) * NU + t] = g1;
          } else {
            const R g2 = X[(15 + v) * NU + t];
            const R* Mt = sMet[le];  // Mt[3 d + c] = (J^-1)_{dc}
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

  // phase 3: triangle planes of the 20 fields, in registers until phase 5;
  // their values at the edge points (gradcoru_fpts), in registers until EF
  // may overwrite the state; the normal viscous flux at the triangle nodes
  // (both faces of a line)
  constexpr int NP = EB * 20 * n, NIT = (NP + NT_ - 1) / NT_;
  R xv[NIT][NTN];
  mf4v fe[NIT][M::TE];
#pragma unroll
  for (int j = 0; j < NIT; ++j) {
    const int it = tid + j * NT_, itc = it < NP ? it : 0;
    const int le = itc / (20 * n), fk = itc - le * (20 * n), fld = fk / n, k = fk - fld * n;
    const R* x = XS(le) + fld * NU + NTN * k;
#pragma unroll
    for (int t = 0; t < NTN; ++t) xv[j][t] = x[t];
#pragma unroll
    for (int t = 0; t < M::TE; ++t) fe[j][t] = mf4v{0, 0, 0, 0};
#pragma unroll
    for (int t = 0; t < NTN; ++t) oe.col(t, xv[j][t], fe[j]);
  }
  // (from the first thread on; phase 4 goes from the last, so that the waves share the surplus)
  for (int it = tid; it < EB * NTN; it += NT_) {
    const int le = it / NTN, t = it - le * NTN, e = e0 + le;
    if (e >= E) continue;
    const R* X = XS(le) + t;
    R fm[20], fp[20];
#pragma unroll
    for (int fld = 0; fld < 20; ++fld) {
      R sm = R(0), sp = R(0);
#pragma unroll
      for (int k = 0; k < n; ++k) {
        const R x = X[fld * NU + NTN * k];
        sm += op.lb[k] * x;
        sp += op.rb[k] * x;
      }
      fm[fld] = sm;
      fp[fld] = sp;
    }
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      const R* w = side ? fp : fm;
      const int po = sg.po_base + e * F::PPE + side * NTN;
      R nn[3];
      if constexpr (WARP) {
        wedge_tri_normal(tri, &sV[le][0], t, side, nn);
      } else {
        const R sgn = (FR(le)[side].info & 1) ? R(1) : R(-1);
#pragma unroll
        for (int c = 0; c < 3; ++c) nn[c] = sgn * FG(le)[side][c];
      }
      R u[5], q[3][5], V[4];
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        u[v] = w[v];
#pragma unroll
        for (int d = 0; d < 3; ++d) q[d][v] = w[5 + d * 5 + v];
      }
      normal_viscous(u, q, nn, g, V);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) Vf[(size_t)po * 4 + kk * NTN + t] = V[kk];
    }
  }
  lds_barrier();
#pragma unroll
  for (int j = 0; j < NIT; ++j) {
    const int it = tid + j * NT_;
    if (it < NP) {
      const int le = it / (20 * n), fk = it - le * (20 * n), fld = fk / n, k = fk - fld * n;
      R* EF = ES(le) + fld * C::EFS + n * k;
#pragma unroll
      for (int q = 0; q < 3 * n; ++q) EF[(q / n) * NFP + q % n] = fe[j][q / 4][q % 4];
    }
  }
  lds_barrier();

  // phase 4: normal viscous flux at the quadrilateral-face points
  for (int it = NT_ - 1 - tid; it < EB * 3 * NFP; it += NT_) {
    const int le = it / (3 * NFP), r1 = it - le * (3 * NFP), e = e0 + le;
    if (e >= E) continue;
    const int ed = r1 / NFP, r2 = r1 - ed * NFP;
    const int po = sg.po_base + e * F::PPE + F::foff(2 + ed);
    R nn[3];
    if constexpr (WARP) {
      wedge_quad_normal(op, &sV[le][0], ed, r2, nn);
    } else {
      const R sgn = (FR(le)[2 + ed].info & 1) ? R(1) : R(-1);
#pragma unroll
      for (int c = 0; c < 3; ++c) nn[c] = sgn * FG(le)[2 + ed][c];
    }
    const R* EF = ES(le) + r1;
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
  Mf4Op<M::TT, NTN> ot;
  ot.load(tab + B::tq, lane);
  const float azi = tab[B::zint + lane], azp = tab[B::zproj + lane];
  lds_barrier();

  // phase 5: triangle-plane interpolation of the 20 fields to the triangle
  // quadrature points (first factor of M7 / M10), over the state
#pragma unroll
  for (int j = 0; j < NIT; ++j) {
    const int it = tid + j * NT_, itc = it < NP ? it : 0;
    const int le = itc / (20 * n), fk = itc - le * (20 * n);
    mf4v s[M::TT];
#pragma unroll
    for (int t = 0; t < M::TT; ++t) s[t] = mf4v{0, 0, 0, 0};
#pragma unroll
    for (int t = 0; t < NTN; ++t) ot.col(t, xv[j][t], s);
    if (it < NP) {
      R* T = TS(le) + fk * M::TQS;
      if constexpr (M::TQS % 4 == 0) {
#pragma unroll
        for (int t = 0; t < M::TT; ++t) reinterpret_cast<mf4v*>(T)[t] = s[t];
      } else {
        typedef float f2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int t = 0; t < NTQ / 2 + NTQ % 2; ++t)
          reinterpret_cast<f2*>(T)[t] = f2{s[t / 2][2 * (t % 2)], s[t / 2][2 * (t % 2) + 1]};
      }
    }
  }
  lds_barrier();

  // phase 6: lane and lane + 32 hold one quadrature column: zeta
  // interpolation (uqpts, gradcoru_qpts) of the 20 fields to all levels of
  // the half at once, then per level the flux (tdisf) and the zeta
  // projection; rows 0..3 of the projection on the matrix cores, row 4
  // (p = 4) on the vector unit
  const int half = lane >> 5, cc = wave * 32 + (lane & 31);
  const bool col = cc < EB * NTQ;
  const int ccc = col ? cc : 0, cle = ccc / NTQ, ctq = ccc - cle * NTQ;
  constexpr int L0 = M::L0;
  mf4v acc[3][NVF];
  R acc4[3][NVF];
  {
    const R* T = TS(cle) + ctq;
    mf4v w[20];
#pragma unroll
    for (int fld = 0; fld < 20; ++fld) {
      w[fld] = mf4v{0, 0, 0, 0};
#pragma unroll
      for (int k = 0; k < n; ++k) w[fld] = mf4<3>(azi, T[(fld * n + k) * M::TQS], w[fld], k);
    }
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int v = 0; v < NVF; ++v) {
        acc[d][v] = mf4v{0, 0, 0, 0};
        acc4[d][v] = R(0);
      }
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
#pragma unroll
    for (int r = 0; r < L0; ++r) {
      constexpr int H = m - L0;                       // levels of the upper half
      const int k1 = L0 + (r < H ? r : H - 1);        // its level at this step
      R u[5], q[3][5], f[3][5];
#pragma unroll
      for (int fld = 0; fld < 20; ++fld) {
        if (fld < 5)
          u[fld] = w[fld][r];
        else
          q[(fld - 5) / 5][(fld - 5) % 5] = w[fld][r];
      }
      point_flux(u, q, g, f);
      if constexpr (WARP) {
        R det;
        wedge_metric(&sV[cle][0], cqx, cqy, half ? op.xq[k1] : op.xq[r], S, det);  // det J J^-1 here
      }
      R p4 = R(0), a4 = R(0);
      if constexpr (n > 4) {
        p4 = half ? (r < H ? op.Pj[n - 1][k1] : R(0)) : op.Pj[n - 1][r];
        a4 = half ? (r < H ? op.AP[n - 1][k1] : R(0)) : op.AP[n - 1][r];
      }
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int v = V0; v < 5; ++v) {
          const R ft = S[d][0] * f[0][v] + S[d][1] * f[1][v] + S[d][2] * f[2][v];
          acc[d][v - V0] = mf4<3>(azp, ft, acc[d][v - V0], d == 2 ? 4 + r : r);
          if constexpr (n > 4) acc4[d][v - V0] += (d == 2 ? a4 : p4) * ft;
        }
    }
  }
  Mf4Op<M::TPG, M::KP> opj;
  // share of the projection's row tiles (one share: the waves loop over the
  // columns; more: every wave has at most one 64-column part of one share)
  const int pg = M::G > 1 && wave < M::IW * M::G ? wave / M::IW : 0;
  opj.load(tab + (LIN ? B::proj : B::projc) + pg * Mf4Op<M::TPG, M::KP>::FLOATS, lane);
  lds_barrier();  // every column has read T1; Z may now overwrite it
  {
    // values in the order (d, v, k), summed over the halves two at a time:
    // the lower half gets and writes the even ones, the upper the odd ones
    auto val = [&](int i) -> R {
      const int dv = i / n, k = i - dv * n;
      return k < 4 ? acc[dv / NVF][dv % NVF][k < 4 ? k : 0] : acc4[dv / NVF][dv % NVF];
    };
    constexpr int NV = 3 * NVF * n;
    R* Z = ZS(cle) + ctq * n;
#pragma unroll
    for (int i = 0; i < NV; i += 2) {
      const bool two = i + 1 < NV;
      const R s = half_sums(val(i), val(two ? i + 1 : i));
      const int z0 = (i / n) * M::ZVS + i % n, z1 = two ? ((i + 1) / n) * M::ZVS + (i + 1) % n : z0;
      if (col && (two || !half)) Z[half ? z1 : z0] = s;
    }
  }
  lds_barrier();

  // phase 7: triangle-plane projection-divergence of one (variable, plane)
  // per lane, this wave's share of the row tiles; LIN: the energy residual
  // takes kap L(rho v) (row 0, from the disu kernel)
  for (int wp = wave; wp < M::IW * M::G; wp += W) {
    constexpr int NJ = EB * NVF * n;
    const int it = (wp - pg * M::IW) * 64 + lane, itc = it < NJ ? it : 0;
    const int le = itc / (NVF * n), r0 = itc - le * (NVF * n), vv = r0 / n, k = r0 - vv * n, e = e0 + le, v = vv + V0;
    const bool ok = it < NJ && e < E;
    R* out = Rp + (size_t)(ok ? e : e0) * 5 * NU + NTN * k;
    const int t0 = pg * 4 * M::TPG;
    R lin[4 * M::TPG];
    if constexpr (LIN) {
#pragma unroll
      for (int t = 0; t < 4 * M::TPG; ++t) lin[t] = out[t0 + t < NTN ? t0 + t : 0];
    }
    const R* Z = ZS(le) + vv * M::ZVS + k;
    mf4v s[M::TPG];
#pragma unroll
    for (int t = 0; t < M::TPG; ++t) s[t] = mf4v{0, 0, 0, 0};
#pragma unroll
    for (int tq = 0; tq < NTQ; ++tq)
#pragma unroll
      for (int d = 0; d < 3; ++d) opj.col(3 * tq + d, Z[d * NVF * M::ZVS + tq * n], s);
    if (ok) {
#pragma unroll
      for (int t = 0; t < 4 * M::TPG; ++t) {
        R x = s[t / 4][t % 4];
        if (LIN && v == 4) x += g.kap * lin[t];
        if (t0 + t < NTN) out[v * NU + t0 + t] = x;
      }
    }
  }
#undef XS
#undef JS
#undef ES
#undef FR
#undef FG
#undef TS
#undef ZS
}

}  // namespace fr
