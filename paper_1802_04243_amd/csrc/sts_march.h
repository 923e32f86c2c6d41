// One Jacobi pass (FP64) over a column strip of the grid by one wave, which
// walks up y.  Included by sts_kernels.hip inside its namespaces; uses its
// elementary functions.
//
// Lane l takes the column x0 - 3 + l; the three lanes at each end are halo.
// The rows the equations of row k read (k-2 .. k+1, with one more of rho
// ahead in the implicit schemes) stand in a ring of rows in LDS that belongs
// to the wave alone, so nothing waits at a barrier; the next row's loads are
// issued a whole row of arithmetic ahead.  What two neighbouring volumes
// share -- the conduction and shear conductances, Gamma on the corners, the
// fluxes and their limiters, the face-centre velocities, the terms of the
// pressure equation -- is computed once, by the volume on whose low side the
// face lies, and handed to the other: across a row by a lane shift, from row
// to row in a register.  Every value is formed by the same expression as in
// the tile kernels (t_update, u_pseudo, v_pseudo, pass_body), so the two
// agree bitwise.
//
// Bound: dependent FP64 instructions at two waves per SIMD (some 200 VGPRs; a
// third wave spills them and is slower).  A row of a wave takes about 430 VALU
// instructions, 7.4 per volume with the halo lanes where the tiles take 15.8
// (implicit TVD 14.4 and 24.6); the VALU is busy 0.55 of the time (implicit
// TVD 0.67), and for 0.3 to 0.45 of its cycles a wave waits for memory or LDS.
// Measured (pass, 5120x1152): explicit TVD 224 ->
// 153 us, explicit upwind 219 -> 153, implicit upwind 245 -> 165, implicit TVD
// 329 -> 237; 0.61 GB of HBM traffic.  Prefetching two rows ahead instead of
// one, and loading the uniform values anew in every section, were slower.
constexpr int MH = 3;             // halo lanes on each side
static_assert(64 - 2 * MH == STRIP_W && MH == HB, "the work items are cut for these strips");
constexpr int MPAD = 2;           // LDS entries beyond the wave at each end
constexpr int MROW = 64 + 2 * MPAD;
constexpr int MFLD = 6;           // u, v, p, T, rho, Gamma
template <bool IM>
constexpr int march_rows = IM ? 5 : 4;

typedef const __attribute__((address_space(4))) double *CDbl;

// the value of the next (i + 1) and of the previous (i - 1) lane's column
template <int CTRL>
__device__ __forceinline__ double lane_shift(double x) {
  union {
    double d;
    int i[2];
  } a, b;
  a.d = x;
  b.i[0] = __builtin_amdgcn_update_dpp(0, a.i[0], CTRL, 0xf, 0xf, true);
  b.i[1] = __builtin_amdgcn_update_dpp(0, a.i[1], CTRL, 0xf, 0xf, true);
  return b.d;
}
__device__ __forceinline__ double next_lane(double x) { return lane_shift<0x130>(x); }
__device__ __forceinline__ double prev_lane(double x) { return lane_shift<0x138>(x); }
__device__ __forceinline__ int next_lane(int x) {
  return __builtin_amdgcn_update_dpp(0, x, 0x130, 0xf, 0xf, true);
}
__device__ __forceinline__ int prev_lane(int x) {
  return __builtin_amdgcn_update_dpp(0, x, 0x138, 0xf, 0xf, true);
}

// the kernel's arguments, read through a pointer to their segment
struct SweepArgs {
  Params P;
  const double *o, *C;  // u of the old iterate, C_u; the other fields (v, p, T; C_v, C_T,
  double *n;            // C_p) follow at a distance of `field` doubles; u of the new iterate
  long field;
  Resid X;
};
typedef const __attribute__((address_space(4))) SweepArgs *KArgs;
typedef const __attribute__((address_space(4))) Params KParams;
template <class T>
__device__ __forceinline__ T fresh(T a) {  // opaque: loads through it stay where they are
  asm volatile("" : "+s"(a));
  return a;
}
// Ends a section of a row: the next one reads its neighbours from LDS again
// (kept across the sections they would not fit the registers)
#define SECTION()                      \
  do {                                 \
    asm volatile("" ::: "memory");     \
    __builtin_amdgcn_sched_barrier(0); \
  } while (0)
// geometry factors of a row (Params::gy6), uniform
struct RowGeo {
  double d, id, s, is, wl, wr;
  __device__ __forceinline__ explicit RowGeo(CDbl p) {
    d = p[0], id = p[1], s = p[2], is = p[3], wl = p[4], wr = p[5];
  }
};

// the row's own and neighbouring values in the ring: each section reads what
// it uses
#define Q_TP (*at(s0, FT))
#define Q_gP (*at(s0, FG))
#define Q_gW (at(s0, FG)[-1])
#define Q_gN (*at(sp, FG))
#define Q_rP (*at(s0, FR))
#define Q_rW (at(s0, FR)[-1])
#define Q_gs (*at(sm1, FG))
#define Q_rS (*at(sm1, FR))
#define Q_u00 (*at(s0, FU))
#define Q_uE (at(s0, FU)[1])
#define Q_uW (at(s0, FU)[-1])
#define Q_uN0 (*at(sp, FU))
#define Q_uNE (at(sp, FU)[1])
#define Q_uS0 (*at(sm1, FU))
#define Q_uSE (at(sm1, FU)[1])
#define Q_v00 (*at(s0, FV))
#define Q_vN0 (*at(sp, FV))
#define Q_vW0 (at(s0, FV)[-1])
#define Q_vNW (at(sp, FV)[-1])
#define Q_vS0 (*at(sm1, FV))
#define Q_vE0 (at(s0, FV)[1])

// Columns [x0, x0 + w) (w <= STRIP_W), rows [y0, y1).  solid: the window (three
// cells around) holds a solid cell, so every row takes the general rules.
// row: the strip's residual partials (RS).
template <bool IM, bool TV, bool RS>
__device__ __forceinline__ void march(double *ring, const KArgs ka, int x0, int w, int y0, int y1,
                                      bool solid, double *row) {
  KParams &P = ka->P;
  constexpr int NRW = march_rows<IM>;
  constexpr int LA = IM ? 2 : 1;  // the newest row in the ring while row k is computed
  const int lane = threadIdx.x & 63;
  const int nx = P.nx, ny = P.ny;
  const int gi = x0 - MH + lane;
  const bool io = !P.per;
  const bool own = lane >= MH && lane < MH + w;
  // loads: wrapped in a periodic x, else inside the frame
  const int ci = P.per ? wrapi(gi, nx) : clampi(gi, -XPAD, nx + XPAD - 1);
  const int ui = P.per ? wrapi(gi, nx) : clampi(gi, -XPAD, nx + XPAD);
  const unsigned cb = 8u * (unsigned)(XO + ci), ub = 8u * (unsigned)(XO + ui);
  const long pitch = P.pitch;
  // array row of the grid row j of a field; one base per iterate and the
  // distance of its fields, to keep the scalar registers free
  const long fld = ka->field;
  const double *const ob = ka->o + (P.off - XO), *const cbp = ka->C + (P.off - XO);
  auto ld = [&](const double *a, int f, int j, unsigned at) {
    return *(const double *)((const char *)(a + f * fld + (long)j * pitch) + at);
  };

  // per-lane geometry
  const double *gx = P.gx6 + 6 * (ci + XPAD);
  const double dxi = gx[0], idx = gx[1], sx = gx[2], isx = gx[3], wlx = gx[4], wrx = gx[5];
  const double dxl = prev_lane(dxi);
  const CDbl gyp = (CDbl)P.gy6 + 6 * XPAD;  // rows of the y geometry
  const CDbl inl = (CDbl)P.inl;              // inlet data of the rows
  const double dt = P.dt, idt = P.idt, PA = P.A, PB = P.B, C1 = P.C1, C2 = P.C2, C3 = P.C3;

  // the ring: row j at slot j mod NRW, addressed through the rotating offsets
  double *const my = ring + lane + MPAD;
  auto at = [&](int slot, int f) { return my + (slot * MFLD + f) * MROW; };
  enum { FU, FV, FP, FT, FR, FG };

  // fluid cells around the lane, per row of the ring: bit q is the cell
  // gi - 2 + q (general rows only)
  auto fluid = [&](int j) {
    const unsigned char *fl = P.fl + (P.off + (long)clampi(j, -XPAD, ny + XPAD - 1) * pitch + ci);
    return (int)*fl;
  };
  auto around = [&](int f) {
    const int a = prev_lane(f), b = next_lane(f);
    return prev_lane(a) | a << 1 | f << 2 | b << 3 | next_lane(b) << 4;
  };
  int fm2 = 31, fm1 = 31, f0 = 31, fp = 31, fq = 31;  // rows k-2 .. k+2

  struct Row {
    double u, v, p, T;
  };
  auto fetch = [&](int j, Row &r) {
    r.u = ld(ob, 0, j, ub);
    r.v = ld(ob, 1, j, cb);
    r.p = ld(ob, 2, j, cb);
    r.T = ld(ob, 3, j, cb);
  };
  auto stash = [&](int slot, const Row &r) {
    *at(slot, FU) = r.u;
    *at(slot, FV) = r.v;
    *at(slot, FP) = r.p;
    *at(slot, FT) = r.T;
    *at(slot, FR) = ddiv(r.p, r.T);
    *at(slot, FG) = sqrt(r.T);
    // the other lanes' values are read below: LDS operations of one wave
    // complete in order, only the compiler has to keep them so
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  struct RowConst {
    double T, u, v, p;
  };
  auto constants = [&](int j, RowConst &c) {
    c.u = ld(cbp, 0, j, ub);
    c.v = ld(cbp, 1, j, cb);
    c.T = ld(cbp, 2, j, cb);
    c.p = ld(cbp, 3, j, cb);
  };

  // rows of the equations: kf .. y1 (the v-face y1 is the last one needed)
  const int kf = y0 > 0 ? y0 - 1 : 0;
  const bool xl = io && gi == 0, xh = io && gi == nx - 1, xn = io && gi == nx;
  // a strip or row next to a boundary (its rules are compiled out elsewhere)
  const bool xedge = io && (x0 - MH < 2 || x0 + w + MH > nx - 2);
  const bool uin = P.per || (gi >= 1 && gi <= nx - 1);
  // v stencil i-2 .. i+1 (in the general rows' cell stencils every cell must
  // also be fluid)
  const bool tvx = !io || (gi >= 2 && gi + 1 <= nx - 1);
  const bool tvu = !io || (gi >= 2 && gi + 1 <= nx);       // u-face stencil

  // slots of the rows k-2, k-1, k, k+1 (and k+2)
  int sm2 = 0, sm1 = 1, s0 = 2, sp = 3, sq = NRW - 1;
  // Gamma linear in x at the u-face, of the newest row with equations ahead
  auto gface = [&](bool eg, int slot, int j) {
    const double g0 = *at(slot, FG), gl = at(slot, FG)[-1];
    double g = wlx * gl + wrx * g0;
    if (eg) {
      if (xl) g = inl[4 * clampi(j, 0, ny - 1) + 2];
      if (xn) g = gl;
    }
    return g;
  };
  // face density rho^v on the face j between the rows of slots b and c (a, d
  // the rows outside them)
  auto rho_v = [&](int j, int a, int b, int c, int d, bool ok) {
    const double vf = *at(c, FV), rs = *at(b, FR), rn = *at(c, FR);
    if (j == 0) return rn;
    if (j == ny) return rs;
    double r = upw(rs, rn, vf);
    if (TV && ok) {
      const RowGeo g0(gyp + 6 * (j - 1)), g1(gyp + 6 * j), g2(gyp + 6 * (j + 1));
      r += psi_sf(*at(a, FR), rs, rn, *at(d, FR), g0.s, g1.s, g2.s, g1.wr, g1.wl, vf) * (rn - rs);
    }
    return r;
  };

  const bool edge = xedge || solid;
  // rows whose four cells j-2 .. j+1 of the own column exist
  auto four = [&](int j) { return j >= 2 && j + 1 <= ny - 1; };
  auto mid = [](int m) { return (m >> 2 & 1) != 0; };  // the own cell
  Row nr;
  RowConst cn;
  {
    // the rows kf-2 .. kf+LA-1 into the ring; every load before the first wait
    Row a, b, c, d;
    fetch(kf - 2, a);
    fetch(kf - 1, b);
    fetch(kf, c);
    if (IM) fetch(kf + 1, d);
    fetch(kf + LA, nr);
    constants(kf, cn);
    stash(sm2, a);
    stash(sm1, b);
    stash(s0, c);
    if (IM) stash(sp, d);
  }
  // what the row below hands up to row kf
  if (edge) {
    const int a = fluid(kf - 2), b = fluid(kf - 1), c = fluid(kf), d = fluid(kf + 1);
    fm1 = around(a), f0 = around(b), fp = around(c), fq = around(d);
  }
  const RowGeo gb0(gyp + 6 * (kf - 1)), g00(gyp + 6 * kf);
  double gxk = gface(true, s0, kf);
  const double gxb = gface(true, sm1, kf - 1);
  const bool low = kf == 0;
  double cS = low ? 0.0 : g00.wl * gxb + g00.wr * gxk;  // Gamma on the corner (i, kf)
  double dST = C1 * hmean(gb0.d, *at(sm1, FG), g00.d, *at(s0, FG)) * dxi * (2.0 * g00.is);
  double dSu = PB * cS * sx * g00.is;
  double dSv = PB * *at(sm1, FG) * dxi * gb0.id;
  double uSf, rvS = 0.0, FS = 0.0, pST = 0.0, ps0 = 0.0, ps1 = 0.0, psV = 0.0, FWb = 0.0;
  {
    const double uc = 0.5 * (*at(s0, FU) + at(s0, FU)[1]);
    uSf = g00.wl * (0.5 * (*at(sm1, FU) + at(sm1, FU)[1])) + g00.wr * uc;
  }
  if constexpr (IM) {
    // fluxes of the face kf and of the row below, and their limiters
    const double v = *at(s0, FV), vW = at(s0, FV)[-1], vb = *at(sm1, FV), u = *at(sm1, FU);
    const bool ok4 = four(kf) && mid(fm1 & f0 & fp & fq);
    rvS = rho_v(kf, sm2, sm1, s0, sp, ok4);
    FS = rvS * v * dxi;
    const double rl = at(sm1, FR)[-1], rr = *at(sm1, FR);
    double ru = upw(rl, rr, u);
    const double sxl = prev_lane(sx), sxh = next_lane(sx);
    if (TV && tvx && (f0 & 15) == 15)
      ru += psi_sf(at(sm1, FR)[-2], rl, rr, at(sm1, FR)[1], sxl, sx, sxh, wrx, wlx, u) * (rr - rl);
    if (xl) ru = u > 0.0 ? inl[4 * clampi(kf - 1, 0, ny - 1) + 3] : rr;
    if (xn) ru = rl;
    FWb = ru * u * gb0.d;
    if (TV && four(kf)) {
      const RowGeo g1(gyp + 6 * (kf + 1));
      if (ok4) pST = psi_sf(*at(sm2, FT), *at(sm1, FT), *at(s0, FT), *at(sp, FT), gb0.s, g00.s, g1.s, g00.wr, g00.wl, v);
      const double f1 = *at(sm2, FU), f2 = *at(sm1, FU), f3 = *at(s0, FU), f4 = *at(sp, FU);
      ps0 = psi_sf(f1, f2, f3, f4, gb0.s, g00.s, g1.s, g00.wr, g00.wl, v);
      ps1 = psi_sf(f1, f2, f3, f4, gb0.s, g00.s, g1.s, g00.wr, g00.wl, vW);
    }
    if (TV && kf >= 2 && kf + 1 <= ny)
      psV = psi_c(*at(sm2, FV), vb, v, *at(sp, FV), RowGeo(gyp + 6 * (kf - 2)).d, gb0.d, g00.d, 0.5 * (vb + v));
  }
  // the pressure equation of the row below, as far as it is known
  double Tn = 1.0, uh = 0.0, du = 0.0, ax = 0.0, apx = 0.0, bx = 0.0, cpm = 0.0, ruM = 0.0;
  double aS = 0.0, bS = 0.0, vhS = 0.0, dvS = 0.0, pnB = 0.0, ruE = 0.0, rvB = 0.0;
  double m0 = 0.0, m1 = 0.0, m2 = 0.0, m3 = 0.0, bad = 0.0;  // increments (RS)

  int fnx = edge ? fluid(kf + 2) : 31;
  for (int k = kf; k <= y1; k++) {
    const RowGeo gb(gyp + 6 * (k - 1)), g0(gyp + 6 * k), gt(gyp + 6 * (k + 1)), gn(gyp + 6 * (k + 2));
    stash(IM ? sq : sp, nr);
    const RowConst cc = cn;
    if (k < y1) {
      fetch(k + LA + 1, nr);
      constants(k + 1, cn);
    }
    if (edge) {
      fm2 = fm1, fm1 = f0, f0 = fp, fp = fq;
      fq = around(fnx);
      fnx = fluid(k + 3);
    }
    double vh, dv, rvk, aN, bN, Tk = 0.0, uhk = 0.0, duk = 0.0, axk = 0.0, apxk = 0.0, bxk = 0.0,
                                ruk = 0.0;

    auto equations = [&](auto egc) {
      constexpr bool EG = decltype(egc)::value;
      const bool XL = EG && xl, XH = EG && xh;
      // solid neighbours of the cell, and the face's own conditions
      const bool SW = EG && !XL && !(f0 & 2), SE = EG && !XH && !(f0 & 8);
      const bool SS = EG && k > 0 && !mid(fm1), SN = EG && k < ny - 1 && !mid(fp);
      const bool YL = EG && k == 0, YH = EG && k == ny - 1;
      const KArgs ke = EG ? fresh(ka) : ka;  // rarely used values are loaded where they are
      KParams &P = ke->P;
      const bool sj = EG && P.otype == 2;
      const double dyj = g0.d, dV = dxi * dyj;
      // face density on the low x-face (a lane shift stands outside branches: it
      // reads nothing from lanes that are switched off)
      const double sxl = prev_lane(sx), sxh = next_lane(sx);
      {
        const double rl = Q_rW, rr = Q_rP;
        ruk = upw(rl, rr, Q_u00);
        if (TV && (!EG || (f0 & 15) == 15))
          ruk += psi_sf(at(s0, FR)[-2], rl, rr, at(s0, FR)[1], sxl, sx, sxh, wrx, wlx, Q_u00) * (rr - rl);
        if (XL) ruk = Q_u00 > 0.0 ? inl[4 * k + 3] : Q_rP;
        if (EG && xn) ruk = Q_rW;
      }
      // mass fluxes through the four faces, of the low ones' limiters of T
      double FW = 0.0, FE = 0.0, FN = 0.0, pW = 0.0, pE = 0.0, pN = 0.0, rvN = 0.0;
      if constexpr (IM) {
        rvN = rho_v(k + 1, sm1, s0, sp, sq, !EG || (four(k + 1) && mid(fm1 & f0 & fp & fq)));
        FW = ruk * Q_u00 * dyj;
        FE = next_lane(FW);
        FN = rvN * Q_vN0 * dxi;
        if (TV) {
          if (!EG || (f0 & 15) == 15)
            pW = psi_sf(at(s0, FT)[-2], at(s0, FT)[-1], Q_TP, at(s0, FT)[1], sxl, sx, sxh, wrx, wlx, Q_u00);
          pE = next_lane(pW);
          if (!EG || (four(k + 1) && mid(fm1 & f0 & fp & fq)))
            pN = psi_sf(*at(sm1, FT), Q_TP, *at(sp, FT), *at(sq, FT), g0.s, gt.s, gn.s,
                        gt.wr, gt.wl, Q_vN0);
        }
      }
      // of the row above the strip only the v-face below it is needed
      const bool whole = k < y1;
      // ---- energy ----
      SECTION();
      if (whole) {
        double nW = at(s0, FT)[-1], nE = at(s0, FT)[1], nS = *at(sm1, FT), nN = *at(sp, FT);
        double DW = C1 * hmean(dxl, Q_gW, dxi, Q_gP) * dyj * (2.0 * isx);
        if (XL) {
          nW = inl[4 * k + 1];
          DW = C1 * hmean2(Q_gP, inl[4 * k + 2]) * dyj * (2.0 * idx);
        }
        double DE = next_lane(DW);
        if (XH) {
          nE = Q_TP;
          DE = 0.0;
        }
        if (SW)
          DW = sj ? C1 * Q_gP * dyj * iwall(dxi, P.kt, Q_rP)
                  : C1 * hmean2(Q_gP, P.sq_obsT) * dyj * (2.0 * idx);
        if (SE)
          DE = sj ? C1 * Q_gP * dyj * iwall(dxi, P.kt, Q_rP)
                  : C1 * hmean2(Q_gP, P.sq_obsT) * dyj * (2.0 * idx);
        double DS = dST;
        if (YL) {
          const int wc = P.per ? ci : clampi(ci, 0, nx - 1);
          if (P.wtype0 == 0) {
            nS = P.wl[4 * wc];
            DS = C1 * hmean2(Q_gP, P.wl[4 * wc + 2]) * dxi * (2.0 * g0.id);
          } else if (P.wtype0 == 2) {
            nS = P.wl[4 * wc];
            DS = C1 * Q_gP * dxi * iwall(dyj, P.kt, Q_rP);
          } else {
            nS = Q_TP;
            DS = 0.0;
          }
        }
        if (SS)
          DS = sj ? C1 * Q_gP * dxi * iwall(dyj, P.kt, Q_rP)
                  : C1 * hmean2(Q_gP, P.sq_obsT) * dxi * (2.0 * g0.id);
        dST = C1 * hmean(dyj, Q_gP, gt.d, Q_gN) * dxi * (2.0 * gt.is);
        double DN = dST;
        if (SN)
          DN = sj ? C1 * Q_gP * dxi * iwall(dyj, P.kt, Q_rP)
                  : C1 * hmean2(Q_gP, P.sq_obsT) * dxi * (2.0 * g0.id);
        if (YH) {
          const int wc = P.per ? ci : clampi(ci, 0, nx - 1);
          if (P.wtype1 == 0) {
            nN = P.wl[4 * wc + 1];
            DN = C1 * hmean2(Q_gP, P.wl[4 * wc + 3]) * dxi * (2.0 * g0.id);
          } else if (P.wtype1 == 2) {
            nN = P.wl[4 * wc + 1];
            DN = C1 * Q_gP * dxi * iwall(dyj, P.kt, Q_rP);
          } else {
            nN = Q_TP;
            DN = 0.0;
          }
        }
        double aW, aE, aS_, aN_, a0;
        if (IM) {
          aW = dmax(0.0, FW) - FW * pW + DW;
          aE = dmax(0.0, -FE) - FE * pE + DE;
          aS_ = dmax(0.0, FS) - FS * pST + DS;
          aN_ = dmax(0.0, -FN) - FN * pN + DN;
          a0 = dt * ((aW + aE + aS_ + aN_) + ((FE - FW) + (FN - FS))) + Q_rP * dV;
        } else {
          aW = DW;
          aE = DE;
          aS_ = DS;
          aN_ = DN;
          a0 = dt * (aW + aE + aS_ + aN_) + Q_rP * dV;
        }
        const double vc = 0.5 * (Q_v00 + Q_vN0), uc = 0.5 * (Q_u00 + Q_uE);
        double vWf = wlx * (0.5 * (Q_vW0 + Q_vNW)) + wrx * vc;
        double vEf = next_lane(vWf);
        if (XL) vWf = 0.0;
        if (XH) vEf = vc;
        if (SW) vWf = sj ? slip_vel(0.0, vc, dxi, P.kz / Q_rP) : 0.0;
        if (SE) vEf = sj ? slip_vel(0.0, vc, dxi, P.kz / Q_rP) : 0.0;
        const double uNi = gt.wl * uc + gt.wr * (0.5 * (Q_uN0 + Q_uNE));
        double uNf = uNi, uS_ = uSf;
        if (SS) uS_ = sj ? slip_vel(0.0, uc, dyj, P.kz / Q_rP) : 0.0;
        if (SN) uNf = sj ? slip_vel(0.0, uc, dyj, P.kz / Q_rP) : 0.0;
        if (YL)
          uS_ = P.wtype0 == 0 ? P.wu0 : (P.wtype0 == 2 ? slip_vel(P.wu0, uc, dyj, P.kz / Q_rP) : uc);
        if (YH)
          uNf = P.wtype1 == 0 ? P.wu1 : (P.wtype1 == 2 ? slip_vel(P.wu1, uc, dyj, P.kz / Q_rP) : uc);
        uSf = uNi;
        const double ux = (Q_uE - Q_u00) * idx;
        const double vy = (Q_vN0 - Q_v00) * g0.id;
        const double vx = (vEf - vWf) * idx, uy = (uNf - uS_) * g0.id;
        const double dvg = ux + vy;
        const double Sc = C2 * Q_gP * (2.0 * (ux * ux + vy * vy) + (vx + uy) * (vx + uy) -
                                       2.0 / 3.0 * dvg * dvg) *
                              dV +
                          C3 * *at(s0, FP) * dvg * dV;
        Tk = ddiv(dt * (aW * nW + aE * nE + aS_ * nS + aN_ * nN + Sc) + cc.T, a0);
        if (EG && !mid(f0)) Tk = Q_TP;
      }
      SECTION();
      // Gamma on the corners (i, k + 1); that of the next column
      const double gxn = gface(EG, sp, k + 1);
      double cN = gt.wl * gxk + gt.wr * gxn;
      if (YH) cN = 0.0;
      const double cE = next_lane(cS);
      // ---- u ----
      if (whole) {
        SECTION();
        const double rl = Q_rW, rr = Q_rP, gl = Q_gW, gr = Q_gP;
        const double M = (rr * dxi + rl * dxl) * dyj / 2.0;
        const double len = 0.5 * (dxl + dxi);
        const double gnode = wlx * gl + wrx * gr;
        double nS = Q_uS0, nN = Q_uN0, DS = dSu;
        const double DNi = PB * cN * sx * gt.is;
        double DN = DNi;
        if (EG && k > 0 && !(fm1 & 6))
          DS = sj ? PB * gnode * len * iwall(dyj, P.kz, wlx * rl + wrx * rr)
                  : PB * 0.5 * (gnode + P.sq_obsT) * len * (2.0 * g0.id);
        if (EG && k < ny - 1 && !(fp & 6))
          DN = sj ? PB * gnode * len * iwall(dyj, P.kz, wlx * rl + wrx * rr)
                  : PB * 0.5 * (gnode + P.sq_obsT) * len * (2.0 * g0.id);
        if (YL) {
          const int wu = P.per ? ui : clampi(ui, 0, nx);
          if (P.wtype0 == 0) {
            nS = P.wu0;
            DS = PB * 0.5 * (gnode + P.wu[2 * wu]) * len * (2.0 * g0.id);
          } else if (P.wtype0 == 2) {
            nS = P.wu0;
            DS = PB * gnode * len * iwall(dyj, P.kz, wlx * rl + wrx * rr);
          } else {
            nS = Q_u00;
            DS = 0.0;
          }
        }
        if (YH) {
          const int wu = P.per ? ui : clampi(ui, 0, nx);
          if (P.wtype1 == 0) {
            nN = P.wu1;
            DN = PB * 0.5 * (gnode + P.wu[2 * wu + 1]) * len * (2.0 * g0.id);
          } else if (P.wtype1 == 2) {
            nN = P.wu1;
            DN = PB * gnode * len * iwall(dyj, P.kz, wlx * rl + wrx * rr);
          } else {
            nN = Q_u00;
            DN = 0.0;
          }
        }
        dSu = DNi;
        const double DE = PB * gr * dyj * idx, DW = prev_lane(DE);
        double aS_, aN_, aW, aE, conv;
        if constexpr (IM) {
          const double Fs0 = FS, Fs1 = prev_lane(FS), Fn0 = FN, Fn1 = prev_lane(FN);
          const double ubW = 0.5 * (Q_uW + Q_u00), ubE = 0.5 * (Q_u00 + Q_uE);
          const double FbW = rl * ubW * dyj, FbE = rr * ubE * dyj;
          double ps0_ = 0.0, ps1_ = 0.0, pn0_ = 0.0, pn1_ = 0.0, pw = 0.0, pe = 0.0;
          if (TV) {
            ps0_ = ps0;
            ps1_ = ps1;
            if (!EG || (k - 1 >= 0 && k + 2 <= ny - 1)) {
              const double f1 = Q_uS0, f3 = Q_uN0, f4 = *at(sq, FU), s2 = gn.s;
              pn0_ = psi_sf(f1, Q_u00, f3, f4, g0.s, gt.s, s2, gt.wr, gt.wl, Q_vN0);
              pn1_ = psi_sf(f1, Q_u00, f3, f4, g0.s, gt.s, s2, gt.wr, gt.wl, Q_vNW);
            }
            ps0 = pn0_;
            ps1 = pn1_;
            const double dxll = prev_lane(dxl);
            if (!EG || tvu) pw = psi_c(at(s0, FU)[-2], Q_uW, Q_u00, Q_uE, dxll, dxl, dxi, ubW);
            pe = next_lane(pw);
          }
          aS_ = 0.5 * (dmax(0.0, Fs0) - Fs0 * ps0_ + dmax(0.0, Fs1) - Fs1 * ps1_) + DS;
          aN_ = 0.5 * (dmax(0.0, -Fn0) - Fn0 * pn0_ + dmax(0.0, -Fn1) - Fn1 * pn1_) + DN;
          aW = dmax(0.0, FbW) - FbW * pw + 4.0 / 3.0 * DW;
          aE = dmax(0.0, -FbE) - FbE * pe + 4.0 / 3.0 * DE;
          conv = 0.5 * (Fn0 - Fs0 + Fn1 - Fs1) + FbE - FbW;
        } else {
          aS_ = DS;
          aN_ = DN;
          aW = 4.0 / 3.0 * DW;
          aE = 4.0 / 3.0 * DE;
          conv = 0.0;
        }
        const double a0 = aS_ + aN_ + aW + aE + conv + M * idt;
        const double Xc = cN * (Q_vN0 - Q_vNW) - cS * (Q_v00 - Q_vW0) - 2.0 / 3.0 * gr * (Q_vN0 - Q_v00) +
                          2.0 / 3.0 * gl * (Q_vNW - Q_vW0);
        const double b = cc.u + PB * Xc;
        const double ia0 = drcp(a0);
        uhk = (aS_ * nS + aN_ * nN + aW * Q_uW + aE * Q_uE + b) * ia0;
        duk = PA * dyj * ia0;
        if (EG && !(uin && (f0 & 6) == 6)) {
          uhk = Q_u00;
          duk = 0.0;
        }
      }
      // ---- v (the face between the rows k - 1 and k) ----
      {
        SECTION();
        const double rs = Q_rS, rn = Q_rP, gn = Q_gP, dys = gb.d, dyn = g0.d;
        const double M = (rn * dyn + rs * dys) * dxi / 2.0;
        const double len = 0.5 * (dys + dyn);
        const double gnode = g0.wl * Q_gs + g0.wr * gn;
        double nW = Q_vW0, nE = Q_vE0;
        double DW = PB * cS * g0.s * isx;
        double DE = next_lane(DW);
        if (XL) {
          nW = 0.0;
          DW = PB * 0.5 * (gnode + cS) * len * (2.0 * idx);
        }
        if (XH) {
          nE = Q_v00;
          DE = 0.0;
        }
        if (EG && !XL && !((fm1 | f0) & 2))
          DW = sj ? PB * gnode * len * iwall(dxi, P.kz, g0.wl * rs + g0.wr * rn)
                  : PB * 0.5 * (gnode + P.sq_obsT) * len * (2.0 * idx);
        if (EG && !XH && !((fm1 | f0) & 8))
          DE = sj ? PB * gnode * len * iwall(dxi, P.kz, g0.wl * rs + g0.wr * rn)
                  : PB * 0.5 * (gnode + P.sq_obsT) * len * (2.0 * idx);
        const double DS = dSv, DN = PB * gn * dxi * g0.id;
        dSv = DN;
        double aW, aE, aS_, aN_, conv;
        if constexpr (IM) {
          const double Fw0 = FW, Fw1 = FWb, Fe0 = FE, Fe1 = next_lane(FWb);
          const double vbS = 0.5 * (Q_vS0 + Q_v00), vbN = 0.5 * (Q_v00 + Q_vN0);
          const double fbS = rs * vbS * dxi, FbN = rn * vbN * dxi;
          const double sxl = prev_lane(sx), sxh = next_lane(sx);
          double pw0 = 0.0, pw1 = 0.0, pe0 = 0.0, pe1 = 0.0, ps = 0.0, pn = 0.0;
          if (TV) {
            if (!EG || tvx) {
              const double f1 = at(s0, FV)[-2], f4 = Q_vE0;
              pw0 = psi_sf(f1, nW, Q_v00, f4, sxl, sx, sxh, wrx, wlx, Q_u00);
              pw1 = psi_sf(f1, nW, Q_v00, f4, sxl, sx, sxh, wrx, wlx, Q_uS0);
            }
            pe0 = next_lane(pw0);
            pe1 = next_lane(pw1);
            ps = psV;
            if (!EG || (k - 1 >= 0 && k + 2 <= ny))
              pn = psi_c(Q_vS0, Q_v00, Q_vN0, *at(sq, FV), dys, dyn, gt.d, vbN);
            psV = pn;
          }
          aW = 0.5 * (dmax(0.0, Fw0) - Fw0 * pw0 + dmax(0.0, Fw1) - Fw1 * pw1) + DW;
          aE = 0.5 * (dmax(0.0, -Fe0) - Fe0 * pe0 + dmax(0.0, -Fe1) - Fe1 * pe1) + DE;
          aS_ = dmax(0.0, fbS) - fbS * ps + 4.0 / 3.0 * DS;
          aN_ = dmax(0.0, -FbN) - FbN * pn + 4.0 / 3.0 * DN;
          conv = 0.5 * (Fe0 - Fw0 + Fe1 - Fw1) + FbN - fbS;
        } else {
          aW = DW;
          aE = DE;
          aS_ = 4.0 / 3.0 * DS;
          aN_ = 4.0 / 3.0 * DN;
          conv = 0.0;
        }
        const double a0 = aW + aE + aS_ + aN_ + conv + M * idt;
        const double Xc = cE * (Q_uE - Q_uSE) - cS * (Q_u00 - Q_uS0) - 2.0 / 3.0 * gn * (Q_uE - Q_u00) +
                          2.0 / 3.0 * Q_gs * (Q_uSE - Q_uS0);
        const double b = cc.v + PB * Xc;
        const double ia0 = drcp(a0);
        vh = (aW * nW + aE * nE + aS_ * Q_vS0 + aN_ * Q_vN0 + b) * ia0;
        dv = PA * dxi * ia0;
        if (EG && (k == 0 || !mid(fm1 & f0))) {
          vh = Q_v00;
          dv = 0.0;
        }
      }
      if (IM) {
        FWb = FW;
        FS = FN;
        pST = pN;
        rvk = rvS;
        rvS = rvN;
      } else {
        rvk = rho_v(k, sm2, sm1, s0, sp, !EG || (four(k) && mid(fm2 & fm1 & f0 & fp)));
      }
      cS = cN;
      gxk = gxn;
      // the x part of the pressure equation of row k
      const double aWp = ruk * duk * dyj, bWp = ruk * uhk * dyj;
      const double aEp = next_lane(aWp), bEp = next_lane(bWp);
      axk = aWp + aEp;
      apxk = aWp * at(s0, FP)[-1] + aEp * at(s0, FP)[1];
      bxk = bEp - bWp;
      aN = rvk * dv * dxi;
      bN = rvk * vh * dxi;
    };
    if (k == ny) {  // the top wall: no unknown on its face
      vh = *at(s0, FV);
      dv = 0.0;
      rvk = *at(sm1, FR);
      aN = 0.0;
      bN = rvk * vh * dxi;
    } else if (edge || k < 3 || k >= ny - 3) {
      equations(std::true_type{});
    } else {
      equations(std::false_type{});
    }

    // ---- pressure and velocities of row k - 1 ----
    if (k > kf) {
      const int j = k - 1;
      const KArgs kr = ka;
      double *const nb = kr->n + (P.off - XO);
      const double dV = dxi * gb.d;
      const double a0 = ddiv(dV, Tn) + (ax + aS + aN) * dt;
      const double bp = cpm - (bx + bN - bS) * dt;
      double pn = ((apx + aS * *at(sm2, FP) + aN * *at(s0, FP)) * dt + bp) * drcp(a0);
      const bool cell = mid(fm1);  // row k - 1
      if (!cell) pn = *at(sm1, FP);
      const double pnW = prev_lane(pn);
      if (own && j >= y0) {
        const double uo = *at(sm1, FU), vo = *at(sm1, FV);
        const bool usol = uin && (fm1 & 6) == 6, vsol = j >= 1 && mid(fm2 & fm1);
        const double un = usol ? uh - du * (pn - pnW) : uo;
        const double vn = vsol ? vhS - dvS * (pn - pnB) : vo;
        auto st = [&](double *a, int jj, unsigned b, double x) {
          *(double *)((char *)(a + (long)jj * pitch) + b) = x;
        };
        st(nb + 3 * fld, j, cb, Tn);
        st(nb + 2 * fld, j, cb, pn);
        st(nb, j, ub, un);
        st(nb + 1 * fld, j, cb, vn);
        const bool ucopy = (io && gi == nx - 1) || (P.per && gi == 0);
        const unsigned kc = 8u * (unsigned)(XO + nx);
        if (ucopy) st(nb, j, kc, un);  // outlet / periodic copy
        if constexpr (RS) {
          const double gw = ruM * un * gb.d;
          st(kr->X.gu + (P.off - XO), j, ub, gw);
          st(kr->X.gv + (P.off - XO), j, cb, rvB * vn * dxi);
          if (ucopy) st(kr->X.gu + (P.off - XO), j, kc, P.per ? gw : ruE * un * gb.d);
          if (j == ny - 1) st(kr->X.gv + (P.off - XO), ny, cb, rvk * *at(s0, FV) * dxi);
          m0 = fmax(m0, fabs(un - uo));
          m1 = fmax(m1, fabs(vn - vo));
          bad += (double)(!isfinite(un)) + (double)(!isfinite(vn));
          if (cell) {
            m2 = fmax(m2, fabs(pn - *at(sm1, FP)));
            m3 = fmax(m3, fabs(Tn - *at(sm1, FT)));
            bad += (double)(!isfinite(pn)) + (double)(!isfinite(Tn));
          }
        }
      }
      pnB = pn;
    }
    Tn = Tk, uh = uhk, du = duk, ax = axk, apx = apxk, bx = bxk, cpm = cc.p;
    aS = aN, bS = bN, vhS = vh, dvS = dv;
    if constexpr (RS) ruM = ruk, ruE = next_lane(ruk), rvB = rvk;
    // rotate the ring
    const int t = sm2;
    sm2 = sm1, sm1 = s0, s0 = sp;
    if (IM) sp = sq, sq = t;
    else sp = t;
  }
  if constexpr (RS) {
    m0 = wave_max(m0), m1 = wave_max(m1), m2 = wave_max(m2), m3 = wave_max(m3), bad = wave_sum(bad);
    if (lane == 0) {
      row[0] = m0, row[1] = m1, row[2] = m2, row[3] = m3;
      row[4] = 0.0, row[5] = 0.0, row[6] = bad, row[7] = 0.0;
    }
  }
}

// Rows of a strip whose cells are all solid: everything keeps its value, the
// old iterate's (the two state buffers need not agree there: a caller may
// have written to one of them).  Lane l takes the column x0 + l, four rows are
// loaded before the first is stored.  RS: the mass fluxes, as in the passes.
template <bool RS>
__device__ __forceinline__ void carry(const KArgs ka, int x0, int w, int y0, int y1, double *row) {
  KParams &P = ka->P;
  const int lane = threadIdx.x & 63;
  const bool own = lane < w;
  const int nx = P.nx, ny = P.ny, gi = x0 + (own ? lane : 0);
  const long pitch = P.pitch, fld = ka->field;
  const double *const o = ka->o + P.off;
  double *const n = ka->n + P.off;
  const bool copy = P.per && gi == 0;  // (no solid cell lies at an outlet)
  constexpr int AHEAD = 4;
  double bad = 0.0;
  for (int y = y0; y < y1; y += AHEAD) {
    double q[AHEAD][4];
#pragma unroll
    for (int a = 0; a < AHEAD; a++)
#pragma unroll
      for (int f = 0; f < 4; f++) q[a][f] = o[f * fld + min(y + a, y1 - 1) * pitch + gi];
#pragma unroll
    for (int a = 0; a < AHEAD; a++) {
      const int j = y + a;
      if (j >= y1 || !own) continue;
#pragma unroll
      for (int f = 0; f < 4; f++) n[f * fld + j * pitch + gi] = q[a][f];
      if (copy) n[j * pitch + nx] = q[a][0];
      if constexpr (RS) {
        const int gw = P.per ? wrapi(gi - 1, nx) : gi - 1;
        auto rho = [&](int i, int jj) { return ddiv(o[2 * fld + jj * pitch + i], o[3 * fld + jj * pitch + i]); };
        const double u = q[a][0], v = q[a][1], r = ddiv(q[a][2], q[a][3]);
        const double dx = P.gx6[6 * (gi + XPAD)], dy = P.gy6[6 * (j + XPAD)];
        const double fu = upw(rho(gw, j), r, u) * u * dy;
        double *const gu = ka->X.gu + P.off, *const gv = ka->X.gv + P.off;
        gu[j * pitch + gi] = fu;
        if (copy) gu[j * pitch + nx] = fu;
        gv[j * pitch + gi] = (j == 0 ? r : upw(rho(gi, j - 1), r, v)) * v * dx;
        if (j == ny - 1) gv[ny * pitch + gi] = r * o[fld + ny * pitch + gi] * dx;
        bad += (double)(!isfinite(u)) + (double)(!isfinite(v));
      }
    }
  }
  if constexpr (RS) {
    bad = wave_sum(bad);
    if (lane == 0)
      for (int k = 0; k < NRES; k++) row[k] = k == 6 ? bad : 0.0;
  }
}
#undef Q_TP
#undef Q_gP
#undef Q_gW
#undef Q_gN
#undef Q_rP
#undef Q_rW
#undef Q_gs
#undef Q_rS
#undef Q_u00
#undef Q_uE
#undef Q_uW
#undef Q_uN0
#undef Q_uNE
#undef Q_uS0
#undef Q_uSE
#undef Q_v00
#undef Q_vN0
#undef Q_vW0
#undef Q_vNW
#undef Q_vS0
#undef Q_vE0
#undef SECTION
