// Three-dimensional SIMPLE-TS step: kernels and the C ABI of include/sts3.h.
//
// The explicit schemes run a pass as two kernels that march in z over tiles of
// columns, with the current planes in LDS and registers (k3_sweep_eqs,
// k3_sweep_pv).  The implicit schemes, whose coefficients take the fluxes of
// many more neighbours, run it as a chain of streaming stencil kernels, one
// thread per unknown, each reading its neighbours through the L1/L2 caches:
//   Gamma on the cell edges along each direction      (k3_edge<c>)
//   energy equation (pl30-pl33, pl28, pl29), and the pseudo velocities and
//   d of each component (pl14-pl16, pl18-pl21 read for any component a),
//   all from the old iterate                          (k3_eqs)
//   pressure equation (pl23, pl24), six neighbours, and rho = p/T,
//   Gamma = sqrt(T) of the new iterate               (k3_pressure)
//   velocity update (pl18, pl19) and the new iterate's face densities
//   (pl10-pl11 read per direction)                   (k3_velocity<a>)
// The step prologue computes rho, Gamma and the face densities of the state
// (k3_cell, k3_rf) and stores the per-step constants (the level n-1 parts of
// b^u, b^v, b^w, b^T, b^p and, for the explicit schemes, the explicit
// convective terms pl15_11 / pl31_1: k3_const).  After the last pass k3_resid
// reduces the increments and the continuity residual in fixed-order block
// partials.  Host arrays are scattered and gathered by k3_impose and k3_pack.
//
// Every field array holds (nz+1+2G) x (ny+1+2G) rows of a pitch of at least
// nx+1+2G doubles (x fastest): one index serves cells and the faces of every
// direction, and G = 2 ghost layers around the domain let every neighbour of
// a stencil be loaded at a constant offset.  In a periodic direction the
// kernels of the prologue and of the implicit chain that write an array read
// by a stencil also write the periodic images of the entries within G of
// either end (face n is the image of face 0); the sweeps read the other end
// instead, and k3_images writes the images of their last state once per step.
// The step constants have none: nothing reads them beside their own cell or
// face.  Elsewhere the ghost entries hold finite values that no equation uses.
#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/sts3.h"
#include "sts_internal.h"

namespace sts3 {
namespace {

constexpr int BX = 64, BY = 4, NTB = BX * BY;  // 256 threads per block
constexpr int NR = 8;                           // residual partials per block
constexpr int G = 2;                            // ghost layers

struct P3 {
  int n[3];
  int per[3];
  int io;  // inlet / outlet in x
  int wt[3][2];
  double wv[3][2][3];
  double wT[3][2], sqwT[3][2];
  double A, B, C1, C2, C3, g[3];
  double u_in, T_in, p_in, rho_in, sqT_in;
  double dt, idt;
  long sy, sz, off;  // strides; index of (0, 0, 0)
  // per direction, index 0 = the first cell or face (G ghost entries before):
  // widths d, their inverses id; at face i (between cells i-1 and i) the
  // weights of cells i-1 and i in the linear interpolation to the face,
  // wlo = d_i / (d_{i-1} + d_i) and whi = d_{i-1} / (d_{i-1} + d_i), and the
  // inverse centre distance ic = 2 / (d_{i-1} + d_i); interleaved, five
  // values per index (one pointer per direction keeps the kernels' uniform
  // values within the scalar register file)
  const double *geo[3];
};
constexpr int NGEO = 5;  // d, 1/d, wlo, whi, ic

struct Fld {
  double *q[5];  // u, v, w, p, T
};

struct Work {
  double *rho, *gam;
  double *rf[3];            // face densities
  double *qh[3], *dq[3];    // pseudo velocities and d
  double *cq[3], *cT, *cp;  // per-step constants
  double *ge[3];            // Gamma on the cell edges along each direction
};

// ---------------------------------------------------------------------------
// indexing
// ---------------------------------------------------------------------------
__device__ __forceinline__ long lin(const P3 &P, int i, int j, int k) {
  return P.off + (long)k * P.sz + (long)j * P.sy + i;
}
__device__ __forceinline__ long stride(const P3 &P, int e) {
  return e == 0 ? 1 : (e == 1 ? P.sy : P.sz);
}
// value of an array at x (+ s along e); x may lie up to G outside the domain
__device__ __forceinline__ double cv(const P3 &P, const double *a, const int x[3], int e = 0,
                                     int s = 0) {
  return a[lin(P, x[0], x[1], x[2]) + s * stride(P, e)];
}
__device__ __forceinline__ double fv(const P3 &P, const double *a, int f, const int x[3],
                                     int e = 0, int s = 0) {
  (void)f;
  return cv(P, a, x, e, s);
}
__device__ __forceinline__ double W(const P3 &P, int e, int i) { return P.geo[e][NGEO * i]; }
__device__ __forceinline__ double IW(const P3 &P, int e, int i) { return P.geo[e][NGEO * i + 1]; }
__device__ __forceinline__ double WLO(const P3 &P, int e, int i) { return P.geo[e][NGEO * i + 2]; }
__device__ __forceinline__ double WHI(const P3 &P, int e, int i) { return P.geo[e][NGEO * i + 3]; }
__device__ __forceinline__ double IC(const P3 &P, int e, int i) { return P.geo[e][NGEO * i + 4]; }
// store v at x and, in periodic directions, at the images of x within the
// ghost layers (FM: bit e set where the array's index along e is a face
// index, 0 for a cell array)
template <int FM>
__device__ void put(const P3 &P, double *a, const int x[3], double v) {
  const long m = lin(P, x[0], x[1], x[2]);
  a[m] = v;
  int o[3][3], no[3];
#pragma unroll
  for (int e = 0; e < 3; e++) {
    no[e] = 1;
    o[e][0] = 0;
    if (P.per[e]) {
      if (x[e] <= (((FM >> e) & 1) ? G : G - 1)) o[e][no[e]++] = P.n[e];
      if (x[e] >= P.n[e] - G) o[e][no[e]++] = -P.n[e];
    }
  }
  if (no[0] + no[1] + no[2] == 3) return;
  for (int a0 = 0; a0 < no[0]; a0++)
    for (int a1 = 0; a1 < no[1]; a1++)
      for (int a2 = 0; a2 < no[2]; a2++)
        if (a0 | a1 | a2) a[m + o[0][a0] + (long)o[1][a1] * P.sy + (long)o[2][a2] * P.sz] = v;
}
__device__ __forceinline__ bool has_cell(const P3 &P, int e, int i) {
  return P.per[e] || (i >= 0 && i < P.n[e]);
}
__device__ __forceinline__ bool has_face(const P3 &P, int e, int i) {
  return P.per[e] || (i >= 0 && i <= P.n[e]);
}
// side s (0 low, 1 high) of cell index xe along e: 0 interior, 1 wall,
// 2 inlet, 3 outlet
__device__ __forceinline__ int side(const P3 &P, int e, int xe, int s) {
  if (P.per[e]) return 0;
  if (s == 0 && xe == 0) return (e == 0 && P.io) ? 2 : 1;
  if (s == 1 && xe == P.n[e] - 1) return (e == 0 && P.io) ? 3 : 1;
  return 0;
}
__device__ __forceinline__ bool solved(const P3 &P, int a, int fa) {
  return P.per[a] ? fa < P.n[a] : (fa > 0 && fa < P.n[a]);
}
// area of the e-faces of cell x
__device__ __forceinline__ double area(const P3 &P, int e, const int x[3]) {
  const int b = e == 0 ? 1 : 0, t = e == 2 ? 1 : 2;
  return W(P, b, x[b]) * W(P, t, x[t]);
}

// ---------------------------------------------------------------------------
// elementary functions (Sec. 3.2)
// ---------------------------------------------------------------------------
__device__ __forceinline__ double upw(double f1, double f2, double vel) {
  return vel > 0.0 ? f1 : f2;
}
// a / b as a reciprocal refined by Newton steps and a residual correction
// (within one ulp of the IEEE quotient), and 1 / b
__device__ __forceinline__ double ddiv(double a, double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = __builtin_fma(__builtin_fma(-b, r, 1.0), r, r);
  const double q = a * r;
  return __builtin_fma(__builtin_fma(-b, q, a), r, q);
}
__device__ __forceinline__ double drcp(double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = __builtin_fma(__builtin_fma(-b, r, 1.0), r, r);
  return __builtin_fma(__builtin_fma(-b, r, 1.0), r, r);
}
// van Leer psi(r) = (r + |r|) / (1 + |r|) of r = a/b, written as 2a / (a + b)
// where a and b have one sign (0 otherwise)
__device__ __forceinline__ double vanleer(double a, double b) {
  const bool same = (a > 0.0 && b > 0.0) || (a < 0.0 && b < 0.0);
  const double q = ddiv(2.0 * a, a + b);
  return same ? q : 0.0;
}
// psi_s of the face i along e between nodes 2 and 3 (cells i-1 and i), with
// the stencil widths d1..d4 and the face's weights d2/(d2+d3), d3/(d2+d3)
__device__ __forceinline__ double psi_s(const P3 &P, int e, int i, double f1, double f2, double f3,
                                        double f4, double vel) {
  const double d1 = W(P, e, i - 2), d2 = W(P, e, i - 1), d3 = W(P, e, i), d4 = W(P, e, i + 1);
  if (vel > 0.0) return WHI(P, e, i) * vanleer((d2 + d3) * (f2 - f1), (d1 + d2) * (f3 - f2));
  return -WLO(P, e, i) * vanleer((d2 + d3) * (f4 - f3), (d3 + d4) * (f3 - f2));
}
__device__ __forceinline__ double psi_c(double f1, double f2, double f3, double f4, double d1,
                                        double d2, double d3, double vel) {
  if (vel > 0.0) return 0.5 * vanleer(d2 * (f2 - f1), d1 * (f3 - f2));
  return -0.5 * vanleer(d2 * (f4 - f3), d3 * (f3 - f2));
}
__device__ __forceinline__ double hmean(double dl, double gl, double dr, double gr) {
  return ddiv((dl + dr) * gl * gr, dl * gr + dr * gl);
}
__device__ __forceinline__ double hmean2(double a, double b) { return ddiv(2.0 * a * b, a + b); }

// thread -> point of an index space of extent (X, Y, Z): one block per
// BX x BY tile of an x-y plane, blockIdx.z the plane.  (Dealing each XCD a
// contiguous slab of planes, as the 2-D pass deals tile bands, was measured
// and made no kernel faster: these kernels are bound by their per-thread
// load chains, not by L2 misses.)
// A wave covers one row of its tile (BX = 64 lanes), so y and z are uniform
// across it: taken from the first lane, they live in scalar registers, and
// the widths, weights and boundary tests along y and z become scalar loads
// and scalar branches.
static_assert(BX == 64, "one tile row per wave");
__device__ __forceinline__ bool point(int X, int Y, int Z, int x[3]) {
  x[0] = blockIdx.x * BX + threadIdx.x;
  x[1] = __builtin_amdgcn_readfirstlane((int)(blockIdx.y * BY + threadIdx.y));
  x[2] = blockIdx.z;
  return x[0] < X && x[1] < Y && x[2] < Z;
}

// ---------------------------------------------------------------------------
// cell properties and face densities
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(NTB) void k3_cell(P3 P, Fld S, Work Wk) {
  int x[3];
  if (!point(P.n[0], P.n[1], P.n[2], x)) return;
  const long m = lin(P, x[0], x[1], x[2]);
  const double p = S.q[3][m], T = S.q[4][m];
  put<0>(P, Wk.rho, x, ddiv(p, T));
  put<0>(P, Wk.gam, x, sqrt(T));
}

// face density of the A-face f with velocity vel there, from rho in Wk
template <int A, bool TV>
__device__ __forceinline__ double rf_at(const P3 &P, const Work &Wk, const int f[3], double vel) {
  const int fa = f[A];
  double r;
  if (!P.per[A] && fa == 0) {
    const double rr = cv(P, Wk.rho, f);
    r = (A == 0 && P.io) ? upw(P.rho_in, rr, vel) : rr;
  } else if (!P.per[A] && fa == P.n[A]) {
    r = cv(P, Wk.rho, f, A, -1);
  } else {
    const double rl = cv(P, Wk.rho, f, A, -1), rr = cv(P, Wk.rho, f);
    r = upw(rl, rr, vel);
    if (TV && has_cell(P, A, fa - 2) && has_cell(P, A, fa + 1))
      r += psi_s(P, A, fa, cv(P, Wk.rho, f, A, -2), rl, rr, cv(P, Wk.rho, f, A, 1), vel) *
           (rr - rl);
  }
  return r;
}

// The low faces of a cell in all three directions, and the high one of the
// last cell of a direction that is not periodic: one launch instead of three
// (the directions share rho): 0.12 ms on 512x128x128, TVD 0.20.
template <int A, bool TV>
__device__ __forceinline__ void rf_face(const P3 &P, const Fld &S, const Work &Wk, const int f[3]) {
  put<1 << A>(P, Wk.rf[A], f, rf_at<A, TV>(P, Wk, f, S.q[A][lin(P, f[0], f[1], f[2])]));
}
template <int A, bool TV>
__device__ __forceinline__ void rf_faces(const P3 &P, const Fld &S, const Work &Wk, const int x[3]) {
  rf_face<A, TV>(P, S, Wk, x);
  if (P.per[A] || x[A] != P.n[A] - 1) return;
  int f[3] = {x[0], x[1], x[2]};
  f[A]++;
  rf_face<A, TV>(P, S, Wk, f);
}
template <bool TV>
__global__ __launch_bounds__(NTB) void k3_rf(P3 P, Fld S, Work Wk) {
  int x[3];
  if (!point(P.n[0], P.n[1], P.n[2], x)) return;
  rf_faces<0, TV>(P, S, Wk, x);
  rf_faces<1, TV>(P, S, Wk, x);
  rf_faces<2, TV>(P, S, Wk, x);
}

// mass flux through the e-face of cell x on side s (0 low, 1 high)
__device__ __forceinline__ double flux(const P3 &P, const Fld &S, const Work &Wk, int e,
                                       const int x[3], int s) {
  int y[3] = {x[0], x[1], x[2]};
  y[e] += s;
  return fv(P, Wk.rf[e], e, y) * fv(P, S.q[e], e, y) * area(P, e, x);
}

// ---------------------------------------------------------------------------
// energy equation
// ---------------------------------------------------------------------------
// T of the neighbour of cell x across side s of direction e, as the
// convective terms take it (inlet T_in, wall and outlet the cell's own)
__device__ __forceinline__ double T_nb(const P3 &P, const double *T, int e, const int x[3],
                                       int s, double TP) {
  const int k = side(P, e, x[e], s);
  if (k == 2) return P.T_in;
  if (k) return TP;
  return cv(P, T, x, e, s ? 1 : -1);
}

// explicit convective term of T (pl31_1) at level n-1 (S, rho, rf of n-1)
template <bool TV>
__device__ double T_explicit(const P3 &P, const Fld &S, const Work &Wk, const int x[3]) {
  const double *T = S.q[4];
  const double TP = cv(P, T, x);
  double sum = 0.0;
#pragma unroll
  for (int e = 0; e < 3; e++) {
    const double TL = T_nb(P, T, e, x, 0, TP), TH = T_nb(P, T, e, x, 1, TP);
    int yh[3] = {x[0], x[1], x[2]};
    yh[e] += 1;
    const double vl = fv(P, S.q[e], e, x), vh = fv(P, S.q[e], e, yh);
    const double Fl = flux(P, S, Wk, e, x, 0), Fh = flux(P, S, Wk, e, x, 1);
    double pl = 0.0, ph = 0.0;
    if (TV) {
      const int xe = x[e];
      if (has_cell(P, e, xe - 1) && has_cell(P, e, xe + 2))
        ph = psi_s(P, e, xe + 1, cv(P, T, x, e, -1), TP, TH, cv(P, T, x, e, 2), vh);
      if (has_cell(P, e, xe - 2) && has_cell(P, e, xe + 1))
        pl = psi_s(P, e, xe, cv(P, T, x, e, -2), TL, TP, TH, vl);
    }
    sum += -Fh * (upw(TP, TH, vh) + (TH - TP) * ph) + Fl * (upw(TL, TP, vl) + (TP - TL) * pl);
  }
  return sum;
}

// cell-centre value of component e in cell x (+ s along f)
__device__ __forceinline__ double qcell(const P3 &P, const Fld &S, int e, const int x[3], int f,
                                        int s) {
  int y[3] = {x[0], x[1], x[2]};
  y[f] += s;
  int z[3] = {y[0], y[1], y[2]};
  z[e] += 1;
  return 0.5 * (fv(P, S.q[e], e, y) + fv(P, S.q[e], e, z));
}
// component e at the centre of the f-face on side s of cell x: bilinear in
// the nearest nodes; the wall's velocity (no slip) or the cell's (slip) on a
// wall, 0 (tangential) at the inlet, the cell's at the outlet
__device__ double qface(const P3 &P, const Fld &S, int e, int f, const int x[3], int s) {
  const double qc = qcell(P, S, e, x, f, 0);
  const int k = side(P, f, x[f], s);
  if (k == 1) return P.wt[f][s] == STS3_NOSLIP ? P.wv[f][s][e] : qc;
  if (k == 2) return 0.0;
  if (k == 3) return qc;
  const double qn = qcell(P, S, e, x, f, s ? 1 : -1);
  return s ? WLO(P, f, x[f] + 1) * qc + WHI(P, f, x[f] + 1) * qn
           : WHI(P, f, x[f]) * qc + WLO(P, f, x[f]) * qn;
}

// new T of cell x (pl28-pl33)
template <bool TV>
__device__ __forceinline__ void energy_at(const P3 &P, const Fld &S, const Work &Wk,
                                          double *Tout, const int x[3]) {
  const double *T = S.q[4];
  const double TP = cv(P, T, x), gP = cv(P, Wk.gam, x), rP = cv(P, Wk.rho, x);
  const double dV = W(P, 0, x[0]) * W(P, 1, x[1]) * W(P, 2, x[2]);
  double sa = 0.0, sn = 0.0, sF = 0.0;
#pragma unroll
  for (int e = 0; e < 3; e++) {
    const double ar = area(P, e, x), de = W(P, e, x[e]);
#pragma unroll
    for (int s = 0; s < 2; s++) {
      const int k = side(P, e, x[e], s);
      double D, nb;
      if (k == 1) {
        if (P.wt[e][s] == STS3_NOSLIP) {
          nb = P.wT[e][s];
          D = P.C1 * hmean2(gP, P.sqwT[e][s]) * ar * 2.0 * IW(P, e, x[e]);
        } else {
          nb = TP;
          D = 0.0;
        }
      } else if (k == 2) {
        nb = P.T_in;
        D = P.C1 * hmean2(gP, P.sqT_in) * ar * 2.0 * IW(P, e, x[e]);
      } else if (k == 3) {
        nb = TP;
        D = 0.0;
      } else {
        const int sg = s ? 1 : -1;
        const double dn = W(P, e, x[e] + sg), gn = cv(P, Wk.gam, x, e, sg);
        nb = cv(P, T, x, e, sg);
        D = P.C1 * (s ? hmean(de, gP, dn, gn) : hmean(dn, gn, de, gP)) * ar * IC(P, e, x[e] + s);
      }
      const double Fv = flux(P, S, Wk, e, x, s);
      double psi = 0.0;
      if (TV) {
        int yf[3] = {x[0], x[1], x[2]};
        yf[e] += s;
        const double vel = fv(P, S.q[e], e, yf);
        const int xe = x[e];
        if (s == 0 && has_cell(P, e, xe - 2) && has_cell(P, e, xe + 1))
          psi = psi_s(P, e, xe, cv(P, T, x, e, -2), cv(P, T, x, e, -1), TP, cv(P, T, x, e, 1), vel);
        if (s == 1 && has_cell(P, e, xe - 1) && has_cell(P, e, xe + 2))
          psi = psi_s(P, e, xe + 1, cv(P, T, x, e, -1), TP, cv(P, T, x, e, 1), cv(P, T, x, e, 2),
                      vel);
      }
      const double a = (s ? fmax(0.0, -Fv) : fmax(0.0, Fv)) - Fv * psi + D;
      sF += s ? Fv : -Fv;
      sa += a;
      sn += a * nb;
    }
  }
  const double a0 = P.dt * (sa + sF) + rP * dV;
  // dissipation (strain rates from the face values) and pressure work
  double dd[3], div = 0.0;
#pragma unroll
  for (int e = 0; e < 3; e++) {
    dd[e] = (fv(P, S.q[e], e, x, e, 1) - fv(P, S.q[e], e, x)) * IW(P, e, x[e]);
    div += dd[e];
  }
  double phi = 2.0 * (dd[0] * dd[0] + dd[1] * dd[1] + dd[2] * dd[2]);
#pragma unroll
  for (int e = 0; e < 3; e++)
#pragma unroll
    for (int f = e + 1; f < 3; f++) {
      const double sef = (qface(P, S, e, f, x, 1) - qface(P, S, e, f, x, 0)) * IW(P, f, x[f]) +
                         (qface(P, S, f, e, x, 1) - qface(P, S, f, e, x, 0)) * IW(P, e, x[e]);
      phi += sef * sef;
    }
  phi -= 2.0 / 3.0 * div * div;
  const double src = P.C2 * gP * phi * dV + P.C3 * cv(P, S.q[3], x) * div * dV;
  const long m = lin(P, x[0], x[1], x[2]);
  put<0>(P, Tout, x, ddiv(P.dt * (sn + src) + Wk.cT[m], a0));
}

// ---------------------------------------------------------------------------
// momentum of component A
// ---------------------------------------------------------------------------
// Gamma on the edge of the A-momentum volume at face f towards side s of
// direction b (the edge runs along the third direction): bilinear in the
// four cells around it; 0 on a wall (it multiplies wall-normal velocities
// only), sqrt(T_in) at the inlet, the last cells along A at the outlet
template <int A>
__device__ __forceinline__ double gam_edge(const P3 &P, const Work &Wk, int b, const int f[3],
                                           int s) {
  return cv(P, Wk.ge[3 - A - b], f, b, s);
}

// Gamma on the edges along direction C (k3_edge): at the a-face and b-face
// positions of the edge ({a, b} the two other directions) and cell index
// along C; bilinear in the four cells around it.  An edge on one boundary:
// 0 on a wall (it multiplies wall-normal velocities only), sqrt(T_in) at the
// inlet, at the outlet the last cells interpolated along the other
// direction; an edge on two boundaries is never used (0).
template <int C>
__global__ __launch_bounds__(NTB) void k3_edge(P3 P, Work Wk) {
  constexpr int a = C == 0 ? 1 : 0, b = C == 2 ? 1 : 2;
  int x[3];
  if (!point(P.n[0] + (C != 0), P.n[1] + (C != 1), P.n[2] + (C != 2), x)) return;
  if ((P.per[a] && x[a] == P.n[a]) || (P.per[b] && x[b] == P.n[b])) return;  // images
  const bool ba = !P.per[a] && (x[a] == 0 || x[a] == P.n[a]);
  const bool bb = !P.per[b] && (x[b] == 0 || x[b] == P.n[b]);
  double g = 0.0;
  if (ba != bb) {
    const int d = ba ? a : b, o = ba ? b : a;
    if (d == 0 && P.io) {
      if (x[d] == 0) {
        g = P.sqT_in;
      } else {
        int l[3] = {x[0], x[1], x[2]}, r[3] = {x[0], x[1], x[2]};
        l[d] = r[d] = P.n[d] - 1;
        l[o] -= 1;
        g = WLO(P, o, x[o]) * cv(P, Wk.gam, l) + WHI(P, o, x[o]) * cv(P, Wk.gam, r);
      }
    }
  } else if (!ba) {
#pragma unroll
    for (int ia = 0; ia < 2; ia++)
#pragma unroll
      for (int ib = 0; ib < 2; ib++) {
        int y[3] = {x[0], x[1], x[2]};
        y[a] = x[a] - 1 + ia;
        y[b] = x[b] - 1 + ib;
        const double wa = ia ? WHI(P, a, x[a]) : WLO(P, a, x[a]);
        const double wb = ib ? WHI(P, b, x[b]) : WLO(P, b, x[b]);
        g += wa * wb * cv(P, Wk.gam, y);
      }
  }
  put<(1 << a) | (1 << b)>(P, Wk.ge[C], x, g);
}

// neighbour of component A at face f across side s (-1, +1) of direction b
template <int A>
__device__ __forceinline__ double q_nb(const P3 &P, const double *q, int b, const int f[3],
                                       int s, double qP) {
  if (b == A) return fv(P, q, A, f, A, s);
  const int k = side(P, b, f[b], s > 0);
  if (k == 1) return P.wt[b][s > 0] == STS3_NOSLIP ? P.wv[b][s > 0][A] : qP;
  if (k == 2) return 0.0;
  if (k == 3) return qP;
  return fv(P, q, A, f, b, s);
}

// explicit convective term of component A (pl15_11) at level n-1
template <int A, bool TV>
__device__ double q_explicit(const P3 &P, const Fld &S, const Work &Wk, const int f[3]) {
  const double *q = S.q[A];
  const double qP = fv(P, q, A, f);
  int l[3] = {f[0], f[1], f[2]};
  l[A] -= 1;
  double sum = 0.0;
#pragma unroll
  for (int b = 0; b < 3; b++) {
    const double qL = q_nb<A>(P, q, b, f, -1, qP), qH = q_nb<A>(P, q, b, f, 1, qP);
    if (b == A) {
      const double Ap = area(P, A, f);
      const double ubH = 0.5 * (qP + qH), ubL = 0.5 * (qL + qP);
      const double FbH = cv(P, Wk.rho, f) * ubH * Ap, FbL = cv(P, Wk.rho, l) * ubL * Ap;
      double pH = 0.0, pL = 0.0;
      if (TV) {
        const int fa = f[A];
        if (has_face(P, A, fa - 1) && has_face(P, A, fa + 2))
          pH = psi_c(qL, qP, qH, fv(P, q, A, f, A, 2), W(P, A, fa - 1), W(P, A, fa),
                     W(P, A, fa + 1), ubH);
        if (has_face(P, A, fa - 2) && has_face(P, A, fa + 1))
          pL = psi_c(fv(P, q, A, f, A, -2), qL, qP, qH, W(P, A, fa - 2), W(P, A, fa - 1),
                     W(P, A, fa), ubL);
      }
      sum += -FbH * (upw(qP, qH, ubH) + (qH - qP) * pH) + FbL * (upw(qL, qP, ubL) + (qP - qL) * pL);
    } else {
      const int fb = f[b];
      double pl = 0.0, ph = 0.0;
      const bool okh = TV && has_cell(P, b, fb - 1) && has_cell(P, b, fb + 2);
      const bool okl = TV && has_cell(P, b, fb - 2) && has_cell(P, b, fb + 1);
      const double q1h = okh ? fv(P, q, A, f, b, -1) : 0.0, q4h = okh ? fv(P, q, A, f, b, 2) : 0.0;
      const double q1l = okl ? fv(P, q, A, f, b, -2) : 0.0, q4l = okl ? fv(P, q, A, f, b, 1) : 0.0;
#pragma unroll
      for (int sd = 0; sd < 2; sd++) {
        const int *cx = sd ? f : l;
        int bh[3] = {cx[0], cx[1], cx[2]};
        bh[b] += 1;
        const double vl = fv(P, S.q[b], b, cx), vh = fv(P, S.q[b], b, bh);
        const double Fl = flux(P, S, Wk, b, cx, 0), Fh = flux(P, S, Wk, b, cx, 1);
        if (okh)
          ph = psi_s(P, b, fb + 1, q1h, qP, qH, q4h, vh);
        if (okl)
          pl = psi_s(P, b, fb, q1l, qL, qP, q4l, vl);
        sum += 0.5 * (-Fh * (upw(qP, qH, vh) + (qH - qP) * ph) +
                      Fl * (upw(qL, qP, vl) + (qP - qL) * pl));
      }
    }
  }
  return sum;
}

// pseudo velocity and d of component A at its face f (pl14-pl16, pl18-pl21)
template <int A, bool TV>
__device__ __forceinline__ void mom_at(const P3 &P, const Fld &S, const Work &Wk, const int f[3]) {
  if (P.per[A] && f[A] == P.n[A]) return;  // the image of face 0
  const long m = lin(P, f[0], f[1], f[2]);
  const double *q = S.q[A];
  const double qP = q[m];
  if (!solved(P, A, f[A])) {
    put<1 << A>(P, Wk.qh[A], f, qP);
    put<1 << A>(P, Wk.dq[A], f, 0.0);
    return;
  }
  int l[3] = {f[0], f[1], f[2]};
  l[A] -= 1;
  const double dal = W(P, A, f[A] - 1), dar = W(P, A, f[A]);
  const double rl = cv(P, Wk.rho, l), rr = cv(P, Wk.rho, f);
  const double gl = cv(P, Wk.gam, l), gr = cv(P, Wk.gam, f);
  const double Ap = area(P, A, f), len = 0.5 * (dal + dar);
  const double M = (rr * dar + rl * dal) * Ap / 2.0;
  const double gnode = WLO(P, A, f[A]) * gl + WHI(P, A, f[A]) * gr;
  double sa = 0.0, sn = 0.0, conv = 0.0, X = 0.0;
#pragma unroll
  for (int b = 0; b < 3; b++) {
    const double qL = q_nb<A>(P, q, b, f, -1, qP), qH = q_nb<A>(P, q, b, f, 1, qP);
    double aL, aH;
    if (b == A) {
      const double DL = P.B * gl * Ap * IW(P, A, f[A] - 1), DH = P.B * gr * Ap * IW(P, A, f[A]);
      const double ubL = 0.5 * (qL + qP), ubH = 0.5 * (qP + qH);
      const double FbL = rl * ubL * Ap, FbH = rr * ubH * Ap;
      double pL = 0.0, pH = 0.0;
      if (TV) {
        const int fa = f[A];
        if (has_face(P, A, fa - 2) && has_face(P, A, fa + 1))
          pL = psi_c(fv(P, q, A, f, A, -2), qL, qP, qH, W(P, A, fa - 2), dal, dar, ubL);
        if (has_face(P, A, fa - 1) && has_face(P, A, fa + 2))
          pH = psi_c(qL, qP, qH, fv(P, q, A, f, A, 2), dal, dar, W(P, A, fa + 1), ubH);
      }
      const double cl = fmax(0.0, FbL) - FbL * pL;
      const double ch = fmax(0.0, -FbH) - FbH * pH;
      conv += FbH - FbL;
      aL = cl + 4.0 / 3.0 * DL;
      aH = ch + 4.0 / 3.0 * DH;
    } else {
      const int t = 3 - A - b;
      const double d3 = W(P, t, f[t]);
      double D[2];
#pragma unroll
      for (int s = 0; s < 2; s++) {
        const int k = side(P, b, f[b], s);
        if (k == 1)
          D[s] = P.wt[b][s] == STS3_NOSLIP
                     ? P.B * (gnode + P.sqwT[b][s]) * len * d3 * IW(P, b, f[b])
                     : 0.0;
        else if (k == 2)
          D[s] = P.B * (gnode + gam_edge<A>(P, Wk, b, f, 0)) * len * d3 * IW(P, b, f[b]);
        else if (k == 3)
          D[s] = 0.0;
        else
          D[s] = P.B * gam_edge<A>(P, Wk, b, f, s) * len * d3 * IC(P, b, f[b] + s);
      }
      double cl = 0.0, ch = 0.0;
      const int fb = f[b];
      const bool okl = TV && has_cell(P, b, fb - 2) && has_cell(P, b, fb + 1);
      const bool okh = TV && has_cell(P, b, fb - 1) && has_cell(P, b, fb + 2);
#pragma unroll
      for (int sd = 0; sd < 2; sd++) {
        const int *cx = sd ? f : l;
        int bh[3] = {cx[0], cx[1], cx[2]};
        bh[b] += 1;
        const double vl = fv(P, S.q[b], b, cx), vh = fv(P, S.q[b], b, bh);
        const double Fl = flux(P, S, Wk, b, cx, 0), Fh = flux(P, S, Wk, b, cx, 1);
        double pl = 0.0, ph = 0.0;
        if (okl)
          pl = psi_s(P, b, fb, fv(P, q, A, f, b, -2), qL, qP, fv(P, q, A, f, b, 1), vl);
        if (okh)
          ph = psi_s(P, b, fb + 1, fv(P, q, A, f, b, -1), qP, qH, fv(P, q, A, f, b, 2), vh);
        cl += 0.5 * (fmax(0.0, Fl) - Fl * pl);
        ch += 0.5 * (fmax(0.0, -Fh) - Fh * ph);
        conv += 0.5 * (Fh - Fl);
      }
      aL = cl + D[0];
      aH = ch + D[1];
      // cross-diffusion for the tangential direction b
      int rh[3] = {f[0], f[1], f[2]}, lh[3] = {l[0], l[1], l[2]};
      rh[b] += 1;
      lh[b] += 1;
      const double *qb = S.q[b];
      const double b_rl = fv(P, qb, b, f), b_rh = fv(P, qb, b, rh);
      const double b_ll = fv(P, qb, b, l), b_lh = fv(P, qb, b, lh);
      X += (gam_edge<A>(P, Wk, b, f, 1) * (b_rh - b_lh) - gam_edge<A>(P, Wk, b, f, 0) * (b_rl - b_ll)) *
               d3 -
           2.0 / 3.0 * (gr * (b_rh - b_rl) - gl * (b_lh - b_ll)) * d3;
    }
    sa += aL + aH;
    sn += aL * qL + aH * qH;
  }
  const double a0 = sa + conv + M * P.idt;
  const double b = Wk.cq[A][m] + P.B * X;
  const double ia0 = drcp(a0);
  put<1 << A>(P, Wk.qh[A], f, (sn + b) * ia0);
  put<1 << A>(P, Wk.dq[A], f, P.A * Ap * ia0);
}

// The implicit schemes' equations that read only the old iterate, energy and
// the three momentum components, in one launch: the thread at index x takes
// the cell x and the low face of that cell in each direction (the threads
// one past the last cell along a direction take that direction's last faces
// only).  Their inputs overlap (velocities, face densities, rho, Gamma and
// the edge Gamma around x), so a block's neighbour loads are served by the
// caches of one launch instead of being fetched again by each.  (A grid
// banded by x per XCD halved the launch's L2 misses but not its time: the
// launch holds more uniform values than the scalar registers take, and its
// spill traffic through vector lanes grew with that layout.)
template <bool TV>
__global__ __launch_bounds__(NTB) void k3_eqs(P3 P, Fld S, Work Wk, double *Tout) {
  int x[3];
  if (!point(P.n[0] + 1, P.n[1] + 1, P.n[2] + 1, x)) return;
  const bool i0 = x[0] < P.n[0], i1 = x[1] < P.n[1], i2 = x[2] < P.n[2];
  if (i0 && i1 && i2) energy_at<TV>(P, S, Wk, Tout, x);
  if (i1 && i2) mom_at<0, TV>(P, S, Wk, x);
  if (i0 && i2) mom_at<1, TV>(P, S, Wk, x);
  if (i0 && i1) mom_at<2, TV>(P, S, Wk, x);
}

// ---------------------------------------------------------------------------
// pressure and velocities
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(NTB) void k3_pressure(P3 P, Fld S, Work Wk, const double *Tn,
                                                   double *pout) {
  int x[3];
  if (!point(P.n[0], P.n[1], P.n[2], x)) return;
  const long m = lin(P, x[0], x[1], x[2]);
  const double pP = S.q[3][m];
  const double dV = W(P, 0, x[0]) * W(P, 1, x[1]) * W(P, 2, x[2]);
  double sa = 0.0, sap = 0.0, sb = 0.0;
#pragma unroll
  for (int e = 0; e < 3; e++) {
    int xh[3] = {x[0], x[1], x[2]};
    xh[e] += 1;
    const double ar = area(P, e, x);
    const double rL = fv(P, Wk.rf[e], e, x), rH = fv(P, Wk.rf[e], e, xh);
    const double aL = rL * fv(P, Wk.dq[e], e, x) * ar, aH = rH * fv(P, Wk.dq[e], e, xh) * ar;
    const double bL = rL * fv(P, Wk.qh[e], e, x) * ar, bH = rH * fv(P, Wk.qh[e], e, xh) * ar;
    const double pL = side(P, e, x[e], 0) ? pP : cv(P, S.q[3], x, e, -1);
    const double pH = side(P, e, x[e], 1) ? pP : cv(P, S.q[3], x, e, 1);
    sa += aL + aH;
    sap += aL * pL + aH * pH;
    sb += bH - bL;
  }
  const double Tm = Tn[m];
  const double a0 = ddiv(dV, Tm) + sa * P.dt;
  const double pm = ddiv(sap * P.dt + (Wk.cp[m] - sb * P.dt), a0);
  put<0>(P, pout, x, pm);
  // rho and Gamma of the new iterate, which the next pass reads (nothing
  // later in this pass reads those of the old one)
  put<0>(P, Wk.rho, x, ddiv(pm, Tm));
  put<0>(P, Wk.gam, x, sqrt(Tm));
}

template <int A>
__device__ __forceinline__ double q_update(const P3 &P, const Work &Wk, const double *pn,
                                           const int f[3]) {
  return fv(P, Wk.qh[A], A, f) - fv(P, Wk.dq[A], A, f) * (cv(P, pn, f) - cv(P, pn, f, A, -1));
}

// new velocity of component A (pl18, pl19); RF: also the face density of the
// new iterate at the face (the next pass's, from the rho the pressure kernel
// stored), which replaces the old one (read by nothing later in this pass
// but the residuals of the last pass, which launches without RF)
template <int A, bool RF, bool TV>
__global__ __launch_bounds__(NTB) void k3_velocity(P3 P, Fld S, Work Wk, const double *pn,
                                                   double *qout) {
  int f[3];
  if (!point(P.n[0] + (A == 0), P.n[1] + (A == 1), P.n[2] + (A == 2), f)) return;
  const int fa = f[A];
  if (P.per[A] && fa == P.n[A]) return;  // the image of face 0
  const long m = lin(P, f[0], f[1], f[2]);
  double qn;
  if (solved(P, A, fa)) {
    qn = q_update<A>(P, Wk, pn, f);
  } else if (A == 0 && P.io && fa == P.n[0]) {  // outlet: zero gradient
    int g[3] = {f[0], f[1], f[2]};
    g[A] = fa - 1;
    qn = q_update<A>(P, Wk, pn, g);
  } else {
    qn = S.q[A][m];  // inlet u_in, wall faces 0
  }
  put<1 << A>(P, qout, f, qn);
  if (RF) put<1 << A>(P, Wk.rf[A], f, rf_at<A, TV>(P, Wk, f, qn));
}

// ---------------------------------------------------------------------------
// The explicit schemes' pass as two sweeps that march in z
// ---------------------------------------------------------------------------
// A block of MY waves takes MX x MY columns of cells and walks up z: a plane
// is loaded once (with a halo of two cells in x and y for rho, one for the
// rest), rho = p/T and Gamma = sqrt(T) are formed while it is staged in LDS,
// its x and y neighbours are read from there, and what the planes above need
// of it stays in registers.  So a pass reads each old field about once
// instead of gathering some 80 neighbour values per cell through the caches
// (479 B per cell across L2), and Gamma on the edges and the face densities
// need no launches of their own.  Three LDS planes in turn: the plane being
// written is never one that a wave may still read, so one barrier per plane
// is enough.  Two blocks share a CU (LDS: 62 KB each; 230 VGPRs).
// Measured (512x128x128, explicit upwind): k3_sweep_eqs 0.38 ms where the
// edge and equation launches took 1.04 ms, 9.7 instead of 27.4 VALU wave
// instructions per cell, 1.5 GB at 3.9 TB/s; k3_sweep_pv 0.33 ms where the
// pressure and velocity launches took 0.48 ms (a step of 10 passes 16.4 ->
// 8.3 ms).  Both are bound by memory: latency at two waves per SIMD in the
// first (the constants of a plane loaded where they are used, not a plane
// ahead, cost 0.11 ms), traffic in the second.
constexpr int MX = 64, MY = 4;
constexpr int MXH = MX + 4;
struct Plane3 {
  double u[MY + 2][MXH], v[MY + 2][MXH], w[MY + 2][MXH], T[MY + 2][MXH], g[MY + 2][MXH];
  double r[MY + 4][MXH];
};

// block -> tile: consecutive blocks go to the 8 XCDs in turn; every XCD takes
// one contiguous range of tiles, so that the halos are found in its L2
__device__ __forceinline__ int xcd_block(int b, int n) {
  const int k = b & 7, q = n >> 3, r = n & 7;
  return k * q + (k < r ? k : r) + (b >> 3);
}
// index x of a direction of n cells: the other end's where it is periodic
__device__ __forceinline__ int around(int x, int n, int per) {
  return per ? (x < 0 ? x + n : (x >= n ? x - n : x)) : x;
}
// an element of a plane: uniform base, 32-bit byte offset (a plane of 4 GiB
// would take the 29 arrays past the device memory)
__device__ __forceinline__ double ldp(const double *plane, unsigned at) {
  return *(const double *)((const char *)plane + at);
}
__device__ __forceinline__ void stp(double *plane, unsigned at, double v) {
  *(double *)((char *)plane + at) = v;
}
// psi_s from its widths and the face's weights
__device__ __forceinline__ double psi_w(double f1, double f2, double f3, double f4, double d1,
                                        double d2, double d3, double d4, double wlo, double whi,
                                        double vel) {
  const bool up = vel > 0.0;
  const double a = (d2 + d3) * (up ? f2 - f1 : f4 - f3);
  const double b = (up ? d1 + d2 : d3 + d4) * (f3 - f2);
  return (up ? whi : -wlo) * vanleer(a, b);
}

// the neighbours of the cell in its plane (s) and in the one above (sp)
#define N3_gW0 s.g[ry][cx - 1]
#define N3_gE0 s.g[ry][cx + 1]
#define N3_gS0 s.g[ry - 1][cx]
#define N3_gN0 s.g[ry + 1][cx]
#define N3_uE0 s.u[ry][cx + 1]
#define N3_uEp sp.u[ry][cx + 1]
#define N3_vN0 s.v[ry + 1][cx]
#define N3_vNp sp.v[ry + 1][cx]
#define N3_wW0 s.w[ry][cx - 1]
#define N3_wE0 s.w[ry][cx + 1]
#define N3_wS0 s.w[ry - 1][cx]
#define N3_wN0 s.w[ry + 1][cx]
#define N3_wWp sp.w[ry][cx - 1]
#define N3_wEp sp.w[ry][cx + 1]
#define N3_wSp sp.w[ry - 1][cx]
#define N3_wNp sp.w[ry + 1][cx]
#define N3_gSW s.g[ry - 1][cx - 1]
#define N3_gSE s.g[ry - 1][cx + 1]
#define N3_gNW s.g[ry + 1][cx - 1]
#define N3_uW s.u[ry][cx - 1]
#define N3_uS s.u[ry - 1][cx]
#define N3_uN s.u[ry + 1][cx]
#define N3_uSE s.u[ry - 1][cx + 1]
#define N3_uNE s.u[ry + 1][cx + 1]
#define N3_vS s.v[ry - 1][cx]
#define N3_vW s.v[ry][cx - 1]
#define N3_vE s.v[ry][cx + 1]
#define N3_vNW s.v[ry + 1][cx - 1]
#define N3_vNE s.v[ry + 1][cx + 1]
#define N3_rW s.r[ry + 1][cx - 1]
#define N3_rS s.r[ry][cx]
// Each equation reads its neighbours from LDS again: kept across equations
// they would not fit the registers
#define N3_SECTION(name)                     \
  const KArgs name = fresh(ka);              \
  __builtin_amdgcn_sched_barrier(0)

// The kernel's arguments, read through a pointer to their segment that
// N3_SECTION makes opaque: every equation loads the uniform values it uses
// again (scalar loads, scalar cache) instead of holding some 150 of them in
// scalar registers, which spilled into vector lanes (291 lane instructions)
struct Sweep {
  P3 P;
  Fld S;
  Work Wk;
  double *Tout;
  int tx, ty, seg;
};
typedef const __attribute__((address_space(4))) Sweep *KArgs;
typedef const __attribute__((address_space(4))) double *CDbl;
template <class T>
__device__ __forceinline__ T fresh(T a) {
  asm volatile("" : "+s"(a) : : "memory");
  return a;
}
// geometry of one direction around index i (uniform)
struct Geo3 {
  double wmm, wm, iwm, w, iw, wlo, whi, ic, wh, wloH, whiH, ich;
  __device__ __forceinline__ explicit Geo3(CDbl p) {
    wmm = p[-2 * NGEO], wm = p[-NGEO], iwm = p[1 - NGEO];
    w = p[0], iw = p[1], wlo = p[2], whi = p[3], ic = p[4];
    wh = p[NGEO], wloH = p[NGEO + 2], whiH = p[NGEO + 3], ich = p[NGEO + 4];
  }
};

// T, the pseudo velocities, d and the face densities of the old iterate S
// (pl30-pl33, pl28, pl29; pl14-pl16, pl18-pl21; pl10, pl11) on the low faces
// of every cell; the cells before a last boundary face also write that face.
template <bool TV>
__global__ __launch_bounds__(MX * MY) __attribute__((amdgpu_waves_per_eu(2, 2))) void k3_sweep_eqs(
    const Sweep A) {
  __shared__ Plane3 pl[3];
  const P3 &P = A.P;
  const int tx = A.tx, ty = A.ty, seg = A.seg;
  const KArgs ka = (KArgs)__builtin_amdgcn_kernarg_segment_ptr();
  const int b = xcd_block(blockIdx.x, gridDim.x);
  const int x0 = (b % tx) * MX, y0 = (b / tx % ty) * MY, z0 = (b / (tx * ty)) * seg;
  const int z1 = min(z0 + seg, P.n[2]);
  const int lane = threadIdx.x, wy = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
  const int n0 = P.n[0], n1 = P.n[1];
  const int i = x0 + lane, j = y0 + wy;
  // columns and rows past the second ghost layer are clamped (no cell of the
  // domain uses them); in a periodic direction the halo is read from the
  // other end, so no periodic images are written between the passes
  const unsigned sy = (unsigned)P.sy;
  auto offset = [&](int x, int y) {
    x = around(min(x, n0 + 1), n0, P.per[0]), y = around(min(y, n1 + 1), n1, P.per[1]);
    return 8u * ((unsigned)(y + G) * sy + (unsigned)(x + G));
  };
  auto plane = [&](int k) { return (long)(around(k, P.n[2], P.per[2]) + G) * P.sz; };
  const unsigned own = offset(i, j);
  // halo rows -2, -1, MY, MY + 1 (one per wave) and, in wave 0, the two halo
  // columns on both sides of the rows -1 .. MY
  const int hr = wy == 0 ? -2 : (wy == 1 ? -1 : (wy == 2 ? MY : MY + 1));
  const bool hfull = wy == 1 || wy == 2;  // the outer rows are needed for rho only
  const unsigned hoff = offset(i, y0 + hr);
  const int cr = lane >> 2, cq4 = lane & 3;
  const bool cols = wy == 0 && lane < 4 * (MY + 2);
  const int ccol = cq4 < 2 ? cq4 : MX + cq4;  // LDS column
  const unsigned coff = cols ? offset(x0 - 2 + ccol, y0 - 1 + cr) : own;

  struct Fetch {  // a plane's values: own column, halo row, halo columns
    double p, T, u, v, w, hp, hT, hu, hv, hw, cp, cT;  // hu, hv, hw also serve the columns
  };
  auto fetch = [&](int k, Fetch &f) {
    const long base = plane(k);
    const double *u = ka->S.q[0] + base, *v = ka->S.q[1] + base, *w = ka->S.q[2] + base,
                 *p = ka->S.q[3] + base, *T = ka->S.q[4] + base;
    f.p = ldp(p, own);
    f.T = ldp(T, own);
    f.u = ldp(u, own);
    f.v = ldp(v, own);
    f.w = ldp(w, own);
    f.hp = ldp(p, hoff);
    f.hT = ldp(T, hoff);
    if (hfull) {
      f.hu = ldp(u, hoff);
      f.hv = ldp(v, hoff);
      f.hw = ldp(w, hoff);
    }
    if (cols) {
      f.cp = ldp(p, coff);
      f.cT = ldp(T, coff);
      f.hu = ldp(u, coff);
      f.hv = ldp(v, coff);
      f.hw = ldp(w, coff);
    }
  };

  // geometry: x per lane, y uniform
  const bool io = !P.per[0];  // x is periodic or inlet / outlet
  const int ig = min(i, n0 - 1), jg = min(j, n1 - 1);
  const double dxll = TV ? W(P, 0, ig - 2) : 0.0, dxl = W(P, 0, ig - 1), dx = W(P, 0, ig), dxh = W(P, 0, ig + 1);
  const double idxl = IW(P, 0, ig - 1), idx = IW(P, 0, ig);
  const bool xl = io && i == 0, xh = io && i == n0 - 1;
  const double icx = IC(P, 0, ig), icxh = xh ? 0.0 : IC(P, 0, ig + 1);
  const double wlox = WLO(P, 0, ig), whix = WHI(P, 0, ig);
  // the last cells' values stand for those on the outlet face
  const double wloxE = xh ? 1.0 : WLO(P, 0, ig + 1), whixE = xh ? 0.0 : WHI(P, 0, ig + 1);
  const bool yl = !P.per[1] && j == 0, yh = !P.per[1] && j == n1 - 1;
  const bool tvx = TV && (!io || (i >= 2 && i + 1 < n0)),
             tvy = TV && (P.per[1] || (j >= 2 && j + 1 < n1));
  const bool active = i < n0 && j < n1;
  // a block with cells next to a boundary in x or y
  const bool edge = (io && (x0 == 0 || x0 + MX >= n0)) || (!P.per[1] && (y0 == 0 || y0 + MY >= n1));
  const int cx = lane + 2, ry = wy + 1;
  const CDbl geoy = (CDbl)(P.geo[1] + NGEO * jg), geoz = (CDbl)P.geo[2];

  // own column: planes k-1 (m), k (0), k+1 (p), rho also k-2 (mm); and of the
  // plane's neighbours what a later plane uses
  double Tm = 1, T0 = 1, Tp = 1, gm = 1, g0 = 1, gp = 1, rmm = 1, rm = 1, r0 = 1, rp = 1;
  double p0 = 1, pp = 1;
  double um = 0, u0 = 0, up = 0, vm = 0, v0 = 0, vp = 0, wm = 0, w0 = 0, wp = 0;
  double gxm = 1, gym = 1, gxEm = 1, gyNm = 1, uEm = 0, vNm = 0;

  // put a fetched plane into LDS slot q and shift the own column
  auto stash = [&](int q, const Fetch &f) {
    Plane3 &s = pl[q];
    const double r = ddiv(f.p, f.T), g = sqrt(f.T);
    s.u[ry][cx] = f.u;
    s.v[ry][cx] = f.v;
    s.w[ry][cx] = f.w;
    s.T[ry][cx] = f.T;
    s.g[ry][cx] = g;
    s.r[ry + 1][cx] = r;
    s.r[hr + 2][cx] = ddiv(f.hp, f.hT);
    if (hfull) {
      s.u[hr + 1][cx] = f.hu;
      s.v[hr + 1][cx] = f.hv;
      s.w[hr + 1][cx] = f.hw;
      s.T[hr + 1][cx] = f.hT;
      s.g[hr + 1][cx] = sqrt(f.hT);
    }
    if (cols) {
      s.u[cr][ccol] = f.hu;
      s.v[cr][ccol] = f.hv;
      s.w[cr][ccol] = f.hw;
      s.T[cr][ccol] = f.cT;
      s.g[cr][ccol] = sqrt(f.cT);
      s.r[cr + 1][ccol] = ddiv(f.cp, f.cT);
    }
    p0 = pp, pp = f.p;
    Tm = T0, T0 = Tp, Tp = f.T;
    gm = g0, g0 = gp, gp = g;
    rmm = rm, rm = r0, r0 = rp, rp = r;
    um = u0, u0 = up, up = f.u;
    vm = v0, v0 = vp, vp = f.v;
    wm = w0, w0 = wp, wp = f.w;
  };
  // step constants of the current plane and of the next
  struct Const4 {
    double T, q[3];
  };
  auto constants = [&](int k, Const4 &c) {
    const long base = (long)(k + G) * P.sz;
    c.T = ldp(ka->Wk.cT + base, own);
    for (int e = 0; e < 3; e++) c.q[e] = ldp(ka->Wk.cq[e] + base, own);
  };
  Fetch nx;
  Const4 cn;
  {
    // the first three planes and the constants, all loads before the first wait
    Fetch a, c;
    const long base = plane(z0 - 2);
    const double p2 = ldp(A.S.q[3] + base, own), T2 = ldp(A.S.q[4] + base, own);
    fetch(z0 - 1, a);
    fetch(z0, c);
    fetch(z0 + 1, nx);
    constants(z0, cn);
    rp = ddiv(p2, T2);
    stash(2, a);
    stash(0, c);
    __syncthreads();
    const Plane3 &s = pl[2];  // the plane z0 - 1, whose own column is now T0, g0, ...
    const Geo3 gy(geoy);
    gxm = xl ? P.sqT_in : wlox * s.g[ry][cx - 1] + whix * g0;
    gym = gy.wlo * s.g[ry - 1][cx] + gy.whi * g0;
    gxEm = wloxE * g0 + whixE * s.g[ry][cx + 1];
    gyNm = gy.wloH * g0 + gy.whiH * s.g[ry + 1][cx];
    uEm = s.u[ry][cx + 1];
    vNm = s.v[ry + 1][cx];
  }
  int q0 = 0;  // LDS slot of plane k
  for (int k = z0; k < z1; k++) {
    const int q1 = q0 == 2 ? 0 : q0 + 1;
    stash(q1, nx);
    __syncthreads();
    const Const4 c0 = cn;
    if (k + 1 < z1) {
      fetch(k + 2, nx);
      constants(k + 1, cn);
    }
    const Plane3 &s = pl[q0], &sp = pl[q1];
    q0 = q1;
    if (!active) continue;  // (every wave still meets every barrier)

    const long base = (long)(k + G) * P.sz;
    auto store = [&](double *a, double v) { stp(a + base, own, v); };
    // EG: some cell of the block lies on a boundary of the domain (the
    // boundary rules are compiled out of the other blocks' planes)
    auto equations = [&](auto eg) {
      constexpr bool EG = decltype(eg)::value;
      const bool XL = EG && xl, XH = EG && xh, YL = EG && yl, YH = EG && yh;
      const bool ZL = EG && !ka->P.per[2] && k == 0, ZH = EG && !ka->P.per[2] && k == ka->P.n[2] - 1;
      N3_SECTION(ke);
      // ---- energy -----------------------------------------------------------
      {
        const Geo3 gy(fresh(geoy)), gz(fresh(geoz) + NGEO * k);
        const double arx = gy.w * gz.w, ary = dx * gz.w, arz = dx * gy.w, dV = dx * gy.w * gz.w;
        double sa, sn;
        {
          const double TW = s.T[ry][cx - 1], TE = s.T[ry][cx + 1];
          const double gl = XL ? ke->P.sqT_in : N3_gW0, nl = XL ? ke->P.T_in : TW;
          const double dl = XL ? dx : dxl, il = XL ? 2.0 * idx : icx;
          const double aL = ke->P.C1 * hmean(dl, gl, dx, g0) * arx * il;
          const double aH = ke->P.C1 * hmean(dx, g0, dxh, N3_gE0) * arx * icxh;  // 0 at the outlet
          const double nh = XH ? T0 : TE;
          sa = aL + aH;
          sn = aL * nl + aH * nh;
        }
        {
          const double TS = s.T[ry - 1][cx], TN = s.T[ry + 1][cx];
          double aL, aH, nl = TS, nh = TN;
          if (YL) {
            nl = (ke->P.wt[1][0] == STS3_NOSLIP) ? ke->P.wT[1][0] : T0;
            aL = (ke->P.wt[1][0] == STS3_NOSLIP) ? ke->P.C1 * hmean2(g0, ke->P.sqwT[1][0]) * ary * 2.0 * gy.iw : 0.0;
          } else {
            aL = ke->P.C1 * hmean(gy.wm, N3_gS0, gy.w, g0) * ary * gy.ic;
          }
          if (YH) {
            nh = (ke->P.wt[1][1] == STS3_NOSLIP) ? ke->P.wT[1][1] : T0;
            aH = (ke->P.wt[1][1] == STS3_NOSLIP) ? ke->P.C1 * hmean2(g0, ke->P.sqwT[1][1]) * ary * 2.0 * gy.iw : 0.0;
          } else {
            aH = ke->P.C1 * hmean(gy.w, g0, gy.wh, N3_gN0) * ary * gy.ich;
          }
          sa += aL + aH;
          sn += aL * nl + aH * nh;
        }
        {
          double aL, aH, nl = Tm, nh = Tp;
          if (ZL) {
            nl = (ke->P.wt[2][0] == STS3_NOSLIP) ? ke->P.wT[2][0] : T0;
            aL = (ke->P.wt[2][0] == STS3_NOSLIP) ? ke->P.C1 * hmean2(g0, ke->P.sqwT[2][0]) * arz * 2.0 * gz.iw : 0.0;
          } else {
            aL = ke->P.C1 * hmean(gz.wm, gm, gz.w, g0) * arz * gz.ic;
          }
          if (ZH) {
            nh = (ke->P.wt[2][1] == STS3_NOSLIP) ? ke->P.wT[2][1] : T0;
            aH = (ke->P.wt[2][1] == STS3_NOSLIP) ? ke->P.C1 * hmean2(g0, ke->P.sqwT[2][1]) * arz * 2.0 * gz.iw : 0.0;
          } else {
            aH = ke->P.C1 * hmean(gz.w, g0, gz.wh, gp) * arz * gz.ich;
          }
          sa += aL + aH;
          sn += aL * nl + aH * nh;
        }
        const double a0 = ke->P.dt * sa + r0 * dV;
        const double d0 = (N3_uE0 - u0) * idx, d1 = (N3_vN0 - v0) * gy.iw, d2 = (wp - w0) * gz.iw;
        const double div = d0 + d1 + d2;
        double phi = 2.0 * (d0 * d0 + d1 * d1 + d2 * d2);
        const double uc = 0.5 * (u0 + N3_uE0), vc = 0.5 * (v0 + N3_vN0), wc = 0.5 * (w0 + wp);
        // u on the y-faces and v on the x-faces of the cell
        {
          double l = gy.whi * uc + gy.wlo * (0.5 * (N3_uS + N3_uSE)), h = gy.wloH * uc + gy.whiH * (0.5 * (N3_uN + N3_uNE));
          if (YL) l = (ke->P.wt[1][0] == STS3_NOSLIP) ? ke->P.wv[1][0][0] : uc;
          if (YH) h = (ke->P.wt[1][1] == STS3_NOSLIP) ? ke->P.wv[1][1][0] : uc;
          const double l2 = XL ? 0.0 : whix * vc + wlox * (0.5 * (N3_vW + N3_vNW));
          const double h2 = wloxE * vc + whixE * (0.5 * (N3_vE + N3_vNE));
          const double sh = (h - l) * gy.iw + (h2 - l2) * idx;
          phi += sh * sh;
        }
        // u on the z-faces and w on the x-faces
        {
          double l = gz.whi * uc + gz.wlo * (0.5 * (um + uEm)), h = gz.wloH * uc + gz.whiH * (0.5 * (up + N3_uEp));
          if (ZL) l = (ke->P.wt[2][0] == STS3_NOSLIP) ? ke->P.wv[2][0][0] : uc;
          if (ZH) h = (ke->P.wt[2][1] == STS3_NOSLIP) ? ke->P.wv[2][1][0] : uc;
          const double l2 = XL ? 0.0 : whix * wc + wlox * (0.5 * (N3_wW0 + N3_wWp));
          const double h2 = wloxE * wc + whixE * (0.5 * (N3_wE0 + N3_wEp));
          const double sh = (h - l) * gz.iw + (h2 - l2) * idx;
          phi += sh * sh;
        }
        // v on the z-faces and w on the y-faces
        {
          double l = gz.whi * vc + gz.wlo * (0.5 * (vm + vNm)), h = gz.wloH * vc + gz.whiH * (0.5 * (vp + N3_vNp));
          if (ZL) l = (ke->P.wt[2][0] == STS3_NOSLIP) ? ke->P.wv[2][0][1] : vc;
          if (ZH) h = (ke->P.wt[2][1] == STS3_NOSLIP) ? ke->P.wv[2][1][1] : vc;
          double l2 = gy.whi * wc + gy.wlo * (0.5 * (N3_wS0 + N3_wSp)), h2 = gy.wloH * wc + gy.whiH * (0.5 * (N3_wN0 + N3_wNp));
          if (YL) l2 = (ke->P.wt[1][0] == STS3_NOSLIP) ? ke->P.wv[1][0][2] : wc;
          if (YH) h2 = (ke->P.wt[1][1] == STS3_NOSLIP) ? ke->P.wv[1][1][2] : wc;
          const double sh = (h - l) * gz.iw + (h2 - l2) * gy.iw;
          phi += sh * sh;
        }
        phi -= 2.0 / 3.0 * div * div;
        const double src = ke->P.C2 * g0 * phi * dV + ke->P.C3 * p0 * div * dV;
        store(ke->Tout, ddiv(ke->P.dt * (sn + src) + c0.T, a0));
      }

      N3_SECTION(kg);
      const Geo3 gy(fresh(geoy)), gz(fresh(geoz) + NGEO * k);
      // Gamma on the edges around the low faces of the cell
      const double gxS = XL ? kg->P.sqT_in : wlox * N3_gSW + whix * N3_gS0, gxN = XL ? kg->P.sqT_in : wlox * N3_gNW + whix * N3_gN0;
      const double gx0 = XL ? kg->P.sqT_in : wlox * N3_gW0 + whix * g0, gy0 = gy.wlo * N3_gS0 + gy.whi * g0;
      const double gxp = XL ? kg->P.sqT_in : wlox * sp.g[ry][cx - 1] + whix * gp;
      const double gyp = gy.wlo * sp.g[ry - 1][cx] + gy.whi * gp;
      const double gez = gy.wlo * gxS + gy.whi * gx0;                // (i, j)
      const double gezN = gy.wloH * gx0 + gy.whiH * gxN;             // (i, j + 1)
      const double gxE = wloxE * g0 + whixE * N3_gE0, gyN = gy.wloH * g0 + gy.whiH * N3_gN0;
      const double gezE = gy.wlo * (wloxE * N3_gS0 + whixE * N3_gSE) + gy.whi * gxE;  // (i + 1, j)
      const double gey = gz.wlo * gxm + gz.whi * gx0, geyT = gz.wloH * gx0 + gz.whiH * gxp;
      const double geyE = gz.wlo * gxEm + gz.whi * gxE;
      const double gex = gz.wlo * gym + gz.whi * gy0, gexT = gz.wloH * gy0 + gz.whiH * gyp;
      const double gexN = gz.wlo * gyNm + gz.whi * gyN;
      const double t23 = 2.0 / 3.0, f43 = 4.0 / 3.0;

      N3_SECTION(ku);
      // ---- u ------------------------------------------------------------------
      {
        const Geo3 gy(fresh(geoy)), gz(fresh(geoz) + NGEO * k);
        const double arx = gy.w * gz.w;
        const double len = 0.5 * (dxl + dx), M = (r0 * dx + N3_rW * dxl) * arx / 2.0;
        const double DL = ku->P.B * N3_gW0 * arx * idxl, DH = ku->P.B * g0 * arx * idx;
        const double aW = f43 * DL, aE = f43 * DH;
        double sa = aW + aE, sn = aW * N3_uW + aE * N3_uE0;
        {
          double GL = gez, GH = gezN, iL = gy.ic, iH = gy.ich, ql = N3_uS, qh = N3_uN;
          if (YL) GL = gx0 + ku->P.sqwT[1][0], iL = (ku->P.wt[1][0] == STS3_NOSLIP) ? gy.iw : 0.0, ql = (ku->P.wt[1][0] == STS3_NOSLIP) ? ku->P.wv[1][0][0] : u0;
          if (YH) GH = gx0 + ku->P.sqwT[1][1], iH = (ku->P.wt[1][1] == STS3_NOSLIP) ? gy.iw : 0.0, qh = (ku->P.wt[1][1] == STS3_NOSLIP) ? ku->P.wv[1][1][0] : u0;
          const double aL = ku->P.B * GL * len * gz.w * iL, aH = ku->P.B * GH * len * gz.w * iH;
          sa += aL + aH;
          sn += aL * ql + aH * qh;
        }
        double X = (gezN * (N3_vN0 - N3_vNW) - gez * (v0 - N3_vW)) * gz.w - t23 * (g0 * (N3_vN0 - v0) - N3_gW0 * (N3_vNW - N3_vW)) * gz.w;
        {
          double GL = gey, GH = geyT, iL = gz.ic, iH = gz.ich, ql = um, qh = up;
          if (ZL) GL = gx0 + ku->P.sqwT[2][0], iL = (ku->P.wt[2][0] == STS3_NOSLIP) ? gz.iw : 0.0, ql = (ku->P.wt[2][0] == STS3_NOSLIP) ? ku->P.wv[2][0][0] : u0;
          if (ZH) GH = gx0 + ku->P.sqwT[2][1], iH = (ku->P.wt[2][1] == STS3_NOSLIP) ? gz.iw : 0.0, qh = (ku->P.wt[2][1] == STS3_NOSLIP) ? ku->P.wv[2][1][0] : u0;
          const double aL = ku->P.B * GL * len * gy.w * iL, aH = ku->P.B * GH * len * gy.w * iH;
          sa += aL + aH;
          sn += aL * ql + aH * qh;
        }
        X += (geyT * (wp - N3_wWp) - gey * (w0 - N3_wW0)) * gy.w - t23 * (g0 * (wp - w0) - N3_gW0 * (N3_wWp - N3_wW0)) * gy.w;
        const double ia0 = drcp(sa + M * ku->P.idt);
        const double bb = c0.q[0] + ku->P.B * X;
        store(ku->Wk.qh[0], XL ? u0 : (sn + bb) * ia0);
        store(ku->Wk.dq[0], XL ? 0.0 : ku->P.A * arx * ia0);
      }
      N3_SECTION(kv);
      // ---- v ------------------------------------------------------------------
      {
        const Geo3 gy(fresh(geoy)), gz(fresh(geoz) + NGEO * k);
        const double ary = dx * gz.w;
        const double len = 0.5 * (gy.wm + gy.w), M = (r0 * gy.w + N3_rS * gy.wm) * ary / 2.0;
        const double DL = kv->P.B * N3_gS0 * ary * gy.iwm, DH = kv->P.B * g0 * ary * gy.iw;
        const double aS = f43 * DL, aN = f43 * DH;
        double sa, sn;
        {
          const double GL = XL ? gy0 + kv->P.sqT_in : gez, iL = XL ? idx : icx;
          const double aL = kv->P.B * GL * len * gz.w * iL, aH = kv->P.B * gezE * len * gz.w * icxh;
          sa = aL + aH;
          sn = aL * (XL ? 0.0 : N3_vW) + aH * (XH ? v0 : N3_vE);
        }
        sa += aS + aN;
        sn += aS * N3_vS + aN * N3_vN0;
        double X = (gezE * (N3_uE0 - N3_uSE) - gez * (u0 - N3_uS)) * gz.w - t23 * (g0 * (N3_uE0 - u0) - N3_gS0 * (N3_uSE - N3_uS)) * gz.w;
        {
          double GL = gex, GH = gexT, iL = gz.ic, iH = gz.ich, ql = vm, qh = vp;
          if (ZL) GL = gy0 + kv->P.sqwT[2][0], iL = (kv->P.wt[2][0] == STS3_NOSLIP) ? gz.iw : 0.0, ql = (kv->P.wt[2][0] == STS3_NOSLIP) ? kv->P.wv[2][0][1] : v0;
          if (ZH) GH = gy0 + kv->P.sqwT[2][1], iH = (kv->P.wt[2][1] == STS3_NOSLIP) ? gz.iw : 0.0, qh = (kv->P.wt[2][1] == STS3_NOSLIP) ? kv->P.wv[2][1][1] : v0;
          const double aL = kv->P.B * GL * len * dx * iL, aH = kv->P.B * GH * len * dx * iH;
          sa += aL + aH;
          sn += aL * ql + aH * qh;
        }
        X += (gexT * (wp - N3_wSp) - gex * (w0 - N3_wS0)) * dx - t23 * (g0 * (wp - w0) - N3_gS0 * (N3_wSp - N3_wS0)) * dx;
        const double ia0 = drcp(sa + M * kv->P.idt);
        const double bb = c0.q[1] + kv->P.B * X;
        store(kv->Wk.qh[1], YL ? v0 : (sn + bb) * ia0);
        store(kv->Wk.dq[1], YL ? 0.0 : kv->P.A * ary * ia0);
      }
      N3_SECTION(kw);
      // ---- w ------------------------------------------------------------------
      {
        const Geo3 gy(fresh(geoy)), gz(fresh(geoz) + NGEO * k);
        const double arz = dx * gy.w;
        const double gn = gz.wlo * gm + gz.whi * g0;
        const double len = 0.5 * (gz.wm + gz.w), M = (r0 * gz.w + rm * gz.wm) * arz / 2.0;
        const double DL = kw->P.B * gm * arz * gz.iwm, DH = kw->P.B * g0 * arz * gz.iw;
        const double aB = f43 * DL, aT = f43 * DH;
        double sa, sn;
        {
          const double GL = XL ? gn + kw->P.sqT_in : gey, iL = XL ? idx : icx;
          const double aL = kw->P.B * GL * len * gy.w * iL, aH = kw->P.B * geyE * len * gy.w * icxh;
          sa = aL + aH;
          sn = aL * (XL ? 0.0 : N3_wW0) + aH * (XH ? w0 : N3_wE0);
        }
        double X = (geyE * (N3_uE0 - uEm) - gey * (u0 - um)) * gy.w - t23 * (g0 * (N3_uE0 - u0) - gm * (uEm - um)) * gy.w;
        {
          double GL = gex, GH = gexN, iL = gy.ic, iH = gy.ich, ql = N3_wS0, qh = N3_wN0;
          if (YL) GL = gn + kw->P.sqwT[1][0], iL = (kw->P.wt[1][0] == STS3_NOSLIP) ? gy.iw : 0.0, ql = (kw->P.wt[1][0] == STS3_NOSLIP) ? kw->P.wv[1][0][2] : w0;
          if (YH) GH = gn + kw->P.sqwT[1][1], iH = (kw->P.wt[1][1] == STS3_NOSLIP) ? gy.iw : 0.0, qh = (kw->P.wt[1][1] == STS3_NOSLIP) ? kw->P.wv[1][1][2] : w0;
          const double aL = kw->P.B * GL * len * dx * iL, aH = kw->P.B * GH * len * dx * iH;
          sa += aL + aH;
          sn += aL * ql + aH * qh;
        }
        X += (gexN * (N3_vN0 - vNm) - gex * (v0 - vm)) * dx - t23 * (g0 * (N3_vN0 - v0) - gm * (vNm - vm)) * dx;
        sa += aB + aT;
        sn += aB * wm + aT * wp;
        const double ia0 = drcp(sa + M * kw->P.idt);
        const double bb = c0.q[2] + kw->P.B * X;
        store(kw->Wk.qh[2], ZL ? w0 : (sn + bb) * ia0);
        store(kw->Wk.dq[2], ZL ? 0.0 : kw->P.A * arz * ia0);
      }
      N3_SECTION(kf);
      // ---- face densities -------------------------------------------------------
      const Geo3 fy(fresh(geoy)), fz(fresh(geoz) + NGEO * k);
      {
        double r = upw(XL ? kf->P.rho_in : N3_rW, r0, u0);
        if (TV) {
          const double ps = psi_w(s.r[ry + 1][cx - 2], N3_rW, r0, s.r[ry + 1][cx + 1], dxll, dxl,
                                  dx, dxh, wlox, whix, u0);
          r += tvx ? ps * (r0 - N3_rW) : 0.0;
        }
        store(kf->Wk.rf[0], r);
      }
      {
        double r = YL ? r0 : upw(N3_rS, r0, v0);
        if (tvy)
          r += psi_w(s.r[ry - 1][cx], N3_rS, r0, s.r[ry + 2][cx], fy.wmm, fy.wm, fy.w, fy.wh, fy.wlo, fy.whi, v0) *
               (r0 - N3_rS);
        store(kf->Wk.rf[1], r);
      }
      {
        double r = ZL ? r0 : upw(rm, r0, w0);
        if (TV && (kf->P.per[2] || (k >= 2 && k + 1 < kf->P.n[2])))
          r += psi_w(rmm, rm, r0, rp, fz.wmm, fz.wm, fz.w, fz.wh, fz.wlo, fz.whi, w0) * (r0 - rm);
        store(kf->Wk.rf[2], r);
      }
      gxm = gx0, gym = gy0, gxEm = gxE, gyNm = gyN, uEm = N3_uE0, vNm = N3_vN0;
      // the last boundary faces: no unknowns, the last cell's density
      if (XH) {
        const long m = lin(P, kf->P.n[0], j, k);
        kf->Wk.qh[0][m] = N3_uE0;
        kf->Wk.dq[0][m] = 0.0;
        kf->Wk.rf[0][m] = r0;
      }
      if (YH) {
        const long m = lin(P, i, kf->P.n[1], k);
        kf->Wk.qh[1][m] = N3_vN0;
        kf->Wk.dq[1][m] = 0.0;
        kf->Wk.rf[1][m] = r0;
      }
      if (ZH) {
        const long m = lin(P, i, j, kf->P.n[2]);
        kf->Wk.qh[2][m] = wp;
        kf->Wk.dq[2][m] = 0.0;
        kf->Wk.rf[2][m] = r0;
      }
    };
    if (edge || (!ka->P.per[2] && (k == 0 || k == ka->P.n[2] - 1))) equations(std::true_type{});
    else equations(std::false_type{});
  }
}
#undef N3_gW0
#undef N3_gE0
#undef N3_gS0
#undef N3_gN0
#undef N3_uE0
#undef N3_uEp
#undef N3_vN0
#undef N3_vNp
#undef N3_wW0
#undef N3_wE0
#undef N3_wS0
#undef N3_wN0
#undef N3_wWp
#undef N3_wEp
#undef N3_wSp
#undef N3_wNp
#undef N3_gSW
#undef N3_gSE
#undef N3_gNW
#undef N3_uW
#undef N3_uS
#undef N3_uN
#undef N3_uSE
#undef N3_uNE
#undef N3_vS
#undef N3_vW
#undef N3_vE
#undef N3_vNW
#undef N3_vNE
#undef N3_rW
#undef N3_rS
#undef N3_SECTION

// The pressure equation (pl23, pl24) and the velocities (pl18, pl19) of a
// pass.  A block of VY + 1 waves of 64 columns walks up z; its first column
// and first row only serve the new pressure on the low side of the owned
// ones (exchanged through LDS), the plane below stays in registers.  VY = 7:
// blocks of 8 waves, two on a CU; 9 waves leave room for one (0.345 against
// 0.33 ms), 4 waves read more halo rows (0.35 ms).
constexpr int VX = 63, VY = 7;
__global__ __launch_bounds__(64 * (VY + 1)) __attribute__((amdgpu_waves_per_eu(4))) void k3_sweep_pv(P3 P, Fld S, Fld N, Work Wk, int tx,
                                                             int ty, int seg) {
  __shared__ double pl[2][VY + 1][64];
  const int b = xcd_block(blockIdx.x, gridDim.x);
  const int x0 = (b % tx) * VX, y0 = (b / tx % ty) * VY, z0 = (b / (tx * ty)) * seg;
  const int n0 = P.n[0], n1 = P.n[1], n2 = P.n[2];
  const int z1 = min(z0 + seg, n2);
  const int lane = threadIdx.x, wy = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
  const int i = x0 - 1 + lane, j = y0 - 1 + wy;
  // the low halo of a periodic direction is the last cell; past the domain
  // the last cell again, which nothing uses
  const int iw = i < 0 ? (P.per[0] ? n0 - 1 : 0) : min(i, n0 - 1);
  const int jw = j < 0 ? (P.per[1] ? n1 - 1 : 0) : min(j, n1 - 1);
  auto offset = [&](int x, int y) {
    x = around(x, n0, P.per[0]), y = around(y, n1, P.per[1]);
    return 8u * ((unsigned)(y + G) * (unsigned)P.sy + (unsigned)(x + G));
  };
  const unsigned own = offset(iw, jw), we = offset(iw - 1, jw), ea = offset(iw + 1, jw),
                 so = offset(iw, jw - 1), no = offset(iw, jw + 1);
  auto plane = [&](int k) { return (long)(around(k, n2, P.per[2]) + G) * P.sz; };
  const bool owned = lane >= 1 && i < n0 && wy >= 1 && j < n1;
  const double dx = W(P, 0, iw), dy = W(P, 1, jw);
  const bool xs = P.per[0] || i > 0, ys = P.per[1] || j > 0;
  // below the first plane: nothing on a wall, else one more plane of pressures
  const bool below = z0 > 0 || P.per[2];
  const int first = below ? z0 - 1 : z0;
  long base = plane(first);
  double rfz = ldp(Wk.rf[2] + base, own), dqz = ldp(Wk.dq[2] + base, own),
         qhz = ldp(Wk.qh[2] + base, own);
  double pm = ldp(S.q[3] + plane(first - 1), own), p0 = ldp(S.q[3] + base, own), pnm = 0.0;
  int buf = 0;
  for (int t = first; t < z1; t++) {
    const int k = around(t, n2, P.per[2]);
    base = plane(t);
    const long above = plane(t + 1);
    const double Tn = ldp(N.q[4] + base, own), cp = ldp(Wk.cp + base, own);
    const double *pb = S.q[3] + base;
    const double pW = ldp(pb, we), pE = ldp(pb, ea), pS = ldp(pb, so),
                 pN = ldp(pb, no), pp = ldp(S.q[3] + above, own);
    const double rx = ldp(Wk.rf[0] + base, own), rxE = ldp(Wk.rf[0] + base, ea);
    const double dqx = ldp(Wk.dq[0] + base, own), dqxE = ldp(Wk.dq[0] + base, ea);
    const double qhx = ldp(Wk.qh[0] + base, own), qhxE = ldp(Wk.qh[0] + base, ea);
    const double ryy = ldp(Wk.rf[1] + base, own), ryN = ldp(Wk.rf[1] + base, no);
    const double dqy = ldp(Wk.dq[1] + base, own), dqyN = ldp(Wk.dq[1] + base, no);
    const double qhy = ldp(Wk.qh[1] + base, own), qhyN = ldp(Wk.qh[1] + base, no);
    const double rzT = ldp(Wk.rf[2] + above, own), dqzT = ldp(Wk.dq[2] + above, own),
                 qhzT = ldp(Wk.qh[2] + above, own);
    const double dz = W(P, 2, k), dV = dx * dy * dz;
    const double arx = dy * dz, ary = dx * dz, arz = dx * dy;
    double sa, sap, sb;
    {
      const double aL = rx * dqx * arx, aH = rxE * dqxE * arx;
      const double bL = rx * qhx * arx, bH = rxE * qhxE * arx;
      sa = aL + aH;
      sap = aL * pW + aH * pE;  // a = 0 where there is no neighbour
      sb = bH - bL;
    }
    {
      const double aL = ryy * dqy * ary, aH = ryN * dqyN * ary;
      const double bL = ryy * qhy * ary, bH = ryN * qhyN * ary;
      sa += aL + aH;
      sap += aL * pS + aH * pN;
      sb += bH - bL;
    }
    {
      const double aL = rfz * dqz * arz, aH = rzT * dqzT * arz;
      const double bL = rfz * qhz * arz, bH = rzT * qhzT * arz;
      sa += aL + aH;
      sap += aL * pm + aH * pp;
      sb += bH - bL;
    }
    const double a0 = ddiv(dV, Tn) + sa * P.dt;
    const double pn = ddiv(sap * P.dt + (cp - sb * P.dt), a0);
    pl[buf][wy][lane] = pn;
    __syncthreads();
    if (owned && t >= z0) {
      auto store = [&](double *a, double v) { stp(a + base, own, v); };
      store(N.q[3], pn);
      if (xs) {
        const double un = qhx - dqx * (pn - pl[buf][wy][lane - 1]);
        store(N.q[0], un);
        if (!P.per[0] && i == n0 - 1) {  // outlet: zero gradient
          stp(N.q[0] + base, ea, un);
        }
      }
      if (ys) store(N.q[1], qhy - dqy * (pn - pl[buf][wy - 1][lane]));
      if (P.per[2] || k > 0) store(N.q[2], qhz - dqz * (pn - pnm));
    }
    buf ^= 1;
    pm = p0, p0 = pp, pnm = pn;
    rfz = rzT, dqz = dqzT, qhz = qhzT;
  }
}

// The periodic images of the new state and of the face densities, once per
// step: the sweeps read a periodic direction's other end, everything else
// (the prologue, the residuals, the implicit passes, the host) the images.
__global__ __launch_bounds__(NTB) void k3_images(P3 P, Fld N, Work Wk) {
  const int i = (int)(blockIdx.x * BX + threadIdx.x) - G, j = (int)(blockIdx.y * BY + threadIdx.y) - G;
  if (i > P.n[0] + G || j > P.n[1] + G) return;
  for (int k = (int)blockIdx.z - G; k <= P.n[2] + G; k += gridDim.z) {
    const int x[3] = {i, j, k};
    int y[3];
    bool image = false, inside = true;
    for (int e = 0; e < 3; e++) {
      y[e] = around(x[e], P.n[e], P.per[e]);
      image |= y[e] != x[e];
      inside &= P.per[e] || (x[e] >= 0 && x[e] <= P.n[e]);
    }
    if (!image || !inside) continue;
    const long to = lin(P, x[0], x[1], x[2]), from = lin(P, y[0], y[1], y[2]);
    for (int f = 0; f < 5; f++) N.q[f][to] = N.q[f][from];
    for (int e = 0; e < 3; e++) Wk.rf[e][to] = Wk.rf[e][from];
  }
}

// ---------------------------------------------------------------------------
// per-step constants (prologue), from the state S as level n-1, with rho and
// the face densities of S in Wk
// ---------------------------------------------------------------------------
template <int A, bool EX, bool TV>
__device__ __forceinline__ void const_face(const P3 &P, const Fld &S, const Work &Wk, const int f[3],
                                           double r) {
  const long m = lin(P, f[0], f[1], f[2]);
  double c = 0.0;
  if (solved(P, A, f[A])) {
    int l[3] = {f[0], f[1], f[2]};
    l[A] -= 1;
    const double dal = W(P, A, f[A] - 1), dar = W(P, A, f[A]);
    const double Mm = (r * dar + cv(P, Wk.rho, l) * dal) * area(P, A, f) / 2.0;
    c = Mm * P.idt * S.q[A][m] + P.g[A] * Mm + (EX ? q_explicit<A, TV>(P, S, Wk, f) : 0.0);
  }
  Wk.cq[A][m] = c;
  if (f[A] == P.n[A] - 1) Wk.cq[A][m + stride(P, A)] = 0.0;  // never solved
}

// The constants of a plane's cells (group 0) and of their low faces along
// x, y, z (groups 1 to 3), the groups of a plane in neighbouring blocks: one
// launch, and the fields that the groups share are read while they are in L2.
// Bound by the load chains of the explicit convective terms (no LDS).  One
// thread for a cell and its faces needs 129 registers (upwind; TVD 161) and
// takes 0.55 ms (1.31) on 512x128x128, the groups 76 (115) and 0.54 ms (1.17).
// The groups follow each other along z, or along y (tall) on a grid of more
// planes than a quarter of the launch limit.
template <bool EX, bool TV>
__global__ __launch_bounds__(NTB) void k3_const(P3 P, Fld S, Work Wk, bool tall) {
  const int by = tall ? blockIdx.y >> 2 : blockIdx.y, bz = tall ? blockIdx.z : blockIdx.z >> 2;
  const int x[3] = {(int)(blockIdx.x * BX + threadIdx.x),
                    __builtin_amdgcn_readfirstlane(by * BY + threadIdx.y), bz};
  if (x[0] >= P.n[0] || x[1] >= P.n[1]) return;
  const long m = lin(P, x[0], x[1], x[2]);
  const double r = Wk.rho[m];
  switch ((tall ? blockIdx.y : blockIdx.z) & 3) {
    case 0: {
      const double dV = W(P, 0, x[0]) * W(P, 1, x[1]) * W(P, 2, x[2]);
      Wk.cp[m] = r * dV;
      Wk.cT[m] = r * S.q[4][m] * dV + (EX ? P.dt * T_explicit<TV>(P, S, Wk, x) : 0.0);
      return;
    }
    case 1: return const_face<0, EX, TV>(P, S, Wk, x, r);
    case 2: return const_face<1, EX, TV>(P, S, Wk, x, r);
    case 3: return const_face<2, EX, TV>(P, S, Wk, x, r);
  }
}

// ---------------------------------------------------------------------------
// residuals of the last pass: increments of the unknowns, continuity
// residual; block partials in a fixed order, then one block folds them
// ---------------------------------------------------------------------------
__device__ void block_reduce(double v[NR], double *out) {
  __shared__ double red[NTB / 64][NR];
  const int t = threadIdx.y * BX + threadIdx.x, lane = t & 63, wv = t >> 6;
#pragma unroll
  for (int q = 0; q < NR; q++) {
    double a = v[q];
    for (int o = 32; o > 0; o >>= 1) {
      const double b = __shfl_down(a, o, 64);
      a = (q == 6 || q == 7) ? a + b : fmax(a, b);
    }
    if (lane == 0) red[wv][q] = a;
  }
  __syncthreads();
  if (t < NR) {
    double a = red[0][t];
    for (int w = 1; w < NTB / 64; w++) a = (t == 6 || t == 7) ? a + red[w][t] : fmax(a, red[w][t]);
    out[t] = a;
  }
}

// Cells with their low faces (and the high one of a direction's last cell),
// over the tiles of all planes in turn: every field is read once, a block
// reduces once and one launch folds the blocks' rows.  Bound by memory: the
// 14 fields it reads of 512x128x128 take 0.20 ms, 4.7 TB/s; a kernel for the
// cells, one per face direction and two folds took 0.58 ms.
template <int A>
__device__ __forceinline__ void resid_face(const P3 &P, const Fld &O, const Fld &N, const int f[3],
                                           double qn, double v[NR]) {
  if (solved(P, A, f[A])) v[A] = fmax(v[A], fabs(qn - O.q[A][lin(P, f[0], f[1], f[2])]));
  v[7] += (double)(!isfinite(qn));
}
template <int A>
__device__ __forceinline__ double resid_faces(const P3 &P, const Fld &O, const Fld &N, const Work &Wk,
                                              const int x[3], double v[NR]) {
  int xh[3] = {x[0], x[1], x[2]};
  xh[A] += 1;
  const double ar = area(P, A, x), ql = N.q[A][lin(P, x[0], x[1], x[2])];
  const double qh = fv(P, N.q[A], A, xh);
  resid_face<A>(P, O, N, x, ql, v);
  if (xh[A] == P.n[A]) resid_face<A>(P, O, N, xh, N.q[A][lin(P, xh[0], xh[1], xh[2])], v);
  return fv(P, Wk.rf[A], A, xh) * qh * ar - fv(P, Wk.rf[A], A, x) * ql * ar;
}
__global__ __launch_bounds__(NTB) void k3_resid(P3 P, Fld O, Fld N, Work Wk, double *part) {
  double v[NR] = {0, 0, 0, 0, 0, 0, 0, 0};
  const int tx = (P.n[0] + BX - 1) / BX, ty = (P.n[1] + BY - 1) / BY;
  const long tiles = (long)tx * ty * P.n[2];
  for (long t = blockIdx.x; t < tiles; t += gridDim.x) {
    const int k = (int)(t / (tx * ty)), r = (int)(t - (long)k * (tx * ty));
    const int x[3] = {r % tx * BX + (int)threadIdx.x,
                      r / tx * BY + __builtin_amdgcn_readfirstlane(threadIdx.y), k};
    if (x[0] >= P.n[0] || x[1] >= P.n[1]) continue;
    const long m = lin(P, x[0], x[1], x[2]);
    const double dV = W(P, 0, x[0]) * W(P, 1, x[1]) * W(P, 2, x[2]);
    const double pn = N.q[3][m], Tn = N.q[4][m];
    v[3] = fmax(v[3], fabs(pn - O.q[3][m]));
    v[4] = fmax(v[4], fabs(Tn - O.q[4][m]));
    double R = (pn / Tn * dV - Wk.cp[m]) / P.dt;
    R += resid_faces<0>(P, O, N, Wk, x, v);
    R += resid_faces<1>(P, O, N, Wk, x, v);
    R += resid_faces<2>(P, O, N, Wk, x, v);
    v[5] = fmax(v[5], fabs(R));
    v[6] += R;
    v[7] += (double)(!isfinite(pn)) + (double)(!isfinite(Tn));
  }
  block_reduce(v, part + (long)blockIdx.x * NR);
}

// fold the rows of all blocks (fixed order)
__global__ __launch_bounds__(NTB) void k3_resid_fold(const double *part, int nrows, double *out) {
  double v[NR] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int b = threadIdx.y * BX + threadIdx.x; b < nrows; b += NTB)
#pragma unroll
    for (int q = 0; q < NR; q++)
      v[q] = (q == 6 || q == 7) ? v[q] + part[(long)b * NR + q] : fmax(v[q], part[(long)b * NR + q]);
  block_reduce(v, out);
}
constexpr int RES_BLOCKS3 = 2048;  // eight per CU, as many as it holds

// ---------------------------------------------------------------------------
// dense host layout <-> padded fields
// ---------------------------------------------------------------------------
struct Ext {
  int D[3], E[3];  // dense extents, padded extents
};
constexpr int RWB = 256;

__global__ __launch_bounds__(RWB) void k3_pack(P3 P, Ext E, const double *q, double *d) {
  const int i = blockIdx.x * RWB + threadIdx.x;
  if (i >= E.D[0]) return;
  for (int k = blockIdx.z; k < E.D[2]; k += gridDim.z)
    for (int j = blockIdx.y; j < E.D[1]; j += gridDim.y)
      d[((long)k * E.D[1] + j) * E.D[0] + i] = q[lin(P, i, j, k)];
}

// Field f (0..2 velocity, 3 p, 4 T) over the whole padded array: from the
// dense array src, else the constant v0 (init), else the field `own`.  A
// periodic direction's last face copies face 0, the outlet face its
// neighbour, the inlet face holds u_in and wall faces 0.  Ghost entries get
// the periodic images, or a finite constant in a direction without.
__device__ __forceinline__ double imposed(const P3 &P, int f, const Ext &E, const double *src,
                                          const double *own, bool init, double v0, int x0, int x1,
                                          int x2) {
  int x[3] = {x0, x1, x2};
  bool in = true;
#pragma unroll
  for (int e = 0; e < 3; e++) {
    const int top = E.D[e];
    if (x[e] >= 0 && x[e] < top) continue;
    if (P.per[e] && x[e] < top + G) x[e] += x[e] < 0 ? P.n[e] : -P.n[e];
    else in = false;
  }
  if (!in) return f >= 3 ? 1.0 : 0.0;
#pragma unroll
  for (int a = 0; a < 3; a++) {
    if (a != f) continue;
    if (P.per[a]) {
      if (x[a] == P.n[a]) x[a] = 0;
    } else if (a == 0 && P.io) {
      if (x[0] == 0) return P.u_in;
      if (x[0] == P.n[0]) x[0]--;
    } else if (x[a] == 0 || x[a] == P.n[a]) {
      return 0.0;
    }
  }
  if (src) return src[((long)x[2] * E.D[1] + x[1]) * E.D[0] + x[0]];
  return init ? v0 : own[lin(P, x[0], x[1], x[2])];
}
__global__ __launch_bounds__(RWB) void k3_impose(P3 P, int f, Ext E, const double *src, const double *own,
                                                 bool init, double v0, double *out) {
  const int i = (int)(blockIdx.x * RWB + threadIdx.x) - G;
  if (i >= E.E[0] - G) return;
  for (int k = (int)blockIdx.z - G; k < E.E[2] - G; k += gridDim.z)
    for (int j = (int)blockIdx.y - G; j < E.E[1] - G; j += gridDim.y)
      out[lin(P, i, j, k)] = imposed(P, f, E, src, own, init, v0, i, j, k);
}

}  // namespace
}  // namespace sts3

// ===========================================================================
// host side
// ===========================================================================
using namespace sts3;

struct sts3_ctx {
  P3 P;
  int n[3];
  long pitch, sy, sz, off;
  size_t field_bytes;
  hipStream_t stream;
  bool own_stream;
  int device;
  std::vector<void *> allocs;
  Fld st[2];
  int cur;
  Work Wk;
  double *d_d[3];  // per direction: NGEO values per index (G ghosts each end)
  double *part, *dres;
  double *hres;   // pinned
  double *hpack;  // pinned, after hres: small boxes' five dense fields, else NULL
  int nblocks;  // of k3_resid
  bool stepped;
  std::vector<double> wid[3];
  int bc[3];
  double u_in;
};

namespace {
sts_status fail3(sts_status s, const char *msg) { return sts::report_error(s, msg); }

#define HIP3(call)                                                         \
  do {                                                                     \
    hipError_t e_ = (call);                                                \
    if (e_ != hipSuccess) {                                                \
      std::string m_ = std::string(#call) + " failed: " + hipGetErrorString(e_); \
      return fail3(STS_EDEVICE, m_.c_str());                               \
    }                                                                      \
  } while (0)

// as HIP3, for sts3_create after the context exists: releases it first
#define HIP3_CREATE(call)                                                  \
  do {                                                                     \
    hipError_t e_ = (call);                                                \
    if (e_ != hipSuccess) {                                                \
      std::string m_ = std::string(#call) + " failed: " + hipGetErrorString(e_); \
      sts3_destroy(c);                                                     \
      return fail3(STS_EDEVICE, m_.c_str());                               \
    }                                                                      \
  } while (0)

constexpr unsigned MAX_GRID = 65535;  // blocks of a launch along y and z
dim3 grid_of(const sts3_ctx *c, int X, int Y, int Z) {
  (void)c;
  return dim3((X + BX - 1) / BX, (Y + BY - 1) / BY, Z);
}
dim3 grid_face(const sts3_ctx *c, int a) {
  return grid_of(c, c->n[0] + (a == 0), c->n[1] + (a == 1), c->n[2] + (a == 2));
}

void launch_rf(sts3_ctx *c, const Fld &S, bool tv) {
  const dim3 b(BX, BY), gc = grid_of(c, c->n[0], c->n[1], c->n[2]);
  if (tv) hipLaunchKernelGGL(k3_rf<true>, gc, b, 0, c->stream, c->P, S, c->Wk);
  else hipLaunchKernelGGL(k3_rf<false>, gc, b, 0, c->stream, c->P, S, c->Wk);
}

// Per-step constants from S, and rho, Gamma and the face densities of S,
// which the first pass reads as those of its old iterate (EX, TV: explicit
// convective terms of that scheme; tvd: TVD face densities).  Three launches
// instead of eight, and two instead of six for the residual, take a step of
// 10 passes of 160x32x32 from 0.334 to 0.303 ms, of 512x128x128 from 8.36 to
// 8.00.
template <bool EX, bool TV>
void launch_prologue3(sts3_ctx *c, const Fld &S, bool tvd) {
  const dim3 b(BX, BY), gc = grid_of(c, c->n[0], c->n[1], c->n[2]);
  hipLaunchKernelGGL(k3_cell, gc, b, 0, c->stream, c->P, S, c->Wk);
  launch_rf(c, S, tvd);
  const bool tall = 4 * gc.z > MAX_GRID;
  hipLaunchKernelGGL((k3_const<EX, TV>), dim3(gc.x, tall ? 4 * gc.y : gc.y, tall ? gc.z : 4 * gc.z), b, 0,
                     c->stream, c->P, S, c->Wk, tall);
}

// increments and continuity residual of the last pass
void launch_resid3(sts3_ctx *c, const Fld &O, const Fld &N) {
  const dim3 b(BX, BY);
  hipLaunchKernelGGL(k3_resid, dim3(c->nblocks), b, 0, c->stream, c->P, O, N, c->Wk, c->part);
  hipLaunchKernelGGL(k3_resid_fold, dim3(1), b, 0, c->stream, c->part, c->nblocks, c->dres);
}

// One explicit pass from O to N as the two z-marching sweeps.  The planes of
// a block: as many as leave about `blocks` blocks (one and a half to three
// rounds of the chip, which holds 512 and 512), but at least two: each block
// first loads three planes (two in k3_sweep_pv), so shorter segments repeat
// more of that than the extra blocks gain.  Measured per pass on 512x128x128
// and 160x32x32: at least 2 planes 0.75 ms and 29 us, 1 plane 0.75 ms and
// 31 us, 4 planes 0.75 ms and 35 us; 512 blocks instead of 1024: 0.78 ms.
template <bool TV>
void launch_sweeps(sts3_ctx *c, const Fld &O, const Fld &N) {
  const int *n = c->n;
  auto segment = [&](int tiles, int blocks) {
    return (int)std::max<long>(2, std::min<long>((long)n[2] * tiles / blocks, n[2]));
  };
  int tx = (n[0] + MX - 1) / MX, ty = (n[1] + MY - 1) / MY, seg = segment(tx * ty, 1024);
  const dim3 g1(tx * ty * ((n[2] + seg - 1) / seg)), b1(MX, MY);
  const Sweep A{c->P, O, c->Wk, N.q[4], tx, ty, seg};
  hipLaunchKernelGGL((k3_sweep_eqs<TV>), g1, b1, 0, c->stream, A);
  tx = (n[0] + VX - 1) / VX, ty = (n[1] + VY - 1) / VY, seg = segment(tx * ty, 1536);
  const dim3 g2(tx * ty * ((n[2] + seg - 1) / seg)), b2(64, VY + 1);
  hipLaunchKernelGGL(k3_sweep_pv, g2, b2, 0, c->stream, c->P, O, N, c->Wk, tx, ty, seg);
}

// One pass from O to N.  rho, Gamma and the face densities of O are in Wk on
// entry (from the prologue, or the previous pass's pressure and velocity
// kernels); a pass other than the last leaves those of N there.
template <bool IM, bool TV>
void launch_pass3d(sts3_ctx *c, const Fld &O, const Fld &N, bool last) {
  if constexpr (!IM) {
    launch_sweeps<TV>(c, O, N);
    if (last && (c->P.per[0] || c->P.per[1] || c->P.per[2]))
      hipLaunchKernelGGL(k3_images,
                         grid_of(c, c->n[0] + 1 + 2 * G, c->n[1] + 1 + 2 * G,
                                 std::min<int>(c->n[2] + 1 + 2 * G, MAX_GRID)),
                         dim3(BX, BY), 0, c->stream, c->P, N, c->Wk);
  } else {
    const dim3 b(BX, BY), gc = grid_of(c, c->n[0], c->n[1], c->n[2]);
    hipLaunchKernelGGL((k3_edge<0>), grid_of(c, c->n[0], c->n[1] + 1, c->n[2] + 1), b, 0, c->stream,
                       c->P, c->Wk);
    hipLaunchKernelGGL((k3_edge<1>), grid_of(c, c->n[0] + 1, c->n[1], c->n[2] + 1), b, 0, c->stream,
                       c->P, c->Wk);
    hipLaunchKernelGGL((k3_edge<2>), grid_of(c, c->n[0] + 1, c->n[1] + 1, c->n[2]), b, 0, c->stream,
                       c->P, c->Wk);
    const dim3 ge = grid_of(c, c->n[0] + 1, c->n[1] + 1, c->n[2] + 1);
    hipLaunchKernelGGL(k3_eqs<TV>, ge, b, 0, c->stream, c->P, O, c->Wk, N.q[4]);
    hipLaunchKernelGGL(k3_pressure, gc, b, 0, c->stream, c->P, O, c->Wk, N.q[4], N.q[3]);
    if (last) {
      hipLaunchKernelGGL((k3_velocity<0, false, TV>), grid_face(c, 0), b, 0, c->stream, c->P, O, c->Wk, N.q[3], N.q[0]);
      hipLaunchKernelGGL((k3_velocity<1, false, TV>), grid_face(c, 1), b, 0, c->stream, c->P, O, c->Wk, N.q[3], N.q[1]);
      hipLaunchKernelGGL((k3_velocity<2, false, TV>), grid_face(c, 2), b, 0, c->stream, c->P, O, c->Wk, N.q[3], N.q[2]);
    } else {
      hipLaunchKernelGGL((k3_velocity<0, true, TV>), grid_face(c, 0), b, 0, c->stream, c->P, O, c->Wk, N.q[3], N.q[0]);
      hipLaunchKernelGGL((k3_velocity<1, true, TV>), grid_face(c, 1), b, 0, c->stream, c->P, O, c->Wk, N.q[3], N.q[1]);
      hipLaunchKernelGGL((k3_velocity<2, true, TV>), grid_face(c, 2), b, 0, c->stream, c->P, O, c->Wk, N.q[3], N.q[2]);
    }
  }
  if (last) launch_resid3(c, O, N);
}

size_t field_elems(const int n[3], long *pitch) {
  const long p = (long)((n[0] + 1 + 2 * G + 31) / 32) * 32;
  if (pitch) *pitch = p;
  return (size_t)p * (n[1] + 1 + 2 * G) * (n[2] + 1 + 2 * G);
}

// Host arrays are dense (x fastest, extents n + (f == e)), device fields
// padded: one contiguous copy to or from a device array, and a kernel that
// scatters or gathers.  On the host the five fields of 512 x 128 x 128 took
// 60 ms to read and as long to set, mostly page faults of a padded copy.
Ext ext_of(const sts3_ctx *c, int f) {
  return Ext{{c->n[0] + (f == 0), c->n[1] + (f == 1), c->n[2] + (f == 2)},
             {(int)c->pitch, c->n[1] + 1 + 2 * G, c->n[2] + 1 + 2 * G}};
}
size_t dense_bytes(const sts3_ctx *c, int f) {
  const Ext E = ext_of(c, f);
  return sizeof(double) * E.D[0] * E.D[1] * E.D[2];
}
size_t fields_bytes(const sts3_ctx *c) {
  size_t n = 0;
  for (int f = 0; f < 5; f++) n += dense_bytes(c, f);
  return n;
}
// Small boxes' fields are packed into pinned memory by the kernels themselves:
// a copy to pageable memory costs some 20 us whatever its size.
constexpr size_t PACK_MOST = 1u << 20;
dim3 rows_grid(int w, int h, int d) { return dim3((w + RWB - 1) / RWB, std::min(h, 4096), std::min(d, 4096)); }

// Both state buffers from host arrays (NULL keeps a field, or gives it its
// value of `init`), boundary values and ghosts included.
sts_status set_state3(sts3_ctx *c, const double *const q[5], const double *init) {
  const Fld &S = c->st[c->cur], &N = c->st[c->cur ^ 1];
  double *stage = c->Wk.qh[0];
  for (int f = 0; f < 5; f++) {
    const Ext E = ext_of(c, f);
    if (q[f])
      HIP3(hipMemcpyAsync(stage, q[f], sizeof(double) * E.D[0] * E.D[1] * E.D[2], hipMemcpyHostToDevice,
                          c->stream));
    hipLaunchKernelGGL(k3_impose, rows_grid(E.E[0], E.E[1], E.E[2]), dim3(RWB), 0, c->stream, c->P, f, E,
                       q[f] ? stage : nullptr, S.q[f], init != nullptr, init ? init[f] : 0.0, N.q[f]);
    HIP3(hipGetLastError());
    // both state buffers: faces that the passes do not write keep these values
    HIP3(hipMemcpyAsync(S.q[f], N.q[f], c->field_bytes, hipMemcpyDeviceToDevice, c->stream));
  }
  HIP3(hipMemsetAsync(stage, 0, c->field_bytes, c->stream));
  HIP3(hipStreamSynchronize(c->stream));
  return STS_OK;
}
constexpr int NFIELDS = 29;  // 2 states x 5, rho, gam, rf x3, qh x3, dq x3, cq x3, cT, cp, ge x3
}  // namespace

extern "C" sts_status sts3_device_bytes(const int n[3], size_t *bytes) {
  if (!n || !bytes) return fail3(STS_EINVAL, "NULL argument");
  for (int e = 0; e < 3; e++)
    if (n[e] < 4) return fail3(STS_EINVAL, "every direction needs >= 4 cells");
  const size_t fe = field_elems(n, nullptr);
  *bytes = NFIELDS * fe * sizeof(double);
  return STS_OK;
}

extern "C" void sts3_destroy(sts3_ctx *c) {
  if (!c) return;
  if (c->device >= 0) (void)hipSetDevice(c->device);
  if (c->stream) (void)hipStreamSynchronize(c->stream);
  for (void *p : c->allocs) (void)hipFree(p);
  if (c->hres) (void)hipHostFree(c->hres);
  if (c->own_stream && c->stream) (void)hipStreamDestroy(c->stream);
  delete c;
}

extern "C" sts_status sts3_create(const sts3_setup *s, void *hip_stream, sts3_ctx **out) {
  if (!s || !out) return fail3(STS_EINVAL, "NULL argument");
  for (int e = 0; e < 3; e++) {
    if (s->n[e] < 4) return fail3(STS_EINVAL, "every direction needs >= 4 cells");
    if (!s->d[e]) return fail3(STS_EINVAL, "cell widths missing");
    for (int i = 0; i < s->n[e]; i++)
      if (!(s->d[e][i] > 0) || !isfinite(s->d[e][i]))
        return fail3(STS_EINVAL, "cell widths must be positive and finite");
    const int bc = s->bc[e];
    if (e == 0 && bc != STS3_PERIODIC && bc != STS3_INLET_OUTLET)
      return fail3(STS_EINVAL, "x is inlet/outlet or periodic");
    if (e > 0 && bc != STS3_PERIODIC && bc != STS3_WALLS)
      return fail3(STS_EINVAL, "y and z are walls or periodic");
    for (int w = 0; w < 2; w++) {
      if (s->wall_type[e][w] != STS3_NOSLIP && s->wall_type[e][w] != STS3_SLIP)
        return fail3(STS_EINVAL, "unknown wall type");
      if (bc == STS3_WALLS && s->wall_type[e][w] == STS3_NOSLIP && !(s->wall_T[e][w] > 0))
        return fail3(STS_EINVAL, "wall temperatures must be > 0");
    }
  }
  if (!(s->Ma > 0) || !(s->Re > 0) || !(s->Pr > 0) || !(s->gamma > 1))
    return fail3(STS_EINVAL, "Ma, Re, Pr must be > 0 and gamma > 1");
  if (!(s->T_in > 0) || !(s->p_in > 0) || !isfinite(s->u_in))
    return fail3(STS_EINVAL, "T_in, p_in must be > 0 and u_in finite");
  size_t bytes = 0;
  sts_status st = sts3_device_bytes(s->n, &bytes);
  if (st != STS_OK) return st;

  sts3_ctx *c = new sts3_ctx();
  c->device = -1;
  c->hres = nullptr;
  c->stream = nullptr;
  c->own_stream = false;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    delete c;
    return fail3(STS_EDEVICE, "no HIP device");
  }
  c->device = dev;
  for (int e = 0; e < 3; e++) {
    c->n[e] = s->n[e];
    c->bc[e] = s->bc[e];
    c->wid[e].assign(s->d[e], s->d[e] + s->n[e]);
  }
  c->u_in = s->u_in;
  const size_t fe = field_elems(c->n, &c->pitch);
  c->sy = c->pitch;
  c->sz = c->pitch * (c->n[1] + 1 + 2 * G);
  c->off = (long)G * c->sz + (long)G * c->sy + G;
  c->field_bytes = fe * sizeof(double);
  auto alloc = [&](size_t b, void **p) -> bool {
    if (hipMalloc(p, b) != hipSuccess) return false;
    c->allocs.push_back(*p);
    return true;
  };
  std::vector<double *> fields(NFIELDS);
  for (int k = 0; k < NFIELDS; k++)
    if (!alloc(c->field_bytes, (void **)&fields[k])) {
      sts3_destroy(c);
      return fail3(STS_ENOMEM, "device allocation failed");
    }
  int k = 0;
  for (int b = 0; b < 2; b++)
    for (int f = 0; f < 5; f++) c->st[b].q[f] = fields[k++];
  c->Wk.rho = fields[k++];
  c->Wk.gam = fields[k++];
  for (int a = 0; a < 3; a++) c->Wk.rf[a] = fields[k++];
  for (int a = 0; a < 3; a++) c->Wk.qh[a] = fields[k++];
  for (int a = 0; a < 3; a++) c->Wk.dq[a] = fields[k++];
  for (int a = 0; a < 3; a++) c->Wk.cq[a] = fields[k++];
  c->Wk.cT = fields[k++];
  c->Wk.cp = fields[k++];
  for (int a = 0; a < 3; a++) c->Wk.ge[a] = fields[k++];
  for (int e = 0; e < 3; e++)
    if (!alloc(sizeof(double) * NGEO * (c->n[e] + 2 * G), (void **)&c->d_d[e])) {
      sts3_destroy(c);
      return fail3(STS_ENOMEM, "device allocation failed");
    }
  c->nblocks = (int)std::min<long>(RES_BLOCKS3, (long)((c->n[0] + BX - 1) / BX) * ((c->n[1] + BY - 1) / BY) *
                                                    c->n[2]);
  if (!alloc(sizeof(double) * NR * (size_t)c->nblocks, (void **)&c->part) ||
      !alloc(256, (void **)&c->dres) ||
      hipHostMalloc((void **)&c->hres, 256 + (fields_bytes(c) <= PACK_MOST ? fields_bytes(c) : 0)) != hipSuccess) {
    c->hres = nullptr;
    sts3_destroy(c);
    return fail3(STS_ENOMEM, "allocation failed");
  }
  c->hpack = fields_bytes(c) <= PACK_MOST ? c->hres + 32 : nullptr;
  if (hip_stream) {
    c->stream = (hipStream_t)hip_stream;
  } else {
    if (hipStreamCreate(&c->stream) != hipSuccess) {
      c->stream = nullptr;
      sts3_destroy(c);
      return fail3(STS_EDEVICE, "hipStreamCreate failed");
    }
    c->own_stream = true;
  }
  // parameters (eqs pl2-pl6 coefficients as in the 2-D library)
  P3 &P = c->P;
  memset(&P, 0, sizeof P);
  for (int e = 0; e < 3; e++) {
    P.n[e] = c->n[e];
    P.per[e] = s->bc[e] == STS3_PERIODIC;
    P.g[e] = s->g[e];
    P.geo[e] = c->d_d[e] + NGEO * G;
    for (int w = 0; w < 2; w++) {
      P.wt[e][w] = s->wall_type[e][w];
      P.wT[e][w] = s->wall_T[e][w];
      P.sqwT[e][w] = s->wall_T[e][w] > 0 ? sqrt(s->wall_T[e][w]) : 0.0;
      for (int v = 0; v < 3; v++) P.wv[e][w][v] = s->wall_vel[e][w][v];
    }
  }
  P.io = s->bc[0] == STS3_INLET_OUTLET;
  const double g = s->gamma;
  P.A = 1.0 / (g * s->Ma * s->Ma);
  P.B = 1.0 / s->Re;
  P.C1 = g / (s->Re * s->Pr);
  P.C2 = g * (g - 1.0) * s->Ma * s->Ma / s->Re;
  P.C3 = -(g - 1.0);
  P.u_in = s->u_in;
  P.T_in = s->T_in;
  P.p_in = s->p_in;
  P.rho_in = s->p_in / s->T_in;
  P.sqT_in = sqrt(s->T_in);
  P.sy = c->sy;
  P.sz = c->sz;
  P.off = c->off;
  // widths with G ghosts at each end: periodic images, or the end cell's
  for (int e = 0; e < 3; e++) {
    const int ne = c->n[e];
    auto width = [&](int i) {
      const int w = P.per[e] ? ((i % ne) + ne) % ne : std::min(std::max(i, 0), ne - 1);
      return c->wid[e][w];
    };
    std::vector<double> g;
    for (int i = -G; i < ne + G; i++) {
      const double dl = width(i - 1), d = width(i);
      g.push_back(d);
      g.push_back(1.0 / d);
      g.push_back(d / (dl + d));
      g.push_back(dl / (dl + d));
      g.push_back(2.0 / (dl + d));
    }
    HIP3_CREATE(hipMemcpy(c->d_d[e], g.data(), sizeof(double) * g.size(), hipMemcpyHostToDevice));
  }
  // clear every array (frame entries stay finite), then the initial state
  for (int k2 = 0; k2 < NFIELDS; k2++)
    HIP3_CREATE(hipMemsetAsync(fields[k2], 0, c->field_bytes, c->stream));
  c->cur = 0;
  c->stepped = false;
  const double *const none[5] = {};
  const double init[5] = {P.io ? s->u_in : 0.0, 0.0, 0.0, s->p_in, s->T_in};
  st = set_state3(c, none, init);
  if (st != STS_OK) {
    sts3_destroy(c);
    return st;
  }
  *out = c;
  return STS_OK;
}

extern "C" sts_status sts3_set_fields(sts3_ctx *c, const double *const q[5]) {
  if (!c || !q) return fail3(STS_EINVAL, "NULL argument");
  HIP3(hipSetDevice(c->device));
  const sts_status st = set_state3(c, q, nullptr);
  if (st != STS_OK) return st;
  c->stepped = false;
  return STS_OK;
}

extern "C" sts_status sts3_fields(sts3_ctx *c, double *const q[5]) {
  if (!c || !q) return fail3(STS_EINVAL, "NULL argument");
  HIP3(hipSetDevice(c->device));
  double *stage = c->Wk.qh[0];
  bool used = false;
  size_t at[5], end = 0;
  for (int f = 0; f < 5; f++) {
    if (!q[f]) continue;
    const Ext E = ext_of(c, f);
    const size_t bytes = dense_bytes(c, f);
    at[f] = end;
    end += bytes / sizeof(double);
    hipLaunchKernelGGL(k3_pack, rows_grid(E.D[0], E.D[1], E.D[2]), dim3(RWB), 0, c->stream, c->P, E,
                       c->st[c->cur].q[f], c->hpack ? c->hpack + at[f] : stage);
    HIP3(hipGetLastError());
    if (c->hpack) continue;
    sts::host_prefault(q[f], bytes);
    HIP3(hipMemcpyAsync(q[f], stage, bytes, hipMemcpyDeviceToHost, c->stream));
    used = true;
  }
  if (used) HIP3(hipMemsetAsync(stage, 0, c->field_bytes, c->stream));
  HIP3(hipStreamSynchronize(c->stream));
  for (int f = 0; c->hpack && f < 5; f++)
    if (q[f]) memcpy(q[f], c->hpack + at[f], dense_bytes(c, f));
  return STS_OK;
}

extern "C" sts_status sts3_step(sts3_ctx *c, double dt, int n_inner, int scheme) {
  if (!c) return fail3(STS_EINVAL, "ctx is NULL");
  if (!(dt > 0) || !isfinite(dt)) return fail3(STS_EINVAL, "dt must be > 0");
  if (n_inner < 1) return fail3(STS_EINVAL, "n_inner must be >= 1");
  if (scheme & ~(STS_IMPLICIT | STS_TVD)) return fail3(STS_EINVAL, "unknown scheme bits");
  HIP3(hipSetDevice(c->device));
  c->P.dt = dt;
  c->P.idt = 1.0 / dt;
  const bool im = scheme & STS_IMPLICIT, tv = scheme & STS_TVD;
  const Fld S0 = c->st[c->cur];
  if (im) launch_prologue3<false, false>(c, S0, tv);
  else if (tv) launch_prologue3<true, true>(c, S0, true);
  else launch_prologue3<true, false>(c, S0, false);
  for (int k = 0; k < n_inner; k++) {
    const Fld O = c->st[c->cur], N = c->st[c->cur ^ 1];
    const bool last = k == n_inner - 1;
    if (im && tv) launch_pass3d<true, true>(c, O, N, last);
    else if (im) launch_pass3d<true, false>(c, O, N, last);
    else if (tv) launch_pass3d<false, true>(c, O, N, last);
    else launch_pass3d<false, false>(c, O, N, last);
    c->cur ^= 1;
  }
  HIP3(hipGetLastError());
  HIP3(hipMemcpyAsync(c->hres, c->dres, NR * sizeof(double), hipMemcpyDeviceToHost, c->stream));
  c->stepped = true;
  return STS_OK;
}

extern "C" sts_status sts3_residuals(sts3_ctx *c, double out[7]) {
  if (!c || !out) return fail3(STS_EINVAL, "NULL argument");
  HIP3(hipSetDevice(c->device));
  HIP3(hipStreamSynchronize(c->stream));
  for (int k = 0; k < 7; k++) out[k] = c->stepped ? c->hres[k] : 0.0;
  if (c->stepped && c->hres[7] != 0.0) return fail3(STS_ENONFINITE, "the last step produced non-finite values");
  return STS_OK;
}
