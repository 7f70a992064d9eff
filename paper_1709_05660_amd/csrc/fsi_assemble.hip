// Device assembly of the finest residual and its exact Jacobian, and the
// Newton loop on the device (include/fsi_assembly.h).
//
// One workgroup per element of one colour.  The element residual's rows are
// sums over quadrature points of test functions weighted by a few coefficients
// per point, which depend on the element state through a few sums per point
// (gradients and values of the fields).  The workgroup differentiates the
// coefficients along each of these sums (one-direction dual numbers: value and
// derivative), so the element Jacobian is a product of the test-function
// table, the points' small tangent matrices and the table again; it is formed
// on the matrix cores and added into the CSR values at positions found once,
// when the assembly is created.  Elements of one colour share no node, so
// every entry is written once per launch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <memory>
#include <vector>

#include "../../include/fsi_assembly.h"
#include "fsi_internal.h"
#include "fsi_pivot.h"

namespace fsi {

// ------------------------------------------------------------ one-direction duals
struct D1 {
  double v, g;
};
__device__ __forceinline__ D1 dc(double c) { return {c, 0.0}; }
__device__ __forceinline__ D1 operator+(D1 a, D1 b) { return {a.v + b.v, a.g + b.g}; }
__device__ __forceinline__ D1 operator-(D1 a, D1 b) { return {a.v - b.v, a.g - b.g}; }
__device__ __forceinline__ D1 operator-(D1 a) { return {-a.v, -a.g}; }
__device__ __forceinline__ D1 operator*(D1 a, D1 b) { return {a.v * b.v, a.g * b.v + a.v * b.g}; }
__device__ __forceinline__ D1 operator*(double s, D1 b) { return {s * b.v, s * b.g}; }
__device__ __forceinline__ D1 operator+(D1 a, double c) { return {a.v + c, a.g}; }
__device__ __forceinline__ D1 operator/(D1 a, D1 b) {
  const double q = a.v / b.v;
  return {q, (a.g - q * b.g) / b.v};
}

struct AsmView {
  int ne, ndof, ncolor;
  const int *l2g, *tgt, *color_ptr, *color_elems, *rowptr, *col;
  const uint8_t *solid, *dir;
  const double *N, *dN, *psi, *w, *yprev;
  double vol, mu, rho, mu_s, dt, rho_s;
  int transient;
};

template <int DIM>
struct Shape {
  static constexpr int NA = DIM == 3 ? 27 : 9, NP = DIM + 1, NL = 2 * DIM * NA + NP, NQ = DIM == 3 ? 27 : 9;
};

// The sums over the element's nodes at one quadrature point: the reference
// gradients of displacement and velocity, velocity, displacement and
// pressure.
template <int DIM>
struct Sums {
  // per point: Gd[c][j], Gu[c][j], uq[c], dq[c], pq
  static constexpr int GD = 0, GU = DIM * DIM, UQ = 2 * DIM * DIM, DQ = UQ + DIM, PQ = DQ + DIM, NS = PQ + 1;
};

// sum s of point q for the element state ye; phi[q][a]: the node's reference
// gradient (two in 2D, then a zero) and its value
template <int DIM>
__device__ __forceinline__ double point_sum(const double *phi, const double *spsi, const double *ye, int q, int s) {
  constexpr int NA = Shape<DIM>::NA, NP = Shape<DIM>::NP;
  using S = Sums<DIM>;
  double acc = 0.0;
  if (s < S::PQ) {
    const int j = s < S::UQ ? s % DIM : 3;
    const int f = s < S::GU ? s / DIM : s < S::UQ ? DIM + (s - S::GU) / DIM : s < S::DQ ? DIM + s - S::UQ : s - S::DQ;
    const double *yc = ye + f * NA, *t = phi + q * NA * 4 + j;
    for (int a = 0; a < NA; ++a) acc += t[a * 4] * yc[a];
  } else {
    for (int j = 0; j < NP; ++j) acc += spsi[q * NP + j] * ye[2 * DIM * NA + j];
  }
  return acc;
}

// What follows from a point's sums without the direction of differentiation,
// once per point and state: det F, F^{-1} and, for the fluid, the velocity
// gradient in current coordinates gu = Gu F^{-1}.
template <int DIM>
struct Point {
  static constexpr int DET = 0, FI = 1, GC = FI + DIM * DIM, NP = GC + DIM * DIM;
};
template <int DIM>
__device__ __forceinline__ void point_kinematics(const double *S, bool fluid, double *out) {
  using SS = Sums<DIM>;
  using P = Point<DIM>;
  double F[DIM][DIM], Fi[DIM][DIM], det;
#pragma unroll
  for (int c = 0; c < DIM; ++c)
#pragma unroll
    for (int j = 0; j < DIM; ++j) F[c][j] = c == j ? S[SS::GD + c * DIM + j] + 1.0 : S[SS::GD + c * DIM + j];
  if constexpr (DIM == 2) {
    det = F[0][0] * F[1][1] - F[0][1] * F[1][0];
    Fi[0][0] = F[1][1] / det;
    Fi[1][1] = F[0][0] / det;
    Fi[0][1] = -(F[0][1] / det);
    Fi[1][0] = -(F[1][0] / det);
  } else {
    double cof[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const int i1 = (i + 1) % 3, i2 = (i + 2) % 3, j1 = (j + 1) % 3, j2 = (j + 2) % 3;
        cof[i][j] = F[i1][j1] * F[i2][j2] - F[i1][j2] * F[i2][j1];
      }
    det = F[0][0] * cof[0][0] + F[0][1] * cof[0][1] + F[0][2] * cof[0][2];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) Fi[i][j] = cof[j][i] / det;
  }
  out[P::DET] = det;
#pragma unroll
  for (int c = 0; c < DIM; ++c)
#pragma unroll
    for (int b = 0; b < DIM; ++b) {
      out[P::FI + c * DIM + b] = Fi[c][b];
      double g = 0.0;
      if (fluid)
#pragma unroll
        for (int j = 0; j < DIM; ++j) g += S[SS::GU + c * DIM + j] * Fi[j][b];
      out[P::GC + c * DIM + b] = g;
    }
}

// The fields of a point's state, read from its sums and kinematics.
template <int DIM>
struct Fields {
  const double *S, *K;
  using SS = Sums<DIM>;
  using P = Point<DIM>;
  __device__ __forceinline__ double det() const { return K[P::DET]; }
  __device__ __forceinline__ double Gd(int c, int j) const { return S[SS::GD + c * DIM + j]; }
  __device__ __forceinline__ double F(int c, int j) const { return c == j ? Gd(c, j) + 1.0 : Gd(c, j); }
  __device__ __forceinline__ double Fi(int c, int j) const { return K[P::FI + c * DIM + j]; }
  __device__ __forceinline__ double gu(int c, int j) const { return K[P::GC + c * DIM + j]; }
  __device__ __forceinline__ double u(int c) const { return S[SS::UQ + c]; }
  __device__ __forceinline__ double d(int c) const { return S[SS::DQ + c]; }
  __device__ __forceinline__ double p() const { return S[SS::PQ]; }
};
// The same differentiated along sum s.  Along the entry (m, n) of the
// displacement gradient F changes by a rank-one matrix: d det = det Fi[n][m],
// d Fi[i][j] = -Fi[i][m] Fi[n][j], d gu[i][j] = -gu[i][m] Fi[n][j]; along that
// of the velocity gradient d gu[m][j] = Fi[n][j].
template <int DIM>
struct DualFields {
  Fields<DIM> f;
  int s, m, n;
  bool gd, gv;
  using SS = Sums<DIM>;
  using P = Point<DIM>;
  double row[DIM], fi[DIM], gc[DIM], ddet;   // row n of F^{-1} and its factors
  __device__ __forceinline__ DualFields(const double *S, const double *K, int s_) : f{S, K}, s(s_) {
    gd = s < SS::GU;
    gv = !gd && s < SS::UQ;
    m = gd || gv ? (s % (DIM * DIM)) / DIM : 0;
    n = gd || gv ? s % DIM : 0;
    ddet = gd ? f.det() * f.Fi(n, m) : 0.0;
#pragma unroll
    for (int j = 0; j < DIM; ++j) {
      row[j] = f.Fi(n, j);
      fi[j] = gd ? -f.Fi(j, m) : 0.0;
      gc[j] = gd ? -f.gu(j, m) : gv && j == m ? 1.0 : 0.0;
    }
  }
  __device__ __forceinline__ D1 unit(double v, int i) const { return {v, s == i ? 1.0 : 0.0}; }
  __device__ __forceinline__ D1 det() const { return {f.det(), ddet}; }
  __device__ __forceinline__ D1 Gd(int c, int j) const { return unit(f.Gd(c, j), SS::GD + c * DIM + j); }
  __device__ __forceinline__ D1 F(int c, int j) const { return unit(f.F(c, j), SS::GD + c * DIM + j); }
  // (row c given apart: a runtime index into registers would go to memory)
  __device__ __forceinline__ D1 Fi(int c, int j) const { return {f.Fi(c, j), fi[c] * row[j]}; }
  __device__ __forceinline__ D1 gu(int c, int j) const { return {f.gu(c, j), gc[c] * row[j]}; }
  __device__ __forceinline__ D1 gu_row(int c, double gcc, int j) const { return {f.gu(c, j), gcc * row[j]}; }
  __device__ __forceinline__ D1 u(int c) const { return unit(f.u(c), SS::UQ + c); }
  __device__ __forceinline__ D1 d(int c) const { return unit(f.d(c), SS::DQ + c); }
  __device__ __forceinline__ D1 p() const { return unit(f.p(), SS::PQ); }
};

// structural coupling of local row lr with local column lc (the builder's rule)
__device__ __forceinline__ bool coupled_d(int dim, int na, bool solid, bool transient, int lr, int lc) {
  const int nd = dim * na;
  const int rblk = lr < nd ? 0 : (lr < 2 * nd ? 1 : 2);
  const int cblk = lc < nd ? 0 : (lc < 2 * nd ? 1 : 2);
  const int rc = (lr % nd) / na, cc = (lc % nd) / na;
  if (!solid) {
    if (rblk == 0) return true;
    if (rblk == 1) return cblk == 0 && rc == cc;
    return cblk != 2;
  }
  if (rblk == 0) return cblk != 1 || (transient && rc == cc);
  if (rblk == 1) return (cblk == 1 || (transient && cblk == 0)) && rc == cc;
  return cblk == 0;
}

// Every element residual row is a sum over the quadrature points of one test
// function (N_a, or psi_j for the pressure rows) and its reference gradient
// weighted by a few per-point coefficients: for the momentum rows of
// component c the coefficients of N_a and of dN_a/dX_j, likewise for the mesh
// motion (fluid) or kinematic (solid) rows, and one coefficient for the
// pressure rows.  Order: the coefficients of the gradient, then that of N_a
// (four in 2D too, one of them zero).
template <int DIM>
struct Terms {
  static constexpr int MOM = 0, MESH = DIM * 4, PR = 2 * DIM * 4, NK = PR + 1;
  // with a tangent of their own: the momentum and pressure coefficients (those
  // of the mesh motion and of the kinematics are linear in one sum)
  static constexpr int TPR = DIM * 4, NT = TPR + 1;
};
// groups of columns that share a field component (displacement, velocity,
// pressure): a column of node b sums its group's tangents along the gradient
// and the value, weighted by the node's table entries
template <int DIM>
struct Groups {
  static constexpr int NG = 2 * DIM + 1;
  static __device__ __forceinline__ int group(int s) {
    using S = Sums<DIM>;
    return s < S::GU ? s / DIM
           : s < S::UQ ? DIM + (s - S::GU) / DIM
           : s < S::DQ ? DIM + s - S::UQ
           : s < S::PQ ? s - S::DQ
                       : 2 * DIM;
  }
  static __device__ __forceinline__ int slot(int s) {
    using S = Sums<DIM>;
    return s < S::UQ ? s % DIM : s < S::PQ ? 3 : 0;
  }
};

// The coefficients of one point for the rows of component c (the pressure
// rows with c = 0): their derivatives along sum s (tan, stride 4 between
// coefficients) and, for vals not null, their values (the residual), the
// formulas of the host builder (steady, or one Crank-Nicolson step when cn,
// f0 then the state at t_n).
template <int DIM>
__device__ __forceinline__ void point_terms(const AsmView &v, bool solid, bool cn, const DualFields<DIM> &k1,
                                            const Fields<DIM> &k0, double w, int c, double *tan, double *vals) {
  using T = Terms<DIM>;
  const double dt = v.dt, rho = v.rho, mu = v.mu;
  auto put = [&](int j, D1 x) {   // momentum coefficient j
    tan[(c * 4 + j) * 4] = x.g;
    if (vals) vals[T::MOM + c * 4 + j] = x.v;
  };
  auto put_mesh = [&](int j, double x) {
    if (vals) vals[T::MESH + c * 4 + j] = x;
  };
  D1 S = dc(0.0), Pr;
  if (!solid) {
    const D1 wJ1 = w * k1.det();
    double gcc = k1.gc[0];
    D1 sig[DIM], guc[DIM];
#pragma unroll
    for (int b = 1; b < DIM; ++b) gcc = c == b ? k1.gc[b] : gcc;
#pragma unroll
    for (int b = 0; b < DIM; ++b) {
      guc[b] = k1.gu_row(c, gcc, b);
      // column c of gu: row b times entry c of the direction's row
      double rc = k1.row[0];
#pragma unroll
      for (int j = 1; j < DIM; ++j) rc = c == j ? k1.row[j] : rc;
      sig[b] = mu * (guc[b] + D1{k1.f.gu(b, c), k1.gc[b] * rc});
      if (b == c) sig[b] = sig[b] - k1.p();
    }
    if (!cn) {
      D1 t = dc(0.0);
#pragma unroll
      for (int b = 0; b < DIM; ++b) t = t + guc[b] * k1.u(b);
      S = rho * (wJ1 * t);
    } else {
      const double wJ0 = w * k0.det();
      D1 divw1 = dc(0.0), divw0 = dc(0.0);
#pragma unroll
      for (int i = 0; i < DIM; ++i)
#pragma unroll
        for (int j = 0; j < DIM; ++j) {
          const D1 Gw = (1.0 / dt) * k1.Gd(i, j) + (-k0.Gd(i, j) / dt);
          divw1 = divw1 + Gw * k1.Fi(j, i);
          divw0 = divw0 + k0.Fi(j, i) * Gw;
        }
      D1 t1 = -(divw1 * k1.u(c));
      D1 t2 = (-k0.u(c)) * divw0;
#pragma unroll
      for (int b = 0; b < DIM; ++b) {
        const D1 wq = (1.0 / dt) * k1.d(b) + (-k0.d(b) / dt);
        t1 = t1 + guc[b] * k1.u(b) - guc[b] * wq;
        t2 = t2 + k0.gu(c, b) * k0.u(b) + (-k0.gu(c, b)) * wq;
      }
      t1 = (0.5 * rho) * t1 + (rho / dt) * k1.u(c);
      t2 = (0.5 * rho) * t2 + (-(rho / dt) * k0.u(c));
      S = wJ1 * t1 + wJ0 * t2;
    }
    const double k_ale = 1.0 / v.vol;
#pragma unroll
    for (int j = 0; j < DIM; ++j) {
      D1 t = dc(0.0);
#pragma unroll
      for (int b = 0; b < DIM; ++b) t = t + sig[b] * k1.Fi(j, b);
      D1 Tm = wJ1 * t;
      if (cn) {
        double t0 = 0.0;
        const double wJ0 = w * k0.det();
#pragma unroll
        for (int b = 0; b < DIM; ++b) {
          double s0 = mu * (k0.gu(c, b) + k0.gu(b, c));
          if (b == c) s0 -= k0.p();
          t0 += s0 * k0.Fi(j, b);
        }
        Tm = 0.5 * Tm + 0.5 * wJ0 * t0;
      }
      put(j, Tm);
      put_mesh(j, (w * k_ale) * k1.f.Gd(c, j));
    }
    put(3, S);
    put_mesh(3, 0.0);
    if (c == 0) {
      D1 div = dc(0.0);
#pragma unroll
      for (int b = 0; b < DIM; ++b) div = div + k1.gu(b, b);
      Pr = wJ1 * div;
    }
  } else {
    // Piola stress J sigma F^{-T}, sigma = -p I + mu_s F F^T
    D1 sig[DIM];
    double sg0[DIM];
#pragma unroll
    for (int b = 0; b < DIM; ++b) {
      D1 t = dc(0.0);
#pragma unroll
      for (int j = 0; j < DIM; ++j) t = t + k1.F(c, j) * k1.F(b, j);
      sig[b] = v.mu_s * t;
      if (b == c) sig[b] = sig[b] - k1.p();
      if (cn) {
        double t0 = 0.0;
#pragma unroll
        for (int j = 0; j < DIM; ++j) t0 += k0.F(c, j) * k0.F(b, j);
        sg0[b] = v.mu_s * t0 - (b == c ? k0.p() : 0.0);
      }
    }
    const D1 det = k1.det();
#pragma unroll
    for (int b = 0; b < DIM; ++b) {
      D1 t = dc(0.0);
#pragma unroll
      for (int j = 0; j < DIM; ++j) t = t + sig[j] * k1.Fi(b, j);
      D1 Tm = det * t;
      if (cn) {
        double t0 = 0.0;
#pragma unroll
        for (int j = 0; j < DIM; ++j) t0 += sg0[j] * k0.Fi(b, j);
        Tm = 0.5 * (Tm + k0.det() * t0);
      }
      put(b, w * Tm);
      put_mesh(b, 0.0);
    }
    double A = k1.f.u(c);
    if (cn) {
      S = (v.rho_s / dt) * (det * k1.u(c) + (-k0.det() * k0.u(c)));
      A = (-1.0 / dt) * k1.f.d(c) + 0.5 * k1.f.u(c) + (k0.d(c) / dt + 0.5 * k0.u(c));
    }
    put(3, w * S);
    put_mesh(3, w * A);
    Pr = w * (det + (-1.0));
  }
  if (DIM == 2) {
    put(2, dc(0.0));
    put_mesh(2, 0.0);
  }
  if (c == 0) {
    tan[T::TPR * 4] = Pr.g;
    if (vals) vals[T::PR] = Pr.v;
  }
}

// Assembly of one element.  Phase 1: the point sums of the element state (and
// of the state at t_n) and what follows from them.  Phase 2: the tangents of
// every (point, sum, component) and the points' coefficients, into LDS.  Phase
// 3, the element Jacobian: each wave takes the columns of 16 nodes of one
// field component and the rows of one component at a time.  One point is one
// step of the 16x16x4 product: A holds the row node's table entries, B the
// tangents times the column node's, formed in registers (so the tangents are
// read from LDS, a few addresses per wave, and never multiplied out there).
// The entries' positions and present sums are loaded before the products.
// Rows or columns past the element's nodes repeat its last node and are
// dropped.
// A launch is a colour (256 of 2,048 elements in 3D, 1,024 of 4,096 in 2D), so
// one workgroup's latency bounds it in 3D: loads, sums, tangents (16 us with 8
// waves), then products whose 2,500 steps take 17 us of the FP64 matrix cores,
// and the scattered additions.  With 16 waves a launch takes 48 us (8 waves:
// 55, 12: 51) against 443 us for dual numbers along all 166 local dofs and a
// contraction on the vector units; in 2D 18 us against 39.  An assembly:
// 32x8x8 3,577 -> 408 us, 128x32 time step 158 -> 86 us.
template <int DIM, int NT, int WPS>
__global__ __launch_bounds__(NT, WPS) void k_assemble(AsmView v, const double *__restrict__ y, double *__restrict__ r,
                                                 double *__restrict__ jval, const int *__restrict__ map, int cbase) {
  constexpr int NA = Shape<DIM>::NA, NP = Shape<DIM>::NP, NL = Shape<DIM>::NL, NQ = Shape<DIM>::NQ;
  using S = Sums<DIM>;
  using T = Terms<DIM>;
  using G = Groups<DIM>;
  typedef Mfma16<double> MM;
  constexpr int NS = S::NS, NTL = (NA + 15) / 16, NG = G::NG;   // node tiles
  __shared__ double ye[NL], ye0[NL];
  __shared__ __align__(32) double phi[NQ * NA * 4];
  __shared__ double spsi[NQ * NP], sw[NQ];
  constexpr int NKIN = Point<DIM>::NP;
  __shared__ double sums[NQ * NS], sums0[NQ * NS], vals[NQ * T::NK], kin[NQ * NKIN], kin0[NQ * NKIN];
  __shared__ __align__(32) double tan[NQ * NG * T::NT * 4];
  const int e = v.color_elems[cbase + blockIdx.x];
  const bool solid = v.solid[e] != 0, transient = v.transient != 0;
  for (int i = threadIdx.x; i < NL; i += NT) {
    const int g = v.l2g[(int64_t)e * NL + i];
    ye[i] = y[g];
    ye0[i] = transient ? v.yprev[g] : 0.0;
  }
  for (int i = threadIdx.x; i < NQ * NA; i += NT) {
#pragma unroll
    for (int j = 0; j < 3; ++j) phi[i * 4 + j] = j < DIM ? v.dN[i * DIM + j] : 0.0;
    phi[i * 4 + 3] = v.N[i];
  }
  for (int i = threadIdx.x; i < NQ * NP; i += NT) spsi[i] = v.psi[i];
  for (int i = threadIdx.x; i < NQ; i += NT) sw[i] = v.w[i];
  if (DIM == 2)   // the third gradient slots stay zero
    for (int i = threadIdx.x; i < NQ * NG * T::NT * 4; i += NT) tan[i] = 0.0;
  __syncthreads();
  for (int i = threadIdx.x; i < NQ * NS; i += NT) {
    sums[i] = point_sum<DIM>(phi, spsi, ye, i / NS, i % NS);
    if (transient) sums0[i] = point_sum<DIM>(phi, spsi, ye0, i / NS, i % NS);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < (transient ? 2 : 1) * NQ; i += NT) {
    const int q = i % NQ;
    point_kinematics<DIM>((i < NQ ? sums : sums0) + q * NS, !solid, (i < NQ ? kin : kin0) + q * NKIN);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < NQ * NS * DIM; i += NT) {
    const int q = i % NQ, c = (i / NQ) % DIM, s = i / (NQ * DIM);
    const DualFields<DIM> k1(sums + q * NS, kin + q * NKIN, s);
    const Fields<DIM> k0{sums0 + q * NS, kin0 + q * NKIN};
    point_terms<DIM>(v, solid, transient, k1, k0, sw[q], c, tan + (q * NG + G::group(s)) * T::NT * 4 + G::slot(s),
                     s == 0 ? vals + q * T::NK : nullptr);
  }
  __syncthreads();
  for (int lr = threadIdx.x; lr < NL; lr += NT) {
    const int tr = v.tgt[(int64_t)e * NL + lr];
    if (tr < 0) continue;
    double acc = 0.0;
    if (lr < 2 * DIM * NA) {
      const double *t = phi + (lr % NA) * 4, *c = vals + (lr / NA) * 4;
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc += t[q * NA * 4 + j] * c[q * T::NK + j];
    } else {
      for (int q = 0; q < NQ; ++q) acc += spsi[q * NP + lr - 2 * DIM * NA] * vals[q * T::NK + T::PR];
    }
    r[tr] += acc;
  }
  const int lane = threadIdx.x & 63, jl = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int *emap = map + (int64_t)e * NL * NL;
  // a tile's entries: their positions (rows lr0 + 16 rt + .., nr rows in all; column lc or -1) and what is there
  struct Entries {
    int pos[4];
    double old[4];
  };
  auto positions = [&](int lr0, int rt, int nr, int lc, Entries &t) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int a = rt * 16 + MM::row(k, kq);
      t.pos[k] = a < nr && lc >= 0 ? emap[(lr0 + a) * NL + lc] : -1;
    }
  };
  auto load = [&](Entries &t) {
#pragma unroll
    for (int k = 0; k < 4; ++k) t.old[k] = jval[max(t.pos[k], 0)];
  };
  auto add = [&](const Entries &t, const dx4 &c, double f) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (t.pos[k] >= 0) jval[t.pos[k]] = t.old[k] + f * c[k];
  };
  const dx4 zero = {0, 0, 0, 0};
  // Items: 16 nodes' columns of a displacement or velocity component for the
  // rows of one momentum component or of the pressure, the pressure columns,
  // the mesh motion or kinematic rows of every component.
  constexpr int NC = 2 * DIM * NTL, NV = NC * DIM, NI = NV + DIM + DIM * NTL + NC;
  for (int it = wave; it < NI; it += NT / 64) {
    if (it < NV + DIM) {
      const bool prc = it >= NV;   // the pressure columns
      const int c = it % DIM, g = prc ? 2 * DIM : it / DIM / NTL, ct = prc ? 0 : it / DIM % NTL;
      if (solid && !prc && g >= DIM && !(transient && g - DIM == c)) continue;
      const int b = ct * 16 + jl, nb = prc ? NP : NA, bc = min(b, nb - 1);
      const int lc = b < nb ? (prc ? 2 * DIM * NA : g * NA) + b : -1;
      dx4 acc[NTL];
      Entries en[NTL];
#pragma unroll
      for (int rt = 0; rt < NTL; ++rt) {
        acc[rt] = zero;
        positions(c * NA, rt, NA, lc, en[rt]);
      }
#pragma unroll
      for (int rt = 0; rt < NTL; ++rt) load(en[rt]);
      const double *t = tan + (g * T::NT + c * 4 + kq) * 4;
      if (prc) {
        for (int q = 0; q < NQ; ++q) {
          const double x = t[q * NG * T::NT * 4] * spsi[q * NP + bc];
#pragma unroll
          for (int rt = 0; rt < NTL; ++rt)
            acc[rt] = MM::mma(phi[(q * NA + min(rt * 16 + jl, NA - 1)) * 4 + kq], x, acc[rt]);
        }
      } else {
        const double *pb = phi + bc * 4;
#pragma unroll 3
        for (int q = 0; q < NQ; ++q) {
          const double *tq = t + q * NG * T::NT * 4, *pq = pb + q * NA * 4;
          const double x = fma(tq[3], pq[3], fma(tq[2], pq[2], fma(tq[1], pq[1], tq[0] * pq[0])));
#pragma unroll
          for (int rt = 0; rt < NTL; ++rt)
            acc[rt] = MM::mma(phi[(q * NA + min(rt * 16 + jl, NA - 1)) * 4 + kq], x, acc[rt]);
        }
      }
#pragma unroll
      for (int rt = 0; rt < NTL; ++rt) add(en[rt], acc[rt], 1.0);
    } else if (it < NV + DIM + DIM * NTL) {
      // fluid: w / vol grad N_a . grad N_b in the displacement; solid: w N_a
      // N_b in the velocity and, in a time step, the displacement
      const int c = (it - NV - DIM) / NTL, ct = (it - NV - DIM) % NTL;
      const int b = ct * 16 + jl, bc = min(b, NA - 1);
      dx4 acc[NTL];
      Entries ed[NTL], eu[NTL];
#pragma unroll
      for (int rt = 0; rt < NTL; ++rt) {
        acc[rt] = zero;
        positions((DIM + c) * NA, rt, NA, b < NA && (!solid || transient) ? c * NA + b : -1, ed[rt]);
        positions((DIM + c) * NA, rt, NA, b < NA && solid ? (DIM + c) * NA + b : -1, eu[rt]);
      }
#pragma unroll
      for (int rt = 0; rt < NTL; ++rt) {
        load(ed[rt]);
        load(eu[rt]);
      }
      const bool on = solid ? kq == 3 : kq < DIM;
      const double k_ale = 1.0 / v.vol;
#pragma unroll 3
      for (int q = 0; q < NQ; ++q) {
        const double wq = solid ? sw[q] : sw[q] * k_ale;
        const double x = on ? wq * phi[(q * NA + bc) * 4 + kq] : 0.0;
#pragma unroll
        for (int rt = 0; rt < NTL; ++rt)
          acc[rt] = MM::mma(phi[(q * NA + min(rt * 16 + jl, NA - 1)) * 4 + kq], x, acc[rt]);
      }
#pragma unroll
      for (int rt = 0; rt < NTL; ++rt) {
        add(ed[rt], acc[rt], solid ? -1.0 / v.dt : 1.0);
        add(eu[rt], acc[rt], transient ? 0.5 : 1.0);
      }
    } else {
      // the pressure rows, four points a step
      const int g = (it - NV - DIM - DIM * NTL) / NTL, ct = (it - NV - DIM - DIM * NTL) % NTL;
      if (solid && g >= DIM) continue;
      const int b = ct * 16 + jl, bc = min(b, NA - 1);
      Entries en;
      positions(2 * DIM * NA, 0, NP, b < NA ? g * NA + b : -1, en);
      load(en);
      dx4 acc = zero;
#pragma unroll
      for (int q0 = 0; q0 < NQ; q0 += 4) {
        const bool ok = q0 + kq < NQ;
        const int q = min(q0 + kq, NQ - 1);
        const double *t = tan + ((q * NG + g) * T::NT + T::TPR) * 4, *pb = phi + (q * NA + bc) * 4;
        const double x = fma(t[3], pb[3], fma(t[2], pb[2], fma(t[1], pb[1], t[0] * pb[0])));
        acc = MM::mma(ok ? spsi[q * NP + min(jl, NP - 1)] : 0.0, ok ? x : 0.0, acc);
      }
      add(en, acc, 1.0);
    }
  }
}

// CSR position of every (element, local row, local column) entry of the
// element Jacobian that the assembly stores, else -1: rows without a target,
// Dirichlet rows and columns, and structurally uncoupled pairs are not stored.
__global__ void k_asm_map(AsmView v, int dim, int na, int nl, int64_t total, int *map) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const int64_t el = idx / nl;
  const int e = (int)(el / nl), lr = (int)(el % nl), jd = (int)(idx % nl);
  const int tr = v.tgt[(int64_t)e * nl + lr], gc = v.l2g[(int64_t)e * nl + jd];
  int pos = -1;
  if (tr >= 0 && !v.dir[tr] && !v.dir[gc] && coupled_d(dim, na, v.solid[e] != 0, v.transient != 0, lr, jd)) {
    int lo = v.rowptr[tr], hi = v.rowptr[tr + 1];
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (v.col[mid] < gc)
        lo = mid + 1;
      else
        hi = mid;
    }
    if (lo < v.rowptr[tr + 1] && v.col[lo] == gc) pos = lo;
  }
  map[idx] = pos;
}

// Dirichlet rows: r = y - g and a unit diagonal
__global__ void k_dirichlet_rows(const int *rows, const int *diag, int n, const double *y, const double *gval,
                                 double *r, double *jval) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= n) return;
  const int i = rows[t];
  r[i] = y[i] - gval[t];
  jval[diag[t]] = 1.0;
}
// Dirichlet dofs set to their values
__global__ void k_set_dirichlet(const int *rows, const double *gval, int n, double *y) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) y[rows[i]] = gval[i];
}

__global__ void k_neg_free(const double *r, const uint8_t *dir, int n, double *b) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) b[i] = dir[i] ? 0.0 : -r[i];
}

// device memory of the assembler: plain allocations owned here, freed when
// the assembler is destroyed or when its creation fails part way
struct AsmMem {
  std::vector<void *> v;
  AsmMem() = default;
  AsmMem(const AsmMem &) = delete;
  AsmMem &operator=(const AsmMem &) = delete;
  ~AsmMem() {
    if (!v.empty()) (void)hipDeviceSynchronize();   // no kernel of a failed creation still reads them
    for (void *p : v) (void)hipFree(p);
  }
  template <typename T>
  T *alloc(int64_t n) {
    void *p = nullptr;
    if (n <= 0) return nullptr;
    if (hipMalloc(&p, sizeof(T) * (size_t)n) != hipSuccess) throw Error(FSI_E_OOM, "device allocation");
    v.push_back(p);
    return static_cast<T *>(p);
  }
  template <typename T>
  T *up(const T *h, int64_t n) {
    T *d = alloc<T>(n);
    if (n > 0) hip_check(hipMemcpy(d, h, sizeof(T) * (size_t)n, hipMemcpyHostToDevice), "H2D");
    return d;
  }
};

struct Assembly {
  AsmView v{};
  int dim = 2, nnz = 0;
  std::vector<int> h_color_ptr;
  int ndir = 0;
  int *d_dir_rows = nullptr, *d_dir_diag = nullptr;
  double *d_dir_val = nullptr;
  double *b = nullptr, *x = nullptr, *r = nullptr, *partial = nullptr, *nrm = nullptr;
  double *yprev = nullptr;   // the state at t_n of a time step (the view reads it), else null
  int *map = nullptr;        // CSR positions of the element Jacobians' entries (ne x nl x nl), -1 if not stored
  AsmMem mem;
};

template <int DIM, int NT, int WPS>
static void launch_assemble_dim(Assembly &A, const double *y, double *r, double *jval, hipStream_t st) {
  for (int c = 0; c < A.v.ncolor; ++c) {
    const int n = A.h_color_ptr[c + 1] - A.h_color_ptr[c];
    if (n > 0) k_assemble<DIM, NT, WPS><<<n, NT, 0, st>>>(A.v, y, r, jval, A.map, A.h_color_ptr[c]);
  }
}

static void assemble(Assembly &A, const double *y, double *r, double *jval, hipStream_t st) {
  launch_fill_f64(r, A.v.ndof, 0.0, st);
  launch_fill_f64(jval, A.nnz, 0.0, st);
  if (A.dim == 2)
    launch_assemble_dim<2, 256, 4>(A, y, r, jval, st);   // 128 threads: 117 us per assembly, 192: 98, 384: 133
  else
    launch_assemble_dim<3, 1024, 4>(A, y, r, jval, st);
  if (A.ndir)
    k_dirichlet_rows<<<(A.ndir + 255) / 256, 256, 0, st>>>(A.d_dir_rows, A.d_dir_diag, A.ndir, y, A.d_dir_val, r,
                                                            jval);
  hip_check(hipGetLastError(), "assembly launch");
}

static Assembly *create(const fsi_element_data &ed, const fsi_csr &J, hipStream_t st) {
  if ((ed.dim != 2 && ed.dim != 3) || ed.ne < 1 || !ed.l2g || !ed.tgt || !ed.solid || !ed.color_ptr ||
      !ed.color_elems || !ed.N || !ed.dN || !ed.psi || !ed.w || !ed.dirichlet || !ed.dval)
    throw Error(FSI_E_INVALID, "element data incomplete");
  const int na = ed.dim == 3 ? 27 : 9, nl = 2 * ed.dim * na + ed.dim + 1, nq = ed.dim == 3 ? 27 : 9;
  if (ed.na != na || ed.nl != nl || ed.nq != nq || ed.np != ed.dim + 1 || J.nrows != ed.ndof || J.ncols != ed.ndof ||
      !J.rowptr || !J.colind || J.nnz >= ((int64_t)1 << 31) || ed.ndof >= ((int64_t)1 << 31))
    throw Error(FSI_E_INVALID, "element data and pattern sizes do not match");
  std::unique_ptr<Assembly> A(new Assembly());
  A->dim = ed.dim;
  A->nnz = (int)J.nnz;
  A->h_color_ptr.assign(ed.color_ptr, ed.color_ptr + ed.ncolor + 1);
  for (int64_t q = 0; q < (int64_t)ed.ne * nl; ++q)
    if (ed.l2g[q] < 0 || ed.l2g[q] >= ed.ndof || ed.tgt[q] < -1 || ed.tgt[q] >= ed.ndof)
      throw Error(FSI_E_INVALID, "element data: a dof out of range");
  if (A->h_color_ptr.front() != 0 || A->h_color_ptr.back() != ed.ne)
    throw Error(FSI_E_INVALID, "element data: colours do not list every element");
  AsmMem &M = A->mem;
  AsmView &v = A->v;
  v.ne = ed.ne;
  v.ndof = (int)ed.ndof;
  v.ncolor = ed.ncolor;
  v.l2g = M.up(ed.l2g, (int64_t)ed.ne * nl);
  v.tgt = M.up(ed.tgt, (int64_t)ed.ne * nl);
  v.color_ptr = M.up(ed.color_ptr, ed.ncolor + 1);
  v.color_elems = M.up(ed.color_elems, ed.ne);
  std::vector<int32_t> rp(J.nrows + 1);
  for (int64_t i = 0; i <= J.nrows; ++i) rp[i] = (int32_t)J.rowptr[i];
  v.rowptr = M.up(rp.data(), J.nrows + 1);
  v.col = M.up(J.colind, J.nnz);
  v.solid = M.up(ed.solid, ed.ne);
  v.dir = M.up(ed.dirichlet, ed.ndof);
  v.N = M.up(ed.N, (int64_t)nq * na);
  v.dN = M.up(ed.dN, (int64_t)nq * na * ed.dim);
  v.psi = M.up(ed.psi, (int64_t)nq * (ed.dim + 1));
  v.w = M.up(ed.w, nq);
  v.transient = ed.y_prev ? 1 : 0;
  A->yprev = ed.y_prev ? M.up(ed.y_prev, ed.ndof) : nullptr;
  v.yprev = A->yprev;
  v.vol = ed.vol;
  v.mu = ed.mu;
  v.rho = ed.rho;
  v.mu_s = ed.mu_s;
  v.dt = ed.dt;
  v.rho_s = ed.rho_s;
  std::vector<int> drows, ddiag;
  std::vector<double> dvals;
  for (int64_t i = 0; i < ed.ndof; ++i)
    if (ed.dirichlet[i]) {
      const int32_t *a = J.colind + J.rowptr[i], *b = J.colind + J.rowptr[i + 1];
      const int32_t *f = std::lower_bound(a, b, (int32_t)i);
      if (f == b || *f != i) throw Error(FSI_E_INVALID, "a Dirichlet row of the pattern holds no diagonal");
      drows.push_back((int)i);
      ddiag.push_back((int)(f - J.colind));
      dvals.push_back(ed.dval[i]);
    }
  A->ndir = (int)drows.size();
  A->d_dir_rows = M.up(drows.data(), (int64_t)drows.size());
  A->d_dir_diag = M.up(ddiag.data(), (int64_t)ddiag.size());
  A->d_dir_val = M.up(dvals.data(), (int64_t)dvals.size());
  const int n = (int)ed.ndof;
  A->b = M.alloc<double>(n);
  A->x = M.alloc<double>(n);
  A->r = M.alloc<double>(n);
  A->partial = M.alloc<double>(krylov_blocks(n));
  A->nrm = M.alloc<double>(4);
  const int64_t nmap = (int64_t)ed.ne * nl * nl;
  A->map = M.alloc<int>(nmap);
  k_asm_map<<<(unsigned)((nmap + 255) / 256), 256, 0, st>>>(v, ed.dim, na, nl, nmap, A->map);
  hip_check(hipGetLastError(), "assembly map");
  hip_check(hipStreamSynchronize(st), "assembly map");
  return A.release();
}

static double dev_norm(Assembly &A, const double *x, int n, hipStream_t st) {
  launch_kdot(n, x, n, 1, x, A.partial, A.nrm, st);
  double h = 0.0;
  hip_check(hipMemcpyAsync(&h, A.nrm, sizeof(double), hipMemcpyDeviceToHost, st), "D2H norm");
  hip_check(hipStreamSynchronize(st), "norm");
  return std::sqrt(h);
}

static fsi_status newton(Assembly &A, MG &mg, double *y, const fsi_newton_opts &no, const fsi_krylov_opts &ko,
                         fsi_newton_info *info, hipStream_t st) {
  Level &F = mg.lv.back();
  if (F.n != A.v.ndof || F.J.nnz != A.nnz) throw Error(FSI_E_INVALID, "the handle's finest pattern is not the assembly's");
  if (no.max_newton < 1 || !(no.tol > 0.0)) throw Error(FSI_E_INVALID, "invalid Newton options");
  fsi_newton_info inf{};
  const int n = A.v.ndof;
  fsi_status st_out = FSI_NOT_CONVERGED;
  for (int k = 0; k < no.max_newton; ++k) {
    assemble(A, y, A.r, F.J.val, st);   // the finest values go straight into the handle
    const double rn = dev_norm(A, A.r, n, st);
    if (k == 0) inf.res0 = rn;
    inf.res_last = rn;
    k_neg_free<<<(n + 255) / 256, 256, 0, st>>>(A.r, A.v.dir, n, A.b);
    galerkin(mg, st);
    refactor(mg, st);
    fsi_krylov_opts kk = ko;
    kk.x0_nonzero = 0;
    fsi_solve_info si{};
    const fsi_status s = fgmres(mg, A.b, A.x, kk, &si, st);
    if (s < 0) return s;
    inf.krylov_iters += si.iters;
    launch_axpy_f64(n, 1.0, A.x, y, st);
    const double en = dev_norm(A, A.x, n, st), yn = dev_norm(A, y, n, st);
    inf.steps = k + 1;
    inf.last_update = yn > 0 ? en / yn : en;
    if (en <= no.tol * yn) {
      inf.converged = 1;
      st_out = FSI_OK;
      break;
    }
  }
  if (info) *info = inf;
  return st_out;
}

// Crank-Nicolson steps: the current state becomes the state at t_n, Newton
// from it gives the state at t_{n+1}
static fsi_status cn_steps(Assembly &A, MG &mg, double *y, int nsteps, const fsi_newton_opts &no,
                           const fsi_krylov_opts &ko, fsi_newton_info *info, hipStream_t st) {
  if (!A.v.transient || !A.yprev) throw Error(FSI_E_INVALID, "the assembly holds no state at t_n (a steady problem)");
  if (nsteps < 1) throw Error(FSI_E_INVALID, "nsteps < 1");
  for (int k = 0; k < nsteps; ++k) {
    hip_check(hipMemcpyAsync(A.yprev, y, sizeof(double) * A.v.ndof, hipMemcpyDeviceToDevice, st), "state at t_n");
    fsi_newton_info inf{};
    const fsi_status r = newton(A, mg, y, no, ko, &inf, st);
    if (info) info[k] = inf;
    if (r != FSI_OK) return r;
  }
  return FSI_OK;
}

// full multigrid: Newton on each mesh, coarsest first, each mesh started from
// the prolongation of the previous mesh's iterate (relative to a base state
// that carries the boundary values, when one is given)
static fsi_status fmg(int nlev, Assembly *const *A, MG *const *M, double *const *y, const double *const *base,
                      const int32_t *caps, const fsi_newton_opts &no, const fsi_krylov_opts &ko,
                      fsi_newton_info *info, hipStream_t st) {
  for (int j = 0; j < nlev; ++j) {
    if (!A[j] || !M[j] || !y[j] || (base && !base[j])) throw Error(FSI_E_INVALID, "null handle or vector");
    if (caps && caps[j] < 1) throw Error(FSI_E_INVALID, "a Newton step limit below 1");
    if (M[j]->lv.back().n != A[j]->v.ndof) throw Error(FSI_E_INVALID, "a handle's finest size is not its assembly's");
    if (j > 0 && (M[j]->nlevels < 2 || M[j]->lv[M[j]->nlevels - 2].n != A[j - 1]->v.ndof))
      throw Error(FSI_E_INVALID, "mesh j-1 is not the level below the finest of handle j");
  }
  fsi_status out = FSI_NOT_CONVERGED;
  for (int j = 0; j < nlev; ++j) {
    Assembly &a = *A[j];
    MG &mg = *M[j];
    if (j > 0) {
      const Level &F = mg.lv.back();
      const int nc = A[j - 1]->v.ndof;
      if (base) launch_axpy_f64(nc, -1.0, base[j - 1], y[j - 1], st);
      launch_spmv(F.P.v64(), y[j - 1], (const double *)nullptr, y[j], kSpmvSet, F.P.lpr, st);
      if (base) {
        launch_axpy_f64(nc, 1.0, base[j - 1], y[j - 1], st);
        launch_axpy_f64(a.v.ndof, 1.0, base[j], y[j], st);
      }
      if (a.ndir) k_set_dirichlet<<<(a.ndir + 255) / 256, 256, 0, st>>>(a.d_dir_rows, a.d_dir_val, a.ndir, y[j]);
      hip_check(hipGetLastError(), "fmg prolongation");
    }
    fsi_newton_opts o = no;
    if (caps) o.max_newton = caps[j];
    fsi_newton_info inf{};
    const fsi_status s = newton(a, mg, y[j], o, ko, &inf, st);
    if (info) info[j] = inf;
    if (s < 0) return s;
    if (j + 1 == nlev) out = s;
  }
  return out;
}

}  // namespace fsi

using namespace fsi;

extern "C" {

fsi_status fsi_assembly_create(const fsi_element_data *ed, const fsi_csr *J, void *hip_stream,
                               struct fsi_assembly **out) {
  try {
    if (!ed || !J || !out) throw Error(FSI_E_INVALID, "null argument");
    *out = reinterpret_cast<fsi_assembly *>(create(*ed, *J, (hipStream_t)hip_stream));
    return FSI_OK;
  } catch (const Error &e) {
    set_error(e.msg);
    return e.code;
  }
}

fsi_status fsi_assembly_run(struct fsi_assembly *h, const double *y_dev, double *r_dev, double *jval_dev,
                            void *hip_stream) {
  try {
    Assembly *A = reinterpret_cast<Assembly *>(h);
    if (!A || !y_dev || !r_dev || !jval_dev) throw Error(FSI_E_INVALID, "null argument");
    assemble(*A, y_dev, r_dev, jval_dev, (hipStream_t)hip_stream);
    return FSI_OK;
  } catch (const Error &e) {
    set_error(e.msg);
    return e.code;
  }
}

fsi_status fsi_newton_solve(struct fsi_assembly *h, struct fsi_mg *mh, double *y_dev, const fsi_newton_opts *nopts,
                            const fsi_krylov_opts *kopts, fsi_newton_info *info, void *hip_stream) {
  try {
    Assembly *A = reinterpret_cast<Assembly *>(h);
    MG *mg = reinterpret_cast<MG *>(mh);
    if (!A || !mg || !y_dev || !nopts || !kopts) throw Error(FSI_E_INVALID, "null argument");
    hipStream_t st = hip_stream ? (hipStream_t)hip_stream : mg->own_stream;
    return newton(*A, *mg, y_dev, *nopts, *kopts, info, st);
  } catch (const Error &e) {
    set_error(e.msg);
    return e.code;
  }
}

fsi_status fsi_cn_steps(struct fsi_assembly *h, struct fsi_mg *mh, double *y_dev, int32_t nsteps,
                        const fsi_newton_opts *nopts, const fsi_krylov_opts *kopts, fsi_newton_info *info,
                        void *hip_stream) {
  try {
    Assembly *A = reinterpret_cast<Assembly *>(h);
    MG *mg = reinterpret_cast<MG *>(mh);
    if (!A || !mg || !y_dev || !nopts || !kopts) throw Error(FSI_E_INVALID, "null argument");
    hipStream_t st = hip_stream ? (hipStream_t)hip_stream : mg->own_stream;
    return cn_steps(*A, *mg, y_dev, nsteps, *nopts, *kopts, info, st);
  } catch (const Error &e) {
    set_error(e.msg);
    return e.code;
  }
}

fsi_status fsi_fmg_solve(int32_t nlev, struct fsi_assembly *const *a, struct fsi_mg *const *mg,
                         double *const *y_dev, const double *const *base_dev, const int32_t *max_newton,
                         const fsi_newton_opts *nopts, const fsi_krylov_opts *kopts, fsi_newton_info *info,
                         void *hip_stream) {
  try {
    if (nlev < 1 || !a || !mg || !y_dev || !nopts || !kopts) throw Error(FSI_E_INVALID, "null argument or nlev < 1");
    if (nopts->max_newton < 1 || !(nopts->tol > 0.0)) throw Error(FSI_E_INVALID, "invalid Newton options");
    hipStream_t st = hip_stream ? (hipStream_t)hip_stream : (mg[0] ? reinterpret_cast<MG *>(mg[0])->own_stream : nullptr);
    return fmg(nlev, reinterpret_cast<Assembly *const *>(a), reinterpret_cast<MG *const *>(mg), y_dev, base_dev,
               max_newton, *nopts, *kopts, info, st);
  } catch (const Error &e) {
    set_error(e.msg);
    return e.code;
  }
}

fsi_status fsi_assembly_destroy(struct fsi_assembly *h) {
  Assembly *A = reinterpret_cast<Assembly *>(h);
  if (!A) return FSI_OK;
  (void)hipDeviceSynchronize();
  delete A;   // frees its device memory
  return FSI_OK;
}

}  // extern "C"
