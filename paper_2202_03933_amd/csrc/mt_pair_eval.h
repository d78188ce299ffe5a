// Evaluation of one (slave, master) element pair, forward and backward, as
// device functions shared by the single-interface kernels and the persistent
// batched kernels.
//
// The clip polygon of a pair is computed once (k_pair_poly, in LDS) and
// stored structure-of-arrays in HBM with each vertex's provenance; the
// integration and its reverse mode read it from there, and use LDS only for
// what they need again after the quadrature (Stash) and for the sums per
// slave element.
//
// Quadrature works in the monomial basis m(xi) = (1, xi1, xi2, xi1 xi2) of
// the bilinear element: N(xi) = C m(xi) with C = H / 4,
//   H = [[1,-1,-1, 1], [1, 1,-1,-1], [1, 1, 1, 1], [1,-1, 1,-1]],
// (row k: (1, s1, s2, s1 s2), (s1, s2) the corner of node k), H H^T = 4 I.
// A quad's map x(xi) = sum_k N_k(xi) X_k = c + e1 xi1 + e2 xi2 + f xi1 xi2
// has coefficients (c, e1, e2, f) = C^T X and nodes X = H (c, e1, e2, f).
#pragma once

#include "mt_geometry.h"
#include "mt_internal.h"

namespace mt {

// Triangle rules as (l0, l1, l2, w) rows, barycentric coordinates with
// weights summing to one: 7 points of degree 5 (Radon's rule) and 3 points of
// degree 2 (the rule of Fig. 1).  The point index is uniform across a
// wavefront, so reads are scalar constant-cache loads.
__constant__ double c_rule7[7][4] = {
    {1.0 / 3.0, 1.0 / 3.0, 1.0 / 3.0, 9.0 / 40.0},
    {0.7974269853530873, 0.10128650732345634, 0.10128650732345634, 0.12593918054482714},
    {0.10128650732345634, 0.7974269853530873, 0.10128650732345634, 0.12593918054482714},
    {0.10128650732345634, 0.10128650732345634, 0.7974269853530873, 0.12593918054482714},
    {0.05971587178976982, 0.4701420641051151, 0.4701420641051151, 0.1323941527885062},
    {0.4701420641051151, 0.05971587178976982, 0.4701420641051151, 0.1323941527885062},
    {0.4701420641051151, 0.4701420641051151, 0.05971587178976982, 0.1323941527885062}};
__constant__ double c_rule3[3][4] = {{2.0 / 3.0, 1.0 / 6.0, 1.0 / 6.0, 1.0 / 3.0},
                                     {1.0 / 6.0, 2.0 / 3.0, 1.0 / 6.0, 1.0 / 3.0},
                                     {1.0 / 6.0, 1.0 / 6.0, 2.0 / 3.0, 1.0 / 3.0}};

template <int NQ>
__device__ __forceinline__ void rule_point(int q, double& l0, double& l1, double& l2, double& w) {
  const double* r = NQ == 3 ? c_rule3[q] : c_rule7[q];
  l0 = r[0];
  l1 = r[1];
  l2 = r[2];
  w = r[3];
}

// ---- clip polygons in HBM (layout: PolyBuf) ------------------------------------
struct GPoly {
  const double* __restrict__ u;
  const double* __restrict__ v;
  const uint8_t* __restrict__ l;
  int64_t stride, p;
  __device__ __forceinline__ double U(int i) const { return u[(int64_t)i * stride + p]; }
  __device__ __forceinline__ double V(int i) const { return v[(int64_t)i * stride + p]; }
  __device__ __forceinline__ uint8_t L(int i) const { return l[(int64_t)i * stride + p]; }
};

// Polygon of pair p (at its entry of the buffer).
__device__ __forceinline__ GPoly gpoly(const PolyBuf& b, int64_t p) {
  return GPoly{b.u, b.v, b.lab, b.stride, b.at(p)};
}
__device__ __forceinline__ uint8_t gpoly_nf(const PolyBuf& b, int64_t p) { return b.nf[b.at(p)]; }

// Writes a clip polygon (n vertices) and its provenance to entry idx of a
// polygon buffer.
__device__ __forceinline__ void poly_store(const RegPoly& q, int n, bool flip, const PolyBuf& out, int64_t idx) {
  out.nf[idx] = (uint8_t)(n | (flip ? 0x80 : 0));
#pragma unroll
  for (int i = 0; i < CAP0; ++i)
    if (i < n) {
      out.u[(int64_t)i * out.stride + idx] = q.u[i];
      out.v[(int64_t)i * out.stride + idx] = q.v[i];
      out.lab[(int64_t)i * out.stride + idx] = (uint8_t)q.lab[i];
    }
}

// Frame, projection, orientation, clip and cleanup of pair p; stores the
// polygon and its provenance.  Returns the clip status bits (PS_*), with
// PS_LOST when the polygon is no longer a segment at these coordinates (the
// pair then contributes nothing).
__device__ __forceinline__ int store_pair_polygon(const double Xs[4][3], const double Xm[4][3], const double* ns,
                                                   const KParams& kp, const LdsPoly& P, const PolyBuf& out,
                                                   int64_t p) {
  double f[12];
  slave_frame_p(Xs, ns, f);
  RegPoly q;
  int st;
  bool flip;
  const int n = pair_geometry(Xs, Xm, f, kp.eps_d, kp.eps_a, flip, P, q, st);
  poly_store(q, n, flip, out, out.at(p));
  return st | (n >= 3 ? 0 : PS_LOST);
}

// ---- monomial basis helpers ------------------------------------------------------

// y = H x
__device__ __forceinline__ void h_apply(const double x[4], double y[4]) {
  const double am = x[0] - x[2], ap = x[0] + x[2], bm = x[1] - x[3], bp = x[1] + x[3];
  y[0] = am - bm;
  y[1] = am + bm;
  y[2] = ap + bp;
  y[3] = ap - bp;
}
// y = H^T x
__device__ __forceinline__ void ht_apply(const double x[4], double y[4]) {
  const double s03 = x[0] + x[3], s12 = x[1] + x[2];
  y[0] = s03 + s12;
  y[1] = s12 - s03;
  y[2] = (x[2] + x[3]) - (x[0] + x[1]);
  y[3] = (x[0] + x[2]) - (x[1] + x[3]);
}
// Y = s H X H^T for a row-major 4x4 X.
__device__ __forceinline__ void h_sandwich(const double X[16], double s, double Y[16]) {
  double T[16];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const double col[4] = {X[c], X[4 + c], X[8 + c], X[12 + c]};
    double y[4];
    h_apply(col, y);
#pragma unroll
    for (int r = 0; r < 4; ++r) T[r * 4 + c] = y[r];
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    double y[4];
    h_apply(T + 4 * r, y);
#pragma unroll
    for (int k = 0; k < 4; ++k) Y[r * 4 + k] = s * y[k];
  }
}
// Y = s H^T X H for a row-major 4x4 X.
__device__ __forceinline__ void ht_sandwich(const double X[16], double s, double Y[16]) {
  double T[16];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const double col[4] = {X[c], X[4 + c], X[8 + c], X[12 + c]};
    double y[4];
    ht_apply(col, y);
#pragma unroll
    for (int r = 0; r < 4; ++r) T[r * 4 + c] = y[r];
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    double y[4];
    ht_apply(T + 4 * r, y);
#pragma unroll
    for (int k = 0; k < 4; ++k) Y[r * 4 + k] = s * y[k];
  }
}

// Launders an index so that loads through it are not merged with earlier
// loads of the same address (the values are reloaded instead of being kept
// in registers across the quadrature loop).
__device__ __forceinline__ int launder(int i) {
  asm volatile("" : "+v"(i));
  return i;
}

// Reciprocal: hardware estimate refined by two Newton-Raphson steps.
__device__ __forceinline__ double rcp_nr(double d) {
#pragma clang fp contract(fast)
  double r = __builtin_amdgcn_rcp(d);
  r = fma(r, fma(-d, r, 1.0), r);
  r = fma(r, fma(-d, r, 1.0), r);
  return r;
}

// Map coefficients (c, e1, e2, f) of a projected quad.
struct QMap {
  double cu, cv, e1u, e1v, e2u, e2v, fu, fv;
};

__device__ __forceinline__ QMap qmap(const V2 X[4]) {
#pragma clang fp contract(fast)
  QMap m;
  m.cu = 0.25 * ((X[0].u + X[1].u) + (X[2].u + X[3].u));
  m.cv = 0.25 * ((X[0].v + X[1].v) + (X[2].v + X[3].v));
  m.e1u = 0.25 * ((X[1].u - X[0].u) + (X[2].u - X[3].u));
  m.e1v = 0.25 * ((X[1].v - X[0].v) + (X[2].v - X[3].v));
  m.e2u = 0.25 * ((X[2].u - X[1].u) + (X[3].u - X[0].u));
  m.e2v = 0.25 * ((X[2].v - X[1].v) + (X[3].v - X[0].v));
  m.fu = 0.25 * ((X[0].u - X[1].u) + (X[2].u - X[3].u));
  m.fv = 0.25 * ((X[0].v - X[1].v) + (X[2].v - X[3].v));
  return m;
}

// Inverse bilinear map in scaled form.  With d = p - c and the cross product
// a x b = au bv - av bu, x(xi) = p means
//   (e1 x f) xi1^2 + (J0 - d x f) xi1 - d x e2 = 0,
//   (e2 x f) xi2^2 - (J0 + d x f) xi2 - d x e1 = 0,   J0 = e1 x e2,
// and the Jacobian's determinant at the solution is the root of the common
// discriminant with the sign of J0.  Divided by J0, with
//   al = (e1 x f) / J0, be = (e2 x f) / J0, t1 = d x e2 / J0,
//   t2 = e1 x d / J0, b1 = 1 - d x f / J0, b2 = 2 - b1:
//   D = sqrt(b1^2 + 4 al t1),  xi1 = 2 t1 / (b1 + D),  xi2 = 2 t2 / (b2 + D),
// det J = J0 D.  (b1 + D) / 2 and (b2 + D) / 2 are the determinants at
// (0, xi2) and (xi1, 0) over J0, so on a convex quad nothing cancels.
// The vectors are kept times 2 / J0: t1, t2 come out doubled.
//
// On a convex quad (the determinants at its corners, J0 (1 +- al +- be), have
// the sign of J0) the root with that sign is the only one in the element.
// Where a corner is reentrant the map folds inside the element, both roots
// can lie in it, and the one meant is the one that Newton's method reaches
// from the centre: a2 is then NaN, and no test lets the closed form through.
struct IMap {
  double cu, cv, e1u, e1v, e2u, e2v, fu, fv;  // c; 2 e1 / J0, 2 e2 / J0, 2 f / J0
  double a2;                                  // 2 al (convex_a2)
  double j0;                                  // J0
};

// The slave quad's map, with its centre as the origin (c = 0).
struct SMap {
  double e1u, e1v, e2u, e2v, fu, fv, a2, j0;
};

// 2 al from e1, e2 as they are and f times 2 / J0.
__device__ __forceinline__ double convex_a2(double e1u, double e1v, double e2u, double e2v, double fu, double fv) {
#pragma clang fp contract(fast)
  const double a2 = e1u * fv - e1v * fu, b2 = e2u * fv - e2v * fu;
  return fabs(a2) + fabs(b2) < 2.0 ? a2 : __builtin_nan("");
}

// Node k of a quad from its scaled map.
__device__ __forceinline__ V2 map_node(const IMap& m, int k) {
#pragma clang fp contract(fast)
  const double h = 0.5 * m.j0;
  const double h1 = (k == 1 || k == 2) ? h : -h;
  const double h2 = k >= 2 ? h : -h;
  const double h12 = (k & 1) ? -h : h;
  return V2{m.cu + h1 * m.e1u + h2 * m.e2u + h12 * m.fu, m.cv + h1 * m.e1v + h2 * m.e2v + h12 * m.fv};
}
__device__ __forceinline__ IMap widen(const SMap& m) {
  return IMap{0.0, 0.0, m.e1u, m.e1v, m.e2u, m.e2v, m.fu, m.fv, m.a2, m.j0};
}

// The scalars of one point's two quadratic equations (t1, t2 doubled).
struct IPoint {
  double t1, t2, b1, b2;
};

__device__ __forceinline__ IPoint ipoint(const IMap& m, double pu, double pv) {
#pragma clang fp contract(fast)
  const double du = pu - m.cu, dv = pv - m.cv;
  IPoint p;
  p.t1 = du * m.e2v - dv * m.e2u;
  p.t2 = dv * m.e1u - du * m.e1v;
  const double q = du * m.fv - dv * m.fu;
  p.b1 = 1.0 - 0.5 * q;
  p.b2 = 1.0 + 0.5 * q;
  return p;
}
__device__ __forceinline__ IPoint ipoint(const SMap& m, double pu, double pv) {
#pragma clang fp contract(fast)
  IPoint p;
  p.t1 = pu * m.e2v - pv * m.e2u;
  p.t2 = pv * m.e1u - pu * m.e1v;
  const double q = pu * m.fv - pv * m.fu;
  p.b1 = 1.0 - 0.5 * q;
  p.b2 = 1.0 + 0.5 * q;
  return p;
}

// Newton's method from xi = 0 on the same scalars: at most maxit steps, the
// first with the Jacobian at 0; stops once the next step is at most tol in
// both components, tested without the division.  rd = J0 / det J.
template <class Map>
__device__ __forceinline__ void inverse_newton(const Map& m, const IPoint& p, double tol, int maxit, double& x1,
                                               double& x2, double& rd, unsigned& noconv) {
#pragma clang fp contract(fast)
  const double h = 0.25 * m.j0;
  const double al = h * (m.e1u * m.fv - m.e1v * m.fu), be = h * (m.e2u * m.fv - m.e2v * m.fu);
  const double t1 = 0.5 * p.t1, t2 = 0.5 * p.t2;
  x1 = t1;
  x2 = t2;
  bool conv = false;
  for (int it = 1; it < maxit && !conv; ++it) {
    const double det = 1.0 + al * x1 - be * x2;
    const double n1 = (al * x1 + p.b1) * x1 - t1;
    const double n2 = (p.b2 - be * x2) * x2 - t2;
    conv = fmax(fabs(n1), fabs(n2)) <= tol * fabs(det);
    if (conv) break;
    const double r = rcp_nr(det);
    x1 -= n1 * r;
    x2 -= n2 * r;
  }
  rd = rcp_nr(1.0 + al * x1 - be * x2);
  noconv += conv ? 0u : 1u;
}

// sqrt(a) and 1 / sqrt(a) of a positive a from the hardware estimate y of
// the latter: with e = 1 - a y^2, 1 / sqrt(a) = y (1 + e / 2 + 3 e^2 / 8 + O(e^3)).
__device__ __forceinline__ void sqrt_rsqrt(double a, double& root, double& rroot) {
#pragma clang fp contract(fast)
  const double y = __builtin_amdgcn_rsq(a);
  const double t = a * y;
  const double e = fma(-t, y, 1.0);
  const double q = e * fma(0.375, e, 0.5);
  root = fma(t, q, t);
  rroot = fma(y, q, y);
}

// 1 / d from the hardware estimate r: with e = 1 - d r, 1 / d = r (1 + e + e^2 + O(e^3)).
__device__ __forceinline__ double rcp3(double d) {
#pragma clang fp contract(fast)
  const double r = __builtin_amdgcn_rcp(d);
  const double e = fma(-d, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// Points whose squared determinant over that at the centre, or product of
// denominators (4 on a parallelogram), is not above this bound are left to
// Newton's method: rounding of the solution grows with the reciprocal of the
// determinant, and from about 1/32 on the iteration reports it.
constexpr double INV_MIN = 0x1p-10;

// Inverse bilinear maps of point p on the slave quad (a) and the master quad
// (b), and rda, rdb = J0 / det J there.  Closed form when kp.direct (a
// tolerance no tighter than its rounding error and at least the default
// number of steps allowed) and both quads are convex: 54 FP64 instructions and three estimates for
// both maps, where Newton's interleaved loop took about 35 per map and step
// and a wavefront as many steps as its slowest lane.  Wavy 1024 x 1024 /
// 777 x 777 (3.24M pairs, alone): forward 0.60 -> 0.38 ms, reverse sweep
// 0.95 -> 0.76 ms; 64 batched interfaces (13M pairs): forward and backward
// 9.35 -> 6.79 ms.  Newton's method for tighter settings, other quads and
// points near a fold of the map.  Maps that do not converge are counted in
// noconv.
__device__ __forceinline__ void inverse2(const SMap& A, const IMap& B, double pu, double pv, const KParams& kp,
                                         double& a1, double& a2, double& b1, double& b2, double& rda, double& rdb,
                                         unsigned& noconv) {
#pragma clang fp contract(fast)
  const IPoint pa = ipoint(A, pu, pv), pb = ipoint(B, pu, pv);
  const double sa = pa.b1 * pa.b1 + A.a2 * pa.t1, sb = pb.b1 * pb.b1 + B.a2 * pb.t1;
  double da, db;
  sqrt_rsqrt(sa, da, rda);
  sqrt_rsqrt(sb, db, rdb);
  const double ga = pa.b1 + da, ha = pa.b2 + da, gb = pb.b1 + db, hb = pb.b2 + db;
  const double ma = ga * ha, mb = gb * hb;
  const double r = rcp3(ma * mb);
  const double ra = r * mb, rb = r * ma;
  a1 = pa.t1 * (ha * ra);
  a2 = pa.t2 * (ga * ra);
  b1 = pb.t1 * (hb * rb);
  b2 = pb.t2 * (gb * rb);
  const bool ok = kp.direct && sa > INV_MIN && sb > INV_MIN && ma > INV_MIN && mb > INV_MIN;
  if (!ok) {
    inverse_newton(A, pa, kp.newton_tol, kp.newton_maxit, a1, a2, rda, noconv);
    inverse_newton(B, pb, kp.newton_tol, kp.newton_maxit, b1, b2, rdb, noconv);
  }
}

// The same for the master quad alone.
__device__ __forceinline__ void inverse1(const IMap& B, double pu, double pv, const KParams& kp, double& b1,
                                         double& b2, unsigned& noconv) {
#pragma clang fp contract(fast)
  const IPoint pb = ipoint(B, pu, pv);
  const double sb = pb.b1 * pb.b1 + B.a2 * pb.t1;
  double db, rdb;
  sqrt_rsqrt(sb, db, rdb);
  const double gb = pb.b1 + db, hb = pb.b2 + db;
  const double mb = gb * hb;
  const double r = rcp3(mb);
  b1 = pb.t1 * (hb * r);
  b2 = pb.t2 * (gb * r);
  if (!(kp.direct && sb > INV_MIN && mb > INV_MIN))
    inverse_newton(B, pb, kp.newton_tol, kp.newton_maxit, b1, b2, rdb, noconv);
}

// ---- plane and maps of one pair ---------------------------------------------------
// The axes are the search's, evaluated in its order: the stored polygons are
// in them, at small elements far from the origin its g1 and g2 (sums of
// coordinates) are rounded well above an element's own rounding, and the
// heights of distant surfaces feel a tilt of the normal.  The lengths and
// quotients come from a refined reciprocal square root instead of IEEE
// square roots and divisions (about 60 instructions against 200), and each
// quad is projected through its four map coefficients.

// a = v / |v|: the reciprocal square root's root and each quotient corrected
// by its residual (the rounded values of the IEEE operations, up to rare ties).
__device__ __forceinline__ void unit3(const double v[3], double a[3]) {
  const double q = (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2];
  double l, rl;
  sqrt_rsqrt(q, l, rl);
  l = fma(fma(-l, l, q), 0.5 * rl, l);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double t = v[d] * rl;
    a[d] = fma(fma(-t, l, v[d]), rl, t);
  }
}

// The axes R = (t1, t2, n0) of the slave plane; ns: the plane normal of the
// continuous field, else null.
__device__ __forceinline__ void plane_axes(const double X[4][3], const double* ns, double R[3][3]) {
  double g1[3], g2[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    g1[d] = 0.25 * (((X[1][d] - X[0][d]) + X[2][d]) - X[3][d]);
    g2[d] = 0.25 * (((X[2][d] + X[3][d]) - X[0][d]) - X[1][d]);
  }
  if (ns) {
#pragma unroll
    for (int d = 0; d < 3; ++d) R[2][d] = ns[d];
    const double gn = (g1[0] * ns[0] + g1[1] * ns[1]) + g1[2] * ns[2];
#pragma unroll
    for (int d = 0; d < 3; ++d) g1[d] = g1[d] - gn * ns[d];
  } else {
    const double n[3] = {g1[1] * g2[2] - g1[2] * g2[1], g1[2] * g2[0] - g1[0] * g2[2], g1[0] * g2[1] - g1[1] * g2[0]};
    unit3(n, R[2]);
  }
  unit3(g1, R[0]);
  R[1][0] = R[2][1] * R[0][2] - R[2][2] * R[0][1];
  R[1][1] = R[2][2] * R[0][0] - R[2][0] * R[0][2];
  R[1][2] = R[2][0] * R[0][1] - R[2][1] * R[0][0];
}

// Map coefficients (c, e1, e2, f) of a quad in space, relative to the point
// o.  The nodes are taken relative to it first: these differences are exact
// to rounding of an element's size, sums of the coordinates are not.
__device__ __forceinline__ void coefficients(const double X[4][3], const double o[3], double C[4][3]) {
#pragma clang fp contract(fast)
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double x0 = X[0][d] - o[d], x1 = X[1][d] - o[d], x2 = X[2][d] - o[d], x3 = X[3][d] - o[d];
    C[0][d] = 0.25 * ((x0 + x1) + (x2 + x3));
    C[1][d] = 0.25 * ((x1 - x0) + (x2 - x3));
    C[2][d] = 0.25 * ((x2 - x1) + (x3 - x0));
    C[3][d] = 0.25 * ((x0 - x1) + (x2 - x3));
  }
}

__device__ __forceinline__ double dot3(const double a[3], const double b[3]) {
#pragma clang fp contract(fast)
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}
// The slave plane's axes R = (t1, t2, n0), the maps of the projected quads
// and the heights' coefficients (slave: of e1, e2, f; its centre has height
// 0).  ns: the plane normal of the continuous field, else null.  The stored
// polygons are relative to the rounded centre x0 of the search; the maps are
// relative to the centre itself, (ou, ov) in the polygons' coordinates.
__device__ __forceinline__ void pair_setup(const double Xs[4][3], const double Xm[4][3], const double* ns,
                                           double R[3][3], SMap& ms, IMap& mm, double hs[3], double hm[4], double& ou,
                                           double& ov) {
#pragma clang fp contract(fast)
  double C[4][3], B[4][3], x0[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) x0[d] = 0.25 * (((Xs[0][d] + Xs[1][d]) + Xs[2][d]) + Xs[3][d]);
  coefficients(Xs, x0, C);
  coefficients(Xm, x0, B);
  plane_axes(Xs, ns, R);
  {
    const double e1u = dot3(C[1], R[0]), e1v = dot3(C[1], R[1]), e2u = dot3(C[2], R[0]), e2v = dot3(C[2], R[1]);
    const double fu = dot3(C[3], R[0]), fv = dot3(C[3], R[1]);
#pragma unroll
    for (int k = 0; k < 3; ++k) hs[k] = dot3(C[k + 1], R[2]);
    ms.j0 = e1u * e2v - e2u * e1v;
    const double r = 2.0 * rcp3(ms.j0);
    ms.e1u = e1u * r;
    ms.e1v = e1v * r;
    ms.e2u = e2u * r;
    ms.e2v = e2v * r;
    ms.fu = fu * r;
    ms.fv = fv * r;
    ms.a2 = convex_a2(e1u, e1v, e2u, e2v, ms.fu, ms.fv);
  }
  ou = dot3(C[0], R[0]);
  ov = dot3(C[0], R[1]);
#pragma unroll
  for (int d = 0; d < 3; ++d) B[0][d] -= C[0][d];
  double u[4], v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    u[k] = dot3(B[k], R[0]);
    v[k] = dot3(B[k], R[1]);
    hm[k] = dot3(B[k], R[2]);
  }
  mm.cu = u[0];
  mm.cv = v[0];
  mm.j0 = u[1] * v[2] - u[2] * v[1];
  const double r = 2.0 * rcp3(mm.j0);
  mm.e1u = u[1] * r;
  mm.e1v = v[1] * r;
  mm.e2u = u[2] * r;
  mm.e2v = v[2] * r;
  mm.fu = u[3] * r;
  mm.fv = v[3] * r;
  mm.a2 = convex_a2(u[1], v[1], u[2], v[2], mm.fu, mm.fv);
}

// Values a lane needs again after the quadrature, kept in LDS meanwhile
// instead of in registers (or instead of gathering the nodes and rebuilding
// the plane a second time, about 600 instructions of the reverse sweep's
// 5,100); lane-interleaved, no bank conflicts.
struct Stash {
  double* p;
  int stride;
  __device__ __forceinline__ double& operator[](int i) const { return p[i * stride]; }
  // for reading back: the laundered offset keeps the compiler from holding
  // the stored values in registers after all
  __device__ __forceinline__ Stash back() const { return Stash{p + launder(0), stride}; }
};
constexpr int FWD_STASH = 13;  // heights' coefficients; then the sums per slave element
constexpr int BWD_STASH = 16;  // heights' coefficients and R; then the sums per slave element

// ---- forward -------------------------------------------------------------------
// Sums over the pairs of each slave element within a wavefront (the lanes
// hold 64 consecutive pairs, sorted by slave element): every lane has put its
// N values in its column of st; the lane of an element's first pair here adds
// up the columns of its run, in pair order.  Returns whether this lane is
// one; the whole wavefront calls it.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int N>
__device__ __forceinline__ bool run_sums(const Stash& st, bool valid, bool head, double v[N]) {
  wave_lds_sync();
  const int lane = (int)(threadIdx.x & 63);
  const uint64_t heads = __ballot(valid && head), live = __ballot(valid);
  if (!(valid && head)) return false;
  // the run ends before the next head, or behind the last valid lane
  const uint64_t above = lane == 63 ? 0ull : ~0ull << (lane + 1);
  const uint64_t stop = (heads | ~live) & above;
  const int len = (stop ? __builtin_ctzll(stop) : 64) - lane;
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = st[k];
  for (int r = 1; r < len; ++r)
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] += st.p[k * st.stride + r];
  return true;
}

// Entry of the sums of slave element s in the tile of pair p: the element's
// own, or the tile's when the element's pairs began in an earlier tile
// (first: the lane of the tile's first pair, before which the element
// already had pairs).
__device__ __forceinline__ int64_t sums_entry(const ElemSums& E, int s, int64_t p, bool began_before) {
  return began_before ? (int64_t)E.n_el + p / TILE_PAIRS : (int64_t)s;
}

// Blocks of one pair from the monomial moments of its quadrature: mu_ij =
// sum w xi1^i xi2^j (i, j <= 2) and Mm[p][r] = sum w m_p(xi) m_r(eta) (Mx:
// its columns r = 1..3; column 0 is mu's first four): M = C Mm C^T to
// blk[c * stride + p], and, summed over the pairs of the slave element,
// D = C Dm C^T (Dm[p][r] the moment of m_p m_r) and g = C gm with
// gm = Mm ht_m - Dm ht_s (ht the heights' coefficients); for the dual basis
// Phi = A N (ms: the slave map) D, M, g <- A D, A M, A g.  Staging D and g per
// slave element instead of per pair cuts the values written from 36 to about
// 22 per pair at three pairs per element.  The whole wavefront calls it
// (valid: the lane has a pair; prev: the slave element of the pair before).
template <bool DUAL>
__device__ __forceinline__ void store_blocks(const SMap& ms, const double mu[9], const double Mx[12],
                                             const double gm[4], bool valid, int s, int prev, int64_t p,
                                             const Stash& st, double* __restrict__ blk, int64_t stride,
                                             const ElemSums& E) {
#pragma clang fp contract(fast)
  double A[16];
  if (valid) {
    const double Mm[16] = {mu[0], Mx[0], Mx[1], Mx[2], mu[1], Mx[3], Mx[4], Mx[5],
                           mu[2], Mx[6], Mx[7], Mx[8], mu[3], Mx[9], Mx[10], Mx[11]};
    double M[16];
    h_sandwich(Mm, 0.0625, M);
    if (DUAL) {
      const IMap w = widen(ms);
      const V2 S[4] = {map_node(w, 0), map_node(w, 1), map_node(w, 2), map_node(w, 3)};
      dual_coefficients(S, A);
      double Ms[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) Ms[k] = M[k];
      const bool some = mu[0] != 0.0;  // (no segment: possibly no coefficients either)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int k = 0; k < 4; ++k)
          M[4 * j + k] =
              some ? A[4 * j] * Ms[k] + A[4 * j + 1] * Ms[4 + k] + A[4 * j + 2] * Ms[8 + k] + A[4 * j + 3] * Ms[12 + k]
                   : 0.0;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) blk[(int64_t)k * stride + p] = M[k];
#pragma unroll
    for (int k = 0; k < 9; ++k) st[k] = mu[k];
#pragma unroll
    for (int k = 0; k < 4; ++k) st[9 + k] = gm[k];
  }
  const bool first = (threadIdx.x & 63) == 0;
  double v[13];
  if (!run_sums<13>(st, valid, first || prev != s, v)) return;
  const double Dm[16] = {v[0], v[1], v[2], v[3], v[1], v[4], v[3], v[6],
                         v[2], v[3], v[5], v[7], v[3], v[6], v[7], v[8]};
  const double gv[4] = {v[9], v[10], v[11], v[12]};
  double D[16], g[4];
  h_sandwich(Dm, 0.0625, D);
  h_apply(gv, g);
#pragma unroll
  for (int j = 0; j < 4; ++j) g[j] *= 0.25;
  if (DUAL) {
    double Ds[16], gs[4];
#pragma unroll
    for (int k = 0; k < 16; ++k) Ds[k] = D[k];
#pragma unroll
    for (int k = 0; k < 4; ++k) gs[k] = g[k];
    const bool some = v[0] != 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        D[4 * j + k] =
            some ? A[4 * j] * Ds[k] + A[4 * j + 1] * Ds[4 + k] + A[4 * j + 2] * Ds[8 + k] + A[4 * j + 3] * Ds[12 + k]
                 : 0.0;
      g[j] = some ? A[4 * j] * gs[0] + A[4 * j + 1] * gs[1] + A[4 * j + 2] * gs[2] + A[4 * j + 3] * gs[3] : 0.0;
    }
  }
  const int64_t at = sums_entry(E, s, p, first && prev == s);
#pragma unroll
  for (int k = 0; k < 16; ++k) E.v[(int64_t)k * E.stride + at] = D[k];
#pragma unroll
  for (int k = 0; k < 4; ++k) E.v[(int64_t)(16 + k) * E.stride + at] = g[k];
}

// gm of a pair from its moments and the heights' coefficients.
__device__ __forceinline__ void gap_moments(const double mu[9], const double Mx[12], const double hs[3],
                                            const double hm[4], double gm[4]) {
#pragma clang fp contract(fast)
  const double D1[4] = {mu[1], mu[4], mu[3], mu[6]}, D2[4] = {mu[2], mu[3], mu[5], mu[7]},
               D3[4] = {mu[3], mu[6], mu[7], mu[8]};
#pragma unroll
  for (int p = 0; p < 4; ++p)
    gm[p] = (mu[p] * hm[0] + Mx[3 * p] * hm[1] + Mx[3 * p + 1] * hm[2] + Mx[3 * p + 2] * hm[3]) -
            (D1[p] * hs[0] + D2[p] * hs[1] + D3[p] * hs[2]);
}

// Moments of pair p of slave element s from its stored polygon
// (nf = count | flip << 7), for
//   D[j][k] = sum w A_t Phi_j N_k(xi),  M[j][l] = sum w A_t Phi_j N_l(eta),
//   g[j]    = sum w A_t Phi_j (sum_l N_l(eta) hm_l - sum_k N_k(xi) hs_k)
// (store_blocks), over the fan triangles from vertex 0 and the rule points.
// The vertex of the next triangle is loaded before the points of this one.
// A pair that is no segment (lost after a coordinate update) has none.
template <int NQ>
__device__ __forceinline__ void pair_moments(const MeshPtrs& SM, int s, int4 cs, const MeshPtrs& MM, int4 cm,
                                             const GPoly& P, int nf, const KParams& kp, const Stash& st, SMap& ms,
                                             double mu[9], double Mx[12], double gm[4], unsigned& noconv) {
  const int n = nf & 0x7f;
  IMap mm;
  double ou, ov;
  {
    double Xs[4][3], Xm[4][3], R[3][3], hs[3], hm[4];
    load_nodes(SM.x, SM.y, SM.z, cs, Xs);
    load_nodes(MM.x, MM.y, MM.z, cm, Xm);
    pair_setup(Xs, Xm, elem_nrm(SM, s), R, ms, mm, hs, hm, ou, ov);
#pragma unroll
    for (int k = 0; k < 3; ++k) st[k] = hs[k];
#pragma unroll
    for (int k = 0; k < 4; ++k) st[3 + k] = hm[k];
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) mu[k] = 0.0;
#pragma unroll
  for (int k = 0; k < 12; ++k) Mx[k] = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) gm[k] = 0.0;
  if (n < 3) return;
  {
#pragma clang fp contract(fast)
    const double u0 = P.U(0) - ou, v0 = P.V(0) - ov;
    double u1 = P.U(1) - ou - u0, v1 = P.V(1) - ov - v0;
    double un = P.U(2), vn = P.V(2);
    for (int i = 1; i + 1 < n; ++i) {
      const double u2 = un - ou - u0, v2 = vn - ov - v0;
      if (i + 2 < n) {
        un = P.U(i + 2);
        vn = P.V(i + 2);
      }
      const double At = 0.5 * (u1 * v2 - v1 * u2);
#pragma unroll 1
      for (int q = 0; q < NQ; ++q) {
        double l0, l1, l2, w;
        rule_point<NQ>(q, l0, l1, l2, w);
        double a1, a2, b1, b2, rda, rdb;
        inverse2(ms, mm, u0 + l1 * u1 + l2 * u2, v0 + l1 * v1 + l2 * v2, kp, a1, a2, b1, b2, rda, rdb, noconv);
        const double t0 = w * At, t1 = t0 * a1, t2 = t0 * a2, t3 = t1 * a2;
        mu[0] += t0;
        mu[1] += t1;
        mu[2] += t2;
        mu[3] += t3;
        mu[4] += t1 * a1;
        mu[5] += t2 * a2;
        mu[6] += t3 * a1;
        mu[7] += t3 * a2;
        mu[8] += t3 * (a1 * a2);
        const double b12 = b1 * b2, t[4] = {t0, t1, t2, t3};
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          Mx[3 * p] += t[p] * b1;
          Mx[3 * p + 1] += t[p] * b2;
          Mx[3 * p + 2] += t[p] * b12;
        }
      }
      u1 = u2;
      v1 = v2;
    }
  }
  const Stash sb = st.back();
  const double hs[3] = {sb[0], sb[1], sb[2]}, hm[4] = {sb[3], sb[4], sb[5], sb[6]};
  gap_moments(mu, Mx, hs, hm, gm);
}

// ---- backward ------------------------------------------------------------------

// The line of edge k (node k to node k + 1) of a quad, in the parameters of
// its map: direction D (scaled as the map), a point M0 on it, and the
// parameter that is constant along it, sg = -1 or 1 (xi2 on even edges, xi1
// on odd ones).
struct EdgeLine {
  double du, dv, mu, mv, sg;
  bool odd;
};

__device__ __forceinline__ EdgeLine edge_line(const IMap& m, int k) {
#pragma clang fp contract(fast)
  EdgeLine e;
  e.odd = k & 1;
  e.sg = (k == 1 || k == 2) ? 1.0 : -1.0;
  const double h = 0.5 * m.j0 * e.sg;
  e.du = (e.odd ? m.e2u : m.e1u) + e.sg * m.fu;
  e.dv = (e.odd ? m.e2v : m.e1v) + e.sg * m.fv;
  e.mu = m.cu + h * (e.odd ? m.e1u : m.e2u);
  e.mv = m.cv + h * (e.odd ? m.e1v : m.e2v);
  return e;
}

// Adjoint (xu, xv) of the intersection X of edge lines A and B.  X moves with
// line A's normal displacement at X and with line B's: with normals nA, nB,
// (xu, xv) = pA + pB, pA along nA and pB along nB, acts on the points of the
// two lines at X, i.e. on the maps at the parameters xa, xb of X there.
// Parallel lines (no defined intersection) contribute nothing.
__device__ __forceinline__ void cross_adjoint(const EdgeLine& A, double ja, const EdgeLine& B, double jb, double X,
                                              double Y, double xu, double xv, double xa[2], double pa[2],
                                              double xb[2], double pb[2]) {
#pragma clang fp contract(fast)
  const double den = A.du * B.dv - A.dv * B.du;
  const double scale = (fabs(A.du) + fabs(A.dv)) * (fabs(B.du) + fabs(B.dv));
  const bool ok = fabs(den) > 1e-14 * scale;
  const double rden = ok ? rcp3(den) : 0.0;
  const double al = (xu * B.du + xv * B.dv) * rden, be = -(xu * A.du + xv * A.dv) * rden;
  pa[0] = -al * A.dv;
  pa[1] = al * A.du;
  pb[0] = -be * B.dv;
  pb[1] = be * B.du;
  // X = M0 + t (J0 / 2) D on each line: t along the line itself, so that it
  // is as accurate on nearly parallel lines
  const double la = 0.5 * ja * (A.du * A.du + A.dv * A.dv), lb = 0.5 * jb * (B.du * B.du + B.dv * B.dv);
  const double r = rcp3(la * lb);
  const double ta = ((X - A.mu) * A.du + (Y - A.mv) * A.dv) * (r * lb);
  const double tb = ((X - B.mu) * B.du + (Y - B.mv) * B.dv) * (r * la);
  xa[0] = A.odd ? A.sg : ta;
  xa[1] = A.odd ? ta : A.sg;
  xb[0] = B.odd ? B.sg : tb;
  xb[1] = B.odd ? tb : B.sg;
}

// Pull the adjoint (xu, xv) of clip vertex (X, Y) back to the coefficients
// of the two maps through its provenance: a slave node; a master node (two
// neighbouring master edges meet there); otherwise the intersection of two
// edge lines.  Clip edge l of a flipped master is its edge 3 - l.  The
// adjoint of a map's point at x adds m(x) times it to (c, e1, e2, f)-bar
// (the slave's c-bar is not needed: its plane moves with it).
__device__ __forceinline__ void vertex_adjoint(uint8_t lab, double X, double Y, double xu, double xv, const SMap& ms,
                                               const IMap& mm, bool flip, double cbs[6], double cbm[8]) {
#pragma clang fp contract(fast)
  double xa[2], pa[2] = {0.0, 0.0}, xb[2] = {0.0, 0.0}, pb[2] = {0.0, 0.0};
  const int la = lab >> 4, lb = flip ? 3 - (lab & 3) : lab & 3;
  if (lab & 0x80) {
    const int k = lab & 3;
    xa[0] = (k == 1 || k == 2) ? 1.0 : -1.0;
    xa[1] = k >= 2 ? 1.0 : -1.0;
    pa[0] = xu;
    pa[1] = xv;
  } else if (la < 4) {
    cross_adjoint(edge_line(widen(ms), la), ms.j0, edge_line(mm, lb), mm.j0, X, Y, xu, xv, xa, pa, xb, pb);
  } else {
    const int ka = flip ? 3 - (la & 3) : la & 3;
    xa[0] = xa[1] = 0.0;
    if (((ka ^ lb) & 1) == 0) {
      // opposite master edges
      double x2[2], p2[2];
      cross_adjoint(edge_line(mm, ka), mm.j0, edge_line(mm, lb), mm.j0, X, Y, xu, xv, x2, p2, xb, pb);
      const double x12 = x2[0] * x2[1];
      cbm[0] += p2[0];
      cbm[1] += p2[1];
      cbm[2] += x2[0] * p2[0];
      cbm[3] += x2[0] * p2[1];
      cbm[4] += x2[1] * p2[0];
      cbm[5] += x2[1] * p2[1];
      cbm[6] += x12 * p2[0];
      cbm[7] += x12 * p2[1];
    } else {
      const int k = lb == ((ka + 1) & 3) ? lb : ka;
      xb[0] = (k == 1 || k == 2) ? 1.0 : -1.0;
      xb[1] = k >= 2 ? 1.0 : -1.0;
      pb[0] = xu;
      pb[1] = xv;
    }
  }
  const double xa12 = xa[0] * xa[1], xb12 = xb[0] * xb[1];
  cbs[0] += xa[0] * pa[0];
  cbs[1] += xa[0] * pa[1];
  cbs[2] += xa[1] * pa[0];
  cbs[3] += xa[1] * pa[1];
  cbs[4] += xa12 * pa[0];
  cbs[5] += xa12 * pa[1];
  cbm[0] += pb[0];
  cbm[1] += pb[1];
  cbm[2] += xb[0] * pb[0];
  cbm[3] += xb[0] * pb[1];
  cbm[4] += xb[1] * pb[0];
  cbm[5] += xb[1] * pb[1];
  cbm[6] += xb12 * pb[0];
  cbm[7] += xb12 * pb[1];
}

// Adjoint of the in-plane projection (u, v) = ((X - x0).t1, (X - x0).t2) of
// the slave nodes and of the slave frame (x0, n0 = g1 x g2 / |g1 x g2|,
// t1 = g1 / |g1|, t2 = n0 x t1): given ub, vb of the nodes, writes their
// coordinate gradients Xsb.  With the continuous normal field (ns, the
// element's plane normal: n0 = ns, t1 = the part of g1 orthogonal to n0,
// normalised) the gradient with respect to n0 is added to n0b instead.
__device__ __forceinline__ void projection_adjoint(const double Xs[4][3], const double* ns, const double ub[4],
                                                   const double vb[4], double Xsb[4][3], double n0b_out[3]) {
#pragma clang fp contract(fast)
  double f[12];
  slave_frame_p(Xs, ns, f);
  double x0b[3] = {0, 0, 0}, t1b[3] = {0, 0, 0}, t2b[3] = {0, 0, 0}, n0b[3] = {0, 0, 0};
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double dd = Xs[k][d] - f[d];
      const double gg = ub[k] * f[6 + d] + vb[k] * f[9 + d];
      Xsb[k][d] = gg;
      x0b[d] -= gg;
      t1b[d] += ub[k] * dd;
      t2b[d] += vb[k] * dd;
    }
  // t2 = n0 x t1
  const double* n0 = f + 3;
  const double* t1 = f + 6;
  n0b[0] += t1[1] * t2b[2] - t1[2] * t2b[1];
  n0b[1] += t1[2] * t2b[0] - t1[0] * t2b[2];
  n0b[2] += t1[0] * t2b[1] - t1[1] * t2b[0];
  t1b[0] += t2b[1] * n0[2] - t2b[2] * n0[1];
  t1b[1] += t2b[2] * n0[0] - t2b[0] * n0[2];
  t1b[2] += t2b[0] * n0[1] - t2b[1] * n0[0];
  double g1[3], g2[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    g1[d] = 0.25 * (((Xs[1][d] - Xs[0][d]) + Xs[2][d]) - Xs[3][d]);
    g2[d] = 0.25 * (((Xs[2][d] + Xs[3][d]) - Xs[0][d]) - Xs[1][d]);
  }
  if (ns) {
    // t1 = w / |w|, w = g1 - (g1.n0) n0; n0 is an input
    const double gn = g1[0] * n0[0] + g1[1] * n0[1] + g1[2] * n0[2];
    double w[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) w[d] = g1[d] - gn * n0[d];
    const double rlw = 1.0 / sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2]);
    const double tt = t1[0] * t1b[0] + t1[1] * t1b[1] + t1[2] * t1b[2];
    double wb[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) wb[d] = (t1b[d] - t1[d] * tt) * rlw;
    const double nw = n0[0] * wb[0] + n0[1] * wb[1] + n0[2] * wb[2];
    double g1b[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      g1b[d] = wb[d] - n0[d] * nw;
      n0b_out[d] += n0b[d] - g1[d] * nw - gn * wb[d];
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double c0 = 0.25 * x0b[d], c1 = 0.25 * g1b[d];
      Xsb[0][d] += c0 - c1;
      Xsb[1][d] += c0 + c1;
      Xsb[2][d] += c0 + c1;
      Xsb[3][d] += c0 - c1;
    }
    return;
  }
  // frame from the slave nodes: g1, g2, n = g1 x g2, n0 = n/|n|, t1 = g1/|g1|
  const double nn[3] = {g1[1] * g2[2] - g1[2] * g2[1], g1[2] * g2[0] - g1[0] * g2[2], g1[0] * g2[1] - g1[1] * g2[0]};
  const double rln = 1.0 / sqrt(nn[0] * nn[0] + nn[1] * nn[1] + nn[2] * nn[2]);
  const double rlg = 1.0 / sqrt(g1[0] * g1[0] + g1[1] * g1[1] + g1[2] * g1[2]);
  const double tt = t1[0] * t1b[0] + t1[1] * t1b[1] + t1[2] * t1b[2];
  const double nt = n0[0] * n0b[0] + n0[1] * n0b[1] + n0[2] * n0b[2];
  double g1b[3], g2b[3], nbv[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    g1b[d] = (t1b[d] - t1[d] * tt) * rlg;
    nbv[d] = (n0b[d] - n0[d] * nt) * rln;
  }
  g1b[0] += g2[1] * nbv[2] - g2[2] * nbv[1];
  g1b[1] += g2[2] * nbv[0] - g2[0] * nbv[2];
  g1b[2] += g2[0] * nbv[1] - g2[1] * nbv[0];
  g2b[0] = nbv[1] * g1[2] - nbv[2] * g1[1];
  g2b[1] = nbv[2] * g1[0] - nbv[0] * g1[2];
  g2b[2] = nbv[0] * g1[1] - nbv[1] * g1[0];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double c0 = 0.25 * x0b[d], c1 = 0.25 * g1b[d], c2 = 0.25 * g2b[d];
    Xsb[0][d] += c0 - c1 - c2;
    Xsb[1][d] += c0 + c1 - c2;
    Xsb[2][d] += c0 + c1 + c2;
    Xsb[3][d] += c0 - c1 + c2;
  }
}

// Backward of one pair: gradient of
// L = sum WD[j][k] D[j][k] + sum WM[j][l] M[j][l] + sum wg[j] g[j]
// with respect to the slave (Xsb) and master (Xmb) nodal coordinates, from
// the stored polygon (nf = count | flip << 7).  Per rule point the
// integrand is F = 1/2 ma^T Q ma + ma^T W mb (ma = m(xi), mb = m(eta)), with
// Q = C^T (WD + WD^T) C - (wt ht_s^T + ht_s wt^T), W = C^T WM C + wt ht_m^T,
// wt = C^T wg, ht the heights' coefficients; reverse mode runs through the
// quadrature, the inverse maps (implicit-function derivative), the clip
// vertices (line intersections, each vertex once: the fan's pending vertex is
// carried to the next triangle) to the coefficients (u, v, height) of the two
// maps in the plane's axes R = (t1, t2, n0), and from there to the nodes:
//  - a rotation of the axes by the small vector w (components along t1, t2,
//    n0) turns every coefficient p into p - w x p, so wb = -sum p x pb;
//  - element normals: w follows g1 = (a, 0, 0), g2 = (b, c, 0) (components in
//    R): wz = dg1_v / a, wy = -dg1_h / a, wx = (dg2_h - dg1_h b / a) / c;
//    continuous field: wy = dn_u, wx = -dn_v, wz = (dg1_v - g1_h dn_v) / a
//    with the plane normal n, whose gradient is n0b (along n it is left out:
//    n is normalised);
//  - the maps' origin is the slave's centre.
// a, b, c are the slave map's: 2 / a = e2v, 2 / c = e1u, 2 b / (a c) = e2u.
// Bound by VALU issue and, at two waves per SIMD (256 registers), by the
// latency of its gathers.  The coefficient form of the vertex and axes
// adjoints (two map points per vertex, one 3-vector per pair) against four
// line end points and nine axis components took it from 0.76 to 0.57 ms on
// the wavy interface of 3.24M pairs, the forward from 0.38 to 0.31 ms.
template <int NQ, bool DUAL, bool NODAL = false>
__device__ __forceinline__ void pair_backward(const MeshPtrs& SM, int s, int4 cs, const MeshPtrs& MM, int4 cm,
                                              const GPoly& P, int nf, const KParams& kp, const Stash& st,
                                              const double WD_in[16], const double WM_in[16], const double wg_in[4],
                                              double Xsb[4][3], double Xmb[4][3], double n0b[3], unsigned& noconv) {
  const int n = nf & 0x7f;
  const bool flip = (nf & 0x80) != 0;
  if (n < 3) {  // no segment (a pair lost after a coordinate update)
#pragma unroll
    for (int d = 0; d < 3; ++d) {
#pragma unroll
      for (int k = 0; k < 4; ++k) Xsb[k][d] = Xmb[k][d] = 0.0;
      n0b[d] = 0.0;
    }
    return;
  }
  SMap ms;
  IMap mm;
  double Qs[10], W[16], wt[4], ou, ov;
  {
#pragma clang fp contract(fast)
    double Xs[4][3], Xm[4][3], R[3][3], hs[3], hm[4];
    load_nodes(SM.x, SM.y, SM.z, cs, Xs);
    load_nodes(MM.x, MM.y, MM.z, cm, Xm);
    pair_setup(Xs, Xm, NODAL ? elem_nrm(SM, s) : nullptr, R, ms, mm, hs, hm, ou, ov);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      st[k] = hs[k];
#pragma unroll
      for (int d = 0; d < 3; ++d) st[7 + 3 * k + d] = R[k][d];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) st[3 + k] = hm[k];
    // dual basis: the blocks are A times the standard ones, so the standard
    // sweep runs on the weights A^T W (the dependence of A on the slave
    // nodes is added by dual_adjoint)
    double WD[16], WM[16], wg[4];
    if (DUAL) {
      const IMap w = widen(ms);
      const V2 S[4] = {map_node(w, 0), map_node(w, 1), map_node(w, 2), map_node(w, 3)};
      double A[16];
      dual_coefficients(S, A);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          WD[4 * m + k] = A[m] * WD_in[k] + A[4 + m] * WD_in[4 + k] + A[8 + m] * WD_in[8 + k] + A[12 + m] * WD_in[12 + k];
          WM[4 * m + k] = A[m] * WM_in[k] + A[4 + m] * WM_in[4 + k] + A[8 + m] * WM_in[8 + k] + A[12 + m] * WM_in[12 + k];
        }
        wg[m] = A[m] * wg_in[0] + A[4 + m] * wg_in[1] + A[8 + m] * wg_in[2] + A[12 + m] * wg_in[3];
      }
    } else {
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        WD[k] = WD_in[k];
        WM[k] = WM_in[k];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) wg[k] = wg_in[k];
    }
    ht_apply(wg, wt);
#pragma unroll
    for (int k = 0; k < 4; ++k) wt[k] *= 0.25;
    double WDs[16], Q[16];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int k = 0; k < 4; ++k) WDs[4 * j + k] = WD[4 * j + k] + WD[4 * k + j];
    ht_sandwich(WDs, 0.0625, Q);
    ht_sandwich(WM, 0.0625, W);
    const double hts[4] = {0.0, hs[0], hs[1], hs[2]};
    int z = 0;
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int r = p; r < 4; ++r) Qs[z++] = Q[4 * p + r] - (wt[p] * hts[r] + hts[p] * wt[r]);
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int r = 0; r < 4; ++r) W[4 * p + r] += wt[p] * hm[r];
  }
  // Qs: q00 q01 q02 q03 q11 q12 q13 q22 q23 q33
  // adjoints of the maps' coefficients: cbs of the slave's (e1, e2, f), cbm
  // of the master's (c, e1, e2, f), hsb and hmb of their heights
  double cbs[6], cbm[8], hsb[3], hmb[4];
#pragma unroll
  for (int k = 0; k < 6; ++k) cbs[k] = 0.0;
#pragma unroll
  for (int k = 0; k < 8; ++k) cbm[k] = 0.0;
#pragma unroll
  for (int k = 0; k < 3; ++k) hsb[k] = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) hmb[k] = 0.0;
  {
#pragma clang fp contract(fast)
    const double u0 = P.U(0) - ou, v0 = P.V(0) - ov;
    double u1 = P.U(1) - ou - u0, v1 = P.V(1) - ov - v0;
    double un = P.U(2), vn = P.V(2);
    double x0bu = 0.0, x0bv = 0.0, pendu = 0.0, pendv = 0.0;
    for (int i = 1; i + 1 < n; ++i) {
      const double u2 = un - ou - u0, v2 = vn - ov - v0;
      if (i + 2 < n) {
        un = P.U(i + 2);
        vn = P.V(i + 2);
      }
      const double At = 0.5 * (u1 * v2 - v1 * u2);
      double Atb = 0.0;
      double pb1u = 0.0, pb1v = 0.0, pb2u = 0.0, pb2v = 0.0;
#pragma unroll 1
      for (int q = 0; q < NQ; ++q) {
        double l0, l1, l2, w;
        rule_point<NQ>(q, l0, l1, l2, w);
        double a1, a2, b1, b2, rda, rdb;
        inverse2(ms, mm, u0 + l1 * u1 + l2 * u2, v0 + l1 * v1 + l2 * v2, kp, a1, a2, b1, b2, rda, rdb, noconv);
        const double a12 = a1 * a2, b12 = b1 * b2;
        const double qa0 = Qs[0] + Qs[1] * a1 + Qs[2] * a2 + Qs[3] * a12;
        const double qa1 = Qs[1] + Qs[4] * a1 + Qs[5] * a2 + Qs[6] * a12;
        const double qa2 = Qs[2] + Qs[5] * a1 + Qs[7] * a2 + Qs[8] * a12;
        const double qa3 = Qs[3] + Qs[6] * a1 + Qs[8] * a2 + Qs[9] * a12;
        const double wb0 = W[0] + W[1] * b1 + W[2] * b2 + W[3] * b12;
        const double wb1 = W[4] + W[5] * b1 + W[6] * b2 + W[7] * b12;
        const double wb2 = W[8] + W[9] * b1 + W[10] * b2 + W[11] * b12;
        const double wb3 = W[12] + W[13] * b1 + W[14] * b2 + W[15] * b12;
        const double wa1 = W[1] + W[5] * a1 + W[9] * a2 + W[13] * a12;
        const double wa2 = W[2] + W[6] * a1 + W[10] * a2 + W[14] * a12;
        const double wa3 = W[3] + W[7] * a1 + W[11] * a2 + W[15] * a12;
        const double F = (0.5 * qa0 + wb0) + (0.5 * qa1 + wb1) * a1 + (0.5 * qa2 + wb2) * a2 + (0.5 * qa3 + wb3) * a12;
        const double G = wt[0] + wt[1] * a1 + wt[2] * a2 + wt[3] * a12;
        const double wA = w * At;
        Atb += w * F;
        const double ga3 = qa3 + wb3;
        // implicit-function adjoint: lambda = J^-T xibar at the solution (the
        // scaled Jacobian times J0 / (2 det J))
        const double ra = 0.5 * wA * rda, rb = 0.5 * wA * rdb;
        const double ya1 = ra * ((qa1 + wb1) + a2 * ga3), ya2 = ra * ((qa2 + wb2) + a1 * ga3);
        const double yb1 = rb * (wa1 + b2 * wa3), yb2 = rb * (wa2 + b1 * wa3);
        const double lau = (ms.e2v + ms.fv * a1) * ya1 - (ms.e1v + ms.fv * a2) * ya2;
        const double lav = (ms.e1u + ms.fu * a2) * ya2 - (ms.e2u + ms.fu * a1) * ya1;
        const double lbu = (mm.e2v + mm.fv * b1) * yb1 - (mm.e1v + mm.fv * b2) * yb2;
        const double lbv = (mm.e1u + mm.fu * b2) * yb2 - (mm.e2u + mm.fu * b1) * yb1;
        const double wAG = wA * G;
        hsb[0] -= wAG * a1;
        hsb[1] -= wAG * a2;
        hsb[2] -= wAG * a12;
        hmb[0] += wAG;
        hmb[1] += wAG * b1;
        hmb[2] += wAG * b2;
        hmb[3] += wAG * b12;
        cbs[0] -= a1 * lau;
        cbs[1] -= a1 * lav;
        cbs[2] -= a2 * lau;
        cbs[3] -= a2 * lav;
        cbs[4] -= a12 * lau;
        cbs[5] -= a12 * lav;
        cbm[0] -= lbu;
        cbm[1] -= lbv;
        cbm[2] -= b1 * lbu;
        cbm[3] -= b1 * lbv;
        cbm[4] -= b2 * lbu;
        cbm[5] -= b2 * lbv;
        cbm[6] -= b12 * lbu;
        cbm[7] -= b12 * lbv;
        const double pbu = lau + lbu, pbv = lav + lbv;
        x0bu += l0 * pbu;
        x0bv += l0 * pbv;
        pb1u += l1 * pbu;
        pb1v += l1 * pbv;
        pb2u += l2 * pbu;
        pb2v += l2 * pbv;
      }
      // triangle area, then vertex i is complete
      const double hA = 0.5 * Atb;
      x0bu += hA * (v1 - v2);
      x0bv += hA * (u2 - u1);
      vertex_adjoint(P.L(i), u0 + u1, v0 + v1, pendu + pb1u + hA * v2, pendv + pb1v - hA * u2, ms, mm, flip, cbs, cbm);
      pendu = pb2u - hA * v1;
      pendv = pb2v + hA * u1;
      u1 = u2;
      v1 = v2;
    }
    vertex_adjoint(P.L(n - 1), u0 + u1, v0 + v1, pendu, pendv, ms, mm, flip, cbs, cbm);
    vertex_adjoint(P.L(0), u0, v0, x0bu, x0bv, ms, mm, flip, cbs, cbm);
  }
  {
#pragma clang fp contract(fast)
    const Stash back = st.back();
    // adjoints of the coefficients, components (t1, t2, n0)
    double Sb[4][3] = {{0, 0, 0}, {cbs[0], cbs[1], hsb[0]}, {cbs[2], cbs[3], hsb[1]}, {cbs[4], cbs[5], hsb[2]}};
    const double Mb[4][3] = {{cbm[0], cbm[1], hmb[0]}, {cbm[2], cbm[3], hmb[1]}, {cbm[4], cbm[5], hmb[2]},
                             {cbm[6], cbm[7], hmb[3]}};
    double wx = 0.0, wy = 0.0, wz = 0.0;  // minus the sum of p x pb
    auto add = [&](double u, double v, double h, const double b[3]) {
      wx -= v * b[2] - h * b[1];
      wy -= h * b[0] - u * b[2];
      wz -= u * b[1] - v * b[0];
    };
    const double js = 0.5 * ms.j0, jm = 0.5 * mm.j0;
    add(js * ms.e1u, js * ms.e1v, back[0], Sb[1]);
    add(js * ms.e2u, js * ms.e2v, back[1], Sb[2]);
    add(js * ms.fu, js * ms.fv, back[2], Sb[3]);
    add(mm.cu, mm.cv, back[3], Mb[0]);
    add(jm * mm.e1u, jm * mm.e1v, back[4], Mb[1]);
    add(jm * mm.e2u, jm * mm.e2v, back[5], Mb[2]);
    add(jm * mm.fu, jm * mm.fv, back[6], Mb[3]);
    const double ra = 0.5 * ms.e2v;  // 1 / a
    Sb[1][1] += wz * ra;
    double nu = 0.0, nv = 0.0;
    if (NODAL) {
      nu = wy;
      nv = -wx - wz * ra * back[0];
    } else {
      Sb[1][2] -= wy * ra + wx * (0.5 * ms.e2u);
      Sb[2][2] += wx * (0.5 * ms.e1u);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) Sb[0][k] = -Mb[0][k];
    // to space, coefficients to nodes (C = H / 4)
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double r0 = back[7 + d], r1 = back[10 + d], r2 = back[13 + d];
      double c[4], x[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) c[k] = 0.25 * (Sb[k][0] * r0 + Sb[k][1] * r1 + Sb[k][2] * r2);
      h_apply(c, x);
#pragma unroll
      for (int k = 0; k < 4; ++k) Xsb[k][d] = x[k];
#pragma unroll
      for (int k = 0; k < 4; ++k) c[k] = 0.25 * (Mb[k][0] * r0 + Mb[k][1] * r1 + Mb[k][2] * r2);
      h_apply(c, x);
#pragma unroll
      for (int k = 0; k < 4; ++k) Xmb[k][d] = x[k];
      n0b[d] = NODAL ? nu * r0 + nv * r1 : 0.0;
    }
  }
}

// The slave components of a pair's gradient (and with the continuous normal
// field the plane normal's), summed over the pairs of the slave element into
// E.  The whole wavefront calls it (valid: the lane has a pair; prev: the
// slave element of the pair before).
template <bool NODAL>
__device__ __forceinline__ void store_slave_gradient(const double Xsb[4][3], const double n0b[3], bool valid, int s,
                                                     int prev, int64_t p, const Stash& st, const ElemSums& E) {
  constexpr int N = NODAL ? BWD_SUMS_NODAL : BWD_SUMS;
  static_assert(N <= BWD_STASH, "the sums fit the stash");
  if (valid) {
#pragma unroll
    for (int k = 0; k < 12; ++k) st[k] = Xsb[k / 3][k % 3];
    if (NODAL)
#pragma unroll
      for (int k = 0; k < 3; ++k) st[12 + k] = n0b[k];
  }
  const bool first = (threadIdx.x & 63) == 0;
  double v[N];
  if (!run_sums<N>(st, valid, first || prev != s, v)) return;
  const int64_t at = sums_entry(E, s, p, first && prev == s);
#pragma unroll
  for (int k = 0; k < N; ++k) E.v[(int64_t)k * E.stride + at] = v[k];
}

}  // namespace mt
