// F = h^2-scaled compact right-hand side for
//  (a) a sum of Gaussian sources f = sum_s a_s exp(-|x - c_s|^2 / (2 sigma^2)),
//  (b) a separable source f = sum_s c_s X_s(x) Y_s(y) Z_s(z) given by samples of
//      each factor and its derivatives up to fourth order at the unknown nodes,
// and (c) the plane term of nonhomogeneous Dirichlet data on a z face, and
// (d) the data term of nonzero Neumann data on a Neumann face.
//
// Interior part, eq. (scheme) right side times h^2 (mixed fourth-derivative
// coefficient h^4/180, the value that makes the scheme sixth order):
//   h^2 [ c_K f + (h^2/12)(1 - kappa/30) lap f + (h^4/360) lap^2 f
//         + (h^4/180)(f_xxyy + f_xxzz + f_yyzz) ].
// Neumann face with normal axis n (eq. (3DN), beta = 0): +- 2h R_N with
//   R_N = (h^2/6)(1 - kappa/20) f_n + (h^4/120) f_nnn + (7h^4/360)(f_n t1t1 + f_n t2t2)
// (+ on the low face, - on the high face).
// Sommerfeld z face (eqs. (3DIMP), (3DDISCS)): + e^{ikh} mu3 [2h Fbar + mu1 (h^5/3) Lbar]
// with fbar_m = d^m/dz'^m (e^{ikz'} f), Lbar = fbar_xxz + fbar_yyz and
//   Fbar = (h^2/6 + k^2h^4/45) fbar_1 - (ikh^4/90) fbar_2 + (h^4/120)(fbar_3 - Lbar),
// z' = z at the bottom face and z' = top - z at the top face.
// Dirichlet data g on a z face: the unknown plane next to the face couples to
// the face plane through the in-plane operator G of eq. (scheme)'s delta_z^2
// term, G = I + (1 + kappa/30)/6 (D_x + D_y) + (1/30) D_x D_y (D = h^2 delta^2),
// so F -= G g on that plane.
// Neumann data beta = du/dn (n the face's axis, derivative along +n), eq.
// (3DN): the ghost relation carries -2h B with
//   B = (1 - kappa/6 + kappa^2/120) beta - (h^4/180)(beta_t1t1t2t2 + beta_t1^4 + beta_t2^4)
//       - (k^2 h^4/180)(beta_t1t1 + beta_t2t2),
// so the face's unknown plane gets F += 2h B (low face) or F -= 2h B (high face).
//
// Gaussian derivatives: d^n/dx^n exp(-t^2/2), t = (x - c)/sigma, equals
// (-1/sigma)^n He_n(t) exp(-t^2/2) with the probabilists' Hermite polynomials.
#include <type_traits>

#include "h6_internal.h"

namespace h6 {
namespace {

constexpr int kMaxSrc = 64;

// grid and coefficient data shared by every source form
struct RhsCoef {
  int n[3];        // interior counts
  int dims[3];     // unknown counts
  int qlo[3];      // q index of the first unknown per axis
  int face[6];
  double h;
  double2 cK, c_lap, c_bil, c_mix;               // interior coefficients (already times h^2)
  double2 nN1, nN3, nNm;                         // Neumann R_N coefficients (times 2h)
  double2 ik, sA, sB, sC, e1mu3, mu1h5;          // Sommerfeld coefficients
};

struct RhsArgs {
  RhsCoef c;
  int nsrc;
  double inv_sigma;
  double cx[kMaxSrc], cy[kMaxSrc], cz[kMaxSrc];
  double2 amp[kMaxSrc];
};

__device__ __forceinline__ void gauss_derivs(double x, double c, double is, double (&g)[5]) {
#pragma clang fp contract(off)
  const double t = (x - c) * is;
  const double e = exp(-0.5 * t * t);
  const double t2 = t * t;
  const double he[5] = {1.0, t, t2 - 1.0, t * (t2 - 3.0), t2 * t2 - 6.0 * t2 + 3.0};
  double s = 1.0;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    g[k] = s * he[k] * e;
    s *= -is;
  }
}

__device__ __forceinline__ double2 cm(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 ca(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 cs(double2 a, double s) { return make_double2(a.x * s, a.y * s); }
// factor arithmetic: real (Gaussians) or complex (separable tables)
__device__ __forceinline__ double fm(double a, double b) { return a * b; }
__device__ __forceinline__ double2 fm(double2 a, double2 b) { return cm(a, b); }
__device__ __forceinline__ double fa(double a, double b) { return a + b; }
__device__ __forceinline__ double2 fa(double2 a, double2 b) { return ca(a, b); }
__device__ __forceinline__ double fs(double a, double s) { return a * s; }
__device__ __forceinline__ double2 fs(double2 a, double s) { return cs(a, s); }
__device__ __forceinline__ double2 cmf(double2 a, double b) { return cs(a, b); }
__device__ __forceinline__ double2 cmf(double2 a, double2 b) { return cm(a, b); }

// One source is a product X(x) Y(y) Z(z).  Along a row of nodes (fixed y, z)
// every term of F, face terms of the y and z faces included, is a row constant
// times X, its second or its fourth derivative, so
//   F(x) = sum_s C[0]_s X_s + C[1]_s (d2 X)_s + C[2]_s (d4 X)_s.
// The constants of one source and row from the derivatives of Y and Z there;
// qy, qz: node indices.
template <typename S>
__device__ __forceinline__ void row_coefs(const RhsCoef& a, const S (&gy)[5], const S (&gz)[5], int qy, int qz,
                                          double2 (&C)[3]) {
  const S p00 = fm(gy[0], gz[0]), p20 = fm(gy[2], gz[0]), p02 = fm(gy[0], gz[2]), p22 = fm(gy[2], gz[2]);
  const S p40 = fm(gy[4], gz[0]), p04 = fm(gy[0], gz[4]), lap = fa(p20, p02);
  // c_bil multiplies lap^2 f = quartic terms + 2 mixed ones, c_mix the mixed ones
  const double2 mixc = ca(cs(a.c_bil, 2.0), a.c_mix);
  C[0] = ca(ca(cmf(a.cK, p00), cmf(a.c_lap, lap)), ca(cmf(a.c_bil, fa(p40, p04)), cmf(mixc, p22)));
  C[1] = ca(cmf(a.c_lap, p00), cmf(mixc, lap));
  C[2] = cmf(a.c_bil, p00);
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const double sg = side == 0 ? 1.0 : -1.0;
    if (a.face[2 + side] == H6_NEUMANN && qy == (side == 0 ? 0 : a.n[1] + 1)) {
      const S p10 = fm(gy[1], gz[0]), p30 = fm(gy[3], gz[0]), p12 = fm(gy[1], gz[2]);
      C[0] = ca(C[0], cs(ca(ca(cmf(a.nN1, p10), cmf(a.nN3, p30)), cmf(a.nNm, p12)), sg));
      C[1] = ca(C[1], cs(cmf(a.nNm, p10), sg));
    }
    if (a.face[4 + side] == H6_DIRICHLET || qz != (side == 0 ? 0 : a.n[2] + 1)) continue;
    const S p01 = fm(gy[0], gz[1]), p03 = fm(gy[0], gz[3]), p21 = fm(gy[2], gz[1]);
    if (a.face[4 + side] == H6_NEUMANN) {
      C[0] = ca(C[0], cs(ca(ca(cmf(a.nN1, p01), cmf(a.nN3, p03)), cmf(a.nNm, p21)), sg));
      C[1] = ca(C[1], cs(cmf(a.nNm, p01), sg));
    } else {                                   // Sommerfeld: z'-derivatives f and its first three z' derivatives
      const S f1 = fs(p01, sg), f3 = fs(p03, sg);
      const double2 ik = a.ik, ik2 = cm(ik, ik), ik3 = cm(ik2, ik);
      const double2 one = make_double2(1.0, 0.0);
      const double2 fb1 = ca(cmf(ik, p00), cmf(one, f1));
      const double2 fb2 = ca(ca(cmf(ik2, p00), cs(cmf(ik, f1), 2.0)), cmf(one, p02));
      const double2 fb3 = ca(ca(cmf(ik3, p00), cs(cmf(ik2, f1), 3.0)), ca(cs(cmf(ik, p02), 3.0), cmf(one, f3)));
      const double2 L0 = ca(cmf(ik, p20), cmf(one, fs(p21, sg)));      // Lbar: parts of X and of its second derivative
      const double2 L2 = ca(cmf(ik, p00), cmf(one, f1));
      const double2 F0 = ca(ca(cm(a.sA, fb1), cs(cm(a.sB, fb2), -1.0)), cm(a.sC, ca(fb3, cs(L0, -1.0))));
      C[0] = ca(C[0], cm(a.e1mu3, ca(cs(F0, 2.0 * a.h), cm(a.mu1h5, L0))));
      C[1] = ca(C[1], cm(a.e1mu3, ca(cs(cm(a.sC, L2), -2.0 * a.h), cm(a.mu1h5, L2))));
    }
  }
}

// The same for the Neumann x faces: at the end nodes of the row F gets
// +- (C[3]_s (d X)_s + C[4]_s (d3 X)_s), + on the low face.
template <typename S>
__device__ __forceinline__ void xface_coefs(const RhsCoef& a, const S (&gy)[5], const S (&gz)[5], double2& C3,
                                            double2& C4) {
  const S p00 = fm(gy[0], gz[0]), lap = fa(fm(gy[2], gz[0]), fm(gy[0], gz[2]));
  C3 = ca(cmf(a.nN1, p00), cmf(a.nNm, lap));
  C4 = cmf(a.nN3, p00);
}

// coordinate of node q, rounded before the centre is subtracted (as everywhere
// else; a fused multiply-add would shift every t by up to an ulp of the node)
__device__ __forceinline__ double node_coord(int q, double h) {
#pragma clang fp contract(off)
  const double x = q * h;
  return x;
}

// Sources of the row kernel.  factor(s, axis, i, g): derivatives 0..4 of the
// axis factor of source s at the i-th unknown; amp(s): its coefficient (zero
// past the last source, whose factor is then source 0's).
struct GaussSrc {
  using S = double;
  const RhsArgs& a;
  __device__ __forceinline__ int count() const { return a.nsrc; }
  __device__ __forceinline__ void factor(int s, int axis, int i, double (&g)[5]) const {
    const double* c = axis == 0 ? a.cx : axis == 1 ? a.cy : a.cz;
    gauss_derivs(node_coord(i + a.c.qlo[axis], a.c.h), c[s < a.nsrc ? s : 0], a.inv_sigma, g);
  }
  __device__ __forceinline__ double2 amp(int s) const { return s < a.nsrc ? a.amp[s] : make_double2(0.0, 0.0); }
};

// tab[a]: per term s and derivative order o the samples of the axis-a factor at
// its unknown nodes, tab[a][(s * 5 + o) * dims[a] + i]
struct TableSrc {
  using S = double2;
  const RhsCoef& c;
  int nterms;
  const double2* coef;
  const double2* tab[3];
  __device__ __forceinline__ int count() const { return nterms; }
  __device__ __forceinline__ void factor(int s, int axis, int i, double2 (&g)[5]) const {
    const double2* t = tab[axis] + size_t(s < nterms ? s : 0) * 5 * c.dims[axis] + i;
#pragma unroll
    for (int o = 0; o < 5; ++o) g[o] = t[size_t(o) * c.dims[axis]];
  }
  __device__ __forceinline__ double2 amp(int s) const { return s < nterms ? coef[s] : make_double2(0.0, 0.0); }
};

typedef double d4 __attribute__((ext_vector_type(4)));

// F as a matrix product on the FP64 matrix cores (v_mfma_f64_16x16x4): rows =
// (re, im) of eight grid rows, columns = 16 nodes along x, k = four sources
// (lane group g = lane / 16) times the orders 0, 2, 4.  Every lane computes the
// row constants and the factors it feeds to the instruction itself, so a wave
// needs no LDS: it holds the constants of 2 x 8 rows and 4 NQ sources and walks
// along x.  Complex factors (tables) take a second product with the constants
// times i.  Tile row 4 e + g is part e & 1 of grid row 2 g + (e >> 1), so a
// lane ends with two whole complex values.  More than 4 NQ sources: the rest
// is added by further passes over the wave's own rows.
// The terms of Neumann x faces go into the tiles that hold the end nodes as two
// more orders; a kernel of its own for them cost every such call 2 to 5 us and 25 us
// with 64 sources (31^3: 64 -> 39).
// The pass is bound by the store of F: 256 x 258 x 258, eight Gaussians, takes
// 69 us (4.0 TB/s of stores), against 970 us with every node forming 22
// derivative products per source from three exponentials.  Three waves per SIMD
// (few registers short of it by default: 128 x 128 x 128, 64 Gaussians, Neumann x
// 182 -> 143 us), two for tables of more than four terms (256 x 258 x 256, six terms:
// three 112 us, two 95).  Errors against
// 80-bit arithmetic over 32 face patterns, source counts and wavenumbers: 3.5e-16 on
// average (3.6e-16 node by node), 1.6e-16 for tables (1.7e-16).
constexpr int kRhsTiles = 2, kRhsRows = 8 * kRhsTiles;      // grid rows per wave

// XF: Neumann x faces; the tiles that hold an end node take their two orders more.
template <typename Src, int NQ, bool XF>
__device__ __forceinline__ void rhs_rows(const RhsCoef& a, const Src& src, double2* __restrict__ F) {
  using S = typename Src::S;
  constexpr bool kCplx = sizeof(S) == 16;
  constexpr int NO = XF ? 5 : 3;
  const int lane = threadIdx.x & 63, g = lane >> 4, c16 = lane & 15;
  const int nx = a.dims[0], ny = a.dims[1], nrows = ny * a.dims[2];
  const int row0 = (blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * kRhsRows;
  if (row0 >= nrows) return;
  // this lane's A rows: tile row c16 = part of grid row
  const int sub = 2 * (c16 & 3) + (c16 >> 3), part = (c16 >> 2) & 1;
  for (int s0 = 0; s0 == 0 || s0 < src.count(); s0 += 4 * NQ) {
    double2 C[kRhsTiles][NQ][NO];
#pragma unroll
    for (int t = 0; t < kRhsTiles; ++t) {
      const int row = min(row0 + 8 * t + sub, nrows - 1);
      const int j = row % ny, l = row / ny;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int sidx = s0 + 4 * q + g;
        S gy[5], gz[5];
        src.factor(sidx, 1, j, gy);
        src.factor(sidx, 2, l, gz);
        double2 c3[3];
        row_coefs<S>(a, gy, gz, j + a.qlo[1], l + a.qlo[2], c3);
#pragma unroll
        for (int o = 0; o < 3; ++o) C[t][q][o] = c3[o];
        if constexpr (XF) xface_coefs<S>(a, gy, gz, C[t][q][3], C[t][q][4]);
        const double2 am = src.amp(sidx);
#pragma unroll
        for (int o = 0; o < NO; ++o) {
          const double2 v = cm(am, C[t][q][o]);
          // A value of this lane's part against a real factor, and against an imaginary one
          C[t][q][o] = make_double2(part ? v.y : v.x, part ? v.x : -v.y);
        }
      }
    }
    for (int x0 = 16 * blockIdx.y; x0 < nx; x0 += 16 * gridDim.y) {
      const int x = x0 + c16, xc = min(x, nx - 1);
      d4 acc[kRhsTiles];
#pragma unroll
      for (int t = 0; t < kRhsTiles; ++t) acc[t] = d4{0.0, 0.0, 0.0, 0.0};
      S g0[NQ];
      const double end = x == 0 ? 1.0 : x == nx - 1 ? -1.0 : 0.0;
      auto add = [&](const double2 (&c)[NQ][NO], int q, int o, S gv, d4& v) {
        if constexpr (kCplx) {
          v = __builtin_amdgcn_mfma_f64_16x16x4f64(c[q][o].x, gv.x, v, 0, 0, 0);
          v = __builtin_amdgcn_mfma_f64_16x16x4f64(c[q][o].y, gv.y, v, 0, 0, 0);
        } else {
          v = __builtin_amdgcn_mfma_f64_16x16x4f64(c[q][o].x, gv, v, 0, 0, 0);
        }
      };
      // orders 4 and 2 of every source (and the face's 3 and 1) first: their products are
      // h or h^2 smaller, and added one by one to the large ones each would round the sum
      // once more
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        S gx[5];
        src.factor(s0 + 4 * q + g, 0, xc, gx);
        g0[q] = gx[0];
#pragma unroll
        for (int o = 2; o > 0; --o)
#pragma unroll
          for (int t = 0; t < kRhsTiles; ++t) add(C[t], q, o, gx[2 * o], acc[t]);
        if constexpr (XF)
          if (x0 == 0 || x0 + 16 >= nx) {
            S g1{}, g3{};
            if (end != 0.0) {
              g1 = fs(gx[1], end);
              g3 = fs(gx[3], end);
            }
#pragma unroll
            for (int t = 0; t < kRhsTiles; ++t) {
              add(C[t], q, 4, g3, acc[t]);
              add(C[t], q, 3, g1, acc[t]);
            }
          }
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int t = 0; t < kRhsTiles; ++t) add(C[t], q, 0, g0[q], acc[t]);
      if (x < nx) {
#pragma unroll
        for (int t = 0; t < kRhsTiles; ++t)
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            const int row = row0 + 8 * t + 2 * g + p;
            if (row >= nrows) continue;
            double2* o = F + size_t(row) * nx + x;
            double2 v = make_double2(acc[t][2 * p], acc[t][2 * p + 1]);
            if (s0 > 0) v = ca(v, *o);
            *o = v;
          }
      }
    }
  }
}

template <int NQ, bool XF>
__global__ __launch_bounds__(256, 3) void rhs_kernel(RhsArgs a, double2* __restrict__ F) {
  const GaussSrc src{a};
  rhs_rows<GaussSrc, NQ, XF>(a.c, src, F);
}

template <int NQ, bool XF>
__global__ __launch_bounds__(256, NQ == 2 ? 2 : 3) void rhs_separable_kernel(
    RhsCoef a, int nterms, const double2* __restrict__ coef, const double2* __restrict__ tx,
    const double2* __restrict__ ty, const double2* __restrict__ tz, double2* __restrict__ F) {
  const TableSrc src{a, nterms, coef, {tx, ty, tz}};
  rhs_rows<TableSrc, NQ, XF>(a, src, F);
}

// Dirichlet data g (n'x x n'y, x fastest) on a z face: Fp -= G g on the
// adjacent unknown plane Fp.  D_x, D_y take the neighbour outside the unknown
// range as 0 next to a Dirichlet face and as the mirror value (index 1 or
// n' - 2) next to a Neumann face.
struct PlaneRule {
  int nx, ny;
  int xlo_n, xhi_n, ylo_n, yhi_n;   // 1 where that in-plane face is Neumann
};

// index of the neighbour of i (i = -1 or n) under the face rule, or -1 for a zero value
__device__ __forceinline__ int ext_index(int i, int n, int lo_n, int hi_n) {
  if (i >= 0 && i < n) return i;
  if (n < 2) return -1;
  if (i < 0) return lo_n ? 1 : -1;
  return hi_n ? n - 2 : -1;
}

__device__ __forceinline__ double2 dx_row(const double2* __restrict__ g, const PlaneRule& r, int i, int j) {
  const double2* row = g + size_t(j) * r.nx;
  const int im = ext_index(i - 1, r.nx, r.xlo_n, r.xhi_n), ip = ext_index(i + 1, r.nx, r.xlo_n, r.xhi_n);
  double2 v = cs(row[i], -2.0);
  if (im >= 0) v = ca(v, row[im]);
  if (ip >= 0) v = ca(v, row[ip]);
  return v;
}

__global__ __launch_bounds__(256) void dirichlet_plane_kernel(const double2* __restrict__ g,
                                                              double2* __restrict__ Fp, PlaneRule r,
                                                              double2 ca_, double cb) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= r.nx * r.ny) return;
  const int i = idx % r.nx, j = idx / r.nx;
  const int jm = ext_index(j - 1, r.ny, r.ylo_n, r.yhi_n), jp = ext_index(j + 1, r.ny, r.ylo_n, r.yhi_n);
  const double2 g0 = g[idx];
  const double2 dx0 = dx_row(g, r, i, j);
  // D_y g and D_y D_x g at (i, j)
  double2 dy = cs(g0, -2.0), dyx = cs(dx0, -2.0);
  if (jm >= 0) {
    dy = ca(dy, g[size_t(jm) * r.nx + i]);
    dyx = ca(dyx, dx_row(g, r, i, jm));
  }
  if (jp >= 0) {
    dy = ca(dy, g[size_t(jp) * r.nx + i]);
    dyx = ca(dyx, dx_row(g, r, i, jp));
  }
  const double2 Gg = ca(ca(g0, cm(ca_, ca(dx0, dy))), cs(dyx, cb));
  const double2 f = Fp[idx];
  Fp[idx] = make_double2(f.x - Gg.x, f.y - Gg.y);
}

double2 d2(cplx c) { return make_double2(c.real(), c.imag()); }

RhsCoef rhs_coef(h6_plan P) {
  RhsCoef a{};
  for (int ax = 0; ax < 3; ++ax) {
    a.n[ax] = P->p.n[ax];
    a.dims[ax] = P->dims[ax];
    a.qlo[ax] = P->p.bc[2 * ax] != H6_DIRICHLET ? 0 : 1;
  }
  for (int f = 0; f < 6; ++f) a.face[f] = P->p.bc[f];
  const double h = P->p.h;
  const cplx I(0.0, 1.0), k = P->k, kap = P->kappa, ikh = I * k * h;
  a.h = h;
  const double h2 = h * h, h4 = h2 * h2;
  a.cK = d2(h2 * (1.0 - kap / 12.0 + kap * kap / 360.0));
  a.c_lap = d2(h2 * (h2 / 12.0) * (1.0 - kap / 30.0));
  a.c_bil = d2(cplx(h2 * h4 / 360.0));
  a.c_mix = d2(cplx(h2 * h4 / 180.0));
  a.nN1 = d2(2.0 * h * (h2 / 6.0) * (1.0 - kap / 20.0));
  a.nN3 = d2(cplx(2.0 * h * h4 / 120.0));
  a.nNm = d2(cplx(2.0 * h * 7.0 * h4 / 360.0));
  const cplx mu3 = 1.0 / (1.0 + (2.0 * ikh / 3.0) * (1.0 + 2.0 * kap / 15.0));
  const cplx mu1 = (ikh / 90.0 + (1.0 + kap / 30.0) / (6.0 * mu3)) / (1.0 + 2.0 * ikh / 3.0);
  a.ik = d2(I * k);
  a.sA = d2(h2 / 6.0 + k * k * h4 / 45.0);
  a.sB = d2(I * k * h4 / 90.0);
  a.sC = d2(cplx(h4 / 120.0));
  a.e1mu3 = d2(std::exp(ikh) * mu3);
  a.mu1h5 = d2(mu1 * h * h4 / 3.0);
  return a;
}

// launch of the row kernels: four waves of kRhsRows rows per workgroup; go(NQ, XF, grid)
template <typename F>
void rhs_launch(h6_plan P, int count, F&& go) {
  const size_t nrows = size_t(P->dims[1]) * P->dims[2];
  const unsigned wg = unsigned((nrows + 4 * kRhsRows - 1) / (4 * kRhsRows));
  // small grids: the x tiles of a row group are shared out until there are
  // about two waves per SIMD (each share forms the row constants again)
  const unsigned tiles = unsigned(P->dims[0] + 15) / 16, split = (512 + wg - 1) / wg;
  const dim3 grid(wg, split < tiles ? split : tiles);
  constexpr std::integral_constant<int, 1> one{};
  constexpr std::integral_constant<int, 2> two{};
  if (P->xmirror) {
    if (count <= 4) go(one, std::true_type{}, grid);
    else go(two, std::true_type{}, grid);
  } else {
    if (count <= 4) go(one, std::false_type{}, grid);
    else go(two, std::false_type{}, grid);
  }
}

// Neumann data on face plane (axis ax, side): beta = sum_s coef[s] T1_s(t1) T2_s(t2)
// from tables tab1 / tab2 ([(s * 5 + o) * n_t + i], o = derivative order).
struct NeumannFace {
  int n1, n2;                 // unknowns along the tangential axes t1 < t2
  size_t s1, s2;              // strides of t1, t2 in the vector layout
  size_t base;                // offset of the face's unknown plane
  double2 a0, c4, c2;         // 2h (1 - kappa/6 + kappa^2/120), -2h h^4/180, -2h k^2 h^4/180 (signed)
};

__global__ __launch_bounds__(256) void neumann_data_kernel(NeumannFace fc, int nterms,
                                                           const double2* __restrict__ coef,
                                                           const double2* __restrict__ tab1,
                                                           const double2* __restrict__ tab2,
                                                           double2* __restrict__ F) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= fc.n1 * fc.n2) return;
  const int i1 = idx % fc.n1, i2 = idx / fc.n1;
  double2 d00 = make_double2(0, 0), d4 = make_double2(0, 0), d2 = make_double2(0, 0);
  for (int s = 0; s < nterms; ++s) {
    double2 a[5], b[5];
    for (int o = 0; o < 5; ++o) {
      a[o] = tab1[size_t(s * 5 + o) * fc.n1 + i1];
      b[o] = tab2[size_t(s * 5 + o) * fc.n2 + i2];
    }
    const double2 c = coef[s];
    d00 = ca(d00, cm(c, cm(a[0], b[0])));
    d4 = ca(d4, cm(c, ca(ca(cm(a[2], b[2]), cm(a[4], b[0])), cm(a[0], b[4]))));
    d2 = ca(d2, cm(c, ca(cm(a[2], b[0]), cm(a[0], b[2]))));
  }
  const double2 add = ca(ca(cm(fc.a0, d00), cm(fc.c4, d4)), cm(fc.c2, d2));
  const size_t o = fc.base + size_t(i1) * fc.s1 + size_t(i2) * fc.s2;
  const double2 f = F[o];
  F[o] = make_double2(f.x + add.x, f.y + add.y);
}

}  // namespace

hipError_t launch_rhs(h6_plan P, int nsrc, const double* centres, const double* amps,
                      double sigma, double2* F, hipStream_t s) {
  if (nsrc > kMaxSrc) return hipErrorInvalidValue;
  RhsArgs a{};
  a.c = rhs_coef(P);
  a.nsrc = nsrc;
  // no source: the row kernel still multiplies a factor by zero, so it has to be finite
  // (1 / sigma and its fourth power overflow for the smallest sigma)
  a.inv_sigma = nsrc > 0 ? 1.0 / sigma : 0.0;
  for (int i = 0; i < nsrc; ++i) {
    a.cx[i] = centres[3 * i];
    a.cy[i] = centres[3 * i + 1];
    a.cz[i] = centres[3 * i + 2];
    a.amp[i] = make_double2(amps[2 * i], amps[2 * i + 1]);
  }
  hipEvent_t ev;
  timing_begin(P, KC_RHS, s, &ev);
  rhs_launch(P, nsrc, [&](auto NQ, auto XF, dim3 grid) {
    hipLaunchKernelGGL((rhs_kernel<NQ(), XF()>), grid, dim3(256), 0, s, a, F);
  });
  timing_end(P, KC_RHS, s, ev, double(P->N) * sizeof(double2));
  return hipGetLastError();
}

hipError_t launch_rhs_separable(h6_plan P, int nterms, const double* coef, const double* const tab[3],
                                double2* F, hipStream_t s) {
  // device copy of the coefficients and the three factor tables, in one
  // plan-owned buffer grown on demand
  const size_t total = size_t(nterms) * (1 + 5 * (size_t(P->dims[0]) + P->dims[1] + P->dims[2]));
  hipError_t e = hipSuccess;
  if (total * sizeof(double2) > P->sep_bytes) {
    (void)hipFree(P->d_sep);
    P->d_sep = nullptr;
    P->sep_bytes = 0;
    e = hipMalloc(&P->d_sep, total * sizeof(double2));
    if (e != hipSuccess) return e;
    P->sep_bytes = total * sizeof(double2);
  }
  double2* base = static_cast<double2*>(P->d_sep);
  const double2* dcoef = base;
  const double2* dtab[3];
  e = hipMemcpyAsync(base, coef, size_t(nterms) * sizeof(double2), hipMemcpyHostToDevice, s);
  size_t at = size_t(nterms);
  for (int ax = 0; ax < 3 && e == hipSuccess; ++ax) {
    const size_t cnt = size_t(nterms) * 5 * P->dims[ax];
    dtab[ax] = base + at;
    e = hipMemcpyAsync(base + at, tab[ax], cnt * sizeof(double2), hipMemcpyHostToDevice, s);
    at += cnt;
  }
  if (e != hipSuccess) return e;
  hipEvent_t ev;
  timing_begin(P, KC_RHS, s, &ev);
  const RhsCoef a = rhs_coef(P);
  rhs_launch(P, nterms, [&](auto NQ, auto XF, dim3 grid) {
    hipLaunchKernelGGL((rhs_separable_kernel<NQ(), XF()>), grid, dim3(256), 0, s, a, nterms, dcoef, dtab[0], dtab[1],
                       dtab[2], F);
  });
  timing_end(P, KC_RHS, s, ev, double(P->N) * sizeof(double2));
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the host tables may be released once the call returns
  return hipStreamSynchronize(s);
}

hipError_t launch_rhs_dirichlet_z(h6_plan P, int side, const double2* g, double2* F, hipStream_t s) {
  PlaneRule r{};
  r.nx = P->dims[0];
  r.ny = P->dims[1];
  r.xlo_n = P->p.bc[0] == H6_NEUMANN;
  r.xhi_n = P->p.bc[1] == H6_NEUMANN;
  r.ylo_n = P->p.bc[2] == H6_NEUMANN;
  r.yhi_n = P->p.bc[3] == H6_NEUMANN;
  const size_t plane = size_t(r.nx) * r.ny;
  double2* Fp = F + (side == 0 ? size_t(0) : plane * (P->dims[2] - 1));
  const double2 ca_ = d2((1.0 + P->kappa / 30.0) / 6.0);
  const unsigned nb = unsigned((plane + 255) / 256);
  hipLaunchKernelGGL(dirichlet_plane_kernel, dim3(nb), dim3(256), 0, s, g, Fp, r, ca_, 1.0 / 30.0);
  return hipGetLastError();
}

hipError_t launch_rhs_neumann(h6_plan P, int face, int nterms, const double* coef, const double* t1,
                              const double* t2, double2* F, hipStream_t s) {
  const int ax = face / 2, side = face % 2;
  const int ta = ax == 0 ? 1 : 0, tb = ax == 2 ? 1 : 2;       // tangential axes, increasing
  const size_t stride[3] = {1, size_t(P->dims[0]), size_t(P->dims[0]) * P->dims[1]};
  NeumannFace fc{};
  fc.n1 = P->dims[ta];
  fc.n2 = P->dims[tb];
  fc.s1 = stride[ta];
  fc.s2 = stride[tb];
  fc.base = side == 0 ? 0 : stride[ax] * size_t(P->dims[ax] - 1);
  const double h = P->p.h, h4 = h * h * h * h;
  const cplx kap = P->kappa, k2 = P->k * P->k;
  const double sg = side == 0 ? 2.0 * h : -2.0 * h;
  fc.a0 = d2(sg * (1.0 - kap / 6.0 + kap * kap / 120.0));
  fc.c4 = d2(cplx(-sg * h4 / 180.0));
  fc.c2 = d2(-sg * k2 * h4 / 180.0);
  const size_t total = size_t(nterms) * (1 + 5 * (size_t(fc.n1) + fc.n2));
  hipError_t e = hipSuccess;
  if (total * sizeof(double2) > P->sep_bytes) {
    (void)hipFree(P->d_sep);
    P->d_sep = nullptr;
    P->sep_bytes = 0;
    e = hipMalloc(&P->d_sep, total * sizeof(double2));
    if (e != hipSuccess) return e;
    P->sep_bytes = total * sizeof(double2);
  }
  double2* base = static_cast<double2*>(P->d_sep);
  double2* d1 = base + nterms;
  double2* dt2 = d1 + size_t(nterms) * 5 * fc.n1;
  e = hipMemcpyAsync(base, coef, size_t(nterms) * sizeof(double2), hipMemcpyHostToDevice, s);
  if (e == hipSuccess)
    e = hipMemcpyAsync(d1, t1, size_t(nterms) * 5 * fc.n1 * sizeof(double2), hipMemcpyHostToDevice, s);
  if (e == hipSuccess)
    e = hipMemcpyAsync(dt2, t2, size_t(nterms) * 5 * fc.n2 * sizeof(double2), hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return e;
  const unsigned nb = unsigned((size_t(fc.n1) * fc.n2 + 255) / 256);
  hipLaunchKernelGGL(neumann_data_kernel, dim3(nb), dim3(256), 0, s, fc, nterms, base, d1, dt2, F);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return hipStreamSynchronize(s);
}

}  // namespace h6
