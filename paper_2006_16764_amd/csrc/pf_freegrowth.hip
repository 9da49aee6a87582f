// Free-growth model (pure melt, phi in [0, 1], temperature T; Sec. 4.1):
// residual, FD Jv and analytic Jv of the part of the theta step that depends
// on the new state, and the explicit part fixed by the previous state, on
// order-1 elements (2-D and 3-D, through quad2/quad3 of pf_element.h) and on
// order-2 (biquadratic, 9-node) elements in 2-D.
//
// 2-D, both orders: one pass over tiles of elements whose corner contributions
// are summed in LDS in a fixed order (pf_tile2.h; order 2 below).  3-D: two
// passes, one thread per element evaluates the element vectors into the
// element buffer, then the gather of pf_residual.hip forms the node sums.  The
// analytic tangent differentiates the pointwise terms by hand, the anisotropic
// flux through the Hessian-vector product of pf_element.h.
#include <type_traits>

#include "pf_tile2.h"

namespace pf {

namespace {

constexpr int kFgBlock = 128;

// Pointwise terms of the residual: s[0], f[0] (phi rows), s[1], f[1] (T rows).
// a2 receives a^2.
template <int DIM>
__device__ __forceinline__ void fg_residual_point(const Geo& G, const FgConst& C, double phi,
                                                  const double* g, double tem, const double* gT,
                                                  double dphi, double dT, double hist, double* s,
                                                  double (*f)[3], double& a2) {
  Aniso<DIM> A;
  A.template flux<2>(g, G);
  const double om = 1.0 - phi, pom = phi * om;
  // G2 = bg phi (1-phi)(1-2phi)/W^2 - 5 beta (Tm - T) phi^2 (1-phi)^2 / W
  const double G2 = pom * fma(C.c_dw, om - phi, -C.c_drv * ((C.Tm - tem) * pom));
  s[0] = fma(A.a2 * dphi, G.idt, C.theta * G2);
  const double ph = fma(C.theta * G.idt, dphi, hist);
  s[1] = fma(G.idt, dT, -C.Lcp * ph);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    f[0][k] = k < DIM ? (C.theta * C.bg) * A.J[k] : 0.0;
    f[1][k] = k < DIM ? (C.theta * C.alpha) * gT[k] : 0.0;
  }
  a2 = A.a2;
}

// The same differentiated along (tp, tT): the T rows are linear, and with
// pom = phi (1 - phi), dpom = (1 - 2 phi) tp,
//   dG2 = dpom (c_dw (1 - 2 phi) - 2 c_drv (Tm - T) pom)
//         + pom (c_drv pom tT - 2 c_dw tp).
template <int DIM>
__device__ __forceinline__ void fg_tangent_point(const Geo& G, const FgConst& C, double phi,
                                                 const double* g, double tem, double dphi, double tp,
                                                 const double* tg, double tT, const double* tgT,
                                                 double* s, double (*f)[3]) {
  Aniso<DIM> A;
  A.template flux<2>(g, G);
  double Hv[3] = {0.0, 0.0, 0.0}, da, gtv, gmv;
  A.template hvp_c<false>(g, tg, 0.0, Hv, da, gtv, gmv);
  const double om = 1.0 - phi, pom = phi * om, w = om - phi;
  const double dr = C.c_drv * ((C.Tm - tem) * pom);
  const double dG2 = fma(w * tp, fma(C.c_dw, w, -2.0 * dr),
                         pom * fma(C.c_drv * pom, tT, (-2.0 * C.c_dw) * tp));
  s[0] = fma(fma((A.a + A.a) * da, dphi, A.a2 * tp), G.idt, C.theta * dG2);
  s[1] = G.idt * fma(-C.Lcp * C.theta, tp, tT);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    f[0][k] = k < DIM ? (C.theta * C.bg) * Hv[k] : 0.0;
    f[1][k] = k < DIM ? (C.theta * C.alpha) * tgT[k] : 0.0;
  }
}

// Order 1.  Residual: gradient fields {phi, T}; value fields {dphi, dT, hist}.
template <int DIM>
struct PhysFgRes : PointFree {
  // 3-D: points and rows unrolled (rows one at a time: 575 us against 561)
  static constexpr int kGxUnroll = 3;
  static constexpr int kGyUnroll = PF_GY_UNROLL;
  const Geo& G;
  const FgConst& C;
  double ca, car, a2;
  __device__ PhysFgRes(const Geo& g, const FgConst& c) : G(g), C(c), ca(0.0), car(0.0), a2(0.0) {}
  __device__ __forceinline__ void weight(double wx) { car = fma(wx, a2, car); }
  __device__ __forceinline__ void row(double wrow) {
    ca = fma(wrow, car, ca);
    car = 0.0;
  }
  __device__ __forceinline__ void operator()(const double* gv, const double (*gg)[3],
                                             const double* vv, double* s, double (*f)[3],
                                             double*) {
    fg_residual_point<DIM>(G, C, gv[0], gg[0], gv[1], gg[1], vv[0], vv[1], vv[2], s, f, a2);
  }
};

// Order 1.  Tangent: gradient fields {phi, tp, tT}; value fields {T, dphi}.
template <int DIM>
struct PhysFgJvp : PointFree {
  // 3-D: points unrolled, rows one at a time (rows unrolled spill: 1018 us
  // against 674 on 256 x 128 x 128)
  static constexpr int kGxUnroll = 3;
  static constexpr int kGyUnroll = 1;
  const Geo& G;
  const FgConst& C;
  __device__ PhysFgJvp(const Geo& g, const FgConst& c) : G(g), C(c) {}
  __device__ __forceinline__ void weight(double) {}
  __device__ __forceinline__ void row(double) {}
  __device__ __forceinline__ void operator()(const double* gv, const double (*gg)[3],
                                             const double* vv, double* s, double (*f)[3],
                                             double*) {
    fg_tangent_point<DIM>(G, C, gv[0], gg[0], vv[0], vv[1], gv[1], gg[1], gv[2], gg[2], s, f);
  }
};

// 2-D: the element vector of the element whose first corner is node base.  ca: the
// cell integral of a^2.
template <int MODE>
__device__ __forceinline__ void fg_element(const Geo& G, const FgConst& C, long long base,
                                           const double2* __restrict__ U,
                                           const double2* __restrict__ Up,
                                           const double2* __restrict__ V,
                                           const double* __restrict__ eps_dev,
                                           const HistArg& H, double (&out)[2][4],
                                           double& ca) {
  const long long s1 = G.nn[0];
  const double eps = (MODE == MODE_FD) ? *eps_dev : 0.0;
  constexpr int NG = MODE == MODE_JVP ? 3 : 2, NV = MODE == MODE_JVP ? 2 : 3;
  double ng[NG][4], nv[NV][4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const long long node = base + (a & 1) + (a >> 1) * s1;
    double2 u = U[node];
    const double2 up = Up[node];
    if constexpr (MODE == MODE_JVP) {
      const double2 v = V[node];
      ng[0][a] = u.x;
      ng[1][a] = v.x;
      ng[2][a] = v.y;
      nv[0][a] = u.y;
      nv[1][a] = u.x - up.x;
    } else {
      if constexpr (MODE == MODE_FD) {
        const double2 v = V[node];
        u.x = fma(eps, v.x, u.x);
        u.y = fma(eps, v.y, u.y);
      }
      ng[0][a] = u.x;
      ng[1][a] = u.y;
      nv[0][a] = u.x - up.x;
      nv[1][a] = u.y - up.y;
      nv[2][a] = C.use_hist ? H.at(node, up) : 0.0;
    }
  }
  double dummy[1][4];
#pragma unroll
  for (int a = 0; a < 4; ++a) out[0][a] = out[1][a] = 0.0;
  if constexpr (MODE == MODE_JVP) {
    PhysFgJvp<2> ph(G, C);
    quad2<3, 2, 2, 0>(G, ng, nv, out, dummy, ph);
  } else {
    PhysFgRes<2> ph(G, C);
    quad2<2, 3, 2, 0>(G, ng, nv, out, dummy, ph);
    ca = ph.ca;
  }
}

// (three wavefronts per SIMD: the analytic product would take 210 VGPRs and two;
// 1024^2 48.4 -> 45.7 us)
template <int MODE, bool kSquare>
__global__ void __launch_bounds__(kTile2Threads, 3)
    k_fg_tile2(Geo G, Tiles2 T, FgConst C, const double2* __restrict__ U, const double2* __restrict__ Up,
               const double2* __restrict__ V, const double* __restrict__ eps_dev,
               HistArg H, const double2* __restrict__ F0, double2* __restrict__ F,
               double* __restrict__ coef) {
  __shared__ double sh[2 * 3 * kTile2Slots<kSquare>];
  const Tile2 P = tile2_pos<kSquare>(T, G);
  double out[2][4] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
  double ca = 0.0;
  if (P.elem) {
    fg_element<MODE>(G, C, P.base, U, Up, V, eps_dev, H, out, ca);
    if (MODE == MODE_RES && coef && P.node)
      coef[P.ex + (long long)G.n[0] * P.ey] = ca / (4.0 * G.jac);
  }
  double acc[2], more[2];
  tile2_sum<2, kSquare>(T, P, out, sh, acc, more);
  tile2_write<kSquare>(T, P, G.nn[0], acc[0], acc[1], more[0], more[1], F, MODE == MODE_FD, F0, eps_dev);
}

// 3-D element vectors, one element per lane, into the element buffer.  kReload:
// the corners are read again at every Gauss plane and the element vector lies in
// the lane's own LDS slots: at most 246 VGPRs, two wavefronts per SIMD, where
// the same with both in registers takes 304 to 360 and one.  256 x 128 x 128
// elements: residual 751 -> 561 us, analytic Jv 899 -> 674 us, difference
// quotient 807 -> 639 us.
//
// Corners and element vector in registers for meshes whose wavefronts all run at
// once at one per SIMD: there no second wavefront hides the reloads' latency.
// Residual and analytic Jv with corners in registers, then reloaded: 33^3 17.1,
// 17.5 and 21.9, 23.6 us; 40^3 (500 workgroups) 19.0, 19.5 and 23.8, 25.2; 44^3
// (666) 27.1, 29.9 and 25.6, 26.6.
constexpr unsigned kOneWaveBlocks = 1024 * 64 / kFgBlock;  // 1024 SIMDs

template <int MODE, bool kReload>
__global__ void __launch_bounds__(kFgBlock, kReload ? 2 : 1)
    k_fg_elem3(Geo G, FgConst C, const double2* __restrict__ U, const double2* __restrict__ Up,
               const double2* __restrict__ V, const double* __restrict__ eps_dev,
               HistArg H, double* __restrict__ E, double* __restrict__ coef) {
  const long long e = (long long)blockIdx.x * kFgBlock + threadIdx.x;
  if (e >= G.n_elems) return;
  const long long n0 = G.n[0], n1 = G.n[1];
  const long long ex = e % n0;
  const long long rest = e / n0;
  const long long ey = rest % n1, ez = rest / n1;
  const long long base = ex + (long long)G.nn[0] * (ey + (long long)G.nn[1] * ez);
  // the element vector from the corners that load(gz, ng, nv) reads
  auto element = [&](auto& load, auto& ph, auto NG, auto NV) {
    if constexpr (kReload) {
      __shared__ double sh[2][8][kFgBlock];
      const int t = (int)threadIdx.x;
#pragma unroll
      for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int a = 0; a < 8; ++a) sh[o][a][t] = 0.0;
      StridedAcc acc{&sh[0][0][t], nullptr, kFgBlock};
      quad3g<NG(), NV(), 2, 0>(G, load, acc, ph);
#pragma unroll
      for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int a = 0; a < 8; ++a) E[(long long)(o * 8 + a) * G.n_elems + e] = sh[o][a][t];
    } else {
      double ng[NG()][8], nv[NV()][8], out[2][8], none[1][8];
      load(0, ng, nv);
#pragma unroll
      for (int a = 0; a < 8; ++a) out[0][a] = out[1][a] = 0.0;
      quad3<NG(), NV(), 2, 0>(G, ng, nv, out, none, ph);
#pragma unroll
      for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int a = 0; a < 8; ++a) E[(long long)(o * 8 + a) * G.n_elems + e] = out[o][a];
    }
  };
  constexpr std::integral_constant<int, 2> two;
  constexpr std::integral_constant<int, 3> three;
  if constexpr (MODE == MODE_JVP) {
    auto load = [&](int, double (&ng)[3][8], double (&nv)[2][8]) {
      __asm__ volatile("" ::: "memory");
      const long long s1 = G.nn[0], s2 = (long long)G.nn[0] * G.nn[1];
#pragma unroll
      for (int a = 0; a < 8; ++a) {
        const long long node = base + (a & 1) + ((a >> 1) & 1) * s1 + (a >> 2) * s2;
        const double2 u = U[node], v = V[node];
        ng[0][a] = u.x;
        ng[1][a] = v.x;
        ng[2][a] = v.y;
        nv[0][a] = u.y;
        nv[1][a] = u.x - Up[node].x;
      }
    };
    PhysFgJvp<3> ph(G, C);
    element(load, ph, three, two);
  } else {
    const double eps = (MODE == MODE_FD) ? *eps_dev : 0.0;
    const ReloadRes<MODE == MODE_FD> load{G, U, Up, V, C.use_hist ? H.rate : nullptr, base, eps};
    PhysFgRes<3> ph(G, C);
    element(load, ph, two, three);
    if (MODE == MODE_RES && coef) coef[e] = ph.ca / (8.0 * G.jac);
  }
}

// ----------------------------------------------------------------- order 2 (2-D)
// 1-D quadratic Lagrange basis (nodes -1, 0, 1) at the 3 Gauss points.
struct P2 {
  static constexpr double s = 0.77459666924148337704;  // sqrt(3/5)
  __host__ __device__ static constexpr double xi(int q) { return q == 0 ? -s : (q == 1 ? 0.0 : s); }
  __host__ __device__ static constexpr double b(int a, int q) {
    return a == 0 ? 0.5 * xi(q) * (xi(q) - 1.0) : (a == 1 ? 1.0 - xi(q) * xi(q) : 0.5 * xi(q) * (xi(q) + 1.0));
  }
  __host__ __device__ static constexpr double d(int a, int q) {
    return a == 0 ? xi(q) - 0.5 : (a == 1 ? -2.0 * xi(q) : xi(q) + 0.5);
  }
};

// Order 2 in one pass: a workgroup evaluates a 16 x 16 tile of 9-node elements,
// one per lane, and owns the grid nodes of the 15 x 15 elements beyond the
// tile's first row and column (as pf_tile2.h: 1.14 evaluations per element).
// Lane (tx, ty), tx, ty >= 1, holds element (ex, ey) and owns its grid nodes
// (2 ex + i, 2 ey + j), i, j in {0, 1}; the contributions of local nodes with
// lx = 2 or ly = 2 go to the neighbours through LDS.  Sums run over (left,
// below), below, left, own.
//
// Node (lx, ly) of element (ex, ey) is grid node (2 ex + lx, 2 ey + ly); the
// grid spacing G.h is half the element size, so d/dx = G.ih[0] d/dxi and the
// Jacobian of the reference map is G.h0 G.h1.
//
// Bound by FP64 issue (no element vectors in memory: 144 B per element each
// way before).  The rule is sum-factorised: per row of Gauss points the fields
// are contracted along y once for its three points, and the outputs are
// contracted along x per row before they are spread along y.  2048^2 elements,
// analytic Jv: 719 us with dense points, a gather pass and a history pass,
// 349 us now.
constexpr int kQ2Pass = 5;  // local nodes passed on: (2,2), (0,2), (1,2), (2,0), (2,1)

template <int MODE, bool kSquare>
__global__ void __launch_bounds__(kTile2Threads, 2)
    k_fg_q2(Geo G, Tiles2 T, FgConst C, const double2* __restrict__ U, const double2* __restrict__ Up,
            const double2* __restrict__ V, const double* __restrict__ eps_dev, HistArg H,
            const double2* __restrict__ F0, double2* __restrict__ F, double* __restrict__ coef) {
  __shared__ double sh[2][kQ2Pass][kTile2Slots<kSquare>];
  const long long nn0 = G.nn[0];
  double out[2][3][3];
#pragma unroll
  for (int o = 0; o < 2; ++o)
#pragma unroll
    for (int ly = 0; ly < 3; ++ly)
#pragma unroll
      for (int lx = 0; lx < 3; ++lx) out[o][ly][lx] = 0.0;
  const int t = (int)threadIdx.x;
  Tile2 P = tile2_pos<kSquare>(T, C.n_macro[0], C.n_macro[1], 0);
  P.base = 2LL * P.ex + nn0 * (2LL * P.ey);
  if (P.elem) {
    const double eps = (MODE == MODE_FD) ? *eps_dev : 0.0;
    // gradient fields: residual {phi, T}, tangent {phi, tp, tT}; value fields:
    // residual {dphi, dT, hist}, tangent {T, dphi}
    constexpr int NG = MODE == MODE_JVP ? 3 : 2, NV = MODE == MODE_JVP ? 2 : 3;
    double g[NG][3][3], w[NV][3][3];
#pragma unroll
    for (int ly = 0; ly < 3; ++ly)
#pragma unroll
      for (int lx = 0; lx < 3; ++lx) {
        const long long node = P.base + lx + nn0 * ly;
        double2 u = U[node];
        const double2 up = Up[node];
        if constexpr (MODE == MODE_JVP) {
          const double2 v = V[node];
          g[0][ly][lx] = u.x;
          g[1][ly][lx] = v.x;
          g[2][ly][lx] = v.y;
          w[0][ly][lx] = u.y;
          w[1][ly][lx] = u.x - up.x;
        } else {
          if constexpr (MODE == MODE_FD) {
            const double2 v = V[node];
            u.x = fma(eps, v.x, u.x);
            u.y = fma(eps, v.y, u.y);
          }
          g[0][ly][lx] = u.x;
          g[1][ly][lx] = u.y;
          w[0][ly][lx] = u.x - up.x;
          w[1][ly][lx] = u.y - up.y;
          w[2][ly][lx] = C.use_hist ? H.at(node, up) : 0.0;
        }
      }
    const double ih0 = G.ih[0], ih1 = G.ih[1], jac = G.h[0] * G.h[1];
    double ca = 0.0;
#pragma unroll 1
    for (int qy = 0; qy < 3; ++qy) {
      // along y: values (and y derivatives of the gradient fields) on the row
      double gy[NG][3], dy[NG][3], wy[NV][3];
#pragma unroll
      for (int lx = 0; lx < 3; ++lx) {
#pragma unroll
        for (int f = 0; f < NG; ++f) {
          gy[f][lx] = P2::b(0, qy) * g[f][0][lx] + P2::b(1, qy) * g[f][1][lx] + P2::b(2, qy) * g[f][2][lx];
          dy[f][lx] = (P2::d(0, qy) * g[f][0][lx] + P2::d(1, qy) * g[f][1][lx] +
                       P2::d(2, qy) * g[f][2][lx]) * ih1;
        }
#pragma unroll
        for (int f = 0; f < NV; ++f)
          wy[f][lx] = P2::b(0, qy) * w[f][0][lx] + P2::b(1, qy) * w[f][1][lx] + P2::b(2, qy) * w[f][2][lx];
      }
      // the row's outputs along x: value and x-flux part, y-flux part
      double rs[2][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}}, ry[2][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
      double car = 0.0;
#pragma unroll
      for (int qx = 0; qx < 3; ++qx) {
        const double b0 = P2::b(0, qx), b1 = P2::b(1, qx), b2 = P2::b(2, qx);
        const double d0 = P2::d(0, qx), d1 = P2::d(1, qx), d2 = P2::d(2, qx);
        double val[NG], dx[NG], dv[NG], wv[NV];
#pragma unroll
        for (int f = 0; f < NG; ++f) {
          val[f] = b0 * gy[f][0] + b1 * gy[f][1] + b2 * gy[f][2];
          dx[f] = (d0 * gy[f][0] + d1 * gy[f][1] + d2 * gy[f][2]) * ih0;
          dv[f] = b0 * dy[f][0] + b1 * dy[f][1] + b2 * dy[f][2];
        }
#pragma unroll
        for (int f = 0; f < NV; ++f) wv[f] = b0 * wy[f][0] + b1 * wy[f][1] + b2 * wy[f][2];
        double s[2], fl[2][3], a2 = 0.0;
        const double gp[3] = {dx[0], dv[0], 0.0}, gq[3] = {dx[1], dv[1], 0.0};
        if constexpr (MODE == MODE_JVP) {
          const double gr[3] = {dx[2], dv[2], 0.0};
          fg_tangent_point<2>(G, C, val[0], gp, wv[0], wv[1], val[1], gq, val[2], gr, s, fl);
        } else {
          fg_residual_point<2>(G, C, val[0], gp, val[1], gq, wv[0], wv[1], wv[2], s, fl, a2);
        }
        car = fma(Q1::w(qx), a2, car);
#pragma unroll
        for (int o = 0; o < 2; ++o) {
          const double ws = Q1::w(qx) * s[o], wx = Q1::w(qx) * ih0 * fl[o][0], wf = Q1::w(qx) * fl[o][1];
#pragma unroll
          for (int lx = 0; lx < 3; ++lx) {
            rs[o][lx] = fma(ws, P2::b(lx, qx), fma(wx, P2::d(lx, qx), rs[o][lx]));
            ry[o][lx] = fma(wf, P2::b(lx, qx), ry[o][lx]);
          }
        }
      }
      const double wrow = Q1::w(qy) * jac;
      ca = fma(wrow, car, ca);
#pragma unroll
      for (int ly = 0; ly < 3; ++ly) {
        const double cb = wrow * P2::b(ly, qy), cd = wrow * ih1 * P2::d(ly, qy);
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
          for (int lx = 0; lx < 3; ++lx)
            out[o][ly][lx] = fma(cb, rs[o][lx], fma(cd, ry[o][lx], out[o][ly][lx]));
      }
    }
    if (MODE == MODE_RES && coef && P.node) {
      // element mean of a^2 on its four grid cells (the preconditioner's grid)
      const double c = ca / (4.0 * jac);
#pragma unroll
      for (int sy = 0; sy < 2; ++sy)
#pragma unroll
        for (int sx = 0; sx < 2; ++sx)
          coef[(2 * P.ex + sx) + (long long)G.n[0] * (2 * P.ey + sy)] = c;
    }
  }
#pragma unroll
  for (int o = 0; o < 2; ++o) {
    sh[o][0][t] = out[o][2][2];
    sh[o][1][t] = out[o][2][0];
    sh[o][2][t] = out[o][2][1];
    sh[o][3][t] = out[o][0][2];
    sh[o][4][t] = out[o][1][2];
  }
  if (!kSquare && t < 2 * kQ2Pass) (&sh[0][0][0])[t * kTile2Slots<kSquare> + kTile2Threads] = 0.0;
  __syncthreads();
  if (!P.node) return;
  const Around2 A = around2<kSquare>(T, P);
  double a[2][2][2];  // [j][i][output]
#pragma unroll
  for (int o = 0; o < 2; ++o) {
    a[0][0][o] = ((sh[o][0][A.lb] + sh[o][1][A.b]) + sh[o][3][A.l]) + out[o][0][0];
    a[0][1][o] = sh[o][2][A.b] + out[o][0][1];
    a[1][0][o] = sh[o][4][A.l] + out[o][1][0];
    a[1][1][o] = out[o][1][1];
  }
  auto put = [&](long long node, double a0, double a1) {
    if constexpr (MODE == MODE_FD) {
      const double e = eps_dev[0];
      const double2 f0 = F0[node];
      a0 = e == 0.0 ? 0.0 : (a0 - f0.x) / e;
      a1 = e == 0.0 ? 0.0 : (a1 - f0.y) / e;
    }
    F[node] = make_double2(a0, a1);
  };
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if ((i == 1 && P.ex == C.n_macro[0]) || (j == 1 && P.ey == C.n_macro[1])) continue;
      put(P.base + i + nn0 * j, a[j][i][0], a[j][i][1]);
    }
  if (!kSquare && P.more) {
    // the nodes beyond the element along x (hx = 0) or y
    const bool x = T.hx == 0;
    const long long node = P.base + (x ? 2 : 2 * nn0);
    put(node, sh[0][0][A.more] + (x ? out[0][0][2] : out[0][2][0]),
        sh[1][0][A.more] + (x ? out[1][0][2] : out[1][2][0]));
    if (x ? P.ey < C.n_macro[1] : P.ex < C.n_macro[0])
      put(node + (x ? nn0 : 1), x ? out[0][1][2] : out[0][2][1], x ? out[1][1][2] : out[1][2][1]);
  }
}

FgConst fg_const(const pf_problem* pb, double theta, int use_hist) {
  const pf_freegrowth_params& f = pb->fg;
  FgConst C{};
  C.bg = f.beta * f.Gamma;
  C.c_dw = f.beta * f.Gamma / (f.W * f.W);
  C.c_drv = 5.0 * f.beta / f.W;
  C.Tm = f.Tm;
  C.alpha = f.alpha;
  C.Lcp = f.Lcp;
  C.theta = theta;
  C.use_hist = use_hist;
  C.n_macro[0] = pb->params.n[0];
  C.n_macro[1] = pb->params.n[1];
  return C;
}

template <int MODE>
int launch_mode(pf_problem* pb, const FgConst& C, const double* U, const double* Uprev,
                const double* v, const double* F0, const double* eps_dev, double* out0,
                double* coef, const HistArg& H, hipStream_t s) {
  const Geo& G = pb->geo;
  auto U2 = reinterpret_cast<const double2*>(U);
  auto P2p = reinterpret_cast<const double2*>(Uprev);
  auto V2 = reinterpret_cast<const double2*>(v);
  auto F02 = reinterpret_cast<const double2*>(F0);
  auto out2 = reinterpret_cast<double2*>(out0);
  if (pb->params.order == 2) {
    const Tiles2 T = tiles2(C.n_macro[0], C.n_macro[1]);
    if (T.square())
      hipLaunchKernelGGL((k_fg_q2<MODE, true>), dim3(T.nt), dim3(kTile2Threads), 0, s, G, T, C, U2, P2p, V2,
                         eps_dev, H, F02, out2, coef);
    else
      hipLaunchKernelGGL((k_fg_q2<MODE, false>), dim3(T.nt), dim3(kTile2Threads), 0, s, G, T, C, U2, P2p, V2,
                         eps_dev, H, F02, out2, coef);
    PF_HIP_CHECK(hipGetLastError());
    return PF_OK;
  }
  if (G.dim == 2) {
    const Tiles2 T = tiles2(G);
    if (T.square())
      hipLaunchKernelGGL((k_fg_tile2<MODE, true>), dim3(T.nt), dim3(kTile2Threads), 0, s, G, T, C, U2, P2p, V2,
                         eps_dev, H, F02, out2, coef);
    else
      hipLaunchKernelGGL((k_fg_tile2<MODE, false>), dim3(T.nt), dim3(kTile2Threads), 0, s, G, T, C, U2, P2p, V2,
                         eps_dev, H, F02, out2, coef);
    PF_HIP_CHECK(hipGetLastError());
    return PF_OK;
  }
  const dim3 eb((unsigned)((G.n_elems + kFgBlock - 1) / kFgBlock));
  if (eb.x > kOneWaveBlocks)
    hipLaunchKernelGGL((k_fg_elem3<MODE, true>), eb, dim3(kFgBlock), 0, s, G, C, U2, P2p, V2, eps_dev, H,
                       pb->elem_buf, coef);
  else
    hipLaunchKernelGGL((k_fg_elem3<MODE, false>), eb, dim3(kFgBlock), 0, s, G, C, U2, P2p, V2, eps_dev, H,
                       pb->elem_buf, coef);
  PF_HIP_CHECK(hipGetLastError());
  return launch_gather3(pb, out0, F0, eps_dev, MODE == MODE_FD ? 1 : 0, s);
}

}  // namespace

long long fg_elem_buf_len(const pf_problem* pb) {
  return pb->geo.dim == 3 ? (long long)2 * 8 * pb->geo.n_elems : 1;
}

int launch_fg(pf_problem* pb, int mode, const double* U, const double* Uprev, const double* v,
              const double* F0, const double* eps_dev, double* out0, double* coef, hipStream_t s,
              const double* Unm1) {
  if (mode != MODE_RES && mode != MODE_FD && mode != MODE_JVP) {
    set_error("the free-growth model has no VJP");
    return PF_ERR_INVALID_ARG;
  }
  const FgConst C = fg_const(pb, pb->params.theta, 1);
  const HistArg H = hist_arg(pb, Unm1);
  if (mode == MODE_RES) return launch_mode<MODE_RES>(pb, C, U, Uprev, v, F0, eps_dev, out0, coef, H, s);
  if (mode == MODE_FD) return launch_mode<MODE_FD>(pb, C, U, Uprev, v, F0, eps_dev, out0, nullptr, H, s);
  return launch_mode<MODE_JVP>(pb, C, U, Uprev, v, F0, eps_dev, out0, nullptr, H, s);
}

int fg_explicit(pf_problem* pb, const double* Un, double* E, hipStream_t s) {
  const double th = pb->params.theta;
  if (th == 1.0) {
    PF_HIP_CHECK(hipMemsetAsync(E, 0, pb->n_dof * sizeof(double), s));
    return PF_OK;
  }
  // the residual at (U^n; U^n) with weight 1 and no history is the spatial
  // operator at U^n: the time and rate terms vanish
  const FgConst C = fg_const(pb, 1.0, 0);
  PF_TRY(launch_mode<MODE_RES>(pb, C, Un, Un, nullptr, nullptr, nullptr, E, nullptr, HistArg{}, s));
  return blas_axpby(1.0 - th, E, 0.0, E, E, pb->n_dof, s);
}

}  // namespace pf
