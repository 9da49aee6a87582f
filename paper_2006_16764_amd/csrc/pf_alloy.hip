// Alloy model (directional solidification, Sec. 4.3): residual, FD Jv and
// analytic Jv of the part of the theta step that depends on the new state,
// and the explicit part fixed by the previous state.
//
// 2-D: the single-pass tiles of pf_tile2.h.  3-D: two passes, k_alloy_elem3
// evaluates every element once (one thread per element; Gauss rule by the
// sum-factorised quad3 of pf_element.h) into the element buffer, then the
// shared gather kernel forms the node sums in a fixed order.  Unlike the thermal u
// equation the solute equation is nonlinear (one-sided mobility,
// anti-trapping current, cu phihat source), so both fields go through the
// Gauss rule.  The analytic tangent differentiates the pointwise
// terms by hand, the anisotropic flux through the Hessian-vector product of
// pf_element.h.
#include "pf_tile2.h"

namespace pf {

namespace {

constexpr int kAlloyBlock = 128;
constexpr double kInv2Sqrt2 = 0.35355339059327376220;  // 1/(2 sqrt 2)

// 1/sqrt(x), x > 0: hardware estimate refined by two Newton steps
__device__ __forceinline__ double rsqrt_nr(double x) {
  double r = __builtin_amdgcn_rsq(x);
  r = r * fma(-0.5 * x * r, r, 1.5);
  return r * fma(-0.5 * x * r, r, 1.5);
}

// The frozen temperature G4 = (x - x_iso - v t)/l_T at the element's points: its
// value at the first node, and its rise along the element.
struct Frozen {
  double first, rise, here;
  __device__ Frozen(const AlloyConst& C, int ex)
      : first(fma(fma((double)ex, C.h0, C.x0), C.g4a, C.g4b)), rise(C.h0 * C.g4a), here(0.0) {}
  __device__ __forceinline__ void point(int gx) { here = fma(Q1::b1(gx), rise, first); }
};

// Residual: gradient fields {phi, u}; value fields {phi - phi^n, u - u^n, hist},
// hist = (1 - theta)(phi^n - phi^(n-1))/dt.  a2 receives cu a^2, the mobility
// factor of the time term (the preconditioner's phi-block coefficient).
template <int DIM>
struct PhysAlloyRes {
  // 3-D: points unrolled, rows one at a time (with rows unrolled too, 18
  // VGPRs spill at two wavefronts per SIMD)
  static constexpr int kGxUnroll = 3;
  static constexpr int kGyUnroll = 1;
  const Geo& G;
  const AlloyConst& C;
  Frozen T;
  double ca, car, a2;
  __device__ PhysAlloyRes(const Geo& g, const AlloyConst& c, int ex)
      : G(g), C(c), T(c, ex), ca(0.0), car(0.0), a2(0.0) {}
  __device__ __forceinline__ void point(int gx) { T.point(gx); }
  __device__ __forceinline__ void weight(double wx) { car = fma(wx, a2, car); }
  __device__ __forceinline__ void row(double wrow) {
    ca = fma(wrow, car, ca);
    car = 0.0;
  }
  __device__ __forceinline__ void operator()(const double* gv, const double (*gg)[3],
                                             const double* vv, double* s, double (*f)[3],
                                             double*) {
    const double phi = gv[0], u = gv[1], dphi = vv[0], du = vv[1], hist = vv[2];
    Aniso<DIM> A;
    A.template flux<2>(gg[0], G);
    const double cu = fma(C.omk, u, 1.0);
    const double om = fma(-phi, phi, 1.0);
    const double R = om * fma(-G.lam * om, u + T.here, phi);
    a2 = cu * A.a2;
    s[0] = fma(a2 * dphi, G.idt, -C.theta * R);
    const double ph = fma(C.theta * G.idt, dphi, hist), pc = ph * cu;
    s[1] = fma(C.hopk * G.idt, du, -0.5 * pc);
    const double mob = (C.theta * G.D * 0.5) * (1.0 - phi);
    const double at = (kInv2Sqrt2 * pc) * rsqrt_nr(A.q + G.delta2);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      f[0][k] = k < DIM ? C.theta * A.J[k] : 0.0;
      f[1][k] = k < DIM ? fma(mob, gg[1][k], at * gg[0][k]) : 0.0;
    }
  }
};

// Tangent along (tp, tu): gradient fields {phi, u, tp, tu}; value fields
// {phi - phi^n, hist}.  With cu, mob, ph, rs = Q^(-1/2), at = cu ph rs/(2 sqrt 2)
// as in the residual and gv = g . grad tp:
//   d(cu a^2 dphi) = dphi (omk tu a^2 + cu 2 a da) + cu a^2 tp,
//   dph = theta tp/dt,  d(ph cu) = dph cu + ph omk tu,  drs = -rs gv/Q,
//   d(mob grad u + at g) = mob grad tu - (theta D/2) tp grad u + at grad tp + dat g.
// On dual numbers the same took about half as many operations again: 3-D
// analytic Jv on 512 x 128 x 128 2190 -> 1990 us.
template <int DIM>
struct PhysAlloyJvp {
  // points unrolled, rows one at a time (measured at 1024 x 256 x 256)
  static constexpr int kGxUnroll = 3;
  static constexpr int kGyUnroll = 1;
  const Geo& G;
  const AlloyConst& C;
  Frozen T;
  __device__ PhysAlloyJvp(const Geo& g, const AlloyConst& c, int ex) : G(g), C(c), T(c, ex) {}
  __device__ __forceinline__ void point(int gx) { T.point(gx); }
  __device__ __forceinline__ void weight(double) {}
  __device__ __forceinline__ void row(double) {}
  __device__ __forceinline__ void operator()(const double* gv, const double (*gg)[3],
                                             const double* vv, double* s, double (*f)[3],
                                             double*) {
    const double phi = gv[0], u = gv[1], tp = gv[2], tu = gv[3], dphi = vv[0], hist = vv[1];
    Aniso<DIM> A;
    A.template flux<2>(gg[0], G);
    double Hv[3] = {0.0, 0.0, 0.0}, da, gtv, gmv;
    A.template hvp_c<false>(gg[0], gg[2], 0.0, Hv, da, gtv, gmv);
    const double cu = fma(C.omk, u, 1.0), dcu = C.omk * tu;
    const double om = fma(-phi, phi, 1.0), w = u + T.here;
    // dR/dphi = (1 - phi^2)(3 + 4 lambda phi (u + G4)) - 2, dR/du = -lambda (1 - phi^2)^2
    const double Rp = fma(om, fma(4.0 * G.lam * phi, w, 3.0), -2.0);
    const double dR = fma(Rp, tp, (-G.lam * om) * (om * tu));
    const double dm = fma(dcu, A.a2, cu * ((A.a + A.a) * da));
    s[0] = fma(fma(dm, dphi, (cu * A.a2) * tp), G.idt, -C.theta * dR);
    const double ti = C.theta * G.idt;
    const double ph = fma(ti, dphi, hist), pc = ph * cu;
    const double dpc = fma(ti * tp, cu, ph * dcu);
    s[1] = fma(C.hopk * G.idt, tu, -0.5 * dpc);
    const double hd = C.theta * G.D * 0.5;
    const double mob = hd * (1.0 - phi), dmob = -hd * tp;
    const double rs = kInv2Sqrt2 * rsqrt_nr(A.q + G.delta2);
    const double at = pc * rs, dat = rs * fma(-pc * A.iQ, gtv, dpc);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      f[0][k] = k < DIM ? C.theta * Hv[k] : 0.0;
      f[1][k] = k < DIM ? fma(mob, gg[3][k], fma(dmob, gg[1][k], fma(at, gg[2][k], dat * gg[0][k]))) : 0.0;
    }
  }
};

template <int DIM, int MODE>
struct AlloyElement {
  static constexpr int NA = 1 << DIM;
  template <int NG, int NV, class Phys>
  __device__ __forceinline__ static void quad(const Geo& G, const double (&ng)[NG][NA],
                                              const double (&nv)[NV][NA], double (&os)[2][NA],
                                              Phys& ph) {
    double dummy[1][NA];
    if constexpr (DIM == 3) quad3<NG, NV, 2, 0>(G, ng, nv, os, dummy, ph);
    else quad2<NG, NV, 2, 0>(G, ng, nv, os, dummy, ph);
  }
  // ex: the element along axis 0.  u0/u1: (phi, u) of the state (the perturbed
  // state for FD), p0/p1 of the previous state, hs: history rate, v0/v1:
  // direction.
  __device__ __forceinline__ static void run(const Geo& G, const AlloyConst& C, int ex,
                                             const double (&u0)[NA], const double (&u1)[NA],
                                             const double (&p0)[NA], const double (&p1)[NA],
                                             const double (&hs)[NA], const double (&v0)[NA], const double (&v1)[NA],
                                             double (&out)[2][NA], double& ge) {
#pragma unroll
    for (int a = 0; a < NA; ++a) out[0][a] = out[1][a] = 0.0;
    if constexpr (MODE == MODE_JVP) {
      double ng[4][NA], nv[2][NA];
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        ng[0][a] = u0[a];
        ng[1][a] = u1[a];
        ng[2][a] = v0[a];
        ng[3][a] = v1[a];
        nv[0][a] = u0[a] - p0[a];
        nv[1][a] = hs[a];
      }
      PhysAlloyJvp<DIM> ph(G, C, ex);
      quad<4, 2>(G, ng, nv, out, ph);
      ge = 0.0;
    } else {
      double ng[2][NA], nv[3][NA];
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        ng[0][a] = u0[a];
        ng[1][a] = u1[a];
        nv[0][a] = u0[a] - p0[a];
        nv[1][a] = u1[a] - p1[a];
        nv[2][a] = hs[a];
      }
      PhysAlloyRes<DIM> ph(G, C, ex);
      quad<2, 3>(G, ng, nv, out, ph);
      ge = ph.ca;
    }
  }
};

template <int DIM, int MODE>
__device__ __forceinline__ void alloy_element(const Geo& G, const AlloyConst& C, int ex,
                                              long long base, const double2* __restrict__ U,
                                              const double2* __restrict__ Up,
                                              const double2* __restrict__ V,
                                              const double* __restrict__ eps_dev,
                                              const HistArg& H, double (&out)[2][1 << DIM],
                                              double& ge) {
  constexpr int NA = 1 << DIM;
  const long long s1 = G.nn[0], s2 = (long long)G.nn[0] * G.nn[1];
  const double eps = (MODE == MODE_FD) ? *eps_dev : 0.0;
  double u0[NA], u1[NA], p0[NA], p1[NA], hs[NA], v0[NA], v1[NA];
#pragma unroll
  for (int a = 0; a < NA; ++a) {
    const long long node = base + (a & 1) + ((a >> 1) & 1) * s1 + (DIM == 3 ? ((a >> 2) & 1) * s2 : 0);
    double2 u = U[node];
    const double2 up = Up[node];
    double2 v = make_double2(0.0, 0.0);
    if (MODE != MODE_RES) v = V[node];
    if (MODE == MODE_FD) {
      u.x = fma(eps, v.x, u.x);
      u.y = fma(eps, v.y, u.y);
    }
    u0[a] = u.x;
    u1[a] = u.y;
    p0[a] = up.x;
    p1[a] = up.y;
    v0[a] = v.x;
    v1[a] = v.y;
    hs[a] = C.use_hist ? H.at(node, up) : 0.0;
  }
  AlloyElement<DIM, MODE == MODE_FD ? MODE_RES : MODE>::run(G, C, ex, u0, u1, p0, p1, hs, v0, v1,
                                                            out, ge);
}

template <int MODE, bool kSquare>
__global__ void __launch_bounds__(kTile2Threads)
    k_alloy_tile2(Geo G, Tiles2 T, AlloyConst C, const double2* __restrict__ U,
                  const double2* __restrict__ Up, const double2* __restrict__ V,
                  const double* __restrict__ eps_dev, HistArg H, const double2* __restrict__ F0,
                  double2* __restrict__ F, double* __restrict__ coef) {
  __shared__ double sh[2 * 3 * kTile2Slots<kSquare>];
  const Tile2 P = tile2_pos<kSquare>(T, G);
  double out[2][4] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
  double ge = 0.0;
  if (P.elem) {
    alloy_element<2, MODE>(G, C, P.ex, P.base, U, Up, V, eps_dev, H, out, ge);
    if (MODE == MODE_RES && coef && P.node)
      coef[P.ex + (long long)G.n[0] * P.ey] = ge / (4.0 * G.jac);
  }
  double acc[2], more[2];
  tile2_sum<2, kSquare>(T, P, out, sh, acc, more);
  tile2_write<kSquare>(T, P, G.nn[0], acc[0], acc[1], more[0], more[1], F, MODE == MODE_FD, F0, eps_dev);
}

// 3-D element vectors, one element per lane, into the element buffer.  kReload:
// the residual (and the difference quotient's residual) reads its corners again
// at every Gauss plane and keeps its element vector in its own LDS slots: 240
// VGPRs, two wavefronts per SIMD, where the same with both in registers takes
// 332 and one.  512 x 128 x 128: residual 1466 -> 1279 us, difference quotient
// 1522 -> 1447 us.  The tangent carries two more gradient fields and spills at
// two wavefronts (4226 us against 1990 at one), and at one the reloads only
// cost time (2092 us): corners and element vector stay in registers.
//
// So they do for meshes whose wavefronts all run at once at one per SIMD: there
// no second wavefront hides the reloads' latency.  Residual with corners in
// registers and reloaded: 33^3 18.7 and 24.5 us, 36^3 (396 workgroups) 19.4 and
// 25.2, 40^3 (520) 28.4 and 26.7, 48^3 30.0 and 28.7.
constexpr unsigned kOneWaveBlocks = 1024 * 64 / kAlloyBlock;  // 1024 SIMDs

template <int MODE, bool kReload>
__global__ void __launch_bounds__(kAlloyBlock, kReload ? 2 : 1)
    k_alloy_elem3(Geo G, AlloyConst C, const double2* __restrict__ U,
                  const double2* __restrict__ Up, const double2* __restrict__ V,
                  const double* __restrict__ eps_dev, HistArg H, double* __restrict__ E,
                  double* __restrict__ coef) {
  // blockIdx.y is the element layer: coordinates from 32-bit arithmetic
  const int pe = G.n[0] * G.n[1];
  const int q = (int)blockIdx.x * kAlloyBlock + (int)threadIdx.x;
  if (q >= pe) return;
  const int ey = q / G.n[0];
  const int ex = q - ey * G.n[0];
  const int ez = (int)blockIdx.y;
  const long long e = (long long)ez * pe + q;
  const long long base = ex + (long long)G.nn[0] * (ey + (long long)G.nn[1] * ez);
  if constexpr (!kReload) {
    double out[2][8];
    double ge = 0.0;
    alloy_element<3, MODE>(G, C, ex, base, U, Up, V, eps_dev, H, out, ge);
    if (MODE == MODE_RES && coef) coef[e] = ge / (8.0 * G.jac);
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
      for (int a = 0; a < 8; ++a) E[(long long)(o * 8 + a) * G.n_elems + e] = out[o][a];
  } else {
    __shared__ double sh[2][8][kAlloyBlock];
    const int t = (int)threadIdx.x;
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
      for (int a = 0; a < 8; ++a) sh[o][a][t] = 0.0;
    const double eps = (MODE == MODE_FD) ? *eps_dev : 0.0;
    const ReloadRes<MODE == MODE_FD> load{G, U, Up, V, C.use_hist ? H.rate : nullptr, base, eps};
    StridedAcc acc{&sh[0][0][t], nullptr, kAlloyBlock};
    PhysAlloyRes<3> ph(G, C, ex);
    quad3g<2, 3, 2, 0>(G, load, acc, ph);
    if (MODE == MODE_RES && coef) coef[e] = ph.ca / (8.0 * G.jac);
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
      for (int a = 0; a < 8; ++a) E[(long long)(o * 8 + a) * G.n_elems + e] = sh[o][a][t];
  }
}

__global__ void k_history(long long n, const double2* __restrict__ Un,
                             const double2* __restrict__ Unm1, double c, double* __restrict__ hist) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    hist[i] = c * (Un[i].x - Unm1[i].x);
}

template <int MODE>
int launch_mode(pf_problem* pb, const AlloyConst& C, const double* U, const double* Uprev,
                const double* v, const double* F0, const double* eps_dev, double* out0,
                double* coef, const HistArg& H, hipStream_t s) {
  const Geo& G = pb->geo;
  auto U2 = reinterpret_cast<const double2*>(U);
  auto P2 = reinterpret_cast<const double2*>(Uprev);
  auto V2 = reinterpret_cast<const double2*>(v);
  if (G.dim == 2) {
    const Tiles2 T = tiles2(G);
    auto F02 = reinterpret_cast<const double2*>(F0);
    auto F2 = reinterpret_cast<double2*>(out0);
    if (T.square())
      hipLaunchKernelGGL((k_alloy_tile2<MODE, true>), dim3(T.nt), dim3(kTile2Threads), 0, s, G, T, C, U2, P2,
                         V2, eps_dev, H, F02, F2, coef);
    else
      hipLaunchKernelGGL((k_alloy_tile2<MODE, false>), dim3(T.nt), dim3(kTile2Threads), 0, s, G, T, C, U2, P2,
                         V2, eps_dev, H, F02, F2, coef);
    PF_HIP_CHECK(hipGetLastError());
    return PF_OK;
  }
  const dim3 eb((unsigned)(((long long)G.n[0] * G.n[1] + kAlloyBlock - 1) / kAlloyBlock),
                (unsigned)G.n[2]);
  constexpr bool kForms = MODE != MODE_JVP;
  if (kForms && eb.x * eb.y > kOneWaveBlocks)
    hipLaunchKernelGGL((k_alloy_elem3<MODE, kForms>), dim3(eb), dim3(kAlloyBlock), 0, s, G, C, U2, P2, V2,
                       eps_dev, H, pb->elem_buf, coef);
  else
    hipLaunchKernelGGL((k_alloy_elem3<MODE, false>), dim3(eb), dim3(kAlloyBlock), 0, s, G, C, U2, P2, V2,
                       eps_dev, H, pb->elem_buf, coef);
  PF_HIP_CHECK(hipGetLastError());
  return launch_gather3(pb, out0, F0, eps_dev, MODE == MODE_FD ? 1 : 0, s);
}

}  // namespace

AlloyConst alloy_const(const pf_problem* pb, double t, double theta, int use_hist) {
  const pf_alloy_params& a = pb->alloy;
  AlloyConst C{};
  C.omk = 1.0 - a.k;
  C.hopk = 0.5 * (1.0 + a.k);
  C.g4a = 1.0 / a.l_T;
  C.g4b = -(a.x_iso + a.v_pull * t) / a.l_T;
  C.x0 = -pb->params.half_width[0];
  C.h0 = pb->geo.h[0];
  C.theta = theta;
  C.use_hist = use_hist;
  return C;
}

int launch_alloy(pf_problem* pb, int mode, const double* U, const double* Uprev, const double* v,
                 const double* F0, const double* eps_dev, double* out0, double* coef,
                 hipStream_t s, const double* Unm1) {
  if (mode != MODE_RES && mode != MODE_FD && mode != MODE_JVP) {
    set_error("the alloy model has no VJP");
    return PF_ERR_INVALID_ARG;
  }
  const AlloyConst C = alloy_const(pb, pb->t_new, pb->params.theta, 1);
  const HistArg H = hist_arg(pb, Unm1);
  if (mode == MODE_RES) return launch_mode<MODE_RES>(pb, C, U, Uprev, v, F0, eps_dev, out0, coef, H, s);
  if (mode == MODE_FD) return launch_mode<MODE_FD>(pb, C, U, Uprev, v, F0, eps_dev, out0, nullptr, H, s);
  return launch_mode<MODE_JVP>(pb, C, U, Uprev, v, F0, eps_dev, out0, nullptr, H, s);
}

int alloy_explicit(pf_problem* pb, const double* Un, double t_n, double* E, hipStream_t s) {
  const double th = pb->params.theta;
  if (th == 1.0) {
    PF_HIP_CHECK(hipMemsetAsync(E, 0, pb->n_dof * sizeof(double), s));
    return PF_OK;
  }
  // the residual at (U^n; U^n) with weight 1 and no history is the spatial
  // operator at U^n: the time and rate terms vanish
  const AlloyConst C = alloy_const(pb, t_n, 1.0, 0);
  PF_TRY(launch_mode<MODE_RES>(pb, C, Un, Un, nullptr, nullptr, nullptr, E, nullptr, HistArg{}, s));
  return blas_axpby(1.0 - th, E, 0.0, E, E, pb->n_dof, s);
}

HistArg hist_arg(const pf_problem* pb, const double* Unm1) {
  return HistArg{Unm1 ? nullptr : pb->hist, reinterpret_cast<const double2*>(Unm1),
                 (1.0 - pb->params.theta) / pb->params.dt};
}

int history_rate(pf_problem* pb, const double* Un, const double* Unm1, hipStream_t s) {
  const long long n = pb->geo.n_nodes;
  long long blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  const unsigned nb = (unsigned)blocks;
  hipLaunchKernelGGL(k_history, dim3(nb), dim3(256), 0, s, n,
                     reinterpret_cast<const double2*>(Un), reinterpret_cast<const double2*>(Unm1),
                     (1.0 - pb->params.theta) / pb->params.dt, pb->hist);
  PF_HIP_CHECK(hipGetLastError());
  return PF_OK;
}

}  // namespace pf
