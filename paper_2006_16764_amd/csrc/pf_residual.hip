// 2-D residual-family kernels: F(U), fused finite-difference Jv, analytic Jv
// and the vector-Jacobian products, all from one element routine
// (pf_element.h) with the single-pass node sums of pf_tile2.h; deterministic,
// no atomics, no colouring.  The VJP's two parameter sums are reduced per
// workgroup in a fixed tree (every element counted by the one tile that owns
// its first node) and then across workgroups in a fixed order.
//
// Also here: the gather pass of the two-pass 3-D alloy and free-growth kernels
// and the dispatch of the residual family over models and dimensions.
#include "pf_tile2.h"

namespace pf {

namespace {

// Wavefronts per SIMD asked of the compiler, where that spills nothing: left to
// itself it takes 204 VGPRs for the analytic product (two wavefronts) and 142 for
// the residual (three).  1024^2, 20 calls back to back: analytic product 45.4 ->
// 39.6 us, residual 27.5 -> 26.4 us; with one more the product spills 51 registers and takes
// 101 us.
template <int MODE>
constexpr int kTile2Waves = MODE == MODE_RES || MODE == MODE_FD    ? 4
                            : MODE == MODE_JVP || MODE == MODE_VJPU ? 3
                            : MODE == MODE_VJPP                     ? 2
                                                                    : 1;

template <int MODE, bool kSquare>
__global__ void __launch_bounds__(kTile2Threads, kTile2Waves<MODE>)
    k_tile2(Geo G, Tiles2 T, const double2* __restrict__ U, const double2* __restrict__ Up,
            const double2* __restrict__ V, const double* __restrict__ eps_dev,
            const double2* __restrict__ F0, double2* __restrict__ out0,
            double2* __restrict__ out1, double* __restrict__ vjp_part, double* __restrict__ coef) {
  constexpr int NO = (MODE == MODE_VJP) ? 4 : 2;
  __shared__ double sh[NO * 3 * kTile2Slots<kSquare>];
  const Tile2 P = tile2_pos<kSquare>(T, G);
  double out[NO][4];
#pragma unroll
  for (int o = 0; o < NO; ++o)
#pragma unroll
    for (int a = 0; a < 4; ++a) out[o][a] = 0.0;
  double ge = 0.0, gl = 0.0;
  if (P.elem) {
    double u0[4], u1[4], p0[4], p1[4], v0[4], v1[4];
    double eps = 0.0;
    if (MODE == MODE_FD) eps = eps_dev[0];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const long long node = P.base + (a & 1) + (a >> 1) * (long long)G.nn[0];
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
    }
    Element<2, MODE>::run(G, u0, u1, p0, p1, v0, v1, out, ge, gl);
    if (MODE == MODE_RES && coef && P.node)
      coef[P.ex + (long long)G.n[0] * P.ey] = ge / (4.0 * G.jac);
  }
  double acc[NO], more[NO];
  tile2_sum<NO, kSquare>(T, P, out, sh, acc, more);
  if (out0)
    tile2_write<kSquare>(T, P, G.nn[0], acc[0], acc[1], more[0], more[1], out0, MODE == MODE_FD, F0, eps_dev);
  if (MODE == MODE_VJP && out1)
    tile2_write<kSquare>(T, P, G.nn[0], acc[2 % NO], acc[3 % NO], more[2 % NO], more[3 % NO], out1, false,
                         nullptr, nullptr);
  if (MODE == MODE_VJP || MODE == MODE_VJPP) {
    // fixed-order workgroup reduction of the two parameter sums
    __syncthreads();
    double* red = sh;
    const int t = (int)threadIdx.x;
    red[t] = P.node ? ge : 0.0;  // ge, gl are 0 where the element does not exist
    red[kTile2Threads + t] = P.node ? gl : 0.0;
    __syncthreads();
    for (int w = kTile2Threads / 2; w > 0; w >>= 1) {
      if (t < w) {
        red[t] += red[t + w];
        red[kTile2Threads + t] += red[kTile2Threads + t + w];
      }
      __syncthreads();
    }
    if (t == 0) {
      vjp_part[blockIdx.x] = red[0];
      vjp_part[gridDim.x + blockIdx.x] = red[kTile2Threads];
    }
  }
}

// Sum of the element contributions around every node of a 3-D mesh (one
// thread per node, fixed order): out0 = sums, or (sums - F0)/eps when fd.
__global__ void __launch_bounds__(256)
    k_gather3(Geo G, const double* __restrict__ E, double2* __restrict__ out0,
              const double2* __restrict__ F0, const double* __restrict__ eps_dev, int fd) {
  // blockIdx.y is the node plane: coordinates from 32-bit arithmetic
  const int pn = G.nn[0] * G.nn[1];
  const int q = (int)blockIdx.x * (int)blockDim.x + (int)threadIdx.x;
  if (q >= pn) return;
  const int iy = q / G.nn[0];
  const int ix = q - iy * G.nn[0];
  const int iz = (int)blockIdx.y;
  const long long i = (long long)iz * pn + q;
  double acc[2] = {0.0, 0.0};
#pragma unroll
  for (int bz = 0; bz < 2; ++bz) {
    const int ez = iz - 1 + bz;
    if (ez < 0 || ez >= G.n[2]) continue;
#pragma unroll
    for (int by = 0; by < 2; ++by) {
      const int ey = iy - 1 + by;
      if (ey < 0 || ey >= G.n[1]) continue;
#pragma unroll
      for (int bx = 0; bx < 2; ++bx) {
        const int ex = ix - 1 + bx;
        if (ex < 0 || ex >= G.n[0]) continue;
        const long long e = ex + (long long)G.n[0] * (ey + (long long)G.n[1] * ez);
        const int a = (1 - bx) + 2 * (1 - by) + 4 * (1 - bz);
#pragma unroll
        for (int o = 0; o < 2; ++o) acc[o] += E[(long long)(o * 8 + a) * G.n_elems + e];
      }
    }
  }
  if (fd) {
    const double eps = *eps_dev;
    const double2 f0 = F0[i];
    double2 o;
    if (eps == 0.0) {
      o.x = 0.0;
      o.y = 0.0;
    } else {
      const double ie = 1.0 / eps;
      o.x = (acc[0] - f0.x) * ie;
      o.y = (acc[1] - f0.y) * ie;
    }
    out0[i] = o;
    return;
  }
  out0[i] = make_double2(acc[0], acc[1]);
}

template <int MODE>
int launch_tile2(const Geo& G, const double* U, const double* Uprev, const double* v,
                 const double* F0, const double* eps_dev, double* out0, double* out1,
                 double* vjp_part, double* coef, hipStream_t s) {
  const Tiles2 T = tiles2(G);
  auto d2 = [](const double* p) { return reinterpret_cast<const double2*>(p); };
  auto o2 = [](double* p) { return reinterpret_cast<double2*>(p); };
  if (T.square())
    hipLaunchKernelGGL((k_tile2<MODE, true>), dim3(T.nt), dim3(kTile2Threads), 0, s, G, T, d2(U), d2(Uprev),
                       d2(v), eps_dev, d2(F0), o2(out0), o2(out1), vjp_part, coef);
  else
    hipLaunchKernelGGL((k_tile2<MODE, false>), dim3(T.nt), dim3(kTile2Threads), 0, s, G, T, d2(U), d2(Uprev),
                       d2(v), eps_dev, d2(F0), o2(out0), o2(out1), vjp_part, coef);
  PF_HIP_CHECK(hipGetLastError());
  return PF_OK;
}

// 2-D thermal modes.  MODE_VJPP's one output goes through out0.
int launch_dim2(const Geo& G, int mode, const double* U, const double* Uprev, const double* v,
                const double* F0, const double* eps_dev, double* out0, double* out1,
                double* vjp_part, double* coef, hipStream_t s) {
  switch (mode) {
    case MODE_RES:
      return launch_tile2<MODE_RES>(G, U, Uprev, v, F0, eps_dev, out0, out1, vjp_part, coef, s);
    case MODE_FD:
      return launch_tile2<MODE_FD>(G, U, Uprev, v, F0, eps_dev, out0, out1, vjp_part, coef, s);
    case MODE_JVP:
      return launch_tile2<MODE_JVP>(G, U, Uprev, v, F0, eps_dev, out0, out1, vjp_part, coef, s);
    case MODE_VJPU:
      return launch_tile2<MODE_VJPU>(G, U, Uprev, v, F0, eps_dev, out0, out1, vjp_part, coef, s);
    case MODE_VJPP:
      return launch_tile2<MODE_VJPP>(G, U, Uprev, v, F0, eps_dev, out0, out1, vjp_part, coef, s);
    default:
      return launch_tile2<MODE_VJP>(G, U, Uprev, v, F0, eps_dev, out0, out1, vjp_part, coef, s);
  }
}

}  // namespace

int launch_residual2(const Geo& G, const double* U, const double* Uprev, double* F, hipStream_t s) {
  return launch_tile2<MODE_RES>(G, U, Uprev, nullptr, nullptr, nullptr, F, nullptr, nullptr, nullptr,
                                s);
}

int launch_gather3(pf_problem* pb, double* out0, const double* F0, const double* eps_dev, int fd,
                   hipStream_t s) {
  const Geo& G = pb->geo;
  const dim3 nb((unsigned)(((long long)G.nn[0] * G.nn[1] + 255) / 256), (unsigned)G.nn[2]);
  hipLaunchKernelGGL(k_gather3, dim3(nb), dim3(256), 0, s, G, pb->elem_buf,
                     reinterpret_cast<double2*>(out0), reinterpret_cast<const double2*>(F0),
                     eps_dev, fd);
  PF_HIP_CHECK(hipGetLastError());
  return PF_OK;
}

int launch_residual_family(pf_problem* pb, int mode, const double* U, const double* Uprev,
                           const double* v, const double* F0, const double* eps_dev,
                           double* out0, double* out1, double* vjp_part, hipStream_t s,
                           double* coef) {
  if (pb->model == 1) return launch_alloy(pb, mode, U, Uprev, v, F0, eps_dev, out0, coef, s);
  if (pb->model == 2) return launch_fg(pb, mode, U, Uprev, v, F0, eps_dev, out0, coef, s);
  // MODE_VJPP: out1 receives (dF/dUprev)^T w; its kernels write their one
  // output through out0 (which the parameter sums alone leave NULL)
  if (mode == MODE_VJPP) {
    out0 = out1;
    out1 = nullptr;
  }
  if (pb->geo.dim == 3)
    return launch_fused3(pb, mode, U, Uprev, v, F0, eps_dev, out0, out1, vjp_part, coef, s);
  return launch_dim2(pb->geo, mode, U, Uprev, v, F0, eps_dev, out0, out1, vjp_part, coef, s);
}

// Number of per-block partial sums the VJP writes (one per workgroup).
int vjp_blocks(const pf_problem* pb, int mode) {
  if (pb->geo.dim == 3) return fused3_tiles(pb->geo, mode);
  return (int)tiles2(pb->geo).nt;
}

}  // namespace pf
