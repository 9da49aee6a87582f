// Single-pass node sums of the 2-D order-1 element kernels.
//
// A workgroup of 256 lanes evaluates a 16 x 16 tile of elements, one per lane,
// and owns the 15 x 15 nodes whose four elements all lie in the tile: the
// tile's first element row and column are evaluated by the neighbouring tile
// too (256/225 = 1.14 evaluations per element).  Lane (tx, ty) holds element
// (ex, ey) and owns node (ex, ey), the element's first corner, when tx, ty >= 1;
// the contributions of the three other corners go through LDS.  The sum over
// the node's elements runs in the fixed order (left, below), below, left, own.
//
// Why: the former pair of kernels (element vectors to memory, then a gather)
// moved 128 B of element vectors per element against 64-80 B of input and
// output and took two launches.  The 14 % of evaluations done twice cost less
// at every size measured: analytic Jv on 1024^2 59.2 -> 39.6 us, residual on 387 x 251
// 10.9 -> 8.0 us.  The evaluation is bound by FP64 issue and latency, so one
// element per lane (all loads in flight at once, many waves) serves small and
// large meshes alike.
#pragma once

#include "pf_element.h"

namespace pf {

constexpr int kTile2 = 16;               // elements per tile side
constexpr int kTile2Own = kTile2 - 1;    // owned nodes per tile side
constexpr int kTile2Threads = kTile2 * kTile2;

inline unsigned tile2_blocks(const Geo& G) {
  return (unsigned)(((G.nn[0] + kTile2Own - 1) / kTile2Own) *
                    (long long)((G.nn[1] + kTile2Own - 1) / kTile2Own));
}

struct Tile2 {
  int tx, ty;
  int ex, ey;      // this lane's element, and the node it owns
  bool elem;       // the element exists
  bool node;       // the lane owns node (ex, ey)
  long long base;  // index of node (ex, ey); only meaningful when elem or node
};

// Tiles are dealt to the XCDs in contiguous runs (neighbours share halo rows).
__device__ __forceinline__ Tile2 tile2_pos(const Geo& G) {
  const unsigned ntx = (unsigned)((G.nn[0] + kTile2Own - 1) / kTile2Own);
  const unsigned t = xcd_tile(blockIdx.x, gridDim.x);
  Tile2 P;
  P.tx = (int)threadIdx.x % kTile2;
  P.ty = (int)threadIdx.x / kTile2;
  P.ex = (int)(t % ntx) * kTile2Own - 1 + P.tx;
  P.ey = (int)(t / ntx) * kTile2Own - 1 + P.ty;
  P.elem = P.ex >= 0 && P.ex < G.n[0] && P.ey >= 0 && P.ey < G.n[1];
  P.node = P.tx > 0 && P.ty > 0 && P.ex < G.nn[0] && P.ey < G.nn[1];
  P.base = P.ex + (long long)G.nn[0] * P.ey;
  return P;
}

// acc[o] = node sum of output o at the lane's node; out must be zero where the
// element does not exist.  sh: NO * 3 * kTile2Threads doubles of LDS.
template <int NO>
__device__ __forceinline__ void tile2_sum(const Tile2& P, const double (&out)[NO][4],
                                          double* __restrict__ sh, double (&acc)[NO]) {
  const int t = (int)threadIdx.x;
#pragma unroll
  for (int o = 0; o < NO; ++o)
#pragma unroll
    for (int a = 1; a < 4; ++a) sh[(o * 3 + a - 1) * kTile2Threads + t] = out[o][a];
  __syncthreads();
  // lanes of the first row or column own no node: any address in range will do
  const int l = P.tx > 0 ? t - 1 : t, b = P.ty > 0 ? t - kTile2 : t;
  const int lb = P.tx > 0 && P.ty > 0 ? t - kTile2 - 1 : t;
#pragma unroll
  for (int o = 0; o < NO; ++o) {
    const double* s = sh + o * 3 * kTile2Threads;
    acc[o] = ((s[2 * kTile2Threads + lb] + s[kTile2Threads + b]) + s[l]) + out[o][0];
  }
}

// The node's result: the sums, or (sums - F0)/eps for the FD product
// (eps_dev[1] = 1/eps, 0 when eps is 0: the product is 0 then).
__device__ __forceinline__ void tile2_write(const Tile2& P, double a0, double a1,
                                            double2* __restrict__ out, bool fd,
                                            const double2* __restrict__ F0,
                                            const double* __restrict__ eps_dev) {
  if (!P.node) return;
  if (fd) {
    const double ie = eps_dev[1];
    const double2 f0 = F0[P.base];
    a0 = ie == 0.0 ? 0.0 : (a0 - f0.x) * ie;
    a1 = ie == 0.0 ? 0.0 : (a1 - f0.y) * ie;
  }
  out[P.base] = make_double2(a0, a1);
}

}  // namespace pf
