// Single-pass node sums of the 2-D element kernels.
//
// A workgroup of 256 lanes evaluates a tile of elements, one per lane, and owns
// the nodes whose four elements all lie in the tile.  Tiles are 16 x 16 elements
// and own 15 x 15 nodes: the first element row and column are evaluated by the
// neighbouring tile too (256/225 = 1.14 evaluations per element).  Lane (tx, ty)
// holds element (ex, ey) and owns node (ex, ey), the element's first corner,
// when tx, ty >= 1; the contributions of the three other corners go through LDS.
// The sum over the node's elements runs in the fixed order (left, below), below,
// left, own.
//
// Narrow meshes take tiles as wide (high) as the mesh: no column (row) is
// evaluated twice, lanes that a 16 x 16 tile would leave without an element hold
// further rows (columns), and the last lane of a row (column) also owns the node
// beyond its element.  Taken where it leaves at most 7/8 of the tiles.  Square
// tiles and these, per 10^6 elements: one across, residual 250 and 25 us, analytic
// Jv 398 and 37, all-outputs VJP 1419 and 80; four across, residual 65 and 24; 16
// across, analytic Jv 57 and 33 us.
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

constexpr int kTile2 = 16;  // elements per side of the square tile
constexpr int kTile2Threads = kTile2 * kTile2;
// LDS slots per value: one per lane, and a zero for missing neighbours.  Lanes of
// a square tile's first row and column own no node: their sums are not used.
template <bool kSquare>
constexpr int kTile2Slots = kTile2Threads + (kSquare ? 0 : 1);

// The tiles of a mesh: tx x ty lanes.  hx = 1 where the first column of lanes
// belongs to the neighbouring tile, 0 where the tile is as wide as the mesh (tx
// elements; the last lanes own two nodes); hy alike.  ntx tiles along x, nt in all.
// mul: lane / tx = lane * mul >> 20 for lanes below 1024.
struct Tiles2 {
  int tx, ty, hx, hy;
  unsigned ntx, nt, mul;
  bool square() const { return hx && hy; }
};

inline Tiles2 tiles2(int n0, int n1) {
  auto count = [](int n, int lanes, int halo) {
    return halo ? ((unsigned)n + 1 + (unsigned)lanes - 2) / ((unsigned)lanes - 1) : 1u;
  };
  auto make = [&](int tx, int ty, int hx, int hy) {
    const unsigned ntx = count(n0, tx, hx);
    return Tiles2{tx, ty, hx, hy, ntx, ntx * count(n1, ty, hy),
                  ((1u << 20) + (unsigned)tx - 1) / (unsigned)tx};
  };
  const Tiles2 square = make(kTile2, kTile2, 1, 1);
  Tiles2 best = square;
  auto take = [&](const Tiles2& T) {
    if (8 * T.nt <= 7 * square.nt && T.nt < best.nt) best = T;
  };
  if (n0 <= kTile2Threads / 2) take(make(n0, kTile2Threads / n0, 0, 1));
  if (n1 <= kTile2Threads / 2) take(make(kTile2Threads / n1, n1, 1, 0));
  return best;
}
inline Tiles2 tiles2(const Geo& G) { return tiles2(G.n[0], G.n[1]); }

struct Tile2 {
  int tx, ty;
  int ex, ey;      // this lane's element, and the node it owns
  bool elem;       // the element exists
  bool node;       // the lane owns node (ex, ey)
  bool more;       // and (ex + 1, ey) (hx = 0) or (ex, ey + 1) (hy = 0)
  long long base;  // index of node (ex, ey); only meaningful when elem or node
};

// Of n0 x n1 elements with rows of nn0 nodes.  Tiles are dealt to the XCDs in
// contiguous runs (neighbours share halo rows).
//
// kSquare: T is of square tiles, whose sides are constants then (T is set to
// them).  The kernels are compiled for these and for any shape: with the shape an
// argument alone, the order-2 tangent spills (2048^2 elements 331 us against 327)
// and the free-growth residual on 1024^2 takes 38.4 us against 37.7.
template <bool kSquare>
__device__ __forceinline__ Tile2 tile2_pos(Tiles2& T, int n0, int n1, int nn0) {
  if constexpr (kSquare) {
    T.tx = T.ty = kTile2;
    T.hx = T.hy = 1;
  }
  const unsigned t = xcd_tile(blockIdx.x, gridDim.x);
  Tile2 P;
  P.ty = kSquare ? (int)threadIdx.x / kTile2 : (int)((threadIdx.x * T.mul) >> 20);
  P.tx = kSquare ? (int)threadIdx.x % kTile2 : (int)threadIdx.x - P.ty * T.tx;
  P.ex = (int)(t % T.ntx) * (T.tx - T.hx) - T.hx + P.tx;
  P.ey = (int)(t / T.ntx) * (T.ty - T.hy) - T.hy + P.ty;
  const bool in = kSquare || P.ty < T.ty;  // lanes beyond the tile hold nothing
  P.elem = in && P.ex >= 0 && P.ex < n0 && P.ey >= 0 && P.ey < n1;
  P.node = in && P.tx >= T.hx && P.ty >= T.hy && P.ex <= n0 && P.ey <= n1;
  P.more = !kSquare && P.node && (T.hx == 0 ? P.tx == T.tx - 1 : T.hy == 0 && P.ty == T.ty - 1);
  P.base = P.ex + (long long)nn0 * P.ey;
  return P;
}
template <bool kSquare>
__device__ __forceinline__ Tile2 tile2_pos(Tiles2& T, const Geo& G) {
  return tile2_pos<kSquare>(T, G.n[0], G.n[1], G.nn[0]);
}

// LDS slots of the elements to the left, below, and left below of a lane's node,
// and of the element left below of its second one.
struct Around2 {
  int l, b, lb, more;
};
template <bool kSquare>
__device__ __forceinline__ Around2 around2(const Tiles2& T, const Tile2& P) {
  const int t = (int)threadIdx.x, zero = kSquare ? t : kTile2Threads;
  return Around2{P.tx > 0 ? t - 1 : zero, P.ty > 0 ? t - T.tx : zero,
                 P.tx > 0 && P.ty > 0 ? t - T.tx - 1 : zero,
                 P.more ? (T.hx == 0 ? t - T.tx : t - 1) : zero};
}

// acc[o] = node sum of output o at the lane's node, more[o] at its second one; out
// must be zero where the element does not exist.  sh: NO * 3 * kTile2Slots<kSquare> doubles of LDS.
template <int NO, bool kSquare>
__device__ __forceinline__ void tile2_sum(const Tiles2& T, const Tile2& P, const double (&out)[NO][4],
                                          double* __restrict__ sh, double (&acc)[NO], double (&more)[NO]) {
  constexpr int kSlots = kTile2Slots<kSquare>;
  const int t = (int)threadIdx.x;
#pragma unroll
  for (int o = 0; o < NO; ++o)
#pragma unroll
    for (int a = 1; a < 4; ++a) sh[(o * 3 + a - 1) * kSlots + t] = out[o][a];
  if (!kSquare && t < NO * 3) sh[t * kSlots + kTile2Threads] = 0.0;
  __syncthreads();
  const Around2 A = around2<kSquare>(T, P);
#pragma unroll
  for (int o = 0; o < NO; ++o) {
    const double* s = sh + o * 3 * kSlots;
    acc[o] = ((s[2 * kSlots + A.lb] + s[kSlots + A.b]) + s[A.l]) + out[o][0];
    // the lane's element is the one to the left (below) of the second node
    more[o] = kSquare ? 0.0 : s[2 * kSlots + A.more] + (T.hx == 0 ? out[o][1] : out[o][2]);
  }
}

// The results at the lane's nodes: the sums, or (sums - F0)/eps for the FD product
// (eps_dev[1] = 1/eps, 0 when eps is 0: the product is 0 then).
template <bool kSquare>
__device__ __forceinline__ void tile2_write(const Tiles2& T, const Tile2& P, int nn0, double a0, double a1,
                                            double m0, double m1, double2* __restrict__ out, bool fd,
                                            const double2* __restrict__ F0,
                                            const double* __restrict__ eps_dev) {
  auto put = [&](long long node, double a0, double a1) {
    if (fd) {
      const double ie = eps_dev[1];
      const double2 f0 = F0[node];
      a0 = ie == 0.0 ? 0.0 : (a0 - f0.x) * ie;
      a1 = ie == 0.0 ? 0.0 : (a1 - f0.y) * ie;
    }
    out[node] = make_double2(a0, a1);
  };
  if (P.node) put(P.base, a0, a1);
  if (!kSquare && P.more) put(P.base + (T.hx == 0 ? 1 : nn0), m0, m1);
}

}  // namespace pf
