// Single-pass 3-D residual family (F, fused FD Jv, analytic Jv, VJP).
//
// A workgroup of 256 lanes owns a tile of 16 x 16 element columns and marches
// through a chunk of element layers in z.  Per layer the next-but-one node plane (17 x
// 17 nodes of U, U^n and the direction/cotangent V) is copied into LDS, every
// lane evaluates one element (pf_element.h) and the node sums are formed from
// the element vectors in LDS in a fixed order:
//   plane k = (top contributions of layer k-1, carried in LDS)
//           + (bottom contributions of layer k).
// Nodes strictly inside the tile box are complete and written once.  Nodes on
// the tile's side faces or on its first/last plane also receive contributions
// from neighbouring tiles; their partial sums go to a side buffer that holds,
// per tile and densely, only those ring nodes (the first and last planes
// whole, the perimeter of every plane between them), and k_fixup3 -- one
// slot of the tile per lane, for the ring nodes that tile owns -- adds the partials
// of the <= 8 tiles that share such a node, in a fixed tile order.  No atomics:
// results are bitwise reproducible.
#include <algorithm>
#include <type_traits>

#include "pf_element.h"

namespace pf {

namespace {

constexpr int TX = 16, TY = 16;
constexpr int PX = TX + 1, PY = TY + 1;
constexpr int PN = PX * PY;  // nodes per staged plane
constexpr int kThreads = TX * TY;
// side buffer: per tile the first plane (PN nodes), the last plane (PN) and
// the perimeter ring of each of the kz - 1 planes between them (RING nodes)
constexpr int RING = 2 * (TX + TY);
__host__ __device__ constexpr int side_nodes(int kz) { return 2 * PN + (kz - 1) * RING; }

// Position of node (lx, ly) on the perimeter of the lxmax x lymax node box of
// a tile plane: bottom edge left to right, right edge upwards, top edge right
// to left, left edge downwards (2 (lxmax + lymax) positions).
__device__ __forceinline__ int ring_pos(int lx, int ly, int lxmax, int lymax) {
  int p = 2 * (lxmax + lymax) - ly;
  p = ly == lymax && lx > 0 ? 2 * lxmax + lymax - lx : p;
  p = lx == lxmax && ly < lymax ? lxmax + ly : p;
  return ly == 0 && lx < lxmax ? lx : p;
}

// Inverse of ring_pos; false for positions beyond the perimeter.
__device__ __forceinline__ bool ring_node(int r, int lxmax, int lymax, int& lx, int& ly) {
  if (r < lxmax) {
    lx = r;
    ly = 0;
    return true;
  }
  r -= lxmax;
  if (r < lymax) {
    lx = lxmax;
    ly = r;
    return true;
  }
  r -= lymax;
  if (r < lxmax) {
    lx = lxmax - r;
    ly = lymax;
    return true;
  }
  r -= lxmax;
  if (r < lymax) {
    lx = 0;
    ly = lymax - r;
    return true;
  }
  return false;
}

// Side-buffer node slot (0 .. side_nodes - 1) of ring node (lx, ly, lz) of a tile with
// node extents lxmax, lymax, kzmax.
__device__ __forceinline__ int side_slot(int lx, int ly, int lz, int lxmax, int lymax, int kzmax) {
  if (lz == 0) return lx + PX * ly;
  if (lz == kzmax) return PN + lx + PX * ly;
  return 2 * PN + (lz - 1) * RING + ring_pos(lx, ly, lxmax, lymax);
}

// Tile counts, and the element layers of a z-chunk.
struct Tiles {
  int ntx, nty, ntz, kz;
};

// Node planes go from HBM straight into LDS (global_load_lds_dwordx4, one
// double2 per lane, no registers) two planes ahead through a ring of three
// plane slots.
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) void glb_void_t;

// One double2 per active lane from src into the LDS slot of the lane's node:
// the instruction writes lane i of the wave at base + 16 i, so the destination
// is the wave's first node (n rounded down to a multiple of 64).
__device__ __forceinline__ void dma16(const double2* src, double2* lds_row, int n) {
  __builtin_amdgcn_global_load_lds((glb_void_t*)src, (lds_void_t*)(lds_row + (n & ~63)), 16, 0, 0);
}

// s_waitcnt vmcnt(0): this wave's outstanding memory operations, the plane
// copies into LDS included, have completed.
__device__ __forceinline__ void wait_vm() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// waves per SIMD of the analytic product and the lean adjoint products (a
// build-time knob: 1 or 2)
#ifndef PF_TAN_WAVES
#define PF_TAN_WAVES 2
#endif
template <int MODE>
constexpr int kWavesPerSimd = (MODE == MODE_RES || MODE == MODE_FD) ? 2 : MODE == MODE_VJP ? 1 : PF_TAN_WAVES;

// Corner source of Element::run_src built from three callables.
template <class C, class P, class L>
struct LdsCorners {
  C c;
  P p;
  L l;
  double* out0;  // this lane's slot of output field 0, corner 0
  int ostride;   // between output fields
  int cstride;   // between corners
  __device__ __forceinline__ void corner(int a, double2& u, double2& pp, double2& v) { c(a, u, pp, v); }
  __device__ __forceinline__ void plane(int gz) { p(gz); }
  __device__ __forceinline__ void loaded(int gz) { l(gz); }
  __device__ __forceinline__ double* out(int o) { return out0 + o * ostride; }
  __device__ __forceinline__ int stride() const { return cstride; }
};

template <int MODE>
struct ModeInfo {
  static constexpr int NO = MODE == MODE_VJP ? 4 : 2;  // doubles per node output
  static constexpr bool kHasV = MODE != MODE_RES;
  // Residual, FD and analytic products: output 1 is the exact linear part
  // alone, M y + theta D K x of two nodal fields, which is formed at the nodes
  // (NodalLin) instead of per element.
  static constexpr bool kNodal = MODE == MODE_RES || MODE == MODE_FD || MODE == MODE_JVP;
  static constexpr int NE = kNodal ? 1 : NO;  // fields of the element vectors
};

// Coefficients of the nodal linear part, see k_fused3.
struct NodalLin {
  double m, kx, ky, q;
};

NodalLin nodal_lin(const Geo& G) {
  const double hx6 = G.h[0] / 6.0, hy6 = G.h[1] / 6.0, hz6 = G.h[2] / 6.0;
  return NodalLin{G.idt * hx6 * hy6 * hz6, G.Dth * G.ih[0] * hy6 * hz6, G.Dth * hx6 * G.ih[1] * hz6,
                  G.Dth * hx6 * hy6 * G.ih[2]};
}

__device__ __forceinline__ long long gnode(const Geo& G, int x, int y, int z) {
  return x + (long long)G.nn[0] * (y + (long long)G.nn[1] * z);
}

// Waves per SIMD (the launch bound): two for the residual, the FD product and
// -- reading their corner values from the staged planes at every Gauss plane
// -- the analytic product and the two lean adjoint products; one for the
// adjoint with all outputs, which needs the whole register file.  kCoef (residual
// only): also write the cell means of a^2 for the preconditioner -- a
// separate instantiation, so that the plain residual carries no branch or
// store for it and profiles name the two kernels apart.
//
// Nodal linear part (ModeInfo::kNodal).  The tile's elements contribute to
// M y + theta D K x the tensor products of their 1-D matrices, and over the
// tile those assemble to products of 1-D three-point rows, the mass rows
// (h/6)(f_l + 2 a f + f_r) and the stiffness rows (1/h)((f - f_l) + (f - f_r)),
// with a the number of the tile's elements beside the node along that axis and
// absent neighbours left out.  Every difference is taken on the field itself
// and the mass rows act on the differences: differences of mass sums would lose
// two digits where x is smooth.  With P_k the share of plane k,
// m (Mx My y) + kx (My Kx x) + ky (Mx Ky x), and Q_k = q Mx My (x_k - x_(k+1)),
// an element layer between planes k and k + 1 adds 2 P_k + P_(k+1) + Q_k to
// plane k and P_k + 2 P_(k+1) - Q_k to plane k + 1.
// y, x and x_k - x_(k+1) of a plane are formed once per node, in LDS with a
// border of zeros, where the sums read 9 neighbours at fixed offsets.
// The residual's kernels are bound by FP64 issue (the vector ALUs issue in 81 %
// of its cycles): about 55 operations per node instead of 210 per element
// and a second field in the element vectors' LDS exchange.
//
// The node phase between a layer's two barriers is a third of a layer's time
// when its LDS reads wait for each other and one wave takes the 33 nodes beyond
// the 256 lanes after its own (6200 of 19000 clocks); with the reads of all
// slots issued together, both parts in one stream of instructions and one store
// per node it is 4300 of 17000, which the other workgroup of the compute unit
// fills with element work.  Measured (with k_fixup3): residual 257^3 nodes 1160
// -> 1040 us, FD product 1385 -> 1262 and on 129^3 201 -> 174, analytic product
// 1850 -> 1760, adjoint on 130 x 98 x 114 367 -> 326.
template <int MODE, bool kCoef = false>
__global__ void __launch_bounds__(kThreads, kWavesPerSimd<MODE>)
    k_fused3(Geo G, Tiles T, NodalLin L, const double2* __restrict__ U, const double2* __restrict__ Up,
             const double2* __restrict__ V, const double* __restrict__ eps_dev,
             const double2* __restrict__ F0, double2* __restrict__ out0, double2* __restrict__ out1,
             double* __restrict__ side, double* __restrict__ vjp_part, double* __restrict__ coef) {
  using MI = ModeInfo<MODE>;
  constexpr int NO = MI::NO, NE = MI::NE;
  constexpr bool kNodal = MI::kNodal;
  // residual and FD product hold their corner values in registers over the
  // Gauss planes; the others read them from the staged planes at every one
  constexpr bool kSrc = !(MODE == MODE_RES || MODE == MODE_FD);
  __shared__ double2 su[3][PN];
  __shared__ double2 sp[3][PN];
  __shared__ double2 sv[MI::kHasV ? 3 : 1][MI::kHasV ? PN : 1];
  // FD product: F0 of planes kz and kz + 1, so that the node writes need no load
  __shared__ double2 sf[MODE == MODE_FD ? 2 : 1][MODE == MODE_FD ? PN : 1];
  // element vectors for the node sums, all 8 corners; zeros for lanes without
  // an element and in the slot kThreads
  constexpr int kCb = kThreads + 1;
  __shared__ double cb[NE][8][kCb];

  const int tid = threadIdx.x;
  const int tile = (int)xcd_tile(blockIdx.x, gridDim.x);
  const int tx = tile % T.ntx;
  const int ty = (tile / T.ntx) % T.nty;
  const int tz = tile / (T.ntx * T.nty);
  const int x0 = tx * TX, y0 = ty * TY, z0 = tz * T.kz;
  const int lxmax = min(TX, G.n[0] - x0);  // last local node index in x
  const int lymax = min(TY, G.n[1] - y0);
  const int kzmax = min(T.kz, G.n[2] - z0);  // element layers in this chunk
  const int ei = tid % TX, ej = tid / TX;  // this lane's element column
  const bool has_elem = ei < lxmax && ej < lymax;
  // FD product: eps_dev holds eps and 1/eps (0 when eps is 0)
  const double eps = (MODE == MODE_FD) ? eps_dev[0] : 0.0;
  const double ieps = (MODE == MODE_FD) ? eps_dev[1] : 0.0;

  // A plane has more nodes than lanes.  Node sums: lane t takes node (t % 16,
  // t / 16), and one wave the 33 nodes of the last column and row, another
  // wave every layer, so that the four SIMDs share that work.  Copies (nodes
  // in storage order): likewise for the nodes beyond the first kThreads.
  constexpr int kSecond = PX + TY;
  static_assert(kSecond <= 64 && PN - kThreads <= 64 && TX == 16, "one wave takes the second part");
  // the lane's index, formed anew where it is used: what follows from it (node
  // coordinates, neighbours' offsets, flags) is then not kept in registers over
  // the element evaluation
  auto lane = [&]() {
    int t = tid;
    __asm__ volatile("" : "+v"(t));
    return t;
  };
  auto turn = [&](int t, int kz) { return __builtin_amdgcn_readfirstlane(t >> 6) == (kz & 3); };
  struct Node {
    int lx, ly, n;
    bool ok;  // in the tile's box
  };
  auto node1 = [&](int t) {
    const int lx = t % TX, ly = t / TX;
    return Node{lx, ly, lx + PX * ly, lx <= lxmax && ly <= lymax};
  };
  // lanes past the last of the 33 repeat it, so that the sums need no branch
  auto node2 = [&](int t) {
    const int k = min(t & 63, kSecond - 1);
    const int lx = k < PY ? TX : k - PY, ly = k < PY ? k : TY;
    return Node{lx, ly, lx + PX * ly, (t & 63) < kSecond && lx <= lxmax && ly <= lymax};
  };
  // per node of the plane: the contributions of the layer below, carried in
  // LDS (no registers held across the element evaluation).  Nodal linear part:
  // carry[1] also holds 2 P of the layer above.
  __shared__ double carry[NO][PN];
  for (int n = tid; n < PN; n += kThreads)
#pragma unroll
    for (int o = 0; o < NO; ++o) carry[o][n] = 0.0;
  // Nodal linear part: (y, x) and x_k - x_(k+1) of the plane kz + 1 and its
  // nodes' P (the lane's first node in a register)
  constexpr int kRow = PX + 1, kFields = kNodal ? kRow * (PY + 2) + 1 : 1;
  __shared__ double2 yx[kFields];
  __shared__ double xd[kFields];
  __shared__ double pn2[kNodal ? kSecond : 1];
  double pn1 = 0.0;

  // Plane z into ring slot `slot` by direct copies into LDS; the copies
  // complete by the wave's next wait_vm().
  auto dma_part = [&](int n, int slot, int z) {
    const int lx = n % PX, ly = n / PX;
    if (lx <= lxmax && ly <= lymax) {
      const long long g = gnode(G, x0 + lx, y0 + ly, z);
      dma16(U + g, su[slot], n);
      dma16(Up + g, sp[slot], n);
      if (MI::kHasV) dma16(V + g, sv[slot], n);
    }
  };
  auto dma_plane = [&](int slot, int z) {
    const int t = lane();
    dma_part(t, slot, z);
    if (turn(t, z) && (t & 63) < PN - kThreads) dma_part(kThreads + (t & 63), slot, z);
  };
  auto dma_f0 = [&](int lz) {
    if constexpr (MODE == MODE_FD) {
      auto part = [&](int n) {
        const int lx = n % PX, ly = n / PX;
        if (lx <= lxmax && ly <= lymax) dma16(F0 + gnode(G, x0 + lx, y0 + ly, z0 + lz), sf[lz & 1], n);
      };
      const int t = lane();
      part(t);
      if (turn(t, lz) && (t & 63) < PN - kThreads) part(kThreads + (t & 63));
    }
  };

  // FD product: U + eps V of node N in place of U, one layer before the plane is
  // read (at the corner reads it took 16 operations and 8 LDS reads per element:
  // 257^3 nodes 1268 -> 1253 us).
  auto perturb = [&](const Node& N, int slot) {
    if constexpr (MODE == MODE_FD) {
      if (!N.ok) return;
      double2 u = su[slot][N.n];
      const double2 v = sv[slot][N.n];
      u.x = fma(eps, v.x, u.x);
      u.y = fma(eps, v.y, u.y);
      su[slot][N.n] = u;
    }
  };
  // The fields of the nodal linear part at node N of the staged plane in `slot`.
  auto fields = [&](const Node& N, int slot) {
    if (!N.ok) return;
    const int q = kRow + 1 + N.lx + kRow * N.ly;
    double y, x;
    if constexpr (MODE == MODE_JVP) {
      const double2 v = sv[slot][N.n];
      y = fma(-G.hth, v.x, v.y);
      x = v.y;
    } else {
      const double2 u = su[slot][N.n], p = sp[slot][N.n];
      y = fma(-G.hth, u.x - p.x, u.y - p.y);
      x = u.y;
    }
    xd[q] = yx[q].y - x;
    yx[q] = make_double2(y, x);
  };
  // P of node (lx, ly) of the plane whose fields are formed, and Q of the plane
  // below it.
  auto nodal = [&](int lx, int ly, double& P, double& Q) {
    const double l = lx > 0 ? 1.0 : 0.0, r = lx < lxmax ? 1.0 : 0.0;
    const double d = ly > 0 ? 1.0 : 0.0, t = ly < lymax ? 1.0 : 0.0;
    const double ax = l + r, ay = d + t;
    const double ax2 = ax + ax, ay2 = ay + ay;
    double m[3][3], x[3][3], z[3][3];
#pragma unroll
    for (int dy = 0; dy < 3; ++dy)
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        const int q = lx + dx + kRow * (ly + dy);
        const double2 v = yx[q];
        m[dy][dx] = v.x;
        x[dy][dx] = v.y;
        z[dy][dx] = xd[q];
      }
    // mass rows along x and y, and the stiffness rows
    auto mass = [](double a2, const double (&f)[3]) { return fma(a2, f[1], f[0] + f[2]); };
    double Mm[3], Mz[3], Kx[3], Ky[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      Mm[k] = mass(ax2, m[k]);
      Mz[k] = mass(ax2, z[k]);
      Kx[k] = fma(l, x[k][1], -x[k][0]) + fma(r, x[k][1], -x[k][2]);
      Ky[k] = fma(d, x[1][k], -x[0][k]) + fma(t, x[1][k], -x[2][k]);
    }
    P = fma(L.m, mass(ay2, Mm), fma(L.kx, mass(ay2, Kx), L.ky * mass(ax2, Ky)));
    Q = L.q * mass(ay2, Mz);
  };

  const long long tile_base = (long long)tile * side_nodes(T.kz);
  // Write the sum of a node of plane lz: final value or side-buffer partial
  // (always the latter on the tile's last column and row: kSide).  One store
  // per output whichever it is: every wave has nodes of both kinds.
  double2* const side_base = reinterpret_cast<double2*>(side) + tile_base * (NO / 2);
  auto emit = [&](auto kSide, const Node& N, int lz, const double* acc) {
    const int lx = N.lx, ly = N.ly;
    const bool ring = kSide() || lx == 0 || lx == lxmax || ly == 0 || ly == lymax || lz == 0 || lz == kzmax;
    double2* const ps = side_base + side_slot(lx, ly, lz, lxmax, lymax, kzmax) * (NO / 2);
    const long long g = gnode(G, x0 + lx, y0 + ly, z0 + lz);
    if constexpr (MODE == MODE_FD) {
      // the tile that owns the node in the fixup (below its upper extent
      // along every axis, or on the mesh's upper face) subtracts F0 from its
      // partial, so that the fixup needs no F0: Jv = (sum of partials)/eps
      const bool owned = (lx < lxmax || tx == T.ntx - 1) && (ly < lymax || ty == T.nty - 1) &&
                         (lz < kzmax || tz == T.ntz - 1);
      double2 f0 = sf[lz & 1][N.n];
      if (ring && !owned) f0 = make_double2(0.0, 0.0);
      const double sc = ring ? 1.0 : ieps;
      *(ring ? ps : out0 + g) = make_double2((acc[0] - f0.x) * sc, (acc[1] - f0.y) * sc);
    } else {
      if (ring || out0) *(ring ? ps : out0 + g) = make_double2(acc[0], acc[1]);
      if (NO == 4 && (ring || out1)) *(ring ? ps + 1 : out1 + g) = make_double2(acc[2 % NO], acc[3 % NO]);
    }
  };

  // Node n of plane kz: its sum is complete (bottom corners of layer kz and
  // the carried part) and written; the top corners are carried to plane kz + 1.
  // Every element's slot is read without a branch (the zero slot for absent
  // ones), so that all LDS reads of a node are in flight together: with one
  // branch per element the reads of a layer's two sums cost 8 LDS latencies.
  auto finish = [&](const Node& N, int kz, double& pn, double (&acc)[NO]) {
    const int lx = N.lx, ly = N.ly, n = N.n;
    double P = 0.0, Q = 0.0;
    if constexpr (kNodal) nodal(lx, ly, P, Q);
    const bool le = lx > 0, re = lx < TX, de = ly > 0, te = ly < TY;
    const int e = lx + TX * ly;
    const int slot[4] = {le && de ? e - TX - 1 : kThreads, re && de ? e - TX : kThreads,
                         le && te ? e - 1 : kThreads, re && te ? e : kThreads};
    double up[NE];
#pragma unroll
    for (int o = 0; o < NE; ++o) {
      // corner 3 - k of the k-th element around the node
      acc[o] = cb[o][3][slot[0]] + cb[o][2][slot[1]] + cb[o][1][slot[2]] + cb[o][0][slot[3]];
      up[o] = cb[o][7][slot[0]] + cb[o][6][slot[1]] + cb[o][5][slot[2]] + cb[o][4][slot[3]];
      acc[o] += carry[o][n];
    }
    if constexpr (kNodal) {
      acc[0] *= G.theta;
      acc[1] = carry[1][n] + (P + Q);
      carry[1][n] = (pn - Q) + (kz + 1 < kzmax ? 4.0 : 2.0) * P;
      pn = P;
    }
#pragma unroll
    for (int o = 0; o < NE; ++o) carry[o][n] = up[o];
  };
  const auto first_part = std::integral_constant<bool, false>{};
  const auto second_part = std::integral_constant<bool, true>{};

  double ge = 0.0, gl = 0.0;
  for (int n = tid; n < NE * 8 * kCb; n += kThreads) (&cb[0][0][0])[n] = 0.0;
  for (int n = tid; kNodal && n < kFields; n += kThreads) {
    yx[n] = make_double2(0.0, 0.0);
    xd[n] = 0.0;
  }
  dma_plane(0, z0);
  dma_plane(1, z0 + 1);
  dma_f0(0);
  wait_vm();
  __syncthreads();
  if constexpr (kNodal) {
    for (int slot = 0; slot < 2; ++slot) {
      perturb(node1(tid), slot);
      if (turn(tid, 0)) perturb(node2(tid), slot);
    }
    fields(node1(tid), 0);
    if (turn(tid, 0)) fields(node2(tid), 0);
    __syncthreads();
    auto start = [&](const Node& N, double& pn) {
      double Q;
      nodal(N.lx, N.ly, pn, Q);
      carry[1][N.n] = pn + pn;
    };
    start(node1(tid), pn1);
    if (turn(tid, 0)) start(node2(tid), pn2[min(tid & 63, kSecond - 1)]);
    __syncthreads();
  }
  for (int kz = 0; kz < kzmax; ++kz) {
    // ring slots: plane kz in kz % 3
    const int bot = kz % 3, top = (kz + 1) % 3;
    auto at = [&](int a) {
      return ((a & 4) ? top : bot) * PN + (ei + (a & 1)) + PX * (ej + ((a >> 1) & 1));
    };
    // the next-but-one plane: slot (kz + 2) % 3 last held plane kz - 1, which
    // no lane reads any more
    auto ahead = [&]() {
      if (kz + 2 <= kzmax) dma_plane((kz + 2) % 3, z0 + kz + 2);
      dma_f0(kz + 1);
    };
    double u0[8], u1[8], p0[8], p1[8], v0[8], v1[8];
    if (!kSrc && has_elem) {
#pragma unroll
      for (int a = 0; a < 8; ++a) {
        const int n = at(a);
        const double2 u = su[0][n];
        u0[a] = u.x;
        u1[a] = u.y;
        p0[a] = sp[0][n].x;
        p1[a] = v0[a] = v1[a] = 0.0;
      }
    }
    // copied once the corner values are in registers (the compiler orders LDS
    // reads of the ring after copies into it)
    if (!(kSrc && has_elem)) ahead();
    if (has_elem) {
      double eg = 0.0, lg = 0.0;
      if constexpr (kSrc) {
        // corner values straight from the staged planes at every Gauss plane;
        // the next-but-one plane is copied after the first plane's reads (its
        // copy then overlaps the first plane's work: the reads of the next
        // planes wait for it)
        auto corner = [&](int a, double2& u, double2& p, double2& v) {
          const int n = at(a);
          u = su[0][n];
          p = sp[0][n];
          v = sv[0][n];
        };
        auto plane = [&](int) { __asm__ volatile("" ::: "memory"); };
        auto loaded = [&](int gz) {
          if (gz == 0) ahead();
        };
        LdsCorners<decltype(corner), decltype(plane), decltype(loaded)> src{corner, plane, loaded,
                                                                            &cb[0][0][tid], 8 * kCb, kCb};
        Element<3, MODE>::run_src(G, src, eg, lg);
      } else {
        double out[2][8];
        Element<3, MODE>::run(G, u0, u1, p0, p1, v0, v1, out, eg, lg);
#pragma unroll
        for (int a = 0; a < 8; ++a) cb[0][a][tid] = out[0][a];
      }
      if (MODE == MODE_RES) {
        // cell mean of a^2 for the preconditioner (weights sum to 8 jac)
        if (kCoef) coef[(x0 + ei) + (long long)G.n[0] * ((y0 + ej) + (long long)G.n[1] * (z0 + kz))] =
            eg / (8.0 * G.jac);
      } else {
        ge += eg;
        gl += lg;
      }
    }
    if constexpr (kNodal) {
      const int t = lane();
      fields(node1(t), top);
      if (turn(t, kz)) fields(node2(t), top);
    }
    // the copies of this layer are complete here, before the node writes go
    // out: waiting for them at the end of the layer would wait for the writes
    // as well
    wait_vm();
    lds_barrier();
    // the wave of the other workgroup on this SIMD is in its element
    // evaluation most of the time and fills what this phase leaves idle
    // (residual 1094 -> 1079 us at 256^3; the tangent and adjoint kernels gain
    // nothing)
    if (!kSrc) __builtin_amdgcn_s_setprio(2);
    {
      const int t = lane();
      const Node N = node1(t);
      double acc[NO];
      const bool ahead2 = MODE == MODE_FD && kz + 2 <= kzmax;
      if (ahead2) perturb(N, (kz + 2) % 3);
      if (turn(t, kz)) {
        const Node N2 = node2(t);
        double acc2[NO];
        if (ahead2) perturb(N2, (kz + 2) % 3);
        finish(N, kz, pn1, acc);
        finish(N2, kz, pn2[min(t & 63, kSecond - 1)], acc2);
        if (N.ok) emit(first_part, N, kz, acc);
        if (N2.ok) emit(second_part, N2, kz, acc2);
      } else {
        finish(N, kz, pn1, acc);
        if (N.ok) emit(first_part, N, kz, acc);
      }
    }
    if (!kSrc) __builtin_amdgcn_s_setprio(0);
    lds_barrier();
  }
  {
    auto last = [&](const Node& N) {
      if (!N.ok) return;
      double acc[NO];
#pragma unroll
      for (int o = 0; o < NO; ++o) acc[o] = carry[o][N.n];
      if constexpr (kNodal) acc[0] *= G.theta;
      emit(second_part, N, kzmax, acc);
    };
    last(node1(tid));
    if (turn(tid, kzmax)) last(node2(tid));
  }

  if (MODE == MODE_VJP || MODE == MODE_VJPP) {
    // fixed-order block reduction of the parameter sums (cb reused as scratch)
    double* red = &cb[0][0][0];
    red[tid] = ge;
    red[kThreads + tid] = gl;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
      if (tid < w) {
        red[tid] += red[tid + w];
        red[kThreads + tid] += red[kThreads + tid + w];
      }
      __syncthreads();
    }
    if (tid == 0) {
      vjp_part[tile] = red[0];
      vjp_part[gridDim.x + tile] = red[kThreads];
    }
  }
}

// Tiles containing coordinate c along an axis with tile width w and tile count
// nt: t[0] (node l[0] of it) and, for two, t[1] (l[1]); returns whether there
// are two, else t[1], l[1] repeat the first.
__device__ __forceinline__ bool axis_tiles(int c, int w, int nt, int (&t)[2], int (&l)[2]) {
  const int hi = c / w;
  const bool face = c % w == 0;
  const bool below = face && hi > 0, above = hi < nt;
  t[0] = below ? hi - 1 : hi;
  l[0] = below ? w : c - hi * w;
  t[1] = above ? hi : t[0];
  l[1] = above ? c - hi * w : l[0];
  return below && above;
}

// fix_parts workgroups per tile, one slot per lane: the ring nodes the tile
// owns -- those whose local coordinates are below the tile's upper extent along
// every axis, or on the mesh's upper face along that axis -- each receive the
// sum of the partials of all tiles sharing the node, taken in increasing tile
// order.  The tile's own side-buffer slots enumerate its ring nodes (a superset
// of the owned ones).  Bound by the latency of the partials' loads, which are
// issued together (at most 8, only those that exist): 257^3 nodes, 79 us with one
// workgroup per tile and the loads one after the other, 62 us now; 129^3 nodes,
// 18 -> 9.
__host__ __device__ constexpr int fix_parts(int kz) { return (side_nodes(kz) + 255) / 256; }

template <int MODE>
__global__ void __launch_bounds__(256)
    k_fixup3(Geo G, Tiles T, const double* __restrict__ side,
             const double* __restrict__ eps_dev, double2* __restrict__ out0,
             double2* __restrict__ out1) {
  constexpr int NO = ModeInfo<MODE>::NO;
  const int block = (int)xcd_tile(blockIdx.x, gridDim.x);
  const int parts = fix_parts(T.kz), nside = side_nodes(T.kz);
  const int tile = block / parts;
  const int tx = tile % T.ntx;
  const int ty = (tile / T.ntx) % T.nty;
  const int tz = tile / (T.ntx * T.nty);
  const int x0 = tx * TX, y0 = ty * TY, z0 = tz * T.kz;
  const int lxmax = min(TX, G.n[0] - x0);
  const int lymax = min(TY, G.n[1] - y0);
  const int kzmax = min(T.kz, G.n[2] - z0);
  const bool lastx = tx == T.ntx - 1, lasty = ty == T.nty - 1, lastz = tz == T.ntz - 1;
  const double ie = MODE == MODE_FD ? eps_dev[1] : 0.0;  // 1/eps
  const int i = (block % parts) * 256 + (int)threadIdx.x;
  if (i >= nside) return;
  int lx, ly, lz;
  if (i < PN) {
    lz = 0;
    lx = i % PX;
    ly = i / PX;
  } else if (i < 2 * PN) {
    if (!lastz) return;  // the next tile's first plane
    lz = kzmax;
    lx = (i - PN) % PX;
    ly = (i - PN) / PX;
  } else {
    const int j = i - 2 * PN;
    lz = 1 + j / RING;
    if (lz >= kzmax || !ring_node(j % RING, lxmax, lymax, lx, ly)) return;
  }
  if (lx > lxmax || ly > lymax) return;
  if ((lx == lxmax && !lastx) || (ly == lymax && !lasty)) return;  // a neighbour's node
  const int x = x0 + lx, y = y0 + ly, z = z0 + lz;
  int txs[2], lxs[2], tys[2], lys[2], tzs[2], lzs[2];
  const bool nx = axis_tiles(x, TX, T.ntx, txs, lxs);
  const bool ny = axis_tiles(y, TY, T.nty, tys, lys);
  const bool nz = axis_tiles(z, T.kz, T.ntz, tzs, lzs);
  const double2* const side2 = reinterpret_cast<const double2*>(side);
  double2 v[8][NO / 2];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int a = k & 1, b = (k >> 1) & 1, c = k >> 2;
#pragma unroll
    for (int o = 0; o < NO / 2; ++o) v[k][o] = make_double2(0.0, 0.0);
    if ((a == 0 || nx) && (b == 0 || ny) && (c == 0 || nz)) {
      const long long t = txs[a] + (long long)T.ntx * (tys[b] + (long long)T.nty * tzs[c]);
      const int slot = side_slot(lxs[a], lys[b], lzs[c], min(TX, G.n[0] - TX * txs[a]),
                                 min(TY, G.n[1] - TY * tys[b]), min(T.kz, G.n[2] - T.kz * tzs[c]));
#pragma unroll
      for (int o = 0; o < NO / 2; ++o) v[k][o] = side2[(t * nside + slot) * (NO / 2) + o];
    }
  }
#pragma unroll
  for (int k = 1; k < 8; ++k)
#pragma unroll
    for (int o = 0; o < NO / 2; ++o) {
      v[0][o].x += v[k][o].x;
      v[0][o].y += v[k][o].y;
    }
  const long long g = gnode(G, x, y, z);
  if (MODE == MODE_FD) {
    // the owning tile's partial already holds -F0 (k_fused3)
    out0[g] = make_double2(v[0][0].x * ie, v[0][0].y * ie);
  } else {
    if (out0) out0[g] = v[0][0];
    if (NO == 4 && out1) out1[g] = v[0][NO / 2 - 1];
  }
}

// The z-chunks of a mode: the division of the mesh into tiles whose estimated
// time is least.  `resident` workgroups run at a time, one or two per compute
// unit; two on a compute unit take 1.67 times as long per layer as one (residual:
// 8.0 and 4.8 us), and a chunk costs one layer besides its own.  Short chunks
// where the mesh has few tiles, and equal ones: 16 layers each, the rest in the
// last chunk, were before.  Residual 64^3 89 -> 31 us, 20^3 92 -> 14, 100 x 150 x
// 60 155 -> 90; adjoint 129 x 97 x 113 326 -> 287; 256^3 1054 with 16 layers, 1048
// with 32.
//
// The division depends on the mesh and the mode alone (results are reproducible
// and alike for all callers).  Its side buffer takes at most what 16 layers
// each would take, or kSideMost doubles per output.
constexpr int kCus = 256, kMostLayers = 32, kMostShort = 8 * kCus;
constexpr long long kSideMost = (long long)kMostShort * side_nodes(15);
static_assert(kSideMost * 2 * sizeof(double) <= 64LL << 20, "fits the fixed array of the call without allocation");

Tiles tiles_for(const Geo& G, int resident) {
  Tiles T;
  T.ntx = (G.n[0] + TX - 1) / TX;
  T.nty = (G.n[1] + TY - 1) / TY;
  const long long columns = (long long)T.ntx * T.nty;
  double best = 0.0;
  T.kz = 0;
  for (int c = 1; c <= kMostLayers; ++c) {
    const int nz = (G.n[2] + c - 1) / c;
    const int kz = (G.n[2] + nz - 1) / nz;  // nz equal chunks
    const long long tiles = columns * nz, rounds = tiles / resident, rest = tiles % resident;
    if (nz > (G.n[2] + 15) / 16 && tiles > kMostShort) continue;
    const double full = resident > kCus ? 1.67 : 1.0;
    const double cost = (kz + 1) * (rounds * full + (rest == 0 ? 0.0 : rest <= kCus ? 1.0 : full));
    if (T.kz == 0 || cost <= best) {
      best = cost;
      T.kz = kz;
    }
  }
  T.ntz = (G.n[2] + T.kz - 1) / T.kz;
  return T;
}

// Workgroups of a mode that run at a time.  (With the all-outputs product's
// division the previous-state product, at two waves per SIMD, took 178 us on 129 x
// 97 x 113 and 361 on 4 x 4 x 20000; with its own 159 and 283.)
template <int MODE>
constexpr int kResident = kCus * kWavesPerSimd<MODE>;

int tile_count(const Tiles& T) { return T.ntx * T.nty * T.ntz; }

// side: the tile-face partial sums, fused3_side_len(G) doubles (the first
// tiles x side_nodes x NO of them are used).
template <int MODE>
int launch_mode(const Geo& G, double* side, const double* U, const double* Uprev, const double* v,
                const double* F0, const double* eps_dev, double* out0, double* out1,
                double* vjp_part, double* coef, hipStream_t s) {
  const Tiles T = tiles_for(G, kResident<MODE>);
  const unsigned nt = (unsigned)tile_count(T);
  const NodalLin L = nodal_lin(G);
  auto d2 = [](const double* p) { return reinterpret_cast<const double2*>(p); };
  bool with_coef = false;
  if constexpr (MODE == MODE_RES) with_coef = coef != nullptr;
  if constexpr (MODE == MODE_RES) {
    if (with_coef)
      hipLaunchKernelGGL((k_fused3<MODE_RES, true>), dim3(nt), dim3(kThreads), 0, s, G, T, L, d2(U),
                         d2(Uprev), d2(v), eps_dev, d2(F0), reinterpret_cast<double2*>(out0),
                         reinterpret_cast<double2*>(out1), side, vjp_part, coef);
  }
  if (!with_coef)
    hipLaunchKernelGGL((k_fused3<MODE, false>), dim3(nt), dim3(kThreads), 0, s, G, T, L, d2(U),
                       d2(Uprev), d2(v), eps_dev, d2(F0), reinterpret_cast<double2*>(out0),
                       reinterpret_cast<double2*>(out1), side, vjp_part, nullptr);
  PF_HIP_CHECK(hipGetLastError());
  hipLaunchKernelGGL((k_fixup3<MODE>), dim3(nt * fix_parts(T.kz)), dim3(256), 0, s, G, T, side,
                     eps_dev, reinterpret_cast<double2*>(out0), reinterpret_cast<double2*>(out1));
  PF_HIP_CHECK(hipGetLastError());
  return PF_OK;
}

}  // namespace

long long fused3_side_len(const Geo& G) {
  long long most = 0;
  auto mode = [&](int resident, int NO) {
    const Tiles T = tiles_for(G, resident);
    most = std::max(most, (long long)tile_count(T) * side_nodes(T.kz) * NO);
  };
  mode(kResident<MODE_RES>, 2);
  mode(kResident<MODE_JVP>, 2);
  mode(kResident<MODE_VJPU>, 2);
  mode(kResident<MODE_VJPP>, 2);
  mode(kResident<MODE_VJP>, 4);
  return most;
}

int fused3_tiles(const Geo& G, int mode) {
  return tile_count(tiles_for(G, mode == MODE_VJPP ? kResident<MODE_VJPP> : kResident<MODE_VJP>));
}

// At least what chunks of 16 layers would take, the size that callers with a
// fixed buffer document (the division in use exceeds it only below kSideMost
// doubles per output).
long long fused3_residual_side_len(const Geo& G) {
  const Tiles T = tiles_for(G, kResident<MODE_RES>);
  const long long by16 = (long long)T.ntx * T.nty * ((G.n[2] + 15) / 16) * side_nodes(16);
  return std::max(by16, (long long)tile_count(T) * side_nodes(T.kz)) * ModeInfo<MODE_RES>::NO;
}

int launch_fused3_residual(const Geo& G, double* side, const double* U, const double* Uprev,
                           double* F, hipStream_t s) {
  return launch_mode<MODE_RES>(G, side, U, Uprev, nullptr, nullptr, nullptr, F, nullptr, nullptr,
                               nullptr, s);
}

int launch_fused3(pf_problem* pb, int mode, const double* U, const double* Uprev, const double* v,
                  const double* F0, const double* eps_dev, double* out0, double* out1,
                  double* vjp_part, double* coef, hipStream_t s) {
  const Geo& G = pb->geo;
  double* side = pb->side_buf;
  switch (mode) {
    case MODE_RES:
      return launch_mode<MODE_RES>(G, side, U, Uprev, v, F0, eps_dev, out0, out1, vjp_part, coef, s);
    case MODE_FD:
      return launch_mode<MODE_FD>(G, side, U, Uprev, v, F0, eps_dev, out0, out1, vjp_part, nullptr, s);
    case MODE_JVP:
      return launch_mode<MODE_JVP>(G, side, U, Uprev, v, F0, eps_dev, out0, out1, vjp_part, nullptr, s);
    case MODE_VJPU:
      return launch_mode<MODE_VJPU>(G, side, U, Uprev, v, F0, eps_dev, out0, out1, vjp_part, nullptr, s);
    case MODE_VJPP:
      return launch_mode<MODE_VJPP>(G, side, U, Uprev, v, F0, eps_dev, out0, out1, vjp_part, nullptr, s);
    default:
      return launch_mode<MODE_VJP>(G, side, U, Uprev, v, F0, eps_dev, out0, out1, vjp_part, nullptr, s);
  }
}

}  // namespace pf
