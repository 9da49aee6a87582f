// The 2-D V-cycle in few launches.  Included by pf_gmg.hip after the level
// definitions (LvK, V2, div_diag).
//
// A 2-D level is small (a 1025^2 grid of FP64 pairs is 17 MB, less than the last
// cache holds) and a sweep over it costs a launch, about 3 us, rather than its
// memory traffic: a V-cycle of a 512^2 mesh took 43 launches.  So several steps
// run per launch on a region held by one workgroup, overlapping its neighbours
// by one node per step:
//   k_down2   both pre-smoothing steps, the residual and its restriction;
//   k_up2     the prolongation and both post-smoothing steps;
//   k_cheb2   4 or 8 steps of the coarsest solve (coarsest grids that do not
//             fit one workgroup);
//   k_tail2   the whole cycle from the first level of at most 1024 nodes down,
//             by one workgroup.
// One lane holds one node of the region and keeps its stencil weights, its
// right-hand side and its direction in registers; the iterates go through LDS.
// Each step's result is wrong in the region's outermost ring of still valid
// nodes, so the valid part shrinks by one node per step: with 16 x 16 lanes
// k_down2 owns 10 x 10 fine nodes (5 x 5 coarse ones) and k_up2 12 x 12; with
// 32 x 32 lanes k_cheb2 owns 16 x 16 nodes (8 steps) or 24 x 24 (4 steps);
// regions2 gives narrow grids others.  The
// nodes evaluated more than once cost less than the launches.  One V-cycle, FP64,
// by launch per step and now: 64^2 77 -> 30 us, 150^2 67 -> 22, 512^2 172 -> 61,
// 1024^2 252 -> 99, 1023 x 1001 (one level) 292 -> 128.
//
// Regions of 32 x 32 lanes for k_down2 and k_up2 evaluate fewer nodes twice, but
// their 16 wavefronts step more slowly than 4: 512^2 62 us, 1024^2 103 us.

constexpr int kReg2 = 16;                  // region side of k_down2 and k_up2
constexpr int kDown2 = (kReg2 - 6) / 2;    // coarse nodes per side owned by k_down2
constexpr int kUp2 = kReg2 - 4;            // fine nodes per side owned by k_up2
constexpr int kRegC2 = 32;                 // side of k_cheb2's square region
constexpr int kCheb2Lanes = kRegC2 * kRegC2;
constexpr int kTail2Lanes = 1024;          // most nodes of k_tail2's first level
constexpr int kTail2Levels = 6;            // most levels k_tail2 takes

// Stencil of one node, phi and u blocks, zero towards missing neighbours, and
// the reciprocals of the two diagonals (a node takes them up to 16 times; a
// division each time cost as much as the stencil's sums).
template <class T>
struct Node2 {
  T w0[9], w1[9];
  T rd0, rd1;
};
__device__ __forceinline__ float rcp_diag(float d) { return __builtin_amdgcn_rcpf(d); }
__device__ __forceinline__ double rcp_diag(double d) { return 1.0 / d; }

// Weights of node (ix, iy) from the phi-block cell coefficients c (memory or
// LDS); all zero for nodes outside the mesh.
template <class T>
__device__ __forceinline__ void node2(const LvK& g, const T* c, int ix, int iy, bool in, Node2<T>& N) {
  T cc[1][2][2];
  const bool ex[2] = {in && ix > 0, in && ix < g.n[0]}, ey[2] = {in && iy > 0, in && iy < g.n[1]};
  const bool ez[2] = {true, true};
#pragma unroll
  for (int by = 0; by < 2; ++by)
#pragma unroll
    for (int bx = 0; bx < 2; ++bx)
      cc[0][by][bx] = ex[bx] && ey[by] ? c[(ix - 1 + bx) + (long long)g.n[0] * (iy - 1 + by)] : (T)0;
  stencil_weights<2, T>(g, cc, ex, ey, ez, N.w0, N.w1);
  N.rd0 = in ? rcp_diag(N.w0[4]) : (T)0;
  N.rd1 = in ? rcp_diag(N.w1[4]) : (T)0;
}

// (A x)_i with the neighbours at xs[at + dx + dy * row].  lo/hi: whether the
// neighbour column and row on that side may be read (else the node itself
// stands in: its weight is 0, or the result is not used).
template <class T>
__device__ __forceinline__ void apply2(const Node2<T>& N, const typename V2<T>::type* xs, int at,
                                       int row, bool xlo, bool xhi, bool ylo, bool yhi, T& y0, T& y1) {
  // one sum per row of the stencil: three short chains instead of a long one
  T s0[3], s1[3];
#pragma unroll
  for (int ty = 0; ty < 3; ++ty) {
    const int oy = ty == 0 ? (ylo ? -row : 0) : (ty == 2 ? (yhi ? row : 0) : 0);
    s0[ty] = 0;
    s1[ty] = 0;
#pragma unroll
    for (int tx = 0; tx < 3; ++tx) {
      const int ox = tx == 0 ? (xlo ? -1 : 0) : (tx == 2 ? (xhi ? 1 : 0) : 0);
      const auto v = xs[at + oy + ox];
      s0[ty] += N.w0[tx + 3 * ty] * v.x;
      s1[ty] += N.w1[tx + 3 * ty] * v.y;
    }
  }
  y0 = (s0[0] + s0[2]) + s0[1];
  y1 = (s1[0] + s1[2]) + s1[1];
}

// Coefficients of a level's two smoothing steps, per block.
template <class T>
struct Cheb2 {
  T be0[2], al1[2], be1[2];
};

// Right-hand side of a node: the level's array, or the FP64 input r64.
template <class T, bool TOP>
__device__ __forceinline__ typename V2<T>::type rhs2(const typename V2<T>::type* b, const double2* r64,
                                                     long long i) {
  if constexpr (TOP) {
    const double2 v = r64[i];
    typename V2<T>::type o;
    o.x = (T)v.x;
    o.y = (T)v.y;
    return o;
  } else {
    return b[i];
  }
}

// The sum over the 3 x 3 fine nodes around a coarse node, weights 1/2, 1, 1/2
// per axis; r at fine neighbour (dx, dy) is load(dx, dy), not called for nodes
// outside the mesh.
template <class T, class Load>
__device__ __forceinline__ typename V2<T>::type restrict2(const LvK& fg, int cx, int cy, Load load) {
  T a0 = 0, a1 = 0;
#pragma unroll
  for (int dy = -1; dy <= 1; ++dy) {
    const int fy = 2 * cy + dy;
    if (fy < 0 || fy >= fg.nn[1]) continue;
    const T wy = dy == 0 ? (T)1 : (T)0.5;
#pragma unroll
    for (int dx = -1; dx <= 1; ++dx) {
      const int fx = 2 * cx + dx;
      if (fx < 0 || fx >= fg.nn[0]) continue;
      const T w = (dx == 0 ? (T)1 : (T)0.5) * wy;
      const auto v = load(dx, dy);
      a0 += w * v.x;
      a1 += w * v.y;
    }
  }
  typename V2<T>::type o;
  o.x = a0;
  o.y = a1;
  return o;
}

// x + (P e) at fine node (ix, iy), e the coarse values (row length cn0).
template <class T>
__device__ __forceinline__ typename V2<T>::type prolong2(typename V2<T>::type x,
                                                         const typename V2<T>::type* e, int cn0, int ix,
                                                         int iy) {
  const int ox = ix & 1, oy = iy & 1;
  const int I = (ix >> 1) + cn0 * (iy >> 1);
  const auto e00 = e[I], e10 = e[I + ox], e01 = e[I + cn0 * oy], e11 = e[I + ox + cn0 * oy];
  T a0 = e00.x, a1 = e00.y;
  a0 += ox ? e10.x : (T)0;
  a1 += ox ? e10.y : (T)0;
  a0 += oy ? e01.x : (T)0;
  a1 += oy ? e01.y : (T)0;
  a0 += ox && oy ? e11.x : (T)0;
  a1 += ox && oy ? e11.y : (T)0;
  const T w = (ox ? (T)0.5 : (T)1) * (oy ? (T)0.5 : (T)1);
  x.x += w * a0;
  x.y += w * a1;
  return x;
}

// This lane's place in a region whose first node is (x0, y0).
struct Lane2 {
  int tx, ty, ix, iy;
  bool in;               // the node is in the mesh
  bool xlo, xhi, ylo, yhi;  // neighbours inside the region
  long long i;           // node index (0 outside the mesh)
};
__device__ __forceinline__ Lane2 lane2(const LvK& g, int x0, int y0, int tx, int ty, int w, int h) {
  Lane2 L;
  L.tx = tx;
  L.ty = ty;
  L.ix = x0 + tx;
  L.iy = y0 + ty;
  const bool held = ty < h;  // lanes beyond the region hold nothing and read themselves
  L.in = held && L.ix >= 0 && L.ix < g.nn[0] && L.iy >= 0 && L.iy < g.nn[1];
  L.xlo = held && tx > 0;
  L.xhi = held && tx < w - 1;
  L.ylo = held && ty > 0;
  L.yhi = held && ty < h - 1;
  L.i = L.in ? L.ix + (long long)g.nn[0] * L.iy : 0;
  return L;
}
template <int R>
__device__ __forceinline__ Lane2 lane2(const LvK& g, int x0, int y0) {
  return lane2(g, x0, y0, (int)threadIdx.x % R, (int)threadIdx.x / R, R, R);
}

// The regions of a k_cheb2 launch of S steps: w x h lanes, of which the S
// outermost columns (hx = S) and rows (hy = S) overlap the neighbouring regions;
// ntx regions along x, nt in all.  mul: lane / w = lane * mul >> 20.
struct Regions2 {
  int w, h, hx, hy;
  unsigned ntx, nt, mul;
};
inline Regions2 regions2(const LvK& g, int S) {
  auto make = [&](int w, int h, int hx, int hy) {
    const unsigned ox = (unsigned)(w - 2 * hx), oy = (unsigned)(h - 2 * hy);
    Regions2 R{w, h, hx, hy, ((unsigned)g.nn[0] + ox - 1) / ox, 0, ((1u << 20) + (unsigned)w - 1) / (unsigned)w};
    R.nt = R.ntx * (((unsigned)g.nn[1] + oy - 1) / oy);
    return R;
  };
  // narrow grids: regions as wide (high) as the grid, which overlap along one
  // axis only, where that gives fewer (FP64 cycle
  // of 1 x 10^6 elements 2162 -> 145 us, of 4 x 250000 551 -> 99 us)
  Regions2 best = make(kRegC2, kRegC2, S, S);
  const int most = kCheb2Lanes / (2 * S + 1);
  auto take = [&](const Regions2& R) {
    if (R.nt < best.nt) best = R;
  };
  if (g.nn[0] <= most) take(make(g.nn[0], kCheb2Lanes / g.nn[0], 0, S));
  if (g.nn[1] <= most) take(make(kCheb2Lanes / g.nn[1], g.nn[1], S, 0));
  return best;
}

// Pre-smoothing from zero, residual and restriction: x (fine nodes) and bc
// (coarse nodes) of the tile the workgroup owns.
template <class T, bool TOP>
__global__ void __launch_bounds__(kReg2 * kReg2)
    k_down2(LvK g, LvK cg, const T* __restrict__ c, const typename V2<T>::type* __restrict__ b,
            const double2* __restrict__ r64, Cheb2<T> K, typename V2<T>::type* __restrict__ x,
            typename V2<T>::type* __restrict__ bc) {
  using T2 = typename V2<T>::type;
  __shared__ T2 xs[2][kReg2 * kReg2];
  constexpr int O = kDown2;
  const int ntx = (cg.nn[0] + O - 1) / O;
  const int tile = (int)xcd_tile(blockIdx.x, gridDim.x);
  const int X0 = (tile % ntx) * O, Y0 = (tile / ntx) * O;
  const Lane2 L = lane2<kReg2>(g, 2 * X0 - 3, 2 * Y0 - 3);
  const int t = (int)threadIdx.x;
  T2 bb{};
  if (L.in) bb = rhs2<T, TOP>(b, r64, L.i);
  Node2<T> N;
  node2<T>(g, c, L.ix, L.iy, L.in, N);
  // x1 = beta_0 D^-1 b, also the step's direction
  T2 v;
  v.x = (K.be0[0] * bb.x) * N.rd0;
  v.y = (K.be0[1] * bb.y) * N.rd1;
  xs[0][t] = v;
  __syncthreads();
  T y0, y1;
  apply2<T>(N, xs[0], t, kReg2, L.xlo, L.xhi, L.ylo, L.yhi, y0, y1);
  v.x = v.x + (K.al1[0] * v.x + (K.be1[0] * (bb.x - y0)) * N.rd0);
  v.y = v.y + (K.al1[1] * v.y + (K.be1[1] * (bb.y - y1)) * N.rd1);
  xs[1][t] = v;
  if (L.in && L.tx >= 3 && L.tx < 3 + 2 * O && L.ty >= 3 && L.ty < 3 + 2 * O) x[L.i] = v;
  __syncthreads();
  apply2<T>(N, xs[1], t, kReg2, L.xlo, L.xhi, L.ylo, L.yhi, y0, y1);
  v.x = bb.x - y0;
  v.y = bb.y - y1;
  xs[0][t] = v;
  __syncthreads();
  if (t < O * O) {
    const int cx = t % O, cy = t / O;
    if (X0 + cx < cg.nn[0] && Y0 + cy < cg.nn[1]) {
      const T2* r = &xs[0][(2 * cx + 3) + kReg2 * (2 * cy + 3)];
      bc[(X0 + cx) + (long long)cg.nn[0] * (Y0 + cy)] = restrict2<T>(
          g, X0 + cx, Y0 + cy, [&](int dx, int dy) { return r[dx + kReg2 * dy]; });
    }
  }
}

// Prolongation of the coarse correction e and post-smoothing: out (or the FP64
// z64) at the nodes of the tile the workgroup owns.  out must not be x.
template <class T, bool TOP>
__global__ void __launch_bounds__(kReg2 * kReg2)
    k_up2(LvK g, LvK cg, const T* __restrict__ c, const typename V2<T>::type* __restrict__ b,
          const double2* __restrict__ r64, Cheb2<T> K, const typename V2<T>::type* __restrict__ x,
          const typename V2<T>::type* __restrict__ e, typename V2<T>::type* __restrict__ out,
          double2* __restrict__ z64, double* __restrict__ part) {
  using T2 = typename V2<T>::type;
  __shared__ T2 xs[2][kReg2 * kReg2];
  constexpr int O = kUp2;
  const int ntx = (g.nn[0] + O - 1) / O;
  const int tile = (int)xcd_tile(blockIdx.x, gridDim.x);
  const Lane2 L = lane2<kReg2>(g, (tile % ntx) * O - 2, (tile / ntx) * O - 2);
  const int t = (int)threadIdx.x;
  T2 bb{}, v{};
  if (L.in) {
    bb = rhs2<T, TOP>(b, r64, L.i);
    v = prolong2<T>(x[L.i], e, cg.nn[0], L.ix, L.iy);
  }
  Node2<T> N;
  node2<T>(g, c, L.ix, L.iy, L.in, N);
  xs[0][t] = v;
  __syncthreads();
  T y0, y1;
  apply2<T>(N, xs[0], t, kReg2, L.xlo, L.xhi, L.ylo, L.yhi, y0, y1);
  const T d0 = (K.be0[0] * (bb.x - y0)) * N.rd0, d1 = (K.be0[1] * (bb.y - y1)) * N.rd1;
  v.x += d0;
  v.y += d1;
  xs[1][t] = v;
  __syncthreads();
  apply2<T>(N, xs[1], t, kReg2, L.xlo, L.xhi, L.ylo, L.yhi, y0, y1);
  v.x += K.al1[0] * d0 + (K.be1[0] * (bb.x - y0)) * N.rd0;
  v.y += K.al1[1] * d1 + (K.be1[1] * (bb.y - y1)) * N.rd1;
  const bool own = L.in && L.tx >= 2 && L.tx < 2 + O && L.ty >= 2 && L.ty < 2 + O;
  if constexpr (TOP) {
    const double2 z = own ? make_double2((double)v.x, (double)v.y) : make_double2(0.0, 0.0);
    if (own) z64[L.i] = z;
    if (part) put_partial<kReg2 * kReg2>(fma(z.x, z.x, z.y * z.y), part);
  } else if (own) {
    out[L.i] = v;
  }
}

// Steps of the coarsest Chebyshev solve, [step][block].
template <class T, int S>
struct ChebSteps {
  T al[S][2], be[S][2];
};

// S steps of the coarsest solve: the first ones, from x = 0 (FIRST), or from
// (x, d); results to (xout, dout), the last ones (LAST) to xout alone, or to z64
// in a hierarchy of one level (TOP).  The outputs must not be the inputs.
template <class T, int S, bool FIRST, bool LAST, bool TOP>
__global__ void __launch_bounds__(kCheb2Lanes)
    k_cheb2(LvK g, Regions2 R, const T* __restrict__ c, const typename V2<T>::type* __restrict__ b,
            const double2* __restrict__ r64, ChebSteps<T, S> K,
            const typename V2<T>::type* __restrict__ x, const typename V2<T>::type* __restrict__ d,
            typename V2<T>::type* __restrict__ xout, typename V2<T>::type* __restrict__ dout,
            double2* __restrict__ z64, double* __restrict__ part) {
  using T2 = typename V2<T>::type;
  __shared__ T2 xs[2][kCheb2Lanes];
  const unsigned tile = xcd_tile(blockIdx.x, gridDim.x);
  const int t = (int)threadIdx.x, ty = (int)(((unsigned)t * R.mul) >> 20), tx = t - ty * R.w;
  const Lane2 L = lane2(g, (int)(tile % R.ntx) * (R.w - 2 * R.hx) - R.hx,
                        (int)(tile / R.ntx) * (R.h - 2 * R.hy) - R.hy, tx, ty, R.w, R.h);
  T2 bb{}, v{}, dv{};
  if (L.in) {
    bb = rhs2<T, TOP>(b, r64, L.i);
    if (!FIRST) {
      v = x[L.i];
      dv = d[L.i];
    }
  }
  Node2<T> N;
  node2<T>(g, c, L.ix, L.iy, L.in, N);
  int k = 0;
  if (FIRST) {
    dv.x = (K.be[0][0] * bb.x) * N.rd0;
    dv.y = (K.be[0][1] * bb.y) * N.rd1;
    v = dv;
    k = 1;
  }
  for (; k < S; ++k) {
    // two buffers: a lane may store step k + 1's iterate while others still
    // read step k's, never the one before it
    xs[k & 1][t] = v;
    __syncthreads();
    T y0, y1;
    apply2<T>(N, xs[k & 1], t, R.w, L.xlo, L.xhi, L.ylo, L.yhi, y0, y1);
    dv.x = K.al[k][0] * dv.x + (K.be[k][0] * (bb.x - y0)) * N.rd0;
    dv.y = K.al[k][1] * dv.y + (K.be[k][1] * (bb.y - y1)) * N.rd1;
    v.x += dv.x;
    v.y += dv.y;
  }
  const bool own = L.in && L.tx >= R.hx && L.tx < R.w - R.hx && L.ty >= R.hy && L.ty < R.h - R.hy;
  if constexpr (TOP && LAST) {
    const double2 z = own ? make_double2((double)v.x, (double)v.y) : make_double2(0.0, 0.0);
    if (own) z64[L.i] = z;
    if (part) put_partial<kCheb2Lanes>(fma(z.x, z.x, z.y * z.y), part);
  } else if (own) {
    xout[L.i] = v;
    if (!LAST) dout[L.i] = dv;
  }
}

// The levels from the first of at most kTail2Lanes nodes down to the coarsest.
template <class T>
struct Tail2 {
  LvK g[kTail2Levels];
  const T* c[kTail2Levels];
  Cheb2<T> K[kTail2Levels];
  int off[kTail2Levels];  // first LDS slot of the level's right-hand side and iterate
  int levels, slots;
  ChebSteps<T, kCoarseDegree> coarse;
};

// One workgroup: the V-cycle from level 0 of the tail, lane t holding node t of
// the level at hand.  Right-hand sides and iterates of all its levels stay in
// LDS (slots <= 4/3 kTail2Lanes + a few).  Input b or r64, output x or z64 (TOP).
constexpr int kTail2Slots = kTail2Lanes + kTail2Lanes / 2;
template <class T, bool TOP>
__global__ void __launch_bounds__(kTail2Lanes)
    k_tail2(Tail2<T> A, const typename V2<T>::type* __restrict__ b, const double2* __restrict__ r64,
            typename V2<T>::type* __restrict__ x, double2* __restrict__ z64) {
  using T2 = typename V2<T>::type;
  __shared__ T2 bs[kTail2Slots], es[kTail2Slots];
  __shared__ T2 xs[2][kTail2Lanes];
  __shared__ T cs[kTail2Slots];  // cell coefficients (a level has fewer cells than nodes)
  const int t = (int)threadIdx.x;
  T2 bb{}, v{};
  Node2<T> N;
  int ix = 0, iy = 0;
  bool in = false, xlo = false, xhi = false, ylo = false, yhi = false;
  // this lane's node of level l and its weights
  auto enter = [&](int l) {
    const LvK& g = A.g[l];
    iy = t / g.nn[0];
    ix = t - iy * g.nn[0];
    in = iy < g.nn[1];
    xlo = in && ix > 0;
    xhi = in && ix < g.n[0];
    ylo = in && iy > 0;
    yhi = in && iy < g.n[1];
    node2<T>(g, &cs[A.off[l]], ix, iy, in, N);
  };
  auto apply = [&](int l, int buf, T& y0, T& y1) {
    apply2<T>(N, xs[buf], t, A.g[l].nn[0], xlo, xhi, ylo, yhi, y0, y1);
  };
  T y0, y1;
  const int last = A.levels - 1;
  if (t < A.g[0].nn[0] * A.g[0].nn[1]) bs[A.off[0] + t] = rhs2<T, TOP>(b, r64, t);
  for (int l = 0; l <= last; ++l)
    if (t < A.g[l].n[0] * A.g[l].n[1]) cs[A.off[l] + t] = A.c[l][t];
  __syncthreads();
  for (int l = 0; l < last; ++l) {
    enter(l);
    const Cheb2<T>& K = A.K[l];
    bb.x = bb.y = 0;
    if (in) bb = bs[A.off[l] + t];
    v.x = (K.be0[0] * bb.x) * N.rd0;
    v.y = (K.be0[1] * bb.y) * N.rd1;
    xs[0][t] = v;
    __syncthreads();
    apply(l, 0, y0, y1);
    v.x = v.x + (K.al1[0] * v.x + (K.be1[0] * (bb.x - y0)) * N.rd0);
    v.y = v.y + (K.al1[1] * v.y + (K.be1[1] * (bb.y - y1)) * N.rd1);
    xs[1][t] = v;
    if (in) es[A.off[l] + t] = v;
    __syncthreads();
    apply(l, 1, y0, y1);
    v.x = bb.x - y0;
    v.y = bb.y - y1;
    xs[0][t] = v;
    __syncthreads();
    const LvK& cg = A.g[l + 1];
    if (t < cg.nn[0] * cg.nn[1]) {
      const int cy = t / cg.nn[0], cx = t - cy * cg.nn[0], row = A.g[l].nn[0];
      const T2* r = &xs[0][2 * cx + row * (2 * cy)];
      bs[A.off[l + 1] + t] =
          restrict2<T>(A.g[l], cx, cy, [&](int dx, int dy) { return r[dx + row * dy]; });
    }
    __syncthreads();
  }
  // coarsest level: kCoarseDegree Chebyshev steps from zero
  enter(last);
  bb.x = bb.y = 0;
  if (in) bb = bs[A.off[last] + t];
  T2 dv;
  dv.x = (A.coarse.be[0][0] * bb.x) * N.rd0;
  dv.y = (A.coarse.be[0][1] * bb.y) * N.rd1;
  v = dv;
  auto step = [&](int k) {
    apply(last, k & 1, y0, y1);
    dv.x = A.coarse.al[k][0] * dv.x + (A.coarse.be[k][0] * (bb.x - y0)) * N.rd0;
    dv.y = A.coarse.al[k][1] * dv.y + (A.coarse.be[k][1] * (bb.y - y1)) * N.rd1;
    v.x += dv.x;
    v.y += dv.y;
  };
  if (A.g[last].nn[0] * A.g[last].nn[1] <= 64) {
    // one wavefront holds the grid: its LDS accesses complete in order, so the
    // steps need no workgroup barrier, only the compiler kept from moving them
    if (t < 64)
      for (int k = 1; k < kCoarseDegree; ++k) {
        xs[k & 1][t] = v;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        step(k);
      }
  } else {
    for (int k = 1; k < kCoarseDegree; ++k) {
      xs[k & 1][t] = v;
      __syncthreads();
      step(k);
    }
  }
  // back up: es of a level holds its iterate, then its corrected iterate
  for (int l = last - 1; l >= 0; --l) {
    if (in) es[A.off[l + 1] + t] = v;
    __syncthreads();
    const int cn0 = A.g[l + 1].nn[0];
    enter(l);
    const Cheb2<T>& K = A.K[l];
    bb.x = bb.y = v.x = v.y = 0;
    if (in) {
      bb = bs[A.off[l] + t];
      v = prolong2<T>(es[A.off[l] + t], &es[A.off[l + 1]], cn0, ix, iy);
    }
    xs[0][t] = v;
    __syncthreads();
    apply(l, 0, y0, y1);
    const T d0 = (K.be0[0] * (bb.x - y0)) * N.rd0;
    const T d1 = (K.be0[1] * (bb.y - y1)) * N.rd1;
    v.x += d0;
    v.y += d1;
    xs[1][t] = v;
    __syncthreads();
    apply(l, 1, y0, y1);
    v.x += K.al1[0] * d0 + (K.be1[0] * (bb.x - y0)) * N.rd0;
    v.y += K.al1[1] * d1 + (K.be1[1] * (bb.y - y1)) * N.rd1;
  }
  if (in) {
    if constexpr (TOP) z64[t] = make_double2((double)v.x, (double)v.y);
    else x[t] = v;
  }
}
