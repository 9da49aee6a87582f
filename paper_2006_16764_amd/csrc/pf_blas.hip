// BLAS-1 kernels of the Krylov solver: dot products and norms with
// deterministic reductions, the multi-vector products of classical
// Gram-Schmidt, and vector updates.  HBM-bound: every kernel streams its vectors
// once with 16-byte loads; on small vectors the launches and the sums inside a
// block are what counts.
//
// Reductions run in a fixed order over a fixed grid.  Vectors of at most
// kSmallPairs entry pairs: one workgroup of 1024 lanes per basis vector forms
// its final sums, one launch.  Longer ones: block partials, then k_reduce.
// Letting the block that finishes last add the partials instead of a second
// launch was measured slower (norm of 64^2 4.6 us against 2.9 + 2.4, products on
// 512^2 39 us): stores, counter and loads beyond the XCD's own L2 take about
// 1 us each, one after the other, and counter increments 25 ns each.
#include "pf_internal.h"

namespace pf {

namespace {

constexpr int kRedThreads = 256;
constexpr int kSmallThreads = 1024;
// where one workgroup's sweep costs as much as the second launch: Jacobi step of
// 64^2 (4225 pairs) 2.34 -> 2.06 ms, of 80^2 2.19 -> 2.01 ms, of 120^2 (14641)
// 1.69 -> 1.79 ms
constexpr long long kSmallPairs = 8192;
constexpr int kChunk = 16;  // most vectors per multi-dot block row

// Sums of M values (a power of two <= 64) over the wavefront's lanes by a
// butterfly: each halving of the lanes also halves the values a lane carries,
// M - 1 + log2(64/M) exchanges instead of 6 M.  Lane l ends with the sum of
// value l / (64 / M) in v[0].
template <int M, int OFF = 32>
__device__ __forceinline__ void wave_sums(double* v) {
  if constexpr (M > 1) {
    const bool up = (threadIdx.x & OFF) != 0;
#pragma unroll
    for (int i = 0; i < M / 2; ++i) {
      const double keep = up ? v[i + M / 2] : v[i], send = up ? v[i] : v[i + M / 2];
      v[i] = keep + __shfl_xor(send, OFF, 64);
    }
    wave_sums<M / 2, OFF / 2>(v);
  } else if constexpr (OFF > 0) {
    v[0] += __shfl_xor(v[0], OFF, 64);
    wave_sums<1, OFF / 2>(v);
  }
}

// Block sums of M values per lane (WAVES wavefronts, added in order): thread
// i < M returns with the sum of value i.  sh: WAVES * M doubles.
template <int M, int WAVES>
__device__ __forceinline__ double block_sums(double* v, double* sh) {
  wave_sums<M>(v);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  constexpr int per = 64 / M;
  if (lane % per == 0) sh[wid * M + lane / per] = v[0];
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x < M) {
#pragma unroll
    for (int w = 0; w < WAVES; ++w) t += sh[w * M + threadIdx.x];
  }
  return t;
}

// eps = sqrt(2^-52) (1 + sqrt(uu)) / sqrt(vv), 0 when v = 0, and its reciprocal
// (read by the product kernels instead of dividing).
__device__ __forceinline__ void write_fd_eps(double uu, double vv, double* eps) {
  const double nu = sqrt(uu), nv = sqrt(vv);
  const double e = (nv > 0.0) ? 1.4901161193847656e-08 * (1.0 + nu) / nv : 0.0;
  eps[0] = e;
  eps[1] = e == 0.0 ? 0.0 : 1.0 / e;
}

// A result for the host, which polls the slot in mapped memory while the stream
// runs on (blas_wait): a store the host sees at once, not at the kernel's end.
__device__ __forceinline__ void put_host(double* slot, double v) {
  __hip_atomic_store(slot, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// What a norm's last kernel does with |x|^2 beyond storing it: a copy for the
// host, and the FD step from it as |v|^2 with |U|^2 at uu (both may be NULL).
struct NormOut {
  double* out;
  double* out_host;
  const double* uu;
  double* eps;
  __device__ __forceinline__ void put(double t) const {
    *out = t;
    if (out_host) put_host(out_host, t);
    if (eps) write_fd_eps(*uu, t, eps);
  }
};

// |x_i|^2 of this lane's entry pairs.
template <int THREADS>
__device__ __forceinline__ double lane_norm(const double* __restrict__ x, long long n) {
  const double2* x2 = reinterpret_cast<const double2*>(x);
  double acc = 0.0;
#pragma unroll 4
  for (long long i = (long long)blockIdx.x * THREADS + threadIdx.x; i < n / 2;
       i += (long long)gridDim.x * THREADS) {
    const double2 v = x2[i];
    acc = fma(v.x, v.x, acc);
    acc = fma(v.y, v.y, acc);
  }
  return acc;
}

__global__ void __launch_bounds__(kRedThreads)
    k_norm(const double* __restrict__ x, long long n, double* __restrict__ partials) {
  __shared__ double sh[kRedThreads / 64];
  double acc = lane_norm<kRedThreads>(x, n);
  const double t = block_sums<1, kRedThreads / 64>(&acc, sh);
  if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

__global__ void __launch_bounds__(kSmallThreads)
    k_norm_small(const double* __restrict__ x, long long n, NormOut O) {
  __shared__ double sh[kSmallThreads / 64];
  double acc = lane_norm<kSmallThreads>(x, n);
  const double t = block_sums<1, kSmallThreads / 64>(&acc, sh);
  if (threadIdx.x == 0) O.put(t);
}

// z = a x + b y as k_axpby, and |z|^2 in the order of k_norm / k_norm_small.
template <int THREADS>
__device__ __forceinline__ double lane_axpby_norm(double a, const double* __restrict__ x, double b,
                                                  const double* __restrict__ y,
                                                  double* __restrict__ z, long long n) {
  const double2* x2 = reinterpret_cast<const double2*>(x);
  const double2* y2 = reinterpret_cast<const double2*>(y);
  double2* z2 = reinterpret_cast<double2*>(z);
  double acc = 0.0;
  for (long long i = (long long)blockIdx.x * THREADS + threadIdx.x; i < n / 2;
       i += (long long)gridDim.x * THREADS) {
    const double2 u = x2[i], v = y2[i];
    const double2 w = make_double2(fma(a, u.x, b * v.x), fma(a, u.y, b * v.y));
    z2[i] = w;
    acc = fma(w.x, w.x, acc);
    acc = fma(w.y, w.y, acc);
  }
  return acc;
}

__global__ void __launch_bounds__(kRedThreads)
    k_axpby_norm(double a, const double* __restrict__ x, double b, const double* __restrict__ y,
                 double* __restrict__ z, long long n, double* __restrict__ partials) {
  __shared__ double sh[kRedThreads / 64];
  double acc = lane_axpby_norm<kRedThreads>(a, x, b, y, z, n);
  const double t = block_sums<1, kRedThreads / 64>(&acc, sh);
  if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

__global__ void __launch_bounds__(kSmallThreads)
    k_axpby_norm_small(double a, const double* __restrict__ x, double b, const double* __restrict__ y,
                       double* __restrict__ z, long long n, NormOut O) {
  __shared__ double sh[kSmallThreads / 64];
  double acc = lane_axpby_norm<kSmallThreads>(a, x, b, y, z, n);
  const double t = block_sums<1, kSmallThreads / 64>(&acc, sh);
  if (threadIdx.x == 0) O.put(t);
}

// The sum of nparts partials of one row, on thread 0: fixed order per thread,
// then the block's.
__device__ __forceinline__ double row_sum(const double* __restrict__ partials, int nparts, double* sh) {
  double acc = 0.0;
#pragma unroll 4
  for (int b = threadIdx.x; b < nparts; b += kRedThreads) acc += partials[b];
  return block_sums<1, kRedThreads / 64>(&acc, sh);
}

// out[j] = sum of row j's partials; one block per row.  out_host (may be NULL):
// the same values for the host.
__global__ void __launch_bounds__(kRedThreads)
    k_reduce(const double* __restrict__ partials, int nparts, double* __restrict__ out,
             double* __restrict__ out_host) {
  __shared__ double sh[kRedThreads / 64];
  const int j = blockIdx.x;
  const double t = row_sum(partials + (long long)j * nparts, nparts, sh);
  if (threadIdx.x == 0) {
    out[j] = t;
    if (out_host) put_host(out_host + j, t);
  }
}

__global__ void __launch_bounds__(kRedThreads)
    k_reduce_norm(const double* __restrict__ partials, int nparts, NormOut O) {
  __shared__ double sh[kRedThreads / 64];
  const double t = row_sum(partials, nparts, sh);
  if (threadIdx.x == 0) O.put(t);
}

// Products of K vectors with w over this lane's entry pairs: acc[q] for
// k0 + q < k.
template <int K, int THREADS>
__device__ __forceinline__ void lane_dots(const double* __restrict__ V, long long ld, int k0, int k,
                                          const double* __restrict__ w, long long n, double* acc) {
#pragma unroll
  for (int q = 0; q < K; ++q) acc[q] = 0.0;
  const double2* w2 = reinterpret_cast<const double2*>(w);
  for (long long i = (long long)blockIdx.x * THREADS + threadIdx.x; i < n / 2;
       i += (long long)gridDim.x * THREADS) {
    const double2 wi = w2[i];
#pragma unroll
    for (int q = 0; q < K; ++q) {
      if (k0 + q < k) {
        const double2 vi = reinterpret_cast<const double2*>(V + (long long)(k0 + q) * ld)[i];
        acc[q] = fma(vi.x, wi.x, acc[q]);
        acc[q] = fma(vi.y, wi.y, acc[q]);
      }
    }
  }
}

// partials[(k0 + q) * gridDim.x + block]; blockIdx.y takes K vectors.
template <int K>
__global__ void __launch_bounds__(kRedThreads)
    k_multidot(const double* __restrict__ V, long long ld, int k, const double* __restrict__ w,
               long long n, double* __restrict__ partials) {
  __shared__ double sh[kRedThreads / 64 * K];
  const int k0 = blockIdx.y * K;
  double acc[K];
  lane_dots<K, kRedThreads>(V, ld, k0, k, w, n, acc);
  const double t = block_sums<K, kRedThreads / 64>(acc, sh);
  const int r = k0 + (int)threadIdx.x;
  if (threadIdx.x < K && r < k) partials[(long long)r * gridDim.x + blockIdx.x] = t;
}

// One workgroup per vector (blockIdx.y).
__global__ void __launch_bounds__(kSmallThreads)
    k_multidot_small(const double* __restrict__ V, long long ld, const double* __restrict__ w,
                     long long n, double* __restrict__ out, double* __restrict__ out_host) {
  __shared__ double sh[kSmallThreads / 64];
  const int r = blockIdx.y;
  double acc[1];
  lane_dots<1, kSmallThreads>(V, ld, r, r + 1, w, n, acc);
  const double t = block_sums<1, kSmallThreads / 64>(acc, sh);
  if (threadIdx.x == 0) {
    out[r] = t;
    if (out_host) put_host(out_host + r, t);
  }
}

// x[i] += sum_j coef[j] * V_j[i] (runtime k, coefficients in the kernel's
// arguments), or x[i] = that sum (assign)
struct Coefs {
  double c[kMaxGmresM];
};
__global__ void __launch_bounds__(256)
    k_combine(const double* __restrict__ V, long long ld, int k, Coefs coef, double* __restrict__ x,
              long long n, int assign) {
  const long long n2 = n / 2;
  double2* x2 = reinterpret_cast<double2*>(x);
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n2;
       i += (long long)gridDim.x * blockDim.x) {
    // assign: x = sum_j coef[j] V_j, the same sums as from an x of zeros
    double2 a = assign ? make_double2(0.0, 0.0) : x2[i];
    for (int j = 0; j < k; ++j) {
      const double c = coef.c[j];
      const double2 v = reinterpret_cast<const double2*>(V + (long long)j * ld)[i];
      a.x = fma(c, v.x, a.x);
      a.y = fma(c, v.y, a.y);
    }
    x2[i] = a;
  }
}

// Products of one Gram-Schmidt step with a delayed second projection, in one
// sweep.  t = V_j (the previous direction, projected once) and w = V_{j+1} (the
// new operator output); rows:
//   k < j: V_k . t,   j: t . t,   j + 1 + k (k < j): V_k . w,
//   2j + 1: t . w,    2j + 2: w . w.
// blockIdx.y takes V_k for k in [KMAX y, KMAX (y + 1)); chunk 0 also forms the
// three products of t and w.  The 2 KMAX + 3 sums of a block go through
// wave_sums together: one by one (with two barriers each) they cost most of the
// kernel, 34 us with 9 to 16 vectors on 512^2, 19 now.
template <int KMAX>
__global__ void __launch_bounds__(kRedThreads)
    k_dcgs_dots(const double* __restrict__ V, long long ld, int j, long long n,
                double* __restrict__ partials) {
  constexpr int kWaves = kRedThreads / 64;
  __shared__ double sh[kWaves * 2 * KMAX], sh3[kWaves * 4];
  const int nb = gridDim.x;
  const int k0 = blockIdx.y * KMAX;
  const bool first = blockIdx.y == 0;
  const long long n2 = n / 2;
  const double2* t2 = reinterpret_cast<const double2*>(V + (long long)j * ld);
  const double2* w2 = reinterpret_cast<const double2*>(V + (long long)(j + 1) * ld);
  double a[2 * KMAX];  // V . t, then V . w
  double s3[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < 2 * KMAX; ++q) a[q] = 0.0;
  for (long long i = (long long)blockIdx.x * kRedThreads + threadIdx.x; i < n2;
       i += (long long)nb * kRedThreads) {
    const double2 t = t2[i], w = w2[i];
#pragma unroll
    for (int q = 0; q < KMAX; ++q) {
      if (k0 + q < j) {
        const double2 v = reinterpret_cast<const double2*>(V + (long long)(k0 + q) * ld)[i];
        a[q] = fma(v.x, t.x, a[q]);
        a[q] = fma(v.y, t.y, a[q]);
        a[KMAX + q] = fma(v.x, w.x, a[KMAX + q]);
        a[KMAX + q] = fma(v.y, w.y, a[KMAX + q]);
      }
    }
    if (first) {
      s3[0] = fma(t.x, t.x, s3[0]);
      s3[0] = fma(t.y, t.y, s3[0]);
      s3[1] = fma(t.x, w.x, s3[1]);
      s3[1] = fma(t.y, w.y, s3[1]);
      s3[2] = fma(w.x, w.x, s3[2]);
      s3[2] = fma(w.y, w.y, s3[2]);
    }
  }
  if (j > 0) {
    const double r = block_sums<2 * KMAX, kWaves>(a, sh);
    const int q = (int)threadIdx.x % KMAX, of_w = (int)threadIdx.x / KMAX;
    if (threadIdx.x < 2 * KMAX && k0 + q < j)
      partials[(long long)(of_w * (j + 1) + k0 + q) * nb + blockIdx.x] = r;
  }
  if (first) {
    const double r = block_sums<4, kWaves>(s3, sh3);
    const int row = threadIdx.x == 0 ? j : 2 * j + (int)threadIdx.x;
    if (threadIdx.x < 3) partials[(long long)row * nb + blockIdx.x] = r;
  }
}

// The same with one workgroup per basis vector: block k < j the products of
// V_k, block j those of t and w.
__global__ void __launch_bounds__(kSmallThreads)
    k_dcgs_small(const double* __restrict__ V, long long ld, int j, long long n,
                 double* __restrict__ out, double* __restrict__ out_host) {
  __shared__ double sh[kSmallThreads / 64 * 4];
  const int k = blockIdx.x;
  const double2* t2 = reinterpret_cast<const double2*>(V + (long long)j * ld);
  const double2* w2 = reinterpret_cast<const double2*>(V + (long long)(j + 1) * ld);
  const double2* v2 = reinterpret_cast<const double2*>(V + (long long)k * ld);  // t itself for k = j
  double s[4] = {0.0, 0.0, 0.0, 0.0};  // v.t, v.w, w.w
#pragma unroll 4
  for (long long i = threadIdx.x; i < n / 2; i += kSmallThreads) {
    const double2 t = t2[i], w = w2[i], v = v2[i];
    s[0] = fma(v.x, t.x, s[0]);
    s[0] = fma(v.y, t.y, s[0]);
    s[1] = fma(v.x, w.x, s[1]);
    s[1] = fma(v.y, w.y, s[1]);
    s[2] = fma(w.x, w.x, s[2]);
    s[2] = fma(w.y, w.y, s[2]);
  }
  const double r = block_sums<4, kSmallThreads / 64>(s, sh);
  const int q = threadIdx.x;
  if (q < (k == j ? 3 : 2)) {
    const int row = q == 0 ? k : (q == 1 ? j + 1 + k : 2 * j + 2);
    out[row] = r;
    if (out_host) put_host(out_host + row, r);
  }
}

// Sums of three values over the wavefront, on every lane.
__device__ __forceinline__ void wave_all3(double& a, double& b, double& c) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    a += __shfl_xor(a, off, 64);
    b += __shfl_xor(b, off, 64);
    c += __shfl_xor(c, off, 64);
  }
}

// The two updates of that step in one sweep, in place:
//   t <- (t - sum_{k<j} s_k V_k) / rho                  (the final V_j; j > 0)
//   w <- (w - sum_{k<j} h_k V_k - h_j t_new) / eta
// with s_k = V_k . t, h_k = V_k . w (rows of the products above, still on the
// device), rho^2 = t.t - sum s_k^2, h_j = (t.w - sum s_k h_k)/rho and eta the norm
// of the projected w by Pythagoras, eta^2 = w.w - sum h_k^2 - h_j^2, or 1 when
// that keeps fewer than six digits (the caller then takes the norm itself).
// Every wavefront forms these scalars from the products (j < 64: one product
// per lane), so the sweep follows the products without the host between them;
// the host, which needs them for the Hessenberg column, gets rho, h_j, eta and
// whether eta was replaced in scal_host[0..3].
__global__ void __launch_bounds__(256)
    k_dcgs_update(double* __restrict__ V, long long ld, int j, const double* __restrict__ dots,
                  long long n, double* __restrict__ scal_host) {
  const double* cs = dots;
  const double* ch = dots + j + 1;
  const int lane = threadIdx.x & 63;
  const double sl = lane < j ? cs[lane] : 0.0, hl = lane < j ? ch[lane] : 0.0;
  double ss = sl * sl, sh = sl * hl, hh = hl * hl;
  wave_all3(ss, sh, hh);
  const double tt = dots[j], tw = dots[2 * j + 1], ww = dots[2 * j + 2];
  const double rho = j > 0 ? sqrt(fmax(tt - ss, 0.0)) : 1.0;
  const double hj = j > 0 ? (tw - sh) / rho : tw;
  const double u2 = ww - fma(hj, hj, hh);
  const bool replaced = !(u2 > 1e-12 * ww);
  const double eta = replaced ? 1.0 : sqrt(u2);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    put_host(scal_host, rho);
    put_host(scal_host + 1, hj);
    put_host(scal_host + 2, eta);
    put_host(scal_host + 3, replaced ? 1.0 : 0.0);
  }
  const double inv_rho = 1.0 / rho, inv_eta = 1.0 / eta;
  const long long n2 = n / 2;
  double2* t2 = reinterpret_cast<double2*>(V + (long long)j * ld);
  double2* w2 = reinterpret_cast<double2*>(V + (long long)(j + 1) * ld);
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n2;
       i += (long long)gridDim.x * blockDim.x) {
    double2 t = t2[i], w = w2[i];
    for (int k = 0; k < j; ++k) {
      const double2 v = reinterpret_cast<const double2*>(V + (long long)k * ld)[i];
      const double a = cs[k], b = ch[k];
      t.x = fma(-a, v.x, t.x);
      t.y = fma(-a, v.y, t.y);
      w.x = fma(-b, v.x, w.x);
      w.y = fma(-b, v.y, w.y);
    }
    t.x *= inv_rho;
    t.y *= inv_rho;
    w.x = fma(-hj, t.x, w.x) * inv_eta;
    w.y = fma(-hj, t.y, w.y) * inv_eta;
    if (j > 0) t2[i] = t;  // V_0 is final as given
    w2[i] = w;
  }
}

// y = x * alpha (invert = 0) or x / alpha (invert = 1), alpha on the device
__global__ void __launch_bounds__(256)
    k_scale(const double* __restrict__ x, const double* __restrict__ alpha, int invert,
            double* __restrict__ y, long long n) {
  const double a = invert ? 1.0 / *alpha : *alpha;
  const long long n2 = n / 2;
  const double2* x2 = reinterpret_cast<const double2*>(x);
  double2* y2 = reinterpret_cast<double2*>(y);
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n2;
       i += (long long)gridDim.x * blockDim.x) {
    const double2 v = x2[i];
    y2[i] = make_double2(a * v.x, a * v.y);
  }
}

__global__ void __launch_bounds__(256)
    k_axpby(double a, const double* __restrict__ x, double b, const double* __restrict__ y,
            double* __restrict__ z, long long n) {
  const long long n2 = n / 2;
  const double2* x2 = reinterpret_cast<const double2*>(x);
  const double2* y2 = reinterpret_cast<const double2*>(y);
  double2* z2 = reinterpret_cast<double2*>(z);
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n2;
       i += (long long)gridDim.x * blockDim.x) {
    const double2 u = x2[i], v = y2[i];
    z2[i] = make_double2(fma(a, u.x, b * v.x), fma(a, u.y, b * v.y));
  }
}

__global__ void k_sub_scalars(double* acc, const double* x, int k) {
  const int j = threadIdx.x;
  if (j < k) acc[j] -= x[j];
}

unsigned grid_for(long long n2, int threads, unsigned cap) {
  long long b = (n2 + threads - 1) / threads;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (unsigned)b;
}

inline bool small(long long n) { return n / 2 <= kSmallPairs; }

int reduce_rows(pf_problem* pb, int rows, double* out_dev, double* out_host, hipStream_t s) {
  hipLaunchKernelGGL(k_reduce, dim3(rows), dim3(kRedThreads), 0, s, pb->red_partials, pb->n_red_blocks,
                     out_dev, out_host);
  PF_HIP_CHECK(hipGetLastError());
  return PF_OK;
}

int reduce_norm(pf_problem* pb, const NormOut& O, int nparts, hipStream_t s) {
  hipLaunchKernelGGL(k_reduce_norm, dim3(1), dim3(kRedThreads), 0, s, pb->red_partials, nparts, O);
  PF_HIP_CHECK(hipGetLastError());
  return PF_OK;
}

int norm_sq(pf_problem* pb, const double* x, long long n, const NormOut& O, hipStream_t s) {
  if (small(n)) {
    hipLaunchKernelGGL(k_norm_small, dim3(1), dim3(kSmallThreads), 0, s, x, n, O);
    PF_HIP_CHECK(hipGetLastError());
    return PF_OK;
  }
  hipLaunchKernelGGL(k_norm, dim3(pb->n_red_blocks), dim3(kRedThreads), 0, s, x, n, pb->red_partials);
  PF_HIP_CHECK(hipGetLastError());
  return reduce_norm(pb, O, pb->n_red_blocks, s);
}

}  // namespace

int blas_multidot(pf_problem* pb, const double* V, long long ld, int k, const double* w,
                  long long n, double* out_dev, hipStream_t s, double* out_host) {
  if (k <= 0) return PF_OK;
  if (k == 1 && V == w) return norm_sq(pb, V, n, NormOut{out_dev, out_host, nullptr, nullptr}, s);
  if (small(n)) {
    hipLaunchKernelGGL(k_multidot_small, dim3(1, k), dim3(kSmallThreads), 0, s, V, ld, w, n, out_dev,
                       out_host);
    PF_HIP_CHECK(hipGetLastError());
    return PF_OK;
  }
  const int nb = pb->n_red_blocks;
  if (k == 1)
    hipLaunchKernelGGL(k_multidot<1>, dim3(nb), dim3(kRedThreads), 0, s, V, ld, k, w, n, pb->red_partials);
  else if (k <= 4)
    hipLaunchKernelGGL(k_multidot<4>, dim3(nb), dim3(kRedThreads), 0, s, V, ld, k, w, n, pb->red_partials);
  else
    hipLaunchKernelGGL(k_multidot<kChunk>, dim3(nb, (k + kChunk - 1) / kChunk), dim3(kRedThreads), 0, s,
                       V, ld, k, w, n, pb->red_partials);
  PF_HIP_CHECK(hipGetLastError());
  return reduce_rows(pb, k, out_dev, out_host, s);
}

int blas_axpby_norm(pf_problem* pb, double a, const double* x, double b, const double* y, double* z,
                    long long n, double* out_dev, hipStream_t s) {
  const NormOut O{out_dev, nullptr, nullptr, nullptr};
  if (small(n)) {
    hipLaunchKernelGGL(k_axpby_norm_small, dim3(1), dim3(kSmallThreads), 0, s, a, x, b, y, z, n, O);
    PF_HIP_CHECK(hipGetLastError());
    return PF_OK;
  }
  hipLaunchKernelGGL(k_axpby_norm, dim3(pb->n_red_blocks), dim3(kRedThreads), 0, s, a, x, b, y, z, n,
                     pb->red_partials);
  PF_HIP_CHECK(hipGetLastError());
  return reduce_norm(pb, O, pb->n_red_blocks, s);
}

int blas_dot(pf_problem* pb, const double* x, const double* y, long long n, double* out_dev,
             hipStream_t s) {
  return blas_multidot(pb, x, n, 1, y, n, out_dev, s);
}

int blas_dcgs_dots(pf_problem* pb, const double* V, long long ld, int j, long long n,
                   double* out_dev, hipStream_t s, double* out_host) {
  if (j < 0 || 2 * j + 3 > kRedRows) return PF_ERR_INVALID_ARG;
  if (small(n)) {
    hipLaunchKernelGGL(k_dcgs_small, dim3(j + 1), dim3(kSmallThreads), 0, s, V, ld, j, n, out_dev,
                       out_host);
    PF_HIP_CHECK(hipGetLastError());
    return PF_OK;
  }
  const int nb = pb->n_red_blocks;
  double* part = pb->red_partials;
  // the smallest accumulator set that holds the basis: fewer sums per block
  if (j <= 2)
    hipLaunchKernelGGL(k_dcgs_dots<2>, dim3(nb), dim3(kRedThreads), 0, s, V, ld, j, n, part);
  else if (j <= 4)
    hipLaunchKernelGGL(k_dcgs_dots<4>, dim3(nb), dim3(kRedThreads), 0, s, V, ld, j, n, part);
  else if (j <= 8)
    hipLaunchKernelGGL(k_dcgs_dots<8>, dim3(nb), dim3(kRedThreads), 0, s, V, ld, j, n, part);
  else
    hipLaunchKernelGGL(k_dcgs_dots<16>, dim3(nb, (j + 15) / 16), dim3(kRedThreads), 0, s, V, ld, j, n,
                       part);
  PF_HIP_CHECK(hipGetLastError());
  return reduce_rows(pb, 2 * j + 3, out_dev, out_host, s);
}

int blas_dcgs_update(double* V, long long ld, int j, const double* dots_dev, long long n,
                     double* scal_host, hipStream_t s) {
  static_assert(kMaxGmresM <= 64, "one product per lane");
  hipLaunchKernelGGL(k_dcgs_update, dim3(grid_for(n / 2, 256, 8192)), dim3(256), 0, s, V, ld, j,
                     dots_dev, n, scal_host);
  PF_HIP_CHECK(hipGetLastError());
  return PF_OK;
}

// A NaN that no kernel produces (results that are NaN carry another payload).
static constexpr uint64_t kUnset = 0x7ff4a5a5deadbeefULL;

void blas_arm(pf_problem* pb, int slot, int count) {
  auto* p = reinterpret_cast<uint64_t*>(pb->host_pinned + slot);
  for (int i = 0; i < count; ++i) __atomic_store_n(p + i, kUnset, __ATOMIC_RELEASE);
}

int blas_wait(pf_problem* pb, int slot, int count, hipStream_t s) {
  const auto* p = reinterpret_cast<const uint64_t*>(pb->host_pinned + slot);
  bool drained = false;
  for (int i = 0; i < count; ++i)
    for (unsigned spin = 1; __atomic_load_n(p + i, __ATOMIC_ACQUIRE) == kUnset; ++spin) {
      if (drained) {
        set_error("a reduction ended without its result");
        return PF_ERR_HIP;
      }
      __builtin_ia32_pause();
      if (spin % 1024) continue;
      // the stream's own state ends the wait if the result never comes
      const hipError_t e = hipStreamQuery(s);
      if (e == hipErrorNotReady) {
        (void)hipGetLastError();
        continue;
      }
      PF_HIP_CHECK(e);
      drained = true;  // one more look at the slot
    }
  return PF_OK;
}

int blas_combine(const double* V, long long ld, int k, const double* coef, double* x, long long n,
                 hipStream_t s, bool assign) {
  if (k < 0 || k > kMaxGmresM) return PF_ERR_INVALID_ARG;
  if (k == 0 && !assign) return PF_OK;
  Coefs c{};
  for (int j = 0; j < k; ++j) c.c[j] = coef[j];
  hipLaunchKernelGGL(k_combine, dim3(grid_for(n / 2, 256, 8192)), dim3(256), 0, s, V, ld, k, c, x, n,
                     assign ? 1 : 0);
  PF_HIP_CHECK(hipGetLastError());
  return PF_OK;
}

int blas_scale_copy(const double* x, const double* alpha_dev, int invert, double* y, long long n,
                    hipStream_t s) {
  hipLaunchKernelGGL(k_scale, dim3(grid_for(n / 2, 256, 8192)), dim3(256), 0, s, x, alpha_dev,
                     invert, y, n);
  PF_HIP_CHECK(hipGetLastError());
  return PF_OK;
}

int blas_axpby(double a, const double* x, double b, const double* y, double* z, long long n,
               hipStream_t s) {
  hipLaunchKernelGGL(k_axpby, dim3(grid_for(n / 2, 256, 8192)), dim3(256), 0, s, a, x, b, y, z, n);
  PF_HIP_CHECK(hipGetLastError());
  return PF_OK;
}

int blas_fd_eps(pf_problem* pb, const double* U, const double* v, long long n, double* eps_dev,
                hipStream_t s) {
  double* uu = pb->red_out + kSlotFdU;
  PF_TRY(norm_sq(pb, U, n, NormOut{uu, nullptr, nullptr, nullptr}, s));
  return blas_fd_eps_cached(pb, uu, v, n, eps_dev, s);
}

int blas_fd_eps_cached(pf_problem* pb, const double* unorm2_dev, const double* v, long long n,
                       double* eps_dev, hipStream_t s) {
  return norm_sq(pb, v, n, NormOut{pb->red_out + kSlotFdV, nullptr, unorm2_dev, eps_dev}, s);
}

int blas_fd_eps_parts(pf_problem* pb, const double* unorm2_dev, int nparts, double* eps_dev, hipStream_t s) {
  return reduce_norm(pb, NormOut{pb->red_out + kSlotFdV, nullptr, unorm2_dev, eps_dev}, nparts, s);
}

int blas_reduce_partials(const double* partials, int nparts, int k, double* out_dev, hipStream_t s) {
  hipLaunchKernelGGL(k_reduce, dim3(k), dim3(kRedThreads), 0, s, partials, nparts, out_dev, nullptr);
  PF_HIP_CHECK(hipGetLastError());
  return PF_OK;
}

int blas_sub_scalars(double* acc_dev, const double* x_dev, int k, hipStream_t s) {
  hipLaunchKernelGGL(k_sub_scalars, dim3(1), dim3(64), 0, s, acc_dev, x_dev, k);
  PF_HIP_CHECK(hipGetLastError());
  return PF_OK;
}

}  // namespace pf
