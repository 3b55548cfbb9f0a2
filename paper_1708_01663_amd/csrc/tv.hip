// Proximal map of lam * TV_iso + box (eq. R_def; step eq. algo1 with
// lam = gamma * tau) by the fast gradient projection (FGP) method of Beck and
// Teboulle (2009) applied to the dual problem.
//
// With grad the forward difference (zero last difference) and div = -grad^T:
//   x(r)    = clip(z + lam div r, lo, hi)                 primal of the dual point r
//   p_k     = P_disk(r_k + grad x(r_k) / (8 lam))          projected dual ascent, 2D
//   t_{k+1} = (1 + sqrt(1 + 4 t_k^2)) / 2
//   r_{k+1} = p_k + ((t_k - 1) / t_{k+1}) (p_k - p_{k-1})
// starting from p_0 = r_1 = 0, t_1 = 1; the output is clip(z + lam div p_K).
//
// The inner iterations run in launches of up to eight (temporal blocking): a
// block iterates on a 16 x 16 tile plus an 8-pixel halo, one thread per pixel
// with z and both duals in registers, and writes the exact tile back.  The state
// (z and four dual arrays, 20 bytes per pixel in FP32) stays resident in L2
// between launches at n <= 512.  An image of at most 32 x 32 pixels is one block
// and one launch.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>
#include <vector>

#include "internal.hpp"

namespace cisor {

constexpr int TVB = 16;              // tile side
constexpr int TVK = 8;               // halo, and iterations per launch
constexpr int TVS = TVB + 2 * TVK;   // staged side: TVS x TVS = 1024 threads
constexpr int TV_THREADS = TVS * TVS;
constexpr int TV_MAXW = 120;         // iterations of one launch on a whole image
template <typename R, int NW> struct TvWeights {
  R w[NW];
};

// The value of the previous (next) lane of the wave; lane 0 (63) receives 0.
template <int CTRL> __device__ __forceinline__ int dpp_shift(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}
template <int CTRL, typename R> __device__ __forceinline__ R lane_shift(R v) {
  if constexpr (sizeof(R) == 4) {
    return __builtin_bit_cast(R, dpp_shift<CTRL>(__builtin_bit_cast(int, v)));
  } else {
    typedef int int2v __attribute__((ext_vector_type(2)));
    int2v p = __builtin_bit_cast(int2v, v);
    p[0] = dpp_shift<CTRL>(p[0]);
    p[1] = dpp_shift<CTRL>(p[1]);
    return __builtin_bit_cast(R, p);
  }
}
constexpr int DPP_WAVE_SHL = 0x130, DPP_WAVE_SHR = 0x138;

// (a, b) projected onto the unit disk.  FP32: the reciprocal root with one
// Newton step in place of a square root and two divisions (a third of the
// iteration's instructions); either rounds each component by about an ulp.
__device__ __forceinline__ void tv_disk(double &a, double &b) {
  const double nrm = sqrt(a * a + b * b);
  if (nrm > 1.0) {
    a /= nrm;
    b /= nrm;
  }
}
__device__ __forceinline__ void tv_disk(float &a, float &b) {
  const float nn = a * a + b * b;
  if (nn > 1.0f) {
    if (nn < 1e37f) {
      const float y = __builtin_amdgcn_rsqf(nn);
      const float s = fmaf(0.5f * y, fmaf(-nn * y, y, 1.0f), y);
      a *= s;
      b *= s;
    } else {   // the squares overflow, or nearly
      const float nrm = sqrtf(nn);
      a /= nrm;
      b /= nrm;
    }
  }
}

// kb consecutive FGP iterations.  One FGP iteration reads its neighbours at
// distance one, so after m iterations the values in the staged region are exact
// at least m pixels away from its edge (or everywhere, when the region is the
// whole image, WHOLE); after kb <= TVK iterations the tile itself is exact and
// is written back.  FIRST starts from zero duals.  With x set (the last launch,
// kb < TVK) it writes the prox clip(z + lam div p) of the tile instead.
// A thread keeps its pixel's z, r and p in registers; a row of the region is
// half a wave, so horizontal neighbours come from the adjacent lane (DPP) and
// only the vertical ones (one value of r, one of x) go through LDS: four LDS
// operations and two barriers an iteration.  With every value in LDS (17
// operations an iteration) a launch of eight iterations at 256^2 took
// 10.4 us, now 6.0 us; bound by the dependent chain of an iteration (two
// barriers, the LDS reads and the projection onto the disk: a reciprocal root
// with a Newton step in FP32, a root and two divisions in FP64) over 16 waves a CU.
// Values outside the image are zero and stay zero, and r1 (r2) is zero in the
// last row (column) from the start on, so div r needs no boundary test.
template <typename R, bool WHOLE, bool FIRST, int NW>
__global__ void __launch_bounds__(TV_THREADS) k_fgp_block(const R *z, const R *rin, const R *pin, R *pout, R *rout,
                                                          R *x, int n, R lam, R lo, R hi, R inv_step,
                                                          TvWeights<R, NW> mw, int kb) {
  __shared__ R s1[TVS][TVS], sx[TVS][TVS];
  const int N = n * n;
  const int li = threadIdx.x / TVS, lj = threadIdx.x % TVS;
  const int gi = (WHOLE ? 0 : (int)blockIdx.y * TVB - TVK) + li, gj = (WHOLE ? 0 : (int)blockIdx.x * TVB - TVK) + lj;
  const bool in = gi >= 0 && gi < n && gj >= 0 && gj < n;
  const size_t g = (size_t)gi * n + gj;
  R zv = 0, r1 = 0, r2 = 0, p1 = 0, p2 = 0;
  if (in) {
    zv = z[g];
    if constexpr (!FIRST) {
      r1 = rin[g];
      r2 = rin[N + g];
      p1 = pin[g];
      p2 = pin[N + g];
    }
  }
  // forward differences that exist (the region's own edge counts as the
  // image's: what that spoils stays within the halo)
  const bool d1 = in && gi < n - 1 && li + 1 < TVS, d2 = in && gj < n - 1 && lj + 1 < TVS;
  const int up = li > 0 ? li - 1 : 0, dn = li + 1 < TVS ? li + 1 : li;
  // x = clip(z + lam div v) on every thread (zero outside the image); s1 holds
  // v1 for the row below
  auto primal = [&](R v1, R v2) -> R {
    const R left = lane_shift<DPP_WAVE_SHR>(v2);
    const R b = li > 0 ? s1[up][lj] : R(0);
    const R d = lj > 0 ? left : R(0);
    const R v = fmin(fmax(zv + lam * (v1 - b + v2 - d), lo), hi);
    return in ? v : R(0);
  };
  for (int m = 0; m < kb; ++m) {
    // rows that the tile still depends on after this iteration (the output x
    // reads p one row up) and the row on either side that they read: the
    // other waves only keep the barriers
    const int margin = kb - m + (x ? 1 : 0);
    const bool act = WHOLE || (li >= TVK - margin && li < TVK + TVB + margin);
    R x0 = 0, xr = 0;
    if (act) s1[li][lj] = r1;
    __syncthreads();
    if (act) {
      x0 = primal(r1, r2);
      sx[li][lj] = x0;
      xr = lane_shift<DPP_WAVE_SHL>(x0);
    }
    __syncthreads();
    if (act && in) {
      const R xd = sx[dn][lj];
      const R g1 = d1 ? xd - x0 : R(0);
      const R g2 = d2 ? xr - x0 : R(0);
      R a = r1 + g1 * inv_step;
      R b = r2 + g2 * inv_step;
      tv_disk(a, b);
      const R w = mw.w[m];
      r1 = a + w * (a - p1);
      r2 = b + w * (b - p2);
      p1 = a;
      p2 = b;
    }
  }
  const bool tile = WHOLE || (li >= TVK && li < TVK + TVB && lj >= TVK && lj < TVK + TVB);
  if (x) {
    s1[li][lj] = p1;
    __syncthreads();
    const R v = primal(p1, p2);
    if (in && tile) x[g] = v;
  } else if (in && tile) {
    pout[g] = p1;
    pout[N + g] = p2;
    rout[g] = r1;
    rout[N + g] = r2;
  }
}

template <typename R> __global__ void k_clip(const R *z, R *x, int N, R lo, R hi) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < N) x[i] = fmin(fmax(z[i], lo), hi);
}

// ---------------------------------------------------------------- 3D volumes
// The same FGP on an n^3 volume (voxel q = (i n + j) n + l, axes of strides
// n^2, n, 1): dual step 1 / (12 lam) (||grad||^2 <= 4 d with d = 3), the dual
// projected voxel by voxel onto the unit ball of R^3, every expression in FP64.
// One FGP iteration is one launch: a block forms x(r) on its tile and on the
// layer past each forward face in LDS, then takes the dual ascent with its
// momentum, p in place and r into the other of two buffers.  The tile is 64
// voxels long on the fastest axis, so that every access is a whole 256-byte
// row (32 on volumes of at most 32^3): 16 long it takes 6.6 us an iteration at
// 64^3, 32 long 4.8, 64 long 4.35 (8.6 for the former two launches), of which an
// empty launch is 1.5 and one that only stores p and r 2.5; the volume and its
// duals stay in L2.
template <int L> struct T3 {
  static constexpr int TL = L, TJ = 4, TI = 128 / L, THREADS = TI * TJ * TL;
  static constexpr int FACES = TJ * TL + TI * TL + TI * TJ;   // voxels past the forward faces
  static_assert(FACES <= THREADS, "a thread forms at most one of them");
};

// Element at a byte offset below 4 GiB from a uniform base (n <= 512).
template <typename R> __device__ __forceinline__ R ld32(const R *base, unsigned off) {
  return *reinterpret_cast<const R *>(reinterpret_cast<const char *>(base) + off);
}

// clip(z + lam div r) at voxel (i, j, l); ZERO: r is zero.  r_a is zero in the
// last layer of its axis (it starts there and has no gradient to follow).
// Rounding is monotone, so clipping the rounded value is rounding the clipped.
template <typename R, bool ZERO>
__device__ __forceinline__ R tv3_x(const R *z, const R *r, int i, int j, int l, int n, double lam, R lo, R hi) {
  const int N = n * n * n;
  const unsigned q = (unsigned)((i * n + j) * n + l) * (unsigned)sizeof(R);
  double d = 0.0;
  if constexpr (!ZERO) {
    const unsigned st[3] = {(unsigned)(n * n) * (unsigned)sizeof(R), (unsigned)n * (unsigned)sizeof(R),
                            (unsigned)sizeof(R)};
    const int ix[3] = {i, j, l};
    R v[3], u[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {   // loaded without a branch, used where they exist
      const R *ra = r + (size_t)a * N;
      v[a] = ld32(ra, q);
      u[a] = ld32(ra, q - (ix[a] > 0 ? st[a] : 0u));
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      d += (double)v[a];
      d -= (double)(ix[a] > 0 ? u[a] : R(0));
    }
  }
  return fmin(fmax((R)((double)ld32(z, q) + lam * d), lo), hi);
}

// 1 / max(1, sqrt(nn)).  Rounded to FP32 afterwards (R = float): the
// reciprocal root with two Newton steps (about 1e-15) for a square root and a
// division.
template <typename R> __device__ __forceinline__ double tv3_scale(double nn) {
  if constexpr (sizeof(R) == 8) {
    return 1.0 / fmax(1.0, sqrt(nn));
  } else {
    if (!(nn > 1.0)) return 1.0;
    if (!(nn < 1e300)) return 1.0 / sqrt(nn);
    double y = __builtin_amdgcn_rsq(nn);
    y = fma(0.5 * y, fma(-nn * y, y, 1.0), y);
    return fma(0.5 * y, fma(-nn * y, y, 1.0), y);
  }
}

template <typename R, bool FIRST, int L>
__global__ void __launch_bounds__(T3<L>::THREADS) k_fgp3_step(const R *z, const R *rin, R *p, R *rout, int n, double lam,
                                                          R lo, R hi, double inv_step, double w) {
  constexpr int T3I = T3<L>::TI, T3J = T3<L>::TJ, T3L = T3<L>::TL;
  __shared__ R sx[T3I + 1][T3J + 1][T3L + 1];
  const int N = n * n * n, tid = threadIdx.x;
  const int i0 = blockIdx.z * T3I, j0 = blockIdx.y * T3J, l0 = blockIdx.x * T3L;
  const int li = tid / (T3J * T3L), lj = tid / T3L % T3J, ll = tid % T3L;
  const int i = i0 + li, j = j0 + lj, l = l0 + ll;
  const bool in = i < n && j < n && l < n;
  const unsigned q = (unsigned)((i * n + j) * n + l) * (unsigned)sizeof(R);
  R rv[3] = {}, pv[3] = {};
  if (in) {
    if constexpr (!FIRST) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        rv[a] = ld32(rin + (size_t)a * N, q);
        pv[a] = ld32((const R *)p + (size_t)a * N, q);
      }
    }
    sx[li][lj][ll] = tv3_x<R, FIRST>(z, rin, i, j, l, n, lam, lo, hi);
  }
  if (tid < T3<L>::FACES) {
    int fi, fj, fl;
    if (tid < T3J * T3L) {
      fi = T3I, fj = tid / T3L, fl = tid % T3L;
    } else if (tid < T3J * T3L + T3I * T3L) {
      fi = (tid - T3J * T3L) / T3L, fj = T3J, fl = tid % T3L;
    } else {
      fi = (tid - (T3J + T3I) * T3L) / T3J, fj = tid % T3J, fl = T3L;
    }
    if (i0 + fi < n && j0 + fj < n && l0 + fl < n)
      sx[fi][fj][fl] = tv3_x<R, FIRST>(z, rin, i0 + fi, j0 + fj, l0 + fl, n, lam, lo, hi);
  }
  __syncthreads();
  if (!in) return;
  const double xc = (double)sx[li][lj][ll];
  const double g[3] = {i < n - 1 ? (double)sx[li + 1][lj][ll] - xc : 0.0,
                       j < n - 1 ? (double)sx[li][lj + 1][ll] - xc : 0.0,
                       l < n - 1 ? (double)sx[li][lj][ll + 1] - xc : 0.0};
  double v[3], nrm = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    v[a] = (double)rv[a] + g[a] * inv_step;
    nrm += v[a] * v[a];
  }
  const double sc = tv3_scale<R>(nrm);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double pn = v[a] * sc;
    char *const ro = reinterpret_cast<char *>(rout + (size_t)a * N), *const po = reinterpret_cast<char *>(p + (size_t)a * N);
    *reinterpret_cast<R *>(ro + q) = (R)(pn + w * (pn - (double)pv[a]));
    *reinterpret_cast<R *>(po + q) = (R)pn;
  }
}

// x = clip(z + lam div p); x may be z.
template <typename R>
__global__ void __launch_bounds__(256) k_fgp3_final(const R *z, const R *p, R *x, int n, double lam, R lo,
                                                    R hi) {
  const int q = blockIdx.x * 256 + threadIdx.x;
  if (q >= n * n * n) return;
  x[q] = tv3_x<R, false>(z, p, q / (n * n), q / n % n, q % n, n, lam, lo, hi);
}

// The prox on a dim-dimensional grid of side n from the work area `work` of
// 9 N reals (2D: a copy of z, made only where x overlaps it, and two ping-pong
// pairs of [2][N] duals; 3D: [3][N] p and two of r), enqueued on stream s.  Every
// launch is a kernel (no memset or copy call), so the prox can be captured in
// a graph, and the work area needs no initial contents: the first iteration's
// duals are zero without being read.
template <typename R> static bool overlap(const R *z, const R *x, int N) { return x < z + N && z < x + N; }

template <typename R>
static void tv_prox3_run(hipStream_t s, int n, R *work, const R *z, R *x, double lam, double lo, double hi,
                         int iters) {
  const int N = n * n * n;
  R *p = work, *rin = work + 3 * (size_t)N, *rout = rin + 3 * (size_t)N;
  const double inv_step = 1.0 / (12.0 * lam);
  double t = 1.0;
  auto step = [&](auto first, auto len) {
    constexpr int L = decltype(len)::value;
    using TT = T3<L>;
    const double tn = (1.0 + std::sqrt(1.0 + 4.0 * t * t)) / 2.0;
    hipLaunchKernelGGL((k_fgp3_step<R, decltype(first)::value, L>),
                       dim3((n + TT::TL - 1) / TT::TL, (n + TT::TJ - 1) / TT::TJ, (n + TT::TI - 1) / TT::TI),
                       dim3(TT::THREADS), 0, s, z, rin, p, rout, n, lam, (R)lo, (R)hi, inv_step, (t - 1.0) / tn);
    std::swap(rin, rout);
    t = tn;
  };
  const std::integral_constant<int, 32> l32{};
  const std::integral_constant<int, 64> l64{};
  for (int k = 0; k < iters; ++k) {
    if (k == 0) n <= 32 ? step(std::true_type{}, l32) : step(std::true_type{}, l64);
    else n <= 32 ? step(std::false_type{}, l32) : step(std::false_type{}, l64);
  }
  // the last kernel reads z at the voxel it writes only, so x may be z; where
  // they overlap otherwise the result goes through the work area
  const bool shifted = x != z && overlap<R>(z, x, N);
  hipLaunchKernelGGL(k_fgp3_final<R>, dim3((N + 255) / 256), dim3(256), 0, s, z, p, shifted ? rin : x, n, lam,
                     (R)lo, (R)hi);
  if (shifted) launch_copy<R>(s, x, rin, (size_t)N);
}

template <typename R>
static void tv_prox2_run(hipStream_t s, int n, R *work, const R *z, R *x, double lam, double lo, double hi,
                         int iters) {
  const int N = n * n;
  R *zc = work;
  R *pin = work + N, *pout = pin + 2 * (size_t)N, *rin = pout + 2 * (size_t)N, *rout = rin + 2 * (size_t)N;
  const R inv_step = (R)(1.0 / (8.0 * lam));
  const bool whole = n <= TVS;
  // several blocks read z around the tiles that others write in the last launch
  if (!whole && overlap<R>(z, x, N)) {
    launch_copy<R>(s, zc, z, (size_t)N);
    z = zc;
  }
  const dim3 grid(whole ? 1 : (n + TVB - 1) / TVB, whole ? 1 : (n + TVB - 1) / TVB);
  double t = 1.0;
  auto launch = [&](auto wh, auto first, auto nw, int kb, R *xo) {
    constexpr int NW = decltype(nw)::value;
    TvWeights<R, NW> mw{};
    for (int m = 0; m < kb; ++m) {
      const double tn = (1.0 + std::sqrt(1.0 + 4.0 * t * t)) / 2.0;
      mw.w[m] = (R)((t - 1.0) / tn);
      t = tn;
    }
    hipLaunchKernelGGL((k_fgp_block<R, decltype(wh)::value, decltype(first)::value, NW>), grid, dim3(TV_THREADS), 0, s,
                       z, rin, pin, pout, rout, xo, n, (R)lam, (R)lo, (R)hi, inv_step, mw, kb);
    std::swap(pin, pout);
    std::swap(rin, rout);
  };
  const std::true_type yes{};
  const std::false_type no{};
  for (int done = 0, left = iters; left > 0;) {
    // the last launch also forms the prox, which reads p one pixel further
    // out: it runs fewer than TVK iterations
    int kb;
    if (whole) {
      kb = std::min(left, TV_MAXW);
      const std::integral_constant<int, TV_MAXW> nw{};
      R *xo = kb == left ? x : nullptr;
      done ? launch(yes, no, nw, kb, xo) : launch(yes, yes, nw, kb, xo);
    } else {
      kb = left == TVK ? TVK - 1 : std::min(left, TVK);
      const std::integral_constant<int, TVK> nw{};
      R *xo = kb == left ? x : nullptr;
      done ? launch(no, no, nw, kb, xo) : launch(no, yes, nw, kb, xo);
    }
    left -= kb;
    done += kb;
  }
}

template <typename R>
static int tv_prox_run(hipStream_t s, int dim, int n, R *work, const R *z, R *x, double lam, double lo, double hi,
                       int iters) {
  const int N = dim == 3 ? n * n * n : n * n;
  if (lam <= 0.0 || iters == 0)   // no regulariser, or a zero dual: x = clip(z)
    hipLaunchKernelGGL(k_clip<R>, dim3((N + 255) / 256), dim3(256), 0, s, z, x, N, (R)lo, (R)hi);
  else if (dim == 3)
    tv_prox3_run<R>(s, n, work, z, x, lam, lo, hi, iters);
  else
    tv_prox2_run<R>(s, n, work, z, x, lam, lo, hi, iters);
  return hipGetLastError() == hipSuccess ? CISOR_OK : CISOR_E_DEVICE;
}

template <typename R>
int launch_tv_prox(Ctx &c, const R *z, R *x, double lam, double lo, double hi, int iters) {
  return tv_prox_run<R>(c.stream, c.dim, c.n, (R *)c.tvbuf, z, x, lam, lo, hi, iters);
}

// Isotropic TV of an n x n image (the regulariser of eq. R_def): the sum over
// pixels of the Euclidean norm of the forward differences, zero at the last
// index of each axis.  FP64 block partials, summed on the host in block order.
constexpr int TVV_BLOCKS = 512;
template <typename R> __global__ void __launch_bounds__(256) k_tv_value_part(const R *x, int n, double *part) {
  __shared__ double scratch[16];
  double v[1] = {0.0};
  const int N = n * n;
  for (int q = blockIdx.x * 256 + threadIdx.x; q < N; q += gridDim.x * 256) {
    const int i = q / n, j = q - i * n;
    const double c = (double)x[q];
    const double gi = (i + 1 < n) ? (double)x[q + n] - c : 0.0;
    const double gj = (j + 1 < n) ? (double)x[q + 1] - c : 0.0;
    v[0] += sqrt(gi * gi + gj * gj);
  }
  block_sum<1>(v, scratch);
  if (threadIdx.x == 0) part[blockIdx.x] = v[0];
}

// The same sum over the voxels of an n^3 volume.
template <typename R> __global__ void __launch_bounds__(256) k_tv3_value_part(const R *x, int n, double *part) {
  __shared__ double scratch[16];
  double v[1] = {0.0};
  const int N = n * n * n;
  for (int q = blockIdx.x * 256 + threadIdx.x; q < N; q += gridDim.x * 256) {
    const int st[3] = {n * n, n, 1};
    const int ix[3] = {q / (n * n), (q / n) % n, q % n};
    const double c = (double)x[q];
    double s2 = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double g = ix[a] + 1 < n ? (double)x[q + st[a]] - c : 0.0;
      s2 += g * g;
    }
    v[0] += sqrt(s2);
  }
  block_sum<1>(v, scratch);
  if (threadIdx.x == 0) part[blockIdx.x] = v[0];
}

template <typename R> int launch_tv_value(Ctx &c, const R *x, double *tv) {
  // partials in the gradient-term buffer, which holds at least N doubles
  const int nb = std::min(TVV_BLOCKS, (c.N + 255) / 256);
  double *part = (double *)c.gpart;
  if (c.dim == 3)
    hipLaunchKernelGGL(k_tv3_value_part<R>, dim3(nb), dim3(256), 0, c.stream, x, c.n, part);
  else
    hipLaunchKernelGGL(k_tv_value_part<R>, dim3(nb), dim3(256), 0, c.stream, x, c.n, part);
  std::vector<double> h(nb);
  CISOR_HIP_CHECK(hipMemcpyAsync(h.data(), part, sizeof(double) * nb, hipMemcpyDeviceToHost, c.stream));
  CISOR_HIP_CHECK(hipStreamSynchronize(c.stream));
  double s = 0.0;
  for (double v : h) s += v;
  *tv = s;
  return std::isfinite(s) ? CISOR_OK : CISOR_E_NONFINITE;
}

template int launch_tv_value<float>(Ctx &, const float *, double *);
template int launch_tv_value<double>(Ctx &, const double *, double *);
template int launch_tv_prox<float>(Ctx &, const float *, float *, double, double, double, int);
template int launch_tv_prox<double>(Ctx &, const double *, double *, double, double, double, int);

}  // namespace cisor

// ------------------------------------------------ the non-allocating prox
// cisor_tv_prox_noalloc runs the same kernels as cisor_tv_prox on a work area
// that lives in this file-scope device array instead of a context buffer, so
// it calls no allocator.  Each GPU holds its own copy of the array; its device
// address is looked up once per device (hipGetSymbolAddress with that device
// current) and kept, and only that address is ever handed to kernels (the
// array's name is a host-side stand-in in host code).
static __device__ __align__(256) unsigned char scratch[CISOR_TV_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

int scratch_of_current_device(void **out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return CISOR_E_DEVICE;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return CISOR_E_DEVICE;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return CISOR_OK;
}
}  // namespace

extern "C" int cisor_tv_prox_noalloc(int dim, int n, int precision, const void *z, void *x, double lam, double lo,
                                     double hi, int inner_iters, void *stream) {
  if ((dim != 2 && dim != 3) || n < 1 || (precision != 0 && precision != 1) || !z || !x || !(lam >= 0) ||
      !std::isfinite(lam) || !(lo <= hi) || inner_iters < 0)
    return CISOR_E_ARG;
  const long long N = dim == 3 ? (long long)n * n * n : (long long)n * n;
  if (N > CISOR_TV_NOALLOC_MAX_N) return CISOR_E_SIZE;
  void *work = nullptr;
  if (int rc = scratch_of_current_device(&work)) return rc;
  hipStream_t s = (hipStream_t)stream;
  if (precision == 0)
    return cisor::tv_prox_run<float>(s, dim, n, (float *)work, (const float *)z, (float *)x, lam, lo, hi,
                                     inner_iters);
  return cisor::tv_prox_run<double>(s, dim, n, (double *)work, (const double *)z, (double *)x, lam, lo, hi,
                                    inner_iters);
}
