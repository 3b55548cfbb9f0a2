// Receiver projection and its adjoint (the one dense contraction of the path).
//
//   projection      y_t = H diag(u_t) f           (eq. Z_def), [T][M]
//   misfit          w_t = y_t - y_meas,t, D = 1/2 sum |w|^2 (eq. D_def, FP64)
//   back-projection q_t = H^H w_t, b_t = f q_t    (right-hand side of eq. u_and_v)
//
// The projection contracts over the N pixels (K = N, large) into a small
// M x T output, so it is split over K: each block produces a partial tile,
// and a second kernel sums the partials in FP64 in a fixed order.  The FP32
// path runs on the BF16 matrix units with its operands split in three parts
// where these hold them exactly, or for few transmitters on
// v_mfma_f32_16x16x4_f32; the FP64 path on v_mfma_f64_16x16x4_f64.
#include <type_traits>

#include "internal.hpp"

namespace cisor {

constexpr int PJ_KCHUNK = PROJ_KCHUNK;  // pixels per split-K chunk

// ---------------------------------------------------------------- FP64 projection
// Complex128 contexts, and complex64 ones with more than 64 transmitters:
// every product and sum in FP64 on v_mfma_f64_16x16x4_f64 (four real products
// per complex one).  Lane l supplies A[l%16][l/16] and B[l/16][l%16] and holds
// C[4 r + l/16][l%16] in accumulator register r.  A block of eight waves owns
// MA x TB tiles of 16 receivers x 16 transmitters over one K chunk; each wave
// contracts an eighth of the chunk and the waves' sums are added in wave order
// at the end, so that a small problem still has waves on many SIMDs.  Operands go from
// global memory to registers as they are: within a group of 16 pixels lane
// group l/16 takes the four consecutive pixels 4 (l/16) .. + 4, one per
// MFMA step (the order of the sum is free), 256 contiguous bytes a row.
// Rows past M or T repeat the last one and are not stored; pixels past the
// chunk are zeros.
// Bound by the FP64 matrix rate and the fields' bytes about equally at 36 x
// 98304 x 81.  Against one thread per receiver with eight FMA sums on operands
// staged in LDS: 260 -> 123 us at 36 x 98304 x 81, and 160 -> 10.7 us at 32 x
// 1024 x 8, where that left two blocks.
typedef double doublex4 __attribute__((ext_vector_type(4)));
constexpr int PD_WAVES = 8;

template <typename R, int MA, int TB>
__global__ void __launch_bounds__(64 * PD_WAVES, 2) k_project_f64(const cplx_t<R> *H, const R *f, const cplx_t<R> *u,
                                                                  cd *part, int M, int N, int T) {
  using C = cplx_t<R>;
  __shared__ cd red[PD_WAVES][16][17];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r16 = lane & 15, g = lane >> 4;
  const int m0 = blockIdx.x * 16 * MA, t0 = blockIdx.y * 16 * TB, kc = blockIdx.z;
  const int k0 = kc * PJ_KCHUNK, kend = min(k0 + PJ_KCHUNK, N);
  const C *hp[MA], *up[TB];
#pragma unroll
  for (int i = 0; i < MA; ++i) hp[i] = H + (size_t)min(m0 + 16 * i + r16, M - 1) * N;
#pragma unroll
  for (int j = 0; j < TB; ++j) up[j] = u + (size_t)min(t0 + 16 * j + r16, T - 1) * N;
  doublex4 re[MA][TB], im[MA][TB];
#pragma unroll
  for (int i = 0; i < MA; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j) re[i][j] = im[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
  constexpr int KW = PJ_KCHUNK / PD_WAVES;   // pixels per wave
  static_assert(KW % 16 == 0, "a wave contracts whole groups of 16 pixels");
  const int kw = k0 + wave * KW, ke = min(kw + KW, kend);
  for (int kb = kw; kb < ke; kb += 16) {
    const int k = kb + 4 * g;
    C h[MA][4], x[TB][4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bool ok = k + s < ke;
      const int kk = min(k + s, N - 1);   // loaded without a branch, zeroed past the end
      const R fk = f[kk];
#pragma unroll
      for (int i = 0; i < MA; ++i) {
        const C v = hp[i][kk];
        h[i][s] = ok ? v : mk<C>(0, 0);
      }
#pragma unroll
      for (int j = 0; j < TB; ++j) {
        const C v = cscale(up[j][kk], fk);
        x[j][s] = ok ? v : mk<C>(0, 0);
      }
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
      for (int i = 0; i < MA; ++i) {
        const double hr = h[i][s].x, hi = h[i][s].y;
#pragma unroll
        for (int j = 0; j < TB; ++j) {
          const double xr = x[j][s].x, xi = x[j][s].y;
          re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(hr, xr, re[i][j], 0, 0, 0);
          im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(hr, xi, im[i][j], 0, 0, 0);
          re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-hi, xi, re[i][j], 0, 0, 0);
          im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(hi, xr, im[i][j], 0, 0, 0);
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < MA; ++i) {
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][r16][4 * r + g] = mk<cd>(re[i][j][r], im[i][j][r]);
      __syncthreads();
      if (threadIdx.x < 256) {
        const int tt = threadIdx.x >> 4, mm = threadIdx.x & 15, t = t0 + 16 * j + tt, m = m0 + 16 * i + mm;
        cd sum = red[0][tt][mm];
#pragma unroll
        for (int w = 1; w < PD_WAVES; ++w) sum = cadd(sum, red[w][tt][mm]);
        if (t < T && m < M) part[((size_t)kc * T + t) * M + m] = sum;
      }
    }
  }
}

// The tile: the widest that leaves at least 512 blocks (two per CU), else one
// 16 x 16 tile; a third receiver tile only where it fits M better.
template <typename R>
static void launch_project_f64(Ctx &c, const R *f, const cplx_t<R> *u, cd *part, int kchunks) {
  const int mt = (c.M + 15) / 16, tt = (c.T + 15) / 16;
  auto go = [&](auto ma, auto tb) {
    constexpr int MA = decltype(ma)::value, TB = decltype(tb)::value;
    hipLaunchKernelGGL((k_project_f64<R, MA, TB>), dim3((mt + MA - 1) / MA, (tt + TB - 1) / TB, kchunks),
                       dim3(64 * PD_WAVES), 0, c.stream, (const cplx_t<R> *)c.H, f, u, part, c.M, c.N, c.T);
  };
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  auto blocks = [&](int ma, int tb) { return (long long)((mt + ma - 1) / ma) * ((tt + tb - 1) / tb) * kchunks; };
  const int ma = mt % 3 == 0 || mt > 4 ? 3 : 2;
  if (blocks(ma, 2) >= 512) return ma == 3 ? go(I3{}, I2{}) : go(I2{}, I2{});
  if (blocks(2, 1) >= 512) return go(I2{}, I1{});
  go(I1{}, I1{});
}

// ---------------------------------------------------------------- FP32 on the BF16 matrix units
// Every FP32 operand is split into three BF16 parts, x = h + m + l (h and m the
// nearest BF16 of what is left, with an exact remainder), and a product takes the
// six part products h h, h m, m h, h l, m m and l h; what is dropped is below
// 2^-24 of it.  v_mfma_f32_32x32x16_bf16 has sixteen times the rate of
// v_mfma_f32_32x32x2_f32, so the 24 part products of a complex product take half
// the matrix time of the three FP32 products of Gauss's form, and avoid the
// cancellation in it.  RMS error against FP64 at 256^2 x 60 x 360 on random
// operands, relative: projection 5.7e-7 in Gauss's form, 2.0e-7 here;
// back-projection 4.9e-7 and 1.4e-7; at no size, scale or spread of magnitudes
// measured was it larger.  With all six products in one sum the projection's was
// (6.0e-7): only h h goes into the long sum.
// The parts hold an operand exactly down to 2^-110, where the last one leaves the
// subnormals of BF16 (unscaled, 2.6e-6 at 1e-35 and 2.5e-4 at 1e-37, where FP32
// products keep 6e-7).  The fields and residuals are therefore scaled by 2^23; the
// receiver matrix is looked over once, when the context is made (h_split).  Where
// it has smaller components, and in a block whose sums end non-finite (operands
// from 2^105 on, infinities), the outputs are formed from FP32 products instead
// (v_mfma_f32_32x32x2_f32, Gauss's form).
// Lane l supplies A[l%32][8(l/32)..+8] and B[8(l/32)..+8][l%32] and holds
// C[8(r/4) + 4(l/32) + r%4][l%32] in accumulator register r.
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
constexpr int BS_PARTS = 3;
// The operand that comes with a call is scaled by this, and the sums back: its
// smallest parts are then normal numbers whatever its own size.
constexpr float BF16_UP = 0x1p23f, BF16_DOWN = 0x1p-23f;
// Zero where every sum is finite, else NaN.
__device__ __forceinline__ float split_finite(const floatx16 &a, const floatx16 &b) {
  float z = 0.0f;
#pragma unroll
  for (int r = 0; r < 16; ++r) z = fmaf(a[r], 0.0f, fmaf(b[r], 0.0f, z));
  return z;
}

// The three BF16 parts of two values, packed in one dword each.
__device__ __forceinline__ void bf16_split(float a, float b, unsigned (&part)[BS_PARTS]) {
  constexpr float MAXB = 3.38953139e38f;   // largest BF16: the nearest one of a larger FP32 value is infinite
  float x[2] = {a, b};
#pragma unroll
  for (int k = 0; k < BS_PARTS; ++k) {
    floatx2 v = {x[0], x[1]};
    if (k == 0) v = floatx2{__builtin_amdgcn_fmed3f(a, -MAXB, MAXB), __builtin_amdgcn_fmed3f(b, -MAXB, MAXB)};
    part[k] = __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
    if (k + 1 < BS_PARTS) {
      x[0] -= __builtin_bit_cast(float, part[k] << 16);
      x[1] -= __builtin_bit_cast(float, part[k] & 0xffff0000u);
    }
  }
}
// Whether any thread of the block asks for it (as a uniform value).
__device__ __forceinline__ bool block_any(bool v) { return __builtin_amdgcn_readfirstlane(__syncthreads_or(v)) != 0; }
// big + small += a b over the parts: only h h goes into big, so that a long sum
// rounds once per 16 terms at its own size instead of six times.
__device__ __forceinline__ void bf16_mfma6(const bf16x8 (&a)[BS_PARTS], const bf16x8 (&b)[BS_PARTS], floatx16 &big,
                                           floatx16 &small) {
#pragma unroll
  for (int s = BS_PARTS - 1; s >= 1; --s)
#pragma unroll
    for (int i = 0; i <= s; ++i) small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[s - i], small, 0, 0, 0);
  big = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], big, 0, 0, 0);
}
__device__ __forceinline__ bf16x8 bf16_neg(bf16x8 x) {
  typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(bf16x8, __builtin_bit_cast(uintx4, x) ^ 0x80008000u);
}
// Two consecutive complex values, 8-byte aligned.
struct __attribute__((packed, aligned(8))) cf2 {
  cf v[2];
};

// Projection: a block of 4 waves covers 64 receivers x 64 transmitters (one
// 32x32 quadrant per wave) for one K chunk, 32 pixels a step.  The next step's
// H, u and f are loaded into registers while the current step runs on the
// matrix cores; they are multiplied and split on the way to LDS, where a row
// holds its six parts (re h m l, im h m l) of 32 pixels.  Rows past M or T repeat
// the last one and are not stored, pixels past the chunk are zeros.  Staging
// (splits, LDS) and the matrix cores take about 30 us each of the 89 at
// 256^2 x 60 x 360 (105 on the FP32 units): latency between barriers bounds it, so
// three blocks fit a CU; with two (95 us) the 768 blocks run one and a half
// rounds, and two LDS buffers of 16 pixels take 99.
constexpr int PJ_OFF32_N = 1 << 26;
constexpr int PJ_KS = 32, PJ_ROW = 2 * BS_PARTS * PJ_KS + 8;   // BF16 elements per LDS row

// The tile of k_project_bf16 from FP32 products, P1 = Hr Xr, P2 = Hi Xi and
// P3 = (Hr + Hi)(Xr + Xi): Re = P1 - P2, Im = P3 - P1 - P2 (Gauss).  Lane l supplies
// A[l%32][l/32] and B[l/32][l%32] of v_mfma_f32_32x32x2_f32.
typedef cf PjRow32[PJ_KS + 1];
// AHEAD: the next step's operands are loaded during the current one (the kernel
// that tries the BF16 units first has no registers for them).
template <bool AHEAD>
__device__ __forceinline__ void project_tile_f32(const cf *H, const float *f, const cf *u, cd *part, int M, int N,
                                                 int T, PjRow32 *sh, PjRow32 *su) {
  constexpr int PER = 64 * PJ_KS / 256;
  const int m0 = blockIdx.x * 64, kc = blockIdx.z;
  const int k0 = kc * PJ_KCHUNK, kend = min(k0 + PJ_KCHUNK, N);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int am = (wave & 1) * 32 + (lane & 31), bt = (wave >> 1) * 32 + (lane & 31), kl = lane >> 5;
  floatx16 p1 = {0}, p2 = {0}, p3 = {0};
  cf rh[PER], ru[PER];
  auto load = [&](int kb, int e) {
    const int i = threadIdx.x + 256 * e, row = i / PJ_KS, k = kb + i % PJ_KS;
    rh[AHEAD ? e : 0] = (m0 + row < M && k < kend) ? H[(size_t)(m0 + row) * N + k] : mk<cf>(0, 0);
    ru[AHEAD ? e : 0] = (row < T && k < kend) ? cscale(u[(size_t)row * N + k], f[k]) : mk<cf>(0, 0);
  };
  auto load_ahead = [&](int kb) {
    if constexpr (AHEAD) {
#pragma unroll
      for (int e = 0; e < PER; ++e) load(kb, e);
    }
  };
  load_ahead(k0);
  for (int kb = k0; kb < kend; kb += PJ_KS) {
#pragma unroll AHEAD ? PER : 1
    for (int e = 0; e < PER; ++e) {
      if constexpr (!AHEAD) load(kb, e);
      const int i = threadIdx.x + 256 * e;
      sh[i / PJ_KS][i % PJ_KS] = rh[AHEAD ? e : 0];
      su[i / PJ_KS][i % PJ_KS] = ru[AHEAD ? e : 0];
    }
    __syncthreads();
    if (kb + PJ_KS < kend) load_ahead(kb + PJ_KS);
#pragma unroll AHEAD ? PJ_KS / 2 : 2
    for (int kk = 0; kk < PJ_KS; kk += 2) {
      const cf a = sh[am][kk + kl], b = su[bt][kk + kl];
      p1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, p1, 0, 0, 0);
      p2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, p2, 0, 0, 0);
      p3 = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x + a.y, b.x + b.y, p3, 0, 0, 0);
    }
    __syncthreads();
  }
  if (bt >= T) return;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = m0 + (wave & 1) * 32 + 8 * (r / 4) + 4 * (lane >> 5) + (r % 4);
    const double d1 = p1[r], d2 = p2[r], d3 = p3[r];
    if (m < M) part[((size_t)kc * T + bt) * M + m] = mk<cd>(d1 - d2, d3 - d1 - d2);
  }
}

__global__ void __launch_bounds__(256) k_project_f32(const cf *H, const float *f, const cf *u, cd *part, int M, int N,
                                                     int T) {
  __shared__ PjRow32 sh[64], su[64];
  project_tile_f32<true>(H, f, u, part, M, N, T, sh, su);
}

template <typename OFF>   // holds 64 N
__global__ void __launch_bounds__(256, 3) k_project_bf16(const cf *H, const float *f, const cf *u, cd *part, int M,
                                                         int N, int T) {
  constexpr int PER = 64 * PJ_KS / 2 / 256;   // pixel pairs per thread and operand
  __shared__ __attribute__((aligned(16))) unsigned short sh[64][PJ_ROW], su[64][PJ_ROW];
  static_assert(sizeof(sh) >= 64 * sizeof(PjRow32), "the FP32 tile uses the same LDS");
  auto f32_tile = [&] {
    project_tile_f32<false>(H, f, u, part, M, N, T, reinterpret_cast<PjRow32 *>(sh), reinterpret_cast<PjRow32 *>(su));
  };
  const int m0 = blockIdx.x * 64, kc = blockIdx.z;
  const int k0 = kc * PJ_KCHUNK;
  const int kend = min(k0 + PJ_KCHUNK, N);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wm = wave & 1, wt = wave >> 1;
  floatx16 re = {0}, im = {0}, res = {0}, ims = {0};
  const int pr = threadIdx.x % (PJ_KS / 2), row = threadIdx.x / (PJ_KS / 2);
  constexpr int RS = 256 / (PJ_KS / 2);    // rows between a thread's elements
  cf2 rh[PER], ru[PER];
  float rf[2];
  // elements from the block's first row
  OFF oh[PER], ou[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    oh[e] = (OFF)(min(m0 + row + RS * e, M - 1) - m0) * (OFF)N;
    ou[e] = (OFF)min(row + RS * e, T - 1) * (OFF)N;
  }
  const cf *Hb = H + (size_t)m0 * N;
  auto load = [&](int kb) {
    const int k = kb + 2 * pr;
    if (kb + PJ_KS <= N) {   // (uniform) whole pairs
      rf[0] = f[k];
      rf[1] = f[k + 1];
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        rh[e] = *reinterpret_cast<const cf2 *>(Hb + (oh[e] + k));
        ru[e] = *reinterpret_cast<const cf2 *>(u + (ou[e] + k));
      }
    } else {
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        const int kd = min(k + d, N - 1);
        rf[d] = f[kd];
#pragma unroll
        for (int e = 0; e < PER; ++e) {
          rh[e].v[d] = Hb[oh[e] + kd];
          ru[e].v[d] = u[ou[e] + kd];
        }
      }
    }
  };
  auto put = [&](unsigned short *dst, cf a, cf b) {
    unsigned p[BS_PARTS], q[BS_PARTS];
    bf16_split(a.x, b.x, p);
    bf16_split(a.y, b.y, q);
#pragma unroll
    for (int k = 0; k < BS_PARTS; ++k) {
      *reinterpret_cast<unsigned *>(dst + k * PJ_KS + 2 * pr) = p[k];
      *reinterpret_cast<unsigned *>(dst + (BS_PARTS + k) * PJ_KS + 2 * pr) = q[k];
    }
  };
  load(k0);
  for (int kb = k0; kb < kend; kb += PJ_KS) {
    const bool ok0 = kb + 2 * pr < kend, ok1 = kb + 2 * pr + 1 < kend;
    const cf z = mk<cf>(0, 0);
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const cf x0 = cscale(ru[e].v[0], rf[0] * BF16_UP), x1 = cscale(ru[e].v[1], rf[1] * BF16_UP);
      put(sh[row + RS * e], ok0 ? rh[e].v[0] : z, ok1 ? rh[e].v[1] : z);
      put(su[row + RS * e], ok0 ? x0 : z, ok1 ? x1 : z);
    }
    __syncthreads();
    if (kb + PJ_KS < kend) load(kb + PJ_KS);
    const unsigned short *ha = sh[wm * 32 + (lane & 31)] + 8 * (lane >> 5);
    const unsigned short *xb = su[wt * 32 + (lane & 31)] + 8 * (lane >> 5);
#pragma unroll
    for (int q = 0; q < PJ_KS; q += 16) {
      bf16x8 hr[BS_PARTS], hi[BS_PARTS], x[BS_PARTS];
#pragma unroll
      for (int k = 0; k < BS_PARTS; ++k) {
        hr[k] = *reinterpret_cast<const bf16x8 *>(ha + k * PJ_KS + q);
        hi[k] = *reinterpret_cast<const bf16x8 *>(ha + (BS_PARTS + k) * PJ_KS + q);
        x[k] = *reinterpret_cast<const bf16x8 *>(xb + k * PJ_KS + q);
      }
      bf16_mfma6(hr, x, re, res);
      bf16_mfma6(hi, x, im, ims);
#pragma unroll
      for (int k = 0; k < BS_PARTS; ++k) x[k] = *reinterpret_cast<const bf16x8 *>(xb + (BS_PARTS + k) * PJ_KS + q);
      bf16_mfma6(hr, x, im, ims);
#pragma unroll
      for (int k = 0; k < BS_PARTS; ++k) x[k] = bf16_neg(x[k]);
      bf16_mfma6(hi, x, re, res);
    }
    __syncthreads();
  }
  if (block_any(split_finite(re, res) + split_finite(im, ims) != 0.0f)) return f32_tile();
  const int t = wt * 32 + (lane & 31);
  if (t >= T) return;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = m0 + wm * 32 + 8 * (r / 4) + 4 * (lane >> 5) + (r % 4);
    const cd sum = mk<cd>((double)re[r] + (double)res[r], (double)im[r] + (double)ims[r]);
    if (m < M) part[((size_t)kc * T + t) * M + m] = cscale(sum, (double)BF16_DOWN);
  }
}

// ---------------------------------------------------------------- narrow FP32 projection
// Narrow variant for at most 16 transmitters (one 16-wide transmitter tile),
// on v_mfma_f32_16x16x4f32: lane l supplies A[l%16][l/16] and B[l/16][l%16]
// and holds C[4*(l/16) + r][l%16] in accumulator register r.  Four waves own
// 16 receivers each (64 per block) against the same 16 transmitters, so no
// matrix-core work is spent on absent transmitters and H is still read once;
// reading it bounds this shape, so the products are FP32's own, three per
// complex one (Gauss): P1 = Hr Xr, P2 = Hi Xi, P3 = (Hr + Hi)(Xr + Xi); Re = P1 -
// P2, Im = P3 - P1 - P2.
typedef float floatx4 __attribute__((ext_vector_type(4)));
constexpr int PJ_NARROW_T = 16;   // transmitters of the narrow projection tiles

template <int KS>
__global__ void __launch_bounds__(256) k_project_mfma16(const cf *H, const float *f, const cf *u, cd *part, int M,
                                                        int N, int T) {
  constexpr int PH = 64 * KS / 256, PU = PJ_NARROW_T * KS / 256;
  static_assert(PH * 256 == 64 * KS && PU * 256 == PJ_NARROW_T * KS, "tile loads must cover the tiles");
  __shared__ cf sh[64][KS + 1];
  __shared__ cf su[PJ_NARROW_T][KS + 1];
  const int m0 = blockIdx.x * 64, kc = blockIdx.z;
  const int k0 = kc * PJ_KCHUNK;
  const int kend = min(k0 + PJ_KCHUNK, N);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  floatx4 acc1 = {0}, acc2 = {0}, acc3 = {0};   // Gauss's three products
  // raw loads ahead of the MFMAs: forming f u here would wait for them.  Rows past M
  // or T are skipped: a step of a small problem is bound by the loads it issues
  // (32^2 x 1 x 32 receivers 18.3 us, 19.8 with the last row repeated)
  static_assert(256 % KS == 0, "one pixel per thread and step");
  const int kk = threadIdx.x % KS, row = threadIdx.x / KS;
  constexpr int RS = 256 / KS;
  cf rh[PH] = {}, ru[PU] = {};
  float rf = 0.0f;
  auto load = [&](int kb) {
    const int k = min(kb + kk, N - 1);
    rf = f[k];
#pragma unroll
    for (int e = 0; e < PH; ++e)
      if (m0 + row + RS * e < M) rh[e] = H[(size_t)(m0 + row + RS * e) * N + k];
#pragma unroll
    for (int e = 0; e < PU; ++e)
      if (row + RS * e < T) ru[e] = u[(size_t)(row + RS * e) * N + k];
  };
  load(k0);
  for (int kb = k0; kb < kend; kb += KS) {
    const bool ok = kb + kk < kend;
#pragma unroll
    for (int e = 0; e < PH; ++e) sh[row + RS * e][kk] = ok ? rh[e] : mk<cf>(0, 0);
#pragma unroll
    for (int e = 0; e < PU; ++e) {
      const cf x = cscale(ru[e], rf);
      su[row + RS * e][kk] = ok ? x : mk<cf>(0, 0);
    }
    __syncthreads();
    if (kb + KS < kend) load(kb + KS);
    const int am = wave * 16 + (lane & 15);
    const int bt = lane & 15;
    const int kl = lane >> 4;
#pragma unroll
    for (int q = 0; q < KS; q += 4) {
      const cf a = sh[am][q + kl];
      const cf b = su[bt][q + kl];
      acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, acc1, 0, 0, 0);
      acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, acc2, 0, 0, 0);
      acc3 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x + a.y, b.x + b.y, acc3, 0, 0, 0);
    }
    __syncthreads();
  }
  const int t = lane & 15;
  if (t >= T) return;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int m = m0 + wave * 16 + 4 * (lane >> 4) + r;
    const double p1 = acc1[r], p2 = acc2[r], p3 = acc3[r];
    if (m < M) part[((size_t)kc * T + t) * M + m] = mk<cd>(p1 - p2, p3 - p1 - p2);
  }
}

// Sum the split-K partials in FP64, form y (or w = y - y_meas) and block
// partials of |w|^2.  A block owns PROJ_REDUCE_OUT outputs; its 256 threads
// are RD_LANES chunk lanes per output, lane l summing chunks l, l + RD_LANES, ...,
// and the lanes' sums are added in lane order: a fixed order, independent of
// timing, with short dependent chains even for thousands of chunks.
constexpr int RD_LANES = 256 / PROJ_REDUCE_OUT;

template <typename R>
__global__ void __launch_bounds__(256) k_project_reduce(const cd *part, int kchunks, const cplx_t<R> *y_meas,
                                                        cplx_t<R> *y, double *dpart, int MT,
                                                        const float *__restrict__ mask) {
  using C = cplx_t<R>;
  __shared__ double lr[RD_LANES][PROJ_REDUCE_OUT], li[RD_LANES][PROJ_REDUCE_OUT];
  __shared__ double scratch[16];
  const int o = threadIdx.x % PROJ_REDUCE_OUT, l = threadIdx.x / PROJ_REDUCE_OUT;
  const int i = blockIdx.x * PROJ_REDUCE_OUT + o;
  double sr = 0.0, si = 0.0;
  if (i < MT) {
    for (int k = l; k < kchunks; k += RD_LANES) {
      const cd p = part[(size_t)k * MT + i];
      sr += p.x;
      si += p.y;
    }
  }
  lr[l][o] = sr;
  li[l][o] = si;
  __syncthreads();
  double acc[1] = {0.0};
  if (l == 0 && i < MT) {
    double ar = 0.0, ai = 0.0;
#pragma unroll
    for (int j = 0; j < RD_LANES; ++j) {
      ar += lr[j][o];
      ai += li[j][o];
    }
    if (y_meas) {
      const C ym = y_meas[i];
      ar -= ym.x;
      ai -= ym.y;
      if (mask && mask[i] == 0.0f) ar = ai = 0.0;   // a switched-off receiver has no datum
    }
    y[i] = mk<C>((R)ar, (R)ai);
    acc[0] = ar * ar + ai * ai;
  }
  block_sum<1>(acc, scratch);
  if (threadIdx.x == 0) dpart[blockIdx.x] = acc[0];
}

// D = 1/2 sum of the n block partials: each of the 64 lanes sums a strided
// subset, lane 0 adds the 64 sums in lane order.
__global__ void __launch_bounds__(64) k_sum_dpart(const double *dpart, int n, double *out) {
  __shared__ double ls[64];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 64) s += dpart[i];
  ls[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x != 0) return;
  double t = 0.0;
  for (int j = 0; j < 64; ++j) t += ls[j];
  out[0] = 0.5 * t;
}

template <typename R>
int launch_project(Ctx &c, const R *f, const cplx_t<R> *u, const cplx_t<R> *y_meas, cplx_t<R> *y,
                   double *D_host, double *D_dev) {
  const int kchunks = (c.N + PJ_KCHUNK - 1) / PJ_KCHUNK;
  cd *part = (cd *)c.gemm_part;
  if constexpr (std::is_same<R, float>::value) {
    if (c.T <= PJ_NARROW_T) {
      dim3 g((c.M + 63) / 64, 1, kchunks);
      hipLaunchKernelGGL(k_project_mfma16<32>, g, dim3(256), 0, c.stream, (const cf *)c.H, f, u, part, c.M, c.N,
                         c.T);
    } else if (c.T <= 64) {
      dim3 g((c.M + 63) / 64, 1, kchunks);
      // 32-bit row offsets below 2^26 pixels: 64-bit ones cost 20 spilled registers
      // (90.4 against 89.2 us at 256^2 x 60 x 360)
      const auto kern = !c.h_split           ? k_project_f32
                        : c.N < PJ_OFF32_N ? k_project_bf16<unsigned>
                                           : k_project_bf16<size_t>;
      hipLaunchKernelGGL(kern, g, dim3(256), 0, c.stream, (const cf *)c.H, f, u, part, c.M, c.N, c.T);
    } else {
      launch_project_f64<float>(c, f, u, part, kchunks);
    }
  } else {
    launch_project_f64<double>(c, f, u, part, kchunks);
  }
  const int MT = c.M * c.T;
  const int nb = (MT + PROJ_REDUCE_OUT - 1) / PROJ_REDUCE_OUT;
  hipLaunchKernelGGL(k_project_reduce<R>, dim3(nb), dim3(256), 0, c.stream, part, kchunks, y_meas, y, c.dpart, MT,
                     (const float *)c.rx_mask);
  if (D_dev) hipLaunchKernelGGL(k_sum_dpart, dim3(1), dim3(64), 0, c.stream, c.dpart, nb, D_dev);
  if (D_host) {
    hipLaunchKernelGGL(k_sum_dpart, dim3(1), dim3(64), 0, c.stream, c.dpart, nb, c.dpart + nb);
    CISOR_HIP_CHECK(hipMemcpyAsync(D_host, c.dpart + nb, sizeof(double), hipMemcpyDeviceToHost, c.stream));
    CISOR_HIP_CHECK(hipStreamSynchronize(c.stream));
  }
  return hipGetLastError() == hipSuccess ? CISOR_OK : CISOR_E_DEVICE;
}

// ---------------------------------------------------------------- FP64 back-projection
// q[t][k] = sum_m conj(H[m][k]) w[t][m]; optional b = f q.  The lane layout is
// k_project_f64's with rows = transmitters (A[l%16][l/16] = w) and columns =
// pixels (B[l/16][l%16] = H, 256 contiguous bytes a row).  A wave owns TB
// transmitter tiles x KA pixel tiles and reads both operands from global
// memory (w is a few hundred kilobytes and stays in L2); the waves are
// independent.  Against 16 FMA sums per thread with w staged in LDS:
// 107 -> 83 us at 36 x 98304 x 81, of which writing q and b is about 50.
template <int TB, int KA>
__global__ void __launch_bounds__(256, 2) k_backproject_f64(const cd *H, const cd *w, cd *q, const double *f, cd *b,
                                                            int M, int N, int T) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r16 = lane & 15, g = lane >> 4;
  const int k0 = (blockIdx.x * 4 + wave) * 16 * KA, t0 = blockIdx.y * 16 * TB;
  if (k0 >= N) return;
  const cd *wp[TB], *hp[KA];
#pragma unroll
  for (int j = 0; j < TB; ++j) wp[j] = w + (size_t)min(t0 + 16 * j + r16, T - 1) * M;
#pragma unroll
  for (int i = 0; i < KA; ++i) hp[i] = H + min(k0 + 16 * i + r16, N - 1);
  doublex4 re[TB][KA], im[TB][KA];
#pragma unroll
  for (int j = 0; j < TB; ++j)
#pragma unroll
    for (int i = 0; i < KA; ++i) re[j][i] = im[j][i] = doublex4{0.0, 0.0, 0.0, 0.0};
  for (int mb = 0; mb < M; mb += 4) {
    const bool ok = mb + g < M;
    const int m = min(mb + g, M - 1);   // loaded without a branch, zeroed past the end
    cd a[TB], h[KA];
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      const cd v = wp[j][m];
      a[j] = ok ? v : mk<cd>(0.0, 0.0);
    }
#pragma unroll
    for (int i = 0; i < KA; ++i) {
      const cd v = hp[i][(size_t)m * N];
      h[i] = ok ? v : mk<cd>(0.0, 0.0);
    }
#pragma unroll
    for (int j = 0; j < TB; ++j) {
#pragma unroll
      for (int i = 0; i < KA; ++i) {
        re[j][i] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[j].x, h[i].x, re[j][i], 0, 0, 0);
        im[j][i] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[j].y, h[i].x, im[j][i], 0, 0, 0);
        re[j][i] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[j].y, h[i].y, re[j][i], 0, 0, 0);
        im[j][i] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[j].x, h[i].y, im[j][i], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < KA; ++i) {
    const int k = k0 + 16 * i + r16;
    if (k >= N) continue;
    const double fk = b ? f[k] : 0.0;
#pragma unroll
    for (int j = 0; j < TB; ++j) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int t = t0 + 16 * j + 4 * r + g;
        if (t >= T) continue;
        const cd val = mk<cd>(re[j][i][r], im[j][i][r]);
        q[(size_t)t * N + k] = val;
        if (b) b[(size_t)t * N + k] = cscale(val, fk);
      }
    }
  }
}

// Two pixel tiles a wave where that still gives 2048 waves (two per SIMD); three
// transmitter tiles only where they are all there are, else two: at 240^2 x 300
// receivers 104 us for a pass over H with two and 193 with three, so four take
// 181 us in two passes of two (377 with three and one of three; 336 with FMA sums).
static void launch_backproject_f64(Ctx &c, const cd *w, cd *q, const double *f, cd *b) {
  const int tt = (c.T + 15) / 16;
  auto go = [&](auto tb, auto ka) {
    constexpr int TB = decltype(tb)::value, KA = decltype(ka)::value;
    hipLaunchKernelGGL((k_backproject_f64<TB, KA>), dim3((c.N + 64 * KA - 1) / (64 * KA), (tt + TB - 1) / TB), dim3(256),
                       0, c.stream, (const cd *)c.H, w, q, f, b, c.M, c.N, c.T);
  };
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  const bool wide = (long long)(c.N / 32) * (tt == 3 ? 1 : (tt + 1) / 2) >= 2048;
  if (wide) return tt == 3 ? go(I3{}, I2{}) : tt >= 2 ? go(I2{}, I2{}) : go(I1{}, I2{});
  go(I1{}, I1{});
}

// ---------------------------------------------------------------- MFMA back-projection (FP32)
// Q[t][k] = sum_m W[t][m] conj(H[m][k]) on the BF16 matrix units in three parts
// per operand (see above): rows = transmitters, columns = pixels.
//   Re Q = sum Wr Hr + Wi Hi,  Im Q = sum Wi Hr - Wr Hi
// A block of four waves owns 64 transmitters x 128 pixels; wave w holds
// transmitter half w%2 and pixel half w/2 (two 32-pixel column blocks), so H is
// read from HBM exactly once per 64 transmitters.  W and H are split and staged
// in LDS 16 receivers at a time, W with the receivers contiguous, H as it lies
// ([receiver][pixel]): its operands, eight receivers of a pixel, come through
// the transposing LDS read.  81-85 us at 256^2 x 60 x 360 (94 on the FP32 units),
// two blocks per CU: the second LDS buffer saves a barrier a step, and the turned
// rows below seven eighths of the bank conflicts (88 us without).
constexpr int BP_MS = 16, BP_PT = 128, BP_TT = 64;
constexpr int BP_WROW = 2 * BS_PARTS * BP_MS + 16;   // BF16 elements per transmitter's LDS row
// Pixel k of receiver m lies at bp_pos(m, k): rows turned by 32 elements (16
// banks) each, so that the four rows of a transposing read miss each other's banks.
__device__ __forceinline__ int bp_pos(int m, int k) { return (k + 32 * (m & 3)) & (BP_PT - 1); }

// The tile of k_backproject_bf16 from FP32 products, P1 = Wr Hr, P2 = Wi Hi and
// P3 = (Wr + Wi)(Hr - Hi): Re = P1 + P2, Im = P3 - P1 + P2 (lane layout as in
// project_tile_f32).
typedef cf BpWRow32[BP_MS + 1];
typedef cf BpHRow32[BP_PT + 1];
template <bool AHEAD>
__device__ __forceinline__ void backproject_tile_f32(const cf *H, const cf *w, cf *q, const float *f, cf *b, int M,
                                                     int N, int T, BpWRow32 *sw, BpHRow32 *shh) {
  constexpr int PW = BP_TT * BP_MS / 256, PH = BP_MS * BP_PT / 256;
  const int k0 = blockIdx.x * BP_PT, t0 = blockIdx.y * BP_TT;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wt = wave & 1, wp = wave >> 1, kl = lane >> 5;
  floatx16 p1[2] = {{0}, {0}}, p2[2] = {{0}, {0}}, p3[2] = {{0}, {0}};
  cf rw[PW], rh[PH];
  auto load_w = [&](int m0, int e) {
    const int i = threadIdx.x + 256 * e, t = t0 + i / BP_MS, m = m0 + i % BP_MS;
    rw[AHEAD ? e : 0] = (t < T && m < M) ? w[(size_t)t * M + m] : mk<cf>(0, 0);
  };
  auto load_h = [&](int m0, int e) {
    const int i = threadIdx.x + 256 * e, m = m0 + i / BP_PT, k = k0 + i % BP_PT;
    rh[AHEAD ? e : 0] = (m < M && k < N) ? H[(size_t)m * N + k] : mk<cf>(0, 0);
  };
  auto load_ahead = [&](int m0) {
    if constexpr (AHEAD) {
#pragma unroll
      for (int e = 0; e < PW; ++e) load_w(m0, e);
#pragma unroll
      for (int e = 0; e < PH; ++e) load_h(m0, e);
    }
  };
  load_ahead(0);
  for (int m0 = 0; m0 < M; m0 += BP_MS) {
#pragma unroll AHEAD ? PW : 1
    for (int e = 0; e < PW; ++e) {
      if constexpr (!AHEAD) load_w(m0, e);
      const int i = threadIdx.x + 256 * e;
      sw[i / BP_MS][i % BP_MS] = rw[AHEAD ? e : 0];
    }
#pragma unroll AHEAD ? PH : 1
    for (int e = 0; e < PH; ++e) {
      if constexpr (!AHEAD) load_h(m0, e);
      const int i = threadIdx.x + 256 * e;
      shh[i / BP_PT][i % BP_PT] = rh[AHEAD ? e : 0];
    }
    __syncthreads();
    if (m0 + BP_MS < M) load_ahead(m0 + BP_MS);
#pragma unroll AHEAD ? BP_MS / 2 : 1
    for (int mm = 0; mm < BP_MS; mm += 2) {
      const cf a = sw[wt * 32 + (lane & 31)][mm + kl];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const cf h = shh[mm + kl][wp * 64 + j * 32 + (lane & 31)];
        p1[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, h.x, p1[j], 0, 0, 0);
        p2[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, h.y, p2[j], 0, 0, 0);
        p3[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x + a.y, h.x - h.y, p3[j], 0, 0, 0);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int k = k0 + wp * 64 + j * 32 + (lane & 31);
    if (k >= N) continue;
    const float fk = b ? f[k] : 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int t = t0 + wt * 32 + 8 * (r / 4) + 4 * (lane >> 5) + (r % 4);
      if (t >= T) continue;
      const double d1 = p1[j][r], d2 = p2[j][r], d3 = p3[j][r];
      const cf val = mk<cf>((float)(d1 + d2), (float)(d3 - d1 + d2));
      q[(size_t)t * N + k] = val;
      if (b) b[(size_t)t * N + k] = mk<cf>(val.x * fk, val.y * fk);
    }
  }
}

__global__ void __launch_bounds__(256) k_backproject_f32(const cf *H, const cf *w, cf *q, const float *f, cf *b, int M,
                                                         int N, int T) {
  __shared__ BpWRow32 sw[BP_TT];
  __shared__ BpHRow32 shh[BP_MS];
  backproject_tile_f32<true>(H, w, q, f, b, M, N, T, sw, shh);
}

__global__ void __launch_bounds__(256, 2) k_backproject_bf16(const cf *H, const cf *w, cf *q, const float *f, cf *b,
                                                          int M, int N, int T) {
  constexpr int PW = BP_TT * BP_MS / 2 / 256, PH = BP_MS * BP_PT / 2 / 256;   // pairs per thread
  __shared__ __attribute__((aligned(16))) unsigned short sw2[2][BP_TT][BP_WROW];
  __shared__ __attribute__((aligned(16))) unsigned short sh2[2][2 * BS_PARTS][BP_MS][BP_PT];
  static_assert(sizeof(sw2) >= BP_TT * sizeof(BpWRow32) && sizeof(sh2) >= BP_MS * sizeof(BpHRow32),
                "the FP32 tile uses the same LDS");
  auto f32_tile = [&] {
    backproject_tile_f32<false>(H, w, q, f, b, M, N, T, reinterpret_cast<BpWRow32 *>(sw2),
                                reinterpret_cast<BpHRow32 *>(sh2));
  };
  const int k0 = blockIdx.x * BP_PT, t0 = blockIdx.y * BP_TT;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wt = wave & 1, wp = wave >> 1;
  floatx16 re[2] = {{0}, {0}}, im[2] = {{0}, {0}}, res[2] = {{0}, {0}}, ims[2] = {{0}, {0}};
  // next step's W and H staged in registers during the current step's MFMAs;
  // rows past T and receivers past M repeat the last one (the latter zeroed on
  // the way to LDS), pixels past N are not stored
  const int wr = threadIdx.x / (BP_MS / 2), wpair = threadIdx.x % (BP_MS / 2);
  const int hr = threadIdx.x / (BP_PT / 2), hpair = threadIdx.x % (BP_PT / 2);
  cf rw[PW][2];
  cf2 rh[PH];
  auto load = [&](int m0) {
#pragma unroll
    for (int e = 0; e < PW; ++e) {
      const size_t base = (size_t)min(t0 + wr + e * (512 / BP_MS), T - 1) * M;
#pragma unroll
      for (int d = 0; d < 2; ++d) rw[e][d] = w[base + min(m0 + 2 * wpair + d, M - 1)];
    }
#pragma unroll
    for (int e = 0; e < PH; ++e) {
      const cf *row = H + (size_t)min(m0 + hr + e * (512 / BP_PT), M - 1) * N;
      const int k = k0 + 2 * hpair;
      if (k0 + BP_PT <= N) {   // (uniform)
        rh[e] = *reinterpret_cast<const cf2 *>(row + k);
      } else {
        rh[e].v[0] = row[min(k, N - 1)];
        rh[e].v[1] = row[min(k + 1, N - 1)];
      }
    }
  };
  auto store = [&](int m0, int buf) {
    auto &sw = sw2[buf];
    auto &sh = sh2[buf];
    const cf z = mk<cf>(0, 0);
    unsigned p[BS_PARTS], r[BS_PARTS];
#pragma unroll
    for (int e = 0; e < PW; ++e) {
      const int m = m0 + 2 * wpair;
      const cf a0 = m < M ? cscale(rw[e][0], BF16_UP) : z, a1 = m + 1 < M ? cscale(rw[e][1], BF16_UP) : z;
      bf16_split(a0.x, a1.x, p);
      bf16_split(a0.y, a1.y, r);
      unsigned short *dst = sw[wr + e * (512 / BP_MS)] + 2 * wpair;
#pragma unroll
      for (int k = 0; k < BS_PARTS; ++k) {
        *reinterpret_cast<unsigned *>(dst + k * BP_MS) = p[k];
        *reinterpret_cast<unsigned *>(dst + (BS_PARTS + k) * BP_MS) = r[k];
      }
    }
#pragma unroll
    for (int e = 0; e < PH; ++e) {
      const int mm = hr + e * (512 / BP_PT);
      const bool ok = m0 + mm < M;
      const cf h0 = ok ? rh[e].v[0] : z, h1 = ok ? rh[e].v[1] : z;
      bf16_split(h0.x, h1.x, p);
      bf16_split(h0.y, h1.y, r);
#pragma unroll
      for (int k = 0; k < BS_PARTS; ++k) {
        *reinterpret_cast<unsigned *>(&sh[k][mm][bp_pos(mm, 2 * hpair)]) = p[k];
        *reinterpret_cast<unsigned *>(&sh[BS_PARTS + k][mm][bp_pos(mm, 2 * hpair)]) = r[k];
      }
    }
  };
  load(0);
  store(0, 0);
  if (BP_MS < M) load(BP_MS);
  __syncthreads();
  for (int m0 = 0, buf = 0; m0 < M; m0 += BP_MS, buf ^= 1) {
    auto &sw = sw2[buf];
    auto &sh = sh2[buf];
    const unsigned short *wa = sw[wt * 32 + (lane & 31)] + 8 * (lane >> 5);
    bf16x8 ar[BS_PARTS], ai[BS_PARTS], an[BS_PARTS];   // Wr, Wi, -Wr
#pragma unroll
    for (int k = 0; k < BS_PARTS; ++k) {
      ar[k] = *reinterpret_cast<const bf16x8 *>(wa + k * BP_MS);
      ai[k] = *reinterpret_cast<const bf16x8 *>(wa + (BS_PARTS + k) * BP_MS);
      an[k] = bf16_neg(ar[k]);
    }
    // lane l of the transposing read: four receivers of pixel l % 16 of its 16-lane group
    const int trow = 8 * (lane >> 5) + ((lane & 15) >> 2), tcol = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      bf16x8 br[BS_PARTS], bi[BS_PARTS];
#pragma unroll
      for (int k = 0; k < 2 * BS_PARTS; ++k) {
        typedef __attribute__((address_space(3))) shortx4 *lds4;
        unsigned short *src = &sh[k][trow][bp_pos(trow, wp * 64 + j * 32 + tcol)];
        const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)src);
        const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(src + 4 * BP_PT));
        const bf16x8 v = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        if (k < BS_PARTS) br[k] = v;
        else bi[k - BS_PARTS] = v;
      }
      bf16_mfma6(ar, br, re[j], res[j]);
      bf16_mfma6(ai, bi, re[j], res[j]);
      bf16_mfma6(ai, br, im[j], ims[j]);
      bf16_mfma6(an, bi, im[j], ims[j]);
    }
    // the other buffer was last read before the barrier that ended the previous step
    if (m0 + BP_MS < M) {
      store(m0 + BP_MS, buf ^ 1);
      if (m0 + 2 * BP_MS < M) load(m0 + 2 * BP_MS);
      __syncthreads();
    }
  }
  const float fin = split_finite(re[0], res[0]) + split_finite(re[1], res[1]) + split_finite(im[0], ims[0]) +
                    split_finite(im[1], ims[1]);
  if (block_any(fin != 0.0f)) return f32_tile();
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int k = k0 + wp * 64 + j * 32 + (lane & 31);
    if (k >= N) continue;
    const float fk = b ? f[k] : 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int t = t0 + wt * 32 + 8 * (r / 4) + 4 * (lane >> 5) + (r % 4);
      if (t >= T) continue;
      const cf val = cscale(mk<cf>(re[j][r] + res[j][r], im[j][r] + ims[j][r]), BF16_DOWN);
      q[(size_t)t * N + k] = val;
      if (b) b[(size_t)t * N + k] = mk<cf>(val.x * fk, val.y * fk);
    }
  }
}

// Narrow variant for at most 16 transmitters on v_mfma_f32_16x16x4f32 (lane
// layout as in k_project_mfma16): rows = the 16 transmitters (A operand
// W[l%16][m + l/16]), columns = pixels (B operand H[m + l/16][l%16]).  Each of
// the four waves owns 16 pixels (64 per block), so every pixel column of H is
// read once and no matrix-core work is spent on absent transmitters.
constexpr int BP16_PT = 64;

__global__ void __launch_bounds__(256) k_backproject_mfma16(const cf *H, const cf *w, cf *q, const float *f, cf *b,
                                                            int M, int N, int T) {
  constexpr int PH = BP_MS * BP16_PT / 256;
  static_assert(PH * 256 == BP_MS * BP16_PT && PJ_NARROW_T * BP_MS == 256, "tile loads must cover the tiles");
  __shared__ cf sw[PJ_NARROW_T][BP_MS + 1];
  __shared__ cf shh[BP_MS][BP16_PT + 1];
  const int k0 = blockIdx.x * BP16_PT;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // Gauss's three products: P1 = Wr Hr, P2 = Wi Hi, P3 = (Wr + Wi)(Hr - Hi);
  // Re = P1 + P2, Im = P3 - P1 + P2
  floatx4 acc1 = {0}, acc2 = {0}, acc3 = {0};
  cf rw, rh[PH];
  auto load = [&](int m0) {
    {
      const int tt = threadIdx.x / BP_MS, mm = threadIdx.x % BP_MS;
      const int m = m0 + mm;
      rw = (tt < T && m < M) ? w[(size_t)tt * M + m] : mk<cf>(0, 0);
    }
#pragma unroll
    for (int e = 0; e < PH; ++e) {
      const int i = threadIdx.x + 256 * e;
      const int mm = i / BP16_PT, kk = i % BP16_PT;
      const int m = m0 + mm, k = k0 + kk;
      rh[e] = (m < M && k < N) ? H[(size_t)m * N + k] : mk<cf>(0, 0);
    }
  };
  load(0);
  for (int m0 = 0; m0 < M; m0 += BP_MS) {
    sw[threadIdx.x / BP_MS][threadIdx.x % BP_MS] = rw;
#pragma unroll
    for (int e = 0; e < PH; ++e) {
      const int i = threadIdx.x + 256 * e;
      shh[i / BP16_PT][i % BP16_PT] = rh[e];
    }
    __syncthreads();
    if (m0 + BP_MS < M) load(m0 + BP_MS);
    const int ar = lane & 15;
    const int kl = lane >> 4;
#pragma unroll
    for (int mm = 0; mm < BP_MS; mm += 4) {
      const cf a = sw[ar][mm + kl];
      const cf h = shh[mm + kl][wave * 16 + (lane & 15)];
      acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, h.x, acc1, 0, 0, 0);
      acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, h.y, acc2, 0, 0, 0);
      acc3 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x + a.y, h.x - h.y, acc3, 0, 0, 0);
    }
    __syncthreads();
  }
  const int k = k0 + wave * 16 + (lane & 15);
  if (k >= N) return;
  const float fk = b ? f[k] : 0.0f;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int t = 4 * (lane >> 4) + r;
    if (t >= T) continue;
    const double p1 = acc1[r], p2 = acc2[r], p3 = acc3[r];
    const cf val = mk<cf>((float)(p1 + p2), (float)(p3 - p1 + p2));
    q[(size_t)t * N + k] = val;
    if (b) b[(size_t)t * N + k] = mk<cf>(val.x * fk, val.y * fk);
  }
}

template <typename R>
int launch_backproject(Ctx &c, const cplx_t<R> *w, cplx_t<R> *q, const R *f, cplx_t<R> *b) {
  if constexpr (std::is_same<R, float>::value) {
    if (c.T <= PJ_NARROW_T) {
      dim3 g((c.N + BP16_PT - 1) / BP16_PT);
      hipLaunchKernelGGL(k_backproject_mfma16, g, dim3(256), 0, c.stream, (const cf *)c.H, w, q, f, b, c.M, c.N,
                         c.T);
      return hipGetLastError() == hipSuccess ? CISOR_OK : CISOR_E_DEVICE;
    }
    dim3 g((c.N + BP_PT - 1) / BP_PT, (c.T + BP_TT - 1) / BP_TT);
    hipLaunchKernelGGL(c.h_split ? k_backproject_bf16 : k_backproject_f32, g, dim3(256), 0, c.stream, (const cf *)c.H,
                       w, q, f, b, c.M, c.N, c.T);
  } else {
    launch_backproject_f64(c, w, q, f, b);
  }
  return hipGetLastError() == hipSuccess ? CISOR_OK : CISOR_E_DEVICE;
}

template int launch_project<float>(Ctx &, const float *, const cf *, const cf *, cf *, double *, double *);
template int launch_project<double>(Ctx &, const double *, const cd *, const cd *, cd *, double *, double *);
template int launch_backproject<float>(Ctx &, const cf *, cf *, const float *, cf *);
template int launch_backproject<double>(Ctx &, const cd *, cd *, const double *, cd *);

}  // namespace cisor
