// Learned warm start for the Lippmann-Schwinger solves: a 4-level convolutional
// encoder-decoder that maps (f, u_in, first-Born scattered field) on the grid to the scattered
// field u - u_in (2 channels), trained on fields produced by the solver itself.
//
// Everything runs in BF16 on the matrix cores with FP32 accumulation:
//   * 3x3 convolution (stride 1, zero padding 1) as an implicit GEMM
//     [pixels x 9 Cin] x [9 Cin x Cout] on v_mfma_f32_32x32x16_bf16, NHWC
//     activations, weights stored [3][3][Cout][Cin]; bias and ReLU fused.
//   * The data gradient of a convolution is the same convolution applied to
//     the output gradient with the weights flipped in space and transposed in
//     channels, so it reuses the forward kernel.
//   * The weight gradient is a GEMM [Cout x pixels] x [pixels x Cin] per tap,
//     split over pixels, with partial tiles summed in a fixed order.
//   * 2x2 average pooling, nearest x2 upsampling, channel concatenation, the
//     relative-L2 loss and Adam (FP32 master weights) are elementwise kernels.
// Layout of a lane's MFMA operands (32x32x16): lane l supplies A[l%32][8(l/32)..+8]
// and B[8(l/32)..+8][l%32]; accumulator register r holds
// C[8(r/4) + 4(l/32) + r%4][l%32].
#include <cmath>
#include <cstring>
#include <new>
#include <random>
#include <vector>

#include "internal.hpp"

namespace cisor {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t bf16_t;

__host__ __device__ __forceinline__ bf16_t f2bf(float f) {
  uint32_t u = __builtin_bit_cast(uint32_t, f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (bf16_t)((u >> 16) | ((u & 0xffff) ? 0x40 : 0));  // inf/nan
  u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest even
  return (bf16_t)(u >> 16);
}
__host__ __device__ __forceinline__ float bf2f(bf16_t h) { return __builtin_bit_cast(float, (uint32_t)h << 16); }

// Orders a wave's own LDS stores and reads (its DS operations complete in
// order; only the compiler must keep them).
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------------------ conv forward
constexpr int CV_BK = 32, CV_PAD = 8;

// y[p][co] = act(bias[co] + sum_{tap, ci} x[shift(p, tap)][ci] w[tap][co][ci])
// x: [B][H][W][Ci] bf16, w: [9][Co][Ci] bf16, y: [B][H][W][Co] bf16 or f32.
// Implicit GEMM [pixels x 9 Ci] x [9 Ci x Co]: a block of four waves owns a
// tile of BM = 128 MI pixels x BN = 32 NI output channels; wave w holds the
// 32 MI x 32 NI sub-tile of pixel rows [32 MI w, 32 MI (w + 1)) in MI x NI
// accumulators of v_mfma_f32_32x32x16_bf16, so every A fragment read from LDS
// feeds NI instructions and every B fragment MI.  Lane l supplies A[l%32][8(l/32)..+8]
// and B[l%32][8(l/32)..+8] (K contiguous) and holds C[8(r/4) + 4(l/32) + r%4][l%32].
// Requires Ci % 32 == 0, Co % BN == 0, (B*H*W) % BM == 0.
template <bool RELU, bool OUT_F32, int MI, int NI>
__global__ void __launch_bounds__(256) k_conv3x3(const bf16_t *__restrict__ x, const bf16_t *__restrict__ w,
                                                 const float *__restrict__ bias, void *__restrict__ y, int H, int W,
                                                 int Ci, int Co, const bf16_t *__restrict__ x2, int C1,
                                                 int s_steps, float *__restrict__ part) {
  constexpr int BM = 128 * MI, BN = 32 * NI;
  constexpr int AL = BM * 4 / 256;                 // 16-byte A pieces per thread per step
  constexpr int BL = (BN * 4 + 255) / 256;         // 16-byte B pieces per thread per step
  __shared__ __attribute__((aligned(16))) bf16_t As[BM][CV_BK + CV_PAD];
  __shared__ __attribute__((aligned(16))) bf16_t Bs[BN][CV_BK + CV_PAD];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int m0 = blockIdx.x * BM, co0 = blockIdx.y * BN;
  const int HW = H * W;
  f32x16 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = f32x16{0};
  // the pixel rows this thread stages: BM rows x 4 segments of 8 channels
  int pb[AL], py[AL], pxx[AL];
#pragma unroll
  for (int i = 0; i < AL; ++i) {
    const int P = m0 + ((tid + 256 * i) >> 2);
    pb[i] = P / HW;
    const int rem = P - pb[i] * HW;
    py[i] = rem / W;
    pxx[i] = rem - py[i] * W;
  }
  // Steps run over (tap, 32-channel slice); the global loads of step it + 1
  // are issued into registers before the MFMAs of step it, so their latency
  // overlaps with the matrix work.  With x2 set, the input is the channel
  // concatenation of x (C1 channels) and the nearest-neighbour 2x upsampling
  // of x2 (Ci - C1 channels at H/2 x W/2), read in place: a 32-channel slice
  // lies in one of the two (C1 is a multiple of 32).
  const int csteps = Ci / CV_BK, nsteps = 9 * csteps;
  const int Cx = x2 ? C1 : Ci, H2 = H >> 1, W2 = W >> 1;
  u32x4 ra[AL], rb[BL];
  auto load = [&](int it) {
    const int tap = it / csteps, ci0 = (it - tap * csteps) * CV_BK;
    const int dy = tap / 3 - 1, dx = tap % 3 - 1;
    const bool up = x2 && ci0 >= C1;
#pragma unroll
    for (int i = 0; i < AL; ++i) {
      const int part = (tid + 256 * i) & 3;
      const int yy = py[i] + dy, xx = pxx[i] + dx;
      ra[i] = u32x4{0, 0, 0, 0};
      if (yy >= 0 && yy < H && xx >= 0 && xx < W) {
        const bf16_t *src = up ? x2 + ((size_t)(pb[i] * H2 + (yy >> 1)) * W2 + (xx >> 1)) * (Ci - C1) + (ci0 - C1)
                               : x + ((size_t)(pb[i] * H + yy) * W + xx) * Cx + ci0;
        ra[i] = *reinterpret_cast<const u32x4 *>(src + part * 8);
      }
    }
#pragma unroll
    for (int i = 0; i < BL; ++i) {
      const int c = tid + 256 * i;
      if (c < BN * 4) {
        const int co = c >> 2, part = c & 3;
        rb[i] = *reinterpret_cast<const u32x4 *>(w + ((size_t)tap * Co + co0 + co) * Ci + ci0 + part * 8);
      }
    }
  };
  // split K: block z runs steps [z s_steps, (z + 1) s_steps) and, with part
  // set, writes its FP32 partial sums (no bias, no activation) to part[z]
  const int it0 = blockIdx.z * s_steps, it1 = min(nsteps, it0 + s_steps);
  load(it0);
  for (int it = it0; it < it1; ++it) {
#pragma unroll
    for (int i = 0; i < AL; ++i) {
      const int c = tid + 256 * i;
      *reinterpret_cast<u32x4 *>(&As[c >> 2][(c & 3) * 8]) = ra[i];
    }
#pragma unroll
    for (int i = 0; i < BL; ++i) {
      const int c = tid + 256 * i;
      if (c < BN * 4) *reinterpret_cast<u32x4 *>(&Bs[c >> 2][(c & 3) * 8]) = rb[i];
    }
    __syncthreads();
    if (it + 1 < it1) load(it + 1);
#pragma unroll
    for (int kk = 0; kk < CV_BK; kk += 16) {
      bf16x8 a[MI], bv[NI];
#pragma unroll
      for (int i = 0; i < MI; ++i)
        a[i] = *reinterpret_cast<const bf16x8 *>(&As[(wave * MI + i) * 32 + (lane & 31)][kk + 8 * (lane >> 5)]);
#pragma unroll
      for (int j = 0; j < NI; ++j)
        bv[j] = *reinterpret_cast<const bf16x8 *>(&Bs[j * 32 + (lane & 31)][kk + 8 * (lane >> 5)]);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], bv[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
  if (part) {
    float *dst = part + (size_t)blockIdx.z * gridDim.x * BM * Co;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int co = co0 + j * 32 + (lane & 31);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int P = m0 + (wave * MI + i) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          dst[(size_t)P * Co + co] = acc[i][j][r];
        }
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    const int co = co0 + j * 32 + (lane & 31);
    const float bb = bias ? bias[co] : 0.0f;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int P = m0 + (wave * MI + i) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        float v = acc[i][j][r] + bb;
        if (RELU) v = fmaxf(v, 0.0f);
        if (OUT_F32)
          reinterpret_cast<float *>(y)[(size_t)P * Co + co] = v;
        else
          reinterpret_cast<bf16_t *>(y)[(size_t)P * Co + co] = f2bf(v);
      }
    }
  }
}

// Input and output forms of the tiled convolution (inference path):
//   TIN_X     x (or [x | up2(x2)] with x2 set), NHWC at the layer's resolution
//   TIN_POOL  the 2x2 average of x given at twice the layer's resolution,
//             summed and rounded as k_avgpool does
//   TIN_NET   the network input formed from (f, u_in, u_B) as k_net_input does
//             (Ci = 32)
//   TOUT_BF16 / TOUT_F32  y in NHWC
//   TOUT_U0   u0 = u_in + (y0 + i y1) written as complex values, as
//             k_net_output does (channels 0 and 1 of the first channel block)
enum { TIN_X = 0, TIN_POOL = 1, TIN_NET = 2 };
//   TOUT_MASK  y in NHWC, zero where io.mask is not positive (the data gradient
//   through the ReLU of the layer below)
enum { TOUT_BF16 = 0, TOUT_F32 = 1, TOUT_U0 = 2, TOUT_MASK = 3 };
struct TileIO {
  const float *f = nullptr;   // TIN_NET: [B, H W]
  const cf *uin = nullptr;    // TIN_NET, TOUT_U0: [B, H W]
  const cf *ub = nullptr;     // TIN_NET: [B, H W] or null (zeros)
  cf *u0 = nullptr;           // TOUT_U0: [B, H W]
  const bf16_t *mask = nullptr;   // TOUT_MASK: the layer's input activation, laid out as y
};

// Registers of one halo piece before it is formed: the piece itself, the four
// pieces that pool into it, or the five network-input values.
template <int TIN> struct HaloRaw {
  struct type {
    u32x4 v[1] = {};
  };
};
template <> struct HaloRaw<TIN_POOL> {
  struct type {
    u32x4 v[4] = {};
  };
};
template <> struct HaloRaw<TIN_NET> {
  struct type {
    float v[5] = {};
  };
};

// The same convolution with the input staged once per 32-channel slice: a
// block owns a TH x 16 pixel tile (TH = 8 MI: 128 MI pixels) of one image and
// BN = 32 NI output channels; per slice it stages the tile with its one-pixel
// halo ((TH + 2) x 18 pixels, zero outside the image) and the slice's weights
// of all nine taps in LDS, then runs the nine taps' MFMAs from there, so each
// input value is fetched once per slice instead of once per tap.  The next
// slice's halo and weights are fetched into registers while a slice's MFMAs
// run.  Wave w holds the pixel rows [2 MI w, 2 MI (w + 1)) of the tile (32
// pixels per MFMA row block).  The K order is (slice, tap).  With TPB > 1
// (Ci = 32) a block runs TPB consecutive tiles with the weights staged once.
// Requires Ci % 32 == 0, Co % BN == 0, H % TH == 0, W % 16 == 0.
template <bool RELU, int TOUT, int MI, int NI, int TPB, int TIN>
__global__ void __launch_bounds__(256) k_conv3x3_tile(const bf16_t *__restrict__ x, const bf16_t *__restrict__ w,
                                                      const float *__restrict__ bias, void *__restrict__ y, int H,
                                                      int W, int Ci, int Co, const bf16_t *__restrict__ x2, int C1,
                                                      TileIO io) {
  constexpr int TH = 8 * MI, TW = 16, HH = TH + 2, HW2 = TW + 2, BN = 32 * NI;
  constexpr int APIECES = HH * HW2 * 4, BPIECES = 9 * BN * 4;   // 16-byte pieces per slice
  constexpr int AREG = (APIECES + 255) / 256, BREG = (BPIECES + 255) / 256;   // pieces per thread
  __shared__ __attribute__((aligned(16))) bf16_t Ah[HH * HW2][CV_BK + CV_PAD];
  __shared__ __attribute__((aligned(16))) bf16_t Bw[9 * BN][CV_BK + CV_PAD];
  __shared__ float Uo[TOUT == TOUT_U0 ? TH * TW : 1][2];   // TOUT_U0: channels 0, 1 of the tile
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int tiles_x = W / TW, tiles_y = H / TH;
  const int co0 = blockIdx.y * BN;
  const int Cx = x2 ? C1 : Ci, H2 = H >> 1, W2 = W >> 1;
  const int csteps = Ci / CV_BK;
  // tile -> (image, top row, left column)
  auto tile_at = [&](int tl, int &bimg, int &y0, int &x0) {
    bimg = tl / (tiles_x * tiles_y);
    const int trem = tl - bimg * tiles_x * tiles_y;
    y0 = (trem / tiles_x) * TH;
    x0 = (trem % tiles_x) * TW;
  };
  // The halo is fetched in two steps so that a prefetch does not wait on its
  // loads: load_halo issues the raw loads of each 16-byte piece (8 channels)
  // into registers, store_halo forms the piece (pooling average or network
  // input) and writes it to LDS.  Pixels outside the image stay zero.
  using Raw = typename HaloRaw<TIN>::type;
  auto load_raw = [&](int bimg, int yy, int xx, int ci, Raw &r) {
    if constexpr (TIN == TIN_NET) {
      if (ci == 0) {
        const size_t i = ((size_t)bimg * H + yy) * W + xx;
        r.v[0] = io.f[i];
        r.v[1] = io.uin[i].x;
        r.v[2] = io.uin[i].y;
        if (io.ub) {
          r.v[3] = io.ub[i].x;
          r.v[4] = io.ub[i].y;
        }
      }
    } else if constexpr (TIN == TIN_POOL) {
      const int W0 = 2 * W;
      const bf16_t *src = x + ((size_t)(bimg * 2 * H + 2 * yy) * W0 + 2 * xx) * Ci + ci;
      r.v[0] = *reinterpret_cast<const u32x4 *>(src);
      r.v[1] = *reinterpret_cast<const u32x4 *>(src + Ci);
      r.v[2] = *reinterpret_cast<const u32x4 *>(src + (size_t)W0 * Ci);
      r.v[3] = *reinterpret_cast<const u32x4 *>(src + (size_t)W0 * Ci + Ci);
    } else {
      const bf16_t *src = x2 && ci >= C1
                              ? x2 + ((size_t)(bimg * H2 + (yy >> 1)) * W2 + (xx >> 1)) * (Ci - C1) + (ci - C1)
                              : x + ((size_t)(bimg * H + yy) * W + xx) * Cx + ci;
      r.v[0] = *reinterpret_cast<const u32x4 *>(src);
    }
  };
  auto form = [&](const Raw &r) -> u32x4 {
    if constexpr (TIN == TIN_NET) {
      u32x4 v = u32x4{0, 0, 0, 0};
      bf16_t *e = reinterpret_cast<bf16_t *>(&v);
#pragma unroll
      for (int j = 0; j < 5; ++j) e[j] = f2bf(r.v[j]);
      return v;
    } else if constexpr (TIN == TIN_POOL) {
      float acc[8] = {};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bf16_t *e = reinterpret_cast<const bf16_t *>(&r.v[q]);
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] += bf2f(e[j]);
      }
      u32x4 o;
      bf16_t *oe = reinterpret_cast<bf16_t *>(&o);
#pragma unroll
      for (int j = 0; j < 8; ++j) oe[j] = f2bf(0.25f * acc[j]);
      return o;
    } else {
      return r.v[0];
    }
  };
  auto load_halo = [&](int bimg, int y0, int x0, int ci0, Raw (&r)[AREG]) {
#pragma unroll
    for (int k = 0; k < AREG; ++k) {
      const int c = tid + 256 * k;
      r[k] = Raw{};
      if (c >= APIECES) continue;
      const int pix = c >> 2, part4 = c & 3;
      const int yy = y0 + pix / HW2 - 1, xx = x0 + pix % HW2 - 1;
      if (yy >= 0 && yy < H && xx >= 0 && xx < W) load_raw(bimg, yy, xx, ci0 + part4 * 8, r[k]);
    }
  };
  auto store_halo = [&](const Raw (&r)[AREG]) {
#pragma unroll
    for (int k = 0; k < AREG; ++k) {
      const int c = tid + 256 * k;
      if (c < APIECES) *reinterpret_cast<u32x4 *>(&Ah[c >> 2][(c & 3) * 8]) = form(r[k]);
    }
  };
  // weight pieces of one slice into registers, then into LDS
  auto load_weights = [&](int ci0, u32x4 (&r)[BREG]) {
#pragma unroll
    for (int k = 0; k < BREG; ++k) {
      const int c = min(tid + 256 * k, BPIECES - 1);   // the tail re-reads the last piece
      const int row = c >> 2, part4 = c & 3;           // row = tap * BN + co
      const int tap = row / BN, co = row - tap * BN;
      r[k] = *reinterpret_cast<const u32x4 *>(w + ((size_t)tap * Co + co0 + co) * Ci + ci0 + part4 * 8);
    }
  };
  auto store_weights = [&](const u32x4 (&r)[BREG]) {
#pragma unroll
    for (int k = 0; k < BREG; ++k) {
      const int c = tid + 256 * k;
      if (c < BPIECES) *reinterpret_cast<u32x4 *>(&Bw[c >> 2][(c & 3) * 8]) = r[k];
    }
  };
  f32x16 acc[MI][NI];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] = f32x16{0};
  };
  auto mfma_slice = [&]() {
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int dy = tap / 3, dx = tap % 3;   // halo offsets (the halo starts one pixel up and left)
#pragma unroll
      for (int kk = 0; kk < CV_BK; kk += 16) {
        bf16x8 a[MI], bv[NI];
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          const int p = (wave * MI + i) * 32 + (lane & 31);
          const int hp = (p / TW + dy) * HW2 + (p % TW) + dx;
          a[i] = *reinterpret_cast<const bf16x8 *>(&Ah[hp][kk + 8 * (lane >> 5)]);
        }
#pragma unroll
        for (int j = 0; j < NI; ++j)
          bv[j] = *reinterpret_cast<const bf16x8 *>(&Bw[tap * BN + j * 32 + (lane & 31)][kk + 8 * (lane >> 5)]);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], bv[j], acc[i][j], 0, 0, 0);
      }
    }
  };
  // epilogue of one tile: accumulator row q of MFMA row block g is tile row
  // (32 g + q) / 16, column (32 g + q) % 16
  auto store_out = [&](int bimg, int y0, int x0) {
    auto pixel = [&](int g, int q) {
      const int py = (g * 32 + q) / TW, px = (g * 32 + q) % TW;
      return ((size_t)bimg * H + y0 + py) * W + x0 + px;
    };
    if constexpr (TOUT == TOUT_U0) {
      // channels 0 and 1 of the tile through LDS, then one complex value per
      // thread: u0 = u_in + (y0 + i y1)
      const int co = lane & 31;
      if (co0 == 0 && co < 2) {
        const float bb = bias ? bias[co] : 0.0f;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int q = (wave * MI + i) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            Uo[q][co] = acc[i][0][r] + bb;
          }
      }
      __syncthreads();
      if (co0 == 0)
        for (int q = tid; q < TH * TW; q += 256) {
          const size_t P = ((size_t)bimg * H + y0 + q / TW) * W + x0 + q % TW;
          const cf a = io.uin[P];
          io.u0[P] = mk<cf>(a.x + Uo[q][0], a.y + Uo[q][1]);
        }
      return;
    }
    if constexpr (TOUT == TOUT_F32) {
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int co = co0 + j * 32 + (lane & 31);
        const float bb = bias ? bias[co] : 0.0f;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const size_t P = pixel(wave * MI + i, 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3));
            float v = acc[i][j][r] + bb;
            if (RELU) v = fmaxf(v, 0.0f);
            reinterpret_cast<float *>(y)[P * Co + co] = v;
          }
        }
      }
      return;
    }
    // bf16: 32 channels at a time through the wave's own rows of the halo's LDS
    // (no wave reads the halo any more), so that a lane stores, and masks, 16
    // bytes instead of two (the 128^2 x 16 network forward: 222 -> 214 us)
    static_assert(128 * MI <= HH * HW2, "the tile's outputs are staged in the halo's LDS");
    bf16_t (*out)[CV_BK + CV_PAD] = Ah + wave * MI * 32;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const float bb = bias ? bias[co0 + j * 32 + (lane & 31)] : 0.0f;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float v = acc[i][j][r] + bb;
          if (RELU) v = fmaxf(v, 0.0f);
          out[i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)][lane & 31] = f2bf(v);
        }
      }
      wave_lds_order();
#pragma unroll
      for (int k = 0; k < 2 * MI; ++k) {
        const int q = (lane >> 2) + 16 * k;   // pixel of the wave's 32 MI
        const size_t P = pixel(wave * MI, q) * Co + co0 + j * 32 + (lane & 3) * 8;
        u32x4 v = *reinterpret_cast<const u32x4 *>(&out[q][(lane & 3) * 8]);
        if constexpr (TOUT == TOUT_MASK) {
          const u32x4 m = *reinterpret_cast<const u32x4 *>(io.mask + P);
#pragma unroll
          for (int d = 0; d < 4; ++d) {   // positive bf16: sign clear, and not zero (NaN is not positive either)
            const uint32_t lo = m[d] << 16, hi = m[d] & 0xffff0000u;
            if (!(__builtin_bit_cast(float, lo) > 0.0f)) v[d] &= 0xffff0000u;
            if (!(__builtin_bit_cast(float, hi) > 0.0f)) v[d] &= 0x0000ffffu;
          }
        }
        *reinterpret_cast<u32x4 *>(reinterpret_cast<bf16_t *>(y) + P) = v;
      }
      wave_lds_order();
    }
  };
  int bimg, y0, x0;
  Raw hr[AREG];
  u32x4 wr[BREG];
  if constexpr (TPB == 1) {
    tile_at(blockIdx.x, bimg, y0, x0);
    clear();
    load_halo(bimg, y0, x0, 0, hr);
    load_weights(0, wr);
    for (int sl = 0; sl < csteps; ++sl) {
      store_halo(hr);
      store_weights(wr);
      __syncthreads();
      if (sl + 1 < csteps) {
        load_halo(bimg, y0, x0, (sl + 1) * CV_BK, hr);
        load_weights((sl + 1) * CV_BK, wr);
      }
      mfma_slice();
      __syncthreads();
    }
    store_out(bimg, y0, x0);
  } else {
    // one 32-channel slice (Ci = 32): each tile's halo is fetched into
    // registers while the previous tile's MFMAs run
    load_weights(0, wr);
    store_weights(wr);
    tile_at(blockIdx.x * TPB, bimg, y0, x0);
    load_halo(bimg, y0, x0, 0, hr);
    store_halo(hr);
    __syncthreads();
    for (int t = 0; t < TPB; ++t) {
      int nb = 0, ny = 0, nx = 0;
      if (t + 1 < TPB) {
        tile_at(blockIdx.x * TPB + t + 1, nb, ny, nx);
        load_halo(nb, ny, nx, 0, hr);
      }
      clear();
      mfma_slice();
      __syncthreads();   // every wave is done with this tile's halo
      store_out(bimg, y0, x0);
      if (t + 1 < TPB) {
        __syncthreads();   // and with the outputs staged there
        store_halo(hr);
        __syncthreads();
        bimg = nb;
        y0 = ny;
        x0 = nx;
      }
    }
  }
}

// Split-K epilogue: y = act(sum_z part[z] + bias), the partial sums added in
// split order (deterministic); four consecutive channels per thread.
template <bool RELU, bool OUT_F32>
__global__ void k_conv_splitk_reduce(const float *__restrict__ part, int splits, size_t MC,
                                     const float *__restrict__ bias, int Co, void *__restrict__ y) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < MC / 4; i += (size_t)gridDim.x * blockDim.x) {
    float4 a = reinterpret_cast<const float4 *>(part)[i];
    for (int z = 1; z < splits; ++z) {
      const float4 b = reinterpret_cast<const float4 *>(part + (size_t)z * MC)[i];
      a.x += b.x;
      a.y += b.y;
      a.z += b.z;
      a.w += b.w;
    }
    const int co = (int)((4 * i) % Co);
    float v[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] += bias ? bias[co + k] : 0.0f;
      if (RELU) v[k] = fmaxf(v[k], 0.0f);
    }
    if (OUT_F32) {
      reinterpret_cast<float4 *>(y)[i] = make_float4(v[0], v[1], v[2], v[3]);
    } else {
      uint2 o;
      bf16_t *e = reinterpret_cast<bf16_t *>(&o);
#pragma unroll
      for (int k = 0; k < 4; ++k) e[k] = f2bf(v[k]);
      reinterpret_cast<uint2 *>(y)[i] = o;
    }
  }
}

// ------------------------------------------------------------------ conv weight gradient
// part[split][tap][co][ci] = sum over the pixels of a split of dy[p][co] x[shift(p, tap)][ci],
// and with bpart the bias gradient bpart[split][co] = sum dy[p][co].
// A GEMM with the pixels as its long inner dimension, whose operands lie with
// the channels contiguous.  A block of eight waves owns 32 output x 32 input
// channels and all nine taps (nine 32x32 accumulators per wave), so x and dy
// are staged once instead of once per tap; each wave walks its own 16-pixel
// wide strips down the image (a task is rh rows of one strip) and needs no
// block barrier until the eight waves' sums are added at the end.  Per row it
// stages 18 x pixels (one of halo on each side) and 16 dy pixels in its part
// of the LDS as they lie in memory ([pixel][32 channels], 64 bytes a pixel, no
// bank conflicts) and reads MFMA operands, eight consecutive pixels of one
// channel per lane, with the transposing LDS read (four 16-bit values of a
// column per lane; 16 lanes cover 4 pixels x 16 channels).  A tap's horizontal
// shift is a pixel offset of that read and its vertical shift one of the last
// three rows, which stay in registers: nine MFMAs per row for four reads'
// worth of fresh operands.  The next two rows are fetched into registers
// meanwhile.  With x2 set the input is [x (C1 channels) | up2(x2)] as in the
// forward convolution.  Pixels outside the image are zeros, so any width runs
// (a strip past the edge is cut).
// Bound by launch and fill latency at the network's sizes (256 blocks, one
// per CU): the 15 layers of a 128^2 x 16 batch take 265 us against
// 986 us for one tap per block with element-wise transposing LDS stores.
constexpr int WG_RB = 2;                                // rows per batch
constexpr int WG_WAVES = 8;
constexpr int WG_XP = 18, WG_DP = 16;                   // staged pixels per row
constexpr int WG_XROW = WG_XP * 32, WG_DROW = WG_DP * 32;   // bf16 elements per staged row
constexpr int WG_STAGE = (WG_RB + 2) * WG_XROW + WG_RB * WG_DROW;
constexpr int WG_RED = WG_WAVES * 1024;                 // floats of one tap's eight wave sums
struct WgArgs {
  const bf16_t *x, *dy, *x2;
  float *part, *bpart;
  int H, W, Ci, Co, C1, rh, segs, strips, tasks;
};
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// Eight consecutive pixels of one channel: lane l takes channel l % 32, pixels
// 8 (l / 32) .. + 8 of a staged row ([pixel][32]) that starts at p.
__device__ __forceinline__ bf16x8 tr_frag(const bf16_t *p) {
  typedef __attribute__((address_space(3))) s16x4 *lds4;
  const int l = threadIdx.x & 63;
  const bf16_t *q = p + (8 * (l >> 5) + ((l & 15) >> 2)) * 32 + 16 * ((l >> 4) & 1) + 4 * (l & 3);
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)q);
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(q + 4 * 32));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <typename OFF>   // holds the element offsets of an image
__global__ void __launch_bounds__(64 * WG_WAVES, 2) k_conv3x3_wgrad(WgArgs a) {
  constexpr int XB = (WG_RB * WG_XP * 4 + 63) / 64;   // x pieces (16 bytes) per lane and batch
  constexpr int XP = (2 * WG_XP * 4 + 63) / 64;       // of the two rows above a task's first batch
  __shared__ __attribute__((aligned(16))) bf16_t stage[WG_WAVES][WG_STAGE];
  static_assert(sizeof(stage) >= sizeof(float) * WG_RED, "the sums are added in the staging area");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int ci0 = blockIdx.x * 32, co0 = blockIdx.y * 32;
  const int H = a.H, W = a.W;
  const bool up = a.x2 && ci0 >= a.C1;
  const int Cx = up ? a.Ci - a.C1 : (a.x2 ? a.C1 : a.Ci), cx0 = up ? ci0 - a.C1 : ci0;
  const bf16_t *xs = up ? a.x2 : a.x;
  const int sh = up ? 1 : 0, Hs = H >> sh, Ws = W >> sh;
  bf16_t *sx = stage[wave], *sd = sx + (WG_RB + 2) * WG_XROW;
  f32x16 acc[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) acc[t] = f32x16{0};
  float bsum = 0.0f;
  const bool bias = a.bpart && ci0 == 0;
  int x0 = 0, y1 = 0;
  const bf16_t *xi = nullptr, *di = nullptr;   // the image's x and dy from channel cx0, co0 on
  // piece i of nr consecutive x rows from row yy on (zero outside the image)
  auto load_x = [&](int i, int nr, int yy) -> u32x4 {
    const int row = i / (WG_XP * 4), rem = i - row * (WG_XP * 4);
    const int y = yy + row, xx = x0 - 1 + (rem >> 2);
    u32x4 v = u32x4{0, 0, 0, 0};
    if (row < nr && y >= 0 && y < H && xx >= 0 && xx < W)
      v = *reinterpret_cast<const u32x4 *>(xi + (((OFF)(y >> sh) * Ws + (xx >> sh)) * Cx + (rem & 3) * 8));
    return v;
  };
  u32x4 rx[XB], rd[WG_RB];
  auto load_batch = [&](int yb) {   // x rows yb + 1 .. yb + WG_RB, dy rows yb .. (zero past the task)
#pragma unroll
    for (int k = 0; k < XB; ++k) rx[k] = load_x(lane + 64 * k, WG_RB, yb + 1);
#pragma unroll
    for (int k = 0; k < WG_RB; ++k) {
      const int xx = x0 + (lane >> 2);
      rd[k] = u32x4{0, 0, 0, 0};
      if (yb + k < y1 && xx < W)
        rd[k] = *reinterpret_cast<const u32x4 *>(di + (((OFF)(yb + k) * W + xx) * a.Co + (lane & 3) * 8));
    }
  };
  for (int task = blockIdx.z * WG_WAVES + wave; task < a.tasks; task += gridDim.z * WG_WAVES) {
    const int seg = task % a.segs, rest = task / a.segs;
    x0 = (rest % a.strips) * 16;
    const int img = rest / a.strips;
    xi = xs + (size_t)img * Hs * Ws * Cx + cx0;
    di = a.dy + (size_t)img * H * W * a.Co + co0;
    const int y0 = seg * a.rh;
    y1 = min(y0 + a.rh, H);
    u32x4 rp[XP];
#pragma unroll
    for (int k = 0; k < XP; ++k) rp[k] = load_x(lane + 64 * k, 2, y0 - 1);
    load_batch(y0);
#pragma unroll
    for (int k = 0; k < XP; ++k)
      if (lane + 64 * k < 2 * WG_XP * 4) *reinterpret_cast<u32x4 *>(sx + (lane + 64 * k) * 8) = rp[k];
    wave_lds_order();
    bf16x8 f0[3], f1[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      f0[d] = tr_frag(sx + d * 32);
      f1[d] = tr_frag(sx + WG_XROW + d * 32);
    }
    for (int yb = y0; yb < y1; yb += WG_RB) {
#pragma unroll
      for (int k = 0; k < XB; ++k)
        if (lane + 64 * k < WG_RB * WG_XP * 4)
          *reinterpret_cast<u32x4 *>(sx + 2 * WG_XROW + (lane + 64 * k) * 8) = rx[k];
#pragma unroll
      for (int k = 0; k < WG_RB; ++k) *reinterpret_cast<u32x4 *>(sd + k * WG_DROW + lane * 8) = rd[k];
      wave_lds_order();
      if (yb + WG_RB < y1) load_batch(yb + WG_RB);
#pragma unroll
      for (int r = 0; r < WG_RB; ++r) {
        const bf16x8 d = tr_frag(sd + r * WG_DROW);
        bf16x8 f2[3];
#pragma unroll
        for (int s = 0; s < 3; ++s) f2[s] = tr_frag(sx + (2 + r) * WG_XROW + s * 32);
        if (bias) {
#pragma unroll
          for (int j = 0; j < 8; ++j) bsum += (float)d[j];
        }
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          acc[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d, f0[s], acc[s], 0, 0, 0);
          acc[3 + s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d, f1[s], acc[3 + s], 0, 0, 0);
          acc[6 + s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d, f2[s], acc[6 + s], 0, 0, 0);
        }
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          f0[s] = f1[s];
          f1[s] = f2[s];
        }
      }
      wave_lds_order();
    }
  }
  // the waves' sums, one tap at a time, added in wave order
  float *red = reinterpret_cast<float *>(&stage[0][0]);
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r)
      red[wave * 1024 + (8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * 32 + (lane & 31)] = acc[t][r];
    __syncthreads();
    for (int e = threadIdx.x; e < 1024; e += 64 * WG_WAVES) {
      float s = red[e];
#pragma unroll
      for (int w = 1; w < WG_WAVES; ++w) s += red[w * 1024 + e];
      a.part[(((size_t)blockIdx.z * 9 + t) * a.Co + co0 + e / 32) * a.Ci + ci0 + e % 32] = s;
    }
  }
  if (!bias) return;
  __syncthreads();
  red[threadIdx.x] = bsum;
  __syncthreads();
  if (threadIdx.x < 32) {
    float s = 0.0f;
    for (int w = 0; w < 2 * WG_WAVES; ++w) s += red[w * 32 + threadIdx.x];
    a.bpart[(size_t)blockIdx.z * a.Co + co0 + threadIdx.x] = s;
  }
}

// out[i] = sum of the `splits` partials part[k][i] of several arrays in one
// launch (a launch per layer and array would cost more than the sums).  A
// block owns 32 consecutive 16-byte groups of one array; eight lanes a group
// sum every eighth split, and the lanes are added in order.
constexpr int RED_ITEMS = 32;
struct RedItem {
  const float *part;
  float *out;
  unsigned n;        // elements, a multiple of 4
  int splits;
  unsigned block0;   // first block of the array
};
struct RedList {
  RedItem it[RED_ITEMS];
  int count = 0;
  unsigned blocks = 0;
  void add(const float *part, float *out, size_t n, int splits) {
    it[count++] = RedItem{part, out, (unsigned)n, splits, blocks};
    blocks += (unsigned)((n + 127) / 128);
  }
};
__global__ void __launch_bounds__(256) k_sum_splits(RedList l) {
  __shared__ float4 sh[8][32];
  int k = 0;
  while (k + 1 < l.count && blockIdx.x >= l.it[k + 1].block0) ++k;
  const RedItem it = l.it[k];
  const int c = threadIdx.x & 31, z0 = threadIdx.x >> 5;
  const unsigned g = (blockIdx.x - it.block0) * 32 + c;
  float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (4 * g < it.n) {
    for (int z = z0; z < it.splits; z += 8) {
      const float4 v = reinterpret_cast<const float4 *>(it.part + (size_t)z * it.n)[g];
      s.x += v.x;
      s.y += v.y;
      s.z += v.z;
      s.w += v.w;
    }
  }
  sh[z0][c] = s;
  __syncthreads();
  if (z0 || 4 * g >= it.n) return;
#pragma unroll
  for (int z = 1; z < 8; ++z) {
    s.x += sh[z][c].x;
    s.y += sh[z][c].y;
    s.z += sh[z][c].z;
    s.w += sh[z][c].w;
  }
  reinterpret_cast<float4 *>(it.out)[g] = s;
}

// w'[tap][ci][co] = w[8 - tap][co][ci] of every layer (the data gradient is
// the forward convolution with w'); wt has the layout of the parameter vector.
struct FlipList {
  struct { unsigned woff; int Ci, Co; } l[16];
  int count = 0;
};
__global__ void k_flip_transpose(const bf16_t *w, bf16_t *wt, FlipList f) {
  const unsigned off = f.l[blockIdx.y].woff;
  const unsigned Ci = f.l[blockIdx.y].Ci, Co = f.l[blockIdx.y].Co, n = 9 * Ci * Co;
  for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const unsigned tap = i / (Ci * Co), rem = i % (Ci * Co), ci = rem / Co, co = rem % Co;
    wt[off + i] = w[off + ((8 - tap) * Co + co) * Ci + ci];
  }
}

// dz = dy * (y > 0)
__global__ void k_relu_bwd(const bf16_t *dy, const bf16_t *y, bf16_t *dz, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    dz[i] = bf2f(y[i]) > 0.0f ? dy[i] : (bf16_t)0;
}

// 2x2 average pooling, NHWC, eight channels (one 16-byte vector) per thread
// (C is a multiple of 8).
__global__ void k_avgpool(const bf16_t *x, bf16_t *y, int B, int H, int W, int C) {
  const int Ho = H / 2, Wo = W / 2, C8 = C / 8;
  const size_t n = (size_t)B * Ho * Wo * C8;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const int c = (int)(i % C8) * 8;
    const size_t p = i / C8;
    const int xo = p % Wo, yo = (p / Wo) % Ho, b = (int)(p / ((size_t)Wo * Ho));
    const size_t base = ((size_t)(b * H + 2 * yo) * W + 2 * xo) * C + c;
    const size_t off[4] = {base, base + C, base + (size_t)W * C, base + (size_t)W * C + C};
    float acc[8] = {};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint4 v = *reinterpret_cast<const uint4 *>(x + off[q]);
      const bf16_t *e = reinterpret_cast<const bf16_t *>(&v);
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] += bf2f(e[j]);
    }
    uint4 o;
    bf16_t *oe = reinterpret_cast<bf16_t *>(&o);
#pragma unroll
    for (int j = 0; j < 8; ++j) oe[j] = f2bf(0.25f * acc[j]);
    *reinterpret_cast<uint4 *>(y + p * C + c) = o;
  }
}
// Eight bf16 values of one 16-byte piece.
__device__ __forceinline__ void unpack8(const uint4 &v, float (&o)[8]) {
  const bf16_t *e = reinterpret_cast<const bf16_t *>(&v);
#pragma unroll
  for (int j = 0; j < 8; ++j) o[j] = bf2f(e[j]);
}
// Rounds v to bf16, zero where the activation y is not positive (ReLU), and
// stores the eight values.
__device__ __forceinline__ void store8_masked(bf16_t *dst, const float (&v)[8], const bf16_t *y) {
  float m[8];
  unpack8(*reinterpret_cast<const uint4 *>(y), m);
  uint4 o;
  bf16_t *e = reinterpret_cast<bf16_t *>(&o);
#pragma unroll
  for (int j = 0; j < 8; ++j) e[j] = m[j] > 0.0f ? f2bf(v[j]) : (bf16_t)0;
  *reinterpret_cast<uint4 *>(dst) = o;
}
// Gradient at an encoder level's output y [B][H][W][C], its ReLU applied: the
// pooled path dyp / 4 ([B][H/2][W/2][C]) plus the skip part, the first C of the
// Ct channels of the decoder's input gradient gc.
__global__ void k_pool_skip_bwd(const bf16_t *dyp, const bf16_t *gc, const bf16_t *y, bf16_t *dx, int B, int H, int W,
                                int C, int Ct) {
  const int C8 = C / 8, Ho = H / 2, Wo = W / 2;
  const size_t n = (size_t)B * H * W * C8;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const int c = (int)(i % C8) * 8;
    const size_t p = i / C8;
    const int xx = p % W, yy = (p / W) % H, b = (int)(p / ((size_t)W * H));
    float v[8], g[8];
    unpack8(*reinterpret_cast<const uint4 *>(dyp + ((size_t)(b * Ho + yy / 2) * Wo + xx / 2) * C + c), v);
    unpack8(*reinterpret_cast<const uint4 *>(gc + p * Ct + c), g);
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = 0.25f * v[j] + g[j];
    store8_masked(dx + p * C + c, v, y + p * C + c);
  }
}
// Gradient at the output y [B][H][W][C] of the level below a decoder level,
// its ReLU applied: the sum over each 2x2 block of the last C of the Ct
// channels of the decoder's input gradient gc ([B][2H][2W][Ct]).
__global__ void k_upsample_bwd(const bf16_t *gc, const bf16_t *y, bf16_t *dx, int B, int H, int W, int C, int Ct) {
  const int C8 = C / 8;
  const size_t n = (size_t)B * H * W * C8, row = (size_t)2 * W * Ct;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const int c = (int)(i % C8) * 8;
    const size_t p = i / C8;
    const int xx = p % W, yy = (p / W) % H, b = (int)(p / ((size_t)W * H));
    const bf16_t *src = gc + ((size_t)(b * 2 * H + 2 * yy) * 2 * W + 2 * xx) * Ct + Ct - C + c;
    float v[8], g[3][8];
    unpack8(*reinterpret_cast<const uint4 *>(src), v);
    unpack8(*reinterpret_cast<const uint4 *>(src + Ct), g[0]);
    unpack8(*reinterpret_cast<const uint4 *>(src + row), g[1]);
    unpack8(*reinterpret_cast<const uint4 *>(src + row + Ct), g[2]);
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = v[j] + g[0][j] + g[1][j] + g[2][j];
    store8_masked(dx + p * C + c, v, y + p * C + c);
  }
}

// network input: channels (f, Re u_in, Im u_in, Re u_B, Im u_B, 0, ...) as
// bf16, 32 channels; u_B (the first-Born scattered field) may be absent (zeros).
__global__ void k_net_input(const float *f, const cf *uin, const cf *ub, bf16_t *x, int B, int N) {
  const size_t n = (size_t)B * N;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const cf b = ub ? ub[i] : mk<cf>(0.0f, 0.0f);
    uint4 v = make_uint4(0, 0, 0, 0);
    bf16_t *e = reinterpret_cast<bf16_t *>(&v);
    e[0] = f2bf(f[i]);
    e[1] = f2bf(uin[i].x);
    e[2] = f2bf(uin[i].y);
    e[3] = f2bf(b.x);
    e[4] = f2bf(b.y);
    uint4 *o = reinterpret_cast<uint4 *>(x + i * 32);   // 32 channels: one data vector, three zero vectors
    o[0] = v;
    o[1] = o[2] = o[3] = make_uint4(0, 0, 0, 0);
  }
}
// u0 = u_in + (out0 + i out1)
__global__ void k_net_output(const float *out, const cf *uin, cf *u0, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    u0[i] = mk<cf>(uin[i].x + out[i * 32], uin[i].y + out[i * 32 + 1]);
}
// Relative L2 loss per sample, averaged over the batch:
//   L = (1/B) sum_b ||out_b - (u_b - uin_b)||^2 / ||u_b - uin_b||^2
// k_rel_l2_part sums both norms over LOSS_PARTS parts of a sample (one block
// each: a block per sample left 240 CUs idle), k_rel_l2 adds the parts and
// writes the per-sample loss and the output gradient (bf16, 32 channels).
constexpr int LOSS_PARTS = 32;
__global__ void __launch_bounds__(256) k_rel_l2_part(const float *out, const cf *uin, const cf *u, double *part,
                                                     int N) {
  __shared__ double scratch[2 * 16];
  const int b = blockIdx.y;
  double acc[2] = {0.0, 0.0};
  for (int q = blockIdx.x * 256 + threadIdx.x; q < N; q += LOSS_PARTS * 256) {
    const size_t i = (size_t)b * N + q;
    const float2 o = *reinterpret_cast<const float2 *>(out + i * 32);
    const double tr = (double)u[i].x - uin[i].x, ti = (double)u[i].y - uin[i].y;
    const double er = o.x - tr, ei = o.y - ti;
    acc[0] += er * er + ei * ei;
    acc[1] += tr * tr + ti * ti;
  }
  block_sum<2>(acc, scratch);
  if (threadIdx.x == 0) {
    part[2 * (b * LOSS_PARTS + blockIdx.x)] = acc[0];
    part[2 * (b * LOSS_PARTS + blockIdx.x) + 1] = acc[1];
  }
}
__global__ void __launch_bounds__(256) k_rel_l2(const float *out, const cf *uin, const cf *u, const double *part,
                                                bf16_t *dout, double *loss_b, int N, int B) {
  const int b = blockIdx.y;
  double e2 = 0.0, t2 = 0.0;
  for (int k = 0; k < LOSS_PARTS; ++k) {
    e2 += part[2 * (b * LOSS_PARTS + k)];
    t2 += part[2 * (b * LOSS_PARTS + k) + 1];
  }
  const double tt = fmax(t2, 1e-30);
  if (blockIdx.x == 0 && threadIdx.x == 0) loss_b[b] = e2 / tt;
  const float scale = (float)(2.0 / (tt * B));
  // four threads a pixel, eight of its 32 channels each
  const int seg = threadIdx.x & 3;
  for (int q = blockIdx.x * 64 + (threadIdx.x >> 2); q < N; q += gridDim.x * 64) {
    const size_t i = (size_t)b * N + q;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (seg == 0) {
      const float2 o = *reinterpret_cast<const float2 *>(out + i * 32);
      bf16_t *e = reinterpret_cast<bf16_t *>(&v);
      const float tr = u[i].x - uin[i].x, ti = u[i].y - uin[i].y;
      e[0] = f2bf(scale * (o.x - tr));
      e[1] = f2bf(scale * (o.y - ti));
    }
    *reinterpret_cast<uint4 *>(dout + i * 32 + seg * 8) = v;
  }
}

// Global-norm gradient clipping: FP64 block partials of |g|^2, then one block
// turns them into the factor min(1, clip / |g|) (1 when clip <= 0).
__global__ void __launch_bounds__(256) k_sqnorm_part(const float *g, size_t n, double *part) {
  __shared__ double scratch[16];
  double acc[1] = {0.0};
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    acc[0] += (double)g[i] * g[i];
  block_sum<1>(acc, scratch);
  if (threadIdx.x == 0) part[blockIdx.x] = acc[0];
}
__global__ void k_clip_factor(const double *part, int nparts, double clip, float *factor) {
  if (threadIdx.x != 0) return;
  double s = 0.0;
  for (int i = 0; i < nparts; ++i) s += part[i];
  const double nrm = sqrt(s);
  factor[0] = (clip > 0.0 && nrm > clip) ? (float)(clip / nrm) : 1.0f;
}

__global__ void k_adam(float *w, const float *g, const float *gscale, float *m, float *v, bf16_t *wb, size_t n,
                       float lr, float b1, float b2, float eps, float c1, float c2) {
  const float sc = gscale[0];
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const float gi = g[i] * sc;
    const float mi = b1 * m[i] + (1 - b1) * gi;
    const float vi = b2 * v[i] + (1 - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    w[i] = wi;
    if (wb) wb[i] = f2bf(wi);
  }
}
__global__ void k_to_bf16(const float *a, bf16_t *b, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    b[i] = f2bf(a[i]);
}

static dim3 grid1(size_t n) { return dim3((unsigned)std::min<size_t>((n + 255) / 256, 8192)); }

// ------------------------------------------------------------------ launch helpers
template <int MI, int NI>
static void conv_fwd_t(hipStream_t s, const bf16_t *x, const bf16_t *w, const float *bias, void *y, int M, int H,
                       int W, int Ci, int Co, bool relu, bool out_f32, const bf16_t *x2, int C1, int splits,
                       int s_steps, float *part) {
  const dim3 g(M / (128 * MI), Co / (32 * NI), splits);
  float *pp = splits > 1 ? part : nullptr;
  if (relu && !out_f32)
    hipLaunchKernelGGL((k_conv3x3<true, false, MI, NI>), g, dim3(256), 0, s, x, w, bias, y, H, W, Ci, Co, x2, C1,
                       s_steps, pp);
  else if (!relu && !out_f32)
    hipLaunchKernelGGL((k_conv3x3<false, false, MI, NI>), g, dim3(256), 0, s, x, w, bias, y, H, W, Ci, Co, x2, C1,
                       s_steps, pp);
  else if (relu)
    hipLaunchKernelGGL((k_conv3x3<true, true, MI, NI>), g, dim3(256), 0, s, x, w, bias, y, H, W, Ci, Co, x2, C1,
                       s_steps, pp);
  else
    hipLaunchKernelGGL((k_conv3x3<false, true, MI, NI>), g, dim3(256), 0, s, x, w, bias, y, H, W, Ci, Co, x2, C1,
                       s_steps, pp);
  if (splits <= 1) return;
  const size_t MC = (size_t)M * Co;
  const dim3 gr((unsigned)std::min<size_t>((MC / 4 + 255) / 256, 8192));
  if (relu && !out_f32)
    hipLaunchKernelGGL((k_conv_splitk_reduce<true, false>), gr, dim3(256), 0, s, part, splits, MC, bias, Co, y);
  else if (!relu && !out_f32)
    hipLaunchKernelGGL((k_conv_splitk_reduce<false, false>), gr, dim3(256), 0, s, part, splits, MC, bias, Co, y);
  else if (relu)
    hipLaunchKernelGGL((k_conv_splitk_reduce<true, true>), gr, dim3(256), 0, s, part, splits, MC, bias, Co, y);
  else
    hipLaunchKernelGGL((k_conv_splitk_reduce<false, true>), gr, dim3(256), 0, s, part, splits, MC, bias, Co, y);
}

// Launch shape of one convolution: the block tile (mi x 128 pixels, ni x 32
// channels) and the split of its K = 9 Ci loop over blocks.
struct ConvPlan {
  int mi = 1, ni = 1, splits = 1, s_steps = 0;
};
// Tile: the largest one that divides the layer and still gives at least 256
// blocks (one per CU), else the smallest; forced 1..6 picks an entry of the
// table (test hook).  Split K: a layer left with fewer than 1024 blocks (four
// waves per SIMD) has its 32-channel steps spread over up to 8 splits of at
// least 16 steps each (auto_split; shorter loops do not repay the extra pass
// over the partials), or over `splits` (> 0, test hook).
static bool conv_plan(int M, int Ci, int Co, int forced, int splits, bool auto_split, ConvPlan &p) {
  struct Tile { int mi, ni; };
  static const Tile tiles[] = {{2, 4}, {1, 4}, {2, 2}, {1, 2}, {2, 1}, {1, 1}};
  if (forced) {
    p.mi = tiles[forced - 1].mi;
    p.ni = tiles[forced - 1].ni;
    if (M % (128 * p.mi) || Co % (32 * p.ni)) return false;
  } else {
    p.mi = p.ni = 1;
    for (const Tile &t : tiles) {
      const int bm = 128 * t.mi, bn = 32 * t.ni;
      if (M % bm || Co % bn) continue;
      if ((long long)(M / bm) * (Co / bn) >= 256) {
        p.mi = t.mi;
        p.ni = t.ni;
        break;
      }
    }
  }
  const int nsteps = 9 * (Ci / 32);
  const long long blocks = (long long)(M / (128 * p.mi)) * (Co / (32 * p.ni));
  int want = 1;
  if (splits > 0)
    want = std::min(splits, nsteps);
  else if (auto_split && blocks < 1024)
    want = (int)std::min<long long>({(1024 + blocks - 1) / blocks, 8, std::max(1, nsteps / 16)});
  p.s_steps = (nsteps + want - 1) / want;
  p.splits = (nsteps + p.s_steps - 1) / p.s_steps;
  return true;
}

// One launch of k_conv3x3_tile; false for a combination of forms that has no
// kernel (the caller then takes the unfused path).
template <int MI, int NI, int TPB>
static bool conv_tile_t(hipStream_t s, const bf16_t *x, const bf16_t *w, const float *bias, void *y, int B, int H,
                        int W, int Ci, int Co, bool relu, int tout, int tin, const bf16_t *x2, int C1,
                        const TileIO &io) {
  const dim3 g(B * (H / (8 * MI)) * (W / 16) / TPB, Co / (32 * NI));
#define TILE_L(R, O, I)                                                                                               \
  hipLaunchKernelGGL((k_conv3x3_tile<R, O, MI, NI, TPB, I>), g, dim3(256), 0, s, x, w, bias, y, H, W, Ci, Co, x2, C1, \
                     io)
  if (tin == TIN_X && tout == TOUT_BF16) {
    if (relu)
      TILE_L(true, TOUT_BF16, TIN_X);
    else
      TILE_L(false, TOUT_BF16, TIN_X);
  } else if (tin == TIN_X && tout == TOUT_MASK && !relu) {
    TILE_L(false, TOUT_MASK, TIN_X);
  } else if (tin == TIN_X && tout == TOUT_F32) {
    if (relu)
      TILE_L(true, TOUT_F32, TIN_X);
    else
      TILE_L(false, TOUT_F32, TIN_X);
  } else if (tin == TIN_X && tout == TOUT_U0 && !relu) {
    TILE_L(false, TOUT_U0, TIN_X);
  } else if (tin == TIN_POOL && tout == TOUT_BF16 && relu) {
    TILE_L(true, TOUT_BF16, TIN_POOL);
  } else if (tin == TIN_NET && tout == TOUT_BF16 && relu) {
    TILE_L(true, TOUT_BF16, TIN_NET);
  } else {
    return false;
  }
#undef TILE_L
  return true;
}

// Plan of the tiled launch: the tile of 128 mi pixels x 32 ni channels
// (mi, ni <= 2), the largest that still gives 512 blocks (two blocks per CU),
// else the one with the most blocks; one-slice layers (Ci = 32) run
// TILES_PER_BLOCK tiles per block when 512 blocks remain.  K is not split: with
// the slices pipelined, splitting K plus its reduction pass cost more than the
// longer K loop at every layer of the warm-start network.
struct TilePlan {
  int mi = 0, ni = 0, tpb = 1;
};
constexpr int TILES_PER_BLOCK = 2;
static bool tile_plan(int B, int H, int W, int Ci, int Co, TilePlan &p) {
  if (W % 16 || Ci % 32 || Ci <= 0) return false;
  struct Tile { int mi, ni; };
  static const Tile tiles[] = {{2, 2}, {1, 2}, {2, 1}, {1, 1}};
  p = TilePlan{};
  long long best = -1;
  for (const Tile &t : tiles) {
    if (H % (8 * t.mi) || Co % (32 * t.ni)) continue;
    const long long blocks = (long long)B * (H / (8 * t.mi)) * (W / 16) * (Co / (32 * t.ni));
    if (blocks >= 512) {
      p.mi = t.mi;
      p.ni = t.ni;
      break;
    }
    if (blocks > best) {
      best = blocks;
      p.mi = t.mi;
      p.ni = t.ni;
    }
  }
  if (!p.mi) return false;
  const long long ntiles = (long long)B * (H / (8 * p.mi)) * (W / 16);
  if (Ci == 32 && ntiles % TILES_PER_BLOCK == 0 && ntiles / TILES_PER_BLOCK * (Co / (32 * p.ni)) >= 512)
    p.tpb = TILES_PER_BLOCK;
  return true;
}

// Tiled launch (k_conv3x3_tile) with the input form tin and output form tout;
// false when the tiled kernel does not apply (the caller then launches
// k_conv3x3, or the unfused kernels).
static bool conv_fwd_tiled(hipStream_t s, const bf16_t *x, const bf16_t *w, const float *bias, void *y, int B, int H,
                           int W, int Ci, int Co, bool relu, int tout, int tin, const bf16_t *x2, int C1,
                           const TileIO &io = TileIO{}) {
  if ((tin != TIN_X && x2) || (tin == TIN_NET && Ci != 32)) return false;
  TilePlan p;
  if (!tile_plan(B, H, W, Ci, Co, p)) return false;
  bool ok = false;
  switch (p.mi * 10 + p.ni + (p.tpb > 1 ? 100 : 0)) {
#define TILE_T(a, b, t)                                                                                              \
  case a * 10 + b + (t > 1 ? 100 : 0):                                                                               \
    ok = conv_tile_t<a, b, t>(s, x, w, bias, y, B, H, W, Ci, Co, relu, tout, tin, x2, C1, io);                        \
    break;
    TILE_T(2, 2, 1)
    TILE_T(1, 2, 1)
    TILE_T(2, 1, 1)
    TILE_T(1, 1, 1)
    TILE_T(2, 2, TILES_PER_BLOCK)
    TILE_T(1, 2, TILES_PER_BLOCK)
    TILE_T(2, 1, TILES_PER_BLOCK)
    TILE_T(1, 1, TILES_PER_BLOCK)
#undef TILE_T
  }
  return ok;
}

// x2 != null: the input is [x (C1 channels) | up2(x2) (Ci - C1 channels)].
// ws: FP32 split-K workspace of ws_elems floats (null: no split).
static int conv_fwd(hipStream_t s, const bf16_t *x, const bf16_t *w, const float *bias, void *y, int B, int H, int W,
                    int Ci, int Co, bool relu, bool out_f32, int forced = 0, const bf16_t *x2 = nullptr,
                    int C1 = 0, float *ws = nullptr, size_t ws_elems = 0, int splits = 0) {
  const int M = B * H * W;
  if (Ci % 32 || Co % 32 || M % 128 || forced < 0 || forced > 6 || splits < 0) return CISOR_E_ARG;
  if (x2 && (C1 <= 0 || C1 >= Ci || C1 % 32 || H % 2 || W % 2)) return CISOR_E_ARG;
  if (!forced && splits <= 1 &&
      conv_fwd_tiled(s, x, w, bias, y, B, H, W, Ci, Co, relu, out_f32 ? TOUT_F32 : TOUT_BF16, TIN_X, x2, C1))
    return hipGetLastError() == hipSuccess ? CISOR_OK : CISOR_E_DEVICE;
  ConvPlan p;
  if (!conv_plan(M, Ci, Co, forced, splits, ws != nullptr, p)) return CISOR_E_ARG;
  if (p.splits > 1 && (!ws || (size_t)p.splits * M * Co > ws_elems)) {
    if (splits > 1) return CISOR_E_ARG;   // an explicit split needs the workspace
    p.s_steps = 9 * (Ci / 32);
    p.splits = 1;
  }
  switch (p.mi * 10 + p.ni) {
#define CONV_T(a, b)                                                                                                  \
  case a * 10 + b:                                                                                                     \
    conv_fwd_t<a, b>(s, x, w, bias, y, M, H, W, Ci, Co, relu, out_f32, x2, C1, p.splits, p.s_steps, ws);              \
    break;
    CONV_T(2, 4)
    CONV_T(1, 4)
    CONV_T(2, 2)
    CONV_T(1, 2)
    CONV_T(2, 1)
    default: conv_fwd_t<1, 1>(s, x, w, bias, y, M, H, W, Ci, Co, relu, out_f32, x2, C1, p.splits, p.s_steps, ws); break;
#undef CONV_T
  }
  return hipGetLastError() == hipSuccess ? CISOR_OK : CISOR_E_DEVICE;
}

// Partial weight (and, with bpart, bias) gradients of one layer into at most
// max_splits partials of 9 Co Ci (Co) elements; returns the number written.
// One block per CU over all channel pairs, and tasks of as many rows as still
// give every wave one: longer tasks read less halo, more of them keep the
// CUs busy.
constexpr int WG_BLOCKS = 256;
static int conv_wgrad(hipStream_t s, const bf16_t *x, const bf16_t *dy, float *part, float *bpart, int B, int H,
                      int W, int Ci, int Co, int max_splits, const bf16_t *x2 = nullptr, int C1 = 0) {
  WgArgs a{};
  a.x = x, a.dy = dy, a.x2 = x2, a.part = part, a.bpart = bpart;
  a.H = H, a.W = W, a.Ci = Ci, a.Co = Co, a.C1 = C1;
  a.strips = (W + 15) / 16;
  const int pairs = (Ci / 32) * (Co / 32);
  int splits = std::max(1, std::min(max_splits, WG_BLOCKS / pairs));
  for (a.rh = 32; a.rh > 4; a.rh /= 2)
    if ((long long)B * a.strips * ((H + a.rh - 1) / a.rh) >= (long long)splits * WG_WAVES) break;
  a.segs = (H + a.rh - 1) / a.rh;
  a.tasks = B * a.strips * a.segs;
  splits = std::min(splits, (a.tasks + WG_WAVES - 1) / WG_WAVES);
  const bool narrow = (double)H * W * std::max(Ci, Co) < 4294967296.0;
  hipLaunchKernelGGL(narrow ? k_conv3x3_wgrad<unsigned> : k_conv3x3_wgrad<size_t>, dim3(Ci / 32, Co / 32, splits),
                     dim3(64 * WG_WAVES), 0, s, a);
  return splits;
}

// ------------------------------------------------------------------ the network
struct ConvLayer {
  int Ci, Co;
  bool relu;
  size_t woff, boff;   // offsets in the FP32 parameter vector
};

constexpr int GN_BLOCKS = 512;

struct Net {
  int H = 0, W = 0, base = 32, max_batch = 0;
  hipStream_t stream = nullptr;
  std::vector<ConvLayer> L;
  size_t nparams = 0;
  float *params = nullptr, *grads = nullptr, *adam_m = nullptr, *adam_v = nullptr;
  bf16_t *wb = nullptr;      // bf16 copy of the parameter vector (weights used by the kernels)
  bf16_t *wt = nullptr;      // flipped/transposed weights, at the parameter vector's offsets
  float *wg_part = nullptr;  // weight-gradient split partials
  size_t wg_part_elems = 0;
  float *kws = nullptr;      // split-K partials of the forward convolutions
  size_t kws_elems = 0;
  long long adam_t = 0;
  // activations (bf16, NHWC) and gradients, allocated for max_batch
  std::vector<bf16_t *> act, gact;
  std::vector<size_t> act_elems;
  float *out = nullptr;      // head output, fp32 [B][H][W][32]
  double *loss_b = nullptr, *loss_part = nullptr;   // per-sample loss, partial norms of k_rel_l2_part
  double *gn_part = nullptr; // gradient-norm partials [GN_BLOCKS]
  float *gscale = nullptr;   // clipping factor applied by Adam
  std::vector<void *> allocs;
};

// activation slots
enum {
  A_X0, A_E1A, A_E1B, A_P1, A_E2A, A_E2B, A_P2, A_E3A, A_E3B, A_P3, A_BA, A_BB, A_D3A, A_D3B, A_D2A, A_D2B, A_D1A,
  A_D1B, A_COUNT
};
// gradients: the same slots, the decoder inputs' [skip | upsampled] and the head's output
enum { G_C3 = A_COUNT, G_C2, G_C1, G_OUT, G_COUNT };

template <typename T> static int nn_alloc(Net &n, T *&p, size_t elems) {
  void *q = nullptr;
  if (hipMalloc(&q, std::max<size_t>(elems * sizeof(T), 16)) != hipSuccess) return CISOR_E_NOMEM;
  n.allocs.push_back(q);
  p = (T *)q;
  return CISOR_OK;
}

static int net_build(Net &n) {
  const int c1 = n.base, c2 = 2 * n.base, c3 = 4 * n.base, c4 = 8 * n.base;
  auto add = [&](int ci, int co, bool relu) { n.L.push_back({ci, co, relu, 0, 0}); };
  add(32, c1, true); add(c1, c1, true);          // enc1
  add(c1, c2, true); add(c2, c2, true);          // enc2
  add(c2, c3, true); add(c3, c3, true);          // enc3
  add(c3, c4, true); add(c4, c4, true);          // bottleneck
  add(c3 + c4, c3, true); add(c3, c3, true);     // dec3
  add(c2 + c3, c2, true); add(c2, c2, true);     // dec2
  add(c1 + c2, c1, true); add(c1, c1, true);     // dec1
  add(c1, 32, false);                            // head (2 of 32 outputs used)
  size_t off = 0;
  for (auto &l : n.L) {
    l.woff = off;
    off += (size_t)9 * l.Ci * l.Co;
    l.boff = off;
    off += l.Co;
  }
  n.nparams = off;
  const size_t B = n.max_batch, P1 = (size_t)n.H * n.W, P2 = P1 / 4, P3 = P1 / 16, P4 = P1 / 64;
  const size_t sizes[G_COUNT] = {B * P1 * 32, B * P1 * c1, B * P1 * c1, B * P2 * c1, B * P2 * c2, B * P2 * c2,
                                 B * P3 * c2, B * P3 * c3, B * P3 * c3, B * P4 * c3, B * P4 * c4, B * P4 * c4,
                                 B * P3 * c3, B * P3 * c3, B * P2 * c2, B * P2 * c2, B * P1 * c1, B * P1 * c1,
                                 B * P3 * (c3 + c4), B * P2 * (c2 + c3), B * P1 * (c1 + c2), B * P1 * 32};
  n.act.assign(A_COUNT, nullptr);
  n.gact.assign(G_COUNT, nullptr);
  n.act_elems.assign(sizes, sizes + A_COUNT);
  int rc;
  for (int i = 0; i < G_COUNT; ++i) {
    if (i < A_COUNT && (rc = nn_alloc(n, n.act[i], sizes[i]))) return rc;
    if ((rc = nn_alloc(n, n.gact[i], sizes[i]))) return rc;
  }
  // split-K workspace: the largest need of any forward layer at max_batch
  const int lev[15] = {1, 1, 2, 2, 4, 4, 8, 8, 4, 4, 2, 2, 1, 1, 1};
  for (int l = 0; l < (int)n.L.size(); ++l) {
    const int M = (int)(B * P1) / (lev[l] * lev[l]);
    ConvPlan p;
    if (conv_plan(M, n.L[l].Ci, n.L[l].Co, 0, 0, true, p) && p.splits > 1)
      n.kws_elems = std::max(n.kws_elems, (size_t)p.splits * M * n.L[l].Co);
  }
  if (n.kws_elems && (rc = nn_alloc(n, n.kws, n.kws_elems))) return rc;
  if ((rc = nn_alloc(n, n.params, n.nparams)) || (rc = nn_alloc(n, n.grads, n.nparams)) ||
      (rc = nn_alloc(n, n.adam_m, n.nparams)) || (rc = nn_alloc(n, n.adam_v, n.nparams)) ||
      (rc = nn_alloc(n, n.wb, n.nparams)) || (rc = nn_alloc(n, n.out, B * P1 * 32)) ||
      (rc = nn_alloc(n, n.loss_b, B)) || (rc = nn_alloc(n, n.loss_part, 2 * LOSS_PARTS * B)) || (rc = nn_alloc(n, n.gn_part, GN_BLOCKS)) ||
      (rc = nn_alloc(n, n.gscale, 1)))
    return rc;
  // split partials of every layer's weight and bias gradients at once: a
  // layer has at most WG_BLOCKS blocks of 9 x 32 x 32 weights
  for (auto &l : n.L) {
    const size_t pairs = (size_t)(l.Ci / 32) * (l.Co / 32), splits = std::max<size_t>(1, WG_BLOCKS / pairs);
    n.wg_part_elems += splits * ((size_t)9 * l.Ci * l.Co + l.Co);
  }
  if ((rc = nn_alloc(n, n.wt, n.nparams)) || (rc = nn_alloc(n, n.wg_part, n.wg_part_elems))) return rc;
  return CISOR_OK;
}

static const bf16_t *wptr(const Net &n, int l) { return n.wb + n.L[l].woff; }
static const float *bptr(const Net &n, int l) { return n.params + n.L[l].boff; }

// The decoder convolutions read the skip tensor and the low-resolution tensor
// in place.  fused (inference): the network input and the pooled tensors are
// formed inside the convolutions that read them too; otherwise they are
// materialised, as the weight gradients of training read them.
static int net_forward(Net &n, const float *f, const cf *uin, const cf *ub, int B, bool fused, cf *u0 = nullptr) {
  hipStream_t s = n.stream;
  const int H = n.H, W = n.W;
  const int c1 = n.base, c2 = 2 * n.base, c3 = 4 * n.base, c4 = 8 * n.base;
  auto &A = n.act;
  const size_t N = (size_t)H * W;
  int rc = 0;
  TileIO io;
  io.f = f;
  io.uin = uin;
  io.ub = ub;
  io.u0 = u0;
#define CONV(l, in, outp, h, w)                                                                                \
  if ((rc = conv_fwd(s, in, wptr(n, l), bptr(n, l), outp, B, h, w, n.L[l].Ci, n.L[l].Co, n.L[l].relu, false, 0,  \
                     nullptr, 0, n.kws, n.kws_elems)))                                                             \
    return rc;
  // fused: the network input formed and the 2x2 pooling done inside the
  // convolutions that read them (the training path keeps them materialised)
#define FUSED_IN(l, tin, in, outp, h, w)                                                                          \
  (fused && conv_fwd_tiled(s, in, wptr(n, l), bptr(n, l), outp, B, h, w, n.L[l].Ci, n.L[l].Co, n.L[l].relu,       \
                           TOUT_BF16, tin, nullptr, 0, io))
  if (!FUSED_IN(0, TIN_NET, nullptr, A[A_E1A], H, W)) {
    hipLaunchKernelGGL(k_net_input, grid1(B * N), dim3(256), 0, s, f, uin, ub, A[A_X0], B, (int)N);
    CONV(0, A[A_X0], A[A_E1A], H, W);
  }
  CONV(1, A[A_E1A], A[A_E1B], H, W);
  if (!FUSED_IN(2, TIN_POOL, A[A_E1B], A[A_E2A], H / 2, W / 2)) {
    hipLaunchKernelGGL(k_avgpool, grid1(n.act_elems[A_P1] / 8), dim3(256), 0, s, A[A_E1B], A[A_P1], B, H, W, c1);
    CONV(2, A[A_P1], A[A_E2A], H / 2, W / 2);
  }
  CONV(3, A[A_E2A], A[A_E2B], H / 2, W / 2);
  if (!FUSED_IN(4, TIN_POOL, A[A_E2B], A[A_E3A], H / 4, W / 4)) {
    hipLaunchKernelGGL(k_avgpool, grid1(n.act_elems[A_P2] / 8), dim3(256), 0, s, A[A_E2B], A[A_P2], B, H / 2, W / 2,
                       c2);
    CONV(4, A[A_P2], A[A_E3A], H / 4, W / 4);
  }
  CONV(5, A[A_E3A], A[A_E3B], H / 4, W / 4);
  if (!FUSED_IN(6, TIN_POOL, A[A_E3B], A[A_BA], H / 8, W / 8)) {
    hipLaunchKernelGGL(k_avgpool, grid1(n.act_elems[A_P3] / 8), dim3(256), 0, s, A[A_E3B], A[A_P3], B, H / 4, W / 4,
                       c3);
    CONV(6, A[A_P3], A[A_BA], H / 8, W / 8);
  }
#undef FUSED_IN
  CONV(7, A[A_BA], A[A_BB], H / 8, W / 8);
  if ((rc = conv_fwd(s, A[A_E3B], wptr(n, 8), bptr(n, 8), A[A_D3A], B, H / 4, W / 4, n.L[8].Ci, n.L[8].Co, n.L[8].relu,
                     false, 0, A[A_BB], c3, n.kws, n.kws_elems)))
    return rc;
  CONV(9, A[A_D3A], A[A_D3B], H / 4, W / 4);
  if ((rc = conv_fwd(s, A[A_E2B], wptr(n, 10), bptr(n, 10), A[A_D2A], B, H / 2, W / 2, n.L[10].Ci, n.L[10].Co, n.L[10].relu,
                     false, 0, A[A_D3B], c2, n.kws, n.kws_elems)))
    return rc;
  CONV(11, A[A_D2A], A[A_D2B], H / 2, W / 2);
  if ((rc = conv_fwd(s, A[A_E1B], wptr(n, 12), bptr(n, 12), A[A_D1A], B, H, W, n.L[12].Ci, n.L[12].Co, n.L[12].relu,
                     false, 0, A[A_D2B], c1, n.kws, n.kws_elems)))
    return rc;
  CONV(13, A[A_D1A], A[A_D1B], H, W);
#undef CONV
  // head: with u0 set (inference), fused, u0 = u_in + (y0 + i y1) written by
  // the convolution itself; else the FP32 output, then u0 from it
  if (!(fused && u0 &&
        conv_fwd_tiled(s, A[A_D1B], wptr(n, 14), bptr(n, 14), nullptr, B, H, W, n.L[14].Ci, n.L[14].Co,
                       n.L[14].relu, TOUT_U0, TIN_X, nullptr, 0, io))) {
    if ((rc = conv_fwd(s, A[A_D1B], wptr(n, 14), bptr(n, 14), n.out, B, H, W, n.L[14].Ci, n.L[14].Co, false, true, 0,
                       nullptr, 0, n.kws, n.kws_elems)))
      return rc;
    if (u0)
      hipLaunchKernelGGL(k_net_output, grid1((size_t)B * N), dim3(256), 0, s, n.out, uin, u0, (size_t)B * N);
  }
  return hipGetLastError() == hipSuccess ? CISOR_OK : CISOR_E_DEVICE;
}

// Data gradient of layer l: gx = conv(gy, w') with w' the flipped weights,
// and, with mask, the ReLU of the layer that produced its input.
static int layer_dgrad(Net &n, int l, const bf16_t *gy, bf16_t *gx, const bf16_t *mask, int B, int h, int w) {
  const ConvLayer &L = n.L[l];
  TileIO io;
  io.mask = mask;
  if (conv_fwd_tiled(n.stream, gy, n.wt + L.woff, nullptr, gx, B, h, w, L.Co, L.Ci, false,
                     mask ? TOUT_MASK : TOUT_BF16, TIN_X, nullptr, 0, io))
    return hipGetLastError() == hipSuccess ? CISOR_OK : CISOR_E_DEVICE;
  if (int rc = conv_fwd(n.stream, gy, n.wt + L.woff, nullptr, gx, B, h, w, L.Co, L.Ci, false, false)) return rc;
  const size_t nx = (size_t)B * h * w * L.Ci;
  if (mask) hipLaunchKernelGGL(k_relu_bwd, grid1(nx), dim3(256), 0, n.stream, gx, mask, gx, nx);
  return CISOR_OK;
}

// Every buffer named G[...] of a convolution's output holds the gradient
// before that convolution's ReLU: the kernels that produce it apply the mask.
static int net_backward(Net &n, int B) {
  hipStream_t s = n.stream;
  const int H = n.H, W = n.W;
  const int c1 = n.base, c2 = 2 * n.base, c3 = 4 * n.base, c4 = 8 * n.base;
  auto &A = n.act;
  auto &G = n.gact;
  FlipList flip;
  for (auto &l : n.L) flip.l[flip.count++] = {(unsigned)l.woff, l.Ci, l.Co};
  hipLaunchKernelGGL(k_flip_transpose, dim3(64, flip.count), dim3(256), 0, s, n.wb, n.wt, flip);
  RedList red;
  float *part = n.wg_part;
  int rc = CISOR_OK;
  // weight and bias gradients of layer l (input xin, or [xin (C1) | up2(xup)])
  auto wgrad = [&](int l, const bf16_t *xin, const bf16_t *gy, int h, int w, const bf16_t *xup = nullptr, int C1 = 0) {
    const ConvLayer &L = n.L[l];
    const size_t nw = (size_t)9 * L.Ci * L.Co;
    const int most = std::max(1, WG_BLOCKS / ((L.Ci / 32) * (L.Co / 32)));
    float *bpart = part + (size_t)most * nw;
    const int splits = conv_wgrad(s, xin, gy, part, bpart, B, h, w, L.Ci, L.Co, most, xup, C1);
    red.add(part, n.grads + L.woff, nw, splits);
    red.add(bpart, n.grads + L.boff, L.Co, splits);
    part = bpart + (size_t)most * L.Co;
  };
  auto dgrad = [&](int l, const bf16_t *gy, bf16_t *gx, const bf16_t *mask, int h, int w) {
    if (rc == CISOR_OK) rc = layer_dgrad(n, l, gy, gx, mask, B, h, w);
  };
  // a decoder level (layers l + 1 and l): from G[b] to the gradient gc of its input
  auto decoder = [&](int l, int b, int a, const bf16_t *skip, int Cs, const bf16_t *low, bf16_t *gc, int h, int w) {
    wgrad(l + 1, A[a], G[b], h, w);
    dgrad(l + 1, G[b], G[a], A[a], h, w);
    wgrad(l, skip, G[a], h, w, low, Cs);
    dgrad(l, G[a], gc, nullptr, h, w);
  };
  auto up_bwd = [&](const bf16_t *gc, int slot, int h, int w, int C, int Ct) {   // h, w: the lower level's size
    hipLaunchKernelGGL(k_upsample_bwd, grid1((size_t)B * h * w * C / 8), dim3(256), 0, s, gc, A[slot], G[slot], B, h, w,
                       C, Ct);
  };
  auto pool_bwd = [&](const bf16_t *gp, const bf16_t *gc, int slot, int h, int w, int C, int Ct) {
    hipLaunchKernelGGL(k_pool_skip_bwd, grid1((size_t)B * h * w * C / 8), dim3(256), 0, s, gp, gc, A[slot], G[slot], B,
                       h, w, C, Ct);
  };
  wgrad(14, A[A_D1B], G[G_OUT], H, W);
  dgrad(14, G[G_OUT], G[A_D1B], A[A_D1B], H, W);
  decoder(12, A_D1B, A_D1A, A[A_E1B], c1, A[A_D2B], G[G_C1], H, W);
  up_bwd(G[G_C1], A_D2B, H / 2, W / 2, c2, c1 + c2);
  decoder(10, A_D2B, A_D2A, A[A_E2B], c2, A[A_D3B], G[G_C2], H / 2, W / 2);
  up_bwd(G[G_C2], A_D3B, H / 4, W / 4, c3, c2 + c3);
  decoder(8, A_D3B, A_D3A, A[A_E3B], c3, A[A_BB], G[G_C3], H / 4, W / 4);
  up_bwd(G[G_C3], A_BB, H / 8, W / 8, c4, c3 + c4);
  // an encoder level (layers l + 1 and l) from G[b] to the gradient of its pooled input
  auto encoder = [&](int l, int b, int a, int in, int h, int w) {
    wgrad(l + 1, A[a], G[b], h, w);
    dgrad(l + 1, G[b], G[a], A[a], h, w);
    wgrad(l, A[in], G[a], h, w);
    if (l) dgrad(l, G[a], G[in], nullptr, h, w);
  };
  encoder(6, A_BB, A_BA, A_P3, H / 8, W / 8);
  pool_bwd(G[A_P3], G[G_C3], A_E3B, H / 4, W / 4, c3, c3 + c4);
  encoder(4, A_E3B, A_E3A, A_P2, H / 4, W / 4);
  pool_bwd(G[A_P2], G[G_C2], A_E2B, H / 2, W / 2, c2, c2 + c3);
  encoder(2, A_E2B, A_E2A, A_P1, H / 2, W / 2);
  pool_bwd(G[A_P1], G[G_C1], A_E1B, H, W, c1, c1 + c2);
  encoder(0, A_E1B, A_E1A, A_X0, H, W);
  if (rc) return rc;
  hipLaunchKernelGGL(k_sum_splits, dim3(red.blocks), dim3(256), 0, s, red);
  return hipGetLastError() == hipSuccess ? CISOR_OK : CISOR_E_DEVICE;
}

}  // namespace cisor

using namespace cisor;

struct cisor_net {
  Net n;
};

extern "C" {

int cisor_net_create(int height, int width, int base, int max_batch, unsigned long long seed, void *stream,
                     cisor_net **out) {
  if (!out || height < 16 || width < 16 || height % 16 || width % 16 || base < 32 || base % 32 || max_batch < 1 ||
      ((size_t)height * width * max_batch) % 8192)
    return CISOR_E_ARG;
  *out = nullptr;
  cisor_net *h = new (std::nothrow) cisor_net();
  if (!h) return CISOR_E_NOMEM;
  Net &n = h->n;
  n.H = height;
  n.W = width;
  n.base = base;
  n.max_batch = max_batch;
  n.stream = (hipStream_t)stream;
  int rc = net_build(n);
  if (rc) {
    for (void *p : n.allocs) (void)hipFree(p);
    delete h;
    return rc;
  }
  // He-normal initialisation (seeded), zero biases; padded input channels of
  // the first layer and padded outputs of the head stay zero.
  std::vector<float> p(n.nparams, 0.0f);
  std::mt19937_64 gen(seed);
  for (size_t l = 0; l < n.L.size(); ++l) {
    const ConvLayer &L = n.L[l];
    const int ci_used = (l == 0) ? 5 : L.Ci;
    const int co_used = (l + 1 == n.L.size()) ? 2 : L.Co;
    std::normal_distribution<float> nd(0.0f, std::sqrt(2.0f / (9.0f * ci_used)) * (l + 1 == n.L.size() ? 0.1f : 1.0f));
    for (int tap = 0; tap < 9; ++tap)
      for (int co = 0; co < co_used; ++co)
        for (int ci = 0; ci < ci_used; ++ci) p[L.woff + ((size_t)tap * L.Co + co) * L.Ci + ci] = nd(gen);
  }
  if (hipMemcpy(n.params, p.data(), sizeof(float) * n.nparams, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemset(n.adam_m, 0, sizeof(float) * n.nparams) != hipSuccess ||
      hipMemset(n.adam_v, 0, sizeof(float) * n.nparams) != hipSuccess) {
    for (void *q : n.allocs) (void)hipFree(q);
    delete h;
    return CISOR_E_DEVICE;
  }
  hipLaunchKernelGGL(k_to_bf16, grid1(n.nparams), dim3(256), 0, n.stream, n.params, n.wb, n.nparams);
  *out = h;
  return hipGetLastError() == hipSuccess ? CISOR_OK : CISOR_E_DEVICE;
}

int cisor_net_destroy(cisor_net *h) {
  if (!h) return CISOR_E_ARG;
  (void)hipStreamSynchronize(h->n.stream);
  for (void *p : h->n.allocs) (void)hipFree(p);
  delete h;
  return CISOR_OK;
}

int cisor_net_set_stream(cisor_net *h, void *stream) {
  if (!h) return CISOR_E_ARG;
  h->n.stream = (hipStream_t)stream;
  return CISOR_OK;
}

int cisor_net_num_params(const cisor_net *h, long long *n) {
  if (!h || !n) return CISOR_E_ARG;
  *n = (long long)h->n.nparams;
  return CISOR_OK;
}

int cisor_net_get_params(cisor_net *h, float *params) {
  if (!h || !params) return CISOR_E_ARG;
  CISOR_HIP_CHECK(hipMemcpyAsync(params, h->n.params, sizeof(float) * h->n.nparams, hipMemcpyDeviceToDevice,
                                 h->n.stream));
  return CISOR_OK;
}

int cisor_net_set_params(cisor_net *h, const float *params) {
  if (!h || !params) return CISOR_E_ARG;
  Net &n = h->n;
  CISOR_HIP_CHECK(hipMemcpyAsync(n.params, params, sizeof(float) * n.nparams, hipMemcpyDeviceToDevice, n.stream));
  hipLaunchKernelGGL(k_to_bf16, grid1(n.nparams), dim3(256), 0, n.stream, n.params, n.wb, n.nparams);
  n.adam_t = 0;
  CISOR_HIP_CHECK(hipMemsetAsync(n.adam_m, 0, sizeof(float) * n.nparams, n.stream));
  CISOR_HIP_CHECK(hipMemsetAsync(n.adam_v, 0, sizeof(float) * n.nparams, n.stream));
  return CISOR_OK;
}

int cisor_net_forward(cisor_net *h, const float *f, const void *u_in, const void *u_born, void *u0, int batch) {
  if (!h || !f || !u_in || !u0 || batch < 1 || batch > h->n.max_batch) return CISOR_E_ARG;
  Net &n = h->n;
  if (((size_t)batch * n.H * n.W) % 8192) return CISOR_E_ARG;
  return net_forward(n, f, (const cf *)u_in, (const cf *)u_born, batch, true, (cf *)u0);
}

int cisor_net_loss_grad(cisor_net *h, const float *f, const void *u_in, const void *u_born, const void *u, int batch,
                        double *loss, float *grad_out) {
  if (!h || !f || !u_in || !u || batch < 1 || batch > h->n.max_batch) return CISOR_E_ARG;
  Net &n = h->n;
  if (((size_t)batch * n.H * n.W) % 8192) return CISOR_E_ARG;
  int rc = net_forward(n, f, (const cf *)u_in, (const cf *)u_born, batch, false);
  if (rc) return rc;
  const int N = n.H * n.W;
  hipLaunchKernelGGL(k_rel_l2_part, dim3(LOSS_PARTS, batch), dim3(256), 0, n.stream, n.out, (const cf *)u_in,
                     (const cf *)u, n.loss_part, N);
  hipLaunchKernelGGL(k_rel_l2, dim3(64, batch), dim3(256), 0, n.stream, n.out, (const cf *)u_in, (const cf *)u,
                     (const double *)n.loss_part, n.gact[G_OUT], n.loss_b, N, batch);
  if ((rc = net_backward(n, batch))) return rc;
  if (loss) {
    std::vector<double> lb(batch);
    CISOR_HIP_CHECK(hipMemcpyAsync(lb.data(), n.loss_b, sizeof(double) * batch, hipMemcpyDeviceToHost, n.stream));
    CISOR_HIP_CHECK(hipStreamSynchronize(n.stream));
    double s = 0;
    for (double v : lb) s += v;
    *loss = s / batch;
  }
  if (grad_out)
    CISOR_HIP_CHECK(hipMemcpyAsync(grad_out, n.grads, sizeof(float) * n.nparams, hipMemcpyDeviceToDevice, n.stream));
  return CISOR_OK;
}

int cisor_net_train_step(cisor_net *h, const float *f, const void *u_in, const void *u_born, const void *u, int batch,
                         double lr, double clip, double *loss) {
  if (!h || !(lr > 0) || !std::isfinite(clip)) return CISOR_E_ARG;
  int rc = cisor_net_loss_grad(h, f, u_in, u_born, u, batch, loss, nullptr);
  if (rc) return rc;
  Net &n = h->n;
  hipLaunchKernelGGL(k_sqnorm_part, dim3(GN_BLOCKS), dim3(256), 0, n.stream, n.grads, n.nparams, n.gn_part);
  hipLaunchKernelGGL(k_clip_factor, dim3(1), dim3(64), 0, n.stream, n.gn_part, GN_BLOCKS, clip, n.gscale);
  n.adam_t += 1;
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.0f - std::pow(b1, (float)n.adam_t), c2 = 1.0f - std::pow(b2, (float)n.adam_t);
  hipLaunchKernelGGL(k_adam, grid1(n.nparams), dim3(256), 0, n.stream, n.params, n.grads, n.gscale, n.adam_m,
                     n.adam_v, n.wb, n.nparams, (float)lr, b1, b2, 1e-8f, c1, c2);
  return hipGetLastError() == hipSuccess ? CISOR_OK : CISOR_E_DEVICE;
}

// Single-layer hooks (BF16 operands, FP32 accumulation) for kernel-level tests.
int cisor_nn_conv3x3(const void *x, const void *w, const float *bias, void *y, int B, int H, int W, int Ci, int Co,
                     int relu, int out_f32, int tile, void *stream) {
  if (!x || !w || !y || B < 1 || H < 1 || W < 1) return CISOR_E_ARG;
  return conv_fwd((hipStream_t)stream, (const bf16_t *)x, (const bf16_t *)w, bias, y, B, H, W, Ci, Co, relu != 0,
                  out_f32 != 0, tile);
}

int cisor_nn_conv3x3_ex(const void *x, const void *x2, int C1, const void *w, const float *bias, void *y, int B,
                        int H, int W, int Ci, int Co, int relu, int out_f32, int tile, int splits, float *workspace,
                        size_t workspace_elems, void *stream) {
  if (!x || !w || !y || B < 1 || H < 1 || W < 1 || splits < 1) return CISOR_E_ARG;
  return conv_fwd((hipStream_t)stream, (const bf16_t *)x, (const bf16_t *)w, bias, y, B, H, W, Ci, Co, relu != 0,
                  out_f32 != 0, tile, (const bf16_t *)x2, x2 ? C1 : 0, workspace, workspace_elems, splits);
}

int cisor_nn_conv3x3_wgrad(const void *x, const void *dy, float *dw, float *scratch, int B, int H, int W, int Ci,
                           int Co, int max_splits, void *stream) {
  if (!x || !dy || !dw || !scratch || Ci % 32 || Co % 32 || max_splits < 1) return CISOR_E_ARG;
  const int splits = conv_wgrad((hipStream_t)stream, (const bf16_t *)x, (const bf16_t *)dy, scratch, nullptr, B, H, W,
                                Ci, Co, max_splits);
  RedList l;
  l.add(scratch, dw, (size_t)9 * Co * Ci, splits);
  hipLaunchKernelGGL(k_sum_splits, dim3(l.blocks), dim3(256), 0, (hipStream_t)stream, l);
  return hipGetLastError() == hipSuccess ? CISOR_OK : CISOR_E_DEVICE;
}

}  // extern "C"
