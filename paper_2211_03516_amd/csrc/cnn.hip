// Learned initialiser: a small 3x3 convolutional network trained and run on
// MFMA matrix cores (gfx950 v_mfma_f32_32x32x16_bf16).
//
// Every convolution is one GEMM over the im2col matrix of its input:
//   forward          z[p][co]     = sum_kc col(a)[p][kc]   W[co][kc]
//   data gradient    da[p][ci]    = sum_kc col(g)[p][kc]   Wflip[ci][kc]
//   weight gradient  dW^T[kc][co] = sum_p  col(a)[p][kc]   g[p][co]
// with p a pixel of the batch, kc = (tap, channel) and Wflip the kernel
// turned by 180 degrees with input and output channels swapped (the
// transposed convolution as a convolution).  Activations are NHWC BF16 with
// channels padded to a multiple of 8.  No im2col matrix is written to memory:
// a workgroup stages an image tile with its one-pixel border in LDS once and
// reads it at the nine shifts.  The weight gradient's workgroups each add
// up their tiles, and a second kernel adds their FP32 sums in a fixed order,
// so training is deterministic.

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <type_traits>
#include <vector>

#include "vam_cnn.h"
#include "vam_internal.h"

namespace vam {
namespace cnn {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr uint64_t kCnnMagic = 0x56414d434e4e3031ull;  // "VAMCNN01"
constexpr int kMaxChannels = 64;
constexpr int BK = 32;          // rows of packed weights are padded to multiples of this
constexpr int kMaxSplits = 256;  // workgroups of a weight gradient: one a CU

__device__ inline uint16_t f2bf(float f) {  // round to nearest even
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
// Two values as a BF16 pair, to nearest even (one v_cvt_pk_bf16_f32).
__device__ inline uint32_t f2bf_pair(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}
__device__ inline float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ inline bool bf_positive(uint16_t h) { return h != 0 && !(h & 0x8000u); }

enum Epi { EPI_RELU_BF16 = 0, EPI_OUT_F32 = 1, EPI_MASK_BF16 = 2 };

struct ConvArgs {
  const uint16_t* X;       // NHWC [pixels][CP]
  int H, W;                // image size
  int tiles_x, tiles_y, tiles;  // 16 x 16 tiles of an image, and of the batch
  const uint16_t* B;       // packed weights (weight_place)
  int rows, kp;            // output channels (padded), im2col entries (padded)
  void* C;                 // BF16 [pixels][rows], or FP32 [pixels] (EPI_OUT_F32)
  const float* bias;       // EPI_RELU_BF16, EPI_OUT_F32
  const uint16_t* mask;    // EPI_MASK_BF16: BF16 [pixels][rows]
  const float* x;          // EPI_OUT_F32: network input [n][2][H][W], or NULL for z itself
  float s1;
};

constexpr int kTile = 16, kTileP = kTile + 2;  // tile edge, with its border

// Channel of a 32-channel block in MFMA row m: register r of lane l of an
// accumulator is row 8 (r / 4) + 4 (l / 32) + r % 4, and holds channel 16 (r / 8)
// + 8 (l / 32) + r % 8 so.
__host__ __device__ constexpr int row_channel(int m) {
  const int r = 4 * (m / 8) + m % 4, half = m / 4 % 2;
  return 16 * (r / 8) + 8 * half + r % 8;
}

// Place of weight (channel co, im2col entry k) in the packed array of a layer
// whose rows have kp entries: for every block of 32 channels and every 16
// entries, the 64 lanes' 8 entries one after the other.
__host__ __device__ inline int weight_place(int co, int k, int kp) {
  const int c = co % 32, r = 8 * (c / 16) + c % 8, half = c / 8 % 2;  // row_channel's inverse
  const int m = 8 * (r / 4) + 4 * half + r % 4, lane = m + 32 * (k / 8 % 2);
  return ((co / 32 * (kp / 16) + k / 16) * 64 + lane) * 8 + k % 8;
}

// Element offset, in a staged tile of `pitch` elements a pixel, of the k-th
// entry of a pixel's im2col row of CP channels a tap.
template <int CP, int PITCH>
constexpr int col_offset(int k) {
  const int tap = k / CP, c = k % CP;
  return (tap / 3 * kTileP + tap % 3) * PITCH + c;
}

// out = epilogue(sum_k W[co][k] col(X)[p][k]) for 16 x 16 pixel tiles, eight
// waves per workgroup, NB blocks of 32 output channels.
//
// What bounds it: at 64 channels a layer moves 2 x 33 MB a batch of 16 x 128^2
// (13 us at the rate of a large copy) and needs 16 us of matrix work at the
// rate of a large product, so both have to overlap and neither may be repeated.
//  * A workgroup keeps its waves' share of the packed weights in registers (a
//    wave has one block of 32 channels: 144 registers at 64 channels) and goes
//    over tiles, so the weights are read once per workgroup.
//  * A tile with its border is staged once (18 x 18 pixels) and read at nine
//    shifts: every LDS address is one base plus a constant.  Pixels lie an odd
//    number of 16-byte units apart, so 16 lanes read 16 different bank groups.
//  * The next tile's loads are issued before the current tile's products and
//    written to the other LDS buffer after them: one barrier a tile.
//  * Weights are the MFMA's first operand, their rows in the order row_channel,
//    and pixels its second: a lane holds two runs of eight channels of one
//    pixel, so outputs (and masks) move 16 bytes at a time.
//  * Packed weights lie in the order the waves load them (weight_place).
//  * The LDS reads run four ahead of the products.
// The products of an output are added in ascending k, 16 at a time, from
// zero: the same bits as any other tiling of that order.
// Measured at 16 x 128^2, 64 to 64 channels: 25 us (27 with a mask); the general
// matrix kernel before, which gathered the nine shifts from memory for every
// 128 pixels and read all weights with them, 46 us (53).  At 64 images 82 us, 3.3
// TB/s.  All weights in registers spilled (44 us).
template <int CP, int NB, int EPI>
__global__ __launch_bounds__(512) void k_conv(ConvArgs g) {
  constexpr int U = CP / 8, PITCH = (U | 1) * 8, PIX = kTileP * kTileP;
  constexpr int KS = (9 * CP + 15) / 16, CHUNKS = PIX * U, PER = (CHUNKS + 511) / 512;
  constexpr int MB = NB == 2 ? 2 : 1;  // 32-pixel blocks (two tile rows) of a wave
  // weights of the last KL steps stay in LDS, so that everything fits 256
  // registers (two waves a SIMD) without spilling
  constexpr int KL = NB == 2 && KS > 28 ? KS - 28 : 0, KR = KS - KL;
  __shared__ __attribute__((aligned(16))) uint16_t tile[2][PIX * PITCH];
  __shared__ __attribute__((aligned(16))) uint16_t wl[(KL ? KL : 1) * NB * 64 * 8];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane >> 5;
  const int nb = NB == 2 ? wave & 1 : 0, mg = NB == 2 ? wave >> 1 : wave;
  bf16x8 w[KR];
#pragma unroll
  for (int s = 0; s < KR; ++s) w[s] = *(const bf16x8*)(g.B + ((nb * (g.kp / 16) + s) * 64 + lane) * 8);
  __shared__ __attribute__((aligned(32))) float bias[kMaxChannels];
  if (EPI != EPI_MASK_BF16 && threadIdx.x < kMaxChannels) bias[threadIdx.x] = g.bias[threadIdx.x];
  for (int i = threadIdx.x; i < KL * NB * 64; i += 512) {
    const int s = i / (NB * 64), rest = i % (NB * 64);
    *(uint4*)(wl + i * 8) = *(const uint4*)(g.B + ((rest / 64 * (g.kp / 16) + KR + s) * 64 + rest % 64) * 8);
  }
  // lane's pixel in block b: tile row 2 (mg MB + b) + (lane / 16) % 2, column lane % 16.
  // The upper half of the wave takes the second 8 of a step's 16 entries:
  // the next channels, the next tap, or the next row of taps.
  const int row0 = 2 * mg * MB + ((lane >> 4) & 1), col = lane & 15;
  const int base = (row0 * kTileP + col) * PITCH;
  const int at_chan = base + half * 8, at_tap = base + half * (PITCH - (CP - 8)),
            at_row = base + half * ((kTileP - 2) * PITCH - (CP - 8));
  uint4 r[PER];
  auto origin = [&](int t, int& img, int& y0, int& x0) {
    img = t / (g.tiles_x * g.tiles_y);
    const int rest = t - img * (g.tiles_x * g.tiles_y), ty = rest / g.tiles_x;
    y0 = ty * kTile;
    x0 = (rest - ty * g.tiles_x) * kTile;
  };
  // buffer loads: an offset past the image reads zeros, the border's value
  const uint32_t image_bytes = (uint32_t)g.H * g.W * CP * 2;
  auto fetch = [&](int t) {
    int img, y0, x0;
    origin(t, img, y0, x0);
    const __amdgpu_buffer_rsrc_t X = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(g.X + (int64_t)img * g.H * g.W * CP), (short)0, image_bytes, 0x00020000);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = k * 512 + threadIdx.x, px = i / U, ch = i - px * U;
      const int y = y0 + px / kTileP - 1, x = x0 + px % kTileP - 1;
      const bool inside = (unsigned)y < (unsigned)g.H && (unsigned)x < (unsigned)g.W && i < CHUNKS;
      const auto v = __builtin_amdgcn_raw_buffer_load_b128(
          X, inside ? (y * g.W + x) * (CP * 2) + ch * 16 : (int)image_bytes, 0, 0);
      __builtin_memcpy(&r[k], &v, 16);
    }
  };
  auto stage = [&](uint16_t* to) {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = k * 512 + threadIdx.x, px = i / U, ch = i - px * U;
      if (i < CHUNKS) *(uint4*)(to + px * PITCH + ch * 8) = r[k];
    }
  };
  int t = blockIdx.x, cur = 0;
  if (t < g.tiles) {
    fetch(t);
    stage(tile[0]);
  }
  __syncthreads();
  for (; t < g.tiles; t += gridDim.x, cur ^= 1) {
    const bool more = t + (int)gridDim.x < g.tiles;
    if (more) fetch(t + gridDim.x);
    int img, y0, x0;
    origin(t, img, y0, x0);
    // outputs (and masks) of the image as a buffer: lanes outside it, or past
    // the last channel, get an offset past its end, where stores do nothing
    const int out_bytes = g.H * g.W * g.rows * 2;
    int at_out[MB][2];
    uint4 mask[MB][2];  // loaded with the next tile, before any store
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int y = y0 + row0 + 2 * b, x = x0 + col, co = nb * 32 + 16 * j + 8 * half;
        at_out[b][j] = y < g.H && x < g.W && co < g.rows ? ((y * g.W + x) * g.rows + co) * 2 : out_bytes;
        if constexpr (EPI == EPI_MASK_BF16) {
          const __amdgpu_buffer_rsrc_t M = __builtin_amdgcn_make_buffer_rsrc(
              const_cast<uint16_t*>(g.mask + (int64_t)img * g.H * g.W * g.rows), (short)0, out_bytes, 0x00020000);
          const auto v = __builtin_amdgcn_raw_buffer_load_b128(M, at_out[b][j], 0, 0);
          __builtin_memcpy(&mask[b][j], &v, 16);
        }
      }
    const uint16_t* in = tile[cur];
    f32x16 acc[MB];
#pragma unroll
    for (int b = 0; b < MB; ++b)
      for (int i = 0; i < 16; ++i) acc[b][i] = 0.0f;
    auto products = [&](auto first, auto end) {
      constexpr int S0 = decltype(first)::value, S1 = decltype(end)::value, READS = (S1 - S0) * MB + (S0 == KR ? KL : 0);
      constexpr int AHEAD = READS < 4 ? READS : 4;
#pragma unroll
      for (int s = S0; s < S1; ++s) {
        const int lo = 16 * s, hi = lo + 8;
        const int o = col_offset<CP, PITCH>(lo);
        // past the last tap (weights zero) the upper half rereads the lower's and
        // takes zeros (an infinity there would make NaN)
        const bf16x8 ws = s < KR ? w[s < KR ? s : 0] : *(const bf16x8*)(wl + (((s - KR) * NB + nb) * 64 + lane) * 8);
        const int at = hi >= 9 * CP ? base : lo / CP == hi / CP ? at_chan : hi / CP % 3 != 0 ? at_tap : at_row;
#pragma unroll
        for (int b = 0; b < MB; ++b) {
          bf16x8 a = *(const bf16x8*)(in + at + o + b * 2 * kTileP * PITCH);
          if (hi >= 9 * CP && half != 0) a = bf16x8{};
          acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ws, a, acc[b], 0, 0, 0);
        }
      }
      // schedule: AHEAD LDS reads, then a product and a read in turn
      __builtin_amdgcn_sched_group_barrier(0x100, AHEAD, 0);
#pragma unroll
      for (int i = 0; i < READS - AHEAD; ++i) {
        if (S0 != KR || i % 3 != 2) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // KL: three reads, two products
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, AHEAD, 0);
    };
    products(std::integral_constant<int, 0>{}, std::integral_constant<int, KR>{});
    if constexpr (KL > 0) products(std::integral_constant<int, KR>{}, std::integral_constant<int, KS>{});
    // into LDS before this tile's stores are issued: loads and stores complete
    // in order, so waiting for the loads later would wait for the stores too
    if (more) stage(tile[cur ^ 1]);
    if constexpr (EPI == EPI_OUT_F32) {
#pragma unroll
      for (int b = 0; b < MB; ++b) {
        const int y = y0 + row0 + 2 * b, x = x0 + col;
        if (y >= g.H || x >= g.W || half != 0) continue;  // channel 0 is row 0
        const int64_t hw = (int64_t)g.H * g.W, p = img * hw + y * g.W + x;
        const float z = acc[b][0] + bias[0];
        ((float*)g.C)[p] = g.x ? g.x[p + (img + 1) * hw] + z / g.s1 : z;
      }
    } else {
      const __amdgpu_buffer_rsrc_t C = __builtin_amdgcn_make_buffer_rsrc(
          (uint16_t*)g.C + (int64_t)img * g.H * g.W * g.rows, (short)0, out_bytes, 0x00020000);
#pragma unroll
      for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
          u32x4 v;
          if constexpr (EPI == EPI_RELU_BF16) {
            const float* bj = bias + nb * 32 + 16 * j + 8 * half;
            float bv[8];
            __builtin_memcpy(bv, __builtin_assume_aligned(bj, 32), 32);
#pragma unroll
            for (int i = 0; i < 4; ++i)
              v[i] = f2bf_pair(fmaxf(acc[b][8 * j + 2 * i] + bv[2 * i], 0.0f),
                               fmaxf(acc[b][8 * j + 2 * i + 1] + bv[2 * i + 1], 0.0f));
          } else {
            const uint32_t m[4] = {mask[b][j].x, mask[b][j].y, mask[b][j].z, mask[b][j].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              // a ReLU's output is positive or zero, so both tests are on the bits
              const uint32_t lo = bf_positive((uint16_t)m[i]) ? 0xffffu : 0u;
              const uint32_t hi = bf_positive((uint16_t)(m[i] >> 16)) ? 0xffff0000u : 0u;
              v[i] = f2bf_pair(acc[b][8 * j + 2 * i], acc[b][8 * j + 2 * i + 1]) & (lo | hi);
            }
          }
          __builtin_amdgcn_raw_buffer_store_b128(v, C, at_out[b][j], 0, 0);
        }
    }
    __syncthreads();
  }
}

struct WgradArgs {
  const uint16_t* X;       // layer input, NHWC [pixels][cp]
  const uint16_t* G;       // output gradient, NHWC [pixels][cpg]
  int H, W, cp, cpg;
  int tiles_x, tiles_y, tiles;  // 8 x 16 tiles of an image, and of the batch
  float* part;             // [workgroup][9 cp rows, .., row bias_row][cpg]
  int64_t stride;          // elements of a workgroup's sums
  int bias_row;
};

// Sums of a workgroup's tiles: part[kc][co] = sum_p col(X)[p][kc] G[p][co], and
// the column sums of G (the bias gradient) in row bias_row.  Three waves, one
// row of taps each, for every one of the CIB x COB blocks of 32 x 32 (input x
// output) channels: twelve at 64 x 64, three on every SIMD (nine waves of a
// tap each left one SIMD with three and the others with two).
//
// Both operands run along pixels, the outer dimension of NHWC: they are
// read from row-major LDS tiles with the transposing ds_read_b64_tr_b16 (16
// lanes fetch 4 pixels x 16 channels and each receives one channel's 4
// pixels), 16 pixels of a tile row per MFMA step.  Pixels lie 64 or 192 bytes
// apart, so the 4 pixels x 32 channels of 32 lanes cover all 64 banks (2.7 clocks
// a wave's read; 4.2 at pitches of 64, 68, 72 or 80 elements).  A tile's border
// is staged once for all nine taps.  The next tile is loaded while this one is
// multiplied.
// Measured at 16 x 128^2, 64 to 64 channels: 31 us (64 images: 96 us, 2.8 TB/s),
// the general matrix kernel before 74 us; a second tile in flight spilled
// (35 us), nine waves of one tap each took 32 us (64 images: 113 us).
template <int CIB, int COB>
__global__ __launch_bounds__(192 * CIB * COB) void k_wgrad(WgradArgs g) {
  constexpr int TH = 8, PIX = (TH + 2) * kTileP, PIXG = TH * kTile;
  constexpr int PA = CIB == 1 ? 32 : 96, PG = COB == 1 ? 32 : 96;  // elements between pixels
  constexpr int UA = 4 * CIB, UG = 4 * COB;                        // 8-channel chunks staged per pixel
  constexpr int NT = 192 * CIB * COB;
  constexpr int PERA = (PIX * UA + NT - 1) / NT, PERG = (PIXG * UG + NT - 1) / NT;
  constexpr int BUF = PIX * PA + PIXG * PG;
  __shared__ __attribute__((aligned(16))) uint16_t tile[2][BUF];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int dy = wave % 3, ci = wave / 3 % CIB, cj = wave / 3 / CIB;  // tap row, block of channels
  typedef short s4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s4 lds_s4;
  // transposing read: lane l supplies pixel 8 (l / 32) + (l / 4) % 4, channels
  // 16 ((l / 16) % 2) + 4 (l % 4) .. + 3, and receives channel l % 32 of pixels
  // 8 (l / 32) .. + 3 (the second read: 4 pixels on)
  const int pix = 8 * (lane >> 5) + ((lane >> 2) & 3), chan = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  const int at_a = (dy * kTileP + pix) * PA + 32 * ci + chan, at_g = PIX * PA + pix * PG + 32 * cj + chan;
  auto operand = [&](uint16_t* at, int pitch) {
    const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)at);
    const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(at + 4 * pitch));
    bf16x8 v;
    __builtin_memcpy(&v, &lo, 8);
    __builtin_memcpy((char*)&v + 8, &hi, 8);
    return v;
  };
  uint4 r[PERA + PERG];
  float bias[8] = {};  // 8 channels of the thread's chunk (NT is a multiple of UG)
  auto fetch = [&](int t) {
    const int img = t / (g.tiles_x * g.tiles_y), rest = t - img * (g.tiles_x * g.tiles_y), ty = rest / g.tiles_x;
    const int y0 = ty * TH, x0 = (rest - ty * g.tiles_x) * kTile;
    // offsets past the image read zeros
    const int bytes_a = g.H * g.W * g.cp * 2, bytes_g = g.H * g.W * g.cpg * 2;
    const __amdgpu_buffer_rsrc_t X = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(g.X + (int64_t)img * g.H * g.W * g.cp), (short)0, bytes_a, 0x00020000);
    const __amdgpu_buffer_rsrc_t G = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(g.G + (int64_t)img * g.H * g.W * g.cpg), (short)0, bytes_g, 0x00020000);
#pragma unroll
    for (int k = 0; k < PERA; ++k) {
      const int i = k * NT + threadIdx.x, px = i / UA, ch = i % UA;
      const int y = y0 + px / kTileP - 1, x = x0 + px % kTileP - 1;
      const bool in = px < PIX && ch * 8 < g.cp && (unsigned)y < (unsigned)g.H && (unsigned)x < (unsigned)g.W;
      const auto v = __builtin_amdgcn_raw_buffer_load_b128(X, in ? (y * g.W + x) * (g.cp * 2) + ch * 16 : bytes_a, 0, 0);
      __builtin_memcpy(&r[k], &v, 16);
    }
#pragma unroll
    for (int k = 0; k < PERG; ++k) {
      const int i = k * NT + threadIdx.x, px = i / UG, ch = i % UG;
      const int y = y0 + px / kTile, x = x0 + px % kTile;
      const bool in = px < PIXG && ch * 8 < g.cpg && y < g.H && x < g.W;
      const auto v = __builtin_amdgcn_raw_buffer_load_b128(G, in ? (y * g.W + x) * (g.cpg * 2) + ch * 16 : bytes_g, 0, 0);
      __builtin_memcpy(&r[PERA + k], &v, 16);
    }
  };
  auto stage = [&](uint16_t* to) {
#pragma unroll
    for (int k = 0; k < PERA; ++k) {
      const int i = k * NT + threadIdx.x, px = i / UA;
      if (px < PIX) *(uint4*)(to + px * PA + i % UA * 8) = r[k];
    }
#pragma unroll
    for (int k = 0; k < PERG; ++k) {
      const int i = k * NT + threadIdx.x, px = i / UG;
      if (px < PIXG) *(uint4*)(to + PIX * PA + px * PG + i % UG * 8) = r[PERA + k];
      const uint4 v = r[PERA + k];
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        bias[2 * q] += __uint_as_float(w[q] << 16);
        bias[2 * q + 1] += __uint_as_float(w[q] & 0xffff0000u);
      }
    }
  };
  f32x16 acc[3];
#pragma unroll
  for (int dx = 0; dx < 3; ++dx)
    for (int i = 0; i < 16; ++i) acc[dx][i] = 0.0f;
  __shared__ int again;
  if (threadIdx.x == 0) again = 0;
  int t = blockIdx.x, cur = 0;
  if (t < g.tiles) {
    fetch(t);
    stage(tile[0]);
  }
  __syncthreads();
  for (; t < g.tiles; t += gridDim.x, cur ^= 1) {
    const bool more = t + (int)gridDim.x < g.tiles;
    if (more) fetch(t + gridDim.x);
    uint16_t* in = tile[cur];
#pragma unroll
    for (int y = 0; y < TH; ++y) {
      const bf16x8 b = operand(in + at_g + y * kTile * PG, PG);
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        const bf16x8 a = operand(in + at_a + (y * kTileP + dx) * PA, PA);
        acc[dx] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[dx], 0, 0, 0);
      }
    }
    // schedule: the 8 LDS reads of a row a row ahead of its 3 products
    __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
#pragma unroll
    for (int y = 1; y < TH; ++y) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
    if (more) stage(tile[cur ^ 1]);
    __syncthreads();
  }
  // Pixels of the last tiles outside the image have zero gradients, but a
  // neighbour of theirs may be infinite, and 0 x Inf is NaN: sums that are not
  // finite are formed again without those pixels.
  if (g.H % TH != 0 || g.W % kTile != 0) {
    float zero[6] = {};  // six chains
#pragma unroll
    for (int dx = 0; dx < 3; ++dx)
#pragma unroll
      for (int i = 0; i < 16; ++i) zero[2 * dx + (i & 1)] = fmaf(acc[dx][i], 0.0f, zero[2 * dx + (i & 1)]);
    if (zero[0] + zero[1] + zero[2] + zero[3] + zero[4] + zero[5] != 0.0f) again = 1;
    __syncthreads();
    if (again != 0) {
#pragma unroll
      for (int dx = 0; dx < 3; ++dx)
        for (int i = 0; i < 16; ++i) acc[dx][i] = 0.0f;
#pragma unroll
      for (int q = 0; q < 8; ++q) bias[q] = 0.0f;
      for (t = blockIdx.x; t < g.tiles; t += gridDim.x) {
        fetch(t);
        stage(tile[0]);
        __syncthreads();
        const int rest = t % (g.tiles_x * g.tiles_y), rows = min(TH, g.H - rest / g.tiles_x * TH);
        const int columns = g.W - rest % g.tiles_x * kTile - 8 * (lane >> 5);  // of the lane's 8 pixels
#pragma unroll 1
        for (int y = 0; y < rows; ++y) {
          const bf16x8 b = operand(tile[0] + at_g + y * kTile * PG, PG);
#pragma unroll
          for (int dx = 0; dx < 3; ++dx) {
            bf16x8 a = operand(tile[0] + at_a + (y * kTileP + dx) * PA, PA);
#pragma unroll
            for (int q = 0; q < 8; ++q)
              if (q >= columns) a[q] = (__bf16)0.0f;
            acc[dx] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[dx], 0, 0, 0);
          }
        }
        __syncthreads();
      }
    }
  }
  float* part = g.part + (int64_t)blockIdx.x * g.stride;
#pragma unroll
  for (int dx = 0; dx < 3; ++dx)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      // accumulator layout: register r of lane l holds row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32
      const int c = 32 * ci + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), co = 32 * cj + (lane & 31);
      if (c < g.cp && co < g.cpg) part[(int64_t)((3 * dy + dx) * g.cp + c) * g.cpg + co] = acc[dx][r];
    }
  // column sums of G: the threads of a chunk added in thread order
  float* sums = (float*)tile[0];
  static_assert(sizeof(tile) >= NT * 8 * sizeof(float), "bias sums fit the tile");
#pragma unroll
  for (int q = 0; q < 8; ++q) sums[threadIdx.x * 8 + q] = bias[q];
  __syncthreads();
  if ((int)threadIdx.x < g.cpg) {
    float v = 0.0f;
    for (int k = threadIdx.x / 8; k < NT; k += UG) v += sums[k * 8 + threadIdx.x % 8];
    part[(int64_t)g.bias_row * g.cpg + threadIdx.x] = v;
  }
}

// a0[p][c] = bf16(s_c x[img][c][h][w]) for c < 2, zero for 2 <= c < 8.
__global__ void k_pack_input(const float* __restrict__ x, int64_t npix, int hw, float s0, float s1,
                             uint16_t* __restrict__ a0) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= npix) return;
  const int64_t img = p / hw, off = p - img * hw;
  const float x0 = x[img * 2 * hw + off], x1 = x[img * 2 * hw + hw + off];
  uint4 v;
  v.x = (uint32_t)f2bf(s0 * x0) | ((uint32_t)f2bf(s1 * x1) << 16);
  v.y = v.z = v.w = 0;
  *(uint4*)(a0 + p * 8) = v;
}

// Residual r = z + s1 x1 - s1 t; g[p][0] = bf16(2 r / npix), other channels
// 0; per-block sum of r^2 in FP64 (fixed-order tree).
__global__ __launch_bounds__(256) void k_loss(const float* __restrict__ z, const float* __restrict__ x,
                                              const float* __restrict__ tgt, int64_t npix, int hw, float s1,
                                              uint16_t* __restrict__ g, double* __restrict__ part) {
  __shared__ double sh[256];
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double r2 = 0.0;
  if (p < npix) {
    const int64_t img = p / hw, off = p - img * hw;
    const float r = z[p] + s1 * x[img * 2 * hw + hw + off] - s1 * tgt[p];
    r2 = (double)r * r;
    uint4 v;
    v.x = f2bf(2.0f * r / (float)npix);
    v.y = v.z = v.w = 0;
    *(uint4*)(g + p * 8) = v;
  }
  sh[threadIdx.x] = r2;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// *out = scale * sum of part[0 .. n): thread j adds part[j], part[j + 256],
// ... in order, then a fixed-shape tree adds the 256 sums (one workgroup of
// 256 threads; the same order on every call).
__global__ __launch_bounds__(256) void k_sum_in_order(const double* part, int n, double scale, double* out) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) s += part[i];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sh[0] * scale;
}

// grad W[co][tap][ci] = sum over splits of part[z][tap * cinp + ci][co]
// and grad b[co] = sum over splits of part[z][kp][co] (the bias row)
// (part entry o = kc * ldc + co).  A workgroup takes 64 consecutive entries
// o; its 16 waves add the splits z = w, w + 16, ... (w = wave) in order,
// reading 64 consecutive floats per split, and the 16 sums are added in
// wave order: a fixed order on every call.  (Four waves kept too few loads in
// flight: 19 us for 256 splits of 577 x 64.)
constexpr int kReduceWaves = 16;
__global__ __launch_bounds__(kReduceWaves * 64) void k_wgrad_reduce(const float* __restrict__ part, int splits,
                                                                    int64_t stride, int ldc, int cinp, int cin,
                                                                    int cout, int kp, float* __restrict__ grad,
                                                                    float* __restrict__ bgrad) {
  __shared__ double sh[kReduceWaves][64];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int64_t o = (int64_t)blockIdx.x * 64 + l;
  const int kc = (int)(o / ldc), co = (int)(o - (int64_t)kc * ldc);
  const int tap = kc / cinp, ci = kc - tap * cinp;
  // padding rows and columns were never written
  const bool used = o < stride && co < cout && (kc == kp || (tap < 9 && ci < cin));
  double s = 0.0;
  if (used)
    for (int z = w; z < splits; z += kReduceWaves) s += part[z * stride + o];
  sh[w][l] = s;
  __syncthreads();
  if (w != 0 || !used) return;
  double v = sh[0][l];
  for (int k = 1; k < kReduceWaves; ++k) v += sh[k][l];
  if (kc == kp)
    bgrad[co] = (float)v;
  else
    grad[(co * 9 + tap) * cin + ci] = (float)v;
}

// Forward weights W(co, kc) with kc = tap * cinp + ci and, for the data
// gradient, Wflip(ci, kc') = W[co][8 - tap'][ci] with kc' = tap' * coutp + co,
// at their places (weight_place), zero in the padding of channels (to blocks
// of 32) and entries; and the layer's biases, zero beyond cout (read four at
// a time).
static inline int round32(int c) { return (c + 31) / 32 * 32; }
__global__ void k_pack_weights(const float* __restrict__ W, const float* __restrict__ b, int cin, int cout, int cinp,
                               int coutp, int kp, int kpb, uint16_t* __restrict__ wb, uint16_t* __restrict__ wf,
                               float* __restrict__ bias) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kMaxChannels) bias[i] = i < cout ? b[i] : 0.0f;
  {
    const int co = i / kp, kc = i % kp, tap = kc / cinp, ci = kc % cinp;
    if (co < (coutp + 31) / 32 * 32)
      wb[weight_place(co, kc, kp)] = f2bf(co < cout && tap < 9 && ci < cin ? W[(co * 9 + tap) * cin + ci] : 0.0f);
  }
  if (wf) {
    const int ci = i / kpb, kc = i % kpb, tap = kc / coutp, co = kc % coutp;
    if (ci < (cinp + 31) / 32 * 32)
      wf[weight_place(ci, kc, kpb)] =
          f2bf(ci < cin && co < cout && tap < 9 ? W[(co * 9 + (8 - tap)) * cin + ci] : 0.0f);
  }
}

__global__ void k_adam(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, int64_t n, float lr, float b1, float b2, float eps, float c1,
                       float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

}  // namespace cnn
}  // namespace vam

struct vam_cnn {
  uint64_t magic;
  int device;
  int L, C, H, W, maxn;
  float s0, s1;
  std::vector<int> cin, cout, cinp, coutp, kp, kpb;
  std::vector<int64_t> woff, boff;
  int64_t nparam;
  float *master, *m1, *m2, *grad;
  float* bias;                     // [layers][kMaxChannels], padded copies of the biases
  std::vector<uint16_t*> wb, wf;   // per layer (index l - 1)
  std::vector<uint16_t*> act;      // a_0 .. a_{L-1}
  float* z;
  uint16_t* g[2];
  float* part;
  double* lpart;
  double* loss;
  int adam_t;
};

namespace vam {
namespace cnn {

static inline unsigned nblocks(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }
static inline int round_up(int x, int m) { return (x + m - 1) / m * m; }

static bool valid(const vam_cnn* h) { return h && h->magic == kCnnMagic; }

static void free_cnn(vam_cnn* h) {
  std::vector<void*> ptrs = {h->master, h->m1, h->m2, h->grad, h->bias, h->z, h->g[0], h->g[1],
                             h->part, h->lpart, h->loss};
  for (auto p : h->wb) ptrs.push_back(p);
  for (auto p : h->wf) ptrs.push_back(p);
  for (auto p : h->act) ptrs.push_back(p);
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  h->magic = 0;
  delete h;
}

template <int CP, int EPI>
static void launch_conv(const ConvArgs& a, hipStream_t s) {
  // one workgroup a CU (eight waves with the weights in registers fill it), two
  // where fewer channels leave room
  const dim3 grid((unsigned)std::min(a.tiles, CP > 32 ? 256 : 512));
  if constexpr (EPI != EPI_OUT_F32) {
    if (a.rows > 32) {
      hipLaunchKernelGGL((k_conv<CP, 2, EPI>), grid, dim3(512), 0, s, a);
      return;
    }
  }
  hipLaunchKernelGGL((k_conv<CP, 1, EPI>), grid, dim3(512), 0, s, a);
}

// The convolution of n images X with cp channels (a multiple of 8, <= 64).
template <int EPI>
static vam_status conv(ConvArgs a, int n, int H, int W, int cp, hipStream_t s) {
  a.H = H;
  a.W = W;
  a.tiles_x = (W + kTile - 1) / kTile;
  a.tiles_y = (H + kTile - 1) / kTile;
  a.tiles = n * a.tiles_x * a.tiles_y;
  switch (cp) {
    case 8: launch_conv<8, EPI>(a, s); break;
    case 16: launch_conv<16, EPI>(a, s); break;
    case 24: launch_conv<24, EPI>(a, s); break;
    case 32: launch_conv<32, EPI>(a, s); break;
    case 40: launch_conv<40, EPI>(a, s); break;
    case 48: launch_conv<48, EPI>(a, s); break;
    case 56: launch_conv<56, EPI>(a, s); break;
    default: launch_conv<64, EPI>(a, s); break;
  }
  VAM_HIP_TRY(hipGetLastError(), "launching a convolution");
  return VAM_OK;
}

// Sums of the weight gradient; returns the number of workgroups (splits).
static int wgrad(WgradArgs a, int n, int H, int W, hipStream_t s) {
  a.H = H;
  a.W = W;
  a.tiles_x = (W + kTile - 1) / kTile;
  a.tiles_y = (H + 7) / 8;
  a.tiles = n * a.tiles_x * a.tiles_y;
  const int splits = std::min(a.tiles, kMaxSplits);
  if (a.cp > 32 && a.cpg > 32) hipLaunchKernelGGL((k_wgrad<2, 2>), dim3(splits), dim3(768), 0, s, a);
  else if (a.cp > 32) hipLaunchKernelGGL((k_wgrad<2, 1>), dim3(splits), dim3(384), 0, s, a);
  else if (a.cpg > 32) hipLaunchKernelGGL((k_wgrad<1, 2>), dim3(splits), dim3(384), 0, s, a);
  else hipLaunchKernelGGL((k_wgrad<1, 1>), dim3(splits), dim3(192), 0, s, a);
  return splits;
}

static vam_status pack_all(vam_cnn* h, hipStream_t s) {
  for (int l = 1; l <= h->L; ++l) {
    const int i = l - 1;
    const int n = std::max(round32(h->coutp[i]) * h->kp[i], round32(h->cinp[i]) * h->kpb[i]);
    hipLaunchKernelGGL(k_pack_weights, dim3(nblocks(n, 256)), dim3(256), 0, s, h->master + h->woff[i],
                       h->master + h->boff[i], h->cin[i], h->cout[i], h->cinp[i], h->coutp[i], h->kp[i], h->kpb[i],
                       h->wb[i], h->wf[i], h->bias + (int64_t)i * kMaxChannels);
  }
  VAM_HIP_TRY(hipGetLastError(), "launching the weight packing");
  return VAM_OK;
}

#define CNN_TRY(expr)                   \
  do {                                  \
    vam_status st_ = (expr);            \
    if (st_ != VAM_OK) return st_;      \
  } while (0)

// Forward pass of n images; leaves a_0 .. a_{L-1} in the workspace, and either
// z there (y NULL) or the output y = x1 + z / s1 in y.
static vam_status forward(vam_cnn* h, const float* x, int n, float* y, hipStream_t s) {
  const int64_t npix = (int64_t)n * h->H * h->W;
  hipLaunchKernelGGL(k_pack_input, dim3(nblocks(npix, 256)), dim3(256), 0, s, x, npix, h->H * h->W, h->s0, h->s1,
                     h->act[0]);
  VAM_HIP_TRY(hipGetLastError(), "launching the input packing");
  for (int l = 1; l <= h->L; ++l) {
    const int i = l - 1;
    ConvArgs a = {};
    a.X = h->act[i];
    a.B = h->wb[i];
    a.kp = h->kp[i];
    a.rows = h->coutp[i];
    a.bias = h->bias + (int64_t)i * kMaxChannels;
    if (l < h->L) {
      a.C = h->act[l];
      CNN_TRY((conv<EPI_RELU_BF16>(a, n, h->H, h->W, h->cinp[i], s)));
    } else {
      a.C = y ? y : h->z;
      a.x = y ? x : nullptr;
      a.s1 = h->s1;
      CNN_TRY((conv<EPI_OUT_F32>(a, n, h->H, h->W, h->cinp[i], s)));
    }
  }
  return VAM_OK;
}

}  // namespace cnn
}  // namespace vam

using namespace vam;
using namespace vam::cnn;

extern "C" {

vam_status vam_cnn_create(int32_t layers, int32_t channels, int32_t height, int32_t width, int32_t max_batch,
                          float in_scale0, float in_scale1, vam_cnn_t* out) {
  clear_error();
  if (!out) return fail(VAM_ERR_INVALID_ARG, "NULL output handle");
  *out = nullptr;
  if (layers < 2 || layers > 32) return fail(VAM_ERR_INVALID_ARG, "layers must be in [2, 32]");
  if (channels < 8 || channels > 64 || channels % 8) return fail(VAM_ERR_INVALID_ARG, "channels must be 8..64, a multiple of 8");
  if (height < 1 || width < 1 || width > 1024 || height > 1024) return fail(VAM_ERR_INVALID_ARG, "image size outside [1, 1024]");
  if (max_batch < 1) return fail(VAM_ERR_INVALID_ARG, "max_batch must be positive");
  const int64_t npix = (int64_t)max_batch * height * width;
  if (npix % BK) return fail(VAM_ERR_INVALID_ARG, "max_batch * height * width must be a multiple of 32");
  if (npix * 576 >= (1LL << 40) || npix >= 0x7fffffffLL) return fail(VAM_ERR_INVALID_ARG, "batch too large");
  if (!(in_scale0 > 0.0f) || !(in_scale1 > 0.0f)) return fail(VAM_ERR_INVALID_ARG, "input scales must be positive");
  vam_cnn* h = new (std::nothrow) vam_cnn();
  if (!h) return fail(VAM_ERR_OUT_OF_MEMORY, "allocating the CNN handle");
  h->magic = kCnnMagic;
  (void)hipGetDevice(&h->device);
  h->L = layers;
  h->C = channels;
  h->H = height;
  h->W = width;
  h->maxn = max_batch;
  h->s0 = in_scale0;
  h->s1 = in_scale1;
  int64_t off = 0;
  int kmax = 0, cmax = 8;
  for (int l = 1; l <= layers; ++l) {
    const int ci = l == 1 ? 2 : channels, co = l == layers ? 1 : channels;
    h->cin.push_back(ci);
    h->cout.push_back(co);
    h->cinp.push_back(round_up(ci, 8));
    h->coutp.push_back(round_up(co, 8));
    h->kp.push_back(round_up(9 * round_up(ci, 8), BK));
    h->kpb.push_back(round_up(9 * round_up(co, 8), BK));
    h->woff.push_back(off);
    off += (int64_t)co * 9 * ci;
    h->boff.push_back(off);
    off += co;
    kmax = std::max({kmax, h->kp.back(), h->kpb.back()});
    cmax = std::max(cmax, round_up(co, 8));
  }
  h->nparam = off;
  const unsigned lblocks = nblocks(npix, 256);
  hipError_t e = hipSuccess;
  auto alloc = [&](void** p, size_t bytes) {
    if (e == hipSuccess) e = hipMalloc(p, std::max<size_t>(bytes, 256));
  };
  alloc((void**)&h->master, h->nparam * 4);
  alloc((void**)&h->m1, h->nparam * 4);
  alloc((void**)&h->m2, h->nparam * 4);
  alloc((void**)&h->grad, h->nparam * 4);
  alloc((void**)&h->bias, (size_t)layers * kMaxChannels * 4);
  h->wb.assign(layers, nullptr);
  h->wf.assign(layers, nullptr);
  h->act.assign(layers, nullptr);
  for (int i = 0; i < layers; ++i) {
    alloc((void**)&h->wb[i], (size_t)round32(h->coutp[i]) * h->kp[i] * 2);
    if (i > 0) alloc((void**)&h->wf[i], (size_t)round32(h->cinp[i]) * h->kpb[i] * 2);
    alloc((void**)&h->act[i], (size_t)npix * h->cinp[i] * 2);
  }
  alloc((void**)&h->z, (size_t)npix * 4);
  alloc((void**)&h->g[0], (size_t)npix * cmax * 2);
  alloc((void**)&h->g[1], (size_t)npix * cmax * 2);
  alloc((void**)&h->part, (size_t)kMaxSplits * (kmax + 1) * cmax * 4);  // one set of sums per workgroup
  alloc((void**)&h->lpart, (size_t)lblocks * 8);
  alloc((void**)&h->loss, 8);
  if (e == hipSuccess) e = hipMemset(h->master, 0, h->nparam * 4);
  if (e == hipSuccess) e = hipMemset(h->m1, 0, h->nparam * 4);
  if (e == hipSuccess) e = hipMemset(h->m2, 0, h->nparam * 4);
  if (e == hipSuccess) e = hipMemset(h->grad, 0, h->nparam * 4);
  if (e != hipSuccess) {
    vam_status st = hip_check(e, "allocating the CNN workspace");
    free_cnn(h);
    return st;
  }
  vam_status st = pack_all(h, nullptr);
  if (st == VAM_OK && hipDeviceSynchronize() != hipSuccess) st = fail(VAM_ERR_HIP, "initialising the CNN");
  if (st != VAM_OK) {
    free_cnn(h);
    return st;
  }
  *out = h;
  return VAM_OK;
}

vam_status vam_cnn_destroy(vam_cnn_t h) {
  clear_error();
  if (!valid(h)) return fail(VAM_ERR_BAD_HANDLE, "not a live CNN handle");
  (void)hipSetDevice(h->device);
  (void)hipDeviceSynchronize();
  free_cnn(h);
  return VAM_OK;
}

int64_t vam_cnn_param_count(vam_cnn_t h) { return valid(h) ? h->nparam : -1; }

vam_status vam_cnn_set_params(vam_cnn_t h, const float* params) {
  clear_error();
  if (!valid(h)) return fail(VAM_ERR_BAD_HANDLE, "not a live CNN handle");
  if (!params) return fail(VAM_ERR_INVALID_ARG, "NULL parameters");
  VAM_HIP_TRY(hipSetDevice(h->device), "hipSetDevice");
  VAM_HIP_TRY(hipMemcpy(h->master, params, h->nparam * 4, hipMemcpyHostToDevice), "copying parameters");
  VAM_HIP_TRY(hipMemset(h->m1, 0, h->nparam * 4), "clearing Adam moments");
  VAM_HIP_TRY(hipMemset(h->m2, 0, h->nparam * 4), "clearing Adam moments");
  h->adam_t = 0;
  CNN_TRY(pack_all(h, nullptr));
  VAM_HIP_TRY(hipDeviceSynchronize(), "packing weights");
  return VAM_OK;
}

vam_status vam_cnn_get_params(vam_cnn_t h, float* params) {
  clear_error();
  if (!valid(h)) return fail(VAM_ERR_BAD_HANDLE, "not a live CNN handle");
  if (!params) return fail(VAM_ERR_INVALID_ARG, "NULL parameters");
  VAM_HIP_TRY(hipSetDevice(h->device), "hipSetDevice");
  VAM_HIP_TRY(hipDeviceSynchronize(), "synchronising");
  VAM_HIP_TRY(hipMemcpy(params, h->master, h->nparam * 4, hipMemcpyDeviceToHost), "copying parameters");
  return VAM_OK;
}

vam_status vam_cnn_get_state(vam_cnn_t h, float* state, int64_t* adam_steps) {
  clear_error();
  if (!valid(h)) return fail(VAM_ERR_BAD_HANDLE, "not a live CNN handle");
  if (!state || !adam_steps) return fail(VAM_ERR_INVALID_ARG, "NULL argument");
  VAM_HIP_TRY(hipSetDevice(h->device), "hipSetDevice");
  VAM_HIP_TRY(hipDeviceSynchronize(), "synchronising");
  VAM_HIP_TRY(hipMemcpy(state, h->master, h->nparam * 4, hipMemcpyDeviceToHost), "copying parameters");
  VAM_HIP_TRY(hipMemcpy(state + h->nparam, h->m1, h->nparam * 4, hipMemcpyDeviceToHost), "copying moments");
  VAM_HIP_TRY(hipMemcpy(state + 2 * h->nparam, h->m2, h->nparam * 4, hipMemcpyDeviceToHost), "copying moments");
  *adam_steps = h->adam_t;
  return VAM_OK;
}

vam_status vam_cnn_set_state(vam_cnn_t h, const float* state, int64_t adam_steps) {
  clear_error();
  if (!valid(h)) return fail(VAM_ERR_BAD_HANDLE, "not a live CNN handle");
  if (!state) return fail(VAM_ERR_INVALID_ARG, "NULL state");
  if (adam_steps < 0 || adam_steps > (int64_t)1 << 40) return fail(VAM_ERR_INVALID_ARG, "bad Adam step count");
  VAM_HIP_TRY(hipSetDevice(h->device), "hipSetDevice");
  VAM_HIP_TRY(hipDeviceSynchronize(), "synchronising");
  VAM_HIP_TRY(hipMemcpy(h->master, state, h->nparam * 4, hipMemcpyHostToDevice), "copying parameters");
  VAM_HIP_TRY(hipMemcpy(h->m1, state + h->nparam, h->nparam * 4, hipMemcpyHostToDevice), "copying moments");
  VAM_HIP_TRY(hipMemcpy(h->m2, state + 2 * h->nparam, h->nparam * 4, hipMemcpyHostToDevice), "copying moments");
  h->adam_t = (int)adam_steps;
  CNN_TRY(pack_all(h, nullptr));
  VAM_HIP_TRY(hipDeviceSynchronize(), "packing weights");
  return VAM_OK;
}

vam_status vam_cnn_get_grads(vam_cnn_t h, float* grads) {
  clear_error();
  if (!valid(h)) return fail(VAM_ERR_BAD_HANDLE, "not a live CNN handle");
  if (!grads) return fail(VAM_ERR_INVALID_ARG, "NULL gradients");
  VAM_HIP_TRY(hipSetDevice(h->device), "hipSetDevice");
  VAM_HIP_TRY(hipDeviceSynchronize(), "synchronising");
  VAM_HIP_TRY(hipMemcpy(grads, h->grad, h->nparam * 4, hipMemcpyDeviceToHost), "copying gradients");
  return VAM_OK;
}

vam_status vam_cnn_forward(vam_cnn_t h, const float* x, int32_t n, float* y, hipStream_t s) {
  clear_error();
  if (!valid(h)) return fail(VAM_ERR_BAD_HANDLE, "not a live CNN handle");
  if (!x || !y) return fail(VAM_ERR_INVALID_ARG, "NULL buffer");
  if (n < 1 || n > h->maxn) return fail(VAM_ERR_INVALID_ARG, "batch %d outside [1, %d]", n, h->maxn);
  VAM_HIP_TRY(hipSetDevice(h->device), "hipSetDevice");
  return forward(h, x, n, y, s);
}

vam_status vam_cnn_loss_grad(vam_cnn_t h, const float* x, const float* t, int32_t n, double* loss_out,
                             hipStream_t s) {
  clear_error();
  if (!valid(h)) return fail(VAM_ERR_BAD_HANDLE, "not a live CNN handle");
  if (!x || !t) return fail(VAM_ERR_INVALID_ARG, "NULL buffer");
  if (n < 1 || n > h->maxn) return fail(VAM_ERR_INVALID_ARG, "batch %d outside [1, %d]", n, h->maxn);
  const int64_t npix = (int64_t)n * h->H * h->W;
  if (npix % BK) return fail(VAM_ERR_INVALID_ARG, "n * height * width must be a multiple of 32");
  VAM_HIP_TRY(hipSetDevice(h->device), "hipSetDevice");
  CNN_TRY(forward(h, x, n, nullptr, s));
  const int L = h->L;
  const unsigned lblocks = nblocks(npix, 256);
  // g_L = d loss / d z (8 channels, channel 0 used)
  uint16_t* gcur = h->g[0];
  uint16_t* gnext = h->g[1];
  hipLaunchKernelGGL(k_loss, dim3(lblocks), dim3(256), 0, s, h->z, x, t, npix, h->H * h->W, h->s1,
                     gcur, h->lpart);
  hipLaunchKernelGGL(k_sum_in_order, dim3(1), dim3(256), 0, s, h->lpart, (int)lblocks, 1.0 / (double)npix, h->loss);
  VAM_HIP_TRY(hipGetLastError(), "launching the CNN loss");
  for (int l = L; l >= 1; --l) {
    const int i = l - 1;
    // weight gradient: dW^T[kc][co] = sum_p col(a_{l-1})[p][kc] g_l[p][co] in
    // rows 0 .. 9 cinp - 1, and row kp = sum_p g_l[p][co] (the bias gradient)
    WgradArgs a = {};
    a.X = h->act[i];
    a.cp = h->cinp[i];
    a.G = gcur;
    a.cpg = h->coutp[i];
    a.part = h->part;
    a.stride = (int64_t)(h->kp[i] + 1) * h->coutp[i];
    a.bias_row = h->kp[i];
    const int splits = wgrad(a, n, h->H, h->W, s);
    hipLaunchKernelGGL(k_wgrad_reduce, dim3(nblocks(a.stride, 64)), dim3(kReduceWaves * 64), 0, s, h->part, splits,
                       a.stride, h->coutp[i], h->cinp[i], h->cin[i], h->cout[i], h->kp[i], h->grad + h->woff[i],
                       h->grad + h->boff[i]);
    VAM_HIP_TRY(hipGetLastError(), "launching the gradient reductions");
    if (l == 1) break;
    // data gradient through the ReLU of a_{l-1}
    ConvArgs d = {};
    d.X = gcur;
    d.B = h->wf[i];
    d.kp = h->kpb[i];
    d.rows = h->cinp[i];
    d.C = gnext;
    d.mask = h->act[i];
    CNN_TRY((conv<EPI_MASK_BF16>(d, n, h->H, h->W, h->coutp[i], s)));
    std::swap(gcur, gnext);
  }
  if (loss_out) {
    VAM_HIP_TRY(hipMemcpyAsync(loss_out, h->loss, 8, hipMemcpyDeviceToHost, s), "reading the loss");
    VAM_HIP_TRY(hipStreamSynchronize(s), "synchronising");
  }
  return VAM_OK;
}

vam_status vam_cnn_adam_step(vam_cnn_t h, float lr, float beta1, float beta2, float eps, hipStream_t s) {
  clear_error();
  if (!valid(h)) return fail(VAM_ERR_BAD_HANDLE, "not a live CNN handle");
  if (!(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f) || !(eps > 0.0f))
    return fail(VAM_ERR_INVALID_ARG, "Adam parameters out of range");
  VAM_HIP_TRY(hipSetDevice(h->device), "hipSetDevice");
  h->adam_t += 1;
  const float c1 = 1.0f - (float)std::pow((double)beta1, h->adam_t);
  const float c2 = 1.0f - (float)std::pow((double)beta2, h->adam_t);
  hipLaunchKernelGGL(k_adam, dim3(nblocks(h->nparam, 256)), dim3(256), 0, s, h->master, h->m1, h->m2, h->grad,
                     h->nparam, lr, beta1, beta2, eps, c1, c2);
  VAM_HIP_TRY(hipGetLastError(), "launching Adam");
  return pack_all(h, s);
}

}  // extern "C"
