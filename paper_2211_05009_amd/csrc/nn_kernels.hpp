// nn_kernels.hpp -- BF16 MFMA kernels of the warm-start surrogate (gfx950).
//
// Activations are NHWC bfloat16 (stored as uint16_t), channel counts
// multiples of 32; a tensor view is (pointer, channel stride, channel
// offset) so a layer can read or write one channel slice of a wider
// concatenation buffer.  Weights of a 3x3 convolution are [9][ci][co]
// (tap = 3 dy + dx, dy, dx in {0, 1, 2} for offsets -1, 0, +1).
//
// The three passes of a convolution:
//   forward : Y[p, o]      = sum_{t,c} X[p + d_t, c] W[t, c, o]  (+ bias, ReLU)
//   dgrad   : GX[p, c]     = sum_{t,o} GY[p - d_t, o] W[t, c, o]
//   wgrad   : GW[t, c, o] += sum_p     X[p + d_t, c] GY[p, o]
// all on v_mfma_f32_16x16x32_bf16 (FP32 accumulate): forward and dgrad as a
// direct convolution from an LDS patch (k_conv_tile) or, for widths it does
// not serve, a pipelined implicit GEMM (k_conv_mn);
// wgrad streamed over strips of image rows with all nine taps per block
// (k_wgrad_rows: widths 16-128) or as a pipelined GEMM over pixel chunks
// (k_wgrad: any width), the per-strip or per-chunk partials added in a
// fixed order (k_sum_parts).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace lbm {
namespace nn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(uint16_t b) {
  return __uint_as_float(((uint32_t)b) << 16);
}
// round to nearest even (finite inputs)
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

enum { FWD = 0, DGRAD = 1, WGRAD = 2 };

// Channels 0 .. 7 of pixel (x, y) of the encoded input canvas: 0 = cavity mask
// (rows y < round(128 Ar)), 1 = (x + 1/2) / 128, 2 = (y + 1/2) / 128, 3 =
// Re / 3000, 4 = Ar / 2, the others (and channels 8 .. 31) zero.
__device__ __forceinline__ uint4 encode_vec(double re, double ar, int x, int y) {
  const int ny = (int)rint(128.0 * ar);
  const float ch[5] = {y < ny ? 1.f : 0.f, (x + 0.5f) / 128.f, (y + 0.5f) / 128.f,
                       (float)(re / 3000.0), (float)(ar / 2.0)};
  return make_uint4(f2bf(ch[0]) | ((uint32_t)f2bf(ch[1]) << 16),
                    f2bf(ch[2]) | ((uint32_t)f2bf(ch[3]) << 16), f2bf(ch[4]), 0);
}

struct ConvArgs {
  int n, h, w, ci, co;
  const uint16_t *x;   // FWD / WGRAD: input activations; DGRAD: output gradient
  int xs, xo;
  const uint16_t *g;   // WGRAD: output gradient
  int gs, go;
  const uint16_t *wt;  // FWD / DGRAD: bf16 weights [9][ci][co]
  const uint16_t *wf;  // FWD / DGRAD (optional): the same weights in this pass's
                       // MFMA fragment order (k_pack_weights)
  const float *bias;   // FWD: per output channel (may be null)
  int relu;            // FWD: apply max(0, .)
  void *out;           // FWD: bf16 Y; DGRAD: bf16 GX; WGRAD: float GW [9 ci][co]
  int os, oo;
  int accumulate;      // DGRAD: add into GX
  const uint16_t *mask;  // DGRAD (optional): zero GX where mask <= 0 (the
                         // ReLU of the layer that produced the input; same
                         // stride and offset as out), before the bf16 rounding
  // FWD, k_conv_tile (optional): the layer's output also goes, as the next
  // op would write it, to
  uint16_t *pool_out;  // its 2 x 2 average pool, dense [n][h/2][w/2][co]
  uint16_t *up_out;    // its nearest 2x upsampling, a slice (ups, upo) of
  int ups, upo;        // [n][2h][2w]
  // FWD, k_conv_tile (optional), the network's ends: the input is the encoding
  // of an image's (Re, Ar) pair enc[2 b], enc[2 b + 1] and x is not read (32
  // input channels); channels 0 .. 2 of the rounded output also go, as FP32,
  // to head [n][h][w][3]
  const double *enc;
  float *head;
  int kchunk;          // WGRAD: pixels per block (multiple of 32)
  float *part;         // WGRAD: per-chunk partials [gridDim.z][9 ci][co], added
                       // into GW in chunk order by k_sum_parts (deterministic)
};

constexpr int kLdsK = 32 + 8;   // padded row of a staged 64 x 32 operand slice

// The hardware deals the blocks of a launch round-robin over the 8 XCDs
// (block L to XCD L % 8), each with its own L2.  xcd_block maps L to a
// block index such that each XCD runs one contiguous range of indices, so
// neighbouring tiles, which share halo rows and input strips, meet in one L2.
__device__ __forceinline__ int xcd_block(int L, int nb) {
  const int k = L & 7, q = nb >> 3, r = nb & 7;
  return k * q + (k < r ? k : r) + (L >> 3);
}

// ---------------------------------------------------------------------------
// Forward and input-gradient passes as one pipelined implicit GEMM.
//   FWD  : M = pixels, N = co, K = 9 ci;  A(p, (t,c)) = X[p + d_t][c],
//          B((t,c), o) = W[t][c][o] (16-byte vectors along n, stored into
//          LDS transposed, element by element: the weights are small).
//   DGRAD: M = pixels, N = ci, K = 9 co;  A(p, (t,o)) = GY[p - d_t][o],
//          B((t,o), c) = W[t][c][o] (contiguous along k = o).
// A block of 256 threads (WM x WN waves, each TM x TN MFMA 16 x 16 x 32
// tiles) computes a BM x BN tile, BM = 16 WM TM, BN = 16 WN TN.  K advances
// in slices of 32 (one tap, 32 channels: channel counts are multiples of 32,
// so a slice never straddles a tap); each slice is loaded from global memory
// into registers while the previous one is multiplied out of LDS, and the
// two LDS buffers alternate, so one barrier per slice suffices.
constexpr int kBK = 32;

template <int MODE, int WM, int WN, int TM, int TN>
__global__ __launch_bounds__(256) void k_conv_mn(ConvArgs a) {
  static_assert(WM * WN == 4, "four waves");
  constexpr int BM = 16 * WM * TM, BN = 16 * WN * TN;
  // 16-byte vectors per thread and operand (4 per row of 32 k)
  constexpr int AV = (BM * 4 + 255) / 256, BV = (BN * 4 + 255) / 256;
  __shared__ uint16_t As[2][BM * kLdsK];
  __shared__ uint16_t Bs[2][BN * kLdsK];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int HW = a.h * a.w, M = a.n * HW;
  const int C = MODE == FWD ? a.ci : a.co;      // channels along k within a tap
  const int N = MODE == FWD ? a.co : a.ci;
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
  const int nk = 9 * C / kBK;

  // staging: vector v of this thread covers row r = (tid + 256 v) / 4, k = 8 ((tid) % 4)
  const int kq = (tid & 3) * 8;
  int apix[AV], ay[AV], ax[AV];
#pragma unroll
  for (int v = 0; v < AV; ++v) {   // rows beyond BM or M load zeros (ay out of range)
    const int m = (tid >> 2) + 64 * v < BM ? m0 + (tid >> 2) + 64 * v : M;
    const int b = m / HW, r = m - b * HW;
    ay[v] = m < M ? r / a.w : -1000000;
    ax[v] = r - (r / a.w) * a.w;
    apix[v] = b * HW;
  }
  uint4 ra[AV], rb[BV];
  auto load = [&](int ks) {
    const int k0 = ks * kBK, tap = k0 / C, c0 = k0 - tap * C + kq;
    const int dy = tap / 3 - 1, dx = tap % 3 - 1;
#pragma unroll
    for (int v = 0; v < AV; ++v) {
      const int qy = MODE == FWD ? ay[v] + dy : ay[v] - dy;
      const int qx = MODE == FWD ? ax[v] + dx : ax[v] - dx;
      if (qy >= 0 && qy < a.h && qx >= 0 && qx < a.w)
        ra[v] = *(const uint4 *)(a.x + (size_t)(apix[v] + qy * a.w + qx) * a.xs + a.xo + c0);
      else
        ra[v] = make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < BV; ++v) {
      if (MODE == FWD) {   // W[tap][c][o]: row k = tid % 32, 8 n from 8 (tid / 32 + 8 v)
        const int kb = tid & 31, nb = 8 * ((tid >> 5) + 8 * v);
        const int cc = k0 - tap * C + kb;
        rb[v] = (nb < BN && n0 + nb < N)
                    ? *(const uint4 *)(a.wt + ((size_t)tap * a.ci + cc) * a.co + n0 + nb)
                    : make_uint4(0, 0, 0, 0);
      } else {             // W[tap][c][o], k = o: row n = tid / 4 + 64 v, 8 k
        const int n = n0 + (tid >> 2) + 64 * v;
        rb[v] = ((tid >> 2) + 64 * v < BN && n < N)
                    ? *(const uint4 *)(a.wt + ((size_t)tap * a.ci + n) * a.co + c0)
                    : make_uint4(0, 0, 0, 0);
      }
    }
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int v = 0; v < AV; ++v)
      if ((tid >> 2) + 64 * v < BM)
        *(uint4 *)&As[buf][((tid >> 2) + 64 * v) * kLdsK + kq] = ra[v];
#pragma unroll
    for (int v = 0; v < BV; ++v) {
      if (MODE == FWD) {
        const int kb = tid & 31, nb = 8 * ((tid >> 5) + 8 * v);
        if (nb < BN) {
          const uint16_t *e = (const uint16_t *)&rb[v];
#pragma unroll
          for (int j = 0; j < 8; ++j) Bs[buf][(nb + j) * kLdsK + kb] = e[j];
        }
      } else if ((tid >> 2) + 64 * v < BN) {
        *(uint4 *)&Bs[buf][((tid >> 2) + 64 * v) * kLdsK + kq] = rb[v];
      }
    }
  };

  floatx4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  const int fr = lane & 15, fk = (lane >> 4) * 8;
  load(0);
  stage(0);
  __syncthreads();
  for (int ks = 0; ks < nk; ++ks) {
    const int buf = ks & 1;
    if (ks + 1 < nk) load(ks + 1);
    bf16x8 fa[TM], fb[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
      fa[i] = *(const bf16x8 *)&As[buf][(wm * TM * 16 + i * 16 + fr) * kLdsK + fk];
#pragma unroll
    for (int j = 0; j < TN; ++j)
      fb[j] = *(const bf16x8 *)&Bs[buf][(wn * TN * 16 + j * 16 + fr) * kLdsK + fk];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    if (ks + 1 < nk) stage(buf ^ 1);
    __syncthreads();
  }

  // epilogue: lane holds rows 4 (lane / 16) + e, column lane % 16 of each tile
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn * TN * 16 + j * 16 + (lane & 15);
      if (n >= N) continue;
      const float bn = (MODE == FWD && a.bias) ? a.bias[n] : 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + wm * TM * 16 + i * 16 + (lane >> 4) * 4 + e;
        if (m >= M) continue;
        float v = acc[i][j][e];
        uint16_t *o = (uint16_t *)a.out + (size_t)m * a.os + a.oo + n;
        if (MODE == FWD) {
          v += bn;
          if (a.relu) v = fmaxf(v, 0.f);
        } else {
          if (a.accumulate) v += bf2f(*o);
          if (a.mask && !(bf2f(a.mask[o - (uint16_t *)a.out]) > 0.f)) v = 0.f;
        }
        *o = f2bf(v);
      }
    }
}

// ---------------------------------------------------------------------------
// The same two passes as direct convolutions, out[p][n] = sum over chunks of
// 32 input channels, then over the 9 taps, of IN[p +- d_t][k] W[t][n][k]
// (FWD: n = output channel, k = input channel; DGRAD the other way round and
// the taps mirrored).  A block of four waves computes BR rows x BC columns of
// one image by 32 channels, two waves along the pixels and two along the
// channels; a wave holds RT rows x 16 columns x 16 channels as RT MFMA tiles
// (channels x pixels: a lane's four results are four channels of one pixel).
//
// What bounds it: at the batch sizes of the network a layer has one or two
// waves per SIMD, so what matters is that neither LDS nor the vector memory
// path nor a barrier holds the MFMAs up.
//  * Weights never enter LDS: a wave needs its own 9 fragments of a chunk,
//    and reads the next chunk's from a copy laid out in fragment order (9
//    loads of 1 KB each, pack_weights) while it works on this one's.
//  * A patch row's fragment (16 pixels, shifted by dx) serves the up to three
//    output rows it is a tap of: 3 (RT + 2) LDS reads for 9 RT MFMAs, in an
//    order that still adds each output's taps 0 to 8 in turn.
//  * The patch (halo included; pixels outside the image come back as zeros
//    from buffer loads) lies in LDS with 64 bytes a pixel, the 16-byte groups
//    of every second quad of columns swapped by twos: no two lanes of a read
//    meet on a bank (4.3 clocks per wave read; 80 bytes a pixel took 8.0).
//  * Two patch buffers, the stores of chunk c + 1 and the loads of c + 2 and of
//    the weights spread between the MFMAs of chunk c: one barrier a chunk.
//  * The epilogue works in registers; v_permlane16_swap pairs two rows so
//    that every store is 16 bytes.
// Layers with one chunk (ONE) have nothing to prefetch: a single buffer and
// 100 registers instead of 211 let a CU hold five blocks instead of two.
// Measured (batch 8, the network's 15 layers, against whole-row tiles with
// patch and weights staged through LDS): forward 248 -> 182 us, input gradient
// 270 -> 188 us; 384 > 128 channels at 32 x 64 29.0 -> 17.0 us (850 TFLOP/s),
// 32 > 32 at 128 x 256 14.5 -> 10.5 us (3.2 TB/s, 6.7 us at a copy's rate).
// The network's ends, without the encoding and extracting kernels around them:
// a forecast of 8 samples 228 -> 216 us.

// the value of the neighbouring lane (lane ^ 1)
__device__ __forceinline__ float lane_xor1(float v) {
  return __uint_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0xB1, 0xF, 0xF, true));
}

// v_permlane16_swap: [a0 a1 a2 a3], [b0 b1 b2 b3] (rows of 16 lanes) become
// [a0 b0 a2 b2], [a1 b1 a3 b3]
__device__ __forceinline__ void swap16(float &a, float &b) {
  const auto r =
      __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}

// ENDS: with ConvArgs enc and head (the others carry no code for them: it costs
// registers, and 2 % of a training step).
template <int MODE, int RT, int WR, int WC, bool ONE, bool ENDS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(ONE ? 4 : 2))) void
k_conv_tile(ConvArgs a, int ntx, int nty) {
  static_assert(WR * WC == 2 && RT % 2 == 0, "two waves along the pixels");
  static_assert(!ENDS || (MODE == FWD && ONE), "the network's ends");
  constexpr int BR = RT * WR, BC = 16 * WC;
  // patch rows of a multiple of 4 pixels, so that a row's columns have the
  // same banks whatever the row
  constexpr int PW = BC + 4, PP = (BR + 2) * PW;
  constexpr int PV = (PP * 4 + 255) / 256;   // 16-byte patch vectors per thread
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  __shared__ __align__(16) uint16_t Sm[ONE ? 1 : 2][PP * 32];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = WR == 2 ? wave >> 1 : 0, wc = WC == 2 ? wave >> 1 : 0;
  const int C = MODE == FWD ? a.ci : a.co, N = MODE == FWD ? a.co : a.ci;
  // block -> channels fastest, then tile column, tile row, image: the blocks
  // of one XCD share patches and halos in its L2
  const int ntn = N / 32, b = xcd_block(blockIdx.x, gridDim.x);
  const int n0 = b % ntn * 32 + (wave & 1) * 16;   // this wave's first channel
  const int pt = b / ntn, tx = pt % ntx, ty = pt / ntx % nty, img = pt / (ntx * nty);
  const int y0 = ty * BR, x0 = tx * BC;
  const int fr = lane & 15, g = lane >> 4;

  // byte offsets in the image of this thread's patch vectors (out of the
  // buffer's range where there is no pixel: such loads return zeros)
  int poff[PV];
  const int pkq = (tid & 3) * 8;
#pragma unroll
  for (int u = 0; u < PV; ++u) {
    const int pp = (tid + 256 * u) >> 2, py = pp / PW, px = pp - py * PW;
    const int gy = y0 + py - 1, gx = x0 + px - 1;
    poff[u] = (pp < PP && px < BC + 2 && gy >= 0 && gy < a.h && gx >= 0 && gx < a.w)
                  ? ((gy * a.w + gx) * a.xs + pkq) * 2
                  : 0x7ffffff0;
  }
  const uint32_t xbytes = (uint32_t)(a.h * a.w * a.xs - a.xo) * 2;
  auto image = [&](bool on) {   // the input image (empty: loads cost nothing)
    return __builtin_amdgcn_make_buffer_rsrc((void *)(a.x + (size_t)img * a.h * a.w * a.xs + a.xo),
                                             0, on ? xbytes : 0, 0x00020000);
  };
  // weight fragments: lane's 8 k of channel fr, k = 8 g; from the packed copy
  // [n / 16][chunk][tap][lane][8], or straight from the rows [tap][n][k]
  const uint16_t *wsrc;
  int wlane, wtap, wchunk;
  if (a.wf) {
    wsrc = a.wf + (size_t)n0 * C * 9;
    wlane = lane * 8;
    wtap = 512;
    wchunk = 9 * 512;
  } else {   // DGRAD
    wsrc = a.wt + (size_t)n0 * C;
    wlane = fr * C + g * 8;
    wtap = N * C;
    wchunk = 32;
  }
  float bv[4] = {0.f, 0.f, 0.f, 0.f};
  if (MODE == FWD && a.bias) {
#pragma unroll
    for (int e = 0; e < 4; ++e) bv[e] = a.bias[n0 + 4 * g + e];
  }

  floatx4 acc[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) acc[r] = floatx4{0.f, 0.f, 0.f, 0.f};
  // LDS element of this lane's fragment in patch row 0, per tap column
  int abase[3];
#pragma unroll
  for (int dx = 0; dx < 3; ++dx) {
    const int px = wc * 16 + fr + (MODE == FWD ? dx : 2 - dx);
    abase[dx] = (wr * RT * PW + px) * 32 + ((g * 8) ^ ((px & 4) << 2));
  }
  u32x4 rp[PV];
  auto put = [&](int bf, int u) {
    const int pp = (tid + 256 * u) >> 2, px = pp % PW;
    if (pp < PP) *(u32x4 *)&Sm[bf][pp * 32 + (pkq ^ ((px & 4) << 2))] = rp[u];
  };
  bf16x8 w0[9], w1[9];
  {
    const auto rs = image(true);
    if (ENDS && a.enc) {
      const double re = a.enc[2 * img], ar = a.enc[2 * img + 1];
#pragma unroll
      for (int u = 0; u < PV; ++u) {
        const int pp = (tid + 256 * u) >> 2, py = pp / PW;
        const uint4 v = encode_vec(re, ar, x0 + pp - py * PW - 1, y0 + py - 1);
        const bool on = pkq == 0 && poff[u] != 0x7ffffff0;
        rp[u] = on ? u32x4{v.x, v.y, v.z, v.w} : u32x4{0, 0, 0, 0};
      }
    } else {
#pragma unroll
      for (int u = 0; u < PV; ++u)
        rp[u] = __builtin_amdgcn_raw_buffer_load_b128(rs, poff[u], 0, 0);
    }
#pragma unroll
    for (int t = 0; t < 9; ++t) w0[t] = *(const bf16x8 *)(wsrc + t * (size_t)wtap + wlane);
#pragma unroll
    for (int u = 0; u < PV; ++u) put(0, u);
    if (!ONE) {
#pragma unroll
      for (int u = 0; u < PV; ++u)
        rp[u] = __builtin_amdgcn_raw_buffer_load_b128(rs, poff[u], 64, 0);
    }
  }

  // One chunk (channels c0 .. c0 + 31) out of buffer bf with weights w; with
  // chunks to come, also the next one's patch into the other buffer, its
  // weights into wn and the loads of the patch after it.
  auto chunk = [&](auto last_t, int bf, int c0, bf16x8(&w)[9], bf16x8(&wn)[9]) {
    constexpr bool LAST = decltype(last_t)::value;
    __syncthreads();
    const uint16_t *P = Sm[bf];
    const auto rs = image(c0 + 64 < C);
    const uint16_t *wp = wsrc + (size_t)(c0 / 32 + 1) * wchunk + wlane;
    bf16x8 fa[2][3];
    auto read_row = [&](int i) {
      const int row = MODE == FWD ? i : RT + 1 - i;
#pragma unroll
      for (int dx = 0; dx < 3; ++dx)
        fa[i & 1][dx] = *(const bf16x8 *)(P + abase[dx] + row * PW * 32);
    };
    read_row(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < RT + 2; ++i) {
      if (i + 1 < RT + 2) read_row(i + 1);
      if (!LAST) {
        constexpr int WI = (9 + RT + 1) / (RT + 2), S0 = PV < RT + 2 ? (RT + 2 - PV) / 2 : 0;
        static_assert(PV <= RT + 2, "one patch vector per row step");
#pragma unroll
        for (int q = 0; q < WI; ++q)
          if (i * WI + q < 9)
            wn[i * WI + q] = *(const bf16x8 *)(wp + (size_t)(i * WI + q) * wtap);
        if (i >= S0 && i - S0 < PV) {
          put(bf ^ 1, i - S0);
          rp[i - S0] =
              __builtin_amdgcn_raw_buffer_load_b128(rs, poff[i - S0], (c0 + 64) * 2, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int dx = 0; dx < 3; ++dx)
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) {
          const int q = i - dy;
          if (q < 0 || q >= RT) continue;
          const int r = MODE == FWD ? q : RT - 1 - q;
          acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[dy * 3 + dx], fa[i & 1][dx], acc[r],
                                                           0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int c0 = 0;; c0 += 64) {
    if (ONE || c0 + 32 >= C) {
      chunk(std::true_type{}, 0, c0, w0, w1);
      break;
    }
    chunk(std::false_type{}, 0, c0, w0, w1);
    if (c0 + 64 >= C) {
      chunk(std::true_type{}, 1, c0 + 32, w1, w0);
      break;
    }
    chunk(std::false_type{}, 1, c0 + 32, w1, w0);
  }

  // Epilogue, rows in pairs: after the swap the lanes of even groups of 16
  // hold 8 channels of row r, those of odd groups the same channels of r + 1.
  const int x = x0 + wc * 16 + fr, yb = y0 + wr * RT, ch = n0 + 8 * (g >> 1);
#pragma unroll
  for (int r = 0; r < RT; r += 2) {
    if (yb + r >= a.h) break;
    float v[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = acc[r][e];
      v[4 + e] = acc[r + 1][e];
      if (MODE == FWD) {
        v[e] += bv[e];
        v[4 + e] += bv[e];
        if (a.relu) {
          v[e] = fmaxf(v[e], 0.f);
          v[4 + e] = fmaxf(v[4 + e], 0.f);
        }
      }
      swap16(v[e], v[4 + e]);
    }
    const int y = yb + r + (g & 1);
    if (y < a.h) {
      uint16_t *o = (uint16_t *)a.out + ((size_t)(img * a.h + y) * a.w + x) * a.os + a.oo + ch;
      if (MODE == DGRAD) {
        if (a.accumulate) {
          const uint4 old = *(const uint4 *)o;
          const uint16_t *ov = (const uint16_t *)&old;
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] += bf2f(ov[e]);
        }
        if (a.mask) {
          const uint4 mv = *(const uint4 *)(a.mask + (o - (uint16_t *)a.out));
          const uint16_t *mk = (const uint16_t *)&mv;
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (!(bf2f(mk[e]) > 0.f)) v[e] = 0.f;
        }
      }
      uint4 pk;
      uint16_t *pv = (uint16_t *)&pk;
#pragma unroll
      for (int e = 0; e < 8; ++e) pv[e] = f2bf(v[e]);
      *(uint4 *)o = pk;
      if (ENDS && a.head && ch == 0) {
        float *hd = a.head + ((size_t)(img * a.h + y) * a.w + x) * 3;
#pragma unroll
        for (int e = 0; e < 3; ++e) hd[e] = bf2f(pv[e]);
      }
      if (MODE == FWD && a.up_out) {   // the 2 x 2 copies at twice the resolution
        uint16_t *u = a.up_out +
                      ((size_t)(img * 2 * a.h + 2 * y) * (2 * a.w) + 2 * x) * a.ups + a.upo + ch;
        *(uint4 *)u = pk;
        *(uint4 *)(u + a.ups) = pk;
        *(uint4 *)(u + (size_t)2 * a.w * a.ups) = pk;
        *(uint4 *)(u + (size_t)(2 * a.w + 1) * a.ups) = pk;
      }
    }
    // 2 x 2 means of the rounded outputs, in k_pool_fwd's order (the image's
    // height is even where there is a pool: the pair is whole)
    if (MODE == FWD && a.pool_out) {
      uint4 pk;
      uint16_t *pv = (uint16_t *)&pk;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float p00 = bf2f(f2bf(v[e])), p01 = lane_xor1(p00), p10 = p00, p11 = p01;
        swap16(p00, p10);   // row r and row r + 1 in every lane
        swap16(p01, p11);
        float sm = 0.f;
        sm += p00;
        sm += p01;
        sm += p10;
        sm += p11;
        pv[e] = f2bf(0.25f * sm);
      }
      if ((lane & 17) == 0)   // even columns, even groups
        *(uint4 *)(a.pool_out +
                   ((size_t)(img * (a.h / 2) + (yb + r) / 2) * (a.w / 2) + x / 2) * a.co + ch) = pk;
    }
  }
}

// ---------------------------------------------------------------------------
// Weight gradient as a pipelined GEMM over a chunk of pixels:
//   part[z][m = (t, c)][o] = sum_{p in chunk z} X[p + d_t][c] GY[p][o]
// M = 9 ci, N = co, K = pixels.  Both operands are pixel-major in memory
// (NHWC) while the MFMA takes 8 consecutive k per lane, so each operand is
// transposed on its way into LDS: a loader thread reads 4 consecutive
// pixels x 8 channels (four 16-byte loads) and writes, per channel, the 4
// pixels as one 64-bit LDS store (As[m][k], Bs[n][k], k contiguous).  A
// block computes a 64 x BN tile with four waves (2 x 2), K advances by 64
// pixels; the next slice is loaded into registers while the current one is
// multiplied out of the other LDS buffer.
constexpr int kWBK = 64, kWLd = kWBK + 8;   // pixels per slice, padded LDS row

template <int BN>
__global__ __launch_bounds__(256) void k_wgrad(ConvArgs a) {
  constexpr int TN = BN / 32;                       // 16-wide n tiles per wave (2 x 2 waves)
  __shared__ __align__(16) uint16_t As[2][64 * kWLd];
  __shared__ __align__(16) uint16_t Bs[2][BN * kWLd];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int HW = a.h * a.w, M = 9 * a.ci, N = a.co;
  const int m0 = blockIdx.x * 64, n0 = blockIdx.y * BN;
  const int p_begin = blockIdx.z * a.kchunk;
  const int p_end = min(p_begin + a.kchunk, a.n * HW);
  // loader roles: threads 0-127 take A (8 rows x 4 pixels each), threads
  // 128 .. 128 + 2 BN - 1 take B (8 columns x 4 pixels each)
  const bool isA = tid < 128;
  const int li = isA ? tid : tid - 128;
  const int rg = li >> 4, pq = li & 15;            // row / column group, pixel quad
  const bool active = isA || li < 2 * BN;
  // A rows 8 rg .. 8 rg + 7: tap and first channel (8 rows share a tap)
  const int am = m0 + 8 * rg;
  const int atap = am / a.ci, ac = am - atap * a.ci;
  const int ady = atap / 3 - 1, adx = atap % 3 - 1;
  const bool arow_ok = am < M;
  const int bn = n0 + 8 * rg;
  const bool bcol_ok = bn < N;

  uint4 r[4];
  auto load = [&](int k0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int p = k0 + 4 * pq + j;
      r[j] = make_uint4(0, 0, 0, 0);
      if (!active || p >= p_end) continue;
      if (isA) {
        if (!arow_ok) continue;
        const int b = p / HW, q = p - b * HW, py = q / a.w, px = q - py * a.w;
        const int qy = py + ady, qx = px + adx;
        if (qy >= 0 && qy < a.h && qx >= 0 && qx < a.w)
          r[j] = *(const uint4 *)(a.x + ((size_t)b * HW + (size_t)qy * a.w + qx) * a.xs + a.xo +
                                  ac);
      } else if (bcol_ok) {
        r[j] = *(const uint4 *)(a.g + (size_t)p * a.gs + a.go + bn);
      }
    }
  };
  auto stage = [&](int buf) {
    if (!active) return;
    uint16_t *dst = isA ? &As[buf][0] : &Bs[buf][0];
    const uint16_t *e0 = (const uint16_t *)&r[0], *e1 = (const uint16_t *)&r[1];
    const uint16_t *e2 = (const uint16_t *)&r[2], *e3 = (const uint16_t *)&r[3];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      uint2 v;
      v.x = (uint32_t)e0[c] | ((uint32_t)e1[c] << 16);
      v.y = (uint32_t)e2[c] | ((uint32_t)e3[c] << 16);
      *(uint2 *)&dst[(8 * rg + c) * kWLd + 4 * pq] = v;
    }
  };

  floatx4 acc[2][TN];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int fr = lane & 15, fk = (lane >> 4) * 8;
  load(p_begin);
  stage(0);
  __syncthreads();
  int buf = 0;
  for (int k0 = p_begin; k0 < p_end; k0 += kWBK) {
    const bool more = k0 + kWBK < p_end;
    if (more) load(k0 + kWBK);
#pragma unroll
    for (int kk = 0; kk < kWBK; kk += 32) {
      bf16x8 fa[2], fb[TN];
#pragma unroll
      for (int i = 0; i < 2; ++i)
        fa[i] = *(const bf16x8 *)&As[buf][(wm * 32 + i * 16 + fr) * kWLd + kk + fk];
#pragma unroll
      for (int j = 0; j < TN; ++j)
        fb[j] = *(const bf16x8 *)&Bs[buf][(wn * TN * 16 + j * 16 + fr) * kWLd + kk + fk];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
    if (more) stage(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + wm * 32 + i * 16 + (lane >> 4) * 4 + e;
        const int n = n0 + wn * TN * 16 + j * 16 + (lane & 15);
        if (m < M && n < N) a.part[((size_t)blockIdx.z * M + m) * N + n] = acc[i][j][e];
      }
}

// Weight gradient streamed over image rows, for widths 16, 32, 64 and 128.
//   part[z][(t, c)][o] = sum over the pixels p of strip z of X[p + d_t][c] GY[p][o]
// A strip is `rows` consecutive image rows of the batch (it may run on from
// one image into the next); a block owns one strip, 32 input channels
// (c0 ..), NB = 32 NT output channels (o0 ..) and all nine taps, so each
// input and output-gradient element of the strip is loaded once per block
// (k_wgrad loads them once per 64-row tile of the 9 ci taps x channels).
// The reduction runs over pixels: a lane's 8 consecutive MFMA k are 8
// consecutive x of one row, so both operands are stored into LDS with x
// contiguous (channel rows):
//   input rows in a ring of 2U + 2 image rows, each [32 c][W + 8], the 8
//   zeros after a channel row doubling as the pad before the next one, so
//   x = -1 and x = W read zeros;
//   output-gradient rows of the current and the next iteration.
// Per tap row the three x offsets come from one aligned 16-byte read and
// two 4-byte reads by funnel shifts (v_alignbit); rows above the top or
// below the bottom of a pixel's image give zero operands.  An iteration
// covers U rows (U W pixels, a multiple of 128: U W / 32 k-steps; U <= h):
// the next iteration's rows are loaded into registers while the current
// one is multiplied out, then written into ring slots the current
// iteration does not read, so one barrier per iteration suffices.  KW groups of four waves split each
// iteration's k-steps and add their sums in LDS at the end (fixed order),
// so a block does KW times the work of one group and the strips, hence the
// partials, are KW times fewer.  With bpart set, blocks of the first
// channel tile also add up GY of their strip in FP32, the bias gradient's
// partial bpart[z][o] (fixed order: per thread, then a fixed LDS tree).
template <int W, int U, int NT, int KW>
__global__ __launch_bounds__(256 * KW) void k_wgrad_rows(ConvArgs a, int rows, float *bpart) {
  static_assert(U * W % 128 == 0 && W % 16 == 0, "an iteration is a multiple of 128 pixels");
  constexpr int NTH = 256 * KW;
  constexpr int RP = W + 8, NR = 2 * U + 2, NB = 32 * NT, KS = U * W / 32;
  static_assert(KS % KW == 0, "groups share the k-steps evenly");
  constexpr int NIN = U * W, NGO = U * W * NT;   // loader tasks: 4 pixels x 8 channels
  constexpr int IN_T = (NIN + NTH - 1) / NTH, GO_T = (NGO + NTH - 1) / NTH;
  constexpr int GCG = 4 * NT;                    // 8-channel groups of the NB outputs
  constexpr int IS_EL = NR * 32 * RP + 8, GS_EL = U * NB * RP;
  __shared__ __align__(16) uint16_t Is[IS_EL];
  __shared__ __align__(16) uint16_t Gs[2][GS_EL];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int grp = wave >> 2, gw = wave & 3;      // k-step group, wave within it
  const int wc = gw & 1, wn = gw >> 1;
  const int fr = lane & 15, fk = (lane >> 4) * 8;
  // block -> (strip, output tile, channel tile); consecutive blocks of one
  // XCD share a strip
  const int tcn = a.ci / 32, ton = a.co / NB;
  const int id = xcd_block(blockIdx.x, gridDim.x);
  const int z = id / (tcn * ton), cx = id % tcn, ox = (id / tcn) % ton;
  const int c0 = 32 * cx, o0 = NB * ox;
  const int nrow = a.n * a.h;
  const int r0 = z * rows, r1 = min(r0 + rows, nrow);
  const int nit = (r1 - r0 + U - 1) / U;
  const bool do_bias = bpart != nullptr && cx == 0;

  float bs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // 4 consecutive pixels x 8 channels of one row -> channel rows of LDS
  auto put = [&](uint16_t *dst, const uint4 (&r)[4]) {
    const uint16_t *e0 = (const uint16_t *)&r[0], *e1 = (const uint16_t *)&r[1];
    const uint16_t *e2 = (const uint16_t *)&r[2], *e3 = (const uint16_t *)&r[3];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      uint2 v;
      v.x = (uint32_t)e0[c] | ((uint32_t)e1[c] << 16);
      v.y = (uint32_t)e2[c] | ((uint32_t)e3[c] << 16);
      *(uint2 *)&dst[c * RP] = v;
    }
  };
  auto bias_add = [&](const uint4 (&r)[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t w4[4] = {r[e].x, r[e].y, r[e].z, r[e].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bs[2 * j] += __uint_as_float(w4[j] << 16);
        bs[2 * j + 1] += __uint_as_float(w4[j] & 0xFFFF0000u);
      }
    }
  };
  // rows outside the batch read row 0 and are zeroed (no branch around loads)
  auto fetch = [&](const uint16_t *base, int stride, int row, int quad, uint4 (&r)[4]) {
    const bool ok = row >= 0 && row < nrow;
    const uint16_t *src = base + ((size_t)(ok ? row : 0) * W + 4 * quad) * stride;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint4 v = *(const uint4 *)(src + (size_t)e * stride);
      r[e] = ok ? v : make_uint4(0, 0, 0, 0);
    }
  };
  const uint16_t *xb = a.x + a.xo + c0, *gyb = a.g + a.go + o0;
  // ring slot of image row `row`: rows r0 - 1, r0, ... take slots 0, 1, ...
  auto slot_of = [&](int row) { return (row - r0 + 1) % NR; };

  // prologue: zero pads, input rows r0 - 1 .. r0 + U, GY rows r0 .. r0 + U - 1
  for (int i = tid; i < NR * 32 + 1; i += NTH) *(uint4 *)&Is[i * RP] = make_uint4(0, 0, 0, 0);
  for (int q = tid; q < (U + 2) * W; q += NTH) {
    const int cg = q & 3, quad = (q >> 2) % (W / 4), u = (q >> 2) / (W / 4);
    uint4 r[4];
    fetch(xb + 8 * cg, a.xs, r0 - 1 + u, quad, r);
    put(&Is[(slot_of(r0 - 1 + u) * 32 + 8 * cg) * RP + 8 + 4 * quad], r);
  }
  for (int q = tid; q < NGO; q += NTH) {
    const int cg = q % GCG, quad = (q / GCG) % (W / 4), u = q / GCG / (W / 4);
    uint4 r[4];
    fetch(gyb + 8 * cg, a.gs, r0 + u, quad, r);
    put(&Gs[0][(u * NB + 8 * cg) * RP + 4 * quad], r);
    if (do_bias) bias_add(r);
  }

  floatx4 acc[9][NT];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[t][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  uint4 rin[IN_T][4], rgo[GO_T][4];
  __syncthreads();

  for (int it = 0; it < nit; ++it) {
    const int rb = r0 + it * U, buf = it & 1;
    const bool more = it + 1 < nit;
    if (more) {   // rows of the next iteration: input rb + U + 1 .., GY rb + U ..
#pragma unroll
      for (int j = 0; j < IN_T; ++j) {
        const int q = tid + NTH * j;
        if (q < NIN) {
          const int cg = q & 3, quad = (q >> 2) % (W / 4), u = (q >> 2) / (W / 4);
          fetch(xb + 8 * cg, a.xs, rb + U + 1 + u, quad, rin[j]);
        }
      }
#pragma unroll
      for (int j = 0; j < GO_T; ++j) {
        const int q = tid + NTH * j;
        if (q < NGO) {
          const int cg = q % GCG, quad = (q / GCG) % (W / 4), u = q / GCG / (W / 4);
          fetch(gyb + 8 * cg, a.gs, rb + U + u, quad, rgo[j]);
        }
      }
    }
    const int yb = rb % a.h, sb = (it * U) % NR;
#pragma unroll
    for (int kk = 0; kk < KS / KW; ++kk) {
      const int ks = kk * KW + grp;
      const int j0 = ks * 32 + fk, u = j0 / W, x0 = j0 % W;
      int y = yb + u;
      if (y >= a.h) y -= a.h;
      bf16x8 fb[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        fb[nt] = *(const bf16x8 *)&Gs[buf][(u * NB + wn * 16 * NT + nt * 16 + fr) * RP + x0];
#pragma unroll
      for (int dy = 0; dy < 3; ++dy) {
        const int yy = y + dy - 1;
        int s = sb + u + dy;
        if (s >= NR) s -= NR;
        const uint16_t *p = &Is[(s * 32 + wc * 16 + fr) * RP + 8 + x0];
        uint4 d = *(const uint4 *)p;
        uint32_t e = *(const uint32_t *)(p + 8), f = *(const uint32_t *)(p - 2);
        if (yy < 0 || yy >= a.h) {
          d = make_uint4(0, 0, 0, 0);
          e = f = 0;
        }
        const uint32_t s1 = __builtin_amdgcn_alignbit(d.y, d.x, 16);
        const uint32_t s2 = __builtin_amdgcn_alignbit(d.z, d.y, 16);
        const uint32_t s3 = __builtin_amdgcn_alignbit(d.w, d.z, 16);
        const uint4 am = make_uint4(__builtin_amdgcn_alignbit(d.x, f, 16), s1, s2, s3);
        const uint4 ap = make_uint4(s1, s2, s3, __builtin_amdgcn_alignbit(e, d.w, 16));
        const bf16x8 fm = __builtin_bit_cast(bf16x8, am), f0 = __builtin_bit_cast(bf16x8, d),
                     fp = __builtin_bit_cast(bf16x8, ap);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          acc[3 * dy][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fm, fb[nt], acc[3 * dy][nt], 0, 0, 0);
          acc[3 * dy + 1][nt] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(f0, fb[nt], acc[3 * dy + 1][nt], 0, 0, 0);
          acc[3 * dy + 2][nt] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(fp, fb[nt], acc[3 * dy + 2][nt], 0, 0, 0);
        }
      }
    }
    if (more) {
#pragma unroll
      for (int j = 0; j < IN_T; ++j) {
        const int q = tid + NTH * j;
        if (q < NIN) {
          const int cg = q & 3, quad = (q >> 2) % (W / 4), u = (q >> 2) / (W / 4);
          put(&Is[(slot_of(rb + U + 1 + u) * 32 + 8 * cg) * RP + 8 + 4 * quad], rin[j]);
        }
      }
#pragma unroll
      for (int j = 0; j < GO_T; ++j) {
        const int q = tid + NTH * j;
        if (q < NGO) {
          const int cg = q % GCG, quad = (q / GCG) % (W / 4), u = q / GCG / (W / 4);
          put(&Gs[buf ^ 1][(u * NB + 8 * cg) * RP + 4 * quad], rgo[j]);
          if (do_bias) bias_add(rgo[j]);
        }
      }
    }
    __syncthreads();
  }

  // groups 1 .. KW - 1 hand their sums to group 0 through LDS, three taps
  // at a time (the ring is free after the loop's last barrier)
  if (KW > 1) {
    float *xch = (float *)Is;   // [group - 1][3 taps][NT][4][256 lanes]
    static_assert((KW - 1) * 3 * NT * 4 * 256 * 4 <= IS_EL * 2, "exchange fits the ring");
#pragma unroll
    for (int t0 = 0; t0 < 9; t0 += 3) {
      if (grp > 0)
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              xch[((((grp - 1) * 3 + t) * NT + nt) * 4 + e) * 256 + (tid & 255)] =
                  acc[t0 + t][nt][e];
      __syncthreads();
      if (grp == 0)
#pragma unroll
        for (int g = 1; g < KW; ++g)
#pragma unroll
          for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
              for (int e = 0; e < 4; ++e)
                acc[t0 + t][nt][e] += xch[((((g - 1) * 3 + t) * NT + nt) * 4 + e) * 256 + tid];
      __syncthreads();
    }
  }
  const int N = a.co;
  if (grp == 0) {
    float *dst = a.part + (size_t)z * 9 * a.ci * N;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int c = c0 + wc * 16 + (lane >> 4) * 4 + e;
          const int o = o0 + wn * 16 * NT + nt * 16 + (lane & 15);
          dst[(size_t)(t * a.ci + c) * N + o] = acc[t][nt][e];
        }
  }
  if (do_bias) {   // threads tid = g (mod GCG) hold channel group g
    float *red = (float *)Is;   // NTH x 9 floats; the last barrier has passed
    static_assert(NTH * 9 * 4 <= IS_EL * 2, "bias tree fits the ring");
#pragma unroll
    for (int j = 0; j < 8; ++j) red[tid * 9 + j] = bs[j];
    __syncthreads();
    for (int h = NTH / GCG / 2; h > 0; h >>= 1) {
      if (tid / GCG < h)
#pragma unroll
        for (int j = 0; j < 8; ++j) red[tid * 9 + j] += red[(tid + h * GCG) * 9 + j];
      __syncthreads();
    }
    if (tid < GCG)
#pragma unroll
      for (int j = 0; j < 8; ++j) bpart[(size_t)z * N + o0 + 8 * tid + j] = red[tid * 9 + j];
  }
}

// Weight copies in k_conv_tile's fragment order, [n / 16][chunk of 32 k][tap]
// [lane][8] with lane = n % 16 + 16 (k % 32 / 8), of up to 16 convolutions at
// once (the parameter layout of the surrogate: conv k's weights at element
// off[k]): into wf for the forward pass (n = output, k = input channel) and
// wd for the input gradient (the other way round); either may be null.  One
// thread per lane vector.
struct ConvTable {
  int count;
  long long off[16];
  int ci[16], co[16];
};
__global__ void k_pack_weights(const uint16_t *w, uint16_t *wf, uint16_t *wd, ConvTable tb,
                               long long total) {
  long long i = (blockIdx.x * (long long)blockDim.x + threadIdx.x) * 8;
  if (i >= total) return;
  int k = 0;
  while (k < tb.count && i >= 9LL * tb.ci[k] * tb.co[k]) {
    i -= 9LL * tb.ci[k] * tb.co[k];
    ++k;
  }
  if (k >= tb.count) return;
  const int ci = tb.ci[k], co = tb.co[k];
  const uint16_t *src = w + tb.off[k];
  const int lane = (int)(i >> 3) & 63, q = (int)(i >> 9), t = q % 9;
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    uint16_t *dst = pass == 0 ? wf : wd;
    if (!dst) continue;
    const int nc = (pass == 0 ? ci : co) / 32;
    const int n = q / 9 / nc * 16 + (lane & 15), k0 = q / 9 % nc * 32 + (lane >> 4) * 8;
    uint4 v;
    uint16_t *e = (uint16_t *)&v;
#pragma unroll
    for (int j = 0; j < 8; ++j)
      e[j] = pass == 0 ? src[((long long)t * ci + k0 + j) * co + n]
                       : src[((long long)t * ci + n) * co + k0 + j];
    *(uint4 *)(dst + tb.off[k] + i) = v;
  }
}

// out[i] += sum over k of part[k][i] for i < n: the deterministic second half
// of the split reductions (weight and bias gradients, loss).  A block takes
// 16 outputs; its 16 thread groups sum the k = g, g + 16, ... in order, and
// the group sums are added in group order, so the result is fixed while
// 16 loads per output are in flight.
constexpr int kSumOut = 16, kSumGroups = 16;
__global__ __launch_bounds__(256) void k_sum_parts(const float *part, int nparts, long long n,
                                                   float *out) {
  const int o = threadIdx.x % kSumOut, g = threadIdx.x / kSumOut;
  const long long i = blockIdx.x * (long long)kSumOut + o;
  float s = 0.f;
  if (i < n)
#pragma unroll 8
    for (int k = g; k < nparts; k += kSumGroups) s += part[(size_t)k * n + i];
  __shared__ float sh[kSumGroups][kSumOut];
  sh[g][o] = s;
  __syncthreads();
  if (g == 0 && i < n) {
    float t = 0.f;
#pragma unroll
    for (int q = 0; q < kSumGroups; ++q) t += sh[q][o];
    out[i] += t;
  }
}

// out[0] += the sum of part[0 .. nparts): one block, thread t adding
// part[t], part[t + 256], ... (loads in flight together), then a fixed LDS
// tree; the loss's per-block sums.
__global__ __launch_bounds__(256) void k_sum_scalar(const float *part, int nparts, float *out) {
  float s = 0.f;
#pragma unroll 8
  for (int k = threadIdx.x; k < nparts; k += 256) s += part[k];
  __shared__ float sh[256];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] += sh[0];
}

// Partial sums of up to eight layers' weight and bias gradients in one launch:
// out[i] (+)= sum over k of part[k][i] for each segment of the table (blocks
// below s[0].blocks take segment 0, and so on).  A thread adds 4 consecutive
// outputs (16-byte loads); the block's `groups` thread groups (a power of two
// dividing 256) take k = g, g + groups, ... in order and the group sums are
// added in group order, so the result is fixed for a given shape.  Many
// groups serve few outputs with many partials, one group many outputs.  n, the
// pointers' element offsets: multiples of 4.
struct SumSeg {
  const float *part;
  long long n;
  float *out;
  int nparts, groups, blocks;
  int add;   // 1: out += sum, 0: out = sum
};
constexpr int kSumSegs = 16;
struct SumTable {
  int count;
  SumSeg s[kSumSegs];
};
__global__ __launch_bounds__(256) void k_sum_parts_v4(SumTable tb) {
  int seg = 0, b = blockIdx.x;
  while (seg + 1 < tb.count && b >= tb.s[seg].blocks) b -= tb.s[seg++].blocks;
  const SumSeg &sg = tb.s[seg];
  const float *part = sg.part;
  float *out = sg.out;
  const int nparts = sg.nparts, G = sg.groups, V = 256 / G;
  const long long n4 = sg.n / 4;
  const bool add = sg.add;
  const int g = threadIdx.x / V, vi = threadIdx.x - g * V;
  const long long i = (long long)b * V + vi;   // vector index
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  if (i < n4) {
    const float4 *p4 = (const float4 *)part + i;
#pragma unroll 4
    for (int k = g; k < nparts; k += G) {
      const float4 v = p4[(size_t)k * n4];
      acc.x += v.x;
      acc.y += v.y;
      acc.z += v.z;
      acc.w += v.w;
    }
  }
  __shared__ float4 sh[256];
  sh[threadIdx.x] = acc;
  __syncthreads();
  if (g == 0 && i < n4) {
    float4 t = sh[vi];
    for (int q = 1; q < G; ++q) {
      const float4 v = sh[q * V + vi];
      t.x += v.x;
      t.y += v.y;
      t.z += v.z;
      t.w += v.w;
    }
    float4 *o = (float4 *)out + i;
    if (add) {
      const float4 r = *o;
      t.x += r.x;
      t.y += r.y;
      t.z += r.z;
      t.w += r.w;
    }
    *o = t;
  }
}

// Bias gradient, first half: part[block][o] = sum of GY[p][o] over the
// block's chunk of pixels (co a multiple of 8, at most 256; gs, go multiples
// of 8).  Thread t takes channels 8 (t % (co / 8)) .. + 7 of the pixels
// p0 + t / (co / 8), + 256 / (co / 8), ... with 16-byte loads (the 256
// threads cover whole pixel rows, so a wavefront reads contiguous memory),
// then the pixel groups are added in a fixed tree order.  k_sum_parts adds
// the chunks into gb.
__global__ __launch_bounds__(256) void k_bias_grad(const uint16_t *g, int gs, int go, int npix,
                                                   int co, int chunk, float *part) {
  const int cv = co / 8, groups = 256 / cv;
  const int t = threadIdx.x, q = t % cv, grp = t / cv;
  const int p0 = blockIdx.x * chunk, p1 = min(p0 + chunk, npix);
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (grp < groups)
    for (int p = p0 + grp; p < p1; p += groups) {
      const uint4 v = *(const uint4 *)(g + (size_t)p * gs + go + 8 * q);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        s[2 * j] += __uint_as_float(w[j] << 16);
        s[2 * j + 1] += __uint_as_float(w[j] & 0xFFFF0000u);
      }
    }
  __shared__ float sh[256][9];
#pragma unroll
  for (int j = 0; j < 8; ++j) sh[t][j] = s[j];
  __syncthreads();
  int top = 1;
  while (top < groups) top <<= 1;
  for (int h = top / 2; h > 0; h >>= 1) {   // fixed tree over the pixel groups
    if (grp < h && grp + h < groups)
#pragma unroll
      for (int j = 0; j < 8; ++j) sh[t][j] += sh[t + h * cv][j];
    __syncthreads();
  }
  if (grp == 0)
#pragma unroll
    for (int j = 0; j < 8; ++j) part[(size_t)blockIdx.x * co + 8 * q + j] = sh[t][j];
}

// Elementwise kernels over groups of 8 channels (16 bytes; channel counts,
// strides and offsets are multiples of 8): thread i takes group i % (c / 8)
// of pixel i / (c / 8).
struct Bf8 {
  uint16_t v[8];
};
__device__ __forceinline__ Bf8 ld8(const uint16_t *p) {
  Bf8 r;
  *(uint4 *)r.v = *(const uint4 *)p;
  return r;
}
__device__ __forceinline__ void st8(uint16_t *p, const Bf8 &r) { *(uint4 *)p = *(const uint4 *)r.v; }

// 2 x 2 average pooling (h, w: input size, even).
__global__ void k_pool_fwd(const uint16_t *x, int xs, int xo, int n, int h, int w, int c,
                           uint16_t *y) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const int cg = c / 8, ho = h / 2, wo = w / 2;
  if (i >= (long long)n * ho * wo * cg) return;
  const int g = (int)(i % cg);
  const long long pix = i / cg;
  const int ox = (int)(pix % wo), oy = (int)((pix / wo) % ho), b = (int)(pix / ((long long)wo * ho));
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int dy = 0; dy < 2; ++dy)
#pragma unroll
    for (int dx = 0; dx < 2; ++dx) {
      const Bf8 v = ld8(x + ((size_t)(b * h + 2 * oy + dy) * w + 2 * ox + dx) * xs + xo + 8 * g);
#pragma unroll
      for (int j = 0; j < 8; ++j) s[j] += bf2f(v.v[j]);
    }
  Bf8 r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r.v[j] = f2bf(0.25f * s[j]);
  st8(y + pix * c + 8 * g, r);
}

// Gradient of the pooling, written into (or added to) a slice of gx; with
// mask set, zero where mask <= 0 (mask has gx's stride and offset: the ReLU
// of the layer that produced the pooled input; k_up_bwd likewise).
__global__ void k_pool_bwd(const uint16_t *gy, int n, int h, int w, int c, uint16_t *gx, int gxs,
                           int gxo, int accumulate, const uint16_t *mask) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const int cg = c / 8;
  if (i >= (long long)n * h * w * cg) return;
  const int g = (int)(i % cg);
  const long long pix = i / cg;
  const int px = (int)(pix % w), py = (int)((pix / w) % h), b = (int)(pix / ((long long)w * h));
  const int ho = h / 2, wo = w / 2;
  const Bf8 v = ld8(gy + ((size_t)(b * ho + py / 2) * wo + px / 2) * c + 8 * g);
  uint16_t *o = gx + (size_t)pix * gxs + gxo + 8 * g;
  Bf8 old{};
  if (accumulate) old = ld8(o);
  Bf8 mk{};
  if (mask) mk = ld8(mask + (o - gx));
  Bf8 r;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    float t = 0.25f * bf2f(v.v[j]);
    if (accumulate) t += bf2f(old.v[j]);
    if (mask && !(bf2f(mk.v[j]) > 0.f)) t = 0.f;
    r.v[j] = f2bf(t);
  }
  st8(o, r);
}

// Nearest 2x upsampling (h, w: input size) into a channel slice of y.
__global__ void k_up_fwd(const uint16_t *x, int n, int h, int w, int c, uint16_t *y, int ys,
                         int yo) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const int H = 2 * h, W = 2 * w, cg = c / 8;
  if (i >= (long long)n * H * W * cg) return;
  const int g = (int)(i % cg);
  const long long pix = i / cg;
  const int px = (int)(pix % W), py = (int)((pix / W) % H), b = (int)(pix / ((long long)W * H));
  st8(y + (size_t)pix * ys + yo + 8 * g,
      ld8(x + ((size_t)(b * h + py / 2) * w + px / 2) * c + 8 * g));
}

__global__ void k_up_bwd(const uint16_t *gy, int gys, int gyo, int n, int h, int w, int c,
                         uint16_t *gx, const uint16_t *mask) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const int cg = c / 8;
  if (i >= (long long)n * h * w * cg) return;
  const int g = (int)(i % cg);
  const long long pix = i / cg;
  const int px = (int)(pix % w), py = (int)((pix / w) % h), b = (int)(pix / ((long long)w * h));
  const int W = 2 * w;
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int dy = 0; dy < 2; ++dy)
#pragma unroll
    for (int dx = 0; dx < 2; ++dx) {
      const Bf8 v =
          ld8(gy + ((size_t)(b * 2 * h + 2 * py + dy) * W + 2 * px + dx) * gys + gyo + 8 * g);
#pragma unroll
      for (int j = 0; j < 8; ++j) s[j] += bf2f(v.v[j]);
    }
  if (mask) {
    const Bf8 mk = ld8(mask + pix * c + 8 * g);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (!(bf2f(mk.v[j]) > 0.f)) s[j] = 0.f;
  }
  Bf8 r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r.v[j] = f2bf(s[j]);
  st8(gx + pix * c + 8 * g, r);
}

// g *= (y > 0) over a channel slice [npix][c] of both tensors.
__global__ void k_relu_bwd(const uint16_t *y, int ys, int yo, uint16_t *g, int gs, int go,
                           long long npix, int c) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const int cg = c / 8;
  if (i >= npix * cg) return;
  const long long p = i / cg;
  const int k = (int)(i % cg);
  const Bf8 yv = ld8(y + p * ys + yo + 8 * k);
  uint16_t *gp = g + p * gs + go + 8 * k;
  Bf8 gv = ld8(gp);
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (!(bf2f(yv.v[j]) > 0.f)) gv.v[j] = 0;
  st8(gp, gv);
}

// Masked mean-squared error over the first `cu` (<= 8) channels of pred
// (stride ps): loss[block] = the block's sum of mask (pred - t)^2 / count
// (k_sum_parts adds the blocks); grad = 2 mask (pred - t) / count (bf16,
// dense: gs channels, zero beyond cu).  t: FP32 [npix][cu]; mask FP32
// [npix].  One thread per 16-byte vector of grad (gs / 8 per pixel, so a
// wavefront stores contiguous memory); the first of a pixel reads its first
// 8 channels of pred (ps a multiple of 8, 16-byte aligned) and does the sums.
__global__ __launch_bounds__(256) void k_mse(const uint16_t *pred, int ps, const float *t,
                                             const float *mask, long long npix, int cu,
                                             float inv_count, uint16_t *grad, int gs,
                                             float *loss) {
  const int vp = gs / 8;   // vectors per pixel
  const long long q = blockIdx.x * 256LL + threadIdx.x;
  float l = 0.f;
  if (q < npix * vp) {
    const long long p = q / vp;
    uint4 out = make_uint4(0, 0, 0, 0);
    if (q - p * vp == 0) {
      const float mk = mask[p];
      const Bf8 pv = ld8(pred + p * ps);
      Bf8 gv;
#pragma unroll
      for (int ch = 0; ch < 8; ++ch) {
        float g = 0.f;
        if (ch < cu) {
          const float d = bf2f(pv.v[ch]) - t[p * cu + ch];
          l += mk * d * d;
          g = 2.f * mk * d * inv_count;
        }
        gv.v[ch] = f2bf(g);
      }
      out = *(const uint4 *)gv.v;
    }
    ((uint4 *)grad)[q] = out;
  }
  for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
  __shared__ float part[4];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = l;
  __syncthreads();
  if (threadIdx.x == 0) loss[blockIdx.x] = (part[0] + part[1] + part[2] + part[3]) * inv_count;
}

// Adam on FP32 master weights; refreshes the bf16 copy (may be null).
__global__ void k_adam(float *w, float *m, float *v, const float *g, uint16_t *wb, long long n,
                       float lr, float b1, float b2, float eps, float c1, float c2) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float wi = w[i] - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
  w[i] = wi;
  if (wb) wb[i] = f2bf(wi);
}

// float -> bf16 copy
__global__ void k_to_bf16(const float *a, uint16_t *b, long long n) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i < n) b[i] = f2bf(a[i]);
}

}  // namespace nn
}  // namespace lbm
