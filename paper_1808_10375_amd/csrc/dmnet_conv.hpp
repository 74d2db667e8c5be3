// dmnet_conv.hpp -- the 3x3 convolutions of the warm-start network on the
// matrix cores: forward and data gradient as implicit GEMMs with bfloat16
// operands and float32 accumulation (v_mfma_f32_16x16x32_bf16), for channel
// counts that are multiples of 32.
//
// Operands live in memory as the matrix cores read them:
//   activations (and output gradients), "chunk layout": bfloat16
//     [C / 32][n * H * W][32], 32 channels of a pixel contiguous (64 bytes).
//     The producing kernel rounds (to nearest even) and writes this layout,
//     so no pass of its own converts or transposes an activation, and a
//     concatenation is just two lists of chunks (the first may be read at
//     half resolution, which is the nearest 2x upsampling).
//   weights, "fragment order": bfloat16 [Co / 16][9][chunks][64][8], 16
//     output channels x 32 input channels of one tap as the 64 lanes of an A
//     operand hold them.
// The products run tap by tap and chunk by chunk inside a tap, the order of
// the channel-last kernel in dmnet_kernels.hpp, so both give the same bits.
#pragma once
#include "dmnet_kernels.hpp"

namespace dmn {

constexpr int kChunk = 32;  // channels per chunk (the K step of the product)

// Fragment-order copies of one convolution's bfloat16 weights w[Co][Ci][9]:
//   wf: forward (rows: output channels, chunks: input channels)
//   wt: data gradient (rows: input channels, chunks: output channels, taps
//       flipped)
// Co and Ci multiples of 32.
__global__ void k_pack3(const uint16_t* __restrict__ w, int co, int ci,
                        uint16_t* __restrict__ wf, uint16_t* __restrict__ wt) {
  const long total = (long)co * ci * 9;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < 2 * total;
       e += (long)gridDim.x * blockDim.x) {
    const bool fwd = e < total;
    const long f = fwd ? e : e - total;
    const int nc = (fwd ? ci : co) / kChunk;
    const int q = (int)(f & 7), lane = (int)(f >> 3) & 63;
    const long g = f >> 9;
    const int ch = (int)(g % nc), t = (int)(g / nc % 9), rt = (int)(g / nc / 9);
    const int row = rt * 16 + (lane & 15), k = ch * kChunk + 8 * (lane >> 4) + q;
    if (fwd) wf[f] = w[((long)row * ci + k) * 9 + t];
    else wt[f] = w[((long)k * ci + row) * 9 + (8 - t)];
  }
}

// ---------------------------------------------------------------------------
// y[o][P] = b[o] + sum_{c, t} w[o][c][t] x[c][P + off_t] (zero padding),
// optional ReLU, over all n samples; to y16 (chunk layout) and / or y32
// (float32 NCHW, sample stride y_ns), either may be NULL.
//
// Pixels are numbered q = (smp (H + 1) + i) (W + 1) + j with one zero row
// after each sample and one zero column after each row, so that a tap is a
// constant offset of q and a run of TP consecutive q needs one run of
// TP + 2 PW + 2 inputs (PW = W + 1) -- or, when the rows are longer than the
// tile, three runs of TP + 2.  A block stages that run once for all channels
// and reads every tap's operand there: 16 lanes x 4 parts of 16 bytes are 1 KB of
// consecutive LDS, free of bank conflicts.  Where LDS does not hold all channels
// (ROWS), it takes one tap row after another, TP + 2 inputs of all channels, or
// of `grp` chunks at a time, which come again for each tap of the row (the
// products run tap by tap).  The weights pass through LDS too,
// kConvG steps (tap, chunk) at a time in two buffers, the group after next on
// its way to registers.  Outputs at padding positions are dropped (3% of the
// work at W = 64, 27% at W = 8).
// Wave tile: OT x 16 output channels by PT x 16 positions; WO of the block's
// NW waves side by side in channels, NW / WO in positions.  At OT = PT = 4 a
// step of 16 products (256 cycles of a SIMD) reads 8 KB of LDS per wave, which
// is the LDS rate; what bounds a block is the chain stage, products, store,
// hidden by the other blocks of its compute unit.  64 samples of the 4-level
// 32-channel network at 64 x 64: 22-27 us for 32 -> 32 channels at 64^2, 42 us
// for 96 -> 32, 42 us for 192 -> 64 at 32^2.  With every wave reading its
// operands of every tap from the caches (k_conv3_mfma_cl), and a pass that
// converts and transposes each input, the forward pass over 300 frames took
// 4.4 ms against 2.0.  16 samples of 64 x 64 with 128, 256 and 512 channels take
// 1.04 ms with ROWS; 1.52 ms with that kernel, and 1.68 ms when the groups were
// staged with all three tap rows for every tap.
// ---------------------------------------------------------------------------
constexpr int kConvG = 4;  // steps per weight group

template <int OT, int PT, int WO, int NW>
struct ConvCfg {
  static constexpr int TP = (NW / WO) * PT * 16;  // positions per block
  static constexpr int TO = WO * OT * 16;        // output channels per block
  static constexpr int WG = kConvG * TO / 16 * 64;  // 16-byte parts of a weight group
};

// distance between the three tap rows of a staged run
__host__ __device__ inline int conv_row_step(int TP, int W) {
  return W + 1 < TP + 2 ? W + 1 : TP + 2;
}

// q / d of 0 <= q < 2^31 by a multiplication (Granlund and Montgomery, "Division
// by invariant integers using multiplication", PLDI 1994): a block's set-up
// divides about ten positions per thread, which with real divisions took
// longer than its products
struct FastDiv {
  uint32_t m, s, d;
  FastDiv() = default;
  explicit FastDiv(uint32_t div) : d(div) {
    for (s = 0; (1u << s) < div; ++s) {}
    m = (uint32_t)((((uint64_t)1 << 32) * (((uint64_t)1 << s) - div)) / div + 1);
  }
  __device__ __forceinline__ int div(int q) const {
    return (int)((__umulhi((uint32_t)q, m) + (uint32_t)q) >> s);
  }
};

struct ConvSrc {
  const uint16_t* p;  // chunk layout
  int nch;            // chunks
  int up;             // 1: stored at half resolution
};

typedef unsigned int nb_u32x4 __attribute__((ext_vector_type(4)));

template <int OT, int PT, int WO, int NW, bool ROWS>
__global__ __launch_bounds__(64 * NW) void k_conv3(ConvSrc s0, ConvSrc s1, int H, int W, int n,
                                               FastDiv dps, FastDiv dpw, int grp,
                                               const uint16_t* __restrict__ A,
                                               const float* __restrict__ bias,
                                               uint16_t* __restrict__ y16,
                                               float* __restrict__ y32, long y_ns, int relu) {
  using C = ConvCfg<OT, PT, WO, NW>;
  constexpr int TP = C::TP, WG = C::WG, NT = 64 * NW, NA = WG / NT, G = kConvG;
  extern __shared__ nb_u32x4 lds[];
  nb_u32x4* const ws = lds;           // [2][step of the group][16 channels][64]
  nb_u32x4* const xs = lds + 2 * WG;  // [chunk of the group][position][4 parts]
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wo = wave % WO, wp = wave / WO;
  const int PW = W + 1, PS = (H + 1) * PW, HW = H * W;
  const int RS = conv_row_step(TP, W);
  const int nx = (TP + 2 + (ROWS ? 0 : 2 * RS)) * 4;  // 16-byte parts of inputs per chunk
  const int q0 = blockIdx.x * TP, o0 = blockIdx.y * C::TO;
  const int n0 = s0.nch, up = s0.up, nch = n0 + s1.nch;
  const int H0 = H >> up, W0 = W >> up;
  const nb_u32x4* __restrict__ b0 = reinterpret_cast<const nb_u32x4*>(s0.p);
  const nb_u32x4* __restrict__ b1 = reinterpret_cast<const nb_u32x4*>(s1.p);
  const size_t st0 = (size_t)n * H0 * W0 * 4, st1 = (size_t)n * HW * 4;
  const nb_u32x4 zero = {0u, 0u, 0u, 0u};
  // chunks c0 .. c1 - 1 of the run (of its tap row dy) to LDS, seven parts a
  // thread in flight
  auto stage = [&](int c0, int c1, int dy) {
    constexpr int U = 7;
    for (int i0 = t; i0 < nx; i0 += NT * U) {
      size_t p0[U], p1[U];
      bool ok[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int id = i0 + NT * k, u = id >> 2;
        int q;
        if (ROWS) {
          q = q0 + (dy - 1) * PW - 1 + u;
        } else if (RS == PW) {
          q = q0 - PW - 1 + u;
        } else {
          const int seg = u / (TP + 2);
          q = q0 + (seg - 1) * PW - 1 + (u - seg * (TP + 2));
        }
        const int qc = q < 0 ? 0 : q;
        const int smp = dps.div(qc), r = qc - smp * PS;
        const int y = dpw.div(r), x = r - y * PW;
        ok[k] = id < nx && q >= 0 && smp < n && y < H && x < W;
        p0[k] = (size_t)((smp * H0 + (y >> up)) * W0 + (x >> up)) * 4 + (t & 3);
        p1[k] = (size_t)((smp * H + y) * W + x) * 4 + (t & 3);
      }
      for (int c = c0; c < c1; ++c) {
        nb_u32x4 v[U];
        if (c < n0) {
#pragma unroll
          for (int k = 0; k < U; ++k) v[k] = ok[k] ? b0[c * st0 + p0[k]] : zero;
        } else {
#pragma unroll
          for (int k = 0; k < U; ++k) v[k] = ok[k] ? b1[(c - n0) * st1 + p1[k]] : zero;
        }
#pragma unroll
        for (int k = 0; k < U; ++k)
          if (i0 + NT * k < nx) xs[(c - c0) * nx + i0 + NT * k] = v[k];
      }
    }
  };
  // weights: step s = tap * nch + chunk of 16-channel tile o is at (o steps + s) 64
  const int steps = 9 * nch, groups = (steps + G - 1) / G;
  const nb_u32x4* __restrict__ aw =
      reinterpret_cast<const nb_u32x4*>(A) + (size_t)(o0 / 16) * steps * 64 + lane;
  nb_u32x4 ar[NA];
  auto load_w = [&](int g) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int r = wave + NW * i;  // 64-part row: step r / (TO / 16), tile r % (TO / 16)
      const int s = g * G + r / (C::TO / 16);
      ar[i] = s < steps ? aw[((size_t)(r % (C::TO / 16)) * steps + s) * 64] : zero;
    }
  };
  auto store_w = [&](int g) {
#pragma unroll
    for (int i = 0; i < NA; ++i) ws[(g & 1) * WG + t + NT * i] = ar[i];
  };
  nb_f32x4 acc[OT][PT];
#pragma unroll
  for (int o = 0; o < OT; ++o)
#pragma unroll
    for (int p = 0; p < PT; ++p) acc[o][p] = nb_f32x4{0.f, 0.f, 0.f, 0.f};
  const int xb = (wp * PT * 16 + (lane & 15)) * 4 + (lane >> 4);
  const int ab = wo * OT * 64 + lane;
  load_w(0);
  stage(0, ROWS ? grp : nch, 0);
  store_w(0);
  if (groups > 1) load_w(1);
  __syncthreads();
  int tap = 0, ch = 0, cg = 0;  // tap, chunk and (ROWS) chunk within its group
  for (int g = 0; g < groups; ++g) {
    // the other weight buffer's readers passed the barrier that ended group g - 1
    if (g + 1 < groups) store_w(g + 1);
    if (g + 2 < groups) load_w(g + 2);
#pragma unroll
    for (int d = 0; d < G; ++d) {
      const int s = g * G + d;
      if (s < steps) {
        const int dy = tap / 3, dx = tap - 3 * dy;
        if (ROWS && s > 0 && cg == 0 && (grp < nch || dx == 0)) {
          __syncthreads();
          stage(ch, ch + grp < nch ? ch + grp : nch, dy);
          __syncthreads();
        }
        const int xo = xb + (ROWS ? cg : ch) * nx + ((ROWS ? 0 : dy * RS) + dx) * 4;
        nb_s16x8 a[OT], b[PT];
#pragma unroll
        for (int o = 0; o < OT; ++o)
          a[o] = __builtin_bit_cast(nb_s16x8,
                                    ws[(g & 1) * WG + d * (C::TO / 16 * 64) + ab + o * 64]);
#pragma unroll
        for (int p = 0; p < PT; ++p) b[p] = __builtin_bit_cast(nb_s16x8, xs[xo + p * 64]);
#pragma unroll
        for (int o = 0; o < OT; ++o)
#pragma unroll
          for (int p = 0; p < PT; ++p) acc[o][p] = nb_mma(a[o], b[p], acc[o][p]);
        if (ROWS && ++cg == grp) cg = 0;
        if (++ch == nch) { ch = cg = 0; ++tap; }
      }
    }
    __syncthreads();
  }
  const int ob = o0 + wo * OT * 16 + 4 * (lane >> 4);
#pragma unroll
  for (int p = 0; p < PT; ++p) {
    const int q = q0 + (wp * PT + p) * 16 + (lane & 15);
    const int smp = dps.div(q), r = q - smp * PS;
    const int i = dpw.div(r), j = r - i * PW;
    if (smp >= n || i >= H || j >= W) continue;
    const int pix = i * W + j;
#pragma unroll
    for (int o = 0; o < OT; ++o) {
      const int oc = ob + o * 16;
      float v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        v[k] = acc[o][p][k] + (bias ? bias[oc + k] : 0.f);
        if (relu) v[k] = fmaxf(v[k], 0.f);
      }
      if (y16) {
        const uint2 w = make_uint2(
            (uint32_t)f_to_bf16_bits(v[0]) | ((uint32_t)f_to_bf16_bits(v[1]) << 16),
            (uint32_t)f_to_bf16_bits(v[2]) | ((uint32_t)f_to_bf16_bits(v[3]) << 16));
        *reinterpret_cast<uint2*>(y16 + (((size_t)(oc / 32) * n + smp) * HW + pix) * 32 +
                                  oc % 32) = w;
      }
      if (y32) {
        float* __restrict__ yn = y32 + (long)smp * y_ns + pix;
#pragma unroll
        for (int k = 0; k < 4; ++k) yn[(long)(oc + k) * HW] = v[k];
      }
    }
  }
}

// The network's first convolution (one input channel, 3x3, ReLU): its 9
// products fit one K step, whose operands each lane gathers as k_conv3_mfma
// does (the same bits); it is bound by its output.  yc a multiple of 32.
// Block: 4 waves x 64 pixels x 32 output channels.
// grid (ceil(n H W / 256), yc / 32)
__global__ __launch_bounds__(256) void k_conv3_first(const float* __restrict__ x, int H, int W,
                                                     long x_ns, int n,
                                                     const uint16_t* __restrict__ w,
                                                     const float* __restrict__ bias,
                                                     uint16_t* __restrict__ y16,
                                                     float* __restrict__ y32, long y_ns) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int HW = H * W, NP = n * HW;
  const int o0 = blockIdx.y * 32, kb = 8 * (lane >> 4);
  nb_s16x8 a[2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int e = 0; e < 8; ++e)
      a[rt][e] = kb + e < 9 ? (short)w[(o0 + 16 * rt + (lane & 15)) * 9 + kb + e] : (short)0;
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) {
    const int P = blockIdx.x * 256 + wave * 64 + 16 * ct + (lane & 15);
    const bool ok = P < NP;
    const int smp = ok ? P / HW : 0;
    const int p = ok ? P - smp * HW : 0;
    const int i = p / W, j = p - i * W;
    nb_s16x8 b;
#pragma unroll
    for (int e = 0; e < 8; ++e)
      b[e] = (short)f_to_bf16_bits(ok ? im2col3(x, x_ns, 1, H, W, smp, i, j, kb + e, 9) : 0.f);
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      const nb_f32x4 acc = nb_mma(a[rt], b, nb_f32x4{0.f, 0.f, 0.f, 0.f});
      const int oc = 16 * rt + 4 * (lane >> 4);
      float v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = fmaxf(acc[k] + bias[o0 + oc + k], 0.f);
      if (!ok) continue;
      *reinterpret_cast<uint2*>(y16 + ((size_t)blockIdx.y * NP + P) * 32 + oc) = make_uint2(
          (uint32_t)f_to_bf16_bits(v[0]) | ((uint32_t)f_to_bf16_bits(v[1]) << 16),
          (uint32_t)f_to_bf16_bits(v[2]) | ((uint32_t)f_to_bf16_bits(v[3]) << 16));
      if (y32) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          y32[(long)smp * y_ns + (long)(o0 + oc + k) * HW + p] = v[k];
      }
    }
  }
}

// 2x2 average of src (float32, C channels, H x W, sample stride s_ns) in
// chunk layout, and in float32 where dst is given; C a multiple of 32.  One
// thread per
// (8 channels, output pixel), pixels fastest.
__global__ void k_avgpool2_chunk(const float* __restrict__ src, long s_ns,
                                 uint16_t* __restrict__ d16, float* __restrict__ dst, long d_ns,
                                 int C, int H, int W, int n) {
  const int Ho = H / 2, Wo = W / 2, HWo = Ho * Wo;
  const long np = (long)n * HWo, total = np * (C / 8);
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < total;
       e += (long)gridDim.x * blockDim.x) {
    const long P = e % np;
    const int c8 = (int)(e / np) * 8;
    const int smp = (int)(P / HWo), p = (int)(P - (long)smp * HWo);
    const int i = p / Wo, j = p - i * Wo;
    const float* __restrict__ s = src + smp * s_ns + (long)c8 * H * W + (2 * i) * W + 2 * j;
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const float* __restrict__ sk = s + (long)k * H * W;
      v[k] = 0.25f * (sk[0] + sk[1] + sk[W] + sk[W + 1]);
      if (dst) dst[smp * d_ns + (long)(c8 + k) * HWo + p] = v[k];
    }
    uint32_t u[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      u[k] = (uint32_t)f_to_bf16_bits(v[2 * k]) | ((uint32_t)f_to_bf16_bits(v[2 * k + 1]) << 16);
    *reinterpret_cast<uint4*>(d16 + ((size_t)(c8 / 32) * np + P) * 32 + c8 % 32) =
        make_uint4(u[0], u[1], u[2], u[3]);
  }
}

// x (float32 [n][C][H*W], sample stride x_ns) in chunk layout, C a multiple of
// 32
__global__ void k_to_chunk16(const float* __restrict__ x, int C, int HW, long x_ns, int n,
                             uint16_t* __restrict__ d16) {
  const long np = (long)n * HW, total = np * (C / 8);
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < total;
       e += (long)gridDim.x * blockDim.x) {
    const long P = e % np;
    const int c8 = (int)(e / np) * 8;
    const int smp = (int)(P / HW), p = (int)(P - (long)smp * HW);
    const float* __restrict__ s = x + (long)smp * x_ns + (long)c8 * HW + p;
    uint32_t u[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float a = s[(long)(2 * k) * HW], b = s[(long)(2 * k + 1) * HW];
      u[k] = (uint32_t)f_to_bf16_bits(a) | ((uint32_t)f_to_bf16_bits(b) << 16);
    }
    *reinterpret_cast<uint4*>(d16 + ((size_t)(c8 / 32) * np + P) * 32 + c8 % 32) =
        make_uint4(u[0], u[1], u[2], u[3]);
  }
}

// ---------------------------------------------------------------------------
// What the backward pass of a 3x3 convolution needs of its output gradient g
// (float32 [n][C][H][W], sample stride g_ns), in one pass over it: g plus,
// where gp is given, the gradient of a 2x2 average pooling (0.25 gp of the
// pooled pixel), zero where the activation is not positive, as
//   dz16  chunk layout (data gradient), dzn  bfloat16 NCHW (weight gradient),
//   dbp[block][c]  the block's float32 sums (bias gradient, unrounded).
// The five kernels that did this (pooling gradient, mask, two conversions,
// bias sums) read and wrote the gradient seven times.
// Block: 32 channels x 64 pixels a step, kPrepPix pixels; C a multiple of 32, H*W
// of 64, W of 8.  grid (ceil(n H W / kPrepPix), C / 32)
// ---------------------------------------------------------------------------
constexpr int kPrepPix = 256;
__global__ __launch_bounds__(256) void k_grad_prep(const float* __restrict__ g, long g_ns,
                                                   const float* __restrict__ act, long a_ns,
                                                   const float* __restrict__ gp, long gp_ns,
                                                   int C, int H, int W, int n,
                                                   uint16_t* __restrict__ dz16,
                                                   uint16_t* __restrict__ dzn,
                                                   float* __restrict__ dbp) {
  __shared__ uint16_t tile[64][32 + 8];  // [pixel][channel]
  const int t = threadIdx.x, cl = t >> 3, c = blockIdx.y * 32 + cl;
  const int HW = H * W, NP = n * HW;
  float sum = 0.f;
  for (int P0 = blockIdx.x * kPrepPix; P0 < min(NP, (int)(blockIdx.x + 1) * kPrepPix); P0 += 64) {
    const int smp = P0 / HW, p = P0 - smp * HW + 8 * (t & 7);
    const long off = (long)c * HW + p;
    const float4* __restrict__ gs = reinterpret_cast<const float4*>(g + smp * g_ns + off);
    const float4* __restrict__ as = reinterpret_cast<const float4*>(act + smp * a_ns + off);
    const float4 g0 = gs[0], g1 = gs[1], a0 = as[0], a1 = as[1];
    float v[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
    const float a[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
    if (gp) {
      const int i = p / W, j = p - i * W;
      const float* __restrict__ q =
          gp + smp * gp_ns + (long)c * (HW / 4) + (i / 2) * (W / 2) + j / 2;
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] += 0.25f * q[k / 2];
    }
    uint16_t h[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (!(a[k] > 0.f)) v[k] = 0.f;
      sum += v[k];
      h[k] = f_to_bf16_bits(v[k]);
    }
    uint32_t u[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = (uint32_t)h[2 * k] | ((uint32_t)h[2 * k + 1] << 16);
    *reinterpret_cast<uint4*>(dzn + ((long)smp * C + c) * HW + p) =
        make_uint4(u[0], u[1], u[2], u[3]);
#pragma unroll
    for (int k = 0; k < 8; ++k) tile[8 * (t & 7) + k][cl] = h[k];
    __syncthreads();
    // 64 pixels x 32 channels are 4 KB of consecutive chunk layout
    *reinterpret_cast<uint4*>(dz16 + ((size_t)blockIdx.y * NP + P0) * 32 + t * 8) =
        *reinterpret_cast<const uint4*>(&tile[t >> 2][8 * (t & 3)]);
    __syncthreads();
  }
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) sum += __shfl_xor(sum, o, 64);
  if ((t & 7) == 0) dbp[(long)blockIdx.x * C + c] = sum;
}

// db[c] = sum over blocks of dbp[block][c]; one block of 256 threads per c
__global__ __launch_bounds__(256) void k_bias_sum(const float* __restrict__ dbp, int blocks,
                                                  int C, float* __restrict__ db) {
  __shared__ float red[4];
  const int c = blockIdx.x, t = threadIdx.x;
  float s = 0.f;
  for (int b = t; b < blocks; b += 256) s += dbp[(long)b * C + c];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((t & 63) == 0) red[t >> 6] = s;
  __syncthreads();
  if (t == 0) db[c] = (red[0] + red[1]) + (red[2] + red[3]);
}

}  // namespace dmn
