// dm_mfma.hpp -- the BF16x3 precision form of the view update for F = 128:
// the 2-D DFT as dense complex matrix products with the DFT matrix W on the
// matrix cores (v_mfma_f32_16x16x32_bf16), every real product split into
// hi*hi + hi*lo + lo*hi of bfloat16 pieces with float32 accumulation.  The
// modulus scale, error norms and updates stay float32.
//
// Three kernels around the spectrum buffer T [N][M][F][F]:
//   (1) k_mf_rows_fwd  T = Z W            Z = 2 P O - psi      (Eqs. 2-3)
//   (2) k_mf_cols      U = W T, modulus projection (definition of F_c),
//                      V = conj(W) U' / F^2, written back over T
//   (3) k_mf_rows_inv  Z' = V conj(W), psi' = psi + beta (Z' - P O), the
//                      per-view object numerator and eps_psi partials
// All three are persistent.  Wave w of a block forms the outputs 16 w .. 16 w
// + 15 of every line, so its part of the split W (real/imaginary x hi/lo, 16
// fragments, 64 registers) is loaded once and stays in registers.  The lines
// come 16 at a time: the block reads them along memory, splits every value
// once and writes the A fragments of the 16 lines to LDS (16 KB, two buffers
// in turn, one barrier per 16 lines, the next lines split while the products
// of the last run), from which all eight waves multiply.
// At 700 x 5 x 128^2 (700 GFLOP a pass of the three, 0.28 ms at the matrix
// peak) they take 276, 382 and 334 us, matrix cores busy 30, 47 and 24% of
// the time; the rest is the latency of a step, with one block of eight waves
// a compute unit (two blocks would need 128 registers a thread, and their
// spills' waits cost more).  With W in LDS and each wave loading its own
// operand fragments (64 bytes a lane, rows 1 KB apart; in the column kernel
// every wave loading and splitting all lines) they took 352, 662 and 383 us.
//
// Operand layout of v_mfma_f32_16x16x32_bf16 (one wave, 64 lanes):
//   A (16 x 32):  lane l holds row l%16, k = 8*(l/16) + e, e = 0..7
//   B (32 x 16):  lane l holds col l%16, k = 8*(l/16) + e
//   C (16 x 16):  lane l holds col l%16, rows 4*(l/16) + r, r = 0..3
// W is stored in B-fragment order, Wf[mat][ks][nt][lane] (16 bytes each),
// mat = 0..3 for Re hi, Re lo, Im hi, Im lo; because W is symmetric the
// same fragment also serves as the A operand of row tile nt.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dm_kernels.hpp"

namespace dmk {

typedef __bf16 mf_bf16x8 __attribute__((ext_vector_type(8)));
typedef float mf_f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t mf_u32x4 __attribute__((ext_vector_type(4)));

constexpr int kMfF = 128;                    // frame edge of this form
constexpr int kMfKs = kMfF / 32;             // k steps of 32
constexpr int kMfNt = kMfF / 16;             // 16-wide tiles
constexpr int kMfFrag = kMfKs * kMfNt * 64;  // uint4 per matrix
constexpr int kMfWords = 4 * kMfFrag;        // uint4 of the whole table (128 KB)
constexpr int kMfMaxModes = 8;

// float -> bfloat16 bits, round to nearest even (the conversion gfx950 does
// in hardware, two values per v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t mf_bf16_rne(float f) {
  return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)f);
}

__device__ __forceinline__ mf_u32x4 mf_neg(mf_u32x4 v) {
  return v ^ 0x80008000u;
}

__device__ __forceinline__ mf_f32x4 mf_mma(mf_u32x4 a, mf_u32x4 b, mf_f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(mf_bf16x8, a),
                                                 __builtin_bit_cast(mf_bf16x8, b), c, 0, 0, 0);
}

// c += a * b with the three-term split (a, b given as hi/lo pieces)
__device__ __forceinline__ mf_f32x4 mf_mma3(mf_u32x4 ah, mf_u32x4 al, mf_u32x4 bh, mf_u32x4 bl,
                                            mf_f32x4 c) {
  c = mf_mma(ah, bh, c);
  c = mf_mma(ah, bl, c);
  c = mf_mma(al, bh, c);
  return c;
}

// A operand of a complex product, split: re, im and -im pieces
struct MfA {
  mf_u32x4 rh, rl, ih, il;
};

// acc_re += Ar Wr - Ai Wi ; acc_im += Ar Wi + Ai Wr   (product with W)
// acc_re += Ar Wr + Ai Wi ; acc_im += Ai Wr - Ar Wi   (product with conj W)
// (the sign goes to A after its last plain use, in place)
template <bool CONJ>
__device__ __forceinline__ void mf_cmma(MfA a, mf_u32x4 wrh, mf_u32x4 wrl, mf_u32x4 wih,
                                        mf_u32x4 wil, mf_f32x4& re, mf_f32x4& im) {
  re = mf_mma3(a.rh, a.rl, wrh, wrl, re);
  if constexpr (!CONJ) {
    im = mf_mma3(a.rh, a.rl, wih, wil, im);
    im = mf_mma3(a.ih, a.il, wrh, wrl, im);
    re = mf_mma3(mf_neg(a.ih), mf_neg(a.il), wih, wil, re);
  } else {
    im = mf_mma3(a.ih, a.il, wrh, wrl, im);
    re = mf_mma3(a.ih, a.il, wih, wil, re);
    im = mf_mma3(mf_neg(a.rh), mf_neg(a.rl), wih, wil, im);
  }
}

// a wave's W fragments (output tile nt) in registers
struct MfW {
  mf_u32x4 f[kMfKs][4];
};
__device__ __forceinline__ void mf_load_w(MfW& w, const mf_u32x4* __restrict__ wf, int nt,
                                          int lane) {
#pragma unroll
  for (int ks = 0; ks < kMfKs; ++ks)
#pragma unroll
    for (int mat = 0; mat < 4; ++mat)
      w.f[ks][mat] = wf[((mat * kMfKs + ks) * kMfNt + nt) * 64 + lane];
}

// A fragments of 16 lines in LDS: [mat][ks][slot] of 16 bytes, mat = re hi, re
// lo, im hi, im lo.  Line r's values k = 32 ks + 8 j + e sit in slot
// (r ^ (j + 4 ks)) + 16 j: a wave that holds one line along k then writes all
// banks, and a fragment read still takes 256 consecutive bytes per 16 lanes.
constexpr int kMfABuf = 4 * kMfKs * 64;  // mf_u32x4 per buffer (16 KB)
__device__ __forceinline__ int mf_slot(int r, int j, int ks) {
  return (r ^ (j + 4 * ks)) + 16 * j;
}

// four consecutive values of line r from k = 4 kq on, split, to the buffer
__device__ __forceinline__ void mf_put4(mf_u32x4* buf, const float2 (&z)[4], int r, int kq) {
  const int ks = kq >> 3, j = (kq >> 1) & 3;
  uint32_t h[2][4], l[2][4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    h[0][e] = mf_bf16_rne(z[e].x);
    l[0][e] = mf_bf16_rne(z[e].x - __uint_as_float(h[0][e] << 16));
    h[1][e] = mf_bf16_rne(z[e].y);
    l[1][e] = mf_bf16_rne(z[e].y - __uint_as_float(h[1][e] << 16));
  }
  uint2* d = reinterpret_cast<uint2*>(buf + ks * 64 + mf_slot(r, j, ks)) + (kq & 1);
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    d[(2 * c) * kMfKs * 128] = make_uint2(h[c][0] | (h[c][1] << 16), h[c][2] | (h[c][3] << 16));
    d[(2 * c + 1) * kMfKs * 128] =
        make_uint2(l[c][0] | (l[c][1] << 16), l[c][2] | (l[c][3] << 16));
  }
}

// re, im (16 lines x 16 outputs) += lines in the buffer times W (or conj W)
template <bool CONJ>
__device__ __forceinline__ void mf_lines(const mf_u32x4* buf, const MfW& w, int lane, mf_f32x4& re,
                                         mf_f32x4& im) {
  auto frag = [&](int ks) {
    const int s = mf_slot(lane & 15, lane >> 4, ks);
    MfA a;
    a.rh = buf[(0 * kMfKs + ks) * 64 + s];
    a.rl = buf[(1 * kMfKs + ks) * 64 + s];
    a.ih = buf[(2 * kMfKs + ks) * 64 + s];
    a.il = buf[(3 * kMfKs + ks) * 64 + s];
    return a;
  };
  // one step's fragments at a time, so that W stays in registers; the other
  // waves of the SIMD hide the reads
#pragma unroll
  for (int ks = 0; ks < kMfKs; ++ks) {
    const MfA a = frag(ks);
    mf_cmma<CONJ>(a, w.f[ks][0], w.f[ks][1], w.f[ks][2], w.f[ks][3], re, im);
    __builtin_amdgcn_sched_barrier(0);
  }
}

constexpr int kMfThreads = 512;
constexpr int kMfTiles = kMfF / 16;  // 16-line tiles per frame

// ---------------------------------------------------------------------------
// (1) row transform: T[r][c] = sum_k Z[r][k] W[k][c], one (view, mode) frame
// after another, 16 rows a step; the next step's psi, P and O are in flight
// during the products.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kMfThreads) void k_mf_rows_fwd(const ScanDev* __restrict__ scans,
                                                               const int2* __restrict__ vmap,
                                                               int total_views, int M,
                                                               const uint4* __restrict__ wf) {
  __shared__ mf_u32x4 ab[2 * kMfABuf];
  constexpr int F = kMfF, FF = F * F;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  MfW w;
  mf_load_w(w, reinterpret_cast<const mf_u32x4*>(wf), wave, lane);
  const int r = t >> 5, kq = t & 31;  // this thread's line and run of four values
  const unsigned to = 4 * (lane >> 4) * F + 16 * wave + (lane & 15);
  const int total = total_views * M;
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int2 vm = vmap[item / M];
    const int m = item % M;
    const ScanDev& sc = scans[vm.x];
    const int j = uni(vm.y);
    const int W = uni(sc.W);
    const int y0 = uni(kidx(sc.pos)[2 * j]), x0 = uni(kidx(sc.pos)[2 * j + 1]);
    // wave-uniform bases, one 32-bit offset per lane
    const float2* __restrict__ psi = sc.psi + ((size_t)j * M + m) * FF;
    const float2* __restrict__ P = sc.P + (size_t)m * FF;
    const float2* __restrict__ O = sc.O + (size_t)y0 * W + x0;
    float2* __restrict__ T = sc.tspec + ((size_t)j * M + m) * FF;
    const unsigned lo = r * W + 4 * kq;
    float4 sv[2], pv[2];
    float2 ov[4];
    auto load = [&](int rt) {
      const float4* s4 = reinterpret_cast<const float4*>(psi + rt * 16 * F);
      const float4* p4 = reinterpret_cast<const float4*>(P + rt * 16 * F);
      const float2* o2 = O + (size_t)rt * 16 * W;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        sv[e] = s4[2u * t + e];
        pv[e] = p4[2u * t + e];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) ov[e] = o2[lo + e];
    };
    auto put = [&](int rt) {
      const float2 p[4] = {make_float2(pv[0].x, pv[0].y), make_float2(pv[0].z, pv[0].w),
                           make_float2(pv[1].x, pv[1].y), make_float2(pv[1].z, pv[1].w)};
      const float2 s[4] = {make_float2(sv[0].x, sv[0].y), make_float2(sv[0].z, sv[0].w),
                           make_float2(sv[1].x, sv[1].y), make_float2(sv[1].z, sv[1].w)};
      float2 z[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float2 phi = cmul(p[e], ov[e]);
        z[e] = make_float2(2.f * phi.x - s[e].x, 2.f * phi.y - s[e].y);
      }
      mf_put4(ab + (rt & 1) * kMfABuf, z, r, kq);
    };
    load(0);
    put(0);
    load(1);
#pragma unroll 1
    for (int rt = 0; rt < kMfTiles; ++rt) {
      const mf_u32x4* buf = ab + (rt & 1) * kMfABuf;
      // one barrier a step: past it the other buffer's readers (step rt - 1)
      // are done, so the next step's lines are split and written while this
      // step's products run
      __syncthreads();
      if (rt + 1 < kMfTiles) put(rt + 1);
      if (rt + 2 < kMfTiles) load(rt + 2);
      mf_f32x4 re{0.f, 0.f, 0.f, 0.f}, im{0.f, 0.f, 0.f, 0.f};
      mf_lines<false>(buf, w, lane, re, im);
      float2* __restrict__ Tr = T + rt * 16 * F;
#pragma unroll
      for (int q = 0; q < 4; ++q) Tr[to + q * F] = make_float2(re[q], im[q]);
    }
  }
}

// ---------------------------------------------------------------------------
// (2) column transform, modulus projection and inverse column transform for
// 16 columns n0 .. n0+15 of every mode of one view, in place in T; the 16
// columns are the lines, wave w forms the frequencies a = 16 w .. 16 w + 15.
//   U^T[n][a] = sum_k T[k][n] W[k][a]
//   U' = U * sqrt(I / sum_m |U_m|^2) / F^2
//   V^T[n][a'] = sum_a U'^T[n][a] conj(W)[a][a']
// ---------------------------------------------------------------------------
// M is a template parameter: with a run-time mode count the spectra of eight
// modes, kept in registers across branches, spill.
template <int M>
__global__ __launch_bounds__(kMfThreads) void k_mf_cols(const ScanDev* __restrict__ scans,
                                                        const int2* __restrict__ vmap,
                                                        int total_views,
                                                        const uint4* __restrict__ wf) {
  // two buffers, taken in turn by the M forward and the M inverse steps of an
  // item, one barrier per step (as above)
  __shared__ mf_u32x4 ab[2 * kMfABuf];
  constexpr int F = kMfF, FF = F * F;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  MfW w;
  mf_load_w(w, reinterpret_cast<const mf_u32x4*>(wf), wave, lane);
  const int kq = 4 * wave + (lane >> 4);  // this thread's run of four values of line lane % 16
  const int a = 16 * wave + (lane & 15);  // this lane's frequency, columns 4 (lane / 16) + r
  const int total = total_views * kMfNt;
  float2 z[4];
  float iv[4];
  // mode m of an item's columns; its intensities
  auto load = [&](int item, int m) {
    const int2 vm = vmap[item / kMfNt];
    const float2* __restrict__ Tl = scans[vm.x].tspec + ((size_t)uni(vm.y) * M + m) * FF +
                                    16 * (item % kMfNt) + (4 * kq) * F + (lane & 15);
#pragma unroll
    for (int e = 0; e < 4; ++e) z[e] = Tl[e * F];
  };
  auto load_iv = [&](int item) {
    const int2 vm = vmap[item / kMfNt];
    const float* __restrict__ Ij = scans[vm.x].I + (size_t)uni(vm.y) * FF +
                                   16 * (item % kMfNt) + a * F + 4 * (lane >> 4);
#pragma unroll
    for (int q = 0; q < 4; ++q) iv[q] = Ij[q];
  };
  if ((int)blockIdx.x < total) {
    load(blockIdx.x, 0);
    mf_put4(ab, z, lane & 15, kq);
    if (M > 1) load(blockIdx.x, 1);
    load_iv(blockIdx.x);
  }
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int2 vm = vmap[item / kMfNt];
    const int n0 = 16 * (item % kMfNt);
    const int next = item + gridDim.x;
    float2* __restrict__ T = scans[vm.x].tspec + (size_t)uni(vm.y) * M * FF;
    mf_f32x4 ure[M], uim[M];
    // past a step's barrier the other buffer is free: the next step's lines
    // are written there while this step's products run
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const mf_u32x4* buf = ab + (m & 1) * kMfABuf;
      __syncthreads();
      if (m + 1 < M) mf_put4(ab + ((m + 1) & 1) * kMfABuf, z, lane & 15, kq);
      if (m + 2 < M) load(item, m + 2);
      ure[m] = mf_f32x4{0.f, 0.f, 0.f, 0.f};
      uim[m] = mf_f32x4{0.f, 0.f, 0.f, 0.f};
      mf_lines<false>(buf, w, lane, ure[m], uim[m]);
    }
    const float inv_ff = 1.0f / (float)FF;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float s = 0.f;
#pragma unroll
      for (int m = 0; m < M; ++m) s += ure[m][r] * ure[m][r] + uim[m][r] * uim[m][r];
      const float i0 = fmaxf(iv[r], 0.f);
      const float g = (s > FLT_MIN) ? sqrtf(i0 / s) * inv_ff : 0.f;
#pragma unroll
      for (int m = 0; m < M; ++m) { ure[m][r] *= g; uim[m][r] *= g; }
    }
    // the next item's first loads: in flight over the inverse steps
    if (next < total) {
      load(next, 0);
      load_iv(next);
    }
    // element (n, a) of U'^T: ks = a / 32 = w / 2, j = (a % 32) / 8
    auto put_u = [&](int m, int step) {
      uint16_t* const ua = reinterpret_cast<uint16_t*>(ab + (step & 1) * kMfABuf);
      const int ks = wave >> 1, jj = 2 * (wave & 1) + ((lane & 15) >> 3);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int n = 4 * (lane >> 4) + r;
        const int slot = (ks * 64 + mf_slot(n, jj, ks)) * 8 + (lane & 7);
        const float vr = ure[m][r], vi = uim[m][r];
        const uint32_t rh = mf_bf16_rne(vr), ih = mf_bf16_rne(vi);
        const uint32_t rl = mf_bf16_rne(vr - __uint_as_float(rh << 16));
        const uint32_t il = mf_bf16_rne(vi - __uint_as_float(ih << 16));
        ua[0 * kMfKs * 512 + slot] = (uint16_t)rh;
        ua[1 * kMfKs * 512 + slot] = (uint16_t)rl;
        ua[2 * kMfKs * 512 + slot] = (uint16_t)ih;
        ua[3 * kMfKs * 512 + slot] = (uint16_t)il;
      }
    };
    // step M's buffer was last read in step M - 2, before step M - 1's barrier
    put_u(0, M);
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const mf_u32x4* buf = ab + ((M + m) & 1) * kMfABuf;
      __syncthreads();
      if (m + 1 < M) {
        put_u(m + 1, M + m + 1);
      } else if (next < total) {
        mf_put4(ab, z, lane & 15, kq);  // 2 M steps: the next item starts with buffer 0
        if (M > 1) load(next, 1);
      }
      mf_f32x4 vre = mf_f32x4{0.f, 0.f, 0.f, 0.f}, vim = mf_f32x4{0.f, 0.f, 0.f, 0.f};
      mf_lines<true>(buf, w, lane, vre, vim);
      // V^T[n][a'] -> T[a'][n0 + n]; lane holds a' = 16 w + lane%16,
      // n = 4 (lane/16) + r
      float2* __restrict__ Tm = T + (size_t)m * FF;
      float4* dst = reinterpret_cast<float4*>(Tm + a * F + n0 + 4 * (lane >> 4));
      dst[0] = make_float4(vre[0], vim[0], vre[1], vim[1]);
      dst[1] = make_float4(vre[2], vim[2], vre[3], vim[3]);
    }
  }
}

// ---------------------------------------------------------------------------
// (3) inverse row transform and the view update, one half (64 rows) of a view
// after another, 16 rows of each mode a step (modes inside, so that the object
// numerator of the 16 rows stays in registers).  The halves' eps_psi partials
// go to parts 2j and 2j + 1.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kMfThreads) void k_mf_rows_inv(const ScanDev* __restrict__ scans,
                                                               const int2* __restrict__ vmap,
                                                               int total_views, int M,
                                                               const uint4* __restrict__ wf) {
  __shared__ mf_u32x4 ab[2 * kMfABuf];
  __shared__ float red[2 * (kMfThreads / 64)];
  constexpr int F = kMfF, FF = F * F;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  MfW w;
  mf_load_w(w, reinterpret_cast<const mf_u32x4*>(wf), wave, lane);
  const int r = t >> 5, kq = t & 31;
  const int col = 16 * wave + (lane & 15), rl = 4 * (lane >> 4);
  for (int item = blockIdx.x; item < 2 * total_views; item += gridDim.x) {
    const int2 vm = vmap[item >> 1];
    const int rt0 = (item & 1) * (kMfTiles / 2), rt1 = rt0 + kMfTiles / 2;
    const ScanDev& sc = scans[vm.x];
    const int j = uni(vm.y);
    const int W = uni(sc.W);
    const float beta = sc.beta;
    const int y0 = uni(kidx(sc.pos)[2 * j]), x0 = uni(kidx(sc.pos)[2 * j + 1]);
    const float2* __restrict__ O = sc.O + (size_t)(y0 + rl) * W + x0 + col;
    const float2* __restrict__ V = sc.tspec + (size_t)j * M * FF + r * F + 4 * kq;
    float2* __restrict__ psi = sc.psi + (size_t)j * M * FF + rl * F + col;
    const float2* __restrict__ P = sc.P + rl * F + col;
    float2* __restrict__ oj = sc.opart + (size_t)j * FF + rl * F + col;
    float e_d = 0.f, e_n = 0.f;
    float4 vv[2];
    auto load = [&](int rt, int m) {
      const float4* v4 = reinterpret_cast<const float4*>(V + (size_t)m * FF + rt * 16 * F);
      vv[0] = v4[0]; vv[1] = v4[1];
    };
    auto put = [&](int step) {
      const float2 z[4] = {make_float2(vv[0].x, vv[0].y), make_float2(vv[0].z, vv[0].w),
                           make_float2(vv[1].x, vv[1].y), make_float2(vv[1].z, vv[1].w)};
      mf_put4(ab + (step & 1) * kMfABuf, z, r, kq);
    };
    const int steps = (rt1 - rt0) * M;
    int lrt = rt0, lm = 0;  // the step whose lines are loaded next
    auto load_next = [&]() {
      load(lrt, lm);
      if (++lm == M) { lm = 0; ++lrt; }
    };
    load_next();
    put(0);
    if (steps > 1) load_next();
    int step = 0;
#pragma unroll 1
    for (int rt = rt0; rt < rt1; ++rt) {
      float2 oacc[4], ov[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        oacc[q] = make_float2(0.f, 0.f);
        ov[q] = O[(size_t)(16 * rt + q) * W];
      }
#pragma unroll 1
      for (int m = 0; m < M; ++m, ++step) {
        const mf_u32x4* buf = ab + (step & 1) * kMfABuf;
        // the update's operands go out before the products
        float2 pr[4], pv[4];
        float2* __restrict__ pm = psi + (size_t)m * FF + rt * 16 * F;
        const float2* __restrict__ Pm = P + (size_t)m * FF + rt * 16 * F;
#pragma unroll
        for (int q = 0; q < 4; ++q) { pr[q] = Pm[q * F]; pv[q] = pm[q * F]; }
        __syncthreads();  // as in the row transform
        if (step + 1 < steps) put(step + 1);
        if (step + 2 < steps) load_next();
        mf_f32x4 re{0.f, 0.f, 0.f, 0.f}, im{0.f, 0.f, 0.f, 0.f};
        mf_lines<true>(buf, w, lane, re, im);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float2 phi = cmul(pr[q], ov[q]);
          const float2 d = make_float2(beta * (re[q] - phi.x), beta * (im[q] - phi.y));
          const float2 pn = cadd(pv[q], d);
          pm[q * F] = pn;
          e_d += cabs2(d);
          e_n += cabs2(pn);
          oacc[q] = cadd(oacc[q], cmulc(pr[q], pn));
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) oj[(16 * rt + q) * F] = oacc[q];
    }
    block_sum2<kMfThreads>(e_d, e_n, red);
    if (t == 0) {
      float* e = sc.err_psi + 4 * (size_t)j + 2 * (item & 1);
      e[0] = e_d;
      e[1] = e_n;
    }
    __syncthreads();  // red and the buffers are reused by the next item
  }
}

}  // namespace dmk
