// dm_mixed.hpp -- the view update (Eq. 3 with F_c, Section II) for frames
// whose edge is not a power of two: F = 4 Q (188 = 4 * 47, 200 = 4 * 50, the
// frame sizes the paper's own measurements use).  Three kernels around the
// spectrum buffer, as for F = 256: row DFTs, then column DFTs with the mode
// sum and modulus scale and the inverse column DFTs, then inverse row DFTs
// with the update.
//
// A wave transforms 16 lines in registers, without LDS or barriers: lane
// (n2 = lane / 16, line = lane % 16) holds x[4 n1 + n2], n1 < Q, and with
// n = 4 n1 + n2, k = k1 + Q k2
//   X[k1 + Q k2] = sum_{n2} W_4^{n2 k2} W_F^{n2 k1} sum_{n1} x[4 n1 + n2] W_Q^{n1 k1}.
// The Q-point DFTs run in the lane.  Q = 47 uses the symmetry of W_Q for odd Q:
// with u_n = x_n + x_{Q-n}, v_n = x_n - x_{Q-n} and c_n + i s_n = W_Q^{n p},
//   Y_p     = x_0 + sum_n c_n u_n + i sum_n s_n v_n,
//   Y_{Q-p} = x_0 + sum_n c_n u_n - i sum_n s_n v_n
// (a quarter of the products of the direct sum, every factor a literal of an
// unrolled FMA).  Q = 50 is 2 x 5 x 5 in place.  Both give their outputs in
// pairs A = Y[kA], B = Y[kB]; the four-point DFT over n2 crosses the lanes of
// a line, two values at a time: v_permlane32_swap gives the lower half-wave
// both halves' A and the upper one both B, v_permlane16_swap then does the
// same with sums and differences, so that lane (h = lane / 32, b = lane / 16 %
// 2) ends with X[k + Q b] and X[k + Q (b + 2)], k = h ? kB : kA.  The inverse
// runs the same steps backwards and returns values to the lane they came
// from.
//
// The spectrum buffer is k-major, T[kx][row], its lines padded to whole blocks
// of 16 rows: the row kernels touch it in runs of 16 rows, exactly one 128-byte
// cache line each (unpadded, a run met two lines that other XCDs wrote too),
// the column kernel along its lines, 32 bytes a line and instruction.
//
// What bounds it: moving the spectra and the views, at 60-75% of a copy's rate,
// and at 188^2 also the products of the 47-point DFTs (2116 FMAs a lane, 45 a
// value and dimension).  At 1500 x 4 x 188^2 rows, columns and inverse rows take
// 0.85, 1.20 and 1.29 ms, at 2521 x 1 x 200^2 0.41, 0.51 and 0.68 ms.  The form
// before kept the lines in LDS with Q + 1 threads a line, each reading 32 bytes
// of LDS per 8 FMAs between four barriers a transform: 0.91, 2.07, 1.27 ms and
// 0.54, 0.86, 0.86 ms.  The row kernels stream the views and the spectra past
// the caches (non-temporal: inverse rows 0.77 -> 0.68 ms at 200^2), which holds
// the probe and object in them; the column kernel does not (1.23 against 1.20
// ms at 188^2).
#pragma once
#include <hip/hip_runtime.h>
#include <float.h>

#include <type_traits>

#include "dm_kernels.hpp"

namespace dmk {

template <int F>
struct Mix;
template <>
struct Mix<188> {
  static constexpr int Q = 47, NP = 24, LB = 12;  // pairs, blocks of 16 lines
  static constexpr int LDT = 16 * LB, FT = 188 * LDT;  // spectrum line, frame (complex)
  static constexpr int kB(int i) { return 47 - i; }
  static constexpr bool hasB(int i) { return i > 0; }
};
template <>
struct Mix<200> {
  static constexpr int Q = 50, NP = 25, LB = 13;
  static constexpr int LDT = 16 * LB, FT = 200 * LDT;
  static constexpr int kB(int i) { return 25 + i; }
  static constexpr bool hasB(int) { return true; }
};

// f(integral_constant<int, B>) ... f(integral_constant<int, E - 1>)
template <int B, int E, class Fn>
__device__ __forceinline__ void static_for(Fn&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// Holds a value at this point of the program: the code that forms it stays
// before, and so do the registers of its operands.  Without, the compiler
// forms the values of a long unrolled block where they are first used, keeps
// every load alive until then and spills.
__device__ __forceinline__ void pin(float2& a) { asm volatile("" : "+v"(a.x), "+v"(a.y)); }

// cos and sin of 2 pi m / N in double at compile time (Taylor series of the
// angle reduced to an eighth turn)
struct CosSin {
  double c, s;
};
constexpr CosSin cos_sin_turn(int m, int n) {
  m %= n;
  if (m < 0) m += n;
  // octant: angle = 2 pi (8 m mod n ... ) folded to [0, pi/4]
  int o = (8 * m) / n;       // 0 .. 7
  const int r = 8 * m - o * n;  // remainder in eighth turns, r / n in [0, 1)
  const bool flip = o & 1;   // mirror odd octants at their end
  const double t = (flip ? (double)(n - r) : (double)r) / n;
  const double x = t * 0.78539816339744830961566084581988;  // pi / 4
  const double x2 = x * x;
  double c = 1.0, s = x, tc = 1.0, ts = x;
  for (int k = 1; k < 14; ++k) {
    tc *= -x2 / ((2 * k - 1) * (2 * k));
    ts *= -x2 / ((2 * k) * (2 * k + 1));
    c += tc;
    s += ts;
  }
  if (flip) ++o;  // angle = o pi / 4 - x
  const double h = 0.70710678118654752440084436210485;
  double oc = 0, os = 0;
  switch (o & 7) {
    case 0: oc = 1; os = 0; break;
    case 1: oc = h; os = h; break;
    case 2: oc = 0; os = 1; break;
    case 3: oc = -h; os = h; break;
    case 4: oc = -1; os = 0; break;
    case 5: oc = -h; os = -h; break;
    case 6: oc = 0; os = -1; break;
    default: oc = h; os = -h; break;
  }
  const double sx = flip ? -s : s;
  return CosSin{oc * c - os * sx, os * c + oc * sx};
}

// a * exp(DIR 2 pi i M / N)
template <int DIR, int M, int N>
__device__ __forceinline__ float2 mix_tw(float2 a) {
  constexpr CosSin w = cos_sin_turn(M, N);
  constexpr float c = (float)w.c, s = (float)(DIR * w.s);
  return make_float2(a.x * c - a.y * s, a.x * s + a.y * c);
}

template <int DIR>
__device__ __forceinline__ void dft5(float2& a0, float2& a1, float2& a2, float2& a3, float2& a4) {
  constexpr CosSin w1 = cos_sin_turn(1, 5), w2 = cos_sin_turn(2, 5);
  constexpr float c1 = (float)w1.c, c2 = (float)w2.c;
  constexpr float s1 = (float)(DIR * w1.s), s2 = (float)(DIR * w2.s);
  const float2 t1 = cadd(a1, a4), t2 = cadd(a2, a3), t3 = csub(a1, a4), t4 = csub(a2, a3);
  const float2 b1 = make_float2(a0.x + c1 * t1.x + c2 * t2.x, a0.y + c1 * t1.y + c2 * t2.y);
  const float2 b2 = make_float2(a0.x + c2 * t1.x + c1 * t2.x, a0.y + c2 * t1.y + c1 * t2.y);
  const float2 d1 = make_float2(s1 * t3.x + s2 * t4.x, s1 * t3.y + s2 * t4.y);
  const float2 d2 = make_float2(s2 * t3.x - s1 * t4.x, s2 * t3.y - s1 * t4.y);
  a0 = cadd(a0, cadd(t1, t2));
  a1 = make_float2(b1.x - d1.y, b1.y + d1.x);
  a4 = make_float2(b1.x + d1.y, b1.y - d1.x);
  a2 = make_float2(b2.x - d2.y, b2.y + d2.x);
  a3 = make_float2(b2.x + d2.y, b2.y - d2.x);
}

// 25-point DFT of a[S i + S0], i < 25; output k is left at index
// S (5 (k % 5) + k / 5) + S0
template <int DIR, int S, int S0, int N>
__device__ __forceinline__ void dft25(float2 (&a)[N]) {
  static_for<0, 5>([&](auto i2) {
    constexpr int o = S * i2 + S0;
    dft5<DIR>(a[o], a[o + 5 * S], a[o + 10 * S], a[o + 15 * S], a[o + 20 * S]);
    static_for<1, 5>([&](auto k1) {
      a[o + 5 * S * k1] = mix_tw<DIR, i2 * k1, 25>(a[o + 5 * S * k1]);
    });
  });
  // a[S (5 k1 + i2) + S0] = y_{i2}[k1]: over i2 for each k1
  static_for<0, 5>([&](auto k1) {
    constexpr int o = S * 5 * k1 + S0;
    dft5<DIR>(a[o], a[o + S], a[o + 2 * S], a[o + 3 * S], a[o + 4 * S]);
  });
}
// index i < 25 at which output k of dft25 is left
constexpr int pos25(int k) { return 5 * (k % 5) + k / 5; }

// sum over the pairs u, v of output p (and Q - p) of the 47-point DFT:
// a[0] = x_0, a[n] = u_n, a[47 - n] = v_n for 1 <= n <= 23.
// The terms are added small ones first, which keeps the rounding of the long
// sums down: the forward transform's lines are largest in the middle of the
// frame (n = 23, where the probe is), the inverse's at the lowest frequencies
// (n = 0, and by the symmetry n = 1).  With both from n = 0 up, psi' after two
// iterations at 1500 x 4 x 188^2 was 4.80e-7 off the 64-bit result (relative
// L2), now 4.20e-7, in the same time.  (Output 0, summed while the terms are
// formed, keeps their order: 2% of the pass at that size.)
template <int DIR, int P>
__device__ __forceinline__ void out47(const float2 (&a)[47], float2& A, float2& B) {
  if constexpr (P == 0) {
    float2 su = a[0];
    static_for<1, 24>([&](auto n) { su = cadd(su, a[n]); });
    A = su;
    B = make_float2(0.f, 0.f);
  } else {
    float2 su = DIR < 0 ? a[0] : make_float2(0.f, 0.f);
    float2 sv = make_float2(0.f, 0.f);
    static_for<1, 24>([&](auto i) {
      constexpr int n = DIR < 0 ? i : 24 - i;
      constexpr CosSin w = cos_sin_turn(n * P, 47);
      constexpr float c = (float)w.c, s = (float)(DIR * w.s);
      su.x += c * a[n].x;
      su.y += c * a[n].y;
      sv.x += s * a[47 - n].x;
      sv.y += s * a[47 - n].y;
    });
    if constexpr (DIR > 0) su = cadd(su, a[0]);
    A = make_float2(su.x - sv.y, su.y + sv.x);
    B = make_float2(su.x + sv.y, su.y - sv.x);
  }
}

// exchanges of two values between the half-waves (v0's upper half with v1's
// lower half) and between the rows of 16 lanes (v0's odd rows with v1's even)
__device__ __forceinline__ void swap_halves(float& v0, float& v1) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v0), __float_as_uint(v1), false,
                                                  false);
  v0 = __uint_as_float(r[0]);
  v1 = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap_rows(float& v0, float& v1) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v0), __float_as_uint(v1), false,
                                                  false);
  v0 = __uint_as_float(r[0]);
  v1 = __uint_as_float(r[1]);
}

// What a lane knows of its place: line of the wave, n2 = 2 h + b
struct MixLane {
  int line, n2, h, b;
  __device__ __forceinline__ explicit MixLane(int lane)
      : line(lane & 15), n2(lane >> 4), h(lane >> 5), b((lane >> 4) & 1) {}
};

// Twiddles W_F^{n2 k1} in LDS, [k1][n2]
template <int F>
__device__ __forceinline__ void mix_load_twiddles(const float2* __restrict__ tw, float2* twl,
                                                  int t, int nt) {
  constexpr int Q = Mix<F>::Q;
  for (int i = t; i < 4 * Q; i += nt) twl[i] = tw[(i >> 2) * (i & 3)];
  __syncthreads();
}

// DFT4 over n2 of the pair (A, B): X[b], X[b + 2] of the lane's k1
__device__ __forceinline__ void cross_fwd(float2 A, float2 B, int b, float2& x0, float2& x1) {
  swap_halves(A.x, B.x);
  swap_halves(A.y, B.y);
  float2 s = cadd(A, B), d = csub(A, B);
  swap_rows(s.x, d.x);
  swap_rows(s.y, d.y);
  // rows b = 1 hold d_0, d_1: X_1 = d_0 - i d_1, X_3 = d_0 + i d_1
  const float2 e = make_float2(b ? d.y : d.x, b ? -d.x : d.y);
  x0 = cadd(s, e);
  x1 = csub(s, e);
}
// its inverse (unnormalised)
__device__ __forceinline__ void cross_inv(float2 x0, float2 x1, int b, float2& A, float2& B) {
  float2 e = cadd(x0, x1), o = csub(x0, x1);
  // rows b = 1: o_1 = X_1 - X_3 enters z_1, z_3 as +- i o_1
  o = make_float2(b ? -o.y : o.x, b ? o.x : o.y);
  swap_rows(e.x, o.x);
  swap_rows(e.y, o.y);
  A = cadd(e, o);
  B = csub(e, o);
  swap_halves(A.x, B.x);
  swap_halves(A.y, B.y);
}

// Forward transform of the wave's lines, a[n1] = x[4 n1 + n2];
// emit(integral_constant i, X0, X1) gets X[k + Q b] and X[k + Q (b + 2)], k = kA = i or
// kB(i) by half-wave (where the upper half has none, its values are 0).
template <int F, class Emit>
__device__ __forceinline__ void mix_fwd(float2 (&a)[Mix<F>::Q], const float2* twl,
                                        const MixLane& ln, Emit&& emit) {
  using C = Mix<F>;
  if constexpr (F == 188) {
    static_for<1, 24>([&](auto n) {
      const float2 x = a[n], y = a[47 - n];
      a[n] = cadd(x, y);
      a[47 - n] = csub(x, y);
    });
  } else {
    dft25<-1, 2, 0>(a);
    dft25<-1, 2, 1>(a);
  }
  static_for<0, C::NP>([&](auto i) {
    float2 A, B;
    if constexpr (F == 188) {
      out47<-1, i>(a, A, B);
    } else {
      constexpr int p = 2 * pos25(i);
      const float2 o = mix_tw<-1, i, 50>(a[p + 1]);
      A = cadd(a[p], o);
      B = csub(a[p], o);
    }
    if constexpr (i > 0) A = cmul(A, twl[i * 4 + ln.n2]);
    if constexpr (C::hasB(i)) B = cmul(B, twl[C::kB(i) * 4 + ln.n2]);
    float2 x0, x1;
    cross_fwd(A, B, ln.b, x0, x1);
    emit(i, x0, x1);
    __builtin_amdgcn_sched_barrier(0);
  });
}

// Inverse, first part: x[2 i], x[2 i + 1] = the X0, X1 of mix_fwd -> a, what
// mix_inv_out forms the outputs from.
template <int F>
__device__ __forceinline__ void mix_inv_in(const float2 (&x)[2 * Mix<F>::NP],
                                           float2 (&a)[Mix<F>::Q], const float2* twl,
                                           const MixLane& ln) {
  using C = Mix<F>;
  static_for<0, C::NP>([&](auto i) {
    float2 A, B;
    cross_inv(x[2 * i], x[2 * i + 1], ln.b, A, B);
    auto conj_tw = [&](float2 z, int k) {
      const float2 w = twl[k * 4 + ln.n2];
      return make_float2(z.x * w.x + z.y * w.y, z.y * w.x - z.x * w.y);
    };
    if constexpr (i > 0) A = conj_tw(A, i);
    if constexpr (C::hasB(i)) B = conj_tw(B, C::kB(i));
    if constexpr (F == 188) {
      if constexpr (i == 0) {
        a[0] = A;
      } else {
        a[i] = cadd(A, B);
        a[47 - i] = csub(A, B);
      }
      if constexpr (i > 0) pin(a[47 - i]);
      pin(a[i]);
    } else {
      a[2 * i] = cadd(A, B);
      a[2 * i + 1] = mix_tw<1, i, 50>(csub(A, B));
      pin(a[2 * i]);
      pin(a[2 * i + 1]);
    }
    __builtin_amdgcn_sched_barrier(0);
  });
  if constexpr (F == 200) {
    dft25<1, 2, 0>(a);
    dft25<1, 2, 1>(a);
  }
}
// Second part: outputs come in NP groups of two (one in group 0 at 188);
// mix_n(i, e) is the n1 of output e of group i, mix_inv_out gives both.
template <int F>
constexpr int mix_n(int i, int e) {
  return F == 188 ? (e ? 47 - i : i) : 2 * i + e;
}
template <int F, int I>
__device__ __forceinline__ void mix_inv_out(const float2 (&a)[Mix<F>::Q], float2 (&z)[2]) {
  if constexpr (F == 188) {
    out47<1, I>(a, z[0], z[1]);
  } else {
    z[0] = a[2 * pos25(I)];
    z[1] = a[2 * pos25(I) + 1];
  }
}

// Byte offset of a dropped access: past the end of every buffer that is stored
// to, with any offset within a frame added.  Only an object of 1 GiB and more
// is larger (up to 2 GiB): a load of it then returns some value of the object
// instead of 0, which like the 0 goes no further than its tile cell.
constexpr int kMixOob = 0x40000000;

// Byte offset of X0 of pair i in a k-major frame; X1 is 2 Q lines further.  The
// padding's rows past the frame hold nothing of use (transforms of the last
// rows again, which the column kernel neither reads nor scales): what is formed
// from them is neither stored nor summed.
template <int F>
struct MixSpec {
  int base, step;
  __device__ __forceinline__ MixSpec(const MixLane& ln, int line) {
    using C = Mix<F>;
    base = (((ln.h ? C::kB(0) : 0) + C::Q * ln.b) * C::LDT + line) * 8;
    step = (F == 188 && ln.h) ? -C::LDT * 8 : C::LDT * 8;
  }
  __device__ __forceinline__ int at(int i, const MixLane& ln) const {
    return (F == 188 && i == 0 && ln.h) ? kMixOob : base + i * step;
  }
  static constexpr int kX1 = 2 * Mix<F>::Q * Mix<F>::LDT * 8;
};

// Lines pass between memory and the lanes in chunks of CW values through a
// wave's own LDS tile of its 16 lines: an instruction then moves 64 / CW lines x
// CW consecutive values instead of 16 lines x 32 bytes (reading x[4 n1 + n2]
// straight from memory the row kernels took 1.47 and 2.43 ms at 1500 x 4 x
// 188^2).  The row kernels take 64 values (512 bytes) a line; the column
// kernel, whose tiles have to fit its waves' slots of LDS, 32.  Tile lines are
// CW + 4 values apart: the lanes' reads of x[4 n1 + n2] then cover all banks.
constexpr int kRowCW = 64, kColCW = 32;
template <int CW>
constexpr int kMixTile = 16 * (CW + 4);  // float2 per tile
template <int F, int CW>
constexpr int kMixChunks = (F + CW - 1) / CW;

// Element (i, lane) of chunk CH, i < kI: with L = 64 / (values used of a
// line) lines an instruction, line L i + lane / (64 / L) of the wave's, value
// CW CH + lane % (64 / L).  (200 leaves a last chunk of 8 values: eight lines an
// instruction.)  Lines past the frame load its last ones again and store
// nothing; values past the line load 0 and store nothing.  A dropped access
// gets a lane offset out of range and a scalar offset within it (the range
// check subtracts the scalar offset).
template <int F, int CW, int CH>
struct MixIO {
  static constexpr int kWidth = F - CW * CH < CW ? F - CW * CH : CW;
  static constexpr int kSpan = kWidth <= 8 ? 8 : CW;  // lanes a line
  static constexpr int L = 64 / kSpan, kI = 16 / L;
  static_assert(F % L == 0 && 16 % L == 0, "the lines of an instruction are in the frame together");
  // per-lane byte offset in lines of `stride` values
  __device__ __forceinline__ static int load_off(int lane, int stride) {
    const int v = lane % kSpan;
    return v < kWidth ? ((lane / kSpan) * stride + v) * 8 : kMixOob;
  }
  __device__ __forceinline__ static bool in(int lane, int line0, int i) {
    return line0 + L * i < F && (kWidth == kSpan || lane % kSpan < kWidth);
  }
  __device__ __forceinline__ static int store_off(int lane, int stride, int line0, int i) {
    return in(lane, line0, i) ? ((lane / kSpan) * stride + lane % kSpan) * 8 : kMixOob;
  }
  // scalar offset; base: the wave's first line
  __device__ __forceinline__ static int s(int i, int line0, int stride, int base) {
    return base + min(L * i, F - L - line0) * stride * 8 + CW * CH * 8;
  }
  __device__ __forceinline__ static int tile(int lane, int i) {
    return (L * i + lane / kSpan) * (CW + 4) + lane % kSpan;
  }
};

// The chunks whose outputs pass p (groups of outputs CW / 4 p ... of the
// inverse) leaves in a wave's two tiles: pairs of 188 are n1 and 47 - n1.
template <int F, int CW>
constexpr int kMixPasses = (Mix<F>::NP + CW / 4 - 1) / (CW / 4);
template <int F, int CW>
constexpr int mix_chunk(int pass, int slot) {
  return F == 188 ? (slot ? kMixChunks<F, CW> - 1 - pass : pass) : 2 * pass + slot;
}
template <int F, int CW>
constexpr int mix_slots(int pass) {
  const int c = mix_chunk<F, CW>(pass, 1);
  return c >= kMixChunks<F, CW> || c == mix_chunk<F, CW>(pass, 0) ? 1 : 2;
}

// LDS accesses of a wave run in program order; this keeps the compiler to it
// where lanes read what other lanes wrote
__device__ __forceinline__ void wave_lds_fence() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// chunk CH of the lines from the tile to the lanes: a[n1] = x[4 n1 + n2]
template <int F, int CW, int CH>
__device__ __forceinline__ void mix_take(float2 (&a)[Mix<F>::Q], const float2* tile,
                                         const MixLane& ln) {
  constexpr int N = CW / 4;
  wave_lds_fence();
#pragma unroll
  for (int k = 0; k < N; ++k)
    if (CH * N + k < Mix<F>::Q) {
      a[CH * N + k] = tile[ln.line * (CW + 4) + 4 * k + ln.n2];
      pin(a[CH * N + k]);
    }
  wave_lds_fence();
}

// the outputs of a pass to the two tiles
template <int F, int CW, int PASS>
__device__ __forceinline__ void mix_give(const float2 (&a)[Mix<F>::Q], float2* tiles,
                                         const MixLane& ln) {
  using C = Mix<F>;
  constexpr int N = CW / 4;
  wave_lds_fence();
  static_for<N * PASS, (N * PASS + N < C::NP ? N * PASS + N : C::NP)>([&](auto i) {
    float2 z[2];
    mix_inv_out<F, i>(a, z);
    static_for<0, 2>([&](auto e) {
      if constexpr (e == 0 || C::hasB(i)) {
        constexpr int n = mix_n<F>(i, e), ch = n / N;
        constexpr int slot = ch == mix_chunk<F, CW>(PASS, 0) ? 0 : 1;
        static_assert(ch == mix_chunk<F, CW>(PASS, slot), "the pass holds this chunk");
        tiles[slot * kMixTile<CW> + ln.line * (CW + 4) + 4 * (n % N) + ln.n2] = z[e];
      }
    });
    __builtin_amdgcn_sched_barrier(0);
  });
  wave_lds_fence();
}

// Slot (view * nblk + line block) of block b when every line block of a view
// runs on one XCD: the dispatcher sends block b to XCD b % 8, so XCD x takes
// the views v = x, x + 8, ... whole, one after the other; the cache lines that
// neighbouring line blocks share (intensities, ragged ends of rows) are then
// fetched into its L2 once.  Bijective on whole groups of 8 views; the remaining blocks keep
// their index.
__device__ __forceinline__ int xcd_view_slot(int b, int n, int nblk) {
  const int full = (n / (8 * nblk)) * (8 * nblk);
  if (b >= full) return b;
  const int x = b & 7, i = b >> 3;
  return (8 * (i / nblk) + x) * nblk + i % nblk;
}

// (1) Z = 2 P O - psi and the DFT along rows: one wave per 16 rows of a frame,
// a quarter of a chunk's psi, P and O in flight while the one before is used
// (more needs registers that cost a wave per SIMD).
// grid (views x LB, modes)
template <int F>
__global__ __launch_bounds__(64, 4) void k_mix_rows_fwd(const ScanDev* __restrict__ scans,
                                                        const int2* __restrict__ vmap,
                                                        const float2* __restrict__ tw, int M) {
  using C = Mix<F>;
  constexpr int Q = C::Q, FF = F * F, CW = kRowCW, NCH = kMixChunks<F, CW>;
  __shared__ float2 twl[4 * Q];
  __shared__ float2 tile[kMixTile<CW>];
  mix_load_twiddles<F>(tw, twl, threadIdx.x, 64);
  const int lane = threadIdx.x;
  const MixLane ln(lane);
  const int slot = xcd_view_slot(blockIdx.x, gridDim.x, C::LB);
  const int2 vm = vmap[slot / C::LB];
  const ScanDev& sc = scans[vm.x];
  const int j = uni(vm.y), m = blockIdx.y;
  const int line0 = (slot % C::LB) * 16;
  const int W = uni(sc.W);
  const int y0 = uni(kidx(sc.pos)[2 * j]), x0 = uni(kidx(sc.pos)[2 * j + 1]);
  const size_t frame = ((size_t)j * M + m) * FF;
  const rsrc_t rpsi = make_rsrc(sc.psi + frame, (uint32_t)(FF * 8));
  const rsrc_t rP = make_rsrc(sc.P + (size_t)m * FF, (uint32_t)(FF * 8));
  const rsrc_t rO = make_rsrc(sc.O, (uint32_t)((size_t)uni(sc.H) * W * 8));
  const int sF = line0 * F * 8, sO = ((y0 + line0) * W + x0) * 8;
  float2 a[Q];
  constexpr int U = 4;
  float2 s[2][U], p[2][U], o[2][U];
  // batch bt: quarter bt % 4 of chunk bt / 4
  auto load = [&](auto bt) {
    using K = MixIO<F, CW, bt / 4>;
    constexpr int i0 = (bt % 4) * U;
    asm volatile("" ::: "memory");
    const int vF = K::load_off(lane, F), vO = K::load_off(lane, W);
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (i0 + k < K::kI) {
        s[bt & 1][k] = bload2_nt(rpsi, vF, K::s(i0 + k, line0, F, sF));
        p[bt & 1][k] = bload2(rP, vF, K::s(i0 + k, line0, F, sF));
        o[bt & 1][k] = bload2(rO, vO, K::s(i0 + k, line0, W, sO));
      }
    asm volatile("" ::: "memory");
  };
  load(std::integral_constant<int, 0>{});
  static_for<0, 4 * NCH>([&](auto bt) {
    using K = MixIO<F, CW, bt / 4>;
    constexpr int i0 = (bt % 4) * U;
    if constexpr (bt + 1 < 4 * NCH) load(std::integral_constant<int, bt + 1>{});
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (i0 + k < K::kI) {
        const float2 phi = cmul(p[bt & 1][k], o[bt & 1][k]);
        tile[K::tile(lane, i0 + k)] =
            make_float2(2.f * phi.x - s[bt & 1][k].x, 2.f * phi.y - s[bt & 1][k].y);
      }
    if constexpr (bt % 4 == 3) mix_take<F, CW, bt / 4>(a, tile, ln);
  });
  const rsrc_t rT =
      make_rsrc(sc.tspec + ((size_t)j * M + m) * C::FT, (uint32_t)(C::FT * 8));
  const MixSpec<F> sp(ln, line0 + ln.line);
  mix_fwd<F>(a, twl, ln, [&](auto i, float2 x0v, float2 x1v) {
    const int v = sp.at(i, ln);
    bstore2_nt(rT, x0v, v, 0);
    bstore2_nt(rT, x1v, v, MixSpec<F>::kX1);
  });
}

// (2) DFT along the columns of 16 lines kx of every mode of one view, the mode
// sum, the modulus scale and the inverse DFT, in place in the spectrum buffer.
// A wave takes the modes w, w + NW, ... (one mode a wave up to 8 modes, above
// six waves): it transforms them one after the other, keeps the last one's
// spectrum in registers and transforms the others again once the scale is
// known.  With several waves the mode powers go through LDS: one slot of 2 NP x
// 64 per wave, then the scale.  A wave's tiles share its slot where they do not
// meet its powers, i.e. up to 8 modes; above they follow the scale (six waves,
// because eight would not fit).  A single mode needs only the tiles.
constexpr int kMixWaves = 8, kMixWavesMany = 6;
constexpr int mix_cols_waves(int M) { return M <= kMixWaves ? M : kMixWavesMany; }
template <int F>
constexpr size_t mix_cols_lds(int M) {
  const size_t slots = M == 1 ? 0 : (size_t)(mix_cols_waves(M) + 1) * 2 * Mix<F>::NP * 64 * 4;
  return slots +
         (M == 1 ? 1 : M > kMixWaves ? kMixWavesMany : 0) * 2 * kMixTile<kColCW> * sizeof(float2);
}

template <int F, bool ONE>
__global__ __launch_bounds__(ONE ? 64 : 64 * kMixWaves, F == 200 && !ONE ? 3 : 2) void k_mix_cols(
    const ScanDev* __restrict__ scans, const int2* __restrict__ vmap,
    const float2* __restrict__ tw, int M, int direct) {
  using C = Mix<F>;
  constexpr int Q = C::Q, NP = C::NP, FF = F * F, NE = 2 * NP, CW = kColCW;
  __shared__ float2 twl[4 * Q];
  extern __shared__ __align__(16) float pw[];  // [wave][NE][64], then the scale [NE][64]
  static_assert(2 * kMixTile<kColCW> * 8 <= NE * 64 * 4, "the tiles fit a wave's slot");
  const int t = threadIdx.x, nt = blockDim.x;
  mix_load_twiddles<F>(tw, twl, t, nt);
  const MixLane ln(t & 63);
  const int lane = t & 63, w = ONE ? 0 : uni(t >> 6), NW = ONE ? 1 : nt >> 6;
  const int slot = xcd_view_slot(blockIdx.x, gridDim.x, C::LB);
  const int2 vm = vmap[slot / C::LB];
  const ScanDev& sc = scans[vm.x];
  const int j = uni(vm.y);
  const int line0 = (slot % C::LB) * 16;
  const int line = line0 + ln.line;
  const rsrc_t rI = make_rsrc(sc.I + (size_t)j * FF, (uint32_t)(FF * 4));
  const float beta = sc.beta, inv_ff = 1.0f / (float)FF;
  // g = sqrt(I / S) / F^2 (0 where S vanishes), or beta g - 1/F^2 for the
  // update without psi
  auto scale = [&](float iv, float s) {
    const float g = (s > FLT_MIN) ? sqrtf(fmaxf(iv, 0.f) / s) * inv_ff : 0.f;
    return direct ? beta * g - inv_ff : g;
  };
  // frequency ky of entry e of a lane in place (h, b)
  auto freq = [&](int e, int h, int b) {
    const int i = e >> 1;
    return (h ? C::kB(i) : i) + Q * (b + 2 * (e & 1));
  };
  const int sT = line0 * C::LDT * 8;
  float2* const tiles = M <= kMixWaves
                            ? reinterpret_cast<float2*>(pw + w * NE * 64)
                            : reinterpret_cast<float2*>(pw + (NW + 1) * NE * 64) +
                                  w * 2 * kMixTile<CW>;
  float2 x[NE];
  const int nm = (M - w + NW - 1) / NW;  // this wave's modes
  for (int it = 0; it < 2 * nm - 1; ++it) {
    const int m = w + NW * (it < nm ? it : it - nm);
    const rsrc_t rT =
        make_rsrc(sc.tspec + ((size_t)j * M + m) * C::FT, (uint32_t)(C::FT * 8));
    float2 a[Q];
    {
      // three chunks of the lines in flight
      constexpr int NCH = kMixChunks<F, CW>, D = 3;
      float2 r[D][8];
      auto load = [&](auto c) {
        using K = MixIO<F, CW, c>;
        asm volatile("" ::: "memory");
        const int v = K::load_off(lane, C::LDT);
#pragma unroll
        for (int i = 0; i < K::kI; ++i) r[c % D][i] = bload2(rT, v, K::s(i, line0, C::LDT, sT));
        asm volatile("" ::: "memory");
      };
      static_for<0, D>(load);
      static_for<0, NCH>([&](auto c) {
        using K = MixIO<F, CW, c>;
#pragma unroll
        for (int i = 0; i < K::kI; ++i) tiles[K::tile(lane, i)] = r[c % D][i];
        if constexpr (c + D < NCH) load(std::integral_constant<int, c + D>{});
        mix_take<F, CW, c>(a, tiles, ln);
      });
    }
    mix_fwd<F>(a, twl, ln, [&](auto i, float2 x0v, float2 x1v) {
      x[2 * i] = x0v;
      x[2 * i + 1] = x1v;
    });
    if constexpr (ONE) {
      // the wave's own powers are the mode sum; batches of 8 intensities
      constexpr int U = 8;
#pragma unroll
      for (int e0 = 0; e0 < NE; e0 += U) {
        float iv[U];
#pragma unroll
        for (int k = 0; k < U; ++k)
          if (e0 + k < NE)
            iv[k] = bload1(rI, line < F ? (freq(e0 + k, ln.h, ln.b) * F + line) * 4 : kMixOob, 0);
#pragma unroll
        for (int k = 0; k < U; ++k)
          if (e0 + k < NE) x[e0 + k] = cscale(x[e0 + k], scale(iv[k], cabs2(x[e0 + k])));
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      float* const gs = pw + NW * NE * 64;
      if (it < nm) {
        float* const mine = pw + w * NE * 64 + lane;
        if (it == 0) {
#pragma unroll
          for (int e = 0; e < NE; ++e) mine[e * 64] = cabs2(x[e]);
        } else {
#pragma unroll
          for (int e = 0; e < NE; ++e) mine[e * 64] += cabs2(x[e]);
        }
        if (it + 1 < nm) continue;
        __syncthreads();
        // the block's threads share the scale's entries; an entry's place
        // follows from its lane
        for (int q = t; q < NE * 64; q += nt) {
          const int e = q >> 6;  // uniform in a wave
          const int ky = freq(e, ln.h, ln.b);
          const float iv = bload1(rI, line < F ? (ky * F + line) * 4 : kMixOob, 0);
          float s = 0.f;
          for (int k = 0; k < NW; ++k) s += pw[k * NE * 64 + q];
          gs[q] = scale(iv, s);
        }
        __syncthreads();
      }
#pragma unroll
      for (int e = 0; e < NE; ++e) x[e] = cscale(x[e], gs[e * 64 + lane]);
    }
    mix_inv_in<F>(x, a, twl, ln);
    static_for<0, kMixPasses<F, CW>>([&](auto pass) {
      mix_give<F, CW, pass>(a, tiles, ln);
      static_for<0, mix_slots<F, CW>(pass)>([&](auto slot) {
        using K = MixIO<F, CW, mix_chunk<F, CW>(pass, slot)>;
#pragma unroll
        for (int i = 0; i < K::kI; ++i)
          bstore2(rT, tiles[slot * kMixTile<CW> + K::tile(lane, i)],
                  K::store_off(lane, C::LDT, line0, i), K::s(i, line0, C::LDT, sT));
      });
    });
  }
}

// (3) inverse DFT along rows, psi' = psi + beta (Z' - P O), the view's object
// numerator sum_m conj(P_m) psi'_m and the eps_psi partial sums for 16 rows of
// a view.  A wave takes the modes w, w + NW, ... (NW = min(M, kMixWaves) waves);
// the outputs of its transform go to two tiles, two chunks of columns a pass,
// where the update finds them row by row and leaves the mode's part of the
// numerator in their place, to be added over the waves.  DIRECT: the
// column kernel scaled the spectra by beta g - 1/F^2, the inverse is beta Z' -
// Z, and psi' = (2 - beta) P O + that (Eq. 3 with psi = 2 P O - Z): psi is not
// read and the eps_psi partials are zero.
template <int F>
constexpr size_t mix_inv_lds(int M) {
  return (size_t)(M < kMixWaves ? M : kMixWaves) * 2 * kMixTile<kRowCW> * sizeof(float2);
}

template <int F, bool DIRECT, bool ONE>
__global__ __launch_bounds__(ONE ? 64 : 64 * kMixWaves, 2) void k_mix_rows_inv(
    const ScanDev* __restrict__ scans, const int2* __restrict__ vmap,
    const float2* __restrict__ tw, int M) {
  using C = Mix<F>;
  constexpr int Q = C::Q, NP = C::NP, FF = F * F, CW = kRowCW;
  __shared__ float2 twl[4 * Q];
  __shared__ float red[kMixWaves][2];
  extern __shared__ float2 tiles[];  // [wave][2][tile]
  const int t = threadIdx.x, nt = blockDim.x;
  mix_load_twiddles<F>(tw, twl, t, nt);
  const int lane = t & 63, w = ONE ? 0 : uni(t >> 6), NW = ONE ? 1 : nt >> 6;
  const MixLane ln(lane);
  float2* const mine = tiles + w * 2 * kMixTile<CW>;
  const int bslot = xcd_view_slot(blockIdx.x, gridDim.x, C::LB);
  const int2 vm = vmap[bslot / C::LB];
  const ScanDev& sc = scans[vm.x];
  const int j = uni(vm.y);
  const int lb = bslot % C::LB, line0 = lb * 16;
  const int W = uni(sc.W);
  const float beta = sc.beta;
  const int y0 = uni(kidx(sc.pos)[2 * j]), x0 = uni(kidx(sc.pos)[2 * j + 1]);
  const MixSpec<F> sp(ln, line0 + ln.line);
  const int sF = line0 * F * 8;
  const rsrc_t rO = make_rsrc(sc.O, (uint32_t)((size_t)uni(sc.H) * W * 8));
  const int sO = ((y0 + line0) * W + x0) * 8;
  const rsrc_t ropart = make_rsrc(sc.opart + (size_t)j * FF, (uint32_t)(FF * 8));
  float e_d = 0.f, e_n = 0.f;
  for (int m0 = 0; m0 < M; m0 += NW) {
    // keeps what one round reads (the twiddles) out of the registers of the next
    asm volatile("" ::: "memory");
    const int m = m0 + w;
    const bool on = ONE || m < M;  // uniform in a wave
    const size_t frame = ((size_t)j * M + (on ? m : 0)) * FF;
    const rsrc_t rT = make_rsrc(sc.tspec + ((size_t)j * M + (on ? m : 0)) * C::FT,
                                (uint32_t)(C::FT * 8));
    const rsrc_t rpsi = make_rsrc(sc.psi + frame, (uint32_t)(FF * 8));
    const rsrc_t rP = make_rsrc(sc.P + (size_t)(on ? m : 0) * FF, (uint32_t)(FF * 8));
    float2 a[Q];
    if (on) {
      float2 x[2 * NP];
      static_for<0, NP>([&](auto i) {
        const int v = sp.at(i, ln);
        x[2 * i] = bload2_nt(rT, v, 0);
        x[2 * i + 1] = bload2_nt(rT, v, MixSpec<F>::kX1);
      });
      mix_inv_in<F>(x, a, twl, ln);
    }
    static_for<0, kMixPasses<F, CW>>([&](auto pass) {
      constexpr int kSlots = mix_slots<F, CW>(pass);
      if (on) {
        // the update of the pass's chunks, four indices a batch: the first
        // batch's operands are in flight over the outputs, then the next one's
        constexpr int U = 4, NB = kSlots * 4;
        float2 p[2][U], o[2][U], s[2][U];
        auto load = [&](auto bt) {
          using K = MixIO<F, CW, mix_chunk<F, CW>(pass, bt / 4)>;
          constexpr int i0 = (bt % 4) * U;
          asm volatile("" ::: "memory");
          const int vF = K::load_off(lane, F), vO = K::load_off(lane, W);
#pragma unroll
          for (int k = 0; k < U; ++k)
            if (i0 + k < K::kI) {
              p[bt & 1][k] = bload2(rP, vF, K::s(i0 + k, line0, F, sF));
              o[bt & 1][k] = bload2(rO, vO, K::s(i0 + k, line0, W, sO));
              if constexpr (!DIRECT) s[bt & 1][k] = bload2_nt(rpsi, vF, K::s(i0 + k, line0, F, sF));
            }
          asm volatile("" ::: "memory");
        };
        load(std::integral_constant<int, 0>{});
        mix_give<F, CW, pass>(a, mine, ln);
        static_for<0, NB>([&](auto bt) {
          using K = MixIO<F, CW, mix_chunk<F, CW>(pass, bt / 4)>;
          constexpr int i0 = (bt % 4) * U;
          if constexpr (bt + 1 < NB) load(std::integral_constant<int, bt + 1>{});
#pragma unroll
          for (int k = 0; k < U; ++k)
            if (i0 + k < K::kI) {
              const int v = K::store_off(lane, F, line0, i0 + k);
              const int sr = K::s(i0 + k, line0, F, sF);
              const bool in = K::in(lane, line0, i0 + k);
              float2* const cell = mine + (bt / 4) * kMixTile<CW> + K::tile(lane, i0 + k);
              const float2 z = *cell, pp = p[bt & 1][k];
              const float2 phi = cmul(pp, o[bt & 1][k]);
              float2 pn;
              if constexpr (DIRECT) {
                pn = make_float2((2.f - beta) * phi.x + z.x, (2.f - beta) * phi.y + z.y);
              } else {
                const float2 d = make_float2(beta * (z.x - phi.x), beta * (z.y - phi.y));
                pn = cadd(s[bt & 1][k], d);
                e_d += in ? cabs2(d) : 0.f;
              }
              e_n += in ? cabs2(pn) : 0.f;
              bstore2_nt(rpsi, pn, v, sr);
              const float2 q = cmulc(pp, pn);
              if constexpr (ONE) bstore2(ropart, q, v, sr);
              else *cell = q;
            }
        });
      }
      if constexpr (!ONE) {
        const int nw = min(NW, M - m0);
        __syncthreads();
        static_for<0, kSlots>([&](auto slot) {
          using K = MixIO<F, CW, mix_chunk<F, CW>(pass, slot)>;
          for (int i = w; i < K::kI; i += NW) {
            const int v = K::store_off(lane, F, line0, i), so = K::s(i, line0, F, sF);
            float2 q = m0 ? bload2(ropart, v, so) : make_float2(0.f, 0.f);
            for (int k = 0; k < nw; ++k)
              q = cadd(q, tiles[(k * 2 + slot) * kMixTile<CW> + K::tile(lane, i)]);
            bstore2(ropart, q, v, so);
          }
        });
        __syncthreads();
      }
    });
  }
  e_d = wave_sum(e_d);
  e_n = wave_sum(e_n);
  if constexpr (!ONE) {
    if (lane == 0) { red[w][0] = e_d; red[w][1] = e_n; }
    __syncthreads();
    e_d = e_n = 0.f;
    for (int k = 0; k < NW; ++k) { e_d += red[k][0]; e_n += red[k][1]; }
  }
  if (t == 0) {
    const int part = j * C::LB + lb;
    sc.err_psi[2 * part] = e_d;
    sc.err_psi[2 * part + 1] = e_n;
  }
}

}  // namespace dmk
