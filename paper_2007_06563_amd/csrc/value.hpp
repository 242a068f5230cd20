// MCMK convolution on float32 values: the same arithmetic as the bitsliced
// kernels (kernels.hpp), bit for bit, computed one value per lane instead of
// 32 per word.
//
// Why: a bitsliced MAC of (5,3) -> (5,4) takes 203 instructions per 32 values,
// 6.3 a value, and its smallest piece of work is a wave of 2,048 accumulator
// chains that no reordering may split; a layer of a few hundred such waves
// leaves most of the chip idle. One float32 operation per step of the MAC takes
// 7 instructions a value (4 rounding toward zero) up to 10 fraction bits in the
// accumulator, 13 to 16 above to nearest (float64 ones counted twice), and its
// smallest piece is 64 chains.
//
// How float32 gives the format's own results. A value of (wE, wF) is an exact
// float32. Operands are scaled by powers of two, so that the format's smallest
// normal number is float32's, 2^-126, in products and sums.
//  - Product. With K = 2^k + 1, k = 23 - wF_acc: c = RN(K w x),
//    d = RN(c - w x), r = c - d is the product rounded to wF_acc fraction bits
//    (Veltkamp's splitting). w x has at most 2 (wF_in + 1) <= 22 bits, so 2^k w x
//    is an even multiple of c's last place and c's own rounding, ties to even,
//    is the one asked for; d is then exactly 2^k w x. K w (or K x) is exact.
//    Types whose products are exact in the accumulator skip this.
//  - Sum. s = RN(acc + r) in float32, then the same splitting of s. Rounding
//    twice gives the single rounding's result for the sum of two numbers of p
//    bits when the first rounding keeps at least 2p + 1 bits: p = wF_acc + 1
//    <= 11. Ties of the second rounding have p + 1 bits, so the argument above
//    holds for them too.
//    Wider accumulators rounding to nearest are held and added in float64 (53
//    bits: p <= 26), split by the same steps.
//  - Toward zero, float32's own rounding is set toward zero and the bits below
//    the format's last place are cleared; truncating twice is exact for any p.
//  - Underflow. The hardware mode flushes float32 results below 2^-126 to a
//    zero of their sign: the rounded product r is produced by a subtraction
//    whose exact result it is, so it is flushed after rounding as the format
//    asks, and a sum below the smallest normal number is always exact, so
//    flushing it before rounding is the same. Of float64's operations only
//    products are flushed, so there the sum passes through one.
//  - Zero signs are IEEE's in every step.
//  - Overflow and inputs that are infinite or NaN do not fit this. The workgroup
//    knows the largest operands staged so far and the chunks of taps that hold an
//    infinity or NaN; such a chunk, and one whose sums could leave the format's range
//    by those operands and the sums before it, takes a slower route (careful_chunk),
//    wave by wave. The bitsliced kernels take one time for all inputs; this one:
//    8x56x56x64 -> 64, 576 taps, (5,3) -> (5,4): ordinary inputs 147 us, an infinity
//    in each image 151, 1 % infinities or nothing but NaN 186, the largest finite
//    number in each image 204, bitsliced 157; (4,3) -> (4,4) with sums that overflow
//    everywhere 216, bitsliced 151.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "codec.hpp"
#include "kernels.hpp"
#include "lanes.hpp"

#pragma clang fp contract(off)

namespace hobflops {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) float lds_f32;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;

__device__ __forceinline__ float pow2f(int e) { return __int_as_float((e + 127) << 23); }

// The arithmetic of one variant V (wE, wF_IN, wF_ACC, wF_OUT, kRound, kAct).
template <class V>
struct ValueMath {
  static constexpr int wE = V::wE, wI = V::wF_IN, wA = V::wF_ACC;
  static constexpr bool kRtz = V::kRound != 0;
  static constexpr bool kExact = wA >= 2 * wI + 1;  // products are exact in the accumulator
  static constexpr bool kWide = !kRtz && wA > 10;   // sums in float64
  using Acc = typename std::conditional<kWide, double, float>::type;
  static constexpr int kBias = (1 << (wE - 1)) - 1;
  // products and sums are scaled by 2^kScale, IFM values by 2^kScaleX
  static constexpr int kScale = -126 + kBias, kScaleX = kScale / 2;
  static constexpr int k = 23 - wA;
  static constexpr uint32_t kMask = ~((1u << k) - 1u);
  // The smallest nonzero product is 2^(-126 - kBias) scaled; where 2^k times it
  // would be flushed, c and d are formed 2^kLift larger and r scaled back (one
  // more instruction): a flushed d beside a normal c would not cancel.
  static constexpr int kLift = kRtz || kExact || k >= kBias ? 0 : kBias - k;
  static constexpr int kScaleW = kScale - kScaleX + kLift;
  // exponent of the first power of two out of range
  static constexpr int kTop = (1 << wE) - kBias;
  // What the steps rest on (and product on a bound of its own): products and sums
  // scaled as above, and the plain sum of products of the slower route, stay in
  // float32's range; an accumulator value is a float32 with bits to round at. The
  // kernels round their result once more, by quantize_narrow, whose additions follow
  // the hardware's rounding mode: set_mode makes that the variant's own.
  static_assert(wE >= 2 && wE <= 6, "scaled values and products leave float32's range");
  static_assert(wA >= wI && wA <= 22 && V::wF_OUT <= 22, "no bit of float32 to round at");
  // The smallest sum out of range before its rounding, scaled: to nearest, half a
  // unit in the last place below 2^kTop rounds up to it (a tie goes to 2^kTop, whose
  // last place is even).
  static constexpr uint32_t kOverflow =
      ((uint32_t)(127 + kTop + kScale) << 23) - (kRtz ? 0u : 1u << (k - 1));
  // Sums that start at |acc| <= A and take up to 32 terms of at most P (before
  // their rounding) stay in range if A + 32 P < kRoom 2^kTop. With u half a unit in
  // the last place of 1, a term grows by 1 + u when rounded, and a rounding adds at
  // most 2^kTop u / 2 while the sums are in range, or a factor of 1 + u.
  static constexpr double room() {
    if (kRtz) return 1.0 - 0x1p-20;  // the estimate's own rounding
    const double u = 1.0 / (double)(2LL << wA);
    double f = 1.0;
    for (int i = 0; i < 33; ++i) f /= 1.0 + u;
    const double a = 1.0 - 16.0 * u;
    return (1.0 - 0x1p-20) / (1.0 + u) * (a > f ? a : f);
  }
  static constexpr float kRoom = (float)room();

  // MODE: float32 rounding nearest or toward zero; float32 results and float64
  // products below the smallest normal number flushed, such operands read as
  // they are (bits 5:4 and 7:6 = 1).
  static __device__ __forceinline__ void set_mode() {
    __builtin_amdgcn_s_setreg(1 | (0 << 6) | (7 << 11), 0x50 | (kRtz ? 3 : 0));
  }
  static __device__ __forceinline__ float trunc(float v) {
    return __uint_as_float(__float_as_uint(v) & kMask);
  }
  // the multiplier's second form of a weight: K w
  static __device__ __forceinline__ float prescale(float w) {
    return kRtz || kExact ? w : w * (float)((1 << k) + 1);
  }
  static __device__ __forceinline__ float product(float w, float wk, float x) {
    if constexpr (kRtz) return kExact ? w * x : trunc(w * x);
    if constexpr (kExact) return w * x;
    static_assert(kRtz || kExact || wI <= 10, "2^k w x is no even multiple of c's last place");
    const float c = wk * x;
    const float d = __builtin_fmaf(-w, x, c);
    const float r = c - d;
    return kLift ? r * pow2f(-kLift) : r;
  }
  // acc + r in the format; a float64 accumulator is scaled by 2^-896 more, so
  // that 2^-1022 is the format's smallest normal number. With kTrack, track takes the
  // largest magnitude of the term and of the sum before its rounding, NaN apart.
  template <bool kTrack>
  static __device__ __forceinline__ Acc add(Acc acc, float r, float& track) {
    if constexpr (kWide) {
      // float64 additions keep numbers below 2^-1022, the multiplication does not
      const double t = __builtin_fma(acc, 0x1p896, (double)r);
      if constexpr (kTrack) track_max(track, (float)t, r);
      const double s = t * 0x1p-896;
      const double u = s * (double)((1LL << (52 - wA)) + 1);
      const double v = u - s;
      return u - v;
    } else {
      const float s = acc + r;
      if constexpr (kTrack) track_max(track, s, r);
      if constexpr (kRtz) return trunc(s);
      const float u = s * (float)((1 << k) + 1);
      const float v = u - s;
      return u - v;
    }
  }
  static __device__ __forceinline__ void track_max(float& track, float a, float b) {
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(track) : "v"(a), "v"(b));
  }
  // the accumulator's value, unscaled (exact), and back
  static __device__ __forceinline__ float value(Acc acc) {
    if constexpr (kWide) return (float)(acc * __builtin_ldexp(1.0, 896 - kScale));
    return acc * pow2f(-kScale);
  }
  static __device__ __forceinline__ Acc scaled(float v) {
    if constexpr (kWide) return (double)v * __builtin_ldexp(1.0, kScale - 896);
    return v * pow2f(kScale);
  }
  // the accumulator's magnitude, scaled like a float32 one; NaN as it is
  static __device__ __forceinline__ float magnitude(Acc acc) {
    if constexpr (kWide) return __builtin_fabsf((float)(acc * 0x1p896));
    return __builtin_fabsf(acc);
  }
  static __device__ __forceinline__ bool finite(float v) { return v - v == 0.0f; }
  // The same step on unscaled values with every check written out: infinities
  // and NaN follow IEEE-754, overflow gives a signed infinity.
  static __device__ __forceinline__ float range(float v) {
    uint32_t b = __float_as_uint(v);
    const uint32_t a = b & 0x7FFFFFFFu, s = b & 0x80000000u;
    b = a < (uint32_t)(127 - kBias) << 23 ? s : b;
    b = a >= (uint32_t)(127 + kTop) << 23 && a <= 0x7F800000u ? s | 0x7F800000u : b;
    return __uint_as_float(b);
  }
  static __device__ __forceinline__ float round_checked(float v) {
    uint32_t b = __float_as_uint(v);
    if constexpr (!kRtz) b += ((b >> k) & 1u) + ((1u << (k - 1)) - 1u);
    return range(__uint_as_float((b & kMask) | (v != v ? 0x7FC00000u : 0u)));
  }
  static __device__ __forceinline__ float add_checked(float acc, float r) {
    if constexpr (kWide) {
      const double s = (double)acc + (double)r;
      const double u = s * (double)((1LL << (52 - wA)) + 1);
      const double v = u - s;
      return s - s == 0.0 ? range((float)(u - v)) : (float)s;  // infinite and NaN sums as they are
    } else {
      return round_checked(acc + r);
    }
  }
  static __device__ __forceinline__ float mac_checked(float acc, float w, float x) {
    return add_checked(acc, round_checked((w * pow2f(-kScaleX - kScaleW)) * x));
  }
  // The largest magnitude of an operand (a product of operands) for which no
  // sum of `taps` of them can reach 2^kTop: rounding is monotone, so the sums
  // stay below those of `taps` equal terms P rounded up, which grow by P (1 + u)
  // a tap, u half a unit in the last place, and stop growing at 2^(wF + 2) P,
  // where P is less than half a unit of the sum.
  static double bound(double taps) {
    const double u = ldexp(1.0, -(wA + 1));
    const double grow = taps * (kRtz ? 1.0 : exp(2.0 * taps * u)), stop = ldexp(1.0, wA + 2);
    return ldexp(1.0, kTop) * (1.0 - 4.0 * u) / (grow < stop ? grow : stop);
  }
};

// Code -> float32 scaled by 2^scale. kChecked: infinities and NaN as
// float32's; otherwise such codes give some number (the caller looks for them).
template <int wE, int wF, int kScale, bool kChecked>
__device__ __forceinline__ uint32_t decode_scaled(uint32_t code) {
  constexpr int sh_s = wF + wE;
  constexpr uint32_t bias = (uint32_t)(127 - ((1 << (wE - 1)) - 1) + kScale) << 23;
  const uint32_t v = (__builtin_amdgcn_ubfe(code, 0, sh_s) << (23 - wF)) + bias;
  const uint32_t x0 = (uint32_t)__builtin_amdgcn_sbfe((int)code, sh_s + 1, 1);
  uint32_t mag = x0 & v;
  if constexpr (kChecked) {
    const uint32_t x1 = (uint32_t)__builtin_amdgcn_sbfe((int)code, sh_s + 2, 1);
    mag = x1 ? 0x7F800000u | (x0 & 0x00400000u) : mag;
  }
  // v_bfi: the sign bit from the shifted code
  return __builtin_amdgcn_bitop3_b32(0x7FFFFFFFu, mag, code << (31 - sh_s), 0xCA);
}

constexpr int kRow = 36;  // floats of an LDS row: 32 taps, rows 16-byte aligned, 4 banks apart

// A workgroup of WP x WM waves computes 2 RP WP positions x 32 RM WM kernels.
// A wave holds RM m-tiles x 2 RP positions: lane j of half h kernel j of each
// m-tile and positions h RP .. h RP + RP - 1, RM * RP chains a lane.
//
// Taps are taken in the fixed order in chunks of at most 32: the channels of
// one (ky, kx, channel word), or, where a channel word holds fewer than
// kFlatC channels, 32 consecutive taps across pixels. For a chunk the workgroup
// turns the plane words of its positions and weight rows into float32 values
// in LDS ([position][tap] and [kernel][tap]); every MAC operand is then read
// four taps at a time, an IFM value as a broadcast within each half wave. The
// words of the next chunk are loaded while this one is computed, and the LDS
// tiles are double buffered, so there is one barrier a chunk. A chunk is filled
// up to a multiple of four taps with w = -0, x = +0: adding -0 changes nothing.
//
// Staging goes by sets of four 32-value groups, one per row of 16 lanes, a
// plane word a lane (two where a code has more than 16 bits), through the
// lane transpose; a set leaves two words a lane.
template <class V, int RM, int RP, int WP, int WM>
struct ValueTile {
  static constexpr int kWaves = WP * WM, kThreads = 64 * kWaves;
  static constexpr int kPos = 2 * RP * WP, kKern = 32 * RM * WM;
  static constexpr int kXSets = (kPos + 3) / 4, kWSets = kKern / 4;
  static constexpr int XS = (kXSets + kWaves - 1) / kWaves, WS = (kWSets + kWaves - 1) / kWaves;
};

template <class V, bool kFlat, int RM, int RP, int WP, int WM>
__global__ __launch_bounds__(64 * WP * WM) void conv2d_value_kernel(
    const uint32_t* __restrict__ ifm, const uint32_t* __restrict__ w, uint32_t* __restrict__ ofm,
    ConvParams p, float bound) {
  using T = ValueTile<V, RM, RP, WP, WM>;
  using A = ValueMath<V>;
  constexpr int NIN = V::NIN, NOUT = V::NOUT, XS = T::XS, WS = T::WS, NW = T::kWaves;
  constexpr bool kHigh = NIN > 16;  // a second plane word a lane
  __shared__ float xs[2][T::kXSets * 4][kRow];
  __shared__ float ws[2][T::kKern][kRow];
  __shared__ float nonfinite[RM * RP][T::kThreads];  // see the careful step
  // What the staging waves found (see `found`): the largest finite codes of x and of
  // w so far, their signs apart; the number of chunks from which on sums have to be
  // looked at or, while that is not so, of chunks up to the last one with an infinity
  // or NaN; and the latter number.
  __shared__ alignas(16) uint32_t seen[4];

  const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wp = wave % WP, wm = wave / WP;
  const int p0 = blockIdx.x * T::kPos, mt0 = blockIdx.y * (RM * WM);
  const int taps = p.KH * p.KW * p.C;
  const int nch = kFlat ? (taps + 31) / 32 : p.KH * p.KW * p.CG;
  if (tid < 4) seen[tid] = 0u;

  // staging: this lane's group of a set, and its plane
  const int row = lane >> 4, l = lane & 15;
  const int grp = ((row & 1) << 1) | (row >> 1);
  const RowT rt = row_transpose_setup(l);
  // byte offset of tap (0, 0)'s plane word, and that tap's input row and column
  uint32_t xoff[XS];
  int xiy[XS], xix[XS];
  auto place = [&](int i, int* n) {  // position i of the tile -> tap (0, 0) and image
    const int q = p0 + i < p.P ? p0 + i : 0;
    const int ox = q % p.OW, t = q / p.OW, oy = t % p.OH;
    *n = t / p.OH;
    // a position past the end has no tap inside its image
    return make_int2(p0 + i < p.P && i < T::kPos ? oy * p.stride - p.pad : -(1 << 30),
                     ox * p.stride - p.pad);
  };
#pragma unroll
  for (int i = 0; i < XS; ++i) {
    int n;
    const int2 e = place(4 * (wave + i * NW) + grp, &n);
    xiy[i] = e.x;
    xix[i] = e.y;
    // modulo 2^32 (positions past the end and taps above the image are never read)
    const uint32_t at = (uint32_t)(n * p.H + e.x) * (uint32_t)p.W + (uint32_t)e.y;
    xoff[i] = (at * (uint32_t)(p.CG * NIN) + min(l, NIN - 1)) * 4u;
  }

  struct Chunk {
    int ky, kx, cg, tap0, nc;
  };
  auto advance = [&](Chunk& c) {
    c.tap0 += c.nc;
    if constexpr (kFlat) {
      c.nc = min(32, taps - c.tap0);
    } else {
      if (++c.cg == p.CG) {
        c.cg = 0;
        if (++c.kx == p.KW) {
          c.kx = 0;
          ++c.ky;
        }
      }
      c.nc = min(32, p.C - 32 * c.cg);
    }
  };
  auto inside = [&](int i, const Chunk& c) {
    return (uint32_t)(xiy[i] + c.ky) < (uint32_t)p.H && (uint32_t)(xix[i] + c.kx) < (uint32_t)p.W;
  };
  auto word = [](const uint32_t* base, uint32_t byte) {
    return *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(base) + byte);
  };
  const uint32_t hi_step = (uint32_t)(min(l + 16, NIN - 1) - min(l, NIN - 1)) * 4u;
  struct Raw {
    uint32_t x[XS][kHigh ? 2 : 1], w[WS][kHigh ? 2 : 1];
  };
  auto fetch = [&](const Chunk& c, Raw& raw) {
    if constexpr (!kFlat) {
      // modulo 2^32: a tap row beside the image may lie far past it
      const uint32_t d = (((uint32_t)c.ky * (uint32_t)p.W + (uint32_t)c.kx) * (uint32_t)p.CG +
                          (uint32_t)c.cg) * (uint32_t)(4 * NIN);
#pragma unroll
      for (int i = 0; i < XS; ++i) {
        const uint32_t o = inside(i, c) ? xoff[i] + d : 0u;
        raw.x[i][0] = word(ifm, o);
        if constexpr (kHigh) raw.x[i][1] = word(ifm, o + (inside(i, c) ? hi_step : 0u));
      }
    }
#pragma unroll
    for (int i = 0; i < WS; ++i) {
      const int s = min(wave + i * NW, T::kWSets - 1);
      const int t = 4 * (s & 7) + grp, mt = min(mt0 + (s >> 3), p.MT - 1);
      const uint32_t o =
          ((uint32_t)(c.tap0 + min(t, c.nc - 1)) * (uint32_t)p.MT + mt) * (uint32_t)(4 * NIN) +
          (uint32_t)min(l, NIN - 1) * 4u;
      raw.w[i][0] = word(w, o);
      if constexpr (kHigh) raw.w[i][1] = word(w, o + hi_step);
    }
  };
  // the codes of a flat chunk's IFM values, bit by bit: lane j is tap tap0 + j
  auto gather = [&](const Chunk& c, int i) {
    const int t = c.tap0 + min(j, c.nc - 1), s = t / p.C, ch = t - s * p.C;
    int n;
    const int2 e = place(i, &n);
    const int iy = e.x + s / p.KW, ix = e.y + s % p.KW;
    const bool ok = (uint32_t)iy < (uint32_t)p.H && (uint32_t)ix < (uint32_t)p.W && j < c.nc;
    const uint32_t* src = ifm + (ok ? (uint32_t)((n * p.H + iy) * p.W + ix) * (uint32_t)NIN : 0u);
    uint32_t q[NIN], code = 0u;
    __builtin_memcpy(q, src, 4 * NIN);
#pragma unroll
    for (int b = 0; b < NIN; ++b) code |= __builtin_amdgcn_ubfe(q[b], ch, 1) << b;
    return ok ? code : 0u;
  };
  // Reports the largest codes of x and of w that a lane staged for chunk ch, special if
  // one of the wave's is an infinity or NaN (cx, cw are then the largest finite ones).
  constexpr uint32_t kSignBit = 1u << (A::wE + A::wI), kSpecial = 4u * kSignBit;
  auto found = [&](uint32_t cx, uint32_t cw, bool special, int ch) {
    volatile uint32_t* const s = &seen[0];
    const uint32_t ux = wave_max(cx), uw = wave_max(cw);
    if (lane != 0) return;
    if (special) s[3] = (uint32_t)(ch + 1);
    atomicMax(&seen[0], ux);
    atomicMax(&seen[1], uw);
    __threadfence_block();
    // read after both: of two waves that each raise one, the later finds both
    const float big = __uint_as_float(decode_scaled<A::wE, A::wI, A::kScaleX, false>(s[0])) *
                      __uint_as_float(decode_scaled<A::wE, A::wI, A::kScaleW, false>(s[1]));
    if (special || !(big < bound)) atomicMax(&seen[2], big < bound ? (uint32_t)(ch + 1) : ~0u);
  };
  // The same number, computed where it is used: the addresses of rarely taken
  // branches then do not hold registers throughout the loop.
  auto here = [](int v) {
    asm volatile("" : "+v"(v));
    return v;
  };
  // Raw words of chunk ch -> float32 values of buffer ch & 1. Infinities and NaN are
  // noticed by their codes, which are larger than the finite ones': sx and sw are the
  // largest ones that earlier chunks are known to hold.
  auto stage = [&](const Chunk& c, Raw& raw, int ch, uint32_t sx, uint32_t sw) {
    const int buf = ch & 1;
    auto put_x = [&](int i, int j, uint32_t code, auto checked) {
      xs[buf][i][j] = __uint_as_float(
          decode_scaled<A::wE, A::wI, A::kScaleX, decltype(checked)::value>(code));
    };
    auto put_w = [&](int kern, int t, uint32_t code, auto checked) {
      ws[buf][kern][t ^ 2] = __uint_as_float(  // see the MAC
          decode_scaled<A::wE, A::wI, A::kScaleW, decltype(checked)::value>(code));
    };
    const uint32_t keep = c.nc < 32 ? (1u << c.nc) - 1u : ~0u;
    // all of this wave's sets through the transpose together: its steps depend
    // on each other, so one set alone would wait at each
    constexpr int X = kFlat ? 0 : XS;
    uint32_t P[X + WS], Q[X + WS];
#pragma unroll
    for (int i = 0; i < X; ++i) {
      const bool ok = inside(i, c);
      P[i] = ok && l < NIN ? raw.x[i][0] & keep : 0u;
      Q[i] = 0u;
      if constexpr (kHigh) Q[i] = ok && l + 16 < NIN ? raw.x[i][1] & keep : 0u;
    }
#pragma unroll
    for (int i = 0; i < WS; ++i) {
      const int t = 4 * ((wave + i * NW) & 7) + grp;
      static_assert(A::wE + A::wI < 16);  // the sign is among the first word's planes
      const uint32_t fill = l == A::wE + A::wI ? ~0u : 0u;  // -0
      P[X + i] = t < c.nc ? (l < NIN ? raw.w[i][0] : 0u) : fill;
      Q[X + i] = 0u;
      if constexpr (kHigh) Q[X + i] = t < c.nc && l + 16 < NIN ? raw.w[i][1] : 0u;
    }
    row_transpose(P, rt);
    if constexpr (kHigh) row_transpose(Q, rt);
#pragma unroll
    for (int i = 0; i < X + WS; ++i) {  // the words of groups h and 2 + h
      uint32_t a, b;
      stage16_from_pairs(P[i], Q[i], a, b);
      P[i] = a;
      Q[i] = b;
    }
    uint32_t a[XS], b[XS];  // the codes of groups h and 2 + h of the sets of x
#pragma unroll
    for (int i = 0; i < XS; ++i) {
      const int s = wave + i * NW;
      if (T::kXSets % NW != 0 && s >= T::kXSets) break;  // uniform
      if constexpr (kFlat) {
        a[i] = gather(c, 4 * s + h);
        b[i] = gather(c, 4 * s + 2 + h);
      } else {
        a[i] = P[i];
        b[i] = Q[i];
      }
    }
    // the largest codes, their signs apart: of all, or of the finite ones
    auto put_all = [&](uint32_t& cx, uint32_t& cw, int lane, auto checked) {
      const int j = lane & 31, h = lane >> 5;
      auto key = [&](uint32_t code) {
        code &= ~kSignBit;
        return decltype(checked)::value && code >= kSpecial ? 0u : code;
      };
      cx = cw = 0u;
#pragma unroll
      for (int i = 0; i < XS; ++i) {
        const int s = wave + i * NW;
        if (T::kXSets % NW != 0 && s >= T::kXSets) break;  // uniform
        put_x(4 * s + h, j, a[i], checked);
        put_x(4 * s + 2 + h, j, b[i], checked);
        cx = max(cx, max(key(a[i]), key(b[i])));
      }
#pragma unroll
      for (int i = 0; i < WS; ++i) {
        const int s = wave + i * NW;
        if (T::kWSets % NW != 0 && s >= T::kWSets) break;  // uniform
        const int kern = (s >> 3) * 32 + j, t0 = 4 * (s & 7) + h;
        put_w(kern, t0, P[X + i], checked);
        put_w(kern, t0 + 2, Q[X + i], checked);
        cw = max(cw, max(key(P[X + i]), key(Q[X + i])));
      }
    };
    uint32_t cx, cw;
    put_all(cx, cw, lane, std::false_type{});
    if (__builtin_expect(__any(cx > sx || cw > sw), 0)) {
      const bool special = __any(max(cx, cw) >= kSpecial);
      if (special) put_all(cx, cw, here(lane), std::true_type{});
      found(cx, cw, special, ch);
    }
  };

  A::set_mode();
  typename A::Acc acc[RM][RP];
#pragma unroll
  for (int m = 0; m < RM; ++m)
#pragma unroll
    for (int r = 0; r < RP; ++r) acc[m][r] = 0;

  // The MACs of four taps.
  auto four = [&](const f32x4(&xv)[RP], const f32x4(&wv)[RM]) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
      for (int m = 0; m < RM; ++m) {
        // weights lie two taps apart from the IFM values in their group of
        // four, so that the two operands of a tap, each loaded four to an
        // aligned register quad, come from different VGPR banks
        const float wt = wv[m][t ^ 2], wk = A::prescale(wt);
        float none = 0.0f;
#pragma unroll
        for (int r = 0; r < RP; ++r)
          acc[m][r] = A::template add<false>(acc[m][r], A::product(wt, wk, xv[r][t]), none);
      }
    }
  };

  // A chunk with an infinity or NaN among the workgroup's operands, or (kTrack) in
  // which a sum may leave the range. The steps of `four` make NaN of a special
  // operand and of the chain that meets it, for good; what IEEE-754 makes of that
  // chain (an infinity of either sign, or NaN) comes from the plain sum of its
  // products, whose finite part is not used, kept beside the accumulator: in LDS
  // between such chunks. Sums out of range are looked for after each few taps, which
  // are then taken again one by one with the range checks written out.
  bool kept = false;  // nonfinite is set (uniform over the wave)
  auto careful_chunk = [&](int buf, int nt, auto tracked) {
    constexpr bool kTrack = decltype(tracked)::value;
    constexpr int S = A::kWide ? 2 : 4;  // taps a step: what the registers hold
    typedef float vec __attribute__((ext_vector_type(S)));
    typedef __attribute__((address_space(3))) vec lds_vec;
    const int tid = here(threadIdx.x), j = tid & 31, h = (tid >> 5) & 1;
    const lds_f32* xb = (const lds_f32*)&xs[buf][(wp * 2 + h) * RP][0];
    const lds_f32* wb = (const lds_f32*)&ws[buf][wm * RM * 32 + j][0];
    float nf[RM][RP];
#pragma unroll
    for (int m = 0; m < RM; ++m)
#pragma unroll
      for (int r = 0; r < RP; ++r) nf[m][r] = kept ? nonfinite[m * RP + r][tid] : 0.0f;
#pragma unroll 1
    for (int t0 = 0; t0 < nt; t0 += S) {
      vec xv[RP], wv[RM];
#pragma unroll
      for (int r = 0; r < RP; ++r) xv[r] = *(const lds_vec*)(xb + r * kRow + t0);
#pragma unroll
      for (int m = 0; m < RM; ++m)
        wv[m] = *(const lds_vec*)(wb + m * 32 * kRow + (S == 2 ? t0 ^ 2 : t0));
      auto w_of = [&](int m, int t) { return wv[m][S == 2 ? t : t ^ 2]; };
      typename A::Acc before[RM][RP];
      float track = 0.0f;
#pragma unroll
      for (int m = 0; m < RM; ++m)
#pragma unroll
        for (int r = 0; r < RP; ++r) before[m][r] = acc[m][r];
#pragma unroll
      for (int t = 0; t < S; ++t)
#pragma unroll
        for (int m = 0; m < RM; ++m) {
          const float wt = w_of(m, t), wk = A::prescale(wt);
#pragma unroll
          for (int r = 0; r < RP; ++r) {
            float p = A::product(wt, wk, xv[r][t]);
            // an infinity that came through the product as one becomes NaN
            if constexpr (A::kRtz || A::kExact) p = __builtin_fmaf(p, 0.0f, p);
            acc[m][r] = A::template add<kTrack>(acc[m][r], p, track);
          }
        }
      if (!kTrack || !__any(!(track < __uint_as_float(A::kOverflow)))) {
#pragma unroll
        for (int t = 0; t < S; ++t)
#pragma unroll
          for (int m = 0; m < RM; ++m)
#pragma unroll
            for (int r = 0; r < RP; ++r) nf[m][r] = __builtin_fmaf(w_of(m, t), xv[r][t], nf[m][r]);
        continue;
      }
      float out[RM][RP];
#pragma unroll
      for (int m = 0; m < RM; ++m)
#pragma unroll
        for (int r = 0; r < RP; ++r)
          out[m][r] = A::finite(nf[m][r]) ? A::value(before[m][r]) : nf[m][r];
#pragma unroll 1
      for (int t = t0; t < t0 + S; ++t) {
        float x1[RP], w1[RM];
#pragma unroll
        for (int r = 0; r < RP; ++r) x1[r] = xb[r * kRow + t];
#pragma unroll
        for (int m = 0; m < RM; ++m) w1[m] = wb[m * 32 * kRow + (t ^ 2)];
#pragma unroll
        for (int m = 0; m < RM; ++m)
#pragma unroll
          for (int r = 0; r < RP; ++r) out[m][r] = A::mac_checked(out[m][r], w1[m], x1[r]);
      }
#pragma unroll
      for (int m = 0; m < RM; ++m)
#pragma unroll
        for (int r = 0; r < RP; ++r) {
          const bool ok = A::finite(out[m][r]);
          nf[m][r] = ok ? 0.0f : out[m][r];
          acc[m][r] = A::scaled(ok ? out[m][r] : __builtin_nanf(""));
        }
    }
#pragma unroll
    for (int m = 0; m < RM; ++m)
#pragma unroll
      for (int r = 0; r < RP; ++r) nonfinite[m * RP + r][tid] = nf[m][r];
    kept = true;
  };

  // All chunks in order: step ch computes chunk ch and stages chunk ch + 1; the
  // first only stages.
  __syncthreads();
  Chunk nx{0, 0, 0, 0, kFlat ? min(32, taps) : min(32, p.C)};
  int nq = 0;  // groups of four taps of the chunk to compute
  Raw raw;
  for (int ch = -1; ch < nch; ++ch) {
    const bool more = ch + 1 < nch;
    if (more) fetch(nx, raw);
    const lds_f32* xb = (const lds_f32*)&xs[ch & 1][(wp * 2 + h) * RP][0];
    const lds_f32* wb = (const lds_f32*)&ws[ch & 1][wm * RM * 32 + j][0];
    auto load = [&](int q, f32x4(&xv)[RP], f32x4(&wv)[RM]) {
#pragma unroll
      for (int r = 0; r < RP; ++r) xv[r] = *(const lds_f32x4*)(xb + r * kRow + 4 * q);
#pragma unroll
      for (int m = 0; m < RM; ++m) wv[m] = *(const lds_f32x4*)(wb + m * 32 * kRow + 4 * q);
    };
    // What is known of chunk ch's operands. Another wave may have staged the next
    // chunk by now: its operands then count as well, which is on the safe side.
    const u32x4 now = *(volatile lds_u32x4*)&seen[0];
    uint32_t sx = 0u, sw = 0u;  // now's, for the staging
    auto fast_chunk = [&] {
      // operands of the next four taps are requested before this four's MACs
      f32x4 xa[RP], wa[RM], xc[RP], wc[RM];
      load(0, xa, wa);
      int q = 0;
      for (; q + 2 <= nq; q += 2) {
        load(q + 1, xc, wc);
        four(xa, wa);
        load(q + 2 < nq ? q + 2 : q, xa, wa);
        four(xc, wc);
      }
      if (q < nq) four(xa, wa);
    };
    // The chunk's route, from the sums before it: 0 the fast one, 1 with care for
    // infinities and NaN, 2 for sums that leave the range as well.
    auto route = [&](const typename A::Acc(&sum)[RM][RP]) {
      sx = __builtin_amdgcn_readfirstlane(now.x);
      sw = __builtin_amdgcn_readfirstlane(now.y);
      if (__builtin_expect(__builtin_amdgcn_readfirstlane(now.z) <= (uint32_t)ch, 1)) return 0;
      const float big = __uint_as_float(decode_scaled<A::wE, A::wI, A::kScaleX, false>(sx)) *
                        __uint_as_float(decode_scaled<A::wE, A::wI, A::kScaleW, false>(sw));
      float a = 0.0f;
#pragma unroll
      for (int m = 0; m < RM; ++m)
#pragma unroll
        for (int r = 0; r < RP; ++r) A::track_max(a, A::magnitude(sum[m][r]), 0.0f);
      if (__any(!(a + 32.0f * (big * pow2f(-A::kLift)) < A::kRoom * pow2f(A::kTop + A::kScale))))
        return 2;
      return __builtin_amdgcn_readfirstlane(now.w) > (uint32_t)ch ? 1 : 0;
    };
    if constexpr (T::kWaves <= 8) {
      // Two waves a SIMD would wait for the route's answer: the chunk is computed first
      // and again where it needs care (14x14x256 -> 256 at batch 16, 56x64 tiles: 310
      // us with the route chosen before, 303). Care is of one kind here, as two of them
      // between staging and barrier cost 4 %.
      if (nq > 0) {
        typename A::Acc before[RM][RP];
#pragma unroll
        for (int m = 0; m < RM; ++m)
#pragma unroll
          for (int r = 0; r < RP; ++r) before[m][r] = acc[m][r];
        fast_chunk();
        if (__builtin_expect(route(before) != 0, 0)) {
#pragma unroll
          for (int m = 0; m < RM; ++m)
#pragma unroll
            for (int r = 0; r < RP; ++r) acc[m][r] = before[m][r];
          careful_chunk(ch & 1, 4 * nq, std::true_type{});
        }
      }
    } else if (nq > 0) {
      const int kind = route(acc);
      if (kind == 0)
        fast_chunk();
      else if (kind == 1)
        careful_chunk(ch & 1, 4 * nq, std::false_type{});
      else
        careful_chunk(ch & 1, 4 * nq, std::true_type{});
    }
    if (more) stage(nx, raw, ch + 1, sx, sw);
    nq = (nx.nc + 3) >> 2;
    advance(nx);
    __syncthreads();
  }
  float out[RM][RP];
#pragma unroll
  for (int m = 0; m < RM; ++m)
#pragma unroll
    for (int r = 0; r < RP; ++r) out[m][r] = A::value(acc[m][r]);
  if (kept) {
#pragma unroll
    for (int m = 0; m < RM; ++m)
#pragma unroll
      for (int r = 0; r < RP; ++r) {
        const float nf = nonfinite[m * RP + r][tid];
        if (!A::finite(nf)) out[m][r] = nf;
      }
  }

  // Epilogue: activation, conversion to the output format, store. Lane j of a
  // half holds kernel 32 mt + j of a position: planes come out of the lane
  // transpose, values and codes are stored 32 lanes side by side.
#pragma unroll
  for (int m = 0; m < RM; ++m) {
    const int mt = mt0 + wm * RM + m;
    uint32_t code[RP + (RP & 1)];
#pragma unroll
    for (int r = 0; r < RP + (RP & 1); ++r) {
      const float v = r < RP ? out[m][r < RP ? r : 0] : 0.0f;
      uint32_t b = __float_as_uint(v);
      if constexpr (V::kAct != 0) b = (b & 0x80000000u) != 0u && v == v ? 0u : b;
      code[r] = quantize_narrow(b, V::wE, V::wF_OUT);
    }
    if (p.ofm_kind == kOfmPlanes) {
      lane_transpose(code, j);
#pragma unroll
      for (int r = 0; r < RP; ++r) {
        const int pos = p0 + (wp * 2 + h) * RP + r;
        if (pos < p.P && mt < p.MT && j < NOUT) ofm[((size_t)pos * p.MT + mt) * NOUT + j] = code[r];
      }
    } else {
      const int kern = mt * 32 + j;
#pragma unroll
      for (int r = 0; r < RP; ++r) {
        const int pos = p0 + (wp * 2 + h) * RP + r;
        const uint32_t v = p.ofm_kind == kOfmF32 ? decode_narrow(code[r], V::wE, V::wF_OUT) : code[r];
        if (pos < p.P && kern < p.M) ofm[(size_t)pos * p.M + kern] = v;
      }
    }
  }
}

// Global average pooling on values, for few (image, channel word) groups: the
// bitsliced kernel gives a group to a lane, whose chain of H W adds of some 130
// instructions then sets the time (16x7x7x1024, (5,4): 512 such lanes, 15.4 us).
// Here a half wave takes a group, a lane a channel: a set (see the convolution)
// is two positions of the wave's two groups, its words are loaded kAhead sets
// together, and each value is added in four operations. About 10 instructions
// per group and position instead of 2, so the bitsliced kernel keeps launches of
// many groups (launch_pool).
template <class V>
__global__ __launch_bounds__(256) void avgpool_value_kernel(const uint32_t* __restrict__ in,
                                                            uint32_t* __restrict__ out,
                                                            PoolParams p) {
  using A = ValueMath<V>;
  constexpr int NIN = V::NIN, NOUT = V::NOUT, kAhead = 8, kSign = V::wE + V::wF_IN;
  constexpr bool kHigh = NIN > 16;
  const int lane = threadIdx.x & 63, j = lane & 31, h = lane >> 5;
  const int row = lane >> 4, l = lane & 15;
  const int64_t groups = (int64_t)p.N * p.CG;
  const int64_t first = 2 * ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6));
  if (first >= groups) return;  // uniform over the wave
  // row r of a set: group first + (r >> 1), position (r & 1) of the two
  const int64_t q = first + (row >> 1) < groups ? first + (row >> 1) : groups - 1;
  const int64_t n = q / p.CG, cg = q - n * p.CG;
  const uint32_t* src = in + ((size_t)n * p.HW * p.CG + cg) * NIN;
  const size_t step = (size_t)p.CG * NIN;
  const int lo = min(l, NIN - 1), hi = min(l + 16, NIN - 1);
  const RowT rt = row_transpose_setup(l);
  const PoolPairs pairs{(uint32_t)p.HW};
  // Every position in order, 2 kAhead at a time. Where those hold an infinity or NaN
  // or their sums may leave the range, and once a sum of the wave is infinite or
  // NaN, they are added again with the range checks written out.
  static_assert(2 * kAhead <= 32);  // of kRoom
  uint32_t mx = 0u;
  A::set_mode();
  typename A::Acc acc = 0;
  float none = 0.0f;
  for (uint32_t s0 = 0; pairs.more(s0); s0 += kAhead) {
    uint32_t P[kAhead], Q[kAhead], any = 0u;
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const uint32_t* at = src + (size_t)pairs.at(s0 + k, row & 1) * step;
      P[k] = at[lo];
      Q[k] = kHigh ? at[hi] : 0u;
    }
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const bool have = pairs.have(s0 + k, row & 1);
      // past the end: -0, which changes no sum
      P[k] = have ? (l < NIN ? P[k] : 0u) : (l == kSign ? ~0u : 0u);
      if constexpr (kHigh) Q[k] = have ? (l + 16 < NIN ? Q[k] : 0u) : (l + 16 == kSign ? ~0u : 0u);
      any |= kHigh ? Q[k] : P[k];
    }
    const bool special = __any(l == ((NIN - 1) & 15) && any != 0u);
    row_transpose(P, rt);
    if constexpr (kHigh) row_transpose(Q, rt);
    const typename A::Acc before = acc;
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      uint32_t a, b;
      stage16_from_pairs(P[k], Q[k], a, b);
      P[k] = a;
      Q[k] = b;
      const uint32_t va = decode_scaled<V::wE, V::wF_IN, A::kScale, false>(a);
      const uint32_t vb = decode_scaled<V::wE, V::wF_IN, A::kScale, false>(b);
      mx = max(mx, max(va & 0x7FFFFFFFu, vb & 0x7FFFFFFFu));
      acc = A::template add<false>(acc, __uint_as_float(va), none);
      acc = A::template add<false>(acc, __uint_as_float(vb), none);
    }
    const float most = A::magnitude(before) + (float)(2 * kAhead) * __uint_as_float(mx);
    if (__builtin_expect(__any(special || !(most < A::kRoom * pow2f(A::kTop + A::kScale))), 0)) {
      float v = A::value(before);
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {
        v = A::add_checked(v, __uint_as_float(decode_scaled<V::wE, V::wF_IN, 0, true>(P[k])));
        v = A::add_checked(v, __uint_as_float(decode_scaled<V::wE, V::wF_IN, 0, true>(Q[k])));
      }
      acc = A::scaled(v);
    }
  }
  const float v = A::value(acc);
  // the product of two accumulator values is exact in float32
  static_assert(2 * (V::wF_ACC + 1) <= 24);
  const float scale =
      __uint_as_float(decode_scaled<V::wE, V::wF_ACC, 0, true>(p.scale));
  uint32_t code[2] = {quantize_narrow(__float_as_uint(v * scale), V::wE, V::wF_OUT), 0u};
  lane_transpose(code, j);
  if (first + h < groups && j < NOUT) out[(size_t)(first + h) * NOUT + j] = code[0];
}

// Tile shapes (RM, RP, WP, WM) of the kernel, largest first; the choice among
// them and the bitsliced kernels is made by value_plan (abi.hip).
template <class V, int RM, int RP, int WP, int WM>
hipError_t launch_value_tile(const uint32_t* ifm, const uint32_t* w, uint32_t* ofm,
                             const ConvParams& p, float bound, hipStream_t stream) {
  using T = ValueTile<V, RM, RP, WP, WM>;
  const dim3 grid((unsigned)((p.P + T::kPos - 1) / T::kPos),
                  (unsigned)((p.MT + RM * WM - 1) / (RM * WM)));
  if constexpr (T::kPos <= 32 && RM == 1) {
    if (p.C < kFlatC) {
      hipLaunchKernelGGL((conv2d_value_kernel<V, true, RM, RP, WP, WM>), grid, dim3(T::kThreads),
                         0, stream, ifm, w, ofm, p, bound);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((conv2d_value_kernel<V, false, RM, RP, WP, WM>), grid, dim3(T::kThreads), 0,
                     stream, ifm, w, ofm, p, bound);
  return hipGetLastError();
}

template <class V>
hipError_t launch_value(const uint32_t* ifm, const uint32_t* w, uint32_t* ofm, const ConvParams& p,
                        int tile, hipStream_t stream) {
  // of the product of the largest x and w as the kernel scales them
  using A = ValueMath<V>;
  const float bound = (float)ldexp(A::bound((double)p.KH * p.KW * p.C), A::kScale + A::kLift);
  switch (tile) {
    case kTile112x64: return launch_value_tile<V, 1, 7, 8, 2>(ifm, w, ofm, p, bound, stream);
    case kTile56x64: return launch_value_tile<V, 1, 7, 4, 2>(ifm, w, ofm, p, bound, stream);
    case kTile32x64: return launch_value_tile<V, 2, 2, 8, 1>(ifm, w, ofm, p, bound, stream);
    case kTile32x32: return launch_value_tile<V, 1, 2, 8, 1>(ifm, w, ofm, p, bound, stream);
    case kTile16x32: return launch_value_tile<V, 1, 1, 8, 1>(ifm, w, ofm, p, bound, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace hobflops
