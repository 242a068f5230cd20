// Bit transposes across the lanes of a wave, without LDS: 32 codes held one per
// lane <-> the plane words of their 32-value group. Used by the pack and unpack
// kernels and by the convolution on float32 values.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hobflops {

// 32 x 32 bit transpose across each 32-lane half of a wave: lane j returns
// the word whose bit i is bit j of lane i's x. Five stages d = 16, 8, 4, 2, 1
// swap the off-diagonal d x d blocks of lane pairs (j, j ^ d): the lower lane
// takes its partner's bits i (i & d == 0) into positions i + d, the upper one
// its partner's bits i + d into positions i. The stages act on disjoint pairs
// of (lane bit, word bit) coordinates, so they may run in any order.
//
// No stage goes through LDS. The stages d = 8, 4, 2, 1 stay inside 16-lane
// rows: a DPP move brings the partner's word (row rotate by 8, quad
// permutes, and for d = 4 a mirror of each 8 lanes followed by the quad
// permute j ^ 3), then one rotate and one bit select (v_bitop3_b32, truth
// table 0xCA: mask ? r : x) with per-lane rotate amounts and masks set up once
// (row_transpose_setup). The stage d = 16 pairs rows 0-1 and 2-3 of a wave;
// it takes two words a, b at once: v_permlane16_swap_b32 gives every lane of
// row 0 the words of a's lanes j and j + 16 and every lane of row 1 those of
// b's, and two byte permutes form P (low halves) and Q (high halves). After
// it, row 0 (2) of P holds a's result at lanes 0-15 of its half and row 0 (2)
// of Q a's result at lanes 16-31, rows 1 and 3 the same for b ("pair
// layout"); a second swap of P and Q gives back the plain layout.
struct RowT {
  uint32_t rot[4], mask[4];  // stages d = 8, 4, 2, 1
};

__device__ __forceinline__ RowT row_transpose_setup(int j) {
  RowT t;
  constexpr uint32_t kLow[4] = {0x00FF00FFu, 0x0F0F0F0Fu, 0x33333333u, 0x55555555u};
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int d = 8 >> s;
    const bool upper = (j & d) != 0;
    t.rot[s] = upper ? d : 32 - d;               // rotate right: by d, or left by d
    t.mask[s] = upper ? kLow[s] : ~kLow[s];      // the positions taken from the partner
  }
  return t;
}

// The word of lane j ^ (8 >> S) of the same 16-lane row (DPP moves).
template <int S>
__device__ __forceinline__ uint32_t row_xor(uint32_t x) {
  if constexpr (S == 0) {
    return __builtin_amdgcn_mov_dpp(x, 0x128, 0xF, 0xF, false);  // row_ror:8
  } else if constexpr (S == 1) {
    const uint32_t m = __builtin_amdgcn_mov_dpp(x, 0x141, 0xF, 0xF, false);  // j ^ 7
    return __builtin_amdgcn_mov_dpp(m, 0x1B, 0xF, 0xF, false);  // quad_perm [3,2,1,0]: j ^ 3
  } else if constexpr (S == 2) {
    return __builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
  } else {
    return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
  }
}

// The largest x of the wave, the same in every lane.
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
  x = max(x, row_xor<0>(x));
  x = max(x, row_xor<1>(x));
  x = max(x, row_xor<2>(x));
  x = max(x, row_xor<3>(x));
  auto row = [&](int lane) { return (uint32_t)__builtin_amdgcn_readlane(x, lane); };
  const uint32_t a = max(row(0), row(16)), b = max(row(32), row(48));
  return max(a, b);
}

// The stages d = 8, 4, 2, 1 on N words.
template <int N>
__device__ __forceinline__ void row_transpose(uint32_t (&x)[N], const RowT& t) {
#define HOBFLOPS_STAGE(S)                                                       \
  {                                                                             \
    uint32_t p[N];                                                              \
    _Pragma("unroll") for (int u = 0; u < N; ++u) p[u] = row_xor<S>(x[u]);      \
    _Pragma("unroll") for (int u = 0; u < N; ++u) {                             \
      const uint32_t r = __builtin_amdgcn_alignbit(p[u], p[u], t.rot[S]);       \
      x[u] = __builtin_amdgcn_bitop3_b32(t.mask[S], r, x[u], 0xCA);             \
    }                                                                           \
  }
  HOBFLOPS_STAGE(0)
  HOBFLOPS_STAGE(1)
  HOBFLOPS_STAGE(2)
  HOBFLOPS_STAGE(3)
#undef HOBFLOPS_STAGE
}

// Exchanges rows 1 and 3 of a with rows 0 and 2 of b.
__device__ __forceinline__ void row_swap(uint32_t& a, uint32_t& b) {
  const auto s = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = s[0];
  b = s[1];
}

// Low and high 16-bit halves of two words: lo = lo16(a) | lo16(b) << 16,
// hi = hi16(a) | hi16(b) << 16.
__device__ __forceinline__ uint32_t halves_lo(uint32_t a, uint32_t b) {
  return __builtin_amdgcn_perm(b, a, 0x05040100u);
}
__device__ __forceinline__ uint32_t halves_hi(uint32_t a, uint32_t b) {
  return __builtin_amdgcn_perm(b, a, 0x07060302u);
}

// The stage d = 16 on words a, b in the plain layout; P and Q in the pair
// layout. kHigh false: the words' high halves are zero and Q (then zero) is
// not formed.
template <bool kHigh>
__device__ __forceinline__ void stage16_to_pairs(uint32_t a, uint32_t b, uint32_t& P,
                                                 uint32_t& Q) {
  row_swap(a, b);
  P = halves_lo(a, b);
  if constexpr (kHigh) Q = halves_hi(a, b);
}

// The stage d = 16 on words a, b given in the pair layout (P: a's lanes 0-15
// in row 0 and b's in row 1, Q: their lanes 16-31; rows 2 and 3 likewise for
// the wave's second half); a and b come out in the plain layout.
__device__ __forceinline__ void stage16_from_pairs(uint32_t P, uint32_t Q, uint32_t& a,
                                                   uint32_t& b) {
  a = halves_lo(P, Q);
  b = halves_hi(P, Q);
  row_swap(a, b);
}

// Whole transpose, plain layout in and out, of U (even) words.
template <int U>
__device__ __forceinline__ void lane_transpose(uint32_t (&x)[U], int j) {
  static_assert(U % 2 == 0, "words go through the d = 16 stage in pairs");
  uint32_t P[U / 2], Q[U / 2];
#pragma unroll
  for (int v = 0; v < U / 2; ++v) stage16_to_pairs<true>(x[2 * v], x[2 * v + 1], P[v], Q[v]);
  const RowT t = row_transpose_setup(j);
  row_transpose(P, t);
  row_transpose(Q, t);
#pragma unroll
  for (int v = 0; v < U / 2; ++v) {
    row_swap(P[v], Q[v]);
    x[2 * v] = P[v];
    x[2 * v + 1] = Q[v];
  }
}

// Group (within the chunk's pass set) of a lane's word of pair v in the pair
// layout: row r of the passes (2v, 2v + 1) holds group
// 2 (2v + (r & 1)) + (r >> 1); the lane's plane is lane & 15 in P, 16 more
// in Q.
__device__ __forceinline__ int pair_group(int v, int lane) {
  const int r = lane >> 4;
  return 4 * v + 2 * (r & 1) + (r >> 1);
}

}  // namespace hobflops
