// Cutting an fp32 tensor into two fp16 planes, shared by the kernels that multiply fp32 operands on the
// fp16 matrix cores with three piece products per fp32 product (igemm_f32_p3.hip, conv_k3_f32.hip,
// conv_k3v_f32.hip, conv_k3c64_f32.hip).
//
//   A tensor gets one power-of-two scale 2^se chosen from its largest magnitude so that the scaled values
//   stay below 2^15 (se = 141 - biased exponent of the largest magnitude; scaling by a power of two is
//   exact).  A scaled value v is cut into
//       h1 = fp16(v)                      (round to nearest: 11 significant bits)
//       H2 = fp16((v - h1) * 2^11)        (the remainder, exact in fp32, scaled up so that it keeps fp16's
//                                          normal range wherever h1 does; 11 more bits)
//   so v = h1 + 2^-11 H2 up to 2^-22 |v| (each piece rounds at half a unit of its 11th bit; typically a quarter
//   of that).  A product of two such values is taken as
//       h1 h1'  +  2^-11 (h1 H2' + H2 h1')
//   with v_mfma_f32_32x32x16_f16, which multiplies fp16 exactly and accumulates in fp32: the first term into
//   one accumulator set, the two cross terms into a second one that is scaled by 2^-11 and added at the end,
//   and the sum is scaled back by 2^-(se + se').  Dropped: 2^-22 H2 H2', at most 2^-22 of |v v'|; with the cuts'
//   own rounding a product is within 3 * 2^-22 of |v v'| in the worst case, a few times the rounding an fp32
//   multiply-add makes anyway and far below what accumulating a long reduction in fp32 adds.
//   Values more than 2^28 below the tensor's largest magnitude fall under fp16's normal range after scaling.  Planes in
//   memory carry them by H2 alone (h1 = 0) with 11 significant bits, an absolute error below 2^-39 of the largest magnitude,
//   and the product of two such values (one from each operand, below 2^-56 of the largest product) is dropped; an operand
//   cut inside a kernel keeps the subnormal h1 and H2 with what is left, an error below 2^-50.
#pragma once
#include <hip/hip_runtime.h>

namespace glowmi {

typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

constexpr float kLowPieceWeight = 0x1p-11f;            // weight of the second accumulator set

// Scale exponent of a tensor from the bits of its largest magnitude (sign cleared).
__device__ __forceinline__ int scale_exponent(unsigned max_bits) {
  int eb = (int)(max_bits >> 23) & 0xff;
  if (eb < 1) eb = 1;                                  // all zero (or subnormal): any scale will do
  return 141 - eb;
}

// Largest of the lanes' words: every lane returns it.  Lane permutations inside the vector unit (DPP): neighbours, pairs,
// halves of a row of 16, rows, then row ends to the rows behind them; lane 63 has seen all.
__device__ __forceinline__ unsigned wave_max_u32(unsigned m) {
  auto take = [&m](unsigned o) { m = o > m ? o : m; };
  take((unsigned)__builtin_amdgcn_update_dpp((int)m, (int)m, 0xB1, 0xf, 0xf, false));    // quad_perm [1,0,3,2]
  take((unsigned)__builtin_amdgcn_update_dpp((int)m, (int)m, 0x4E, 0xf, 0xf, false));    // quad_perm [2,3,0,1]
  take((unsigned)__builtin_amdgcn_update_dpp((int)m, (int)m, 0x141, 0xf, 0xf, false));   // row_half_mirror
  take((unsigned)__builtin_amdgcn_update_dpp((int)m, (int)m, 0x140, 0xf, 0xf, false));   // row_mirror
  take((unsigned)__builtin_amdgcn_update_dpp((int)m, (int)m, 0x142, 0xa, 0xf, false));   // row_bcast15 into rows 1 and 3
  take((unsigned)__builtin_amdgcn_update_dpp((int)m, (int)m, 0x143, 0xc, 0xf, false));   // row_bcast31 into rows 2 and 3
  return (unsigned)__builtin_amdgcn_readlane((int)m, 63);
}

// Largest of n words at src, by one wavefront on its own (no LDS, no barrier); every lane returns it.
__device__ __forceinline__ unsigned wave_max_words(const unsigned* __restrict__ src, int n) {
  unsigned m = 0;
  for (int i = (int)(threadIdx.x & 63); i < n; i += 64) {
    const unsigned v = src[i];
    m = v > m ? v : m;
  }
  return wave_max_u32(m);
}

// Largest magnitude (bits) among 8 * N prefetched values held as N pairs of float4: of the lane, over the wavefront.  A NaN
// among numbers is left out of it (an infinity is not): it reaches the results it belongs to through its pieces.
template <int N, typename V4>
__device__ __forceinline__ unsigned lane_max_of(const V4 (&pre)[N][2]) {
  float m = 0.f;
#pragma unroll
  for (int q = 0; q < N; ++q)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 4; e += 2)                   // magnitudes are a source modifier, and no quieting in front
        asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(pre[q][h][e]), "v"(pre[q][h][e + 1]));
  return __builtin_bit_cast(unsigned, m) & 0x7fffffffu;
}
template <int N, typename V4>
__device__ __forceinline__ unsigned wave_max_of(const V4 (&pre)[N][2]) { return wave_max_u32(lane_max_of(pre)); }

// The largest of the eight words the wavefronts of a workgroup left at `words` (LDS).
__device__ __forceinline__ unsigned max_of_eight(const unsigned* words) {
  const v4u a = *reinterpret_cast<const v4u*>(words), b = *reinterpret_cast<const v4u*>(words + 4);
  unsigned m = a[0];
#pragma unroll
  for (int e = 1; e < 4; ++e) m = a[e] > m ? a[e] : m;
#pragma unroll
  for (int e = 0; e < 4; ++e) m = b[e] > m ? b[e] : m;
  return (unsigned)__builtin_amdgcn_readfirstlane((int)m);
}

// The cut as planes in memory hold it (a form that callers may keep): below fp16's normal range h1 is zero and the second
// piece carries the value.
__device__ __forceinline__ void cut8(const float (&v)[8], int se, v4u& p1, v4u& p2) {
  _Float16 h1[8], h2[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float x = __builtin_ldexpf(v[i], se);
    h1[i] = (_Float16)x;
    if (__builtin_fabsf(x) < 0x1p-14f) h1[i] = (_Float16)0.f;
    h2[i] = (_Float16)((x - (float)h1[i]) * 2048.f);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    p1[i] = __builtin_bit_cast(unsigned, v2h{h1[2 * i], h1[2 * i + 1]});
    p2[i] = __builtin_bit_cast(unsigned, v2h{h2[2 * i], h2[2 * i + 1]});
  }
}

// The cut inside a kernel: 3.5 instructions a value instead of ten (scale, 2^11 times that, half a packed conversion, and
// the remainder as one fma from fp16 back to fp16).  A subnormal h1 stays: the matrix instructions keep it.
__device__ __forceinline__ void cut8_in_place(const float (&x)[8], int se, v4u& p1, v4u& p2) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const v2f v = {__builtin_ldexpf(x[2 * i], se), __builtin_ldexpf(x[2 * i + 1], se)};
    const v2h h1 = __builtin_convertvector(v, v2h);    // round to nearest
    const v2h h2 = {(_Float16)__builtin_fmaf((float)h1[0], -2048.f, v[0] * 2048.f),
                    (_Float16)__builtin_fmaf((float)h1[1], -2048.f, v[1] * 2048.f)};   // exact before the one rounding
    p1[i] = __builtin_bit_cast(unsigned, h1);
    p2[i] = __builtin_bit_cast(unsigned, h2);
  }
}
struct Cut2 { _Float16 h1, h2; };
__device__ __forceinline__ Cut2 cut2(float x, int se) {
  const float v = __builtin_ldexpf(x, se);
  Cut2 c;
  c.h1 = (_Float16)v;
  c.h2 = (_Float16)__builtin_fmaf((float)c.h1, -2048.f, v * 2048.f);
  return c;
}

// A filter's planes in memory hold pieces of eight reduction indices, 16 bytes each, in one of two orders, and the first word
// behind them says which:
//   rows        [output channel][reduction / 8], one scale: word 0 is the bits of the tensor's largest magnitude;
//   by channel  [reduction / 8][output channel], the order conv_patch_f32 reads best, a scale per output channel: word i is the
//               bits of channel i's largest magnitude, word 0 with kByChannel.
// Every kernel over planes reads either, so planes made once serve the filter whichever kernel a call takes.
constexpr unsigned kByChannel = 0x80000000u;
struct PlaneOrder {
  unsigned row, piece;                                   // bytes from a channel's piece to the next channel's, to its next piece
  bool by_channel;
  // words: behind the planes; pieces: of a channel; known: made in this call by conv_patch_f32, whose order needs no asking (a
  // trip to memory ahead of the first fragments: 0.4 us of a residual block)
  __device__ __forceinline__ PlaneOrder(const unsigned* words, int channels, int pieces, bool known = false) {
    by_channel = true;
    if (!known) by_channel = (__builtin_amdgcn_readfirstlane((int)words[0]) & (int)kByChannel) != 0;   // uniform
    set(channels, pieces);
  }
  // the same from the first word itself
  __device__ __forceinline__ PlaneOrder(unsigned first_word, int channels, int pieces) {
    by_channel = (__builtin_amdgcn_readfirstlane((int)first_word) & (int)kByChannel) != 0;
    set(channels, pieces);
  }
  __device__ __forceinline__ void set(int channels, int pieces) {
    row = by_channel ? 16u : 16u * (unsigned)pieces;
    piece = by_channel ? 16u * (unsigned)channels : 16u;
  }
  // the bits of the largest magnitude that channel ch was scaled by
  __device__ __forceinline__ unsigned max_bits(const unsigned* words, int ch) const { return words[by_channel ? (unsigned)ch : 0u] & ~kByChannel; }
};

// The two operands' largest magnitudes (bits) -> what the accumulators are scaled back by, and what is added to
// every result: 0, or NaN when an operand holds an infinity or a NaN (its largest "magnitude" is then not finite and
// no scale fits: the whole call's results are NaN rather than finite numbers that are wrong).
struct ScaleBack { int neg_se; float poison; };
__device__ __forceinline__ ScaleBack scale_back(unsigned x_max_bits, unsigned w_max_bits) {
  ScaleBack s;
  s.neg_se = -(scale_exponent(x_max_bits) + scale_exponent(w_max_bits));
  const bool finite = x_max_bits < 0x7f800000u && w_max_bits < 0x7f800000u;
  s.poison = finite ? 0.f : __builtin_nanf("");
  return s;
}
// The same from the scale exponents in use and whether every magnitude seen was finite.
__device__ __forceinline__ ScaleBack scale_back_of(int se_x, int se_w, bool finite) {
  ScaleBack s;
  s.neg_se = -(se_x + se_w);
  s.poison = finite ? 0.f : __builtin_nanf("");
  return s;
}

// A finished sum from the two accumulator sets of scaled operands.
__device__ __forceinline__ float join_sets(float hi, float lo, ScaleBack sb) {
  return __builtin_ldexpf(__builtin_fmaf(lo, kLowPieceWeight, hi), sb.neg_se) + sb.poison;
}

}  // namespace glowmi
