// Pieces shared by the int8 kernels that walk the reduction in 16-code chunks (igemm_i8.hip, conv_small_i8.hip).  A chunk
// never straddles a filter tap: a tap of cg channels has ceil(cg / 16) chunks, the last one with cg % 16 codes (or 16).
// One load then fetches a chunk at any channel count, 16 bytes at whatever byte address the pixel's channels start; the
// bytes past the tap's channels belong to the next pixel (filter: the next tap) and meet zeros on the filter side.
#pragma once
#include <hip/hip_runtime.h>

#include "igemm.h"

namespace glowmi {

// Position of a chunk in the reduction: filter row and column, first channel.
struct Chunk {
  int r, s, c;
};

// Divided out on the host: a division by a number the compiler does not know is about forty dependent instructions.
struct ChunkWalk {
  FastDiv div_cpt;
  int cpt, chunks;                       // chunks per tap, chunks of the reduction
  int dr, ds, dc;                        // one step = (dr * S + ds) taps and dc channels
  int end_pixels, end_filters;           // the last output pixels, filters of a group, whose chunks may run past the end of a tensor
#if defined(__HIPCC__)
  __device__ __forceinline__ Chunk at(int chunk, const Problem& p) const {
    Chunk k;
    const int t = div_cpt.div(chunk);
    k.c = (chunk - t * cpt) * 16;
    k.r = p.div_s.div(t);
    k.s = t - k.r * p.s;
    return k;
  }
  __device__ __forceinline__ void step(Chunk& k, int S) const {   // one carry per digit
    k.c += dc;
    const bool wc = k.c >= cpt * 16;
    k.c -= wc ? cpt * 16 : 0;
    k.s += ds + (wc ? 1 : 0);
    const bool ws = k.s >= S;
    k.s -= ws ? S : 0;
    k.r += dr + (ws ? 1 : 0);
  }
  // reduction codes in the chunks before this one
  __device__ __forceinline__ int codes_before(int chunk, const Problem& p) const {
    if (chunk >= chunks) return p.Kgemm;
    const int t = div_cpt.div(chunk);
    return t * p.cg + (chunk - t * cpt) * 16;
  }
#endif
};

// A 16-byte load that starts in the last 15 bytes of a tensor runs past its end, and a dword of it that straddles the end is
// lost with whatever codes lie in front of it.  The output pixels with taps in those bytes: all from the first output row that
// reaches the input's last rows (of its last image, or the last images where one is smaller than that).
inline int pixels_at_end(const Problem& p) {
  const long long image = (long long)p.h * p.w_, near = (15 + (long long)p.c - 1) / p.c;   // input pixels in the last bytes
  if (near > image) {
    const long long images = (near + image - 1) / image;
    return images < p.n ? (int)(images * p.oh * p.ow) : p.M;
  }
  const int first_row = p.h - (int)((near + p.w_ - 1) / p.w_);
  const long long reach = (long long)first_row + p.pad_t - (p.r - 1);                      // oy * stride from which it is read
  const long long oy = reach <= 0 ? 0 : (reach + p.stride_h - 1) / p.stride_h;
  return oy < p.oh ? (int)(p.oh - oy) * p.ow : 0;
}
inline int filters_at_end(const Problem& p) { return (15 + p.Kgemm - 1) / p.Kgemm; }

inline ChunkWalk make_chunk_walk(const Problem& p, int step) {
  ChunkWalk w;
  w.cpt = (p.cg + 15) / 16;
  w.div_cpt = make_fastdiv((uint32_t)w.cpt);
  w.chunks = p.r * p.s * w.cpt;
  const int taps = step / w.cpt;
  w.dc = (step - taps * w.cpt) * 16;
  w.dr = taps / p.s;
  w.ds = taps - w.dr * p.s;
  w.end_pixels = pixels_at_end(p);
  w.end_filters = filters_at_end(p);
  return w;
}

#if defined(__HIPCC__)
typedef int i8x16 __attribute__((ext_vector_type(4)));   // sixteen codes

// 16 bytes shifted down by `over` bytes (0..15), zeros from above.
__device__ __forceinline__ i8x16 shift_down(i8x16 v, unsigned over) {
  const unsigned q = over >> 2, b = over & 3u;
  unsigned d[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int x = 0;
#pragma unroll
    for (int j = i; j < 4; ++j) x = (int)q == j - i ? v[j] : x;
    d[i] = (unsigned)x;
  }
  return i8x16{(int)__builtin_amdgcn_alignbyte(d[1], d[0], b), (int)__builtin_amdgcn_alignbyte(d[2], d[1], b),
               (int)__builtin_amdgcn_alignbyte(d[3], d[2], b), (int)__builtin_amdgcn_alignbyte(0u, d[3], b)};
}

// Mask of the first `valid` bytes (any integer; at least 16 keeps all) of 16.
__device__ __forceinline__ i8x16 byte_mask(int valid) {
  i8x16 m;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int n = valid - 4 * i;
    m[i] = n >= 4 ? -1 : n <= 0 ? 0 : (int)((1u << (8 * n)) - 1u);
  }
  return m;
}

// The first n (1 .. 15) of 16 codes, to any address.
__device__ __forceinline__ void store_front(signed char* dst, i8x16 v, int n) {
  int lo = v[0], hi = v[1];
  if (n & 8) {
    __builtin_memcpy(dst, &v, 8);
    dst += 8;
    lo = v[2];
    hi = v[3];
  }
  if (n & 4) {
    __builtin_memcpy(dst, &lo, 4);
    dst += 4;
    lo = hi;
  }
  if (n & 2) {
    __builtin_memcpy(dst, &lo, 2);
    dst += 2;
    lo = (int)((unsigned)lo >> 16);
  }
  if (n & 1) *dst = (signed char)lo;
}

// acc plus the signed bytes of v (ones = 0x01010101), or acc (ones = 0)
__device__ __forceinline__ int sum_bytes(i8x16 v, int ones, int acc) {
#pragma unroll
  for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_sdot4(v[i], ones, acc, false);
  return acc;
}
#endif

}  // namespace glowmi
