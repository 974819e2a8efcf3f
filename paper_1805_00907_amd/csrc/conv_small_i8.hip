// int8 Convolution on few output pixels with a reduction of up to a few thousand codes (the late layers of a network at
// small batch): the quantized contraction of Section 4 of the paper, offsets taken out afterwards, requantize and Relu on
// the accumulators (Section 4.3, operator stacking of Section 5.2).
//
// Such a layer is latency.  Tiled over the output it has fewer tiles than the chip has CUs, and each walks the reduction
// slab by slab, half a microsecond of staging instructions per slab (3x3 168->104 stride 2 on 35x35: 12 tiles, 12 us); a
// split reduction pays a second kernel.  Here it is ONE launch with one memory round trip:
//   - a workgroup owns 32 pixels x 32 channels; its eight wavefronts split the reduction in steps of two 16-code chunks
//     (i8_chunks.h) and every wavefront issues all loads of its steps before touching any;
//   - no LDS staging: a lane loads a chunk of its pixel's input and of its channel's filter straight into the operand
//     layout of v_mfma_i32_32x32x32_i8 (lanes 0..31 the even chunk of a step, 32..63 the odd one);
//   - a tap outside the image is the code of real zero (selected after the load), a chunk past the reduction has a
//     zero filter, the bytes of a short chunk past its tap are masked on the filter side;
//   - the eight partial tiles are summed through LDS, four channels of a pixel per thread, then the offsets, bias, addend,
//     requantize, one dword of codes per thread.
// A CU pulls 64 bytes of operands per reduction code of its tile from the caches at some 45 B/ns, so a tile's reduction is
// bounded (2560 codes); deeper ones are sliced over the grid when that gives enough workgroups (a finishing kernel
// sums them), or stay on the tiled kernels.
#include <hip/hip_runtime.h>

#include "arguments.h"
#include "i8_chunks.h"
#include "igemm.h"
#include "quant_epilogue.h"

namespace glowmi {
namespace {

typedef i8x16 v4i;
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int CQ_WAVES = 8;
constexpr int CQ_THREADS = 64 * CQ_WAVES;
constexpr int CQ_MAX_STEPS = 10;                 // per wavefront: eight registers each
constexpr int CQ_PITCH = 36;                     // ints per pixel of a partial tile (32 channels): rows start on other banks
constexpr unsigned OOB = 0x80000000u;            // tensors are below 2 GiB: past the end, the load returns zeros

struct Grid {
  FastDiv div_tiles_n, div_tiles_m, div_groups;
  int tiles_n, tiles_m, total;                   // channel tiles per group, pixel tiles, all workgroups
  int steps_per_split;                           // of two chunks
  ChunkWalk chunk;                               // one step of the walk: 2 chunks
};

template <int STEPS>
__global__ __launch_bounds__(CQ_THREADS, STEPS <= 4 ? 4 : 2) void conv_small_i8_kernel(const Problem p, const Grid gr) {
  fetch_arguments(p, gr);
  __shared__ __align__(16) int part[CQ_WAVES * 32 * CQ_PITCH];
  __shared__ int sums[64];                       // filter code sums per channel, input code sums per pixel
  int* wsum = sums;
  int* xsum = sums + 32;

  // consecutive workgroups go round-robin to the eight XCDs: each XCD takes a contiguous run of tiles, channel tiles
  // innermost, and finds the pixels they share in its own L2
  const int per_xcd = gridDim.x >> 3;
  const int wk = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (wk >= gr.total) return;
  int t = gr.div_tiles_n.div(wk);
  const int tn = wk - t * gr.tiles_n;
  int t2 = gr.div_tiles_m.div(t);
  const int tm = t - t2 * gr.tiles_m;
  const int split = gr.div_groups.div(t2);
  const int g = t2 - split * p.groups;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lh = lane >> 5;
  const int m = tm * 32 + l32;                   // this lane's pixel (column operand)
  const int n = tn * 32 + l32;                   // this lane's channel of the group (row operand)
  if (tid < 64) sums[tid] = 0;

  // a 16-byte load at the end of a tensor of any size stays inside the 16-byte block of its last byte
  const unsigned x_size = p.x_bytes < 16u ? 16u : p.x_bytes, w_size = p.w_bytes < 16u ? 16u : p.w_bytes;
  const __amdgpu_buffer_rsrc_t rsrc_x =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.x), 0, (int)x_size, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_w =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w), 0, (int)w_size, 0x00020000);

  int ih0 = -(1 << 24), iw0 = 0;                 // a row past M has no tap inside
  int pix_base = 0;
  if (m < p.M) {
    const int img = p.div_ohow.div(m);
    const int rem = m - img * (p.oh * p.ow);
    const int oh = p.div_ow.div(rem);
    const int ow = rem - oh * p.ow;
    ih0 = oh * p.stride_h - p.pad_t;
    iw0 = ow * p.stride_w - p.pad_l;
    pix_base = ((img * p.h + ih0) * p.w_ + iw0) * p.c + g * p.cg;
  }
  const unsigned w_base = n < p.kg ? (unsigned)(g * p.kg + n) * (unsigned)p.Kgemm : OOB;

  const int first = split * gr.steps_per_split;  // steps of this slice
  const int end_chunk = (first + gr.steps_per_split) * 2 < gr.chunk.chunks ? (first + gr.steps_per_split) * 2 : gr.chunk.chunks;
  int chunk = (first + wave * STEPS) * 2 + lh;
  Chunk at = gr.chunk.at(chunk, p);

  const bool ragged = p.cg % 16 != 0;
  // chunks that would run past the end of a tensor are fetched from its last 16 bytes and shifted (only tiles that see them)
  const bool at_end = ragged && (tm * 32 + 32 > p.M - gr.chunk.end_pixels || tn * 32 + 32 > p.kg - gr.chunk.end_filters);

  v4i a[STEPS], b[STEPS];
  unsigned inside = 0, brief = 0;
  unsigned long long over_a = 0, over_b = 0;     // four bits per load
#pragma unroll
  for (int i = 0; i < STEPS; ++i) {
    const bool kok = chunk < end_chunk;
    const int ih = ih0 + at.r, iw = iw0 + at.s;
    const bool in = kok && (unsigned)ih < (unsigned)p.h && (unsigned)iw < (unsigned)p.w_;
    unsigned xo = in ? (unsigned)(pix_base + (at.r * p.w_ + at.s) * p.c + at.c) : OOB;
    unsigned wo = kok && w_base != OOB ? w_base + (unsigned)((at.r * p.s + at.s) * p.cg + at.c) : OOB;
    inside |= (in ? 1u : 0u) << i;
    brief |= ((at.c + 16 > p.cg ? 1u : 0u) | (kok ? 0u : 0x10000u)) << i;
    if (at_end) {
      const unsigned oa = xo != OOB && xo > x_size - 16u ? xo - (x_size - 16u) : 0u;
      const unsigned ob = wo != OOB && wo > w_size - 16u ? wo - (w_size - 16u) : 0u;
      xo -= oa;
      wo -= ob;
      over_a |= (unsigned long long)oa << (4 * i);
      over_b |= (unsigned long long)ob << (4 * i);
    }
    a[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, xo, 0, 0);
    b[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, wo, 0, 0);
    chunk += 2;
    gr.chunk.step(at, p.s);
  }
  __syncthreads();                               // the code sums are zeroed (the loads stay in flight)

  const int xo_fill = (p.x_off & 0xff) * 0x01010101;
  const v4i short_mask = byte_mask(p.cg % 16);
  const bool need_xsum = p.w_off != 0;
  v16i acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0;
  int wacc = 0, xacc = 0;
#pragma unroll
  for (int i = 0; i < STEPS; ++i) {
    v4i va = a[i], vb = b[i];
    if (at_end) {
      va = shift_down(va, (unsigned)(over_a >> (4 * i)) & 15u);
      vb = shift_down(vb, (unsigned)(over_b >> (4 * i)) & 15u);
    }
    const bool in = inside & (1u << i);
    const bool cut = brief & (1u << i);
#pragma unroll
    for (int e = 0; e < 4; ++e) va[e] = in ? va[e] : xo_fill;
    if (ragged) {
#pragma unroll
      for (int e = 0; e < 4; ++e) vb[e] = cut ? vb[e] & short_mask[e] : vb[e];
    }
    if (need_xsum) {                             // the sum of a pixel's codes counts real chunks only
      v4i vx;
      const bool past = brief & (0x10000u << i);
#pragma unroll
      for (int e = 0; e < 4; ++e) vx[e] = past ? 0 : (ragged && cut) ? va[e] & short_mask[e] : va[e];
      xacc = sum_bytes(vx, 0x01010101, xacc);
    }
    wacc = sum_bytes(vb, 0x01010101, wacc);
    // filter fragment as the row operand: result rows = channels, columns = pixels
    acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(vb, va, acc, 0, 0, 0);
  }

  // ---- partial tiles [wavefront][pixel][channel] and code sums -> LDS.  Register e of lane (l32, lh) is channel
  // (e/4)*8 + 4*lh + e%4 of pixel l32.
  atomicAdd(&wsum[l32], wacc);
  if (need_xsum) atomicAdd(&xsum[l32], xacc);
#pragma unroll
  for (int q = 0; q < 4; ++q)
    *reinterpret_cast<v4i*>(part + (wave * 32 + l32) * CQ_PITCH + q * 8 + 4 * lh) =
        v4i{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
  __syncthreads();
  if (tid >= 256) return;

  // ---- four channels of one pixel per thread
  const int px = tid >> 3, c0 = (tid & 7) * 4;
  const int row = tm * 32 + px, col = tn * 32 + c0;
  if (row >= p.M || col >= p.kg) return;
  v4i v = {0, 0, 0, 0};
#pragma unroll
  for (int w = 0; w < CQ_WAVES; ++w) v += *reinterpret_cast<const v4i*>(part + (w * 32 + px) * CQ_PITCH + c0);
  // sum (x - xo)(w - wo) = sum x*w - xo * sum w - wo * sum x + count * xo * wo, all modulo 2^32 (the true value fits)
  const int count = gr.chunk.codes_before(end_chunk, p) - gr.chunk.codes_before(first * 2, p);
  const unsigned rowterm = (unsigned)count * (unsigned)(p.x_off * p.w_off) - (need_xsum ? (unsigned)p.w_off * (unsigned)xsum[px] : 0u);
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = (int)((unsigned)v[e] + rowterm - (unsigned)p.x_off * (unsigned)wsum[c0 + e]);
  const size_t o = (size_t)row * p.k + g * p.kg + col;
  const bool whole = ((p.kg | p.k) & 3) == 0;    // uniform: four channels are all there or none is
  if (p.split_k > 1) {
    int* __restrict__ dst = static_cast<int*>(p.partial) + (size_t)split * p.M * p.k + o;
    if (whole) {
      *reinterpret_cast<v4i*>(dst) = v;
    } else {
      for (int e = 0; e < 4 && col + e < p.kg; ++e) dst[e] = v[e];
    }
    return;
  }
  const int* __restrict__ bias = static_cast<const int*>(p.bias);
  const signed char* addend = static_cast<const signed char*>(p.addend);   // may be the output itself
  int q[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const bool live = col + e < p.kg;
    unsigned x = (unsigned)v[e];
    if (bias && live) x += (unsigned)bias[g * p.kg + col + e];
    if (addend && live) x += (unsigned)rescale_term((int)addend[o + e] - p.r_off, p.r_mant, p.r_shift);
    q[e] = p.shift >= 33 ? requantize_as<true>((int)x, p.mant, p.shift, p.y_off, p.lo, p.hi)
                         : requantize_as<false>((int)x, p.mant, p.shift, p.y_off, p.lo, p.hi);   // uniform
  }
  signed char* Y = static_cast<signed char*>(p.y) + o;
  if (whole) {
    *reinterpret_cast<unsigned*>(Y) = pack_codes(q[0], q[1], q[2], q[3]);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (col + e < p.kg) Y[e] = (signed char)q[e];
  }
}

template <int STEPS>
hipError_t launch_cq(const Problem& p, hipStream_t stream, const Grid& gr) {
  hipLaunchKernelGGL(conv_small_i8_kernel<STEPS>, dim3((unsigned)((gr.total + 7) / 8 * 8)), dim3(CQ_THREADS), 0, stream, p, gr);
  return hipGetLastError();
}

long long cq_tiles(const Problem& p) { return (long long)((p.M + 31) / 32) * ((p.kg + 31) / 32) * p.groups; }
int cq_steps(const Problem& p) { return (p.r * p.s * ((p.cg + 15) / 16) + 1) / 2; }

bool cq_shape(const Problem& p) {
  return !p.b_is_kn && p.chain_n == 0 && p.x_bytes <= 0x7FFFFFFFu && p.w_bytes <= 0x7FFFFFFFu && cq_tiles(p) < (1LL << 24);
}

}  // namespace

bool conv_small_i8_applicable(const Problem& p) {
  if (!cq_shape(p) || cq_steps(p) > CQ_WAVES * CQ_MAX_STEPS) return false;
  // Up to three tiles per CU (3x3 72->64 stride 2 on 65x96 at batch 4, 396 tiles: 7.9 -> 7.2 us; 3x3 56->512 on 23x16, 368:
  // 7.7 -> 6.8; 3x3 72->120 on 33x45 at batch 5, 932: 8.2 -> 10.6); a reduction of one slab of the tiled kernel is no
  // chain there (1x1 72->232 on 17x17, 728 tiles: 5.3 -> 5.7 us; 1x1 80->552 on 5x6, 306: 5.0 -> 4.6).
  // And up to 48 MB of operands through the caches in all (3x3 256->256 on 14x14: batch 4, 29 MB, 10.4 -> 8.7 us; batch 8,
  // 58 MB, 12.6 -> 12.9).
  if (cq_tiles(p) * cq_steps(p) > (48LL << 20) / 2048) return false;
  return cq_tiles(p) <= knob_or(KNOB_I8_SMALL_MAX_TILES, cq_steps(p) <= 4 ? 384 : 768);
}

// The reduction sliced over the grid: number of slices, 0 if the layer is not of that kind.
int conv_small_i8_splits(const Problem& p) {
  if (!cq_shape(p)) return 0;
  const int steps = cq_steps(p), per_split = CQ_WAVES * 4;
  const int splits = (steps + per_split - 1) / per_split;
  const long long tiles = cq_tiles(p);
  // (3x3 512->512 on 7x7: batch 1, 32 tiles, 10.2 -> 7.2 us; batch 4, 112 tiles, 11.0 -> 11.6)
  if (splits < 2 || splits > 64 || tiles > 64 || tiles * splits > knob_or(KNOB_I8_SMALL_MAX_TILES, 768)) return 0;
  return splits;
}

hipError_t launch_conv_small_i8(const Problem& p, hipStream_t stream, const char** variant) {
  Grid gr;
  gr.tiles_m = (p.M + 31) / 32;
  gr.tiles_n = (p.kg + 31) / 32;
  gr.div_tiles_n = make_fastdiv((uint32_t)gr.tiles_n);
  gr.div_tiles_m = make_fastdiv((uint32_t)gr.tiles_m);
  gr.div_groups = make_fastdiv((uint32_t)p.groups);
  gr.chunk = make_chunk_walk(p, 2);
  const int steps = cq_steps(p);
  gr.steps_per_split = p.split_k > 1 ? CQ_WAVES * 4 : steps;
  gr.total = (int)(cq_tiles(p) * p.split_k);
  *variant = p.split_k > 1 ? "conv_small_i8_splitk" : "conv_small_i8";
  const int per_wave = (gr.steps_per_split + CQ_WAVES - 1) / CQ_WAVES;
  switch (per_wave) {
    case 1: return launch_cq<1>(p, stream, gr);
    case 2: return launch_cq<2>(p, stream, gr);
    case 3: case 4: return launch_cq<4>(p, stream, gr);
    case 5: case 6: return launch_cq<6>(p, stream, gr);
    case 7: case 8: return launch_cq<8>(p, stream, gr);
    default: return launch_cq<CQ_MAX_STEPS>(p, stream, gr);
  }
}

}  // namespace glowmi
