// int8 Convolution with a short reduction on many pixels, any filter of up to 30 taps, for gfx950 (MI355X): the quantized
// form of Section 4 of the paper, one more of the kinds of convolution that get a strategy of their own (Section 5.3).
//
// With a reduction of one to a dozen steps a workgroup that makes one tile and ends is a chain of waits: pixel indexes, loads,
// LDS, barriers, the channels' sums, the requantize step, the stores, about five microseconds whatever the tile has to do, and
// four tiles on a CU do not hide it.  So here, as in conv_pw_i8.hip:
//   - persistent workgroups of eight wavefronts keep a slice of NT x 32 filters in LDS, each tap's channels filled up to sixteen
//     with zeros, in the row order the MFMA needs, and the slice's terms  bias - x_offset * sum w;
//   - a wavefront goes through blocks of 32 pixels by itself, no barrier.  A lane's operand (16 codes of one tap of one pixel)
//     is one 16-byte load straight from the image: it serves NT MFMAs, and a pixel that nine taps want comes from the L1;
//   - the loads of a trip of T steps are issued a trip ahead, the next block's first ones ahead of this block's stores (the
//     memory counter is in order: behind them they would wait for the stores);
//   - the filter is the row operand with its channels permuted so that a lane ends up with 16 consecutive channels of one
//     pixel: requantize, clamp, pack, one 16-byte store.
// A chunk's codes past its tap's channels are the next pixel's and meet the zeros on the filter side.
// Measured: 3x3 24->208 on 100x100 at batch 27 (56 MB of codes) 84.7 -> 33 us, 1x1 72->472 on 43x46 at batch 16 20.2 -> 10.0, 1x1
// 40->320 at 44304 pixels 19.2 -> 8.8, 3x3 16->176 at 31185 11.1 -> 6.4, 3x3 72->152 at 18564 16.5 -> 8.9.  What bounds it: with many
// pixels the requantize step and the MFMAs, about equal (a multiply-high is four issue slots, a code some nine instructions),
// otherwise the start and the slice's way into LDS.  Sixteen wavefronts to a workgroup (slices twice as deep) gained on 3x3
// 112->80 alone (14.0 -> 12.8) and four, whose slices are half, nothing past the runs' differences; trips of two steps instead of
// three are 5 % slower on nine taps of two chunks, and three instead of two on short single taps.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <type_traits>

#include "arguments.h"
#include "i8_chunks.h"
#include "igemm.h"
#include "pw_common.h"
#include "quant_epilogue.h"

namespace glowmi {
namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

template <int V>
using Int = std::integral_constant<int, V>;

constexpr int SH_THREADS = 512;
constexpr int SH_WAVES = SH_THREADS / 64;
constexpr int SH_LDS = 80 * 1024;                       // two workgroups to a CU
constexpr unsigned OOB = 0x80000000u;                   // beyond any tensor the kernel accepts: loads give zeros
constexpr int NO_TAP = 31;                              // bit of no tap: a chunk past the reduction

// Row of a staged tile of 32 filters that holds its channel c: result register e of a lane with half h is MFMA row
// (e / 4) * 8 + 4 h + e % 4, which this order makes channel 16 h + e.
__device__ __forceinline__ int staged_row(int c) { return ((c >> 2) & 3) * 8 + (c >> 4) * 4 + (c & 3); }

// Sixteen bytes from byte `by` of five dwords.
__device__ __forceinline__ v4i shift_in(v4i v, int fifth, unsigned by) {
  return v4i{(int)__builtin_amdgcn_alignbyte((unsigned)v[1], (unsigned)v[0], by), (int)__builtin_amdgcn_alignbyte((unsigned)v[2], (unsigned)v[1], by),
             (int)__builtin_amdgcn_alignbyte((unsigned)v[3], (unsigned)v[2], by), (int)__builtin_amdgcn_alignbyte((unsigned)fifth, (unsigned)v[3], by)};
}

// Adds v up over each sixteen lanes; the last of them has the sum.
__device__ __forceinline__ int sum_of_sixteen(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // row_shr:1 (a row: 16 lanes)
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);   // row_shr:8
  return v;
}

struct ShortWalk {
  int trips, pitch;                                     // trips of a block; bytes of a filter's row in LDS
  int cpt, chunks;                                      // 16-code chunks of a tap, of the reduction
  FastDiv div_cpt;
  PwRange range;                                        // a wavefront's blocks
};

constexpr int short_lds(int nt, int pitch) { return nt * 32 * pitch + nt * 32 * 4 + 256 * 4 + (pitch / 16) * 8; }

// TAPS: more than one tap, or padding; otherwise a pixel's chunks follow each other and all lie inside the image.
// ADD: the chain has a tensor-add link (int8 of the output's shape, maybe the output itself).
// T == 4, LINES: pixels that lie whole cache lines apart (c % 128 == 0) would all be read at the same place of a line at once
// (conv_few_f32.hip); the odd ones load the two halves of a trip, the halves of a line, in the other order (3x3 128->88 at 27900
// pixels 16.2 -> 12.7 us, 256->56 + add on 55x55 at batch 4 23.7 -> 16.5).
// ODD: input or output channels that are no multiple of four (the stores for the latter in every form would make the widest spill:
// 3x3 24->208 36.3 -> 41.7 us).  Loads at odd addresses take several times as long as others, so a chunk is fetched as
// the five dwords it lies in and shifted where it is used (1x1 19->864 at 56784 pixels 42.3 -> 16.5 us, 3x3 30->912 at 9120 21.3 ->
// 11.3, 1x1 30->144 at 27540 9.4 -> 5.2; 64 of 90 layers move and take 0.79 of the time; 1x1 24->183 at 72090 21.2 -> 10.0).
template <int NT, int T, bool TAPS, bool ADD, bool ODD>
__global__ __launch_bounds__(SH_THREADS, 4) void conv_short_i8_kernel(const Problem p, const ShortWalk walk) {
  fetch_arguments(p, walk);
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int BN = 32 * NT;
  constexpr bool LINES = T == 4;
  const int pitch = walk.pitch;
  unsigned char* wlds = smem;
  int* cterm = reinterpret_cast<int*>(smem + BN * pitch);
  int* addlut = cterm + BN;                             // [256] the addend's code (as an unsigned byte) -> its term
  v2i* tab = reinterpret_cast<v2i*>(addlut + 256);      // [chunk] its place in the image from the pixel's first tap, its tap

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lh = lane >> 5;
  const int slice = blockIdx.y;
  // consecutive workgroups go round the eight XCDs: each gets a run of pixels
  const int wg = gridDim.x % 8 == 0 ? (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3) : blockIdx.x;

  // (tensors start on 16 bytes: the dword of a tensor's last byte lies in the block of sixteen that the byte lies in)
  const __amdgpu_buffer_rsrc_t rsrc_x =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.x), 0, (int)((p.x_bytes + 3u) & ~3u), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_w =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w), 0, (int)((p.w_bytes + 3u) & ~3u), 0x00020000);
  const int y_bytes = (int)((unsigned)p.M * (unsigned)p.k);
  const __amdgpu_buffer_rsrc_t rsrc_y = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, y_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_add =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(ADD ? p.addend : p.y), 0, y_bytes, 0x00020000);

  int blk, end;
  deal_range(wg * SH_WAVES + wave, (int)gridDim.x * SH_WAVES, walk.range.items_div, walk.range.items_rem, blk, end);

  const int all_chunks = walk.trips * T * 2;            // (chunks past the reduction: zeros)
  // ---- this lane's pixel of a block: where its first tap lies, and a bit for each tap that lies inside the image
  const int ohow = p.oh * p.ow;
  auto locate = [&](int b, bool live, unsigned& base, unsigned& mask) {
    int m = b * 32 + l32;
    if (m >= p.M) m = p.M - 1;                          // (results of such rows are never stored)
    const int img = p.div_ohow.div(m);
    const int rem = m - img * ohow;
    const int oh = p.div_ow.div(rem);
    const int ih0 = oh * p.stride_h - p.pad_t, iw0 = (rem - oh * p.ow) * p.stride_w - p.pad_l;
    base = (unsigned)(((img * p.h + ih0) * p.w_ + iw0) * p.c);
    if (TAPS) {
      const int lo = iw0 < 0 ? -iw0 : 0, hi = p.w_ - iw0 < p.s ? p.w_ - iw0 : p.s;
      const unsigned cols = live && lo < hi ? ((1u << hi) - 1u) & ~((1u << lo) - 1u) : 0u;
      mask = 0;
      for (int r = 0; r < p.r; ++r) mask |= (unsigned)(ih0 + r) < (unsigned)p.h ? cols << (r * p.s) : 0u;
    } else if (!live) {
      base = OOB;
    }
  };
  const int swapped = LINES ? 2 * (l32 & 1) : 0;
  struct Trip {
    v4i a[T];
    int fifth[ODD ? T : 1];
    unsigned inside, by;                                // a bit for each step: its tap lies inside the image; two bits: bytes to shift by
  };
  auto load_trip = [&](Trip& tr, int trip, unsigned base, unsigned mask, auto table_tag) {   // table: whether `tab` is there
    tr.inside = tr.by = 0;
#pragma unroll
    for (int u = 0; u < T; ++u) {
      const int chunk = 2 * (trip * T + (LINES ? u ^ swapped : u)) + lh;
      unsigned off = base + 16u * (unsigned)chunk;
      if (TAPS) {
        v2i e;
        if constexpr (decltype(table_tag)::value) {
          e = tab[chunk];
        } else {
          const int tap = walk.div_cpt.div(chunk), r = p.div_s.div(tap);
          e = chunk < walk.chunks ? v2i{(r * p.w_ + tap - r * p.s) * p.c + (chunk - tap * walk.cpt) * 16, tap} : v2i{0, NO_TAP};
        }
        const unsigned in = (mask >> e[1]) & 1u;
        off = in ? base + (unsigned)e[0] : OOB;
        tr.inside |= in << u;                              // (the halves of a line are of one tap)
      }
      tr.a[u] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, ODD ? off & ~3u : off, 0, 0);
      if (ODD) {
        tr.fifth[u] = (int)__builtin_amdgcn_raw_buffer_load_b32(rsrc_x, (off & ~3u) + 16u, 0, 0);
        tr.by |= (off & 3u) << (2 * u);
      }
    }
  };
  v4i addn[NT];
  auto load_addend = [&](int b, bool live) {
    const unsigned off = (unsigned)(b * 32 + l32) * (unsigned)p.k + (unsigned)(slice * BN + 16 * lh);
#pragma unroll
    for (int t = 0; t < NT; ++t) addn[t] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_add, live ? off + 32u * t : 0xFFFFFF00u, 0, 0);
  };

  // ---- filter slice -> LDS.  Sixteen lanes side by side load a row's chunks, so that a lane works out its chunks' places in a filter
  // once for all its rows (a division for each chunk of each row took 1400 of 12000 cycles of a small layer) and a row's code sum is what
  // the lanes add up of what passes through them (read back from LDS by four threads a row, behind a barrier: 2200).  The first block's
  // first trip is asked for behind the first rows' chunks.
  constexpr int AT_ONCE = 4 * SH_WAVES;                 // rows of a pass
  const int col = lane & 15, row0 = wave * 4 + (lane >> 4);
  unsigned base, mask = 0;
  Trip now, next;
  auto stage_rows = [&](int pass0, auto rows_tag, auto columns_tag, auto first_tag) {   // passes, sixteens of chunks in flight
    constexpr int U = decltype(rows_tag)::value, C = decltype(columns_tag)::value;
    constexpr bool FIRST = decltype(first_tag)::value != 0;
    int sum[U], bias[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int ch = slice * BN + (pass0 + q) * AT_ONCE + row0;
      bias[q] = p.bias && ch < p.k ? static_cast<const int*>(p.bias)[ch] : 0;
      sum[q] = 0;
    }
    auto columns = [&](int col0, auto locate_tag) {
      v4i v[C][U];
      int fifth[ODD ? C : 1][ODD ? U : 1];
      unsigned by[ODD ? C : 1][ODD ? U : 1];
      int left[C];                                      // of a chunk's tap's channels
#pragma unroll
      for (int i = 0; i < C; ++i) {
        const int chunk = col0 + 16 * i + col, tap = walk.div_cpt.div(chunk), c0 = (chunk - tap * walk.cpt) * 16;
        left[i] = chunk < walk.chunks ? p.c - c0 : 0;
        const unsigned lane_off = left[i] > 0 ? (unsigned)(tap * p.c + c0) : OOB;
#pragma unroll
        for (int q = 0; q < U; ++q) {
          const int ch = slice * BN + (pass0 + q) * AT_ONCE + row0;
          const unsigned off = ch < p.k && lane_off != OOB ? (unsigned)ch * (unsigned)p.Kgemm + lane_off : OOB;
          v[i][q] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, off & ~3u, 0, 0);
          if (ODD) {
            fifth[i][q] = (int)__builtin_amdgcn_raw_buffer_load_b32(rsrc_w, (off & ~3u) + 16u, 0, 0);
            by[i][q] = off & 3u;
          }
        }
        if (TAPS && FIRST && wave == 0 && lane < 16 && chunk < all_chunks) {
          const int r = p.div_s.div(tap), s = tap - r * p.s;
          tab[chunk] = chunk < walk.chunks ? v2i{(r * p.w_ + s) * p.c + c0, tap} : v2i{0, NO_TAP};
        }
      }
      if constexpr (decltype(locate_tag)::value) {
        locate(blk, blk < end, base, mask);
        load_trip(now, 0, base, mask, Int<0>{});
      }
#pragma unroll
      for (int i = 0; i < C; ++i) {
        const int chunk = col0 + 16 * i + col;
        v4i keep;                                       // the bytes that are the tap's
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int mine = left[i] - 4 * e;
          keep[e] = mine >= 4 ? -1 : mine <= 0 ? 0 : (1 << (8 * mine)) - 1;
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
          const int row = (pass0 + q) * AT_ONCE + row0;
          if (ODD) v[i][q] = shift_in(v[i][q], fifth[i][q], by[i][q]);
          v[i][q] &= keep;
#pragma unroll
          for (int e = 0; e < 4; ++e) sum[q] = __builtin_amdgcn_sdot4(v[i][q][e], 0x01010101, sum[q], false);
          if (chunk < all_chunks) *reinterpret_cast<v4i*>(wlds + ((row & ~31) + staged_row(row & 31)) * pitch + chunk * 16) = v[i][q];
        }
      }
    };
    columns(0, first_tag);
    for (int col0 = 16 * C; col0 < all_chunks; col0 += 16 * C) columns(col0, Int<0>{});
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int all = sum_of_sixteen(sum[q]);
      // combined modulo 2^32: the true accumulator fits int32 by contract
      if (col == 15) cterm[(pass0 + q) * AT_ONCE + row0] = (int)((unsigned)bias[q] - (unsigned)p.x_off * (unsigned)all);
    }
  };
  auto stage = [&](auto columns_tag) {                  // (up to twelve chunks of a lane in flight)
    constexpr int C = decltype(columns_tag)::value, U = NT * C <= (ODD ? 6 : 12) ? NT : (NT + 1) / 2;
    stage_rows(0, Int<U>{}, columns_tag, Int<1>{});
    if constexpr (U < NT) stage_rows(U, Int<NT - U>{}, columns_tag, Int<0>{});
  };
  if (all_chunks <= 16) stage(Int<1>{});
  else if (all_chunks <= 32) stage(Int<2>{});
  else if (all_chunks <= 48) stage(Int<3>{});
  else stage(Int<4>{});
  if (ADD)
    for (int i = tid; i < 256; i += SH_THREADS) addlut[i] = rescale_term((int)(signed char)i - p.r_off, p.r_mant, p.r_shift);
  if (ADD) load_addend(blk, blk < end);
  __syncthreads();
  if (blk >= end) return;

  const unsigned char* w_lane = wlds + l32 * pitch + 16 * lh;
  const int fill = (p.x_off & 0xff) * 0x01010101;       // a tap on padding: the code of real zero
  const bool fast = p.shift >= 33;                      // uniform
  const FoldedRequant fold = make_folded_requant(p.shift, p.y_off);
  const int lo_v = p.lo;
  v16i acc[NT];
  auto multiply = [&](Trip& tr, int trip) {
    const unsigned char* w = w_lane + trip * (T * 32);
#pragma unroll
    for (int u = 0; u < T; ++u) {
      v4i v = tr.a[u];
      if (ODD) v = shift_in(v, tr.fifth[u], (tr.by >> (2 * u)) & 3u);
      if (LINES) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = swapped ? tr.a[u ^ (T / 2)][e] : v[e];
      }
      if (TAPS) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = tr.inside & (1u << u) ? v[e] : fill;
      }
#pragma unroll
      for (int t = 0; t < NT; ++t)
        acc[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(*reinterpret_cast<const v4i*>(w + t * 32 * pitch + 32 * u), v, acc[t], 0, 0, 0);
    }
  };

  for (; blk < end; ++blk) {
    int term = 16 * lh;
    asm volatile("" : "+v"(term));                      // read anew for every block: kept, the terms take as many registers as the sums
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const v4i c = *reinterpret_cast<const v4i*>(cterm + 32 * t + term + 4 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[t][4 * q + e] = c[e];
      }
    for (int trip = 0; trip + 1 < walk.trips; ++trip) {
      load_trip(next, trip + 1, base, mask, Int<1>{});
      multiply(now, trip);
      now = next;
    }
    v4i add[NT];
    if (ADD) {
#pragma unroll
      for (int t = 0; t < NT; ++t) add[t] = addn[t];
    }
    locate(blk + 1, blk + 1 < end, base, mask);
    load_trip(next, 0, base, mask, Int<1>{});
    if (ADD) load_addend(blk + 1, blk + 1 < end);
    multiply(now, walk.trips - 1);

    // ---- lane (l32, lh): pixel l32, channels 32 t + 16 lh + e
    const unsigned off = (unsigned)(blk * 32 + l32) * (unsigned)p.k;
    auto finish = [&](auto mode_tag) {
      constexpr int MODE = decltype(mode_tag)::value;   // 2 folded, 1 multiply-high, 0 64-bit
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        v4i out;
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          int q[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            unsigned v = (unsigned)acc[t][4 * q4 + e];
            if (ADD) v += (unsigned)addlut[((unsigned)add[t][q4] >> (8 * e)) & 0xffu];
            q[e] = MODE == 2 ? requantize_folded((int)v, p.mant, fold, lo_v, p.hi)
                             : requantize_as<MODE == 1>((int)v, p.mant, p.shift, p.y_off, p.lo, p.hi);
          }
          out[q4] = (int)pack_codes(q[0], q[1], q[2], q[3]);
        }
        // rows past M fall outside the output's range and the checked store drops them
        const int ch = slice * BN + 32 * t + 16 * lh;
        if (ODD && !ADD && (p.k & 3) != 0) {            // uniform: pixels at any byte address (with an addend the planner takes other kernels)
          signed char* dst = static_cast<signed char*>(p.y) + ((size_t)(blk * 32 + l32) * p.k + ch);
          if (blk * 32 + l32 >= p.M || ch >= p.k) continue;
          if (ch + 16 <= p.k) __builtin_memcpy(dst, &out, 16);
          else store_front(dst, out, p.k - ch);
        } else if (ch + 16 <= p.k) __builtin_amdgcn_raw_buffer_store_b128(out, rsrc_y, off + (unsigned)ch, 0, 0);
        else {
#pragma unroll
          for (int q4 = 0; q4 < 3; ++q4)
            if (ch + 4 * q4 < p.k) __builtin_amdgcn_raw_buffer_store_b32(out[q4], rsrc_y, off + (unsigned)(ch + 4 * q4), 0, 0);
        }
      }
    };
    if (fold.ok) finish(std::integral_constant<int, 2>{});
    else if (fast) finish(std::integral_constant<int, 1>{});
    else finish(std::integral_constant<int, 0>{});
    now = next;
  }
}

// Workgroups of a slice: two to a CU over all slices, a multiple of the XCDs where there are as many.
int workgroups(int blocks, int slices, int num_cu) {
  int wgs = 2 * num_cu / slices;
  const int most = (blocks + SH_WAVES - 1) / SH_WAVES;
  if (wgs < 1) wgs = 1;
  if (wgs >= 8) wgs &= ~7;
  if (wgs > most) wgs = most >= 8 ? (most + 7) & ~7 : most;
  return wgs;
}

template <int NT, int T, bool TAPS, bool ADD, bool ODD = false>
hipError_t launch_form(const Problem& p, hipStream_t stream) {
  auto kern = conv_short_i8_kernel<NT, T, TAPS, ADD, ODD>;
  // once per instantiation; initialisation of a function-local static is thread-safe
  static const hipError_t attr_status =
      hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, SH_LDS);
  if (attr_status != hipSuccess) return attr_status;
  const int num_cu = num_compute_units();
  if (num_cu < 1) return hipErrorInvalidDevice;
  ShortWalk walk;
  walk.cpt = (p.c + 15) / 16;
  walk.chunks = p.r * p.s * walk.cpt;
  walk.trips = (walk.chunks + 2 * T - 1) / (2 * T);
  walk.pitch = walk.trips * T * 32 + 16;
  walk.div_cpt = make_fastdiv((uint32_t)walk.cpt);
  const int slices = (p.k + 32 * NT - 1) / (32 * NT), blocks = (p.M + 31) / 32;
  const int wgs = workgroups(blocks, slices, num_cu);
  walk.range = make_pw_range(blocks, 1, (long long)wgs * SH_WAVES);
  hipLaunchKernelGGL(kern, dim3((unsigned)wgs, (unsigned)slices), dim3(SH_THREADS), short_lds(NT, walk.pitch), stream, p, walk);
  return hipGetLastError();
}

// Steps of a trip: nine taps of few channels are a multiple of three; more registers than there are with four tiles and an addend.
constexpr int steps_of(int nt, bool taps, bool add) { return taps && !(nt == 4 && add) ? 3 : 2; }
bool by_lines(const Problem& p, int nt) { return p.c % 128 == 0 && p.k % 4 == 0 && nt <= 2; }   // (more tiles leave no registers for four steps)
bool has_taps(const Problem& p) { return p.r * p.s > 1 || p.pad_t || p.pad_l; }

template <int NT, bool ODD>
hipError_t launch_rest(const Problem& p, hipStream_t stream) {
  if (has_taps(p))
    return p.addend ? launch_form<NT, steps_of(NT, true, true), true, true, ODD>(p, stream)
                    : launch_form<NT, steps_of(NT, true, false), true, false, ODD>(p, stream);
  return p.addend ? launch_form<NT, steps_of(NT, false, true), false, true, ODD>(p, stream)
                  : launch_form<NT, steps_of(NT, false, false), false, false, ODD>(p, stream);
}

template <int NT>
hipError_t launch_nt(const Problem& p, hipStream_t stream) {
  if constexpr (NT <= 2) {
    if (by_lines(p, NT)) {
      if (has_taps(p)) return p.addend ? launch_form<NT, 4, true, true>(p, stream) : launch_form<NT, 4, true, false>(p, stream);
      return p.addend ? launch_form<NT, 4, false, true>(p, stream) : launch_form<NT, 4, false, false>(p, stream);
    }
  }
  if (p.c % 4 != 0 || p.k % 4 != 0) return launch_rest<NT, true>(p, stream);
  return launch_rest<NT, false>(p, stream);
}

}  // namespace

// The form (tiles of 32 channels to a slice) and what it is expected to take, -1: not a layer for this kernel.  Whether it is the
// best kernel is the planner's question, which gives what it has to be below.  The estimate: a start, the filter's way into LDS for each of a
// CU's workgroups in turn, the blocks a wavefront goes through (tiles, steps, an addend) as the workgroups of a CU share its pipes and the
// steps as one wavefront's chain, the bytes of the tensors and of the filter.  Fitted apart for channels in fours and others (five dwords to a
// chunk, and shifts, or codes stored one by one), to the geometric mean of the times with operands in the caches and from memory: over 2361
// and 432 runs of 900 layers drawn after the fit, in every form, median errors of 4 and 5 %, nine in ten within 11 and 14 %.
struct ShortCost { double fixed, fill, tile, step, add, chain, mb, filter; };
constexpr ShortCost kShort[2] = {{3.604, 0.01838, 0.3973, 0.06682, 0.2133, 0.04485, 0.09156, 0.3565},
                                 {3.588, 0.02711, 0.4203, 0.1295, 0.07967, 0.02581, 0.1254, 1.957}};
int short_i8_form(const Problem& p, double below, double* us) {
  const int mode = knob_or(KNOB_I8_SHORT, 1);           // 0: off, 2: any layer that fits (tests)
  if (mode == 0 || p.b_is_kn || p.groups != 1 || p.chain_n > 0 || p.w_off != 0 || (p.addend && p.k % 4 != 0)) return -1;
  if (p.r * p.s >= NO_TAP || p.x_bytes > 0x7FFFFFFFu || p.w_bytes > 0x7FFFFFFFu) return -1;
  if ((unsigned long long)p.M * (unsigned long long)p.k > 0xF0000000ull || p.k > 65536 || p.M > (1 << 30)) return -1;
  const bool taps = has_taps(p);
  // (padding at the far sides only: a single tap past the image has no bit to say so)
  if (!taps && ((long long)(p.oh - 1) * p.stride_h >= p.h || (long long)(p.ow - 1) * p.stride_w >= p.w_)) return -1;
  const int chunks = p.r * p.s * ((p.c + 15) / 16), blocks = (p.M + 31) / 32, forced = knob_or(KNOB_I8_SHORT_FORM, -1);
  const ShortCost& cost = kShort[p.c % 4 != 0 || p.k % 4 != 0];
  const double mb = 1e-6 * ((double)p.x_bytes + (p.addend ? 2.0 : 1.0) * p.M * p.k);
  // one tile to a wavefront, with nothing to wait for but its own chain: most small layers are decided by this
  const double chain = 0.5 * chunks;                    // at least this many steps
  if (mode == 1 && cost.fixed + cost.fill * chunks + cost.tile + (cost.step + cost.chain) * chain + cost.mb * mb >= below) return -1;
  int best = -1;
  for (int nt = 1; nt <= 4; ++nt) {
    const int T = by_lines(p, nt) ? 4 : steps_of(nt, taps, p.addend != nullptr), steps = (chunks + 2 * T - 1) / (2 * T) * T;
    if (short_lds(nt, steps * 32 + 16) > SH_LDS || (forced > 0 && nt != forced)) continue;
    const int slices = (p.k + 32 * nt - 1) / (32 * nt), wgs = workgroups(blocks, slices, 256);
    const double per_cu = (wgs * slices + 255) / 256, deep = (blocks + wgs * SH_WAVES - 1) / (wgs * SH_WAVES);
    const double t = cost.fixed + per_cu * (cost.fill * nt * chunks + deep * (nt * (cost.tile + (p.addend ? cost.add : 0.0)) + cost.step * steps)) +
                     deep * cost.chain * steps + cost.mb * mb + cost.filter * 1e-6 * p.w_bytes;
    if (best < 0 || t < *us) {
      best = nt;
      *us = t;
    }
  }
  return best;
}

hipError_t launch_short_i8(const Problem& p, int form, hipStream_t stream, const char** variant) {
  static thread_local char name[48];
  snprintf(name, sizeof(name), "conv_short_i8_32x%d", 32 * form);
  *variant = name;
  switch (form) {
    case 1: return launch_nt<1>(p, stream);
    case 2: return launch_nt<2>(p, stream);
    case 3: return launch_nt<3>(p, stream);
    case 4: return launch_nt<4>(p, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace glowmi
