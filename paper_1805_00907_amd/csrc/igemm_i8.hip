// int8 implicit-GEMM Convolution / FullyConnected for gfx950 (MI355X), the quantized form of
// Section 4 of the paper: int8 codes with per-tensor scale/offset (Section 4.1), int32 accumulation,
// and the rescale to the output range folded into the producing operation (Section 4.3), with Relu
// as a plain integer max against the output offset (same-scale max, Section 4.3).
//
// The matrix cores multiply raw codes (v_mfma_i32_32x32x32_i8).  Offsets are taken out afterwards:
//   sum (x - xo)(w - wo) = sum x*w - xo * sum_k w - wo * sum_k x + Kcount * xo * wo
// where padded taps are staged as the code xo (real value 0), so they cancel exactly.  The row sums
// are collected with dot-product instructions while the tiles are staged.  Everything after the
// accumulator is integer arithmetic, so results are reproducible bit for bit.
//
// Tiling: BM x BN output tile per workgroup of 4 or 8 wavefronts, reduction slabs of 128 codes staged in
// double-buffered LDS as K-contiguous rows of 128 + 16 pad bytes (conflict-free ds_read_b128), XCD-aware
// workgroup order.  The MFMA is issued with the filter fragment as its row operand, so a lane ends up with
// four consecutive output channels of one pixel: they are requantized, packed into one dword, transposed
// through LDS and leave the chip as 16-byte stores along the channel axis.
//
// The reduction is walked in 16-code chunks (i8_chunks.h), so any channel count is fetched 16 bytes at a time; the filter
// side is masked while it is staged.  The form before this one packed taps densely and gathered channel counts that are not a multiple of 16 byte by byte
// (16 loads and as many tap steps per chunk): 3x3 72->120 on 33x45 at batch 5 took 31.6 us.
// Two slabs are in flight in registers while a third is multiplied: with six to ten slabs per tile, which is
// what most of these layers have, a load's latency per slab was most of the kernel.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>

#include "arguments.h"
#include "i8_chunks.h"
#include "igemm.h"
#include "quant_epilogue.h"

namespace glowmi {
namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef i8x16 v4i;
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int BKQ = 128;                 // codes per reduction slab
constexpr int LDQ = BKQ + 16;            // LDS row pitch in bytes (36 dwords: conflict-free b128 reads)
constexpr int KV = BKQ / 16;             // 16-byte chunks per K-contiguous row
constexpr int INVALID_ROW = -(1 << 24);

constexpr unsigned OOB = 0x80000000u;    // beyond any int8 tensor the library accepts: loads give zeros

// How the launch walks tiles and chunks.
struct Walk {
  FastDiv div_tiles_n, div_tiles_m, div_groups;
  int tiles_n, tiles_m, total_work;
  int padded;                            // some row of some tile has taps outside the image, or lies past M
  ChunkWalk chunk;                       // one step: a slab of every wavefront group
};

__device__ __forceinline__ int requantize(int acc, int mant, int shift, int y_off, int lo, int hi) {
  return shift >= 33 ? requantize_as<true>(acc, mant, shift, y_off, lo, hi)
                     : requantize_as<false>(acc, mant, shift, y_off, lo, hi);   // uniform branch
}

// The ops of a general chain on one int32 accumulator value (quantized form: a scalar multiply only
// changed the scale on the host, bounds are integers on the accumulator's grid, an added tensor's code
// difference is rescaled to the accumulator's current scale).  `off` indexes [M][k] tensors.
__device__ __forceinline__ int apply_chain_i8(const Problem& p, int v, size_t off) {
  for (int o = 0; o < p.chain_n; ++o) {
    const ChainOpDev& op = p.chain[o];
    if (op.kind == CHAIN_ADD_TENSOR)
      v += rescale_term((int)static_cast<const signed char*>(op.tensor)[off] - op.t_off, op.t_mant, op.t_shift);
    else if (op.kind == CHAIN_MAX_SCALAR) v = v < op.ia ? op.ia : v;
    else if (op.kind == CHAIN_CLIP) { v = v < op.ia ? op.ia : v; v = v > op.ib ? op.ib : v; }
  }
  return v;
}

// KGRP groups of WAVES_M x WAVES_N wavefronts share a tile: group i multiplies slabs i, i + KGRP, ... in LDS buffers of
// its own and the partial tiles are summed through LDS at the end, every group finishing its share of the outputs.
// A grid that leaves a wavefront or two per SIMD spends a slab's time on the latency of its ~150 instructions, not
// on issuing them, so the chain of slabs is what has to get shorter (3x3 72->120 on 33x45 at batch 5, 232 tiles of
// six slabs: 10.6 us with one group).
template <int BM, int BN, int WAVES_M, int WAVES_N, int KGRP, bool B_KN, bool CHAINV = false>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N * KGRP, BM * BN / (WAVES_M * WAVES_N) <= (B_KN ? 1024 : 2048) ? 4 : 2) void igemm_i8_kernel(const Problem p, const Walk walk) {
  fetch_arguments(p, walk);
  constexpr int NTHREADS = 64 * WAVES_M * WAVES_N;      // of one group
  constexpr int ALL_THREADS = NTHREADS * KGRP;
  constexpr int ROWS_PER_PASS = NTHREADS / KV;
  constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  static_assert(TM >= 1 && TN >= 1 && WTM % 32 == 0 && WTN % 32 == 0, "tile shape");
  static_assert(BM % ROWS_PER_PASS == 0 && BN % ROWS_PER_PASS == 0, "tile rows per pass");
  constexpr int A_PASSES = BM / ROWS_PER_PASS;
  constexpr int B_PASSES = BN / ROWS_PER_PASS;          // K-contiguous filter rows
  constexpr int B_UNITS = (BKQ / 4) * (BN / 4);         // FC weight: 4k x 4n byte blocks per slab
  constexpr int B_UPT = B_UNITS / NTHREADS;             // blocks per thread
  static_assert(B_UNITS % NTHREADS == 0, "FC weight tile does not divide over the threads");
  static_assert(A_PASSES + B_PASSES <= 8, "four bits per load in one register");
  constexpr int A_BYTES = BM * LDQ, B_BYTES = BN * LDQ;
  constexpr int OUT_PITCH = BN + 16;                    // output tile staged in LDS, bytes per pixel row
  constexpr int XCH = KGRP > 1 ? KGRP * BM * BN * 4 : 0;  // partial tiles of the groups
  static_assert(2 * KGRP * (A_BYTES + B_BYTES) >= XCH + BM * OUT_PITCH + (BM + 2 * BN + 256) * 4, "epilogue reuses the staging LDS");
  static_assert(KGRP == 1 || (TM == 1 && TN == 1), "the groups share the outputs of one MFMA block per wavefront");

  extern __shared__ __align__(16) unsigned char ldsq[];

  const int per_xcd = gridDim.x >> 3;
  const int w = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (w >= walk.total_work) return;
  int t_ = walk.div_tiles_n.div(w);
  const int tn = w - t_ * walk.tiles_n;
  int t2_ = walk.div_tiles_m.div(t_);
  const int tm = t_ - t2_ * walk.tiles_m;
  const int split = walk.div_groups.div(t2_);
  const int g = t2_ - split * p.groups;

  const int all_tid = threadIdx.x;
  const int grp = KGRP > 1 ? __builtin_amdgcn_readfirstlane(all_tid / NTHREADS) : 0;
  const int tid = KGRP > 1 ? all_tid % NTHREADS : all_tid;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;

  // A 16-byte load at the end of a tensor of any size stays inside the 16-byte block of its last byte.
  const unsigned x_size = p.x_bytes < 16u ? 16u : p.x_bytes, w_size = p.w_bytes < 16u ? 16u : p.w_bytes;
  const __amdgpu_buffer_rsrc_t rsrc_x =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.x), 0, (int)x_size, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_w =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w), 0, (int)w_size, 0x00020000);

  const int kvec = tid % KV;
  const int row0 = tid / KV;
  int a_base[A_PASSES], a_ih0[A_PASSES], a_iw0[A_PASSES];
  {
    const int ohow = p.oh * p.ow;
#pragma unroll
    for (int q = 0; q < A_PASSES; ++q) {
      const int m = tm * BM + row0 + q * ROWS_PER_PASS;
      if (m < p.M) {
        const int img = p.div_ohow.div(m);
        const int rem = m - img * ohow;
        const int oh = p.div_ow.div(rem);
        const int ow = rem - oh * p.ow;
        a_ih0[q] = oh * p.stride_h - p.pad_t;
        a_iw0[q] = ow * p.stride_w - p.pad_l;
        a_base[q] = ((img * p.h + a_ih0[q]) * p.w_ + a_iw0[q]) * p.c + g * p.cg;
      } else {
        a_ih0[q] = INVALID_ROW;
        a_iw0[q] = INVALID_ROW;
        a_base[q] = 0;
      }
    }
  }

  const int slab_begin = split * p.slabs_per_split;
  const int total_slabs = (walk.chunk.chunks + KV - 1) / KV;
  int slab_end = slab_begin + p.slabs_per_split;
  if (slab_end > total_slabs) slab_end = total_slabs;
  const int k_count = walk.chunk.codes_before(slab_end * KV, p) - walk.chunk.codes_before(slab_begin * KV, p);   // codes of this split
  Chunk at = walk.chunk.at((slab_begin + grp) * KV + kvec, p);   // of the next slab to load

  const int xo_fill = (p.x_off & 0xff) * 0x01010101;    // padding = the code of real zero
  const bool need_xsum = p.w_off != 0;
  const bool padded = walk.padded != 0;                 // some tap of some pixel falls on padding (or a row lies past M)
  const bool ragged = p.cg % 16 != 0;                   // a tap's last chunk has cg % 16 codes: the bytes of those
  const v4i short_mask = byte_mask(p.cg % 16);
  // Chunks that run past the end of a tensor (its last pixels', or last filters', short chunks) are fetched from its last
  // 16 bytes and shifted: only tiles that see such pixels or filters look for them.
  const bool at_end = p.cg % 16 != 0 && (tm * BM + BM > p.M - walk.chunk.end_pixels || tn * BN + BN > p.kg - walk.chunk.end_filters);

  struct Stage {                                        // one slab on its way to LDS
    v4i a[A_PASSES], b[B_KN ? B_UPT : B_PASSES];
    unsigned inside;                                    // bit q: the tap of row q lies inside the image; SHORT, PAST
    unsigned over;                                      // 4 bits per load: bytes to shift down
  };
  constexpr unsigned SHORT = 1u << 30, PAST = 1u << 31; // the chunk is a tap's short last one, lies past the reduction
  Stage st[2];
  int asum[A_PASSES];                                   // running sum of staged input codes per row
  int bsum[B_KN ? B_UPT * 4 : B_PASSES];                // running sum of staged filter codes
#pragma unroll
  for (int q = 0; q < A_PASSES; ++q) asum[q] = 0;
#pragma unroll
  for (int q = 0; q < (B_KN ? B_UPT * 4 : B_PASSES); ++q) bsum[q] = 0;

  auto load_global = [&](int slab, Stage& sg) {
    const bool kok = at.r < p.r;                        // past the last tap: nothing of this chunk counts
    const int tap_off = (at.r * p.w_ + at.s) * p.c + at.c;
    sg.inside = (at.c + 16 > p.cg ? SHORT : 0u) | (kok ? 0u : PAST);
    sg.over = 0;
    unsigned off[A_PASSES];
    if (padded) {
#pragma unroll
      for (int q = 0; q < A_PASSES; ++q) {
        const int ih = a_ih0[q] + at.r, iw = a_iw0[q] + at.s;
        const bool in = kok && (unsigned)ih < (unsigned)p.h && (unsigned)iw < (unsigned)p.w_;
        sg.inside |= in ? 1u << q : 0u;
        off[q] = in ? (unsigned)(a_base[q] + tap_off) : OOB;
      }
    } else {
#pragma unroll
      for (int q = 0; q < A_PASSES; ++q) off[q] = kok ? (unsigned)(a_base[q] + tap_off) : OOB;
    }
    if (at_end) {
#pragma unroll
      for (int q = 0; q < A_PASSES; ++q) {
        const unsigned last = x_size - 16u, o = off[q] != OOB && off[q] > last ? off[q] - last : 0u;
        off[q] -= o;
        sg.over |= o << (4 * q);
      }
    }
#pragma unroll
    for (int q = 0; q < A_PASSES; ++q) sg.a[q] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, off[q], 0, 0);
    if (!B_KN) {
      const unsigned koff = (unsigned)((at.r * p.s + at.s) * p.cg + at.c);
#pragma unroll
      for (int q = 0; q < B_PASSES; ++q) {
        const int n = tn * BN + row0 + q * ROWS_PER_PASS;
        unsigned o = kok && n < p.kg ? (unsigned)(g * p.kg + n) * (unsigned)p.Kgemm + koff : OOB;
        if (at_end) {
          const unsigned last = w_size - 16u, over = o != OOB && o > last ? o - last : 0u;
          o -= over;
          sg.over |= over << (4 * (A_PASSES + q));
        }
        sg.b[q] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, o, 0, 0);
      }
    } else {
      // FC weight [Kgemm][k], N contiguous: each thread takes 4 k-rows x 4 columns.  Columns past the last one: the
      // row's last four, shifted (their results are not stored).
#pragma unroll
      for (int q = 0; q < B_UPT; ++q) {
        const int u = tid + q * NTHREADS;
        const int ng = u % (BN / 4), kgp = u / (BN / 4);
        const int col = tn * BN + ng * 4;
        if (p.k >= 4) {
          const unsigned c4 = (unsigned)(col <= p.k - 4 ? col : p.k - 4);
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) {
            const int kgr = slab * BKQ + kgp * 4 + kk;
            sg.b[q][kk] = __builtin_amdgcn_raw_buffer_load_b32(rsrc_w, kgr < p.Kgemm ? (unsigned)kgr * (unsigned)p.k + c4 : OOB, 0, 0);
          }
        } else {
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) {
            const int kgr = slab * BKQ + kgp * 4 + kk;
            int d = 0;
            for (int e = 0; e < p.k; ++e)
              d |= (int)__builtin_amdgcn_raw_buffer_load_b8(rsrc_w, kgr < p.Kgemm && col == 0 ? (unsigned)(kgr * p.k + e) : OOB, 0, 0) << (8 * e);
            sg.b[q][kk] = d;
          }
        }
      }
    }
    walk.chunk.step(at, p.s);
  };

  auto store_lds = [&](int buf, Stage& sg, bool live) {
    const int ones = live ? 0x01010101 : 0;              // uniform
    v4i mask = {-1, -1, -1, -1};                         // (past the reduction the filter's loads gave zeros)
    if (ragged) {
#pragma unroll
      for (int e = 0; e < 4; ++e) mask[e] = sg.inside & SHORT ? short_mask[e] : -1;
    }
    unsigned char* As = ldsq + (grp * 2 + buf) * (A_BYTES + B_BYTES);
    unsigned char* Bs = As + A_BYTES;
#pragma unroll
    for (int q = 0; q < A_PASSES; ++q) {
      v4i v = sg.a[q];
      if (at_end) v = shift_down(v, (sg.over >> (4 * q)) & 15u);
      if (padded) {
        const bool in = sg.inside & (1u << q);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = in ? v[e] : xo_fill;
      }
      if (need_xsum) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = sg.inside & PAST ? 0 : v[e] & mask[e];
        asum[q] = sum_bytes(v, ones, asum[q]);
      }
      *reinterpret_cast<v4i*>(As + (row0 + q * ROWS_PER_PASS) * LDQ + kvec * 16) = v;
    }
    if (!B_KN) {
#pragma unroll
      for (int q = 0; q < B_PASSES; ++q) {
        v4i v = sg.b[q];
        if (at_end) v = shift_down(v, (sg.over >> (4 * (A_PASSES + q))) & 15u);
        if (ragged) v &= mask;
        *reinterpret_cast<v4i*>(Bs + (row0 + q * ROWS_PER_PASS) * LDQ + kvec * 16) = v;
        bsum[q] = sum_bytes(v, ones, bsum[q]);
      }
    } else {
      // transpose the 4 x 4 byte block: every column becomes one dword of 4 consecutive k
#pragma unroll
      for (int q = 0; q < B_UPT; ++q) {
        const int u = tid + q * NTHREADS;
        const int ng = u % (BN / 4), kgp = u / (BN / 4);
        const int col = tn * BN + ng * 4;
        v4i d = sg.b[q];
        if (p.k >= 4 && col > p.k - 4) {
          const int sh = col - (p.k - 4) < 4 ? 8 * (col - (p.k - 4)) : 31;
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) d[kk] = (int)((unsigned)d[kk] >> sh);
        }
        const unsigned t0 = __builtin_amdgcn_perm((unsigned)d[1], (unsigned)d[0], 0x05010400u);
        const unsigned t1 = __builtin_amdgcn_perm((unsigned)d[3], (unsigned)d[2], 0x05010400u);
        const unsigned t2 = __builtin_amdgcn_perm((unsigned)d[1], (unsigned)d[0], 0x07030602u);
        const unsigned t3 = __builtin_amdgcn_perm((unsigned)d[3], (unsigned)d[2], 0x07030602u);
        const v4i o = {(int)__builtin_amdgcn_perm(t1, t0, 0x05040100u), (int)__builtin_amdgcn_perm(t1, t0, 0x07060302u),
                       (int)__builtin_amdgcn_perm(t3, t2, 0x05040100u), (int)__builtin_amdgcn_perm(t3, t2, 0x07060302u)};
#pragma unroll
        for (int nn = 0; nn < 4; ++nn) {
          *reinterpret_cast<int*>(Bs + (ng * 4 + nn) * LDQ + kgp * 4) = o[nn];
          bsum[q * 4 + nn] = __builtin_amdgcn_sdot4(o[nn], ones, bsum[q * 4 + nn], false);
        }
      }
    }
  };

  // acc[i][j]: 32 output channels (rows of the MFMA result) x 32 pixels (columns)
  v16i acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0;

  const int lrow = lane & 31;
  const int lhalf = lane >> 5;

  auto compute = [&](int buf) {
    const unsigned char* As = ldsq + (grp * 2 + buf) * (A_BYTES + B_BYTES);
    const unsigned char* Bs = As + A_BYTES;
#pragma unroll
    for (int k32 = 0; k32 < BKQ / 32; ++k32) {
      // each lane feeds 16 consecutive codes of its row; lanes 32..63 take the upper 16 of the 32
      v4i a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i)
        a[i] = *reinterpret_cast<const v4i*>(As + (wm * WTM + i * 32 + lrow) * LDQ + k32 * 32 + lhalf * 16);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        b[j] = *reinterpret_cast<const v4i*>(Bs + (wn * WTN + j * 32 + lrow) * LDQ + k32 * 32 + lhalf * 16);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)   // filter fragment as the row operand: result rows = channels
          acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b[j], a[i], acc[i][j], 0, 0, 0);
    }
  };

  // A group's slab number n is in its LDS buffer n % 2 while slab n + 1 waits in stage (n + 1) % 2 and slab n + 2 is being
  // fetched into the stage slab n came from.  No load sits in a branch whose paths join while it is in flight (the
  // compiler would wait for all of them there): a full pair of slabs per trip, then the one to three that are left.  The
  // groups run in step; where group 0 has one slab more the others stage it too, without summing or multiplying it.
  if (slab_begin < slab_end) {
    int slab = slab_begin + grp;
    int left = (slab_end - slab_begin + KGRP - 1) / KGRP;
    auto advance = [&](int u, bool store) {              // multiply the slab in LDS, stage the one after it
      if (KGRP == 1 || slab < slab_end) compute(u);
      if (store) store_lds(u ^ 1, st[u ^ 1], KGRP == 1 || slab + KGRP < slab_end);
      __syncthreads();
      slab += KGRP;
      --left;
    };
    load_global(slab, st[0]);
    if (left > 1) {
      load_global(slab + KGRP, st[1]);
      store_lds(0, st[0], true);
      __syncthreads();
      while (left > 3) {
        load_global(slab + 2 * KGRP, st[0]);
        advance(0, true);
        load_global(slab + 2 * KGRP, st[1]);
        advance(1, true);
      }
      if (left == 3) {
        load_global(slab + 2 * KGRP, st[0]);
        advance(0, true);
        advance(1, true);
        advance(0, false);
      } else {
        advance(0, true);
        advance(1, false);
      }
    } else {
      store_lds(0, st[0], KGRP == 1 || slab < slab_end);
      __syncthreads();
      advance(0, false);
    }
  }

  // ---- epilogue.  LDS (staging buffers are free now):
  //   out   [BM][OUT_PITCH] bytes : requantized tile, pixel-major
  //   xsum  [BM] int, wsum [BN] int : code sums;  cterm [BN] int : per-channel additive term
  //   and, with several groups, their partial tiles ahead of it: [group][four registers][wavefront's lanes] of int4
  if constexpr (KGRP > 1) {
    v4i* xch = reinterpret_cast<v4i*>(ldsq);
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      v4i v;
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] = acc[0][0][q4 * 4 + t];
      xch[(grp * 4 + q4) * NTHREADS + tid] = v;
    }
  }
  unsigned char* out = ldsq + XCH;
  int* xsum = reinterpret_cast<int*>(out + BM * OUT_PITCH);
  int* wsum = xsum + BM;
  int* cterm = wsum + BN;
  int* addlut = cterm + BN;                             // [256] the addend's code (as an unsigned byte) -> its term
  constexpr int CHUNKS = BN / 16;                       // 16-byte pieces of a pixel row of the tile
  for (int i = all_tid; i < BM + BN; i += ALL_THREADS) xsum[i] = 0;
  __syncthreads();
  const bool adding = !CHAINV && p.addend && p.split_k == 1;   // uniform: tensor-add link of the chain
  if (adding) {
    // The addend's tile into `out`, whole 16-byte pieces whatever the alignment (the tensor's last ones fetched from its
    // last 16 bytes and shifted); its codes' terms once per workgroup.  Byte by byte, each rescaled for itself, a layer
    // with an addend took twice as long as without (3x3 16 -> 512 on 37x37 at batch 24 50 us instead of 26).
    const unsigned y_size = (unsigned)p.M * (unsigned)p.k < 16u ? 16u : (unsigned)p.M * (unsigned)p.k;
    const __amdgpu_buffer_rsrc_t rsrc_add = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.addend), 0, (int)y_size, 0x00020000);
    for (int i = all_tid; i < 256; i += ALL_THREADS) addlut[i] = rescale_term((int)(signed char)i - p.r_off, p.r_mant, p.r_shift);
    for (int u = all_tid; u < BM * CHUNKS; u += ALL_THREADS) {
      const int lr = u / CHUNKS, ch = u % CHUNKS;
      const int row = tm * BM + lr, col = tn * BN + ch * 16;
      unsigned off = row < p.M && col < p.kg ? (unsigned)row * (unsigned)p.k + (unsigned)(g * p.kg + col) : OOB;
      const unsigned over = off != OOB && off > y_size - 16u ? off - (y_size - 16u) : 0u;
      v4i v = __builtin_amdgcn_raw_buffer_load_b128(rsrc_add, off - over, 0, 0);
      if (over) v = shift_down(v, over);
      *reinterpret_cast<v4i*>(out + lr * OUT_PITCH + ch * 16) = v;
    }
  }
  if (need_xsum) {
#pragma unroll
    for (int q = 0; q < A_PASSES; ++q) atomicAdd(&xsum[row0 + q * ROWS_PER_PASS], asum[q]);
  }
  if (!B_KN) {
#pragma unroll
    for (int q = 0; q < B_PASSES; ++q) atomicAdd(&wsum[row0 + q * ROWS_PER_PASS], bsum[q]);
  } else {
#pragma unroll
    for (int q = 0; q < B_UPT; ++q) {
      const int u = tid + q * NTHREADS;
      const int ng = u % (BN / 4);
#pragma unroll
      for (int nn = 0; nn < 4; ++nn) atomicAdd(&wsum[ng * 4 + nn], bsum[q * 4 + nn]);
    }
  }
  __syncthreads();
  // The correction terms are combined modulo 2^32 (unsigned): each may exceed the final value, the
  // true accumulator fits int32 by contract, so the wrapped sum is exact.
  const int* __restrict__ bias = static_cast<const int*>(p.bias);
  for (int i = all_tid; i < BN; i += ALL_THREADS) {
    const int col = tn * BN + i;
    unsigned ct = (unsigned)k_count * (unsigned)(p.x_off * p.w_off) - (unsigned)p.x_off * (unsigned)wsum[i];
    if (p.split_k == 1 && bias && col < p.kg) ct += (unsigned)bias[g * p.kg + col];
    cterm[i] = (int)ct;
  }
  __syncthreads();

  // this thread's outputs: with several groups, registers 4 q4 .. 4 q4 + 3 for the q4 of its group, summed over the groups
  constexpr int Q4S = 4 / KGRP;
  if constexpr (KGRP > 1) {
    const v4i* xch = reinterpret_cast<const v4i*>(ldsq);
#pragma unroll
    for (int i = 0; i < Q4S; ++i) {
      v4i v = {0, 0, 0, 0};
#pragma unroll
      for (int k = 0; k < KGRP; ++k) v += xch[(k * 4 + grp * Q4S + i) * NTHREADS + tid];
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[0][0][i * 4 + t] = v[t];
    }
  }

  if (p.split_k == 1) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int lr = wm * WTM + i * 32 + lrow;                        // pixel row inside the tile
      const unsigned rowterm = need_xsum ? (unsigned)p.w_off * (unsigned)xsum[lr] : 0u;
      const int row = tm * BM + lr;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
#pragma unroll
        for (int q4 = 0; q4 < Q4S; ++q4) {
          const int lc = wn * WTN + j * 32 + (grp * Q4S + q4) * 8 + lhalf * 4;   // first of 4 consecutive channels
          const v4i ct = *reinterpret_cast<const v4i*>(cterm + lc);
          unsigned* four = reinterpret_cast<unsigned*>(out + lr * OUT_PITCH + lc);
          const unsigned codes = adding ? *four : 0u;
          unsigned packed = 0;
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            int v = (int)((unsigned)acc[i][j][q4 * 4 + t] + (unsigned)ct[t] - rowterm);
            if (CHAINV) {                                             // general op list
              const int col = tn * BN + lc + t;
              if (row < p.M && col < p.kg) v = apply_chain_i8(p, v, (size_t)row * p.k + g * p.kg + col);
            } else if (adding) {
              v += addlut[(codes >> (8 * t)) & 0xffu];
            }
            packed |= ((unsigned)requantize(v, p.mant, p.shift, p.y_off, p.lo, p.hi) & 0xffu) << (t * 8);
          }
          *four = packed;
        }
      }
    }
    __syncthreads();
    // copy out: 16 bytes of one pixel row per thread and pass, at whatever address the row starts
    signed char* __restrict__ Y = static_cast<signed char*>(p.y);
    for (int u = all_tid; u < BM * CHUNKS; u += ALL_THREADS) {
      const int lr = u / CHUNKS, ch = u % CHUNKS;
      const int row = tm * BM + lr, col = tn * BN + ch * 16;
      if (row >= p.M || col >= p.kg) continue;
      signed char* dst = Y + (size_t)row * p.k + g * p.kg + col;
      const v4i codes = *reinterpret_cast<const v4i*>(out + lr * OUT_PITCH + ch * 16);
      if (col + 16 <= p.kg) __builtin_memcpy(dst, &codes, 16);
      else store_front(dst, codes, p.kg - col);
    }
  } else {
    int* __restrict__ part = static_cast<int*>(p.partial);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int lr = wm * WTM + i * 32 + lrow;
      const int row = tm * BM + lr;
      const unsigned rowterm = need_xsum ? (unsigned)p.w_off * (unsigned)xsum[lr] : 0u;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
#pragma unroll
        for (int e = 0; e < 4 * Q4S; ++e) {
          const int lc = wn * WTN + j * 32 + (grp * Q4S + (e >> 2)) * 8 + lhalf * 4 + (e & 3);
          const int col = tn * BN + lc;
          if (row >= p.M || col >= p.kg) continue;
          part[((size_t)split * p.M + row) * p.k + g * p.kg + col] =
              (int)((unsigned)acc[i][j][e] + (unsigned)cterm[lc] - rowterm);
        }
      }
    }
  }
}

// A thread owns W consecutive outputs (W = 4 when the row length allows: 16-byte loads of the int32
// partials, one dword of codes stored) and walks the splits eight at a time with the loads in flight
// together.  Integer sums: any order gives the same result.
template <int W>
__global__ __launch_bounds__(256) void splitk_finish_i8(const int* __restrict__ partial,
                                                        const int* __restrict__ bias,
                                                        const signed char* addend, int r_off, int r_mant,
                                                        int r_shift, signed char* y, int total, int k,
                                                        int split_k, int mant, int shift, int y_off,
                                                        int lo, int hi) {
  fetch_arguments(partial, bias, addend, r_off, r_mant, r_shift, y, total, k, split_k, mant, shift, y_off, lo, hi);
  typedef unsigned vec __attribute__((ext_vector_type(W)));
  const int groups = total / W;                      // W divides total (the launcher checks)
  for (int gi = blockIdx.x * blockDim.x + threadIdx.x; gi < groups; gi += gridDim.x * blockDim.x) {
    const size_t i = (size_t)gi * W;
    vec v = {};
    for (int s = 0; s < split_k; s += 8) {
      vec t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int su = s + u < split_k ? s + u : s;
        t[u] = *reinterpret_cast<const vec*>(partial + (size_t)su * total + i);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (s + u < split_k) v += t[u];
    }
    if (bias) v += *reinterpret_cast<const vec*>(bias + i % k);      // W divides k: no wrap inside the vector
    int q[W];
#pragma unroll
    for (int e = 0; e < W; ++e) {
      unsigned a = v[e];
      if (addend) a += (unsigned)rescale_term((int)addend[i + e] - r_off, r_mant, r_shift);
      q[e] = requantize((int)a, mant, shift, y_off, lo, hi);
    }
    if (W == 4) {
      *reinterpret_cast<unsigned*>(y + i) = pack_codes(q[0], q[1], q[2], q[3]);
    } else {
#pragma unroll
      for (int e = 0; e < W; ++e) y[i + e] = (signed char)q[e];
    }
  }
}

// Finish of a split reduction whose element-wise chain is a general op list.
__global__ __launch_bounds__(256) void splitk_finish_chain_i8(const Problem p, int total) {
  fetch_arguments(p, total);
  const int* __restrict__ partial = static_cast<const int*>(p.partial);
  const int* __restrict__ bias = static_cast<const int*>(p.bias);
  signed char* y = static_cast<signed char*>(p.y);
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    unsigned a = 0;
    for (int s = 0; s < p.split_k; ++s) a += (unsigned)partial[(size_t)s * total + i];
    if (bias) a += (unsigned)bias[i % p.k];
    const int v = apply_chain_i8(p, (int)a, (size_t)i);
    y[i] = (signed char)requantize(v, p.mant, p.shift, p.y_off, p.lo, p.hi);
  }
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int KGRP, bool B_KN, bool CHAINV = false>
hipError_t launch_variant(const Problem& p, const Plan& plan, hipStream_t stream) {
  auto kern = igemm_i8_kernel<BM, BN, WAVES_M, WAVES_N, KGRP, B_KN, CHAINV>;
  constexpr int lds_bytes = 2 * KGRP * (BM + BN) * LDQ;
  constexpr int nthreads = 64 * WAVES_M * WAVES_N * KGRP;
  // once per instantiation; initialisation of a function-local static is thread-safe
  static const hipError_t attr_status = hipFuncSetAttribute(
      reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
  if (attr_status != hipSuccess) return attr_status;
  const long long total_work = (long long)plan.tiles_m * plan.tiles_n * p.groups * plan.split_k;
  const long long grid_x = ((total_work + 7) / 8) * 8;
  Walk walk;
  walk.div_tiles_n = make_fastdiv((uint32_t)plan.tiles_n);
  walk.div_tiles_m = make_fastdiv((uint32_t)plan.tiles_m);
  walk.div_groups = make_fastdiv((uint32_t)p.groups);
  walk.tiles_n = plan.tiles_n;
  walk.tiles_m = plan.tiles_m;
  walk.total_work = (int)total_work;
  walk.padded = p.pad_t != 0 || p.pad_l != 0 || (p.oh - 1) * p.stride_h + p.r > p.h || (p.ow - 1) * p.stride_w + p.s > p.w_ ||
                p.M % BM != 0;
  walk.chunk = make_chunk_walk(p, KV * KGRP);
  dim3 grid((unsigned)grid_x, 1, 1), block(nthreads, 1, 1);
  hipLaunchKernelGGL(kern, grid, block, lds_bytes, stream, p, walk);
  return hipGetLastError();
}

struct TileI8 { int bm, bn, wm, wn, kgrp; const char* name; };
constexpr TileI8 kTilesI8[] = {
    {64, 64, 2, 2, 1, "64x64w4"},       // 0: default
    {128, 64, 4, 2, 1, "128x64w8"},     // 1
    {128, 128, 2, 4, 1, "128x128w8"},   // 2
    {128, 128, 2, 2, 1, "128x128w4"},   // 3
    {0, 0, 0, 0, 0, ""}, {0, 0, 0, 0, 0, ""},   // 4, 5: the kernel for large contractions, 128 x 128 and 128 x 64
    {64, 64, 2, 2, 2, "64x64w4k2"},     // 6
    {64, 64, 2, 2, 4, "64x64w4k4"},     // 7
};
constexpr int kNumTilesI8 = sizeof(kTilesI8) / sizeof(kTilesI8[0]);

template <int BM, int BN, int WM, int WN, int KGRP>
hipError_t launch_tile(const Problem& p, const Plan& plan, hipStream_t stream, bool fc) {
  return fc ? launch_variant<BM, BN, WM, WN, KGRP, true>(p, plan, stream)
            : launch_variant<BM, BN, WM, WN, KGRP, false>(p, plan, stream);
}

}  // namespace

namespace {
// What tiles of several wavefront groups take (microseconds; 20 layers of 21 to 47 slabs, within 15 %).
double groups_us(const Problem& p, long long tiles, int split, int slabs, int kgrp) {
  const double slab = (p.cg % 16 == 0 ? 0.31 : 0.43) * (kgrp == 4 ? 1.0 : 2.0), slots = 1024 / kgrp;
  const double rounds = (double)(long long)((tiles * split + slots - 1) / slots);
  return rounds * (4.6 + slab * slabs) + (split > 1 ? 4.0 + 0.6e-6 * 4.0 * split * (double)p.M * p.k : 0.0);
}

// What a convolution takes in microseconds on the kernel `pl` has it on, 0: not known.  Fitted to 2400 layers of 16 to 768 channels and
// 49 to 400000 pixels, to the geometric mean of the times with operands in the caches and from memory (median errors: conv_small_i8 and
// its sliced form 4 %, tiles 3 to 5 %, the wide kernel 4 and 6 %).  Tiles: to begin with, per workgroup of a CU in turn, per slab of
// those, more per slab where channels end inside sixteen and inside four, per megabyte of the tensors, for a split, per megabyte of its parts.
struct TileCost { double fixed, per_cu, slab, ragged, by_value, mb, split, part; };
constexpr TileCost kTileCost[kNumTilesI8] = {
    {5.01, 0.0, 0.350, 0.119, 0.055, 0.072, 5.47, 0.0}, {2.50, 1.586, 0.478, 0.152, 0.083, 0.114, 0.0, 0.0},
    {4.91, 1.363, 0.578, 0.250, 0.097, 0.235, 0.0, 0.0}, {}, {}, {}, {5.81, 0.0, 0.258, 0.146, 0.058, 0.076, 0.0, 0.0},
    {0.0, 6.055, 0.287, 0.126, 0.060, 0.081, 1.94, 1.141},
};
double planned_us(const Problem& p, const Plan& pl) {
  const double out = 1e-6 * (double)p.M * p.k, mb = 1e-6 * ((double)p.x_bytes + p.w_bytes) + (p.addend ? 2.0 : 1.0) * out;
  const double parts = pl.split_k > 1 ? 4.0 * pl.split_k * out : 0.0;
  if (pl.kernel == KERNEL_SMALL || pl.kernel == KERNEL_SMALL_SPLIT) {
    const long long t32 = (long long)((p.M + 31) / 32) * ((p.k + 31) / 32) * pl.split_k;
    const double rounds = (double)((t32 + 255) / 256), chunks = p.r * p.s * ((p.cg + 15) / 16);
    if (pl.kernel == KERNEL_SMALL_SPLIT) return 5.83 + 1.78 * rounds + 0.353 * parts + 0.345 * mb;
    return 3.90 + rounds * (0.107 + (p.cg % 4 != 0 ? 0.0366 : 0.0161) * chunks) + (p.cg % 16 != 0 ? 0.0203 : 0.0071) * chunks +
           1.25 * out + 0.067 * mb;
  }
  const double t = (double)pl.tiles_m * pl.tiles_n * pl.split_k;
  double per_cu = t < 1024 ? (double)(int)((t + 255) / 256) : t / 256;
  if (per_cu < 1.0) per_cu = 1.0;
  const double slabs = per_cu * pl.slabs_per_split;
  if (pl.kernel == KERNEL_WIDE) {
    const double fetch = (t > 256 ? t / 256 : 1.0) * pl.slabs_per_split;
    return pl.bn == 128 ? 4.70 + 0.587 * slabs + 0.049 * fetch + 0.765 * out + 0.100 * mb
                        : 5.83 + 0.231 * slabs + 0.244 * fetch + 0.369 * out + 0.106 * mb + (pl.split_k > 1 ? 1.81 : 0.0) + 0.489 * parts;
  }
  if (pl.kernel != KERNEL_TILED) return 0.0;
  const TileCost& c = kTileCost[pl.tile];
  return c.fixed + c.per_cu * per_cu + slabs * (c.slab + (p.cg % 16 != 0 ? c.ragged : 0.0) + (p.cg % 4 != 0 ? c.by_value : 0.0)) + c.mb * mb +
         (pl.split_k > 1 ? c.split : 0.0) + c.part * parts;
}
constexpr double kMargin = 1.02;                        // what a kernel's estimate has to be below the planned one's by

Plan plan_i8_rest(const Problem& p, bool allow_split) {
  Plan pl;
  pl.kernel = KERNEL_TILED;
  pl.tile = 0;
  pl.bm = pl.bn = pl.bk = 0;
  pl.tiles_m = pl.tiles_n = 1;
  pl.slabs = 1;
  pl.split_k = 1;
  pl.slabs_per_split = 1;
  int forced = knob_or(KNOB_I8_TILE, -1);         // experiments and tests: force a tile variant
  if (p.chain_n > 0) forced = 0;                  // a general chain: only the generic 64 x 64 kernel implements it
  if (forced < 0) {
    // kernels of their own, no workspace
    if (dw_i8_applicable(p)) { pl.kernel = KERNEL_DW; return pl; }
    if (smallc_i8_applicable(p) && !p.addend) { pl.kernel = KERNEL_SMALLC; return pl; }
    if (pw_i8_applicable(p)) { pl.kernel = KERNEL_PW; return pl; }
    if (k3c64_i8_applicable(p)) { pl.kernel = KERNEL_K3C64; return pl; }
    if (fc_small_i8_applicable(p)) { pl.kernel = KERNEL_FC_SMALL; return pl; }
    if (conv_small_i8_applicable(p)) { pl.kernel = KERNEL_SMALL; return pl; }
    const int slices = allow_split ? conv_small_i8_splits(p) : 0;
    if (slices > 1) {
      pl.kernel = KERNEL_SMALL_SPLIT;
      pl.split_k = slices;
      return pl;
    }
  }
  pl.bk = BKQ;
  pl.slabs = (p.r * p.s * ((p.cg + 15) / 16) + KV - 1) / KV;
  int tile = 0;
  if (forced >= 0 && forced < kNumTilesI8 && kTilesI8[forced].bm > 0) tile = forced;
  // Large contractions (deep reduction, enough pixels and channels for 128-wide tiles) take the
  // kernel built for them.
  if (wide_i8_applicable(p)) {
    if (forced == 4 || forced == 5) return plan_wide_i8(p, (forced == 4 || p.b_is_kn) ? 128 : 64, allow_split);
    if (forced < 0 && p.Kgemm >= 256 && p.M >= 96 && p.kg >= 128 && !pw_i8_applicable(p)) {
      // convolutions with at most one 128 x 128 tile per CU take 128 x 64 tiles: twice the workgroups
      // for the same bytes per workgroup (measured: 3x3 512->512 on 7x7 at batch 32 21.8 -> 19.6 us,
      // 1x1 512->2048 on 7x7 9.1 -> 8.5 us; 1x1 256->1024 on 14x14 with 392 tiles stays at 128 x 128)
      const long long t128 = (long long)((p.M + 127) / 128) * ((p.kg + 127) / 128) * p.groups;
      const Plan wide = plan_wide_i8(p, (!p.b_is_kn && t128 <= 256) ? 64 : 128, allow_split);
      // Channels that are no multiple of sixteen: not on reductions of less than five slabs, where the generic tiles are as fast
      // or faster (3x3 stride 2 40->328 on 100x100 at batch 21 31.8 us, 35.3 there; 1x1 296->984 on 37x57 at batch 15 41.9 and
      // 47.1), nor where tiles of four wavefront groups get through their slabs sooner (3x3 152->424 on 24x24 at batch 4 10.6
      // and 12.3); elsewhere 0.54 to 0.9 of the generic tiles' time (3x3 744->960 on 18x18 at batch 12 88 -> 54).
      const long long t64 = (long long)((p.M + 63) / 64) * ((p.kg + 63) / 64) * p.groups;
      const double wide_us = 6.0 + 0.55 * wide.slabs_per_split + (wide.split_k > 1 ? 3.5 : 0.0);
      const bool sooner = t64 <= 256 && pl.slabs >= 8 && groups_us(p, t64, 1, pl.slabs, 4) < wide_us;
      if (p.b_is_kn || p.cg % 16 == 0 || (wide.slabs >= 5 && !sooner)) return wide;
    }
  }
  if (forced < 0) {
    const long long t64 = (long long)((p.M + 63) / 64) * ((p.kg + 63) / 64) * p.groups;
    const long long t128 = (long long)((p.M + 127) / 128) * ((p.kg + 127) / 128) * p.groups;
    // up to about one 64 x 64 tile per CU: several wavefront groups per tile, the chain of slabs is what counts (3x3 72->120 on
    // 33x45 at batch 5, 232 tiles: 10.4 us with one group, 8.2 with two; FC 76x808x208, 8 tiles: 12.0, 9.6, 8.9 with four);
    // at twice that many tiles the groups only take each other's room (3x3 19->119 on 68x94 at batch 3, 600 tiles: 10.6 -> 14.2)
    // (and four groups fill a CU: beyond 256 tiles they take a second round, 3x3 256->40 on 48x30 at batch 12, 270 tiles: 20.0 us,
    // 14.5 with two)
    if (t64 <= 320 && pl.slabs >= 2) tile = pl.slabs >= 8 && t64 <= 256 ? 7 : 6;
    // many tiles: the larger ones read each operand fewer times (3x3 120->128 on 56x56 at batch 16: 33 us with 64 x 64 tiles,
    // 26 us with 128 x 128; 1x1 344->176 stride 2 on 85x86 at batch 11, three slabs: 11.1 -> 10.1 us with 128 x 64; with a
    // slab or two the output is what counts, and there have to be four tiles per CU: 1x1 40->896 on 40x40 at batch 24
    // 36.1 us with 128 x 64, 30.4 with 128 x 128)
    else if (!p.b_is_kn && t128 >= (pl.slabs >= 4 ? 256 : 1000) && p.kg > 64) tile = 2;
    else if (t64 >= 900) tile = 1;
  }
  pl.tile = tile;
  pl.bm = kTilesI8[tile].bm;
  pl.bn = kTilesI8[tile].bn;
  pl.tiles_m = (p.M + pl.bm - 1) / pl.bm;
  pl.tiles_n = (p.kg + pl.bn - 1) / pl.bn;
  pl.split_k = 1;
  pl.slabs_per_split = pl.slabs;
  const long long t = (long long)pl.tiles_m * pl.tiles_n * p.groups;
  // Split the reduction when the tiles alone cannot fill the chip: among the split factors that keep
  // at least four slabs per workgroup, the smallest that fills >= 90 % of the resident-workgroup
  // slots of its last round, else the one that fills them best.  With several wavefront groups per tile, whose workgroups fill a
  // CU or half of one and get through their slabs several times as fast, the one that takes the least by their measured times:
  // a start and so much per slab for each round, and a second kernel for the parts (3x3 288->112 on 31x46 at batch 3, 134 tiles,
  // 21 slabs: 11.8 us unsplit, 27 in five).
  const int kgrp = kTilesI8[tile].kgrp;
  const long long slots = 1024 / kgrp;
  const int min_slabs = kgrp > 1 ? 21 : 8;
  if (allow_split && t < slots && pl.slabs >= min_slabs) {
    int max_split = pl.slabs / 4 < 64 ? pl.slabs / 4 : 64;
    if (t >= 256 && max_split > p.Kgemm / 3072) max_split = p.Kgemm / 3072;   // int32 partials are 4x the output
    int best = 1;
    double best_u = 0.0, best_us = 0.0;
    for (int sk = 1; sk <= max_split; ++sk) {
      const int sps = (pl.slabs + sk - 1) / sk;
      const int real = (pl.slabs + sps - 1) / sps;
      if (real != sk) continue;
      const long long blocks = t * sk;
      if (kgrp > 1) {
        const double us = groups_us(p, t, sk, sps, kgrp);
        if (sk == 1 || us < best_us) { best_us = us; best = sk; }
        continue;
      }
      const double u = (double)blocks / (double)(((blocks + slots - 1) / slots) * slots);
      if (u > best_u + 1e-9) { best_u = u; best = sk; }
      if (u >= 0.9) { best = sk; break; }
    }
    if (knob_is_set(KNOB_I8_SPLIT)) {                      // experiments: clamped to what the slabs allow
      best = knob(KNOB_I8_SPLIT);
      if (best < 1) best = 1;
      if (best > max_split) best = max_split;
    }
    if (best > 1) {
      pl.slabs_per_split = (pl.slabs + best - 1) / best;
      pl.split_k = (pl.slabs + pl.slabs_per_split - 1) / pl.slabs_per_split;
    }
  }
  return pl;
}

// A kernel that needs no workspace in place of `rest`; the queries name what they named before.
Plan instead_of(const Problem& p, const Plan& rest, int kernel, int form, double us) {
  Plan pl;
  pl.kernel = kernel;
  pl.tile = form;
  pl.bm = pl.bn = pl.bk = 0;
  pl.tiles_m = pl.tiles_n = pl.slabs = pl.split_k = pl.slabs_per_split = 1;
  pl.us = (float)us;
  pl.stood_in_for = rest.kernel == KERNEL_FEW ? rest.stood_in_for
                                              : rest.split_k > 1 ? (size_t)rest.split_k * (size_t)p.M * (size_t)p.k * 4u : 0u;
  return pl;
}

// Convolutions on few pixels: conv_few_i8 in place of the tiled kernel and of both forms of conv_small_i8 where its estimate is
// lower than theirs by two in a hundred.  Of the time of those, over 1200 layers drawn after the fit, operands in the caches and from
// memory: one launch of conv_small_i8 0.83 and 0.92 (250 layers move), its slices 0.82 and 0.86 (36), tiles 0.75 and 0.81 (41); the
// worst layer 1.09.
Plan few_or(const Problem& p, const Plan& rest) {
  const int mode = knob_or(KNOB_I8_FEW, 1);             // 0: off, 2: any size (tests)
  // (with fewer chunks conv_small_i8 is as fast, and such calls are as long as their way through here, 0.1 us of 4.3)
  if (mode == 1 && rest.kernel == KERNEL_SMALL && p.r * p.s * ((p.cg + 15) / 16) < 16) return rest;
  double us = 0.0;
  const int form = few_i8_form(p, &us);
  if (form < 0) return rest;
  if (mode != 2) {
    if (kMargin * us > planned_us(p, rest)) return rest;
    for (const Knob k : {KNOB_I8_TILE, KNOB_I8_SPLIT, KNOB_I8_SMALL_MAX_TILES})
      if (knob_is_set(k)) return rest;                   // another kernel is asked for
  }
  return instead_of(p, rest, KERNEL_FEW, form, us);
}

// Convolutions whose filters fit the LDS of a CU in slices: conv_short_i8 where its estimate is lower than that of the kernel that
// would run by two in a hundred.  Of the time of those, over 900 drawn layers, operands in the caches and from memory together: tiles 0.69 (245
// move, the slowest 0.98), the wide kernel 0.73 (53, 0.94), conv_small_i8 as below.  All choices together lie 1.6 % above the best one for each.
// The kernels for one kind of layer stay (1x1 256->64 on 56x56 at batch 32 8.6 us, 10.4 here).
Plan short_or(const Problem& p, const Plan& rest) {
  const int mode = knob_or(KNOB_I8_SHORT, 1);           // 0: off, 2: any layer that fits (tests)
  if (mode != 2 && rest.kernel != KERNEL_WIDE && rest.kernel != KERNEL_TILED && rest.kernel != KERNEL_FEW && rest.kernel != KERNEL_SMALL) return rest;
  // (128 x 128 tiles of several taps over whole cache lines of channels: equal, 3x3 128->256 on 56x56 at batch 6 17.7 us, 18.1
  // here, at batch 12 28.6 and 26.0)
  if (mode != 2 && rest.kernel == KERNEL_WIDE && p.c % 128 == 0 && p.r * p.s > 1 && rest.bn == 128) return rest;
  // (conv_small_i8's time, fitted to 689 layers: median error 3 %.  By it and the margins 129 of those 900 move, 0.89 of their time, two above 1.08
  // of it, 3x3 stride 2 104->688 on 31x31 at batch 3 8.9 -> 10.6 us)
  auto small_us = [&]() {
    const long long t32 = (long long)((p.M + 31) / 32) * ((p.k + 31) / 32);
    const double rounds = (double)((t32 + 255) / 256), chunks = p.r * p.s * ((p.c + 15) / 16), out = 1e-6 * (double)p.M * p.k;
    return 4.196 + rounds * (0.197 + (p.c % 4 != 0 ? 0.0415 : 0.0211) * chunks) + (p.c % 16 != 0 ? 0.0155 : 0.0) * chunks + 0.347 * out +
           0.0851 * (1e-6 * ((double)p.x_bytes + p.w_bytes) + (p.addend ? 2.0 : 1.0) * out) + (p.addend ? 0.232 : 0.0);
  };
  const double other = mode == 2 ? 0.0 : rest.kernel == KERNEL_FEW ? (double)rest.us : rest.kernel == KERNEL_SMALL ? small_us() : planned_us(p, rest);
  double us = 0.0;
  const int form = short_i8_form(p, other / kMargin, &us);
  if (form < 0) return rest;
  // (where a slice holds one tile of a long reduction, the estimate is anywhere from 0.66 to 1.12 of the time)
  // (conv_small_i8 with several taps: within 8 % the two are as fast, 3x3 stride 2 48->376 on 36x36 at batch 5 5.6 us on either)
  const double margin = form == 1 && p.r * p.s * ((p.cg + 15) / 16) >= 72 ? 1.3 : rest.kernel == KERNEL_SMALL && p.r * p.s > 1 ? 1.08 : kMargin;
  if (mode != 2 && margin * us > other) return rest;
  if (mode != 2)
    for (const Knob k : {KNOB_I8_TILE, KNOB_I8_SPLIT, KNOB_I8_SMALL_MAX_TILES, KNOB_I8_WIDE_SPLIT, KNOB_I8_WIDE_NBUF, KNOB_I8_FEW})
      if (knob_is_set(k)) return rest;                   // another kernel is asked for
  return instead_of(p, rest, KERNEL_SHORT, form, us);
}
}  // namespace

Plan plan_i8(const Problem& p, bool allow_split) {
  const Plan rest = plan_i8_rest(p, allow_split);
  const bool may_move = !p.b_is_kn && (rest.kernel == KERNEL_TILED || rest.kernel == KERNEL_SMALL || rest.kernel == KERNEL_SMALL_SPLIT);
  return short_or(p, may_move || knob_or(KNOB_I8_FEW, 1) == 2 ? few_or(p, rest) : rest);
}

hipError_t launch_i8(const Problem& p_in, const Plan& plan, hipStream_t stream, const char** variant) {
  switch (plan.kernel) {
    case KERNEL_DW: return launch_dw_i8(p_in, stream, variant);
    case KERNEL_SMALLC: return launch_smallc_i8(p_in, stream, variant);
    case KERNEL_PW: return launch_pw_i8(p_in, stream, variant);
    case KERNEL_K3C64: return launch_k3c64_i8(p_in, stream, variant);
    case KERNEL_FC_SMALL: return launch_fc_small_i8(p_in, stream, variant);
    case KERNEL_SMALL: return launch_conv_small_i8(p_in, stream, variant);
    case KERNEL_SHORT: return launch_short_i8(p_in, plan.tile, stream, variant);
    case KERNEL_FEW: return launch_few_i8(p_in, plan.tile, stream, variant);
    default: break;
  }
  if (plan.split_k > 1 && !p_in.partial) return hipErrorInvalidValue;   // the ABI layer never plans a split without a workspace
  Problem p = p_in;
  p.split_k = plan.split_k;
  p.slabs_per_split = plan.slabs_per_split;
  const bool fc = p.b_is_kn != 0;
  hipError_t e;
  if (plan.kernel == KERNEL_SMALL_SPLIT) {
    e = launch_conv_small_i8(p, stream, variant);
  } else if (plan.kernel == KERNEL_WIDE) {
    e = launch_wide_i8(p, plan, stream, variant);
  } else if (p.chain_n > 0) {
    if (fc || plan.tile != 0) return hipErrorInvalidValue;
    *variant = "igemm_i8_64x64w4_conv_chainv";
    e = launch_variant<64, 64, 2, 2, 1, false, true>(p, plan, stream);
  } else {
    static thread_local char name[64];
    snprintf(name, sizeof(name), "igemm_i8_%s_%s", kTilesI8[plan.tile].name, fc ? "fc" : "conv");
    *variant = name;
    switch (plan.tile) {
      case 0: e = launch_tile<64, 64, 2, 2, 1>(p, plan, stream, fc); break;
      case 1: e = launch_tile<128, 64, 4, 2, 1>(p, plan, stream, fc); break;
      case 2: e = launch_tile<128, 128, 2, 4, 1>(p, plan, stream, fc); break;
      case 3: e = launch_tile<128, 128, 2, 2, 1>(p, plan, stream, fc); break;
      case 6: e = launch_tile<64, 64, 2, 2, 2>(p, plan, stream, fc); break;
      case 7: e = launch_tile<64, 64, 2, 2, 4>(p, plan, stream, fc); break;
      default: return hipErrorInvalidValue;
    }
  }
  if (e != hipSuccess) return e;
  if (plan.split_k > 1 && p.chain_n > 0) {
    const int total = p.M * p.k;
    int blocks = (total + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(splitk_finish_chain_i8, dim3(blocks), dim3(256), 0, stream, p, total);
    e = hipGetLastError();
  } else if (plan.split_k > 1) {
    const int total = p.M * p.k;
    const bool wide = p.k % 4 == 0 && (reinterpret_cast<uintptr_t>(p.bias) & 15) == 0;   // y, partial are 16-byte aligned
    int blocks = (total / (wide ? 4 : 1) + 255) / 256;
    if (blocks > 2048) blocks = 2048;
    auto finish_kernel = wide ? splitk_finish_i8<4> : splitk_finish_i8<1>;
    hipLaunchKernelGGL(finish_kernel, dim3(blocks), dim3(256), 0, stream,
                       static_cast<const int*>(p.partial), static_cast<const int*>(p.bias),
                       static_cast<const signed char*>(p.addend), p.r_off, p.r_mant, p.r_shift,
                       static_cast<signed char*>(p.y), total, p.k, plan.split_k, p.mant, p.shift,
                       p.y_off, p.lo, p.hi);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace glowmi
