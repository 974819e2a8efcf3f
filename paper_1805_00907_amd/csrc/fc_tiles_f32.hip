// fp32 FullyConnected with some dozens to some hundreds of rows on the fp16 matrix cores, in one launch: y = x w (+ bias,
// Relu), x [M][K], w [K][N].  (The fp16-piece products and their scales: f16_pieces.h.)
//
// The kernels over packed planes pay launches and passes over both operands before they multiply, the fp32 matrix cores
// multiply at 60 TFLOP/s; in between lie the classifier layers of a batch.  Here both operands are cut on the way from
// memory to the matrix cores:
//   - a workgroup owns 64 (32) rows and 64 columns; its eight wavefronts take every eighth chunk of 16 reduction indices,
//     each the whole tile, so that no value is fetched twice in a workgroup and the loop has no barrier;
//   - the columns of w lie side by side in memory: lane (column, half) loads its eight indices of a column one by one, 128
//     bytes of a row of w at a time, and the cut values are the matrix operand as they are;
//   - x arrives as 64 bytes of 16 rows per load and goes, cut, through 4 KB of LDS of the wavefront's own (fetched in the
//     operand's own layout, 32 bytes of 32 rows at a time, it comes at a quarter of the rate);
//   - a wavefront scales either operand by the largest magnitude it has seen; values that outgrow it scale the sums down;
//   - every eight chunks the accumulators of the h1 h1' products are folded into sums in LDS.  One chain of rounded additions
//     per output and wavefront was less exact than the contraction over planes at deep reductions (256x9216x4096 2.4e-7 of
//     the result's norm against 1.7e-7, now 1.4e-7); it costs 4 to 7 % from 2000 indices on, most of it LDS traffic;
//   - at the end the wavefronts exchange their sums through LDS and finish an eighth of the tile each.
// Bound by the vector unit (the cuts: 32 values a lane and chunk) and the 64 bytes a clock of a CU's memory path, closely
// followed by the matrix cores.  Measured: 256x4096x4096 52 us, 1000x1024x512 12.3, 150x301x77 6.5 (82, 21, 13 on the kernels
// over planes and on the fp32 matrix cores).
// Few tiles: the reduction is also split over the grid, and the partial sums go through the workspace.
#include <hip/hip_runtime.h>

#include "arguments.h"
#include "f16_pieces.h"
#include "igemm.h"
#include "lds_direct.h"

namespace glowmi {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

constexpr int FT_WAVES = 8, FT_COLS = 64, FT_CHUNK = 16, FT_FOLD = 8;   // FT_FOLD: chunks of a wavefront between folds, even
constexpr unsigned FT_OOB = 0x80000000u;                 // operands are smaller: whatever is added or set below, past the end

__device__ __forceinline__ void cut4_in_place(const v4f& x, int se, v2u& p1, v2u& p2) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const v2f v = {__builtin_ldexpf(x[2 * i], se), __builtin_ldexpf(x[2 * i + 1], se)};
    const v2h h1 = __builtin_convertvector(v, v2h);
    const v2h h2 = {(_Float16)__builtin_fmaf((float)h1[0], -2048.f, v[0] * 2048.f),
                    (_Float16)__builtin_fmaf((float)h1[1], -2048.f, v[1] * 2048.f)};
    p1[i] = __builtin_bit_cast(unsigned, h1);
    p2[i] = __builtin_bit_cast(unsigned, h2);
  }
}

// Scale of one operand of a wavefront: for magnitudes up to `limit` (bits).
struct RunningScale {
  int se = 140;
  unsigned limit = 0x00ffffffu;
  __device__ __forceinline__ bool fits(unsigned lane_max) const { return lane_max <= limit; }
  __device__ __forceinline__ void grow(unsigned max_bits) {
    if (max_bits <= limit) return;
    se = scale_exponent(max_bits);
    limit = max_bits | 0x007fffffu;
  }
};

template <int MB>
__global__ __launch_bounds__(64 * FT_WAVES, 2) void fc_tiles_f32_kernel(const Problem p, const FastDiv tiles_m, const FastDiv tiles_n, int total, int chunks,
                                                                        int chunks_per_split) {
  fetch_arguments(p, tiles_m, tiles_n, total, chunks, chunks_per_split);
  constexpr int ROWS = 32 * MB, LOADS = ROWS / 16;
  constexpr int PLANE = ROWS * 32;                       // bytes of a plane of a wavefront's chunk of x
  extern __shared__ __align__(16) unsigned char lds[];

  // consecutive tiles, the row tiles of a column strip first, on one XCD: its L2 serves the strip to all of them
  const int per_xcd = (int)(gridDim.x >> 3);
  int tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  if (tile >= total) return;
  const int strips = tiles_m.div(tile), tm = tile - strips * (int)tiles_m.d;
  const int split = tiles_n.div(strips), tn = strips - split * (int)tiles_n.d;
  const int tid = threadIdx.x, lane = tid & 63, lrow = lane & 31, lhalf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = p.Kgemm, N = p.k;
  const int first = split * chunks_per_split;
  const int end = first + chunks_per_split < chunks ? first + chunks_per_split : chunks;

  const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.x), 0, (int)p.x_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w), 0, (int)p.w_bytes, 0x00020000);

  // rows past the last one lie past the end of x
  const unsigned x_at = (unsigned)(tm * ROWS + (lane >> 2)) * (unsigned)K * 4u + 16u * (lane & 3);
  // (the second 32 columns of a tile may not be there: what they load then is never stored)
  const int col0 = tn * FT_COLS + lrow;
  const unsigned w_at = (col0 < N ? (unsigned)col0 * 4u : FT_OOB) + (unsigned)(8 * lhalf) * (unsigned)N * 4u;
  v4f raw_x[2][LOADS];
  float raw_w[2][2][8];
  // rows of w past the last one lie past its end; past the last index of a row of x lies the next row (masked below)
  auto load = [&](int set, int chunk) {
    const unsigned dead = chunk < end ? 0u : FT_OOB;     // uniform
    const unsigned k0 = (unsigned)chunk * FT_CHUNK;
    // (opaque: the compiler would otherwise carry a register through the loop for every load)
    unsigned xa = (x_at + 4u * k0) | dead, at = (w_at + k0 * (unsigned)N * 4u) | dead;
    asm("" : "+v"(xa), "+v"(at));
#pragma unroll
    for (int j = 0; j < LOADS; ++j)
      raw_x[set][j] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, xa + (unsigned)(16 * j) * (unsigned)K * 4u, 0, 0));
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const unsigned row = at + (unsigned)i * (unsigned)N * 4u;
      raw_w[set][0][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc_w, row, 0, 0));
      raw_w[set][1][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc_w, row + 128u, 0, 0));
    }
  };

  v16f acc[MB][2], acc_lo[MB][2];                        // the h1 h1' products; the cross terms (weight 2^-11)
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        acc[a][b][e] = 0.f;
        acc_lo[a][b][e] = 0.f;
      }
  RunningScale sx, sw;
  bool finite = true;

  unsigned char* mine = lds + wave * 2 * PLANE;
  unsigned char* put = mine + (lane >> 2) * 32 + (lane & 3) * 8;
  const unsigned char* get = mine + lrow * 32 + lhalf * 16;
  auto multiply = [&](int set, int chunk) {
    v4f (&x)[LOADS] = raw_x[set];
    float (&w)[2][8] = raw_w[set];
    if ((chunk + 1) * FT_CHUNK > K) {                    // uniform: the last chunk, ragged
      const int left = K - chunk * FT_CHUNK - 4 * (lane & 3);
#pragma unroll
      for (int j = 0; j < LOADS; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) x[j][e] = e < left ? x[j][e] : 0.f;
    }
    float mx = 0.f, mw = 0.f;
#pragma unroll
    for (int j = 0; j < LOADS; ++j)
#pragma unroll
      for (int e = 0; e < 4; e += 2) asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(mx) : "v"(x[j][e]), "v"(x[j][e + 1]));
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 8; e += 2) asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(mw) : "v"(w[b][e]), "v"(w[b][e + 1]));
    const unsigned bx = __builtin_bit_cast(unsigned, mx) & 0x7fffffffu, bw = __builtin_bit_cast(unsigned, mw) & 0x7fffffffu;
    if (__builtin_amdgcn_ballot_w64(!sx.fits(bx) || !sw.fits(bw)) != 0) {
      const int before = sx.se + sw.se;
      const unsigned ax = wave_max_u32(bx), aw = wave_max_u32(bw);
      finite = finite && ax < 0x7f800000u && aw < 0x7f800000u;
      sx.grow(ax);
      sw.grow(aw);
      const int by = sx.se + sw.se - before;
#pragma unroll
      for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            acc[a][b][e] = __builtin_ldexpf(acc[a][b][e], by);
            acc_lo[a][b][e] = __builtin_ldexpf(acc_lo[a][b][e], by);
          }
    }
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
      v2u p1, p2;
      cut4_in_place(x[j], sx.se, p1, p2);
      *reinterpret_cast<v2u*>(put + j * 512) = p1;
      *reinterpret_cast<v2u*>(put + PLANE + j * 512) = p2;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the wavefront's own LDS, in order
    __builtin_amdgcn_wave_barrier();
    v8h x1[MB], x2[MB];
#pragma unroll
    for (int a = 0; a < MB; ++a) {
      x1[a] = __builtin_bit_cast(v8h, *reinterpret_cast<const v4u*>(get + a * 1024));
      x2[a] = __builtin_bit_cast(v8h, *reinterpret_cast<const v4u*>(get + PLANE + a * 1024));
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      v4u c1, c2;
      cut8_in_place(w[b], sw.se, c1, c2);
      const v8h w1 = __builtin_bit_cast(v8h, c1), w2 = __builtin_bit_cast(v8h, c2);
      __builtin_amdgcn_sched_barrier(0);
      if (b == 1) load(set, chunk + 2 * FT_WAVES);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int a = 0; a < MB; ++a) acc_lo[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x1[a], w2, acc_lo[a][b], 0, 0, 0);
#pragma unroll
      for (int a = 0; a < MB; ++a) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x1[a], w1, acc[a][b], 0, 0, 0);
#pragma unroll
      for (int a = 0; a < MB; ++a) acc_lo[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x2[a], w1, acc_lo[a][b], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // Sums of short runs round less: every FT_FOLD chunks acc goes into LDS of the wavefront's own, at the scale of that moment.
  constexpr int NQ = MB * 8;                             // quads of registers of the tile
  v4f* const kept = reinterpret_cast<v4f*>(lds + FT_WAVES * 2 * PLANE) + wave * NQ * 64 + lane;
  // (Every sixteen: 3 % faster, but 6 to 9 % further from 64-bit sums than the contraction over planes at 1500 to 2200
  // indices.  Left to the LDS to add, ds_add_f32: three times the time of the call.)
  int kept_se = 0, since_fold = 0;
  bool any_kept = false;                                 // uniform, as the two above
  auto add_kept = [&] {                                  // brought to the present scale
    const int by = sx.se + sw.se - kept_se;
#pragma unroll
    for (int q = 0; q < NQ; q += 4) {                    // four reads in flight
      v4f v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = kept[(q + i) * 64];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc[(q + i) / 8][(q + i) / 4 % 2][(q + i) % 4 * 4 + e] += __builtin_ldexpf(v[i][e], by);
    }
  };

  int chunk = first + wave;
  load(0, chunk);
  load(1, chunk + FT_WAVES);
  // in pairs; the one after the last is all zeros
  do {
    if (since_fold == FT_FOLD) {
      if (any_kept) add_kept();
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        v4f v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = acc[q / 8][q / 4 % 2][q % 4 * 4 + e];
          acc[q / 8][q / 4 % 2][q % 4 * 4 + e] = 0.f;
        }
        kept[q * 64] = v;
      }
      kept_se = sx.se + sw.se;
      since_fold = 0;
      any_kept = true;
    }
    since_fold += 2;
    multiply(0, chunk);
    multiply(1, chunk + FT_WAVES);
    chunk += 2 * FT_WAVES;
  } while (chunk < end);

  // ---- the wavefronts swap their sums: each finishes OQ of the tile's NQ quads of registers.  Register e of a block is row
  // (e/4)*8 + 4*lhalf + e%4 of its 32, column lane % 32.
  constexpr int OQ = NQ / FT_WAVES;
  if (any_kept) add_kept();
  const ScaleBack sb = scale_back_of(sx.se, sw.se, finite);
  v4f* xch = reinterpret_cast<v4f*>(lds);
  float res[OQ][4];
  __syncthreads();                                       // everyone is done with the planes
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    v4f send;
#pragma unroll
    for (int e = 0; e < 4; ++e) send[e] = join_sets(acc[q / 8][q / 4 % 2][q % 4 * 4 + e], acc_lo[q / 8][q / 4 % 2][q % 4 * 4 + e], sb);
    if (q / OQ != wave) xch[(wave * NQ + q) * 64 + lane] = send;
    else {
#pragma unroll
      for (int e = 0; e < 4; ++e) res[q % OQ][e] = send[e];
    }
  }
  __syncthreads();
#pragma unroll
  for (int d = 1; d < FT_WAVES; ++d) {
    const int from = (wave + d) % FT_WAVES;
#pragma unroll
    for (int q = 0; q < OQ; ++q) {
      const v4f got = xch[(from * NQ + wave * OQ + q) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) res[q][e] += got[e];
    }
  }
  const unsigned y_bytes = (unsigned)p.M * (unsigned)N * 4u;
  const bool partial = p.split_k > 1;                    // uniform
  float* out = partial ? static_cast<float*>(p.partial) + (size_t)split * p.M * N : static_cast<float*>(p.y);
  const __amdgpu_buffer_rsrc_t rsrc_y = __builtin_amdgcn_make_buffer_rsrc(out, 0, (int)y_bytes, 0x00020000);
  const float* __restrict__ bias = static_cast<const float*>(p.bias);
  const bool act = p.act == 1 && !partial;
#pragma unroll
  for (int q = 0; q < OQ; ++q) {
    const int quad = wave * OQ + q;
    const int row = tm * ROWS + (quad >> 3) * 32 + (quad & 3) * 8 + lhalf * 4;
    const int col = tn * FT_COLS + (quad >> 2 & 1) * 32 + lrow;
    const float bv = bias && !partial && col < N ? bias[col] : 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float v = res[q][e] + bv;
      if (act) v = clamp_act(v, p.act_lo, p.act_hi);
      const unsigned off = row + e < p.M && col < N ? ((unsigned)(row + e) * (unsigned)N + (unsigned)col) * 4u : FT_OOB;
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), rsrc_y, off, 0, 0);
    }
  }
}

template <int MB>
hipError_t launch_ft(const Problem& p, const Plan& plan, hipStream_t stream) {
  constexpr int lds_bytes = FT_WAVES * MB * (2 * 32 * 32 + 8 * 64 * 16);   // the planes of x, the folded sums (then the exchange)
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(fc_tiles_f32_kernel<MB>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
  if (attr != hipSuccess) return attr;
  const int total = plan.tiles_m * plan.tiles_n * plan.split_k;
  hipLaunchKernelGGL(fc_tiles_f32_kernel<MB>, dim3((unsigned)((total + 7) / 8 * 8)), dim3(64 * FT_WAVES), lds_bytes, stream, p,
                     make_fastdiv((uint32_t)plan.tiles_m), make_fastdiv((uint32_t)plan.tiles_n), total, plan.slabs, plan.slabs_per_split);
  return hipGetLastError();
}

}  // namespace

// The tiles and the split of the reduction for a FullyConnected, and its time; false: not a layer for this kernel.
bool plan_fc_tiles_f32(const Problem& p, bool allow_split, Plan* plan, double* us) {
  const int mode = knob_or(KNOB_F32_FC_TILES, 1);        // 0: off, 2: any size, 3, 4: any size, 32 or 64 rows (tests, experiments)
  if (mode == 0 || !p.b_is_kn || p.groups != 1 || p.addend || p.chain_n > 0) return false;
  if (p.x_bytes > (1u << 30) || p.w_bytes > (1u << 30) || (long long)p.M * p.k * 4 > (1LL << 30)) return false;   // 31-bit offsets
  if (p.k > (1 << 18) || p.Kgemm > (1 << 22)) return false;   // loads past the end stay below 2^32
  double best = 0.0;
  const int chunks = (p.Kgemm + FT_CHUNK - 1) / FT_CHUNK;
  for (int mb = 1; mb <= 2; ++mb) {
    if (mode >= 3 && mb != mode - 2) continue;
    const int tm = (p.M + 32 * mb - 1) / (32 * mb), tn = (p.k + FT_COLS - 1) / FT_COLS;
    const long long tiles = (long long)tm * tn;
    if (tiles > (1 << 24)) continue;
    for (int split = 1; split <= 64; ++split) {
      if (split > 1 && (!allow_split || tiles * split > 512 || chunks / split < 2 * FT_WAVES)) break;
      if (knob_is_set(KNOB_F32_FC_TILES_SPLIT) && allow_split && split != knob(KNOB_F32_FC_TILES_SPLIT)) continue;
      const int per = (chunks + split - 1) / split;
      if ((chunks + per - 1) / per != split) continue;
      // measured; a trip of the eight wavefronts takes longer when every CU is at it, and trips come in pairs
      const double rounds = (double)((tiles * split + 255) / 256), fill = (double)(tiles * split) / (256.0 * rounds);
      const int trips = (per + 2 * FT_WAVES - 1) / (2 * FT_WAVES) * 2;
      const double t = (mb == 2 ? 4.2 : 3.4) + 1.5 * fill + (rounds - 1.0) * (mb == 2 ? 2.0 : 1.5) +
                       rounds * trips * (mb == 2 ? 1.03 + 0.27 * fill : 0.78 + 0.15 * fill) +
                       (split > 1 ? 1.6 + 0.8e-6 * 4.0 * p.M * p.k * split : 0.0);
      if (best > 0.0 && t >= best) continue;
      best = t;
      plan->kernel = KERNEL_FC_TILES;
      plan->bm = 32 * mb;
      plan->bn = FT_COLS;
      plan->bk = FT_CHUNK;
      plan->tiles_m = tm;
      plan->tiles_n = tn;
      plan->slabs = chunks;
      plan->split_k = split;
      plan->slabs_per_split = per;
      plan->pack_bytes = 0;
    }
  }
  *us = best;
  return best > 0.0;
}

hipError_t launch_fc_tiles_f32(const Problem& p, const Plan& plan, hipStream_t stream, const char** variant) {
  *variant = plan.bm == 64 ? "fc_tiles_f32_64x64" : "fc_tiles_f32_32x64";
  return plan.bm == 64 ? launch_ft<2>(p, plan, stream) : launch_ft<1>(p, plan, stream);
}

}  // namespace glowmi
