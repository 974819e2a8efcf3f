// int8 FullyConnected with few rows (batch 1..64) and a reduction of a few thousand: the quantized
// form of Section 4 of the paper (int8 codes with scale/offset, int32 accumulation, rescale folded
// into the producer) for the layer that the lowering of Section 3.4 turns into MatMul + BatchedAdd.
//
// Such a layer is a few megabytes of weights and a few million multiply-accumulates: what it costs
// is latency.  Tiled over the output with the reduction split over workgroups it needs a second
// kernel to sum the partial tiles, and two dependent kernels plus their memory round trips are most
// of its time.  Here it is ONE launch with one memory round trip:
//   - a workgroup owns a strip of 32 output columns and a block of 32 rows; its eight wavefronts
//     split the reduction, up to 256 weight rows each per pass, and every wavefront issues all loads of
//     its slice at once (up to eight 16-byte loads per lane of weights, eight of activations) before
//     touching any; any K, N and alignment of the rows (FC 76x808x208 9.6 us on the tiled kernel);
//   - the weight slice [k][32 columns] goes into a private LDS region as it lies in memory, and the
//     K-contiguous MFMA fragments are read from it with the transposing load ds_read_b64_tr_b8 (within
//     16 lanes, result byte e of lane i is byte i%8 of the 8 bytes addressed by lane 2e + i/8);
//     the activation fragments (K-contiguous rows) come straight from global memory;
//   - v_mfma_i32_32x32x32_i8 with the weight fragment as the row operand: a lane ends with groups of
//     four consecutive output columns of one row; raw codes are multiplied and the offsets removed
//     afterwards with per-column / per-row code sums taken from the fragments (v_dot4);
//   - the eight partial results are summed through LDS in a fixed order, then bias, requantize,
//     clamp (Relu = lower bound), pack, one 4-byte store per group.
#include <hip/hip_runtime.h>

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

constexpr int FS_WAVES = 8;
constexpr int FS_THREADS = 64 * FS_WAVES;
constexpr int FS_COLS = 32;                      // output columns per workgroup
constexpr int FS_MAX_STEPS = 8;                  // MFMA steps (32 weight rows each) per wavefront and pass
constexpr int FS_PITCH = FS_COLS;                // bytes per staged weight row

// STEPS: 32-row MFMA steps per wavefront and pass.  The smallest number that covers the reduction in one pass, so that a
// short reduction is spread over all eight wavefronts too (FC 18x552x4072: two steps instead of three wavefronts with eight).
template <int STEPS>
__global__ __launch_bounds__(FS_THREADS, STEPS <= 4 ? 4 : 2) void fc_small_i8_kernel(const Problem p) {
  fetch_arguments(p);
  constexpr int KW = 32 * STEPS;                           // weight rows per wavefront and pass
  constexpr int WLOADS = STEPS;                            // 16-byte weight loads per lane and pass
  constexpr int REGION = KW * FS_PITCH > 4096 ? KW * FS_PITCH : 4096;   // bytes per wavefront: its weight slice, later its 4 KB of partial sums
  extern __shared__ __align__(16) unsigned char lds[];     // the wavefronts' regions, then the code sums
  int* wsum = reinterpret_cast<int*>(lds + FS_WAVES * REGION);      // [32] sum over k of W[k][n0 + c]
  int* xsum = wsum + FS_COLS;                                        // [32] sum over k of A[m][k]

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lrow = lane & 31, lhalf = lane >> 5;
  const int n0 = blockIdx.x * FS_COLS;
  const int m0 = blockIdx.y * 32;                          // first activation row of this workgroup
  const int K = p.Kgemm, N = p.k, M = p.M;
  unsigned char* region = lds + wave * REGION;

  // a 16-byte load at the end of activations of any size stays inside the 16-byte block of its last byte
  const unsigned a_size = p.x_bytes < 16u ? 16u : p.x_bytes, w_size = p.w_bytes;
  const __amdgpu_buffer_rsrc_t rsrc_a =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.x), 0, (int)a_size, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_w =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w), 0, (int)w_size, 0x00020000);

  if (tid < FS_COLS + 32) wsum[tid] = 0;                    // xsum follows wsum

  v16i acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0;
  int wacc = 0, xacc = 0;
  const bool need_xsum = p.w_off != 0;
  // K % 16 != 0: a row's last run of activations is short (the weights past K are zeros), one that would
  // run past the tensor's end is fetched from its last 16 bytes and shifted
  const bool ragged = K % 16 != 0;
  const bool at_end = ragged && (unsigned)(m0 + 32) * (unsigned)K + 15u > a_size;   // a run of this block starts in the last 15 bytes

  // Weight staging: load i of a lane covers row 32i + lane/2 of the slice, 16 columns at 16*(lane%2).
  // Fragment reads (per 16-lane group: columns 16*cb .. +15 of the strip, reduction half lhalf): lane i16
  // addresses 8 bytes of row 16*lhalf + 8u + i16/2 (u = 0, 1) at columns 16*cb + 8*(i16%2) and receives
  // the 8 codes of column 16*cb + i16 for rows 16*lhalf + 8u .. +7.
  const int srow = lane >> 1, scol = 16 * (lane & 1);
  const int i16 = lane & 15, cb = (lane >> 4) & 1;
  const unsigned frag_off = (unsigned)((16 * lhalf + (i16 >> 1)) * FS_PITCH + 16 * cb + 8 * (i16 & 1));

  const int passes = (K + FS_WAVES * KW - 1) / (FS_WAVES * KW);
  for (int pass = 0; pass < passes; ++pass) {
    const int k0 = (pass * FS_WAVES + wave) * KW;          // first weight row of this wavefront's slice
    // ---- all loads of the slice.  Rows at or past K lie past the end of the weight tensor (zeros).
    // A 16-byte run that would straddle the end of the tensor (last row of the last strip when N is
    // not a multiple of 16) is fetched from the last 16 bytes instead and shifted when it is stored.
    v4i wv[WLOADS];
    unsigned wshift = 0;                                   // 4 bits per load: bytes to shift down
#pragma unroll
    for (int i = 0; i < WLOADS; ++i) {
      const unsigned off = (unsigned)(k0 + 32 * i + srow) * (unsigned)N + (unsigned)(n0 + scol);
      const unsigned last = w_size - 16u;
      const bool straddle = off > last && off < w_size;
      wshift |= (straddle ? off - last : 0u) << (4 * i);
      wv[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, straddle ? last : off, 0, 0);
    }
    v4i av[STEPS];
    unsigned ashift = 0;
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      const int m = m0 + lrow, k = k0 + 32 * s + 16 * lhalf;
      // rows past M and codes past K: an offset past the end, the range-checked load returns zeros
      unsigned off = (m < M && k < K) ? (unsigned)m * (unsigned)K + (unsigned)k : 0x80000000u;
      if (at_end) {
        const unsigned over = off != 0x80000000u && off > a_size - 16u ? off - (a_size - 16u) : 0u;
        off -= over;
        ashift |= over << (4 * s);
      }
      av[s] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_a, off, 0, 0);
    }
    // ---- weights -> the wavefront's LDS region, as they lie in memory
#pragma unroll
    for (int i = 0; i < WLOADS; ++i) {
      v4i v = wv[i];
      const unsigned sh = (wshift >> (4 * i)) & 15u;
      if (sh) v = shift_down(v, sh);                       // rare
      *reinterpret_cast<v4i*>(region + (32 * i + srow) * FS_PITCH + scol) = v;
    }
    // (a wavefront's LDS operations execute in order: no barrier between its own writes and reads)
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      const unsigned char* q = region + 32 * s * FS_PITCH + frag_off;
      const v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((v2i __attribute__((address_space(3)))*)(q));
      const v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((v2i __attribute__((address_space(3)))*)(q + 8 * FS_PITCH));
      const v4i bw = {lo[0], lo[1], hi[0], hi[1]};         // column n0 + lrow, rows k0 + 32s + 16*lhalf .. +15
      v4i a = av[s];
      if (at_end) a = shift_down(a, (ashift >> (4 * s)) & 15u);
      if (need_xsum) {
        if (ragged) a &= byte_mask(K - (k0 + 32 * s + 16 * lhalf));
        xacc = sum_bytes(a, 0x01010101, xacc);
      }
      wacc = sum_bytes(bw, 0x01010101, wacc);
      // weight fragment as the row operand: result rows = output columns, result columns = activation rows
      acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(bw, a, acc, 0, 0, 0);
    }
  }

  // ---- code sums and partial results of the eight wavefronts -> LDS
  __syncthreads();                                         // wsum / xsum zeroed; all fragment reads done
  atomicAdd(&wsum[lrow], wacc);
  if (need_xsum) atomicAdd(&xsum[lrow], xacc);
  // [4 groups of four columns][64 lanes] of int4 per wavefront
  v4i* part = reinterpret_cast<v4i*>(region);
#pragma unroll
  for (int g = 0; g < 4; ++g) part[g * 64 + lane] = v4i{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
  __syncthreads();
  if (wave >= 4) return;

  // ---- wavefront g finishes column group g: sum the partials in wavefront order, remove the offsets
  //   sum (a - ao)(w - wo) = sum a*w - ao * sum_k w - wo * sum_k a + K * ao * wo       (modulo 2^32:
  // exact because the true value fits), add the bias, requantize, clamp, pack, store.
  // Register e of lane (lrow, lhalf) is output column n0 + (e/4)*8 + 4*lhalf + e%4 of row lrow.
  const int* bias = static_cast<const int*>(p.bias);
  const int m = m0 + lrow;
  const unsigned rowterm = (unsigned)K * (unsigned)(p.x_off * p.w_off) - (need_xsum ? (unsigned)p.w_off * (unsigned)xsum[lrow] : 0u);
  signed char* __restrict__ Y = static_cast<signed char*>(p.y);
  const int c0 = 8 * wave + 4 * lhalf;                     // first of four consecutive columns of the strip
  if (m >= M || n0 + c0 >= N) return;
  v4i v = {0, 0, 0, 0};
#pragma unroll
  for (int w = 0; w < FS_WAVES; ++w) v += reinterpret_cast<const v4i*>(lds + w * REGION)[wave * 64 + lane];
  int q[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int n = n0 + c0 + t;
    unsigned x = (unsigned)v[t] + rowterm - (unsigned)p.x_off * (unsigned)wsum[c0 + t];
    if (bias && n < N) x += (unsigned)bias[n];
    q[t] = p.shift >= 33 ? requantize_as<true>((int)x, p.mant, p.shift, p.y_off, p.lo, p.hi)
                         : requantize_as<false>((int)x, p.mant, p.shift, p.y_off, p.lo, p.hi);   // uniform
  }
  if (N % 4 == 0) {                                        // a group of four columns is wholly inside or outside
    *reinterpret_cast<unsigned*>(Y + (size_t)m * N + n0 + c0) = pack_codes(q[0], q[1], q[2], q[3]);
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (n0 + c0 + t < N) Y[(size_t)m * N + n0 + c0 + t] = (signed char)q[t];
  }
}

int fs_max_rows() {
  return knob_or(KNOB_I8_FC_SMALL_MAX_M, 64);   // the knob: experiments and tests
}

}  // namespace

bool fc_small_i8_applicable(const Problem& p) {
  if (!p.b_is_kn || p.groups != 1 || p.addend) return false;
  if (p.w_bytes < 16u || p.w_bytes > 0x7FFFFFFFu || p.x_bytes > 0x7FFFFFFFu) return false;   // rows past K must lie past the end
  // 32-bit byte offsets, also for the rows past K that the last pass addresses (and gets zeros for)
  if ((long long)(p.Kgemm + FS_WAVES * 32 * FS_MAX_STEPS) * p.k >= (1LL << 32)) return false;
  if (p.M > fs_max_rows() && knob_is_set(KNOB_I8_FC_SMALL_MAX_M)) return false;
  // rows of weights at odd byte addresses come at half the rate: several passes of them are better split over the grid
  // (9x3001x777: 8.8 us there, 12.3 here)
  if (p.k % 4 != 0 && p.Kgemm > 32 * FS_WAVES * FS_MAX_STEPS) return false;
  if (p.M <= 64) {
    if (p.Kgemm > 8192) return false;                      // longer reductions: the split kernels amortise their second launch
    // larger weight matrices are a bandwidth problem again and the tiled kernels stream them faster
    // (measured: 16 x 4096 x 4096, 16 MB, 12.6 us tiled vs 18.2 us here; 16 x 4096 x 1000, 4 MB, 10.9 vs 9.5 us)
    return p.w_bytes <= (8u << 20);
  }
  // More rows: a block of 32 rows re-reads the weights, a strip the activations, so up to three tiles per CU and 48 MB through
  // the caches in all (76x808x208 9.6 -> 4.3 us, 175x472x1088 7.1 -> 4.1, 128x2048x1000 12.7 -> 8.4 against the tiled kernel).
  // The kernel for large contractions takes such calls where rows come in sixteens; where they only come in fours this one is the
  // faster (196x2360x344 7.7 us, 11.3 there; of 90 such calls of 96 to 1000 rows all but seven, 0.80 of the time at the median).
  if (wide_i8_applicable(p) && p.Kgemm % 16 == 0 && p.k % 16 == 0 && p.M >= 96 && p.k >= 128 && p.Kgemm >= 1536) return false;
  const long long tiles = (long long)((p.M + 31) / 32) * ((p.k + FS_COLS - 1) / FS_COLS);
  return p.Kgemm <= 4096 && tiles <= 768 && tiles * p.Kgemm * 64 <= (48LL << 20);
}

template <int STEPS>
hipError_t launch_fs(const Problem& p, hipStream_t stream) {
  constexpr int region = 32 * STEPS * FS_PITCH > 4096 ? 32 * STEPS * FS_PITCH : 4096;
  constexpr int lds_bytes = FS_WAVES * region + (FS_COLS + 32) * (int)sizeof(int);
  // once per instantiation; initialisation of a function-local static is thread-safe
  static const hipError_t attr_status = hipFuncSetAttribute(
      reinterpret_cast<const void*>(fc_small_i8_kernel<STEPS>), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
  if (attr_status != hipSuccess) return attr_status;
  // one workgroup per strip of 32 columns and block of 32 rows (measured with 64 rows: both row blocks
  // in one workgroup 10.5 us, in two workgroups 8.8 us: twice the workgroups in flight, half the loads
  // per lane)
  dim3 grid((unsigned)((p.k + FS_COLS - 1) / FS_COLS), (unsigned)((p.M + 31) / 32), 1), block(FS_THREADS, 1, 1);
  hipLaunchKernelGGL(fc_small_i8_kernel<STEPS>, grid, block, lds_bytes, stream, p);
  return hipGetLastError();
}

hipError_t launch_fc_small_i8(const Problem& p, hipStream_t stream, const char** variant) {
  *variant = p.M <= 64 && p.Kgemm % 16 == 0 && p.k % 4 == 0 ? "fc_small_i8" : "fc_strip_i8";   // strip: ragged sizes, more rows
  const int steps = (p.Kgemm + 32 * FS_WAVES - 1) / (32 * FS_WAVES);
  if (steps <= 1) return launch_fs<1>(p, stream);
  if (steps <= 2) return launch_fs<2>(p, stream);
  if (steps <= 4) return launch_fs<4>(p, stream);
  return launch_fs<FS_MAX_STEPS>(p, stream);
}

}  // namespace glowmi
