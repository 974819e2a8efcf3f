// fp32 FullyConnected with few rows (batch 1..64) in ONE launch with one pass over the weights.
//
// Section 3.4 of the paper lowers FullyConnected to a matrix multiplication followed by a broadcasted
// add; with a handful of rows the layer is a stream of the weight matrix through the chip, and what it
// costs beyond that stream is latency: kernels that follow each other on a stream, and dependent
// memory round trips inside a kernel.  The tiled kernels split the reduction over workgroups and
// finish in a second kernel; here a column strip of the output is owned by one workgroup and the
// reduction is split over its sixteen wavefronts instead, summed through LDS in a fixed order:
//
//   - workgroup = (strip of 16 * VW output columns, block of 16 rows); strips narrow enough that a
//     matrix with N = 1000..4096 columns still gives every CU (or at least a quarter of them, which is
//     enough L2 -> CU bandwidth for a few megabytes) a workgroup.  Neighbouring strips read the two
//     halves of the same cache lines; consecutive strips go to the same XCD, so the second reader finds
//     the line in that XCD's L2;
//   - a wavefront owns a contiguous range of 16-row steps of the reduction.  Lane (c, q) loads
//     W[k0 + 4q + t][n0 + VW c ..] for t = 0..3 straight into MFMA operand layout (no LDS staging) and
//     the float4 A[row c][k0 + 4q ..]; v_mfma_f32_16x16x4_f32 (t, j) multiplies reduction index
//     k0 + 4q + t into column n0 + VW c + j.  Loads run a chunk of steps ahead of the MFMAs in a second
//     register set, so a wavefront pays one memory latency, not one per step;
//   - every load is a range-checked buffer load: rows past K, columns past N and rows past M read zeros,
//     so ragged shapes need no branches;
//   - the sixteen partial results are summed through LDS in wavefront order (deterministic), then
//     bias + activation, one store.
#include <hip/hip_runtime.h>

#include "arguments.h"
#include "igemm.h"

namespace glowmi {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));

constexpr int FSF_WAVES = 16;
constexpr int FSF_THREADS = 64 * FSF_WAVES;
constexpr int FSF_STEP = 16;                 // reduction indices per step

template <int VW> struct VecOf;
template <> struct VecOf<1> { typedef float type; };
template <> struct VecOf<2> { typedef v2f type; };
template <> struct VecOf<4> { typedef v4f type; };

template <int VW>
__device__ __forceinline__ typename VecOf<VW>::type load_w(__amdgpu_buffer_rsrc_t rsrc, unsigned off) {
  if constexpr (VW == 1) return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, off, 0, 0));
  else if constexpr (VW == 2) return __builtin_bit_cast(v2f, __builtin_amdgcn_raw_buffer_load_b64(rsrc, off, 0, 0));
  else return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0));
}

template <int VW>
__device__ __forceinline__ float elem(const typename VecOf<VW>::type& v, int j) {
  if constexpr (VW == 1) return v;
  else return v[j];
}

template <int VW>
__global__ __launch_bounds__(FSF_THREADS) void fc_small_f32_kernel(const Problem p, int strips, int steps_per_wave) {
  fetch_arguments(p, strips, steps_per_wave);
  constexpr int U = 4 / VW < 1 ? 1 : 4 / VW;       // steps per chunk: 16 weight registers per set
  constexpr int COLS = 16 * VW;
  typedef typename VecOf<VW>::type wvec;
  __shared__ float red[FSF_WAVES * VW * 4 * 64];

  // consecutive strips on one XCD (workgroup ids go round-robin over the 8 XCDs)
  const int per_xcd = gridDim.x >> 3;
  const int strip = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (strip >= strips) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = lane & 15, q = lane >> 4;
  const int n0 = strip * COLS;
  const int m0 = blockIdx.y * 16;
  const int K = p.Kgemm, N = p.k, M = p.M;

  const __amdgpu_buffer_rsrc_t rsrc_w =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w), 0, (int)p.w_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_a =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.x), 0, (int)p.x_bytes, 0x00020000);
  constexpr unsigned OOB = 0xFFFFFF00u;            // beyond any tensor this library accepts

  const int col = n0 + c * VW;
  const bool col_ok = col < N;                     // N % VW == 0: the whole vector is inside or outside
  const bool row_ok = m0 + c < M;                  // as the A operand lane c holds activation row m0 + c
  const unsigned a_row = (unsigned)(m0 + c) * (unsigned)K;

  const int s_begin = wave * steps_per_wave;
  int s_end = s_begin + steps_per_wave;
  const int total_steps = (K + FSF_STEP - 1) / FSF_STEP;
  if (s_end > total_steps) s_end = total_steps;

  v4f acc[VW];
#pragma unroll
  for (int j = 0; j < VW; ++j) acc[j] = v4f{0.f, 0.f, 0.f, 0.f};

  v4f a0[U], a1[U];
  wvec b0[U][4], b1[U][4];
  auto load_chunk = [&](int s0, v4f (&a)[U], wvec (&b)[U][4]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k0 = (s0 + u) * FSF_STEP + 4 * q;            // K % 4 == 0: the lane's four indices are in or out together
      const bool kok = s0 + u < s_end && k0 < K;
      const unsigned aoff = (kok && row_ok) ? (a_row + (unsigned)k0) * 4u : OOB;
      a[u] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rsrc_a, aoff, 0, 0));
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const unsigned woff = (kok && col_ok) ? ((unsigned)(k0 + t) * (unsigned)N + (unsigned)col) * 4u : OOB;
        b[u][t] = load_w<VW>(rsrc_w, woff);
      }
    }
  };
  auto mma_chunk = [&](const v4f (&a)[U], const wvec (&b)[U][4]) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int j = 0; j < VW; ++j)
          acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][t], elem<VW>(b[u][t], j), acc[j], 0, 0, 0);
  };

  // Two register sets: the loads of the next chunk are in flight while this one is multiplied.  The
  // loads are issued unconditionally (steps past the wavefront's range get the out-of-range offset and
  // cost no memory traffic): a load inside a branch would make the compiler wait for every outstanding
  // load at the join, which serialises the two sets.
  load_chunk(s_begin, a0, b0);
  for (int s = s_begin; s < s_end; s += 2 * U) {
    load_chunk(s + U, a1, b1);
    mma_chunk(a0, b0);
    load_chunk(s + 2 * U, a0, b0);
    mma_chunk(a1, b1);
  }

  // ---- partial results -> LDS; summed in wavefront order by the first VW * 256 threads
#pragma unroll
  for (int j = 0; j < VW; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) red[((wave * VW + j) * 4 + e) * 64 + lane] = acc[j][e];
  __syncthreads();
  const int tid = threadIdx.x;
  if (tid >= VW * 256) return;
  const int idx = tid >> 6;                        // j * 4 + e
  const int j = idx >> 2, e = idx & 3;
  float v = 0.f;
#pragma unroll
  for (int w = 0; w < FSF_WAVES; ++w) v += red[((w * VW + j) * 4 + e) * 64 + lane];
  // 16 x 16 result: register e of lane (c, q) is row 4q + e, column slot c = column n0 + VW c + j
  const int row = m0 + 4 * q + e, ocol = n0 + c * VW + j;
  if (row >= M || ocol >= N) return;
  const float* __restrict__ bias = static_cast<const float*>(p.bias);
  if (bias) v += bias[ocol];
  if (p.act == 1) v = fmaxf(v, 0.f);
  static_cast<float*>(p.y)[(size_t)row * N + ocol] = v;
}

// ---- one to four rows on the vector units, the whole reduction of a strip of columns in one workgroup, any K and N.
//
// At these sizes a call is a latency, and the kernel that streams the matrix through every CU needs a second one for its
// partial sums.  Here a workgroup of sixteen wavefronts owns 4 LPR columns: LPR lanes of four columns, 1024 / LPR rows at a
// time, eight of those in flight.  The row's values come through LDS; the lanes' sums meet by lane permutations and then
// through LDS in wavefront order (deterministic).  A CU takes in 16 lines of 64 bytes as slowly as 16 whole ones, so strips
// are as wide as eight rows in flight per lane cover the reduction, and a matrix of some megabytes is better off on every CU:
// 1 x 512 x 1000 5.4 us streamed, 4.2 here; 1 x 2048 x 1000 7.2 both; 2 x 2048 x 1000 7.4 and 8.7.  Rows that do not start
// on 16 bytes, which the other kernels fetch value by value: 1 x 500 x 130 11.3 -> 4.2, 3 x 1536 x 777 12.5 -> 10.2.
constexpr int FR_THREADS = 1024;
constexpr int FR_DEPTH = 8;                  // rows of a lane in flight

template <int MR, int LPR>
__global__ __launch_bounds__(FR_THREADS) void fc_rows_f32_kernel(const Problem p, int strips) {
  fetch_arguments(p, strips);
  constexpr int ROWS = FR_THREADS / LPR;           // weight rows per pass
  constexpr int COLS = 4 * LPR;
  __shared__ float red[16 * MR * COLS];
  extern __shared__ float xs[];                    // [MR][passes * ROWS]

  const int per_xcd = gridDim.x >> 3;              // consecutive strips share lines: one XCD
  const int strip = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  if (strip >= strips) return;
  const int tid = threadIdx.x;
  const int quad = tid % LPR, row0 = tid / LPR;
  const int K = p.Kgemm, N = p.k;
  const __amdgpu_buffer_rsrc_t rsrc_w =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w), 0, (int)p.w_bytes, 0x00020000);
  constexpr unsigned OOB = 0xFFFFFF00u;
  const int col = strip * COLS + 4 * quad;
  const unsigned first = ((unsigned)row0 * (unsigned)N + (unsigned)col) * 4u;
  const unsigned pass_step = (unsigned)ROWS * (unsigned)N * 4u;
  const int passes = (K + ROWS - 1) / ROWS;
  auto load = [&](int pass) {                      // rows past the last one read zeros; columns past it are not stored
    const unsigned off = col < N && row0 + pass * ROWS < K ? first + (unsigned)pass * pass_step : OOB;
    return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, off, 0, 0));
  };
  v4f w[FR_DEPTH];
#pragma unroll
  for (int d = 0; d < FR_DEPTH; ++d) w[d] = load(d);
  const float* __restrict__ x = static_cast<const float*>(p.x);
  const int kpad = passes * ROWS;
#pragma unroll
  for (int m = 0; m < MR; ++m)
    for (int k = tid; k < kpad; k += FR_THREADS) xs[m * kpad + k] = m < p.M && k < K ? x[(size_t)m * K + k] : 0.f;
  __syncthreads();
  v4f acc[MR];
#pragma unroll
  for (int m = 0; m < MR; ++m) acc[m] = v4f{0.f, 0.f, 0.f, 0.f};
  for (int pass = 0; pass < passes; pass += FR_DEPTH) {
#pragma unroll
    for (int d = 0; d < FR_DEPTH; ++d) {
      const v4f v = w[d];
      w[d] = load(pass + d + FR_DEPTH);            // past the end: no memory traffic
      const int k = row0 + (pass + d < passes ? pass + d : 0) * ROWS;
#pragma unroll
      for (int m = 0; m < MR; ++m) {
        const float xv = xs[m * kpad + k];         // past the last pass the weights are zeros
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[m][j] = __builtin_fmaf(xv, v[j], acc[m][j]);
      }
    }
  }
  const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int m = 0; m < MR; ++m)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float s = acc[m][j];
#pragma unroll
      for (int d = 32; d >= LPR; d >>= 1) s += __shfl_xor(s, d, 64);
      if (lane < LPR) red[(wave * MR + m) * COLS + 4 * lane + j] = s;
    }
  __syncthreads();
  if (tid >= MR * COLS) return;
  const int m = tid / COLS, ocol = strip * COLS + tid % COLS;
  if (m >= p.M || ocol >= N) return;
  float v = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) v += red[(i * MR) * COLS + tid];
  const float* __restrict__ bias = static_cast<const float*>(p.bias);
  if (bias) v += bias[ocol];
  if (p.act == 1) v = fmaxf(v, 0.f);
  static_cast<float*>(p.y)[(size_t)m * N + ocol] = v;
}

template <int MR, int LPR>
hipError_t launch_rows_variant(const Problem& p, hipStream_t stream) {
  constexpr int ROWS = FR_THREADS / LPR;
  const int strips = (p.k + 4 * LPR - 1) / (4 * LPR);
  const size_t lds = (size_t)MR * ((p.Kgemm + ROWS - 1) / ROWS * ROWS) * sizeof(float);
  hipLaunchKernelGGL((fc_rows_f32_kernel<MR, LPR>), dim3((unsigned)((strips + 7) / 8 * 8)), dim3(FR_THREADS), lds, stream, p, strips);
  return hipGetLastError();
}

template <int MR>
hipError_t launch_rows(const Problem& p, int lanes, hipStream_t stream) {
  switch (lanes) {
    case 4: return launch_rows_variant<MR, 4>(p, stream);
    case 8: return launch_rows_variant<MR, 8>(p, stream);
    default: return launch_rows_variant<MR, 16>(p, stream);
  }
}

template <int VW>
hipError_t launch_fsf(const Problem& p, hipStream_t stream) {
  constexpr int COLS = 16 * VW;
  const int strips = (p.k + COLS - 1) / COLS;
  const int total_steps = (p.Kgemm + FSF_STEP - 1) / FSF_STEP;
  const int steps_per_wave = (total_steps + FSF_WAVES - 1) / FSF_WAVES;
  dim3 grid((unsigned)(((strips + 7) / 8) * 8), (unsigned)((p.M + 15) / 16), 1), block(FSF_THREADS, 1, 1);
  hipLaunchKernelGGL(fc_small_f32_kernel<VW>, grid, block, 0, stream, p, strips, steps_per_wave);
  return hipGetLastError();
}

// Strip width in units of 16 columns: the widest loads that still give about three quarters of the CUs
// a workgroup (wider strips read whole cache lines per row; narrower ones reach more CUs).
int width_of(const Problem& p) {
  const int forced = knob_or(KNOB_F32_FC_SMALL_VW, 0);
  if ((forced == 4 && p.k % 4 == 0) || (forced == 2 && p.k % 2 == 0) || forced == 1) return forced;
  const int row_blocks = (p.M + 15) / 16;
  if (p.k % 4 == 0 && (long long)((p.k + 63) / 64) * row_blocks >= 192) return 4;
  if (p.k % 2 == 0 && (long long)((p.k + 31) / 32) * row_blocks >= 192) return 2;
  return 1;
}

}  // namespace

int fc_small_f32_width(const Problem& p) { return width_of(p); }

bool fc_small_f32_applicable(const Problem& p) {
  if (!p.b_is_kn || p.groups != 1 || p.addend || p.chain_n > 0) return false;
  if (knob_or(KNOB_F32_FC_SMALL_OFF, 0) != 0) return false;
  if (p.M > 64 || p.Kgemm % 4 != 0 || p.Kgemm < 64) return false;
  // One workgroup per column strip pulls its strip of the matrix at the rate ONE CU sustains from
  // memory: about 45 GB/s when the weights are resident in the last-level cache and a third of that
  // when they come from HBM.  Measured per launch, (rows x K x N): launched back to back on warm weights
  // 1 x 2048 x 1000 8.4 us here vs 11.3 us for the weight-streaming kernel + finishing kernel,
  // 64 x 2048 x 1000 9.5 vs 13.0 us (tiled), 16 x 4096 x 1000 14.5 vs 10.6 us; with the weights cold (other
  // layers in between) 1 x 2048 x 1000 13.1 vs 10.8 us, 64 x 2048 x 1000 15.5 vs 15.0 us.  So up to 16 rows
  // the streaming kernel, which spreads the matrix over every CU, stays the planner's choice (the knob
  // F32_FC_SMALL_MIN_M lowers the bound for tests and experiments); with 17 to 64 rows this kernel
  // replaces the tiled one for matrices of a few megabytes.
  if (p.M < knob_or(KNOB_F32_FC_SMALL_MIN_M, 17)) return false;
  const long long max_kb = knob_or(KNOB_F32_FC_SMALL_MAX_KB, 8704);      // the knob: experiments and tests
  if ((long long)p.w_bytes > (max_kb << 10) || p.w_bytes > 0x7FFFFFFFu || p.x_bytes > 0x7FFFFFFFu) return false;
  return true;
}

bool fc_rows_f32_applicable(const Problem& p) {
  if (!p.b_is_kn || p.groups != 1 || p.addend || p.chain_n > 0 || p.M > 4 || p.Kgemm > 8192) return false;
  const int mode = knob_or(KNOB_F32_FC_ROWS, 1);         // 0: off, 2: any size (tests)
  if (mode == 0 || knob_is_set(KNOB_F32_FC_SMALL_MIN_M)) return false;
  if (mode == 2) return true;
  if (p.k % 4 != 0 || p.Kgemm % 4 != 0) return p.w_bytes <= (16u << 20);
  return p.M == 1 && p.Kgemm > 128 && p.Kgemm <= 2048 && p.w_bytes <= (4u << 20);
}

hipError_t launch_fc_rows_f32(const Problem& p, hipStream_t stream, const char** variant) {
  const int lanes = p.Kgemm <= 512 ? 16 : p.Kgemm <= 1024 ? 8 : 4;   // eight rows in flight per lane cover the reduction
  *variant = "fc_rows_f32";
  if (p.M == 1) return launch_rows<1>(p, lanes, stream);
  if (p.M == 2) return launch_rows<2>(p, lanes, stream);
  return launch_rows<4>(p, lanes, stream);
}

hipError_t launch_fc_small_f32(const Problem& p, hipStream_t stream, const char** variant) {
  switch (width_of(p)) {
    case 4: *variant = "fc_small_f32_w64"; return launch_fsf<4>(p, stream);
    case 2: *variant = "fc_small_f32_w32"; return launch_fsf<2>(p, stream);
    default: *variant = "fc_small_f32_w16"; return launch_fsf<1>(p, stream);
  }
}

}  // namespace glowmi
