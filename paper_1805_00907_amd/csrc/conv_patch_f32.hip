// fp32 convolutions of ordinary size on the fp16 matrix cores: 1x1 and 3x3 filters, stride 1 or 2, any map and channel
// counts.  The arithmetic is that of the other kernels over fp16 pieces (f16_pieces.h): three
// exact fp16 products per fp32 product, fp32 accumulation.
//
// The 3x3 tile kernels (conv_k3*_f32.hip) own a CU per tile of 200 pixels x 128 channels, so they need a large map at a
// large batch; below that, and for strides and pointwise layers, a layer ran on the contraction over planes (a pass that
// measures the input, one that cuts it, every element then fetched once per filter tap) or on the fp32 matrix cores.
// Here a tile is 64 or 128 pixels x 32 to 128 channels and the input is read once:
//   - a workgroup loads the input patch of its pixel tile, CC channels at a time, measures it, scales it and cuts it into
//     two fp16 planes in LDS, which all taps then read at shifted addresses.  The planes are double buffered and there is
//     one barrier per chunk: while a chunk is multiplied, the next one goes from registers into the other planes and the
//     one after it into the registers;
//   - a wavefront multiplies 64 pixels x 32 channels: every filter fragment meets two pixel fragments.  The eight
//     or four wavefronts of a workgroup cover the tile, and where it has fewer such blocks, KS wavefronts share one: each
//     takes every KS-th run of 16 channels, and they add up through LDS at the end;
//   - the filter's fragments go from memory into registers, DB steps ahead: no LDS traffic and no barrier for them;
//   - the accumulators of the h1 h1' products are folded into a second set after every eight or nine steps.  One chain of
//     rounded additions per output was less exact than the contraction over planes that some of these layers came from (3x3
//     392 -> 200 on 92x75 2.7e-7 of the result's norm against 1.1e-7, 512 -> 512 on 28x28 4.3e-7); so it is no further from
//     64-bit sums than that kernel (1.1e-7 and 1.6e-7), for 2 % of the time;
//   - a 3x3 layer of many channels on few pixels has its reduction in parts, whose sums splitk_finish_f32 adds up: 512->512 stride 2 on
//     14x14 at batch 16, filter given, 45 -> 23.5 us; 520 drawn layers 0.83 of their time with operands in the caches and 0.79 from memory.
// What bounds it: LDS and vector memory bandwidth next to the matrix cores, and what a workgroup does before its first and
// behind its last chunk.  A form with 32 x 32 blocks per wavefront and the filter in an LDS ring read 32 KB of fragments per
// 32 reduction indices of a 64 x 64 tile, 256 cycles against 192 of matrix work, and did not get past a third of the matrix
// rate; here it is 16 KB from LDS and 8 KB from memory.  The instructions that are neither go between the matrix ones.
// Measured, microseconds with the filter cut in the call, before (igemm_f32, igemm_f32_p3) -> here: 3x3 stride 2 128 -> 128
// on 56x56 at batch 16 49 -> 23, 3x3 128 -> 128 on 28x28 at batch 8 30 -> 14.8, 3x3 152 -> 152 on 57x57 at batch 13
// 133 -> 87, 3x3 32 -> 344 on 102x102 at batch 4 93 -> 41, 1x1 608 -> 152 on 57x57 at batch 13 92 -> 60.
// The input's scale is per patch (within a tile the exponent only goes down, the accumulators are scaled along), the
// filter's per output channel.  Planes made ahead of time (glowmi_conv2d_pack_filter) are in this kernel's order where the
// channels come in sixteens or the planner takes it for the descriptor they were made with: the packed call is then one launch, 3x3
// stride 2 128 -> 128 on 56x56 at batch 16 24.4 -> 20.8 us, 3x3 128 -> 64 on 85x85 13.4 -> 9.8, 1x1 248 -> 952 on 20x20 at batch 3
// 13.6 -> 9.3.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>

#include "arguments.h"
#include "f16_pieces.h"
#include "igemm.h"
#include "lds_direct.h"
#include "write_through.h"

namespace glowmi {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr unsigned OOBX = 0xFFFFFF00u;           // beyond any fp32 tensor this kernel accepts
constexpr unsigned OOBW = 0x80000000u;           // beyond a filter plane (kPlaneReach), also after adding an offset
constexpr unsigned PASTW = 0x40000000u;          // inside one or PASTW, which itself takes any offset past the plane
constexpr long long kPlaneReach = 1LL << 30;     // a filter plane and what a chunk's steps may address behind its end
constexpr int kChunkPieces = 32;                 // of eight channels: the widest chunk

// R: filter extent, ST: stride, PXB: 64-pixel blocks, CHB: 32-channel blocks of a tile, W: wavefronts (8: a workgroup
// owns a CU, 4: two share it).
template <int R, int ST, int PXB, int CHB, int W>
struct Patch {
  static constexpr int THREADS = 64 * W;
  static constexpr int PX = 64 * PXB, BN = 32 * CHB;
  static constexpr int KS = W / (PXB * CHB);                 // wavefronts that share a block of the tile
  // 16-channel steps per tap and wavefront: one where a 3x3 chunk's nine taps make a trip long enough; a chunk is at
  // least 32 channels (64 for pointwise)
  static constexpr int MS = R == 1 ? (KS == 1 ? 4 : 2) : (KS == 1 ? 2 : 1);
  static constexpr int CC = 16 * KS * MS;                    // channels per chunk
  static constexpr int NS = R * R * MS;                      // steps per chunk and wavefront
  static constexpr int SETS = R == 1 ? 2 : 1;                // chunks in registers: a pointwise one is over before the next has arrived
  static constexpr int UNROLL = SETS;                        // chunks per loop pass
  static constexpr int DB = R == 1 ? 4 : 3;                  // steps whose filter fragments are in flight (nine: no faster)
  static constexpr int MAXP = R == 1 ? PX : ST == 1 ? (PX == 64 ? 120 : 208) : (PX == 64 ? 320 : 600);   // patch pixels
  static constexpr int ROW = 2 * CC;                         // bytes of a pixel in a plane
  static constexpr int PIECES = CC / 8;                      // of eight channels, per pixel
  static constexpr int PASSES = (MAXP * PIECES + THREADS - 1) / THREADS;
  // rows of the planes: as many as whole passes of the workgroup write, where the LDS holds them (no branch then)
  static constexpr int ROWS = 4 * PASSES * THREADS * 16 <= (W == 8 ? 150 : 75) * 1024 ? PASSES * THREADS / PIECES : MAXP;
  static constexpr int ITEMS = ROWS * PIECES;
  static constexpr int APLANE = ROWS * ROW, PAIR = 2 * APLANE;
  static constexpr int FOLD = R == 3 ? 1 : 8 / NS;          // chunks between folds of the accumulators (18 steps: one in the middle, too)
  static constexpr int CUT_FROM = NS > 2 ? 1 : 0;            // the steps beside which the next chunk is cut
  static constexpr int CUT_STEPS = PASSES < NS - CUT_FROM ? PASSES : NS - CUT_FROM;
  static constexpr int XCH = KS > 1 ? W * 8 * 64 * 16 : 0;   // exchange of partial tiles, in place of the planes
  static constexpr int WORDS_AT = 2 * PAIR > XCH ? 2 * PAIR : XCH;
  static constexpr int LDS = WORDS_AT + 64 + PX * 4;         // + the wavefronts' largest magnitudes, the pixels' output positions
  static_assert(KS >= 1 && PXB * CHB * KS == W && (NS * UNROLL) % DB == 0, "work of a wavefront");
  static_assert(PIECES <= kChunkPieces, "kPlaneReach");
  static_assert(LDS <= (W == 8 ? 160 : 80) * 1024, "LDS of one CU");
  // A pixel's 16-byte pieces sit at piece ^ swizzle(key), key = the pixel's position at the tile's own pitch: 16
  // consecutive lanes have 16 consecutive keys, and (position, piece) then names 16 different bank groups (the host
  // makes the patch pitch congruent to the tile's columns modulo 4).
  static __device__ __forceinline__ int swizzle(int key) { return ROW == 64 ? (key >> 2) & 3 : ROW == 128 ? (key >> 1) & 7 : key & 15; }
};

struct Tiles {
  int th, tw, pitch, half;       // tile rows, columns; patch row pitch; 3x3 stride 2: where the odd columns start
  int patch_h, patch_w;          // patch extents in input pixels
  int tiles_y, tiles_x, tiles_c, total;
  FastDiv div_tw, div_pitch, div_tiles_c, div_tiles_x, div_tiles_y;
  int chunks;                    // of channels: of a workgroup
};
constexpr int PLAIN = 0, ADD_LINK = 1, PARTS = 2;   // what a launch does behind the products: PARTS leaves sums of a part of the chunks each

template <int V> struct Const { static constexpr int value = V; };

template <int R, int ST, int PXB, int CHB, int W, int LINK, bool THROUGH>
__global__ __launch_bounds__(64 * W, 2) void conv_patch_f32_kernel(const Problem p, const Tiles tl) {
  fetch_arguments(p, tl);
  using T = Patch<R, ST, PXB, CHB, W>;
  constexpr bool ADD = LINK == ADD_LINK;
  extern __shared__ __align__(16) unsigned char lds[];
  unsigned* maxw = reinterpret_cast<unsigned*>(lds + T::WORDS_AT);
  int* out_pix = reinterpret_cast<int*>(lds + T::WORDS_AT + 64);

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (W == 4 && tid < 16 && (tid & 4)) maxw[tid] = 0;   // the words of wavefronts 4 .. 7, which there are not
  const int wn = wave % CHB;
  const int wm = (wave / CHB) % PXB;
  const int kset = wave / (CHB * PXB);
  const int lrow = lane & 31, lhalf = lane >> 5;

  // Consecutive workgroups go round-robin to the eight XCDs: each XCD takes a contiguous run of tiles, channel tiles
  // innermost, so that the tiles that share a patch find it in their XCD's L2.
  const int per_xcd = gridDim.x >> 3;
  const int t = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  if (t >= tl.total) return;
  const int t1 = tl.div_tiles_c.div(t);
  const int ct = t - t1 * tl.tiles_c;
  int img = 0, ty = 0, tx = t1;                         // pointwise: tile tx of the whole batch's pixels
  if (R != 1) {
    const int t2 = tl.div_tiles_x.div(t1);
    tx = t1 - t2 * tl.tiles_x;
    img = tl.div_tiles_y.div(t2);
    ty = t2 - img * tl.tiles_y;
  }

  // ---- filter fragments: planes of pieces in either order (by channel unless the caller had them made for another kernel, and
  // then slower: a load's lanes are a filter apart); lane: channel lrow of the wavefront's 32, eight indices lhalf of the step's
  // 16.  Step st of a chunk: tap st / MS, channels 16 ((st % MS) KS + kset) .. of the chunk.
  // Pieces of eight channels per tap, the filter's last one filled up with zeros: they meet whatever lies behind a pixel's
  // last channel (the next pixel; behind the tensor zeros).
  const int c8 = (p.c + 7) >> 3;
  const unsigned wpb = 16u * (unsigned)(R * R * c8) * (unsigned)p.k;   // bytes of one plane
  const __amdgpu_buffer_rsrc_t rsrc_w1 = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w_planes), 0, (int)wpb, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_w2 = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<unsigned char*>(static_cast<const unsigned char*>(p.w_planes)) + wpb, 0, (int)wpb, 0x00020000);
  const int ch = ct * T::BN + wn * 32 + lrow;
  // this workgroup's chunks: all or, with its part's first channel and the end of its last
  const int c_first = LINK == PARTS ? (int)blockIdx.y * tl.chunks * T::CC : 0;
  const int c_end = LINK == PARTS && c_first + tl.chunks * T::CC < p.c ? c_first + tl.chunks * T::CC : p.c;
  const int chunks = LINK == PARTS ? (c_end - c_first + T::CC - 1) / T::CC : tl.chunks;
  const PlaneOrder order(p.w_range, p.k, R * R * c8, p.packed_is_cut == 0);
  const unsigned b_base = ch < p.k ? (unsigned)((c_first >> 3) + 2 * kset + lhalf) * order.piece + (unsigned)ch * order.row : OOBW;
  const unsigned tap_step = (unsigned)c8 * order.piece, chunk_step = (unsigned)(T::CC >> 3) * order.piece;
  v4i fb[T::DB][2];                                     // [step in flight][plane]
  auto chunk_at = [&](int chunk) { return chunk < chunks ? (unsigned)chunk * chunk_step : PASTW; };
  auto load_b = [&](int slot, unsigned from, int st) {  // slot, st: compile-time; from: chunk_at of the chunk
    unsigned at = from + (unsigned)(st / T::MS) * tap_step + (unsigned)(st % T::MS * 2 * T::KS) * order.piece;
    asm("" : "+s"(at));                                   // one sum, added to the lane's base: split up it costs eight to twenty registers
    fb[slot][0] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rsrc_w1, b_base + at, 0, 0));
    fb[slot][1] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rsrc_w2, b_base + at, 0, 0));
  };

  // ---- patch: piece q of this thread is item tid + 512 q: pixel item / PIECES, channels 8 (item % PIECES) .. of a chunk;
  // where it comes from in the input and where it goes in the planes
  const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.x), 0, (int)p.x_bytes, 0x00020000);
  unsigned raw_off[T::PASSES], cut_at[T::PASSES];
  int raw_c[T::PASSES];
#pragma unroll
  for (int q = 0; q < T::PASSES; ++q) {
    const int item = tid + q * T::THREADS;
    const int pp = item / T::PIECES, piece = item % T::PIECES;
    raw_c[q] = 8 * piece;
    raw_off[q] = OOBX;
    int key = pp;
    if (R == 1) {
      const int m = tx * T::PX + pp;
      if (pp < T::PX && m < p.M) {
        int pix = m;
        if (ST != 1 || p.oh != p.h || p.ow != p.w_) {    // uniform
          const int im = p.div_ohow.div(m);
          const int rem = m - im * (p.oh * p.ow);
          const int oy = p.div_ow.div(rem);
          pix = (im * p.h + oy * ST) * p.w_ + (rem - oy * p.ow) * ST;
        }
        raw_off[q] = ((unsigned)pix * (unsigned)p.c + (unsigned)raw_c[q]) * 4u;
      }
    } else {
      const int py = tl.div_pitch.div(pp);
      int px = pp - py * tl.pitch;
      key = (ST == 2 ? py >> 1 : py) * tl.tw + px;
      if (ST == 2) px = px < tl.half ? 2 * px : px < 2 * tl.half ? 2 * (px - tl.half) + 1 : tl.patch_w;   // even columns, then odd ones
      const int iy = ty * tl.th * ST - p.pad_t + py, ix = tx * tl.tw * ST - p.pad_l + px;
      if (pp < T::MAXP && py < tl.patch_h && px < tl.patch_w && (unsigned)iy < (unsigned)p.h && (unsigned)ix < (unsigned)p.w_)
        raw_off[q] = ((unsigned)((img * p.h + iy) * p.w_ + ix) * (unsigned)p.c + (unsigned)raw_c[q]) * 4u;
    }
    cut_at[q] = pp * T::ROW + ((piece ^ T::swizzle(key)) << 4);
  }
  auto load_raw = [&](v4f (&dst)[T::PASSES][2], int chunk) {   // past the last chunk: zeros
    const int c0 = c_first + chunk * T::CC;
#pragma unroll
    for (int q = 0; q < T::PASSES; ++q) {
      const unsigned off = raw_off[q] != OOBX && c0 + raw_c[q] < c_end ? raw_off[q] + (unsigned)c0 * 4u : OOBX;
      dst[q][0] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, off, 0, 0));
      dst[q][1] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, off + 16u, 0, 0));
    }
  };
  typedef v4f Raw[T::PASSES][2];                        // a chunk on its way into the planes
  Raw pre[T::SETS];                                     // chunk j in set j % SETS
  auto leave_max = [&](const Raw& raw, int parity) {
    const unsigned share_max = wave_max_of(raw);
    if (lane == 0) maxw[parity * 8 + wave] = share_max;
  };
  int se_x = 141;                                       // scale exponent of the planes written last
  bool finite = true;
  auto take_scale = [&](int parity) {                   // of the chunk whose magnitudes were left last
    const unsigned m = max_of_eight(maxw + parity * 8);
    finite = finite && m < 0x7f800000u;
    const int need = scale_exponent(m);
    se_x = need < se_x ? need : se_x;
  };
  auto cut = [&](const Raw& raw, int parity, int part) {   // a CUT_STEPS-th of a chunk, into the planes of that parity
#pragma unroll
    for (int q = 0; q < T::PASSES; ++q) {
      if (q * T::CUT_STEPS / T::PASSES != part) continue;
      if ((q + 1) * T::THREADS <= T::ITEMS || tid + q * T::THREADS < T::ITEMS) {
        const float v[8] = {raw[q][0][0], raw[q][0][1], raw[q][0][2], raw[q][0][3],
                            raw[q][1][0], raw[q][1][1], raw[q][1][2], raw[q][1][3]};
        v4u p1, p2;
        cut8_in_place(v, se_x, p1, p2);
        unsigned char* dst = lds + parity * T::PAIR + cut_at[q];
        *reinterpret_cast<v4u*>(dst) = p1;
        *reinterpret_cast<v4u*>(dst + T::APLANE) = p2;
      }
    }
  };

  // ---- before the first chunk: chunk 0 in the planes, the next SETS in registers, the magnitudes of chunk 1 left behind
  Raw pre0;
  load_raw(pre0, 0);
#pragma unroll
  for (int j = 1; j <= T::SETS; ++j) load_raw(pre[j % T::SETS], j);
#pragma unroll
  for (int d = 0; d < T::DB; ++d) load_b(d, chunk_at(d / T::NS), d % T::NS);

  // ---- what the epilogue needs, fetched now: the channel's bias, the filter's scale, where the pixels lie in the output
  const float* __restrict__ bias = static_cast<const float*>(p.bias);
  const float bv = LINK != PARTS && ch < p.k && bias ? bias[ch] : 0.f;
  const unsigned w_max_bits = order.max_bits(p.w_range, ch < p.k ? ch : 0);
  if (tid < T::PX) {
    int pix = -1;
    if (R == 1) {
      const int m = tx * T::PX + tid;
      if (m < p.M) pix = m;
    } else {
      const int r = tl.div_tw.div(tid), c = tid - r * tl.tw;
      const int oy = ty * tl.th + r, ox = tx * tl.tw + c;
      if (r < tl.th && oy < p.oh && ox < p.ow) pix = (img * p.oh + oy) * p.ow + ox;
    }
    out_pix[tid] = pix;
  }

  // ---- fragment addresses: the wavefront's two blocks of 32 pixels at tap (0, 0)
  int pp0[2], key0[2];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int tp = wm * 64 + b * 32 + lrow;
    pp0[b] = key0[b] = tp;
    if (R != 1) {
      int r = tl.div_tw.div(tp), c = tp - r * tl.tw;
      if (r >= tl.th) {                                 // past the tile: any pixel of it
        r = 0;
        c = 0;
      }
      pp0[b] = r * ST * tl.pitch + c;
      key0[b] = r * tl.tw + c;
    }
  }

  v16f acc[2], acc_lo[2];                               // the h1 h1' products; the cross terms (weight 2^-11)
  v16f total[2];                                        // what acc is folded into
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      acc[b][e] = 0.f;
      acc_lo[b][e] = 0.f;
      total[b][e] = 0.f;
    }

  leave_max(pre0, 0);
  __syncthreads();
  take_scale(0);
#pragma unroll
  for (int i = 0; i < T::CUT_STEPS; ++i) cut(pre0, 0, i);
  int se_acc = se_x;                                    // scale exponent of the accumulators
  leave_max(pre[1 % T::SETS], 1);
  // The compiler's counts of loads in flight then describe the loop alone; joined with those of this part they are too low,
  // and a chunk waited for the loads of the one before it.
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));

  // ---- the chunks.  A step's pixel fragments are read while the step before it is multiplied.
  auto chunk_steps = [&](int chunk, auto unrolled) {
    constexpr int U = decltype(unrolled)::value;        // which chunk of a loop pass
    const int parity = T::UNROLL == 2 ? U : chunk & 1;
    Raw& next = pre[(U + 1) % T::SETS];
    const unsigned char* planes = lds + parity * T::PAIR;
    v8h fa[2][2][2];                                    // [set][block][plane]
    auto read_a = [&](int st) {                         // compile-time
      const int tap = st / T::MS, tr = R == 1 ? 0 : tap / 3, ts = R == 1 ? 0 : tap % 3;
      const int piece = (st % T::MS * T::KS + kset) * 2 + lhalf;
      // tap (tr, ts) in the patch: whole rows and columns; stride 2 keeps the odd columns apart
      const int d_pp = tr * tl.pitch + (ST == 2 ? (ts & 1) * tl.half + (ts >> 1) : ts);
      const int d_key = ST == 2 ? (tr >> 1) * tl.tw + (ts & 1) * tl.half + (ts >> 1) : tr * tl.tw + ts;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const unsigned char* at = planes + (pp0[b] + d_pp) * T::ROW + ((piece ^ T::swizzle(key0[b] + d_key)) << 4);
        fa[st & 1][b][0] = __builtin_bit_cast(v8h, *reinterpret_cast<const v4i*>(at));
        fa[st & 1][b][1] = __builtin_bit_cast(v8h, *reinterpret_cast<const v4i*>(at + T::APLANE));
      }
    };
    auto fold = [&] {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          total[b][e] += acc[b][e];
          acc[b][e] = 0.f;
        }
    };
    if (U % T::FOLD == 0 && chunk % T::FOLD == 0) fold();   // uniform
    const unsigned from[3] = {(unsigned)chunk * chunk_step, chunk_at(chunk + 1), chunk_at(chunk + 2)};   // (DB <= 2 NS)
    __syncthreads();                                    // this chunk's planes and the next one's magnitudes are there
    read_a(0);
    if (se_x < se_acc) {                                // uniform: larger values than any chunk before
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          acc[b][e] = __builtin_ldexpf(acc[b][e], se_x - se_acc);
          acc_lo[b][e] = __builtin_ldexpf(acc_lo[b][e], se_x - se_acc);
          total[b][e] = __builtin_ldexpf(total[b][e], se_x - se_acc);
        }
      se_acc = se_x;
    }
    if (T::CUT_FROM == 0) take_scale(parity ^ 1);       // for the next chunk's planes
#pragma unroll
    for (int st = 0; st < T::NS; ++st) {
      const int cur = st & 1, slot = (U * T::NS + st) % T::DB;
      if (T::NS > 9 && st == T::NS / 2) {
        int always = 1;                                 // opaque: without the branch the registers run out (14 to 25 spills a chunk)
        asm volatile("" : "+s"(always));
        if (always) fold();
      }
      __builtin_amdgcn_sched_barrier(0);
      if (st + 1 < T::NS) read_a(st + 1);
      const v8h b1 = __builtin_bit_cast(v8h, fb[slot][0]), b2 = __builtin_bit_cast(v8h, fb[slot][1]);
#pragma unroll
      for (int b = 0; b < 2; ++b) acc_lo[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[cur][b][0], b2, acc_lo[b], 0, 0, 0);
#pragma unroll
      for (int b = 0; b < 2; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[cur][b][0], b1, acc[b], 0, 0, 0);
#pragma unroll
      for (int b = 0; b < 2; ++b) acc_lo[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[cur][b][1], b1, acc_lo[b], 0, 0, 0);
      const int ahead = st + T::DB;                     // DB <= 2 NS
      load_b(slot, from[ahead / T::NS], ahead % T::NS);
      constexpr int LAST_CUT = T::CUT_FROM + T::CUT_STEPS - 1;
      const bool cutting = st >= T::CUT_FROM && st <= LAST_CUT;
      if (T::CUT_FROM == 1 && st == 0) take_scale(parity ^ 1);
      if (cutting) cut(next, parity ^ 1, st - T::CUT_FROM);
      if (st == LAST_CUT) load_raw(next, chunk + 1 + T::SETS);
      if (st == T::NS - 1) leave_max(pre[U % T::SETS], parity);   // chunk + 2
      // everything else goes between the matrix instructions: each leaves room for seven
#pragma unroll
      for (int m = 0; m < 6; ++m) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // matrix
        if (cutting) __builtin_amdgcn_sched_group_barrier(0x002, 12, 0);   // vector
        else __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // LDS read
      }
    }
  };
  int chunk = 0;
  for (; chunk + T::UNROLL <= chunks; chunk += T::UNROLL) {
    chunk_steps(chunk, Const<0>());
    if (T::UNROLL == 2) chunk_steps(chunk + 1, Const<T::UNROLL - 1>());
  }
  if (T::UNROLL == 2 && chunk < chunks) chunk_steps(chunk, Const<0>());   // behind the loop: a way out of its middle costs waits

  // ---- epilogue.  Register e of a block is pixel (e/4)*8 + 4*lhalf + e%4 of its 32, channel ch.  The KS wavefronts of
  // a block swap their partial sums: each finishes OQ of the block's eight quads of registers.
  const ScaleBack sb = scale_back_of(se_acc, scale_exponent(w_max_bits), finite && w_max_bits < 0x7f800000u);
  constexpr int OQ = 8 / T::KS;
  float res[OQ][4];
  float joined[32];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int e = 0; e < 16; ++e) joined[b * 16 + e] = __builtin_fmaf(acc_lo[b][e], kLowPieceWeight, acc[b][e]) + total[b][e];
  if (T::KS > 1) {
    v4f* xch = reinterpret_cast<v4f*>(lds);
    const int pair = wave % (PXB * CHB);
    __syncthreads();                                    // everyone is done with the planes
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const v4f send = {joined[4 * q], joined[4 * q + 1], joined[4 * q + 2], joined[4 * q + 3]};
      if (q / OQ != kset) xch[((pair * T::KS + kset) * 8 + q) * 64 + lane] = send;
      else {
#pragma unroll
        for (int e = 0; e < 4; ++e) res[q % OQ][e] = send[e];
      }
    }
    __syncthreads();
#pragma unroll
    for (int d = 1; d < T::KS; ++d) {
      const int from = (kset + d) % T::KS;
#pragma unroll
      for (int q = 0; q < OQ; ++q) {
        const v4f got = xch[((pair * T::KS + from) * 8 + kset * OQ + q) * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) res[q][e] += got[e];
      }
    }
  } else {
#pragma unroll
    for (int q = 0; q < OQ; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) res[q][e] = joined[(4 * q + e) % 32];
  }
  const unsigned y_bytes = (unsigned)((long long)p.M * p.k * 4);   // below 4 GiB on this kernel
  void* const y = LINK == PARTS ? static_cast<unsigned char*>(p.partial) + (size_t)blockIdx.y * y_bytes : p.y;
  const __amdgpu_buffer_rsrc_t rsrc_y = __builtin_amdgcn_make_buffer_rsrc(y, 0, (int)y_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_add =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(ADD ? p.addend : p.y), 0, (int)y_bytes, 0x00020000);
  unsigned off[OQ * 4];
#pragma unroll
  for (int q = 0; q < OQ; ++q) {
    const int quad = kset * OQ + q;
    const int px0 = wm * 64 + (quad >> 2) * 32 + (quad & 3) * 8 + lhalf * 4;
    const v4i pix = *reinterpret_cast<const v4i*>(out_pix + px0);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      off[q * 4 + e] = pix[e] >= 0 && ch < p.k ? ((unsigned)pix[e] * (unsigned)p.k + (unsigned)ch) * 4u : OOBX;
  }
  float addv[OQ * 4];
  if (ADD) {                                            // all in flight together: one wait, not one per store
#pragma unroll
    for (int e = 0; e < OQ * 4; ++e)
      addv[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc_add, off[e], 0, 0));
  }
  const bool act = LINK != PARTS && p.act == 1;
#pragma unroll
  for (int e = 0; e < OQ * 4; ++e) {
    float v = __builtin_ldexpf(res[e / 4][e % 4], sb.neg_se) + sb.poison + bv;
    if (ADD) v += addv[e];
    if (act) v = clamp_act(v, p.act_lo, p.act_hi);
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), rsrc_y, off[e], 0, THROUGH ? kThrough : 0);
  }
}

// The filter [k][r][s][c] as two planes [Kgemm / 8][k][8], each output channel by a scale of its own, in one launch.  The
// eight consecutive reduction indices of a channel are 16 bytes and the channels lie side by side, so the fragment of 32
// channels x 16 indices that a wavefront multiplies is two runs of 512 bytes; as rows of one channel it is 32 lines of which
// 32 bytes each are wanted, and a CU fetches it at a quarter of the rate (8 KB in 0.22 instead of 0.058 us).
// A workgroup takes eight channels, so that it writes whole 128-byte lines (one channel at a time, 16 bytes of eight lines
// here and there, 512 x 4608 took 9 us instead of 5): a wavefront finds each one's largest magnitude and its bits go into
// words[channel]; then the workgroup cuts its part of the reduction of all eight.  Where eight channels at a time leave CUs
// idle, `parts` workgroups share them, each measuring for itself.
// One launch cuts the filters of several layers of a sequence (kCutJobs at most).
constexpr int CUT_ROWS = 8;
struct CutJob {
  const float* w;
  unsigned short* dst;
  unsigned* words;
  int rows, taps, c, parts, first_block;
  FastDiv div_c8;
};
template <int N>
struct CutJobs {
  int n;
  CutJob job[N];
};
template <int N>
__global__ __launch_bounds__(64 * CUT_ROWS) void cut_filter_kernel(const CutJobs<N> jobs) {
  fetch_arguments(jobs);
  __shared__ unsigned largest[CUT_ROWS];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int j = 0;
  while (N > 1 && j + 1 < jobs.n && (int)blockIdx.x >= jobs.job[j + 1].first_block) ++j;   // uniform
  const float* __restrict__ w = jobs.job[j].w;
  unsigned short* __restrict__ dst = jobs.job[j].dst;
  unsigned* __restrict__ words = jobs.job[j].words;
  const int rows = jobs.job[j].rows, taps = jobs.job[j].taps, c = jobs.job[j].c, parts = jobs.job[j].parts;
  const int c8 = (c + 7) >> 3, row8 = taps * c8, depth = taps * c;   // a channel's pieces of eight; its weights
  const bool ragged = (c & 7) != 0;                     // uniform
  const size_t plane_elems = (size_t)rows * row8 * 8;
  const int at = (int)blockIdx.x - jobs.job[j].first_block;
  const int blocks = (N > 1 && j + 1 < jobs.n ? jobs.job[j + 1].first_block : (int)gridDim.x) - jobs.job[j].first_block;   // a multiple of 8
  // the parts of a group on one XCD, whose L2 serves the measuring of all but the first
  const int block = (at & 7) * (blocks >> 3) + (at >> 3);
  const int group = block / parts, part = block - group * parts;
  if (group * CUT_ROWS >= rows) return;
  // 16 bytes from any weight on, zeros past the last one (buffer loads are checked word by word)
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(w), 0, (int)(4u * (unsigned)rows * (unsigned)depth), 0x00020000);
  auto load = [&](unsigned weight) { return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rsrc, 4u * weight, 0, 0)); };
  // what this thread will cut, asked for first: two trips to memory become one
  constexpr int HELD = 4, STEP = 64;
  const int r = (int)threadIdx.x & (CUT_ROWS - 1), row = group * CUT_ROWS + r;
  const int per = (row8 + parts - 1) / parts;
  const int first = part * per + (int)threadIdx.x / CUT_ROWS;
  const int end = row < rows ? ((part + 1) * per < row8 ? (part + 1) * per : row8) : 0;
  auto piece = [&](int g, v4f (&v)[2]) {                 // eight weights of this thread's channel, a tap's last ones filled up
    const int tap = ragged ? jobs.job[j].div_c8.div(g) : 0;
    const int ch = (g - tap * c8) * 8;                   // (not ragged: the weights lie in the order of the pieces)
    // (no branch around the loads: the compiler would wait for them where its paths join)
    const unsigned from = g < end ? (unsigned)row * (unsigned)depth + (unsigned)(tap * c + ch) : 0x3fffffc0u;
    v[0] = load(from);
    v[1] = load(from + 4);
    if (ragged) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e / 4][e % 4] = ch + e < c ? v[e / 4][e % 4] : 0.f;
    }
  };
  v4f held[HELD][2];
#pragma unroll
  for (int q = 0; q < HELD; ++q) piece(first + q * STEP, held[q]);
  {
    const int mine = group * CUT_ROWS + wave;
    unsigned m = 0;
    if (mine < rows) {
      const unsigned from = (unsigned)mine * (unsigned)depth;
      const int quads = (depth + 3) >> 2;
      constexpr int PAIRS = 5;                          // of loads in flight
      for (int g0 = lane; g0 < quads; g0 += 128 * PAIRS) {
        v4f v[PAIRS][2];
#pragma unroll
        for (int q = 0; q < 2 * PAIRS; ++q) {
          const int g = g0 + 64 * q < quads ? g0 + 64 * q : quads - 1;
          v[q / 2][q % 2] = load(from + 4u * (unsigned)g);
          if (ragged) {                                 // the next channel's first weights do not count
#pragma unroll
            for (int e = 0; e < 4; ++e) v[q / 2][q % 2][e] = 4 * g + e < depth ? v[q / 2][q % 2][e] : 0.f;
          }
        }
        const unsigned o = lane_max_of(v);
        m = o > m ? o : m;
      }
      m = wave_max_u32(m);
      if (part == 0 && lane == 0) words[mine] = mine == 0 ? m | kByChannel : m;
    }
    if (lane == 0) largest[wave] = m;
  }
  __syncthreads();
  const int se = scale_exponent(largest[r]);
  auto write = [&](int g, const v4f (&w8)[2]) {
    const float v[8] = {w8[0][0], w8[0][1], w8[0][2], w8[0][3], w8[1][0], w8[1][1], w8[1][2], w8[1][3]};
    v4u p1, p2;
    cut8_in_place(v, se, p1, p2);
    unsigned short* out = dst + ((size_t)g * rows + row) * 8;
    *reinterpret_cast<v4u*>(out) = p1;
    *reinterpret_cast<v4u*>(out + plane_elems) = p2;
  };
#pragma unroll
  for (int q = 0; q < HELD; ++q)
    if (first + q * STEP < end) write(first + q * STEP, held[q]);
  for (int g = first + HELD * STEP; g < end; g += STEP) {
    v4f w8[2];
    piece(g, w8);
    write(g, w8);
  }
}

int patch_pitch(int tw, int st) {
  // at least the patch's columns; congruent to the tile's columns modulo 4 (stride 2, where output rows are two patch
  // rows apart: twice the pitch, possible for even columns)
  if (st == 1) return tw + 4;
  int pitch = 2 * tw + 2;
  while (tw % 2 == 0 && (2 * pitch) % 4 != tw % 4) ++pitch;
  return pitch;
}

// The rows x columns of at most px pixels with the fewest tiles over the map whose patch fits; ties: the smaller patch.
struct MapTile { int th, tw, tiles; };
MapTile pick_map_tile(const Problem& p, int px, int max_patch) {
  const int st = p.stride_h;
  MapTile best = {0, 0, 0};
  int best_patch = 0;
  for (int th = 1; th <= px / 4; ++th) {
    const int rows = (p.oh + th - 1) / th;
    int tw = px / th;
    while (tw > 4 && ((th - 1) * st + 3) * patch_pitch(tw, st) > max_patch) --tw;
    const int cols = (p.ow + tw - 1) / tw;
    const int even = (p.ow + cols - 1) / cols;           // the same number of tiles with fewer columns each
    if (even >= 4) tw = even;
    const int patch = ((th - 1) * st + 3) * patch_pitch(tw, st);
    if (patch > max_patch) continue;
    if (best.th == 0 || rows * cols < best.tiles || (rows * cols == best.tiles && patch < best_patch)) {
      best = {th, tw, rows * cols};
      best_patch = patch;
    }
    if (rows == 1) break;
  }
  return best;
}

template <int R, int ST, int PXB, int CHB, int W>
void fill_tiles(const Problem& p, Tiles* t) {
  using T = Patch<R, ST, PXB, CHB, W>;
  t->th = 1;
  t->tw = T::PX;
  if (R == 1) {
    t->pitch = T::PX;
    t->half = 0;
    t->patch_h = 1;
    t->patch_w = T::PX;
    t->tiles_y = 1;
    t->tiles_x = (p.M + T::PX - 1) / T::PX;
  } else {
    const MapTile m = pick_map_tile(p, T::PX, T::MAXP);
    t->th = m.th;
    t->tw = m.tw;
    t->pitch = patch_pitch(t->tw, ST);
    t->half = ST == 2 ? t->tw + 1 : 0;
    t->patch_h = (t->th - 1) * ST + 3;
    t->patch_w = (t->tw - 1) * ST + 3;
    t->tiles_y = (p.oh + t->th - 1) / t->th;
    t->tiles_x = (p.ow + t->tw - 1) / t->tw;
  }
  t->tiles_c = (p.k + T::BN - 1) / T::BN;
  t->div_tw = make_fastdiv((uint32_t)t->tw);
  t->div_pitch = make_fastdiv((uint32_t)t->pitch);
  t->div_tiles_c = make_fastdiv((uint32_t)t->tiles_c);
  t->div_tiles_x = make_fastdiv((uint32_t)t->tiles_x);
  t->div_tiles_y = make_fastdiv((uint32_t)t->tiles_y);
  t->chunks = (p.c + T::CC - 1) / T::CC;
  const long long total = (R == 1 ? 1LL : (long long)p.n) * t->tiles_y * t->tiles_x * t->tiles_c;
  t->total = total < (1LL << 30) ? (int)total : -1;
}

template <int R, int ST, int PXB, int CHB, int W, int LINK, bool THROUGH>
hipError_t launch_patch_as(const Problem& p, int parts, hipStream_t stream, const char** variant) {
  using T = Patch<R, ST, PXB, CHB, W>;
  auto kern = conv_patch_f32_kernel<R, ST, PXB, CHB, W, LINK, THROUGH>;
  static const hipError_t attr_status = hipFuncSetAttribute(
      reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS);
  if (attr_status != hipSuccess) return attr_status;
  Tiles t;
  fill_tiles<R, ST, PXB, CHB, W>(p, &t);
  if (t.total <= 0) return hipErrorInvalidValue;
  if (LINK == PARTS) {
    if (parts < 2 || parts > t.chunks || !p.partial) return hipErrorInvalidValue;
    const int each = (t.chunks + parts - 1) / parts;
    if ((t.chunks + each - 1) / each != parts) return hipErrorInvalidValue;
    t.chunks = each;
  }
  static thread_local char name[64];
  snprintf(name, sizeof(name), "conv_patch_f32_f16x3_%dx%ds%d_%dx%dw%d%s", R, R, ST, T::PX, T::BN, W, LINK == PARTS ? "_parts" : LINK == ADD_LINK ? "_add" : "");
  *variant = name;
  hipLaunchKernelGGL(kern, dim3((unsigned)((t.total + 7) / 8 * 8), LINK == PARTS ? (unsigned)parts : 1u), dim3(T::THREADS), T::LDS, stream, p, t);
  return hipGetLastError();
}

// (a branch in the kernel instead costs up to half of what it gains, in instructions fetched behind the last chunk)
template <int R, int ST, int PXB, int CHB, int W, int LINK>
hipError_t launch_patch(const Problem& p, int parts, hipStream_t stream, const char** variant) {
  return through_pays(LINK == PARTS ? p.partial : p.y, p.k) ? launch_patch_as<R, ST, PXB, CHB, W, LINK, true>(p, parts, stream, variant)
                                                           : launch_patch_as<R, ST, PXB, CHB, W, LINK, false>(p, parts, stream, variant);
}

// ---- forms: pixels x channels of a tile, wavefronts.  Eight wavefronts per tile where the tiles do not fill the machine
// twice, four (and two workgroups per CU, one's start and end behind the other's middle) where they do.
constexpr int FORMS = 6;

template <int R, int ST, int LINK>
hipError_t launch_patch_form(const Problem& p, int form, int parts, hipStream_t stream, const char** variant) {
  if constexpr (R == 3) {
    if (form == 1) return launch_patch<R, ST, 1, 4, 8, LINK>(p, parts, stream, variant);
  }
  if constexpr (R == 1 || ST == 1) {
    switch (form) {
      case 0: return launch_patch<R, ST, 1, 2, 8, LINK>(p, parts, stream, variant);
      case 2: return launch_patch<R, ST, 1, 1, 8, LINK>(p, parts, stream, variant);
      case 3: return launch_patch<R, ST, 1, 2, 4, LINK>(p, parts, stream, variant);
      case 4: return launch_patch<R, ST, 1, 4, 4, LINK>(p, parts, stream, variant);
      case 5: return launch_patch<R, ST, 2, 1, 4, LINK>(p, parts, stream, variant);
    }
  }
  return hipErrorInvalidValue;
}

template <int LINK>
hipError_t launch_patch_shape(const Problem& p, int form, int parts, hipStream_t stream, const char** variant) {
  if constexpr (LINK != PARTS) {
    if (p.r == 1) return p.stride_h == 1 ? launch_patch_form<1, 1, LINK>(p, form, parts, stream, variant)
                                         : launch_patch_form<1, 2, LINK>(p, form, parts, stream, variant);
  }
  if (p.r != 3) return hipErrorInvalidValue;
  return p.stride_h == 1 ? launch_patch_form<3, 1, LINK>(p, form, parts, stream, variant)
                         : launch_patch_form<3, 2, LINK>(p, form, parts, stream, variant);
}

// What a form costs, in microseconds, fitted to 78 layers of 0.05 to 59 GFLOP in all forms (median error 4 %; choosing by it
// costs 0.15 % over the best form of each layer, 5 % at most): 4.3 for the two launches (1 where the filter was cut ahead of
// the call), 1 per megabyte of filter to cut, 0.1 per megabyte of input and output, and per round of workgroups a start and end and so much per chunk of channels.  A
// four-wavefront workgroup that has a CU to itself takes 0.7 of what two take that share it.  Above 20 GFLOP the estimates are
// low, up to 25 % (512 -> 512 on 28x28 at batch 16: 142, measured 188), for all forms alike: nothing but the choice among forms
// goes by them there.  (A tile of 128 pixels x 64 channels lost its place to 64 x 64 with the second accumulator set, for which
// it has no registers: 64 -> 64 on 112x112 at batch 16 60 -> 71 us, 64 x 64 63.)
struct FormCost { int px, bn, waves, cc1, cc3; float round1, chunk1, round3, chunk3; };
constexpr FormCost kForms[FORMS] = {
    {64, 64, 8, 128, 64, 3.48f, 0.97f, 3.23f, 2.51f},
    {64, 128, 8, 0, 32, 0.f, 0.f, 3.51f, 2.02f},
    {64, 32, 8, 256, 128, 4.02f, 1.64f, 3.97f, 2.95f},
    {64, 64, 4, 64, 32, 2.57f, 1.09f, 3.79f, 2.21f},
    {64, 128, 4, 64, 32, 2.95f, 1.36f, 4.82f, 3.54f},
    {128, 32, 4, 64, 32, 3.10f, 1.62f, 4.87f, 2.53f},
};

// Parts of the reduction where the tiles leave CUs idle, each with workgroups of its own; splitk_finish_f32 sums them up.  What that takes was
// fitted to 3551 runs of 260 3x3 layers of 96 to 768 channels on up to 9000 pixels (median error 4 %); the margin is that of both estimates.
constexpr int kMostParts = 8;
constexpr double kPartsMargin = 1.10;
// Layers that parts are measured on: 486 drawn ones that the estimates give to them, 0.84 of the time in one part with operands in the caches
// and 0.80 from memory, the slowest 1.02 by both; in place of the contraction over planes 34, 0.71 and 0.75, the slowest 0.92.  Beyond: 488->16 on
// 107x107 at batch 8 1.06; in place of the contraction over planes 2000->232 stride 2 on 9x7 at batch 25 1.23; a filter of more than 16 MB
// 624->816 on 17x17 at batch 2 31 -> 42 us.
bool parts_measured(const Problem& p) { return p.c >= 96 && p.c <= 2048 && p.M <= 40000 && p.w_bytes <= (16u << 20); }
constexpr int kMostOverPlanes = 1400;
// Wavefronts that share the reduction of a form's block.  With no fewer runs than in one part, and two chunks and more to a part, sums lie at
// 0.72 to 1.006 of the distance from 64-bit ones that they have without parts (520 layers, median 0.97); 26 layers of fewer runs lay at 0.97 to
// 1.09, 8 of one chunk to a part at 0.99 to 1.02.
int sharing(const FormCost& c) { return c.waves / (c.px / 64 * (c.bn / 32)); }

double fixed_cost(const Problem& p, bool cut_ahead) {
  return (cut_ahead ? 1.0 : 4.3 + 1e-6 * p.w_bytes) + 1e-7 * ((double)p.x_bytes + 4.0 * p.M * p.k);
}

// The cheapest form for the layer and its cost; a 3x3 stride-2 layer has one form (two of its patches do not fit a CU; a
// chunk of it takes 1.35 times as long).  split: the cheapest form in parts, with forced_parts of them or, where that is below one, as many
// as are fastest; one where it takes longer than the form for the whole.  Whether the filter was cut ahead counts in the costs and in neither
// choice (both go by a call over planes): calls with and without them sum in the same order.
int cheapest_form(const Problem& p, int forced, int forced_parts, double* cost, PatchParts* split, double* split_us) {
  const bool pointwise = p.r == 1;
  MapTile map[2] = {{0, 0, 0}, {0, 0, 0}};               // of 64 and of 128 pixels
  if (!pointwise) {
    map[0] = pick_map_tile(p, 64, p.stride_h == 1 ? 120 : 320);
    if (p.stride_h == 1) map[1] = pick_map_tile(p, 128, 208);
  }
  auto takes = [&](int f) {
    return !(pointwise ? kForms[f].cc1 == 0 : p.stride_h == 2 && f != 1) && (forced < 0 || f == forced);
  };
  auto tiles_of = [&](const FormCost& c) {
    const double px_tiles = pointwise ? (double)((p.M + c.px - 1) / c.px) : (double)p.n * map[c.px == 128].tiles;
    return px_tiles * ((p.k + c.bn - 1) / c.bn);
  };
  auto chunks_of = [&](const FormCost& c) { return (p.c + (pointwise ? c.cc1 : c.cc3) - 1) / (pointwise ? c.cc1 : c.cc3); };
  auto chunk_us = [&](const FormCost& c) { return pointwise ? (double)c.chunk1 : p.stride_h == 2 ? 1.35 * c.chunk3 : (double)c.chunk3; };
  auto rounds_of = [](const FormCost& c, double workgroups) {
    const double rounds = workgroups / (c.waves == 8 ? 256 : 512);
    return c.waves == 4 && rounds <= 0.5 ? 0.7 : rounds <= 3.0 ? (double)(int)(rounds + 0.999999) : rounds + 0.5;
  };
  double steps = 0.0, split_steps = 0.0;                 // of the forms chosen, beside what is fixed
  int best = -1;
  for (int f = 0; f < FORMS; ++f) {
    if (!takes(f)) continue;
    const FormCost& c = kForms[f];
    const double t = rounds_of(c, tiles_of(c)) * ((pointwise ? c.round1 : c.round3) + chunks_of(c) * chunk_us(c));
    if (best < 0 || t < steps) {
      best = f;
      steps = t;
    }
  }
  const double fixed = fixed_cost(p, p.packed_is_cut != 0), over_planes = fixed_cost(p, true);
  *cost = fixed + steps;
  if (!split || pointwise || best < 0 || !(forced_parts > 1 || parts_measured(p))) return best;
  PatchParts in_parts = {0, 1};
  const int runs = sharing(kForms[best]);
  auto split_cost = [&](double fixed) { return kPartsMargin * (3.0 + 1.03 * fixed + split_steps + 0.067e-6 * p.w_bytes); };
  const double below = (over_planes + steps) / kPartsMargin - (3.0 + 1.03 * over_planes + 0.067e-6 * p.w_bytes) + 1e-6;   // of split_steps
  for (int f = 0; f < FORMS; ++f) {
    if (!takes(f)) continue;
    const FormCost& c = kForms[f];
    const int chunks = chunks_of(c);
    const double tiles = tiles_of(c), chunk = chunk_us(c);
    // no number of parts takes less than the products in full rounds: most layers that stay whole are decided by this
    if (forced_parts <= 1 && 0.94 * tiles * chunks * chunk / (c.waves == 8 ? 256 : 512) + 0.83 * 0.7 * c.round3 >= below) continue;
    for (int s = 2; s <= kMostParts; ++s) {
      const int each = (chunks + s - 1) / s;
      if ((chunks + each - 1) / each != s || (forced_parts > 0 && s != forced_parts)) continue;
      if (forced_parts <= 1 && (each < 2 || s * sharing(c) < runs)) continue;
      // (a part's tiles are dealt to the eight XCDs: three times 84 tiles are 33 workgroups to an XCD of 32 CUs)
      const double workgroups = 8.0 * (((long long)tiles + 7) / 8) * s, full = workgroups / (c.waves == 8 ? 256 : 512);
      const double r = rounds_of(c, workgroups);
      const double u = 0.83 * r * c.round3 + 0.94 * r * each * chunk + 1.02 * (full < 1.0 ? full : 1.0) + 1.34e-6 * s * (double)p.M * p.k;
      if (in_parts.parts == 1 || u < split_steps) {
        in_parts = {f, s};
        split_steps = u;
      }
    }
  }
  *split_us = split_cost(fixed);
  if (in_parts.parts > 1 && (forced_parts > 1 || split_cost(over_planes) < over_planes + steps)) *split = in_parts;
  return best;
}

}  // namespace

// The form to run a layer in, -1: not a layer for this kernel.  An addend does not count: the workspace queries do not know
// of it, and a call must not plan what they did not ask room for.
int patch_f32_form(const Problem& p, double* us_out, PatchParts* split) {
  if (split) *split = {0, 1};
  const int mode = knob_or(KNOB_F32_PATCH, 1);          // 0: off, 2: any size (tests)
  if (mode == 0 || (mode == 1 && knob_or(KNOB_F32_P3, 1) == 0)) return -1;   // either switch: such layers stay on the fp32 matrix cores
  if (p.b_is_kn || p.chain_n > 0 || p.groups != 1) return -1;
  if (p.r != p.s || (p.r != 1 && p.r != 3) || p.stride_h != p.stride_w || (p.stride_h != 1 && p.stride_h != 2)) return -1;
  if (p.r == 1 && (p.pad_t != 0 || p.pad_l != 0 || (p.oh - 1) * p.stride_h >= p.h || (p.ow - 1) * p.stride_w >= p.w_)) return -1;
  if (p.x_bytes > 0xF0000000u || p.w_bytes > (1u << 30) || (long long)p.M * p.k * 4 > 0xF0000000LL) return -1;   // 32-bit byte offsets
  if (((long long)p.r * p.s * ((p.c + 7) / 8) + kChunkPieces) * 16 * p.k > kPlaneReach) return -1;   // a tap's channels are filled up to eight
  const int knob_form = knob_or(KNOB_F32_PATCH_TILE, -1), forced = knob_form < FORMS ? knob_form : -1;   // (no such form: the rule's)
  // Against what the layer would take elsewhere: on the fp32 matrix cores 8 us (6 for pointwise) and 50 or 75 TFLOP/s, or what
  // its tensors take at 3 TB/s; on the one-launch kernel for few pixels 3.5 us and 32 TFLOP/s.  The margin covers both
  // estimates' errors where the kernels are close.
  const double us = 2e-6 * p.M * (double)p.k * p.Kgemm;
  const double rate = p.c % 4 == 0 ? 75.0 : 50.0;       // TFLOP/s; channels that do not start on 16 bytes are fetched one by one
  const bool small = conv_small_f32_applicable(p) || conv_small_f32_splits(p) > 0;
  const double bytes = (double)p.x_bytes + p.w_bytes + 4.0 * p.M * p.k;
  double other = p.r == 3 ? 8.0 + us / rate : 6.0 + (us / rate > bytes / 3e6 ? us / rate : bytes / 3e6);
  if (small && 3.5 + us / 32.0 < other) other = 3.5 + us / 32.0;
  // (The contraction over planes does not come into it: of 60 deep 3x3 stride 2 layers with planes given it takes 0.69 to 1.42,
  // at the mean 1.03 of the time, and lies up to 1.32 times as far from 64-bit sums, 1.12 at the median.)
  // (With the filter cut ahead many a small pointwise layer is as fast on either, 5 to 6 us: those stay.)
  // (a pointwise layer of few channels, which fill a quarter of a chunk, longer: 16->824 stride 2 at 2312 pixels 6.5 us with tiles, 7.6)
  const double margin = p.packed_is_cut && p.r == 1 ? (p.c < 32 ? 4.5 : 3.2) : p.r == 1 || small ? 1.6 : 0.5;
  // no form takes less than a start, an end and a chunk of the cheapest: most small layers are decided without a search for tiles
  if (mode == 1 && fixed_cost(p, p.packed_is_cut != 0) + (p.r == 1 ? 2.4 : 4.1) + margin >= other) return -1;
  const int parts = knob_or(KNOB_F32_PATCH_PARTS, mode == 2 ? 1 : -1);
  double cost = 0.0, split_us = 0.0;
  const int form = cheapest_form(p, forced, parts, &cost, parts == 1 ? nullptr : split, &split_us);
  *us_out = cost;
  if (mode == 2 || cost + margin < other) return form;
  if (split && split->parts > 1 && (split_us + margin >= other || p.c > kMostOverPlanes)) split->parts = 1;
  return -1;
}

namespace {
// Both planes of the filter, a tap's channels filled up to whole pieces of eight.
size_t cut_plane_bytes(const Problem& p) { return ((size_t)p.r * p.s * ((p.c + 7) / 8) * 32 * (size_t)p.k + 255) / 256 * 256; }
}  // namespace

size_t patch_f32_pack_bytes(const Problem& p) { return cut_plane_bytes(p) + 4 * (size_t)p.k; }
// (Whole pieces of eight channels take the same bytes in either order; the channels' words then lie in the trailer's place.)
bool patch_f32_order_fits(const Problem& p) {
  return p.groups == 1 && p.r == p.s && (p.r == 1 || p.r == 3) && p.c % 8 == 0 && 4 * (size_t)p.k <= kPlaneTrailerBytes;
}

namespace {
unsigned* cut_words(const Problem& p, const void* planes) {
  return reinterpret_cast<unsigned*>(static_cast<unsigned char*>(const_cast<void*>(planes)) + cut_plane_bytes(p));
}
}  // namespace

// Cuts the filters of n layers (at most kCutJobs), each into its own p.planes.
hipError_t launch_cut_filters(const Problem* const* layers, int n, hipStream_t stream) {
  if (n < 1 || n > kCutJobs) return hipErrorInvalidValue;
  CutJobs<kCutJobs> jobs;
  jobs.n = n;
  int blocks = 0;
  for (int i = 0; i < n; ++i) {
    const Problem& p = *layers[i];
    if (!p.planes) return hipErrorInvalidValue;         // the ABI layer never plans this kernel without a workspace
    CutJob& j = jobs.job[i];
    j.w = static_cast<const float*>(p.w);
    j.dst = static_cast<unsigned short*>(const_cast<void*>(p.planes));
    j.words = cut_words(p, p.planes);
    j.rows = p.k;
    j.taps = p.r * p.s;
    j.c = p.c;
    const int c8 = (p.c + 7) / 8, row8 = j.taps * c8;
    j.div_c8 = make_fastdiv((uint32_t)c8);
    const int groups = (p.k + CUT_ROWS - 1) / CUT_ROWS;
    j.parts = 256 / groups;
    if (j.parts > (row8 + 15) / 16) j.parts = (row8 + 15) / 16;   // at least two wavefronts' work each
    if (j.parts > 8) j.parts = 8;
    if (j.parts < 1) j.parts = 1;
    j.first_block = blocks;
    blocks += (groups * j.parts + 7) / 8 * 8;
  }
  if (n == 1) {
    CutJobs<1> one;
    one.n = 1;
    one.job[0] = jobs.job[0];
    hipLaunchKernelGGL(cut_filter_kernel<1>, dim3((unsigned)blocks), dim3(64 * CUT_ROWS), 0, stream, one);
  } else {
    hipLaunchKernelGGL(cut_filter_kernel<kCutJobs>, dim3((unsigned)blocks), dim3(64 * CUT_ROWS), 0, stream, jobs);
  }
  return hipGetLastError();
}

hipError_t launch_patch_f32(const Problem& p_in, int form, int parts, hipStream_t stream, const char** variant) {
  Problem p = p_in;
  if (!p.filter_is_cut && !p.packed_is_cut) {
    const Problem* one = &p;
    const hipError_t e = launch_cut_filters(&one, 1, stream);
    if (e != hipSuccess) return e;
  }
  p.w_planes = p.packed_is_cut ? p.w_packed : p.planes;
  p.w_range = cut_words(p, p.w_planes);
  if (parts > 1) return launch_patch_shape<PARTS>(p, form, parts, stream, variant);
  return p.addend ? launch_patch_shape<ADD_LINK>(p, form, 1, stream, variant) : launch_patch_shape<PLAIN>(p, form, 1, stream, variant);
}

}  // namespace glowmi
