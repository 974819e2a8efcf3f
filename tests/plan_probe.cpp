// What the planner chooses for a call, without launching it: the prepare half of the convolution entry points and the
// planners behind the FullyConnected ones, for tests that need no GPU (plan_probe.py builds and loads this).
#include <algorithm>
#include <chrono>
#include <cstdint>
#include <cstring>
#include <vector>

#include "../paper_1805_00907_amd/csrc/api_internal.h"

using namespace glowmi;

namespace {
void* fake(uintptr_t at) { return reinterpret_cast<void*>(at << 36); }   // aligned, disjoint, never dereferenced

size_t used(const Problem& p, const Plan& pl) {
  return pl.pack_bytes + (pl.split_k > 1 ? (size_t)pl.split_k * (size_t)p.M * (size_t)p.k * 4u : 0u);
}

// Median nanoseconds of planning an fp32 call with room for whatever it likes, in turn: with that switch, with none.
template <typename PlanFn>
void versus(const char* knob, int32_t value, int32_t repeats, int64_t* out, PlanFn plan) {
  std::vector<int64_t> ns[2];
  for (int32_t i = 0; i < 2 * repeats; ++i) {
    glowmi_tuning_reset();
    if (i % 2 == 0) glowmi_tuning_set(knob, value);
    const auto a = std::chrono::steady_clock::now();
    plan();
    ns[i % 2].push_back(std::chrono::duration_cast<std::chrono::nanoseconds>(std::chrono::steady_clock::now() - a).count());
  }
  glowmi_tuning_reset();
  for (int t = 0; t < 2; ++t) {
    std::nth_element(ns[t].begin(), ns[t].begin() + repeats / 2, ns[t].end());
    out[t] = ns[t][repeats / 2];
  }
}
}  // namespace

extern "C" {

struct ProbePlan {
  int32_t status, kernel, tile, split_k;
  uint64_t workspace;    // bytes the planned launch uses
};

// mode: 0 fp32, 1 int8.  ws_bytes: of the workspace handed over, 0: none.
void probe_conv(const glowmi_conv_desc* d, int32_t mode, int32_t addend, int32_t packed, int32_t w_offset, uint64_t ws_bytes,
                ProbePlan* out) {
  PreparedCall call;
  glowmi_chain chain;
  std::memset(&chain, 0, sizeof(chain));
  chain.addend = addend ? fake(5) : nullptr;
  chain.addend_q.scale = 0.03f;
  chain.act = GLOWMI_ACT_RELU;
  void* ws = ws_bytes ? fake(6) : nullptr;
  if (mode == 0) {
    out->status = prepare_conv2d_chain(static_cast<const float*>(fake(1)), static_cast<const float*>(fake(2)), nullptr,
                                       static_cast<float*>(fake(4)), d, &chain, ws, ws_bytes, &call, packed ? fake(7) : nullptr);
  } else {
    const glowmi_qparam xq = {0.03f, 3}, wq = {0.01f, w_offset}, yq = {0.04f, -5};
    out->status = prepare_qconv2d_chain(static_cast<const int8_t*>(fake(1)), xq, static_cast<const int8_t*>(fake(2)), wq, nullptr,
                                        static_cast<int8_t*>(fake(4)), yq, d, &chain, ws, ws_bytes, &call);
  }
  if (out->status != GLOWMI_OK) return;
  out->kernel = call.plan.kernel;
  out->tile = call.plan.tile;
  out->split_k = call.plan.split_k;
  out->workspace = used(call.p, call.plan);
}

// The FullyConnected calls of those extents with a workspace as large as they like.
static void fill(Problem& p, int32_t M, int32_t K, int32_t N) {
  std::memset(&p, 0, sizeof(p));
  p.allow_pack = 1;
  p.n = M; p.h = p.w_ = 1; p.c = p.cg = K; p.k = p.kg = N; p.r = p.s = 1; p.oh = p.ow = 1;
  p.stride_h = p.stride_w = 1; p.groups = 1; p.M = M; p.Kgemm = K; p.split_k = 1; p.b_is_kn = 1;
  p.div_ohow = p.div_ow = p.div_s = make_fastdiv(1);
  p.div_cg = make_fastdiv((uint32_t)K);
  p.x = fake(1); p.w = fake(2); p.y = fake(4);
}

void probe_fc(int32_t M, int32_t K, int32_t N, ProbePlan* out) {
  Problem p;
  fill(p, M, K, N);
  p.x_bytes = 4u * (uint32_t)M * (uint32_t)K; p.w_bytes = 4u * (uint32_t)K * (uint32_t)N;
  const Plan pl = plan_f32(p, true);
  out->status = GLOWMI_OK;
  out->kernel = pl.kernel;
  out->tile = pl.tile;
  out->split_k = pl.split_k;
  out->workspace = used(p, pl);
}

void probe_conv_versus(const glowmi_conv_desc* d, int32_t packed, const char* knob, int32_t value, int32_t repeats, int64_t* out) {
  ProbePlan plan;
  versus(knob, value, repeats, out, [&]() { probe_conv(d, 0, 0, packed, 0, (uint64_t)1 << 36, &plan); });
}
void probe_fc_versus(int32_t M, int32_t K, int32_t N, const char* knob, int32_t value, int32_t repeats, int64_t* out) {
  ProbePlan plan;
  versus(knob, value, repeats, out, [&]() { probe_fc(M, K, N, &plan); });
}

void probe_qfc(int32_t M, int32_t K, int32_t N, int32_t w_offset, ProbePlan* out) {
  Problem p;
  fill(p, M, K, N);
  p.x_bytes = (uint32_t)M * (uint32_t)K; p.w_bytes = (uint32_t)K * (uint32_t)N;
  p.w_off = w_offset; p.mant = 1 << 30; p.shift = 31; p.lo = -128; p.hi = 127;
  const Plan pl = plan_i8(p, true);
  out->status = GLOWMI_OK;
  out->kernel = pl.kernel;
  out->tile = pl.tile;
  out->split_k = pl.split_k;
  out->workspace = used(p, pl);
}

const char* probe_kernel_name(int32_t kernel) {
  switch (kernel) {
    case KERNEL_TILED: return "tiled";
    case KERNEL_SKINNY16: return "skinny16";
    case KERNEL_SMALL: return "small";
    case KERNEL_SMALL_SPLIT: return "small_split";
    case KERNEL_SMALLC: return "smallc";
    case KERNEL_PW: return "pw";
    case KERNEL_K3C64: return "k3c64";
    case KERNEL_FC_SMALL: return "fc_small";
    case KERNEL_WIDE: return "wide";
    case KERNEL_K3: return "k3";
    case KERNEL_P3: return "p3";
    case KERNEL_DW: return "dw";
    case KERNEL_FC_ROWS: return "fc_rows";
    case KERNEL_FC_TILES: return "fc_tiles";
    case KERNEL_FEW: return "few";
    case KERNEL_SHORT: return "short";
    case KERNEL_FC_FEW: return "fc_few";
    case KERNEL_PATCH: return "patch";
    default: return "?";
  }
}

}  // extern "C"
