// Pieces of the ABI layer (api.hip) that the other host-side translation units use: the error
// record behind glowmi_last_error(), and "prepare" / "run" halves of the convolution entry points so
// that a caller issuing several layers (sequence.hip) can validate ALL of them before the first launch.
#pragma once
#include "../../include/glowmi.h"
#include "igemm.h"

namespace glowmi {

// Records the message glowmi_last_error() returns on this thread; returns `s`.
glowmi_status fail(glowmi_status s, const char* fmt, ...) __attribute__((format(printf, 2, 3)));

// One validated, planned layer call: everything needed to launch it later without further checks.
struct PreparedCall {
  Problem p;
  Plan plan;
  bool quantized;
};

// Validate the arguments of glowmi_conv2d_chain / glowmi_qconv2d_chain and plan the launch (tile,
// split of the reduction given the workspace).  Nothing is launched.  w_planes: the filter's bf16 planes made
// ahead of time (glowmi_conv2d_pack_filter), or null.  parts: whether conv_patch_f32 may take a reduction in parts.
glowmi_status prepare_conv2d_chain(const float* x, const float* w, const float* bias, float* y,
                                   const glowmi_conv_desc* d, const glowmi_chain* chain, void* workspace,
                                   size_t workspace_bytes, PreparedCall* out, const void* w_planes = nullptr, bool parts = true);
glowmi_status prepare_qconv2d_chain(const int8_t* x, glowmi_qparam xq, const int8_t* w, glowmi_qparam wq,
                                    const int32_t* bias, int8_t* y, glowmi_qparam yq, const glowmi_conv_desc* d,
                                    const glowmi_chain* chain, void* workspace, size_t workspace_bytes,
                                    PreparedCall* out);
// Bytes for the planes of a layer's filter where the planner takes the kernel that cuts it into an order of its own
// (conv_patch_f32), else 0.
size_t conv2d_cut_bytes(const glowmi_conv_desc* d);
// What glowmi_conv2d_workspace_bytes names, without the parts of conv_patch_f32's reductions: the layers of a sequence run without them, so that
// what a layer runs on does not depend on how much scratch its neighbours want.
size_t conv2d_whole_bytes(const glowmi_conv_desc* d);
// One launch for the filters of n (at most kCutJobs) prepared calls of that kernel, each with a place of its own (p.planes).
glowmi_status run_cuts(PreparedCall* const* calls, int n, hipStream_t stream);
// Launch a prepared call on `stream`.
glowmi_status run_prepared(const PreparedCall& call, hipStream_t stream);
// Launches three prepared calls that follow each other in a sequence as one kernel that writes the third's output alone, where there
// is one for them; false, and nothing is launched, where there is none.
bool run_in_one_launch(const PreparedCall* calls, hipStream_t stream, glowmi_status* st);

}  // namespace glowmi
