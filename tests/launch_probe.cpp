// What a call hands to the runtime, without a GPU: this program's own hipLaunchKernel, hipFuncSetAttribute and what a
// launch needs beside them stand in for the runtime's, note what they are given and launch nothing (launch_probe.py builds and drives it).
//
// Reads commands, one a line, and answers each with one line.
//   knob NAME VALUE                    -> ok
//   reset                              -> ok
//   seq QUANTIZED LAYERS ADD n h w c   -> status, the variant's name, then for every launch  name|dynamic LDS bytes|limit set for that kernel
//       followed by LAYERS times  k r  (stride 1, padding r / 2); ADD: bit i adds the sequence input in layer i
//   versus NAME VALUE REPEATS          -> median times of the last seq command's call, in nanoseconds: with that knob set, with none set
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstdint>
#include <iostream>
#include <map>
#include <sstream>
#include <string>
#include <vector>

#include "../include/glowmi.h"

namespace {
struct Launch {
  std::string name;
  size_t lds, limit;
};
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;           // filled before main, by the library's own initialisation
  return m;
}
std::map<const void*, size_t> limits;
std::vector<Launch> launches;
size_t pushed;
bool note = true;

void* fake(uintptr_t at) { return reinterpret_cast<void*>(at << 36); }   // aligned, disjoint, never dereferenced
}  // namespace

extern "C" {
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*) {
  names()[host] = device;
}
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute a, int value) {
  if (a == hipFuncAttributeMaxDynamicSharedMemorySize) limits[f] = (size_t)value;
  return hipSuccess;
}
// (a launch passes its extents to the kernel's host function this way)
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t lds, hipStream_t) {
  pushed = lds;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t* lds, hipStream_t*) {
  *lds = pushed;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t lds, hipStream_t) {
  if (note) launches.push_back({names()[f], lds, limits.count(f) ? limits[f] : 0});
  return hipSuccess;
}
hipError_t hipGetDevice(int* device) {
  *device = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* value, hipDeviceAttribute_t, int) {
  *value = 256;                                          // (the library asks for the number of compute units alone)
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* blocks, const void*, int, size_t) {
  *blocks = 2;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
}

int main() {
  std::vector<glowmi_seq_layer> layers;
  std::string line;
  bool quantized = true;
  auto call = [&]() {
    const size_t arena = glowmi_seq_arena_bytes(layers.data(), (int32_t)layers.size(), quantized);
    if (quantized)
      return glowmi_seq_qconv2d(static_cast<const int8_t*>(fake(1)), {0.03f, 3}, layers.data(), (int32_t)layers.size(),
                                static_cast<int8_t*>(fake(2)), fake(3), arena, nullptr);
    return glowmi_seq_conv2d(static_cast<const float*>(fake(1)), layers.data(), (int32_t)layers.size(), static_cast<float*>(fake(2)), fake(3),
                             arena, nullptr);
  };
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    std::string what;
    in >> what;
    if (what == "knob") {
      std::string name;
      int value;
      in >> name >> value;
      std::cout << (glowmi_tuning_set(name.c_str(), value) == GLOWMI_OK ? "ok" : "no such knob") << std::endl;
    } else if (what == "reset") {
      glowmi_tuning_reset();
      std::cout << "ok" << std::endl;
    } else if (what == "seq") {
      int n_layers, add, n, h, w, c;
      in >> quantized >> n_layers >> add >> n >> h >> w >> c;
      layers.clear();
      for (int i = 0; i < n_layers; ++i) {
        int k, r;
        in >> k >> r;
        glowmi_seq_layer l = {};
        l.desc = {n, h, w, c, k, r, r, 1, 1, r / 2, r / 2, r / 2, r / 2, 1};
        l.w = fake(16 + i);
        l.wq = {0.01f, 0};
        l.yq = {0.04f, -5};
        l.act = GLOWMI_ACT_RELU;
        l.add_input = add >> i & 1;
        layers.push_back(l);
        c = k;
      }
      launches.clear();
      std::cout << call() << ' ' << glowmi_last_variant();
      for (const Launch& l : launches) std::cout << ' ' << l.name << '|' << l.lds << '|' << l.limit;
      std::cout << std::endl;
    } else if (what == "versus") {
      std::string name;
      int value, repeats;
      in >> name >> value >> repeats;
      note = false;
      std::vector<long long> ns[2];
      for (int i = 0; i < 2 * repeats; ++i) {            // in turn, call by call
        glowmi_tuning_reset();
        if (i % 2 == 0) glowmi_tuning_set(name.c_str(), value);
        const auto a = std::chrono::steady_clock::now();
        call();
        ns[i % 2].push_back(std::chrono::duration_cast<std::chrono::nanoseconds>(std::chrono::steady_clock::now() - a).count());
      }
      note = true;
      for (auto& v : ns) std::nth_element(v.begin(), v.begin() + repeats / 2, v.end());
      std::cout << ns[0][repeats / 2] << ' ' << ns[1][repeats / 2] << std::endl;
    } else {
      std::cout << "?" << std::endl;
    }
  }
}
