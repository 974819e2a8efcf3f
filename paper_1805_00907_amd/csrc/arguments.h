// A kernel's arguments, all of them on their way before the first is wanted.
//
// The compiler reads an argument where it is used.  The arguments of these kernels lie in eight and more cache lines, none of which
// is in the scalar cache when a workgroup starts, and a kernel that comes upon one line after the other waits for each: three to
// eight times some 300 cycles before its first load of a tensor (3x3 stride 2 128->128 on 56x56 at batch 16: 1200 of 34300 cycles).
// Asked for together they cost one wait, and the reads that follow find them in the cache.  Measured, times of the whole call with and
// without: 3x3 256->256 on 14x14 at batch 1 8.8 -> 8.4 us, 1x2048x1000 6.4 -> 6.3, small int8 layers 4.3 -> 4.0, a block of four launches
// 35.7 -> 34.6; launched back to back on the same buffers 300 drawn calls take 0.90 of their time.  conv_pw_f32, which asks for its
// filter and its first pixels before it needs most arguments, gained nothing (64->256 + add at batch 32 51.5 -> 51.9) and does without.
#pragma once
#include <hip/hip_runtime.h>

namespace glowmi {

#define GLOWMI_LINE(at) "s_load_dword %0, %1, " #at "\n\t"
#define GLOWMI_LINES4(a, b, c, d) GLOWMI_LINE(a) GLOWMI_LINE(b) GLOWMI_LINE(c) GLOWMI_LINE(d)
#define GLOWMI_FETCH(lines) asm volatile(lines "s_waitcnt lgkmcnt(0)" : "=&s"(word) : "s"(arguments))

// First in a kernel, with its parameters: their sizes say how many lines there are.  (The words themselves are not kept.)
template <class... A>
__device__ __forceinline__ void fetch_arguments(const A&...) {
  typedef const unsigned __attribute__((address_space(4))) * Arguments;
  const Arguments arguments = (Arguments)__builtin_amdgcn_kernarg_segment_ptr();
  constexpr int LINES = (int)(((sizeof(A) + ...) + 63) / 64);
  unsigned word;
  if constexpr (LINES >= 16)
    GLOWMI_FETCH(GLOWMI_LINES4(0x0, 0x40, 0x80, 0xc0) GLOWMI_LINES4(0x100, 0x140, 0x180, 0x1c0) GLOWMI_LINES4(0x200, 0x240, 0x280, 0x2c0)
                     GLOWMI_LINES4(0x300, 0x340, 0x380, 0x3c0));
  else if constexpr (LINES >= 12)
    GLOWMI_FETCH(GLOWMI_LINES4(0x0, 0x40, 0x80, 0xc0) GLOWMI_LINES4(0x100, 0x140, 0x180, 0x1c0) GLOWMI_LINES4(0x200, 0x240, 0x280, 0x2c0));
  else if constexpr (LINES >= 10)
    GLOWMI_FETCH(GLOWMI_LINES4(0x0, 0x40, 0x80, 0xc0) GLOWMI_LINES4(0x100, 0x140, 0x180, 0x1c0) GLOWMI_LINE(0x200) GLOWMI_LINE(0x240));
  else if constexpr (LINES == 9)
    GLOWMI_FETCH(GLOWMI_LINES4(0x0, 0x40, 0x80, 0xc0) GLOWMI_LINES4(0x100, 0x140, 0x180, 0x1c0) GLOWMI_LINE(0x200));
  else if constexpr (LINES >= 8)
    GLOWMI_FETCH(GLOWMI_LINES4(0x0, 0x40, 0x80, 0xc0) GLOWMI_LINES4(0x100, 0x140, 0x180, 0x1c0));
  else if constexpr (LINES >= 4)
    GLOWMI_FETCH(GLOWMI_LINES4(0x0, 0x40, 0x80, 0xc0));
  else if constexpr (LINES >= 2)
    GLOWMI_FETCH(GLOWMI_LINE(0x0) GLOWMI_LINE(0x40));
}

#undef GLOWMI_FETCH
#undef GLOWMI_LINES4
#undef GLOWMI_LINE

}  // namespace glowmi
