// A kernel's arguments, all of them on their way before the first is wanted.
//
// The compiler reads an argument where it is used.  The arguments of these kernels lie in two to sixteen cache lines (most in
// nine to twelve), none of which is in the scalar cache when a workgroup starts, and a kernel that comes upon one line after the other waits
// for each: three to eight times some 300 cycles before its first load of a tensor (3x3 stride 2 128->128 on 56x56 at batch 16: 1200 of 34300 cycles).
// Asked for together they cost one wait, and the reads that follow find them in the cache.  Measured, times of the whole call with and
// without: 3x3 256->256 on 14x14 at batch 1 8.8 -> 8.4 us, 1x2048x1000 6.4 -> 6.3, small int8 layers 4.3 -> 4.0, a block of four launches
// 35.7 -> 34.6; launched back to back on the same buffers 300 drawn calls take 0.90 of their time.  conv_pw_f32, which asks for its
// filter and its first pixels before it needs most arguments, gained nothing (64->256 + add at batch 32 51.5 -> 51.9) and does without.
#pragma once
#include <hip/hip_runtime.h>

namespace glowmi {

#define GLOWMI_LINE(at) "s_load_dword %0, %1, " #at "\n\t"
#define GLOWMI_LINES2 GLOWMI_LINE(0x0) GLOWMI_LINE(0x40)
#define GLOWMI_LINES3 GLOWMI_LINES2 GLOWMI_LINE(0x80)
#define GLOWMI_LINES4 GLOWMI_LINES3 GLOWMI_LINE(0xc0)
#define GLOWMI_LINES5 GLOWMI_LINES4 GLOWMI_LINE(0x100)
#define GLOWMI_LINES6 GLOWMI_LINES5 GLOWMI_LINE(0x140)
#define GLOWMI_LINES7 GLOWMI_LINES6 GLOWMI_LINE(0x180)
#define GLOWMI_LINES8 GLOWMI_LINES7 GLOWMI_LINE(0x1c0)
#define GLOWMI_LINES9 GLOWMI_LINES8 GLOWMI_LINE(0x200)
#define GLOWMI_LINES10 GLOWMI_LINES9 GLOWMI_LINE(0x240)
#define GLOWMI_LINES11 GLOWMI_LINES10 GLOWMI_LINE(0x280)
#define GLOWMI_LINES12 GLOWMI_LINES11 GLOWMI_LINE(0x2c0)
#define GLOWMI_LINES13 GLOWMI_LINES12 GLOWMI_LINE(0x300)
#define GLOWMI_LINES14 GLOWMI_LINES13 GLOWMI_LINE(0x340)
#define GLOWMI_LINES15 GLOWMI_LINES14 GLOWMI_LINE(0x380)
#define GLOWMI_LINES16 GLOWMI_LINES15 GLOWMI_LINE(0x3c0)
#define GLOWMI_FETCH(n) if constexpr (LINES == n) asm volatile(GLOWMI_LINES##n "s_waitcnt lgkmcnt(0)" : "=&s"(word) : "s"(arguments))

// Cache lines of a kernel's parameters: each lies at the next multiple of its alignment.
template <class... A>
constexpr int argument_lines() {
  size_t at = 0;
  ((at = (at + alignof(A) - 1) / alignof(A) * alignof(A) + sizeof(A)), ...);
  return (int)((at + 63) / 64);
}

// First in a kernel, with its parameters: their sizes say how many lines there are.  (The words themselves are not kept.)  One line (of
// cut_filter_kernel's forms, that for one filter) is asked for by whatever reads it first.
template <class... A>
__device__ __forceinline__ void fetch_arguments(const A&...) {
  typedef const unsigned __attribute__((address_space(4))) * Arguments;
  const Arguments arguments = (Arguments)__builtin_amdgcn_kernarg_segment_ptr();
  constexpr int LINES = argument_lines<A...>();
  static_assert(LINES <= 16, "as many lines as there are forms below");
  unsigned word;
  GLOWMI_FETCH(2);
  GLOWMI_FETCH(3);
  GLOWMI_FETCH(4);
  GLOWMI_FETCH(5);
  GLOWMI_FETCH(6);
  GLOWMI_FETCH(7);
  GLOWMI_FETCH(8);
  GLOWMI_FETCH(9);
  GLOWMI_FETCH(10);
  GLOWMI_FETCH(11);
  GLOWMI_FETCH(12);
  GLOWMI_FETCH(13);
  GLOWMI_FETCH(14);
  GLOWMI_FETCH(15);
  GLOWMI_FETCH(16);
}

#undef GLOWMI_FETCH
#undef GLOWMI_LINES16
#undef GLOWMI_LINES15
#undef GLOWMI_LINES14
#undef GLOWMI_LINES13
#undef GLOWMI_LINES12
#undef GLOWMI_LINES11
#undef GLOWMI_LINES10
#undef GLOWMI_LINES9
#undef GLOWMI_LINES8
#undef GLOWMI_LINES7
#undef GLOWMI_LINES6
#undef GLOWMI_LINES5
#undef GLOWMI_LINES4
#undef GLOWMI_LINES3
#undef GLOWMI_LINES2
#undef GLOWMI_LINE

}  // namespace glowmi
