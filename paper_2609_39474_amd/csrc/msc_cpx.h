// Complex arithmetic, the LDS bank swizzle and the XCD-aware block order of the
// transform passes.
#pragma once

#include <hip/hip_runtime.h>

namespace msc {

template <class CT>
struct cpx {
  CT x, y;
};

template <class CT>
__device__ __forceinline__ cpx<CT> cmul(cpx<CT> a, cpx<CT> b) {
#pragma clang fp contract(on)
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <class CT>
__device__ __forceinline__ cpx<CT> cadd(cpx<CT> a, cpx<CT> b) {
  return {a.x + b.x, a.y + b.y};
}
template <class CT>
__device__ __forceinline__ cpx<CT> csub(cpx<CT> a, cpx<CT> b) {
  return {a.x - b.x, a.y - b.y};
}
// multiply by +i (s > 0) or -i (s < 0)
template <class CT>
__device__ __forceinline__ cpx<CT> cmuli(cpx<CT> a, int s) {
  return s > 0 ? cpx<CT>{-a.y, a.x} : cpx<CT>{a.y, -a.x};
}

// XCD-aware order of the column passes: a grid of G blocks, G a multiple of 8
// (the host pads it), is dealt to the 8 XCDs round-robin; block b takes work
// item (b mod 8) G/8 + b/8, so that each XCD gets a contiguous range of items
// (adjacent columns, whose values share cache lines) and its L2 serves them.
__device__ __forceinline__ int xcd_item(int b, int G) { return (G & 7) ? b : (b & 7) * (G >> 3) + (b >> 3); }
__host__ __device__ constexpr int pad8(int n) { return (n + 7) / 8 * 8; }

// Bank swizzle of the intermediate stages: element i of a line is stored at
// i with its position inside a 128-byte row XORed with the row number, so the
// strided writes of the early stages (stride 8 or 4 Ns elements) fall on
// different banks; a bijection within every aligned row group, so a line of
// N >= G elements keeps its footprint.
template <class CT>
__device__ __forceinline__ int lds_swz(int i) {
  constexpr int G = 128 / (int)sizeof(cpx<CT>);  // elements per 128-byte row: 8 (FP64), 16 (FP32)
  return i ^ ((i / G) & (G - 1));
}

}  // namespace msc
