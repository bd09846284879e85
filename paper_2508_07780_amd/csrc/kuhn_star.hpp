// Row sums of the assembled Kuhn star from a box of nodes in LDS, shared by the resident and the step kernels.
#pragma once

#include "resident.hpp"

namespace dd {
namespace {

// The value as something the compiler does not know: what is derived from it (unpacked indices,
// addresses, flags, table entries) is formed again in every step instead of being kept in
// registers for the whole solve, which would take several times the registers there are.
__device__ __forceinline__ uint32_t fresh(uint32_t v) { asm volatile("" : "+v"(v)); return v; }
__device__ __forceinline__ int fresh(int v) { asm volatile("" : "+v"(v)); return v; }
// A result formed here, not moved past a barrier with its operands held until then.
__device__ __forceinline__ void here(float& v) { asm volatile("" : "+v"(v)); }
// w * (the star's value n h / 6), the sign in the instruction; n = 0: nothing
template <int N, class Args>
__device__ __forceinline__ float star_mul(const Args& a, float w) {
  constexpr int m = N < 0 ? -N : N;
  const float v = m == 1 ? a.sb1 : m == 2 ? a.sb2 : m == 4 ? a.sb4 : m == 6 ? a.sb6 : a.sb12;
  return w * (N < 0 ? -v : v);
}
template <int N, class Args>
__device__ __forceinline__ float star_fma(const Args& a, float w, float t) {
  constexpr int m = N < 0 ? -N : N;
  const float v = m == 1 ? a.sb1 : m == 2 ? a.sb2 : m == 4 ? a.sb4 : m == 6 ? a.sb6 : a.sb12;
  return __builtin_fmaf(w, N < 0 ? -v : v, t);
}

// Args: a kernel's arguments with the star's values (StarValues) as sk1 .. sb12.
// Slot S of the row sums of the Kuhn star at LDS box node p: r += K u, and the div-div row of
// (eps - 1) u (forward, w = eps - 1) or q += B u (adjoint).  The star's zero entries are left out;
// the order of the operations is that of the step kernels'.
template <int S, bool ADJ, class Args>
__device__ __forceinline__ void star_slot(const Args& a, const float4& x, float (&r)[3], float (&q)[3]) {
#pragma clang fp contract(off)
  constexpr StarSlot s = kStar[S];
  if (s.k) {
    const float k = s.k == 6 ? a.sk6 : -a.sk1;
    r[0] = __builtin_fmaf(k, x.x, r[0]);
    r[1] = __builtin_fmaf(k, x.y, r[1]);
    r[2] = __builtin_fmaf(k, x.z, r[2]);
  }
  const float w0 = ADJ ? x.x : x.w * x.x, w1 = ADJ ? x.y : x.w * x.y, w2 = ADJ ? x.z : x.w * x.z;
  float (&o)[3] = ADJ ? q : r;
  float t[3];
#define DD_STAR_ROW(c)                                                       \
  t[c] = s.b[3 * c + 1] ? star_mul<s.b[3 * c + 1]>(a, w1) : 0.f;             \
  if (s.b[3 * c]) t[c] = s.b[3 * c + 1] ? star_fma<s.b[3 * c]>(a, w0, t[c]) : star_mul<s.b[3 * c]>(a, w0); \
  if (s.b[3 * c + 2]) t[c] = star_fma<s.b[3 * c + 2]>(a, w2, t[c]);          \
  o[c] += t[c];
  DD_STAR_ROW(0) DD_STAR_ROW(1) DD_STAR_ROW(2)
#undef DD_STAR_ROW
}

template <int S, int M, bool ADJ>
struct StarSums {
  // M nodes at a time; two slots' loads in flight
  template <class Args>
  static __device__ __forceinline__ void run(const Args& a, const float4* box, const int* cell, int sx, int sxy, float (*r)[3],
                                             float (*q)[3]) {
    constexpr int S2 = S + 1 < 15 ? S + 1 : S;
    float4 x[M], y[M];
#pragma unroll
    for (int j = 0; j < M; ++j) {
      const float4* p = box + fresh(cell[j]);
      x[j] = p[kStar[S].x + sx * kStar[S].y + sxy * kStar[S].z];
      y[j] = p[kStar[S2].x + sx * kStar[S2].y + sxy * kStar[S2].z];
    }
#pragma unroll
    for (int j = 0; j < M; ++j) {
      star_slot<S, ADJ>(a, x[j], r[j], q[j]);
      if (S2 > S) star_slot<S2, ADJ>(a, y[j], r[j], q[j]);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        here(r[j][c]);
        if (ADJ) here(q[j][c]);
      }
    }
    StarSums<S + 2, M, ADJ>::run(a, box, cell, sx, sxy, r, q);
  }
};
template <int M, bool ADJ>
struct StarSums<16, M, ADJ> {
  template <class Args>
  static __device__ __forceinline__ void run(const Args&, const float4*, const int*, int, int, float (*)[3], float (*)[3]) {}
};

}  // namespace
}  // namespace dd
