// Sums and moves across the lanes of a 64-lane wavefront.
#pragma once
#include <hip/hip_runtime.h>

namespace td {

// Reads of tables that no thread of the launch writes, at uniform addresses:
// scalar loads
#if defined(__HIP_DEVICE_COMPILE__)
template <class X>
using uniform_ptr = const __attribute__((address_space(4))) X*;
#else
template <class X>
using uniform_ptr = const X*;
#endif

// Cross-lane moves without LDS. A shuffle is an LDS instruction with an LDS
// round trip in its dependent chain, and the nonlocal phases are such chains:
// six reduction steps per atom and stage. gfx950 exchanges wavefront halves
// and rows of 16 lanes with a register swap; the steps inside a row are DPP
// moves.
struct Pair64 {
  double x, y;
};
__device__ __forceinline__ Pair64 join2(unsigned xl, unsigned xh, unsigned yl, unsigned yh) {
  return Pair64{__hiloint2double((int)xh, (int)xl), __hiloint2double((int)yh, (int)yl)};
}
// x = (a's lower half, b's lower half), y = (a's upper half, b's upper half)
__device__ __forceinline__ Pair64 swap32(double a, double b) {
#if defined(__HIP_DEVICE_COMPILE__)
  const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return join2(l[0], h[0], l[1], h[1]);
#else
  return Pair64{a, b};
#endif
}
// the same for the even and odd rows of 16 lanes
__device__ __forceinline__ Pair64 swap16(double a, double b) {
#if defined(__HIP_DEVICE_COMPILE__)
  const auto l = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto h = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return join2(l[0], h[0], l[1], h[1]);
#else
  return Pair64{a, b};
#endif
}
// DPP controls: lane ^ 1, lane ^ 2 (quad permutations), lane ^ 7 (mirror of
// eight lanes), lane ^ 8 (rotation of a row by eight)
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kXor7 = 0x141, kXor8 = 0x128;
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
#if defined(__HIP_DEVICE_COMPILE__)
  const int l = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
  const int h = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(h, l);
#else
  return v;
#endif
}
// sum over the lanes that differ in bit 5 / in bit 4
__device__ __forceinline__ double sum32(double v) {
  const Pair64 p = swap32(v, v);
  return p.x + p.y;
}
__device__ __forceinline__ double sum16(double v) {
  const Pair64 p = swap16(v, v);
  return p.x + p.y;
}
// sum over groups of eight / of four lanes
__device__ __forceinline__ double sum_quad(double v) {
  v += dpp<kXor2>(v);
  return v + dpp<kXor1>(v);
}
__device__ __forceinline__ double sum_oct(double v) { return sum_quad(v + dpp<kXor7>(v)); }

__device__ __forceinline__ double wave_sum(double v) {
  v = sum16(sum32(v));
  return sum_oct(v + dpp<kXor8>(v));
}

// Wavefront sums of eight values at once by recursive halving: at each of the
// exchanges over lane bits 5, 4, 3 a lane keeps half of its values and sends
// the other half; three more steps finish the sum over bits 2..0. Every lane
// returns the full sum of value (lane >> 3) & 7.
__device__ __forceinline__ double wave_sum8(const double (&v)[8], int lane) {
  double a[4], b[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const Pair64 p = swap32(v[i], v[i + 4]);
    a[i] = p.x + p.y;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const Pair64 p = swap16(a[i], a[i + 2]);
    b[i] = p.x + p.y;
  }
  const bool hi = lane & 8;
  const double keep = hi ? b[1] : b[0], send = hi ? b[0] : b[1];
  return sum_oct(keep + dpp<kXor8>(send));
}

// Wavefront sums of 16 values in the same way over lane bits 5..2 (the last
// exchange goes to lane ^ 7: its low bits are summed over next anyway): every
// lane returns the full sum of value lane >> 2.
__device__ __forceinline__ double wave_sum16(const double (&v)[16], int lane) {
  double a[8], b[4], c[2];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const Pair64 p = swap32(v[i], v[i + 8]);
    a[i] = p.x + p.y;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const Pair64 p = swap16(a[i], a[i + 4]);
    b[i] = p.x + p.y;
  }
  const bool h8 = lane & 8, h4 = lane & 4;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double keep = h8 ? b[i + 2] : b[i], send = h8 ? b[i] : b[i + 2];
    c[i] = keep + dpp<kXor8>(send);
  }
  const double keep = h4 ? c[1] : c[0], send = h4 ? c[0] : c[1];
  return sum_quad(keep + dpp<kXor7>(send));
}

}  // namespace td
