// What the 256 x 256 forward and adjoint kernels share: the split of a stamp
// over a 1,024-thread workgroup and the LDS layout of its exchanges (each
// transform stage of the adjoint is the forward's, run backwards).
#pragma once

#include "gfc_device.hpp"

namespace gfc {

namespace w256 {
constexpr int W = 256;
constexpr int NC = W / 2;           // packed columns
constexpr int D = 8;                // column decimation: lane (c, h) takes rows k_y = 8m + h
constexpr int M = W / D;            // bins per lane in the column phase
constexpr int BLOCK = NC * D;       // 1,024 threads
constexpr int NWAVE = BLOCK / 64;
constexpr int HROWS = W / 2;        // rows per half of the stamp
// LDS has 32 banks of 4 bytes and serves a 64-bit access 16 lanes at a time:
// the 16 lanes are conflict-free when their float2 addresses differ mod 16.
// Row stride of a half, TS = 2 (mod 16): lanes (column c', h) write rows
// 8k + h, addresses 2 h + c' (mod 16); lanes (row y', r) of the row phase
// read columns 8 m + r (and 128 - 8 m - r): 2 y' +- r.
constexpr int TS = 130;
// Slots of the wavefront-private exchanges: entry (i, j) of slot s at
// s * S + 9 i + j.  Column combine (slot = column c', j = h), S = 8 (mod 16):
// writes 8 c' + h, reads 8 c' + 9 h.  Row stage (slot = row y', j = r),
// S = 2 (mod 16): writes 2 y' + r, reads 2 y' + 9 r.
constexpr int CXS = 72;
constexpr int RXS = 82;
// Row stride of the combine twiddle table (float2): odd, so rows h start in
// distinct banks.
constexpr int TWC = 33;
constexpr int LDS_F2 = HROWS * TS;  // 133 KB
static_assert(NWAVE * 8 * CXS <= LDS_F2, "the column exchange slices lie in the half buffer");
static_assert(8 * RXS <= 8 * TS && (8 * TS) % 16 == 0, "a row exchange slice lies in its wavefront's rows");
}  // namespace w256

// Orders a wavefront's LDS accesses across this point (they execute in
// order on the hardware; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) v2f* GlobalF2;

__device__ __forceinline__ float2 ld2(GlobalF2 a, int i) {
  const v2f v = a[i];
  return make_float2(v.x, v.y);
}

}  // namespace gfc
