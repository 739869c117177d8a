// Filtered rows between the fused normalise + filter kernels and the blocked
// backprojection: 16-bit samples of 8 slices side by side,
//   rows[z / 8][angle][plane][bin][z % 8],
// so that a window of bins is one contiguous piece for 8 slices, read 16 bytes
// per lane straight into LDS.  FP32 rows take two FP16 planes (the rounded
// sample and 2^11 times what it misses), the same 4 bytes.  In sinogram order the 64 rows
// of a window lie a power of two apart: the loads then queue on few sets of the
// first-level cache (they cost 12 to 30 ms of 128 rows of the 2048-cubed scan).
// Without room for whole blocks, fewer than 8 slices lie in one block as wide as
// there are.
#pragma once

#include "tp_internal.h"

namespace tp {
namespace {

enum { kStF16 = 0, kStBF16 = 1, kStF32 = 2 };

// Per storage type: row planes, weight planes, angles per staged block (FP32 rows
// at 4: 16 slices of 256 x 256 from 180 angles 0.060 ms, at 8 0.053).
template <int ST> struct Blocked;
template <> struct Blocked<kStF16> { static constexpr int PB = 1, PA = 1, A = 8; };
template <> struct Blocked<kStBF16> { static constexpr int PB = 1, PA = 2, A = 8; };
template <> struct Blocked<kStF32> { static constexpr int PB = 2, PA = 2, A = 8; };

// A power of two that puts the rows high in FP16's range: they stay below 7
// (13.82 = -ln 1e-6 times the filters' absolute sum of at most 1/2), 2^12 times
// them below 65504.
constexpr float kRowScale = 4096.0f;

// Sample v of bin j: `row` points at (z / 8, angle, plane 0, bin 0, z % 8) of
// blocks `wide` slices wide.
template <int ST> __device__ __forceinline__ void store_blocked(uint16_t* row, int n, int wide, int j, float v) {
    const int at = __mul24(j, wide);
    if constexpr (ST == kStF16) {
        row[at] = __half_as_ushort(__float2half_rn(v));
    } else if constexpr (ST == kStBF16) {
        const float b = __uint_as_float(static_cast<uint32_t>(f32_to_bf16_rne(v)) << 16);
        row[at] = __half_as_ushort(__float2half_rn(b * kRowScale));
    } else {
        const float s = v * kRowScale;
        const __half hi = __float2half_rn(s);
        row[at] = __half_as_ushort(hi);
        row[n * wide + at] = __half_as_ushort(__float2half_rn((s - __half2float(hi)) * kLowScale));
    }
}

}  // namespace
}  // namespace tp
