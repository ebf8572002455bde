// What the decompression kernels share: the marker of an escaped residual, scans over the lanes of a
// wavefront, the rounding to a 16-bit output type, buffer descriptors.
#pragma once
#include "comet_kernels.h"

namespace comet {

namespace {

constexpr int32_t kEscape = -32768;
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// ---- DPP: value of another lane of the same 16-lane row (0 where there is none) ----
template <int CTRL, int ROW_MASK, bool BOUND>
__device__ inline int32_t dpp0(int32_t v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, BOUND);
}

// Inclusive scan over runs of lanes.  MODE 0: runs of `width` <= 16 lanes packed
// inside 16-lane rows (pos = position in the run); MODE 1: one run per 32-lane
// half; MODE 2: one run over the whole wavefront.
template <int MODE>
__device__ inline int32_t run_scan(int32_t v, uint32_t pos, uint32_t width) {
    if (MODE == 0) {
        int32_t t;
        t = dpp0<0x111, 0xf, true>(v); if (width > 1u) v += (pos >= 1u) ? t : 0;
        t = dpp0<0x112, 0xf, true>(v); if (width > 2u) v += (pos >= 2u) ? t : 0;
        t = dpp0<0x114, 0xf, true>(v); if (width > 4u) v += (pos >= 4u) ? t : 0;
        t = dpp0<0x118, 0xf, true>(v); if (width > 8u) v += (pos >= 8u) ? t : 0;
        return v;
    }
    v += dpp0<0x111, 0xf, true>(v);
    v += dpp0<0x112, 0xf, true>(v);
    v += dpp0<0x114, 0xf, true>(v);
    v += dpp0<0x118, 0xf, true>(v);
    v += dpp0<0x142, 0xa, false>(v);            // lane 15 of rows 0, 2 into rows 1, 3
    if (MODE == 2) v += dpp0<0x143, 0xc, false>(v);   // lane 31 into rows 2, 3
    return v;
}

// Element type of the output: OUT = 0 fp32, 1 IEEE half, 2 bfloat16.  A 16-bit output is the fp32
// result rounded to nearest, ties to even (NaN stays NaN).
template <int OUT> __device__ inline uint32_t narrow16(float v) {
    if (OUT == 1) return (uint32_t)__builtin_bit_cast(unsigned short, (_Float16)v);
    const uint32_t u = __float_as_uint(v);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x0040u;       // NaN: keep it one
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// buffer descriptor over [p, p + bytes): accesses at offsets >= bytes are dropped (loads give 0)
__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}

}  // namespace

}  // namespace comet
