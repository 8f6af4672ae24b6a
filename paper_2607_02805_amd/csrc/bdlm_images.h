// bdlm_images.h -- LDS row images of bf16 tokens and their operand reads, shared by the kernels
// that stage whole token rows (bdlm_seq16.hip, bdlm_maskw.hip), and decay sums in double
// (bdlm_mix.hip, bdlm_maskw.hip).  Internal.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bdlm_device.h"

namespace bdlm {

// Row images, permuted so that staging and operand reads meet each of 64 banks once, by the lanes
// that move 256 bytes.  (The counters still show conflicts in 17 to 28 % of the sequence
// kernels' LDS cycles, a part of them from weighted tiles written 8 bytes in every 16, which
// are not in these images.)  B, C: 16-byte piece
// c of token t (staging writes whole rows, operand reads 16 tokens by one piece).
template <int NS>
__device__ __forceinline__ int c_at(int t, int c) {
    if constexpr (NS == 128) return t * 16 + (c ^ (4 * (t & 3) + ((t >> 2) & 3)));
    else if constexpr (NS == 64) return t * 8 + (c ^ (4 * ((t >> 1) & 1) + ((t >> 2) & 3)));
    else if constexpr (NS == 32) return t * 4 + (c ^ ((t >> 2) & 3));
    else return t * 2 + (c ^ ((t >> 3) & 1));
}
// x: 16-byte piece c of token t.
__device__ __forceinline__ int x_at(int t, int c) { return t * 8 + (c ^ (2 * ((t >> 1) & 3)) ^ ((t >> 3) & 1)); }

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
// LDS transpose read (gfx950): every lane reads four bf16 at its own 8-byte-aligned
// address, and within each group of 16 lanes, lane 4a + b receives element b of the words
// read by lanes a, a + 4, a + 8 and a + 12 of its group, in that order.  So when lane s
// of group kg reads the quad (token 4kg + s / 4, quad s % 4 of four column quads), lane (kg,
// col) receives column col of tokens 4kg .. 4kg + 3.
__device__ __forceinline__ s16x4 ds_read_tr(const uint2 *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(const_cast<uint2 *>(p)));
}
__device__ __forceinline__ int tr_tok(int lane) { return 4 * (lane >> 4) + ((lane & 15) >> 2); }
// x operand over tokens: lane (grp, col) gets tokens 16 jt + 4 grp .. +3 of column 16 pt + col.
__device__ __forceinline__ s16x4 x_read(const uint4 *sX, int jt, int pt, int lane) {
    const int a = lane & 3;
    return ds_read_tr(reinterpret_cast<const uint2 *>(sX) + 2 * x_at(16 * jt + tr_tok(lane), 2 * pt + (a >> 1)) + (a & 1));
}
__device__ __forceinline__ f32x4 quad_val(s16x4 v) {
    return f32x4{bf16_to_f32(v[0]), bf16_to_f32(v[1]), bf16_to_f32(v[2]), bf16_to_f32(v[3])};
}
__device__ __forceinline__ s16x4 lo4(uint4 v) { return as_s16x4(uint2{v.x, v.y}); }
__device__ __forceinline__ s16x4 hi4(uint4 v) { return as_s16x4(uint2{v.z, v.w}); }

// Inclusive sum of doubles over the wave (wave_inclusive_sum's steps on both halves).
template <int CTRL, int ROW_MASK, bool BOUND_ZERO>
__device__ __forceinline__ double dpp_d(double v) {
    const int2 u = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(double, int2{__builtin_amdgcn_update_dpp(0, u.x, CTRL, ROW_MASK, 0xf, BOUND_ZERO),
                                           __builtin_amdgcn_update_dpp(0, u.y, CTRL, ROW_MASK, 0xf, BOUND_ZERO)});
}
__device__ __forceinline__ double wave_inclusive_sum_d(double v) {
    v += dpp_d<0x111, 0xf, true>(v);
    v += dpp_d<0x112, 0xf, true>(v);
    v += dpp_d<0x114, 0xf, true>(v);
    v += dpp_d<0x118, 0xf, true>(v);
    v += dpp_d<0x142, 0xa, false>(v);
    v += dpp_d<0x143, 0xc, false>(v);
    return v;
}

}  // namespace bdlm
