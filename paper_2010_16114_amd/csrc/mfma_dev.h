// mfma_dev.h -- device helpers shared by the int8 matrix-core kernels (mfma.hip,
// mfma_dense.hip).
#pragma once
#include "device_common.h"

namespace cox {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kLimbs = 3;
constexpr int kQBits = 22;       // |R| <= 2^22 keeps the top limb within int8

// The three signed limbs of R, R = d0 + 256 d1 + 65536 d2 (|R| <= 2^22).
__device__ __forceinline__ void split_limbs(int R, int& d0, int& d1, int& d2)
{
    d0 = ((R + 128) & 255) - 128;
    const int R1 = (R - d0) >> 8;
    d1 = ((R1 + 128) & 255) - 128;
    d2 = (R1 - d1) >> 8;
}

// Allele-count bytes -> int8 counts.  FP8 E4M3 codes of 0, 1, 2 are 0x00, 0x38,
// 0x40, whose top three bits are the count itself (000, 001, 010); other codes
// are rejected before any matrix-core pass runs.
template <int XT>
__device__ __forceinline__ uint32_t counts4(uint32_t w)
{
    if constexpr (XT == XT_FP8)
        return (w >> 5) & 0x07070707u;
    else
        return w;
}

// int8 counts of a raw run.
template <int XT>
__device__ __forceinline__ v4i decode_a(v4i raw)
{
    v4i v;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = (int)counts4<XT>((uint32_t)raw[q]);
    return v;
}

// Byte transpose of a 4 x 4 block: d[r] holds bytes (x_r0, x_r1, x_r2, x_r3);
// o[c] receives (x_0c, x_1c, x_2c, x_3c).  __builtin_amdgcn_perm(hi, lo, sel)
// picks byte sel_k of the 8-byte value hi:lo for result byte k.
__device__ __forceinline__ void transpose4x4(const uint32_t (&d)[4], uint32_t (&o)[4])
{
    const uint32_t lo01 = __builtin_amdgcn_perm(d[1], d[0], 0x05010400u);  // x00 x10 x01 x11
    const uint32_t hi01 = __builtin_amdgcn_perm(d[1], d[0], 0x07030602u);  // x02 x12 x03 x13
    const uint32_t lo23 = __builtin_amdgcn_perm(d[3], d[2], 0x05010400u);  // x20 x30 x21 x31
    const uint32_t hi23 = __builtin_amdgcn_perm(d[3], d[2], 0x07030602u);  // x22 x32 x23 x33
    o[0] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);                 // x00 x10 x20 x30
    o[1] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);                 // x01 x11 x21 x31
    o[2] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
    o[3] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
}

}  // namespace cox
