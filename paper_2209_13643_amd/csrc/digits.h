// Balanced base-256 digits of ring words, as the recoders store them.
#pragma once
#include "common.h"

// Balanced base-256 digits of x: x = sum_j d_j 2^(8j) (mod 2^64), d_j in
// [-128, 127].  Adding 0x80 to every byte position (with carries) and flipping
// the top bit of every byte yields the eight digits as two's-complement bytes.
__device__ __forceinline__ u64 balanced_digits(u64 x)
{
    const u64 h = 0x8080808080808080ull;
    return (x + h) ^ h;
}

// The digits of four words, digit by digit: out[d] holds digit d of w[0..3] in bytes 0..3.
__device__ __forceinline__ void digits_of_4(const u64 (&w)[4], uint32_t (&out)[8])
{
    uint32_t h[2][4];
#pragma unroll
    for (int t = 0; t < 4; ++t) { const u64 d = balanced_digits(w[t]); h[0][t] = (uint32_t)d; h[1][t] = (uint32_t)(d >> 32); }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        // a 4 x 4 byte transpose in eight byte permutes
        const uint32_t x0 = __builtin_amdgcn_perm(h[q][1], h[q][0], 0x05010400), y0 = __builtin_amdgcn_perm(h[q][3], h[q][2], 0x05010400);
        const uint32_t x1 = __builtin_amdgcn_perm(h[q][1], h[q][0], 0x07030602), y1 = __builtin_amdgcn_perm(h[q][3], h[q][2], 0x07030602);
        out[4 * q + 0] = __builtin_amdgcn_perm(y0, x0, 0x05040100); out[4 * q + 1] = __builtin_amdgcn_perm(y0, x0, 0x07060302);
        out[4 * q + 2] = __builtin_amdgcn_perm(y1, x1, 0x05040100); out[4 * q + 3] = __builtin_amdgcn_perm(y1, x1, 0x07060302);
    }
}
