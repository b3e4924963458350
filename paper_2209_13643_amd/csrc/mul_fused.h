// Interface of the one-launch element-wise products (mul_fused.hip).
#pragma once
#include "common.h"

struct FusedMul {
    const u64 *x[3], *y[3], *a[3], *b[3], *c[3];
    u64* z[3];
    u64* box;                            // mul_fused_box_bytes(parties, n) bytes
    size_t n;
    int trunc_bits, mask_from_sign;      // truncation: two parties only; mask_from_sign: y holds sign shares s, the factor is 1 - s
    unsigned tiles;                      // filled by the launcher
};
size_t mul_fused_box_bytes(int parties, size_t n);
int launch_mul_fused(mpc_ctx* c, hipStream_t st, int parties, FusedMul q);

// max-pool backward; triples 1 on 2 n_out words, triples 2 on n_out
struct FusedPoolBwd {
    const u64 *g[3], *s1[3], *s2[3], *a1[3], *b1[3], *c1[3], *a2[3], *b2[3], *c2[3];
    u64* gx[3];
    u64* box;                            // poolbwd_fused_box_bytes(parties, n_out) bytes
    size_t n_out; int H, W, C;
    unsigned tiles;
};
size_t poolbwd_fused_box_bytes(int parties, size_t n_out);
int launch_poolbwd_fused(mpc_ctx* c, hipStream_t st, int parties, FusedPoolBwd q);
