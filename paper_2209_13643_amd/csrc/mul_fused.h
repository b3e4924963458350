// Interface of the one-launch element-wise products (mul_fused.hip).
#pragma once
#include "common.h"
#include "overlap.h"

struct FusedMul {
    const u64 *x[3], *y[3], *a[3], *b[3], *c[3];
    u64* z[3];
    u64* box;                            // mul_fused_box_bytes(parties, n) bytes
    size_t n;
    int trunc_bits, mask_from_sign;      // truncation: two parties only; mask_from_sign: y holds sign shares s, the factor is 1 - s
    unsigned tiles;                      // filled by the launcher
};
// whether the call may run as one launch (overlap.h)
inline bool mul_outputs_apart(int parties, const FusedMul& q)
{
    Spans<15> in; Spans<3> out;
    for (int i = 0; i < parties; ++i) {
        for (const u64* p : { q.x[i], q.y[i], q.a[i], q.b[i], q.c[i] }) in.words(p, q.n);
        out.words(q.z[i], q.n);
    }
    return outputs_apart(out, in, true);
}
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
inline bool poolbwd_outputs_apart(int parties, const FusedPoolBwd& q)
{
    Spans<27> in; Spans<3> out;
    for (int i = 0; i < parties; ++i) {
        for (const u64* p : { q.g[i], q.s2[i], q.a2[i], q.b2[i], q.c2[i] }) in.words(p, q.n_out);
        for (const u64* p : { q.s1[i], q.a1[i], q.b1[i], q.c1[i] }) in.words(p, 2 * q.n_out);
        out.words(q.gx[i], 4 * q.n_out);
    }
    return outputs_apart(out, in, false);
}
size_t poolbwd_fused_box_bytes(int parties, size_t n_out);
int launch_poolbwd_fused(mpc_ctx* c, hipStream_t st, int parties, FusedPoolBwd q);

// masked rescale of a three-party sharing (in place): party 0 opens z + r + 2^62 and shifts, the others negate their share of r >> bits
struct FusedTrunc3 {
    u64* z[3]; const u64 *r[3], *rt[3];
    u64* box;                            // trunc3_fused_box_bytes(n) bytes
    size_t n; int bits;
    unsigned tiles;
};
inline bool trunc3_outputs_apart(const FusedTrunc3& q)
{
    Spans<9> in; Spans<3> out;
    for (int i = 0; i < 3; ++i) { in.words(q.z[i], q.n); in.words(q.r[i], q.n); in.words(q.rt[i], q.n); out.words(q.z[i], q.n); }
    return outputs_apart(out, in, true);
}
size_t trunc3_fused_box_bytes(size_t n);
int launch_trunc3_fused(mpc_ctx* c, hipStream_t st, FusedTrunc3 q);
