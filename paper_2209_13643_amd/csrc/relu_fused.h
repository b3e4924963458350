// Interface of the one-launch secure ReLU (relu_fused.hip) to the entry points (relu.hip, three_party.hip).
#pragma once
#include "common.h"

struct FusedReluParty {
    const u64 *x, *r, *r1;               // input share, A2B mask (three parties: r to party + 1, r1 to party + 2)
    const u64 *ta, *tb, *tc;             // AND triples
    const u8* rb; const u64* ra;         // B2A
    const u64 *ma, *mb, *mc;             // select
    u64* y; u8* s_bit; u64* s_arith;     // outputs (the last two optional)
};
struct FusedRelu {
    FusedReluParty p[3];
    u64* box;                            // receive buffers, relu_fused_(msb_)box_bytes(parties, n) bytes
    size_t n;
    unsigned tiles;                      // filled by the launcher
};
size_t relu_fused_box_bytes(int parties, size_t n);
int launch_relu_fused(mpc_ctx* c, hipStream_t st, int parties, FusedRelu q, int topo);
// the sign-only chain; offsets of the triples in the packed buffers
struct PackedTriples { size_t off[13]; size_t words[6]; };      // words[l]: packed words of level l
size_t relu_fused_msb_box_bytes(int parties, size_t n);
int launch_relu_fused_msb(mpc_ctx* c, hipStream_t st, int parties, FusedRelu q, const PackedTriples& g);
// 2x2 max-pool of [B][H][W][C] (n_out = B * H/2 * W/2 * C outputs); material of the two conversions in m1 (2 n_out
// elements) and m2 (n_out); x, y and the sign shares of FusedReluParty are not used; s1, s2 optional
struct FusedPool {
    FusedReluParty m1[3], m2[3];
    const u64* x[3]; u64* y[3]; u64 *s1[3], *s2[3];
    u64* box;                            // maxpool_fused_box_bytes(parties, packed, n_out) bytes
    size_t n_out; int H, W, C;
    unsigned tiles;                      // filled by the launcher
};
size_t maxpool_fused_box_bytes(int parties, bool packed, size_t n_out);
// g1, g2: packed layouts of the two conversions (sign-only chain), or null (whole words)
int launch_maxpool_fused(mpc_ctx* c, hipStream_t st, int parties, FusedPool q, int topo, const PackedTriples* g1, const PackedTriples* g2);
