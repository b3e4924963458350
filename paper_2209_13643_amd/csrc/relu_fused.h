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
struct PackedTriples { size_t off[13]; };
size_t relu_fused_msb_box_bytes(int parties, size_t n);
int launch_relu_fused_msb(mpc_ctx* c, hipStream_t st, int parties, FusedRelu q, const PackedTriples& g);
