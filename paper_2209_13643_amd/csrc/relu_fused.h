// Interface of the one-launch secure ReLU (relu_fused.hip) to the entry points (relu.hip).
#pragma once
#include "common.h"
#include "msb_pack.h"

struct FusedReluParty {
    const u64 *x, *r;                    // input share, A2B mask
    const u64 *ta, *tb, *tc;             // AND triples
    const u8* rb; const u64* ra;         // B2A
    const u64 *ma, *mb, *mc;             // select
    u64* y; u8* s_bit; u64* s_arith;     // outputs (the last two optional)
};
struct FusedRelu {
    FusedReluParty p[2];
    u64* box;                            // receive buffers, relu_fused_box_bytes(n) bytes
    size_t n;
    unsigned tiles;                      // filled by the launcher
};
size_t relu_fused_box_bytes(size_t n);
int launch_relu_fused(mpc_ctx* c, hipStream_t st, FusedRelu q, int topo);
// the sign-only chain; triples in the packed layout of `g`
size_t relu_fused_msb_box_bytes(size_t n);
int launch_relu_fused_msb(mpc_ctx* c, hipStream_t st, FusedRelu q, const MsbGeom& g);
