// Interface of the one-launch secure ReLU (relu_fused.hip) to the entry points (relu.hip, three_party.hip).
#pragma once
#include "common.h"
#include "overlap.h"

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
template <int NI>
inline void add_material(Spans<NI>& in, const FusedReluParty& p, size_t n, size_t triple_words)
{
    in.words(p.r, n); in.words(p.r1, n); in.words(p.ta, triple_words); in.words(p.tb, triple_words); in.words(p.tc, triple_words);
    in.bytes(p.rb, n); in.words(p.ra, n); in.words(p.ma, n); in.words(p.mb, n); in.words(p.mc, n);
}
// whether the call may run as one launch (overlap.h); triple_words: words of one of a party's AND triple arrays
inline bool relu_outputs_apart(int parties, const FusedRelu& q, size_t triple_words)
{
    Spans<33> in; Spans<9> out;
    for (int i = 0; i < parties; ++i) {
        in.words(q.p[i].x, q.n); add_material(in, q.p[i], q.n, triple_words);
        out.words(q.p[i].y, q.n); out.bytes(q.p[i].s_bit, q.n); out.words(q.p[i].s_arith, q.n);
    }
    return outputs_apart(out, in, true);
}
// copies (two parties): the exchange by copies inside the launch (wire.h) instead of by remote store
size_t relu_fused_box_bytes(int parties, size_t n, bool copies = false);
int launch_relu_fused(mpc_ctx* c, hipStream_t st, int parties, FusedRelu q, int topo, bool copies = false);
// the sign-only chain; offsets of the triples in the packed buffers
struct PackedTriples { size_t off[13]; size_t words[6]; };      // words[l]: packed words of level l
size_t relu_fused_msb_box_bytes(int parties, size_t n, bool copies = false);
int launch_relu_fused_msb(mpc_ctx* c, hipStream_t st, int parties, FusedRelu q, const PackedTriples& g, bool copies = false);
// 2x2 max-pool of [B][H][W][C] (n_out = B * H/2 * W/2 * C outputs); material of the two conversions in m1 (2 n_out
// elements) and m2 (n_out); x, y and the sign shares of FusedReluParty are not used; s1, s2 optional
struct FusedPool {
    FusedReluParty m1[3], m2[3];
    const u64* x[3]; u64* y[3]; u64 *s1[3], *s2[3];
    u64* box;                            // maxpool_fused_box_bytes(parties, packed, n_out) bytes
    size_t n_out; int H, W, C;
    unsigned tiles;                      // filled by the launcher
};
inline bool pool_outputs_apart(int parties, const FusedPool& q, size_t triple_words1, size_t triple_words2)
{
    Spans<63> in; Spans<9> out;
    for (int i = 0; i < parties; ++i) {
        in.words(q.x[i], 4 * q.n_out);
        add_material(in, q.m1[i], 2 * q.n_out, triple_words1); add_material(in, q.m2[i], q.n_out, triple_words2);
        out.words(q.y[i], q.n_out); out.words(q.s1[i], 2 * q.n_out); out.words(q.s2[i], q.n_out);
    }
    return outputs_apart(out, in, false);
}
size_t maxpool_fused_box_bytes(int parties, bool packed, size_t n_out);
// g1, g2: packed layouts of the two conversions (sign-only chain), or null (whole words)
int launch_maxpool_fused(mpc_ctx* c, hipStream_t st, int parties, FusedPool q, int topo, const PackedTriples* g1, const PackedTriples* g2);
