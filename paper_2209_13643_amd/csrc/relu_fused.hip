// Secure ReLU, all rounds in one launch (exchange by remote store on a single-queue lane).
//
// A workgroup is one wave per party (two or three), and its waves work on the same elements.  A party's wave reads its
// own share, its own material and what it has received; a round's masked words are stored into the peers' receive
// buffers in device memory, and the workgroup barrier that follows is the round: nothing but the waves of a workgroup
// depend on each other, so no wave ever waits for another workgroup.  Between rounds (G, P) stay in registers, and a
// receive buffer holds one round of one workgroup's elements, so what streams from HBM is the input, the offline
// material and the output, each once: 690 bytes per element of both parties instead of the 2498 that one launch per
// round moves.  2 097 152 elements: 0.95 ms as ten launches, 0.323 ms here (4.5 TB/s of compulsory bytes).
//
// What bounds it is the exchange through vector memory: a build that exchanges through LDS takes 0.25 ms (5.8 TB/s, more
// than a large copy reaches).  Of the difference, 0.05 ms went with the stores of the masked words and 0.035 with their
// loads; how much of that is their traffic and how much the order of the loads is not separated: vector loads return in
// order, and a round asks for the next level's triples before it loads the received words, so it cannot end before those
// triples have come from memory.  That is all of a small call: 16 411 elements, eleven rounds, take 27 us.  The receive
// buffers have to stay in the L2: with a grid of 2048 workgroups and two buffers per party (33 MB) they were written
// back to memory (0.64 GB per call) and the call took 0.345 ms; with one buffer and a second barrier per round, and 1024
// workgroups, they are 8 MB, and four lanes converting at once still fit (batch-128 VGG16 on four lanes: 11.7 ms with
// two buffers, 11.2 ms with one).  The material is read once, hence the non-temporal loads (0.376 -> 0.345 ms).
#include "common.h"
#include "msb_pack.h"
#include "relu_steps.h"
#include "wire.h"
#include "relu_fused.h"

#include <type_traits>

namespace {

constexpr int kRows = 4;            // most words an element sends in one round

template <int V> struct Operands { Pack<V> P, G; u64 top[V]; };         // top: bit 63 of P

// Alg. 2 on a wave's elements, up to P = U ^ V and G = U & V of the two words the prefix network adds.  Two parties:
// the words x_0, x_1; three: the carry-save sum of x_0, x_1, x_2 and its majority shifted up.  row: loads the
// wave's words of an array; t1: offset of triple 1; whole: bytes between two rows of the receive buffers; before_last:
// loads to issue ahead of the last wait.
template <int NP, int V, typename Row, typename Next>
__device__ __forceinline__ Operands<V> a2b(const FusedReluParty& p, const Wire<NP>& wire, int party, u64 m0, const Pack<V>& x,
                                           unsigned slot, unsigned whole, Row&& row, size_t t1, Next&& before_last)
{
    Operands<V> o;
    const Pack<V> r = row(p.r);
    Pack<V> a = row(p.ta), b = row(p.tb), c = row(p.tc), d, g;
    if constexpr (NP == 2) {
        wire.drained();
        wire.put(slot, r);                                               // the mask half of the own word
        wire.opened();
        const Pack<V> rr = wire.template from<V>(0, slot);
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const u64 own = x.v[k] ^ r.v[k], U = party == 0 ? own : rr.v[k], Vv = party == 0 ? rr.v[k] : own;
            d.v[k] = U ^ a.v[k]; g.v[k] = Vv ^ b.v[k];
            o.P.v[k] = U ^ Vv; o.top[k] = o.P.v[k] >> 63;
        }
    } else {
        const Pack<V> r1 = row(p.r1);
        wire.drained();
        wire.put_to(0, slot, r1); wire.put_to(1, slot, r);               // r1 to party + 2, r to party + 1
        const Pack<V> na = row(p.ta + t1), nb = row(p.tb + t1), nc = row(p.tc + t1);
        wire.opened();
        const Pack<V> w1 = wire.template from<V>(0, slot), w2 = wire.template from<V>(1, slot);      // words of party + 1, party + 2
        Pack<V> S, Wd;
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const u64 own = x.v[k] ^ r.v[k] ^ r1.v[k];
            const u64 U = party == 0 ? own : party == 1 ? w2.v[k] : w1.v[k];
            const u64 Vv = party == 1 ? own : party == 2 ? w2.v[k] : w1.v[k];
            Wd.v[k] = party == 2 ? own : party == 0 ? w2.v[k] : w1.v[k];
            S.v[k] = U ^ Vv ^ Wd.v[k];
            d.v[k] = U ^ Wd.v[k] ^ a.v[k]; g.v[k] = Vv ^ Wd.v[k] ^ b.v[k];
        }
        wire.drained();
        wire.put(slot, d); wire.put(slot + whole, g);
        wire.opened();
        const Pack<V> rd = wire.template xored<V>(slot), rg = wire.template xored<V>(slot + whole);
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const u64 K = (fin(d.v[k] ^ rd.v[k], g.v[k] ^ rg.v[k], a.v[k], b.v[k], c.v[k], m0) ^ Wd.v[k]) << 1;
            o.P.v[k] = S.v[k] ^ K; o.top[k] = o.P.v[k] >> 63;
            d.v[k] = S.v[k] ^ na.v[k]; g.v[k] = K ^ nb.v[k];
        }
        a = na; b = nb; c = nc;
    }
    wire.drained();
    wire.put(slot, d); wire.put(slot + whole, g);
    before_last();
    wire.opened();
    const Pack<V> rd = wire.template xored<V>(slot), rg = wire.template xored<V>(slot + whole);
#pragma unroll
    for (int k = 0; k < V; ++k) o.G.v[k] = fin(d.v[k] ^ rd.v[k], g.v[k] ^ rg.v[k], a.v[k], b.v[k], c.v[k], m0);
    return o;
}

// B2A of the sign share and the select product.  s: the share, one byte per element; y and the additive share out.
template <int NP, int V>
__device__ __forceinline__ void select(const Wire<NP>& wire, u64 m0, unsigned lane, unsigned slot, unsigned whole, unsigned masked,
                                       const Pack<V>& x, const Pack<V>& ra, const Pack<V>& ma, const Pack<V>& mb, const Pack<V>& mc,
                                       Pack<V>& y, Pack<V>& sa)
{
    wire.drained();
    wire.template put_flags<V>(lane * V, masked);
    wire.opened();
    const unsigned v = masked ^ wire.template flags<V>(lane * V);
    Pack<V> e, f;
#pragma unroll
    for (int k = 0; k < V; ++k) {
        // s = v xor rb = v + rb - 2 v rb on additive shares of rb
        const u64 vk = (v >> (8 * k)) & 1;
        sa.v[k] = (vk ? (u64)0 - ra.v[k] : ra.v[k]) + (vk & m0);
        e.v[k] = x.v[k] - ma.v[k];
        f.v[k] = (m0 & 1) - sa.v[k] - mb.v[k];
    }
    wire.drained();
    wire.put(slot, e); wire.put(slot + whole, f);
    wire.opened();
    const Pack<V> re = wire.template summed<V>(slot), rf = wire.template summed<V>(slot + whole);
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const u64 eo = e.v[k] + re.v[k], fo = f.v[k] + rf.v[k];
        y.v[k] = mc.v[k] + eo * (mb.v[k] + (fo & m0)) + ma.v[k] * fo;
    }
}

template <int W> struct LevelTriples { Pack<W> a1, b1, c1, a2, b2, c2; };

// y = ReLU(x) on a wave's elements, whole-word adder.  row: loads the wave's words of an array of n; rb: its random
// bits.  s: the sign bit shares (one byte per element), sa: the additive ones.
template <int V> struct Converted { Pack<V> y, sa; unsigned s; };
template <int NP, int V, int TOPO, typename Row>
__device__ __forceinline__ Converted<V> convert_words(const FusedReluParty& p, const Wire<NP>& wire, int party, unsigned lane, unsigned slot,
                                                      size_t n, const Pack<V>& x, unsigned rb_at, const u8* rb_base, Row&& row)
{
    const u64 m0 = party == 0 ? ~(u64)0 : 0;
    constexpr unsigned whole = kWave * V * 8u;
    auto triples = [&](auto tag) {
        constexpr int L = decltype(tag)::value, t = NP - 1 + 2 * L;
        LevelTriples<V> r;
        r.a1 = row(p.ta + t * n); r.b1 = row(p.tb + t * n); r.c1 = row(p.tc + t * n);
        if constexpr (L < 5) { r.a2 = row(p.ta + (t + 1) * n); r.b2 = row(p.tb + (t + 1) * n); r.c2 = row(p.tc + (t + 1) * n); }
        return r;
    };
    LevelTriples<V> next;
    Operands<V> o = a2b<NP, V>(p, wire, party, m0, x, slot, whole, row, n, [&] { next = triples(std::integral_constant<int, 0>{}); });
    Pack<V>&P = o.P, &G = o.G;
    // prefix levels: mask and send level L's operands, fetch the next level's triples, open, finish
    auto level = [&](auto tag) {
        constexpr int L = decltype(tag)::value;
        const LevelTriples<V> t = next;
        Pack<V> d1, g1, d2, g2;
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const u64 X = op_x<TOPO, L>(P.v[k]);
            d1.v[k] = X ^ t.a1.v[k]; g1.v[k] = op_y<TOPO, L>(G.v[k]) ^ t.b1.v[k];
            if constexpr (L < 5) { d2.v[k] = X ^ t.a2.v[k]; g2.v[k] = op_y<TOPO, L>(P.v[k]) ^ t.b2.v[k]; }
        }
        wire.drained();
        wire.put(slot, d1); wire.put(slot + whole, g1);
        if constexpr (L < 5) { wire.put(slot + 2 * whole, d2); wire.put(slot + 3 * whole, g2); }
        if constexpr (L < 5) next = triples(std::integral_constant<int, L + 1>{});
        wire.opened();
        const Pack<V> rd1 = wire.template xored<V>(slot), rg1 = wire.template xored<V>(slot + whole);
        Pack<V> rd2, rg2;
        if constexpr (L < 5) { rd2 = wire.template xored<V>(slot + 2 * whole); rg2 = wire.template xored<V>(slot + 3 * whole); }
#pragma unroll
        for (int k = 0; k < V; ++k) {
            G.v[k] ^= fin(d1.v[k] ^ rd1.v[k], g1.v[k] ^ rg1.v[k], t.a1.v[k], t.b1.v[k], t.c1.v[k], m0);
            if constexpr (L < 5)
                P.v[k] = keep_p<TOPO, L>(P.v[k]) ^ fin(d2.v[k] ^ rd2.v[k], g2.v[k] ^ rg2.v[k], t.a2.v[k], t.b2.v[k], t.c2.v[k], m0);
        }
    };
    level(std::integral_constant<int, 0>{}); level(std::integral_constant<int, 1>{}); level(std::integral_constant<int, 2>{});
    level(std::integral_constant<int, 3>{}); level(std::integral_constant<int, 4>{}); level(std::integral_constant<int, 5>{});

    // sign share = bit 63 of the sum's half-add xor the carry out of bits 0..62
    const Pack<V> ra = row(p.ra), ma = row(p.ma), mb = row(p.mb), mc = row(p.mc);
    const unsigned rb = ld_flags<V>(rb_base + rb_at);
    Converted<V> r;
    r.s = 0;
#pragma unroll
    for (int k = 0; k < V; ++k) r.s |= (unsigned)(o.top[k] ^ ((G.v[k] >> 62) & 1)) << (8 * k);
    select<NP, V>(wire, m0, lane, slot, whole, r.s ^ rb, x, ra, ma, mb, mc, r.y, r.sa);
    return r;
}

template <int NP, int V, int TOPO>
__global__ __launch_bounds__(NP * kWave, 4) void k_relu_fused(FusedRelu q)
{
    const int party = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int lane = threadIdx.x % kWave;
    const FusedReluParty& p = q.p[party];
    const size_t n = q.n;
    const Wire<NP> wire(q.box, party, (size_t)kRows * kWave * V);
    unsigned slot = lane * V * 8u;

    for (size_t tile = blockIdx.x; tile < q.tiles; tile += gridDim.x) {
        // the wave's elements: base + off .. ; a ragged last tile takes the last 64 V elements and stores its own only
        const size_t first = tile * (kWave * V);
        const size_t base = first + kWave * V <= n ? first : n >= kWave * V ? n - kWave * V : 0;
        const unsigned rest = n < kWave * V ? (unsigned)n - V : kWave * V - V;
        unsigned off = lane * V < rest ? lane * V : rest;
        // opaque per tile: otherwise the addresses of all rows are formed ahead of the loop and spilled
        asm volatile("" : "+v"(off), "+v"(slot));
        auto row = [&](const u64* t) { return ld_once<V>(t + base, off * 8u); };
        const Pack<V> x = row(p.x);
        const Converted<V> r = convert_words<NP, V, TOPO>(p, wire, party, lane, slot, n, x, off, p.rb + base, row);
        if (base + off >= first) {
            st_words<V>(p.y + base, off * 8u, r.y);
            if (p.s_bit) st_flags<V>(p.s_bit + base + off, r.s);
            if (p.s_arith) st_words<V>(p.s_arith + base, off * 8u, r.sa);
        } else if (V == 2 && base + off + 1 == first) {                // an odd count: only the second element is the tile's own
            (p.y + base)[off + 1] = r.y.v[V - 1];
            if (p.s_bit) (p.s_bit + base)[off + 1] = (u8)(r.s >> 8);
            if (p.s_arith) (p.s_arith + base)[off + 1] = r.sa.v[V - 1];
        }
    }
}

// ---- sign-only chain on packed words ------------------------------------------------
// A wave works on 64 V elements.  Level l keeps one word per 2^(l+1) elements: the first log2(V) levels combine two
// words of the same lane, every later one the words of lanes j and j ^ d: both lanes form the same word, load the same
// triple words and store the same masked words, so no lane ever moves data and element k of the lane finds its carry
// in the lane's own word at the end.
// 2 097 152 elements: 0.378 ms as ten launches, 0.141 ms here (256 compulsory bytes per element: 3.8 TB/s; what is
// left is the exchange through vector memory, as for whole words).  Four elements per lane, whose loads touch every
// line twice: 0.144 ms; 1024 workgroups: 0.145 ms.
__device__ __forceinline__ u64 from_lane_xor(u64 v, int mask)
{
    const unsigned lo = __shfl_xor((unsigned)v, mask), hi = __shfl_xor((unsigned)(v >> 32), mask);
    return ((u64)hi << 32) | lo;
}

// y = ReLU(x) on a wave's elements from `base` (a multiple of 64 V) on; lane's elements at lane V.  RAGGED: the tile may
// reach past the packed words of the call's elements (word indices are clamped then).
template <int NP, int V, bool RAGGED, typename Row>
__device__ __forceinline__ Converted<V> convert_packed(const FusedReluParty& p, const PackedTriples& g, const Wire<NP>& wire, int party,
                                                       unsigned lane, size_t base, const Pack<V>& x, unsigned rb_at, const u8* rb_base, Row&& row)
{
    const u64 m0 = party == 0 ? ~(u64)0 : 0;
    // rows of whole words and of packed words in the receive buffers
    constexpr unsigned whole = kWave * V * 8u, packed = kWave * V / 2 * 8u;
    const unsigned slot = lane * V * 8u;
    // level L: a lane forms words(L) words, at word index at(L) of the tile
    auto at = [&](auto tag) { constexpr int L = decltype(tag)::value; return (2 << L) <= V ? lane * (V >> (L + 1)) : (lane * V) >> (L + 1); };
    auto triples = [&](auto tag) {
        constexpr int L = decltype(tag)::value, W = (2 << L) <= V ? V >> (L + 1) : 1, t = NP - 1 + 2 * L;
        unsigned w = at(tag);
        if constexpr (RAGGED) {
            const size_t have = g.words[L] - (base >> (L + 1));                 // of this level from the tile's first one on
            if (w + W > have) w = have < W ? 0 : (unsigned)have - W;
        }
        auto tri = [&](const u64* q, int k) { return ld_once<W>(q + g.off[k] + (base >> (L + 1)), w * 8u); };
        LevelTriples<W> r;
        r.a1 = tri(p.ta, t); r.b1 = tri(p.tb, t); r.c1 = tri(p.tc, t);
        if constexpr (L < 5) { r.a2 = tri(p.ta, t + 1); r.b2 = tri(p.tb, t + 1); r.c2 = tri(p.tc, t + 1); }
        return r;
    };

    LevelTriples<V == 1 ? 1 : V / 2> t0;
    Operands<V> o = a2b<NP, V>(p, wire, party, m0, x, slot, whole, row, g.off[1], [&] { t0 = triples(std::integral_constant<int, 0>{}); });
    Pack<V>&P = o.P, &G = o.G;
    // mask and send, fetch the next level's triples (returned), open and finish
    auto level = [&](auto tag, const auto& tr) {
        constexpr int L = decltype(tag)::value, d = 1 << L;
        constexpr u64 A = sel_mask(L), B = low_mask(L);
        constexpr bool inlane = (2 << L) <= V;
        constexpr int W = inlane ? V >> (L + 1) : 1;
        const unsigned w = at(tag) * 8u;
        Pack<W> d1, g1, d2, g2, Gk;
#pragma unroll
        for (int k = 0; k < W; ++k) {
            u64 Glo, Ghi, Plo, Phi;
            if constexpr (inlane) { Glo = G.v[2 * k]; Ghi = G.v[2 * k + 1]; Plo = P.v[2 * k]; Phi = P.v[2 * k + 1]; }
            else {
                constexpr int bit = d / V;                        // lanes that hold the two halves differ in this bit
                const u64 Go = from_lane_xor(G.v[0], bit), Po = from_lane_xor(P.v[0], bit);
                const bool up = lane & bit;
                Glo = up ? Go : G.v[0]; Ghi = up ? G.v[0] : Go; Plo = up ? Po : P.v[0]; Phi = up ? P.v[0] : Po;
            }
            const u64 X = (Plo & A) | rotl<d>(Phi & A);                             // P[p]
            Gk.v[k] = (Glo & A) | rotl<d>(Ghi & A);                                 // G[p]
            d1.v[k] = X ^ tr.a1.v[k];
            g1.v[k] = (rotl<d>(Glo & B) | rotl<2 * d>(Ghi & B)) ^ tr.b1.v[k];       // G[p - d] moved to p
            if constexpr (L < 5) {
                d2.v[k] = X ^ tr.a2.v[k];
                g2.v[k] = (rotl<d>(Plo & B) | rotl<2 * d>(Phi & B)) ^ tr.b2.v[k];   // P[p - d] moved to p
            }
        }
        wire.drained();
        wire.put(w, d1); wire.put(w + packed, g1);
        if constexpr (L < 5) { wire.put(w + 2 * packed, d2); wire.put(w + 3 * packed, g2); }
        constexpr int W1 = (4 << L) <= V ? V >> (L + 2) : 1;
        LevelTriples<W1> next;
        if constexpr (L < 5) next = triples(std::integral_constant<int, L + 1>{});
        wire.opened();
        const Pack<W> rd1 = wire.template xored<W>(w), rg1 = wire.template xored<W>(w + packed);
        Pack<W> rd2, rg2;
        if constexpr (L < 5) { rd2 = wire.template xored<W>(w + 2 * packed); rg2 = wire.template xored<W>(w + 3 * packed); }
#pragma unroll
        for (int k = 0; k < W; ++k) {
            G.v[k] = Gk.v[k] ^ fin(d1.v[k] ^ rd1.v[k], g1.v[k] ^ rg1.v[k], tr.a1.v[k], tr.b1.v[k], tr.c1.v[k], m0);
            if constexpr (L < 5) P.v[k] = fin(d2.v[k] ^ rd2.v[k], g2.v[k] ^ rg2.v[k], tr.a2.v[k], tr.b2.v[k], tr.c2.v[k], m0);
        }
        return next;
    };
    const auto t1 = level(std::integral_constant<int, 0>{}, t0);
    const auto t2 = level(std::integral_constant<int, 1>{}, t1);
    const Pack<V> ra = row(p.ra), ma = row(p.ma);
    const auto t3 = level(std::integral_constant<int, 2>{}, t2);
    const Pack<V> mb = row(p.mb), mc = row(p.mc);
    const auto t4 = level(std::integral_constant<int, 3>{}, t3);
    const auto t5 = level(std::integral_constant<int, 4>{}, t4);
    level(std::integral_constant<int, 5>{}, t5);

    // element i's carry into bit 63 sits at bit (62 + i) mod 64 of word i / 64
    const unsigned rb = ld_flags<V>(rb_base + rb_at);
    Converted<V> r;
    r.s = 0;
#pragma unroll
    for (int k = 0; k < V; ++k) r.s |= (unsigned)((o.top[k] ^ (G.v[0] >> ((62 + lane * V + k) & 63))) & 1) << (8 * k);
    select<NP, V>(wire, m0, lane, slot, whole, r.s ^ rb, x, ra, ma, mb, mc, r.y, r.sa);
    return r;
}

template <int NP, int V>
__device__ __forceinline__ void msb_tile(const FusedReluParty& p, const PackedTriples& g, const Wire<NP>& wire, int party, size_t base, size_t n)
{
    unsigned lane = threadIdx.x % kWave;
    const unsigned rest = V == 1 && n - base < kWave ? (unsigned)(n - base) - 1 : kWave * V - V;
    unsigned off = lane * V < rest ? lane * V : rest;             // V > 1: the caller passes whole tiles only
    asm volatile("" : "+v"(off), "+v"(lane));
    auto row = [&](const u64* q) { return ld_once<V>(q + base, off * 8u); };
    const Pack<V> x = row(p.x);
    const Converted<V> r = convert_packed<NP, V, false>(p, g, wire, party, lane, base, x, off, p.rb + base, row);
    if (off != lane * V) return;              // past the end: a lane that worked on the last element again, at another bit position
    st_words<V>(p.y + base, off * 8u, r.y);
    if (p.s_bit) st_flags<V>(p.s_bit + base + off, r.s);
    if (p.s_arith) st_words<V>(p.s_arith + base, off * 8u, r.sa);
}

// tiles 0 .. wide-1: 128 elements each, two per lane; the others 64 elements, one per lane (the last one ragged)
constexpr int kMsbV = 2;
constexpr size_t kMsbBox = 2 * kWave * kMsbV;      // words: two rows of whole words, or four of level 0
template <int NP>
__global__ __launch_bounds__(NP * kWave, 4) void k_relu_fused_msb(FusedRelu q, PackedTriples g, unsigned wide)
{
    const int party = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const Wire<NP> wire(q.box, party, kMsbBox);
    for (unsigned tile = blockIdx.x; tile < q.tiles; tile += gridDim.x) {
        if (tile < wide) msb_tile<NP, kMsbV>(q.p[party], g, wire, party, (size_t)tile * kWave * kMsbV, q.n);
        else             msb_tile<NP, 1>(q.p[party], g, wire, party, ((size_t)wide * kMsbV + (tile - wide)) * kWave, q.n);
    }
}

constexpr size_t kPoolBox = (size_t)kRows * kWave * 2;        // words: four rows of the first level's pairs
// ---- 2x2 max-pool: two tournament levels, each max(p, q) = q + ReLU(p - q) ----------------
// A wave works on 64 outputs: the first level's pair of differences of an output are two elements of one lane, the
// second level's difference one, so both conversions and the sums around them stay in registers.
// 32 x 32 x 32 x 64 inputs (524 288 outputs): 0.283 ms as gathers, two one-launch conversions and a sum (eight launches),
// 0.251 ms here (whole words; 512 workgroups 0.311 ms), sign-only 0.145 -> 0.137 ms; 32 x 8 x 8 x 256: 81 -> 64 us.
template <int NP, bool PACKED, int TOPO>
__global__ __launch_bounds__(NP * kWave, 4) void k_maxpool_fused(FusedPool q, PackedTriples g1, PackedTriples g2)
{
    const int party = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const Wire<NP> wire(q.box, party, kPoolBox);
    const FusedReluParty &p1 = q.m1[party], &p2 = q.m2[party];
    const u64* const x = q.x[party];
    const unsigned C = (unsigned)q.C, Wo = (unsigned)q.W / 2, Ho = (unsigned)q.H / 2;
    for (unsigned tile = blockIdx.x; tile < q.tiles; tile += gridDim.x) {
        const size_t o0 = (size_t)tile * kWave;
        unsigned lane = threadIdx.x % kWave;
        const unsigned last = q.n_out - o0 < kWave ? (unsigned)(q.n_out - o0) - 1 : kWave - 1;
        unsigned at = lane < last ? lane : last;                    // past the end: the last output again, not stored
        asm volatile("" : "+v"(at), "+v"(lane));
        size_t t = o0 + at;
        const unsigned ch = (unsigned)(t % C); t /= C;
        const unsigned wo = (unsigned)(t % Wo); t /= Wo;
        const unsigned ho = (unsigned)(t % Ho); const size_t b = t / Ho;
        const u64* const w = x + ((b * q.H + 2 * ho) * q.W + 2 * wo) * C + ch;
        const size_t dh = (size_t)q.W * C;
        const u64 p00 = w[0], p01 = w[C], p10 = w[dh], p11 = w[dh + C];
        Pack<2> d1;
        d1.v[0] = p00 - p01; d1.v[1] = p10 - p11;
        auto row1 = [&](const u64* m) { return ld_once<2>(m + 2 * o0, at * 16u); };
        Converted<2> r1;
        if constexpr (PACKED) r1 = convert_packed<NP, 2, true>(p1, g1, wire, party, lane, 2 * o0, d1, 2 * at, p1.rb + 2 * o0, row1);
        else                  r1 = convert_words<NP, 2, TOPO>(p1, wire, party, lane, lane * 16u, 2 * q.n_out, d1, 2 * at, p1.rb + 2 * o0, row1);
        const u64 u = p01 + r1.y.v[0], v = p11 + r1.y.v[1];
        Pack<1> d2;
        d2.v[0] = u - v;
        asm volatile("" : "+v"(at), "+v"(lane));
        auto row2 = [&](const u64* m) { return ld_once<1>(m + o0, at * 8u); };
        Converted<1> r2;
        if constexpr (PACKED) r2 = convert_packed<NP, 1, false>(p2, g2, wire, party, lane, o0, d2, at, p2.rb + o0, row2);
        else                  r2 = convert_words<NP, 1, TOPO>(p2, wire, party, lane, lane * 8u, q.n_out, d2, at, p2.rb + o0, row2);
        if (at != lane) continue;
        q.y[party][o0 + at] = v + r2.y.v[0];
        if (q.s1[party]) st_words<2>(q.s1[party] + 2 * o0, at * 16u, r1.sa);
        if (q.s2[party]) q.s2[party][o0 + at] = r2.sa.v[0];
    }
}

// Workgroups of a launch, [parties - 2]: as many as their receive buffers fit the L2 of their XCD (a three-party
// workgroup has six of them).  Whole words, 2 097 152 elements: two parties 512 / 1024 / 2048 workgroups 0.335 / 0.323 /
// 0.331 ms; three parties 256 / 512 / 768 / 1024 workgroups 0.73 / 0.65 / 0.71 / 0.75 ms (2.12 ms as eleven launches).
// Sign-only: two parties 1024 / 2048 workgroups 0.145 / 0.141 ms; three parties 1024 / 1536 / 2048 workgroups 0.369 /
// 0.360 / 0.365 ms (0.99 ms as eleven launches).
constexpr unsigned kBlocks[2] = { 1024, 512 }, kMsbBlocks[2] = { 2048, 1536 };
constexpr int kMaxBlockPairs[2] = { 2, 6 };        // ordered pairs of parties: receive buffers per workgroup

// two elements per thread (16-byte accesses) once one element per thread would need a second round of workgroups
int width(size_t n, unsigned blocks) { return n > (size_t)blocks * kWave ? 2 : 1; }
unsigned tiles_of(size_t n, int v) { return (unsigned)((n + kWave * v - 1) / (kWave * v)); }
unsigned wide_tiles(size_t n, unsigned blocks) { return width(n, blocks) == kMsbV ? (unsigned)(n / (kWave * kMsbV)) : 0; }
unsigned msb_tiles(size_t n, unsigned blocks)
{
    const unsigned wide = wide_tiles(n, blocks);
    return wide + tiles_of(n - (size_t)wide * kWave * kMsbV, 1);
}
unsigned least(unsigned a, unsigned b) { return a < b ? a : b; }

template <int NP, int V>
void launch(hipStream_t st, const FusedRelu& q, int topo)
{
    const dim3 grid(least(q.tiles, kBlocks[NP - 2])), block(NP * kWave);
    if constexpr (NP == 2)
        if (topo) { hipLaunchKernelGGL((k_relu_fused<NP, V, 1>), grid, block, 0, st, q); return; }
    hipLaunchKernelGGL((k_relu_fused<NP, V, 0>), grid, block, 0, st, q);
}

}  // namespace

size_t relu_fused_box_bytes(int parties, size_t n)
{
    const unsigned blocks = kBlocks[parties - 2];
    const int v = width(n, blocks);
    return (size_t)least(tiles_of(n, v), blocks) * kMaxBlockPairs[parties - 2] * (kRows * kWave * v) * sizeof(u64);
}

int launch_relu_fused(mpc_ctx* c, hipStream_t st, int parties, FusedRelu q, int topo)
{
    if (q.n == 0 || q.n >= ((size_t)1 << 37)) return MPC_EINVAL;
    const int v = width(q.n, kBlocks[parties - 2]);
    q.tiles = tiles_of(q.n, v);
    if (parties == 2) { if (v == 2) launch<2, 2>(st, q, topo); else launch<2, 1>(st, q, topo); }
    else              { if (v == 2) launch<3, 2>(st, q, 0);    else launch<3, 1>(st, q, 0); }
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

size_t relu_fused_msb_box_bytes(int parties, size_t n)
{
    const unsigned blocks = kMsbBlocks[parties - 2];
    return (size_t)least(msb_tiles(n, blocks), blocks) * kMaxBlockPairs[parties - 2] * kMsbBox * sizeof(u64);
}

int launch_relu_fused_msb(mpc_ctx* c, hipStream_t st, int parties, FusedRelu q, const PackedTriples& g)
{
    if (q.n == 0 || q.n >= ((size_t)1 << 37)) return MPC_EINVAL;
    const unsigned blocks = kMsbBlocks[parties - 2], wide = wide_tiles(q.n, blocks);
    q.tiles = msb_tiles(q.n, blocks);
    const dim3 grid(least(q.tiles, blocks));
    if (parties == 2) hipLaunchKernelGGL(k_relu_fused_msb<2>, grid, dim3(2 * kWave), 0, st, q, g, wide);
    else              hipLaunchKernelGGL(k_relu_fused_msb<3>, grid, dim3(3 * kWave), 0, st, q, g, wide);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

size_t maxpool_fused_box_bytes(int parties, bool packed, size_t n_out)
{
    const unsigned blocks = (packed ? kMsbBlocks : kBlocks)[parties - 2];
    return (size_t)least(tiles_of(n_out, 1), blocks) * kMaxBlockPairs[parties - 2] * kPoolBox * sizeof(u64);
}

int launch_maxpool_fused(mpc_ctx* c, hipStream_t st, int parties, FusedPool q, int topo, const PackedTriples* g1, const PackedTriples* g2)
{
    if (q.n_out == 0 || q.n_out >= ((size_t)1 << 36)) return MPC_EINVAL;
    const bool packed = g1 != nullptr;
    q.tiles = tiles_of(q.n_out, 1);
    const dim3 grid(least(q.tiles, (packed ? kMsbBlocks : kBlocks)[parties - 2])), block(parties * kWave);
    const PackedTriples none{};
    if (parties == 2) {
        if (packed)    hipLaunchKernelGGL((k_maxpool_fused<2, true, 0>), grid, block, 0, st, q, *g1, *g2);
        else if (topo) hipLaunchKernelGGL((k_maxpool_fused<2, false, 1>), grid, block, 0, st, q, none, none);
        else           hipLaunchKernelGGL((k_maxpool_fused<2, false, 0>), grid, block, 0, st, q, none, none);
    } else {
        if (packed)    hipLaunchKernelGGL((k_maxpool_fused<3, true, 0>), grid, block, 0, st, q, *g1, *g2);
        else           hipLaunchKernelGGL((k_maxpool_fused<3, false, 0>), grid, block, 0, st, q, none, none);
    }
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}
