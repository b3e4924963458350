// Secure ReLU, all rounds in one launch (exchange by remote store on a single-queue lane).
//
// A workgroup is one wave per party (two or three), and its waves work on the same elements.  A party's wave reads its
// own share, its own material and what it has received; a round's masked words are stored into the peers' receive
// buffers in device memory, and the workgroup barrier that follows is the round: nothing but the waves of a workgroup
// depend on each other, so no wave ever waits for another workgroup.  Between rounds (G, P) stay in registers, and a
// receive buffer holds one round of one workgroup's elements, so what streams from HBM is the input, the offline
// material and the output, each once: 690 bytes per element of both parties instead of the 2498 that one launch per
// round moves.  2 097 152 elements: 0.95 ms as ten launches, 0.307-0.311 ms here (4.7 TB/s of compulsory bytes; two boxes).
//
// What bounds it is memory plus the exchange through the L2: a build that exchanges through LDS takes 0.255 ms (5.7 TB/s,
// more than a large copy reaches), and the number of resident workgroups no longer matters (768 / 1024 / 2048: 0.305 /
// 0.307 / 0.315 ms).  The order of the loads (issue_point below) keeps the rounds from waiting for memory: with the next
// level's triples asked for ahead of the received words, and those loaded one after the other, the call took 0.342 and
// 0.328 ms on the same two boxes, and a workgroup began each tile with nothing in flight.  The receive
// buffers should stay in the L2: with a grid of 2048 workgroups and two buffers per party (33 MB) they were written
// back to memory (0.64 GB per call) and the call took 5 % longer; with one buffer and a second barrier per round, and 1024
// workgroups, they are 8 MB, and four lanes converting at once still fit (batch-128 VGG16 on four lanes: 11.7 ms with
// two buffers, 11.2 ms with one).  The sign-only chain gives some of that up (msb_v below).  The material is read once, hence
// the non-temporal loads (10 % at the same size).
#include "common.h"
#include "msb_pack.h"
#include "relu_steps.h"
#include "wire.h"
#include "relu_fused.h"

#include <type_traits>

namespace {

constexpr int kRows = 4;            // most words an element sends in one round

template <int V> struct Operands { Pack<V> P, G; u64 top[V]; };         // top: bit 63 of P

// Order of the loads.  Vector loads return in order, so a round's received words are loaded first, together, and behind
// them what comes from memory for later rounds: the masks (a, b) of the round after the next, which have to be there when
// the next round's words are masked, and the c of the next round, needed when that is finished.  An operand thus has one
// whole round to arrive in.
__device__ __forceinline__ void issue_point() { __builtin_amdgcn_sched_barrier(0); }

// What a wave needs when it turns to its elements: the A2B masks (r1: three parties) and triple 0's a and b.
template <int NP, int V> struct Head { Pack<V> r, r1, a, b; };
template <int NP, int V, typename Row> __device__ __forceinline__ void load_masks(Head<NP, V>& h, const FusedReluParty& p, Row&& row)
{
    h.r = row(p.r);
    if constexpr (NP == 3) h.r1 = row(p.r1);
}
template <int NP, int V, typename Row> __device__ __forceinline__ void load_first(Head<NP, V>& h, const FusedReluParty& p, Row&& row)
{
    h.a = row(p.ta); h.b = row(p.tb);
}

// Alg. 2 on a wave's elements, up to P = U ^ V and G = U & V of the two words the prefix network adds.  Two parties:
// the words x_0, x_1; three: the carry-save sum of x_0, x_1, x_2 and its majority shifted up.  row: loads the
// wave's words of an array; t1: offset of triple 1; whole: bytes between two rows of the receive buffers; masks0: loads
// level 0's masks; masks1: level 1's masks and level 0's c.
template <int NP, int V, bool COPY, typename Row, typename Masks0, typename Masks1>
__device__ __forceinline__ Operands<V> a2b(const FusedReluParty& p, const Wire<NP, COPY>& wire, int party, u64 m0, const Pack<V>& x,
                                           const Head<NP, V>& h, unsigned slot, unsigned whole, Row&& row, size_t t1,
                                           Masks0&& masks0, Masks1&& masks1)
{
    Operands<V> o;
    Pack<V> a = h.a, b = h.b, c, d, g;
    if constexpr (NP == 2) {
        wire.drained();
        wire.put(slot, h.r);                                             // the mask half of the own word
        wire.opened();
        const auto got = wire.template received<V>(slot);
        issue_point();
        c = row(p.tc); masks0();
        issue_point();
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const u64 own = x.v[k] ^ h.r.v[k], rr = got.q[0].v[k], U = party == 0 ? own : rr, Vv = party == 0 ? rr : own;
            d.v[k] = U ^ a.v[k]; g.v[k] = Vv ^ b.v[k];
            o.P.v[k] = U ^ Vv; o.top[k] = o.P.v[k] >> 63;
        }
    } else {
        wire.drained();
        wire.put_to(0, slot, h.r1); wire.put_to(1, slot, h.r);           // r1 to party + 2, r to party + 1
        wire.opened();
        const auto got = wire.template received<V>(slot);                // words of party + 1, party + 2
        issue_point();
        const Pack<V> na = row(p.ta + t1), nb = row(p.tb + t1);
        c = row(p.tc);
        issue_point();
        Pack<V> S, Wd;
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const u64 own = x.v[k] ^ h.r.v[k] ^ h.r1.v[k], w1 = got.q[0].v[k], w2 = got.q[1].v[k];
            const u64 U = party == 0 ? own : party == 1 ? w2 : w1;
            const u64 Vv = party == 1 ? own : party == 2 ? w2 : w1;
            Wd.v[k] = party == 2 ? own : party == 0 ? w2 : w1;
            S.v[k] = U ^ Vv ^ Wd.v[k];
            d.v[k] = U ^ Wd.v[k] ^ a.v[k]; g.v[k] = Vv ^ Wd.v[k] ^ b.v[k];
        }
        wire.drained();
        wire.put(slot, d); wire.put(slot, g, whole);
        wire.opened();
        const auto rd = wire.template received<V>(slot), rg = wire.template received<V>(slot, whole);
        issue_point();
        const Pack<V> nc = row(p.tc + t1);
        masks0();
        issue_point();
        const Pack<V> sd = rd.xored(), sg = rg.xored();
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const u64 K = (fin(d.v[k] ^ sd.v[k], g.v[k] ^ sg.v[k], a.v[k], b.v[k], c.v[k], m0) ^ Wd.v[k]) << 1;
            o.P.v[k] = S.v[k] ^ K; o.top[k] = o.P.v[k] >> 63;
            d.v[k] = S.v[k] ^ na.v[k]; g.v[k] = K ^ nb.v[k];
        }
        a = na; b = nb; c = nc;
    }
    wire.drained();
    wire.put(slot, d); wire.put(slot, g, whole);
    wire.opened();
    const auto rd = wire.template received<V>(slot), rg = wire.template received<V>(slot, whole);
    issue_point();
    masks1();
    issue_point();
    const Pack<V> sd = rd.xored(), sg = rg.xored();
#pragma unroll
    for (int k = 0; k < V; ++k) o.G.v[k] = fin(d.v[k] ^ sd.v[k], g.v[k] ^ sg.v[k], a.v[k], b.v[k], c.v[k], m0);
    return o;
}

// B2A of the sign share and the select product.  masked: the share xor rb, one byte per element; y and the additive share
// out.  after_flags, after_words: loads for the wave's next elements.
template <int NP, int V, bool COPY, typename Row, typename AfterFlags, typename AfterWords>
__device__ __forceinline__ void select(const FusedReluParty& p, const Wire<NP, COPY>& wire, u64 m0, unsigned lane, unsigned slot, unsigned whole,
                                       unsigned masked, const Pack<V>& x, const Pack<V>& ra, const Pack<V>& ma, const Pack<V>& mb,
                                       Row&& row, AfterFlags&& after_flags, AfterWords&& after_words, Pack<V>& y, Pack<V>& sa)
{
    wire.drained();
    wire.template put_flags<V>(lane * V, masked);
    wire.opened();
    const unsigned got = wire.template flags<V>(lane * V);
    issue_point();
    const Pack<V> mc = row(p.mc);
    after_flags();
    issue_point();
    const unsigned v = masked ^ got;
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
    wire.put(slot, e); wire.put(slot, f, whole);
    wire.opened();
    const auto re = wire.template received<V>(slot), rf = wire.template received<V>(slot, whole);
    issue_point();
    after_words();
    issue_point();
    const Pack<V> se = re.summed(), sf = rf.summed();
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const u64 eo = e.v[k] + se.v[k], fo = f.v[k] + sf.v[k];
        y.v[k] = mc.v[k] + eo * (mb.v[k] + (fo & m0)) + ma.v[k] * fo;
    }
}

template <int W> struct LevelMasks { Pack<W> a1, b1, a2, b2; };
template <int W> struct LevelC { Pack<W> c1, c2; };

// y = ReLU(x) on a wave's elements, whole-word adder.  row: loads the wave's words of an array of n; rb: its random
// bits.  s: the sign bit shares (one byte per element), sa: the additive ones.
template <int V> struct Converted { Pack<V> y, sa; unsigned s; };
template <int NP, int V, int TOPO, bool COPY, typename Row, typename AfterFlags, typename AfterWords>
__device__ __forceinline__ Converted<V> convert_words(const FusedReluParty& p, const Wire<NP, COPY>& wire, int party, unsigned lane, unsigned slot,
                                                      size_t n, const Pack<V>& x, const Head<NP, V>& h, unsigned rb_at, const u8* rb_base,
                                                      Row&& row, AfterFlags&& after_flags, AfterWords&& after_words)
{
    const u64 m0 = party == 0 ? ~(u64)0 : 0;
    constexpr unsigned whole = kWave * V * 8u;
    auto masks = [&](auto tag) {
        constexpr int L = decltype(tag)::value, t = NP - 1 + 2 * L;
        LevelMasks<V> r;
        r.a1 = row(p.ta + t * n); r.b1 = row(p.tb + t * n);
        if constexpr (L < 5) { r.a2 = row(p.ta + (t + 1) * n); r.b2 = row(p.tb + (t + 1) * n); }
        return r;
    };
    auto thirds = [&](auto tag) {
        constexpr int L = decltype(tag)::value, t = NP - 1 + 2 * L;
        LevelC<V> r;
        r.c1 = row(p.tc + t * n);
        if constexpr (L < 5) r.c2 = row(p.tc + (t + 1) * n);
        return r;
    };
    LevelMasks<V> now, next;
    LevelC<V> third;
    Operands<V> o = a2b<NP, V>(p, wire, party, m0, x, h, slot, whole, row, n,
                               [&] { now = masks(std::integral_constant<int, 0>{}); },
                               [&] { next = masks(std::integral_constant<int, 1>{}); third = thirds(std::integral_constant<int, 0>{}); });
    Pack<V>&P = o.P, &G = o.G;
    unsigned rb = 0;
    Pack<V> ra, ma, mb;
    // prefix levels: mask and send level L's operands, open, fetch for the rounds to come, finish
    auto level = [&](auto tag) {
        constexpr int L = decltype(tag)::value;
        // A party's masked words are formed twice, for the peers and again when the round is finished: held in between they
        // would take 8 V registers.
        Pack<V> d1, g1, d2, g2;
        auto form = [&] {
#pragma unroll
            for (int k = 0; k < V; ++k) {
                const u64 X = op_x<TOPO, L>(P.v[k]);
                d1.v[k] = X ^ now.a1.v[k]; g1.v[k] = op_y<TOPO, L>(G.v[k]) ^ now.b1.v[k];
                if constexpr (L < 5) { d2.v[k] = X ^ now.a2.v[k]; g2.v[k] = op_y<TOPO, L>(P.v[k]) ^ now.b2.v[k]; }
            }
        };
        form();
        wire.drained();
        wire.put(slot, d1); wire.put(slot, g1, whole);
        if constexpr (L < 5) { wire.put(slot, d2, 2 * whole); wire.put(slot, g2, 3 * whole); }
        if constexpr (!TOPO) {
#pragma unroll
            for (int k = 0; k < V; ++k) asm volatile("" : "+v"(P.v[k]), "+v"(G.v[k]));
        }
        wire.opened();
        const auto rd1 = wire.template received<V>(slot), rg1 = wire.template received<V>(slot, whole);
        Received<NP, V> rd2, rg2;
        if constexpr (L < 5) { rd2 = wire.template received<V>(slot, 2 * whole); rg2 = wire.template received<V>(slot, 3 * whole); }
        issue_point();
        LevelMasks<V> later; LevelC<V> next_third;
        if constexpr (L < 5) next_third = thirds(std::integral_constant<int, L + 1>{});
        if constexpr (L < 4) later = masks(std::integral_constant<int, L + 2>{});
        if constexpr (L == 4) rb = ld_flags<V>(rb_base + rb_at);
        if constexpr (L == 5) { ra = row(p.ra); ma = row(p.ma); mb = row(p.mb); }
        issue_point();
        form();
        const Pack<V> sd1 = rd1.xored(), sg1 = rg1.xored();
        Pack<V> sd2, sg2;
        if constexpr (L < 5) { sd2 = rd2.xored(); sg2 = rg2.xored(); }
#pragma unroll
        for (int k = 0; k < V; ++k) {
            G.v[k] ^= fin(d1.v[k] ^ sd1.v[k], g1.v[k] ^ sg1.v[k], now.a1.v[k], now.b1.v[k], third.c1.v[k], m0);
            if constexpr (L < 5)
                P.v[k] = keep_p<TOPO, L>(P.v[k]) ^ fin(d2.v[k] ^ sd2.v[k], g2.v[k] ^ sg2.v[k], now.a2.v[k], now.b2.v[k], third.c2.v[k], m0);
        }
        now = next; next = later; third = next_third;
    };
    level(std::integral_constant<int, 0>{}); level(std::integral_constant<int, 1>{}); level(std::integral_constant<int, 2>{});
    level(std::integral_constant<int, 3>{}); level(std::integral_constant<int, 4>{}); level(std::integral_constant<int, 5>{});

    // sign share = bit 63 of the sum's half-add xor the carry out of bits 0..62
    Converted<V> r;
    r.s = 0;
#pragma unroll
    for (int k = 0; k < V; ++k) r.s |= (unsigned)(o.top[k] ^ ((G.v[k] >> 62) & 1)) << (8 * k);
    select<NP, V>(p, wire, m0, lane, slot, whole, r.s ^ rb, x, ra, ma, mb, row, after_flags, after_words, r.y, r.sa);
    return r;
}

// Registers: a GEMM wave leaves 136 of a SIMD's.  128 here (two parties, prefix network of Kogge and Stone); the
// prefix tree needs 131 (held at 128 it spills four: 70 001 / 2 097 152 elements 14.4 / 312.7 us, 13.0 / 306.5 at 131), the copying
// exchange 135 and 139, the operands of three rounds of three parties 156 (512 workgroups are less than two waves per SIMD
// either way).  Max-pool of whole words: 136, with the prefix tree 141, three parties 159.  What is wider waits for a unit
// without a GEMM wave.
template <int NP, int V, int TOPO, bool COPY>
__global__ __launch_bounds__(NP * kWave, (NP == 3 || COPY || TOPO) && V == 2 ? 3 : 4) void k_relu_fused(FusedRelu q)
{
    const int party = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int lane = threadIdx.x % kWave;
    const FusedReluParty& p = q.p[party];
    const size_t n = q.n;
    const Wire<NP, COPY> wire(q.box, party, (size_t)kRows * kWave * V);
    unsigned slot = lane * V * 8u;

    // a tile's elements for the wave: base + off .. ; a ragged last tile takes the last 64 V elements and stores its own only
    const unsigned rest = n < kWave * V ? (unsigned)n - V : kWave * V - V;
    unsigned off = lane * V < rest ? lane * V : rest;
    auto base_of = [&](size_t tile) {
        const size_t first = tile * (kWave * V);
        return first + kWave * V <= n ? first : n >= kWave * V ? n - kWave * V : 0;
    };
    size_t tile = blockIdx.x, base = base_of(tile);
    auto row = [&](const u64* t) { return ld_once<V>(t + base, off * 8u); };
    Head<NP, V> h;
    load_masks(h, p, row);
    Pack<V> x = row(p.x);
    load_first(h, p, row);
    for (;;) {
        const size_t first = tile * (kWave * V), after = tile + gridDim.x;
        const bool more = after < q.tiles;                       // uniform; the next tile's first operands are loaded under this one's last rounds
        const size_t next_base = base_of(more ? after : tile);
        auto next_row = [&](const u64* t) { return ld_once<V>(t + next_base, off * 8u); };
        // opaque per tile: otherwise the addresses of all rows are formed ahead of the loop and spilled
        asm volatile("" : "+v"(off), "+v"(slot));
        Head<NP, V> nh; Pack<V> nx;
        const Converted<V> r = convert_words<NP, V, TOPO>(p, wire, party, lane, slot, n, x, h, off, p.rb + base, row,
                                                          [&] { if (more) load_masks(nh, p, next_row); },
                                                          [&] { if (more) { nx = next_row(p.x); load_first(nh, p, next_row); } });
        if (base + off >= first) {
            st_words<V>(p.y + base, off * 8u, r.y);
            if (p.s_bit) st_flags<V>(p.s_bit + base + off, r.s);
            if (p.s_arith) st_words<V>(p.s_arith + base, off * 8u, r.sa);
        } else if (V == 2 && base + off + 1 == first) {                // an odd count: only the second element is the tile's own
            (p.y + base)[off + 1] = r.y.v[V - 1];
            if (p.s_bit) (p.s_bit + base)[off + 1] = (u8)(r.s >> 8);
            if (p.s_arith) (p.s_arith + base)[off + 1] = r.sa.v[V - 1];
        }
        if (!more) break;
        tile = after; base = next_base; h = nh; x = nx;
    }
}

// ---- sign-only chain on packed words ------------------------------------------------
// A wave works on 64 V elements.  Level l keeps one word per 2^(l+1) elements: the first log2(V) levels combine two
// words of the same lane, every later one the words of lanes j and j ^ d: both lanes form the same word, load the same
// triple words and store the same masked words, so no lane ever moves data and element k of the lane finds its carry
// in the lane's own word at the end.
// 2 097 152 elements: 0.378 ms as ten launches, 0.135 ms here (256 compulsory bytes per element: 4.0 TB/s).  With two elements
// per lane 0.151 ms (0.131 through LDS; the levels' vector work, the same for every level, is half of the rest), with the
// received words behind the next triples 0.155 ms.
__device__ __forceinline__ u64 from_lane_xor(u64 v, int mask)
{
    const unsigned lo = __shfl_xor((unsigned)v, mask), hi = __shfl_xor((unsigned)(v >> 32), mask);
    return ((u64)hi << 32) | lo;
}

template <int W> struct LevelTriples { Pack<W> a1, b1, c1, a2, b2, c2; };
// words a lane forms at level L of the sign-only chain
constexpr int level_words(int V, int L) { return (2 << L) <= V ? V >> (L + 1) : 1; }

// y = ReLU(x) on a wave's elements from `base` (a multiple of 64 V) on; lane's elements at lane V.  RAGGED: the tile may
// reach past the packed words of the call's elements (word indices are clamped then).
template <int NP, int V, bool RAGGED, bool COPY, typename Row, typename AfterFlags, typename AfterWords>
__device__ __forceinline__ Converted<V> convert_packed(const FusedReluParty& p, const PackedTriples& g, const Wire<NP, COPY>& wire, int party,
                                                       unsigned lane, size_t base, const Pack<V>& x, const Head<NP, V>& h,
                                                       unsigned rb_at, const u8* rb_base, Row&& row,
                                                       AfterFlags&& after_flags, AfterWords&& after_words)
{
    const u64 m0 = party == 0 ? ~(u64)0 : 0;
    // rows of whole words and of packed words in the receive buffers
    constexpr unsigned whole = kWave * V * 8u, packed = kWave * V / 2 * 8u;
    const unsigned slot = lane * V * 8u;
    // level L: a lane forms level_words(V, L) words, at word index at(L) of the tile
    auto at = [&](auto tag) { constexpr int L = decltype(tag)::value; return (2 << L) <= V ? lane * (V >> (L + 1)) : (lane * V) >> (L + 1); };
    auto triples = [&](auto tag) {
        constexpr int L = decltype(tag)::value, W = level_words(V, L), t = NP - 1 + 2 * L;
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
    constexpr std::integral_constant<int, 0> l0{}; constexpr std::integral_constant<int, 1> l1{}; constexpr std::integral_constant<int, 2> l2{};
    constexpr std::integral_constant<int, 3> l3{}; constexpr std::integral_constant<int, 4> l4{}; constexpr std::integral_constant<int, 5> l5{};
    LevelTriples<level_words(V, 0)> t0; LevelTriples<level_words(V, 1)> t1; LevelTriples<level_words(V, 2)> t2;
    LevelTriples<level_words(V, 3)> t3; LevelTriples<level_words(V, 4)> t4; LevelTriples<level_words(V, 5)> t5;

    Operands<V> o = a2b<NP, V>(p, wire, party, m0, x, h, slot, whole, row, g.off[1], [&] { t0 = triples(l0); }, [&] { t1 = triples(l1); });
    Pack<V>&P = o.P, &G = o.G;
    // mask and send, open, fetch for the rounds to come (ahead), finish
    auto level = [&](auto tag, const auto& tr, auto&& ahead) {
        constexpr int L = decltype(tag)::value, d = 1 << L;
        constexpr u64 A = sel_mask(L), B = low_mask(L);
        constexpr bool inlane = (2 << L) <= V;
        constexpr int W = level_words(V, L);
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
        wire.put(w, d1); wire.put(w, g1, packed);
        if constexpr (L < 5) { wire.put(w, d2, 2 * packed); wire.put(w, g2, 3 * packed); }
        wire.opened();
        const auto rd1 = wire.template received<W>(w), rg1 = wire.template received<W>(w, packed);
        Received<NP, W> rd2, rg2;
        if constexpr (L < 5) { rd2 = wire.template received<W>(w, 2 * packed); rg2 = wire.template received<W>(w, 3 * packed); }
        issue_point();
        ahead();
        issue_point();
        const Pack<W> sd1 = rd1.xored(), sg1 = rg1.xored();
        Pack<W> sd2, sg2;
        if constexpr (L < 5) { sd2 = rd2.xored(); sg2 = rg2.xored(); }
#pragma unroll
        for (int k = 0; k < W; ++k) {
            G.v[k] = Gk.v[k] ^ fin(d1.v[k] ^ sd1.v[k], g1.v[k] ^ sg1.v[k], tr.a1.v[k], tr.b1.v[k], tr.c1.v[k], m0);
            if constexpr (L < 5) P.v[k] = fin(d2.v[k] ^ sd2.v[k], g2.v[k] ^ sg2.v[k], tr.a2.v[k], tr.b2.v[k], tr.c2.v[k], m0);
        }
    };
    unsigned rb = 0;
    Pack<V> ra, ma, mb;
    level(l0, t0, [&] { t2 = triples(l2); });
    level(l1, t1, [&] { t3 = triples(l3); });
    level(l2, t2, [&] { t4 = triples(l4); });
    level(l3, t3, [&] { t5 = triples(l5); });
    level(l4, t4, [&] { rb = ld_flags<V>(rb_base + rb_at); ra = row(p.ra); });
    level(l5, t5, [&] { ma = row(p.ma); mb = row(p.mb); });

    // element i's carry into bit 63 sits at bit (62 + i) mod 64 of word i / 64
    Converted<V> r;
    r.s = 0;
#pragma unroll
    for (int k = 0; k < V; ++k) r.s |= (unsigned)((o.top[k] ^ (G.v[0] >> ((62 + lane * V + k) & 63))) & 1) << (8 * k);
    select<NP, V>(p, wire, m0, lane, slot, whole, r.s ^ rb, x, ra, ma, mb, row, after_flags, after_words, r.y, r.sa);
    return r;
}

// The workgroup's tiles of 64 V elements: tile blockIdx.x and every gridDim.x-th after it from `tile` to below `end`;
// tile t starts at element at0 + (t - tile0) 64 V.  Returns the workgroup's first tile from `end` on.
template <int NP, int V, bool COPY>
__device__ __forceinline__ unsigned msb_tiles(const FusedReluParty& p, const PackedTriples& g, const Wire<NP, COPY>& wire, int party,
                                              unsigned tile, unsigned tile0, unsigned end, size_t at0, size_t n)
{
    if (tile >= end) return tile;
    unsigned lane = threadIdx.x % kWave;
    auto base_of = [&](unsigned t) { return at0 + (size_t)(t - tile0) * (kWave * V); };
    auto off_of = [&](size_t b) {
        const unsigned rest = V == 1 && n - b < kWave ? (unsigned)(n - b) - 1 : kWave * V - V;      // V > 1: whole tiles only
        return lane * V < rest ? lane * V : rest;
    };
    size_t base = base_of(tile);
    unsigned off = off_of(base);
    auto row = [&](const u64* q) { return ld_once<V>(q + base, off * 8u); };
    Head<NP, V> h;
    load_masks(h, p, row);
    Pack<V> x = row(p.x);
    load_first(h, p, row);
    for (;;) {
        const unsigned after = tile + gridDim.x;
        const bool more = after < end;
        const size_t next_base = base_of(more ? after : tile);
        unsigned next_off = off_of(next_base);
        auto next_row = [&](const u64* q) { return ld_once<V>(q + next_base, next_off * 8u); };
        asm volatile("" : "+v"(off), "+v"(lane), "+v"(next_off));
        Head<NP, V> nh; Pack<V> nx;
        const Converted<V> r = convert_packed<NP, V, false>(p, g, wire, party, lane, base, x, h, off, p.rb + base, row,
                                                            [&] { if (more) load_masks(nh, p, next_row); },
                                                            [&] { if (more) { nx = next_row(p.x); load_first(nh, p, next_row); } });
        if (off == lane * V) {            // else past the end: a lane that worked on the last element again, at another bit position
            st_words<V>(p.y + base, off * 8u, r.y);
            if (p.s_bit) st_flags<V>(p.s_bit + base + off, r.s);
            if (p.s_arith) st_words<V>(p.s_arith + base, off * 8u, r.sa);
        }
        if (!more) return after;
        tile = after; base = next_base; off = next_off; h = nh; x = nx;
    }
}

// tiles 0 .. wide-1: 64 V elements each, V per lane; the others 64 elements, one per lane (the last one ragged).  Two
// parties: four per lane, the rounds and the vector work of the deeper levels shared by twice the elements of two per lane
// (2 097 152 elements 150 -> 135 us on one box, 143 -> 137 on another; VGG16 of 32 images on one lane 2.31 -> 2.25 ms, on four
// lanes, where the 168 registers no longer fit beside the GEMM's, 0.7 % more).  A launch writes 121 MiB, of which 32 are
// results, with two per lane 47: the buffers are 8 MB either way, but rows of four words a lane leave the L2 more often.  Three
// parties: two per lane (four 2 % slower).
constexpr int msb_v(int parties) { return parties == 2 ? 4 : 2; }
constexpr size_t msb_box(int v) { return 2 * kWave * (size_t)v; }      // words: two rows of whole words, or four of level 0
template <int NP, bool COPY>
__global__ __launch_bounds__(NP * kWave, NP == 2 ? 3 : 4) void k_relu_fused_msb(FusedRelu q, PackedTriples g, unsigned wide)
{
    const int party = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const Wire<NP, COPY> wire(q.box, party, msb_box(wide ? msb_v(NP) : 1));
    const unsigned tile = msb_tiles<NP, msb_v(NP)>(q.p[party], g, wire, party, blockIdx.x, 0, wide, 0, q.n);
    msb_tiles<NP, 1>(q.p[party], g, wire, party, tile, wide, q.tiles, (size_t)wide * msb_v(NP) * kWave, q.n);
}

constexpr size_t kPoolBox = (size_t)kRows * kWave * 2;        // words: four rows of the first level's pairs
// ---- 2x2 max-pool: two tournament levels, each max(p, q) = q + ReLU(p - q) ----------------
// A wave works on 64 outputs: the first level's pair of differences of an output are two elements of one lane, the
// second level's difference one, so both conversions and the sums around them stay in registers.
// The window and the first masks of the next tile are loaded under the second conversion's last rounds.
// 32 x 32 x 32 x 64 inputs (524 288 outputs): 0.283 ms as gathers, two one-launch conversions and a sum (eight launches),
// 0.251 ms here (whole words; 512 workgroups 0.311 ms), sign-only 0.145 -> 0.137 ms; 32 x 8 x 8 x 256: 81 -> 64 us.
template <int NP, bool PACKED, int TOPO>
__global__ __launch_bounds__(NP * kWave, PACKED ? 4 : 3) void k_maxpool_fused(FusedPool q, PackedTriples g1, PackedTriples g2)
{
    const int party = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const Wire<NP> wire(q.box, party, kPoolBox);
    const FusedReluParty &p1 = q.m1[party], &p2 = q.m2[party];
    const u64* const x = q.x[party];
    const unsigned C = (unsigned)q.C, Wo = (unsigned)q.W / 2, Ho = (unsigned)q.H / 2;
    unsigned lane = threadIdx.x % kWave;
    unsigned tile = blockIdx.x;
    // a tile's first output and the lane's place in it (past the end: the last output again, not stored)
    auto at_of = [&](size_t o0) {
        const unsigned last = q.n_out - o0 < kWave ? (unsigned)(q.n_out - o0) - 1 : kWave - 1;
        return lane < last ? lane : last;
    };
    struct Window { u64 p00, p01, p10, p11; };
    auto window = [&](size_t o0, unsigned at) {
        size_t t = o0 + at;
        const unsigned ch = (unsigned)(t % C); t /= C;
        const unsigned wo = (unsigned)(t % Wo); t /= Wo;
        const unsigned ho = (unsigned)(t % Ho); const size_t b = t / Ho;
        const u64* const w = x + ((b * q.H + 2 * ho) * q.W + 2 * wo) * C + ch;
        const size_t dh = (size_t)q.W * C;
        return Window{ w[0], w[C], w[dh], w[dh + C] };
    };
    size_t o0 = (size_t)tile * kWave;
    unsigned at = at_of(o0);
    auto row1 = [&](const u64* m) { return ld_once<2>(m + 2 * o0, at * 16u); };
    auto row2 = [&](const u64* m) { return ld_once<1>(m + o0, at * 8u); };
    Head<NP, 2> h1;
    load_masks(h1, p1, row1);
    Window w = window(o0, at);
    load_first(h1, p1, row1);
    for (;;) {
        const unsigned after = tile + gridDim.x;
        const bool more = after < q.tiles;
        const size_t next_o0 = (size_t)(more ? after : tile) * kWave;
        unsigned next_at = at_of(next_o0);
        auto next_row1 = [&](const u64* m) { return ld_once<2>(m + 2 * next_o0, next_at * 16u); };
        asm volatile("" : "+v"(at), "+v"(lane), "+v"(next_at));
        Head<NP, 1> h2;
        auto masks2 = [&] { load_masks(h2, p2, row2); };
        auto first2 = [&] { load_first(h2, p2, row2); };
        Pack<2> d1;
        d1.v[0] = w.p00 - w.p01; d1.v[1] = w.p10 - w.p11;
        Converted<2> r1;
        if constexpr (PACKED) r1 = convert_packed<NP, 2, true>(p1, g1, wire, party, lane, 2 * o0, d1, h1, 2 * at, p1.rb + 2 * o0, row1, masks2, first2);
        else                  r1 = convert_words<NP, 2, TOPO>(p1, wire, party, lane, lane * 16u, 2 * q.n_out, d1, h1, 2 * at, p1.rb + 2 * o0, row1, masks2, first2);
        const u64 u = w.p01 + r1.y.v[0], v = w.p11 + r1.y.v[1];
        Pack<1> d2;
        d2.v[0] = u - v;
        asm volatile("" : "+v"(at), "+v"(lane));
        Head<NP, 2> nh; Window nw;
        auto masks1 = [&] { if (more) load_masks(nh, p1, next_row1); };
        auto first1 = [&] { if (more) { nw = window(next_o0, next_at); load_first(nh, p1, next_row1); } };
        Converted<1> r2;
        if constexpr (PACKED) r2 = convert_packed<NP, 1, false>(p2, g2, wire, party, lane, o0, d2, h2, at, p2.rb + o0, row2, masks1, first1);
        else                  r2 = convert_words<NP, 1, TOPO>(p2, wire, party, lane, lane * 8u, q.n_out, d2, h2, at, p2.rb + o0, row2, masks1, first1);
        if (at == lane) {
            q.y[party][o0 + at] = v + r2.y.v[0];
            if (q.s1[party]) st_words<2>(q.s1[party] + 2 * o0, at * 16u, r1.sa);
            if (q.s2[party]) q.s2[party][o0 + at] = r2.sa.v[0];
        }
        if (!more) break;
        tile = after; o0 = next_o0; at = next_at; h1 = nh; w = nw;
    }
}

// Workgroups of a launch, [parties - 2]: as many as their receive buffers fit the L2 of their XCD (a three-party
// workgroup has six of them).  Whole words, 2 097 152 elements: two parties 512 / 1024 / 2048 workgroups 0.315 / 0.307 /
// 0.315 ms; three parties 384 / 512 / 640 / 768 / 1024 workgroups 0.707 / 0.592 / 0.680 / 0.624 / 0.639 ms (2.12 ms as eleven
// launches), 300 000 elements 111 / 95 / 102 / 100 / 104 us.
// Sign-only: two parties 768 / 1024 / 1280 workgroups 0.144 / 0.141 / 0.145 ms; three parties 768 .. 2048 workgroups level
// (0.99 ms as eleven launches).
constexpr unsigned kBlocks[2] = { 1024, 512 }, kMsbBlocks[2] = { 1024, 1536 }, kMsbPoolBlocks[2] = { 2048, 1536 };
constexpr int kMaxBlockPairs[2] = { 2, 6 };        // ordered pairs of parties: receive buffers per workgroup

// two elements per thread (16-byte accesses) once one element per thread would need a second round of workgroups
int width(size_t n, unsigned blocks) { return n > (size_t)blocks * kWave ? 2 : 1; }
unsigned tiles_of(size_t n, int v) { return (unsigned)((n + kWave * v - 1) / (kWave * v)); }
// sign-only chain: wide tiles and all tiles of a call
unsigned wide_tiles(int parties, size_t n)
{
    return width(n, kMsbBlocks[parties - 2]) == 2 ? (unsigned)(n / (kWave * msb_v(parties))) : 0;
}
unsigned msb_tile_count(int parties, size_t n)
{
    const unsigned wide = wide_tiles(parties, n);
    return wide + tiles_of(n - (size_t)wide * kWave * msb_v(parties), 1);
}
unsigned least(unsigned a, unsigned b) { return a < b ? a : b; }

template <int NP, int V, bool COPY>
void launch(hipStream_t st, const FusedRelu& q, int topo)
{
    const dim3 grid(least(q.tiles, kBlocks[NP - 2])), block(NP * kWave);
    if constexpr (NP == 2)
        if (topo) { hipLaunchKernelGGL((k_relu_fused<NP, V, 1, COPY>), grid, block, 0, st, q); return; }
    hipLaunchKernelGGL((k_relu_fused<NP, V, 0, COPY>), grid, block, 0, st, q);
}

}  // namespace

size_t relu_fused_box_bytes(int parties, size_t n, bool copies)
{
    const unsigned blocks = kBlocks[parties - 2];
    const int v = width(n, blocks);
    return (size_t)least(tiles_of(n, v), blocks) * kMaxBlockPairs[parties - 2] * (copies ? 2 : 1) * (kRows * kWave * v) * sizeof(u64);
}

int launch_relu_fused(mpc_ctx* c, hipStream_t st, int parties, FusedRelu q, int topo, bool copies)
{
    if (q.n == 0 || q.n >= ((size_t)1 << 37) || (copies && parties != 2)) return MPC_EINVAL;
    const int v = width(q.n, kBlocks[parties - 2]);
    q.tiles = tiles_of(q.n, v);
    if (copies)            { if (v == 2) launch<2, 2, true>(st, q, topo);  else launch<2, 1, true>(st, q, topo); }
    else if (parties == 2) { if (v == 2) launch<2, 2, false>(st, q, topo); else launch<2, 1, false>(st, q, topo); }
    else                   { if (v == 2) launch<3, 2, false>(st, q, 0);    else launch<3, 1, false>(st, q, 0); }
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

size_t relu_fused_msb_box_bytes(int parties, size_t n, bool copies)
{
    return (size_t)least(msb_tile_count(parties, n), kMsbBlocks[parties - 2]) * kMaxBlockPairs[parties - 2] * (copies ? 2 : 1) *
           msb_box(wide_tiles(parties, n) ? msb_v(parties) : 1) * sizeof(u64);
}

int launch_relu_fused_msb(mpc_ctx* c, hipStream_t st, int parties, FusedRelu q, const PackedTriples& g, bool copies)
{
    if (q.n == 0 || q.n >= ((size_t)1 << 37) || (copies && parties != 2)) return MPC_EINVAL;
    const unsigned blocks = kMsbBlocks[parties - 2], wide = wide_tiles(parties, q.n);
    q.tiles = msb_tile_count(parties, q.n);
    const dim3 grid(least(q.tiles, blocks));
    if (copies)            hipLaunchKernelGGL((k_relu_fused_msb<2, true>), grid, dim3(2 * kWave), 0, st, q, g, wide);
    else if (parties == 2) hipLaunchKernelGGL((k_relu_fused_msb<2, false>), grid, dim3(2 * kWave), 0, st, q, g, wide);
    else                   hipLaunchKernelGGL((k_relu_fused_msb<3, false>), grid, dim3(3 * kWave), 0, st, q, g, wide);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

size_t maxpool_fused_box_bytes(int parties, bool packed, size_t n_out)
{
    const unsigned blocks = (packed ? kMsbPoolBlocks : kBlocks)[parties - 2];
    return (size_t)least(tiles_of(n_out, 1), blocks) * kMaxBlockPairs[parties - 2] * kPoolBox * sizeof(u64);
}

int launch_maxpool_fused(mpc_ctx* c, hipStream_t st, int parties, FusedPool q, int topo, const PackedTriples* g1, const PackedTriples* g2)
{
    if (q.n_out == 0 || q.n_out >= ((size_t)1 << 36)) return MPC_EINVAL;
    const bool packed = g1 != nullptr;
    q.tiles = tiles_of(q.n_out, 1);
    const dim3 grid(least(q.tiles, (packed ? kMsbPoolBlocks : kBlocks)[parties - 2])), block(parties * kWave);
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
