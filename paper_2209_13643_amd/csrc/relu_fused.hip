// Secure ReLU, all rounds in one launch (exchange by remote store on a single-queue lane).
//
// A workgroup is one wave per party, and both waves work on the same elements.  A party's wave reads its own share,
// its own material and what it has received; a round's masked words are stored into the peer's receive buffer in
// device memory, and the workgroup barrier that follows is the round: nothing but the two waves of a workgroup
// depends on each other, so no wave ever waits for another workgroup.  Between rounds (G, P) stay in registers, and a
// receive buffer holds one round of one workgroup's elements, so what streams from HBM is the input, the offline
// material and the output, each once: 690 bytes per element of both parties instead of the 2498 that one launch per
// round moves.  2 097 152 elements: 0.95 ms as ten launches, 0.323 ms here (4.5 TB/s of compulsory bytes).
//
// What bounds it is the vector memory path: a build that exchanges through LDS takes 0.25 ms (5.8 TB/s, what a large
// copy reaches), the stores of the masked words cost 0.05 and their loads 0.035 ms of the difference.  The receive
// buffers have to stay in the L2: with a grid of 2048 workgroups and two buffers per party (33 MB) they were written
// back to memory (0.64 GB per call) and the call took 0.345 ms; with one buffer and a second barrier per round, and 1024
// workgroups, they are 8 MB, and four lanes converting at once still fit (batch-128 VGG16 on four lanes: 11.7 ms with
// two buffers, 11.2 ms with one).  The material is read once, hence the non-temporal loads (0.376 -> 0.345 ms).
#include "common.h"
#include "relu_steps.h"
#include "relu_fused.h"

#include <type_traits>

namespace {

constexpr int kWave = 64;
constexpr int kRows = 4;            // most words an element sends in one round

typedef u64 u64v2u __attribute__((ext_vector_type(2), aligned(8)));

// V consecutive words at scalar base + 32-bit byte offset, any 8-byte aligned address, read once
template <int V> __device__ __forceinline__ Pack<V> ld_once(const u64* p, unsigned off)
{
    const u8* a = reinterpret_cast<const u8*>(p) + off;
    Pack<V> r;
    if constexpr (V >= 2) {
#pragma unroll
        for (int k = 0; k < V; k += 2) {
            const u64v2u t = __builtin_nontemporal_load(reinterpret_cast<const u64v2u*>(a + 8 * k));
            r.v[k] = t.x; r.v[k + 1] = t.y;
        }
    }
    else r.v[0] = __builtin_nontemporal_load(reinterpret_cast<const u64*>(a));
    return r;
}

template <int V> __device__ __forceinline__ void st_words(u64* p, unsigned off, const Pack<V>& w)
{
    u8* a = reinterpret_cast<u8*>(p) + off;
    if constexpr (V == 1) *reinterpret_cast<u64*>(a) = w.v[0];
#pragma unroll
    for (int k = 0; k + 1 < V; k += 2) *reinterpret_cast<u64v2u*>(a + 8 * k) = u64v2u{ w.v[k], w.v[k + 1] };
}
// V consecutive bytes at any address, one per element
template <int V> struct ByteWord;
template <> struct ByteWord<1> { typedef u8 type; };
template <> struct ByteWord<2> { typedef uint16_t type __attribute__((aligned(1))); };
template <> struct ByteWord<4> { typedef uint32_t type __attribute__((aligned(1))); };
template <int V> __device__ __forceinline__ unsigned ld_flags(const u8* p) { return *reinterpret_cast<const typename ByteWord<V>::type*>(p); }
template <int V> __device__ __forceinline__ void st_flags(u8* p, unsigned w) { *reinterpret_cast<typename ByteWord<V>::type*>(p) = (typename ByteWord<V>::type)w; }

template <int V, int TOPO>
__global__ __launch_bounds__(2 * kWave, 4) void k_relu_fused(FusedRelu q)
{
    const int party = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int lane = threadIdx.x % kWave;
    const FusedReluParty& p = q.p[party];
    const size_t n = q.n;
    const u64 m0 = party == 0 ? ~(u64)0 : 0;             // the party that adds the product of the opened words
    constexpr size_t kBox = (size_t)kRows * kWave * V;
    u64* const in = q.box + ((size_t)blockIdx.x * 2 + party) * kBox;
    u64* const out = q.box + ((size_t)blockIdx.x * 2 + (party ^ 1)) * kBox;
    unsigned slot = lane * V * 8u;
    // row `row` of this round's words, into the peer's receive buffer / out of the own one
    auto put = [&](int row, const Pack<V>& w) { w.st(reinterpret_cast<u64*>(reinterpret_cast<u8*>(out) + (slot + row * kWave * V * 8u)), 0); };
    auto get = [&](int row) { return Pack<V>::ld(reinterpret_cast<const u64*>(reinterpret_cast<const u8*>(in) + (slot + row * kWave * V * 8u)), 0); };
    auto opened = [] { __syncthreads(); };      // both waves have stored their words of the round
    auto drained = [] { __syncthreads(); };     // both waves hold the words of the last round: the buffers are free
    auto fin = [&](u64 d, u64 g, u64 a, u64 b, u64 c) { return c ^ (d & b) ^ (g & a) ^ (d & g & m0); };

    for (size_t tile = blockIdx.x; tile < q.tiles; tile += gridDim.x) {
        // the wave's elements: base + off .. ; a ragged last tile takes the last 64 V elements and stores its own only
        const size_t first = tile * (kWave * V);
        const size_t base = first + kWave * V <= n ? first : n >= kWave * V ? n - kWave * V : 0;
        const unsigned rest = n < kWave * V ? (unsigned)n - V : kWave * V - V;
        unsigned off = lane * V < rest ? lane * V : rest;
        // opaque per tile: otherwise the addresses of all 43 rows are formed ahead of the loop and spilled
        asm volatile("" : "+v"(off), "+v"(slot));
        auto row = [&](const u64* t) { return ld_once<V>(t + base, off * 8u); };
        auto tri = [&](const u64* t, int k) { return row(t + (size_t)k * n); };

        const Pack<V> x = row(p.x), r = row(p.r);
        Pack<V> a1 = tri(p.ta, 0), b1 = tri(p.tb, 0), c1 = tri(p.tc, 0), a2, b2, c2;
        drained();
        put(0, r);                                                     // Alg. 2: the mask half of the own word
        opened();
        Pack<V> P, G, sd, sg;
        u64 top[V];
        {
            const Pack<V> rr = get(0);
#pragma unroll
            for (int k = 0; k < V; ++k) {
                const u64 o = x.v[k] ^ r.v[k], U = party == 0 ? o : rr.v[k], Vv = party == 0 ? rr.v[k] : o;
                sd.v[k] = U ^ a1.v[k]; sg.v[k] = Vv ^ b1.v[k];
                P.v[k] = U ^ Vv; top[k] = P.v[k] >> 63;
            }
            drained();
            put(0, sd); put(1, sg);
        }
        Pack<V> na1 = tri(p.ta, 1), nb1 = tri(p.tb, 1), nc1 = tri(p.tc, 1);
        Pack<V> na2 = tri(p.ta, 2), nb2 = tri(p.tb, 2), nc2 = tri(p.tc, 2);
        opened();
        {
            const Pack<V> rd = get(0), rg = get(1);
#pragma unroll
            for (int k = 0; k < V; ++k) G.v[k] = fin(sd.v[k] ^ rd.v[k], sg.v[k] ^ rg.v[k], a1.v[k], b1.v[k], c1.v[k]);
        }
        // prefix levels: mask and send level L's operands, fetch the next level's triples, open, finish
        auto level = [&](auto tag) {
            constexpr int L = decltype(tag)::value;
            a1 = na1; b1 = nb1; c1 = nc1; a2 = na2; b2 = nb2; c2 = nc2;
            Pack<V> d1, g1, d2, g2;
#pragma unroll
            for (int k = 0; k < V; ++k) {
                const u64 X = op_x<TOPO, L>(P.v[k]);
                d1.v[k] = X ^ a1.v[k]; g1.v[k] = op_y<TOPO, L>(G.v[k]) ^ b1.v[k];
                if constexpr (L < 5) { d2.v[k] = X ^ a2.v[k]; g2.v[k] = op_y<TOPO, L>(P.v[k]) ^ b2.v[k]; }
            }
            drained();
            put(0, d1); put(1, g1);
            if constexpr (L < 5) { put(2, d2); put(3, g2); }
            if constexpr (L < 5) { na1 = tri(p.ta, 3 + 2 * L); nb1 = tri(p.tb, 3 + 2 * L); nc1 = tri(p.tc, 3 + 2 * L); }
            if constexpr (L < 4) { na2 = tri(p.ta, 4 + 2 * L); nb2 = tri(p.tb, 4 + 2 * L); nc2 = tri(p.tc, 4 + 2 * L); }
            opened();
            const Pack<V> rd1 = get(0), rg1 = get(1);
            Pack<V> rd2, rg2;
            if constexpr (L < 5) { rd2 = get(2); rg2 = get(3); }
#pragma unroll
            for (int k = 0; k < V; ++k) {
                G.v[k] ^= fin(d1.v[k] ^ rd1.v[k], g1.v[k] ^ rg1.v[k], a1.v[k], b1.v[k], c1.v[k]);
                if constexpr (L < 5)
                    P.v[k] = keep_p<TOPO, L>(P.v[k]) ^ fin(d2.v[k] ^ rd2.v[k], g2.v[k] ^ rg2.v[k], a2.v[k], b2.v[k], c2.v[k]);
            }
        };
        level(std::integral_constant<int, 0>{}); level(std::integral_constant<int, 1>{}); level(std::integral_constant<int, 2>{});
        level(std::integral_constant<int, 3>{}); level(std::integral_constant<int, 4>{}); level(std::integral_constant<int, 5>{});

        // sign share = bit 63 of U ^ V xor the carry out of bits 0..62; masked with the random bit and opened
        const Pack<V> ra = row(p.ra), ma = row(p.ma), mb = row(p.mb), mc = row(p.mc);
        const unsigned rb = ld_flags<V>(p.rb + base + off);
        unsigned s = 0;                                                // the bits of an element are bytes of s
#pragma unroll
        for (int k = 0; k < V; ++k) s |= (unsigned)(top[k] ^ ((G.v[k] >> 62) & 1)) << (8 * k);
        drained();
        st_flags<V>(reinterpret_cast<u8*>(out) + lane * V, s ^ rb);
        opened();
        const unsigned v = s ^ rb ^ ld_flags<V>(reinterpret_cast<const u8*>(in) + lane * V);
        Pack<V> sa, e, f;
#pragma unroll
        for (int k = 0; k < V; ++k) {
            // s = v xor rb = v + rb - 2 v rb on additive shares of rb
            const u64 vk = (v >> (8 * k)) & 1;
            sa.v[k] = (vk ? (u64)0 - ra.v[k] : ra.v[k]) + (vk & m0);
            e.v[k] = x.v[k] - ma.v[k];
            f.v[k] = (m0 & 1) - sa.v[k] - mb.v[k];
        }
        drained();
        put(0, e); put(1, f);
        opened();
        Pack<V> y;
        {
            const Pack<V> re = get(0), rf = get(1);
#pragma unroll
            for (int k = 0; k < V; ++k) {
                const u64 eo = e.v[k] + re.v[k], fo = f.v[k] + rf.v[k];
                y.v[k] = mc.v[k] + eo * (mb.v[k] + (fo & m0)) + ma.v[k] * fo;
            }
        }
        if (base + off >= first) {
            st_words<V>(p.y + base, off * 8u, y);
            if (p.s_bit) st_flags<V>(p.s_bit + base + off, s);
            if (p.s_arith) st_words<V>(p.s_arith + base, off * 8u, sa);
        } else if (V == 2 && base + off + 1 == first) {                // an odd count: only the second element is the tile's own
            (p.y + base)[off + 1] = y.v[V - 1];
            if (p.s_bit) (p.s_bit + base)[off + 1] = (u8)(s >> 8);
            if (p.s_arith) (p.s_arith + base)[off + 1] = sa.v[V - 1];
        }
    }
}

// ---- sign-only chain on packed words ------------------------------------------------
// A wave works on 64 V elements.  Level l keeps one word per 2^(l+1) elements: the first log2(V) levels combine two
// words of the same lane, every later one the words of lanes j and j ^ d: both lanes form the same word, load the same
// triple words and store the same masked words, so no lane ever moves data and element k of the lane finds its carry
// in the lane's own word at the end.
// 2 097 152 elements: 0.378 ms as ten launches, 0.141 ms here (256 compulsory bytes per element: 3.8 TB/s; what is
// left is the vector memory path of the exchange, as for whole words).  Four elements per lane, whose loads touch every
// line twice: 0.144 ms; 1024 workgroups: 0.145 ms.
__device__ __forceinline__ u64 from_lane_xor(u64 v, int mask)
{
    const unsigned lo = __shfl_xor((unsigned)v, mask), hi = __shfl_xor((unsigned)(v >> 32), mask);
    return ((u64)hi << 32) | lo;
}

struct MsbTile {
    const FusedReluParty& p; const MsbGeom& g;
    u64 *in, *out;
    int party, lane;
    u64 m0;
};

template <int W> struct LevelTriples { Pack<W> a1, b1, c1, a2, b2, c2; };

template <int V>
__device__ __forceinline__ void msb_tile(const MsbTile& t, size_t base, size_t n)
{
    const FusedReluParty& p = t.p;
    const u64 m0 = t.m0;
    const unsigned rest = V == 1 && n - base < kWave ? (unsigned)(n - base) - 1 : kWave * V - V;
    unsigned off = t.lane * V < rest ? t.lane * V : rest;         // V > 1: the caller passes whole tiles only
    unsigned lane = t.lane;
    asm volatile("" : "+v"(off), "+v"(lane));
    auto row = [&](const u64* q) { return ld_once<V>(q + base, off * 8u); };
    auto opened = [] { __syncthreads(); };
    auto drained = [] { __syncthreads(); };
    auto fin = [&](u64 d, u64 g, u64 a, u64 b, u64 c) { return c ^ (d & b) ^ (g & a) ^ (d & g & m0); };
    // words at word index `w` of the peer's / the own receive buffer; rows of whole words and of packed words
    constexpr unsigned kWhole = kWave * V, kPacked = kWave * V / 2;
    auto put = [&](unsigned w, const auto& v) { v.st(reinterpret_cast<u64*>(reinterpret_cast<u8*>(t.out) + w * 8u), 0); };
    auto get = [&](unsigned w, auto tag) {
        return Pack<decltype(tag)::value>::ld(reinterpret_cast<const u64*>(reinterpret_cast<const u8*>(t.in) + w * 8u), 0);
    };
    typedef std::integral_constant<int, V> VT;

    // level L: a lane forms words(L) words, at word index at(L) of the tile
    auto at = [&](auto tag) { constexpr int L = decltype(tag)::value; return (2 << L) <= V ? lane * (V >> (L + 1)) : (lane * V) >> (L + 1); };
    auto triples = [&](auto tag) {
        constexpr int L = decltype(tag)::value, W = (2 << L) <= V ? V >> (L + 1) : 1;
        const unsigned w = at(tag);
        auto tri = [&](const u64* q, int k) { return ld_once<W>(q + t.g.toff[k] + (base >> (L + 1)), w * 8u); };
        LevelTriples<W> r;
        r.a1 = tri(p.ta, 1 + 2 * L); r.b1 = tri(p.tb, 1 + 2 * L); r.c1 = tri(p.tc, 1 + 2 * L);
        if constexpr (L < 5) { r.a2 = tri(p.ta, 2 + 2 * L); r.b2 = tri(p.tb, 2 + 2 * L); r.c2 = tri(p.tc, 2 + 2 * L); }
        return r;
    };

    const Pack<V> x = row(p.x), r = row(p.r), a0 = row(p.ta), b0 = row(p.tb), c0 = row(p.tc);
    drained();
    put(lane * V, r);
    opened();
    Pack<V> P, G, sd, sg;
    LevelTriples<V == 1 ? 1 : V / 2> t0;
    u64 top = 0;                                                  // bit k: bit 63 of U ^ V of element k
    {
        const Pack<V> rr = get(lane * V, VT{});
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const u64 o = x.v[k] ^ r.v[k], U = t.party == 0 ? o : rr.v[k], Vv = t.party == 0 ? rr.v[k] : o;
            sd.v[k] = U ^ a0.v[k]; sg.v[k] = Vv ^ b0.v[k];
            P.v[k] = U ^ Vv; top |= (P.v[k] >> 63) << k;
        }
        drained();
        put(lane * V, sd); put(lane * V + kWhole, sg);
        t0 = triples(std::integral_constant<int, 0>{});
        opened();
        const Pack<V> rd = get(lane * V, VT{}), rg = get(lane * V + kWhole, VT{});
#pragma unroll
        for (int k = 0; k < V; ++k) G.v[k] = fin(sd.v[k] ^ rd.v[k], sg.v[k] ^ rg.v[k], a0.v[k], b0.v[k], c0.v[k]);
    }
    // mask and send, fetch the next level's triples (returned), open and finish
    auto level = [&](auto tag, const auto& tr) {
        constexpr int L = decltype(tag)::value, d = 1 << L;
        constexpr u64 A = sel_mask(L), B = low_mask(L);
        constexpr bool inlane = (2 << L) <= V;
        constexpr int W = inlane ? V >> (L + 1) : 1;
        const unsigned w = at(tag);
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
        drained();
        put(w, d1); put(w + kPacked, g1);
        if constexpr (L < 5) { put(w + 2 * kPacked, d2); put(w + 3 * kPacked, g2); }
        constexpr int W1 = (4 << L) <= V ? V >> (L + 2) : 1;
        LevelTriples<W1> next;
        if constexpr (L < 5) next = triples(std::integral_constant<int, L + 1>{});
        opened();
        typedef std::integral_constant<int, W> WT;
        const Pack<W> rd1 = get(w, WT{}), rg1 = get(w + kPacked, WT{});
        Pack<W> rd2, rg2;
        if constexpr (L < 5) { rd2 = get(w + 2 * kPacked, WT{}); rg2 = get(w + 3 * kPacked, WT{}); }
#pragma unroll
        for (int k = 0; k < W; ++k) {
            G.v[k] = Gk.v[k] ^ fin(d1.v[k] ^ rd1.v[k], g1.v[k] ^ rg1.v[k], tr.a1.v[k], tr.b1.v[k], tr.c1.v[k]);
            if constexpr (L < 5) P.v[k] = fin(d2.v[k] ^ rd2.v[k], g2.v[k] ^ rg2.v[k], tr.a2.v[k], tr.b2.v[k], tr.c2.v[k]);
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

    // element i's carry into bit 63 sits at bit (62 + i) mod 64 of word i / 64; the bits of an element are bytes of s
    const unsigned rb = ld_flags<V>(p.rb + base + off);
    unsigned s = 0;
#pragma unroll
    for (int k = 0; k < V; ++k) s |= (unsigned)(((top >> k) ^ (G.v[0] >> ((62 + lane * V + k) & 63))) & 1) << (8 * k);
    drained();
    st_flags<V>(reinterpret_cast<u8*>(t.out) + lane * V, s ^ rb);
    opened();
    const unsigned v = s ^ rb ^ ld_flags<V>(reinterpret_cast<const u8*>(t.in) + lane * V);
    Pack<V> sa, e, f;
#pragma unroll
    for (int k = 0; k < V; ++k) {
        // s = v xor rb = v + rb - 2 v rb on additive shares of rb
        const u64 vk = (v >> (8 * k)) & 1;
        sa.v[k] = (vk ? (u64)0 - ra.v[k] : ra.v[k]) + (vk & m0);
        e.v[k] = x.v[k] - ma.v[k];
        f.v[k] = (m0 & 1) - sa.v[k] - mb.v[k];
    }
    drained();
    put(lane * V, e); put(lane * V + kWhole, f);
    opened();
    Pack<V> y;
    {
        const Pack<V> re = get(lane * V, VT{}), rf = get(lane * V + kWhole, VT{});
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const u64 eo = e.v[k] + re.v[k], fo = f.v[k] + rf.v[k];
            y.v[k] = mc.v[k] + eo * (mb.v[k] + (fo & m0)) + ma.v[k] * fo;
        }
    }
    if (off != lane * V) return;              // past the end: a lane that worked on the last element again, at another bit position
    st_words<V>(p.y + base, off * 8u, y);
    if (p.s_bit) st_flags<V>(p.s_bit + base + off, s);
    if (p.s_arith) st_words<V>(p.s_arith + base, off * 8u, sa);
}

// tiles 0 .. wide-1: 128 elements each, two per lane; the others 64 elements, one per lane (the last one ragged)
constexpr int kMsbV = 2;
constexpr size_t kMsbBox = 2 * kWave * kMsbV;      // words: two rows of whole words, or four of level 0
__global__ __launch_bounds__(2 * kWave, 4) void k_relu_fused_msb(FusedRelu q, MsbGeom g, unsigned wide)
{
    const int party = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    constexpr size_t kBox = kMsbBox;
    const MsbTile t{ q.p[party], g, q.box + ((size_t)blockIdx.x * 2 + party) * kBox, q.box + ((size_t)blockIdx.x * 2 + (party ^ 1)) * kBox,
                     party, (int)(threadIdx.x % kWave), party == 0 ? ~(u64)0 : 0 };
    for (unsigned tile = blockIdx.x; tile < q.tiles; tile += gridDim.x) {
        if (tile < wide) msb_tile<kMsbV>(t, (size_t)tile * kWave * kMsbV, q.n);
        else             msb_tile<1>(t, ((size_t)wide * kMsbV + (tile - wide)) * kWave, q.n);
    }
}

constexpr int kFusedBlocks = 1024;      // two waves per SIMD; 512 and 2048 workgroups are 4 and 2 % slower

template <int V> unsigned fused_tiles(size_t n) { return (unsigned)((n + kWave * V - 1) / (kWave * V)); }
// two elements per thread (16-byte accesses) once one element per thread would need a second round of workgroups
inline int fused_width(size_t n) { return n > (size_t)kFusedBlocks * kWave ? 2 : 1; }

template <int V>
int launch(mpc_ctx* c, hipStream_t st, FusedRelu& q, int topo)
{
    q.tiles = fused_tiles<V>(q.n);
    const dim3 grid(q.tiles < (unsigned)kFusedBlocks ? q.tiles : kFusedBlocks), block(2 * kWave);
    if (topo) hipLaunchKernelGGL((k_relu_fused<V, 1>), grid, block, 0, st, q);
    else      hipLaunchKernelGGL((k_relu_fused<V, 0>), grid, block, 0, st, q);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

}  // namespace

size_t relu_fused_box_bytes(size_t n)
{
    const int v = fused_width(n);
    const size_t tiles = v == 2 ? fused_tiles<2>(n) : fused_tiles<1>(n);
    return (tiles < kFusedBlocks ? tiles : kFusedBlocks) * 2 * (kRows * kWave * v) * sizeof(u64);
}

int launch_relu_fused(mpc_ctx* c, hipStream_t st, FusedRelu q, int topo)
{
    if (q.n == 0 || q.n >= ((size_t)1 << 37)) return MPC_EINVAL;
    return fused_width(q.n) == 2 ? launch<2>(c, st, q, topo) : launch<1>(c, st, q, topo);
}

constexpr int kMsbBlocks = 2048;
// two elements per lane once one per lane would need a second round of workgroups
static unsigned msb_wide_tiles(size_t n) { return n > (size_t)kMsbBlocks * kWave ? (unsigned)(n / (kWave * kMsbV)) : 0; }
static unsigned msb_tiles(size_t n)
{
    const unsigned wide = msb_wide_tiles(n);
    return wide + (unsigned)((n - (size_t)wide * kWave * kMsbV + kWave - 1) / kWave);
}

size_t relu_fused_msb_box_bytes(size_t n)
{
    const size_t tiles = msb_tiles(n);
    return (tiles < kMsbBlocks ? tiles : kMsbBlocks) * 2 * kMsbBox * sizeof(u64);
}

int launch_relu_fused_msb(mpc_ctx* c, hipStream_t st, FusedRelu q, const MsbGeom& g)
{
    if (q.n == 0 || q.n >= ((size_t)1 << 37)) return MPC_EINVAL;
    q.tiles = msb_tiles(q.n);
    hipLaunchKernelGGL(k_relu_fused_msb, dim3(q.tiles < kMsbBlocks ? q.tiles : kMsbBlocks), dim3(2 * kWave), 0, st, q, g, msb_wide_tiles(q.n));
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}
