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

namespace {

constexpr int kWave = 64;
constexpr int kRows = 4;            // most words an element sends in one round

typedef u64 u64v2u __attribute__((ext_vector_type(2), aligned(8)));

// V consecutive words at scalar base + 32-bit byte offset, any 8-byte aligned address, read once
template <int V> __device__ __forceinline__ Pack<V> ld_once(const u64* p, unsigned off)
{
    const u8* a = reinterpret_cast<const u8*>(p) + off;
    Pack<V> r;
    if constexpr (V == 2) { const u64v2u t = __builtin_nontemporal_load(reinterpret_cast<const u64v2u*>(a)); r.v[0] = t.x; r.v[1] = t.y; }
    else r.v[0] = __builtin_nontemporal_load(reinterpret_cast<const u64*>(a));
    return r;
}

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
        u64 s[V], masked[V];
#pragma unroll
        for (int k = 0; k < V; ++k) { s[k] = top[k] ^ ((G.v[k] >> 62) & 1); masked[k] = s[k] ^ (p.rb + base)[off + k]; }
        u8* const outb = reinterpret_cast<u8*>(out) + lane * V;
        const u8* const inb = reinterpret_cast<const u8*>(in) + lane * V;
        drained();
#pragma unroll
        for (int k = 0; k < V; ++k) outb[k] = (u8)masked[k];
        opened();
        Pack<V> sa, e, f;
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const u64 v = masked[k] ^ (u64)inb[k];
            // s = v xor rb = v + rb - 2 v rb on additive shares of rb
            sa.v[k] = (v ? (u64)0 - ra.v[k] : ra.v[k]) + (v & m0);
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
#pragma unroll
        for (int k = 0; k < V; ++k) {
            if (base + off + k < first) continue;
            (p.y + base)[off + k] = y.v[k];
            if (p.s_bit) (p.s_bit + base)[off + k] = (u8)s[k];
            if (p.s_arith) (p.s_arith + base)[off + k] = sa.v[k];
        }
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
