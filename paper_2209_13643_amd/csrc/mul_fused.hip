// Element-wise Alg. 1 and what is built on it (ReLU backward, max-pool backward) in one launch, exchange by remote
// store: a workgroup is one wave per party (wire.h), the masked words go through receive buffers that stay in the L2,
// and every operand is read once and every result written once.  Bound by HBM.
#include "common.h"
#include "mul_fused.h"
#include "wire.h"

namespace {

constexpr int kRows = 2;                  // masked words of the two operands
constexpr unsigned kBlocks = 2048;        // receive buffers of two parties: 8 MB
constexpr int kPairs[2] = { 2, 6 };       // ordered pairs of parties

// One element-wise product on a wave's elements: z = c + e b + a f (+ e f), e = open(x - a), f = open(y - b).
template <int NP, int V>
__device__ __forceinline__ Pack<V> product(const Wire<NP>& wire, u64 m0, unsigned slot, const Pack<V>& x, const Pack<V>& y,
                                           const Pack<V>& a, const Pack<V>& b, const Pack<V>& c)
{
    constexpr unsigned row = kWave * V * 8u;
    Pack<V> e, f, z;
#pragma unroll
    for (int k = 0; k < V; ++k) { e.v[k] = x.v[k] - a.v[k]; f.v[k] = y.v[k] - b.v[k]; }
    wire.drained();
    wire.put(slot, e); wire.put(slot, f, row);
    wire.opened();
    const auto ge = wire.template received<V>(slot), gf = wire.template received<V>(slot, row);
    const Pack<V> re = ge.summed(), rf = gf.summed();
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const u64 eo = e.v[k] + re.v[k], fo = f.v[k] + rf.v[k];
        z.v[k] = c.v[k] + eo * (b.v[k] + (fo & m0)) + a.v[k] * fo;
    }
    return z;
}

// a party's shares of 1 - s
template <int V> __device__ __forceinline__ Pack<V> one_minus(const Pack<V>& s, u64 m0)
{
    Pack<V> r;
#pragma unroll
    for (int k = 0; k < V; ++k) r.v[k] = (m0 & 1) - s.v[k];
    return r;
}

// 2 097 152 elements, two parties: mask, copy and finish kernels 0.097 ms, this one 0.037 ms (5.4 TB/s).
template <int NP, int V>
__global__ __launch_bounds__(NP * kWave, 8) void k_mul_fused(FusedMul q)
{
    const int party = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int lane = threadIdx.x % kWave;
    const u64 m0 = party == 0 ? ~(u64)0 : 0;
    const Wire<NP> wire(q.box, party, (size_t)kRows * kWave * V);
    const size_t n = q.n;
    for (size_t tile = blockIdx.x; tile < q.tiles; tile += gridDim.x) {
        // a ragged last tile takes the last 64 V elements and stores its own only
        const size_t first = tile * (kWave * V);
        const size_t base = first + kWave * V <= n ? first : n >= kWave * V ? n - kWave * V : 0;
        const unsigned rest = n < kWave * V ? (unsigned)n - V : kWave * V - V;
        const unsigned off = lane * V < rest ? lane * V : rest;
        auto row = [&](const u64* t) { return ld_once<V>(t + base, off * 8u); };
        const Pack<V> x = row(q.x[party]), a = row(q.a[party]), b = row(q.b[party]), c = row(q.c[party]);
        Pack<V> y = row(q.y[party]);
        if (q.mask_from_sign) y = one_minus(y, m0);
        Pack<V> z = product<NP, V>(wire, m0, lane * V * 8u, x, y, a, b, c);
        if (NP == 2 && q.trunc_bits) {
#pragma unroll
            for (int k = 0; k < V; ++k) z.v[k] = party == 0 ? z.v[k] >> q.trunc_bits : (u64)0 - (((u64)0 - z.v[k]) >> q.trunc_bits);
        }
        if (base + off >= first) st_words<V>(q.z[party] + base, off * 8u, z);
        else if (V == 2 && base + off + 1 == first) (q.z[party] + base)[off + 1] = z.v[V - 1];
    }
}

// Max-pool backward on 64 outputs per wave: grad_u = g (1 - s2), grad_v = g - grad_u; P = (grad_u, grad_v) (1 - s1); the
// window receives P[0], grad_u - P[0], P[1], grad_v - P[1].  524 288 outputs: eight launches 0.10 ms, this one 0.030 ms.
template <int NP>
__global__ __launch_bounds__(NP * kWave, 6) void k_poolbwd_fused(FusedPoolBwd q)
{
    const int party = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const unsigned lane = threadIdx.x % kWave;
    const u64 m0 = party == 0 ? ~(u64)0 : 0;
    const Wire<NP> wire(q.box, party, (size_t)kRows * kWave * 2);
    const unsigned C = (unsigned)q.C, Wo = (unsigned)q.W / 2, Ho = (unsigned)q.H / 2;
    for (unsigned tile = blockIdx.x; tile < q.tiles; tile += gridDim.x) {
        const size_t o0 = (size_t)tile * kWave;
        const unsigned last = q.n_out - o0 < kWave ? (unsigned)(q.n_out - o0) - 1 : kWave - 1;
        const unsigned at = lane < last ? lane : last;              // past the end: the last output again, not stored
        auto row1 = [&](const u64* m) { return ld_once<2>(m + 2 * o0, at * 16u); };
        auto row2 = [&](const u64* m) { return ld_once<1>(m + o0, at * 8u); };
        const Pack<1> g = row2(q.g[party]);
        const Pack<1> gu = product<NP, 1>(wire, m0, lane * 8u, g, one_minus(row2(q.s2[party]), m0),
                                          row2(q.a2[party]), row2(q.b2[party]), row2(q.c2[party]));
        Pack<2> pair;
        pair.v[0] = gu.v[0]; pair.v[1] = g.v[0] - gu.v[0];
        const Pack<2> P = product<NP, 2>(wire, m0, lane * 16u, pair, one_minus(row1(q.s1[party]), m0),
                                         row1(q.a1[party]), row1(q.b1[party]), row1(q.c1[party]));
        if (at != lane) continue;
        size_t t = o0 + at;
        const unsigned ch = (unsigned)(t % C); t /= C;
        const unsigned wo = (unsigned)(t % Wo); t /= Wo;
        const unsigned ho = (unsigned)(t % Ho); const size_t b = t / Ho;
        u64* const w = q.gx[party] + ((b * q.H + 2 * ho) * q.W + 2 * wo) * C + ch;
        const size_t dh = (size_t)q.W * C;
        w[0] = P.v[0];  w[C] = pair.v[0] - P.v[0];
        w[dh] = P.v[1]; w[dh + C] = pair.v[1] - P.v[1];
    }
}

// The masked rescale of three parties: parties 1 and 2 store z_i + r_i into party 0's two receive buffers.  Twelve traversals of
// the words instead of the 21 of mask, copy and finish kernels: 2 097 152 elements 65 us as
// three launches, 34 here (5.9 TB/s).
template <int V>
__global__ __launch_bounds__(3 * kWave, 6) void k_trunc3_fused(FusedTrunc3 q)
{
    const int party = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const unsigned lane = threadIdx.x % kWave, slot = lane * V * 8u;
    const size_t n = q.n, row_bytes = kWave * V * 8;
    u8* const wg = reinterpret_cast<u8*>(q.box) + (size_t)blockIdx.x * 2 * row_bytes;
    for (size_t tile = blockIdx.x; tile < q.tiles; tile += gridDim.x) {
        // a ragged last tile takes the last 64 V elements and stores its own only
        const size_t first = tile * (kWave * V);
        const size_t base = first + kWave * V <= n ? first : n >= kWave * V ? n - kWave * V : 0;
        const unsigned rest = n < kWave * V ? (unsigned)n - V : kWave * V - V;
        const unsigned off = lane * V < rest ? lane * V : rest;
        auto row = [&](const u64* t) { return ld_once<V>(t + base, off * 8u); };
        Pack<V> z = row(q.z[party]), rt = row(q.rt[party]);
        const Pack<V> r = row(q.r[party]);
#pragma unroll
        for (int k = 0; k < V; ++k) z.v[k] += r.v[k];
        __syncthreads();                     // party 0 holds the words of the last tile
        if (party) z.st(reinterpret_cast<u64*>(wg + (party - 1) * row_bytes + slot), 0);
        __syncthreads();
        if (party == 0) {
            const Pack<V> a = Pack<V>::ld(reinterpret_cast<const u64*>(wg + slot), 0), b = Pack<V>::ld(reinterpret_cast<const u64*>(wg + row_bytes + slot), 0);
#pragma unroll
            for (int k = 0; k < V; ++k)
                z.v[k] = ((z.v[k] + a.v[k] + b.v[k] + ((u64)1 << 62)) >> q.bits) - ((u64)1 << (62 - q.bits)) - rt.v[k];
        } else {
#pragma unroll
            for (int k = 0; k < V; ++k) z.v[k] = (u64)0 - rt.v[k];
        }
        if (base + off >= first) st_words<V>(q.z[party] + base, off * 8u, z);
        else if (V == 2 && base + off + 1 == first) (q.z[party] + base)[off + 1] = z.v[V - 1];
    }
}

// two elements per thread once one per thread would need a second round of workgroups
int width(size_t n) { return n > (size_t)kBlocks * kWave ? 2 : 1; }
unsigned tiles_of(size_t n, int v) { return (unsigned)((n + kWave * v - 1) / (kWave * v)); }
unsigned blocks_for(unsigned tiles) { return tiles < kBlocks ? tiles : kBlocks; }

}  // namespace

size_t mul_fused_box_bytes(int parties, size_t n)
{
    const int v = width(n);
    return (size_t)blocks_for(tiles_of(n, v)) * kPairs[parties - 2] * (kRows * kWave * v) * sizeof(u64);
}

int launch_mul_fused(mpc_ctx* c, hipStream_t st, int parties, FusedMul q)
{
    if (q.n == 0 || q.n >= ((size_t)1 << 37)) return MPC_EINVAL;
    const int v = width(q.n);
    q.tiles = tiles_of(q.n, v);
    const dim3 grid(blocks_for(q.tiles)), block(parties * kWave);
    if (parties == 2) {
        if (v == 2) hipLaunchKernelGGL((k_mul_fused<2, 2>), grid, block, 0, st, q);
        else        hipLaunchKernelGGL((k_mul_fused<2, 1>), grid, block, 0, st, q);
    } else {
        if (v == 2) hipLaunchKernelGGL((k_mul_fused<3, 2>), grid, block, 0, st, q);
        else        hipLaunchKernelGGL((k_mul_fused<3, 1>), grid, block, 0, st, q);
    }
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

size_t poolbwd_fused_box_bytes(int parties, size_t n_out)
{
    return (size_t)blocks_for(tiles_of(n_out, 1)) * kPairs[parties - 2] * (kRows * kWave * 2) * sizeof(u64);
}

int launch_poolbwd_fused(mpc_ctx* c, hipStream_t st, int parties, FusedPoolBwd q)
{
    if (q.n_out == 0 || q.n_out >= ((size_t)1 << 36)) return MPC_EINVAL;
    q.tiles = tiles_of(q.n_out, 1);
    const dim3 grid(blocks_for(q.tiles)), block(parties * kWave);
    if (parties == 2) hipLaunchKernelGGL(k_poolbwd_fused<2>, grid, block, 0, st, q);
    else              hipLaunchKernelGGL(k_poolbwd_fused<3>, grid, block, 0, st, q);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

size_t trunc3_fused_box_bytes(size_t n)
{
    const int v = width(n);
    return (size_t)blocks_for(tiles_of(n, v)) * 2 * (kWave * v) * sizeof(u64);
}

int launch_trunc3_fused(mpc_ctx* c, hipStream_t st, FusedTrunc3 q)
{
    if (q.n == 0 || q.n >= ((size_t)1 << 37)) return MPC_EINVAL;
    const int v = width(q.n);
    q.tiles = tiles_of(q.n, v);
    const dim3 grid(blocks_for(q.tiles)), block(3 * kWave);
    if (v == 2) hipLaunchKernelGGL(k_trunc3_fused<2>, grid, block, 0, st, q);
    else        hipLaunchKernelGGL(k_trunc3_fused<1>, grid, block, 0, st, q);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}
