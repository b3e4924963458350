// Exchange of masked words inside a launch (by remote store): a workgroup is one wave per party, all of them on the same
// elements, and a round is "every wave stores its words into the peers' receive buffers, workgroup barrier, every wave
// reads its own receive buffers".  Shared by the kernels that run several protocol rounds in one launch.
#pragma once
#include "common.h"
#include "relu_steps.h"

constexpr int kWave = 64;

typedef u64 u64v2u __attribute__((ext_vector_type(2), aligned(8)));

// V consecutive words at scalar base + 32-bit byte offset, any 8-byte aligned address, read once.  Four words per lane are two
// accesses to the same lines, of which the second should find them: not non-temporal (sign-only ReLU of 2 097 152 elements
// 141 -> 135 us).
template <int V> __device__ __forceinline__ Pack<V> ld_once(const u64* p, unsigned off)
{
    const u8* a = reinterpret_cast<const u8*>(p) + off;
    Pack<V> r;
    if constexpr (V >= 2) {
#pragma unroll
        for (int k = 0; k < V; k += 2) {
            const u64v2u* const at = reinterpret_cast<const u64v2u*>(a + 8 * k);
            const u64v2u t = V > 2 ? *at : __builtin_nontemporal_load(at);
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

// What a wave received from its peers, loaded but not yet combined (XOR shares / additive shares): a round's words are
// asked for together before the first of them is used.
template <int NP, int W> struct Received {
    Pack<W> q[NP - 1];
    __device__ __forceinline__ Pack<W> xored() const
    {
        Pack<W> r = q[0];
        if constexpr (NP == 3) {
#pragma unroll
            for (int k = 0; k < W; ++k) r.v[k] ^= q[1].v[k];
        }
        return r;
    }
    __device__ __forceinline__ Pack<W> summed() const
    {
        Pack<W> r = q[0];
        if constexpr (NP == 3) {
#pragma unroll
            for (int k = 0; k < W; ++k) r.v[k] += q[1].v[k];
        }
        return r;
    }
};

// The receive buffers of a workgroup, one per ordered pair of parties: party i's buffer s holds what party
// (i + 1 + s) mod NP sent last.  `box_words` words each.
// COPY (two parties): a party stores its words into a send buffer of its own, and after the barrier the peer's wave moves
// them into its receive buffer, using each word as it passes; two buffers per party.  The receive buffer is not read back:
// its stores are the exchange that the protocol asks for, one more word through the L2 per word sent.
template <int NP, bool COPY = false>
struct Wire {
    static_assert(!COPY || NP == 2, "the copying exchange is written for two parties");
    u8* in; u8* out[NP - 1]; size_t step;
    u8* peer;                                 // COPY: the peer's send buffer
    __device__ __forceinline__ Wire(u64* box, int party, size_t box_words)
    {
        step = box_words * 8;
        u8* const wg = reinterpret_cast<u8*>(box) + (size_t)blockIdx.x * (NP * (NP - 1) * (COPY ? 2 : 1)) * step;
        in = wg + (size_t)party * (NP - 1) * step;
        if constexpr (COPY) { out[0] = wg + (size_t)(2 + party) * step; peer = wg + (size_t)(3 - party) * step; return; }
#pragma unroll
        for (int s = 0; s < NP - 1; ++s) {
            int to = party + NP - 1 - s; if (to >= NP) to -= NP;             // the party whose buffer s is filled from here
            out[s] = wg + ((size_t)to * (NP - 1) + s) * step;
        }
    }
    // off: the lane's place; row: a uniform distance, kept apart so that it goes to the scalar base
    template <int W> __device__ __forceinline__ void put_to(int s, unsigned off, const Pack<W>& w, unsigned row = 0) const { w.st(reinterpret_cast<u64*>(out[s] + row + off), 0); }
    template <int W> __device__ __forceinline__ void put(unsigned off, const Pack<W>& w, unsigned row = 0) const
    {
#pragma unroll
        for (int s = 0; s < NP - 1; ++s) put_to(s, off, w, row);
    }
    template <int W> __device__ __forceinline__ Pack<W> from(int s, unsigned off, unsigned row = 0) const
    {
        if constexpr (COPY) {
            const Pack<W> w = Pack<W>::ld(reinterpret_cast<const u64*>(peer + row + off), 0);
            w.st(reinterpret_cast<u64*>(in + row + off), 0);
            return w;
        } else return Pack<W>::ld(reinterpret_cast<const u64*>(in + s * step + row + off), 0);
    }
    template <int W> __device__ __forceinline__ Received<NP, W> received(unsigned off, unsigned row = 0) const
    {
        Received<NP, W> r;
#pragma unroll
        for (int i = 0; i < NP - 1; ++i) r.q[i] = from<W>(i, off, row);
        return r;
    }
    template <int V> __device__ __forceinline__ void put_flags(unsigned off, unsigned w) const
    {
#pragma unroll
        for (int s = 0; s < NP - 1; ++s) st_flags<V>(out[s] + off, w);
    }
    template <int V> __device__ __forceinline__ unsigned flags(unsigned off) const
    {
        unsigned w = ld_flags<V>((COPY ? peer : in) + off);
        if constexpr (COPY) st_flags<V>(in + off, w);
        if constexpr (NP == 3) w ^= ld_flags<V>(in + step + off);
        return w;
    }
    __device__ __forceinline__ static void opened() { __syncthreads(); }      // every wave has stored its words of the round
    __device__ __forceinline__ static void drained() { __syncthreads(); }     // every wave holds the words of the last round: the buffers are free
};

// One party's side of a Beaver AND; m0: all ones for the party that adds the product of the opened words.
__device__ __forceinline__ u64 fin(u64 d, u64 g, u64 a, u64 b, u64 c, u64 m0) { return c ^ (d & b) ^ (g & a) ^ (d & g & m0); }
