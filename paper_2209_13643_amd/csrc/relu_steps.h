// Per-element steps of the secure ReLU that the stage kernels (one launch per protocol round) and the fused
// kernels (all rounds in one launch) share: vector access, the Beaver AND, and the adder topologies.
#pragma once
#include "common.h"

struct alignas(16) u64x2 { u64 a, b; };

template <int V> struct Pack;
template <> struct Pack<1> {
    u64 v[1];
    __device__ static Pack ld(const u64* p, size_t i) { Pack r; r.v[0] = p[i]; return r; }
    __device__ void st(u64* p, size_t i) const { p[i] = v[0]; }
};
template <> struct Pack<2> {
    u64 v[2];
    __device__ static Pack ld(const u64* p, size_t i)
    {
        const u64x2 t = *reinterpret_cast<const u64x2*>(p + i);
        Pack r; r.v[0] = t.a; r.v[1] = t.b; return r;
    }
    __device__ void st(u64* p, size_t i) const
    {
        u64x2 t; t.a = v[0]; t.b = v[1];
        *reinterpret_cast<u64x2*>(p + i) = t;
    }
};

template <> struct Pack<4> {
    u64 v[4];
    __device__ static Pack ld(const u64* p, size_t i)
    {
        const u64x2 t = *reinterpret_cast<const u64x2*>(p + i), u = *reinterpret_cast<const u64x2*>(p + i + 2);
        Pack r; r.v[0] = t.a; r.v[1] = t.b; r.v[2] = u.a; r.v[3] = u.b; return r;
    }
    __device__ void st(u64* p, size_t i) const
    {
        u64x2 t, u; t.a = v[0]; t.b = v[1]; u.a = v[2]; u.b = v[3];
        *reinterpret_cast<u64x2*>(p + i) = t; *reinterpret_cast<u64x2*>(p + i + 2) = u;
    }
};

// V consecutive bytes (one per element): a single 16- or 32-bit access when V is 2 or 4
template <int V> __device__ __forceinline__ void ld_bytes(const u8* p, size_t i, u8 (&out)[V])
{
    if constexpr (V == 4) { const uint32_t w = *reinterpret_cast<const uint32_t*>(p + i);
                            out[0] = (u8)w; out[1] = (u8)(w >> 8); out[2] = (u8)(w >> 16); out[3] = (u8)(w >> 24); }
    else if constexpr (V == 2) { const uint16_t w = *reinterpret_cast<const uint16_t*>(p + i);
                                 out[0] = (u8)w; out[1] = (u8)(w >> 8); }
    else out[0] = p[i];
}
template <int V> __device__ __forceinline__ void st_bytes(u8* p, size_t i, const u8 (&in)[V])
{
    if constexpr (V == 4) *reinterpret_cast<uint32_t*>(p + i) = (uint32_t)in[0] | ((uint32_t)in[1] << 8) | ((uint32_t)in[2] << 16) | ((uint32_t)in[3] << 24);
    else if constexpr (V == 2) *reinterpret_cast<uint16_t*>(p + i) = (uint16_t)((uint16_t)in[0] | ((uint16_t)in[1] << 8));
    else p[i] = in[0];
}

// Beaver AND, one party's side (Eq. 4; Alg. 4 for the party that adds d & g):
// d, g are the opened masked operands, (a, b, c) this party's triple words.
template <int PARTY>
__device__ __forceinline__ u64 and_finish(u64 d, u64 g, u64 a, u64 b, u64 c)
{
    u64 t = c ^ (d & b) ^ (g & a);
    if (PARTY == 0) t ^= d & g;
    return t;
}

// ---- adder topologies -----------------------------------------------------------
// TOPO 0: Kogge-Stone, level l combines every position p with p - 2^l.
// TOPO 1: the prefix tree of the listing in Sec. 4.2, level l joins blocks of
// 2^l bits: the upper half of each 2^(l+1)-bit block (om) combines with the top
// bit of its lower half (im), copied over the upper half by a multiply (mu).
constexpr u64 tree_im(int l) { u64 m = 0; for (int b = 0; b < 64; b += 2 << l) m |= (u64)1 << (b + (1 << l) - 1); return m; }
constexpr u64 tree_om(int l)
{
    const int half = 1 << l; u64 m = 0;
    for (int b = 0; b < 64; b += 2 * half) m |= (half == 64 ? ~(u64)0 : (((u64)1 << half) - 1)) << (b + half);
    return m;
}
constexpr u64 tree_mu(int l) { u64 m = 0; for (int k = 1; k <= (1 << l); ++k) m |= (u64)1 << k; return m; }
// left operand of a level's ANDs, from P
template <int TOPO, int L> __device__ __forceinline__ u64 op_x(u64 P) { if constexpr (TOPO) return P & tree_om(L); else return P; }
// right operand, from G (first AND) or P (second AND)
template <int TOPO, int L> __device__ __forceinline__ u64 op_y(u64 w)
{
    if constexpr (TOPO) return (w & tree_im(L)) * tree_mu(L); else return w << (1 << L);
}
// the part of P a level leaves untouched
template <int TOPO, int L> __device__ __forceinline__ u64 keep_p(u64 P) { if constexpr (TOPO) return P & ~tree_om(L); else return 0; }
