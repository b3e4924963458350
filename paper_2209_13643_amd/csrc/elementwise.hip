// Streaming element-wise kernels: masking, opening, truncation, wire copy,
// and the recoding of ring words into balanced base-256 digit planes.
// All of them are HBM-bound; they use 16-byte accesses and grid-stride loops.
#include "common.h"
#include "digits.h"
#include "recode_tiles.h"

#include <algorithm>
#include <type_traits>

namespace {

constexpr int kThreads = 256;

inline int grid_for(size_t items, int per_thread = 1)
{
    size_t blocks = (items + (size_t)kThreads * per_thread - 1) / ((size_t)kThreads * per_thread);
    const size_t cap = 256 * 16;          // 16 workgroups per CU keep HBM busy
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    return (int)blocks;
}

struct alignas(16) u64x2 { u64 a, b; };

template <int OP>  // 0: x - y, 1: x + y
__global__ __launch_bounds__(kThreads) void k_binary(const u64* __restrict__ x, const u64* __restrict__ y,
                                                     u64* __restrict__ out, size_t n)
{
    const size_t n2 = n / 2;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const u64x2* x2 = reinterpret_cast<const u64x2*>(x);
    const u64x2* y2 = reinterpret_cast<const u64x2*>(y);
    u64x2* o2 = reinterpret_cast<u64x2*>(out);
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n2; i += stride) {
        u64x2 p = x2[i], q = y2[i], r;
        if (OP == 0) { r.a = p.a - q.a; r.b = p.b - q.b; }
        else         { r.a = p.a + q.a; r.b = p.b + q.b; }
        o2[i] = r;
    }
    if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
        const size_t i = n - 1;
        out[i] = OP == 0 ? x[i] - y[i] : x[i] + y[i];
    }
}

// scalar fallback when a pointer is only 8-byte aligned
template <int OP>
__global__ __launch_bounds__(kThreads) void k_binary_scalar(const u64* __restrict__ x, const u64* __restrict__ y,
                                                            u64* __restrict__ out, size_t n)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        out[i] = OP == 0 ? x[i] - y[i] : x[i] + y[i];
}

__global__ __launch_bounds__(kThreads) void k_copy16(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n16)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
}

__global__ __launch_bounds__(kThreads) void k_copy1(const u8* __restrict__ src, u8* __restrict__ dst, size_t n)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

// Local two-party truncation: party 0 shifts, party 1 negates, shifts, negates.
__global__ __launch_bounds__(kThreads) void k_truncate(u64* __restrict__ z, size_t n, int bits, int party)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const u64 v = z[i];
        z[i] = party == 0 ? (v >> bits) : (u64)0 - (((u64)0 - v) >> bits);
    }
}

// 16 consecutive k of one row to the eight planes of one k block
__device__ __forceinline__ void store_unit(const u64 (&v)[16], u8* out, long long digit_stride)
{
    uint32_t w[8][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const u64 four[4] = { v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3] };
        uint32_t d[8];
        digits_of_4(four, d);
#pragma unroll
        for (int k = 0; k < 8; ++k) w[k][q] = d[k];
    }
#pragma unroll
    for (int d = 0; d < 8; ++d) *reinterpret_cast<uint4*>(out + (size_t)d * digit_stride) = make_uint4(w[d][0], w[d][1], w[d][2], w[d][3]);
}

// One thread recodes one (row, k-block): 16 ring words in, one 16-byte unit
// out per digit plane.  Consecutive lanes take consecutive rows so that the
// plane stores are contiguous.  The 16 words of every operand are loaded at clamped indices with no branch between
// them and masked afterwards: with a range check around each word the loads ran one after the other (a recoding of
// any size took at least 12 us, now 5).
__device__ __forceinline__ void recode_body(const RecodeArgs& a, int tap /* == ntaps: zero padding block(s) */, int b,
                                            unsigned bx, unsigned nbx)
{
    // tap_stride may be negative (filters read in reverse tap order)
    const bool padtap = tap >= a.ntaps;
    const long long at = (long long)b * a.src_batch_stride + (padtap ? 0 : (long long)tap * a.tap_stride);
    const u64* src = a.src + at;
    const u64* src2 = a.src2 ? a.src2 + at : nullptr;
    const u64* src3 = a.src3 ? a.src3 + at : nullptr;
    u8* dst = a.dst + (size_t)b * a.dst_batch_stride;
    const int kb_count = padtap ? a.KB_total - a.ntaps * a.KB_tap : a.KB_tap;
    const size_t items = (size_t)kb_count * a.plane_rows;
    const size_t stride = (size_t)nbx * blockDim.x;
    for (size_t it = (size_t)bx * blockDim.x + threadIdx.x; it < items; it += stride) {
        const int kbl = (int)(it / a.plane_rows);
        const int row = (int)(it - (size_t)kbl * a.plane_rows);
        const int kb_out = (padtap ? a.ntaps * a.KB_tap : tap * a.KB_tap) + kbl;
        const int k0 = kbl * 16;
        // valid words of the unit: k0 .. k0 + have - 1
        const int have = (padtap || row >= a.rows) ? 0 : a.K - k0 < 16 ? (a.K - k0 > 0 ? a.K - k0 : 0) : 16;
        const long long base = (long long)(row < a.rows ? row : 0) * a.row_stride + (long long)(k0 < a.K ? k0 : 0) * a.k_stride;
        auto load = [&](const u64* q, u64 (&w)[16]) {
#pragma unroll
            for (int t = 0; t < 16; ++t) w[t] = q[base + (long long)(t < have ? t : 0) * a.k_stride];
        };
        u64 v[16], w[16];
        load(src, v);
        if (src2) {
            load(src2, w);
#pragma unroll
            for (int t = 0; t < 16; ++t) v[t] += w[t];
        }
        if (src3) {
            load(src3, w);
#pragma unroll
            for (int t = 0; t < 16; ++t) v[t] += w[t];
        }
#pragma unroll
        for (int t = 0; t < 16; ++t) v[t] = t < have ? v[t] : 0;
        store_unit(v, dst + ((size_t)kb_out * a.plane_rows + row) * 16, a.digit_stride);
    }
}

__global__ __launch_bounds__(kThreads) void k_recode(RecodeArgs a)
{
    recode_body(a, blockIdx.y, blockIdx.z, blockIdx.x, gridDim.x);
}

// Recoding of a matrix whose k index is contiguous in memory (left operands,
// NHWC activations, filters read with their channel roles swapped): a workgroup takes a 64-row x 64-k tile of one
// filter tap, reads it with lanes along k (coalesced 16-byte loads), scatters the digits into LDS in
// plane order, and writes each plane's 16-byte units with lanes along rows
// (coalesced again).  bx = row tile, by = (tap, group of 4 k blocks).
__device__ __forceinline__ void recode_rows_body(const RecodeArgs& a, int b, unsigned bx, unsigned by, uint32_t (*tile)[4][64][4])
{
    const RecodeTile rt = recode_tile(a.ntaps, a.KB_tap, a.KB_total, by);
    const int row0 = bx * 64, tap = rt.tap, kb0 = rt.kb0, kb_lim = rt.kb_lim, kb_first = tap * a.KB_tap;
    const bool padtap = rt.zero;                                 // the k blocks behind the last tap: zero
    if (row0 >= a.plane_rows || kb0 >= kb_lim) return;           // uniform per workgroup
    const long long at = (long long)b * a.src_batch_stride + (padtap ? 0 : (long long)tap * a.tap_stride);
    const u64* src = a.src + at;
    const u64* src2 = a.src2 ? a.src2 + at : nullptr;
    const u64* src3 = a.src3 ? a.src3 + at : nullptr;
    u8* dst = a.dst + (size_t)b * a.dst_batch_stride;
    const int k_lim = padtap ? 0 : a.K;
    const bool vec = (a.row_stride % 2 == 0) && (((uintptr_t)src | (uintptr_t)src2 | (uintptr_t)src3) & 15) == 0;
    // thread's segments: 4 words each, segment p at row (threadIdx.x + 256 p) / 16 of the tile
    const int s4 = threadIdx.x & 15, k = kb0 * 16 + s4 * 4;
    // 16-byte accesses allowed; threads past the last k read column 0 with the others instead of a way of their own
    const bool beyond = k >= k_lim, whole = vec && (beyond ? k_lim > 3 : k + 3 < k_lim);
    const int kc = beyond ? 0 : k;
    // The loads of two segments in one straight line per way of access and kind of sum.  With the way chosen anew for
    // every operand the ways joined in between, and the next operand's loads waited for the joined registers; with the
    // threads past the last k on the word-wise way, every wave of a tile that K leaves ragged ran both: 300 x 4000 words
    // 8.3 -> 7.1 us.
#pragma unroll
    for (int p0 = 0; p0 < 4; p0 += 2) {
        auto row_of = [&](int p) { return row0 + (int)(threadIdx.x >> 4) + 16 * (p0 + p); };
        u64 v[2][4];
        auto gather = [&](auto whole_tag, auto sum_tag) {
            constexpr bool W = decltype(whole_tag)::value, sum = decltype(sum_tag)::value;       // sum: src and src2 alone
            auto load = [&](const u64* q, u64 (&w)[2][4]) {
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const int r = row_of(p);
                    const u64* t = q + (size_t)(r < a.rows ? r : 0) * a.row_stride;
                    if constexpr (W) {
                        const u64x2 lo = reinterpret_cast<const u64x2*>(t + kc)[0], hi = reinterpret_cast<const u64x2*>(t + kc)[1];
                        w[p][0] = lo.a; w[p][1] = lo.b; w[p][2] = hi.a; w[p][3] = hi.b;
                    } else {
#pragma unroll
                        for (int u = 0; u < 4; ++u) w[p][u] = t[k + u < k_lim ? k + u : 0];
                    }
                }
            };
            auto add = [&](const u64* q) {
                u64 w[2][4];
                load(q, w);
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[p][u] += w[p][u];
            };
            load(src, v);
            if constexpr (sum) add(src2);
            else {
                if (src2) add(src2);
                if (src3) add(src3);
            }
        };
        if (!whole)             gather(std::false_type{}, std::false_type{});
        else if (src2 && !src3) gather(std::true_type{}, std::true_type{});
        else                    gather(std::true_type{}, std::false_type{});
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const bool row_ok = row_of(p) < a.rows;
            u64 four[4]; uint32_t d[8];
#pragma unroll
            for (int u = 0; u < 4; ++u) four[u] = row_ok && k + u < k_lim ? v[p][u] : 0;
            digits_of_4(four, d);
#pragma unroll
            for (int q = 0; q < 8; ++q) tile[q][s4 >> 2][(threadIdx.x >> 4) + 16 * (p0 + p)][s4 & 3] = d[q];
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int u = threadIdx.x + 256 * q;
        const int d = u >> 8, kbl = (u >> 6) & 3, row = u & 63;
        if (row0 + row < a.plane_rows && kb0 + kbl < kb_lim) {
            const uint4 val = *reinterpret_cast<const uint4*>(&tile[d][kbl][row][0]);
            *reinterpret_cast<uint4*>(dst + (size_t)d * a.digit_stride + ((size_t)(kb_first + kb0 + kbl) * a.plane_rows + row0 + row) * 16) = val;
        }
    }
}

__global__ __launch_bounds__(kThreads) void k_recode_rows(RecodeBatch rb)
{
    __shared__ uint32_t tile[8][4][64][4];
    const int set = blockIdx.z / rb.batch, b = blockIdx.z - set * rb.batch;
    recode_rows_body(rb.a[set], b, blockIdx.x, blockIdx.y, tile);
}

// Sets of both kinds in one launch over a flat list of workgroups: set q owns the
// ids [first[q], first[q+1]), decoded as (x, y, batch item) with its own extents gx, gy.
// Contiguous-k sets (rows_kind) use the tile recoder above with (x, y) = (row tile, group
// of 4 k blocks); generic sets use one thread per (row, k block) with y = tap.
struct RecodeMixed { RecodeBatch rb; unsigned first[kMaxRecodeSets + 1]; unsigned gx[kMaxRecodeSets], gy[kMaxRecodeSets];
                     bool rows_kind[kMaxRecodeSets]; int count; };
__global__ __launch_bounds__(kThreads) void k_recode_mixed(RecodeMixed m)
{
    __shared__ uint32_t tile[8][4][64][4];
    int q = 0;
    while (q + 1 < m.count && blockIdx.x >= m.first[q + 1]) ++q;       // uniform per workgroup
    const RecodeArgs& a = m.rb.a[q];
    unsigned id = blockIdx.x - m.first[q];
    const unsigned x = id % m.gx[q]; id /= m.gx[q];
    const unsigned y = id % m.gy[q]; const int b = (int)(id / m.gy[q]);
    if (m.rows_kind[q]) recode_rows_body(a, b, x, y, tile);
    else                recode_body(a, (int)y, b, x, m.gx[q]);
}

// Digit planes of the transposed im2col matrix of an NHWC tensor: plane row
// (tap, ci), contraction index = output pixel (b, ho, wo).  One thread fills
// one 16-byte unit per digit: 16 consecutive output pixels of one (tap, ci).
// Lanes run along the rows, i.e. along ci, so loads and stores are contiguous.
__global__ __launch_bounds__(kThreads) void k_recode_im2col_t(Im2colTBatch bt)
{
    const Im2colTArgs& a = bt.a[blockIdx.z];
    const int rows = a.KH * a.KW * a.Cin;
    const long long npix = (long long)a.B * a.Ho * a.Wo;
    const size_t items = (size_t)a.KB_total * rows;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t it = (size_t)blockIdx.x * blockDim.x + threadIdx.x; it < items; it += stride) {
        const int kb = (int)(it / rows);
        const int row = (int)(it - (size_t)kb * rows);
        const int tap = row / a.Cin, ci = row - tap * a.Cin;
        const int dy = tap / a.KW, dx = tap - dy * a.KW;
        // loads at clamped pixels with no branch between them, masked afterwards
        const long long m = (long long)kb * 16;
        int wo = (int)(m % a.Wo); long long t2 = m / a.Wo;
        int ho = (int)(t2 % a.Ho); int b = (int)(t2 / a.Ho);
        size_t idx[16]; unsigned ok = 0;
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const int hi = ho * a.stride + dy - a.pad, wi = wo * a.stride + dx - a.pad;
            const bool in = m + t < npix && hi >= 0 && hi < a.H && wi >= 0 && wi < a.W;
            ok |= (unsigned)in << t;
            idx[t] = in ? (((size_t)b * a.H + hi) * a.W + wi) * a.Cin + ci : 0;
            if (++wo == a.Wo) { wo = 0; if (++ho == a.Ho) { ho = 0; ++b; } }
        }
        u64 v[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) v[t] = a.src[idx[t]];
        if (a.src2) {
            u64 w[16];
#pragma unroll
            for (int t = 0; t < 16; ++t) w[t] = a.src2[idx[t]];
#pragma unroll
            for (int t = 0; t < 16; ++t) v[t] += w[t];
        }
#pragma unroll
        for (int t = 0; t < 16; ++t) v[t] = (ok >> t) & 1 ? v[t] : 0;
        store_unit(v, a.dst + ((size_t)kb * rows + row) * 16, a.digit_stride);
    }
}

// The same planes for a 3x3 filter of stride 1 and padding 1, whose output pixels are the input's: one thread fills the
// three units of a filter row (dx = 0, 1, 2) of one (dy, ci), which read the same 16 pixels moved by one: 18 loads instead
// of 48, at indices Cin words apart (pixel p of the flattened batch reads p + (dy - 1) W + dx - 1; a neighbour inside the
// image row is the neighbour in the run).  Fourteen launches of a VGG16 training step of 32 images
// 418 -> 331 us in all.
__global__ __launch_bounds__(kThreads) void k_recode_im2col3_t(Im2colTBatch bt)
{
    const Im2colTArgs& a = bt.a[blockIdx.z];
    const int rows = 9 * a.Cin, per_kb = 3 * a.Cin;
    const int npix = a.B * a.H * a.W;
    const size_t items = (size_t)a.KB_total * per_kb;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t it = (size_t)blockIdx.x * blockDim.x + threadIdx.x; it < items; it += stride) {
        const int kb = (int)(it / per_kb), q = (int)(it - (size_t)kb * per_kb);
        const int dy = q / a.Cin, ci = q - dy * a.Cin;
        const int m = kb * 16;
        int wo = m % a.W, ho = m / a.W % a.H;
        unsigned ok = 0, left = 0, right = 0;           // bit t: pixel m + t has an input row, and a left / right neighbour in it
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const int hi = ho + dy - 1;
            const bool in = m + t < npix && hi >= 0 && hi < a.H;
            ok |= (unsigned)in << t; left |= (unsigned)(in && wo > 0) << t; right |= (unsigned)(in && wo + 1 < a.W) << t;
            if (++wo == a.W) { wo = 0; if (++ho == a.H) ho = 0; }
        }
        // loads at clamped pixels with no branch between them, masked afterwards
        const int p0 = m + (dy - 1) * a.W - 1;
        size_t idx[18];
#pragma unroll
        for (int t = 0; t < 18; ++t) {
            const int p = p0 + t;
            idx[t] = (size_t)(p < 0 ? 0 : p < npix ? p : npix - 1) * a.Cin + ci;
        }
        u64 v[18];
#pragma unroll
        for (int t = 0; t < 18; ++t) v[t] = a.src[idx[t]];
        if (a.src2) {
            u64 w[18];
#pragma unroll
            for (int t = 0; t < 18; ++t) w[t] = a.src2[idx[t]];
#pragma unroll
            for (int t = 0; t < 18; ++t) v[t] += w[t];
        }
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
            const unsigned there = dx == 0 ? left : dx == 1 ? ok : right;
            u64 unit[16];
#pragma unroll
            for (int t = 0; t < 16; ++t) unit[t] = (there >> t) & 1 ? v[t + dx] : 0;
            store_unit(unit, a.dst + ((size_t)kb * rows + (dy * 3 + dx) * a.Cin + ci) * 16, a.digit_stride);
        }
    }
}

// Element-wise Alg. 1 after the exchange (blockIdx.y = party): e, f from the
// own and the received masked words, z_i = c_i + e*b_i + a_i*f (+ e*f), then the
// optional local truncation.  With `mask_from_sign` the second operand is the
// ReLU input mask 1 - s formed from the additive sign shares in y.
__global__ __launch_bounds__(kThreads) void k_mul_finish(MulArgs q)
{
    const int i = blockIdx.y;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < q.n; k += stride) {
        const u64 e = q.se[i][k] + q.re[i][k], f = q.sf[i][k] + q.rf[i][k];
        u64 z = q.c[i][k] + e * q.b[i][k] + q.a[i][k] * f;
        if (i == 0) z += e * f;
        if (q.trunc_bits) z = i == 0 ? (z >> q.trunc_bits) : (u64)0 - (((u64)0 - z) >> q.trunc_bits);
        q.z[i][k] = z;
    }
}

// masks of the element-wise product (blockIdx.y = party): se = x - a, sf = y - b
__global__ __launch_bounds__(kThreads) void k_mul_mask(MulArgs q)
{
    const int i = blockIdx.y;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < q.n; k += stride) {
        u64 y = q.y[i][k];
        if (q.mask_from_sign) y = (i == 0 ? (u64)1 : (u64)0) - y;
        q.se[i][k] = q.x[i][k] - q.a[i][k];
        q.sf[i][k] = y - q.b[i][k];
    }
}

// Max-pool backward, between its two products (blockIdx.y = party):
// grad_v = g - grad_u, and the pair (grad_u, grad_v) interleaved as the first
// tournament level stored its pairs.
__global__ __launch_bounds__(kThreads) void k_poolbwd_pairs(PoolBwdArgs q)
{
    const int i = blockIdx.y;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t o = (size_t)blockIdx.x * blockDim.x + threadIdx.x; o < q.n_out; o += stride) {
        const u64 gu = q.gu[i][o];
        q.pairs[i][2 * o] = gu;
        q.pairs[i][2 * o + 1] = q.g[i][o] - gu;
    }
}

// ... and after the second product P = pairs * mask1: the four window positions
// receive P[2o], grad_u - P[2o], P[2o+1], grad_v - P[2o+1] (NHWC input layout).
__global__ __launch_bounds__(kThreads) void k_poolbwd_scatter(PoolBwdArgs q)
{
    const int i = blockIdx.y;
    const int Ho = q.H / 2, Wo = q.W / 2;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t o = (size_t)blockIdx.x * blockDim.x + threadIdx.x; o < q.n_out; o += stride) {
        const int ch = (int)(o % q.C); size_t t = o / q.C;
        const int wo = (int)(t % Wo); t /= Wo;
        const int ho = (int)(t % Ho); const int b = (int)(t / Ho);
        const size_t base = (((size_t)b * q.H + 2 * ho) * q.W + 2 * wo) * q.C + ch;
        const size_t dw = q.C, dh = (size_t)q.W * q.C;
        const u64 p0 = q.prod[i][2 * o], p1 = q.prod[i][2 * o + 1];
        const u64 gu = q.pairs[i][2 * o], gv = q.pairs[i][2 * o + 1];
        u64* gx = q.gx[i];
        gx[base] = p0;            gx[base + dw] = gu - p0;
        gx[base + dh] = p1;       gx[base + dh + dw] = gv - p1;
    }
}

// Zero-dilation for the input gradient of a strided convolution (blockIdx.y = tensor):
// every destination word is written, a source word where its pixel is a multiple of the stride.
__global__ __launch_bounds__(kThreads) void k_dilate(DilateArgs q)
{
    const u64* src = q.src[blockIdx.y]; u64* dst = q.dst[blockIdx.y];
    if (!src) return;
    const size_t total = (size_t)q.B * q.Hd * q.Wd * q.C;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t o = (size_t)blockIdx.x * blockDim.x + threadIdx.x; o < total; o += stride) {
        const int ch = (int)(o % q.C); size_t t = o / q.C;
        const int wd = (int)(t % q.Wd); t /= q.Wd;
        const int hd = (int)(t % q.Hd); const int b = (int)(t / q.Hd);
        u64 v = 0;
        if (hd % q.stride == 0 && wd % q.stride == 0) {
            const int ho = hd / q.stride, wo = wd / q.stride;
            if (ho < q.Ho && wo < q.Wo) v = src[(((size_t)b * q.Ho + ho) * q.Wo + wo) * q.C + ch];
        }
        dst[o] = v;
    }
}

// Several recodings in one launch: blockIdx.z = set * batch + batch item.
__global__ __launch_bounds__(kThreads) void k_recode_multi(RecodeBatch rb)
{
    const int set = blockIdx.z / rb.batch, b = blockIdx.z - set * rb.batch;
    const RecodeArgs& a = rb.a[set];
    const int taps = a.ntaps + (a.KB_total > a.ntaps * a.KB_tap ? 1 : 0);
    if ((int)blockIdx.y < taps) recode_body(a, blockIdx.y, b, blockIdx.x, gridDim.x);
}

// Several element-wise subtractions / copies in one launch: blockIdx.y = segment.
// PUT: every difference is also stored into out2, the peer's receive buffer
// (exchange by remote store: the mask kernel is the sender).
template <bool PUT>
__global__ __launch_bounds__(kThreads) void k_sub_multi(SubBatch sb)
{
    const SubSeg& q = sb.s[blockIdx.y];
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    if (q.vec) {
        const size_t n2 = q.n / 2;
        const u64x2* x2 = reinterpret_cast<const u64x2*>(q.x);
        const u64x2* y2 = reinterpret_cast<const u64x2*>(q.a);
        u64x2* o2 = reinterpret_cast<u64x2*>(q.out);
        u64x2* p2 = reinterpret_cast<u64x2*>(q.out2);
        for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n2; i += stride) {
            u64x2 p = x2[i], r = y2[i];
            p.a -= r.a; p.b -= r.b;
            o2[i] = p;
            if constexpr (PUT) p2[i] = p;
        }
        if ((q.n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
            q.out[q.n - 1] = q.x[q.n - 1] - q.a[q.n - 1];
            if constexpr (PUT) q.out2[q.n - 1] = q.out[q.n - 1];
        }
    } else {
        for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < q.n; i += stride) {
            const u64 v = q.x[i] - q.a[i];
            q.out[i] = v;
            if constexpr (PUT) q.out2[i] = v;
        }
    }
}

__global__ __launch_bounds__(kThreads) void k_copy_multi(CopyBatch cb)
{
    const CopySeg& q = cb.s[blockIdx.y];
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    if (q.vec) {
        const uint4* s4 = reinterpret_cast<const uint4*>(q.src); uint4* d4 = reinterpret_cast<uint4*>(q.dst);
        const size_t n16 = q.bytes / 16;
        for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) d4[i] = s4[i];
    } else {
        for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < q.bytes; i += stride) q.dst[i] = q.src[i];
    }
}

// out = x + y + w: the opening of a three-party additive sharing.
__global__ __launch_bounds__(kThreads) void k_sum3(const u64* __restrict__ x, const u64* __restrict__ y,
                                                   const u64* __restrict__ w, u64* __restrict__ out, size_t n)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) out[i] = x[i] + y[i] + w[i];
}

inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

template <int OP>
int launch_binary(mpc_ctx* c, hipStream_t st, const u64* x, const u64* y, u64* out, size_t n)
{
    if (aligned16(x) && aligned16(y) && aligned16(out))
        hipLaunchKernelGGL(k_binary<OP>, dim3(grid_for(n / 2 + 1)), dim3(kThreads), 0, st, x, y, out, n);
    else
        hipLaunchKernelGGL(k_binary_scalar<OP>, dim3(grid_for(n)), dim3(kThreads), 0, st, x, y, out, n);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

}  // namespace

int launch_sub(mpc_ctx* c, hipStream_t st, const u64* x, const u64* a, u64* out, size_t n)
{
    return launch_binary<0>(c, st, x, a, out, n);
}

int launch_add(mpc_ctx* c, hipStream_t st, const u64* x, const u64* y, u64* out, size_t n)
{
    return launch_binary<1>(c, st, x, y, out, n);
}

// The "wire": a plain device copy kernel (kept as a kernel rather than
// hipMemcpyAsync so that the same path can be captured into a HIP graph).
int launch_copy(mpc_ctx* c, hipStream_t st, const void* src, void* dst, size_t bytes)
{
    if (bytes == 0) return MPC_OK;
    if (aligned16(src) && aligned16(dst) && bytes % 16 == 0) {
        const size_t n16 = bytes / 16;
        hipLaunchKernelGGL(k_copy16, dim3(grid_for(n16)), dim3(kThreads), 0, st,
                           (const uint4*)src, (uint4*)dst, n16);
    } else {
        hipLaunchKernelGGL(k_copy1, dim3(grid_for(bytes)), dim3(kThreads), 0, st,
                           (const u8*)src, (u8*)dst, bytes);
    }
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

int launch_sum3(mpc_ctx* c, hipStream_t st, const u64* x, const u64* y, const u64* w, u64* out, size_t n)
{
    if (n == 0) return MPC_OK;
    hipLaunchKernelGGL(k_sum3, dim3(grid_for(n)), dim3(kThreads), 0, st, x, y, w, out, n);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

int launch_truncate(mpc_ctx* c, hipStream_t st, u64* z, size_t n, int bits, int party)
{
    hipLaunchKernelGGL(k_truncate, dim3(grid_for(n)), dim3(kThreads), 0, st, z, n, bits, party);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

// contiguous k, and taps (if any) of at least two whole k blocks: the tile recoder; else one thread per (row, k block)
static bool rows_form(const RecodeArgs& a) { return a.k_stride == 1 && (a.ntaps == 1 || a.KB_tap >= 2); }
static unsigned rows_gy(const RecodeArgs& a) { return recode_tile_count(a.ntaps, a.KB_tap, a.KB_total); }

int launch_recode_multi(mpc_ctx* c, hipStream_t st, const RecodeArgs* sets, int count)
{
    if (count < 1 || count > kMaxRecodeSets) return MPC_EINVAL;
    bool rows_kind = true;          // every set a plain matrix with contiguous k?
    for (int i = 0; i < count; ++i)
        if (!rows_form(sets[i]) || sets[i].batch != sets[0].batch) rows_kind = false;
    if (rows_kind) {
        RecodeBatch rb{};
        int rows = 0; unsigned gy = 0;
        for (int i = 0; i < count; ++i) {
            rb.a[i] = sets[i];
            if (sets[i].plane_rows > rows) rows = sets[i].plane_rows;
            if (rows_gy(sets[i]) > gy) gy = rows_gy(sets[i]);
        }
        rb.batch = sets[0].batch;
        if ((size_t)count * rb.batch > 65535 || gy > 65535) return MPC_EINVAL;
        dim3 grid((rows + 63) / 64, gy, count * rb.batch);
        hipLaunchKernelGGL(k_recode_rows, grid, dim3(kThreads), 0, st, rb);
        MPC_HIP(c, hipGetLastError());
        return MPC_OK;
    }
    RecodeBatch rb{};
    size_t items = 0; int taps = 0;
    for (int i = 0; i < count; ++i) {
        rb.a[i] = sets[i];
        if (sets[i].batch != sets[0].batch) return MPC_EINVAL;
        const size_t it = (size_t)sets[i].KB_tap * sets[i].plane_rows;
        if (it > items) items = it;
        const int t = sets[i].ntaps + (sets[i].KB_total > sets[i].ntaps * sets[i].KB_tap ? 1 : 0);
        if (t > taps) taps = t;
    }
    rb.batch = sets[0].batch;
    if ((size_t)count * rb.batch > 65535) return MPC_EINVAL;
    dim3 grid(grid_for(items), taps, count * rb.batch);
    hipLaunchKernelGGL(k_recode_multi, grid, dim3(kThreads), 0, st, rb);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

// Up to kMaxRecodeSets recodings of either kind (contiguous k, or generic with taps) in one launch.
int launch_recode_any(mpc_ctx* c, hipStream_t st, const RecodeArgs* sets, int count)
{
    if (count < 1 || count > kMaxRecodeSets) return MPC_EINVAL;
    RecodeMixed m{};
    unsigned long long total = 0;
    for (int i = 0; i < count; ++i) {
        const RecodeArgs& a = sets[i];
        m.rb.a[i] = a;
        m.rows_kind[i] = rows_form(a);
        if (m.rows_kind[i]) {
            m.gx[i] = (unsigned)((a.plane_rows + 63) / 64); m.gy[i] = rows_gy(a);
        } else {
            m.gx[i] = (unsigned)grid_for((size_t)a.KB_tap * a.plane_rows);
            m.gy[i] = (unsigned)(a.ntaps + (a.KB_total > a.ntaps * a.KB_tap ? 1 : 0));
        }
        if (m.gx[i] == 0 || m.gy[i] == 0 || a.batch < 1) return MPC_EINVAL;
        m.first[i] = (unsigned)total;
        total += (unsigned long long)m.gx[i] * m.gy[i] * a.batch;
        if (total >= (1ull << 31)) return MPC_EINVAL;
    }
    m.first[count] = (unsigned)total;
    m.count = count;
    hipLaunchKernelGGL(k_recode_mixed, dim3((unsigned)total), dim3(kThreads), 0, st, m);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

int launch_sub_multi(mpc_ctx* c, hipStream_t st, const SubSeg* segs, int count)
{
    if (count < 1 || count > kMaxSegs) return MPC_EINVAL;
    SubBatch sb{}; size_t nmax = 0;
    for (int i = 0; i < count; ++i) {
        sb.s[i] = segs[i];
        sb.s[i].vec = aligned16(segs[i].x) && aligned16(segs[i].a) && aligned16(segs[i].out) &&
                      (!segs[i].out2 || aligned16(segs[i].out2));
        if (segs[i].n > nmax) nmax = segs[i].n;
        if ((segs[i].out2 != nullptr) != (segs[0].out2 != nullptr)) return MPC_EINVAL;    // all or none
    }
    if (segs[0].out2) hipLaunchKernelGGL(k_sub_multi<true>, dim3(grid_for(nmax / 2 + 1), count), dim3(kThreads), 0, st, sb);
    else              hipLaunchKernelGGL(k_sub_multi<false>, dim3(grid_for(nmax / 2 + 1), count), dim3(kThreads), 0, st, sb);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

int launch_copy_multi(mpc_ctx* c, hipStream_t st, const CopySeg* segs, int count)
{
    if (count < 1 || count > kMaxSegs) return MPC_EINVAL;
    CopyBatch cb{}; size_t bmax = 0;
    for (int i = 0; i < count; ++i) {
        cb.s[i] = segs[i];
        cb.s[i].vec = aligned16(segs[i].src) && aligned16(segs[i].dst) && segs[i].bytes % 16 == 0;
        if (segs[i].bytes > bmax) bmax = segs[i].bytes;
    }
    hipLaunchKernelGGL(k_copy_multi, dim3(grid_for(bmax / 16 + 1), count), dim3(kThreads), 0, st, cb);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

int launch_recode_im2col_t(mpc_ctx* c, hipStream_t st, const Im2colTArgs* sets, int count)
{
    if (count < 1 || count > 3) return MPC_EINVAL;
    Im2colTBatch bt{};
    for (int i = 0; i < count; ++i) bt.a[i] = sets[i];
    const Im2colTArgs& s = sets[0];          // the sets of a launch have one geometry
    // Three units a thread: its wave stores Cin units side by side, which fill a cache line from 8 channels on.  With fewer the
    // lines are written in parts, which the caches make up for while the planes are small; filter gradients, us, one unit a
    // thread / three: 8 x 32 x 32 x 1 36.2 / 37.6, 32 x 32 x 32 x 3 58.4 / 57.8, 8 x 112 x 112 x 3 114 / 124, 8 x 224 x 224 x 3 461 / 538,
    // 32 x 64 x 64 x 4 141 / 142, 8 x 224 x 224 x 4 508 / 538, 8 x 224 x 224 x 8 622 / 613.
    const long long npix = (long long)s.B * s.H * s.W;
    const bool rows_of_three = s.KH == 3 && s.KW == 3 && s.stride == 1 && s.pad == 1 && npix + 2ll * s.W + 32 < (1ll << 31) &&
                               (s.Cin >= 8 || (s.Cin > 1 && npix <= 16384ll * s.Cin));
    const size_t items = (size_t)s.KB_total * s.KH * s.Cin * (rows_of_three ? 1 : s.KW);
    if (rows_of_three) hipLaunchKernelGGL(k_recode_im2col3_t, dim3(grid_for(items), 1, count), dim3(kThreads), 0, st, bt);
    else               hipLaunchKernelGGL(k_recode_im2col_t, dim3(grid_for(items), 1, count), dim3(kThreads), 0, st, bt);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

int launch_mul_mask(mpc_ctx* c, hipStream_t st, const MulArgs& q)
{
    hipLaunchKernelGGL(k_mul_mask, dim3(grid_for(q.n), 2), dim3(kThreads), 0, st, q);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

int launch_mul_finish(mpc_ctx* c, hipStream_t st, const MulArgs& q)
{
    hipLaunchKernelGGL(k_mul_finish, dim3(grid_for(q.n), 2), dim3(kThreads), 0, st, q);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

int launch_dilate(mpc_ctx* c, hipStream_t st, const DilateArgs& q)
{
    const size_t total = (size_t)q.B * q.Hd * q.Wd * q.C;
    hipLaunchKernelGGL(k_dilate, dim3(grid_for(total), 4), dim3(kThreads), 0, st, q);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

int launch_poolbwd_pairs(mpc_ctx* c, hipStream_t st, const PoolBwdArgs& q)
{
    hipLaunchKernelGGL(k_poolbwd_pairs, dim3(grid_for(q.n_out), 2), dim3(kThreads), 0, st, q);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

int launch_poolbwd_scatter(mpc_ctx* c, hipStream_t st, const PoolBwdArgs& q)
{
    hipLaunchKernelGGL(k_poolbwd_scatter, dim3(grid_for(q.n_out), 2), dim3(kThreads), 0, st, q);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

int launch_recode(mpc_ctx* c, hipStream_t st, const RecodeArgs& a)
{
    if (rows_form(a)) return launch_recode_multi(c, st, &a, 1);
    const bool has_pad = a.KB_total > a.ntaps * a.KB_tap;
    const size_t items = (size_t)a.KB_tap * a.plane_rows;
    dim3 grid(grid_for(items), a.ntaps + (has_pad ? 1 : 0), a.batch);
    hipLaunchKernelGGL(k_recode, grid, dim3(kThreads), 0, st, a);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}
