// Masking, exchange by remote store and recoding of a linear layer's opened operands in one launch (single-queue lanes).
// A workgroup is two waves per party (two parties or three) on the same words: every wave masks its share (e_i = x_i - a_i),
// stores it into the peer's receive buffer in device memory, and after the workgroup barrier recodes what its party
// contracts: party 0 its own share plus the received word (a_0 + e = x_0 + e_1), party 1 the opened e.  Bound by memory:
// every share and mask is read once and every plane written once, six traversals of the operand, and the receive buffers
// stay in the L2.  As three launches (mask and send, open and recode, recode) there were eleven; 32 x 56 x 56 x 64
// words took 104 us in all, here 77 (4.0 TB/s).  Calls, same box, three launches / one: per-head Q K^T 342 / 305 us, A V 636 / 465,
// 1x1 convolution of 64 to 256 channels 362 / 334, 3x3 of 128 channels 233 / 222 (on another box, with all else that changed
// meanwhile, 328 / 296, 346 / 313 and 221 / 218: the last is bound by its GEMM), 8 products of 64 x 64 x 64 27.4 / 19.0.
// Plain calls write the planes of the masks from the same pass, seven traversals instead of twelve (left) and seventeen
// (right operand).
// Three parties: an operand's masks, broadcast, sum and recoding were four launches and 84 us for 64 x 16 x 16 x 128 words,
// 47 here.
// Non-temporal loads lose (3x3: 235 us): the operand was often written just before and is in the last-level cache.
#include "open_recode.h"
#include "digits.h"

#include <type_traits>

namespace {

typedef u64 u64v2u __attribute__((ext_vector_type(2), aligned(8)));

constexpr int kPartyThreads = 128;
// Tile of a workgroup where k is contiguous: KBT k blocks wide and 128 / KBT rows high, so that a thread has 16 words of it
// (narrow operands fill only the first k blocks of a wide tile: a 3x3 convolution of 3 channels, 32 x 56 x 56, takes 134 us a
// call on tiles of 64 k, 111 on tiles of 16).
constexpr int tile_rows(int KBT) { return 128 / KBT; }
// 32-bit words between k blocks of a plane in LDS: the blocks that a wave scatters to lie in different banks
constexpr int block_pitch(int KBT) { return tile_rows(KBT) * 4 + 64 / KBT; }
constexpr int kTileWords = 8 * (512 + 64);
int tile_blocks(int KB_total) { return KB_total > 2 ? 4 : KB_total; }
// Workgroups of a launch, as many as are resident at once: two parties three to a compute unit (168 registers; held at 128
// for a fourth they are spilled, and the 3x3 convolution takes 228 us), two in plain calls (228); three parties two and one.
// None fits beside a GEMM wave's 376 on a SIMD: another lane's opening waits for the GEMM's units.
// 512 / 768 / 1024 workgroups of folded calls: level within 1-2 %.
constexpr unsigned max_blocks(int parties, OpenPlanes planes)
{
    return parties == 2 ? (planes == OpenPlanes::kFolded ? 768 : 512) : planes == OpenPlanes::kMasks ? 256 : 512;
}
constexpr int waves_per_simd(int parties, OpenPlanes planes) { return planes == OpenPlanes::kMasks ? 2 : 3; }

struct OpenBatch { OpenSet s[kMaxOpenSets]; int count; unsigned tiles; u8* box; };

// The receive buffers: per workgroup and ordered pair of parties, kWords words per thread.  Party i's buffer k holds what
// party (i + 1 + k) mod NP sent last.
template <int NP>
struct Exchange {
    static constexpr int kWords = NP == 2 ? 8 : 4;
    static constexpr unsigned kBox = kPartyThreads * kWords * 8;
    static_assert((size_t)NP * (NP - 1) * kBox == open_box_bytes(NP), "buffers of a workgroup");
    u8 *in, *out[NP - 1]; unsigned at;
    __device__ __forceinline__ Exchange(u8* box, int party, int t)
    {
        u8* const wg = box + (size_t)blockIdx.x * open_box_bytes(NP);
        in = wg + party * (NP - 1) * kBox;
#pragma unroll
        for (int k = 0; k < NP - 1; ++k) {
            int to = party + NP - 1 - k; if (to >= NP) to -= NP;
            out[k] = wg + (to * (NP - 1) + k) * kBox;
        }
        at = (unsigned)t * 16;
    }
    // kWords words to every peer, and the sum of what the peers sent; 16 bytes per lane and access, lanes side by side
    __device__ __forceinline__ void swap(const u64 (&mine)[kWords], u64 (&theirs)[kWords]) const
    {
        __syncthreads();                   // the peers hold the last words they were sent
#pragma unroll
        for (int k = 0; k < NP - 1; ++k)
#pragma unroll
            for (int q = 0; q < kWords / 2; ++q)
                *reinterpret_cast<u64v2u*>(out[k] + q * (kPartyThreads * 16) + at) = u64v2u{ mine[2 * q], mine[2 * q + 1] };
        __syncthreads();
        u64v2u w[NP - 1][kWords / 2];
#pragma unroll
        for (int k = 0; k < NP - 1; ++k)
#pragma unroll
            for (int q = 0; q < kWords / 2; ++q) w[k][q] = *reinterpret_cast<const u64v2u*>(in + k * kBox + q * (kPartyThreads * 16) + at);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < kWords / 2; ++q) {
            theirs[2 * q] = w[0][q].x; theirs[2 * q + 1] = w[0][q].y;
            if constexpr (NP == 3) { theirs[2 * q] += w[1][q].x; theirs[2 * q + 1] += w[1][q].y; }
        }
    }
};

// Contiguous k: lanes along k read the tile, digits go to LDS in plane order, planes are written with lanes along rows.
// H = 1: tiles of which at most half the rows are there (few-row products), half the loads and one exchange.
template <int NP, OpenPlanes PLANES, int KBT, int H>
__device__ __forceinline__ void open_rows(const OpenSet& s, const Exchange<NP>& ex, int party, int t, int b, int row0, int kb0, uint32_t* tile)
{
    const u64* x = s.x[party] + (long long)b * s.src_batch_stride;
    const u64* a = s.a[party] + (long long)b * s.src_batch_stride;
    // thread's segments: 4 words each, segment p at row t / lanes + step p of the tile
    constexpr int lanes = 4 * KBT, step = kPartyThreads / lanes, pitch = block_pitch(KBT);
    const int s4 = t % lanes, k = kb0 * 16 + s4 * 4;
    const bool beyond = k >= s.K, whole = beyond ? s.K > 3 : k + 3 < s.K;
    const int kc = beyond ? 0 : k;
    u64 v[2 * H][4], m[2 * H][4];
    // all loads in one straight line per way of access
    auto load = [&](auto whole_tag, const u64* q, u64 (&w)[2 * H][4]) {
#pragma unroll
        for (int p = 0; p < 2 * H; ++p) {
            const int r = row0 + t / lanes + step * p;
            const u64* const e = q + (long long)(r < s.rows ? r : 0) * s.row_stride;
            if constexpr (decltype(whole_tag)::value) {
                const u64v2u lo = *reinterpret_cast<const u64v2u*>(e + kc);
                const u64v2u hi = *reinterpret_cast<const u64v2u*>(e + kc + 2);
                w[p][0] = lo.x; w[p][1] = lo.y; w[p][2] = hi.x; w[p][3] = hi.y;
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) w[p][u] = e[k + u < s.K ? k + u : 0];
            }
        }
    };
    if (whole) { load(std::true_type{}, x, v); load(std::true_type{}, a, m); }
    else       { load(std::false_type{}, x, v); load(std::false_type{}, a, m); }
    auto scatter = [&](int p, const u64 (&w)[4]) {
        const int r = t / lanes + step * p;
        const bool row_ok = row0 + r < s.rows;
        u64 four[4]; uint32_t d[8];
#pragma unroll
        for (int u = 0; u < 4; ++u) four[u] = row_ok && k + u < s.K ? w[u] : 0;
        digits_of_4(four, d);
#pragma unroll
        for (int q = 0; q < 8; ++q) tile[(q * KBT + (s4 >> 2)) * pitch + r * 4 + (s4 & 3)] = d[q];
    };
    auto store = [&](u8* dst) {
        const int kbl = t / tile_rows(KBT), row = t % tile_rows(KBT);
        if (!dst || row0 + row >= s.plane_rows || kb0 + kbl >= s.KB_total) return;
        u8* const o = dst + (size_t)b * s.dst_batch_stride + ((size_t)(kb0 + kbl) * s.plane_rows + row0 + row) * 16;
#pragma unroll
        for (int q = 0; q < 8; ++q)
            *reinterpret_cast<uint4*>(o + (size_t)q * s.digit_stride) = *reinterpret_cast<const uint4*>(&tile[(q * KBT + kbl) * pitch + row * 4]);
    };
    constexpr int W = Exchange<NP>::kWords;
#pragma unroll
    for (int h = 0; h < 8 * H / W; ++h) {
        u64 e[W], got[W];
#pragma unroll
        for (int q = 0; q < W; ++q) e[q] = v[(h * W + q) / 4][q % 4] - m[(h * W + q) / 4][q % 4];
        ex.swap(e, got);
        // party 0 recodes the opened words (the parties of kOpened in turn, and a third of the planes each: no faster)
        if (PLANES != OpenPlanes::kFolded && party) continue;
#pragma unroll
        for (int p = h * W / 4; p < (h + 1) * W / 4; ++p) {
            u64 four[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = 4 * p + u - h * W;
                four[u] = (PLANES == OpenPlanes::kFolded && party == 0 ? v[p][u] : e[q]) + got[q];
                if (PLANES == OpenPlanes::kMasks && s.add_open) m[p][u] += four[u];
            }
            scatter(p, four);
        }
    }
    __syncthreads();
    store(s.dst[party]);
    if constexpr (PLANES == OpenPlanes::kMasks) {
        __syncthreads();
#pragma unroll
        for (int p = 0; p < 2 * H; ++p) scatter(p, m[p]);
        __syncthreads();
        store(s.mask_dst[party]);
    }
}

// Contiguous rows (an operand stored [K][N], a filter): a thread takes one (row, k block of a tap), lanes along rows.
template <int NP, OpenPlanes PLANES>
__device__ __forceinline__ void open_columns(const OpenSet& s, const Exchange<NP>& ex, int party, int t, int b, unsigned bx, unsigned kb)
{
    const int tap = s.ntaps == 1 ? 0 : (int)kb / s.KB_tap;             // == ntaps: padding behind the last tap
    const int row = (int)bx * kPartyThreads + t, k0 = ((int)kb - tap * s.KB_tap) * 16;
    const bool there = row < s.rows && tap < s.ntaps && k0 < s.K;
    const int have = there ? (s.K - k0 < 16 ? s.K - k0 : 16) : 0;      // valid words of the unit
    const long long at = (long long)b * s.src_batch_stride + (there ? tap * s.tap_stride + row * s.row_stride + k0 * s.k_stride : 0);
    const u64 *x = s.x[party] + at, *a = s.a[party] + at;
    u64 v[16], m[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = x[(long long)(u < have ? u : 0) * s.k_stride];
#pragma unroll
    for (int u = 0; u < 16; ++u) m[u] = a[(long long)(u < have ? u : 0) * s.k_stride];
    auto store = [&](u8* dst, const u64 (&w)[16]) {
        if (!dst || row >= s.plane_rows) return;
        uint32_t unit[8][4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            u64 four[4]; uint32_t d[8];
#pragma unroll
            for (int u = 0; u < 4; ++u) four[u] = 4 * p + u < have ? w[4 * p + u] : 0;
            digits_of_4(four, d);
#pragma unroll
            for (int q = 0; q < 8; ++q) unit[q][p] = d[q];
        }
        u8* const o = dst + (size_t)b * s.dst_batch_stride + ((size_t)kb * s.plane_rows + row) * 16;
#pragma unroll
        for (int q = 0; q < 8; ++q)
            *reinterpret_cast<uint4*>(o + (size_t)q * s.digit_stride) = make_uint4(unit[q][0], unit[q][1], unit[q][2], unit[q][3]);
    };
    constexpr int W = Exchange<NP>::kWords;
#pragma unroll
    for (int h = 0; h < 16 / W; ++h) {
        u64 e[W], got[W];
#pragma unroll
        for (int q = 0; q < W; ++q) e[q] = v[W * h + q] - m[W * h + q];
        ex.swap(e, got);
#pragma unroll
        for (int q = 0; q < W; ++q) {
            v[W * h + q] = (PLANES == OpenPlanes::kFolded && party == 0 ? v[W * h + q] : e[q]) + got[q];
            if (PLANES == OpenPlanes::kMasks && party == 0 && s.add_open) m[W * h + q] += v[W * h + q];
        }
    }
    store(s.dst[party], v);
    if constexpr (PLANES == OpenPlanes::kMasks) store(s.mask_dst[party], m);
}

template <int NP, OpenPlanes PLANES>
__global__ __launch_bounds__(NP * kPartyThreads, waves_per_simd(NP, PLANES)) void k_open_recode(OpenBatch g)
{
    __shared__ __align__(16) uint32_t lds[NP == 2 || PLANES == OpenPlanes::kMasks ? NP : 1][kTileWords];
    const int party = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kPartyThreads));
    const int t = threadIdx.x % kPartyThreads;
    uint32_t* const tile = lds[sizeof(lds) / sizeof(lds[0]) == 1 ? 0 : party];
    const Exchange<NP> ex(g.box, party, t);
    for (unsigned id = blockIdx.x; id < g.tiles; id += gridDim.x) {
        const OpenSet& s = g.s[g.count > 1 && id >= g.s[1].first ? 1 : 0];
        unsigned q = id - s.first;
        const unsigned bx = q % s.gx; q /= s.gx;
        const unsigned by = q % s.gy; const int b = (int)(q / s.gy);
        if (!s.kbt) { open_columns<NP, PLANES>(s, ex, party, t, b, bx, by); continue; }
        const int row0 = (int)bx * tile_rows(s.kbt), kb0 = (int)by * s.kbt;
        if (s.kbt == 1)                    open_rows<NP, PLANES, 1, 2>(s, ex, party, t, b, row0, kb0, tile);
        else if (s.kbt == 2)               open_rows<NP, PLANES, 2, 2>(s, ex, party, t, b, row0, kb0, tile);
        else if (s.plane_rows - row0 > 16) open_rows<NP, PLANES, 4, 2>(s, ex, party, t, b, row0, kb0, tile);
        else                               open_rows<NP, PLANES, 4, 1>(s, ex, party, t, b, row0, kb0, tile);
    }
}

template <int NP, OpenPlanes PLANES>
void launch(hipStream_t st, const OpenBatch& g, size_t box_bytes)
{
    // as many workgroups as have buffers, all of them with the same number of tiles (but for the last few)
    unsigned long long blocks = box_bytes / open_box_bytes(NP);
    if (blocks > max_blocks(NP, PLANES)) blocks = max_blocks(NP, PLANES);
    const unsigned long long rounds = (g.tiles + blocks - 1) / blocks;
    blocks = (g.tiles + rounds - 1) / rounds;
    hipLaunchKernelGGL((k_open_recode<NP, PLANES>), dim3((unsigned)blocks), dim3(NP * kPartyThreads), 0, st, g);
}

// tiles of a set; fills kbt, gx and gy
unsigned long long lay_tiles(OpenSet& s)
{
    s.kbt = s.k_stride == 1 && s.ntaps == 1 ? tile_blocks(s.KB_total) : 0;
    const int high = s.kbt ? tile_rows(s.kbt) : kPartyThreads, wide = s.kbt ? s.kbt : 1;
    s.gx = (unsigned)((s.plane_rows + high - 1) / high);
    s.gy = (unsigned)((s.KB_total + wide - 1) / wide);
    return (unsigned long long)s.gx * s.gy * s.batch;
}

}  // namespace

// A tile takes its time however few of its 2048 words there are, and a launch with more tiles than workgroups takes them in
// rounds, where the kernels it replaces have threads for the words that exist.  Two parties lose with long operands of few
// contiguous rows ([K][N] with few columns, [K][M] with few rows); tiles across k of narrow operands stay ahead (3x3
// convolutions of 1 to 3 channels 0.94-0.96 of the other kernels' time).  Three parties lose with either, in plain calls, whose
// other launches are more, only after many rounds.  Calls, us, this launch / separate kernels: 3 x 20000 x 4 twice 49.3 / 36.2,
// the same transposed 62.2 / 31.6, folded 47.6 / 34.7, 17 x 3000 x 8 sixteen times 53.8 / 43.4; three parties, prepared, 3000 x 2 x 40
// sixteen times 65.5 / 54.0, plain 71.8 / 74.0, 3 x 3000 x 4 sixteen times 95.4 / 63.0.  From a sixth of the words on they are level.
bool open_pays(int parties, OpenPlanes planes, const OpenSet* sets, int count)
{
    unsigned long long tiles = 0, words = 0, col_tiles = 0, col_words = 0;
    for (int i = 0; i < count; ++i) {
        OpenSet s = sets[i];
        const unsigned long long t = lay_tiles(s), w = (unsigned long long)s.rows * s.K * s.ntaps * s.batch;
        tiles += t; words += w;
        if (!s.kbt) { col_tiles += t; col_words += w; }
    }
    const unsigned blocks = max_blocks(parties, planes);
    if (tiles <= blocks) return true;
    if (parties == 2) return col_tiles * 2 < tiles || col_words * 6 >= col_tiles * 2048;
    return words * 6 >= tiles * 2048 || (planes == OpenPlanes::kMasks && tiles <= 8ull * blocks);
}

size_t open_most_tiles(int plane_rows, int KB_total, int batch)
{
    const size_t rows = (size_t)plane_rows, kbt = (size_t)tile_blocks(KB_total), high = (size_t)tile_rows((int)kbt);
    const size_t by_rows = (rows + high - 1) / high * ((KB_total + kbt - 1) / kbt), by_columns = (rows + kPartyThreads - 1) / kPartyThreads * KB_total;
    return (by_rows > by_columns ? by_rows : by_columns) * batch;
}
size_t open_most_blocks(int parties)
{
    const unsigned plain = max_blocks(parties, OpenPlanes::kMasks), other = max_blocks(parties, parties == 2 ? OpenPlanes::kFolded : OpenPlanes::kOpened);
    return plain > other ? plain : other;
}

int launch_open_recode(mpc_ctx* c, hipStream_t st, int parties, OpenPlanes planes, const OpenSet* sets, int count, u8* box, size_t box_bytes)
{
    if (parties < 2 || parties > 3 || count < 1 || count > kMaxOpenSets || !box || box_bytes < open_box_bytes(parties)) return MPC_EINVAL;
    if (parties == (planes == OpenPlanes::kFolded ? 3 : planes == OpenPlanes::kOpened ? 2 : 0)) return MPC_EINVAL;
    OpenBatch g{};
    unsigned long long tiles = 0;
    for (int i = 0; i < count; ++i) {
        OpenSet& s = g.s[i];
        s = sets[i];
        if (s.rows < 1 || s.K < 1 || s.batch < 1 || s.plane_rows < s.rows || (long long)s.KB_total * 16 < s.K) return MPC_EINVAL;
        if (!can_open(s) || s.ntaps < 1 || s.KB_tap < 1) return MPC_EINVAL;
        s.first = (unsigned)tiles;
        tiles += lay_tiles(s);
        if (tiles >= (1ull << 31)) return MPC_EINVAL;
    }
    g.count = count; g.tiles = (unsigned)tiles; g.box = box;
    if (planes == OpenPlanes::kFolded)      launch<2, OpenPlanes::kFolded>(st, g, box_bytes);
    else if (planes == OpenPlanes::kOpened) launch<3, OpenPlanes::kOpened>(st, g, box_bytes);
    else if (parties == 2)                  launch<2, OpenPlanes::kMasks>(st, g, box_bytes);
    else                                    launch<3, OpenPlanes::kMasks>(st, g, box_bytes);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}
