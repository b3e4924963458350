// Ring GEMM over Z_2^64 on the int8 matrix cores.
//
// A ring word is split into eight balanced base-256 digits d_j in [-128,127].
// Mod 2^64 only digit pairs with i + j <= 7 contribute, so one ring MAC is 36
// int8 products; products with equal s = i + j share one int32 accumulator
// (exact while (s+1) * K * 2^14 < 2^31 for s <= 3; for s >= 4 only the low
// 64 - 8s <= 32 bits matter, so wrap-around there is harmless).  The epilogue
// recombines sum_s acc_s * 2^(8s) mod 2^64, adds the party's addend (c_i or a
// partial sum), optionally truncates, and stores.
//
// One wave per SIMD, the whole register file per wave: a wave owns a 32x64
// output tile = 2 x 8 digit-sum groups x 16 accumulator registers (256 AGPRs)
// and issues 72 v_mfma_i32_32x32x32_i8 per 32-deep K step.  A workgroup of
// WGM x WGN waves streams the eight digit planes of its (32*WGM)-row left tile
// and (64*WGN)-row right tile through a three-slot LDS ring filled by direct
// global->LDS loads (no staging registers).  Every load is "scalar base +
// per-lane constant offset": the lane offsets are fixed for the whole kernel
// and the bases advance with scalar arithmetic, so the loader costs almost no
// vector ALU work.  Inside a K step an operand register is refilled from the
// next ring slot right after its last use, and the global loads for step t+3
// are issued in the same MFMA shadow.  The planes' [kb][row][16] layout makes
// the global reads and the ds_read_b128 operand fetches contiguous in lane
// order.
//
// The contraction may run over two operand segments (party i contracts
// [e | a_i] against [b_i' ; f]) and, for convolutions, the left tile loader
// gathers filter taps from NHWC activation planes (implicit im2col); taps
// that fall into the zero padding read the all-zero row that ends every
// activation plane.
//
// Products with few output tiles take another form (k_sliced_gemm): a workgroup
// has one 32 x 32 tile, its waves slices of the contraction, and operands go
// straight into registers.
#include <atomic>
#include "common.h"
#include "overlap.h"

#include <type_traits>
#include <utility>

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int KS = 2;   // 16-wide k blocks per pipeline stage = one MFMA K step

// Division by a number the host knows: n / d for n < 2^31, exact with mul = ceil(2^(31 + s) / d), s = ceil(log2 d)
// (Granlund and Montgomery, "Division by invariant integers using multiplication").
struct Divider {
    unsigned mul; int shift;
    __host__ static Divider by(unsigned d)
    {
        int s = 0;
        while ((1ull << s) < d) ++s;
        return Divider{ (unsigned)(((1ull << (31 + s)) + d - 1) / d), 31 + s };
    }
    __device__ __forceinline__ unsigned operator()(unsigned n) const { return (unsigned)(((u64)n * mul) >> shift); }
};

// What a launch passes to the kernel: everything of a party in one place, and the divisors of the tile order.  A
// workgroup runs through its set-up alone, mostly as one chain of scalar instructions and loads, before it can ask for
// its first tile; with divisions in the kernel and a party's operands picked field by field that was 490 instructions
// (convolutions 710-800), as long as the matrix work of a 64-deep contraction; now 370 (540-610) (per-head Q K^T 334 -> 330 us).
struct GemmParty {
    GemmSeg seg[2];
    const u64 *addend, *addend2; u64* out;
    int tiles, per_xcd;                     // tiles of the party, and how many of them an XCD owns
};
struct GemmDev {
    GemmParty p[3];
    int M, N, rows_L, nseg, nparty, trunc_bits, ksplit, steps_per_split;
    long long out_bstride;
    u64* partial;
    unsigned heavy_blocks;                  // > 0: so many workgroups of party 1 come first, then party 0's
    unsigned per_item, batch, panel_tiles, tiles_n, last_width;
    int by_columns;                         // k_sliced_gemm: the order of an item's tiles
    Divider by_item, by_batch, by_panel, by_last_width, by_Wo, by_Ho;
    ConvGeom conv;
};
// Widest output whose words the epilogue addresses by a 32-bit lane offset: the last lane's is (4 N + 31) words.
constexpr int kLaneOffsetMaxN = (1 << 27) - 8;
constexpr u64 last_lane_offset(u64 N) { return (4 * N + 31) * 8; }
static_assert(last_lane_offset(kLaneOffsetMaxN) < (1ull << 32), "the widest output's lane offsets fit 32 bits");
static_assert(last_lane_offset(kLaneOffsetMaxN + 1) >= (1ull << 32), "and no wider one's do");

// LDS ring depth: three slots for the one-workgroup-per-unit tiles; two for the small tile of short
// contractions, which then fits twice on a compute unit

// NH: 32-column halves of a wave's output tile (2: 32 x 64, all 256 accumulator registers, one wave per SIMD;
// 1: 32 x 32, 128 accumulator registers, two waves per SIMD).
template <int WGM, int WGN, int NS, int NH>
struct Cfg {
    static constexpr int WN = 32 * NH;
    static constexpr int TM = 32 * WGM, TN = WN * WGN, NW = WGM * WGN, NT = 64 * NW;
    static constexpr int LM = TM < 64 ? 64 : TM;      // left rows held: whole 64-row loads (a 32-row tile reads its rows clamped)
    static constexpr int L_UNITS = 8 * KS * LM, R_UNITS = 8 * KS * TN;   // 16-byte units per stage
    static constexpr int STAGE_UNITS = L_UNITS + R_UNITS;
    static constexpr size_t LDS_BYTES = (size_t)NS * STAGE_UNITS * 16;
    // Tiles are loaded in chunks of 64 rows x 16 bytes (one wave-wide load).
    // Wave w loads digits w, w+NW, ... (DPW of them) of every k block and row
    // chunk: load j <-> digit w + NW*(j % DPW), k block (j / DPW) % KS,
    // row chunk j / (DPW * KS).
    static constexpr int RCM = LM / 64, RCN = TN / 64;
    static constexpr int DPW = 8 / NW;
    static constexpr int LPW = DPW * KS * RCM, RPW = DPW * KS * RCN;     // loads per wave per stage
    static_assert(LM % 64 == 0 && TN % 64 == 0, "operand tiles are whole numbers of 64-row chunks");
    static_assert(8 % NW == 0, "digits divide evenly over waves");
};

template <typename F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// s_waitcnt immediate that waits for vmcnt <= n only (gfx9 encoding)
constexpr int vmcnt_imm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }

// One wave-wide direct global->LDS load: lane l's 16 bytes at base + voff(l)
// land at lds_slot + LDS_OFF + 16*l.  Issued through inline assembly so that
// completion is tracked by this kernel's own vmcnt waits (see the main loop).
template <int LDS_OFF>
__device__ __forceinline__ void load_lds16(const u8* base, unsigned voff, unsigned lds_slot)
{
    asm volatile("s_add_u32 m0, %0, %1\n\tglobal_load_lds_dwordx4 %2, %3"
                 :: "s"(lds_slot), "n"(LDS_OFF), "v"(voff), "s"(base) : "memory", "scc");
}

// Recombination sum_s d_s 2^(8s) mod 2^64 of a word's eight digit sums in 32-bit pieces: those of weights 0..3 add up exactly
// as 64-bit terms built from two shifts each; of weights 4..7 only the low 32 bits reach the result, and those land in the
// high word.
__device__ __forceinline__ u64 recombine(const int (&d)[8])
{
    u64 acc64 = (u64)(long long)d[0];
#pragma unroll
    for (int sg = 1; sg < 4; ++sg)
        acc64 += (u64)((unsigned)d[sg] << (8 * sg)) | ((u64)(unsigned)(d[sg] >> (32 - 8 * sg)) << 32);
    const unsigned high = (unsigned)d[4] + ((unsigned)d[5] << 8) + ((unsigned)d[6] << 16) + ((unsigned)d[7] << 24);
    return acc64 + ((u64)high << 32);
}

template <int WGM, int WGN, bool CONV, int NS, int NH>
__device__ __forceinline__ void gemm_tile(const GemmDev& g)
{
    using C = Cfg<WGM, WGN, NS, NH>;
    extern __shared__ uint4 lds[];
    const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)lds;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WGM, wn = wave / WGM;
    const int i32 = lane & 31, g2 = lane >> 5;
    // One-dimensional grid.  Workgroups go to the eight XCDs (each with its own L2) round-robin by their
    // linear id, and XCD r owns a contiguous range of the tile sequence, so that the workgroups resident on
    // an XCD at one time are neighbours in that sequence.  The sequence runs over (split, batch item), then
    // panels of GN column tiles, then row tiles, then the column tiles of the panel: what an XCD holds at a
    // time is a block of a few row tiles by up to GN column tiles of one item, whose left and right tiles
    // are fetched into that L2 once (convolutions: neighbouring pixel tiles also share the rows their filter
    // taps overlap on).  Measured with the fetch counter: the 256-wide 1x1 convolution on 56 x 56 x 64 moved
    // 983 MiB with the row tiles of one column running first, per-head Q K^T 1032 MiB with the tiles dealt
    // round-robin; in this order 547 and 539 MiB (the minimum is 539 and 528).
    //  - parties with equal work: both parties' workgroups of a tile one after the other (they share e and f);
    //  - parties that contract different lengths: party 1's workgroups (the long ones) fill the chip first,
    //    party 0's follow as units free up.
    const unsigned id = blockIdx.x;
    int party; unsigned q, tile;
    if (g.heavy_blocks) {
        party = id < g.heavy_blocks ? 1 : 0;
        q = (party ? id : id - g.heavy_blocks) >> 3;
    } else {
        const unsigned sl = id >> 3;
        party = g.nparty == 2 ? (int)(sl & 1) : 0;
        q = g.nparty == 2 ? sl >> 1 : sl;
    }
    const GemmParty P = g.p[party];
    tile = (id & 7) * (unsigned)P.per_xcd + q;
    if (q >= (unsigned)P.per_xcd || tile >= (unsigned)P.tiles) return;      // padding of the last group of eight
    constexpr unsigned GN = NH == 1 && C::TN == 64 ? 8 : 4;
    const unsigned t2 = g.by_item(tile), tq = tile - t2 * g.per_item;
    const unsigned panel = g.by_panel(tq), rem = tq - panel * g.panel_tiles;
    const bool whole_panel = g.tiles_n - panel * GN >= GN;
    const unsigned row_tile = whole_panel ? rem / GN : g.by_last_width(rem);
    const int mt = (int)row_tile;
    const int nt = (int)(panel * GN + rem - row_tile * (whole_panel ? GN : g.last_width));
    const int split = (int)g.by_batch(t2);
    const int bidx = (int)(t2 - (unsigned)split * g.batch);
    const int m0 = mt * C::TM, n0 = nt * C::TN;

    // ---- per-party operands as scalars
    const GemmSeg &sg0 = P.seg[0], &sg1 = P.seg[1];
    const int KB0 = sg0.KB, KB1 = g.nseg > 1 ? sg1.KB : 0;        // a party's second segment may be empty
    // K steps of this workgroup: all of them, or one slice when the contraction is split
    const int T_all = (KB0 + KB1) / KS;
    const int st0 = split * g.steps_per_split;
    const int T = T_all - st0 < g.steps_per_split ? T_all - st0 : g.steps_per_split;
    if (T <= 0) return;             // cannot happen: the launcher gives each party ceil(steps / steps_per_split) slices
    const long long krowL = (long long)g.rows_L * 16;      // bytes between k blocks of a left plane
    const long long krowR = (long long)g.N * 16;

    // ---- per-lane constant byte offsets
    // conv: pixel index of filter tap (0,0), biased so that it is never negative, nor the zero row's distance from any tap's
    // base (a filter higher than the whole batch: 5x5 on three images of 1 x 1; the last tap here is the one past the end)
    int bias = CONV ? g.conv.pad * g.conv.W + g.conv.pad : 0;
    if (CONV && g.conv.npix < (long long)g.conv.KH * g.conv.W + g.conv.KW) {
        const int need = g.conv.KH * g.conv.W + g.conv.KW - (int)g.conv.npix;
        bias = bias > need ? bias : need;
    }
    unsigned voffL[C::RCM];
    unsigned long long lvalid[C::RCM];      // conv: bit per filter tap that hits the image
#pragma unroll
    for (int rc = 0; rc < C::RCM; ++rc) {
        int m = m0 + rc * 64 + lane; if (m > g.M - 1) m = g.M - 1;
        if (CONV) {
            const int t = (int)g.by_Wo((unsigned)m), wo = m - t * g.conv.Wo;
            const int b = (int)g.by_Ho((unsigned)t), ho = t - b * g.conv.Ho;
            const int hi0 = ho * g.conv.stride - g.conv.pad, wi0 = wo * g.conv.stride - g.conv.pad;
            const long long pix00 = ((long long)b * g.conv.H + hi0) * g.conv.W + wi0;
            voffL[rc] = (unsigned)((pix00 + bias) * 16);
            unsigned long long v = 0;
            for (int kh = 0; kh < g.conv.KH; ++kh)
                for (int kw = 0; kw < g.conv.KW; ++kw) {
                    const int hi = hi0 + kh, wi = wi0 + kw;
                    if (hi >= 0 && hi < g.conv.H && wi >= 0 && wi < g.conv.W)
                        v |= 1ull << (kh * g.conv.KW + kw);
                }
            lvalid[rc] = v;
        } else {
            voffL[rc] = (unsigned)m * 16u; lvalid[rc] = ~0ull;
        }
    }
    unsigned voffR[C::RCN];
#pragma unroll
    for (int rc = 0; rc < C::RCN; ++rc) {
        int n = n0 + rc * 64 + lane; if (n > g.N - 1) n = g.N - 1;
        voffR[rc] = (unsigned)n * 16u;
    }
    const int ntaps = CONV ? g.conv.KH * g.conv.KW : 0;
    const int CB = CONV ? g.conv.CB : 1, KWf = CONV ? g.conv.KW : 1, Wimg = CONV ? g.conv.W : 0;
    const long long npix = CONV ? g.conv.npix : 0;          // the zero row of a plane has index npix

    // ---- loader state (all scalar).  segL / segR already point at this wave's
    // first digit plane; dsL / dsR are the byte strides between the digit
    // planes a wave loads (NW planes apart).
    const u8 *segL, *segR; long long dsL, dsR;
    auto set_segment = [&](int seg) {
        const GemmSeg& q = seg ? sg1 : sg0;
        segL = q.L + (size_t)bidx * q.L_bstride + (long long)wave * q.L_dstride;
        segR = q.R + (size_t)bidx * q.R_bstride + (long long)wave * q.R_dstride;
        dsL = q.L_dstride * C::NW; dsR = q.R_dstride * C::NW;
    };
    // cursor at K step st0
    int c_seg = st0 * KS >= KB0 ? 1 : 0;
    int c_kb = st0 * KS - (c_seg ? KB0 : 0);
    int c_tap = CONV ? c_kb / CB : 0, c_cb = CONV ? c_kb - c_tap * CB : 0;
    int c_kw = CONV ? c_tap % KWf : 0;
    int c_dpix = CONV ? (c_tap / KWf) * Wimg + c_kw : 0;
    long long c_offL = (long long)c_kb * krowL, c_offR = (long long)c_kb * krowR;       // c_kb * krowL / krowR
    set_segment(c_seg);
    auto cursor_next = [&]() {      // advance by one k block
        ++c_kb; c_offL += krowL; c_offR += krowR;
        if (CONV) {
            if (++c_cb == CB) {
                c_cb = 0; ++c_tap;
                if (++c_kw == KWf) { c_kw = 0; c_dpix += Wimg - (KWf - 1); } else ++c_dpix;
            }
        }
        if (c_seg == 0 && c_kb == KB0) {
            c_seg = 1; c_kb = 0; c_tap = 0; c_cb = 0; c_dpix = 0; c_kw = 0; c_offL = 0; c_offR = 0;
            set_segment(1);
        }
    };

    // State of the stage being issued, captured once per stage; the stage's
    // loads are then issued one by one between MFMAs.
    const u8* s_L[KS]; const u8* s_R[KS];
    unsigned s_zoff[KS]; int s_tap[KS];
    unsigned s_slotL, s_slotR; long long s_dsL, s_dsR;
    auto stage_begin = [&](int slot) {
        // KS divides every segment, so a stage never straddles two segments
        // (the cursor may move on to the next segment at the end of this stage)
        s_dsL = dsL; s_dsR = dsR;
        s_slotL = lds_base + (unsigned)(slot * C::STAGE_UNITS * 16) + (unsigned)(wave * KS * C::LM * 16);
        s_slotR = lds_base + (unsigned)((slot * C::STAGE_UNITS + C::L_UNITS) * 16) + (unsigned)(wave * KS * C::TN * 16);
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            s_R[kk] = segR + c_offR;
            if (CONV) {
                // base such that base + (pix00 + bias)*16 is the tap pixel's unit in channel block c_cb
                s_L[kk] = segL + ((long long)c_cb * (npix + 1) + c_dpix - bias) * 16;
                s_zoff[kk] = (unsigned)((npix - c_dpix + bias) * 16);   // lands on the zero row instead
                s_tap[kk] = c_tap;
            } else {
                s_L[kk] = segL + c_offL;
            }
            cursor_next();
        }
    };
    // q-th load of the stage (left tile first), q a compile-time constant
    auto issue_one = [&](auto q_tag) {
        constexpr int q = decltype(q_tag)::value;
        if constexpr (q < C::LPW) {
            constexpr int dj = q % C::DPW, kk = (q / C::DPW) % KS, rc = q / (C::DPW * KS);
            unsigned voff = voffL[rc];
            if (CONV) {
                const bool ok = s_tap[kk] < ntaps && ((lvalid[rc] >> (s_tap[kk] & 63)) & 1);
                voff = ok ? voff : s_zoff[kk];
            }
            // destination unit: ((d*KS + kk)*LM + rc*64) with d = wave + NW*dj
            load_lds16<((C::NW * dj * KS + kk) * C::LM + rc * 64) * 16>(s_L[kk] + dj * s_dsL, voff, s_slotL);
        } else {
            constexpr int r = q - C::LPW;
            constexpr int dj = r % C::DPW, kk = (r / C::DPW) % KS, rc = r / (C::DPW * KS);
            load_lds16<((C::NW * dj * KS + kk) * C::TN + rc * 64) * 16>(s_R[kk] + dj * s_dsR, voffR[rc], s_slotR);
        }
    };
    constexpr int PER_STAGE = C::LPW + C::RPW;
    constexpr int EVERY = 36 * NH / PER_STAGE < 4 ? 36 * NH / PER_STAGE : 4;       // MFMAs per load
    static_assert(EVERY >= 2, "every load of a stage has a place between the MFMAs");
    auto issue_all = [&](int slot) {
        stage_begin(slot);
        static_for<PER_STAGE>([&](auto q) { issue_one(q); });
    };

    v16i acc[NH][8];
#pragma unroll
    for (int c = 0; c < NH; ++c)
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[c][s][v] = 0;

    v4i A[8], B[NH][8];
    auto read_A = [&](int slot, int d) {
        const uint4 a = lds[(size_t)slot * C::STAGE_UNITS + (d * KS + g2) * C::LM + wm * 32 + i32];
        A[d] = v4i{ (int)a.x, (int)a.y, (int)a.z, (int)a.w };
    };
    auto read_B = [&](int slot, int d) {
#pragma unroll
        for (int c = 0; c < NH; ++c) {
            const uint4 b = lds[(size_t)slot * C::STAGE_UNITS + C::L_UNITS + (d * KS + g2) * C::TN + wn * C::WN + c * 32 + i32];
            B[c][d] = v4i{ (int)b.x, (int)b.y, (int)b.z, (int)b.w };
        }
    };

    // ---- output pointers, and the addend c_i of the epilogue.  Its loads (indices clamped
    // into the matrix, no per-word branch) are issued all at once at the start of the
    // epilogue.  Issuing them from inside the last steps hides their latency (4 % on
    // 64-deep contractions) but keeps 64 more registers live across the main loop; the
    // kernel stays below 128 vector registers instead, so that a wave of a streaming
    // kernel from another lane fits beside it on the same SIMD (512 registers in all: 136 are
    // left; which of the one-launch kernels keep to that stands at their launch bounds)
    // and fills the issue slots the MFMAs leave free: 7-13 % on the inter-batch pipeline.
    const bool partial = g.ksplit > 1;      // raw partial products go to the workspace; a second kernel finishes
    const u64* addend = (P.addend && !partial) ? P.addend + (size_t)bidx * g.out_bstride : nullptr;
    const u64* addend2 = (P.addend2 && !partial) ? P.addend2 + (size_t)bidx * g.out_bstride : nullptr;
    u64* out = partial ? g.partial + (((size_t)split * g.nparty + party) * g.batch + bidx) * g.out_bstride
                       : P.out + (size_t)bidx * g.out_bstride;
    const int rbase = m0 + wm * 32 + g2 * 4;
    const int shift = partial ? 0 : g.trunc_bits;
    // Word v of a lane's column half lies row_of(v) rows below the lane's first row: a uniform distance.  In tiles that
    // lie inside the output (uniform) a word is addressed as scalar base + one 32-bit lane offset, without vector
    // arithmetic and without bounds checks.  (With an address product, a branch on the addend and three on the
    // truncation per word, and branches between the MFMAs of the last two steps, per-head Q K^T took 358 us and the
    // 1x1 convolution on 56 x 56 x 64 to 256 channels 381 us; so 334 and 361 us.)
    auto row_of = [](int v) { return (v >> 2) * 8 + (v & 3); };
    const bool interior = m0 + C::TM <= g.M && n0 + C::TN <= g.N && g.N <= kLaneOffsetMaxN;
    const unsigned lane_off = ((unsigned)(g2 * 4) * (unsigned)g.N + (unsigned)i32) * 8u;
    const size_t wave_at = (size_t)(m0 + wm * 32) * g.N + (n0 + wn * C::WN);
    u64 addw[NH][16];
    auto load_addend = [&]() {
        if (!addend) {
#pragma unroll
            for (int c = 0; c < NH; ++c)
#pragma unroll
                for (int v = 0; v < 16; ++v) addw[c][v] = 0;
        } else if (interior) {
            const u64* base = addend + wave_at;
#pragma unroll
            for (int c = 0; c < NH; ++c)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    addw[c][v] = *reinterpret_cast<const u64*>(reinterpret_cast<const u8*>(base + (size_t)row_of(v) * g.N + c * 32) + lane_off);
        } else {
#pragma unroll
            for (int c = 0; c < NH; ++c) {
                const int col = n0 + wn * C::WN + c * 32 + i32;
                const int colc = col < g.N ? col : g.N - 1;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = rbase + row_of(v);
                    const int rowc = row < g.M ? row : g.M - 1;
                    addw[c][v] = addend[(size_t)rowc * g.N + colc];
                }
            }
        }
    };

    // ---- main loop.  Ring slot t%NS holds K step t.  At the top of step t the
    // slot of step t+1 must have landed (this wave's loads: all but the most
    // recent PER_STAGE); the barrier makes every wave's part visible and
    // retires slot t%NS, whose operands every wave already holds in registers,
    // so the loads of step t+NS can go there.  Inside the step the MFMAs run
    // block by block over the right-operand digit j (left digits 7-j .. 0);
    // an operand register is refilled from the next slot right after its last
    // use, in an order that gives every refill at least ~14 MFMAs of cover,
    // and one global->LDS load is issued after every fourth MFMA (every third
    // where twelve loads share 36 MFMAs): a wave can
    // issue one instruction per four cycles, so everything that is not an MFMA
    // has to sit in the seven free issue slots an 8-pass MFMA leaves behind.
    issue_all(0);
    if (1 < T) issue_all(1);
    if (NS > 2 && 2 < T) issue_all(2);
    // slot 0 must have landed: everything but the stages issued after it
    static_assert(NS == 2 || NS == 3, "ring depth");
    static_assert((NS - 1) * PER_STAGE <= 63, "vmcnt is a six-bit counter");
    if (NS > 2 && T > 2) __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * PER_STAGE));
    else if (T > 1)      __builtin_amdgcn_s_waitcnt(vmcnt_imm(1 * PER_STAGE));
    else                 __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __syncthreads();
#pragma unroll
    for (int d = 0; d < 8; ++d) { read_A(0, d); read_B(0, d); }

    int slot = 0;                        // t % NS
    // The last NS steps have forms of their own, so that no step branches between its MFMAs: kFull prefetches operands
    // and issues a stage; kNext only prefetches while a later stage is in flight; kNext1 when none is; kLast neither.
    enum { kFull, kNext, kNext1, kLast };
    auto step = [&](auto form_tag) {
        constexpr int form = decltype(form_tag)::value;
        constexpr bool have_next = form != kLast, fill = form == kFull;
        // slot t+1 must have landed; with three slots the loads of step t+2 may still be in flight
        if constexpr (NS > 2 && (form == kFull || form == kNext)) __builtin_amdgcn_s_waitcnt(vmcnt_imm(PER_STAGE));
        else if constexpr (have_next)                             __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        if constexpr (have_next) __syncthreads();
        const int nslot = slot + 1 == NS ? 0 : slot + 1;
        if constexpr (fill) stage_begin(slot);
        // MFMA number n (0..71) <-> block j, left digit i, column half c
        static_for<8>([&](auto jt) {
            constexpr int j = decltype(jt)::value;
            static_for<8 - j>([&](auto it) {
                constexpr int i = 7 - j - decltype(it)::value;
                static_for<NH>([&](auto ct) {
                    constexpr int c = decltype(ct)::value;
                    // MFMAs before this block: sum_{j'<j} NH*(8-j') = NH*j*(17-j)/2
                    constexpr int n = NH * (j * (17 - j) / 2 + (7 - j - i)) + c;
                    acc[c][i + j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[i], B[c][j], acc[c][i + j], 0, 0, 0);
                    if constexpr (fill && n % EVERY == 1 && n / EVERY < PER_STAGE) issue_one(std::integral_constant<int, n / EVERY>{});
                });
                if constexpr (i == 7 - j && have_next) read_A(nslot, i);       // last use of A[7-j] in this step
                // keep this interleaving: without the fence the scheduler packs the
                // MFMAs back to back and everything else into one exposed cluster
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (have_next) read_B(nslot, j);                          // last use of B[.][j]
        });
        slot = nslot;
    };
    int t = 0;
    for (; t + NS < T; ++t) step(std::integral_constant<int, kFull>{});
    if (NS > 2 && t + 2 < T) { step(std::integral_constant<int, kNext>{}); ++t; }
    if (t + 1 < T) step(std::integral_constant<int, kNext1>{});
    step(std::integral_constant<int, kLast>{});

    load_addend();
    // The explicit accumulator reads below are opaque to the compiler's hazard
    // handling: give the last MFMA (8 passes) time to retire before the first read.
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");

    // ---- epilogue: recombine, add, truncate, store.
    static_for<NH>([&](auto ct) {
        constexpr int c = decltype(ct)::value;
        const int col = n0 + wn * C::WN + c * 32 + i32;
        u64 (&add)[16] = addw[c];
        if (addend2) {                  // partial sums of a two-phase call: loaded here, all 16 at once
            const int colc = col < g.N ? col : g.N - 1;
            u64 more[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = rbase + row_of(v);
                const int rowc = row < g.M ? row : g.M - 1;
                more[v] = addend2[(size_t)rowc * g.N + colc];
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) add[v] += more[v];
        }
        // The accumulators are read out explicitly (left to itself the compiler copies all
        // 256 accumulator registers into vector registers at the loop exit, which leaves no
        // room for anything else to stay live across the main loop); the two column halves
        // are fenced from each other, inside a half the 16 words are independent chains.
        u64 z[16];
        static_for<16>([&](auto vt) {
            constexpr int v = decltype(vt)::value;
            int d[8];
            asm volatile("v_accvgpr_read_b32 %0, %8\n\tv_accvgpr_read_b32 %1, %9\n\tv_accvgpr_read_b32 %2, %10\n\tv_accvgpr_read_b32 %3, %11\n\t"
                         "v_accvgpr_read_b32 %4, %12\n\tv_accvgpr_read_b32 %5, %13\n\tv_accvgpr_read_b32 %6, %14\n\tv_accvgpr_read_b32 %7, %15"
                         : "=&v"(d[0]), "=&v"(d[1]), "=&v"(d[2]), "=&v"(d[3]), "=&v"(d[4]), "=&v"(d[5]), "=&v"(d[6]), "=&v"(d[7])
                         : "a"(acc[c][0][v]), "a"(acc[c][1][v]), "a"(acc[c][2][v]), "a"(acc[c][3][v]),
                           "a"(acc[c][4][v]), "a"(acc[c][5][v]), "a"(acc[c][6][v]), "a"(acc[c][7][v]));
            z[v] = recombine(d) + add[v];
        });
        // local truncation (shift and party are uniform over the workgroup): party 0 shifts, party 1 negates around the shift
        if (shift && party == 0) {
#pragma unroll
            for (int v = 0; v < 16; ++v) z[v] >>= shift;
        } else if (shift) {
#pragma unroll
            for (int v = 0; v < 16; ++v) z[v] = (u64)0 - (((u64)0 - z[v]) >> shift);
        }
        if (interior) {
            u64* base = out + wave_at + c * 32;
#pragma unroll
            for (int v = 0; v < 16; ++v)
                *reinterpret_cast<u64*>(reinterpret_cast<u8*>(base + (size_t)row_of(v) * g.N) + lane_off) = z[v];
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = rbase + row_of(v);
                if (row < g.M && col < g.N) out[(size_t)row * g.N + col] = z[v];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    });
}

template <int WGM, int WGN, bool CONV, int NS, int NH>
__global__ __launch_bounds__(64 * WGM * WGN, NH == 1 ? 2 : 1) void k_limb_gemm(GemmDev g) { gemm_tile<WGM, WGN, CONV, NS, NH>(g); }
// the tile of products with at most 32 rows
template <bool CONV>
__global__ __launch_bounds__(256, 2) void k_few_rows_gemm(GemmDev g) { gemm_tile<1, 4, CONV, 3, 1>(g); }

// ---- products with few output tiles --------------------------------------------------
// (Chosen by sliced_waves below, with what it measured.)
// A workgroup has one 32 x 32 output tile, and its KW waves share the contraction: each contracts a slice of the K steps
// with operands loaded straight into registers (the planes' layout is that of the matrix operands; nothing is shared
// between the waves, so nothing goes through LDS), then the 64-bit partial words are added up in LDS and finished there:
// one launch, no partial products in memory.
//
// The MFMAs run in nested angles: level l holds the digit pairs (l, j) and (i, l) with i, j >= l.  With level l the
// operand digits l and 7 - l have had their last use, and are refilled for the next step at once; the next step asks for
// them in the same order, 11 to 21 MFMAs later (twice that with the SIMD's second wave), which covers an L2 access.
template <bool CONV, int KW>
__global__ __launch_bounds__(64 * KW, 2) void k_sliced_gemm(GemmDev g)
{
    __shared__ u64 part[KW][16][64];
    const int lane = threadIdx.x & 63, i32 = lane & 31, g2 = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const unsigned id = blockIdx.x;
    // a party's workgroups one after the other; of two, party 1's, the longer ones, come first
    const int nth = id < g.heavy_blocks ? 0 : id < 2 * g.heavy_blocks ? 1 : 2;
    const int party = g.nparty == 2 ? 1 - nth : nth;
    const unsigned q = (id - (unsigned)nth * g.heavy_blocks) >> 3;
    const GemmParty& P = g.p[party];
    const unsigned tile = (id & 7) * (unsigned)P.per_xcd + q;
    if (q >= (unsigned)P.per_xcd || tile >= (unsigned)P.tiles) return;
    const unsigned t2 = g.by_item(tile), rem = tile - t2 * g.per_item;
    const unsigned split = g.by_batch(t2), item = t2 - split * g.batch;
    // Order of an item's tiles: along the shorter side of the output first, so that an XCD, which has a run of them, reads a
    // stretch of the longer operand once and the shorter one whole.  Along the rows of a wide output every XCD read most of
    // the right operand.  The launch, us, on the larger tiles / here along rows / now: 128 x 512 x 4096 45.0 / 49.4 / 38.8,
    // 256 x 512 x 2048 43.9 / 46.2 / 39.1, 128 x 1024 x 2048 42.2 / 43.3 / 36.2 (folded 37.4 / 35.7 / 28.8).
    const unsigned major = g.by_panel(rem), minor = rem - major * g.panel_tiles;
    const unsigned mt = g.by_columns ? minor : major, nt = g.by_columns ? major : minor;
    const int m0 = (int)mt * 32, n0 = (int)nt * 32;
    const int T0 = P.seg[0].KB / KS, T = T0 + (g.nseg > 1 ? P.seg[1].KB / KS : 0);
    // the workgroup's steps (all, or a slice of a contraction split over workgroups as well), and this wave's
    const int begin = (int)split * g.steps_per_split, end = begin + g.steps_per_split < T ? begin + g.steps_per_split : T;
    const int per = (end - begin + KW - 1) / KW, first = begin + wave * per, last = first + per < end ? first + per : end;
    const bool partial = g.ksplit > 1;
    const u64* const addend = partial ? nullptr : P.addend; const u64* const addend2 = partial ? nullptr : P.addend2;
    u64* const out = partial ? g.partial + ((size_t)split * g.nparty + party) * g.batch * g.out_bstride : P.out;

    // the workgroup's words: thread t has words t and t + 64 KW (of 1024), in the accumulators' order
    constexpr int WPT = 16 / KW;
    size_t at[WPT]; bool ok[WPT]; u64 add[WPT];
#pragma unroll
    for (int k = 0; k < WPT; ++k) {
        const int v = wave + KW * k, row = m0 + (v >> 2) * 8 + g2 * 4 + (v & 3), col = n0 + i32;
        ok[k] = row < g.M && col < g.N;
        at[k] = (size_t)item * g.out_bstride + (size_t)(row < g.M ? row : g.M - 1) * g.N + (col < g.N ? col : g.N - 1);
        add[k] = (addend ? addend[at[k]] : 0) + (addend2 ? addend2[at[k]] : 0);
    }

    v16i acc[8];
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[s][v] = 0;
    if (first < last) {
        const int rowL = m0 + i32 < g.M ? m0 + i32 : g.M - 1, rowR = n0 + i32 < g.N ? n0 + i32 : g.N - 1;
        const unsigned krowL = (unsigned)g.rows_L * 16u, krowR = (unsigned)g.N * 16u;
        // convolution: image position of filter tap (0, 0)
        int hi0 = 0, wi0 = 0, pix0 = 0;
        if (CONV) {
            const int t = (int)g.by_Wo((unsigned)rowL), wo = rowL - t * g.conv.Wo;
            const int b = (int)g.by_Ho((unsigned)t), ho = t - b * g.conv.Ho;
            hi0 = ho * g.conv.stride - g.conv.pad; wi0 = wo * g.conv.stride - g.conv.pad;
            pix0 = (b * g.conv.H + hi0) * g.conv.W + wi0;
        }
        // cursor: the next step to load.  Lanes 0..31 read its first k block, lanes 32..63 its second.
        int seg = first >= T0 ? 1 : 0;
        int left = seg ? T - first : T0 - first;              // steps of the segment from the cursor on
        const u8 *baseL, *baseR; long long dsL, dsR;
        unsigned voffL, voffR;
        int cb = 0, kh = 0, kw = 0;
        auto enter = [&](int kb) {          // k block kb of the segment (uniform) under the cursor
            const GemmSeg& sg = P.seg[seg];
            baseL = sg.L + (size_t)item * sg.L_bstride; baseR = sg.R + (size_t)item * sg.R_bstride;
            dsL = sg.L_dstride; dsR = sg.R_dstride;
            const int k = kb + g2;
            voffR = (unsigned)k * krowR + (unsigned)rowR * 16u;
            if (CONV) { const int tap = k / g.conv.CB; cb = k - tap * g.conv.CB; kh = tap / g.conv.KW; kw = tap - kh * g.conv.KW; }
            else voffL = (unsigned)k * krowL + (unsigned)rowL * 16u;
        };
        auto gather = [&]() {               // convolution: the lane's unit of the left planes; taps outside the image read the zero row
            if (!CONV) return;
            const int hi = hi0 + kh, wi = wi0 + kw;
            const bool in = kh < g.conv.KH && hi >= 0 && hi < g.conv.H && wi >= 0 && wi < g.conv.W;
            const int pix = in ? pix0 + kh * g.conv.W + kw : (int)g.conv.npix;
            voffL = ((unsigned)cb * (unsigned)(g.conv.npix + 1) + (unsigned)pix) * 16u;
        };
        auto next = [&](bool more) {        // on to the next step (more: there is one)
            if (--left == 0) {
                if (seg == 0 && more) { seg = 1; left = T - T0; enter(0); }
            } else {
                voffR += 2 * krowR;
                if (CONV) {
                    cb += 2;
                    while (cb >= g.conv.CB) { cb -= g.conv.CB; if (++kw == g.conv.KW) { kw = 0; ++kh; } }
                } else voffL += 2 * krowL;
            }
            gather();
        };
        enter((first - (seg ? T0 : 0)) * KS);
        gather();
        v4i A[8], B[8];
        auto load_A = [&](int d) { const uint4 x = *reinterpret_cast<const uint4*>(baseL + d * dsL + voffL); A[d] = v4i{ (int)x.x, (int)x.y, (int)x.z, (int)x.w }; };
        auto load_B = [&](int d) { const uint4 x = *reinterpret_cast<const uint4*>(baseR + d * dsR + voffR); B[d] = v4i{ (int)x.x, (int)x.y, (int)x.z, (int)x.w }; };
        static_for<4>([&](auto l) { load_A(l); load_B(l); load_A(7 - l); load_B(7 - l); });
        auto step = [&](auto refill) {
            constexpr bool more = decltype(refill)::value;
            if (more) next(true);
            static_for<4>([&](auto lt) {
                constexpr int l = decltype(lt)::value;
                auto mm = [&](auto it, auto jt) {
                    constexpr int i = decltype(it)::value, j = decltype(jt)::value;
                    acc[i + j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[i], B[j], acc[i + j], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                };
                auto pair = [&](auto kt) {          // (l, k) and (k, l)
                    constexpr int k = decltype(kt)::value;
                    mm(std::integral_constant<int, l>{}, std::integral_constant<int, k>{});
                    if constexpr (k != l) mm(std::integral_constant<int, k>{}, std::integral_constant<int, l>{});
                };
                // partners l .. 7 - l of digit l in the order of their refills: l, 7 - l, l + 1, 6 - l, ...
                static_for<4 - l>([&](auto dt) {
                    constexpr int d = decltype(dt)::value;
                    pair(std::integral_constant<int, l + d>{});
                    pair(std::integral_constant<int, 7 - l - d>{});
                });
                if constexpr (more) { load_A(l); load_B(l); load_A(7 - l); load_B(7 - l); __builtin_amdgcn_sched_barrier(0); }
            });
        };
        for (int t = first; t + 1 < last; ++t) step(std::true_type{});
        step(std::false_type{});
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        int d[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) d[s] = acc[s][v];
        part[wave][v][lane] = recombine(d);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < WPT; ++k) {
        u64 z = add[k];
#pragma unroll
        for (int w = 0; w < KW; ++w) z += part[w][wave + KW * k][lane];
        if (g.trunc_bits && !partial) z = party == 0 ? z >> g.trunc_bits : (u64)0 - (((u64)0 - z) >> g.trunc_bits);
        if (ok[k]) out[at[k]] = z;
    }
}

// Second pass of a split contraction: out = sum over splits of the partial
// products + addends, then truncation.  One thread per output word.
__global__ __launch_bounds__(256) void k_splitk_finish(GemmArgs g)
{
    const size_t per = (size_t)g.batch * g.out_bstride;            // words per party
    const size_t total = per * g.nparty;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        const int party = (int)(i / per);
        const size_t w = i - (size_t)party * per;
        u64 z = 0;
        for (int sp = 0; sp < g.ksplit_p[party]; ++sp) z += g.partial[((size_t)sp * g.nparty + party) * per + w];
        if (g.addend[party]) z += g.addend[party][w];
        if (g.addend2[party]) z += g.addend2[party][w];
        if (g.trunc_bits) z = party == 0 ? (z >> g.trunc_bits) : (u64)0 - (((u64)0 - z) >> g.trunc_bits);
        g.out[party][w] = z;
    }
}

// finishing pass of a contraction split over workgroups
void launch_finish(hipStream_t st, const GemmArgs& g)
{
    const size_t total = (size_t)g.batch * g.out_bstride * g.nparty;
    size_t blocks = (total + 255) / 256; if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_splitk_finish, dim3((unsigned)blocks), dim3(256), 0, st, g);
}

template <int WGM, int WGN, bool CONV, int NS = 3, int NH = 2>
int launch_cfg(mpc_ctx* c, hipStream_t st, const GemmArgs& g)
{
    using C = Cfg<WGM, WGN, NS, NH>;
    // once per device and kernel: allow the large dynamic LDS allocation (lanes may live on several host threads)
    static std::atomic<bool> attr_set[16];
    void (*kern)(GemmDev);
    if constexpr (C::TM == 32) kern = k_few_rows_gemm<CONV>;
    else                       kern = k_limb_gemm<WGM, WGN, CONV, NS, NH>;
    if (c->device < 0 || c->device >= 16) return MPC_EINVAL;
    if (!attr_set[c->device].load(std::memory_order_acquire)) {
        MPC_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS_BYTES));
        attr_set[c->device].store(true, std::memory_order_release);
    }
    GemmArgs ga = g;
    ga.tiles_m = (g.M + C::TM - 1) / C::TM; ga.tiles_n = (g.N + C::TN - 1) / C::TN;
    long long wgs = 0;
    for (int p = 0; p < 2; ++p) {
        const long long tiles = p < g.nparty ? (long long)ga.tiles_m * ga.tiles_n * g.batch * g.ksplit_p[p] : 0;
        if (tiles >= (1ll << 30)) return MPC_EINVAL;
        ga.tiles_party[p] = (int)tiles;
        wgs += (tiles + 7) / 8 * 8;
    }
    // equal slice counts: the interleaved order of the kernel assumes equal blocks
    if (!ga.heavy_first && g.nparty == 2 && ga.tiles_party[0] != ga.tiles_party[1]) return MPC_EINVAL;
    if (wgs >= (1ll << 31)) return MPC_EINVAL;
    GemmDev d{};
    for (int p = 0; p < 2; ++p) {
        GemmParty& q = d.p[p];
        q.seg[0] = g.seg[p][0]; q.seg[1] = g.seg[p][1];
        q.addend = g.addend[p]; q.addend2 = g.addend2[p]; q.out = g.out[p];
        q.tiles = ga.tiles_party[p]; q.per_xcd = (ga.tiles_party[p] + 7) / 8;
    }
    d.M = g.M; d.N = g.N; d.rows_L = g.rows_L; d.nseg = g.nseg; d.nparty = g.nparty; d.trunc_bits = g.trunc_bits;
    d.ksplit = g.ksplit; d.steps_per_split = g.steps_per_split; d.out_bstride = g.out_bstride; d.partial = g.partial;
    d.heavy_blocks = ga.heavy_first ? (unsigned)(d.p[1].per_xcd * 8) : 0;
    constexpr unsigned GN = NH == 1 && C::TN == 64 ? 8 : 4;        // column tiles of a panel
    d.per_item = (unsigned)ga.tiles_m * (unsigned)ga.tiles_n; d.batch = (unsigned)g.batch;
    d.panel_tiles = GN * (unsigned)ga.tiles_m; d.tiles_n = (unsigned)ga.tiles_n;
    d.last_width = d.tiles_n % GN ? d.tiles_n % GN : GN;
    d.by_item = Divider::by(d.per_item); d.by_batch = Divider::by(d.batch); d.by_panel = Divider::by(d.panel_tiles);
    d.by_last_width = Divider::by(d.last_width);
    d.conv = g.conv;
    d.by_Wo = Divider::by(CONV ? (unsigned)g.conv.Wo : 1); d.by_Ho = Divider::by(CONV ? (unsigned)g.conv.Ho : 1);
    dim3 grid((unsigned)wgs, 1, 1);
    const int pi = prof_begin(c, MPC_PROF_GEMM_KERNEL, st);
    hipLaunchKernelGGL(kern, grid, dim3(C::NT), C::LDS_BYTES, st, d);
    if (g.ksplit > 1) launch_finish(st, ga);
    prof_end(c, MPC_PROF_GEMM_KERNEL, pi, st);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

// g.ksplit_p[p] slices of g.steps_per_split steps per party
template <bool CONV, int KW>
int launch_sliced(mpc_ctx* c, hipStream_t st, const GemmArgs& g)
{
    GemmDev d{};
    const int tiles_m = (g.M + 31) / 32, tiles_n = (g.N + 31) / 32;
    const long long tiles = (long long)tiles_m * tiles_n * g.batch;
    unsigned blocks = 0;
    for (int p = 0; p < g.nparty; ++p) {
        GemmParty& q = d.p[p];
        q.seg[0] = g.seg[p][0]; q.seg[1] = g.seg[p][1];
        q.addend = g.addend[p]; q.addend2 = g.addend2[p]; q.out = g.out[p];
        const long long t = tiles * (g.ksplit > 1 ? g.ksplit_p[p] : 1);
        if (t >= (1ll << 27)) return MPC_EINVAL;
        q.tiles = (int)t; q.per_xcd = (int)((t + 7) / 8);
        blocks += (unsigned)q.per_xcd * 8;
    }
    d.M = g.M; d.N = g.N; d.rows_L = g.rows_L; d.nseg = g.nseg; d.nparty = g.nparty; d.trunc_bits = g.trunc_bits;
    d.ksplit = g.ksplit; d.steps_per_split = g.steps_per_split; d.partial = g.partial;
    d.out_bstride = g.out_bstride;
    d.heavy_blocks = (unsigned)(d.p[g.nparty == 2 ? 1 : 0].per_xcd * 8);          // of the party that comes first (three: of each)
    d.per_item = (unsigned)tiles_m * (unsigned)tiles_n; d.batch = (unsigned)g.batch;
    d.by_columns = tiles_n > tiles_m;
    d.panel_tiles = (unsigned)(d.by_columns ? tiles_m : tiles_n);
    d.by_item = Divider::by(d.per_item); d.by_batch = Divider::by(d.batch); d.by_panel = Divider::by(d.panel_tiles);
    d.conv = g.conv;
    d.by_Wo = Divider::by(CONV ? (unsigned)g.conv.Wo : 1); d.by_Ho = Divider::by(CONV ? (unsigned)g.conv.Ho : 1);
    const int pi = prof_begin(c, MPC_PROF_GEMM_KERNEL, st);
    hipLaunchKernelGGL((k_sliced_gemm<CONV, KW>), dim3(blocks), dim3(64 * KW), 0, st, d);
    if (g.ksplit > 1) launch_finish(st, g);
    prof_end(c, MPC_PROF_GEMM_KERNEL, pi, st);
    MPC_HIP(c, hipGetLastError());
    return MPC_OK;
}

}  // namespace

// How many ways to split the contraction so that a small output still fills
// the chip: aim for about 256 workgroups, keep at least 4 K steps per slice.
// 32 k per step; with balanced digits (|d| <= 128) the digit-sum groups that
// matter beyond their low 32 bits hold at most four pairs, so 4 * 2^14 * k < 2^31.
constexpr int kMaxStepsExact = 1023;

// Output tile of a workgroup: 0 = 64 x 128 (2 x 2 waves), 1 = 128 x 64 (4 x 1 waves) when a second 64-column half
// would be empty, 2 = 64 x 64 (2 x 2 waves of 32 x 32 with half the accumulator registers, two-slot ring: two
// workgroups per compute unit, two waves per SIMD) for short contractions, where a workgroup's life is mostly
// pipeline fill and epilogue and a second resident wave hides them.
// 3 = 32 x 128 (1 x 4 waves of 32 x 32) for at most 32 rows, where a 64-row tile multiplies padding: with two rows and
// weights of 25088 x 4096 the matrix pipeline was as busy as the memory (616 us a call, 413 us on this tile: 6.0 TB/s of weight planes; 32 rows 641 and 476 us; level
// where a call is all launches).
// Batched products of few rows that meet tile 2's rule stay on tile 2 where half of tile 3's columns would be padding:
// GEMM launch of 768 products with 4 / 32 rows, tile 2 against 3, K = 64: N = 32 29 / 35 and 41 / 47 us, N = 64 33 / 46 and
// 43 / 56; N = 96 (8 / 32 rows) 60 / 76 and 50 / 68, N = 128 66 / 82 and 61 / 73; K = 256, N = 64 98 / 113 and 104 / 119.  Below 512
// products and on longer contractions tile 3 takes the place of the 128 x 64 tile: 96 products, K = 64 and N = 64, 16 / 18
// and 11 / 13 us; K = 512, 768 products, 275 / 290 and 173 / 186.
// Tile 2 is chosen when the longest contraction of the launch has at most g_small_max_steps K steps (32 terms each)
// and the output has at least g_small_min_tiles tiles of 64 x 64 (mpc_set_gemm_small_tile changes both).
// A launch whose parties contract different lengths (the folded calls: party 0 one segment, party 1 two) also takes
// tile 2 at any contraction length once the output has kAsymMinTiles tiles of 64 x 64: short and long workgroups then
// mix two to a compute unit, and the launch loses less to the imbalance (BERT-base layers 2-9 % faster; at 512 tiles,
// configs[1]'s convolution, the two tilings are even, and the wide tile keeps room for another lane's streaming waves).
static std::atomic<int> g_small_max_steps{ 16 }, g_small_min_tiles{ 512 };
// The setting is the process's: a launch reads it once, and everything chosen for the launch follows from that reading.
struct Tuning { int max_steps, min_tiles; };
static Tuning tuning() { return { g_small_max_steps.load(std::memory_order_relaxed), g_small_min_tiles.load(std::memory_order_relaxed) }; }
constexpr long long kAsymMinTiles = 768;
static int tile_kind(const Tuning& tune, int M, int N, int batch, int longest_steps, bool asymmetric)
{
    const long long tiles64 = (long long)((M + 63) / 64) * ((N + 63) / 64) * batch;
    const bool few_rows = M <= 32;
    if (longest_steps <= tune.max_steps && tiles64 >= tune.min_tiles && !(few_rows && N > 64)) return 2;
    if (few_rows) return 3;
    // (not the batched products one 64-column tile wide, per-head A*V: those are 5 % faster on the 128 x 64 tile)
    if (asymmetric && tune.max_steps > 0 && tiles64 >= kAsymMinTiles && !(batch > 1 && N <= 64)) return 2;
    return (((N - 1) % 128) < 64 && (N <= 64 || M >= 4096)) ? 1 : 0;
}

// Waves of a workgroup that share a 32 x 32 tile's contraction (k_sliced_gemm), or 0 for the tiles above.  Few tiles and a
// contraction of at most 64 steps: a workgroup's life is latency, and the finishing pass of a contraction split over
// workgroups one more launch.  Eight waves as long as every compute unit has one workgroup at most, then four.  Folded
// prepared calls, tiles above / 4 waves / 8 waves, us (13.9 is the host's time of a call):
//   64 x 256 x 128 (16 workgroups)       20.4 / 14.1 / 14.0     256 x 1024 x 512 (256)    32.3 / 28.1 / 27.5
//   64 x 1024 x 128                      24.2 / 22.4 / 20.7     512 x 512 x 384 (384)     29.8 / 22.9 / 25.7
//   64 x 2048 x 128, 128 steps           28.7 / 35.7 / 31.5     512 x 1024 x 512 (512)    43.4 / 37.7 / 42.4
//   256 x 512 x 512 (256)                28.5 / 20.0 / 19.7     1024 x 128 x 512 (1024)   29.5 / 22.0 / 25.3
//   1024 x 1024 x 512                    70.2 / 66.4 / 77.0     1024 x 512 x 768 (1536)   54.6 / 58.6 / 69.2
// Beyond 1024 workgroups the larger tiles' reuse of operands wins, beyond 64 steps the split over more workgroups (512 steps:
// 48 / 108 / 98).  Convolutions: 8 x 14 x 14 x 128, 3x3, 42.2 / 32.7 / 37.0; 4 x 14 x 14 x 64 27.5 / 18.6 / 17.9.
// mpc_set_gemm_small_tile(0, ...) switches this form off as well.
//
// Longer contractions with at most 256 workgroups: by cost, in steps of a 64 x 128 tile.  The contraction is then split over
// workgroups too, over as many as the chip holds at once and the caller's partial products have room for (*slices, of which
// the finishing pass costs 5).  At once: every party's workgroups are dealt to the XCDs in eights, and an XCD with one more
// than its 32 compute units runs two rounds (folded 22 x 21586 x 472 in 165 + 90 workgroups 85 us, in 150 + 75 52).  Tiles
// above: rounds of workgroups x (steps per slice + 14), a step of the 32-row tile counting half; sliced: steps per wave + 4, a
// step counting 1.5, as eight waves ask the L2 for 128 KB in it (2.2 us with the chip full; of a strided convolution, which
// uses half of every line it reads, 2.25).  Of 1702 drawn products and convolutions with such contractions none beyond 32
// rows then takes the slower form by more than 2 %, and 1398 of the 1446 that gain as much take it.  The launch, us,
// tiles above / sliced:
//   2 x 25088 x 10      50.3 / 27.8     60 x 8000 x 400      49.3 / 40.8     64 x 8000 x 2000 (left above)    125 / 155
//   64 x 2048 x 128     29.5 / 19.5     100 x 20000 x 100    90.2 / 64.7     1073 x 12347 x 89 (left above)   188 / 232
//   32 x 4096 x 1000    35.4 / 30.0     300 x 4000 x 200     53.8 / 49.8     316 x 25053 x 158 (left above)   204 / 226
//   30 x 1100 x 4000    37.2 / 28.4     200 x 3001 x 333     49.0 / 43.6     3x3 convolution of 4 x 7 x 7 x 256  35.5 / 30.3
constexpr int kSlicedMaxSteps = 64, kFinishCost = 5;
constexpr long long kSlicedMaxBlocks = 1024, kSlicedWideBlocks = 256;
static int sliced_waves(const Tuning& tune, const GemmArgs& g, int longest, const int steps[3], int* slices)
{
    *slices = 1;
    if (tune.max_steps == 0) return 0;
    const long long tiles = (long long)((g.M + 31) / 32) * ((g.N + 31) / 32) * g.batch, blocks = tiles * g.nparty;
    if (blocks > kSlicedMaxBlocks || tile_kind(tune, g.M, g.N, g.batch, longest, false) == 2) return 0;
    // a lane's offset inside a plane is 32 bits wide
    if ((g.conv.enabled ? (g.conv.npix + 1) * g.conv.CB : (long long)longest * KS * g.rows_L) * 16 >= (1ll << 31)) return 0;
    if ((long long)longest * KS * g.N * 16 >= (1ll << 31)) return 0;
    // Few rows and a handful of steps: the 32 x 128 tiles in one round, where this form has two (two workgroups of four waves to
    // a compute unit).  The launch, us, those tiles / four waves: 57 products of 8 x 8 x 240 9.6 / 12.2, 21 of 1 x 21 x 595
    // 9.5 / 11.9, 102 of 12 x 66 x 111 (6 steps) 13.0 / 14.8; from 8 steps on this form is level or ahead (21 of 28 x 97 x 432
    // 0.88-0.93 of the tiles' time).
    if (g.nparty <= 2 && g.M <= 32 && g.N > 64 && longest <= 6 && blocks > 2 * kSlicedWideBlocks &&
        (long long)((g.N + 127) / 128) * g.batch * g.nparty <= 256) return 0;
    if (longest <= kSlicedMaxSteps) return blocks <= kSlicedWideBlocks ? 8 : 4;
    if (blocks > kSlicedWideBlocks || g.nparty > 2) return 0;
    auto blocks_of = [&](int per, long long t) {
        long long n = 0;
        for (int p = 0; p < g.nparty; ++p) n += (t * ((steps[p] + per - 1) / per) + 7) / 8 * 8;
        return n;
    };
    int s = 1;
    while (s < g.ksplit && (longest + s) / (s + 1) >= 8 && blocks_of((longest + s) / (s + 1), tiles) <= kSlicedWideBlocks) ++s;
    const int per = (longest + s - 1) / s;
    const double cost = (per + 7) / 8 * (g.conv.enabled && g.conv.stride > 1 ? 2.25 : 1.5) + 4 + (s > 1 ? kFinishCost : 0);
    const int kind = tile_kind(tune, g.M, g.N, g.batch, 1 << 30, false), tm = kind == 1 ? 128 : kind == 3 ? 32 : 64, tn = kind == 1 ? 64 : 128;
    const long long large = blocks_of(g.steps_per_split, (long long)((g.M + tm - 1) / tm) * ((g.N + tn - 1) / tn) * g.batch);
    const double cost_large = ((large + 255) / 256) * (g.steps_per_split * (kind == 3 ? 0.5 : 1.0) + 14) + (g.ksplit > 1 ? kFinishCost : 0);
    if (cost >= cost_large || (per + 7) / 8 > kMaxStepsExact) return 0;
    *slices = s;
    return 8;
}

// steps[p]: K steps party p contracts (steps[1] = 0 for a one-party launch).  Returns the number of slices
// of the longer contraction; a party with fewer steps gets ceil(its steps / slice length) slices.
static int ksplit_for(int M, int N, int batch, const int steps[2])
{
    const int nparty = steps[1] > 0 ? 2 : 1;
    const int longest = steps[0] > steps[1] ? steps[0] : steps[1];
    const int kind = tile_kind(tuning(), M, N, batch, longest, nparty == 2 && steps[0] != steps[1]);
    const int tm = kind == 1 ? 128 : kind == 3 ? 32 : 64, tn = kind == 0 || kind == 3 ? 128 : 64;
    const long long tiles_pp = (long long)((M + tm - 1) / tm) * ((N + tn - 1) / tn) * batch;      // per party
    // the int32 digit sums of one workgroup stay exact for at most kMaxStepsExact steps
    const int s_exact = (longest + kMaxStepsExact - 1) / kMaxStepsExact;
    int s = s_exact;
    if (tiles_pp * nparty < 160 && longest >= 8) {
        // One workgroup per compute unit at a time: pick the slice count that minimises
        // (rounds of workgroups over the 256 units) x (steps per slice + fixed cost per
        // workgroup: pipeline fill, epilogue, its share of the finishing pass).
        long long best = -1;
        const int s_max = longest / 4 < 32 ? longest / 4 : 32;
        for (int q = s_exact < 1 ? 1 : s_exact; q <= s_max; ++q) {
            const int per = (longest + q - 1) / q;
            long long wgs = 0;
            for (int p = 0; p < nparty; ++p) wgs += tiles_pp * ((steps[p] + per - 1) / per);
            const long long rounds = (wgs + 255) / 256;
            const long long cost = rounds * (per + 6);
            if (best < 0 || cost < best) { best = cost; s = q; }
        }
    }
    if (s <= 1) return 1;
    const int per = (longest + s - 1) / s;
    return (longest + per - 1) / per;          // no empty slice
}

int gemm_ksplit(int M, int N, int batch, int nparty, int total_steps)
{
    const int steps[2] = { total_steps, nparty > 1 ? total_steps : 0 };
    return ksplit_for(M, N, batch, steps);
}

int gemm_ksplit2(int M, int N, int batch, int steps0, int steps1)
{
    const int steps[2] = { steps0, steps1 };
    return ksplit_for(M, N, batch, steps);
}

extern "C" int mpc_set_gemm_small_tile(int max_steps, int min_tiles)
{
    if (max_steps < 0 || min_tiles < 1) return MPC_EINVAL;
    g_small_max_steps.store(max_steps, std::memory_order_relaxed);
    g_small_min_tiles.store(min_tiles, std::memory_order_relaxed);
    return MPC_OK;
}

// slices of `per` steps for every party, none empty
static void split_over(GemmArgs& g, const int steps[3], int per)
{
    g.steps_per_split = per; g.ksplit = 1;
    for (int p = 0; p < 2; ++p) {
        g.ksplit_p[p] = p < g.nparty ? (steps[p] + per - 1) / per : 0;
        if (g.ksplit_p[p] > g.ksplit) g.ksplit = g.ksplit_p[p];
    }
}

// The checks of a launch and the choice of its kernel; completes g.  MPC_OK: f may be launched.
struct Form { int waves, slices, kind; };          // waves: of k_sliced_gemm, or 0: a tile of `kind`
static int choose_form(GemmArgs& g, Form* f)
{
    if (g.nparty < 1 || g.nparty > 3 || g.nseg < 1 || g.nseg > 2) return MPC_EINVAL;
    int longest = 0, steps[3] = { 0, 0, 0 };
    for (int p = 0; p < g.nparty; ++p)
        for (int s = 0; s < g.nseg; ++s) steps[p] += g.seg[p][s].KB / KS;
    if (g.nparty == 3 && (steps[1] != steps[0] || steps[2] != steps[0])) return MPC_EINVAL;
    longest = steps[0] > steps[1] ? steps[0] : steps[1];
    if (g.ksplit < 1 || !g.partial) g.ksplit = 1;
    const int per = (longest + g.ksplit - 1) / g.ksplit;
    if (per < 1 || per > kMaxStepsExact) return MPC_ERANGE;
    split_over(g, steps, per);
    // the longer contraction first (party 1's by construction of the callers)
    g.heavy_first = g.nparty == 2 && steps[1] > steps[0];
    if (g.nparty == 2 && steps[1] < steps[0]) return MPC_EINVAL;
    if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return MPC_EINVAL;
    for (int p = 0; p < g.nparty; ++p)
        for (int s = 0; s < g.nseg; ++s)
            if (g.seg[p][s].KB < (s == 0 ? 1 : 0) || g.seg[p][s].KB % KS) return MPC_EINVAL;     // a second segment may be empty
    // per-lane byte offsets inside one k block of a plane are 32-bit
    if ((long long)g.rows_L * 16 >= (1ll << 32) || (long long)g.N * 16 >= (1ll << 32)) return MPC_EINVAL;
    // A 1x1 convolution of stride 1 without padding reads pixel m for output row m: its planes are those of a matrix with
    // one row more (the zero row), and the plain kernel contracts them without gather, bounds of taps and divisions.
    // (An odd number of channel blocks is filled up from the zero row, which only the gather does.)  56 x 56 x 64
    // to 256 channels, 32 images: 361 -> 350 us a call with the shorter set-up.
    if (g.conv.enabled && g.conv.KH == 1 && g.conv.KW == 1 && g.conv.stride == 1 && g.conv.pad == 0 && g.conv.CB % KS == 0)
        g.conv = ConvGeom{};
    const Tuning tune = tuning();
    f->waves = sliced_waves(tune, g, longest, steps, &f->slices);
    if (f->waves) split_over(g, steps, (longest + f->slices - 1) / f->slices);
    else if (g.nparty == 3) return MPC_EINVAL;               // the tiles below know two parties
    // 64x128 workgroup tiles, or 128x64 when a second 64-column half would be empty
    f->kind = g.ksplit > 1 ? tile_kind(tune, g.M, g.N, g.batch, 1 << 30, false) : tile_kind(tune, g.M, g.N, g.batch, longest, g.heavy_first != 0);
    return MPC_OK;
}

static int launch_form(mpc_ctx* c, hipStream_t st, const GemmArgs& g, const Form& f)
{
    const int kind = f.kind;
    if (f.waves) {
        if (g.conv.enabled) return f.waves == 8 ? launch_sliced<true, 8>(c, st, g) : launch_sliced<true, 4>(c, st, g);
        return f.waves == 8 ? launch_sliced<false, 8>(c, st, g) : launch_sliced<false, 4>(c, st, g);
    }
    if (g.conv.enabled)
        return kind == 3 ? launch_cfg<1, 4, true, 3, 1>(c, st, g) : kind == 2 ? launch_cfg<2, 2, true, 2, 1>(c, st, g)
             : kind == 1 ? launch_cfg<4, 1, true>(c, st, g) : launch_cfg<2, 2, true>(c, st, g);
    return kind == 3 ? launch_cfg<1, 4, false, 3, 1>(c, st, g) : kind == 2 ? launch_cfg<2, 2, false, 2, 1>(c, st, g)
         : kind == 1 ? launch_cfg<4, 1, false>(c, st, g) : launch_cfg<2, 2, false>(c, st, g);
}

int launch_limb_gemm(mpc_ctx* c, hipStream_t st, const GemmArgs& g_in)
{
    GemmArgs g = g_in;
    Form f{};
    if (g.nparty > 2) return MPC_EINVAL;
    MPC_TRY(choose_form(g, &f));
    return launch_form(c, st, g, f);
}

// whether no party's output shares memory with another party's addend
static bool parties_apart(const GemmArgs& g)
{
    const size_t n = (size_t)g.batch * g.out_bstride;
    for (int i = 0; i < 3; ++i) {
        Spans<1> out; Spans<4> in;
        out.words(g.out[i], n);
        for (int j = 0; j < 3; ++j) if (j != i) { in.words(g.addend[j], n); in.words(g.addend2[j], n); }
        if (!outputs_apart(out, in, false)) return false;
    }
    return true;
}

// Three parties of equal lengths (g.nparty is not read): few tiles in one launch, others, and calls whose party 2 stores over
// what parties 0 and 1 add, in two.
int launch_limb_gemm3(mpc_ctx* c, hipStream_t st, const GemmArgs& g_in)
{
    GemmArgs g = g_in;
    Form f{};
    g.nparty = 3;
    if (choose_form(g, &f) == MPC_OK && parties_apart(g)) return launch_form(c, st, g, f);
    g = g_in;
    g.nparty = 2;
    MPC_TRY(launch_limb_gemm(c, st, g));
    g.nparty = 1;
    for (int s = 0; s < 2; ++s) g.seg[0][s] = g_in.seg[2][s];
    g.addend[0] = g_in.addend[2]; g.addend2[0] = g_in.addend2[2]; g.out[0] = g_in.out[2];
    return launch_limb_gemm(c, st, g);
}
